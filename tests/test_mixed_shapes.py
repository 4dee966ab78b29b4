"""Plans whose tile shapes no kernel has are refused before anything is
launched, also where prefill-shaped tiles and block decodes would share a
launch. Runs without a GPU: a refused call touches no device pointer."""
import ctypes

import numpy as np
import pytest

import workloads
from paper_2607_04206_amd import _lib
from paper_2607_04206_amd._lib import lib
from tests.test_plan import HEADER, plan_of


@pytest.mark.parametrize("d,field,value", [(128, "prefill_rows", 64), (64, "prefill_rows", 256), (128, "prefill_rows", 512),
                                           (64, "prefill_rows", 0)])
def test_unknown_tile_shape_is_refused(d, field, value):
    wl = workloads.make_workload("shapes", 3, hq=8, hkv=8, d=d, decodes=[(64, 300)], prefills=[200, 1100])
    p = plan_of(wl)
    blob = np.array(p.host, copy=True)
    h = np.frombuffer(blob.data, HEADER, count=1)
    assert h["n_decode_tiles"][0] > 0 and h["n_prefill_tiles"][0] > 0 and h["decode_qw"][0] == 1
    at = HEADER.fields[field][1]
    blob[at:at + 4] = np.frombuffer(np.int32(value).tobytes(), np.uint8)
    buf = ctypes.create_string_buffer(blob.tobytes(), blob.nbytes + 64)
    base = ctypes.addressof(buf)
    ptr = ctypes.c_void_p((1 << 20) + 16)  # aligned, never dereferenced
    status = lib.sangam_attn_forward(base, ptr, ptr, ptr, ptr, ptr, ptr, wl.num_pool_pages, ptr, len(wl.page_ids), ptr, None,
                                     ptr, 1 << 30, None)
    assert _lib.STATUS_NAMES[status] == "SANGAM_ERR_UNSUPPORTED"
