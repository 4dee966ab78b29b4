"""Export and import at the packed size from which the stores are nontemporal
(128 MiB of K and V), at odd numbers of KV heads and with a partial last page:
every byte moved, no other slot written."""
import numpy as np
import pytest
import torch

from paper_2607_04206_amd import kv

pytestmark = pytest.mark.gpu


# rows x heads x dim x 4 bytes: exactly 128 MiB, then above it
@pytest.mark.parametrize("hkv,d,rows", [(16, 64, 32768), (16, 64, 32769), (8, 128, 32768), (8, 128, 32769), (7, 64, 80001), (5, 128, 60007)])
def test_copies_around_the_stream_size(hkv, d, rows):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    dev = torch.device("cuda:0")
    print(f"[case] kv stream {hkv} heads, D {d}, {rows} rows", flush=True)
    kv_len = np.array([rows - 1000, 983, 17], np.int32)
    counts = -(-kv_len // 16)
    indptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    pool = int(indptr[-1]) + 9
    rng = np.random.default_rng(rows + d)
    src, dst = (rng.permutation(pool)[:indptr[-1]].astype(np.int32) for _ in range(2))
    gen = torch.Generator(device=dev).manual_seed(rows)
    k, v = (torch.randint(-32768, 32768, (pool, hkv, 16, d), generator=gen, device=dev, dtype=torch.int16).view(torch.bfloat16)
            for _ in range(2))
    plans = [kv.plan(kv_len=kv_len, page_indptr=indptr, page_ids=p, num_kv_heads=hkv, head_dim=d, num_pool_pages=pool, device=dev)
             for p in (src, dst)]
    packed = kv.kv_export(plans[0], k, v)
    back = [torch.full_like(k.view(torch.int16), 0x7FC1).view(torch.bfloat16) for _ in range(2)]
    want = [b.clone() for b in back]
    kv.kv_import(plans[1], *packed, *back)
    pos = np.concatenate([np.arange(n) for n in kv_len])
    entry = np.concatenate([indptr[i] + np.arange(n) // 16 for i, n in enumerate(kv_len)])
    slot = torch.from_numpy(pos % 16).to(dev)
    for p, pool_in, out, w in zip(packed, (k, v), back, want):
        rows_in = pool_in[torch.from_numpy(src[entry].astype(np.int64)).to(dev), :, slot]
        assert torch.equal(p.view(torch.int16), rows_in.contiguous().view(torch.int16))
        w[torch.from_numpy(dst[entry].astype(np.int64)).to(dev), :, slot] = rows_in
        assert torch.equal(out.view(torch.int16), w.view(torch.int16))
