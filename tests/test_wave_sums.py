"""The two waves that share a decode tile's rows (one or two query heads a
tile) each hold a part of every 64 keys; their sums meet as
fma(s1, O1, s0 * O0). Which product is fused shows in the last bit of the fp32
split partials, which these inputs make computable: equal keys within a wave
(every weight is 1) and small integers as values."""
import numpy as np
import pytest
import torch

from tests.test_plan import parse

SPLITS, D, H, N = 17, 64, 2, 32  # 17 splits: more than a tile merges, so the partials stay as [split][row][head][D]


def rounded(x):
    return np.float64(np.float32(x))


@pytest.mark.gpu
@pytest.mark.parametrize("larger", [0, 1])
def test_partials_are_fused_in_wave_order(larger):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2607_04206_amd import attn
    dev = torch.device("cuda:0")
    L, scale, low = 64 * SPLITS, np.float32(0.125), -0.75
    rng = np.random.default_rng(larger)
    wave = np.arange(L) % 64 // 32
    k = np.zeros((L, H, D), np.float32)
    k[:, :, 0] = np.where(wave == larger, 0.0, low)[:, None]  # the score of a key, with q = e0
    v = rng.integers(-100, 101, (L, H, D)).astype(np.float32)
    q = np.zeros((N, H, D), np.float32)
    q[:, :, 0] = 1.0
    bf = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(torch.bfloat16).to(dev)  # noqa: E731
    paged = lambda x: bf(x.reshape(L // 16, 16, H, D).transpose(0, 2, 1, 3))  # noqa: E731
    ids = np.arange(L // 16, dtype=np.int32)
    p = attn.plan(q_indptr=[0, N], q_offset=[L - N], kv_len=[L], page_indptr=[0, len(ids)], page_ids=ids, num_q_heads=H,
                  num_kv_heads=H, head_dim=D, num_pool_pages=len(ids), sm_scale=float(scale), force_kv_splits=SPLITS, device=dev)
    h, items, *_ = parse(p)
    assert items["num_splits"][0] == SPLITS and h["reserved"] == 0 and h["decode_kw"] == 2
    ws = torch.empty(p.workspace_bytes, dtype=torch.uint8, device=dev)
    attn.forward(p, bf(q), bf(k[L - N:]), bf(v[L - N:]), paged(k), paged(v), torch.from_numpy(ids).to(dev), workspace=ws)
    at = int(items["ws_o"][0])
    got = ws.cpu().numpy().view(np.float32)[at:at + SPLITS * N * H * D].reshape(SPLITS, N, H, D)
    assert (got == got[:, :1]).all()  # the rows are alike
    got = got[:, 0].astype(np.float64)
    sums = v.reshape(SPLITS, 2, 32, H, D).sum(2, dtype=np.float64)
    # the factor of the wave with the smaller scores: exp2 to 1 ulp of the hardware's
    m = rounded(np.float64(low) * np.float64(np.float32(scale * np.float32(1.44269504088896340736))))
    near = np.float32(2.0 ** m)
    for step in range(-2, 3):
        s = np.ones(2)
        s[1 - larger] = np.float64((near.view(np.int32) + step).astype(np.int32).view(np.float32))
        total = 2 * rounded(16 * s[0] + 16 * s[1])
        o = rounded(s[1] * sums[:, 1] + rounded(s[0] * sums[:, 0]))  # the products of 24 and 12 bits are exact in fp64
        if (got == rounded(o * rounded(1.0 / total))).all():
            return
    raise AssertionError("no factor gives these partials")
