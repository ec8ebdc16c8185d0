"""GPU parity of the row softmax at the edges of its row forms: lengths around every
lanes-per-row and chunk limit, odd head counts, scores at odd element offsets, rows
whose scores are huge, -inf or the type's lowest value, masked rows, and heads split
over waves or not."""
import numpy as np
import pytest
import torch

import oracle
from tests.helpers import canary_buffer, canary_intact, dev, host, scores_close
from workloads import random_storage

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513,
         1023, 1024, 1025]


def _plan(L, H):
    import paper_2110_10221_amd as rag

    plan = rag.Plan(torch.from_numpy(L).cuda(), int(L.sum()), int(L.max()), H)
    rag.ragged_offsets(plan)
    return plan


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("L,H", [(EDGES[:20], 3), (EDGES[20:], 1), ([9, 40, 100, 200, 300, 600], 17), ([8] * 7, 2),
                                 ([1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32], 19),
                                 ([130] * 140, 5)])
@pytest.mark.parametrize("shift", [0, 1])
def test_row_forms(dtype, L, H, shift):
    import paper_2110_10221_amd as rag

    L = np.array(L, np.int32)
    rng = np.random.default_rng(int(L.sum()) + H)
    n = oracle.score_elems(L, H)
    s = random_storage(rng, (n,), dtype, 4.0)
    print(f"softmax {dtype} B={L.size} H={H} shift={shift}", flush=True)
    plan = _plan(L, H)
    s_whole = torch.full((n + 64,), float("nan"), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
    S = s_whole[shift:shift + n]
    S.copy_(dev(s, dtype))
    whole, P = canary_buffer(n + shift, dtype)
    rag.ragged_softmax(plan, S, P[shift:])
    torch.cuda.synchronize()
    assert not plan.data_errors()
    assert canary_intact(whole, n + shift) and (shift == 0 or bool(torch.isnan(P[:shift].float()).all()))
    got = host(P[shift:], dtype)
    assert scores_close(got, oracle.softmax(dtype, L, H, s), L, H, dtype)
    rag.ragged_softmax(plan, S)                                # in place: the same bits
    torch.cuda.synchronize()
    assert np.array_equal(host(S, dtype), got)
    assert bool(torch.isnan(s_whole[shift + n:].float()).all())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_masked_row_forms(dtype):
    # causal: row i has i + 1 scores, so every row form runs at every length
    import paper_2110_10221_amd as rag

    L, H = np.array([600, 5, 65], np.int32), 3
    rng = np.random.default_rng(5)
    n = oracle.score_elems(L, H)
    s = random_storage(rng, (n,), dtype, 3.0)
    plan = _plan(L, H)
    S = dev(s, dtype)
    P = torch.zeros_like(S)
    print(f"masked softmax {dtype}", flush=True)
    rag.ragged_softmax_causal(plan, S, P)
    torch.cuda.synchronize()
    got, vals, o = host(P.float(), "f32"), host(S.float(), "f32").astype(np.float64), 0
    for l in L:
        x = vals[o:o + H * l * l].reshape(l, H, l)
        mask = np.arange(l)[None, None, :] <= np.arange(l)[:, None, None]
        e = np.where(mask, np.exp(x - np.where(mask, x, -np.inf).max(-1, keepdims=True)), 0.0)
        ref = e / e.sum(-1, keepdims=True)
        g = got[o:o + H * l * l].reshape(l, H, l)
        # one rounding to the storage type, plus the fp32 exponential and sums
        tol = (2.0 ** -8 if dtype == "bf16" else 0.0) * ref + 1e-5 * ref.max(-1, keepdims=True)
        assert np.all(np.abs(g - ref) <= tol)
        o += H * l * l


def test_extreme_scores():
    import paper_2110_10221_amd as rag

    L, H = np.array([6, 40, 300], np.int32), 2
    n = oracle.score_elems(L, H)
    rng = np.random.default_rng(2)
    x = rng.standard_normal(n).astype(np.float32)
    off = 0
    for l in L:
        rows = x[off:off + H * l * l].reshape(-1, l)
        rows[0] = -np.inf
        rows[0, l - 1] = 1.0                                   # one finite score, in the row's last place
        rows[1] = np.finfo(np.float32).min                     # all equal to the type's lowest value: uniform
        rows[2] = 3e38
        rows[3, 0] = -np.inf
        off += H * l * l
    S = torch.from_numpy(x).cuda()
    plan = _plan(L, H)
    print("softmax extremes", flush=True)
    rag.ragged_softmax(plan, S)
    torch.cuda.synchronize()
    got, off = S.cpu().numpy(), 0
    for l in L:
        rows = x[off:off + H * l * l].reshape(-1, l)
        ref = torch.softmax(torch.from_numpy(rows.astype(np.float64)), -1).numpy()
        assert np.allclose(got[off:off + H * l * l].reshape(-1, l), ref, rtol=1e-5, atol=1e-7)
        off += H * l * l
