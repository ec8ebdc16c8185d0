"""GPU parity of the bf16 linear operator's small-launch tiles (32 x 32, 64 x 64,
64 x 128, 128 x 128 and 128 x 256 in one round, chosen by the launch's size) at the edges of each: ragged
tokens, partial feature tiles, reductions of one 64-k block and of a number the
stages do not divide, padded rows, in-place residuals; and the layer's plan built
by such a launch."""
import numpy as np
import pytest
import torch

import oracle
from tests.helpers import canary_buffer, canary_intact, close, dev, host
from workloads import random_storage

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,K,N", [
    (1, 64, 64), (31, 128, 64), (33, 192, 192), (100, 64, 64), (300, 320, 320),   # 32 x 32
    (1000, 512, 512), (777, 64, 1088), (1501, 256, 320), (2500, 320, 1600),       # 64 x 64
    (900, 192, 1600), (1700, 448, 832), (2236, 2048, 512),                         # 64 x 128
    (1300, 64, 2112), (3000, 192, 1088), (2236, 512, 1536),                        # 128 x 128
    (4300, 1024, 960), (2000, 1088, 4032), (10241, 1216, 448),                     # 128 x 256, one round
])
@pytest.mark.parametrize("act,res", [(oracle.ACT_NONE, True), (oracle.ACT_GELU_ERF, False)])
def test_small_tiles(T, K, N, act, res):
    import paper_2110_10221_amd as rag

    rng = np.random.default_rng(T + K + N)
    x, w = random_storage(rng, (T, K), "bf16"), random_storage(rng, (N, K), "bf16", 0.05)
    b = random_storage(rng, (N,), "bf16", 0.5)
    r = random_storage(rng, (T, N), "bf16") if res else None
    print(f"small linear T={T} K={K} N={N} act={act} res={res}", flush=True)
    xw = torch.full((T, K + 8), float("nan"), dtype=torch.bfloat16, device="cuda")  # NaN between the rows
    xw[:, :K] = dev(x, "bf16")
    whole, y = canary_buffer(T * N, "bf16")
    y = y.view(T, N)
    if res:  # in place
        y.copy_(dev(r, "bf16"))
    rag.packed_linear(xw[:, :K], dev(w, "bf16"), y, dev(b, "bf16") if not res else None, y if res else None, act)
    torch.cuda.synchronize()
    assert canary_intact(whole, T * N)
    rows = np.unique(np.r_[0:min(T, 40), T // 2, max(0, T - 40):T])
    ref = oracle.linear("bf16", x[rows], w, b if not res else None, r[rows] if res else None, act)
    assert close(host(y, "bf16")[rows], ref, "bf16")


@pytest.mark.parametrize("lengths,heads", [([5, 70, 33], 2), ([64] * 40 + [3] * 100, 4), ([17] * 256, 8),
                                           ([200, 1, 300] * 5, 8), ([64] * 23 + [30], 16), ([40] * 13, 24),
                                           ([100] * 8, 6), ([50] * 10, 12)])
def test_layer_builds_its_plan_in_a_small_launch(lengths, heads):
    # the plan's workgroups behind each tile form: bit-identical to a plan built ahead
    import paper_2110_10221_amd as rag

    L = np.array(lengths, np.int32)
    T, d, dff = int(L.sum()), 64 * heads, 128 * heads
    rng = np.random.default_rng(T)
    shapes = {"w_qkv": (3 * d, d), "b_qkv": (3 * d,), "w_o": (d, d), "b_o": (d,), "ln1_g": (d,), "ln1_b": (d,),
              "w_ff1": (dff, d), "b_ff1": (dff,), "w_ff2": (d, dff), "b_ff2": (d,), "ln2_g": (d,), "ln2_b": (d,)}
    w = {n: dev(random_storage(rng, s, "bf16", 0.05), "bf16") for n, s in shapes.items()}
    x = dev(random_storage(rng, (T, d), "bf16"), "bf16")
    out, plans = [], []
    for flags in (0, rag.RAG_LAYER_BUILD_PLAN):
        plan = rag.Plan(torch.from_numpy(L).cuda(), T, int(L.max()), heads)
        if not flags:
            rag.ragged_offsets(plan)
        ws = torch.empty(rag.encoder_layer_workspace(T, int(L.max()), d, heads, dff), dtype=torch.uint8, device="cuda")
        y = torch.empty_like(x)
        rag.encoder_layer(plan, x, y, w, dff, ws, flags=flags)
        torch.cuda.synchronize()
        assert not plan.data_errors()
        out.append(y)
        plans.append(plan)
    assert torch.equal(out[0].view(torch.int16), out[1].view(torch.int16))
    n_av, n_q = int(plans[0].status[2]), int(plans[0].status[1])
    for name, n in (("tok_off", None), ("att_off", None), ("order", None), ("tok_seq", T), ("av_items", 3 * n_av),
                    ("qkt_items", 4 * n_q), ("status", None)):
        assert torch.equal(getattr(plans[0], name)[:n], getattr(plans[1], name)[:n]), name


@pytest.mark.parametrize("T,K,N,ldy_pad", [
    (1300, 1536, 2112, 0),    # 54 tiles of 256 x 256, all as quarters, ragged both ways
    (8300, 1600, 2112, 8),    # 256 whole tiles, then the quarters of 41; 25 steps of 64 k
    (16384, 2048, 1024, 0),   # exactly one whole round
    (16129, 1536, 960, 0),    # one round, its last tiles partial
])
@pytest.mark.parametrize("bias,res", [(True, True), (False, False)])
def test_long_reductions(T, K, N, ldy_pad, bias, res):
    import paper_2110_10221_amd as rag

    rng = np.random.default_rng(T + K + N)
    print(f"long-reduction linear T={T} K={K} N={N} bias={bias} res={res}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T)
    xw = torch.full((T, K + 8), float("nan"), dtype=torch.bfloat16, device="cuda")  # NaN between the rows
    xw[:, :K] = torch.randn(T, K, device="cuda", generator=gen).to(torch.bfloat16)
    w = random_storage(rng, (N, K), "bf16", 0.05)
    b = random_storage(rng, (N,), "bf16", 0.5) if bias else None
    ld = N + ldy_pad
    whole, yv = canary_buffer(T * ld, "bf16")
    y = yv.view(T, ld)[:, :N]
    rows = np.unique(np.r_[0:20, 120:136, 250:260, T // 2, T - 270:T - 250, T - 20:T])
    r = None
    if res:  # in place
        y.copy_(torch.randn(T, N, device="cuda", generator=gen).to(torch.bfloat16))
        r = host(y[rows], "bf16")
    rag.packed_linear(xw[:, :K], dev(w, "bf16"), y, dev(b, "bf16") if bias else None, y if res else None)
    torch.cuda.synchronize()
    assert canary_intact(whole, T * ld)
    if ldy_pad:
        assert bool(torch.isnan(yv.view(T, ld)[:, N:].float()).all())
    assert bool(torch.isfinite(y.float()).all())
    ref = oracle.linear("bf16", host(xw[rows, :K], "bf16"), w, b, r, oracle.ACT_NONE)
    assert close(host(y[rows], "bf16"), ref, "bf16")
