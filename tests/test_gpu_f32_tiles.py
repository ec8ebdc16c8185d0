"""GPU parity of the fp32 matrix kernels at the edges of their tiles and dispatch:
sizes that are multiples of nothing, rows that start at any element (4-byte copies)
next to 16-byte aligned ones, last rounds that run as quarter tiles, both tile
sizes of vgemm and trmm, and leading dimensions past the 32-bit offsets."""
import numpy as np
import pytest
import torch

import oracle
from tests.helpers import canary_buffer, canary_intact, close, dev, host
from workloads import make_trmm_operands, make_vgemm_operands, random_storage

pytestmark = pytest.mark.gpu


def _form(T, N):
    """The tiles of an fp32 linear call (see rag::linear_form_f32): 128 or 64, plus one where
    the last round runs as quarters."""
    import ctypes

    import paper_2110_10221_amd as rag

    f = rag.library()._ZN3rag15linear_form_f32Ellbl
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int64, ctypes.c_int64, ctypes.c_bool, ctypes.c_int64]
    return f(T, N, True, torch.cuda.get_device_properties(0).multi_processor_count)


@pytest.mark.parametrize("T,K,N,pad,shift,form", [
    (1, 1, 1, 0, 0, 65), (1, 1, 1, 2, 1, 65),                         # one element
    (33, 31, 65, 0, 0, 65), (64, 4, 64, 4, 0, 65), (65, 36, 130, 3, 1, 65),  # k below, at and past one 32-k step
    (63, 32, 31, 0, 0, 65), (64, 64, 64, 1, 1, 65), (97, 100, 33, 4, 4, 65),  # 16-byte aligned rows (pad, shift % 4 == 0) and not
    (2300, 100, 520, 0, 0, 65), (2300, 101, 519, 0, 0, 65),           # 324 tiles of 64 x 64, 68 as quarters
    (8200, 68, 520, 0, 0, 65), (4100, 33, 1030, 1, 1, 65),            # four rounds of them, then quarters
    (4300, 68, 1030, 0, 0, 129), (4300, 33, 1030, 1, 1, 129),         # 306 tiles of 128 x 128, 50 as quarters of 64 x 64
    (16300, 36, 250, 4, 0, 128), (16300, 35, 250, 0, 0, 128),         # one round of 128 x 128 tiles
    (3000, 36, 1000, 0, 0, 64),                                       # whole 64 x 64 tiles alone
])
def test_linear_any_shape(T, K, N, pad, shift, form):
    assert _form(T, N) == form
    import paper_2110_10221_amd as rag

    rng = np.random.default_rng(T + 7 * K + N)
    x, w = random_storage(rng, (T, K), "f32"), random_storage(rng, (N, K), "f32", 0.1)
    b, r = random_storage(rng, (N,), "f32"), random_storage(rng, (T, N), "f32")
    print(f"f32 linear T={T} K={K} N={N} pad={pad} shift={shift}", flush=True)
    ld = K + pad + shift
    xw = torch.full((T * ld + 8,), float("nan"), device="cuda")   # NaN between and past the rows
    xv = xw[shift:shift + T * ld].view(T, ld)[:, :K]
    xv.copy_(dev(x, "f32"))
    whole, y = canary_buffer(T * N, "f32")
    y = y.view(T, N)
    rag.packed_linear(xv, dev(w, "f32"), y, dev(b, "f32"), dev(r, "f32"), oracle.ACT_GELU_ERF)
    torch.cuda.synchronize()
    assert canary_intact(whole, T * N)
    rows = np.unique(np.r_[0:min(T, 24), T // 2, max(0, T - 24):T])
    assert close(host(y, "f32")[rows], oracle.linear("f32", x[rows], w, b, r[rows], oracle.ACT_GELU_ERF), "f32", N)


@pytest.mark.parametrize("T,K,N,ld", [
    (70, 40, 9, 12_000_000),     # past 2^31 bytes within 64 rows: the plain-FMA kernel
    (140, 64, 9, 8_000_000),     # within 128 rows only: 64 x 64 tiles
    (300, 36, 2600, 5_000_001),  # the same on rows at any element
    (3, 40, 9, 1 << 26),         # few rows: rows past the last whose offsets wrap
])
def test_linear_rows_past_32_bit_offsets(T, K, N, ld):
    import paper_2110_10221_amd as rag

    rng = np.random.default_rng(3)
    x, w = random_storage(rng, (T, K), "f32"), random_storage(rng, (N, K), "f32")
    print(f"f32 linear, ldx {ld}", flush=True)
    xv = torch.empty(T, ld, device="cuda")[:, :K]
    xv.copy_(dev(x, "f32"))
    y = torch.empty(T, N, device="cuda")
    rag.packed_linear(xv, dev(w, "f32"), y)
    L, B = make_trmm_operands(T, N, rng, "f32")
    lv = torch.empty(T, ld, device="cuda")[:, :T]
    lv.copy_(dev(L, "f32"))
    c = torch.empty(T, N, device="cuda")
    rag.ragged_trmm(lv, dev(B, "f32"), c)
    torch.cuda.synchronize()
    assert close(host(y, "f32"), oracle.linear("f32", x, w, None, None, oracle.ACT_NONE), "f32", N)
    assert close(host(c, "f32"), oracle.trmm("f32", T, N, L, B), "f32", N)


def _strided(T, N, ld):
    """[T, N] with leading dimension ld in a buffer of NaN, and the buffer."""
    buf = torch.full((T, ld), float("nan"), device="cuda")
    return buf, buf[:, :N]


# Tile rows past the last one whose 32-bit store offset, row * ld * 4 mod 2^32, falls on a
# valid row again (strides of 2^25 .. 2^27) or between the valid rows (the others).
@pytest.mark.parametrize("T,K,N,ld", [(1, 64, 4096, 1 << 26), (1, 33, 4096, 1 << 27), (16, 32, 16384, 1 << 25),
                                      (8, 32, 64, 60_000_000), (8, 36, 16384, 20_000_000), (70, 31, 9, 1 << 25)])
def test_linear_output_stride_past_32_bit_offsets(T, K, N, ld):
    import paper_2110_10221_amd as rag

    rng = np.random.default_rng(T + K)
    x, w = random_storage(rng, (T, K), "f32"), random_storage(rng, (N, K), "f32")
    b, r = random_storage(rng, (N,), "f32"), random_storage(rng, (T, N), "f32")
    print(f"f32 linear T={T} N={N}, ldy {ld}", flush=True)
    buf, y = _strided(T, N, ld)
    y.copy_(dev(r, "f32"))
    rag.packed_linear(dev(x, "f32"), dev(w, "f32"), y, dev(b, "f32"), y, oracle.ACT_GELU_ERF)
    torch.cuda.synchronize()
    assert close(host(y, "f32"), oracle.linear("f32", x, w, b, r, oracle.ACT_GELU_ERF), "f32", N)
    assert sum(int((~torch.isnan(row)).sum()) for row in buf) == T * N


@pytest.mark.parametrize("n,m,ld", [(1, 64, 1 << 26), (4, 68, 1 << 26), (40, 68, 1 << 25), (8, 33, 60_000_000)])
def test_trmm_output_stride_past_32_bit_offsets(n, m, ld):
    import paper_2110_10221_amd as rag

    rng = np.random.default_rng(n + m)
    L, B = make_trmm_operands(n, m, rng, "f32")
    print(f"trmm f32 n={n} m={m}, ldc {ld}", flush=True)
    buf, c = _strided(n, m, ld)
    rag.ragged_trmm(dev(L, "f32").view(n, n), dev(B, "f32").view(n, m), c)
    torch.cuda.synchronize()
    assert close(host(c, "f32"), oracle.trmm("f32", n, m, L, B), "f32", m)
    assert sum(int((~torch.isnan(row)).sum()) for row in buf) == n * m


@pytest.mark.parametrize("dims,sampled", [
    ([[64, 64, 64], [65, 63, 33], [3, 3, 1], [128, 256, 32], [130, 260, 36], [31, 1, 500]], False),
    ([[8320, 2048, 5], [130, 300, 64]], True),             # over 16 tiles per problem: 128 x 128 parts
    ([[8320, 2048, 8], [129, 257, 33]], True),
])
def test_vgemm_mixed_alignments(dims, sampled):
    import paper_2110_10221_amd as rag

    dims = np.array(dims, np.int32)
    rng = np.random.default_rng(int(dims.sum()))
    a, b = make_vgemm_operands(dims, rng, "f32")
    print(f"vgemm f32 dims={dims.tolist()}", flush=True)
    off = oracle.vgemm_offsets(dims)
    plan = rag.VgemmPlan(torch.from_numpy(dims).cuda(), host_dims=dims)
    rag.vgemm_offsets(plan)
    n_c = int(off.c_off[-1])
    whole, c = canary_buffer(n_c, "f32")
    rag.ragged_vgemm(plan, dev(a, "f32"), dev(b, "f32"), c)
    torch.cuda.synchronize()
    assert not plan.data_errors() and canary_intact(whole, n_c)
    got = host(c, "f32")
    for p, (m, n, k) in enumerate(dims.tolist()):
        rows = np.unique(np.r_[0, m - 1, rng.integers(0, m, 12)]) if sampled else np.arange(m)
        A = a[off.a_off[p]:off.a_off[p + 1]].reshape(m, k)[rows]
        ref = oracle.vgemm("f32", [[len(rows), n, k]], A.reshape(-1), b[off.b_off[p]:off.b_off[p + 1]])
        g = got[off.c_off[p]:off.c_off[p + 1]].reshape(m, n)[rows]
        assert close(g, ref.reshape(len(rows), n), "f32", n), (m, n, k)


@pytest.mark.parametrize("n,m,pad", [(32, 64, 0), (33, 64, 3), (64, 128, 0), (96, 68, 4), (130, 70, 1), (260, 132, 0),
                                     (4100, 4000, 0), (4097, 3969, 1)])  # the last two: 128 x 128 tiles
def test_trmm_tiles(n, m, pad):
    import paper_2110_10221_amd as rag

    rng = np.random.default_rng(n + m)
    L, B = make_trmm_operands(n, m, rng, "f32")            # NaN above the diagonal
    print(f"trmm f32 n={n} m={m} pad={pad}", flush=True)
    lw = torch.full((n, n + pad), float("nan"), device="cuda")
    lw[:, :n] = dev(L, "f32").view(n, n)
    bw = torch.full((n, m + pad), float("nan"), device="cuda")
    bw[:, :m] = dev(B, "f32").view(n, m)
    whole, c = canary_buffer(n * m, "f32")
    c = c.view(n, m)
    rag.ragged_trmm(lw[:, :n], bw[:, :m], c)
    torch.cuda.synchronize()
    assert canary_intact(whole, n * m)
    rows = np.unique(np.r_[0:min(n, 40), n // 2, n - 2:n]) if n > 1000 else np.arange(n)
    assert close(host(c, "f32")[rows], oracle.trmm_rows("f32", n, m, L, B, rows), "f32", m)


@pytest.mark.parametrize("n,m,r", [(4100, 4000, 3070), (200, 68, 100)])  # 128 x 128 tiles and 64 x 64 ones
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_trmm_row_of_infinities(n, m, r, bad):
    # a non-finite row r of B reaches the rows of C from r on, and at most those of the
    # 64-row block it lies in
    import paper_2110_10221_amd as rag

    rng = np.random.default_rng(r)
    L, B = make_trmm_operands(n, m, rng, "f32")
    print(f"trmm f32 n={n} m={m}, row {r} of B {bad}", flush=True)
    Bd = dev(B, "f32").view(n, m)
    Bd[r] = bad
    c = torch.empty(n, m, device="cuda")
    rag.ragged_trmm(dev(L, "f32").view(n, n), Bd, c)
    torch.cuda.synchronize()
    clean = r // 64 * 64
    rows = np.arange(max(0, clean - 70), clean)
    assert bool(torch.isfinite(c[:clean]).all()) and not bool(torch.isfinite(c[r:]).any())
    assert close(host(c, "f32")[rows], oracle.trmm_rows("f32", n, m, L, B, rows), "f32", m)
