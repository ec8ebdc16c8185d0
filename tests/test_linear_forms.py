"""The tile form a packed linear call takes (host arithmetic, no GPU needed), at sizes where
every form was timed: the rule must not name one measured slower."""
import ctypes
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2110_10221_amd", "libragged.so")
needs_lib = pytest.mark.skipif(not os.path.exists(LIB), reason="libragged.so not built")

CUS = 256
# 0: 128 x 256 tiles, two per CU; 1 .. 4: 32 x 32, 64 x 64, 64 x 128, 128 x 128; 5: 128 x 256,
# one round; 6: 256 x 256 (and 128 x 128 quarters)


def form(T, K, N, act=0, residual=False, plan_batch=0):
    import paper_2110_10221_amd as rag

    f = rag.library()._ZN3rag16linear_form_bf16Elllibll  # rag::linear_form_bf16
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int, ctypes.c_bool, ctypes.c_int64, ctypes.c_int64]
    return f(T, K, N, act, residual, plan_batch, CUS)


@needs_lib
@pytest.mark.parametrize("T,K,N,res,forms", [
    # few tokens: most of a 128-row quarter is empty (us, best of the small tiles / 256 x 256)
    (1, 4224, 14272, 0, (1, 2)),      # 18.7 / 26.5
    (8, 3968, 13760, 0, (1, 2)),      # 17.6 / 25.1
    (32, 4096, 16384, 0, (1, 2)),     # 21.5 / 34.9
    (100, 4096, 12288, 0, (2, 3)),    # 23.3 / 28.7
    (257, 4096, 5120, 0, (2, 3)),     # 21.9 / 29.2
    (897, 4032, 2112, 1, (3,)),       # 22.7 / 26.2
    # enough of them: the 256 x 256 kernel
    (1300, 1536, 2112, 0, (6,)), (5200, 2048, 512, 0, (6,)),          # 18.9 / 17.7
    (4000, 4096, 1024, 0, (6,)), (2000, 2048, 4992, 0, (6,)),         # 54.9 (form 0) / 53.1
    (1926, 6912, 4288, 0, (6,)), (4622, 3968, 2048, 0, (6,)),         # 149.6 / 147.5, 91.7 / 87.9
    (16384, 2048, 1024, 0, (6,)), (35475, 4096, 1024, 0, (6,)),       # 68.8 / 62.7, 298 / 270
    (10076, 2048, 512, 0, (5,)), (35475, 1024, 4096, 0, (0,)),
    # (2580 tokens: the last 256-token row of tiles is a twelfth full)
    (2580, 6144, 1536, 1, (4,)),      # 52.4 / 84.0
    (2580, 1536, 1536, 1, (4,)),      # 16.0 / 24.7
    (2580, 2048, 6144, 0, (0,)),      # 59.1 / 68.8
    (2236, 4096, 1024, 1, (6,)), (4980, 5440, 448, 0, (6,)),    # 30.9 / 28.0, 37.6 / 33.7
    (2700, 2048, 6144, 0, (6,)), (2580, 1536, 4608, 0, (6,)),   # 76 / 66, 39.0 / 38.6
    (2442, 1536, 4608, 0, (0,)),      # 39.5 / 42.0
    (6000, 1536, 1536, 1, (6,)),      # 40.7 / 39.4
])
def test_long_reduction_form(T, K, N, res, forms):
    assert form(T, K, N, 0, bool(res)) in forms


@needs_lib
@pytest.mark.parametrize("T,K,N,act,res,forms", [
    # one round of 128 x 256 tiles, two on some CUs (us, form 0 / best of the small tiles)
    (4000, 768, 3072, 1, 0, (0,)),     # 29.5 / 32.6
    (5174, 1024, 2048, 1, 0, (0,)),    # 33.9 / 37.8
    (2600, 1024, 4096, 1, 0, (0,)),    # 33.7 / 37.3
    (1592, 2816, 5888, 1, 0, (0,)),    # 72.6 / 75.1
    (5200, 768, 2304, 0, 0, (0,)),     # 25.2 / 27.8
    (4000, 1024, 3072, 0, 0, (0,)),    # 30.7 / 34.5
    (4000, 768, 2304, 0, 0, (0,)),     # 23.4 / 25.0
    (16000, 768, 768, 0, 1, (0,)),     # 29.3 / 30.8
    (13000, 768, 768, 0, 1, (3,)),     # 27.6 / 25.5
    (20000, 512, 512, 0, 1, (3,)),     # 22.5 / 20.3
    (13000, 576, 576, 0, 1, (3, 4)),   # 22.6 / 17.5: partial feature tiles
    (2236, 512, 1536, 0, 0, (4,)), (777, 1024, 4096, 1, 0, (4,)), (20000, 1024, 3072, 0, 0, (0,)),
])
def test_short_reduction_form(T, K, N, act, res, forms):
    assert form(T, K, N, act, bool(res)) in forms


@needs_lib
@pytest.mark.parametrize("T,d,batch,forms", [
    # QKV projections: the form without a plan, and with one of `batch` sequences
    (2454, 512, 40, (4, 0)),     # the layer: 64.3 us with form 4, 59.4
    (2580, 512, 128, (4, 0)),    # 67.2, 60.4
    (2442, 512, 16, (4, 4)),     # 16 CUs are free: 59.3, 60.4
    (2236, 512, 32, (4, 4)),     # 40 are
    (2454, 1024, 40, (5, 0)),    # 119.1, 114.5
    (2442, 1024, 16, (5, 5)),    # 113.4, 115.8
    (507, 512, 8, (2, 2)),       # 32.5, 36.6: two workgroups per CU
    (1000, 2048, 40, (5, 5)),    # the projection alone: 28.8, 39.5
    (507, 1536, 8, (6, 6)),      # 72.7, 83.9
])
def test_form_leaves_the_plan_room(T, d, batch, forms):
    assert (form(T, d, 3 * d), form(T, d, 3 * d, plan_batch=batch)) == forms


@needs_lib
@pytest.mark.parametrize("expected,shapes", [
    (1, [(1, 64, 64), (31, 128, 64), (33, 192, 192), (100, 64, 64), (300, 320, 320)]),
    (2, [(1000, 512, 512), (777, 64, 1088), (1501, 256, 320), (2500, 320, 1600)]),
    (3, [(900, 192, 1600), (1700, 448, 832), (2236, 2048, 512)]),
    (4, [(1300, 64, 2112), (3000, 192, 1088), (2236, 512, 1536)]),
    (5, [(4300, 1024, 960), (2000, 1088, 4032), (10241, 1216, 448)]),
    (6, [(1300, 1536, 2112), (8300, 1600, 2112), (16384, 2048, 1024), (16129, 1536, 960)]),
])
def test_parity_shapes_reach_their_form(expected, shapes):
    # the shapes by which the GPU tests cover each form
    for s in shapes:
        assert form(*s, 0, True) == expected, s
        if expected < 6:
            assert form(*s, 1) == expected, s


@needs_lib
@pytest.mark.parametrize("T,N,expected", [
    (500, 4096, 64), (3000, 1024, 64),   # quarters of 128 x 128 tiles: 38.5 (38.6), 56.7 (54.1) us
    (777, 2304, 64), (2300, 520, 65),
    (4300, 1030, 129),            # 306 tiles of 128 x 128, the last 50 as quarters
    (5000, 1024, 129), (4096, 2048, 128), (10076, 512, 129), (1, 4096, 65),
])
def test_f32_form(T, N, expected):
    import paper_2110_10221_amd as rag

    f = rag.library()._ZN3rag15linear_form_f32Ellbl  # rag::linear_form_f32
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int64, ctypes.c_int64, ctypes.c_bool, ctypes.c_int64]
    assert f(T, N, True, CUS) == expected
    assert f(T, N, False, CUS) in (64, 65)
