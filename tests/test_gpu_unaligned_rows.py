"""Linears of at most 64 rows whose rows of weights do not start on cache lines: neighbouring column tiles go to one XCD in runs, and every tile
has to be taken exactly once whatever their number is modulo the XCDs."""
import ctypes

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 5e-3       # the largest error over the largest result: fp16 rounding of y 4.9e-4 and fp32 sums, a margin of 10


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2506_02006_amd import binding
    return binding


@pytest.fixture(autouse=True)
def planned_tiles(B):
    yield
    for key in (B.TUNE_TILED, B.TUNE_SMALL):
        B.set_tuning(key, 0)


@pytest.mark.parametrize("kind", ["dense", "dense128", "w4", "w8"])
@pytest.mark.parametrize("M", [1, 16, 33])
def test_every_tile_once(B, kind, M):
    """1, 11, 12, 13, 15, 16, 17 and 23 tiles (256 columns, 8-bit up to 16 rows and dense128 128), the last one of eight columns, one to sixteen parts of K."""
    width = 128 if (kind == "w8" and M <= 16) or kind == "dense128" else 256
    if kind.startswith("dense"):                             # tiles of 256 columns without the LDS ring, and of 128 wherever they can run
        B.set_tuning(*((B.TUNE_SMALL, 6) if width == 128 else (B.TUNE_TILED, 1)))
    plan = (ctypes.c_int * 5)()
    g = torch.Generator(device="cuda").manual_seed(M)
    for K in (128, 1152):
        for tiles in (1, 11, 12, 13, 15, 16, 17, 23):
            N = width * (tiles - 1) + 8
            w = torch.randn((K, N), generator=g, device="cuda") * 0.05
            x = torch.randn((M, K), generator=g, device="cuda").half()
            if kind.startswith("dense"):
                rec, k, fn = (w.half(),), B.KIND_FP16, B.linear_fp16
                d = rec[0]
            elif kind == "w4":
                rec, k, fn = B.quantize_layer(w), B.KIND_W4A16, B.linear_w4a16
                d = B.dequantize_w4(*rec, torch.float32)
            else:
                rec, k, fn = B.quantize_layer_w8(w), B.KIND_W8A16, B.linear_w8a16
                d = B.dequantize_w8(*rec, torch.float32)
            if kind != "w8" or M <= 16:
                assert B.lib().morph_plan_decode(k, M, K, N, plan) == 0 and list(plan[:2]) == [1, tiles], (K, tiles, list(plan))
            y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
            fn(x, *rec, B.new_workspace(B.workspace_bytes(k, M, K, N)), out=y)
            want = x.cpu().double() @ d.cpu().double()
            err = (y.cpu().double() - want).abs().max() / want.abs().max()
            assert err <= TOL, (K, tiles, float(err))
