"""Linears of at most 64 rows whose rows of weights do not start on cache lines: neighbouring column tiles go to one XCD in runs, and every tile
has to be taken exactly once whatever their number is modulo the XCDs."""
import numpy as np
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


@pytest.mark.parametrize("kind", ["dense", "w4", "w8"])
@pytest.mark.parametrize("M", [1, 16, 33])
def test_every_tile_once(B, kind, M):
    """1, 11, 12, 13, 15, 16, 17 and 23 tiles (256 columns, 8-bit up to 16 rows 128), the last one of eight columns, one to sixteen parts of K."""
    width = 128 if kind == "w8" and M <= 16 else 256
    g = torch.Generator(device="cuda").manual_seed(M)
    for K in (128, 1152):
        for tiles in (1, 11, 12, 13, 15, 16, 17, 23):
            N = width * (tiles - 1) + 8
            w = torch.randn((K, N), generator=g, device="cuda") * 0.05
            x = torch.randn((M, K), generator=g, device="cuda").half()
            if kind == "dense":
                rec, k, fn = (w.half(),), B.KIND_FP16, B.linear_fp16
                d = rec[0]
            elif kind == "w4":
                rec, k, fn = B.quantize_layer(w), B.KIND_W4A16, B.linear_w4a16
                d = B.dequantize_w4(*rec, torch.float32)
            else:
                rec, k, fn = B.quantize_layer_w8(w), B.KIND_W8A16, B.linear_w8a16
                d = B.dequantize_w8(*rec, torch.float32)
            y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
            fn(x, *rec, B.new_workspace(B.workspace_bytes(k, M, K, N)), out=y)
            want = x.cpu().double() @ d.cpu().double()
            err = (y.cpu().double() - want).abs().max() / want.abs().max()
            assert err <= TOL, (K, tiles, float(err))
