"""Dense linears of at most 64 rows, in column tiles of 256 and of 128: K shared out over the splits and the waves' halves or quarters in k-steps of 32, with none to
three left after the last round of four (none to 66 of them to a wave), and in runs of 128 rows (none to 17 of them)."""
import ctypes

import numpy as np
import pytest

from paper_2506_02006_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"fp16": 2e-3, "bf16": 1.2e-2}     # one rounding of the result (2^-12 / 2^-9 of values up to a few rms) and fp32 sums, a margin of 3


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2506_02006_amd import binding
    return binding


# column tiles of 256 without the LDS ring, and of 128 wherever they can run
WIDTHS = {256: ("TUNE_TILED", 1), 128: ("TUNE_SMALL", 6)}


def set_width(B, width):
    B.set_tuning(getattr(B, WIDTHS[width][0]), WIDTHS[width][1])


def layout(B, M, K, N):
    """(column width, tiles, splits) of the launch"""
    plan = (ctypes.c_int * 5)()
    assert B.lib().morph_plan_decode(B.KIND_FP16, M, K, N, plan) == 0 and plan[0] == 1
    return 128 if plan[4] == 2 else 256, plan[1], plan[2]


@pytest.fixture(autouse=True)
def planned_splits(B):
    yield
    for key in (B.TUNE_DECODE_SPLIT, B.TUNE_TILED, B.TUNE_SMALL):
        B.set_tuning(key, 0)


@pytest.mark.parametrize("width", list(WIDTHS))
@pytest.mark.parametrize("fmt", ["fp16", "bf16"])
@pytest.mark.parametrize("M", [1, 16, 17, 32, 64])
@pytest.mark.parametrize("K,splits", [(128, (1,)), (384, (1, 2, 3)), (640, (2, 3, 5)), (1024, (1, 4, 8)), (1408, (1, 3, 7, 11)), (4224, (1, 2, 5, 16))])
def test_dense_k_steps_left_over(B, oracle, K, splits, M, fmt, width):
    """Row 1 of x is infinite: what a wave reads beyond its part of a row must not reach another row's sums."""
    N = 264
    dt = torch.float16 if fmt == "fp16" else torch.bfloat16
    g = torch.Generator().manual_seed(K + M)
    x, w = torch.randn((M, K), generator=g).to(dt), (0.05 * torch.randn((K, N), generator=g)).to(dt)
    if M > 1:
        x[1] = float("inf")
    keep = [r for r in range(M) if r != 1]
    want = (x[keep].double() @ w.double()).numpy()
    fn = B.linear_fp16 if fmt == "fp16" else B.linear_bf16
    ws = B.new_workspace(B.workspace_bytes(B.KIND_FP16, M, K, N) + (32 << 20))
    xd, wd = x.cuda(), w.cuda()
    set_width(B, width)
    for S in splits:
        B.set_tuning(B.TUNE_DECODE_SPLIT, S)
        assert layout(B, M, K, N) == (width, -(-N // width), S)
        got = fn(xd, wd, ws)[keep].double().cpu().numpy()
        r = oracle.error_metric(got, want)
        assert r["finite"] and r["err"] <= TOL[fmt], (S, r)


@pytest.mark.parametrize("width", [256, None])
@pytest.mark.parametrize("fmt", ["fp16", "bf16"])
@pytest.mark.parametrize("K,N", [(256, 264), (512, 264), (1024, 4096), (2048, 4096), (4096, 2048), (8192, 2048)])
def test_dense_splits_as_planned(B, oracle, K, N, fmt, width):
    """Results on the planner's own splits (test_abi.py has their numbers, of tiles of 256 columns and of the planner's choice): workgroups of four k-steps, and the splits whose
    starts lie whole megabytes apart."""
    dt = torch.float16 if fmt == "fp16" else torch.bfloat16
    g = torch.Generator().manual_seed(K + N)
    x, w = torch.randn((64, K), generator=g).to(dt), (0.05 * torch.randn((K, N), generator=g)).to(dt)
    want = (x.double() @ w.double()).numpy()
    fn = B.linear_fp16 if fmt == "fp16" else B.linear_bf16
    xd, wd = x.cuda(), w.cuda()
    if width:
        set_width(B, width)
    for M in (1, 16, 32, 64):
        assert layout(B, M, K, N)[0] == (width or (128 if M <= 32 else 256))
        r = oracle.error_metric(fn(xd[:M].contiguous(), wd, B.new_workspace(B.workspace_bytes(B.KIND_FP16, M, K, N))).double().cpu().numpy(), want[:M])
        assert r["finite"] and r["err"] <= TOL[fmt], (M, r)


def test_dense_one_workgroup_needs_no_workspace(B):
    """K of 384 and less stays in one part, which is what calls without a workspace rely on."""
    for K in (128, 256, 384):
        x, w = torch.randn((4, K)).half().cuda(), torch.randn((K, 264)).half().cuda()
        y = torch.empty((4, 264), dtype=torch.float16, device="cuda")
        assert B.lib().morph_linear_fp16(x.data_ptr(), w.data_ptr(), y.data_ptr(), 4, K, 264, None, 0, torch.cuda.current_stream().cuda_stream) == 0
        want = x.float() @ w.float()
        assert (y.float() - want).norm() <= 1e-3 * want.norm()
