"""Dense linears of up to 64 rows in column tiles of 128, all rows in one workgroup.

Bound, per element, against an fp64 product: fp32 sums of K products of at most K + 64 additions each off by 2^-24 of their magnitude, and y rounded to its
16 bits by u |y| (and half the smallest subnormal, 2^-25).  So |y - ref| <= (K + 64) 2^-24 sum|x||w| + u |ref| + 2^-25."""
import ctypes

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2506_02006_amd import binding
    return binding


# (key, value): nothing; nobody looks for the others' sums, every workgroup recomputes them; the hand-over through memory
HOOKS = {"plain": None, "recompute": ("TUNE_DECODE_SCATTER", 3), "far": ("TUNE_SMALL_FAR", 1)}


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["fp16", "bf16"])
@pytest.mark.parametrize("hook", list(HOOKS))
# beyond 32 rows: sixteen parts of 17 and 18 k-steps (quarters of four and five) on half a tile and on one tile and a half; ten parts of fourteen; one part of
# twenty, no hand-over; two parts of 34, off cache lines; rows at both ends of the range and on both sides of 48 = three tiles of rows.  Up to 32: parts of four
# k-steps, one to a wave; fifteen parts; parts of five to seven; one row, a full tile of rows, one more than that, two full tiles
@pytest.mark.parametrize("M,K,N", [(33, 8832, 64), (64, 8832, 192), (47, 4480, 2112), (48, 4480, 2112), (49, 640, 16400), (64, 2176, 13832),
                                   (1, 8192, 1032), (5, 512, 136), (16, 768, 776), (17, 1280, 5128), (32, 4480, 5120), (24, 896, 8968)])
def test_tiles_of_128_columns(B, M, K, N, hook, dtype):
    g = torch.Generator(device="cuda").manual_seed(M + K + N)
    w = (torch.randn((K, N), generator=g, device="cuda") * 0.05).to(dtype)
    x = torch.randn((M, K), generator=g, device="cuda").to(dtype)
    fn = B.linear_fp16 if dtype == torch.float16 else B.linear_bf16
    plan = (ctypes.c_int * 5)()
    assert B.lib().morph_plan_decode(B.KIND_FP16, M, K, N, plan) == 0
    assert list(plan[:2]) == [1, -(-N // 128)] and plan[4] == 2, "the planner leaves it to another kernel"
    out = torch.full((M + 1, N), 77.0, dtype=dtype, device="cuda")
    if HOOKS[hook]:
        B.set_tuning(getattr(B, HOOKS[hook][0]), HOOKS[hook][1])
    try:
        fn(x, w, B.new_workspace(B.workspace_bytes(B.KIND_FP16, M, K, N)), out=out[:M])
        torch.cuda.synchronize()
    finally:
        if HOOKS[hook]:
            B.set_tuning(getattr(B, HOOKS[hook][0]), 0)
    assert bool((out[M] == 77.0).all()), "wrote past the last row"
    xd, wd = x.double(), w.double()
    ref = xd @ wd
    u = 2.0 ** -11 if dtype == torch.float16 else 2.0 ** -8
    bound = (K + 64) * 2.0 ** -24 * (xd.abs() @ wd.abs()) + u * ref.abs() + 2.0 ** -25
    worst = ((out[:M].double() - ref).abs() / bound).max()
    print(f"M={M} K={K} N={N} {hook} {dtype}: {float(worst):.3f} of the bound", flush=True)
    assert worst <= 1.0
