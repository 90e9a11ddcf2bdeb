"""The LDS-ring kernels at the sizes where they can go wrong: one row more than a tile, ragged last columns, K of one group (fewer
groups than a workgroup has parts), K split as far as it goes, and every partial sum recomputed (nobody waits).

Bound, per element, against an fp64 product with the dequantized weights: a weight rounded to x's 16-bit format is off by at most
u_w |w| (and half the smallest subnormal, 2^-25 in fp16); fp32 sums of K products of at most K + 64 additions each off by 2^-24 of
their magnitude; y rounded to 16 bits by u_y |y|.  So |y - ref| <= (u_w + (K + 64) 2^-24) sum|x||w| + 2^-25 sum|x| + u_y |ref| + 2^-25."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2506_02006_amd import synth

pytestmark = pytest.mark.gpu

KINDS = ("dense", "w4", "w8")
TILES = [(1, m) for m in (4, 5, 6, 7, 8)] + [(2, m) for m in (5, 6, 7, 8)] + [(3, m) for m in (4, 6)] + [(4, m) for m in (5, 6, 7, 8)]
ROWS_OF = {1: 1, 2: 2, 3: 1, 4: 2}
COLS_OF = {1: 256, 2: 256, 3: 128, 4: 128}


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_02006_amd import binding
    binding.lib()
    binding.warmup()
    return binding


class Problem:
    def __init__(self, B, kind, bf, M, K, N):
        self.B, self.kind, self.bf, self.M, self.K, self.N = B, kind, bf, M, K, N
        g = torch.Generator(device="cuda").manual_seed(synth.BASE_SEED + M + 3 * K + 7 * N)
        dt = torch.bfloat16 if bf else torch.float16
        self.x = torch.randn((M, K), generator=g, device="cuda").to(dt)
        w = torch.randn((K, N), generator=g, device="cuda") * 0.02
        if kind == "dense":
            self.w = (w.to(dt),)
            W = self.w[0].double()
        elif kind == "w4":
            self.w = B.quantize_layer(w)
            W = B.dequantize_w4(*self.w).double()
        else:
            self.w = B.quantize_layer_w8(w)
            W = B.dequantize_w8(*self.w).double()
        self.ref = self.x.double() @ W
        u = 2.0 ** -8 if bf else 2.0 ** -11          # half a unit in the last of 8 (11) significant bits
        size = self.x.double().abs() @ W.abs()
        self.bound = ((0.0 if kind == "dense" else u) + (K + 64) * 2.0 ** -24) * size + 2.0 ** -25 * self.x.double().abs().sum(1, keepdim=True) \
            + u * self.ref.abs() + 2.0 ** -25

    def call(self):
        B = self.B
        return {("dense", 0): B.linear_fp16, ("dense", 1): B.linear_bf16, ("w4", 0): B.linear_w4a16, ("w4", 1): B.linear_w4a16_bf16,
              ("w8", 0): B.linear_w8a16, ("w8", 1): B.linear_w8a16_bf16}[(self.kind, self.bf)]

    def workspace(self):
        B = self.B
        return B.new_workspace(B.workspace_bytes({"dense": B.KIND_FP16, "w4": B.KIND_W4A16, "w8": B.KIND_W8A16}[self.kind], self.M, self.K, self.N))

    def run(self):
        fn, ws = self.call(), self.workspace()
        out = torch.full((self.M + 1, self.N), 77.0, dtype=self.x.dtype, device="cuda")
        y = fn(self.x, *self.w, ws=ws, out=out[: self.M])
        torch.cuda.synchronize()
        assert bool((out[self.M] == 77.0).all()), "wrote past the last row"
        return y

    def check(self):
        y = self.run()
        worst = float(((y.double() - self.ref).abs() / self.bound).max())
        assert worst <= 1.0, f"{worst} of the bound"
        return y


def no_wait(B, p):
    """The same bits when every workgroup recomputes the others' parts instead of waiting for them."""
    y = p.check()
    B.set_tuning(B.TUNE_DECODE_SCATTER, 3)
    try:
        assert torch.equal(p.check().view(torch.int16), y.view(torch.int16))
    finally:
        B.set_tuning(B.TUNE_DECODE_SCATTER, 0)


@pytest.mark.parametrize("layout,mt", TILES)
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("bf", [0, 1])
def test_every_tile(B, kind, bf, layout, mt):
    if kind == "dense" and (layout, mt) == (3, 6):
        pytest.skip("not built: the LDS holds too few stages")
    bm, bn = 16 * mt * ROWS_OF[layout], COLS_OF[layout]
    B.set_tuning(B.TUNE_TILED, 16 * layout + mt)
    try:
        for M, K, N, split in ((65, 128, 8, 1), (max(bm + 1, 66), 896, bn + 8, 3), (max(bm, 65), 2560, 2 * bn - 8, 16), (2 * bm + 3, 1152, bn, 1)):
            print(f"ring {kind} bf={bf} layout={layout} mt={mt} M={M} K={K} N={N} S={split}", flush=True)
            B.set_tuning(B.TUNE_TILED_SPLIT, split)
            no_wait(B, Problem(B, kind, bf, M, K, N))
    finally:
        B.set_tuning(B.TUNE_TILED, 0)
        B.set_tuning(B.TUNE_TILED_SPLIT, 0)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("bf", [0, 1])
def test_planned(B, kind, bf):
    """The planner's own choice at both sides of its lines: 16 / 17, 32 / 33 and 64 / 65 rows, and the matrices beyond 26e6 weights."""
    for M, K, N in ((17, 128, 8), (32, 2048, 520), (33, 1792, 264), (64, 4096, 1032), (64, 5120, 5128), (33, 5120, 5128), (33, 2048, 16392), (64, 2048, 16392), (65, 128, 8), (65, 4096, 1032), (100, 1024, 4104)):
        print(f"ring planned {kind} bf={bf} M={M} K={K} N={N}", flush=True)
        p = Problem(B, kind, bf, M, K, N)
        no_wait(B, p)
        if kind == "dense" and M <= 64:                          # and without tiles of 128 columns, which take most of the matrices that the ring runs else
            B.set_tuning(B.TUNE_TILED, 2)
            try:
                no_wait(B, p)
            finally:
                B.set_tuning(B.TUNE_TILED, 0)
        if kind == "w4" and not bf and M <= 64:                  # either storage order: the same bits
            ws = B.new_workspace(B.workspace_bytes(B.KIND_W4A16_NATIVE, M, K, N))
            nat = B.linear_w4a16_native(p.x, B.repack_w4_native(p.w[0]), p.w[1], p.w[2], ws=ws)
            assert np.array_equal(nat.cpu().numpy().view(np.uint16), p.run().cpu().numpy().view(np.uint16))


@pytest.mark.parametrize("kind", KINDS)
def test_workspace_of_the_older_kernels(B, kind):
    """A workspace that covers only what the kernels without the ring need still serves the call, by those kernels.  (The size asked for
    covers both formats of x: where the ring's plan for this one needs no more than the smaller size, the ring takes the call.)"""
    tag = {"dense": B.KIND_FP16, "w4": B.KIND_W4A16, "w8": B.KIND_W8A16}[kind]
    fn = {"dense": B.linear_fp16, "w4": B.linear_w4a16, "w8": B.linear_w8a16}[kind]
    taken = 0
    for M, K, N in ((160, 2048, 6144), (100, 2048, 2048), (320, 3072, 9216), (72, 3072, 8192), (320, 4096, 9216)):   # (the last: codes on the ring with K split)
        B.set_tuning(B.TUNE_TILED, 1)
        try:
            p = Problem(B, kind, 0, M, K, N)
            need = B.workspace_bytes(tag, M, K, N)
            older = p.check()
        finally:
            B.set_tuning(B.TUNE_TILED, 0)
        if need >= B.workspace_bytes(tag, M, K, N):
            continue
        ring = p.check()
        got = fn(p.x, *p.w, ws=B.new_workspace(need) if need else None)
        same = [torch.equal(got.view(torch.int16), y.view(torch.int16)) for y in (older, ring)]
        assert any(same)
        taken += same[0] and not torch.equal(older, ring)
    assert taken, "no shape where the older kernels stood in for the ring"


@pytest.mark.parametrize("kind", ["w4", "w8"])
@pytest.mark.parametrize("bf", [0, 1])
@pytest.mark.parametrize("M,K,N", [(65, 2048, 6144), (100, 14336, 4096), (160, 2048, 6144), (256, 4096, 4096)])
def test_codes_beyond_64_rows_stay_exact(B, kind, bf, M, K, N):
    """Where codes are multiplied as they are, y is the 16-bit rounding of a sum with fp32 errors only: relative to |y| these add up like a walk of
    at most K steps of 2^-25, 2^-18 for the largest K here, so that a rounding to 16 bits (steps of 2^-10 .. 2^-11 of y in fp16, eight times that in
    bfloat16) goes another way in about 2 * 2^-18 / 2^-11 = 1.6 % of the elements; zero points taken off large sums may triple that.  Weights rounded
    to 16 bits (2^-12 of y and more) change a quarter of them and more."""
    print(f"exact codes {kind} bf={bf} M={M} K={K} N={N}", flush=True)
    p = Problem(B, kind, bf, M, K, N)
    y = p.run()
    share = float((y != p.ref.to(y.dtype)).double().mean())
    assert share <= 0.05, share


@pytest.mark.parametrize("kind", ["w4", "w8"])
def test_weights_beyond_the_fp16_range(B, kind):
    """Masters of up to 3e5 (the format's scales allow it) and small rows: the products stay in range, so the results are finite and right."""
    M, K, N = 100, 4096, 4096
    g = torch.Generator(device="cuda").manual_seed(synth.BASE_SEED + 81)
    w = torch.randn((K, N), generator=g, device="cuda") * 6e4
    x = (torch.randn((M, K), generator=g, device="cuda") * 2.0 ** -12).to(torch.float16)
    rec = B.quantize_layer(w) if kind == "w4" else B.quantize_layer_w8(w)
    W = (B.dequantize_w4 if kind == "w4" else B.dequantize_w8)(*rec).double()
    assert float(W.abs().max()) > 65504
    fn, tag = (B.linear_w4a16, B.KIND_W4A16) if kind == "w4" else (B.linear_w8a16, B.KIND_W8A16)
    y = fn(x, *rec, ws=B.new_workspace(B.workspace_bytes(tag, M, K, N))).double()
    ref = x.double() @ W
    assert bool(torch.isfinite(y).all()) and float((y - ref).norm() / ref.norm()) <= 2.0 ** -11


@pytest.mark.parametrize("kind,hidden,inter,M", [("fp16", 4096, 9216, 64), ("w8", 2048, 4096, 40), ("w8", 4096, 11008, 64)])
def test_stack_on_the_workspace_of_the_older_kernels(B, kind, hidden, inter, M):
    """A step through a stack takes a workspace that covers only what the kernels without the ring need, as a single linear does."""
    tag = {"fp16": B.KIND_FP16, "w8": B.KIND_W8A16}[kind]
    st = B.LayerStack(hidden, inter, M)
    g = torch.Generator(device="cuda").manual_seed(synth.BASE_SEED + 83)
    shapes = st._shapes()
    layer = {}
    for name, (K, N) in shapes.items():
        w = torch.randn((K, N), generator=g, device="cuda") * 0.02
        layer[name] = ("fp16", w.to(torch.float16)) if kind == "fp16" else ("w8",) + tuple(B.quantize_layer_w8(w))
    st.add_layer(layer)
    x = torch.randn((M, hidden), generator=g, device="cuda").to(torch.float16)
    want = st.forward(x.clone())
    plan = (ctypes.c_int * 5)()
    def ring():                                              # the dense linears that the ring takes
        return [name for name, (K, N) in shapes.items() if kind == "fp16" and B.lib().morph_plan_decode(tag, M, K, N, plan) == 0 and plan[0] == 0]
    assert ring() == (["gate_up"] if kind == "fp16" else [])
    B.set_tuning(B.TUNE_TILED, 1)
    try:
        assert not ring()
        need = max(B.workspace_bytes(tag, M, K, N) for K, N in shapes.values())
        older = st.forward(x.clone())
    finally:
        B.set_tuning(B.TUNE_TILED, 0)
    asked = max(B.workspace_bytes(tag, M, K, N) for K, N in shapes.values())
    print(f"stack {kind} {hidden} {inter} M={M}: {need} and {asked} bytes", flush=True)
    assert need < asked, "the ring needs no more here: another shape is wanted"
    st.ws = B.new_workspace(need)
    got = st.forward(x.clone())
    # each of the linears ran on one of the two families; a step's own rounding is 2^-11 per linear (four, and four row steps)
    for ref in (want, older):
        assert float((got.double() - ref.double()).norm() / ref.double().norm()) <= 8 * 2.0 ** -11


@pytest.mark.parametrize("kind,bf,M,K,N", [("w8", 0, 256, 4096, 6144), ("dense", 0, 256, 14336, 4096), ("w4", 0, 2048, 13824, 5120), ("w8", 1, 33, 14336, 1024),
                                           ("w8", 1, 17, 1024, 28672)])
def test_the_planner_keeps_to_the_faster_kernel(B, kind, bf, M, K, N):
    """Shapes on which the ring is 5 to 30 % slower than the kernels without it, with weights from memory: the planner's choice takes no longer than
    those (best of up to 60 blocks of launches over copies of the weights, in turn, until that is seen; 5 % for the clock)."""
    p = Problem(B, kind, bf, M, K, N)
    copies = [p.w] + [tuple(t.clone() for t in p.w) for _ in range(max(1, min(23, (600 << 20) // sum(t.numel() * t.element_size() for t in p.w))))]
    out = torch.empty((M, N), dtype=p.x.dtype, device="cuda")
    fn, best = p.call(), {0: 1e9, 1: 1e9}
    try:
        for block in range(60):
            if block > 5 and best[0] <= 1.05 * best[1]:
                break
            for key in best:
                B.set_tuning(B.TUNE_TILED, key)
                ws = p.workspace()
                fn(p.x, *copies[0], ws=ws, out=out)
                t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                t0.record()
                for w in copies:
                    fn(p.x, *w, ws=ws, out=out)
                t1.record()
                t1.synchronize()
                best[key] = min(best[key], t0.elapsed_time(t1) * 1e3 / len(copies))
    finally:
        B.set_tuning(B.TUNE_TILED, 0)
    print(f"planner {kind} bf={bf} M={M} K={K} N={N}: {best[0]:.1f} us, without the ring {best[1]:.1f} us", flush=True)
    assert best[0] <= 1.05 * best[1], best
