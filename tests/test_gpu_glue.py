"""The elementwise + row-norm steps at the widths where the vectors per thread change (512 threads of 8 columns: multiples of
4096, the widest rows are read twice), and on gates whose exponential overflows, infinities and NaN."""
import numpy as np
import pytest

from paper_2506_02006_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"fp16": 2e-3, "bf16": 8e-3}      # of the largest value of a step: one rounding of the result, 2^-12 (2^-9), of values up to about 5 rms, and a margin of 4

# element by element: the rounding of the result and 2e-5 for fp32 (the exponential at 88: 127 x 2^-24 of its argument in powers of two); half the
# smallest fp16 number, the smallest normal bfloat16 one
REL = {"fp16": 2.0 ** -11 + 2e-5, "bf16": 2.0 ** -8 + 2e-5}
TINY = {"fp16": 2.0 ** -25, "bf16": 2.0 ** -126}


def swiglu_fp32(gu, H):
    """The step by its definition: fp32 up to the products, the row's mean square in 64 bits."""
    x, u = gu[:, :H].float(), gu[:, H:].float()
    h = (x / (1.0 + torch.exp(-x)) * u).double()
    return (h / torch.sqrt((h * h).mean(dim=1, keepdim=True) + 1e-6)).numpy()


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2506_02006_amd import binding
    return binding


@pytest.mark.parametrize("fmt", ["fp16", "bf16"])
@pytest.mark.parametrize("M,H", [(3, H) for H in (8, 4096, 4104, 8192, 8200, 12288, 12296, 16384, 16392, 40008)] + [(M, H) for M in (256, 257) for H in (8, 4104, 8200, 16392)])
def test_glue_at_the_edges_of_the_vectors_per_thread(B, oracle, M, H, fmt):
    """... for a few rows and for about as many as there are compute units."""
    rng = np.random.default_rng([synth.BASE_SEED, 600, H])
    dt = torch.float16 if fmt == "fp16" else torch.bfloat16
    dev = lambda cols, s: torch.from_numpy((rng.standard_normal((M, cols)) * s).astype(np.float32)).to(dt).cuda()
    f64 = lambda t: t.double().cpu().numpy()
    qkv, a, b, gu = dev(3 * H, 2.0), dev(H, 1.0), dev(H, 3.0), dev(2 * H, 2.0)
    for op, p, q, want in ((B.GLUE_QKV, qkv, None, oracle.glue_qkv(f64(qkv))), (B.GLUE_RESIDUAL, a, b, oracle.glue_residual(f64(a), f64(b))),
                           (B.GLUE_SWIGLU, gu, None, oracle.glue_swiglu(f64(gu))), (B.GLUE_RMS, a, None, oracle.rms(f64(a)))):
        r = oracle.error_metric(f64(B.glue(op, p, q)), want)
        assert r["finite"] and r["err"] <= TOL[fmt], (op, r)


@pytest.mark.parametrize("fmt", ["fp16", "bf16"])
@pytest.mark.parametrize("H,col", [(4104, 100), (4104, 4100), (16392, 100), (16392, 16390), (20488, 16390)])
def test_swiglu_on_gates_that_overflow_the_exponential(B, fmt, H, col):
    """One special gate per row: finite ones far out on either side leave every column as the definition has it (in fp32, where the
    exponential overflows beyond 88.72), the special one among them; what is infinite or NaN by the definition (silu(inf) = inf,
    silu(-inf) = NaN) is so here, and only where it is there.  The special column is in a thread's first vector, in its last, and in one that is read twice."""
    dt = torch.float16 if fmt == "fp16" else torch.bfloat16
    gates = [-87.0, -87.5, -88.0, -88.5, -89.0, -104.0, -60000.0, 60000.0, float("inf"), float("-inf"), float("nan")]
    g = torch.Generator().manual_seed(7)
    gu = torch.randn((len(gates), 2 * H), generator=g).to(dt)
    for i, v in enumerate(gates):
        gu[i, col], gu[i, H + col] = v, 1.0
    want = swiglu_fp32(gu, H)
    got = B.glue(B.GLUE_SWIGLU, gu.cuda()).double().cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
    for i in range(8):
        assert (np.abs(got[i] - want[i]) <= REL[fmt] * np.abs(want[i]) + TINY[fmt]).all(), gates[i]


@pytest.mark.parametrize("fmt", ["fp16", "bf16"])
def test_swiglu_of_every_gate(B, fmt):
    """All finite values of the format, each in a row of its own kind: the short quotient has to serve them from -87 up, the division below."""
    dt = torch.float16 if fmt == "fp16" else torch.bfloat16
    x = torch.arange(65536, dtype=torch.int32).to(torch.int16).view(dt)
    x = x[torch.isfinite(x) & (x.abs() < 60000.0)].sort().values          # rows of gates of like size, so that no row hides its small ones
    H = 64
    x = x[:x.numel() // H * H].view(-1, H)
    gu = torch.cat([x, torch.ones_like(x)], 1)
    want, got = swiglu_fp32(gu, H), B.glue(B.GLUE_SWIGLU, gu.cuda()).double().cpu().numpy()
    assert (np.abs(got - want) <= REL[fmt] * np.abs(want) + TINY[fmt]).all()


def test_swiglu_gates_whose_reciprocal_is_subnormal(B):
    """1 / (1 + exp(-x)) is below the smallest normal number for gates under -87.3; against up values of 10^36 the quotient is what
    the row is made of."""
    H = 4104
    gates = [-87.0, -87.5, -88.0, -88.5]
    gu = torch.zeros((len(gates), 2 * H), dtype=torch.bfloat16)
    for i, v in enumerate(gates):
        gu[i, 100], gu[i, H + 100] = v, 2.0 ** 120
    want = swiglu_fp32(gu, H)
    assert (np.abs(want[:, 100]) > 60.0).all()
    got = B.glue(B.GLUE_SWIGLU, gu.cuda()).double().cpu().numpy()
    assert (np.abs(got - want) <= REL["bf16"] * np.abs(want)).all()
