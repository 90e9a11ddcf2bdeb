"""A launch that fails is reported once and not tried again: the C++ half of the binding is bound to stand-ins for the library's functions that
fail at the first call and would succeed at a second.  Nothing is launched through them."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

ERR_DEVICE = 6


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_02006_amd import binding
    binding.lib()
    return binding


def test_a_failed_launch_raises_and_is_not_repeated(B):
    K, N, M = 128, 256, 4
    w = torch.randn((K, N), device="cuda")
    x = {dt: torch.randn((M, K), device="cuda").to(dt) for dt in (torch.float16, torch.bfloat16)}
    w4, w8, w4n = B.quantize_layer(w), B.quantize_layer_w8(w), B.quantize_layer_native(w)
    ws = B.new_workspace(1 << 20)
    h, bf = torch.float16, torch.bfloat16
    calls = [
        ("morph_linear_fp16", lambda: B.linear_fp16(x[h], w.to(h), ws)), ("morph_linear_bf16", lambda: B.linear_bf16(x[bf], w.to(bf), ws)),
        ("morph_linear_w4a16", lambda: B.linear_w4a16(x[h], *w4, ws)), ("morph_linear_w4a16_bf16", lambda: B.linear_w4a16_bf16(x[bf], *w4, ws)),
        ("morph_linear_w8a16", lambda: B.linear_w8a16(x[h], *w8, ws)), ("morph_linear_w8a16_bf16", lambda: B.linear_w8a16_bf16(x[bf], *w8, ws)),
        ("morph_linear_w4a16_native", lambda: B.linear_w4a16_native(x[h], *w4n, ws)),
        ("morph_linear_w4a16_native_bf16", lambda: B.linear_w4a16_native_bf16(x[bf], *w4n, ws)),
        ("morph_glue", lambda: B.glue(B.GLUE_RMS, x[h])), ("morph_glue_bf16", lambda: B.glue(B.GLUE_RMS, x[bf])),
        ("morph_cosine_rows", lambda: B.cosine_rows(x[h], x[h])), ("morph_cosine_rows_bf16", lambda: B.cosine_rows(x[bf], x[bf])),
        ("morph_quantize_layer", lambda: B.quantize_layer(w)), ("morph_quantize_layer_w8", lambda: B.quantize_layer_w8(w)),
        ("morph_quantize_layer_native_only", lambda: B.quantize_layer_native(w)),
        ("morph_dequantize_w4", lambda: B.dequantize_w4(*w4)), ("morph_dequantize_w8", lambda: B.dequantize_w8(*w8)),
        ("morph_dequantize_w4_native", lambda: B.dequantize_w4_native(*w4n)),
    ]
    real = [ctypes.cast(getattr(B.lib(), name), ctypes.c_void_p).value for name in B._CALL_FNS]
    count = [0]

    def fail_once():
        count[0] += 1
        return ERR_DEVICE if count[0] == 1 else 0

    stub = ctypes.CFUNCTYPE(ctypes.c_int)(fail_once)
    try:
        for name, call in calls:
            bound = list(real)
            bound[B._CALL_FNS.index(name)] = ctypes.cast(stub, ctypes.c_void_p).value
            B._call.bind(bound)
            count[0] = 0
            with pytest.raises(B.MorphError) as e:
                call()
            assert e.value.status == ERR_DEVICE and name + ":" in str(e.value) and count[0] == 1
    finally:
        B._call.bind(real)
    for name, call in calls:                             # and with the library's own functions all of them succeed
        call()
    torch.cuda.synchronize()
