"""The quantized format's formula in numpy, and weights at the ends of the floating range (for the tests of quantizer and oracle)."""
import numpy as np

GROUP = 128


def extreme_columns(K, N):
    """Standard normal weights; every eleventh column gets one kind of extreme values in every group of 128 rows."""
    w = np.random.default_rng([250602006, 72, K, N]).standard_normal((K, N)).astype(np.float32)
    inf, nan = np.float32(np.inf), np.float32(np.nan)
    kinds = [{3: inf, 5: -1e5}, {3: -inf, 5: 1e5}, {0: inf, 127: -inf}, {64: nan}, {9: 3e38, 10: -1e5}, {9: 3e38, 10: -3e38},
             {1: nan, 2: inf, 3: -7e4}, {r: nan for r in range(GROUP)}, {100: 1e30, 101: -2e5}, {100: 1e9, 101: -1e7}, {0: 2e14, 1: -1.4e14}]
    for n in range(N):
        for g in range(K // GROUP):
            for r, v in kinds[n % len(kinds)].items():
                w[g * GROUP + r, n] = v
    return w


def formula_record(w, L):
    """Codes [K,N], scales fp16 and zero points [K/128,N]: lo = min(0, w), hi = max(0, w), s = (hi - lo) / L rounded up to fp16 within 2^-14 .. 65504,
    z = clamp(rint(-lo / s), 0, L), q = clamp(rint(w / s) + z, 0, L); NaN counts in no range and has the code of 0."""
    with np.errstate(all="ignore"):
        g = w.reshape(-1, GROUP, w.shape[1])
        lo = np.fmin.reduce(np.concatenate([g, np.zeros_like(g[:, :1])], 1), 1)
        hi = np.fmax.reduce(np.concatenate([g, np.zeros_like(g[:, :1])], 1), 1)
        s32 = ((hi - lo) / np.float32(L)).astype(np.float32)
        s = s32.astype(np.float16)
        up = np.nextafter(s, np.float16(np.inf))
        s = np.where(s.astype(np.float32) < s32, up, s).astype(np.float16)
        s = np.clip(s, np.float16(2.0 ** -14), np.float16(65504)).astype(np.float16)
        sf = s.astype(np.float32)
        z = np.clip(np.rint(-lo / sf), 0, L).astype(np.int64)
        t = np.clip(np.nan_to_num(np.rint(g / sf[:, None]), nan=0.0, posinf=L, neginf=-L), -L, L).astype(np.int64)
        q = np.clip(t + z[:, None], 0, L).reshape(w.shape)
    return q, s, z
