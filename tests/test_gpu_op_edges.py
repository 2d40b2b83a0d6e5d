"""pow at the edges of its fast path's integer steps: subnormal bases (scaled
into the normal range), bases on both sides of every significand split at
sqrt(1/2), the largest and smallest normal bases; within the 3 ulp and with the
special cases of test_gpu_ops.  sin and cos at every quadrant edge, both signs,
up to where FP32 has even integers only: exact there."""
import numpy as np
import pytest

from test_gpu_ops import _check_pow, _eval, env  # noqa: F401

pytestmark = pytest.mark.gpu

SPLIT = np.array([0x3f3504f2, 0x3f3504f3, 0x3f3504f4, 0x3f800000, 0x3f7fffff], dtype=np.uint32).view(np.float32)


@pytest.mark.parametrize("base", ["mult(x, 3e-39)", "mult(x, 1e-44)", "mult(x, 4e-38)", "mult(x, 1e38)"])
def test_pow_scaled_bases(env, base):  # noqa: F811
    got = _eval(env, [base, "mult(y, 0.8)", f"pow({base}, mult(y, 0.8))"])
    _check_pow(got[0], got[1], got[2], f"pow({base}, 0.8 y)")
    got = _eval(env, [base, f"pow({base}, if(x, 1.0, y))", f"pow({base}, if(x, -1.0, y))"])
    _check_pow(got[0], np.full_like(got[0], 1), got[1], f"pow({base}, 1)")
    if np.abs(got[0]).max() > 2.0 ** -127:
        _check_pow(got[0], np.full_like(got[0], -1), got[2], f"pow({base}, -1)")
    else:  # every reciprocal overflows
        assert np.all(np.isinf(got[2]) & (np.signbit(got[2]) == np.signbit(got[0])))


@pytest.mark.parametrize("exponent", [-126, -125, -64, -1, 0, 1, 63, 126])
def test_pow_significand_split(env, exponent):  # noqa: F811
    bases = [float(np.ldexp(v, exponent)) for v in SPLIT]
    texts = ["y"] + [t for b in bases for t in (f"if(x, {b!r}, y)", f"pow(if(x, {b!r}, y), y)")]
    got = _eval(env, texts)
    for j, b in enumerate(bases):
        assert np.all(got[1 + 2 * j] == np.float32(b))
        _check_pow(got[1 + 2 * j], got[0], got[2 + 2 * j], f"pow({b!r}, y)")


@pytest.mark.parametrize("scale", [1, 2 ** 10, 2 ** 22, 2 ** 23, 2 ** 25])
def test_sin_cos_quadrants(env, scale):  # noqa: F811
    ns = [s * (scale + j * 0.5) for j in range(9) for s in (1, -1)]
    ns = [float(np.float32(n)) for n in ns]
    got = _eval(env, [t for n in ns for t in (f"sin(if(x, {n!r}, y))", f"cos(if(x, {n!r}, y))")])
    for j, n in enumerate(ns):
        q = int(2 * n) % 4
        assert np.all(got[2 * j] == (0, 1, 0, -1)[q]), n
        assert np.all(got[2 * j + 1] == (1, 0, -1, 0)[q]), n
