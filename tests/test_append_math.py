"""The 8-bit append's quotient, on the host: the fp64 product with the reciprocal of the scale, rounded to
binary32, is the correctly rounded binary32 quotient for every bf16 value."""
import numpy as np
import pytest


@pytest.mark.parametrize("kind", ["usual", "any bits", "special"])
def test_product_with_the_reciprocal_is_the_quotient(kind):
    rng = np.random.default_rng(3)
    x = (np.arange(1 << 16, dtype=np.uint32) << 16).view(np.float32)
    x = x[~np.isnan(x)]
    scales = {"usual": (rng.uniform(1, 2, 400) * 2.0 ** rng.integers(-20, 20, 400)).astype(np.float32),
              "any bits": rng.integers(1, 0x7F800000, 400).astype(np.uint32).view(np.float32),
              "special": np.array([1, 448, 1 / 448, 2.0 ** -126, 1.4e-45, 3.4e38, float.fromhex("0x1.af286cp-8"),
                                   float.fromhex("0x1.fffffep+0"), float.fromhex("0x1.000002p+0")], np.float32)}[kind]
    with np.errstate(all="ignore"):
        for s in scales:
            quotient = x / s
            product = (x.astype(np.float64) * (1.0 / np.float64(s))).astype(np.float32)
            # quotients this small all give code zero, whichever way they round
            tiny = (np.abs(quotient) < 2.0 ** -100) & (np.abs(product) < 2.0 ** -100)
            assert np.all((quotient.view(np.uint32) == product.view(np.uint32)) | tiny)
