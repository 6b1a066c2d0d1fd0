"""Rounding error of the run-time-length passes: no larger than that of the mixed-radix passes.

The error of one application G A x (relative L2 against long double) is compared with the one that
the mixed-radix passes, which these lengths ran on before, had for the same inputs on an MI355X.
Tolerance: 2 per cent above that figure; another seed moves an error at these sizes by 1 per cent
at most."""
import numpy as np
import pytest
import torch

from paper_1508_02045_amd import fgh

pytestmark = pytest.mark.gpu


def error(N, dtype):
    """Relative L2 error of G A x: a two-valued scalar A of contrast 100 and standard normal x."""
    rng = np.random.default_rng(1000 + sum(N))
    d = len(N)
    A = 1.0 + 99.0 * (rng.random(N) < 0.3)
    x = rng.standard_normal((d,) + N).astype(dtype)
    prec = fgh.FGH_FP64 if dtype == np.float64 else fgh.FGH_FP32_REFINED
    plan = fgh.Plan(N, precision=prec, A=torch.from_numpy(A).cuda())
    y = plan.apply(torch.from_numpy(x).cuda()).cpu().numpy()
    plan.close()
    k = np.meshgrid(*[np.round(np.fft.fftfreq(n) * n).astype(np.longdouble) for n in N], indexing="ij")
    kk = sum(f * f for f in k)
    kk[(0,) * d] = 1
    axes = tuple(range(1, d + 1))
    Z = np.fft.fftn(A.astype(np.longdouble) * x, axes=axes)
    assert Z.dtype == np.clongdouble
    t = sum(f * z for f, z in zip(k, Z)) / kk
    ref = np.fft.ifftn(np.stack([f * t for f in k]), axes=axes).real
    e = float(np.linalg.norm((y - ref).astype(np.float64)) / np.linalg.norm(ref.astype(np.float64)))
    print(N, np.dtype(dtype).name, f"{e:.3e}", flush=True)
    return e


@pytest.mark.parametrize("N,mixed", [((51, 51), 4.108e-16), ((75, 75), 3.809e-16), ((85, 85), 4.111e-16),
                                     ((105, 105), 3.814e-16), ((165, 165), 4.465e-16), ((225, 225), 4.306e-16),
                                     ((255, 289), 5.071e-16), ((75, 75, 75), 4.523e-16), ((85, 85, 85), 5.033e-16),
                                     ((143, 121, 77), 5.224e-16)])
def test_register_radices(N, mixed):
    """Products of two register radices, 9 to 17 among them, in double precision."""
    assert error(N, np.float64) <= 1.02 * mixed


@pytest.mark.parametrize("N,mixed64,mixed32", [((441, 441), 4.868e-16, 2.485e-07), ((525, 525), 4.559e-16, 2.371e-07),
                                               ((945, 945), 5.074e-16, 2.701e-07), ((999, 999), 6.613e-16, 3.107e-07),
                                               ((1023, 767), 6.103e-16, 3.247e-07), ((511, 509), 1.174e-15, 6.331e-07),
                                               ((201, 151, 101), 8.954e-16, 4.803e-07)])
def test_dense_steps(N, mixed64, mixed32):
    """Dense steps of composite length (49, 35, 63, 111, 93) and of prime length, in both precisions."""
    assert error(N, np.float64) <= 1.02 * mixed64
    assert error(N, np.float32) <= 1.02 * mixed32


@pytest.mark.parametrize("N,mixed", [((51, 51), 2.222e-07), ((75, 75), 2.079e-07), ((105, 105), 2.068e-07),
                                     ((225, 225), 2.267e-07), ((375, 375), 2.488e-07), ((127, 129), 3.597e-07),
                                     ((1021, 1021), 1.150e-06), ((75, 75, 75), 2.445e-07), ((105, 105, 105), 2.456e-07),
                                     ((89, 97, 101), 4.531e-07)])
def test_single_precision(N, mixed):
    """Smooth and prime lengths in single precision, whose multiplier weights are formed in it."""
    assert error(N, np.float32) <= 1.02 * mixed
