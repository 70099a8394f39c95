"""The Rosenbrock steps' reciprocal against the division, bit for bit (up to
the payload of a NaN), over the whole range of FP64: the normal numbers, those
whose reciprocal is subnormal, the subnormal ones (whose reciprocal overflows
below 2^-1024), zeros, infinities and NaN.  A registered system evaluates both:
its first component grows where they differ, its second where 1/x differs from
3 (1 / (3 x)), which is now and then the case and shows that a difference is
seen.
"""
import numpy as np
import pytest
import torch

from paper_2609_02876_amd import binding as B

pytestmark = pytest.mark.gpu

SOURCE = """
struct System {
  template <class T>
  __device__ static T differ(const T& a, const T& b) { return T(0); }
  __device__ static double differ(const double& a, const double& b) {
    return double(a != b) * double(1 - int(a != a) * int(b != b)) +
           double(copysign(1.0, a) != copysign(1.0, b)) * double(a == b);
  }
  template <class T>
  __device__ static void rhs(const T* y, const T* p, T* f) {
    const T r = T(1) / p[0];
    f[0] = differ(ens::inverse(p[0]), r);
    f[1] = differ(T(3) * (T(1) / (T(3) * p[0])), r);
  }
  template <class T>
  __device__ static void vjp(const T* y, const T* p, const T* w, T* gy, T* gp) {
    gy[0] = T(0);
    gy[1] = T(0);
  }
};
"""
N = 1 << 20


def _of_exponents(lo, hi, rng):
    e = rng.integers(lo + 1023, hi + 1023, N, dtype=np.uint64)
    m = rng.integers(0, 1 << 52, N, dtype=np.uint64)
    s = rng.integers(0, 2, N, dtype=np.uint64)
    return ((s << np.uint64(63)) | (e << np.uint64(52)) | m).view(np.float64)


@pytest.fixture(scope="module")
def system():
    B.register_system("gpu_inverse", SOURCE, 2, 1)
    return "gpu_inverse"


@pytest.mark.parametrize("which", ["normal", "near_one", "subnormal_result", "subnormal",
                                   "overflow", "special"])
def test_inverse_is_the_division(system, which):
    print(f"case inverse {which}", flush=True)
    rng = np.random.default_rng(5)
    x = {"normal": lambda: _of_exponents(-1022, 1021, rng),
         "near_one": lambda: _of_exponents(-3, 3, rng),
         "subnormal_result": lambda: _of_exponents(1021, 1024, rng),
         "subnormal": lambda: rng.integers(1 << 50, 1 << 52, N, dtype=np.uint64).view(np.float64),
         "overflow": lambda: rng.integers(1, 1 << 50, N, dtype=np.uint64).view(np.float64),
         "special": lambda: np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 1.0, -3.0, 5e-324,
                                      2.0 ** -1024, 2.0 ** -1022, 2.0 ** 1022,
                                      1.7976931348623157e308])}[which]()
    y0 = torch.zeros(2, x.size, dtype=torch.float64, device="cuda")
    p = torch.tensor(x[None], device="cuda")
    ys, status = B.ensemble_solve(system, "tsit5", y0, p, 0.0, 1.0, 1e-3, 1e-3)
    ys = ys.cpu().numpy()[0]
    assert int(status.abs().max()) == 0
    assert int((ys[0] != 0).sum()) == 0
    if which == "near_one":
        assert int((ys[1] != 0).sum()) > 1000
