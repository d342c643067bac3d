"""A user's field function that needs more registers than two waves to a SIMD
leave it gets all 512; one that spills little stays at two waves.  Read from
the compiler's resource remarks; no GPU is needed."""
import re

import pytest

from paper_2204_05586_amd import native

# n coefficients for each component, formed from the parameters once and kept
# through the fine steps: 8 n registers beside the integrator's own.
POLYNOMIALS = """
__device__ void mss_user_field(double t, const double* p, double* f) {
  double a[4][%d];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < %d; ++i) a[j][i] = (i + 1) * p[j & 1] / (16.0 * (j + 1));
  const double u = 1e3 * t;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    double v = 0.0;
#pragma unroll
    for (int i = %d - 1; i >= 0; --i) v = v * u * 0.5 + a[j][i];
    f[j] = 1e-2 * v;
  }
}
"""


def _kernels(n):
    """{kernel: (registers, scratch bytes)} of the integrators."""
    s = native.Sampler(POLYNOMIALS % (n, n, n), ["-Rpass-analysis=kernel-resource-usage"])
    found = re.findall(r"Function Name: mss_user_(\w+).*? VGPRs: (\d+).*?AGPRs: (\d+)"
                       r".*?ScratchSize \[bytes/lane\]: (\d+)", s.log, re.S)
    s.close()
    return {k: (int(v) + int(a), int(b)) for k, v, a, b in found if k != "work_chained"}


@pytest.mark.parametrize("n, all_registers", [(1, False), (16, False), (32, True)])
def test_registers_of_a_user_function(n, all_registers):
    kernels = _kernels(n)
    assert set(kernels) == {"integrate_2", "integrate_3", "work_integrate"}
    most = max(r for r, _ in kernels.values())
    scratch = max(b for _, b in kernels.values())
    print(n, kernels)
    assert (most > 256) == all_registers
    assert scratch <= 512
