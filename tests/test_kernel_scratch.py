"""The integrators keep an interval in registers: none of a compiled field's
kernels uses scratch memory.  Read from the compiler's resource remarks; no GPU
is needed."""
import re

from paper_2204_05586_amd import native

DRIVE = """
__device__ void mss_user_field(double t, const double* p, double* f) {
  double s, c;
  mss::sincos_cw(mss::kTwoPi * (p[0] * t), &s, &c);
  f[0] = p[1] * c;
  f[2] = p[0];
  f[3] = 2.3;
}
"""


def test_no_scratch_in_compiled_integrators():
    s = native.Sampler(DRIVE, ["-Rpass-analysis=kernel-resource-usage"])
    scratch = dict(re.findall(r"Function Name: (\w+).*?ScratchSize \[bytes/lane\]: (\d+)", s.log,
                              re.S))
    s.close()
    assert {k: int(v) for k, v in scratch.items()} == {
        "mss_user_integrate_2": 0, "mss_user_integrate_3": 0, "mss_user_work_integrate": 0,
        "mss_user_work_chained": 0}
