"""How long a wave of a chained run sleeps between polls: by the units that
still have to pass before the one it waits for.  A state arrives word by word,
so the word looked at may be the waited-for unit's while others are not: that
is the end of the line, not its far end.  Checked by the device compiler; no
GPU is needed."""
from paper_2204_05586_amd import native

# (tag waited for, tag seen, units ahead)
CASES = [
    (1, 0, 0), (2, 0, 1), (2, 1, 0), (70, 3, 66), (70, 69, 0),
    (2, 2, 0), (70, 70, 0),  # partly arrived
    (2 ** 31, 0, 2 ** 31 - 1), (2 ** 31, 2 ** 31, 0),
]


def test_units_ahead():
    checks = "\n".join(f"static_assert(mss::units_ahead({t}u, {h}u) == {a}u, \"{t} {h}\");"
                       for t, h, a in CASES)
    native.Sampler(f"""
#include "mss_work_device.h"
{checks}
__device__ void mss_user_field(double t, const double* params, double* field) {{ field[2] = 1.0; }}
""").close()
