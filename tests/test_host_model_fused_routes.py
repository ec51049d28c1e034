"""Which way the product with output quantization goes (one kernel, or the product and then the quantizer), and what a bound on
workgroups means for it, read from the launches on the CPU execution model of the kernels; no workgroup is simulated."""
import numpy as np
import pytest

import scale_layout as sl
from test_host_model import hostmodel, put, run_case  # noqa: F401


def launches(hostmodel, tmp_path, M, N, steps, axis, units, wg=0):  # noqa: F811
    """[(workgroups, LDS bytes)] of one call on a device of `units` units; tiled scales."""
    K = steps * 128
    names = []
    for name, rows in (("a", M), ("b", N)):
        names += [put(tmp_path, name + "q.bin", np.zeros((rows, K), np.uint8)), put(tmp_path, name + "s.bin", np.zeros(sl.tiled_bytes(rows, K // 32), np.uint8))]
    line = f"gemmq 0 {M} {N} {K} {N} {axis} {' '.join(names)} {tmp_path / 'out'} tiled" + (f" wg={wg}" if wg else "")
    res, calls = run_case(hostmodel, tmp_path, [line], WAVESIM_CUS=units, WAVESIM_BLOCKS=0)
    assert calls[0][0] == 0
    line, = [v for v in res.stdout.splitlines() if v.startswith("launches")]
    return [tuple(int(x) for x in v.split(":")) for v in line.split()[1:]]


@pytest.mark.parametrize("axis", [1, 2, 3])
def test_a_bound_that_bounds_nothing(hostmodel, tmp_path, axis):  # noqa: F811
    """As many workgroups as the device has units, or more, is no bound; fewer keep the call in one kernel."""
    free = launches(hostmodel, tmp_path, 256, 512, 12, axis, units=4)
    assert len(free) == 2
    for wg in (4, 5, 1 << 20):
        assert launches(hostmodel, tmp_path, 256, 512, 12, axis, units=4, wg=wg) == free
    assert [n for n, _ in launches(hostmodel, tmp_path, 256, 512, 12, axis, units=4, wg=3)] == [3]
