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
    free = launches(hostmodel, tmp_path, 256, 512, 13, axis, units=4)
    assert len(free) == 2
    for wg in (4, 5, 1 << 20):
        assert launches(hostmodel, tmp_path, 256, 512, 13, axis, units=4, wg=wg) == free
    assert [n for n, _ in launches(hostmodel, tmp_path, 256, 512, 13, axis, units=4, wg=3)] == [3]


# M, N, axis, most K steps that stay in one kernel (0: none do; 99: all do) on 256 units
LINES = [(512, 1024, 1, 3), (512, 1024, 3, 3), (1024, 1536, 1, 7), (1280, 2048, 2, 12), (2048, 2048, 3, 12),   # at most a round of 128x128 tiles
         (1920, 2432, 1, 7), (2560, 2560, 2, 12), (1920, 2432, 3, 0),                                          # more than one
         (2816, 3072, 1, 0), (3072, 4096, 1, 0), (3328, 4096, 1, 99), (4096, 4096, 1, 99), (4352, 4096, 1, 0), (4096, 4096, 2, 0), (4096, 4096, 3, 0)]


@pytest.mark.parametrize("M,N,axis,steps", LINES)
def test_lines_between_the_two_ways(hostmodel, tmp_path, M, N, axis, steps):  # noqa: F811
    tile = 256 if -(-M // 256) * -(-N // 256) >= 128 else 128
    for n in {2, min(max(steps, 2), 13), min(max(steps, 2), 13) + 1}:
        got = launches(hostmodel, tmp_path, M, N, n, axis, units=256)
        if n <= steps:
            assert [g for g, _ in got] == [min(256, M // tile * (N // tile))], n
        else:
            assert len(got) == 2 and got[-1][1] == 0, n   # the quantizer asks for no dynamic LDS
