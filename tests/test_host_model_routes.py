"""Which kernel a product is launched on, read from the launch itself (workgroups and LDS bytes) on the CPU execution model
of the kernels; no operand is read."""
import subprocess
import os

import pytest

from test_host_model import hostmodel  # noqa: F401  (fixture)


def routes(hostmodel, tmp_path, calls, **env):
    """[(format, M, N, K steps of 128 operand bytes, BF16 output, ldc or 0, bytes that c is off 16, tiled, bound)] ->
    [(workgroups, LDS bytes)]"""
    lines = []
    for fmt, M, N, steps, bf16, ldc, off, tiled, wg in calls:
        K = steps * {"fp8": 128, "fp4": 256, "bf16": 64}[fmt]
        lines.append(f"route {fmt} {M} {N} {K} {'bf16' if bf16 else 'f32'} {ldc or N} {off}" + (" tiled" if tiled else "") + (f" wg={wg}" if wg else ""))
    case = tmp_path / "routes.txt"
    case.write_text("\n".join(lines) + "\n")
    res = subprocess.run([hostmodel, str(case)], capture_output=True, text=True, timeout=300,
                         env=dict(os.environ, WAVESIM_BLOCKS="0", **{k: str(v) for k, v in env.items()}))
    assert res.returncode == 0, (res.stdout + res.stderr)[-2000:]
    out = [tuple(int(v) for v in line.split()[1:]) for line in res.stdout.splitlines() if line.startswith("route")]
    assert len(out) == len(calls) and all(o[0] == 0 for o in out)
    return [o[1:] for o in out]


@pytest.mark.parametrize("bf16", [True, False], ids=["bf16", "f32"])
def test_bound_holds_where_rows_of_c_are_far_apart(hostmodel, tmp_path, bf16):
    """Whole 128x128 tiles keep the bound on workgroups for every distance of the rows of C that 128-row tiles can address
    (below 16 MiB); the resident 256-row tiles address 8 MiB at most."""
    mib = (1 << 20) // (2 if bf16 else 4)
    calls = [("fp8", 896, 512, 4, bf16, ldc, 0, tiled, wg) for wg in (1, 3) for tiled in (True, False)
             for ldc in (512, 8 * mib - 8, 8 * mib, 10 * mib, 16 * mib - 8)]
    for call, (workgroups, _) in zip(calls, routes(hostmodel, tmp_path, calls)):
        assert workgroups == call[-1], call


def test_tile_is_chosen_for_the_units_of_the_device(hostmodel, tmp_path):
    """A device of n units runs a product on the kernel and tile of a 256-unit device that is held to n workgroups (shapes at
    which the contention of a fully used chip, counted in the first case only, does not change the choice)."""
    shapes = [("fp8", 2048, 2048, 32, True), ("fp8", 1024, 4096, 32, True), ("fp8", 512, 6144, 32, True), ("bf16", 1024, 1024, 16, False),
              ("fp4", 512, 1024, 12, True), ("fp8", 256, 1024, 8, False)]
    for units in (32, 64):
        own = routes(hostmodel, tmp_path, [s + (0, 0, True, 0) for s in shapes], WAVESIM_CUS=units)
        held = routes(hostmodel, tmp_path, [s + (0, 0, True, units) for s in shapes])
        full = routes(hostmodel, tmp_path, [s + (0, 0, True, 0) for s in shapes])
        lds = lambda r: [v[1] for v in r]  # noqa: E731
        assert lds(own) == lds(held)
        assert lds(own) != lds(full)
