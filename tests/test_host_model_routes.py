"""Which kernel a product is launched on, read from the launch itself (workgroups and LDS bytes) on the CPU execution model
of the kernels; no operand is read."""
import os
import subprocess

import pytest

from route_cases import K_STEP, ROUTES, TAIL_SHAPES, launch
from test_host_model import hostmodel  # noqa: F401  (fixture)


def routes(hostmodel, tmp_path, calls, **env):
    """[(format, M, N, K steps of 128 operand bytes, BF16 output, ldc or 0, bytes that c is off 16, tiled, bound)] ->
    [(workgroups, LDS bytes)]"""
    lines = []
    for fmt, M, N, steps, bf16, ldc, off, tiled, wg in calls:
        lines.append(f"route {fmt} {M} {N} {steps * K_STEP[fmt]} {'bf16' if bf16 else 'f32'} {ldc or N} {off}" + (" tiled" if tiled else "") + (f" wg={wg}" if wg else ""))
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


# Calls that the staged kernel, or a 256-row tile on the one-tile kernel, made up to 20 % slower, and neighbours that stay there.
FASTEST = [
    # one-tile 128x128 workgroups, two to a unit, against the staged kernel; row-major scales, few of them, FP32 out
    (("fp4", 2064, 3528, 21, True, 0, True, 0), ("one-tile", 128, 128)),
    (("fp8", 2254, 2584, 10, True, 0, True, 0), ("one-tile", 128, 128)),
    (("bf16", 1451, 3900, 104, True, 0, False, 0), ("one-tile", 128, 128)),
    (("fp8", 2254, 2584, 10, True, 0, False, 0), ("staged", 128, 64)),
    (("fp4", 651, 5566, 65, True, 0, True, 0), ("staged", 64, 128)),
    (("fp4", 564, 6688, 4, False, 0, True, 0), ("staged", 64, 64)),
    # few K steps, several tiles per workgroup: resident 128x128 tiles; more steps, row-major MXFP4, half the units idle: staged
    (("fp8", 896, 2688, 4, True, 0, False, 40), ("resident", 128, 128)),
    (("fp8", 5888, 128, 5, False, 0, True, 40), ("resident", 128, 128)),
    (("fp4", 1024, 4352, 5, True, 0, False, 0), ("staged", 64, 64)),
    (("fp4", 384, 1408, 4, True, 0, True, 100), ("staged", 64, 64)),
    (("fp8", 896, 5504, 11, True, 0, True, 40), ("staged", 128, 128)),
    # 256-row tiles that cannot go resident (fewer rows; rows of C that end off 16 bytes) against smaller ones
    (("fp8", 137, 74069, 38, True, 0, True, 0), ("staged", 64, 128)),
    (("fp8", 200, 49152, 32, True, 0, True, 0), ("one-tile", 256, 192)),
    (("fp8", 6144, 6922, 27, True, 0, False, 0), ("one-tile", 256, 256)),
    (("fp8", 6144, 6928, 27, True, 0, False, 0), ("resident", 256, 256)),
    # tiles of 96 columns in several rounds, or with few K steps, against the others; from 24 (35) steps on they are faster
    (("fp8", 768, 6144, 16, True, 0, True, 0), ("staged", 64, 64)),
    (("fp8", 850, 5120, 20, True, 0, False, 0), ("staged", 64, 64)),
    (("fp8", 251, 5504, 20, True, 0, True, 0), ("staged", 128, 64)),
    (("fp8", 265, 3360, 16, False, 0, False, 0), ("staged", 32, 64)),
    (("fp8", 441, 2352, 20, True, 0, True, 0), ("staged", 128, 64)),
    (("fp8", 200, 5120, 48, True, 0, True, 0), ("staged", 64, 96)),
    # a rest of few tiles that quarters would hardly compute sooner
    (("fp8", 12544, 2688, 51, True, 0, True, 0), ("resident", 256, 192)),
]


@pytest.mark.parametrize("table", [FASTEST, ROUTES], ids=["fastest", "gpu"])
def test_calls_take_the_kernel_named_for_them(hostmodel, tmp_path, table):
    calls = [("fp8" if fmt == "e5m2" else fmt, M, N, steps, bf16, N + pad, 0, tiled, bound)
             for (fmt, M, N, steps, bf16, pad, tiled, bound), _ in table]
    for (call, want), got in zip(table, routes(hostmodel, tmp_path, calls)):
        assert got == launch(call, *want), call


def test_rest_as_quarters(hostmodel, tmp_path):
    """The last launch of the call is that of the quarters, of every format, output and layout."""
    calls, want = [], []
    for M, N, kbytes in TAIL_SHAPES:
        rest = -(-M // 256) * -(-N // 256) % 256
        for fmt, steps in (("fp8", kbytes // 128), ("fp4", kbytes // 128), ("bf16", kbytes // 64)):   # (BF16 of the same K: twice the bytes)
            for bf16 in (True, False):
                for tiled in (True, False):
                    calls.append((fmt, M, N, steps, bf16, N, 0, tiled, 0))
                    want.append((4 * rest, launch((fmt, M, N, steps, bf16, 0, tiled, 0), "staged", 128, 128)[1]))
    assert routes(hostmodel, tmp_path, calls) == want


def test_nothing_is_launched_where_a_kernel_is_refused(hostmodel, tmp_path):
    """A product of two launches: whatever is refused before a launch is refused before the first one."""
    M, N, kbytes = TAIL_SHAPES[0]
    case = tmp_path / "case.txt"
    case.write_text(f"route fp8 {M} {N} {kbytes} bf16 {N} 0 tiled\n")
    for fails, status, launched in ((0, 6, 0), (1, 6, 0), (2, 0, 2)):   # both kernels ask for LDS
        res = subprocess.run([hostmodel, str(case)], capture_output=True, text=True, env=dict(os.environ, WAVESIM_BLOCKS="0", WAVESIM_FAIL_ATTRIBUTE=str(fails)))
        lines = {v.split()[0]: v.split()[1:] for v in res.stdout.splitlines()}
        assert (int(lines["status"][0]), len(lines["launches"])) == (status, launched), fails
