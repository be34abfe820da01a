"""Register budget of the HIP kernels, from the compiler's resource remarks
recorded when the library is built: no kernel spills to scratch memory (a
spill in a step kernel costs more HBM traffic than the stencil itself)."""
import json
import os

import pytest

from paper_2110_03345_amd import build_lib


def _resources():
    if not os.path.exists(build_lib.RESOURCES):
        pytest.skip("library not built here (no resource remarks)")
    with open(build_lib.RESOURCES) as f:
        return json.load(f)


def test_no_kernel_spills_registers():
    res = _resources()
    steps = [k for k in res if "step2d_" in k or "step3d_" in k]
    assert len(steps) >= 40, len(steps)
    spills = {k: v["scratch"] for k, v in res.items() if v.get("scratch", 0) > 0}
    assert not spills, spills


def test_single_shot_3d_steps_meet_their_occupancy_target():
    """The leapfrog 3D kernels that ask for 4 waves per SIMD (radius-2 or
    narrower row blocks, and the 8-wave forward) stay within 128 VGPRs: the
    target is a compiler attribute, and this checks that it held."""
    import re
    res = _resources()
    seen = 0
    for name, r in res.items():
        m = re.search(r"step3d_kernelILi(\d)ELb(\d)ELi(\d)ELi(\d)ELi(\d)E", name)
        if not m:
            continue
        R, adj, ry, waves, mode = (int(x) for x in m.groups())
        if mode == 0 and (ry <= 2 or (not adj and waves == 8)):
            seen += 1
            assert r["vgpr"] <= 128, (name, r)
    assert seen >= 4, seen


def test_3d_steps_counted_on_for_four_waves_meet_them():
    """Every single-shot 3D kernel whose chunk length counts on four waves per SIMD
    (512 VGPRs a lane over four: 128), in both cache policies: the forward steps
    with one stencil field (modes 0, 1, 2, 4, four points a thread), the adjoint
    steps imaging from a stored v (5, 6, four) and the fused adjoint (0, two).
    All of them have to be there: a pattern that matches nothing proves nothing."""
    import re
    res = _resources()
    want = {(R, adj, vx, mode, stream) for R in (4, 5) for stream in (0, 1)
            for adj, vx, modes in ((0, 4, (0, 1, 2, 4)), (1, 4, (5, 6)), (1, 2, (0,))) for mode in modes}
    seen = {}
    for name, r in res.items():
        m = re.search(r"step3d_kernelILi(\d)ELb(\d)ELi(\d)ELi4ELi(\d)ELb(\d)E", name)
        if m:
            seen[tuple(int(x) for x in m.groups())] = r
    assert not want - set(seen), want - set(seen)
    bad = {k: seen[k] for k in want if seen[k]["vgpr"] > 128 or seen[k]["occupancy"] < 4}
    assert not bad, bad


def test_2d_sweeps_fit_their_block():
    """The kernels of the sweeps kept on the chip run 16 waves a block on one CU."""
    res = _resources()
    sweeps = {k: r for k, r in res.items() if "step2d_resident" in k}
    assert len(sweeps) == 15, sorted(sweeps)
    bad = {k: r for k, r in sweeps.items() if r["vgpr"] > 128 or r["occupancy"] < 4}
    assert not bad, bad


def test_batched_3d_steps_meet_the_single_shots_occupancy():
    """The batched forms of the same kernels, whose slots' parameters come from a
    table in memory: four waves per SIMD as well."""
    import re
    res = _resources()
    want = {(R, adj, vx, mode) for R in (4, 5)
            for adj, vx, modes in ((0, 4, (0, 1, 2, 4)), (1, 4, (5, 6)), (1, 2, (0,))) for mode in modes}
    seen = {}
    for name, r in res.items():
        m = re.search(r"step3d_batchedILi(\d)ELb(\d)ELi(\d)ELi4ELi(\d)E", name)
        if m:
            seen[tuple(int(x) for x in m.groups())] = r
    assert not want - set(seen), want - set(seen)
    bad = {k: seen[k] for k in want if seen[k]["vgpr"] > 128 or seen[k]["occupancy"] < 4}
    assert not bad, bad
