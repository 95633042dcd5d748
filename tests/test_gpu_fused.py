"""The multi-step variants (LBAC_KERNEL_FUSED2 / _FUSED3): one launch takes S =
2 or 3 steps with the populations between them kept in LDS.  Each of the S
stages does the one-step kernels' arithmetic on every node, so they must agree
with them bit for bit, for every grid, launch shape, step count and graph
chunking; and with the FP64 oracle to the FP32 bound."""
import sys

import numpy as np
import pytest

from oracle import lib as O
from paper_2203_05230_amd import workloads as W

pytestmark = pytest.mark.gpu

FUSED2, FUSED3 = 3, 4
VARIANTS = [FUSED2, FUSED3]


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def full_widths(variant):
    """Tile widths of the multi-step kernels that are not multiples of 64: the
    last wavefront then holds tile columns besides the halo."""
    return [96, 160, 224, 288]


def run(lb, case, phi0, steps, launch, graph=0, chunks=None):
    sim = lb.Simulation({**case, "precision": "f32"}, phi0)
    sim.set_launch(*launch)
    if graph:
        sim.set_graph_chunk(graph)
    for n in (chunks or [steps]):
        sim.step(n)
    return sim


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("model", ["improved", "conventional"])
def test_bitwise_equal_to_one_step_kernels(gpu_lib, model, variant):
    say("case: multi-step variant", variant, "vs block variant,", model)
    case = {**W.single_vortex_case(320, U=0.05, period_T=100.0), "model": model}
    phi0 = W.circle(320, 1.0)
    base = run(gpu_lib, case, phi0, 13, (256, 64, 0)).phi()
    fw = full_widths(variant)
    for bx, strip in ((256, 64), (64, 5), (128, 320), (256, 1), (64, 17), (128, 2), (256, 3), (192, 40), (320, 7),
                      (192, 1), (320, 320), (fw[1], 9), (fw[2], 64), (fw[3], 1), (fw[2], 320), (fw[2], 2), (fw[0], 11),
                      (240, 9), (240, 320)):
        phi = run(gpu_lib, case, phi0, 13, (bx, strip, variant)).phi()
        assert np.array_equal(phi, base), (bx, strip, variant)


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("nx,ny", [(100, 37), (65, 130), (1, 64), (64, 1), (3, 5), (300, 70), (257, 9)])
def test_ragged_and_degenerate_grids(gpu_lib, nx, ny, variant):
    say("case: multi-step variant", variant, "ragged grid", nx, ny)
    case = dict(nx=nx, ny=ny, eps=1.0, tau=0.8, delta=1e-10, vel="uniform", ux=0.03, uy=-0.02)
    rng = np.random.default_rng(nx * 1000 + ny)
    phi0 = W.circle(max(nx, ny), 1.5, R_frac=0.3, yc_frac=0.5)[:ny, :nx] * 0.9 + 0.05 * rng.random((ny, nx))
    base = run(gpu_lib, case, phi0, 11, (64, 7, 0)).phi()
    fw = full_widths(variant)
    for bx, strip in ((64, 7), (128, 4), (256, 1), (64, 64), (256, 2), (192, 3), (320, 5), (fw[2], 4), (fw[1], 13),
                      (fw[3], 2), (fw[0], 6), (240, 5)):
        phi = run(gpu_lib, case, phi0, 11, (bx, strip, variant)).phi()
        assert np.array_equal(phi, base), (bx, strip, variant)


@pytest.mark.parametrize("variant", VARIANTS)
def test_step_counts_and_graph_chunks(gpu_lib, variant):
    """Counts that are not multiples of S end with one-step launches; graph
    chunks may hold an odd number of launches, so the buffers swap parity
    across replays."""
    say("case: multi-step variant", variant, "step counts and graph replay")
    import torch

    case = W.single_vortex_case(96, U=0.05, period_T=100.0)
    phi0 = W.circle(96, 1.0)
    chunks = [1, 2, 3, 8, 5, 6, 12, 7, 1]
    ref = gpu_lib.Simulation({**case, "precision": "f32"}, phi0)
    ref.set_launch(128, 16, 0)
    fw = full_widths(variant)
    sims = [run(gpu_lib, case, phi0, 0, (bx, 16, variant), graph=g, chunks=[0])
            for g, bx in ((0, 128), (6, 128), (8, fw[2]), (4, fw[1]))]
    for n in chunks:
        ref.step(n)
        for s in sims:
            s.step(n)
        x = torch.ones(1000, device="cuda").sum()  # unrelated eager work between replays
        torch.cuda.synchronize()
        assert float(x) == 1000.0
        want = ref.phi()
        for s, g in zip(sims, (0, 6, 8, 4)):
            assert np.array_equal(s.phi(), want), (n, g)
    assert ref.time() == sum(chunks) and all(s.time() == sum(chunks) for s in sims)
    m = [s.mass() for s in sims]
    assert all(v == ref.mass() for v in m)


@pytest.mark.parametrize("variant", VARIANTS)
def test_fp32_parity_with_oracle(gpu_lib, variant):
    say("case: multi-step variant", variant, "vs FP64 oracle, 128x128, 1001 steps")
    case = W.single_vortex_case(128, eps=1.0, U=0.02, period_T=2000.0)
    phi0 = W.circle(128, 1.0)
    p = O.Params(128, 128, eps=1.0, tau=0.8, delta=1e-10, vel_kind=O.VEL_VORTEX, U=0.02, period_T=2000.0)
    ref = O.run(p, phi0, 1001)
    sim = run(gpu_lib, case, phi0, 1001, (128, 32, variant))
    err = float(np.linalg.norm(sim.phi() - ref) / np.linalg.norm(ref))
    say("  rel L2 %.3e" % err)
    assert err <= 1e-5


@pytest.mark.parametrize("variant", VARIANTS)
def test_checkpoint_resume_in_the_middle(gpu_lib, variant):
    say("case: multi-step variant", variant, "checkpoint and resume")
    case = W.single_vortex_case(80, U=0.05, period_T=100.0)
    phi0 = W.circle(80, 1.0)
    a = run(gpu_lib, case, phi0, 9, (64, 8, variant))
    blob = a.get_state()
    a.step(10)
    b = gpu_lib.Simulation({**case, "precision": "f32"}, W.circle(80, 2.0))
    b.set_launch(64, 8, variant)
    b.set_state(blob)
    b.step(10)
    assert b.time() == a.time() == 19
    assert np.array_equal(a.phi(), b.phi())


@pytest.mark.parametrize("launch,n", [((128, 128, 4), 2047), ((128, 512, 4), 4097), ((64, 50, 3), 1001)])
def test_heights_that_round_to_another_strip_count(gpu_lib, launch, n):
    """Strip heights whose nearest whole period would add a strip the next one
    above does not (17 strips of 126 rows against 16 of 132), on grids whose
    tiles do not all run at once; 50 rows, 20 strips of 52, stay the nearest."""
    case = {**W.single_vortex_case(n, eps=1.0, U=0.04, period_T=200.0), "precision": "f32"}
    phi0 = W.circle(n, 1.0)
    a, b = [gpu_lib.Simulation(case, phi0) for _ in range(2)]
    a.set_launch(*launch)
    b.set_launch(256, 64, 0)
    for s in (a, b):
        s.step(7)
    assert np.array_equal(a.phi(), b.phi())
    a.close()
    b.close()


def test_needs_fp32_collision(gpu_lib):
    case = W.single_vortex_case(32)
    sim = gpu_lib.Simulation({**case, "precision": "f64"}, W.circle(32, 1.0))
    for variant in VARIANTS:
        with pytest.raises(gpu_lib.LbacError):
            sim.set_launch(128, 16, variant)
    with pytest.raises(gpu_lib.LbacError):
        sim.set_launch(128, 16, 5)
    sim.close()


# ---- shifted 16-bit storage with the multi-step kernel ------------------------
# The populations pass through 16 bits at the launch's load and store only; the
# S - 1 steps in between keep them in FP32 in LDS.  So the result depends on S
# (how often the storage rounds) but on nothing else: every tile shape and
# strip height of one variant gives the same bits.

def run16(lb, prec, case, phi0, steps, launch):
    sim = lb.Simulation({**case, "precision": prec}, phi0)
    sim.set_launch(*launch)
    sim.step(steps)
    return sim


@pytest.mark.parametrize("prec", ["f32_f16store", "f32_bf16store"])
@pytest.mark.parametrize("variant", VARIANTS)
def test_shifted_storage_bitwise_over_launch_shapes(gpu_lib, prec, variant):
    say("case: multi-step variant", variant, prec, "over launch shapes")
    case = W.single_vortex_case(320, U=0.05, period_T=100.0)
    phi0 = W.circle(320, 1.0)
    base = run16(gpu_lib, prec, case, phi0, 12, (224, 40, variant)).phi()
    for bx, strip in ((256, 64), (64, 5), (128, 320), (96, 1), (160, 9), (320, 7), (192, 3), (240, 11), (240, 1)):
        phi = run16(gpu_lib, prec, case, phi0, 12, (bx, strip, variant)).phi()
        assert np.array_equal(phi, base), (bx, strip)


@pytest.mark.parametrize("prec,tol10", [("f32_f16store", 3e-4), ("f32_bf16store", 3e-3)])
def test_shifted_storage_short_run_against_oracle(gpu_lib, prec, tol10):
    """The bounds of the one-step 16-bit kernels (test_gpu_parity): nine steps
    as three launches of three, plus one one-step launch."""
    say("case: 10 steps", prec, "three-step kernel")
    case = W.single_vortex_case(128, eps=1.0, U=0.05, period_T=200.0)
    phi0 = W.circle(128, 1.0)
    ref = O.run(O.Params(128, 128, eps=1.0, tau=0.8, delta=1e-10, vel_kind=O.VEL_VORTEX, U=0.05, period_T=200.0),
                phi0, 10)
    sim = run16(gpu_lib, prec, case, phi0, 10, (224, 16, FUSED3))
    assert float(np.linalg.norm(sim.phi() - ref) / np.linalg.norm(ref)) <= tol10


@pytest.mark.parametrize("prec", ["f32_f16store", "f32_bf16store"])
def test_shifted_storage_mass_and_bytes(gpu_lib, prec):
    """Mass drift over 999 steps (333 launches) within the bound of the
    one-step 16-bit kernels; 40 bytes per node per launch (8 16-bit planes and
    the FP32 phi* plane, read and written once)."""
    say("case: mass", prec, "three-step kernel")
    case = W.single_vortex_case(256, eps=1.0, period_T=2048.0)
    sim = gpu_lib.Simulation({**case, "precision": prec}, W.circle(256, 1.0))
    sim.set_launch(224, 40, FUSED3)
    assert sim.steps_per_launch() == 3 and sim.bytes_per_node() == 40.0
    m0 = sim.mass()
    sim.step(999)
    assert abs(sim.mass() - m0) / m0 <= 1e-6
    sim.close()


@pytest.mark.parametrize("prec", ["f32_f16store", "f32_bf16store"])
def test_shifted_storage_reflection_symmetry(gpu_lib, prec):
    """The mirrored frame of downward strips with 16-bit planes: the run from
    the mirrored field is the mirror image bit for bit."""
    say("case: reflection symmetry,", prec, "three-step kernel")
    nx, ny = 150, 97
    rng = np.random.default_rng(7)
    phi0 = W.circle(160, 1.5, R_frac=0.25, yc_frac=0.4)[:ny, :nx] * 0.9 + 0.05 * rng.random((ny, nx))
    case = dict(nx=nx, ny=ny, eps=1.0, tau=0.7, delta=1e-10, vel="uniform", ux=0.03, uy=0.021)
    a = run16(gpu_lib, prec, case, phi0, 15, (224, 12, FUSED3))
    b = run16(gpu_lib, prec, {**case, "uy": -0.021}, np.ascontiguousarray(phi0[::-1]), 15, (224, 12, FUSED3))
    assert np.array_equal(b.phi(), a.phi()[::-1])


def test_tile_widths_of_the_multi_step_kernels_only(gpu_lib):
    """Tiles of 96, 160, 192, 224, 240, 288 and 320 columns exist for the
    multi-step kernels only; the one-step launches such a
    context makes (a remainder, or with the closure on) use 256-column tiles,
    bit for bit the same."""
    case = W.single_vortex_case(200, U=0.05, period_T=100.0)
    phi0 = W.circle(200, 1.0)
    sim = gpu_lib.Simulation({**case, "precision": "f32"}, phi0)
    for variant in (0, 1, 2):
        for bx in [192, 240, 320] + full_widths(FUSED3):
            with pytest.raises(gpu_lib.LbacError):
                sim.set_launch(bx, 16, variant)
    for variant in VARIANTS:
        for bx in (32, 80, 244, 248, 352):
            with pytest.raises(gpu_lib.LbacError):
                sim.set_launch(bx, 16, variant)
    sim.close()
    base = run(gpu_lib, case, phi0, 7, (256, 16, 0)).phi()
    for variant in VARIANTS:
        for bx in [192, 240, 320] + full_widths(variant):
            assert np.array_equal(run(gpu_lib, case, phi0, 7, (bx, 16, variant)).phi(), base), (bx, variant)


@pytest.mark.parametrize("variant,steps", [(FUSED2, 2), (FUSED3, 3), (0, 1)])
def test_steps_per_launch(gpu_lib, variant, steps):
    case = W.single_vortex_case(32)
    sim = gpu_lib.Simulation({**case, "precision": "f32"}, W.circle(32, 1.0))
    sim.set_launch(64, 8, variant)
    assert sim.steps_per_launch() == steps
    assert sim.bytes_per_node() == 72.0
    sim.close()


@pytest.mark.parametrize("prec,launches", [
    ("f32", [(256, 16, 0), (128, 5, 1), (256, 9, 2), (224, 12, FUSED3), (160, 7, FUSED3), (192, 20, FUSED2)]),
    ("f64", [(256, 16, 0), (64, 6, 2)]),
])
def test_reflection_symmetry_is_exact(gpu_lib, prec, launches):
    """D2Q9 with a uniform velocity is symmetric under y -> -y with v -> -v.
    The node arithmetic rounds mirror-symmetrically (the multi-step kernels
    compute downward strips in the mirrored frame and rely on it), so the run
    from the mirrored field with the mirrored velocity is the mirror image of
    the original bit for bit, for every kernel variant and launch shape."""
    say("case: reflection symmetry,", prec)
    nx, ny = 150, 97
    rng = np.random.default_rng(7)
    phi0 = W.circle(160, 1.5, R_frac=0.25, yc_frac=0.4)[:ny, :nx] * 0.9 + 0.05 * rng.random((ny, nx))
    case = dict(nx=nx, ny=ny, eps=1.0, tau=0.7, delta=1e-10, vel="uniform", ux=0.03, uy=0.021, precision=prec)
    mirrored = {**case, "uy": -0.021}
    for launch in launches:
        a = gpu_lib.Simulation(case, phi0)
        b = gpu_lib.Simulation(mirrored, np.ascontiguousarray(phi0[::-1]))
        for s in (a, b):
            s.set_launch(*launch)
            s.step(14)
        pa, pb = a.phi(), b.phi()
        a.close()
        b.close()
        assert np.array_equal(pb, pa[::-1]), launch
