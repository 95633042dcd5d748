"""The patch kernels (the launches of a context whose shape nobody set, on
grids whose strips cannot fill the device) against the one-step strip kernels:
bit for bit, in every shape the rule chooses between and for every remainder
of a step count, on sizes at and off the patches' edges."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2203_05230_amd import closure as driver  # noqa: E402
from paper_2203_05230_amd import lbac, workloads as W  # noqa: E402


@pytest.fixture(autouse=True)
def the_library(gpu_lib):
    """Every test here needs the GPU and the built library (gpu_lib also opens
    the device through torch first, which finds none once another HIP runtime has)."""


def say(*a):
    print(*a, flush=True)


def sims(nx, ny, precision, model="improved", closure=False, vel="vortex"):
    case = dict(nx=nx, ny=ny, eps=0.8, tau=0.7, vel=vel, U=0.03, period_T=37.0, ux=0.04, uy=-0.03, precision=precision,
                model=model)
    rng = np.random.default_rng(nx * 1000 + ny)
    phi0 = W.circle(nx, 0.8, R_frac=0.3, yc_frac=0.5, ny=ny) * (1.0 - 1e-3 * rng.random((ny, nx)))
    out = []
    for _ in range(2):
        s = lbac.Simulation(case, phi0)
        if closure:
            s.set_closure(driver.init_weights(5, out_scale=0.05), 0.02)
        out.append(s)
    out[1].set_launch(64, 8, 0)  # one-step strips
    return out


def check(a, b, steps):
    for n in steps:
        a.step(n)
        b.step(n)
        assert a.time() == b.time()
        assert np.array_equal(a.phi(), b.phi()), n
    a.close()
    b.close()


# FP32 patches from 8x8 to 48x16, FP64 from 4x4 to 24x16, 16-bit storage from
# 12x12 to 60x28; sizes on the patches' edges, one off them, smaller than a grown
# patch, and degenerate
@pytest.mark.parametrize("nx,ny", [(1, 1), (1, 70), (33, 1), (5, 3), (31, 32), (64, 64), (129, 127), (200, 203), (256, 256),
                                   (303, 290), (384, 385), (512, 500), (1040, 1000)])
@pytest.mark.parametrize("precision", ["f32", "f64", "f32_f16store", "f32_bf16store"])
def test_patches_equal_strips(nx, ny, precision):
    say("case: patches", nx, ny, precision)
    a, b = sims(nx, ny, precision)
    check(a, b, (1, 2, 3, 4, 5, 13))


@pytest.mark.parametrize("precision", ["f32", "f64", "f32_f16store"])
def test_patches_equal_strips_conventional_model(precision):
    say("case: patches, conventional model", precision)
    for nx, ny in ((70, 61), (530, 410)):
        a, b = sims(nx, ny, precision, model="conventional", vel="uniform")
        check(a, b, (3, 14))


# closure patches from 8x8 to 52x20
@pytest.mark.parametrize("nx,ny", [(9, 7), (96, 101), (200, 190), (400, 420), (1000, 700)])
def test_patches_equal_strips_with_the_closure(nx, ny):
    say("case: patches with the closure", nx, ny)
    a, b = sims(nx, ny, "f32", closure=True)
    check(a, b, (1, 2, 3, 9))


@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_long_runs_and_graphs(precision):
    """Runs past the table of time factors (256 steps), in pieces, from graphs, and after a restored state."""
    say("case: patches, long runs", precision)
    a, b = sims(75, 66, precision)
    a.step(700)
    for n in (255, 1, 256, 188):
        b.step(n)
    assert np.array_equal(a.phi(), b.phi())
    blob = a.get_state()
    a.set_graph_chunk(300)
    b.set_state(blob)
    a.step(650)
    b.step(650)
    assert a.time() == b.time() == 1350 and np.array_equal(a.phi(), b.phi())
    a.close()
    b.close()


def test_autotune_keeps_the_faster_and_the_state():
    say("case: autotune on a small grid")
    a, b = sims(96, 96, "f32")
    a.step(7)
    b.step(7)
    us = a.autotune(3)
    assert us > 0 and a.time() == 7
    a.step(20)
    b.step(20)
    assert np.array_equal(a.phi(), b.phi())
    bx, strip, variant = a.get_launch()
    a.set_launch(bx, strip, variant)  # a reported shape can be set
    a.step(5)
    b.step(5)
    assert np.array_equal(a.phi(), b.phi())
    a.close()
    b.close()


# the two-pass launches (strips that mark, then the marked patches): grids
# whose last patch is one to a few nodes wide or high, a disk across the
# periodic edges, strips of one row, up and down
@pytest.mark.parametrize("nx,ny", [(145, 97), (147, 98), (160, 100), (33, 25), (1, 40), (300, 13), (17, 300)])
@pytest.mark.parametrize("launch", [(224, 40, 4), (64, 6, 4), (128, 32, 3), (96, 8, 3)])
def test_two_pass_closure_equals_one_step(nx, ny, launch):
    say("case: two-pass closure", nx, ny, launch)
    case = dict(nx=nx, ny=ny, eps=0.8, tau=0.7, vel="uniform", ux=0.05, uy=-0.04, precision="f32")
    phi0 = W.circle(nx, 0.8, R_frac=0.3, xc_frac=0.0, yc_frac=1.0, ny=ny)
    phi0 = np.maximum(phi0, np.roll(phi0, (ny // 2, nx // 2), (0, 1)))
    out = []
    for shape in (launch, (64, 8, 0)):
        s = lbac.Simulation(case, phi0)
        s.set_closure(driver.init_weights(5, out_scale=0.05), 0.02)
        s.set_launch(*shape)
        s.step(launch[2] - 1)
        a = s.phi()
        s.step(6 * (launch[2] - 1))
        out.append((a, s.phi()))
        s.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


# the smaller patches of FP64 and of the closure, off the patches' edges
@pytest.mark.parametrize("precision,closure,nx,ny", [
    ("f64", False, 61, 63), ("f64", False, 101, 99), ("f64", False, 145, 151), ("f64", False, 199, 209),
    ("f64", False, 255, 253), ("f64", False, 301, 299), ("f32", True, 127, 121), ("f32", True, 201, 197),
    ("f32", True, 255, 249), ("f32", True, 299, 301), ("f32", True, 601, 590)])
def test_small_patches_equal_strips(precision, closure, nx, ny):
    say("case: small patches", precision, closure, nx, ny)
    a, b = sims(nx, ny, precision, closure=closure)
    check(a, b, (3, 2, 1, 11))


@pytest.mark.parametrize("nx,ny", [(120, 90), (1700, 1300)])
def test_default_launches_with_the_closure_at_theta_zero(nx, ny):
    """theta = 0 puts nearly every node in the band: patches on a small grid,
    one-step launches on a large one."""
    say("case: closure at theta 0", nx, ny)
    a, b = sims(nx, ny, "f32")
    for s in (a, b):
        s.set_closure(driver.init_weights(5, out_scale=0.05), 0.0)
    check(a, b, (4, 7))


@pytest.mark.parametrize("precision,model", [("f32", "improved"), ("f64", "improved"), ("f64", "conventional")])
@pytest.mark.parametrize("nx,ny", [(399, 401), (770, 765), (1000, 1021)])
def test_middle_patches_equal_strips(nx, ny, precision, model):
    """FP32 patches of 48 x 16 and FP64 ones of 24 x 16, off their edges."""
    say("case: middle patches", precision, model, nx, ny)
    a, b = sims(nx, ny, precision, model=model)
    check(a, b, (4, 1, 6))


@pytest.mark.parametrize("model", ["improved", "conventional"])
def test_fp64_default_launches_on_large_grids(model):
    """Single steps take strips of a height chosen by the grid, longer runs
    patches, beyond 2048 nodes a side and off the tiles' and patches' edges;
    on a wide, low grid the strips are as high as the grid."""
    for nx, ny, steps in ((2050, 2049, (1, 2, 3, 5)), (16500, 17, (1, 1, 4))):
        say("case: FP64 default launches", model, nx, ny)
        a, b = sims(nx, ny, "f64", model=model)
        check(a, b, steps)


@pytest.mark.parametrize("theta", [5e-8, 1e-9, 1e-4])
@pytest.mark.parametrize("launch", [None, (224, 40, 4), (96, 8, 3)])
def test_two_pass_closure_at_small_theta(theta, launch):
    """The band test of the marking strips at thetas near the rounding of phi:
    a disk whose tails pass through them (and whose inside does, but for what
    rounds to 1), small enough for two-pass launches on its grid."""
    say("case: two-pass closure, theta", theta, launch)
    nx, ny = 1501, 1203
    case = dict(nx=nx, ny=ny, eps=0.8, tau=0.7, vel="vortex", U=0.03, period_T=37.0, precision="f32")
    phi0 = W.circle(nx, 0.8, R_frac=0.12, yc_frac=0.5, ny=ny)
    a, b = out = [lbac.Simulation(case, phi0) for _ in range(2)]
    for s in out:
        s.set_closure(driver.init_weights(5, out_scale=0.05), theta)
    if launch:
        a.set_launch(*launch)
    b.set_launch(64, 8, 0)
    assert a.steps_per_launch() == (3 if launch is None else launch[2] - 1)
    check(a, b, (3, 7))


def drops(nx, ny):
    y, x = np.mgrid[0:ny, 0:nx]
    return 0.5 + 0.5 * np.tanh(10.0 * np.sin(2 * np.pi * x / 64.0) * np.sin(2 * np.pi * y / 64.0))


@pytest.mark.parametrize("launch", [None, (224, 40, 4), (160, 8, 3)])
def test_closure_with_a_wide_band(launch):
    """Where most of a large grid is in the band, launches that would take two
    passes take patches of one step instead, from the first one on, and two
    passes again once the band is thin; the launches in graphs follow.  All of
    it the same bits as one-step strips."""
    say("case: closure, wide band", launch)
    nx, ny = 1501, 1203
    case = dict(nx=nx, ny=ny, eps=0.8, tau=0.7, vel="vortex", U=0.03, period_T=37.0, precision="f32")
    thin = W.circle(nx, 0.8, R_frac=0.3, yc_frac=0.5, ny=ny)
    out = []
    for shape in (launch, (64, 8, 0)):
        s = lbac.Simulation(case, drops(nx, ny))
        s.set_closure(driver.init_weights(5, out_scale=0.05), 0.02)
        if shape:
            s.set_launch(*shape)
        out.append(s)
    a, b = out
    if launch is None:
        assert a.steps_per_launch() == 1
    t = lbac.Simulation(case, thin)
    state = t.get_state()
    t.close()
    for graph in (0, 60):
        a.set_graph_chunk(graph)
        for n in (7, 300, 5):  # past a look at the band
            a.step(n)
            b.step(n)
            assert np.array_equal(a.phi(), b.phi()), (graph, n)
        for s in out:
            s.set_state(state)
        if launch is None:
            assert a.steps_per_launch() == 3
        for n in (7, 60):
            a.step(n)
            b.step(n)
            assert np.array_equal(a.phi(), b.phi()), (graph, n)
        wide = lbac.Simulation(case, drops(nx, ny))
        blob = wide.get_state()
        wide.close()
        for s in out:
            s.set_state(blob)
    a.close()
    b.close()
