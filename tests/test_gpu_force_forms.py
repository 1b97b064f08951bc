"""The staged force pass's forms (one sweep, two sweeps, pipelined) against the
unstaged kernel, which the parity tests compare with the oracle: the same
arithmetic in the same order, so bitwise, at tiles whose edges fall inside
and on waves, with a ragged last tile, more neighbours than the packed slots or
the pipelined form hold, failed particles, contact between two specimens, and
a specimen that run control has stopped."""
import numpy as np
import pytest

from paper_1901_07374_amd import inputs as I

pytestmark = pytest.mark.gpu

KEYS = ("force", "v", "u", "F", "Q", "sig", "D")
# LDS bytes per slot of each form (FP64, mixed)
BYTES = {"one": (208, 128), "two": (148, None), "pipe": (232, 168)}


@pytest.fixture(scope="module")
def tl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1901_07374_amd import tlsph
    return tlsph


def wide(dx):
    """Support of 1.8 dx: 26 neighbours, more than the packed slots hold."""
    return I.notched_bar(dx=dx, h=1.8 * dx)


PROBLEMS = {
    "bar": lambda: I.notched_bar(dx=0.27e-3),
    "bar_large": lambda: I.notched_bar(dx=0.2e-3),
    "wide": lambda: wide(0.5e-3),
    "wide_large": lambda: wide(0.27e-3),
    "contact_av": lambda: I.with_materials(I.bar_collision(dx=0.13e-3, gap=0.0), **I.DAMPING),
    "stopped": lambda: I.bar_batch(n_spec=3, counts=(70000, 50000, 60000)),
}
# problem, precision, lanes, tile, the form it takes
CASES = [
    ("bar", "fp64", 2, 163, "pipe"), ("bar", "fp64", 2, 192, "pipe"), ("bar", "fp64", 2, 195, "pipe"),
    ("bar", "fp64", 2, 66, "two"), ("bar", "fp64", 4, 65, "two"), ("bar", "fp64", 1, 66, "two"),
    ("bar", "fp64", 2, 96, "one"), ("bar", "fp64", 1, 100, "one"),
    ("bar_large", "mixed", 2, 128, "pipe"), ("bar_large", "mixed", 2, 227, "pipe"),
    ("bar_large", "mixed", 2, 195, "one"),
    ("bar", "mixed", 2, 100, "one"), ("bar", "mixed", 4, 100, "one"),
    ("wide", "fp64", 2, 66, "one"), ("wide", "mixed", 2, 66, "one"),
    ("wide_large", "fp64", 2, 67, "two"), ("wide_large", "fp64", 4, 64, "two"),
    ("contact_av", "fp64", 2, 192, "pipe"), ("stopped", "fp64", 2, 193, "pipe"),
]


@pytest.mark.parametrize("problem,precision,lanes,tile,form", CASES)
def test_forms_are_bitwise_the_unstaged_pass(tl, problem, precision, lanes, tile, form):
    p = PROBLEMS[problem]()
    st = I.random_state(p, seed=11, v_scale=1.0, u_scale=1e-7)
    outs = []
    for shape in ((False, 4, 256, 256, 0), (True, lanes, 256, 256, tile)):
        g = tl.Sim(p, precision=tl.FP64 if precision == "fp64" else tl.MIXED,
                   flags=tl.STORE_FORCE, k_cap=32)
        g.set_launch_shape(*shape)
        g.set_state(st)
        if problem == "stopped":
            g.set_run_control([{"group": 2 * q + 1, "axis": 2, "sign": -1.0, "drop": 0.5,
                                "min_peak": 1e12, "step_cap": 2 if q == 1 else 0}
                               for q in range(p.n_spec)])
            g.run(4, check_every=1)
            assert g.run_status()["steps"][1] == 2
        else:
            g.step(3)
        outs.append({k: g.get(k) for k in KEYS})
        inf = g.info()
    print(problem, precision, lanes, tile, p.n, inf, flush=True)
    assert inf["staged"] and inf["tile"] == tile and inf["lanes_per_particle"] == lanes
    per_slot = BYTES[form][precision == "mixed"]
    assert inf["lds_bytes"] % per_slot == 0 and inf["lds_bytes"] > tile * per_slot
    for k in KEYS:
        assert np.array_equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("precision,tile", [("fp64", 193), ("fp64", 208), ("mixed", 128)])
def test_groups_of_several_specimens_in_a_wave(tl, precision, tile):
    """Specimens whose ramps differ (time steps, time constants), and whose first
    particles are in groups, so that a wave of the pipelined pass holds lanes of
    two specimens with groups of both."""
    p = I.bar_batch(n_spec=3, counts=(90000, 70000, 80000))
    mats = [dict(m, dt=m["dt"] * f) for m, f in zip(p.materials, (1.0, 0.9, 0.8))]
    groups = [dict(g, tau=1e-3 * (1 + k)) for k, g in enumerate(p.bc_groups)]
    bc = p.bc_group.copy()
    for q in range(3):   # every third particle, alternating between the specimen's groups
        i = np.arange(p.spec_offsets[q], p.spec_offsets[q + 1], 3)
        bc[i] = 2 * q + (i % 2)
    p = I.Problem(p.name, p.X, p.V0, p.spec_offsets, mats, bc, groups, p.v_init, p.steps, p.dx)
    st = I.random_state(p, seed=13, v_scale=1.0, u_scale=1e-7)
    outs = []
    for shape in ((False, 4, 256, 256, 0), (True, 2, 256, 256, tile)):
        g = tl.Sim(p, precision=tl.FP64 if precision == "fp64" else tl.MIXED, k_cap=32)
        g.set_launch_shape(*shape)
        g.set_state(st)
        g.step(3)
        outs.append({k: g.get(k) for k in KEYS if k != "force"})
        inf = g.info()
    print(precision, tile, p.n, inf, flush=True)
    assert inf["lds_bytes"] % BYTES["pipe"][precision == "mixed"] == 0
    for k in outs[0]:
        assert np.array_equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("tile,form", [(80, "one"), (120, "two"), (128, "two"), (129, "pipe"),
                                       (144, "pipe")])
def test_form_at_the_rules_lines(tl, tile, form):
    """Two lanes, FP64: two workgroups of 80 share a CU in one sweep and in the
    pipelined form, whose image does not pay at that size; up to 128 particles two
    share it in two sweeps alone; above, one does in any form."""
    test_forms_are_bitwise_the_unstaged_pass(tl, "bar", "fp64", 2, tile, form)


def mild(scale):
    """Two zones of spacings 1 and 1.1: a graded bar whose tiles stay small."""
    return I.graded_notched_bar(R=2e-3, L=10e-3, rho=1e-3, bounds=(2e-3,),
                                spacings=(scale * 0.2e-3, scale * 0.22e-3))


@pytest.mark.parametrize("lanes,tile,form", [(1, 64, "two"), (1, 128, "two"), (2, 128, "two"),
                                             (2, 112, "two"), (4, 64, "two"), (4, 112, "two"),
                                             (2, 64, "one"), (4, 80, "one")])
def test_graded_forms_are_bitwise_the_unstaged_pass(tl, lanes, tile, form):
    """Each pair's own support: its radii's plane in the image, the constant
    factor in what the first sweep keeps, more neighbours than the packed slots."""
    p = mild(0.521)
    st = I.random_state(p, seed=17, v_scale=1.0, u_scale=1e-7)
    outs = []
    for shape in ((False, 4, 256, 256, 0), (True, lanes, 256, 256, tile)):
        g = tl.Sim(p, flags=tl.STORE_FORCE, k_cap=64)
        g.set_launch_shape(*shape)
        g.set_state(st)
        g.step(3)
        outs.append({k: g.get(k) for k in KEYS})
        inf = g.info()
    print(lanes, tile, p.n, inf, flush=True)
    per_slot = BYTES[form][0] + 8
    assert inf["lds_bytes"] % per_slot == 0 and inf["lds_bytes"] > tile * per_slot
    for k in KEYS:
        assert np.array_equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("problem,precision,tile", [
    ("bar", "fp64", 163), ("bar", "fp64", 195), ("bar_large", "mixed", 128),
    ("bar_large", "mixed", 227), ("contact_av", "fp64", 192), ("stopped", "fp64", 193)])
def test_pipelined_pass_without_stored_forces(tl, problem, precision, tile):
    """The finish's two stores are then the wave's last, which its wait for the
    next tile's copies counts on exactly (with forces stored it waits for more)."""
    p = PROBLEMS[problem]()
    st = I.random_state(p, seed=19, v_scale=1.0, u_scale=1e-7)
    outs = []
    for shape in ((False, 4, 256, 256, 0), (True, 2, 256, 256, tile)):
        g = tl.Sim(p, precision=tl.FP64 if precision == "fp64" else tl.MIXED, k_cap=32)
        g.set_launch_shape(*shape)
        g.set_state(st)
        if problem == "stopped":
            g.set_run_control([{"step_cap": 2 if q == 1 else 0} for q in range(p.n_spec)])
            g.run(6, check_every=1)
        else:
            g.step(6)
        outs.append({k: g.get(k) for k in KEYS if k != "force"})
        inf = g.info()
    print(problem, precision, tile, p.n, inf, flush=True)
    assert inf["lds_bytes"] % BYTES["pipe"][precision == "mixed"] == 0
    for k in outs[0]:
        assert np.array_equal(outs[0][k], outs[1][k]), k


def test_kernel_names(tl):
    """The context names the kernels it launches."""
    g = tl.Sim(PROBLEMS["bar"]())
    for shape, force, deform in (
            ((False, 4, 128, 256, 0), "k_pass_b", "k_pass_a"),
            ((True, 2, 256, 0, 80), "k_pass_b_one", "k_pass_a_staged"),
            ((True, 2, 256, -64, 128), "k_pass_b_wide", "k_pass_a_staged"),
            ((True, 4, 256, 64, 64), "k_pass_b_staged", "k_pass_a"),
            ((True, 2, 256, 256, 192), "k_pass_b_staged", "k_pass_a")):
        g.set_launch_shape(*shape)
        assert g.kernel_names() == {"force_pass": force, "deformation_pass": deform}, shape
    g = tl.Sim(PROBLEMS["bar_large"](), precision=tl.MIXED)
    g.set_launch_shape(True, 2, 256, 0, 128)
    assert g.kernel_names()["deformation_pass"] == "k_pass_a_staged"   # (below 450k particles)
