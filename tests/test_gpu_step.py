"""Batched steps in one kernel (chains of at most 256 beads): the chain's
workgroup collides the nodes set aside for it, the tiles all others.  Bits
equal those of the form that re-collides the chain's nodes after the collide
(launch mode 2); a single box also matches the FP64 oracle."""
from __future__ import annotations

import numpy as np
import pytest

from lbtest import chain, gpu_system, initial_pops, max_rel_pop_err, oracle_state, params, say

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0903_5067_amd as lbm
    lbm.lib()


def _run(boxes, xs, prec, overlap, graph, calls):
    s = gpu_system(boxes, prec, xs=xs)
    s.set_launch(batched=True, graph_steps=graph, overlap=overlap)
    for n in calls:
        s.step(n)
    assert all(o["health"] == 0 for o in s.observables())
    out = s.export_state()["boxes"]
    s.close()
    return out


def _equal(a, b):
    for i, (p, q) in enumerate(zip(a, b)):
        for k in ("n", "x", "v", "f", "fc"):
            assert np.array_equal(p[k], q[k]), (i, k)


# one bead; both sides of 16, 32 and 64 beads (lanes per bead, threads per
# workgroup), 128 / 129 and the longest chain; a box that one stencil wraps
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("L,N", [(2, 1), (4, 16), (7, 17), (16, 32), (16, 33), (24, 64), (24, 65), (32, 128),
                                 (32, 129), (32, 256)])
def test_one_kernel_step_matches_fixup_form_and_oracle(orc, L, N, prec):
    say("one-kernel step", L, N, prec)
    p = params(L=L, N=N, kT=1e-2, omega_s=1.2, omega_b=0.8, omega_g=1.4, seed=21, box_id=3)
    x = chain(p)
    got = _run([p], [x], prec, True, 0, (5, 3))
    _equal(got, _run([p], [x], prec, False, 0, (8,)))
    o = oracle_state(orc, p, initial_pops(orc, p), x)
    o.run(8)
    if prec == FP64:
        assert np.max(np.abs(got[0]["n"] - o.n)) < 1e-12
        assert np.max(np.abs(got[0]["x"] - o.x)) < 1e-10
    else:
        assert max_rel_pop_err(got[0]["n"], o.n, orc) < 1e-5


def _left_set_aside(p, x0, v0, x1):
    """Beads whose end position's stencil reaches past the nodes that may be
    set aside from (x0, v0): the start's stencil, one node wider on a side
    closer than twice the ballistic path plus four thermal ones."""
    m = np.minimum(2 * np.abs(v0) * p["tau_lb"] + 4 * np.sqrt(p["kT"] / p["mass"]) * p["tau_lb"], 0.5)
    i, fr = np.floor(x0), x0 - np.floor(x0)
    lo, hi = i - (fr < m), i + 1 + (fr > 1 - m)
    return (np.floor(x1) < lo).any(1) | (np.floor(x1) + 1 > hi).any(1)


@pytest.mark.parametrize("prec,graph", [(FP64, 0), (FP32, 0), (FP64, 4), (FP32, 4)])
def test_beads_that_leave_their_set_aside_nodes(prec, graph):
    """A chain at rest, shrunk by 7 %, flies apart within its
    first steps: its impulses land on nodes the tiles have collided, which
    the next step's start (or the run's end) re-collides.  A quiet box and one
    without a chain in the batch; runs of 1, 4 and 7 steps."""
    say("left set-aside nodes", prec, graph)
    boxes = [params(L=16, N=16, kT=0.0, therm=0, seed=5, box_id=0),
             params(L=12, N=0, kT=1e-2, seed=5, box_id=1),
             params(L=24, N=60, kT=1e-2, seed=5, box_id=2)]
    xs = [chain(b) for b in boxes]
    xs[0] = xs[0][0] + 0.93 * (xs[0] - xs[0][0])
    ref = gpu_system(boxes, prec, xs=xs)
    ref.set_launch(batched=True, overlap=False)
    left = 0
    for _ in range(4):
        a = ref.export_state()["boxes"][0]
        ref.step(1)
        left += int(_left_set_aside(boxes[0], a["x"], a["v"], ref.export_state()["boxes"][0]["x"]).sum())
    ref.close()
    assert left > 0
    want = _run(boxes, xs, prec, False, 0, (12,))
    _equal(_run(boxes, xs, prec, True, graph, (1, 4, 7)), want)


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_many_tiles_and_wide_workgroups(prec):
    """The launch shapes by batch: more tiles than the small-batch shape takes
    (256-thread workgroups), and a long chain in a batch of short ones."""
    say("step launch shapes", prec)
    many = [params(L=104, N=48, kT=1e-2, seed=8, box_id=0), params(L=10, N=10, kT=1e-2, seed=8, box_id=1)]
    mixed = [params(L=20, N=200, kT=1e-2, seed=8, box_id=0), params(L=10, N=10, kT=1e-2, seed=8, box_id=1),
             params(L=9, N=24, kT=1e-2, seed=8, box_id=2)]
    for boxes in (many, mixed):
        xs = [chain(b) for b in boxes]
        got = _run(boxes, xs, prec, True, 2, (5,))
        _equal(got, _run(boxes, xs, prec, False, 0, (5,)))
        _equal(got[1:2], _run(boxes[1:2], xs[1:2], prec, True, 0, (5,)))   # a box alone


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_checkpoint_of_uneven_boxes(prec):
    """Export and import through the staging buffer: boxes whose planes fit it
    in one piece, in several, and with a ragged last tile; the exported
    populations are the stored ones (rho0 not 1: w_i rho0 rounds), an import
    of them exports the same, a state given as one oversized list of arrays is
    refused, and a run goes on from an import as from the export."""
    import paper_0903_5067_amd as lbm
    say("checkpoint of uneven boxes", prec)
    boxes = [params(L=11, N=9, kT=1e-2, rho0=0.864, seed=4, box_id=0), params(L=2, N=0, kT=1e-2, seed=4, box_id=1),
             params(L=20, N=30, kT=1e-2, rho0=0.9, seed=4, box_id=2)]
    s = gpu_system(boxes, prec, xs=[chain(b) for b in boxes])
    s.step(5)
    a = s.export_state()
    obs = s.observables()
    for b, o, p in zip(a["boxes"], obs, boxes):
        assert abs(b["n"].sum() - o["mass"]) < 1e-9 * o["mass"]
    s.import_state(a)
    c = s.export_state()
    s.step(3)
    d = s.export_state()
    s.import_state(a)
    s.step(3)
    _equal(a["boxes"], c["boxes"])
    _equal(d["boxes"], s.export_state()["boxes"])
    with pytest.raises(lbm.LBError):
        s.import_state({"step": a["step"], "boxes": a["boxes"][:2]})
    s.close()


# 512 / 513 beads: both widths of the large-chain kernel; dense boxes (32 N >=
# L^3) of one node range, of several with a ragged end, and the largest; cell
# rows of the list build that pass a multiple of 16 cells (L = 40: 24 cells)
# and ones that do not; several chains in a box
@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("L,N,chain_len", [(13, 257, 0), (14, 512, 32), (20, 513, 0), (32, 1024, 64), (24, 512, 0),
                                           (40, 400, 0), (40, 700, 100)])
def test_large_chain_kernels_match_oracle(orc, L, N, chain_len, prec):
    say("large chain edges", L, N, chain_len, prec)
    p = params(L=L, N=N, chain_len=chain_len, kT=0.05, md_dt=0.005, tau_lb=0.05, seed=31, box_id=2)
    x = chain(p)
    got = _run([p], [x], prec, True, 0, (3, 2))
    o = oracle_state(orc, p, initial_pops(orc, p), x)
    o.run(5)
    if prec == FP64:
        assert np.max(np.abs(got[0]["n"] - o.n)) < 1e-12
        assert np.max(np.abs(got[0]["x"] - o.x)) < 1e-10
    else:
        assert max_rel_pop_err(got[0]["n"], o.n, orc) < 1e-5


@pytest.mark.parametrize("L,N,chain_len", [(8, 1, 0), (10, 17, 0), (14, 65, 13), (16, 129, 0)])
def test_adjoint_lane_layouts_match_oracle_tangent(orc, L, N, chain_len):
    """The reverse coupling kernel at the edges of its lanes per bead and
    threads per workgroup, against the oracle's exact tangent."""
    say("adjoint lane layouts", L, N, chain_len)
    p = params(L=L, N=N, chain_len=chain_len, kT=1e-3, omega_s=1.2, omega_b=0.9, seed=17, box_id=1)
    x0, n0 = chain(p), initial_pops(orc, p, amp=0.01, seed=11)
    s = gpu_system([p], FP64, xs=[x0], pops=[n0])
    vh = s.window_forward(6, 4)
    cw = np.random.default_rng(5).normal(size=vh.shape)
    grad = s.window_backward(cw)[0]
    ho, dh = oracle_state(orc, p, n0, x0).window_tangent(6)
    assert np.max(np.abs(vh - ho)) < 1e-10
    ref = np.einsum("tna,tnak->k", cw, dh)
    np.testing.assert_allclose(grad, ref, rtol=1e-7, atol=1e-7 * np.max(np.abs(ref)))
    s.close()


def test_runs_whose_collides_carry_the_node_tables():
    """A box large enough that its collide, not its large chain, sets the step
    time (136^3): FP32 runs put the node tables into the collides.  A hot
    chain's beads leave their tables within the steps; bits as with the
    re-collision after the collide, in one run and in two."""
    say("node tables in the collide")
    p = params(L=136, N=300, seed=7, box_id=0, kT=1.0, therm=0, md_dt=0.02, md_substeps=10, tau_lb=0.2, zeta=1.0,
               k_fene=7.0, r0_fene=2.0)
    x = chain(p)
    s = gpu_system([p], FP32, xs=[x])
    s.set_launch(batched=True, overlap=False)
    left = 0
    for _ in range(8):
        a = s.bead_positions()
        s.step(1)
        # a stencil outside the 3x3x3 nodes around the nearest node of the start
        left += int((np.abs(np.floor(s.bead_positions()) + 0.5 - np.floor(a + 0.5)) > 1.0).any(1).sum())
    want = s.export_state()["boxes"]
    s.close()
    assert left > 0
    _equal(_run([p], [x], FP32, True, 0, (8,)), want)
    _equal(_run([p], [x], FP32, True, 4, (5, 3)), want)


@pytest.mark.parametrize("substeps", [1, 4, 5, 6, 11])
def test_impulses_of_any_number_of_substeps(orc, substeps):
    """The impulses of a large chain are made from its substep records, five
    at a time: every remainder, against the oracle."""
    say("records of", substeps, "substeps")
    p = params(L=40, N=300, kT=1e-2, seed=9, md_dt=0.01, md_substeps=substeps, tau_lb=0.01 * substeps)
    x = chain(p)
    n0 = initial_pops(orc, p, amp=0.01, seed=3)
    s = gpu_system([p], FP64, xs=[x], pops=[n0])
    s.couple()
    o = oracle_state(orc, p, n0, x)
    dp = o.couple()
    assert np.abs(s.pending_impulse()[0] - dp).max() < 1e-13
    s.step(5)
    o.collide_stream(dp)
    o.run(4)
    st = s.export_state()["boxes"][0]
    s.close()
    assert max_rel_pop_err(st["n"], o.n, orc) < 1e-11


@pytest.mark.parametrize("L", [150, 163])
def test_observables_of_large_boxes(orc, L):
    """The sums of a box above 12000 tiles (one round of blocks, its records
    summed at once; two rounds, the records in ranges; the last block short)
    against the oracle's, on populations of which many are negative."""
    say("observables", L)
    p = params(L=L, N=0, kT=0.0, therm=0)
    n = initial_pops(orc, p, amp=1.5, seed=5)
    s = gpu_system([p], FP64, pops=[n])
    got = s.observables(allow_unhealthy=True)[0]
    s.close()
    want = oracle_state(orc, p, n, np.zeros((0, 3))).observables()
    assert got["neg"] == want[orc.OBS["neg"]]
    assert got["mass"] == pytest.approx(want[0], rel=1e-12)
    np.testing.assert_allclose(got["p_total"], want[10:13], atol=1e-7)   # 4e6 nodes of ~1, summed in FP64
    np.testing.assert_allclose(got["mode_sq"], want[19:38], rtol=1e-9, atol=1e-20)


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_packed_state_and_arrays_are_the_same(prec):
    """lb_export_state / lb_import_state (one buffer) against lb_export_arrays /
    lb_import_arrays, and what the array calls refuse."""
    import ctypes

    import paper_0903_5067_amd as lbm
    say("packed state", prec)
    boxes = [params(L=9, N=12, kT=1e-2, seed=6, box_id=0), params(L=4, N=0, kT=1e-2, seed=6, box_id=1)]
    s = gpu_system(boxes, prec, xs=[chain(b) for b in boxes])
    s.step(4)
    L, st = lbm.lib(), s.export_state()
    buf = np.empty(L.lb_state_host_bytes(s.h) // 8)
    assert L.lb_export_state(s.h, buf.ctypes.data_as(ctypes.c_void_p), buf.nbytes) == lbm.LB_OK
    arrs = [b[k] for b in st["boxes"] for k in ("n", "x", "v", "f", "fc")]
    assert int(buf[:1].view(np.uint64)[0]) == st["step"] == 4
    assert np.array_equal(buf[1:], np.concatenate([a.reshape(-1) for a in arrs]))
    s.import_state(st)   # FP64 deviations come back to the last bit of n_i: both runs go on from an import
    s.step(3)
    want = s.export_state()["boxes"]
    assert L.lb_import_state(s.h, buf.ctypes.data_as(ctypes.c_void_p), buf.nbytes) == lbm.LB_OK
    s.step(3)
    _equal(s.export_state()["boxes"], want)
    step, null = ctypes.c_uint64(), ctypes.c_void_p()
    ptrs = [a.ctypes.data for a in arrs]
    for bad in (ptrs[:5], [None] + ptrs[1:], ptrs[:2] + [None] + ptrs[3:]):
        p = (ctypes.c_void_p * len(bad))(*bad)
        assert L.lb_export_arrays(s.h, ctypes.byref(step), p, len(bad)) == lbm.LB_EINVAL
        assert L.lb_import_arrays(s.h, 4, p, len(bad)) == lbm.LB_EINVAL
    p = (ctypes.c_void_p * 10)(*(ptrs[:6] + [null] * 4))   # no beads in the second box
    assert L.lb_export_arrays(s.h, ctypes.byref(step), p, 10) == lbm.LB_OK and step.value == 7
    _equal(st["boxes"], want)
    assert L.lb_import_arrays(s.h, 7, p, 10) == lbm.LB_OK
    s.close()


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("n", [3, 129])
def test_wide_chains_that_leave_their_set_aside_nodes(prec, n):
    """The 512-thread shapes for 65 to 128 beads, few chains and more than half
    as many as the GPU has CUs, one of them flying apart."""
    say("wide chains", prec, n)
    boxes = [params(L=16, N=100, kT=0.0, therm=0, seed=5, box_id=0)]
    boxes += [params(L=11, N=65 + i % 64, kT=1e-2, seed=5, box_id=i) for i in range(1, n)]
    xs = [chain(b) for b in boxes]
    xs[0] = xs[0][0] + 0.93 * (xs[0] - xs[0][0])
    ref = gpu_system(boxes, prec, xs=xs)
    ref.set_launch(batched=True, overlap=False)
    left = 0
    for _ in range(4):
        a = ref.export_state()["boxes"][0]
        ref.step(1)
        left += int(_left_set_aside(boxes[0], a["x"], a["v"], ref.export_state()["boxes"][0]["x"]).sum())
    ref.close()
    assert left > 0
    want = _run(boxes, xs, prec, False, 0, (7,))
    _equal(_run(boxes, xs, prec, True, 0, (1, 2, 4)), want)


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_observables_with_and_without_ranges_of_records(orc, prec):
    """Boxes whose block records are summed at once beside ones that sum ranges
    of them first (above 256 records: 104^3), in either order; in the static
    array the same bits, and against the boxes alone."""
    say("record ranges", prec)
    boxes = [params(L=104, N=0, kT=1e-2, box_id=0), params(L=10, N=7, kT=1e-2, box_id=1), params(L=103, N=0, kT=1e-2, box_id=2),
             params(L=105, N=30, kT=1e-2, box_id=3)]
    xs = [chain(b) for b in boxes]
    s = gpu_system(boxes, prec, xs=xs)
    s.step(2)
    got, static = s.observables(), s.observables(static=True)
    s.close()
    for i, b in enumerate(boxes):
        one = gpu_system([b], prec, xs=[xs[i]])
        one.step(2)
        for o in (static[i], one.observables()[0]):
            for k, v in got[i].items():
                assert np.array_equal(v, o[k]), (i, k)
        one.close()
        assert got[i]["mass"] == pytest.approx(int(b["L"]) ** 3, rel=1e-6) and got[i]["mode_sq"][4] > 0


@pytest.mark.parametrize("prec,resident", [(FP32, True), (FP32, False), (FP64, True)])
def test_large_chains_in_two_boxes_whose_collide_sets_the_time(prec, resident):
    """Two sparse boxes with a large chain each, so many nodes that the collide
    sets the step time: in FP32 the collides carry the node tables of both
    (workgroups of two list entries, the overflow fix-up sorted by box), in
    launch mode 3 and in FP64 the two queues alternate.  The second chain is
    hot: its beads leave their tables.  Bits as with the re-collision after
    the collide."""
    say("two large chains, collide-bound", prec, resident)
    hot = dict(kT=1.0, therm=0, zeta=1.0, k_fene=7.0, r0_fene=2.0)
    base = dict(seed=7, md_dt=0.02, md_substeps=10, tau_lb=0.2)
    boxes = [params(L=107, N=280, box_id=0, **base, kT=1e-2, k_fene=7.0, r0_fene=2.0, zeta=1.0),
             params(L=107, N=300, box_id=1, **base, **hot)]
    xs = [chain(b) for b in boxes]
    s = gpu_system(boxes, prec, xs=xs)
    s.set_launch(batched=True, overlap=False)
    left = 0
    for _ in range(8):
        a = s.bead_positions()[280:]
        s.step(1)
        left += int((np.abs(np.floor(s.bead_positions()[280:]) + 0.5 - np.floor(a + 0.5)) > 1.0).any(1).sum())
    assert all(o["health"] == 0 for o in s.observables())
    want = s.export_state()["boxes"]
    s.close()
    assert left > 0
    s = gpu_system(boxes, prec, xs=xs)
    s.set_launch(batched=True, overlap=True, resident=resident)
    for n in (5, 3):
        s.step(n)
    assert all(o["health"] == 0 for o in s.observables())
    _equal(s.export_state()["boxes"], want)
    s.close()


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("batch", ["small chains", "fluid", "large chain"])
def test_every_launch_shape_of_the_batched_collide(prec, batch):
    """k_collide over several boxes in every launch shape: with chains of at
    most 256 beads re-collided after it, with no chain, and with the stamps of
    the deferred segments around a large chain.  The autotuner's choice too."""
    import paper_0903_5067_amd as lbm
    say("batched collide shapes", prec, batch)
    boxes = {"small chains": [params(L=16, N=20, kT=1e-2, box_id=0), params(L=9, N=40, kT=1e-2, box_id=1)],
             "fluid": [params(L=16, N=0, kT=1e-2, box_id=0), params(L=11, N=0, kT=1e-2, box_id=1)],
             "large chain": [params(L=40, N=300, kT=1e-2, box_id=0), params(L=11, N=0, kT=1e-2, box_id=1)]}[batch]
    s = gpu_system(boxes, prec, xs=[chain(b) for b in boxes])
    s.set_launch(batched=True, overlap=batch != "small chains")
    a = s.export_state()
    want = None
    for v in list(range(lbm.N_COLLIDE_VARIANTS)) + ["autotuned"]:
        if v == "autotuned":
            s.autotune(reps=2)
        else:
            s.set_collide_variant(v)
        s.import_state(a)
        s.step(5)
        got = s.export_state()["boxes"]
        want = want or got
        _equal(got, want)
    assert s.observables()[0]["health"] == 0
    s.close()


@pytest.mark.parametrize("N,k", [(16, 4), (16, 1), (100, 3)])
def test_window_whose_beads_leave_their_set_aside_nodes(orc, N, k):
    """A chain that flies apart inside a window: the impulses outside the
    set-aside nodes are re-collided in the forward run and, from the tape
    slots of the step before, in the replay; trajectory and gradient against
    the oracle's exact tangent."""
    say("window, left set-aside nodes", N, k)
    p = params(L=16, N=N, kT=0.0, therm=0, omega_s=1.2, omega_b=0.9, seed=5)
    x0 = chain(p)
    x0 = x0[0] + 0.93 * (x0 - x0[0])
    n0 = initial_pops(orc, p, amp=0.01, seed=11)
    o, left = oracle_state(orc, p, n0, x0), 0
    for _ in range(6):
        a, v = o.x.copy(), o.v.copy()
        o.run(1)
        left += int(_left_set_aside(p, a, v, o.x).sum())
    assert left > 0
    s = gpu_system([p], FP64, xs=[x0], pops=[n0])
    vh = s.window_forward(6, k)
    cw = np.random.default_rng(5).normal(size=vh.shape)
    grad = s.window_backward(cw)[0]
    assert s.observables()[0]["health"] == 0
    ho, dh = oracle_state(orc, p, n0, x0).window_tangent(6)
    assert np.max(np.abs(vh - ho)) < 1e-10
    ref = np.einsum("tna,tnak->k", cw, dh)
    np.testing.assert_allclose(grad, ref, rtol=1e-7, atol=1e-7 * np.max(np.abs(ref)))
    s.close()


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("L,N,chain_len,modes", [(16, 16, 0, (0, 1, 2)), (16, 33, 0, (1,)), (20, 100, 0, (0, 1, 2)), (16, 200, 0, (1,)),
                                                 (40, 300, 0, (0, 1, 2)), (16, 512, 32, (0, 1)), (48, 600, 0, (1,))])
def test_beads_beyond_any_box_address_nothing_outside(L, N, chain_len, modes, prec):
    """Positions and velocities as a broken bond leaves them (far past the box,
    not finite): the steps end with health bits set, and the same system goes
    on from an imported state as if nothing had been."""
    import ctypes

    import paper_0903_5067_amd as lbm
    say("broken bonds", L, N, prec)
    p = params(L=L, N=N, chain_len=chain_len, kT=1e-2, seed=6)
    for mode in modes:
        say("launch mode", mode)
        s = gpu_system([p], prec, xs=[chain(p)])
        s.set_launch(batched=mode > 0, overlap=mode != 2)
        good = s.export_state()
        s.import_state(good)
        s.step(3)
        want = s.export_state()["boxes"]
        bad = {"step": 0, "boxes": [{k: a.copy() for k, a in good["boxes"][0].items()}]}
        b = bad["boxes"][0]
        b["x"][0], b["x"][3], b["x"][N // 2] = 1e18, -3e25, (1e300, 5.0, -1e17)
        b["v"][5], b["v"][N - 1] = 1e200, np.nan
        s.import_state(bad)
        s.step(3)
        assert s.observables(allow_unhealthy=True)[0]["health"] != 0
        s.import_state(good)
        s.step(3)
        with pytest.raises(lbm.LBError):   # the health word stays
            s.export_state()
        got = {k: np.empty_like(a) for k, a in good["boxes"][0].items()}
        ptrs = (ctypes.c_void_p * 5)(*[a.ctypes.data for a in got.values()])
        assert lbm.lib().lb_export_arrays(s.h, ctypes.byref(ctypes.c_uint64()), ptrs, 5) == lbm.LB_ENUMERIC
        _equal([got], want)
        s.close()
