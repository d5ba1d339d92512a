"""Branches of the launch and kernel dispatch at the sizes where they can go wrong: load order,
workgroup size and defaults by domain size and lookup, states at rest, pools with face members, the
pressure condition inside the collide kernel against the face kernel, read-back through pinned
memory or a device buffer, byte and 16-bit neighbour codes, call buffers on both sides of a block,
and the distance, line and labelling passes of the pre-processing at word, window, packing and tile
edges. Step results are compared bitwise (all variants evaluate the same operations), distances
and masks exactly."""
import dataclasses
import time
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle as O
from oracle import prep as OP
from paper_2007_12266_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

PRECISIONS = ("fp64", "mixed", "fp32dev")


@pytest.fixture(scope="module")
def lbm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2007_12266_amd import lbm as mod
    mod.load_library()
    return mod


def _prec(lbm, name):
    return {"fp64": lbm.FP64, "mixed": lbm.FP32_MIXED, "fp32dev": lbm.FP32_DEV}[name]


def _box(shape, seed, solid_frac=0.1, periodic=(True, True, True)):
    rng = np.random.default_rng(seed)
    return inputs.Problem(labels=np.where(rng.random(shape) < solid_frac, 0, 1).astype(np.int32),
                          label_kind=np.array([inputs.KIND_SOLID, inputs.KIND_PORE_INIT], np.int8),
                          label_affinity=np.array([0.4, 0.0]),
                          init_phi=inputs.bernoulli_phase(shape, 0.5, seed + 1),
                          periodic=periodic, tau_a=0.7, tau_b=0.8, force=(0, 0, 1e-5))


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("voxels", [(32, 32, 32), (33, 32, 32), (64, 64, 64), (65, 64, 64)])
def test_size_dependent_kernels_are_bitwise_identical(lbm, voxels, precision):
    """Open boxes of 32768 and 33792 voxels (default workgroups of 64 and of 256) and of 262144 and
    266240 (all loads first, or not): the default configuration equals streaming accesses in
    workgroups of 256, which have one variant for all sizes."""
    prob = _box(voxels, 5, solid_frac=0.0)
    out = []
    for stream in (0, 1):
        dom = lbm.Domain(prob, precision=_prec(lbm, precision))
        n = dom.n_pore
        assert dom.tuning()["collide_block"] == (64 if n <= 32768 else 256)
        if stream:
            dom.set_tuning(phase_stream=1, collide_stream=1, phase_block=256, collide_block=256)
        dom.step(9)
        out.append(dom.save())
        dom.close()
    assert out[0] == out[1]


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("mode", ["table", "rank", "compact"])
def test_pressure_faces_do_not_depend_on_how_steps_are_called(lbm, mode, precision):
    """The pressure condition is applied by the collide kernel inside a stretch of steps and by the
    face kernel where one ends: one call of 70 steps (a captured chunk and single steps), 70 calls,
    and calls that end on odd steps with reductions and read-back between give the same state."""
    prob = inputs.displacement_problem(shape=(20, 18, 22), seed_geom=31, porosity_target=0.4)
    nm = {"table": lbm.NBR_TABLE, "rank": lbm.NBR_RANK, "compact": lbm.NBR_COMPACT}[mode]
    blobs = []
    for calls in ((70,), (1,) * 70, (3, 64, 2, 1)):
        dom = lbm.Domain(prob, precision=_prec(lbm, precision), neighbour_mode=nm, reduce_every=7)
        for n in calls:
            dom.step(n)
            if len(calls) > 1:
                dom.reduce()
                dom.pore_field("uz")
        blobs.append((dom.save(), [h["qz"] for h in dom.history()]))
        dom.close()
    assert blobs[0] == blobs[1] == blobs[2]


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("steps", [0, 1, 2, 65])
def test_saved_states_continue_and_save_again(lbm, steps, precision):
    """A state saved after an even or an odd step loads into another domain, saves as the same
    bytes before any step, reads back the same fields, and goes on bit for bit; so does it after
    the launch configuration was timed on it."""
    prob = _box((14, 17, 23), 8, periodic=(True, False, True))
    a = lbm.Domain(prob, precision=_prec(lbm, precision))
    a.step(steps)
    blob = a.save()
    b = lbm.Domain(prob, precision=_prec(lbm, precision))
    b.step(3)
    b.load(blob)
    assert b.save() == blob
    for name in ("Na", "phi", "rho", "uz"):
        assert np.array_equal(a.pore_field(name), b.pore_field(name))
    b.autotune(2)
    assert b.save() == blob
    assert a.step(5).save() == b.step(5).save()
    a.close()
    b.close()


@pytest.mark.parametrize("edge", [101, 102])
def test_read_back_on_both_sides_of_the_pinned_limit(lbm, edge):
    """Boxes of 1,040,502 and 1,050,804 voxels: a field below 8 MiB is written to pinned
    memory, one above goes through the device buffer and its chunks. N_a sums to the mass either
    way, and the dense field holds the same values."""
    prob = _box((101, 102, edge), 3, solid_frac=0.0)
    dom = lbm.Domain(prob)
    dom.step(2)
    na = dom.pore_field("Na")
    assert (na.nbytes > 8 << 20) == (edge == 102)
    assert abs(na.sum() - dom.reduce()["mass_a"]) <= 1e-12 * na.sum()
    assert np.array_equal(np.sort(na), np.sort(dom.field("Na").reshape(-1)))
    dom.close()


@pytest.mark.parametrize("per", [(False, False, False), (True, True, True), (True, False, False)])
@pytest.mark.parametrize("nx", [1, 4, 31, 32, 33, 63, 64, 65, 96, 100, 129, 260, 1030])
def test_distances_at_word_and_window_edges(lbm, nx, per):
    """Row lengths around the half words of the row windows and the shapes of its workgroups, with
    features dense, sparse (distances beyond the windows of the row and of the lines) and one voxel
    at the end of a row."""
    rng = np.random.default_rng(nx)
    shape = (11, 26, nx) if nx < 500 else (3, 5, nx)
    last = np.zeros(shape, bool)
    last[1, 2, nx - 1] = True
    for feat in (rng.random(shape) < 0.3, rng.random(shape) < 3.0 / (shape[0] * shape[1] * nx), last):
        want = OP.edt_sq(feat, per)
        want = np.where(want >= OP.INF, -1, want)
        assert np.array_equal(lbm.prep_distance(feat, per), want)
        if nx < 500:
            out = torch.empty(shape, dtype=torch.int32, device="cuda")
            lbm.prep_distance_noalloc(torch.from_numpy(feat.astype(np.uint8)).cuda(), out,
                                      periodic=per, stream=torch.cuda.current_stream().cuda_stream)
            assert np.array_equal(out.cpu().numpy(), want)


@pytest.mark.parametrize("shape", [(3, 128, 70), (3, 129, 70), (239, 137, 9), (240, 137, 9),
                                   (240, 480, 4), (240, 481, 4), (256, 20, 6), (257, 95, 6),
                                   (257, 96, 6), (3, 128, 72), (240, 137, 8), (5, 20, 256),
                                   (5, 20, 264), (3, 9, 40), (240, 480, 8)])
@pytest.mark.parametrize("per", [(False, False, False), (True, True, False)])
def test_distances_with_row_and_line_passes_in_one_and_apart(lbm, shape, per):
    """Plane heights, counts and row lengths (words packed within the pass, or before) on both sides
    of the rules, dense and sparse features, walls."""
    rng = np.random.default_rng(shape[1])
    for density, walls in ((0.2, 0), (0.0005, 0), (0.002, 7)):
        feat = rng.random(shape) < density
        want = OP.edt_sq(feat, per, [bool(walls >> a & 1) for a in range(3)])
        want = np.where(want >= OP.INF, -1, want)
        assert np.array_equal(lbm.prep_distance(feat, per, wall_axes=walls), want)


@pytest.mark.parametrize("nx", [30, 32, 64, 68, 130])
@pytest.mark.parametrize("inlet", [False, True])
def test_drainage_with_byte_and_wide_distances(lbm, nx, inlet):
    """Rows that are and are not a multiple of 4 (lines packed in fours, or not), runs that cross
    word ends, and a wide channel whose spheres exceed a squared radius of 255 (32-bit passes)."""
    rng = np.random.default_rng(nx + inlet)
    per = (True, True, False)
    rock = rng.random((20, 24, nx)) < 0.9
    channel = np.ones((40, 44, max(nx, 44)), bool)
    channel[:, 0, :] = channel[:, :, 0] = False
    for pore, target in ((rock, 0.5), (channel, 0.6)):
        nw, got = lbm.prep_drain(pore, per, target, inlet=inlet)
        want = OP.drain(pore, per, target, inlet=inlet)
        assert np.array_equal(nw, want["nw"]) and got["k"] == want["k"]
        assert got["evaluations"] == want["evaluations"]
    assert got["kmax"] > 255


@pytest.mark.parametrize("shape", [(17, 16, 65), (16, 33, 64), (33, 15, 130), (1, 17, 63)])
@pytest.mark.parametrize("per", [(False, False, False), (True, True, False)])
def test_invasion_through_winding_pores_across_tiles(lbm, shape, per):
    """Pores just above the percolation threshold, whose components wind across the tiles of 16 x 16
    words, the words of a row and the periodic faces."""
    rng = np.random.default_rng(shape[1])
    for porosity in (0.33, 0.38):
        pore = rng.random(shape) < porosity
        pore[0, 0, 0] = True
        nw, got = lbm.prep_drain(pore, per, 0.0, inlet=True)
        want = OP.drain(pore, per, 0.0, inlet=True)
        assert np.array_equal(nw, want["nw"]) and got["k"] == want["k"]


@pytest.mark.parametrize("precision", PRECISIONS)
def test_pool_member_with_faces_costs_the_others_nothing(lbm, precision):
    """A pool of 15 periodic members and one with pressure faces steps in at most 1.6 times what
    one of 16 periodic members takes: 1.02 to 1.06 with the kernels as they are, 1.9 to 2.6 with a
    kernel that holds its arguments in scratch memory."""
    rocks = []
    for k in range(16):
        solid, _ = inputs.grf_rock((64, 64, 64), 4.0, 0.25, 40 + k)
        rocks.append(dataclasses.replace(_box((64, 64, 64), 40 + k),
                                         labels=np.where(solid > 0, 0, 1).astype(np.int32)))
    face = inputs.displacement_problem(shape=(64, 64, 64), seed_geom=5, porosity_target=0.25)
    took = []
    for probs in (rocks, rocks[:15] + [face]):
        pool = lbm.Pool(1 << 34, precision=_prec(lbm, precision), max_slots=16, chunk_steps=64)
        doms = [lbm.Domain(p, precision=_prec(lbm, precision)) for p in probs]
        for d in doms:
            pool.admit(d)
        best = float("inf")
        for _ in range(6):
            torch.cuda.synchronize()
            start = time.perf_counter()
            pool.step(128)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - start)
        took.append(best)
        pool.close()
        for d in doms:
            d.close()
    assert took[1] <= 1.6 * took[0]


@pytest.mark.parametrize("mode,edge,stream,limited", [("rank", 93, 0, False), ("table", 93, 0, True),
                                                      ("compact", 93, 0, True), ("rank", 122, 0, False),
                                                      ("compact", 122, 1, True),
                                                      ("rank", 140, 1, True)])
def test_default_launch_configuration_by_size_and_lookup(lbm, mode, edge, stream, limited):
    """Open boxes above 786432 voxels, of 384 to 512 MiB and above 512 MiB in FP64: streaming and
    workgroup limits begin later with the rank lookup, whose dependent loads need the waves."""
    nm = {"table": lbm.NBR_TABLE, "rank": lbm.NBR_RANK, "compact": lbm.NBR_COMPACT}[mode]
    dom = lbm.Domain(_box((edge, edge, edge), 1, solid_frac=0.0), neighbour_mode=nm)
    tuned = dom.tuning()
    assert (dom.info()["device_bytes"] > 384 << 20) == (edge > 93)
    assert (dom.info()["device_bytes"] > 512 << 20) == (edge == 140)
    assert tuned["phase_stream"] == tuned["collide_stream"] == stream
    assert (tuned["phase_wg"], tuned["collide_wg"]) == ((5, 2) if limited else (0, 0))
    dom.close()


@pytest.mark.parametrize("shape", [(101, 103, 100), (104, 101, 100), (33, 130, 260)])
@pytest.mark.parametrize("per", [(False, False, False), (False, True, False)])
def test_byte_passes_on_both_sides_of_the_four_line_rule(lbm, shape, per):
    """Images just below and above 2^20 voxels (a line to a thread, four to a thread) whose rows and
    lines leave remainders: pores so open that most searches go beyond the windows (squared radii of
    82 to 255), and narrow ones."""
    rng = np.random.default_rng(shape[1])
    for density, target in ((0.0004, 0.5), (0.08, 0.4)):
        pore = rng.random(shape) >= density
        nw, got = lbm.prep_drain(pore, per, target)
        want = OP.drain(pore, per, target)
        assert np.array_equal(nw, want["nw"]) and got["k"] == want["k"]
        assert density > 0.01 or 81 < got["k"] <= 255


@pytest.mark.parametrize("nx", [1, 2, 4, 5, 16, 31, 32, 33, 48, 63, 64, 65])
def test_distances_in_short_periodic_rows(lbm, nx):
    """Periodic rows around one and two half words, whose windows go on with the row's own ends."""
    rng = np.random.default_rng(nx)
    for density in (0.5, 0.08, 1.5 / nx, 0.2 / nx):
        feat = rng.random((3, 40, nx)) < density
        want = OP.edt_sq(feat, (True, False, False))
        want = np.where(want >= OP.INF, -1, want)
        assert np.array_equal(lbm.prep_distance(feat, (True, False, False)), want)


@pytest.mark.parametrize("shape", [(2, 3, 4), (64, 64, 127), (64, 64, 128), (64, 65, 128), (128, 128, 128)])
def test_call_buffers_on_both_sides_of_the_block_limit(lbm, shape):
    """Images whose 4-byte buffers are below, at and above 2 MiB, and whose 1-byte buffers reach it:
    some, none or all of a call's buffers share an allocation."""
    rng = np.random.default_rng(shape[2])
    pore = rng.random(shape) < 0.4
    nw = pore & (rng.random(shape) < 0.02)
    kind = np.array([inputs.KIND_SOLID, inputs.KIND_PORE_INIT, inputs.KIND_SOLID], np.int8)
    lab = pore.astype(np.int32)
    per = (False, False, False)
    assert np.array_equal(lbm.prep_relabel(lab, kind, nw, per, 2.0, 2),
                          OP.relabel(lab, kind, nw, per, 2.0, 2))
    assert np.array_equal(lbm.prep_mixing_layer(lab, kind, 2, 1), OP.mixing_layer(lab, kind, 2, 1))
    mask, got = lbm.prep_drain(pore, per, 0.6, inlet=True)
    want = OP.drain(pore, per, 0.6, inlet=True)
    assert np.array_equal(mask, want["nw"]) and got["k"] == want["k"]


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("edge", [80, 81, 102])
def test_large_states_save_and_load(lbm, edge, precision):
    """Boxes of 512,000, 531,441 and 1,061,208 voxels: the component densities of a saved state go
    through pinned memory up to 8 MiB and in parts above (first in FP64 and FP32-mixed, then in
    FP32-dev). The state loads, saves as the same bytes and goes on bit for bit."""
    prob = _box((edge, edge, edge), 6, solid_frac=0.0)
    a, b = (lbm.Domain(prob, precision=_prec(lbm, precision)) for _ in range(2))
    blob = a.step(3).save()
    b.load(blob)
    assert b.save() == blob
    assert np.array_equal(a.pore_field("Nb"), b.pore_field("Nb"))
    assert a.step(2).save() == b.step(2).save()
    a.close()
    b.close()


def test_read_back_by_more_threads_than_pinned_buffers(lbm):
    """Ten threads, each with a domain on a stream of its own, step, reduce and read at once: some
    read through pinned memory and some through their device buffers, all what one thread reads."""
    probs = [_box((20, 22, 24 + k), 60 + k) for k in range(10)]

    def work(dom):
        out = []
        for _ in range(12):
            dom.step(3)
            out.append((dom.reduce(), dom.pore_field("phi").tobytes(), dom.save()))
        return out

    want = []
    for p in probs:
        dom = lbm.Domain(p)
        want.append(work(dom))
        dom.close()
    streams = [torch.cuda.Stream() for _ in probs]
    doms = [lbm.Domain(p, stream=s.cuda_stream) for p, s in zip(probs, streams)]
    with ThreadPoolExecutor(len(doms)) as pool:
        assert list(pool.map(work, doms)) == want
    for d in doms:
        d.close()


@pytest.mark.parametrize("edge", [50, 52, 57, 65, 80])
def test_read_back_in_one_to_eight_parts(lbm, edge):
    """Fields of 0.95 to 3.9 MiB, copied out of pinned memory by one thread for each 512 KiB: in pore
    order the values of the dense field, which is formed from a copy of its own."""
    dom = lbm.Domain(_box((edge, edge, edge), 9, solid_frac=0.0))
    dom.step(2)
    for name in ("Na", "uz"):
        got = dom.pore_field(name)
        assert np.array_equal(got, dom.field(name).reshape(-1)[dom.pore_index()])
    assert abs(dom.pore_field("Na").sum() - dom.reduce()["mass_a"]) <= 1e-12 * got.size
    dom.close()


@pytest.mark.parametrize("thin", [1, 2, 3, 7, 8, 9, 15, 16, 17])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("per", [(False, False, False), (True, True, True)])
def test_thin_images_in_each_axis(lbm, axis, thin, per):
    """Lines along y or z of 1 to 17 voxels, around the segments and the windows, which on a periodic
    line wrap more than once, in rows packed in eights and not, on planes of few and of many rows:
    distances, with walls, and (bytes) a drainage."""
    rng = np.random.default_rng(10 * thin + axis)
    for nx, other in ((40, 70), (37, 130), (300, 12)):
        shape = (thin, other, nx) if axis == 0 else (other, thin, nx)
        for density, walls in ((0.1, 0), (3.0 / (thin * other * nx), 7)):
            feat = rng.random(shape) < density
            want = OP.edt_sq(feat, per, [bool(walls >> a & 1) for a in range(3)])
            want = np.where(want >= OP.INF, -1, want)
            assert np.array_equal(lbm.prep_distance(feat, per, wall_axes=walls), want)
        pore = rng.random(shape) < 0.9
        mask, got = lbm.prep_drain(pore, per, 0.5)
        want = OP.drain(pore, per, 0.5)
        assert np.array_equal(mask, want["nw"]) and got["k"] == want["k"]


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("mode", ["table", "rank", "compact"])
@pytest.mark.parametrize("faces", [False, True])
def test_large_domain_at_rest(lbm, faces, mode, precision):
    """Domains above 262144 pore voxels count the phase of a state at rest without its neighbours: the
    initial phase is read back as given, counted and summed, two steps from it follow the oracle, and
    the phase counted at rest after a growth is the one that the fields show. Bounds: of each field's
    largest value 1e-12 in FP64, 1e-6 where populations are float (2e-8 relative to their rest
    values, 0.06, against velocities of 1e-3 and up), 1e-5 where everything is."""
    nm = {"table": lbm.NBR_TABLE, "rank": lbm.NBR_RANK, "compact": lbm.NBR_COMPACT}[mode]
    prob = _box((70, 66, 68), 21, solid_frac=0.1)
    if faces:
        prob = inputs.displacement_problem(shape=(80, 70, 72), seed_geom=4, porosity_target=0.75)
    tol = {"fp64": 1e-12, "mixed": 1e-6, "fp32dev": 1e-5}[precision]
    pore = prob.solid_mask() == 0
    dom = lbm.Domain(prob, precision=_prec(lbm, precision), neighbour_mode=nm)
    assert dom.n_pore > 1 << 18
    phi = prob.phase0()[pore]
    assert np.abs(dom.field("phi")[pore] - phi).max() <= (1e-6 if precision == "fp32dev" else 1e-14)
    assert dom.reduce()["sw_count"] == (phi > 0).mean()
    assert dom.phase_volume() == int((phi > 0).sum())
    ref = O.state_for(prob).run(2)
    dom.step(2)
    got, want = dom.fields(), ref.fields()
    for k in ("Na", "Nb", "phi", "rho", "ux", "uy", "uz"):
        scale = max(np.abs(want[c][pore]).max() for c in (("ux", "uy", "uz") if k[0] == "u" else (k,)))
        if precision == "fp32dev" and not faces:
            break   # a random phase has gradients below 1e-5, which this precision counts as none
        assert np.abs(got[k][pore] - want[k][pore]).max() <= tol * scale, k
    if not faces:
        assert dom.phase_volume() == dom.morph(delta=0.7)["volume_before"]
        assert np.array_equal(dom.pore_field("phi") > 0, dom.field("phi").reshape(-1)[dom.pore_index()] > 0)
        assert dom.phase_volume() == int((dom.pore_field("phi") > 0).sum())
    dom.close()
