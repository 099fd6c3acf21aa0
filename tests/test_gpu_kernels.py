"""GPU kernels at the sizes where their work split changes (tiles, remainders,
the smallest and largest of a dispatch's ranges), against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2012_02207_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def fmm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2012_02207_amd import fmm as F
    return F


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


# 1024 sinks are the most that get a workgroup each; more share one by fours
@pytest.mark.parametrize("n,nsink", [(1, 1), (2, 2), (255, 1), (1025, 63), (1030, 1024), (1030, 1025), (3001, 1027)])
@pytest.mark.parametrize("eps_soft", [0.0, 1e-3])
def test_direct_sum_splits(fmm, n, nsink, eps_soft):
    """Compensated on both sides, so the sums agree to the rounding of their
    terms (a few 2^-53 each, of either sign) relative to the sum of the terms'
    sizes; the potential's terms have one sign."""
    pos, _, mass = W.plummer(max(n, 8), 31)
    pos, mass = pos[:n].copy(), mass[:n].copy()
    if n > 100:
        pos[5] = pos[77]  # a coincident pair contributes nothing without softening
    sinks = np.random.default_rng(n).permutation(n)[:nsink]
    print(f"[gpu] direct n={n} nsink={nsink} eps_soft={eps_soft}", flush=True)
    acc, pot = fmm.direct(_dev(pos), _dev(mass), eps_soft=eps_soft, sinks=_dev(sinks.astype(np.int32)))
    ad, pd = oracle.direct(pos, mass, eps_soft=eps_soft, sinks=sinks.astype(np.int64))
    d = pos[None] - pos[sinks][:, None]
    s2 = (d * d).sum(-1) + eps_soft ** 2
    s2[s2 == 0.0] = np.inf
    size = (mass * np.sqrt((d * d).sum(-1)) * s2 ** -1.5).sum(1)
    assert (np.abs(acc.cpu().numpy() - ad) <= 2e-15 * size[:, None] + 1e-300).all()
    np.testing.assert_allclose(pot.cpu().numpy(), pd, rtol=2e-15, atol=0.0)


# up to 4096 leaves the estimate's near sums take sixteen wavefronts per leaf;
# leaves of one body to more than 64, masses beyond the range of the unscaled
# division (2^-500 .. 2^500) among them
@pytest.mark.parametrize("n,n_leaf,scale", [(1, 64, 1.0), (66, 64, 1.0), (130, 128, 1e-160), (700, 1, 1.0),
                                            (5000, 1, 1.0), (4500, 3, 1e-200), (9000, 200, 1.0)])
def test_estimate_near_sums(fmm, n, n_leaf, scale):
    """The scalar-force estimate is summed in the oracle's order: bit for bit."""
    pos, mass = W.uniform_cube(n, 17)
    mass[::7] = 0.0
    mass[1::5] *= scale
    if n > 100:
        pos[3] = pos[60]  # coincident bodies count nothing
        pos[61] = pos[60] + 1e-170
    print(f"[gpu] estimate n={n} n_leaf={n_leaf}", flush=True)
    f = fmm.FMM(p=2, err_tol=1e-3, n_leaf=n_leaf)
    f.forces(_dev(pos), _dev(mass))
    o = oracle.Oracle()
    o.run(pos, mass, p=2, err_tol=1e-3, n_leaf=n_leaf, stage="walk")
    assert np.array_equal(f.export("f_part"), o.get("f_part"))
    assert np.array_equal(f.export("fmin"), o.get("fmin"))
    f.close()


def _clumps(n, seed):
    """Points at every scale: a cube, tight clumps, exact duplicates (level-21
    cells) and a line of points that splits into single-child chains."""
    rng = np.random.default_rng(seed)
    pos = rng.uniform(-1.0, 1.0, (n, 3))
    k = n // 4
    pos[:k] = 0.25 + rng.normal(size=(k, 3)) * 10.0 ** rng.uniform(-9, -1, (k, 1))
    if n > 40:
        pos[k:k + n // 8] = pos[k]
    return pos, np.full(n, 1.0 / n)


# the cells are written in tiles of 1024 bodies, from windows of n_leaf + 1
@pytest.mark.parametrize("n,n_leaf", [(1, 64), (2, 1), (64, 64), (65, 64), (1024, 7), (1025, 64), (2047, 1),
                                      (2049, 1024), (5000, 100), (3071, 1023)])
def test_cells_match_oracle(fmm, n, n_leaf):
    """Cells, leaves and centres of the oracle's tree, bit for bit."""
    pos, mass = _clumps(n, 40 + n)
    print(f"[gpu] cells n={n} n_leaf={n_leaf}", flush=True)
    f = fmm.FMM(p=1, n_leaf=n_leaf)
    f.build(_dev(pos), _dev(mass))
    o = oracle.Oracle()
    o.run(pos, mass, p=1, err_tol=1e-7, n_leaf=n_leaf, stage="upward")
    for k in ("cell_level", "cell_begin", "cell_end", "cell_parent", "cell_child0", "cell_nchild"):
        assert np.array_equal(f.export(k).astype(np.int64), o.get(k).astype(np.int64)), k
    assert f.stats()["nleaf"] == (o.get("cell_nchild") == 0).sum()
    assert np.array_equal(f.export("mult"), o.get("mult"))  # the leaf list reached every leaf
    f.close()


def test_noalloc_many_calls(fmm):
    """Repeated calls take the same part of the fixed scratch each time."""
    pos, _, mass = W.plummer(4096, 9)
    p, m = _dev(pos), _dev(mass)
    f = fmm.FMM(p=6, err_tol=1e-6)
    first = None
    for _ in range(60):
        a, _ = f.forces(p, m, noalloc=True)
        first = a if first is None else first
    assert torch.equal(first, a)
    f.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,n_leaf,eps_soft", [(700, 1, 0.0), (4097, 64, 1e-4), (9001, 16, 0.0), (5000, 130, 0.0),
                                               (70001, 64, 0.0)])
def test_near_field_segment_lengths(fmm, precision, n, n_leaf, eps_soft):
    """Segments of 8 entries to a 1024th of the bodies, leaves of one body to
    more than a wavefront's 64: the forces agree with the oracle as the whole
    lists' do (FP64 1e-12 median; mixed its bound, 1.5e-7), and a batch of two
    systems repeats each system's sums bit for bit."""
    pos, _, mass = W.plummer(n, 60)
    print(f"[gpu] near-field segments n={n} n_leaf={n_leaf} {precision}", flush=True)
    f = fmm.FMM(p=6, err_tol=1e-6, n_leaf=n_leaf, precision=precision)
    acc, pot = f.forces(_dev(pos), _dev(mass), eps_soft=eps_soft)
    o = oracle.Oracle()
    oacc, opot = o.run(pos, mass, p=6, err_tol=1e-6, n_leaf=n_leaf, eps_soft=eps_soft)
    rel = np.linalg.norm(acc.cpu().numpy() - oacc, axis=1) / np.linalg.norm(oacc, axis=1)
    assert np.median(rel) <= (1e-12 if precision == "fp64" else 1.5e-7), np.median(rel)
    if n < 20000:
        q, _, mq = W.plummer(333, 61)
        both, _ = f.forces_batch(_dev(np.concatenate([q, pos])), _dev(np.concatenate([mq, mass])),
                                 np.array([0, 333, 333 + n]), eps_soft=eps_soft)
        assert torch.equal(both[333:], acc)
    f.close()


# orders at the edges of the upward kernels' splits: P2M values per lane (p <= 10,
# 14, 22, 30), M2M tasks in one round of threads or two, the eight-children
# layout (p <= 22) and the streamed one
@pytest.mark.parametrize("p", [1, 7, 10, 11, 14, 15, 16, 21, 22, 23, 30])
def test_upward_orders(fmm, p):
    """Multipoles and norms of the oracle, bit for bit: leaves of one body to
    many batches, offsets whose high powers underflow (the division's general
    path) and masses of zero."""
    pos, mass = _clumps(600, 90)
    pos[5:25] = pos[5] + np.random.default_rng(1).normal(size=(20, 3)) * 1e-7
    pos[30:50] = 1e-30 * np.random.default_rng(2).normal(size=(20, 3))
    mass[::9] = 0.0
    print(f"[gpu] upward p={p}", flush=True)
    f = fmm.FMM(p=p, n_leaf=24)
    f.build(_dev(pos), _dev(mass))
    o = oracle.Oracle()
    o.run(pos, mass, p=p, err_tol=1e-7, n_leaf=24, stage="upward")
    assert np.array_equal(f.export("mult"), o.get("mult"))
    assert np.array_equal(f.export("pk"), o.get("pk"))
    f.close()


# the matrix-core M2L: one and two tiles of 16 pairs at a time (p <= 20), orders
# owned by two, three and four slots of a wavefront, lists of one pair to several
# segments
@pytest.mark.parametrize("p,n,n_leaf,err_tol", [(17, 400, 40, 1e-3), (18, 3000, 8, 1e-6), (20, 9000, 4, 1e-8),
                                                (21, 3000, 16, 1e-6), (23, 2000, 8, 1e-6), (25, 2500, 16, 1e-6),
                                                (29, 1500, 4, 1e-9)])
def test_high_order_m2l(fmm, p, n, n_leaf, err_tol):
    """Local expansions and forces of the oracle to rounding (the FP64 parity
    bounds: median 1e-12, maximum 1e-9), with the same lists."""
    pos, _, mass = W.plummer(n, 80 + p)
    print(f"[gpu] high order p={p} n={n} n_leaf={n_leaf}", flush=True)
    f = fmm.FMM(p=p, err_tol=err_tol, n_leaf=n_leaf)
    acc, _ = f.forces(_dev(pos), _dev(mass))
    o = oracle.Oracle()
    oacc, _ = o.run(pos, mass, p=p, err_tol=err_tol, n_leaf=n_leaf)
    rel = np.linalg.norm(acc.cpu().numpy() - oacc, axis=1) / np.linalg.norm(oacc, axis=1)
    assert np.median(rel) <= 1e-12 and rel.max() <= 1e-9, (np.median(rel), rel.max())
    lg, lo = f.export("local"), o.get("local")
    scale = np.abs(lo).max(axis=1, keepdims=True) + 1e-300
    assert np.median(np.abs(lg - lo) / scale) < 1e-12
    a2, _ = f.forces(_dev(pos), _dev(mass))
    assert torch.equal(acc, a2)
    f.close()


# four sinks to a workgroup up to p = 8 and one above; coefficients loaded an
# order ahead but for p = 11 and 12; from order 1, lists of one pair to several
# segments
@pytest.mark.parametrize("p,n,n_leaf,err_tol", [(1, 300, 8, 1e-2), (8, 3000, 8, 1e-5), (9, 3000, 4, 1e-6),
                                                (10, 20000, 16, 1e-6), (11, 3000, 8, 1e-6), (12, 20000, 16, 1e-6),
                                                (13, 3000, 8, 1e-7), (16, 20000, 16, 1e-8)])
def test_register_m2l(fmm, p, n, n_leaf, err_tol):
    """Local expansions and forces of the oracle to rounding (the FP64 parity
    bounds: median 1e-12, maximum 1e-9)."""
    pos, _, mass = W.plummer(n, 90 + p)
    print(f"[gpu] m2l p={p} n={n} n_leaf={n_leaf}", flush=True)
    f = fmm.FMM(p=p, err_tol=err_tol, n_leaf=n_leaf)
    acc, _ = f.forces(_dev(pos), _dev(mass))
    o = oracle.Oracle()
    oacc, _ = o.run(pos, mass, p=p, err_tol=err_tol, n_leaf=n_leaf)
    rel = np.linalg.norm(acc.cpu().numpy() - oacc, axis=1) / np.linalg.norm(oacc, axis=1)
    assert np.median(rel) <= 1e-12 and rel.max() <= 1e-9, (np.median(rel), rel.max())
    lg, lo = f.export("local"), o.get("local")
    scale = np.abs(lo).max(axis=1, keepdims=True) + 1e-300
    assert np.median(np.abs(lg - lo) / scale) < 1e-12
    f.close()


# up to 8192 bodies are sorted, and lists of up to 20480 entries grouped, by one
# workgroup of 1024 threads
@pytest.mark.parametrize("n,n_leaf", [(1, 64), (63, 4), (1023, 64), (1025, 30), (3000, 40), (8191, 200), (8192, 300),
                                      (8193, 300)])
def test_one_workgroup_sorts(fmm, n, n_leaf):
    """Keys, order (ties in the caller's) and lists of the oracle, bit for bit,
    the lists ascending by sink and source."""
    pos, mass = _clumps(n, 70 + n)
    print(f"[gpu] sorts n={n} n_leaf={n_leaf}", flush=True)
    f = fmm.FMM(p=3, err_tol=1e-4, n_leaf=n_leaf)
    f.forces(_dev(pos), _dev(mass))
    o = oracle.Oracle()
    o.run(pos, mass, p=3, err_tol=1e-4, n_leaf=n_leaf, stage="walk")
    assert np.array_equal(f.export("keys"), o.get("keys"))
    assert np.array_equal(f.export("perm").astype(np.int64), o.get("perm"))
    assert np.array_equal(f.export("rootbox"), o.get("rootbox"))
    for k in ("est_far", "est_near", "m2l", "p2p"):
        want = np.asarray(o.get(k), dtype=np.int64).reshape(-1, 2)
        want = want[np.lexsort((want[:, 1], want[:, 0]))]
        print(k, len(want), flush=True)
        assert np.array_equal(f.export(k).astype(np.int64).reshape(-1, 2), want), k
    f.close()


# the mixed near field sums a chunk of a source leaf without a test per pair
# and again with it if a pair had no distance
@pytest.mark.parametrize("groups", [0, 1, 3])
@pytest.mark.parametrize("copies,n_leaf", [((30, 1, 2), 8), ((64, 65, 100), 64), ((200, 7), 100)])
def test_mixed_pairs_without_distance(fmm, copies, n_leaf, groups):
    """Coincident bodies (in one chunk, and in two of a leaf of more than 64)
    and a separation that FP32 rounds to zero add nothing to each other, and the
    other pairs of their chunks count.  Every pair directly but those of two
    cells without extent (theta small), so a sum is off by its FP32 roundings
    alone: 64 + 16 units of 2^-24 of the sum of the terms' sizes."""
    rng = np.random.default_rng(8)
    sites = rng.uniform(-1, 1, (len(copies), 3))
    tiny = np.array([[1e-26, 0.3, 0.3], [-1e-26, 0.3, 0.3]])
    box = np.array([[x, y, z] for x in (-1, 1) for y in (-1, 1) for z in (-1, 1)], dtype=np.float64)
    pos = np.concatenate([np.repeat(sites, copies, axis=0), tiny, box, rng.uniform(-1, 1, (211, 3))])
    pos = pos[rng.permutation(len(pos))]
    mass = rng.uniform(0.5, 1.5, len(pos))
    print(f"[gpu] mixed near field copies={copies} n_leaf={n_leaf} groups={groups}", flush=True)
    f = fmm.FMM(p=4, err_tol=1e-6, n_leaf=n_leaf, precision="mixed", theta=1e-3, p2p_groups=groups)
    acc, pot = f.forces(_dev(pos), _dev(mass))
    d = (pos[None] - pos[:, None]).astype(np.float32)
    d2 = (d * d).sum(-1)
    on = (d2 > 0) & ~np.eye(len(pos), dtype=bool)
    rinv = np.where(on, 1.0 / np.sqrt(np.where(on, d2, 1.0).astype(np.float64)), 0.0)
    term = (mass[None] * rinv**3)[..., None] * d.astype(np.float64)
    u = 80 * 2.0**-24
    assert (np.abs(acc.cpu().numpy() - term.sum(1)) <= u * np.abs(term).sum(1)).all()
    assert (np.abs(pot.cpu().numpy() + (mass[None] * rinv).sum(1)) <= u * (mass[None] * rinv).sum(1)).all()
    f.close()


# longer lists are split by the sink's top 8 bits, or by 9 to 16 in two passes,
# into parts sorted in LDS: up to 256 cells, parts of many sinks and of one, cell
# ids of more than 16 bits, and parts too long for LDS (close pairs make chains of
# cells without lists, and the leaves' long lists share few parts) either way
@pytest.mark.parametrize("kind,n,n_leaf,theta,p,err_tol", [
    ("uniform", 160, 1, 1e-3, 1, 1e-6), ("uniform", 900, 1, 1e-3, 1, 1e-6),
    ("uniform", 20000, 4, 0.5, 3, 1e-4),
    ("uniform", 60000, 1, 1.0, 3, 1e-2),
    ("pairs", 1000, 1, 1e-3, 1, 1e-6), ("pairs", 2000, 1, 1e-3, 1, 1e-6)])
def test_list_parts(fmm, kind, n, n_leaf, theta, p, err_tol):
    """The oracle's lists, ascending by sink and source."""
    rng = np.random.default_rng(n)
    pos = rng.uniform(-1, 1, (n, 3))
    if kind == "pairs":
        pos[n // 2:] = pos[:n // 2] + 1e-6
    mass = np.full(n, 1.0 / n)
    print(f"[gpu] list parts {kind} n={n}", flush=True)
    f = fmm.FMM(p=p, err_tol=err_tol, n_leaf=n_leaf, theta=theta)
    f.forces(_dev(pos), _dev(mass))
    o = oracle.Oracle()
    o.run(pos, mass, p=p, err_tol=err_tol, n_leaf=n_leaf, theta=theta, stage="walk")
    for k in ("est_far", "est_near", "m2l", "p2p"):
        want = np.asarray(o.get(k), dtype=np.int64).reshape(-1, 2)
        want = want[np.lexsort((want[:, 1], want[:, 0]))]
        print(k, len(want), flush=True)
        assert np.array_equal(f.export(k).astype(np.int64).reshape(-1, 2), want), k
    f.close()


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("first", ["forces", "jerk"])
def test_frozen_under_direct_precision(fmm, first, graph):
    """A frozen evaluation under precision "direct" is the FP64 one, bit for
    bit: leaves of more than one tile of sinks, split and unsplit lists."""
    pos, vel, mass = (_dev(a) for a in W.plummer(6000, 12))
    moved = pos + 1e-3 * vel
    print(f"[gpu] frozen under direct, after {first}, graph={graph}", flush=True)
    f = fmm.FMM(p=6, err_tol=1e-6)
    f.forces(pos, mass)
    want = f.forces_frozen(moved, mass)
    f.close()
    f = fmm.FMM(p=6, err_tol=1e-6, precision="fp64" if first == "forces" else "direct")
    if first == "forces":
        f.forces(pos, mass)
        f.set_params(precision="direct")
    else:  # evaluates in FP64 whatever the precision
        f.jerk(pos, vel, mass)
    got = [torch.full_like(t, 7.0) for t in want]
    for _ in range(2):
        f.forces_frozen(moved, mass, out=got, graph=graph)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    f.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
def test_batch_isolates_a_bad_system(fmm, precision, bad):
    """Systems of a batch feel only their own bodies: one whose positions are
    not finite, at the start of the sorted order, leaves the others' sums as
    they are alone, bit for bit."""
    pos, mass = W.uniform_cube(70, 3)
    pos[10:14] = bad
    q, _, mq = W.plummer(700, 4)
    print(f"[gpu] batch with a bad system {bad} {precision}", flush=True)
    f = fmm.FMM(p=4, err_tol=1e-5, precision=precision)
    alone = f.forces(_dev(q), _dev(mq))
    both = f.forces_batch(_dev(np.concatenate([pos, q, pos])), _dev(np.concatenate([mass, mq, mass])),
                          np.array([0, 70, 770, 840]))
    assert torch.equal(both[0][70:770], alone[0]) and torch.equal(both[1][70:770], alone[1])
    f.close()


def test_calls_after_a_failed_one(fmm):
    """A call that runs out of scratch on the way leaves nothing running on the
    buffers that the next call takes: small calls right behind such ones, in the
    fixed scratch and in a context's own under a limit, give what they give on
    their own."""
    big, _, mbig = (_dev(a) for a in W.plummer(65536, 15))
    pos, _, mass = (_dev(a) for a in W.plummer(3000, 16))
    f = fmm.FMM(p=20, err_tol=1e-9, n_leaf=8)
    want = f.forces(pos, mass)
    for _ in range(4):
        print("[gpu] noalloc after a failed call", flush=True)
        with pytest.raises(fmm.FmmError) as e:
            f.forces(big, mbig, noalloc=True)
        assert e.value.status == fmm.FMM_ENOMEM
        got = f.forces(pos, mass, noalloc=True)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    f.close()
    f = fmm.FMM(p=8, err_tol=1e-6)
    f.forces(big, mbig)
    need = f.stats()["workspace_bytes"]
    f.close()
    f = fmm.FMM(p=8, err_tol=1e-6)
    want = f.forces(pos, mass)
    for part in (0.15, 0.3, 0.45, 0.6, 0.75, 0.9):
        print(f"[gpu] forces after a call failed at {part} of its workspace", flush=True)
        f.set_workspace_limit(int(part * need))
        with pytest.raises(fmm.FmmError) as e:
            f.forces(big, mbig)
        assert e.value.status == fmm.FMM_ENOMEM
        f.set_workspace_limit(0)
        got = f.forces(pos, mass)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    f.close()


@pytest.mark.parametrize("graph", [False, True])
def test_no_adjoint_of_a_failed_frozen_evaluation(fmm, graph):
    """A frozen evaluation that runs out of workspace has changed the bodies and
    not finished the expansions: there is nothing left to differentiate."""
    pos, vel, mass = (_dev(a) for a in W.plummer(3000, 18))
    print(f"[gpu] adjoint after a failed frozen evaluation, graph={graph}", flush=True)
    f = fmm.FMM(p=6, err_tol=1e-6)
    acc, _ = f.forces(pos, mass)
    f.set_workspace_limit(f.stats()["workspace_bytes"])
    f.set_params(precision="mixed")  # needs the normalised moments too
    with pytest.raises(fmm.FmmError) as e:
        f.forces_frozen(pos + 0.1 * vel, mass, graph=graph)
    assert e.value.status == fmm.FMM_ENOMEM
    with pytest.raises(fmm.FmmError) as e:
        f.adjoint_last(acc, vel)
    assert e.value.status == fmm.FMM_ENOTBUILT
    f.close()


# internal cells' sums: a workgroup per run of levels of up to 2048 cells, a launch
# per larger level, in any succession
@pytest.mark.parametrize("kind", ["chain", "two widths"])
def test_cell_sums_of_clumped_trees(fmm, kind):
    """Masses and centres of the oracle, bit for bit, where the widest level is
    not the deepest internal one."""
    rng = np.random.default_rng(5)
    pos = rng.uniform(-1.0, 1.0, (24000, 3))
    if kind == "chain":  # a few cells on each of many levels below the widest
        pos[:12] = 0.3 + 1e-7 * rng.normal(size=(12, 3))
    else:  # wide, narrow, wide again
        pos[:12000] = 0.3 + 1e-4 * pos[:12000]
    mass = rng.uniform(0.5, 1.5, len(pos))
    print(f"[gpu] cell sums, {kind}", flush=True)
    f = fmm.FMM(p=1, n_leaf=4)
    f.build(_dev(pos), _dev(mass))
    level, nchild = f.export("cell_level"), f.export("cell_nchild")
    internal = np.bincount(level[nchild > 0])
    wide = np.bincount(level)[:len(internal)] > 2048
    assert wide.any() and not wide[0] and not wide[-1 if kind == "chain" else 8]
    assert kind == "chain" or wide[9:].any() and wide[:8].any()
    o = oracle.Oracle()
    o.run(pos, mass, p=1, err_tol=1e-7, n_leaf=4, stage="upward")
    for k in ("cell_mass", "cell_com"):
        assert np.array_equal(f.export(k), o.get(k).reshape(f.export(k).shape)), k
    f.close()


@pytest.mark.parametrize("count,big", [(200, ()), (3000, ()), (3000, (0, 1499, 2999)), (70000 // 16, (7,))])
def test_lists_of_few_sinks(fmm, count, big):
    """Batches whose interaction lists are empty, or have entries for a few of
    thousands of sinks: every list's offsets are the running counts of its
    entries, and the large systems' sums are those of their own calls."""
    rng = np.random.default_rng(count)
    size = np.ones(count, dtype=np.int64)
    size[list(big)] = 300
    off = np.concatenate([[0], np.cumsum(size)])
    pos, mass = rng.uniform(-1, 1, (off[-1], 3)), rng.uniform(0.5, 1.5, off[-1])
    print(f"[gpu] lists of few sinks: {count} systems, {len(big)} large", flush=True)
    f = fmm.FMM(p=4, err_tol=1e-3, n_leaf=16)
    acc, pot = f.forces_batch(_dev(pos), _dev(mass), off)
    st, nc = f.stats(), len(f.export("cell_level"))
    assert (st["n_m2l"] > 0) == bool(big) and (st["n_est_far"] > 0) == bool(big)
    for k in ("est_far", "est_near", "m2l", "p2p"):
        pairs = f.export(k)  # rebuilt from the offsets
        assert (np.diff(pairs[:, 0]) >= 0).all() and pairs.min(initial=0) >= 0 and pairs.max(initial=0) < nc, k
    p2p = f.export("p2p")
    assert set(map(tuple, p2p[p2p[:, 0] == p2p[:, 1]])) >= {(s, s) for s in np.flatnonzero(size == 1)}
    single = np.repeat(size == 1, size)
    assert not acc.cpu().numpy()[single].any() and not pot.cpu().numpy()[single].any()
    for s in big:
        a, q = f.forces(_dev(pos[off[s]:off[s + 1]]), _dev(mass[off[s]:off[s + 1]]))
        assert torch.equal(acc[off[s]:off[s + 1]], a) and torch.equal(pot[off[s]:off[s + 1]], q)
    f.close()


# lists of 8 entries or more (32 in FP64) are cut in these systems: a batch has more
# segments than the partial sums have room for, so most lists are summed by one
# wavefront in the batch and by several in a call of their own
@pytest.mark.parametrize("precision,count,n", [("mixed", 16, 4096), ("mixed", 60, 2000), ("fp64", 48, 4096)])
def test_large_batch_equals_single_calls(fmm, precision, count, n):
    """Every system of a batch of half a million list entries and more sums as
    it does alone, bit for bit."""
    kinds = [W.plummer(n, 200)[::2], W.kroupa_with_central(n, 201)[::2], W.uniform_cube(n, 202)]
    pos = np.concatenate([kinds[s % 3][0] for s in range(count)])
    mass = np.concatenate([kinds[s % 3][1] for s in range(count)])
    print(f"[gpu] batch of {count} x {n} {precision}", flush=True)
    f = fmm.FMM(p=5, err_tol=1e-6, precision=precision)
    acc, pot = f.forces_batch(_dev(pos), _dev(mass), np.arange(count + 1) * n)
    st = f.stats()
    assert st["n_p2p_cells"] > 65536 * 8
    alone = [f.forces(_dev(q), _dev(m)) for q, m in kinds]
    for s in range(count):
        a, q = alone[s % 3]
        assert torch.equal(acc[s * n:(s + 1) * n], a) and torch.equal(pot[s * n:(s + 1) * n], q), s
    f.close()


@pytest.mark.parametrize("n,n_leaf", [(1500, 64), (4096, 64), (5000, 5), (20000, 30)])
def test_near_field_under_a_limit(fmm, n, n_leaf):
    """With less room for partial sums more lists are summed unsplit: the
    same bits, for forces in both precisions, jerk and gradient, and the same
    again in frozen steps."""
    pos, vel, mass = (_dev(a) for a in W.plummer(n, 300))
    out = []
    for limit in (0, 1 << 34):
        print(f"[gpu] near field n={n} n_leaf={n_leaf} limit={limit}", flush=True)
        f = fmm.FMM(p=6, err_tol=1e-6, n_leaf=n_leaf)
        f.set_workspace_limit(limit)
        r = [*f.jerk(pos, vel, mass, eps_soft=1e-4), *f.adjoint(pos, mass, vel, eps_soft=1e-4)]
        r += f.forces(pos, mass)
        r += f.adjoint_last(r[-2], vel)
        r += f.forces_frozen(pos + 1e-3 * vel, mass, graph=True)
        f.set_params(precision="mixed")
        r += f.forces(pos, mass)
        r += f.forces_frozen(pos + 1e-3 * vel, mass)
        out.append(r)
        f.close()
    for a, b in zip(*out):
        assert torch.equal(a, b)


# M2L lists of more than 512 pairs (a 384th of the bodies, if that is more) are cut,
# also in batches of over four million pairs
@pytest.mark.parametrize("precision,p,count,n,n_leaf", [("fp64", 5, 12, 30000, 64), ("mixed", 5, 12, 30000, 64),
                                                        ("fp64", 4, 40, 8000, 6), ("mixed", 11, 40, 8000, 6),
                                                        ("fp64", 18, 12, 5000, 6), ("fp64", 16, 4, 6000, 6)])
def test_batch_m2l_segments(fmm, precision, p, count, n, n_leaf):
    """Every system of a batch sums as it does alone, bit for bit."""
    kinds = [W.plummer(n, 200)[::2], W.kroupa_with_central(n, 201)[::2], W.uniform_cube(n, 202)]
    pos = np.concatenate([kinds[s % 3][0] for s in range(count)])
    mass = np.concatenate([kinds[s % 3][1] for s in range(count)])
    print(f"[gpu] batch of {count} x {n} {precision} p={p} n_leaf={n_leaf}", flush=True)
    f = fmm.FMM(p=p, err_tol=1e-6, precision=precision, n_leaf=n_leaf)
    acc, pot = f.forces_batch(_dev(pos), _dev(mass), np.arange(count + 1) * n)
    assert count < 40 or f.stats()["n_m2l"] > 2 * 512 * 8192
    alone, longest = [], 0
    for q, m in kinds:
        alone.append(f.forces(_dev(q), _dev(m)))
        longest = max(longest, np.bincount(f.export("m2l")[:, 0]).max())
    assert longest > 512
    for s in range(count):
        a, q = alone[s % 3]
        assert torch.equal(acc[s * n:(s + 1) * n], a) and torch.equal(pot[s * n:(s + 1) * n], q), s
    f.close()


@pytest.mark.parametrize("p,n,n_leaf", [(17, 9000, 6), (22, 12000, 8)])
def test_high_order_m2l_under_a_limit(fmm, p, n, n_leaf):
    """Without slots for partial expansions (a workspace limit, the fixed
    scratch) long lists are summed by one workgroup: the same bits."""
    pos, vel, mass = (_dev(a) for a in W.kroupa_with_central(n, 400))
    out = []
    for limit in (0, 1 << 34):
        print(f"[gpu] high-order M2L p={p} n={n} limit={limit}", flush=True)
        f = fmm.FMM(p=p, err_tol=1e-6, n_leaf=n_leaf)
        f.set_workspace_limit(limit)
        out.append([*f.forces(pos, mass), *f.adjoint(pos, mass, vel)])
        assert np.bincount(f.export("m2l")[:, 0]).max() > 512
    out.append([*f.forces(pos, mass, noalloc=True), *out[0][2:]])
    f.close()
    for r in out[1:]:
        for a, b in zip(out[0], r):
            assert torch.equal(a, b)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("count,n,n_leaf", [(1, 3000, 64), (1, 9000, 100), (700, 50, 8), (3, 20000, 64)])
def test_body_pair_count(fmm, precision, count, n, n_leaf):
    """The near field's body pairs are those of its list."""
    pos, _, mass = W.plummer(count * n, 21)
    print(f"[gpu] body pairs {count} x {n} n_leaf={n_leaf} {precision}", flush=True)
    f = fmm.FMM(p=4, err_tol=1e-5, n_leaf=n_leaf, precision=precision)
    for _ in range(2):
        f.forces_batch(_dev(pos), _dev(mass), np.arange(count + 1) * n)
    size = f.export("cell_end").astype(np.int64) - f.export("cell_begin")
    p2p = f.export("p2p")
    assert f.stats()["n_p2p_pairs"] == (size[p2p[:, 0]] * size[p2p[:, 1]]).sum() - count * n
    f.close()


# leaves of more than 64 bodies (512 from 2048 leaves on) take a workgroup of eight
# wavefronts each, others one wavefront
@pytest.mark.parametrize("p", [1, 3, 10, 15, 16, 21, 30])
@pytest.mark.parametrize("n,n_leaf,copies", [(1000, 1024, 0), (1500, 200, 65), (30000, 8, 600)])
def test_upward_large_leaves(fmm, p, n, n_leaf, copies):
    """Multipoles and norms of the oracle, bit for bit: leaves about the bounds,
    by n_leaf and by coincident bodies, beside small ones."""
    pos, mass = W.uniform_cube(n, 50 + n)
    pos[100:100 + copies] = pos[100]
    pos[200 + copies:264 + copies] = pos[99]
    mass[::9] = 0.0
    print(f"[gpu] upward p={p} n={n} n_leaf={n_leaf} copies={copies}", flush=True)
    f = fmm.FMM(p=p, n_leaf=n_leaf)
    f.build(_dev(pos), _dev(mass))
    assert copies < 600 or f.stats()["nleaf"] > 2048
    o = oracle.Oracle()
    o.run(pos, mass, p=p, err_tol=1e-7, n_leaf=n_leaf, stage="upward")
    assert np.array_equal(f.export("mult"), o.get("mult"))
    assert np.array_equal(f.export("pk"), o.get("pk"))
    f.close()


@pytest.mark.parametrize("n,n_leaf,kind", [(530000, 1024, "cube"), (600001, 1000, "mixed")])
def test_estimate_of_large_leaves(fmm, n, n_leaf, kind):
    """Up to 4096 leaves that hold more than 8192 blocks of 64 bodies: the sums of
    leaves of 64 and more (a lane per body) and of the others, each body's in the
    defining order, so bit for bit the running sums of its list in numpy."""
    pos, mass = W.uniform_cube(n, 7)
    if kind == "mixed":  # leaves of all sizes, coincident bodies, no mass
        pos[:n // 2] *= 0.2
        pos[5:25] = pos[5]
        mass[::3] = 0.0
    print(f"[gpu] estimate of large leaves n={n} n_leaf={n_leaf}", flush=True)
    f = fmm.FMM(p=1, err_tol=1.0, n_leaf=n_leaf)
    f.forces(_dev(pos), _dev(mass))
    assert f.stats()["nleaf"] <= 4096
    perm = f.export("perm").astype(np.int64)
    x, m = pos[perm], mass[perm]
    cb, ce, parent = f.export("cell_begin"), f.export("cell_end"), f.export("cell_parent")
    far, fpart, near = f.export("fcell_est"), f.export("f_part"), f.export("est_near").astype(np.int64)
    size = ce - cb
    leaves = np.unique(near[:, 0])
    picked = [leaves[size[leaves] == k][0] for k in np.unique(size[leaves])[::max(1, n_leaf // 12)]]
    picked += [leaves[np.argmax(size[leaves])], leaves[np.argmin(size[leaves])]]
    assert max(size[c] for c in picked) > 64
    for c in picked:
        sources = near[near[:, 0] == c, 1]
        j = np.concatenate([np.arange(cb[a], ce[a]) for a in sources])
        top, path = 0.0, []
        q = c
        while q >= 0:
            path.append(q)
            q = parent[q]
        for q in path[::-1]:
            top = top + far[q]
        for i in {int(cb[c]), int(ce[c]) - 1, int(cb[c]) + int(size[c]) // 2}:
            d = x[j] - x[i]
            d2 = (d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2]
            term = np.where(d2 > 0.0, m[j] / np.where(d2 > 0.0, d2, 1.0), 0.0)
            assert fpart[i] == top + np.cumsum(term)[-1], (c, i)
    f.close()
