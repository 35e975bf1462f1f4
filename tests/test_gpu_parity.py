"""Parity of the HIP path (through the C ABI) with the CPU oracle.

The contract is bit equality: offspring genotypes, objectives, descriptors,
cells and the whole archive after every generation.  The tolerances the method
asks for (1e-5 relative for genotypes/objectives/descriptors, bit-exact cells
and insertion outcomes, 1e-4 relative end-to-end QD-score) are therefore met
with margin; the assertions below check equality and, separately, those
tolerances.

Sizes: small configurations that the oracle runs in seconds but that still
span several 256-gene chunks, a ragged last chunk and several waves, plus the
full benchmark shapes checked on sampled offspring.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2202_01258_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def qd():
    from paper_2202_01258_amd import qd as Q
    return Q


def say(msg):
    print(msg, flush=True)


def assert_archive_equal(gpu, ora, n, what=""):
    np.testing.assert_array_equal(gpu["occ"], ora["occ"], err_msg=f"occupancy {what}")
    filled = ora["occ"] == 1
    np.testing.assert_array_equal(gpu["fit"][filled], ora["fit"][filled], err_msg=f"fit {what}")
    np.testing.assert_array_equal(gpu["desc"][filled], ora["desc"][filled], err_msg=f"desc {what}")
    np.testing.assert_array_equal(gpu["geno"][filled, :n], ora["geno"][filled, :n],
                                  err_msg=f"genotypes {what}")


def rel_err(a, b, floor):
    a = np.asarray(a, np.float64)
    b = np.asarray(b, np.float64)
    return np.max(np.abs(a - b) / np.maximum(np.abs(b), floor)) if a.size else 0.0


SMALL = {
    "rastrigin_grid_b128": dict(),
    "sphere_grid_b16384": dict(batch=1000),
    "rastrigin_proj_cvt_b65536": dict(batch=600),
    "rastrigin_ragged": dict(n=257, batch=77),
    # projection descriptors spread over the whole box: few genes drawn from the
    # full range, so the nearest-centroid search meets most fine buckets
    "proj_spread_cvt": dict(n=8, batch=3000, C=2000, init_lo=-5.12, init_hi=5.12, seed=3),
    # the same on a Lloyd CVT (centroids moved by three Lloyd iterations)
    "proj_spread_lloyd": dict(n=8, batch=2000, C=500, init_lo=-5.12, init_hi=5.12, seed=4,
                              cvt_samples=20000, cvt_iters=3),
    # a short genotype (two offspring per wave) on a CVT, descriptors over the
    # whole box: the (theta_0, theta_1) descriptor through the candidate lists
    "sphere_cvt_spread": dict(tess=W.CVT, C=500, grid=(0, 0), batch=300, init_lo=-5.12,
                              init_hi=5.12, seed=6),
}


def small_workload(name):
    if name == "rastrigin_ragged":
        return W.workload("rastrigin_grid_b128", n=257, batch=77, seed=5)
    if name in ("proj_spread_cvt", "proj_spread_lloyd"):
        return W.workload("rastrigin_proj_cvt_b65536", **SMALL[name])
    if name == "sphere_cvt_spread":
        return W.workload("sphere_grid_b16384", **SMALL[name])
    return W.workload(name, **SMALL[name])


@pytest.mark.parametrize("name", list(SMALL))
def test_first_batch_bit_exact(name):
    w = small_workload(name)
    say(f"first batch {name} n={w['n']} batch={w['batch']}")
    a = qd().Archive(w, keep_offspring=True)
    gb = a.last_batch()
    o = O.Oracle(w)
    o.init()
    ob = o.last_batch()
    np.testing.assert_array_equal(gb["geno"], o.last_offspring())
    np.testing.assert_array_equal(gb["fit"], ob["fit"])
    np.testing.assert_array_equal(gb["desc"], ob["desc"])
    np.testing.assert_array_equal(gb["cell"], ob["cell"])
    np.testing.assert_array_equal(gb["won"], ob["won"])
    assert_archive_equal(a.snapshot(), o.archive(), o.n, "after the first batch")
    if w["tess"] == W.CVT:
        np.testing.assert_array_equal(a.views()["centroids"].cpu().numpy(), o.centroids())


@pytest.mark.parametrize("C,D,S,L", [(64, 2, 3000, 5), (37, 4, 2000, 3), (1500, 2, 7777, 1),
                                     (1000, 2, 20000, 2), (300, 4, 5000, 2)])
def test_lloyd_centroids_bit_exact(C, D, S, L):
    """Centroids after L Lloyd iterations over S points (several LDS tiles of
    centroids, ragged point and tile counts) equal the oracle's."""
    base = "rastrigin_proj_cvt_b65536" if D == 2 else "mlp64_cvt_b8192"
    w = W.workload(base, C=C, batch=16, cvt_samples=S, cvt_iters=L, seed=2)
    say(f"lloyd C={C} D={D} S={S} L={L}")
    a = qd().Archive(w)
    o = O.Oracle(w)
    o.setup()
    got = a.views()["centroids"].cpu().numpy()
    np.testing.assert_array_equal(got, o.centroids())
    plain = W.workload(base, C=C, batch=16, seed=2)
    q = O.Oracle(plain)
    q.setup()
    assert np.any(got != q.centroids()), "Lloyd iterations moved no centroid"


@pytest.mark.parametrize("task,n,nb", [
    # one offspring per wave: block and chunk ends of the genotype and of its half
    (W.RASTRIGIN_PROJ, 2, 1), (W.RASTRIGIN_PROJ, 7, 3), (W.RASTRIGIN_PROJ, 255, 5), (W.RASTRIGIN_PROJ, 258, 5),
    (W.RASTRIGIN_PROJ, 514, 9), (W.RASTRIGIN_PROJ, 1029, 3), (W.RASTRIGIN, 128, 2), (W.SPHERE, 129, 3),
    # two per wave, the last wave with one
    (W.RASTRIGIN, 30, 2049), (W.RASTRIGIN_PROJ, 131, 2051), (W.SPHERE, 260, 2049),
    # four per wave, the last wave with one, two and three
    (W.SPHERE, 5, 8193), (W.RASTRIGIN, 127, 8195), (W.RASTRIGIN, 133, 8194), (W.RASTRIGIN_PROJ, 250, 8193),
    (W.RASTRIGIN_PROJ, 777, 8195), (W.RASTRIGIN_PROJ, 3, 8194), (W.RASTRIGIN_PROJ, 127, 8193),
    (W.RASTRIGIN_PROJ, 128, 8195), (W.SPHERE, 399, 8194), (W.RASTRIGIN, 513, 8195),
])
def test_genes_ragged(task, n, nb):
    """Ragged genotype lengths and batches, with kept genotypes, against the
    oracle: the first batch and one generation."""
    w = W.workload("rastrigin_proj_cvt_b65536", task=task, n=n, batch=nb, C=300, seed=11,
                   init_lo=-5.12, init_hi=5.12)
    say(f"ragged genes task={task} n={n} N_B={nb}")
    a = qd().Archive(w, keep_offspring=True)
    o = O.Oracle(w)
    o.init()
    for g in (0, 1):
        if g:
            a.generation(g)
            o.generation(g)
        gb, ob = a.last_batch(), o.last_batch()
        np.testing.assert_array_equal(gb["geno"], o.last_offspring(), err_msg=f"generation {g}")
        for k in ("fit", "desc", "cell", "won"):
            np.testing.assert_array_equal(gb[k], ob[k], err_msg=f"{k} of generation {g}")
    assert_archive_equal(a.snapshot(), o.archive(), o.n, "after one generation")


@pytest.mark.parametrize("grid,nb", [
    ((1, 1), 3), ((7, 1), 40), ((1, 9), 200),               # 8 cells per workgroup: its ends,
    ((128, 128), 8192),                                     # the last cell count and batch that take it
    ((128, 128), 8191), ((145, 113), 20000),                # 32: the first batch and cell count past those
    ((31, 1), 14), ((32, 1), 15), ((33, 1), 15), ((65, 1), 31),
])
def test_winner_kernel_cells_per_workgroup(grid, nb):
    """Both choices of cells per workgroup at the ends of their ranges: first
    batch and three generations against the oracle."""
    w = W.workload("rastrigin_grid_b128", n=7, batch=nb, grid=grid, C=grid[0] * grid[1], seed=9,
                   init_lo=-5.12, init_hi=5.12)
    say(f"winner kernel grid={grid} N_B={nb}")
    a = qd().Archive(w)
    o = O.Oracle(w)
    o.init()
    for g in range(4):
        if g:
            a.generation(g)
            o.generation(g)
        gb, ob = a.last_batch(), o.last_batch()
        for k in ("fit", "desc", "cell", "won"):
            np.testing.assert_array_equal(gb[k], ob[k], err_msg=f"{k} of generation {g}")
    assert_archive_equal(a.snapshot(), o.archive(), o.n, "after three generations")


@pytest.mark.parametrize("C,S,L", [
    (1, 10, 1), (2, 1, 2), (3, 100, 3), (5, 4000, 2),      # grids of one and two buckets a side
    (5, (1 << 20) - 1, 1), (5, 1 << 20, 1), (5, (1 << 20) + 1, 2),   # count in a sum's word, and apart
    (4100, 255, 4), (4100, 30001, 1),                      # most cells without points; many rings
])
def test_lloyd_lists_bit_exact(C, S, L):
    """Lloyd's lists per bucket in two dimensions at the ends of their ranges:
    centroids and first batch against the oracle (brute force)."""
    w = W.workload("rastrigin_proj_cvt_b65536", n=16, C=C, batch=300, cvt_samples=S, cvt_iters=L,
                   seed=3, init_lo=-5.12, init_hi=5.12)
    say(f"lloyd lists C={C} S={S} L={L}")
    a = qd().Archive(w)
    o = O.Oracle(w)
    o.init()
    np.testing.assert_array_equal(a.views()["centroids"].cpu().numpy(), o.centroids())
    np.testing.assert_array_equal(a.last_batch()["cell"], o.last_batch()["cell"])


@pytest.mark.parametrize("D", [2, 4])
@pytest.mark.parametrize("S", [(1 << 20) - 1, 1 << 20, (1 << 20) + 1])
def test_lloyd_count_of_one_cell_at_the_packed_limit(D, S):
    """One cell gets all the points: its count and sums at and around the number
    of points from which the count has a word of its own."""
    base = "rastrigin_proj_cvt_b65536" if D == 2 else "mlp64_cvt_b8192"
    w = W.workload(base, C=1, batch=16, cvt_samples=S, cvt_iters=1, seed=2)
    say(f"lloyd one cell D={D} S={S}")
    a = qd().Archive(w)
    o = O.Oracle(w)
    o.setup()
    np.testing.assert_array_equal(a.views()["centroids"].cpu().numpy(), o.centroids())


@pytest.mark.parametrize("C,L", [(1, 0), (2, 0), (3, 2), (37, 0), (500, 3), (3003, 0)])
def test_cvt_candidate_lists_complete(C, L):
    """A fine bucket's count and list are those of the definition worked out
    over every centroid in double: nearest-point distance to the padded box at
    most the smallest farthest-corner distance, in ascending index."""
    w = W.workload("rastrigin_proj_cvt_b65536", n=16, C=C, batch=16, seed=5,
                   cvt_samples=2000 if L else 0, cvt_iters=L)
    say(f"candidate lists against the definition, C={C} L={L}")
    a = qd().Archive(w)
    v = a.views()
    R = a.layout.cand_res
    cnt, pts = v["cand_count"].cpu().numpy(), v["cand_pts"].cpu().numpy()
    cent = v["centroids"].cpu().numpy().astype(np.float64)
    for b in range(R * R):
        # the box as the kernel forms it: w = 1 / R, padded by 1e-6
        box = [((i * (1.0 / R)) - 1e-6, (i + 1) * (1.0 / R) + 1e-6) for i in (b // R, b % R)]
        far = sum(np.maximum(cent[:, k] - lo, hi - cent[:, k]) ** 2 for k, (lo, hi) in enumerate(box))
        near = sum(np.maximum(0.0, np.maximum(lo - cent[:, k], cent[:, k] - hi)) ** 2
                   for k, (lo, hi) in enumerate(box))
        want = np.nonzero(near <= far.min() * (1.0 + 1e-5) + 1e-12)[0]
        assert cnt[b] == len(want), (b, cnt[b], len(want))
        if len(want) <= qd().CAND_SLOTS:
            np.testing.assert_array_equal(pts[b, : len(want), 2].view(np.int32), want)
            np.testing.assert_array_equal(pts[b, : len(want), :2], cent[want].astype(np.float32))


@pytest.mark.parametrize("C,seed", [(10000, 0), (2000, 3), (37, 1)])
def test_cvt_candidate_lists_hold_the_nearest_centroid(C, seed):
    """Every listed fine bucket holds, in ascending order, the brute-force
    nearest centroid (the oracle's) of points all over it: random points,
    bucket corners and points one fp32 step either side of bucket edges."""
    w = W.workload("rastrigin_proj_cvt_b65536", C=C, batch=64, seed=seed)
    say(f"candidate lists C={C} seed={seed}")
    a = qd().Archive(w)
    v = a.views()
    R = a.layout.cand_res
    assert R > 0 and R * R <= 4 * C < (R + 1) * (R + 1)
    cnt = v["cand_count"].cpu().numpy()
    pts = v["cand_pts"].cpu().numpy()
    cent = v["centroids"].cpu().numpy()
    assert cnt.min() >= 1
    assert (cnt <= qd().CAND_SLOTS).mean() > 0.999
    o = O.Oracle(w)
    o.setup()
    np.testing.assert_array_equal(cent, o.centroids())
    rng = np.random.default_rng(seed)
    edges = (np.arange(R + 1) / R).astype(np.float32)
    near = np.concatenate([edges, np.nextafter(edges, np.float32(0)),
                           np.nextafter(edges, np.float32(1))]).clip(0, 1)
    u = np.concatenate([
        rng.random((4000, 2), dtype=np.float32),
        np.stack([rng.choice(near, 4000), rng.random(4000, dtype=np.float32)], 1),
        np.stack([rng.random(4000, dtype=np.float32), rng.choice(near, 4000)], 1),
        np.stack([rng.choice(near, 2000), rng.choice(near, 2000)], 1),
    ]).astype(np.float32)
    lo, hi = np.float32(-5.12), np.float32(5.12)
    span = np.float32(hi - lo)
    for k, (u0, u1) in enumerate(u):
        d = (np.float32(u0) * span + lo, np.float32(u1) * span + lo)
        d = np.clip(np.array(d, np.float32), lo, hi)
        best = O.cvt_cell(d, w["lo"], w["hi"], cent)
        un = (d - lo) / span
        q = np.minimum(np.floor(un * np.float32(R)), R - 1).astype(int)
        b = q[0] * R + q[1]
        if cnt[b] > qd().CAND_SLOTS:
            continue
        listed = pts[b, :cnt[b], 2].view(np.int32)
        assert np.all(np.diff(listed) > 0), (b, listed)
        assert best in listed, (k, d, b, best, listed)


@pytest.mark.parametrize("name", list(SMALL))
def test_generations_driven_bit_exact(name):
    """Each generation: offspring from the GPU's own pre-generation archive,
    then cells and insertion driven from the GPU's objectives/descriptors."""
    w = small_workload(name)
    a = qd().Archive(w, keep_offspring=True)
    o = O.Oracle(w)
    o.setup()
    for g in range(1, 6):
        say(f"driven {name} generation {g}")
        pre = a.snapshot()
        a.generation(g)
        gb = a.last_batch()
        o.set_archive(pre["geno"], pre["fit"], pre["desc"], pre["occ"])
        for j in range(w["batch"]):
            geno, fit, desc, par = o.offspring(g, j)
            np.testing.assert_array_equal(par, gb["parents"][j], err_msg=f"parents j={j}")
            np.testing.assert_array_equal(gb["geno"][j], geno, err_msg=f"genotype j={j}")
            assert gb["fit"][j] == fit, (j, gb["fit"][j], fit)
            np.testing.assert_array_equal(gb["desc"][j], desc, err_msg=f"desc j={j}")
        cell, won = o.insert_driven(gb["fit"], gb["desc"], gb["geno"])
        np.testing.assert_array_equal(gb["cell"], cell)
        np.testing.assert_array_equal(gb["won"], won)
        assert_archive_equal(a.snapshot(), o.archive(), o.n, f"after generation {g}")


@pytest.mark.parametrize("name,kw,G", [
    ("rastrigin_grid_b128", {}, 100),                        # the full configuration
    ("sphere_grid_b16384", dict(batch=2048), 40),
    ("sphere_grid_b16384", {}, 500),                         # the full configuration
    ("rastrigin_proj_cvt_b65536", dict(batch=2048), 12),
    ("rastrigin_proj_cvt_b65536", {}, 3),                    # the benchmark configuration
    # its shape with a spread first batch: ~10^4 filled cells, distinct parents
    ("rastrigin_proj_cvt_b65536_spread", {}, 3),
    # first batch over the whole box: thousands of new cells and winners in
    # every early generation (regeneration and compaction at full load)
    ("rastrigin_grid_b128", dict(batch=4096, init_lo=-5.12, init_hi=5.12, seed=2), 40),
    ("sphere_grid_b16384", dict(batch=4096, init_lo=-5.12, init_hi=5.12, seed=3), 10),
    # the generation kernel's offspring-per-wave thresholds (one up to 2048, two
    # up to 8192, four above), each side, with ragged last waves
    ("rastrigin_grid_b128", dict(batch=2049, init_lo=-5.12, init_hi=5.12, seed=4), 20),
    ("sphere_grid_b16384", dict(batch=8192, init_lo=-5.12, init_hi=5.12, seed=6), 10),
    ("rastrigin_proj_cvt_b65536", dict(batch=8193, n=300, seed=5), 3),
])
def test_end_to_end_qd_score(name, kw, G):
    w = W.workload(name, **kw)
    say(f"end to end {name} {kw} G={G}")
    a = qd().Archive(w)
    o = O.Oracle(w)
    o.init()
    for g in range(1, G + 1):
        a.generation(g)
        o.generation(g)
    gs, os_ = a.stats(), o.stats()
    assert gs["num_occupied"] == os_["coverage"]
    assert abs(gs["qd_score"] - os_["qd_score"]) <= 1e-4 * abs(os_["qd_score"])
    assert gs["qd_score"] == pytest.approx(os_["qd_score"], rel=1e-12)
    assert gs["best"] == np.float32(os_["best"])
    assert_archive_equal(a.snapshot(), o.archive(), o.n, f"after {G} generations")


def test_keep_offspring_does_not_change_the_path():
    w = W.workload("rastrigin_proj_cvt_b65536", batch=1500)
    a0 = qd().Archive(w, keep_offspring=False)
    a1 = qd().Archive(w, keep_offspring=True)
    for g in range(1, 4):
        a0.generation(g)
        a1.generation(g)
    s0, s1 = a0.snapshot(), a1.snapshot()
    for k in ("key", "fit", "desc", "geno"):
        np.testing.assert_array_equal(s0[k], s1[k])


def test_replay_is_deterministic():
    w = W.workload("sphere_grid_b16384", batch=3000)
    a = qd().Archive(w)
    a.generation(1)
    b = qd().Archive(w)
    b.generation(1)
    for k in ("key", "fit", "desc", "geno", "occ_list"):
        np.testing.assert_array_equal(a.snapshot()[k], b.snapshot()[k])


@pytest.mark.parametrize("name,kw", [("sphere_grid_b16384", dict(batch=3000)),
                                     ("mlp64_cvt_b8192", dict(batch=24, T=20))])
def test_generations_in_one_call_equal_single_calls(name, kw):
    """qd_generations(first, count) leaves the archive and the last batch
    exactly as count qd_generation() calls do."""
    w = W.workload(name, **kw)
    say(f"generations in one call: {name} {kw}")
    a = qd().Archive(w, keep_offspring=True)
    for g in range(1, 6):
        a.generation(g)
    b = qd().Archive(w, keep_offspring=True)
    b.generations(1, 5)
    b.generations(6, 0)                  # count 0: nothing
    sa, sb = a.snapshot(), b.snapshot()
    for k in ("key", "fit", "desc", "geno", "occ_list"):
        np.testing.assert_array_equal(sa[k], sb[k], err_msg=k)
    la, lb = a.last_batch(), b.last_batch()
    for k in ("geno", "fit", "desc", "cell", "won"):
        np.testing.assert_array_equal(la[k], lb[k], err_msg=k)


def check_driven_generation(a, o, w, g):
    """Runs generation g on the GPU from its current archive and checks it
    against the oracle started from the same archive: every offspring's cell
    and the whole insertion, sampled offspring, and the winners' rows."""
    pre = a.snapshot()
    a.generation(g)
    gb = a.last_batch()
    o.set_archive(pre["geno"], pre["fit"], pre["desc"], pre["occ"])
    rng = np.random.default_rng(g)
    for j in np.concatenate([[0, 1, w["batch"] - 1], rng.integers(0, w["batch"], 12)]):
        geno, fit, desc, par = o.offspring(g, int(j))
        np.testing.assert_array_equal(par, gb["parents"][j])
        assert gb["fit"][j] == fit
        np.testing.assert_array_equal(gb["desc"][j], desc)
    # the winners' genotypes, made by the oracle from the archive before the
    # insertion (afterwards new cells would change the selection)
    winners = np.nonzero(gb["won"])[0][:8]
    expect = {int(j): o.offspring(g, int(j))[0] for j in winners}
    cell, won = o.insert_driven(gb["fit"], gb["desc"])
    np.testing.assert_array_equal(gb["cell"], cell)
    np.testing.assert_array_equal(gb["won"], won)
    post = a.snapshot()
    oa = o.archive()
    np.testing.assert_array_equal(post["occ"], oa["occ"])
    filled = oa["occ"] == 1
    np.testing.assert_array_equal(post["fit"][filled], oa["fit"][filled])
    np.testing.assert_array_equal(post["desc"][filled], oa["desc"][filled])
    # winners' rows: regenerated on the GPU, recomputed here
    for j, geno in expect.items():
        np.testing.assert_array_equal(post["geno"][gb["cell"][j]], geno)
    # the tolerance the method states, for the record
    assert rel_err(post["fit"][filled], oa["fit"][filled], 1e-6) <= 1e-5
    return int(won.sum())


@pytest.mark.parametrize("name,batch", [("rastrigin_proj_cvt_b65536", 65536),
                                        ("rastrigin_proj_cvt_b65536", 131072),
                                        ("rastrigin_proj_cvt_b65536_spread", 65536)])
def test_full_size_rastrigin_projection_sampled(name, batch):
    """n = 1000, CVT 10^4 at N_B = 65536 (the benchmark's launch configuration)
    and at 131072 (the top of the batch-size sweep), and the same shape with
    a spread first batch (nearly every cell filled, thousands of winners per
    generation).  Every offspring's cell and the whole insertion are checked
    (driven), and sampled offspring genotypes/objectives/descriptors from the
    oracle."""
    w = W.workload(name, batch=batch)
    say(f"full size rastrigin projection N_B={batch}: init")
    a = qd().Archive(w)
    o = O.Oracle(w)
    o.setup()
    np.testing.assert_array_equal(a.views()["centroids"].cpu().numpy(), o.centroids())
    for g in (1, 2):
        say(f"full size rastrigin projection: generation {g}")
        check_driven_generation(a, o, w, g)


def test_benchmark_configuration_at_generation_200_driven():
    """The benchmark configuration run on the GPU alone for the paper's 199
    generations, then generation 200 checked against the oracle from the
    archive the GPU reached: parity deep into the run that is timed."""
    w = W.workload("rastrigin_proj_cvt_b65536")
    say("benchmark configuration: init, 199 free-running generations")
    a = qd().Archive(w)
    a.generations(1, 199)
    o = O.Oracle(w)
    o.setup()
    say("benchmark configuration: generation 200, driven")
    check_driven_generation(a, o, w, 200)
    assert a.stats()["num_occupied"] >= 1


MLP_SMALL = {
    "mlp64_cvt_b8192": ("mlp64_cvt_b8192", dict(batch=48, T=250)),
    "mlp128_cvt_b65536": ("mlp128_cvt_b65536", dict(batch=16, T=40, C=500)),
    # failure at new-state component 0 below a threshold: at -0.05 (h = 64)
    # 28 of the 64 first-batch episodes fail at the first step (death flags
    # in both modes), 3 later (truncated, or flagged when discarding) and 33
    # run to the end; at -0.03 (h = 128, two waves) 14 of 24 fail at the
    # first step, 6 later and 4 run to the end
    "mlp64_death_truncate": ("mlp64_cvt_b8192",
                             dict(batch=64, T=60, death_mode=1, death_below=-0.05)),
    "mlp64_death_discard": ("mlp64_cvt_b8192",
                            dict(batch=64, T=60, death_mode=2, death_below=-0.05)),
    "mlp128_death_truncate": ("mlp128_cvt_b65536",
                              dict(batch=24, T=40, C=500, death_mode=1, death_below=-0.03)),
    "mlp128_death_discard": ("mlp128_cvt_b65536",
                             dict(batch=24, T=40, C=500, death_mode=2, death_below=-0.03)),
    # a batch that is not a multiple of the 16 offspring an LDS-CVT insertion
    # workgroup takes, on a CVT smaller than one centroid per lane
    "mlp64_odd_batch_small_cvt": ("mlp64_cvt_b8192", dict(batch=37, T=12, C=13)),
    # the largest CVT whose centroids the insertion stages in LDS, and the
    # smallest one searched by rings instead
    "mlp64_cvt_2048_lds": ("mlp64_cvt_b8192", dict(batch=40, T=8, C=2048)),
    "mlp64_cvt_2049_rings": ("mlp64_cvt_b8192", dict(batch=40, T=8, C=2049)),
    # policies on a 4-D grid of 5^4 cells (grid insertion with D = 4); the
    # box is narrowed around 0.5, where these descriptors lie, so the batch
    # spreads over 17 cells and reaches 85 in three generations
    "mlp64_grid_4d": ("mlp64_cvt_b8192", dict(batch=40, T=20, tess=W.GRID, grid=(5, 5, 5, 5),
                                              C=625, lo=(0.498,) * 4, hi=(0.502,) * 4)),
}


@pytest.mark.parametrize("name", list(MLP_SMALL))
def test_mlp_bit_exact(name):
    base, kw = MLP_SMALL[name]
    w = W.workload(base, **kw)
    say(f"mlp {name} {kw}: first batch")
    a = qd().Archive(w, keep_offspring=True)
    o = O.Oracle(w)
    o.init()
    np.testing.assert_array_equal(a.views()["env"].cpu().numpy()[: o.env_len], o.env())
    gb, ob = a.last_batch(), o.last_batch()
    np.testing.assert_array_equal(gb["geno"], o.last_offspring())
    np.testing.assert_array_equal(gb["fit"], ob["fit"])
    np.testing.assert_array_equal(gb["desc"], ob["desc"])
    np.testing.assert_array_equal(gb["cell"], ob["cell"])
    assert_archive_equal(a.snapshot(), o.archive(), o.n, "first batch")
    deaths = int(np.isnan(gb["fit"]).sum())
    for g in (1, 2, 3):
        say(f"mlp {name}: generation {g}")
        a.generation(g)
        o.generation(g)
        gb, ob = a.last_batch(), o.last_batch()
        np.testing.assert_array_equal(gb["geno"], o.last_offspring())
        np.testing.assert_array_equal(gb["fit"], ob["fit"])
        np.testing.assert_array_equal(gb["desc"], ob["desc"])
        np.testing.assert_array_equal(gb["won"], ob["won"])
        assert_archive_equal(a.snapshot(), o.archive(), o.n, f"generation {g}")
    assert a.stats()["qd_score"] == pytest.approx(o.stats()["qd_score"], rel=1e-12)
    if w.get("death_mode", 0):
        # the failure rule was exercised: the first batch holds death flags
        assert deaths > 0


@pytest.mark.parametrize("name,batch,T,keep,death", [
    ("mlp64_cvt_b8192", 1, 1, True, 0),        # one individual, a spare wave beside it
    ("mlp64_cvt_b8192", 5, 64, False, 0),      # odd batch; exactly one ring of steps
    ("mlp64_cvt_b8192", 64, 65, True, 1),
    ("mlp128_cvt_b65536", 1, 63, False, 0),    # eight waves per individual
    ("mlp128_cvt_b65536", 256, 3, True, 2),    # its largest batch
    ("mlp128_cvt_b65536", 40, 129, False, 1),
    ("mlp128_cvt_b65536", 257, 66, False, 2),  # two waves per individual
])
def test_mlp_waves_per_individual(name, batch, T, keep, death):
    """Each choice of waves per individual at the ends of its range and at
    episode lengths around the reward ring's size, against the oracle."""
    w = W.workload(name, batch=batch, T=T, C=200, death_mode=death, death_below=-0.06)
    say(f"waves per individual: {name} N_B={batch} T={T} keep={keep} death={death}")
    a = qd().Archive(w, keep_offspring=keep)
    o = O.Oracle(w)
    o.init()
    for g in (0, 1, 2):
        if g:
            a.generation(g)
            o.generation(g)
        gb, ob = a.last_batch(), o.last_batch()
        if keep:
            np.testing.assert_array_equal(gb["geno"], o.last_offspring())
        for k in ("fit", "desc", "cell", "won"):
            np.testing.assert_array_equal(gb[k], ob[k], err_msg=f"{k} of generation {g}")
    assert_archive_equal(a.snapshot(), o.archive(), o.n, "after two generations")


@pytest.mark.parametrize("name,batch,samples", [("mlp64_cvt_b8192", 8192, 6),
                                                ("mlp64_cvt_b8192", 131072, 4),
                                                ("mlp128_cvt_b65536", 65536, 2)])
def test_mlp_full_size_sampled(name, batch, samples):
    """The full policy shapes (N_B 8192 / 65536, T 250 / 1000) and the h = 64
    shape at the top of the batch-size sweep: sampled offspring rollouts
    against the oracle, all cells and insertion driven."""
    w = W.workload(name, batch=batch)
    say(f"mlp full size {name} N_B={batch}: init")
    a = qd().Archive(w)
    o = O.Oracle(w)
    o.setup()
    np.testing.assert_array_equal(a.views()["env"].cpu().numpy()[: o.env_len], o.env())
    say(f"mlp full size {name}: generation 1")
    pre = a.snapshot()
    a.generation(1)
    gb = a.last_batch()
    o.set_archive(pre["geno"], pre["fit"], pre["desc"], pre["occ"])
    rng = np.random.default_rng(0)
    for j in np.concatenate([[0, w["batch"] - 1], rng.integers(0, w["batch"], samples - 2)]):
        say(f"  oracle rollout j={j}")
        geno, fit, desc, par = o.offspring(1, int(j))
        np.testing.assert_array_equal(par, gb["parents"][j])
        assert gb["fit"][j] == fit, (j, gb["fit"][j], fit)
        np.testing.assert_array_equal(gb["desc"][j], desc)
    cell, won = o.insert_driven(gb["fit"], gb["desc"])
    np.testing.assert_array_equal(gb["cell"], cell)
    np.testing.assert_array_equal(gb["won"], won)
    post, oa = a.snapshot(), o.archive()
    np.testing.assert_array_equal(post["occ"], oa["occ"])
    filled = oa["occ"] == 1
    np.testing.assert_array_equal(post["fit"][filled], oa["fit"][filled])


@pytest.mark.parametrize("name,G,count", [("mlp64_cvt_b8192", 100, None),
                                          ("mlp128_cvt_b65536", 50, 512)])
def test_policy_configuration_at_last_generation_driven(name, G, count):
    """A policy configuration (27-64-64-8, T = 250, N_B = 8192; 27-128-128-8,
    T = 1000, N_B = 65536) run on the GPU alone for the paper's G - 1
    generations, then generation G checked from the archive the GPU reached:
    rollouts against the oracle's (all 8192 of the first configuration, 512
    of the second; the oracle runs them on every host thread), every cell
    and the insertion, and the winners' regenerated rows."""
    w = W.workload(name)
    say(f"policy configuration {name}: init, {G - 1} free-running generations")
    a = qd().Archive(w)
    a.generations(1, G - 1)
    o = O.Oracle(w)
    o.setup()
    g = G
    say(f"policy configuration {name}: generation {G}, driven")
    pre = a.snapshot()
    a.generation(g)
    gb = a.last_batch()
    o.set_archive(pre["geno"], pre["fit"], pre["desc"], pre["occ"])
    rng = np.random.default_rng(g)
    js = (np.arange(w["batch"]) if count is None else
          np.unique(np.concatenate([[0, w["batch"] - 1], rng.integers(0, w["batch"], count)])))
    say(f"  oracle rollouts: {js.size} on {O.set_threads(0)} threads")
    fit, desc, par = o.offspring_many(g, js)
    np.testing.assert_array_equal(par, gb["parents"][js])
    np.testing.assert_array_equal(gb["fit"][js].view(np.uint32), fit.view(np.uint32))
    np.testing.assert_array_equal(gb["desc"][js], desc)
    # winners' genotypes from the archive before the insertion
    expect = {int(j): o.offspring(g, int(j))[0] for j in np.nonzero(gb["won"])[0][:4]}
    cell, won = o.insert_driven(gb["fit"], gb["desc"])
    np.testing.assert_array_equal(gb["cell"], cell)
    np.testing.assert_array_equal(gb["won"], won)
    post, oa = a.snapshot(), o.archive()
    np.testing.assert_array_equal(post["occ"], oa["occ"])
    filled = oa["occ"] == 1
    np.testing.assert_array_equal(post["fit"][filled], oa["fit"][filled])
    np.testing.assert_array_equal(post["desc"][filled], oa["desc"][filled])
    for j, geno in expect.items():
        np.testing.assert_array_equal(post["geno"][gb["cell"][j]], geno)


def test_policy_configuration_end_to_end():
    """27-64-64-8, T = 250, N_B = 8192, CVT 1024 (the configuration in full
    size) free-running for 4 generations on both sides: every rollout, the
    archive and the QD-score (1e-4 relative asked; equal here)."""
    G = 4
    w = W.workload("mlp64_cvt_b8192")
    say(f"policy configuration end to end, G={G}, oracle on {O.set_threads(0)} threads")
    a = qd().Archive(w)
    o = O.Oracle(w)
    o.init()
    for g in range(1, G + 1):
        a.generation(g)
        o.generation(g)
        say(f"  generation {g}")
        gb, ob = a.last_batch(), o.last_batch()
        np.testing.assert_array_equal(gb["fit"].view(np.uint32), ob["fit"].view(np.uint32))
        np.testing.assert_array_equal(gb["desc"], ob["desc"])
        np.testing.assert_array_equal(gb["won"], ob["won"])
    gs, os_ = a.stats(), o.stats()
    assert gs["num_occupied"] == os_["coverage"]
    assert abs(gs["qd_score"] - os_["qd_score"]) <= 1e-4 * abs(os_["qd_score"])
    assert gs["qd_score"] == pytest.approx(os_["qd_score"], rel=1e-12)
    assert_archive_equal(a.snapshot(), o.archive(), o.n, f"after {G} generations")


@pytest.mark.parametrize("kw", [dict(batch=1), dict(n=2, batch=5), dict(n=101, batch=9),
                                dict(C=1, grid=(1, 1), batch=33),
                                dict(n=65537, batch=6)])     # long rows with a ragged tail
def test_edge_shapes(kw):
    w = W.workload("rastrigin_grid_b128", **kw)
    say(f"edge shape {kw}")
    a = qd().Archive(w, keep_offspring=True)
    o = O.Oracle(w)
    o.init()
    for g in range(1, 4):
        a.generation(g)
        o.generation(g)
        np.testing.assert_array_equal(a.last_batch()["geno"], o.last_offspring())
    assert_archive_equal(a.snapshot(), o.archive(), o.n, f"{kw}")


def test_empty_archive_sets_the_flag_and_inserts_nothing():
    """Every first-batch policy fails at once (death flags): the archive stays
    empty, and the next generation reports the empty archive (flag bit 0)
    instead of selecting parents, with every offspring marked not inserted."""
    w = W.workload("mlp64_cvt_b8192", batch=16, T=5, C=64, death_mode=2,
                   death_below=float("inf"))
    say("empty archive")
    a = qd().Archive(w)
    st = a.stats()
    assert st["num_occupied"] == 0 and st["flags"] == 0 and np.isnan(st["best"])
    assert np.isnan(a.last_batch()["fit"]).all()
    o = O.Oracle(w)
    o.init()
    assert o.stats()["coverage"] == 0
    a.generation(1)
    gb = a.last_batch()
    assert np.isnan(gb["fit"]).all()
    assert (gb["parents"] == -1).all() and (gb["cell"] == -1).all() and not gb["won"].any()
    st = a.stats()
    assert st["num_occupied"] == 0 and st["flags"] & 1
    with pytest.raises(RuntimeError, match="empty archive"):
        o.generation(1)                   # the oracle finds no parent either


def test_fast_division_equals_ieee_on_all_inputs():
    """Short reciprocal sequences replace IEEE division in tanh and sigmoid;
    over every input each can receive they must reproduce the IEEE results
    bit for bit."""
    assert qd().check_fast_arith() == [0, 0]


def test_sampler_bit_exact_on_every_magnitude_and_both_signs():
    """All 2^24 magnitudes of the Gaussian sampler (every table row, including
    the tail rows a generation almost never reaches), each with a random
    choice of the unused bits 24..30 and both signs, against the oracle."""
    w = W.workload("sphere_grid_b16384", batch=64)
    a = qd().Archive(w)
    k = np.arange(1 << 24, dtype=np.uint32)
    mid = np.random.default_rng(11).integers(0, 128, size=k.size, dtype=np.uint32) << 24
    for sign in (0, 0x80000000):
        words = k | mid | np.uint32(sign)
        say(f"sampler: 2^24 words, sign bit {sign >> 31}")
        got = a.sample_normals(words)
        want = O.normal(words)
        np.testing.assert_array_equal(got.view(np.uint32), want.view(np.uint32))
    # a count that is not a multiple of the workgroup size
    words = np.random.default_rng(12).integers(0, 2**32, size=1001, dtype=np.uint64).astype(np.uint32)
    np.testing.assert_array_equal(a.sample_normals(words).view(np.uint32),
                                  O.normal(words).view(np.uint32))


def test_normal_table_equals_the_oracle_table():
    """The Gaussian sampler's table that qd_archive_init builds on the host
    and copies into the workspace holds the oracle's bits (each side builds
    it with its own code)."""
    w = W.workload("sphere_grid_b16384", batch=64)
    a = qd().Archive(w)
    a.stream.synchronize()
    got = a.views()["normal_tab"].cpu().numpy()
    want = O.normal_table()
    np.testing.assert_array_equal(got.view(np.uint32), want.view(np.uint32))
