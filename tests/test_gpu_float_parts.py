"""Floats in three bf16 parts: the form of the float operands that the 16-bit matrix instructions multiply.  Asked for here
with the "float_form" option; by itself the library takes it where the estimates say that it is faster."""
import gc

import numpy as np
import pytest
import torch

import mmm_synth as synth
import oracle
import paper_2402_14118_amd as mm
from hip_harness import HipRun, assert_close
from test_gpu_parity import check_workload

pytestmark = pytest.mark.gpu

PLAIN, PARTS = 0, 1


@pytest.fixture(autouse=True)
def parts_on_the_matrix_path():
    mm.mmm_set_option("float_form", PARTS)
    mm.mmm_set_option("matmul_path", mm.MMM_PATH_MATRIX)
    yield
    mm.mmm_set_option("float_form", -1)
    mm.mmm_set_option("matmul_path", -1)


# ---- the edges of tiles, groups, segments, batches of 32 and the blocks of the ring ----------
@pytest.mark.parametrize("rows", [None, 0.6], ids=["all", "rows"])
@pytest.mark.parametrize("M,K,N,bw", [(65, 1, 8, 8), (65, 2, 136, 8), (128, 65, 272, 16), (129, 127, 256, 16), (129, 128, 288, 32),
                                      (66, 129, 264, 8), (190, 257, 544, 32), (70, 1030, 48, 16), (200, 8065, 32, 16)])
def test_edges(M, K, N, bw, rows):
    w = synth.random_masked(M, K, N, bw, 0.4, 0.4, 31 * M + K + N, dist="smallint", p_rows=rows)
    run, (_, _, C_ref, _, _) = check_workload(w, "edges", exact=True)
    run.eng.set_plan(-1, 3)
    run.Cbuf.fill_(float("nan"))
    run.matmul()
    run.matmul(accumulate=True)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(run.C.cpu().numpy(), 2 * C_ref)


@pytest.mark.parametrize("bw", [8, 16, 32])
def test_list_lengths(bw):
    lengths = [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 95, 97, 127, 128, 0]
    segs, N = 16, 256
    K, NB = segs * 128, N // bw
    keep = np.zeros((K, NB), bool)
    rng = np.random.default_rng(bw)
    for s in range(segs):
        for b in range(NB):
            keep[s * 128 + rng.permutation(128)[: lengths[(s + b * bw // max(16, bw)) % len(lengths)]], b] = True
    w = synth.random_masked(80, K, N, bw, 0.5, 1.0, 77 + bw, dist="smallint")
    w.keep_blocks = synth.pack_bits(keep)
    check_workload(w, "lengths", exact=True, ldx=K + 3, ldy=N + 5, ldc=N + 1)


@pytest.mark.parametrize("marked", [False, True], ids=["held", "marked"])
@pytest.mark.parametrize("bw,steps", [(16, 47), (32, 23), (8, 9), (16, 3), (16, 131), (8, 197), (32, 64), (16, 65)])
def test_joined_lists(bw, steps, marked):
    """Batches take units of eight slots from two neighbouring lists: lengths around whole units, and around the three that a step
    counts for at least; with every third block of A marked, whose step has no list for the batches around it.  Past 64 steps the
    lengths in hand are at times enough for a plan of 64 batches, at times for 46 and at times to be fetched anew."""
    lengths = [0, 7, 8, 9, 24, 25, 1, 16, 17, 120, 0, 0, 23, 31, 33, 32, 26, 56]
    K, N = steps * 128, 288
    rng = np.random.default_rng(bw + steps)
    keep = np.zeros((K, N // bw), bool)
    for s in range(steps):
        for b in range(N // bw):   # k = 5 of a segment is in no list
            k = s * 128 + rng.permutation(np.delete(np.arange(128), 5))[: lengths[(s + b * bw // max(16, bw) * 5) % len(lengths)]]
            keep[k, b] = True
    w = synth.random_masked(70, K, N, bw, 0.5, 1.0, 91 + bw, dist="smallint")
    if marked:
        w.X[:, 5::384] = np.float32(2.0 ** 60)   # out of the range of parts, and multiplied by nothing
    w.keep_blocks = synth.pack_bits(keep)
    check_workload(w, "joined", exact=True)


# ---- no less exact than floats as they are ------------------------------------------------------
@pytest.mark.parametrize("dist", ["normal", "uniform"])
@pytest.mark.parametrize("scale_x,scale_y", [(1.0, 1.0), (2.0 ** -100, 2.0 ** 40), (1.0, 0.02)])
@pytest.mark.parametrize("M,K,N,p", [(130, 300, 96, 0.1), (130, 2100, 96, 0.4)])
def test_error_against_double_precision(M, K, N, p, scale_x, scale_y, dist):
    w = synth.random_masked(M, K, N, 16, p, p, 5 + K, dist=dist)
    w.X, w.Y = (w.X * np.float32(scale_x)).astype(np.float32), (w.Y * np.float32(scale_y)).astype(np.float32)
    ab, bb, _, mag = oracle.run_workload(w)
    A = np.where(synth.unpack_bits(ab, K), w.X, 0).astype(np.float64)
    B = np.where(np.repeat(synth.unpack_bits(bb, N // 16), 16, axis=1), w.Y, 0).astype(np.float64)
    exact = A @ B
    error = {}
    for form in (PLAIN, PARTS):
        mm.mmm_set_option("float_form", form)
        _, _, C = HipRun(w).run()
        error[form] = np.linalg.norm(C - exact) / np.linalg.norm(exact)
        # a sum of n products rounded once each is off by less than n 2^-24 |A||B| (six products of parts are left out or
        # rounded below that)
        assert (np.abs(C - exact) <= K * 2.0 ** -24 * mag + 1e-45).all()
    assert error[PARTS] <= error[PLAIN]


@pytest.mark.parametrize("products", [1, 2])
@pytest.mark.parametrize("ex,ey", [(0, 0), (-110, 0), (-110, 53), (-110, -14), (54, 54), (54, -110), (-63, -63), (-58, -60), (-75, -74)])
def test_few_products(ex, ey, products):
    """Sums of one product and of two, up to the ends of the range that parts hold and where products or the parts' products
    are subnormal.  In units of 2^-24 of the products' magnitudes: the three products of parts left out are below 1, the
    others' sums are 2^-7 of the whole and off by less than 0.1, adding the two accumulators rounds by 1 (floats as they
    are: 1), and the first parts' sum of two by 2 where the instruction cuts off.  Each of the six products and two additions
    may lose 2^-149 among subnormals."""
    M, K, N = 96, 128, 64
    rng = np.random.default_rng(abs(1000 * ex + ey) + products)

    def values(shape, e):
        fraction = rng.integers(0, 1 << 23, shape)
        fraction = np.where(rng.random(shape) < 0.3, rng.choice([0, 1, (1 << 23) - 1], shape), fraction)
        return ((1 + fraction / 2.0 ** 23) * rng.choice([-1.0, 1.0], shape) * 2.0 ** e).astype(np.float32)

    w = synth.random_masked(M, K, N, 16, 1.0, 1.0, 1)
    w.Y = values((K, N), ey)
    w.X[:] = 0
    for i in range(M):
        w.X[i, rng.permutation(K)[:products]] = values(products, ex)
    exact = w.X.astype(np.float64) @ w.Y.astype(np.float64)
    mag = np.abs(w.X.astype(np.float64)) @ np.abs(w.Y.astype(np.float64))
    _, _, C = HipRun(w).run()
    units = 2.1 if products == 1 else 4.1
    err = np.abs(C - exact)
    print("worst", (err / mag).max() * 2 ** 24)
    assert (err <= units * 2.0 ** -24 * mag + 8 * 2.0 ** -149).all()


# ---- elements that the parts do not hold: multiplied as floats ----------------------------------
@pytest.mark.parametrize("rows", [None, 0.7], ids=["all", "rows"])
@pytest.mark.parametrize("bw", [8, 16, 32])
@pytest.mark.parametrize("value", [2.0 ** -111, 3e-39, -1e-45, 2.0 ** 55, -3.4028235e38], ids=str)
def test_finite_elements_out_of_range(value, bw, rows):
    """One in A, one in B, in blocks of their own; the other factors are small integers, so every sum is exact in float or
    dominated by the element."""
    w = synth.random_masked(140, 700, 96, bw, 0.4, 0.6, 17 + bw, dist="smallint", p_rows=rows)
    ab = oracle.run_workload(w)[0]
    live = np.ones(w.K, bool) if rows is None else synth.unpack_bits(w.keep_rows.reshape(1, -1), w.K)[0]
    b = synth.unpack_bits(oracle.b_bits(w.Y, bw, w.keep_rows, w.keep_blocks), w.NB)
    i, k = [int(v) for v in np.argwhere(synth.unpack_bits(ab, w.K) & live)[300]]
    w.X[i, k] = value
    k2, jb = [int(v) for v in np.argwhere(b)[-1]]
    assert k // 128 != k2 // 128
    w.Y[k2, jb * bw + 1] = value
    ab, bb, C_ref, mag = oracle.run_workload(w)
    run = HipRun(w)
    a_hip, b_hip, C = run.run()
    np.testing.assert_array_equal(a_hip, ab)
    np.testing.assert_array_equal(b_hip, bb)
    finite = np.isfinite(C_ref)
    np.testing.assert_array_equal(np.isfinite(C), finite)
    assert (np.abs(C[finite] - C_ref[finite]) <= w.K * 2.0 ** -24 * mag[finite] + 1e-45).all()
    mm.mmm_set_option("float_form", PLAIN)
    plain = HipRun(w).run()[2]
    clean = (C_ref == np.rint(C_ref)) & (np.abs(C_ref) < 2 ** 20)       # sums of small integers alone
    np.testing.assert_array_equal(C[clean], plain[clean])


@pytest.mark.parametrize("rows", [None, 0.7], ids=["all", "rows"])
@pytest.mark.parametrize("bw", [8, 16, 32])
def test_marked_steps_everywhere(bw, rows):
    """Marked steps on either side of the 32 that share a word, of the 64 batches that are planned together and of the splits,
    on both places of the ring, with lists of one batch and of several.  A marked step is left out of the loop and redone
    behind it for all rows (A) or all 16 columns (B): those without the element, sums of small integers, show what is lost
    or counted twice."""
    w = synth.random_masked(140, 140 * 128 - 37, 96, bw, 0.1, 1.0, 51 + bw, dist="smallint", p_rows=rows)
    live = np.arange(w.K) if rows is None else np.nonzero(synth.unpack_bits(w.keep_rows.reshape(1, -1), w.K)[0])[0]
    steps = -(-len(live) // 128)
    assert steps > 96
    rng = np.random.default_rng(bw)
    share = rng.choice([0.02, 0.2, 0.6], (w.K // 128 + 1, w.NB)).repeat(128, 0)[: w.K]
    on = rng.random((w.K, w.NB)) < share
    a_steps, b_steps = [0, 31, 32, 63, 64, steps - 1], [1, 33, 62, 65, steps // 3, 2 * (steps // 3) + 1, steps - 1]
    a = synth.unpack_bits(w.keep_a, w.K).copy()
    for i, st in enumerate(a_steps):
        k = int(live[st * 128 + i])
        a[7 + 22 * i, k], w.X[7 + 22 * i, k] = True, 2.0 ** 56
    for i, st in enumerate(b_steps):
        k = int(live[min(st * 128 + 3 * i, len(live) - 1)])
        on[k, i % w.NB], w.Y[k, (i % w.NB) * bw + i % bw] = True, -(2.0 ** 57)
    w.keep_a, w.keep_blocks = synth.pack_bits(a), synth.pack_bits(on)
    _, _, C_ref, mag = oracle.run_workload(w)
    clean = mag < 2.0 ** 24
    assert 0.7 < clean.mean() < 1.0
    run = HipRun(w)
    run.build()
    assert mm.mmm_matmul_form(run.eng.maps) == PARTS
    for split in (1, 3):
        run.eng.set_plan(1, split)
        run.Cbuf.fill_(float("nan"))
        run.matmul()
        torch.cuda.synchronize()
        C = run.C.cpu().numpy()
        np.testing.assert_array_equal(C[clean], C_ref[clean])
        assert (np.abs(C - C_ref) <= w.K * 2.0 ** -24 * mag).all()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan], ids=str)
@pytest.mark.parametrize("where", ["x", "y"])
def test_non_finite_elements(where, value):
    """What the definition gives in the row or column of the element, and nothing elsewhere."""
    w = synth.random_masked(140, 700, 96, 16, 0.4, 0.6, 29, dist="smallint")
    ab, bb, C_ref, _ = oracle.run_workload(w)
    a, b = synth.unpack_bits(ab, w.K), synth.unpack_bits(bb, w.NB)
    i, k = [int(v) for v in np.argwhere(a)[500]]
    jb = int(np.nonzero(b[k])[0][0])
    hit = np.zeros(C_ref.shape, bool)
    if where == "x":
        w.X[i, k] = value
        hit[i] = np.repeat(b[k], 16)
    else:
        w.Y[k, jb * 16 + 3] = value
        hit[:, jb * 16 + 3] = True
    bad = oracle.run_workload(w)[2]
    _, _, C = HipRun(w).run()
    np.testing.assert_array_equal(C[~hit], C_ref[~hit])
    if where == "x":
        np.testing.assert_array_equal(np.isfinite(C), np.isfinite(bad))
        np.testing.assert_array_equal(np.isnan(C), np.isnan(bad))
    else:
        rows = a[:, k]
        assert not np.isfinite(C[rows, jb * 16 + 3]).any()
        rest = C[~rows, jb * 16 + 3]
        assert np.all(np.isnan(rest) | (rest == C_ref[~rows, jb * 16 + 3]))


@pytest.mark.parametrize("rows", [None, 0.7], ids=["all", "rows"])
@pytest.mark.parametrize("bw", [8, 16, 32])
def test_the_multiplication_reads_neither_operand(bw, rows):
    """Elements in and out of range in either operand; X and Y hold something else by the time of the multiplication."""
    w = synth.random_masked(140, 700, 96 + bw, bw, 0.4, 0.6, 23 + bw, dist="normal", p_rows=rows)
    rng = np.random.default_rng(bw)
    odd = np.float32([2.0 ** -111, -3e-39, 1e-45, 2.0 ** 55, -2.0 ** 61])
    # (in some of the blocks of A and in some of the segments of B)
    for v, share in ((w.X[:, :200], 0.001), (w.Y[300:500], 0.002)):
        at = rng.random(v.shape) < share
        v[at] = rng.choice(odd, int(at.sum()))
    _, _, C_ref, mag = oracle.run_workload(w)
    run = HipRun(w)
    run.build()
    run.matmul()
    torch.cuda.synchronize()
    C = run.C.cpu().numpy()
    assert (np.abs(C - C_ref) <= w.K * 2.0 ** -24 * mag + 1e-45).all()
    run.X.fill_(float("nan"))
    run.Y.fill_(float("nan"))
    run.Cbuf.fill_(float("nan"))
    run.matmul()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(run.C.cpu().numpy(), C)


def test_inspection_shows_the_elements_as_they_are():
    rng = np.random.default_rng(3)
    w = synth.random_masked(100, 300, 32, 16, 0.5, 0.5, 4, dist="normal")
    bits = rng.integers(0, 1 << 32, w.X.shape, dtype=np.uint64).astype(np.uint32)       # every exponent, NaN payloads too
    w.X = np.where(rng.random(w.X.shape) < 0.3, bits.view(np.float32), w.X)
    from test_gpu_parity import check_lists
    run = HipRun(w)
    run.build()
    torch.cuda.synchronize()
    check_lists(run, oracle.a_bits(w.X, keep_bits=w.keep_a), w, "lists")


# ---- which form a build takes ---------------------------------------------------------------------
def test_the_form_follows_the_counts_and_the_side_that_is_kept():
    """Seen by the bits of C, which the two forms round differently."""
    mm.mmm_set_option("matmul_path", -1)
    w = synth.random_masked(1500, 2100, 1024, 16, 0.4, 0.5, 8, dist="normal")
    want = {}
    for form in (PLAIN, PARTS):
        mm.mmm_set_option("float_form", form)
        run = HipRun(w)
        run.eng.set_plan(1, 1)
        want[form] = run.run()[2]
    mm.mmm_set_option("float_form", -1)
    assert (want[PLAIN] != want[PARTS]).any()

    def check(run, form):
        run.Cbuf.fill_(float("nan"))
        run.matmul()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(run.C.cpu().numpy(), want[form])

    run = HipRun(w)
    run.eng.set_plan(1, 1)
    run.build()
    check(run, PLAIN)                      # nothing is known
    run.eng.stats()
    check(run, PLAIN)                      # as it was built
    run.build(a=True, b=False)
    check(run, PLAIN)                      # B is kept
    run.build(a=False, b=True)
    check(run, PLAIN)                      # A is
    run.build()
    check(run, PARTS)
    run.build(a=True, b=False)
    check(run, PARTS)
    run.eng.set_plan(0, 1)                 # parts take this tile too, and the builds that follow leave floats as they are
    check(run, PARTS)
    run.build()
    check(run, PLAIN)


@pytest.mark.parametrize("rows", [None, 0.7], ids=["all", "rows"])
@pytest.mark.parametrize("bw", [8, 16, 32])
@pytest.mark.parametrize("side", ["x", "y"])
def test_the_form_follows_the_steps_that_parts_do_not_hold(side, bw, rows):
    """stats() counts them in either form; where they are more than a few, floats stay as they are or become so again."""
    mm.mmm_set_option("matmul_path", -1)
    mm.mmm_set_option("float_form", -1)
    w = synth.random_masked(1500, 4000, 1024, bw, 0.4, 0.5, 8, dist="normal", p_rows=rows)
    run = HipRun(w)
    clean = {"x": run.X.clone(), "y": run.Y.clone()}
    given = run.X if side == "x" else run.Y
    at = torch.rand(given.shape, generator=torch.Generator().manual_seed(bw)) < 0.001
    odd = torch.where(at.cuda(), torch.full_like(given, 1e-38), given)

    def form_after_stats():
        run.build()
        run.matmul()
        run.eng.stats()
        run.build()
        return mm.mmm_matmul_form(run.eng.maps)

    given.copy_(odd)
    assert form_after_stats() == PLAIN     # counted among floats as they are
    given.copy_(clean[side])
    assert form_after_stats() == PARTS
    given.copy_(odd)
    assert form_after_stats() == PLAIN     # counted among parts
    given.copy_(clean[side])
    assert form_after_stats() == PARTS


@pytest.mark.parametrize("M,K,N,bw,p,form", [
    (3631, 206, 3456, 16, 0.169, PLAIN), (3157, 304, 3832, 8, 0.081, PLAIN), (3434, 737, 3680, 16, 0.121, PLAIN),   # passes in parts take 1.34, 1.18 and 1.20 times as long
    (1969, 637, 2752, 16, 0.179, PLAIN),                                  # 1.10 times
    (2048, 2048, 2048, 16, 0.4, PARTS), (1300, 4096, 3000, 8, 0.3, PARTS),   # long lists
])
def test_choice_of_form(M, K, N, bw, p, form):
    """Short lists and a short K are multiplied as floats."""
    mm.mmm_set_option("matmul_path", -1)
    mm.mmm_set_option("float_form", -1)
    run = HipRun(synth.random_masked(M, K, N, bw, 0.2, p, M + K, dist="normal"))
    run.build()
    run.eng.stats()
    run.build()
    assert mm.mmm_matmul_form(run.eng.maps) == form


@pytest.mark.parametrize("value", [1e-38, float("nan")], ids=str)
def test_columns_that_are_switched_off_mark_nothing(value):
    """Whatever they hold.  Seen by the count of marked steps: more than a few would bring floats as they are."""
    mm.mmm_set_option("matmul_path", -1)
    mm.mmm_set_option("float_form", -1)
    w = synth.random_masked(1500, 4000, 1024, 16, 0.4, 0.5, 8, dist="normal", p_rows=0.7)
    off = ~synth.unpack_bits(w.keep_rows.reshape(1, -1), w.K)[0]
    w.X[:, off] = np.float32(value)
    run = HipRun(w)
    for want in (PLAIN, PARTS, PARTS, PARTS):
        run.build()
        assert mm.mmm_matmul_form(run.eng.maps) == want
        run.eng.stats()


def test_a_workspace_without_room_for_parts():
    """That of another type: floats are multiplied as they are, whatever is asked for, and nothing behind it is written."""
    w = synth.random_masked(200, 700, 288, 16, 0.4, 0.5, 9, dist="normal")
    mm.mmm_set_option("float_form", PLAIN)
    want = HipRun(w).run()[2]
    mm.mmm_set_option("float_form", PARTS)
    run = HipRun(w)
    need = mm.mmm_maps_workspace_bytes_for(w.M, w.K, w.N, w.bw, mm.MMM_BF16)
    room = run.eng.workspace.numel()
    assert need < room
    run.eng.close()
    run.eng.workspace.fill_(0x5a)
    run.eng.maps = mm.mmm_maps_init(run.eng.workspace, need, w.M, w.K, w.N, w.bw)
    np.testing.assert_array_equal(run.run()[2], want)
    run.eng.stats()
    np.testing.assert_array_equal(run.run()[2], want)
    assert (run.eng.workspace[need:] == 0x5a).all()


@pytest.mark.parametrize("bw", [8, 16, 32])
def test_a_tile_that_is_fixed_holds_at_once(bw):
    """The tiles with one range of K take parts as well; which tile it is does not change the sums."""
    w = synth.random_masked(200, 1500, 544, bw, 0.4, 0.5, 41 + bw, dist="normal")
    run = HipRun(w)
    run.eng.set_plan(1, 1)
    want = run.run()[2]
    assert mm.mmm_matmul_form(run.eng.maps) == PARTS
    for v in range(mm.mmm_matmul_variant_count()):
        name = mm.mmm_matmul_variant_name(v)
        print("variant", v, name, flush=True)
        run.eng.set_plan(v, 1)
        held = name.startswith("R4") and not name.endswith("K2")
        assert run.eng.plan()[:2] == (v if held else 1, 1)
        run.Cbuf.fill_(float("nan"))
        run.matmul()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(run.C.cpu().numpy(), want)
    mm.mmm_set_option("float_form", PLAIN)
    run.build()
    assert mm.mmm_matmul_form(run.eng.maps) == PLAIN


@pytest.mark.parametrize("form", [PLAIN, PARTS])
def test_autotune_times_the_tiles_of_the_form(form):
    w = synth.random_masked(300, 2100, 384, 16, 0.4, 0.5, 12, dist="normal")
    mm.mmm_set_option("float_form", form)
    run = HipRun(w)
    run.build()
    results = run.eng.autotune(run.X, run.Y, run.C, splits=(1, 2), reps=2)
    names = [mm.mmm_matmul_variant_name(v) for v in range(mm.mmm_matmul_variant_count())]
    usable = [v for v, n in enumerate(names) if n.startswith("R4") and not (form == PARTS and n.endswith("K2"))]
    assert sorted({r[1] for r in results}) == usable and results == sorted(results)
    fixed = run.eng.plan()[:2]
    assert fixed == (results[0][1:] if form == PLAIN else next(r[1:] for r in results if r[1] == 1))
    # the form is decided anew by the builds that follow: a plan found for parts keeps them where they pay
    mm.mmm_set_option("float_form", -1)
    wide = synth.random_masked(1500, 2100, 1024, 16, 0.4, 0.5, 8, dist="normal")
    run = HipRun(wide)
    run.build()
    run.eng.stats()
    run.build()
    assert mm.mmm_matmul_form(run.eng.maps) == PARTS
    run.eng.autotune(run.X, run.Y, run.C, reps=2)
    run.build()
    assert mm.mmm_matmul_form(run.eng.maps) == PARTS and run.eng.plan()[0] == 1


@pytest.mark.parametrize("captured", ["build", "matmul"])
def test_a_captured_call_fixes_the_form(captured):
    """A graph's build or multiplication runs between calls of other forms otherwise."""
    w = synth.random_masked(200, 700, 288, 16, 0.4, 0.5, 9, dist="smallint")
    C_ref = oracle.run_workload(w)[2]
    mm.mmm_set_option("float_form", -1)
    run = HipRun(w)
    run.build()
    run.matmul()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run.build() if captured == "build" else run.matmul()
    mm.mmm_set_option("float_form", PARTS)
    run.eng.stats()
    for _ in range(3):
        run.Cbuf.fill_(float("nan"))
        if captured == "matmul":
            run.build()
        graph.replay()
        if captured == "build":
            run.matmul()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(run.C.cpu().numpy(), C_ref)
        run.build()
        run.matmul()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(run.C.cpu().numpy(), C_ref)


def test_the_form_is_free_again_when_the_graphs_are_gone():
    w = synth.random_masked(200, 700, 288, 16, 0.4, 0.5, 9, dist="smallint")
    C_ref = oracle.run_workload(w)[2]
    mm.mmm_set_option("float_form", PLAIN)
    run = HipRun(w)
    run.build()
    run.matmul()
    torch.cuda.synchronize()
    graphs = [torch.cuda.CUDAGraph() for _ in range(3)]
    for graph, calls in zip(graphs, ([run.build, run.matmul], [run.matmul], [run.matmul])):
        with torch.cuda.graph(graph):
            for call in calls:
                call()
    mm.mmm_set_option("float_form", PARTS)

    def form_of_a_build():
        for _ in range(3):             # (the runtime lets go of a graph that has run some calls later)
            run.build()
            torch.cuda.synchronize()
        return mm.mmm_matmul_form(run.eng.maps)

    while len(graphs) > 1:
        assert form_of_a_build() == PLAIN
        for graph in graphs:
            run.Cbuf.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            np.testing.assert_array_equal(run.C.cpu().numpy(), C_ref)
        del graph, graphs[0]
        gc.collect()
        torch.cuda.synchronize()
    assert form_of_a_build() == PLAIN
    graphs.clear()
    gc.collect()
    torch.cuda.synchronize()
    assert form_of_a_build() == PARTS
    run.matmul()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(run.C.cpu().numpy(), C_ref)
    graph = torch.cuda.CUDAGraph()     # that outlives the handle
    with torch.cuda.graph(graph):
        run.matmul()
    graph.replay()
    torch.cuda.synchronize()
    run.eng.close()
    del graph
    gc.collect()
    torch.cuda.synchronize()
