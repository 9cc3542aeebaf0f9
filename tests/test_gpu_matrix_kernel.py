"""The kernels at the edges of their geometry: blocks of A of 64 rows x 128 columns (64 for doubles in
the builder), groups of 16 columns, segments of 128 k whose lists are walked in batches of 16 or 32 slots, column tiles of
256 (128).  Exact on integer inputs, against the CPU oracle, for every element type."""
import numpy as np
import pytest
import torch

import mmm_synth as synth
import oracle
import paper_2402_14118_amd as mm
from hip_harness import HipRun

pytestmark = pytest.mark.gpu

DTYPES = [synth.DT_F32, synth.DT_BF16, synth.DT_F16, synth.DT_F64]
IDS = ["f32", "bf16", "f16", "f64"]


def _run(w, split=1, variant=-1, **ld):
    ab, bb, C_ref, _ = oracle.run_workload(w)
    run = HipRun(w, **ld)
    run.eng.set_path(mm.MMM_PATH_MATRIX)
    run.eng.set_plan(variant, split)
    a, b, C = run.run()
    assert run.eng.path() == mm.MMM_PATH_MATRIX
    np.testing.assert_array_equal(a, ab)
    np.testing.assert_array_equal(b, bb)
    np.testing.assert_array_equal(C, C_ref)
    return run, C_ref


@pytest.mark.parametrize("dtype", DTYPES, ids=IDS)
@pytest.mark.parametrize("M,K,N,bw", [
    (65, 1, 8, 8),            # one k; half a column group
    (65, 2, 136, 8),          # half a group behind whole ones, across a column tile of 128
    (128, 64, 16, 16), (128, 65, 272, 16), (129, 127, 256, 16), (129, 128, 288, 32), (66, 129, 264, 8),
    (190, 257, 544, 32),      # three segments, the ring reused; three column tiles of 256
    (70, 1030, 48, 16),       # nine segments
])
def test_edges(M, K, N, bw, dtype):
    w = synth.random_masked(M, K, N, bw, 0.4, 0.4, 31 * M + K + N, dist="smallint", dtype=dtype)
    _run(w)
    print("split", M, K, N, bw, flush=True)
    _run(w, split=3)


@pytest.mark.parametrize("dtype", DTYPES, ids=IDS)
@pytest.mark.parametrize("bw", [8, 16, 32])
def test_list_lengths(bw, dtype):
    """Segments whose lists have every length around the batch and quad sizes: segment s of column group g holds
    lengths[(s + g) % len] occupied rows; the rest of B is switched off and holds values that would show."""
    lengths = [0, 1, 3, 4, 5, 15, 16, 17, 31, 32, 33, 127, 128, 0, 64]
    M, segs, N = 80, 16, 128
    K, NB = segs * 128, N // bw
    keep = np.zeros((K, NB), bool)
    rng = np.random.default_rng(bw)
    for s in range(segs):
        for b in range(NB):
            n = lengths[(s + b * bw // max(16, bw)) % len(lengths)]
            keep[s * 128 + rng.permutation(128)[:n], b] = True
    w = synth.random_masked(M, K, N, bw, 0.5, 1.0, 77 + bw, dist="smallint", dtype=dtype)
    w.keep_blocks = synth.pack_bits(keep)
    _run(w)
    _run(w, split=4)


@pytest.mark.parametrize("dtype", DTYPES, ids=IDS)
def test_many_steps(dtype):
    """More steps than a wave holds list lengths for at a time (62), in whole and with K in two ranges, the last one of an
    odd number of steps; waves without columns in the last column tile."""
    for segs in (63, 125):
        w = synth.random_masked(70, segs * 128 - 5, 80, 16, 0.05, 0.05, segs, dist="smallint", dtype=dtype)
        for variant in (0, 1) if dtype == synth.DT_F64 else (0, 1, 6, 7):
            print("segments", segs, "variant", variant, flush=True)
            _run(w, variant=variant)


@pytest.mark.parametrize("dtype", [synth.DT_F32, synth.DT_BF16, synth.DT_F16], ids=["f32", "bf16", "f16"])
@pytest.mark.parametrize("M,p_rows", [(389, 1.0), (261, 0.1)])      # seven, five blocks of A below each other, the last one ragged
def test_many_blocks_per_builder_workgroup(M, p_rows, dtype):
    w = synth.random_masked(M, 53001, 32, 16, 0.1, 0.1, M, dist="smallint", dtype=dtype, p_rows=p_rows)
    _run(w)


@pytest.mark.parametrize("dtype,form", [(synth.DT_F32, 0), (synth.DT_F32, 1), (synth.DT_BF16, -1), (synth.DT_F16, -1), (synth.DT_F64, -1)],
                         ids=["f32", "parts", "bf16", "f16", "f64"])
@pytest.mark.parametrize("M,K,N,p_rows", [
    (389, 11400, 32, 1.0),     # 630 blocks of A, seven below each other: two, two, two and a ragged one per workgroup
    (129, 25600, 16, 0.1),     # 600 in three rows: the fewest that go in twos
    (70, 65400, 16, 1.0),      # 1022 in two rows: the most
    (389, 14000, 32, 0.3),     # 770 in seven rows: row-compacted floats in parts too
])
def test_two_blocks_per_builder_workgroup(M, K, N, p_rows, dtype, form):
    if dtype == synth.DT_F64:   # blocks half as wide
        K //= 2
    mm.mmm_set_option("float_form", form)
    try:
        _run(synth.random_masked(M, K, N, 16, 0.1, 0.1, M, dist="smallint", dtype=dtype, p_rows=p_rows))
    finally:
        mm.mmm_set_option("float_form", -1)


@pytest.mark.parametrize("M,N,split", [(2100, 16, 1), (40, 4112, 3), (1000, 2576, 1), (1030, 3344, 4)])
def test_numbering_of_tiles(M, N, split):
    """One column of tiles, one row of them, panels of tile columns with a narrower last one: every tile once, whatever its size."""
    for variant in range(mm.mmm_matmul_variant_count()):
        print("variant", variant, flush=True)
        _run(synth.random_masked(M, 260, N, 16, 0.2, 0.3, M + N, dist="smallint", dtype=synth.DT_BF16), split, variant)


@pytest.mark.parametrize("dtype", DTYPES, ids=IDS)
def test_every_variant_and_row_count(dtype):
    for variant in range(mm.mmm_matmul_variant_count()):
        short = mm.mmm_matmul_variant_name(variant).startswith("R2")
        if short and dtype == synth.DT_F64:
            continue      # doubles of so few rows take the pair kernel
        for M in ((17, 32) if short else (65, 191)):
            for bw in (16, 32):
                print("variant", variant, M, bw, flush=True)
                _run(synth.random_masked(M, 300, 544, bw, 0.3, 0.5, variant * 10 + M, dist="smallint", dtype=dtype), variant=variant)


@pytest.mark.parametrize("dtype", DTYPES, ids=IDS)
def test_leading_dimensions_and_accumulate(dtype):
    """Odd leading dimensions put the rows of 16-bit matrices on 2-byte boundaries."""
    w = synth.random_masked(100, 333, 80, 16, 0.4, 0.5, 5, dist="smallint", dtype=dtype, p_rows=0.6)
    run, C_ref = _run(w, ldx=335, ldy=83, ldc=91)
    run.eng.matmul(run.X, run.Y, run.C, accumulate=True)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(run.C.cpu().numpy(), 2 * C_ref)
    assert torch.isnan(run.Cbuf[:, 80:]).all()


@pytest.mark.parametrize("dtype", [synth.DT_F32, synth.DT_BF16, synth.DT_F64], ids=["f32", "bf16", "f64"])
def test_values_that_must_not_reach_the_arithmetic(dtype):
    """NaN and Inf where the masks drop them, at the ragged edges of every tile."""
    w = synth.random_masked(97, 200, 136, 8, 0.3, 0.3, 6, dist="smallint", dtype=dtype)
    C_ref = oracle.run_workload(w)[2]
    w.X = np.where(synth.unpack_bits(w.keep_a, w.K), w.X, np.nan).astype(w.X.dtype)
    w.Y = np.where(np.repeat(synth.unpack_bits(w.keep_blocks, w.NB), w.bw, axis=1), w.Y, np.inf).astype(w.Y.dtype)
    if dtype == synth.DT_BF16:
        w.X_bits, w.Y_bits = synth.round_to_bf16(w.X)[0], synth.round_to_bf16(w.Y)[0]
    run = HipRun(w)
    run.eng.set_path(mm.MMM_PATH_MATRIX)
    np.testing.assert_array_equal(run.run()[2], C_ref)


@pytest.mark.parametrize("dtype", DTYPES, ids=IDS)
@pytest.mark.parametrize("M,K,N,bw", [
    (1, 7, 8, 8), (3, 8, 72, 8), (2, 1025, 96, 32),     # fewer than eight k; a whole byte of k; one k behind the last whole byte
    (5, 2049, 144, 16), (20, 4097, 272, 16), (40, 9001, 40, 8), (7, 17000, 64, 32),   # ranges of 16, 32, 64 words of k
    (18, 66001, 32, 16),                                # more k than the bitmap in LDS holds
    (300, 300, 520, 8), (1030, 70, 32, 16), (1040, 2100, 16, 16),   # many rows
])
def test_pair_kernel_shapes(M, K, N, bw, dtype):
    """Every workgroup shape and range size of the pair kernel, with the map of A built and with the mask evaluated in the
    multiplication, at odd leading dimensions."""
    w = synth.random_masked(M, K, N, bw, 0.15, 0.3, M + K + N, dist="smallint", dtype=dtype)
    C_ref = oracle.run_workload(w)[2]
    run = HipRun(w, ldx=K + 1, ldy=N + 3, ldc=N + 1)
    run.eng.set_path(mm.MMM_PATH_PAIRS)
    run.build()
    for fused in (False, True):
        print("fused", fused, flush=True)
        run.Cbuf.fill_(float("nan"))
        if fused:
            run.eng.matmul_fused(run.X, run.Y, run.C, w.pred, w.threshold, run.keep_a)
        else:
            run.matmul()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(run.C.cpu().numpy(), C_ref)
        assert torch.isnan(run.Cbuf[:, N:]).all()


@pytest.mark.parametrize("dtype", DTYPES, ids=IDS)
@pytest.mark.parametrize("K", [1, 7, 8, 9, 63, 64, 65, 4097, 66001])
@pytest.mark.parametrize("M,ldx_more", [(3, 0), (19, 1)])
def test_fused_mask_without_a_bitmap(M, ldx_more, K, dtype):
    """The multiplication that evaluates the mask, where no bitmap is given: whole groups of eight k and what is left of them."""
    w = synth.random_masked(M, K, 72, 8, 0.5, 0.4, 7 * K + M, dist="smallint", dtype=dtype)
    w.keep_a, w.pred, w.threshold = None, synth.PRED_GT, 0.0
    C_ref = oracle.run_workload(w)[2]
    run = HipRun(w, ldx=K + ldx_more)
    run.build(a=False, b=True)
    run.eng.matmul_fused(run.X, run.Y, run.C, w.pred, w.threshold, None)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(run.C.cpu().numpy(), C_ref)


@pytest.mark.parametrize("dtype,form", [(synth.DT_BF16, -1), (synth.DT_F16, -1), (synth.DT_F32, 0), (synth.DT_F32, 1), (synth.DT_F64, -1)],
                         ids=["bf16", "f16", "f32", "parts", "f64"])
@pytest.mark.parametrize("bw", [8, 16, 32])
def test_shorter_lists_over_longer_ones(bw, dtype, form):
    """A build leaves what lies behind a list as it was: here infinities and NaN of a build with every block on.  Lists end one
    slot before, at and behind each unit of eight, and what A holds at other k is not finite either (where A is masked out)."""
    lengths = [0, 1, 7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32, 33, 40, 127]
    M, segs, N = 70, 9, 96
    K, NB = segs * 128, N // bw
    keep = np.zeros((K, NB), bool)
    rng = np.random.default_rng(bw)
    for s in range(segs):
        for b in range(NB):
            keep[s * 128 + rng.permutation(128)[: lengths[(5 * s + b) % len(lengths)]], b] = True
    w = synth.random_masked(M, K, N, bw, 0.5, 1.0, 177 + bw, dist="smallint", dtype=dtype)
    w.keep_blocks = synth.pack_bits(keep)
    C_ref = oracle.run_workload(w)[2]
    mm.mmm_set_option("float_form", form)
    try:
        run = HipRun(w)
        run.eng.set_path(mm.MMM_PATH_MATRIX)
        Y = run.Y.clone()
        run.Y.copy_(torch.where(torch.rand(K, N, device="cuda") < 0.5, 0x7fff, 0x7f80).to(torch.int16) if Y.dtype == torch.int16
                    else torch.where(torch.rand(K, N, device="cuda") < 0.5, float("nan"), float("inf")))
        run.eng.build_maps(run.X, run.Y, w.pred, w.threshold, run.keep_a)
        run.matmul()
        run.Y.copy_(Y)
        np.testing.assert_array_equal(run.run()[2], C_ref)
    finally:
        mm.mmm_set_option("float_form", -1)


@pytest.mark.parametrize("dtype,bw", [(synth.DT_F32, 16), (synth.DT_BF16, 8), (synth.DT_F16, 32)], ids=["f32", "bf16", "f16"])
@pytest.mark.parametrize("K,live", [
    (64, "none"), (65, "last"), (300, 127), (300, 128), (300, 129),     # no segment, the last bit of a row word, whole segments and one row more
    (5000, 1), (5000, "all"), (4097, 640),                              # 40 segments of which one, all, five hold a row
    (65536, 300), (65537, 300), (70001, "last"),                        # a row word per thread, and more
])
def test_numbering_of_rows(K, live, dtype, bw):
    """Row-compacted builds behind a build with every row on: the numbering, map rows of rows that are off, C."""
    N = 544 if K < 10000 else 32                                        # three column tiles; one
    rng = np.random.default_rng(K)
    on = np.zeros(K, bool)
    on[{"none": [], "last": [K - 1], "all": np.arange(K)}.get(live) if isinstance(live, str) else rng.permutation(K)[:live]] = True
    w = synth.random_masked(70, K, N, bw, 0.3, 0.6, K, dist="smallint", dtype=dtype)
    run = HipRun(w)
    run.eng.set_path(mm.MMM_PATH_MATRIX)
    run.build()
    w.keep_rows = synth.pack_bits(on[None, :])
    ab, bb, C_ref, _ = oracle.run_workload(w)
    run.keep_rows = torch.from_numpy(w.keep_rows.view(np.int64)).cuda()
    a, b, C = run.run()
    np.testing.assert_array_equal(a, ab)
    np.testing.assert_array_equal(b, bb)
    np.testing.assert_array_equal(C, C_ref)
    count, kmap, _, _ = run.eng.compacted()
    assert int(count.cpu()[0]) == on.sum()
    np.testing.assert_array_equal(kmap.cpu().numpy()[: on.sum()], np.flatnonzero(on))


@pytest.mark.parametrize("dtype", [synth.DT_F32, synth.DT_F16], ids=["f32", "f16"])
@pytest.mark.parametrize("K,N,bw", [(1, 8, 8), (63, 520, 8), (129, 1032, 8), (200, 8192, 8), (130, 8200, 8), (127, 16416, 16), (65, 66048, 32), (70, 65536, 8)])
def test_map_rows_that_are_off(K, N, bw, dtype):
    """Their words are cleared, whatever a build before had there: 1 to 128 words per row."""
    w = synth.random_masked(3, K, N, bw, 0.5, 1.0, K + N, dist="smallint", dtype=dtype)
    run = HipRun(w)
    run.build()
    assert (run.maps_host()[1] != 0).any()
    w.keep_rows = synth.pack_bits((np.arange(K) % 3 == 1)[None, :])
    run.keep_rows = torch.from_numpy(w.keep_rows.view(np.int64)).cuda()
    run.build()
    np.testing.assert_array_equal(run.maps_host()[1], oracle.run_workload(w)[1])


@pytest.mark.parametrize("dtype", [synth.DT_BF16, synth.DT_F16], ids=["bf16", "f16"])
@pytest.mark.parametrize("bw", [8, 16, 32])
@pytest.mark.parametrize("M", [1, 31, 32, 33, 64, 65])
def test_planes_of_every_tile(M, bw, dtype):
    """Every tile of 16-bit types (a wave copies a part of a plane, one, or two of them; tiles of 32 rows two of the four), rows around
    the planes' ends.  Column k = 5 (mod 7) of A is infinite and its row of B off; whole steps have no list; the last ones begin behind K in
    one range of K."""
    K, N = 128 * 9 + 40, 288
    w = synth.random_masked(M, K, N, bw, 0.5, 0.3, 13 * M + bw, dist="smallint", dtype=dtype)
    k = np.arange(K)
    on = (k % 7 != 5) & (k // 128 % 3 != 1)
    w.keep_blocks = synth.pack_bits(synth.unpack_bits(w.keep_blocks, N // bw).astype(bool) & on[:, None])
    C_ref = oracle.run_workload(w)[2]
    run = HipRun(w)
    run.eng.set_path(mm.MMM_PATH_MATRIX)
    run.X[:, k % 7 == 5] = 0x7f80 if dtype == synth.DT_BF16 else 0x7c00
    for variant in range(mm.mmm_matmul_variant_count()):
        for split in (1, 2):
            run.eng.set_plan(variant, split)
            if run.eng.plan()[0] != variant:
                continue   # computes fewer rows than there are
            print(variant, split, flush=True)
            np.testing.assert_array_equal(run.run()[2], C_ref)


@pytest.mark.parametrize("M,dtype,form", [(4097, synth.DT_F32, 0), (4097, synth.DT_F32, 1), (4097, synth.DT_BF16, -1), (8193, synth.DT_BF16, -1), (1025, synth.DT_F64, -1)],
                         ids=["f32", "parts", "bf16_4097", "bf16", "f64"])
@pytest.mark.parametrize("rows", [False, True])
def test_large_x(M, dtype, form, rows):
    """An X of 32 to 67 MB, several blocks of A for each workgroup of the builder, under both kernels.  Floats: a row of A is one element that parts
    do not hold, in the last block."""
    K, N = 4099, 48
    w = synth.random_masked(M, K, N, 16, 0.05, 0.1, M, dist="smallint", dtype=dtype)
    if rows:
        w.keep_rows = synth.pack_bits((np.arange(K) % 5 == 1)[None, :])
    if dtype == synth.DT_F32:
        keep = synth.unpack_bits(w.keep_a, K).astype(bool)
        keep[M - 1] = np.arange(K) == K - 3          # 4096 is on
        w.keep_a = synth.pack_bits(keep)
        w.X[M - 1, K - 3] = 2.0**60
        blocks = synth.unpack_bits(w.keep_blocks, N // 16).astype(bool)
        blocks[K - 3] = True
        w.keep_blocks = synth.pack_bits(blocks)
    ab, bb, C_ref, _ = oracle.run_workload(w)
    mm.mmm_set_option("float_form", form)
    try:
        run = HipRun(w)
        for path in (mm.MMM_PATH_MATRIX, mm.MMM_PATH_PAIRS):
            run.eng.set_path(path)
            a, b, C = run.run()
            assert mm.mmm_matmul_form(run.eng.maps) == max(form, 0)
            np.testing.assert_array_equal(a, ab)
            np.testing.assert_array_equal(b, bb)
            np.testing.assert_array_equal(C, C_ref)
            if dtype == synth.DT_F32:
                assert (np.abs(C[M - 1]) >= 2.0**60).any()
    finally:
        mm.mmm_set_option("float_form", -1)


@pytest.mark.parametrize("dtype,bw", [(synth.DT_BF16, 16), (synth.DT_F16, 32), (synth.DT_F16, 8)], ids=["bf16", "f16_32", "f16_8"])
@pytest.mark.parametrize("batches", [[1], [4], [0, 0], [1, 0, 2], [0, 1, 1, 4, 3], [1] * 6, [1] * 7, [0] * 8, [2, 3] * 4, [1] * 64 + [4], [4] * 16 + [1] * 3], ids=lambda b: f"{len(b)}_{sum(b)}")
def test_batches_of_a_queue(batches, dtype, bw):
    """16-bit types take three batches at a time and the last one or two by themselves: any number of them over the steps, in one and two ranges of
    K; the last tiles have waves without columns, which only copy."""
    M, K, N = 65, 128 * len(batches), 288 if bw == 32 else 272
    keep = np.zeros((K, N // bw), bool)
    rng = np.random.default_rng(K + bw)
    for s, b in enumerate(batches):
        keep[s * 128 + rng.permutation(128)[: max(32 * b - 5, 0)]] = True
    w = synth.random_masked(M, K, N, bw, 0.5, 1.0, K, dist="smallint", dtype=dtype)
    w.keep_blocks = synth.pack_bits(keep)
    for variant in (0, 1, 2, 6, 7):
        for split in (1, 2):
            print(variant, split, flush=True)
            _run(w, split, variant)


@pytest.mark.parametrize("bw", [8, 16, 32])
def test_order_in_a_step(bw):
    """Doubles in the widest tile read the operands of lists of more than ten k ahead of the next copy: lists around that, and of several batches."""
    lengths = [0, 1, 9, 10, 11, 12, 16, 17, 31, 33, 128, 0, 10, 11]
    M, segs, N = 70, len(lengths), 288
    keep = np.zeros((segs * 128, N // bw), bool)
    rng = np.random.default_rng(bw)
    for s in range(segs):
        for b in range(N // bw):
            keep[s * 128 + rng.permutation(128)[: lengths[(s + b * bw // 32) % segs]], b] = True
    w = synth.random_masked(M, segs * 128, N, bw, 0.5, 1.0, bw, dist="smallint", dtype=synth.DT_F64)
    w.keep_blocks = synth.pack_bits(keep)
    for split in (1, 3):
        _run(w, split, 1)
