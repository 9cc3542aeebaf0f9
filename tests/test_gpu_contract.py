"""What the calls promise beyond the numbers: which operands a product is made from, what a build leaves in the
workspace and for whom, which products are skipped."""
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


# ---- which Y a product is made from ------------------------------------------------------------
@pytest.mark.parametrize("rows", [None, 0.5], ids=["all", "rows"])
@pytest.mark.parametrize("asked", [-1, mm.MMM_PATH_MATRIX, mm.MMM_PATH_PAIRS], ids=["auto", "matrix", "pairs"])
@pytest.mark.parametrize("dtype", DTYPES, ids=IDS)
def test_another_y_than_the_one_built_from(dtype, asked, rows):
    """The product is that of the Y that is passed, whichever kernel is chosen: the matrix kernel has only the values of
    the Y that the maps were built from."""
    w = synth.random_masked(100, 300, 64, 16, 0.3, 0.3, 77, dist="smallint", dtype=dtype, p_rows=rows)
    _, _, C_ref, _ = oracle.run_workload(w)
    run = HipRun(w)
    run.eng.set_path(asked)
    run.build()
    other = run.Y.clone()                                            # the same values elsewhere
    halves = {synth.DT_BF16: torch.bfloat16, synth.DT_F16: torch.float16}
    twice = run.Y.clone()
    twice = (twice.view(halves[dtype]) * 2).view(torch.int16) if dtype in halves else twice * 2
    wide = torch.zeros((w.K, w.N + 8), dtype=run.Y.dtype, device="cuda")    # another leading dimension
    wide[:, : w.N] = run.Y
    for Y, factor in ((run.Y, 1), (other, 1), (twice, 2), (wide, 1), (run.Y, 1)):
        for call in (run.eng.matmul, run.eng.matmul_static_scratch):
            run.Cbuf.fill_(float("nan"))
            call(run.X, Y, run.C)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(run.C.cpu().numpy(), factor * C_ref)


def test_another_y_that_no_kernel_can_read():
    """Rows too far apart for the pair kernel, and not the Y whose values the matrix kernel has."""
    w = synth.random_masked(40, 200, 64, 16, 0.3, 0.5, 88, dist="smallint")
    run = HipRun(w, ldy=(1 << 18) + 8)
    run.build()
    other = torch.zeros((w.K + 1, (1 << 18) + 8), device="cuda")[1:, : w.N]
    other.copy_(run.Y)
    with pytest.raises(mm.MmmError) as e:
        run.eng.matmul(run.X, other, run.C)
    assert e.value.status == mm.binding.MMM_ERR_MAPS_MISMATCH
    run.matmul()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(run.C.cpu().numpy(), oracle.run_workload(w)[2])


# ---- inspection ------------------------------------------------------------------------------
def test_inspection_needs_no_stream_of_the_build():
    """A program builds on a stream of its own, waits for it, gives that stream other work and looks at the lists from
    another stream."""
    w = synth.random_masked(100, 700, 96, 16, 0.3, 0.4, 5, dist="smallint", p_rows=0.5)
    run = HipRun(w)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    run.eng.build_maps(run.X, run.Y, w.pred, w.threshold, run.keep_a, run.keep_rows, run.keep_blocks, stream=side)
    side.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(50_000_000)          # some 20 ms
    counts, entries = run.eng.a_lists()
    colany_c = run.eng.compacted()[2]
    a = synth.unpack_bits(oracle.a_bits(w.X, w.pred, w.threshold, w.keep_a), w.K)
    a = a[:, synth.unpack_bits(w.keep_rows.reshape(1, -1), w.K)[0]]
    want = np.array([[a[i:i + 64, k:k + 128].sum() for k in range(0, a.shape[1], 128)] for i in range(0, w.M, 64)])
    got, got_any = counts.clone(), colany_c.clone()
    torch.cuda.current_stream().synchronize()
    np.testing.assert_array_equal(got.cpu().numpy()[:, : want.shape[1]], want)
    a = np.concatenate([a, np.zeros(((-w.M) % 32, a.shape[1]), bool)]).reshape(-1, 32, a.shape[1]).any(axis=1)
    words = (a.shape[1] + 63) // 64
    np.testing.assert_array_equal(got_any.cpu().numpy().view(np.uint64)[:, :words], synth.pack_bits(a))
    torch.cuda.synchronize()


# ---- columns of A that are zero in all 64 rows of a tile ---------------------------------------
def _structured(M, K, N, bw, p_cols, p_b, p_rows, seed):
    """Every 64 rows of A have their own share p_cols of columns on, dense inside; rows of Y that meet only dead columns of
    a tile hold Inf, which shows in that tile if they are multiplied."""
    w = synth.random_masked(M, K, N, bw, 0.5, p_b, seed, dist="smallint", p_rows=p_rows)
    rng = np.random.default_rng(seed)
    on = rng.random(((M + 63) // 64, K)) < p_cols
    keep = synth.unpack_bits(w.keep_a, K) & np.repeat(on, 64, axis=0)[:M]
    w.keep_a = synth.pack_bits(keep)
    return w, keep


@pytest.mark.parametrize("counted", [True, False], ids=["stats", "no_stats"])
@pytest.mark.parametrize("M,K,N,bw,p_cols,p_b,p_rows", [
    (65, 1280, 48, 16, 0.1, 1.0, None), (200, 1111, 272, 8, 0.1, 0.9, None), (130, 2100, 288, 32, 0.05, 1.0, None),
    (70, 9000, 96, 16, 0.1, 0.9, None),          # more steps than list lengths are held for at a time
    (130, 6000, 272, 16, 0.1, 1.0, 0.3),         # over the live rows of B
    (100, 128, 64, 16, 0.0, 1.0, None),          # nothing on
])
def test_dead_columns_are_not_multiplied(M, K, N, bw, p_cols, p_b, p_rows, counted):
    w, keep = _structured(M, K, N, bw, p_cols, p_b, p_rows, M + K)
    _, _, C_ref, _ = oracle.run_workload(w)
    # the first tile's dead columns: Inf in those rows of Y
    dead = ~keep[:64].any(axis=0)
    w.Y = np.where(dead[:, None], np.float32(np.inf), w.Y)
    run = HipRun(w)
    run.eng.set_path(mm.MMM_PATH_MATRIX)
    run.build()
    if counted:
        run.eng.stats()       # (without counts the lists of packed B are taken as they are: looking makes every call longer)
    for variant, split in [(-1, 0)] + [(v, 1 + v % 3) for v in range(mm.mmm_matmul_variant_count()) if not mm.mmm_matmul_variant_name(v).startswith("R2")]:
        print("variant", variant, "split", split, flush=True)
        run.eng.set_plan(variant, split)
        run.Cbuf.fill_(float("nan"))
        run.matmul()
        torch.cuda.synchronize()
        if counted:
            np.testing.assert_array_equal(run.C.cpu().numpy()[:64], C_ref[:64])
        else:
            got = run.C.cpu().numpy()[:64]
            assert np.isnan(got).any()
            np.testing.assert_array_equal(got[~np.isnan(got)], C_ref[:64][~np.isnan(got)])


@pytest.mark.parametrize("bw", [8, 16, 32])
@pytest.mark.parametrize("M,p_rows", [(64, None), (30, None), (200, None), (30, 0.5), (200, 0.5)])
def test_lists_without_dead_columns_of_every_length(M, p_rows, bw):
    """Segments whose lists hold every number of slots around the batch and quad sizes, before and after the dead columns
    are left out, in every tile; waves without columns; the last segment a short one."""
    lengths = [0, 1, 3, 4, 5, 15, 16, 17, 31, 32, 33, 127, 128, 0, 64]
    segs, N = 66, 160
    K = segs * 128 - 70
    rng = np.random.default_rng(bw + M)
    w = synth.random_masked(M, K, N, bw, 1.0, 0.9, 177 + bw, dist="smallint", p_rows=p_rows)
    on = np.zeros(((M + 63) // 64, segs * 128), bool)
    for t in range(on.shape[0]):
        for s in range(segs):
            on[t, s * 128 + rng.permutation(128)[:lengths[(s + 7 * t) % len(lengths)]]] = True
    w.keep_a = synth.pack_bits(np.repeat(on[:, :K], 64, axis=0)[:M] & (rng.random((M, K)) < 0.7))
    _, _, C_ref, _ = oracle.run_workload(w)
    run = HipRun(w)
    run.eng.set_path(mm.MMM_PATH_MATRIX)
    run.build()
    run.eng.stats()
    for variant in range(mm.mmm_matmul_variant_count()):
        if mm.mmm_matmul_variant_name(variant).startswith("R2") != (M <= 32):
            continue
        for split in (1, 2):
            print("variant", variant, "split", split, flush=True)
            run.eng.set_plan(variant, split)
            run.Cbuf.fill_(float("nan"))
            run.matmul()
            torch.cuda.synchronize()
            np.testing.assert_array_equal(run.C.cpu().numpy(), C_ref)


# ---- the choice between the kernels where A keeps few of its elements --------------------------
@pytest.mark.parametrize("dtype", [synth.DT_BF16, synth.DT_F16], ids=["bf16", "f16"])
@pytest.mark.parametrize("M,K,N,p_a,p_b", [(512, 8192, 4096, 0.03, 0.1), (512, 8192, 4096, 0.03, 0.5)])
def test_16_bit_inputs_with_few_elements_of_a_take_the_matrix_kernel(M, K, N, p_a, p_b, dtype):
    w = synth.random_masked(M, K, N, 16, p_a, p_b, 9, dist="smallint", dtype=dtype)
    run = HipRun(w)
    run.build()
    run.eng.stats()
    assert run.eng.path() == mm.MMM_PATH_MATRIX


# ---- row-compacted mode: the transposed map over k, for calls that want it where the matrix kernel was expected --------
def _compacted(seed, dtype=synth.DT_F32, p_rows=0.3):
    w = synth.random_masked(100, 1500, 288, 16, 0.3, 0.4, seed, dist="smallint", dtype=dtype, p_rows=p_rows)
    run = HipRun(w)
    run.eng.set_path(mm.MMM_PATH_MATRIX)
    return w, run, oracle.run_workload(w)[2]


def _fused(w, run, C, stream=None):
    run.eng.matmul_fused(run.X, run.Y, C, w.pred, w.threshold, run.keep_a, stream=stream)


def test_the_transposed_map_is_made_once_per_build():
    """Seen by what a call does with a map that was cleared behind its back: a call that made it again would be right."""
    w, run, C_ref = _compacted(11)
    bt = run.eng.bt_bits()             # nothing built: the address alone
    for _ in range(2):
        bt.fill_(-1)
        run.build()
        for _ in range(2):
            _fused(w, run, run.C)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(run.C.cpu().numpy(), C_ref)
        run.eng.set_path(mm.MMM_PATH_PAIRS)
        run.matmul()
        run.eng.set_path(mm.MMM_PATH_MATRIX)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(run.C.cpu().numpy(), C_ref)
        bt.zero_()
        _fused(w, run, run.C)
        torch.cuda.synchronize()
        assert not run.C.any()


def test_the_transposed_map_from_several_streams():
    """The stream whose call makes the map is held up; calls on other streams, in front of that, wait for the map."""
    w, run, C_ref = _compacted(12)
    run.eng.bt_bits().fill_(-1)
    streams = [torch.cuda.Stream() for _ in range(3)]
    outs = [torch.full_like(run.C, float("nan")) for _ in streams]
    for _ in range(3):
        run.build()
        for s in streams:
            s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(streams[0]):
            torch.cuda._sleep(20_000_000)          # some 10 ms
        for s, C in zip(streams, outs):
            _fused(w, run, C, stream=s)
        torch.cuda.synchronize()
        for C in outs:
            np.testing.assert_array_equal(C.cpu().numpy(), C_ref)
            C.fill_(float("nan"))
        torch.cuda.synchronize()


def test_the_transposed_map_in_a_graph():
    """A captured call is right at every replay, also after builds of other rows between the replays."""
    w, run, C_ref = _compacted(13)
    w2, _, C2_ref = _compacted(14, p_rows=0.6)
    w2.X, w2.keep_a = w.X, w.keep_a
    C2_ref = oracle.run_workload(w2)[2]
    run.build()
    _fused(w, run, run.C)              # made and seen to be made before the capture
    torch.cuda.synchronize()
    _fused(w, run, run.C)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _fused(w, run, run.C)
    for source, want in ((w, C_ref), (w2, C2_ref), (w, C_ref), (w2, C2_ref)):
        run.Y.copy_(torch.from_numpy(source.Y))
        run.keep_rows.copy_(torch.from_numpy(source.keep_rows.view(np.int64)))
        run.keep_blocks.copy_(torch.from_numpy(source.keep_blocks.view(np.int64)))
        run.build()
        for _ in range(2):
            run.Cbuf.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            np.testing.assert_array_equal(run.C.cpu().numpy(), want)
        run.Cbuf.fill_(float("nan"))
        _fused(w, run, run.C)          # and beside it, not captured
        torch.cuda.synchronize()
        np.testing.assert_array_equal(run.C.cpu().numpy(), want)


def test_the_transposed_map_after_replayed_builds():
    """Builds of other rows that come from a graph, which the handle does not see, and calls that are not captured."""
    w, run, C_ref = _compacted(15)
    w2, _, _ = _compacted(16, p_rows=0.6)
    w2.X, w2.keep_a = w.X, w.keep_a
    C2_ref = oracle.run_workload(w2)[2]
    bt = run.eng.bt_bits()
    run.build()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run.build()
    for source, want in ((w, C_ref), (w2, C2_ref), (w, C_ref), (w2, C2_ref)):
        run.Y.copy_(torch.from_numpy(source.Y))
        run.keep_rows.copy_(torch.from_numpy(source.keep_rows.view(np.int64)))
        run.keep_blocks.copy_(torch.from_numpy(source.keep_blocks.view(np.int64)))
        bb = oracle.b_bits(source.Y, w.bw, source.keep_rows, source.keep_blocks)
        graph.replay()
        for _ in range(2):
            run.Cbuf.fill_(float("nan"))
            _fused(w, run, run.C)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(run.C.cpu().numpy(), want)
        bt.fill_(-1)
        got = run.eng.bt_bits()
        np.testing.assert_array_equal(got.cpu().numpy().view(np.uint64), synth.pack_bits(synth.unpack_bits(bb, w.NB).T))
