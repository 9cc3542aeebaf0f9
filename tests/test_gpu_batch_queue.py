"""The matrix kernel's queue of list batches (16-bit types, floats in parts): 64 (parts: 46 to 64) are planned at a time, whatever steps they
belong to, so lists of every length fall on the seams of the plan.  Small whole numbers: sums are exact in any order."""
import numpy as np
import pytest

import mmm_synth as synth
import paper_2402_14118_amd as mm
from test_gpu_parity import check_workload

pytestmark = pytest.mark.gpu

FORMS = [(synth.DT_BF16, -1), (synth.DT_F16, -1), (synth.DT_F32, 1)]


@pytest.fixture(autouse=True)
def matrix_path():
    mm.mmm_set_option("matmul_path", mm.MMM_PATH_MATRIX)
    yield
    mm.mmm_set_option("matmul_path", -1)
    mm.mmm_set_option("float_form", -1)


@pytest.mark.parametrize("dtype,form", FORMS, ids=["bf16", "f16", "parts"])
@pytest.mark.parametrize("bw,steps,longest", [(16, 61, 32), (16, 62, 32), (16, 63, 33), (16, 64, 33), (8, 67, 128), (32, 150, 128), (32, 20, 128)])
def test_seams_of_the_plan(bw, steps, longest, dtype, form):
    mm.mmm_set_option("float_form", form)
    M, K, N = 70, steps * 128 - 3, 96
    rng = np.random.default_rng(bw * steps)
    keep = np.zeros((K, N // bw), bool)
    for b in range(N // bw):
        for s in range(steps):   # short, long and empty lists, at random and in runs
            n = 0 if rng.random() < 0.1 else rng.integers(1, longest + 1) if (s + 5 * b) // 7 % 2 else rng.integers(1, 20)
            at = s * 128 + rng.permutation(128)[:n]
            keep[at[at < K], b] = True
    w = synth.random_masked(M, K, N, bw, 0.5, 1.0, bw + steps, dist="smallint", dtype=dtype)
    w.keep_blocks = synth.pack_bits(keep)
    check_workload(w, "seams", exact=True)
