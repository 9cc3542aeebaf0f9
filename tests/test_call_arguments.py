"""Arguments of the Python entry points, checked without a GPU: what they hand to the C ABI, which refuses these calls
(nothing is built) before it touches a device."""
import numpy as np
import pytest
import torch

import paper_2402_14118_amd as mm
from paper_2402_14118_amd import binding as B


@pytest.fixture
def engine():
    """An engine on maps of a workspace that is never touched."""
    eng = object.__new__(mm.MaskedMatmul)
    need = mm.mmm_maps_workspace_bytes(64, 128, 64, 16)
    eng.maps, eng.dtype, eng.bw = mm.mmm_maps_init(0x7000_0000_0000, need, 64, 128, 64, 16), mm.MMM_F32, 16
    yield eng
    eng.close()


@pytest.mark.parametrize("accumulate", [False, True, 0, 1, np.bool_(True), 1.0, np.float32(0.0), np.int64(1)], ids=repr)
def test_accumulate_takes_whatever_int_takes(engine, accumulate):
    X, Y, C = torch.zeros(64, 128), torch.zeros(128, 64), torch.zeros(64, 64)
    for call in (engine.matmul, engine.matmul_static_scratch, engine.matmul_fused):
        with pytest.raises(mm.MmmError) as e:
            call(X, Y, C, accumulate=accumulate, stream=0)
        assert e.value.status == B.MMM_ERR_MAPS_MISMATCH
