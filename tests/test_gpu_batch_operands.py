"""GPU: where every activation of a small batch meets its weight.  Samples that are zero but for one column return the weights of
that column, exactly."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


# four samples with 1, 2, 4 and 8 column groups per wavefront (4 bits: not with 8); eight with 1 and (5 bits and more) 4; one on the matrix
# pipe, rows of many tiles and (up to 4 bits) of few.  The columns: every place of a word, in the first tile, one in the middle and the
# ragged last one
@pytest.mark.parametrize("out,in_,B", [(8200, 288, 4), (4200, 288, 3), (2100, 800, 2), (100, 8192 + 96, 4), (8200, 288, 8), (2049, 4096 + 96, 5), (8200, 288, 1),
                                      (8200, 4096 + 96, 1)])
def test_one_column_at_a_time(out, in_, B):
    import paper_2508_06041_amd as dp
    lin = synth.make_linear(out, in_, 8, 1, seed=out + in_, device="cuda", keep_codes=False)
    model = dp.Model(1)
    model.dpllm_load_linear(0, lin["planes"], lin["luts"], 1)
    planes = synth.planes_np(lin["planes"])
    columns = [w * 32 + c for w in (0, (in_ // 32) // 2, in_ // 32 - 1) for c in range(32)]
    for k in range(1, 9):
        lut = synth.lut_np(lin["luts"][k]).view(np.float16)
        for i in range(0, len(columns), B):
            cols = [columns[(i + b) % len(columns)] for b in range(B)]
            X = torch.zeros(B, in_, dtype=torch.float16)
            X[torch.arange(B), torch.tensor(cols)] = 1.0
            y = model.dpllm_gemv(0, k, X.cuda()).cpu().numpy()
            for b, c in enumerate(cols):
                code = np.zeros(out, dtype=np.int64)
                for plane in range(k):
                    code = code * 2 + ((planes[plane, :, c // 32] >> (c % 32)) & 1)
                assert np.array_equal(y[b], lut[np.arange(out), code]), (k, c)
    model.close()
