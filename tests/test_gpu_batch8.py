"""GPU: five to eight right-hand sides in one pass over the planes, against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


# two passes of four or one pass; fewer column tiles than wavefronts; more than a thousand row blocks (65604 rows);
# rows and tiles that no block or group divides
@pytest.mark.parametrize("out,in_", [(1, 32), (130, 4096 + 160), (1000, 1056), (4127, 288), (8200, 544), (16390, 96), (65604, 1184)])
def test_gemv_five_to_eight_samples(out, in_):
    import paper_2508_06041_amd as dp
    many = out > 60000
    p, ks = (5, (3, 4, 5)) if many else (8, range(1, 9))
    lin = synth.make_linear(out, in_, p, 1, seed=out + in_, device="cuda", keep_codes=False)
    model = dp.Model(1)
    model.dpllm_load_linear(0, lin["planes"], lin["luts"], 1)
    planes = synth.planes_np(lin["planes"])
    X = synth.make_x(in_, 8, seed=out)
    xmax = float(X.double().abs().max())
    for k in ks:
        lut = synth.lut_np(lin["luts"][k])
        ref = oracle.gemv(planes, k, lut, synth.lut_np(X))
        # half a unit of the fp16 result, and fp32 sums of in_ exact products (random signs)
        wmax = np.abs(lut.view(np.float16).astype(np.float64)).max(axis=1)
        bound = 2.0 ** -10 * np.abs(ref) + 2.0 * np.sqrt(in_) * 2.0 ** -24 * wmax * xmax + 2.0 ** -24
        for B in ((8,) if many else (5, 6, 7, 8)):
            y = torch.full((B + 1, out), 7.0, dtype=torch.float16, device="cuda")     # one row more than may be written
            model.dpllm_gemv(0, k, X[:B].cuda(), y=y[:B])
            assert (np.abs(y[:B].double().cpu().numpy() - ref[:B]) <= bound[:B]).all(), (k, B)
            assert (y[B] == 7.0).all()
    model.close()


def test_eight_samples_add_as_four_do():
    """The sums of five to eight right-hand sides are no longer chains of additions than those of four: the same bits, where
    both take one pass of 64 rows per workgroup."""
    import paper_2508_06041_amd as dp
    out, in_ = 129 * 64, 4096 + 32
    lin = synth.make_linear(out, in_, 8, 3, seed=5, device="cuda", keep_codes=False)
    model = dp.Model(1)
    model.dpllm_load_linear(0, lin["planes"], lin["luts"], 3)
    X = synth.make_x(in_, 8, seed=6).cuda()
    for k in range(3, 9):
        halves = [model.dpllm_gemv(0, k, X[i:i + 4].contiguous()) for i in (0, 4)]
        assert torch.equal(model.dpllm_gemv(0, k, X), torch.cat(halves)), k
    model.close()


# 33 and 64 row blocks, where 5 bits and more take one pass with four column groups and fewer bits two passes with two: the fewest column tiles
# that take it, a last step of one tile and a ragged last word
@pytest.mark.parametrize("out,in_", [(2049, 4096), (4096, 4096 - 32), (2600, 9216 + 32)])
def test_gemv_five_to_eight_samples_of_a_narrow_launch(out, in_):
    import paper_2508_06041_amd as dp
    lin = synth.make_linear(out, in_, 8, 3, seed=out + in_, device="cuda", keep_codes=False)
    model = dp.Model(1)
    model.dpllm_load_linear(0, lin["planes"], lin["luts"], 3)
    planes = synth.planes_np(lin["planes"])
    X = synth.make_x(in_, 8, seed=out)
    xmax = float(X.double().abs().max())
    k_dev = torch.zeros(1, dtype=torch.int32, device="cuda")
    for k in range(3, 9):
        lut = synth.lut_np(lin["luts"][k])
        ref = oracle.gemv(planes, k, lut, synth.lut_np(X))
        wmax = np.abs(lut.view(np.float16).astype(np.float64)).max(axis=1)
        bound = 2.0 ** -10 * np.abs(ref) + 2.0 * np.sqrt(in_) * 2.0 ** -24 * wmax * xmax + 2.0 ** -24
        for B in (5, 8):
            for dev in (False, True):        # the bitwidth on the device: the launch is the one for one pass, whichever it is
                y = torch.full((B + 1, out), 7.0, dtype=torch.float16, device="cuda")     # one row more than may be written
                k_dev.fill_(k)
                model.dpllm_gemv(0, -1 if dev else k, X[:B].cuda(), y=y[:B], k_dev=k_dev)
                assert (np.abs(y[:B].double().cpu().numpy() - ref[:B]) <= bound[:B]).all(), (k, B, dev)
                assert (y[B] == 7.0).all()
    model.close()


# 65, 94 and 128 row blocks, one pass with two column groups: few columns (5 bits and more only) and many, an odd last step of one tile
@pytest.mark.parametrize("out,in_", [(65 * 64 - 63, 4096 - 32), (6000, 1056), (8192, 4096 + 160)])
def test_gemv_five_to_eight_samples_with_two_column_groups(out, in_):
    import paper_2508_06041_amd as dp
    lin = synth.make_linear(out, in_, 8, 2, seed=out + in_, device="cuda", keep_codes=False)
    model = dp.Model(1)
    model.dpllm_load_linear(0, lin["planes"], lin["luts"], 2)
    planes = synth.planes_np(lin["planes"])
    X = synth.make_x(in_, 8, seed=out)
    xmax = float(X.double().abs().max())
    for k in range(2, 9):
        lut = synth.lut_np(lin["luts"][k])
        ref = oracle.gemv(planes, k, lut, synth.lut_np(X))
        # half a unit of the fp16 result, and fp32 sums of in_ exact products (random signs)
        wmax = np.abs(lut.view(np.float16).astype(np.float64)).max(axis=1)
        bound = 2.0 ** -10 * np.abs(ref) + 2.0 * np.sqrt(in_) * 2.0 ** -24 * wmax * xmax + 2.0 ** -24
        for B in (5, 8):
            y = torch.full((B + 1, out), 7.0, dtype=torch.float16, device="cuda")     # one row more than may be written
            model.dpllm_gemv(0, k, X[:B].cuda(), y=y[:B])
            assert (np.abs(y[:B].double().cpu().numpy() - ref[:B]) <= bound[:B]).all(), (k, B)
            assert (y[B] == 7.0).all()
    model.close()
