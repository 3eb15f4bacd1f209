"""GPU: a GEMV leaves the same bits whether the call names the bitwidth or the device does, and whichever pairs are attached."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def check(out, in_, batches, p=8, kmin=2):
    import paper_2508_06041_amd as dp
    lin = synth.make_linear(out, in_, p, kmin, seed=out + in_, device="cuda", keep_codes=False)
    model = dp.Model(1)
    model.dpllm_load_linear(0, lin["planes"], lin["luts"], kmin)
    X = synth.make_x(in_, 8, seed=out).cuda()
    k_dev = torch.zeros(1, dtype=torch.int32, device="cuda")
    pairs = [None, (p - 1, p), (min(3, p), min(6, p))]
    named = {}
    for pair in pairs:
        if pair is not None:
            model.dpllm_set_selector(0, *pair, dp.DPLLM_SEL_LINREG, alpha=0.0, beta=1.0, T=0.5)
        for k in range(kmin, p + 1):
            k_dev.fill_(k)
            for B in batches:
                x = X[:B].contiguous() if B > 1 else X[0]
                y = model.dpllm_gemv(0, k, x)
                assert torch.equal(named.setdefault((k, B), y), y), (pair, k, B)
                assert torch.equal(model.dpllm_gemv(0, -1, x, k_dev=k_dev), y), (pair, k, B)
    model.close()


# one right-hand side: blocks of 64 rows, up to 4096 columns (where both pipes are in use) and more; 64 to 8 rows per workgroup
@pytest.mark.parametrize("out,in_", [(8256, 4096), (9000, 544), (8200, 4096 + 32), (16390, 96), (4127, 288), (2049, 1056), (300, 8192 + 32)])
def test_one_right_hand_side(out, in_):
    check(out, in_, (1,))


# few rows of 64 column tiles and more, where four bits take four column groups and the other bitwidths eight: one pass and two
@pytest.mark.parametrize("out,in_", [(1, 8192), (500, 8192 + 32), (1100, 11008), (300, 32 * 513)])
def test_batch_on_few_rows(out, in_):
    check(out, in_, (2, 3, 4, 7))


# five to eight samples, one pass or two by the bitwidth: 33 and 64 row blocks (an odd number of blocks of 16 rows, the fewest column tiles), 65
# and 128 on few column tiles and on many; a linear of four bits, whose launch is the one for two passes
@pytest.mark.parametrize("out,in_,p", [(2049, 4096, 8), (4096, 4096 - 32, 8), (2600, 9216 + 32, 6), (4097, 1056, 8), (8192, 1024, 5), (6000, 32, 8),
                                      (4097, 4096 - 32, 8), (8192, 4096 + 160, 6), (2049, 4096, 4), (6000, 1056, 4), (4096, 2048, 8), (8256, 544, 8)])
def test_five_to_eight_samples(out, in_, p):
    check(out, in_, (5, 8), p)
