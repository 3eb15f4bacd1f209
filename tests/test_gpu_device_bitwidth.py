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
