"""GPU: a linear whose arena is larger than 4 GiB, where the offsets of the tables do not fit 32 bits."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


def test_tables_behind_4_gib_of_planes():
    """The planes alone are 4 GiB: the tables of both bitwidths lie beyond.  Some rows against the oracle: a lone GEMV with the bitwidth
    named and on the device, a batch, and a step."""
    import paper_2508_06041_amd as dp
    out, in_, p, kmin = 262144, 16384, 8, 7
    assert dp.binding.dpllm_linear_device_bytes(out, in_, p, kmin) > 2 ** 32
    g = torch.Generator(device="cuda").manual_seed(1)
    planes = torch.randint(-2 ** 31, 2 ** 31, (p, out, in_ // 32), dtype=torch.int32, device="cuda", generator=g)
    luts = {k: torch.randn(out, 1 << k, device="cuda", generator=g).half() for k in (7, 8)}
    model = dp.Model(1)
    model.dpllm_load_linear(0, planes, luts, kmin)
    rows = torch.cat([torch.tensor([0, 63, 64, out // 2, out - 1]), torch.randint(0, out, (59,), generator=torch.Generator().manual_seed(2))])
    some = synth.planes_np(planes[:, rows.cuda()].contiguous())
    X = synth.make_x(in_, 3, seed=3)
    xmax = float(X.double().abs().max())
    y, e = torch.empty(out, dtype=torch.float16, device="cuda"), torch.zeros(1, device="cuda")
    for k in (7, 8):
        lut = synth.lut_np(luts[k][rows.cuda()])
        ref = oracle.gemv(some, k, lut, synth.lut_np(X))
        # half a unit of the fp16 result, and fp32 sums of in_ exact products (random signs)
        wmax = np.abs(lut.view(np.float16).astype(np.float64)).max(axis=1)
        bound = 2.0 ** -10 * np.abs(ref) + 2.0 * np.sqrt(in_) * 2.0 ** -24 * wmax * xmax + 2.0 ** -24
        k_dev = torch.full((1,), k, dtype=torch.int32, device="cuda")
        model.dpllm_set_selector(0, k, k, dp.DPLLM_SEL_NONE)
        model.dpllm_decode_step([X[0].cuda()], [y], torch.zeros_like(k_dev), e)
        got = {"named": model.dpllm_gemv(0, k, X[0].cuda()), "device": model.dpllm_gemv(0, -1, X[0].cuda(), k_dev=k_dev),
               "batch": model.dpllm_gemv(0, k, X.cuda()), "step": y}
        for how, v in got.items():
            v = v.reshape(-1, out)[:, rows.cuda()].double().cpu().numpy()
            assert (np.abs(v - ref[:len(v)]) <= bound[:len(v)]).all(), (k, how)
    model.close()
