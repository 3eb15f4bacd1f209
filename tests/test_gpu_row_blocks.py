"""GPU: launches of so many rows that a workgroup takes several blocks of 64 of them, against the CPU oracle on some of the rows."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


# 2049 row blocks on 1025 workgroups, the last of which has one and a ragged one; fewer column tiles than wavefronts, rows whose activations a
# wavefront keeps (up to 4096 columns) and longer ones
@pytest.mark.parametrize("in_", [96, 1184, 4096 + 96])
def test_several_row_blocks_per_workgroup(in_):
    import paper_2508_06041_amd as dp
    out, p, kmin = 2048 * 64 + 37, 8, 2
    g = torch.Generator(device="cuda").manual_seed(in_)
    planes = torch.randint(-2 ** 31, 2 ** 31, (p, out, in_ // 32), dtype=torch.int32, device="cuda", generator=g)
    luts = {k: torch.randn(out, 1 << k, device="cuda", generator=g).half() for k in range(kmin, p + 1)}
    model = dp.Model(1)
    model.dpllm_load_linear(0, planes, luts, kmin)
    # whole blocks of the first workgroups' first and second turn, of the middle, and the last rows
    rows = torch.cat([torch.arange(b * 64, min(out, b * 64 + 64)) for b in (0, 1, 512, 1023, 1024, 1025, 1026, 2047, 2048)]).cuda()
    some = synth.planes_np(planes[:, rows].contiguous())
    X = synth.make_x(in_, 8, seed=in_)
    xmax = float(X.double().abs().max())
    k_dev = torch.zeros(1, dtype=torch.int32, device="cuda")
    for k in range(kmin, p + 1):
        lut = synth.lut_np(luts[k][rows])
        ref = oracle.gemv(some, k, lut, synth.lut_np(X))
        # half a unit of the fp16 result, and fp32 sums of in_ exact products (random signs)
        wmax = np.abs(lut.view(np.float16).astype(np.float64)).max(axis=1)
        bound = 2.0 ** -10 * np.abs(ref) + 2.0 * np.sqrt(in_) * 2.0 ** -24 * wmax * xmax + 2.0 ** -24
        k_dev.fill_(k)
        for B in (1, 3, 8):
            x = X[:B].cuda() if B > 1 else X[0].cuda()
            y = model.dpllm_gemv(0, k, x)
            assert torch.equal(model.dpllm_gemv(0, -1, x, k_dev=k_dev), y), (k, B)
            assert (np.abs(y.reshape(B, out)[:, rows].double().cpu().numpy() - ref[:B]) <= bound[:B]).all(), (k, B)
    model.close()
