"""GPU: the launches that give a workgroup 64, 32, 16 or 8 rows, and the bitwidths 1 and 2, against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dp():
    import paper_2508_06041_amd as dp
    assert torch.cuda.is_available()
    return dp


def bound(y_ref, lut, x_bits, in_):
    """Per row: half a unit of the fp16 result, and fp32 sums of `in_` exact products (random signs)."""
    wmax = np.abs(lut.view(np.float16).astype(np.float64)).max(axis=1)
    xmax = float(np.abs(x_bits.view(np.float16).astype(np.float64)).max())
    return 2.0 ** -10 * np.abs(y_ref) + 2.0 * np.sqrt(in_) * 2.0 ** -24 * wmax * xmax + 2.0 ** -24


# blocks of 64 rows 1, 3, 33 .. 130 (eight to one column groups); column tiles no multiple of the groups; rows no
# multiple of the workgroup's
@pytest.mark.parametrize("out,in_", [(1, 32), (70, 160), (185, 8192 + 224), (2049, 1056), (3000, 416), (4127, 288), (8200, 544), (16390, 96)])
def test_gemv_every_bitwidth_and_batch(dp, out, in_):
    lin = synth.make_linear(out, in_, 8, 1, seed=out + in_, device="cuda", keep_codes=False)
    model = dp.Model(1)
    model.dpllm_load_linear(0, lin["planes"], lin["luts"], 1)
    planes = synth.planes_np(lin["planes"])
    X = synth.make_x(in_, 5, seed=out)
    for k in range(1, 9):
        lut = synth.lut_np(lin["luts"][k])
        ref = oracle.gemv(planes, k, lut, synth.lut_np(X))
        for B in (1, 3, 5):
            got = model.dpllm_gemv(0, k, (X[:B] if B > 1 else X[0]).cuda()).double().cpu().numpy().reshape(B, out)
            for b in range(B):
                assert (np.abs(got[b] - ref[b]) <= bound(ref[b], lut, synth.lut_np(X[b]), in_)).all(), (k, B, b)
    model.close()


# two, four and eight column groups, wavefronts of several steps (the tile of the next step is asked for while this one is
# decoded), the last step with a tile for some of the groups only
@pytest.mark.parametrize("out,in_", [(300, 32 * 1035), (2500, 6688), (4200, 12320)])
def test_gemv_several_steps(dp, out, in_):
    lin = synth.make_linear(out, in_, 8, 1, seed=out + in_, device="cuda", keep_codes=False)
    model = dp.Model(1)
    model.dpllm_load_linear(0, lin["planes"], lin["luts"], 1)
    planes = synth.planes_np(lin["planes"])
    X = synth.make_x(in_, 7, seed=out)
    for k in (1, 3, 4, 5, 8):
        lut = synth.lut_np(lin["luts"][k])
        ref = oracle.gemv(planes, k, lut, synth.lut_np(X))
        for B in (1, 4, 7):
            got = model.dpllm_gemv(0, k, (X[:B] if B > 1 else X[0]).cuda()).double().cpu().numpy().reshape(B, out)
            for b in range(B):
                assert (np.abs(got[b] - ref[b]) <= bound(ref[b], lut, synth.lut_np(X[b]), in_)).all(), (k, B, b)
    model.close()


# few rows of 64 column tiles and more: a batch at k = 4 takes four column groups, in a launch for four or, where the device says k, for eight
@pytest.mark.parametrize("out,in_,B", [(1, 8192, 2), (500, 8192 + 32, 4), (1100, 11008, 3), (300, 32 * 513, 7)])
def test_four_bit_batch_on_few_rows(dp, out, in_, B):
    lin = synth.make_linear(out, in_, 5, 3, seed=out + in_, device="cuda", keep_codes=False)
    model = dp.Model(1)
    model.dpllm_load_linear(0, lin["planes"], lin["luts"], 3)
    lut = synth.lut_np(lin["luts"][4])
    X = synth.make_x(in_, B, seed=out)
    ref = oracle.gemv(synth.planes_np(lin["planes"]), 4, lut, synth.lut_np(X))
    k_dev = torch.full((1,), 4, dtype=torch.int32, device="cuda")
    for got in (model.dpllm_gemv(0, 4, X.cuda()), model.dpllm_gemv(0, -1, X.cuda(), k_dev=k_dev)):
        got = got.double().cpu().numpy()
        for b in range(B):
            assert (np.abs(got[b] - ref[b]) <= bound(ref[b], lut, synth.lut_np(X[b]), in_)).all(), b
    model.close()


@pytest.mark.parametrize("out,in_", [(40, 160), (20000, 96)])
def test_two_bits_unused_infinite_centroid(dp, out, in_):
    """Columns past the end of a row carry code 0; an infinite centroid of that code must not reach the sum."""
    rng = np.random.default_rng(out)
    planes = rng.integers(0, 2 ** 32, size=(2, out, in_ // 32), dtype=np.uint32)
    planes[1] |= ~planes[0]                       # the code 0 does not occur
    luts = {1: rng.standard_normal((out, 2)).astype(np.float16), 2: rng.standard_normal((out, 4)).astype(np.float16)}
    luts[2][:, 0] = np.inf
    luts = {k: v.view(np.uint16) for k, v in luts.items()}
    model = dp.Model(1)
    model.dpllm_load_linear(0, planes, luts, 1)
    X = synth.make_x(in_, 3, seed=1)
    finite = luts[2].copy()
    finite[:, 0] = 0
    ref = oracle.gemv(planes, 2, finite, synth.lut_np(X))
    for B in (1, 3):
        got = model.dpllm_gemv(0, 2, (X[:B] if B > 1 else X[0]).cuda()).double().cpu().numpy().reshape(B, out)
        for b in range(B):
            assert (np.abs(got[b] - ref[b]) <= bound(ref[b], finite, synth.lut_np(X[b]), in_)).all(), (B, b)
    model.close()


def test_two_bits_subnormal_centroids(dp):
    out, in_ = 96, 256
    rng = np.random.default_rng(0)
    planes = rng.integers(0, 2 ** 32, size=(2, out, in_ // 32), dtype=np.uint32)
    luts = {k: rng.integers(1, 64, size=(out, 1 << k)).astype(np.uint16) for k in (1, 2)}    # up to 63 x 2^-24
    model = dp.Model(1)
    model.dpllm_load_linear(0, planes, luts, 1)
    X = 512.0 * synth.make_x(in_, 3, seed=2)
    for k in (1, 2):
        ref = oracle.gemv(planes, k, luts[k], synth.lut_np(X))
        for B in (1, 3):
            got = model.dpllm_gemv(0, k, (X[:B] if B > 1 else X[0]).cuda()).double().cpu().numpy().reshape(B, out)
            for b in range(B):
                assert (np.abs(got[b] - ref[b]) <= bound(ref[b], luts[k], synth.lut_np(X[b]), in_)).all(), (k, B, b)
    model.close()


def test_decode_step_with_a_two_bit_child(dp):
    """A pair (2, 3): bitwidths below 3 share the launches of the others."""
    shapes = [(260, 384), (70, 384), (200, 260 // 4 * 4 + 28)]
    lins = [synth.make_linear(o, i, 4, 2, seed=o + i) for o, i in shapes]
    model = dp.Model(len(lins))
    xs, ys = [], []
    for i, lin in enumerate(lins):
        model.dpllm_load_linear(i, synth.planes_np(lin["planes"]), {k: synth.lut_np(v) for k, v in lin["luts"].items()}, 2)
        model.dpllm_set_selector(i, 2, 3, dp.DPLLM_SEL_LINREG, alpha=0.0, beta=1.0, T=0.5 if i == 1 else 2.0)
        xs.append(synth.make_x(shapes[i][1], 1, seed=i)[0].cuda())
        ys.append(torch.empty(shapes[i][0], dtype=torch.float16, device="cuda"))
    k_dev = torch.zeros(len(lins), dtype=torch.int32, device="cuda")
    e_dev = torch.zeros(len(lins), dtype=torch.float32, device="cuda")
    model.dpllm_decode_step(xs, ys, k_dev, e_dev)
    assert k_dev.tolist() == [2, 3, 2]
    for lin, x, y, k, (out, in_) in zip(lins, xs, ys, (2, 3, 2), shapes):
        lut = synth.lut_np(lin["luts"][k])
        ref = oracle.gemv(synth.planes_np(lin["planes"]), k, lut, synth.lut_np(x))
        assert (np.abs(y.double().cpu().numpy() - ref) <= bound(ref, lut, synth.lut_np(x), in_)).all()
    model.close()


# eight column groups for a batch (4 bits: four): the most row blocks and the fewest column tiles that take them, one row, a last step of
# one tile whose last words lie past the row
@pytest.mark.parametrize("out,in_", [(2048, 8192), (1, 28672), (1017, 8192 + 32), (500, 9216 + 96)])
def test_gemv_batch_of_few_rows_on_long_columns(dp, out, in_):
    lin = synth.make_linear(out, in_, 8, 1, seed=out + in_, device="cuda", keep_codes=False)
    model = dp.Model(1)
    model.dpllm_load_linear(0, lin["planes"], lin["luts"], 1)
    planes = synth.planes_np(lin["planes"])
    X = synth.make_x(in_, 7, seed=out)
    k_dev = torch.zeros(1, dtype=torch.int32, device="cuda")
    for k in range(1, 9):
        lut = synth.lut_np(lin["luts"][k])
        ref = oracle.gemv(planes, k, lut, synth.lut_np(X))
        for B in (2, 4, 7):
            y = torch.full((B + 1, out), 7.0, dtype=torch.float16, device="cuda")     # one row more than may be written
            k_dev.fill_(k)
            model.dpllm_gemv(0, -1 if B == 4 else k, X[:B].cuda(), y=y[:B], k_dev=k_dev)
            got = y.double().cpu().numpy()
            assert (got[B] == 7.0).all()
            for b in range(B):
                assert (np.abs(got[b] - ref[b]) <= bound(ref[b], lut, synth.lut_np(X[b]), in_)).all(), (k, B, b)
    model.close()
