"""GPU tests of the selectors that run inside the GEMV launch of a small dependency level: rows of G dealt out to the
launch's workgroups in slices of 4096 columns, partial products handed over through slots of the workspace, the decision
taken by every workgroup from the slots of its own linear."""
import math

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


def _lone_linear(dp, in_, r, seed, out=70):
    lin = synth.make_linear(out, in_, 4, 3, seed=seed)
    model = dp.Model(1)
    planes, luts = synth.planes_np(lin["planes"]), {k: synth.lut_np(v) for k, v in lin["luts"].items()}
    model.dpllm_load_linear(0, planes, luts, 3)
    G = (torch.randn(r, in_, generator=torch.Generator().manual_seed(seed)) / math.sqrt(r)).half()
    return model, planes, luts, G


# ranks around the 16 rows of a row group, the 256 workgroups the tasks are dealt out to and the 512 threads that collect
# them; rows below one chunk of 512 columns, of one slice (4096) exactly, and with a ragged last chunk or slice
@pytest.mark.parametrize("in_,r", [(32, 3), (1056, 17), (4096, 64), (4128, 16), (11008, 64), (16416, 40), (4096, 300), (8224, 1024)])
def test_step_selectors_match_oracle(dp, in_, r):
    model, planes, luts, G = _lone_linear(dp, in_, r, seed=in_ + r)
    xs = synth.make_x(in_, 4, seed=r)
    est = [oracle.estimate(synth.lut_np(G), synth.lut_np(x)) for x in xs]
    T = synth.nudge_threshold(float(np.median(est)), torch.tensor(est))
    model.dpllm_set_selector(0, 3, 4, dp.DPLLM_SEL_PROJ, G=G.cuda(), T=T)
    x_dev = torch.zeros(in_, dtype=torch.float16, device="cuda")
    y = torch.zeros(planes.shape[1], dtype=torch.float16, device="cuda")
    k_dev, e_dev = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.float32, device="cuda")
    for x, e_ref in zip(xs, est):       # another vector every time: a slot left over from the step before would show
        x_dev.copy_(x)
        model.dpllm_decode_step([x_dev], [y], k_dev, e_dev)
        assert math.isclose(float(e_dev), e_ref, rel_tol=3e-7)
        k = oracle.decide(e_ref, T, 3, 4)
        assert int(k_dev) == k
        ref = oracle.gemv(planes, k, luts[k], synth.lut_np(x))
        assert np.linalg.norm(y.float().cpu().numpy() - ref) <= 2e-3 * np.linalg.norm(ref)
    model.close()


@pytest.mark.parametrize("in_,r", [(1056, 17), (8224, 64), (4096, 600)])
def test_step_takes_products_nobody_delivers_itself(dp, in_, r):
    """A graph captured while no linear has an estimator, replayed after the pair in use has changed to one with a
    projection: same bits as an eager step under that pair."""
    model, planes, luts, G = _lone_linear(dp, in_, r, seed=in_ * 3 + r)
    x = synth.make_x(in_, 1, seed=r)[0].cuda()
    e_ref = oracle.estimate(synth.lut_np(G), synth.lut_np(x))
    model.dpllm_set_selector(0, 3, 4, dp.DPLLM_SEL_PROJ, G=G.cuda(), T=float(np.float32(1.1 * e_ref)))
    model.dpllm_set_selector(0, 4, 4, dp.DPLLM_SEL_NONE)
    y = torch.zeros(planes.shape[1], dtype=torch.float16, device="cuda")
    k_dev, e_dev = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.float32, device="cuda")
    xp, yp = model.pointers([x]), model.pointers([y])
    model.dpllm_decode_step(xp, yp, k_dev, e_dev)
    torch.cuda.synchronize()
    assert int(k_dev) == 4
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        model.dpllm_decode_step(xp, yp, k_dev, e_dev)
    model.dpllm_set_active_pair(0, 3, 4)
    model.dpllm_decode_step(xp, yp, k_dev, e_dev)
    torch.cuda.synchronize()
    want = (k_dev.clone(), e_dev.clone(), y.clone())
    assert int(k_dev) == 3 and math.isclose(float(e_dev), e_ref, rel_tol=3e-7)
    for _ in range(3):
        y.zero_(), k_dev.zero_(), e_dev.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(k_dev, want[0]) and torch.equal(e_dev, want[1]) and torch.equal(y, want[2])
    model.close()


def test_selector_on_the_buffer_its_own_linear_writes(dp):
    """A selector input that is the linear's own output buffer: the estimate comes from what the buffer held before the
    GEMV wrote it, so the selectors of such a level are done before its GEMV launch starts."""
    model, planes, luts, G = _lone_linear(dp, 256, 32, seed=91, out=256)
    x = synth.make_x(256, 1, seed=92)[0].cuda()
    before = synth.make_x(256, 1, seed=93)[0].cuda()
    e_ref = oracle.estimate(synth.lut_np(G), synth.lut_np(before))
    model.dpllm_set_selector(0, 3, 4, dp.DPLLM_SEL_PROJ, G=G.cuda(), T=float(np.float32(0.9 * e_ref)))
    y = torch.zeros(256, dtype=torch.float16, device="cuda")
    model.dpllm_set_selector_input(0, y)
    k_dev, e_dev = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.float32, device="cuda")
    for _ in range(3):
        y.copy_(before)
        model.dpllm_decode_step([x], [y], k_dev, e_dev)
        assert math.isclose(float(e_dev), e_ref, rel_tol=3e-7) and int(k_dev) == 4
        ref = oracle.gemv(planes, 4, luts[4], synth.lut_np(x))
        assert np.linalg.norm(y.float().cpu().numpy() - ref) <= 2e-3 * np.linalg.norm(ref)
    model.close()


@pytest.mark.parametrize("own_launch", [True, False])
def test_step_captured_without_estimators_follows_a_later_pair(dp, own_launch):
    """A graph captured while no linear has an estimator, replayed after the pair in use has changed to one with a
    projection: estimates of the vector the replay finds, not of the one an eager step in between left products of.
    own_launch: the selectors run in front of the GEMV launch (the selector reads what its linear writes)."""
    model, planes, luts, G = _lone_linear(dp, 256, 32, seed=41, out=256)
    x = synth.make_x(256, 1, seed=42)[0].cuda()
    vectors = synth.make_x(256, 3, seed=43)
    vectors[1] *= 3.0
    est = [oracle.estimate(synth.lut_np(G), synth.lut_np(v)) for v in vectors]
    T = synth.nudge_threshold(float(np.median(est)), torch.tensor(est))
    model.dpllm_set_selector(0, 3, 4, dp.DPLLM_SEL_PROJ, G=G.cuda(), T=T)
    model.dpllm_set_selector(0, 4, 4, dp.DPLLM_SEL_NONE)
    y, sel = torch.zeros(256, dtype=torch.float16, device="cuda"), torch.zeros(256, dtype=torch.float16, device="cuda")
    read = y if own_launch else sel
    model.dpllm_set_selector_input(0, read)
    k_dev, e_dev = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.float32, device="cuda")
    xp, yp = model.pointers([x]), model.pointers([y])
    model.dpllm_decode_step(xp, yp, k_dev, e_dev)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        model.dpllm_decode_step(xp, yp, k_dev, e_dev)
    model.dpllm_set_active_pair(0, 3, 4)
    for v, e_ref in zip(vectors, est):
        read.copy_(vectors[0])
        model.dpllm_decode_step(xp, yp, k_dev, e_dev)
        read.copy_(v)
        graph.replay()
        torch.cuda.synchronize()
        assert math.isclose(float(e_dev), e_ref, rel_tol=3e-7)
        k = oracle.decide(e_ref, T, 3, 4)
        assert int(k_dev) == k
        ref = oracle.gemv(planes, k, luts[k], synth.lut_np(x))
        assert np.linalg.norm(y.float().cpu().numpy() - ref) <= 2e-3 * np.linalg.norm(ref)
    model.close()


@pytest.mark.parametrize("in_,r", [(4096, 64), (1056, 48)])
def test_step_with_a_workspace_from_before_its_selectors(dp, in_, r):
    """A workspace of the size the model asked for when no pair was attached: too small for the tasks of r rows, large
    enough for the parts of one selector.  The step runs its selectors in launches of their own."""
    model, planes, luts, G = _lone_linear(dp, in_, r, seed=in_ + 7 * r)
    model.dpllm_set_workspace()
    x = synth.make_x(in_, 1, seed=r)[0]
    e_ref = oracle.estimate(synth.lut_np(G), synth.lut_np(x))
    model.dpllm_set_selector(0, 3, 4, dp.DPLLM_SEL_PROJ, G=G.cuda(), T=float(np.float32(0.9 * e_ref)))
    assert model.workspace.numel() < model.dpllm_workspace_bytes()
    model._ws_stale = False              # as a caller of the C functions that keeps the workspace it has
    y = torch.zeros(planes.shape[1], dtype=torch.float16, device="cuda")
    k_dev, e_dev = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.float32, device="cuda")
    for _ in range(2):
        k_dev.zero_(), e_dev.zero_(), y.zero_()
        model.dpllm_decode_step([x.cuda()], [y], k_dev, e_dev)
        assert int(k_dev) == 4 and math.isclose(float(e_dev), e_ref, rel_tol=3e-7)
        ref = oracle.gemv(planes, 4, luts[4], synth.lut_np(x))
        assert np.linalg.norm(y.float().cpu().numpy() - ref) <= 2e-3 * np.linalg.norm(ref)
    model.close()


@pytest.mark.parametrize("in_,r", [(1056, 17), (8224, 64), (4096, 600), (32, 3)])
def test_step_computes_the_products_nobody_delivers(dp, in_, r):
    """Workgroups that stop looking for the products of their linear's selector compute them: with no look but the first one,
    and with the selector work left out of the launch, where every slot is empty.  Same bits as with the work shared."""
    model, planes, luts, G = _lone_linear(dp, in_, r, seed=in_ * 5 + r)
    X = synth.make_x(in_, 2, seed=r)
    X[1] *= 2.0
    est = [oracle.estimate(synth.lut_np(G), synth.lut_np(x)) for x in X]
    model.dpllm_set_selector(0, 3, 4, dp.DPLLM_SEL_PROJ, G=G.cuda(), T=float(np.float32(0.5 * sum(est))))
    x, y = torch.zeros(in_, dtype=torch.float16, device="cuda"), torch.zeros(planes.shape[1], dtype=torch.float16, device="cuda")
    k_dev, e_dev = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.float32, device="cuda")
    want = {}
    for polls in (64, 0, -1, 64):
        model.dpllm_debug_set_polls(polls)
        for rep in range(4):
            which = rep % 2
            x.copy_(X[which])
            y.zero_(), k_dev.zero_(), e_dev.zero_()
            model.dpllm_decode_step([x], [y], k_dev, e_dev)
            assert math.isclose(float(e_dev), est[which], rel_tol=3e-7) and int(k_dev) == 3 + which, (polls, rep)
            got = (e_dev.clone(), y.clone())
            want.setdefault(which, got)
            assert all(torch.equal(a, b) for a, b in zip(got, want[which])), (polls, rep)
    with pytest.raises(dp.DpllmError):
        model.dpllm_debug_set_polls(-2)
    model.close()
