"""GPU tests of the ways a dependency level of a decode step gets its bitwidths: selectors inside the GEMV launch, a part
launch and the decision in the prologue of every workgroup, or launches of their own for both; the choice rests on the
workgroups of the launch and the rows of G they would share (runs_selectors in dpllm_api.hip).  Against the CPU oracle."""
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


class Net:
    """Linears with random codes and tables (p = 4, 3 and 4 bits), scaled so that a chain keeps its size."""

    def __init__(self, dp, shapes, ranks, seed=0):
        rng = np.random.default_rng(seed)
        self.dp, self.shapes, n = dp, shapes, len(shapes)
        self.model, self.lin = dp.Model(n), []
        for i, (out, in_) in enumerate(shapes):
            planes = rng.integers(0, 2 ** 32, size=(4, out, in_ // 32), dtype=np.uint32)
            luts = {k: (rng.standard_normal((out, 1 << k)) / math.sqrt(in_)).astype(np.float16).view(np.uint16) for k in (3, 4)}
            self.model.dpllm_load_linear(i, planes, luts, 3)
            G = None if ranks[i] == 0 else (rng.standard_normal((ranks[i], in_)) * 0.1 / math.sqrt(in_)).astype(np.float16)
            self.lin.append({"planes": planes, "luts": luts, "G": G, "alpha": 0.0, "beta": 0.0})
            if G is None:
                self.lin[i].update(alpha=float(np.float32(0.01)), beta=0.25)
        self.k = torch.zeros(n, dtype=torch.int32, device="cuda")
        self.e = torch.zeros(n, dtype=torch.float32, device="cuda")
        self.ys = [torch.zeros(out, dtype=torch.float16, device="cuda") for out, _ in shapes]

    def estimate(self, i, x):
        L = self.lin[i]
        return oracle.linreg_estimate(x, L["alpha"], L["beta"]) if L["G"] is None else oracle.estimate(L["G"].view(np.uint16), x)

    def select(self, T):
        for i, L in enumerate(self.lin):
            kind = self.dp.DPLLM_SEL_LINREG if L["G"] is None else self.dp.DPLLM_SEL_PROJ
            G = None if L["G"] is None else torch.from_numpy(L["G"]).cuda()
            L["T"] = float(np.float32(T[i]))
            self.model.dpllm_set_selector(i, 3, 4, kind, G=G, alpha=L["alpha"], beta=L["beta"], T=L["T"])

    def check(self, xs, sels, tag):
        """Every estimate, bitwidth and result from the buffers as they are on the device after the step."""
        es, ks = self.e.cpu().numpy(), self.k.cpu().numpy()
        for i, (x, s) in enumerate(zip(xs, sels)):
            e_ref = self.estimate(i, s)
            assert abs(float(es[i]) - e_ref) <= 3e-7 * e_ref, (tag, i)
            k = oracle.decide(e_ref, self.lin[i]["T"], 3, 4)
            assert int(ks[i]) == k, (tag, i)
            ref = oracle.gemv(self.lin[i]["planes"], k, self.lin[i]["luts"][k], x)
            err = np.linalg.norm(self.ys[i].double().cpu().numpy() - ref)
            assert err <= 2e-3 * np.linalg.norm(ref), (tag, i)


# 96 and 192 blocks of 64 rows (32 and 64 rows per workgroup), 344, 688 and 1064 workgroups; rows of G on either side of six
# (256 workgroups), two (512) and one (more) per sharing workgroup
@pytest.mark.parametrize("out,in_,count,r,hybrid", [
    (2048, 256, 3, 64, True), (2048, 256, 3, 528, False), (4096, 256, 3, 64, True), (4096, 256, 3, 512, False), (4096, 256, 3, 528, True),
    (4096, 256, 3, 528, False), (11008, 256, 2, 64, True), (11008, 256, 2, 256, False), (11008, 256, 2, 528, True), (11008, 256, 4, 48, False),
    (11008, 256, 4, 96, True), (17000, 160, 4, 32, False)])
def test_level_matches_oracle(dp, out, in_, count, r, hybrid):
    """hybrid: the last linear is on the linear regression."""
    net = Net(dp, [(out, in_)] * count, [r] * (count - 1) + [0 if hybrid else r], seed=out + r)
    X = synth.make_x(in_, 2, seed=r)
    X[1] *= 2.0
    refs = [[net.estimate(i, synth.lut_np(x)) for x in X] for i in range(count)]
    # the first linear lies between the two vectors, the others on one side of both
    net.select([0.5 * sum(e) if i == 0 else (0.5 * min(e) if i == 1 else 1.5 * max(e)) for i, e in enumerate(refs)])
    x = torch.zeros(in_, dtype=torch.float16, device="cuda")
    xs = [x] * count
    xp, yp = net.model.pointers(xs), net.model.pointers(net.ys)

    def step(v, go):
        x.copy_(v)
        net.k.zero_(), net.e.zero_()
        go()
        torch.cuda.synchronize()

    eager = lambda: net.model.dpllm_decode_step(xp, yp, net.k, net.e)
    apart = lambda: [net.model.dpllm_decode_step_parts(xp, yp, net.k, net.e, p) for p in (dp.DPLLM_STEP_SELECT, dp.DPLLM_STEP_GEMV)]
    step(X[0], eager)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        eager()
    for turn in range(2):
        for v in X:
            bits = synth.lut_np(v)
            for name, go in (("eager", eager), ("apart", apart), ("graph", graph.replay)):
                for y in net.ys:
                    y.zero_()
                step(v, go)
                net.check([bits] * count, [bits] * count, (name, turn))
    net.model.close()


def test_selectors_of_later_levels_run_in_launches_of_every_kind(dp):
    """Selectors with an input of their own run with an earlier level: of 1040 workgroups (launches in front), and of a few
    (inside); their linears collect the products in a later launch.  One whose input that level writes stays where it is."""
    shapes = [(16640, 160)] * 4 + [(256, 16640), (512, 256), (256, 512), (128, 256)]
    net = Net(dp, shapes, [32, 32, 0, 16, 48, 64, 300, 17], seed=7)
    x = torch.zeros(160, dtype=torch.float16, device="cuda")
    wide, late = torch.zeros(16640, dtype=torch.float16, device="cuda"), torch.zeros(512, dtype=torch.float16, device="cuda")
    xs = [x] * 4 + [net.ys[0], net.ys[4], net.ys[5], net.ys[6]]
    sels = [x] * 4 + [wide, net.ys[4], late, net.ys[5]]
    net.select([math.inf] * 8)
    for i in (4, 6, 7):
        net.model.dpllm_set_selector_input(i, sels[i])
    xp, yp = net.model.pointers(xs), net.model.pointers(net.ys)
    go = lambda: net.model.dpllm_decode_step(xp, yp, net.k, net.e)
    inputs = [(synth.make_x(160, 1, seed=s)[0], synth.make_x(16640, 1, seed=s + 10)[0], synth.make_x(512, 1, seed=s + 20)[0]) for s in (1, 2)]

    def put(turn):
        for buf, v in zip((x, wide, late), inputs[turn % 2]):
            buf.copy_(v * (1 + turn % 2))

    put(0)
    go()
    first = net.e.tolist()
    net.select([e * (0.8 if i % 2 else 1.25) for i, e in enumerate(first)])
    go()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        go()
    for turn in range(6):
        put(turn)
        net.k.zero_(), net.e.zero_()
        (graph.replay if turn >= 3 else go)()
        torch.cuda.synchronize()
        host = lambda ts: [t.cpu().numpy().view(np.uint16) for t in ts]
        net.check(host(xs), [s[:shapes[i][1]] for i, s in enumerate(host(sels))], turn)
    net.model.close()
