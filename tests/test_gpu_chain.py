"""GPU tests of steps of many levels that run as one launch (gemv_chain_kernel): results and products of selectors handed over
inside the launch, rows dealt out in blocks of 64, 32 or 16, vectors longer than the eight wavefronts park at a time.  Against
the CPU oracle, linear by linear, from the buffers as they are on the device after the step.  Shapes this small take a launch per
level by themselves: the tests ask for the one launch (dpllm_debug_set_one_launch) and see that they get it."""
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


class Chain:
    """Levels of linears; every level reads, from `skip` elements on, the result of the first linear of the level before.
    levels: [[out, ...], ...]; the columns of a level are what the one before offers, down to a multiple of 32."""

    def __init__(self, dp, levels, first_in, p, pairs, seed, ranks=(17, 0, 64, 1, 130, -1), late=True):
        rng = np.random.default_rng(seed)
        self.dp, self.x0 = dp, torch.zeros(first_in, dtype=torch.float16, device="cuda")
        self.late = torch.zeros(max(max(l) for l in levels) + first_in, dtype=torch.float16, device="cuda")
        self.src, self.ys, self.sel, self.lin, sizes = [], [], [], [], []
        feed, n_in = self.x0, first_in
        for li, outs in enumerate(levels):
            for o in outs:
                sizes.append((o, n_in))
                self.src.append(feed[:n_in])
                self.ys.append(torch.zeros(o, dtype=torch.float16, device="cuda"))
            skip = 8 * (li % 3) if outs[0] >= 64 else 0
            feed, n_in = self.ys[-len(outs)][skip:], (outs[0] - skip) // 32 * 32
            if n_in == 0:
                feed, n_in = self.x0, first_in
        self.model, n = dp.Model(len(sizes)), len(sizes)
        for i, (o, k_in) in enumerate(sizes):
            planes = rng.integers(0, 2 ** 32, size=(p, o, k_in // 32), dtype=np.uint32)
            kmin = min(l for l, _ in pairs)
            luts = {k: (rng.standard_normal((o, 1 << k)) / math.sqrt(k_in)).astype(np.float16).view(np.uint16) for k in range(kmin, p + 1)}
            self.model.dpllm_load_linear(i, planes, luts, kmin)
            r = ranks[i % len(ranks)]
            G = (rng.standard_normal((r, k_in)) * 0.1 / math.sqrt(k_in)).astype(np.float16) if r > 0 else None
            self.lin.append({"planes": planes, "luts": luts, "G": G, "r": r, "pair": pairs[i % len(pairs)]})
            own = late and i % 5 == 2
            self.sel.append(self.late[:k_in] if own else self.src[i])
        self.k, self.e = torch.zeros(n, dtype=torch.int32, device="cuda"), torch.zeros(n, dtype=torch.float32, device="cuda")
        self.xp, self.yp = self.model.pointers(self.src), self.model.pointers(self.ys)
        for i in range(n):
            if self.sel[i] is not self.src[i]:
                self.model.dpllm_set_selector_input(i, self.sel[i])
        self.model.dpllm_debug_set_one_launch(1)

    def select(self, T):
        for i, L in enumerate(self.lin):
            l, h = L["pair"]
            L["T"] = float(np.float32(T[i]))
            if L["r"] < 0:
                self.model.dpllm_set_selector(i, l, l, self.dp.DPLLM_SEL_NONE)
            elif L["r"] == 0:
                self.model.dpllm_set_selector(i, l, h, self.dp.DPLLM_SEL_LINREG, alpha=0.125, beta=0.25, T=L["T"])
            else:
                self.model.dpllm_set_selector(i, l, h, self.dp.DPLLM_SEL_PROJ, G=torch.from_numpy(L["G"]).cuda(), T=L["T"])

    def put(self, seed):
        self.x0.copy_(synth.make_x(self.x0.numel(), 1, seed=seed)[0] * (1 + seed % 3))
        self.late.copy_(synth.make_x(self.late.numel() // 32 * 32 + 32, 1, seed=seed + 50)[0][:self.late.numel()])

    def step(self, one=True):
        self.model.dpllm_decode_step(self.xp, self.yp, self.k, self.e)
        assert (self.model.dpllm_debug_step_launches() == 2) == one

    def level_by_level(self):
        """The same step with a launch per level (it writes the tables anew: replays come behind the next step in one launch)."""
        self.model.dpllm_debug_set_one_launch(-1)
        self.step(one=False)
        self.model.dpllm_debug_set_one_launch(1)

    def state(self):
        torch.cuda.synchronize()
        return [t.clone() for t in [self.k, self.e] + self.ys]

    def clear(self):
        for t in [self.k, self.e] + self.ys:
            t.zero_()

    def calibrate(self, seeds, one=True):
        """Thresholds between, below and above the estimates of two inputs in turn."""
        self.select([math.inf] * len(self.lin))
        est = []
        for s in seeds:
            self.put(s)
            self.step(one)
            est.append(self.e.tolist())
        self.select([0.5 * (a + b) if i % 3 == 0 else (0.4 if i % 3 == 1 else 2.5) * max(a, b) for i, (a, b) in enumerate(zip(*est))])

    def check(self, tag):
        bits = lambda t: t.cpu().numpy().view(np.uint16)
        es, ks = self.e.cpu().numpy(), self.k.cpu().numpy()
        for i, L in enumerate(self.lin):
            l, h = L["pair"]
            s = bits(self.sel[i])
            if L["r"] < 0:
                e_ref, k = 0.0, l
            else:
                e_ref = oracle.linreg_estimate(s, 0.125, 0.25) if L["r"] == 0 else oracle.estimate(L["G"].view(np.uint16), s)
                k = oracle.decide(e_ref, L["T"], l, h)
            assert abs(float(es[i]) - e_ref) <= 3e-7 * abs(e_ref), (tag, i)
            assert int(ks[i]) == k, (tag, i)
            ref = oracle.gemv(L["planes"], k, L["luts"][k], bits(self.src[i]))
            assert np.linalg.norm(self.ys[i].double().cpu().numpy() - ref) <= 2e-3 * np.linalg.norm(ref), (tag, i)


# small and ragged linears (rows around 16, 32 and 64, columns below one tile, with a ragged last tile and chunk)
SMALL = [[64], [65, 1, 63], [33], [544, 17], [1000], [15, 130], [96, 4, 4, 4, 4, 4, 4], [200]] * 3 + [[512], [77]]
# levels that are dealt out in blocks of 64 and 32 rows, vectors of more than 4096 elements, with and without a ragged last chunk
LARGE = [[4128, 8200], [352, 64], [8224], [96], [4096, 4096, 4100], [160], [11008, 11008], [128], [28672], [64], [64]] + [[64]] * 15


@pytest.mark.parametrize("name,p,pairs", [("small", 4, [(3, 4), (2, 3), (4, 4)]), ("small", 6, [(4, 5), (5, 6), (3, 6)]),
                                          ("small", 8, [(7, 8), (1, 8), (6, 7), (3, 5)]), ("large", 4, [(3, 4)]), ("large", 6, [(5, 6), (4, 5)])])
def test_chain_matches_oracle(dp, name, p, pairs):
    net = Chain(dp, SMALL if name == "small" else LARGE, 96 if name == "small" else 64, p, pairs, seed=p)
    net.calibrate((1, 2))
    clean = {}
    for seed in (1, 2):
        net.put(seed)
        net.clear()
        net.step()
        clean[seed] = net.state()
        net.check((name, seed))
    assert not torch.equal(clean[1][0], clean[2][0])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        net.step()
    for rep in range(12):
        seed = 1 + rep % 2
        net.put(seed)
        net.clear()
        (net.step, graph.replay, net.level_by_level)[rep % 3]()
        got = net.state()
        if rep % 3 < 2:
            assert all(torch.equal(a, b) for a, b in zip(got, clean[seed])), rep
        else:
            net.check((name, "level by level", rep))
    net.model.close()


def test_target_switches_between_replays(dp):
    """The bitwidths, the planes asked for ahead and the selectors' rows of G follow a switch of target in a captured step."""
    net = Chain(dp, SMALL, 96, 8, [(3, 4)], seed=11, ranks=(17, 64), late=False)
    net.calibrate((3, 4))
    for i, L in enumerate(net.lin):
        net.model.dpllm_set_target_entry(1, i, 3, 4, math.inf)
    wide = [dict(L) for L in net.lin]
    for i, L in enumerate(wide):
        G = torch.from_numpy((L["G"] * np.float16(0.5)).astype(np.float16)).cuda()
        net.model.dpllm_set_selector(i, 6, 8, dp.DPLLM_SEL_PROJ, G=G[:9].contiguous(), T=-math.inf)
        net.model.dpllm_set_active_pair(i, 3, 4)
        net.model.dpllm_set_target_entry(2, i, 6, 8, -math.inf)
    net.put(3)
    net.step()
    base = net.state()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        net.step()
    for target in (1, 2, 0, 2, 1, 0):
        net.model.dpllm_set_target(target)
        net.clear()
        graph.replay()
        got = net.state()
        if target == 0:
            assert all(torch.equal(a, b) for a, b in zip(got, base))
            net.check("target 0")
        else:
            assert got[0].tolist() == [3 if target == 1 else 8] * len(net.lin)
            for i in (0, 5, len(net.lin) - 1):
                k = int(got[0][i])
                ref = oracle.gemv(net.lin[i]["planes"], k, net.lin[i]["luts"][k], net.src[i].cpu().numpy().view(np.uint16))
                assert np.linalg.norm(net.ys[i].double().cpu().numpy() - ref) <= 2e-3 * np.linalg.norm(ref), (target, i)
    net.model.close()


@pytest.mark.parametrize("pairs,unused", [([(3, 4)], (5, 6)), ([(3, 4)], (7, 8)), ([(5, 6)], (7, 8)), ([(3, 4), (4, 5)], (7, 8))])
def test_pairs_that_are_not_active_change_nothing(dp, pairs, unused):
    """How many planes are asked for ahead follows the active pairs; a wider one beside them leaves every bit as it is."""
    net = Chain(dp, SMALL, 96, 8, pairs, seed=31)
    net.calibrate((1, 2))
    net.put(1)
    net.step()
    alone = net.state()
    net.model.dpllm_set_selector(len(net.lin) - 1, *unused, dp.DPLLM_SEL_LINREG, alpha=0.5, beta=0.5, T=0.0)
    net.model.dpllm_set_active_pair(len(net.lin) - 1, *net.lin[-1]["pair"])
    net.clear()
    net.step()
    assert all(torch.equal(a, b) for a, b in zip(net.state(), alone))
    net.check(unused)
    net.model.close()


def test_two_chains_beside_one_another(dp):
    """Two models on two streams: each launch works with the workgroups that found a place."""
    nets = [Chain(dp, SMALL, 96, 4, [(3, 4)], seed=s) for s in (21, 22)]
    clean = []
    for net in nets:
        net.calibrate((5, 6))
        net.put(5)
        net.step()
        clean.append(net.state())
    streams = [torch.cuda.Stream() for _ in nets]
    for rep in range(6):
        for net in nets:
            net.clear()
        torch.cuda.synchronize()
        for _ in range(8):
            for net, s in zip(nets, streams):
                with torch.cuda.stream(s):
                    net.step()
        for net, want in zip(nets, clean):
            assert all(torch.equal(a, b) for a, b in zip(net.state(), want)), rep
    for net in nets:
        net.model.close()


@pytest.mark.parametrize("name,p,pairs", [("small", 4, [(3, 4)]), ("large", 6, [(5, 6), (4, 5)])])
def test_workgroups_that_join_later(dp, name, p, pairs):
    """However many workgroups share the first levels, the results are the same bits, eager and replayed."""
    net = Chain(dp, SMALL if name == "small" else LARGE, 96 if name == "small" else 64, p, pairs, seed=71)
    net.calibrate((1, 2))
    net.put(1)
    net.step()
    clean = net.state()
    net.check(name)
    for seats in (1, 2, 7, 100, 255, 256, 1000, 0):
        net.model.dpllm_debug_set_one_launch(1, seats)
        for rep in range(3):
            net.clear()
            net.step()
            assert all(torch.equal(a, b) for a, b in zip(net.state(), clean)), (seats, rep)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            net.step()
        for rep in range(3):
            net.clear()
            graph.replay()
            assert all(torch.equal(a, b) for a, b in zip(net.state(), clean)), (seats, rep, "replay")
    net.model.close()


def test_a_chain_beside_other_work(dp):
    """Copies and matrix products on a second stream hold compute units while the step starts and while it runs."""
    net = Chain(dp, LARGE, 64, 6, [(5, 6), (4, 5)], seed=81)
    net.calibrate((1, 2))
    net.put(1)
    net.step()
    clean = net.state()
    a, b = torch.randn(4096, 4096, device="cuda").half(), torch.empty(1 << 27, dtype=torch.float16, device="cuda")
    work = [lambda: torch.mm(a, a), lambda: b[:1 << 26].copy_(b[1 << 26:])]
    side = torch.cuda.Stream()
    for rep in range(8):
        net.clear()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for i in range(30):
                work[(i // 3 if rep % 3 == 2 else rep) % 2]()
        for _ in range(6):
            net.step()
        assert all(torch.equal(u, v) for u, v in zip(net.state(), clean)), rep
    net.model.close()


@pytest.mark.parametrize("case", ["overlap", "shared", "offset"])
def test_steps_it_does_not_serve_run_level_by_level(dp, case):
    """A vector that spans two results, one result buffer for several linears, a vector that starts off the mailbox's words: the
    results of linears one after the other."""
    net = Chain(dp, [[96]] * 6 + [[112]] + [[96]] * 19, 96, 4, [(3, 4)], seed=31, ranks=(17, 64), late=False)
    both = torch.zeros(400, dtype=torch.float16, device="cuda")
    if case == "overlap":
        net.ys[3], net.ys[4] = both[:96], both[96:192]
        net.src[5] = net.sel[5] = both[48:144]
        net.src[4] = net.sel[4] = net.ys[3]
    elif case == "shared":
        net.ys[10] = net.ys[7]
        net.src[11] = net.sel[11] = net.ys[7]
    else:
        net.ys[6] = both[1:113]
        net.src[7] = net.sel[7] = both[8:104]
    net.xp, net.yp = net.model.pointers(net.src), net.model.pointers(net.ys)
    net.calibrate((7, 8), one=False)
    net.put(7)
    net.clear()
    net.step(one=False)
    ks, es, ys = net.k.tolist(), net.e.tolist(), [y.clone() for y in net.ys]
    net.clear()
    for i in range(len(net.lin)):
        e, k = net.model.dpllm_estimate(i, 3, 4, net.sel[i])
        net.model.dpllm_gemv(i, -1, net.src[i].contiguous(), y=net.ys[i], k_dev=k)
        assert int(k) == ks[i] and math.isclose(float(e), es[i], rel_tol=3e-4), i
    for i, (a, b) in enumerate(zip(net.ys, ys)):
        if not (case == "shared" and i == 7):
            assert (a.double() - b.double()).norm() <= 2e-2 * b.double().norm(), i
    net.model.close()


def test_more_linears_in_a_level_than_its_record_holds(dp):
    """57 linears on one vector: a launch per level."""
    net = Chain(dp, [[64] * 56, [64] * 57], 64, 4, [(3, 4)], seed=41, late=False)
    net.calibrate((1, 2), one=False)
    net.put(1)
    net.step(one=False)
    net.check("57")
    net.model.close()


@pytest.mark.parametrize("values", [(math.inf,), (-math.inf, 1.0), (math.nan,), (math.inf, math.nan)])
def test_infinities_and_nan_travel_through_mailboxes(dp, values):
    """A result that is not finite, all bits set among them, is handed over like any other: the launch ends, and every result is
    what a launch per level leaves (an infinity, NaN, or a number to the rounding of the sums)."""
    net = Chain(dp, SMALL, 96, 4, [(3, 4)], seed=51, late=False)
    net.calibrate((1, 2))
    net.put(1)
    bits = net.x0.view(torch.int16)
    for i, v in enumerate(values):
        net.x0[7 * i + 3] = v
        if math.isnan(v):
            bits[7 * i + 3] = -1                     # 0xffff
    net.clear()
    net.step()
    got = net.state()
    net.clear()
    net.level_by_level()
    want = net.state()
    assert torch.equal(got[0], want[0]) and int(got[0][0]) > 0
    for a, b in zip(got[2:], want[2:]):
        assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.isinf(a), torch.isinf(b))
        keep = torch.isfinite(b)
        assert (a[keep].double() - b[keep].double()).norm() <= 2e-2 * b[keep].double().norm()
    assert not bool(torch.isfinite(torch.cat(got[2:])).all())
    net.model.close()


def _big(dp, shapes, p, pairs, seed, rank=16):
    """One linear per shape, each fed by the one before, with random planes made on the device."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    model, lin = dp.Model(len(shapes)), []
    for i, (out, in_) in enumerate(shapes):
        planes = torch.randint(-2 ** 31, 2 ** 31, (p, out, in_ // 32), dtype=torch.int32, device="cuda", generator=g)
        luts = {k: (torch.randn(out, 1 << k, device="cuda", generator=g) / math.sqrt(in_)).half() for k in range(3, p + 1)}
        model.dpllm_load_linear(i, planes, luts, 3)
        Gs = [(torch.randn(rank, in_, device="cuda", generator=g) * 0.1 / math.sqrt(in_)).half() for _ in pairs]
        for (l, h), G in zip(pairs, Gs):
            model.dpllm_set_selector(i, l, h, dp.DPLLM_SEL_PROJ, G=G, T=0.0)
        keep = i in (0, len(shapes) - 1)             # what the oracle is asked about
        lin.append({"planes": planes if keep else None, "luts": luts if keep else None, "G": Gs if keep else None})
    return model, lin


# 24 levels either side of the line between the two kinds of step; at 3 or 4 bits a level is 24 .. 42 MB, at 7 or 8 55 .. 84.
# Linears that do not depend on one another, with 1024 workgroups where the work is cut for 3 or 4 bits and 2048 where for 7 or 8
@pytest.mark.parametrize("shapes,chained,one", [([(15360, 4096), (4096, 15360)] * 12, True, True), ([(15360, 5120), (5120, 15360)] * 12, True, False),
                                                ([(16384, 16384)] * 8, False, False)])
def test_a_captured_step_follows_the_pair_in_use(dp, shapes, chained, one):
    """How a captured step is launched does not depend on the pairs in use: a graph captured under one pair runs another after
    dpllm_set_active_pair and an eager step between, in both directions."""
    pairs = [(3, 4), (7, 8)]
    model, lin = _big(dp, shapes, 8, pairs, seed=61)
    n = len(shapes)
    x0 = synth.make_x(shapes[0][1], 1, seed=62)[0].cuda()
    ys = [torch.zeros(out, dtype=torch.float16, device="cuda") for out, _ in shapes]
    xs = [x0] + ys[:-1] if chained else [x0] * n
    k, e = torch.zeros(n, dtype=torch.int32, device="cuda"), torch.zeros(n, dtype=torch.float32, device="cuda")

    def use(pair, T):
        for i in range(n):
            model.dpllm_set_active_pair(i, *pair)
            model.dpllm_set_threshold(i, *pair, T[i])

    def step():
        model.dpllm_decode_step(xs, ys, k, e)
        assert (model.dpllm_debug_step_launches() == 2) == one

    want, T = {}, {}
    for pair in pairs:
        T[pair] = [math.inf if i % 2 else -math.inf for i in range(n)]
        use(pair, T[pair])
        step()
        torch.cuda.synchronize()
        want[pair] = [t.clone() for t in [k, e] + ys]
        assert k.tolist() == [pair[0] if i % 2 else pair[1] for i in range(n)]
        for i in (0, n - 1):
            x = xs[i].cpu().numpy().view(np.uint16)
            got_k = int(k[i])
            ref = oracle.gemv(lin[i]["planes"].cpu().numpy().view(np.uint32), got_k, lin[i]["luts"][got_k].cpu().numpy().view(np.uint16), x)
            assert np.linalg.norm(ys[i].double().cpu().numpy() - ref) <= 2e-3 * np.linalg.norm(ref), (pair, i)
            ref = oracle.estimate(lin[i]["G"][pairs.index(pair)].cpu().numpy().view(np.uint16), x)
            assert math.isclose(float(e[i]), ref, rel_tol=3e-7)
    for captured, other in (pairs, pairs[::-1]):
        use(captured, T[captured])
        step()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step()
        for pair in (other, captured, other):
            use(pair, T[pair])
            for t in ys:
                t.zero_()
            step()
            for rep in range(2):
                for t in [k, e] + ys:
                    t.zero_()
                graph.replay()
                torch.cuda.synchronize()
                assert all(torch.equal(a, b) for a, b in zip([k, e] + ys, want[pair])), (captured, pair, rep)
    model.close()


# either side of the lines of the rule: levels, columns that eight wavefronts share evenly or not, rows of G per level, weights
@pytest.mark.parametrize("shapes,rank,one", [([(4096, 4096)] * 24, 64, True), ([(4096, 4096)] * 23, 64, False), ([(4096, 4096)] * 24, 256, True),
                                             ([(4096, 4096)] * 24, 272, False), ([(3584, 3584)] * 24, 16, True), ([(3072, 3072)] * 24, 16, False),
                                             ([(5120, 5120)] * 24, 16, False), ([(8192, 7680)] + [(8192, 8192)] * 23, 16, False)])
def test_which_steps_are_one_launch(dp, shapes, rank, one):
    model, _ = _big(dp, shapes, 3, [(3, 3)], seed=91, rank=rank)
    ys = [torch.zeros(out, dtype=torch.float16, device="cuda") for out, _ in shapes]
    xs = [synth.make_x(shapes[0][1], 1, seed=92)[0].cuda()] + ys[:-1]
    k, e = torch.zeros(len(shapes), dtype=torch.int32, device="cuda"), torch.zeros(len(shapes), dtype=torch.float32, device="cuda")
    model.dpllm_decode_step(xs, ys, k, e)
    torch.cuda.synchronize()
    assert (model.dpllm_debug_step_launches() == 2) == one and k.tolist() == [3] * len(shapes)
    first = [t.clone() for t in ys]
    for i in range(len(shapes)):                     # linear by linear
        model.dpllm_gemv(i, 3, xs[i], y=ys[i])
    for i, (a, b) in enumerate(zip(ys, first)):
        assert (a.double() - b.double()).norm() <= 2e-2 * a.double().norm() > 0, i
    model.close()
