"""Calls recorded into a graph, replayed between eager calls: neither sees
the other's maximum or scratch, whatever their order."""
import pytest
import torch

from paper_2503_10855_amd import synth

pytestmark = pytest.mark.gpu
THETA = 0.1
SIGMA = {5: 1.0, 9: 2.0}
BRIGHT, DARK = 3.0, 0.25    # a replay leaves a larger maximum than the eager calls'


@pytest.fixture(scope="module")
def hx():
    from paper_2503_10855_amd import hx as mod
    return mod


def images(h, w, seed):
    return [torch.from_numpy(synth.image(h, w, seed, i)).cuda() * s
            for i, s in enumerate((BRIGHT, DARK, DARK, 1.0))]


@pytest.mark.parametrize("ks,form", [(5, "auto"), (5, "recompute"), (5, "depth1"), (9, "auto"),
                                     (5, "stages"), (9, "stages")])
@pytest.mark.parametrize("where", ["own stream", "side stream"])
def test_eager_calls_between_replays_of_a_per_image_call(hx, ks, form, where):
    """Capture on the stream that makes the eager calls and on another one;
    after each replay of a bright image, eager calls on darker ones, an odd
    and an even number of them."""
    h, w = 300, 500
    srcs = images(h, w, 411)
    eager, side = torch.cuda.Stream(), torch.cuda.Stream()
    with hx.Pipeline(ksize=ks, sigma=SIGMA[ks], theta=THETA, max_pixels=h * w, max_images=1) as p:
        p.set_schedule(64, 16, 1)
        want = [p.edge_detect_stages(s) for s in srcs]
        p.sync()
        sched = {"recompute": (256, 64, 4, hx.PASS_RECOMPUTE), "depth1": (64, 16, 1)}.get(form)
        p.set_schedule(*sched) if sched else p.set_schedule()

        def call(src, stream):
            if form == "stages":
                with torch.cuda.stream(stream):
                    return p.edge_detect_stages(src, stream=stream)
            m = torch.zeros(1, device="cuda")
            torch.cuda.synchronize()
            return {"mask": p.edge_detect(src, dmax=m, stream=stream), "M": m}

        def check(got, i):
            torch.cuda.synchronize()
            for k, v in got.items():
                assert torch.equal(v, want[i][k]), (i, k)

        with torch.cuda.stream(eager):
            check(call(srcs[1], eager), 1)
        x = srcs[0].clone()
        out = {"mask": torch.zeros((h, w), dtype=torch.uint8, device="cuda"),
               "M": torch.zeros(1, device="cuda")}
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=eager if where == "own stream" else side):
            if form == "stages":
                out = p.edge_detect_stages(x)
            else:
                p.edge_detect(x, out["mask"], dmax=out["M"])
        for rep in range(4):
            for i in (0, 3):
                x.copy_(srcs[i])
                torch.cuda.synchronize()
                print(f"k{ks} {form} {where} replay {rep} image {i}", flush=True)
                with torch.cuda.stream(eager):
                    g.replay()
                check(out, i)
                for n in range(1 + rep):   # on the eager stream and another
                    check(call(srcs[1 + n % 2], (eager, side)[n // 2]), 1 + n % 2)


def test_recorded_calls_on_two_streams_of_one_capture(hx):
    """A capture that forks to a second stream and joins it: the recorded
    calls share one scratch set, so the graph must keep them in order."""
    h, w = 700, 900
    srcs = images(h, w, 412)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with hx.Pipeline(theta=THETA, max_pixels=h * w, max_images=1) as p:
        want_m = torch.zeros(4, device="cuda")
        want = [p.edge_detect(s, dmax=want_m[i:i + 1]) for i, s in enumerate(srcs)]
        p.sync()
        masks = [torch.zeros_like(m) for m in want]
        dm = torch.zeros(4, device="cuda")
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=a):
            b.wait_stream(a)
            for i, s in enumerate((a, b, a, b)):
                p.edge_detect(srcs[i], masks[i], dmax=dm[i:i + 1], stream=s)
            a.wait_stream(b)
        for rep in range(3):
            print(f"replay {rep}", flush=True)
            dm.fill_(-1.0)
            for m in masks:
                m.fill_(7)
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(dm, want_m)
            assert all(torch.equal(m, r) for m, r in zip(masks, want))


@pytest.mark.parametrize("contexts,graphs", [(1, 1), (2, 2), (4, 2)])
@pytest.mark.parametrize("form", ["auto", "recompute", "store", "large"])
def test_eager_batches_between_replays_of_a_batch(hx, contexts, graphs, form):
    """Batched calls recorded into graphs (more of them than contexts can be
    spared, too), replayed on new contents between eager calls on more
    batches than there are contexts, of other sizes and forms: a replay's
    table and scratch are its own."""
    shapes = [(1080, 1920)] * 4 if form == "large" else [(200, 300), (64, 64), (333, 251)]
    kind = {"recompute": hx.PASS_RECOMPUTE, "store": hx.PASS_STORE}.get(form)
    sets = [[torch.from_numpy(synth.image(h, w, 413 + s, i)).cuda() * sc
             for i, (h, w) in enumerate(shapes)] for s, sc in enumerate((BRIGHT, DARK, 1.0))]
    others = [[torch.from_numpy(synth.image(50 + 90 * b + i, 700 - 80 * b, 416, i)).cuda() * DARK
               for i in range(1 + 7 * (b % 3))] for b in range(6)]
    n_max = max(len(s) for s in sets + others)
    with hx.Pipeline(theta=THETA, max_pixels=1 << 24, max_images=n_max,
                     batch_contexts=contexts) as p:
        def batched(srcs, **kw):
            dm = torch.zeros(len(srcs), device="cuda")
            return p.edge_detect_batched(srcs, dmax=dm, **kw), dm

        p.set_schedule(64, 16, 1)
        want = []
        for srcs in sets + others:
            dm = torch.zeros(len(srcs), device="cuda")
            want.append(([p.edge_detect(s, dmax=dm[i:i + 1]) for i, s in enumerate(srcs)], dm))
        p.sync()

        def check(got, i):
            torch.cuda.synchronize()
            assert torch.equal(got[1], want[i][1]), i
            assert all(torch.equal(a, b) for a, b in zip(got[0], want[i][0])), i

        p.set_schedule(*((256, 32, 4, kind) if kind else ()))
        check(batched(sets[0]), 0)
        recs = []
        for _ in range(graphs):
            x = [torch.empty_like(s) for s in sets[0]]
            masks = [torch.zeros(s.shape, dtype=torch.uint8, device="cuda") for s in x]
            dm = torch.zeros(len(x), device="cuda")
            torch._foreach_copy_(x, sets[1])
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                p.edge_detect_batched(x, masks, dmax=dm)
            recs.append((g, x, masks, dm))
        p.set_schedule()
        side = torch.cuda.Stream()
        for rep in range(3):
            for j, (g, x, masks, dm) in enumerate(recs):
                for i in (0, 1, 2):
                    torch._foreach_copy_(x, sets[i])
                    dm.fill_(-1.0)
                    print(f"{form} {contexts} contexts graph {j} replay {rep} set {i}", flush=True)
                    g.replay()
                    check((masks, dm), i)
                    for b in range(6):
                        with torch.cuda.stream(side if b % 2 else torch.cuda.default_stream()):
                            got = batched(others[b], stream=torch.cuda.current_stream())
                        check(got, 3 + b)
                    check(batched(sets[(i + 1) % 3]), (i + 1) % 3)
        print("tuner beside a recorded call", flush=True)
        p.autotune_batch(sets[2])
        for g, x, masks, dm in recs:
            torch._foreach_copy_(x, sets[0])
            g.replay()
            check((masks, dm), 0)


def test_recorded_per_image_speculate(hx):
    """A fixed SPECULATE per-image call, recorded more often than there are
    contexts, with eager calls of the same form between the replays."""
    h, w = 500, 777
    srcs = images(h, w, 417)
    with hx.Pipeline(theta=THETA, max_pixels=h * w, max_images=1, batch_contexts=2,
                     pass_mode=hx.PASS_SPECULATE) as p:
        want_m = torch.zeros(4, device="cuda")
        want = [p.edge_detect(s, dmax=want_m[i:i + 1]) for i, s in enumerate(srcs)]
        p.sync()
        masks = [torch.zeros_like(m) for m in want]
        dm = torch.zeros(4, device="cuda")
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for i, s in enumerate(srcs):
                p.edge_detect(s, masks[i], dmax=dm[i:i + 1])
        em = torch.zeros(1, device="cuda")
        for rep in range(4):
            print(f"replay {rep}", flush=True)
            dm.fill_(-1.0)
            g.replay()
            e = p.edge_detect(srcs[rep], dmax=em)
            torch.cuda.synchronize()
            assert torch.equal(dm, want_m) and em[0] == want_m[rep] and torch.equal(e, want[rep])
            assert all(torch.equal(m, r) for m, r in zip(masks, want))
