"""The surrogate's hand-written kernels against its FP64 oracle on the same
BF16-rounded parameters and inputs: forward probabilities, the full gradient
of the loss, a decreasing training loss, and the spread estimator's fallback
to the plain simulator."""
import numpy as np
import pytest

from oracle import gnn as OG
from paper_2603_14895_amd import workloads as W
from tests.gpu_util import log

pytestmark = pytest.mark.gpu


def _hub_graph():
    """Chung-Lu background plus hub nodes with 300-1500 in- and out-arcs, so
    the block-per-row aggregation paths (rows above 256 arcs) run too."""
    rng = np.random.default_rng(99)
    base = W.chung_lu(1500, 6.0, 2.5, 4343)
    ptr, src = base.numpy()
    dst = np.repeat(np.arange(base.n), np.diff(ptr))
    edges = set(zip(src.tolist(), dst.tolist()))
    for hub, k in ((3, 300), (77, 700), (1234, 1499)):
        for u in rng.choice(base.n, size=k, replace=False).tolist():
            if u != hub:
                edges.add((u, hub))
                edges.add((hub, u))
    return W.from_edges(base.n, sorted(edges), "hubs")


@pytest.fixture(scope="module", params=["small", "hubs"])
def setup(request):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_14895_amd import fsg
    gr = W.chung_lu(400, 8.0, 2.5, 4242) if request.param == "small" else _hub_graph()
    rev = W.reverse_graph(gr)
    g = fsg.DeviceGraph(*gr.numpy())
    gr_ = fsg.DeviceGraph(*rev.numpy())
    rng = np.random.default_rng(7)
    n = gr.n
    masks = (rng.random((3, n)) < 0.05).astype(np.uint8)
    betas = [0.012, 0.03, 0.047]
    ys = rng.random((3, n)).astype(np.float32)
    params = OG.glorot(11).astype(np.float32)
    return dict(fsg=fsg, gr=gr, g=g, rev=gr_, masks=masks, betas=betas, ys=ys, params=params)


def test_forward_matches_oracle(setup):
    import torch
    S = setup
    net = S["fsg"].GNN(1)
    net.set_params(S["params"])
    prob = net.forward(S["g"], torch.tensor(S["masks"], device="cuda"), S["betas"]).cpu().numpy()
    ptr, src = S["gr"].numpy()
    for s in range(3):
        ref, _ = OG.forward(S["params"].astype(np.float64), ptr, src, S["masks"][s].astype(float),
                            S["betas"][s], bf=True)
        err = np.abs(prob[s] - ref)
        log(f"[gnn] forward set {s}: max abs err {err.max():.2e}, mean {err.mean():.2e}")
        # every BF16 activation is its definition rounded once, so only the
        # FP32 head (and a rare MFMA-sum rounding at a BF16 tie) separates them
        assert err.max() < 1e-3 and err.mean() < 1e-5


def test_gradient_matches_oracle(setup):
    import torch
    S = setup
    net = S["fsg"].GNN(2)
    net.set_params(S["params"])
    loss = net.train_step(S["g"], S["rev"], torch.tensor(S["masks"], device="cuda"), S["betas"],
                          torch.tensor(S["ys"], device="cuda"), 0.0, update=False)
    gg = net.get_grads().astype(np.float64)
    ptr, src = S["gr"].numpy()
    rl, rg = OG.loss_and_grad(S["params"].astype(np.float64), ptr, src,
                              [m.astype(float) for m in S["masks"]], S["betas"],
                              [y.astype(float) for y in S["ys"]], bf=True)
    cos = float(gg @ rg / (np.linalg.norm(gg) * np.linalg.norm(rg)))
    big = np.abs(rg) > 1e-3 * np.abs(rg).max()
    rel = np.abs(gg - rg)[big] / np.abs(rg)[big]
    log(f"[gnn] loss gpu {loss:.6f} oracle {rl:.6f}; grad cosine {cos:.6f}, "
        f"rel err median {np.median(rel):.2e} p99 {np.quantile(rel, 0.99):.2e} max {rel.max():.2e}")
    assert abs(loss - rl) < 1e-4 * max(1.0, abs(rl))
    assert cos >= 0.999
    # elementwise on every entry above 1e-3 of the largest
    assert rel.max() <= 2e-2, (np.nonzero(big)[0][np.argmax(rel)], rel.max())


def test_training_reduces_loss(setup):
    import torch
    S = setup
    net = S["fsg"].GNN(3)
    m = torch.tensor(S["masks"], device="cuda")
    y = torch.tensor(S["ys"] * 0.0 + S["masks"] * 0.9 + 0.05, device="cuda", dtype=torch.float32)
    losses = [net.train_step(S["g"], S["rev"], m, S["betas"], y, 3e-3) for _ in range(60)]
    log(f"[gnn] loss {losses[0]:.4f} -> {losses[-1]:.4f}")
    assert losses[-1] < 0.7 * losses[0]


def test_estimator_fallback_is_plain_mc(setup):
    S = setup
    fsg = S["fsg"]
    members = [fsg.GNN(10 + i) for i in range(3)]
    est = fsg.SpreadEstimator(members, S["g"], gamma=0.1, max_steps=40, B_fallback=256, tau=0.0)
    seeds = np.array([3, 17, 99], dtype=np.int32)
    sp, unc, fb = est.estimate(seeds, 0.04, 1234, tau=-1.0)
    assert fb
    _, cnt, _, _ = fsg.simulate(S["g"], "sir", seeds, 256, 1234, beta=0.04, gamma=0.1,
                                max_steps=40, want_states=False)
    assert abs(sp - float(cnt.sum().item()) / 256) < 1e-9
    sp2, unc2, fb2 = est.estimate(seeds, 0.04, 1234, tau=1e30)
    assert not fb2 and unc2 == pytest.approx(unc)


def test_adam_matches_oracle_bit_for_bit(setup):
    """The optimiser step on seeded gradients (not from the network): FP32
    parameters, both moments and the BF16 weight copies after each of three
    steps equal the oracle's single-precision Adam bit for bit."""
    S = setup
    net = S["fsg"].GNN(4)
    p = S["params"].copy()
    net.set_params(p)
    m = np.zeros_like(p)
    v = np.zeros_like(p)
    rng = np.random.default_rng(2024)
    for t, lr in enumerate((1e-3, 3e-3, 1e-3), start=1):
        g = (rng.normal(size=p.size) * 10.0 ** rng.uniform(-9, 0, size=p.size)).astype(np.float32)
        g[::97] = 0.0
        net.apply_update(g, lr)
        p, m, v = OG.adam_step(p, m, v, g, t, lr)
        gp = net.get_params()
        gm, gv, gwb, gt = net.get_state()
        assert gt == t
        for name, a, b in (("params", gp, p), ("m", gm, m), ("v", gv, v)):
            bad = np.nonzero(a.view(np.uint32) != b.view(np.uint32))[0]
            assert bad.size == 0, (t, name, bad[:5], a[bad[:5]], b[bad[:5]])
        assert (gwb == OG.weight_copies(p)).all(), t


def test_three_train_steps_match_oracle(setup):
    """Three full training steps (forward, backward, Adam) against the oracle's
    network and Adam.  Moments follow the gradient elementwise (the first
    within 2e-2 of the same moment of |g|, the second within 4e-2 relative,
    on entries above 1e-3 of the largest); a parameter whose three gradients are
    all such entries moves as the oracle's does (Adam's step has size about lr
    whatever the gradient's scale, so the bound is in units of lr); any other
    parameter stays within its largest possible move, 3 lr."""
    import torch
    S = setup
    net = S["fsg"].GNN(5)
    p = S["params"].copy()
    net.set_params(p)
    m = np.zeros_like(p)
    v = np.zeros_like(p)
    ptr, src = S["gr"].numpy()
    masks_t = torch.tensor(S["masks"], device="cuda")
    ys_t = torch.tensor(S["ys"], device="cuda")
    lr = 1e-3
    sure = np.ones(p.size, dtype=bool)
    m_abs = np.zeros(p.size)  # the first moment of |g|: the scale of m without cancellation
    for t in range(1, 4):
        net.train_step(S["g"], S["rev"], masks_t, S["betas"], ys_t, lr)
        _, rg = OG.loss_and_grad(p.astype(np.float64), ptr, src,
                                 [mm.astype(float) for mm in S["masks"]], S["betas"],
                                 [y.astype(float) for y in S["ys"]], bf=True)
        big = np.abs(rg) > 1e-3 * np.abs(rg).max()
        sure &= big
        p, m, v = OG.adam_step(p, m, v, rg.astype(np.float32), t, lr)
        m_abs = 0.9 * m_abs + 0.1 * np.abs(rg)
        gp = net.get_params()
        gm, gv, gwb, gt = net.get_state()
        assert gt == t
        mb = m_abs > 1e-3 * m_abs.max()
        rel_m = np.abs(gm - m)[mb] / m_abs[mb]
        vb = v > 1e-6 * v.max()
        rel_v = np.abs(gv - v)[vb] / v[vb]
        dp = np.abs(gp.astype(np.float64) - p)
        log(f"[gnn] train step {t}: m rel max {rel_m.max():.2e}, v rel max {rel_v.max():.2e}, "
            f"param diff max {dp[sure].max() / lr:.2e} lr (determined), {dp.max() / lr:.2e} lr (all)")
        assert rel_m.max() <= 2e-2 and rel_v.max() <= 4e-2
        assert dp[sure].max() <= 2e-2 * lr * t
        assert dp.max() <= 2 * lr * t + 1e-7


@pytest.mark.parametrize("n,deg,sets", [(1, 0.0, 1), (15, 3.0, 1), (16, 3.0, 3), (63, 4.0, 1), (65, 4.0, 5),
                                        (130, 120.0, 2), (300, 290.0, 1), (700, 6.0, 4)])
def test_sizes_at_the_edges_of_tiles(n, deg, sets):
    """Row counts around the 16- and 64-row tiles and the partial sums' blocks,
    one to five sets, empty neighbourhoods, graphs whose every row is wide:
    forward and gradient against the FP64 oracle with the same BF16 rounding
    points.  A product's FP32 sums are of at most 128 terms and a mean is
    exact, so an activation differs by a BF16 unit (2^-8) only at a tie: 1e-3
    on a probability, 2e-2 of the largest entry on a gradient."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_14895_amd import fsg
    gr = W.erdos_renyi_directed(n, deg, 700 + n) if deg > 0 else W.from_edges(n, [])
    g, rev = fsg.DeviceGraph(*gr.numpy()), fsg.DeviceGraph(*W.reverse_graph(gr).numpy())
    rng = np.random.default_rng(n)
    masks = (rng.random((sets, n)) < 0.1).astype(np.uint8)
    masks[:, 0] = 1
    betas = [float(np.float32(x)) for x in rng.uniform(0.01, 0.05, sets)]
    ys = rng.random((sets, n)).astype(np.float32)
    params = OG.glorot(31).astype(np.float32)
    net = fsg.GNN(5)
    net.set_params(params)
    tm = torch.tensor(masks, device="cuda")
    prob = net.forward(g, tm, betas).cpu().numpy()
    ptr, src = gr.numpy()
    for s in range(sets):
        ref, _ = OG.forward(params.astype(np.float64), ptr, src, masks[s].astype(float), betas[s], bf=True)
        assert np.abs(prob[s] - ref).max() < 1e-3
    loss = net.train_step(g, rev, tm, betas, torch.tensor(ys, device="cuda"), 0.0, update=False)
    gg = net.get_grads().astype(np.float64)
    rl, rg = OG.loss_and_grad(params.astype(np.float64), ptr, src, [m.astype(float) for m in masks], betas,
                              [y.astype(float) for y in ys], bf=True)
    assert abs(loss - rl) < 1e-4 * max(1.0, abs(rl))
    assert np.abs(gg - rg).max() <= 2e-2 * np.abs(rg).max()


@pytest.mark.parametrize("members", [1, 3, 4, 5, 9])
def test_estimator_members_side_by_side(setup, members):
    """A spread estimate runs its members four at a time; every member's
    spread is the sum of its own forward pass."""
    import torch
    S = setup
    fsg = S["fsg"]
    nets = [fsg.GNN(40 + i) for i in range(members)]
    est = fsg.SpreadEstimator(nets, S["g"], gamma=0.1, max_steps=40, B_fallback=64,
                              gate=dict(tau=float("inf")))
    seeds = np.array([1, 5, 9, 60], dtype=np.int32)
    sp, unc, fb = est.estimate(seeds, 0.03, 77)
    mask = torch.zeros((1, S["gr"].n), dtype=torch.uint8)
    mask[0, torch.as_tensor(seeds, dtype=torch.int64)] = 1
    own = [float(net.forward(S["g"], mask.cuda(), [0.03]).double().sum()) for net in nets]
    assert not fb and abs(sp - np.mean(own)) <= 1e-5 * np.mean(own)  # FP32 sums of n terms in a tree
    if members > 1:
        assert abs(unc - np.std(own, ddof=1) / np.mean(own)) <= 1e-4


def test_forward_of_600000_seed_sets():
    """More seed sets than one launch over sets and their parts takes: every
    set's probabilities are those it has in a call of few sets."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_14895_amd import fsg
    n, sets = 3, 600_000
    g = fsg.DeviceGraph(*W.from_edges(n, [(0, 1), (1, 2), (2, 1)], "three").numpy())
    net = fsg.GNN(5)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(12)
    masks = (torch.rand((sets, n), generator=gen, device="cuda") < 0.4).to(torch.uint8)
    betas = torch.rand(sets, generator=gen, device="cuda").mul_(0.05).cpu().numpy()
    prob = net.forward(g, masks, betas)
    for lo in (0, 65_000, 524_000, sets - 2000):
        part = net.forward(g, masks[lo:lo + 2000].contiguous(), betas[lo:lo + 2000])
        assert torch.equal(prob[lo:lo + 2000], part), lo
    g.close()


def test_estimator_repeated_seeds_stay_in_the_workspace(setup):
    """A seed array longer than the graph (seeds repeated): the same spread as
    each seed once, nothing written past the workspace."""
    import torch
    S = setup
    fsg = S["fsg"]
    members = [fsg.GNN(30 + i) for i in range(2)]
    est = fsg.SpreadEstimator(members, S["g"], gamma=0.1, max_steps=40, B_fallback=64, tau=1e30)
    room = est.ws_bytes + (8 << 20)
    buf = torch.full((room + 256,), 0xA5, dtype=torch.uint8, device="cuda")
    est.ws_addr = (buf.data_ptr() + 255) & ~255
    end = est.ws_addr - buf.data_ptr() + est.ws_bytes
    once = np.array([3, 17, 99], dtype=np.int32)
    want = est.estimate(once, 0.04, 1234)
    got = est.estimate(np.tile(once, (est.ws_bytes + (4 << 20)) // 12), 0.04, 1234)
    assert got == want
    assert bool((buf[end:] == 0xA5).all())
