"""Warm-start MLP on the GPU (through the C ABI) against the FP64 oracle of
oracle/mlp.py: the features of the method's own links, the forward pass,
the gradient (FP16 form: 2e-2 of the largest component; FP32 test
instantiation: 1e-5) and Adam steps, and the warm-started link solver,
which must find the plain solver's roots (the Newton tolerance judges the
guess) -- also with an untrained network."""
import numpy as np
import pytest

import oracle
import workloads
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mdl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2209_10411_amd as m
    m.lib()
    return m


def oracle_features(cfg, sim, node, d, owner):
    parts = sim.particles()
    body = []
    for p in cfg.particles:
        _, c, _, _ = oracle.body_properties(p.cp_xyz, p.cp_k, cfg.quad_h)
        body.append((np.asarray(p.cp_xyz) - c, np.asarray(p.cp_k)))
    lat = oracle.lattice()
    E = lat[0] if isinstance(lat, tuple) else lat["e"]
    out = []
    for n, i, o in zip(node, d, owner):
        x = np.array([n % cfg.nx, (n // cfg.nx) % cfg.ny, n // (cfg.nx * cfg.ny)], float)
        cpb, k = body[o]
        out.append(omlp.features(cpb, k, parts[o]["x"], parts[o]["quat"], x, np.asarray(E[i], float),
                                 dims=(cfg.nx, cfg.ny, cfg.nz), periodic=cfg.periodic))
    return np.array(out)


@pytest.mark.parametrize("which", ["walled", "periodic"])
def test_link_features_match_oracle(mdl, which):
    cfg = workloads.small_settling(n=32, nz=48, R=5.0) if which == "walled" else workloads.suspension_small()
    sim = mdl.Simulation(cfg)
    sim.step(3)
    node, d, owner, q = sim.links()
    feat, target = mdl.mlp_collect(sim)
    f = feat.float().cpu().numpy()
    t = target.cpu().numpy()
    assert f.shape == (len(q), 87)
    assert np.array_equal(t[:, 0], q.astype(np.float32)) and np.all(t[:, 1:] == 0)
    sel = np.arange(0, len(q), max(1, len(q) // 400))
    ref = oracle_features(cfg, sim, node[sel], d[sel], owner[sel]).astype(np.float16).astype(np.float64)
    ulp = np.spacing(np.abs(ref).astype(np.float16)).astype(np.float64)
    assert np.all(np.abs(f[sel] - ref) <= ulp), np.abs(f[sel] - ref).max()
    sim.close()


def rand_batch(rng, n=256):
    X = rng.normal(0, 0.6, size=(n, 87))
    X[:, 6] = (np.arange(n) % 4 == 0).astype(float)
    T = rng.normal(0.4, 0.3, size=(n, 4))
    return X, T


def params(seed):
    rng = np.random.default_rng(seed)
    return workloads.mlp_init(seed) + rng.normal(0, 0.05, size=omlp.P)


@pytest.mark.parametrize("precision", [0, 1])
def test_forward_and_gradient_match_oracle(mdl, precision):
    import torch
    theta = params(11).astype(np.float32)
    net = mdl.Mlp(theta)
    X, T = rand_batch(np.random.default_rng(12))
    if precision == 0:
        Xd = torch.tensor(X, dtype=torch.float16, device="cuda:0")
        Xr = X.astype(np.float16).astype(np.float64)
        th = theta.astype(np.float16).astype(np.float64)
        tol = 2e-2
    else:
        Xd = torch.tensor(X, dtype=torch.float32, device="cuda:0")
        Xr = X.astype(np.float32).astype(np.float64)
        th = theta.astype(np.float64)
        tol = 1e-5
    Td = torch.tensor(T, dtype=torch.float32, device="cuda:0")
    Tr = T.astype(np.float32).astype(np.float64)
    out = net.forward(Xd, precision).cpu().numpy()
    ref, _ = omlp.forward(th, Xr)
    assert np.abs(out - ref).max() <= tol * np.abs(ref).max()
    g, loss = net.grad(Xd, Td, precision)
    gr = omlp.grad(th, Xr, Tr)
    assert np.abs(g - gr).max() <= tol * np.abs(gr).max(), np.abs(g - gr).max() / np.abs(gr).max()
    assert loss == pytest.approx(omlp.loss(th, Xr, Tr), rel=tol)


@pytest.mark.parametrize("n", [250, 33, 1])
def test_matrix_core_forward_matches_oracle_and_fma_form(mdl, n):
    """Precision 2 (hidden layers on the matrix cores, 32 samples a block,
    ragged last block) against the oracle on the same FP16-rounded inputs
    and weights, and against the FMA form (precision 0), which differs only
    in the order of the FP32 sums."""
    import torch
    theta = params(21).astype(np.float32)
    net = mdl.Mlp(theta)
    X, _ = rand_batch(np.random.default_rng(22), n)
    Xd = torch.tensor(X, dtype=torch.float16, device="cuda:0")
    out = net.forward(Xd, 2).cpu().numpy()
    ref, _ = omlp.forward(theta.astype(np.float16).astype(np.float64), X.astype(np.float16).astype(np.float64))
    scale = np.abs(ref).max()
    assert out.shape == (n, 4) and np.all(np.isfinite(out))
    assert np.abs(out - ref).max() <= 2e-2 * scale, np.abs(out - ref).max() / scale
    fma = net.forward(Xd, 0).cpu().numpy()
    assert np.abs(out - fma).max() <= 4e-3 * scale, np.abs(out - fma).max() / scale


def test_adam_steps_match_oracle(mdl):
    """FP32 instantiation, two minibatches; eps large enough that tiny
    gradients do not make the step sign-sensitive to rounding."""
    import torch
    theta = params(13)
    net = mdl.Mlp(theta.astype(np.float32))
    X, T = rand_batch(np.random.default_rng(14), n=512)
    Xd = torch.tensor(X, dtype=torch.float32, device="cuda:0")
    Td = torch.tensor(T, dtype=torch.float32, device="cuda:0")
    hp = dict(lr=1e-3, epochs=1, batch=256, eps=1e-3, precision=1)
    net.train(Xd, Td, **hp)
    ref = omlp.train(theta.astype(np.float32).astype(np.float64), X.astype(np.float32).astype(np.float64),
                     T.astype(np.float32).astype(np.float64), epochs=1, batch=256, lr=1e-3, eps=1e-3)
    assert np.abs(net.params() - ref).max() <= 1e-6


def shuffled_samples(mdl, sim, seed=0):
    import torch
    feat, target = mdl.mlp_collect(sim)
    g = torch.Generator(device="cpu").manual_seed(seed)
    perm = torch.randperm(feat.shape[0], generator=g).to(feat.device)
    return feat[perm].contiguous(), target[perm].contiguous()


def test_training_on_the_methods_links_reduces_the_loss(mdl):
    cfg = workloads.small_settling(n=32, nz=48, R=5.0)
    sim = mdl.Simulation(cfg)
    feat, target = shuffled_samples(mdl, sim)
    net = mdl.Mlp(workloads.mlp_init(15).astype(np.float32))
    _, l0 = net.grad(feat[:4096], target[:4096])
    net.train(feat, target, lr=3e-3, epochs=200, batch=64)
    _, l1 = net.grad(feat[:4096], target[:4096])
    print(f"links {feat.shape[0]}: loss {l0:.4e} -> {l1:.4e}", flush=True)
    assert l1 < 0.2 * l0
    sim.close()


@pytest.mark.parametrize("trained", [True, False])
def test_warm_start_finds_the_plain_roots(mdl, trained):
    cfg = workloads.small_settling(n=32, nz=48, R=5.0)
    net = mdl.Mlp(workloads.mlp_init(16).astype(np.float32))
    if trained:
        s0 = mdl.Simulation(cfg)
        feat, target = shuffled_samples(mdl, s0)
        net.train(feat, target, lr=3e-3, epochs=200, batch=64)
        s0.close()
    plain, warm = mdl.Simulation(cfg), mdl.Simulation(cfg)
    warm.set_warmstart(net)
    plain.nr_histogram()
    warm.nr_histogram()
    plain.step(10)
    warm.step(10)
    n0, d0, o0, q0 = plain.links()
    n1, d1, o1, q1 = warm.links()
    assert np.array_equal(n0, n1) and np.array_equal(d0, d1)
    dq = np.abs(q1 - q0)
    h0, r0 = plain.nr_histogram()
    h1, r1 = warm.nr_histogram()
    it = np.arange(65)
    print(f"trained={trained}: |dq| median {np.median(dq):.2e} max {dq.max():.2e}; "
          f"mean iterations plain {(h0 * it).sum() / h0.sum():.2f} warm {(h1 * it).sum() / h1.sum():.2f}; "
          f"residual plain {r0:.1e} warm {r1:.1e}", flush=True)
    assert np.median(dq) <= 1e-13 and dq.max() <= 2e-7 and np.mean(dq > 1e-11) < 0.01
    assert r1 <= 1e-10 and r0 <= 1e-10
    plain.close()
    warm.close()


def test_warm_start_on_a_held_out_system(mdl, tmp_path):
    """The warm start evaluated on a system the network never saw (seed 24;
    trained on the links of seeds 21-23 over 20 steps), plain and warm from
    one checkpointed state.  Measured result: the network learns the mean of
    q, not the sub-lattice surface position (held-out loss about var(q)), and
    the Newton iteration inside the eight-sample bracket does not need fewer
    evaluations from its guess (3.39 against 3.22 at 3 epochs; longer
    training overfits: held-out loss 1.1-2.0 at 30-200 epochs, evaluations
    3.22-3.23).  Asserted: the roots are the plain ones and the evaluation
    count does not drop -- the warm start gains nothing here."""
    import torch
    feats, targets = [], []
    for seed in (21, 22, 23):
        s = mdl.Simulation(workloads.small_settling(seed=seed, n=32, nz=48, R=5.0))
        for _ in range(4):
            f, t = mdl.mlp_collect(s)
            feats.append(f.clone())
            targets.append(t.clone())
            s.step(5)
        s.close()
    feat, target = torch.cat(feats), torch.cat(targets)
    perm = torch.randperm(feat.shape[0], generator=torch.Generator().manual_seed(0)).to(feat.device)
    feat, target = feat[perm].contiguous(), target[perm].contiguous()
    held = workloads.small_settling(seed=24, n=32, nz=48, R=5.0)
    net = mdl.Mlp(workloads.mlp_init(16).astype(np.float32))
    net.train(feat, target, lr=3e-3, epochs=3, batch=64)
    sim = mdl.Simulation(held)
    hf, ht = mdl.mlp_collect(sim)
    _, l_held = net.grad(hf[:4096], ht[:4096])
    var_q = float(ht[:4096, 0].float().var())
    sim.step(3)
    ck = str(tmp_path / "held.ckpt")
    sim.save(ck)
    sim.nr_histogram()
    sim.step(20)
    hp, _ = sim.nr_histogram()
    _, _, _, q_plain = sim.links()
    sim.load(ck)
    sim.set_warmstart(net)
    sim.nr_histogram()
    sim.step(20)
    hw, rw = sim.nr_histogram()
    _, _, _, q_warm = sim.links()
    sim.close()
    it = np.arange(len(hp))
    mp, mw = (hp * it).sum() / hp.sum(), (hw * it).sum() / hw.sum()
    print(f"held-out loss {l_held:.4e} (var q {var_q:.4e}); mean evaluations plain {mp:.3f} warm {mw:.3f}",
          flush=True)
    assert l_held > 0.5 * var_q  # the mean, not the surface position
    assert mw >= mp - 0.01  # no gain from the guess
    dq = np.abs(q_warm - q_plain)
    assert len(q_warm) == len(q_plain) and np.median(dq) <= 1e-13 and rw <= 1e-10


def _at_rest(cfg):
    """No gravity and no initial motion: the fluid stays at rest, so the
    bodies feel no load and keep their poses through a step."""
    cfg.g_particle = np.zeros(3)
    for p in cfg.particles:
        p.v = np.zeros(3)
        p.omega = np.zeros(3)
    return cfg


def test_contact_samples_match_oracle(mdl):
    """Closest-point samples (task bit 1) of the candidate pairs of a packed
    periodic suspension at rest: inputs equal to the oracle's features of the
    partner's centroid (within an FP16 ulp), targets equal to the oracle's
    stationary point of the pair in the lower body's frame."""
    cfg = _at_rest(workloads.suspension_small(n_bodies=40, box=64, seed=52))
    sim = mdl.Simulation(cfg)
    ref = oracle.Oracle(cfg)
    sim.step(1)
    body = []
    for p in cfg.particles:
        _, c, _, _ = oracle.body_properties(p.cp_xyz, p.cp_k, cfg.quad_h)
        body.append((np.asarray(p.cp_xyz) - c, np.asarray(p.cp_k)))
    parts = [ref.particle(i) for i in range(len(cfg.particles))]
    gparts = sim.particles()
    dims = (cfg.nx, cfg.ny, cfg.nz)
    for a, b in zip(gparts, parts):  # at rest: the poses of the contact sub-step (modulo the box)
        dx = a["x"] - b["x"]
        dx -= np.array(dims) * np.round(dx / np.array(dims))
        assert np.abs(dx).max() < 1e-12
    expect = []
    for i in range(len(parts)):
        for j in range(i + 1, len(parts)):
            d = parts[j]["x"] - parts[i]["x"]
            d -= np.array(dims) * np.floor(d / np.array(dims) + 0.5)
            if np.linalg.norm(d) > parts[i]["rb"] + parts[j]["rb"]:
                continue
            r, xm = ref.pair_geometry(i, j)[:2]
            if r < 0:
                continue
            cpb, k = body[i]
            x_in = omlp.features(cpb, k, parts[i]["x"], parts[i]["quat"], parts[j]["x"], np.zeros(3), dims=dims,
                                 periodic=cfg.periodic, task=1)
            off = omlp.features(cpb, k, parts[i]["x"], parts[i]["quat"], xm, np.zeros(3), dims=dims,
                                periodic=cfg.periodic, task=1)[:3]
            expect.append((x_in, off))
    feat, target = mdl.mlp_collect_contact(sim)
    f = feat.float().cpu().numpy()
    t = target.cpu().numpy()
    print(f"{len(expect)} candidate pairs solved by the oracle, {len(f)} samples", flush=True)
    assert len(f) == len(expect) and len(f) >= 3
    for s, (x_in, off) in enumerate(expect):
        ref16 = x_in.astype(np.float16).astype(np.float64)
        ulp = np.spacing(np.abs(ref16).astype(np.float16)).astype(np.float64)
        assert np.all(np.abs(f[s] - ref16) <= ulp), (s, np.abs(f[s] - ref16).max())
        assert t[s, 0] == 0.0
        assert np.abs(t[s, 1:] - off).max() < 1e-6, (s, t[s, 1:], off)
    sim.close()


@pytest.mark.parametrize("trained", [True, False])
def test_warm_started_contacts_match_plain(mdl, trained):
    """Forty bodies with contact, the pair stationary points warm-started by
    the network's closest-point outputs (trained on the method's own pair
    solutions, or untrained): the same contacts and trajectories as the plain
    start (the iteration's tolerance, the fallback and the between-centroids
    check judge the guess); solves and Newton evaluations reported."""
    import torch
    cfg = workloads.suspension_small(n_bodies=40, box=64, seed=52)
    net = mdl.Mlp(workloads.mlp_init(17).astype(np.float32))
    if trained:
        s0 = mdl.Simulation(cfg)
        fs, ts = [], []
        for _ in range(12):
            s0.step(1)
            f, t = mdl.mlp_collect_contact(s0)
            fs.append(f.clone())
            ts.append(t.clone())
        s0.close()
        feat, target = torch.cat(fs), torch.cat(ts)
        perm = torch.randperm(feat.shape[0], generator=torch.Generator().manual_seed(0)).to(feat.device)
        net.train(feat[perm].contiguous(), target[perm].contiguous(), lr=3e-3, epochs=300, batch=64)
    plain, warm = mdl.Simulation(cfg), mdl.Simulation(cfg)
    warm.set_warmstart(net)
    plain.contact_nr_stats()
    warm.contact_nr_stats()
    plain.step(15)
    warm.step(15)
    s0_, i0_ = plain.contact_nr_stats()
    s1_, i1_ = warm.contact_nr_stats()
    print(f"trained={trained}: pair solves {s0_} / {s1_}, Newton evaluations per solve plain {i0_ / s0_:.2f} "
          f"warm {i1_ / s1_:.2f}", flush=True)
    assert s0_ == s1_ and s0_ > 0
    assert plain.contact_stats() == warm.contact_stats()
    for a, b in zip(plain.particles(), warm.particles()):
        assert np.abs(a["x"] - b["x"]).max() < 1e-9
        assert np.abs(a["v"] - b["v"]).max() < 1e-9
    plain.close()
    warm.close()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 250, 257, 1000])
def test_gradient_of_ragged_batches(mdl, n):
    """Batches smaller than the sixteen slices, slices of one tile and a part
    of one, and of several tiles (FP32 form, the bound of the test above)."""
    import torch
    rng = np.random.default_rng(300 + n)
    X, T = rand_batch(rng, n)
    theta = params(9)
    net = mdl.Mlp(theta.astype(np.float32))
    th, Xr, Tr = theta.astype(np.float32).astype(np.float64), X.astype(np.float32), T.astype(np.float32)
    g, loss = net.grad(torch.tensor(Xr, device="cuda:0"), torch.tensor(Tr, device="cuda:0"), 1)
    gr = omlp.grad(th, Xr.astype(np.float64), Tr.astype(np.float64))
    assert np.abs(g - gr).max() <= 1e-5 * np.abs(gr).max()
    assert loss == pytest.approx(omlp.loss(th, Xr.astype(np.float64), Tr.astype(np.float64)), rel=1e-5)


@pytest.mark.parametrize("n,layer", [(5, "W1"), (40, "W1"), (5, "W2"), (300, "W2")])
def test_gradient_with_a_weight_beyond_fp16(mdl, n, layer):
    """A weight that FP16 holds as infinite saturates its unit (or, in the
    second layer, the unit it feeds) for every sample; the gradients of the
    layers above it stay finite, also where a slice ends within a tile.  (The
    FP16 form's bound of the test above; the oracle takes a large finite
    weight, which saturates tanh as well.)"""
    import torch
    rng = np.random.default_rng(400 + n)
    X, T = rand_batch(rng, n)
    X[:, 0] = np.where(np.abs(X[:, 0]) < 0.1, 0.3, X[:, 0])
    theta = params(15).astype(np.float32)
    big = 0 * 64 + 3 if layer == "W1" else 87 * 64 + 64 + 5 * 64 + 3
    theta[big] = 1e6
    th = theta.astype(np.float16).astype(np.float64)
    th[big] = 6e4
    Xr, Tr = X.astype(np.float16), T.astype(np.float32)
    g, loss = mdl.Mlp(theta).grad(torch.tensor(Xr, device="cuda:0"), torch.tensor(Tr, device="cuda:0"), 0)
    gr = omlp.grad(th, Xr.astype(np.float64), Tr.astype(np.float64))
    # what the infinite weight itself carries back (second layer: to unit 5 of
    # the first) is 0 times infinity; the rest is held to the bound
    ok = np.ones(omlp.P, bool)
    if layer == "W2":
        ok[np.arange(87) * 64 + 5] = False
        ok[87 * 64 + 5] = False
    assert np.all(np.isfinite(g[ok]))
    assert np.abs(g[ok] - gr[ok]).max() <= 2e-2 * np.abs(gr[ok]).max()
    assert loss == pytest.approx(omlp.loss(th, Xr.astype(np.float64), Tr.astype(np.float64)), rel=2e-2)
