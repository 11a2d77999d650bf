"""Parity of the robust sample selection (crom_sampling_residual,
crom_sampling_candidates, crom_robust_sampling) with the FP64 oracle (GPU).

* Residual vectors: the fused decode-and-compare kernel against the oracle's
  decode of every node, for the 1D (d = 1) and 3D (d = 3, Euclidean norm)
  decoders, node counts that leave a ragged last batch, several sets and
  parameters.  Bound: each term of the sum is off by at most the decode
  error, so |res_gpu - res| <= n_mu * sqrt(d) * TOL_VALUE * max|g| (TOL_VALUE
  the decode's normwise value tolerance: FP32 1e-5, BF16 1e-4).
* Candidates: integer work, bit-exact against the oracle's ranking on the
  same FP64 residual vectors (ties, NaN, members, fewer eligible nodes than
  asked for).
* The greedy loop: the GPU's rounds are replayed by the oracle along the
  GPU's own path.  Where the candidates' oracle residuals or metrics are
  closer than the tolerance the ranking is not unique, so what is checked is
  that every choice is valid within it; the metrics of the candidate sets
  must match the oracle's to TOL_METRIC (relative)."""
import numpy as np
import pytest

from oracle import heat, mlp, sampling
from oracle.inversion import GNOptions
from workloads import Elastic3D, Heat1D, rng, uniform_points, xavier_mlp

pytestmark = pytest.mark.gpu

TOL_VALUE = {"fp32": 1e-5, "bf16": 1e-4}
# FP32 rollouts: the final latents carry ~1e-6 relative error from the
# normal equations; 1e-4 leaves a factor of 10 over the largest seen.
TOL_METRIC = 1e-4


def _dev_net(layers, m, prec, cuda):
    from paper_2206_02607_amd import crom
    return crom.Decoder.from_layers([(np.asarray(W, np.float32), np.asarray(b, np.float32)) for W, b in layers],
                                    m, precision=prec, device=cuda)


@pytest.mark.parametrize("shape", ["1d", "3d"])
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_residual_matches_oracle(cuda, shape, prec):
    import torch
    from paper_2206_02607_amd import crom
    g = rng(11)
    if shape == "1d":
        m, r, d, width, depth, P = 1, 3, 1, 32, 5, 1000
    else:
        m, r, d, width, depth, P = 3, 16, 3, 256, 6, 333
    layers = xavier_mlp(g, m, r, d, width, depth, bias_scale=0.1)
    if shape == "3d":
        layers[-1] = (layers[-1][0] * 0.01, layers[-1][1] * 0.01)
    x = uniform_points(g, P, m).astype(np.float32)
    n_set, n_mu = 3, 4
    q = g.uniform(-1, 1, size=(n_set, n_mu, r))
    odec = mlp.MLPDecoder(layers, m)
    vals = np.stack([[odec.value(x.astype(np.float64), q[s, k]) for k in range(n_mu)] for s in range(n_set)])
    ref = vals[0] + 0.1 * g.standard_normal(size=(n_mu, P, d)) * np.abs(vals).max()
    want = np.sqrt(((vals - ref[None]) ** 2).sum(axis=-1)).sum(axis=1)          # [n_set, P]
    dec = _dev_net(layers, m, prec, cuda)
    res, met = crom.sampling_residual(dec, torch.from_numpy(x).to(cuda), torch.from_numpy(q).to(cuda),
                                      torch.from_numpy(ref).to(cuda))
    res, met = res.cpu().numpy(), met.cpu().numpy()
    bound = n_mu * np.sqrt(d) * TOL_VALUE[prec] * np.abs(vals).max()
    err = np.abs(res - want).max()
    print(f"{shape} {prec}: max |res| {want.max():.3e} error {err:.2e} bound {bound:.2e}")
    assert err <= bound
    for s in range(n_set):
        assert abs(met[s] - sampling.metric(want[s])) <= 2 * bound


def test_residual_of_exact_reference_is_zero(cuda):
    """ref = the GPU's own decode: every term vanishes exactly."""
    import torch
    from paper_2206_02607_amd import crom
    w = Heat1D()
    dec = _dev_net(w.layers, 1, "fp32", cuda)
    x = torch.linspace(0, 1, 777, dtype=torch.float32, device=cuda).reshape(-1, 1)
    q = torch.from_numpy(rng(3).uniform(-1, 1, size=(2, 5, 3))).to(cuda)
    ref = torch.empty(5, 777, 1, dtype=torch.float64, device=cuda)
    for k in range(5):
        ref[k] = dec.decode(x, q[1, k]).to(torch.float64)
    res, met = crom.sampling_residual(dec, x, q, ref)
    assert torch.all(res[1] == 0) and met[1].item() == 0.0
    assert torch.all(res[0] > 0)


def _ranked(res, member, n):
    return sampling.max_indices(res, list(np.flatnonzero(member)), n)


@pytest.mark.parametrize("P,n", [(5000, 10), (3000, 64), (7, 10), (1, 1)])
def test_candidates_bit_exact(cuda, P, n):
    import torch
    from paper_2206_02607_amd import crom
    g = rng(P + n)
    res = np.round(g.uniform(0, 1, size=P), 2)            # many ties
    res[g.choice(P, size=min(P, 3), replace=False)[:1]] = np.nan
    member = (g.uniform(size=P) < 0.3).astype(np.uint8)
    for mem in (None, member):
        got = crom.sampling_candidates(torch.from_numpy(res).to(cuda), n,
                                       None if mem is None else torch.from_numpy(mem).to(cuda)).cpu().numpy()
        want = _ranked(res, np.zeros(P, np.uint8) if mem is None else mem, n)
        want = want + [-1] * (n - len(want))
        np.testing.assert_array_equal(got, np.asarray(want, dtype=np.int32))


def _loop_case(seed=0):
    w = Heat1D(seed=seed)
    P = 61
    nodes = (np.arange(P) / (P - 1.0)).reshape(-1, 1)
    clamp = np.zeros(P, np.uint8)
    clamp[[0, P - 1]] = 1
    nus = np.array([0.3, 0.5, 0.8])
    q0 = rng(seed + 100).uniform(-1, 1, size=(3, w.r))
    dt, n_steps = 1e-4, 8
    ref = np.stack([heat.heat1d_modes(w.ic, nu, n_steps * dt, nodes) for nu in nus])[:, :, None]
    return w, nodes, clamp, nus, q0, dt, n_steps, ref


@pytest.mark.parametrize("linearized", [True, False])
def test_greedy_loop_follows_oracle(cuda, linearized):
    import torch
    from paper_2206_02607_amd import crom
    w, nodes, clamp, nus, q0, dt, n_steps, ref = _loop_case()
    dec = _dev_net(w.layers, 1, "fp32", cuda)
    init = [7, 19, 33, 48]
    n_try, max_samples = 4, 9
    gopts = dict(max_iter=1 if linearized else 3, linearized=linearized, tol_step=1e-7)
    out = crom.robust_sampling(dec, torch.from_numpy(nodes.astype(np.float32)).to(cuda),
                               torch.from_numpy(ref).to(cuda), q0, nus, dt, init, n_steps, target=0.0, n_try=n_try,
                               max_samples=max_samples, opts=crom.GNOptions(**gopts),
                               node_clamp=torch.from_numpy(clamp).to(cuda), trace=True)
    assert out.rounds == max_samples - len(init) and not out.reached
    assert list(out.samples[:len(init)]) == init and len(set(out.samples.tolist())) == max_samples
    odec = mlp.MLPDecoder(w.layers, 1)
    fl = sampling.heat_final_latent(odec, nodes, q0, nus, dt, n_steps, GNOptions(**{**gopts, "tol_step": 1e-10}),
                                    clamp)
    M = list(init)
    for rnd in range(out.rounds):
        res = sampling.residual(odec, nodes, ref, M, fl)
        tol_res = TOL_METRIC * res.max()
        cand = [int(c) for c in out.candidates[rnd]]
        assert not set(cand) & set(M) and len(set(cand)) == n_try
        outside = sorted((i for i in range(len(nodes)) if i not in M), key=lambda i: -res[i])
        tau = res[outside[n_try - 1]]
        assert all(res[c] >= tau - tol_res for c in cand), f"round {rnd}: not among the largest residuals"
        assert all(res[a] >= res[b] - tol_res for a, b in zip(cand, cand[1:])), f"round {rnd}: order"
        mets = np.array([sampling.metric(sampling.residual(odec, nodes, ref, M + [c], fl)) for c in cand])
        rel = np.abs(out.metrics[rnd] - mets) / mets
        print(f"round {rnd}: candidates {cand} metric error {rel.max():.2e}")
        assert rel.max() <= TOL_METRIC
        j = cand.index(int(out.samples[len(M)]))
        assert mets[j] <= mets.min() * (1 + 2 * TOL_METRIC)
        M.append(cand[j])
    assert M == list(out.samples)
    assert abs(out.metric - mets[j]) <= TOL_METRIC * mets[j]


def test_stops_at_target_and_zero_rounds(cuda):
    """max_samples = n_init evaluates the initial set only (its metric is
    the oracle's); a target above the first chosen metric stops after one
    round."""
    import torch
    from paper_2206_02607_amd import crom
    w, nodes, clamp, nus, q0, dt, n_steps, ref = _loop_case(1)
    dec = _dev_net(w.layers, 1, "fp32", cuda)
    args = (dec, torch.from_numpy(nodes.astype(np.float32)).to(cuda), torch.from_numpy(ref).to(cuda), q0, nus, dt)
    opts = crom.GNOptions(max_iter=1, linearized=True)
    init = [5, 25, 40]
    only = crom.robust_sampling(*args, init, n_steps, target=0.0, max_samples=3, opts=opts,
                                node_clamp=torch.from_numpy(clamp).to(cuda))
    assert only.rounds == 0 and list(only.samples) == init
    odec = mlp.MLPDecoder(w.layers, 1)
    fl = sampling.heat_final_latent(odec, nodes, q0, nus, dt, n_steps, GNOptions(max_iter=1, linearized=True), clamp)
    m0 = sampling.metric(sampling.residual(odec, nodes, ref, init, fl))
    assert abs(only.metric - m0) <= TOL_METRIC * m0
    one = crom.robust_sampling(*args, init, n_steps, target=0.0, max_samples=4, opts=opts,
                               node_clamp=torch.from_numpy(clamp).to(cuda))
    again = crom.robust_sampling(*args, init, n_steps, target=one.metric * (1 + 1e-9), opts=opts,
                                 node_clamp=torch.from_numpy(clamp).to(cuda))
    if one.metric < only.metric:
        assert again.reached and again.rounds == 1 and list(again.samples) == list(one.samples)
    high = crom.robust_sampling(*args, init, n_steps, target=2 * m0, opts=opts,
                                node_clamp=torch.from_numpy(clamp).to(cuda))
    assert high.reached and high.rounds == 0


def test_elastic_residual_loop_runs(cuda):
    """The neo-Hookean rollout inside the loop (q_prev carried between steps):
    one round from 6 samples, its candidates' metrics against the oracle's
    elastic rollouts."""
    import torch
    from paper_2206_02607_amd import crom
    from oracle import elastic
    w = Elastic3D()
    layers = [(np.asarray(W, np.float32), np.asarray(b, np.float32)) for W, b in w.layers]
    dec = crom.Decoder.from_layers(layers, 3, precision="fp32", device=cuda)
    sel = w.sample_idx[:80]
    nodes = w.nodes[sel]
    P = nodes.shape[0]
    clamp = (nodes[:, 0] == 0.0).astype(np.uint8)
    coef = np.array([[w.lam, w.mu, w.rho0, *w.gravity], [w.lam, 1.5 * w.mu, w.rho0, *w.gravity]])
    q0 = np.stack([w.q0, w.q0])
    n_steps = 2
    odec = mlp.MLPDecoder(layers, 3)
    gn = dict(max_iter=1, linearized=True)

    def final_latent(k, samples):
        idx = np.asarray(samples)
        q_prev, q = q0[k].copy(), q0[k].copy()
        for _ in range(n_steps):
            qn, _, _ = elastic.elastic_step(odec, nodes[idx].astype(np.float64), q, q_prev, coef[k, 0], coef[k, 1],
                                            coef[k, 2], coef[k, 3:], w.dt, GNOptions(**gn), clamp[idx])
            q_prev, q = q, qn
        return q

    ref = np.stack([odec.value(nodes.astype(np.float64), q0[k]) * 1.01 for k in range(2)])
    init = [3, 17, 29, 41, 55, 70]
    out = crom.robust_sampling(dec, torch.from_numpy(nodes.astype(np.float32)).to(cuda),
                               torch.from_numpy(ref).to(cuda), q0, coef, w.dt, init, n_steps, target=0.0, n_try=3,
                               max_samples=7, opts=crom.GNOptions(**gn), pde="neohookean",
                               node_clamp=torch.from_numpy(clamp).to(cuda), trace=True)
    assert out.rounds == 1
    cand = [int(c) for c in out.candidates[0]]
    mets = np.array([sampling.metric(sampling.residual(odec, nodes, ref, init + [c], final_latent)) for c in cand])
    rel = np.abs(out.metrics[0] - mets) / mets
    print("elastic candidate metrics", mets, "error", rel.max())
    assert rel.max() <= 1e-3


# Width 128 in BF16: a value is the decode's, bit for bit, and a node's norms
# are added in the latents' order whichever kernel takes the call: few 64-node
# batches per compute unit, and whole and cut last rounds of 256-node groups.
@pytest.mark.parametrize("n_set,n_mu,P,r", [(1, 3, 1, 8), (2, 2, 333, 8), (4, 3, 16001, 8), (6, 2, 16384, 8),
                                            (10, 2, 16384, 8), (600, 2, 70, 8), (5, 3, 12011, 16)])
def test_residual_is_the_sum_of_decode_differences(cuda, n_set, n_mu, P, r):
    import torch
    from paper_2206_02607_amd import crom
    g = rng(13)
    layers = xavier_mlp(g, 2, r, 1, 128, 5, bias_scale=0.1)
    dec = _dev_net(layers, 2, "bf16", cuda)
    x = torch.from_numpy(uniform_points(g, P, 2).astype(np.float32)).to(cuda)
    q = torch.from_numpy(g.uniform(-1, 1, size=(n_set, n_mu, r))).to(cuda)
    ref = torch.from_numpy(g.standard_normal(size=(n_mu, P, 1))).to(cuda)
    res, _ = crom.sampling_residual(dec, x, q, ref)
    for s in range(0, n_set, max(1, n_set // 3)):
        want = torch.zeros(P, dtype=torch.float64, device=cuda)
        for k in range(n_mu):
            want = want + (dec.decode(x, q[s, k]).to(torch.float64) - ref[k]).abs()[:, 0]
        assert torch.equal(res[s], want)
