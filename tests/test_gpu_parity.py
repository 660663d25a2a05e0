"""GPU parity: the HIP path (through the C ABI) against the FP64 oracle on the
same seeded inputs and float32 parameters."""
import ctypes
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2104_10013_amd import ddpinn, workloads as W
from parity_util import compare

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def run(prob, params=None, fused=True, **kw):
    pb = ddpinn.Problem(prob, fused=fused, **kw)
    if params is not None:
        pb.set_params(params)
    lt, g = pb.loss_and_grad()
    torch.cuda.synchronize()
    return pb, lt.cpu().numpy(), [x.cpu().numpy() for x in pb.split(g.cpu())]


def _params(prob, seed):
    if seed is None:
        return [s.params for s in prob.subdomains]
    return [W.perturb_params(s.params, seed, 0.1) for s in prob.subdomains]


@pytest.mark.parametrize("seed", [None, 11, 12, 13])
def test_c1_cpinn_poisson_full(seed):
    prob = W.c1_cpinn_poisson(seed=0)
    params = _params(prob, seed)
    _say(f"c1 full, perturbation {seed}")
    pb, lt, g = run(prob, params)
    wl, wg = compare(prob, params, lt, g)
    _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
    pb.close()


@pytest.mark.parametrize("seed", [None, 21])
def test_c2_xpinn_poisson_scaled(seed):
    prob = W.c2_xpinn_poisson(seed=1, scale=0.1)
    params = _params(prob, seed)
    _say(f"c2 scale 0.1, perturbation {seed}")
    pb, lt, g = run(prob, params)
    wl, wg = compare(prob, params, lt, g)
    _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
    pb.close()


def test_c2_xpinn_poisson_full_size_bench_launch():
    """Full-size 16-subdomain workload in the launch configuration the
    benchmark times (fused, work plan chosen by the autotuner), and with the
    default plan."""
    prob = W.c2_xpinn_poisson(seed=0)
    params = _params(prob, None)
    terms, grads = oracle.loss_and_grad(prob, params)
    for tuned in (True, False):
        _say(f"c2 full size, autotuned plan {tuned}")
        pb = ddpinn.Problem(prob, fused=True)
        if tuned:
            _say(f"  plan {pb.autotune(iters=3)}")
        lt, g = pb.loss_and_grad()
        torch.cuda.synchronize()
        wl, wg = compare(prob, params, lt.cpu().numpy(), [x.cpu().numpy() for x in pb.split(g.cpu())],
                         ref=(terms, grads))
        _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
        pb.close()


def test_ragged_mixed_widths_and_depths():
    """Widths across every class (incl. non-multiples of 16), depth 1..6,
    point counts that are not tile multiples, one subdomain without residual
    points, interface counts of 1 and 67."""
    widths = [[2, 20, 1], [2, 33, 33, 1], [2, 50, 50, 50, 50, 1], [2, 80] + [80] * 5 + [1]]
    prob = W.custom_box_problem("xpinn", "poisson2d", 2, 2, widths, [1, 65, 130, 0], n_bnd_seg=3, n_iface=67,
                                seed=3)
    prob.interfaces[0].xy = prob.interfaces[0].xy[:1].copy()
    params = _params(prob, 5)
    _say("ragged mixed widths")
    pb, lt, g = run(prob, params, chunk_points=64)
    compare(prob, params, lt, g)
    pb.close()


@pytest.mark.parametrize("method", ["cpinn", "xpinn"])
def test_two_subdomain_methods(method):
    prob = W.custom_box_problem(method, "poisson2d", 2, 1, [[2, 48, 48, 48, 1], [2, 24, 24, 1]], [300, 257],
                                n_bnd_seg=40, n_iface=129, seed=7)
    params = _params(prob, 8)
    _say(f"two subdomains {method}")
    pb, lt, g = run(prob, params)
    compare(prob, params, lt, g)
    pb.close()


def test_c3_cpinn_burgers_scaled():
    prob = W.c3_cpinn_burgers(seed=0, scale=0.2)
    params = _params(prob, 31)
    _say("c3 burgers scale 0.2")
    pb, lt, g = run(prob, params)
    wl, wg = compare(prob, params, lt, g)
    _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
    pb.close()


def test_c4_xpinn_kovasznay_scaled():
    prob = W.c4_xpinn_kovasznay(seed=0, scale=0.1)
    params = _params(prob, 41)
    _say("c4 kovasznay scale 0.1")
    pb, lt, g = run(prob, params)
    wl, wg = compare(prob, params, lt, g)
    _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
    pb.close()


def test_fused_matches_plain_and_is_deterministic():
    prob = W.c2_xpinn_poisson(seed=2, scale=0.1)
    _say("fused vs plain")
    pf, lt_f, g_f = run(prob, fused=True)
    lt2, g2 = pf.loss_and_grad()
    torch.cuda.synchronize()
    assert np.array_equal(lt_f, lt2.cpu().numpy())
    assert np.array_equal(np.concatenate(g_f), g2.cpu().numpy())
    pp, lt_p, g_p = run(prob, fused=False)
    np.testing.assert_allclose(lt_p, lt_f, rtol=2e-6, atol=0)
    for a, b in zip(g_p, g_f):
        assert np.linalg.norm(a - b) <= 2e-6 * np.linalg.norm(b)
    pf.close()
    pp.close()


@pytest.mark.parametrize("fused", [True, False])
def test_adam_step_matches_formula(fused):
    prob = W.c1_cpinn_poisson(seed=0, scale=0.3)
    _say(f"adam fused={fused}")
    pb = ddpinn.Problem(prob, fused=fused)
    p0 = pb.get_params()
    _, g = pb.loss_and_grad()
    g = g.cpu().numpy().astype(np.float64)
    lt = pb.step(1)
    st = pb.get_state()
    assert st["t"] == 1
    # (1 - beta) are formed in float32 by the kernel: 1 - 0.999f = 0.00099998713...
    one_m_b1 = float(np.float32(1) - np.float32(0.9))
    one_m_b2 = float(np.float32(1) - np.float32(0.999))
    np.testing.assert_allclose(st["m"], one_m_b1 * g, rtol=1e-6, atol=1e-30)
    np.testing.assert_allclose(st["v"], one_m_b2 * g * g, rtol=1e-6, atol=1e-30)
    for q in range(prob.n_sd):
        gq = pb.split(g)[q]
        ref = p0[q].astype(np.float64) - prob.subdomains[q].lr * gq / (np.abs(gq) + 1e-8)
        np.testing.assert_allclose(st["params"][q], ref, rtol=1e-6, atol=1e-6 * prob.subdomains[q].lr)
    pb.close()


def test_training_trajectory_loosely_follows_oracle():
    """100 Adam steps of the 4-subdomain cPINN Poisson problem at full size:
    every subdomain's loss follows the FP64 oracle's trajectory."""
    prob = W.c1_cpinn_poisson(seed=0)
    n = 100
    _say("trajectory 100 steps")
    pb = ddpinn.Problem(prob, fused=True)
    hist = []
    for _ in range(n):
        hist.append(pb.step(1).cpu().numpy().copy())
    ps_ref, hist_ref = oracle.train(prob, [s.params for s in prob.subdomains], n)
    hist = np.stack(hist)
    np.testing.assert_allclose(hist[:, :, 0], hist_ref[:, :, 0], rtol=1e-3)
    pb.close()


def test_checkpoint_resume_bitwise():
    """50 steps, save, restore into a new problem, 50 more: the same bits as
    100 straight steps."""
    prob = W.c1_cpinn_poisson(seed=0, scale=0.2)
    _say("checkpoint resume")
    a = ddpinn.Problem(prob, fused=True)
    a.step(50)
    st = a.get_state()
    a.step(50)
    pa = a.get_params()
    b = ddpinn.Problem(prob, fused=True)
    b.set_state(st)
    b.step(50)
    pb_ = b.get_params()
    for x, y in zip(pa, pb_):
        assert np.array_equal(x, y)
    assert b.get_state()["t"] == 100
    a.close()
    b.close()


def test_stitched_eval_matches_oracle():
    prob = W.c2_xpinn_poisson(seed=0, scale=0.05)
    _say("stitched eval")
    pb = ddpinn.Problem(prob, fused=True)
    idx = np.arange(0, prob.eval_xy.shape[0], 37)
    u = pb.eval(prob.eval_xy[idx], prob.eval_owner[idx]).cpu().numpy()
    ref = oracle.eval_stitched(prob, [s.params for s in prob.subdomains], prob.eval_xy[idx], prob.eval_owner[idx])
    np.testing.assert_allclose(u, ref, rtol=1e-5, atol=1e-6)
    pb.close()


def test_nonfinite_loss_is_reported():
    prob = W.c1_cpinn_poisson(seed=0, scale=0.1)
    _say("non-finite flag")
    pb = ddpinn.Problem(prob, fused=True)
    pb.sync()
    bad = [s.params.copy() for s in prob.subdomains]
    bad[2][:] = np.nan
    pb.set_params(bad)
    pb.loss_and_grad()
    with pytest.raises(ddpinn.DDPError) as ei:
        pb.sync()
    assert ei.value.code == ddpinn.DDP_ENONFINITE
    pb.set_params([s.params for s in prob.subdomains])
    pb.loss_and_grad()
    pb.sync()
    pb.close()


def test_autograd_function_backward():
    prob = W.c1_cpinn_poisson(seed=0, scale=0.1)
    _say("autograd function")
    pb = ddpinn.Problem(prob, fused=True)
    flat = torch.tensor(np.concatenate([s.params for s in prob.subdomains]), device="cuda", requires_grad=True)
    J = ddpinn.DDPLoss.apply(flat, pb)
    w = torch.tensor([1.0, 2.0, 0.5, -1.0], device="cuda")
    (J * w).sum().backward()
    _, g = pb.loss_and_grad()
    ref = torch.cat([g[pb.offsets[q]:pb.offsets[q + 1]] * w[q] for q in range(4)])
    assert torch.equal(flat.grad, ref)
    pb.close()


@pytest.mark.parametrize("name", ["c3_cpinn_burgers", "c4_xpinn_kovasznay", "c1_cpinn_poisson"])
def test_full_size_configs_at_init(name):
    """Every workload at its full size, fused launch, initial parameters."""
    prob = W.make_problem(name, seed=0)
    params = _params(prob, None)
    _say(f"{name} full size")
    pb, lt, g = run(prob, params)
    wl, wg = compare(prob, params, lt, g)
    _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
    pb.close()


def test_c4_adjoint_vs_central_fd_of_oracle_loss():
    """The GPU gradient of a Navier-Stokes subdomain loss against central
    differences (h = 1e-3, FP64) of the oracle's J_q on sampled parameters."""
    prob = W.c4_xpinn_kovasznay(seed=0, scale=0.02)
    params = _params(prob, 5)
    _say("c4 adjoint vs central FD")
    pb, lt, g = run(prob, params)
    rng = np.random.default_rng(0)
    for q in (0, 4):
        idx = rng.choice(len(params[q]), 12, replace=False)
        base = [torch.tensor(p, dtype=torch.float64) for p in params]
        for i in idx:
            h = 1e-3
            bp = [b.clone() for b in base]
            bm = [b.clone() for b in base]
            bp[q][i] += h
            bm[q][i] -= h
            jp = float(oracle.subdomain_terms(prob, q, bp)[0].detach())
            jm = float(oracle.subdomain_terms(prob, q, bm)[0].detach())
            fd = (jp - jm) / (2 * h)
            scale = np.linalg.norm(g[q]) / np.sqrt(len(g[q]))
            assert abs(g[q][i] - fd) <= 1e-3 * max(abs(fd), scale), (q, i, g[q][i], fd)
    pb.close()


def test_autotune_keeps_results_and_caches(tmp_path):
    prob = W.c2_xpinn_poisson(seed=3, scale=0.1)
    _say("autotune")
    pb, lt0, g0 = run(prob)
    cache = tmp_path / "tune.jsonl"
    choice = pb.autotune(iters=2, cache_path=cache)
    assert choice["recompute"] in (0, 1) and choice["concurrent"] in (0, 1) and choice["tail"] in (0, 30)
    assert cache.exists() and len(cache.read_text().splitlines()) == 1
    lt1, g1 = pb.loss_and_grad()
    torch.cuda.synchronize()
    compare(prob, [s.params for s in prob.subdomains], lt1.cpu().numpy(), [x.cpu().numpy() for x in pb.split(g1.cpu())])
    # a second problem with the same signature takes the cached choice without a search
    pb2 = ddpinn.Problem(prob, fused=True)
    assert pb2.autotune(iters=2, cache_path=cache) == choice
    assert len(cache.read_text().splitlines()) == 1
    pb.step(2)
    pb.sync()
    pb.close()
    pb2.close()


# --------------------------------------------------------------------------
# inverse diffusion (Eq. heq): u- and K-network per subdomain, paired items


@pytest.mark.parametrize("seed", [None, 51])
def test_c5_inverse_scaled(seed):
    prob = W.c5_xpinn_inverse_diffusion(seed=0, scale=0.03)
    params = _params(prob, seed)
    _say(f"c5 scale 0.03, perturbation {seed}")
    pb, lt, g = run(prob, params)
    wl, wg = compare(prob, params, lt, g)
    _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
    pb.close()


def test_c5_inverse_full_size_bench_launch():
    prob = W.c5_xpinn_inverse_diffusion(seed=0)
    params = _params(prob, None)
    _say("c5 full size")
    pb, lt, g = run(prob, params)
    wl, wg = compare(prob, params, lt, g)
    _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
    pb.close()


def test_concurrent_launches_match_sequential_bitwise():
    """Items that need the two train kernels (networks up to 80 and wider):
    the two persistent launches side by side on two streams give the same
    bits as one after the other, in a loss-and-gradient pass and over graph
    steps with Adam; full size against the oracle."""
    prob = W.c5_xpinn_inverse_diffusion(seed=0, scale=0.05)
    params = _params(prob, 7)
    out = {}
    for conc in (0, 1):
        _say(f"c5 scale 0.05 concurrent {conc}")
        pb, lt, g = run(prob, params, concurrent=conc)
        pb.step(3)
        pb.sync()
        out[conc] = (lt, g, pb.get_params())
        pb.close()
    assert np.array_equal(out[0][0], out[1][0])
    for a, b in zip(out[0][1], out[1][1]):
        assert np.array_equal(a, b)
    for a, b in zip(out[0][2], out[1][2]):
        assert np.array_equal(np.asarray(a), np.asarray(b))
    compare(prob, params, out[1][0], out[1][1])
    prob = W.c5_xpinn_inverse_diffusion(seed=0)
    params = _params(prob, None)
    _say("c5 full size concurrent 1")
    pb, lt, g = run(prob, params, concurrent=1)
    wl, wg = compare(prob, params, lt, g)
    _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
    pb.close()


def test_c5_inverse_narrow_ragged_fused_and_plain():
    """Narrow and mixed widths for both networks (non-multiples of 16), short
    point sets that end inside a tile, fused and per-subdomain launches."""
    prob = W.c5_xpinn_inverse_diffusion(seed=3, scale=0.01)
    rng = np.random.default_rng(0)
    choices = [[2, 20, 1], [2, 33, 33, 1], [2, 40, 40, 40, 1], [2, 17, 17, 17, 17, 1]]
    for q, s in enumerate(prob.subdomains):
        s.widths = list(choices[q % 4])
        s.aux_widths = list(choices[(q + 1) % 4])
        s.params = np.concatenate([W.glorot_params(rng, s.widths), W.glorot_params(rng, s.aux_widths)])
    params = _params(prob, 7)
    for fused in (True, False):
        _say(f"c5 narrow ragged fused={fused}")
        pb, lt, g = run(prob, params, fused=fused, chunk_points=64)
        compare(prob, params, lt, g)
        pb.close()


def test_c5_stitched_eval_and_adam_step():
    prob = W.c5_xpinn_inverse_diffusion(seed=0, scale=0.02)
    params = _params(prob, 61)
    _say("c5 eval and one Adam step")
    pb = ddpinn.Problem(prob, fused=True)
    pb.set_params(params)
    idx = np.arange(0, prob.eval_xy.shape[0], 23)
    uk = pb.eval(prob.eval_xy[idx], prob.eval_owner[idx]).cpu().numpy()
    ref = oracle.eval_stitched(prob, params, prob.eval_xy[idx], prob.eval_owner[idx])
    assert uk.shape == ref.shape == (idx.size, 2)
    np.testing.assert_allclose(uk, ref, rtol=1e-5, atol=1e-6)
    _, grads = oracle.loss_and_grad(prob, params)
    pb.step(1)
    got = pb.get_params()
    for q, s in enumerate(prob.subdomains):
        th, _, _ = oracle.adam_step(params[q].astype(np.float64), 0.0, 0.0, grads[q], 1, s.lr)
        # step 1 moves every parameter by about lr * sign(g): compare the step
        step = got[q].astype(np.float64) - params[q].astype(np.float64)
        ref_step = th - params[q].astype(np.float64)
        big = np.abs(grads[q]) > 1e-3 * np.abs(grads[q]).max()
        np.testing.assert_allclose(step[big], ref_step[big], rtol=2e-3, atol=2e-6 * s.lr)
    pb.close()


def test_extreme_network_sizes_and_an_empty_subdomain():
    """Maximum sizes (width 112 with 8 hidden layers, the widest class and
    deepest stash), the narrowest networks (widths 1, 3 and 16), Navier-Stokes
    outputs on a wide net, and a subdomain without any points (zero loss and
    gradient, parameters unchanged by Adam)."""
    widths = [[2] + [112] * 8 + [1], [2, 1, 1], [2, 3, 3, 3, 1], [2] + [16] * 7 + [1]]
    prob = W.custom_box_problem("xpinn", "poisson2d", 2, 2, widths, [150, 70, 1, 0], n_bnd_seg=5, n_iface=19,
                                seed=11)
    # the fourth box keeps no points at all: no data, no interfaces
    s3 = prob.subdomains[3]
    s3.bnd_xy, s3.bnd_g = s3.bnd_xy[:0], s3.bnd_g[:0]
    prob.interfaces = [e for e in prob.interfaces if 3 not in (e.a, e.b)]
    params = _params(prob, 13)
    _say("extreme sizes and an empty subdomain")
    pb, lt, g = run(prob, params, chunk_points=64)
    compare(prob, params, lt, g)
    assert np.all(lt[3] == 0) and np.all(g[3] == 0)
    pb.step(1)
    assert np.array_equal(pb.get_params()[3], params[3])
    pb.close()
    prob = W.custom_box_problem("xpinn", "ns2d_steady", 2, 1, [[2] + [112] * 3 + [3], [2, 7, 7, 3]], [90, 40],
                                n_bnd_seg=6, n_iface=23, seed=12, coef=(40.0,), domain=(-0.5, 1.0, -0.5, 1.5))
    params = _params(prob, 14)
    _say("navier-stokes width 112")
    pb, lt, g = run(prob, params)
    compare(prob, params, lt, g)
    pb.close()


def test_c5_training_trajectory_loosely_follows_oracle():
    """30 Adam steps of a small inverse problem (both networks per cell): the
    per-subdomain losses follow the FP64 oracle's trajectory."""
    prob = W.c5_xpinn_inverse_diffusion(seed=1, scale=0.02)
    n = 30
    _say("c5 trajectory 30 steps")
    pb = ddpinn.Problem(prob, fused=True)
    hist = np.stack([pb.step(1).cpu().numpy().copy() for _ in range(n)])
    _, hist_ref = oracle.train(prob, [s.params for s in prob.subdomains], n)
    np.testing.assert_allclose(hist[:, :, 0], hist_ref[:, :, 0], rtol=2e-3)
    pb.close()


@pytest.mark.parametrize("method,nx,nt", W.TABLE3_PARTITIONS)
def test_space_time_burgers_partitions_full_size(method, nx, nt):
    """Every space-time partition of the viscous Burgers comparison (80k
    residual points, 2-20x5-1 networks), at init and perturbed; the 4 x 4
    XPINN and 16-strip cPINN cases also in the autotuned plan and the plain
    path."""
    prob = W.make_problem(f"burgers_st_{method}_{nx}x{nt}", seed=0)
    variants = [(None, True, False)]
    if (method, nx, nt) in (("xpinn", 4, 4), ("cpinn", 16, 1)):
        variants += [(61, True, True), (61, False, False)]
    for seed, fused, tuned in variants:
        params = _params(prob, seed)
        _say(f"burgers {method} {nx}x{nt} perturbation {seed} fused {fused} autotuned {tuned}")
        pb = ddpinn.Problem(prob, fused=fused)
        pb.set_params(params)
        if tuned:
            _say(f"  plan {pb.autotune(iters=3)}")
        lt, g = pb.loss_and_grad()
        torch.cuda.synchronize()
        wl, wg = compare(prob, params, lt.cpu().numpy(), [x.cpu().numpy() for x in pb.split(g.cpu())])
        _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
        pb.close()


def test_space_time_burgers_training_trajectory_loosely_follows_oracle():
    """20 Adam steps of the 2 x 2 space-time XPINN case at a fifth of its
    points: the per-subdomain losses follow the FP64 oracle's trajectory."""
    prob = W.burgers_space_time("xpinn", 2, 2, seed=2, scale=0.2)
    n = 20
    _say("burgers space-time trajectory 20 steps")
    pb = ddpinn.Problem(prob, fused=True)
    hist = np.stack([pb.step(1).cpu().numpy().copy() for _ in range(n)])
    _, hist_ref = oracle.train(prob, [s.params for s in prob.subdomains], n)
    np.testing.assert_allclose(hist[:, :, 0], hist_ref[:, :, 0], rtol=1e-3)
    pb.close()


@pytest.mark.parametrize("scale,seed", [(0.1, 71), (1.0, None)])
def test_ns_cpinn_kovasznay(scale, seed):
    """Navier-Stokes with cPINN interfaces: the momentum and mass fluxes of
    Table 1 matched across the 12 interfaces of the 3 x 3 Kovasznay problem."""
    prob = W.ns_cpinn_kovasznay(seed=0, scale=scale)
    params = _params(prob, seed)
    for fused in ((True, False) if scale < 1 else (True,)):
        _say(f"ns cpinn scale {scale} perturbation {seed} fused {fused}")
        pb, lt, g = run(prob, params, fused=fused)
        wl, wg = compare(prob, params, lt, g)
        _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
        pb.close()


def test_ns_cpinn_ragged_mixed_widths():
    """cPINN Navier-Stokes on 2 x 2 boxes of widths 17..96 with tile-ragged
    point counts and 1..67 interface points."""
    widths = [[2, 17, 17, 3], [2, 40, 40, 40, 3], [2, 64] * 1 + [64] * 3 + [3], [2, 96, 96, 3]]
    prob = W.custom_box_problem("cpinn", "ns2d_steady", 2, 2, widths, [65, 130, 1, 77], n_bnd_seg=5,
                                n_iface=67, seed=9, coef=(40.0,), domain=(-0.5, 1.0, -0.5, 1.5))
    prob.interfaces[1].xy = prob.interfaces[1].xy[:1].copy()
    params = _params(prob, 10)
    _say("ns cpinn ragged mixed widths")
    pb, lt, g = run(prob, params, chunk_points=64)
    compare(prob, params, lt, g)
    pb.close()


@pytest.mark.parametrize("seed", [None, 81])
def test_space_time_burgers_hybrid(seed):
    """cPINN flux matching across the space interfaces and XPINN residual
    continuity across the time interfaces of the 4 x 4 space-time Burgers
    decomposition, in one launch."""
    prob = W.make_problem("burgers_st_hybrid_4x4", seed=0)
    assert {e.method for e in prob.interfaces} == {"cpinn", "xpinn"}
    params = _params(prob, seed)
    _say(f"burgers hybrid 4x4 perturbation {seed}")
    pb, lt, g = run(prob, params)
    wl, wg = compare(prob, params, lt, g)
    _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
    pb.close()


# ---------------------------------------------------------------------------
# activation choice and trainable slopes (Sec. 3, Table 4)


def _slope_identity_gaps(sd, theta, grad):
    """a^k dJ/da^k - (<W^k, dJ/dW^k> + <b^k, dJ/db^k>) relative to the terms'
    size, for every hidden layer of each of the subdomain's networks."""
    gaps, off = [], 0
    th, g = theta.astype(np.float64), grad.astype(np.float64)
    for wd in [sd.widths] + ([sd.aux_widths] if sd.aux_widths is not None else []):
        lay = []
        for k in range(1, len(wd)):
            n = wd[k] * wd[k - 1] + wd[k]
            lay.append(slice(off, off + n))
            off += n
        for k in range(len(wd) - 2):
            lhs = th[off + k] * g[off + k]
            prod = th[lay[k]] * g[lay[k]]
            gaps.append(abs(lhs - prod.sum()) / max(np.abs(prod).sum(), 1e-30))
        off += len(wd) - 2
    return gaps


@pytest.mark.parametrize("scale,seed", [(0.05, 91), (1.0, None)])
def test_table4_adaptive_inverse(scale, seed):
    """The inverse problem with Table 4's networks (adaptive tanh / sin / cos
    per subdomain, 3 x 80 for u and K): loss terms and gradients, slopes
    included, against the oracle; at full size also the slope identity of
    every layer on the GPU's own gradient."""
    prob = W.c5_table4_adaptive(seed=0, scale=scale)
    params = _params(prob, seed)
    _say(f"table 4 adaptive scale {scale} perturbation {seed}")
    pb, lt, g = run(prob, params)
    wl, wg = compare(prob, params, lt, g)
    _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
    if scale == 1.0:
        worst = max(max(_slope_identity_gaps(s, params[q], g[q])) for q, s in enumerate(prob.subdomains))
        _say(f"  slope identity worst {worst:.2e}")
        assert worst < 1e-4
    pb.close()


def _mixed_activation_problem(method, pde):
    """2 x 2 boxes across width classes: a plain tanh network, then adaptive
    sin, cos and tanh networks (neighbours of different kinds)."""
    if pde == "poisson2d":
        widths = [[2, 20, 20, 1], [2, 40, 40, 40, 1], [2, 64, 64, 1], [2, 96, 96, 96, 1]]
        prob = W.custom_box_problem(method, pde, 2, 2, widths, [65, 130, 1, 200], n_bnd_seg=7, n_iface=67, seed=12)
    else:
        widths = [[2, 17, 17, 3], [2, 48, 48, 3], [2, 33, 33, 33, 3], [2, 80, 80, 3]]
        prob = W.custom_box_problem(method, pde, 2, 2, widths, [70, 64, 129, 90], n_bnd_seg=5, n_iface=41, seed=13,
                                    coef=(40.0,), domain=(-0.5, 1.0, -0.5, 1.5))
    W.with_activations(prob, ("tanh", "sin", "cos", "tanh"))
    s0 = prob.subdomains[0]
    s0.adaptive, s0.params = False, s0.params[:W.param_count(s0.widths)].copy()
    return prob


@pytest.mark.parametrize("method,pde", [("xpinn", "poisson2d"), ("cpinn", "poisson2d"), ("cpinn", "ns2d_steady")])
def test_mixed_activations_across_classes(method, pde):
    prob = _mixed_activation_problem(method, pde)
    params = _params(prob, 14)
    for fused in (True, False):
        _say(f"mixed activations {method} {pde} fused {fused}")
        pb, lt, g = run(prob, params, fused=fused, chunk_points=64)
        wl, wg = compare(prob, params, lt, g)
        _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
        pb.close()


def test_adaptive_sin_burgers_space_time():
    """Adaptive sin and cos networks on the space-time Burgers problem (only
    u_xx in the second-order stream)."""
    prob = W.with_activations(W.burgers_space_time("xpinn", 2, 2, seed=3, scale=0.02), ("sin", "cos"))
    params = _params(prob, 15)
    _say("adaptive burgers space-time")
    pb, lt, g = run(prob, params)
    compare(prob, params, lt, g)
    pb.close()


def test_table4_eval_adam_and_trajectory():
    """Stitched evaluation with the activations and slopes, one Adam step
    (slopes included) and 20 steps of loss history against the oracle."""
    prob = W.c5_table4_adaptive(seed=1, scale=0.02)
    params = _params(prob, 16)
    _say("table 4 eval, Adam step, trajectory")
    pb = ddpinn.Problem(prob, fused=True)
    pb.set_params(params)
    idx = np.arange(0, prob.eval_xy.shape[0], 23)
    uk = pb.eval(prob.eval_xy[idx], prob.eval_owner[idx]).cpu().numpy()
    ref = oracle.eval_stitched(prob, params, prob.eval_xy[idx], prob.eval_owner[idx])
    np.testing.assert_allclose(uk, ref, rtol=1e-5, atol=1e-6)
    _, grads = oracle.loss_and_grad(prob, params)
    pb.step(1)
    got = pb.get_params()
    for q, s in enumerate(prob.subdomains):
        th, _, _ = oracle.adam_step(params[q].astype(np.float64), 0.0, 0.0, grads[q], 1, s.lr)
        step = got[q].astype(np.float64) - params[q].astype(np.float64)
        ref_step = th - params[q].astype(np.float64)
        big = np.abs(grads[q]) > 1e-3 * np.abs(grads[q]).max()
        np.testing.assert_allclose(step[big], ref_step[big], rtol=2e-3, atol=2e-6 * s.lr)
    pb.close()
    pb = ddpinn.Problem(prob, fused=True)
    pb.set_params(params)
    hist = np.stack([pb.step(1).cpu().numpy().copy() for _ in range(20)])
    _, hist_ref = oracle.train(prob, params, 20)
    np.testing.assert_allclose(hist[:, :, 0], hist_ref[:, :, 0], rtol=2e-3)
    pb.close()


def test_mfma_probe_rate():
    """The attainable FP32 MFMA rate: positive, at most the published peak
    (157.3 TFLOP/s, with a margin for timing), and well above what a
    one-wave-per-SIMD latency-bound loop would show."""
    t = ddpinn.mfma_probe(2000)
    _say(f"mfma probe {t:.1f} TFLOP/s")
    assert 60.0 < t < 165.0


def test_cpinn_burgers_time_interfaces():
    """cPINN across space and time interfaces of 2 x 3 space-time boxes: the
    time component u of the space-time flux and its adjoint."""
    prob = W.burgers_space_time("cpinn", 2, 3, seed=4, scale=0.05)
    assert any(tuple(e.normal) == (0.0, 1.0) for e in prob.interfaces)
    params = _params(prob, 17)
    _say("cpinn burgers with time interfaces")
    for fused in (True, False):
        pb, lt, g = run(prob, params, fused=fused)
        compare(prob, params, lt, g)
        pb.close()


def test_general_activation_kernels_match_plain_bitwise():
    """A tanh problem runs in the plain kernels; the same problem with one
    extra, unconnected sin subdomain runs in the general-activation kernels.
    With one tile per work item (the same summation order), the tanh
    subdomains' loss terms and gradients agree bit for bit."""
    base = W.custom_box_problem("xpinn", "poisson2d", 2, 2,
                                [[2, 20, 20, 1], [2, 48, 48, 48, 1], [2, 64, 64, 1], [2, 80, 80, 80, 1]],
                                [130, 257, 64, 199], n_bnd_seg=9, n_iface=77, seed=21)
    extra = W.custom_box_problem("xpinn", "poisson2d", 1, 1, [[2, 33, 33, 1]], [90], n_bnd_seg=5, n_iface=1,
                                 seed=22, domain=(2.0, 3.0, 0.0, 1.0))
    W.with_activations(extra, ("sin",))
    mixed = W.custom_box_problem("xpinn", "poisson2d", 2, 2,
                                 [[2, 20, 20, 1], [2, 48, 48, 48, 1], [2, 64, 64, 1], [2, 80, 80, 80, 1]],
                                 [130, 257, 64, 199], n_bnd_seg=9, n_iface=77, seed=21)
    mixed.subdomains.append(extra.subdomains[0])
    params = _params(base, 23)
    _say("general-activation kernels vs plain, bitwise")
    pa, la, ga = run(base, params, chunk_points=64)
    pb, lb, gb = run(mixed, params + [extra.subdomains[0].params], chunk_points=64)
    assert np.array_equal(la, lb[:4])
    for q in range(4):
        assert np.array_equal(ga[q], gb[q])
    pa.close()
    pb.close()


@pytest.mark.parametrize("others", [0, 1, 2, 3])
def test_second_stream_beside_any_caller_stream(others):
    """The stream of the second train launch is chosen by what runs beside the
    caller's; whichever hardware queue the caller's stream has, after any
    number of other streams, the bits are those of one launch after the other."""
    prob = W.c5_xpinn_inverse_diffusion(seed=0, scale=0.05)
    params = _params(prob, 7)
    streams = [torch.cuda.Stream() for _ in range(others + 1)]
    for s in streams:
        with torch.cuda.stream(s):
            torch.zeros(8, device="cuda").add_(1)
    out = []
    for conc in (0, 1):
        _say(f"{others} other streams, concurrent {conc}")
        with torch.cuda.stream(streams[-1]):
            pb, lt, g = run(prob, params, concurrent=conc)
        out.append((lt, g))
        pb.close()
    assert np.array_equal(out[0][0], out[1][0])
    for a, b in zip(out[0][1], out[1][1]):
        assert np.array_equal(a, b)


def test_phase_timing_of_the_fused_step():
    """Train time split by point kind on the 16-subdomain problem: residual
    items dominate, every phase is timed, and the phases add up to at least
    the whole launch (their separate launches cannot overlap)."""
    prob = W.c2_xpinn_poisson(seed=0)
    pb = ddpinn.Problem(prob, fused=True)
    pb.step(2)
    ph = pb.time_phases(5)
    kt = pb.time_kernels(5)
    _say(f"phases {ph} kernels {kt}")
    assert ph["residual_ms"] > ph["interface_ms"] > 0 and ph["data_ms"] > 0
    assert ph["residual_ms"] + ph["interface_ms"] + ph["data_ms"] >= 0.9 * ph["all_ms"]
    assert 0.5 * kt["train_ms"] < ph["all_ms"] < 2.0 * kt["train_ms"]
    pl = ddpinn.Problem(prob, fused=False)
    with pytest.raises(ddpinn.DDPError):
        pl.time_phases(1)
    pl.close()
    pb.close()


def test_many_subdomains_random_widths_and_depths():
    """64 subdomains (8 x 8, XPINN Poisson) with a random width from 16 to 112
    and 1-6 hidden layers each, ragged residual counts (some empty) and 1-90
    points per interface: both width-class launches, both paths."""
    rng = np.random.default_rng(31)
    widths = [[2] + [int(rng.integers(16, 113))] * int(rng.integers(1, 7)) + [1] for _ in range(64)]
    counts = [int(c) if c > 20 else 0 for c in rng.integers(0, 400, 64)]
    prob = W.custom_box_problem("xpinn", "poisson2d", 8, 8, widths, counts, n_bnd_seg=6, n_iface=90, seed=32)
    for e in prob.interfaces:
        e.xy = e.xy[: int(rng.integers(1, 91))].copy()
    params = _params(prob, 33)
    for fused in (True, False):
        _say(f"64 random subdomains fused {fused}")
        pb, lt, g = run(prob, params, fused=fused)
        wl, wg = compare(prob, params, lt, g)
        _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
        pb.close()


@pytest.mark.parametrize("name,scale", [("c2_xpinn_poisson", 0.1), ("c5_xpinn_inverse_diffusion", 0.03),
                                        ("c5_table4_adaptive", 0.1), ("c3_cpinn_burgers", 0.2),
                                        ("burgers_st_xpinn_2x2", 0.2), ("burgers_st_cpinn_4x1", 0.2)])
def test_recompute_policy(name, scale):
    """Both activation policies (stash a^k and h^k; stash a^k and rebuild h^k
    in the reverse pass) against the oracle, on both paths.  The space-time
    Burgers cases (narrow networks: layer 1 is short, so the next layer's
    weights are still in flight to LDS at the barrier that hands them to the
    other waves unless every wave waits for its own copies) run the fused
    path three times."""
    prob = W.make_problem(name, seed=0, scale=scale)
    params = _params(prob, 5)
    ref = oracle.loss_and_grad(prob, params)
    reps = 3 if name.startswith("burgers_st") else 1
    for fused in (True, False):
        for rh in (0, 1):
            for _ in range(reps if fused else 1):
                _say(f"{name} scale {scale} fused {fused} recompute {rh}")
                pb, lt, g = run(prob, params, fused=fused, recompute=rh)
                wl, wg = compare(prob, params, lt, g, ref=ref)
                _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
                pb.close()


@pytest.mark.parametrize("name,scale,seed", [("c2_xpinn_poisson", 0.1, 1), ("burgers_st_xpinn_2x2", 0.2, 0),
                                             ("c5_xpinn_inverse_diffusion", 0.03, 0)])
def test_work_plans_against_oracle(name, scale, seed):
    """The work plans the autotuner chooses among (points per item, items per
    workgroup, workgroups per CU, activation policy, tail share of one-tile
    items, and for the inverse problem side-by-side launches) all give the
    oracle's loss and gradient."""
    prob = W.make_problem(name, seed=seed, scale=scale)
    params = _params(prob, 3)
    ref = oracle.loss_and_grad(prob, params)
    conc = (0, 1) if name.startswith("c5") else (0,)
    worst = 0.0
    for chunk in (64, 512, 4096):
        for ips in (1, 8):
            for bpc in (1, 2):
                for rh in (0, 1):
                    for cc in conc:
                        tail = 30 if (ips == 8) == (rh == 1) else 0
                        pb, lt, g = run(prob, params, chunk_points=chunk, items_per_slot=ips, blocks_per_cu=bpc,
                                        recompute=rh, concurrent=cc, tail=tail)
                        try:
                            wl, wg = compare(prob, params, lt, g, ref=ref)
                        except AssertionError:
                            _say(f"{name} plan {chunk}/{ips}/{bpc}/rh{rh}/c{cc} failed")
                            raise
                        worst = max(worst, wl, wg)
                        pb.close()
    _say(f"{name}: every plan within the bar, worst {worst:.2e}")


@pytest.mark.parametrize("widths", [(1, 15, 16, 17), (31, 32, 33, 47), (48, 49, 63, 64), (65, 79, 80, 81),
                                    (95, 96, 97, 112)])
@pytest.mark.parametrize("acts", ["tanh", "mixed"])
def test_every_width_class_at_its_edges(widths, acts):
    """Each width class with its odd or even number of 16-neuron blocks, at its
    edges, one hidden-to-hidden product and several, over more than one tile
    per work item with a last tile of one point: the split bf16 contractions,
    the dW staging and its left-over blocks, the stash of each class, with the
    plain and the general activation rule.  The bound is that of compare."""
    depths = (2, 3, 4, 2)
    prob = W.custom_box_problem("xpinn", "poisson2d", 2, 2, [[2] + [w] * d + [1] for w, d in zip(widths, depths)],
                                [129, 193, 65, 130], n_bnd_seg=9, n_iface=17, seed=sum(widths))
    if acts == "mixed":
        W.with_activations(prob, ("tanh", "sin", "tanh", "cos"))
    params = _params(prob, 31)
    for chunk in (64, 4096):
        _say(f"widths {widths} {acts} chunk {chunk}")
        pb, lt, g = run(prob, params, chunk_points=chunk, items_per_slot=1)
        wl, wg = compare(prob, params, lt, g)
        _say(f"  worst loss rel {wl:.2e} grad rel {wg:.2e}")
        pb.close()


def _eval_by_slots(prob, params, xy, owner):
    """Eq. FSol slot by slot: the mean over the valid owner slots of a point
    (a subdomain listed twice counts twice, an unknown one not at all)."""
    cols = prob.d_out + (1 if prob.pde == W.PDE_DIFFUSION2D_INV else 0)
    acc, cnt = np.zeros((len(xy), cols)), np.zeros(len(xy))
    for q, s in enumerate(prob.subdomains):
        one = oracle.eval_stitched(prob, params, xy, np.where(np.arange(4) == 0, q, -1)[None, :].repeat(len(xy), 0))
        times = (owner == q).sum(1)
        acc += times[:, None] * one
        cnt += times
    return np.where(cnt[:, None] > 0, acc / np.maximum(cnt, 1)[:, None], 0.0)


@pytest.mark.parametrize("n", [1, 16, 17, 255, 4097, 140001])
def test_eval_owners_in_any_order(n):
    """Blocks of points of every fill, with the owners mixed point by point:
    repeated, missing and unknown subdomains, every width class, three
    outputs and the network pairs of the inverse problem.  The bound is that
    of the grid evaluations above."""
    mixed = W.custom_box_problem("xpinn", "ns2d_steady", 4, 2,
                                 [[2] + [w] * d + [3] for w, d in zip((5, 16, 20, 40, 64, 80, 90, 112), (1, 2, 3, 4, 2, 3, 2, 3))],
                                 [9] * 8, n_bnd_seg=3, n_iface=3, seed=3, coef=(40.0,))
    W.with_activations(mixed, ("tanh", "sin", "cos"))
    rng = np.random.default_rng(n)
    for prob in (mixed, W.c5_xpinn_inverse_diffusion(seed=1, scale=0.005)):
        params = _params(prob, 17)
        _say(f"eval of {prob.name} at {n} points")
        pb = ddpinn.Problem(prob, fused=True)
        pb.set_params(params)
        xy = rng.uniform(0.0, 1.0, (n, 2)).astype(np.float32)
        owner = rng.integers(-2, prob.n_sd + 2, (n, 4)).astype(np.int32)
        owner[rng.random(n) < 0.5, 1:] = -1
        got = pb.eval(xy, owner).cpu().numpy()
        np.testing.assert_allclose(got, _eval_by_slots(prob, params, xy, owner), rtol=1e-5, atol=1e-6)
        pb.close()


@pytest.mark.parametrize("name,scale", [("c1_cpinn_poisson", 0.2), ("c5_xpinn_inverse_diffusion", 0.01)])
def test_steps_in_one_call_equal_single_steps(name, scale):
    """23 steps in one call (graphs of several steps, then single ones) leave
    the bits of 23 calls of one step, with one train launch and with two."""
    prob = W.make_problem(name, seed=0, scale=scale)
    ends = []
    for calls in ([23], [1] * 23, [9, 14]):
        pb = ddpinn.Problem(prob, fused=True)
        for n in calls:
            lt = pb.step(n).clone()
        st = pb.get_state()
        ends.append((lt.cpu().numpy(), np.concatenate(st["params"]), st["m"], st["v"], st["t"]))
        pb.close()
    for other in ends[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(ends[0], other))


@pytest.mark.parametrize("name,scale", [("c2_xpinn_poisson", 0.05), ("c5_xpinn_inverse_diffusion", 0.01)])
def test_gradients_captured_by_the_caller(name, scale):
    """loss_and_grad inside a caller's graph, with one train launch and with
    two side by side: every replay gives the eager bits, with eager calls in
    between."""
    prob = W.make_problem(name, seed=0, scale=scale)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        pb = ddpinn.Problem(prob, fused=True, stream=stream)
        lt, g = (x.clone() for x in pb.loss_and_grad())
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            clt, cg = pb.loss_and_grad()
        for _ in range(3):
            clt.zero_(), cg.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(clt, lt) and torch.equal(cg, g)
            elt, eg = pb.loss_and_grad()
            assert torch.equal(elt, lt) and torch.equal(eg, g)
    torch.cuda.synchronize()
    pb.close()


def test_parameters_from_any_memory():
    """Device, pageable and pinned host parameters leave the same bits through
    the flat and the per-subdomain call, short ones are refused, and a pointer
    that is not the device's own, or is not a float's address, is copied (or
    refused by the runtime) and never read by a kernel."""
    prob = W.c1_cpinn_poisson(seed=0, scale=0.1)
    params = _params(prob, 3)
    flat = torch.from_numpy(np.concatenate(params))
    total = flat.numel()
    pb = ddpinn.Problem(prob, fused=True)
    zeros = torch.zeros(total, device="cuda")

    def now():
        pb.sync()
        return np.concatenate(pb.get_params())

    pb.set_params([p for p in params])
    lt, g = (x.clone() for x in pb.loss_and_grad())
    for kind, t in (("device", flat.cuda()), ("pageable", flat), ("pinned", flat.pin_memory()),
                    ("double", flat.double()), ("longer", torch.cat([flat, flat]).cuda())):
        _say(f"flat parameters: {kind}")
        pb.set_params_flat(zeros)
        pb.set_params_flat(t)
        assert np.array_equal(now(), flat.numpy()), kind
        lt2, g2 = pb.loss_and_grad()
        assert torch.equal(lt, lt2) and torch.equal(g, g2), kind
    short = flat.cuda()[:total - 1]
    with pytest.raises(ddpinn.DDPError):
        pb.set_params_flat(short)
    with pytest.raises(ddpinn.DDPError):
        pb.set_params([torch.zeros(int(pb.n_params[0]) - 1, device="cuda")])
    assert np.array_equal(now(), flat.numpy())
    # the C entry with on_device = 1
    lib = ddpinn.load_library()
    host = np.ascontiguousarray(params[1], np.float32)
    raw = torch.zeros(4 * len(host) + 4, dtype=torch.uint8, device="cuda")
    raw[2:2 + 4 * len(host)] = torch.from_numpy(host.view(np.uint8)).cuda()
    torch.cuda.synchronize()
    for kind, ptr in (("pageable", host.ctypes.data), ("odd address", raw.data_ptr() + 2)):
        _say(f"on_device = 1 with {kind} memory")
        pb.set_params_flat(zeros)
        rc = lib.ddp_set_params(pb._h, 1, ptr, 1)
        torch.cuda.synchronize()
        got = pb.get_params()[1]
        assert np.array_equal(got, host if rc == ddpinn.DDP_OK else np.zeros_like(host)), (kind, rc)
    pb.close()


def test_parameters_captured_by_the_caller():
    """Device parameters taken inside a caller's graph: every replay takes what
    the buffer then holds."""
    prob = W.c1_cpinn_poisson(seed=0, scale=0.1)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        pb = ddpinn.Problem(prob, fused=True, stream=stream)
        buf = torch.zeros(int(pb.offsets[-1]), device="cuda")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            pb.set_params_flat(buf)
        for r in range(3):
            want = np.concatenate(_params(prob, r))
            buf.copy_(torch.from_numpy(want))
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(np.concatenate(pb.get_params()), want)
    torch.cuda.synchronize()
    pb.close()


def _hidden(widths, k):
    """Offset of hidden matrix W^k in a network's flat parameters, and the width."""
    w = widths[1]
    return 3 * w + (k - 2) * (w * w + w), w


def _extremes():
    """Hidden weights out of the ordinary range: name -> (value, layer, row,
    column) of what is written."""
    inf, nan = np.inf, np.nan
    return {"none": [], "inf in W2": [(inf, 2, 1, 5)], "-inf in W3": [(-inf, 3, 2, 1)],
            "inf and -inf": [(inf, 3, 0, 0), (-inf, 3, 0, 1)], "largest": [(3.4028235e38, 2, 4, 3)],
            "rounds up in bf16": [(-3.397e38, 3, 1, 1)], "1e30": [(1e30, 3, 1, 2)], "nan": [(nan, 2, 1, 1)],
            "1e-36": [(1e-36, 2, 1, 1)]}


def _with_extremes(prob, params, muts):
    out = [p.copy() for p in params]
    for p, s in zip(out, prob.subdomains):
        for v, k, m, j in muts:
            off, w = _hidden(s.widths, k)
            p[off + m * w + j] = v
    return out


@pytest.mark.parametrize("widths", [(5, 16, 20, 32), (33, 48, 60, 64), (70, 80, 90, 112)])
@pytest.mark.parametrize("adaptive", [False, True])
def test_eval_beyond_the_ordinary_range(widths, adaptive):
    """Infinite and very large weights and points at infinity saturate the
    neurons they feed, as in float32 arithmetic, and NaN stays with its point
    or network: the same finite points as the oracle's, and the bound of the
    grid evaluations there; a finite point's bits do not depend on the points
    beside it."""
    prob = W.custom_box_problem("xpinn", "poisson2d", 2, 2, [[2] + [w] * 3 + [1] for w in widths], [9] * 4,
                                n_bnd_seg=3, n_iface=3, seed=sum(widths))
    if adaptive:
        W.with_activations(prob, ("tanh",))
    params = _params(prob, 23)
    rng = np.random.default_rng(7)
    n = 333
    xy = rng.uniform(0.0, 1.0, (n, 2)).astype(np.float32)
    owner = np.full((n, 4), -1, np.int32)
    owner[:, 0] = rng.integers(0, 4, n)
    owner[::5, 1] = (owner[::5, 0] + 1) % 4
    far = xy.copy()
    far[::17, 0] = [np.inf, -np.inf, np.nan, 3e38] * 5
    pb = ddpinn.Problem(prob, fused=True)
    for name, muts in _extremes().items():
        _say(f"eval, widths {widths}, adaptive {adaptive}: {name}")
        q = _with_extremes(prob, params, muts)
        if adaptive and name == "none":
            q[1][-2] = np.inf   # a slope
        pb.set_params(q)
        near, got = (pb.eval(x, owner).cpu().numpy() for x in (xy, far))
        with np.errstate(all="ignore"):
            want = oracle.eval_stitched(prob, q, far, owner)
        assert np.array_equal(np.isfinite(got), np.isfinite(want)), name
        ok = np.isfinite(want)
        np.testing.assert_allclose(got[ok], want[ok], rtol=1e-5, atol=1e-6, err_msg=name)
        same = np.isfinite(far).all(1) & (far[:, 0] == xy[:, 0])
        assert np.array_equal(near[same], got[same], equal_nan=True), name
    pb.close()


@pytest.mark.parametrize("widths", [(20, 32, 60, 16), (80, 100, 48, 112)])
@pytest.mark.parametrize("adaptive", [False, True])
def test_gradients_beyond_the_ordinary_range(widths, adaptive):
    """An infinite, NaN or very large weight in subdomain 0: the loss terms and
    gradient entries that the oracle finds finite are finite (large finite
    weights: the value terms, whose derivatives exceed float32), the terms
    within 1e-5 of it, and the subdomain that shares no interface with it keeps
    its bits."""
    prob = W.custom_box_problem("xpinn", "poisson2d", 2, 2, [[2] + [w] * 3 + [1] for w in widths],
                                [150, 70, 64, 130], n_bnd_seg=9, n_iface=17, seed=sum(widths))
    if adaptive:
        W.with_activations(prob, ("tanh",))
    params = _params(prob, 5)
    pb, lt0, g0 = run(prob, params)
    for name, muts in _extremes().items():
        _say(f"gradients, widths {widths}, adaptive {adaptive}: {name}")
        q = [params[0].copy()] + params[1:]
        q[0] = _with_extremes(prob, params, muts)[0]
        pb.set_params(q)
        lt, g = (x.cpu().numpy() for x in pb.loss_and_grad())
        g = pb.split(g)
        assert np.array_equal(lt[3], lt0[3]) and np.array_equal(g[3], g0[3]), name
        with np.errstate(all="ignore"):
            want, wg = oracle.loss_and_grad(prob, q)
        value_only = any(np.isfinite(m[0]) and abs(m[0]) > 1 for m in muts)
        cols = [1, 3] if value_only else [0, 1, 2, 3, 4]
        ok = np.isfinite(want[:, cols])
        assert np.array_equal(np.isfinite(lt[:, cols]), ok), name
        np.testing.assert_allclose(lt[:, cols][ok], want[:, cols][ok], rtol=1e-5, err_msg=name)
        if not value_only and len(muts) < 2:
            assert all(np.array_equal(np.isfinite(a), np.isfinite(b)) for a, b in zip(g, wg)), name
    pb.close()


@pytest.mark.parametrize("widths", [(20, 32, 60, 16), (80, 100, 48, 112)])
@pytest.mark.parametrize("adaptive", [False, True])
def test_gradients_of_tiny_losses(widths, adaptive):
    """Loss weights of 2^-90 and 2^-100: the gradient scales with them as float32
    does.  An entry is a sum of at most 1e5 terms that may round at 2^-149, the
    spacing of the subnormals, and the norm is above 2^-104, so the difference is
    below 1e5 * 2^-45 < 2^-28 of it."""
    out = []
    for k in (90, 100):
        prob = W.custom_box_problem("xpinn", "poisson2d", 2, 2, [[2] + [w] * 3 + [1] for w in widths],
                                    [150, 70, 64, 130], n_bnd_seg=9, n_iface=17, seed=sum(widths),
                                    loss_w=(2.0 ** -k,) * 4)
        if adaptive:
            W.with_activations(prob, ("tanh",))
        _say(f"widths {widths}, adaptive {adaptive}: loss weights 2^-{k}")
        pb, lt, g = run(prob, _params(prob, 5))
        out.append(np.concatenate(g).astype(np.float64) * 2.0 ** k)
        pb.close()
    assert np.linalg.norm(out[0]) > 2.0 ** -4
    assert np.linalg.norm(out[0] - out[1]) < 2.0 ** -28 * np.linalg.norm(out[0])


@pytest.mark.parametrize("name", ["c5_xpinn_inverse_diffusion", "burgers_st_xpinn_4x4", "ns_cpinn_kovasznay"])
def test_items_run_in_float32_against_oracle(name):
    """Loss weights of 2^-90 send every work item through the float32 run, on
    every operator and kind of item: the gradient against the oracle's, scaled
    by 2^90, within the bars of compare."""
    prob = W.make_problem(name, seed=0, scale=0.02 if name.startswith("c5") else 0.2)
    params = _params(prob, 11)
    ref = oracle.loss_and_grad(prob, params)
    w = [s.loss_w for s in prob.subdomains]
    for s in prob.subdomains:
        s.loss_w = tuple(float(np.float32(v)) * 2.0 ** -90 for v in s.loss_w)
    _say(f"{name}: loss weights times 2^-90")
    pb, lt, g = run(prob, params)
    lt = lt.astype(np.float64)
    lt[:, 0] *= 2.0 ** 90
    for s, v in zip(prob.subdomains, w):
        s.loss_w = v
    compare(prob, params, lt, [x.astype(np.float64) * 2.0 ** 90 for x in g], ref=ref)
    pb.close()


def test_backward_on_another_stream_outlives_the_problem():
    """The index that scales the gradient is kept by the problem and read on the
    stream of the backward pass: once the problem is gone its memory is not
    given out again before that stream has read it."""
    prob = W.c1_cpinn_poisson(seed=0, scale=0.1)
    pb = ddpinn.Problem(prob, fused=True)
    flat = torch.from_numpy(np.concatenate(_params(prob, 3))).cuda().requires_grad_(True)
    ddpinn.DDPLoss.apply(flat, pb).sum().backward()
    index = pb.subdomain_of_param()
    ptr, n, want = index.data_ptr(), index.numel(), flat.grad.clone()
    flat.grad = None
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        loss = ddpinn.DDPLoss.apply(flat, pb).sum()
        torch.cuda.synchronize()
        pb.close()
        torch.cuda._sleep(200_000_000)
        loss.backward()
    del index, loss, pb
    got = [torch.empty(n, dtype=torch.int64, device="cuda") for _ in range(4)]
    assert ptr not in [t.data_ptr() for t in got]
    torch.cuda.synchronize()
    assert torch.equal(flat.grad, want)


def test_long_steps_after_a_new_plan():
    """The graph of several steps belongs to the plan it was made under: after
    autotune the next long call makes its own, and the bits are those of single
    steps under the same plan."""
    prob = W.c1_cpinn_poisson(seed=0, scale=0.1)
    pb = ddpinn.Problem(prob, fused=True)
    pb.step(12)
    at = pb.get_state()
    plan = pb.autotune(iters=1)
    other = ddpinn.Problem(prob, fused=True, **plan)
    other.set_state(at)
    pb.step(25)
    for _ in range(25):
        other.step(1)
    a, b = pb.get_state(), other.get_state()
    assert a["t"] == b["t"] == 37
    assert np.array_equal(np.concatenate(a["params"]), np.concatenate(b["params"]))
    assert np.array_equal(a["m"], b["m"]) and np.array_equal(a["v"], b["v"])
    pb.close()
    other.close()


def _signature_before_revisions(prob, fused):
    """The autotune cache key of libraries that did not hash their revision."""
    h = 1469598103934665603

    def mix(v):
        nonlocal h
        for b in int(v).to_bytes(8, "little", signed=True):
            h = (h ^ b) * 1099511628211 % 2 ** 64

    for v in (ddpinn._PDE[prob.pde], ddpinn._METHOD[prob.method], fused,
              torch.cuda.get_device_properties(0).multi_processor_count, prob.n_sd):
        mix(v)
    for s in prob.subdomains:
        aux = s.aux_widths is not None
        for w in list(s.widths) + (list(s.aux_widths) if aux else []):
            mix(w)
        for v in (ddpinn._ACT[s.act], s.adaptive, len(s.res_xy), len(s.bnd_xy), len(s.aux_xy) if aux else 0):
            mix(v)
    for e in prob.interfaces:
        for v in (e.a, e.b, len(e.xy), ddpinn._METHOD[e.method or prob.method]):
            mix(v)
    return h


def test_autotune_does_not_take_a_plan_found_for_other_kernels(tmp_path):
    """A choice cached by a library with other kernels is searched for again."""
    prob = W.c1_cpinn_poisson(seed=0, scale=0.1)
    cache = tmp_path / "tune.jsonl"
    cache.write_text('{"signature": "%016x", "chunk_points": 4096, "items_per_slot": 3, "blocks_per_cu": 1, '
                     '"recompute": 1, "concurrent": 0, "tail": 7, "ms": 0.1}\n' % _signature_before_revisions(prob, 1))
    pb = ddpinn.Problem(prob, fused=True)
    choice = pb.autotune(iters=1, cache_path=cache)
    assert choice["chunk_points"] != 4096 and choice["tail"] != 7
    lines = cache.read_text().splitlines()
    assert len(lines) == 2
    assert pb.autotune(iters=1, cache_path=cache) == choice and cache.read_text().splitlines() == lines
    pb.close()


def test_a_term_of_tiny_weight_beside_others_keeps_its_bits():
    """Interface terms weighted 2^-100 beside others of weight 1 have tiny seeds,
    but not a tiny loss: their items run as with weight 1, with the same bits of
    every loss term."""
    terms = []
    for w in (1.0, 2.0 ** -100):
        prob = W.custom_box_problem("xpinn", "poisson2d", 2, 2, [[2] + [w_] * 3 + [1] for w_ in (20, 32, 60, 80)],
                                    [150, 70, 64, 130], n_bnd_seg=9, n_iface=17, seed=3, loss_w=(1.0, 1.0, w, w))
        pb, lt, g = run(prob, _params(prob, 5))
        terms.append(lt[:, 1:])
        pb.close()
    assert np.array_equal(terms[0], terms[1])


@pytest.mark.parametrize("name,scale", [("c2_xpinn_poisson", 0.05), ("c5_xpinn_inverse_diffusion", 0.01),
                                        ("c5_table4_adaptive", 0.05)])
def test_float32_items_on_every_path(name, scale):
    """An infinite weight sends items through the float32 run: the static-scratch
    entry (fewer workgroups), side-by-side launches and one after the other, a
    repeat and an Adam step leave the same bits, the per-subdomain path the same
    finite entries; the loss is reported as not finite, and finite parameters
    afterwards give the bits they gave before."""
    prob = W.make_problem(name, seed=0, scale=scale)
    params = _params(prob, 9)
    bad = [p.copy() for p in params]
    off, w = _hidden(prob.subdomains[0].widths, 2)
    bad[0][off + w + 2] = np.inf
    outs = []
    for kw in (dict(concurrent=1), dict(concurrent=0), dict(fused=False)):
        _say(f"{name}: {kw}")
        pb = ddpinn.Problem(prob, **kw)
        pb.set_params(params)
        lt0, g0 = (x.clone() for x in pb.loss_and_grad())
        pb.set_params(bad)
        for entry in (pb.loss_and_grad, pb.loss_and_grad_static, pb.loss_and_grad):
            lt, g = entry()
            outs.append((kw, lt.cpu().numpy(), g.cpu().numpy()))
        with pytest.raises(ddpinn.DDPError) as e:
            pb.sync()
        assert e.value.code == ddpinn.DDP_ENONFINITE
        step = pb.step(1).cpu().numpy()
        assert np.array_equal(step, outs[-1][1], equal_nan=True)
        pb.set_params(params)
        lt, g = pb.loss_and_grad()
        assert torch.equal(lt, lt0) and torch.equal(g, g0)
        pb.close()
    _, lt0, g0 = outs[0]
    assert np.isfinite(g0).any() and not np.isfinite(g0).all()
    for kw, lt, g in outs:
        if kw.get("fused", True):
            assert np.array_equal(lt, lt0, equal_nan=True) and np.array_equal(g, g0, equal_nan=True)
        else:
            assert np.array_equal(np.isfinite(lt), np.isfinite(lt0)) and np.array_equal(np.isfinite(g), np.isfinite(g0))


def _boxes(pde, widths, acts, seed):
    """A 4x2 or 2x1 box problem (the inverse problem: its cells) with the given
    widths, three hidden layers, work items of several tiles with a ragged last
    one, and interfaces between all of them."""
    if pde == "inverse":
        prob = W.c5_xpinn_inverse_diffusion(seed=3, scale=0.006)
        rng = np.random.default_rng(seed)
        for q, s in enumerate(prob.subdomains):
            s.widths = [2] + [widths[q % len(widths)]] * 3 + [1]
            s.aux_widths = [2] + [widths[(q + 3) % len(widths)]] * 2 + [1]
            s.params = np.concatenate([W.glorot_params(rng, s.widths), W.glorot_params(rng, s.aux_widths)])
    else:
        out, coef = (3, (40.0,)) if pde == "ns2d_steady" else (1, (0.05,) if pde == "burgers1d" else ())
        nx, ny = (4, 2) if len(widths) > 1 else (2, 1)
        n = nx * ny
        prob = W.custom_box_problem("cpinn" if seed % 2 else "xpinn", pde, nx, ny,
                                    [[2] + [widths[q % len(widths)]] * 3 + [out] for q in range(n)],
                                    [130 + 7 * q for q in range(n)], n_bnd_seg=9, n_iface=17, seed=seed, coef=coef)
    return W.with_activations(prob, acts) if acts else prob


@pytest.mark.parametrize("pde", ["poisson2d", "burgers1d", "ns2d_steady", "inverse"])
@pytest.mark.parametrize("acts", [None, ("tanh", "sin", "tanh", "cos")])
def test_every_kernel_and_class_against_oracle(pde, acts):
    """Every train kernel with every width class it holds: one width at a time
    (the kernel of that class), all widths at once (the groups up to 80 and up to
    112), and the per-subdomain path (the widest kernel for all).  The compiler
    holds values of the wide classes in accumulation registers or memory, and
    has saved some under a partial mask of lanes, which gives errors of order
    one: each kernel is checked by itself, at ten times the bar of the other
    tests."""
    for widths in [(w,) for w in (16, 32, 48, 64, 80, 96, 112)] + [(16, 112, 32, 96, 48, 80, 64, 20)]:
        for seed in (1, 2):
            prob = _boxes(pde, widths, acts, seed)
            params = _params(prob, 13)
            ref = oracle.loss_and_grad(prob, params)
            for fused in (True, False) if len(widths) > 1 else (True,):
                _say(f"{pde} {acts} widths {widths} seed {seed} fused {fused}")
                pb, lt, g = run(prob, params, fused=fused, items_per_slot=1, chunk_points=4096)
                compare(prob, params, lt, g, ref=ref, loss_rtol=1e-4, grad_rtol=1e-4)
                pb.close()
            if pde == "inverse":
                break
