"""GPU parity of the Sim3 residual, its hand-written backward, the Sim3
exponential, the Gauss-Newton step, the autograd Function and per-event
refinement against the float64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle import residual as R
from oracle import sim3
from gpu_util import dev, t

pytestmark = pytest.mark.gpu

REL = 1e-4   # relative error bound (infinity norm) of float32 per-pair terms vs float64


@pytest.fixture(scope="module")
def ctx():
    import paper_2603_17201_amd as fl
    c = fl.Context(0)
    yield c
    c.close()


def rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-300)


def s32(S):
    return t(sim3.to_f32_rows(S))


def multi_view(n, seed):
    rng = np.random.default_rng(seed)
    d = synth.gen_c4(n=n, seed=seed, pix_sigma=0.0, outlier_frac=0.0)
    T = np.array([sim3.exp(np.concatenate([rng.normal(size=3) * 0.1, rng.normal(size=3) * 0.5, [0.0]]))[:12]
                  for _ in range(5)])
    kf = rng.integers(0, 5, n).astype(np.int32)
    _, q, uv, _ = R.project(d["S_true"], d["xyz"], kf, T, d["cam"])
    uv = uv + rng.normal(0, 1.0, uv.shape)
    out = rng.random(n) < 0.1
    th = rng.uniform(0, 2 * np.pi, n)
    uv[out] += 20 * np.stack([np.cos(th[out]), np.sin(th[out])], 1)
    keep = q[:, 2] > 0.1
    return d, d["xyz"][keep], uv[keep].astype(np.float32), kf[keep], T


@pytest.fixture(scope="module")
def c4():
    d = synth.gen_c4()
    d["S0"] = sim3.compose(sim3.exp(d["xi0"]), d["S_true"])
    return d


def test_forward_matches_fp64(ctx, c4):
    S0 = c4["S0"]
    r, w, loss = ctx.residual_fwd(t(c4["xyz"]), t(c4["uv"]), None, None, s32(S0), c4["cam"], c4["huber_delta"])
    r64, w64, L64 = R.forward(sim3.from_matrix(sim3.to_matrix(S0)), c4["xyz"], c4["uv"], None, None, c4["cam"],
                              c4["huber_delta"])
    assert rel(r.cpu().numpy(), r64) < REL
    assert rel(w.cpu().numpy(), w64) < REL
    assert abs(loss.item() - L64) / L64 < REL


def test_backward_matches_fp64_and_fd(ctx, c4):
    S0 = c4["S0"]
    g, H = ctx.residual_bwd(t(c4["xyz"]), t(c4["uv"]), None, None, s32(S0), c4["cam"], c4["huber_delta"])
    g64, H64, _ = R.grad_hess(S0, c4["xyz"], c4["uv"], None, None, c4["cam"], c4["huber_delta"])
    assert rel(g.cpu().numpy(), g64) < REL
    assert rel(H.cpu().numpy(), R.H_upper(H64)) < REL
    fd = R.fd_grad(S0, c4["xyz"], c4["uv"], None, None, c4["cam"], c4["huber_delta"], h=1e-4)
    assert rel(g.cpu().numpy(), fd) < 2 * REL
    # deterministic: same bits on a second call
    g2, H2 = ctx.residual_bwd(t(c4["xyz"]), t(c4["uv"]), None, None, s32(S0), c4["cam"], c4["huber_delta"])
    assert torch.equal(g, g2) and torch.equal(H, H2)


def test_backward_with_keyframe_poses(ctx):
    d, xyz, uv, kf, T = multi_view(30000, 5)
    S0 = sim3.compose(sim3.exp(d["xi0"]), d["S_true"])
    g, H = ctx.residual_bwd(t(xyz), t(uv), t(kf), t(T.astype(np.float32)), s32(S0), d["cam"], 2.45)
    g64, H64, _ = R.grad_hess(S0, xyz, uv, kf, T, d["cam"], 2.45)
    assert rel(g.cpu().numpy(), g64) < REL
    assert rel(H.cpu().numpy(), R.H_upper(H64)) < REL


def test_sim3_exp_mul_matches_expm(ctx):
    rng = np.random.default_rng(2)
    for scale in (1e-7, 1e-3, 0.05, 0.5, 2.0):
        xi = rng.normal(size=7) * scale
        S_in = sim3.exp(rng.normal(size=7) * 0.3)
        S_out, S32 = ctx.sim3_exp_mul(t(xi), t(S_in))
        exp = sim3.compose(sim3.exp(xi), S_in)
        assert np.max(np.abs(S_out.cpu().numpy() - exp)) < 1e-12 * max(1.0, np.max(np.abs(exp))), scale
        assert np.max(np.abs(S32.cpu().numpy() - sim3.to_f32_rows(exp))) < 1e-6


def test_sim3_exp_series_branches(ctx):
    # sigma on both sides of each switch between series lengths (2.5e-4, 4e-3,
    # 1e-2) and of the switch to the summed series, of both signs; rotation
    # angles on both sides of the small-angle switch (1e-2)
    rng = np.random.default_rng(9)
    S_in = sim3.exp(rng.normal(size=7) * 0.3)
    for sig in (0.0, 1e-9, 2.4e-4, -2.4e-4, 2.6e-4, 3.9e-3, -3.9e-3, 4.1e-3, 9.9e-3, -9.9e-3, 1.01e-2, -1.01e-2):
        for th in (0.0, 3e-5, 9.9e-3, 1.01e-2):
            w = rng.normal(size=3)
            w *= th / np.linalg.norm(w)
            xi = np.concatenate([w, rng.normal(size=3) * 0.05, [sig]])
            S_out, _ = ctx.sim3_exp_mul(t(xi), t(S_in))
            exp = sim3.compose(sim3.exp(xi), S_in)
            assert np.max(np.abs(S_out.cpu().numpy() - exp)) < 1e-12 * max(1.0, np.max(np.abs(exp))), (sig, th)


def test_gn_step_matches_oracle(ctx, c4):
    d, xyz, uv, kf, T = multi_view(20000, 8)
    S0 = sim3.compose(sim3.exp(d["xi0"]), d["S_true"])
    g64, H64, _ = R.grad_hess(S0, xyz, uv, kf, T, d["cam"], 2.45)
    S = t(S0.copy())
    S32 = torch.empty(16, dtype=torch.float32, device=dev())
    ctx.gn_step(t(g64), t(R.H_upper(H64)), S, S32)
    exp = sim3.compose(sim3.exp(np.linalg.solve(H64, -g64)), S0)
    assert np.max(np.abs(S.cpu().numpy() - exp)) < 1e-9


def test_autograd_function(ctx, c4):
    import paper_2603_17201_amd as fl
    S0 = t(c4["S0"])
    xi = torch.zeros(7, dtype=torch.float64, device=dev(), requires_grad=True)
    loss = fl.Sim3Residual.apply(xi, S0, t(c4["xyz"]), t(c4["uv"]), None, None, c4["cam"], c4["huber_delta"], ctx)
    (2.0 * loss).backward()
    g64, _, L64 = R.grad_hess(c4["S0"], c4["xyz"], c4["uv"], None, None, c4["cam"], c4["huber_delta"])
    assert abs(loss.item() - L64) / L64 < REL
    assert rel(xi.grad.cpu().numpy(), 2.0 * g64) < REL
    # central differences of the Function itself around xi = 0
    h = 1e-4
    fd = np.zeros(7)
    for i in range(7):
        e = torch.zeros(7, dtype=torch.float64, device=dev())
        e[i] = h
        lp = fl.Sim3Residual.apply(e, S0, t(c4["xyz"]), t(c4["uv"]), None, None, c4["cam"], c4["huber_delta"], ctx)
        lm = fl.Sim3Residual.apply(-e, S0, t(c4["xyz"]), t(c4["uv"]), None, None, c4["cam"], c4["huber_delta"], ctx)
        fd[i] = (lp.item() - lm.item()) / (2 * h)
    # float32 losses limit the difference quotient: compare on the dominant components
    big = np.abs(g64) > 1e-3 * np.max(np.abs(g64))
    assert np.max(np.abs(fd[big] - g64[big])) / np.max(np.abs(g64)) < 1e-3


def test_sim3_grad_xi_matches_numerical_left_jacobian(ctx):
    # J_l(xi) column i is d/dh log(exp(xi + h e_i) exp(xi)^-1) at h = 0
    # (central differences of scipy's expm / logm in float64); the kernel
    # returns scale * J_l^T g.
    rng = np.random.default_rng(21)
    for scale in (1e-6, 0.05, 0.3, 1.0):
        xi = rng.normal(size=7) * scale
        h = 1e-6
        J = np.zeros((7, 7))
        for i in range(7):
            e = np.zeros(7)
            e[i] = h
            Sp = sim3.compose(sim3.exp(xi + e), sim3.inverse(sim3.exp(xi)))
            Sm = sim3.compose(sim3.exp(xi - e), sim3.inverse(sim3.exp(xi)))
            J[:, i] = (sim3.log(Sp) - sim3.log(Sm)) / (2 * h)
        g = rng.normal(size=7)
        out = ctx.sim3_grad_xi(t(xi), t(g), t(np.array([2.5]))).cpu().numpy()
        assert rel(out, 2.5 * J.T @ g) < 1e-7, scale
        out1 = ctx.sim3_grad_xi(t(xi), t(g)).cpu().numpy()
        assert rel(out1, J.T @ g) < 1e-7, scale


def test_autograd_function_away_from_zero(ctx, c4):
    # At xi = 0.05 on every component the Function's gradient is dL/dxi of
    # L(exp(xi) S0): compared with float64 central differences of the
    # oracle's loss at the same xi.
    import paper_2603_17201_amd as fl
    S0 = t(c4["S0"])
    xi1 = np.full(7, 0.05)
    xi = torch.tensor(xi1, dtype=torch.float64, device=dev(), requires_grad=True)
    loss = fl.Sim3Residual.apply(xi, S0, t(c4["xyz"]), t(c4["uv"]), None, None, c4["cam"], c4["huber_delta"], ctx)
    (3.0 * loss).backward()
    h = 1e-5
    fd = np.zeros(7)
    for i in range(7):
        e = np.zeros(7)
        e[i] = h
        fd[i] = (R.loss_at(xi1 + e, c4["S0"], c4["xyz"], c4["uv"], None, None, c4["cam"], c4["huber_delta"])
                 - R.loss_at(xi1 - e, c4["S0"], c4["xyz"], c4["uv"], None, None, c4["cam"], c4["huber_delta"])) / (2 * h)
    L64 = R.loss_at(xi1, c4["S0"], c4["xyz"], c4["uv"], None, None, c4["cam"], c4["huber_delta"])
    assert abs(loss.item() - L64) / L64 < REL
    assert rel(xi.grad.cpu().numpy(), 3.0 * fd) < REL
    # the left-perturbation gradient alone is not dL/dxi here
    g_left, _, _ = R.grad_hess(sim3.compose(sim3.exp(xi1), c4["S0"]), c4["xyz"], c4["uv"], None, None, c4["cam"],
                               c4["huber_delta"])
    assert rel(g_left, fd) > 10 * REL


def test_refine_events_matches_oracle_gn(ctx):
    import paper_2603_17201_amd as fl
    ev = synth.gen_c2()
    out = oracle.search_fuse(ev, use_grid=True)
    b = fl.DeviceBatch(ev, device=dev())
    res = ctx.search_fuse_graph(b, ev.params)
    got = res.numpy()
    for k in got:
        assert np.array_equal(got[k], out[k]), k
    # oracle GN on the accepted pairs
    acc = np.nonzero((out["decision"] == oracle.ADD) | (out["decision"] == oracle.FUSE))[0]
    kf = (np.searchsorted(ev.pair_offset, acc, side="right") - 1).astype(np.int32)
    mp = acc - ev.pair_offset[kf]
    kp = ev.kp_offset[kf] + out["best_idx"][acc]
    xyz, uv = ev.mp_xyz[mp], ev.kp_xy[kp]
    T32 = ev.kf_T.astype(np.float32).astype(np.float64)   # the keyframe poses the GPU sees
    S_ref = R.gauss_newton(ev.S_init, xyz, uv, kf, T32, ev.cams[0], 2.45, iters=10)
    finals = {}
    for mode in ("scan", "graph", "batched"):
        event_S = t(ev.S_init.reshape(1, 13).copy())
        nm = torch.zeros(1, dtype=torch.int32, device=dev())
        ref = (10, 2.45, event_S, None, nm)
        if mode == "graph":
            ctx.search_fuse_graph(b, ev.params, refine=ref)
        elif mode == "batched":
            got2 = ctx.search_fuse_batched(b, ev.params, refine=ref).numpy()
            for k in got2:
                assert np.array_equal(got2[k], out[k]), k
        else:
            ctx.refine_events(b, res, ref)
        S_gpu = event_S.cpu().numpy()[0]
        finals[mode] = S_gpu
        assert nm.item() == len(acc)
        err = np.linalg.norm(sim3.log(sim3.compose(S_gpu, sim3.inverse(S_ref))))
        assert err < 1e-6, (mode, err)
        # and the refinement moved toward the truth
        e_true = np.linalg.norm(sim3.log(sim3.compose(S_gpu, sim3.inverse(ev.S_true))))
        e_init = np.linalg.norm(sim3.log(sim3.compose(ev.S_init, sim3.inverse(ev.S_true))))
        assert e_true < e_init
    # the list-driven refinements see the same pairs (their order follows the
    # order in which tiles finish, so the float64 sums may differ in rounding)
    d = np.linalg.norm(sim3.log(sim3.compose(finals["graph"], sim3.inverse(finals["batched"]))))
    assert d < 1e-9, d


def test_zero_pairs(ctx):
    z3 = torch.zeros((0, 3), dtype=torch.float32, device=dev())
    z2 = torch.zeros((0, 2), dtype=torch.float32, device=dev())
    S = s32(sim3.identity())
    _, _, loss = ctx.residual_fwd(z3, z2, None, None, S, synth.scenes._cam_row(synth.CAM_752), 2.45)
    g, H = ctx.residual_bwd(z3, z2, None, None, S, synth.scenes._cam_row(synth.CAM_752), 2.45)
    assert loss.item() == 0.0 and torch.all(g == 0) and torch.all(H == 0)


def _event_gn(B, out, e, iters=10):
    """Float64 Gauss-Newton of event e of batch B on the pairs the oracle
    accepted, with the keyframe poses the device sees (float32)."""
    ekf, emp = B.event_kf_offset, B.event_mp_offset
    xyz, uv, kfl = [], [], []
    for k in range(int(ekf[e]), int(ekf[e + 1])):
        p0, p1 = int(B.pair_offset[k]), int(B.pair_offset[k + 1])
        d = out["decision"][p0:p1]
        acc = np.nonzero((d == oracle.ADD) | (d == oracle.FUSE))[0]
        local = B.pair_mp[p0 + acc] if B.pair_mp is not None else acc
        xyz.append(B.mp_xyz[int(emp[e]) + np.asarray(local, np.int64)])
        uv.append(B.kp_xy[int(B.kp_offset[k]) + out["best_idx"][p0 + acc]])
        kfl.append(np.full(len(acc), k - int(ekf[e]), np.int32))
    xyz, uv, kfl = np.concatenate(xyz), np.concatenate(uv), np.concatenate(kfl)
    if len(xyz) == 0:
        return None, 0
    T32 = B.kf_T[int(ekf[e]):int(ekf[e + 1])].astype(np.float32).astype(np.float64)
    S = R.gauss_newton(B.events[e].S_init, xyz, uv, kfl, T32, B.cams[int(ekf[e])], 2.45, iters=iters)
    return S, len(xyz)


def test_refine_multi_event_batch(ctx):
    """Several uneven events in one launch (the refinement grid split among
    them), one of which accepts no pair, in both launch modes."""
    import paper_2603_17201_amd as fl
    e0 = synth.gen_c3(seed=321, n_kf=10, n_mp=5000, id_base=1000, fresh_base=10 ** 9)
    e1 = synth.gen_tiny(62, n_kf=3, n_mp=400)
    e2 = synth.gen_c2(seed=207, n_kf=5, n_mp=3000)
    e3 = synth.gen_tiny(63, n_kf=2, n_mp=150)
    e3.kp_desc = e3.kp_desc ^ np.uint8(0xFF)   # every distance far above the threshold
    B = synth.concat_events([e0, e1, e2, e3])
    exp = oracle.search_fuse(B, use_grid=True)
    refs = [_event_gn(B, exp, e) for e in range(4)]
    assert refs[3][1] == 0 and all(n > 100 for _, n in refs[:3])
    b = fl.DeviceBatch(B, device=dev())
    S0 = np.stack([ev.S_init for ev in B.events])
    for mode in ("batched", "graph"):
        S = t(S0.copy())
        nm = torch.zeros(4, dtype=torch.int32, device=dev())
        ref = (10, 2.45, S, None, nm)
        res = (ctx.search_fuse_batched(b, B.params, refine=ref) if mode == "batched"
               else ctx.search_fuse_graph(b, B.params, refine=ref))
        got = res.numpy()
        for k in got:
            assert np.array_equal(got[k], exp[k]), (mode, k)
        S_gpu, n_gpu = S.cpu().numpy(), nm.cpu().numpy()
        for e, (S_ref, n_ref) in enumerate(refs):
            assert n_gpu[e] == n_ref, (mode, e)
            if S_ref is None:   # no pair: the system is singular and the Sim3 is left as it was
                assert np.array_equal(S_gpu[e], S0[e]), (mode, e)
                continue
            err = np.linalg.norm(sim3.log(sim3.compose(S_gpu[e], sim3.inverse(S_ref))))
            assert err < 1e-6, (mode, e, err)


def test_stream_largest_event_graph_with_refine(ctx):
    """The largest event of the 200-event stream (73 keyframes, 97,969 points,
    7.15 M dense pairs) in the stream's launch configuration (graph replay
    with ten refinement steps): every output bit-exact against the oracle and
    the refined Sim3 against float64 Gauss-Newton on the same pairs."""
    import paper_2603_17201_amd as fl
    ev = synth.gen_c5_event(59)
    B = synth.concat_events([ev])
    assert int(B.pair_offset[-1]) == 73 * 97969
    exp = oracle.search_fuse(B, use_grid=True)
    S_ref, n_ref = _event_gn(B, exp, 0)
    assert n_ref > 50000
    b = fl.DeviceBatch(B, device=dev())
    try:
        for tuning in ((2, 2, 1, 1), (1, 2, 2, 1)):
            ctx.set_tuning(*tuning)
            S = t(ev.S_init.reshape(1, 13).copy())
            nm = torch.zeros(1, dtype=torch.int32, device=dev())
            got = ctx.search_fuse_graph(b, B.params, refine=(10, 2.45, S, None, nm)).numpy()
            for k in got:
                assert np.array_equal(got[k], exp[k]), (tuning, k)
            assert int(nm.item()) == n_ref, tuning
            err = np.linalg.norm(sim3.log(sim3.compose(S.cpu().numpy()[0], sim3.inverse(S_ref))))
            assert err < 1e-6, (tuning, err)
    finally:
        ctx.set_tuning()


def test_ten_uneven_events_one_launch(ctx):
    """Ten uneven 60-keyframe events (4.68 M sparse pairs) in one graph launch
    with ten refinement steps each, as the benchmark times them: every
    search output bit-exact, every event's Sim3 within 1e-6 of float64
    Gauss-Newton on the oracle's accepted pairs."""
    import paper_2603_17201_amd as fl
    evs = [synth.gen_c3(seed=303 + i, id_base=1000 + 10 ** 6 * i, fresh_base=10 ** 9 + 10 ** 7 * i)
           for i in range(10)]
    B = synth.concat_events(evs)
    assert int(B.pair_offset[-1]) == 4675858
    exp = oracle.search_fuse(B, use_grid=True)
    refs = [_event_gn(B, exp, e) for e in range(10)]
    b = fl.DeviceBatch(B, device=dev())
    S0 = np.stack([ev.S_init for ev in evs])
    S = t(S0.copy())
    nm = torch.zeros(10, dtype=torch.int32, device=dev())
    got = ctx.search_fuse_graph(b, B.params, refine=(10, 2.45, S, None, nm)).numpy()
    for k in got:
        assert np.array_equal(got[k], exp[k]), k
    S_gpu, n_gpu = S.cpu().numpy(), nm.cpu().numpy()
    for e, (S_ref, n_ref) in enumerate(refs):
        assert n_gpu[e] == n_ref, e
        err = np.linalg.norm(sim3.log(sim3.compose(S_gpu[e], sim3.inverse(S_ref))))
        assert err < 1e-6, (e, err)


def test_two_contexts_on_two_streams(ctx):
    """Consecutive events alternating between two contexts on two streams
    (one event's search overlapping the previous one's refinement), graph
    launches with ten refinement steps: every event's outputs bit-exact and
    its Sim3 within 1e-6 of float64 Gauss-Newton."""
    import paper_2603_17201_amd as fl
    evs = [synth.gen_c3(seed=330 + i, n_kf=10 + 2 * i, n_mp=6000 + 500 * i, id_base=1000 + 10 ** 6 * i,
                        fresh_base=10 ** 9 + 10 ** 7 * i) for i in range(6)]
    Bs = [synth.concat_events([ev]) for ev in evs]
    exps = [oracle.search_fuse(B, use_grid=True) for B in Bs]
    refs = [_event_gn(B, exp, 0) for B, exp in zip(Bs, exps)]
    ctx2 = fl.Context(0)
    try:
        ctxs = [ctx, ctx2]
        streams = [torch.cuda.current_stream(), torch.cuda.Stream()]
        bs = [fl.DeviceBatch(B, device=dev()) for B in Bs]
        outs = [fl.FuseOutputs.empty(b.n_pairs, dev()) for b in bs]
        S = [t(ev.S_init.reshape(1, 13).copy()) for ev in evs]
        nm = torch.zeros(len(evs), dtype=torch.int32, device=dev())
        torch.cuda.synchronize()
        for rep in range(2):
            for i in range(len(evs)):
                k = i % 2
                ctxs[k].search_fuse_graph(bs[i], Bs[i].params, outs[i], refine=(10, 2.45, S[i], None, nm[i:i + 1]),
                                          stream=streams[k])
            torch.cuda.synchronize()
            for i, (exp, (S_ref, n_ref)) in enumerate(zip(exps, refs)):
                got = outs[i].numpy()
                for key in got:
                    assert np.array_equal(got[key], exp[key]), (rep, i, key)
                assert int(nm[i].item()) == n_ref, (rep, i)
                if rep == 0:
                    err = np.linalg.norm(sim3.log(sim3.compose(S[i].cpu().numpy()[0], sim3.inverse(S_ref))))
                    assert err < 1e-6, (i, err)
                S[i].copy_(t(evs[i].S_init.reshape(1, 13).copy()))
    finally:
        ctx2.close()


def _accepted(ev, out):
    acc = np.nonzero((out["decision"] == oracle.ADD) | (out["decision"] == oracle.FUSE))[0]
    kf = (np.searchsorted(ev.pair_offset, acc, side="right") - 1).astype(np.int32)
    mp = acc - ev.pair_offset[kf]
    kp = ev.kp_offset[kf] + out["best_idx"][acc]
    return ev.mp_xyz[mp], ev.kp_xy[kp], kf


@pytest.mark.parametrize("lm", [0.0, synth.ROBUST_LM_LAMBDA])
def test_robust_refinement_matches_oracle(ctx, lm):
    """The verification search on an event with 10% wrong associations, then
    two rounds of five evaluations, the second on the pairs within 3.035 px:
    Gauss-Newton and Levenberg-Marquardt, through the scan path, the graph
    and the eager batched call, against the float64 oracle."""
    import paper_2603_17201_amd as fl
    ev = synth.gen_c2_misplaced()
    P = synth.verification_params()
    out = oracle.search_fuse(ev, params=P, use_grid=True)
    xyz, uv, kf = _accepted(ev, out)
    T32 = ev.kf_T.astype(np.float32).astype(np.float64)
    it, rounds, tau = synth.ROBUST_ITERS, synth.ROBUST_ROUNDS, synth.ROBUST_OUTLIER_PX
    # the device takes the Huber threshold and the inlier bound as float32
    d32, tau32 = float(np.float32(2.45)), float(np.float32(tau))
    S_ref, n_ref = R.refine_robust(ev.S_init, xyz, uv, kf, T32, ev.cams[0], d32, iters=it, rounds=rounds,
                                   outlier_px=tau32, lm_lambda=lm)
    assert n_ref < len(xyz) - 1000   # the wrong associations are dropped
    b = fl.DeviceBatch(ev, device=dev())
    res = ctx.search_fuse_batched(b, P)
    for mode in ("scan", "graph", "batched"):
        event_S = t(ev.S_init.reshape(1, 13).copy())
        nm = torch.zeros(1, dtype=torch.int32, device=dev())
        ref = (it, 2.45, event_S, None, nm, rounds, tau, lm)
        if mode == "graph":
            ctx.search_fuse_graph(b, P, refine=ref)
        elif mode == "batched":
            got = ctx.search_fuse_batched(b, P, refine=ref).numpy()
            for k in got:
                assert np.array_equal(got[k], out[k]), k
        else:
            ctx.refine_events(b, res, ref)
        S_gpu = event_S.cpu().numpy()[0]
        err = np.linalg.norm(sim3.log(sim3.compose(S_gpu, sim3.inverse(S_ref))))
        assert err < 1e-6, (mode, lm, err)
        assert nm.item() == n_ref, (mode, lm, nm.item(), n_ref)


def test_robust_refinement_rejects_bad_arguments(ctx):
    import paper_2603_17201_amd as fl
    ev = synth.gen_c1()
    b = fl.DeviceBatch(ev, device=dev())
    S = t(ev.S_init.reshape(1, 13).copy())
    for ref in [(5, 2.45, S, None, None, 2, 0.0, 0.0),       # no inlier bound
                (5, 2.45, S, None, None, 2, 3.0, -1.0),      # negative damping
                (500, 2.45, S, None, None, 3, 3.0, 0.0),     # more than 1000 evaluations
                (5, 2.45, S, None, None, -1, 3.0, 0.0)]:
        with pytest.raises(fl.FlError):
            ctx.search_fuse_batched(b, ev.params, refine=ref)


@pytest.fixture(scope="module")
def bidir():
    return synth.gen_bidir()


def test_sim3_inverse_matches_oracle(ctx, bidir):
    for S in (bidir["S0"], bidir["S_true"], sim3.exp(np.array([0.3, -0.2, 0.1, 1.0, -2.0, 0.5, 0.4]))):
        S_inv, S32 = ctx.sim3_inverse(t(S))
        exp = sim3.inverse(S)
        assert np.max(np.abs(S_inv.cpu().numpy() - exp)) < 1e-14 * max(1.0, np.max(np.abs(exp)))
        assert np.max(np.abs(S32.cpu().numpy() - sim3.to_f32_rows(exp))) < 1e-6


def test_inverse_direction_matches_fp64(ctx, bidir):
    """Points of the current side observed on the loop side through S^-1:
    residuals, weights and loss from the forward call given S^-1's float32
    form; g and H with respect to S from the inverse backward, against the
    float64 oracle."""
    xyz, uv, kf, T = bidir["bwd"]
    S0, cam = bidir["S0"], bidir["cam"]
    _, S32_inv = ctx.sim3_inverse(t(S0))
    r, w, loss = ctx.residual_fwd(t(xyz), t(uv), t(kf), t(T), S32_inv, cam, 2.45)
    r64, w64, L64 = R.forward_inv(S0, xyz, uv, kf, T.astype(np.float64), cam, 2.45)
    assert rel(r.cpu().numpy(), r64) < REL
    assert rel(w.cpu().numpy(), w64) < REL
    assert abs(loss.item() - L64) / L64 < REL
    g, H = ctx.residual_bwd(t(xyz), t(uv), t(kf), t(T), S32_inv, cam, 2.45, inverse=True)
    g64, H64, _ = R.grad_hess_inv(S0, xyz, uv, kf, T.astype(np.float64), cam, 2.45)
    assert rel(g.cpu().numpy(), g64) < REL
    assert rel(H.cpu().numpy(), R.H_upper(H64)) < REL


def test_two_sided_gauss_newton_matches_oracle(ctx, bidir):
    """Ten Gauss-Newton steps on both directions through the C ABI: two
    backward calls, their sums added, one step, the inverse refreshed."""
    fwd, bwd, cam = bidir["fwd"], bidir["bwd"], bidir["cam"]
    S = t(bidir["S0"].copy())
    S32 = torch.empty(16, dtype=torch.float32, device=dev())
    S32_inv = torch.empty(16, dtype=torch.float32, device=dev())
    ctx.sim3_exp_mul(t(np.zeros(7)), S.clone(), S, S32)
    Xf, Uf, Kf, Tf = (t(a) for a in fwd)
    Xb, Ub, Kb, Tb = (t(a) for a in bwd)
    for _ in range(10):
        ctx.sim3_inverse(S, None, S32_inv)
        g1, H1 = ctx.residual_bwd(Xf, Uf, Kf, Tf, S32, cam, 2.45)
        g2, H2 = ctx.residual_bwd(Xb, Ub, Kb, Tb, S32_inv, cam, 2.45, inverse=True)
        ctx.gn_step(g1 + g2, H1 + H2, S, S32)
    f64 = fwd[:3] + (fwd[3].astype(np.float64),)
    b64 = bwd[:3] + (bwd[3].astype(np.float64),)
    S_ref = R.gauss_newton_bidir(bidir["S0"], f64, b64, cam, 2.45, iters=10)
    S_gpu = S.cpu().numpy()
    err = np.linalg.norm(sim3.log(sim3.compose(S_gpu, sim3.inverse(S_ref))))
    assert err < 1e-6, err
    e_true = np.linalg.norm(sim3.log(sim3.compose(S_gpu, sim3.inverse(bidir["S_true"]))))
    e_init = np.linalg.norm(sim3.log(sim3.compose(bidir["S0"], sim3.inverse(bidir["S_true"]))))
    assert e_true < 0.1 * e_init


def _event_pairs(B, out, e):
    """The accepted pairs of event e of batch B (points, observations, local
    keyframe index) and the event's keyframe poses as the device sees them."""
    ekf, emp = B.event_kf_offset, B.event_mp_offset
    xyz, uv, kfl = [], [], []
    for k in range(int(ekf[e]), int(ekf[e + 1])):
        p0, p1 = int(B.pair_offset[k]), int(B.pair_offset[k + 1])
        d = out["decision"][p0:p1]
        acc = np.nonzero((d == oracle.ADD) | (d == oracle.FUSE))[0]
        local = B.pair_mp[p0 + acc] if B.pair_mp is not None else acc
        xyz.append(B.mp_xyz[int(emp[e]) + np.asarray(local, np.int64)])
        uv.append(B.kp_xy[int(B.kp_offset[k]) + out["best_idx"][p0 + acc]])
        kfl.append(np.full(len(acc), k - int(ekf[e]), np.int32))
    T32 = B.kf_T[int(ekf[e]):int(ekf[e + 1])].astype(np.float32).astype(np.float64)
    return np.concatenate(xyz), np.concatenate(uv), np.concatenate(kfl), T32


@pytest.mark.parametrize("lm", [0.0, synth.ROBUST_LM_LAMBDA])
def test_robust_refinement_multi_event_batch(ctx, lm):
    """Rounds with an inlier bound (and Levenberg-Marquardt) on four events
    in one launch: two with wrong associations, one uneven with sparse
    pairs, one that accepts no pair.  The events leave their rounds at
    different steps; each must match its own float64 refinement."""
    import paper_2603_17201_amd as fl
    e0 = synth.gen_c2(seed=231, n_kf=5, n_mp=4000, misplace=(0.1, 6.0, 9.0))
    e1 = synth.gen_c3(seed=322, n_kf=8, n_mp=4000, id_base=10 ** 6, fresh_base=2 * 10 ** 9)
    e2 = synth.gen_c2(seed=232, n_kf=4, n_mp=3000, misplace=(0.15, 6.0, 9.0))
    e3 = synth.gen_tiny(64, n_kf=2, n_mp=150)
    e3.kp_desc = e3.kp_desc ^ np.uint8(0xFF)   # no candidate within the threshold
    B = synth.concat_events([e0, e1, e2, e3])
    P = synth.verification_params()
    exp = oracle.search_fuse(B, params=P, use_grid=True)
    it, rounds, tau = synth.ROBUST_ITERS, synth.ROBUST_ROUNDS, synth.ROBUST_OUTLIER_PX
    d32, tau32 = float(np.float32(2.45)), float(np.float32(tau))
    refs = []
    for e in range(3):
        xyz, uv, kfl, T32 = _event_pairs(B, exp, e)
        refs.append(R.refine_robust(B.events[e].S_init, xyz, uv, kfl, T32, B.cams[int(B.event_kf_offset[e])], d32,
                                    iters=it, rounds=rounds, outlier_px=tau32, lm_lambda=lm))
    assert all(n > 100 for _, n in refs)
    b = fl.DeviceBatch(B, device=dev())
    S0 = np.stack([ev.S_init for ev in B.events])
    for mode in ("batched", "graph"):
        S = t(S0.copy())
        nm = torch.zeros(4, dtype=torch.int32, device=dev())
        ref = (it, 2.45, S, None, nm, rounds, tau, lm)
        res = (ctx.search_fuse_batched(b, P, refine=ref) if mode == "batched"
               else ctx.search_fuse_graph(b, P, refine=ref))
        got = res.numpy()
        for k in got:
            assert np.array_equal(got[k], exp[k]), (mode, k)
        S_gpu, n_gpu = S.cpu().numpy(), nm.cpu().numpy()
        for e, (S_ref, n_ref) in enumerate(refs):
            assert n_gpu[e] == n_ref, (mode, lm, e, n_gpu[e], n_ref)
            err = np.linalg.norm(sim3.log(sim3.compose(S_gpu[e], sim3.inverse(S_ref))))
            assert err < 1e-6, (mode, lm, e, err)
        assert n_gpu[3] == 0 and np.array_equal(S_gpu[3], S0[3]), mode


def _inverse_set(fl, sets, cams):
    """InversePairs over the events' sets (xyz, uv, kf, T) (None: no pair);
    keyframes of every set concatenated, each with its event's camera."""
    off, xs, us, ks, Ts, Cs = [0], [], [], [], [], []
    n_kf = 0
    for st, cam in zip(sets, cams):
        if st is None:
            off.append(off[-1])
            continue
        x, u, k, T = st
        xs.append(x)
        us.append(u)
        ks.append(k + n_kf)
        Ts.append(T)
        Cs.append(np.tile(np.asarray(cam[:4], np.float32), (len(T), 1)))
        n_kf += len(T)
        off.append(off[-1] + len(x))
    cat = lambda a: np.ascontiguousarray(np.concatenate(a))
    return fl.InversePairs(np.array(off, np.int64), t(cat(xs)), t(cat(us)), t(cat(ks).astype(np.int32)),
                           t(cat(Ts).astype(np.float32)), t(cat(Cs)))


def test_two_sided_refinement_in_the_batched_launch(ctx):
    """The refinement inside the batched launch on both directions of a loop:
    the event's accepted pairs observed through S and 8,000 current-side
    points observed in four loop-side keyframes through S^-1, one system per
    step; against the float64 two-sided Gauss-Newton, in every launch mode.
    The other direction moves the result by ~1e-4, far above the bound."""
    import paper_2603_17201_amd as fl
    ev = synth.gen_c2()
    out = oracle.search_fuse(ev, use_grid=True)
    acc = np.nonzero((out["decision"] == oracle.ADD) | (out["decision"] == oracle.FUSE))[0]
    kf = (np.searchsorted(ev.pair_offset, acc, side="right") - 1).astype(np.int32)
    mp = acc - ev.pair_offset[kf]
    kp = ev.kp_offset[kf] + out["best_idx"][acc]
    xyz, uv = ev.mp_xyz[mp], ev.kp_xy[kp]
    T32 = ev.kf_T.astype(np.float32).astype(np.float64)
    xb, ub, kb, Tb = synth.gen_inverse_pairs(ev.S_true, 8000, seed=707)
    inv = _inverse_set(fl, [(xb, ub, kb, Tb)], [ev.cams[0]])
    S_ref = R.gauss_newton_bidir(ev.S_init, (xyz, uv, kf, T32), (xb, ub, kb, Tb.astype(np.float64)), ev.cams[0],
                                 2.45, iters=10)
    S_one = R.gauss_newton(ev.S_init, xyz, uv, kf, T32, ev.cams[0], 2.45, iters=10)
    assert np.linalg.norm(sim3.log(sim3.compose(S_one, sim3.inverse(S_ref)))) > 1e-5
    b = fl.DeviceBatch(ev, device=dev())
    res = ctx.search_fuse_graph(b, ev.params)
    for mode in ("batched", "graph", "scan"):
        event_S = t(ev.S_init.reshape(1, 13).copy())
        nm = torch.zeros(1, dtype=torch.int32, device=dev())
        ref = (10, 2.45, event_S, None, nm, 0, 0.0, 0.0, inv)
        if mode == "graph":
            got = ctx.search_fuse_graph(b, ev.params, refine=ref).numpy()
        elif mode == "batched":
            got = ctx.search_fuse_batched(b, ev.params, refine=ref).numpy()
        else:
            ctx.refine_events(b, res, ref)
            got = res.numpy()
        for k in got:
            assert np.array_equal(got[k], out[k]), (mode, k)
        assert nm.item() == len(acc) + len(xb), mode   # every point is in front of its keyframe
        S_gpu = event_S.cpu().numpy()[0]
        err = np.linalg.norm(sim3.log(sim3.compose(S_gpu, sim3.inverse(S_ref))))
        assert err < 1e-6, (mode, err)


def test_two_sided_refinement_multi_event_batch(ctx):
    """Four events in one launch with uneven inverse sets: one with none, one
    whose search accepts no pair (its system comes from the other direction
    alone), and a keyframe index out of range that must add nothing."""
    import paper_2603_17201_amd as fl
    e0 = synth.gen_c3(seed=321, n_kf=10, n_mp=5000, id_base=1000, fresh_base=10 ** 9)
    e1 = synth.gen_tiny(62, n_kf=3, n_mp=400)
    e2 = synth.gen_c2(seed=207, n_kf=5, n_mp=3000)
    e3 = synth.gen_tiny(63, n_kf=2, n_mp=150)
    e3.kp_desc = e3.kp_desc ^ np.uint8(0xFF)   # every distance far above the threshold
    B = synth.concat_events([e0, e1, e2, e3])
    exp = oracle.search_fuse(B, use_grid=True)
    sets = [synth.gen_inverse_pairs(e0.S_true, 3000, seed=710), None,
            synth.gen_inverse_pairs(e2.S_true, 5000, seed=712), synth.gen_inverse_pairs(e3.S_true, 2000, seed=713)]
    cams = [B.cams[int(B.event_kf_offset[e])] for e in range(4)]
    cam_bwd = np.array(list(synth.CAM_752) + [0.0, 0.0], np.float32)
    # the inverse sets are seen by 752x480 cameras whatever the event's camera
    inv = _inverse_set(fl, sets, [cam_bwd] * 4)
    # one pair of event 2 names a keyframe outside the set: it adds nothing
    bad = int(inv.event_offset[2]) + 17
    kfi = inv.kf_idx.cpu().numpy()
    kfi[bad] = 1000
    inv.kf_idx = t(kfi)
    refs = []
    for e in range(4):
        fx = _event_pairs(B, exp, e)
        st = sets[e]
        if st is not None and e == 2:
            keep = np.ones(len(st[0]), bool)
            keep[17] = False
            st = (st[0][keep], st[1][keep], st[2][keep], st[3])
        n_f = len(fx[0])
        if st is None:
            S_ref = R.gauss_newton(B.events[e].S_init, *fx, cams[e], 2.45, iters=10) if n_f else None
            refs.append((S_ref, n_f))
            continue
        S_ref = R.gauss_newton_bidir(B.events[e].S_init, fx, st[:3] + (st[3].astype(np.float64),), cams[e], 2.45,
                                     iters=10, cam_bwd=cam_bwd)
        refs.append((S_ref, n_f + len(st[0])))
    assert refs[3][1] == 2000   # event 3: the other direction only
    b = fl.DeviceBatch(B, device=dev())
    S0 = np.stack([ev.S_init for ev in B.events])
    for mode in ("batched", "graph"):
        S = t(S0.copy())
        nm = torch.zeros(4, dtype=torch.int32, device=dev())
        ref = (10, 2.45, S, None, nm, 0, 0.0, 0.0, inv)
        res = (ctx.search_fuse_batched(b, B.params, refine=ref) if mode == "batched"
               else ctx.search_fuse_graph(b, B.params, refine=ref))
        got = res.numpy()
        for k in got:
            assert np.array_equal(got[k], exp[k]), (mode, k)
        S_gpu, n_gpu = S.cpu().numpy(), nm.cpu().numpy()
        for e, (S_ref, n_ref) in enumerate(refs):
            assert n_gpu[e] == n_ref, (mode, e, n_gpu[e], n_ref)
            err = np.linalg.norm(sim3.log(sim3.compose(S_gpu[e], sim3.inverse(S_ref))))
            assert err < 1e-6, (mode, e, err)


def test_two_sided_refinement_rejects_bad_arguments(ctx):
    """Offsets that do not start at 0, and the robust variants (the other
    direction is Gauss-Newton only), are refused before any launch."""
    import paper_2603_17201_amd as fl
    from paper_2603_17201_amd import _abi
    ev = synth.gen_tiny(64, n_kf=2, n_mp=200)
    b = fl.DeviceBatch(ev, device=dev())
    xb, ub, kb, Tb = synth.gen_inverse_pairs(ev.S_true, 100, seed=714)
    S = t(ev.S_init.reshape(1, 13).copy())
    cam4 = t(np.tile(np.asarray(ev.cams[0][:4], np.float32), (len(Tb), 1)))
    for off, rounds, lm, code in (([1, 100], 0, 0.0, _abi.FL_EINVAL), ([0, 100], 0, 0.5, _abi.FL_ENOTSUP),
                                  ([0, 100], 2, 0.0, _abi.FL_ENOTSUP)):
        inv = fl.InversePairs(np.asarray(off, np.int64), t(xb), t(ub), t(kb), t(Tb), cam4)
        ref = (5, 2.45, S, None, None, rounds, 3.0 if rounds else 0.0, lm, inv)
        with pytest.raises(fl.FlError) as ei:
            ctx.search_fuse_batched(b, ev.params, refine=ref)
        assert ei.value.code == code, (off, rounds, lm, ei.value)


@pytest.mark.parametrize("n", [0, 1, 63, 256, 257, 2049, 14337, 262144, 262145])
def test_residual_sums_over_every_grid_shape(ctx, n):
    """One block and many, blocks with a few pairs, more rows of partials than
    one round of loads takes, the largest grid and pairs beyond it: loss, g
    and H against float64 to the bound of the other residual tests, and the
    one-launch form of the autograd function against the separate calls: the
    same float32 Sim3 to the bit and sums that differ by their float64 order
    at most."""
    d = synth.gen_c4(n=max(n, 1))
    xyz, uv = d["xyz"][:n], d["uv"][:n]
    xi, S_true = d["xi0"], d["S_true"]
    S0, S32 = ctx.sim3_exp_mul(t(xi), t(S_true))
    _, _, loss = ctx.residual_fwd(t(xyz), t(uv), None, None, S32, d["cam"], 2.45)
    g, H = ctx.residual_bwd(t(xyz), t(uv), None, None, S32, d["cam"], 2.45)
    if n:
        S64 = S0.cpu().numpy()
        L64 = R.forward(S64, xyz, uv, None, None, d["cam"], 2.45)[2]
        g64, H64, _ = R.grad_hess(S64, xyz, uv, None, None, d["cam"], 2.45)
        assert abs(loss.item() - L64) / L64 < REL
        assert rel(g.cpu().numpy(), g64) < REL
        assert rel(H.cpu().numpy(), R.H_upper(H64)) < REL
    else:
        assert loss.item() == 0.0 and not g.any() and not H.any()
    scale = t(np.array([1.7]))
    gx = ctx.sim3_grad_xi(t(xi), g, scale).cpu().numpy()
    one32, one = ctx._residual_fwd_xi(t(xi), t(S_true), t(xyz), t(uv), None, None, d["cam"], 2.45)
    gone = ctx._residual_bwd_xi(t(xi), scale, t(xyz), t(uv), None, None, S32, d["cam"], 2.45).cpu().numpy()
    assert torch.equal(one32, S32)
    assert abs(one.item() - loss.item()) <= 1e-14 * loss.item()
    assert np.max(np.abs(gone - gx)) <= 1e-13 * np.max(np.abs(gx))


@pytest.mark.parametrize("n_kf", [5, 64, 128, 129])
def test_refinement_at_the_keyframe_table_limit(ctx, n_kf):
    """Keyframe poses in LDS up to 128 keyframes of an event, from device
    memory beyond, and two events that hold one, two, three and more accepted
    pairs a thread between them: the oracle's accepted pairs, and float64
    Gauss-Newton on them to the bound of the other refinement tests."""
    import paper_2603_17201_amd as fl
    few = synth.gen_c2(seed=211, n_kf=n_kf, n_mp=900, n_kp=40)
    many = synth.gen_c2(seed=212, n_kf=4, n_mp=4000, n_kp=800)
    B = synth.concat_events([few, many])
    exp = oracle.search_fuse(B, use_grid=True)
    S = t(np.stack([ev.S_init for ev in B.events]))
    nm = torch.zeros(2, dtype=torch.int32, device=dev())
    got = ctx.search_fuse_batched(fl.DeviceBatch(B, device=dev()), B.params, refine=(6, 2.45, S, None, nm)).numpy()
    for k in got:
        assert np.array_equal(got[k], exp[k]), k
    for e in range(2):
        S_ref, n_ref = _event_gn(B, exp, e, iters=6)
        assert nm[e].item() == n_ref
        assert np.linalg.norm(sim3.log(sim3.compose(S[e].cpu().numpy(), sim3.inverse(S_ref)))) < 1e-6


def test_two_sided_pairs_that_are_not_finite_add_nothing(ctx):
    """Pairs of the other direction whose point or depth is not a number or
    infinite add nothing, like those behind their keyframe: the same Sim3 as
    without them (another order of the float32 sums of a quad at most)."""
    import paper_2603_17201_amd as fl
    ev = synth.gen_c2(seed=213, n_kf=4, n_mp=2000, n_kp=500)
    xyz, uv, kf, T = synth.gen_inverse_pairs(ev.S_true, 700, seed=9)
    bad = np.array([[np.nan, 1, 2], [1, np.inf, 2], [0, 0, -np.inf], [np.nan] * 3], np.float32)
    cam = t(np.tile(np.array(synth.CAM_752[:4], np.float32), (len(T), 1)))
    b = fl.DeviceBatch(ev, device=dev())
    out = []
    for extra in (0, len(bad)):
        x = np.concatenate([xyz, bad[:extra]])
        inv = fl.InversePairs([0, len(x)], t(x), t(np.concatenate([uv, uv[:extra]])), t(np.concatenate([kf, kf[:extra]])),
                              t(T), cam)
        S = t(ev.S_init.reshape(1, 13).copy())
        nm = torch.zeros(1, dtype=torch.int32, device=dev())
        ctx.search_fuse_batched(b, ev.params, refine=(6, 2.45, S, None, nm, 0, 0.0, 0.0, inv))
        out.append((S.cpu().numpy()[0], nm.item()))
    assert out[0][1] == out[1][1]
    assert np.linalg.norm(sim3.log(sim3.compose(out[1][0], sim3.inverse(out[0][0])))) < 1e-6


@pytest.mark.parametrize("lm", [None, synth.ROBUST_LM_LAMBDA])
def test_refinement_of_more_pairs_than_the_registers_hold(ctx, lm):
    """128 events leave two workgroups of 512 threads each: of the three large
    ones the first has pairs for the registers and the LDS of its threads, the
    second fills both, the third has pairs beyond them.  Gauss-Newton, and
    Levenberg-Marquardt in rounds."""
    import paper_2603_17201_amd as fl
    big = [synth.gen_c2(seed=241 + n, n_kf=n, n_mp=6000) for n in (4, 6, 8)]
    evs = big[:1] + [synth.gen_tiny(700 + i, n_kf=2, n_mp=40, n_kp=(8, 14)) for i in range(125)] + big[1:]
    B = synth.concat_events(evs)
    P = B.params
    exp = oracle.search_fuse(B, use_grid=True)
    at = (0, 126, 127)
    it, rounds, tau = synth.ROBUST_ITERS, synth.ROBUST_ROUNDS, synth.ROBUST_OUTLIER_PX
    refs = []
    for e in at:
        if lm is None:
            refs.append(_event_gn(B, exp, e))
            continue
        xyz, uv, kfl, T32 = _event_pairs(B, exp, e)
        refs.append(R.refine_robust(B.events[e].S_init, xyz, uv, kfl, T32, B.cams[int(B.event_kf_offset[e])],
                                    float(np.float32(2.45)), iters=it, rounds=rounds,
                                    outlier_px=float(np.float32(tau)), lm_lambda=lm))
    n_acc = [len(_event_pairs(B, exp, e)[0]) for e in at]
    assert 3072 < n_acc[0] < 4096 < n_acc[1] < 5120 < n_acc[2], n_acc
    b = fl.DeviceBatch(B, device=dev())
    S0 = np.stack([ev.S_init for ev in B.events])
    for run in (ctx.search_fuse_batched, ctx.search_fuse_graph):
        S = t(S0.copy())
        nm = torch.zeros(len(evs), dtype=torch.int32, device=dev())
        ref = (10, 2.45, S, None, nm) if lm is None else (it, 2.45, S, None, nm, rounds, tau, lm)
        got = run(b, P, refine=ref).numpy()
        for k in got:
            assert np.array_equal(got[k], exp[k]), (run.__name__, k)
        S_gpu, n_gpu = S.cpu().numpy(), nm.cpu().numpy()
        for e, (S_ref, n_ref) in zip(at, refs):
            assert n_gpu[e] == n_ref, (run.__name__, e, n_gpu[e], n_ref)
            err = np.linalg.norm(sim3.log(sim3.compose(S_gpu[e], sim3.inverse(S_ref))))
            assert err < 1e-6, (run.__name__, e, err)


NOT_FINITE = [np.nan, np.inf, -np.inf]


@pytest.mark.parametrize("bad", NOT_FINITE)
@pytest.mark.parametrize("what", ["padding", "observation", "pose", "intrinsics"])
def test_excluded_pairs_of_the_other_direction_add_nothing_whatever_they_hold(ctx, what, bad):
    """Pairs of the other direction whose depth is not positive, or whose point
    and observation are both not finite, with a value that is not finite in
    their observation, keyframe pose or intrinsics: the count and the Sim3 of
    the launch without them (another order of the float32 sums of a quad at
    most), in each launch that refines."""
    import paper_2603_17201_amd as fl
    ev = synth.gen_c2(seed=213, n_kf=4, n_mp=2000, n_kp=500)
    xyz, uv, kf, T = synth.gen_inverse_pairs(ev.S_true, 700, seed=9)
    T = np.asarray(T, np.float32)
    cam = np.tile(np.array(synth.CAM_752[:4], np.float32), (len(T), 1))
    # a further keyframe, with every point far behind it
    extra_T = np.array([[1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, -1e6]], np.float32)
    extra_cam, m = cam[:1].copy(), 70
    x_bad, u_bad = xyz[:m].copy(), uv[:m].copy()
    if what == "padding":
        x_bad[:], u_bad[:] = bad, bad
        extra_T[0, 6:9] = 0.0   # zero times the point: a depth that is not a number
    elif what == "observation":
        u_bad[:] = bad
    elif what == "pose":
        extra_T[0, [0, 4, 9, 10]] = bad
    else:
        extra_cam[:] = bad
    n_T = len(T)
    b = fl.DeviceBatch(ev, device=dev())
    res = ctx.search_fuse_graph(b, ev.params)
    out = {}
    for extra in (False, True):
        x, u, k = (np.concatenate([xyz, x_bad]), np.concatenate([uv, u_bad]),
                   np.concatenate([kf, np.full(m, n_T, np.int32)])) if extra else (xyz, uv, kf)
        inv = fl.InversePairs([0, len(x)], t(x), t(u), t(k.astype(np.int32)), t(np.concatenate([T, extra_T])),
                              t(np.concatenate([cam, extra_cam])))
        for mode in ("batched", "graph", "scan"):
            S = t(ev.S_init.reshape(1, 13).copy())
            nm = torch.zeros(1, dtype=torch.int32, device=dev())
            ref = (6, 2.45, S, None, nm, 0, 0.0, 0.0, inv)
            if mode == "scan":
                ctx.refine_events(b, res, ref)
            else:
                (ctx.search_fuse_batched if mode == "batched" else ctx.search_fuse_graph)(b, ev.params, refine=ref)
            out[mode, extra] = (S.cpu().numpy()[0], nm.item())
    for mode in ("batched", "graph", "scan"):
        (S0, n0), (S1, n1) = out[mode, False], out[mode, True]
        assert n0 == n1 > 700, (mode, n0, n1)
        assert not np.array_equal(S0, ev.S_init), mode
        err = np.linalg.norm(sim3.log(sim3.compose(S1, sim3.inverse(S0))))
        assert err < 1e-6, (mode, err)


@pytest.mark.parametrize("bad", NOT_FINITE)
@pytest.mark.parametrize("lm", [None, synth.ROBUST_LM_LAMBDA])
@pytest.mark.parametrize("matched", [False, True])
def test_keyframe_poses_that_are_not_finite_add_nothing(ctx, matched, lm, bad):
    """An event whose first keyframe's pose is not finite (every depth not a
    number or negative, the image rows any of the three): the accepted pairs of
    the other keyframes alone are refined, whether the first keyframe has some
    (left out, float64 reference on the rest) or none (threads without a pair
    read that pose)."""
    import paper_2603_17201_amd as fl
    ev = synth.gen_c2(seed=214, n_kf=4, n_mp=3000, n_kp=600)
    n0 = int(ev.kp_offset[1])
    if not matched:
        ev.kp_desc[:n0] ^= np.uint8(0xFF)   # every distance far above the threshold
    B = synth.concat_events([ev])
    exp = oracle.search_fuse(B, use_grid=True)
    xyz, uv, kfl, T32 = _event_pairs(B, exp, 0)
    assert (np.count_nonzero(kfl == 0) > 100) == matched
    rest = kfl != 0
    B.kf_T = np.array(B.kf_T, np.float32)
    T0 = B.kf_T.reshape(-1, 12)[0]
    T0[:] = [bad, 0, 0, 0, bad, 0, 0, 0, 1, bad, bad, -np.inf if bad == -np.inf else -1e6]
    if np.isnan(bad):
        T0[6:9] = bad
    it, rounds, tau = synth.ROBUST_ITERS, synth.ROBUST_ROUNDS, synth.ROBUST_OUTLIER_PX
    if lm is None:
        S_ref = R.gauss_newton(ev.S_init, xyz[rest], uv[rest], kfl[rest], T32, B.cams[0], 2.45, iters=10)
        n_ref = int(rest.sum())
    else:
        S_ref, n_ref = R.refine_robust(ev.S_init, xyz[rest], uv[rest], kfl[rest], T32, B.cams[0],
                                       float(np.float32(2.45)), iters=it, rounds=rounds,
                                       outlier_px=float(np.float32(tau)), lm_lambda=lm)
    b = fl.DeviceBatch(B, device=dev())
    res = ctx.search_fuse_graph(b, B.params)
    for mode in ("batched", "graph", "scan"):
        S = t(ev.S_init.reshape(1, 13).copy())
        nm = torch.zeros(1, dtype=torch.int32, device=dev())
        ref = (10, 2.45, S, None, nm) if lm is None else (it, 2.45, S, None, nm, rounds, tau, lm)
        if mode == "scan":
            ctx.refine_events(b, res, ref)
        else:
            (ctx.search_fuse_batched if mode == "batched" else ctx.search_fuse_graph)(b, B.params, refine=ref)
        assert nm.item() == n_ref, (mode, nm.item(), n_ref)
        err = np.linalg.norm(sim3.log(sim3.compose(S.cpu().numpy()[0], sim3.inverse(S_ref))))
        assert err < 1e-6, (mode, err)


def test_events_without_keyframes_are_refined_from_the_other_direction(ctx):
    """The first, the third and the last of four events have no keyframe and no
    point, the first and the last some hundred pairs of the other direction
    (one workgroup, and two): float64 two-sided Gauss-Newton on those; the third
    is left as it was."""
    import paper_2603_17201_amd as fl
    ev = synth.gen_c2(seed=215, n_kf=3, n_mp=2000, n_kp=500)
    B = synth.concat_events([ev])
    exp = oracle.search_fuse(B, use_grid=True)
    fx = _event_pairs(B, exp, 0)
    B.event_kf_offset = np.array([0, 0, 3, 3, 3], np.int32)
    B.event_mp_offset = np.array([0, 0, ev.n_mp, ev.n_mp, ev.n_mp], np.int32)
    sets = [synth.gen_inverse_pairs(ev.S_true, 300, seed=31), None, None, synth.gen_inverse_pairs(ev.S_true, 900, seed=32)]
    cam_bwd = np.array(list(synth.CAM_752) + [0.0, 0.0], np.float32)
    inv = _inverse_set(fl, sets, [cam_bwd] * 4)
    none = tuple(a[:0] for a in fx[:3]) + (fx[3],)
    refs = [(ev.S_init, 0) if st is None else
            (R.gauss_newton_bidir(ev.S_init, none, st[:3] + (st[3].astype(np.float64),), cam_bwd, 2.45, iters=10,
                                  cam_bwd=cam_bwd), len(st[0])) for st in sets]
    refs[1] = (R.gauss_newton(ev.S_init, *fx, B.cams[0], 2.45, iters=10), len(fx[0]))
    b = fl.DeviceBatch(B, device=dev())
    for run in (ctx.search_fuse_batched, ctx.search_fuse_graph):
        S = t(np.stack([ev.S_init] * 4))
        nm = torch.zeros(4, dtype=torch.int32, device=dev())
        got = run(b, B.params, refine=(10, 2.45, S, None, nm, 0, 0.0, 0.0, inv)).numpy()
        for k in got:
            assert np.array_equal(got[k], exp[k]), (run.__name__, k)
        for e, (S_ref, n_ref) in enumerate(refs):
            assert nm[e].item() == n_ref, (run.__name__, e, nm[e].item(), n_ref)
            err = np.linalg.norm(sim3.log(sim3.compose(S[e].cpu().numpy(), sim3.inverse(S_ref))))
            assert err < 1e-6, (run.__name__, e, err)


def test_event_without_keyframes_after_one_whose_pose_is_not_a_number(ctx):
    """257 events: the workgroup of event 0, whose keyframes' poses are not a
    number, goes on to event 256, which has no keyframe and is refined from the
    other direction alone; the ones between have neither."""
    import paper_2603_17201_amd as fl
    ev = synth.gen_tiny(216, n_kf=2, n_mp=60, n_kp=(20, 30))
    B = synth.concat_events([ev])
    B.kf_T = np.full_like(np.asarray(B.kf_T, np.float32), np.nan)
    n = 257
    B.event_kf_offset = np.array([0] + [2] * n, np.int32)
    B.event_mp_offset = np.array([0] + [ev.n_mp] * n, np.int32)
    st = synth.gen_inverse_pairs(ev.S_true, 300, seed=33)
    cam = np.array(list(synth.CAM_752) + [0.0, 0.0], np.float32)
    inv = _inverse_set(fl, [None] * (n - 1) + [st], [cam] * n)
    none = (np.zeros((0, 3)), np.zeros((0, 2)), np.zeros(0, np.int32), np.zeros((2, 12)))
    S_ref = R.gauss_newton_bidir(ev.S_init, none, st[:3] + (st[3].astype(np.float64),), cam, 2.45, iters=10, cam_bwd=cam)
    b = fl.DeviceBatch(B, device=dev())
    for run in (ctx.search_fuse_batched, ctx.search_fuse_graph):
        S = t(np.stack([ev.S_init] * n))
        nm = torch.zeros(n, dtype=torch.int32, device=dev())
        run(b, B.params, refine=(10, 2.45, S, None, nm, 0, 0.0, 0.0, inv))
        S = S.cpu().numpy()
        assert nm.cpu().tolist() == [0] * (n - 1) + [len(st[0])], run.__name__
        assert all(np.array_equal(S[e], ev.S_init) for e in range(n - 1)), run.__name__
        err = np.linalg.norm(sim3.log(sim3.compose(S[-1], sim3.inverse(S_ref))))
        assert err < 1e-6, (run.__name__, err)
