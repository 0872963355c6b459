"""What is measured: the calls a loop-closing program makes, over their real range.

Scenes follow the generators of ``synth/`` (an arc of covisible keyframes, ORB-like keypoints over 8 octaves of which
half are planted observations, 256-bit descriptors with 5% of the bits flipped, a loop Sim3 a little off the truth),
drawn with torch on the device so that fresh inputs are cheap.  Families:

* ``plain``  one keyframe against a point list, the per-call search (``Context.search_fuse``)
* ``event``  one loop event or several in one launch: batched search, ADD resolution and Sim3 refinement
* ``residual``  the differentiable reprojection residual, forward and backward
* ``two_sided``  one Gauss-Newton step on the matches of both directions of a loop
* ``graph``  essential-graph optimisation of Sim3 keyframe poses
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2603_17201_amd as fl

CAM_752 = (458.0, 458.0, 367.0, 248.0, 752.0, 480.0)
CAM_512 = (190.0, 190.0, 256.0, 256.0, 512.0, 512.0)
N_OCT, SCALE = 8, 1.2
HUBER = 2.45
F64 = torch.float64
OUT = ("best_idx", "best_dist", "second_dist", "decision", "target")


def listed():
    return [
        # the per-call search on the current keyframe: one keyframe, fusion thresholds
        dict(name="plain_1kf", family="plain", cam=752, n_mp=2000, n_kp=1000, win=3.0, ratio=0.0),
        # loop verification's projection search: one keyframe in one launch, wide window, ratio test; the smallest batch
        dict(name="verify_1kf", family="event", events=1, cam=752, n_kf=1, n_mp=2000, kp_lo=1000, kp_hi=1000,
             sparse=False, win=10.0, ratio=0.75, refine="none", graph=False),
        # the ordinary loop event: 20 covisible keyframes, every point against each, then ten Gauss-Newton steps
        dict(name="event_20kf", family="event", events=1, cam=752, n_kf=20, n_mp=15000, kp_lo=1200, kp_hi=1200,
             sparse=False, win=3.0, ratio=0.0, refine="gn", graph=False),
        # a mid-size event of uneven keyframes replayed from a captured graph, refined on both directions' matches
        dict(name="event_33kf_graph", family="event", events=1, cam=512, n_kf=33, n_mp=41377, kp_lo=300, kp_hi=2500,
             sparse=False, win=3.0, ratio=0.0, refine="two_sided", graph=True),
        # an uneven event whose pairs are the covisibility list, not every point against every keyframe
        dict(name="event_60kf_sparse", family="event", events=1, cam=512, n_kf=60, n_mp=60000, kp_lo=300, kp_hi=2500,
             sparse=True, win=3.0, ratio=0.0, refine="gn", graph=False),
        # the verification window followed by the robust refinement (rounds with an inlier bound, Levenberg-Marquardt)
        dict(name="event_20kf_robust", family="event", events=1, cam=752, n_kf=20, n_mp=15000, kp_lo=1200, kp_hi=1200,
             sparse=False, win=10.0, ratio=0.75, refine="lm", graph=False),
        # the largest event of the stream: 73 keyframes, 97,969 points, 7.15 M pairs
        dict(name="event_73kf", family="event", events=1, cam=752, n_kf=73, n_mp=97969, kp_lo=300, kp_hi=2500,
             sparse=False, win=3.0, ratio=0.0, refine="gn", graph=False),
        # ten uneven events in one launch (offline or multi-session closing): 4.7 M listed pairs
        dict(name="events_10_sparse", family="event", events=10, cam=512, n_kf=60, n_mp=60000, kp_lo=300, kp_hi=2500,
             sparse=True, win=3.0, ratio=0.0, refine="gn", graph=False),
        # the differentiable residual inside an autograd program: forward, then the hand-written backward
        dict(name="residual_50k", family="residual", n=50000),
        # one two-sided Gauss-Newton step: 20,000 pairs each way over four keyframes a side
        dict(name="two_sided_20k", family="two_sided", n_fwd=20000, n_bwd=19999, views=4),
        # loop correction of one loop of 1,000 keyframes: ten Levenberg-Marquardt iterations, direct solve
        dict(name="graph_1000_1lap", family="graph", n=1000, laps=1, iters=10),
        # the same map after three loops: cross edges widen the reordered band
        dict(name="graph_1000_3laps", family="graph", n=1000, laps=3, iters=10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes over their logarithm, options as in the list."""
    kind = rng.choice(["plain", "event", "event", "event", "events", "residual", "two_sided", "graph"])
    if kind == "plain":
        return dict(family="plain", cam=rng.choice([752, 512]), n_mp=_log_int(rng, 200, 20000),
                    n_kp=_log_int(rng, 300, 2500), win=rng.choice([3.0, 10.0]), ratio=rng.choice([0.0, 0.75]))
    if kind in ("event", "events"):
        many = kind == "events"
        lo, n_kf = _log_int(rng, 300, 2000), _log_int(rng, 5, 40) if many else _log_int(rng, 1, 80)
        # one or two views hardly determine a Sim3: those searches go without refinement
        refine = rng.choice(["none", "gn", "gn", "rounds", "lm", "two_sided"]) if n_kf >= 5 else "none"
        return dict(family="event", events=rng.randint(2, 6) if many else 1, cam=rng.choice([752, 512]), n_kf=n_kf,
                    n_mp=_log_int(rng, 2000, 30000) if many else _log_int(rng, 2000, 90000),
                    kp_lo=lo, kp_hi=rng.randint(lo, 2500), sparse=rng.random() < 0.4, win=rng.choice([3.0, 3.0, 10.0]),
                    ratio=rng.choice([0.0, 0.75]), refine=refine, graph=rng.random() < 0.25)
    if kind == "residual":
        return dict(family="residual", n=_log_int(rng, 500, 400000))
    if kind == "two_sided":
        return dict(family="two_sided", n_fwd=_log_int(rng, 500, 200000), n_bwd=_log_int(rng, 500, 200000),
                    views=rng.randint(1, 12))
    return dict(family="graph", n=_log_int(rng, 60, 1000), laps=rng.choice([1, 1, 2, 3]), iters=rng.choice([5, 10]))


# ---------------------------------------------------------------------------
# scenes (float64 torch on the device)

def _dev():
    return torch.device("cuda", 0)


def _rng(seed):
    g = torch.Generator(device=_dev())
    g.manual_seed(int(seed))
    return g


def _hat(w):
    """[w]x of [..., 3]."""
    z = torch.zeros_like(w[..., 0])
    return torch.stack([z, -w[..., 2], w[..., 1], w[..., 2], z, -w[..., 0], -w[..., 1], w[..., 0], z],
                       -1).reshape(*w.shape[:-1], 3, 3)


def _rot(axis, angle):
    """Rotations by `angle` (radians) about unit `axis` [..., 3]."""
    K = _hat(axis)
    a = torch.as_tensor(angle, dtype=F64, device=axis.device)[..., None, None]
    return torch.eye(3, dtype=F64, device=axis.device) + torch.sin(a) * K + (1 - torch.cos(a)) * (K @ K)


def _unit(g, *shape):
    v = torch.randn((*shape, 3), dtype=F64, device=_dev(), generator=g)
    return v / v.norm(dim=-1, keepdim=True)


def _uniform(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(shape, dtype=F64, device=_dev(), generator=g)


def _normal(g, sigma, *shape):
    return sigma * torch.randn(shape, dtype=F64, device=_dev(), generator=g)


def _ints(g, lo, hi, *shape):
    return torch.randint(lo, hi, shape, device=_dev(), generator=g)


def _loop_sim3(g):
    """A loop correction (scale 0.95-1.05, up to 5 deg, 0.1 m) and a start 0.1 deg, 1 cm and 0.2% off it."""
    R = _rot(_unit(g), _uniform(g, 0.0, math.radians(5.0)))
    t, s = 0.1 * _unit(g), _uniform(g, 0.95, 1.05)
    Rp = _rot(_unit(g), math.radians(0.1))
    return (R, t, s), (Rp @ R, Rp @ t + 0.01 * _unit(g), 1.002 * s)


def _flat(S):
    return torch.cat([S[0].reshape(9), S[1], S[2].reshape(1)])


def _poses(cam, n):
    """World -> camera poses on an arc facing its centre."""
    radius, step = (5.0, 3.0 / 19.0) if cam is CAM_752 else (3.0, 0.1)
    phi = (torch.arange(n, dtype=F64, device=_dev()) - 0.5 * (n - 1)) * (step / radius)
    axis = torch.tensor([0.0, 1.0, 0.0], dtype=F64, device=_dev()).expand(n, 3)
    R = _rot(axis, phi)
    c = torch.stack([radius * torch.sin(phi), torch.zeros_like(phi), radius - radius * torch.cos(phi)], -1)
    return R, -(R @ c[:, :, None])[:, :, 0]


def _camera(S, R, t):
    """T_k o S for every pose: (R, t, s)."""
    return R @ S[0], (R @ S[1][:, None])[..., 0] + t, S[2]


def _sim3_f32(S):
    """Search form of [..] Sim3s (R, t, s): sR, t, 1/s, padding."""
    R, t, s = S
    n = R.shape[0]
    return torch.cat([(s * R).reshape(n, 9), t, (1.0 / s).expand(n, 1), torch.zeros(n, 3, dtype=F64, device=R.device)],
                     1).float()


def _flips(g, desc):
    """Descriptors with each bit flipped with probability 0.05."""
    bits = torch.rand(desc.shape[0], 32, 8, device=_dev(), generator=g) < 0.05
    w = (2 ** torch.arange(8, device=_dev())).to(torch.uint8)
    return desc ^ (bits.to(torch.uint8) * w).sum(-1, dtype=torch.uint8)


def _scene(g, cam, n_kf, n_mp, kp_lo, kp_hi, sparse, id_base):
    """One event: points seen from the middle keyframe (or, sparse, from an anchor of their own and a run of
    neighbours), and keypoints: 50% planted on visible points, 20% planted ones already owned by another point, the
    rest outliers; a tenth of the first are owned by their own point (already observed)."""
    fx, fy, cx, cy, W, H = cam
    dev = _dev()
    S_true, S_init = _loop_sim3(g)
    R, t = _poses(cam, n_kf)
    C = _camera(S_true, R, t)
    anchor = _ints(g, 0, n_kf, n_mp) if sparse else torch.full((n_mp,), n_kf // 2, device=dev)
    u, v = _uniform(g, 0, W, n_mp), _uniform(g, 0, H, n_mp)
    z = _uniform(g, 0.5, 20.0, n_mp)
    q = torch.stack([(u - cx) / fx * z, (v - cy) / fy * z, z], -1)
    X = ((q - C[1][anchor])[:, None, :] @ C[0][anchor])[:, 0] / S_true[2]
    o_ref = _ints(g, 0, N_OCT, n_mp)
    dmax = 0.95 * q.norm(dim=-1) / S_true[2] * SCALE ** o_ref
    xyz, dmax = X.float(), dmax.float()
    desc = _ints(g, 0, 256, n_mp, 32).to(torch.uint8)
    ids = id_base + torch.arange(n_mp, dtype=torch.int32, device=dev)
    # covisibility: the pair list, keyframe by keyframe
    seen = torch.ones(n_kf, n_mp, dtype=torch.bool, device=dev)
    if sparse:
        k = torch.arange(1, 41, dtype=F64, device=dev)
        cdf = torch.cumsum(0.875 ** (k - 1), 0)
        # run lengths by their quantiles, dealt out at random: the list is as long for every seed
        at = (torch.randperm(n_mp, device=dev, generator=g) + 0.5) / n_mp
        run = (1 + torch.searchsorted(cdf / cdf[-1], at.double())).clamp(max=n_kf)
        first = torch.minimum((anchor - (run - 1) // 2).clamp(min=0), n_kf - run)
        kk = torch.arange(n_kf, device=dev)[:, None]
        seen = (kk >= first) & (kk < first + run)
    per_kf = seen.sum(1)
    pair_mp = seen.nonzero()[:, 1].to(torch.int32) if sparse else None
    # keypoints
    n_kp = _ints(g, kp_lo, kp_hi + 1, n_kf)
    parts = {f: [] for f in ("xy", "oct", "desc", "owner")}
    fresh = 1_000_000_000 + 100 * id_base
    Xd = xyz.double()
    for k, n in enumerate(n_kp.tolist()):
        p = Xd @ (S_true[2] * C[0][k]).T + C[1][k]
        pu, pv = fx * p[:, 0] / p[:, 2] + cx, fy * p[:, 1] / p[:, 2] + cy
        vis = (seen[k] & (p[:, 2] > 0) & (pu >= 0) & (pu < W) & (pv >= 0) & (pv < H)).nonzero()[:, 0]
        m = min(round(0.7 * n), vis.numel())
        pick = vis[torch.randperm(vis.numel(), device=dev, generator=g)[:m]]
        d = p[pick].norm(dim=-1) / S_true[2]
        octave = torch.ceil(torch.log(dmax[pick].double() / d) / math.log(SCALE)).clamp(0, N_OCT - 1)
        owner = torch.full((n,), -1, dtype=torch.int64, device=dev)
        n_free = round(m * 5 / 7)
        owner[n_free:m] = fresh + torch.arange(m - n_free, device=dev)
        owner[:n_free // 10] = ids[pick[:n_free // 10]].long()
        fresh += m - n_free
        noise = _normal(g, 1.0, m, 2)
        xy = torch.cat([torch.stack([pu[pick], pv[pick]], -1) + noise,
                        _uniform(g, 0, 1, n - m, 2) * torch.tensor([W, H], dtype=F64, device=dev)])
        octave = torch.cat([octave.long(), _ints(g, 0, N_OCT, n - m)])
        dk = torch.cat([_flips(g, desc[pick]), _ints(g, 0, 256, n - m, 32).to(torch.uint8)])
        order = torch.randperm(n, device=dev, generator=g)
        for f, a in (("xy", xy.float()), ("oct", octave.to(torch.int8)), ("desc", dk), ("owner", owner.int())):
            parts[f].append(a[order])
    cams = torch.tensor(list(cam) + [0.0, 0.0], dtype=torch.float32).expand(n_kf, 8)
    return SimpleNamespace(
        cams=cams.numpy(), kf_T=torch.cat([R.reshape(n_kf, 9), t], 1).float().cpu().numpy(),
        kf_sim3=_sim3_f32(_camera(S_init, R, t)).cpu().numpy(), S_init=_flat(S_init), S_true=S_true,
        mp_xyz=xyz, mp_desc=desc, mp_dmax=dmax, mp_id=ids, n_kp=n_kp.cpu().numpy(),
        kp_xy=torch.cat(parts["xy"]), kp_oct=torch.cat(parts["oct"]), kp_desc=torch.cat(parts["desc"]),
        kp_owner=torch.cat(parts["owner"]), per_kf=per_kf.cpu().numpy(), pair_mp=pair_mp)


def _views(g, n, views, S):
    """n points seen in `views` keyframes through T_k o S, 1 px noise, 10% of them 20 px off."""
    fx, fy, cx, cy, W, H = CAM_752
    R = _rot(_unit(g, views), _uniform(g, 0.0, math.radians(6.0), views))
    t = _unit(g, views) * _uniform(g, 0.0, 0.5, views, 1)
    kf = _ints(g, 0, views, n)
    C = _camera(S, R, t)
    u, v, z = _uniform(g, 0, W, n), _uniform(g, 0, H, n), _uniform(g, 1.0, 10.0, n)
    q = torch.stack([(u - cx) / fx * z, (v - cy) / fy * z, z], -1)
    X = ((q - C[1][kf])[:, None, :] @ C[0][kf])[:, 0] / S[2]
    off = (torch.rand(n, device=_dev(), generator=g) < 0.1).double()[:, None]
    a = _uniform(g, 0, 2 * math.pi, n)
    uv = torch.stack([u, v], -1) + _normal(g, 1.0, n, 2) + off * 20.0 * torch.stack([torch.cos(a), torch.sin(a)], -1)
    return X.float(), uv.float(), kf.int(), torch.cat([R.reshape(views, 9), t], 1).float()


def _inverse(S):
    R, t, s = S
    return R.T, -(R.T @ t) / s, 1.0 / s


def _mul(A, B):
    return A[0] @ B[0], A[2][..., None] * (A[0] @ B[1][..., None])[..., 0] + A[1], A[2] * B[2]


def _inv(S):
    Rt = S[0].transpose(-1, -2)
    return Rt, -(Rt @ S[1][..., None])[..., 0] / S[2][..., None], 1.0 / S[2]


def _pose_graph(g, n, laps):
    """n keyframes round a 5 m loop `laps` times: odometry and covisibility edges to the next three, eight loop edges,
    and on later laps edges to the three keyframes of the lap before at the same place; the start chains the odometry
    with drift."""
    i = torch.arange(n, dtype=F64, device=_dev())
    a = 2 * math.pi * laps * i / n
    rad = 5.0 + (0.25 * laps * i / n if laps > 1 else 0.0 * i)
    y = torch.tensor([0.0, 1.0, 0.0], dtype=F64, device=_dev())
    R = _rot(y.expand(n, 3), -a)
    c = torch.stack([rad * torch.cos(a), 0.1 * torch.sin(3 * a), rad * torch.sin(a)], -1)
    S = (R, -(R @ c[..., None])[..., 0], torch.ones(n, dtype=F64, device=_dev()))
    edges = {(j, j + d) for d in range(1, 4) for j in range(n - d)} | {(n - 1 - k, k) for k in range(8)}
    if laps > 1:
        period = n / laps
        for j in range(math.ceil(period), n):
            j0 = round(j - period) - 1
            edges |= {(m, j) for m in range(max(j0, 0), min(j0 + 3, j - 3))}
    edges = np.array(sorted(edges), np.int32)
    E = len(edges)
    ei, ej = (torch.from_numpy(edges[:, s].astype(np.int64)).to(_dev()) for s in (0, 1))
    pick = lambda P, k: (P[0][k], P[1][k], P[2][k])  # noqa: E731
    M = _mul(pick(S, ej), _inv(pick(S, ei)))
    Rn = _rot(_unit(g, E), math.radians(0.1) * torch.randn(E, dtype=F64, device=_dev(), generator=g).abs())
    M = (Rn @ M[0], (Rn @ M[1][..., None])[..., 0] + _normal(g, 0.01, E, 3), M[2] * torch.exp(_normal(g, 0.001, E)))
    # the start, chained on the host
    Mh = [x.cpu() for x in M]
    at = {(int(p), int(q)): k for k, (p, q) in enumerate(edges)}
    drift = (_rot(y, math.radians(0.02)).cpu(), torch.tensor([0.002, 0.0, 0.0], dtype=F64), torch.tensor(1.002, dtype=F64))
    chain = [tuple(x[0].cpu() for x in S)]
    for j in range(n - 1):
        k = at[(j, j + 1)]
        chain.append(_mul(_mul(drift, tuple(x[k] for x in Mh)), chain[-1]))
    S0 = torch.stack([_flat(s) for s in chain])
    return S0.to(_dev()), torch.cat([M[0].reshape(E, 9), M[1], M[2][:, None]], 1).contiguous(), edges


def _params(case):
    return SimpleNamespace(win_px=case.get("win", 3.0), scale_factor=SCALE, n_octaves=N_OCT, grid_cols=64, grid_rows=48,
                           hamming_th=50, nn_ratio=case.get("ratio", 0.0))


def _cam(case):
    return CAM_752 if case["cam"] == 752 else CAM_512


def _events(case, g):
    """The events of a case and the batch arrays a program hands to DeviceBatch."""
    evs = [_scene(g, _cam(case), case["n_kf"], case["n_mp"], case["kp_lo"], case["kp_hi"], case["sparse"],
                  1000 + e * 1_000_000) for e in range(case["events"])]
    host = lambda f: np.concatenate([getattr(e, f).cpu().numpy() for e in evs])  # noqa: E731
    tab = lambda f: np.concatenate([getattr(e, f) for e in evs])  # noqa: E731
    offs = lambda v, dt: np.concatenate([[0], np.cumsum(v)]).astype(dt)  # noqa: E731
    n_ev = len(evs)
    src = SimpleNamespace(
        event_kf_offset=offs([case["n_kf"]] * n_ev, np.int32), event_mp_offset=offs([case["n_mp"]] * n_ev, np.int32),
        cams=tab("cams"), kf_sim3=tab("kf_sim3"), kf_T=tab("kf_T"), kp_offset=offs(tab("n_kp"), np.int32),
        pair_offset=offs(tab("per_kf"), np.int64), pair_mp=host("pair_mp") if case["sparse"] else None,
        **{f: host(f) for f in ("mp_xyz", "mp_desc", "mp_dmax", "mp_id", "kp_xy", "kp_oct", "kp_desc", "kp_owner")})
    return evs, src


def _other_direction(case, g, evs):
    """Each event's matches of the other direction: a quarter of its points, seen in four loop-side keyframes."""
    sides = [_views(g, case["n_mp"] // 4, 4, _inverse(e.S_true)) for e in evs]
    xyz, uv, kf, T = (torch.cat([s[i] + (4 * e if i == 2 else 0) for e, s in enumerate(sides)]).contiguous() for i in range(4))
    cam = torch.tensor(CAM_752[:4], dtype=torch.float32, device=_dev()).repeat(4 * len(evs), 1).contiguous()
    offset = np.arange(len(evs) + 1, dtype=np.int64) * (case["n_mp"] // 4)
    return offset, xyz, uv, kf, T, cam


# ---------------------------------------------------------------------------
# the calls

_context = []


def _ctx():
    """The one context such a program keeps."""
    if not _context:
        _context.append(fl.Context(0))
    return _context[0]


def prepare(case, seed):
    g = _rng(seed)
    ctx = _ctx()
    st = SimpleNamespace(case=case, ctx=ctx, params=_params(case))
    fam = case["family"]
    if fam == "plain":
        ev = _scene(g, _cam(case), 1, case["n_mp"], case["n_kp"], case["n_kp"], False, 1000)
        st.args = (ev.mp_xyz, ev.mp_desc, ev.mp_dmax, ev.mp_id, ev.kp_xy, ev.kp_oct, ev.kp_desc, ev.kp_owner,
                   ev.kf_sim3[0], ev.cams[0], st.params)
        st.out = fl.FuseOutputs.empty(case["n_mp"], _dev())
    elif fam == "event":
        evs, src = _events(case, g)
        st.batch = fl.DeviceBatch(src, device=_dev())
        st.out = fl.FuseOutputs.empty(st.batch.n_pairs, _dev())
        st.S0 = torch.stack([e.S_init for e in evs]).contiguous()
        st.S = st.S0.clone()
        st.S32 = torch.empty(len(evs), 16, dtype=torch.float32, device=_dev())
        st.n = torch.empty(len(evs), dtype=torch.int32, device=_dev())
        st.refine = None
        if case["refine"] != "none":
            more = {"gn": (10, 0, 0.0, 0.0), "rounds": (5, 2, 3.035, 0.0), "lm": (5, 2, 3.035, 1e-3),
                    "two_sided": (10, 0, 0.0, 0.0)}[case["refine"]]
            st.refine = (more[0], HUBER, st.S, st.S32, st.n) + more[1:]
            if case["refine"] == "two_sided":
                st.refine += (fl.InversePairs(*_other_direction(case, g, evs)),)
    elif fam == "residual":
        S = _loop_sim3(g)[0]
        st.xyz, st.uv, _, _ = _pinhole_pairs(g, case["n"], S)
        st.S0 = _flat(S)
        st.xi0 = torch.tensor([math.radians(1.0), 0.0, 0.0, 0.0, 0.05, 0.0, 0.02], dtype=F64, device=_dev())
        st.cam8 = np.array(list(CAM_752) + [0.0, 0.0], np.float32)
    elif fam == "two_sided":
        S, S0 = _loop_sim3(g)
        st.fwd, st.bwd = _views(g, case["n_fwd"], case["views"], S), _views(g, case["n_bwd"], case["views"], _inverse(S))
        st.S0 = _flat(S0)
        st.S = st.S0.clone()
        st.S32_0 = _sim3_f32((S0[0][None], S0[1][None], S0[2])).reshape(16).contiguous()
        st.S32 = st.S32_0.clone()
        st.cam8 = np.array(list(CAM_752) + [0.0, 0.0], np.float32)
    else:
        st.S0, st.M, st.edges = _pose_graph(g, case["n"], case["laps"])
        st.S = st.S0.clone()
    return st


def _pinhole_pairs(g, n, S):
    """_views with one keyframe at the identity."""
    fx, fy, cx, cy, W, H = CAM_752
    u, v, z = _uniform(g, 0, W, n), _uniform(g, 0, H, n), _uniform(g, 1.0, 10.0, n)
    q = torch.stack([(u - cx) / fx * z, (v - cy) / fy * z, z], -1)
    X = (q - S[1]) @ S[0] / S[2]
    off = (torch.rand(n, device=_dev(), generator=g) < 0.1).double()[:, None]
    a = _uniform(g, 0, 2 * math.pi, n)
    uv = torch.stack([u, v], -1) + _normal(g, 1.0, n, 2) + off * 20.0 * torch.stack([torch.cos(a), torch.sin(a)], -1)
    return X.float(), uv.float(), None, None


def run(st):
    fam, ctx = st.case["family"], st.ctx
    if fam == "plain":
        o = ctx.search_fuse(*st.args, out=st.out)
        return {f: getattr(o, f) for f in OUT}
    if fam == "event":
        if st.refine:
            st.S.copy_(st.S0)   # the event's starting Sim3; the call refines it in place
        call = ctx.search_fuse_graph if st.case["graph"] else ctx.search_fuse_batched
        o = call(st.batch, st.params, out=st.out, refine=st.refine)
        got = {f: getattr(o, f) for f in OUT}
        # the refined Sim3 as the next search takes it: the pairs' terms are float32 and their list is in the order the
        # tiles finished, so the digits of the float64 form below float32 are not the same from run to run
        return {**got, "S32": st.S32, "n": st.n} if st.refine else got
    if fam == "residual":
        xi = st.xi0.clone().requires_grad_(True)
        loss = fl.Sim3Residual.apply(xi, st.S0, st.xyz, st.uv, None, None, st.cam8, HUBER, ctx)
        loss.backward()
        return {"loss": loss.detach(), "grad": xi.grad}
    if fam == "two_sided":
        st.S.copy_(st.S0)
        st.S32.copy_(st.S32_0)
        r, w, loss = ctx.residual_fwd(*st.fwd, st.S32, st.cam8, HUBER)
        g1, H1 = ctx.residual_bwd(*st.fwd, st.S32, st.cam8, HUBER)
        _, Si32 = ctx.sim3_inverse(st.S)
        g2, H2 = ctx.residual_bwd(*st.bwd, Si32, st.cam8, HUBER, inverse=True)
        g, H = g1 + g2, H1 + H2
        ctx.gn_step(g, H, st.S, st.S32)
        return {"r": r, "w": w, "loss": loss, "g": g, "H": H, "S": st.S}
    st.S.copy_(st.S0)
    cost, used = ctx.pose_graph_optimize(st.S, st.M, st.edges, iters=st.case["iters"])
    return {"S": st.S, "cost": cost, "used": used}


def work(case):
    """Each input read once and each output written once; operations of the projection of every pair, of ten steps of
    g and H over the accepted pairs, of the residual, and of the banded factorisation."""
    fam = case["family"]
    if fam == "plain":
        return {"bytes": 61 * case["n_mp"] + 45 * case["n_kp"], "flops": 65 * case["n_mp"]}
    if fam == "event":
        kps = case["n_kf"] * (case["kp_lo"] + case["kp_hi"]) / 2
        k = np.arange(1, 41)
        p = 0.125 * 0.875 ** (k - 1)
        run_mean = float((np.minimum(k, case["n_kf"]) * p).sum() / p.sum())
        pairs = case["n_mp"] * (run_mean if case["sparse"] else case["n_kf"])
        b = 48 * case["n_mp"] + 45 * kps + pairs * (17 if case["sparse"] else 13)
        steps = 0 if case["refine"] == "none" else 10
        inv = case["n_mp"] // 4 if case["refine"] == "two_sided" else 0
        matched = min(0.7 * kps, pairs)
        return {"bytes": case["events"] * (b + (32 * matched + 24 * inv if steps else 0)),
                "flops": case["events"] * (65 * pairs + steps * 250 * (matched + inv))}
    if fam == "residual":
        return {"bytes": 40 * case["n"], "flops": (60 + 250) * case["n"]}
    if fam == "two_sided":
        return {"bytes": 36 * case["n_fwd"] + 24 * (case["n_fwd"] + case["n_bwd"]),
                "flops": 60 * case["n_fwd"] + 280 * (case["n_fwd"] + case["n_bwd"])}
    band = {1: 49, 2: 98, 3: 168}[case["laps"]]
    edges = case["n"] * (3 if case["laps"] == 1 else 6)
    return {"bytes": case["iters"] * (8 * 13 * 2 * (case["n"] + edges) + 8 * 7 * case["n"] * band),
            "flops": case["iters"] * 7 * case["n"] * (band * band + 4 * band)}


# ---------------------------------------------------------------------------
# the same outputs in 64 bits, in plain torch

def exact(case, seed):
    st = prepare(case, seed)
    fam = case["family"]
    if fam == "plain":
        return None   # whole numbers only
    if fam == "event":
        if not st.refine:
            return None
        n = case["events"]
        S, counts = [], []
        for e in range(n):
            s, c = _refined(st, e)
            S.append(_flat(s))
            counts.append(c)
        S = torch.stack(S)
        S32 = torch.cat([S[:, 12:] * S[:, :9], S[:, 9:12], 1.0 / S[:, 12:], torch.zeros(n, 3, dtype=F64, device=S.device)], 1)
        return {**{f: None for f in OUT}, "S32": S32, "n": None}
    if fam == "residual":
        xi = st.xi0
        S = _mul(_exp(xi), _split(st.S0))
        _, _, loss, g, _ = _terms(S, None, st.xyz.double(), st.uv.double(), _cams64(1))
        return {"loss": loss, "grad": _left_jacobian(xi).T @ g}
    if fam == "two_sided":
        S = _split(st.S0)
        a = [x.double() if x.is_floating_point() else x.long() for x in st.fwd]
        b = [x.double() if x.is_floating_point() else x.long() for x in st.bwd]
        r, w, loss, g1, H1 = _terms(S, a[3][a[2]], a[0], a[1], _cams64(1))
        _, _, _, g2, H2 = _terms(S, b[3][b[2]], b[0], b[1], _cams64(1), inverse=True)
        g, H = g1 + g2, H1 + H2
        S = _mul(_exp(-torch.linalg.solve(H, g)), S)
        up = torch.triu_indices(7, 7, device=H.device)
        return {"r": r, "w": w, "loss": loss.reshape(1), "g": g, "H": H[up[0], up[1]], "S": _flat(S)}
    return _graph_lm(st)


def _split(v):
    return v[..., :9].reshape(*v.shape[:-1], 3, 3), v[..., 9:12], v[..., 12]


def _exp(xi):
    """exp of tangents [..., 7] (omega, upsilon, sigma) through the 4x4 generator."""
    A = torch.zeros(*xi.shape[:-1], 4, 4, dtype=F64, device=xi.device)
    A[..., :3, :3] = _hat(xi[..., :3]) + xi[..., 6, None, None] * torch.eye(3, dtype=F64, device=xi.device)
    A[..., :3, 3] = xi[..., 3:6]
    Q = torch.linalg.matrix_exp(A)
    s = torch.exp(xi[..., 6])
    return Q[..., :3, :3] / s[..., None, None], Q[..., :3, 3], s


def _integral(A):
    """integral_0^1 exp(tau A) d tau of [..., n, n]."""
    n = A.shape[-1]
    B = torch.zeros(*A.shape[:-2], 2 * n, 2 * n, dtype=F64, device=A.device)
    B[..., :n, :n] = A
    B[..., :n, n:] = torch.eye(n, dtype=F64, device=A.device)
    return torch.linalg.matrix_exp(B)[..., :n, n:]


def _ad(xi):
    A = torch.zeros(*xi.shape[:-1], 7, 7, dtype=F64, device=xi.device)
    W = _hat(xi[..., :3])
    A[..., :3, :3] = W
    A[..., 3:6, :3] = _hat(xi[..., 3:6])
    A[..., 3:6, 3:6] = W + xi[..., 6, None, None] * torch.eye(3, dtype=F64, device=xi.device)
    A[..., 3:6, 6] = -xi[..., 3:6]
    return A


def _left_jacobian(xi):
    return _integral(_ad(xi))


def _cams64(n, cam=CAM_752):
    return torch.tensor(cam[:4], dtype=F64, device=_dev()).expand(n, 4)


def _residuals(S, T, X, uv, cam, inverse=False):
    """p, q, r, |r| and the pairs in front of their keyframe."""
    M = _inverse(S) if inverse else S
    p = M[2] * (X @ M[0].T) + M[1]
    q = p if T is None else (T[:, :9].reshape(-1, 3, 3) @ p[..., None])[..., 0] + T[:, 9:]
    ok = q[:, 2] > 0
    z = torch.where(ok, q[:, 2], torch.ones_like(q[:, 2]))
    r = torch.stack([cam[:, 0] * q[:, 0] / z + cam[:, 2], cam[:, 1] * q[:, 1] / z + cam[:, 3]], -1) - uv
    r = torch.where(ok[:, None], r, torch.zeros_like(r))
    return p, q, z, r, r.norm(dim=-1), ok


def _terms(S, T, X, uv, cam, inverse=False, keep=None):
    """r, w, the Huber loss, g and H of the pairs (those of `keep`) at S."""
    cam = cam.expand(X.shape[0], 4)
    p, q, z, r, e, ok = _residuals(S, T, X, uv, cam, inverse)
    w = torch.where(e <= HUBER, torch.ones_like(e), HUBER / e.clamp(min=1e-300)) * ok
    rho = torch.where(e <= HUBER, 0.5 * e * e, HUBER * e - 0.5 * HUBER * HUBER) * ok
    zero = torch.zeros_like(z)
    D = torch.stack([cam[:, 0] / z, zero, -cam[:, 0] * q[:, 0] / z ** 2, zero, cam[:, 1] / z,
                     -cam[:, 1] * q[:, 1] / z ** 2], -1).reshape(-1, 2, 3)
    M = D if T is None else D @ T[:, :9].reshape(-1, 3, 3)
    P = p
    if inverse:
        M, P = -(M @ (S[0].T / S[2])), X
    J = torch.cat([-(M @ _hat(P)), M, M @ P[..., None]], -1)
    k = w if keep is None else w * keep
    g = ((k[:, None, None] * J) * r[..., None]).sum((0, 1))
    Jf = J.reshape(-1, 7)
    H = Jf.T @ (k.repeat_interleave(2)[:, None] * Jf)
    return r, w, (rho if keep is None else rho * keep).sum(), g, H


def _fma(a, b, c):
    """float32 fused multiply-add."""
    return (a.double() * b.double() + c.double()).float()


_POP = [bin(i).count("1") for i in range(256)]


def _accepted(st, k, e):
    """The accepted pairs of keyframe k (event e): point index in the batch, keypoint index in the batch.  The
    definition of the search by brute force over the keyframe's keypoints, in its float32 operations."""
    b, P, dev = st.batch, st.params, _dev()
    A = torch.from_numpy(b.h_kf_sim3[k]).to(dev)
    fx, fy, cx, cy, W, H = (torch.tensor(float(x), device=dev) for x in b.h_kf_K[k][:6])
    o0, o1 = (int(x) for x in b.h_pair_offset[k:k + 2])
    m0 = int(b.h_event_mp_offset[e])
    mp = m0 + (b.pair_mp[o0:o1].long() if b.pair_mp is not None else torch.arange(o1 - o0, device=dev))
    k0, k1 = (int(x) for x in b.h_kp_offset[k:k + 2])
    mp = mp[~torch.isin(b.mp_id[mp], b.kp_owner[k0:k1])]
    x, y, z = b.mp_xyz[mp].unbind(-1)
    q = [_fma(A[3 * i + 2], z, _fma(A[3 * i + 1], y, _fma(A[3 * i], x, A[9 + i]))) for i in range(3)]
    iz = (1.0 / q[2].double()).float()
    u, v = _fma(fx, q[0] * iz, cx), _fma(fy, q[1] * iz, cy)
    vis = (q[2] > 0) & (u >= 0) & (u < W) & (v >= 0) & (v < H)
    d = _fma(q[0], q[0], _fma(q[1], q[1], q[2] * q[2])).double().sqrt().float() * A[12]
    sf = torch.tensor([SCALE ** n for n in range(N_OCT)], dtype=F64, device=dev).float()
    hit = d[:, None] * sf >= b.mp_dmax[mp][:, None]
    pred = torch.where(hit.any(1), hit.float().argmax(1), N_OCT - 1)
    r = torch.tensor(P.win_px, dtype=torch.float32, device=dev) * sf[pred]
    mp, u, v, r, pred = (a[vis] for a in (mp, u, v, r, pred))
    kx, ky = b.kp_xy[k0:k1].unbind(-1)
    ko = b.kp_oct[k0:k1].long()
    pts, kps = [], []
    for c in range(0, mp.numel(), 16384):
        s = slice(c, c + 16384)
        lo, hi = (a[s, None] for a in (u - r, u + r))
        m = (kx >= lo) & (kx <= hi) & (ky >= (v - r)[s, None]) & (ky <= (v + r)[s, None])
        m &= (ko >= pred[s, None] - 1) & (ko <= pred[s, None])
        i, j = m.nonzero().unbind(-1)
        pts.append(i + c)
        kps.append(j)
    if not pts:
        return mp[:0], mp[:0]
    pts, kps = torch.cat(pts), torch.cat(kps)
    pop = torch.tensor(_POP, device=dev)
    h = pop[(b.mp_desc[mp[pts]] ^ b.kp_desc[k0 + kps]).long()].sum(-1)
    key = h * 65536 + kps
    none = 1 << 40
    best = torch.full((mp.numel(),), none, device=dev).scatter_reduce(0, pts, key, "amin")
    rest = torch.where(key == best[pts], none, h)
    second = torch.full((mp.numel(),), 0x7FFF, device=dev).scatter_reduce(0, pts, rest, "amin")
    bh = best // 65536
    ok = bh <= P.hamming_th
    if 0 < P.nn_ratio < 1:
        ok &= bh.float() < torch.tensor(P.nn_ratio, dtype=torch.float32, device=dev) * second.float()
    return mp[ok], k0 + best[ok] % 65536


def _refined(st, e):
    """The refined Sim3 of event e and the pairs of its last evaluation."""
    b, case, dev = st.batch, st.case, _dev()
    X, uv, T, cam = [], [], [], []
    for k in range(int(b.h_event_kf_offset[e]), int(b.h_event_kf_offset[e + 1])):
        mp, kp = _accepted(st, k, e)
        X.append(b.mp_xyz[mp].double())
        uv.append(b.kp_xy[kp].double())
        T.append(torch.from_numpy(b.h_kf_T[k]).to(dev).double().expand(mp.numel(), 12))
        cam.append(torch.from_numpy(b.h_kf_K[k][:4]).to(dev).double().expand(mp.numel(), 4))
    X, uv, T, cam = (torch.cat(a) for a in (X, uv, T, cam))
    S = _split(st.S0[e])
    iters, rounds, bound, lam0 = st.refine[0], max(st.refine[5], 1), st.refine[6], st.refine[7]
    other = None
    if case["refine"] == "two_sided":
        V = st.refine[8]
        s = slice(int(V.event_offset[e]), int(V.event_offset[e + 1]))
        kf = V.kf_idx[s].long()
        other = (V.kf_T[kf].double(), V.xyz[s].double(), V.uv[s].double(), V.kf_cam[kf].double())
    for rnd in range(rounds):
        keep = None
        if rnd:
            _, _, _, _, err, ok = _residuals(S, T, X, uv, cam)
            keep = (ok & (err <= float(np.float32(bound)))).double()
        acc = None
        for j in range(iters):
            _, _, loss, g, H = _terms(S, T, X, uv, cam, keep=keep)
            if other:
                _, _, _, g2, H2 = _terms(S, *other, inverse=True)
                g, H = g + g2, H + H2
            if lam0 == 0.0:
                S = _mul(_exp(-torch.linalg.solve(H, g)), S)
                continue
            if j == 0:
                acc, lam = (S, g, H, float(loss)), float(np.float32(lam0))
            else:
                rho = (acc[3] - float(loss)) / acc[3]
                if rho > 1e-6:
                    acc, lam = (S, g, H, float(loss)), max(lam * 0.1, 1e-12)
                elif rho >= -1e-6:
                    break
                else:
                    lam = min(lam * 10.0, 1e16)
            if j < iters - 1:
                S = _mul(_exp(-torch.linalg.solve(acc[2] + lam * torch.diag(acc[2].diagonal()), acc[1])), acc[0])
        if acc:
            S = acc[0]
    return S, 0


def _log(S):
    R, t, s = S
    v = 0.5 * torch.stack([R[..., 2, 1] - R[..., 1, 2], R[..., 0, 2] - R[..., 2, 0], R[..., 1, 0] - R[..., 0, 1]], -1)
    sn = v.norm(dim=-1)
    th = torch.atan2(sn, 0.5 * (R.diagonal(dim1=-2, dim2=-1).sum(-1) - 1.0))
    w = v * torch.where(th < 1e-4, 1 + th ** 2 / 6, th / sn.clamp(min=1e-300))[..., None]
    sig = torch.log(s)
    V = _integral(_hat(w) + sig[..., None, None] * torch.eye(3, dtype=F64, device=R.device))
    return torch.cat([w, torch.linalg.solve(V, t[..., None])[..., 0], sig[..., None]], -1)


def _adjoint(S):
    R, t, s = S
    A = torch.zeros(*s.shape, 7, 7, dtype=F64, device=R.device)
    A[..., :3, :3] = R
    A[..., 3:6, :3] = _hat(t) @ R
    A[..., 3:6, 3:6] = s[..., None, None] * R
    A[..., 3:6, 6] = -t
    A[..., 6, 6] = 1.0
    return A


def _graph_lm(st):
    """Levenberg-Marquardt on the dense normal equations, node 0 held (on the host)."""
    S, M = _split(st.S0.cpu()), _split(st.M.cpu())
    n, E = S[2].shape[0], len(st.edges)
    i, j = torch.from_numpy(st.edges.astype(np.int64)).T
    at = lambda P, k: (P[0][k], P[1][k], P[2][k])  # noqa: E731
    Mi = _inv(M)

    def err(P):
        Ed = _mul(Mi, _mul(at(P, j), _inv(at(P, i))))
        return Ed, _log(Ed)

    lam, cost = 1e-4, []
    Ed, e = err(S)
    F = float((e * e).sum())
    fresh = True
    for _ in range(st.case["iters"]):
        cost.append(F)
        if fresh:
            K = torch.linalg.inv(_left_jacobian(e))
            Jj, Ji = K @ _adjoint(Mi), -K @ _adjoint(Ed)
            g = torch.zeros(n, 7, dtype=F64)
            g.index_add_(0, i, (Ji.transpose(1, 2) @ e[..., None])[..., 0])
            g.index_add_(0, j, (Jj.transpose(1, 2) @ e[..., None])[..., 0])
            H = torch.zeros(n * n, 7, 7, dtype=F64)
            for a, Ja in ((i, Ji), (j, Jj)):
                for c, Jc in ((i, Ji), (j, Jj)):
                    H.index_add_(0, a * n + c, Ja.transpose(1, 2) @ Jc)
            H = H.reshape(n, n, 7, 7).transpose(1, 2).reshape(7 * n, 7 * n)[7:, 7:]
        L = H.clone()
        L.diagonal().mul_(1.0 + lam)
        d = torch.cholesky_solve(-g.reshape(-1)[7:, None], torch.linalg.cholesky(L))
        step = torch.cat([torch.zeros(1, 7, dtype=F64), d.reshape(n - 1, 7)])
        C = _mul(_exp(step), S)
        Ec, ec = err(C)
        Fc = float((ec * ec).sum())
        fresh = Fc < F
        if fresh:
            S, Ed, e, F, lam = C, Ec, ec, Fc, max(lam / 10, 1e-12)
        else:
            lam = min(lam * 10, 1e12)
    cost.append(F)
    out = torch.cat([S[0].reshape(n, 9), S[1], S[2][:, None]], 1)
    return {"S": out, "cost": torch.tensor(cost, dtype=F64), "used": None}
