"""GPU parity of search-and-fuse against the CPU oracle: every output of every
pair bit-exact, for the plain per-keyframe path, the batched persistent path
and the graph-replayed path, on the hand-worked case, small ragged events,
the full loop-event workloads, multi-event batches, every tuning and the
list-overflow paths."""
import itertools

import numpy as np
import pytest
import torch

import oracle
import synth
from cases import conflict_case, hand_case, with_near_duplicates
from gpu_util import FIELDS, assert_same, dev, plain_per_keyframe, t

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2603_17201_amd as fl
    c = fl.Context(0)
    yield c
    c.close()


def batched(ctx, src, params=None, graph=False, use_dmax=True, use_id=True):
    import paper_2603_17201_amd as fl
    b = fl.DeviceBatch(src, device=dev(), use_dmax=use_dmax, use_id=use_id)
    p = params if params is not None else src.params
    out = ctx.search_fuse_graph(b, p) if graph else ctx.search_fuse_batched(b, p)
    return out.numpy()


def test_hand_case(ctx):
    ev, exp = hand_case()
    for mode in ("plain", "batched", "graph"):
        got = plain_per_keyframe(ctx, ev, ev.params) if mode == "plain" else batched(ctx, ev, graph=mode == "graph")
        assert_same(got, exp, mode)


@pytest.mark.parametrize("order", [list(p) for p in itertools.islice(itertools.permutations(range(6)), 0, 720, 181)])
def test_conflict_rule(ctx, order):
    ev = conflict_case(order)
    exp = oracle.search_fuse(ev)
    assert_same(plain_per_keyframe(ctx, ev, ev.params), exp, "plain")
    assert_same(batched(ctx, ev), exp, "batched")


@pytest.mark.parametrize("seed", range(10))
def test_tiny_events(ctx, seed):
    sparse = seed % 3 == 2
    ev = synth.gen_tiny(100 + seed, n_kf=1 + seed % 5, n_mp=37 + 61 * seed, n_kp=(3 + seed, 90 + 40 * seed),
                        sparse=sparse, skip_frac=0.05)
    for use_dmax, use_id in [(True, True), (False, True), (True, False)]:
        exp = oracle.search_fuse(ev, use_dmax=use_dmax, use_id=use_id)
        assert_same(batched(ctx, ev, use_dmax=use_dmax, use_id=use_id), exp, f"batched {seed} {use_dmax} {use_id}")
        assert_same(plain_per_keyframe(ctx, ev, ev.params, use_dmax, use_id), exp, f"plain {seed}")


def test_c1_single_call(ctx):
    ev = synth.gen_c1()
    exp = oracle.search_fuse(ev, use_grid=True)
    assert_same(plain_per_keyframe(ctx, ev, ev.params), exp, "plain")
    assert_same(plain_per_keyframe(ctx, ev, ev.params, with_grid=True), exp, "plain+grid")
    assert_same(batched(ctx, ev), exp, "batched")


@pytest.fixture(scope="module")
def c2():
    ev = synth.gen_c2(skip_frac=0.05)
    return ev, oracle.search_fuse(ev, use_grid=True)


def test_c2_plain(ctx, c2):
    ev, exp = c2
    assert_same(plain_per_keyframe(ctx, ev, ev.params), exp, "plain")


def test_c2_batched_and_graph(ctx, c2):
    ev, exp = c2
    assert_same(batched(ctx, ev), exp, "batched")
    for _ in range(3):   # replays of the captured graph
        assert_same(batched(ctx, ev, graph=True), exp, "graph")


def test_c2_every_tuning_and_repeat(ctx, c2):
    import paper_2603_17201_amd as fl
    ev, exp = c2
    b = fl.DeviceBatch(ev, device=dev())
    try:
        for ppl, mode, wpc, xa in itertools.product((1, 2, 4), (0, 1, 2), (1, 2), (0, 1)):
            ctx.set_tuning(ppl, mode, wpc, xa)
            got = ctx.search_fuse_batched(b, ev.params).numpy()
            assert_same(got, exp, f"tuning {ppl} {mode} {wpc} {xa}")
    finally:
        ctx.set_tuning()
    first = ctx.search_fuse_batched(b, ev.params).numpy()
    for _ in range(5):
        assert_same(ctx.search_fuse_batched(b, ev.params).numpy(), first, "repeat")


def test_c2_stats_match_oracle_counters(ctx, c2):
    import paper_2603_17201_amd as fl
    ev, exp = c2
    b = fl.DeviceBatch(ev, device=dev())
    ctx.set_stats(True)
    try:
        got = ctx.search_fuse_batched(b, ev.params).numpy()
        torch.cuda.synchronize()
        st = ctx.get_stats()
    finally:
        ctx.set_stats(False)
    assert_same(got, exp, "stats run")
    for k in ("n_visible", "n_cells", "n_kp_scanned", "n_cand"):
        assert st[k] == exp[k], (k, st[k], exp[k])


def test_list_overflow_paths(ctx):
    ev = synth.gen_c2(n_kf=4, n_mp=4000, skip_frac=0.02)
    exp = oracle.search_fuse(ev)
    ctx.debug_set_list_cap(16)
    try:
        assert_same(batched(ctx, ev), exp, "batched overflow")
        assert_same(plain_per_keyframe(ctx, ev, ev.params), exp, "plain overflow")
    finally:
        ctx.debug_set_list_cap(0)


def test_c3_sparse_pairs(ctx):
    ev = synth.gen_c3()
    exp = oracle.search_fuse(ev, use_grid=True)
    assert_same(batched(ctx, ev), exp, "c3 batched")
    assert_same(batched(ctx, ev, graph=True), exp, "c3 graph")


def test_multi_event_batch(ctx):
    evs = [synth.gen_c3(seed=310 + i, n_kf=8 + 5 * i, n_mp=3000 + 1000 * i, id_base=1000 + 10 ** 6 * i,
                        fresh_base=10 ** 9 + 10 ** 7 * i) for i in range(3)]
    evs.append(synth.gen_tiny(55, n_kf=3, n_mp=500))
    B = synth.concat_events(evs)
    exp = oracle.search_fuse(B, use_grid=True)
    assert_same(batched(ctx, B), exp, "multi batched")
    assert_same(batched(ctx, B, graph=True), exp, "multi graph")


def test_edge_cases(ctx):
    import paper_2603_17201_amd as fl
    ev = synth.gen_tiny(7, n_kf=3, n_mp=150, n_kp=(20, 40))
    # NaN / Inf coordinates and a point behind every camera
    X = ev.mp_xyz.copy()
    X[0] = [np.nan, 0, 1]
    X[1] = [0, 0, np.inf]
    X[2] = [0, 0, -1e6]
    ev.mp_xyz = X
    exp = oracle.search_fuse(ev)
    assert_same(batched(ctx, ev), exp, "nonfinite")
    assert_same(plain_per_keyframe(ctx, ev, ev.params), exp, "nonfinite plain")
    # an empty keyframe in the middle of a batch
    n0, n1 = int(ev.kp_offset[1]), int(ev.kp_offset[2])
    keep = np.r_[0:n0, n1:int(ev.kp_offset[-1])]
    ev.kp_offset = np.array([0, n0, n0, n0 + int(ev.kp_offset[-1]) - n1], np.int32)
    ev.kp_xy, ev.kp_oct, ev.kp_desc, ev.kp_owner = (ev.kp_xy[keep], ev.kp_oct[keep], ev.kp_desc[keep],
                                                    ev.kp_owner[keep])
    exp = oracle.search_fuse(ev)
    assert_same(batched(ctx, ev), exp, "empty keyframe")
    assert_same(plain_per_keyframe(ctx, ev, ev.params), exp, "empty keyframe plain")
    # sparse pairs naming points outside the event
    sp = synth.gen_tiny(8, n_kf=2, n_mp=60, n_kp=(10, 30), sparse=True)
    sp.pair_mp = sp.pair_mp.copy()
    sp.pair_mp[0] = -5
    sp.pair_mp[-1] = 60
    exp = oracle.search_fuse(sp)
    assert exp["decision"][0] == oracle.INVALID
    assert_same(batched(ctx, sp), exp, "invalid pairs")
    # no pairs at all
    b = fl.DeviceBatch(ev, device=dev())
    b.h_pair_offset = np.zeros_like(b.h_pair_offset)
    b.n_pairs = 0
    b.pair_mp = t(np.zeros(1, np.int32))
    out = ctx.search_fuse_batched(b, ev.params)
    assert out.decision.numel() == 0


def test_grid_build_matches_definition(ctx):
    ev = synth.gen_c3(n_kf=4, n_mp=2000)
    p = ev.params
    for k in range(ev.n_kf):
        a, b = int(ev.kp_offset[k]), int(ev.kp_offset[k + 1])
        xy = ev.kp_xy[a:b]
        cs, ck = ctx.build_grid(t(xy), ev.cams[k], p)
        cs, ck = cs.cpu().numpy(), ck.cpu().numpy()
        ecs, eck = oracle.build_grid(xy, ev.cams[k], p)
        assert np.array_equal(cs, ecs) and np.array_equal(ck, eck)


def test_host_validation_errors(ctx):
    import paper_2603_17201_amd as fl
    ev = synth.gen_tiny(9, n_kf=2, n_mp=50)
    b = fl.DeviceBatch(ev, device=dev())
    bad = synth.LoopParams(n_octaves=40)
    with pytest.raises(fl.FlError) as e:
        ctx.search_fuse_batched(b, bad)
    assert e.value.code == -4
    with pytest.raises(ValueError):   # host tensor where a device tensor is required
        ctx.search_fuse(torch.zeros((4, 3)), t(np.zeros((4, 32), np.uint8)), None, None,
                        t(np.zeros((1, 2), np.float32)), t(np.zeros(1, np.int8)), t(np.zeros((1, 32), np.uint8)),
                        t(np.zeros(1, np.int32)), np.zeros(16, np.float32), ev.cams[0], ev.params)


def test_valu_rate_probe(ctx):
    # the issue-rate probe used for roofline reporting: a plausible rate
    # (between 1 and 200 T lane-ops/s) and its argument range enforced
    rate = ctx.valu_rate(iters=2000)
    assert 1e12 < rate < 2e14, rate
    import paper_2603_17201_amd as fl
    with pytest.raises(ValueError):
        ctx.valu_rate(iters=0)
    assert fl.last_error()


def test_staging_ring_reuse_with_changing_tables(ctx):
    # 60 eager calls cycling through three batches: every call uploads new
    # tables, so each staging buffer is rewritten several times, each time
    # after a fence that follows its previous fetch; every result must hold
    import paper_2603_17201_amd as fl
    evs = [synth.gen_tiny(70 + i, n_kf=2 + i, n_mp=300 + 50 * i) for i in range(3)]
    exps = [oracle.search_fuse(ev) for ev in evs]
    bs = [fl.DeviceBatch(ev, device=dev()) for ev in evs]
    outs = [fl.FuseOutputs.empty(b.n_pairs, dev()) for b in bs]
    for it in range(60):
        i = it % 3
        ctx.search_fuse_batched(bs[i], evs[i].params, outs[i])
        if it % 7 == 0 or it >= 57:
            assert_same(outs[i].numpy(), exps[i], f"call {it}")


def test_graph_ring_reuse_with_changing_tables(ctx):
    # 30 graph launches cycling through three batches of one shape (so the
    # captured graphs are reused): each graph's table buffer is rewritten
    # after a fence that follows its previous replay; every result must hold
    import paper_2603_17201_amd as fl
    evs = [synth.gen_tiny(80 + i, n_kf=3, n_mp=400) for i in range(3)]
    exps = [oracle.search_fuse(ev) for ev in evs]
    bs = [fl.DeviceBatch(ev, device=dev()) for ev in evs]
    outs = [fl.FuseOutputs.empty(b.n_pairs, dev()) for b in bs]
    for it in range(30):
        i = it % 3
        ctx.search_fuse_graph(bs[i], evs[i].params, outs[i])
        if it % 4 == 0 or it >= 27:
            assert_same(outs[i].numpy(), exps[i], f"graph call {it}")


def _accepted(o):
    return int(((o["decision"] == oracle.ADD) | (o["decision"] == oracle.FUSE)).sum())


def test_projection_search_one_keyframe(ctx):
    """Loop verification's single projection search: every point against one
    keyframe with near-duplicate keypoints, the wider window and the ratio
    test on; the plain call and a batched launch, bit-exact."""
    ev = with_near_duplicates(synth.gen_c1())
    P = synth.verification_params()
    exp = oracle.search_fuse(ev, params=P)
    loose = oracle.search_fuse(ev, params=synth.LoopParams(win_px=P.win_px))
    assert _accepted(exp) < _accepted(loose)   # the ratio test rejects some matches here
    assert_same(plain_per_keyframe(ctx, ev, P), exp, "PS1 plain")
    assert_same(batched(ctx, ev, params=P), exp, "PS1 batched")
    assert_same(batched(ctx, ev, params=P, graph=True), exp, "PS1 graph")


def test_projection_search_three_keyframes_one_launch(ctx):
    """Loop verification's triple projection search in one launch: the same
    points against three keyframes (one event, dense pairs), and three
    independent one-keyframe searches batched together; ratio test on."""
    P = synth.verification_params()
    ev = synth.gen_c2(seed=212, n_kf=3, n_mp=15000)
    exp = oracle.search_fuse(ev, params=P, use_grid=True)
    assert_same(batched(ctx, ev, params=P), exp, "PS3 one event")
    assert_same(batched(ctx, ev, params=P, graph=True), exp, "PS3 one event, graph")
    evs = [with_near_duplicates(synth.gen_c1(seed=101 + i), seed=7 + i) for i in range(3)]
    B = synth.concat_events(evs)
    exp3 = oracle.search_fuse(B, params=P)
    assert _accepted(exp3) < _accepted(oracle.search_fuse(B, params=synth.LoopParams(win_px=P.win_px)))
    assert_same(batched(ctx, B, params=P), exp3, "PS3 three events")


def test_c2_with_ratio_test(ctx):
    """The full loop event with the ratio test on (0.75) and the fusion
    window."""
    ev = synth.gen_c2()
    P = synth.LoopParams(nn_ratio=0.75)
    exp = oracle.search_fuse(ev, params=P, use_grid=True)
    assert_same(batched(ctx, ev, params=P), exp, "c2 ratio")


def test_keyframe_at_the_packed_key_limit(ctx):
    # a keyframe of FL_MAX_KP = 65,535 keypoints (the 16-bit index of the
    # packed key) between two ordinary ones: too large for LDS, so the
    # batched launch takes its global-grid mode; the plain path runs each
    # keyframe on its own
    import paper_2603_17201_amd as fl
    ev = synth.gen_c2(seed=515, n_mp=4000, kp_counts=[1200, fl.MAX_KP, 1200])
    exp = oracle.search_fuse(ev, use_grid=True)
    assert int(exp["best_idx"].max()) > 60000   # indices near the limit are matched
    assert_same(batched(ctx, ev), exp, "batched")
    assert_same(batched(ctx, ev, graph=True), exp, "graph")
    assert_same(plain_per_keyframe(ctx, ev, ev.params), exp, "plain")


@pytest.mark.parametrize("big", [6000, 20000])
def test_one_large_keyframe_among_small_ones(ctx, big):
    # one keyframe of `big` keypoints among 1,200-keypoint ones: the LDS
    # footprint is sized by the largest, so the launch stages fewer octave
    # buckets (6,000) or falls back to global grids (20,000) for every
    # keyframe; every tuning stays bit-exact
    ev = synth.gen_c2(seed=616 + big, n_mp=3000, kp_counts=[1200, 1200, big, 1200, 1200])
    exp = oracle.search_fuse(ev, use_grid=True)
    saved = ctx.get_tuning()
    try:
        for ppl, mode in itertools.product((1, 2, 4), (0, 1, 2)):
            ctx.set_tuning(ppl, mode, 1, 1)
            assert_same(batched(ctx, ev), exp, f"ppl {ppl} mode {mode}")
    finally:
        ctx.set_tuning(saved.pairs_per_lane, saved.lds_mode, saved.wg_per_cu, saved.xcd_aware)


@pytest.mark.parametrize("win", [12.0, 25.0, 90.0])
def test_windows_of_many_rows(ctx, win):
    # windows of 3 to 65 grid rows (10 pixels each, octaves 0 to 7): the scan
    # takes four rows at a time, the lanes of a wave with different numbers
    import dataclasses
    ev = synth.gen_tiny(41, n_kf=3, n_mp=700, n_kp=(150, 260), skip_frac=0.05)
    P = dataclasses.replace(ev.params, win_px=win)
    exp = oracle.search_fuse(ev, params=P)
    assert_same(plain_per_keyframe(ctx, ev, P), exp, "plain")
    saved = ctx.get_tuning()
    try:
        for ppl, mode in itertools.product((1, 4), (0, 1, 2)):
            ctx.set_tuning(ppl, mode, 1, 1)
            assert_same(batched(ctx, ev, params=P), exp, f"ppl {ppl} mode {mode}")
            assert_same(batched(ctx, ev, params=P, use_dmax=False), oracle.search_fuse(ev, params=P, use_dmax=False),
                        f"no gate, ppl {ppl} mode {mode}")
    finally:
        ctx.set_tuning(saved.pairs_per_lane, saved.lds_mode, saved.wg_per_cu, saved.xcd_aware)


@pytest.mark.parametrize("wg_per_cu", [1, 2])
def test_accepted_pairs_of_every_event_are_counted(ctx, wg_per_cu):
    # 330 keyframes of 110 events, more than there are workgroups: most
    # workgroups take several events, large events several workgroups, and
    # every seventh event accepts nothing; the refinement finds each event's
    # accepted pairs among the workgroups' lists
    import paper_2603_17201_amd as fl
    evs = []
    for i in range(110):
        e = synth.gen_tiny(500 + i, n_kf=3, n_mp=2500 if i % 10 == 3 else 70 + 13 * (i % 9), n_kp=(20, 60),
                           sparse=i % 4 == 2)
        if i % 7 == 0:
            e.kp_desc = e.kp_desc ^ np.uint8(0xFF)   # every distance far above the threshold
        evs.append(e)
    B = synth.concat_events(evs)
    exp = oracle.search_fuse(B)
    accepted = np.isin(exp["decision"], (2, 3))   # ADD, FUSE
    kf_pairs = np.add.reduceat(np.append(accepted, False), B.pair_offset[:-1].astype(np.int64))
    kf_pairs[np.diff(B.pair_offset) == 0] = 0
    n_ref = np.array([kf_pairs[a:b].sum() for a, b in zip(B.event_kf_offset[:-1], B.event_kf_offset[1:])])
    assert (n_ref == 0).sum() >= 16 and n_ref.max() > 20
    b = fl.DeviceBatch(B, device=dev())
    S0 = np.stack([e.S_init for e in evs])
    saved = ctx.get_tuning()
    try:
        ctx.set_tuning(saved.pairs_per_lane, saved.lds_mode, wg_per_cu, saved.xcd_aware)
        for run in (ctx.search_fuse_batched, ctx.search_fuse_graph):
            nm = torch.full((110,), -7, dtype=torch.int32, device=dev())
            got = run(b, B.params, refine=(1, 2.45, t(S0.copy()), None, nm)).numpy()
            assert_same(got, exp, run.__name__)
            # a step counts the pairs in front of their keyframe: all accepted ones, or
            # none (-1) where its system is singular
            n = nm.cpu().numpy()
            assert ((n == n_ref) | (n == -1) & (n_ref < 4)).all(), (n[n != n_ref], n_ref[n != n_ref])
    finally:
        ctx.set_tuning(saved.pairs_per_lane, saved.lds_mode, saved.wg_per_cu, saved.xcd_aware)


@pytest.mark.parametrize("n_kp", [1, 1023, 1024, 1025, 8192, 8193])
def test_plain_search_over_keypoint_counts(ctx, n_kp):
    # one keypoint a thread, a second one, and the last list that is put
    # together on the chip; windows of up to eight rows, grid given or not
    import dataclasses
    ev = synth.gen_tiny(77, n_kf=1, n_mp=333, n_kp=(n_kp, n_kp), skip_frac=0.1)
    P = dataclasses.replace(ev.params, win_px=10.0)
    exp = oracle.search_fuse(ev, params=P)
    for with_grid in (False, True):
        assert_same(plain_per_keyframe(ctx, ev, P, with_grid=with_grid), exp, f"grid given: {with_grid}")
    cs, ck = ctx.build_grid(t(ev.kp_xy), ev.cams[0], P)
    cs_ref, ck_ref = oracle.build_grid(ev.kp_xy, ev.cams[0], P)
    assert np.array_equal(cs.cpu().numpy(), cs_ref) and np.array_equal(ck.cpu().numpy(), ck_ref)


def test_plain_search_of_more_points_than_a_launch_has_lanes_for(ctx):
    """2^29 + 300 points, eight lanes each, are more threads than one launch
    may have: the event's points at both ends and across the 2^28th and the
    2^29th, all others behind the keyframe, against the search of those points
    alone (the claims of one keypoint from both ends among them)."""
    import paper_2603_17201_amd as fl
    n = (1 << 29) + 300
    if torch.cuda.mem_get_info(dev())[0] < 80 << 30:
        pytest.skip("needs 40 GB of device memory")
    ev = synth.gen_c2(seed=311, n_kf=1, n_mp=2000, n_kp=800)
    at = [(0, 500), ((1 << 28) - 250, (1 << 28) + 250), ((1 << 29) - 250, n)]
    m = sum(b - a for a, b in at)
    # every point twice, at two of the places
    pick = np.concatenate([np.arange(m // 2), np.arange(m - m // 2)])
    x, d = np.ascontiguousarray(ev.mp_xyz[pick]), np.ascontiguousarray(ev.mp_desc[pick])
    rest = (t(ev.kp_xy), t(ev.kp_oct), t(ev.kp_desc), t(ev.kp_owner), ev.kf_sim3[0], ev.cams[0], ev.params)
    ids = np.arange(m, dtype=np.int32) + 10 ** 9
    exp = ctx.search_fuse(t(x), t(d), None, t(ids), *rest).numpy()
    assert (exp["decision"] == oracle.ADD).sum() > 50
    # the others behind the keyframe
    A, c = np.float64(ev.kf_sim3[0][:9]).reshape(3, 3), np.float64(ev.kf_sim3[0][9:12])
    X = t(np.linalg.solve(A, np.array([0.0, 0.0, -5.0]) - c).astype(np.float32)).repeat(n, 1)
    D = torch.zeros((n, 32), dtype=torch.uint8, device=dev())
    I = torch.full((n,), -1, dtype=torch.int32, device=dev())
    o = 0
    for a, b in at:
        X[a:b], D[a:b], I[a:b] = t(x[o:o + b - a]), t(d[o:o + b - a]), t(ids[o:o + b - a])
        o += b - a
    out = ctx.search_fuse(X, D, None, I, *rest)
    none = dict(best_idx=-1, best_dist=0x7FFF, second_dist=0x7FFF, decision=oracle.NOT_VISIBLE, target=-1)
    for f in FIELDS:
        got = getattr(out, f)
        assert np.array_equal(np.concatenate([got[a:b].cpu().numpy() for a, b in at]), exp[f]), f
        for a, b in at:
            got[a:b] = none[f]
        assert bool((got == none[f]).all()), f


def test_claimed_and_helped_tiles_of_several_events_and_passes(ctx):
    # 27,000 tiles of four events over 256 workgroups: ranges long enough that
    # their second half is claimed, some within one event (others help with
    # them) and some across two or three; eager with refinement, and in two
    # passes (twice the tiles), the second with windows of several rows
    import paper_2603_17201_amd as fl
    B = synth.concat_events([synth.gen_c2(seed=231, n_kf=2, n_mp=400), synth.gen_c2(seed=232, n_kf=5, n_mp=200000),
                             synth.gen_c2(seed=233, n_kf=3, n_mp=2000), synth.gen_c2(seed=234, n_kf=4, n_mp=180000)])
    exp = oracle.search_fuse(B, use_grid=True)
    accepted = np.isin(exp["decision"], (oracle.ADD, oracle.FUSE))
    n_ref = [int(accepted[int(B.pair_offset[a]):int(B.pair_offset[z])].sum())
             for a, z in zip(B.event_kf_offset[:-1], B.event_kf_offset[1:])]
    b = fl.DeviceBatch(B, device=dev())
    assert b.n_pairs / 64 / 256 > 96
    for run in (ctx.search_fuse_batched, ctx.search_fuse_graph):
        S = t(np.stack([e.S_init for e in B.events]))
        nm = torch.zeros(4, dtype=torch.int32, device=dev())
        assert_same(run(b, B.params, refine=(1, 2.45, S, None, nm)).numpy(), exp, run.__name__)
        assert nm.cpu().tolist() == n_ref, run.__name__
    P2 = synth.verification_params()
    exp2 = oracle.search_fuse(B, params=P2, use_grid=True)
    outs = ctx.search_fuse_passes(b, [(B.params, None, None), (P2, None, None)])
    for o, e in zip(outs, (exp, exp2)):
        assert_same(o.numpy(), e, "passes")
