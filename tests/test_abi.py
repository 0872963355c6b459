"""The C ABI library loads, exports every function include/fastloop.h
declares, and rejects invalid arguments on the host before any device work
(no GPU needed: fl_validate_batch is host-only)."""
import ctypes
import os
import re

import numpy as np
import pytest

import paper_2603_17201_amd as fl
from paper_2603_17201_amd import _abi

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "fastloop.h")


def declared():
    src = open(HEADER).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(fl_[a-z0-9_]+)\s*\(", src)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(fl.LIB_PATH):
        from paper_2603_17201_amd import build
        build.build()
    return fl.load()


def test_every_declared_symbol_is_exported(lib):
    names = declared()
    assert len(names) >= 18
    for n in names:
        assert hasattr(lib, n), n
    # and the binding declares exactly the header's functions
    assert sorted(s[0] for s in _abi.SIGNATURES) == names


def test_header_constants_match_binding():
    src = open(HEADER).read()
    for name, val in (("FL_MAX_PASSES", _abi.MAX_PASSES), ("FL_PGO_MAX_BAND_NODES", _abi.PGO_MAX_BAND_NODES),
                      ("FL_PGO_SOLVER_AUTO", _abi.PGO_SOLVER_AUTO), ("FL_PGO_SOLVER_CG", _abi.PGO_SOLVER_CG),
                      ("FL_PGO_SOLVER_DIRECT", _abi.PGO_SOLVER_DIRECT),
                      ("FL_PGO_SOLVER_DIRECT_WIDE", _abi.PGO_SOLVER_DIRECT_WIDE)):
        m = re.search(r"#define\s+%s\s+(\d+)" % name, src)
        assert m and int(m.group(1)) == val, name


def test_struct_sizes_match_header():
    assert ctypes.sizeof(_abi.Sim3) == 64
    assert ctypes.sizeof(_abi.Pinhole) == 32
    assert ctypes.sizeof(_abi.Params) == 32
    assert ctypes.sizeof(_abi.FuseOut) == 40
    assert ctypes.sizeof(_abi.Refine) == 56
    assert ctypes.sizeof(_abi.RefineInverse) == 56
    assert ctypes.sizeof(_abi.Pass) == 80
    assert ctypes.sizeof(_abi.PoseGraph) == 40
    assert ctypes.sizeof(_abi.PgoParams) == 64


def _batch(n_kf=2, n_mp=10, n_kp=(5, 7), dense=True):
    kp_off = np.concatenate([[0], np.cumsum(n_kp)]).astype(np.int32)
    pair_off = (np.arange(n_kf + 1) * n_mp).astype(np.int64)
    tables = dict(
        ekf=np.array([0, n_kf], np.int32), emp=np.array([0, n_mp], np.int32), kp_off=kp_off,
        pair_off=pair_off, sim3=np.zeros((n_kf, 16), np.float32),
        K=np.tile(np.array([458, 458, 367, 248, 752, 480, 0, 0], np.float32), (n_kf, 1)))
    b = _abi.Batch()
    b.n_events, b.n_kf, b.n_mp, b.n_kp_total, b.n_pairs = 1, n_kf, n_mp, int(kp_off[-1]), int(pair_off[-1])
    b.event_kf_offset = tables["ekf"].ctypes.data_as(ctypes.c_void_p)
    b.event_mp_offset = tables["emp"].ctypes.data_as(ctypes.c_void_p)
    b.kp_offset = tables["kp_off"].ctypes.data_as(ctypes.c_void_p)
    b.pair_offset = tables["pair_off"].ctypes.data_as(ctypes.c_void_p)
    b.kf_sim3 = tables["sim3"].ctypes.data_as(ctypes.c_void_p)
    b.kf_K = tables["K"].ctypes.data_as(ctypes.c_void_p)
    fake = 0x10000   # never dereferenced: validation is host-only
    for f in ("kp_xy", "kp_octave", "kp_desc", "kp_owner", "mp_xyz", "mp_desc"):
        setattr(b, f, fake)
    o = _abi.FuseOut(fake, fake, fake, fake, fake)
    P = _abi.Params(3.0, 1.2, 8, 64, 48, 50, 0.0, 0)
    return b, P, o, tables


def test_validate_accepts_a_consistent_batch(lib):
    b, P, o, t = _batch()
    assert lib.fl_validate_batch(ctypes.byref(b), ctypes.byref(P), ctypes.byref(o)) == 0


@pytest.mark.parametrize("case,code", [
    ("null_kp_xy", _abi.FL_EINVAL), ("negative_n_mp", _abi.FL_EINVAL), ("misaligned_desc", _abi.FL_EINVAL),
    ("grid_overflow", _abi.FL_ERANGE), ("octaves_33", _abi.FL_ERANGE), ("octaves_0", _abi.FL_ERANGE),
    ("too_many_kp", _abi.FL_ERANGE), ("nonfinite_K", _abi.FL_EINVAL), ("zero_width", _abi.FL_EINVAL),
    ("kp_offset_total", _abi.FL_EINVAL), ("pair_offset_dense", _abi.FL_EINVAL), ("flags", _abi.FL_EINVAL),
    ("win_nan", _abi.FL_EINVAL), ("event_offset_start", _abi.FL_EINVAL), ("null_output", _abi.FL_EINVAL),
    ("pairs_2_31", _abi.FL_ERANGE),
])
def test_validate_rejects(lib, case, code):
    b, P, o, t = _batch()
    if case == "null_kp_xy":
        b.kp_xy = None
    elif case == "negative_n_mp":
        b.n_mp = -1
    elif case == "misaligned_desc":
        b.mp_desc = 0x10004
    elif case == "grid_overflow":
        P.grid_cols, P.grid_rows = 100, 100
    elif case == "octaves_33":
        P.n_octaves = 33
    elif case == "octaves_0":
        P.n_octaves = 0
    elif case == "too_many_kp":
        t["kp_off"][1:] = [70000, 70007]
        b.n_kp_total = 70007
    elif case == "nonfinite_K":
        t["K"][1, 0] = np.inf
    elif case == "zero_width":
        t["K"][0, 4] = 0.0
    elif case == "kp_offset_total":
        b.n_kp_total = 99
    elif case == "pair_offset_dense":
        t["pair_off"][1] = 9
    elif case == "flags":
        P.flags = 1
    elif case == "win_nan":
        P.win_px = float("nan")
    elif case == "event_offset_start":
        t["ekf"][0] = 1
    elif case == "null_output":
        o.decision = None
    elif case == "pairs_2_31":
        b.n_pairs = 2 ** 31
    rc = lib.fl_validate_batch(ctypes.byref(b), ctypes.byref(P), ctypes.byref(o))
    assert rc == code, (case, rc, fl.last_error())
    assert fl.last_error()


def test_null_context_is_rejected(lib):
    P = _abi.Params(3.0, 1.2, 8, 64, 48, 50, 0.0, 0)
    K = _abi.Pinhole(458, 458, 367, 248, 752, 480)
    rc = lib.fl_build_grid(None, 0, None, ctypes.byref(K), ctypes.byref(P), None, None, None)
    assert rc == _abi.FL_EINVAL
    rc = lib.fl_set_stats(None, 1)
    assert rc == _abi.FL_EINVAL
    r = ctypes.c_double()
    rc = lib.fl_valu_rate(None, 100, ctypes.byref(r), None)
    assert rc == _abi.FL_EINVAL
    b, P, o, _tables = _batch()
    passes = (_abi.Pass * 2)(_abi.Pass(None, P, o), _abi.Pass(None, P, o))
    rc = lib.fl_search_fuse_passes(None, ctypes.byref(b), 2, passes, None)
    assert rc == _abi.FL_EINVAL
    assert lib.fl_sim3_inverse(None, None, None, None, None) == _abi.FL_EINVAL
    assert lib.fl_pose_graph_optimize(None, None, None, None) == _abi.FL_EINVAL


def test_missing_library_fails_loudly(tmp_path):
    with pytest.raises(RuntimeError):
        _abi._lib, saved = None, _abi._lib
        try:
            _abi.load(str(tmp_path / "nope.so"))
        finally:
            _abi._lib = saved


def test_refine_tags_never_repeat_between_clears(lib):
    # The refinement's partial-sum words carry a 32-bit tag of (launch epoch,
    # step); the epoch of launch L is -L mod 2^32.  Across every clear of the
    # rows and around the 2^22 wrap of the tag's epoch bits, two launches that
    # share a tag must have a clear between them.
    period = 1 << 22
    clears = [L for L in range(1, 3 * period + 8) if L % (period // 4) < 3 or L % period > period - 3
              if lib.fl_debug_refine_rows_cleared(L)]
    assert clears == [period, 2 * period, 3 * period]
    for step in (0, 7, 999):
        seen = {}
        last_clear = 0
        for L in list(range(1, 40)) + list(range(period - 40, period + 40)) + list(range(2 * period - 5, 2 * period + 40)):
            if lib.fl_debug_refine_rows_cleared(L):
                last_clear = L
            tag = lib.fl_debug_refine_tag((-L) & 0xFFFFFFFF, step)
            assert tag != 0   # a zeroed word never matches
            if tag in seen:
                assert seen[tag] < last_clear <= L, (L, seen[tag], last_clear)
            seen[tag] = L
    # launches one period apart share their tag (hence the clears)
    assert lib.fl_debug_refine_tag((-5) & 0xFFFFFFFF, 3) == lib.fl_debug_refine_tag((-5 - period) & 0xFFFFFFFF, 3)
    # distinct steps of one launch have distinct tags
    assert len({lib.fl_debug_refine_tag(12345, s) for s in range(1000)}) == 1000


def test_noalloc_search_rejects_what_its_scratch_cannot_hold(lib):
    # a keyframe of 30,000 keypoints needs more than the 1 MiB static scratch
    # of the allocation-free search: refused on the host, before any device
    # work (the pointers are never dereferenced)
    fake = 0x10000
    P = _abi.Params(3.0, 1.2, 8, 64, 48, 50, 0.0, 0)
    K = _abi.Pinhole(458, 458, 367, 248, 752, 480)
    S = _abi.Sim3()
    o = _abi.FuseOut(fake, fake, fake, fake, fake)
    kf = _abi.Keyframe(30000, fake, fake, fake, fake, None, None)
    rc = lib.fl_search_fuse_noalloc(100000, fake, fake, None, None, ctypes.byref(kf), ctypes.byref(S), ctypes.byref(K),
                                    ctypes.byref(P), ctypes.byref(o), None)
    assert rc == _abi.FL_ERANGE, (rc, fl.last_error())
    assert "scratch" in fl.last_error()
    # and argument errors are those of fl_search_fuse
    kf = _abi.Keyframe(100, None, fake, fake, fake, None, None)
    rc = lib.fl_search_fuse_noalloc(10, fake, fake, None, None, ctypes.byref(kf), ctypes.byref(S), ctypes.byref(K),
                                    ctypes.byref(P), ctypes.byref(o), None)
    assert rc == _abi.FL_EINVAL


def _plan(lib, tiles, weight, stage, slots):
    t = np.asarray(tiles, np.int64)
    w = np.asarray(weight, np.float32)
    bound = np.full(slots + 1, -1, np.int64)
    n = lib.fl_debug_plan_ranges(len(t), t.ctypes.data, w.ctypes.data, stage, slots, bound.ctypes.data)
    assert 1 <= n <= slots, (n, fl.last_error())
    return bound[:n + 1]


def _range_costs(bound, tiles, weight, stage):
    """Cost of each range: its tiles' weights, and `stage` for each keyframe it has tiles of."""
    first = np.concatenate([[0], np.cumsum(tiles)])
    lo = np.maximum(bound[:-1, None], first[None, :-1])
    hi = np.minimum(bound[1:, None], first[None, 1:])
    share = np.maximum(hi - lo, 0)
    return (share * np.asarray(weight)[None, :]).sum(1) + stage * (share > 0).sum(1)


def test_ranges_of_a_plan_cover_the_tiles_and_share_their_cost(lib):
    # No keyframe, keyframes without tiles, one tile a slot, as many keyframes
    # as slots and more, few and many tiles a slot, one dense keyframe among
    # sparse ones.  Every tile is in one range and the ranges rise.  Where the
    # longest range is minimised (no more keyframes than slots, at most 64
    # tiles a slot), it is at most the even share and the dearest keyframe's
    # staging and tile, or the 1.25 times that which is tried next.  Otherwise
    # a range costs at most one tile and the staging of the keyframe it begins
    # in more than the even share.
    stage = 36.0
    rng = np.random.default_rng(5)
    cases = [([], [], 256), ([0, 0], [2, 2], 256), ([1], [1.8], 256), ([256], [1.8], 256), ([257], [1.8], 256),
             ([5] * 256, [1.8] * 256, 256), ([5] * 257, [1.8] * 257, 256), ([3, 0, 70000, 2], [1.8, 9, 1.8, 40.0], 512),
             ([16384], [1.8], 256), ([16385], [1.8], 256), ([235] * 20, [1.8] * 20, 256), ([1] * 3, [1e3, 1, 1], 2),
             ([7], [1.8], 1), ([0, 7, 3], [1.8] * 3, 1)]
    for _ in range(400):
        n = int(rng.integers(1, 400))
        tiles = np.floor(np.exp(rng.uniform(0, rng.uniform(1, 8), n))).astype(np.int64) * (rng.random(n) > 0.1)
        cases.append((tiles, 1 + rng.exponential(2.0, n).astype(np.float32) * rng.choice([1, 10], n, p=[0.95, 0.05]),
                      int(rng.choice([1, 2, 7, 64, 256, 512]))))
    for tiles, weight, slots in cases:
        tiles = np.asarray(tiles, np.int64)
        weight = np.asarray(weight, np.float32).astype(np.float64)
        b = _plan(lib, tiles, weight, stage, slots)
        total, used = int(tiles.sum()), int((tiles > 0).sum())
        what = (used, total, slots)
        assert b[0] == 0 and b[-1] == total and np.all(np.diff(b) >= 0), what
        if total == 0:
            assert len(b) == 2, what
            continue
        if total <= slots:
            assert len(b) == total + 1 and np.all(np.diff(b) == 1), what
            continue
        cost = _range_costs(b, tiles, weight, stage)
        even = (stage * used + (tiles * weight).sum()) / slots
        top = stage + weight[tiles > 0].max()
        if used > slots or total > 64 * slots:
            assert cost.max() <= even * (1 + 1e-5) + top, what
        else:
            assert np.all(np.diff(b) > 0) and cost.max() <= 1.25 * (even + top) * (1 + 1e-5), what
