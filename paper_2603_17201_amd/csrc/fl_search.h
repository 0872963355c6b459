// Search-and-fuse kernels: the fused batched search, its global-grid
// fallback, the plain per-keyframe search and ADD-conflict resolution.
//
// Loop fusion (paper Sec. III-B, Sec. IV-D3): every map point of the loop
// region is projected through the corrected Sim3 into each connected
// keyframe; keypoints inside a window whose size follows the point's
// predicted octave are compared by 256-bit Hamming distance and the point is
// fused into an owned keypoint or added to a free one.  The work is
// independent per (point, keyframe) pair; the only coupling is several
// points claiming one free keypoint, resolved by the lowest point index.
#pragma once

#include "fl_internal.h"

namespace fl {

constexpr uint8_t kDecUndecided = 0xFF;
constexpr int kSearchBlock = 1024;   // threads of a batched-search workgroup (16 waves)
constexpr int kWavesPerWG = kSearchBlock / 64;

struct SearchConst {
    float sf[32];
    int N;
    int gate;
    int C, R;
    int th;
    float ratio;
    float r0;
};

__device__ __forceinline__ void load_desc(const uint8_t* __restrict__ base, int64_t row, uint4& a, uint4& b) {
    const uint4* p = reinterpret_cast<const uint4*>(base + row * 32);
    a = ldg_u4(p);
    b = ldg_u4(p + 1);
}

__device__ __forceinline__ bool accept_match(const Best& b, int th, float ratio) {
    if (b.key == 0xFFFFFFFFu) return false;
    const int bh = (int)(b.key >> 16);
    if (bh > th) return false;
    if (ratio > 0.0f && ratio < 1.0f) return (float)bh < ratio * (float)b.second;
    return true;
}

// Window box and cell range of a visible point.
struct Window {
    float lx, hx, ly, hy;
    int c0, c1, r0, r1;
};

__device__ __forceinline__ Window make_window(const Proj& p, const KfDesc& kd, const float* sf, float r0w, int C,
                                              int R) {
    Window w;
    const float rad = r0w * sf[p.pred];
    w.lx = p.u - rad;
    w.hx = p.u + rad;
    w.ly = p.v - rad;
    w.hy = p.v + rad;
    w.c0 = cell_of(w.lx, kd.invw, C);
    w.c1 = cell_of(w.hx, kd.invw, C);
    w.r0 = cell_of(w.ly, kd.invh, R);
    w.r1 = cell_of(w.hy, kd.invh, R);
    return w;
}

// Closed box and octave gate, evaluated without branches.
__device__ __forceinline__ bool in_window(const Window& w, float x, float y, int oct, int pred, int gate) {
    const bool box = (x >= w.lx) & (x <= w.hx) & (y >= w.ly) & (y <= w.hy);
    const bool oct_ok = (gate == 0) | ((oct >= pred - 1) & (oct <= pred));
    return box & oct_ok;
}

__device__ __forceinline__ uint32_t owner_slot(int32_t id, int32_t mask) {
    return (hash_id(id) >> 7) & (uint32_t)mask;
}

// Insert an owner id into an open-addressing set with at least one free slot.
__device__ __forceinline__ void owner_insert(int32_t* tab, int32_t mask, int32_t o) {
    uint32_t hh = owner_slot(o, mask);
    for (int probe = 0; probe <= mask; ++probe) {
        const int32_t prev = atomicCAS(&tab[hh], -1, o);
        if (prev == -1 || prev == o) return;
        hh = (hh + 1) & (uint32_t)mask;
    }
}

// Workgroup exclusive scan of a[0..n) in place (n may exceed blockDim): each
// thread sums a run of consecutive elements, the runs are scanned inside each
// wave and the wave totals by wave 0.  s_tmp needs blockDim / 64 + 1 ints
// (s_tmp[blockDim / 64] = total); blockDim is a multiple of 64, at most 4096.
__device__ void block_exclusive_scan(int32_t* a, int n, int32_t* s_tmp) {
    const int tid = threadIdx.x, nt = blockDim.x;
    const int lane = wave_lane(), wid = tid / kWave, nw = nt / kWave;
    const int chunk = (n + nt - 1) / nt;
    const int b = min(tid * chunk, n), e = min(b + chunk, n);
    constexpr int kRun = 4;   // runs up to this length are loaded at once
    int v[kRun];
    int sum = 0;
    if (chunk <= kRun) {
#pragma unroll
        for (int j = 0; j < kRun; ++j) v[j] = b + j < e ? a[b + j] : 0;
#pragma unroll
        for (int j = 0; j < kRun; ++j) sum += v[j];
    } else {
        for (int i = b; i < e; ++i) sum += a[i];
    }
    const int incl = wave_incl_scan(sum);
    if (lane == kWave - 1) s_tmp[wid] = incl;
    __syncthreads();
    if (wid == 0) {
        const int t = lane < nw ? s_tmp[lane] : 0;
        const int x = wave_incl_scan(t);
        if (lane < nw) s_tmp[lane] = x - t;
        if (lane == nw - 1) s_tmp[nw] = x;
    }
    __syncthreads();
    int run = s_tmp[wid] + incl - sum;
    if (chunk <= kRun) {
#pragma unroll
        for (int j = 0; j < kRun; ++j)
            if (b + j < e) {
                a[b + j] = run;
                run += v[j];
            }
    } else {
        for (int i = b; i < e; ++i) {
            const int x = a[i];
            a[i] = run;
            run += x;
        }
    }
    __syncthreads();
}

// 16-byte units of the 16-bit octave-bucket counts in LDS, and the bytes of
// the bucket starts: those units behind one more, whose last entry is the
// first start (0).  The counts alone are a whole number of units a thread
// (64 x 48 cells of 8 groups: 3).
__host__ __device__ inline int search_cs_units(int cells, int nb) { return (int)(((size_t)cells * nb + 7) / 8); }
__host__ __device__ inline size_t search_cs_bytes(int cells, int nb) {
    return 16 * (size_t)(search_cs_units(cells, nb) + 1);
}
constexpr int kCsFirst = 7;   // entry of the first start in the leading unit

// Exclusive scan by a workgroup of kSearchBlock threads of n4 groups of four
// words, each word a packed pair of 16-bit counts, in place (low half first):
// a word becomes (P, P + lo) for P the sum of every count before it.  Every
// sum must stay below 65536, so the halves never carry into each other and
// both are added in one instruction: with four waves on a SIMD the vector
// instructions bound this scan, one for a word's share of the sum and four
// for its result.  Each thread takes a run of consecutive groups: with
// 16-byte accesses at strides of 16, 32 or 48 bytes a wave's lanes share no
// bank, and the groups of a short run stay in registers between the two
// passes.  s_tmp needs one int a wave.
__device__ __forceinline__ void block_exclusive_scan_u16(uint4* w, int n4, int32_t* s_tmp) {
    constexpr int nt = kSearchBlock;
    const int tid = threadIdx.x;
    const int lane = wave_lane(), wid = tid / kWave;
    const int chunk = (n4 + nt - 1) / nt;
    const int b = min(tid * chunk, n4), e = min(b + chunk, n4);
    constexpr int kRun = 3;
    uint4 v[kRun];
#pragma unroll
    for (int j = 0; j < kRun; ++j) v[j] = b + j < e ? w[b + j] : make_uint4(0, 0, 0, 0);
    uint32_t both = 0;
#pragma unroll
    for (int j = 0; j < kRun; ++j) both += (v[j].x + v[j].y) + (v[j].z + v[j].w);
    for (int i = b + kRun; i < e; ++i) both += (w[i].x + w[i].y) + (w[i].z + w[i].w);
    const int sum = (int)((both & 0xFFFFu) + (both >> 16));
    const int incl = wave_incl_scan(sum);
    if (lane == kWave - 1) s_tmp[wid] = incl;
    __syncthreads();
    const int before = __builtin_amdgcn_readlane(wave_incl_scan(lane < wid ? s_tmp[lane] : 0), kWave - 1);
    uint32_t run = (uint32_t)(before + incl - sum) * 0x10001u;   // in both halves
    auto put = [&](int i, uint4 x) {
        auto word = [&](uint32_t& y) {
            const uint32_t c = y;
            y = run + (c << 16);
            run += c + __builtin_amdgcn_alignbit(c, c, 16);
        };
        word(x.x);
        word(x.y);
        word(x.z);
        word(x.w);
        w[i] = x;
    };
#pragma unroll
    for (int j = 0; j < kRun; ++j)
        if (b + j < e) put(b + j, v[j]);
    for (int i = b + kRun; i < e; ++i) put(i, w[i]);
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Keyframe grid in LDS by octave group.  With the octave gate on, a pair
// whose point is predicted at octave p has as candidates the keypoints of
// octaves p - 1 and p; group g = min(p, nb - 1) holds exactly those
// keypoints for g < nb - 1, and the last group every octave from nb - 2 up,
// so a pair reads the cells of one group.  A keypoint of octave o therefore
// sits in up to two groups (o and o + 1 below nb - 1, the last group from
// o = nb - 2 up; octaves below -1 can never be candidates).  With nb = 1
// (the gate off, or too little LDS) group 0 is the plain grid of every
// keypoint.  Slots are ordered by row, then group, then column, so a pair's
// candidates are one run of slots per grid row.  Histogram of the (row,
// group, column) cells (16-bit counts, two per 32-bit word), exclusive scan,
// scatter of slot-ordered records (and descriptors), owner hash set.  On
// return s_cs[j] is the first slot of cell j and s_cs[R * nb * C] the
// number of slots (below 65536).  The order of the records inside a cell is
// arbitrary: the packed (distance, index) key makes every output
// independent of it.

// The groups of a keypoint of octave o: a (or -1) and b (or -1).
__device__ __forceinline__ void groups_of(int o, int nb, int& a, int& b) {
    if (nb == 1) {
        a = 0;
        b = -1;
        return;
    }
    a = (o >= 0 && o <= nb - 2) ? o : -1;
    b = (o + 1 >= 0 && o + 1 <= nb - 2) ? o + 1 : (o >= nb - 2 ? nb - 1 : -1);
}

// 16-bit entry j of a packed array, incremented; returns its old value.
__device__ __forceinline__ int u16_fetch_add(uint32_t* w, int j) {
    const int sh = (j & 1) * 16;
    return (int)((atomicAdd(&w[j >> 1], 1u << sh) >> sh) & 0xFFFFu);
}

// The first kStagePre keypoints of a thread are loaded once, before the LDS
// is cleared and the keyframe's descriptor is there, and kept for the scatter.
// Clearing and scan move 16 bytes at a time.  At 1,000 keypoints and 64 x 48
// cells of 8 groups (48 KB of counts) the staging takes 8,800 cycles; with
// 4-byte accesses and the keypoints loaded where they are used it took 13,000.
constexpr int kStagePre = 2;

// What the staging needs of a keyframe.
struct StageKf {
    int32_t kp_off, n_kp;
    float invw, invh;
};

struct StageKp {
    float x, y;
    int oct, own;
    int ca, cb;   // its cells in up to two groups, or -1
};

// The launch's constants of the staging.
struct StageEnv {
    const float* xy;
    const int8_t* oct;
    const int32_t* own;
    const uint8_t* desc;
    int C, R, nb, hmask;
    __device__ __forceinline__ StageKp load(const StageKf& k, int i) const {
        const int64_t g = (int64_t)k.kp_off + i;
        return {ldg(xy + 2 * g), ldg(xy + 2 * g + 1), (int)ldg(oct + g), ldg(own + g), -1, -1};
    }
};

__device__ __forceinline__ void stage_load(const StageEnv& env, const StageKf& kd, StageKp* pre) {
#pragma unroll
    for (int j = 0; j < kStagePre; ++j) {
        const int i = (int)threadIdx.x + j * kSearchBlock;
        if (i < kd.n_kp) pre[j] = env.load(kd, i);
    }
}

template <bool STAGE_DESC>
__device__ __forceinline__ void stage_build(const StageEnv& env, const StageKf& kd, StageKp* pre, uint4* s_cs,
                                            KpRec* s_rec, uint4* s_desc, int32_t* s_hash, int32_t* s_tmp) {
    constexpr int nt = kSearchBlock;
    const int tid = threadIdx.x;
    const int n = kd.n_kp, C = env.C, R = env.R, nb = env.nb;
    const int n4 = search_cs_units(R * C, nb);
    uint4* w4 = s_cs + 1;   // cell j's count, then its first slot, then (the scatter) the next cell's
    uint32_t* w = reinterpret_cast<uint32_t*>(w4);
    for (int c = tid; c <= n4; c += nt) s_cs[c] = make_uint4(0, 0, 0, 0);
    for (int s = tid; s <= env.hmask; s += nt) s_hash[s] = -1;
    __syncthreads();
    // cell of group g: (row * nb + g) * C + col
    auto cells_of = [&](StageKp& k) {
        const int base = cell_of(k.y, kd.invh, R) * (nb * C) + cell_of(k.x, kd.invw, C);
        int ga, gb;
        groups_of(k.oct, nb, ga, gb);
        k.ca = ga >= 0 ? base + ga * C : -1;
        k.cb = gb >= 0 ? base + gb * C : -1;
    };
    auto count = [&](StageKp& k) {
        cells_of(k);
        if (k.ca >= 0) u16_fetch_add(w, k.ca);
        if (k.cb >= 0) u16_fetch_add(w, k.cb);
    };
    auto list_owner = [&](const StageKp& k) {
        if (k.own >= 0) owner_insert(s_hash, env.hmask, k.own);
    };
    auto scatter = [&](int i, const StageKp& k) {
        KpRec r;
        r.x = k.x;
        r.y = k.y;
        r.idx = i;
        r.oct = k.oct;
        uint4 d0 = make_uint4(0, 0, 0, 0), d1 = d0;
        if (STAGE_DESC && (k.ca >= 0 || k.cb >= 0)) load_desc(env.desc, (int64_t)kd.kp_off + i, d0, d1);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int c = q ? k.cb : k.ca;
            if (c < 0) continue;
            const int slot = u16_fetch_add(w, c);
            s_rec[slot] = r;
            if (STAGE_DESC) {
                s_desc[2 * slot] = d0;
                s_desc[2 * slot + 1] = d1;
            }
        }
    };
#pragma unroll
    for (int j = 0; j < kStagePre; ++j)
        if (tid + j * nt < n) count(pre[j]);
#pragma unroll
    for (int j = 0; j < kStagePre; ++j)
        if (tid + j * nt < n) list_owner(pre[j]);
    for (int i = tid + kStagePre * nt; i < n; i += nt) {
        StageKp k = env.load(kd, i);
        count(k);
        list_owner(k);
    }
    __syncthreads();
    block_exclusive_scan_u16(w4, n4, s_tmp);
#pragma unroll
    for (int j = 0; j < kStagePre; ++j)
        if (tid + j * nt < n) scatter(tid + j * nt, pre[j]);
    for (int i = tid + kStagePre * nt; i < n; i += nt) {
        StageKp k = env.load(kd, i);
        cells_of(k);
        scatter(i, k);
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Global keyframe grids (fallback for keyframes too large for LDS, and
// fl_build_grid): one workgroup per keyframe.

constexpr int kPrepBlock = 256;

// cs[c] = first entry of cell c in ck (cs[cells] = n), the keypoints of a cell
// in increasing index order.  s_cnt: cells + 1 ints of LDS.  With s_ck (at
// least n entries of LDS) the list is put together and sorted there.
__device__ __forceinline__ void build_grid_global(const KfDesc& kd, int cells, int C, int R,
                                                  const float* __restrict__ kp_xy, int32_t* __restrict__ cs,
                                                  int32_t* __restrict__ ck, int32_t* s_cnt, int32_t* s_tmp,
                                                  uint16_t* s_ck = nullptr) {
    const int tid = threadIdx.x, nb = blockDim.x;
    const int n = kd.n_kp;
    const float* xy = kp_xy + 2 * (int64_t)kd.kp_off;
    auto cell = [&](int i) { return cell_of(ldg(xy + 2 * i + 1), kd.invh, R) * C + cell_of(ldg(xy + 2 * i), kd.invw, C); };
    // the cell of the thread's first keypoint is kept for the second pass
    // (and loaded while the counters are cleared)
    const int c0 = tid < n ? cell(tid) : 0;
    for (int c = tid; c <= cells; c += nb) s_cnt[c] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += nb) atomicAdd(&s_cnt[i == tid ? c0 : cell(i)], 1);
    __syncthreads();
    block_exclusive_scan(s_cnt, cells, s_tmp);
    for (int c = tid; c < cells; c += nb) cs[c] = s_cnt[c];
    if (tid == 0) cs[cells] = n;
    __syncthreads();
    for (int i = tid; i < n; i += nb) {
        const int slot = atomicAdd(&s_cnt[i == tid ? c0 : cell(i)], 1);   // ends as the next cell's first
        if (s_ck) s_ck[slot] = (uint16_t)i;
        else ck[slot] = i;
    }
    __syncthreads();
    // keypoints of a cell in increasing index order (deterministic layout)
    auto sort = [&](auto* list) {
        for (int c = tid; c < cells; c += nb) {
            const int b = c ? s_cnt[c - 1] : 0, e = s_cnt[c];
            for (int a = b + 1; a < e; ++a) {
                const auto v = list[a];
                int j = a - 1;
                while (j >= b && list[j] > v) {
                    list[j + 1] = list[j];
                    --j;
                }
                list[j + 1] = v;
            }
        }
    };
    if (s_ck) {
        sort(s_ck);
        __syncthreads();
        for (int i = tid; i < n; i += nb) ck[i] = s_ck[i];
    } else {
        sort(ck);
    }
    __syncthreads();
}

__global__ __launch_bounds__(kPrepBlock) void prep_global_kernel(const BatchHdr* __restrict__ hp) {
    __shared__ int32_t s_cnt[FL_MAX_CELLS + 1];
    __shared__ int32_t s_tmp[kPrepBlock / kWave + 1];
    const BatchHdr& h = *hp;
    for (int k = blockIdx.x; k < h.n_kf; k += gridDim.x) {
        const KfDesc& kd = h.kf[k];
        if (kd.pass != 0) continue;   // the other passes of a keyframe share its grid
        int32_t* cs = h.cell_start + kd.grid_off;
        int32_t* ck = h.cell_kp + kd.kp_off;
        build_grid_global(kd, h.cells, h.grid_cols, h.grid_rows, h.kp_xy, cs, ck, s_cnt, s_tmp);
        for (int s = threadIdx.x; s < kd.n_kp; s += blockDim.x) {
            const int i = ck[s];
            KpRec r;
            r.x = h.kp_xy[2 * ((int64_t)kd.kp_off + i)];
            r.y = h.kp_xy[2 * ((int64_t)kd.kp_off + i) + 1];
            r.idx = i;
            r.oct = (int)h.kp_oct[kd.kp_off + i];
            h.recs[kd.kp_off + s] = r;
            const uint4* src = reinterpret_cast<const uint4*>(h.kp_desc + 32 * ((int64_t)kd.kp_off + i));
            h.desc_sorted[2 * ((int64_t)kd.kp_off + s)] = src[0];
            h.desc_sorted[2 * ((int64_t)kd.kp_off + s) + 1] = src[1];
        }
        int32_t* tab = h.hash + kd.hash_off;
        for (int s = threadIdx.x; s <= kd.hash_mask; s += blockDim.x) tab[s] = -1;
        __syncthreads();
        for (int i = threadIdx.x; i < kd.n_kp; i += blockDim.x) {
            const int32_t o = h.kp_owner[kd.kp_off + i];
            if (o >= 0) owner_insert(tab, kd.hash_mask, o);
        }
        __syncthreads();
    }
}

// What a plain search needs of its keyframe before it starts, in one launch:
// workgroup 0 builds the grid into (caller or scratch) buffers; the other (or
// the only one, given a grid) makes the owner hash set and resets the claims
// and the ADD counter.  Both are chains of short steps over some thousand
// entries, bound by their barriers and round trips: with 1,024 threads a
// keyframe of 1,000 keypoints takes one or two entries a thread at each
// (4.8 us; two launches of 256 threads in turn took 10.3 and 5.1).
constexpr int kSingleBlock = 1024;
constexpr int kSingleLds = 8192;   // keypoints whose list is sorted in LDS

struct PlainPrep {
    const int32_t* kp_owner;
    int32_t* tab;
    int32_t mask;
    int32_t* claim;
    uint32_t* counter;
};

__device__ __forceinline__ void grid_single(const KfDesc& kd, int cells, int C, int R, const float* kp_xy,
                                            int32_t* cell_start, int32_t* cell_kp) {
    __shared__ int32_t s_cnt[FL_MAX_CELLS + 1];
    __shared__ int32_t s_tmp[kSingleBlock / kWave + 1];
    __shared__ uint16_t s_ck[kSingleLds];
    build_grid_global(kd, cells, C, R, kp_xy, cell_start, cell_kp, s_cnt, s_tmp, kd.n_kp <= kSingleLds ? s_ck : nullptr);
}

// Grid of a single keyframe into caller buffers (fl_build_grid).
__global__ __launch_bounds__(kSingleBlock) void grid_single_kernel(KfDesc kd, int cells, int C, int R,
                                                                 const float* __restrict__ kp_xy,
                                                                 int32_t* __restrict__ cell_start,
                                                                 int32_t* __restrict__ cell_kp) {
    grid_single(kd, cells, C, R, kp_xy, cell_start, cell_kp);
}

__global__ __launch_bounds__(kSingleBlock) void plain_prep_kernel(KfDesc kd, int cells, int C, int R,
                                                                const float* __restrict__ kp_xy,
                                                                int32_t* __restrict__ cell_start,
                                                                int32_t* __restrict__ cell_kp, PlainPrep p) {
    const int tid = threadIdx.x, n = kd.n_kp;
    if (blockIdx.x + 1 < gridDim.x) {
        grid_single(kd, cells, C, R, kp_xy, cell_start, cell_kp);
        return;
    }
    const int32_t own = tid < n ? ldg(p.kp_owner + tid) : -1;
    for (int i = tid; i < n; i += kSingleBlock) p.claim[i] = 0x7FFFFFFF;
    if (tid == 0) *p.counter = 0;
    if (p.mask < 2 * kSingleLds) {
        // the set in LDS, then copied out
        __shared__ int32_t s_tab[2 * kSingleLds];
        for (int s = tid; s <= p.mask; s += kSingleBlock) s_tab[s] = -1;
        __syncthreads();
        for (int i = tid; i < n; i += kSingleBlock) {
            const int32_t o = i == tid ? own : ldg(p.kp_owner + i);
            if (o >= 0) owner_insert(s_tab, p.mask, o);
        }
        __syncthreads();
        for (int s = tid; s <= p.mask; s += kSingleBlock) p.tab[s] = s_tab[s];
    } else {
        for (int s = tid; s <= p.mask; s += kSingleBlock) p.tab[s] = -1;
        __syncthreads();
        for (int i = tid; i < n; i += kSingleBlock) {
            const int32_t o = i == tid ? own : ldg(p.kp_owner + i);
            if (o >= 0) owner_insert(p.tab, p.mask, o);
        }
    }
}

// ---------------------------------------------------------------------------
// Per-call tables are fetched by the device from pinned host memory (a plain
// copy kernel, in stream order with the kernels that read them).

// It also advances the claim epoch of the launch that follows (counting
// down, so claims of earlier launches always compare larger) and clears the
// counters of its ranges.
__global__ __launch_bounds__(256) void fetch_blob_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst,
                                                       int n16, uint32_t* __restrict__ epoch,
                                                       RangeCtr* __restrict__ ctr, int n_ctr) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += gridDim.x * blockDim.x) dst[i] = src[i];
    if (blockIdx.x != 0) return;
    for (int i = threadIdx.x; i < n_ctr; i += blockDim.x) {
        ctr[i].claimed = 0;
        ctr[i].helpers = 0;
    }
    if (threadIdx.x == 0) *epoch = *epoch - 1u;
}

// ---------------------------------------------------------------------------
// Wave-aggregated append to a bounded list: one atomic per wave.

template <typename T>
__device__ __forceinline__ void wave_append(bool want, uint32_t* counter, T* list, int32_t cap, const T& e) {
    const unsigned long long m = __ballot(want);
    if (m == 0ull) return;
    const int lane = wave_lane();
    const int leader = __ffsll((long long)m) - 1;
    uint32_t base = 0;
    if (lane == leader) base = atomicAdd(counter, (uint32_t)__popcll(m));
    base = (uint32_t)__shfl((int)base, leader);
    if (want) {
        const uint32_t idx = base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        if (idx < (uint32_t)cap) list[idx] = e;
    }
}

// ---------------------------------------------------------------------------
// Fused batched search.  A tile is one wave's share of a keyframe's pairs (64
// x PPL, pair j on lane j mod 64).  Each workgroup owns a contiguous,
// cost-balanced range of tiles (workgroups are dispatched to the 8 XCDs
// round-robin, and the ranges of one XCD are neighbours in the tile order, so
// the keyframes of an XCD stay in its L2).  The consecutive tiles of one
// keyframe descriptor form a segment: if its keyframe is not the one in LDS,
// the workgroup builds that keyframe's grid, records (and descriptors) and
// owner hash set in LDS; then its waves search the segment's tiles, each wave
// on its own, with no barrier between tiles.  What a tile costs is known only
// once its points are projected, so a long range's second half is claimed tile
// by tile, and a workgroup whose range is done helps the longest of its XCD
// (73 keyframes x 97,969 points: the workgroups ended between 92 and 161 us,
// and the launch takes as long as its last; calls of 224 us became 199).
// Provisional ADDs and accepted pairs go to the workgroup's own list regions
// through LDS counters; a table says which of its accepted pairs are whose
// event's, and the refinement reads them where they are (joining the event's
// list, with a device-scope reservation and a copy, took 6,000 to 8,000 cycles
// at the end of every workgroup).  The ADD conflicts are resolved by the next
// kernel on the stream.
//
// Bound: instruction issue and LDS latency at four waves a SIMD.  A tile of 64
// pairs with two scan steps takes about 400 vector and 40 LDS instructions; the
// vector ones keep a SIMD busy for 63% of a workgroup's time, and 42 fewer of
// them left a call as it was: the chain of dependent operations waits.  The
// tables' uniform values are read by scalar loads where they are used (kept
// across a tile they took 75 vector instructions a tile to bring back from
// spilled lanes).

// Zero in a vector register the compiler cannot see through: an atomic at
// such an offset is left as written (at an address known to be uniform it is
// given a reduction over the wave first, about 25 instructions for one lane).
__device__ __forceinline__ int opaque_zero() {
    int z = 0;
    asm volatile("" : "+v"(z));
    return z;
}

struct KfView {
    const int32_t* cs;          // global grid: cell starts (one bucket per cell)
    const uint16_t* cs16;       // LDS: octave-bucket starts
    int nb;                     // octave buckets per cell
    const KpRec* rec;
    const uint4* desc;          // cell-ordered descriptors (LDS or workspace), or null
    const uint8_t* desc_orig;   // keypoint descriptors by original index (when desc is null)
    const int32_t* hash;
    int32_t hash_mask;
    int32_t n_rec;              // records (slots) in rec
};

// Record slots of a keyframe of kp_cap keypoints in nb octave groups (a
// keypoint sits in up to two groups when nb > 1).
__host__ __device__ inline int search_slots(int kp_cap, int nb) { return nb > 1 ? 2 * kp_cap : kp_cap; }

// LDS bytes of the search kernel (shared with the host).
__host__ __device__ inline size_t search_lds_bytes(int mode, int kp_cap, int cells, int hash_cap, int nb) {
    if (mode == kModeGlobal) return 16;
    const size_t slots = (size_t)search_slots(kp_cap, nb);
    size_t b = 16 * slots;   // records
    if (mode == kModeLdsDesc) b += 32 * slots;
    b += search_cs_bytes(cells, nb);
    b += 4 * (size_t)hash_cap;
    b += 4 * (size_t)(kSearchBlock / kWave + 4);
    return b;
}

// One pair's point, loaded before its evaluation (its descriptor is read
// only for the pair's candidates, when their distances are computed).
struct PairIn {
    int32_t gp, id;
    float x, y, z, dm;
    uint8_t dec;
};

// The launch's point arrays (mp_id may be null; pair_mp is read unless dense).
struct PointEnv {
    const int32_t* pair_mp;
    const int32_t* id;
    const float* xyz;
    const float* dmax;
    bool dense;
    int gate;
};

// The pairs [o, o + 64) of a wave, one a lane, n of them (any n) to be
// searched.  First the point's index in its event (-1: no pair), then the
// point: two dependent loads, in flight during different chunks.  Addresses
// are a scalar base and the lane.
__device__ __forceinline__ PointEnv point_env(cmem<BatchHdr>* h, int gate) {
    return {h->pair_mp, h->mp_id, h->mp_xyz, h->mp_dmax, h->dense != 0, gate};
}

__device__ __forceinline__ int32_t load_index(const PointEnv& env, int64_t pair_off, int64_t o, int n) {
    const uint32_t lane = (uint32_t)wave_lane();
    int32_t lp = -1;
    if ((int)lane < n) lp = env.dense ? (int32_t)(o - pair_off) + (int32_t)lane : ldg(env.pair_mp + o + lane);
    return lp;
}

typedef float v3f __attribute__((ext_vector_type(3), aligned(4)));

__device__ __forceinline__ void load_point(const PointEnv& env, int32_t mp_off, int32_t n_mp, int32_t lp, int n,
                                           PairIn& p) {
    p.dec = FL_INVALID;
    p.gp = 0;
    p.id = -1;
    p.x = p.y = p.z = p.dm = 0.0f;
    if (wave_lane() < n && lp >= 0 && lp < n_mp) {
        p.dec = kDecUndecided;
        p.gp = mp_off + lp;
        p.id = env.id ? ldg(env.id + p.gp) : p.gp;
        const v3f x = *(const gmem<v3f>*)(env.xyz + 3 * (int64_t)p.gp);
        p.x = x.x;
        p.y = x.y;
        p.z = x.z;
        if (env.gate) p.dm = ldg(env.dmax + p.gp);
    }
}

// Search result of one pair beyond its decision.
struct PairRes {
    Best best;
    int32_t target;
    float ku, kv;   // the best candidate's keypoint
};

// The octave scale table sf[n] = scale_factor^n of a launch: its first
// kOctReg entries in registers, every entry in LDS; and the pass's window
// half-width at octave 0.
constexpr int kOctReg = 8;
struct OctaveTable {
    float sf[kOctReg];
    const float* all;   // LDS, n_octaves entries
    int N;
    float r0;
};

// The first n with d * sf[n] >= dmax, else N - 1: the first kOctReg tests
// from the last to the first without branches (entries past N, if any test
// true, come after every real one and are cut to N - 1).
__device__ __forceinline__ int predict_octave(const OctaveTable& T, float d, float dmax) {
    int pred = kOctReg;
#pragma unroll
    for (int n = kOctReg - 1; n >= 0; --n) pred = d * T.sf[n] >= dmax ? n : pred;
    if (T.N > kOctReg && pred == kOctReg)
        while (pred < T.N - 1 && !(d * T.all[pred] >= dmax)) ++pred;
    return min(pred, T.N - 1);
}

// Window half-width r0 * sf[pred] (sf from LDS: a lane-dependent index into
// registers would be compiled as a table in scratch memory).
__device__ __forceinline__ float window_radius(const OctaveTable& T, int pred) { return T.r0 * T.all[pred]; }

// Evaluation of one pair (point p, keyframe kd) in three parts.  The front
// (per lane): observed-set test, Sim3 projection, predicted octave, window,
// and the runs of record slots to read: the window's grid rows of the pair's
// octave group (with the octave gate on, the group holds octaves pred - 1
// and pred only: a quarter of the window's keypoints when the eight octaves
// are equally common).  The scan (the whole wave together): every lane walks
// its runs as one flat sequence, testing box and octave; the records that
// pass go to a per-wave queue, and each time the queue fills (and at the end)
// the wave computes the queued Hamming distances one per lane, so the
// distance instructions run with their lanes full instead of with the few
// lanes that happen to have a candidate at one step.  Best and second best
// are kept per lane in LDS with atomic minima: the packed (distance, index)
// key of a candidate goes to the best slot, and whichever key the update
// leaves out (the old best, or the candidate) offers its distance to the
// second slot; so the second slot ends at the smallest distance of every
// candidate but the best, whatever the order.  The back (per lane): the
// fuse / add decision (provisional for ADD).  st: visible pairs, cells
// scanned, keypoints in them (every octave), candidates.  The wave takes
// kRowSeg rows of every window at a time: at 3 pixels few windows have more;
// at 10 pixels the upper octaves' have up to eight, and walking those by
// themselves, lane by lane, made a 20-keyframe event with outlier rounds 94 us
// instead of 89.
constexpr int kRowSeg = 4;
static_assert(kRowSeg == 4, "four row runs");

// What the front leaves for the scan of one pair.
struct PairScan {
    Window w;
    int pred, grp;
    int b0, d1, d2, d3, c1, c2, c3, total;   // slot = m + b0 + (d_j where m >= c_j)
    int nrows;
    int first;   // entry of the bucket starts of the window's first row, column 0
};

// Per wave: the candidate queue, each lane's best key and second distance,
// and the marks of the scan's item ranges (-1 between uses).
struct WaveCand {
    uint32_t q[kWave];        // owner lane << 17 | slot
    uint32_t best[kWave];
    uint32_t second[kWave];
    int32_t mark[kWave];
};
constexpr size_t kSearchStaticLds = sizeof(WaveCand) * kWavesPerWG + 1024;   // beside the dynamic LDS

// The runs of the window's rows j0 .. j0 + kRowSeg - 1, and how many records
// they hold (named values, not arrays: an array indexed by a lane-dependent
// value would be placed in scratch memory).
template <int MODE>
__device__ __forceinline__ void row_runs(const KfView& v, int C, int j0, PairScan& q) {
    const int row = (MODE == kModeGlobal ? 1 : v.nb) * C;
    auto cs_at = [&](int j) -> int { return MODE == kModeGlobal ? v.cs[j] : (int)v.cs16[j]; };
    auto run = [&](int j, int c_in, int& b_out, int& c_out) {
        const bool in = j0 + j < q.nrows;
        const int idx = q.first + (in ? (j0 + j) * row : 0);
        const int s0 = cs_at(idx + q.w.c0), e0 = cs_at(idx + q.w.c1 + 1);
        b_out = s0 - c_in;
        c_out = c_in + (in ? e0 - s0 : 0);
    };
    int b1, b2, b3;
    run(0, 0, q.b0, q.c1);
    run(1, q.c1, b1, q.c2);
    run(2, q.c2, b2, q.c3);
    run(3, q.c3, b3, q.total);
    q.d1 = b1 - q.b0;
    q.d2 = b2 - b1;
    q.d3 = b3 - b2;
}

template <int MODE, bool STATS>
__device__ __forceinline__ bool search_front(const KfDesc& kd, const KfView& v, const OctaveTable& T, int gate,
                                             int C, int R, PairIn& p, PairScan& q, unsigned long long* st) {
    q.total = 0;
    q.nrows = 0;
    // owner probe (a point already observed in this keyframe is skipped):
    // its first read is issued here and the probe finished after the
    // window, so its latency overlaps the projection
    const bool probe = p.dec == kDecUndecided && p.id >= 0;
    uint32_t hh = 0;
    int32_t hv = -1;
    if (probe) {
        hh = owner_slot(p.id, v.hash_mask);
        hv = v.hash[hh];
    }
    Proj pr;
    const bool vis = project_uv(kd, p.x, p.y, p.z, pr);
    q.pred = gate ? predict_octave(T, pr.d, p.dm) : T.N - 1;
    const float rad = window_radius(T, q.pred);
    Window& w = q.w;
    w.lx = pr.u - rad;
    w.hx = pr.u + rad;
    w.ly = pr.v - rad;
    w.hy = pr.v + rad;
    w.c0 = cell_of(w.lx, kd.invw, C);
    w.c1 = cell_of(w.hx, kd.invw, C);
    w.r0 = cell_of(w.ly, kd.invh, R);
    w.r1 = cell_of(w.hy, kd.invh, R);
    const int nb = MODE == kModeGlobal ? 1 : v.nb;
    auto cs_at = [&](int j) -> int { return MODE == kModeGlobal ? v.cs[j] : (int)v.cs16[j]; };
    q.grp = min(q.pred, nb - 1);
    q.nrows = w.r1 - w.r0 + 1;
    q.first = (int)__umul24(__umul24(w.r0, nb) + q.grp, C);
    row_runs<MODE>(v, C, 0, q);
    if (probe) {
        for (int n = 0; n <= v.hash_mask; ++n) {
            if (hv == p.id) {
                p.dec = FL_SKIP;
                break;
            }
            if (hv < 0) break;
            hh = (hh + 1) & (uint32_t)v.hash_mask;
            hv = v.hash[hh];
        }
    }
    // SKIP before NOT_VISIBLE; neither is searched
    if (p.dec == kDecUndecided && !vis) p.dec = FL_NOT_VISIBLE;
    if (p.dec != kDecUndecided) {
        q.total = 0;
        q.nrows = 0;
        return false;
    }
    if (STATS) {
        ++st[0];
        // cells and keypoints of the window's cells (every octave: the
        // counting launch stages one group)
        for (int row = w.r0; row <= w.r1; ++row) {
            st[1] += (unsigned long long)(w.c1 - w.c0 + 1);
            for (int g = 0; g < nb; ++g) {
                const int j = (row * nb + g) * C;
                st[2] += (unsigned long long)(cs_at(j + w.c1 + 1) - cs_at(j + w.c0));
            }
        }
    }
    return true;
}

// Descriptor of record slot i (keypoint index idx).
template <int MODE>
__device__ __forceinline__ void record_desc(const KfView& v, int i, int idx, uint4& b0, uint4& b1) {
    if (MODE == kModeLdsRec) {
        load_desc(v.desc_orig, idx, b0, b1);
    } else if (MODE == kModeLdsDesc) {
        b0 = v.desc[2 * i];
        b1 = v.desc[2 * i + 1];
    } else {
        b0 = ldg_u4(v.desc + 2 * i);
        b1 = ldg_u4(v.desc + 2 * i + 1);
    }
}

// A candidate of key k for the pair of `owner`: the atomic-minimum update of
// its best and second slots (see above).
__device__ __forceinline__ void offer_lds(WaveCand& wc, int owner, uint32_t k) {
    const uint32_t old = atomicMin(&wc.best[owner], k);
    const uint32_t out = k < old ? old : k;
    if (out != 0xFFFFFFFFu) atomicMin(&wc.second[owner], out >> 16);
}

// The queued candidates, one per lane: the owner's point descriptor (its
// point index from the owner lane) against the keypoint's.  Every lane of
// the wave takes part in the cross-lane read.
template <int MODE>
__device__ __forceinline__ void drain_queue(WaveCand& wc, int qn, const KfView& v, const uint8_t* mp_desc,
                                            int32_t gp) {
    const int lane = wave_lane();
    const uint32_t e = lane < qn ? wc.q[lane] : 0u;
    const int owner = (int)(e >> 17);
    const int32_t ogp = __builtin_amdgcn_ds_bpermute(owner << 2, gp);
    if (lane < qn) {
        const int slot = (int)(e & 0x1FFFFu);
        const int idx = v.rec[slot].idx;
        uint4 a0, a1, b0, b1;
        load_desc(mp_desc, ogp, a0, a1);
        record_desc<MODE>(v, slot, idx, b0, b1);
        offer_lds(wc, owner, ((uint32_t)hamming(a0, a1, b0, b1) << 16) | (uint32_t)idx);
    }
}

// The wave's scan of its lanes' pairs (every lane of the wave calls it; a
// lane with no pair to search has q.total = 0 and q.nrows = 0).  The records
// of the lanes' runs form one sequence of items, lane after lane (lane l's
// q.total items from P_l, the exclusive prefix sum of the totals), taken 64
// at a time, one per lane: a wave makes ceil(N / 64) steps for its N items
// instead of as many as its busiest lane has records.  Lane l marks where its
// items start; the owner of an item is the last mark at or before it, and
// the owner's window and run layout come from the owner lane.
template <int MODE, bool STATS>
__device__ __forceinline__ void search_scan(const KfView& v, int gate, int C, const uint8_t* mp_desc,
                                            const PairIn& p, PairScan& q, WaveCand& wc,
                                            unsigned long long* st) {
    const int lane = wave_lane();
    wc.best[lane] = 0xFFFFFFFFu;
    wc.second[lane] = FL_NO_DIST;
    int qn = 0;
    for (int j0 = 0;;) {
        const int L = q.total;
        const int incl = wave_incl_scan(L);
        const int P = incl - L;
        const int N = __builtin_amdgcn_readlane(incl, kWave - 1);
        // item k of this lane (P <= k < P + L) is record slot
        // k + B + (d1 if k >= A1) + (d2 if k >= A2) + (d3 if k >= A3)
        const int B = q.b0 - P, A1 = P + q.c1, A2 = P + q.c2, A3 = P + q.c3;
        const float lx = q.w.lx, hx = q.w.hx, ly = q.w.ly, hy = q.w.hy;
        int cur = 0;   // owner of the step's first item when no range starts there
        for (int base = 0; base < N; base += kWave) {
            // (one wave's LDS accesses complete in order: the read below sees
            // the marks, and the reset follows the read)
            if (L > 0 && P >= base && P < base + kWave) wc.mark[P - base] = lane;
            int mk = wc.mark[lane];
            wc.mark[lane] = -1;
            if (lane == 0 && mk < 0) mk = cur;
            const unsigned long long starts = __ballot(mk >= 0);   // bit 0 always set
            const unsigned long long upto = lane == kWave - 1 ? ~0ull : ((2ull << lane) - 1ull);
            const int pos = 63 - __builtin_clzll(starts & upto);
            const int o = __shfl(mk, pos);   // owner lane of item base + lane
            cur = __builtin_amdgcn_readlane(o, kWave - 1);
            const int k = base + lane;
            const bool act = k < N;
            const int oB = __shfl(B, o), oA1 = __shfl(A1, o), oA2 = __shfl(A2, o), oA3 = __shfl(A3, o);
            const int od1 = __shfl(q.d1, o), od2 = __shfl(q.d2, o), od3 = __shfl(q.d3, o);
            Window w;
            w.lx = __shfl(lx, o);
            w.hx = __shfl(hx, o);
            w.ly = __shfl(ly, o);
            w.hy = __shfl(hy, o);
            const int opred = __shfl(q.pred, o);
            const int i = k + oB + (od1 & -(int)(k >= oA1)) + (od2 & -(int)(k >= oA2)) + (od3 & -(int)(k >= oA3));
            KpRec rc{};
            if (act) rc = v.rec[min((unsigned)i, (unsigned)(v.n_rec - 1))];   // (in range by construction)
            const bool cand = act && in_window(w, rc.x, rc.y, rc.oct, opred, gate);
            const unsigned long long cm = __ballot(cand);
            if (cm) {
                const int n = __popcll(cm);
                if (qn + n > kWave) {
                    drain_queue<MODE>(wc, qn, v, mp_desc, p.gp);
                    qn = 0;
                }
                if (cand) {
                    wc.q[qn + __popcll(cm & ((1ull << lane) - 1ull))] = ((uint32_t)o << 17) | (uint32_t)i;
                    if (STATS) ++st[3];
                }
                qn += n;
            }
        }
        // the next rows, if any lane's window has them
        j0 += kRowSeg;
        if (__ballot(q.nrows > j0) == 0ull) break;
        row_runs<MODE>(v, C, j0, q);
    }
    if (qn) drain_queue<MODE>(wc, qn, v, mp_desc, p.gp);
}

// The decision of a searched pair from its best and second.
// kp_owner and, if given, kp_xy are the keyframe's; with kp_xy, also the
// accepted keypoint's position (the two loads together).
__device__ __forceinline__ void search_back(int hamming_th, float nn_ratio, const int32_t* kp_owner,
                                            const float* kp_xy, PairIn& p, PairRes& res) {
    if (!accept_match(res.best, hamming_th, nn_ratio)) {
        p.dec = FL_NO_MATCH;
    } else {
        const uint32_t kg = res.best.key & 0xFFFFu;
        const int32_t ow = ldg(kp_owner + kg);
        if (kp_xy) {
            res.ku = ldg(kp_xy + 2 * kg);
            res.kv = ldg(kp_xy + 2 * kg + 1);
        }
        if (ow >= 0) {
            p.dec = FL_FUSE;
            res.target = ow;
        } else {
            p.dec = FL_ADD;   // provisional; losers are relabelled by the resolver
        }
    }
}

// The workgroup's accepted pairs by event: the table entry of the event whose
// pairs are being searched is written when the next begins (or, event < 0, at
// the end).  The workgroup's counts are complete when it is called.
struct MatchSegs {
    int event;
    uint32_t m0;   // first staged pair of the event
    __device__ __forceinline__ void next(const BatchHdr& h, const WgRange& rg, const unsigned long long* s_list,
                                         int e) {
        const uint32_t m = (uint32_t)(s_list[0] >> 32);
        if (threadIdx.x == 0 && event >= 0)
            h.match_seg[rg.chunk + event] = MatchSeg{(int32_t)(rg.priv_off + m0), (int32_t)(m - m0)};
        event = e;
        m0 = m;
    }
};

// A range to help with, chosen by one wave for its workgroup, whose own is
// done: of the ranges all of whose tiles belong to `event` (the workgroup's
// accepted pairs then stay one run), the one with the most unclaimed tiles per
// workgroup on it, if they are at least kHelpTiles: staging a keyframe anew
// costs what two rounds of the sixteen waves do.  The workgroup's list regions
// must have room for what its waves may hold.  Only the ranges of its own XCD
// (every kMaxQueues-th workgroup) are looked at: their points are in its L2, and
// each look goes to memory (with every workgroup reading all 256 counters in
// the launch's last third, loads took 8,000 cycles).  out: the range (or -1).
constexpr int kHelpTiles = 32;

__device__ __forceinline__ void pick_range(const BatchHdr& h, RangeCtr* ctr, int event, uint32_t held, int32_t cap,
                                           unsigned long long used, int* out) {
    const int lane = wave_lane();
    int best = -1, best_i = -1;
    if (max((uint32_t)used, (uint32_t)(used >> 32)) + held <= (uint32_t)cap) {
        for (int i = (int)(blockIdx.x % kMaxQueues) + lane * kMaxQueues; i < (int)gridDim.x; i += kWave * kMaxQueues) {
            const WgRange& r = h.wg_range[i];
            const unsigned long long taken = __hip_atomic_load((gmem<unsigned long long>*)&ctr[i], __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT);
            const int score = (r.t1 - range_shared(r.t0, r.t1, kWavesPerWG) - (int)(uint32_t)taken) / (1 + (int)(taken >> 32));
            if (r.event == event && r.one_event && score > best) {
                best = score;
                best_i = i;
            }
        }
    }
    int m = best;
    for (int off = 32; off > 0; off >>= 1) m = max(m, __shfl_xor(m, off));
    const unsigned long long who = __ballot(best == m);
    const int v = __builtin_amdgcn_readlane(best_i, __ffsll((long long)who) - 1);
    if (lane == 0) {
        out[0] = m >= kHelpTiles ? v : -1;
        if (m >= kHelpTiles)
            __hip_atomic_fetch_add((gmem<uint32_t>*)&ctr[v].helpers, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <int PPL, int MODE, bool STATS>
__global__ __launch_bounds__(kSearchBlock) void search_fused_kernel(const BatchHdr* __restrict__ hp) {
    extern __shared__ __align__(16) unsigned char s_mem[];
    const BatchHdr& h = *hp;
    const int tid = threadIdx.x;
    const int lane = wave_lane();
    __shared__ unsigned long long s_list[1];   // running counts: ADD region (low half), accepted-pair region
    __shared__ WaveCand s_wc[kWavesPerWG];   // each wave's candidate queue, best and second
    __shared__ float s_sf[FL_MAX_OCTAVES];
    __shared__ int s_first[4], s_help[4];
    const int wid = __builtin_amdgcn_readfirstlane(tid / kWave);
    constexpr int nw = kWavesPerWG;

    // Every load of the prologue is issued before the first is waited for: a
    // launch starts with the header, the ranges and the keyframe table in
    // memory only (the table fetch wrote them), and a trip there is about
    // 2,000 cycles.  The range and the keyframe table sit at offsets of the
    // table blob that follow from the grid size, so neither waits for a
    // pointer, and the range holds what the first keyframe's own loads need.
    const char* blob = reinterpret_cast<const char*>(hp);
    const WgRange rg = reinterpret_cast<const WgRange*>(blob + blob_range_offset())[blockIdx.x];
    const KfDesc* kf_tab = reinterpret_cast<const KfDesc*>(blob + blob_kf_offset((int)gridDim.x));
    const float sf_lane = h.sf[tid & (FL_MAX_OCTAVES - 1)];
    const int gate = uniform_i(h.gate), C = uniform_i(h.grid_cols), R = uniform_i(h.grid_rows);
    const int nb = MODE == kModeGlobal ? 1 : uniform_i(h.oct_buckets);
    const int hmask = uniform_i(h.lds_hash_mask);
    const int kp_cap = uniform_i(h.lds_kp_cap);
    const bool want_matches = uniform_i(h.refine_iters) > 0;
    const uint32_t epoch = ldg(h.epoch);   // (a vector register: waited for where it is used)
    unsigned long long st[4] = {0, 0, 0, 0};

    KpRec* s_rec = reinterpret_cast<KpRec*>(s_mem);
    uint4* s_desc = nullptr;
    uint4* s_cs = nullptr;
    int32_t* s_hash = nullptr;
    int32_t* s_tmp = nullptr;
    if (MODE != kModeGlobal) {
        const size_t slots = (size_t)search_slots(kp_cap, nb);
        unsigned char* p = s_mem + 16 * slots;
        if (MODE == kModeLdsDesc) {
            s_desc = reinterpret_cast<uint4*>(p);
            p += 32 * slots;
        }
        s_cs = reinterpret_cast<uint4*>(p);
        p += search_cs_bytes(C * R, nb);
        s_hash = reinterpret_cast<int32_t*>(p);
        p += 4 * (size_t)(hmask + 1);
        s_tmp = reinterpret_cast<int32_t*>(p);
    }
    if (tid < 4) s_first[tid] = INT32_MAX;
    if (tid == 0) s_list[0] = 0;
    s_wc[wid].mark[lane] = -1;
    // the octave scale table in LDS (the octave search and the window radius
    // index it per lane): published, as the counters above, by the first
    // keyframe's staging in the LDS modes
    if (tid < FL_MAX_OCTAVES) s_sf[tid] = sf_lane;
    if (MODE == kModeGlobal) __syncthreads();

    // The wave's tile ta and the one after it, tb, in the range [.., t1) being
    // searched, whose tiles from ts on are claimed.
    int ta = rg.t0 + wid, tb = ta + nw, t1 = rg.t1;
    int ts = range_shared(rg.t0, rg.t1, nw);
    int own = (int)blockIdx.x;
    RangeCtr* const ctr = uniform_p(h.range_ctr);
    constexpr int kChunk = kWave * PPL;
    // entries that every tile the waves may hold (one being searched, ta, tb and
    // one claimed each) could add to the lists
    constexpr uint32_t kHeld = 4 * nw * kChunk;
    auto claim_tile = [&]() -> int {   // lane 0's value
        int v = kNoTile;
        bool room = true;
        if (own != (int)blockIdx.x)
            room = max((uint32_t)s_list[0], (uint32_t)(s_list[0] >> 32)) + kHeld <= (uint32_t)rg.priv_cap;
        if (room && lane == 0)
            v = ts + (int)__hip_atomic_fetch_add((gmem<uint32_t>*)&ctr[own].claimed, 1u, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
        return v;
    };
    // The tile after tb: nw further on, or claimed (tc_v, lane 0's) if that is
    // one to claim; none after a tile past the end.
    int tc_v = kNoTile;
    auto ask_next = [&]() {
        tc_v = kNoTile;
        if (tb + nw >= ts && tb < t1 && ts < t1) tc_v = claim_tile();
    };
    ask_next();

    int slot = rg.slot;
    int staged = -1;
    MatchSegs segs{rg.event, 0};
    for (int seg = 0;; ++seg) {
        int k = rg.kf, tb0 = rg.slot_t0, te = rg.slot_t1, pass = rg.pass, key = rg.stage_key;
        StageKf sk{rg.kp_off, rg.n_kp, rg.invw, rg.invh};
        if (seg == 0) {
            if (rg.t0 >= rg.t1) break;
        } else {
            // the lowest tile any wave still holds (three minima in turn: one
            // is cleared a segment after its last reader)
            if (lane == 0 && ta < t1) atomicMin(&s_first[seg % 3], ta);
            __syncthreads();   // also: every reader of the keyframe is done, its pairs are listed
            const int t = uniform_i(s_first[seg % 3]);
            if (tid == 0) s_first[(seg + 2) % 3] = INT32_MAX;
            if (t >= t1) {
                // nothing is left of the range: help another
                if (wid == 0) pick_range(h, ctr, segs.event, kHeld, rg.priv_cap, s_list[0], s_help);
                __syncthreads();
                const int v = uniform_i(s_help[0]);
                if (v < 0) break;
                own = v;
                const WgRange& r = h.wg_range[v];
                t1 = uniform_i(r.t1);
                ts = range_shared(uniform_i(r.t0), t1, nw);
                slot = uniform_i(r.slot);
                const int a_v = claim_tile(), b_v = claim_tile();
                ta = uniform_i(a_v);
                tb = uniform_i(b_v);
                ask_next();
                continue;
            }
            while (t >= uniform_i(h.tile_prefix[slot + 1])) ++slot;
            k = uniform_i(h.kf_order[slot]);
            tb0 = uniform_i(h.tile_prefix[slot]);
            te = uniform_i(h.tile_prefix[slot + 1]);
            const KfDesc& kn = kf_tab[k];
            pass = uniform_i(kn.pass);
            key = uniform_i(kn.stage_key);
            sk = {uniform_i(kn.kp_off), uniform_i(kn.n_kp), uniform_f(kn.invw), uniform_f(kn.invh)};
        }
        te = min(te, t1);
        StageKp pre[kStagePre];
        const bool build = MODE != kModeGlobal && staged != key;
        cmem<BatchHdr>* const hs = fresh(hp);
        const StageEnv stage{hs->kp_xy, hs->kp_oct, hs->kp_owner, hs->kp_desc, C, R, nb, hmask};
        if (build) stage_load(stage, sk, pre);
        const KfDesc* const kf = kf_tab + k;
        const KfDesc kd = search_kf(fresh(kf));
        // A tile is the pairs [first_pair(t), + kChunk) of the keyframe, up to
        // its last pair se.
        const int64_t se = kd.pair_off + kd.n_pairs;
        auto first_pair = [&](int t) { return kd.pair_off + (int64_t)(t - tb0) * kChunk; };
        // pairs of the 64 from pair o on (any value <= 0: none)
        auto left = [&](int64_t o) { return (int)min(se - o, (int64_t)kWave); };
        if (want_matches && kd.event != segs.event) {
            // (the barrier above: every pair of the events before is listed)
            segs.next(h, rg, s_list, kd.event);
            __syncthreads();
        }
        // The points of a wave's first tile are loaded while the keyframe is
        // staged, those of its next while its current one is evaluated, and
        // with them the point indices of the one after, which is claimed
        // another tile earlier.
        PairIn pn[PPL];
        int32_t ln[PPL];
        auto indices = [&](const PointEnv& points, int t) {
#pragma unroll
            for (int r = 0; r < PPL; ++r) {
                const int64_t o = first_pair(t) + r * kWave;
                ln[r] = load_index(points, kd.pair_off, o, t < te ? left(o) : 0);
            }
        };
        auto pts = [&](const PointEnv& points, int32_t mp_off, int32_t n_mp, int t) {
#pragma unroll
            for (int r = 0; r < PPL; ++r)
                load_point(points, mp_off, n_mp, ln[r], t < te ? left(first_pair(t) + r * kWave) : 0, pn[r]);
        };
        {
            const PointEnv points = point_env(hs, gate);
            indices(points, ta);
            pts(points, kd.mp_off, kd.n_mp, ta);
            indices(points, tb);
        }

        KfView v;
        if (MODE == kModeGlobal) {
            v.cs = h.cell_start + kd.grid_off;
            v.cs16 = nullptr;
            v.nb = 1;
            v.rec = h.recs + kd.kp_off;
            v.n_rec = max(kd.n_kp, 1);
            v.desc = h.desc_sorted + 2 * (int64_t)kd.kp_off;
            v.desc_orig = nullptr;
            v.hash = h.hash + kd.hash_off;
            v.hash_mask = kd.hash_mask;
        } else {
            if (build) {
                stage_build<MODE == kModeLdsDesc>(stage, sk, pre, s_cs, s_rec, s_desc, s_hash, s_tmp);
                staged = key;
            }
            v.cs = nullptr;
            v.cs16 = reinterpret_cast<const uint16_t*>(s_cs) + kCsFirst;
            v.nb = nb;
            v.rec = s_rec;
            v.n_rec = search_slots(kp_cap, nb);
            v.desc = MODE == kModeLdsDesc ? s_desc : nullptr;
            v.desc_orig = nullptr;   // read where it is used
            v.hash = s_hash;
            v.hash_mask = hmask;
        }

        while (ta < te) {
            const int64_t cb = first_pair(ta);
            PairIn p[PPL];
#pragma unroll
            for (int r = 0; r < PPL; ++r) p[r] = pn[r];
            const int tc = tb + nw < ts ? tb + nw : uniform_i(tc_v);
            {
                cmem<KfDesc>* const kc = fresh(kf);
                const PointEnv points = point_env(fresh(hp), gate);
                pts(points, kc->mp_off, kc->n_mp, tb);
                indices(points, tc);
            }
            ta = tb;
            tb = tc;
            ask_next();
#pragma unroll
            for (int r = 0; r < PPL; ++r) {
                const int64_t o = cb + r * kWave;   // lane 0's pair
                const bool active = lane < left(o);
                PairRes res;
                res.target = -1;
                res.ku = res.kv = 0.0f;
                PairScan sq;
                bool searching;
                {
                    cmem<BatchHdr>* const hc = fresh(hp);
                    OctaveTable T;
                    T.all = s_sf;
                    T.N = hc->n_octaves;
                    T.r0 = hc->out[pass].r0;
#pragma unroll
                    for (int n = 0; n < kOctReg; ++n) T.sf[n] = hc->sf[n];
                    searching = search_front<MODE, STATS>(search_kf(fresh(kf)), v, T, gate, C, R, p[r], sq, st);
                }
                WaveCand& wc = s_wc[wid];
                cmem<BatchHdr>* const hc = fresh(hp);
                const int64_t kp_off = fresh(kf)->kp_off;
                if (MODE == kModeLdsRec) v.desc_orig = hc->kp_desc + 32 * kp_off;
                search_scan<MODE, STATS>(v, gate, C, hc->mp_desc, p[r], sq, wc, st);
                res.best.key = wc.best[lane];
                res.best.second = (int)wc.second[lane];
                cmem<BatchHdr>* const hb = fresh(hp);
                cmem<PassOut>* const po = &hb->out[pass];
                if (searching)
                    search_back(po->hamming_th, po->nn_ratio, hb->kp_owner + kp_off,
                                want_matches ? hb->kp_xy + 2 * kp_off : nullptr, p[r], res);
                // Stores and loads are counted together, in order: the next
                // tiles' loads (and the claim) are waited for here, not behind
                // the stores below.
#pragma unroll
                for (int i = 0; i < PPL; ++i)
                    asm volatile("" : "+v"(pn[i].x), "+v"(pn[i].y), "+v"(pn[i].z), "+v"(pn[i].dm), "+v"(pn[i].id),
                                      "+v"(ln[i]));
                asm volatile("" : "+v"(tc_v));
                const uint32_t key = res.best.key;
                const int bidx = key == 0xFFFFFFFFu ? -1 : (int)(key & 0xFFFFu);
                const int kpg = fresh(kf)->claim_off + (bidx < 0 ? 0 : bidx);   // claim slot
                const uint32_t ul = (uint32_t)lane;
                if (active) {
                    stg(po->best_idx + o + ul, (int32_t)bidx);
                    stg(po->best_dist + o + ul, (int16_t)(key == 0xFFFFFFFFu ? FL_NO_DIST : (int)(key >> 16)));
                    stg(po->second_dist + o + ul, (int16_t)res.best.second);
                    stg(po->decision + o + ul, p[r].dec);
                    stg(po->target + o + ul, res.target);
                }
                const bool is_add = active && p[r].dec == FL_ADD;
                const bool acc = want_matches && active && (p[r].dec == FL_ADD || p[r].dec == FL_FUSE);
                if (is_add)
                    __hip_atomic_fetch_min((gmem<unsigned long long>*)(hb->claim + kpg),
                                           (unsigned long long)epoch << 32 | (uint32_t)p[r].gp, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                // one LDS reservation per wave for both lists
                const unsigned long long ma = __ballot(is_add), mm = __ballot(acc);
                if ((ma | mm) == 0) continue;
                unsigned long long at = 0;
                if (lane == 0)
                    at = atomicAdd(&s_list[opaque_zero()],
                                   (unsigned long long)__popcll(mm) << 32 | (unsigned long long)__popcll(ma));
                const uint32_t ba = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at);
                const uint32_t bm = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32));
                if (is_add) {
                    AddRef e;
                    e.pair = (int32_t)(o + lane);
                    e.kp = kpg;
                    e.gp = p[r].gp;
                    e.pass = pass;
                    stg_rec(hb->add_list + rg.priv_off + ba + __builtin_amdgcn_mbcnt_hi((uint32_t)(ma >> 32),
                                __builtin_amdgcn_mbcnt_lo((uint32_t)ma, 0u)), e);
                }
                if (acc) {
                    // the matched keypoint's observation
                    MatchRec me;
                    me.x = p[r].x;
                    me.y = p[r].y;
                    me.z = p[r].z;
                    me.u = res.ku;
                    me.v = res.kv;
                    me.kf = k;
                    me.pad0 = me.pad1 = 0;
                    stg_rec(hb->match_stage + rg.priv_off + bm + __builtin_amdgcn_mbcnt_hi((uint32_t)(mm >> 32),
                                __builtin_amdgcn_mbcnt_lo((uint32_t)mm, 0u)), me);
                }
            }
        }
    }
    __syncthreads();   // every ADD and accepted pair of the workgroup is counted
    if (tid == 0) h.add_count[blockIdx.x] = (uint32_t)s_list[0];
    if (want_matches) segs.next(h, rg, s_list, -1);
    if (STATS) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            unsigned long long xv = st[i];
            for (int off = 32; off > 0; off >>= 1) xv += __shfl_xor(xv, off);
            if (lane == 0 && xv) atomicAdd(&h.stats_out[i], xv);
        }
    }
}

// ADD resolution after a batched search launched without refinement: the
// search workgroups' ADD regions, grid-stride.
constexpr int kResolveBlock = 256;
constexpr int kResolveGrid = 1024;   // workgroups in graph mode (any count is correct)

__global__ __launch_bounds__(kResolveBlock) void resolve_adds_kernel(const BatchHdr* __restrict__ hp) {
    const BatchHdr& h = *hp;
    const unsigned long long tag = (unsigned long long)(*h.epoch) << 32;
    for (int r = blockIdx.x; r < h.n_wg; r += gridDim.x) resolve_region_adds(h, r, tag);
}

// ---------------------------------------------------------------------------
// Plain search: one lane per map point against one keyframe, candidates
// gathered through the caller's (or a freshly built) cell_start / cell_kp
// grid from the keyframe's own arrays.

struct PlainArgs {
    KfDesc kd;
    SearchConst sc;
    int32_t first;   // the launch's first point
    int32_t n_mp;
    int32_t add_cap;
    const float* mp_xyz;
    const uint8_t* mp_desc;
    const float* mp_dmax;
    const int32_t* mp_id;
    const float* kp_xy;
    const int8_t* kp_oct;
    const uint8_t* kp_desc;
    const int32_t* kp_owner;
    const int32_t* cell_start;
    const int32_t* cell_kp;
    const int32_t* hash;
    int32_t* claim;
    uint32_t* counter;
    AddRef* add_list;
    int32_t* best_idx;
    int16_t* best_dist;
    int16_t* second_dist;
    uint8_t* decision;
    int32_t* target;
};

// The plain search gives each point kPlainLanes neighbouring lanes: with one
// lane a point, a call of 2,000 points puts 32 waves on the chip, each walking
// its window's candidates one after the other, four dependent loads apiece.
// Lane j of a point takes the rows j mod 4, every fourth, and of a row's
// candidates every second from j / 4 on; the lanes' best and second are put
// together at the end.  (2,000 points, 1,000 keypoints: 8.0 us, 13.0 with one
// lane a point.)
constexpr int kPlainBlock = 256;
constexpr int kPlainLanes = 8;
constexpr int kPlainSlice = 1 << 28;   // points a launch takes: one may have up to 2^32 - 1 threads

// a's and b's candidates together: the better best key; of the other key and
// the two seconds the smallest distance.
__device__ __forceinline__ void merge_best(Best& a, uint32_t key, int second) {
    const uint32_t lose = max(a.key, key);
    a.key = min(a.key, key);
    a.second = min(a.second, second);
    if (lose != 0xFFFFFFFFu) a.second = min(a.second, (int)(lose >> 16));
}

__global__ __launch_bounds__(kPlainBlock) void search_plain_kernel(PlainArgs a) {
    __shared__ float s_sf[FL_MAX_OCTAVES];
    if (threadIdx.x < FL_MAX_OCTAVES) s_sf[threadIdx.x] = a.sc.sf[threadIdx.x];
    const int64_t o = a.first + ((int64_t)blockIdx.x * kPlainBlock + threadIdx.x) / kPlainLanes;
    const int sub = threadIdx.x % kPlainLanes;
    const bool active = o < a.n_mp;
    const KfDesc& kd = a.kd;
    const SearchConst& sc = a.sc;
    uint8_t dec = active ? kDecUndecided : (uint8_t)0;
    const int32_t gp = (int32_t)o;
    // the point's loads together; the owner set's first entry is on its way
    // while the point is projected
    int32_t id = 0;
    float x = 0.0f, y = 0.0f, z = 0.0f, dmax = 0.0f;
    uint4 a0 = make_uint4(0, 0, 0, 0), a1 = a0;
    if (active) {
        id = a.mp_id ? ldg(a.mp_id + gp) : gp;
        x = ldg(a.mp_xyz + 3 * o);
        y = ldg(a.mp_xyz + 3 * o + 1);
        z = ldg(a.mp_xyz + 3 * o + 2);
        if (sc.gate) dmax = ldg(a.mp_dmax + o);
        load_desc(a.mp_desc, o, a0, a1);
    }
    __syncthreads();
    const bool probe = active && id >= 0;
    uint32_t hh = owner_slot(id, kd.hash_mask);
    int32_t hv = probe ? ldg(a.hash + hh) : -1;
    Proj p;
    const bool vis = project(kd, x, y, z, dmax, sc.gate, s_sf, sc.N, p);
    Best best;
    best.init();
    int32_t target = -1;
    Window w{};
    if (active && vis) w = make_window(p, kd, s_sf, sc.r0, sc.C, sc.R);
    for (int n = 0; probe && n <= kd.hash_mask && hv >= 0; ++n) {
        if (hv == id) {
            dec = FL_SKIP;
            break;
        }
        hh = (hh + 1) & (uint32_t)kd.hash_mask;
        hv = ldg(a.hash + hh);
    }
    if (dec == kDecUndecided && !vis) dec = FL_NOT_VISIBLE;
    if (dec == kDecUndecided) {
        for (int row = w.r0 + sub % 4; row <= w.r1; row += 4) {
            // a caller-supplied grid is clamped to the keypoint range
            const int s = max(ldg(a.cell_start + row * sc.C + w.c0), 0);
            const int e = min(ldg(a.cell_start + row * sc.C + w.c1 + 1), kd.n_kp);
            for (int i = s + sub / 4; i < e; i += kPlainLanes / 4) {
                const int kp = ldg(a.cell_kp + i);
                if ((unsigned)kp >= (unsigned)kd.n_kp) continue;
                const float kx = ldg(a.kp_xy + 2 * kp), ky = ldg(a.kp_xy + 2 * kp + 1);
                const int oct = ldg(a.kp_oct + kp);
                uint4 b0, b1;
                load_desc(a.kp_desc, kp, b0, b1);
                if (in_window(w, kx, ky, oct, p.pred, sc.gate)) best.offer(hamming(a0, a1, b0, b1), kp);
            }
        }
    }
#pragma unroll
    for (int off = 1; off < kPlainLanes; off <<= 1) {
        const uint32_t key = (uint32_t)__shfl_xor((int)best.key, off);
        const int second = __shfl_xor(best.second, off);
        merge_best(best, key, second);
    }
    if (dec == kDecUndecided) {
        if (!accept_match(best, sc.th, sc.ratio)) {
            dec = FL_NO_MATCH;
        } else {
            const int32_t ow = ldg(a.kp_owner + (best.key & 0xFFFFu));
            if (ow >= 0) {
                dec = FL_FUSE;
                target = ow;
            } else {
                dec = FL_ADD;
            }
        }
    }
    const int bidx = best.key == 0xFFFFFFFFu ? -1 : (int)(best.key & 0xFFFFu);
    const bool write = active && sub == 0;
    if (write) {
        a.best_idx[o] = bidx;
        a.best_dist[o] = (int16_t)(best.key == 0xFFFFFFFFu ? FL_NO_DIST : (int)(best.key >> 16));
        a.second_dist[o] = (int16_t)best.second;
        a.decision[o] = dec;
        a.target[o] = target;
    }
    const bool is_add = write && dec == FL_ADD;
    if (is_add) atomicMin(&a.claim[bidx], gp);
    AddRef e;
    e.pair = (int32_t)o;
    e.kp = bidx < 0 ? 0 : bidx;
    e.gp = gp;
    e.pass = 0;
    wave_append(is_add, a.counter, a.add_list, a.add_cap, e);
}

__global__ __launch_bounds__(256) void resolve_plain_kernel(int32_t n_mp, const uint32_t* __restrict__ counter,
                                                          const AddRef* __restrict__ list, int32_t cap,
                                                          const int32_t* __restrict__ claim,
                                                          const int32_t* __restrict__ mp_id,
                                                          const int32_t* __restrict__ best_idx,
                                                          uint8_t* __restrict__ decision,
                                                          int32_t* __restrict__ target) {
    const uint32_t n = *counter;
    const int stride = gridDim.x * blockDim.x;
    if (n <= (uint32_t)cap) {
        for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
            const AddRef e = list[i];
            const int32_t w = claim[e.kp];
            if (w != e.gp) {
                decision[e.pair] = FL_FUSE;
                target[e.pair] = mp_id ? mp_id[w] : w;
            }
        }
        return;
    }
    for (int32_t o = blockIdx.x * blockDim.x + threadIdx.x; o < n_mp; o += stride) {
        if (decision[o] != FL_ADD) continue;
        const int32_t w = claim[best_idx[o]];
        if (w != o) {
            decision[o] = FL_FUSE;
            target[o] = mp_id ? mp_id[w] : w;
        }
    }
}

}  // namespace fl
