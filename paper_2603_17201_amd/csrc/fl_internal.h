// Internal layouts and device helpers of the fastloop library (gfx950).
//
// The batch descriptor lives in device memory (uploaded once per call from a
// pinned staging buffer); every kernel takes only a pointer to it, so one
// captured HIP graph serves batches of any size up to the workspace capacity.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fastloop.h"

namespace fl {

constexpr int kWave = 64;
constexpr int kMaxQueues = 8;        // one work queue per XCD
constexpr int kNAccPad = 36;        // doubles per partial of a float64 reduction

// One keyframe of a batch: search transform, camera, grid and ranges.
struct alignas(16) KfDesc {
    float A[9];          // sR, row-major
    float t[3];
    float inv_s;
    float fx, fy, cx, cy, W, H;
    float invw, invh;    // grid_cols / W, grid_rows / H (float32, rounded once)
    float T[12];         // world->camera SE3 for refinement (R row-major, t)
    int32_t kp_off;      // first keypoint (global index)
    int32_t n_kp;
    int32_t grid_off;    // first cell_start entry (global-grid mode)
    int32_t event;
    int32_t mp_off;      // first point of the event (global index)
    int32_t n_mp;        // points in the event
    int32_t hash_off;    // owner hash table of this keyframe (global-grid mode)
    int32_t hash_mask;
    int32_t n_tiles;
    int32_t pad0, pad2;
    int32_t pad3;
    int64_t pair_off;
    int64_t n_pairs;
    // A launch may search its batch several times (passes); each (keyframe,
    // pass) has a descriptor of its own, keyframe-major.
    int32_t pass;        // thresholds and outputs: BatchHdr::out[pass]
    int32_t stage_key;   // the keyframe in the batch (its grid is the same in every pass)
    int32_t claim_off;   // first ADD claim slot: pass * n_kp_total + kp_off
    int32_t pad1;
};

// One search pass of a launch: its thresholds and its outputs (caller-owned).
struct PassOut {
    int32_t* best_idx;
    int16_t* best_dist;
    int16_t* second_dist;
    uint8_t* decision;
    int32_t* target;
    int32_t hamming_th;
    float nn_ratio;
    float r0;            // window half-width at octave 0, pixels
    int32_t pad;
};

struct alignas(16) EventDesc {
    int32_t kf_begin, kf_end;
    int32_t mp_off, n_mp;
    int32_t seg_off, seg_n;        // the event's entries of the accepted-pair table
    int64_t pair_begin, pair_end;  // pair range (pairs of the event are contiguous)
    int32_t inv_off, inv_n;        // the event's pairs of the other direction (two-sided refinement)
    int32_t list_cap;              // more accepted pairs than this are taken from the decisions instead
    int32_t pad0;
};

// Offsets in the table blob (which starts at the batch header) of the
// workgroups' tile ranges and of the keyframe table: fixed by the header size
// and the search grid, so a workgroup finds its range and first keyframe
// without first loading pointers.
constexpr size_t kBlobAlign = 256;
__host__ __device__ constexpr size_t blob_align(size_t x) { return (x + kBlobAlign - 1) / kBlobAlign * kBlobAlign; }

// Provisional ADD: a pair whose point claimed a free keypoint.
struct alignas(16) AddRef {
    int32_t pair;     // global pair index
    int32_t kp;       // claim slot of the keypoint (KfDesc::claim_off + index)
    int32_t gp;       // global point index
    int32_t pass;     // search pass (its outputs)
};

// The share of the search launch of one workgroup: tiles [t0, t1) of the
// tile order, the slot of tile t0 and its keyframe descriptor, and the
// workgroup's region of the provisional-ADD and accepted-pair staging lists:
// entries [priv_off, priv_off + priv_cap), as many as the pairs it searches
// (each pair adds at most one entry to each list).
struct alignas(16) WgRange {
    int32_t t0, t1, slot, kf;
    int32_t priv_off, priv_cap;
    int32_t chunk;           // the workgroup's place in the tile order
    int32_t event;           // event of tile t0
    // of the first keyframe, so that neither its keypoints' loads nor the
    // pass's thresholds wait for its descriptor
    int32_t slot_t0, slot_t1;   // tile_prefix[slot], tile_prefix[slot + 1]
    int16_t pass;
    int16_t one_event;          // every tile of the range belongs to `event`
    int32_t stage_key;
    int32_t kp_off, n_kp;
    float invw, invh;
};
static_assert(sizeof(WgRange) == 64, "one cache line");

// The waves of a range's workgroup take its first tiles in turn (tile t0 + w,
// then every kWavesPerWG-th); those from range_shared() on are claimed one
// by one, so that workgroups with nothing left can help.  A claim costs some
// 700 cycles of a tile's 8,000: short ranges, which no one could help in time,
// have none to claim, longer ones their second half.
constexpr int kSharedTiles = 96;   // shortest range with tiles to claim
constexpr int kNoTile = 1 << 30;   // past every tile, with room for a stride on top
__host__ __device__ constexpr int range_shared(int t0, int t1, int waves) {
    return t1 - t0 < kSharedTiles ? t1 : t0 + (t1 - t0) / (2 * waves) * waves;
}

// What has been claimed of a range, and the workgroups that came to help.  A
// 128-byte line each: device-scope atomics on one line serialise (about 12 ns
// apiece).  Cleared by the table fetch.
struct alignas(128) RangeCtr {
    uint32_t claimed, helpers;   // read together as one 64-bit word
};

// The accepted pairs one workgroup staged for one event: entries [start,
// start + count) of the staging list.  Workgroup chunk c and event e meet at
// index c + e of the table (both rise along the tile order, so no two meetings
// share an index).
struct MatchSeg {
    int32_t start, count;
};

// Accepted pair kept for refinement: point, observation, keyframe.
struct alignas(16) MatchRec {
    float x, y, z;
    float u, v;
    int32_t kf;
    int32_t pad0, pad1;
};

// Cell-ordered keypoint record: 16 bytes, one dwordx4 load.  idx is the
// keypoint index within its keyframe.
struct alignas(16) KpRec {
    float x, y;
    int32_t idx;
    int32_t oct;
};

enum : int { kModeGlobal = 0, kModeLdsRec = 1, kModeLdsDesc = 2 };

struct alignas(16) BatchHdr {
    int32_t n_events, n_kf, n_mp, n_kp_total;
    int64_t n_pairs;
    int32_t cells, grid_cols, grid_rows, n_octaves;
    int32_t n_pass;             // search passes of the launch (1 .. FL_MAX_PASSES)
    int32_t gate;               // 1: point distance invariance given (octave gate on)
    int32_t dense;
    int32_t stats;              // 1: count visible / cells / keypoints / candidates
    int32_t lds_hash_mask;      // owner hash capacity - 1 in the LDS modes
    int32_t n_wg;               // workgroups of the search launch
    int32_t refine_iters;       // evaluations per round
    float huber_delta;
    int32_t refine_rounds;      // >= 1; rounds after the first keep the pairs within outlier_px
    float outlier_px;
    float lm_lambda;            // > 0: Levenberg-Marquardt from this damping; 0: Gauss-Newton
    int32_t pad_refine;
    int32_t refine_blocks;      // blocks per event
    int32_t refine_scan;        // 1: take accepted pairs from the decisions, not the list
    int32_t resolve_in_refine;  // 1: the refinement kernel resolves the search's ADD conflicts
    int32_t lds_kp_cap;         // keypoint capacity of the LDS records in the LDS modes
    int32_t oct_buckets;        // octave buckets per grid cell in the LDS modes (1 .. 8)
    int32_t pad_buckets[3];
    float sf[32];               // scale_factor^n rounded to float32
    // tables in the uploaded blob
    const KfDesc* kf;
    const EventDesc* ev;
    const int32_t* kf_order;    // keyframes in tile order
    const int32_t* tile_prefix; // [n_kf+1] first tile of each keyframe in tile order
    const WgRange* wg_range;    // [n_wg] each workgroup's tiles and list regions
    RangeCtr* range_ctr;        // [n_wg] what has been taken of them
    // inputs (caller-owned)
    const float* kp_xy;
    const int8_t* kp_oct;
    const uint8_t* kp_desc;
    const int32_t* kp_owner;
    const float* mp_xyz;
    const uint8_t* mp_desc;
    const float* mp_dmax;
    const int32_t* mp_id;
    const int32_t* pair_mp;
    // thresholds and outputs of each pass
    PassOut out[FL_MAX_PASSES];
    // workspace (library-owned)
    int32_t* cell_start;        // global-grid mode: [n_kf * (cells + 1)]
    KpRec* recs;                // global-grid mode: [n_kp_total]
    uint4* desc_sorted;         // global-grid mode: [n_kp_total * 2]
    int32_t* cell_kp;           // global-grid mode: [n_kp_total]
    int32_t* hash;              // global-grid mode: owner hash tables
    unsigned long long* claim;  // [n_pass * n_kp_total] (epoch << 32 | lowest claiming point)
    const uint32_t* epoch;      // tag of this launch's claims, decremented by the table fetch
    AddRef* add_list;           // per-workgroup regions (WgRange::priv_off)
    uint32_t* add_count;        // [n_wg] entries of each workgroup's ADD region
    MatchRec* match_stage;      // per-workgroup regions of accepted pairs (WgRange::priv_off)
    MatchSeg* match_seg;        // [n_wg + n_events] which of them belong to which event
    unsigned long long* stats_out;  // [4]
    // refinement
    double* event_S;            // [n_events][13] caller's, in/out
    fl_sim3* event_S32_out;     // caller's (may be null)
    int32_t* event_n_matched;   // caller's (may be null)
    unsigned long long* refine_rows;   // [2][n_events * refine_blocks][kRefWords] tagged partial-sum words
    // two-sided refinement (caller's; null without it): points of the other
    // side observed through S^-1 in keyframes of their own
    const float* inv_xyz;       // [n][3]
    const float* inv_uv;        // [n][2]
    const int32_t* inv_kf;      // [n] into inv_T / inv_cam
    const float* inv_T;         // [inv_n_kf][12]
    const float* inv_cam;       // [inv_n_kf][4] fx, fy, cx, cy
    int32_t inv_n_kf;
    int32_t pad_inv[3];
};

__host__ __device__ constexpr size_t blob_range_offset() { return blob_align(sizeof(BatchHdr)); }
__host__ __device__ constexpr size_t blob_kf_offset(int grid) {
    return blob_align(blob_range_offset() + sizeof(WgRange) * (size_t)(grid > 1 ? grid : 1));
}


// ---------------------------------------------------------------------------
// float32 helpers whose rounding is fixed: every multiply-add written as
// fmaf is one fused operation, every other operation rounds on its own (the
// library is compiled with -ffp-contract=off).

// floor(x * inv) clamped to [0, n): a negative or NaN product gives cell 0.
// Clamped in float first (the median of the product and both ends; of a NaN
// and the ends it is the lower end), where the conversion's truncation is the
// floor.
__device__ __forceinline__ int cell_of(float x, float inv, int n) {
    return (int)__builtin_amdgcn_fmed3f(x * inv, 0.0f, (float)(n - 1));
}

struct Proj {
    float u, v, d;
    int pred;
};

// Transform by the keyframe's Sim3, pinhole projection and image test:
// false when the point is not visible (u, v and d are then of no meaning);
// u, v and the metric distance d otherwise.  Straight-line code: a wave
// leaves it early only if none of its 64 points is visible.
__device__ __forceinline__ bool project_uv(const KfDesc& k, float x, float y, float z, Proj& p) {
    const float q0 = fmaf(k.A[2], z, fmaf(k.A[1], y, fmaf(k.A[0], x, k.t[0])));
    const float q1 = fmaf(k.A[5], z, fmaf(k.A[4], y, fmaf(k.A[3], x, k.t[1])));
    const float q2 = fmaf(k.A[8], z, fmaf(k.A[7], y, fmaf(k.A[6], x, k.t[2])));
    const float iz = 1.0f / q2;
    p.u = fmaf(k.fx, q0 * iz, k.cx);
    p.v = fmaf(k.fy, q1 * iz, k.cy);
    p.d = sqrtf(fmaf(q0, q0, fmaf(q1, q1, q2 * q2))) * k.inv_s;
    return (q2 > 0.0f) & (p.u >= 0.0f) & (p.u < k.W) & (p.v >= 0.0f) & (p.v < k.H);
}

// Transform, projection, image test and predicted octave: the first n with
// d * sf[n] >= dmax, else N - 1 (gate off: N - 1).
__device__ __forceinline__ bool project(const KfDesc& k, float x, float y, float z, float dmax, int gate,
                                        const float* sf, int N, Proj& p) {
    if (!project_uv(k, x, y, z, p)) return false;
    int pred = N - 1;
    if (gate) {
        for (int n = 0; n < N; ++n) {
            if (p.d * sf[n] >= dmax) { pred = n; break; }
        }
    }
    p.pred = pred;
    return true;
}

__device__ __forceinline__ int hamming(const uint4& a0, const uint4& a1, const uint4& b0, const uint4& b1) {
    int h = __popc(a0.x ^ b0.x);
    h += __popc(a0.y ^ b0.y);
    h += __popc(a0.z ^ b0.z);
    h += __popc(a0.w ^ b0.w);
    h += __popc(a1.x ^ b1.x);
    h += __popc(a1.y ^ b1.y);
    h += __popc(a1.z ^ b1.z);
    h += __popc(a1.w ^ b1.w);
    return h;
}

// Running best / second best over packed keys (h << 16 | idx): the minimum
// key is the lexicographic minimum of (distance, keypoint index), so the
// result does not depend on the order candidates are visited in.
struct Best {
    uint32_t key;   // 0xFFFFFFFF: none
    int second;     // FL_NO_DIST: none
    __device__ __forceinline__ void init() {
        key = 0xFFFFFFFFu;
        second = FL_NO_DIST;
    }
    __device__ __forceinline__ void offer(int h, int idx) {
        const uint32_t k = ((uint32_t)h << 16) | (uint32_t)idx;
        if (k < key) {
            if (key != 0xFFFFFFFFu) second = min(second, (int)(key >> 16));
            key = k;
        } else {
            second = min(second, h);
        }
    }
};

__device__ __forceinline__ uint32_t hash_id(int32_t id) {
    return (uint32_t)id * 0x9E3779B1u;
}

// Tag of the refinement's partial-sum words: the low kTagEpochBits bits of
// the launch epoch (decremented by every table fetch) above ten bits of
// step number (step + 1 < 1024).  Tags repeat every 2^kTagEpochBits
// launches, so the host zeroes the partial-sum rows before every launch
// whose count is a multiple of that period (refine_rows_cleared_before):
// between two clears no two launches share a tag, and a zeroed word (tag 0)
// matches none.
constexpr uint32_t kTagEpochBits = 22;
__host__ __device__ constexpr uint32_t refine_tag(uint32_t epoch, int step) {
    return (epoch << 10) | (uint32_t)(step + 1);
}
__host__ __device__ constexpr bool refine_rows_cleared_before(uint32_t launches) {
    return (launches & ((1u << kTagEpochBits) - 1u)) == 0u;
}

__device__ __forceinline__ int wave_lane() { return threadIdx.x & (kWave - 1); }

// Between a wave's LDS stores and its lanes' loads of each other's values (or
// such loads and the next stores): one wave's LDS accesses complete in order,
// so no instruction is needed, but the compiler must keep theirs, which it
// otherwise only does while it cannot tell the addresses apart.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Global-memory accesses through the global address space: the compiler
// then issues global (not flat) loads and stores, with a scalar base where
// it can.
template <typename T>
using gmem = __attribute__((address_space(1))) T;
template <typename T>
__device__ __forceinline__ T ldg(const T* p) {
    return *(const gmem<T>*)p;   // address-space cast: generic to global
}
template <typename T>
__device__ __forceinline__ void stg(T* p, const T& v) {
    *(gmem<T>*)p = v;
}
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ldg_u4(const uint4* p) {
    const v4u x = *(const gmem<v4u>*)p;
    return make_uint4(x.x, x.y, x.z, x.w);
}
// A record of n 16-byte units stored with n dwordx4 global stores.
template <typename T>
__device__ __forceinline__ void stg_rec(T* p, const T& v) {
    static_assert(sizeof(T) % 16 == 0, "whole 16-byte units");
    const v4u* src = reinterpret_cast<const v4u*>(&v);
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 16; ++i) ((gmem<v4u>*)p)[i] = src[i];
}

// A value known to be the same in every lane, moved to a scalar register
// (the compiler cannot always tell that a loaded value is uniform, and
// would otherwise hold it in a vector register of every lane).
__device__ __forceinline__ int32_t uniform_i(int32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ float uniform_f(float x) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}
__device__ __forceinline__ int64_t uniform_l(int64_t x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
template <typename T>
__device__ __forceinline__ T* uniform_p(T* p) {
    return reinterpret_cast<T*>(uniform_l((int64_t)reinterpret_cast<uintptr_t>(p)));
}

// Tables that no one writes while a kernel runs, read through the constant
// address space: with a uniform address these are scalar loads, from the
// scalar cache.  `fresh` hides the pointer's origin, so the loads stay where
// they are written.  A loop with more uniform values than there are scalar
// registers reads them where it needs them: hoisted out of it they would be
// kept in lanes of vector registers, and every use would be a vector
// instruction.
template <typename T>
using cmem = const __attribute__((address_space(4))) T;
template <typename T>
__device__ __forceinline__ cmem<T>* fresh(const T* p) {
    uint64_t a = reinterpret_cast<uint64_t>(p);
    asm volatile("" : "+s"(a));
    return (cmem<T>*)a;
}

// The search fields of a keyframe descriptor.
__device__ __forceinline__ KfDesc search_kf(cmem<KfDesc>* s) {
    KfDesc k;
#pragma unroll
    for (int i = 0; i < 9; ++i) k.A[i] = s->A[i];
#pragma unroll
    for (int i = 0; i < 3; ++i) k.t[i] = s->t[i];
    k.inv_s = s->inv_s;
    k.fx = s->fx;
    k.fy = s->fy;
    k.cx = s->cx;
    k.cy = s->cy;
    k.W = s->W;
    k.H = s->H;
    k.invw = s->invw;
    k.invh = s->invh;
#pragma unroll
    for (int i = 0; i < 12; ++i) k.T[i] = 0.0f;   // not used by the search
    k.kp_off = s->kp_off;
    k.n_kp = s->n_kp;
    k.grid_off = s->grid_off;
    k.event = s->event;
    k.mp_off = s->mp_off;
    k.n_mp = s->n_mp;
    k.hash_off = s->hash_off;
    k.hash_mask = s->hash_mask;
    k.n_tiles = s->n_tiles;
    k.pad0 = k.pad1 = k.pad2 = k.pad3 = 0;
    k.pair_off = s->pair_off;
    k.n_pairs = s->n_pairs;
    k.pass = s->pass;
    k.stage_key = s->stage_key;
    k.claim_off = s->claim_off;
    return k;
}

// Inclusive prefix sum over the 64 lanes of a wave: shifts by 1, 2, 4, 8
// lanes inside each row of 16 (DPP row_shr), then the last lane of row 0 is
// added to row 1 and of row 2 to row 3 (row_bcast:15), and the last lane of
// row 1 to rows 2 and 3 (row_bcast:31).  Lanes with no source add 0.  Every
// lane of the wave must be active.
__device__ __forceinline__ int wave_incl_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15, rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31, rows 2 and 3
    return x;
}

// ADD conflicts, resolved by a kernel that runs after the whole batched
// search on the same stream.  Of the provisional ADDs on one keypoint the
// lowest point index (the claim it left, tagged with the launch epoch) keeps
// ADD; the others become FUSE to that point (Sec. IV-D3, with the
// lowest-index reading of concurrent additions).  Workgroup r of the search
// listed its provisional ADDs in its region of the ADD list; every thread of
// the calling workgroup takes part.
__device__ inline void resolve_region_adds(const BatchHdr& h, int r, unsigned long long tag) {
    const WgRange g = h.wg_range[r];
    const uint32_t n = h.add_count[r];
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
        const AddRef e = h.add_list[g.priv_off + i];
        const int32_t w = (int32_t)(h.claim[e.kp] - tag);
        if (w != e.gp) {
            const PassOut& po = h.out[e.pass];
            po.decision[e.pair] = FL_FUSE;
            po.target[e.pair] = h.mp_id ? h.mp_id[w] : w;
        }
    }
}

}  // namespace fl
