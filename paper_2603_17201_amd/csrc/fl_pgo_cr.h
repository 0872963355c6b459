// Block cyclic reduction of the essential graph's damped normal equations.
//
// The band solves of fl_pgo.h factor one block column after another in one
// workgroup: a chain as long as the graph.  Here the free keyframes, in their
// band order, are cut into N blocks of B >= b consecutive positions (no edge
// spans more than b), so H is block tridiagonal with dense blocks of
// m = 16 NT >= 7 B scalars (the rows beyond 7 B, and those of positions the
// last block does not have, are held: unit diagonal, zero right-hand side).
// A level eliminates every second block, all at once:
//   cr_eliminate_kernel  A_mm = L L^T and, for the block's neighbours l and r,
//                        Y_l = A_lm L^-T, Y_r = A_rm L^-T, L^-T itself and
//                        y = L^-1 b_m: the rows of [A_lm; A_rm; I; b^T], each
//                        multiplied by L^-T from the right;
//   cr_update_kernel     of the blocks that stay: A_ll -= Y_l Y_l^T (from the
//                        block to its right), A_ll -= Y_r Y_r^T (from the one
//                        to its left), the new coupling A_rl = -Y_r Y_l^T and
//                        the right-hand sides;
// and after ceil(log2 N) levels one block is left.  The unknowns follow from
// the last level back: x_m = L^-T (y - Y_l^T x_l - Y_r^T x_r), two products
// and no triangular solve (cr_back_kernel).  This is a Cholesky factorisation
// under a nested-dissection order: every sum has a fixed order, and a pivot
// that is not positive marks the solve failed.
//
// What bounds it: latency.  A level costs three launches and NT dependent
// panel steps of 16 columns; the arithmetic (about 6 m^3 fused multiply-adds
// per block, on the float64 matrix instructions) is a few microseconds.  On
// 1,000 keyframes, per level: one lap (N = 167 blocks of 48, 8 levels)
// eliminate 9.9, update 4.8, back 4.4 us, three laps (40 blocks of 176, 6
// levels) 57, 12.4 and 13.3 us; a whole iteration 0.22 and 0.65 ms, where the
// band solves took 3.65 and 9.7 ms.
#pragma once

#include <algorithm>

#include "fl_pgo.h"

namespace fl {

typedef double v4d __attribute__((ext_vector_type(4)));

struct CrArgs {
    int32_t n_blocks;   // N
    int32_t block_pos;  // B, band positions of a block
    int32_t n_pos;      // free keyframes
    int32_t m;          // 16 NT
    double* D;          // [N][m][m] diagonal blocks (lower tiles; whole diagonal tiles)
    double* C;          // [N][m][m] C[i]: rows of the next active block, columns of block i; Y_r of an eliminated one
    double* YL;         // [N][m][m] Y_l of an eliminated block (row-major: rows of its left neighbour)
    double* LI;         // [N][m][m] L^-1 of an eliminated block (the transpose of L^-T)
    double* b;          // [N][m] right-hand sides, then y
    double* x;          // [N][m]
    double* lm;         // Levenberg-Marquardt state (kLmFail; kLmUsed stays the 0 it is set to at the start)
};

constexpr int kCrWaves = 8;            // waves of an elimination workgroup
constexpr int kCrTile = 16 * 17;       // doubles of a tile in LDS (rows of 17)
constexpr int kCrUpdBlock = 256;
constexpr int kCrBackBlock = 1024;
constexpr int kCrFillBlock = 256;
constexpr int64_t kCrMaxEntries = 1 << 25;   // entries of one of the four block arrays (1 GiB in all)

// Tile rows of [Y_l; Y_r; I; b] a workgroup carries beside the triangle of
// A_mm, which every workgroup of a block factors for itself (that costs no
// time, the triangle's chain is the same in all, and no exchange is needed).
// A wave keeps its tiles in registers for the whole elimination: with 8 waves a
// thread holds (NT (NT + 1) / 2 + XR NT) / 8 tiles of 4 doubles, which fills
// the 256 registers at NT = 11.  Of the two widest shapes the compiler spills
// 6 (NT = 14) and 93 of them (NT = 16).
constexpr int cr_rows(int nt) { return nt >= 14 ? 2 : nt >= 11 ? 4 : 5; }
constexpr int cr_groups(int nt) { return (3 * nt + 1 + cr_rows(nt) - 1) / cr_rows(nt); }

// 1 / sqrt(d) from the hardware estimate r (relative error below 2^-22) and
// one step of third order, r (1 + e / 2 + 3 e^2 / 8) with e = 1 - d r^2.
__device__ __forceinline__ double cr_rsqrt(double d) {
    const double r = __builtin_amdgcn_rsq(d);
    const double e = fma(-d * r, r, 1.0);
    return fma(r * e, fma(0.375, e, 0.5), r);
}

// Cholesky of the 16 x 16 tile c (accumulator layout) by one wave, four
// columns at a time: every lane factors the 4 x 4 diagonal block and inverts
// its factor for itself (its entries read by all from LDS), lane (row lc, k =
// lr) then holds entry k of its row of the four columns times the inverse,
// which is both operands' layout of the one matrix instruction that updates
// the rest.  Identity rows taken along come out as the rows of L^-T, in sM.
// (4,000 to 5,000 cycles a tile; column by column, with the values passed
// between lanes by readlane, it took 5,000 to 14,000, two thirds of a step.)
// Entries above the diagonal are never used.  Returns whether every pivot was
// positive.
__device__ __forceinline__ bool cr_factor_tile(v4d c, double* sD, double* sX, double* sM) {
    const int l = wave_lane(), lr = l >> 4, lc = l & 15;
    v4d X;
#pragma unroll
    for (int r = 0; r < 4; ++r) X[r] = lr + 4 * r == lc ? 1.0 : 0.0;
    bool ok = true;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            sD[(lr + 4 * r) * 17 + lc] = c[r];
            sX[(lr + 4 * r) * 17 + lc] = X[r];
        }
        wave_lds_sync();
        const double* a = sD + 4 * s * 18;   // the diagonal block, rows of 17
        double d[4], x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            d[q] = sD[lc * 17 + 4 * s + q];
            x[q] = sX[lc * 17 + 4 * s + q];
        }
        const double a10 = a[17], a20 = a[34], a30 = a[51], a21 = a[35], a31 = a[52], a32 = a[53];
        const double r0 = cr_rsqrt(a[0]), l10 = a10 * r0, l20 = a20 * r0, l30 = a30 * r0;
        const double p1 = fma(-l10, l10, a[18]);
        const double r1 = cr_rsqrt(p1), l21 = fma(-l20, l10, a21) * r1, l31 = fma(-l30, l10, a31) * r1;
        const double p2 = fma(-l21, l21, fma(-l20, l20, a[36]));
        const double r2 = cr_rsqrt(p2), l32 = fma(-l31, l21, fma(-l30, l20, a32)) * r2;
        const double p3 = fma(-l32, l32, fma(-l31, l31, fma(-l30, l30, a[54])));
        const double r3 = cr_rsqrt(p3);
        ok = ok && a[0] > 0.0 && p1 > 0.0 && p2 > 0.0 && p3 > 0.0;   // the same in every lane
        // row k of L^-1 = column k of L^-T
        const double i10 = -r1 * (l10 * r0), i21 = -r2 * (l21 * r1), i32 = -r3 * (l32 * r2);
        const double i20 = -r2 * fma(l21, i10, l20 * r0), i31 = -r3 * fma(l32, i21, l31 * r1);
        const double i30 = -r3 * fma(l32, i20, fma(l31, i10, l30 * r0));
        const double m0 = lr == 0 ? r0 : lr == 1 ? i10 : lr == 2 ? i20 : i30;
        const double m1 = lr == 0 ? 0.0 : lr == 1 ? r1 : lr == 2 ? i21 : i31;
        const double m2 = lr < 2 ? 0.0 : lr == 2 ? r2 : i32;
        const double m3 = lr < 3 ? 0.0 : r3;
        const double P = fma(d[3], m3, fma(d[2], m2, fma(d[1], m1, d[0] * m0)));
        const double Q = fma(x[3], m3, fma(x[2], m2, fma(x[1], m1, x[0] * m0)));
        sM[lc * 17 + 4 * s + lr] = Q;
        if (s < 3) {
            c = __builtin_amdgcn_mfma_f64_16x16x4f64(-P, P, c, 0, 0, 0);
            X = __builtin_amdgcn_mfma_f64_16x16x4f64(-Q, P, X, 0, 0, 0);
            wave_lds_sync();
        }
    }
    return ok;
}

// One level: block t = 2 u + 1 of the n_active blocks 0, s, 2 s, ... is
// eliminated by the cr_groups(NT) workgroups of u (last: the one block left,
// block 0, which has no neighbours).  Per panel step k of 16 columns: the
// panel tiles (rows below, and the X rows) times L_kk^-T, one barrier, then
// every tile (i, j > k) -= P_i P_j^T; one barrier.  Wave 0 holds the diagonal
// tiles: it updates the next one first and factors it beside the other waves'
// updates.
template <int NT>
__global__ __launch_bounds__(kCrWaves * 64) void cr_eliminate_kernel(CrArgs a, int s, int n_active, int last) {
    constexpr int XR = cr_rows(NT), G = cr_groups(NT), M = 16 * NT, MM = M * M;
    constexpr int TT = NT * (NT + 1) / 2, XT = XR * NT;
    constexpr int OW = kCrWaves - 1;   // waves of the tiles off the diagonal
    constexpr int TQ = std::max(NT, (TT - NT + XT + OW - 1) / OW);   // tiles of a wave
    __shared__ double sP[(NT + XR) * kCrTile];
    __shared__ double sM[2][kCrTile];
    __shared__ double sD[kCrTile], sX[kCrTile];
    const int u = (int)blockIdx.x / G, grp = (int)blockIdx.x % G;
    const int t = last ? 0 : 2 * u + 1;
    const bool has_l = !last, has_r = !last && t + 1 < n_active;
    const int64_t mb = (int64_t)t * s, lb = mb - s;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int l = wave_lane(), lr = l >> 4, lc = l & 15;

    // kind of X tile row r of this workgroup: 0 Y_l, 1 Y_r, 2 I, 3 b, 4 none
    auto kind_of = [&](int xr, int& row) {
        const int gr = grp * XR + xr;
        const int kd = gr < 3 * NT ? gr / NT : gr == 3 * NT ? 3 : 4;
        row = gr < 3 * NT ? gr % NT : 0;
        if ((kd == 0 && !has_l) || (kd == 1 && !has_r)) return 4;
        return kd;
    };
    {
        bool any = false;   // the same in every thread
        for (int xr = 0; xr < XR; ++xr) {
            int row;
            any = any || kind_of(xr, row) != 4;
        }
        if (!any) return;
    }

    // this wave's tiles: wave 0 the diagonal ones, wave 1 + w of the others,
    // in column order (of column j its NT - 1 - j triangle tiles, then its XR
    // X tiles), w, w + 7, ...; packed in one scalar each: panel row i (X rows
    // from NT) << 8 | column, of an X tile also 1 + kind << 24 | tile row of
    // the kind << 16; -1: none
    v4d tile[TQ];
    int tk[TQ];
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
        int id = w - 1 + OW * q, j = 0;
        // one load for every kind (what a kind does not use is masked below),
        // so that all tiles' loads are in flight together: A_mm, A_ml
        // transposed, A_rm, the right-hand side in row 0
        const double* d = a.D + mb * MM;
        int rs = M, cs = 1;
        tk[q] = -1;
        if (w == 0) {
            if (q < NT) tk[q] = q << 8 | q;
        } else if (id < TT - NT + XT) {
            while (id >= NT - 1 - j + XR) id -= NT - 1 - j++ + XR;
            if (id < NT - 1 - j) {
                tk[q] = (j + 1 + id) << 8 | j;
            } else {
                id -= NT - 1 - j;
                int row;
                const int kd = kind_of(id, row);
                if (kd != 4) tk[q] = (kd + 1) << 24 | row << 16 | (NT + id) << 8 | j;
                if (kd == 0) {
                    d = a.C + lb * MM + 16 * j * M + 16 * row;
                    rs = 1;
                    cs = M;
                } else if (kd == 1) {
                    d = a.C + mb * MM + 16 * row * M + 16 * j;
                } else if (kd == 3) {
                    d = a.b + mb * M + 16 * j;
                    rs = 0;
                }
            }
        }
        if (tk[q] >= 0 && tk[q] >> 24 == 0) d += 16 * (tk[q] >> 8) * M + 16 * (tk[q] & 255);
#pragma unroll
        for (int r = 0; r < 4; ++r) tile[q][r] = d[(lr + 4 * r) * rs + lc * cs];
    }
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
        const int kd = (tk[q] >> 24) - 1, row = tk[q] >> 16 & 255, j = tk[q] & 255;
        if (kd >= 2) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                tile[q][r] = kd == 3 ? (lr + 4 * r == 0 ? tile[q][r] : 0.0) : (row == j && lr + 4 * r == lc ? 1.0 : 0.0);
        }
    }

    bool ok = true;
    // This lane's places in a tile: op (lr, lc) of the accumulator layout (the
    // other rows 4, 8, 12 below), oa (lc, lr) of both operands' layouts, og
    // (lr, lc) of a block in memory.
    int op = lr * 17 + lc, oa = lc * 17 + lr, og = lr * M + lc;
    auto put = [&](double* t, const v4d& v) {
#pragma unroll
        for (int r = 0; r < 4; ++r) t[op + 4 * 17 * r] = v[r];
    };
    if (w == 0) ok = cr_factor_tile(tile[0], sD, sX, sM[0]);
    __syncthreads();
    // a panel tile times L_kk^-T: through LDS into the left operand's layout
    auto panel = [&](const v4d& v, double* t, const double* Mk) {
        put(t, v);
        wave_lds_sync();
        v4d c = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            c = __builtin_amdgcn_mfma_f64_16x16x4f64(t[oa + 4 * kk], Mk[op + 4 * 17 * kk], c, 0, 0, 0);
        wave_lds_sync();
        put(t, c);
        return c;
    };
    auto update = [&](v4d c, const double* Pi, const double* Pj) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            c = __builtin_amdgcn_mfma_f64_16x16x4f64(-Pi[oa + 4 * kk], Pj[oa + 4 * kk], c, 0, 0, 0);
        return c;
    };
#pragma unroll 1
    for (int k = 0; k < NT; ++k) {
        const double* Mk = sM[k & 1];
        // (an offset the compiler cannot follow through the step: it would
        // otherwise keep every tile's addresses in registers for the whole
        // loop and spill them)
        asm volatile("" : "+v"(op), "+v"(oa), "+v"(og));
        // of this wave's tiles, those before q0 lie in columns before k, those
        // from q1 on in columns after it (wave 0: its tile k + 1 is q1)
        const int before = k * (NT - 1 + XR) - k * (k - 1) / 2, upto = before + NT - 1 - k + XR;
        const int q0 = w == 0 ? k + 1 : (before - w + OW) / OW, q1 = w == 0 ? k + 1 : (upto - w + OW) / OW;
        // (four tiles at a time: a branch taken over each tile that has no
        // part in the step costs as much as a matrix instruction)
#pragma unroll
        for (int g = 0; g < TQ; g += 4) {
            if (g + 4 <= q0 || g >= q1) continue;
#pragma unroll
            for (int q = g; q < std::min(g + 4, TQ); ++q) {
                if (q < q0 || q >= q1 || tk[q] < 0) continue;
                const int i = tk[q] >> 8 & 255;
                const v4d c = panel(tile[q], sP + i * kCrTile, Mk);
                const int kd = (tk[q] >> 24) - 1, row = tk[q] >> 16 & 255;
                if (kd < 0) continue;
                if (kd == 3) {
                    if (lr == 0) a.b[mb * M + 16 * k + lc] = c[0];
                } else if (kd == 2) {   // transposed
                    wave_lds_sync();
                    double* d = a.LI + mb * MM + 16 * k * M + 16 * row;
#pragma unroll
                    for (int r = 0; r < 4; ++r) d[og + 4 * r * M] = sP[i * kCrTile + oa + 4 * r];
                } else {
                    double* d = (kd == 0 ? a.YL : a.C) + mb * MM + 16 * row * M + 16 * k;
#pragma unroll
                    for (int r = 0; r < 4; ++r) d[og + 4 * r * M] = c[r];
                }
            }
        }
        if (k == NT - 1) break;
        __syncthreads();
        if (w == 0) {
            __builtin_amdgcn_s_setprio(3);   // the step's longest chain
            v4d nd = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int q = 0; q < NT; ++q)
                if (q == k + 1) nd = tile[q];
            nd = update(nd, sP + (k + 1) * kCrTile, sP + (k + 1) * kCrTile);
            ok = cr_factor_tile(nd, sD, sX, sM[(k + 1) & 1]) && ok;
            __builtin_amdgcn_s_setprio(0);
        }
        const int qu = q1 + (w == 0);
#pragma unroll
        for (int g = 0; g < TQ; g += 4) {
            if (g + 4 <= qu) continue;
#pragma unroll
            for (int q = g; q < std::min(g + 4, TQ); ++q)
                if (q >= qu && tk[q] >= 0)
                    tile[q] = update(tile[q], sP + (tk[q] >> 8 & 255) * kCrTile, sP + (tk[q] & 255) * kCrTile);
        }
        __syncthreads();
    }
    if (!ok && l == 0) a.lm[kLmFail] = 1.0;
}

// Sum over k of P_i[row][k] P_j[col][k] for 16 x 16 entries, P_i and P_j 16
// rows of M doubles: lane group lr takes columns 16 q + 4 lr .. + 3 of both,
// 32 consecutive bytes a lane (any order of k serves, the same in both).
template <int NT, bool VEC>
__device__ __forceinline__ v4d cr_product(v4d c, const double* Pi, const double* Pj, double sign) {
    const int l = wave_lane(), lr = l >> 4, lc = l & 15;
    const double* pa = Pi + (int64_t)lc * (16 * NT) + 4 * lr;
    const double* pb = VEC ? Pj + 4 * lr : Pj + (int64_t)lc * (16 * NT) + 4 * lr;
#pragma unroll 4
    for (int q = 0; q < NT; ++q) {
        v4d x = *(const v4d*)(pa + 16 * q), y = *(const v4d*)(pb + 16 * q);
        if (VEC && lc != 0) y = v4d{0.0, 0.0, 0.0, 0.0};   // a vector: column 0 only
#pragma unroll
        for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f64_16x16x4f64(sign * x[e], y[e], c, 0, 0, 0);
    }
    return c;
}

// The blocks that stay, t = 2 blockIdx.y: one wave per tile of the new A_tt
// (lower), of the new coupling to block t + 2, and per 16 rows of the
// right-hand side.
template <int NT>
__global__ __launch_bounds__(kCrUpdBlock) void cr_update_kernel(CrArgs a, int s, int n_active) {
    constexpr int M = 16 * NT, MM = M * M, TT = NT * (NT + 1) / 2;
    const int t = 2 * (int)blockIdx.y;
    const int l = wave_lane(), lr = l >> 4, lc = l & 15;
    int id = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kCrUpdBlock / kWave) + threadIdx.x / kWave));
    const int64_t kb = (int64_t)t * s, pb = kb - s, nb = kb + s;   // this block, the ones eliminated beside it
    const bool has_p = t > 0, has_n = t + 1 < n_active, has_r = t + 2 < n_active;
    if (id < TT) {
        int j = 0;
        while (id >= NT - j) id -= NT - j++;
        const int i = j + id;
        double* d = a.D + kb * MM + (int64_t)(16 * i) * M + 16 * j;
        v4d c;
#pragma unroll
        for (int r = 0; r < 4; ++r) c[r] = d[(lr + 4 * r) * M + lc];
        if (has_p) c = cr_product<NT, false>(c, a.C + pb * MM + 16 * i * M, a.C + pb * MM + 16 * j * M, -1.0);
        if (has_n) c = cr_product<NT, false>(c, a.YL + nb * MM + 16 * i * M, a.YL + nb * MM + 16 * j * M, -1.0);
#pragma unroll
        for (int r = 0; r < 4; ++r) d[(lr + 4 * r) * M + lc] = c[r];
        return;
    }
    id -= TT;
    if (id < NT * NT) {
        if (!has_r) return;
        const int i = id / NT, j = id % NT;
        v4d c = {0.0, 0.0, 0.0, 0.0};
        c = cr_product<NT, false>(c, a.C + nb * MM + 16 * i * M, a.YL + nb * MM + 16 * j * M, -1.0);
        double* d = a.C + kb * MM + (int64_t)(16 * i) * M + 16 * j;
#pragma unroll
        for (int r = 0; r < 4; ++r) d[(lr + 4 * r) * M + lc] = c[r];
        return;
    }
    id -= NT * NT;
    if (id < NT) {
        double* d = a.b + kb * M + 16 * id;
        v4d c = {0.0, 0.0, 0.0, 0.0};
        if (lc == 0)
#pragma unroll
            for (int r = 0; r < 4; ++r) c[r] = d[lr + 4 * r];
        if (has_p) c = cr_product<NT, true>(c, a.C + pb * MM + 16 * id * M, a.b + pb * M, -1.0);
        if (has_n) c = cr_product<NT, true>(c, a.YL + nb * MM + 16 * id * M, a.b + nb * M, -1.0);
        if (lc == 0)
#pragma unroll
            for (int r = 0; r < 4; ++r) d[lr + 4 * r] = c[r];
    }
}

// x_m = L^-T (y - Y_l^T x_l - Y_r^T x_r) of the blocks a level eliminated:
// thread (seg, j) sums the rows p = seg, seg + SEG, ... of column j of both
// products, then of L^-1; the segments are added in order.
template <int NT>
__global__ __launch_bounds__(kCrBackBlock) void cr_back_kernel(CrArgs a, int s, int n_active, int last) {
    constexpr int M = 16 * NT, MM = M * M, SEG = kCrBackBlock / M, RS = (M + SEG - 1) / SEG;
    __shared__ double sx[2 * M];
    __shared__ double sz[M];
    __shared__ double sp[SEG * M];
    const int t = last ? 0 : 2 * (int)blockIdx.x + 1;
    const bool has_l = !last, has_r = !last && t + 1 < n_active;
    const int64_t mb = (int64_t)t * s;
    const int tid = threadIdx.x, seg = tid / M, j = tid % M;
    if (tid < M) {
        sx[tid] = has_l ? a.x[(mb - s) * M + tid] : 0.0;
        sx[M + tid] = has_r ? a.x[(mb + s) * M + tid] : 0.0;
    }
    __syncthreads();
    if (seg < SEG) {
        double v = 0.0;
        if (has_l) {
            const double* Y = a.YL + mb * MM + j;
#pragma unroll
            for (int q = 0; q < RS; ++q) {
                const int p = seg + SEG * q;
                if (p < M) v = fma(Y[p * M], sx[p], v);
            }
        }
        if (has_r) {
            const double* Y = a.C + mb * MM + j;
#pragma unroll
            for (int q = 0; q < RS; ++q) {
                const int p = seg + SEG * q;
                if (p < M) v = fma(Y[p * M], sx[M + p], v);
            }
        }
        sp[seg * M + j] = v;
    }
    __syncthreads();
    if (tid < M) {
        double v = a.b[mb * M + tid];
        for (int q = 0; q < SEG; ++q) v -= sp[q * M + tid];
        sz[tid] = v;
    }
    __syncthreads();
    if (seg < SEG) {
        const double* T = a.LI + mb * MM + j;
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < RS; ++q) {
            const int p = seg + SEG * q;
            if (p < M) v = fma(T[p * M], sz[p], v);
        }
        sp[seg * M + j] = v;
    }
    __syncthreads();
    if (tid < M) {
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < SEG; ++q) v += sp[q * M + tid];
        a.x[mb * M + tid] = v;
    }
}

// Zero the blocks, the couplings and the right-hand sides; unit diagonal in
// the rows no free keyframe has.
__global__ __launch_bounds__(kCrFillBlock) void cr_fill_kernel(CrArgs a) {
    const int m = a.m;
    const int64_t mm = (int64_t)m * m, total = a.n_blocks * mm;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < total; q += stride) {
        const int64_t blk = q / mm;
        const int e = (int)(q - blk * mm), row = e / m, col = e - row * m;
        const bool held = row >= 7 * a.block_pos || blk * a.block_pos + row / 7 >= a.n_pos;
        a.D[q] = row == col && held ? 1.0 : 0.0;
        a.C[q] = 0.0;
        if (col == 0) a.b[blk * m + row] = 0.0;
    }
}

// Rows 7 P .. 7 P + 6 of the normal equations (free node n at position P),
// one wave per node, lane 7 r + c entry (r, c) of the 7 x 7 blocks: (J_a^T
// J_a)[r][c] over the node's incident edges in their order on the diagonal,
// (J_a^T J_b)[r][c] of each edge to a free node at an earlier position in
// that node's columns, lambda on the diagonal, -g on the right.  A node
// without edges is held.
__global__ __launch_bounds__(256) void cr_assemble_kernel(PgoArgs a, CrArgs cr) {
    const int P = (int)(blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave);
    if (P >= cr.n_pos) return;
    const int n = a.order[P], l = wave_lane();
    const bool ent = l < 49, rhs = l >= 49 && l < 56;
    const int r = ent ? l / 7 : l - 49, c = ent ? l % 7 : 0;
    const int B = cr.block_pos, m = cr.m;
    const int64_t blk = P / B, mm = (int64_t)m * m;
    const int row = 7 * (int)(P - blk * B) + r;
    double acc = 0.0, gr = 0.0;
    const int t0 = a.adj_off[n], t1 = a.adj_off[n + 1];
    if (ent || rhs)
        for (int t = t0; t < t1; ++t) {
            const int k = a.adj[t] >> 1, side = a.adj[t] & 1;
            const double* Ja = a.J + 98 * (int64_t)k + 49 * side;
            const double* Jb = a.J + 98 * (int64_t)k + 49 * (1 - side);
            double ja[7];
#pragma unroll
            for (int rr = 0; rr < 7; ++rr) ja[rr] = Ja[7 * rr + r];
            if (rhs) {
#pragma unroll
                for (int rr = 0; rr < 7; ++rr) gr = fma(ja[rr], a.e[7 * (int64_t)k + rr], gr);
                continue;
            }
            double v = 0.0;
#pragma unroll
            for (int rr = 0; rr < 7; ++rr) v = fma(ja[rr], Ja[7 * rr + c], v);
            acc += v;
            const int pm = a.pos[a.edges[2 * k + 1 - side]];
            if (pm >= 0 && pm < P) {
                double o = 0.0;
#pragma unroll
                for (int rr = 0; rr < 7; ++rr) o = fma(ja[rr], Jb[7 * rr + c], o);
                const int64_t jb = pm / B;   // blk or blk - 1: no edge spans more than B positions
                const int64_t at = (int64_t)row * m + 7 * (int)(pm - jb * B) + c;
                double* d = jb == blk ? cr.D + blk * mm + at : cr.C + jb * mm + at;
                *d += o;   // this lane's own entry: another edge to the same node adds to it
            }
        }
    if (ent) {
        if (r == c) acc = t0 == t1 ? 1.0 : acc * (1.0 + a.lm[kLmLambda]);
        // whole rows of a diagonal block: its upper entries are not read
        cr.D[blk * mm + (int64_t)row * m + 7 * (int)(P - blk * B) + c] = acc;
    } else if (rhs) {
        cr.b[blk * m + row] = t0 == t1 ? 0.0 : -gr;
    }
}

// Candidate poses S_n <- exp(x_n) S_n of the free nodes; held nodes copied.
__global__ __launch_bounds__(64) void cr_candidate_kernel(PgoArgs a, CrArgs cr) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= a.n_nodes) return;
    const int P = a.pos[n];
    const Sim3d Sn = sim3_load(a.S + 13 * (int64_t)n);
    if (P < 0) {
        sim3_store(Sn, a.S_c + 13 * (int64_t)n);
        return;
    }
    const int blk = P / cr.block_pos;
    double d[7];
    for (int c = 0; c < 7; ++c) d[c] = cr.x[(int64_t)blk * cr.m + 7 * (P - blk * cr.block_pos) + c];
    sim3_store(sim3_mul(sim3_exp(d), Sn), a.S_c + 13 * (int64_t)n);
}

}  // namespace fl
