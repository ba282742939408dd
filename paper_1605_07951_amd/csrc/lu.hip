// Batched dense complex LU with partial pivoting and the matching solves.
//
// Factorisation (right-looking, blocked, RSRR Step 2 needs one LU per
// sampling point): for each outer panel of nb columns
//   1. the panel (all rows below the diagonal) is factored in blocks of up to
//      32 columns by a register-resident base kernel, right-looking inside;
//   2. the panel's row interchanges are composed into a permutation of at
//      most 2*nb rows (perm_build) and applied to the columns right of the
//      panel together with the unit-lower triangular solve U12 = L11^-1 A12;
//   3. the trailing matrix is updated on the matrix cores, A22 -= L21 U12,
//      for two panels at once where there are two (in FP32 of 384 rows and
//      more on the FP16 matrix cores with split operands).
// Columns left of the panel are never interchanged ("lazy" left swaps): the
// solve applies each panel's permutation just before that panel's forward
// elimination step, which reproduces the elimination order exactly.  Inside
// one panel the interchanges are applied to every panel column, so the
// solve can work at panel granularity.
//
// Pivot: largest |Re| + |Im| in the column, lowest row index on ties
// (LAPACK's choice).  info = first column (1-based) whose pivot is exactly
// zero; the factorisation continues past it, as getrf does.
#include <algorithm>
#include <climits>

#include "common.h"
#include "kernels.h"

namespace rsrr {

// ----------------------------------------------------------------------------
// Panel base: rows [c0, n) x columns [c0, c0+jb) of one matrix per workgroup,
// held in registers (thread t owns rows t, t+NT, ... of the panel).
//
// Bound by the chain of dependent steps of a column (search, broadcast, update),
// about 1000 cycles, not by bytes or flops, so the steps are kept few: rows never
// move while the panel is factored (a thread tracks the position that the
// interchanges give each of its rows and stores the row there at the end); the
// search runs in registers (DPP) inside a wave; each wave publishes its candidate
// with the candidate's row, so one barrier per column suffices and every thread
// picks the winner itself; pivots and flags are written after the loop.  Columns go
// in groups of GW: the chain of a column touches its
// own group only, the columns after the group take its pivot rows and one rank-GW
// update at the end of the group.  The loop over the groups is rolled (the registers
// rotate by one group), so the code stays in the instruction cache.
// A block of 32 columns of 48 matrices, complex FP32: 29 / 34 / 47 us at 256 / 512 /
// 1024 rows (a form that moved the rows, searched by shuffles with four barriers a
// column and took 8 columns a launch: 73 / 94 / 120 us in four launches, plus the
// products between them).
// perm (optional, 2*jb int2) receives the composed interchanges in the layout of
// perm_build_kernel.
// ----------------------------------------------------------------------------

// Lanes' values moved by a DPP control; lanes without a source get `none`.
template <int CTRL, int ROWS> RSRR_DEV int dpp(int x, int none)
{
    return __builtin_amdgcn_update_dpp(none, x, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS> RSRR_DEV double dpp(double x, double none)
{
    return __hiloint2double(dpp<CTRL, ROWS>(__double2hiint(x), __double2hiint(none)),
                            dpp<CTRL, ROWS>(__double2loint(x), __double2loint(none)));
}
RSRR_DEV int lane_get(int x, int l) { return __builtin_amdgcn_readlane(x, l); }
RSRR_DEV float lane_get(float x, int l) { return __int_as_float(lane_get(__float_as_int(x), l)); }
RSRR_DEV double lane_get(double x, int l)
{
    return __hiloint2double(lane_get(__double2hiint(x), l), lane_get(__double2loint(x), l));
}
template <typename C> RSRR_DEV C lane_get(C x, int l) { x.x = lane_get(x.x, l); x.y = lane_get(x.y, l); return x; }
RSRR_DEV float shfl_get(float x, int l) { return __shfl(x, l); }
RSRR_DEV double shfl_get(double x, int l) { return __shfl(x, l); }
template <typename C> RSRR_DEV C shfl_get(C x, int l) { x.x = __shfl(x.x, l); x.y = __shfl(x.y, l); return x; }

RSRR_DEV int max2(int a, int b) { return a > b ? a : b; }
RSRR_DEV double max2(double a, double b) { return fmax(a, b); }

// Maximum over lanes 0..W-1 (W = 2, 4, 8 or 16, the same values repeated in the other
// lanes or not) or over the whole wave (W = 64); uniform result.
template <int W, typename T> RSRR_DEV T wave_max(T x, T none)
{
    // row_shr 1, 2, 4, 8: lane W - 1 of a row of 16 has lanes 0 .. W-1
    x = max2(x, dpp<0x111, 0xf>(x, none));
    if (W > 2) x = max2(x, dpp<0x112, 0xf>(x, none));
    if (W > 4) x = max2(x, dpp<0x114, 0xf>(x, none));
    if (W > 8) x = max2(x, dpp<0x118, 0xf>(x, none));
    if (W <= 16) return lane_get(x, W - 1);
    x = max2(x, dpp<0x142, 0xa>(x, none));   // row_bcast 15 and 31: lane 63 has all
    x = max2(x, dpp<0x143, 0xc>(x, none));
    return lane_get(x, 63);
}

// Order of the pivot search: |Re| + |Im| as an integer (the bits of a non-negative
// float keep its order, a NaN comes above infinity) or as a double (a NaN counts as
// infinite), so a NaN wins and is reported.
RSRR_DEV int pivot_key(float a) { return __float_as_int(a) & 0x7fffffff; }
RSRR_DEV double pivot_key(double a) { return a == a ? a : (double)INFINITY; }
// (a, pa) before (b, pb): larger key, lower position on ties.
RSRR_DEV bool pivot_before(int a, int pa, int b, int pb)
{
    return ((long long)a << 32 | (unsigned)~pa) > ((long long)b << 32 | (unsigned)~pb);
}
RSRR_DEV bool pivot_before(double a, int pa, double b, int pb) { return a > b || (a == b && pa < pb); }

// The lane with the lowest pos among those of `lanes` (a ballot of hit, not empty; their
// pos are distinct).  More than one is a tie of the pivot search, as between the zero
// rows of a sparse column.
template <int W> RSRR_DEV int lowest_lane(unsigned long long lanes, bool hit, int pos)
{
    if (lanes & (lanes - 1)) {
        const int top = ~wave_max<W>(hit ? ~pos : INT_MIN, INT_MIN);
        lanes &= __ballot(pos == top);
    }
    return __ffsll((long long)lanes) - 1;
}

// a - b c as four fused multiply-adds (the chain of the panel base is bound by the
// number of instructions).
template <typename C> RSRR_DEV C cfms_fused(C a, C b, C c)
{
    a.x = fma(-b.x, c.x, a.x);
    a.y = fma(-b.x, c.y, a.y);
    a.x = fma(b.y, c.y, a.x);
    a.y = fma(-b.y, c.x, a.y);
    return a;
}
RSRR_DEV float cfms_fused(float a, float b, float c) { return fmaf(-b, c, a); }

template <typename C, int NT, int RPT, int JB>
__global__ __launch_bounds__(NT) void panel_lu_kernel(
    C* __restrict__ A, long sA, int lda, int n, int c0, int jb,
    int* __restrict__ ipiv, long sP, int* __restrict__ info, int2* __restrict__ perm, long sPerm,
    const int* __restrict__ active)
{
    typedef real_t<C> R;
    typedef decltype(pivot_key(R())) Key;
    constexpr Key none = sizeof(Key) == 4 ? (Key)INT_MIN : (Key)-1;   // below every key
    constexpr int NW = NT / 64;
    constexpr int GW = JB < 8 ? JB : 8, NG = JB / GW;
    static_assert(NW == 4 || NW == 8 || NW == 16, "the winner is picked inside one row of 16 lanes");
    static_assert(JB % GW == 0 && GW % 2 == 0 && JB <= 64, "whole groups; the buffer parity is fixed per unrolled column");
    const int b = blockIdx.x;
    if (active && !active[b]) return;
    C* Ab = A + (long)b * sA;
    int* pv = ipiv + (long)b * sP;
    const int m = n - c0;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;

    struct __attribute__((aligned(16))) Cand { Key key; int pos; C piv; };
    __shared__ Cand cand[2][NW];
    __shared__ __attribute__((aligned(16))) C rows[2][NW][GW];      // the candidates' rows, this group's columns
    __shared__ __attribute__((aligned(16))) C U[GW][JB];            // the group's pivot rows, the columns after it
    __shared__ C Lg[GW][GW];                                        // and their multipliers
    __shared__ int spiv[JB];   // pivot positions and values, looked at after the loop
    __shared__ C sval[JB];

    C v[RPT][JB];
    int pos[RPT];   // position of the row after the interchanges so far; -1: no row
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int lr = tid + NT * q;
        pos[q] = lr < m ? lr : -1;
#pragma unroll
        for (int c = 0; c < JB; ++c) {
            C e = czero<C>();
            if (lr < m && c < jb) e = Ab[(c0 + lr) + (long)(c0 + c) * lda];
            v[q][c] = e;
        }
    }

    const int ngrp = (jb + GW - 1) / GW;
#pragma unroll 1
    for (int g = 0; g < NG; ++g) {
#pragma unroll
        for (int c8 = 0; c8 < GW; ++c8) {
            const int c = g * GW + c8;
            if (c >= jb) break;
            const int buf = c8 & 1;
            // ---- candidate of the thread, then of the wave (lowest position on ties) ----
            Key bk = none;
            int bp = INT_MAX;
            C bv = czero<C>();
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                const Key a = pos[q] >= c ? pivot_key(cabs1(v[q][c8])) : none;
                if (q == 0 || pivot_before(a, pos[q], bk, bp)) { bk = a; bp = pos[q]; bv = v[q][c8]; }
            }
            const Key wk = wave_max<64>(bk, none);
            if (wk == none) {   // every row of the wave is done or absent
                if (lane == 0) cand[buf][wave] = {none, INT_MAX, czero<C>()};
            } else if (lane == lowest_lane<64>(__ballot(bk == wk), bk == wk, bp)) {
                cand[buf][wave] = {wk, bp, bv};
#pragma unroll
                for (int q = 0; q < RPT; ++q)
                    if (RPT == 1 || pos[q] == bp) {
#pragma unroll
                        for (int j = 0; j < GW; ++j)
                            if (j > c8) rows[buf][wave][j] = v[q][j];
                    }
            }
            __syncthreads();
            const Cand ca = cand[buf][lane & (NW - 1)];
            const Key gk = wave_max<NW>(ca.key, none);   // at least one row is left: gk != none
            const int win = lowest_lane<NW>(__ballot(ca.key == gk) & ((1ull << NW) - 1), ca.key == gk, ca.pos);
            C u[GW];
#pragma unroll
            for (int j = 0; j < GW; ++j)
                if (j > c8) u[j] = rows[buf][win][j];
            const int p = lane_get(ca.pos, win);
            const C piv = lane_get(ca.piv, win);
            const bool zero = is_zero(piv);
            if (tid == 0) { spiv[c] = p; sval[c] = piv; }
            const C rp = zero ? czero<C>() : crecip_scaled(piv);
            // ---- the interchange, the multipliers and the group's columns right of c ----
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                pos[q] = pos[q] == p ? c : (pos[q] == c ? p : pos[q]);
                if (pos[q] > c) {
                    if (!zero) v[q][c8] = cmul(v[q][c8], rp);
#pragma unroll
                    for (int j = 0; j < GW; ++j)
                        if (j > c8) v[q][j] = cfms_fused(v[q][j], v[q][c8], u[j]);
                }
            }
        }
        if (NG > 1 && g + 1 < ngrp) {
            // ---- the columns after the group: its pivot rows U = L11^-1 A, then the rank-GW update ----
            const int left = (ngrp - g - 1) * GW, first = g * GW;
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                const int i = pos[q] - first;
                if (i >= 0 && i < GW) {
#pragma unroll
                    for (int j = 0; j < GW; ++j) Lg[i][j] = v[q][j];
#pragma unroll
                    for (int j = 0; j < JB - GW; ++j)
                        if (j < left) U[i][j] = v[q][GW + j];
                }
            }
            __syncthreads();
            if (tid < left) {
                C x[GW];
#pragma unroll
                for (int i = 0; i < GW; ++i) x[i] = U[i][tid];
#pragma unroll
                for (int j = 0; j < GW; ++j)
#pragma unroll
                    for (int i = j + 1; i < GW; ++i) x[i] = cfms_fused(x[i], Lg[i][j], x[j]);
#pragma unroll
                for (int i = 0; i < GW; ++i) U[i][tid] = x[i];
            }
            __syncthreads();
            // Few rows per thread: a done row's multipliers are set to zero, so that no branch lies
            // between the reads of U and their uses.  More rows: no registers for the copies.
            constexpr bool COPY = RPT * sizeof(C) < 32;
            C l[COPY ? RPT : 1][GW];
            if constexpr (COPY) {
#pragma unroll
                for (int q = 0; q < RPT; ++q)
#pragma unroll
                    for (int i = 0; i < GW; ++i) l[q][i] = pos[q] >= first + GW ? v[q][i] : czero<C>();
            }
#pragma unroll
            for (int k = 1; k < NG; ++k)
                if (k < ngrp - g) {
#pragma unroll
                    for (int i = 0; i < GW; ++i) {
                        C u[GW];
#pragma unroll
                        for (int j = 0; j < GW; ++j) u[j] = U[i][(k - 1) * GW + j];
#pragma unroll
                        for (int q = 0; q < RPT; ++q) {
                            if constexpr (COPY) {
#pragma unroll
                                for (int j = 0; j < GW; ++j)
                                    v[q][k * GW + j] = cfms_fused(v[q][k * GW + j], l[q][i], u[j]);
                            } else if (pos[q] >= first + GW) {
#pragma unroll
                                for (int j = 0; j < GW; ++j)
                                    v[q][k * GW + j] = cfms_fused(v[q][k * GW + j], v[q][i], u[j]);
                            }
                        }
                    }
                }
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                const int i = pos[q] - first;
                if (i >= 0 && i < GW) {
#pragma unroll
                    for (int j = 0; j < JB - GW; ++j)
                        if (j < left) v[q][GW + j] = U[i][j];
                }
            }
        }
        if (NG > 1) {   // the finished group goes last; after NG turns every column is back in place
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                C t[GW];
#pragma unroll
                for (int j = 0; j < GW; ++j) t[j] = v[q][j];
#pragma unroll
                for (int j = 0; j < JB - GW; ++j) v[q][j] = v[q][j + GW];
#pragma unroll
                for (int j = 0; j < GW; ++j) v[q][JB - GW + j] = t[j];
            }
        }
    }
    __syncthreads();
    if (tid < jb) pv[c0 + tid] = c0 + spiv[tid];
    if (wave == 0) {   // the first zero or non-finite pivot
        const C pz = lane < jb ? sval[lane] : from_real<C>((R)1);
        const unsigned long long bad = __ballot(!all_finite(pz)), odd = bad | __ballot(is_zero(pz));
        const int c = __ffsll((long long)odd) - 1;
        if (odd && lane == 0 && info[b] == 0) info[b] = (bad >> c & 1) ? -(c0 + c + 1) : c0 + c + 1;
    }

    int2* pm = perm ? perm + (long)b * sPerm : nullptr;
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int lr = tid + NT * q;
        if (lr < m) {
#pragma unroll
            for (int c = 0; c < JB; ++c)
                if (c < jb) Ab[(c0 + pos[q]) + (long)(c0 + c) * lda] = v[q][c];
            // only the first jb rows can leave their place other than as a pivot: row lr owns slot jb + lr
            if (pm) {
                if (pos[q] < jb) pm[pos[q]] = make_int2(c0 + pos[q], c0 + lr);
                if (lr < jb) pm[jb + lr] = pos[q] >= jb ? make_int2(c0 + pos[q], c0 + lr) : make_int2(-1, -1);
            }
        }
    }
}

// ----------------------------------------------------------------------------
// Compose the interchanges ipiv[k1 .. k1+jb) (applied in order) into a
// permutation of the affected rows: after the swaps, row dst[s] holds the
// old row src[s].  Slots 0..jb-1 are rows k1..k1+jb-1; later slots are the
// distinct rows below that were swapped in; unused slots hold (-1, -1).
// One wavefront per matrix; lane 0 replays the swaps, the wave searches.
// ----------------------------------------------------------------------------
__global__ __launch_bounds__(64) void perm_build_kernel(const int* __restrict__ ipiv, long sP, int k1, int jb,
                                                          int2* __restrict__ perm, long sPerm,
                                                          const int* __restrict__ active)
{
    const int b = blockIdx.x;
    if (active && !active[b]) return;
    const int* pv = ipiv + (long)b * sP;
    int2* pm = perm + (long)b * sPerm;
    const int lane = threadIdx.x;
    __shared__ int rowid[2 * MAX_NB], content[2 * MAX_NB];
    for (int s = lane; s < 2 * jb; s += 64) {
        rowid[s] = (s < jb) ? k1 + s : -1;
        content[s] = (s < jb) ? k1 + s : -1;
    }
    __syncthreads();
    int nout = 0;
    for (int i = 0; i < jb; ++i) {
        const int p = pv[k1 + i];
        int slot;
        if (p < k1 + jb) {
            slot = p - k1;
        } else {
            int found = INT_MAX;
            for (int base = 0; base < nout; base += 64) {
                const int s = base + lane;
                const bool hit = (s < nout) && rowid[jb + s] == p;
                const unsigned long long m = __ballot(hit);
                if (m) { found = base + __ffsll((long long)m) - 1; break; }
            }
            if (found == INT_MAX) {
                slot = jb + nout;
                if (lane == 0) { rowid[slot] = p; content[slot] = p; }
                ++nout;
            } else {
                slot = jb + found;
            }
        }
        __syncthreads();
        if (lane == 0 && slot != i) {
            const int t = content[i];
            content[i] = content[slot];
            content[slot] = t;
        }
        __syncthreads();
    }
    for (int s = lane; s < 2 * jb; s += 64) pm[s] = make_int2(rowid[s], content[s]);
}

// Wave-level ordering of LDS accesses (one wavefront, no workgroup barrier).
RSRR_DEV void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The composition of perm_build_kernel done by the first wavefront of a
// workgroup into pm (2 jb slots, LDS): after the interchanges pv[k1 .. k1+jb),
// row pm[s].x holds the old row pm[s].y.  The caller synchronises the workgroup
// afterwards.
RSRR_DEV void compose_perm_wave(const int* __restrict__ pv, int k1, int jb, int2* pm)
{
    const int lane = threadIdx.x & 63;
    for (int s = lane; s < 2 * jb; s += 64) pm[s] = s < jb ? make_int2(k1 + s, k1 + s) : make_int2(-1, -1);
    wave_sync();
    int nout = 0;
    for (int i = 0; i < jb; ++i) {
        const int p = pv[k1 + i];
        int slot;
        if (p < k1 + jb) {
            slot = p - k1;
        } else {
            int found = INT_MAX;
            for (int base = 0; base < nout; base += 64) {
                const int s = base + lane;
                const bool hit = (s < nout) && pm[jb + s].x == p;
                const unsigned long long m = __ballot(hit);
                if (m) { found = base + __ffsll((long long)m) - 1; break; }
            }
            if (found == INT_MAX) {
                slot = jb + nout;
                if (lane == 0) pm[slot] = make_int2(p, p);
                ++nout;
            } else {
                slot = jb + found;
            }
        }
        wave_sync();
        if (lane == 0 && slot != i) {
            const int t = pm[i].y;
            pm[i].y = pm[slot].y;
            pm[slot].y = t;
        }
        wave_sync();
    }
}

// ----------------------------------------------------------------------------
// A factored block [c0, c0+jb) (jb <= JB) of a panel [p0, p0+pw): its row
// interchanges on the panel's other columns and, right of the block,
// U = L11^-1 A (L11: the unit-lower triangle at (c0, c0)).  One launch for both
// sides.  A column is a group of 2 JB lanes, one lane per affected row (top row
// s, or the s-th displaced row), so a column's gather and scatter are one load
// and one store and nothing is shared between waves; each top lane holds its row
// of L11 in registers and the solve broadcasts x_l across the group.  PS_U
// columns per group are in flight to cover the latency.
// The composed interchanges come from the base kernel (perm) or, for a block of
// several bases, are composed here from ipiv.
// ----------------------------------------------------------------------------
constexpr int PS_NT = 256, PS_U = 4, PS_MAX = 32;

template <typename C, int JB>
__global__ __launch_bounds__(PS_NT) void panel_swap_kernel(
    C* __restrict__ A, long sA, int lda, const int2* __restrict__ perm, long sPerm, const int* __restrict__ ipiv,
    long sP, int p0, int pw, int c0, int jb, const int* __restrict__ active)
{
    constexpr int G = 2 * JB, CW = 64 / G;   // lanes per column, columns side by side in a wave
    const int b = blockIdx.y;
    if (active && !active[b]) return;
    C* Ab = A + (long)b * sA;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int s = lane % G, gb = lane - s;
    __shared__ int2 pm[2 * JB];
    const int2* pb = pm;
    if (ipiv) {
        if (wave == 0) compose_perm_wave(ipiv + (long)b * sP, c0, jb, pm);
        __syncthreads();
    } else {
        pb = perm + (long)b * sPerm;
    }
    int2 e = make_int2(-1, -1);
    if (s < jb) e = pb[s];
    else if (s >= JB && s - JB < jb) e = pb[jb + s - JB];
    const int nl = c0 - p0, ncols = pw - jb;
    const int k0 = (blockIdx.x * (PS_NT / 64) + wave) * CW * PS_U + lane / G;
    C x[PS_U], y[PS_U];
    int col[PS_U];
#pragma unroll
    for (int u = 0; u < PS_U; ++u) {
        const int k = k0 + u * CW;
        col[u] = k >= ncols ? -1 : (k < nl ? p0 + k : c0 + jb + (k - nl));
        x[u] = (col[u] >= 0 && e.y >= 0) ? Ab[e.y + (long)col[u] * lda] : czero<C>();
        y[u] = x[u];
    }
    bool right = false;
#pragma unroll
    for (int u = 0; u < PS_U; ++u) right |= col[u] > c0;
    if (__any(right)) {
        C Lr[JB];
#pragma unroll
        for (int l = 0; l < JB; ++l)
            Lr[l] = (l < s && s < jb) ? Ab[(c0 + s) + (long)(c0 + l) * lda] : czero<C>();
#pragma unroll
        for (int l = 0; l < JB - 1; ++l) {   // rows past jb are zero in Lr
#pragma unroll
            for (int u = 0; u < PS_U; ++u) {
                C xl;
                if constexpr (G == 64) xl = lane_get(y[u], l);
                else xl = shfl_get(y[u], gb + l);
                y[u] = cfms_fused(y[u], Lr[l], xl);
            }
        }
    }
    if (e.x >= 0) {
#pragma unroll
        for (int u = 0; u < PS_U; ++u)
            if (col[u] >= 0) {
                C o = x[u];
                if (s < JB && col[u] > c0) o = y[u];
                Ab[e.x + (long)col[u] * lda] = o;
            }
    }
}

// ----------------------------------------------------------------------------
// Row permutation + triangular solve on a block of columns (the FP64 path
// without diagonal-block inverses).
// X: rows indexed like the factored matrix; columns [0, ncols).
// mode 1: permute, then X[c0:c0+jb] = L11^-1 X[...] with L11 the unit-lower
// diagonal block of LU at (c0, c0).
// mode 2: no permutation, X[c0:c0+jb] = U11^-1 X[...] (non-unit upper).
// ----------------------------------------------------------------------------
constexpr int TS_NT = 256;

// MJB: widest diagonal block staged in LDS; TC: columns per workgroup.
template <typename C, int MJB, int TC>
__global__ __launch_bounds__(TS_NT) void perm_trsm_kernel(
    const C* __restrict__ LU, long sLU, int ldl,
    const int2* __restrict__ perm, long sPerm,
    C* __restrict__ X, long sX, int ldx,
    int c0, int jb, int ncols, int mode, const int* __restrict__ active)
{
    const int b = blockIdx.y;
    if (active && !active[b]) return;
    const C* Lb = LU + (long)b * sLU;
    C* Xb = X + (long)b * sX;
    const int tid = threadIdx.x;
    const int col = tid % TC, grp = tid / TC;
    constexpr int NG = TS_NT / TC;
    const int gcol = blockIdx.x * TC + col;
    const bool colok = gcol < ncols;

    __shared__ C top[MJB][TC + 1];
    __shared__ C Ld[MJB][MJB + 1];
    __shared__ int2 pm[2 * MJB];

    if (mode == 1) {
        const int2* pb = perm + (long)b * sPerm;
        for (int s = tid; s < 2 * jb; s += TS_NT) pm[s] = pb[s];
    }
    // triangle into LDS (column-major read, coalesced along rows)
    for (int e = tid; e < jb * jb; e += TS_NT) {
        const int r = e % jb, c = e / jb;
        Ld[r][c] = Lb[(c0 + r) + (long)(c0 + c) * ldl];
    }
    __syncthreads();

    if (mode == 1) {
        // gather every affected row (reads first, writes after the barrier)
        constexpr int MAXQ = (2 * MJB + NG - 1) / NG;
        C val[MAXQ];
#pragma unroll
        for (int q = 0; q < MAXQ; ++q) {
            const int s = grp + NG * q;
            C e = czero<C>();
            if (s < 2 * jb && colok) {
                const int src = pm[s].y;
                if (src >= 0) e = Xb[src + (long)gcol * ldx];
            }
            val[q] = e;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < MAXQ; ++q) {
            const int s = grp + NG * q;
            if (s < jb) {
                top[s][col] = val[q];
            } else if (s < 2 * jb && colok) {
                const int dst = pm[s].x;
                if (dst >= 0) Xb[dst + (long)gcol * ldx] = val[q];
            }
        }
    } else {
        for (int s = grp; s < jb; s += NG)
            top[s][col] = colok ? Xb[(c0 + s) + (long)gcol * ldx] : czero<C>();
    }
    __syncthreads();

    if (mode == 1) {
        for (int l = 0; l < jb; ++l) {
            const C xl = top[l][col];
            for (int i = l + 1 + grp; i < jb; i += NG) top[i][col] = cfms(top[i][col], Ld[i][l], xl);
            __syncthreads();
        }
    } else {
        for (int l = jb - 1; l >= 0; --l) {
            if (grp == 0) {
                const C d = Ld[l][l];
                top[l][col] = is_zero(d) ? top[l][col] : cmul(top[l][col], crecip(d));
            }
            __syncthreads();
            const C xl = top[l][col];
            for (int i = grp; i < l; i += NG) top[i][col] = cfms(top[i][col], Ld[i][l], xl);
            __syncthreads();
        }
    }

    if (colok)
        for (int s = grp; s < jb; s += NG) Xb[(c0 + s) + (long)gcol * ldx] = top[s][col];
}

// ----------------------------------------------------------------------------
// Row permutation of a block of columns without a solve (LDS only for the
// permutation).  A workgroup takes PR_TC columns: 2*jb threads gather the
// affected rows of all of them (the loads in flight together), then scatter
// them; rows c0..c0+jb-1 go to T (jb x ncols, ldt) when T is given, otherwise
// back into X.  perm == nullptr: identity (copy the block
// rows to T).
// ----------------------------------------------------------------------------
constexpr int PR_TC = 32;

template <typename C>
__global__ __launch_bounds__(2 * MAX_NB) void perm_rows_kernel(
    const int2* __restrict__ perm, long sPerm, C* __restrict__ X, long sX, int ldx,
    C* __restrict__ T, long sT, int ldt, int c0, int jb, int ncols, const int* __restrict__ active)
{
    typedef real_t<C> R;
    const int b = blockIdx.y;
    if (active && !active[b]) return;
    C* Xb = X + (long)b * sX;
    C* Tb = T ? T + (long)b * sT : nullptr;
    const int s = threadIdx.x;
    int2 e = make_int2(-1, -1);
    if (s < 2 * jb) {
        if (perm) e = perm[(long)b * sPerm + s];
        else if (s < jb) e = make_int2(c0 + s, c0 + s);
    }
    // every column's source row first (all loads in flight), one barrier, then the stores
    const int cbase = blockIdx.x * PR_TC;
    C v[PR_TC];
#pragma unroll
    for (int cc = 0; cc < PR_TC; ++cc) {
        const int gcol = cbase + cc;
        v[cc] = czero<C>();
        if (gcol < ncols && e.y >= 0) v[cc] = Xb[e.y + (long)gcol * ldx];
    }
    __syncthreads();
#pragma unroll
    for (int cc = 0; cc < PR_TC; ++cc) {
        const int gcol = cbase + cc;
        if (gcol < ncols) {
            if (s < jb) {
                if (Tb) Tb[s + (long)gcol * ldt] = v[cc];
                else Xb[(c0 + s) + (long)gcol * ldx] = v[cc];
            } else if (e.x >= 0) {
                Xb[e.x + (long)gcol * ldx] = v[cc];
            }
        }
    }
}

// ----------------------------------------------------------------------------
// host drivers
// ----------------------------------------------------------------------------

// Base width of the register-resident panel kernel for m rows: as many columns
// as the registers hold (32 at most: the blocks of the panel are that wide).
template <typename C> static int base_width(int m)
{
    constexpr int words = sizeof(C) / 4;   // registers per element
    if (m <= 512) return 32;
    if (words == 4) return m <= 1024 ? 16 : (m <= 2048 ? 8 : (m <= 4096 ? 4 : 2));
    if (words == 2) return m <= 1024 ? 32 : (m <= 2048 ? 16 : (m <= 4096 ? 8 : 4));
    return m <= 2048 ? 32 : (m <= 4096 ? 16 : 8);
}

template <typename C>
static void panel_lu(hipStream_t st, C* A, long sA, int lda, int n, int c0, int jb,
                     int* ipiv, long sP, int* info, int2* perm, long sPerm, const int* active, int batch)
{
    constexpr int words = sizeof(C) / 4;
    const int m = n - c0;
#define PL(NT, RPT, JB)                                                                                       \
    hipLaunchKernelGGL((panel_lu_kernel<C, NT, RPT, JB>), dim3(batch), dim3(NT), 0, st, A, sA, lda, n, c0, jb, \
                       ipiv, sP, info, perm, sPerm, active)
    // RPT rows per thread against NT threads: measured per column for each range of m (us, 48
    // matrices); more threads repeat the search in more waves, more rows lengthen the update
    if constexpr (words == 4) {
        if (m <= 256) PL(256, 1, 32);         // 1.2
        else if (m <= 512) PL(512, 1, 32);    // 1.5
        else if (m <= 1024) PL(512, 2, 16);   // 1.8
        else if (m <= 2048) PL(1024, 2, 8);   // 2.6
        else if (m <= 4096) PL(1024, 4, 4);   // 3.9
        else PL(1024, 8, 2);                  // 6.2
    } else if constexpr (words == 2) {
        if (m <= 256) PL(256, 1, 32);         // 0.9
        else if (m <= 512) PL(512, 1, 32);    // 1.1 (two rows of 256 threads 1.2)
        else if (m <= 1024) PL(512, 2, 32);   // 1.5
        else if (m <= 2048) PL(512, 4, 16);   // 2.0
        else if (m <= 4096) PL(1024, 4, 8);   // 2.9 (eight rows of 512 threads 3.6)
        else PL(1024, 8, 4);                  // 4.4
    } else {
        if (m <= 256) PL(256, 1, 32);         // 0.7
        else if (m <= 512) PL(256, 2, 32);    // 0.9
        else if (m <= 1024) PL(512, 2, 32);   // 1.0 (four rows of 256 threads 1.25)
        else if (m <= 2048) PL(512, 4, 32);   // 1.5
        else if (m <= 4096) PL(512, 8, 16);   // 2.3
        else PL(1024, 8, 8);                  // 2.9
    }
#undef PL
}

// Interchanges of the factored block [c0, c0+jb) on the other columns of the panel
// [p0, p0+pw) and U = L11^-1 A right of it.  perm: composed by the base kernel, or
// nullptr: composed in the kernel from ipiv.
template <typename C>
static void panel_swap(hipStream_t st, C* A, long sA, int lda, const int2* perm, long sPerm, const int* ipiv,
                       long sP, int p0, int pw, int c0, int jb, const int* active, int batch)
{
    const int ncols = pw - jb;
    if (ncols <= 0) return;
    if (perm) ipiv = nullptr;
#define PSW(JB)                                                                                                \
    do {                                                                                                       \
        constexpr int per = (PS_NT / 64) * (64 / (2 * JB)) * PS_U;                                             \
        hipLaunchKernelGGL((panel_swap_kernel<C, JB>), dim3((ncols + per - 1) / per, batch), dim3(PS_NT), 0,   \
                           st, A, sA, lda, perm, sPerm, ipiv, sP, p0, pw, c0, jb, active);                     \
    } while (0)
    if (jb <= 8) PSW(8);
    else if (jb <= 16) PSW(16);
    else PSW(32);
#undef PSW
}

// FP64 path without diagonal-block inverses (panels of at most 64 columns).
static void perm_trsm(hipStream_t st, const double2* LU, long sLU, int ldl, const int2* perm, long sPerm,
                      double2* X, long sX, int ldx, int c0, int jb, int ncols, int mode,
                      const int* active, int batch)
{
    if (ncols <= 0 || jb <= 0) return;
    constexpr int TC = 32;
    dim3 g((ncols + TC - 1) / TC, batch);
    hipLaunchKernelGGL((perm_trsm_kernel<double2, 64, TC>), g, dim3(TS_NT), 0, st, LU, sLU, ldl, perm, sPerm,
                       X, sX, ldx, c0, jb, ncols, mode, active);
}

template <typename C>
static void perm_rows(hipStream_t st, const int2* perm, long sPerm, C* X, long sX, int ldx,
                      C* T, long sT, int ldt, int c0, int jb, int ncols, const int* active, int batch)
{
    if (ncols <= 0 || jb <= 0) return;
    dim3 g((ncols + PR_TC - 1) / PR_TC, batch);
    hipLaunchKernelGGL(perm_rows_kernel<C>, g, dim3(2 * MAX_NB), 0, st, perm, sPerm, X, sX, ldx, T, sT, ldt, c0, jb,
                       ncols, active);
}

// C = beta C - alpha A B (defaults alpha = beta = 1: C -= A B).  The products
// C = A B with the diagonal-block inverses use alpha = -1, beta = 0.
template <typename C>
static hipError_t gemm_sub(hipStream_t st, int M, int N, int K, const C* A, int lda, long sA,
                           const C* B, int ldb, long sB, C* Cm, int ldc, long sC,
                           int batch, int tag = 0, double alpha = 1.0, double beta = 1.0);
template <>
hipError_t gemm_sub<float2>(hipStream_t st, int M, int N, int K, const float2* A, int lda, long sA, const float2* B,
                           int ldb, long sB, float2* Cm, int ldc, long sC, int batch, int tag, double alpha,
                           double beta)
{
    return cgemm(st, M, N, K, (float)-alpha, A, lda, sA, B, ldb, sB, (float)beta, Cm, ldc, sC, batch, tag);
}
template <>
hipError_t gemm_sub<double2>(hipStream_t st, int M, int N, int K, const double2* A, int lda, long sA,
                            const double2* B, int ldb, long sB, double2* Cm, int ldc, long sC, int batch, int tag,
                            double alpha, double beta)
{
    return zgemm(st, 0, 0, M, N, K, -alpha, A, lda, sA, B, ldb, sB, beta, Cm, ldc, sC, batch, tag);
}

template <>
hipError_t gemm_sub<float>(hipStream_t st, int M, int N, int K, const float* A, int lda, long sA, const float* B,
                           int ldb, long sB, float* Cm, int ldc, long sC, int batch, int tag, double alpha,
                           double beta)
{
    return sgemm(st, M, N, K, (float)-alpha, A, lda, sA, B, ldb, sB, (float)beta, Cm, ldc, sC, batch, tag);
}

// C -= A21 U12 right of a factored block, inside the panel: rows below the block.
template <typename C>
static void panel_update(hipStream_t st, C* A, long sA, int lda, int n, int c0, int jb, int cend, int batch)
{
    const int c1 = c0 + jb;
    if (c1 >= cend || c1 >= n) return;
    (void)gemm_sub<C>(st, n - c1, cend - c1, jb, A + c1 + (long)c0 * lda, lda, sA, A + c0 + (long)c1 * lda, lda, sA,
                      A + c1 + (long)c1 * lda, lda, sA, batch);
}

// Panel factorisation of columns [c0, c0+w) (rows c0..n-1): blocks of PS_MAX
// columns, each a single base or, where the base is narrower, several bases, both
// levels right-looking (block, interchanges and U rows in one launch, update).
// pm: 2*MAX_NB int2 per matrix (stride sPm) as scratch for a base's interchanges.
template <typename C>
static void factor_panel(hipStream_t st, C* A, long sA, int lda, int n, int c0, int w,
                         int* ipiv, long sP, int* info, int2* pm, long sPm, const int* active,
                         int batch)
{
    for (int b0 = c0; b0 < c0 + w; b0 += PS_MAX) {
        const int bw = std::min(PS_MAX, c0 + w - b0);
        const int base = base_width<C>(n - b0);
        for (int s0 = b0; s0 < b0 + bw; s0 += base) {
            const int sw = std::min(base, b0 + bw - s0);
            panel_lu<C>(st, A, sA, lda, n, s0, sw, ipiv, sP, info, pm, sPm, active, batch);
            if (bw > base) {
                panel_swap<C>(st, A, sA, lda, pm, sPm, ipiv, sP, b0, bw, s0, sw, active, batch);
                panel_update<C>(st, A, sA, lda, n, s0, sw, b0 + bw, batch);
            }
        }
        panel_swap<C>(st, A, sA, lda, bw <= base ? pm : nullptr, sPm, ipiv, sP, c0, w, b0, bw, active, batch);
        panel_update<C>(st, A, sA, lda, n, b0, bw, c0 + w, batch);
    }
}

// Diagonal-block inverses of panel p (complex-FP32 path): L11^-1 at
// inv + (2p) nb^2, U11^-1 at inv + (2p+1) nb^2, ld nb.
template <typename C>
static C* panel_inv(const LUWork& w, int p, int nb, int which)
{
    return (C*)w.inv + (long)(2 * p + which) * nb * nb;
}

// 16 x 16 tiles of products of blocks in LDS (column-major, ld TI_LD) on the 16x16x4 matrix
// instructions; the first operand carries the right factor, so that a lane's output runs down a column.
template <typename C> constexpr int TI_N = max_panel<real_t<C>>();
template <typename C> constexpr int TI_LD = TI_N<C> + 4;
constexpr int TI_B = 16, TI_NT = 512;

RSRR_DEV floatx4 mfma16(float x, float y, floatx4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c, 0, 0, 0); }
RSRR_DEV doublex4 mfma16(double x, double y, doublex4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, c, 0, 0, 0);
}
template <typename R> struct vec4_of { typedef floatx4 T; };
template <> struct vec4_of<double> { typedef doublex4 T; };
// column of a lane's output r: four consecutive ones in FP32, every fourth in FP64
template <typename R>
RSRR_DEV int mfma16_col(int g, int r) { return sizeof(R) == 4 ? 4 * g + r : g + 4 * r; }

template <typename C>
struct Tile16 {
    typedef real_t<C> R;
    typename vec4_of<R>::T re = {0, 0, 0, 0}, im = {0, 0, 0, 0}, rn = {0, 0, 0, 0}, in = {0, 0, 0, 0};
    // += A B, A 16 x K and B K x 16 in LDS (first elements, ld TI_LD and LB)
    template <int LB>
    RSRR_DEV void add(const C* A, const C* B, int K, int lane)
    {
        const int li = lane & 15, g = lane >> 4;
        const C* pa = A + g * TI_LD<C> + li;
        const C* pb = B + li * LB + g;
        for (int k = 0; k < K; k += 16) {
            C x[4], y[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                x[u] = pa[(k + 4 * u) * TI_LD<C>];
                y[u] = pb[k + 4 * u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if constexpr (elem_traits<C>::complex) {
                    re = mfma16(y[u].x, x[u].x, re);
                    im = mfma16(y[u].y, x[u].x, im);
                    rn = mfma16(y[u].y, x[u].y, rn);
                    in = mfma16(y[u].x, x[u].y, in);
                } else {
                    re = mfma16(y[u], x[u], re);
                }
            }
        }
    }
    // to LDS at D (ld LB), times sign
    template <int LB>
    RSRR_DEV void put(C* D, R sign, int lane) const
    {
        const int li = lane & 15, g = lane >> 4;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            C* p = D + mfma16_col<R>(g, r) * LB + li;
            if constexpr (elem_traits<C>::complex) {
                p->x = sign * (re[r] - rn[r]);
                p->y = sign * (im[r] + in[r]);
            } else {
                *p = sign * re[r];
            }
        }
    }
};

// Inverses of the two triangles of the jb x jb diagonal block at (c0, c0), or (upper false) of L alone: L11^-1 (unit lower, which =
// 0) at inv + (2p) nb^2 and U11^-1 (upper, which = 1) at inv + (2p+1) nb^2, ld nb, the other triangle
// zero.  One workgroup per triangle and matrix, the triangle in LDS and inverted in place by 16 x 16
// blocks: the diagonal ones by a lane per column (substitution in registers), then the block rows in
// turn, a wave per block of the row, X_ij = -L_ii^-1 sum_{j<=k<i} L_ik X_kj on the matrix cores (U: upwards,
// X_ij = -U_ii^-1 sum_{i<k<=j} U_ik X_kj).
// A zero diagonal entry of U counts as one (as in the solves).  Rows and columns past jb are
// padded with the identity.
// Bound by latency (the load, 16 dependent rows, seven block rows with two barriers each):
// complex FP32 128 rows, 1 / 64 / 256 matrices 27 / 30 / 66 us (32 x 32 blocks on the vector unit, a
// workgroup per block column: 49 / 60 / 141), real FP32 14 / 16 / 21 (24 / 27 / 57), FP64 64 rows 12 / 13 /
// 28 (28 / 31 / 98).  By halves (four products instead of fourteen in turn) 25 us, but up to twice
// the error of L11^-1.  The parts of a complex product have accumulators of their own: one
// chain for two of them measured 1.3 times the error.
template <typename C>
__global__ __launch_bounds__(TI_NT) void tri_inv_kernel(const C* __restrict__ LU, long sLU, int ldl, int c0, int jb,
                                                        C* __restrict__ inv, long sInv, int nb,
                                                        const int* __restrict__ active)
{
    constexpr int N = TI_N<C>, LD = TI_LD<C>;
    const int b = blockIdx.x, which = blockIdx.y;
    if (active && !active[b]) return;
    const C* A = LU + (long)b * sLU + c0 + (long)c0 * ldl;   // the diagonal block, A(r, c) = A[r + c*ldl]
    C* X = (C*)inv + (long)b * sInv + (long)(2 * (c0 / nb) + which) * nb * nb;
    constexpr int PL = TI_B + 4;
    __shared__ C S[N * LD], P[TI_NT / 64][TI_B * PL];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int np = (jb + TI_B - 1) / TI_B * TI_B;   // rows in use
    constexpr int W = 8;                            // columns in flight per thread
    const int r = tid % N;
    for (int cc = tid / N; cc < np; cc += W * (TI_NT / N)) {
        C v[W];
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const int c = cc + q * (TI_NT / N);
            const bool in = r < jb && c < jb && (which == 0 ? r > c : r <= c);
            v[q] = in ? A[r + (long)c * ldl] : from_real<C>((real_t<C>)(r == c ? 1 : 0));
        }
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const int c = cc + q * (TI_NT / N);
            if (c < np) S[c * LD + r] = v[q];
        }
    }
    __syncthreads();
    if (wave < N / TI_B && wave * TI_B < np) {
        const int o = wave * TI_B, col = lane & 15;
        const C* D = S + o * LD + o;
        C x[TI_B];
        if (which == 0) {
#pragma unroll
            for (int i = 0; i < TI_B; ++i) {
                C s = from_real<C>((real_t<C>)(i == col ? 1 : 0));
#pragma unroll
                for (int l = 0; l < i; ++l) s = cfms(s, D[l * LD + i], x[l]);
                x[i] = s;
            }
        } else {
            // the lanes' own diagonal entry inverted at once, handed out by row
            const C d = D[col * LD + col];
            const C dr = is_zero(d) ? from_real<C>((real_t<C>)1) : crecip(d);
#pragma unroll
            for (int i = TI_B - 1; i >= 0; --i) {
                C s = from_real<C>((real_t<C>)(i == col ? 1 : 0));
#pragma unroll
                for (int l = i + 1; l < TI_B; ++l) s = cfms(s, D[l * LD + i], x[l]);
                x[i] = cmul(s, shfl_get(dr, i));
            }
        }
        // (a wave's reads of its block precede its writes)
        if (lane < TI_B) {
#pragma unroll
            for (int i = 0; i < TI_B; ++i) S[(o + col) * LD + o + i] = x[i];
        }
    }
    __syncthreads();
    const int nbk = np / TI_B;
    for (int m = 1; m < nbk; ++m) {
        const int i = which == 0 ? m : nbk - 1 - m, j = which == 0 ? wave : i + 1 + wave;
        const bool on = wave < m;
        Tile16<C> t, x;
        if (on) {
            if (which == 0) t.template add<LD>(S + j * TI_B * LD + i * TI_B, S + j * TI_B * LD + j * TI_B, (i - j) * TI_B, lane);
            else t.template add<LD>(S + (i + 1) * TI_B * LD + i * TI_B, S + j * TI_B * LD + (i + 1) * TI_B, (j - i) * TI_B, lane);
            t.template put<PL>(P[wave], (real_t<C>)1, lane);
        }
        __syncthreads();
        if (on) x.template add<PL>(S + i * TI_B * LD + i * TI_B, P[wave], TI_B, lane);
        // (every read of the block row precedes the barrier above)
        if (on) x.template put<LD>(S + j * TI_B * LD + i * TI_B, (real_t<C>)-1, lane);
        __syncthreads();
    }
    for (int c = tid / N; c < jb; c += TI_NT / N)
        if (r < jb) X[r + (long)c * nb] = S[c * LD + r];
}

template <typename C>
static void tri_inv(hipStream_t st, const C* LU, long sLU, int ldl, int c0, int jb, C* inv, long sInv, int nb,
                    const int* active, int batch, bool upper)
{
    hipLaunchKernelGGL(tri_inv_kernel<C>, dim3(batch, upper ? 2 : 1), dim3(TI_NT), 0, st, LU, sLU, ldl, c0, jb, inv, sInv, nb,
                       active);
}

// D(r0.., 0..cols) = S(r0.., 0..cols): rows r0..n-1 of a column block, per matrix.
template <typename C>
__global__ __launch_bounds__(256) void copy_rows_kernel(int r0, int n, int cols, const C* __restrict__ S, int lds,
                                                         long sS, C* __restrict__ D, int ldd, long sD,
                                                         const int* __restrict__ active)
{
    const int b = blockIdx.y;
    if (active && !active[b]) return;
    const long m = n - r0;
    const long e = (long)blockIdx.x * 256 + threadIdx.x;
    if (e >= m * cols) return;
    const int r = r0 + (int)(e % m), c = (int)(e / m);
    D[b * sD + r + (long)c * ldd] = S[b * sS + r + (long)c * lds];
}

template <typename C>
static void copy_rows(hipStream_t st, int r0, int n, int cols, const C* S, int lds, long sS, C* D, int ldd, long sD,
                      const int* active, int batch)
{
    const long cnt = (long)(n - r0) * cols;
    if (cnt <= 0) return;
    hipLaunchKernelGGL(copy_rows_kernel<C>, dim3((unsigned)((cnt + 255) / 256), batch), dim3(256), 0, st, r0, n, cols,
                       S, lds, sS, D, ldd, sD, active);
}

// ----------------------------------------------------------------------------
// Rows of one size for the split products (FP32): the factorisation of T with w.rs is that of
// diag(2^-rs) T, and the right-hand sides are scaled by 2^-rs where they are narrowed.  A T whose
// largest entries per row lie within RW_SPREAD powers of two keeps rs = 0 and every bit.
//
// With rows of different size the small entries of a row of L meet the large ones of a column of U and fall out
// of the range of FP16 (split.hip): T with half of its rows 10^8 / 10^10 times the others took 3 / 6 to 10
// corrections instead of 2, at 10^12 the redo in FP64, and the preconditioner of the iterative sampling was
// lost. Powers of two per inner index taken from the columns of L21 mend those, but lose columns that are only
// weakly coupled to the rows below; the rows of T itself have no such case. In an emulation of 72 scaled,
// penalised, sparse and block matrices the scaled form took no more corrections than an unscaled FP32
// factorisation wherever that one succeeded, and left smaller errors in the small components.
//
// Whether T needs it is decided cheaply where that is safe: the largest of 16 entries and the
// diagonal entry of a row bounds the row's size from below, ||T||_F every row's from above; within 2^14 nothing
// of weight is lost (2^-40 2^14 = 2^-26).  Only other matrices are read in full.  64 matrices with n = 4096:
// 46 us (64 entries: 95) of a call of 88.9 ms with 16 right-hand sides; with half of the rows 10^10 times the
// others 1.5 ms for the sizes and 3.8 for the scaling, 94.5 ms in all.
// ----------------------------------------------------------------------------
constexpr int RW_SPREAD = 10, RW_SURE = 14, RW_NONE = -(1 << 20);
constexpr int RW_NT = 1024;

RSRR_DEV float part_max(float2 v) { return fmaxf(fabsf(v.x), fabsf(v.y)); }
RSRR_DEV float part_max(float v) { return fabsf(v); }

// need[b] = whether some row of matrix b may be beyond 2^RW_SURE of the largest; else rs = 0
template <typename C>
__global__ __launch_bounds__(RW_NT) void row_sure_kernel(const C* __restrict__ A, long sA, int lda, int n,
                                                         const int* __restrict__ rows, const double* __restrict__ frob,
                                                         int* __restrict__ rs, long sR, int* __restrict__ need)
{
    const int b = blockIdx.x, lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int m = rows ? rows[b] : n;
    __shared__ float lo[RW_NT / 64];
    float least = INFINITY;
    if (frob)
        for (int i0 = g * 64; i0 < m; i0 += RW_NT) {
            const int i = min(i0 + lane, m - 1);
            const C* Ab = A + b * sA + i;
            float t = part_max(Ab[(long)i * lda]);
#pragma unroll
            for (int q = 0; q < 16; ++q) t = fmaxf(t, part_max(Ab[(long)((long)q * m / 16) * lda]));
            least = fminf(least, t);
        }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) least = fminf(least, __shfl_xor(least, off));
    if (lane == 0) lo[g] = least;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < RW_NT / 64; ++q) least = fminf(least, lo[q]);
    // false for a norm that is not finite
    const bool sure = frob && (double)least * (double)(1 << RW_SURE) >= frob[b];
    if (threadIdx.x == 0) need[b * sR] = !sure;
    if (sure)
        for (int i = threadIdx.x; i < n; i += RW_NT) rs[b * sR + i] = 0;
}

// ex[i] = the exponent of row i's largest part (none, or not finite: RW_NONE)
template <typename C>
__global__ __launch_bounds__(RW_NT) void row_expo_kernel(const C* __restrict__ A, long sA, int lda, int n,
                                                         const int* __restrict__ rows, int* __restrict__ ex, long sR,
                                                         const int* __restrict__ need)
{
    constexpr int G = RW_NT / 64;
    const int b = blockIdx.y, lane = threadIdx.x & 63, g = threadIdx.x >> 6, i = blockIdx.x * 64 + lane;
    if (!need[b * sR]) return;
    const int m = rows ? rows[b] : n;
    __shared__ float top[G][64];
    const C* Ab = A + b * sA + min(i, n - 1);
    float t = 0.f;
#pragma unroll 8
    for (int j = g; j < m; j += G) t = fmaxf(t, part_max(Ab[(long)j * lda]));
    top[g][lane] = t;
    __syncthreads();
    if (g > 0 || i >= n) return;
#pragma unroll
    for (int q = 1; q < G; ++q) t = fmaxf(t, top[q][lane]);
    ex[b * sR + i] = i < m && t > 0.f && isfinite(t) ? __builtin_amdgcn_frexp_expf(t) : RW_NONE;
}

// rs = ex relative to the largest row (0 for all within RW_SPREAD), and T scaled by it.  At most 2^96, so that
// scaled right-hand sides of norm one stay in the range of FP32.
template <typename C>
__global__ __launch_bounds__(256) void row_apply_kernel(C* __restrict__ A, long sA, int lda, int n,
                                                        const int* __restrict__ ex, int* __restrict__ rs, long sR,
                                                        const int* __restrict__ need)
{
    const int b = blockIdx.y, t = threadIdx.x;
    if (!need[b * sR]) return;
    const int* e = ex + b * sR;
    __shared__ int hi[256], lo[256];
    int h = RW_NONE, l = -RW_NONE;
    for (int i = t; i < n; i += 256)
        if (e[i] != RW_NONE) {
            h = max(h, e[i]);
            l = min(l, e[i]);
        }
    hi[t] = h;
    lo[t] = l;
    __syncthreads();
    for (int o = 128; o >= 1; o >>= 1) {
        if (t < o) {
            hi[t] = max(hi[t], hi[t + o]);
            lo[t] = min(lo[t], lo[t + o]);
        }
        __syncthreads();
    }
    h = hi[0];
    const bool scale = h != RW_NONE && h - lo[0] > RW_SPREAD;
    if (blockIdx.x == 0)
        for (int i = t; i < n; i += 256) rs[b * sR + i] = scale && e[i] != RW_NONE ? max(e[i] - h, -96) : 0;
    if (!scale) return;
    for (int j = blockIdx.x; j < n; j += gridDim.x) {
        C* col = A + b * sA + (long)j * lda;
        for (int i = t; i < n; i += 256) {
            const int s = e[i] != RW_NONE ? min(h - e[i], 96) : 0;
            if (s == 0) continue;
            if constexpr (elem_traits<C>::complex) col[i] = make_float2(ldexpf(col[i].x, s), ldexpf(col[i].y, s));
            else col[i] = ldexpf(col[i], s);
        }
    }
}

__global__ __launch_bounds__(256) void row_zero_kernel(int n, int* __restrict__ rs, long sR)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) rs[blockIdx.y * sR + i] = 0;
}

// w.rs and the scratch before it (row_scale_of); without split operands nothing is scaled
template <typename C>
static void scale_rows(hipStream_t st, C* A, long sA, int lda, int n, const LUWork& w, int batch)
{
    int *need = w.rs - 1, *ex = need - n;
    if (!w.pack) {
        hipLaunchKernelGGL(row_zero_kernel, dim3((n + 255) / 256, batch), dim3(256), 0, st, n, w.rs, w.sRs);
        return;
    }
    hipLaunchKernelGGL(row_sure_kernel<C>, dim3(batch), dim3(RW_NT), 0, st, A, sA, lda, n, w.rows, w.frob, w.rs, w.sRs,
                       need);
    hipLaunchKernelGGL(row_expo_kernel<C>, dim3((n + 63) / 64, batch), dim3(RW_NT), 0, st, A, sA, lda, n, w.rows, ex,
                       w.sRs, need);
    // eight workgroups of a matrix or more, to fill the chip with few matrices too
    hipLaunchKernelGGL(row_apply_kernel<C>, dim3(std::max(8, std::min(64, 2048 / batch)), batch), dim3(256), 0, st, A,
                       sA, lda, n, ex, w.rs, w.sRs, need);
}

template <typename C>
static hipError_t getrf_impl(hipStream_t st, C* A, long sA, int lda, int n, int nb, const LUWork& w,
                         int batch)
{
    typedef real_t<C> R;
    if constexpr (sizeof(R) == 4) {
        if (w.rs) scale_rows<C>(st, A, sA, lda, n, w, batch);
    }
    // diagonal-block inverses and products on the matrix cores: always in FP32, in
    // FP64 when the caller gives the inverse and scratch buffers
    const bool use_inv = sizeof(R) == 4 || (w.inv != nullptr && w.tmp != nullptr);
    if (nb > max_panel<R>()) nb = max_panel<R>();
    if (nb < MIN_NB) nb = MIN_NB;  // perm/inv storage holds perm_panels(n) panels
    UpdateRecorder* rec = w.rec;
    hipError_t err = hipSuccess;   // the first one
    auto ok = [&](hipError_t e) { if (err == hipSuccess) err = e; };
    // trailing update C(M x N) -= Aop(M x kdepth) Bop(kdepth x N) on `s`, event-timed.  An
    // update done in column parts gives its whole width (Nall) and the part's first column
    // (j0); with split operands the first part (j0 = 0) packs them for all parts (B unless the U
    // rows came packed).
    auto timed_update = [&](hipStream_t s, int M, int N, int kdepth, const C* Aop, int ldaop, long sAop,
                               const C* Bop, C* Cop, int Nall = 0, int j0 = 0, bool bpacked = false) {
        const bool timed = rec && rec->used < rec->cap;
        if (timed) (void)hipEventRecord(rec->ev[2 * rec->used], s);
        if (Nall == 0) Nall = N;
        bool split = false;
        if constexpr (sizeof(R) == 4) {
            // (a part that starts inside a packed block of 32 columns runs in FP32)
            split = w.pack != nullptr && split_ok(M, Nall, kdepth) && j0 % 32 == 0;
            if (split) {
                char* PA = (char*)w.pack + split_column_bytes(n);
                char* PB = PA + split_operand_bytes<C>(M, kdepth);
                if (j0 == 0) {
                    ok(split_pack_a<C>(s, M, kdepth, Aop, ldaop, sAop, nullptr, 0, PA, w.sPack, batch));
                    if (!bpacked) ok(split_pack_b<C>(s, Nall, kdepth, Bop, lda, sA, nullptr, 0, PB, w.sPack, batch));
                }
                ok(gemm_split(s, M, N, kdepth, PA, w.sPack, PB, w.sPack, Nall, j0, true, Cop, lda, sA, batch));
            }
        }
        if (!split) ok(gemm_sub<C>(s, M, N, kdepth, Aop, ldaop, sAop, Bop, lda, sA, Cop, lda, sA, batch, 1));
        if (timed) {
            (void)hipEventRecord(rec->ev[2 * rec->used + 1], s);
            const double fl = (elem_traits<C>::complex ? 8.0 : 2.0) * M * (double)N * kdepth * batch;
            if (rec->lflops) rec->lflops[rec->used] = fl;
            if (rec->lmask) rec->lmask[rec->used] = (s == w.upd && s != nullptr) ? 1 : 0;
            rec->used++;
            rec->flops += fl;
            rec->bytes += (double)sizeof(C) * (2.0 * M * N + (double)M * kdepth + (double)kdepth * N) * batch;
        } else if (rec) {
            rec->dropped++;
        }
    };
    // panel p on stream s: factor, composed interchanges, diagonal-block inverses (FP32 paths)
    auto panel = [&](hipStream_t s, int c0, int jb, int p) -> int2* {
        int2* pm = w.perm + (long)p * 2 * MAX_NB;
        factor_panel<C>(s, A, sA, lda, n, c0, jb, w.ipiv, w.sP, w.info, pm, w.sPerm, w.active, batch);
        hipLaunchKernelGGL(perm_build_kernel, dim3(batch), dim3(64), 0, s, w.ipiv, w.sP, c0, jb, pm, w.sPerm,
                           w.active);
        if (use_inv)
            tri_inv<C>(s, A, sA, lda, c0, jb, (C*)w.inv, w.sInv, nb, w.active, batch, sizeof(R) == 4 || w.solve_inv);
        return pm;
    };
    // Two panels may share one trailing update of depth jb0 + jb1 (the deeper
    // product keeps the matrix cores busier per byte of A22 read and written):
    // panel p+1's columns get panel p's update first; the rows of L21_p are
    // copied and interchanged like panel p+1's rows (the stored L21_p keeps
    // panel p's row order, which the solves expect); the U rows of panel p+1
    // receive panel p's update from that copy; then A22 -= [L21_p' L21_{p+1}]
    // [U12_p; U12_{p+1}] in one product.
    const bool pairing = use_inv && w.pair != nullptr;
    // The U rows of the pair (q0, q1 = q0 + nb) of full panels p, p + 1 on the columns from q2 on,
    // with the rows' interchanges, by the split kernels: true when done (and the update's B packed).
    auto split_pair_rows = [&](hipStream_t s, int q0, int p0, C* TL) -> bool {
        if constexpr (sizeof(C) == sizeof(float2) && elem_traits<C>::complex) {
            const int q2 = q0 + 2 * nb, rest = n - q2;
            C* Ar = A + (long)q2 * lda;
            if (!w.pack || !split_ok(rest, rest, 2 * nb) || !split_urows_ok(nb, Ar + q0, lda, sA)) return false;
            const int2* pm0 = w.perm + (long)p0 * 2 * MAX_NB;
            perm_rows<C>(s, pm0, w.sPerm, Ar, sA, lda, (C*)nullptr, 0, 0, q0, nb, rest, w.active, batch);
            perm_rows<C>(s, pm0 + 2 * MAX_NB, w.sPerm, Ar, sA, lda, (C*)nullptr, 0, 0, q0 + nb, nb, rest, w.active,
                         batch);
            ok(split_urows(s, rest, rest, panel_inv<C>(w, p0, nb, 0), nb, w.sInv, TL, nb, w.sPair,
                           panel_inv<C>(w, p0 + 1, nb, 0), nb, w.sInv, Ar + q0, lda, sA,
                           (char*)w.pack + split_column_bytes(n), w.sPack, batch));
            return true;
        }
        return false;
    };
    // A pair's work before its trailing update: a front part that touches only its own 2 nb columns
    // (panel p, its interchanges and U rows on panel p+1's columns, panel p+1's columns update,
    // panel p+1, the interchanged copy of L21_p) and a back part on the trailing columns (the
    // interchanges and U rows of both panels there, the copy of L21_{p+1}).
    const int ldw = w.ldpair;
    auto front = [&](hipStream_t s, int q0, int pp, C* Wp) {
        const int q1 = q0 + nb;
        C* TL = Wp + (long)ldw * 2 * nb;
        const int2* pm0 = panel(s, q0, nb, pp);
        perm_rows<C>(s, pm0, w.sPerm, A + (long)q1 * lda, sA, lda, (C*)w.tmp, w.sTmp, nb, q0, nb, nb, w.active,
                     batch);
        ok(gemm_sub<C>(s, nb, nb, nb, panel_inv<C>(w, pp, nb, 0), nb, w.sInv, (const C*)w.tmp, nb, w.sTmp,
                       A + q0 + (long)q1 * lda, lda, sA, batch, 0, -1.0, 0.0));
        ok(gemm_sub<C>(s, n - q1, nb, nb, A + q1 + (long)q0 * lda, lda, sA, A + q0 + (long)q1 * lda, lda, sA,
                       A + q1 + (long)q1 * lda, lda, sA, batch));
        const int2* pm1 = panel(s, q1, nb, pp + 1);
        copy_rows<C>(s, q1, n, nb, A + (long)q0 * lda, lda, sA, Wp, ldw, w.sPair, w.active, batch);
        perm_rows<C>(s, pm1, w.sPerm, Wp, w.sPair, ldw, TL, w.sPair, nb, q1, nb, nb, w.active, batch);
    };
    auto back = [&](int q0, int pp, C* Wp) -> bool {
        const int q1 = q0 + nb, q2 = q1 + nb, rest = n - q2;
        C* TL = Wp + (long)ldw * 2 * nb;
        copy_rows<C>(st, q2, n, nb, A + (long)q1 * lda, lda, sA, Wp + (long)ldw * nb, ldw, w.sPair, w.active, batch);
        if (split_pair_rows(st, q0, pp, TL)) return true;
        const int2* pm0 = w.perm + (long)pp * 2 * MAX_NB;
        const int2* pm1 = w.perm + (long)(pp + 1) * 2 * MAX_NB;
        C* Ar2 = A + (long)q2 * lda;
        perm_rows<C>(st, pm0, w.sPerm, Ar2, sA, lda, (C*)w.tmp, w.sTmp, nb, q0, nb, rest, w.active, batch);
        ok(gemm_sub<C>(st, nb, rest, nb, panel_inv<C>(w, pp, nb, 0), nb, w.sInv, (const C*)w.tmp, nb, w.sTmp,
                       Ar2 + q0, lda, sA, batch, 0, -1.0, 0.0));
        perm_rows<C>(st, pm1, w.sPerm, Ar2, sA, lda, (C*)w.tmp, w.sTmp, nb, q1, nb, rest, w.active, batch);
        ok(gemm_sub<C>(st, nb, rest, nb, TL, nb, w.sPair, Ar2 + q0, lda, sA, (C*)w.tmp, nb, w.sTmp, batch));
        ok(gemm_sub<C>(st, nb, rest, nb, panel_inv<C>(w, pp + 1, nb, 0), nb, w.sInv, (const C*)w.tmp, nb,
                       w.sTmp, Ar2 + q1, lda, sA, batch, 0, -1.0, 0.0));
        return false;
    };
    int c0 = 0, p = 0;
    // Look-ahead over full pairs (two nb-wide panels with a trailing block after
    // them).  After the back part of pair i, the trailing update is split: first
    // the 2 nb columns of pair i+1, then, while the rest of the update runs on
    // `st`, pair i+1's front part runs on the side stream (its own pair buffer);
    // the next back part waits for both.
    if (pairing && w.side && w.pair2 && w.ev_a && w.ev_b && n > 2 * nb) {
        C* Wb[2] = {(C*)w.pair, (C*)w.pair2};
        int buf = 0;
        front(st, 0, 0, Wb[0]);
        if (w.first_panel) ok(hipEventRecord(w.first_panel, st));
        for (;;) {
            const int c2 = c0 + 2 * nb, rest = n - c2;
            const bool bpacked = back(c0, p, Wb[buf]);
            C* Aop = Wb[buf] + c2;
            const C* Bop = A + c0 + (long)c2 * lda;
            C* Cop = A + c2 + (long)c2 * lda;
            if (rest <= 2 * nb) {
                // no full pair follows: one update, the loop below finishes the tail
                timed_update(st, rest, rest, 2 * nb, Aop, ldw, w.sPair, Bop, Cop, rest, 0, bpacked);
                c0 = c2;
                p += 2;
                break;
            }
            const int wn = 2 * nb;
            timed_update(st, rest, wn, 2 * nb, Aop, ldw, w.sPair, Bop, Cop, rest, 0, bpacked);
            ok(hipEventRecord(w.ev_a, st));
            // the rest of the update is enqueued before the next pair's panels (a chain of
            // small launches), so the host never holds it back behind them
            if (w.upd && w.ev_c) {
                // the first la_cols columns of the update on the CUs the side stream does not
                // use (while the next panels are factored), the rest on every CU
                const int n1 = w.la_cols > 0 ? std::min(rest - wn, std::max(32, w.la_cols / 32 * 32)) : rest - wn;
                ok(hipStreamWaitEvent(w.upd, w.ev_a, 0));
                timed_update(w.upd, rest, n1, 2 * nb, Aop, ldw, w.sPair, Bop + (long)wn * lda,
                                Cop + (long)wn * lda, rest, wn);
                ok(hipEventRecord(w.ev_c, w.upd));
                ok(hipStreamWaitEvent(st, w.ev_c, 0));
                if (n1 < rest - wn)
                    timed_update(st, rest, rest - wn - n1, 2 * nb, Aop, ldw, w.sPair, Bop + (long)(wn + n1) * lda,
                                    Cop + (long)(wn + n1) * lda, rest, wn + n1);
            } else {
                timed_update(st, rest, rest - wn, 2 * nb, Aop, ldw, w.sPair, Bop + (long)wn * lda,
                                Cop + (long)wn * lda, rest, wn);
            }
            ok(hipStreamWaitEvent(w.side, w.ev_a, 0));
            front(w.side, c2, p + 2, Wb[buf ^ 1]);
            ok(hipEventRecord(w.ev_b, w.side));
            ok(hipStreamWaitEvent(st, w.ev_b, 0));
            c0 = c2;
            p += 2;
            buf ^= 1;
        }
    }
    // without look-ahead: the pairs in turn; then the last panels one by one
    for (; pairing && n - c0 > 2 * nb; c0 += 2 * nb, p += 2) {
        const int c2 = c0 + 2 * nb, rest = n - c2;
        C* Wp = (C*)w.pair;
        front(st, c0, p, Wp);
        if (c0 == 0 && w.first_panel) ok(hipEventRecord(w.first_panel, st));
        const bool bpacked = back(c0, p, Wp);
        timed_update(st, rest, rest, 2 * nb, Wp + c2, ldw, w.sPair, A + c0 + (long)c2 * lda, A + c2 + (long)c2 * lda,
                        rest, 0, bpacked);
    }
    for (; c0 < n; c0 += nb, ++p) {
        const int jb = std::min(nb, n - c0), c1 = c0 + jb, rest = n - c1;
        const int2* pm = panel(st, c0, jb, p);
        if (rest <= 0) break;
        C* Ar = A + (long)c1 * lda;
        if (use_inv) {
            // interchanges on the right block (top rows to the scratch), then U12 = L11^-1 A12 on MFMA
            perm_rows<C>(st, pm, w.sPerm, Ar, sA, lda, (C*)w.tmp, w.sTmp, nb, c0, jb, rest, w.active, batch);
            ok(gemm_sub<C>(st, jb, rest, jb, panel_inv<C>(w, p, nb, 0), nb, w.sInv, (const C*)w.tmp, nb, w.sTmp,
                           Ar + c0, lda, sA, batch, 0, -1.0, 0.0));
        } else {
            if constexpr (sizeof(C) == sizeof(double2))
                perm_trsm(st, A, sA, lda, pm, w.sPerm, Ar, sA, lda, c0, jb, rest, 1, w.active, batch);
        }
        if (c0 == 0 && w.first_panel) ok(hipEventRecord(w.first_panel, st));
        timed_update(st, rest, rest, jb, A + c1 + (long)c0 * lda, lda, sA, A + c0 + (long)c1 * lda,
                        A + c1 + (long)c1 * lda);
    }
    ok(hipGetLastError());
    return err;
}

// Right-hand sides, and those of all matrices, from which the solves' products pack their operands (the
// factor is read once more and written once for that, two launches more a product).  FP32 / split, ms: 128
// right-hand sides 1.03 / 1.04 (n = 1024, 32 matrices) and 2.07 / 2.07 (2048, 16), 256 1.32 / 1.24 and
// 2.66 / 2.37, 512 1.97 / 1.74 and 3.76 / 3.02; one matrix, n = 500 0.39 / 0.41 and n = 2730
// 2.48 / 2.49 at 512, 3.52 / 2.91 at 2730.
constexpr int SPLIT_RHS = 256, SPLIT_RHS_ALL = 2048;

template <typename C>
static hipError_t getrs_impl(hipStream_t st, const C* LU, long sLU, int lda, int n, int nb,
                         const LUWork& w, C* X, long sX, int ldx, int nrhs, int batch)
{
    typedef real_t<C> R;
    const bool use_inv = sizeof(R) == 4 || (w.inv != nullptr && w.tmp != nullptr && w.solve_inv);
    if (nb > max_panel<R>()) nb = max_panel<R>();
    if (nb < MIN_NB) nb = MIN_NB;
    const int np = (n + nb - 1) / nb;
    hipError_t err = hipSuccess;   // the first one
    auto ok = [&](hipError_t e) { if (err == hipSuccess) err = e; };
    // rows at r0 (m of them) -= F (m x K, ld lda) times the K rows of X at c0; the backward sweep's split
    // products take a power of two per column of U, formed before the first
    bool columns = false;
    auto off_diag = [&](int r0, int m, int K, const C* F, int c0) {
        if constexpr (sizeof(C) == sizeof(float2) && elem_traits<C>::complex) {
            const long na = split_operand_bytes<C>(m, K);
            if (w.pack && !w.any_mix && split_ok(m, nrhs, K) && nrhs >= SPLIT_RHS && (long)nrhs * batch >= SPLIT_RHS_ALL &&
                (long)split_column_bytes(n) + na + split_operand_bytes<C>(nrhs, K) <= w.sPack) {
                const long sE = w.sPack / 4;
                const bool back = r0 < c0;
                if (back && !columns) ok(split_columns(st, n, LU, lda, sLU, (int*)w.pack, sE, batch));
                columns |= back;
                const int* E = back ? (const int*)w.pack + c0 : nullptr;
                char* PA = (char*)w.pack + split_column_bytes(n);
                char* PB = PA + na;
                ok(split_pack_a(st, m, K, F, lda, sLU, E, sE, PA, w.sPack, batch));
                ok(split_pack_b(st, nrhs, K, X + c0, ldx, sX, E, sE, PB, w.sPack, batch));
                ok(gemm_split(st, m, nrhs, K, PA, w.sPack, PB, w.sPack, nrhs, 0, true, X + r0, ldx, sX, batch));
                return;
            }
        }
        ok(gemm_sub<C>(st, m, nrhs, K, F, lda, sLU, X + c0, ldx, sX, X + r0, ldx, sX, batch));
    };
    for (int p = 0; p < np; ++p) {
        const int c0 = p * nb, jb = (n - c0 < nb) ? n - c0 : nb;
        const int2* pm = w.perm + (long)p * 2 * MAX_NB;
        if (use_inv) {
            perm_rows<C>(st, pm, w.sPerm, X, sX, ldx, (C*)w.tmp, w.sTmp, nb, c0, jb, nrhs, w.active, batch);
            ok(gemm_sub<C>(st, jb, nrhs, jb, panel_inv<C>(w, p, nb, 0), nb, w.sInv, (const C*)w.tmp, nb, w.sTmp,
                           X + c0, ldx, sX, batch, 0, -1.0, 0.0));
        } else {
            if constexpr (sizeof(C) == sizeof(double2))
                perm_trsm(st, LU, sLU, lda, pm, w.sPerm, X, sX, ldx, c0, jb, nrhs, 1, w.active, batch);
        }
        const int rest = n - c0 - jb;
        if (rest > 0) off_diag(c0 + jb, rest, jb, LU + (c0 + jb) + (long)c0 * lda, c0);
    }
    // Backward sweep with U11.  Panels are taken in pairs (p, p-1): after both
    // diagonal solves (the second preceded by the small coupling product with
    // U[p-1, p]) the rows above are updated once with depth jb(p-1) + jb(p);
    // the columns of U above a pair are contiguous, so no copy is needed.
    auto diag_solve = [&](int p) {
        const int c0 = p * nb, jb = (n - c0 < nb) ? n - c0 : nb;
        if (use_inv) {
            perm_rows<C>(st, nullptr, 0, X, sX, ldx, (C*)w.tmp, w.sTmp, nb, c0, jb, nrhs, w.active, batch);
            ok(gemm_sub<C>(st, jb, nrhs, jb, panel_inv<C>(w, p, nb, 1), nb, w.sInv, (const C*)w.tmp, nb, w.sTmp,
                           X + c0, ldx, sX, batch, 0, -1.0, 0.0));
        } else {
            if constexpr (sizeof(C) == sizeof(double2))
                perm_trsm(st, LU, sLU, lda, nullptr, 0, X, sX, ldx, c0, jb, nrhs, 2, w.active, batch);
        }
    };
    for (int p = np - 1; p >= 0;) {
        const int c0 = p * nb, jb = (n - c0 < nb) ? n - c0 : nb;
        diag_solve(p);
        if (p >= 1) {
            const int c1 = c0 - nb;  // panel p-1 is a full panel of width nb
            off_diag(c1, nb, jb, LU + c1 + (long)c0 * lda, c0);
            diag_solve(p - 1);
            if (c1 > 0) off_diag(0, c1, nb + jb, LU + (long)c1 * lda, c1);
            p -= 2;
        } else {
            p -= 1;
        }
    }
    ok(hipGetLastError());
    return err;
}

// ----------------------------------------------------------------------------
// The whole solve of getrs_impl (FP32, diagonal blocks by their inverses) for one matrix (and at most 16 right-hand sides) per workgroup, for right-hand-side
// blocks that fit in LDS: X is read once, every panel's forward step (interchanges,
// X_p = L11^-1 X_p, rows below -= L21 X_p) and backward step (X_p = U11^-1 X_p,
// rows above -= U12 X_p) runs out of LDS while the factor columns stream from
// memory once, and X is written back at the end.  The same operations as
// the launch-per-step chain, so the same result up to the order of the sums;
// a matrix with active[b] == 0 is left as it is.
//
// The products run on v_mfma_f32_16x16x4f32: the 16 columns of one operand are the real
// and the imaginary parts of 8 right-hand sides, so one instruction for the real and one
// for the imaginary parts of the factor give 16 rows of the complex product (real FP32: 16
// right-hand sides, one instruction).  A
// lane's factor entry (row lane % 16, column lane / 16 of four) goes from memory
// into its registers, and the panel's X_p stays in registers for all rows of the update.
// A row of X in LDS: per 8 right-hand sides 8 real, then 8 imaginary parts.
//
// Bound by the serial chain of panels and by what one compute unit streams and multiplies
// (8 n^2 bytes, 8 right-hand sides: n^2 / 64 pairs of 32-cycle instructions on four SIMDs,
// 109 us at n = 1000).  One launch for the 3 a panel step of the chain, so it is the faster
// way wherever X fits.  Chain / this kernel / the same split on the vector unit, in us: n =
// 256, 8 right-hand sides, 72 matrices 95 / 31 / 91, n = 1000 541 / 319 / 795 (1 matrix 460 / 252 /
// 724, 256 matrices 795 / 409 / 875); 16 right-hand sides, 72 matrices, n = 512 241 / 136 / 534, n =
// 1024 571 / 464 / 1580; n = 2048, 8 right-hand sides, 1 / 32 matrices 950 / 1081 (chain), 874 / 1031.
// Real, 16 right-hand sides, 64 matrices, chain / this kernel: n = 256 75 / 21, n = 1024 421 / 194, n =
// 2025 1117 / 779 (4 right-hand sides, 16 matrices 834 / 707; 64 and 64 1755 / 687).
// ----------------------------------------------------------------------------
constexpr int GS_MAX_RHS = 64, GS_MAX_WG = 512;
constexpr int GS_NT = 512, GS_NW = GS_NT / 64;
constexpr int GS_G = 8;                      // groups of four columns per batch of loads
constexpr int GS_Q = MAX_NB / (4 * GS_G);    // batches per panel

// C = float2: CB blocks of 8 right-hand sides; float: CB blocks of 16
template <typename C, int CB>
__global__ __launch_bounds__(GS_NT) void getrs_lds_kernel(const C* __restrict__ LU, long sLU, int lda, int n, int nb,
                                                          const int2* __restrict__ perm, long sPerm,
                                                          const C* __restrict__ inv, long sInv,
                                                          C* __restrict__ X, long sX, int ldx, int L,
                                                          const int* __restrict__ active)
{
    constexpr bool CX = elem_traits<C>::complex;
    constexpr int LD = 16 * CB;              // floats per row of X
    constexpr int NR = (CX ? 8 : 16) * CB;   // right-hand sides
    constexpr int NX = CB == 1 ? 2 : 1;      // blocks of rows per wave (two need more registers than there are)
    extern __shared__ __attribute__((aligned(16))) float xs[];
    const int b = blockIdx.x, tid = threadIdx.x;
    if (active && !active[b]) return;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, g = lane >> 4;
    const C* A = LU + (long)b * sLU;
    C* Xb = X + (long)b * sX + (long)(blockIdx.y * NR) * ldx;   // this workgroup's right-hand sides
    L = min(L - (int)blockIdx.y * NR, NR);
    // X in and out: 16 rows x 4 right-hand sides per wave
    auto each = [&](auto f) {
        const int nrb = (n + 15) / 16;
        for (int e = wave; e < nrb * (NR / 4); e += GS_NW) {
            const int r = e / (NR / 4) * 16 + li, l = e % (NR / 4) * 4 + g;
            if (r < n) f(r, l, xs + r * LD + (CX ? (l >> 3) * 16 + (l & 7) : l));
        }
    };
    each([&](int r, int l, float* x) {
        const C v = l < L ? Xb[r + (long)l * ldx] : czero<C>();
        if constexpr (CX) {
            x[0] = v.x;
            x[8] = v.y;
        } else {
            x[0] = v;
        }
    });
    const int np = (n + nb - 1) / nb;

    // X_p as the other operand for the real parts of the factor (b1); for the imaginary parts the
    // two halves of 8 columns change places and the first changes sign
    float b1[GS_Q][GS_G][CB];
    const unsigned flip = li < 8 ? 0x80000000u : 0u;
    auto turned = [&](float v) {   // row_ror:8, lane i of 16 takes lane i ^ 8
        const unsigned o = (unsigned)__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, true);
        return __uint_as_float(o ^ flip);
    };
    auto read_x = [&](int c0, int jb) {
        if (jb == 4 * GS_G * GS_Q) {
            const float* x = xs + (c0 + g) * LD + li;
#pragma unroll
            for (int q = 0; q < GS_Q; ++q)
#pragma unroll
                for (int i = 0; i < GS_G; ++i)
#pragma unroll
                    for (int c = 0; c < CB; ++c) b1[q][i][c] = x[(q * GS_G + i) * 4 * LD + c * 16];
        } else {
#pragma unroll
            for (int q = 0; q < GS_Q; ++q)
#pragma unroll
                for (int i = 0; i < GS_G; ++i) {
                    const int k = (q * GS_G + i) * 4 + g;
                    const float* x = xs + (c0 + min(k, jb - 1)) * LD + li;
#pragma unroll
                    for (int c = 0; c < CB; ++c) b1[q][i][c] = k < jb ? x[c * 16] : 0.f;
                }
        }
    };
    // entries (row, 4 (q GS_G + i) + g) of a block of jb columns (past the last: the last again, X is zero there)
    auto load = [&](const C* F, int ldf, int row, int q, int jb, C (&a)[GS_G]) {
        if ((q + 1) * 4 * GS_G <= jb) {
            const unsigned off = (unsigned)(g * ldf + row) * (unsigned)sizeof(C);   // uniform base, 32-bit offset
#pragma unroll
            for (int i = 0; i < GS_G; ++i)
                a[i] = *reinterpret_cast<const C*>(
                    reinterpret_cast<const char*>(F + (long)((q * GS_G + i) * 4) * ldf) + off);
        } else {
#pragma unroll
            for (int i = 0; i < GS_G; ++i)
                a[i] = F[(unsigned)row + (unsigned)(min((q * GS_G + i) * 4 + g, jb - 1) * ldf)];
        }
    };
    auto mult = [&](const C (&a)[GS_G], int q, floatx4 (&acc)[CB]) {
#pragma unroll
        for (int i = 0; i < GS_G; ++i) {
            if constexpr (CX) {
#pragma unroll
                for (int c = 0; c < CB; ++c)
                    acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(b1[q][i][c], a[i].x, acc[c], 0, 0, 0);
#pragma unroll
                for (int c = 0; c < CB; ++c)
                    acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(turned(b1[q][i][c]), a[i].y, acc[c], 0, 0, 0);
            } else {
#pragma unroll
                for (int c = 0; c < CB; ++c)
                    acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(b1[q][i][c], a[i], acc[c], 0, 0, 0);
            }
        }
    };
    // the jb x jb triangle D (ld nb), one block of 16 rows per wave; a batch of columns on the far
    // side of the diagonal is zero
    C d[GS_Q][GS_G];
    auto diag_on = [&](int q, int jb, bool lower) {
        return wave * 16 < jb && q * 4 * GS_G < jb &&
               (lower ? q * 4 * GS_G < wave * 16 + 16 : (q + 1) * 4 * GS_G > wave * 16);
    };
    auto diag_load = [&](const C* D, int jb, bool lower) {
#pragma unroll
        for (int q = 0; q < GS_Q; ++q)
            if (diag_on(q, jb, lower)) load(D, nb, min(wave * 16 + li, jb - 1), q, jb, d[q]);
    };
    // X_p = D X_p (D loaded), then rows [r0, r1) -= F X_p, F the columns c0 .. c0+jb of the factor: a wave
    // takes NX blocks of 16 rows at a time and loads one batch of columns ahead
    auto panel = [&](int r0, int r1, int c0, int jb, bool lower) {
        const int nblk = (r1 - r0 + 15) / 16;
        const C* F = A + (long)c0 * lda;
        C a[2][NX][GS_G];   // [buffer][block]
        auto load_batch = [&](int blk, int q) {
#pragma unroll
            for (int x = 0; x < NX; ++x)
                if (blk + x * GS_NW < nblk)
                    load(F, lda, min(r0 + (blk + x * GS_NW) * 16 + li, r1 - 1), q, jb, a[q & 1][x]);
        };
        read_x(c0, jb);
        {
            floatx4 acc[CB];
#pragma unroll
            for (int c = 0; c < CB; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < GS_Q; ++q)
                if (diag_on(q, jb, lower)) mult(d[q], q, acc);
            load_batch(wave, 0);
            __syncthreads();   // every read of X_p precedes the first write
            const int r = wave * 16 + li;
            if (r < jb) {
#pragma unroll
                for (int c = 0; c < CB; ++c) *reinterpret_cast<floatx4*>(xs + (c0 + r) * LD + c * 16 + 4 * g) = acc[c];
            }
            __syncthreads();
        }
        read_x(c0, jb);
        for (int blk = wave; blk < nblk; blk += NX * GS_NW) {
            floatx4 acc[NX][CB];
#pragma unroll
            for (int x = 0; x < NX; ++x)
#pragma unroll
                for (int c = 0; c < CB; ++c) acc[x][c] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < GS_Q; ++q) {
                if (q * 4 * GS_G < jb) {
                    if (q + 1 < GS_Q && (q + 1) * 4 * GS_G < jb) load_batch(blk, q + 1);
#pragma unroll
                    for (int x = 0; x < NX; ++x)
                        if (x == 0 || blk + x * GS_NW < nblk) mult(a[q & 1][x], q, acc[x]);
                }
            }
            load_batch(blk + NX * GS_NW, 0);
#pragma unroll
            for (int x = 0; x < NX; ++x) {
                const int row = r0 + (blk + x * GS_NW) * 16 + li;
                if (row < r1) {
#pragma unroll
                    for (int c = 0; c < CB; ++c) {
                        floatx4* p = reinterpret_cast<floatx4*>(xs + row * LD + c * 16 + 4 * g);
                        floatx4 v = *p;
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] -= acc[x][c][i];
                        *p = v;
                    }
                }
            }
        }
    };
    const C* Db = inv + (long)b * sInv;
    for (int p = 0; p < np; ++p) {
        const int c0 = p * nb, jb = min(nb, n - c0);
        diag_load(Db + (long)(2 * p) * nb * nb, jb, true);
        // this panel's interchanges: row pm[s].x receives old row pm[s].y
        const int2* pm = perm + (long)b * sPerm + (long)p * 2 * MAX_NB;
        __syncthreads();
        constexpr int W4 = 4 * CB, PQ = (2 * MAX_NB * W4 + GS_NT - 1) / GS_NT;
        floatx4 v[PQ];
        int dst[PQ];
#pragma unroll
        for (int q = 0; q < PQ; ++q) {
            const int e = tid + GS_NT * q;
            dst[q] = -1;
            if (e < 2 * jb * W4) {
                const int2 m = pm[e / W4];
                if (m.y >= 0) {
                    v[q] = *reinterpret_cast<const floatx4*>(xs + m.y * LD + 4 * (e % W4));
                    dst[q] = m.x;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PQ; ++q)
            if (dst[q] >= 0) *reinterpret_cast<floatx4*>(xs + dst[q] * LD + 4 * ((tid + GS_NT * q) % W4)) = v[q];
        __syncthreads();
        panel(c0 + jb, n, c0, jb, true);
    }
    for (int p = np - 1; p >= 0; --p) {
        const int c0 = p * nb, jb = min(nb, n - c0);
        diag_load(Db + (long)(2 * p + 1) * nb * nb, jb, false);
        __syncthreads();
        panel(0, c0, c0, jb, false);
    }
    __syncthreads();
    each([&](int r, int l, float* x) {
        if (l >= L) return;
        if constexpr (CX) Xb[r + (long)l * ldx] = make_float2(x[0], x[8]);
        else Xb[r + (long)l * ldx] = x[0];
    });
}

// LDS of a workgroup: complex 8 or 16, real 16 right-hand sides
template <typename C>
static size_t gs_lds(int n, int nrhs) { return (size_t)n * (elem_traits<C>::complex && nrhs > 8 ? 128 : 64); }
// At most 16 right-hand sides that fit: always (above).  17 to 64 in groups of 16, a workgroup each, which
// read the factor once per group, up to two workgroups per CU (64 right-hand sides, chain / groups: 48
// matrices n = 256 125 / 52 us, n = 1024 769 / 470, 128 matrices 141 / 102 and 1124 / 973).  With any_mix 17
// and more take the chain, whatever the batch: of 2048 matrices with 32 right-hand sides the groups take
// 1.1 (n = 1024) to 1.4 times as long (n = 128).
template <typename C>
static bool getrs_lds_ok(int n, int nrhs, int batch, bool any_mix)
{
    if (nrhs < 1 || nrhs > GS_MAX_RHS || gs_lds<C>(n, nrhs) > (size_t)128 << 10) return false;
    return nrhs <= 16 || (!any_mix && (long)batch * ((nrhs + 15) / 16) <= GS_MAX_WG);
}

template <typename C>
static hipError_t getrs_lds_batched(hipStream_t st, const C* LU, long sLU, int lda, int n, int nb, const LUWork& w,
                                    C* X, long sX, int ldx, int nrhs, int batch)
{
    if (nb > max_panel<float>()) nb = max_panel<float>();
    if (nb < MIN_NB) nb = MIN_NB;
    const size_t lds = gs_lds<C>(n, nrhs);
    const dim3 grid(batch, (nrhs + 15) / 16);
#define GS_L(CB)                                                                                                   \
    hipLaunchKernelGGL((getrs_lds_kernel<C, CB>), grid, dim3(GS_NT), lds, st, LU, sLU, lda, n, nb, w.perm, w.sPerm, \
                       (const C*)w.inv, w.sInv, X, sX, ldx, nrhs, w.active)
    if constexpr (elem_traits<C>::complex) {
        if (nrhs > 8) GS_L(2);
        else GS_L(1);
    } else {
        GS_L(1);
    }
#undef GS_L
    return hipGetLastError();
}

template <>
hipError_t getrf_batched<float>(hipStream_t st, float2* A, long sA, int lda, int n, int nb, const LUWork& w, int batch)
{
    return getrf_impl<float2>(st, A, sA, lda, n, nb, w, batch);
}
template <>
hipError_t getrf_batched<double>(hipStream_t st, double2* A, long sA, int lda, int n, int nb, const LUWork& w,
                                 int batch)
{
    return getrf_impl<double2>(st, A, sA, lda, n, nb, w, batch);
}
template <>
hipError_t getrs_batched<float>(hipStream_t st, const float2* LU, long sLU, int lda, int n, int nb, const LUWork& w,
                                float2* X, long sX, int ldx, int nrhs, int batch)
{
    if (getrs_lds_ok<float2>(n, nrhs, batch, w.any_mix))
        return getrs_lds_batched(st, LU, sLU, lda, n, nb, w, X, sX, ldx, nrhs, batch);
    return getrs_impl<float2>(st, LU, sLU, lda, n, nb, w, X, sX, ldx, nrhs, batch);
}
template <>
hipError_t getrs_batched<double>(hipStream_t st, const double2* LU, long sLU, int lda, int n, int nb,
                                 const LUWork& w, double2* X, long sX, int ldx, int nrhs, int batch)
{
    return getrs_impl<double2>(st, LU, sLU, lda, n, nb, w, X, sX, ldx, nrhs, batch);
}
hipError_t getrf_real_batched(hipStream_t st, float* A, long sA, int lda, int n, int nb, const LUWork& w, int batch)
{
    return getrf_impl<float>(st, A, sA, lda, n, nb, w, batch);
}
hipError_t getrs_real_batched(hipStream_t st, const float* LU, long sLU, int lda, int n, int nb, const LUWork& w,
                              float* X, long sX, int ldx, int nrhs, int batch)
{
    if (getrs_lds_ok<float>(n, nrhs, batch, w.any_mix))
        return getrs_lds_batched(st, LU, sLU, lda, n, nb, w, X, sX, ldx, nrhs, batch);
    return getrs_impl<float>(st, LU, sLU, lda, n, nb, w, X, sX, ldx, nrhs, batch);
}

}  // namespace rsrr
