// Element-wise and reduction kernels of the mixed-precision refinement
// (complex FP32 solves, FP64 residuals) and of the probe/solution copies.
// All operate on a batch of n x L column blocks (stride per point).
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace rsrr {

constexpr int EW_NT = 256;

// Right-hand sides of a factorisation with scaled rows: entry of row i times 2^-rs[i] (rs null: as it is).
RSRR_DEV double row_scaled(double v, const int* rs, long i) { return rs ? ldexp(v, -rs[i]) : v; }

// D_k = (c64) U for every point k.
__global__ __launch_bounds__(EW_NT) void bcast_to_c64_kernel(int n, int L, const double2* __restrict__ U, int ldu,
                                                              float2* __restrict__ D, int ldd, long sD,
                                                              const int* __restrict__ rs, long sRs)
{
    const int k = blockIdx.y;
    const int e = blockIdx.x * EW_NT + threadIdx.x;
    if (e >= n * L) return;
    const int i = e % n, c = e / n;
    const double2 u = U[i + (long)c * ldu];
    D[k * sD + i + (long)c * ldd] =
        make_float2((float)row_scaled(u.x, rs, k * sRs + i), (float)row_scaled(u.y, rs, k * sRs + i));
}

// R_k = U for every point k (FP64).
__global__ __launch_bounds__(EW_NT) void bcast_c128_kernel(int n, int L, const double2* __restrict__ U, int ldu,
                                                            double2* __restrict__ R, int ldr, long sR)
{
    const int k = blockIdx.y;
    const int e = blockIdx.x * EW_NT + threadIdx.x;
    if (e >= n * L) return;
    const int i = e % n, c = e / n;
    R[k * sR + i + (long)c * ldr] = U[i + (long)c * ldu];
}

// X_k = (c128) D_k.
__global__ __launch_bounds__(EW_NT) void widen_kernel(int n, int L, const float2* __restrict__ D, int ldd, long sD,
                                                       double2* __restrict__ X, int ldx, long sX)
{
    const int k = blockIdx.y;
    const int e = blockIdx.x * EW_NT + threadIdx.x;
    if (e >= n * L) return;
    const int i = e % n, c = e / n;
    X[k * sX + i + (long)c * ldx] = to_c128(D[k * sD + i + (long)c * ldd]);
}

// out[k*L + c] = ||X_k(:, c)||_2 (FP64, fixed summation order).
__global__ __launch_bounds__(EW_NT) void colnorm_kernel(int n, int L, const double2* __restrict__ X, int ldx, long sX,
                                                         double* __restrict__ out)
{
    __shared__ double red[EW_NT / 64];
    const int c = blockIdx.x, k = blockIdx.y;
    const double2* col = X + k * sX + (long)c * ldx;
    double v = 0.0;
    for (int i = threadIdx.x; i < n; i += EW_NT) {
        const double2 a = col[i];
        v += a.x * a.x + a.y * a.y;
    }
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < EW_NT / 64; ++w) s += red[w];
        out[(long)k * L + c] = sqrt(s);
    }
}

// D_k(:, c) = (c64) (R_k(:, c) * inv[k*L + c]) for active points.
__global__ __launch_bounds__(EW_NT) void scale_narrow_kernel(int n, int L, const double2* __restrict__ R, int ldr,
                                                              long sR, const double* __restrict__ inv,
                                                              float2* __restrict__ D, int ldd, long sD,
                                                              const int* __restrict__ active,
                                                              const int* __restrict__ rs, long sRs)
{
    const int k = blockIdx.y;
    if (active && !active[k]) return;
    const int e = blockIdx.x * EW_NT + threadIdx.x;
    if (e >= n * L) return;
    const int i = e % n, c = e / n;
    const double s = inv[(long)k * L + c];
    const double2 r = R[k * sR + i + (long)c * ldr];
    D[k * sD + i + (long)c * ldd] =
        make_float2((float)row_scaled(r.x * s, rs, k * sRs + i), (float)row_scaled(r.y * s, rs, k * sRs + i));
}

// X_k(:, c) += scale[k*L + c] * D_k(:, c) for active points.
__global__ __launch_bounds__(EW_NT) void axpy_widen_kernel(int n, int L, const float2* __restrict__ D, int ldd,
                                                            long sD, const double* __restrict__ scale,
                                                            double2* __restrict__ X, int ldx, long sX,
                                                            const int* __restrict__ active)
{
    const int k = blockIdx.y;
    if (active && !active[k]) return;
    const int e = blockIdx.x * EW_NT + threadIdx.x;
    if (e >= n * L) return;
    const int i = e % n, c = e / n;
    const double s = scale[(long)k * L + c];
    const float2 d = D[k * sD + i + (long)c * ldd];
    double2* x = X + k * sX + i + (long)c * ldx;
    double2 v = *x;
    v.x += s * (double)d.x;
    v.y += s * (double)d.y;
    *x = v;
}

// ---- real FP32 correction solves (a real NEP at real points) ----
// The FP64 residual stays complex (its imaginary part is exactly zero for a
// real problem); the real FP32 LU solves with its real part.  If the problem
// is not real after all, the refinement stalls and the point is redone on the
// FP64 complex path.

// D_k(:, c) = (float) (Re R_k(:, c) * inv[k*L + c]) (inv = null: 1) for active points.
__global__ __launch_bounds__(EW_NT) void scale_narrow_real_kernel(int n, int L, const double2* __restrict__ R, int ldr,
                                                                   long sR, const double* __restrict__ inv,
                                                                   float* __restrict__ D, int ldd, long sD,
                                                                   const int* __restrict__ active,
                                                                   const int* __restrict__ rs, long sRs)
{
    const int k = blockIdx.y;
    if (active && !active[k]) return;
    const int e = blockIdx.x * EW_NT + threadIdx.x;
    if (e >= n * L) return;
    const int i = e % n, c = e / n;
    const double s = inv ? inv[(long)k * L + c] : 1.0;
    D[k * sD + i + (long)c * ldd] = (float)row_scaled(R[k * sR + i + (long)c * ldr].x * s, rs, k * sRs + i);
}

// X_k(:, c) = (D_k(:, c), 0) when scale is null, else Re X_k(:, c) += scale[k*L + c] * D_k(:, c),
// for active points.
__global__ __launch_bounds__(EW_NT) void axpy_widen_real_kernel(int n, int L, const float* __restrict__ D, int ldd,
                                                                 long sD, const double* __restrict__ scale,
                                                                 double2* __restrict__ X, int ldx, long sX,
                                                                 const int* __restrict__ active)
{
    const int k = blockIdx.y;
    if (active && !active[k]) return;
    const int e = blockIdx.x * EW_NT + threadIdx.x;
    if (e >= n * L) return;
    const int i = e % n, c = e / n;
    const double d = (double)D[k * sD + i + (long)c * ldd];
    double2* x = X + k * sX + i + (long)c * ldx;
    if (!scale) {
        *x = make_double2(d, 0.0);
    } else {
        double2 v = *x;
        v.x += scale[(long)k * L + c] * d;
        *x = v;
    }
}

// Copy n x m (c128) blocks: Y_k = X_k.
__global__ __launch_bounds__(EW_NT) void copy_c128_kernel(int n, int m, const double2* __restrict__ X, int ldx,
                                                           long sX, double2* __restrict__ Y, int ldy, long sY)
{
    const int k = blockIdx.y;
    const long e = (long)blockIdx.x * EW_NT + threadIdx.x;
    if (e >= (long)n * m) return;
    const int i = (int)(e % n), c = (int)(e / n);
    Y[k * sY + i + (long)c * ldy] = X[k * sX + i + (long)c * ldx];
}

// Scale each column c of X (n x m) by s[c] (in place, FP64).
__global__ __launch_bounds__(EW_NT) void scale_cols_kernel(int n, int m, double2* __restrict__ X, int ldx,
                                                            const double* __restrict__ s)
{
    const long e = (long)blockIdx.x * EW_NT + threadIdx.x;
    if (e >= (long)n * m) return;
    const int i = (int)(e % n), c = (int)(e / n);
    double2* x = X + i + (long)c * ldx;
    const double f = s[c];
    x->x *= f;
    x->y *= f;
}

// ---- ragged-batch helpers ----

// Identity outside the leading nk x nk block of each P x P matrix (both copies
// may be null); the leading block is written by the assembly afterwards.  Only
// the padding is visited (grid-stride): with p = P - n, element e < n p lies in
// column e / p of the rows below the block (zero), the rest in the last p
// columns (identity).
template <typename C>
__global__ __launch_bounds__(EW_NT) void pad_identity_kernel(C* __restrict__ T, int ld, long sT, int P,
                                                              const int* __restrict__ nk)
{
    const int k = blockIdx.y;
    const int n = nk[k], p = P - n;
    const long total = p > 0 ? (long)p * (n + P) : 0;
    for (long e = (long)blockIdx.x * EW_NT + threadIdx.x; e < total; e += (long)gridDim.x * EW_NT) {
        int i, j;
        if (e < (long)n * p) {
            j = (int)(e / p);
            i = n + (int)(e % p);
        } else {
            const long f = e - (long)n * p;
            j = n + (int)(f / P);
            i = (int)(f % P);
        }
        C v;
        v.x = (i == j) ? 1 : 0;
        v.y = 0;
        T[k * sT + i + (long)j * ld] = v;
    }
}

// Fill n x m (c128) blocks with zeros (graph-safe replacement of a memset).
__global__ __launch_bounds__(EW_NT) void zero_c128_kernel(int n, int m, double2* __restrict__ X, int ldx, long sX)
{
    const int k = blockIdx.y;
    const long e = (long)blockIdx.x * EW_NT + threadIdx.x;
    if (e >= (long)n * m) return;
    X[k * sX + (e % n) + (long)(e / n) * ldx] = make_double2(0.0, 0.0);
}

__global__ __launch_bounds__(EW_NT) void zero_int_kernel(int* __restrict__ p, int n)
{
    const int e = blockIdx.x * EW_NT + threadIdx.x;
    if (e < n) p[e] = 0;
}

// Per-point refinement state: active = (getrf info == 0), prev = +inf.
__global__ __launch_bounds__(EW_NT) void ir_init_kernel(int M, const int* __restrict__ info, int* __restrict__ active,
                                                         double* __restrict__ prev, double* __restrict__ resid,
                                                         int* __restrict__ iters)
{
    const int k = blockIdx.x * EW_NT + threadIdx.x;
    if (k >= M) return;
    active[k] = info[k] == 0 ? 1 : 0;
    prev[k] = INFINITY;
    resid[k] = 0.0;
    iters[k] = 0;
}

// Device-side refinement decision for iteration `it` (one thread per point):
// rn, xn: column norms of R_k and X_k (M x Lmax); un: probe column norms
// (M x Lmax, zero for padding columns); frob: ||T_k||_F.  A point stops when
// its backward error max_c ||r_c|| / (||T||_F ||x_c|| + ||u_c||) <= tol_be,
// when the residual did not halve, or at it == maxit.  Writes the scaling
// of the next correction (inv = 1/||r_c||, scl = ||r_c||).
__global__ __launch_bounds__(EW_NT) void ir_decide_kernel(int M, int Lmax, const double* __restrict__ rn,
                                                           const double* __restrict__ xn,
                                                           const double* __restrict__ un,
                                                           const double* __restrict__ frob, double tol_be, int it,
                                                           int maxit, int* __restrict__ active,
                                                           double* __restrict__ prev, double* __restrict__ resid,
                                                           int* __restrict__ iters, double* __restrict__ inv,
                                                           double* __restrict__ scl)
{
    const int k = blockIdx.x * EW_NT + threadIdx.x;
    if (k >= M) return;
    if (!active[k]) return;
    double r = 0.0, eta = 0.0;
    bool nan = false;
    for (int c = 0; c < Lmax; ++c) {
        const double u = un[(long)k * Lmax + c];
        if (!(u > 0.0)) continue;
        const double rr = rn[(long)k * Lmax + c];
        if (!(rr == rr)) nan = true;
        r = fmax(r, rr / u);
        eta = fmax(eta, rr / (frob[k] * xn[(long)k * Lmax + c] + u));
    }
    resid[k] = nan ? INFINITY : r;
    iters[k] = it;
    const bool stop = nan || eta <= tol_be || r > 0.5 * prev[k] || it >= maxit;
    prev[k] = r;
    if (stop) { active[k] = 0; return; }
    for (int c = 0; c < Lmax; ++c) {
        const double rr = rn[(long)k * Lmax + c];
        inv[(long)k * Lmax + c] = rr > 0.0 ? 1.0 / rr : 0.0;
        scl[(long)k * Lmax + c] = rr;
    }
}


// R_b = U_b - T_b X_b (U null: T_b X_b) in FP64 for at most 32 right-hand sides: the
// product is skinny, so it is a stream over T, bound by HBM where there are enough
// rows.  A workgroup takes 64 rows of one matrix; its W waves split
// the columns of T (a contiguous range each) and their partial sums are added in a fixed
// order, so that small matrices and few points still keep many loads in
// flight (one workgroup per 1024 rows that walked all columns ran n = 3000, 32 points,
// L = 2 at 3.7 TB/s on 96 workgroups; n = 200, L = 16, 32 points took 141 us).  Nothing
// is shared before that sum, so there is no barrier in the loop.  Matrices with
// active[b] == 0 are skipped.  The split depends on n and L alone, never on the number of matrices: a
// point's residual has the same bits whatever shares its launch.
//
// Up to 8 columns (resid_stream_kernel): a lane owns a row, the loads of T are
// coalesced, and X(k, c), the same for the whole wave, comes through the scalar cache.  Eight waves at
// every size: fewer matrices need them (2048 rows, one matrix, 8 columns 65 us, four waves 118), and
// for many, four waves of one or two rows per lane take 0.91 to 1.13 times as long (1024 rows, 96 matrices, 4 columns
// 267 us against 293; 256 rows, 384 matrices, 8 columns 91 against 85).
// 9 to 32 columns (resid_mfma_kernel): v_mfma_f64_16x16x4f64 on four 16-row blocks and one or
// two 16-column blocks per wave; a lane loads whole complex entries and the real and
// imaginary parts go through separate instructions (inner index: four consecutive k).
// 17 to 32 columns fill half of a GEMM tile's 64: n = 1024, L = 32, 48 points 441 us there,
// 335 us here (T read once takes 170 us at a copy's rate, the products 177 us).

// The partial sums of the first W waves (acc: NV values per lane) added in order into wave 0's.
template <int NV, int W>
RSRR_DEV void wave_partials(double2 (&acc)[NV], double2* lds, int wave, int lane)
{
    if (wave > 0 && wave < W) {
#pragma unroll
        for (int v = 0; v < NV; ++v) lds[((wave - 1) * NV + v) * 64 + lane] = acc[v];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int w = 1; w < W; ++w)
#pragma unroll
            for (int v = 0; v < NV; ++v) acc[v] = cadd(acc[v], lds[((w - 1) * NV + v) * 64 + lane]);
    }
}

constexpr int RS_W = 8;   // waves

template <int LC>
__global__ __launch_bounds__(64 * RS_W) void resid_stream_kernel(int n, int L, const double2* __restrict__ T, int ldt,
                                                              long sT, const double2* __restrict__ X, int ldx,
                                                              long sX, const double2* __restrict__ U, int ldu,
                                                              long sU, double2* __restrict__ R, int ldr, long sR,
                                                              const int* __restrict__ active)
{
    constexpr int KU = LC <= 4 ? 4 : 2;   // columns of T in flight per row (X(k .. k+KU, :) fits the scalar registers)
    constexpr bool TWO = LC > 4;          // waves 4 to 7 into 0 to 3 first: half the LDS (57 KB for 8 columns)
    constexpr int W = RS_W, WS = TWO ? W / 2 : W;
    __shared__ double2 part[(TWO ? WS : W - 1) * LC * 64];
    const int b = blockIdx.y;
    if (active && !active[b]) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = blockIdx.x * 64 + lane;
    const int per = ((n + W - 1) / W + KU - 1) / KU * KU;
    const int k0 = min(n, wave * per), k1 = min(n, k0 + per);
    const double2* Xb = X + b * sX;
    const double2* Tb = T + b * sT;
    const int rr = min(row, n - 1);   // rows past the end read the last row and are not stored
    int xc[LC];    // columns past L read the last one and are not stored
#pragma unroll
    for (int c = 0; c < LC; ++c) xc[c] = min(c, L - 1);
    double2 acc[LC];
#pragma unroll
    for (int v = 0; v < LC; ++v) acc[v] = make_double2(0.0, 0.0);
    auto step = [&](int k, auto ku) {
        constexpr int KN = decltype(ku)::value;
        double2 t[KN];
#pragma unroll
        for (int u = 0; u < KN; ++u) t[u] = Tb[rr + (long)(k + u) * ldt];
#pragma unroll
        for (int c = 0; c < LC; ++c)
#pragma unroll
            for (int u = 0; u < KN; ++u) {
                const double2 x = Xb[(k + u) + (long)xc[c] * ldx];
                double2& a = acc[c];
                a.x = fma(t[u].x, x.x, a.x);
                a.y = fma(t[u].x, x.y, a.y);
                a.x = fma(-t[u].y, x.y, a.x);
                a.y = fma(t[u].y, x.x, a.y);
            }
    };
    int k = k0;
#pragma unroll 2
    for (; k + KU <= k1; k += KU) step(k, std::integral_constant<int, KU>{});
    for (; k < k1; ++k) step(k, std::integral_constant<int, 1>{});
    if constexpr (TWO) {
        if (wave >= WS) {
#pragma unroll
            for (int c = 0; c < LC; ++c) part[((wave - WS) * LC + c) * 64 + lane] = acc[c];
        }
        __syncthreads();
        if (wave < WS) {
#pragma unroll
            for (int c = 0; c < LC; ++c) acc[c] = cadd(acc[c], part[(wave * LC + c) * 64 + lane]);
        }
        __syncthreads();
    }
    wave_partials<LC, WS>(acc, part, wave, lane);
    if (wave > 0) return;
    double2* Rb = R + b * sR;
    const double2* Ub = U ? U + b * sU : nullptr;
    if (row >= n) return;
#pragma unroll
    for (int c = 0; c < LC; ++c)
        if (c < L) {
            double2 v = acc[c];
            if (Ub) v = csub(Ub[row + (long)c * ldu], v);
            Rb[row + (long)c * ldr] = v;
        }
}

template <int CB, int W>
__global__ __launch_bounds__(64 * W) void resid_mfma_kernel(int n, int L, const double2* __restrict__ T, int ldt,
                                                            long sT, const double2* __restrict__ X, int ldx, long sX,
                                                            const double2* __restrict__ U, int ldu, long sU,
                                                            double2* __restrict__ R, int ldr, long sR,
                                                            const int* __restrict__ active)
{
    constexpr int RB = 4;   // 16-row blocks per wave
    __shared__ double2 part[(W - 1) * RB * 4 * 64];   // one column block at a time
    const int b = blockIdx.y;
    if (active && !active[b]) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 15, kq = lane >> 4;
    const int row0 = blockIdx.x * 16 * RB + li;
    const int per = ((n + W - 1) / W + 3) / 4 * 4;
    const int k0 = min(n, wave * per), k1 = min(n, k0 + per);
    const double2* Tb = T + b * sT;
    const double2* Xc[CB];   // columns past L are not stored
#pragma unroll
    for (int y = 0; y < CB; ++y) Xc[y] = X + b * sX + (long)min(16 * y + li, L - 1) * ldx;
    int rr[RB];
#pragma unroll
    for (int x = 0; x < RB; ++x) rr[x] = min(row0 + 16 * x, n - 1);
    doublex4 accR[RB][CB], accI[RB][CB];
#pragma unroll
    for (int x = 0; x < RB; ++x)
#pragma unroll
        for (int y = 0; y < CB; ++y) accR[x][y] = accI[x][y] = doublex4{0.0, 0.0, 0.0, 0.0};
    // G groups of four k: all loads first; past the wave's range T counts as zero
    auto step = [&](int k, auto groups) {
        constexpr int G = decltype(groups)::value;
        double2 xv[G][CB], t[G][RB];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int kk = k + 4 * g + kq, kc = min(kk, k1 - 1);
#pragma unroll
            for (int y = 0; y < CB; ++y) xv[g][y] = Xc[y][kc];
#pragma unroll
            for (int x = 0; x < RB; ++x) {
                t[g][x] = Tb[rr[x] + (long)kc * ldt];
                if (kk >= k1) t[g][x] = make_double2(0.0, 0.0);
            }
        }
        // the first operand carries X, so that a lane's output runs along the rows of T X
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int x = 0; x < RB; ++x)
#pragma unroll
                for (int y = 0; y < CB; ++y) {
                    const double2 v = xv[g][y], a = t[g][x];
                    accR[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(v.x, a.x, accR[x][y], 0, 0, 0);
                    accI[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(v.y, a.x, accI[x][y], 0, 0, 0);
                    accR[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(-v.y, a.y, accR[x][y], 0, 0, 0);
                    accI[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(v.x, a.y, accI[x][y], 0, 0, 0);
                }
    };
    int k = k0;
    for (; k + 8 <= k1; k += 8) step(k, std::integral_constant<int, 2>{});
    for (; k < k1; k += 4) step(k, std::integral_constant<int, 1>{});
    double2* Rb = R + b * sR;
    const double2* Ub = U ? U + b * sU : nullptr;
#pragma unroll
    for (int y = 0; y < CB; ++y) {
        double2 acc[RB * 4];   // lane li: row, register r: column kq + 4 r
#pragma unroll
        for (int x = 0; x < RB; ++x)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[x * 4 + r] = make_double2(accR[x][y][r], accI[x][y][r]);
        if (y > 0) __syncthreads();   // wave 0 has read the previous block's sums
        wave_partials<RB * 4, W>(acc, part, wave, lane);
        if (wave == 0) {
#pragma unroll
            for (int x = 0; x < RB; ++x) {
                const int row = row0 + 16 * x;
                if (row >= n) continue;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int c = 16 * y + kq + 4 * r;
                    if (c < L) {
                        double2 v = acc[x * 4 + r];
                        if (Ub) v = csub(Ub[row + (long)c * ldu], v);
                        Rb[row + (long)c * ldr] = v;
                    }
                }
            }
        }
    }
}

static dim3 ew_grid(long elems, int B) { return dim3((unsigned)((elems + EW_NT - 1) / EW_NT), B); }
// Ub_k (rows < n, columns < L) = U_q for point k = koff + blockIdx.y of instance blockIdx.z.
__global__ __launch_bounds__(EW_NT) void bcast_group_kernel(const RhsInstance* __restrict__ ins,
                                                             double2* __restrict__ Ub, int ldb, long sB)
{
    const RhsInstance in = ins[blockIdx.z];
    const int k = blockIdx.y;
    const long e = (long)blockIdx.x * EW_NT + threadIdx.x;
    if (k >= in.N || e >= (long)in.n * in.L) return;
    const int i = (int)(e % in.n), c = (int)(e / in.n);
    Ub[(in.koff + k) * sB + i + (long)c * ldb] = in.U[i + (long)c * in.ldu];
}

// S_q columns k L .. k L + L - 1 (rows < n) = X_(koff + k) for point k = blockIdx.y of instance blockIdx.z.
__global__ __launch_bounds__(EW_NT) void copy_out_group_kernel(const RhsInstance* __restrict__ ins,
                                                                const double2* __restrict__ Xb, int ldb, long sB)
{
    const RhsInstance in = ins[blockIdx.z];
    const int k = blockIdx.y;
    const long e = (long)blockIdx.x * EW_NT + threadIdx.x;
    if (k >= in.N || e >= (long)in.n * in.L) return;
    const int i = (int)(e % in.n), c = (int)(e / in.n);
    in.S[i + ((long)k * in.L + c) * in.lds] = Xb[(in.koff + k) * sB + i + (long)c * ldb];
}

hipError_t bcast_group(hipStream_t st, const RhsInstance* ins, int nins, int nmax, int Lmax, int Nmax,
                       double2* Ub, int ldb, long sB)
{
    const dim3 g((unsigned)(((long)nmax * Lmax + EW_NT - 1) / EW_NT), (unsigned)Nmax, (unsigned)nins);
    hipLaunchKernelGGL(bcast_group_kernel, g, dim3(EW_NT), 0, st, ins, Ub, ldb, sB);
    return hipGetLastError();
}

hipError_t copy_out_group(hipStream_t st, const RhsInstance* ins, int nins, int nmax, int Lmax, int Nmax,
                          const double2* Xb, int ldb, long sB)
{
    const dim3 g((unsigned)(((long)nmax * Lmax + EW_NT - 1) / EW_NT), (unsigned)Nmax, (unsigned)nins);
    hipLaunchKernelGGL(copy_out_group_kernel, g, dim3(EW_NT), 0, st, ins, Xb, ldb, sB);
    return hipGetLastError();
}


hipError_t pad_identity(hipStream_t st, float2* T64, double2* T128, int ld, long sT, int P, const int* nk, int M)
{
    // one thread per padding element of a matrix of a 64-wide size bucket (P - n < 64)
    const long cover = std::min((long)P * P, 128L * P);
    if (T64) hipLaunchKernelGGL(pad_identity_kernel<float2>, ew_grid(cover, M), dim3(EW_NT), 0, st, T64, ld, sT,
                                P, nk);
    if (T128) hipLaunchKernelGGL(pad_identity_kernel<double2>, ew_grid(cover, M), dim3(EW_NT), 0, st, T128, ld,
                                 sT, P, nk);
    return hipGetLastError();
}
hipError_t zero_c128(hipStream_t st, int n, int m, double2* X, int ldx, long sX, int B)
{
    hipLaunchKernelGGL(zero_c128_kernel, ew_grid((long)n * m, B), dim3(EW_NT), 0, st, n, m, X, ldx, sX);
    return hipGetLastError();
}
hipError_t zero_int(hipStream_t st, int* p, int n)
{
    hipLaunchKernelGGL(zero_int_kernel, dim3((n + EW_NT - 1) / EW_NT), dim3(EW_NT), 0, st, p, n);
    return hipGetLastError();
}
hipError_t ir_init(hipStream_t st, int M, const int* info, int* active, double* prev, double* resid, int* iters)
{
    hipLaunchKernelGGL(ir_init_kernel, dim3((M + EW_NT - 1) / EW_NT), dim3(EW_NT), 0, st, M, info, active, prev,
                       resid, iters);
    return hipGetLastError();
}
hipError_t ir_decide(hipStream_t st, int M, int Lmax, const double* rn, const double* xn, const double* un,
                     const double* frob, double tol_be, int it, int maxit, int* active, double* prev, double* resid,
                     int* iters, double* inv, double* scl)
{
    hipLaunchKernelGGL(ir_decide_kernel, dim3((M + EW_NT - 1) / EW_NT), dim3(EW_NT), 0, st, M, Lmax, rn, xn, un, frob,
                       tol_be, it, maxit, active, prev, resid, iters, inv, scl);
    return hipGetLastError();
}

hipError_t bcast_to_c64(hipStream_t st, int n, int L, const double2* U, int ldu, float2* D, int ldd, long sD, int B,
                        const int* rs, long sRs)
{
    hipLaunchKernelGGL(bcast_to_c64_kernel, ew_grid((long)n * L, B), dim3(EW_NT), 0, st, n, L, U, ldu, D, ldd, sD, rs,
                       sRs);
    return hipGetLastError();
}
hipError_t bcast_c128(hipStream_t st, int n, int L, const double2* U, int ldu, double2* R, int ldr, long sR, int B)
{
    hipLaunchKernelGGL(bcast_c128_kernel, ew_grid((long)n * L, B), dim3(EW_NT), 0, st, n, L, U, ldu, R, ldr, sR);
    return hipGetLastError();
}
hipError_t widen(hipStream_t st, int n, int L, const float2* D, int ldd, long sD, double2* X, int ldx, long sX, int B)
{
    hipLaunchKernelGGL(widen_kernel, ew_grid((long)n * L, B), dim3(EW_NT), 0, st, n, L, D, ldd, sD, X, ldx, sX);
    return hipGetLastError();
}
hipError_t colnorms(hipStream_t st, int n, int L, const double2* X, int ldx, long sX, double* out, int B)
{
    hipLaunchKernelGGL(colnorm_kernel, dim3(L, B), dim3(EW_NT), 0, st, n, L, X, ldx, sX, out);
    return hipGetLastError();
}
hipError_t scale_narrow(hipStream_t st, int n, int L, const double2* R, int ldr, long sR, const double* inv,
                        float2* D, int ldd, long sD, const int* active, int B, const int* rs, long sRs)
{
    hipLaunchKernelGGL(scale_narrow_kernel, ew_grid((long)n * L, B), dim3(EW_NT), 0, st, n, L, R, ldr, sR, inv, D,
                       ldd, sD, active, rs, sRs);
    return hipGetLastError();
}
hipError_t axpy_widen(hipStream_t st, int n, int L, const float2* D, int ldd, long sD, const double* scale,
                      double2* X, int ldx, long sX, const int* active, int B)
{
    hipLaunchKernelGGL(axpy_widen_kernel, ew_grid((long)n * L, B), dim3(EW_NT), 0, st, n, L, D, ldd, sD, scale, X,
                       ldx, sX, active);
    return hipGetLastError();
}
hipError_t copy_c128(hipStream_t st, int n, int m, const double2* X, int ldx, long sX, double2* Y, int ldy, long sY,
                     int B)
{
    hipLaunchKernelGGL(copy_c128_kernel, ew_grid((long)n * m, B), dim3(EW_NT), 0, st, n, m, X, ldx, sX, Y, ldy, sY);
    return hipGetLastError();
}
hipError_t scale_cols(hipStream_t st, int n, int m, double2* X, int ldx, const double* s)
{
    hipLaunchKernelGGL(scale_cols_kernel, ew_grid((long)n * m, 1), dim3(EW_NT), 0, st, n, m, X, ldx, s);
    return hipGetLastError();
}


bool resid_skinny_ok(int L) { return L >= 1 && L <= 32; }

hipError_t resid_skinny(hipStream_t st, int n, int L, const double2* T, int ldt, long sT, const double2* X, int ldx,
                        long sX, const double2* U, int ldu, long sU, double2* R, int ldr, long sR, const int* active,
                        int B)
{
#define RS_L(LC)                                                                                                     \
    hipLaunchKernelGGL(resid_stream_kernel<LC>, dim3((unsigned)((n + 63) / 64), (unsigned)B), dim3(64 * RS_W), 0, st, \
                       n, L, T, ldt, sT, X, ldx, sX, U, ldu, sU, R, ldr, sR, active)
#define RS_M(CB, W)                                                                                                  \
    hipLaunchKernelGGL((resid_mfma_kernel<CB, W>), dim3((unsigned)((n + 63) / 64), (unsigned)B), dim3(64 * W), 0, st, \
                       n, L, T, ldt, sT, X, ldx, sX, U, ldu, sU, R, ldr, sR, active)
    if (L <= 2) {
        RS_L(2);
    } else if (L <= 4) {
        RS_L(4);
    } else if (L <= 8) {
        RS_L(8);
    } else if (L <= 16) {
        RS_M(1, 4);
    } else {
        RS_M(2, 4);
    }
#undef RS_M
#undef RS_L
    return hipGetLastError();
}

hipError_t scale_narrow_real(hipStream_t st, int n, int L, const double2* R, int ldr, long sR, const double* inv,
                             float* D, int ldd, long sD, const int* active, int B, const int* rs, long sRs)
{
    hipLaunchKernelGGL(scale_narrow_real_kernel, ew_grid((long)n * L, B), dim3(EW_NT), 0, st, n, L, R, ldr, sR, inv,
                       D, ldd, sD, active, rs, sRs);
    return hipGetLastError();
}
hipError_t axpy_widen_real(hipStream_t st, int n, int L, const float* D, int ldd, long sD, const double* scale,
                           double2* X, int ldx, long sX, const int* active, int B)
{
    hipLaunchKernelGGL(axpy_widen_real_kernel, ew_grid((long)n * L, B), dim3(EW_NT), 0, st, n, L, D, ldd, sD, scale,
                       X, ldx, sX, active);
    return hipGetLastError();
}

}  // namespace rsrr
