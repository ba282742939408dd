// Truncated SVD of the normalised sampling matrix (RSRR Step 3) by block
// one-sided Jacobi in FP64.
//
// The columns of A (m x p) are split into blocks of JB_B columns.  A sweep
// pairs every block with every other once (round-robin tournament, all
// pairs of a round independent).  A round is two launches:
//   1. gram:  for every pair and every slice of JRG rows, one workgroup forms
//      the partial Gram matrix [A_I A_J]^H [A_I A_J] (2B x 2B) of its slice;
//   2. rotate: for every pair and every slice of JR rows of the m_apply rows
//      that are rotated, one workgroup sums the pair's Gram slices (fixed
//      order), measures max |G_pq| / sqrt(G_pp G_qq) over p != q (the
//      convergence measure of one-sided Jacobi; columns with |a|^2 <= zthr2,
//      rounding level relative to ||A||_F, count as zero and are neither
//      measured nor rotated, so exactly rank-deficient inputs converge),
//      applies one sweep of two-sided Jacobi rotations to G (parallel
//      ordering) accumulating the unitary V, and applies
//      [A_I A_J] <- [A_I A_J] V to its rows.  The first round of a sweep
//      rotates all pairs of the 2B columns, the others the pairs between the
//      two blocks, so that every pair of columns is rotated once a sweep.
//      Every workgroup of a pair does the same small sweep on the same data,
//      so they agree bitwise; slice 0 records the measure.
// Both products are on the FP64 matrix cores, straight from memory; a round is
// then bound by the dependent steps of the small sweep.
// Splitting the rows keeps every CU busy although a round has only p/(2B)
// pairs.  When every pair's measure is below the tolerance the columns of A
// are orthogonal: A = U Sigma with the column norms as singular values.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace rsrr {

constexpr int JB_B = 16;          // columns per block
constexpr int JB_W = 2 * JB_B;    // columns per pair
constexpr int JB_NT = 256;

// block at tournament position pos in round r (nb even, position 0 fixed)
RSRR_DEV int rr_block(int pos, int r, int nb) { return pos == 0 ? 0 : ((pos - 1 + r) % (nb - 1)) + 1; }

constexpr int JR = 64;            // rows per slice of the rotation (16 per wave)
constexpr int JRG = 128;          // rows per slice of the Gram matrices

RSRR_DEV int jac_col(int s, int bI, int bJ, int p)
{
    const int c = (s < JB_B ? bI : bJ) * JB_B + (s % JB_B);
    return c < p ? c : -1;
}

// 1. partial Gram matrix of rows [slice*JRG, min(m, slice*JRG + JRG)) of pair blockIdx.x.
// The waves take chunks of 16 rows in turn; a lane loads four consecutive rows of its
// column of either block, which are the four inner indices of its MFMA operands (any
// order of the rows gives the same sum).  The blocks (I,I), (I,J) and (J,J) are formed,
// the waves' sums added in order, (J,I) is the conjugate of (I,J).
__global__ __launch_bounds__(JB_NT) void jacobi_gram_kernel(const double2* __restrict__ A, int lda, int m, int p,
                                                             int nb, int round, double2* __restrict__ Gp)
{
    constexpr int NW = JB_NT / 64;
    __shared__ double2 part[NW][3][4][64];
    const int pr = blockIdx.x, slice = blockIdx.y, tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6, li = lane & 15, kq = lane >> 4;
    const int bI = rr_block(pr, round, nb), bJ = rr_block(nb - 1 - pr, round, nb);
    const int rlo = slice * JRG, rhi = min(m, rlo + JRG);
    const int cI = jac_col(li, bI, bJ, p), cJ = jac_col(JB_B + li, bI, bJ, p);
    doublex4 re[3], im[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) re[t] = im[t] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ch = 0; ch < JRG / (16 * NW); ++ch) {
        const int r0 = rlo + 16 * (wave + NW * ch) + 4 * kq;
        double2 x[4], y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            x[u] = (cI >= 0 && r0 + u < rhi) ? A[(r0 + u) + (long)cI * lda] : make_double2(0.0, 0.0);
            y[u] = (cJ >= 0 && r0 + u < rhi) ? A[(r0 + u) + (long)cJ * lda] : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            // G_ij = sum conj(a_i) a_j: first operand i, second operand j
            auto add = [&](int t, double2 a, double2 b) {
                re[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, re[t], 0, 0, 0);
                im[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, im[t], 0, 0, 0);
                re[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.y, re[t], 0, 0, 0);
                im[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.x, im[t], 0, 0, 0);
            };
            add(0, x[u], x[u]);
            add(1, x[u], y[u]);
            add(2, y[u], y[u]);
        }
    }
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[wave][t][r][lane] = make_double2(re[t][r], im[t][r]);
    __syncthreads();
    double2* G = Gp + ((long)pr * gridDim.y + slice) * (JB_W * JB_W);
#pragma unroll
    for (int q = 0; q < 3 * 4 * 64 / JB_NT; ++q) {
        const int e = tid + JB_NT * q, l = e & 63, r = (e >> 6) & 3, t = e >> 8;
        double2 v = part[0][t][r][l];
#pragma unroll
        for (int w = 1; w < NW; ++w) v = cadd(v, part[w][t][r][l]);
        const int i = (l >> 4) + 4 * r, j = l & 15;   // register r of lane l: row l / 16 + 4 r, column l % 16
        if (t == 0) G[i * JB_W + j] = v;
        else if (t == 2) G[(JB_B + i) * JB_W + JB_B + j] = v;
        else {
            G[i * JB_W + JB_B + j] = v;
            G[(JB_B + j) * JB_W + i] = cconj(v);
        }
    }
}

// The rotation that makes columns a, b with Gram entries da, db (diagonal) and g = G_ab
// orthogonal: x_a <- c x_a - conj(e) x_b, x_b <- e x_a + c x_b (e carries the sine).  With
// tau = db - da and w = |tau| + sqrt(tau^2 + 4|g|^2) the tangent is 2|g|/w, so neither
// |g| nor a division by it is needed: one square root, one division, one reciprocal root.
struct JacRot { double c; double2 e; };
RSRR_DEV JacRot jac_rot(double da, double db, double2 g, double zthr2, double thr2)
{
    JacRot r = {1.0, make_double2(0.0, 0.0)};
    const double h2 = g.x * g.x + g.y * g.y;
    if (da > zthr2 && db > zthr2 && h2 > thr2 * (da * db)) {
        const double tau = db - da;
        const double w = fabs(tau) + sqrt(tau * tau + 4.0 * h2);
        const double q = (tau >= 0.0 ? 2.0 : -2.0) / w;
        r.c = 1.0 / sqrt(1.0 + q * q * h2);
        r.e = make_double2(r.c * q * g.x, r.c * q * g.y);
    }
    return r;
}

// 2. sum the Gram slices of pair blockIdx.x, measure, one sweep of rotations on G, and
// rotate the rows of slice blockIdx.y.  A step of the sweep applies JB_W / 2 disjoint
// rotations (a_k, b_k) from both sides at once; thread (qi, qj) owns the 2 x 2 entries of
// G at rows {a_qi, b_qi} x columns {a_qj, b_qj}, works out both rotations itself from the
// current G and writes its entries into the other of two buffers, so a step needs one
// barrier.  240 columns of 240 rows: 22 us a round and 7 us for its Gram matrices (64 + 21 us with
// two barriers a step, 31 steps every round, one division after the other in 16
// threads, and both products on the vector units out of LDS).
__global__ __launch_bounds__(JB_NT) void jacobi_rotate_kernel(double2* __restrict__ A, int lda, int m_apply, int p,
                                                               int nb, int round, const double2* __restrict__ Gp,
                                                               int slices, double tol, double zthr2,
                                                               double* __restrict__ offmax)
{
    static_assert(JB_NT == (JB_W / 2) * (JB_W / 2), "one thread per 2 x 2 block of a step");
    static_assert(JR == 16 * (JB_NT / 64), "16 rows per wave");
    __shared__ double2 G[2][JB_W][JB_W + 1];
    __shared__ double2 V[JB_W][JB_W + 1];
    __shared__ double wmax[JB_NT / 64];
    const int pr = blockIdx.x, slice = blockIdx.y, tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6, li = lane & 15, kq = lane >> 4;
    const int bI = rr_block(pr, round, nb), bJ = rr_block(nb - 1 - pr, round, nb);
    // the wave's 16 rows (row li, column kq + 4 t), needed after the sweep
    const int row = slice * JR + 16 * wave + li;
    double2 x[JB_W / 4];
#pragma unroll
    for (int t = 0; t < JB_W / 4; ++t) {
        const int c = jac_col(kq + 4 * t, bI, bJ, p);
        x[t] = (c >= 0 && row < m_apply) ? A[row + (long)c * lda] : make_double2(0.0, 0.0);
    }
    const double2* src = Gp + (long)pr * slices * (JB_W * JB_W);
    constexpr int PER = JB_W * JB_W / JB_NT;
    {
        // JS_SL slices' loads in flight at once; each entry is summed in slice order
        constexpr int JS_SL = 8;
        double2 g[PER];
#pragma unroll
        for (int t = 0; t < PER; ++t) g[t] = make_double2(0.0, 0.0);
        for (int sl0 = 0; sl0 < slices; sl0 += JS_SL) {
            double2 v[JS_SL][PER];
#pragma unroll
            for (int q = 0; q < JS_SL; ++q) {
                const double2* sp = src + (long)(sl0 + q) * (JB_W * JB_W) + tid;
#pragma unroll
                for (int t = 0; t < PER; ++t) v[q][t] = sl0 + q < slices ? sp[JB_NT * t] : make_double2(0.0, 0.0);
            }
#pragma unroll
            for (int q = 0; q < JS_SL; ++q) {
                if (sl0 + q >= slices) break;
#pragma unroll
                for (int t = 0; t < PER; ++t) g[t] = cadd(g[t], v[q][t]);
            }
        }
#pragma unroll
        for (int t = 0; t < PER; ++t) {
            const int e = tid + JB_NT * t;
            G[0][e / JB_W][e % JB_W] = g[t];
            V[e / JB_W][e % JB_W] = make_double2(e / JB_W == e % JB_W ? 1.0 : 0.0, 0.0);
        }
    }
    __syncthreads();
    double off = 0.0;   // the largest squared measure
    for (int e = tid; e < JB_W * JB_W; e += JB_NT) {
        const int i = e / JB_W, q = e % JB_W;
        if (i == q) continue;
        const double dp = G[0][i][i].x, dq = G[0][q][q].x;
        if (dp > zthr2 && dq > zthr2) {
            const double2 g = G[0][i][q];
            off = fmax(off, (g.x * g.x + g.y * g.y) / (dp * dq));
        }
    }
    for (int o = 32; o >= 1; o >>= 1) off = fmax(off, __shfl_xor(off, o));
    if ((tid & 63) == 0) wmax[tid >> 6] = off;
    __syncthreads();
    off = wmax[0];
    for (int w = 1; w < JB_NT / 64; ++w) off = fmax(off, wmax[w]);
    off = sqrt(off);
    if (slice == 0 && tid == 0) offmax[pr] = off;
    if (off <= tol) return;  // pair already orthogonal: A stays unchanged (uniform over the workgroup)

    const int qi = tid / (JB_W / 2), qj = tid % (JB_W / 2);
    const double thr2 = 0.0625 * tol * tol;
    const bool all = round == 0;
    const int steps = all ? JB_W - 1 : JB_B;
    int cur = 0;
    for (int st = 0; st < steps; ++st) {
        auto pair_of = [&](int k, int& a, int& b) {
            if (all) {
                const int u = rr_block(k, st, JB_W), v = rr_block(JB_W - 1 - k, st, JB_W);
                a = min(u, v);
                b = max(u, v);
            } else {
                a = k;
                b = JB_B + ((k + st) & (JB_B - 1));
            }
        };
        int ra, rb, ca, cb;
        pair_of(qi, ra, rb);
        pair_of(qj, ca, cb);
        const double2 (*Gc)[JB_W + 1] = G[cur];
        double2 (*Gn)[JB_W + 1] = G[cur ^ 1];
        double2 g00 = Gc[ra][ca], g01 = Gc[ra][cb], g10 = Gc[rb][ca], g11 = Gc[rb][cb];
        double2 v00 = V[qi][ca], v01 = V[qi][cb], v10 = V[qi + JB_B][ca], v11 = V[qi + JB_B][cb];
        const JacRot ri = jac_rot(Gc[ra][ra].x, Gc[rb][rb].x, Gc[ra][rb], zthr2, thr2);
        const JacRot rj = jac_rot(Gc[ca][ca].x, Gc[cb][cb].x, Gc[ca][cb], zthr2, thr2);
        // columns a, b: x_a <- c x_a - conj(e) x_b, x_b <- e x_a + c x_b
        auto colop = [&](double2& xa, double2& xb) {
            const double2 t = cmul(cconj(rj.e), xb), u = cmul(rj.e, xa);
            xa = make_double2(rj.c * xa.x - t.x, rj.c * xa.y - t.y);
            xb = make_double2(u.x + rj.c * xb.x, u.y + rj.c * xb.y);
        };
        colop(g00, g01);
        colop(g10, g11);
        colop(v00, v01);
        colop(v10, v11);
        // rows a, b: r_a <- c r_a - e r_b, r_b <- conj(e) r_a + c r_b
        auto rowop = [&](double2& xa, double2& xb) {
            const double2 t = cmul(ri.e, xb), u = cmul(cconj(ri.e), xa);
            xa = make_double2(ri.c * xa.x - t.x, ri.c * xa.y - t.y);
            xb = make_double2(u.x + ri.c * xb.x, u.y + ri.c * xb.y);
        };
        rowop(g00, g10);
        rowop(g01, g11);
        if (qi == qj) {
            // a rotated pair's coupling is zero, its diagonal real
            if (ri.e.x != 0.0 || ri.e.y != 0.0) g01 = g10 = make_double2(0.0, 0.0);
            g00.y = 0.0;
            g11.y = 0.0;
        }
        Gn[ra][ca] = g00; Gn[ra][cb] = g01; Gn[rb][ca] = g10; Gn[rb][cb] = g11;
        V[qi][ca] = v00; V[qi][cb] = v01; V[qi + JB_B][ca] = v10; V[qi + JB_B][cb] = v11;
        cur ^= 1;
        __syncthreads();
    }
    // [A_I A_J] <- [A_I A_J] V on the wave's rows; the first operand carries V, so that a
    // lane's output runs along the rows: register r holds column lane / 16 + 4 r
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        doublex4 re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int t = 0; t < JB_W / 4; ++t) {
            const double2 v = V[kq + 4 * t][h * JB_B + li];
            re = __builtin_amdgcn_mfma_f64_16x16x4f64(v.x, x[t].x, re, 0, 0, 0);
            im = __builtin_amdgcn_mfma_f64_16x16x4f64(v.x, x[t].y, im, 0, 0, 0);
            re = __builtin_amdgcn_mfma_f64_16x16x4f64(-v.y, x[t].y, re, 0, 0, 0);
            im = __builtin_amdgcn_mfma_f64_16x16x4f64(v.y, x[t].x, im, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = jac_col(h * JB_B + kq + 4 * r, bI, bJ, p);
            if (c >= 0 && row < m_apply) A[row + (long)c * lda] = make_double2(re[r], im[r]);
        }
    }
}

// Q(:, i) = A(:, order[i]) * inv[i] for i < k.
__global__ __launch_bounds__(256) void gather_scale_kernel(const double2* __restrict__ A, int lda, int m,
                                                            const int* __restrict__ order,
                                                            const double* __restrict__ inv, double2* __restrict__ Q,
                                                            int ldq, int k)
{
    const long e = (long)blockIdx.x * 256 + threadIdx.x;
    if (e >= (long)m * k) return;
    const int i = (int)(e % m), c = (int)(e / m);
    const double2 a = A[i + (long)order[c] * lda];
    const double s = inv[c];
    Q[i + (long)c * ldq] = make_double2(a.x * s, a.y * s);
}

// ----------------------------------------------------------------------------
// Seeded complex Gaussian matrix (n x m, ld n): entry e uses the counter-based
// generator splitmix64(seed, e) -> two uniforms -> Box-Muller.  Deterministic.
// ----------------------------------------------------------------------------
RSRR_DEV unsigned long long splitmix64(unsigned long long x)
{
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

__global__ __launch_bounds__(256) void gaussian_kernel(double2* __restrict__ X, int n, int m, int ld,
                                                        unsigned long long seed)
{
    const long e = (long)blockIdx.x * 256 + threadIdx.x;
    if (e >= (long)n * m) return;
    const int i = (int)(e % n), j = (int)(e / n);
    const unsigned long long h1 = splitmix64(seed ^ splitmix64((unsigned long long)e * 2ull));
    const unsigned long long h2 = splitmix64(seed ^ splitmix64((unsigned long long)e * 2ull + 1ull));
    const double u1 = ((h1 >> 11) + 1.0) * (1.0 / 9007199254740993.0);  // (0, 1]
    const double u2 = (h2 >> 11) * (1.0 / 9007199254740992.0);         // [0, 1)
    const double r = sqrt(-2.0 * log(u1)) * 0.70710678118654752;
    double sn, cs;
    sincos(6.283185307179586 * u2, &sn, &cs);
    X[i + (long)j * ld] = make_double2(r * cs, r * sn);
}

// ----------------------------------------------------------------------------
// Classical Gram-Schmidt with reorthogonalisation inside one block of bw <= CG_BW
// columns (column c against columns 0..c-1 of the block, twice, then
// normalised).  One workgroup; the block stays in global memory (L2).
// A column whose remaining norm is at most thr * ref[c] (ref = nullptr: 1) is
// numerically dependent on the columns before it and is set to zero: what
// remains of it is rounding noise, and normalising noise would break the
// orthogonality of everything after it.
// ----------------------------------------------------------------------------
constexpr int CG_BW = 8;      // columns per block: the projections on earlier blocks are GEMMs
constexpr int CG_NT = 1024;   // one workgroup per block; many waves keep loads in flight

__global__ __launch_bounds__(CG_NT) void block_cgs2_kernel(double2* __restrict__ Y, int ld, int n, int bw,
                                                            const double* __restrict__ ref, double thr)
{
    constexpr int NW = CG_NT / 64;
    __shared__ double2 red[NW][CG_BW];
    __shared__ double2 coef[CG_BW];
    __shared__ double nred[NW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int c = 0; c < bw; ++c) {
        double2* y = Y + (long)c * ld;
        for (int pass = 0; pass < 2 && c > 0; ++pass) {
            double2 acc[CG_BW];
#pragma unroll
            for (int j = 0; j < CG_BW; ++j) acc[j] = make_double2(0.0, 0.0);
            for (int r = tid; r < n; r += CG_NT) {
                const double2 v = y[r];
#pragma unroll
                for (int j = 0; j < CG_BW; ++j)
                    if (j < c) acc[j] = cfma_cj(acc[j], Y[r + (long)j * ld], v);
            }
#pragma unroll
            for (int j = 0; j < CG_BW; ++j) {
                if (j >= c) break;
                double2 a = acc[j];
                for (int o = 32; o >= 1; o >>= 1) { a.x += __shfl_xor(a.x, o); a.y += __shfl_xor(a.y, o); }
                if (lane == 0) red[wave][j] = a;
            }
            __syncthreads();
            if (tid < c) {
                double2 t = red[0][tid];
                for (int w = 1; w < NW; ++w) t = cadd(t, red[w][tid]);
                coef[tid] = t;
            }
            __syncthreads();
            for (int r = tid; r < n; r += CG_NT) {
                double2 v = y[r];
                for (int j = 0; j < c; ++j) v = cfms(v, Y[r + (long)j * ld], coef[j]);
                y[r] = v;
            }
            __syncthreads();
        }
        double s2 = 0.0;
        for (int r = tid; r < n; r += CG_NT) { const double2 v = y[r]; s2 += v.x * v.x + v.y * v.y; }
        for (int o = 32; o >= 1; o >>= 1) s2 += __shfl_xor(s2, o);
        if (lane == 0) nred[wave] = s2;
        __syncthreads();
        double tot = 0.0;
        for (int w = 0; w < NW; ++w) tot += nred[w];
        const double nn = sqrt(tot);
        const double inv = nn > thr * (ref ? ref[c] : 1.0) ? 1.0 / nn : 0.0;
        for (int r = tid; r < n; r += CG_NT) { const double2 v = y[r]; y[r] = make_double2(v.x * inv, v.y * inv); }
        __syncthreads();
    }
}

hipError_t gaussian(hipStream_t st, double2* X, int n, int m, int ld, unsigned long long seed)
{
    const long e = (long)n * m;
    hipLaunchKernelGGL(gaussian_kernel, dim3((unsigned)((e + 255) / 256)), dim3(256), 0, st, X, n, m, ld, seed);
    return hipGetLastError();
}

// Projection of the block Yj = Y[:, j0:j0+bw] off the finished columns
// Y[:, :j0]:  W = Y[:, :j0]^H Yj,  Yj -= Y[:, :j0] W.  Both products are
// skinny (bw columns), so each is split along its long inner dimension into
// slices that run as one batched MFMA GEMM, and the slices are summed in a
// fixed order (deterministic).
// The slices are as short as it takes to fill the chip: a 64 x 64 tile walks its slice at
// 1.7 us per 16 inner indices, whatever else runs (256 rows a slice at n = 2048: 64
// workgroups, 72 us a product; 64 rows a slice: 31 us, with the faster GEMM).
constexpr int PK_MIN = 64, PK_TILES = 256;
// inner slice of W = Y^H Yj (rows of Y) for j0 finished columns: about PK_TILES tiles
static int pk_rows(int n, int j0)
{
    const long want = ((long)n * ((j0 + 63) / 64) / PK_TILES + PK_MIN - 1) / PK_MIN * PK_MIN;
    return (int)std::max<long>(PK_MIN, want);
}
// inner slice of Yj -= Y W (columns of Y)
static int pk_cols(int n) { return n <= 2048 ? 64 : 128; }

__global__ __launch_bounds__(256) void sum_parts_kernel(const double2* __restrict__ part, int S, int rows, int cols,
                                                         double2* __restrict__ out, int ldo, int sub)
{
    const long e = (long)blockIdx.x * 256 + threadIdx.x;
    const long cnt = (long)rows * cols;
    if (e >= cnt) return;
    double2 acc = make_double2(0.0, 0.0);
    for (int sl = 0; sl < S; ++sl) acc = cadd(acc, part[sl * cnt + e]);
    double2* o = out + (e % rows) + (e / rows) * (long)ldo;
    *o = sub ? make_double2(o->x - acc.x, o->y - acc.y) : acc;
}

static hipError_t sum_parts(hipStream_t st, const double2* part, int S, int rows, int cols, double2* out, int ldo,
                            int sub)
{
    const long cnt = (long)rows * cols;
    hipLaunchKernelGGL(sum_parts_kernel, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, st, part, S, rows, cols,
                       out, ldo, sub);
    return hipGetLastError();
}

static hipError_t project_out(hipStream_t st, double2* Y, int ld, int n, int j0, int bw, double2* W, double2* part)
{
    double2* Yj = Y + (long)j0 * ld;
    const int PK_ROWS = pk_rows(n, j0), PK_COLS = pk_cols(n);
    const int S1 = n / PK_ROWS, r1 = n - S1 * PK_ROWS;
    hipError_t e = hipSuccess;
    if (S1 > 0)
        e = zgemm(st, 1, 0, j0, bw, PK_ROWS, 1.0, Y, ld, PK_ROWS, Yj, ld, PK_ROWS, 0.0, part, j0, (long)j0 * bw, S1);
    if (e == hipSuccess && r1 > 0)
        e = zgemm(st, 1, 0, j0, bw, r1, 1.0, Y + S1 * PK_ROWS, ld, 0, Yj + S1 * PK_ROWS, ld, 0, 0.0,
                  part + (long)S1 * j0 * bw, j0, 0, 1);
    if (e == hipSuccess) e = sum_parts(st, part, S1 + (r1 > 0), j0, bw, W, j0, 0);
    const int S2 = j0 / PK_COLS, r2 = j0 - S2 * PK_COLS;
    if (e == hipSuccess && S2 > 0)
        e = zgemm(st, 0, 0, n, bw, PK_COLS, 1.0, Y, ld, (long)PK_COLS * ld, W, j0, PK_COLS, 0.0, part, n,
                  (long)n * bw, S2);
    if (e == hipSuccess && r2 > 0)
        e = zgemm(st, 0, 0, n, bw, r2, 1.0, Y + (long)S2 * PK_COLS * ld, ld, 0, W + S2 * PK_COLS, j0, 0, 0.0,
                  part + (long)S2 * n * bw, n, 0, 1);
    if (e == hipSuccess) e = sum_parts(st, part, S2 + (r2 > 0), n, bw, Yj, ld, 1);
    return e;
}

// ----------------------------------------------------------------------------
// Orthonormalisation inside a wide block from its Gram matrix.  G = Yb^H Yb
// (bw x bw) is factored G = R^H R column by column; a column is dropped (R row
// and Rinv row and column zero) when its norm after the projections on the
// earlier blocks, sqrt(G_cc), or after the earlier columns of the block,
// sqrt(d_c) with d_c the Cholesky pivot, is at most thr * ref[c] (ref =
// nullptr: thr).  The pivot carries a relative rounding error of about
// n eps G_cc / d_c, so the factorisation stops at the first column whose pivot
// falls below tau * G_cc: flag[0] = that column (bw when none), and columns
// from there on are left to the next block, which sees them projected off
// the columns kept here (the scale that made the pivot small is gone then).
// The first column that is not dropped always has d_c = G_cc, so flag[0] > 0.
// Rinv = R^-1 on the kept columns before the cut, so Yb Rinv has orthonormal
// columns up to eps cond(Yb)^2 (a second pass brings that to eps).  flag[1] =
// number of kept columns before the cut.
//
// One workgroup, bound by the chain of a column's steps.  The elimination G = L D L^H runs
// on [G | I], so L^-1 (and with it Rinv = L^-H D^-1/2) comes out of the same steps:
// thread (ti, tj) keeps the entries (ti + 16 a, tj + 16 b) in registers, the upper
// triangle of G and below it L^-1, and step c publishes row c in one of two LDS buffers
// and subtracts conj(G_ci) / d times it from every row i > c, one barrier a column
// (72-115 us before, with three barriers a column, the triangle in LDS and Rinv by a
// substitution of one thread per column afterwards; 28-39 us now).
constexpr int QB = 64;        // columns per BCGS2 block
constexpr int CH_NT = 256;

__global__ __launch_bounds__(CH_NT) void block_chol_kernel(const double2* __restrict__ Gin, int bw,
                                                            const double* __restrict__ ref, double thr, double tau,
                                                            double2* __restrict__ Rinv, int* __restrict__ flag)
{
    static_assert(CH_NT == 256 && QB == 64, "a 16 x 16 grid of threads with 4 x 4 entries each");
    __shared__ double2 row[2][QB];
    __shared__ double gd[QB], lim2[QB], rd[QB];   // rd: 1 / sqrt(d) of a kept column, 0 otherwise
    const int tid = threadIdx.x, ti = tid >> 4, tj = tid & 15;
    double2 v[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = ti + 16 * a, j = tj + 16 * q;
            v[a][q] = (i <= j && j < bw) ? Gin[i + (long)j * bw] : make_double2(0.0, 0.0);
        }
    if (tid < bw) {
        gd[tid] = Gin[tid + (long)tid * bw].x;
        const double lim = thr * (ref ? ref[tid] : 1.0);
        lim2[tid] = lim * lim;
    }
    if (tid < QB) rd[tid] = 0.0;
    int cut = bw;
#pragma unroll
    for (int ca = 0; ca < 4; ++ca) {
#pragma unroll 1
        for (int ct = 0; ct < 16; ++ct) {
            const int c = 16 * ca + ct;
            if (c >= cut) break;   // uniform
            double2* w = row[c & 1];
            if (ti == ct) {
#pragma unroll
                for (int q = 0; q < 4; ++q) w[tj + 16 * q] = v[ca][q];
            }
            __syncthreads();
            // every thread takes the same decisions from the same values
            const double d = w[c].x, g = gd[c];
            if (!(g > lim2[c]) || !(d == d)) continue;   // dependent on the earlier blocks (or not finite)
            if (d < tau * g) { cut = c; break; }         // the pivot is not resolved: cut here
            if (d <= lim2[c]) continue;                  // dependent on the earlier columns of the block
            if (tid == 0) rd[c] = 1.0 / sqrt(d);
            const double di = 1.0 / d;
            double2 f[4], x[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const double2 t = w[ti + 16 * a];
                f[a] = make_double2(t.x * di, -t.y * di);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j = tj + 16 * q;
                x[q] = w[j];
                if (j == c) x[q] = make_double2(1.0, 0.0);   // the diagonal of L^-1
            }
#pragma unroll
            for (int a = ca; a < 4; ++a)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = ti + 16 * a, j = tj + 16 * q;
                    if (i > c && (j >= i || j <= c)) v[a][q] = cfms(v[a][q], f[a], x[q]);
                }
        }
        if (cut < 16 * (ca + 1)) break;
    }
    __syncthreads();
    // Rinv_kj = conj((L^-1)_jk) / sqrt(d_j)
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int j = ti + 16 * a, k = tj + 16 * q;
            if (j >= bw || k >= bw) continue;
            const double s = j < cut ? rd[j] : 0.0;
            double2 o = make_double2(0.0, 0.0);
            if (k < j && s != 0.0) o = make_double2(v[a][q].x * s, -v[a][q].y * s);
            if (k == j) o.x = s;
            Rinv[k + (long)j * bw] = o;
        }
    if (tid < 64) {
        const int kept = __popcll(__ballot(tid < cut && rd[tid] != 0.0));
        if (tid == 0) {
            flag[0] = cut;
            flag[1] = kept;
        }
    }
}

// G = Yb^H Yb for the bw columns of Yb, split along the rows like project_out.
static hipError_t gram_block(hipStream_t st, const double2* Yb, int ld, int n, int bw, double2* G, double2* part)
{
    const int PK_ROWS = pk_rows(n, bw);
    const int S1 = n / PK_ROWS, r1 = n - S1 * PK_ROWS;
    const long bb = (long)bw * bw;
    hipError_t e = hipSuccess;
    if (S1 > 0) e = zgemm(st, 1, 0, bw, bw, PK_ROWS, 1.0, Yb, ld, PK_ROWS, Yb, ld, PK_ROWS, 0.0, part, bw, bb, S1);
    if (e == hipSuccess && r1 > 0)
        e = zgemm(st, 1, 0, bw, bw, r1, 1.0, Yb + S1 * PK_ROWS, ld, 0, Yb + S1 * PK_ROWS, ld, 0, 0.0,
                  part + (long)S1 * bb, bw, 0, 1);
    if (e == hipSuccess) e = sum_parts(st, part, S1 + (r1 > 0), bw, bw, G, bw, 0);
    return e;
}

// Entries of the partial products: at most PK_TILES tiles of 64 columns (and a slice's rest) of
// W or of a Gram matrix, or the slices of Yj -= Y W.
static size_t bcgs2_part(int n, int m)
{
    const size_t cols = (size_t)((std::max(m, QB) + 63) / 64) * 64;
    const size_t p1 = std::min((size_t)(n / PK_MIN + 1) * cols, (size_t)(PK_TILES + 8) * 64 + 2 * cols) * QB;
    const size_t p2 = (size_t)(m / pk_cols(n) + 1) * n * QB;
    return std::max(p1, p2);
}

size_t bcgs2_work_bytes(int n, int m)
{
    const size_t w = (size_t)m * QB;
    return (w + bcgs2_part(n, m) + 2 * (size_t)QB * QB + (size_t)n * QB) * 16 + 512;
}

// Block classical Gram-Schmidt with reorthogonalisation (BCGS2) of Y (n x m,
// ld): each block of up to QB columns is projected off the finished blocks and
// orthonormalised inside the block from its Gram matrix, twice.  Columns found
// dependent (remaining norm <= 4 eps sqrt(n) times their original norm) come
// out as zero columns, so Q^H Q is the identity on the nonzero columns.  A
// block is cut where its Gram pivots stop being resolved in FP64 (columns of
// very different scale in one block), and the rest starts the next block.
// Once every column of a block is dependent, the range of Y is taken as
// captured and the remaining columns are set to zero: for Gaussian sketch
// columns the chance that a further column would still be independent is
// below 0.01^QB.
// work: bcgs2_work_bytes(n, m) bytes; n0: scratch of m doubles.
hipError_t bcgs2(hipStream_t st, double2* Y, int ld, int n, int m, void* work, double* n0)
{
    const double thr = 4.0 * 2.220446049250313e-16 * sqrt((double)n);
    const double tau = 1e-6;
    double2* W = (double2*)work;
    double2* part = W + (size_t)m * QB;
    double2* G = part + bcgs2_part(n, m);
    double2* Ri = G + (size_t)QB * QB;
    double2* T = Ri + (size_t)QB * QB;
    int* flag = (int*)(T + (size_t)n * QB);
    int hf[2] = {0, 0};
    hipError_t e = colnorms(st, n, m, Y, ld, 0, n0, 1);
    if (e != hipSuccess) return e;
    // column by column on columns [a, b) (two passes per CG_BW sub-block), for a block
    // the Gram route cannot finish; orig: the columns still carry their original scale
    auto exact = [&](int a, int b, bool orig) -> hipError_t {
        for (int s0 = a; s0 < b; s0 += CG_BW) {
            const int sbw = std::min(CG_BW, b - s0);
            for (int pass = 0; pass < 2; ++pass) {
                if (s0 > 0) {
                    hipError_t x = project_out(st, Y, ld, n, s0, sbw, W, part);
                    if (x != hipSuccess) return x;
                }
                hipLaunchKernelGGL(block_cgs2_kernel, dim3(1), dim3(CG_NT), 0, st, Y + (long)s0 * ld, ld, n, sbw,
                                   (pass == 0 && orig) ? n0 + s0 : (const double*)nullptr, thr);
                hipError_t x = hipGetLastError();
                if (x != hipSuccess) return x;
                if (s0 == 0) break;
            }
        }
        return hipSuccess;
    };
    for (int j0 = 0; j0 < m;) {
        int bw = std::min(QB, m - j0);
        double2* Yb = Y + (long)j0 * ld;
        for (int pass = 0; pass < 2; ++pass) {
            if (j0 > 0 && (e = project_out(st, Y, ld, n, j0, bw, W, part)) != hipSuccess) return e;
            if ((e = gram_block(st, Yb, ld, n, bw, G, part)) != hipSuccess) return e;
            hipLaunchKernelGGL(block_chol_kernel, dim3(1), dim3(CH_NT), 0, st, G, bw,
                               pass == 0 ? n0 + j0 : (const double*)nullptr, thr, tau, Ri, flag);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            if ((e = hipMemcpyAsync(hf, flag, sizeof(hf), hipMemcpyDeviceToHost, st)) != hipSuccess) return e;
            if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
            const int ldr = bw;
            if (hf[0] < 1 || (pass == 1 && hf[0] < bw)) {
                // not expected (see block_chol_kernel); finish these columns one by one
                if ((e = exact(j0, j0 + bw, pass == 0)) != hipSuccess) return e;
                break;
            }
            if (pass == 0) {
                if (hf[0] == bw && hf[1] == 0) return zero_c128(st, n, m - j0, Yb, ld, 0, 1);
                bw = hf[0];
            }
            if ((e = zgemm(st, 0, 0, n, bw, bw, 1.0, Yb, ld, 0, Ri, ldr, 0, 0.0, T, n, 0, 1)) != hipSuccess) return e;
            if ((e = copy_c128(st, n, bw, T, n, 0, Yb, ld, 0, 1)) != hipSuccess) return e;
        }
        j0 += bw;
    }
    return hipSuccess;
}

int jacobi_blocks(int p) { int nb = (p + JB_B - 1) / JB_B; return nb + (nb & 1); }

size_t jacobi_work_bytes(int m, int m_apply, int p)
{
    const size_t pairs = (size_t)jacobi_blocks(p) / 2;
    const size_t slices = (size_t)(std::max(m, 1) + JRG - 1) / JRG;
    (void)m_apply;
    return pairs * (slices + 1) * JB_W * JB_W * 16 + pairs * 4 + 256;
}

hipError_t jacobi_round(hipStream_t st, double2* A, int lda, int m, int m_apply, int p, int round, double tol,
                        double zthr2, double* offmax, void* work)
{
    const int nb = jacobi_blocks(p), pairs = nb / 2;
    const int gs = (std::max(m, 1) + JRG - 1) / JRG, as = (m_apply + JR - 1) / JR;
    double2* Gp = (double2*)work;
    hipLaunchKernelGGL(jacobi_gram_kernel, dim3(pairs, gs), dim3(JB_NT), 0, st, A, lda, m, p, nb, round, Gp);
    hipLaunchKernelGGL(jacobi_rotate_kernel, dim3(pairs, as), dim3(JB_NT), 0, st, A, lda, m_apply, p, nb, round, Gp,
                       gs, tol, zthr2, offmax);
    return hipGetLastError();
}

hipError_t gather_scale(hipStream_t st, const double2* A, int lda, int m, const int* order, const double* inv,
                        double2* Q, int ldq, int k)
{
    if (k <= 0) return hipSuccess;
    const long e = (long)m * k;
    hipLaunchKernelGGL(gather_scale_kernel, dim3((unsigned)((e + 255) / 256)), dim3(256), 0, st, A, lda, m, order, inv,
                       Q, ldq, k);
    return hipGetLastError();
}

}  // namespace rsrr
