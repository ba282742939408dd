// Batched complex GEMMs on the CDNA4 matrix cores.
//
// A complex product C += A*B is computed as real MFMA products by splitting
// the complex inner index k into two real indices k' = 2k + c (c = 0 real
// part, c = 1 imaginary part):
//     Re C(i,j) = sum_k' A'(i,k') Br'(k',j),   A'(i,2k+c) = c ? Im A : Re A,
//     Im C(i,j) = sum_k' A'(i,k') Bi'(k',j),   Br'(2k+c,j) = c ? -Im B : Re B,
//                                              Bi'(2k+c,j) = c ?  Re B : Im B.
// (4 real multiplies per complex multiply-add, the "4M" form.)  A' is the
// interleaved complex storage read one float per lane, so the operands come
// straight from the interleaved layout staged in LDS.  The MFMA operand
// slots are swapped (the MFMA "A" operand carries B' and its "B" operand
// carries A'), which makes the output lane index run along rows i: 32 (or 16)
// consecutive lanes then store one contiguous column segment of C.
#include "common.h"
#include "kernels.h"

namespace rsrr {

// ----------------------------------------------------------------------------
// complex FP32: v_mfma_f32_32x32x2f32.  The workgroup has WR x WC waves; each
// wave owns BR x BC blocks of 32x32 outputs, so the WG tile is
// (32 WR BR) x (32 WC BC).  In this 4M form it serves the 128x32 products of
// the panels; wider products go to the 3M kernel below.  The 4M
// kernel is kept general (a 128x128 tile of 2x2 waves of 2x2 blocks runs at
// two waves per SIMD).  beta*C is loaded into the accumulators before
// the k loop (its latency overlaps the first LDS stage), alpha is folded
// into the A operand, and the epilogue only stores.
// ----------------------------------------------------------------------------
constexpr int CG_KT = 16, CG_NT = 256;

// Tile t of a matrix -> (row tile, column tile): groups of TG_ROWS row tiles
// sweep the columns together, so the workgroups in flight on one XCD share a
// few row slices of A and column slices of B in its L2 instead of streaming
// all of A once per column of tiles.
constexpr int TG_ROWS = 8;
__device__ __forceinline__ void tile_order(int t, int tilesM, int tilesN, int* ti, int* tj)
{
    const int span = TG_ROWS * tilesN;
    const int g = t / span, first = g * TG_ROWS;
    const int rows = min(tilesM - first, TG_ROWS);
    const int in = t - g * span;
    *ti = first + in % rows;
    *tj = in / rows;
}

template <int WR, int WC, int BR, int BC, bool VEC, int TAG>
__global__ __launch_bounds__(CG_NT, 2) void cgemm_mfma_kernel(
    int M, int N, int K, float alpha,
    const float2* __restrict__ A, int lda, long sA,
    const float2* __restrict__ B, int ldb, long sB,
    float beta, float2* __restrict__ C, int ldc, long sC,
    int tilesM, int tilesN, int batch, long total_padded)
{
    constexpr int BM = 32 * WR * BR, BN = 32 * WC * BC;
    constexpr int AQ = BM * CG_KT / 2 / CG_NT;   // float4 (2 complex) A loads per thread per stage
    constexpr int BQ = BN * CG_KT / 2 / CG_NT;   // float4 B loads per thread per stage
    static_assert(AQ >= 1 && BQ >= 1, "tile too small for the loader");
    // B rows padded by 4 complex (32 B): the staging stores write 8 k-rows of one
    // column per wave, which then fall on different LDS banks
    __shared__ __attribute__((aligned(16))) float As[2][CG_KT][2 * BM];
    __shared__ __attribute__((aligned(16))) float2 Bs[2][CG_KT][BN + 4];

    const long tile = xcd_remap(blockIdx.x, total_padded);
    const long per = (long)tilesM * tilesN;
    const long b = tile / per;
    if (b >= batch) return;
    const int t = (int)(tile - b * per);
    int ti, tj;
    tile_order(t, tilesM, tilesN, &ti, &tj);
    const int i0 = ti * BM;
    const int j0 = tj * BN;
    const float2* Ab = A + b * sA;
    const float2* Bb = B + b * sB;
    float2* Cb = C + b * sC;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wi = wave % WR, wj = wave / WR;
    const int li = lane & 31, half = lane >> 5;
    const int wrow = i0 + wi * BR * 32, wcol = j0 + wj * BC * 32;

    // ---- prologue: acc = (beta / alpha) C, scaled by alpha once at the end (bitwise the same
    // for alpha = +-1); output layout: lane li = row, reg r = column 8(r/4)+4 half+r%4 ----
    const bool prod = alpha != 0.f;
    const float cs = prod ? beta / alpha : beta, os = prod ? alpha : 1.f;
    floatx16 accR[BR][BC], accI[BR][BC];
#pragma unroll
    for (int x = 0; x < BR; ++x)
#pragma unroll
        for (int y = 0; y < BC; ++y) {
            const int i = wrow + x * 32 + li;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int j = wcol + y * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                float2 c = make_float2(0.f, 0.f);
                if (beta != 0.f && i < M && j < N) c = Cb[i + (long)j * ldc];
                accR[x][y][r] = cs * c.x;
                accI[x][y][r] = cs * c.y;
            }
        }

    floatx4 ra[AQ], rb[BQ];
    auto gload = [&](int k0) {
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            const int p = tid + CG_NT * q;
            const int k = p / (BM / 2), ip = (p % (BM / 2)) * 2;
            const int gi = i0 + ip, gk = k0 + k;
            floatx4 v = {0.f, 0.f, 0.f, 0.f};
            if (gk < K) {
                const float2* src = Ab + gi + (long)gk * lda;
                if (VEC && gi + 1 < M) {
                    v = *reinterpret_cast<const floatx4*>(src);
                } else {
                    if (gi < M) { float2 e = src[0]; v[0] = e.x; v[1] = e.y; }
                    if (gi + 1 < M) { float2 e = src[1]; v[2] = e.x; v[3] = e.y; }
                }
            }
            ra[q] = v;
        }
#pragma unroll
        for (int q = 0; q < BQ; ++q) {
            const int p = tid + CG_NT * q;
            const int j = p / (CG_KT / 2), kp = (p % (CG_KT / 2)) * 2;
            const int gj = j0 + j, gk = k0 + kp;
            floatx4 v = {0.f, 0.f, 0.f, 0.f};
            if (gj < N) {
                const float2* src = Bb + gk + (long)gj * ldb;
                if (VEC && gk + 1 < K) {
                    v = *reinterpret_cast<const floatx4*>(src);
                } else {
                    if (gk < K) { float2 e = src[0]; v[0] = e.x; v[1] = e.y; }
                    if (gk + 1 < K) { float2 e = src[1]; v[2] = e.x; v[3] = e.y; }
                }
            }
            rb[q] = v;
        }
    };
    auto sstore = [&](int buf) {
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            const int p = tid + CG_NT * q;
            const int k = p / (BM / 2), ip = (p % (BM / 2)) * 2;
            *reinterpret_cast<floatx4*>(&As[buf][k][2 * ip]) = ra[q];
        }
#pragma unroll
        for (int q = 0; q < BQ; ++q) {
            const int p = tid + CG_NT * q;
            const int j = p / (CG_KT / 2), kp = (p % (CG_KT / 2)) * 2;
            Bs[buf][kp][j] = make_float2(rb[q][0], rb[q][1]);
            Bs[buf][kp + 1][j] = make_float2(rb[q][2], rb[q][3]);
        }
    };

    const int nst = prod ? (K + CG_KT - 1) / CG_KT : 0;
    if (nst > 0) {
        gload(0);
        sstore(0);
        __syncthreads();
    }
    for (int s = 0; s < nst; ++s) {
        const int buf = s & 1;
        if (s + 1 < nst) gload((s + 1) * CG_KT);
#pragma unroll 4
        for (int k = 0; k < CG_KT; ++k) {
            float a[BR], br[BC], bi[BC];
#pragma unroll
            for (int x = 0; x < BR; ++x) a[x] = As[buf][k][2 * (wi * BR * 32 + x * 32 + li) + half];
#pragma unroll
            for (int y = 0; y < BC; ++y) {
                const float2 bv = Bs[buf][k][wj * BC * 32 + y * 32 + li];
                br[y] = half ? -bv.y : bv.x;
                bi[y] = half ? bv.x : bv.y;
            }
#pragma unroll
            for (int x = 0; x < BR; ++x)
#pragma unroll
                for (int y = 0; y < BC; ++y) {
                    accR[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(br[y], a[x], accR[x][y], 0, 0, 0);
                    accI[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(bi[y], a[x], accI[x][y], 0, 0, 0);
                }
        }
        if (s + 1 < nst) sstore(buf ^ 1);
        __syncthreads();
    }

    // ---- epilogue: store ----
#pragma unroll
    for (int x = 0; x < BR; ++x) {
        const int i = wrow + x * 32 + li;
        if (i >= M) continue;
#pragma unroll
        for (int y = 0; y < BC; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int j = wcol + y * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                if (j < N) Cb[i + (long)j * ldc] = make_float2(os * accR[x][y][r], os * accI[x][y][r]);
            }
    }
}

// ----------------------------------------------------------------------------
// complex FP32, "3M" form (Gauss's three-product trick): with A = Ar + i Ai and
// B = Br + i Bi, the three real products T1 = Ar Br, T2 = Ai Bi and
// T3 = (Ar + Ai)(Br + Bi) give Re AB = T1 - T2 and Im AB = T3 - T1 - T2: 3
// real multiplies per complex multiply-add instead of 4.  Here the MFMA's
// inner index of 2 runs over two consecutive complex k (lanes 0-31: k, lanes
// 32-63: k + 1), so one stage of CG_KT complex k takes 3 * CG_KT / 2 MFMAs per
// 32x32 block against 2 * CG_KT for the 4M kernel.  Staging, tile order and
// output layout are those of the 4M kernel; the sums Ar + Ai and Br + Bi are
// formed in registers from the staged values.  beta C enters the
// accumulators as T1 = beta Re C, T2 = 0, T3 = beta (Re C + Im C).  The error
// is bounded normwise like that of the 4M form with a slightly larger
// constant (Higham, "Stability of a method for multiplying complex matrices
// with three real matrix multiplications", SIMAX 1992), which the FP64
// refinement downstream absorbs.  Three accumulator sets per block: with
// 2x2 blocks per wave that is one wave per SIMD, with two blocks two.  The
// workgroup has 64 WR WC threads.
// ----------------------------------------------------------------------------
template <int WR, int WC, int BR, int BC, bool VEC, int TAG>
__global__ __launch_bounds__(64 * WR * WC, (BR * BC <= 2) ? 512 / (64 * WR * WC) : 1) void cgemm3m_mfma_kernel(
    int M, int N, int K, float alpha,
    const float2* __restrict__ A, int lda, long sA,
    const float2* __restrict__ B, int ldb, long sB,
    float beta, float2* __restrict__ C, int ldc, long sC,
    int tilesM, int tilesN, int batch, long total_padded)
{
    constexpr int NT = 64 * WR * WC;
    constexpr int BM = 32 * WR * BR, BN = 32 * WC * BC;
    constexpr int AQ = BM * CG_KT / 2 / NT;
    constexpr int BQ = BN * CG_KT / 2 / NT;
    static_assert(AQ >= 1 && BQ >= 1, "tile too small for the loader");
    static_assert(CG_KT % 2 == 0, "stages hold pairs of k");
    __shared__ __attribute__((aligned(16))) float As[2][CG_KT][2 * BM];
    __shared__ __attribute__((aligned(16))) float2 Bs[2][CG_KT][BN + 4];

    const long tile = xcd_remap(blockIdx.x, total_padded);
    const long per = (long)tilesM * tilesN;
    const long b = tile / per;
    if (b >= batch) return;
    const int t = (int)(tile - b * per);
    int ti, tj;
    tile_order(t, tilesM, tilesN, &ti, &tj);
    const int i0 = ti * BM;
    const int j0 = tj * BN;
    const float2* Ab = A + b * sA;
    const float2* Bb = B + b * sB;
    float2* Cb = C + b * sC;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wi = wave % WR, wj = wave / WR;
    const int li = lane & 31, half = lane >> 5;
    const int wrow = i0 + wi * BR * 32, wcol = j0 + wj * BC * 32;

    // alpha leaves the inner loop: the accumulators hold (beta / alpha) C + A B and
    // are scaled by alpha once at the end (bitwise the same for alpha = +-1)
    const bool prod = alpha != 0.f;
    const float cs = prod ? beta / alpha : beta, os = prod ? alpha : 1.f;
    floatx16 t1[BR][BC], t2[BR][BC], t3[BR][BC];
#pragma unroll
    for (int x = 0; x < BR; ++x)
#pragma unroll
        for (int y = 0; y < BC; ++y) {
            const int i = wrow + x * 32 + li;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int j = wcol + y * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                float2 c = make_float2(0.f, 0.f);
                if (beta != 0.f && i < M && j < N) c = Cb[i + (long)j * ldc];
                t1[x][y][r] = cs * c.x;
                t2[x][y][r] = 0.f;
                t3[x][y][r] = cs * (c.x + c.y);
            }
        }

    floatx4 ra[AQ], rb[BQ];
    auto gload = [&](int k0) {
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            const int p = tid + NT * q;
            const int k = p / (BM / 2), ip = (p % (BM / 2)) * 2;
            const int gi = i0 + ip, gk = k0 + k;
            floatx4 v = {0.f, 0.f, 0.f, 0.f};
            if (gk < K) {
                const float2* src = Ab + gi + (long)gk * lda;
                if (VEC && gi + 1 < M) {
                    v = *reinterpret_cast<const floatx4*>(src);
                } else {
                    if (gi < M) { float2 e = src[0]; v[0] = e.x; v[1] = e.y; }
                    if (gi + 1 < M) { float2 e = src[1]; v[2] = e.x; v[3] = e.y; }
                }
            }
            ra[q] = v;
        }
#pragma unroll
        for (int q = 0; q < BQ; ++q) {
            const int p = tid + NT * q;
            const int j = p / (CG_KT / 2), kp = (p % (CG_KT / 2)) * 2;
            const int gj = j0 + j, gk = k0 + kp;
            floatx4 v = {0.f, 0.f, 0.f, 0.f};
            if (gj < N) {
                const float2* src = Bb + gk + (long)gj * ldb;
                if (VEC && gk + 1 < K) {
                    v = *reinterpret_cast<const floatx4*>(src);
                } else {
                    if (gk < K) { float2 e = src[0]; v[0] = e.x; v[1] = e.y; }
                    if (gk + 1 < K) { float2 e = src[1]; v[2] = e.x; v[3] = e.y; }
                }
            }
            rb[q] = v;
        }
    };
    auto sstore = [&](int buf) {
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            const int p = tid + NT * q;
            const int k = p / (BM / 2), ip = (p % (BM / 2)) * 2;
            *reinterpret_cast<floatx4*>(&As[buf][k][2 * ip]) = ra[q];
        }
#pragma unroll
        for (int q = 0; q < BQ; ++q) {
            const int p = tid + NT * q;
            const int j = p / (CG_KT / 2), kp = (p % (CG_KT / 2)) * 2;
            Bs[buf][kp][j] = make_float2(rb[q][0], rb[q][1]);
            Bs[buf][kp + 1][j] = make_float2(rb[q][2], rb[q][3]);
        }
    };

    const int nst = prod ? (K + CG_KT - 1) / CG_KT : 0;
    if (nst > 0) {
        gload(0);
        sstore(0);
        __syncthreads();
    }
    for (int s = 0; s < nst; ++s) {
        const int buf = s & 1;
        if (s + 1 < nst) gload((s + 1) * CG_KT);
#pragma unroll 2
        for (int kk = 0; kk < CG_KT; kk += 2) {
            const int k = kk + half;
            float ar[BR], ai[BR], as[BR], br[BC], bi[BC], bs[BC];
#pragma unroll
            for (int x = 0; x < BR; ++x) {
                const float2 av = *reinterpret_cast<const float2*>(&As[buf][k][2 * (wi * BR * 32 + x * 32 + li)]);
                ar[x] = av.x;
                ai[x] = av.y;
                as[x] = av.x + av.y;
            }
#pragma unroll
            for (int y = 0; y < BC; ++y) {
                const float2 bv = Bs[buf][k][wj * BC * 32 + y * 32 + li];
                br[y] = bv.x;
                bi[y] = bv.y;
                bs[y] = bv.x + bv.y;
            }
#pragma unroll
            for (int x = 0; x < BR; ++x)
#pragma unroll
                for (int y = 0; y < BC; ++y) {
                    t1[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(br[y], ar[x], t1[x][y], 0, 0, 0);
                    t2[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(bi[y], ai[x], t2[x][y], 0, 0, 0);
                    t3[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(bs[y], as[x], t3[x][y], 0, 0, 0);
                }
        }
        if (s + 1 < nst) sstore(buf ^ 1);
        __syncthreads();
    }

#pragma unroll
    for (int x = 0; x < BR; ++x) {
        const int i = wrow + x * 32 + li;
        if (i >= M) continue;
#pragma unroll
        for (int y = 0; y < BC; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int j = wcol + y * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                if (j < N)
                    Cb[i + (long)j * ldc] = make_float2(os * (t1[x][y][r] - t2[x][y][r]),
                                                        os * (t3[x][y][r] - t1[x][y][r] - t2[x][y][r]));
            }
    }
}

// ----------------------------------------------------------------------------
// complex FP32 with at most 16 output columns (the solves of narrow probe
// blocks and the lowest levels of the panel recursion): v_mfma_f32_16x16x4f32,
// whose inner index of 4 covers two complex k in the 4M split k' = 2k + c
// (lane group g = lane / 16: complex k = k0 + g / 2, part c = g % 2).  A
// 32-wide instruction would leave three quarters of its columns empty at
// N = 8; this one leaves at most half.  With the operands swapped as in the
// kernels above, lane l and register r of a 16x16 block hold row l % 16 and
// column 4 (l / 16) + r.  Four waves of BR 16x16 blocks stacked in rows: the
// workgroup tile is (64 BR) x 16.
// ----------------------------------------------------------------------------
template <int BR, bool VEC, int TAG>
__global__ __launch_bounds__(CG_NT) void cgemm_narrow_kernel(
    int M, int N, int K, float alpha,
    const float2* __restrict__ A, int lda, long sA,
    const float2* __restrict__ B, int ldb, long sB,
    float beta, float2* __restrict__ C, int ldc, long sC,
    int tilesM, int batch, long total_padded)
{
    constexpr int BM = 64 * BR, BN = 16;
    constexpr int AQ = BM * CG_KT / 2 / CG_NT;   // float4 (2 complex) A loads per thread per stage
    constexpr int BLD = BN * CG_KT / 2;          // float4 B loads per stage (fewer than the threads)
    static_assert(AQ >= 1 && AQ * 2 * CG_NT == BM * CG_KT, "A tile must split evenly over the threads");
    static_assert(BLD <= CG_NT, "one B load per thread at most");
    __shared__ __attribute__((aligned(16))) float As[2][CG_KT][2 * BM];
    __shared__ __attribute__((aligned(16))) float2 Bs[2][CG_KT][BN + 4];

    const long tile = xcd_remap(blockIdx.x, total_padded);
    const long b = tile / tilesM;
    if (b >= batch) return;
    const int i0 = (int)(tile - b * tilesM) * BM;
    const float2* Ab = A + b * sA;
    const float2* Bb = B + b * sB;
    float2* Cb = C + b * sC;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, g = lane >> 4;
    const int kc = g >> 1, part = g & 1;
    const int wrow = i0 + wave * BR * 16;

    const bool prod = alpha != 0.f;   // alpha applied once at the end, as in the kernels above
    const float cs = prod ? beta / alpha : beta, os = prod ? alpha : 1.f;
    floatx4 accR[BR], accI[BR];
#pragma unroll
    for (int x = 0; x < BR; ++x) {
        const int i = wrow + x * 16 + li;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = 4 * g + r;
            float2 c = make_float2(0.f, 0.f);
            if (beta != 0.f && i < M && j < N) c = Cb[i + (long)j * ldc];
            accR[x][r] = cs * c.x;
            accI[x][r] = cs * c.y;
        }
    }

    floatx4 ra[AQ], rb;
    auto gload = [&](int k0) {
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            const int p = tid + CG_NT * q;
            const int k = p / (BM / 2), ip = (p % (BM / 2)) * 2;
            const int gi = i0 + ip, gk = k0 + k;
            floatx4 v = {0.f, 0.f, 0.f, 0.f};
            if (gk < K) {
                const float2* src = Ab + gi + (long)gk * lda;
                if (VEC && gi + 1 < M) {
                    v = *reinterpret_cast<const floatx4*>(src);
                } else {
                    if (gi < M) { float2 e = src[0]; v[0] = e.x; v[1] = e.y; }
                    if (gi + 1 < M) { float2 e = src[1]; v[2] = e.x; v[3] = e.y; }
                }
            }
            ra[q] = v;
        }
        rb = floatx4{0.f, 0.f, 0.f, 0.f};
        if (tid < BLD) {
            const int j = tid / (CG_KT / 2), kp = (tid % (CG_KT / 2)) * 2;
            const int gk = k0 + kp;
            if (j < N) {
                const float2* src = Bb + gk + (long)j * ldb;
                if (VEC && gk + 1 < K) {
                    rb = *reinterpret_cast<const floatx4*>(src);
                } else {
                    if (gk < K) { float2 e = src[0]; rb[0] = e.x; rb[1] = e.y; }
                    if (gk + 1 < K) { float2 e = src[1]; rb[2] = e.x; rb[3] = e.y; }
                }
            }
        }
    };
    auto sstore = [&](int buf) {
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            const int p = tid + CG_NT * q;
            const int k = p / (BM / 2), ip = (p % (BM / 2)) * 2;
            *reinterpret_cast<floatx4*>(&As[buf][k][2 * ip]) = ra[q];
        }
        if (tid < BLD) {
            const int j = tid / (CG_KT / 2), kp = (tid % (CG_KT / 2)) * 2;
            Bs[buf][kp][j] = make_float2(rb[0], rb[1]);
            Bs[buf][kp + 1][j] = make_float2(rb[2], rb[3]);
        }
    };

    const int nst = prod ? (K + CG_KT - 1) / CG_KT : 0;
    if (nst > 0) {
        gload(0);
        sstore(0);
        __syncthreads();
    }
    for (int s = 0; s < nst; ++s) {
        const int buf = s & 1;
        if (s + 1 < nst) gload((s + 1) * CG_KT);
#pragma unroll 4
        for (int kk = 0; kk < CG_KT; kk += 2) {
            const int k = kk + kc;
            float a[BR];
#pragma unroll
            for (int x = 0; x < BR; ++x) a[x] = As[buf][k][2 * (wave * BR * 16 + x * 16 + li) + part];
            const float2 bv = Bs[buf][k][li];
            const float br = part ? -bv.y : bv.x;
            const float bi = part ? bv.x : bv.y;
#pragma unroll
            for (int x = 0; x < BR; ++x) {
                accR[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(br, a[x], accR[x], 0, 0, 0);
                accI[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(bi, a[x], accI[x], 0, 0, 0);
            }
        }
        if (s + 1 < nst) sstore(buf ^ 1);
        __syncthreads();
    }

#pragma unroll
    for (int x = 0; x < BR; ++x) {
        const int i = wrow + x * 16 + li;
        if (i >= M) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = 4 * g + r;
            if (j < N) Cb[i + (long)j * ldc] = make_float2(os * accR[x][r], os * accI[x][r]);
        }
    }
}

template <int WR, int WC, int BR, int BC, bool M3 = false>
static void cgemm_launch(hipStream_t st, int M, int N, int K, float alpha, const float2* A, int lda, long sA,
                         const float2* B, int ldb, long sB, float beta, float2* C, int ldc, long sC, int batch,
                         int tag, bool vec)
{
    constexpr int BM = 32 * WR * BR, BN = 32 * WC * BC;
    const int tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN;
    const long total = round_up_l((long)tm * tn * batch, 8);
#define CG_L(V, T)                                                                                                    \
    do {                                                                                                              \
        if constexpr (M3)                                                                                             \
            hipLaunchKernelGGL((cgemm3m_mfma_kernel<WR, WC, BR, BC, V, T>), dim3((unsigned)total), dim3(64 * WR * WC), \
                               0, st,                                                                                 \
                               M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, tm, tn, batch, total);       \
        else                                                                                                          \
            hipLaunchKernelGGL((cgemm_mfma_kernel<WR, WC, BR, BC, V, T>), dim3((unsigned)total), dim3(CG_NT), 0, st,   \
                               M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, tm, tn, batch, total);       \
    } while (0)
    if (vec) {
        if (tag == 1) CG_L(true, 1); else CG_L(true, 0);
    } else {
        if (tag == 1) CG_L(false, 1); else CG_L(false, 0);
    }
#undef CG_L
}

// Workgroup tile of the complex FP32 trailing update (tag 1), chosen per bucket
// by the ragged batch's autotuner and set around its launches (host thread).
namespace {
thread_local int g_update_tile = UPD_TILE_3M_128x64;
}
void set_update_tile(int t) { g_update_tile = (t >= 0 && t < UPD_TILE_COUNT) ? t : UPD_TILE_3M_128x64; }
int get_update_tile() { return g_update_tile; }
const char* update_tile_name(int t)
{
    switch (t) {
    case UPD_TILE_3M_64x64: return "3m_64x64_4waves";
    case UPD_TILE_4M_128x128: return "4m_128x128_4waves";
    case UPD_TILE_4M_64x64: return "4m_64x64_4waves";
    default: return "3m_128x64_4waves";
    }
}

hipError_t cgemm(hipStream_t st, int M, int N, int K, float alpha,
                 const float2* A, int lda, long sA, const float2* B, int ldb, long sB,
                 float beta, float2* C, int ldc, long sC, int batch, int tag)
{
    if (M <= 0 || N <= 0 || batch <= 0) return hipSuccess;
    const bool vec = ((((uintptr_t)A) | ((uintptr_t)B)) & 15) == 0 && (lda % 2 == 0) && (ldb % 2 == 0)
                     && (sA % 2 == 0) && (sB % 2 == 0);
    // 128x16 tiles of 16x16 blocks for at most 16 columns, 128x32 tiles in the
    // 4M form up to 32 columns (the narrow products of the panels and
    // of narrow probe blocks); 64x64 tiles in the 3M form up to 64 columns (the
    // solves at L = 64); 128x64 tiles in the 3M form for everything wider that the
    // split kernels do not take (small trailing updates, U12 products): with two 32x32 blocks per wave the three
    // accumulator sets still leave two waves per SIMD, which measured faster
    // than 128x128 tiles in either form.  The trailing update's tile can be
    // changed per bucket by the ragged batch's autotuner (set_update_tile).
    if (N <= 16) {
        constexpr int BR = 2, BM = 64 * BR;
        const int tm = (M + BM - 1) / BM;
        const long total = round_up_l((long)tm * batch, 8);
#define CN_L(V, T)                                                                                                 \
    hipLaunchKernelGGL((cgemm_narrow_kernel<BR, V, T>), dim3((unsigned)total), dim3(CG_NT), 0, st, M, N, K, alpha, \
                       A, lda, sA, B, ldb, sB, beta, C, ldc, sC, tm, batch, total)
        if (vec) {
            if (tag == 1) CN_L(true, 1); else CN_L(true, 0);
        } else {
            if (tag == 1) CN_L(false, 1); else CN_L(false, 0);
        }
#undef CN_L
    } else if (N <= 32) {
        cgemm_launch<4, 1, 1, 1>(st, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, tag, vec);
    } else if (tag == 0 && N <= 64) {
        // 33..64 columns (the solves' products at L = 64): 64 x 64 tiles in the 3M form give
        // twice the workgroups of 128 x 64 on these skinny products (solve phase 25.8 -> 21.9 ms
        // per headline step; 64 x 32 and 32 x 64 tiles of two waves, 128 x 32 of four: slower)
        cgemm_launch<2, 2, 1, 1, true>(st, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, tag, vec);
    } else if (tag == 1 && g_update_tile == UPD_TILE_3M_64x64) {
        cgemm_launch<2, 2, 1, 1, true>(st, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, tag, vec);
    } else if (tag == 1 && g_update_tile == UPD_TILE_4M_128x128) {
        cgemm_launch<2, 2, 2, 2>(st, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, tag, vec);
    } else if (tag == 1 && g_update_tile == UPD_TILE_4M_64x64) {
        cgemm_launch<2, 2, 1, 1>(st, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, tag, vec);
    } else {
        cgemm_launch<4, 1, 1, 2, true>(st, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, tag, vec);
    }
    return hipGetLastError();
}

// ----------------------------------------------------------------------------
// real FP32 (the LU of a real NEP at real points): v_mfma_f32_32x32x2f32 with
// the instruction's K = 2 over two consecutive k (lanes 0-31: k, lanes 32-63:
// k + 1).  Same wave/block shapes and output layout as the complex kernel.
// LDS rows are padded so that the staging stores and the two-row operand
// reads spread over the banks.
// ----------------------------------------------------------------------------
constexpr int SG_KT = 16;

template <int WR, int WC, int BR, int BC, bool VEC, int TAG>
__global__ __launch_bounds__(CG_NT, 2) void sgemm_mfma_kernel(
    int M, int N, int K, float alpha,
    const float* __restrict__ A, int lda, long sA,
    const float* __restrict__ B, int ldb, long sB,
    float beta, float* __restrict__ C, int ldc, long sC,
    int tilesM, int tilesN, int batch, long total_padded)
{
    constexpr int BM = 32 * WR * BR, BN = 32 * WC * BC;
    constexpr int AQ = BM * SG_KT / 4 / CG_NT;   // float4 (4 rows) A loads per thread per stage
    constexpr int BLD = BN * SG_KT / 4;            // float4 (4 k) B loads per stage
    constexpr int BQ = (BLD + CG_NT - 1) / CG_NT;  // ... per thread (the last round may be partial)
    static_assert(AQ >= 1 && AQ * 4 * CG_NT == BM * SG_KT, "A tile must split evenly over the threads");
    __shared__ __attribute__((aligned(16))) float As[2][SG_KT][BM + 32];
    __shared__ __attribute__((aligned(16))) float Bs[2][SG_KT][BN + 36];

    const long tile = xcd_remap(blockIdx.x, total_padded);
    const long per = (long)tilesM * tilesN;
    const long b = tile / per;
    if (b >= batch) return;
    const int t = (int)(tile - b * per);
    int ti, tj;
    tile_order(t, tilesM, tilesN, &ti, &tj);
    const int i0 = ti * BM;
    const int j0 = tj * BN;
    const float* Ab = A + b * sA;
    const float* Bb = B + b * sB;
    float* Cb = C + b * sC;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wi = wave % WR, wj = wave / WR;
    const int li = lane & 31, half = lane >> 5;
    const int wrow = i0 + wi * BR * 32, wcol = j0 + wj * BC * 32;

    floatx16 acc[BR][BC];
#pragma unroll
    for (int x = 0; x < BR; ++x)
#pragma unroll
        for (int y = 0; y < BC; ++y) {
            const int i = wrow + x * 32 + li;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int j = wcol + y * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                acc[x][y][r] = (beta != 0.f && i < M && j < N) ? beta * Cb[i + (long)j * ldc] : 0.f;
            }
        }

    floatx4 ra[AQ], rb[BQ];
    auto gload = [&](int k0) {
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            const int p = tid + CG_NT * q;
            const int k = p / (BM / 4), i4 = (p % (BM / 4)) * 4;
            const int gi = i0 + i4, gk = k0 + k;
            floatx4 v = {0.f, 0.f, 0.f, 0.f};
            if (gk < K) {
                const float* src = Ab + gi + (long)gk * lda;
                if (VEC && gi + 3 < M) {
                    v = *reinterpret_cast<const floatx4*>(src);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (gi + e < M) v[e] = src[e];
                }
            }
            ra[q] = v;
        }
#pragma unroll
        for (int q = 0; q < BQ; ++q) {
            const int p = tid + CG_NT * q;
            const int j = p / (SG_KT / 4), k4 = (p % (SG_KT / 4)) * 4;
            const int gj = j0 + j, gk = k0 + k4;
            floatx4 v = {0.f, 0.f, 0.f, 0.f};
            if (p < BLD && j < BN && gj < N) {
                const float* src = Bb + gk + (long)gj * ldb;
                if (VEC && gk + 3 < K) {
                    v = *reinterpret_cast<const floatx4*>(src);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (gk + e < K) v[e] = src[e];
                }
            }
            rb[q] = v;
        }
    };
    auto sstore = [&](int buf) {
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            const int p = tid + CG_NT * q;
            const int k = p / (BM / 4), i4 = (p % (BM / 4)) * 4;
            *reinterpret_cast<floatx4*>(&As[buf][k][i4]) = ra[q];
        }
#pragma unroll
        for (int q = 0; q < BQ; ++q) {
            const int p = tid + CG_NT * q;
            const int j = p / (SG_KT / 4), k4 = (p % (SG_KT / 4)) * 4;
            if (p < BLD) {
#pragma unroll
                for (int e = 0; e < 4; ++e) Bs[buf][k4 + e][j] = rb[q][e];
            }
        }
    };

    const int nst = (K + SG_KT - 1) / SG_KT;
    if (nst > 0) {
        gload(0);
        sstore(0);
        __syncthreads();
    }
    for (int s = 0; s < nst; ++s) {
        const int buf = s & 1;
        if (s + 1 < nst) gload((s + 1) * SG_KT);
#pragma unroll 4
        for (int kp = 0; kp < SG_KT / 2; ++kp) {
            const int k = 2 * kp + half;
            float a[BR], bb[BC];
#pragma unroll
            for (int x = 0; x < BR; ++x) a[x] = alpha * As[buf][k][wi * BR * 32 + x * 32 + li];
#pragma unroll
            for (int y = 0; y < BC; ++y) bb[y] = Bs[buf][k][wj * BC * 32 + y * 32 + li];
#pragma unroll
            for (int x = 0; x < BR; ++x)
#pragma unroll
                for (int y = 0; y < BC; ++y)
                    acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(bb[y], a[x], acc[x][y], 0, 0, 0);
        }
        if (s + 1 < nst) sstore(buf ^ 1);
        __syncthreads();
    }

#pragma unroll
    for (int x = 0; x < BR; ++x) {
        const int i = wrow + x * 32 + li;
        if (i >= M) continue;
#pragma unroll
        for (int y = 0; y < BC; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int j = wcol + y * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                if (j < N) Cb[i + (long)j * ldc] = acc[x][y][r];
            }
    }
}

template <int WR, int WC, int BR, int BC>
static void sgemm_launch(hipStream_t st, int M, int N, int K, float alpha, const float* A, int lda, long sA,
                         const float* B, int ldb, long sB, float beta, float* C, int ldc, long sC, int batch, int tag,
                         bool vec)
{
    constexpr int BM = 32 * WR * BR, BN = 32 * WC * BC;
    const int tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN;
    const long total = round_up_l((long)tm * tn * batch, 8);
#define SG_L(V, T)                                                                                                    \
    hipLaunchKernelGGL((sgemm_mfma_kernel<WR, WC, BR, BC, V, T>), dim3((unsigned)total), dim3(CG_NT), 0, st, M, N, K, \
                       alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, tm, tn, batch, total)
    if (vec) {
        if (tag == 1) SG_L(true, 1); else SG_L(true, 0);
    } else {
        if (tag == 1) SG_L(false, 1); else SG_L(false, 0);
    }
#undef SG_L
}

hipError_t sgemm(hipStream_t st, int M, int N, int K, float alpha, const float* A, int lda, long sA,
                 const float* B, int ldb, long sB, float beta, float* C, int ldc, long sC, int batch, int tag)
{
    if (M <= 0 || N <= 0 || batch <= 0) return hipSuccess;
    const bool vec = ((((uintptr_t)A) | ((uintptr_t)B)) & 15) == 0 && (lda % 4 == 0) && (ldb % 4 == 0) &&
                     (sA % 4 == 0) && (sB % 4 == 0);
    if (N <= 32)
        sgemm_launch<4, 1, 1, 1>(st, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, tag, vec);
    else if (N <= 64)
        sgemm_launch<4, 1, 1, 2>(st, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, tag, vec);
    else
        sgemm_launch<2, 2, 2, 2>(st, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, tag, vec);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------
// complex FP64: v_mfma_f64_16x16x4f64, four waves, op(A) = A or A^H, op(B) = B or B^H.
//
// Bound by the FP64 matrix cores (64 cycles an instruction), so the rest of a stage has to
// stay out of their way: the instruction's inner index runs over four complex k, with
// separate instructions for the real and imaginary parts of A (a lane uses the whole
// complex entry that it reads from LDS: 6 reads for 32 instructions on the 128 x 64 tile;
// an interleaved inner index, which uses half of each entry, needs 4 reads and 12 selects
// for 8), and the stages are copied straight from memory into LDS, two ahead.
// LDS holds an operand that is contiguous along its rows as [k][row] and one that is
// contiguous along k as [row][k] with the k of row i rotated by i / 2, so that the 16
// rows of a fragment fall on different banks; the rotation is in the addresses that the
// lanes load from.  4096 x 64 x 4096, 32 matrices: 4.86 -> 4.44 ms (62 TFLOP/s); 2500 x
// 300 x 2500, 30 matrices: 8.4 -> 7.8 ms; its Hermitian product 300 x 300 x 2500: 1.72 -> 1.17
// ms; without the copies of the next stages the first would take 3.8 ms.
// ----------------------------------------------------------------------------
constexpr int ZG_BN = 64, ZG_KT = 8, ZG_NT = 256, ZG_BUF = 3;

// One operand's stage (ROWS x ZG_KT).  KC: contiguous along k (element (i, k) at p[k + i ld]),
// otherwise along the rows (p[i + k ld]).
template <bool KC, int ROWS> struct ZgStage {
    static constexpr int PER = ROWS * ZG_KT / ZG_NT;
    // row and k of the element that LDS slot e holds
    static RSRR_DEV void at(int e, int& i, int& k)
    {
        if (KC) { i = e / ZG_KT; k = (e % ZG_KT - (i >> 1)) & (ZG_KT - 1); }
        else { i = e % ROWS; k = e / ROWS; }
    }
    static RSRR_DEV int slot(int i, int k) { return KC ? i * ZG_KT + ((k + (i >> 1)) & (ZG_KT - 1)) : k * ROWS + i; }
    static RSRR_DEV long offset(int i, int k, int ld) { return KC ? k + (long)i * ld : i + (long)k * ld; }
};

template <bool CA, bool CB, int BM, int TAG>
__global__ __launch_bounds__(ZG_NT, 2) void zgemm_mfma_kernel(
    int M, int N, int K, double alpha,
    const double2* __restrict__ A, int lda, long sA,
    const double2* __restrict__ B, int ldb, long sB,
    double beta, double2* __restrict__ C, int ldc, long sC,
    int tilesM, int tilesN, int batch, long total_padded, int direct)
{
    constexpr int WR = BM / 32, WC = 4 / WR;          // waves along the rows and columns
    constexpr int XB = 2, YB = ZG_BN / WC / 16;       // 16 x 16 blocks of a wave
    typedef ZgStage<CA, BM> SA;
    typedef ZgStage<!CB, ZG_BN> SB;
    __shared__ __attribute__((aligned(16))) double2 As[ZG_BUF][BM * ZG_KT];
    __shared__ __attribute__((aligned(16))) double2 Bs[ZG_BUF][ZG_BN * ZG_KT];

    const long tile = xcd_remap(blockIdx.x, total_padded);
    const long per = (long)tilesM * tilesN;
    const long b = tile / per;
    if (b >= batch) return;
    const int t = (int)(tile - b * per);
    int ti, tj;
    tile_order(t, tilesM, tilesN, &ti, &tj);
    const int i0 = ti * BM;
    const int j0 = tj * ZG_BN;
    const double2* Ab = A + b * sA;
    const double2* Bb = B + b * sB;
    double2* Cb = C + b * sC;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wi = wave % WR, wj = wave / WR;
    const int li = lane & 15, kq = lane >> 4;
    const int r0 = wi * 32, c0 = wj * 16 * YB;

    // acc = (beta / alpha) C, scaled by alpha once at the end (bitwise the same for
    // alpha = +-1); lane li holds row i, register r holds column lane/16 + 4*r
    // (the f64 MFMA interleaves its four output groups by register)
    const bool prod = alpha != 0.0;
    const double cs = prod ? beta / alpha : beta, os = prod ? alpha : 1.0;
    doublex4 accR[XB][YB], accI[XB][YB];
#pragma unroll
    for (int x = 0; x < XB; ++x)
#pragma unroll
        for (int y = 0; y < YB; ++y) {
            const int i = i0 + r0 + x * 16 + li;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = j0 + c0 + y * 16 + kq + 4 * r;
                double2 c = make_double2(0.0, 0.0);
                if (beta != 0.0 && i < M && j < N) c = Cb[i + (long)j * ldc];
                accR[x][y][r] = cs * c.x;
                accI[x][y][r] = cs * c.y;
            }
        }

    // stage s into LDS buffer buf.  Whole stages of 16-byte aligned operands are copied directly
    // (rows past the end: the last row again, their results are not stored); the last, partial
    // one passes through registers, zero past K.
    auto load = [&](int s, int buf) {
        const int k0 = s * ZG_KT;
        if (direct && k0 + ZG_KT <= K) {
#pragma unroll
            for (int q = 0; q < SA::PER; ++q) {
                int i, k;
                SA::at(q * ZG_NT + tid, i, k);
                const double2* g = Ab + SA::offset(min(i0 + i, M - 1), k0 + k, lda);
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                                 (__attribute__((address_space(3))) void*)&As[buf][q * ZG_NT + wave * 64],
                                                 16, 0, 0);
            }
#pragma unroll
            for (int q = 0; q < SB::PER; ++q) {
                int j, k;
                SB::at(q * ZG_NT + tid, j, k);
                const double2* g = Bb + SB::offset(min(j0 + j, N - 1), k0 + k, ldb);
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                                 (__attribute__((address_space(3))) void*)&Bs[buf][q * ZG_NT + wave * 64],
                                                 16, 0, 0);
            }
        } else {
#pragma unroll
            for (int q = 0; q < SA::PER; ++q) {
                int i, k;
                SA::at(q * ZG_NT + tid, i, k);
                As[buf][q * ZG_NT + tid] = (i0 + i < M && k0 + k < K) ? Ab[SA::offset(i0 + i, k0 + k, lda)]
                                                                      : make_double2(0.0, 0.0);
            }
#pragma unroll
            for (int q = 0; q < SB::PER; ++q) {
                int j, k;
                SB::at(q * ZG_NT + tid, j, k);
                Bs[buf][q * ZG_NT + tid] = (j0 + j < N && k0 + k < K) ? Bb[SB::offset(j0 + j, k0 + k, ldb)]
                                                                      : make_double2(0.0, 0.0);
            }
        }
    };
    // Stage s is complete and visible to every wave, while the copies of stage s + 1 (the last
    // ones issued) may still be in flight.  Every wave has also finished with stage s - 1.
    auto arrived = [&](int s) {
        constexpr int INFLIGHT = SA::PER + SB::PER;
        static_assert(INFLIGHT < 16, "the count's low four bits");
        if (direct && (s + 2) * ZG_KT <= K) __builtin_amdgcn_s_waitcnt(INFLIGHT | 7 << 4);   // vmcnt, lgkmcnt 0
        else __builtin_amdgcn_s_waitcnt(7 << 4);
        asm volatile("s_barrier" ::: "memory");
    };

    const int nst = prod ? (K + ZG_KT - 1) / ZG_KT : 0;
    if (nst > 0) load(0, 0);
    if (nst > 1) load(1, 1);
    int buf = 0;
    for (int s = 0; s < nst; ++s) {
        arrived(s);
        if (s + 2 < nst) load(s + 2, buf == 0 ? 2 : buf - 1);
#pragma unroll
        for (int kg = 0; kg < ZG_KT / 4; ++kg) {
            const int k = kg * 4 + kq;
            double2 a[XB], bv[YB];
#pragma unroll
            for (int x = 0; x < XB; ++x) a[x] = As[buf][SA::slot(r0 + x * 16 + li, k)];
#pragma unroll
            for (int y = 0; y < YB; ++y) bv[y] = Bs[buf][SB::slot(c0 + y * 16 + li, k)];
            // conjugated operands: the sign of their imaginary parts
#pragma unroll
            for (int x = 0; x < XB; ++x) if (CA) a[x].y = -a[x].y;
#pragma unroll
            for (int y = 0; y < YB; ++y) if (CB) bv[y].y = -bv[y].y;
#pragma unroll
            for (int x = 0; x < XB; ++x)
#pragma unroll
                for (int y = 0; y < YB; ++y) {
                    accR[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(bv[y].x, a[x].x, accR[x][y], 0, 0, 0);
                    accI[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(bv[y].y, a[x].x, accI[x][y], 0, 0, 0);
                }
#pragma unroll
            for (int x = 0; x < XB; ++x)
#pragma unroll
                for (int y = 0; y < YB; ++y) {
                    accR[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(-bv[y].y, a[x].y, accR[x][y], 0, 0, 0);
                    accI[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(bv[y].x, a[x].y, accI[x][y], 0, 0, 0);
                }
        }
        buf = buf == 2 ? 0 : buf + 1;
    }

    // epilogue: store
#pragma unroll
    for (int x = 0; x < XB; ++x) {
        const int i = i0 + r0 + x * 16 + li;
        if (i >= M) continue;
#pragma unroll
        for (int y = 0; y < YB; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = j0 + c0 + y * 16 + kq + 4 * r;
                if (j < N) Cb[i + (long)j * ldc] = make_double2(os * accR[x][y][r], os * accI[x][y][r]);
            }
    }
}

template <int BM>
static hipError_t zgemm_launch(hipStream_t st, int opA, int opB, int M, int N, int K, double alpha, const double2* A,
                               int lda, long sA, const double2* B, int ldb, long sB, double beta, double2* C, int ldc,
                               long sC, int batch, int tag)
{
    const int tm = (M + BM - 1) / BM, tn = (N + ZG_BN - 1) / ZG_BN;
    const long total = round_up_l((long)tm * tn * batch, 8);
    const int direct = ((((uintptr_t)A) | ((uintptr_t)B)) & 15) == 0;
    dim3 g((unsigned)total), blk(ZG_NT);
#define ZG_LAUNCH(CA, CB, T)                                                                                   \
    hipLaunchKernelGGL((zgemm_mfma_kernel<CA, CB, BM, T>), g, blk, 0, st, M, N, K, alpha, A, lda, sA, B, ldb, sB, \
                       beta, C, ldc, sC, tm, tn, batch, total, direct)
    if (tag == 1 && !opA && !opB) ZG_LAUNCH(false, false, 1);
    else if (!opA && !opB) ZG_LAUNCH(false, false, 0);
    else if (opA && !opB) ZG_LAUNCH(true, false, 0);
    else if (!opA && opB) ZG_LAUNCH(false, true, 0);
    else ZG_LAUNCH(true, true, 0);
#undef ZG_LAUNCH
    return hipGetLastError();
}

hipError_t zgemm(hipStream_t st, int opA, int opB, int M, int N, int K, double alpha,
                 const double2* A, int lda, long sA, const double2* B, int ldb, long sB,
                 double beta, double2* C, int ldc, long sC, int batch, int tag)
{
    if (M <= 0 || N <= 0 || batch <= 0) return hipSuccess;
    // 128 x 64 tiles where there are two for every CU and the rows they pad cost less than the
    // 8% that they gain over 64 x 64; smaller products keep twice as many workgroups with 64 x 64
    // (projection of 541 / 900 rows, 298 columns: 949 / 1986 us with 128 x 64, 841 / 1695 with 64 x 64;
    // 2400 rows, equal padding, 9.05 ms against 9.67 with 64 x 64 before the larger tile)
    const long t128 = (M + 127) / 128, t64 = (M + 63) / 64;
    const long big = t128 * ((N + ZG_BN - 1) / ZG_BN) * batch;
    if (big >= 512 && 2 * t128 * 20 <= t64 * 21)
        return zgemm_launch<128>(st, opA, opB, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, tag);
    return zgemm_launch<64>(st, opA, opB, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch, tag);
}

}  // namespace rsrr
