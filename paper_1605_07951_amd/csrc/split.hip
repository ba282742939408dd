// FP32 products C -= A B and C = A B on the FP16 matrix cores with split operands (the LU's trailing
// updates, complex and real, and in complex FP32 the wide solves and the preconditioner of the iterative
// sampling).
//
// v_mfma_f32_32x32x16_f16 multiplies at 16 times the rate of the FP32 instruction, with exact products and
// FP32 sums.  Every real FP32 value, scaled by a power of two, is held as hi + lo of two FP16 numbers (the
// splitting of Markidis et al. 2018 and Ootomo and Yokota 2022): hi carries the leading 11 bits, lo the
// next 11 and a sign, so hi + lo is the value to within one unit of FP32 (exactly for three quarters of the
// values).  Three products, hi hi + hi lo + lo hi, are accumulated; lo lo is below 2^-22 of the product.
// The sums do not contain C (one subtraction at the end), and 16 products enter them per rounding instead
// of 2.
//
// The range is that of FP16, so every row of A and every column of B has its own power of two, to a largest
// part in [2^14, 2^15) (depths of at most 256; a deeper product is a sum of slabs with scales of their
// own).  An entry keeps its 22 bits down to 2^-17 of the largest of its row or column, then loses a bit per
// factor of two, and below 2^-40 it is lost: beyond the error of the 22 bits a product is off by up to
// 2^-40 max_k |A_ik| max_k |B_kj|.  Columns of T of different size are in the powers of B's columns.  Rows
// of different size are not: they reach the factors as L_ik ~ d_i / d_k and U_kj ~ d_k, small entries of a
// row of L against large ones of a column of U; so the factorisation takes such a T with its rows brought
// to one size first (lu.hip), and |L| <= 1 then meets rows of U of T's size.  In the solves' backward sweep
// the inner index runs over T's columns; there it takes a power of two of its own (split_columns).
//
// Error against 64 bits, relative to |A||B| and in units of u = 2^-24, K = 128 and 256, split / FP32
// kernels: complex, one size or rows and columns spread over 16 decades: rms 0.32-0.34 / 0.51-0.53, largest
// 1.8-2.5 / 3.1-4.9; the entries of A spread over 3 decades 0.6 / 0.95; both operands' over 3 decades 1.1 /
// 1.6-1.7, over 8 decades 1.7-1.9 / 2.3-2.6, largest 12 / 24.  Real: 0.28-0.31 / 0.43; 0.53-0.56 / 0.78;
// 0.95 / 1.3; 1.5-1.7 / 1.7-2.0.
//
// Bound by the matrix cores and by C, which is read and written once per update.  64 matrices, K = 256, n =
// 3840 / 2048 / 1024: 6.0-6.6 / 1.7-1.8 / 0.44 ms, 292-325 / 301-335 / 311-318 TFLOP/s in the standard
// count of 8 flops per complex multiply-add (up to 975 TFLOP/s in FP16, C at 2.6 TB/s), packing 0.36 / 0.20
// / 0.11 ms; the FP32 3M kernel 13.8 / 4.5 / 1.1 ms.
//
// Real: K = 256, 64 matrices, n = 1768 / 1024 / 512 / 256: 0.54 / 0.17 / 0.045 / 0.018 ms and 0.12 / 0.07 /
// 0.04 / 0.026 ms for the packing, the FP32 kernel 1.48 / 0.52 / 0.14 / 0.045.
//
// The complex product is the 4M form with the interleaved parts as the inner index
// (k' = 2k + part): Re C takes A' (Br, -Bi), Im C takes A' (Bi, Br), which is one sign
// flip and one half-word rotation of the same registers.
//
// The operands are packed once per update into the order in which the instruction
// takes them (a fragment: 32 rows x 8 complex k, 64 lanes x 16 bytes, 1 KB), so a tile is
// staged with plain 16-byte global-to-LDS copies and read back without bank conflicts.
#include "common.h"
#include "kernels.h"

namespace rsrr {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));

constexpr int SP_KC = 8;          // complex k per fragment
constexpr int SP_FRAG = 1024;     // bytes
constexpr int SP_TOP = 14;        // exponent that a row's or column's largest part is scaled to
constexpr int SP_KMAX = 256;

// hi and lo parts of 4 complex values scaled by 2^(e + k), interleaved (re, im) as one lane of a fragment
RSRR_DEV void split4(const float2 (&v)[4], int e, const int2 (&k)[4], uintx4* hi, uintx4* lo)
{
    half8 h, l;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float x = ldexpf(v[q].x, e + k[q].x), y = ldexpf(v[q].y, e + k[q].y);
        h[2 * q] = (_Float16)x;
        h[2 * q + 1] = (_Float16)y;
        l[2 * q] = (_Float16)(x - (float)h[2 * q]);
        l[2 * q + 1] = (_Float16)(y - (float)h[2 * q + 1]);
    }
    *hi = __builtin_bit_cast(uintx4, h);
    *lo = __builtin_bit_cast(uintx4, l);
}
RSRR_DEV void split4(const float2 (&v)[4], int e, uintx4* hi, uintx4* lo)
{
    const int2 none[4] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
    split4(v, e, none, hi, lo);
}

// Exponent that scales a largest part to [2^SP_TOP, 2^(SP_TOP + 1)); zero or non-finite: no scale.
RSRR_DEV int split_expo(float top)
{
    // v_frexp_exp: top = m 2^e with m in [1/2, 1)
    return (top > 0.f && isfinite(top)) ? SP_TOP + 1 - __builtin_amdgcn_frexp_expf(top) : 0;
}

// Exponent of v's larger part times 2^k (v_frexp_exp: x = m 2^e with m in [1/2, 1); 0 for infinities
// and NaN); zero: SP_NONE.
constexpr int SP_NONE = -(1 << 20);
RSRR_DEV int part_expo(float x, int k) { return x != 0.f ? __builtin_amdgcn_frexp_expf(x) + k : SP_NONE; }
RSRR_DEV int part_expo(float2 v, int2 k) { return max(part_expo(v.x, k.x), part_expo(v.y, k.y)); }
// Exponent that scales a largest part with exponent `top` to [2^SP_TOP, 2^(SP_TOP + 1)); zero: no scale.
RSRR_DEV int split_expo(int top) { return top != SP_NONE ? SP_TOP + 1 - top : 0; }

// Bytes of the fragments of an operand of `rows` rows (A) or columns (B); its exponents follow.
// Real operands: two consecutive k in place of the parts of one, 16 k per fragment.
template <typename C>
static __host__ __device__ constexpr int sp_chunks(int K)
{
    return sizeof(C) == sizeof(float2) ? (K + SP_KC - 1) / SP_KC : (K + 2 * SP_KC - 1) / (2 * SP_KC);
}
template <typename C>
static __host__ __device__ long sp_frag_bytes(int rows, int K)
{
    return (long)((rows + 31) / 32) * sp_chunks<C>(K) * 2 * SP_FRAG;
}
// entry k of a row or column with K entries ld apart (real: entries 2 k and 2 k + 1), zero past the end
RSRR_DEV float2 sp_entry(const float2* src, int k, long ld, int K)
{
    return k < K ? src[k * ld] : make_float2(0.f, 0.f);
}
RSRR_DEV float2 sp_entry(const float* src, int k, long ld, int K)
{
    return make_float2(2 * k < K ? src[2 * k * ld] : 0.f, 2 * k + 1 < K ? src[(2 * k + 1) * ld] : 0.f);
}

// the inner index's exponents (LDS, 16-byte aligned) of the parts of entries 4 p .. 4 p + 3
template <typename C>
RSRR_DEV void sp_inner(const int* inner, int p, int2 (&k)[4])
{
    const int4* e = reinterpret_cast<const int4*>(inner) + (sizeof(C) == sizeof(float2) ? p : 2 * p);
    const int4 x = e[0];
    if (sizeof(C) == sizeof(float2)) {
        k[0] = make_int2(x.x, x.x);
        k[1] = make_int2(x.y, x.y);
        k[2] = make_int2(x.z, x.z);
        k[3] = make_int2(x.w, x.w);
    } else {
        const int4 y = e[1];
        k[0] = make_int2(x.x, x.y);
        k[1] = make_int2(x.z, x.w);
        k[2] = make_int2(y.x, y.y);
        k[3] = make_int2(y.z, y.w);
    }
}

// E[k] scales column k of U (k of the n x n factors) to a largest part in [1/2, 1) (zero or non-finite: 0), for
// the products of the solves' backward sweep: their inner index runs over T's columns, whose sizes the rows of
// U and the solution carry inversely to each other.  One workgroup per column, one launch before the sweep.
__global__ __launch_bounds__(256) void split_columns_kernel(const float2* __restrict__ LU, int ld, long sLU,
                                                            int* __restrict__ E, long sE)
{
    const int k = blockIdx.x, b = blockIdx.y, t = threadIdx.x;
    const float2* col = LU + b * sLU + (long)k * ld;
    __shared__ float tops[4];
    float top = 0.f;
#pragma unroll 4
    for (int i = t; i <= k; i += 256) top = fmaxf(top, fmaxf(fabsf(col[i].x), fabsf(col[i].y)));
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) top = fmaxf(top, __shfl_xor(top, off));
    if ((t & 63) == 0) tops[t >> 6] = top;
    __syncthreads();
    if (t == 0) {
        top = fmaxf(fmaxf(tops[0], tops[1]), fmaxf(tops[2], tops[3]));
        E[b * sE + k] = (top > 0.f && isfinite(top)) ? -__builtin_amdgcn_frexp_expf(top) : 0;
    }
}

// INNER: with exponents of the inner index (E).
//
// A (M x K, K <= SP_KMAX): fragment (row block, k chunk, hi/lo) at ((rb * nkc + kc) * 2 + h) KB; lane l
// holds row l % 32 and the 4 complex k at 4 (l / 32); then the exponent of each row's scale.  One
// workgroup per 32 rows, thread (row t % 32, groups of 4 columns t / 32 + 8 q); rows past M are zero.
// Of a deeper product, slab b holds the columns b kstep .. (past Ktot: zero).
template <typename C, bool INNER>
__global__ __launch_bounds__(256) void split_pack_a_kernel(int M, int K, int Ktot, int kstep,
                                                           const C* __restrict__ A, int lda, long sA,
                                                           const int* __restrict__ E, long sE,
                                                           char* __restrict__ P, long sP)
{
    const int rb = blockIdx.x, b = blockIdx.y, t = threadIdx.x;
    const int nkc = sp_chunks<C>(K), Kb = min(K, Ktot - b * kstep);
    const int r = t & 31, part = t >> 5, i = rb * 32 + r;
    __shared__ int tops[8][32];
    __shared__ __attribute__((aligned(16))) int inner[INNER ? SP_KMAX : 4];
    const int ei = INNER && t < Kb ? E[b * sE + t] : 0;
    const C* src = A + b * sA + i;
    constexpr int Q = sp_chunks<C>(SP_KMAX) / 4;
    float2 v[Q][4];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int u = 0; u < 4; ++u)
            v[q][u] = i < M ? sp_entry(src, 4 * (part + 8 * q) + u, lda, Kb) : make_float2(0.f, 0.f);
    if constexpr (INNER) {
        inner[t] = ei;
        __syncthreads();
    }
    int top = SP_NONE;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        int2 ek[4] = {};
        if constexpr (INNER) sp_inner<C>(inner, part + 8 * q, ek);
#pragma unroll
        for (int u = 0; u < 4; ++u) top = max(top, part_expo(v[q][u], ek[u]));
    }
    tops[part][r] = top;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) top = max(top, tops[q][r]);
    const int e = split_expo(top);
    char* Pb = P + b * sP;
    if (part == 0) reinterpret_cast<int*>(Pb + sp_frag_bytes<C>(M, K))[i] = e;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int p = part + 8 * q, kc = p >> 1;
        if (kc >= nkc) break;
        uintx4 hi, lo;
        int2 ek[4] = {};
        if constexpr (INNER) sp_inner<C>(inner, p, ek);
        split4(v[q], e, ek, &hi, &lo);
        uintx4* dst = reinterpret_cast<uintx4*>(Pb + ((long)rb * nkc + kc) * 2 * SP_FRAG);
        dst[r + 32 * (p & 1)] = hi;
        dst[64 + r + 32 * (p & 1)] = lo;
    }
}

// B (K x N, K <= SP_KMAX): the same fragments with the columns in place of the rows, and the
// exponent of each column's scale.  One workgroup per 32 columns, 8 threads per column.
template <typename C, bool INNER>
__global__ __launch_bounds__(256) void split_pack_b_kernel(int N, int K, int Ktot, int kstep,
                                                           const C* __restrict__ B, int ldb, long sB,
                                                           const int* __restrict__ E, long sE,
                                                           char* __restrict__ P, long sP)
{
    const int b = blockIdx.y, t = threadIdx.x;
    const int nkc = sp_chunks<C>(K), Kb = min(K, Ktot - b * kstep);
    const int c = t >> 3, part = t & 7;
    const int j = blockIdx.x * 32 + c;
    const C* src = B + b * sB + (long)j * ldb;
    constexpr int Q = sp_chunks<C>(SP_KMAX) / 4;
    __shared__ __attribute__((aligned(16))) int inner[INNER ? SP_KMAX : 4];
    const int ei = INNER && t < Kb ? -E[b * sE + t] : 0;
    float2 v[Q][4];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int u = 0; u < 4; ++u)
            v[q][u] = j < N ? sp_entry(src, 4 * (part + 8 * q) + u, 1, Kb) : make_float2(0.f, 0.f);
    if constexpr (INNER) {
        inner[t] = ei;
        __syncthreads();
    }
    int top = SP_NONE;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        int2 ek[4] = {};
        if constexpr (INNER) sp_inner<C>(inner, part + 8 * q, ek);
#pragma unroll
        for (int u = 0; u < 4; ++u) top = max(top, part_expo(v[q][u], ek[u]));
    }
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) top = max(top, __shfl_xor(top, off));
    const int e = split_expo(top);
    char* Pb = P + b * sP;
    if (part == 0) reinterpret_cast<int*>(Pb + sp_frag_bytes<C>(N, K))[j] = e;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int p = part + 8 * q, kc = p >> 1;
        if (kc >= nkc) break;
        uintx4 hi, lo;
        int2 ek[4] = {};
        if constexpr (INNER) sp_inner<C>(inner, p, ek);
        split4(v[q], e, ek, &hi, &lo);
        uintx4* dst = reinterpret_cast<uintx4*>(Pb + ((long)blockIdx.x * nkc + kc) * 2 * SP_FRAG);
        dst[c + 32 * (p & 1)] = hi;
        dst[64 + c + 32 * (p & 1)] = lo;
    }
}

// The U rows of a pair of 128-wide panels on the trailing columns, with the packed operand of the
// update that follows: for every column x = [x0; x1] (the 256 rows of the pair after both panels'
// interchanges)
//     u0 = L0^-1 x0,   u1 = L1^-1 (x1 - T u0),
// L0^-1 and L1^-1 the inverses of the panels' unit triangles and T the rows of L21 of the
// first panel beside the second.  Three products of 128 x 128 on 32 columns per workgroup,
// split like the update (their left factors packed once with a power of two per row, the
// columns split here), instead of three GEMM launches and a packing pass that wrote and
// read the 256 rows each time: bound by reading them once and writing them twice (U and
// packed).  n = 4096, 64 matrices, all pairs: 5.3 ms a factorisation (three FP32 3M launches and
// the packing pass 11 ms).
constexpr int UR_NB = 128, UR_KC = UR_NB / SP_KC, UR_LD = UR_NB + 2;
constexpr long UR_OPERAND = (long)(UR_NB / 32) * UR_KC * 2 * SP_FRAG;   // bytes of one packed factor

// The three left factors (128 x 128, ld ldf[f]) packed with a scale per row; expo at eoff.  One
// workgroup per 32 rows, factor and matrix: thread (row t % 32, 16 columns of part t / 32).
struct UrFactors { const float2* p[3]; long stride[3]; int ld[3]; };
__global__ __launch_bounds__(256) void split_pack_rows_kernel(UrFactors F, char* __restrict__ P, long sP, long eoff)
{
    const int rb = blockIdx.x, f = blockIdx.y, b = blockIdx.z, t = threadIdx.x;
    const int r = t & 31, part = t >> 5;
    __shared__ float tops[8][32];
    const float2* src = F.p[f] + b * F.stride[f] + rb * 32 + r;
    float2 v[4][4];
    float top = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            v[q][u] = src[(long)(16 * part + 4 * q + u) * F.ld[f]];
            top = fmaxf(top, fmaxf(fabsf(v[q][u].x), fabsf(v[q][u].y)));
        }
    tops[part][r] = top;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) top = fmaxf(top, tops[q][r]);
    const int e = split_expo(top);
    char* Pb = P + b * sP;
    if (part == 0) reinterpret_cast<int*>(Pb + eoff)[f * UR_NB + rb * 32 + r] = e;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uintx4 hi, lo;
        split4(v[q], e, &hi, &lo);
        uintx4* dst = reinterpret_cast<uintx4*>(Pb + f * UR_OPERAND +
                                                ((long)rb * UR_KC + 2 * part + q / 2) * 2 * SP_FRAG);
        dst[r + 32 * (q & 1)] = hi;
        dst[64 + r + 32 * (q & 1)] = lo;
    }
}

__global__ __launch_bounds__(256, 2) void split_urows_kernel(float2* __restrict__ A, int lda, long sA, int ncols,
                                                             const char* __restrict__ P3, long sP, long eoff,
                                                             char* __restrict__ PB, long expo_off)
{
    __shared__ __attribute__((aligned(16))) char F[UR_KC * 2 * SP_FRAG];   // the split columns
    __shared__ __attribute__((aligned(16))) float2 S[32 * UR_LD];          // a product, column by column
    __shared__ int ex[32];
    const int b = blockIdx.y, t = threadIdx.x;
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int c = t >> 3, part = t & 7;   // column, and every eighth group of four rows of it
    const int j = blockIdx.x * 32 + c;
    const bool ok = j < ncols;
    float2* col = A + b * sA + (long)j * lda;
    auto fetch = [&](const float2* src, float2 (&v)[4][4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const floatx4* p = reinterpret_cast<const floatx4*>(src + 4 * (part + 8 * q));
            const floatx4 x = p[0], y = p[1];
            v[q][0] = make_float2(x[0], x[1]);
            v[q][1] = make_float2(x[2], x[3]);
            v[q][2] = make_float2(y[0], y[1]);
            v[q][3] = make_float2(y[2], y[3]);
        }
    };
    auto store = [&](float2* dst, const float2 (&v)[4][4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            floatx4* p = reinterpret_cast<floatx4*>(dst + 4 * (part + 8 * q));
            p[0] = floatx4{v[q][0].x, v[q][0].y, v[q][1].x, v[q][1].y};
            p[1] = floatx4{v[q][2].x, v[q][2].y, v[q][3].x, v[q][3].y};
        }
    };
    auto top_of = [&](const float2 (&v)[4][4]) {
        float top = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int u = 0; u < 4; ++u) top = fmaxf(top, fmaxf(fabsf(v[q][u].x), fabsf(v[q][u].y)));
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) top = fmaxf(top, __shfl_xor(top, off));
        return top;
    };
    // four-row group q of the thread goes to fragment (part + 8 q) / 2 of dst
    auto put = [&](char* dst, const float2 (&v)[4][4], int e) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int p = part + 8 * q;
            uintx4 hi, lo;
            split4(v[q], e, &hi, &lo);
            uintx4* d = reinterpret_cast<uintx4*>(dst + (long)(p >> 1) * 2 * SP_FRAG);
            d[c + 32 * (p & 1)] = hi;
            d[64 + c + 32 * (p & 1)] = lo;
        }
    };
    const char* Pb = P3 + b * sP;
    const int li = lane & 31, half = lane >> 5;
    // S = factor f times the split columns; wave w takes the rows 32 w .. 32 w + 31
    auto product = [&](int f) {
        const uintx4* fa = reinterpret_cast<const uintx4*>(Pb + f * UR_OPERAND + (long)wave * UR_KC * 2 * SP_FRAG) + lane;
        const uintx4* fb = reinterpret_cast<const uintx4*>(F) + lane;
        const int er = reinterpret_cast<const int*>(Pb + eoff)[f * UR_NB + wave * 32 + li];
        floatx16 re, im;
#pragma unroll
        for (int r = 0; r < 16; ++r) re[r] = im[r] = 0.f;
#pragma unroll 4
        for (int kc = 0; kc < UR_KC; ++kc) {
            uintx4 a[2], br[2], bi[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                a[h] = fa[(kc * 2 + h) * 64];
                const uintx4 v = fb[(kc * 2 + h) * 64];
                br[h] = v ^ 0x80000000u;              // (Br, -Bi)
                bi[h] = (v << 16) | (v >> 16);        // (Bi, Br)
            }
#pragma unroll
            for (int p = 0; p < 3; ++p) {   // lo hi, hi lo, hi hi
                const int ha = p == 0, hb = p == 1;
                re = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, br[hb]),
                                                            __builtin_bit_cast(half8, a[ha]), re, 0, 0, 0);
                im = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, bi[hb]),
                                                            __builtin_bit_cast(half8, a[ha]), im, 0, 0, 0);
            }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int cc = 8 * (r >> 2) + 4 * half + (r & 3);
            const int e = -(er + ex[cc]);
            S[cc * UR_LD + wave * 32 + li] = make_float2(ldexpf(re[r], e), ldexpf(im[r], e));
        }
    };
    float2 v0[4][4] = {}, v1[4][4] = {};
    if (ok) {
        fetch(col, v0);
        fetch(col + UR_NB, v1);
    }
    auto split = [&](const float2 (&v)[4][4]) {
        const int e = split_expo(top_of(v));
        if (part == 0) ex[c] = e;
        put(F, v, e);
        __syncthreads();
    };
    split(v0);
    product(0);
    __syncthreads();
    fetch(S + c * UR_LD, v0);
    split(v0);
    product(1);
    __syncthreads();
    {
        float2 w[4][4];
        fetch(S + c * UR_LD, w);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int u = 0; u < 4; ++u) v1[q][u] = csub(v1[q][u], w[q][u]);
    }
    split(v1);
    product(2);
    __syncthreads();
    fetch(S + c * UR_LD, v1);
    if (ok) {
        store(col, v0);
        store(col + UR_NB, v1);
    }
    // the update's operand: one scale for the 256 rows of the column
    const int e = split_expo(fmaxf(top_of(v0), top_of(v1)));
    char* dst = PB + b * sP + (long)blockIdx.x * 2 * UR_KC * 2 * SP_FRAG;
    if (part == 0) reinterpret_cast<int*>(PB + b * sP + expo_off)[j] = e;
    put(dst, v0, e);
    put(dst + (long)UR_KC * 2 * SP_FRAG, v1, e);
}

// Workgroup tile 128 x 128, four waves of 64 x 64 (2 x 2 blocks of 32 x 32, real and imaginary
// accumulators: 128 registers, two waves per SIMD); stages of SP_ST k chunks in two LDS buffers
// (64 KB, two workgroups per CU: one stores its tile while the other multiplies).
constexpr int SP_ST = 2, SP_T = 128;

// SUB: C -= A B, else C = A B; E: float2 or float.
template <typename E, bool SUB>
__global__ __launch_bounds__(256, 2) void gemm_split_kernel(int M, int N, int nkc, const char* __restrict__ PA,
                                                             long sPA, long expo_a, const char* __restrict__ PB,
                                                             long sPB, long expo_b, int cb0, E* __restrict__ C,
                                                             int ldc, long sC, int tilesM, int tilesN, int batch,
                                                             long total)
{
    constexpr bool CX = elem_traits<E>::complex;
    constexpr int STAGE = 4 * SP_ST * 2 * SP_FRAG;   // bytes of one operand's stage
    __shared__ __attribute__((aligned(16))) char lds[2][2][STAGE];

    const long tile = xcd_remap(blockIdx.x, total);
    const long per = (long)tilesM * tilesN;
    const long b = tile / per;
    if (b >= batch) return;
    // groups of 8 row tiles sweep the columns together (shared slices in the XCD's L2)
    constexpr int ROWS = 8;
    const int t = (int)(tile - b * per);
    const int span = ROWS * tilesN, g = t / span, first = g * ROWS, rows = min(tilesM - first, ROWS), in = t - g * span;
    const int ti = first + in % rows, tj = in / rows;
    const int nrb = (M + 31) / 32, ncb = (N + 31) / 32;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wi = wave & 1, wj = wave >> 1;
    // wave w stages row block w and column block w of the tile (blocks past the end: the last one again)
    const char* ga = PA + b * sPA + (long)min(ti * 4 + wave, nrb - 1) * nkc * 2 * SP_FRAG + lane * 16;
    const char* gb = PB + b * sPB + (long)(cb0 + min(tj * 4 + wave, ncb - 1)) * nkc * 2 * SP_FRAG + lane * 16;
    auto stage = [&](int s, int buf) {
#pragma unroll
        for (int f = 0; f < 2 * SP_ST; ++f) {
            const int kc = min(s * SP_ST + f / 2, nkc - 1);
            const long o = ((long)kc * 2 + f % 2) * SP_FRAG;
            const int l = (wave * 2 * SP_ST + f) * SP_FRAG;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(ga + o),
                                             (__attribute__((address_space(3))) void*)&lds[buf][0][l], 16, 0, 0);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(gb + o),
                                             (__attribute__((address_space(3))) void*)&lds[buf][1][l], 16, 0, 0);
        }
    };
    auto frag = [&](int buf, int op, int block, int f) {
        return *reinterpret_cast<const uintx4*>(&lds[buf][op][(block * 2 * SP_ST + f) * SP_FRAG + lane * 16]);
    };

    floatx16 accR[2][2], accI[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) accR[x][y][r] = accI[x][y][r] = 0.f;

    const int nst = (nkc + SP_ST - 1) / SP_ST;
    // a barrier orders LDS accesses but does not wait for copies into LDS in flight
    auto arrived = [] { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); __syncthreads(); };
    stage(0, 0);
    arrived();
    for (int s = 0; s < nst; ++s) {
        const int buf = s & 1;
        if (s + 1 < nst) stage(s + 1, buf ^ 1);
#pragma unroll
        for (int kc = 0; kc < SP_ST; ++kc) {
            if (SP_ST > 1 && s * SP_ST + kc >= nkc) break;
            uintx4 a[2][2], br[2][2], bi[2][2];   // [block][hi, lo]
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    a[x][h] = frag(buf, 0, wi * 2 + x, kc * 2 + h);
                    const uintx4 v = frag(buf, 1, wj * 2 + x, kc * 2 + h);
                    br[x][h] = CX ? v ^ 0x80000000u : v;        // (Br, -Bi)
                    bi[x][h] = (v << 16) | (v >> 16);           // (Bi, Br)
                }
#pragma unroll
            for (int p = 0; p < 3; ++p) {   // lo hi, hi lo, hi hi
                const int ha = p == 0, hb = p == 1;
#pragma unroll
                for (int x = 0; x < 2; ++x)
#pragma unroll
                    for (int y = 0; y < 2; ++y) {
                        accR[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                            __builtin_bit_cast(half8, br[y][hb]), __builtin_bit_cast(half8, a[x][ha]), accR[x][y], 0,
                            0, 0);
                        if constexpr (CX) accI[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                            __builtin_bit_cast(half8, bi[y][hb]), __builtin_bit_cast(half8, a[x][ha]), accI[x][y], 0,
                            0, 0);
                    }
            }
        }
        arrived();
    }

    // 2^-(scales) acc; lane li = row, register r = column 8 (r / 4) + 4 (lane / 32) + r % 4
    E* Cb = C + b * sC;
    const int* ea = reinterpret_cast<const int*>(PA + b * sPA + expo_a);
    const int* ex = reinterpret_cast<const int*>(PB + b * sPB + expo_b) + cb0 * 32;
    const int li = lane & 31, half = lane >> 5;
    int er[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) er[x] = ea[min(ti * SP_T + (wi * 2 + x) * 32 + li, M - 1)];
#pragma unroll
    for (int y = 0; y < 2; ++y) {
        const int j0 = tj * SP_T + (wj * 2 + y) * 32 + 4 * half;
        if (tj * SP_T + (wj * 2 + y) * 32 >= N) break;
        int e[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) e[r] = ex[min(j0 + 8 * (r >> 2) + (r & 3), N - 1)];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const int i = ti * SP_T + (wi * 2 + x) * 32 + li;
            if (i >= M) continue;
            E* col = Cb + i + (long)j0 * ldc;
            auto value = [&](int r) {
                const int s2 = -(er[x] + e[r]);
                if constexpr (CX) return make_float2(ldexpf(accR[x][y][r], s2), ldexpf(accI[x][y][r], s2));
                else return ldexpf(accR[x][y][r], s2);
            };
            if (tj * SP_T + (wj * 2 + y) * 32 + 32 <= N) {   // whole block: all loads in flight before the first store
                E c[16];
                if constexpr (SUB) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) c[r] = col[(long)(8 * (r >> 2) + (r & 3)) * ldc];
                }
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    col[(long)(8 * (r >> 2) + (r & 3)) * ldc] = SUB ? csub(c[r], value(r)) : value(r);
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int jr = 8 * (r >> 2) + (r & 3);
                    if (j0 + jr < N) {
                        if constexpr (SUB) col[(long)jr * ldc] = csub(col[(long)jr * ldc], value(r));
                        else col[(long)jr * ldc] = value(r);
                    }
                }
            }
        }
    }
}

template <typename C>
long split_operand_bytes(int rows, int K)
{
    return sp_frag_bytes<C>(rows, K) + (long)(rows + 31) / 32 * 32 * 4;
}

// Layout of the LU's pack buffer: the solves' exponents, A, B, then (complex) the three left factors of the U
// rows with their row exponents (the offsets follow from the sizes of the product).
template <typename C>
size_t split_pack_bytes(int n, int K)
{
    return split_column_bytes(n) + 2 * split_operand_bytes<C>(n, K) +
           (elem_traits<C>::complex ? 3 * UR_OPERAND + 3 * UR_NB * 4 : 0);
}

// Depths of at least one panel (the error is below the FP32 kernel's from K = 64 on); fewer
// than 128 rows or columns leave most of a tile empty and do not pay for the packing.
bool split_ok(int M, int N, int K) { return K >= 128 && K <= SP_KMAX && M >= 128 && N >= 128; }

hipError_t split_columns(hipStream_t st, int n, const float2* LU, int ld, long sLU, int* E, long sE, int batch)
{
    hipLaunchKernelGGL(split_columns_kernel, dim3(n, batch), dim3(256), 0, st, LU, ld, sLU, E, sE);
    return hipGetLastError();
}

template <typename C>
hipError_t split_pack_a(hipStream_t st, int M, int K, const C* A, int lda, long sA, const int* E, long sE, void* P,
                        long sP, int batch, int Ktot, int kstep)
{
    if (E)
        hipLaunchKernelGGL((split_pack_a_kernel<C, true>), dim3((M + 31) / 32, batch), dim3(256), 0, st, M, K,
                           Ktot ? Ktot : K, kstep, A, lda, sA, E, sE, (char*)P, sP);
    else
        hipLaunchKernelGGL((split_pack_a_kernel<C, false>), dim3((M + 31) / 32, batch), dim3(256), 0, st, M, K,
                           Ktot ? Ktot : K, kstep, A, lda, sA, E, sE, (char*)P, sP);
    return hipGetLastError();
}

template <typename C>
hipError_t split_pack_b(hipStream_t st, int N, int K, const C* B, int ldb, long sB, const int* E, long sE, void* P,
                        long sP, int batch, int Ktot, int kstep)
{
    if (E)
        hipLaunchKernelGGL((split_pack_b_kernel<C, true>), dim3((N + 31) / 32, batch), dim3(256), 0, st, N, K,
                           Ktot ? Ktot : K, kstep, B, ldb, sB, E, sE, (char*)P, sP);
    else
        hipLaunchKernelGGL((split_pack_b_kernel<C, false>), dim3((N + 31) / 32, batch), dim3(256), 0, st, N, K,
                           Ktot ? Ktot : K, kstep, B, ldb, sB, E, sE, (char*)P, sP);
    return hipGetLastError();
}

bool split_urows_ok(int nb, const float2* A, int lda, long sA)
{
    return nb == UR_NB && (((uintptr_t)A) & 15) == 0 && lda % 2 == 0 && sA % 2 == 0;
}

hipError_t split_urows(hipStream_t st, int M, int N, const float2* L0, int ld0, long s0, const float2* T, int ldt,
                       long sT, const float2* L1, int ld1, long s1, float2* A, int lda, long sA, void* P, long sP,
                       int batch)
{
    constexpr int K = 2 * UR_NB;
    char* Pc = (char*)P;
    const long offb = split_operand_bytes<float2>(M, K), off = offb + split_operand_bytes<float2>(N, K);
    const UrFactors F = {{L0, T, L1}, {s0, sT, s1}, {ld0, ldt, ld1}};
    hipLaunchKernelGGL(split_pack_rows_kernel, dim3(UR_NB / 32, 3, batch), dim3(256), 0, st, F, Pc + off, sP,
                       3 * UR_OPERAND);
    hipLaunchKernelGGL(split_urows_kernel, dim3((N + 31) / 32, batch), dim3(256), 0, st, A, lda, sA, N, Pc + off, sP,
                       3 * UR_OPERAND, Pc + offb, sp_frag_bytes<float2>(N, K));
    return hipGetLastError();
}

template <typename C>
hipError_t gemm_split(hipStream_t st, int M, int N, int K, const void* PA, long sPA, const void* PB, long sPB,
                      int Npack, int j0, bool sub, C* Cm, int ldc, long sC, int batch)
{
    if (M <= 0 || N <= 0 || batch <= 0) return hipSuccess;
    if (j0 % 32 != 0 || j0 + N > Npack) return hipErrorInvalidValue;
    const int tm = (M + SP_T - 1) / SP_T, tn = (N + SP_T - 1) / SP_T;
    const long total = round_up_l((long)tm * tn * batch, 8);
#define SP_L(S)                                                                                                   \
    hipLaunchKernelGGL((gemm_split_kernel<C, S>), dim3((unsigned)total), dim3(256), 0, st, M, N, sp_chunks<C>(K), \
                       (const char*)PA, sPA, sp_frag_bytes<C>(M, K), (const char*)PB, sPB,                        \
                       sp_frag_bytes<C>(Npack, K), j0 / 32, Cm, ldc, sC, tm, tn, batch, total)
    if (sub) SP_L(true);
    else if constexpr (elem_traits<C>::complex) SP_L(false);
    else return hipErrorInvalidValue;   // no real caller
#undef SP_L
    return hipGetLastError();
}

#define SP_INST(C)                                                                                                  \
    template long split_operand_bytes<C>(int, int);                                                                 \
    template size_t split_pack_bytes<C>(int, int);                                                                  \
    template hipError_t split_pack_a<C>(hipStream_t, int, int, const C*, int, long, const int*, long, void*, long,  \
                                        int, int, int);                                                             \
    template hipError_t split_pack_b<C>(hipStream_t, int, int, const C*, int, long, const int*, long, void*, long,  \
                                        int, int, int);                                                             \
    template hipError_t gemm_split<C>(hipStream_t, int, int, int, const void*, long, const void*, long, int, int,   \
                                      bool, C*, int, long, int);
SP_INST(float2)
SP_INST(float)
#undef SP_INST

}  // namespace rsrr
