// C ABI: the moment matrix of the resolvent moment scheme (Sec. 4.1) from the
// sampling matrix, M = S Z (eq. MS).
//
// M_alpha = sum_i c_{alpha,i} X_i with X_i the i-th L-column block of S and
// c_{alpha,i} = omega_i zeta_i^alpha (eq. Malpha), zeta_i = (z_i - gamma)/rho,
// omega_i the barycentric weights of the zeta_i (eq. bary-wt) with every
// factor divided by the capacity C (the scaling Sec. 3.3 recommends against
// under- and overflow).  For a fixed probe column l the blocks form an
// n x N matrix (stride L lds between points) and M's columns alpha L + l an
// n x K matrix: a batch of L products with the small N x K table c^T as the
// right operand.  At most 32 moments: one stream over S (moments_stream_kernel);
// more: one batched FP64 MFMA GEMM.  The table is formed on the device (one
// wavefront per point) from the points copied next to it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "common.h"
#include "ctx.h"
#include "kernels.h"

using namespace rsrr;

// Scratch of rsrr_moments_noalloc: the raw points followed by the N x K
// coefficient table, in a file-scope device array (each GPU the library runs
// on holds its own copy until the process ends).  Host code reaches it only
// through the per-device address that hipGetSymbolAddress returns.
constexpr long MOMENTS_NOALLOC_MAX = 1L << 16;   // complex entries: N + N*K <= 65536 (1 MiB)
static __device__ __align__(256) double2 scratch[MOMENTS_NOALLOC_MAX];

namespace {

std::mutex g_scratch_mu;
std::vector<double2*> g_scratch_ptr;  // by device ordinal

// c_{alpha,i} = omega_i zeta_i^alpha at cw[i si + alpha sa], zeta_i = (z_i - gamma)/rho,
// log omega_i = -sum_{j != i} log((zeta_i - zeta_j)/C): one wavefront per point, its
// lanes over j (the logarithms and angles of a point one after the other in one
// thread took 30 us at N = 64).
__global__ __launch_bounds__(64) void moment_weights_kernel(const double2* __restrict__ z, int N, int K, double gre,
                                                            double gim, double rho, double cap,
                                                            double2* __restrict__ cw, int si, int sa)
{
    const int i = blockIdx.x;
    const double2 zi = make_double2((z[i].x - gre) / rho, (z[i].y - gim) / rho);
    double lr = 0.0, li = 0.0;
    for (int j = threadIdx.x; j < N; j += 64) {
        if (j == i) continue;
        const double2 zj = make_double2((z[j].x - gre) / rho, (z[j].y - gim) / rho);
        const double dx = (zi.x - zj.x) / cap, dy = (zi.y - zj.y) / cap;
        lr -= log(hypot(dx, dy));
        li -= atan2(dy, dx);
    }
    for (int off = 32; off >= 1; off >>= 1) {
        lr += __shfl_xor(lr, off);
        li += __shfl_xor(li, off);
    }
    if (threadIdx.x != 0) return;
    double sn, cs;
    sincos(li, &sn, &cs);
    const double m = exp(lr);
    double2 w = make_double2(m * cs, m * sn);
    for (int a = 0; a < K; ++a) {
        cw[(long)i * si + (long)a * sa] = w;
        w = cmul(w, zi);
    }
}

// M = S Z for the KC moments from a0 on: a thread per (row, probe column) walks the N
// points, reads S once, coalesced along the rows, and keeps its KC sums in registers;
// the coefficients (cw, N x K with the moment fastest) are the same for every lane
// and come through the scalar cache, those of a point as one block (a kernel per KC: with
// indices clamped to K eight points' loads were not in flight at once, 110 against 72 us).
// Bound by the stream over S: n = 4096, N = L = 64, K = 16 (335 MB) 178 us as a GEMM, whose
// 64-wide tiles left three quarters of the matrix core's columns empty, 72 us (4.7 TB/s) here;
// small ones by the latency of N / 8 loads in turn.
constexpr int MS_NT = 256, MS_KMAX = 16;
template <int KC>
__global__ __launch_bounds__(MS_NT) void moments_stream_kernel(int n, int N, int L, const double2* __restrict__ S,
                                                               int lds, const double2* __restrict__ cw, int K, int a0,
                                                               double2* __restrict__ M, int ldm)
{
    const int row = blockIdx.x * MS_NT + threadIdx.x, l = blockIdx.y;
    if (row >= n) return;
    const double2* s = S + row + (long)l * lds;
    const long step = (long)L * lds;
    double2 acc[KC];
#pragma unroll
    for (int a = 0; a < KC; ++a) acc[a] = make_double2(0.0, 0.0);
#pragma unroll 8
    for (int i = 0; i < N; ++i) {
        const double2 v = s[i * step];
        const double2* c = cw + (long)i * K + a0;
#pragma unroll
        for (int a = 0; a < KC; ++a) {
            const double2 w = c[a];
            acc[a].x = fma(w.x, v.x, acc[a].x);
            acc[a].y = fma(w.x, v.y, acc[a].y);
            acc[a].x = fma(-w.y, v.y, acc[a].x);
            acc[a].y = fma(w.y, v.x, acc[a].y);
        }
    }
    double2* m = M + row + (long)l * ldm;
#pragma unroll
    for (int a = 0; a < KC; ++a) m[(long)(a0 + a) * L * ldm] = acc[a];
}

template <int KC>
void moments_stream(hipStream_t st, int kc, int n, int N, int L, const double2* S, int lds, const double2* cw, int K,
                    int a0, double2* M, int ldm)
{
    if constexpr (KC > 1) {
        if (kc < KC) return moments_stream<KC - 1>(st, kc, n, N, L, S, lds, cw, K, a0, M, ldm);
    }
    hipLaunchKernelGGL(moments_stream_kernel<KC>, dim3((n + MS_NT - 1) / MS_NT, L), dim3(MS_NT), 0, st, n, N, L, S, lds,
                       cw, K, a0, M, ldm);
}

rsrr_status check_args(rsrr_ctx* c, int n, int N, int L, const double* S, int lds, const double* z,
                       const double* gamma, double rho, double capacity, int K, double* M, int ldm)
{
    if (!c) return -1;
    if (n < 1) return -2;
    if (N < 1) return -3;
    if (L < 1) return -4;
    if (!S) return -5;
    if (lds < n) return -6;
    if (!z) return -7;
    if (!gamma) return -8;
    if (!(rho > 0)) return -9;
    if (!(capacity > 0)) return -10;
    if (K < 1 || K > N) return -11;
    if (!M) return -12;
    if (ldm < n) return -13;
    for (int i = 0; i < N; ++i)  // coincident points have no barycentric weight
        for (int j = 0; j < i; ++j)
            if (z[2 * i] == z[2 * j] && z[2 * i + 1] == z[2 * j + 1]) return -7;
    return RSRR_OK;
}

// The points and the coefficient table in `work` (N + N*K complex), then M = S Z.
rsrr_status moments_run(rsrr_ctx* c, int n, int N, int L, const double* S, int lds, const double* z,
                        const double* gamma, double rho, double capacity, int K, double* M, int ldm, double2* work)
{
    double2* zd_ = work;
    double2* cw = work + N;
    RSRR_HIP(hipMemcpyAsync(zd_, z, (size_t)N * 16, hipMemcpyHostToDevice, c->stream));
    // Up to 32 moments: the stream (S read once per 16 of them); more: the GEMM, whose tiles are
    // then at least half used.  The grid of the stream has the probe columns in y.
    const bool stream = K <= 32 && L <= 65535;
    hipLaunchKernelGGL(moment_weights_kernel, dim3(N), dim3(64), 0, c->stream, zd_, N, K, gamma[0], gamma[1], rho,
                       capacity, cw, stream ? K : 1, stream ? 1 : N);
    RSRR_HIP(hipGetLastError());
    if (stream) {
        for (int a0 = 0; a0 < K; a0 += MS_KMAX)
            moments_stream<MS_KMAX>(c->stream, std::min(MS_KMAX, K - a0), n, N, L, (const double2*)S, lds, cw, K, a0,
                                    (double2*)M, ldm);
        RSRR_HIP(hipGetLastError());
    } else {
        // batch l: A = S + l lds (n x N, ld L lds), C = M + l ldm (n x K, ld L ldm)
        RSRR_HIP(zgemm(c->stream, 0, 0, n, K, N, 1.0, (const double2*)S, L * lds, lds, cw, N, 0, 0.0, (double2*)M,
                       L * ldm, ldm, L));
    }
    RSRR_HIP(hipStreamSynchronize(c->stream));
    return RSRR_OK;
}

}  // namespace

// Once per device, with that device current (rsrr_create): the device address of `scratch`.
rsrr_status noalloc_scratch_setup(int device, void** out)
{
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if ((int)g_scratch_ptr.size() <= device) g_scratch_ptr.resize(device + 1, nullptr);
    if (!g_scratch_ptr[device]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return RSRR_EDEVICE;
        }
        g_scratch_ptr[device] = (double2*)p;
    }
    *out = g_scratch_ptr[device];
    return RSRR_OK;
}

extern "C" rsrr_status rsrr_moments(rsrr_ctx* c, int n, int N, int L, const double* S, int lds, const double* z,
                                    const double* gamma, double rho, double capacity, int K, double* M, int ldm)
{
    const rsrr_status e = check_args(c, n, N, L, S, lds, z, gamma, rho, capacity, K, M, ldm);
    if (e) return e;
    RSRR_HIP(hipSetDevice(c->device));
    double2* work = (double2*)ws_get(c, WS_COEF, ((size_t)N + (size_t)N * K) * 16);
    if (!work) return RSRR_ENOMEM;
    return moments_run(c, n, N, L, S, lds, z, gamma, rho, capacity, K, M, ldm, work);
}

extern "C" rsrr_status rsrr_moments_noalloc(rsrr_ctx* c, int n, int N, int L, const double* S, int lds,
                                            const double* z, const double* gamma, double rho, double capacity, int K,
                                            double* M, int ldm)
{
    const rsrr_status e = check_args(c, n, N, L, S, lds, z, gamma, rho, capacity, K, M, ldm);
    if (e) return e;
    if ((long)N + (long)N * K > MOMENTS_NOALLOC_MAX) return RSRR_ELIMIT;
    if (!c->noalloc_scratch) return RSRR_EDEVICE;
    RSRR_HIP(hipSetDevice(c->device));
    return moments_run(c, n, N, L, S, lds, z, gamma, rho, capacity, K, M, ldm, (double2*)c->noalloc_scratch);
}
