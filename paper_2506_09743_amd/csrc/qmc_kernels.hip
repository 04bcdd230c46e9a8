// Launch dispatch of libqmc's walker kernels: picks the instantiation of
// the call's arithmetic form (the kernels live in qmc_kernels.h and are
// instantiated by the qmc_form_*.hip units).

#include "qmc_walker.h"

namespace qmc {

hipError_t launch_form_fp64(bool, const DevSystem &, double *, double *, double *, double *, int64_t, int,
                            double, uint64_t, uint64_t, uint32_t, double *, const CallStreams &);
hipError_t launch_form_fp32(bool, const DevSystem &, double *, double *, double *, double *, int64_t, int,
                            double, uint64_t, uint64_t, uint32_t, double *, const CallStreams &);
hipError_t launch_form_bf16(bool, const DevSystem &, double *, double *, double *, double *, int64_t, int,
                            double, uint64_t, uint64_t, uint32_t, double *, const CallStreams &, int);
hipError_t launch_form_explicit(bool, const DevSystem &, double *, double *, double *, double *, int64_t, int,
                                double, uint64_t, uint64_t, uint32_t, double *, const CallStreams &);
hipError_t launch_form_backflow(bool, const DevSystem &, double *, double *, double *, double *, int64_t, int,
                                double, uint64_t, uint64_t, uint32_t, double *, const CallStreams &, bool);

// Sums of the [W][4] accumulators over walkers in an order fixed by W:
// thread t of the one work-group adds rows t, t + T, t + 2T, ... in turn,
// then the T partial sums meet in a binary tree (T = kReduceThreads).
constexpr int kReduceThreads = 1024;

__global__ __launch_bounds__(kReduceThreads) void k_reduce_acc(const double *__restrict__ acc, int64_t W,
                                                               double *__restrict__ out) {
    __shared__ double part[5][kReduceThreads];
    const int t = threadIdx.x;
    double s[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int64_t w = t; w < W; w += kReduceThreads) {
        const double *a = acc + 4 * w;
        s[0] += a[0];
        s[1] += a[1];
        s[2] += a[2];
        s[3] += a[3];
        s[4] += a[3] != 0.0 ? 1.0 : 0.0;
    }
    for (int k = 0; k < 5; ++k) part[k][t] = s[k];
    __syncthreads();
    for (int h = kReduceThreads / 2; h > 0; h >>= 1) {
        if (t < h)
            for (int k = 0; k < 5; ++k) part[k][t] += part[k][t + h];
        __syncthreads();
    }
    if (t < 5) out[t] = part[t][0];
}

// out[p] = sum_w ga[w] A[w][p] + gb[w] B[w][p] over the columns of (A0, B0)
// [W][n0], then of (A1, B1) [W][n1]; a walker of weight zero adds nothing, even
// where its row is not finite.  Bound by reading A and B once.  The columns are
// few and the walkers many, so the walkers are split: a work-group sums one of
// `splits` ranges of them for 64 columns, its four waves taking every fourth
// walker, and k_vjp_finish adds the ranges' sums.  The order is fixed by W.
// Many-body CO, 4099 walkers: 12 + 6 us; as four products with masked copies of
// the Jacobians in torch the same sums took 480 us of kernels and 17 launches.
constexpr int kVjpSplits = 256, kVjpRows = 16;  // most ranges; fewest walkers a range is cut to

struct VjpArgs {
    const double *ga, *gb, *a0, *b0, *a1, *b1;
    int64_t W;
    int n0, n1, splits;
};

__global__ __launch_bounds__(256) void k_vjp(VjpArgs v, double *__restrict__ work) {
    __shared__ double part[4][64];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int p = 64 * (int)blockIdx.x + lane;
    const int64_t w0 = v.W * blockIdx.y / v.splits, w1 = v.W * (blockIdx.y + 1) / v.splits;
    double s = 0.0;
    if (p < v.n0 + v.n1) {
        const bool first = p < v.n0;
        const int64_t n = first ? v.n0 : v.n1;
        const double *__restrict__ a = first ? v.a0 + p : v.a1 + (p - v.n0);
        const double *__restrict__ b = first ? v.b0 + p : v.b1 + (p - v.n0);
#pragma unroll 4
        for (int64_t w = w0 + q; w < w1; w += 4) {
            const double ga = v.ga[w], gb = v.gb[w];
            const double x = a[w * n], y = b[w * n];
            s = ga != 0.0 ? fma(ga, x, s) : s;
            s = gb != 0.0 ? fma(gb, y, s) : s;
        }
    }
    part[q][lane] = s;
    __syncthreads();
    if (q == 0 && p < v.n0 + v.n1)
        work[(int64_t)blockIdx.y * (v.n0 + v.n1) + p] =
            (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
}

__global__ __launch_bounds__(256) void k_vjp_finish(const double *__restrict__ work, int splits, int n,
                                                    double *__restrict__ out) {
    __shared__ double part[4][64];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int p = 64 * (int)blockIdx.x + lane;
    double s = 0.0;
    if (p < n) {
#pragma unroll 8
        for (int k = q; k < splits; k += 4) s += work[(int64_t)k * n + p];
    }
    part[q][lane] = s;
    __syncthreads();
    if (q == 0 && p < n) out[p] = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
}

// Ranges the walkers are cut into (the rows of `work`).
int vjp_splits(int64_t W) {
    const int64_t k = (W + kVjpRows - 1) / kVjpRows;
    return (int)(k < 1 ? 1 : k > kVjpSplits ? kVjpSplits : k);
}

hipError_t launch_vjp(const double *ga, const double *gb, const double *a0, const double *b0, int n0,
                      const double *a1, const double *b1, int n1, int64_t W, double *work, double *out,
                      hipStream_t st) {
    const VjpArgs v{ga, gb, a0, b0, a1, b1, W, n0, n1, vjp_splits(W)};
    const unsigned tiles = (unsigned)((n0 + n1 + 63) / 64);
    hipLaunchKernelGGL(k_vjp, dim3(tiles, (unsigned)v.splits), dim3(256), 0, st, v, work);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_vjp_finish, dim3(tiles), dim3(256), 0, st, work, v.splits, n0 + n1, out);
    return hipGetLastError();
}

hipError_t launch_reduce_acc(const double *acc, int64_t W, double *out, hipStream_t st) {
    hipLaunchKernelGGL(k_reduce_acc, dim3(1), dim3(kReduceThreads), 0, st, acc, W, out);
    return hipGetLastError();
}

static int nmo_bucket(int n_mo) {
    const int b[] = {4, 8, 12, 16, 20, 24, 32};
    for (int v : b)
        if (n_mo <= v) return v;
    return -1;
}

int padded_mo(int n_mo) { return nmo_bucket(n_mo); }

size_t explicit_lds_bytes(const DevSystem &S) {
    int per = 0;
    switch (S.nmo_pad) {
#define QMC_CASE(N) \
    case N: per = walker::walker_lds_explicit<N>(S); break;
        QMC_CASE(4) QMC_CASE(8) QMC_CASE(12) QMC_CASE(16) QMC_CASE(20) QMC_CASE(24) QMC_CASE(32)
#undef QMC_CASE
    }
    const int admit = walker::een_admit(S);
    if (per < admit) per = admit;
    return (size_t)S.WPW * per * sizeof(double);
}

// form: 0 FP64, 1 mixed FP32 (VALU), 2 mixed BF16 on the matrix cores with
// split operands, 3 mixed BF16 single products, 4 FP64 with explicit
// determinants, 5 FP64 with backflow and every configuration factorised,
// 6 FP64 with backflow and the low-rank configuration update.
hipError_t launch_walkers(bool mc, int form, const DevSystem &S, double *X, double *LP, double *SG,
                          double *EL, int64_t W, int n_steps, double sigma, uint64_t seed,
                          uint64_t step0, uint32_t woff, double *ACC, const CallStreams &st) {
    switch (form) {
        case 0: return launch_form_fp64(mc, S, X, LP, SG, EL, W, n_steps, sigma, seed, step0, woff, ACC, st);
        case 1: return launch_form_fp32(mc, S, X, LP, SG, EL, W, n_steps, sigma, seed, step0, woff, ACC, st);
        case 2: return launch_form_bf16(mc, S, X, LP, SG, EL, W, n_steps, sigma, seed, step0, woff, ACC, st, 3);
        case 3: return launch_form_bf16(mc, S, X, LP, SG, EL, W, n_steps, sigma, seed, step0, woff, ACC, st, 1);
        case 4: return launch_form_explicit(mc, S, X, LP, SG, EL, W, n_steps, sigma, seed, step0, woff, ACC, st);
        case 5: return launch_form_backflow(mc, S, X, LP, SG, EL, W, n_steps, sigma, seed, step0, woff, ACC, st, false);
        case 6: return launch_form_backflow(mc, S, X, LP, SG, EL, W, n_steps, sigma, seed, step0, woff, ACC, st, true);
    }
    return hipErrorInvalidValue;
}

}  // namespace qmc
