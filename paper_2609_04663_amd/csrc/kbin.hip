// K-binned scale-aware scope (EMU_SCOPE_KBIN): classes of the reduction
// indices (the gathers of the index groups are in split.hip).  An extension of the
// scale-aware decomposition the paper names as its key next step (Sec. 9)
// along the reduction: the products a_mk b_kn of one k share the magnitude
// class of k, the indices of one class form a group, and every group is
// emulated with its own row/column weights and exponent chains.
//
// class(k) = min(NCLS - 1, floor(-(ceil(log2 max_m |a~_mk|) +
//                                  ceil(log2 max_n |b~_kn|)) / WIDTH)),
// a~ = op(A) with row m scaled by 2^-sA_m, b~ = op(B) with column n scaled by
// 2^-sB_n (the ROWCOL weights); -1 when either maximum is 0 (the index
// contributes exact zeros and is left out).
#include "emu_internal.h"

namespace emu {
namespace {

constexpr int KT = 256;

__device__ inline unsigned long long mbits(double x) {
    return (unsigned long long)__double_as_longlong(x);
}

// mb[k] = max over the other index of |X| 2^-w (finite entries), X stored
// rows x cols (ldx); k runs along the columns (k_is_col) or the rows, and w is
// indexed by the other coordinate.  With k along the columns one atomic maximum
// per k and block, and mb must be zero on entry.
__global__ __launch_bounds__(KT) void weighted_kmax_kernel(const double *__restrict__ X,
                                                           int64_t rows, int64_t cols, int64_t ldx,
                                                           int k_is_col, const int *__restrict__ w,
                                                           unsigned long long *__restrict__ mb) {
    if (k_is_col) {
        // lanes along the columns (coalesced), the block's rows strided
        const int64_t c = (int64_t)blockIdx.x * KT + threadIdx.x;
        if (c >= cols) return;
        const int64_t per = (rows + gridDim.y - 1) / gridDim.y;
        const int64_t r0 = (int64_t)blockIdx.y * per, r1 = r0 + per < rows ? r0 + per : rows;
        double m = 0.0;
        for (int64_t r = r0; r < r1; r += 8) {   // eight loads in flight
            double x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = r + u < r1 ? X[(r + u) * ldx + c] : 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (__builtin_isfinite(x[u]))
                    m = fmax(m, fabs(ldexp(x[u], -w[r + u < r1 ? r + u : r])));
        }
        if (m > 0.0) atomicMax(&mb[c], mbits(m));
    } else {
        // one row per wave, eight loads in flight
        const int lane = threadIdx.x & 63;
        for (int64_t r = (int64_t)blockIdx.x * (KT / 64) + (threadIdx.x >> 6); r < rows;
             r += (int64_t)gridDim.x * (KT / 64)) {
            double m = 0.0;
            for (int64_t c0 = lane; c0 < cols; c0 += 8 * 64) {
                double x[8];
                int e[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int64_t c = c0 + u * 64;
                    x[u] = c < cols ? X[r * ldx + c] : 0.0;
                    e[u] = c < cols ? w[c] : 0;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (__builtin_isfinite(x[u])) m = fmax(m, fabs(ldexp(x[u], -e[u])));
            }
            for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
            if (lane == 0) mb[r] = mbits(m);
        }
    }
}

__device__ inline int ceil_log2_d(double m) {
    int e;
    const double f = frexp(m, &e);
    return (f == 0.5) ? e - 1 : e;
}

__device__ inline int class_of(unsigned long long ma, unsigned long long mb) {
    const double a = __longlong_as_double((long long)ma), b = __longlong_as_double((long long)mb);
    if (!(a > 0.0 && b > 0.0)) return -1;
    const int ne = -(ceil_log2_d(a) + ceil_log2_d(b));   // >= 0: a, b <= 1
    return ne / KBIN_WIDTH < KBIN_MAX - 1 ? ne / KBIN_WIDTH : KBIN_MAX - 1;
}

// The index lists, by one block: each wave classes a run of indices, 64 at a
// time (256 loads of each array in flight), counts them by ballots, and after a
// scan over the waves puts them in their places, so every list ascends.
constexpr int LT = 1024;
__global__ __launch_bounds__(LT) void kbin_lists_kernel(const unsigned long long *__restrict__ ma,
                                                        const unsigned long long *__restrict__ mb,
                                                        int64_t K, int *__restrict__ counts,
                                                        int *__restrict__ idx) {
    __shared__ int at0[LT / 64][KBIN_MAX];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t per = (K + LT - 1) / LT * 64, k0 = per * w, k1 = k0 + per < K ? k0 + per : K;
    constexpr int U = 4;
    auto classes = [&](int64_t k, int (&c)[U]) {
        unsigned long long a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = k + u * 64 + lane;
            a[u] = i < k1 ? ma[i] : 0ull;
            b[u] = i < k1 ? mb[i] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = class_of(a[u], b[u]);
    };
    int n[KBIN_MAX] = {};
    for (int64_t k = k0; k < k1; k += U * 64) {
        int c[U];
        classes(k, c);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < KBIN_MAX; ++i) n[i] += __popcll(__ballot(c[u] == i));
    }
#pragma unroll
    for (int i = 0; i < KBIN_MAX; ++i)
        if (lane == 0) at0[w][i] = n[i];
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int i = 0; i < KBIN_MAX; ++i) {
            const int t0 = t;
            for (int v = 0; v < LT / 64; ++v) {
                const int x = at0[v][i];
                at0[v][i] = t;
                t += x;
            }
            counts[i] = t - t0;
        }
    }
    __syncthreads();
    int at[KBIN_MAX];
#pragma unroll
    for (int i = 0; i < KBIN_MAX; ++i) at[i] = at0[w][i];
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int64_t k = k0; k < k1; k += U * 64) {
        int c[U];
        classes(k, c);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < KBIN_MAX; ++i) {
                const unsigned long long m = __ballot(c[u] == i);
                if (c[u] == i) idx[at[i] + __popcll(m & below)] = (int)(k + u * 64 + lane);
                at[i] += __popcll(m);
            }
    }
}

__global__ void fill_u64_zero_kernel(unsigned long long *p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}

// C = fl(fl(alpha P) + fl(beta C)) (fl(alpha P) when beta == 0), unless the
// call's status word says that the fallback has written C already.
__global__ void axpby_f64_kernel(const double *__restrict__ P, int64_t ldp, double *__restrict__ C,
                                 int64_t ldc, int64_t M, int64_t N, double alpha, double beta,
                                 const unsigned *__restrict__ skip_if) {
    if (skip_if != nullptr && *skip_if != 0u) return;
    for (int64_t r = blockIdx.x; r < M; r += gridDim.x)
        for (int64_t c = threadIdx.x; c < N; c += blockDim.x) {
#pragma clang fp contract(off)
            const double ap = alpha * P[r * ldp + c];
            C[r * ldc + c] = beta == 0.0 ? ap : ap + beta * C[r * ldc + c];
        }
}

int grid_rows(int64_t n) { return (int)(n < 4096 ? (n > 0 ? n : 1) : 4096); }

}  // namespace

hipError_t launch_kbin_classes(const double *A, int64_t lda, bool ta, const double *B, int64_t ldb,
                               bool tb, int64_t M, int64_t N, int64_t K, const int *sa,
                               const int *sb, unsigned long long *ma, unsigned long long *mb,
                               int *counts, int *idx, hipStream_t s) {
    const int fg = (int)((K + 255) / 256 < 1024 ? (K + 255) / 256 : 1024);
    if (!ta) fill_u64_zero_kernel<<<fg, 256, 0, s>>>(ma, K);
    if (tb) fill_u64_zero_kernel<<<fg, 256, 0, s>>>(mb, K);
    // op(A): k along A's columns (stored M x K) or rows (stored K x M); weights sa by m
    auto launch = [&](const double *X, int64_t rows, int64_t cols, int64_t ld, bool k_is_col,
                      const int *w, unsigned long long *out) {
        if (k_is_col) {
            const int64_t gx = (cols + KT - 1) / KT;
            int64_t gy = (rows + 63) / 64;      // 256 rows a slice: 118 us at 1024 x 16384
            if (gy > 65535) gy = 65535;
            if (gx * gy > 16384) gy = 16384 / gx > 1 ? 16384 / gx : 1;
            weighted_kmax_kernel<<<dim3((unsigned)gx, (unsigned)gy), KT, 0, s>>>(X, rows, cols, ld,
                                                                                  1, w, out);
        } else {
            weighted_kmax_kernel<<<grid_rows((rows + KT / 64 - 1) / (KT / 64)), KT, 0, s>>>(
                X, rows, cols, ld, 0, w, out);
        }
    };
    if (ta) launch(A, K, M, lda, false, sa, ma);
    else launch(A, M, K, lda, true, sa, ma);
    // op(B): k along B's rows (stored K x N) or columns (stored N x K); weights sb by n
    if (tb) launch(B, N, K, ldb, true, sb, mb);
    else launch(B, K, N, ldb, false, sb, mb);
    kbin_lists_kernel<<<1, LT, 0, s>>>(ma, mb, K, counts, idx);
    return hipGetLastError();
}

hipError_t launch_axpby_f64(const double *P, int64_t ldp, double *C, int64_t ldc, int64_t M,
                            int64_t N, double alpha, double beta, const unsigned *skip_if,
                            hipStream_t s) {
    axpby_f64_kernel<<<grid_rows(M), 256, 0, s>>>(P, ldp, C, ldc, M, N, alpha, beta, skip_if);
    return hipGetLastError();
}

}  // namespace emu
