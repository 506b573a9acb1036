// Shared parts of the emulated DGEMM kernels: the retained products and their
// order, and the launchers of the three kernels.
#pragma once

#include "gemm_common.h"

namespace emu {

// Product q of the retained set S_d of Eq. (product-selection), in executed
// order: diagonal l = i + j ascending, i ascending inside a diagonal, slice
// indices i, j < 6.  q ascending is the FP64 order of Eq. (fp64reconstruction);
// the sets of the depths d are prefixes of one sequence (for d <= 6 product q
// is A_i B_(l - i) with q = l (l + 1) / 2 + i).
constexpr int pair_code(int q) {
    int n = 0;
    for (int l = 0; l < 11; ++l)
        for (int i = (l > 5 ? l - 5 : 0); i <= (l < 5 ? l : 5); ++i)
            if (n++ == q) return 8 * i + (l - i);
    return -1;
}
constexpr int prod_i(int q) { return pair_code(q) >> 3; }
constexpr int prod_j(int q) { return pair_code(q) & 7; }
constexpr int n_prod(int d) {
    int n = 0;
    for (int i = 0; i < 6; ++i)
        for (int j = 0; j < 6; ++j) n += (i + j < d);
    return n;
}

// One product GEMM on packed operands: C (M x N, ldc) = alpha P + beta C over KB
// k-blocks; sa, sb: row and column weights to restore, or both null.  skip_if:
// when not null, the kernel does nothing (and leaves C) if *skip_if is nonzero.
struct DgemmArgs {
    const uint16_t *Ap, *Bp;
    double *C;
    int64_t M, N, KB, RpadA, RpadB, ldc;
    const int *sa, *sb;
    double alpha, beta;
    const unsigned *skip_if;
};

inline int persistent_workgroups() { return persistent_workgroups(device_cu_count()); }

// gemm_f64s.hip: 32 x 32 x 16 MFMA, output tile (64 BM) x 64
template <int D, int BM, int NS, bool ACC64_LDS>
hipError_t launch_s(const DgemmArgs &a, hipStream_t s);
// gemm_f64w.hip: 16 x 16 x 32 MFMA, output tile (32 BMW) x 64.  PERSIST_OK =
// false: the caller only launches long reductions, or grids of at most one tile
// per CU, which do not take the persistent grid (its instantiation is then not
// built; more tiles would run one per workgroup).
template <int D, int NS, bool ACC64_LDS, int BMW = 1, bool PERSIST_OK = true>
hipError_t launch_w(const DgemmArgs &a, hipStream_t s);
// gemm_f64t.hip: 32 x 32 x 16 MFMA over whole panels, output tile (64 t_bm(D)) x 64
template <int D>
hipError_t launch_t64(const DgemmArgs &a, hipStream_t s);

}  // namespace emu
