// Emulated DGEMM: the N_p(d) retained component products of the fixed
// six-slice split (Eq. fp64productcounts), each evaluated per reduction panel
// of 256 on bf16 MFMA with FP32 accumulation, then widened and added in FP64
// (Eq. fp64reconstruction, Algorithm fp64, Sec. 6.3) -- the FP64
// widen-and-accumulate epilogue is fused into the k-loop.
//
// Exactness of a panel product.  With operand-wide exponents every entry of
// slice A_i is an integer multiple of 2^(vA_i - 8) of magnitude <= 2^vA_i, so a
// panel sum of 256 slice products is an integer multiple of
// 2^(vA_i + vB_j - 16) below 2^24 such units: every partial sum is an FP32
// value and the MFMA accumulation is exact in any order.  The FP64 result then
// depends only on the order of the FP64 additions, which here is the paper's:
// panel ascending, diagonal l = i + j ascending, i ascending inside a diagonal.
//
// Three kernels.  gemm_f64_kernel (gemm_f64s.hip): 32 x 32 x 16 MFMA, 4 waves in a 2 x 2
// grid; wave tile (32 BM) x 32, output tile (64 BM) x 64.  gemm_f64w_kernel
// (gemm_f64w.hip): 16 x 16 x 32 MFMA on a (16 BMW) x 32 wave tile, one barrier
// per k-block; it runs depths d >= 7, small grids and d = 6 where the panels do
// not suit.  gemm_f64t_kernel (gemm_f64t.hip): 32 x 32 x 16 MFMA over whole
// panels, d = 3 .. 6 on grids that fill the CUs (panel_kernel_wanted in
// dgemm_plan.h; the choice among the others is made in launch_gemm_f64).  Per
// k-block of 32 the d planes of both operands are copied straight into LDS (global_load_lds_dwordx4) through a ring of LDS stages.
// Each wave keeps one FP32 accumulator set per product for the whole panel
// (all N_p live, so every fragment read from LDS feeds every product that
// uses it) and an FP64 accumulator tile.
#include "gemm_f64.h"

namespace emu {

hipError_t launch_gemm_f64(const uint16_t *Ap, const uint16_t *Bp, double *C, int64_t M,
                           int64_t N, int64_t KB, int64_t RpadA, int64_t RpadB, int64_t ldc,
                           const int *sa, const int *sb, double alpha, double beta, int d,
                           bool panels, const unsigned *skip_if, hipStream_t s) {
    // First gemm_f64t_kernel where the plan packed the operands for it.  The
    // other calls of depths 1 .. 5 take the wide kernel's 64 x 64 tiles (BMW = 2)
    // where it measured faster than the 32 x 32 x 16 kernel: long reductions
    // (K > 1024) of d = 2 (8 % at 8192^3), and grids of d = 1 .. 3 whose 128- or
    // 256-row tiles would number fewer than the CUs (1.5 - 1.9x at 1000 x 1000
    // x 8200).  Long reductions of d = 4 and 5 come here only with fewer tiles
    // than CUs, where both kernels take the same time within 5 % (32 x 32 x 16 /
    // wide, us: d = 4 1024 x 1024 x 4096 87.2 / 88.7, 1024 x 768 x 8192 141.8 /
    // 149.1, 1400 x 1400 x 8200 326.3 / 326.7; d = 5 900 x 900 x 4096 118.9 /
    // 115.8, 1000 x 1000 x 16384 450.5 / 448.6).  The
    // other long reductions of d = 1 take its 128 x 64 tiles (BMW = 4; 7-40 %
    // faster).  All kernels give the same bits.
    const DgemmArgs a = {Ap, Bp, C, M, N, KB, RpadA, RpadB, ldc, sa, sb, alpha, beta,
                         skip_if};
    const int pw = persistent_workgroups();
    auto few_tiles = [&](int64_t mt) {
        return ((M + mt - 1) / mt) * ((N + DGEMM_NT - 1) / DGEMM_NT) < pw;
    };
    const bool long_k = KB > 32;
    if (panels) {
        switch (d) {
            case 3: return launch_t64<3>(a, s);
            case 4: return launch_t64<4>(a, s);
            case 5: return launch_t64<5>(a, s);
            case 6: return launch_t64<6>(a, s);
            default: return hipErrorInvalidValue;
        }
    }
    switch (d) {
        case 1:
            if (few_tiles(256))
                return launch_w<1, 4, false, 2>(a, s);
            if (long_k)
                return launch_w<1, 4, false, 4, false>(a, s);
            return launch_s<1, 4, 4, false>(a, s);
        case 2:
            if (long_k || few_tiles(128))
                return launch_w<2, 4, false, 2>(a, s);
            return launch_s<2, 2, 4, false>(a, s);
        case 3:
            if (few_tiles(128))
                return launch_w<3, 4, false, 2>(a, s);
            return launch_s<3, 2, 3, false>(a, s);
        case 4:
            // 32 x 64 tiles where they number no more than the CUs (nprod 10 calls,
            // 64 x 64 / 32 x 64, us: 512^3 27.1 / 24.3, 700 x 600 x 800 37.2 / 32.8,
            // 300 x 300 x 1000 37.4 / 32.0; 1024^3, 512 tiles, 48.0 / 53.7)
            if (few_tiles(32) || ((M + 31) / 32) * ((N + DGEMM_NT - 1) / DGEMM_NT) == pw)
                return launch_w<4, 4, false, 1, false>(a, s);
            if (long_k)
                return launch_w<4, 4, false, 2, false>(a, s);
            return launch_s<4, 1, 3, false>(a, s);
        case 5:
            if (long_k)
                return launch_w<5, 3, true, 2, false>(a, s);
            return launch_s<5, 1, 3, true>(a, s);
        case 6: return launch_w<6, 4, false>(a, s);
        case 7: return launch_w<7, 3, false>(a, s);
        case 8: return launch_w<8, 3, true>(a, s);
        case 9: return launch_w<9, 3, true>(a, s);
        case 10: return launch_w<10, 3, true>(a, s);
        case 11: return launch_w<11, 3, true>(a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace emu
