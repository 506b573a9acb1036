// Emulated DGEMM, depths d = 3 .. 6 over whole panels (see gemm_f64.hip for the
// method and the choice): 32 x 32 x 16 MFMA with wave tiles
// of BM 32 x 32 blocks: four waves in a 2 x 2 grid, output tile (64 BM) x 64
// (d = 6 and 5: BM = 1; d = 4 and 3: BM = 2).  Every retained product's
// accumulators (16 registers per block) stay live for the whole panel: the
// first 16 sets in AGPRs, the rest in VGPRs through inline asm; the FP64 tile
// (16 BM doubles per lane) is in VGPRs.  The operand fragments of a 16-index
// sub-step (BM blocks of every A slice, one block of every B slice) are held in
// one register set: each is re-read for the next sub-step right after its last
// MFMA in the current one, except those whose last use comes too late for the
// read to land in time (the double-buffered set below), which are read into a
// second buffer at the start of the sub-step.  The two sub-steps of a k-block
// run the products in two orders chosen for that: sub-step 0 walks B's slices
// downward (the A fragments finish late: they are the double-buffered ones),
// sub-step 1 walks A's slices upward.  The k-block's d planes of both operands
// are copied in 1 KB copies, d (BM + 1) per wave, NS k-blocks ahead through a
// ring of NS LDS stages; one barrier per k-block, between its sub-steps.
#include "gemm_f64.h"

namespace emu {
namespace {

// Fragment codes: A slice i, block b -> 8 b + i (< 32); B slice j -> 32 + j.
constexpr int fa_code(int i, int b) { return 8 * b + i; }
constexpr int fb_code(int j) { return 32 + j; }

// The slot schedule of a k-block (tables, computed once per instantiation).
template <int D, int BM, int W0, int W1>
struct Sched {
    static constexpr int T = n_prod(D) * BM, F = 40;
    // MFMA t of sub-step order o: 64 b + 8 i + j (product A_i B_j on block b)
    int mfma[2][T] = {};
    bool valid[F] = {};
    // Double-buffered: its last use in sub-step 0 falls in the last W0 MFMAs (the
    // read would still be in flight at the barrier that follows), or its last use
    // in sub-step 1 in the last W1 (the compiler waits for every outstanding LDS
    // read before the first MFMA of a k-block, since the k-block's copies count as
    // such events too), or fewer than four MFMAs separate its last use in sub-step
    // 1 from its first use in the next sub-step 0.
    bool db[F] = {};
    // slot after whose MFMA fragment f is read for the next sub-step (order o)
    int read_slot[2][F] = {};

    constexpr Sched() {
        constexpr int npl = D < 6 ? D : 6;
        int n = 0;
        for (int i = 0; i < npl; ++i)
            for (int b = 0; b < BM; ++b)
                for (int j = 0; j < npl; ++j)
                    if (i + j < D) mfma[1][n++] = 64 * b + 8 * i + j;
        n = 0;
        for (int j = npl - 1; j >= 0; --j)
            for (int i = 0; i < npl; ++i)
                for (int b = 0; b < BM; ++b)
                    if (i + j < D) mfma[0][n++] = 64 * b + 8 * i + j;
        int last[2][F] = {}, first[2][F] = {};
        for (int o = 0; o < 2; ++o)
            for (int t = T - 1; t >= 0; --t) {
                const int c = mfma[o][t], fa = fa_code((c >> 3) & 7, c >> 6), fb = fb_code(c & 7);
                for (int f : {fa, fb}) {
                    if (last[o][f] < t) last[o][f] = t;
                    first[o][f] = t;
                    valid[f] = true;
                }
            }
        int rank = 0;
        for (int f = 0; f < F; ++f) {
            if (!valid[f]) continue;
            db[f] = last[0][f] >= T - W0 || last[1][f] >= T - W1 ||
                    (T - 1 - last[1][f]) + first[0][f] < 4;
            for (int o = 0; o < 2; ++o) read_slot[o][f] = db[f] ? rank : last[o][f];
            if (db[f]) ++rank;
        }
    }
};
template <int D, int BM, int W0, int W1>
struct SchedOf {
    static constexpr Sched<D, BM, W0, W1> t{};
};

// Product index q of pair (i, j) for d <= 6: diagonal l = i + j ascending, i ascending.
constexpr int q_of(int i, int j) { return (i + j) * (i + j + 1) / 2 + i; }

template <int D, int BM>
struct CfgT {
    static constexpr int P = n_prod(D);
    static constexpr int NPL = D;                                   // d <= 6
    static constexpr int MT = 64 * BM, NT = 64;
    static constexpr int A_BYTES = MT * 64, B_BYTES = NT * 64;      // one plane of a stage
    static constexpr int STAGE = NPL * (A_BYTES + B_BYTES);
    static constexpr int NS = 160 * 1024 / STAGE < 4 ? 160 * 1024 / STAGE : 4;
    static constexpr int COPIES = NPL * (BM + 1);                   // per wave and k-block
    static constexpr int T = P * BM;                                // MFMAs per sub-step
    static constexpr int Q_VGPR = T > 16 ? 16 / BM : P;             // AGPRs hold 16 sets
    static_assert(D >= 3 && D <= 6, "depths 3 .. 6");
    static_assert(4 * COPIES * 1024 == STAGE, "copy split");
    static_assert(NS >= 3 && (NS - 1) * COPIES <= 63, "LDS stages");
};

template <int D, int BM, int W0, int W1, bool PERSIST>
__global__ __launch_bounds__(256, 1) void gemm_f64t_kernel(
    const uint16_t *__restrict__ Ap, const uint16_t *__restrict__ Bp, double *__restrict__ C,
    int64_t M, int64_t N, int KB, int64_t RpadA, int64_t RpadB, int64_t ldc,
    const int *__restrict__ sa, const int *__restrict__ sb, double alpha, double beta, int nt_m,
    int nt_n, int ntiles, const unsigned *__restrict__ skip_if) {
    if (skip_if != nullptr && *skip_if != 0u) return;
    using K = CfgT<D, BM>;
    constexpr int P = K::P, NPL = K::NPL, NS = K::NS, T = K::T;
    using SC = SchedOf<D, BM, W0, W1>;
    __shared__ __attribute__((aligned(1024))) char lds[NS * K::STAGE];

    // PERSIST: workgroup w0 of G takes tiles w0, w0 + G, ... (`mine` of them) and
    // walks them as one sequence of k-blocks, the copies running on into the
    // next tile; otherwise one tile per workgroup.  Groups of 4 tile rows: the
    // 32 tiles resident on an XCD share each A row-panel 8 ways and each B
    // column-panel 4 ways (measured 0.7-3.4 % less GEMM time than groups of 8
    // at 8192^3, d = 3 .. 6).
    const int G = gridDim.x;
    const int mine = PERSIST ? (ntiles - 1 - (int)blockIdx.x) / G + 1 : 1;
    const int lane = threadIdx.x & 63;
    const unsigned lane16 = (unsigned)lane * 16u;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // Copy c of a k-block by wave w: for c < NPL BM, part 4 (c % BM) + w (16
    // rows, 1 KB) of A plane c / BM; else part w of B plane c - NPL BM.  ak, bk:
    // the copied k-block's slab of plane 0 at the tile's first row / column.
    const char *Ag = reinterpret_cast<const char *>(Ap) + wave * 1024;
    const char *Bg = reinterpret_cast<const char *>(Bp) + wave * 1024;
    const int64_t a_plane = plane_elems(KB, RpadA) * 2, b_plane = plane_elems(KB, RpadB) * 2;
    const int64_t a_kstep = RpadA * 64, b_kstep = RpadB * 64;
    auto issue = [&](const char *ak, const char *bk, char *dst, auto c_c) {
        constexpr int c = decltype(c_c)::value;
        if constexpr (c < NPL * BM)
            copy_1k(ak + (c / BM) * a_plane + (c % BM) * 4096,
                    dst + (c / BM) * K::A_BYTES + (c % BM) * 4096 + wave * 1024, lane16);
        else
            copy_1k(bk + (c - NPL * BM) * b_plane,
                    dst + NPL * K::A_BYTES + (c - NPL * BM) * K::B_BYTES + wave * 1024, lane16);
    };
    // copy cursor: the k-block whose copies are issued next and its stage; after
    // a tile's last k-block it goes on at n_ak, n_bk, the next tile's first one
    // (after the last tile that tile's own: in bounds, unused)
    int c_kb = 0, c_st = 0;
    const char *c_ak, *c_bk, *n_ak, *n_bk;
    auto cursor_next = [&]() {
        ++c_kb;
        const bool wrap = c_kb == KB;
        c_kb = wrap ? 0 : c_kb;
        c_ak = wrap ? n_ak : c_ak + a_kstep;
        c_bk = wrap ? n_bk : c_bk + b_kstep;
        c_st = c_st + 1 == NS ? 0 : c_st + 1;
    };
    auto tile_bases = [&](int it, const char *&ak, const char *&bk) {
        int tm, tn;
        tile_coords_of<4>((int)blockIdx.x + it * G, ntiles, nt_m, nt_n, tm, tn);
        ak = Ag + (int64_t)tm * K::MT * 64;
        bk = Bg + (int64_t)tn * K::NT * 64;
    };
    tile_bases(0, c_ak, c_bk);
    n_ak = c_ak;
    n_bk = c_bk;
    auto stage = [&](int s) -> char * { return lds + s * K::STAGE; };

    const int off0 = frag_offset(lane, 0), off1 = frag_offset(lane, 1);
    const char *const At0 = lds + (wm * 32 * BM) * 64;
    const char *const Bt0 = lds + NPL * K::A_BYTES + (wn * 32) * 64;
    // fragments: [slice][block][buffer]; buffer 1 only for the double-buffered ones
    bf16x8 fa[NPL][BM][2], fb[NPL][2];
    auto read_frag = [&](int so, int off, auto f_c, auto buf_c) {
        constexpr int f = decltype(f_c)::value, u = decltype(buf_c)::value;
        if constexpr (f < 32)
            fa[f % 8][f / 8][u] = lds_frag(At0 + so + (f % 8) * K::A_BYTES + (f / 8) * 32 * 64, off);
        else
            fb[f - 32][u] = lds_frag(Bt0 + so + (f - 32) * K::B_BYTES, off);
    };

    f32x16 acc[P * BM];   // product q, block b at q BM + b
    // Sub-step of order O (= its parity): the T MFMAs, the reads of the next
    // sub-step (stage offset nso, lane offset noff) and NC copies of the
    // cursor's k-block spread over the slots.  MFMA first in every slot: its
    // operands were read a sub-step earlier.
    auto step = [&](auto o_c, auto zero_c, int nso, int noff, auto nc_c) {
        constexpr int O = decltype(o_c)::value;
        constexpr bool zero = decltype(zero_c)::value;
        constexpr int NC = decltype(nc_c)::value;
        char *cdst = stage(c_st);
        static_for<T>([&](auto t_c) {
            constexpr int t = decltype(t_c)::value;
            constexpr int code = SC::t.mfma[O][t], b = code >> 6, i = (code >> 3) & 7,
                          j = code & 7, x = q_of(i, j) * BM + b;
            constexpr int ua = SC::t.db[fa_code(i, b)] ? O : 0;
            constexpr int ub = SC::t.db[fb_code(j)] ? O : 0;
            if constexpr (q_of(i, j) >= K::Q_VGPR) {
                if constexpr (zero) mfma_vacc_zero(acc[x], fa[i][b][ua], fb[j][ub]);
                else mfma_vacc(acc[x], fa[i][b][ua], fb[j][ub]);
            } else {
                acc[x] = mfma(fa[i][b][ua], fb[j][ub], zero ? f32x16{} : acc[x]);
            }
            order_fence();
            static_for<40>([&](auto f_c) {
                constexpr int f = decltype(f_c)::value;
                if constexpr (SC::t.valid[f] && SC::t.read_slot[O][f] == t)
                    read_frag(nso, noff, f_c,
                              std::integral_constant<int, SC::t.db[f] ? 1 - O : 0>{});
            });
            order_fence();
            // NC copies spread over the T slots (the k-th after slot ceil((k + 1) T / NC) - 1)
            if constexpr (NC > 0 && (t * NC) / T != ((t + 1) * NC) / T)
                issue(c_ak, c_bk, cdst, std::integral_constant<int, (t * NC) / T>{});
            order_fence();
        });
    };

    // prologue: k-blocks 0 .. NS - 1 into the stages; wait for k-block 0
    for (int s = 0; s < NS; ++s) {
        static_for<K::COPIES>([&](auto c_c) { issue(c_ak, c_bk, stage(c_st), c_c); });
        cursor_next();
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * K::COPIES) : "memory");
    __syncthreads();
    static_for<40>([&](auto f_c) {
        if constexpr (SC::t.valid[decltype(f_c)::value])
            read_frag(0, off0, f_c, std::integral_constant<int, 0>{});
    });

    int qs = 0;   // stage of the current k-block
    // k-block kb: sub-step 0, wait + barrier, sub-step 1 with the copies of
    // k-block kb + NS (into the stage of kb, which no wave reads any more)
    auto kblock = [&](auto zero_c) {
        const int qn = qs + 1 == NS ? 0 : qs + 1;
        step(std::integral_constant<int, 0>{}, zero_c, qs * K::STAGE, off1,
             std::integral_constant<int, 0>{});
        __builtin_amdgcn_sched_barrier(0);
        // k-block kb + 1 landed: only kb + 2 .. kb + NS - 1 may still be in flight
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * K::COPIES) : "memory");
        pipeline_barrier();
        step(std::integral_constant<int, 1>{}, std::false_type{}, qn * K::STAGE, off0,
             std::integral_constant<int, K::COPIES>{});
        __builtin_amdgcn_sched_barrier(0);
        cursor_next();
        qs = qn;
    };
    for (int it = 0; it < mine; ++it) {
        int tm, tn;
        tile_coords_of<4>((int)blockIdx.x + it * G, ntiles, nt_m, nt_n, tm, tn);
        const int64_t m0 = (int64_t)tm * K::MT, n0 = (int64_t)tn * K::NT;
        if constexpr (PERSIST) tile_bases(it + 1 < mine ? it + 1 : it, n_ak, n_bk);
        double acc64[BM][16];
#pragma unroll
        for (int b = 0; b < BM; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc64[b][r] = 0.0;
        // whole panels (KB is a multiple of 8: the planes are zero-padded to
        // whole panels, which adds exact zeros to the last panel's sums); the
        // panel's k-blocks are unrolled (a loop over them made the compiler
        // spill the FP64 tile around it)
        for (int p0 = 0; p0 < KB; p0 += KB_PER_PANEL) {
            kblock(std::true_type{});
#pragma unroll
            for (int kb = 1; kb < KB_PER_PANEL; ++kb) kblock(std::false_type{});
            // panel end: widen each product exactly and add it in FP64, in order
            // (one product at a time, so that only its values are in flight)
#pragma unroll
            for (int x = K::Q_VGPR * BM; x < P * BM; ++x) mfma_vacc_settle(acc[x]);
            static_for<P>([&](auto q_c) {
                constexpr int q = decltype(q_c)::value;
#pragma unroll
                for (int b = 0; b < BM; ++b)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc64[b][r] += (double)acc[q * BM + b][r];
                __builtin_amdgcn_sched_barrier(0);
            });
        }
        // (the lane is laundered so that the store's addresses are not hoisted
        // out of the tile loop into registers the k-loop needs)
        int sl = lane;
        if constexpr (PERSIST) asm volatile("" : "+v"(sl));
        store_tile<BM, 16>([&](int b, int r) { return acc64[b][r]; },
                           [&](int b, int r) { return m0 + (wm * BM + b) * 32 + acc_row(r); },
                           acc_lrow(sl), [&](int) { return n0 + wn * 32; }, sl & 31,
                           m0 + K::MT <= M && n0 + K::NT <= N, M, N, C, ldc, alpha, beta, sa, sb);
    }
    // the last trips issued (unused) copies: let them land before the
    // workgroup ends and its LDS is handed to another workgroup
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

}  // namespace

template <int D>
hipError_t launch_t64(const DgemmArgs &a, hipStream_t s) {
    constexpr int BM = t_bm(D);
    using K = CfgT<D, BM>;
    if (a.KB < KB_PER_PANEL || a.KB % KB_PER_PANEL != 0 || a.RpadA % K::MT != 0 || a.RpadB % K::NT != 0)
        return hipErrorInvalidValue;
    const int nt_m = (int)((a.M + K::MT - 1) / K::MT), nt_n = (int)((a.N + K::NT - 1) / K::NT);
    const int ntiles = nt_m * nt_n, pw = persistent_workgroups();
    // Reductions up to K = 2048, and d = 3 at any: one persistent workgroup per CU, so the next
    // tile's first copies overlap a tile's epilogue and store, about 7 us per
    // tile where the reduction of 512 itself takes 17 (d = 4; 16384 x 16384 x
    // 512 with one workgroup per tile / persistent, ms: d = 3 2.44 / 2.09, d = 4 3.07 /
    // 2.88, d = 5 4.61 / 4.00, d = 6 5.59 / 5.24; 8192 x 8192 x 2048 1-5 % less).
    // Longer ones keep the dispatcher's balancing: persistent was 2-4 % slower
    // at 8192^3 and 16384 x 8192 x 4096 for d = 4 .. 6, 1-3 % faster for d = 3.
    if ((D == 3 || a.KB <= 64) && ntiles > pw)
        gemm_f64t_kernel<D, BM, 4, 8, true><<<pw, 256, 0, s>>>(
            a.Ap, a.Bp, a.C, a.M, a.N, (int)a.KB, a.RpadA, a.RpadB, a.ldc, a.sa, a.sb, a.alpha,
            a.beta, nt_m, nt_n, ntiles, a.skip_if);
    else
        gemm_f64t_kernel<D, BM, 4, 8, false><<<ntiles, 256, 0, s>>>(
            a.Ap, a.Bp, a.C, a.M, a.N, (int)a.KB, a.RpadA, a.RpadB, a.ldc, a.sa, a.sb, a.alpha,
            a.beta, nt_m, nt_n, ntiles, a.skip_if);
    return hipGetLastError();
}

template hipError_t launch_t64<3>(const DgemmArgs &, hipStream_t);
template hipError_t launch_t64<4>(const DgemmArgs &, hipStream_t);
template hipError_t launch_t64<5>(const DgemmArgs &, hipStream_t);
template hipError_t launch_t64<6>(const DgemmArgs &, hipStream_t);

}  // namespace emu
