// Emulated DGEMM on 32 x 32 tiles (see gemm_f64.hip for the method): 4 waves in
// a 2 x 2 grid, wave tile (32 BM) x 32, output tile (64 BM) x 64.
#include "gemm_f64.h"

namespace emu {
namespace {

template <int D, int BM, int NS, bool ACC64_LDS>
struct Cfg {
    static constexpr int P = n_prod(D);             // retained products N_p(d)
    // FP64 accumulator tile in LDS instead of registers (frees 32 BM VGPRs for
    // the N_p FP32 accumulator sets; touched once per panel)
    static constexpr int ACC64_BYTES = ACC64_LDS ? 4 * 64 * 16 * BM * 8 : 0;
    // products q >= Q_VGPR keep their accumulators in VGPRs (inline-asm MFMA)
    // so that all N_p sets fit: 256 AGPRs hold 16 sets of 16 registers
    static constexpr int Q_VGPR = P * BM > 16 ? 16 / BM : P;
    static constexpr int MT = 64 * BM, NT = DGEMM_NT;
    static constexpr int A_BYTES = MT * 64, B_BYTES = NT * 64;
    static constexpr int STAGE = D * (A_BYTES + B_BYTES);
    static constexpr int NSTAGE = NS;               // LDS stages (copy lead = NS - 1 k-blocks)
    static constexpr int A_PARTS = A_BYTES / 1024, B_PARTS = B_BYTES / 1024;
    static constexpr int COPIES = D * (A_PARTS + B_PARTS) / 4;   // 1 KB copies per wave per k-block
    static constexpr int READS = D * (BM + 1);      // fragment reads per sub-step
    static constexpr int MMAS = P * BM;             // MFMAs per sub-step
    static_assert(A_PARTS == 4 * BM && B_PARTS == 4, "copy split assumes 4 waves");
    static_assert(NS * STAGE + ACC64_BYTES <= 160 * 1024, "LDS");
};

// Per sub-step instruction order.  MFMA t is product t / BM on row block
// t % BM (products in q order); read t loads the t-th distinct operand
// fragment in order of first use by that MFMA sequence, encoded as
// 64 * is_B + 8 * plane + row block.  Reads of the next sub-step go out in
// the order its MFMAs will want them.
template <int D, int BM>
constexpr int read_code(int t) {
    bool seen_a[6][4] = {}, seen_b[6] = {};
    int r = 0;
    for (int u = 0; u < n_prod(D) * BM; ++u) {
        const int q = u / BM, b = u % BM, i = prod_i(q), j = prod_j(q);
        if (!seen_a[i][b]) {
            seen_a[i][b] = true;
            if (r++ == t) return 8 * i + b;
        }
        if (!seen_b[j]) {
            seen_b[j] = true;
            if (r++ == t) return 64 + 8 * j;
        }
    }
    return -1;
}

template <int D, int BM, int NS, bool ACC64_LDS, bool PERSIST>
__global__ __launch_bounds__(256, 1) void gemm_f64_kernel(
    const uint16_t *__restrict__ Ap, const uint16_t *__restrict__ Bp, double *__restrict__ C,
    int64_t M, int64_t N, int KB, int64_t RpadA, int64_t RpadB, int64_t ldc,
    const int *__restrict__ sa, const int *__restrict__ sb, double alpha, double beta, int nt_m,
    int nt_n, int ntiles, const unsigned *__restrict__ skip_if) {
    if (skip_if != nullptr && *skip_if != 0u) return;
    using K = Cfg<D, BM, NS, ACC64_LDS>;
    __shared__ __attribute__((aligned(1024))) char lds[K::NSTAGE * K::STAGE + K::ACC64_BYTES];
    // lane-private FP64 accumulators in LDS: element r of lane l of wave w at
    // ((w * BM + b) * 16 + r) * 64 + l (consecutive lanes, consecutive doubles)
    double *acc64_lds = reinterpret_cast<double *>(lds + K::NSTAGE * K::STAGE);

    // PERSIST: workgroup w0 of G takes tiles w0, w0 + G, ... (`mine` of them)
    // and walks them as one sequence of k-blocks, the copies running on into
    // the next tile; otherwise one tile per workgroup.
    const int G = gridDim.x;
    const int mine = PERSIST ? (ntiles - 1 - (int)blockIdx.x) / G + 1 : 1;
    const int lane = threadIdx.x & 63;
    const unsigned lane16 = (unsigned)lane * 16u;   // copy offset of this lane
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform
    const int wm = wave >> 1, wn = wave & 1;

    const char *Ag = reinterpret_cast<const char *>(Ap);
    const char *Bg = reinterpret_cast<const char *>(Bp);
    const int64_t a_plane = plane_elems(KB, RpadA) * 2;
    const int64_t b_plane = plane_elems(KB, RpadB) * 2;

    // Copy issue for one k-block: wave w moves 1 KB parts [w BM, (w + 1) BM) of
    // every A plane and part w of every B plane (wave-uniform base plus
    // compile-time offsets).  ak, bk: the k-block's slab of plane 0 at the
    // copied tile's first row.
    const int64_t a_base = (int64_t)wave * BM * 1024;
    const int64_t b_base = (int64_t)wave * 1024;
    // Copy j of a k-block (j < COPIES) moves plane c = j / (BM + 1), A part
    // j % (BM + 1) (or the B part when that is BM).
    auto issue_one = [&](const char *ak, const char *bk, char *base, auto j_c) {
        constexpr int j = decltype(j_c)::value, c = j / (BM + 1), r = j % (BM + 1);
        if constexpr (r < BM)
            copy_1k(ak + a_base + c * a_plane + r * 1024,
                    base + wave * BM * 1024 + c * K::A_BYTES + r * 1024, lane16);
        else
            copy_1k(bk + b_base + c * b_plane, base + D * K::A_BYTES + wave * 1024 + c * K::B_BYTES,
                    lane16);
    };
    // Copy cursor: the (tile, k-block) the next copies fetch; past the last
    // k-block of the last tile it stays on that k-block (in bounds, unused).
    int c_tile = 0, c_kb = 0;
    const char *c_ak, *c_bk;
    // tiles in groups of 4 tile-rows per XCD (the tiles of this kernel are up
    // to four times taller than wide; measured 1-10 % less time than groups
    // of 8 at 16384 x 16384 x 512 and 8192 x 8192 x 1024)
    auto cursor_bases = [&]() {
        int tm, tn;
        tile_coords_of<4>((int)blockIdx.x + c_tile * G, ntiles, nt_m, nt_n, tm, tn);
        c_ak = Ag + (int64_t)c_kb * RpadA * 64 + (int64_t)tm * K::MT * 64;
        c_bk = Bg + (int64_t)c_kb * RpadB * 64 + (int64_t)tn * K::NT * 64;
    };
    auto cursor_next = [&]() {
        if (c_kb + 1 < KB) {
            ++c_kb;
            c_ak += RpadA * 64;
            c_bk += RpadB * 64;
        } else if (PERSIST && c_tile + 1 < mine) {
            ++c_tile;
            c_kb = 0;
            cursor_bases();
        }
    };
    auto stage = [&](int qs) -> char * { return lds + qs * K::STAGE; };

    const int off0 = frag_offset(lane, 0), off1 = frag_offset(lane, 1);

    // Fragments of one 16-index sub-step: D planes of A (BM row blocks) and of B.
    struct Frags {
        bf16x8 a[D][BM], b[D];
    };
    const char *const At0 = lds + (wm * 32 * BM) * 64;
    const char *const Bt0 = lds + D * K::A_BYTES + (wn * 32) * 64;
    auto load = [&](int stage_off, int off, Frags &f) {
#pragma unroll
        for (int m = 0; m < D; ++m) {
            f.b[m] = lds_frag(Bt0 + stage_off + m * K::B_BYTES, off);
#pragma unroll
            for (int b = 0; b < BM; ++b)
                f.a[m][b] = lds_frag(At0 + stage_off + m * K::A_BYTES + b * 32 * 64, off);
        }
    };
    // One sub-step: the MMAS MFMAs on `cur`, the READS fragment reads of the
    // next sub-step (stage offset nso, lane offset noff) into `nxt`, and copies
    // [J0, J1) of k-block ckb into stage cdst, in slots of one MFMA, one read and
    // one copy (MFMA first: its operands were read a sub-step earlier), so that
    // reads and copies are issued while MFMAs execute.  The accumulator order
    // (q) encodes the FP64 addition order; the MFMA order inside a panel does
    // not matter (exact panel sums).
    constexpr int SLOTS = K::MMAS > K::READS ? K::MMAS : K::READS;
    auto step = [&](const Frags &cur, f32x16 (&acc)[K::P][BM], auto zero_c, int nso, int noff,
                    Frags &nxt, const char *ak, const char *bk, char *cdst, auto j0_c, auto j1_c) {
        constexpr bool zero = decltype(zero_c)::value;
        constexpr int J0 = decltype(j0_c)::value, J1 = decltype(j1_c)::value;
        static_for<(SLOTS > J1 - J0 ? SLOTS : J1 - J0)>([&](auto t_c) {
            constexpr int t = decltype(t_c)::value;
            if constexpr (t < K::MMAS) {
                constexpr int q = t / BM, b = t % BM, i = prod_i(q), j = prod_j(q);
                if constexpr (q >= K::Q_VGPR) {
                    if constexpr (zero) mfma_vacc_zero(acc[q][b], cur.a[i][b], cur.b[j]);
                    else mfma_vacc(acc[q][b], cur.a[i][b], cur.b[j]);
                } else {
                    acc[q][b] = mfma(cur.a[i][b], cur.b[j], zero ? f32x16{} : acc[q][b]);
                }
            }
            order_fence();
            if constexpr (t < K::READS) {
                constexpr int code = read_code<D, BM>(t);
                constexpr int plane = (code >> 3) & 7, blk = code & 7;
                if constexpr (code >= 64)
                    nxt.b[plane] = lds_frag(Bt0 + nso + plane * K::B_BYTES, noff);
                else
                    nxt.a[plane][blk] = lds_frag(At0 + nso + plane * K::A_BYTES + blk * 32 * 64, noff);
            }
            order_fence();
            if constexpr (t < J1 - J0)
                issue_one(ak, bk, cdst, std::integral_constant<int, J0 + t>{});
            order_fence();
        });
    };

    // Software pipeline over the workgroup's sequence of k-blocks with a ring of
    // NS LDS stages (position q in stage q mod NS).  Trip q (1) reads the
    // sub-step-1 fragments of q while the sub-step-0 MFMAs run; (2) waits until
    // at most the newest NS - 2 k-blocks of its own copies are outstanding (so
    // q + 1 has landed) and for its LDS reads, then barriers: every wave is done
    // reading stage q and every copy of q + 1 has landed; (3) issues the copies
    // of q + NS into stage q and reads the sub-step-0 fragments of q + 1 while
    // the sub-step-1 MFMAs run.  Across a tile boundary q + 1 is the next tile's
    // first k-block, already in place.
    cursor_bases();
    for (int j = 0; j < K::NSTAGE; ++j) {
        static_for<K::COPIES>([&](auto j_c) { issue_one(c_ak, c_bk, stage(j), j_c); });
        cursor_next();
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((K::NSTAGE - 2) * K::COPIES + K::COPIES) : "memory");
    __syncthreads();
    Frags f0, f1;
    load(0, off0, f0);
    int qs = 0;                        // q mod NS
    auto kblock = [&](f32x16 (&acc)[K::P][BM], auto first_c) {
        const int so = qs * K::STAGE;
        const int qn = qs + 1 == K::NSTAGE ? 0 : qs + 1;
        // sub-step 0 of q; reads sub-step 1 of q
        step(f0, acc, first_c, so, off1, f1, c_ak, c_bk, stage(qs),
             std::integral_constant<int, K::COPIES>{}, std::integral_constant<int, K::COPIES>{});
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (K::NSTAGE == 2)
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        else
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((K::NSTAGE - 2) * K::COPIES)
                         : "memory");
        pipeline_barrier();
        // sub-step 1 of q; reads sub-step 0 of q + 1; copies of q + NS into stage q
        step(f1, acc, std::false_type{}, qn * K::STAGE, off0, f0, c_ak, c_bk, stage(qs),
             std::integral_constant<int, 0>{}, std::integral_constant<int, K::COPIES>{});
        __builtin_amdgcn_sched_barrier(0);
        cursor_next();
        qs = qn;
    };

    for (int it = 0; it < mine; ++it) {
        int tm, tn;
        tile_coords_of<4>((int)blockIdx.x + it * G, ntiles, nt_m, nt_n, tm, tn);
        const int64_t m0 = (int64_t)tm * K::MT, n0 = (int64_t)tn * K::NT;
        double acc64[ACC64_LDS ? 1 : BM][16];
#pragma unroll
        for (int b = 0; b < BM; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if constexpr (ACC64_LDS)
                    acc64_lds[((wave * BM + b) * 16 + r) * 64 + lane] = 0.0;
                else
                    acc64[b][r] = 0.0;
            }
        for (int p0 = 0; p0 < KB; p0 += KB_PER_PANEL) {
            const int p1 = min(KB, p0 + KB_PER_PANEL);
            f32x16 acc[K::P][BM];
            kblock(acc, std::true_type{});
            for (int kb = p0 + 1; kb < p1; ++kb) kblock(acc, std::false_type{});
            // panel end: widen each product exactly and add it in FP64, in order
#pragma unroll
            for (int q = K::Q_VGPR; q < K::P; ++q)
#pragma unroll
                for (int b = 0; b < BM; ++b) mfma_vacc_settle(acc[q][b]);
            if constexpr (ACC64_LDS) {
                // eight elements at a time: eight independent FP64 chains keep
                // the FP64 adder busy (one element's 21 adds in a row would wait
                // on each other)
#pragma unroll
                for (int b = 0; b < BM; ++b)
#pragma unroll
                    for (int h = 0; h < 16; h += 8) {
                        double t[8];
#pragma unroll
                        for (int r = 0; r < 8; ++r)
                            t[r] = acc64_lds[((wave * BM + b) * 16 + h + r) * 64 + lane];
#pragma unroll
                        for (int q = 0; q < K::P; ++q)
#pragma unroll
                            for (int r = 0; r < 8; ++r) t[r] += (double)acc[q][b][h + r];
#pragma unroll
                        for (int r = 0; r < 8; ++r)
                            acc64_lds[((wave * BM + b) * 16 + h + r) * 64 + lane] = t[r];
                    }
            } else {
#pragma unroll
                for (int q = 0; q < K::P; ++q)
#pragma unroll
                    for (int b = 0; b < BM; ++b)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc64[b][r] += (double)acc[q][b][r];
            }
        }

        // store; with the scale-aware split the row and column weights go back
        // in here, C_mn = 2^(sa_m + sb_n) C'_mn (exact up to overflow or underflow).
        // (The lane is laundered so that the store's addresses are not hoisted
        // out of the tile loop into registers the k-loop needs.)
        int sl = lane;
        if constexpr (PERSIST) asm volatile("" : "+v"(sl));
        store_tile<BM, 16>(
            [&](int b, int r) {
                return ACC64_LDS ? acc64_lds[((wave * BM + b) * 16 + r) * 64 + sl]
                                 : acc64[ACC64_LDS ? 0 : b][r];
            },
            [&](int b, int r) { return m0 + (wm * BM + b) * 32 + acc_row(r); }, acc_lrow(sl),
            [&](int) { return n0 + wn * 32; }, sl & 31, m0 + K::MT <= M && n0 + K::NT <= N, M, N, C,
            ldc, alpha, beta, sa, sb);
    }
    // the last trips issued (unused) copies: let them land before the workgroup
    // ends and its LDS is handed to another workgroup
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

}  // namespace

template <int D, int BM, int NS, bool ACC64_LDS>
hipError_t launch_s(const DgemmArgs &a, hipStream_t s) {
    using K = Cfg<D, BM, NS, ACC64_LDS>;
    const int nt_m = (int)((a.M + K::MT - 1) / K::MT), nt_n = (int)((a.N + K::NT - 1) / K::NT);
    const int ntiles = nt_m * nt_n;
    // short reductions: persistent workgroups (as in launch_w; every k-block
    // starts on f0, so any number of k-blocks works).  A separate
    // instantiation, so that the one-tile kernel of long reductions carries
    // none of the tile-walking code (it cost up to 7 % at 8192 for d = 5).
    const int pw = persistent_workgroups();
    if (a.KB <= 32 && ntiles > pw)
        gemm_f64_kernel<D, BM, NS, ACC64_LDS, true><<<pw, 256, 0, s>>>(
            a.Ap, a.Bp, a.C, a.M, a.N, (int)a.KB, a.RpadA, a.RpadB, a.ldc, a.sa, a.sb, a.alpha, a.beta, nt_m, nt_n, ntiles, a.skip_if);
    else
        gemm_f64_kernel<D, BM, NS, ACC64_LDS, false><<<ntiles, 256, 0, s>>>(
            a.Ap, a.Bp, a.C, a.M, a.N, (int)a.KB, a.RpadA, a.RpadB, a.ldc, a.sa, a.sb, a.alpha, a.beta, nt_m, nt_n, ntiles, a.skip_if);
    return hipGetLastError();
}

template hipError_t launch_s<1, 4, 4, false>(const DgemmArgs &, hipStream_t);
template hipError_t launch_s<2, 2, 4, false>(const DgemmArgs &, hipStream_t);
template hipError_t launch_s<3, 2, 3, false>(const DgemmArgs &, hipStream_t);
template hipError_t launch_s<4, 1, 3, false>(const DgemmArgs &, hipStream_t);
template hipError_t launch_s<5, 1, 3, true>(const DgemmArgs &, hipStream_t);

}  // namespace emu
