// Emulated DGEMM on 16 x 16 blocks (see gemm_f64.hip for the method).
// Depths d = 6 .. 11 (21 .. 36 products, every slice of both operands).  For
// d >= 7 a 32 x 32 wave tile would need 16 N_p accumulator registers per lane,
// more than the register file holds, so these depths use the 16 x 16 x 32 MFMA
// on a 16 x 32 wave tile (BMW = 1: two 16 x 16 blocks along N): 8 registers
// per product.  Workgroup: 4 waves in a 2 x 2 grid, output tile 32 x 64; one
// k-block of 32 reduction indices (one MFMA depth) per trip and one barrier
// per trip, with the copies and fragment reads spread over the trip's MFMAs
// and copies issued two trips ahead.  d = 6 runs here too where the
// panel kernel (gemm_f64t.hip) does not suit: small grids, reductions that pad
// badly to whole panels or need fewer rounds of these smaller tiles.
// Depths d <= 5 (d planes per operand) can take a 32 x 32 wave tile here
// (BMW = 2: 2 x 2 blocks, 16 registers per product, output tile 64 x 64) or,
// with few products, 64 x 32 (BMW = 4, output tile 128 x 64).
#include "gemm_f64.h"

namespace emu {
namespace {

template <int D, int NS, bool ACC64_LDS, int BMW>
struct CfgW {
    static constexpr int P = n_prod(D);
    static constexpr int NPL = D < 6 ? D : 6;                        // slices read per operand
    // FP64 accumulator tile in LDS (8 BMW doubles per lane) instead of VGPRs
    static constexpr int ACC64_BYTES = ACC64_LDS ? 4 * 64 * 8 * BMW * 8 : 0;
    static constexpr int MT = 32 * BMW, NT = 64;                     // wave tile 16 BMW x 32
    static constexpr int A_BYTES = MT * 64, B_BYTES = NT * 64;       // one plane of a stage
    static constexpr int STAGE = NPL * (A_BYTES + B_BYTES);
    static constexpr int COPIES = STAGE / 1024 / 4;                  // 1 KB copies per wave
    static constexpr int A_COPIES = NPL * MT / 16 / 4;               // the first ones move A
    static constexpr int READS = NPL * (BMW + 2);                    // A: BMW blocks, B: 2
    static constexpr int MMAS = 2 * BMW * P;
    // AGPRs hold 32 / BMW products of 2 BMW blocks; later products use VGPRs
    static constexpr int Q_VGPR = P > 32 / BMW ? 32 / BMW : P;
    static_assert(BMW == 1 || BMW == 2 || BMW == 4, "wave tile");
    static_assert(4 * COPIES * 1024 == STAGE && 4 * A_COPIES * 1024 == NPL * A_BYTES,
                  "copy split");
    static_assert(BMW != 1 || NPL % 2 == 0, "one-block tiles copy planes in pairs");
    static_assert(NS * STAGE + ACC64_BYTES <= 160 * 1024, "LDS");
};

// Read t of a trip loads the t-th distinct fragment in order of first use by
// the trip's MFMA sequence (product q on block b for MFMA 2 q + b), encoded as
// 64 * is_B + 8 * plane + block.
template <int D, int BMW>
constexpr int read_code_w(int t) {
    bool seen_a[6][4] = {}, seen_b[6][2] = {};
    int r = 0;
    for (int u = 0; u < 2 * BMW * n_prod(D); ++u) {
        const int q = u / (2 * BMW), a = (u % (2 * BMW)) / 2, b = u % 2, i = prod_i(q),
                  j = prod_j(q);
        if (!seen_a[i][a]) {
            seen_a[i][a] = true;
            if (r++ == t) return 8 * i + a;
        }
        if (!seen_b[j][b]) {
            seen_b[j][b] = true;
            if (r++ == t) return 64 + 8 * j + b;
        }
    }
    return -1;
}

template <int D, int NS, bool ACC64_LDS, bool PERSIST, int BMW>
__global__ __launch_bounds__(256, 1) void gemm_f64w_kernel(
    const uint16_t *__restrict__ Ap, const uint16_t *__restrict__ Bp, double *__restrict__ C,
    int64_t M, int64_t N, int KB, int64_t RpadA, int64_t RpadB, int64_t ldc,
    const int *__restrict__ sa, const int *__restrict__ sb, double alpha, double beta, int nt_m,
    int nt_n, int ntiles, const unsigned *__restrict__ skip_if) {
    if (skip_if != nullptr && *skip_if != 0u) return;
    using K = CfgW<D, NS, ACC64_LDS, BMW>;
    __shared__ __attribute__((aligned(1024))) char lds[NS * K::STAGE + K::ACC64_BYTES];
    // lane-private FP64 accumulators in LDS: element e = 4 (2 a + b) + r of
    // lane l of wave w at (w * 8 BMW + e) * 64 + l
    double *acc64_lds = reinterpret_cast<double *>(lds + NS * K::STAGE);

    // Persistent workgroups: workgroup w0 of G takes tiles w0, w0 + G, ... (its
    // `mine` tiles), walking one sequence of k-blocks tile after tile, so the
    // copy ring runs on into the next tile's first k-blocks while a tile's
    // FP64 epilogue and store execute.
    const int G = gridDim.x;
    const int mine = PERSIST ? (ntiles - 1 - (int)blockIdx.x) / G + 1 : 1;
    const int lane = threadIdx.x & 63;
    const unsigned lane16 = (unsigned)lane * 16u;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    const char *Ag = reinterpret_cast<const char *>(Ap);
    const char *Bg = reinterpret_cast<const char *>(Bp);
    const int64_t a_plane = plane_elems(KB, RpadA) * 2;
    const int64_t b_plane = plane_elems(KB, RpadB) * 2;

    // Copy c of a k-block by wave w moves 1 KB part g = 4 c + w of the list
    // A parts (plane-major, 2 BMW parts a plane), then B parts: for BMW = 1,
    // c < A_COPIES moves part (w & 1) of A plane 2 c + (w >> 1); for BMW >= 2,
    // c < A_COPIES moves part 4 (c % (BMW / 2)) + w of A plane c / (BMW / 2);
    // the rest move part w of B plane c - A_COPIES.
    // ak, bk: the k-block's slab of plane 0 at the copied tile's first row.
    const int64_t a_off = BMW == 1 ? (int64_t)(wave >> 1) * a_plane + (wave & 1) * 1024
                                   : (int64_t)wave * 1024;
    const int a_dst = BMW == 1 ? (wave >> 1) * K::A_BYTES + (wave & 1) * 1024 : wave * 1024;
    const int64_t b_off = (int64_t)wave * 1024;
    const int b_dst = K::NPL * K::A_BYTES + wave * 1024;
    auto issue_one = [&](const char *ak, const char *bk, char *base, auto c_c) {
        constexpr int c = decltype(c_c)::value;
        // compile-time part of copy c's A offsets
        constexpr int a_pl = BMW == 1 ? 2 * c : c / (BMW > 1 ? BMW / 2 : 1);
        constexpr int a_pt = BMW == 1 ? 0 : 4 * (c % (BMW > 1 ? BMW / 2 : 1));
        if constexpr (c < K::A_COPIES)
            copy_1k(ak + a_off + a_pl * a_plane + a_pt * 1024,
                    base + a_dst + a_pl * K::A_BYTES + a_pt * 1024, lane16);
        else
            copy_1k(bk + b_off + (c - K::A_COPIES) * b_plane,
                    base + b_dst + (c - K::A_COPIES) * K::B_BYTES, lane16);
    };
    // Copy cursor: the (tile, k-block) the next copies fetch; past the last
    // k-block of the last tile it stays on that k-block (in bounds, unused).
    int c_tile = 0, c_kb = 0;
    const char *c_ak, *c_bk;
    auto cursor_bases = [&]() {
        int tm, tn;
        tile_coords_of<8>((int)blockIdx.x + c_tile * G, ntiles, nt_m, nt_n, tm, tn);
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

    // lane's fragment offset inside a 16-row block: row l % 16, chunk l / 16
    const int frow = lane & 15;
    const int foff = frow * 64 + (((lane >> 4) ^ swz(frow)) << 4);
    const char *const At0 = lds + (wm * 16 * BMW) * 64 + foff;
    const char *const Bt0 = lds + K::NPL * K::A_BYTES + (wn * 32) * 64 + foff;

    struct Frags {
        bf16x8 a[K::NPL][BMW], b[K::NPL][2];
    };
    auto read_one = [&](int so, Frags &f, auto t_c) {
        constexpr int code = read_code_w<D, BMW>(decltype(t_c)::value);
        constexpr int plane = (code >> 3) & 7, blk = code & 7;
        if constexpr (code >= 64)
            f.b[plane][blk] =
                *reinterpret_cast<const bf16x8 *>(Bt0 + so + plane * K::B_BYTES + blk * 16 * 64);
        else
            f.a[plane][blk] =
                *reinterpret_cast<const bf16x8 *>(At0 + so + plane * K::A_BYTES + blk * 16 * 64);
    };

    // One trip: the MMAS MFMAs on `cur`; read t of the next k-block (stage
    // offset nso) at slot RS t; copy c of k-block ckb into stage cdst at slot
    // CS c + 2 (reads and copies spread over the MFMA stream).
    constexpr int SLOTS = K::MMAS;
    constexpr int RS = SLOTS >= 2 * K::READS ? 2 : 1;
    constexpr int CS = (SLOTS - 2) / K::COPIES;
    static_assert(RS * (K::READS - 1) < SLOTS && CS >= 1, "slots");
    auto trip = [&](const Frags &cur, f32x4 (&acc)[K::P][2 * BMW], auto zero_c, int nso,
                    Frags &nxt, const char *ak, const char *bk, char *cdst) {
        constexpr bool zero = decltype(zero_c)::value;
        static_for<SLOTS>([&](auto t_c) {
            constexpr int t = decltype(t_c)::value;
            // product q on block e = 2 a + b (A block a, B block b)
            constexpr int q = t / (2 * BMW), e = t % (2 * BMW), a = e / 2, b = e % 2;
            constexpr int i = prod_i(q), j = prod_j(q);
            if constexpr (q >= K::Q_VGPR) {
                if constexpr (zero) mfma16_vacc_zero(acc[q][e], cur.a[i][a], cur.b[j][b]);
                else mfma16_vacc(acc[q][e], cur.a[i][a], cur.b[j][b]);
            } else {
                acc[q][e] = mfma16(cur.a[i][a], cur.b[j][b], zero ? f32x4{} : acc[q][e]);
            }
            order_fence();
            if constexpr (t % RS == 0 && t / RS < K::READS)
                read_one(nso, nxt, std::integral_constant<int, t / RS>{});
            order_fence();
            if constexpr (t >= 2 && (t - 2) % CS == 0 && (t - 2) / CS < K::COPIES)
                issue_one(ak, bk, cdst, std::integral_constant<int, (t - 2) / CS>{});
            order_fence();
        });
    };

    // Ring of NS stages; the k-block at position q of the workgroup's sequence
    // sits in stage q mod NS.  Trip q starts once every wave's copies of q + 1
    // have landed and every wave has read q into registers (one barrier); it
    // then runs the MFMAs of q, reads q + 1 and issues the copies of q + NS into
    // the stage of q.  Across a tile boundary q + 1 is the next tile's first
    // k-block, already in place, so only the first tile waits for a fill.
    cursor_bases();
    for (int j = 0; j < NS; ++j) {
        static_for<K::COPIES>([&](auto c_c) { issue_one(c_ak, c_bk, stage(j), c_c); });
        cursor_next();
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * K::COPIES) : "memory");
    __syncthreads();
    Frags f0, f1;
    static_for<K::READS>([&](auto t_c) { read_one(0, f0, t_c); });
    int qs = 0;                        // q mod NS
    auto one = [&](const Frags &cur, Frags &nxt, f32x4 (&acc)[K::P][2 * BMW], auto zero_c) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * K::COPIES) : "memory");
        pipeline_barrier();
        const int qn = qs + 1 == NS ? 0 : qs + 1;
        trip(cur, acc, zero_c, qn * K::STAGE, nxt, c_ak, c_bk, stage(qs));
        __builtin_amdgcn_sched_barrier(0);
        cursor_next();
        qs = qn;
    };

    for (int it = 0; it < mine; ++it) {
        int tm, tn;
        tile_coords_of<8>((int)blockIdx.x + it * G, ntiles, nt_m, nt_n, tm, tn);
        const int64_t m0 = (int64_t)tm * K::MT, n0 = (int64_t)tn * K::NT;
        double acc64[2 * BMW][4];
#pragma unroll
        for (int e = 0; e < 2 * BMW; ++e)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                acc64[e][r] = 0.0;
                if constexpr (ACC64_LDS)
                    acc64_lds[(wave * 8 * BMW + 4 * e + r) * 64 + lane] = 0.0;
            }
        // trips alternate the fragment buffers: a panel starts on f0 (panels
        // have even length, except the last panel of a tile when KB is odd,
        // and then the workgroup has one tile)
        for (int p0 = 0; p0 < KB; p0 += KB_PER_PANEL) {
            const int p1 = min(KB, p0 + KB_PER_PANEL);
            f32x4 acc[K::P][2 * BMW];
            int kb = p0;
            one(f0, f1, acc, std::true_type{});
            for (++kb; kb < p1; ++kb) {
                one(f1, f0, acc, std::false_type{});
                if (++kb < p1) one(f0, f1, acc, std::false_type{});
            }
            // panel end: widen each product exactly and add it in FP64, in order
#pragma unroll
            for (int q = K::Q_VGPR; q < K::P; ++q)
#pragma unroll
                for (int e = 0; e < 2 * BMW; ++e) mfma16_vacc_settle(acc[q][e]);
            // 8 BMW independent FP64 chains, products in order
            if constexpr (ACC64_LDS) {
#pragma unroll
                for (int x = 0; x < 8 * BMW; ++x)
                    acc64[x / 4][x % 4] = acc64_lds[(wave * 8 * BMW + x) * 64 + lane];
            }
#pragma unroll
            for (int q = 0; q < K::P; ++q)
#pragma unroll
                for (int e = 0; e < 2 * BMW; ++e)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc64[e][r] += (double)acc[q][e][r];
            if constexpr (ACC64_LDS) {
#pragma unroll
                for (int x = 0; x < 8 * BMW; ++x)
                    acc64_lds[(wave * 8 * BMW + x) * 64 + lane] = acc64[x / 4][x % 4];
            }
        }

        // a column holds the 4 BMW values of BMW 16-row blocks (the lane is
        // laundered as in gemm_f64_kernel)
        int sl = lane;
        if constexpr (PERSIST) asm volatile("" : "+v"(sl));
        store_tile<2, 4 * BMW>(
            [&](int b, int r) { return acc64[2 * (r / 4) + b][r % 4]; },
            [&](int, int r) { return m0 + wm * 16 * BMW + (r / 4) * 16 + r % 4; }, (sl >> 4) * 4,
            [&](int b) { return n0 + wn * 32 + b * 16; }, sl & 15,
            m0 + K::MT <= M && n0 + K::NT <= N, M, N, C, ldc, alpha, beta, sa, sb);
    }
    // the last trips issued (unused) copies: let them land before the workgroup
    // ends and its LDS is handed to another workgroup
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

}  // namespace

template <int D, int NS, bool ACC64_LDS, int BMW, bool PERSIST_OK>
hipError_t launch_w(const DgemmArgs &a, hipStream_t s) {
    using K = CfgW<D, NS, ACC64_LDS, BMW>;
    const int nt_m = (int)((a.M + K::MT - 1) / K::MT), nt_n = (int)((a.N + K::NT - 1) / K::NT);
    const int ntiles = nt_m * nt_n;
    // Short reductions (K <= 1024): one persistent workgroup per CU (a
    // multiple of 8: every workgroup keeps its XCD), so the next tile's first
    // copies overlap a tile's epilogue and store (measured at 16384^2 x 512,
    // d = 6: 17 % less time).  Longer reductions: one workgroup per tile
    // (persistent was 4-9 % slower at K = 8192; a separate instantiation keeps
    // their kernel free of the tile-walking code).  With an odd number of
    // k-blocks a second tile would start on the other fragment buffer, so
    // those always take one tile per workgroup.
    const int pw = persistent_workgroups();
    if constexpr (PERSIST_OK) {
        if (a.KB % 2 == 0 && a.KB <= 32 && ntiles > pw) {
            gemm_f64w_kernel<D, NS, ACC64_LDS, true, BMW><<<pw, 256, 0, s>>>(
                a.Ap, a.Bp, a.C, a.M, a.N, (int)a.KB, a.RpadA, a.RpadB, a.ldc, a.sa, a.sb, a.alpha, a.beta, nt_m, nt_n,
                ntiles, a.skip_if);
            return hipGetLastError();
        }
    }
    gemm_f64w_kernel<D, NS, ACC64_LDS, false, BMW><<<ntiles, 256, 0, s>>>(
        a.Ap, a.Bp, a.C, a.M, a.N, (int)a.KB, a.RpadA, a.RpadB, a.ldc, a.sa, a.sb, a.alpha, a.beta, nt_m, nt_n, ntiles, a.skip_if);
    return hipGetLastError();
}

template hipError_t launch_w<1, 4, false, 2>(const DgemmArgs &, hipStream_t);
template hipError_t launch_w<1, 4, false, 4, false>(const DgemmArgs &, hipStream_t);
template hipError_t launch_w<2, 4, false, 2>(const DgemmArgs &, hipStream_t);
template hipError_t launch_w<3, 4, false, 2>(const DgemmArgs &, hipStream_t);
template hipError_t launch_w<4, 4, false, 2, false>(const DgemmArgs &, hipStream_t);
template hipError_t launch_w<4, 4, false, 1, false>(const DgemmArgs &, hipStream_t);
template hipError_t launch_w<5, 3, true, 2, false>(const DgemmArgs &, hipStream_t);
template hipError_t launch_w<6, 4, false>(const DgemmArgs &, hipStream_t);
template hipError_t launch_w<7, 3, false>(const DgemmArgs &, hipStream_t);
template hipError_t launch_w<8, 3, true>(const DgemmArgs &, hipStream_t);
template hipError_t launch_w<9, 3, true>(const DgemmArgs &, hipStream_t);
template hipError_t launch_w<10, 3, true>(const DgemmArgs &, hipStream_t);
template hipError_t launch_w<11, 3, true>(const DgemmArgs &, hipStream_t);

}  // namespace emu
