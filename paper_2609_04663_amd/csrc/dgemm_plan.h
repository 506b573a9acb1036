// Host-side plan of an emulated DGEMM: which kernel runs it and how its packed
// operands lie in the workspace.  Plain C++ without HIP, so that the sizes can
// be checked by a host program.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace emu {

constexpr int KBLK = 32;        // reduction indices per k-block (one LDS stage)
constexpr int ROW_GROUP = 64;   // packed rows are padded to a multiple of this ...
constexpr int KPANEL = 256;     // reduction panel B_K of the FP32/FP64 reconstruction
constexpr int KB_PER_PANEL = KPANEL / KBLK;

// ... and of the GEMM tile that reads them (output tile rows for A, columns for B).
constexpr int DGEMM_NT = 64;
// Slices of each operand that the products of depth d read (indices < 6).
inline int dgemm_planes(int d) { return d < 6 ? d : 6; }

// Memory-channel staggering of the packed operands.  With power-of-two sizes
// the k-block stride (Rpad x 64 B) and the plane stride are multiples of a
// large power of two, and every copy of a tile's k-block (all planes) lands in
// the same few L2 channels.  Two skews break that: Rpad gets ROW_SKEW_TILES
// extra tiles (never read by the GEMM), and consecutive planes are PLANE_SKEW elements further
// apart than their KB x Rpad x 32 elements (a multiple of 512: planes stay
// 1 KB aligned).
constexpr int ROW_SKEW_TILES = 2;
constexpr int64_t PLANE_SKEW = 2048;

// Elements from one component plane to the next.
constexpr int64_t plane_elems(int64_t KB, int64_t Rpad) { return KB * Rpad * KBLK + PLANE_SKEW; }

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

struct Shape {
    int64_t KB, RpadA, RpadB, RliveA, RliveB;
    size_t bytesA, bytesB;
};

// Packed sizes: rows padded to whole GEMM tiles (tile_m, tile_n are multiples
// of ROW_GROUP), reduction padded to whole k-blocks.
inline Shape plan(int64_t M, int64_t N, int64_t K, int nplanes, int64_t tile_m, int64_t tile_n,
                  int64_t KB = 0) {
    Shape s;
    s.KB = KB > 0 ? KB : (K + KBLK - 1) / KBLK;
    s.RliveA = round_up(M, tile_m);
    s.RliveB = round_up(N, tile_n);
    s.RpadA = s.RliveA + ROW_SKEW_TILES * tile_m;
    s.RpadB = s.RliveB + ROW_SKEW_TILES * tile_n;
    s.bytesA = (size_t)nplanes * plane_elems(s.KB, s.RpadA) * 2;
    s.bytesB = (size_t)nplanes * plane_elems(s.KB, s.RpadB) * 2;
    return s;
}

// Persistent grid of the DGEMM kernels: one workgroup per CU (their LDS use
// allows one), rounded down to a multiple of 8.
inline int persistent_workgroups(int cus) { return cus < 8 ? 8 : cus / 8 * 8; }

// Blocks of 64 tile rows of the panel kernel (32 x 32 x 16 MFMA over whole panels).
constexpr int t_bm(int d) { return d == 6 || d == 5 ? 1 : d == 4 || d == 3 ? 2 : 0; }

// Reductions that the panel kernel also gets where it only measured faster for
// most sizes; longer ones are always its own.
constexpr int64_t SHORT_KB = 32;

// Whether a depth-d DGEMM of an M x N output with KB k-blocks of data is to run
// on the panel kernel: d = 3 .. 6, at least a panel, and (64 BM) x 64 tiles that
// fill the CUs (smaller grids keep the kernels with smaller tiles).  It pads
// the reduction to whole panels: always worth it for K > 1024.  Shorter
// reductions take it where two rules hold:
//   * the padding costs less than the kernel gains over the others on whole
//     panels (16384 x 16384 x 512: 3 / 8 / 30 / 15 % for d = 3 .. 6; 3000 x 5000
//     x 300, padded to 512, was 12 / 22 % slower at d = 3 / 4, 13 % faster at
//     d = 5 and 15 % slower at d = 6);
//   * its rounds of workgroups cost no more than those of the kernel it replaces.
//     For d = 3 and 5 that one has the same tiles, for d = 4 and 6 tiles of half
//     the height, so that a panel round counts as two of them, over the gain
//     per round (d = 4 17 %, d = 6 25 %).  Product GEMM at K = 1024, other kernel / panel
//     kernel, us (rounds): d = 4, 1344 x 1536 44.8 (2) / 67.1 (2), 1600 x 1600 61.3 (3)
//     / 67.0 (2), 2176 x 1536 80.9 (4) / 68.0 (2), 3000 x 3000 178.9 (9) / 168.3 (5);
//     d = 6, 1088 x 1024 66.1 (3) / 68.7 (2), 1280 x 1280 86.4 (4) / 69.2 (2),
//     1472 x 1472 106.4 (5) / 103.9 (3).
inline bool panel_kernel_wanted(int d, int64_t M, int64_t N, int64_t KB, int cus) {
    if (d < 3 || d > 6 || KB < KB_PER_PANEL) return false;
    const int64_t mt = 64 * t_bm(d), nt_n = (N + DGEMM_NT - 1) / DGEMM_NT;
    const int64_t pw = persistent_workgroups(cus), tiles = (M + mt - 1) / mt * nt_n;
    if (tiles < pw) return false;
    if (KB > SHORT_KB) return true;
    constexpr int gain[7] = {0, 0, 0, 103, 107, 160, 112};         // per cent
    constexpr int round_gain[7] = {0, 0, 0, 0, 117, 0, 125};
    const int64_t padded = round_up(KB, KB_PER_PANEL);
    if (padded * 100 > KB * gain[d]) return false;
    if (d == 3 || d == 5) return true;
    const int64_t rounds = (tiles + pw - 1) / pw;
    const int64_t half_tiles = (M + mt / 2 - 1) / (mt / 2) * nt_n;
    return rounds * 2 * padded * 100 <= (half_tiles + pw - 1) / pw * KB * round_gain[d];
}

// Scale-aware split scratch: 64-bit maxima for the nA rows of A and the nB
// columns of B, then their int32 exponents.
inline size_t scale_bytes(int64_t nA, int64_t nB) { return 256 + (size_t)(nA + nB) * 12; }

// Workspace areas of one emulated DGEMM after the header: packed planes, then
// (256-byte aligned) the weights of the scale-aware split.
struct DgemmLayout {
    Shape s;
    bool panels;                // for the panel kernel (whole zero-padded panels)
    size_t scale_off, bytes;
};

inline DgemmLayout dgemm_layout_for(bool panels, int d, int64_t M, int64_t N, int64_t K,
                                    bool scaled) {
    DgemmLayout L;
    const int64_t KB = (K + KBLK - 1) / KBLK;
    L.panels = panels;
    // A's tile rows; without the panel kernel a multiple of every other kernel's tile
    L.s = plan(M, N, K, dgemm_planes(d), panels ? 64 * t_bm(d) : d == 1 ? 256 : d <= 3 ? 128 : 64,
               DGEMM_NT, panels ? round_up(KB, KB_PER_PANEL) : KB);
    auto up = [](size_t x) { return (x + 255) / 256 * 256; };
    L.scale_off = up(L.s.bytesA + L.s.bytesB);
    L.bytes = up(L.scale_off + (scaled ? scale_bytes(M, N) : 0));
    return L;
}

// The layout for the kernel that suits the size.  A short reduction for which it
// takes more than `limit` bytes gets the layout of the other kernels, which is
// never larger than the panel kernel's (all kernels give the same bits).
inline DgemmLayout dgemm_layout(int d, int64_t M, int64_t N, int64_t K, bool scaled, int cus,
                                size_t limit = (size_t)-1) {
    const int64_t KB = (K + KBLK - 1) / KBLK;
    DgemmLayout L = dgemm_layout_for(panel_kernel_wanted(d, M, N, KB, cus), d, M, N, K, scaled);
    if (L.panels && KB <= SHORT_KB && L.bytes > limit)
        L = dgemm_layout_for(false, d, M, N, K, scaled);
    return L;
}

// A group of kb <= K reduction indices of a K-binned DGEMM whose groups share
// the area of `area` bytes that a layout of the whole reduction takes.  A shorter
// reduction may suit the panel kernel where the whole one does not (d = 4: 25
// k-blocks pad to 32, 24 to 24, in tiles twice as tall) and would then need more
// than the area; it takes the other kernels' layout, whose size grows with kb.
inline DgemmLayout kbin_group_layout(int d, int64_t M, int64_t N, int64_t kb, int cus,
                                     size_t area) {
    return dgemm_layout(d, M, N, kb, true, cus, area);
}

}  // namespace emu
