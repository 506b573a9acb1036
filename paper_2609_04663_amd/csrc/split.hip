// Split/pack kernels: FP32 three-component split (Eq. fp32split, Sec. 4.2) and
// FP64 fixed six-slice simplified Ozaki split (Eq. fp64split, Sec. 4.3), each
// writing BF16 component planes in the packed MFMA operand format described
// in emu_internal.h.  Work item: one 16-byte packed chunk (8 consecutive
// reduction indices of one packed row), so every output store is a 16-byte
// vector store and a wave writes 1 KB contiguously per component.
#include "emu_internal.h"

namespace emu {
namespace {

constexpr int SPLIT_THREADS = 256;
constexpr int ROWS_PER_BLOCK = 64;    // 64 packed rows x 4 chunks = 256 work items

// Zeros that the loads of entries outside an operand read.
__device__ double g_zero8_f64[8];

__device__ inline unsigned block_or(unsigned v) {
    // OR within the wave, then one atomic per wave.
    for (int off = 32; off > 0; off >>= 1) v |= __shfl_xor(v, off);
    return v;
}

// Decode a (k-block, row-group) pair of SPLIT_THREADS threads and the thread's row/chunk.
struct ItemCoords {
    int64_t kb, prow;
    int q;
};

__device__ inline ItemCoords item_coords(int64_t pair, int RG) {
    ItemCoords c;
    c.kb = pair / RG;
    int64_t rg = pair - c.kb * RG;
    c.prow = rg * ROWS_PER_BLOCK + (threadIdx.x % SPLIT_THREADS >> 2);
    c.q = threadIdx.x & 3;
    return c;
}

// ---------------------------------------------------------------------------
// FP32: A_r = fl_BF16(A^(r)), A^(r+1) = fl_32(A^(r) - A_r), r = 0, 1, 2.
// AS_B = false: X is rows x cols (an A operand, packed row = X row, k = col).
// AS_B = true : X is rows x cols = K x N (a B operand, packed row = column n,
//               k = X row), i.e. B is packed transposed.
// Blocks [b0, b0 + nb) of the launch serve one operand, block b of them the
// items b, b + nb, ...
template <bool AS_B>
__device__ __forceinline__ void split_f32_operand(const float *__restrict__ X, int64_t rows,
                                                  int64_t cols, int64_t ldx, u16 *__restrict__ P,
                                                  int64_t KB, int64_t Rpad, int64_t Rlive,
                                                  unsigned *__restrict__ status, int b, int nb) {
    const int RG = (int)(Rlive / ROWS_PER_BLOCK);
    const int64_t npairs = KB * RG;
    const int64_t prow_lim = AS_B ? cols : rows;
    const int64_t k_lim = AS_B ? rows : cols;
    unsigned st = 0;
    for (int64_t pair = b; pair < npairs; pair += nb) {
        const ItemCoords ic = item_coords(pair, RG);
        const int64_t k0 = ic.kb * KBLK + ic.q * 8;
        float x[8];
        if (!AS_B) {
            const float *src = X + ic.prow * ldx + k0;
            const bool full = ic.prow < prow_lim && k0 + 8 <= k_lim;
            if (full && ((reinterpret_cast<uintptr_t>(src) & 15u) == 0)) {
                const float4 v0 = *reinterpret_cast<const float4 *>(src);
                const float4 v1 = *reinterpret_cast<const float4 *>(src + 4);
                x[0] = v0.x; x[1] = v0.y; x[2] = v0.z; x[3] = v0.w;
                x[4] = v1.x; x[5] = v1.y; x[6] = v1.z; x[7] = v1.w;
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    x[i] = (ic.prow < prow_lim && k0 + i < k_lim) ? src[i] : 0.0f;
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                x[i] = (ic.prow < prow_lim && k0 + i < k_lim) ? X[(k0 + i) * ldx + ic.prow] : 0.0f;
        }
        u16x8 c0, c1, c2;
        split3_f32x8(x, c0, c1, c2, st);
        *reinterpret_cast<u16x8 *>(P + packed_index(0, ic.kb, ic.prow, ic.q, KB, Rpad)) = c0;
        *reinterpret_cast<u16x8 *>(P + packed_index(1, ic.kb, ic.prow, ic.q, KB, Rpad)) = c1;
        *reinterpret_cast<u16x8 *>(P + packed_index(2, ic.kb, ic.prow, ic.q, KB, Rpad)) = c2;
    }
    st = block_or(st);
    if ((threadIdx.x & 63) == 0 && st) atomicOr(status, st);
}

// Operands of one FP32 split launch (the GEMM splits A and B together).
struct F32SplitArgs {
    F32SplitOperand op[2];
    int nops;
    int blocks0;          // blocks of operand 0; the rest serve operand 1
    int64_t KB;
    unsigned *status;
};

__global__ __launch_bounds__(SPLIT_THREADS) void split_f32_kernel(F32SplitArgs a) {
    const bool second = a.nops > 1 && (int)blockIdx.x >= a.blocks0;
    const F32SplitOperand &op = second ? a.op[1] : a.op[0];
    const int b = (int)blockIdx.x - (second ? a.blocks0 : 0);
    const int nb = second ? (int)gridDim.x - a.blocks0 : a.blocks0;
    if (op.as_b)
        split_f32_operand<true>(op.X, op.rows, op.cols, op.ldx, op.P, a.KB, op.Rpad, op.Rlive, a.status, b, nb);
    else
        split_f32_operand<false>(op.X, op.rows, op.cols, op.ldx, op.P, a.KB, op.Rpad, op.Rlive, a.status, b, nb);
}

// ---------------------------------------------------------------------------
// FP64 split.  The operand-wide maximum of every level is a global reduction;
// instead of six dependent passes the split speculates the exponent chain
// v_(r+1) = v_r - step (step = 9 for the symmetric projection, 8 for the
// literal one) and records the true maxima of the residuals it produces.
// Three launches:
//   f64_maxabs_kernel   the level-0 maximum, one partial per block;
//   split_f64_kernel    every block reduces those partials, speculates the
//                       chain, writes all slices, leaves its maxima of the
//                       levels and marks the levels whose exponent it confirms,
//                       finds too small (only where slices are subnormal: they
//                       are rounded coarser than the projection) or not zero;
//   f64_replay_kernel   returns at once when the marks decide every level (the
//                       largest residual has the speculated exponent, or the
//                       level and all after it are zero).  Otherwise
//                       it reduces the recorded maxima, takes the true exponent
//                       of the first wrong level (exact: every earlier level
//                       was computed with verified exponents), re-speculates
//                       the levels after it and recomputes them, pass by pass
//                       until the chain holds; every pass fixes at least one
//                       more level.
// The partial maxima sit in the row skew of the planes (rows Rlive .. Rpad of
// k-block 0, which no GEMM reads), so they cost no workspace and no atomics:
// 4096 blocks' maxima of two levels on two cache lines took 12 of the split
// pass's 42 us at 2048^3 (d = 3).

constexpr int MAX_THREADS = 512;      // threads and blocks per operand of the maximum
constexpr int MAX_BLOCKS = 256;
constexpr int SPLIT_BLOCKS = 1024;    // blocks per operand of the split pass
constexpr int REPLAY_THREADS = 512;   // threads of a replay block: ITEMS items at a time
constexpr int REPLAY_ITEMS = REPLAY_THREADS / SPLIT_THREADS;
// the row skew of one k-block holds a partial per block (tiles have >= 64 rows)
static_assert(ROW_SKEW_TILES * ROW_GROUP * KBLK * 2 >= SPLIT_BLOCKS * 8 && SPLIT_BLOCKS >= MAX_BLOCKS,
              "partial maxima");

__device__ inline int ceil_log2_pos(double m) {
    int e;
    const double f = frexp(m, &e);
    return (f == 0.5) ? e - 1 : e;
}

__device__ inline unsigned long long dbits(double x) {
    return (unsigned long long)__double_as_longlong(x);
}

// Marks of the split pass in F64SplitState::seen, bit r of each for level r: some
// block's maximum has the speculated exponent, a larger one, or is not zero.
__device__ inline unsigned seen_hit(unsigned long long levels) { return (unsigned)levels; }
__device__ inline unsigned seen_above(unsigned long long levels) { return (unsigned)levels << 8; }
__device__ inline unsigned seen_nonzero(unsigned long long levels) { return (unsigned)levels << 16; }

// Operands of one launch and the split of its grid between them.
struct F64SplitArgs {
    F64SplitOperand op[2];
    int nops;
    int blocks0, blocks1; // blocks of operand 0; the rest serve operand 1
    int max0, max1;       // partial level-0 maxima of the operands
    int64_t KB;
    unsigned *status;
    int dcheck;           // depth d of the product set to range-check (A = op 0,
                          // B = op 1), or 0 for none
    int mode;             // EMU_SPLIT_*
    int units0;           // replay work units of operand 0; the rest serve operand 1
};

// Eq. (bf16rangefp64): nonzero magnitudes from 2^-126 to (2 - 2^-7) 2^127.
constexpr double DOMAIN_LO = 0x1p-126, DOMAIN_HI = 0x1.fep127;

// The block's operand (selected, not indexed, so that the arguments stay in the
// kernel-argument segment), its block index and block count within it.
__device__ inline const F64SplitOperand &operand_of_block(const F64SplitArgs &a, int &b, int &nb) {
    const bool second = a.nops > 1 && (int)blockIdx.x >= a.blocks0;
    b = (int)blockIdx.x - (second ? a.blocks0 : 0);
    nb = second ? a.blocks1 : a.blocks0;
    return second ? a.op[1] : a.op[0];
}

// Partial maxima of level r: one double per block.
__device__ inline double *partial_max(const F64SplitOperand &op, int64_t KB, int r) {
    return reinterpret_cast<double *>(op.P + r * plane_elems(KB, op.Rpad) + op.Rlive * KBLK);
}

__device__ inline double wave_max(double m) {
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
    return m;
}

// max |x| over an operand (level-0 maximum) and the input-domain checks of
// Eq. (bf16rangefp64).  A wave reads 512 consecutive entries of a row (eight
// loads of 512 bytes in flight); a matrix without gaps between its rows is
// read as one row.  Bound by HBM: 5.9 TB/s at 8192^2.  (Operands with weights
// take f64_weights_kernel instead.)
__global__ __launch_bounds__(MAX_THREADS) void f64_maxabs_kernel(F64SplitArgs a) {
    __shared__ double red[MAX_THREADS / 64];
    int b, nb;
    const F64SplitOperand &op = operand_of_block(a, b, nb);
    if (b == 0) {   // the state of the passes that follow
        unsigned *w = reinterpret_cast<unsigned *>(op.st);
        for (int i = threadIdx.x; i < (int)(sizeof(F64SplitState) / 4); i += MAX_THREADS) w[i] = 0u;
    }
    double m = 0.0;
    bool nonfinite = false, range = false;
    const bool one_row = op.ldx == op.cols;
    const int64_t rows = one_row ? 1 : op.rows;
    const int64_t cols = one_row ? op.rows * op.cols : op.cols;
    constexpr int U = 8;
    const int64_t segs = (cols + U * 64 - 1) / (U * 64), items = rows * segs;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int64_t it = (int64_t)b * (MAX_THREADS / 64) + wave; it < items;
         it += (int64_t)nb * (MAX_THREADS / 64)) {
        const int64_t r = one_row ? 0 : it / segs;
        const int64_t c0 = (it - r * segs) * (U * 64) + lane;
        const double *row = op.X + r * op.ldx;
        double x[U];
        if (c0 - lane + U * 64 <= cols) {
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = row[c0 + u * 64];
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = c0 + u * 64 < cols ? row[c0 + u * 64] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double ax = fabs(x[u]);
            const bool fin = __builtin_isfinite(x[u]);
            nonfinite |= !fin;
            range |= fin && x[u] != 0.0 && (ax < DOMAIN_LO || ax > DOMAIN_HI);
            m = fmax(m, fin ? ax : 0.0);
        }
    }
    m = wave_max(m);
    const unsigned flags = block_or((nonfinite ? ST_NAN : 0u) | (range ? ST_RANGE : 0u));
    if (lane == 0) {
        red[wave] = m;
        if (flags) atomicOr(a.status, flags);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < MAX_THREADS / 64; ++i) m = fmax(m, red[i]);
        partial_max(op, a.KB, 0)[b] = m;
    }
}

// The eight entries of work item (pair, thread): packed row ic.prow, reduction
// indices k0 .. k0 + 7; zeros outside the operand; weights applied.  scan: look
// for scaled entries below the domain (ST_RANGE into st), see f64_weights_kernel.
template <bool AS_B>
__device__ __forceinline__ void load8_f64(const F64SplitOperand &op, const ItemCoords &ic,
                                          bool scan, double (&x)[8], unsigned &st) {
    const int64_t prow_lim = AS_B ? op.cols : op.rows;
    const int64_t k_lim = AS_B ? op.rows : op.cols;
    const int64_t k0 = ic.kb * KBLK + ic.q * 8, ldx = op.ldx;
    const double *X = op.X;
    const double *src = X + ic.prow * ldx + k0;
    if (!AS_B && ic.prow < prow_lim && k0 + 8 <= k_lim &&
        (reinterpret_cast<uintptr_t>(src) & 15u) == 0) {
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
            const double2 t = *reinterpret_cast<const double2 *>(src + i);
            x[i] = t.x;
            x[i + 1] = t.y;
        }
    } else {
        // branch-free: an entry outside the operand is read from g_zero8_f64,
        // so the eight loads are issued together
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const bool ok = ic.prow < prow_lim && k0 + i < k_lim;
            const double *e = ok ? X + (AS_B ? (k0 + i) * ldx + ic.prow : ic.prow * ldx + k0 + i)
                                 : g_zero8_f64;
            x[i] = *e;
        }
    }
    if (op.sc) {
        const int wexp = ic.prow < prow_lim ? -op.sc[ic.prow] : 0;   // weight 2^-s
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = ldexp(x[i], wexp);
        if (scan) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (x[i] != 0.0 && fabs(x[i]) < DOMAIN_LO) st |= ST_RANGE;
        }
    }
}

// Levels whose slices are normal BF16 values whenever the chain is right:
// every Z is a multiple of 2^(v - 8) of magnitude <= 2^v, so for
// -118 <= v <= 127 a nonzero Z lies in [2^-126, 2^127] and needs at most 8
// significant bits.  There the BF16 pattern is the top half of (float) Z,
// the residual is A - Z, and only a non-finite Z (NaN or Inf input) can
// raise a flag.  Other levels take the general rounding and checks.
__device__ inline bool plain_level(int v) { return v != V_ZERO && v >= -118 && v <= 127; }

// One pass of the six-slice split over a work share (units b, b + nb, ...):
//   Z = fl64(fl64(A^(r) + Sigma) - Sigma), Sigma = c 2^(v_r + 45)
//   (c = 0.75 symmetric, 1 literal), A_r = fl_BF16(Z) (= Z in the domain),
//   A^(r+1) = fl64(A^(r) - A_r); zero slices for a level whose residual is 0.
// Levels r0 .. nlev - 1 are stored, and the maxima |A^(r+1)| of the levels
// after r0 returned in mx (the GEMM never reads slices >= nlev, and they do
// not influence slices < nlev).  General form: any chain, any first level.
// WRITE_THROUGH: the slices are stored past this XCD's L2 (device scope).
template <bool AS_B, bool WRITE_THROUGH>
__device__ __forceinline__ void split_f64_pass(const F64SplitOperand &op, int64_t KB, int b, int nb,
                                               const int (&v)[6], int r0, int nlev, double cst,
                                               bool scan, double (&mx)[6], unsigned &st) {
    double sig[6];
    bool plain[6];
#pragma unroll
    for (int r = 0; r < 6; ++r) {
        sig[r] = (v[r] == V_ZERO) ? 0.0 : ldexp(cst, v[r] + 45);
        plain[r] = plain_level(v[r]);
    }
    const int RG = (int)(op.Rlive / ROWS_PER_BLOCK);
    const int64_t npairs = KB * RG;
    for (int64_t pair = b; pair < npairs; pair += nb) {
        const ItemCoords ic = item_coords(pair, RG);
        double x[8];
        load8_f64<AS_B>(op, ic, scan, x, st);
        // level by level over the eight entries: the branches on the (uniform)
        // form of a level are taken once per item, not once per entry
#pragma unroll
        for (int r = 0; r < 6; ++r) {
            if (r >= nlev) break;
            u16x8 outp{};
            if (plain[r]) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const double t = x[i] + sig[r];
                    const double z = t - sig[r];
                    const u16 h = (u16)(__float_as_uint((float)z) >> 16);
                    if ((h & 0x7F80u) == 0x7F80u) st |= ST_OVERFLOW;
                    x[i] = x[i] - z;
                    outp[i] = h;
                }
            } else if (v[r] != V_ZERO) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const double t = x[i] + sig[r];
                    const double z = t - sig[r];
                    const u16 h = bf16_rne_bits((float)z);    // exact for in-domain slices
                    st |= classify(h, z != 0.0);
                    x[i] = x[i] - (double)bf16_to_float(h);
                    outp[i] = h;
                }
            }
            if (r < r0) continue;
            if (r + 1 < nlev) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const double ax = fabs(x[i]);
                    if (ax > mx[r + 1]) mx[r + 1] = ax;
                }
            }
            u16 *dst = op.P + packed_index(r, ic.kb, ic.prow, ic.q, KB, op.Rpad);
            if constexpr (WRITE_THROUGH) {
                // a 16-byte store of device scope (the two wait states let the
                // store read its data before a VALU instruction may write it)
                asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1"
                             :: "v"(dst), "v"(outp) : "memory");
            } else {
                *reinterpret_cast<u16x8 *>(dst) = outp;
            }
        }
    }
}

// The first pass over a chain whose levels are all plain: the same values,
// with the number of levels fixed at compile time.  About six instructions
// per entry and level, five of them FP64.
template <int NLEV, bool AS_B>
__device__ __forceinline__ void split_f64_plain(const F64SplitOperand &op, int64_t KB, int b, int nb,
                                                const int (&v)[6], double cst, bool scan,
                                                double (&mx)[6], unsigned &st) {
    double sig[NLEV];
#pragma unroll
    for (int r = 0; r < NLEV; ++r) sig[r] = ldexp(cst, v[r] + 45);
    const unsigned RG = (unsigned)(op.Rlive / ROWS_PER_BLOCK);
    const unsigned npairs = (unsigned)(KB * RG);      // at most the planes' bytes / 4096
    const int64_t plane = plane_elems(KB, op.Rpad);
    bool nonfinite = false;
    for (unsigned pair = b; pair < npairs; pair += nb) {
        ItemCoords ic;
        const unsigned kb = pair / RG;
        ic.kb = kb;
        ic.prow = (int64_t)(pair - kb * RG) * ROWS_PER_BLOCK + (threadIdx.x >> 2);
        ic.q = threadIdx.x & 3;
        double x[8];
        load8_f64<AS_B>(op, ic, scan, x, st);
        unsigned outp[NLEV][4];
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
            double w0 = x[i], w1 = x[i + 1];
            // a non-finite entry is non-finite in every slice
            nonfinite |= !__builtin_isfinite(w0) || !__builtin_isfinite(w1);
#pragma unroll
            for (int r = 0; r < NLEV; ++r) {
                const double z0 = (w0 + sig[r]) - sig[r], z1 = (w1 + sig[r]) - sig[r];
                outp[r][i / 2] = __builtin_amdgcn_perm(__float_as_uint((float)z1),
                                                       __float_as_uint((float)z0), 0x07060302u);
                if (r + 1 < NLEV) {
                    w0 = w0 - z0;
                    w1 = w1 - z1;
                    mx[r + 1] = fmax(mx[r + 1], fabs(w0));
                    mx[r + 1] = fmax(mx[r + 1], fabs(w1));
                }
            }
        }
        u16 *dst = op.P + packed_index(0, ic.kb, ic.prow, ic.q, KB, op.Rpad);
#pragma unroll
        for (int r = 0; r < NLEV; ++r)
            *reinterpret_cast<uint4 *>(dst + r * plane) =
                make_uint4(outp[r][0], outp[r][1], outp[r][2], outp[r][3]);
    }
    if (nonfinite) st |= ST_OVERFLOW;
}

// Block maxima of the levels in red[r][0 .. W - 1] (one per wave), after a barrier.
template <int W>
__device__ inline void block_level_max(const double (&mx)[6], int r0, int nlev,
                                       double (&red)[6][W]) {
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int r = 1; r < 6; ++r) {
        if (r <= r0 || r >= nlev) continue;
        const double m = wave_max(mx[r]);
        if ((threadIdx.x & 63) == 0) red[r][w] = m;
    }
    __syncthreads();
}

// The chain speculated from the level-0 maximum.
__device__ inline void speculate_chain(double m0, int step, int (&v)[6]) {
    const int v0 = (m0 == 0.0) ? V_ZERO : ceil_log2_pos(m0);
#pragma unroll
    for (int r = 0; r < 6; ++r) v[r] = (v0 == V_ZERO) ? V_ZERO : v0 - step * r;
}

template <int NLEV>
__global__ __launch_bounds__(SPLIT_THREADS) void split_f64_kernel(F64SplitArgs a) {
    __shared__ double red[6][SPLIT_THREADS / 64];
    int b, nb;
    const F64SplitOperand &op = operand_of_block(a, b, nb);
    const int nmax = a.nops > 1 && (int)blockIdx.x >= a.blocks0 ? a.max1 : a.max0;
    // the operand-wide maximum from the partials of f64_maxabs_kernel, or of
    // f64_weights_kernel, whose sign says that the entries are to be looked through
    const double *part = partial_max(op, a.KB, 0);
    double m0 = 0.0;
    static_assert(MAX_BLOCKS <= SPLIT_THREADS, "one partial per thread");
    if ((int)threadIdx.x < nmax) m0 = part[threadIdx.x];
    const bool wave_scan = op.sc != nullptr && __any(signbit(m0));
    m0 = wave_max(fabs(m0));
    if ((threadIdx.x & 63) == 0) red[0][threadIdx.x >> 6] = wave_scan ? -m0 : m0;
    __syncthreads();
    bool scan = false;
#pragma unroll
    for (int i = 0; i < SPLIT_THREADS / 64; ++i) {
        m0 = fmax(m0, fabs(red[0][i]));
        scan |= signbit(red[0][i]);
    }
    scan = __builtin_amdgcn_readfirstlane(scan);
    m0 = __longlong_as_double(((long long)__builtin_amdgcn_readfirstlane((int)(dbits(m0) >> 32)) << 32) |
                              (unsigned)__builtin_amdgcn_readfirstlane((int)dbits(m0)));
    int v[6];
    speculate_chain(m0, a.mode ? 8 : 9, v);
    if (b == 0 && threadIdx.x == 0)
        for (int r = 0; r < 6; ++r) op.st->v[r] = v[r];
    const double cst = a.mode ? 1.0 : 0.75;
    double mx[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    unsigned st = 0;
    if (plain_level(v[0]) && plain_level(v[NLEV - 1])) {   // v descends
        if (op.as_b) split_f64_plain<NLEV, true>(op, a.KB, b, nb, v, cst, scan, mx, st);
        else split_f64_plain<NLEV, false>(op, a.KB, b, nb, v, cst, scan, mx, st);
    } else {
        if (op.as_b) split_f64_pass<true, false>(op, a.KB, b, nb, v, 0, NLEV, cst, scan, mx, st);
        else split_f64_pass<false, false>(op, a.KB, b, nb, v, 0, NLEV, cst, scan, mx, st);
    }
    st = block_or(st);
    if ((threadIdx.x & 63) == 0 && st) atomicOr(a.status, st);
    if (NLEV == 1) return;
    block_level_max(mx, 0, NLEV, red);
    // lane r of wave 0 holds the block's maximum of level r
    if (threadIdx.x >= 64) return;
    const int r = threadIdx.x;
    bool hit = false, above = false, nonzero = false;
    if (r >= 1 && r < NLEV) {
        double m = red[r][0];
        for (int i = 1; i < SPLIT_THREADS / 64; ++i) m = fmax(m, red[r][i]);
        partial_max(op, a.KB, r)[b] = m;
        int vr = v[1];
#pragma unroll
        for (int t = 2; t < 6; ++t) vr = r == t ? v[t] : vr;
        nonzero = m > 0.0;
        above = m > ldexp(1.0, vr);
        hit = nonzero && !above && ceil_log2_pos(m) == vr;
    }
    const unsigned mask = seen_hit(__ballot(hit)) | seen_above(__ballot(above)) |
                          seen_nonzero(__ballot(nonzero));
    if (threadIdx.x == 0 && mask) {
        // once a level is marked the later blocks skip the atomic
        const unsigned old = __hip_atomic_load(&op.st->seen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (mask & ~old) atomicOr(&op.st->seen, mask);
    }
}

// Verifies the levels after rf of chain v against the maxima mb, from the
// first unverified level on: returns -1 when the chain holds, else the first
// level to recompute, with v corrected there and re-speculated after it.  The
// levels after an identically zero residual are V_ZERO (their slices are zero
// whatever exponent was speculated).
__device__ inline int verify_chain(const unsigned long long (&mb)[6], int rf, int nlev, int step,
                                   int (&v)[6]) {
    int r0 = -1;
    bool done = rf < 0;
    // (compile-time level indices keep v and mb in registers)
#pragma unroll
    for (int r = 1; r < 6; ++r) {
        if (done || r <= rf || r >= nlev) continue;
        if (v[r - 1] == V_ZERO) { v[r] = V_ZERO; continue; }
        const double m = __longlong_as_double((long long)mb[r]);
        if (m == 0.0) {
#pragma unroll
            for (int t = r; t < 6; ++t) v[t] = V_ZERO;
            done = true;
            continue;
        }
        const int vt = ceil_log2_pos(m);
        if (vt == v[r]) continue;
        v[r] = vt;
#pragma unroll
        for (int t = r + 1; t < 6; ++t) v[t] = vt - step * (t - r);
        r0 = r;
        done = true;
    }
    return r0;
}

// Whether every retained panel product is an exact FP32 value for the final
// chains vA, vB.  A slice entry is a multiple of 2^(v - 8) of magnitude at
// most 2^v, so the panel sum of A_i B_j (256 terms) is a multiple of
// u = 2^(vA_i + vB_j - 16) below 2^24 u.  Every partial sum is then a normal
// FP32 value (or 0) when u >= 2^-126 and 2^24 u <= 2^127; outside that range
// the FP32 accumulation may round or overflow.  Pairs with an all-zero slice
// contribute exact zeros.
__device__ inline bool panel_products_in_range(const int (&vA)[6], const int (&vB)[6], int d) {
    bool ok = true;
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            if (i + j >= d || vA[i] == V_ZERO || vB[j] == V_ZERO) continue;
            const int e = vA[i] + vB[j];
            if (e - 16 < -126 || e + 8 > 127) ok = false;
        }
    return ok;
}

// The chains of the launch's operands in one pass (block-shared), and the
// first level each recomputes (-1: the chain holds).
struct Chains {
    int v[2][6], r0[2];
};

// The final chains (one thread of the launch).
__device__ inline void publish_chains(const F64SplitArgs &a, const Chains &c) {
    int v0[6], v1[6];
#pragma unroll
    for (int r = 0; r < 6; ++r) {
        v0[r] = c.v[0][r];
        v1[r] = c.v[1][r];
        a.op[0].st->vfinal[r] = v0[r];
        if (a.nops > 1) a.op[1].st->vfinal[r] = v1[r];
    }
    if (a.dcheck > 0 && a.nops == 2 && !panel_products_in_range(v0, v1, a.dcheck))
        atomicOr(a.status, ST_INEXACT);
}

// The chain of operand o after the split pass, into c: v corrected where a
// level was mis-speculated, and the first level to recompute.  Called by the
// whole block; red is block scratch.
__device__ inline void first_verification(const F64SplitArgs &a, int o, int nlev, Chains &c,
                                          double (&red)[6][REPLAY_THREADS / 64]) {
    const F64SplitOperand &op = o ? a.op[1] : a.op[0];
    int v[6];
#pragma unroll
    for (int r = 0; r < 6; ++r) v[r] = op.st->v[r];
    // The marks confirm the chain when every level before the first identically
    // zero one was hit and none exceeded (the same for all threads)
    const unsigned levels = (1u << nlev) - 2u, seen = op.st->seen;
    const unsigned zero = levels & ~(seen >> 16);   // (seen_nonzero)
    const unsigned before = zero ? levels & ((zero & (0u - zero)) - 1u) : levels;
    unsigned long long mb[6] = {0, 0, 0, 0, 0, 0};
    const bool confirmed =
        v[0] == V_ZERO || ((seen & seen_above(levels)) == 0u && (seen & before) == before);
    if (confirmed) {
#pragma unroll
        for (int r = 1; r < 6; ++r)
            if (zero != 0u && (1u << r) > before) v[r] = V_ZERO;
    } else {
        double mx[6];
#pragma unroll
        for (int r = 1; r < 6; ++r) {
            mx[r] = 0.0;
            if (r >= nlev) continue;
            const double *part = partial_max(op, a.KB, r);
            for (int i = threadIdx.x; i < (o ? a.blocks1 : a.blocks0); i += REPLAY_THREADS)
                mx[r] = fmax(mx[r], part[i]);
        }
        __syncthreads();   // red may still be read by an earlier use
        block_level_max(mx, 0, nlev, red);
#pragma unroll
        for (int r = 1; r < 6; ++r) {
            if (r >= nlev) continue;
            double m = red[r][0];
            for (int i = 1; i < REPLAY_THREADS / 64; ++i) m = fmax(m, red[r][i]);
            mb[r] = dbits(m);
        }
    }
    const int r0 = verify_chain(mb, confirmed ? -1 : 0, nlev, a.mode ? 8 : 9, v);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int r = 0; r < 6; ++r) c.v[o][r] = v[r];
        c.r0[o] = r0;
    }
}

// The chain operand o has in replay pass `pass` >= 2, from the slot the
// previous pass completed (read past the caches: another XCD wrote it).
__device__ inline void replay_chain(const F64SplitArgs &a, int o, int pass, int nlev, Chains &c) {
    const F64ReplaySlot &in = (o ? a.op[1] : a.op[0]).st->slot[pass - 1];
    unsigned long long mb[6];
    int v[6];
#pragma unroll
    for (int r = 0; r < 6; ++r) {
        v[r] = __hip_atomic_load(&in.v[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        mb[r] = __hip_atomic_load(&in.maxbits[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const int rf = __hip_atomic_load(&in.replay_from, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    c.r0[o] = verify_chain(mb, rf, nlev, a.mode ? 8 : 9, v);
#pragma unroll
    for (int r = 0; r < 6; ++r) c.v[o][r] = v[r];
}

// Verification of the speculated chains and, on a mismatch, up to nlev - 1
// replay passes over the operands.  The passes follow each other inside this
// launch: the blocks draw units of work (pass, share) from one counter, in
// order, and the units of a pass start once every unit of the pass before has
// been counted as done.  A unit is only drawn by a running block, which works
// on it before it draws another, so the units that a block waits for are
// always finished or in work: the wait ends whatever number of blocks the
// device runs at a time, and no co-residency is assumed.  A block leaves
// when both chains hold; it has then drawn one unit of that pass, and a pass
// has as many units as the launch has blocks, so nobody waits for a unit that
// was not drawn.  (One unit per block and pass: with two, the draws alone took
// 40 us a pass.)
__global__ __launch_bounds__(REPLAY_THREADS, 4) void f64_replay_kernel(F64SplitArgs a, int nlev) {
    __shared__ double red[6][REPLAY_THREADS / 64];
    __shared__ unsigned drawn;
    __shared__ Chains c;
    first_verification(a, 0, nlev, c, red);
    if (a.nops > 1) {
        first_verification(a, 1, nlev, c, red);
    } else if (threadIdx.x == 0) {
        for (int r = 0; r < 6; ++r) c.v[1][r] = V_ZERO;
        c.r0[1] = -1;
    }
    __syncthreads();
    if (c.r0[0] < 0 && c.r0[1] < 0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) publish_chains(a, c);
        return;
    }
    F64SplitState *ctl = a.op[0].st;
    const unsigned units = gridDim.x;
    const double cst = a.mode ? 1.0 : 0.75;
    for (;;) {
        __syncthreads();   // the last unit's reads of c and red are done
        if (threadIdx.x == 0) {
            drawn = atomicAdd(&ctl->ticket[0], 1u);
            const int pass = 1 + (int)(drawn / units);
            if (pass > 1 && pass < nlev) {
                while (__hip_atomic_load(&ctl->done[pass - 1], __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT) != units)
                    __builtin_amdgcn_s_sleep(32);
                replay_chain(a, 0, pass, nlev, c);
                if (a.nops > 1) replay_chain(a, 1, pass, nlev, c);
            }
        }
        __syncthreads();
        const int pass = 1 + (int)(drawn / units), u = (int)(drawn % units);
        if (pass >= nlev) return;
        // the last pass's chain is final: it has fixed a level in every pass
        const bool holds = c.r0[0] < 0 && c.r0[1] < 0;
        if (u == 0 && threadIdx.x == 0 && (holds || pass == nlev - 1)) publish_chains(a, c);
        if (holds) return;
        const int o = u >= a.units0 ? 1 : 0;
        const F64SplitOperand &op = o ? a.op[1] : a.op[0];
        const int b = o ? u - a.units0 : u, nb = o ? (int)units - a.units0 : a.units0;
        const int r0 = __builtin_amdgcn_readfirstlane(c.r0[o]);
        int v[6];
#pragma unroll
        for (int r = 0; r < 6; ++r) v[r] = __builtin_amdgcn_readfirstlane(c.v[o][r]);
        F64ReplaySlot *out = &op.st->slot[pass];
        if (b == 0 && threadIdx.x == 0) {
            for (int r = 0; r < 6; ++r)
                __hip_atomic_store(&out->v[r], v[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&out->replay_from, r0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (r0 >= 0) {
            double mx[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
            unsigned st = 0;
            const int ib = b * REPLAY_ITEMS + (int)(threadIdx.x / SPLIT_THREADS), nib = nb * REPLAY_ITEMS;
            if (op.as_b) split_f64_pass<true, true>(op, a.KB, ib, nib, v, r0, nlev, cst, false, mx, st);
            else split_f64_pass<false, true>(op, a.KB, ib, nib, v, r0, nlev, cst, false, mx, st);
            st = block_or(st);
            if ((threadIdx.x & 63) == 0 && st) atomicOr(a.status, st);
            block_level_max(mx, r0, nlev, red);
            const int r = threadIdx.x;
            if (r > r0 && r >= 1 && r < nlev) {
                double m = red[r][0];
                for (int i = 1; i < REPLAY_THREADS / 64; ++i) m = fmax(m, red[r][i]);
                // most units find a maximum that is already as large
                if (dbits(m) > __hip_atomic_load(&out->maxbits[r], __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
                    atomicMax(&out->maxbits[r], dbits(m));
            }
        }
        // The next pass reads this slot and rewrites slices from other XCDs:
        // every store and maximum of this unit, all of device scope, has been
        // performed before the unit counts as done.  (A device-scope fence here
        // would write back the whole L2, once per wave: 2.6 times the time of
        // the separate launches this loop replaced.)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) atomicAdd(&ctl->done[pass], 1u);
    }
}

// ---------------------------------------------------------------------------
// Weights of the scale-aware split: s_p = ceil(log2 max|x|) over each row of X
// (by_col = 0) or each column (by_col = 1), non-finite entries ignored, 0 for
// a row without nonzero entries.  The maxima are reduced as bit patterns of
// non-negative doubles (whose unsigned order is the numeric order).

// one block per row, threads across the row
__global__ __launch_bounds__(SPLIT_THREADS) void row_maxbits_kernel(
    const double *__restrict__ X, int64_t rows, int64_t cols, int64_t ldx,
    unsigned long long *__restrict__ mb) {
    __shared__ unsigned long long red[SPLIT_THREADS / 64];
    for (int64_t r = blockIdx.x; r < rows; r += gridDim.x) {
        double m = 0.0;
        for (int64_t c0 = threadIdx.x; c0 < cols; c0 += 8 * SPLIT_THREADS) {   // eight loads in flight
            double x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                x[u] = c0 + u * SPLIT_THREADS < cols ? X[r * ldx + c0 + u * SPLIT_THREADS] : 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (__builtin_isfinite(x[u])) m = fmax(m, fabs(x[u]));
        }
        for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = dbits(m);
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned long long b = red[0];
            for (int i = 1; i < SPLIT_THREADS / 64; ++i) b = red[i] > b ? red[i] : b;
            mb[r] = b;
        }
        __syncthreads();
    }
}

// 64 columns per block and a slice of the rows per blockIdx.y; lanes run
// along the columns (coalesced), the four waves over rows; one atomic maximum
// per column and block.  mb must be zero on entry.
__global__ __launch_bounds__(SPLIT_THREADS) void col_maxbits_kernel(
    const double *__restrict__ X, int64_t rows, int64_t cols, int64_t ldx,
    unsigned long long *__restrict__ mb) {
    __shared__ unsigned long long red[SPLIT_THREADS / 64][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t c = (int64_t)blockIdx.x * 64 + lane;
    const int64_t per = (rows + gridDim.y - 1) / gridDim.y;
    const int64_t r0 = (int64_t)blockIdx.y * per, r1 = r0 + per < rows ? r0 + per : rows;
    double m = 0.0;
    if (c < cols)
        for (int64_t r = r0 + w; r < r1; r += 8 * (SPLIT_THREADS / 64)) {   // eight loads in flight
            double x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t ru = r + u * (SPLIT_THREADS / 64);
                x[u] = ru < r1 ? X[ru * ldx + c] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (__builtin_isfinite(x[u])) m = fmax(m, fabs(x[u]));
        }
    red[w][lane] = dbits(m);
    __syncthreads();
    if (w == 0 && c < cols) {
        unsigned long long b = red[0][lane];
        for (int i = 1; i < SPLIT_THREADS / 64; ++i) b = red[i][lane] > b ? red[i][lane] : b;
        if (b) atomicMax(&mb[c], b);
    }
}

__global__ void maxbits_to_exponent_kernel(const unsigned long long *__restrict__ mb, int64_t n,
                                           int *__restrict__ s) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double m = __longlong_as_double((long long)mb[i]);
        s[i] = (m > 0.0) ? ceil_log2_pos(m) : 0;
    }
}

__global__ void fill_u64_kernel(unsigned long long *p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}

// Magnitude statistics for the scale-aware split: per row or column the largest
// finite and the smallest nonzero finite magnitude (bit patterns; 0 and ~0 for
// none), and the NaN/infinity flag.  They give the weights, the level-0 maximum of
// the scaled operand and its domain checks without reading it a second time.
struct MagStat {
    unsigned long long mx = 0ull, mn = ~0ull;
    bool nonfinite = false;
    __device__ void add(double x) {
        const unsigned long long a = dbits(fabs(x));
        if (!__builtin_isfinite(x)) { nonfinite = true; return; }
        mx = a > mx ? a : mx;
        mn = (a != 0ull && a < mn) ? a : mn;
    }
};

// block-wide result of one row, valid in thread 0
__device__ inline void block_magstat(MagStat &s, unsigned long long (*red)[2]) {
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long a = __shfl_xor(s.mx, off), b = __shfl_xor(s.mn, off);
        s.mx = a > s.mx ? a : s.mx;
        s.mn = b < s.mn ? b : s.mn;
    }
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6][0] = s.mx;
        red[threadIdx.x >> 6][1] = s.mn;
    }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int i = 1; i < SPLIT_THREADS / 64; ++i) {
            s.mx = red[i][0] > s.mx ? red[i][0] : s.mx;
            s.mn = red[i][1] < s.mn ? red[i][1] : s.mn;
        }
    __syncthreads();
}

// one block per row, four loads in flight per thread.  IDX: the row's entries are
// those of the columns idx[0 .. cols), and they are written to G as well.
template <bool IDX>
__global__ __launch_bounds__(SPLIT_THREADS) void row_stats_kernel(
    const double *__restrict__ X, int64_t rows, int64_t cols, int64_t ldx, int64_t cstride,
    const int *__restrict__ idx, double *__restrict__ G, unsigned long long *__restrict__ mx,
    unsigned long long *__restrict__ mn, unsigned *__restrict__ status) {
    __shared__ unsigned long long red[SPLIT_THREADS / 64][2];
    bool nonfinite = false;
    for (int64_t r = blockIdx.x; r < rows; r += gridDim.x) {
        const double *row = X + r * ldx;
        MagStat s;
        for (int64_t c0 = threadIdx.x; c0 < cols; c0 += 4 * SPLIT_THREADS) {
            double x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t c = c0 + u * SPLIT_THREADS;
                x[u] = c < cols ? row[IDX ? idx[c] * cstride : c] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t c = c0 + u * SPLIT_THREADS;
                s.add(x[u]);
                if (IDX && c < cols) G[r * cols + c] = x[u];
            }
        }
        nonfinite |= s.nonfinite;
        block_magstat(s, red);
        if (threadIdx.x == 0) {
            mx[r] = s.mx;
            mn[r] = s.mn;
        }
    }
    if (__any(nonfinite) && (threadIdx.x & 63) == 0) atomicOr(status, ST_NAN);
}

// 64 columns per block and a slice of the rows per blockIdx.y; lanes run along
// the columns, the four waves over rows, four loads in flight; two atomics per
// column and block.  mx and mn must be 0 and ~0 on entry.  IDX: the rows are
// idx[0 .. rows), and they are written to G as well.
template <bool IDX>
__global__ __launch_bounds__(SPLIT_THREADS) void col_stats_kernel(
    const double *__restrict__ X, int64_t rows, int64_t cols, int64_t ldx, int64_t cstride,
    const int *__restrict__ idx, double *__restrict__ G, unsigned long long *__restrict__ mx,
    unsigned long long *__restrict__ mn, unsigned *__restrict__ status) {
    __shared__ unsigned long long red[SPLIT_THREADS / 64][64][2];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t c = (int64_t)blockIdx.x * 64 + lane;
    const int64_t per = (rows + gridDim.y - 1) / gridDim.y;
    const int64_t r0 = (int64_t)blockIdx.y * per, r1 = r0 + per < rows ? r0 + per : rows;
    MagStat s;
    if (c < cols)
        for (int64_t r = r0 + w; r < r1; r += 4 * (SPLIT_THREADS / 64)) {
            double x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t ru = r + u * (SPLIT_THREADS / 64);
                x[u] = ru < r1 ? X[(IDX ? idx[ru] : ru) * ldx + c * cstride] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t ru = r + u * (SPLIT_THREADS / 64);
                s.add(x[u]);
                if (IDX && ru < r1) G[ru * cols + c] = x[u];
            }
        }
    red[w][lane][0] = s.mx;
    red[w][lane][1] = s.mn;
    if (__any(s.nonfinite) && lane == 0) atomicOr(status, ST_NAN);
    __syncthreads();
    if (w == 0 && c < cols) {
        for (int i = 1; i < SPLIT_THREADS / 64; ++i) {
            s.mx = red[i][lane][0] > s.mx ? red[i][lane][0] : s.mx;
            s.mn = red[i][lane][1] < s.mn ? red[i][lane][1] : s.mn;
        }
        if (s.mx) atomicMax(&mx[c], s.mx);
        if (s.mn != ~0ull) atomicMin(&mn[c], s.mn);
    }
}

__global__ void stats_init_kernel(unsigned long long *mx, unsigned long long *mn, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        mx[i] = 0ull;
        mn[i] = ~0ull;
    }
}

// From the statistics of an operand's packed rows: their weights, and in place of
// f64_maxabs_kernel the level-0 maximum of the scaled operand, its range check
// and the cleared state.  A scaled magnitude is at most 1, so only entries below
// 2^-126 leave the range.  Where the smallest one of a row underflows to an exact
// zero (which is in the domain), others of the row may leave it: the sign of the
// block's maximum then tells the split pass to look at every entry.  (A walk of the
// row by the thread here took 2.2 ms for one such row of 16384 entries, in a call of
// 0.25.)
__global__ __launch_bounds__(SPLIT_THREADS) void f64_weights_kernel(F64SplitArgs a) {
    __shared__ double red[SPLIT_THREADS / 64];
    int b, nb;
    const F64SplitOperand &op = operand_of_block(a, b, nb);
    if (b == 0) {
        unsigned *w = reinterpret_cast<unsigned *>(op.st);
        for (int i = threadIdx.x; i < (int)(sizeof(F64SplitState) / 4); i += SPLIT_THREADS) w[i] = 0u;
    }
    const int64_t n = op.as_b ? op.cols : op.rows;
    double m = 0.0;
    bool range = false, scan = false;
    for (int64_t p = (int64_t)b * SPLIT_THREADS + threadIdx.x; p < n; p += (int64_t)nb * SPLIT_THREADS) {
        const double mx = __longlong_as_double((long long)op.mx[p]);
        const int s = mx > 0.0 ? ceil_log2_pos(mx) : 0;
        const_cast<int *>(op.sc)[p] = s;
        m = fmax(m, ldexp(mx, -s));
        if (mx > 0.0) {
            const double t = ldexp(__longlong_as_double((long long)op.mn[p]), -s);
            range |= t > 0.0 && t < DOMAIN_LO;
            scan |= t == 0.0;
        }
    }
    m = wave_max(m);
    scan = __any(scan);
    const unsigned flags = block_or(range ? ST_RANGE : 0u);
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6] = scan ? -m : m;
        if (flags) atomicOr(a.status, flags);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < SPLIT_THREADS / 64; ++i) {
            m = fmax(m, fabs(red[i]));
            scan |= signbit(red[i]);
        }
        partial_max(op, a.KB, 0)[b] = scan ? -m : m;
    }
}

// Test hook: packed planes back to plain row-major planes in X's orientation.
__global__ void unpack_kernel(const u16 *__restrict__ P, int nc, int64_t KB, int64_t Rpad,
                              int64_t rows, int64_t cols, int as_b, u16 *__restrict__ out) {
    const int64_t total = (int64_t)nc * rows * cols;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t c = i / (rows * cols);
        const int64_t rem = i - c * rows * cols;
        const int64_t r = rem / cols, col = rem - r * cols;
        const int64_t prow = as_b ? col : r;
        const int64_t k = as_b ? r : col;
        const int64_t kb = k / KBLK, q = (k % KBLK) / 8;
        out[i] = P[packed_index((int)c, kb, prow, (int)q, KB, Rpad) + (k % 8)];
    }
}

// The verified chain.
__global__ void copy_v_kernel(const F64SplitState *st, int32_t *v) {
    if (threadIdx.x < 6) v[threadIdx.x] = st->vfinal[threadIdx.x];
}

// An operand without entries: every level is zero.
__global__ void f64_empty_kernel(F64SplitState *st) {
    if (threadIdx.x < 6) st->vfinal[threadIdx.x] = V_ZERO;
}

template <typename T>
__global__ void fill_zero_kernel(T *C, int64_t M, int64_t N, int64_t ldc) {
    for (int64_t r = blockIdx.x; r < M; r += gridDim.x)
        for (int64_t c = threadIdx.x; c < N; c += blockDim.x) C[r * ldc + c] = T(0);
}

int grid_for_pairs(int64_t npairs) {
    const int64_t cap = 8192;
    return (int)(npairs < cap ? (npairs > 0 ? npairs : 1) : cap);
}

}  // namespace

// C = beta C (0 when beta == 0: C is then not read), the BLAS result when
// alpha == 0 or K == 0.
template <typename T>
__global__ void scale_c_kernel(T *C, int64_t M, int64_t N, int64_t ldc, T beta) {
    for (int64_t r = blockIdx.x; r < M; r += gridDim.x)
        for (int64_t c = threadIdx.x; c < N; c += blockDim.x)
            C[r * ldc + c] = (beta == T(0)) ? T(0) : beta * C[r * ldc + c];
}

hipError_t launch_scale_c_f32(float *C, int64_t M, int64_t N, int64_t ldc, float beta,
                              hipStream_t s) {
    const int g = (int)(M < 4096 ? (M > 0 ? M : 1) : 4096);
    scale_c_kernel<float><<<g, 256, 0, s>>>(C, M, N, ldc, beta);
    return hipGetLastError();
}

hipError_t launch_scale_c_f64(double *C, int64_t M, int64_t N, int64_t ldc, double beta,
                              hipStream_t s) {
    const int g = (int)(M < 4096 ? (M > 0 ? M : 1) : 4096);
    scale_c_kernel<double><<<g, 256, 0, s>>>(C, M, N, ldc, beta);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float *C, int64_t M, int64_t N, int64_t ldc, hipStream_t s) {
    const int g = (int)(M < 4096 ? M : 4096);
    fill_zero_kernel<float><<<g, 256, 0, s>>>(C, M, N, ldc);
    return hipGetLastError();
}

hipError_t launch_fill_f64(double *C, int64_t M, int64_t N, int64_t ldc, hipStream_t s) {
    const int g = (int)(M < 4096 ? M : 4096);
    fill_zero_kernel<double><<<g, 256, 0, s>>>(C, M, N, ldc);
    return hipGetLastError();
}

hipError_t launch_split_f32(const F32SplitOperand *ops, int nops, int64_t KB, unsigned *status,
                            hipStream_t s) {
    if (nops < 1 || nops > 2) return hipErrorInvalidValue;
    F32SplitArgs a{};
    for (int o = 0; o < nops; ++o) a.op[o] = ops[o];
    a.nops = nops;
    a.KB = KB;
    a.status = status;
    a.blocks0 = grid_for_pairs(KB * (ops[0].Rlive / ROWS_PER_BLOCK));
    const int g = a.blocks0 + (nops > 1 ? grid_for_pairs(KB * (ops[1].Rlive / ROWS_PER_BLOCK)) : 0);
    split_f32_kernel<<<g, SPLIT_THREADS, 0, s>>>(a);
    return hipGetLastError();
}

// Full FP64 split of the operands: level-0 maxima, the speculative pass over all
// levels, and its verification (which replays only on a mismatch).
hipError_t launch_split_f64(const F64SplitOperand *ops, int nops, int64_t KB, int nlev, int mode,
                            int dcheck, unsigned *status, hipStream_t s) {
    if (nops < 1 || nops > 2 || nlev < 1 || nlev > 6 || (dcheck > 0 && nops != 2))
        return hipErrorInvalidValue;
    for (int o = 0; o < nops; ++o)
        if (ops[o].Rlive % ROWS_PER_BLOCK != 0 || ops[o].Rpad - ops[o].Rlive < ROW_SKEW_TILES * ROW_GROUP)
            return hipErrorInvalidValue;
    if (KB == 0) {   // no planes, and nowhere to keep partial maxima
        for (int o = 0; o < nops; ++o) f64_empty_kernel<<<1, 64, 0, s>>>(ops[o].st);
        return hipGetLastError();
    }
    F64SplitArgs a{};
    for (int o = 0; o < nops; ++o) a.op[o] = ops[o];
    a.nops = nops;
    a.KB = KB;
    a.status = status;
    a.dcheck = dcheck;
    a.mode = mode;
    auto clamp = [](int64_t n, int hi) { return (int)(n < 1 ? 1 : n < hi ? n : hi); };
    // one 512-entry segment of a row per wave, at most MAX_BLOCKS blocks per operand
    auto max_blocks = [&](const F64SplitOperand &o) {
        const int64_t segs = o.ldx == o.cols ? (o.rows * o.cols + 511) / 512
                                                                : o.rows * ((o.cols + 511) / 512);
        return clamp((segs + MAX_THREADS / 64 - 1) / (MAX_THREADS / 64), MAX_BLOCKS);
    };
    if (ops[0].sc != nullptr) {
        // scale-aware: weights and maxima from the operands' statistics
        auto row_blocks = [&](const F64SplitOperand &o) {
            return clamp(((o.as_b ? o.cols : o.rows) + SPLIT_THREADS - 1) / SPLIT_THREADS, MAX_BLOCKS);
        };
        a.blocks0 = a.max0 = row_blocks(ops[0]);
        a.blocks1 = a.max1 = nops > 1 ? row_blocks(ops[1]) : 0;
        f64_weights_kernel<<<a.blocks0 + a.blocks1, SPLIT_THREADS, 0, s>>>(a);
    } else {
        a.blocks0 = a.max0 = max_blocks(ops[0]);
        a.blocks1 = a.max1 = nops > 1 ? max_blocks(ops[1]) : 0;
        f64_maxabs_kernel<<<a.blocks0 + a.blocks1, MAX_THREADS, 0, s>>>(a);
    }
    // one 64-row x 32-index item per block, at most SPLIT_BLOCKS blocks per operand
    a.blocks0 = clamp(KB * (ops[0].Rlive / ROWS_PER_BLOCK), SPLIT_BLOCKS);
    a.blocks1 = nops > 1 ? clamp(KB * (ops[1].Rlive / ROWS_PER_BLOCK), SPLIT_BLOCKS) : 0;
    const int g = a.blocks0 + a.blocks1;
    switch (nlev) {
        case 1: split_f64_kernel<1><<<g, SPLIT_THREADS, 0, s>>>(a); break;
        case 2: split_f64_kernel<2><<<g, SPLIT_THREADS, 0, s>>>(a); break;
        case 3: split_f64_kernel<3><<<g, SPLIT_THREADS, 0, s>>>(a); break;
        case 4: split_f64_kernel<4><<<g, SPLIT_THREADS, 0, s>>>(a); break;
        case 5: split_f64_kernel<5><<<g, SPLIT_THREADS, 0, s>>>(a); break;
        default: split_f64_kernel<6><<<g, SPLIT_THREADS, 0, s>>>(a); break;
    }
    // A replay unit per two items (the block's two halves), at most 256 (512 for
    // large operands: two blocks per CU), shared between the operands by their
    // items.  Drawing and counting cost about 30 ns a unit and pass: d = 6 at
    // 2048^3, every level replayed, split phase, us: 250 with 256 units of 512
    // threads, 329 with 512 of 256, 355 with 128 of 1024, 288 with the separate
    // launches of before, which took 20 us more whenever nothing is replayed; at
    // 256^3 69, 78, 123 and 74 (84 with four items a unit).  A launch that finds
    // nothing to do costs less the fewer blocks it has (2.2 us for 320, 4.7 for
    // 2048).
    const int64_t items0 = KB * (ops[0].Rlive / ROWS_PER_BLOCK);
    const int64_t items = items0 + (nops > 1 ? KB * (ops[1].Rlive / ROWS_PER_BLOCK) : 0);
    const int most = clamp(items / REPLAY_ITEMS, (items < 16384 ? 512 : 1024) / REPLAY_ITEMS);
    const int gr = most < nops ? nops : most;
    a.units0 = nops == 1 ? gr : clamp(gr * items0 / items, gr - 1);
    f64_replay_kernel<<<gr, REPLAY_THREADS, 0, s>>>(a, nlev);
    return hipGetLastError();
}

hipError_t launch_scale_exponents(const double *X, int64_t rows, int64_t cols, int64_t ldx,
                                  bool by_col, unsigned long long *mb, int *sexp, hipStream_t s) {
    const int64_t n = by_col ? cols : rows;
    if (n == 0) return hipSuccess;
    const int fg = (int)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024);
    if (by_col) {
        fill_u64_kernel<<<fg, 256, 0, s>>>(mb, n);
        const int64_t gx = (cols + 63) / 64;
        int64_t gy = (rows + 255) / 256;                  // about 256 rows per block
        if (gy > 65535) gy = 65535;
        if (gx * gy > 16384) gy = 16384 / gx > 1 ? 16384 / gx : 1;
        col_maxbits_kernel<<<dim3((unsigned)gx, (unsigned)gy), SPLIT_THREADS, 0, s>>>(X, rows, cols,
                                                                                      ldx, mb);
    } else {
        const int g = (int)(rows < 8192 ? rows : 8192);
        row_maxbits_kernel<<<g, SPLIT_THREADS, 0, s>>>(X, rows, cols, ldx, mb);
    }
    maxbits_to_exponent_kernel<<<fg, 256, 0, s>>>(mb, n, sexp);
    return hipGetLastError();
}

namespace {
// grid of a pass over columns: 64 per block, about 64 rows per slice (with 256 a
// 161-row group of 1024 columns took 21 us on 16 blocks)
dim3 col_grid(int64_t rows, int64_t cols) {
    const int64_t gx = (cols + 63) / 64;
    int64_t gy = (rows + 63) / 64;
    if (gy > 65535) gy = 65535;
    if (gx * gy > 8192) gy = 8192 / gx > 1 ? 8192 / gx : 1;
    return dim3((unsigned)gx, (unsigned)(gy > 0 ? gy : 1));
}
int row_grid(int64_t rows) { return (int)(rows < 8192 ? (rows > 0 ? rows : 1) : 8192); }
hipError_t stats_init(unsigned long long *mx, unsigned long long *mn, int64_t n, hipStream_t s) {
    stats_init_kernel<<<(int)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024), 256, 0, s>>>(mx, mn, n);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_mag_stats(const double *X, int64_t rows, int64_t cols, int64_t ldx, bool by_col,
                            unsigned long long *mx, unsigned long long *mn, unsigned *status,
                            hipStream_t s) {
    const int64_t n = by_col ? cols : rows;
    if (n == 0) return hipSuccess;
    if (by_col) {
        hipError_t e = stats_init(mx, mn, n, s);
        if (e != hipSuccess) return e;
        col_stats_kernel<false><<<col_grid(rows, cols), SPLIT_THREADS, 0, s>>>(
            X, rows, cols, ldx, 1, nullptr, nullptr, mx, mn, status);
    } else {
        row_stats_kernel<false><<<row_grid(rows), SPLIT_THREADS, 0, s>>>(
            X, rows, cols, ldx, 1, nullptr, nullptr, mx, mn, status);
    }
    return hipGetLastError();
}

hipError_t launch_gather_stats(const double *A, int64_t lda, bool ta, const double *B, int64_t ldb,
                               bool tb, int64_t M, int64_t N, const int *idx, int64_t kb, double *GA,
                               double *GB, unsigned long long *mxA, unsigned long long *mnA,
                               unsigned long long *mxB, unsigned long long *mnB, unsigned *status,
                               hipStream_t s) {
    hipError_t e = stats_init(mxB, mnB, N, s);
    if (e != hipSuccess) return e;
    row_stats_kernel<true><<<row_grid(M), SPLIT_THREADS, 0, s>>>(
        A, M, kb, ta ? 1 : lda, ta ? lda : 1, idx, GA, mxA, mnA, status);
    col_stats_kernel<true><<<col_grid(kb, N), SPLIT_THREADS, 0, s>>>(
        B, kb, N, tb ? 1 : ldb, tb ? ldb : 1, idx, GB, mxB, mnB, status);
    return hipGetLastError();
}

hipError_t launch_unpack(const uint16_t *P, int nc, int64_t KB, int64_t Rpad, int64_t rows,
                         int64_t cols, bool as_b, uint16_t *out, hipStream_t s) {
    unpack_kernel<<<2048, 256, 0, s>>>(P, nc, KB, Rpad, rows, cols, as_b ? 1 : 0, out);
    return hipGetLastError();
}

hipError_t launch_copy_v(const F64SplitState *st, int32_t *v, hipStream_t s) {
    copy_v_kernel<<<1, 64, 0, s>>>(st, v);
    return hipGetLastError();
}

}  // namespace emu
