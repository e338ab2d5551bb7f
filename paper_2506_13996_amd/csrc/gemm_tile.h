// Block-tile bf16 MFMA contraction for gfx950, shared by every GEMM of the library: the tiled
// LM-head + cross-entropy path (logits of a sequence tile, dHidden of the tile, dW accumulation),
// the tiled MLP and the tiled linear layer.
//
// One workgroup owns a 256 (r) x 256 (c) block of D and walks k in steps of 64 through two LDS
// stages.  The c index is the MFMA row (register) dimension and r the MFMA column (lane)
// dimension, so a lane holds, for one r, runs of 4 consecutive c: reductions over c stay mostly
// inside a lane and stores along c are vector stores.  The core with two k-contiguous operands
// multiplies with v_mfma_f32_16x16x32_bf16 (accumulator tiles of 16 x 16, 4 registers per lane), the
// k-major ones with v_mfma_f32_32x32x16_bf16 (32 x 32, 16 registers): on random operands
// the 16 x 16 form draws less power per flop (a register-resident loop sustains 1.89 against
// 1.80 PFLOP/s) and the same block GEMM runs 5.5 - 7.5 % faster with it.  The kernels' epilogues
// are written against the layout description every core carries (Lane, kTile, kRuns, kGroups).
//
// An operand is either k-contiguous (a matrix [rows][k]) or k-major (a matrix [k][columns], the
// block taking 256 of its columns).  Three combinations occur:
//     D[r][c] = sum_k X[r][k] * Y[c][k]     both k-contiguous: logits, forward projections, and the products
//                                           with a weight matrix over its row index (dH = dZ W, da = dy Wd,
//                                           dx = dg Wg + du Wu, dx = dy W) against a copy of the weight
//                                           transposed once per call (transpose_piece)
//     D[r][c] = sum_k X[r][k] * Y[k][c]     "mixed": those products of the MLP and the linear layer with the
//                                           weight as it is, where an extent is not whole k-steps and the
//                                           call's workspace has no unused room for the copy
//     D[r][c] = sum_k X[k][r] * Y[k][c]     both k-major: the weight-gradient products, whose k is
//                                           the token row
// Activations and what is made of them are read as they lie; only weights are ever transposed.
//
// Three cores with the same accumulator interface for these blocks, one per layout: DirectCore, MixedCore,
// KMajorCore; halves of a block (HalfCore, KMajorHalfCore) and, for launches of few blocks, blocks of 64 x 64 and 64 x 128
// (RingCoreT, KMajorSplitT) have cores of their own below.
// 4 wavefronts (one per SIMD), 128 x 128 per wavefront, operands DMA'd straight from global memory
// into LDS (global_load_lds_dwordx4), MFMA operands of the two k-slices of a step held in registers,
// one barrier in the middle of a k-step so that the next stage's first operands are read while the
// second half is multiplied.  A k-major tile lands in LDS as 64 k-rows and the MFMA operands are
// formed by the transposing LDS read (ds_read_b64_tr_b16).
//
// Ragged extents cost the k-loop nothing: a lane chooses where its DMA reads from, so the rows (or
// columns) an operand lacks inside a block are read from its last one (finite or not, they only
// reach accumulators that the caller discards), and in the last k-step the k that do not exist are
// read from a chunk of zeros, for both operands (so that no infinity meets a zero).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace alst {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef short i16x8_t __attribute__((ext_vector_type(8)));

constexpr int kBlockR = 256;          // rows of X per block (MFMA lane dimension)
constexpr int kBlockC = 256;          // rows of Y per block (MFMA register dimension)
constexpr int kBlockK = 64;           // k per main-loop step
constexpr int kGroupC = 128;          // c extent one wavefront covers (DirectCore, HalfCore, RingCoreT<8>), of a softmax partial
constexpr int kTileBytes = kBlockR * kBlockK * 2;       // one operand tile in LDS (32 KB)
constexpr int kStageBytes = 4 * kTileBytes;             // X, Y, two stages each (128 KB)
constexpr int kLdsBytes = kStageBytes + 1024;           // + landing area of the L2 warm-up loads
constexpr int kWarmAhead = 3;                           // k-steps between warm-up and DMA of a line

// What a lane reads in place of k that do not exist.
static __device__ __align__(16) uint32_t zero_chunk[4];

// XCD-aware block numbering.  Workgroups are dealt round-robin to the 8 XCDs (each with its own L2);
// the 32 workgroups that are resident together on one XCD get a run of 32 consecutive blocks of an
// order that walks the output in columns PC blocks wide, so that a run is a patch of PR x PC blocks that
// share operand tiles through that L2.  The order has no holes: a last column may be narrower, a launch
// of several products ("parts") numbers their blocks through, and the blocks that do not fill a round of
// 256 are spread evenly over the XCDs.  (Numbering padded patches instead, patch P on XCD P % 8, left an
// XCD with a second patch while others had none: 9 patches took the time of 16.)
// Inside a column the blocks go by patches, a patch's rows fastest, or row by row (by_rows).
constexpr int kXcds = 8, kPerXcd = 32, kRound = kXcds * kPerXcd;
struct PatchGrid {
    int tiles_r, tiles_c;      // output blocks of one part
    int PR, PC;                // patch shape, PR * PC = 32
    // (int: the launches are checked to fit a one-dimensional grid before any kernel sees this)
    __host__ __device__ int blocks() const { return tiles_r * tiles_c; }
    // for the host-side sizing, which also meets shapes no launch can hold
    int64_t padded() const {
        return (int64_t)((tiles_r + PR - 1) / PR) * ((tiles_c + PC - 1) / PC) * 32;
    }
};

// Patch shape: 4 x 8 (12 operand tiles per k-step for 32 blocks), unless 8 x 4 or one of the
// flat shapes 2 x 16, 16 x 2 (18 tiles per k-step) has so much less outside the output that it needs
// under 9/10 of the patches.
inline PatchGrid choose_patches(int tiles_r, int tiles_c) {
    const int shapes[4][2] = {{4, 8}, {8, 4}, {2, 16}, {16, 2}};
    PatchGrid best = {tiles_r, tiles_c, 4, 8};
    for (int i = 1; i < 4; ++i) {
        const PatchGrid g = {tiles_r, tiles_c, shapes[i][0], shapes[i][1]};
        if (10 * g.padded() < 9 * best.padded()) best = g;
    }
    return best;
}

// A launch has fewer than 2^32 threads (more are not refused: their number wraps): workgroups of 256.
constexpr int64_t kGridBlocks = ((int64_t)1 << 24) - kRound;
inline int grid_for_blocks(int64_t blocks) { return (int)((blocks + kRound - 1) / kRound * kRound); }

// Row by row: for a long contraction over rows that are not whole patches.  By patches a run there is parts of two
// behind the first partial one, whose sharers do not cover each other's warm-up lines; row by row it is
// whole rows (63 instead of 64 row blocks: cross-entropy step 16384 x 5120 x 200064, 3 % ignored, 81.2 ->
// 76.9 ms, 16384 x 2560 x 128256 27.0 -> 25.2).  By patches are faster: rows of whole patches (dW of 16 row blocks
// 1 %), short contractions (MLP 192512 x 512 x 1536: 3 % of its projections), and the weight gradients,
// which do without the warm-up (12288 x 2304 x 2816: 3 %).
__host__ __device__ __forceinline__ bool by_rows(const PatchGrid& g, int K) {
    return K >= 1024 && g.tiles_r % g.PR != 0;
}

// Workgroup -> number of its block among the launch's `total`, or -1.
__host__ __device__ __forceinline__ int block_of_workgroup(int bid, int total, bool rows) {
    const int round = bid / kRound, xcd = bid % kXcds, slot = (bid / kXcds) % kPerXcd;
    const int left = total - round * kRound;
    if (left >= kRound) return round * kRound + xcd * kPerXcd + slot;
    if (left <= 0) return -1;
    // The last round is spread evenly, one by one: the first `more` XCDs have one more.  Row by row, half
    // a round and more is dealt in units of 8, the row of a patch, whose sharers then stay together, if the fullest XCD gets no more
    // than a tenth above the mean (one by one, 236 blocks were parts of rows at both ends of every XCD's share:
    // cross-entropy step 16384 x 5120 x 128256, 3 % ignored, 49.3 -> 47.8 ms; but 207 blocks of a weight
    // gradient as 32 and 24 an XCD instead of 26: 283 -> 316 us).
    const int units8 = (left + 7) / 8;
    const int shift = rows && 2 * left >= kRound && (units8 + 7) / 8 * 640 <= left * 11 ? 3 : 0;
    const int units = shift ? units8 : left, per = units / kXcds, more = units % kXcds;
    const int number = ((xcd * per + (xcd < more ? xcd : more)) << shift) + slot;
    return slot < (per + (xcd < more ? 1 : 0)) << shift && number < left ? round * kRound + number : -1;
}

// The last round, if it fills no more than half of the compute units, is worked on in halves: two
// workgroups take a block's upper and lower 128 rows (HalfCore) or, in the weight-gradient products,
// its left and right 128 columns (KMajorHalfCore); the k order is the same, hence the results.  A
// half takes 0.62 to 0.64 of a block's time (66 against 103 us for 128 and 256 blocks of K = 4096),
// so beyond 128 blocks, where some unit would get two, whole blocks are the faster ones.
// numbers: what the launch's workgroups are dealt, blocks below `full` whole, the others as halves.
struct Halving {
    int full, numbers;
    // number -> its block; half: 0, 1 or -1 (whole)
    __host__ __device__ __forceinline__ int block(int number, int& half) const {
        half = -1;
        if (number < full) return number;
        half = (number - full) & 1;
        return full + (number - full) / 2;
    }
};
__host__ __device__ __forceinline__ Halving halve_last_round(int blocks) {
    const int full = blocks / kRound * kRound, left = blocks - full;
    if (2 * left > kRound) return {blocks, blocks};
    return {full, full + 2 * left};
}

// Whether a launch of k-contiguous products runs on persistent workgroups that fetch their next block early
// (DirectCore::Pipe).  K: whole k-steps, at least the 4 that a chain needs.  A chain's start, its larger LDS and its last,
// unused fetch cost a launch of one or two rounds more than they save, unless the contraction is long; us of a
// product without / with:
//   K = 256: 128 blocks 9.5 / 9.8, 256: 14.6 / 15.5, 384: 22.0 / 22.4, 576: 38.8 / 37.6, 2048: 101 / 85
//   K = 1024: 128 blocks 18.6 / 19.1, 256: 31.2 / 30.6, 384: 49.2 / 49.1, 576: 78.0 / 77.7, 2048: 234 / 220
//   K = 4096: 128 blocks 59.2 / 59.3, 256: 97.2 / 95.2, 576: 232 / 229, 2048: 749 / 740
// Kernels with a long epilogue (softmax, SwiGLU) need more rounds.  us of a call, of K and gate / up or logits blocks:
//   MLP forward of 2048 rows, K = 256: 512 blocks 75.8 / 73.8, 1024: 135.6 / 132.8, 1280: 166.0 / 160.5, 2560: 317 / 304
//   K = 1024: 512 blocks 134.7 / 134.8, 1024: 257.5 / 252.2, 1280: 317 / 311; K = 4096: 512 blocks 313.5 / 311.0, 1280: 791 / 776
//   lse and loss of 2048 rows, K = 512: 512 blocks 64.1 / 65.0, 768: 82.0 / 81.7, 1024: 100.0 / 98.7, 1280: 118.2 / 115.7
//   K = 1600: 512 blocks 110.8 / 111.0, 768: 152.3 / 151.2, 1024: 193.9 / 190.7; K = 4096: 512 220.1 / 219.2, 1280: 518 / 507
//   a round begun: MLP forward 3000 x 2048 x 4096 (384) 138 / 140, cross-entropy step 8000 x 512 x 5000 (640) 272 / 277,
//   3001 x 1600 x 50257 (2167) 1796 / 1764
// So from four rounds on they gain in all; with two or three it depends on the last one.
inline bool chain_pays(int64_t blocks, int64_t K, bool long_epilogue) {
    if (K % kBlockK != 0 || K < 4 * kBlockK) return false;
    return long_epilogue ? blocks > 4 * kRound : blocks > 2 * kRound || (blocks >= kRound && K >= 1024);
}

// What a launch of `blocks` blocks takes, in 16ths of a round of whole blocks (a last round in halves:
// 10 / 16, see Halving).
__host__ __device__ __forceinline__ int64_t rounds16(int64_t blocks, bool halves = true) {
    const int64_t left = blocks % kRound;
    return blocks / kRound * 16 + (left == 0 ? 0 : halves && 2 * left <= kRound ? 10 : 16);
}

// Block (tr, tc) of number i < g.blocks() in the order.
__host__ __device__ __forceinline__ void block_at(const PatchGrid& g, int i, bool rows, int& tr, int& tc) {
    const int column = i / (g.tiles_r * g.PC);
    i -= column * g.tiles_r * g.PC;
    const int c0 = column * g.PC, cols = g.tiles_c - c0 < g.PC ? g.tiles_c - c0 : g.PC;
    const int PR = rows ? 1 : g.PR;
    const int r0 = i / (PR * cols) * PR, in = g.tiles_r - r0 < PR ? g.tiles_r - r0 : PR;
    i -= r0 * cols;
    tr = r0 + i % in;
    tc = c0 + i / in;
}

// Gated pair of Y operands: with Y2 given, the Y rows of the block at c0 are runs of RUN = 64 (32)
// rows, run q = rows c0 / 2 + (q / 2) * RUN .. + RUN - 1 of Y (q even) or of Y2 (q odd): the 2 RUN rows of
// a wavefront are RUN rows of Y followed by the same rows of Y2, so a lane that holds the
// product with row j of Y in accumulator tile mt holds the one with row j of Y2 in the tile RUN rows on.
// br = row inside the block; valid = the source row exists (the pointer is then usable anyway).
template <int RUN = 64>
__device__ __forceinline__ const uint16_t* paired_row(const uint16_t* Y, const uint16_t* Y2,
                                                      int64_t ldy, int c0, int br, int rows_y,
                                                      bool& valid) {
    const int run = br >> (RUN == 64 ? 6 : 5);
    const int src = (c0 >> 1) + (run >> 1) * RUN + (br & (RUN - 1));
    valid = src < rows_y;
    return ((run & 1) ? Y2 : Y) + (int64_t)(valid ? src : 0) * ldy;
}

// L2 warm-up.  The blocks of a patch that share an operand tile walk k in step, so each of them
// would meet every line of the tile as an L2 miss at the same moment.  Instead the sharers split
// the tile's rows between them and each touches one dword per line of its share kWarmAhead
// k-steps before the DMA needs it: the miss latency is paid early and once, and the sixteen DMA
// instructions of a k-step find their lines in L2.  Returns this lane's row of X or Y (the
// pointer to its first element); every lane gets a valid row, surplus lanes repeat one.  PR x PC
// is the launch's patch shape (2 x 16, 4 x 8, 8 x 4 or 16 x 2).
__device__ __forceinline__ const uint16_t* warm_row(int PR, int PC, const uint16_t* X, int64_t ldx,
                                                    int r0, int tr, const uint16_t* Y, int64_t ldy,
                                                    int c0, int tc, const uint16_t* Y2, int rows_x,
                                                    int rows_y) {
    const int nx = kBlockR / PC, ny = kBlockC / PR, total = nx + ny, per = (total + 3) / 4;   // per <= 36
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int l = w * per + (lane < per ? lane : per - 1);
    if (l > total - 1) l = total - 1;
    if (l < nx) {
        const int row = r0 + (tc % PC) * nx + l;                      // as the DMA: clamped to X (and Y)
        return X + (int64_t)(row < rows_x ? row : rows_x - 1) * ldx;
    }
    if (Y2) {
        bool valid;
        return paired_row(Y, Y2, ldy, c0, (tr % PR) * ny + (l - nx), rows_y, valid);
    }
    const int row = c0 + (tr % PR) * ny + (l - nx);
    return Y + (int64_t)(row < rows_y ? row : rows_y - 1) * ldy;
}

// The same with a k-major Y[k][ldy]: the 64 k-rows x 512 bytes of a k-step's tile are 256 lines, line
// L = (k-row L / 4, 128-byte piece L % 4).  `step` = elements between the lane's line in one k-step
// and the next.
__device__ __forceinline__ const uint16_t* warm_line_mixed(int PR, int PC, const uint16_t* X,
                                                           int64_t ldx, int r0, int tr,
                                                           const uint16_t* Y, int64_t ldy, int c0,
                                                           int tc, int64_t& step, int rows_x,
                                                           int cols_y, int krows_y) {
    const int nx = kBlockR / PC, ny = kBlockC / PR, total = nx + ny, per = (total + 3) / 4;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int l = w * per + (lane < per ? lane : per - 1);
    if (l > total - 1) l = total - 1;
    if (l < nx) {
        step = kBlockK;
        const int row = r0 + (tc % PC) * nx + l;
        return X + (int64_t)(row < rows_x ? row : rows_x - 1) * ldx;
    }
    const int L = (tr % PR) * ny + (l - nx);
    step = ldy * kBlockK;
    const int col = c0 + (L & 3) * 64;
    const int krow = (L >> 2) < krows_y ? (L >> 2) : krows_y - 1;
    return Y + (int64_t)krow * ldy + (col < cols_y ? col : cols_y - 8);
}

// k-major LDS tiles: an LDS row is one k-row of 512 bytes = 8 granules of 64 bytes
// (32 r or c each); granule g of k-row k lives at granule slot g ^ kswz(k).  One transposing read
// covers k-rows {R .. R+3, R+8 .. R+11} (R % 4 == 0) at one granule: 8 different slots.
__device__ __forceinline__ int kswz(int k) { return (k & 3) | (((k >> 3) & 1) << 2); }

// MFMA operand (8 k of one column per lane) from a k-major tile: two transposing reads.  In each,
// the 16 lanes of a quarter wave address 4 k-rows x 4 pieces of 8 bytes and lane i of the quarter
// receives the 4 k of column i.  `at`: the lane's address for the first 4 k-rows; the next 4
// k-rows are NEXT4 bytes on (2048 in a tile of 256 columns).
template <int NEXT4>
__device__ __forceinline__ bf16x8_t read_kmajor(const unsigned char* at) {
    typedef __attribute__((address_space(3))) i16x4_t* tptr_t;
    typedef __attribute__((address_space(3))) void* lptr_t;
    unsigned char* const p = const_cast<unsigned char*>(at);
    const i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tptr_t)(lptr_t)p);
    const i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tptr_t)(lptr_t)(p + NEXT4));
    return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
// The lane's byte offset inside a k-major tile for granule `gran` (MFMA lane l: column l % 32 of
// the granule, k = 8 (l / 32) .. + 7 of a 16-row slice; add 8192 per slice).
__device__ __forceinline__ int kmajor_lane_offset(int lane, int gran) {
    const int sl = lane & 15, b1 = (lane >> 4) & 1, half = lane >> 5;
    const int f = (sl >> 2) | (half << 2);                   // kswz of the lane's k-rows
    return (8 * half + (sl >> 2)) * 512 + ((gran ^ f) * 64) + b1 * 32 + (sl & 3) * 8;
}

// The same in a tile of 128 columns (LDS rows of 256 bytes, granule slots gran ^ (k & 3); add 4096 per
// slice).
__device__ __forceinline__ int kmajor_half_lane_offset(int lane, int gran) {
    const int sl = lane & 15, b1 = (lane >> 4) & 1, half = lane >> 5;
    return (8 * half + (sl >> 2)) * 256 + ((gran ^ (sl >> 2)) * 64) + b1 * 32 + (sl & 3) * 8;
}

// Between LDS accesses of different lanes of one wavefront: LDS serves them in program order, but the compiler may
// order them anew along the branches of lanes that skip a guarded store (it sees one lane), and let those lanes write
// the next piece before the others have read this one.  No instruction.
template <bool DIVERGENT>
__device__ __forceinline__ void wave_sync() {
    if constexpr (DIVERGENT) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// Values that are the same in every lane of a wavefront, said so to the compiler (it then keeps
// them in scalar registers and branches on them without masking lanes).
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uniform(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
template <class T>
__device__ __forceinline__ const T* uniform(const T* p) {
    return reinterpret_cast<const T*>(uniform((int64_t)reinterpret_cast<uintptr_t>(p)));
}

// Global -> LDS DMA: each lane's BYTES (16 or 4) land at lds + lane * BYTES; `lds` must be uniform
// over the wavefront.
template <int BYTES>
__device__ __forceinline__ void dma_to_lds(const void* g, unsigned char* lds) {
    typedef const __attribute__((address_space(1))) void* gptr_t;
    typedef __attribute__((address_space(3))) void* lptr_t;
    static_assert(BYTES == 16 || BYTES == 4, "one or four dwords per lane");
    if (BYTES == 16) __builtin_amdgcn_global_load_lds((gptr_t)g, (lptr_t)lds, 16, 0, 0);
    else __builtin_amdgcn_global_load_lds((gptr_t)g, (lptr_t)lds, 4, 0, 0);
}

// Combines a value over the lane groups of a wavefront that hold the same r (lanes l, l ^ 16, l ^ 32,
// l ^ 48 for 16 x 16 tiles; l, l ^ 32 for 32 x 32 tiles): every lane gets the result.
template <int GROUPS>
__device__ __forceinline__ float groups_max(float v) {
    if (GROUPS == 4) v = fmaxf(v, __shfl_xor(v, 16));
    return fmaxf(v, __shfl_xor(v, 32));
}
template <int GROUPS>
__device__ __forceinline__ float groups_sum(float v) {
    if (GROUPS == 4) v += __shfl_xor(v, 16);
    return v + __shfl_xor(v, 32);
}

// ---------------------------------------------------------------------------------------------
// KMajorDirectT: the DMA core for a k-major Y (and, with XK, a k-major X): v_mfma_f32_32x32x16_bf16
// ---------------------------------------------------------------------------------------------
// Same pipeline as DirectCore below on 32 x 32 accumulator tiles.  Measured on the dHidden and dW
// GEMMs the 16 x 16 x 32 form gains nothing over this one when operands come through the
// transposing reads, and its register allocation breaks down for two k-major operands.
// XK: X is k-major too.
// MT: 32-wide c tiles per wavefront: 4, or 2 for half a block (128 c; k-major X only).
template <bool XK, int MT = 4>
struct KMajorDirectT {
    static_assert(MT == 4 || (MT == 2 && XK), "a block or the c half of one");
    static constexpr bool YK = true;
    static constexpr int kThreads = 256;
    static constexpr int kMT = MT;    // 32-wide c tiles per wavefront
    static constexpr int kNT = 4;     // 32-wide r tiles per wavefront
    static constexpr int kWaveC = 32 * MT;                 // c one wavefront covers
    typedef f32x16_t acc_t;
    static constexpr int kTile = 32, kRuns = 4, kGroups = 2;

    struct Lane {
        int lane, grp, lrow, wr, wc;
        __device__ __forceinline__ Lane() {
            const int tid = threadIdx.x;
            lane = tid & 63;
            grp = lane >> 5;
            lrow = lane & 31;
            const int wave = tid >> 6;
            wr = wave & 1;
            wc = wave >> 1;
        }
        __device__ __forceinline__ int r(int nt) const { return wr * 128 + nt * 32 + lrow; }
        __device__ __forceinline__ int rbase(int nt) const { return wr * 128 + nt * 32; }
        __device__ __forceinline__ int cw(int mt, int q) const { return mt * 32 + q * 8 + grp * 4; }
        __device__ __forceinline__ int c(int mt, int q) const { return wc * kWaveC + cw(mt, q); }
    };

    // LDS row = 128 bytes = 8 chunks of 16 bytes; chunk kc of row `row` lives at slot
    // kc ^ ((row >> 1) & 7): sixteen consecutive rows at one kc then cover all 64 banks once.
    static __device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

    // acc += the block's product over all of K >= 1 (16-byte aligned rows).  Y is [K][ldy] and the block
    // takes its columns c0 .. c0 + 255; a k-major X is [K][ldx], columns r0 .. r0 + 255, a
    // k-contiguous one [rows_x][ldx] (K a multiple of 8).  Operands may end inside the block: columns of a k-major
    // operand beyond its rows_x / rows_y (a multiple of 8) are read from its last 8, rows of a
    // k-contiguous X beyond rows_x from its last row, and the caller discards those accumulators.
    // KTAIL: K need not be whole k-steps of 64 (see the top of this file).
    // warm (k-contiguous X only): the lane's warm-up line, warm_stride = elements from one k-step's to
    // the next.
    template <bool KTAIL>
    static __device__ __forceinline__ void gemm(const uint16_t* __restrict__ X, int64_t ldx,
                                                int rows_x, const uint16_t* __restrict__ Y,
                                                int64_t ldy, int rows_y, int K, int r0, int c0,
                                                unsigned char* smem, acc_t (&acc)[kMT][kNT],
                                                const uint16_t* warm, int64_t warm_stride) {
        const int tid = threadIdx.x, lane = tid & 63;
        const int w = __builtin_amdgcn_readfirstlane(tid >> 6);       // wave id, provably uniform
        const int wr = w & 1, wc = w >> 1;
        const int l31 = lane & 31, half = lane >> 5;

        // One DMA instruction moves 8 rows x 128 bytes: lane -> (row = lane / 8, LDS chunk slot =
        // lane % 8); the lane fetches the global chunk that belongs in its slot.  Wave w owns rows
        // [64 w, 64 w + 64) of both operand tiles: 8 instructions per operand per k-step.
        // k-major: one DMA instruction moves 2 k-rows x 512 bytes: lane -> (k-row = lane / 32, chunk
        // slot = lane % 32); wave w owns k-rows [16 w, 16 w + 16) of the tile.
        // A Y tile of 128 columns: 4 k-rows x 256 bytes, an LDS row is 4 granules and granule g of
        // k-row k lives at slot g ^ (k & 3) (the 4 k-rows a quarter of a transposing read covers: 4 slots,
        // all 64 banks).
        constexpr int kYq = 2 * MT;                          // DMA instructions per wavefront for a Y tile
        constexpr int kYRow = 128 * MT;                      // bytes of an LDS row of it
        const int lr = lane >> 3, pc = lane & 7;
        auto ykrow = [&](int q) { return MT == 4 ? w * 16 + q * 2 + (lane >> 5) : w * 16 + q * 4 + (lane >> 4); };
        const uint16_t* xg[8];
        const uint16_t* yg[kYq];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int krow = w * 16 + q * 2 + (lane >> 5);
            const int ch = (lane & 31) ^ (kswz(krow) << 2);
            const int row = (w * 8 + q) * 8 + lr;
            const int kc = pc ^ swz(row);
            // (the clamps: see the comment of this function)
            if (XK) xg[q] = X + (int64_t)krow * ldx + (r0 + ch * 8 < rows_x ? r0 + ch * 8 : rows_x - 8);
            else xg[q] = X + (int64_t)(r0 + row < rows_x ? r0 + row : rows_x - 1) * ldx + kc * 8;
            if (q < kYq) {
                const int yrow = ykrow(q);
                const int yc = MT == 4 ? ch : (lane & 15) ^ ((yrow & 3) << 2);
                yg[q % kYq] = Y + (int64_t)yrow * ldy + (c0 + yc * 8 < rows_y ? c0 + yc * 8 : rows_y - 8);
            }
        }
        // elements from one k-step's tile to the next
        const int64_t xstep = XK ? ldx * kBlockK : kBlockK, ystep = ldy * kBlockK;
        const int KT = (K + kBlockK - 1) / kBlockK;
        const int klast = K - (KT - 1) * kBlockK;                     // k of the last k-step, 1 .. 64
        // where instruction q of k-step kt reads from; tail: kt is the last k-step
        auto krow_in = [&](int q) { return w * 16 + q * 2 + (lane >> 5) < klast; };
        auto zeros = [] { return reinterpret_cast<const uint16_t*>(zero_chunk); };
        auto xsrc = [&](int q, int kt, bool tail) -> const uint16_t* {
            const uint16_t* p = xg[q] + kt * xstep;
            if (!tail) return p;
            return (XK ? krow_in(q) : (pc ^ swz(q * 8 + lr)) * 8 < klast) ? p : zeros();
        };
        auto ysrc = [&](int q, int kt, bool tail) -> const uint16_t* {
            const uint16_t* p = yg[q] + kt * ystep;
            return !tail || ykrow(q) < klast ? p : zeros();
        };
        auto issue_loads = [&](int stage, int kt) {
            unsigned char* xs = smem + stage * kTileBytes + w * 8192;
            unsigned char* ys = smem + 2 * kTileBytes + stage * kTileBytes + w * (kYq * 1024);
            const bool tail = KTAIL && kt == KT - 1;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                dma_to_lds<16>(xsrc(q, kt, tail), xs + q * 1024);
                if (q < kYq) dma_to_lds<16>(ysrc(q % kYq, kt, tail), ys + q * 1024);
            }
        };

        // Operand reads.  k-contiguous tiles: one 16-byte read per operand.  k-major: read_kmajor.
        int rofs[4], xofs[4], yofs[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            rofs[s] = ((2 * s + half) ^ swz(l31)) * 16;
            xofs[s] = kmajor_lane_offset(lane, wr * 4 + s);      // s = accumulator tile here
            yofs[s] = 2 * kTileBytes + (MT == 4 ? kmajor_lane_offset(lane, wc * 4 + s)
                                                : kmajor_half_lane_offset(lane, (wc * 2 + s) & 3));
        }
        const int xbase = (wr * 128 + l31) * 128;

        // MFMA operands of the four k-slices of a step: fy[s][t], fx[s][t] for slice s.
        bf16x8_t fy[4][MT], fx[4][4];
        // item 0..MT-1: the Y operand of accumulator row t = item, MT..MT+3: the X operand of column item - MT
        auto read_item = [&](int stage, int s, int item) {
            const unsigned char* base = smem + stage * kTileBytes;
            if (item < MT)
                fy[s][item] = read_kmajor<4 * kYRow>(base + yofs[item] + s * (16 * kYRow));
            else
                fx[s][item - MT] =
                    XK ? read_kmajor<2048>(base + xofs[item - MT] + s * 8192)
                       : *reinterpret_cast<const bf16x8_t*>(base + xbase + (item - MT) * 4096 + rofs[s]);
        };
        // the two MFMAs of slot i (0 .. 2 MT - 1) of a quarter step on slice s
        auto mfma_pair = [&](int s, int i) {
            const int mt = i >> 1, n0 = (i & 1) * 2;
            acc[mt][n0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fy[s][mt], fx[s][n0], acc[mt][n0],
                                                                  0, 0, 0);
            acc[mt][n0 + 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fy[s][mt], fx[s][n0 + 1],
                                                                      acc[mt][n0 + 1], 0, 0, 0);
        };

        // One 4-byte DMA per wavefront and k-step into a landing area nobody reads: it only pulls
        // the line into L2.  `warm` (see warm_row) must be a valid row pointer in every lane.
        // Not for two k-major operands (the weight-gradient products): measured there, the extra
        // L2 lookups cost as much as the early misses save.
        constexpr bool warming = !XK;
        unsigned char* const dump = smem + kStageBytes + w * 256;
        auto warm_step = [&](int kt) {
            // (the last step may lack k-rows, and the lane's line may be one of them: not warmed)
            const int last = KTAIL && KT > 1 ? KT - 2 : KT - 1;
            const int kk = kt < last ? kt : last;
            dma_to_lds<4>(warm + kk * warm_stride, dump);
        };
        // Joins the wavefronts once this wavefront's DMA of the next stage has landed.  The warm-up
        // load issued after that DMA may still be in flight (loads complete in order).
        auto stage_barrier = [&](bool one_behind) {
            if (one_behind) asm volatile("s_waitcnt vmcnt(1) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        };
        if (warming)
            for (int p = 2; p < 2 + kWarmAhead; ++p) warm_step(p);
        issue_loads(0, 0);
        __syncthreads();                       // waits for the DMA (vmcnt) and joins the waves
        if (KT > 1) issue_loads(1, 1);
#pragma unroll
        for (int item = 0; item < MT + 4; ++item) read_item(0, 0, item);
#pragma unroll
        for (int item = 0; item < MT + 4; ++item) read_item(0, 1, item);

        // One k-step = four quarters of sixteen MFMAs, each quarter eight fenced slots of two MFMAs
        // plus the memory instructions that ride along, in this order:
        //   Q0  MFMA slice 0 | read slices 2 and 3 of this stage
        //   Q1  MFMA slice 1 |
        //   -- all of this stage has been read, the next stage has landed: workgroup barrier --
        //   Q2  MFMA slice 2 | DMA of step kt + 2, X half, into this stage | read slice 0 of kt + 1
        //   Q3  MFMA slice 3 | DMA of step kt + 2, Y half                  | read slice 1 of kt + 1
        // Every operand read is issued at least a quarter and a half before its first MFMA, so a
        // burst of DMA writes into LDS delays reads without draining the matrix pipe, and the DMA
        // issue is spread over half a step (left to the scheduler the sixteen DMA instructions
        // come out back to back and the matrix pipe idles behind their issue).
        // LOADS: step kt + 2 exists (TAIL: and is the last).  NEXT: step kt + 1 exists.  The last steps skip
        // the DMA so that none is in flight when the workgroup ends.
        // BEHIND: the previous k-step issued a warm-up load after its DMA.
        auto kstep = [&](int kt, auto loads, auto next, auto tail, bool behind) {
            constexpr bool LOADS = decltype(loads)::value, NEXT = decltype(next)::value;
            constexpr bool TAIL = decltype(tail)::value;
            const int cur = kt & 1;
            unsigned char* const xs = smem + cur * kTileBytes + w * 8192;
            unsigned char* const ys = smem + 2 * kTileBytes + cur * kTileBytes + w * (kYq * 1024);
            constexpr int kSlots = 2 * MT, kItems = MT + 4;       // (half a block: 4 slots, 6 items)
#pragma unroll
            for (int i = 0; i < kSlots; ++i) {
                mfma_pair(0, i);
#pragma unroll
                for (int q = i * 2 * kItems / kSlots; q < (i + 1) * 2 * kItems / kSlots; ++q)
                    read_item(cur, q < kItems ? 2 : 3, q % kItems);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 0; i < kSlots; ++i) {
                mfma_pair(1, i);
                __builtin_amdgcn_sched_barrier(0);
            }
            stage_barrier(behind);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < kSlots; ++i) {
                mfma_pair(2, i);
                if (LOADS)
#pragma unroll
                    for (int q = i * 8 / kSlots; q < (i + 1) * 8 / kSlots; ++q)
                        dma_to_lds<16>(xsrc(q, kt + 2, TAIL), xs + q * 1024);
                if (NEXT)
#pragma unroll
                    for (int q = i * kItems / kSlots; q < (i + 1) * kItems / kSlots; ++q) read_item(cur ^ 1, 0, q);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 0; i < kSlots; ++i) {
                mfma_pair(3, i);
                if (LOADS)
                    dma_to_lds<16>(ysrc(i % kYq, kt + 2, TAIL), ys + i * 1024);
                if (NEXT)
#pragma unroll
                    for (int q = i * kItems / kSlots; q < (i + 1) * kItems / kSlots; ++q) read_item(cur ^ 1, 1, q);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (LOADS && warming) warm_step(kt + 2 + kWarmAhead);
        };
        // a step's barrier may leave one load in flight iff the step before it had LOADS and warmed
        constexpr auto yes = std::true_type{};
        constexpr auto no = std::false_type{};
        int kt = 0;
        for (; kt + (KTAIL ? 3 : 2) < KT; ++kt) kstep(kt, yes, yes, no, warming && kt > 0);
        if (KTAIL && KT >= 3) {
            kstep(kt, yes, yes, yes, warming && kt > 0);
            ++kt;
        }
        if (KT >= 2) {
            kstep(kt, no, yes, no, warming && kt > 0);
            ++kt;
        }
        kstep(kt, no, no, no, false);
    }
};
typedef KMajorDirectT<true> KMajorCore;
// 256 r x 128 c, see HalfCore.  Backward calls with whole blocks / halves: linear 8192 x 2048 x 2048 (64 blocks) 207 / 163 us, 4096 x
// 4096 x 4608 (288) 319 / 292, 16384 x 3072 x 5120 (240: none) 773 / 772, cross-entropy 3001 x 1600 x 50257 (1379) 1371 / 1354.
typedef KMajorDirectT<true, 2> KMajorHalfCore;
typedef KMajorDirectT<false> MixedCore;

// ---------------------------------------------------------------------------------------------
// DirectCore: 4 wavefronts, global -> LDS DMA, both operands k-contiguous, v_mfma_f32_16x16x32_bf16
// ---------------------------------------------------------------------------------------------
// Against the same pipeline on the 32 x 32 x 16 form a plain product of the logits shape is 8 %
// faster (16-row operand reads, half the address arithmetic per k-step; with register-resident
// operands the two forms are level to 4 % apart).  It is the fastest of the cores, so products
// over a weight's row index are run on it against a copy of the weight transposed once per call.
template <int NT>
struct DirectCoreT {
    static constexpr int kThreads = 256;
    static constexpr int kMT = 8;     // 16-wide c tiles per wavefront
    static constexpr int kNT = NT;    // 16-wide r tiles per wavefront: 8, or 4 for half a block (128 r)
    static constexpr int kWaveR = 16 * NT;                 // r one wavefront covers
    static constexpr int kWaveC = kGroupC;
    typedef f32x4_t acc_t;
    static constexpr int kTile = 16, kRuns = 1, kGroups = 4;

    // acc[mt][nt][x]: r = nt * 16 + lane % 16, c = mt * 16 + 4 (lane / 16) + x inside the wavefront's
    // kWaveR x 128.
    struct Lane {
        int lane, grp, lrow, wr, wc;
        // tid: threadIdx.x
        __device__ __forceinline__ Lane(int tid = threadIdx.x) {
            lane = tid & 63;
            grp = lane >> 4;
            lrow = lane & 15;
            const int wave = tid >> 6;
            wr = wave & 1;
            wc = wave >> 1;
        }
        __device__ __forceinline__ int r(int nt) const { return wr * kWaveR + nt * 16 + lrow; }
        __device__ __forceinline__ int rbase(int nt) const { return wr * kWaveR + nt * 16; }
        __device__ __forceinline__ int cw(int mt, int /*q*/) const { return mt * 16 + grp * 4; }
        __device__ __forceinline__ int c(int mt, int q) const { return wc * kGroupC + cw(mt, q); }
    };

    // LDS row of a tile = 128 bytes = 8 chunks of 16 bytes; chunk kc of row `row` lives at slot
    // kc ^ ((row >> 1) & 7): sixteen consecutive rows at one kc then cover all 64 banks once.
    static __device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

    // The operands of one output block: D[r0 + r][c0 + c] = sum_k X[r0 + r][k] Y[c0 + c][k].
    // K >= 1 a multiple of 8 (of 64 without KTAIL), 16-byte aligned rows.  Operands may end inside
    // the block: their rows beyond rows_x / rows_y are read from the last one and the caller
    // discards those accumulators.
    // Y2: gated pair, see paired_row; rows_y is then the rows of Y and of Y2, the rows of the pair
    // beyond it are read from row 0 and the caller discards those columns.
    // warm (see warm_row): the lane's warm-up row; warm_stride = elements between its line of one
    // k-step and the next.
    struct Block {
        const uint16_t* X;
        int64_t ldx;
        const uint16_t* Y;
        int64_t ldy;
        int rows_x, rows_y, K, r0, c0;
        const uint16_t* warm;
        int64_t warm_stride;
        const uint16_t* Y2;
    };

    // The k-loop's state: the DMA sources of the block whose operands are being fetched, the LDS
    // read offsets and the operand registers.  Used in two ways.
    //  * One block per workgroup: gemm() below.
    //  * A chain of blocks on one (persistent) workgroup: start(first); then for every block
    //    run(block, the block after it, acc) followed by the caller's epilogue; finish() after
    //    the last.  The last two k-steps of a block, which otherwise issue no DMA, fetch the
    //    first two k-steps of the block after it into the stages they free, so the next block's
    //    operands travel while the epilogue runs and no block but the first waits for a
    //    prologue.  The last block of a chain names itself as the block after it (the fetch is
    //    then wasted; finish() waits for it so that nothing is in flight when the workgroup
    //    ends).  Every block of a chain must have the same K, a multiple of 64 and >= 256.  Between start() and
    //    finish() the first kLdsBytes of LDS belong to the chain: an epilogue that turns data
    //    around in LDS does it behind them.
    template <bool KTAIL>
    struct Pipe {
        unsigned char* smem;
        int w, lr, pc;                 // wavefront, the lane's row and chunk slot in a DMA instruction
        int rofs[2], xbase, ybase;     // LDS read offsets
        // the block the DMA works for: the lane's sources of k-step 0, the warm-up row, the k-steps
        // and (KTAIL) the k of the last one
        const uint16_t* xg[NT];
        const uint16_t* yg[8];
        const uint16_t* warm;
        int64_t warm_stride;
        int KT_, klast;
        int base;                      // the stage of the block's k-step 0 (0, but for chains of an odd number of k-steps)
        // MFMA operands of the two k-slices of a step: fy[s][t], fx[s][t] for slice s
        bf16x8_t fy[2][8], fx[2][NT];

        __device__ __forceinline__ explicit Pipe(unsigned char* smem_) : smem(smem_) {
            const int tid = threadIdx.x, lane = tid & 63;
            w = uniform(tid >> 6);
            base = 0;
            const int wr = w & 1, wc = w >> 1;
            const int l15 = lane & 15, g = lane >> 4;
            // One DMA instruction moves 8 rows x 128 bytes: lane -> (row = lane / 8, LDS chunk slot
            // = lane % 8); the lane fetches the global chunk that belongs in its slot.  Wave w owns
            // rows [64 w, 64 w + 64) of an operand tile, 8 instructions per k-step (of the 128 rows of
            // X of half a block [32 w, 32 w + 32), 4 instructions).
            lr = lane >> 3;
            pc = lane & 7;
            // Operand reads.  A k-step is two slices of 32 k; lane (row l15 of a 16-row tile,
            // k-group g) reads the 16-byte chunk 4 s + g of its row: one read per operand.
#pragma unroll
            for (int s = 0; s < 2; ++s) rofs[s] = ((4 * s + g) ^ swz(l15)) * 16;
            xbase = (wr * kWaveR + l15) * 128;
            ybase = 2 * kTileBytes + (wc * kGroupC + l15) * 128;
        }
        __device__ __forceinline__ void target(const Block& b) {
            KT_ = (b.K + kBlockK - 1) / kBlockK;
            if (KTAIL) klast = b.K - (KT_ - 1) * kBlockK;
            warm = b.warm;
            warm_stride = b.warm_stride;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int row = (w * 8 + q) * 8 + lr;
                const int kc = pc ^ swz(row);
                if (q < NT) {                       // (the clamps: see Block)
                    const int xr = (w * NT + q) * 8 + lr;
                    const int xrow = b.r0 + xr < b.rows_x ? b.r0 + xr : b.rows_x - 1;
                    xg[q < NT ? q : 0] = b.X + (int64_t)xrow * b.ldx + kc * 8;
                }
                if (b.Y2) {                         // gated pair
                    bool valid;
                    yg[q] = paired_row(b.Y, b.Y2, b.ldy, b.c0, row, b.rows_y, valid) + kc * 8;   // (missing rows: row 0)
                } else {
                    const int yrow = b.c0 + row < b.rows_y ? b.c0 + row : b.rows_y - 1;
                    yg[q] = b.Y + (int64_t)yrow * b.ldy + kc * 8;
                }
            }
        }
        // where a lane reads from in DMA instruction q: `base` (xg[q] or yg[q]) moved on to k-step
        // kt; tail: that is the last k-step, in which the chunks beyond K are zeros
        __device__ __forceinline__ const uint16_t* src(const uint16_t* base, int q, int kt, bool tail) const {
            const uint16_t* const p = base + kt * kBlockK;
            return !tail || (pc ^ swz(q * 8 + lr)) * 8 < klast ? p
                                                               : reinterpret_cast<const uint16_t*>(zero_chunk);
        }
        __device__ __forceinline__ void issue_loads(int stage, int kt) {
            unsigned char* xs = smem + stage * kTileBytes + w * (NT * 1024);
            unsigned char* ys = smem + 2 * kTileBytes + stage * kTileBytes + w * 8192;
            const bool tail = KTAIL && kt == KT_ - 1;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (q < NT) dma_to_lds<16>(src(xg[q < NT ? q : 0], q, kt, tail), xs + q * 1024);
                dma_to_lds<16>(src(yg[q], q, kt, tail), ys + q * 1024);
            }
        }
        // item 0..7: the Y operand of accumulator row t = item, 8..: the X operand of column item - 8
        __device__ __forceinline__ void read_item(int stage, int s, int item) {
            const unsigned char* base = smem + stage * kTileBytes + rofs[s];
            if (item < 8) fy[s][item] = *reinterpret_cast<const bf16x8_t*>(base + ybase + item * 2048);
            else fx[s][item - 8] = *reinterpret_cast<const bf16x8_t*>(base + xbase + (item - 8) * 2048);
        }
        // the four MFMAs of slot i (0 .. 2 NT - 1) of a slice
        __device__ __forceinline__ void mfma_quad(acc_t (&acc)[kMT][kNT], int s, int i) {
            const int mt = NT == 8 ? i >> 1 : i, n0 = NT == 8 ? (i & 1) * 4 : 0;
#pragma unroll
            for (int d = 0; d < 4; ++d)
                acc[mt][n0 + d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fy[s][mt], fx[s][n0 + d],
                                                                          acc[mt][n0 + d], 0, 0, 0);
        }
        // One 4-byte DMA per wavefront and k-step into a landing area nobody reads: it only pulls
        // the line into L2.  `warm` must be a valid row pointer in every lane.  Steps beyond the
        // targeted block's last are steps of `ahead`, the block after it in a chain (or clamped).
        __device__ __forceinline__ void warm_step(int kt, const Block* ahead) {
            unsigned char* const dump = smem + kStageBytes + w * 256;
            if (ahead != nullptr && kt >= KT_) {
                // (the next block's first steps: whole k-steps of Y, K >= 256)
                dma_to_lds<4>(ahead->warm + (kt - KT_) * ahead->warm_stride, dump);
                return;
            }
            const int kk = kt < KT_ - 1 ? kt : KT_ - 1;
            dma_to_lds<4>(warm + kk * warm_stride, dump);
        }
        // Joins the wavefronts once this wavefront's DMA of the next stage has landed.  The warm-up
        // load issued after that DMA may still be in flight (loads complete in order).
        static __device__ __forceinline__ void stage_barrier(bool one_behind) {
            if (one_behind) asm volatile("s_waitcnt vmcnt(1) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }

        // One k-step = two slices of 64 MFMAs, each slice sixteen fenced slots of four MFMAs (64
        // cycles) plus the memory instructions that ride along, in this order:
        //   slice 0, slots 0..7    | read slice 1 of this stage (two operands per slot)
        //   slice 0, slots 8..15   |
        //   -- all of this stage has been read, the next stage has landed: workgroup barrier --
        //   slice 1, slots 0..7    | DMA of step kt + 2, X half, into this stage | read slice 0 of kt + 1
        //   slice 1, slots 8..15   | DMA of step kt + 2, Y half                  | read slice 0 of kt + 1
        // Every operand read is issued at least half a slice before its first MFMA, so a burst of
        // DMA writes into LDS delays reads without draining the matrix pipe, and the DMA issue is
        // spread over half a step (left to the scheduler the sixteen DMA instructions come out
        // back to back and the matrix pipe idles behind their issue).  Inside a slot the MFMAs
        // go first (the sched_group_barrier calls): the wait the compiler puts before a slot's
        // first MFMA then covers reads issued long ago, not the slot's own (1.5 % of the kernel).
        // kt: the step computed (its stage is (kt + base) & 1).  LOADS: the DMA of step dkt + 2 of the
        // targeted block is issued (dkt = kt, or kt - KT when the target is the next block of a
        // chain; TAIL: that is the block's last step).  NEXT: step kt + 1 exists.  Steps without LOADS
        // leave no DMA in flight.
        // BEHIND: the previous k-step issued a warm-up load after its DMA.
        template <bool LOADS, bool NEXT, bool TAIL = false>
        __device__ __forceinline__ void kstep(acc_t (&acc)[kMT][kNT], int kt, int dkt, bool behind,
                                              const Block* ahead) {
            const int cur_stage = (kt + base) & 1;
            unsigned char* const xs = smem + cur_stage * kTileBytes + w * (NT * 1024);
            unsigned char* const ys = smem + 2 * kTileBytes + cur_stage * kTileBytes + w * 8192;
            if constexpr (NT == 4) {
                half_kstep<LOADS, NEXT, TAIL>(acc, cur_stage, xs, ys, dkt, behind);
                if (LOADS) warm_step(dkt + 2 + kWarmAhead, ahead);
                return;
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                mfma_quad(acc, 0, i);
                read_item(cur_stage, 1, 2 * i);
                read_item(cur_stage, 1, 2 * i + 1);
                __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 8; i < 16; ++i) {
                mfma_quad(acc, 0, i);
                __builtin_amdgcn_sched_barrier(0);
            }
            stage_barrier(behind);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                mfma_quad(acc, 1, i);
                if (LOADS) dma_to_lds<16>(src(xg[i % NT], i, dkt + 2, TAIL), xs + i * 1024);
                if (NEXT) read_item(cur_stage ^ 1, 0, i);
                __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
                if (LOADS) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                if (NEXT) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 8; i < 16; ++i) {
                mfma_quad(acc, 1, i);
                if (LOADS) dma_to_lds<16>(src(yg[i - 8], i - 8, dkt + 2, TAIL), ys + (i - 8) * 1024);
                if (NEXT) read_item(cur_stage ^ 1, 0, i);
                __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
                if (LOADS) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                if (NEXT) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (LOADS) warm_step(dkt + 2 + kWarmAhead, ahead);
        }

        // The k-step of half a block: eight slots per slice, the twelve operand reads of a slice and the
        // twelve DMA instructions spread over them in the same order.
        template <bool LOADS, bool NEXT, bool TAIL>
        __device__ __forceinline__ void half_kstep(acc_t (&acc)[kMT][kNT], int cur_stage, unsigned char* xs,
                                                   unsigned char* ys, int dkt, bool behind) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                mfma_quad(acc, 0, i);
#pragma unroll
                for (int q = 0; q < 3; ++q) read_item(cur_stage, 1, 3 * i + q);
                __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 4; i < 8; ++i) {
                mfma_quad(acc, 0, i);
                __builtin_amdgcn_sched_barrier(0);
            }
            stage_barrier(behind);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                mfma_quad(acc, 1, i);
                if (LOADS) {
                    dma_to_lds<16>(src(xg[i % NT], i, dkt + 2, TAIL), xs + i * 1024);
                    dma_to_lds<16>(src(yg[i], i, dkt + 2, TAIL), ys + i * 1024);
                }
                if (NEXT) {
                    read_item(cur_stage ^ 1, 0, i);
                    read_item(cur_stage ^ 1, 0, 8 + i);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
                if (LOADS) __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);
                if (NEXT) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 4; i < 8; ++i) {
                mfma_quad(acc, 1, i);
                if (LOADS) dma_to_lds<16>(src(yg[i], i, dkt + 2, TAIL), ys + i * 1024);
                if (NEXT) read_item(cur_stage ^ 1, 0, i);
                __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
                if (LOADS) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                if (NEXT) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        // ---- one block per workgroup
        __device__ __forceinline__ void single(const Block& b, acc_t (&acc)[kMT][kNT]) {
            const int KT = (b.K + kBlockK - 1) / kBlockK;
            target(b);
            for (int p = 2; p < 2 + kWarmAhead; ++p) warm_step(p, nullptr);
            issue_loads(0, 0);
            __syncthreads();                   // waits for the DMA (vmcnt) and joins the waves
            if (KT > 1) issue_loads(1, 1);
#pragma unroll
            for (int item = 0; item < 8 + NT; ++item) read_item(0, 0, item);
            // a step's barrier may leave one load in flight iff the step before it had LOADS and warmed
            int kt = 0;
            for (; kt + (KTAIL ? 3 : 2) < KT; ++kt) kstep<true, true>(acc, kt, kt, kt > 0, nullptr);
            if (KTAIL && KT >= 3) {
                kstep<true, true, true>(acc, kt, kt, kt > 0, nullptr);
                ++kt;
            }
            if (KT >= 2) {
                kstep<false, true>(acc, kt, kt, kt > 0, nullptr);
                ++kt;
            }
            kstep<false, false>(acc, kt, kt, false, nullptr);
        }

        // ---- a chain of blocks
        __device__ __forceinline__ void start(const Block& first) {
            target(first);
            for (int p = 2; p < 2 + kWarmAhead; ++p) warm_step(p, nullptr);
            issue_loads(0, 0);
            issue_loads(1, 1);
            asm volatile("s_waitcnt vmcnt(16)" ::: "memory");     // step 0 has landed (loads complete in order)
        }
        // acc += the product of `cur`, the targeted block, whose k-step 0 this wavefront's DMA has
        // landed and whose k-step 1 is in flight; fetches the first two k-steps of `next`, targets
        // it and returns when this wavefront's part of its k-step 0 has landed.  The stores of the
        // caller's epilogue are never waited for on their own: the barrier of the next block's
        // k-step 0, half a step in, covers them together with the DMA of its k-step 1.
        __device__ __forceinline__ void run(const Block& cur, const Block& next, acc_t (&acc)[kMT][kNT]) {
            const int KT = uniform(cur.K / kBlockK);
            // every wavefront's part of k-step 0 has landed, and all are done with the block before
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
            for (int item = 0; item < 8 + NT; ++item) read_item(base, 0, item);
            int kt = 0;
            for (; kt + 2 + kWarmAhead < KT; ++kt) kstep<true, true>(acc, kt, kt, kt > 0, nullptr);
            // (the warm-up loads of these steps are for the first steps of `next`)
            for (; kt + 2 < KT; ++kt) kstep<true, true>(acc, kt, kt, kt > 0, &next);
            target(next);
            kstep<true, true>(acc, kt, -2, true, nullptr);
            kstep<true, false>(acc, kt + 1, -1, true, nullptr);
            // all but the 16 DMA instructions of the last half step and the warm-up load behind them
            asm volatile("s_waitcnt vmcnt(17)" ::: "memory");
            base ^= KT & 1;
        }
        __device__ __forceinline__ void finish() { stage_barrier(false); }
    };

    // One block (or half of one) on its own.
    template <bool KTAIL>
    static __device__ __forceinline__ void gemm(const Block& b, unsigned char* smem, acc_t (&acc)[kMT][kNT]) {
        Pipe<KTAIL> pipe(smem);
        pipe.single(b, acc);
    }
};
typedef DirectCoreT<8> DirectCore;
// Half a block, for a last round that leaves half of the compute units or more idle.  It reads 384
// operand rows per k-step where a whole block reads 512 for twice the work, so it takes more than half of
// a block's time.  linear 10000 x 4096 x 4096 (2.5 rounds): 784 -> 765 us; mlp 6000 x 4096 x 14336:
// 6327 -> 6082 us.  (Launches of up to some 32 blocks run on small blocks instead.)
typedef DirectCoreT<4> HalfCore;

// ---------------------------------------------------------------------------------------------
// Small blocks
// ---------------------------------------------------------------------------------------------
// For launches whose 256 x 256 blocks would leave most compute units idle.  What bounds such a launch is how fast
// one compute unit gets operands that are not in its L2: about 57 GB/s, whatever is requested ahead (some
// 45 KB in flight at the latency of the memory-side cache; from L2 it is 150 GB/s).  So the blocks are small: 8 or
// 16 times as many workgroups each fetch a half to a third of what a 128 x 256 half block does, through a
// ring of LDS stages with all the steps ahead in flight that fit.  Same interfaces as the large cores.

// Columns of a launch's small blocks, 64 or 128, or 0: large ones.  Small while they are at most one round, as
// narrow as that allows.  us per product of 64 x 64 / 64 x 128 / large blocks, captured in a graph:
//   512 x 1024 (8 large blocks), K = 256: 4.5 / 5.4 / 7.7, 768: 7.0 / 8.7 / 12.4, 8192: 41 / 58 / 97
//   1024 x 2048 (32), K = 256: 7.5 / 5.7 / 8.1, 768: 13.0 / 9.4 / 12.8, 8192: 81 / 61 / 90
//   2048 x 2048 (64), K = 256: 13.4 / 9.8 / 8.6, 768: 24 / 17 / 13.8, 8192: 152 / 116 / 90
// Weight gradients (whole linear backward calls): 512 x 1024 (8), 2048 rows: 29.9 / 34.0 / 47.6;
// 1024 x 2048 (32), 8192 rows: 94 / 80 / 131.
// count(c): the launch's blocks of 64 x c.
constexpr int kSmallRows = 64;
inline int64_t small_blocks(int64_t rows, int64_t cols, int64_t c) {
    return ((rows + kSmallRows - 1) / kSmallRows) * ((cols + c - 1) / c);
}
template <class Count>
inline int small_block_columns(Count count) {
    return count(64) <= kRound ? 64 : count(128) <= kRound ? 128 : 0;
}

// Columns of the blocks of one launch of two kinds of products, dX (count(c): its blocks of 64 x c) and weight gradients
// (count_w), or 0: a launch for each.  One while the small blocks of both are at most one round (blocks beyond it wait for a
// compute unit, which costs more than the launch).  The launch and the shorter kind cost nothing then; but where a kind would have narrower
// blocks alone, its longest block takes longer in the launch, by about 2 us (dX) or 1.4 us (weight gradients) per
// 1000 of its contraction: may_widen, may_widen_w say whether that contraction is short enough beside the other's.
template <class Count, class CountW>
inline int joint_block_columns(Count count, bool may_widen, CountW count_w, bool may_widen_w) {
    const int both = small_block_columns([&](int64_t c) { return count(c) + count_w(c); });
    if (!may_widen && small_block_columns(count) < both) return 0;
    if (!may_widen_w && small_block_columns(count_w) < both) return 0;
    return both;
}

// Waits until at most `steps` (no more than MOST) steps' DMA of PER instructions each is in flight for this wavefront,
// and for its LDS reads, then joins the wavefronts of the workgroup.
template <int PER, int MOST>
__device__ __forceinline__ void ring_barrier(int steps) {
    static_assert(PER * MOST < 64, "vmcnt has six bits");
    if constexpr (MOST == 0) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    } else {
        if (steps >= MOST) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(MOST * PER) : "memory");
        else ring_barrier<PER, MOST - 1>(steps);
    }
}

// Both operands k-contiguous, 64 (r) x 16 MT (c).  The four wavefronts lie along r, 16 rows each.
template <int MT>
struct RingCoreT {
    static_assert(MT == 2 || MT == 4 || MT == 8, "32, 64 or 128 c");
    static constexpr int kThreads = 256;
    static constexpr int kMT = MT, kNT = 1;
    static constexpr int kWaveR = 16, kWaveC = 16 * MT, kRows = 4 * kWaveR, kCols = kWaveC;
    typedef f32x4_t acc_t;
    static constexpr int kTile = 16, kRuns = 1, kGroups = 4;
    static constexpr int kXBytes = kRows * 128, kStage = kXBytes + kCols * 128;
    static constexpr int kStages = MT == 8 ? 5 : 8, kLds = kStages * kStage;      // 96, 128, 120 KB
    typedef typename DirectCoreT<8>::Block Block;

    struct Lane {
        int lane, grp, lrow, wr;
        static constexpr int wc = 0;
        __device__ __forceinline__ Lane(int tid = threadIdx.x) {
            lane = tid & 63;
            grp = lane >> 4;
            lrow = lane & 15;
            wr = tid >> 6;
        }
        __device__ __forceinline__ int r(int) const { return wr * kWaveR + lrow; }
        __device__ __forceinline__ int rbase(int) const { return wr * kWaveR; }
        __device__ __forceinline__ int cw(int mt, int /*q*/) const { return mt * 16 + grp * 4; }
        __device__ __forceinline__ int c(int mt, int q) const { return cw(mt, q); }
    };

    // As DirectCore's Block says (without the warm-up).
    template <bool KTAIL>
    static __device__ __forceinline__ void gemm(const Block& b, unsigned char* smem, acc_t (&acc)[kMT][kNT]) {
        constexpr int kXq = 2, kYq = MT / 2, kPer = kXq + kYq;    // DMA instructions per wavefront and k-step
        const int lane = threadIdx.x & 63, w = uniform((int)(threadIdx.x >> 6));
        const int lr = lane >> 3, pc = lane & 7, l15 = lane & 15, g = lane >> 4;
        auto swz = [](int row) { return (row >> 1) & 7; };
        const int KT = uniform((b.K + kBlockK - 1) / kBlockK), klast = b.K - (KT - 1) * kBlockK;
        const uint16_t* xg[kXq];
        const uint16_t* yg[kYq];
        int kx[kXq], ky[kYq];                                     // the lane's k inside a step
#pragma unroll
        for (int q = 0; q < kXq; ++q) {
            const int row = (w * kXq + q) * 8 + lr;
            kx[q] = (pc ^ swz(row)) * 8;
            xg[q] = b.X + (int64_t)(b.r0 + row < b.rows_x ? b.r0 + row : b.rows_x - 1) * b.ldx + kx[q];
        }
#pragma unroll
        for (int q = 0; q < kYq; ++q) {
            const int row = (w * kYq + q) * 8 + lr;
            ky[q] = (pc ^ swz(row)) * 8;
            if (b.Y2) {
                bool valid;
                yg[q] = paired_row<kWaveC / 2>(b.Y, b.Y2, b.ldy, b.c0, row, b.rows_y, valid) + ky[q];
            } else {
                yg[q] = b.Y + (int64_t)(b.c0 + row < b.rows_y ? b.c0 + row : b.rows_y - 1) * b.ldy + ky[q];
            }
        }
        auto issue = [&](int kt, int stage) {
            const bool tail = KTAIL && kt == KT - 1;
            auto src = [&](const uint16_t* p, int k) {
                return !tail || k < klast ? p + kt * kBlockK : reinterpret_cast<const uint16_t*>(zero_chunk);
            };
#pragma unroll
            for (int q = 0; q < kXq; ++q) dma_to_lds<16>(src(xg[q], kx[q]), smem + stage + (w * kXq + q) * 1024);
#pragma unroll
            for (int q = 0; q < kYq; ++q) dma_to_lds<16>(src(yg[q], ky[q]), smem + stage + kXBytes + (w * kYq + q) * 1024);
        };
        int rofs[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) rofs[s] = ((4 * s + g) ^ swz(l15)) * 16 + l15 * 128;

#pragma unroll
        for (int kt = 0; kt < kStages - 1; ++kt)
            if (kt < KT) issue(kt, kt * kStage);
        int cur = 0, free = (kStages - 1) * kStage;               // stages, as byte offsets
        auto next = [](int at) { return at == (kStages - 1) * kStage ? 0 : at + kStage; };
        for (int kt = 0; kt < KT; ++kt) {
            // step kt has landed, and every wavefront has read the stage of step kt - 1
            ring_barrier<kPer, kStages - 2>(KT - 1 - kt);
            if (kt + kStages - 1 < KT) issue(kt + kStages - 1, free);
            const unsigned char* const st = smem + cur;
            bf16x8_t fy[2][kMT], fx[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                fx[s] = *reinterpret_cast<const bf16x8_t*>(st + w * (kWaveR * 128) + rofs[s]);
#pragma unroll
                for (int t = 0; t < kMT; ++t)
                    fy[s][t] = *reinterpret_cast<const bf16x8_t*>(st + kXBytes + t * 2048 + rofs[s]);
            }
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int m = 0; m < kMT; ++m)
                    acc[m][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fy[s][m], fx[s], acc[m][0], 0, 0, 0);
            cur = next(cur);
            free = next(free);
        }
        __syncthreads();               // the epilogue turns its data around in the stages
    }
};

// Both operands k-major, 64 (r) x 32 CT (c).  The wavefronts share the block by k (wavefront w: the steps of 32 k w,
// w + 4, ...), which takes a third of the transposing reads that a share by columns takes, and needs no barrier in the loop:
// each has a ring of LDS stages of its own.  The partial sums are added in LDS at the end in wavefront order;
// after that a wavefront holds 32 c x 32 CT / 2 r.
template <int CT>
struct KMajorSplitT {
    static_assert(CT == 4 || CT == 2, "128 or 64 c");
    static constexpr int kThreads = 256, kWaves = 4;
    static constexpr int kRT = 2;                                 // 32-wide r tiles of the block
    static constexpr int kMT = 1, kNT = CT * kRT / kWaves;        // a wavefront's tiles of the summed block
    static constexpr int kWaveC = 32, kRows = 32 * kRT, kCols = 32 * CT;
    typedef f32x16_t acc_t;
    static constexpr int kTile = 32, kRuns = 4, kGroups = 2;
    static constexpr int kStepK = 32, kXBytes = kStepK * kRows * 2, kYRow = 64 * CT, kStage = kXBytes + kStepK * kYRow;
    static constexpr int kStages = CT == 4 ? 3 : 4, kLds = kWaves * kStages * kStage;      // 144 KB, 128 KB

    struct Lane {
        int lane, grp, lrow, wr, wc;
        __device__ __forceinline__ Lane() {
            lane = threadIdx.x & 63;
            grp = lane >> 5;
            lrow = lane & 31;
            const int wave = threadIdx.x >> 6;
            wr = wave % (kRT / kNT);
            wc = wave / (kRT / kNT);
        }
        __device__ __forceinline__ int r(int nt) const { return (wr * kNT + nt) * 32 + lrow; }
        __device__ __forceinline__ int rbase(int nt) const { return (wr * kNT + nt) * 32; }
        __device__ __forceinline__ int cw(int mt, int q) const { return mt * 32 + q * 8 + grp * 4; }
        __device__ __forceinline__ int c(int mt, int q) const { return wc * kWaveC + cw(mt, q); }
    };

    // As KMajorCore's gemm.
    template <bool KTAIL>
    static __device__ __forceinline__ void gemm(const uint16_t* __restrict__ X, int64_t ldx, int rows_x,
                                                const uint16_t* __restrict__ Y, int64_t ldy, int rows_y, int K, int r0,
                                                int c0, unsigned char* smem, acc_t (&out)[kMT][kNT],
                                                const uint16_t* /*warm*/, int64_t /*warm_stride*/) {
        const int lane = threadIdx.x & 63, w = uniform((int)(threadIdx.x >> 6));
        const int KT = uniform((K + kStepK - 1) / kStepK), klast = K - (KT - 1) * kStepK;
        const int steps = (KT - w + kWaves - 1) / kWaves;
        // LDS rows (k) of 128 bytes (64 columns), 8 per DMA instruction: granule (32 columns) g of k-row k at slot
        // g ^ (k / 2 & 1).  Of 256 bytes (128 columns), 4 per instruction: slot g ^ (k & 3).  The 4 k-rows that a
        // quarter of a transposing read covers then fall into different 64 bytes of the 256 that the banks span.
        constexpr int kXq = 4, kYq = 2 * CT, kPer = kXq + kYq, kYk = 16 / CT;    // kYk: k-rows of Y per instruction
        auto slot_x = [](int g, int k) { return g ^ ((k >> 1) & 1); };
        auto slot_y = [](int g, int k) { return CT == 4 ? g ^ (k & 3) : g ^ ((k >> 1) & 1); };
        const uint16_t* xg[kXq];
        const uint16_t* yg[kYq];
        const int xk = lane >> 3, yk = lane / (64 / kYk), ya = lane % (64 / kYk);     // (+ 8 q, + kYk q: the same slots)
        const int xc = r0 + (slot_x((lane & 7) >> 2, xk) * 4 + (lane & 3)) * 8;
        const int yc = c0 + (slot_y(ya >> 2, yk) * 4 + (ya & 3)) * 8;
#pragma unroll
        for (int q = 0; q < kXq; ++q) xg[q] = X + (int64_t)(xk + 8 * q) * ldx + (xc < rows_x ? xc : rows_x - 8);
#pragma unroll
        for (int q = 0; q < kYq; ++q) yg[q] = Y + (int64_t)(yk + kYk * q) * ldy + (yc < rows_y ? yc : rows_y - 8);
        unsigned char* const ring = smem + w * (kStages * kStage);
        auto issue = [&](int i, int stage) {
            const int kt = w + kWaves * i;
            const bool tail = KTAIL && kt == KT - 1;
            const uint16_t* const zeros = reinterpret_cast<const uint16_t*>(zero_chunk);
            const int64_t xs = (int64_t)kt * kStepK * ldx, ys = (int64_t)kt * kStepK * ldy;
#pragma unroll
            for (int q = 0; q < kXq; ++q)
                dma_to_lds<16>(!tail || xk + 8 * q < klast ? xg[q] + xs : zeros, ring + stage + q * 1024);
#pragma unroll
            for (int q = 0; q < kYq; ++q)
                dma_to_lds<16>(!tail || yk + kYk * q < klast ? yg[q] + ys : zeros, ring + stage + kXBytes + q * 1024);
        };
        // a lane's place in a transposing read of a 16-row slice: k-row 8 half + sl / 4 (see kmajor_lane_offset)
        const int sl = lane & 15, kr = 8 * (lane >> 5) + (sl >> 2), within = ((lane >> 4) & 1) * 32 + (sl & 3) * 8;
        int xofs[kRT], yofs[CT];
#pragma unroll
        for (int t = 0; t < kRT; ++t) xofs[t] = kr * 128 + slot_x(t, kr) * 64 + within;
#pragma unroll
        for (int t = 0; t < CT; ++t) yofs[t] = kXBytes + kr * kYRow + slot_y(t, kr) * 64 + within;

        acc_t acc[CT][kRT];
#pragma unroll
        for (int m = 0; m < CT; ++m)
#pragma unroll
            for (int n = 0; n < kRT; ++n)
#pragma unroll
                for (int j = 0; j < 16; ++j) acc[m][n][j] = 0.f;

        int cur = 0, free = (kStages - 1) * kStage;               // stages, as byte offsets
        auto next = [](int at) { return at == (kStages - 1) * kStage ? 0 : at + kStage; };
#pragma unroll
        for (int i = 0; i < kStages - 1; ++i)
            if (i < steps) issue(i, i * kStage);
        for (int i = 0; i < steps; ++i) {
            // this wavefront's reads of the stage that is filled next are done; then its step i has landed
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (i + kStages - 1 < steps) issue(i + kStages - 1, free);
            const int behind = steps - 1 - i;
            if (behind >= kStages - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kStages - 1) * kPer) : "memory");
            else if (kStages == 4 && behind == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kPer) : "memory");
            else if (behind >= 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kPer) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const unsigned char* const st = ring + cur;
            bf16x8_t fy[2][CT], fx[2][kRT];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
#pragma unroll
                for (int t = 0; t < kRT; ++t) fx[s][t] = read_kmajor<4 * 128>(st + xofs[t] + s * (16 * 128));
#pragma unroll
                for (int t = 0; t < CT; ++t) fy[s][t] = read_kmajor<4 * kYRow>(st + yofs[t] + s * (16 * kYRow));
            }
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int m = 0; m < CT; ++m)
#pragma unroll
                    for (int n = 0; n < kRT; ++n)
                        acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fy[s][m], fx[s][n], acc[m][n], 0, 0, 0);
            cur = next(cur);
            free = next(free);
        }
        __syncthreads();               // the rings become the place of the partial sums
        // wavefront d gets the kNT tiles d kNT .. of the block, counted r first: c tile d kNT / kRT
        constexpr int kPiece = kNT * 4096;
        auto tile = [&](int d, int n) -> acc_t& { return acc[(d * kNT + n) / kRT][(d * kNT + n) % kRT]; };
#pragma unroll
        for (int d = 0; d < kWaves; ++d) {
            if (d == w) continue;
            unsigned char* const to = smem + (d * 3 + (w < d ? w : w - 1)) * kPiece + lane * 16;
#pragma unroll
            for (int n = 0; n < kNT; ++n)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const acc_t& t = tile(d, n);
                    *reinterpret_cast<f32x4_t*>(to + (n * 4 + j) * 1024) = f32x4_t{t[4 * j], t[4 * j + 1], t[4 * j + 2], t[4 * j + 3]};
                }
        }
        __syncthreads();
#pragma unroll
        for (int d = 0; d < kWaves; ++d) {
            if (d != w) continue;
            const unsigned char* const from = smem + d * 3 * kPiece + lane * 16;
#pragma unroll
            for (int n = 0; n < kNT; ++n)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    f32x4_t sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int o = 0; o < kWaves; ++o) {
                        const acc_t& t = tile(d, n);
                        const f32x4_t v = o == d ? f32x4_t{t[4 * j], t[4 * j + 1], t[4 * j + 2], t[4 * j + 3]}
                                                 : *reinterpret_cast<const f32x4_t*>(from + (o < d ? o : o - 1) * kPiece + (n * 4 + j) * 1024);
                        sum = o == 0 ? v : sum + v;
                    }
#pragma unroll
                    for (int x = 0; x < 4; ++x) out[0][n][4 * j + x] = sum[x];
                }
        }
        __syncthreads();
    }
};

// ---------------------------------------------------------------------------------------------
// out[c][r] = in[r][c] (bf16), zeros for rows <= r < fill
// ---------------------------------------------------------------------------------------------
// Weights that a product contracts over their row index are transposed once per call, so that
// the product reads both operands along their rows (DirectCore).  in: [rows, ld_in], cols a
// multiple of 8, 16-byte aligned rows; out: [cols, ld_out], fill >= rows a multiple of 8, at most rows rounded up to 64.  One
// workgroup of 256 turns a 64 x 64 piece around in LDS; the pieces of the matrices are numbered through
// (one launch for all: each costs 4.6 us at the smallest sizes).
struct Transpose {
    const uint16_t* in;
    int rows, cols;
    int64_t ld_in;
    uint16_t* out;
    int64_t ld_out;
    int fill;
    __host__ __device__ int64_t pieces() const { return (int64_t)((rows + 63) / 64) * ((cols + 63) / 64); }
};
struct Transposes {
    Transpose m[3];            // (rows = 0: none)
    int64_t pieces() const { return m[0].pieces() + m[1].pieces() + m[2].pieces(); }
};
__device__ __forceinline__ void transpose_piece(const Transpose& t, int64_t i) {
    const uint16_t* __restrict__ const in = t.in;
    uint16_t* __restrict__ const out = t.out;
    const int rows = t.rows, cols = t.cols;
    const int64_t ld_in = t.ld_in, ld_out = t.ld_out;
    const int across = (rows + 63) / 64;
    __shared__ uint16_t piece[64][64 + 2];
    const int r0 = (int)(i % across) * 64, c0 = (int)(i / across) * 64;
    const int tid = threadIdx.x;
    // in: 64 rows x 8 chunks of 8 columns; thread -> (row tid / 8 + 32 j, chunk tid % 8)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int r = tid / 8 + 32 * j, cc = (tid % 8) * 8;
        u32x4_t x = {0u, 0u, 0u, 0u};
        if (r0 + r < rows && c0 + cc < cols)
            x = *reinterpret_cast<const u32x4_t*>(in + (int64_t)(r0 + r) * ld_in + c0 + cc);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            piece[r][cc + 2 * q] = (uint16_t)(x[q] & 0xffffu);
            piece[r][cc + 2 * q + 1] = (uint16_t)(x[q] >> 16);
        }
    }
    __syncthreads();
    // out: 64 rows (columns of in) x 8 chunks of 8
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int c = tid / 8 + 32 * j, rc = (tid % 8) * 8;
        if (c0 + c >= cols || r0 + rc >= t.fill) continue;
        u32x4_t y;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            y[q] = (uint32_t)piece[rc + 2 * q][c] | ((uint32_t)piece[rc + 2 * q + 1][c] << 16);
        *reinterpret_cast<u32x4_t*>(out + (int64_t)(c0 + c) * ld_out + r0 + rc) = y;
    }
}
static __global__ __launch_bounds__(256) void transpose_bf16_kernel(const Transposes ts, int64_t first) {
    int64_t i = first + blockIdx.x;
    int k = 0;
    for (; k < 2 && i >= ts.m[k].pieces(); ++k) i -= ts.m[k].pieces();
    transpose_piece(ts.m[k], i);
}
// (more pieces than a launch holds: several)
static inline bool launch_transposes(const Transposes& ts, hipStream_t s) {
    const int64_t pieces = ts.pieces();
    for (int64_t first = 0; first < pieces; first += kGridBlocks)
        hipLaunchKernelGGL(transpose_bf16_kernel, dim3((unsigned)(pieces - first < kGridBlocks ? pieces - first : kGridBlocks)),
                           dim3(256), 0, s, ts, first);
    return hipGetLastError() == hipSuccess;
}

// ---------------------------------------------------------------------------------------------
// Epilogues shared by the kernels built on the cores (written against the cores' layout traits)
// ---------------------------------------------------------------------------------------------
constexpr int kTurnPitch = 272;     // bytes per row of the LDS turn-around area: 256 + 16 of padding
// LDS of a kernel whose workgroups run chains of blocks (DirectCore::Pipe): the epilogue's
// turn-around area (4 wavefronts x 16 rows) lies behind the stages and the warm-up landing area,
// which belong to the next block's DMA while the epilogue runs.
constexpr int kChainTurnOffset = kLdsBytes;
constexpr int kChainLdsBytes = kChainTurnOffset + 4 * 16 * kTurnPitch;

template <class Core>
__device__ __forceinline__ void zero_acc(typename Core::acc_t (&acc)[Core::kMT][Core::kNT]) {
#pragma unroll
    for (int mt = 0; mt < Core::kMT; ++mt)
#pragma unroll
        for (int nt = 0; nt < Core::kNT; ++nt)
#pragma unroll
            for (int j = 0; j < 4 * Core::kRuns; ++j) acc[mt][nt][j] = 0.f;
}

// D[(r0 + r) * ldd + c0 + c] = bf16(acc) for the block's 256 x 256 accumulators, D row-major with c
// contiguous.  In the accumulators a lane holds 4 consecutive c of one r, so a direct store would
// scatter 8-byte pieces over many rows per instruction: each wavefront instead turns its
// kTile x 128 pieces around in LDS (free once the k-loop is over; each wavefront has its own region
// and LDS serves a wavefront's accesses in order, so no barrier is needed) and stores whole
// 256-byte row segments (non-temporal stores: the output is a stream that nothing reads back while
// it is in L2, and it would push operand lines out of there; -1 % on the K = 4096 products).
// `smem`: 4 * kTile * kTurnPitch bytes of LDS for this.
// GUARD: rows >= rows_out and 8-column chunks beyond cols_out are not written.
template <class Core, bool GUARD>
__device__ __forceinline__ void store_block_bf16(const typename Core::acc_t (&acc)[Core::kMT][Core::kNT],
                                                 uint16_t* __restrict__ D, int64_t ldd, int r0,
                                                 int c0, int rows_out, int cols_out,
                                                 unsigned char* smem) {
    const typename Core::Lane lp;
    unsigned char* const tw = smem + (threadIdx.x >> 6) * (Core::kTile * kTurnPitch);
    constexpr int kChunks = Core::kWaveC / 8, kRowsAtOnce = 64 / kChunks;
    const int lrow = lp.lane / kChunks, lcol = lp.lane % kChunks;            // 4 (8) rows x 16 (8) chunks of 16 B
    const int gc = c0 + lp.wc * Core::kWaveC + lcol * 8;
#pragma unroll
    for (int nt = 0; nt < Core::kNT; ++nt) {
#pragma unroll
        for (int mt = 0; mt < Core::kMT; ++mt)
#pragma unroll
            for (int q = 0; q < Core::kRuns; ++q) {
                bf16x4_t o;
#pragma unroll
                for (int x = 0; x < 4; ++x) o[x] = (__bf16)acc[mt][nt][q * 4 + x];
                *reinterpret_cast<bf16x4_t*>(tw + lp.lrow * kTurnPitch + lp.cw(mt, q) * 2) = o;
            }
        wave_sync<GUARD>();
#pragma unroll
        for (int it = 0; it < Core::kTile / kRowsAtOnce; ++it) {
            const int row = it * kRowsAtOnce + lrow;
            const int gr = r0 + lp.rbase(nt) + row;
            const u32x4_t v = *reinterpret_cast<const u32x4_t*>(tw + row * kTurnPitch + lcol * 16);
            if (!GUARD || (gr < rows_out && gc + 8 <= cols_out))
                __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t*>(D + (int64_t)gr * ldd + gc));
        }
        wave_sync<GUARD>();
    }
}

// Where the block of a weight-gradient product goes: element [c0 + c][r0 + r] of row-major [.., ld]
// arrays.  A gradient is the sum of several launches' products (`first` .. `last`, one launch for a
// short sequence): all but the last leave their fp32 sums in `sums`; the last adds its own to them
// and writes scale times the total to `out`.
struct GradOut {
    float* sums;             // may be `out` (fp32 overwrite)
    void* out;
    int64_t ld;
    float scale;
    int first, last;
    int f32, add;            // out: fp32 or bf16; += or =
};

// r runs along the MFMA lane dimension, so each accumulator register of a wavefront covers runs of
// kTile consecutive floats of rows of `sums` and the accumulate is one fire-and-forget fp32 atomic
// add per register (a plain store when `first`).  Each element belongs to exactly one lane per
// launch; launches on one stream are ordered, so the sums are formed in launch order: deterministic.
// The last launch's workgroups finish the gradient themselves: a separate pass over the fp32 sums
// wrote and read 8 bytes per weight more and started only when all of them were done (two
// micro-batches of 4096 rows on a 128256 x 4096 head, fp32 += : 23.6 -> 21.7 ms).  For that the
// products are turned around in LDS (`smem`, free once the k-loop is over; each wavefront has its own region), so that sums and results travel
// as whole row segments: 512 (fp32) or 256 bytes of a wavefront's 128 r, half or a quarter of that in small blocks.
// Rows r >= r_valid (a multiple of 8) and c >= c_valid are skipped.
template <class Core>
__device__ __forceinline__ void weight_grad_block(const typename Core::acc_t (&acc)[Core::kMT][Core::kNT],
                                                  const GradOut& g, int r0, int c0, int r_valid, int c_valid,
                                                  unsigned char* smem) {
    constexpr int kMT = Core::kMT, kNT = Core::kNT, kRegs = 4 * Core::kRuns;
    const typename Core::Lane lp;
    if (!g.last) {
#pragma unroll
        for (int nt = 0; nt < kNT; ++nt) {
            const int r = r0 + lp.r(nt);
            if (r >= r_valid) continue;
#pragma unroll
            for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
                for (int j = 0; j < kRegs; ++j) {
                    const int c = c0 + lp.c(mt, j >> 2) + (j & 3);
                    if (c >= c_valid) continue;
                    float* dst = g.sums + (int64_t)c * g.ld + r;
                    if (g.first) *dst = acc[mt][nt][j];
                    else unsafeAtomicAdd(dst, acc[mt][nt][j]);
                }
        }
        return;
    }
    // one row of accumulator tiles at a time: 32 c x kR r as fp32 (row pitch: two rows 4 apart, which
    // one store writes, fall into different halves of the banks), then as whole rows, 4 r per lane
    constexpr int kR = kNT * Core::kTile, kRowLanes = kR / 4, kRowsAtOnce = 64 / kRowLanes;
    static_assert((kR == 128 || kR == 64 || kR == 32) && Core::kTile == 32, "a wavefront's r; a turned piece");
    constexpr int kPitch = kR + 8, kBatch = kR == 32 ? 4 : 8;
    float* const tw = reinterpret_cast<float*>(smem) + (threadIdx.x >> 6) * (32 * kPitch);
    const int sub = lp.lane / kRowLanes, c_first = c0 + lp.wc * Core::kWaveC, rq = lp.lane % kRowLanes * 4;
    const int r = r0 + lp.wr * kR + rq;
    const bool rok = r < r_valid;
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt) {
#pragma unroll
        for (int nt = 0; nt < kNT; ++nt)
#pragma unroll
            for (int j = 0; j < kRegs; ++j)
                tw[(lp.cw(0, j >> 2) + (j & 3)) * kPitch + nt * 32 + lp.lrow] = acc[mt][nt][j];
        wave_sync<true>();
#pragma unroll 1
        for (int row0 = 0; row0 < 32; row0 += kRowsAtOnce * kBatch) {
            f32x4_t v[kBatch];
            bool ok[kBatch];
            int64_t at[kBatch];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const int c = c_first + mt * 32 + row0 + kRowsAtOnce * b + sub;
                ok[b] = rok && c < c_valid;
                at[b] = ok[b] ? (int64_t)c * g.ld + r : 0;
            }
            if (g.first) {
#pragma unroll
                for (int b = 0; b < kBatch; ++b) v[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            } else {
#pragma unroll
                for (int b = 0; b < kBatch; ++b)
                    v[b] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(g.sums + at[b]));
            }
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                v[b] += *reinterpret_cast<const f32x4_t*>(tw + (row0 + kRowsAtOnce * b + sub) * kPitch + rq);
                v[b] *= g.scale;
            }
            if (g.f32) {
                float* const out = reinterpret_cast<float*>(g.out);
                if (g.add) {
                    f32x4_t old[kBatch];
#pragma unroll
                    for (int b = 0; b < kBatch; ++b)
                        old[b] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(out + at[b]));
#pragma unroll
                    for (int b = 0; b < kBatch; ++b) v[b] += old[b];
                }
#pragma unroll
                for (int b = 0; b < kBatch; ++b)
                    if (ok[b]) __builtin_nontemporal_store(v[b], reinterpret_cast<f32x4_t*>(out + at[b]));
            } else {
                __bf16* const out = reinterpret_cast<__bf16*>(g.out);
                if (g.add) {
                    bf16x4_t old[kBatch];
#pragma unroll
                    for (int b = 0; b < kBatch; ++b)
                        old[b] = __builtin_nontemporal_load(reinterpret_cast<const bf16x4_t*>(out + at[b]));
#pragma unroll
                    for (int b = 0; b < kBatch; ++b)
#pragma unroll
                        for (int x = 0; x < 4; ++x) v[b][x] += (float)old[b][x];
                }
#pragma unroll
                for (int b = 0; b < kBatch; ++b) {
                    bf16x4_t o;
#pragma unroll
                    for (int x = 0; x < 4; ++x) o[x] = (__bf16)v[b][x];
                    if (ok[b]) __builtin_nontemporal_store(o, reinterpret_cast<bf16x4_t*>(out + at[b]));
                }
            }
        }
        wave_sync<true>();
    }
}

}  // namespace alst
