// Sequence-tiled gated MLP and sequence-tiled linear layer for gfx950: kernels and the C ABI
// (alst_mlp.h, alst_linear.h).
//
// Paper, subsection "TiledMLP": forward and backward of the MLP are run on tiles of the sequence,
// the [tile, intermediate] activations exist only for the tile in flight and backward recomputes
// them.  Per chunk of rows (below), all contractions on the block GEMM of gemm_tile.h (operands with the
// contraction index contiguous):
//
//   forward    a  = silu(x Wg^T) * (x Wu^T)   gated_kernel: both products in one block, SwiGLU in
//                                             the epilogue, g and u never reach memory
//              y  = a Wd^T
//   backward   da = dy Wd                     against Wd^T, transposed once per call
//              a, [dg | du]                   gated_kernel again (g and u recomputed), its epilogue
//                                             reads da; written into the rows of the chunk's group
//              dx = dg Wg + du Wu             one contraction over the 2 I columns of [dg | du]
//                                             against [Wg | Wu]^T, transposed once per call
//                                             (H or I not a multiple of 64 and several groups or fp32
//                                             overwrite outputs: the weights as they are, k-major operands on
//                                             MixedCore, which has no halves for a short last round; dx as two
//                                             contractions over I)
//   per group  dWg += dg^T x, dWu += du^T x, dWd += dy^T a   (fp32, contraction over the group's rows)
//
// The launches work on CHUNKS of consecutive rows whose length is chosen for the hardware
// (chunk_rows), not by the caller's tile: the tile bounds the workspace and with it the chunks, of
// the MLP forward to one tile rounded up to 256 rows, backward to a GROUP of tiles (about 16384
// rows); the linear layer has no scratch per row.  a and [dg | du] of a group are kept for the weight
// gradients, so that the read-modify-write of the fp32 sums is paid once per group.  da lives in
// a's place: the gated epilogue reads an element of da and writes a's over it, from the same lane.
// The weight gradients' operands have the contraction index (the token row) as the slow index and
// are read as they are by the k-major cores: x and dy straight from the caller's arrays, a and
// [dg | du] from the group's buffers.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <initializer_list>
#include <mutex>
#include <stdint.h>
#include <math.h>

#include "../../include/alst_mlp.h"
#include "../../include/alst_linear.h"
#include "../../include/alst_debug.h"
#include "gemm_tile.h"
#include "common.h"

namespace alst {

constexpr int kMlpGroupRows = 16384;
constexpr int kMlpGroupMax = 8;

struct MlpLayout {
    int64_t Tp;            // tile rows rounded up to 256
    int64_t chunk;         // rows per chunk of launches
    int64_t rows;          // backward: rows of a weight-gradient group, whole chunks
    size_t a, dgu, wdt, wgut, acc_g, acc_u, acc_d, total;
    bool weights_t;        // backward multiplies by transposed copies of the weights
};

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// A launch of a chunk: columns of output blocks and k-steps per block; halves: a last round of at most
// half the compute units is worked on in halves (MixedCore has none).
struct ChunkLaunch { int64_t cols, ksteps; bool halves; };
static ChunkLaunch chunk_launch(int64_t cols, int64_t k, bool halves = true) {
    return {(cols + kBlockC - 1) / kBlockC, (k + kBlockK - 1) / kBlockK, halves};
}

// Rows of a chunk, a multiple of 256 and at most `most`: the number with the least estimated time for all
// N rows, in units of a k-step of one block: per launch the rounds of the compute units times (k-steps
// per block + about 4 for its start and epilogue), and about 4 for the launch itself.  (Half of `most` and
// less is not looked at: two such chunks are one launch each fewer.)  room, group: a weight-gradient
// group of whole chunks has at most `room` rows and costs `group` 16ths of a unit.
// What a chunk's length is worth is whole rounds of its narrowest product: 65536 x 4096 x 14336 forward,
// tile 16384: 18.1 / 17.3 / 16.4 / 16.2 ms in chunks of 2048 / 5120 / 4096 / 16384 rows.  Chunks of as many
// rows as some bytes allow, whatever the rounds, were up to 6 % slower than one launch per tile of 8192 or
// more rows: linear 65536 x 4096 x 4096 forward 1.53 against 1.62 ms, MLP 65536 x 1024 x 4096 1.34
// against 1.43.
static int64_t chunk_rows(int64_t N, int64_t most, std::initializer_list<ChunkLaunch> launches, int64_t room = 0,
                          int64_t group = 0) {
    if (N <= most) return most;
    auto cost = [&](int64_t row_blocks) {
        int64_t c = 0;
        for (const ChunkLaunch& l : launches) c += rounds16(row_blocks * l.cols, l.halves) * (l.ksteps + 4) + 16 * 4;
        return c;
    };
    int64_t best = most, least = INT64_MAX;
    for (int64_t rows = most; 2 * rows > most; rows -= kBlockR) {
        const int64_t rest = (N % rows + kBlockR - 1) / kBlockR;
        int64_t c = N / rows * cost(rows / kBlockR) + (rest ? cost(rest) : 0);
        if (room) {
            const int64_t group_rows = room / rows * rows;
            c += (N + group_rows - 1) / group_rows * group;
        }
        if (c < least) { least = c; best = rows; }
    }
    return best;
}

// The most rows of a chunk whose rows are `width` elements wide: 16384, more while they stay below `bytes`
// (what a launch reads several times over, or the next launch reads again, is then mostly in the memory-side
// cache).
static int64_t chunk_rows_max(int64_t width, int64_t bytes, int64_t top) {
    return std::clamp<int64_t>(bytes / (2 * width) / kBlockR * kBlockR, 16384, top);
}
// MLP, width I: a of 16384 / 32768 / 65536 rows 32768 x 4096 x 11008 forward 6.27 / 6.36 ms, 65536 x 1024 x
// 4096 1.39 / 1.38 / 1.37.
static int64_t mlp_chunk_rows_max(int64_t I) { return chunk_rows_max(I, (int64_t)512 << 20, 65536); }

static MlpLayout make_mlp_layout(int64_t N, int64_t H, int64_t I, int64_t tile, bool backward,
                                 uint32_t flags) {
    MlpLayout L = {};
    const int64_t T = tile < N ? tile : N;
    L.Tp = (T + 255) / 256 * 256;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, 256); return at; };
    if (!backward) {
        L.chunk = chunk_rows(N, std::min(L.Tp, mlp_chunk_rows_max(I)),
                             {chunk_launch(2 * I, H), chunk_launch(H, I)});
        L.a = take((size_t)L.Tp * I * 2);
    } else {
        // a and [dg | du] of a chunk, in the room that those of a group of g tiles and the da of one
        // tile take
        int64_t g = kMlpGroupRows / L.Tp;
        g = g < 1 ? 1 : (g > kMlpGroupMax ? kMlpGroupMax : g);
        const int64_t room = (g * 3 + 1) * L.Tp / 3 / kBlockR * kBlockR;
        // fp32 overwrite outputs hold the sums themselves
        const bool in_out = (flags & ALST_FLAG_DW_FP32) && !(flags & ALST_FLAG_DW_ACCUMULATE);
        const bool whole = H % kBlockK == 0 && I % kBlockK == 0;
        // H or I that are not whole k-steps: no room of their own, but a call of one group leaves that of the sums unused
        L.weights_t = whole || (!in_out && N <= std::min(room, mlp_chunk_rows_max(I)));
        // (a group's three weight gradients: each of its blocks about 4 + 5 k-steps for its start and the
        // sums' way through memory)
        const int64_t wgrad_blocks = 3 * ((H + kBlockR - 1) / kBlockR) * ((I + kBlockC - 1) / kBlockC);
        L.chunk = chunk_rows(N, std::min(room, mlp_chunk_rows_max(I)),
                             {chunk_launch(I, H, L.weights_t), chunk_launch(2 * I, H), chunk_launch(H, 2 * I, L.weights_t)},
                             room, rounds16(wgrad_blocks) * 9);
        L.rows = room / L.chunk * L.chunk;
        L.a = take((size_t)(g * 3 + 1) * L.Tp * I * 2);
        L.dgu = L.a + (size_t)L.rows * I * 2;
        // Wd transposed [I, H] and [Wg | Wu] transposed [H, 2 I], made once per call: da = dy Wd and
        // dx = [dg | du] [Wg ; Wu] then read both operands along their rows (the fastest layout
        // of the block GEMM).
        L.wdt = take(whole ? (size_t)I * H * 2 : 0);
        L.wgut = take(whole ? (size_t)H * 2 * I * 2 : 0);
        L.acc_g = take(in_out ? 0 : (size_t)I * H * 4);
        L.acc_u = take(in_out ? 0 : (size_t)I * H * 4);
        L.acc_d = take(in_out ? 0 : (size_t)H * I * 4);
        if (L.weights_t && !whole) {
            L.wdt = L.acc_g;
            L.wgut = L.acc_u;
        }
    }
    L.total = o;
    return L;
}

// ---------------------------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------------------------
struct LinearParams {
    const uint16_t* X;       // [rows_x, ldx]   k contiguous
    const uint16_t* Y;       // [rows_y, ldy]   k contiguous: D[r][c] = sum_k X[r][k] Y[c][k], bf16
                             // [K, ldy]        k-major (y_kmajor; a weight matrix contracted over its
                             //                 row index, as it is): D[r][c] = sum_k X[r][k] Y[k][c],
                             //                 rows_y = its number of columns
    uint16_t* D;             // [.., ldd]
    const uint16_t* X2;      // second product summed into the same D (y_kmajor only, same K and
    const uint16_t* Y2;      // leading dimensions), or null
    int64_t ldx, ldy, ldd;
    int rows_x, rows_y, K;   // D is [rows_x, rows_y]; rows_y and K multiples of 8
    int y_kmajor;
};

// Up to three independent products in one launch: their output blocks are numbered
// through (gemm_tile.h), so the XCDs stay evenly loaded and the tail of one product is filled by
// the first workgroups of the next instead of leaving compute units idle.
constexpr int kMaxBatch = 3;
struct BatchMap {
    PatchGrid g[kMaxBatch];
    int first_block[kMaxBatch + 1];      // first_block[i] .. first_block[i + 1]: blocks of part i
    int n;
    Halving last;                        // (MixedCore: every block whole)
    bool rows;                           // the order of the blocks (by_rows; one product only)
    // which part and which of its blocks (or halves, see Halving) a workgroup works on; false for
    // padding workgroups
    __device__ __forceinline__ bool locate(int bid, int& which, int& tr, int& tc, int& PR, int& PC, int& half) const {
        const int number = block_of_workgroup(bid, last.numbers, rows);
        if (number < 0) return false;
        find(number, which, tr, tc, PR, PC, half);
        return true;
    }
    __device__ __forceinline__ void find(int number, int& which, int& tr, int& tc, int& PR, int& PC, int& half) const {
        const int i = last.block(number, half);
        which = 0;
#pragma unroll
        for (int k = 1; k < kMaxBatch; ++k)
            if (k < n && i >= first_block[k]) which = k;
        PR = g[which].PR;
        PC = g[which].PC;
        block_at(g[which], i - first_block[which], rows, tr, tc);
    }
};
struct LinearBatch {
    LinearParams p[kMaxBatch];
    BatchMap map;
};

// One block, or half of one, of a product of two k-contiguous operands; r0: the rows' first, tr: the
// whole block's.
template <class Core, bool KTAIL, bool GUARD>
__device__ __forceinline__ void linear_block(const LinearParams& p, int PR, int PC, int tr, int tc, int r0,
                                             unsigned char* smem) {
    const int c0 = tc * kBlockC;
    if (r0 >= p.rows_x) return;                    // (the second half of a block that has no such rows)
    typename Core::acc_t acc[Core::kMT][Core::kNT];
    zero_acc<Core>(acc);
    const uint16_t* warm = warm_row(PR, PC, p.X, p.ldx, tr * kBlockR, tr, p.Y, p.ldy, c0, tc, nullptr, p.rows_x,
                                    p.rows_y);
    Core::template gemm<KTAIL>({p.X, p.ldx, p.Y, p.ldy, p.rows_x, p.rows_y, p.K, r0, c0, warm, kBlockK, nullptr},
                               smem, acc);
    store_block_bf16<Core, GUARD>(acc, p.D, p.ldd, r0, c0, p.rows_x, p.rows_y, smem);
}

// KTAIL: K is not whole k-steps.
template <class Core, bool KTAIL>
__global__ __launch_bounds__(Core::kThreads) void linear_kernel(const LinearBatch b) {
    extern __shared__ __align__(16) unsigned char smem[];
    int which, tr, tc, PR, PC, half;
    if (!b.map.locate(blockIdx.x, which, tr, tc, PR, PC, half)) return;
    const LinearParams& p = b.p[which];
    const int r0 = tr * kBlockR, c0 = tc * kBlockC;

    if constexpr (std::is_same<Core, MixedCore>::value) {
        typename Core::acc_t acc[Core::kMT][Core::kNT];
        zero_acc<Core>(acc);
        int64_t step = 0;
        const uint16_t* warm = warm_line_mixed(PR, PC, p.X, p.ldx, r0, tr, p.Y, p.ldy, c0, tc, step, p.rows_x,
                                               p.rows_y, p.K);
        Core::template gemm<KTAIL>(p.X, p.ldx, p.rows_x, p.Y, p.ldy, p.rows_y, p.K, r0, c0, smem, acc, warm, step);
        if (p.X2) {
            __syncthreads();        // every wavefront is done with the first product's LDS stages
            warm = warm_line_mixed(PR, PC, p.X2, p.ldx, r0, tr, p.Y2, p.ldy, c0, tc, step, p.rows_x, p.rows_y, p.K);
            Core::template gemm<KTAIL>(p.X2, p.ldx, p.rows_x, p.Y2, p.ldy, p.rows_y, p.K, r0, c0, smem, acc,
                                       warm, step);
        }
        store_block_bf16<Core, true>(acc, p.D, p.ldd, r0, c0, p.rows_x, p.rows_y, smem);
    } else {
        if (half < 0) linear_block<Core, KTAIL, true>(p, PR, PC, tr, tc, r0, smem);
        else linear_block<HalfCore, KTAIL, true>(p, PR, PC, tr, tc, r0 + half * (kBlockR / 2), smem);
    }
}

// The same in small blocks (RingCoreT); the map's numbers are those of blocks of Core's size.
template <class Core, bool KTAIL>
__device__ __forceinline__ void linear_small_block(const LinearBatch& b, int number, unsigned char* smem) {
    int which, tr, tc, PR, PC, half;
    b.map.find(number, which, tr, tc, PR, PC, half);
    const LinearParams& p = b.p[which];
    const int r0 = tr * Core::kRows, c0 = tc * Core::kCols;
    typename Core::acc_t acc[Core::kMT][Core::kNT];
    zero_acc<Core>(acc);
    Core::template gemm<KTAIL>({p.X, p.ldx, p.Y, p.ldy, p.rows_x, p.rows_y, p.K, r0, c0, nullptr, 0, nullptr}, smem, acc);
    store_block_bf16<Core, true>(acc, p.D, p.ldd, r0, c0, p.rows_x, p.rows_y, smem);
}
template <class Core, bool KTAIL>
__global__ __launch_bounds__(Core::kThreads) void linear_small_kernel(const LinearBatch b) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int number = block_of_workgroup(blockIdx.x, b.map.last.numbers, false);
    if (number >= 0) linear_small_block<Core, KTAIL>(b, number, smem);
}

// The k-contiguous products on persistent workgroups: one workgroup per compute unit walks the
// launch's blocks bid = blockIdx.x, blockIdx.x + gridDim.x, ... (the same block numbering as
// linear_kernel, so the 32 workgroups of an XCD still share a patch) and fetches the first two
// k-steps of its next block while the current block's last two k-steps and epilogue run
// (DirectCore::Pipe).  total = the workgroup numbers of whole blocks; a last round in halves
// comes behind the chain.  Every product of the launch has the same K, a multiple of 64 and >= 256.
// GUARD: some product's rows or columns are not whole blocks.  HALVES: there is a last round in halves; a launch
// of whole rounds is 0.3 to 0.7 % faster without that code in it (98304 x 2048 x 8192: 2409 -> 2393 us).
template <bool GUARD, bool HALVES>
__global__ __launch_bounds__(DirectCore::kThreads) void linear_chain_kernel(const LinearBatch b, int total) {
    typedef DirectCore Core;
    extern __shared__ __align__(16) unsigned char smem[];
    // the next block number from `bid` on that is not padding, or -1
    auto next_block = [&](int bid, Core::Block& blk, int& which) {
        for (; bid < total; bid += gridDim.x) {
            int tr, tc, PR, PC, half;
            if (!b.map.locate(bid, which, tr, tc, PR, PC, half)) continue;
            const LinearParams& p = b.p[which];
            const int r0 = tr * kBlockR, c0 = tc * kBlockC;
            blk = {uniform(p.X), uniform(p.ldx), uniform(p.Y), uniform(p.ldy), uniform(p.rows_x), uniform(p.rows_y),
                   uniform(p.K), uniform(r0), uniform(c0),
                   warm_row(PR, PC, p.X, p.ldx, r0, tr, p.Y, p.ldy, c0, tc, nullptr, p.rows_x, p.rows_y), kBlockK,
                   nullptr};
            which = uniform(which);
            return uniform(bid);
        }
        return -1;
    };
    Core::Block cur, nxt;
    int which, which_next = 0;
    int bid = next_block(blockIdx.x, cur, which);
    Core::Pipe<false> pipe(smem);
    if (bid >= 0) pipe.start(cur);
    const bool chain = bid >= 0;
    while (bid >= 0) {
        const int nbid = next_block(bid + gridDim.x, nxt, which_next);
        if (nbid < 0) {            // the last block: the chain's fetch goes to this block again, unused
            nxt = cur;
            which_next = which;
        }
        typename Core::acc_t acc[Core::kMT][Core::kNT];
        zero_acc<Core>(acc);
        pipe.run(cur, nxt, acc);
        const LinearParams& p = b.p[which];
        store_block_bf16<Core, GUARD>(acc, p.D, p.ldd, cur.r0, cur.c0, p.rows_x, p.rows_y,
                                      smem + kChainTurnOffset);
        cur = nxt;
        which = which_next;
        bid = nbid;
    }
    if (chain) pipe.finish();
    if (!HALVES) return;
    for (bid = b.map.last.full + blockIdx.x; bid < b.map.last.numbers + kRound; bid += gridDim.x) {
        int tr, tc, PR, PC, half;
        if (!b.map.locate(bid, which, tr, tc, PR, PC, half) || half < 0) continue;
        __syncthreads();                // LDS is free
        linear_block<HalfCore, false, GUARD>(b.p[which], PR, PC, tr, tc, tr * kBlockR + half * (kBlockR / 2), smem);
    }
}

// Gate and up projections of a tile with the SwiGLU in the epilogue: the block's Y rows are the
// gated pair (Wg, Wu) of gemm_tile.h, so every lane holds g and u of the same elements and neither
// reaches memory.
//   forward   a = silu(g) * u
//   backward  also reads da and writes dg = da * u * silu'(g), du = da * silu(g) as [dg | du]
// g and u enter the SwiGLU as the fp32 accumulators.
struct GatedParams {
    const uint16_t* X;       // [rows_x, ldx]   the tile's rows of x
    const uint16_t* Wg;      // [I, ldw]
    const uint16_t* Wu;      // [I, ldw]
    const uint16_t* da;      // [rows_x, I]     backward; may be `a`; or null (small blocks):
    const uint16_t* dy;      // [rows_x, ldx]   da = dy Wdt^T is made here
    const uint16_t* Wdt;     // [I, ldw]        Wd transposed
    uint16_t* a;             // [rows_x, I]
    uint16_t* dgu;           // [rows_x, 2I]    backward
    int64_t ldx, ldw;
    int rows_x, I, K;
    PatchGrid grid;
    Halving last;
    bool rows;               // the order of the blocks (by_rows)
};

// 1 / (1 + exp(-g)) with the bits of the quotient: for every exp(-g) (all floats from 0 to infinity compared) the same, but for
// subnormal results (g < -87.3), a fifth of which are 2^-149 off.  v_rcp_f32, which has 1 ulp and makes those 0, and
// one step of Newton's iteration, on a quarter of the denominator so that its reciprocal is a normal number (infinity, which
// the step would turn into NaN, becomes the largest float, whose reciprocal v_rcp_f32 makes 0).  us of MLP forward and backward
// calls with the quotient / this / v_rcp_f32 alone: 16384 x 256 x 1024 219.4 / 213.5 / 209.0, 16384 x 1024 x 4096 1406 / 1392 / 1379,
// 6000 x 4096 x 14336 6023 / 6002 / 5995.
__device__ __forceinline__ float sigmoid(float g) {
    const float quarter = fminf(fmaf(__expf(-g), 0.25f, 0.25f), 3.4028234663852886e38f);
    const float r = __builtin_amdgcn_rcpf(quarter);
    return fmaf(fmaf(-quarter, r, 1.f), r, r) * 0.25f;
}

// The SwiGLU epilogue of a block whose accumulators hold g (tiles mt < kMT / 2) and u (tile mt + kMT / 2)
// of the same elements.  CHECK: rows >= rows_x and 8-column chunks beyond I are neither read nor
// written.  tw: this wavefront's LDS turn-around region (kTile rows of kTurnPitch bytes).
// OWN_DA: da is the lane's, in dacc (rounded to bf16 here, as it is on its way through memory), not in memory.
template <class Core, bool BWD, bool CHECK, bool OWN_DA = false>
__device__ __forceinline__ void gated_epilogue(const GatedParams& p,
                                               const typename Core::acc_t (&acc)[Core::kMT][Core::kNT],
                                               int r0, int c0, unsigned char* tw,
                                               const typename Core::acc_t (*dacc)[Core::kNT] = nullptr) {
    constexpr int kMT = Core::kMT, kNT = Core::kNT;
    constexpr int kHalfMT = kMT / 2;
    // Per wavefront and accumulator column nt: kTile rows x 64 (32) columns of I.  Everything that goes
    // to or comes from memory is turned around in the wavefront's own LDS region (as in
    // store_block_bf16) so that global accesses are whole 128-byte row segments.
    const typename Core::Lane lp;
    constexpr int kRuns = Core::kRuns, kTile = Core::kTile;
    constexpr int kCols = Core::kWaveC / 2, kChunks = kCols / 8, kRowsAtOnce = 64 / kChunks;
    const int lrow = lp.lane / kChunks, lcol = lp.lane % kChunks;  // 8 (16) rows x 8 (4) chunks of 16 B
    const int gc = (c0 >> 1) + lp.wc * kCols + lcol * 8;           // this lane's 8 columns of I
    const bool col_ok = !CHECK || gc + 8 <= p.I;
    const u32x4_t zero4 = {0u, 0u, 0u, 0u};
    // (da is asked for at once: tile by tile, behind the tile's stores, it was eight times a load's latency)
    u32x4_t da[BWD ? kNT : 1][kTile / kRowsAtOnce];
    if (BWD && !OWN_DA) {
#pragma unroll
        for (int nt = 0; nt < kNT; ++nt)
#pragma unroll
            for (int it = 0; it < kTile / kRowsAtOnce; ++it) {
                const int row = r0 + lp.rbase(nt) + it * kRowsAtOnce + lrow;
                const bool ok = !CHECK || (row < p.rows_x && col_ok);
                da[BWD ? nt : 0][it] = ok ? *reinterpret_cast<const u32x4_t*>(p.da + (int64_t)row * p.I + gc) : zero4;
            }
    }
#pragma unroll
    for (int nt = 0; nt < kNT; ++nt) {
        const int row0 = r0 + lp.rbase(nt);
        // the lane's own elements: row lrow of the tile, columns cw(mt, q) + x of the wavefront's 64
        auto own = [&](int mt, int q) { return tw + lp.lrow * kTurnPitch + lp.cw(mt, q) * 2; };
        auto store_rows = [&](const bf16x4_t (&v)[kHalfMT][kRuns], uint16_t* dst, int64_t ld) {
#pragma unroll
            for (int mt = 0; mt < kHalfMT; ++mt)
#pragma unroll
                for (int q = 0; q < kRuns; ++q) *reinterpret_cast<bf16x4_t*>(own(mt, q)) = v[mt][q];
            wave_sync<CHECK>();
#pragma unroll
            for (int it = 0; it < kTile / kRowsAtOnce; ++it) {
                const int row = it * kRowsAtOnce + lrow;
                const u32x4_t val = *reinterpret_cast<const u32x4_t*>(tw + row * kTurnPitch + lcol * 16);
                if (!CHECK || (row0 + row < p.rows_x && col_ok))
                    *reinterpret_cast<u32x4_t*>(dst + (int64_t)(row0 + row) * ld + gc) = val;
            }
            wave_sync<CHECK>();
        };
        bf16x4_t d[kHalfMT][kRuns];
        if (BWD && OWN_DA) {
#pragma unroll
            for (int mt = 0; mt < kHalfMT; ++mt)
#pragma unroll
                for (int q = 0; q < kRuns; ++q)
#pragma unroll
                    for (int x = 0; x < 4; ++x) d[mt][q][x] = (__bf16)dacc[mt][nt][q * 4 + x];
        } else if (BWD) {
#pragma unroll
            for (int it = 0; it < kTile / kRowsAtOnce; ++it) {
                const int row = it * kRowsAtOnce + lrow;
                *reinterpret_cast<u32x4_t*>(tw + row * kTurnPitch + lcol * 16) = da[BWD ? nt : 0][it];
            }
            wave_sync<CHECK>();
#pragma unroll
            for (int mt = 0; mt < kHalfMT; ++mt)
#pragma unroll
                for (int q = 0; q < kRuns; ++q) d[mt][q] = *reinterpret_cast<const bf16x4_t*>(own(mt, q));
            wave_sync<CHECK>();
        }
        bf16x4_t oa[kHalfMT][kRuns], og[kHalfMT][kRuns], ou[kHalfMT][kRuns];
#pragma unroll
        for (int mt = 0; mt < kHalfMT; ++mt)
#pragma unroll
            for (int q = 0; q < kRuns; ++q)
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const float g = acc[mt][nt][q * 4 + x], u = acc[mt + kHalfMT][nt][q * 4 + x];
                    const float sg = sigmoid(g);
                    const float silu = g * sg;
                    oa[mt][q][x] = (__bf16)(silu * u);
                    if (BWD) {
                        const float dd = (float)d[mt][q][x];
                        og[mt][q][x] = (__bf16)(dd * u * (sg * (1.f + g * (1.f - sg))));
                        ou[mt][q][x] = (__bf16)(dd * silu);
                    }
                }
        store_rows(oa, p.a, p.I);
        if (BWD) {
            store_rows(og, p.dgu, 2 * (int64_t)p.I);
            store_rows(ou, p.dgu + p.I, 2 * (int64_t)p.I);
        }
    }
}

// One block, or half of one; r0: the rows' first, tr: the whole block's.
template <class Core, bool BWD, bool KTAIL, bool CHECK>
__device__ __forceinline__ void gated_block(const GatedParams& p, int tr, int tc, int r0, unsigned char* smem) {
    static_assert(Core::kMT * Core::kTile == kGroupC, "a wavefront's 128 Y rows: 64 of Wg, then the same 64 of Wu");
    const int c0 = tc * kBlockC;                         // c0 / 2 = first of the block's 128 columns of I
    if (r0 >= p.rows_x) return;
    typename Core::acc_t acc[Core::kMT][Core::kNT];
    zero_acc<Core>(acc);
    const uint16_t* warm = warm_row(p.grid.PR, p.grid.PC, p.X, p.ldx, tr * kBlockR, tr, p.Wg, p.ldw, c0, tc, p.Wu,
                                    p.rows_x, p.I);
    Core::template gemm<KTAIL>({p.X, p.ldx, p.Wg, p.ldw, p.rows_x, p.I, p.K, r0, c0, warm, kBlockK, p.Wu}, smem, acc);
    gated_epilogue<Core, BWD, CHECK>(p, acc, r0, c0, smem + (threadIdx.x >> 6) * (32 * kTurnPitch));
}

// KTAIL: H is not whole k-steps.
template <bool BWD, bool KTAIL>
__global__ __launch_bounds__(DirectCore::kThreads) void gated_kernel(const GatedParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int number = block_of_workgroup(blockIdx.x, p.last.numbers, p.rows);
    if (number < 0) return;
    int tr, tc, half;
    block_at(p.grid, p.last.block(number, half), p.rows, tr, tc);
    if (half < 0) gated_block<DirectCore, BWD, KTAIL, true>(p, tr, tc, tr * kBlockR, smem);
    else gated_block<HalfCore, BWD, KTAIL, true>(p, tr, tc, tr * kBlockR + half * (kBlockR / 2), smem);
}

// The same in small blocks.  LDS: that of the rings of both products (the narrower one has more stages).
template <class Core, bool BWD>
constexpr int gated_small_lds() {
    constexpr int da = RingCoreT<Core::kMT / 2>::kLds;
    return BWD && da > Core::kLds ? da : Core::kLds;
}
template <class Core, bool BWD, bool KTAIL>
__global__ __launch_bounds__(Core::kThreads) void gated_small_kernel(const GatedParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int number = block_of_workgroup(blockIdx.x, p.last.numbers, false);
    if (number < 0) return;
    int tr, tc;
    block_at(p.grid, number, false, tr, tc);
    const int r0 = tr * Core::kRows, c0 = tc * Core::kCols;          // c0 / 2 = first of the block's 64 columns of I
    unsigned char* const tw = smem + (threadIdx.x >> 6) * (Core::kTile * kTurnPitch);
    typename Core::acc_t acc[Core::kMT][Core::kNT];
    zero_acc<Core>(acc);
    if constexpr (BWD) {
        if (p.dy) {
            // da of the block's rows and columns of I first: as a launch of its own it was 4 - 5 us more, most of them not
            // its loads (512 x 256 x 768 forward and backward: 52.4 -> 48.4 us)
            typedef RingCoreT<Core::kMT / 2> Half;
            typename Core::acc_t dacc[Half::kMT][Half::kNT];
            zero_acc<Half>(dacc);
            Half::template gemm<KTAIL>({p.dy, p.ldx, p.Wdt, p.ldw, p.rows_x, p.I, p.K, r0, c0 / 2, nullptr, 0, nullptr}, smem, dacc);
            Core::template gemm<KTAIL>({p.X, p.ldx, p.Wg, p.ldw, p.rows_x, p.I, p.K, r0, c0, nullptr, 0, p.Wu}, smem, acc);
            gated_epilogue<Core, BWD, true, true>(p, acc, r0, c0, tw, dacc);
            return;
        }
    }
    Core::template gemm<KTAIL>({p.X, p.ldx, p.Wg, p.ldw, p.rows_x, p.I, p.K, r0, c0, nullptr, 0, p.Wu}, smem, acc);
    gated_epilogue<Core, BWD, true>(p, acc, r0, c0, tw);
}

// The same on persistent workgroups (see linear_chain_kernel): K = H a multiple of 64 and >= 256.
// total = the workgroup numbers of whole blocks.  GUARD: rows_x or I is not whole blocks.
template <bool BWD, bool GUARD>
__global__ __launch_bounds__(DirectCore::kThreads) void gated_chain_kernel(const GatedParams p, int total) {
    typedef DirectCore Core;
    extern __shared__ __align__(16) unsigned char smem[];
    auto next_block = [&](int bid, Core::Block& blk) {
        for (; bid < total; bid += gridDim.x) {
            const int number = block_of_workgroup(bid, p.last.numbers, p.rows);
            if (number < 0) continue;
            int tr, tc;
            block_at(p.grid, number, p.rows, tr, tc);
            const int r0 = tr * kBlockR, c0 = tc * kBlockC;
            blk = {uniform(p.X), p.ldx, uniform(p.Wg), p.ldw, p.rows_x, p.I, p.K, uniform(r0), uniform(c0),
                   warm_row(p.grid.PR, p.grid.PC, p.X, p.ldx, r0, tr, p.Wg, p.ldw, c0, tc, p.Wu, p.rows_x, p.I),
                   kBlockK, uniform(p.Wu)};
            return uniform(bid);
        }
        return -1;
    };
    Core::Block cur, nxt;
    int bid = next_block(blockIdx.x, cur);
    Core::Pipe<false> pipe(smem);
    if (bid >= 0) pipe.start(cur);
    const bool chain = bid >= 0;
    unsigned char* const tw = smem + kChainTurnOffset + (threadIdx.x >> 6) * (Core::kTile * kTurnPitch);
    while (bid >= 0) {
        const int nbid = next_block(bid + gridDim.x, nxt);
        if (nbid < 0) nxt = cur;        // the last block: the chain's fetch goes to this block again, unused
        typename Core::acc_t acc[Core::kMT][Core::kNT];
        zero_acc<Core>(acc);
        pipe.run(cur, nxt, acc);
        gated_epilogue<Core, BWD, GUARD>(p, acc, cur.r0, cur.c0, tw);
        cur = nxt;
        bid = nbid;
    }
    if (chain) pipe.finish();
    for (bid = p.last.full + blockIdx.x; bid < p.last.numbers + kRound; bid += gridDim.x) {
        const int number = block_of_workgroup(bid, p.last.numbers, p.rows);
        if (number < p.last.full) continue;              // (none, or a whole block: the chain's)
        int tr, tc, half;
        block_at(p.grid, p.last.block(number, half), p.rows, tr, tc);
        __syncthreads();                // LDS is free
        gated_block<HalfCore, BWD, false, GUARD>(p, tr, tc, tr * kBlockR + half * (kBlockR / 2), smem);
    }
}

struct WgradParams {
    const uint16_t* X;       // [K, ldx]        r (columns 0 .. rows_x): the contiguous index of `out`
    const uint16_t* Y;       // [K, ldy]        c (columns 0 .. rows_y): the row index of `out`
    GradOut out;             // [rows_y, ld]    out[c][r] (+)= sum_k X[k][r] Y[k][c]
    int64_t ldx, ldy;
    int rows_x, rows_y, K;
};

struct WgradBatch {
    WgradParams p[kMaxBatch];
    BatchMap map;
};

// One block, or half of one (columns c0 .. c0 + 127).
template <class Core, bool KTAIL>
__device__ __forceinline__ void wgrad_block(const WgradParams& p, int r0, int c0, unsigned char* smem) {
    if (c0 >= p.rows_y) return;
    typename Core::acc_t acc[Core::kMT][Core::kNT];
    zero_acc<Core>(acc);
    Core::template gemm<KTAIL>(p.X, p.ldx, p.rows_x, p.Y, p.ldy, p.rows_y, p.K, r0, c0, smem, acc, nullptr, 0);
    weight_grad_block<Core>(acc, p.out, r0, c0, p.rows_x, p.rows_y, smem);
}

// KTAIL: K is not whole k-steps.
template <bool KTAIL>
__global__ __launch_bounds__(KMajorCore::kThreads) void wgrad_kernel(const WgradBatch b) {
    extern __shared__ __align__(16) unsigned char smem[];
    int which, tr, tc, PR, PC, half;
    if (!b.map.locate(blockIdx.x, which, tr, tc, PR, PC, half)) return;
    const WgradParams& p = b.p[which];
    if (half < 0) wgrad_block<KMajorCore, KTAIL>(p, tr * kBlockR, tc * kBlockC, smem);
    else wgrad_block<KMajorHalfCore, KTAIL>(p, tr * kBlockR, tc * kBlockC + half * (kBlockC / 2), smem);
}

// The same in small blocks.
template <class Core, bool KTAIL>
__device__ __forceinline__ void wgrad_small_block(const WgradBatch& b, int number, unsigned char* smem) {
    int which, tr, tc, PR, PC, half;
    b.map.find(number, which, tr, tc, PR, PC, half);
    wgrad_block<Core, KTAIL>(b.p[which], tr * Core::kRows, tc * Core::kCols, smem);
}
template <class Core, bool KTAIL>
__global__ __launch_bounds__(Core::kThreads) void wgrad_small_kernel(const WgradBatch b) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int number = block_of_workgroup(blockIdx.x, b.map.last.numbers, false);
    if (number >= 0) wgrad_small_block<Core, KTAIL>(b, number, smem);
}

// dx and the weight gradients of one group in one launch, both in small blocks: neither reads what the other writes, and
// with at most one round of blocks in all, each has a compute unit of its own.  Core, WgradCore: blocks of the same size.
template <class Core, class WgradCore, bool KTAIL>
__global__ __launch_bounds__(Core::kThreads) void backward_small_kernel(const LinearBatch dx, const WgradBatch dw) {
    extern __shared__ __align__(16) unsigned char smem[];
    static_assert(Core::kRows == WgradCore::kRows && Core::kCols == WgradCore::kCols && Core::kThreads == WgradCore::kThreads,
                  "one numbering of blocks");
    const int first = dx.map.last.numbers;
    const int number = block_of_workgroup(blockIdx.x, first + dw.map.last.numbers, false);
    if (number < 0) return;
    if (number < first) linear_small_block<Core, KTAIL>(dx, number, smem);
    else wgrad_small_block<WgradCore, KTAIL>(dw, number - first, smem);
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
template <class Core, class WgradCore>
constexpr int backward_small_lds() { return Core::kLds > WgradCore::kLds ? Core::kLds : WgradCore::kLds; }

static int prepare_mlp_kernels_on_current_device() {
    int rc = ALST_OK;
    auto acc = [&](int r) { if (r != ALST_OK) rc = r; };
    acc(allow_big_lds(linear_kernel<DirectCore, false>));
    acc(allow_big_lds(linear_kernel<DirectCore, true>));
    acc(allow_big_lds(linear_kernel<MixedCore, false>));
    acc(allow_big_lds(linear_kernel<MixedCore, true>));
    acc(allow_big_lds(linear_chain_kernel<false, false>, kChainLdsBytes));
    acc(allow_big_lds(linear_chain_kernel<false, true>, kChainLdsBytes));
    acc(allow_big_lds(linear_chain_kernel<true, false>, kChainLdsBytes));
    acc(allow_big_lds(linear_chain_kernel<true, true>, kChainLdsBytes));
    acc(allow_big_lds(gated_kernel<false, false>));
    acc(allow_big_lds(gated_kernel<false, true>));
    acc(allow_big_lds(gated_kernel<true, false>));
    acc(allow_big_lds(gated_kernel<true, true>));
    acc(allow_big_lds(gated_chain_kernel<false, false>, kChainLdsBytes));
    acc(allow_big_lds(gated_chain_kernel<true, false>, kChainLdsBytes));
    acc(allow_big_lds(gated_chain_kernel<false, true>, kChainLdsBytes));
    acc(allow_big_lds(gated_chain_kernel<true, true>, kChainLdsBytes));
    acc(allow_big_lds(wgrad_kernel<false>));
    acc(allow_big_lds(wgrad_kernel<true>));
    acc(allow_big_lds(linear_small_kernel<RingCoreT<4>, false>, RingCoreT<4>::kLds));
    acc(allow_big_lds(linear_small_kernel<RingCoreT<4>, true>, RingCoreT<4>::kLds));
    acc(allow_big_lds(linear_small_kernel<RingCoreT<8>, false>, RingCoreT<8>::kLds));
    acc(allow_big_lds(linear_small_kernel<RingCoreT<8>, true>, RingCoreT<8>::kLds));
    acc(allow_big_lds(gated_small_kernel<RingCoreT<4>, false, false>, gated_small_lds<RingCoreT<4>, false>()));
    acc(allow_big_lds(gated_small_kernel<RingCoreT<4>, false, true>, gated_small_lds<RingCoreT<4>, false>()));
    acc(allow_big_lds(gated_small_kernel<RingCoreT<4>, true, false>, gated_small_lds<RingCoreT<4>, true>()));
    acc(allow_big_lds(gated_small_kernel<RingCoreT<4>, true, true>, gated_small_lds<RingCoreT<4>, true>()));
    acc(allow_big_lds(gated_small_kernel<RingCoreT<8>, false, false>, gated_small_lds<RingCoreT<8>, false>()));
    acc(allow_big_lds(gated_small_kernel<RingCoreT<8>, false, true>, gated_small_lds<RingCoreT<8>, false>()));
    acc(allow_big_lds(gated_small_kernel<RingCoreT<8>, true, false>, gated_small_lds<RingCoreT<8>, true>()));
    acc(allow_big_lds(gated_small_kernel<RingCoreT<8>, true, true>, gated_small_lds<RingCoreT<8>, true>()));
    acc(allow_big_lds(wgrad_small_kernel<KMajorSplitT<2>, false>, KMajorSplitT<2>::kLds));
    acc(allow_big_lds(wgrad_small_kernel<KMajorSplitT<2>, true>, KMajorSplitT<2>::kLds));
    acc(allow_big_lds(wgrad_small_kernel<KMajorSplitT<4>, false>, KMajorSplitT<4>::kLds));
    acc(allow_big_lds(wgrad_small_kernel<KMajorSplitT<4>, true>, KMajorSplitT<4>::kLds));
    acc(allow_big_lds(backward_small_kernel<RingCoreT<4>, KMajorSplitT<2>, false>, backward_small_lds<RingCoreT<4>, KMajorSplitT<2>>()));
    acc(allow_big_lds(backward_small_kernel<RingCoreT<4>, KMajorSplitT<2>, true>, backward_small_lds<RingCoreT<4>, KMajorSplitT<2>>()));
    acc(allow_big_lds(backward_small_kernel<RingCoreT<8>, KMajorSplitT<4>, false>, backward_small_lds<RingCoreT<8>, KMajorSplitT<4>>()));
    acc(allow_big_lds(backward_small_kernel<RingCoreT<8>, KMajorSplitT<4>, true>, backward_small_lds<RingCoreT<8>, KMajorSplitT<4>>()));
    return rc;
}
// Once per device, whatever the number of host threads that make their first call together.
static int prepare_mlp_kernels() {
    static std::once_flag once[kMaxDevices];
    static int results[kMaxDevices];
    const int dev = current_device_slot();
    if (dev < 0) return ALST_ERR_HIP;
    std::call_once(once[dev], [dev] { results[dev] = prepare_mlp_kernels_on_current_device(); });
    return results[dev];
}

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Numbers the blocks of block_r x block_c of n products through; returns their number (may be beyond a launch).
template <class Batch, class Params>
static int64_t number_blocks(Batch& b, const Params* ps, int n, int block_r, int block_c) {
    b.map.n = n;
    int64_t total = 0;
    for (int i = 0; i < n; ++i) {
        const Params& p = ps[i];
        b.p[i] = p;
        b.map.first_block[i] = (int)total;
        const int tiles_r = (p.rows_x + block_r - 1) / block_r, tiles_c = (p.rows_y + block_c - 1) / block_c;
        b.map.g[i] = choose_patches(tiles_r, tiles_c);
        total += (int64_t)tiles_r * tiles_c;
    }
    for (int i = n; i <= kMaxBatch; ++i) b.map.first_block[i] = (int)total;
    b.map.last = Halving{(int)total, (int)total};
    b.map.rows = false;
    return total;
}
// Small blocks of 64 x c of the n products.
template <class Params>
static int64_t count_small(const Params* ps, int n, int64_t c) {
    int64_t total = 0;
    for (int i = 0; i < n; ++i) total += small_blocks(ps[i].rows_x, ps[i].rows_y, c);
    return total;
}
// Columns of small blocks for the n products (small_block_columns), or 0: large ones.
template <class Params>
static int small_columns(const Params* ps, int n) {
    return small_block_columns([&](int64_t c) { return count_small(ps, n, c); });
}

template <class Core>
static int launch_linear_small(const LinearParams* ps, int n, hipStream_t s) {
    LinearBatch b = {};
    const int64_t total = number_blocks(b, ps, n, Core::kRows, Core::kCols);
    bool ktail = false;
    for (int i = 0; i < n; ++i) ktail = ktail || ps[i].K % kBlockK != 0;
    const dim3 blocks((unsigned)grid_for_blocks(total)), threads(Core::kThreads);
    ProfScope pr(PROF_MLP_LINEAR, s);
    if (ktail) hipLaunchKernelGGL((linear_small_kernel<Core, true>), blocks, threads, Core::kLds, s, b);
    else hipLaunchKernelGGL((linear_small_kernel<Core, false>), blocks, threads, Core::kLds, s, b);
    return hipGetLastError() == hipSuccess ? ALST_OK : ALST_ERR_HIP;
}

// What a launch runs on: small blocks of that many columns, or (0) large ones, one a workgroup or in chains.
struct BlockChoice {
    int columns;
    bool chain;
};
static BlockChoice choose_linear(const LinearParams* ps, int n) {
    BlockChoice c = {};
    if (ps[0].y_kmajor) return c;
    c.columns = small_columns(ps, n);
    if (c.columns) return c;
    int64_t total = 0;
    bool one_k = true;                                            // (a chain is of one K)
    for (int i = 0; i < n; ++i) {
        total += (int64_t)((ps[i].rows_x + kBlockR - 1) / kBlockR) * ((ps[i].rows_y + kBlockC - 1) / kBlockC);
        one_k = one_k && ps[i].K == ps[0].K;
    }
    c.chain = one_k && chain_pays(total, ps[0].K, false);
    return c;
}

// One launch for the n products (n <= kMaxBatch), all of one kind (y_kmajor).
static int launch_linear(const LinearParams* ps, int n, hipStream_t s) {
    const auto [columns, chain] = choose_linear(ps, n);
    if (columns == 64) return launch_linear_small<RingCoreT<4>>(ps, n, s);
    if (columns == 128) return launch_linear_small<RingCoreT<8>>(ps, n, s);
    LinearBatch b = {};
    const int64_t total = number_blocks(b, ps, n, kBlockR, kBlockC);
    if (total > 0x7fffff00) return ALST_ERR_SHAPE;
    bool guard = false, ktail = false;
    for (int i = 0; i < n; ++i) {
        const LinearParams& p = ps[i];
        guard = guard || p.rows_x % kBlockR != 0 || p.rows_y % kBlockC != 0;
        ktail = ktail || p.K % kBlockK != 0;
    }
    if (!ps[0].y_kmajor) b.map.last = halve_last_round((int)total);
    b.map.rows = n == 1 && !ps[0].y_kmajor && by_rows(b.map.g[0], ps[0].K);
    const int blocks = grid_for_blocks(total);
    const int whole = grid_for_blocks(b.map.last.full);           // the chains' workgroup numbers
    ProfScope pr(PROF_MLP_LINEAR, s);
    const dim3 all((unsigned)blocks), persistent((unsigned)std::min(blocks, persistent_grid()));
    const dim3 threads(DirectCore::kThreads);
    if (ps[0].y_kmajor && ktail)
        hipLaunchKernelGGL((linear_kernel<MixedCore, true>), all, threads, kLdsBytes, s, b);
    else if (ps[0].y_kmajor)
        hipLaunchKernelGGL((linear_kernel<MixedCore, false>), all, threads, kLdsBytes, s, b);
    else if (chain && b.map.last.numbers != (int)total) {
        if (guard) hipLaunchKernelGGL((linear_chain_kernel<true, true>), persistent, threads, kChainLdsBytes, s, b, whole);
        else hipLaunchKernelGGL((linear_chain_kernel<false, true>), persistent, threads, kChainLdsBytes, s, b, whole);
    } else if (chain && guard)
        hipLaunchKernelGGL((linear_chain_kernel<true, false>), persistent, threads, kChainLdsBytes, s, b, whole);
    else if (chain)
        hipLaunchKernelGGL((linear_chain_kernel<false, false>), persistent, threads, kChainLdsBytes, s, b, whole);
    else if (ktail)
        hipLaunchKernelGGL((linear_kernel<DirectCore, true>), all, threads, kLdsBytes, s, b);
    else
        hipLaunchKernelGGL((linear_kernel<DirectCore, false>), all, threads, kLdsBytes, s, b);
    return hipGetLastError() == hipSuccess ? ALST_OK : ALST_ERR_HIP;
}

static int launch_linear(const LinearParams& p, hipStream_t s) { return launch_linear(&p, 1, s); }

template <class Core>
static int launch_wgrad_small(const WgradParams* ps, int n, hipStream_t s) {
    WgradBatch b = {};
    const int64_t total = number_blocks(b, ps, n, Core::kRows, Core::kCols);
    const dim3 blocks((unsigned)grid_for_blocks(total)), threads(Core::kThreads);
    ProfScope pr(PROF_MLP_WGRAD, s);
    if (ps[0].K % kBlockK != 0) hipLaunchKernelGGL((wgrad_small_kernel<Core, true>), blocks, threads, Core::kLds, s, b);
    else hipLaunchKernelGGL((wgrad_small_kernel<Core, false>), blocks, threads, Core::kLds, s, b);
    return hipGetLastError() == hipSuccess ? ALST_OK : ALST_ERR_HIP;
}

// The n weight-gradient products (n <= kMaxBatch, all with the same K) in one launch.
static int launch_wgrad(const WgradParams* ps, int n, hipStream_t s) {
    const int columns = small_columns(ps, n);
    if (columns == 64) return launch_wgrad_small<KMajorSplitT<2>>(ps, n, s);
    if (columns == 128) return launch_wgrad_small<KMajorSplitT<4>>(ps, n, s);
    WgradBatch b = {};
    const int64_t total = number_blocks(b, ps, n, kBlockR, kBlockC);
    if (total > 0x7fffff00) return ALST_ERR_SHAPE;
    b.map.last = halve_last_round((int)total);
    const dim3 blocks((unsigned)grid_for_blocks(total)), threads(KMajorCore::kThreads);
    ProfScope pr(PROF_MLP_WGRAD, s);
    if (ps[0].K % kBlockK != 0)
        hipLaunchKernelGGL((wgrad_kernel<true>), blocks, threads, kLdsBytes, s, b);
    else
        hipLaunchKernelGGL((wgrad_kernel<false>), blocks, threads, kLdsBytes, s, b);
    return hipGetLastError() == hipSuccess ? ALST_OK : ALST_ERR_HIP;
}

static int launch_wgrad(const WgradParams& p, hipStream_t s) { return launch_wgrad(&p, 1, s); }

template <class Core, class WgradCore>
static int launch_backward_small(const LinearParams& lp, const WgradParams* ps, int n, hipStream_t s) {
    LinearBatch dx = {};
    WgradBatch dw = {};
    const int64_t total = number_blocks(dx, &lp, 1, Core::kRows, Core::kCols) +
                          number_blocks(dw, ps, n, WgradCore::kRows, WgradCore::kCols);
    const dim3 blocks((unsigned)grid_for_blocks(total)), threads(Core::kThreads);
    constexpr int lds = backward_small_lds<Core, WgradCore>();
    ProfScope pr(PROF_MLP_WGRAD, s);
    if (lp.K % kBlockK != 0 || ps[0].K % kBlockK != 0)
        hipLaunchKernelGGL((backward_small_kernel<Core, WgradCore, true>), blocks, threads, lds, s, dx, dw);
    else hipLaunchKernelGGL((backward_small_kernel<Core, WgradCore, false>), blocks, threads, lds, s, dx, dw);
    return hipGetLastError() == hipSuccess ? ALST_OK : ALST_ERR_HIP;
}

// dx (lp) and the n weight gradients of the group that it completes, in one launch or two.  us of a backward call, two launches /
// one (N x K x M, N x H x I):
//   nothing wider: linear 3800 x 256 x 256 28.8 / 25.8, MLP 2000 x 256 x 512 40.5 / 32.6
//   the weights' blocks wider, their contraction N at most 512 + 6 times dx's: linear 512 x 1024 x 1024 23.1 / 20.1, 4096 x 256 x
//     1024 34.1 / 31.0, 3000 x 512 x 512 29.7 / 29.5, MLP 4000 x 256 x 512 60.5 / 57.0, 6000 x 256 x 512 70.8 / 66.8
//   beyond: linear 2000 x 512 x 200 23.8 / 25.8, 4000 x 256 x 256 29.3 / 33.8, 7900 x 256 x 256 41.9 / 50.3, 14000 x 128 x 256 58.9 / 75.9, MLP
//     7000 x 256 x 256 64.1 / 68.1, 12000 x 128 x 256 78.2 / 89.7
//   dx's blocks wider, its contraction at most 2048 (beside three weight gradients 3072) more than N: linear 2000 x 256 x 3072
//     38.5 / 37.3, 1000 x 320 x 3000 38.6 / 37.4, 600 x 384 x 2600 33.6 / 34.2, MLP 400 x 256 x 1400 46.9 / 45.5
//   beyond: linear 300 x 512 x 2560 31.3 / 33.8, 1000 x 256 x 4096 39.6 / 45.1, 500 x 128 x 8192 55.3 / 75.5, MLP 256 x 128 x 4096 64.8 / 77.3
static int choose_together(const LinearParams& lp, const WgradParams* ps, int n) {       // columns of the blocks, or 0: two launches
    if (lp.y_kmajor) return 0;
    const int64_t k = lp.K, k_w = ps[0].K;
    return joint_block_columns([&](int64_t c) { return small_blocks(lp.rows_x, lp.rows_y, c); }, k <= (n > 1 ? 3072 : 2048) + k_w,
                               [&](int64_t c) { return count_small(ps, n, c); }, k_w <= 512 + 6 * k);
}
static int launch_backward(const LinearParams& lp, const WgradParams* ps, int n, hipStream_t s) {
    const int columns = choose_together(lp, ps, n);
    if (columns == 64) return launch_backward_small<RingCoreT<4>, KMajorSplitT<2>>(lp, ps, n, s);
    if (columns == 128) return launch_backward_small<RingCoreT<8>, KMajorSplitT<4>>(lp, ps, n, s);
    const int rc = launch_linear(lp, s);
    return rc == ALST_OK ? launch_wgrad(ps, n, s) : rc;
}

struct MlpProblem {
    const uint16_t *x, *Wg, *Wu, *Wd, *dy;
    uint16_t *y, *dx;
    void *dWg, *dWu, *dWd;
    int64_t N, H, I, tile;
    unsigned char* ws;
    uint32_t flags;
    hipStream_t stream;
};

static int validate_mlp(const MlpProblem& P, size_t workspace_bytes, bool backward) {
    if (!P.x || !P.Wg || !P.Wu || !P.Wd || !P.ws) return ALST_ERR_NULL;
    if (!backward && !P.y) return ALST_ERR_NULL;
    if (backward && (!P.dy || !P.dx || !P.dWg || !P.dWu || !P.dWd)) return ALST_ERR_NULL;
    if (P.flags & ~(ALST_FLAG_DW_FP32 | ALST_FLAG_DW_ACCUMULATE)) return ALST_ERR_UNSUPPORTED;
    if (P.N < 1 || P.H < 1 || P.I < 1 || P.tile < 1) return ALST_ERR_SHAPE;
    if (P.N > (int64_t)1 << 30 || P.H > (int64_t)1 << 20 || P.I > (int64_t)1 << 20) return ALST_ERR_SHAPE;
    if (P.H % 8 != 0 || P.I % 8 != 0) return ALST_ERR_ALIGN;
    const void* ptrs[] = {P.x, P.Wg, P.Wu, P.Wd, P.ws, P.y, P.dy, P.dx, P.dWg, P.dWu, P.dWd};
    for (const void* q : ptrs)
        if (q && !aligned16(q)) return ALST_ERR_ALIGN;
    const MlpLayout L = make_mlp_layout(P.N, P.H, P.I, P.tile, backward, P.flags);
    // every launch must fit its grid (the widest are [T, 2I] and [2I, H] outputs)
    if (!checked_grid(L.Tp / kBlockR, (2 * P.I + kBlockC - 1) / kBlockC) ||
        !checked_grid((P.I + kBlockR - 1) / kBlockR, (P.H + kBlockC - 1) / kBlockC))
        return ALST_ERR_SHAPE;
    if (workspace_bytes < L.total) return ALST_ERR_WORKSPACE;
    return ALST_OK;
}

template <class Core>
static int launch_gated_small(GatedParams gp, bool bwd, hipStream_t s) {
    gp.grid = choose_patches((gp.rows_x + Core::kRows - 1) / Core::kRows, (2 * gp.I + Core::kCols - 1) / Core::kCols);
    gp.last = {gp.grid.blocks(), gp.grid.blocks()};
    const dim3 blocks((unsigned)grid_for_blocks(gp.grid.blocks())), threads(Core::kThreads);
    const bool ktail = gp.K % kBlockK != 0;
    ProfScope pr(PROF_MLP_LINEAR, s);
    const int lds = bwd ? gated_small_lds<Core, true>() : gated_small_lds<Core, false>();
    if (ktail && bwd) hipLaunchKernelGGL((gated_small_kernel<Core, true, true>), blocks, threads, lds, s, gp);
    else if (ktail) hipLaunchKernelGGL((gated_small_kernel<Core, false, true>), blocks, threads, lds, s, gp);
    else if (bwd) hipLaunchKernelGGL((gated_small_kernel<Core, true, false>), blocks, threads, lds, s, gp);
    else hipLaunchKernelGGL((gated_small_kernel<Core, false, false>), blocks, threads, lds, s, gp);
    return hipGetLastError() == hipSuccess ? ALST_OK : ALST_ERR_HIP;
}

static BlockChoice choose_gated(int rows, int64_t H, int64_t I) {
    BlockChoice c = {};
    c.columns = small_block_columns([&](int64_t cols) { return small_blocks(rows, 2 * I, cols); });
    if (!c.columns) c.chain = chain_pays((rows + kBlockR - 1) / kBlockR * ((I + 127) / 128), H, true);
    return c;
}
// a = silu(x_t Wg^T) * (x_t Wu^T) for `rows` rows of x; backward (da given, or dy_t and Wd transposed to make it from
// if the blocks are small): also [dg | du].
static int launch_gated(const MlpProblem& P, const uint16_t* x_t, int rows, const uint16_t* da, uint16_t* a,
                        uint16_t* dgu, hipStream_t s, const uint16_t* dy_t = nullptr, const uint16_t* wdt = nullptr) {
    GatedParams gp = {};
    gp.dy = dy_t; gp.Wdt = wdt;
    gp.X = x_t; gp.ldx = P.H; gp.rows_x = rows; gp.K = (int)P.H;
    gp.Wg = P.Wg; gp.Wu = P.Wu; gp.ldw = P.H; gp.I = (int)P.I;
    gp.da = da; gp.a = a; gp.dgu = dgu;
    const auto [columns, chain] = choose_gated(rows, P.H, P.I);
    if (columns == 64) return launch_gated_small<RingCoreT<4>>(gp, dgu != nullptr, s);
    if (columns == 128) return launch_gated_small<RingCoreT<8>>(gp, dgu != nullptr, s);
    gp.grid = choose_patches((rows + kBlockR - 1) / kBlockR, (int)((P.I + 127) / 128));
    gp.last = halve_last_round(gp.grid.blocks());
    gp.rows = by_rows(gp.grid, gp.K);
    const int blocks = grid_for_blocks(gp.grid.blocks()), whole = grid_for_blocks(gp.last.full);
    const bool guard = rows % kBlockR != 0 || P.I % 128 != 0, ktail = P.H % kBlockK != 0;
    const dim3 all((unsigned)blocks), persistent((unsigned)std::min(blocks, persistent_grid()));
    const dim3 threads(DirectCore::kThreads);
    ProfScope pr(PROF_MLP_LINEAR, s);
    if (chain) {
        if (guard && da) hipLaunchKernelGGL((gated_chain_kernel<true, true>), persistent, threads, kChainLdsBytes, s, gp, whole);
        else if (guard) hipLaunchKernelGGL((gated_chain_kernel<false, true>), persistent, threads, kChainLdsBytes, s, gp, whole);
        else if (da) hipLaunchKernelGGL((gated_chain_kernel<true, false>), persistent, threads, kChainLdsBytes, s, gp, whole);
        else hipLaunchKernelGGL((gated_chain_kernel<false, false>), persistent, threads, kChainLdsBytes, s, gp, whole);
    } else if (ktail && da) hipLaunchKernelGGL((gated_kernel<true, true>), all, threads, kLdsBytes, s, gp);
    else if (ktail) hipLaunchKernelGGL((gated_kernel<false, true>), all, threads, kLdsBytes, s, gp);
    else if (da) hipLaunchKernelGGL((gated_kernel<true, false>), all, threads, kLdsBytes, s, gp);
    else hipLaunchKernelGGL((gated_kernel<false, false>), all, threads, kLdsBytes, s, gp);
    return hipGetLastError() == hipSuccess ? ALST_OK : ALST_ERR_HIP;
}

static int run_mlp_forward(const MlpProblem& P) {
    int rc = prepare_mlp_kernels();
    if (rc != ALST_OK) return rc;
    const MlpLayout L = make_mlp_layout(P.N, P.H, P.I, P.tile, false, P.flags);
    hipStream_t s = P.stream;
    uint16_t* a = reinterpret_cast<uint16_t*>(P.ws + L.a);
    const int H = (int)P.H, I = (int)P.I;
    for (int64_t i0 = 0; i0 < P.N; i0 += L.chunk) {
        const int rows = (int)std::min(L.chunk, P.N - i0);
        rc = launch_gated(P, P.x + i0 * P.H, rows, nullptr, a, nullptr, s);
        if (rc != ALST_OK) return rc;
        LinearParams lp = {};
        lp.X = a; lp.ldx = I; lp.rows_x = rows; lp.K = I;
        lp.Y = P.Wd; lp.ldy = I; lp.rows_y = H;
        lp.D = P.y + i0 * P.H; lp.ldd = H;
        rc = launch_linear(lp, s);
        if (rc != ALST_OK) return rc;
    }
    return ALST_OK;
}

// The extents of backward's products: dx of `rows` rows, the three weight gradients of a group of `rows` rows.
static LinearParams mlp_dx_extents(const MlpLayout& L, int rows, int H, int I) {
    LinearParams lp = {};
    lp.rows_x = rows; lp.ldx = 2 * (int64_t)I; lp.rows_y = H; lp.ldd = H;
    if (L.weights_t) {
        // one contraction over the 2 I columns of [dg | du] against [Wg | Wu]^T [H, 2 I]
        lp.K = 2 * I; lp.ldy = 2 * (int64_t)I;
    } else {
        // two contractions over I summed in the accumulators, the weights [I, H] as they are: k = i
        lp.K = I; lp.ldy = H; lp.y_kmajor = 1;
    }
    return lp;
}
static void mlp_wgrad_extents(WgradParams (&wp)[kMaxBatch], int64_t rows, int H, int I) {
    wp[0] = {};
    wp[0].K = (int)rows;
    wp[0].ldx = H; wp[0].rows_x = H;                    // x
    wp[0].ldy = 2 * (int64_t)I; wp[0].rows_y = I;       // dg
    wp[1] = wp[0];                                      // x, du
    wp[2] = wp[0];
    wp[2].ldx = I; wp[2].rows_x = I;                    // a
    wp[2].ldy = H; wp[2].rows_y = H;                    // dy
}

static int run_mlp_backward(const MlpProblem& P) {
    int rc = prepare_mlp_kernels();
    if (rc != ALST_OK) return rc;
    const MlpLayout L = make_mlp_layout(P.N, P.H, P.I, P.tile, true, P.flags);
    hipStream_t s = P.stream;
    uint16_t* a = reinterpret_cast<uint16_t*>(P.ws + L.a);
    uint16_t* dgu = reinterpret_cast<uint16_t*>(P.ws + L.dgu);
    const bool f32 = P.flags & ALST_FLAG_DW_FP32, accum = P.flags & ALST_FLAG_DW_ACCUMULATE;
    const bool in_out = f32 && !accum;
    float* acc_g = in_out ? reinterpret_cast<float*>(P.dWg) : reinterpret_cast<float*>(P.ws + L.acc_g);
    float* acc_u = in_out ? reinterpret_cast<float*>(P.dWu) : reinterpret_cast<float*>(P.ws + L.acc_u);
    float* acc_d = in_out ? reinterpret_cast<float*>(P.dWd) : reinterpret_cast<float*>(P.ws + L.acc_d);
    const int H = (int)P.H, I = (int)P.I;
    const int64_t I2 = 2 * (int64_t)I;

    uint16_t* wdt = reinterpret_cast<uint16_t*>(P.ws + L.wdt);
    uint16_t* wgut = reinterpret_cast<uint16_t*>(P.ws + L.wgut);
    if (L.weights_t) {
        ProfScope ps(PROF_MLP_OTHER, s);
        const Transposes ts = {{{P.Wd, H, I, I, wdt, H, H}, {P.Wg, I, H, H, wgut, I2, I}, {P.Wu, I, H, H, wgut + I, I2, I}}};
        if (!launch_transposes(ts, s)) return ALST_ERR_HIP;
    }

    for (int64_t i0 = 0; i0 < P.N; i0 += L.chunk) {
        const int rows = (int)std::min(L.chunk, P.N - i0);
        const int64_t group0 = i0 / L.rows * L.rows;         // first row of the chunk's group
        uint16_t* const a_c = a + (i0 - group0) * I;
        uint16_t* const dgu_c = dgu + (i0 - group0) * I2;
        const uint16_t* x_c = P.x + i0 * P.H;
        const uint16_t* dy_c = P.dy + i0 * P.H;

        if (L.weights_t && choose_gated(rows, H, I).columns) {
            rc = launch_gated(P, x_c, rows, nullptr, a_c, dgu_c, s, dy_c, wdt);
            if (rc != ALST_OK) return rc;
        } else {   // da = dy Wd (contraction over H), then g and u again with a, dg, du made in the epilogue
            LinearParams lp = {};
            lp.X = dy_c; lp.ldx = H; lp.rows_x = rows; lp.K = H;
            if (L.weights_t) { lp.Y = wdt; lp.ldy = H; lp.rows_y = I; }            // Wd^T [I, H]
            else { lp.Y = P.Wd; lp.ldy = I; lp.rows_y = I; lp.y_kmajor = 1; }      // Wd [H, I]: k = h
            lp.D = a_c; lp.ldd = I;
            rc = launch_linear(lp, s);
            if (rc == ALST_OK) rc = launch_gated(P, x_c, rows, a_c, a_c, dgu_c, s);
            if (rc != ALST_OK) return rc;
        }
        // dx = dg Wg + du Wu
        LinearParams lp = mlp_dx_extents(L, rows, H, I);
        lp.X = dgu_c; lp.D = P.dx + i0 * P.H;
        if (L.weights_t) lp.Y = wgut;
        else { lp.Y = P.Wg; lp.X2 = dgu_c + I; lp.Y2 = P.Wu; }
        const int64_t in_group = i0 + rows - group0;
        if (in_group < L.rows && i0 + rows < P.N) {
            rc = launch_linear(lp, s);
            if (rc != ALST_OK) return rc;
            continue;
        }
        // the group is complete
        GradOut out = {nullptr, nullptr, 0, 1.f, group0 == 0, i0 + rows == P.N, f32, accum};
        auto into = [&](float* sums, void* dW, int64_t ld) { out.sums = sums; out.out = dW; out.ld = ld; return out; };
        WgradParams wp[kMaxBatch];
        mlp_wgrad_extents(wp, in_group, H, I);
        wp[0].X = P.x + group0 * H; wp[0].Y = dgu; wp[0].out = into(acc_g, P.dWg, H);                     // dWg[i][h]
        wp[1].X = P.x + group0 * H; wp[1].Y = dgu + I; wp[1].out = into(acc_u, P.dWu, H);                 // dWu[i][h]
        wp[2].X = a; wp[2].Y = P.dy + group0 * H; wp[2].out = into(acc_d, P.dWd, I);                      // dWd[h][i]
        // (weights transposed into the room of the sums: a call of one group, whose gradients don't touch the sums)
        rc = launch_backward(lp, wp, 3, s);
        if (rc != ALST_OK) return rc;
    }
    return ALST_OK;
}

// ---------------------------------------------------------------------------------------------
// the single tiled linear layer: y = x W^T, dx = dy W, dW = dy^T x
// ---------------------------------------------------------------------------------------------
// Rows of a launch of D [N, M] = X [N, K] Y.  One launch for all rows if a row of X is read once (an output of
// at most 8 columns of blocks, a patch's width: 131072 x 1024 x 1024 forward 223 us, in two launches 230;
// 4 M rows are 64 whole rounds and more, far from the limit of a grid); else 16384, more while a chunk of X stays below 128 MB: 32768 x 5120 x 16384 forward 3.80 / 3.92 ms with
// 16384 / 32768 rows.
static int64_t lin_chunk_rows(int64_t N, int64_t K, int64_t M, bool halves = true) {
    const int64_t all = (N + kBlockR - 1) / kBlockR * kBlockR;
    if (M <= 8 * kBlockC) return std::min(all, (int64_t)1 << 22);
    return chunk_rows(N, std::min(all, chunk_rows_max(K, (int64_t)128 << 20, 262144)), {chunk_launch(M, K, halves)});
}

struct LinLayout {
    int64_t Tp;
    size_t acc, wt, total;
    bool weight_t;         // backward multiplies dy by a transposed copy of W
};

// Rows of a weight-gradient group.
static int64_t lin_group_rows(const LinLayout& L) { return std::max<int64_t>(kMlpGroupRows, L.Tp); }

static LinLayout make_lin_layout(int64_t N, int64_t K, int64_t M, int64_t tile, bool backward,
                                 uint32_t flags) {
    LinLayout L = {};
    const int64_t T = tile < N ? tile : N;
    L.Tp = (T + 255) / 256 * 256;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, 256); return at; };
    if (backward) {
        const bool in_out = (flags & ALST_FLAG_DW_FP32) && !(flags & ALST_FLAG_DW_ACCUMULATE);
        L.acc = take(in_out ? 0 : (size_t)M * K * 4);
        // W transposed [K, M], made once per call: dx = dy W then reads both operands along their
        // rows (the fastest layout of the block GEMM).  M that is not whole k-steps: no room of its own, but a call of one
        // group leaves that of the sums unused; else W is read as it is.
        const bool whole = M % kBlockK == 0;
        L.weight_t = whole || (!in_out && N <= lin_group_rows(L));
        L.wt = take(whole ? (size_t)K * M * 2 : 0);
        if (!whole) L.wt = L.acc;
    }
    L.total = o;
    return L;
}

struct LinProblem {
    const uint16_t *x, *W, *dy;
    uint16_t *y, *dx;
    void* dW;
    int64_t N, K, M, tile;
    unsigned char* ws;
    uint32_t flags;
    hipStream_t stream;
};

static int validate_lin(const LinProblem& P, size_t workspace_bytes, bool backward) {
    if (!P.x || !P.W) return ALST_ERR_NULL;
    if (!backward && !P.y) return ALST_ERR_NULL;
    if (backward && (!P.dy || !P.dx || !P.dW)) return ALST_ERR_NULL;
    if (P.flags & ~(ALST_FLAG_DW_FP32 | ALST_FLAG_DW_ACCUMULATE)) return ALST_ERR_UNSUPPORTED;
    if (P.N < 1 || P.K < 1 || P.M < 1 || P.tile < 1) return ALST_ERR_SHAPE;
    if (P.N > (int64_t)1 << 30 || P.K > (int64_t)1 << 20 || P.M > (int64_t)1 << 24) return ALST_ERR_SHAPE;
    // (forward needs no scratch)
    if (make_lin_layout(P.N, P.K, P.M, P.tile, backward, P.flags).total > 0 && !P.ws) return ALST_ERR_NULL;
    if (P.K % 8 != 0 || P.M % 8 != 0) return ALST_ERR_ALIGN;
    const void* ptrs[] = {P.x, P.W, P.dy, P.y, P.dx, P.dW, P.ws};
    for (const void* q : ptrs)
        if (q && !aligned16(q)) return ALST_ERR_ALIGN;
    const LinLayout L = make_lin_layout(P.N, P.K, P.M, P.tile, backward, P.flags);
    if (!checked_grid(L.Tp / kBlockR, (P.M + kBlockC - 1) / kBlockC) ||
        !checked_grid((P.K + kBlockR - 1) / kBlockR, (P.M + kBlockC - 1) / kBlockC))
        return ALST_ERR_SHAPE;
    if (workspace_bytes < L.total) return ALST_ERR_WORKSPACE;
    return ALST_OK;
}

static int run_lin_forward(const LinProblem& P) {
    int rc = prepare_mlp_kernels();
    if (rc != ALST_OK) return rc;
    const int64_t chunk = lin_chunk_rows(P.N, P.K, P.M);
    for (int64_t i0 = 0; i0 < P.N; i0 += chunk) {
        LinearParams lp = {};
        lp.X = P.x + i0 * P.K; lp.ldx = P.K; lp.rows_x = (int)std::min(chunk, P.N - i0); lp.K = (int)P.K;
        lp.Y = P.W; lp.ldy = P.K; lp.rows_y = (int)P.M;
        lp.D = P.y + i0 * P.M; lp.ldd = P.M;
        rc = launch_linear(lp, P.stream);
        if (rc != ALST_OK) return rc;
    }
    return ALST_OK;
}

// The extents of backward's products: dx of `rows` rows, dW of a group of `rows` rows.
static LinearParams lin_dx_extents(const LinLayout& L, int rows, int K, int M) {
    LinearParams lp = {};
    lp.rows_x = rows; lp.ldx = M; lp.K = M; lp.rows_y = K; lp.ldd = K;
    if (L.weight_t) lp.ldy = M;                         // W^T [K, M]
    else { lp.ldy = K; lp.y_kmajor = 1; }               // W [M, K]: k = m
    return lp;
}
static WgradParams lin_wgrad_extents(int64_t rows, int K, int M) {
    WgradParams wp = {};
    wp.K = (int)rows;
    wp.ldx = K; wp.rows_x = K; wp.ldy = M; wp.rows_y = M;
    return wp;
}

static int run_lin_backward(const LinProblem& P) {
    int rc = prepare_mlp_kernels();
    if (rc != ALST_OK) return rc;
    const LinLayout L = make_lin_layout(P.N, P.K, P.M, P.tile, true, P.flags);
    hipStream_t s = P.stream;
    const bool f32 = P.flags & ALST_FLAG_DW_FP32, accum = P.flags & ALST_FLAG_DW_ACCUMULATE;
    const bool in_out = f32 && !accum;
    float* acc = in_out ? reinterpret_cast<float*>(P.dW) : reinterpret_cast<float*>(P.ws + L.acc);
    const int K = (int)P.K, M = (int)P.M;
    uint16_t* wt = reinterpret_cast<uint16_t*>(P.ws + L.wt);
    if (L.weight_t) {
        ProfScope ps(PROF_MLP_OTHER, s);
        const Transposes ts = {{{P.W, M, K, K, wt, M, M}}};
        if (!launch_transposes(ts, s)) return ALST_ERR_HIP;
    }
    const int64_t chunk = lin_chunk_rows(P.N, P.M, P.K, L.weight_t);
    LinearParams lp = {};
    for (int64_t i0 = 0; i0 < P.N; i0 += chunk) {
        lp = lin_dx_extents(L, (int)std::min(chunk, P.N - i0), K, M);
        lp.X = P.dy + i0 * P.M; lp.Y = L.weight_t ? wt : P.W; lp.D = P.dx + i0 * P.K;
        if (i0 + chunk >= P.N) break;                                     // (the last one: with the first group)
        rc = launch_linear(lp, s);
        if (rc != ALST_OK) return rc;
    }
    const int64_t group = lin_group_rows(L);
    for (int64_t i0 = 0; i0 < P.N; i0 += group) {
        // dW[m][k] += sum over the group's rows of dy[t][m] x[t][k]: both operands are read
        // from the caller's arrays as they are
        const int64_t rows = std::min(group, P.N - i0);
        WgradParams wp = lin_wgrad_extents(rows, K, M);
        wp.X = P.x + i0 * P.K; wp.Y = P.dy + i0 * P.M;
        wp.out = {acc, P.dW, K, 1.f, i0 == 0, i0 + rows == P.N, f32, accum};
        rc = i0 == 0 ? launch_backward(lp, &wp, 1, s) : launch_wgrad(wp, s);
        if (rc != ALST_OK) return rc;
    }
    return ALST_OK;
}

}  // namespace alst

using namespace alst;

extern "C" {

size_t alst_tiled_mlp_workspace_bytes(int64_t N, int64_t H, int64_t I, int64_t tile, int backward,
                                      uint32_t flags) {
    if (N < 1 || H < 1 || I < 1 || tile < 1) return 0;
    if (N > (int64_t)1 << 30 || H > (int64_t)1 << 20 || I > (int64_t)1 << 20) return 0;
    return make_mlp_layout(N, H, I, tile, backward != 0, flags).total;
}

int alst_tiled_mlp_forward(const void* x, const void* Wg, const void* Wu, const void* Wd, int64_t N,
                           int64_t H, int64_t I, int64_t tile, void* y, void* workspace,
                           size_t workspace_bytes, uint32_t flags, void* stream) {
    MlpProblem P = {};
    P.x = (const uint16_t*)x; P.Wg = (const uint16_t*)Wg; P.Wu = (const uint16_t*)Wu;
    P.Wd = (const uint16_t*)Wd; P.y = (uint16_t*)y;
    P.N = N; P.H = H; P.I = I; P.tile = tile;
    P.ws = (unsigned char*)workspace; P.flags = flags; P.stream = (hipStream_t)stream;
    const int rc = validate_mlp(P, workspace_bytes, false);
    if (rc != ALST_OK) return rc;
    return run_mlp_forward(P);
}

int alst_tiled_mlp_backward(const void* x, const void* Wg, const void* Wu, const void* Wd,
                            const void* dy, int64_t N, int64_t H, int64_t I, int64_t tile, void* dx,
                            void* dWg, void* dWu, void* dWd, void* workspace, size_t workspace_bytes,
                            uint32_t flags, void* stream) {
    MlpProblem P = {};
    P.x = (const uint16_t*)x; P.Wg = (const uint16_t*)Wg; P.Wu = (const uint16_t*)Wu;
    P.Wd = (const uint16_t*)Wd; P.dy = (const uint16_t*)dy; P.dx = (uint16_t*)dx;
    P.dWg = dWg; P.dWu = dWu; P.dWd = dWd;
    P.N = N; P.H = H; P.I = I; P.tile = tile;
    P.ws = (unsigned char*)workspace; P.flags = flags; P.stream = (hipStream_t)stream;
    const int rc = validate_mlp(P, workspace_bytes, true);
    if (rc != ALST_OK) return rc;
    return run_mlp_backward(P);
}

size_t alst_tiled_linear_workspace_bytes(int64_t N, int64_t K, int64_t M, int64_t tile, int backward,
                                         uint32_t flags) {
    if (N < 1 || K < 1 || M < 1 || tile < 1) return 0;
    if (N > (int64_t)1 << 30 || K > (int64_t)1 << 20 || M > (int64_t)1 << 24) return 0;
    return make_lin_layout(N, K, M, tile, backward != 0, flags).total;
}

int alst_tiled_linear_forward(const void* x, const void* W, int64_t N, int64_t K, int64_t M,
                              int64_t tile, void* y, void* workspace, size_t workspace_bytes,
                              uint32_t flags, void* stream) {
    LinProblem P = {};
    P.x = (const uint16_t*)x; P.W = (const uint16_t*)W; P.y = (uint16_t*)y;
    P.N = N; P.K = K; P.M = M; P.tile = tile;
    P.ws = (unsigned char*)workspace; P.flags = flags; P.stream = (hipStream_t)stream;
    const int rc = validate_lin(P, workspace_bytes, false);
    if (rc != ALST_OK) return rc;
    return run_lin_forward(P);
}

int alst_tiled_linear_backward(const void* x, const void* W, const void* dy, int64_t N, int64_t K,
                               int64_t M, int64_t tile, void* dx, void* dW, void* workspace,
                               size_t workspace_bytes, uint32_t flags, void* stream) {
    LinProblem P = {};
    P.x = (const uint16_t*)x; P.W = (const uint16_t*)W; P.dy = (const uint16_t*)dy;
    P.dx = (uint16_t*)dx; P.dW = dW;
    P.N = N; P.K = K; P.M = M; P.tile = tile;
    P.ws = (unsigned char*)workspace; P.flags = flags; P.stream = (hipStream_t)stream;
    const int rc = validate_lin(P, workspace_bytes, true);
    if (rc != ALST_OK) return rc;
    return run_lin_backward(P);
}

int64_t alst_debug_chunk_rows(int op, int64_t N, int64_t K, int64_t M, int64_t tile) {
    if (op < 0 || op > 3 || N < 1 || K < 1 || M < 1 || tile < 1 || N > (int64_t)1 << 30 || K > (int64_t)1 << 20 ||
        M > (int64_t)1 << (op < 2 ? 20 : 24))
        return -ALST_ERR_SHAPE;
    if (op < 2) return make_mlp_layout(N, K, M, tile, op == 1, 0).chunk;
    if (op == 2) return lin_chunk_rows(N, K, M);
    return lin_chunk_rows(N, M, K, make_lin_layout(N, K, M, tile, true, 0).weight_t);
}

int alst_debug_layer(int op, int64_t N, int64_t K, int64_t M, int64_t tile, uint32_t flags, alst_debug_layer_info* info) {
    if (!info) return ALST_ERR_NULL;
    const int64_t chunk = alst_debug_chunk_rows(op, N, K, M, tile);
    if (chunk < 0) return (int)-chunk;
    if (K % 8 != 0 || M % 8 != 0) return ALST_ERR_ALIGN;
    if (flags & ~(ALST_FLAG_DW_FP32 | ALST_FLAG_DW_ACCUMULATE)) return ALST_ERR_UNSUPPORTED;
    *info = {};
    const int H = (int)K, I = (int)M;
    auto last_rows = [&](int64_t of) { return (int)(N - (N - 1) / of * of); };
    auto product = [&](const LinearParams& lp) {
        const BlockChoice c = choose_linear(&lp, 1);
        info->product_columns = c.columns;
        info->product_chained = c.chain;
    };
    auto gradients = [&](const LinearParams& lp, const WgradParams* ps, int n) {
        const int both = choose_together(lp, ps, n);
        product(lp);
        info->wgrad_columns = small_columns(ps, n);
        info->together = both != 0;
        if (both) info->product_columns = info->wgrad_columns = both;
    };
    if (op < 2) {
        const MlpLayout L = make_mlp_layout(N, K, M, tile, op == 1, flags);
        info->rows = last_rows(L.chunk);
        const BlockChoice g = choose_gated((int)info->rows, K, M);
        info->gated_columns = g.columns;
        info->gated_chained = g.chain;
        if (op == 0) {
            LinearParams lp = {};
            lp.rows_x = (int)info->rows; lp.K = I; lp.rows_y = H;
            product(lp);
        } else {
            info->transposed = L.weights_t;
            WgradParams wp[kMaxBatch];
            mlp_wgrad_extents(wp, last_rows(L.rows), H, I);
            gradients(mlp_dx_extents(L, (int)info->rows, H, I), wp, kMaxBatch);
        }
        return ALST_OK;
    }
    const LinLayout L = make_lin_layout(N, K, M, tile, op == 3, flags);
    if (op == 2) {
        info->rows = last_rows(chunk);
        LinearParams lp = {};
        lp.rows_x = (int)info->rows; lp.K = H; lp.rows_y = I;
        product(lp);
    } else {
        info->rows = last_rows(lin_chunk_rows(N, M, K, L.weight_t));
        info->transposed = L.weight_t;
        const WgradParams wp = lin_wgrad_extents(std::min(lin_group_rows(L), N), H, I);
        gradients(lin_dx_extents(L, (int)info->rows, H, I), &wp, 1);
    }
    return ALST_OK;
}

}  // extern "C"
