// Sequence-tiled LM-head projection + cross-entropy for gfx950: kernels and the C ABI (alst.h).
//
// Per shard of the sequence (paper, section "Sequence Tiling for Reducing Activation Memory
// Footprint": forward and backward of each logits shard are done together and the shard's
// intermediates are dropped before the next shard):
//
//   0. index / gather    rows whose label is ignored take no part in the loss or in either gradient:
//                        once per call the valid rows are numbered densely in sequence order, and
//                        the launches below work on CHUNKS of consecutive dense rows, gathered into
//                        a dense [rows, H] copy (behind the rows of the earlier chunks of their dW
//                        group).  A chunk is as many of the caller's tiles as the scratch holds
//                        anyway for the dW group (one tile under ALST_FLAG_TILE_SCRATCH).  The
//                        number M of dense rows lives on the device: the host walks the chunks of
//                        N rows and the kernels of a chunk beyond the dense rows leave at once, so
//                        nothing waits for the host.
//   1. logits_kernel     Z = H_c W^T in 256x256 blocks, fp32 accumulators.  The logits never
//                        leave the registers: the epilogue picks out the label logit, writes
//                        e = exp(z - ref_i) as bf16 to a [rows, V] scratch ("stash", also laid out
//                        per dW group) and reduces each row over the block's columns to
//                        a sum-of-e partial per 128-column group.  ref_i is ONE reference per
//                        row (0 to begin with), so a row's softmax is e / S_i with S_i = sum_v e:
//                        the scale is a per-row scalar that the consumers of the stash apply.
//   2. row_finish        partials -> S_i, lse_i = ref_i + log S_i, per-row loss; the label entry of
//                        the stash becomes e - S_i (so that e' / S_i = p - onehot), and the row's
//                        dense hidden row is scaled by 1 / S_i in place (the dW operand).  A row
//                        whose S_i left the safe range of the bf16 / fp32 exponents (logits
//                        beyond about +-40) is redone with ref_i = its exact maximum: a second,
//                        conditional launch of 1. and 2. whose workgroups leave at once when no
//                        row of the chunk asked for it.
//   3. dhidden_kernel    dH_i = (g/M) (1/S_i) e'_i W   (contraction over V), rows scattered back
//   4. dw_kernel         acc += (H_c / S)^T e'         once per group of rows (contraction over
//                        the group's dense rows, fp32)
//
// After the last chunk: loss = sum(per-row loss) / M in a fixed order.  The last group's dw_kernel writes
// dW = (g/M) acc.
// The contractions share the block GEMM of gemm_tile.h: logits and dHidden with both operands
// k-contiguous (dHidden against a copy of W transposed once per call), dW with both operands
// k-major (the group's dense hidden rows and dZ rows as they are).  No array of rows is
// transposed.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <math.h>
#include <algorithm>
#include <mutex>

#include "../../include/alst.h"
#include "../../include/alst_debug.h"
#include "gemm_tile.h"
#include "common.h"

namespace alst {

// ---------------------------------------------------------------------------------------------
// workspace
// ---------------------------------------------------------------------------------------------
struct Header {
    int status;            // alst_status set by kernels
    int pad0;
    long long n_valid;     // M
    float inv;             // g / M (0 when M == 0)
    float pad1;
    double loss_sum;
};

// What gather_rows_kernel leaves for the other kernels of a chunk.
struct ChunkInfo {
    int Tc;                // dense rows of the chunk (valid label)
    int Trc;               // Tc rounded up to the block height (256)
    int splits;            // dHidden: ranges the contraction over V is cut into for this chunk
    int ksteps;            //          k-steps of 64 per range (the last range may be shorter)
    int redo;              // set by row_finish: some row of the chunk needs the second logits pass
    int pad[3];
};

// dW is accumulated into the fp32 [V, H] sums once per GROUP of consecutive dense rows, as many as
// some number of tiles has (about kDwGroupRows): the hidden rows and dZ rows of the group's chunks are
// kept one behind the other and one dW GEMM contracts over all of them, so the read-modify-write of
// the 4*V*H-byte accumulator and the GEMM's epilogue are paid once per group instead of once per chunk.
constexpr int kDwGroupRows = 16384;
constexpr int kDwGroupMax = 8;
// ALST_FLAG_TILE_SCRATCH (and the forward-only layout, which keeps no dZ at all): groups of one tile.
static inline int dw_group_size(int64_t Tp, uint32_t flags) {
    if (flags & (ALST_FLAG_TILE_SCRATCH | ALST_FLAG_FORWARD_ONLY)) return 1;
    int64_t g = kDwGroupRows / Tp;
    return (int)(g < 1 ? 1 : (g > kDwGroupMax ? kDwGroupMax : g));
}
constexpr uint32_t kKnownFlags = ALST_FLAG_DW_FP32 | ALST_FLAG_DW_ACCUMULATE | ALST_FLAG_REDUCE_SUM |
                                 ALST_FLAG_TILE_SCRATCH | ALST_FLAG_FORWARD_ONLY;

constexpr int kScanThreads = 1024;   // rows per block of the compaction kernels
// gather_rows_kernel: rows of the sequence a workgroup looks for ignored tokens at a time, workgroups that do so
constexpr int kZeroRows = 16, kZeroBlocksMax = 32768;

struct Layout {
    int64_t Tp, Vp, ng;    // padded tile rows, padded vocabulary, 128-column groups
    int64_t Hk;            // row pitch of the dense hidden copy: H rounded up to whole k-steps
    int g;                 // the caller's tiles per dW group
    int64_t Kg;            // dense rows the group's buffers hold: g * Tp
    int64_t Rc;            // most dense rows per chunk of launches, a multiple of 256
    int64_t step;          // dense rows of a chunk behind which more than Rc follow
    int dh_PR, dh_PC;      // dHidden: patch shape of the block -> tile mapping
    size_t part_bytes;     //          room for fp32 partial products at `part`
    size_t header, cinfo, loss_rows, lse, idx, block_cnt, block_ofs, zlabel, yc, ref, frow, rowstate,
        rmax, ps, part, hc, stash, wt, acc, total;
};

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// dHidden has (rows / 256) * (H / 256) output blocks for a chunk of `rows` dense rows (a multiple
// of 256).  Picks the number of ranges (1..8) the contraction over V is cut into: the one with the
// least estimated time, in units of a k-step of one block (1.5 us on gfx950): rounds of the 256
// compute units (a last one in halves: 5/8) times (k-steps per range + about 4 for the block's start
// and epilogue) and, if cut, the partial products' way through memory (256 KB per block and range
// written and read back at about 5 TB/s: 0.07 units) and the launch that adds them.  A range keeps
// at least 8 k-steps.
// The chunk's row count is known on the device only, so gather_rows_kernel makes the choice; the
// host evaluates the same function for every row count that can be cut (dhidden_most_blocks).
constexpr int kComputeUnits = 256;
// (from 16 rounds of workgroups on the chip is filled to 16/17 or better as it is)
constexpr int64_t kCutBlocks = 16 * kComputeUnits;
// part_rows_cap: the ranges' fp32 partial products (splits * rows rows) must fit that many rows.
__host__ __device__ inline void dhidden_splits(int64_t rows, int64_t H, int64_t V, int64_t part_rows_cap,
                                               int& splits, int& ksteps) {
    const int64_t blocks = (rows / kBlockR) * ((H + kBlockC - 1) / kBlockC);
    const int KT = (int)((V + kBlockK - 1) / kBlockK);
    splits = 1;
    int64_t best = INT64_MAX;
    const int sp_max = blocks >= kCutBlocks ? 1 : 8;
    for (int sp = 1; sp <= sp_max; ++sp) {
        const int per = (KT + sp - 1) / sp;
        if (sp > 1 && (per < 8 || (int64_t)(sp - 1) * per >= KT || sp * rows > part_rows_cap)) break;
        const int64_t cost = rounds16(blocks * sp) * (per + 4) + (sp > 1 ? 48 + blocks * sp * 9 / 8 : 0);
        if (cost < best) { best = cost; splits = sp; }
    }
    ksteps = (KT + splits - 1) / splits;
}

// The most blocks (over all ranges) that dHidden of a chunk of up to `rows` dense rows (a multiple of
// 256) needs, and whether some number of rows has its contraction cut: what gather_rows_kernel may
// choose on the device, for every number of dense rows.  Only below 16 rounds of blocks is a contraction
// cut; from there on the blocks grow with the rows, so of those numbers the largest stands for all.
static int64_t dhidden_most_blocks(int64_t rows, int64_t H, int64_t V, int64_t part_rows, bool& cut) {
    const int64_t tiles_c = (H + kBlockC - 1) / kBlockC, rb_max = rows / kBlockR;
    int64_t most = rb_max * tiles_c;
    cut = false;
    for (int64_t rb = 1; rb <= rb_max && rb * tiles_c < kCutBlocks; ++rb) {
        int sp, ks;
        dhidden_splits(rb * kBlockR, H, V, part_rows, sp, ks);
        if (rb * tiles_c * sp > most) most = rb * tiles_c * sp;
        cut = cut || sp > 1;
    }
    return most;
}

// Ranges of V whose partial products of a full tile the workspace has room for.  The workspace's size is
// part of the interface, so this is not the choice of dhidden_splits: the number (1..8) that fills the
// compute units most evenly (ties: fewest), each range keeping at least 64 k-steps.
static int64_t workspace_ranges(int64_t rows, int64_t H, int64_t V) {
    const int64_t blocks = (rows / kBlockR) * ((H + kBlockC - 1) / kBlockC);
    const int64_t KT = (V + kBlockK - 1) / kBlockK;
    int64_t ranges = 1, best = 0, best_slots = 1;          // share of busy compute units: best / best_slots
    const int sp_max = blocks >= kCutBlocks ? 1 : 8;
    for (int sp = 1; sp <= sp_max; ++sp) {
        const int64_t per = (KT + sp - 1) / sp;
        if (sp > 1 && (per < 64 || (sp - 1) * per >= KT)) break;
        const int64_t slots = (blocks * sp + kComputeUnits - 1) / kComputeUnits * kComputeUnits;
        if (blocks * sp * best_slots > best * slots) { best = blocks * sp; best_slots = slots; ranges = sp; }
    }
    return ranges;
}

// From about here on (k-steps: 1536) calls gain by chunks of one round of dHidden: at 128256 words and more up to
// 1.7 % for H = 2048 to 8192 and none loses (131072 x 4096 276.0 -> 274.8 ms, 32768 x 5120 x 152064 82.0 -> 80.8,
// 32768 x 8192 x 128256 150.9 -> 148.4), at 65536 words between level and 1.6 % slower (H = 1024 to 7168).
constexpr int64_t kLongVocabulary = 98304;

static Layout make_layout(int64_t N, int64_t H, int64_t V, int64_t tile, uint32_t flags) {
    Layout L;
    const int64_t T = tile < N ? tile : N;
    L.Tp = (T + 255) / 256 * 256;
    L.Vp = (V + 255) / 256 * 256;
    L.ng = L.Vp / 128;
    L.Hk = (H + kBlockK - 1) / kBlockK * kBlockK;
    L.g = dw_group_size(L.Tp, flags);
    L.Kg = (int64_t)L.g * L.Tp;
    const bool fwd_only = flags & ALST_FLAG_FORWARD_ONLY;     // no dZ rows, partial products, dW sums
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, 256); return at; };
    L.header = take(sizeof(Header));
    L.cinfo = take(sizeof(ChunkInfo));
    // the O(N) part: 12 bytes per row + 12 bytes per kScanThreads rows
    const size_t nblocks = ((size_t)N + kScanThreads - 1) / kScanThreads;
    L.loss_rows = take((size_t)N * 4);
    L.lse = take((size_t)N * 4);
    L.idx = take((size_t)N * 4);
    L.block_cnt = take(nblocks * 4);
    L.block_ofs = take(nblocks * 8);
    // Per-row arrays, softmax partials and partial dHidden products of one chunk.  The region is
    // sized for one tile (20 bytes per row, 8 per row and 128-column group, the partial products a
    // full tile needs); a chunk then takes as many rows of the dW group as fit it (and a grid) with 24 bytes
    // per row and 4 per row and group (the partial products of dHidden reuse the softmax partials'
    // place, which row_finish has consumed by then).
    const size_t region = (size_t)L.Tp * (20 + 8 * (size_t)L.ng) +
                          (fwd_only ? 0 : (size_t)workspace_ranges(L.Tp, H, V) * L.Tp * H * 4);
    const size_t at = take(region);
    const int64_t fit = (int64_t)(region / (24 + 4 * (size_t)L.ng)) / kBlockR * kBlockR;
    const int64_t rows = (N + kBlockR - 1) / kBlockR * kBlockR, Kn = L.Kg < rows ? L.Kg : rows;
    // (a launch has a workgroup of 256 per row and those of the zeroing, or per output block of the chunk)
    const int64_t cols = std::max((L.Vp + kBlockC - 1) / kBlockC, (H + kBlockC - 1) / kBlockC);
    const int64_t grid = std::min(kGridBlocks - kZeroBlocksMax, kGridBlocks / cols * kBlockR) / kBlockR * kBlockR;
    const int64_t most = std::min(fit, grid), parts = (Kn + most - 1) / most;
    L.Rc = ((Kn + parts - 1) / parts + kBlockR - 1) / kBlockR * kBlockR;     // <= most, a multiple of 256
    // A long vocabulary makes dHidden's blocks long, and over several rounds of them in one launch the
    // workgroups of an XCD no longer walk k together: chunks of about one round then, and not less than
    // 4096 rows (a last one up to a quarter longer: each chunk reads W again).
    L.step = L.Rc;
    const int64_t round_rows = std::max<int64_t>(4096, kRound * (int64_t)kBlockR * kBlockC / H / 4096 * 4096);
    if (!fwd_only && V >= kLongVocabulary && L.Rc > round_rows + round_rows / 4) {
        L.step = round_rows;
        L.Rc = round_rows + round_rows / 4;
    }
    L.zlabel = at;
    L.yc = L.zlabel + (size_t)L.Rc * 4;
    L.ref = L.yc + (size_t)L.Rc * 4;
    L.frow = L.ref + (size_t)L.Rc * 4;
    L.rowstate = L.frow + (size_t)L.Rc * 4;
    L.rmax = L.rowstate + (size_t)L.Rc * 4;
    L.ps = L.part = L.rmax + (size_t)L.Rc * 4;
    // hc and stash hold the dense rows of the whole group: they are the two operands of the
    // group's dW product as they are (k = dense row, the slow index)
    L.hc = take((size_t)L.Kg * L.Hk * 2);
    L.stash = take(fwd_only ? 0 : (size_t)L.Kg * L.Vp * 2);
    // W transposed, [H, Vp], zeros from V to whole k-steps: the second operand of dH = dZ W, k-contiguous
    L.wt = take(fwd_only ? 0 : (size_t)H * L.Vp * 2);
    {
        const PatchGrid pg = choose_patches((int)(L.step / kBlockR), (int)((H + kBlockC - 1) / kBlockC));
        L.dh_PR = pg.PR; L.dh_PC = pg.PC;
        L.part_bytes = at + region - L.part;
    }
    const bool acc_in_dw = (flags & ALST_FLAG_DW_FP32) && !(flags & ALST_FLAG_DW_ACCUMULATE);
    L.acc = take(acc_in_dw || fwd_only ? 0 : (size_t)V * H * 4);
    L.total = o;
    return L;
}

// ---------------------------------------------------------------------------------------------
// small kernels
// ---------------------------------------------------------------------------------------------
__global__ void init_header_kernel(Header* h) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        h->status = 0;
        h->n_valid = 0;
        h->inv = 0.f;
        h->loss_sum = 0.0;
    }
}

__device__ __forceinline__ bool label_valid(int y, int ignore_index, int V) {
    return y != ignore_index && y >= 0 && y < V;
}

// Row compaction of the whole sequence: idx[j] = row of the j-th token with a valid label, in
// sequence order.  Three small kernels over blocks of kScanThreads rows:
//   block_count_kernel   valid rows per block
//   block_offsets_kernel exclusive scan of the block counts (one workgroup), M = their sum
//   scatter_index_kernel rank inside the block + block offset -> idx; rows that take no part get
//                        loss term 0 and lse 0 (forward).
// and, for up to kIndexRows rows, one kernel of one workgroup in place of the four launches (a
// launch costs about 5 us; at 32768 rows the one workgroup takes 8 us).
__device__ __forceinline__ int block_rank(bool valid, int* wave_total, int& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long mask = __ballot(valid);
    const int below = __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0));
    if (lane == 0) wave_total[wave] = __popcll(mask);
    __syncthreads();
    int before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kScanThreads / 64; ++w) {
        const int c = wave_total[w];
        if (w < wave) before += c;
        total += c;
    }
    __syncthreads();
    return before + below;
}

__global__ __launch_bounds__(kScanThreads) void block_count_kernel(
    const int32_t* __restrict__ labels, int64_t N, int ignore_index, int V,
    int32_t* __restrict__ block_cnt, Header* h) {
    __shared__ int wave_total[kScanThreads / 64];
    const int64_t i = (int64_t)blockIdx.x * kScanThreads + threadIdx.x;
    const int y = i < N ? labels[i] : ignore_index;
    const bool valid = i < N && label_valid(y, ignore_index, V);
    if (i < N && y != ignore_index && !valid) atomicMax(&h->status, (int)ALST_ERR_LABEL_RANGE);
    int total;
    (void)block_rank(valid, wave_total, total);
    if (threadIdx.x == 0) block_cnt[blockIdx.x] = total;
}

// One workgroup: block_ofs[b] = sum of block_cnt[0 .. b), M and g/M into the header.
__global__ __launch_bounds__(kScanThreads) void block_offsets_kernel(
    const int32_t* __restrict__ block_cnt, int64_t nblocks, int64_t* __restrict__ block_ofs,
    Header* h, float grad_loss, int sum_mode, int64_t* __restrict__ n_valid_out) {
    __shared__ long long part[kScanThreads];
    const int tid = threadIdx.x;
    // thread t owns the contiguous chunk [t * per, (t + 1) * per)
    const int64_t per = (nblocks + kScanThreads - 1) / kScanThreads;
    const int64_t lo = tid * per, hi = lo + per < nblocks ? lo + per : nblocks;
    long long sum = 0;
    for (int64_t b = lo; b < hi; ++b) sum += block_cnt[b];
    part[tid] = sum;
    __syncthreads();
    if (tid == 0) {
        long long run = 0;
        for (int t = 0; t < kScanThreads; ++t) {
            const long long c = part[t];
            part[t] = run;
            run += c;
        }
        h->n_valid = run;
        // gradient scale: g / M for the mean, g for the sum of the token losses
        h->inv = run > 0 ? (sum_mode ? grad_loss : grad_loss / (float)run) : 0.f;
        if (n_valid_out) *n_valid_out = run;
    }
    __syncthreads();
    long long run = part[tid];
    for (int64_t b = lo; b < hi; ++b) {
        block_ofs[b] = run;
        run += block_cnt[b];
    }
}

__global__ __launch_bounds__(kScanThreads) void scatter_index_kernel(
    const int32_t* __restrict__ labels, int64_t N, int ignore_index, int V,
    const int64_t* __restrict__ block_ofs, int32_t* __restrict__ idx, float* __restrict__ lse,
    float* __restrict__ loss_rows) {
    __shared__ int wave_total[kScanThreads / 64];
    const int64_t i = (int64_t)blockIdx.x * kScanThreads + threadIdx.x;
    const int y = i < N ? labels[i] : ignore_index;
    const bool valid = i < N && label_valid(y, ignore_index, V);
    int total;
    const int rank = block_rank(valid, wave_total, total);
    if (valid) idx[block_ofs[blockIdx.x] + rank] = (int32_t)i;
    else if (i < N) {
        if (lse) lse[i] = 0.f;
        if (loss_rows) loss_rows[i] = 0.f;
    }
}

// The whole compaction in one workgroup: wavefront w owns the consecutive rows [w span, (w + 1) span),
// counts them, and after one scan over the wavefronts numbers them.
constexpr int64_t kIndexRows = 32768;
__global__ __launch_bounds__(kScanThreads) void index_rows_kernel(
    const int32_t* __restrict__ labels, int N, int ignore_index, int V, float grad_loss, int sum_mode,
    int32_t* __restrict__ idx, float* __restrict__ lse, float* __restrict__ loss_rows, Header* h,
    int64_t* __restrict__ n_valid_out) {
    constexpr int kWaves = kScanThreads / 64;
    __shared__ int wave_total[kWaves], wave_bad[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int span = (N + kScanThreads - 1) / kScanThreads * 64, lo = wave * span;
    int count = 0, bad = 0;
    // eight loads in flight; act(row, label) for the wavefront's rows in order, 64 at a time
    auto for_rows = [&](auto act) {
        for (int o = 0; o < span; o += 512) {
            int y[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int i = lo + o + j * 64 + lane;
                y[j] = o + j * 64 < span && i < N ? labels[i] : ignore_index;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) act(lo + o + j * 64 + lane, y[j], o + j * 64 < span);
        }
    };
    for_rows([&](int, int y, bool) {
        const bool valid = label_valid(y, ignore_index, V);
        count += __popcll(__ballot(valid));
        bad |= (y != ignore_index && !valid) ? 1 : 0;
    });
    bad = __ballot(bad != 0) != 0ull ? 1 : 0;
    if (lane == 0) {
        wave_total[wave] = count;
        wave_bad[wave] = bad;
    }
    __syncthreads();
    int before = 0, total = 0;
    bad = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const int c = wave_total[w];
        if (w < wave) before += c;
        total += c;
        bad |= wave_bad[w];
    }
    if (threadIdx.x == 0) {
        h->status = bad ? (int)ALST_ERR_LABEL_RANGE : 0;
        h->n_valid = total;
        h->inv = total > 0 ? (sum_mode ? grad_loss : grad_loss / (float)total) : 0.f;
        h->loss_sum = 0.0;
        if (n_valid_out) *n_valid_out = total;
    }
    for_rows([&](int i, int y, bool mine) {
        const bool valid = label_valid(y, ignore_index, V);
        const unsigned long long mask = __ballot(valid);
        if (valid)
            idx[before + __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0))] = i;
        else if (mine && i < N) {
            if (lse) lse[i] = 0.f;
            if (loss_rows) loss_rows[i] = 0.f;
        }
        before += __popcll(mask);
    });
}

// A row's maximum travels as an integer of the same order (atomicMax).
__device__ __forceinline__ int ordered_int(float v) {
    const int b = __builtin_bit_cast(int, v);
    return b >= 0 ? b : b ^ 0x7fffffff;
}
__device__ __forceinline__ float from_ordered_int(int k) {
    return __builtin_bit_cast(float, k >= 0 ? k : k ^ 0x7fffffff);
}

// Workgroup b < Rc: dense row b of the chunk that starts at dense row `first`.  Copies the hidden
// row of its token into the dense matrix Hc (the chunk's rows; row pitch Hk = H rounded up to whole
// k-steps, zeros behind the H elements) and its label into yc; rows Tc <= b < Trc are zero padding.  Also sets the row's softmax reference for the first logits
// pass (0; backward from a saved lse: that lse, so that e is the probability itself) and marks the
// row as taking part in that pass.  Workgroup 0 leaves the chunk's counts and its dHidden ranges.
// Workgroups from Rc on (first chunk, if a gradient is wanted) take kZeroRows rows of the sequence at a
// time; the dHidden rows of ignored tokens become zeros.  The workgroups behind those transpose W (first chunk, if
// a gradient is wanted: a launch of its own took 3 us more of the smallest calls).
// INDEX (N <= kGatherIndexRows, one chunk): there was no launch that numbers the rows; every workgroup counts the valid labels
// itself, and workgroup 0 leaves the header.  A launch less, for four labels a thread counts in every workgroup; us of a call
// with the launch / without: N = 300 (H = 256, V = 4096) 38.6 / 36.1, 512 40.7 / 38.2, 1024 51.6 / 49.3; with 8 and 16 labels a thread 1500 65.5 /
// 65.4, 2048 69.4 / 72.7, 3000 80.4 / 92.2.
constexpr int kGatherIndexRows = 1024;
struct GatherParams {
    const uint16_t* hidden;      // [N, H]
    const int32_t* labels;       // [N]
    const int32_t* idx;          // [N]        dense row -> row of the sequence
    const float* lse_in;         // [N]        backward from a saved lse, or null
    const Header* hdr;
    ChunkInfo* info;
    uint16_t* Hc;                // [Rc, Hk]   the chunk's rows of the dense matrix
    int32_t* yc;                 // [Rc]
    float* ref;
    int32_t *rowstate, *rmax;
    uint16_t* dHidden;           // [N, H]
    int64_t N, first;
    int64_t Rc;                  // the chunk's rows, rounded up to the block height
    int64_t H, V, dh_part_rows;
    int64_t zero_blocks;
    int Hk, ignore_index;
    // INDEX: what index_rows_kernel writes
    Header* hdr_out;
    int32_t* idx_out;
    float *lse, *loss_rows;      // may be null
    int64_t* n_valid_out;
    float grad_loss;
    int sum_mode;
};
template <bool INDEX>
__global__ __launch_bounds__(256) void gather_rows_kernel(const GatherParams p, const Transpose t) {
    const int64_t b = blockIdx.x;
    if (b >= p.Rc + p.zero_blocks) {
        transpose_piece(t, b - p.Rc - p.zero_blocks);
        return;
    }
    const u32x4_t zero4 = {0u, 0u, 0u, 0u};
    const int src_chunks = (int)(p.H / 8);
    if (b >= p.Rc) {
        const int lane = threadIdx.x & 63;
        for (int64_t row0 = (b - p.Rc) * kZeroRows; row0 < p.N; row0 += p.zero_blocks * kZeroRows) {
            const int64_t i = row0 + lane;
            const bool ignored = lane < kZeroRows && i < p.N && !label_valid(p.labels[i], p.ignore_index, (int)p.V);
            for (unsigned long long mask = __ballot(ignored); mask; mask &= mask - 1) {
                u32x4_t* dst = reinterpret_cast<u32x4_t*>(p.dHidden + (row0 + (__ffsll(mask) - 1)) * p.H);
                for (int c = threadIdx.x; c < src_chunks; c += 256) dst[c] = zero4;
            }
        }
        return;
    }
    long long n_valid = 0;
    int my_row = 0;                // INDEX: the token of dense row b
    if constexpr (INDEX) {
        constexpr int kPer = kGatherIndexRows / 256;
        __shared__ int count[kPer][4];
        __shared__ int row_of_b;
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        unsigned long long mask[kPer];
        bool bad = false;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int i = j * 256 + threadIdx.x;
            const int y = i < p.N ? p.labels[i] : p.ignore_index;
            const bool valid = i < p.N && label_valid(y, p.ignore_index, (int)p.V);
            bad |= y != p.ignore_index && !valid;
            mask[j] = __ballot(valid);
            if (lane == 0) count[j][wave] = __popcll(mask[j]);
        }
        const int any_bad = __syncthreads_or(bad);
        int total = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                if (w == wave) {
                    const int rank = total + __builtin_amdgcn_mbcnt_hi((unsigned)(mask[j] >> 32),
                                                                       __builtin_amdgcn_mbcnt_lo((unsigned)mask[j], 0));
                    if ((mask[j] >> lane & 1) && rank == b) row_of_b = j * 256 + threadIdx.x;
                }
                total += count[j][w];
            }
        n_valid = total;
        if (b == 0) {
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                const int i = j * 256 + threadIdx.x;
                if (i < p.N && !(mask[j] >> lane & 1)) {
                    if (p.lse) p.lse[i] = 0.f;
                    if (p.loss_rows) p.loss_rows[i] = 0.f;
                }
            }
            if (threadIdx.x == 0) {
                p.hdr_out->status = any_bad ? (int)ALST_ERR_LABEL_RANGE : 0;
                p.hdr_out->n_valid = total;
                p.hdr_out->inv = total > 0 ? (p.sum_mode ? p.grad_loss : p.grad_loss / (float)total) : 0.f;
                p.hdr_out->loss_sum = 0.0;
                if (p.n_valid_out) *p.n_valid_out = total;
            }
        }
        __syncthreads();
        if (b < total) {
            my_row = row_of_b;
            if (threadIdx.x == 0) p.idx_out[b] = my_row;
        }
    } else {
        n_valid = p.hdr->n_valid;
    }
    const long long left = n_valid - p.first;
    const int Tc = (int)(left < 0 ? 0 : (left > p.Rc ? p.Rc : left));
    const int Trc = (Tc + kBlockR - 1) / kBlockR * kBlockR;
    if (b == 0 && threadIdx.x == 0) {
        p.info->Tc = Tc;
        p.info->Trc = Trc;
        p.info->redo = 0;
        // dHidden of this chunk: the ranges of V that suit its Trc rows.  The host has looked at every
        // Trc there can be (dhidden_most_blocks): the launch holds the blocks, and the partial products
        // are added up.
        int sp = 1, ks = 0;
        dhidden_splits(Trc, p.H, p.V, p.dh_part_rows, sp, ks);
        p.info->splits = sp;
        p.info->ksteps = ks;
    }
    if (b >= Trc) return;
    const int chunks = p.Hk / 8;
    u32x4_t* dst = reinterpret_cast<u32x4_t*>(p.Hc + b * p.Hk);
    int y = -1;
    float ref = 0.f;
    if (b < Tc) {
        const int64_t row = INDEX ? my_row : p.idx[p.first + b];
        const u32x4_t* src = reinterpret_cast<const u32x4_t*>(p.hidden + row * p.H);
        for (int c = threadIdx.x; c < chunks; c += 256) dst[c] = c < src_chunks ? src[c] : zero4;
        if (threadIdx.x == 0) {
            y = p.labels[row];
            if (p.lse_in) ref = p.lse_in[row];
        }
    } else {
        for (int c = threadIdx.x; c < chunks; c += 256) dst[c] = zero4;
    }
    if (threadIdx.x == 0) {
        p.yc[b] = y;
        p.ref[b] = ref;
        p.rowstate[b] = 1;
        p.rmax[b] = ordered_int(-INFINITY);
    }
}

enum { MODE_FWD = 0, MODE_FUSED = 1, MODE_BWD = 2 };

// A row's e = exp(z - ref) live in bf16 (the stash) and in fp32 sums; both have 8 exponent bits.
// With S = sum_v e inside [kSumLo, kSumHi] no e of weight overflows, the ones that underflow are
// below 2^-66 of the row's mass, and the fp32 products S * |w| of the dHidden contraction stay far
// from overflow.  A row outside is redone with ref = its exact maximum (then 1 <= S <= V).
constexpr float kSumLo = 8.673617379884035e-19f;      // 2^-60
constexpr float kSumHi = 1.2676506002282294e30f;      // 2^100
constexpr float kGroupHi = 1.1805916207174113e21f;    // 2^70
constexpr float kLog2e = 1.4426950408889634f;

struct RowFinishParams {
    const float* ps;         // [ng, Rc]  per 128-column group: sum of e
    const float* zlabel;     // [Rc]      label logit of each dense row
    const int32_t* yc;       // [Rc]      label of each dense row
    const int32_t* idx;      // [Rc]      dense row -> row of the sequence
    const int32_t* rmax;     // [Rc]      maximum of a row whose sum left the safe range (ordered_int)
    ChunkInfo* info;
    float* ref;              // [Rc]      the row's reference; rewritten for a row that is redone
    float* frow;             // [Rc]      1 / S of a finished row (MODE_FUSED), 1 (MODE_BWD)
    int32_t* rowstate;       // [Rc]      1: the row takes part in the next logits pass, 0: finished
    float* lse_t;            // [N]       by row of the sequence
    float* loss_rows_t;      // [N]
    uint16_t* hc;            // [Rc, Hk]  the chunk's dense hidden rows (scaled in place, MODE_FUSED)
    uint16_t* stash;         // [Rc, Vp]
    int64_t Rc;
    int ng, H, Hk, Vp;
};

// Per dense row of the chunk, after a logits pass: S = sum of the per-group sums of e (fixed order,
// so a row's lse depends on nothing but its own partials), lse = ref + log S, the row's loss term
// (both written to the row's original position) and, when gradients follow,
//   * the stash entry of the label becomes e_label - S (MODE_FUSED) or p_label - 1 (MODE_BWD),
//     formed in fp32 from the label logit, so that (stash * f)[v] = p[v] - [v = label] with the
//     relative precision of bf16 in every entry;
//   * frow = f = 1 / S (adjusted by the rounding of the label entry, see below), which dHidden
//     applies to its output rows;
//   * the row's dense hidden row is multiplied by f in place: it is the other operand of the
//     dW product, whose contraction index is the row.
// First pass (REDO = false): a row whose S is outside [kSumLo, kSumHi] is not finished; its
// reference becomes its exact maximum, it stays marked, and the chunk is flagged for the second
// pass.  Second pass (REDO = true): leaves at once unless flagged; finishes the marked rows.
// MODE_BWD has no sums to combine (e is the probability itself): label entries only.
// Block = 16 rows x 64 lanes: thread (x, y) owns groups y, y + 64, ... of row x; the 64 lanes of a
// row are combined through LDS in a fixed order.
constexpr int kCombineRows = 16, kCombineLanes = 64;
template <int MODE, bool REDO>
__global__ __launch_bounds__(kCombineRows * kCombineLanes) void row_finish_kernel(const RowFinishParams p) {
    __shared__ float red[kCombineLanes][kCombineRows];
    const int x = threadIdx.x, y = threadIdx.y;
    if ((int)blockIdx.x * kCombineRows >= p.info->Trc) return;
    if (REDO && !p.info->redo) return;
    const int i = blockIdx.x * kCombineRows + x;          // dense row; Trc is a multiple of 256
    const bool inrow = i < p.info->Tc;                    // every dense row below Tc is valid
    const bool marked = p.rowstate[i] != 0;
    __syncthreads();                                      // every thread of a row has read its mark
    const int64_t Rc = p.Rc;
    const int ng = p.ng;
    float S = 1.f;
    if (MODE != MODE_BWD) {
        float sum = 0.f;
        for (int g = y; g < ng; g += kCombineLanes) sum += p.ps[g * Rc + i];
        red[y][x] = sum;
        __syncthreads();
        S = red[0][x];
#pragma unroll
        for (int l = 1; l < kCombineLanes; ++l) S += red[l][x];
    }
    // (rowstate, ref and frow of row i are written by the row's thread y == 0 only, and read above
    // or below by the same thread or before the barriers)
    if (!inrow) {                                         // padding rows: nothing to finish
        if (y == 0 && !REDO) { p.rowstate[i] = 0; p.frow[i] = 0.f; }
        return;
    }
    if (!marked) return;
    const bool ok = MODE == MODE_BWD || REDO || (S >= kSumLo && S <= kSumHi);
    if (!ok) {
        if (y == 0) {
            const float M = from_ordered_int(p.rmax[i]);
            p.ref[i] = (M == -INFINITY || M != M) ? 0.f : M;
            atomicOr(&p.info->redo, 1);
        }
        return;
    }
    const float ref = p.ref[i], zl = p.zlabel[i];
    // the label's e, as the logits pass formed it before rounding it to bf16, minus S (MODE_BWD:
    // p - 1, S = 1), rounded to bf16 for the stash
    const float el = __builtin_amdgcn_exp2f(fmaf(zl, kLog2e, -(ref * kLog2e)));
    const __bf16 d = (__bf16)(el - S);
    // The row's scale is chosen so that the ROUNDED label entry times the scale is p - 1 to fp32
    // precision (the label entries carry the largest gradients); every other entry of the row then
    // sees the scale off by the label entry's rounding, within the 2^-9 its own rounding has.
    float f = 1.f / S;
    if (MODE != MODE_FWD && (float)d != 0.f) f = ((el - S) / (float)d) / S;     // (d * S may overflow)
    if (y == 0) {
        if (MODE != MODE_BWD) {
            const int orig = p.idx[i];
            const float lse = ref + __logf(S);
            p.lse_t[orig] = lse;
            p.loss_rows_t[orig] = lse - zl;
        }
        if (MODE != MODE_FWD) {
            p.stash[(int64_t)i * p.Vp + p.yc[i]] = __builtin_bit_cast(uint16_t, d);
            p.frow[i] = f;
        }
        p.rowstate[i] = 0;
    }
    if (MODE == MODE_FUSED) {
        uint16_t* row = p.hc + (int64_t)i * p.Hk;
        for (int c = y; c < p.H / 8; c += kCombineLanes) {
            bf16x8_t v = *reinterpret_cast<const bf16x8_t*>(row + c * 8);
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = (__bf16)((float)v[q] * f);
            *reinterpret_cast<bf16x8_t*>(row + c * 8) = v;
        }
    }
}

// loss = (sum of the per-row terms in a fixed order) / M, or the sum itself.  One workgroup of THREADS; the order is
// the same for every number of threads: kLossSums sums of every kLossSums-th term, added up pairwise.  Which launch makes the loss
// depends on the tile and the entry point, the bits of the loss do not.
struct LossParams {
    const float* loss_rows;
    int64_t N;
    Header* h;
    int sum_mode;
    float* loss_out;
};
constexpr int kLossSums = 1024;
template <int THREADS>
__device__ __forceinline__ void loss_reduce(const LossParams& p) {
    constexpr int kPer = kLossSums / THREADS;
    __shared__ double part[kLossSums];
    double s[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) s[q] = 0.0;
    const float* at = p.loss_rows + threadIdx.x;
    const int64_t whole = p.N / kLossSums;
    const int rest = (int)(p.N % kLossSums);
#pragma unroll 8
    for (int64_t k = 0; k < whole; ++k, at += kLossSums)
#pragma unroll
        for (int q = 0; q < kPer; ++q) s[q] += (double)at[q * THREADS];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        if ((int)threadIdx.x + q * THREADS < rest) s[q] += (double)at[q * THREADS];
        part[threadIdx.x + q * THREADS] = s[q];
    }
    __syncthreads();
    for (int w = kLossSums / 2; w > 0; w >>= 1) {
        for (int t = threadIdx.x; t < w; t += THREADS) part[t] += part[t + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const long long M = p.h->n_valid;
        const double L = M > 0 ? (p.sum_mode ? part[0] : part[0] / (double)M) : 0.0;
        p.h->loss_sum = part[0];
        *p.loss_out = (float)L;
        if (!isfinite(L)) atomicMax(&p.h->status, (int)ALST_ERR_NONFINITE);
    }
}
__global__ __launch_bounds__(1024) void loss_reduce_kernel(const LossParams p) { loss_reduce<1024>(p); }

__global__ void copy_f32_kernel(const float* __restrict__ in, float* __restrict__ out, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = in[i];
}

__global__ void shift_labels_kernel(const int32_t* __restrict__ labels, int32_t* __restrict__ out,
                                    int64_t N, int ignore_index) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = i + 1 < N ? labels[i + 1] : ignore_index;
}

// ---------------------------------------------------------------------------------------------
// the three block GEMMs
// ---------------------------------------------------------------------------------------------
struct LogitsParams {
     const uint16_t* hidden_t;   // [Rc, Hk]     the chunk's dense (valid) rows, zero padded to Trc
    const uint16_t* W;          // [V, H]
    const int32_t* labels_t;    // [Rc]         labels of the dense rows
    const ChunkInfo* info;
    const float* ref;           // [Rc]         reference of each dense row: e = exp(z - ref)
    const int32_t* rowstate;    // [Rc]         second pass: rows that are redone (others keep their results)
    int32_t* rmax;              // [Rc]         maximum of rows whose sums leave the safe range (ordered_int)
    float* ps;                  // [ng, Rc]     MODE_FWD / MODE_FUSED
    float* zlabel;              // [Rc]
    uint16_t* stash;            // [Rc, Vp]     MODE_FUSED / MODE_BWD
    int64_t Rc;                 // row stride of ps
    int H, Hk, V, Vp;
    int PR, PC;                 // patch shape of the block -> tile mapping
};

// r = token row of the chunk (MFMA lane dimension), c = vocabulary id (register dimension).
// REDO: the second pass over a chunk, for the rows whose first-pass sums left the safe range; its
// workgroups leave at once unless row_finish flagged the chunk, and rows that are not marked keep
// what the first pass wrote.
// tw: the wavefront's LDS turn-around area, kTile rows.
template <class Core, int MODE, bool REDO>
__device__ __forceinline__ void logits_epilogue(const LogitsParams& p, typename Core::acc_t (&acc)[Core::kMT][Core::kNT],
                                                int T_cur, int r0, int c0, unsigned char* tw, int tid = threadIdx.x) {
    constexpr int kMT = Core::kMT, kNT = Core::kNT;
    static_assert(Core::kWaveC == kGroupC, "a wavefront's c are one group of the softmax partials");
    constexpr int kRegs = 4 * Core::kRuns;          // accumulator registers of a tile
    const typename Core::Lane lp(tid);
    // What the rows need from memory is asked for at once: tile by tile, behind the tile's stores, it was eight
    // times a load's latency (5 % of the kernel at H = 1600, 2.5 % at 4096).  The first pass of the forward modes
    // has ref = 0 everywhere.
    constexpr bool kRef = MODE == MODE_BWD || REDO;
    int y[kNT];
    float ref[kNT];
    bool act[kNT];                                        // this pass writes the row's results
#pragma unroll
    for (int nt = 0; nt < kNT; ++nt) {
        const int i = r0 + lp.r(nt);
        y[nt] = p.labels_t[i];                            // (padding rows: -1)
        ref[nt] = kRef ? p.ref[i] : 0.f;
        act[nt] = !REDO || p.rowstate[i] != 0;
    }
#pragma unroll
    for (int nt = 0; nt < kNT; ++nt) {
        if (c0 + kBlockC > p.V) {                         // columns beyond the vocabulary (last column block)
#pragma unroll
            for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
                for (int j = 0; j < kRegs; ++j)
                    if (c0 + lp.c(mt, j >> 2) + (j & 3) >= p.V) acc[mt][nt][j] = -INFINITY;
        }
        // e = exp(z - ref) as exp2(z * log2(e) - ref * log2(e)); summed in fp32, stored as bf16.
        // In the accumulators a lane holds 4 consecutive columns of one row, so a direct store
        // would scatter 8-byte pieces over many rows per instruction.  The wavefront instead turns
        // its kTile x 128 piece around in LDS (free once the k-loop is over; each wavefront has its
        // own region and LDS serves a wavefront's accesses in order, so no barrier is needed) and
        // stores whole 256-byte row segments.
        const float ref2 = ref[nt] * kLog2e;
        float s = 0.f;
#pragma unroll
        for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
            for (int q = 0; q < Core::kRuns; ++q) {
                bf16x4_t o;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const float z = acc[mt][nt][q * 4 + x];
                    const float e = __builtin_amdgcn_exp2f(kRef ? fmaf(z, kLog2e, -ref2) : z * kLog2e);
                    s += e;
                    o[x] = (__bf16)e;
                }
                if (MODE != MODE_FWD)
                    *reinterpret_cast<bf16x4_t*>(tw + lp.lrow * kTurnPitch + lp.cw(mt, q) * 2) = o;
            }
        if (MODE != MODE_FWD) {
            // (the rows' sums and label logits are stored by some lanes only, between one tile's turn and the next's)
            wave_sync<true>();
            const int lrow = lp.lane >> 4, lcol = lp.lane & 15;        // 4 rows x 16 chunks of 16 B
            const int rb = r0 + lp.rbase(nt);
            uint16_t* const out = p.stash + (int64_t)rb * p.Vp + c0 + lp.wc * kGroupC + lcol * 8;
#pragma unroll
            for (int it = 0; it < Core::kTile / 4; ++it) {
                const int row = it * 4 + lrow;
                const u32x4_t v = *reinterpret_cast<const u32x4_t*>(tw + row * kTurnPitch + lcol * 16);
                if (!REDO || p.rowstate[rb + row] != 0)
                    __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t*>(out + (int64_t)row * p.Vp));
            }
            wave_sync<true>();
        }
        // label logit: exactly one lane of one block holds column y of row i.  Few wavefronts
        // hold any (a tile's rows x 128 of V columns), so the search sits behind a uniform branch.
        const unsigned d = (unsigned)(y[nt] - (c0 + lp.wc * kGroupC));
        const bool mine = act[nt] && y[nt] >= 0 && d < (unsigned)kGroupC &&
                          ((d >> 2) & (unsigned)(Core::kGroups - 1)) == (unsigned)lp.grp;
        if (__ballot(mine) != 0ull) {
            if (mine) {
                float zl = 0.f;
#pragma unroll
                for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
                    for (int j = 0; j < kRegs; ++j)
                        if (d == (unsigned)(lp.cw(mt, j >> 2) + (j & 3))) zl = acc[mt][nt][j];
                p.zlabel[r0 + lp.r(nt)] = zl;
            }
        }
        if (MODE != MODE_BWD) {
            const int i = r0 + lp.r(nt);
            s = groups_sum<Core::kGroups>(s);
            if (lp.grp == 0 && act[nt]) p.ps[((c0 + lp.wc * kGroupC) >> 7) * p.Rc + i] = s;
            if (!REDO) {
                // A row whose total will leave [kSumLo, kSumHi] needs its exact maximum for the second
                // pass.  The group that holds it then has s > kSumHi / 2^17 groups / 128 columns, or
                // (with every other group) s < kSumLo: groups outside [kSumLo, 2^70] report theirs.
                const bool out = !(s >= kSumLo && s <= kGroupHi);
                if (__ballot(out) != 0ull) {
                    float m = -INFINITY;
#pragma unroll
                    for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
                        for (int j = 0; j < kRegs; ++j) m = fmaxf(m, acc[mt][nt][j]);
                    m = groups_max<Core::kGroups>(m);
                    if (out && lp.grp == 0) atomicMax(p.rmax + i, ordered_int(m));
                }
            }
        }
    }
}

// One block.  KTAIL: the hidden size is not whole k-steps.
// Core: DirectCore for a block, HalfCore for one half of its rows, RingCoreT<8> for a small one.
// warm: the block's warm-up row (large blocks).
template <class Core, bool KTAIL, int MODE, bool REDO>
__device__ __forceinline__ void logits_block(const LogitsParams& p, int T_cur, int Trc, int r0, int c0,
                                             const uint16_t* warm, unsigned char* smem) {
    if (r0 >= T_cur) return;        // (a second half of padding rows: the consumers' k-steps end before it)
    typename Core::acc_t acc[Core::kMT][Core::kNT];
    zero_acc<Core>(acc);
    Core::template gemm<KTAIL>({p.hidden_t, p.Hk, p.W, p.H, Trc, p.V, p.H, r0, c0, warm, kBlockK, nullptr}, smem, acc);
    logits_epilogue<Core, MODE, REDO>(p, acc, T_cur, r0, c0, smem + (threadIdx.x >> 6) * (Core::kTile * kTurnPitch));
}

template <bool KTAIL, int MODE, bool REDO>
__global__ __launch_bounds__(DirectCore::kThreads) void logits_kernel(const LogitsParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int T_cur = p.info->Tc, Trc = p.info->Trc;
    if (T_cur == 0) return;
    if (REDO && !p.info->redo) return;
    const PatchGrid pg = {Trc / kBlockR, p.Vp / kBlockC, p.PR, p.PC};
    const Halving last = halve_last_round(pg.blocks());
    const bool rows = by_rows(pg, p.H);
    const int number = block_of_workgroup(blockIdx.x, last.numbers, rows);
    if (number < 0) return;
    int tr, tc, half;
    block_at(pg, last.block(number, half), rows, tr, tc);
    const int r0 = tr * kBlockR, c0 = tc * kBlockC;
    const uint16_t* warm = warm_row(p.PR, p.PC, p.hidden_t, p.Hk, r0, tr, p.W, p.H, c0, tc, nullptr, Trc, p.V);
    if (half < 0) logits_block<DirectCore, KTAIL, MODE, REDO>(p, T_cur, Trc, r0, c0, warm, smem);
    else logits_block<HalfCore, KTAIL, MODE, REDO>(p, T_cur, Trc, r0 + half * (kBlockR / 2), c0, warm, smem);
}

// The first pass on persistent workgroups that fetch their next block's first two k-steps while the current block's
// last two and its epilogue run (DirectCore::Pipe); a last round in halves comes behind the chain.  The
// hidden size is whole k-steps and at least 4 of them.
template <int MODE>
__global__ __launch_bounds__(DirectCore::kThreads) void logits_chain_kernel(const LogitsParams p) {
    typedef DirectCore Core;
    extern __shared__ __align__(16) unsigned char smem[];
    const int T_cur = uniform(p.info->Tc), Trc = uniform(p.info->Trc);
    if (T_cur == 0) return;
    const PatchGrid pg = {Trc / kBlockR, p.Vp / kBlockC, p.PR, p.PC};
    const Halving last = halve_last_round(pg.blocks());
    const bool rows = by_rows(pg, p.H);
    const int whole = (last.full + kRound - 1) / kRound * kRound;          // the chains' workgroup numbers
    auto next_block = [&](int bid, Core::Block& blk) {
        for (; bid < whole; bid += gridDim.x) {
            const int number = block_of_workgroup(bid, last.numbers, rows);
            if (number < 0) continue;
            int tr, tc;
            block_at(pg, number, rows, tr, tc);
            const int r0 = tr * kBlockR, c0 = tc * kBlockC;
            blk = {uniform(p.hidden_t), p.Hk, uniform(p.W), p.H, Trc, p.V, p.H, uniform(r0), uniform(c0),
                   warm_row(p.PR, p.PC, p.hidden_t, p.Hk, r0, tr, p.W, p.H, c0, tc, nullptr, Trc, p.V), kBlockK, nullptr};
            return uniform(bid);
        }
        return -1;
    };
    Core::Block cur, nxt;
    int bid = next_block(blockIdx.x, cur);
    Core::Pipe<false> pipe(smem);
    if (bid >= 0) pipe.start(cur);
    const bool chain = bid >= 0;
    while (bid >= 0) {
        const int nbid = next_block(bid + gridDim.x, nxt);
        if (nbid < 0) nxt = cur;        // the last block: the chain's fetch goes to this block again, unused
        typename Core::acc_t acc[Core::kMT][Core::kNT];
        zero_acc<Core>(acc);
        pipe.run(cur, nxt, acc);
        // (what depends on the lane alone is worked out again for every block: kept over the blocks it is spilled)
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        logits_epilogue<Core, MODE, false>(p, acc, T_cur, cur.r0, cur.c0,
                                           smem + kChainTurnOffset + (tid >> 6) * (Core::kTile * kTurnPitch), tid);
        cur = nxt;
        bid = nbid;
    }
    if (chain) pipe.finish();
    for (bid = last.full + blockIdx.x; bid < last.numbers + kRound; bid += gridDim.x) {
        const int number = block_of_workgroup(bid, last.numbers, rows);
        if (number < last.full) continue;              // (none, or a whole block: the chain's)
        int tr, tc, half;
        block_at(pg, last.block(number, half), rows, tr, tc);
        const int r0 = tr * kBlockR, c0 = tc * kBlockC;
        const uint16_t* warm = warm_row(p.PR, p.PC, p.hidden_t, p.Hk, r0, tr, p.W, p.H, c0, tc, nullptr, Trc, p.V);
        __syncthreads();                // LDS is free
        logits_block<HalfCore, false, MODE, false>(p, T_cur, Trc, r0 + half * (kBlockR / 2), c0, warm, smem);
    }
}

// The same in small blocks.
typedef RingCoreT<8> LogitsSmallCore;
template <bool KTAIL, int MODE, bool REDO>
__global__ __launch_bounds__(LogitsSmallCore::kThreads) void logits_small_kernel(const LogitsParams p) {
    typedef LogitsSmallCore Core;
    extern __shared__ __align__(16) unsigned char smem[];
    const int T_cur = p.info->Tc, Trc = p.info->Trc;
    if (T_cur == 0) return;
    if (REDO && !p.info->redo) return;
    const PatchGrid pg = {Trc / Core::kRows, p.Vp / Core::kCols, p.PR, p.PC};
    const int number = block_of_workgroup(blockIdx.x, pg.blocks(), false);
    if (number < 0) return;
    int tr, tc;
    block_at(pg, number, false, tr, tc);
    logits_block<Core, KTAIL, MODE, REDO>(p, T_cur, Trc, tr * Core::kRows, tc * Core::kCols, nullptr, smem);
}

struct DHiddenParams {
    const uint16_t* dz;      // [Rc, Vp]     the chunk's dense rows
    const uint16_t* Wt;      // [H, Vp]      W transposed (k = vocabulary id contiguous), zero from V to whole k-steps
    uint16_t* dH_t;          // [N, H]       whole dHidden; dense row i goes to row idx[i]
    const int32_t* idx;
    const ChunkInfo* info;
    const Header* hdr;
    const float* frow;       // [Rc]         scale of each dense row's result: 1 / S of its softmax
    float* part;             // [splits, Trc, H] fp32 partial products (splits > 1); the number
                             // of ranges and their length are the chunk's (ChunkInfo)
    int H, V, Vp;
    int PR, PC;              // patch shape of the block -> tile mapping
};

// dH = dZ W runs with both operands k-contiguous (the fastest of the block GEMM's layouts: 9 % on
// this product): W transposed, [H, Vp] with zeros from V to whole k-steps, is made once per call that
// computes gradients (transpose_piece), for the price of reading and writing W once.

// r = token row (lane dimension), c = hidden index (register dimension), k = vocabulary; both
// operands k-contiguous (dZ rows and the rows of W transposed).
// The output has only (rows / 256) * (H / 256) blocks, each with a long contraction: when that
// number does not fill the compute units evenly, the contraction is cut into `splits` ranges, each
// range's blocks write fp32 partial products, and dhidden_reduce_kernel adds them in a fixed
// order.
// warm: the block's warm-up row for k = 0 (large blocks).
template <class Core>
__device__ __forceinline__ void dhidden_block(const DHiddenParams& p, int T_cur, int Trc, int splits, int ksteps,
                                              int split, int r0, int c0, const uint16_t* warm, unsigned char* smem) {
    constexpr int kMT = Core::kMT, kNT = Core::kNT;
    if (r0 >= T_cur) return;
    // k runs over V rounded up to whole k-steps: dZ and Wt are zero there
    const int k0 = split * ksteps * kBlockK;
    const int klen = min(ksteps * kBlockK, (p.V + kBlockK - 1) / kBlockK * kBlockK - k0);     // > 0

    typename Core::acc_t acc[kMT][kNT];
    zero_acc<Core>(acc);

    const uint16_t* const dz = p.dz + k0;
    const uint16_t* const Wk = p.Wt + k0;
    // (a hidden size that ends inside the block: the rows of Wt beyond H are read from its last
    // row, and the epilogue skips those columns)
    Core::template gemm<false>({dz, p.Vp, Wk, p.Vp, Trc, p.H, klen, r0, c0, warm, kBlockK, nullptr}, smem, acc);

    const typename Core::Lane lp;
    if (splits > 1) {
        float* const part = p.part + (int64_t)split * Trc * p.H;
#pragma unroll
        for (int nt = 0; nt < kNT; ++nt) {
            float* row = part + (int64_t)(r0 + lp.r(nt)) * p.H;
#pragma unroll
            for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
                for (int q = 0; q < Core::kRuns; ++q) {
                    const int h = c0 + lp.c(mt, q);
                    if (h >= p.H) continue;             // last column block of a ragged H
                    f32x4_t o;
#pragma unroll
                    for (int x = 0; x < 4; ++x) o[x] = acc[mt][nt][q * 4 + x];
                    *reinterpret_cast<f32x4_t*>(row + h) = o;
                }
        }
        return;
    }
    const float inv = p.hdr->inv;
    float frow[kNT];                                // (all asked for at once, see logits_epilogue)
    int token[kNT];
#pragma unroll
    for (int nt = 0; nt < kNT; ++nt) {
        const int i = r0 + lp.r(nt) < T_cur ? r0 + lp.r(nt) : T_cur - 1;
        frow[nt] = p.frow[i];
        token[nt] = p.idx[i];
    }
#pragma unroll
    for (int nt = 0; nt < kNT; ++nt) {
        const int i = r0 + lp.r(nt);
        if (i >= T_cur) continue;
        const float sc = inv * frow[nt];
        uint16_t* row = p.dH_t + (int64_t)token[nt] * p.H;
#pragma unroll
        for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
            for (int q = 0; q < Core::kRuns; ++q) {
                const int h = c0 + lp.c(mt, q);
                if (h >= p.H) continue;             // last column block of a ragged H
                bf16x4_t o;
#pragma unroll
                for (int x = 0; x < 4; ++x) o[x] = (__bf16)(acc[mt][nt][q * 4 + x] * sc);
                *reinterpret_cast<bf16x4_t*>(row + h) = o;
            }
    }
}

__global__ __launch_bounds__(DirectCore::kThreads) void dhidden_kernel(const DHiddenParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int T_cur = p.info->Tc, Trc = p.info->Trc;
    if (T_cur == 0) return;
    // the ranges are parts of one launch: their blocks are numbered through
    const PatchGrid pg = {Trc / kBlockR, (p.H + kBlockC - 1) / kBlockC, p.PR, p.PC};
    const int splits = p.info->splits, ksteps = p.info->ksteps;
    const Halving last = halve_last_round(pg.blocks() * splits);
    const bool rows = by_rows(pg, ksteps * kBlockK);
    const int number = block_of_workgroup(blockIdx.x, last.numbers, rows);
    if (number < 0) return;
    int tr, tc, half;
    const int i = last.block(number, half), split = i / pg.blocks();
    block_at(pg, i - split * pg.blocks(), rows, tr, tc);
    const int r0 = tr * kBlockR, c0 = tc * kBlockC, k0 = split * ksteps * kBlockK;
    const uint16_t* warm = warm_row(p.PR, p.PC, p.dz + k0, p.Vp, r0, tr, p.Wt + k0, p.Vp, c0, tc, nullptr, Trc, p.H);
    if (half < 0) dhidden_block<DirectCore>(p, T_cur, Trc, splits, ksteps, split, r0, c0, warm, smem);
    else dhidden_block<HalfCore>(p, T_cur, Trc, splits, ksteps, split, r0 + half * (kBlockR / 2), c0, warm, smem);
}

// The same in small blocks (the ranges are those that suit the large ones).
template <class Core>
struct DHiddenSmall {
    const DHiddenParams& p;
    int T_cur, Trc, splits;
    PatchGrid pg;
    __device__ __forceinline__ explicit DHiddenSmall(const DHiddenParams& p_)
        : p(p_), T_cur(p_.info->Tc), Trc(p_.info->Trc), splits(p_.info->splits),
          pg{Trc / Core::kRows, (p_.H + Core::kCols - 1) / Core::kCols, p_.PR, p_.PC} {}
    __device__ __forceinline__ int blocks() const { return T_cur == 0 ? 0 : pg.blocks() * splits; }
    __device__ __forceinline__ void run(int number, unsigned char* smem) const {
        int tr, tc;
        const int split = number / pg.blocks();
        block_at(pg, number - split * pg.blocks(), false, tr, tc);
        dhidden_block<Core>(p, T_cur, Trc, splits, p.info->ksteps, split, tr * Core::kRows, tc * Core::kCols, nullptr, smem);
    }
};
template <class Core>
__global__ __launch_bounds__(Core::kThreads) void dhidden_small_kernel(const DHiddenParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    const DHiddenSmall<Core> dh(p);
    const int number = block_of_workgroup(blockIdx.x, dh.blocks(), false);
    if (number >= 0) dh.run(number, smem);
}

// dH[idx[i]] = (g/M) (1/S_i) * sum over the ranges of the partial products of dense row i, in
// range order.  Chunks whose contraction was not cut were written by dhidden_kernel itself.
// make_loss (the last chunk of a call of up to kLossInReduceRows rows that wants it): workgroup 0 makes the loss and the
// rows come behind it.  That saves a launch where one workgroup of 256 has added up the terms before the rows are done, and is
// a tail behind them where it hasn't; us of a call, a launch of its own / in this one: 512 x 256 x 4096 40.4 / 38.2, 4096 x 256 x
// 4096 90.8 / 87.5, 16384 241.7 / 239.0, 400000 5535 / 5553; 32768 x 64 x 512 227.5 / 229.2, 131072 x 64 x 512 850.9 / 872.4.
constexpr int64_t kLossInReduceRows = 16384;
__global__ __launch_bounds__(256) void dhidden_reduce_kernel(const float* __restrict__ part, int H,
                                                             const int32_t* __restrict__ idx,
                                                             const ChunkInfo* __restrict__ info,
                                                             const Header* __restrict__ hdr,
                                                             const float* __restrict__ frow,
                                                             uint16_t* __restrict__ dH, int make_loss, const LossParams loss) {
    const int i = (int)blockIdx.x - make_loss;
    if (i < 0) {
        loss_reduce<256>(loss);
        return;
    }
    const int splits = info->splits, Trc = info->Trc;
    if (i >= info->Tc || splits <= 1) return;
    const float inv = hdr->inv * frow[i];
    uint16_t* out = dH + (int64_t)idx[i] * H;
    for (int c = threadIdx.x * 4; c < H; c += 256 * 4) {
        f32x4_t a = *reinterpret_cast<const f32x4_t*>(part + (int64_t)i * H + c);
        for (int sp = 1; sp < splits; ++sp)
            a += *reinterpret_cast<const f32x4_t*>(part + ((int64_t)sp * Trc + i) * H + c);
        bf16x4_t o;
#pragma unroll
        for (int x = 0; x < 4; ++x) o[x] = (__bf16)(a[x] * inv);
        *reinterpret_cast<bf16x4_t*>(out + c) = o;
    }
}

struct DWParams {
    const uint16_t* hg;      // [Kg, Hk]     the group's dense hidden rows (H of the Hk columns used)
    const uint16_t* dzg;     // [Kg, Vp]     their dZ rows
    GradOut out;             // [V, H] (scale and last: the kernel finds them)
    const Header* hdr;
    int64_t row0, rows;      // the group's dense rows: row0 .. row0 + rows - 1, as far as they exist
    int H, Hk, V, Vp;
    int PR, PC;              // patch shape of the block -> tile mapping
};

// r = hidden index (lane dimension), c = vocabulary id (register dimension), k = dense token row:
// both operands have k as the slow index (k-major cores).  With the hidden index along the lanes
// the accumulate moves full 128-byte lines of the sums (weight_grad_block).
// Core: KMajorCore for a block, KMajorHalfCore for half of its columns.
template <class Core>
__device__ __forceinline__ void dw_block(const DWParams& p, int Tkc, int64_t left, int r0, int c0,
                                         unsigned char* smem) {
    if (c0 >= p.V) return;
    typename Core::acc_t acc[Core::kMT][Core::kNT];
    zero_acc<Core>(acc);

    if (Tkc > 0)
        Core::template gemm<false>(p.hg, p.Hk, p.H, p.dzg, p.Vp, p.Vp, Tkc, r0, c0, smem, acc, nullptr, 0);

    // the last group with dense rows finishes dW = (g/M) sums
    GradOut out = p.out;
    out.scale = p.hdr->inv;
    out.last = left <= p.rows;
    weight_grad_block<Core>(acc, out, r0, c0, p.H, p.V, smem);
}

__global__ __launch_bounds__(KMajorCore::kThreads) void dw_kernel(const DWParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    int tr, tc, half;
    const int tiles_r = (p.H + kBlockR - 1) / kBlockR;
    // k extent of the group (its dense rows are zero padded to whole blocks)
    const int64_t left = p.hdr->n_valid - p.row0;
    const int Tkc = left <= 0 ? 0 : (int)(((left < p.rows ? left : p.rows) + kBlockK - 1) / kBlockK * kBlockK);
    if (Tkc == 0 && !p.out.first) return;
    const PatchGrid pg = {tiles_r, p.Vp / kBlockC, p.PR, p.PC};
    const Halving last = halve_last_round(pg.blocks());
    const int number = block_of_workgroup(blockIdx.x, last.numbers, false);
    if (number < 0) return;
    block_at(pg, last.block(number, half), false, tr, tc);
    if (half < 0) dw_block<KMajorCore>(p, Tkc, left, tr * kBlockR, tc * kBlockC, smem);
    else dw_block<KMajorHalfCore>(p, Tkc, left, tr * kBlockR, tc * kBlockC + half * (kBlockC / 2), smem);
}

// The same in small blocks.
template <class Core>
struct DWSmall {
    const DWParams& p;
    int64_t left;
    int Tkc;
    PatchGrid pg;
    __device__ __forceinline__ explicit DWSmall(const DWParams& p_)
        : p(p_), left(p_.hdr->n_valid - p_.row0),
          Tkc(left <= 0 ? 0 : (int)(((left < p_.rows ? left : p_.rows) + kBlockK - 1) / kBlockK * kBlockK)),
          pg{(p_.H + Core::kRows - 1) / Core::kRows, (p_.V + Core::kCols - 1) / Core::kCols, p_.PR, p_.PC} {}
    __device__ __forceinline__ int blocks() const { return Tkc == 0 && !p.out.first ? 0 : pg.blocks(); }
    __device__ __forceinline__ void run(int number, unsigned char* smem) const {
        int tr, tc;
        block_at(pg, number, false, tr, tc);
        dw_block<Core>(p, Tkc, left, tr * Core::kRows, tc * Core::kCols, smem);
    }
};
template <class Core>
__global__ __launch_bounds__(Core::kThreads) void dw_small_kernel(const DWParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    const DWSmall<Core> dw(p);
    const int number = block_of_workgroup(blockIdx.x, dw.blocks(), false);
    if (number >= 0) dw.run(number, smem);
}

// dHidden of a group's last chunk and the group's dW in one launch, both in small blocks: neither reads what the other
// writes (dHidden's partial products lie behind the rows that dW reads), and with at most one round of blocks in all, each
// has a compute unit of its own.
template <class Core, class DWCore>
__global__ __launch_bounds__(Core::kThreads) void gradients_small_kernel(const DHiddenParams hp, const DWParams wp) {
    extern __shared__ __align__(16) unsigned char smem[];
    static_assert(Core::kThreads == DWCore::kThreads, "one launch");
    const DHiddenSmall<Core> dh(hp);
    const DWSmall<DWCore> dw(wp);
    const int first = dh.blocks();
    const int number = block_of_workgroup(blockIdx.x, first + dw.blocks(), false);
    if (number < 0) return;
    if (number < first) dh.run(number, smem);
    else dw.run(number - first, smem);
}
template <class Core, class DWCore>
constexpr int gradients_small_lds() { return Core::kLds > DWCore::kLds ? Core::kLds : DWCore::kLds; }

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
static int prepare_kernels_on_current_device() {
    int rc = ALST_OK;
    auto acc = [&](int r) { if (r != ALST_OK) rc = r; };
    acc(allow_big_lds(logits_kernel<false, MODE_FWD, false>));
    acc(allow_big_lds(logits_kernel<true, MODE_FWD, false>));
    acc(allow_big_lds(logits_kernel<false, MODE_FUSED, false>));
    acc(allow_big_lds(logits_kernel<true, MODE_FUSED, false>));
    acc(allow_big_lds(logits_kernel<false, MODE_BWD, false>));
    acc(allow_big_lds(logits_kernel<true, MODE_BWD, false>));
    acc(allow_big_lds(logits_kernel<false, MODE_FWD, true>));
    acc(allow_big_lds(logits_kernel<true, MODE_FWD, true>));
    acc(allow_big_lds(logits_kernel<false, MODE_FUSED, true>));
    acc(allow_big_lds(logits_kernel<true, MODE_FUSED, true>));
    acc(allow_big_lds(logits_chain_kernel<MODE_FWD>, kChainLdsBytes));
    acc(allow_big_lds(logits_chain_kernel<MODE_FUSED>, kChainLdsBytes));
    acc(allow_big_lds(logits_chain_kernel<MODE_BWD>, kChainLdsBytes));
    acc(allow_big_lds(logits_small_kernel<false, MODE_FWD, false>, LogitsSmallCore::kLds));
    acc(allow_big_lds(logits_small_kernel<true, MODE_FWD, false>, LogitsSmallCore::kLds));
    acc(allow_big_lds(logits_small_kernel<false, MODE_FUSED, false>, LogitsSmallCore::kLds));
    acc(allow_big_lds(logits_small_kernel<true, MODE_FUSED, false>, LogitsSmallCore::kLds));
    acc(allow_big_lds(logits_small_kernel<false, MODE_BWD, false>, LogitsSmallCore::kLds));
    acc(allow_big_lds(logits_small_kernel<true, MODE_BWD, false>, LogitsSmallCore::kLds));
    acc(allow_big_lds(logits_small_kernel<false, MODE_FWD, true>, LogitsSmallCore::kLds));
    acc(allow_big_lds(logits_small_kernel<true, MODE_FWD, true>, LogitsSmallCore::kLds));
    acc(allow_big_lds(logits_small_kernel<false, MODE_FUSED, true>, LogitsSmallCore::kLds));
    acc(allow_big_lds(logits_small_kernel<true, MODE_FUSED, true>, LogitsSmallCore::kLds));
    acc(allow_big_lds(dhidden_kernel));
    acc(allow_big_lds(dhidden_small_kernel<RingCoreT<4>>, RingCoreT<4>::kLds));
    acc(allow_big_lds(dhidden_small_kernel<RingCoreT<8>>, RingCoreT<8>::kLds));
    acc(allow_big_lds(dw_kernel));
    acc(allow_big_lds(dw_small_kernel<KMajorSplitT<2>>, KMajorSplitT<2>::kLds));
    acc(allow_big_lds(dw_small_kernel<KMajorSplitT<4>>, KMajorSplitT<4>::kLds));
    acc(allow_big_lds(gradients_small_kernel<RingCoreT<4>, KMajorSplitT<2>>, gradients_small_lds<RingCoreT<4>, KMajorSplitT<2>>()));
    acc(allow_big_lds(gradients_small_kernel<RingCoreT<8>, KMajorSplitT<4>>, gradients_small_lds<RingCoreT<8>, KMajorSplitT<4>>()));
    return rc;
}
// Once per device, whatever the number of host threads that make their first call together.
static int prepare_kernels() {
    static std::once_flag once[kMaxDevices];
    static int results[kMaxDevices];
    const int dev = current_device_slot();
    if (dev < 0) return ALST_ERR_HIP;
    std::call_once(once[dev], [dev] { results[dev] = prepare_kernels_on_current_device(); });
    return results[dev];
}

// A chunk of launches as the host sees it, which knows N only: dense rows first .. first + rows - 1, as far as
// they exist.
struct ChunkPlan {
    int64_t group0;            // first dense row of the chunk's dW group
    int64_t at, rows;          // the chunk's place in the group and length
    int Tr;                    // rows rounded up to the block height
    bool group_done;           // the group's last chunk
    // dHidden: where the fp32 partial products of its ranges go (a place in the workspace) and how many
    // rows of them fit; the most blocks, and whether they may have to be added up
    size_t part;
    int64_t part_rows, dh_blocks;
    bool dh_cut;
};
static ChunkPlan chunk_plan(const Layout& L, int64_t N, int64_t H, int64_t V, int64_t first, bool do_bwd) {
    ChunkPlan c = {};
    c.group0 = first / L.Kg * L.Kg;
    c.at = first - c.group0;
    const int64_t left = std::min(L.Kg - c.at, N - first);
    c.rows = left <= L.Rc ? left : L.step;
    c.Tr = (int)((c.rows + kBlockR - 1) / kBlockR * kBlockR);
    c.group_done = c.at + c.rows == L.Kg || first + c.rows == N;
    if (!do_bwd) return c;
    // The partial products: behind the chunk's per-row arrays, or in the rows of the stash that the group
    // has not reached, if these have more room (the next chunk's logits are written after they are added
    // up).  A short call has nearly all of the stash: N = 512, H = 256, V = 4096 takes 8 ranges where the
    // first place holds 1: the call 116 -> 65 us.
    c.part = L.part;
    size_t bytes = L.part_bytes;
    const size_t behind = (size_t)(L.Kg - c.at - c.Tr) * L.Vp * 2;
    if (behind > bytes) {
        c.part = L.stash + (size_t)(c.at + c.Tr) * L.Vp * 2;
        bytes = behind;
    }
    c.part_rows = (int64_t)(bytes / ((size_t)H * 4));
    c.dh_blocks = dhidden_most_blocks(c.Tr, H, V, c.part_rows, c.dh_cut);
    return c;
}

struct Problem {
    const uint16_t* hidden;
    const uint16_t* W;
    const int32_t* labels;
    const float* lse_in;
    int64_t N, H, V, tile;
    int ignore_index;
    float grad_loss;
    float* loss_out;
    float* lse_out;
    int64_t* n_valid_out;
    uint16_t* dHidden;
    void* dW;
    unsigned char* ws;
    uint32_t flags;
    hipStream_t stream;
};

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// own_scratch: the workspace is the library's own static buffer of workspace_bytes (P.ws is not
// looked at).
static int validate(const Problem& P, size_t workspace_bytes, bool need_fwd_out, bool need_bwd_out,
                    bool need_lse_in, bool own_scratch = false) {
    if (!P.hidden || !P.W || !P.labels || (!own_scratch && !P.ws)) return ALST_ERR_NULL;
    if (need_fwd_out && !P.loss_out) return ALST_ERR_NULL;
    if (need_bwd_out && (!P.dHidden || !P.dW)) return ALST_ERR_NULL;
    if (need_lse_in && !P.lse_in) return ALST_ERR_NULL;
    if (P.flags & ~kKnownFlags) return ALST_ERR_UNSUPPORTED;
    if (need_bwd_out && (P.flags & ALST_FLAG_FORWARD_ONLY)) return ALST_ERR_UNSUPPORTED;
    if (P.N < 1 || P.H < 1 || P.V < 1 || P.tile < 1) return ALST_ERR_SHAPE;
    if (P.N > (int64_t)1 << 30 || P.H > (int64_t)1 << 20 || P.V > (int64_t)1 << 24)
        return ALST_ERR_SHAPE;
    if (P.H % 8 != 0) return ALST_ERR_ALIGN;
    if (!aligned16(P.hidden) || !aligned16(P.W) || (!own_scratch && !aligned16(P.ws)))
        return ALST_ERR_ALIGN;
    if (need_bwd_out && (!aligned16(P.dHidden) || !aligned16(P.dW))) return ALST_ERR_ALIGN;
    const Layout L = make_layout(P.N, P.H, P.V, P.tile, P.flags);
    // tiles beyond these many blocks are refused (what a launch holds, make_layout sees to)
    if (!checked_grid(L.Tp / kBlockR, L.Vp / kBlockC) ||
        !checked_grid((P.H + kBlockR - 1) / kBlockR, L.Vp / kBlockC) ||
        L.Tp / kBlockR * ((P.H + kBlockC - 1) / kBlockC) > 0x7fffff00 ||
        (L.Vp / 256) * (L.Tp / 64) > 0x7fffffff)
        return ALST_ERR_SHAPE;
    if (workspace_bytes < L.total) return own_scratch ? ALST_ERR_NOALLOC_LIMIT : ALST_ERR_WORKSPACE;
    return ALST_OK;
}

// Grids are sized for Tr (the chunk's rows rounded up to the block height); the kernels read the
// number of rows that take part from the device and surplus blocks leave at once.
struct LogitsLaunch {
    int columns;               // of small blocks, or 0: large ones
    bool chain;                // the first pass runs on chains of blocks
    PatchGrid pg;
    int grid;                  // workgroups (a chain has no more than there are compute units)
};
static LogitsLaunch choose_logits(int Tr, int Vp, int64_t H) {
    LogitsLaunch l = {};
    // (small blocks: 128 columns only, a group of the softmax partials)
    if (small_blocks(Tr, Vp, LogitsSmallCore::kCols) <= kRound) {
        l.columns = LogitsSmallCore::kCols;
        l.pg = choose_patches(Tr / LogitsSmallCore::kRows, Vp / LogitsSmallCore::kCols);
    } else {
        l.pg = choose_patches(Tr / kBlockR, Vp / kBlockC);
        l.chain = chain_pays(l.pg.blocks(), H, true);
    }
    l.grid = grid_for_blocks(l.pg.blocks());
    return l;
}
template <int MODE, bool REDO>
static int launch_logits(LogitsParams lp, int Tr, bool ktail, hipStream_t s) {
    const LogitsLaunch l = choose_logits(Tr, lp.Vp, lp.H);
    lp.PR = l.pg.PR; lp.PC = l.pg.PC;
    const dim3 grid((unsigned)l.grid), threads(DirectCore::kThreads);
    constexpr int lds = LogitsSmallCore::kLds;
    if (l.columns && ktail) hipLaunchKernelGGL((logits_small_kernel<true, MODE, REDO>), grid, threads, lds, s, lp);
    else if (l.columns) hipLaunchKernelGGL((logits_small_kernel<false, MODE, REDO>), grid, threads, lds, s, lp);
    else if (!REDO && l.chain)
        hipLaunchKernelGGL((logits_chain_kernel<MODE>), dim3((unsigned)std::min(l.grid, persistent_grid())), threads,
                           kChainLdsBytes, s, lp);
    else if (ktail) hipLaunchKernelGGL((logits_kernel<true, MODE, REDO>), grid, threads, kLdsBytes, s, lp);
    else hipLaunchKernelGGL((logits_kernel<false, MODE, REDO>), grid, threads, kLdsBytes, s, lp);
    return hipGetLastError() == hipSuccess ? ALST_OK : ALST_ERR_HIP;
}

// W transposed for the call's dHidden (nothing to transpose: forward only).
static Transpose weight_transpose(const Layout& L, const uint16_t* W, uint16_t* wt, int64_t H, int64_t V, bool do_bwd) {
    return {W, do_bwd ? (int)V : 0, do_bwd ? (int)H : 0, H, wt, L.Vp, (int)((V + kBlockK - 1) / kBlockK * kBlockK)};
}
// The launch that gathers the rows of the chunk that begins at dense row `first`.
struct GatherLaunch {
    bool numbers;              // it numbers the rows too
    int64_t zero_blocks;       // workgroups that look for ignored tokens
    int64_t pieces;            // workgroups that transpose W
    bool transposes_apart;     // W is transposed by a launch of its own: this one would be more than a grid
};
static GatherLaunch choose_gather(const Layout& L, const Transpose& t, int64_t N, int64_t H, int64_t V, int64_t first, int Tr,
                                  bool do_bwd) {
    GatherLaunch g = {};
    g.numbers = N <= kGatherIndexRows && chunk_plan(L, N, H, V, 0, false).rows == N;
    g.zero_blocks = do_bwd && first == 0 ? std::min<int64_t>((N + kZeroRows - 1) / kZeroRows, kZeroBlocksMax) : 0;
    g.pieces = first == 0 ? t.pieces() : 0;
    g.transposes_apart = g.pieces > kGridBlocks - Tr - g.zero_blocks;
    if (g.transposes_apart) g.pieces = 0;
    return g;
}

// The launches of a chunk's gradients.
struct GradientLaunches {
    int dh_columns, dw_columns;        // of small blocks, or 0: large ones (dw_columns: the group is complete)
    bool together;                     // dHidden and dW in one launch, both in small blocks of dh_columns
    PatchGrid dw;
    int dh_grid, dw_grid;
};
// dHidden in small blocks (a block is 16 of 64 columns or fewer), and dW, which joins its launch while both together are
// at most one round; us of a call, two launches / one: 512 x 256 x 4096 40.1 / 38.1, 512 x 1024 x 1024 46.2 / 42.7, 300 x 256 x 1000
// 36.2 / 30.7.  Where dW's blocks become wider, up to 1024 + 10 times as many rows as a range of V has words: 3500 x 512 x 256 58.1 / 56.4,
// 5000 x 256 x 512 71.0 / 64.5; beyond: 4096 x 256 x 256 53.3 / 54.2, 7000 x 128 x 256 63.2 / 65.6.  Where dHidden's do, ranges
// of up to 2048 more words than rows: beyond, 256 x 64 x 24000 54.1 / 58.0.
static GradientLaunches choose_gradients(const ChunkPlan& c, int64_t H, int64_t V, int64_t Vp) {
    GradientLaunches g = {};
    auto dh_small = [&](int64_t cols) { return c.dh_blocks * 4 * (kBlockC / cols); };
    auto dw_small = [&](int64_t cols) { return small_blocks(H, V, cols); };
    int ranges, ksteps;                // of a chunk whose rows are all there
    dhidden_splits(c.Tr, H, V, c.part_rows, ranges, ksteps);
    const int64_t range = (int64_t)ksteps * kBlockK, group_rows = c.at + c.rows;
    const int both = !c.group_done ? 0 : joint_block_columns(dh_small, range <= 2048 + group_rows,
                                                             dw_small, group_rows <= 1024 + 10 * range);
    g.together = both != 0;
    g.dh_columns = both ? both : small_block_columns(dh_small);
    // (enough workgroups for whatever number of rows and ranges the chunk turns out to have)
    g.dh_grid = g.dh_columns ? kRound : grid_for_blocks(c.dh_blocks);
    if (!c.group_done) return g;
    g.dw_columns = both ? both : small_block_columns(dw_small);
    g.dw = g.dw_columns ? choose_patches((int)((H + kSmallRows - 1) / kSmallRows), (int)((V + g.dw_columns - 1) / g.dw_columns))
                        : choose_patches((int)((H + kBlockR - 1) / kBlockR), (int)(Vp / kBlockC));
    g.dw_grid = both ? 0 : grid_for_blocks(g.dw.blocks());
    return g;
}

// The logits pass of a chunk and the per-row work behind it; for the modes that form the softmax
// sums, followed by the conditional second pass (see row_finish_kernel).
template <int MODE>
static int logits_and_finish(const LogitsParams& lp, const RowFinishParams& fp, int Tr, int tiles, bool ktail,
                             hipStream_t s) {
    const dim3 fgrid(Tr / kCombineRows), fblock(kCombineRows, kCombineLanes);
    int rc;
    {
        ProfScope ps_(PROF_LOGITS, s, tiles);
        rc = launch_logits<MODE, false>(lp, Tr, ktail, s);
    }
    if (rc != ALST_OK) return rc;
    {
        ProfScope small_(PROF_OTHER, s);
        hipLaunchKernelGGL((row_finish_kernel<MODE, false>), fgrid, fblock, 0, s, fp);
        ALST_HIP(hipGetLastError());
    }
    if (MODE == MODE_BWD) return ALST_OK;
    constexpr int M2 = MODE == MODE_BWD ? MODE_FUSED : MODE;      // (MODE_BWD never gets here)
    // (timed with the small kernels: in all but pathological inputs both launches are empty)
    ProfScope small_(PROF_OTHER, s);
    rc = launch_logits<M2, true>(lp, Tr, ktail, s);
    if (rc != ALST_OK) return rc;
    hipLaunchKernelGGL((row_finish_kernel<M2, true>), fgrid, fblock, 0, s, fp);
    ALST_HIP(hipGetLastError());
    return ALST_OK;
}

// do_fwd: produce loss / lse.  do_bwd: produce gradients.  Both: one fused sweep.
static int run(const Problem& P, bool do_fwd, bool do_bwd) {
    int rc = prepare_kernels();
    if (rc != ALST_OK) return rc;
    const Layout L = make_layout(P.N, P.H, P.V, P.tile, P.flags);
    hipStream_t s = P.stream;
    Header* hdr = reinterpret_cast<Header*>(P.ws + L.header);
    ChunkInfo* info = reinterpret_cast<ChunkInfo*>(P.ws + L.cinfo);
    float* loss_rows = reinterpret_cast<float*>(P.ws + L.loss_rows);
    float* lse_buf = P.lse_out ? P.lse_out : reinterpret_cast<float*>(P.ws + L.lse);
    float* zlabel = reinterpret_cast<float*>(P.ws + L.zlabel);
    int32_t* yc = reinterpret_cast<int32_t*>(P.ws + L.yc);
    int32_t* idx = reinterpret_cast<int32_t*>(P.ws + L.idx);
    int32_t* block_cnt = reinterpret_cast<int32_t*>(P.ws + L.block_cnt);
    int64_t* block_ofs = reinterpret_cast<int64_t*>(P.ws + L.block_ofs);
    int32_t* rmax = reinterpret_cast<int32_t*>(P.ws + L.rmax);
    float* ps = reinterpret_cast<float*>(P.ws + L.ps);
    float* ref = reinterpret_cast<float*>(P.ws + L.ref);
    float* frow = reinterpret_cast<float*>(P.ws + L.frow);
    int32_t* rowstate = reinterpret_cast<int32_t*>(P.ws + L.rowstate);
    uint16_t* hc = reinterpret_cast<uint16_t*>(P.ws + L.hc);
    uint16_t* stash = reinterpret_cast<uint16_t*>(P.ws + L.stash);
    uint16_t* wt = reinterpret_cast<uint16_t*>(P.ws + L.wt);
    const bool acc_in_dw = (P.flags & ALST_FLAG_DW_FP32) && !(P.flags & ALST_FLAG_DW_ACCUMULATE);
    float* acc = acc_in_dw ? reinterpret_cast<float*>(P.dW) : reinterpret_cast<float*>(P.ws + L.acc);

    const int H = (int)P.H, V = (int)P.V, Vp = (int)L.Vp, ng = (int)L.ng;
    const int64_t T = P.tile < P.N ? P.tile : P.N;
    const int sum_mode = (P.flags & ALST_FLAG_REDUCE_SUM) ? 1 : 0;

    const Transpose transpose = weight_transpose(L, P.W, wt, P.H, P.V, do_bwd);
    if (choose_gather(L, transpose, P.N, P.H, P.V, 0, 0, do_bwd).numbers) {
        // (gather_rows_kernel numbers the rows)
    } else if (P.N <= kIndexRows) {
        hipLaunchKernelGGL(index_rows_kernel, dim3(1), dim3(kScanThreads), 0, s, P.labels, (int)P.N,
                           P.ignore_index, V, P.grad_loss, sum_mode, idx, do_fwd ? lse_buf : nullptr,
                           do_fwd ? loss_rows : nullptr, hdr, P.n_valid_out);
    } else {
        const int64_t nblocks = (P.N + kScanThreads - 1) / kScanThreads;
        hipLaunchKernelGGL(init_header_kernel, dim3(1), dim3(64), 0, s, hdr);
        hipLaunchKernelGGL(block_count_kernel, dim3((unsigned)nblocks), dim3(kScanThreads), 0, s,
                           P.labels, P.N, P.ignore_index, V, block_cnt, hdr);
        hipLaunchKernelGGL(block_offsets_kernel, dim3(1), dim3(kScanThreads), 0, s, block_cnt,
                           nblocks, block_ofs, hdr, P.grad_loss, sum_mode, P.n_valid_out);
        hipLaunchKernelGGL(scatter_index_kernel, dim3((unsigned)nblocks), dim3(kScanThreads), 0, s,
                           P.labels, P.N, P.ignore_index, V, block_ofs, idx,
                           do_fwd ? lse_buf : nullptr, do_fwd ? loss_rows : nullptr);
    }
    ALST_HIP(hipGetLastError());

    // The row extent of a chunk is always block-aligned (dense rows are zero padded to a multiple of the
    // block height).  A vocabulary that ends inside a column block: the logits kernel reads the last
    // row of W in place of the missing ones and masks those columns; a hidden size that is not whole
    // k-steps: what W's rows and the dense hidden rows have beyond H in the last one is read as zeros.
    const bool ktail_logits = (H % kBlockK) != 0;
    // A hidden size that ends inside a block: dHidden and dW read the last rows of W transposed / columns
    // of the dense hidden rows in place of the missing ones and discard the results; a vocabulary that
    // is not whole k-steps: dZ and W transposed are zero up to whole k-steps.
    const LossParams loss = {loss_rows, P.N, hdr, sum_mode, P.loss_out};
    bool loss_made = false;

    // The host does not know M: it walks the chunks of N rows, the most there can be; the kernels of
    // a chunk beyond the dense rows find Tc = 0 on the device and leave at once.
    for (int64_t first = 0, rows = 0; first < P.N; first += rows) {
        const ChunkPlan c = chunk_plan(L, P.N, P.H, P.V, first, do_bwd);
        rows = c.rows;
        const int Tr = c.Tr;
        const int32_t* idx_t = idx + first;             // the chunk's dense rows -> sequence rows
        // the caller's tiles that begin in this chunk, for the timers
        const int tiles = (int)((first + rows + T - 1) / T - (first + T - 1) / T);
        // (the forward-only layout has the rows of one chunk)
        uint16_t* const hc_t = hc + (do_bwd ? c.at : 0) * L.Hk;
        uint16_t* const stash_t = stash + (do_bwd ? c.at : 0) * L.Vp;
        float* const part = reinterpret_cast<float*>(P.ws + c.part);

        {
            ProfScope small_(PROF_OTHER, s);
            GatherParams gp;
            gp.hidden = P.hidden; gp.labels = P.labels; gp.idx = idx; gp.lse_in = do_fwd ? nullptr : P.lse_in;
            gp.hdr = hdr; gp.info = info; gp.Hc = hc_t; gp.yc = yc; gp.ref = ref; gp.rowstate = rowstate;
            gp.rmax = rmax; gp.dHidden = P.dHidden;
            gp.N = P.N; gp.first = first; gp.Rc = Tr; gp.H = P.H; gp.V = P.V;
            gp.dh_part_rows = c.part_rows;
            gp.Hk = (int)L.Hk; gp.ignore_index = P.ignore_index;
            const GatherLaunch g = choose_gather(L, transpose, P.N, P.H, P.V, first, Tr, do_bwd);
            gp.zero_blocks = g.zero_blocks;
            gp.hdr_out = hdr; gp.idx_out = idx; gp.lse = do_fwd ? lse_buf : nullptr;
            gp.loss_rows = do_fwd ? loss_rows : nullptr; gp.n_valid_out = P.n_valid_out;
            gp.grad_loss = P.grad_loss; gp.sum_mode = sum_mode;
            if (g.transposes_apart && !launch_transposes(Transposes{{transpose}}, s)) return ALST_ERR_HIP;
            const dim3 grid((unsigned)(Tr + g.zero_blocks + g.pieces));
            if (g.numbers) hipLaunchKernelGGL(gather_rows_kernel<true>, grid, dim3(256), 0, s, gp, transpose);
            else hipLaunchKernelGGL(gather_rows_kernel<false>, grid, dim3(256), 0, s, gp, transpose);
            ALST_HIP(hipGetLastError());
        }

        LogitsParams lp;
        lp.hidden_t = hc_t;
        lp.W = P.W;
        lp.labels_t = yc;
        lp.info = info;
        lp.ref = ref; lp.rowstate = rowstate;
        lp.rmax = rmax; lp.ps = ps; lp.zlabel = zlabel; lp.stash = stash_t;
        lp.Rc = L.Rc; lp.H = H; lp.Hk = (int)L.Hk; lp.V = V; lp.Vp = Vp;
        RowFinishParams fp;
        fp.ps = ps; fp.rmax = rmax; fp.zlabel = zlabel; fp.yc = yc; fp.idx = idx_t; fp.info = info;
        fp.ref = ref; fp.frow = frow; fp.rowstate = rowstate;
        fp.lse_t = lse_buf; fp.loss_rows_t = loss_rows; fp.hc = hc_t; fp.stash = stash_t;
        fp.Rc = L.Rc; fp.ng = ng; fp.H = H; fp.Hk = (int)L.Hk; fp.Vp = Vp;
        if (do_fwd && do_bwd) rc = logits_and_finish<MODE_FUSED>(lp, fp, Tr, tiles, ktail_logits, s);
        else if (do_fwd) rc = logits_and_finish<MODE_FWD>(lp, fp, Tr, tiles, ktail_logits, s);
        else rc = logits_and_finish<MODE_BWD>(lp, fp, Tr, tiles, ktail_logits, s);
        if (rc != ALST_OK) return rc;
        if (!do_bwd) continue;

        const GradientLaunches gl = choose_gradients(c, P.H, P.V, L.Vp);
        DWParams wp = {};
        if (c.group_done) {
            wp.hg = hc; wp.dzg = stash; wp.hdr = hdr;
            wp.out = {acc, P.dW, P.H, 0.f, c.group0 == 0, 0, (P.flags & ALST_FLAG_DW_FP32) != 0,
                      (P.flags & ALST_FLAG_DW_ACCUMULATE) != 0};
            wp.row0 = c.group0; wp.rows = L.Kg;
            wp.H = H; wp.Hk = (int)L.Hk; wp.V = V; wp.Vp = Vp;
            wp.PR = gl.dw.PR; wp.PC = gl.dw.PC;
        }
        {
            DHiddenParams dp;
            dp.dz = stash_t; dp.Wt = wt; dp.dH_t = P.dHidden; dp.idx = idx_t;
            dp.info = info; dp.hdr = hdr; dp.frow = frow;
            dp.part = part;
            dp.H = H; dp.V = V; dp.Vp = Vp;
            dp.PR = L.dh_PR; dp.PC = L.dh_PC;
            const dim3 grid((unsigned)gl.dh_grid), threads(DirectCore::kThreads);
            ProfScope ps_(PROF_DHIDDEN, s, tiles);
            if (gl.together && gl.dh_columns == 64)
                hipLaunchKernelGGL((gradients_small_kernel<RingCoreT<4>, KMajorSplitT<2>>), grid, threads,
                                   (gradients_small_lds<RingCoreT<4>, KMajorSplitT<2>>()), s, dp, wp);
            else if (gl.together)
                hipLaunchKernelGGL((gradients_small_kernel<RingCoreT<8>, KMajorSplitT<4>>), grid, threads,
                                   (gradients_small_lds<RingCoreT<8>, KMajorSplitT<4>>()), s, dp, wp);
            else if (gl.dh_columns == 64)
                hipLaunchKernelGGL(dhidden_small_kernel<RingCoreT<4>>, grid, threads, RingCoreT<4>::kLds, s, dp);
            else if (gl.dh_columns == 128)
                hipLaunchKernelGGL(dhidden_small_kernel<RingCoreT<8>>, grid, threads, RingCoreT<8>::kLds, s, dp);
            else
                hipLaunchKernelGGL(dhidden_kernel, grid, threads, kLdsBytes, s, dp);
            if (c.dh_cut) {
                loss_made = do_fwd && first + rows == P.N && P.N <= kLossInReduceRows;
                hipLaunchKernelGGL(dhidden_reduce_kernel, dim3(Tr + loss_made), dim3(256), 0, s, dp.part, H, idx_t,
                                   info, hdr, frow, P.dHidden, (int)loss_made, loss);
            }
            ALST_HIP(hipGetLastError());
        }
        if (c.group_done && !gl.together) {
            const dim3 grid((unsigned)gl.dw_grid), threads(KMajorCore::kThreads);
            ProfScope ps_(PROF_DW, s);
            if (gl.dw_columns == 64) hipLaunchKernelGGL(dw_small_kernel<KMajorSplitT<2>>, grid, threads, KMajorSplitT<2>::kLds, s, wp);
            else if (gl.dw_columns) hipLaunchKernelGGL(dw_small_kernel<KMajorSplitT<4>>, grid, threads, KMajorSplitT<4>::kLds, s, wp);
            else hipLaunchKernelGGL(dw_kernel, grid, threads, kLdsBytes, s, wp);
            ALST_HIP(hipGetLastError());
        }
    }

    if (do_fwd && !loss_made) {
        hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(1024), 0, s, loss);
        ALST_HIP(hipGetLastError());
    }
    return ALST_OK;
}

// ---------------------------------------------------------------------------------------------
// the entry point that allocates nothing
// ---------------------------------------------------------------------------------------------
// The workspace of alst_tiled_ce_forward_backward_noalloc: one array per GPU, held from the moment
// the library's code is loaded on it until the process ends.  In host code the name `scratch` is
// only a handle for hipGetSymbolAddress; what the kernels get is the address that call returns
// for the current device (each GPU has its own copy at its own address).
static __device__ __align__(256) unsigned char scratch[ALST_NOALLOC_SCRATCH_BYTES];

// The device address of `scratch` on the current device, looked up once per device.
static int noalloc_scratch(unsigned char** out) {
    static std::mutex lock;
    static unsigned char* ptrs[kMaxDevices];
    const int dev = current_device_slot();
    if (dev < 0) return ALST_ERR_HIP;
    std::lock_guard<std::mutex> hold(lock);
    if (!ptrs[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return ALST_ERR_HIP;
        ptrs[dev] = static_cast<unsigned char*>(p);
    }
    *out = ptrs[dev];
    return ALST_OK;
}

__global__ void copy_status_kernel(const Header* __restrict__ h, int32_t* __restrict__ out) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *out = h->status;
}

}  // namespace alst

// ---------------------------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------------------------
using namespace alst;

extern "C" {

const char* alst_status_string(int status) {
    switch (status) {
        case ALST_OK: return "ok";
        case ALST_ERR_NULL: return "a required pointer is NULL";
        case ALST_ERR_SHAPE: return "N, H, V and tile must be >= 1 and within the supported range";
        case ALST_ERR_ALIGN: return "H must be a multiple of 8 and base pointers 16-byte aligned";
        case ALST_ERR_WORKSPACE: return "workspace is smaller than alst_tiled_ce_workspace_bytes()";
        case ALST_ERR_LABEL_RANGE: return "a label is neither ignore_index nor inside [0, V)";
        case ALST_ERR_HIP: return "a HIP runtime call or kernel launch failed";
        case ALST_ERR_UNSUPPORTED: return "unknown flag bits, or a flag this entry point does not take";
        case ALST_ERR_NONFINITE: return "the loss is not finite";
        case ALST_ERR_NOALLOC_LIMIT:
            return "the problem needs more scratch than the static buffer of "
                   "alst_tiled_ce_forward_backward_noalloc holds";
        default: return "unknown status";
    }
}

int alst_version(void) { return 100; }

size_t alst_tiled_ce_workspace_bytes(int64_t N, int64_t H, int64_t V, int64_t tile, uint32_t flags) {
    if (N < 1 || H < 1 || V < 1 || tile < 1) return 0;
    if (N > (int64_t)1 << 30 || H > (int64_t)1 << 20 || V > (int64_t)1 << 24) return 0;
    if (flags & ~kKnownFlags) return 0;
    return make_layout(N, H, V, tile, flags).total;
}

int alst_tiled_ce_forward(const void* hidden, const void* W, const int32_t* labels, int64_t N,
                          int64_t H, int64_t V, int64_t tile, int32_t ignore_index, float* loss_out,
                          float* lse_out, int64_t* n_valid_out, void* workspace,
                          size_t workspace_bytes, uint32_t flags, void* stream) {
    Problem P = {};
    P.hidden = (const uint16_t*)hidden; P.W = (const uint16_t*)W; P.labels = labels;
    P.N = N; P.H = H; P.V = V; P.tile = tile; P.ignore_index = ignore_index; P.grad_loss = 1.f;
    P.loss_out = loss_out; P.lse_out = lse_out; P.n_valid_out = n_valid_out;
    P.ws = (unsigned char*)workspace; P.flags = flags; P.stream = (hipStream_t)stream;
    const int rc = validate(P, workspace_bytes, true, false, false);
    if (rc != ALST_OK) return rc;
    return run(P, true, false);
}

int alst_tiled_ce_backward(const void* hidden, const void* W, const int32_t* labels,
                           const float* lse, int64_t N, int64_t H, int64_t V, int64_t tile,
                           int32_t ignore_index, float grad_loss, void* dHidden, void* dW,
                           void* workspace, size_t workspace_bytes, uint32_t flags, void* stream) {
    Problem P = {};
    P.hidden = (const uint16_t*)hidden; P.W = (const uint16_t*)W; P.labels = labels;
    P.lse_in = lse;
    P.N = N; P.H = H; P.V = V; P.tile = tile; P.ignore_index = ignore_index;
    P.grad_loss = grad_loss; P.dHidden = (uint16_t*)dHidden; P.dW = dW;
    P.ws = (unsigned char*)workspace; P.flags = flags; P.stream = (hipStream_t)stream;
    const int rc = validate(P, workspace_bytes, false, true, true);
    if (rc != ALST_OK) return rc;
    return run(P, false, true);
}

int alst_tiled_ce_forward_backward(const void* hidden, const void* W, const int32_t* labels,
                                   int64_t N, int64_t H, int64_t V, int64_t tile,
                                   int32_t ignore_index, float grad_loss, float* loss_out,
                                   float* lse_out, int64_t* n_valid_out, void* dHidden, void* dW,
                                   void* workspace, size_t workspace_bytes, uint32_t flags,
                                   void* stream) {
    Problem P = {};
    P.hidden = (const uint16_t*)hidden; P.W = (const uint16_t*)W; P.labels = labels;
    P.N = N; P.H = H; P.V = V; P.tile = tile; P.ignore_index = ignore_index;
    P.grad_loss = grad_loss; P.loss_out = loss_out; P.lse_out = lse_out;
    P.n_valid_out = n_valid_out; P.dHidden = (uint16_t*)dHidden; P.dW = dW;
    P.ws = (unsigned char*)workspace; P.flags = flags; P.stream = (hipStream_t)stream;
    const int rc = validate(P, workspace_bytes, true, true, false);
    if (rc != ALST_OK) return rc;
    return run(P, true, true);
}

int alst_tiled_ce_forward_backward_noalloc(const void* hidden, const void* W, const int32_t* labels,
                                           int64_t N, int64_t H, int64_t V, int64_t tile,
                                           int32_t ignore_index, float grad_loss, float* loss_out,
                                           float* lse_out, int64_t* n_valid_out, void* dHidden,
                                           void* dW, int32_t* device_status_out, uint32_t flags,
                                           void* stream) {
    Problem P = {};
    P.hidden = (const uint16_t*)hidden; P.W = (const uint16_t*)W; P.labels = labels;
    P.N = N; P.H = H; P.V = V; P.tile = tile; P.ignore_index = ignore_index;
    P.grad_loss = grad_loss; P.loss_out = loss_out; P.lse_out = lse_out;
    P.n_valid_out = n_valid_out; P.dHidden = (uint16_t*)dHidden; P.dW = dW;
    P.flags = flags; P.stream = (hipStream_t)stream;
    int rc = validate(P, ALST_NOALLOC_SCRATCH_BYTES, true, true, false, /*own_scratch=*/true);
    if (rc != ALST_OK) return rc;
    rc = noalloc_scratch(&P.ws);
    if (rc != ALST_OK) return rc;
    // run() starts by resetting the header and writes every other region of the workspace before
    // it reads it, so what the last call left in the array does not matter
    rc = run(P, true, true);
    if (rc != ALST_OK) return rc;
    if (device_status_out) {
        hipLaunchKernelGGL(copy_status_kernel, dim3(1), dim3(64), 0, P.stream,
                           reinterpret_cast<const Header*>(P.ws), device_status_out);
        if (hipGetLastError() != hipSuccess) return ALST_ERR_HIP;
    }
    return ALST_OK;
}

int alst_last_device_status(void* workspace, void* stream) {
    if (!workspace) return ALST_ERR_NULL;
    Header h;
    if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return ALST_ERR_HIP;
    if (hipMemcpy(&h, workspace, sizeof(Header), hipMemcpyDeviceToHost) != hipSuccess)
        return ALST_ERR_HIP;
    const int st = h.status;
    if (st != 0) {
        hipLaunchKernelGGL(init_header_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream,
                           reinterpret_cast<Header*>(workspace));
        if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return ALST_ERR_HIP;
    }
    return st;
}

int alst_tiled_ce_token_losses(const void* workspace, size_t workspace_bytes, int64_t N, int64_t H,
                               int64_t V, int64_t tile, uint32_t flags, float* token_loss_out,
                               void* stream) {
    if (!workspace || !token_loss_out) return ALST_ERR_NULL;
    if (flags & ~kKnownFlags) return ALST_ERR_UNSUPPORTED;
    if (N < 1 || H < 1 || V < 1 || tile < 1) return ALST_ERR_SHAPE;
    if (N > (int64_t)1 << 30 || H > (int64_t)1 << 20 || V > (int64_t)1 << 24) return ALST_ERR_SHAPE;
    const Layout L = make_layout(N, H, V, tile, flags);
    if (workspace_bytes < L.total) return ALST_ERR_WORKSPACE;
    const float* rows = reinterpret_cast<const float*>((const unsigned char*)workspace + L.loss_rows);
    int blocks = (int)((N + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(copy_f32_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, rows,
                       token_loss_out, N);
    return hipGetLastError() == hipSuccess ? ALST_OK : ALST_ERR_HIP;
}

int alst_debug_ce_chunk(int64_t N, int64_t H, int64_t V, int64_t tile, uint32_t flags, int64_t chunk, int64_t dense,
                        alst_debug_ce_chunk_info* info) {
    if (!info) return ALST_ERR_NULL;
    if ((flags & ~kKnownFlags) || (flags & ALST_FLAG_FORWARD_ONLY)) return ALST_ERR_UNSUPPORTED;
    if (N < 1 || H < 1 || V < 1 || tile < 1 || chunk < 0) return ALST_ERR_SHAPE;
    if (N > (int64_t)1 << 30 || H > (int64_t)1 << 20 || V > (int64_t)1 << 24) return ALST_ERR_SHAPE;
    const Layout L = make_layout(N, H, V, tile, flags);
    ChunkPlan c = {};
    int64_t first = 0;
    for (int64_t k = 0; k <= chunk; ++k, first += c.rows) {
        if (first >= N) return ALST_ERR_SHAPE;
        c = chunk_plan(L, N, H, V, first, true);
    }
    if (dense < 0 || dense > c.rows) return ALST_ERR_SHAPE;
    const int64_t Trc = (dense + kBlockR - 1) / kBlockR * kBlockR;
    int ranges, ksteps;
    dhidden_splits(Trc, H, V, c.part_rows, ranges, ksteps);          // as gather_rows_kernel
    info->first = first - c.rows;
    info->rows = c.rows;
    info->group0 = c.group0;
    info->ranges = ranges;
    info->added_up = c.dh_cut;
    const int64_t at = first - c.rows;
    const GatherLaunch g = choose_gather(L, weight_transpose(L, nullptr, nullptr, H, V, true), N, H, V, at, c.Tr, true);
    const LogitsLaunch l = choose_logits(c.Tr, (int)L.Vp, H);
    const GradientLaunches gl = choose_gradients(c, H, V, L.Vp);
    info->dhidden_blocks = (gl.dh_columns ? Trc / kSmallRows * ((H + gl.dh_columns - 1) / gl.dh_columns)
                                          : Trc / kBlockR * ((H + kBlockC - 1) / kBlockC)) * ranges;
    info->dhidden_grid = gl.dh_grid;
    info->dw_blocks = c.group_done ? gl.dw.blocks() : 0;
    info->dw_grid = gl.dw_grid;
    info->gather_grid = c.Tr + g.zero_blocks + g.pieces;
    info->largest_grid = std::max<int64_t>({info->gather_grid, (int64_t)gl.dh_grid, (int64_t)gl.dw_grid, (int64_t)l.grid,
                                            (int64_t)c.Tr + 1});
    info->logits_columns = l.columns;
    info->logits_chained = l.chain;
    info->dhidden_columns = gl.dh_columns;
    info->dw_columns = gl.dw_columns;
    info->together = gl.together;
    info->numbered_by_gather = g.numbers;
    info->transposed_apart = g.transposes_apart;
    info->in_stash = c.part != L.part;
    return ALST_OK;
}

int alst_shift_labels(const int32_t* labels, int32_t* shift_labels, int64_t N, int32_t ignore_index,
                      void* stream) {
    if (!labels || !shift_labels) return ALST_ERR_NULL;
    if (N < 1 || N > (int64_t)1 << 30) return ALST_ERR_SHAPE;
    int blocks = (int)((N + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(shift_labels_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, labels,
                       shift_labels, N, ignore_index);
    return hipGetLastError() == hipSuccess ? ALST_OK : ALST_ERR_HIP;
}

}  // extern "C"
