// Encoder-side compaction of CIVIC, the paper's own (learned, soft) route to a compact sequence:
//   civic_anchor_aggregate  Eq. 8: Z_0 = softmax(Q_A K_0^T / tau) X_0 with K_0 = Norm(LN(X_0)), Q_A = Norm(LN(A)),
//                           softmax over the dense tokens
//   civic_kv_compress       Eq. 9: K_c = Rbar^T K, V_c = Rbar^T V with the column-normalised assignment matrix
// (the attention over the compressed keys, softmax(Q K_c^T / sqrt(d)) V_c, is civic_cross_attn in attn.hip).
//
// Both are dense contractions and run on the bf16 MFMA pipe.  Eq. 9 has a kernel of its own (compress_kernel); the
// products of Eq. 8 go through one kernel, C = alpha * A B^T, whose B operand may be stored either way round: like A, with the
// contraction index contiguous (the products Q_A X_0^T behind the logits), or with the contraction index as the row index, which is
// how X_0 lies in Z_0 = W_A X_0; it is read where it is (transposing LDS reads), no transposed copy is made.  A is always
// contraction-contiguous and zero-padded to a multiple of 64 in that direction (W_A is written that way), so the GEMM has no tail
// there; row and column tails are clamped loads and masked stores.  (Eq. 9 for rows that are not whole 16-byte pieces goes through
// the GEMM as well, with transposed, padded copies of R and X.)
//   - 128 x 128 output tile per 256-thread workgroup, 64 x 64 per wavefront (2 x 2 blocks of
//     v_mfma_f32_32x32x16_bf16, fp32 accumulators), 64 contraction elements per LDS tile.
//   - A and B tiles go from global memory straight into an LDS ring (global_load_lds_dwordx4), 16-byte chunks
//     XOR-swizzled by the row so that operand reads fall on distinct banks; explicit vmcnt waits, fence-free barriers;
//     the fragments of the next k-step are read while the MFMAs of the current one run, in a hand-written order.
//   - Two ring depths: two stages and two workgroups per compute unit for grids that fill the chip (the kernel is then
//     bound by the L2 -> LDS traffic of its tiles, 64 FLOP per byte; a deeper ring at one workgroup per unit was
//     slower, 46.6 against 35.3 us on the 1365 x 4096 x 1152 logits), four stages for grids that leave units without a
//     second workgroup anyway, where the latency of a tile is what a workgroup waits for.
// The softmax of Eq. 8 has two routes.  A logit never exceeds inv_tau in size, so up to 60 the first product's epilogue writes
// exponentials in bf16 and their partial row sums, and the second product divides by those: no logits in memory, no softmax
// launch.  A colder softmax needs its row's maximum: logits in fp32 to scratch, a row kernel into bf16 weights, the second product.
#include <algorithm>
#include <cmath>

#include "civic_internal.h"

namespace civic {

typedef __bf16 enc_bf16x8 __attribute__((ext_vector_type(8)));
typedef float enc_f32x16 __attribute__((ext_vector_type(16)));
typedef float enc_f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char enc_lds_char;

constexpr int kGemmBM = 128, kGemmBN = 128, kGemmBK = 64;
constexpr int kGemmThreads = 256;
constexpr int kGemmTileBytes = kGemmBM * kGemmBK * 2;         // one operand tile: 16 KB

constexpr int kGroupItems = 64;    // items of one grouped launch (longer lists go out in several)

// Items of different row counts packed along the row axis (the ragged Eq. 9 call): item i owns rows [row[i], row[i + 1]).
struct Group {
    int32_t row[kGroupItems + 1];
    uint8_t longest_first[kGroupItems];   // the items by falling row count
};

struct GemmArgs {
    const __bf16* a; const __bf16* b; void* c;
    int64_t lda, ldb, ldc;             // elements between rows of A [m x k], of B as stored, of C [m x n]
    int64_t sa, sb, sc;                // elements between batch items (0 = shared)
    int32_t m, n, k;                   // k a multiple of 64 (A is zero-padded up to it)
    int32_t kb_rows;                   // B stored [k x n]: the rows that exist (<= k); rows beyond re-read the last one
    float alpha;
    // output tiles: counts per matrix, tiles of all matrices of the launch, n-tiles per panel (filled in by launch_gemm)
    int32_t tiles_m, tiles_n, total_tiles, panel;
    // logits and weights of Eq. 8 (kOutLogits, kOutExp): (mean, 1 / ||x - mean||) of the batch item's B rows, `col_pitch`
    // entries per item, and the sum of every A row (both arrays readable up to whole tiles)
    const float2* col_stats; int64_t col_pitch; const float* row_sum;
    // partial row sums [batch][parts][part_pitch], written by kOutExp (parts = 2 * its tiles_n), read by kOutRowNorm
    float* row_part; int32_t parts; int64_t part_pitch;
    float* row_inv;                    // kOutRowNorm: one over the sum of every A row, written when not null, [batch x m]
    // kOutRowNorm: workgroups behind the tiles' that make the token weights, each `sum_chunks` times 64 columns of a batch item (0: none)
    float* col_sum; int32_t sum_groups, sum_chunks;
};

template <int LDS_IMM>
__device__ __forceinline__ void enc_dma16(const void* base, uint32_t byte_off, uint32_t lds_addr)
{
    // 16 bytes per lane from base + byte_off (scalar base, per-lane offset) into LDS at lds_addr + LDS_IMM + lane * 16.  (The compiler
    // counts no wait states into an asm statement: the load may read m0 one state after the scalar write; `base` is enc_uniform's.)
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_addr), "v"(byte_off), "s"(base), "n"(LDS_IMM) : "memory", "scc");
}

// The same pointer in scalar registers, written by a scalar instruction, so that a load inside an asm statement may read it at once:
// from a vector instruction's write five wait states would have to lie in between, which the compiler does not count there.
__device__ __forceinline__ const char* enc_uniform(const void* p)
{
    const uint64_t bits = reinterpret_cast<uint64_t>(p);
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(bits >> 32)));
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(bits)));
    uint64_t copy;
    asm("s_mov_b64 %0, %1" : "=s"(copy) : "s"((static_cast<uint64_t>(hi) << 32) | lo));
    return reinterpret_cast<const char*>(copy);
}

// physical chunk = logical chunk ^ swz(row): rows 0..31 of a 128-byte-pitch tile, same logical chunk -> 32 banks groups
__device__ __forceinline__ int enc_swz(int row) { return (((row >> 1) & 1) << 2) | ((row >> 2) & 3); }
// the same for a 256-byte pitch (16 chunks per row): a tile stored with the contraction index as its rows
__device__ __forceinline__ int enc_swz16(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }

typedef __bf16 enc_bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 enc_bf16x4 __attribute__((ext_vector_type(4)));
typedef short enc_s16x4 __attribute__((ext_vector_type(4)));
typedef short enc_s16x8 __attribute__((ext_vector_type(8)));

// What leaves the kernel for a product value P(i, j) = sum_k A(i, k) B(j, k):
//   kOutBf16     alpha * P as bf16
//   kOutLogits   alpha * inv_j * (P - mean_j * sum_i) as fp32: the logit of Eq. 8 when B holds the dense tokens as they are
//                and sum_i is the sum of A row i (Norm(LN(x)) = (x - mean) * inv, so no normalised copy of X_0 is made)
//   kOutExp      2^(that logit * log2 e - kExpShift) as bf16, zero for columns n .. ldc - 1: softmax weights without their
//                row's factor; and the sum of what every wavefront wrote of a row (its 64 columns), as rounded
//   kOutRowNorm  P over the sum of A row i as bf16, from those partial sums: the row factor of weights written by kOutExp.
//                (Summing the A fragments under the MFMAs instead, 8 packed dot products a k-step, made the product of
//                1365 x 4096 weights with 4096 x 1152 tokens 47.8 us instead of 40.)
enum GemmOut { kOutBf16, kOutLogits, kOutExp, kOutRowNorm };
// |logit| <= inv_tau up to the rounding of Q_A, so with inv_tau <= 60 (86.6 binades) a weight lies in [2^-103, 2^72]: every row's
// weights are normal fp32 and bf16 numbers without knowing the row's maximum, and so are their sums.  (Their products with X_0
// are, but for tokens beyond 2^40 or rows without a weight above 2^-40, which the second product looks for.)
// The fraction of the shift puts the weights of a warm softmax, all near one another, high in their binade (2^0.7 of it), where
// bf16 is finest against the weight and the upper tail still does not spill into the next one.  Normalised weights lie around
// 1 / n_tokens instead, wherever in its binade that is; 300 tokens happen to be the best place, so the error of Z_0 is compared
// there (1152 wide, 100 anchors, inv_tau = 4, against 64 bits): 2.21e-3 normalised, 2.28e-3 with 15.5, 2.20e-3 with 15.3.
constexpr float kExpShift = 15.3f, kMaxDirectInvTau = 60.0f;
// One over a row's sum beyond which its product with the tokens is not left to fp32's range (the row's largest weights are below
// 2^-40 then; never at inv_tau <= 17, and above only for an anchor that every token points away from).
constexpr float kMaxRowFactor = 1.0995116e12f;

// Sum over the eight lanes 8 apart: x + x of lane ^ 8, ^ 16, ^ 32, one after the other (a sum does not depend on whose comes first).
__device__ __forceinline__ float over_row_slots(float v)
{
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xF, 0xF, false));   // row_ror:8
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}
// Token weights by workgroups of the second product's launch, on units that its tiles leave idle: column j's sum over the rows i of
// w(i, j) / sum_i, for `sum_chunks` times 64 columns.  The rows' factors first, from the partial sums as the tiles take them; then the
// columns, in the order of col_sum_kernel (128 row slots, of which a thread has every 32nd here): the same bits as from that kernel.
// (2 x 4096 tokens, 1365 anchors, 1152 wide: the product alone 33.5 us on 198 units and a launch of 6.8 behind it; together 37.4, since
// each of 44 groups reads the partial sums of all rows of its item and their weights past the tiles.)
constexpr int kSumGroupRows = 24 * 1024;                      // (a multiple of 4) rows whose factors are kept in LDS
constexpr int kSumGroupParts = 16, kSumGroupCols = 64;
constexpr size_t kSumGroupBytes = sizeof(float) * (kSumGroupRows + kSumGroupParts * kSumGroupCols);
__device__ __forceinline__ void col_sum_group(const GemmArgs& g, uint32_t group, char* smem)
{
    constexpr int kVirtual = kSumGroupParts, kCols = kSumGroupCols, kSlots = 128, kMine = 4;
    float* const inv = reinterpret_cast<float*>(smem);
    float* const part = inv + kSumGroupRows;                  // [kVirtual][kCols]
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid >> 6;
    const int32_t chunks = (g.kb_rows + kCols - 1) / kCols, per_item = (chunks + g.sum_chunks - 1) / g.sum_chunks;
    const int64_t b = group / static_cast<uint32_t>(per_item);
    const int32_t first = static_cast<int32_t>(group - b * per_item) * g.sum_chunks, last = min(first + g.sum_chunks, chunks);
    for (int r = 4 * tid; r < g.m; r += 4 * kGemmThreads) {   // (rows up to whole tiles are there: m <= part_pitch, a multiple of 128)
        const enc_f32x4* const src = reinterpret_cast<const enc_f32x4*>(g.row_part + b * g.parts * g.part_pitch + r);
        enc_f32x4 t[2] = {enc_f32x4{0.f, 0.f, 0.f, 0.f}, enc_f32x4{0.f, 0.f, 0.f, 0.f}};
        const int64_t pitch = g.part_pitch / 4;
        constexpr int kAhead = 16;                            // pairs of parts in flight
        for (int x0 = 0; x0 < g.parts; x0 += 2 * kAhead) {    // (an even number of parts; past the last the last pair again, not added)
            enc_f32x4 v[2 * kAhead];
#pragma unroll
            for (int x = 0; x < 2 * kAhead; ++x) v[x] = src[min(x0 + x, g.parts - 2 + (x & 1)) * pitch];
#pragma unroll
            for (int x = 0; x < 2 * kAhead; ++x)
                if (x0 + x < g.parts) t[x & 1] += v[x];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) inv[r + e] = 1.0f / (t[0][e] + t[1][e]);
    }
    __syncthreads();
    const int c = tid & 7, slot = tid >> 3;
    for (int32_t chunk = first; chunk < last; ++chunk) {
        const char* const src = reinterpret_cast<const char*>(g.a + b * g.sa + chunk * kCols + 8 * c);
        float acc[kMine][8];
#pragma unroll
        for (int u = 0; u < kMine; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[u][e] = 0.f;
        auto add = [&](int u, const u32x4& v, float f) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[u][2 * e] = fmaf(__uint_as_float(v[e] << 16), f, acc[u][2 * e]);
                acc[u][2 * e + 1] = fmaf(__uint_as_float(v[e] & 0xFFFF0000u), f, acc[u][2 * e + 1]);
            }
        };
        constexpr int kDeep = 6;                              // rows of a slot in flight: 24 loads of 16 bytes a lane
        int r0 = slot;
        for (; r0 - slot + kDeep * kSlots <= g.m; r0 += kDeep * kSlots) {
            u32x4 v[kDeep][kMine];
#pragma unroll
            for (int x = 0; x < kDeep; ++x)
#pragma unroll
                for (int u = 0; u < kMine; ++u) v[x][u] = *reinterpret_cast<const u32x4*>(src + (r0 + x * kSlots + 32 * u) * g.lda * 2);
#pragma unroll
            for (int x = 0; x < kDeep; ++x)
#pragma unroll
                for (int u = 0; u < kMine; ++u) add(u, v[x][u], inv[r0 + x * kSlots + 32 * u]);
        }
        if (r0 - slot < g.m) {                                // fewer are left: a row past the last re-reads it and is not added
            u32x4 v[kDeep][kMine];
#pragma unroll
            for (int x = 0; x < kDeep; ++x)
#pragma unroll
                for (int u = 0; u < kMine; ++u) v[x][u] = *reinterpret_cast<const u32x4*>(src + min(r0 + x * kSlots + 32 * u, g.m - 1) * g.lda * 2);
#pragma unroll
            for (int x = 0; x < kDeep; ++x)
#pragma unroll
                for (int u = 0; u < kMine; ++u)
                    if (r0 + x * kSlots + 32 * u < g.m) add(u, v[x][u], inv[r0 + x * kSlots + 32 * u]);
        }
        __syncthreads();                                      // the sums of the chunk before have been read
#pragma unroll
        for (int u = 0; u < kMine; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                acc[u][e] = over_row_slots(acc[u][e]);
                if (lane < 8) part[(w + 4 * u) * kCols + 8 * lane + e] = acc[u][e];
            }
        __syncthreads();
        const int j = chunk * kCols + tid;
        if (tid < kCols && j < g.kb_rows) {
            float t = 0.f;
#pragma unroll
            for (int x = 0; x < kVirtual; ++x) t += part[x * kCols + tid];
            g.col_sum[b * g.kb_rows + j] = t;
        }
    }
}

// C = A B^T in the form OUT.  A is stored [m x k] (contraction index contiguous).  B_KROWS = false: B stored [n x k], the same
// way.  B_KROWS = true: B stored [k x n], contraction index as the row index - the layout of X_0 in Z_0 = W_A X_0 and of
// K, V in Eq. 9; its tiles (64 contraction rows x 128 columns, 256-byte pitch) are read with the transposing LDS read,
// which hands a lane one column and 4 consecutive contraction rows, so no transposed copy is ever made.
// The product is taken transposed (B fragments as the MFMA's first operand), so a lane owns one row of C and four
// consecutive columns per register quad: row factors are lane scalars and bf16 results leave through LDS in whole 16-byte
// row segments.
// STAGES: tiles in the LDS ring, all but one in flight ahead of the one consumed: 2 (two workgroups per compute unit)
// when the grid fills the chip, 4 (one workgroup per unit) when it does not and a tile's latency is what is waited for.
template <int OUT, bool B_KROWS, int STAGES>
__global__ __launch_bounds__(kGemmThreads, STAGES == 2 ? 2 : 1) void gemm_kernel(GemmArgs g)
{
    extern __shared__ __attribute__((aligned(16))) char gemm_lds[];
    enc_lds_char* const lds = (enc_lds_char*)gemm_lds;       // the A stages, then the B stages
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid >> 6;
    const int col = lane & 31, half = lane >> 5;
    const int wm = w >> 1, wn = w & 1;                        // the wavefront's 64 x 64 quadrant
    // Workgroup -> output tile.  The hardware hands consecutive workgroups to the eight XCDs in turn, each with an L2
    // of its own, so workgroup p takes tile (p mod 8) * (workgroups / 8) + p / 8: every XCD owns a contiguous run of
    // tiles, and the tiles of a matrix are numbered panel by panel (a panel = `panel` tile columns, all tile rows), so
    // that run is a compact block whose A row slabs and B column slabs are shared inside one L2 as the workgroups
    // advance along the contraction together.  With the plain (x, y) numbering every XCD touches every slab and the
    // kernel runs at the speed of the memory behind the L2s.
    constexpr bool kSums = OUT == kOutRowNorm && STAGES == 4;
    const uint32_t tile_blocks = gridDim.x - static_cast<uint32_t>(kSums ? g.sum_groups : 0);
    if constexpr (kSums) {
        static_assert(kSumGroupBytes <= 2 * STAGES * kGemmTileBytes, "the factors and partial sums of the token weights fit the ring");
        if (blockIdx.x >= tile_blocks) { col_sum_group(g, blockIdx.x - tile_blocks, gemm_lds); return; }
    }
    const uint32_t per_xcd = tile_blocks >> 3;
    const uint32_t tile = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if (tile >= static_cast<uint32_t>(g.total_tiles)) return;        // (the grid is padded to a multiple of 8)
    const uint32_t per_mat = static_cast<uint32_t>(g.tiles_m) * g.tiles_n;
    const uint32_t zi = tile / per_mat;
    const uint32_t rr = tile - zi * per_mat;
    const uint32_t pn = rr / (static_cast<uint32_t>(g.panel) * g.tiles_m);
    const uint32_t base_n = pn * g.panel;
    const uint32_t pw = min(static_cast<uint32_t>(g.panel), static_cast<uint32_t>(g.tiles_n) - base_n);
    const uint32_t within = rr - pn * g.panel * g.tiles_m;
    const int m0 = static_cast<int>(within / pw) * kGemmBM;
    const int n0 = static_cast<int>(base_n + within % pw) * kGemmBN;
    const int64_t bz = zi;
    const __bf16* const b_mat = g.b;
    const int32_t k_len = g.k, kb_rows = g.kb_rows;
    const int64_t lda = g.lda, a_first = bz * g.sa, b_first = bz * g.sb;

    // global -> LDS: instruction j of wavefront w fills slots [(4 w + j) * 64, +64) of a tile; slot -> (row, physical chunk)
    const char* a_base = reinterpret_cast<const char*>(g.a + a_first + static_cast<int64_t>(m0) * lda);
    const char* b_base = B_KROWS ? reinterpret_cast<const char*>(b_mat + b_first + n0)
                                 : reinterpret_cast<const char*>(b_mat + b_first + static_cast<int64_t>(n0) * g.ldb);
    const int last_tile = k_len / kGemmBK - 1;
    uint32_t a_off[4], b_off[4], b_off_tail[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int slot = (w * 4 + j) * kWave + lane;
        const int row = slot >> 3;
        const int c = (slot & 7) ^ enc_swz(row);
        a_off[j] = static_cast<uint32_t>(min(row, g.m - 1 - m0)) * static_cast<uint32_t>(lda * 2) + c * 16;
        if constexpr (B_KROWS) {
            const int krow = slot >> 4;                       // contraction row inside the tile
            const int lc = (slot & 15) ^ enc_swz16(krow);     // logical chunk: columns n0 + 8 lc .. + 7
            const int cc = min(lc, (g.n - n0) / 8 - 1);       // (n is a multiple of 8; chunks past it re-read a valid one)
            b_off[j] = static_cast<uint32_t>(krow) * static_cast<uint32_t>(g.ldb * 2) + cc * 16;
            b_off_tail[j] = static_cast<uint32_t>(min(last_tile * kGemmBK + krow, kb_rows - 1) - last_tile * kGemmBK) *
                                static_cast<uint32_t>(g.ldb * 2) + cc * 16;
        } else {
            b_off[j] = static_cast<uint32_t>(min(row, g.n - 1 - n0)) * static_cast<uint32_t>(g.ldb * 2) + c * 16;
            b_off_tail[j] = b_off[j];
        }
    }
    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds)) + w * 4 * kWave * 16);
    // Load j of the eight of a tile into the stage's A and B areas.  (Tiles past the last: the last one again.)
    auto tile_a = [&](int kt) __attribute__((always_inline)) { return enc_uniform(a_base + static_cast<int64_t>(min(kt, last_tile)) * kGemmBK * 2); };
    auto tile_b = [&](int kt) __attribute__((always_inline)) {
        return enc_uniform(b_base + static_cast<int64_t>(min(kt, last_tile)) * kGemmBK * 2 * (B_KROWS ? g.ldb : 1));
    };
    auto issue = [&](const char* ab, const char* bb, bool tail, int j, auto stage_c) __attribute__((always_inline)) {
        constexpr int at = decltype(stage_c)::value * kGemmTileBytes, bt = (STAGES + decltype(stage_c)::value) * kGemmTileBytes;
        const uint32_t off = j < 4 ? a_off[j & 3] : tail ? b_off_tail[j & 3] : b_off[j & 3];
        if (j == 0) enc_dma16<at + 0 * 1024>(ab, off, lds_wave);
        else if (j == 1) enc_dma16<at + 1 * 1024>(ab, off, lds_wave);
        else if (j == 2) enc_dma16<at + 2 * 1024>(ab, off, lds_wave);
        else if (j == 3) enc_dma16<at + 3 * 1024>(ab, off, lds_wave);
        else if (j == 4) enc_dma16<bt + 0 * 1024>(bb, off, lds_wave);
        else if (j == 5) enc_dma16<bt + 1 * 1024>(bb, off, lds_wave);
        else if (j == 6) enc_dma16<bt + 2 * 1024>(bb, off, lds_wave);
        else enc_dma16<bt + 3 * 1024>(bb, off, lds_wave);
    };

    // A reads: row (quadrant row 32 i + col), logical chunk 2 s + half; the swizzle depends on row bits 1..3 only, so the
    // second row block is the first plus a constant.  B the same when it is stored like A; when it is stored with the
    // contraction index as rows, two transposing reads per fragment: a block of 16 lanes fetches a patch of 4
    // contraction rows (8 half + 4 hi + 0..3 of the 16-row step) x 16 columns and every lane receives one column of it.
    enc_lds_char* a_addr[4];
    enc_lds_char* b_addr[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        a_addr[s] = lds + (wm * 64 + col) * 128 + (((2 * s + half) ^ enc_swz(col)) << 4);
        if constexpr (B_KROWS) {
            const int hi = s & 1, j = s >> 1;                 // (the four registers are the (hi, j) combinations)
            const int l16 = lane & 15, g16 = (lane >> 4) & 1;
            const int krow = 8 * half + 4 * hi + (l16 >> 2);
            const int el = wn * 64 + 32 * j + 16 * g16 + 4 * (l16 & 3);
            b_addr[s] = lds + STAGES * kGemmTileBytes + krow * 256 + (((el >> 3) ^ enc_swz16(krow)) << 4) + (el & 7) * 2;
        } else {
            b_addr[s] = lds + STAGES * kGemmTileBytes + (wn * 64 + col) * 128 + (((2 * s + half) ^ enc_swz(col)) << 4);
        }
        asm volatile("" : "+v"(a_addr[s]), "+v"(b_addr[s]));
    }

    enc_f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    const int n_tiles = k_len / kGemmBK;
    auto issue_all = [&](int kt, auto stage_c) __attribute__((always_inline)) {
        const char* const ab = tile_a(kt);
        const char* const bb = tile_b(kt);
#pragma unroll
        for (int j = 0; j < 8; ++j) issue(ab, bb, B_KROWS && kt >= last_tile, j, stage_c);
    };
    issue_all(0, std::integral_constant<int, 0>{});
    if constexpr (STAGES == 4) {
        issue_all(1, std::integral_constant<int, 1>{});
        issue_all(2, std::integral_constant<int, 2>{});
    }
    auto step = [&](int kt, auto stage_c) __attribute__((always_inline)) {
        constexpr int st = decltype(stage_c)::value;
        constexpr std::integral_constant<int, (st + STAGES - 1) % STAGES> fill{};
        // Loads retire in order, 8 per tile and wavefront: tile kt has landed once at most those of the two tiles after it are
        // outstanding (four stages; loads past the last tile are issued all the same, so that the count holds to the end) or none.
        if constexpr (STAGES == 4) __builtin_amdgcn_s_waitcnt(0x4F70);       // vmcnt(16): the count's bits 5:4 sit in bits 15:14
        else __builtin_amdgcn_s_waitcnt(0x0F70);                              // vmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();                         // landed for every wavefront; the stage of tile kt - 1 is free
        asm volatile("" ::: "memory");
        const char* const ab = tile_a(kt + STAGES - 1);
        const char* const bb = tile_b(kt + STAGES - 1);
        const bool tail = B_KROWS && kt + STAGES - 1 >= last_tile;
        if (STAGES == 2 && kt + 1 < n_tiles) issue_all(kt + 1, fill);
        // operand fragments of k-step s + 1 are read while the MFMAs of step s run (in the order written)
        auto read_a = [&](int s, int i) __attribute__((always_inline)) {
            return *reinterpret_cast<const __attribute__((address_space(3))) enc_bf16x8*>(a_addr[s] + st * kGemmTileBytes + i * 32 * 128);
        };
        auto read_b = [&](int s, int j) __attribute__((always_inline)) {
            if constexpr (B_KROWS) {
                const enc_s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) enc_s16x4*)(b_addr[2 * j] + st * kGemmTileBytes + s * 16 * 256));
                const enc_s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) enc_s16x4*)(b_addr[2 * j + 1] + st * kGemmTileBytes + s * 16 * 256));
                const enc_s16x8 v8 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                return __builtin_bit_cast(enc_bf16x8, v8);
            } else {
                return *reinterpret_cast<const __attribute__((address_space(3))) enc_bf16x8*>(b_addr[s] + st * kGemmTileBytes + j * 32 * 128);
            }
        };
        enc_bf16x8 af[2][2], bf[2][2];
        af[0][0] = read_a(0, 0); af[0][1] = read_a(0, 1); bf[0][0] = read_b(0, 0); bf[0][1] = read_b(0, 1);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int cur = s & 1, nxt = cur ^ 1;
            // Four stages, one wavefront to a SIMD: behind each product one operand read of the next 16 contraction elements and one
            // load of a tile to come, where the wavefront would only wait for the product.  (All of them ahead of the four products of
            // a k-step: 41 us on 1365 x 4096 weights times 4096 x 1152 tokens, two items; one by one, spread over the step, 31.  A tile's
            // first operands read in the step before it as well: no gain.  Eight wavefronts, each half with half of a tile's
            // contraction: 38.)  Two stages, two workgroups to a unit: the other one's products run meanwhile.
            if (STAGES == 2 && s + 1 < 4) { af[nxt][0] = read_a(s + 1, 0); af[nxt][1] = read_a(s + 1, 1); bf[nxt][0] = read_b(s + 1, 0); bf[nxt][1] = read_b(s + 1, 1); }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = k >> 1, j = k & 1;
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[cur][j], af[cur][i], acc[i][j], 0, 0, 0);
                if constexpr (STAGES == 4) {
                    if (s + 1 < 4) {
                        if (k < 2) af[nxt][k] = read_a(s + 1, k);
                        else bf[nxt][k - 2] = read_b(s + 1, k - 2);
                    }
                    if (k & 1) issue(ab, bb, tail, 2 * s + (k >> 1), fill);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    for (int kt = 0; kt < n_tiles; kt += STAGES) {
        step(kt, std::integral_constant<int, 0>{});
        if (kt + 1 < n_tiles) step(kt + 1, std::integral_constant<int, 1>{});
        if constexpr (STAGES == 4) {
            if (kt + 2 < n_tiles) step(kt + 2, std::integral_constant<int, 2>{});
            if (kt + 3 < n_tiles) step(kt + 3, std::integral_constant<int, 3>{});
        }
    }

    __builtin_amdgcn_s_waitcnt(0x0F70);                       // (the loads past the last tile, before the ring is written to)

    // register r of block (i, j): row 32 i + col, column 32 j + 8 (r / 4) + 4 half + r % 4 of the wavefront's quadrant
    const int row_q = m0 + wm * 64, col_q = n0 + wn * 64;
    constexpr bool kFp32 = OUT == kOutLogits;
    char* c_base = static_cast<char*>(g.c) + (bz * g.sc) * (kFp32 ? 4 : 2);
    constexpr int kPitch = 64 + 8;                            // elements per staged row (padded against bank conflicts)
    constexpr int kStageBytes = 4 * 64 * kPitch * 2;
    if constexpr (OUT == kOutRowNorm) {                       // the tile's row sums: 2 threads a row, every other part each
        float* const sums = reinterpret_cast<float*>(gemm_lds + kStageBytes);
        const int r = tid & (kGemmBM - 1), first = tid / kGemmBM;
        const float* src = g.row_part + bz * g.parts * g.part_pitch + m0 + r;
        float t = 0.f;
#pragma unroll 16
        for (int part = first; part < g.parts; part += 2) t += src[part * g.part_pitch];
        __syncthreads();                                      // every wavefront has read its last tile: the ring is free
        sums[tid] = t;
        __syncthreads();
    }
    float scale[2], part_sum[2] = {0.f, 0.f}, odd[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = row_q + 32 * i + col;
        scale[i] = g.alpha;
        if constexpr (OUT == kOutRowNorm) {
            const float* const sums = reinterpret_cast<const float*>(gemm_lds + kStageBytes);
            scale[i] = 1.0f / (sums[row - m0] + sums[kGemmBM + row - m0]);
            if (g.row_inv != nullptr && n0 == 0 && wn == 0 && half == 0 && row < g.m) g.row_inv[bz * g.m + row] = scale[i];
        } else if constexpr (OUT == kOutLogits || OUT == kOutExp) {
            scale[i] = g.row_sum[row];
        }
    }
    auto value = [&](int i, int j, int rq, float4 mean, float4 inv, float (&v)[4]) __attribute__((always_inline)) {
        const float mm[4] = {mean.x, mean.y, mean.z, mean.w}, ii[4] = {inv.x, inv.y, inv.z, inv.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float p = acc[i][j][4 * rq + e];
            if constexpr (OUT == kOutLogits) v[e] = ii[e] * fmaf(-mm[e], scale[i], p);
            else if constexpr (OUT == kOutExp) v[e] = __builtin_amdgcn_exp2f(fmaf(ii[e], fmaf(-mm[e], scale[i], p), -kExpShift));
            else v[e] = p * scale[i];
        }
    };
    // (mean, factor) of the lane's four columns of register quad rq; the factor carries alpha (and log2 e)
    auto columns = [&](int j, int rq, float4& mean, float4& inv) __attribute__((always_inline)) {
        if constexpr (OUT == kOutLogits || OUT == kOutExp) {
            const float4* st = reinterpret_cast<const float4*>(g.col_stats + bz * g.col_pitch + col_q + 32 * j + 8 * rq + 4 * half);
            const float4 a = st[0], b = st[1];
            const float f = OUT == kOutExp ? g.alpha * 1.4426950408889634f : g.alpha;
            mean = make_float4(a.x, a.z, b.x, b.z);
            inv = make_float4(a.y * f, a.w * f, b.y * f, b.w * f);
        }
    };
    if constexpr (kFp32) {                                    // (rows of ldc floats, ldc a multiple of 64: whole quads)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                float4 mean, inv;
                columns(j, rq, mean, inv);
                const int cc = col_q + 32 * j + 8 * rq + 4 * half;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int row = row_q + 32 * i + col;
                    float v[4];
                    value(i, j, rq, mean, inv, v);
                    if (row < g.m && cc < g.ldc)
                        *reinterpret_cast<float4*>(reinterpret_cast<float*>(c_base) + static_cast<int64_t>(row) * g.ldc + cc) = make_float4(v[0], v[1], v[2], v[3]);
                }
            }
        return;
    }
    // rows of whole 16-byte pieces (launch-uniform); weights have them by their padding, which is written as zeros
    const int64_t n_out = OUT == kOutExp ? g.ldc : g.n;
    const bool whole = g.ldc % 8 == 0 && n_out % 8 == 0;
    __bf16* const stage = reinterpret_cast<__bf16*>(gemm_lds) + w * 64 * kPitch;
    if (whole && OUT != kOutRowNorm) __syncthreads();         // every wavefront has read its last tile: the ring is free
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
            float4 mean = make_float4(0.f, 0.f, 0.f, 0.f), inv = mean;
            columns(j, rq, mean, inv);
            const int cc = col_q + 32 * j + 8 * rq + 4 * half;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                float v[4];
                value(i, j, rq, mean, inv, v);
                if constexpr (OUT == kOutRowNorm) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) odd[i] = fmaf(v[e], 0.f, odd[i]);
                }
                enc_bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    o[e] = static_cast<__bf16>(OUT == kOutExp && cc + e >= g.n ? 0.f : v[e]);
                    if constexpr (OUT == kOutExp) part_sum[i] += static_cast<float>(o[e]);
                }
                if (whole) {
                    *reinterpret_cast<enc_bf16x4*>(&stage[(32 * i + col) * kPitch + 32 * j + 8 * rq + 4 * half]) = o;
                } else {
                    const int row = row_q + 32 * i + col;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (row < g.m && cc + e < g.n) reinterpret_cast<__bf16*>(c_base)[static_cast<int64_t>(row) * g.ldc + cc + e] = o[e];
                }
            }
        }
    if constexpr (OUT == kOutRowNorm) {
        // Weights without their row's factor reach from 2^-103 to 2^72, so a product with tokens beyond 2^40 may have overflowed, and
        // one of a row of small weights with small tokens vanished.  Such a wavefront makes its results again with the factor
        // applied to the weight first, one fp32 multiply-add each, four columns at a time.
        // (A row whose factor is NaN has met a NaN among the tokens: that is its result.)
        bool again = false;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            again |= row_q + 32 * i + col < g.m && (scale[i] > kMaxRowFactor || (odd[i] != 0.f && scale[i] == scale[i]));
        if (__builtin_expect(__any(again), 0)) {
#pragma unroll 1
            for (int c4 = 4 * half; c4 < 64; c4 += 8)
#pragma unroll 1
                for (int row = row_q + col, i = 0; i < 2; row += 32, ++i) {
                    if (row >= g.m || col_q + c4 >= g.n) continue;
                    const float factor = i == 0 ? scale[0] : scale[1];
                    const __bf16* wgt = g.a + a_first + row * lda;
                    const __bf16* x = b_mat + b_first + col_q + c4;
                    float t[4] = {0.f, 0.f, 0.f, 0.f};
                    for (int k = 0; k < kb_rows; ++k) {
                        const enc_bf16x4 xk = *reinterpret_cast<const enc_bf16x4*>(x + k * g.ldb);
                        const float wk = static_cast<float>(wgt[k]) * factor;
#pragma unroll
                        for (int e = 0; e < 4; ++e) t[e] = fmaf(wk, static_cast<float>(xk[e]), t[e]);
                    }
                    enc_bf16x4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = static_cast<__bf16>(t[e]);
                    *reinterpret_cast<enc_bf16x4*>(reinterpret_cast<__bf16*>(c_base) + static_cast<int64_t>(row) * g.ldc + col_q + c4) = o;
                }
            return;
        }
    }
    if constexpr (OUT == kOutExp) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const float t = part_sum[i] + __shfl_xor(part_sum[i], 32, kWave);
            if (half == 0)                                    // (rows up to whole tiles: the array is that tall)
                g.row_part[(bz * g.parts + (n0 / kGemmBN) * 2 + wn) * g.part_pitch + row_q + 32 * i + col] = t;
        }
    }
    if (!whole) return;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        const int r = it * 8 + (lane >> 3), c8 = (lane & 7) * 8;
        const int row = row_q + r, cc = col_q + c8;
        if (row < g.m && cc < n_out)
            *reinterpret_cast<u32x4*>(reinterpret_cast<__bf16*>(c_base) + static_cast<int64_t>(row) * g.ldc + cc) =
                *reinterpret_cast<const u32x4*>(&stage[r * kPitch + c8]);
    }
}

template <int OUT, bool B_KROWS, int STAGES>
static int launch_gemm_variant(const GemmArgs& g, unsigned blocks, hipStream_t s)
{
    if (g.sum_groups != 0 && !(OUT == kOutRowNorm && STAGES == 4)) return CIVIC_ERR_UNSUPPORTED;   // (sums_fit asks for none there)
    const dim3 grid(blocks + static_cast<unsigned>(g.sum_groups));
    constexpr size_t lds = 2 * STAGES * kGemmTileBytes;
    static_assert(lds >= 4 * 64 * (64 + 8) * 2 + 1024, "the ring holds the staged output tile and the row sums");
    static std::atomic<uint64_t> allowed{0};
    const int rc = allow_dynamic_lds(reinterpret_cast<const void*>(gemm_kernel<OUT, B_KROWS, STAGES>), lds, &allowed);
    if (rc != CIVIC_OK) return rc;
    civic::launch((gemm_kernel<OUT, B_KROWS, STAGES>), grid, dim3(kGemmThreads), lds, s, g);
    return check_launch();
}

// Output tiles from which on a launch has a second workgroup for every unit, or nearly, and takes the ring of two stages.
constexpr int64_t kTwoStageTiles = 2 * 256;

// Whether the token weights go into the second product's launch, and their share of it: its tiles run one to a unit and leave units
// idle (in their only generation or in the second), and those are through with the columns well before the tiles are with their rows:
// a unit reads 60 KB of partial row sums and 50 of weights a microsecond by itself, a tile takes 0.52 for 64 tokens, beside each other
// both take longer, and a launch of their own costs 4 before its work.  (us, so and as a launch of their own, and what is compared: 2 x 4096
// tokens, 1365 anchors, 1152 wide 78.7, 80.4, 21 <= 27; 1 x 8192, 2730, 768 112.8, 119.5, 41 <= 47; 4 x 6144, 1536, 1152 215.4, 215.6,
// 36 <= 37; but 1 x 8192, 2730, 1152 143.8, 139.8, 49 > 47; 3 x 12000, 1333, 768 232, 221, 67 > 65; 1 x 8086, 2695, 1280 160, 149, 56 > 46;
// 2 x 6144, 3072, 1152 224, 217, 48 > 37.)
static bool sums_fit(GemmArgs* g, int64_t batch)
{
    const int64_t total = batch * ((g->m + kGemmBM - 1) / kGemmBM) * ((g->n + kGemmBN - 1) / kGemmBN);
    if (total >= kTwoStageTiles || g->m > kSumGroupRows) return false;   // (their LDS is that of four stages)
    const int64_t idle = (total <= 256 ? 256 : 512) - (total + 7) / 8 * 8, chunks = (g->kb_rows + 63) / 64;
    if (idle <= 0) return false;
    int64_t each = std::max<int64_t>((chunks * batch + idle - 1) / idle, 1);
    while ((chunks + each - 1) / each * batch > idle && each < chunks) ++each;
    const int64_t groups = (chunks + each - 1) / each * batch, rounds = (groups + idle - 1) / idle;
    const double rows = 1.5 + g->m * static_cast<double>(g->parts) * 4.0 / 60e3, columns = 1.0 + g->m * 128.0 / 50e3;
    if (static_cast<double>(rounds) * (rows + static_cast<double>(each) * columns) > 0.31 * (g->k / 64) + 7.0) return false;
    g->sum_chunks = static_cast<int32_t>(each);
    g->sum_groups = static_cast<int32_t>(groups);
    return true;
}

// `batch` batch items.  B_KROWS: B is stored [k x n].
template <int OUT, bool B_KROWS>
static int launch_gemm(const GemmArgs& g_in, int batch, hipStream_t s)
{
    GemmArgs g = g_in;
    g.tiles_n = (g.n + kGemmBN - 1) / kGemmBN;
    g.tiles_m = (g.m + kGemmBM - 1) / kGemmBM;
    const int64_t total = static_cast<int64_t>(batch) * g.tiles_m * g.tiles_n;
    if (total > (int64_t{1} << 30)) return CIVIC_ERR_UNSUPPORTED;
    g.total_tiles = static_cast<int32_t>(total);
    const unsigned grid = static_cast<unsigned>((total + 7) / 8 * 8);
    // panel width: about the square root of an XCD's share of the tiles, so that its block is as tall as it is wide
    int panel = 1;
    while (static_cast<int64_t>(panel + 1) * (panel + 1) <= (total + 7) / 8) ++panel;
    g.panel = panel < g.tiles_n ? panel : g.tiles_n;
    // a grid that leaves compute units without a second workgroup takes the deeper ring
    return total < kTwoStageTiles ? launch_gemm_variant<OUT, B_KROWS, 4>(g, grid, s) : launch_gemm_variant<OUT, B_KROWS, 2>(g, grid, s);
}

// ------------------------------------------------------------------------------------------ row kernels
// Row statistics of Eq. 8, one wavefront per row; rows [0, rows_a) are anchors, the rest dense tokens (items of `tokens`
// rows, whose statistics are `stat_pitch` entries apart).
//   anchor  qa[row, :] = Norm(LN(a)) = (a - mean) / ||a - mean|| as bf16, and the sum of that row as rounded
//   token   (mean, 1 / ||x - mean||) only: the GEMM reads the token's row as it is and applies both to its product
// A row without variance normalises to zero (factor 0).  CH > 0: rows of up to 64 * 8 * CH elements; the row is read once with
// 16-byte loads and stays in registers for the centred second pass.  CH == 0: longer rows, three passes over a row that stays
// in L1/L2 after the first.  (2 x 4096 + 1365 rows of 1152: 9.7 us when the normalised tokens were written out as well, 18.9 MB.)
template <int CH>
__global__ __launch_bounds__(256) void row_stats_kernel(const __bf16* __restrict__ anchors, int64_t rows_a, const __bf16* __restrict__ x0,
                                                        int64_t rows_x, int32_t tokens, int64_t stat_pitch, int32_t dim,
                                                        __bf16* __restrict__ qa, float* __restrict__ qa_sum, float2* __restrict__ stats)
{
    const int lane = threadIdx.x & (kWave - 1);
    int64_t row = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (row >= rows_a + rows_x) return;
    const bool is_anchor = row < rows_a;
    if (!is_anchor) row -= rows_a;
    const u32x4* src = reinterpret_cast<const u32x4*>((is_anchor ? anchors : x0) + row * dim);
    const int n_chunks = dim >> 3;                            // (dim is a multiple of 64)
    constexpr int kHeld = CH > 0 ? CH : 1;
    const int n_rounds = CH > 0 ? CH : (n_chunks + kWave - 1) / kWave;
    u32x4 v[kHeld];
    auto chunk = [&](int c, bool again) {
        const int k = c * kWave + lane;
        if (CH > 0 && again) return v[CH > 0 ? c : 0];
        return k < n_chunks ? src[k] : u32x4{0u, 0u, 0u, 0u};
    };
    if constexpr (CH > 0) {                                   // all loads before the first use
#pragma unroll
        for (int c = 0; c < CH; ++c) v[c] = chunk(c, false);
    }
    float sum = 0.f;
#pragma unroll kHeld
    for (int c = 0; c < n_rounds; ++c) {
        const u32x4 x = chunk(c, true);
#pragma unroll
        for (int e = 0; e < 4; ++e) sum += __uint_as_float(x[e] << 16) + __uint_as_float(x[e] & 0xFFFF0000u);
    }
    const float mean = wave_sum(sum) / static_cast<float>(dim);
    float n2 = 0.f;
#pragma unroll kHeld
    for (int c = 0; c < n_rounds; ++c)
        if (c * kWave + lane < n_chunks) {
            const u32x4 x = chunk(c, true);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float lo = __uint_as_float(x[e] << 16) - mean, hi = __uint_as_float(x[e] & 0xFFFF0000u) - mean;
                n2 = fmaf(lo, lo, n2); n2 = fmaf(hi, hi, n2);
            }
        }
    n2 = wave_sum(n2);
    const float inv = n2 > 0.f ? 1.0f / sqrtf(n2) : 0.f;
    if (!is_anchor) {
        if (lane == 0) stats[row / tokens * stat_pitch + row % tokens] = make_float2(mean, inv);
        return;
    }
    u32x4* dst = reinterpret_cast<u32x4*>(qa + row * dim);
    float q_sum = 0.f;
#pragma unroll kHeld
    for (int c = 0; c < n_rounds; ++c)
        if (c * kWave + lane < n_chunks) {
            const u32x4 x = chunk(c, true);
            u32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const enc_bf16x2 t = {static_cast<__bf16>((__uint_as_float(x[e] << 16) - mean) * inv),
                                      static_cast<__bf16>((__uint_as_float(x[e] & 0xFFFF0000u) - mean) * inv)};
                const uint32_t word = __builtin_bit_cast(uint32_t, t);
                o[e] = word;
                q_sum += __uint_as_float(word << 16) + __uint_as_float(word & 0xFFFF0000u);
            }
            dst[c * kWave + lane] = o;
        }
    q_sum = wave_sum(q_sum);
    if (lane == 0) qa_sum[row] = q_sum;
}

// p[row, 0..cols) = softmax(s[row, 0..cols)) as bf16, p[row, cols..ld_p) = 0; one wavefront per row.  Rows of up to
// 64 * 4 * CH logits (ld_s a multiple of 4) stay in registers between the maximum, the exponentials and the store: one
// trip to memory; longer rows take the three-pass loop.
template <int CH>
__global__ __launch_bounds__(256) void row_softmax_kernel(const float* __restrict__ s, int64_t rows, int32_t cols, int64_t ld_s,
                                                          __bf16* __restrict__ p, int64_t ld_p)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t row = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const float* src = s + row * ld_s;
    __bf16* dst = p + row * ld_p;
    if constexpr (CH > 0) {
        float4 v[CH];
        float mx = -INFINITY;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int j = (c * kWave + lane) * 4;
            v[c] = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
            if (j < cols) v[c] = *reinterpret_cast<const float4*>(src + j);   // (ld_s is padded: the vector stays inside the row)
            if (j + 1 >= cols) v[c].y = -INFINITY;
            if (j + 2 >= cols) v[c].z = -INFINITY;
            if (j + 3 >= cols) v[c].w = -INFINITY;
            mx = fmaxf(mx, fmaxf(fmaxf(v[c].x, v[c].y), fmaxf(v[c].z, v[c].w)));
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, kWave));
        float sum = 0.f;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            v[c].x = __expf(v[c].x - mx); v[c].y = __expf(v[c].y - mx); v[c].z = __expf(v[c].z - mx); v[c].w = __expf(v[c].w - mx);
            sum += (v[c].x + v[c].y) + (v[c].z + v[c].w);
        }
        const float inv = 1.0f / wave_sum(sum);
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int j = (c * kWave + lane) * 4;
            if (j < ld_p) {                                                   // (ld_p is a multiple of 64)
                const __bf16 o[4] = {static_cast<__bf16>(v[c].x * inv), static_cast<__bf16>(v[c].y * inv),
                                     static_cast<__bf16>(v[c].z * inv), static_cast<__bf16>(v[c].w * inv)};
                u32x2 packed;
                packed.x = static_cast<uint32_t>(__builtin_bit_cast(uint16_t, o[0])) | (static_cast<uint32_t>(__builtin_bit_cast(uint16_t, o[1])) << 16);
                packed.y = static_cast<uint32_t>(__builtin_bit_cast(uint16_t, o[2])) | (static_cast<uint32_t>(__builtin_bit_cast(uint16_t, o[3])) << 16);
                *reinterpret_cast<u32x2*>(dst + j) = packed;
            }
        }
    } else {
        float mx = -INFINITY;
        for (int j = lane; j < cols; j += kWave) mx = fmaxf(mx, src[j]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, kWave));
        float sum = 0.f;
        for (int j = lane; j < cols; j += kWave) sum += __expf(src[j] - mx);
        const float inv = 1.0f / wave_sum(sum);
        for (int j = lane; j < ld_p; j += kWave) dst[j] = static_cast<__bf16>(j < cols ? __expf(src[j] - mx) * inv : 0.f);
    }
}

// out[b, j] = sum over rows of p[b, row, j] * row_scale[b, row] (1 where row_scale is null): the weight a dense token receives
// from all anchors together.  One pass over the weights, so memory-bound: a workgroup owns 64 columns (one 128-byte line of
// every row) and its 1024 threads are 8 column chunks x 128 row slots, 16 bytes a load, four rows in flight per thread; the
// slots meet in a fixed order (shuffles, then LDS), so the sums are the same every time.  1365 x 4096 weights, two items: 313 us
// as one thread per column walking all rows (32 workgroups, one 2-byte load in flight each), 6.8 us so.
constexpr int kColSumThreads = 1024, kColSumCols = 64;
__global__ __launch_bounds__(kColSumThreads) void col_sum_kernel(const __bf16* __restrict__ p, int32_t rows, int32_t cols, int64_t ld_p,
                                                                 int64_t batch_stride, const float* __restrict__ row_scale,
                                                                 float* __restrict__ out)
{
    constexpr int kSlots = kColSumThreads / 8, kWaves = kColSumThreads / kWave, kRows = 4;
    __shared__ float part[kWaves][kColSumCols];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
    const int c = threadIdx.x & 7, slot = threadIdx.x >> 3;
    const int j0 = blockIdx.x * kColSumCols;                  // (ld_p is a multiple of 64: whole chunks, zeros past cols)
    const int64_t b = blockIdx.y;
    const char* src = reinterpret_cast<const char*>(p + b * batch_stride + j0 + 8 * c);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int r = slot; r < rows; r += kRows * kSlots) {
        u32x4 v[kRows];
        float f[kRows];
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            v[u] = u32x4{0u, 0u, 0u, 0u};
            f[u] = 1.0f;
            if (r + u * kSlots < rows) {
                v[u] = *reinterpret_cast<const u32x4*>(src + (r + u * kSlots) * ld_p * 2);
                if (row_scale != nullptr) f[u] = row_scale[b * rows + r + u * kSlots];
            }
        }
#pragma unroll
        for (int u = 0; u < kRows; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[2 * e] = fmaf(__uint_as_float(v[u][e] << 16), f[u], acc[2 * e]);
                acc[2 * e + 1] = fmaf(__uint_as_float(v[u][e] & 0xFFFF0000u), f[u], acc[2 * e + 1]);
            }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {                             // the wavefront's 8 row slots
#pragma unroll
        for (int off = 8; off < kWave; off <<= 1) acc[e] += __shfl_xor(acc[e], off, kWave);
        if (lane < 8) part[wv][8 * lane + e] = acc[e];
    }
    __syncthreads();
    const int j = threadIdx.x;
    if (j < kColSumCols && j0 + j < cols) {
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) t += part[w][j];
        out[b * cols + j0 + j] = t;
    }
}

constexpr int kColParts = 32;             // partial column sums per column (col_part_sum_kernel below)

// out[b, c, r] = in[b, r, c] * inv[c] for r < rows, 0 for rows <= r < ld_out; 32 x 32 tiles through LDS.  inv[c] is one
// over column c's sum, taken here from its kColParts partial sums part[p, c] (0 for a column that sums to zero); with
// part null the values are copied unscaled.
template <typename TIN>
__device__ __forceinline__ void transpose_pad_block(const TIN* __restrict__ in, int32_t rows, int32_t cols, int64_t ld_in,
                                                    int64_t in_batch, const float* __restrict__ part,
                                                    __bf16* __restrict__ out, int64_t ld_out, int64_t out_batch, int64_t b)
{
    __shared__ float tile[32][33];
    __shared__ float inv_s[32];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
    const int r0 = blockIdx.x * 32, c0 = blockIdx.y * 32;
    if (part != nullptr && threadIdx.x < 32) {
        const int c = c0 + threadIdx.x;
        float t = 0.f;
        if (c < cols) {
#pragma unroll
            for (int p = 0; p < kColParts; ++p) t += part[static_cast<int64_t>(p) * cols + c];
        }
        inv_s[threadIdx.x] = t != 0.f ? 1.0f / t : 0.f;      // (read after the barrier below)
    }
    for (int k = ty; k < 32; k += 8) {
        const int r = r0 + k, c = c0 + tx;
        float v = 0.f;
        if (r < rows && c < cols) {
            if constexpr (std::is_same<TIN, float>::value) v = in[b * in_batch + static_cast<int64_t>(r) * ld_in + c];
            else v = static_cast<float>(in[b * in_batch + static_cast<int64_t>(r) * ld_in + c]);
        }
        tile[k][tx] = v;
    }
    __syncthreads();
    for (int k = ty; k < 32; k += 8) {
        const int c = c0 + k, r = r0 + tx;
        if (c < cols && r < ld_out) {
            const float sc = part ? inv_s[k] : 1.0f;
            out[b * out_batch + static_cast<int64_t>(c) * ld_out + r] = static_cast<__bf16>(tile[tx][k] * sc);
        }
    }
}

template <typename TIN>
__global__ __launch_bounds__(256) void transpose_pad_kernel(const TIN* __restrict__ in, int32_t rows, int32_t cols, int64_t ld_in,
                                                            int64_t in_batch, const float* __restrict__ part,
                                                            __bf16* __restrict__ out, int64_t ld_out, int64_t out_batch)
{
    transpose_pad_block<TIN>(in, rows, cols, ld_in, in_batch, part, out, ld_out, out_batch, blockIdx.z);
}

// Column sums of r [rows, cols], first step: block (x, y) adds the rows 4 y .. 4 y + 3 of every 4 kColParts of 64 columns (a row of
// the four for each wavefront, coalesced 256-byte reads, four in flight, meeting in LDS) into part[y, c]; whoever divides by a column's
// sum adds its kColParts partial sums in order.
__device__ __forceinline__ void col_part_sum_block(const float* __restrict__ r, int32_t rows, int32_t cols, float* __restrict__ part)
{
    __shared__ float lds_part[4][kWave];
    constexpr int kAhead = 4, kStride = 4 * kColParts;
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
    const int c = blockIdx.x * kWave + lane;
    float acc = 0.f;
    if (c < cols)
        for (int64_t m = blockIdx.y * 4 + wv; m < rows; m += kAhead * kStride) {
            float v[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) v[u] = r[(m + u * kStride < rows ? m + u * kStride : m) * cols + c];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) acc = m + u * kStride < rows ? acc + v[u] : acc;
        }
    lds_part[wv][lane] = acc;
    __syncthreads();
    if (wv == 0 && c < cols)
        part[static_cast<int64_t>(blockIdx.y) * cols + c] = (lds_part[0][lane] + lds_part[1][lane]) + (lds_part[2][lane] + lds_part[3][lane]);
}

__global__ __launch_bounds__(256) void col_part_sum_kernel(const float* __restrict__ r, int32_t rows, int32_t cols, float* __restrict__ part)
{
    col_part_sum_block(r, rows, cols, part);
}

// The same for the items of a group (grid z): every item its own rows, its own kColParts x cols partial sums.
__global__ __launch_bounds__(256) void col_part_sum_grouped_kernel(const float* __restrict__ r, int32_t cols, float* __restrict__ part, Group grp)
{
    const int i = blockIdx.z;
    const int64_t r0 = grp.row[i];
    col_part_sum_block(r + r0 * cols, grp.row[i + 1] - grp.row[i], cols, part + static_cast<int64_t>(i) * kColParts * cols);
}

// ------------------------------------------------------------------------------------------ Eq. 9
// X_c = Rbar^T X for X = K and V, Rbar the columns of R over their sums, rounded to bf16, in two launches: partial column sums of R
// (col_part_sum_kernel), then the product, which takes R as it lies, divides by its columns' sums and rounds on the way into LDS: no
// transposed copy of Rbar in memory.  (Rounding R first and dividing the result instead needs no sums ahead of the product, but a
// column whose sum is far from the entries' size or that nearly cancels then needs a route of its own, and results change.)
//   - 128 x 128 outputs per workgroup of four wavefronts, a quadrant of 64 x 64 each, in steps of 64 contraction rows, two workgroups
//     to a unit; one sum per output over all rows in order, whatever the launch holds besides: items of a batch, packed or not, come
//     out the same bits
//   - R goes through registers one step ahead, into tiles [64 rows x 128 columns] like those of X, which go straight into LDS; both
//     operands are read with the transposing LDS read
//   - one barrier a step: a wavefront writes the next step's R, asks for the R after that and for the next X, and waits for X when
//     the step's products are done
// Both launches (us): eight items of 85 to 1365 rows, 256 x 1152 out 25.1; 4 x 2048 rows, 512 x 1024 out 32.3; 6 x 1024, 256 x 1152
// 19.2; 16 x 700, 128 x 768 19.8; 24 x 24, 512 x 1280 31.1; 1 x 85, 256 x 1152 11.8.  With a transposed copy of Rbar made between
// the two: 29.8, 35.0, 22.6, 24.4, 30.6, 19.3.  (The R of two steps in registers instead of one's: the same within 2 %, but 33.0 for
// 24 x 24.)
struct CompressArgs {
    const float* r;                       // [rows x m], shared by all items or packed like them
    const float* part;                    // [kColParts x m] partial column sums; PACKED: of every item, one after the other
    const __bf16* x[2];                   // K, V [rows x n]
    __bf16* out[2];                       // [items x m x n]
    int32_t m, n, tiles_m, tiles_n, slabs;
    int32_t n_rows;                       // of every item; PACKED: from grp
    Group grp;
};
constexpr int kCmpTile = 64 * 128 * 2;                        // bytes of one operand tile of 64 contraction rows

// QUADS: m a multiple of 4, so that rows of R are aligned to 16 bytes and made of whole quads of columns, and below 2^24, so that 64
// rows are below 2^32 bytes.
template <bool PACKED, bool QUADS>
__global__ __launch_bounds__(256, 2) void compress_kernel(CompressArgs g)
{
    constexpr int kStep = 64, kCmpStage = 2 * kCmpTile;
    extern __shared__ __attribute__((aligned(16))) char cmp_lds[];
    enc_lds_char* const lds = (enc_lds_char*)cmp_lds;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // the wavefront's quadrant
    const int col = lane & 31, half = lane >> 5, wm = w >> 1, wn = w & 1;
    // Column slabs (one tile column of an item and tensor, all its tile rows) go to the XCDs in turn, the longest items' first: an
    // XCD's L2 holds the slab of X for its tile rows, and no XCD works on alone.
    const uint32_t slot = blockIdx.x >> 3, per_item = static_cast<uint32_t>(g.tiles_n) * 2u;
    const uint32_t up = slot / static_cast<uint32_t>(g.tiles_m), slab = up * 8u + (blockIdx.x & 7u);
    if (slab >= static_cast<uint32_t>(g.slabs)) return;
    const uint32_t rank = slab / per_item, in_item = slab - rank * per_item, tensor = in_item / static_cast<uint32_t>(g.tiles_n);
    const int m0 = static_cast<int>(slot - up * g.tiles_m) * 128, n0 = static_cast<int>(in_item - tensor * g.tiles_n) * 128;
    int64_t item = rank, r_first = 0, x_first = rank * static_cast<int64_t>(g.n_rows);
    int32_t rows = g.n_rows;
    if constexpr (PACKED) {
        item = g.grp.longest_first[rank];
        r_first = x_first = g.grp.row[item];
        rows = g.grp.row[item + 1] - g.grp.row[item];
    }
    const float* const r_item = g.r + r_first * g.m;
    const __bf16* const x_item = (tensor ? g.x[1] : g.x[0]) + x_first * g.n;
    const int steps = (rows + kStep - 1) / kStep;

    // R: thread -> four columns of rows row_r, row_r + 8, ... of the step's 64
    const int col4 = (tid & 31) * 4, row_r = tid >> 5;
    // bytes of a row of R; elements where rows are not whole quads or 64 of them take more than 32 bits of bytes
    const uint32_t r_pitch = static_cast<uint32_t>(g.m) * (QUADS ? 4u : 1u), x_pitch = static_cast<uint32_t>(g.n) * 2u;
    const uint32_t r_col = static_cast<uint32_t>(QUADS ? min(col4, g.m - 4 - m0) : 0) * 4u;
    uint32_t r_off[8];                                        // from the step's first row
#pragma unroll
    for (int j = 0; j < 8; ++j) r_off[j] = static_cast<uint32_t>(row_r + 8 * j) * r_pitch + r_col;
    enc_f32x4 rv[8];                                          // the next step's R, or on its way there
    // row j of the thread's eight of a step whose first row is at `base` and whose last row is at `last_row`
    auto fetch_row = [&](const char* base, uint32_t last_row, int j) __attribute__((always_inline)) {
        // (global by type: a pointer put together from scalars is a generic one, whose loads count as LDS accesses as well)
        const auto p = (const __attribute__((address_space(1))) char*)base + static_cast<uint64_t>(min(r_off[j], last_row)) * (QUADS ? 1u : 4u);
        if constexpr (QUADS) {
            rv[j] = *(const __attribute__((address_space(1))) enc_f32x4*)p;
        } else {
            const int last = g.m - 1 - m0;
            const auto f = (const __attribute__((address_space(1))) float*)p;
            rv[j] = enc_f32x4{f[min(col4, last)], f[min(col4 + 1, last)], f[min(col4 + 2, last)], f[min(col4 + 3, last)]};
        }
    };
    // (steps, rows and columns past the end re-read the last one)
    auto step_base = [&](int step) __attribute__((always_inline)) { return enc_uniform(r_item + m0 + static_cast<int64_t>(min(step, steps - 1)) * kStep * g.m); };
    auto step_last = [&](int step) __attribute__((always_inline)) {
        return static_cast<uint32_t>(min(rows - 1 - min(step, steps - 1) * kStep, kStep - 1)) * r_pitch + r_col;
    };
    auto fetch_r = [&](int step) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 8; ++j) fetch_row(step_base(step), step_last(step), j);
    };
    // rows of `step` past the item become zeros (only the last step has any)
    auto clear_tail = [&](int step) __attribute__((always_inline)) {
        if (__builtin_expect((step + 1) * kStep > rows, 0)) {
            const int live = rows - (step * kStep + row_r);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const bool in = 8 * j < live;
                rv[j].x = in ? rv[j].x : 0.f; rv[j].y = in ? rv[j].y : 0.f;
                rv[j].z = in ? rv[j].z : 0.f; rv[j].w = in ? rv[j].w : 0.f;
            }
        }
    };
    // Row j of the thread's eight, over its columns' sums and rounded, into the stage of its step's parity.
    float4 inv;
    u32x2 word;
    auto round_r = [&](int j) __attribute__((always_inline)) {
        const enc_f32x4 v = rv[j];
        const enc_bf16x2 lo = {static_cast<__bf16>(v.x * inv.x), static_cast<__bf16>(v.y * inv.y)};
        const enc_bf16x2 hi = {static_cast<__bf16>(v.z * inv.z), static_cast<__bf16>(v.w * inv.w)};
        word = u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
    };
    auto write_r = [&](int j, auto stage_c) __attribute__((always_inline)) {
        const int kr = row_r + 8 * j;
        *reinterpret_cast<__attribute__((address_space(3))) u32x2*>(
            lds + decltype(stage_c)::value * kCmpStage + kr * 256 + (((col4 >> 3) ^ enc_swz16(kr)) << 4) + (col4 & 4) * 2) = word;
    };
    // X: instruction j of wavefront w fills slots [(4 w + j) * 64, +64) of the tile
    uint32_t x_off[4], x_col[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int s = (w * 4 + j) * kWave + lane, kr = s >> 4;
        const int lc = (s & 15) ^ enc_swz16(kr);              // logical chunk: columns n0 + 8 lc .. + 7
        x_col[j] = min(lc, (g.n - n0) / 8 - 1) * 16;          // (n is a multiple of 8; chunks past it re-read a valid one)
        x_off[j] = kr * x_pitch + x_col[j];
    }
    const uint32_t lds_x = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds)) + kCmpTile + w * 4 * kWave * 16);
    auto x_base = [&](int step) __attribute__((always_inline)) { return enc_uniform(reinterpret_cast<const char*>(x_item + n0) + static_cast<int64_t>(min(step, steps - 1)) * kStep * g.n * 2); };
    auto x_last = [&](int step) __attribute__((always_inline)) { return static_cast<uint32_t>(rows - 1 - min(step, steps - 1) * kStep) * x_pitch; };
    auto issue_x = [&](const char* base, uint32_t last_row, int j, int st) __attribute__((always_inline)) {
        const uint32_t off = min(x_off[j], last_row + x_col[j]);              // (rows past the item re-read its last)
        const uint32_t dst = lds_x + st * kCmpStage;
        if (j == 0) enc_dma16<0 * 1024>(base, off, dst);
        else if (j == 1) enc_dma16<1 * 1024>(base, off, dst);
        else if (j == 2) enc_dma16<2 * 1024>(base, off, dst);
        else enc_dma16<3 * 1024>(base, off, dst);
    };
    // operand reads of a 16-row step: 4 contraction rows x 16 columns a block of 16 lanes, a lane receives one column
    enc_lds_char* a_addr[4];
    enc_lds_char* b_addr[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int hi = s & 1, j = s >> 1, l16 = lane & 15, g16 = (lane >> 4) & 1;
        const int kr = 8 * half + 4 * hi + (l16 >> 2), el = 32 * j + 16 * g16 + 4 * (l16 & 3);
        const int ea = wm * 64 + el, eb = wn * 64 + el;
        a_addr[s] = lds + kr * 256 + (((ea >> 3) ^ enc_swz16(kr)) << 4) + (ea & 7) * 2;
        b_addr[s] = lds + kCmpTile + kr * 256 + (((eb >> 3) ^ enc_swz16(kr)) << 4) + (eb & 7) * 2;
        asm volatile("" : "+v"(a_addr[s]), "+v"(b_addr[s]));
    }
    enc_f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // X of the next step has landed (its loads are older than the last eight, of R) and so have all LDS accesses, of every wavefront
    auto landed = [&]() __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0070 | (QUADS ? 8 : 0)); // vmcnt, lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // A step: sixteen products, and behind each of them a little of everything else, so that one wavefront's vector instructions run
    // under the other's product.  R and X past the last step are fetched all the same, the last rows again, and R written as zeros: a
    // branch around loads has the compiler move registers of loads under way, and wait for them.
    auto step = [&](int kt, auto stage_c) __attribute__((always_inline)) {
        constexpr int st = decltype(stage_c)::value;
        constexpr std::integral_constant<int, st ^ 1> other{};
        clear_tail(kt + 1);
        const char* const xb = x_base(kt + 1);
        const uint32_t xl = x_last(kt + 1);
        const char* const rb = step_base(kt + 2);
        const uint32_t rl = step_last(kt + 2);
        auto read = [&](enc_lds_char* const (&addr)[4], int s, int j) __attribute__((always_inline)) {
            const enc_s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) enc_s16x4*)(addr[2 * j] + st * kCmpStage + s * 16 * 256));
            const enc_s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) enc_s16x4*)(addr[2 * j + 1] + st * kCmpStage + s * 16 * 256));
            const enc_s16x8 v8 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            return __builtin_bit_cast(enc_bf16x8, v8);
        };
        enc_bf16x8 af[2][2], bf[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i) { af[0][i] = read(a_addr, 0, i); bf[0][i] = read(b_addr, 0, i); }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int cur = s & 1, nxt = cur ^ 1;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = k >> 1, j = k & 1;
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[cur][j], af[cur][i], acc[i][j], 0, 0, 0);
                if (s + 1 < 4) {                              // the next 16 rows' operands
                    if (k < 2) af[nxt][k] = read(a_addr, s + 1, k);
                    else bf[nxt][k - 2] = read(b_addr, s + 1, k - 2);
                }
                if (s == 0) issue_x(xb, xl, k, st ^ 1);       // the next step's X
                const int row = 2 * s + (k >> 1);             // the next step's R, then the row to take its registers
                if ((k & 1) == 0) {
                    round_r(row);
                } else {
                    write_r(row, other);
                    if (s > 0) fetch_row(rb, rl, row - 2);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        fetch_row(rb, rl, 6);
        fetch_row(rb, rl, 7);
        landed();
    };
    auto start = [&](auto stage_c) __attribute__((always_inline)) {
        constexpr int st = decltype(stage_c)::value;
        float p[kColParts];
        if (tid < 128) {
            const float* const sums = g.part + (PACKED ? item * kColParts * g.m : 0) + min(m0 + tid, g.m - 1);
#pragma unroll
            for (int i = 0; i < kColParts; ++i) p[i] = sums[static_cast<int64_t>(i) * g.m];
        }
        fetch_r(0);
#pragma unroll
        for (int j = 0; j < 4; ++j) issue_x(x_base(0), x_last(0), j, st);
        float* const inv_s = reinterpret_cast<float*>(cmp_lds + (st ^ 1) * kCmpStage);   // (written to from the first step on, behind another barrier)
        if (tid < 128) {
            float t = 0.f;
#pragma unroll
            for (int i = 0; i < kColParts; ++i) t += p[i];
            inv_s[tid] = t != 0.f ? 1.0f / t : 0.f;           // (a column that sums to zero weighs nothing)
        }
        __syncthreads();
        inv = *reinterpret_cast<const float4*>(inv_s + col4);
        clear_tail(0);
#pragma unroll
        for (int j = 0; j < 8; ++j) { round_r(j); write_r(j, stage_c); }
        fetch_r(1);
        landed();
    };
    // Steps in pairs, stage 1 and stage 0, with a single one in front where their number is odd.  (A loop that can end between the
    // two leaves the compiler in doubt about which loads of R are under way, and the first of the two waits for all.)
    constexpr std::integral_constant<int, 0> stage0{};
    constexpr std::integral_constant<int, 1> stage1{};
    int kt = steps & 1;
    if (kt) {
        start(stage0);
        step(0, stage0);
    } else {
        start(stage1);
    }
    for (; kt < steps; kt += 2) {
        step(kt, stage1);
        step(kt + 1, stage0);
    }
    __builtin_amdgcn_s_waitcnt(0x0070);                       // (R past the end)
    __syncthreads();                                          // the ring is free

    // Register r of block (i, j): row 32 i + col, column 32 j + 8 (r / 4) + 4 half + r % 4 of the quadrant; through LDS into whole
    // 16-byte pieces of rows.
    constexpr int kPitch = 64 + 8;
    __bf16* const stage = reinterpret_cast<__bf16*>(cmp_lds) + w * 64 * kPitch;
    __bf16* const out = (tensor ? g.out[1] : g.out[0]) + item * g.m * g.n;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                enc_bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = static_cast<__bf16>(acc[i][j][4 * rq + e]);
                *reinterpret_cast<enc_bf16x4*>(&stage[(32 * i + col) * kPitch + 32 * j + 8 * rq + 4 * half]) = o;
            }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        const int r = it * 8 + (lane >> 3), c8 = (lane & 7) * 8;
        const int row = m0 + wm * 64 + r, cc = n0 + wn * 64 + c8;
        if (row < g.m && cc < g.n)
            *reinterpret_cast<u32x4*>(out + static_cast<int64_t>(row) * g.n + cc) = *reinterpret_cast<const u32x4*>(&stage[r * kPitch + c8]);
    }
}

// Eq. 9 of `items` items whose partial column sums are there; rows of whole 16-byte pieces in X (n a multiple of 8).
template <bool PACKED, bool QUADS>
static int launch_compress_variant(const CompressArgs& g, hipStream_t s)
{
    constexpr size_t lds = 2 * 2 * kCmpTile;
    static_assert(lds >= 4 * 64 * (64 + 8) * 2, "the ring holds the staged output");
    civic::launch((compress_kernel<PACKED, QUADS>), dim3(static_cast<unsigned>((g.slabs + 7) / 8 * 8 * g.tiles_m)), dim3(256), lds, s, g);
    return check_launch();
}

// (packed: the items' rows are in g.grp)
static int launch_compress(const CompressArgs& g_in, int64_t items, bool packed, hipStream_t s)
{
    CompressArgs g = g_in;
    g.tiles_m = (g.m + 127) / 128;
    g.tiles_n = (g.n + 127) / 128;
    const int64_t slabs = items * 2 * g.tiles_n;
    if (slabs * g.tiles_m > (int64_t{1} << 30)) return CIVIC_ERR_UNSUPPORTED;
    g.slabs = static_cast<int32_t>(slabs);
    const bool quads = g.m % 4 == 0 && g.m < (1 << 24);
    if (packed) return quads ? launch_compress_variant<true, true>(g, s) : launch_compress_variant<true, false>(g, s);
    return quads ? launch_compress_variant<false, true>(g, s) : launch_compress_variant<false, false>(g, s);
}

static int64_t pad64(int64_t x) { return (x + 63) / 64 * 64; }
static size_t align256(size_t x) { return (x + 255) / 256 * 256; }

struct AggPlan {                         // byte offsets into the workspace of civic_anchor_aggregate
    int64_t t_pad, t_tile;              // tokens rounded up to 64 (contraction tiles) and to 128 (whole output tiles)
    int64_t m_tile;                     // anchors rounded up to 128
    size_t qa, qa_sum, stats, row_part, row_inv, s, p, total;
};

static void agg_plan(int32_t batch, int32_t n_tokens, int32_t n_anchors, int32_t dim, AggPlan* p)
{
    p->t_pad = pad64(n_tokens);
    p->t_tile = (static_cast<int64_t>(n_tokens) + kGemmBN - 1) / kGemmBN * kGemmBN;
    p->m_tile = (static_cast<int64_t>(n_anchors) + kGemmBM - 1) / kGemmBM * kGemmBM;
    size_t off = 0;
    p->qa = off; off += align256(static_cast<size_t>(n_anchors) * dim * 2);
    p->qa_sum = off; off += align256(static_cast<size_t>(p->m_tile) * 4);
    p->stats = off; off += align256(static_cast<size_t>(batch) * p->t_tile * 8);
    p->row_part = off; off += align256(static_cast<size_t>(batch) * (p->t_tile / kGemmBN * 2) * p->m_tile * 4);
    p->row_inv = off; off += align256(static_cast<size_t>(batch) * n_anchors * 4);
    p->s = off;  off += align256(static_cast<size_t>(batch) * n_anchors * p->t_pad * 4);
    p->p = off;  off += align256(static_cast<size_t>(batch) * n_anchors * p->t_pad * 2);
    p->total = off;
}

struct CompressPlan {                    // byte offsets into the workspace of civic_kv_compress
    int64_t m_pad;
    size_t part, rt, xt, total;          // (rt and xt are written for widths of no whole 16-byte pieces only)
};

static void compress_plan(int32_t batch, int32_t n_rows, int32_t n_mem, int32_t width, CompressPlan* p)
{
    p->m_pad = pad64(n_rows);
    size_t off = 0;
    p->part = off; off += align256(static_cast<size_t>(n_mem) * 4 * kColParts);
    p->rt = off;  off += align256(static_cast<size_t>(n_mem) * p->m_pad * 2);
    // (a transposed copy of K, then V, only for widths whose rows are not whole 16-byte chunks)
    p->xt = off;  off += width % 8 ? align256(static_cast<size_t>(batch) * width * p->m_pad * 2) : 0;
    p->total = off;
}

static bool agg_sizes_ok(int32_t batch, int32_t n_tokens, int32_t n_anchors, int32_t dim)
{
    return batch >= 0 && n_tokens > 0 && n_anchors > 0 && dim > 0;
}

}  // namespace civic

extern "C" size_t civic_anchor_aggregate_workspace_bytes(int32_t batch, int32_t n_tokens, int32_t n_anchors, int32_t dim)
{
    if (!civic::agg_sizes_ok(batch, n_tokens, n_anchors, dim)) return 0;
    civic::AggPlan p;
    civic::agg_plan(batch, n_tokens, n_anchors, dim, &p);
    return p.total;
}

extern "C" int civic_anchor_aggregate(const void* x0, const void* anchors, int dtype, int32_t batch, int32_t n_tokens,
                                      int32_t n_anchors, int32_t dim, float inv_tau, void* z0, float* token_weight,
                                      void* workspace, size_t workspace_bytes, void* stream)
{
    using namespace civic;
    const int esz = dtype_size(dtype);
    if (!esz || !agg_sizes_ok(batch, n_tokens, n_anchors, dim)) return CIVIC_ERR_INVALID_ARG;
    if (!(inv_tau >= 0.f) || std::isinf(inv_tau)) return CIVIC_ERR_INVALID_ARG;
    if (batch > 0 && (!x0 || !anchors || !z0)) return CIVIC_ERR_INVALID_ARG;
    if (!aligned16(x0) || !aligned16(anchors) || !aligned16(z0) || (reinterpret_cast<uintptr_t>(token_weight) & 3u)) return CIVIC_ERR_INVALID_ARG;
    if (dim % 64) return CIVIC_ERR_UNSUPPORTED;                          // the first contraction runs over dim in tiles of 64
    if (dtype != CIVIC_BF16) return CIVIC_ERR_UNSUPPORTED;               // z0 leaves the MFMA path as bf16
    if (batch > 65535 || static_cast<int64_t>(n_tokens) * dim * 2 >= (int64_t{1} << 32) ||
        static_cast<int64_t>(n_anchors) * pad64(n_tokens) * 2 >= (int64_t{1} << 32))
        return CIVIC_ERR_UNSUPPORTED;                                     // 32-bit row offsets inside one batch item
    AggPlan p;
    agg_plan(batch, n_tokens, n_anchors, dim, &p);
    if (!workspace || workspace_bytes < p.total || !aligned16(workspace)) return CIVIC_ERR_WORKSPACE;
    if (batch == 0) return CIVIC_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);
    __bf16* qa = reinterpret_cast<__bf16*>(ws + p.qa);
    float* qa_sum = reinterpret_cast<float*>(ws + p.qa_sum);
    float2* stats = reinterpret_cast<float2*>(ws + p.stats);
    float* row_part = reinterpret_cast<float*>(ws + p.row_part);
    float* row_inv = reinterpret_cast<float*>(ws + p.row_inv);
    __bf16* pw = reinterpret_cast<__bf16*>(ws + p.p);
    const int64_t rows_x = static_cast<int64_t>(batch) * n_tokens, rows_w = static_cast<int64_t>(batch) * n_anchors;

    // Q_A = Norm(LN(A)) and the statistics of X_0's rows: one launch over the rows of both
    {
        const dim3 grid(static_cast<unsigned>((n_anchors + rows_x + 3) / 4));
        const int chunks = (dim / 8 + kWave - 1) / kWave;                              // 16-byte pieces per lane
#define CIVIC_LN_CASE(N) civic::launch((row_stats_kernel<N>), grid, dim3(256), 0, s, static_cast<const __bf16*>(anchors), \
                                            static_cast<int64_t>(n_anchors), static_cast<const __bf16*>(x0), rows_x, n_tokens, p.t_tile, dim, qa, qa_sum, stats)
        if (chunks <= 1) CIVIC_LN_CASE(1);
        else if (chunks <= 2) CIVIC_LN_CASE(2);
        else if (chunks <= 3) CIVIC_LN_CASE(3);
        else if (chunks <= 4) CIVIC_LN_CASE(4);
        else if (chunks <= 8) CIVIC_LN_CASE(8);
        else CIVIC_LN_CASE(0);
#undef CIVIC_LN_CASE
    }
    int rc = check_launch();
    if (rc != CIVIC_OK) return rc;
    // Q_A times the dense tokens as they lie; the epilogue makes logits of the products
    GemmArgs g1;
    g1.kb_rows = 0;
    g1.a = qa; g1.b = static_cast<const __bf16*>(x0);
    g1.lda = dim; g1.ldb = dim; g1.ldc = p.t_pad;
    g1.sa = 0; g1.sb = static_cast<int64_t>(n_tokens) * dim; g1.sc = static_cast<int64_t>(n_anchors) * p.t_pad;
    g1.m = n_anchors; g1.n = n_tokens; g1.k = dim; g1.alpha = inv_tau;
    g1.col_stats = stats; g1.col_pitch = p.t_tile; g1.row_sum = qa_sum; g1.row_inv = nullptr;
    g1.col_sum = nullptr; g1.sum_groups = 0; g1.sum_chunks = 0;
    g1.row_part = row_part; g1.parts = static_cast<int32_t>(p.t_tile / kGemmBN * 2); g1.part_pitch = p.m_tile;
    // Z_0 = W_A X_0, X_0 read where it lies (tokens are its rows: the contraction index is the row index)
    GemmArgs g2;
    g2.a = pw; g2.b = static_cast<const __bf16*>(x0); g2.c = z0;
    g2.lda = p.t_pad; g2.ldb = dim; g2.ldc = dim;
    g2.sa = static_cast<int64_t>(n_anchors) * p.t_pad; g2.sb = static_cast<int64_t>(n_tokens) * dim; g2.sc = static_cast<int64_t>(n_anchors) * dim;
    g2.m = n_anchors; g2.n = dim; g2.k = static_cast<int32_t>(p.t_pad); g2.kb_rows = n_tokens; g2.alpha = 1.0f;
    g2.col_stats = nullptr; g2.col_pitch = 0; g2.row_sum = nullptr; g2.row_inv = nullptr;
    g2.col_sum = nullptr; g2.sum_groups = 0; g2.sum_chunks = 0;
    g2.row_part = row_part; g2.parts = g1.parts; g2.part_pitch = g1.part_pitch;
    auto token_weights = [&](const float* row_scale) {
        civic::launch(col_sum_kernel, dim3(static_cast<unsigned>((n_tokens + kColSumCols - 1) / kColSumCols), static_cast<unsigned>(batch)),
                      dim3(kColSumThreads), 0, s, pw, n_anchors, n_tokens, p.t_pad, static_cast<int64_t>(n_anchors) * p.t_pad, row_scale, token_weight);
        return check_launch();
    };
    // Small enough inverse temperatures: the first product leaves as exponentials (a logit never exceeds inv_tau), the second
    // divides by their row sums, and no logits are written.  2 x (1365 x 4096): fp32 logits out, a softmax over their rows and
    // bf16 weights back in were 44.7 + 44.7 + 22.4 MB more and a launch of 12.9 us.
    if (inv_tau <= kMaxDirectInvTau) {
        g1.c = pw;
        rc = launch_gemm<kOutExp, false>(g1, batch, s);
        if (rc != CIVIC_OK) return rc;
        const bool with_sums = token_weight && sums_fit(&g2, batch);
        g2.col_sum = with_sums ? token_weight : nullptr;
        g2.row_inv = token_weight && !with_sums ? row_inv : nullptr;
        rc = launch_gemm<kOutRowNorm, true>(g2, batch, s);
        if (rc != CIVIC_OK || !token_weight || with_sums) return rc;
        return token_weights(row_inv);
    }
    // Colder softmaxes need their row's maximum: logits in fp32, a softmax over their rows into bf16 weights (zero in the
    // padding), then the second product
    float* sl = reinterpret_cast<float*>(ws + p.s);
    g1.c = sl;
    rc = launch_gemm<kOutLogits, false>(g1, batch, s);
    if (rc != CIVIC_OK) return rc;
    {
        const dim3 grid(static_cast<unsigned>((rows_w + 3) / 4));
        const int chunks = static_cast<int>((p.t_pad / 4 + kWave - 1) / kWave);       // float4 per lane
#define CIVIC_SOFTMAX_CASE(N) civic::launch((row_softmax_kernel<N>), grid, dim3(256), 0, s, sl, rows_w, n_tokens, p.t_pad, pw, p.t_pad)
        if (chunks <= 4) CIVIC_SOFTMAX_CASE(4);
        else if (chunks <= 8) CIVIC_SOFTMAX_CASE(8);
        else if (chunks <= 16) CIVIC_SOFTMAX_CASE(16);
        else if (chunks <= 32) CIVIC_SOFTMAX_CASE(32);
        else CIVIC_SOFTMAX_CASE(0);
#undef CIVIC_SOFTMAX_CASE
    }
    rc = check_launch();
    if (rc == CIVIC_OK && token_weight) rc = token_weights(nullptr);
    if (rc != CIVIC_OK) return rc;
    return launch_gemm<kOutBf16, true>(g2, batch, s);
}

// For tests, on the host alone (no part of civic.h): workgroups that make the token weights inside the second product's launch, and the
// columns of each over 64 in *chunks; 0 where they are a launch of their own.
extern "C" int civic_aggregate_sum_groups(int32_t batch, int32_t n_tokens, int32_t n_anchors, int32_t dim, int32_t* chunks)
{
    using namespace civic;
    AggPlan p;
    agg_plan(batch, n_tokens, n_anchors, dim, &p);
    GemmArgs g = {};
    g.m = n_anchors; g.n = dim; g.k = static_cast<int32_t>(p.t_pad); g.kb_rows = n_tokens; g.parts = static_cast<int32_t>(p.t_tile / kGemmBN * 2);
    const bool with_sums = sums_fit(&g, batch);
    if (chunks) *chunks = with_sums ? g.sum_chunks : 0;
    return with_sums ? g.sum_groups : 0;
}

extern "C" size_t civic_kv_compress_workspace_bytes(int32_t batch, int32_t n_rows, int32_t n_mem, int32_t width)
{
    if (batch < 0 || n_rows <= 0 || n_mem <= 0 || width <= 0) return 0;
    civic::CompressPlan p;
    civic::compress_plan(batch, n_rows, n_mem, width, &p);
    return p.total;
}

extern "C" int civic_kv_compress(const void* k, const void* v, int dtype, const float* r, int32_t batch, int32_t n_rows,
                                 int32_t n_mem, int32_t width, void* k_c, void* v_c, void* workspace, size_t workspace_bytes,
                                 void* stream)
{
    using namespace civic;
    const int esz = dtype_size(dtype);
    if (!esz || batch < 0 || n_rows <= 0 || n_mem <= 0 || width <= 0) return CIVIC_ERR_INVALID_ARG;
    if (!r || (batch > 0 && (!k || !v || !k_c || !v_c))) return CIVIC_ERR_INVALID_ARG;
    if (!aligned16(k) || !aligned16(v) || !aligned16(k_c) || !aligned16(v_c) || !aligned16(r)) return CIVIC_ERR_INVALID_ARG;
    if (dtype != CIVIC_BF16) return CIVIC_ERR_UNSUPPORTED;
    if (batch > 65535 || pad64(n_rows) * static_cast<int64_t>(width) * 2 >= (int64_t{1} << 32) ||
        pad64(n_rows) * static_cast<int64_t>(n_mem) * 2 >= (int64_t{1} << 32))
        return CIVIC_ERR_UNSUPPORTED;
    CompressPlan p;
    compress_plan(batch, n_rows, n_mem, width, &p);
    if (!workspace || workspace_bytes < p.total || !aligned16(workspace)) return CIVIC_ERR_WORKSPACE;
    if (batch == 0) return CIVIC_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);
    float* part = reinterpret_cast<float*>(ws + p.part);
    civic::launch(col_part_sum_kernel, dim3(static_cast<unsigned>((n_mem + kWave - 1) / kWave), kColParts), dim3(256), 0, s, r, n_rows,
                       n_mem, part);
    int rc = check_launch();
    if (rc != CIVIC_OK) return rc;
    if (width % 8 == 0) {
        CompressArgs c;
        c.r = r; c.part = part; c.x[0] = static_cast<const __bf16*>(k); c.x[1] = static_cast<const __bf16*>(v);
        c.out[0] = static_cast<__bf16*>(k_c); c.out[1] = static_cast<__bf16*>(v_c);
        c.m = n_mem; c.n = width; c.n_rows = n_rows;
        return launch_compress(c, batch, false, s);
    }
    // rows that are not whole 16-byte pieces: transposed, padded copies of them and of Rbar
    __bf16* rt = reinterpret_cast<__bf16*>(ws + p.rt);
    __bf16* xt = reinterpret_cast<__bf16*>(ws + p.xt);
    // Rbar^T [n_mem x m_pad]: every column of R over its sum, transposed, zero beyond n_rows
    civic::launch((transpose_pad_kernel<float>), dim3(static_cast<unsigned>(p.m_pad / 32), static_cast<unsigned>((n_mem + 31) / 32), 1u),
                       dim3(256), 0, s, r, n_rows, n_mem, static_cast<int64_t>(n_mem), int64_t{0}, part, rt, p.m_pad, int64_t{0});
    rc = check_launch();
    if (rc != CIVIC_OK) return rc;
    GemmArgs g;
    g.col_stats = nullptr; g.col_pitch = 0; g.row_sum = nullptr; g.row_inv = nullptr; g.row_part = nullptr; g.parts = 0; g.part_pitch = 0; g.col_sum = nullptr; g.sum_groups = 0; g.sum_chunks = 0;
    g.a = rt; g.lda = p.m_pad; g.ldc = width;
    g.sa = 0; g.sc = static_cast<int64_t>(n_mem) * width;
    g.m = n_mem; g.n = width; g.k = static_cast<int32_t>(p.m_pad); g.alpha = 1.0f;
    const void* src[2] = {k, v};
    void* dst[2] = {k_c, v_c};
    for (int t = 0; t < 2; ++t) {
        // X^T [width x m_pad] per batch item, then X_c = Rbar^T (X^T)^T
        civic::launch((transpose_pad_kernel<__bf16>), dim3(static_cast<unsigned>(p.m_pad / 32), static_cast<unsigned>((width + 31) / 32),
                                                                static_cast<unsigned>(batch)),
                           dim3(256), 0, s, static_cast<const __bf16*>(src[t]), n_rows, width, static_cast<int64_t>(width),
                           static_cast<int64_t>(n_rows) * width, static_cast<const float*>(nullptr), xt, p.m_pad,
                           static_cast<int64_t>(width) * p.m_pad);
        rc = check_launch();
        if (rc != CIVIC_OK) return rc;
        g.b = xt; g.c = dst[t]; g.kb_rows = 0;
        g.ldb = p.m_pad; g.sb = static_cast<int64_t>(width) * p.m_pad;
        rc = launch_gemm<kOutBf16, false>(g, batch, s);
        if (rc != CIVIC_OK) return rc;
    }
    return CIVIC_OK;
}

// ---------------------------------------------------------------------------------------------- ragged batches
namespace civic {

// host [batch + 1], starting at 0, strictly increasing (every item has at least one row)
static bool offsets_ok(const int64_t* off, int32_t batch)
{
    if (!off || off[0] != 0) return false;
    for (int32_t b = 0; b < batch; ++b)
        if (off[b + 1] <= off[b] || off[b + 1] - off[b] > INT32_MAX) return false;
    return true;
}

}  // namespace civic

namespace civic {

// Bytes of the workspace of civic_kv_compress_ragged: every item's partial column sums, and room for a transposed, rounded copy of
// Rbar in whole steps of 64 rows, which is not written (the product makes it on the way into LDS): the size is part of what callers
// rely on.  Sets *pad_total to the items' rows in such steps.
static size_t ragged_workspace(int32_t batch, const int64_t* off, int32_t n_mem, int64_t* pad_total)
{
    *pad_total = 0;
    for (int32_t b = 0; b < batch; ++b) *pad_total += pad64(off[b + 1] - off[b]);
    return align256(static_cast<size_t>(batch) * n_mem * 4 * kColParts) + align256(static_cast<size_t>(n_mem) * *pad_total * 2);
}

}  // namespace civic

extern "C" size_t civic_kv_compress_ragged_workspace_bytes(int32_t batch, const int64_t* row_offsets, int32_t n_mem, int32_t width)
{
    if (batch <= 0 || n_mem <= 0 || width <= 0 || !civic::offsets_ok(row_offsets, batch)) return 0;
    int64_t pad_total;
    return civic::ragged_workspace(batch, row_offsets, n_mem, &pad_total);
}

extern "C" int civic_kv_compress_ragged(const void* k, const void* v, int dtype, const float* r, int32_t batch,
                                        const int64_t* row_offsets, int32_t n_mem, int32_t width, void* k_c, void* v_c,
                                        void* workspace, size_t workspace_bytes, void* stream)
{
    using namespace civic;
    const int esz = dtype_size(dtype);
    if (!esz || batch < 0 || n_mem <= 0 || width <= 0) return CIVIC_ERR_INVALID_ARG;
    if (batch == 0) return CIVIC_OK;
    if (!offsets_ok(row_offsets, batch)) return CIVIC_ERR_INVALID_ARG;
    if (!r || !k || !v || !k_c || !v_c) return CIVIC_ERR_INVALID_ARG;
    if (!aligned16(k) || !aligned16(v) || !aligned16(k_c) || !aligned16(v_c) || !aligned16(r)) return CIVIC_ERR_INVALID_ARG;
    if (dtype != CIVIC_BF16) return CIVIC_ERR_UNSUPPORTED;
    // every item's first row must be 16-byte aligned in K, V and R: whole 16-byte pieces per row
    if (width % 8 || n_mem % 4) return CIVIC_ERR_UNSUPPORTED;
    if (row_offsets[batch] > INT32_MAX) return CIVIC_ERR_UNSUPPORTED;       // (row numbers travel as 32-bit kernel arguments)
    for (int32_t b = 0; b < batch; ++b) {                                     // 32-bit row offsets inside one item, as in civic_kv_compress
        const int64_t padded = pad64(row_offsets[b + 1] - row_offsets[b]);
        if (padded * width * 2 >= (int64_t{1} << 32) || padded * n_mem * 2 >= (int64_t{1} << 32)) return CIVIC_ERR_UNSUPPORTED;
    }
    int64_t pad_total;
    const size_t need = ragged_workspace(batch, row_offsets, n_mem, &pad_total);
    if (pad_total > INT32_MAX) return CIVIC_ERR_UNSUPPORTED;
    if (!workspace || workspace_bytes < need || !aligned16(workspace)) return CIVIC_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    // Groups of up to kGroupItems items, two launches each.
    for (int32_t b0 = 0; b0 < batch; b0 += kGroupItems) {
        const int32_t nb = batch - b0 < kGroupItems ? batch - b0 : kGroupItems;
        CompressArgs c;
        c.r = r; c.x[0] = static_cast<const __bf16*>(k); c.x[1] = static_cast<const __bf16*>(v);
        c.out[0] = static_cast<__bf16*>(k_c) + static_cast<int64_t>(b0) * n_mem * width;
        c.out[1] = static_cast<__bf16*>(v_c) + static_cast<int64_t>(b0) * n_mem * width;
        c.m = n_mem; c.n = width; c.n_rows = 0;
        for (int32_t i = 0; i <= kGroupItems; ++i)                            // (entries past the group repeat its end)
            c.grp.row[i] = static_cast<int32_t>(row_offsets[b0 + (i <= nb ? i : nb)]);
        for (int32_t i = 0; i < kGroupItems; ++i) c.grp.longest_first[i] = static_cast<uint8_t>(i);
        std::stable_sort(c.grp.longest_first, c.grp.longest_first + nb, [&](uint8_t x, uint8_t y) {
            return c.grp.row[x + 1] - c.grp.row[x] > c.grp.row[y + 1] - c.grp.row[y];
        });
        float* part = static_cast<float*>(workspace) + static_cast<int64_t>(b0) * n_mem * kColParts;
        c.part = part;
        civic::launch(col_part_sum_grouped_kernel, dim3(static_cast<unsigned>((n_mem + kWave - 1) / kWave), kColParts, static_cast<unsigned>(nb)),
                      dim3(256), 0, s, r, n_mem, part, c.grp);
        int rc = check_launch();
        if (rc != CIVIC_OK) return rc;
        rc = launch_compress(c, nb, true, s);
        if (rc != CIVIC_OK) return rc;
    }
    return CIVIC_OK;
}
