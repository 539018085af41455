// civic_select: exact constrained top-k (cell floors, frame floors, global budget) with ascending,
// order-preserving output.  Latency-bound: a sample's scores are 8-128 KB.
//
// One workgroup per sample (1024 threads, 512 up to 2048 tokens) keeps everything in LDS: a 32-bit sort key per
// token and one mark bit per token.  The strict order "higher score first, equal scores to the lower index" becomes
// (key ascending, index ascending) after mapping the float bits to an unsigned key (with -0 folded
// onto +0).
//   cells   small cells: one thread per cell (from registers up to 4 x 4), or a team of 16 lanes, picks the
//           cell's best remaining member cell_floor times (smallest key, then smallest index = the tie rule).
//           large cells: one wavefront per cell runs the select below.
//   frames  one wavefront per frame: the select below over the frame's unmarked tokens (256 bins).
//   budget  the same select run by the whole workgroup over the unmarked tokens of the sample (512 to
//           2048 bins, by the tokens).
//   select  one histogram pass over buckets that are linear in the score, a search for the bucket that
//           holds the m-th token (by every wavefront for itself), one marking pass; the few tokens of that bucket are ranked against
//           each other directly.  Degenerate score distributions fall back to an exact radix select
//           over the key digits (see select_first).
//   output  popcounts of the 64-bit mark words -> LDS prefix scan -> every set bit writes its index
//           at (prefix of its word + set bits below it): ascending kept_idx without any sort.
#include "select_device.h"

namespace civic {

// One workgroup selects sample `b` of the tensors a.scores, a.kept_idx and a.keep_flags point at.
template <int T>
__global__ __launch_bounds__(T) void select_kernel(SelArgs a)
{
    constexpr int kSelThreads = T, kSelWaves = T / kWave;
    extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
    const SelLds m(smem, a);
    uint32_t* const bcast = m.bcast;
    uint32_t* const marks = m.marks;
    uint32_t* const word_prefix = m.word_prefix;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6, b = blockIdx.x;
    select_marks<T>(a, m, a.scores + static_cast<int64_t>(b) * a.nv);

    // ---- ascending output
    const int32_t words = a.nv_pad / 64;                     // <= 512, one per thread
    int32_t* out = a.kept_idx + static_cast<int64_t>(b) * a.kept;
    if (words <= kWave) {
        // Up to 4096 tokens: the mark words fit one per lane, so every wavefront scans all of them itself and
        // takes the prefixes of its own words from the scan's lanes; nothing goes through LDS, no barrier.
        const u32x2 mine = *reinterpret_cast<const u32x2*>(marks + 2 * min(lane, words - 1));
        const uint32_t cnt = lane < words ? __popc(mine.x) + __popc(mine.y) : 0u;
        const uint32_t before = wave_incl_scan(cnt, lane) - cnt;
#pragma unroll
        for (int u = 0; u < kWave / kSelWaves; ++u) {        // the wavefront's tokens: 64 per 1024, words wave, wave + kSelWaves, ...
            const int w = wave + u * kSelWaves;
            if (w >= words) break;
            const uint32_t lo = __builtin_amdgcn_readlane(mine.x, w), hi = __builtin_amdgcn_readlane(mine.y, w);
            const uint32_t base = __builtin_amdgcn_readlane(before, w);
            const uint64_t word = (static_cast<uint64_t>(hi) << 32) | lo;
            const int32_t v = w * kWave + lane;
            const bool bit = (word >> lane) & 1ull;
            if (bit) {
                const uint32_t pos = base + static_cast<uint32_t>(__popcll(word & ((1ull << lane) - 1ull)));
                if (pos < static_cast<uint32_t>(a.kept)) out[pos] = v;
            }
            if (a.keep_flags && v < a.nv) a.keep_flags[static_cast<int64_t>(b) * a.nv + v] = bit ? 1 : 0;
        }
        return;
    }
    uint32_t pc = 0;
    if (tid < words) pc = __popc(marks[2 * tid]) + __popc(marks[2 * tid + 1]);
    const uint32_t incl = wave_incl_scan(pc, lane);
    if (lane == kWave - 1) bcast[wave] = incl;
    __syncthreads();
    uint32_t wave_base = 0;
    {
        uint32_t tot[kSelWaves];                             // independent reads; a loop to `wave` would wait on each in turn
#pragma unroll
        for (int x = 0; x < kSelWaves; x += 4) {
            const u32x4 t = *reinterpret_cast<const u32x4*>(bcast + x);
            tot[x] = t.x; tot[x + 1] = t.y; tot[x + 2] = t.z; tot[x + 3] = t.w;
        }
#pragma unroll
        for (int x = 0; x < kSelWaves; ++x) wave_base += x < wave ? tot[x] : 0u;
    }
    if (tid < words) word_prefix[tid] = wave_base + incl - pc;
    __syncthreads();

    for (int32_t v0 = tid; v0 < a.nv_pad; v0 += kSelBatch * kSelThreads) {
        u32x2 mw[kSelBatch];
        uint32_t wp[kSelBatch];
#pragma unroll
        for (int u = 0; u < kSelBatch; ++u) {                // a batch of reads from clamped indices, then the stores
            const int32_t w = min(v0 + u * kSelThreads, a.nv_pad - 1) >> 6;
            mw[u] = *reinterpret_cast<const u32x2*>(marks + 2 * w);
            wp[u] = word_prefix[w];
        }
#pragma unroll
        for (int u = 0; u < kSelBatch; ++u) {
            const int32_t v = v0 + u * kSelThreads;
            if (v >= a.nv_pad) break;
            const uint64_t word = (static_cast<uint64_t>(mw[u].y) << 32) | mw[u].x;
            const bool bit = (word >> lane) & 1ull;
            if (bit) {
                const uint32_t pos = wp[u] + static_cast<uint32_t>(__popcll(word & ((1ull << lane) - 1ull)));
                if (pos < static_cast<uint32_t>(a.kept)) out[pos] = v;
            }
            if (a.keep_flags && v < a.nv) a.keep_flags[static_cast<int64_t>(b) * a.nv + v] = bit ? 1 : 0;
        }
    }
}


}  // namespace civic

namespace civic {

// The argument checks of civic_select (host only, nothing is launched).
int select_check(const float* scores, int32_t batch, const civic_grid* grid, const int32_t* kept_idx)
{
    GridInfo gi;
    if (grid_info(grid, &gi) != CIVIC_OK) return CIVIC_ERR_INVALID_ARG;
    if (batch < 0) return CIVIC_ERR_INVALID_ARG;
    if (batch > 0 && (!scores || (gi.kept > 0 && !kept_idx))) return CIVIC_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(scores) | reinterpret_cast<uintptr_t>(kept_idx)) & 3u) return CIVIC_ERR_INVALID_ARG;
    if (gi.nv > CIVIC_MAX_VISUAL_TOKENS) return CIVIC_ERR_UNSUPPORTED;
    return CIVIC_OK;
}

}  // namespace civic

namespace civic {

// What the kernel needs to know about a sample of grid `gi` (checked), and the dynamic LDS it takes in bytes.
SelArgs make_sel_args(const float* scores, int32_t* kept_idx, uint8_t* keep_flags, const GridInfo& gi, size_t* lds_bytes)
{
    SelArgs a;
    a.scores = scores; a.kept_idx = kept_idx; a.keep_flags = keep_flags;
    a.frames = gi.frames; a.height = gi.height; a.width = gi.width; a.hw = gi.hw; a.nv = gi.nv;
    a.nv_pad = (gi.nv + 63) / 64 * 64;
    a.cell_h = gi.cell_h < gi.height ? gi.cell_h : gi.height;
    a.cell_w = gi.cell_w < gi.width ? gi.cell_w : gi.width;
    a.cell_floor = gi.cell_floor; a.frame_floor = gi.frame_floor;
    a.cells_y = (gi.height + a.cell_h - 1) / a.cell_h;
    a.cells_x = (gi.width + a.cell_w - 1) / a.cell_w;
    a.floor_sum = gi.floor_sum; a.fill = gi.fill; a.kept = gi.kept;
    a.big_cells = static_cast<int64_t>(a.cell_h) * a.cell_w > kSmallCell ? 1 : 0;
    a.cell_kept_frame = gi.cell_kept_frame;
    a.quad_scores = (reinterpret_cast<uintptr_t>(scores) & 15u) == 0 && gi.nv % 4 == 0;
    auto magic = [](int64_t d) { return d <= 1 ? 0u : static_cast<uint32_t>(((int64_t{1} << 32) + d - 1) / d); };
    a.magic_cells_f = magic(static_cast<int64_t>(a.cells_y) * a.cells_x);
    a.magic_cells_x = magic(a.cells_x);
    a.magic_qpr = magic(a.cell_w / 4);
    a.cell_team = 0; a.cell_team_shift = 0;
    // Cells of 64-256 tokens whose rows are made of aligned quads of keys get 16 lanes each; smaller ones are
    // faster with a thread of their own (measured: 4 x 4 cells 1.0 us against 1.3 us, 8 x 8 cells 2.4 against 1.5).
    if (a.cell_w % 4 == 0 && a.cells_x * a.cell_w == a.width && !a.big_cells && a.cell_h * (a.cell_w / 4) >= 16) {
        a.cell_team = 16; a.cell_team_shift = 4;
    }
    // keys | histograms | per-team words | mark bits | word prefixes, rounded up to 16 bytes | per-wavefront extremes | candidate count
    const size_t lds_words = (static_cast<size_t>(a.nv_pad) + kSelHistWords + kSelMaxWaves * 8 + a.nv_pad / 32 + a.nv_pad / 64 + 3) / 4 * 4 +
                             2 * kSelMaxWaves + 4;
    a.lds_words = static_cast<int32_t>(lds_words);
    *lds_bytes = sizeof(uint32_t) * lds_words;
    return a;
}

// The limit of dynamic LDS is raised once per device and kernel, for the largest sample there is.
int allow_select_lds(const void* kernel, std::atomic<uint64_t>* done)
{
    constexpr size_t max_pad = (CIVIC_MAX_VISUAL_TOKENS + 63) / 64 * 64;
    constexpr size_t max_lds = sizeof(uint32_t) * ((max_pad + kSelHistWords + kSelMaxWaves * 8 + max_pad / 32 + max_pad / 64 + 3) / 4 * 4 +
                                                   2 * kSelMaxWaves + 4);
    return allow_dynamic_lds(kernel, max_lds, done);
}

}  // namespace civic

extern "C" int civic_select(const float* scores, int32_t batch, const civic_grid* grid, int32_t* kept_idx,
                            uint8_t* keep_flags, void* workspace, size_t workspace_bytes, void* stream)
{
    using namespace civic;
    (void)workspace; (void)workspace_bytes;
    const int rc_check = select_check(scores, batch, grid, kept_idx);
    if (rc_check != CIVIC_OK) return rc_check;
    if (batch == 0) return CIVIC_OK;
    GridInfo gi;
    grid_info(grid, &gi);
    size_t lds = 0;
    const SelArgs a = make_sel_args(scores, kept_idx, keep_flags, gi, &lds);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (gi.nv <= kSelSmallTokens) {
        civic::launch(select_kernel<kSelSmallThreads>, dim3(static_cast<unsigned>(batch)), dim3(kSelSmallThreads), lds, s, a);
        return check_launch();
    }
    if (lds > 64 * 1024) {
        static std::atomic<uint64_t> allowed{0};
        const int rc = allow_select_lds(reinterpret_cast<const void*>(select_kernel<kSelMaxThreads>), &allowed);
        if (rc != CIVIC_OK) return rc;
    }
    civic::launch(select_kernel<kSelMaxThreads>, dim3(static_cast<unsigned>(batch)), dim3(kSelMaxThreads), lds, s, a);
    return check_launch();
}
