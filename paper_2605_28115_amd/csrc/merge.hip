// Selection and compact merge of the front (civic_compact_prefill, civic_compact_prefill_ragged) in one launch: what civic_select
// and civic_compact do one after the other, for callers that want both.
//
// A selection keeps one compute unit busy for 4 to 14 us while 255 wait, and a merge launch after it starts cold and reads the kept
// list back before it knows its first row.  Here every workgroup that moves rows makes the sample's selection by itself
// (select_device.h: deterministic, so all of a sample's workgroups hold the same marks), finds the sources of its own compact rows
// in the marks and copies them: the same selection up to 256 times over costs no more time than once, and there is no second
// launch, no kept list to read and no idle chip between the two.  Rows whose place does not depend on the selection - text
// before the first frame and after the last - are moved by workgroups of their own meanwhile, as long as two workgroups fit a unit.
//   - a workgroup's rows are a contiguous run of compact rows, so its output is one linear run of 16-byte vectors; a thread divides
//     its vector number by the vectors per row (multiply-high) and looks the row's source up in LDS
//   - 8 or 16 wavefronts a unit with 10 or 6 loads of 16 bytes each in flight per lane
// Kernel times (us), selection + merge as launches of their own and as one: a 32 x 32 image of 2048-channel rows 5.4 + 4.7 and 7.6;
// four prompts of two such images, 4096 channels 7.2 + 13.6 and 18.1; two 64 x 64 grids of 1152 channels 7.5 + 8.8 and 12.4; 16 frames
// of 24 x 24, 4096 channels 16.4 + 14.4 and 28.6; eight prompts of different grids 6.8 + 14.7 and 21.4.
#include <algorithm>

#include "select_device.h"

namespace civic {

constexpr int kMergeRows = 2048;                 // rows whose sources are held in LDS at a time
constexpr int kMergeUnits = 256;                 // compute units
constexpr int kMergeGroupBytes = 8 * 1024;       // a workgroup of 512 threads moves at least this much: one load per thread
constexpr int kMergeTextBytes = 64 * 1024;       // moved by a workgroup that only copies text
constexpr int kMergeLongBytes = 128 * 1024;      // moved by a workgroup of a large batch of long samples

struct MergeItem {
    SelArgs sel;
    int64_t row0, comp0;                         // the sample's first dense and compact row
    int32_t seq_len, seq_c;
    int32_t head, tail;                          // text rows at the sample's ends that workgroups of their own move
    int32_t sel_groups, text_groups;
    uint32_t magic_hw;                           // ceil(2^32 / hw), 0 for hw = 1
};
// Samples of one shape.
struct MergeBatch {
    MergeItem it;
    int32_t n;
    int32_t start[CIVIC_MAX_FRAMES];             // sequence index of each frame's first token
    __device__ __forceinline__ const MergeItem& item(int) const { return it; }
    __device__ __forceinline__ const int32_t* starts(int) const { return start; }
    __device__ __forceinline__ int64_t place(int i) const { return i; }
};
// Samples of different shape: each brings its own description, with pointers to its own scores and kept indices.
struct MergeTable {
    MergeItem items[kMergeItems];
    int32_t n;
    int32_t start[kMergeItems][kMergeItemFrames];
    __device__ __forceinline__ const MergeItem& item(int i) const { return items[i]; }
    __device__ __forceinline__ const int32_t* starts(int i) const { return start[i]; }
    __device__ __forceinline__ int64_t place(int) const { return 0; }
};

struct MergeTensors {
    const u32x4* hidden;
    const int32_t* pos_ids;
    u32x4* hidden_c;
    int32_t* pos_c;
    int32_t* src_idx;
    int64_t pos_axis_in, pos_axis_out;
    int32_t vpr;                                 // 16-byte vectors per row
    uint32_t magic_vpr;                          // ceil(2^32 / vpr), 0 for vpr = 1
};

// What the kernel is launched with, as its one argument: it lies at the front of the argument segment as it lies on the host.  The kernel
// reads it there, and again after the selection: values that were read before and are needed after it would fill the scalar registers
// across it (60 of them spilled).
template <typename MAP>
struct MergeArgs { MAP map; MergeTensors t; };
template <typename MAP>
__device__ __forceinline__ const MergeArgs<MAP>& merge_args()
{
    static_assert(std::is_trivially_copyable<MergeArgs<MAP>>::value && std::is_standard_layout<MergeArgs<MAP>>::value &&
                      alignof(MergeArgs<MAP>) <= 16 && sizeof(MergeArgs<MAP>) <= 4096,
                  "passed byte for byte, where the segment begins");
    auto p = (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const MergeArgs<MAP>*)p;
}

template <typename MAP, int T>
__global__ __launch_bounds__(T, T / 128) void merge_kernel(MergeArgs<MAP>)
{
    constexpr int kSelThreads = T, kSelWaves = T / kWave;
    constexpr int kMergeUnroll = T == kSelMaxThreads ? 6 : 10;         // 16-byte loads in flight per thread (in 64 and in 128 registers)
    extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
    const MAP& map = merge_args<MAP>().map;
    // grid y: every sample's selecting workgroups, then every sample's text workgroups
    const bool text_only = static_cast<int>(blockIdx.y) >= map.n;
    const int y = static_cast<int>(blockIdx.y) - (text_only ? map.n : 0);
    int32_t first, last;                                               // the workgroup's share of the rows
    {
        // rows [first, last) of the compact rows between the ends, or of the two ends put together
        const MergeItem& it = map.item(y);
        const int groups = text_only ? it.text_groups : it.sel_groups;
        if (static_cast<int>(blockIdx.x) >= groups) return;
        const int32_t total = text_only ? it.head + it.tail : it.seq_c - it.head - it.tail;
        first = static_cast<int32_t>(static_cast<int64_t>(total) * blockIdx.x / groups);
        last = static_cast<int32_t>(static_cast<int64_t>(total) * (blockIdx.x + 1) / groups);
        if (first >= last) return;
    }
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    int32_t my_start = 0;                                              // (in flight under the selection)
    if (!text_only) {
        const SelArgs& a = map.item(y).sel;
        if (tid < a.frames) my_start = map.starts(y)[tid];
        select_marks<T>(a, SelLds(smem, a), a.scores + map.place(y) * a.nv);
    }

    const MergeArgs<MAP>& args = merge_args<MAP>();
    const MergeItem& it = args.map.item(y);
    const MergeTensors& t = args.t;
    const SelArgs& a = it.sel;
    const int64_t place = args.map.place(y);
    const SelLds m(smem, a);
    const int64_t row0 = it.row0 + place * it.seq_len, comp0 = it.comp0 + place * it.seq_c;
    const int32_t F = a.frames, hw = a.hw, words = a.nv_pad / 64;
    int32_t* const row_src = reinterpret_cast<int32_t*>(m.hist);       // [kMergeRows], in the histograms' place
    int32_t* const fstart = row_src + kMergeRows;                      // [frames]: text tokens before frame f
    int32_t* const kb = fstart + CIVIC_MAX_FRAMES;                     // [frames + 1]: kept tokens before frame f
    static_assert(kMergeRows + 2 * CIVIC_MAX_FRAMES + 1 <= kSelHistWords, "the tables fit the histograms' place");
    const bool text_between = it.seq_c - it.head - it.tail != a.kept;  // text rows among those placed by the selection
    uint32_t before = 0;                                               // up to 64 mark words: kept tokens before word `lane`
    const int32_t fs0 = args.map.starts(y)[0], fs_last = args.map.starts(y)[F - 1] - (F - 1) * hw;
    if (!text_only) {
        // Kept tokens before every mark word of 64: up to 64 words every wavefront has them all in its lanes, more go through LDS.
        uint32_t pc = 0;
        const int32_t my_word = words <= kWave ? lane : tid;
        if (my_word < words) {
            const u32x2 mw = *reinterpret_cast<const u32x2*>(m.marks + 2 * my_word);
            pc = __popc(mw.x) + __popc(mw.y);
        }
        const uint32_t incl = wave_incl_scan(pc, lane);
        before = incl - pc;
        if (words > kWave) {
            if (lane == kWave - 1) m.bcast[wave] = incl;
            __syncthreads();
#pragma unroll
            for (int x = 0; x < kSelWaves; x += 4) {
                const u32x4 s4 = *reinterpret_cast<const u32x4*>(m.bcast + x);
                const uint32_t tot[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) before += x + e < wave ? tot[e] : 0u;
            }
        }
        if (my_word < words && (words > kWave || wave == 0)) m.word_prefix[my_word] = before;
        if (F > 1 || text_between) {                                   // (one frame without text around it needs no table)
            if (tid < F) fstart[tid] = my_start - tid * hw;
            __syncthreads();
        } else if (words > kWave) {
            __syncthreads();
        }
        if (text_between) {
            if (tid <= F) {
                const int32_t v = tid * hw;
                uint32_t n = static_cast<uint32_t>(a.kept);
                if (tid < F) {
                    const u32x2 mw = *reinterpret_cast<const u32x2*>(m.marks + 2 * (v >> 6));
                    const uint64_t word = (static_cast<uint64_t>(mw.y) << 32) | mw.x;
                    n = m.word_prefix[v >> 6] + static_cast<uint32_t>(__popcll(word & ((1ull << (v & 63)) - 1ull)));
                }
                kb[tid] = static_cast<int32_t>(n);
            }
            __syncthreads();
        }
    }
    int32_t* const kept_idx = a.kept_idx + place * a.kept;

    for (int32_t j0 = first, nrows; j0 < last; j0 += nrows) {          // (nrows at most last - j0: j0 stays in range)
        nrows = min(kMergeRows, last - j0);
        const int32_t slot0 = text_only ? j0 : j0 + it.head;           // compact row of the run's first row
        // text of both ends: rows from `split` on lie behind the rows in between
        const int32_t split = text_only ? min(max(it.head - j0, 0), nrows) : nrows;
        const int32_t gap = text_only ? it.seq_c - it.head - it.tail : 0;
        if (j0 != first) __syncthreads();                              // the sources of the run before are still read
        if (text_only) {
            const int32_t dropped = it.seq_len - it.head - it.tail;
            for (int32_t r = tid; r < nrows; r += kSelThreads) row_src[r] = j0 + r + (r >= split ? dropped : 0);
        } else {
            // Kept tokens: the i-th of them, of frame f, is compact row fstart[f] + i.  Only mark words whose tokens can land in
            // the run are looked at, one token a lane.
            const int32_t win_lo = slot0 - fs_last, win_hi = slot0 + nrows - fs0;
            for (int32_t w = wave; w < words; w += kSelWaves) {
                const u32x2 mw = *reinterpret_cast<const u32x2*>(m.marks + 2 * w);
                const uint64_t word = (static_cast<uint64_t>(mw.y) << 32) | mw.x;
                const int32_t base = static_cast<int32_t>(words <= kWave ? __builtin_amdgcn_readlane(before, w) : m.word_prefix[w]);
                const int32_t past = base + static_cast<int32_t>(__popcll(word));
                if (base >= win_hi || past <= win_lo) continue;
                if ((word >> lane) & 1ull) {
                    const int32_t v = w * kWave + lane, i = base + static_cast<int32_t>(__popcll(word & ((1ull << lane) - 1ull)));
                    const int32_t fs = F > 1 ? fstart[div_magic(v, it.magic_hw)] : fs0, r = fs + i - slot0;
                    if (r >= 0 && r < nrows) {
                        row_src[r] = fs + v;
                        if (i < a.kept) kept_idx[i] = v;               // (every kept token has one compact row: written once)
                    }
                }
            }
            // the other rows are text: the tokens dropped before them added back
            for (int32_t r = text_between ? tid : nrows; r < nrows; r += kSelThreads) {
                const int32_t j = slot0 + r;
                int32_t lo = 0, hi = F;                                // frames whose compact rows begin at or before j
                while (lo < hi) {
                    const int32_t mid = (lo + hi) >> 1;
                    if (fstart[mid] + kb[mid] <= j) lo = mid + 1; else hi = mid;
                }
                if (lo == 0) row_src[r] = j;
                else if (j >= fstart[lo - 1] + kb[lo]) row_src[r] = j + lo * hw - kb[lo];
            }
        }
        __syncthreads();

        // ids of the first rows: their loads fly with the rows' own
        auto source = [&](int32_t r) { return min(max(row_src[r], 0), it.seq_len - 1); };
        const int32_t r_id = min(tid, nrows - 1);
        const int32_t id_src = source(r_id);
        int32_t id[3];
#pragma unroll
        for (int x = 0; x < 3; ++x) id[x] = t.pos_ids[x * t.pos_axis_in + row0 + id_src];

        const u32x4* const in = t.hidden + row0 * t.vpr;
        u32x4* const out = t.hidden_c + (comp0 + slot0) * t.vpr;
        const int32_t n_vec = nrows * t.vpr, split_vec = split * t.vpr;
        const int64_t gap_vec = static_cast<int64_t>(gap) * t.vpr;
        for (int32_t i0 = 0; i0 < n_vec; i0 += kMergeUnroll * kSelThreads) {
            u32x4 val[kMergeUnroll];
#pragma unroll
            for (int u = 0; u < kMergeUnroll; ++u) {                   // (a clamped index repeats the last vector: no load is conditional)
                const int32_t i = min(i0 + u * kSelThreads + tid, n_vec - 1);
                const int32_t r = div_magic(i, t.magic_vpr), c = i - r * t.vpr;
                val[u] = load_streaming(in + static_cast<int64_t>(source(r)) * t.vpr + c);
            }
            // (A model normalises these rows next.  us for the path alone, and with a layer norm over the rows and a product over the
            // attention's output, inputs that change from pass to pass; stores cached, non-temporal and written through: 4 x 938 rows of 4096
            // 71.1, 68.7, 69.9 and 257.8, 259.0, 257.3; eight ragged prompts 73.4, 71.6, 72.0 and 248.0, 251.2, 246.2; heads of 64 55.0, 55.0,
            // 53.8 and 134.1, 135.7, 131.7; 16 / 8 heads 63.5, 58.1, 62.4 and 137.1, 138.7, 135.8.)
#pragma unroll
            for (int u = 0; u < kMergeUnroll; ++u) {
                const int32_t i = i0 + u * kSelThreads + tid;
                if (i < n_vec) store_through(out + i + (i >= split_vec ? gap_vec : 0), val[u]);
            }
        }
        auto put_ids = [&](int32_t r, int32_t src, const int32_t (&p)[3]) {
            const int64_t o = comp0 + slot0 + r + (r >= split ? gap : 0);
            t.src_idx[o] = src;
#pragma unroll
            for (int x = 0; x < 3; ++x) t.pos_c[x * t.pos_axis_out + o] = p[x];
        };
        if (tid < nrows) put_ids(tid, id_src, id);
        for (int32_t r = tid + kSelThreads; r < nrows; r += kSelThreads) {
            const int32_t src = source(r);
#pragma unroll
            for (int x = 0; x < 3; ++x) id[x] = t.pos_ids[x * t.pos_axis_in + row0 + src];
            put_ids(r, src, id);
        }
    }
}

static uint32_t merge_magic(int64_t d) { return d <= 1 ? 0u : static_cast<uint32_t>(((int64_t{1} << 32) + d - 1) / d); }

// A sample's description without its place and its workgroups; the LDS it takes.
static MergeItem merge_item(const float* scores, int32_t* kept_idx, const civic_grid* grid, const int64_t* frame_start, int64_t seq_len,
                            int32_t* start, size_t* lds)
{
    GridInfo gi;
    grid_info(grid, &gi);
    MergeItem it;
    it.sel = make_sel_args(scores, kept_idx, nullptr, gi, lds);
    it.row0 = 0; it.comp0 = 0;
    it.seq_len = static_cast<int32_t>(seq_len);
    it.seq_c = static_cast<int32_t>(seq_len - gi.nv + gi.kept);
    it.head = static_cast<int32_t>(frame_start[0]);
    it.tail = static_cast<int32_t>(seq_len - frame_start[gi.frames - 1] - gi.hw);
    it.sel_groups = it.text_groups = 0;
    it.magic_hw = merge_magic(gi.hw);
    for (int32_t f = 0; f < gi.frames; ++f) start[f] = static_cast<int32_t>(frame_start[f]);
    return it;
}

// Rows that selecting workgroups move.
static int64_t placed_rows(const MergeItem& it, bool text_apart) { return it.seq_c - (text_apart ? it.head + it.tail : 0); }

// Selecting workgroups of each of `batch` samples with `bytes` of rows to move.  Up to half as many samples as units: one workgroup to
// a unit.  More samples: workgroups that fill the units twice over, two for each sample at least, and for long samples one for every
// 128 KB up to eight times over: what a selection costs is small beside their rows, and many small workgroups end together.  (us,
// front, one workgroup to a unit and so: 129 samples of 16 x 16, 1024 channels 39.0, 36.8, 300 of them 83.4, 78.8; 129 of 32 x 32, 2048
// channels 205, 181, 300 of them 535, 485; 300 of 64 x 64, 1152 channels 1242, 1154.)
static int64_t merge_share(int32_t batch, int64_t bytes)
{
    if (batch <= kMergeUnits / 2) return kMergeUnits / batch;
    const int64_t least = std::max(2 * kMergeUnits / batch, 2), most = (8 * kMergeUnits + batch - 1) / batch;
    return std::max(least, std::min(most, bytes / kMergeLongBytes));
}

// How many workgroups move an item's rows when `units` of the launch's selecting workgroups are its share.
static void merge_groups(MergeItem* it, int64_t units, int64_t row_bytes, bool text_apart)
{
    if (!text_apart) it->head = it->tail = 0;
    auto groups = [&](int64_t rows, int64_t bytes, int64_t most) {
        const int64_t n = std::min<int64_t>((rows * row_bytes + bytes - 1) / bytes, std::max<int64_t>(most, 1));
        return static_cast<int32_t>(std::min(n, rows));
    };
    it->sel_groups = groups(it->seq_c - it->head - it->tail, kMergeGroupBytes, units);
    it->text_groups = groups(static_cast<int64_t>(it->head) + it->tail, kMergeTextBytes, units);
}

static MergeTensors merge_tensors(const void* hidden, int64_t row_bytes, const int32_t* pos_ids, void* hidden_c, int32_t* pos_c,
                                  int32_t* src_idx, int64_t pos_axis_in, int64_t pos_axis_out)
{
    MergeTensors t;
    t.hidden = static_cast<const u32x4*>(hidden); t.pos_ids = pos_ids;
    t.hidden_c = static_cast<u32x4*>(hidden_c); t.pos_c = pos_c; t.src_idx = src_idx;
    t.pos_axis_in = pos_axis_in; t.pos_axis_out = pos_axis_out;
    t.vpr = static_cast<int32_t>(row_bytes / 16);
    t.magic_vpr = merge_magic(t.vpr);
    return t;
}

template <typename MAP, int T>
static int merge_launch(const MAP& map, const MergeTensors& t, int32_t widest, bool text, size_t lds, void* stream)
{
    if (widest == 0) return CIVIC_OK;                                  // no compact rows (and so no kept token)
    if (lds > 64 * 1024) {
        static std::atomic<uint64_t> allowed{0};
        const int rc = allow_select_lds(reinterpret_cast<const void*>(merge_kernel<MAP, T>), &allowed);
        if (rc != CIVIC_OK) return rc;
    }
    const dim3 grid(static_cast<unsigned>(widest), static_cast<unsigned>(text ? 2 * map.n : map.n));
    civic::launch((merge_kernel<MAP, T>), grid, dim3(T), lds, static_cast<hipStream_t>(stream), MergeArgs<MAP>{map, t});
    return check_launch();
}

// Text gets workgroups of its own where two workgroups fit a unit's LDS, and for launches whose samples take several each.
constexpr size_t kMergePairLds = 80 * 1024;

// Beyond 2^19 visual tokens in samples of more than 2048 the selection as a launch of its own is the faster one: there are samples for
// enough units then, and a sample's selection takes too long to be made by all its workgroups.  (us, front, in one launch and in two: 64
// samples of 64 x 64, 1152 channels 177, 182; 64 of 8 x 32 x 32, 512 channels 225, 225; 32 of 128 x 128 218, 218; 64 of 96 x 96 247, 243,
// 128 of them 523, 506; 64 of 180 x 180 895, 877.)
bool merge_in_one_launch(int32_t batch, int64_t nv) { return nv <= kSelSmallTokens || batch * nv <= (int64_t{1} << 19); }

int merge_batch_launch(const void* hidden, int dtype, int32_t dim, const int32_t* pos_ids, int32_t batch, int64_t seq_len,
                       const civic_grid* grid, const int64_t* frame_start, const float* scores, int32_t* kept_idx, void* hidden_c,
                       int32_t* pos_c, int32_t* src_idx, int64_t pos_axis_in, int64_t pos_axis_out, void* stream)
{
    if (batch == 0) return CIVIC_OK;
    const int64_t row_bytes = static_cast<int64_t>(dim) * dtype_size(dtype);
    MergeBatch map;
    size_t lds = 0;
    for (int32_t f = 0; f < CIVIC_MAX_FRAMES; ++f) map.start[f] = 0;
    map.it = merge_item(scores, kept_idx, grid, frame_start, seq_len, map.start, &lds);
    map.n = batch;
    const bool text_apart = lds <= kMergePairLds && batch <= kMergeUnits / 2;
    merge_groups(&map.it, merge_share(batch, placed_rows(map.it, text_apart) * row_bytes), row_bytes, text_apart);
    const MergeTensors t = merge_tensors(hidden, row_bytes, pos_ids, hidden_c, pos_c, src_idx, pos_axis_in, pos_axis_out);
    const int32_t widest = std::max(map.it.sel_groups, map.it.text_groups);
    const bool text = map.it.text_groups > 0;
    return map.it.sel.nv <= kSelSmallTokens ? merge_launch<MergeBatch, kSelSmallThreads>(map, t, widest, text, lds, stream)
                                            : merge_launch<MergeBatch, kSelMaxThreads>(map, t, widest, text, lds, stream);
}

int merge_samples_launch(const void* hidden, int dtype, int32_t dim, const int32_t* pos_ids, const float* scores, int32_t* kept_idx,
                         void* hidden_c, int32_t* pos_c, int32_t* src_idx, const RaggedSample* samples, int32_t n, int64_t pos_axis_in,
                         int64_t pos_axis_out, void* stream)
{
    const int64_t row_bytes = static_cast<int64_t>(dim) * dtype_size(dtype);
    MergeTable map;
    size_t lds = 0;
    int64_t rows = 0;
    int32_t largest = 0;
    map.n = n;
    for (int i = 0; i < kMergeItems; ++i) {
        for (int f = 0; f < kMergeItemFrames; ++f) map.start[i][f] = 0;
        if (i >= n) { map.items[i] = map.items[0]; continue; }         // (never read: the grid has n samples)
        const RaggedSample& x = samples[i];
        size_t one = 0;
        map.items[i] = merge_item(scores + x.vis0, kept_idx + x.kept0, x.grid, x.frame_start, x.seq_len, map.start[i], &one);
        map.items[i].row0 = x.row0; map.items[i].comp0 = x.comp0;
        largest = std::max(largest, map.items[i].sel.nv);
        lds = std::max(lds, one);
    }
    for (int i = 0; i < n; ++i) rows += placed_rows(map.items[i], lds <= kMergePairLds);
    int32_t widest = 0;
    bool text = false;
    for (int i = 0; i < n; ++i) {
        MergeItem& it = map.items[i];
        const int64_t share = rows > 0 ? (kMergeUnits * placed_rows(it, lds <= kMergePairLds) + rows / 2) / rows : 0;
        merge_groups(&it, share, row_bytes, lds <= kMergePairLds);
        widest = std::max(widest, std::max(it.sel_groups, it.text_groups));
        text = text || it.text_groups > 0;
    }
    const MergeTensors t = merge_tensors(hidden, row_bytes, pos_ids, hidden_c, pos_c, src_idx, pos_axis_in, pos_axis_out);
    return largest <= kSelSmallTokens ? merge_launch<MergeTable, kSelSmallThreads>(map, t, widest, text, lds, stream)
                                      : merge_launch<MergeTable, kSelMaxThreads>(map, t, widest, text, lds, stream);
}

}  // namespace civic
