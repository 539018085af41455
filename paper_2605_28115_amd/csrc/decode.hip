// civic_decode_attn: one generated token attending to the compact prompt in the contiguous KV cache (the
// per-token work inside the autoregressive decoding cost C_dec of Eq. 2 / Eq. 7; the cache is the one
// civic_kv_write fills).  HBM-bound: every K and V row of the context is read once, 2 * H_kv * n_ctx * d
// elements per sample, and nothing else of size moves.
//
// The context of a (batch item, KV head) is split over several workgroups so that a launch of a few dozen
// (item, head) pairs still covers the chip; a workgroup serves all query heads of its KV head at once (up to 8
// per pass, 16 on the matrix cores), so K and V are read once per group, not once per query head.
// The vector kernel (fp32, one or two bf16 heads per KV head, head_dim above 128):
//   - A cache row is read by LPR adjacent lanes, 16 bytes each (LPR = row bytes / 16 rounded up to a power of two),
//     64 / LPR rows per wavefront instruction; a lane's loads of a round (U rows of K and the same rows of V) are
//     issued before anything is computed, so a workgroup whose share is one round makes a single trip to memory.
//   - Logits: packed bf16 dot products (v_dot2_f32_bf16) of the lane's 8 channels against every query head,
//     summed over the row's lanes; every lane of the row then holds the row's logits.
//   - Each (wavefront, row slot) runs its own online softmax over the rows it meets: no barrier and no LDS in
//     the loop.  The lane keeps the 8 output channels of its chunk for every head in fp32.
//   - At the end the partial states of the workgroup's 4, 8 or 16 wavefronts meet, in registers and LDS; it writes the final
//     rows (one split) or its (max, sum, unnormalised output) into the workspace, which a second small launch
//     combines.
#include <algorithm>
#include <cmath>

#include "civic_internal.h"

namespace civic {

constexpr int kDecThreads = 256;
constexpr int kDecWaves = kDecThreads / kWave;
constexpr int kDecU = 4;                 // cache rows per lane and round

constexpr int kDecFullUnits = 384;       // (sample, KV head, head block) triples that keep the chip busy without a split

constexpr int kDecRaggedUnits = 256;     // the same where every sample has its own context length
constexpr int kDecRaggedKeys = 512, kDecVecRaggedKeys = 256;   // rows per piece of a ragged launch that fills the chip
constexpr int kDecTailKeys = 448;         // rows by which the longest context may exceed the average before it is cut
constexpr int kDecRaggedItems = 256;     // samples of one launch when every sample has its own context length

struct DecodeArgs {
    const void* q; const void* kc; const void* vc; void* out; float* ws;
    int64_t s_max;
    int32_t batch, n_q_heads, n_kv_heads, head_dim, group, head_blocks;
    int32_t n_ctx, splits, keys_per_split;
    int32_t heads_first;                  // grid order (decode_grid)
    int32_t cpr;                          // 16-byte chunks per cache row
    float scale_log2;                     // softmax scale * log2(e)
};

// civic_decode_attn_ragged: sample b attends to its cache rows [0, ctx[b]), cut into pieces of keys_per_split rows.  (The grid
// covers the longest sample, workgroups past a sample's pieces leave at once: finding a piece's sample in a table of first
// pieces instead was 1.3 us slower on 5 samples of 27..216 rows, two dependent reads of the kernel arguments.)
struct DecodeTable {
    int32_t ctx[kDecRaggedItems];
};
struct NoTable {};

typedef __bf16 dec_bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 dec_bf16x8 __attribute__((ext_vector_type(8)));
typedef float dec_f32x4 __attribute__((ext_vector_type(4)));

// acc + a.lo * b.lo + a.hi * b.hi for two words of packed bf16 pairs.  (The words come in as scalars on purpose:
// a bit cast applied directly to an element of a vector variable reads the vector's first element.)
__device__ __forceinline__ float dot2_words(uint32_t a, uint32_t b, float acc)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(dec_bf16x2, a), __builtin_bit_cast(dec_bf16x2, b), acc, false);
}

// Sum over the LPR adjacent lanes that share a cache row; every one of them receives the total.  Inside a row of
// 16 lanes the exchange is a data-parallel-primitive (DPP) operand of the add itself: lane pairs, then the two
// pairs of a quad, then the mirrored lane of the other quad of a half row (whose four lanes all hold that quad's
// sum by then), then the mirrored lane of the other half row.  No LDS round trip: a shuffle through LDS per step
// made the logits of a round a chain of 64 dependent waits.  Rows wider than 16 lanes finish with shuffles.
template <int CTRL>
__device__ __forceinline__ float dpp_moved(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}

template <int LPR>
__device__ __forceinline__ float row_sum(float v)
{
    if constexpr (LPR >= 2) v += dpp_moved<0xB1>(v);        // quad_perm [1,0,3,2]
    if constexpr (LPR >= 4) v += dpp_moved<0x4E>(v);        // quad_perm [2,3,0,1]
    if constexpr (LPR >= 8) v += dpp_moved<0x141>(v);       // row_half_mirror
    if constexpr (LPR >= 16) v += dpp_moved<0x140>(v);      // row_mirror
    if constexpr (LPR >= 32) v += __shfl_xor(v, 16, kWave);
    if constexpr (LPR >= 64) v += __shfl_xor(v, 32, kWave);
    return v;
}

// Sum and maximum over the 64 / LPR row slots of a wavefront (lanes LPR apart), in every lane: a rotation inside rows of 16
// lanes, then swaps of rows and of half-waves (v_permlane16_swap, v_permlane32_swap).  No LDS.
template <int LPR, typename OP>
__device__ __forceinline__ float over_slots(float v, OP op)
{
    if constexpr (LPR <= 8) v = op(v, dpp_moved<0x128>(v));    // row_ror:8
    if constexpr (LPR <= 16) {
        const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = op(__uint_as_float(p[0]), __uint_as_float(p[1]));
    }
    if constexpr (LPR <= 32) {
        const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = op(__uint_as_float(p[0]), __uint_as_float(p[1]));
    }
    return v;
}
template <int LPR> __device__ __forceinline__ float slots_sum(float v) { return over_slots<LPR>(v, [](float x, float y) { return x + y; }); }
template <int LPR> __device__ __forceinline__ float slots_max(float v) { return over_slots<LPR>(v, [](float x, float y) { return fmaxf(x, y); }); }

// States of the vector kernel's workgroup that meet in LDS: one per wavefront where a wavefront holds 8 row slots, one per slot
// elsewhere.  Sums in registers take two lane swaps a value and halving of the slots, LDS one round trip a slot (21 x 16 rows, 8 / 8
// bf16 heads of 64, 8 slots: 3.7 us in registers, 4.1 in LDS; 85 x 23 rows, 28 / 4 fp32 heads of 64, 4 slots: 7.7 and 6.9).  Wide
// workgroups always meet in registers first: their slots would take up to 133 KB of LDS (8 wavefronts, 8 fp32 heads of 128).
constexpr int decode_states(int lpr, int waves) { return lpr == 8 || waves > kDecWaves ? waves : waves * (kWave / lpr); }

// A workgroup's place: block of query heads, KV head, sample, split (decode_grid has the orders).  Passes over the same rows and the
// workgroups of a group's query heads lie n_kv_heads times the splits apart: on one XCD where that is a multiple of 8.  (Next to each other
// they are on different ones: 40 of 500..1500 rows, 28 / 4 fp32 heads 55 us so, 66 then; 8 x 400, 32 / 8 one workgroup a query head 7.6, 9.9.)
struct DecodePlace { int hb, g, b, split; };
template <bool RAGGED>
__device__ __forceinline__ DecodePlace decode_place(const DecodeArgs& a)
{
    DecodePlace p;
    if (a.heads_first) {
        p.hb = blockIdx.x / a.n_kv_heads; p.g = blockIdx.x - p.hb * a.n_kv_heads;
        p.b = blockIdx.z; p.split = blockIdx.y;
        if constexpr (RAGGED)
            if ((a.splits & 1) == 0) p.split = (p.split + p.b + (p.b >> 2) + (p.b >> 3)) % a.splits;
    } else {
        p.hb = blockIdx.y / a.n_kv_heads; p.g = blockIdx.y - p.hb * a.n_kv_heads;
        p.b = blockIdx.z; p.split = blockIdx.x;
    }
    return p;
}

// WAVES: wavefronts of a workgroup (kDecWaves, or a wide one's)
template <bool BF16, int HG, int LPR, int WAVES, typename TABLE>
__global__ __launch_bounds__(WAVES * kWave) void decode_partial_kernel(DecodeArgs a, TABLE t)
{
    constexpr bool RAGGED = std::is_same<TABLE, DecodeTable>::value;
    constexpr int E = BF16 ? 8 : 4;       // elements per 16-byte chunk
    constexpr int ESZ = BF16 ? 2 : 4;
    constexpr int RPS = kWave / LPR;      // cache rows per wavefront instruction
    constexpr int SLOTS = WAVES * RPS;   // independent softmax streams per workgroup
    extern __shared__ __attribute__((aligned(16))) float dec_lds[];
    constexpr int STATES = decode_states(LPR, WAVES);
    // of every state that meets in LDS: [HG][d] outputs, [HG] maxima, [HG] sums
    float* sm_o = dec_lds;
    float* sm_m = dec_lds + STATES * HG * a.head_dim;
    float* sm_l = sm_m + STATES * HG;

    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid >> 6;
    const int r = lane / LPR, c = lane % LPR;
    const bool chunk_live = c < a.cpr;
    const DecodePlace at = decode_place<RAGGED>(a);
    const int hb = at.hb, g = at.g;
    const int d = a.head_dim;
    const int b = at.b, split = at.split;
    int n_ctx = a.n_ctx, n_splits = a.splits;
    if constexpr (RAGGED) {
        n_ctx = t.ctx[b];
        if (split * a.keys_per_split >= n_ctx) return;
        n_splits = (n_ctx + a.keys_per_split - 1) / a.keys_per_split;
    }
    const int k0 = split * a.keys_per_split;
    const int k1 = min(k0 + a.keys_per_split, n_ctx);

    // the lane's chunk of every query head of the pass (heads past the group repeat the last one; never written)
    u32x4 qw[HG];
#pragma unroll
    for (int hh = 0; hh < HG; ++hh) {
        const int hg = min(hb * HG + hh, a.group - 1);
        const int64_t row = static_cast<int64_t>(b) * a.n_q_heads + g * a.group + hg;
        qw[hh] = u32x4{0u, 0u, 0u, 0u};
        if (chunk_live) qw[hh] = *reinterpret_cast<const u32x4*>(static_cast<const char*>(a.q) + (row * d + c * E) * ESZ);
    }
    const int64_t head_row0 = (static_cast<int64_t>(b) * a.n_kv_heads + g) * a.s_max;
    const char* kbase = static_cast<const char*>(a.kc) + (head_row0 * d + c * E) * ESZ;
    const char* vbase = static_cast<const char*>(a.vc) + (head_row0 * d + c * E) * ESZ;
    const int64_t row_bytes = static_cast<int64_t>(d) * ESZ;

    float m[HG], l[HG], acc[HG][E];
#pragma unroll
    for (int hh = 0; hh < HG; ++hh) {
        m[hh] = -INFINITY; l[hh] = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) acc[hh][e] = 0.f;
    }

    // Round: the workgroup's next SLOTS * U rows; slot (w, r) takes rows key0 + (u * WAVES + w) * RPS + r.  The
    // loads of the next round are issued before the current one is computed.
    u32x4 kq[kDecU], vq[kDecU], kn[kDecU], vn[kDecU];
    auto fetch = [&](int key0, u32x4* kd, u32x4* vd) {
#pragma unroll
        for (int u = 0; u < kDecU; ++u) {
            const int key = key0 + (u * WAVES + w) * RPS + r;
            kd[u] = u32x4{0u, 0u, 0u, 0u};
            vd[u] = u32x4{0u, 0u, 0u, 0u};
            if (key < k1 && chunk_live) {
                kd[u] = load_streaming(reinterpret_cast<const u32x4*>(kbase + key * row_bytes));
                vd[u] = load_streaming(reinterpret_cast<const u32x4*>(vbase + key * row_bytes));
            }
        }
    };
    fetch(k0, kn, vn);
    for (int key0 = k0; key0 < k1; key0 += SLOTS * kDecU) {
#pragma unroll
        for (int u = 0; u < kDecU; ++u) { kq[u] = kn[u]; vq[u] = vn[u]; }
        if (key0 + SLOTS * kDecU < k1) fetch(key0 + SLOTS * kDecU, kn, vn);
        float s[kDecU][HG];
#pragma unroll
        for (int u = 0; u < kDecU; ++u) {
            const int key = key0 + (u * WAVES + w) * RPS + r;
#pragma unroll
            for (int hh = 0; hh < HG; ++hh) {
                float part = 0.f;
                if constexpr (BF16) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) part = dot2_words(kq[u][e], qw[hh][e], part);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) part = fmaf(__uint_as_float(kq[u][e]), __uint_as_float(qw[hh][e]), part);
                }
                const float tot = row_sum<LPR>(part) * a.scale_log2;
                s[u][hh] = key < k1 ? tot : -INFINITY;
            }
        }
#pragma unroll
        for (int hh = 0; hh < HG; ++hh) {
            float m_new = m[hh];
#pragma unroll
            for (int u = 0; u < kDecU; ++u) m_new = fmaxf(m_new, s[u][hh]);
            const float m_use = m_new == -INFINITY ? 0.f : m_new;       // a slot that has met no row yet
            const float alpha = __builtin_amdgcn_exp2f(m[hh] - m_use);  // exp2(-inf) = 0 on the first rows
            float p[kDecU], psum = 0.f;
#pragma unroll
            for (int u = 0; u < kDecU; ++u) { p[u] = __builtin_amdgcn_exp2f(s[u][hh] - m_use); psum += p[u]; }
            l[hh] = l[hh] * alpha + psum;
            m[hh] = m_new;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                float o = acc[hh][e] * alpha;
#pragma unroll
                for (int u = 0; u < kDecU; ++u) {
                    float ve;
                    if constexpr (BF16) ve = (e & 1) ? __uint_as_float(vq[u][e >> 1] & 0xFFFF0000u) : __uint_as_float(vq[u][e >> 1] << 16);
                    else ve = __uint_as_float(vq[u][e]);
                    o = fmaf(p[u], ve, o);
                }
                acc[hh][e] = o;
            }
        }
    }

    int state = w * RPS + r;
    bool writes = true;
    if constexpr (STATES == WAVES) {                           // a wavefront's slots meet in registers first
#pragma unroll
        for (int hh = 0; hh < HG; ++hh) {
            const float mw = slots_max<LPR>(m[hh]);
            const float f = m[hh] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[hh] - mw);
            m[hh] = mw;
            l[hh] = slots_sum<LPR>(l[hh] * f);
#pragma unroll
            for (int e = 0; e < E; ++e) acc[hh][e] = slots_sum<LPR>(acc[hh][e] * f);
        }
        state = w;
    }
    // the workgroup's states meet in LDS
#pragma unroll
    for (int hh = 0; hh < HG; ++hh) {
        if constexpr (STATES == WAVES) writes = hh % RPS == r;   // (every slot holds the sums: slot r writes heads r, r + RPS, ...)
        if (writes && c == 0) { sm_m[state * HG + hh] = m[hh]; sm_l[state * HG + hh] = l[hh]; }
        if (writes && chunk_live) {
            float4* dst = reinterpret_cast<float4*>(sm_o + (state * HG + hh) * d + c * E);
#pragma unroll
            for (int e = 0; e < E; e += 4) dst[e / 4] = make_float4(acc[hh][e], acc[hh][e + 1], acc[hh][e + 2], acc[hh][e + 3]);
        }
    }
    __syncthreads();
    for (int i = tid; i < HG * d; i += WAVES * kWave) {
        const int hh = i / d, ch = i - hh * d;
        const int hg = hb * HG + hh;
        if (hg >= a.group) continue;
        float mx = sm_m[hh];
#pragma unroll
        for (int x = 1; x < STATES; ++x) mx = fmaxf(mx, sm_m[x * HG + hh]);
        float o = 0.f, lt = 0.f;
#pragma unroll
        for (int x = 0; x < STATES; ++x) {
            const float ms = sm_m[x * HG + hh];
            const float wgt = ms == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ms - mx);
            o = fmaf(wgt, sm_o[(x * HG + hh) * d + ch], o);
            lt = fmaf(wgt, sm_l[x * HG + hh], lt);
        }
        if (n_splits == 1) {
            const int64_t row = static_cast<int64_t>(b) * a.n_q_heads + g * a.group + hg;
            const float val = o / lt;                              // n_ctx >= 1: at least one row was met
            if constexpr (BF16) static_cast<__bf16*>(a.out)[row * d + ch] = static_cast<__bf16>(val);
            else static_cast<float*>(a.out)[row * d + ch] = val;
        } else {
            const int64_t row = static_cast<int64_t>(b) * a.n_q_heads + g * a.group + hg;
            float* dst = a.ws + (row * a.splits + split) * (d + 2);
            if (ch == 0) { dst[0] = mx; dst[1] = lt; }
            dst[2 + ch] = o;
        }
    }
}

// The same for bf16 caches with head_dim <= 128 and at least three query heads per KV head, on the matrix cores: all query heads
// of a KV head (up to 16 per pass) are the columns of one MFMA tile, so the vector work per cache row no longer grows with the
// heads, and a workgroup that has little context gets through it in a few memory latencies.  (Per 64 rows of 128 channels and
// four heads the kernel above needs about 450 vector instructions a wavefront and 1.4 us; bound by that, not by memory, whenever
// a workgroup runs alone.)
//   - A wavefront takes 32 keys a step.  K rows are read as they lie (lane = key, 16-byte chunks of the row in any order that Q
//     shares) and are the first operand of v_mfma_f32_16x16x32_bf16.  The two 16-key tiles of a step hold keys 8 a + r and
//     8 a + 4 + r in row 4 a + r: a lane then owns the logits of 8 consecutive keys of one head, which is the second operand
//     of O^T += V^T P^T as it stands.
//   - V^T rows may be any permutation of the channels: a lane reads channels 8 i .. 8 i + 7 of its 8 keys, 16 bytes each, and
//     v_perm gathers 8 operands (channel 8 i + j of the 8 keys) out of them: no LDS, no transposed copy.
//   - Weights enter as sums of three bf16 terms, which hold every bit of the fp32 weight (two hold 16: the results then differ
//     from the rounded exact ones four times as often as with fp32 weights).  The third costs 8 MFMAs a step, which memory hides,
//     and registers, which scalar base addresses gave back (with vector ones 20 were spilled: 64 samples of 117..3584 rows 99 us).
//   - Each wavefront runs its own online softmax; the states meet in LDS at the end.
// Against the kernel above (us): 64 x 938 rows, 32 / 8 heads 45.5 -> 40.9 (6.0 TB/s); 64 x 3584 154 -> 140 (6.7 TB/s); 4 x 938
// 10.6 -> 9.0; 16 x 2000 with 64 / 8 heads 43.8 -> 27.7, 32 x 2000 with 32 / 2 43.8 -> 19.6.  With one or two heads the vector
// work is less than the gathering here (32 x 1000, 16 / 16 heads of 64: 22.5 there, 26.0 here; 8 x 1280, 16 / 8 heads 12.8, 13.8),
// so those stay there.
template <int WAVES, typename TABLE>
__global__ __launch_bounds__(WAVES * kWave, 2) void decode_mfma_kernel(DecodeArgs a, TABLE tab)
{
    constexpr bool RAGGED = std::is_same<TABLE, DecodeTable>::value;
    constexpr int THREADS = WAVES * kWave, KT = 4;             // K chunks of 32 channels
    extern __shared__ __attribute__((aligned(16))) float dec_lds[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);    // (uniform for the compiler: loads take scalar base addresses)
    const int l16 = lane & 15, kq = lane >> 4;
    const DecodePlace place = decode_place<RAGGED>(a);
    const int hb = place.hb, g = place.g, b = place.b, split = place.split, d = a.head_dim;
    int n_ctx = a.n_ctx, n_splits = a.splits;
    if constexpr (RAGGED) {
        n_ctx = tab.ctx[b];
        if (split * a.keys_per_split >= n_ctx) return;
        n_splits = (n_ctx + a.keys_per_split - 1) / a.keys_per_split;
    }
    const int k0 = split * a.keys_per_split;
    const int k1 = min(k0 + a.keys_per_split, n_ctx);
    const int heads = min(16, a.group - 16 * hb);              // query heads of this pass
    // of every wavefront: [heads][d] outputs, [heads] maxima, [heads] sums
    float* const sm_o = dec_lds;
    float* const sm_m = dec_lds + WAVES * heads * d;
    float* const sm_l = sm_m + WAVES * heads;

    const uint32_t row_bytes = static_cast<uint32_t>(d) * 2;
    const int64_t first_row = (static_cast<int64_t>(b) * a.n_kv_heads + g) * a.s_max + k0;
    const char* const kbase = static_cast<const char*>(a.kc) + first_row * row_bytes;
    const char* const vbase = static_cast<const char*>(a.vc) + first_row * row_bytes;
    const int n_keys = k1 - k0;

    // Loads of the 32 keys from `key` on (relative to k0); keys past the end re-read the last one (their logits are masked)
    auto fetch = [&](int key_v, u32x4 (&kf)[2][KT], u32x4 (&vf)[8]) __attribute__((always_inline)) {
        const int key = __builtin_amdgcn_readfirstlane(key_v);
        const int last = n_keys - 1 - key;
        const char* const kb = kbase + static_cast<int64_t>(key) * row_bytes;
        const char* const vb = vbase + static_cast<int64_t>(key) * row_bytes;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const uint32_t off = static_cast<uint32_t>(min(8 * (l16 >> 2) + 4 * s + (l16 & 3), last)) * row_bytes;
#pragma unroll
            for (int t = 0; t < KT; ++t)
                if (32 * t < d) kf[s][t] = load_streaming(reinterpret_cast<const u32x4*>(kb + (off + (32 * t + 8 * kq < d ? 64 * t + 16 * kq : 0))));
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t off = static_cast<uint32_t>(min(8 * kq + e, last)) * row_bytes + (8 * l16 < d ? l16 * 16 : 0);
            vf[e] = load_streaming(reinterpret_cast<const u32x4*>(vb + off));
        }
    };
    u32x4 kf[2][2][KT], vf[2][8];
    const int step = 32 * WAVES;
    int key = 32 * w;
    if (key < n_keys) fetch(key, kf[0], vf[0]);
    // Q^T: channels 32 t + 8 kq .. + 7 of head l16
    dec_bf16x8 qf[KT];
    {
        const int64_t row = static_cast<int64_t>(b) * a.n_q_heads + g * a.group + hb * 16 + min(l16, heads - 1);
        const char* qb = static_cast<const char*>(a.q) + row * row_bytes + kq * 16;
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            u32x4 x = u32x4{0u, 0u, 0u, 0u};
            if (32 * t + 8 * kq < d) x = *reinterpret_cast<const u32x4*>(qb + 64 * t);
            qf[t] = __builtin_bit_cast(dec_bf16x8, x);
        }
    }
    dec_f32x4 o[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = dec_f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;                              // of head l16; l: the lane's own keys

    // logits (times log2 e) of the lane's keys 8 kq .. + 7 of the step at `at`, head l16; keys past the end -infinity
    auto logits = [&](int at, u32x4 (&ck)[2][KT], float (&z)[8]) __attribute__((always_inline)) {
        if ((d & 31) != 0) {                                    // lanes past the row hold a piece of its front: 0 x it has to be 0
#pragma unroll
            for (int t = 0; t < KT; ++t)
                if (32 * t < d && 32 * t + 32 > d) {
#pragma unroll
                    for (int x = 0; x < 2; ++x)
                        if (32 * t + 8 * kq >= d) ck[x][t] = u32x4{0u, 0u, 0u, 0u};
                }
        }
        dec_f32x4 s[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            s[x] = dec_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < KT; ++t)
                if (32 * t < d) s[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(dec_bf16x8, ck[x][t]), qf[t], s[x], 0, 0, 0);
        }
        const int lim = n_keys - at - 8 * kq;                   // the lane's keys below this exist
#pragma unroll
        for (int e = 0; e < 8; ++e) z[e] = e < lim ? s[e >> 2][e & 3] * a.scale_log2 : -INFINITY;
    };
    auto compute = [&](int at, u32x4 (&ck)[2][KT], u32x4 (&cv)[8]) __attribute__((always_inline)) {
        float p[8], m_new = m;
        logits(at, ck, p);
#pragma unroll
        for (int e = 0; e < 8; ++e) m_new = fmaxf(m_new, p[e]);
        m_new = slots_max<16>(m_new);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;   // every key so far has a logit of -infinity: weight 0
        if (__any(m_new != m)) {
            const float alpha = __builtin_amdgcn_exp2f(m - m_use);   // exp2(-inf) = 0 on the first step
            l *= alpha;
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) o[j][r] *= alpha;
            m = m_new;
        }
        u32x4 ph, pm, pl;                                       // the weights as sums of three bf16 terms: 24 bits, all of fp32's
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float p0 = __builtin_amdgcn_exp2f(p[2 * e] - m_use), p1 = __builtin_amdgcn_exp2f(p[2 * e + 1] - m_use);
            l += p0 + p1;
            const dec_bf16x2 hi = {static_cast<__bf16>(p0), static_cast<__bf16>(p1)};
            ph[e] = __builtin_bit_cast(uint32_t, hi);
            const float r0 = p0 - __uint_as_float(ph[e] << 16), r1 = p1 - __uint_as_float(ph[e] & 0xFFFF0000u);
            const dec_bf16x2 mid = {static_cast<__bf16>(r0), static_cast<__bf16>(r1)};
            pm[e] = __builtin_bit_cast(uint32_t, mid);
            const dec_bf16x2 lo = {static_cast<__bf16>(r0 - __uint_as_float(pm[e] << 16)),
                                   static_cast<__bf16>(r1 - __uint_as_float(pm[e] & 0xFFFF0000u))};
            pl[e] = __builtin_bit_cast(uint32_t, lo);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            u32x4 v;                                            // channel 8 l16 + j of keys 8 kq .. + 7
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t w0 = cv[2 * e][j >> 1], w1 = cv[2 * e + 1][j >> 1];
                v[e] = __builtin_amdgcn_perm(w1, w0, (j & 1) ? 0x07060302u : 0x05040100u);
            }
            o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(dec_bf16x8, v), __builtin_bit_cast(dec_bf16x8, ph), o[j], 0, 0, 0);
            o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(dec_bf16x8, v), __builtin_bit_cast(dec_bf16x8, pm), o[j], 0, 0, 0);
            o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(dec_bf16x8, v), __builtin_bit_cast(dec_bf16x8, pl), o[j], 0, 0, 0);
        }
    };
    // two steps per pass of the loop: the other buffer is in flight while one is computed
    while (key < n_keys) {
        if (key + step < n_keys) fetch(key + step, kf[1], vf[1]);
        compute(key, kf[0], vf[0]);
        key += step;
        if (key >= n_keys) break;
        if (key + step < n_keys) fetch(key + step, kf[0], vf[0]);
        compute(key, kf[1], vf[1]);
        key += step;
    }
    l = slots_sum<16>(l);
    // An infinity of V has met the trailing terms of its weight, or the weight of a key past the end (0 x infinity, infinity -
    // infinity): the wavefront's results are made again from the final maximum, one fp32 multiply-add per key that exists.
    float odd = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) odd = fmaf(o[j][r], 0.f, odd);
    if (__builtin_expect(__any(odd != 0.f), 0)) {
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = dec_f32x4{0.f, 0.f, 0.f, 0.f};
        const float m_use = m == -INFINITY ? 0.f : m;
#pragma unroll 1
        for (int at = 32 * w; at < n_keys; at += step) {
            float p[8];
            fetch(at, kf[0], vf[0]);
            logits(at, kf[0], p);
#pragma unroll
            for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(p[e] - m_use);
#pragma unroll 1
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float wgt = __shfl(p[e], 16 * x + l16, kWave);
                    const int key_at = at + 8 * x + e;
                    if (key_at < n_keys) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int ch = 8 * (4 * kq + r);
                            if (ch >= d) continue;
                            const u32x4 v = *reinterpret_cast<const u32x4*>(vbase + static_cast<int64_t>(key_at) * row_bytes + ch * 2);
#pragma unroll
                            for (int j = 0; j < 8; ++j)
                                o[j][r] = fmaf(wgt, (j & 1) ? __uint_as_float(v[j >> 1] & 0xFFFF0000u) : __uint_as_float(v[j >> 1] << 16), o[j][r]);
                        }
                    }
                }
        }
    }

    if (l16 < heads) {                                          // register r of o[j]: channel 8 (4 kq + r) + j
        if (kq == 0) { sm_m[w * heads + l16] = m; sm_l[w * heads + l16] = l; }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int ch = 8 * (4 * kq + r);
            if (ch < d) {
                float4* dst = reinterpret_cast<float4*>(sm_o + (w * heads + l16) * d + ch);
                dst[0] = make_float4(o[0][r], o[1][r], o[2][r], o[3][r]);
                dst[1] = make_float4(o[4][r], o[5][r], o[6][r], o[7][r]);
            }
        }
    }
    __syncthreads();
    const int half_d = d / 2;
    for (int i = tid; i < heads * half_d; i += THREADS) {
        const int hh = i / half_d, ch = (i - hh * half_d) * 2;
        float mx = sm_m[hh];
#pragma unroll
        for (int x = 1; x < WAVES; ++x) mx = fmaxf(mx, sm_m[x * heads + hh]);
        float o0 = 0.f, o1 = 0.f, lt = 0.f;
#pragma unroll
        for (int x = 0; x < WAVES; ++x) {                       // (a wavefront without a key of any weight: m = -inf)
            const float mw = sm_m[x * heads + hh], f = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - mx);
            const float2 v = *reinterpret_cast<const float2*>(sm_o + (x * heads + hh) * d + ch);
            o0 = fmaf(f, v.x, o0); o1 = fmaf(f, v.y, o1);
            lt = fmaf(f, sm_l[x * heads + hh], lt);
        }
        const int64_t row = static_cast<int64_t>(b) * a.n_q_heads + g * a.group + hb * 16 + hh;
        if (n_splits == 1) {
            const float inv = 1.0f / lt;
            const dec_bf16x2 val = {static_cast<__bf16>(o0 * inv), static_cast<__bf16>(o1 * inv)};
            *reinterpret_cast<dec_bf16x2*>(static_cast<__bf16*>(a.out) + row * d + ch) = val;
        } else {
            float* dst = a.ws + (row * a.splits + split) * (d + 2);
            if (ch == 0) *reinterpret_cast<float2*>(dst) = make_float2(mx, lt);
            *reinterpret_cast<float2*>(dst + 2 + ch) = make_float2(o0, o1);
        }
    }
}

// Combines the splits of one (batch item, query head): out = sum_s w_s o_s / sum_s w_s l_s, w_s = 2^(m_s - max m).
// Latency-bound (a few KB per workgroup), so everything that can be asked for at once is: a thread's first 8 partial outputs are
// requested together with the (max, sum) pairs, later ones 8 at a time whether or not 8 are left; beyond 8 splits two groups of
// threads take every other one.  (With what a division by 8 leaves fetched one by one, 4 x 938 rows took 12.6 us in 15 splits,
// 10.3 us in 8 of twice the length.)
constexpr int kDecMaxSplits = 1024;
template <bool BF16, int THREADS, int GROUPS, typename TABLE>
__global__ __launch_bounds__(THREADS) void decode_merge_kernel(const float* __restrict__ ws, void* __restrict__ out, int32_t splits,
                                                               int32_t d, int32_t n_q_heads, int32_t keys_per_split, TABLE t)
{
    constexpr int kWaves = THREADS / kWave, COLS = THREADS / GROUPS;
    __shared__ float wgt[kDecMaxSplits];
    __shared__ float red[2 * kWaves];
    __shared__ float meet[GROUPS > 1 ? THREADS : 1];
    const int64_t row = blockIdx.x;
    const float* src = ws + row * splits * (d + 2);
    if constexpr (std::is_same<TABLE, DecodeTable>::value) {   // a sample of one piece has its result already
        splits = (t.ctx[row / n_q_heads] + keys_per_split - 1) / keys_per_split;
        if (splits == 1) return;
    }
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
    const int x = tid % COLS, y = tid / COLS;                  // the thread's channel and group
    constexpr int kBatch = 8;
    float o_pre[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
        const int s = y + j * GROUPS;
        o_pre[j] = (s < splits && x < d) ? src[s * (d + 2) + 2 + x] : 0.f;
    }
    const float m_own = tid < splits ? src[tid * (d + 2)] : -INFINITY, l_own = tid < splits ? src[tid * (d + 2) + 1] : 0.f;
    float mloc = m_own;
    for (int s = tid + THREADS; s < splits; s += THREADS) mloc = fmaxf(mloc, src[s * (d + 2)]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mloc = fmaxf(mloc, __shfl_xor(mloc, off, kWave));
    if (lane == 0) red[wv] = mloc;
    __syncthreads();
    float mx = red[0];
#pragma unroll
    for (int i = 1; i < kWaves; ++i) mx = fmaxf(mx, red[i]);
    float lsum = 0.f;
    for (int s = tid; s < splits; s += THREADS) {
        const float ms = s == tid ? m_own : src[s * (d + 2)];
        const float wt = ms == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ms - mx);
        wgt[s] = wt;
        lsum = fmaf(wt, s == tid ? l_own : src[s * (d + 2) + 1], lsum);
    }
    lsum = wave_sum(lsum);
    if (lane == 0) red[kWaves + wv] = lsum;
    __syncthreads();
    float l_all = red[kWaves];
#pragma unroll
    for (int i = 1; i < kWaves; ++i) l_all += red[kWaves + i];
    const float inv = 1.0f / l_all;
    for (int c0 = 0; c0 < d; c0 += COLS) {
        const int ch = c0 + x;
        float o[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int s = y + j * GROUPS;
            const float v = c0 == 0 ? o_pre[j] : (s < splits && ch < d) ? src[s * (d + 2) + 2 + ch] : 0.f;
            o[j] = s < splits ? wgt[s] * v : 0.f;
        }
        for (int s0 = kBatch * GROUPS; s0 < splits; s0 += kBatch * GROUPS) {
            float v[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const int s = s0 + y + j * GROUPS;
                v[j] = (s < splits && ch < d) ? src[s * (d + 2) + 2 + ch] : 0.f;
            }
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const int s = s0 + y + j * GROUPS;
                if (s < splits) o[j] = fmaf(wgt[s], v[j], o[j]);
            }
        }
        float val = ((o[0] + o[1]) + (o[2] + o[3])) + ((o[4] + o[5]) + (o[6] + o[7]));
        if constexpr (GROUPS > 1) {                            // (one pass over the channels then: d <= COLS)
            meet[tid] = val;
            __syncthreads();
            if (y > 0) return;
#pragma unroll
            for (int i = 1; i < GROUPS; ++i) val += meet[i * COLS + x];
        }
        if (ch < d) {
            if constexpr (BF16) static_cast<__bf16*>(out)[row * d + ch] = static_cast<__bf16>(val * inv);
            else static_cast<float*>(out)[row * d + ch] = val * inv;
        }
    }
}

// Block shape and split count for these sizes (shared by the launch and the workspace query).
struct DecodePlan {
    bool mfma;
    int hg, lpr, head_blocks, round_keys;
    int waves;                           // of a workgroup: kDecWaves, or a wide one's
    bool wide_short, wide_full;          // where wide workgroups are the faster way: contexts short or even
    bool wide_heads;                     // the same with one for each query head, where wide_heads_pay as well
    int64_t heads_row_bytes, heads_most; // bytes that these read of a context row into all L2s, and what they may read (wide_heads_pay)
    int whole_keys;                      // contexts up to this are not cut
    // pieces of different contexts: whole samples from ragged_units pairs on; else no more than ragged_groups, or of ragged_keys rows
    int ragged_units, ragged_keys, ragged_groups;
    int32_t splits, keys_per_split;      // of one context length for all samples
    int32_t max_splits;                  // per sample, at most: what the workspace is sized for
    size_t ws_bytes, lds_bytes;
};

// Wavefronts of a wide workgroup: as many as the registers of a unit hold.
static int decode_wide_waves(const DecodePlan& p) { return !p.mfma && p.hg <= 2 ? 16 : 8; }

static size_t decode_lds(const DecodePlan& p, int32_t head_dim)
{
    return sizeof(float) * (p.mfma ? p.waves : decode_states(p.lpr, p.waves)) * static_cast<size_t>(p.hg) * (head_dim + 2);
}

// Where 192 to 256 workgroups that take a whole context each are not the faster way after all; p->splits is what the contexts would be
// cut into otherwise (us, cut and whole).
//   - one or two heads a pass, samples of different length, as many pairs as units: these are not cut anyway, and narrow workgroups
//     are the better ones (32 samples, 16 / 8 heads of 128: of 300..600 rows 14.2, 15.1, of 1000..1300 27.8, 30.2; 28 samples 28.0, 27.0)
//   - 4 and more heads a pass on the vector units are bound by their instructions, and 192 workgroups leave a quarter of the units
//     without any: with one length from some length on (48 x 2000 rows, 32 / 4 fp32 heads 98, 108; 48 x 800 50.9, 47.4, but 51 x 2500
//     143, 135; 24 x 2500, 32 / 8 bf16 heads of 256 89, 95; 24 x 1500 fp32 of 128 53.5, 51.0; 12 x 1500, 56 / 8 45.2, 48.0; 48 of
//     300..600, 32 / 4 of 128 35.6, 37.6, but of 64 23.3, 19.9, and 24 of 300..600, 32 / 8 25.0, 24.1)
//   - two passes over the same rows, n_kv_heads times the splits apart in the grid (decode_place): cut they may meet on an XCD, whole
//     they do only if n_kv_heads is a multiple of 8 (24 x 2500, 28 / 4 fp32 heads 76, 85 and 32 x 2500 86, 103, in 6 and 4 splits; 28 x 2500
//     103, 90, in 5; 24 x 800 33.1, 30.3, but 31 x 500 23.4, 24.7; samples of different length 26 of 600..900 36.9, 32.9, of 1600..2000 59.9, 66.9)
static bool wide_full_pays(const DecodePlan& p, int64_t units, int64_t n_ctx, int32_t n_kv_heads, bool ragged)
{
    if (p.mfma) return true;
    if (p.hg <= 2) return !ragged || units < kDecRaggedUnits;
    if (ragged) return (units >= 200 || p.hg == 4 || p.lpr <= 16) && (p.head_blocks == 1 || n_ctx <= 900);
    if (p.hg == 4 && p.head_blocks > 1 && n_kv_heads % 8 != 0)
        return static_cast<int64_t>(n_kv_heads) * p.splits % 8 != 0 || (n_ctx <= 800 && units <= 240);
    return units >= 200 || n_ctx <= (p.hg > 4 ? 800 : p.head_blocks == 1 ? 1500 : 700);
}

// Workgroups of one query head each read their KV head's rows as often as there are heads.  A group's workgroups lie n_kv_heads apart
// in the grid, so they are on one XCD, and all but the first read from its L2, only where n_kv_heads is a multiple of 8; else every XCD
// of the 8 / gcd(n_kv_heads, 8) that have some of them fetches the rows, and above a number of bytes that costs more than a launch
// saves (us, first for caches that the passes find in the last-level cache, then for such as they do not; cut and so: 16 x 300 rows, 16
// / 1 bf16 heads 10.1 / 10.5, 8.4 / 10.0, 8 x 512, 8 / 1 9.2 / 9.5, 8.8 / 11.0, but 16 x 420 9.8 / 10.5, 8.9 / 11.7 and 32 x 300, 8 / 1
// 9.4 / 9.6, 9.8 / 12.0; in fp32 16 x 270, 16 / 4 11.8 / 12.7, 9.4 / 11.2, but 16 x 384 12.0 / 13.4, 12.4 / 13.8 and 64 x 270, 4 / 1
// 11.9 / 12.7, 12.9 / 15.6; samples of different length, which take longer cut: 16 of 100..500, 16 / 1 12.3 / 13.1, 10.1 / 11.8, but of
// 500..768 12.3 / 13.3, 14.0 / 15.7, and 8 of 500..768, 32 / 4 10.2 / 10.5, 10.8 / 12.2).
static bool wide_heads_pay(const DecodePlan& p, int64_t rows) { return p.wide_heads && rows * p.heads_row_bytes <= p.heads_most; }

static void go_wide(DecodePlan* p, bool heads, int32_t longest, int32_t head_dim, int group)
{
    if (heads) { p->mfma = false; p->hg = 1; p->head_blocks = group; }
    p->waves = decode_wide_waves(*p);
    p->splits = 1;
    p->keys_per_split = longest;
    p->lds_bytes = decode_lds(*p, head_dim);
}

static int decode_plan(int dtype, int32_t batch, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, int64_t n_ctx,
                       DecodePlan* p, bool ragged = false)
{
    const int esz = dtype_size(dtype);
    if (!esz || batch < 0 || n_q_heads <= 0 || n_kv_heads <= 0 || head_dim <= 0 || n_ctx < 0) return CIVIC_ERR_INVALID_ARG;
    if (n_q_heads % n_kv_heads) return CIVIC_ERR_INVALID_ARG;
    if ((static_cast<int64_t>(head_dim) * esz) % 16) return CIVIC_ERR_INVALID_ARG;
    const int cpr = head_dim * esz / 16;
    if (cpr > kWave || n_ctx > INT32_MAX || batch > 65535) return CIVIC_ERR_UNSUPPORTED;
    const int group = n_q_heads / n_kv_heads;
    p->mfma = dtype == CIVIC_BF16 && head_dim <= 128 && group > 2;
    // blocks of the vector kernel's 1, 2, 4 or 8 heads: the limit on the sizes and the workspace go by them, whichever kernel runs
    const int vec_heads = group >= 8 ? 8 : group > 2 ? 4 : group, vec_blocks = (group + vec_heads - 1) / vec_heads;
    if (static_cast<int64_t>(n_kv_heads) * vec_blocks > 65535) return CIVIC_ERR_UNSUPPORTED;
    p->hg = p->mfma ? std::min(group, 16) : vec_heads;          // query heads per pass
    p->head_blocks = (group + p->hg - 1) / p->hg;
    p->lpr = 8;
    while (p->lpr < cpr) p->lpr *= 2;
    const int64_t units = static_cast<int64_t>(batch > 0 ? batch : 1) * n_kv_heads * p->head_blocks;
    const int64_t round_keys = p->mfma ? 32 * kDecWaves : static_cast<int64_t>(kDecWaves) * (kWave / p->lpr) * kDecU;
    const bool heavy = !p->mfma && p->hg > 4;                  // 8 heads on the vector units: a round is long, two workgroups fill a unit
    const int64_t whole_keys = round_keys * (p->mfma || heavy ? 2 : 4);
    p->round_keys = static_cast<int>(round_keys);
    // whole rounds per split, no split shorter than one round
    auto cut = [&](int64_t splits, int64_t round, int32_t* n, int32_t* keys) {
        const int64_t max_splits = (n_ctx + round - 1) / round;
        splits = std::max<int64_t>(std::min(std::min(splits, max_splits), static_cast<int64_t>(kDecMaxSplits)), 1);
        int64_t kps = (n_ctx + splits - 1) / splits;
        kps = std::max((kps + round - 1) / round * round, round);
        *n = static_cast<int32_t>(n_ctx > 0 ? (n_ctx + kps - 1) / kps : 1);
        *keys = static_cast<int32_t>(kps);
    };
    // What the workspace has room for: about four workgroups per compute unit, in rounds of the vector kernel (the size decides
    // which calls civic_decode_attn_noalloc takes).  What is launched below is never more: at most 512 or 256 workgroups, of at
    // most twice the heads, in rounds as long or longer.  And the pieces of a ragged launch.
    int32_t unused;
    const int64_t room_units = static_cast<int64_t>(batch > 0 ? batch : 1) * n_kv_heads * vec_blocks;
    cut((1024 + room_units - 1) / room_units, static_cast<int64_t>(kDecWaves) * (kWave / p->lpr) * kDecU, &p->max_splits, &unused);
    p->ragged_keys = p->mfma || heavy ? kDecRaggedKeys : kDecVecRaggedKeys;
    p->ragged_groups = p->mfma || heavy ? 512 : 1024;
    p->ragged_units = heavy ? kDecFullUnits : kDecRaggedUnits;
    if (ragged) {
        const int64_t pieces = std::max<int64_t>(p->max_splits, (n_ctx + p->ragged_keys - 1) / p->ragged_keys);
        p->max_splits = static_cast<int32_t>(std::min<int64_t>(pieces, kDecMaxSplits));
    }
    // What is launched: nothing to combine once the (item, KV head) pairs fill the chip by themselves (64 x 938 rows, 8 KV
    // heads: one split 45.5 us, two 52; 64 x 3584: 153 against 172); otherwise two workgroups per unit in at most 8 splits, which
    // one trip of the combining launch reads (16 x 938: 4 splits 18.7 us, 8 splits 20.8; 4 x 938: 8 splits 10.3 us, 15 splits
    // 12.6), or one per unit in more (1 x 3584: 28 splits 11.9 us, 57 splits 13.0, 8 splits 16).  Nor is a context cut that one
    // workgroup gets through before a second launch would have started (1 x 256 rows, 32 / 8 heads: 7.0 us whole, 7.8 in two).
    p->whole_keys = static_cast<int>(whole_keys);
    // The vector kernel with 4 or 8 heads a pass is bound by its instructions and takes more workgroups per unit: 4 splits (74 x 968
    // rows, 16 / 4 fp32 heads of 96: 63 us in one, 49 in four; 22 x 392, 32 / 8 of 128: 22.5 in two, 21.3 in four), or 8 where
    // several passes read the same rows, which then run on one XCD (decode_place) and share its L2 (24 x 2500, 28 / 4
    // of 128: 93 us in two, 65 in eight).  As long as a split is two rounds, and the workspace has the room (there 6, 75 us).
    int64_t wanted = units >= kDecFullUnits || n_ctx <= whole_keys ? 1 : std::max(std::min<int64_t>(512 / units, 8), 256 / units);
    // The same 4 where the matrix cores would run one workgroup on most units and two on some through a long context (80 x 2918
    // rows, 16 / 4 heads of 72, 320 pairs: 87 us in one, 74 in four).
    const int64_t busy = !p->mfma && p->head_blocks > 1 ? 8 : 4, shortest = (p->mfma ? 8 : 2 * busy) * round_keys;
    const bool more = p->mfma ? units > 256 : p->hg > 2;
    if (more && wanted < busy && units < kDecFullUnits && n_ctx > whole_keys && n_ctx >= shortest)
        wanted = std::min<int64_t>(busy, (1024 + room_units - 1) / room_units);
    cut(wanted, round_keys, &p->splits, &p->keys_per_split);
    p->ws_bytes = p->max_splits > 1 ? sizeof(float) * static_cast<size_t>(batch) * n_q_heads * p->max_splits * (head_dim + 2) : 0;
    p->waves = kDecWaves;
    p->lds_bytes = decode_lds(*p, head_dim);
    // Wide workgroups and one split, where contexts would be cut (us, as it was and so):
    //   - up to 256 query heads with three rounds of 16 wavefronts or less: a workgroup for each of them, which is bound by its
    //     instructions and through before a second launch would have started (1 x 469 rows, 16 / 8 heads of 128 8.9, 6.4, and 9.5, 8.1 for
    //     caches that no pass has touched before; 8 x 300, 32 / 8 of 64 in fp32 10.6, 7.4).  Two rounds where matrix cores would take contexts
    //     of one length (8 x 512, 32 / 8 9.0, 7.9 and untouched 9.8, 9.5, but 8 x 768 10.4, 9.8 and 11.9, 13.1; 8 of 500..768 12.2, 10.1 and
    //     13.1, 12.3), and where one pass over the rows would do for a single KV head's 4 or 8 heads (8 x 384, 8 / 1 in fp32 12.1, 12.7
    //     and untouched 12.6, 14.3).  With 4 or 8 heads on the vector units contexts need not be cut for that (1 x 130, 32 / 4 fp32 heads 11.9, 7.1).
    //   - matrix cores, up to 128 pairs with 5 / 4 rounds of 8 wavefronts (16 x 300, 32 / 8 10.2, 8.5; 8 x 400 9.2, 10.2)
    //   - 192 to 256 pairs (of them and passes) up to 3072 rows: one such workgroup to a unit reads at its rate and nothing is left to
    //     combine (24 x 600 rows, 32 / 8 heads of 128 19.5, 14.4; 60 x 1200, 28 / 4 30.8, 26.7; 28 x 2400, 16 / 8 fp32 of 64 45.3, 43.2;
    //     32 x 2400, 16 / 8 of 128 53.1, 51.1, but of 4000 85, 90; 160 pairs: 20 x 1200, 16 / 8 19.7, 20.7)
    // (wide_full_pays has where the third does not hold)
    const bool cut_up = n_ctx > whole_keys;
    const int spread = std::min(group, n_kv_heads % 8 == 0 ? 1 : n_kv_heads % 4 == 0 ? 2 : n_kv_heads % 2 == 0 ? 4 : 8);
    p->heads_row_bytes = static_cast<int64_t>(2) * n_kv_heads * head_dim * esz * spread;
    const int64_t rounds = (n_ctx + 16 * (kWave / p->lpr) * kDecU - 1) / (16 * (kWave / p->lpr) * kDecU);
    p->heads_most = spread == 1 ? INT64_MAX : !p->mfma ? 44000000 : !ragged ? 20000000 : rounds <= 2 ? 24000000 : 12000000;
    p->wide_heads = static_cast<int64_t>(batch) * n_q_heads <= 256 && (cut_up || (p->hg > 2 && !p->mfma && n_ctx > round_keys)) &&
                    rounds <= ((p->mfma ? !ragged : spread == 8 && p->head_blocks == 1) ? 2 : 3);
    p->wide_short = p->mfma && cut_up && units <= 128 && n_ctx <= 5 * 32 * 8 / 4;
    p->wide_full = cut_up && units >= 192 && units <= 256 && n_ctx <= 3072 && wide_full_pays(*p, units, n_ctx, n_kv_heads, ragged);
    if (!ragged) {
        const bool heads = wide_heads_pay(*p, static_cast<int64_t>(batch) * n_ctx);
        if (heads || p->wide_short || p->wide_full) go_wide(p, heads, static_cast<int32_t>(n_ctx), head_dim, group);
    }
    return CIVIC_OK;
}

// How samples of different context lengths are cut into pieces of one length (the last piece of a sample is what is left):
//   - not at all when the pairs fill the chip and the longest context is within 448 rows of the average: its workgroups then
//     outlast the others by less than a second launch costs (96 samples of 100..800 rows: 41 us, 45-50 us cut; from 256
//     pairs on: 40 samples of 152..300, 32 / 8 heads 13.2 us, 16.2-19.3 cut; 40 of 85..600, 16 / 8 heads 16.3, 17.7-24.5 cut)
//   - else into the shortest pieces that make at most 512 workgroups, or pieces of 512 rows if that takes longer ones
//     (64 samples of 117..3584 rows, 8 KV heads: 97 us; 118 us in pieces of 128, 103 of 1024, 129 uncut; the same grid for
//     every sample, laid out for the longest context, took 133 us, half of its workgroups with nothing to do)
//   - the vector kernel with up to 4 heads a pass into at most 1024 workgroups, or pieces of 256 rows (64 samples of 345..2500,
//     16 / 4 fp32 heads of 96: 63 us, 69 in pieces of 512; 24 of 345..2500, 16 / 8 bf16 heads of 128: 28.0, 30.5; 17 of 57..457:
//     10.1, 11.2), but no more than 512 of a single round of 32 rows.  (With 8 heads a pass 512 as well, and whole samples from
//     384 pairs on only: 80 of 694..1388, 32 / 4 fp32 heads of 64 58 us, 69 in 1024 or whole.)
// Never more pieces per sample than the workspace holds, max_splits.
static void cut_ragged(const int32_t* ctx_of, int32_t batch, int64_t units, int32_t head_dim, int group, DecodePlan* p)
{
    int64_t rows = 0;
    int32_t longest = 0;
    for (int32_t i = 0; i < batch; ++i) { rows += ctx_of[i]; longest = std::max(longest, ctx_of[i]); }
    const bool heads = wide_heads_pay(*p, rows);
    if (heads || p->wide_short || (p->wide_full && longest - rows / batch <= kDecTailKeys)) return go_wide(p, heads, longest, head_dim, group);
    const int64_t per_sample = units / batch;
    int64_t kps = p->round_keys;
    if (longest <= p->whole_keys || (units >= p->ragged_units && longest - rows / batch <= kDecTailKeys)) kps = longest;
    for (;; kps += p->round_keys) {                           // (ends: a piece as long as the longest context is one per sample)
        const int64_t most = (longest + kps - 1) / kps;
        if (most > p->max_splits) continue;
        int64_t pieces = 0;
        for (int32_t i = 0; i < batch; ++i) pieces += (ctx_of[i] + kps - 1) / kps;
        if (pieces * per_sample <= (kps < 64 ? 512 : p->ragged_groups) || kps >= p->ragged_keys) break;
    }
    p->keys_per_split = static_cast<int32_t>(kps);
    p->splits = static_cast<int32_t>((longest + kps - 1) / kps);
}

// Order of the workgroups.  The hardware hands consecutive ones to the eight XCDs in turn, and an XCD's to its units.  With the splits
// innermost an even number of them puts the last pieces of all samples on the same XCDs, and of samples of different length these are
// the ones that do not exist: the other XCDs have more of the work.  So the heads are innermost, then the splits; and since 32 units
// would see the same split of every few samples where their number is even, each sample begins with another one then (us, splits
// innermost, heads innermost, and with a split of its own: 24 samples of 100..2000 rows, 32 / 8 heads of 128 38.9, 38.0, 27.2; 80 of
// 60..4000, 28 / 4 99.8, 96.9, 71.0; 24 of 100..2000, 16 / 8 fp32 51.5, 41.2, 39.2; five splits, 40 of 85..2500 48.0, 47.3, 50.5; seven, 64 of
// 117..3584 91.6, 89.1, 90.6).  The samples outermost: with the splits there a first pass over caches that were not touched before took
// 132 us instead of 119 (64 of 117..3584).
// Where several passes read the same rows the splits stay innermost: a power of two of them keeps the passes on one XCD, where they
// share its L2 (40 x 1000, 28 / 4 fp32 heads of 128 52.0, 68.9 with the heads innermost; 40 of 500..1500 55.2, 63.5).
static bool decode_heads_first(const DecodePlan& p) { return p.head_blocks == 1 && p.splits > 1; }

static dim3 decode_grid(const DecodeArgs& a, const DecodePlan& p)
{
    const unsigned heads = static_cast<unsigned>(a.n_kv_heads * p.head_blocks), batch = static_cast<unsigned>(a.batch), splits = static_cast<unsigned>(p.splits);
    return a.heads_first ? dim3(heads, splits, batch) : dim3(splits, heads, batch);
}

template <bool BF16, int HG, int LPR, int WAVES, typename TABLE>
static int launch_decode_waves(const DecodeArgs& a, const TABLE& t, const DecodePlan& p, hipStream_t s)
{
    const dim3 grid = decode_grid(a, p);
    if (p.lds_bytes > 64 * 1024) {
        static std::atomic<uint64_t> allowed{0};
        // (of the widest rows: the limit is set once for all launches of the instance)
        constexpr size_t most = sizeof(float) * decode_states(LPR, WAVES) * HG * (LPR * (BF16 ? 8 : 4) + 2);
        const int rc = allow_dynamic_lds(reinterpret_cast<const void*>(decode_partial_kernel<BF16, HG, LPR, WAVES, TABLE>), most, &allowed);
        if (rc != CIVIC_OK) return rc;
    }
    civic::launch((decode_partial_kernel<BF16, HG, LPR, WAVES, TABLE>), grid, dim3(WAVES * kWave), p.lds_bytes, s, a, t);
    return check_launch();
}

template <bool BF16, int HG, int LPR, typename TABLE>
static int launch_decode_kernel(const DecodeArgs& a, const TABLE& t, const DecodePlan& p, hipStream_t s)
{
    return p.waves == kDecWaves ? launch_decode_waves<BF16, HG, LPR, kDecWaves>(a, t, p, s)
                                : launch_decode_waves<BF16, HG, LPR, HG <= 2 ? 16 : 8>(a, t, p, s);   // (decode_wide_waves)
}

template <bool BF16, int HG, typename TABLE>
static int launch_decode_lpr(const DecodeArgs& a, const TABLE& t, const DecodePlan& p, hipStream_t s)
{
    if constexpr (!BF16 || HG <= 2) {                           // (bf16 rows of up to 16 chunks with more heads: the matrix cores)
        if (p.lpr == 8) return launch_decode_kernel<BF16, HG, 8>(a, t, p, s);
        if (p.lpr == 16) return launch_decode_kernel<BF16, HG, 16>(a, t, p, s);
    }
    switch (p.lpr) {
        case 32: return launch_decode_kernel<BF16, HG, 32>(a, t, p, s);
        case 64: return launch_decode_kernel<BF16, HG, 64>(a, t, p, s);
        default: return CIVIC_ERR_UNSUPPORTED;
    }
}

template <bool BF16, typename TABLE>
static int launch_decode(const DecodeArgs& a, const TABLE& t, const DecodePlan& p, hipStream_t s)
{
    int rc;
    if (p.mfma) {
        const dim3 grid = decode_grid(a, p);
        if (p.waves == kDecWaves) {
            static_assert(sizeof(float) * kDecWaves * 16 * (128 + 2) <= 64 * 1024, "no launch needs more LDS than every launch may have");
            civic::launch((decode_mfma_kernel<kDecWaves, TABLE>), grid, dim3(kDecThreads), p.lds_bytes, s, a, t);
        } else {
            if (p.lds_bytes > 64 * 1024) {
                static std::atomic<uint64_t> allowed{0};
                rc = allow_dynamic_lds(reinterpret_cast<const void*>(decode_mfma_kernel<8, TABLE>), sizeof(float) * 8 * 16 * (128 + 2), &allowed);
                if (rc != CIVIC_OK) return rc;
            }
            civic::launch((decode_mfma_kernel<8, TABLE>), grid, dim3(8 * kWave), p.lds_bytes, s, a, t);
        }
        rc = check_launch();
    } else switch (p.hg) {
        case 1: rc = launch_decode_lpr<BF16, 1>(a, t, p, s); break;
        case 2: rc = launch_decode_lpr<BF16, 2>(a, t, p, s); break;
        case 4: rc = launch_decode_lpr<BF16, 4>(a, t, p, s); break;
        default: rc = launch_decode_lpr<BF16, 8>(a, t, p, s);
    }
    if (rc != CIVIC_OK || p.splits == 1) return rc;
    const dim3 rows(static_cast<unsigned>(a.batch) * static_cast<unsigned>(a.n_q_heads));
#define CIVIC_DEC_MERGE(T, G) civic::launch((decode_merge_kernel<BF16, T, G, TABLE>), rows, dim3(T), 0, s, a.ws, a.out, p.splits, a.head_dim, \
                                            a.n_q_heads, p.keys_per_split, t)
    if (p.splits <= 8) CIVIC_DEC_MERGE(128, 1);
    else if (a.head_dim <= 128) CIVIC_DEC_MERGE(256, 2);
    else CIVIC_DEC_MERGE(256, 1);
#undef CIVIC_DEC_MERGE
    return check_launch();
}

// Everything but the choice of the workspace: `ws` holds at least plan.ws_bytes when the plan splits.
static int decode_attn(const void* q, const void* k_cache, const void* v_cache, void* out, int dtype, int32_t batch,
                       int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, int64_t s_max, int64_t n_ctx,
                       float softmax_scale, const DecodePlan& p, float* ws, void* stream, const int32_t* ctx_of = nullptr)
{
    DecodeArgs a;
    a.q = q; a.kc = k_cache; a.vc = v_cache; a.out = out; a.ws = ws;
    a.s_max = s_max;
    a.batch = batch; a.n_q_heads = n_q_heads; a.n_kv_heads = n_kv_heads; a.head_dim = head_dim;
    a.group = n_q_heads / n_kv_heads; a.head_blocks = p.head_blocks;
    a.n_ctx = static_cast<int32_t>(n_ctx); a.splits = p.splits; a.keys_per_split = p.keys_per_split;
    a.cpr = head_dim * dtype_size(dtype) / 16;
    const float scale = softmax_scale > 0.f ? softmax_scale : 1.0f / std::sqrt(static_cast<float>(head_dim));
    a.scale_log2 = scale * 1.4426950408889634f;
    hipStream_t s = static_cast<hipStream_t>(stream);
    a.heads_first = decode_heads_first(p);
    if (!ctx_of) return dtype == CIVIC_BF16 ? launch_decode<true>(a, NoTable{}, p, s) : launch_decode<false>(a, NoTable{}, p, s);
    DecodePlan pr = p;
    cut_ragged(ctx_of, batch, static_cast<int64_t>(batch) * n_kv_heads * p.head_blocks, head_dim, a.group, &pr);
    a.head_blocks = pr.head_blocks;
    a.heads_first = decode_heads_first(pr);
    a.keys_per_split = pr.keys_per_split;
    a.splits = pr.splits;
    DecodeTable t;
    for (int i = 0; i < kDecRaggedItems; ++i) t.ctx[i] = i < batch ? ctx_of[i] : 0;
    return dtype == CIVIC_BF16 ? launch_decode<true>(a, t, pr, s) : launch_decode<false>(a, t, pr, s);
}

// Argument checks shared by the two entry points (all before any HIP call).  CIVIC_OK with *nothing = true when
// there is no row to compute.
static int decode_check(const void* q, const void* k_cache, const void* v_cache, void* out, int dtype, int32_t batch,
                        int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, int64_t s_max, int64_t n_ctx,
                        float softmax_scale, DecodePlan* p, bool* nothing, bool ragged = false)
{
    *nothing = false;
    const int rc = decode_plan(dtype, batch, n_q_heads, n_kv_heads, head_dim, n_ctx, p, ragged);
    if (rc != CIVIC_OK) return rc;
    if (s_max < 0 || n_ctx > s_max) return CIVIC_ERR_INVALID_ARG;
    if (!(softmax_scale >= 0.f) || std::isinf(softmax_scale)) return CIVIC_ERR_INVALID_ARG;
    if (batch == 0) { *nothing = true; return CIVIC_OK; }
    if (n_ctx < 1) return CIVIC_ERR_INVALID_ARG;                 // a softmax over no row has no value
    if (!q || !k_cache || !v_cache || !out) return CIVIC_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(out)) return CIVIC_ERR_INVALID_ARG;
    return CIVIC_OK;
}

}  // namespace civic

// For tests, on the host alone (no part of civic.h): how a launch is taken, of one context length n_ctx[0] for all samples or, `ragged`,
// of n_ctx[i] each.  shape: wavefronts of a workgroup, query heads a pass, passes, splits, whether on the matrix cores.
extern "C" int civic_decode_shape(int dtype, int32_t batch, const int32_t* n_ctx, int32_t ragged, int32_t n_q_heads, int32_t n_kv_heads,
                                  int32_t head_dim, int32_t* shape)
{
    using namespace civic;
    if (batch < 1 || batch > kDecRaggedItems || !n_ctx || !shape) return CIVIC_ERR_INVALID_ARG;
    DecodePlan p;
    const int32_t longest = ragged ? *std::max_element(n_ctx, n_ctx + batch) : n_ctx[0];
    const int rc = decode_plan(dtype, batch, n_q_heads, n_kv_heads, head_dim, longest, &p, ragged != 0);
    if (rc != CIVIC_OK) return rc;
    if (ragged) cut_ragged(n_ctx, batch, static_cast<int64_t>(batch) * n_kv_heads * p.head_blocks, head_dim, n_q_heads / n_kv_heads, &p);
    shape[0] = p.waves; shape[1] = p.hg; shape[2] = p.head_blocks; shape[3] = p.splits; shape[4] = p.mfma ? 1 : 0;
    return CIVIC_OK;
}

namespace civic {

// ------------------------------------------------------------------------------ no allocation at all
// civic_decode_attn_noalloc keeps the partial results of the splits in a buffer that belongs to the library's
// code object instead of one the caller brings: every GPU that loads the library holds its own copy of this
// array, at its own address, until the process ends.
constexpr size_t kDecStaticBytes = CIVIC_DECODE_NOALLOC_MAX_BYTES;
static __device__ __align__(256) unsigned char dec_static_scratch[kDecStaticBytes];

// The array's address on the current device.  In host code the array's name stands for the symbol, not for
// device memory: its address is asked for once per device, with that device current, and kept.
static int static_scratch_ptr(void** ptr)
{
    constexpr int kMaxDevices = 64;
    static std::atomic<void*> cached[kMaxDevices];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return record_hip_error(e);
    if (dev >= 0 && dev < kMaxDevices) {
        void* p = cached[dev].load(std::memory_order_acquire);
        if (p) { *ptr = p; return CIVIC_OK; }
    }
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(dec_static_scratch));
    if (e != hipSuccess || !p) return record_hip_error(e != hipSuccess ? e : hipErrorInvalidSymbol);
    if (dev >= 0 && dev < kMaxDevices) cached[dev].store(p, std::memory_order_release);
    *ptr = p;
    return CIVIC_OK;
}

}  // namespace civic

extern "C" int civic_decode_attn_noalloc(const void* q, const void* k_cache, const void* v_cache, void* out, int dtype,
                                         int32_t batch, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                                         int64_t s_max, int64_t n_ctx, float softmax_scale, void* stream)
{
    using namespace civic;
    DecodePlan p;
    bool nothing = false;
    const int rc = decode_check(q, k_cache, v_cache, out, dtype, batch, n_q_heads, n_kv_heads, head_dim, s_max, n_ctx,
                                softmax_scale, &p, &nothing);
    if (rc != CIVIC_OK || nothing) return rc;
    if (p.ws_bytes > kDecStaticBytes) return CIVIC_ERR_WORKSPACE;      // more partial results than the array holds
    void* scratch = nullptr;
    if (p.ws_bytes > 0) {
        const int rs = static_scratch_ptr(&scratch);
        if (rs != CIVIC_OK) return rs;
    }
    // every element of the array that the combine launch reads is written by this call's first launch: nothing
    // has to start at zero
    return decode_attn(q, k_cache, v_cache, out, dtype, batch, n_q_heads, n_kv_heads, head_dim, s_max, n_ctx, softmax_scale,
                       p, static_cast<float*>(scratch), stream);
}

extern "C" size_t civic_decode_attn_workspace_bytes(int dtype, int32_t batch, int32_t n_q_heads, int32_t n_kv_heads,
                                                    int32_t head_dim, int64_t n_ctx)
{
    civic::DecodePlan p;
    if (civic::decode_plan(dtype, batch, n_q_heads, n_kv_heads, head_dim, n_ctx, &p) != CIVIC_OK) return 0;
    return p.ws_bytes;
}

extern "C" int civic_decode_attn(const void* q, const void* k_cache, const void* v_cache, void* out, int dtype,
                                 int32_t batch, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, int64_t s_max,
                                 int64_t n_ctx, float softmax_scale, void* workspace, size_t workspace_bytes, void* stream)
{
    using namespace civic;
    DecodePlan p;
    bool nothing = false;
    const int rc = decode_check(q, k_cache, v_cache, out, dtype, batch, n_q_heads, n_kv_heads, head_dim, s_max, n_ctx,
                                softmax_scale, &p, &nothing);
    if (rc != CIVIC_OK || nothing) return rc;
    if (p.ws_bytes > 0 && (!workspace || workspace_bytes < p.ws_bytes || !aligned16(workspace))) return CIVIC_ERR_WORKSPACE;
    return decode_attn(q, k_cache, v_cache, out, dtype, batch, n_q_heads, n_kv_heads, head_dim, s_max, n_ctx, softmax_scale,
                       p, static_cast<float*>(workspace), stream);
}

// ---------------------------------------------------------------------------------------------- ragged caches
namespace civic {

// The longest context of samples [b0, b0 + nb); -1 if one of them is shorter than one row or longer than the caches.
static int64_t longest_ctx(const int32_t* n_ctx, int32_t b0, int32_t nb, int64_t s_max)
{
    int64_t longest = 0;
    for (int32_t i = 0; i < nb; ++i) {
        const int64_t n = n_ctx[b0 + i];
        if (n < 1 || n > s_max) return -1;
        longest = n > longest ? n : longest;
    }
    return longest;
}

}  // namespace civic

extern "C" size_t civic_decode_attn_ragged_workspace_bytes(int dtype, int32_t batch, const int32_t* n_ctx, int32_t n_q_heads,
                                                           int32_t n_kv_heads, int32_t head_dim)
{
    using namespace civic;
    if (batch <= 0 || !n_ctx) return 0;
    size_t need = 0;                                          // the groups run one after the other and share the workspace
    for (int32_t b0 = 0; b0 < batch; b0 += kDecRaggedItems) {
        const int32_t nb = batch - b0 < kDecRaggedItems ? batch - b0 : kDecRaggedItems;
        const int64_t longest = longest_ctx(n_ctx, b0, nb, INT32_MAX);
        DecodePlan p;
        if (longest < 0 || decode_plan(dtype, nb, n_q_heads, n_kv_heads, head_dim, longest, &p, true) != CIVIC_OK) return 0;
        need = p.ws_bytes > need ? p.ws_bytes : need;
    }
    return need;
}

extern "C" int civic_decode_attn_ragged(const void* q, const void* k_cache, const void* v_cache, void* out, int dtype,
                                        int32_t batch, const int32_t* n_ctx, int32_t n_q_heads, int32_t n_kv_heads,
                                        int32_t head_dim, int64_t s_max, float softmax_scale, void* workspace,
                                        size_t workspace_bytes, void* stream)
{
    using namespace civic;
    const int esz = dtype_size(dtype);
    if (!esz || batch < 0) return CIVIC_ERR_INVALID_ARG;
    if (batch > 0 && !n_ctx) return CIVIC_ERR_INVALID_ARG;
    // Groups of up to kDecRaggedItems samples, each the launch or two of civic_decode_attn over pieces of one length; every
    // group is checked before the first launch.
    for (int pass = 0; pass < 2; ++pass)
        for (int32_t b0 = 0; b0 < batch; b0 += kDecRaggedItems) {
            const int32_t nb = batch - b0 < kDecRaggedItems ? batch - b0 : kDecRaggedItems;
            const int64_t longest = longest_ctx(n_ctx, b0, nb, s_max);
            if (longest < 0) return CIVIC_ERR_INVALID_ARG;
            const char* qb = static_cast<const char*>(q) + static_cast<int64_t>(b0) * n_q_heads * head_dim * esz;
            char* ob = static_cast<char*>(out) + static_cast<int64_t>(b0) * n_q_heads * head_dim * esz;
            const int64_t cache_at = static_cast<int64_t>(b0) * n_kv_heads * s_max * head_dim * esz;
            const char* kb = static_cast<const char*>(k_cache) + cache_at;
            const char* vb = static_cast<const char*>(v_cache) + cache_at;
            DecodePlan p;
            bool nothing = false;
            int rc = decode_check(q ? qb : nullptr, k_cache ? kb : nullptr, v_cache ? vb : nullptr, out ? ob : nullptr, dtype, nb, n_q_heads,
                                  n_kv_heads, head_dim, s_max, longest, softmax_scale, &p, &nothing, true);
            if (rc != CIVIC_OK) return rc;
            if (p.ws_bytes > 0 && (!workspace || workspace_bytes < p.ws_bytes || !aligned16(workspace))) return CIVIC_ERR_WORKSPACE;
            if (pass == 0 || nothing) continue;
            rc = decode_attn(qb, kb, vb, ob, dtype, nb, n_q_heads, n_kv_heads, head_dim, s_max, longest, softmax_scale, p,
                             static_cast<float*>(workspace), stream, n_ctx + b0);
            if (rc != CIVIC_OK) return rc;
        }
    return CIVIC_OK;
}
