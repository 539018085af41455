// civic_prefill_attn: dense grouped-query prefill attention over the compact sequence (the
// beta * N_l * (L+M_p)^2 * D_l term of Eq. 7; softmax(Q K^T / sqrt(d)) V as in Eq. 9).
//
// bf16 path (MFMA-bound): flash-style, one 512-thread workgroup = 8 wavefronts x 32 query rows over
// one KV head.  With four or more query heads per KV head the wavefronts are 4 heads x 2 row tiles
// (64 rows), so one K/V tile staged in LDS serves the whole group and all wavefronts share the
// causal extent; smaller groups put more row tiles of the same head in the workgroup.
//   - K/V tiles of 64 keys go from global memory straight into a small LDS ring
//     (global_load_lds_dwordx4, 16 bytes per lane), one tile ahead of the one being consumed; Q is
//     staged the same way, so the kernel has no register-destination global load, and the ring is
//     tracked with explicit vmcnt waits and fence-free workgroup barriers.  Rows keep a 256-byte
//     pitch and the 16-byte chunks are XOR-swizzled, so neither the 128-bit K reads nor the
//     transposing V reads hit a bank conflict.
//   - Scores are computed TRANSPOSED, S^T = K Q^T with v_mfma_f32_32x32x16_bf16: a lane owns one
//     query column, so softmax row statistics are in-lane reductions plus one exchange between the
//     two half-waves, and the rescale factor is a per-lane scalar.  The exponentiated tile, rounded
//     to bf16, is already laid out as the B operand of O^T += V^T P^T; the matching A operand comes
//     from the row-major V tile through the LDS transpose read ds_read_b64_tr_b16.
//   - Little vector work per score: a probability is exp2(fma(score, scale * log2 e, -offset)), one
//     fused multiply-add and one v_exp_f32; the offset is the first tile's row maximum and moves
//     later only when the row sums show that a tile outgrew it (no per-tile maximum pass).
//   - fp32 accumulation, row sums taken from the rounded probabilities with v_dot2c_f32_bf16, bf16
//     output (nearest even) staged through LDS into whole 16-byte row segments.
//   - Workgroups are ordered heaviest causal row tile first (row tile on grid y, the rest of the block
//     index decoded with multiply-high constants from the launch: no integer division ahead of Q's loads).
//   - Masking costs a compare and a select per score and only on tiles that cross the diagonal or the end
//     of the sequence; a wavefront that cannot see the second half of such a tile computes the first only.
//   - civic_prefill_attn_kv: the workgroup of a KV head's first head block also copies the K/V rows of its
//     own query rows into the caches (8 threads per row, same address for K and V).
//
// fp32 path and head sizes the bf16 MFMA path does not cover: fp32 matrix instructions, the keys of a 16-row tile split over a
// workgroup's wavefronts.
#include <algorithm>
#include <array>
#include <cmath>
#include <type_traits>

#include "civic_internal.h"

// LDS fragments (K rows, transposed V) are read this many MFMAs ahead of the MFMA that consumes them (build-time
// knob for A/B runs; 2-4 measure within 1 % of each other, 2 needs the fewest registers).
#ifndef CIVIC_ATTN_DIST
#define CIVIC_ATTN_DIST 2
#endif

namespace civic {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kRaggedItems = 64;          // items of one ragged launch (longer lists go out in several)

struct AttnArgs {
    const void* q; const void* k; const void* v; void* out;
    int64_t qs[3], ks[3], os[3];          // element strides: batch, token, head
    int32_t batch, seq, n_q_heads, n_kv_heads, head_dim, causal;
    int32_t kv_seq;                       // keys per sample (= seq except for civic_cross_attn, which has no mask)
    float scale;                          // softmax scale (natural-exponent domain)
    int32_t heads_per_block, row_tiles;   // MFMA path: block shape and number of 32*rows_per_block tiles; fp32 path: tiles of 16 rows
    int32_t pass_tiles;                   // fp32 path: row tiles of a pass over the units (f32_grid)
    int32_t paired;                       // MFMA path: a workgroup walks two row tiles, a heavy and a light one
    int32_t item_shift;                   // MFMA path, ragged: every fourth row tile begins with the next item (shift_items)
    // block index -> (head block, kv head, batch) without integer division: q heads per kv head,
    // head blocks per kv head, log2(heads_per_block), ceil(2^32 / d) for d = head blocks, kv heads (0 for d = 1)
    int32_t group, head_blocks, hb_shift;
    uint32_t magic_head_blocks, magic_kv_heads;
    // fused KV-cache write (MFMA path; null = none): caches are dense [batch, n_kv_heads, s_max, head_dim]
    void* k_cache; void* v_cache;
    int64_t s_max, pos0;
    // rotary embedding of Q from a (cos, sin) table [batch, seq, head_dim / 2] (null = none): civic_prefill_attn_rope
    const float2* q_cs;
    // ragged queries (civic_cross_attn_ragged; read by the RAGGED instantiations only): `batch` items packed along the
    // token axis, item b owning query and output rows [item_row[b], item_row[b + 1]); `seq` is the longest item
    int32_t item_row[kRaggedItems + 1];
    int32_t kv_packed;                    // ragged: keys and values are packed along the token axis like the queries
};

// ---------------------------------------------------------------------------------- fp32 matrix-core path
// fp32 inputs, and head sizes the bf16 kernel does not cover: all arithmetic in fp32 on v_mfma_f32_16x16x4f32.  A workgroup of
// four wavefronts owns 16 query rows of one head and its wavefronts take every fourth tile of keys, each with an online
// softmax of its own; the four states meet in LDS at the end.  Splitting the keys is what fills the chip: these shapes have few
// rows (469 rows x 16 heads are 480 workgroups of 16 rows), and one wavefront needs 64 clocks for 16 x 16 x 16 multiply-adds.
// No operand goes through LDS on its way to the matrix cores.  The contraction of Q K^T may run over the channels in any order
// that both operands share, and the rows of V^T may be any permutation of the channels, so a lane takes the 16-byte pieces that
// lie there: channels 16 t + 4 (lane / 16) .. + 3 of key lane % 16 serve four consecutive MFMAs, channels 64 T + 4 (lane % 16) ..
// + 3 of one key are four rows of V^T.  S^T leaves a lane with four consecutive keys of one query, which is the B operand of
// O^T += V^T P^T as it stands.  L1 delivers 16 KB per 16 x 16 tile and wavefront, 32 bytes a clock and unit at full MFMA rate.
// 469 rows, 16 / 8 heads of 128, causal: 175 us on the vector units (one row per wavefront), 20.7 us here.
template <bool BF16>
__device__ __forceinline__ float4 load_quad(const void* p, int64_t i)
{
    if constexpr (BF16) {
        const u32x2 w = *reinterpret_cast<const u32x2*>(static_cast<const uint16_t*>(p) + i);
        return make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xFFFF0000u), __uint_as_float(w.y << 16),
                           __uint_as_float(w.y & 0xFFFF0000u));
    } else {
        return *reinterpret_cast<const float4*>(static_cast<const float*>(p) + i);
    }
}

constexpr int kF32Rows = 16, kF32Waves = 4;
constexpr int kMaxGridZ = 65535;
static constexpr size_t f32_lds_bytes(int nt) { return sizeof(float) * (kF32Waves * kF32Rows * (64 * nt + 4 + 2) + kF32Waves); }

// NT: head_dim rounded up to 64, over 64.  SUB: sub-tiles of 16 keys a tile (launch_f32_for says which).  TAIL: head_dim ends inside
// a step of 16 channels (as a check in the loop it cost 0.4 of 43 us on 469 rows with 16 / 8 heads of 128, which have no tail).
// FULL: head_dim is 64 NT.  Its steps are known then, and the loop has no branches around them: loads and products of different steps
// mix, and a tile's first products do not wait for all of its K rows.
template <bool BF16, int NT, int SUB, bool TAIL, bool FULL>
__global__ __launch_bounds__(kF32Waves * kWave, NT <= 3 ? 2 : 1) void attn_f32_kernel(AttnArgs a)
{
    static_assert(!(TAIL && FULL), "a full head has no tail");
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) float f32_lds[];
    constexpr int KEYS = 16 * SUB;                             // SUB sub-tiles of 16 keys a tile
    constexpr int PITCH = 64 * NT + 4;                         // floats per staged row (padded against bank conflicts)
    float* const st_m = f32_lds + kF32Waves * kF32Rows * PITCH, * const st_l = st_m + kF32Waves * kF32Rows, * const st_odd = st_l + kF32Waves * kF32Rows;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid >> 6;
    const int l16 = lane & 15, kq = lane >> 4;
    // Grid x: the query heads, those of KV head g at g, g + n_kv_heads, ...; y: the samples; z: the row tiles, f32_grid has the order.
    const int group = a.group, hg = a.magic_kv_heads ? static_cast<int>(__umulhi(blockIdx.x, a.magic_kv_heads)) : static_cast<int>(blockIdx.x);
    const int g = static_cast<int>(blockIdx.x) - hg * a.n_kv_heads, h = g * group + hg;
    int b = blockIdx.y, y = blockIdx.z;
    if (b >= a.batch) { const int up = b / a.batch; b -= up * a.batch; y += up * kMaxGridZ; }
    if (y >= a.row_tiles) return;
    if (a.pass_tiles < a.row_tiles) {
        const int pass = y / a.pass_tiles, first = pass * a.pass_tiles;
        if (pass & 1) y = first + min(first + a.pass_tiles, a.row_tiles) - 1 - y;
    }
    const int row_tile = a.row_tiles - 1 - y;                  // the heaviest causal tiles first
    const int d = FULL ? 64 * NT : a.head_dim, i0 = row_tile * kF32Rows;
    const int rows = min(kF32Rows, a.seq - i0);
    const int64_t kv_off = b * a.ks[0] + g * a.ks[2];

    // Q: scaled, rotated if asked, staged as fp32 (rows past the sequence repeat the last one; never written)
    for (int idx = tid; idx < kF32Rows * (d / 4); idx += kF32Waves * kWave) {
        const int r = idx / (d / 4), c = (idx - r * (d / 4)) * 4;
        float4 x = load_quad<BF16>(a.q, b * a.qs[0] + (i0 + min(r, rows - 1)) * a.qs[1] + h * a.qs[2] + c);
        x.x *= a.scale; x.y *= a.scale; x.z *= a.scale; x.w *= a.scale;
        *reinterpret_cast<float4*>(f32_lds + r * PITCH + c) = x;
    }
    // KV-cache write of the tile's own K and V rows (the first head of every KV group does it)
    if (a.k_cache != nullptr && h == g * group) {
        constexpr int EPP = BF16 ? 8 : 4, ESZ = BF16 ? 2 : 4;  // elements per 16-byte piece
        const int pieces = d / EPP;
        for (int idx = tid; idx < rows * pieces; idx += kF32Waves * kWave) {
            const int r = idx / pieces, c = (idx - r * pieces) * EPP;
            const int64_t src = (kv_off + (i0 + r) * a.ks[1] + c) * ESZ;
            const int64_t dst = (((static_cast<int64_t>(b) * a.n_kv_heads + g) * a.s_max + a.pos0 + i0 + r) * d + c) * ESZ;
            *reinterpret_cast<u32x4*>(static_cast<char*>(a.k_cache) + dst) = *reinterpret_cast<const u32x4*>(static_cast<const char*>(a.k) + src);
            *reinterpret_cast<u32x4*>(static_cast<char*>(a.v_cache) + dst) = *reinterpret_cast<const u32x4*>(static_cast<const char*>(a.v) + src);
        }
    }
    __syncthreads();
    if (a.q_cs != nullptr) {                                   // rotary embedding: pairs (c, c + d/2) of a query row
        for (int idx = tid; idx < kF32Rows * (d / 2); idx += kF32Waves * kWave) {
            const int r = idx / (d / 2), c = idx - r * (d / 2);
            const float2 t = a.q_cs[(static_cast<int64_t>(b) * a.seq + i0 + min(r, rows - 1)) * (d / 2) + c];
            float* q = f32_lds + r * PITCH + c;
            rope_pair(q[0], q[d / 2], t.x, t.y, q[0], q[d / 2]);
        }
        __syncthreads();
    }
    float4 qf[4 * NT];                                         // B operand: channels 16 t + 4 kq .. + 3 of query l16
#pragma unroll
    for (int t = 0; t < 4 * NT; ++t) {
        const int c = 16 * t + 4 * kq;
        qf[t] = c < d ? *reinterpret_cast<const float4*>(f32_lds + l16 * PITCH + c) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();                                           // the area becomes the wavefronts' results

    f32x4 o[NT][4];                                            // O^T: register r of (T, e): channel 64 T + 16 kq + 4 r + e, query l16
#pragma unroll
    for (int T = 0; T < NT; ++T)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[T][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;                              // l: the lane's own keys only
    const int n_keys = a.causal ? i0 + rows : a.kv_seq;        // keys some row of the tile sees
    const int qi = i0 + l16;
    // From the tile of this key on some query does not see every key of a tile.  A hidden key's weight is 0, and 0 x V has to
    // stay 0 whatever that row of V holds: infinities and NaN are taken out there, and put back at the end for the rows that see
    // them (in the loop that would cost the registers it runs in).
    const int mixed0 = (a.causal ? i0 + 1 : n_keys) / KEYS * KEYS;
    bool odd = false;
    // (a key past the last one re-reads it: its score is masked)
    auto k_row = [&](int key) { return kv_off + static_cast<int64_t>(min(key, n_keys - 1)) * a.ks[1]; };
    float4 kf[SUB][4 * NT];
    auto fetch_k = [&](int key0) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < SUB; ++s) {
            const int64_t base = k_row(key0 + 16 * s + l16);
#pragma unroll
            for (int t = 0; t < 4 * NT; ++t)
                if (16 * t < d) kf[s][t] = load_quad<BF16>(a.k, base + min(16 * t + 4 * kq, d - 4));
        }
    };
    int key0 = w * KEYS;
    if (key0 < n_keys) fetch_k(key0);
    for (; key0 < n_keys; key0 += kF32Waves * KEYS) {
        if constexpr (TAIL) {                                  // lanes past the row hold the end of it: 0 x it has to be 0
#pragma unroll
            for (int t = 0; t < 4 * NT; ++t)
                if (16 * t < d && 16 * t + 16 > d) {
#pragma unroll
                    for (int s = 0; s < SUB; ++s)
                        if (16 * t + 4 * kq >= d) kf[s][t] = make_float4(0.f, 0.f, 0.f, 0.f);
                }
        }
        // S^T: sub-tiles of 16 keys, two partial sums each (independent MFMA chains)
        f32x4 sc[SUB][2];
#pragma unroll
        for (int s = 0; s < SUB; ++s) sc[s][0] = sc[s][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 4 * NT; ++t)
            if (16 * t < d) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int s = 0; s < SUB; ++s) {
                        const float kv[4] = {kf[s][t].x, kf[s][t].y, kf[s][t].z, kf[s][t].w};
                        const float qv[4] = {qf[t].x, qf[t].y, qf[t].z, qf[t].w};
                        sc[s][e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[e], qv[e], sc[s][e & 1], 0, 0, 0);
                    }
            }
        // V rows of this tile, in flight under the softmax: step e of sub-tile s multiplies keys 16 s + 4 kq + e
        float4 vf[SUB][4][NT];
#pragma unroll
        for (int s = 0; s < SUB; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t base = k_row(key0 + 16 * s + 4 * kq + e);
#pragma unroll
                for (int T = 0; T < NT; ++T) {
                    const int c = 64 * T + 4 * l16;
                    vf[s][e][T] = load_quad<BF16>(a.v, base + (c < d ? c : 0));
                }
            }
        const bool more = key0 + kF32Waves * KEYS < n_keys;
        const int lim = a.causal ? min(qi + 1, n_keys) : n_keys;   // the lane sees keys below lim
        float p[SUB][4], m_new = m;
#pragma unroll
        for (int s = 0; s < SUB; ++s)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float z = sc[s][0][r] + sc[s][1][r];
                p[s][r] = key0 + 16 * s + 4 * kq + r < lim ? z : -INFINITY;
                m_new = fmaxf(m_new, p[s][r]);
            }
        m_new = fmaxf(m_new, __shfl_xor(m_new, 16, kWave));
        m_new = fmaxf(m_new, __shfl_xor(m_new, 32, kWave));
        const float m_use = m_new == -INFINITY ? 0.f : m_new;  // a query that has met no key of this wavefront yet
        const float alpha = expf(m - m_use);
        float sum = 0.f;
#pragma unroll
        for (int s = 0; s < SUB; ++s)
#pragma unroll
            for (int r = 0; r < 4; ++r) { p[s][r] = expf(p[s][r] - m_use); sum += p[s][r]; }
        l = fmaf(l, alpha, sum);
        m = m_new;
#pragma unroll
        for (int T = 0; T < NT; ++T)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[T][e] *= alpha;
        if (more) fetch_k(key0 + kF32Waves * KEYS);            // the next tile's K rows fly under the second product
        if (key0 >= mixed0) {
            auto finite = [&](float& x) __attribute__((always_inline)) {
                if (!(fabsf(x) < INFINITY)) { x = 0.f; odd = true; }
            };
#pragma unroll
            for (int s = 0; s < SUB; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int T = 0; T < NT; ++T) { finite(vf[s][e][T].x); finite(vf[s][e][T].y); finite(vf[s][e][T].z); finite(vf[s][e][T].w); }
        }
#pragma unroll
        for (int s = 0; s < SUB; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int T = 0; T < NT; ++T) {
                    const float vv[4] = {vf[s][e][T].x, vf[s][e][T].y, vf[s][e][T].z, vf[s][e][T].w};
#pragma unroll
                    for (int c = 0; c < 4; ++c) o[T][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[c], p[s][e], o[T][c], 0, 0, 0);
                }
    }
    l += __shfl_xor(l, 16, kWave);
    l += __shfl_xor(l, 32, kWave);

    // the four states of the tile meet: out = sum_w f_w o_w / sum_w f_w l_w, f_w = exp(m_w - max m)
    if (kq == 0) { st_m[w * kF32Rows + l16] = m; st_l[w * kF32Rows + l16] = l; }
    odd = __any(odd);
    if (lane == 0) st_odd[w] = odd ? 1.f : 0.f;
#pragma unroll
    for (int T = 0; T < NT; ++T)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *reinterpret_cast<float4*>(f32_lds + (w * kF32Rows + l16) * PITCH + 64 * T + 16 * kq + 4 * r) =
                make_float4(o[T][0][r], o[T][1][r], o[T][2][r], o[T][3][r]);
    __syncthreads();
    for (int idx = tid; idx < rows * (d / 4); idx += kF32Waves * kWave) {
        const int r = idx / (d / 4), c = (idx - r * (d / 4)) * 4;
        float mx = st_m[r];
#pragma unroll
        for (int x = 1; x < kF32Waves; ++x) mx = fmaxf(mx, st_m[x * kF32Rows + r]);   // finite: every row sees a key
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        float lt = 0.f;
#pragma unroll
        for (int x = 0; x < kF32Waves; ++x) {
            const float f = expf(st_m[x * kF32Rows + r] - mx);
            const float4 t = *reinterpret_cast<const float4*>(f32_lds + (x * kF32Rows + r) * PITCH + c);
            lt = fmaf(f, st_l[x * kF32Rows + r], lt);
            acc.x = fmaf(f, t.x, acc.x); acc.y = fmaf(f, t.y, acc.y); acc.z = fmaf(f, t.z, acc.z); acc.w = fmaf(f, t.w, acc.w);
        }
        if (__builtin_expect(st_odd[0] + st_odd[1] + st_odd[2] + st_odd[3] != 0.f, 0)) {
            const int lim = a.causal ? i0 + r + 1 : n_keys;    // an infinity or NaN that the row sees is the result, whatever its weight
            for (int key = mixed0; key < lim; ++key) {
                const float4 v = load_quad<BF16>(a.v, k_row(key) + c);
                acc.x += fabsf(v.x) < INFINITY ? 0.f : v.x; acc.y += fabsf(v.y) < INFINITY ? 0.f : v.y;
                acc.z += fabsf(v.z) < INFINITY ? 0.f : v.z; acc.w += fabsf(v.w) < INFINITY ? 0.f : v.w;
            }
        }
        const float inv = 1.f / lt;
        const int64_t at = b * a.os[0] + (i0 + r) * a.os[1] + h * a.os[2] + c;
        if constexpr (BF16) {
            const bf16x4 v = {static_cast<__bf16>(acc.x * inv), static_cast<__bf16>(acc.y * inv), static_cast<__bf16>(acc.z * inv),
                              static_cast<__bf16>(acc.w * inv)};
            *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(a.out) + at) = v;
        } else {
            *reinterpret_cast<float4*>(static_cast<float*>(a.out) + at) = make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
        }
    }
}

// Grid and order of the workgroups.  The hardware hands consecutive workgroups to the eight XCDs in turn: with the heads innermost, the
// query heads of a KV head and all their row tiles land on the same few, and its K and V in those L2s (2 x 1024 rows, 8 heads of 256
// 188 -> 130 us, 1 x 1500, 8 of 96 85 -> 68; the row tiles innermost brought all K and V to every XCD).
// Under the causal mask row tiles go out by falling weight.  Up to four workgroups to a unit they go in passes of one workgroup to a
// unit, every other pass in reverse, so that the unit with the heaviest first takes the lightest second: all start at once or nearly
// so, and nothing evens out the units later (1 x 469, 16 / 8 heads of 128 23.1 -> 20.7 us, 1 x 1024, 8 / 8 40.0 -> 31.8, 1 x 700, 16 / 8
// 38.4 -> 33.9).  Around four to a unit either order may be the faster, in passes 2 % on average over 140 sizes (without and in them:
// 2 x 1050, 4 / 2 of 96 42.2, 36.3, 4 x 450, 8 / 8 of 64 19.6, 18.5, 8 x 128, 16 / 8 19.8, 19.2, but 8 x 117 18.9, 19.6, and the worst
// 4 x 200, 16 / 8 20.0, 21.1).  More workgroups than that even out by themselves (4 x 200, 32 / 8 33.7 and 34.3 in passes).
static dim3 f32_grid(AttnArgs& a)
{
    constexpr int64_t kUnits = 256;                            // compute units
    a.row_tiles = static_cast<int32_t>((static_cast<int64_t>(a.seq) + kF32Rows - 1) / kF32Rows);
    const int64_t per_rt = static_cast<int64_t>(a.n_q_heads) * a.batch;
    a.pass_tiles = a.causal && per_rt <= kUnits && per_rt * a.row_tiles <= 4 * kUnits ? static_cast<int32_t>(kUnits / per_rt) : a.row_tiles;
    a.magic_kv_heads = a.n_kv_heads <= 1 ? 0u : static_cast<uint32_t>(((int64_t{1} << 32) + a.n_kv_heads - 1) / a.n_kv_heads);
    // (row tiles past what a grid has in z continue behind the samples in y)
    return dim3(static_cast<unsigned>(a.n_q_heads), static_cast<unsigned>(a.batch * ((a.row_tiles + kMaxGridZ - 1) / kMaxGridZ)),
                static_cast<unsigned>(std::min(a.row_tiles, kMaxGridZ)));
}

template <bool BF16, int NT, int SUB, bool TAIL, bool FULL>
static int launch_f32_tail(const AttnArgs& a_in, hipStream_t s)
{
    AttnArgs a = a_in;
    const dim3 grid = f32_grid(a);
    constexpr size_t lds = f32_lds_bytes(NT);
    if (lds > 64 * 1024) {
        static std::atomic<uint64_t> allowed{0};
        const int rc = allow_dynamic_lds(reinterpret_cast<const void*>(attn_f32_kernel<BF16, NT, SUB, TAIL, FULL>), lds, &allowed);
        if (rc != CIVIC_OK) return rc;
    }
    civic::launch((attn_f32_kernel<BF16, NT, SUB, TAIL, FULL>), grid, dim3(kF32Waves * kWave), lds, s, a);
    return check_launch();
}

template <bool BF16, int NT, int SUB>
static int launch_f32(const AttnArgs& a, hipStream_t s)
{
    if (a.head_dim == 64 * NT) return launch_f32_tail<BF16, NT, SUB, false, true>(a, s);
    return a.head_dim % 16 ? launch_f32_tail<BF16, NT, SUB, true, false>(a, s) : launch_f32_tail<BF16, NT, SUB, false, false>(a, s);
}

template <bool BF16>
static int launch_f32_for(const AttnArgs& a, hipStream_t s)
{
    // 16 keys a tile (times with the row tiles innermost in the grid; f32_grid's order takes up to a third off both sides)
    //   - up to 64 keys, one tile for each wavefront, where the instructions of the longer tile are most of the time (17 rows,
    //     4 / 2 fp32 heads of 64 / 128: 4.4 / 6.0 us, 5.3 / 7.7 in tiles of 32, 4.2 / 5.8 with one row per wavefront on the vector
    //     units; 32 x 64 rows, 16 / 8 heads of 128: 33.1, 41.2 and 172.8)
    //   - for fp32 heads of 64 and 128, whose loop has no branches, and between them up to 1024 keys: more wavefronts fit a unit (us in
    //     tiles of 32 and 16: 469 rows, 16 / 8 heads of 128 26.2 and 24.7; 8 x 100, 32 / 8 of 128 36.0 and 28.2; 4 x 300, 16 / 16 of 64
    //     25.1 and 22.1; 3 x 400, 16 / 16 of 96 48.5 and 43.5, but 1500, 8 / 8 of 96 83.3 and 86.5, 469, 16 / 8 of 40 14.4 and 15.1)
    //   - for heads wider than 128, where two workgroups then fit a unit (up to 192) and nothing is spilled (beyond): 469
    //     rows, 16 / 8 fp32 heads of 192 / 256: 36.0 / 72.4 us, 56.6 / 120.7 in tiles of 32; bf16 45.8 / 102, 69.7 / 144
    // and 32 elsewhere.
    const bool few = a.kv_seq <= 64 || (!BF16 && (a.head_dim == 64 || a.head_dim == 128 || (a.head_dim > 64 && a.kv_seq <= 1024)));
    if (a.head_dim <= 64) return few ? launch_f32<BF16, 1, 1>(a, s) : launch_f32<BF16, 1, 2>(a, s);
    if (a.head_dim <= 128) return few ? launch_f32<BF16, 2, 1>(a, s) : launch_f32<BF16, 2, 2>(a, s);
    if (a.head_dim <= 192) return launch_f32<BF16, 3, 1>(a, s);
    return launch_f32<BF16, 4, 1>(a, s);
}

// --------------------------------------------------------------------------------------- MFMA path
constexpr int kBN = 64;                 // keys per LDS tile

typedef short s16x4 __attribute__((ext_vector_type(4)));

// LDS transpose read (gfx950): the 16 lanes of a group each name 4 consecutive bf16 of a 4 x 16 block
// (lane i -> row i/4, columns 4(i%4)..+3); lane i receives column i of the block, rows 0..3.
__device__ __forceinline__ s16x4 lds_read_tr16(const __bf16* p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (s16x4 __attribute__((address_space(3)))*)(const_cast<__bf16*>(p)));
}

// K/V tiles live in LDS with a fixed row pitch of PITCH 16-byte chunks and an XOR swizzle of the chunk
// index by a function of the row, so that no padding is needed (global -> LDS loads write 64
// consecutive 16-byte slots per wavefront instruction) and both the 128-bit K reads (16 lanes = 16
// consecutive rows, same logical chunk) and the transposing 64-bit V reads (32 lanes = 4 consecutive
// rows x 4 chunks) fall on distinct banks.
template <int PITCH>
__device__ __forceinline__ int swz(int row)
{
    if constexpr (PITCH == 16) return ((row & 3) << 2) | ((row >> 2) & 3);
    else if constexpr (PITCH == 12) return (row >> 2) & 3;   // (rows 12 chunks apart start in 4 different quarters of the 16 by themselves)
    else return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
}


typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) char lds_char;

// 16 bytes per lane from global memory (scalar base + per-lane byte offset) straight into LDS at
// lds_addr + LDS_IMM + lane * 16 (lds_addr wave-uniform).  Issued as inline assembly on purpose: the pipeline
// tracks these loads with explicit s_waitcnt vmcnt(N), and an LDS read the compiler could see racing
// with an asynchronous LDS write would make it drain the whole load queue first.  m0 is written and not
// declared: the register is reserved (the compiler rejects it as a clobber), never allocated, and set by the
// compiler only directly in front of an instruction that reads it, of which this file has none.
// The compiler counts no wait states into an asm statement.  A load into LDS may read m0 one wait state after a scalar instruction wrote
// it; `base` comes from uniform_ptr, which sees to the ones that it needs.
template <int LDS_IMM>
__device__ __forceinline__ void dma16(const void* base, uint32_t byte_off, uint32_t lds_addr)
{
    // (the LDS address is lds_addr + LDS_IMM, added here so that one scalar register serves every instruction
    // of a tile instead of one register per instruction)
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_addr), "v"(byte_off), "s"(base), "n"(LDS_IMM) : "memory", "scc");
}

// dma16 with the LDS immediate BASE_IMM + j * 1024 for a loop index j that is a constant after unrolling
// (at most 16 instructions per wavefront and tile).
template <int BASE_IMM, int J = 0>
__device__ __forceinline__ void dma16_at(const void* base, uint32_t byte_off, uint32_t lds_addr,
                                         std::integral_constant<int, BASE_IMM> imm, int j)
{
    if constexpr (J < 16) {
        if (j == J) dma16<BASE_IMM + J * kWave * 16>(base, byte_off, lds_addr);
        else dma16_at<BASE_IMM, J + 1>(base, byte_off, lds_addr, imm, j);
    }
}

// Workgroup barrier without the memory fence __syncthreads() implies (which would wait for every
// outstanding load, including the prefetches that are meant to stay in flight).
__device__ __forceinline__ void block_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The same pointer, written by a scalar instruction.  A load reads its base five wait states after a vector instruction wrote that at
// the earliest (v_readfirstlane, or v_readlane of a spilled pair), which the compiler does not see to for a load inside an asm
// statement; a scalar instruction waits for the vector one in hardware, and what it wrote may be read at once.  (Five states in front
// of every load instead: 0.5 to 1 % of a launch.)
__device__ __forceinline__ const char* scalar_copy(const char* p)
{
    uint64_t copy;
    asm("s_mov_b64 %0, %1" : "=s"(copy) : "s"(p));
    return reinterpret_cast<const char*>(copy);
}

// A wave-uniform pointer with both halves forced into scalar registers, for loads.
__device__ __forceinline__ const char* uniform_ptr(const void* p)
{
    const uint64_t bits = reinterpret_cast<uint64_t>(p);
    // the builtin returns a signed int: widen each half as unsigned
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(bits >> 32)));
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(bits)));
    return scalar_copy(reinterpret_cast<const char*>((static_cast<uint64_t>(hi) << 32) | lo));
}

template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    // s_waitcnt immediate (gfx9): vmcnt = bits [3:0] and [15:14]; expcnt and lgkmcnt left at their maxima
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// DP: head_dim rounded up to 64, 80, 96 or 128; WAVES: wavefronts per workgroup (4 or 8); STAGES: K/V
// tiles in flight in LDS.
template <int DP, int WAVES, int STAGES>
struct AttnTile {
    static constexpr int THREADS = WAVES * kWave;
    static constexpr int KSTEPS = DP / 16;      // MFMA k-steps of Q K^T
    static constexpr int DT = (DP + 31) / 32;   // 32-row tiles of O^T
    static constexpr int PITCH = DP == 64 ? 8 : DP <= 96 && WAVES == 4 ? 12 : 16;   // 16-byte chunks per LDS row
    static constexpr int PITCHB = PITCH * 16;              // ... in bytes
    static constexpr int TILEB = kBN * PITCHB;             // bytes per K (or V) tile
    static constexpr int NI = kBN * PITCH / THREADS;       // global->LDS instructions per wavefront, tile and tensor
    static constexpr int TLOADS = 2 * NI;                  // ... per tile (K and V)
    static constexpr int VBASE = STAGES * TILEB;           // byte offset of the V stages
    static constexpr int OROW = 32 * DT + 8;               // elements per staged output row (padded against bank conflicts)
    // Every wavefront has an area that first stages its Q tile (32 rows in the K tile layout) and later its output tile.  With
    // 8 wavefronts it lies behind the rings, since a second row tile's Q arrives while they are in use.  With 4 wavefronts there is one
    // row tile, and the rings themselves serve: the four Q tiles fill stage 1 of K and V, which the first key tile does not touch, and
    // the output comes when all keys are done.  64 KB instead of 99 at 128 channels: two workgroups fit a unit.
    // 65 to 96 channels in workgroups of 4 wavefronts: rows of 12 pieces, 48 KB, three workgroups a unit (items of 24..1600 rows over
    // 512 keys, 16 heads of 72 34.7 us in rows of 16 pieces, 32.6 so; a ragged batch of 50..2700 rows, 16 / 8 89.4, 75.0).
    // Up to 80 channels are five k-steps of Q K^T instead of six (the two 31.1 and 73.2 then; 8 x 4096, 16 heads of 72 831, 808).
    static constexpr int QW = 32 * PITCHB;
    static constexpr int WAREA = QW > 32 * OROW * 2 ? QW : 32 * OROW * 2;
    static constexpr bool IN_RINGS = WAVES == 4;
    static constexpr int LDS_BYTES = 2 * STAGES * TILEB + (IN_RINGS ? 0 : WAVES * WAREA);
    static_assert(!IN_RINGS || (2 * QW == TILEB && WAVES * WAREA <= 2 * STAGES * TILEB), "the rings hold four Q tiles in stage 1, four output tiles");
    static_assert(WAVES == 4 || WAVES == 8, "block shapes are 4 or 8 wavefronts");
    static_assert(STAGES == 2, "every wait below is for all outstanding loads, which fits a ring of two");
};

// Waits until at most `younger` tiles' worth of loads (TL per tile) are outstanding, younger <= MAXY.
template <int MAXY, int TL>
__device__ __forceinline__ void wait_tiles(int younger)
{
    if constexpr (MAXY == 0) wait_vmcnt<0>();
    else {
        if (younger >= MAXY) wait_vmcnt<MAXY * TL>();
        else wait_tiles<MAXY - 1, TL>(younger);
    }
}

template <int DP, int WAVES, int STAGES, bool RAGGED = false>
__global__ __launch_bounds__(WAVES * kWave, 2) void attn_mfma_kernel(AttnArgs a)
{
    using T = AttnTile<DP, WAVES, STAGES>;
    constexpr int kAttnWaves = WAVES, kStages = STAGES;
    constexpr int KSTEPS = T::KSTEPS, DT = T::DT, PITCH = T::PITCH, PITCHB = T::PITCHB, TILEB = T::TILEB;
    constexpr int NI = T::NI, TLOADS = T::TLOADS, VBASE = T::VBASE;
    extern __shared__ __attribute__((aligned(16))) __bf16 smem[];
    lds_char* const lds = (lds_char*)smem;    // K stages at [0, VBASE), V stages at [VBASE, 2 VBASE), then the wavefronts' areas

    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid >> 6;
    const int col = lane & 31, half = lane >> 5;
    const int HB = a.heads_per_block, RB = kAttnWaves >> a.hb_shift;   // heads and 32-row sub-tiles per block
    const int group = a.group, head_blocks = a.head_blocks;

    // blockIdx.y -> the workgroup's row tiles, the heaviest causal ones first (the linear dispatch order runs
    // through x first); blockIdx.x -> (head block, kv head, batch).  The quotients come from multiply-high with
    // constants prepared at launch: a chain of integer divisions here would delay the first load by half a
    // microsecond.  A paired launch gives workgroup y the row tiles n-1-y and then y (y-1 when n is odd, where
    // the heaviest tile stays alone): under the causal mask tile t has t+1 key tiles, so every workgroup gets
    // the same number of them, one workgroup per compute unit covers the launch, and the second tile's Q and
    // first K/V tile are fetched under the first one's last tiles and output stores.
    auto div_magic = [](uint32_t n, uint32_t magic) { return magic ? __umulhi(n, magic) : n; };
    int rt = a.row_tiles - 1 - static_cast<int>(blockIdx.y);
    int rt_next = !T::IN_RINGS && a.paired ? static_cast<int>(blockIdx.y) - (a.row_tiles & 1) : -1;
    const uint32_t bid = blockIdx.x;
    const uint32_t bid_hb = div_magic(bid, a.magic_head_blocks);      // = kv head + n_kv_heads * batch
    const int hb = static_cast<int>(bid - bid_hb * head_blocks);
    int item = static_cast<int>(div_magic(bid_hb, a.magic_kv_heads));
    const int g = static_cast<int>(bid_hb) - item * a.n_kv_heads;
    // (shift_items; the one integer division here, and only in launches that gain far more by it)
    if constexpr (RAGGED)
        if (a.item_shift) item = (item + static_cast<int>(blockIdx.y >> 2)) % a.batch;
    const int b = item;

    const int h = g * group + hb * HB + (w & (HB - 1));
    const int wrow = (w >> a.hb_shift) * 32;                  // this wavefront's first query row inside a row tile
    // Query rows of this sample and where they start.  Ragged launches (no mask, one row tile per workgroup): item b's
    // rows come from the table in the arguments, and a workgroup whose row tile lies past its item's end has nothing
    // to do (the grid covers the longest item); it leaves before any load or barrier.
    int seq_item = a.seq, kv_seq_item = a.kv_seq;
    int64_t q_first = b * a.qs[0], o_first = b * a.os[0], kv_first = b * a.ks[0];
    if constexpr (RAGGED) {
        const int32_t first = a.item_row[b];
        seq_item = a.item_row[b + 1] - first;
        q_first = static_cast<int64_t>(first) * a.qs[1];
        o_first = static_cast<int64_t>(first) * a.os[1];
        if (a.kv_packed) {                                    // keys and values packed like the queries (self-attention)
            kv_seq_item = seq_item;
            kv_first = static_cast<int64_t>(first) * a.ks[1];
        }
        if (rt * RB * 32 >= seq_item) return;
    }
    const int seq = seq_item, kv_seq = kv_seq_item;
    const float sl2 = a.scale * 1.4426950408889634f;          // scale * log2(e)

    // geometry of the row tile being computed
    int row0, block_row0, block_rows_end, qi, n_tiles;
    auto set_rows = [&](int t) {
        block_row0 = t * RB * 32;
        row0 = block_row0 + wrow;                             // this wavefront's first query row
        block_rows_end = min(block_row0 + RB * 32, seq);
        qi = row0 + col;                                      // this lane's query row
        const int kv_end = a.causal ? block_rows_end : kv_seq; // keys [0, kv_end) are visible to the block
        n_tiles = (kv_end + kBN - 1) / kBN;
    };
    set_rows(rt);
    const __bf16* kp = static_cast<const __bf16*>(a.k) + kv_first + g * a.ks[2];
    const __bf16* vp = static_cast<const __bf16*>(a.v) + kv_first + g * a.ks[2];
    const uint32_t row_bytes = static_cast<uint32_t>(a.ks[1]) * 2u;   // K/V token stride

    // Q first: its loads are the longest wait of the prologue, everything else is set up in their shadow.
    // Q goes through LDS as well (same swizzled layout as a K tile, 32 rows per wavefront, in the wavefront's
    // own area), so that the main loop holds no register-destination global load: the
    // compiler then never emits a vmcnt wait of its own there.
    const uint32_t q_lds = T::IN_RINGS ? (w & 1) * T::QW + TILEB + (w >> 1) * VBASE : 2 * VBASE + w * T::WAREA;
    const char* const qb = uniform_ptr(static_cast<const __bf16*>(a.q) + q_first + h * a.qs[2]);
    const uint32_t q_row_bytes = static_cast<uint32_t>(a.qs[1]) * 2u;
    const uint32_t q_lds_uni = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds)) + q_lds);
    // Slot -> (row, physical chunk) as for a K tile: instruction j covers rows 4j .. 4j+3 when a row has 16
    // chunks (8j .. 8j+7 when it has 8), and the chunk swizzle repeats every 16 rows, so instructions j and
    // j + 16/rows-per-instruction differ by a constant row offset only.
    auto q_slot_off = [&](int j, int first_row, bool clamp) {
        const int slot = j * kWave + lane;
        const int row = slot / PITCH;
        const int c = (slot % PITCH) ^ swz<PITCH>(row);
        const uint32_t cb = (c * 8 < a.head_dim) ? c * 16 : 0;
        const int r = clamp ? min(first_row + row, seq - 1) : first_row + row;
        return static_cast<uint32_t>(r) * q_row_bytes + cb;
    };
    auto issue_q = [&](int first_row) {                       // any row tile: rows past the sequence re-read its last row
        const char* base = scalar_copy(qb);
#pragma unroll
        for (int j = 0; j < PITCH / 2; ++j)
            dma16_at(base, q_slot_off(j, first_row, true), q_lds_uni, std::integral_constant<int, 0>{}, j);
    };
    // The Q rows of a workgroup's second row tile, which is never the last of the sequence (no clamping): the
    // offsets of the first 16 rows stay in registers, the tile's first row enters through the scalar base.
    constexpr int QJ = 16 * PITCH / kWave;                    // instructions per 16 rows
    uint32_t q_voff[QJ];
#pragma unroll
    for (int j = 0; j < QJ; ++j) q_voff[j] = q_slot_off(j, 0, false);
    auto issue_q_next = [&](int first_row) {
        const char* base0 = uniform_ptr(qb + static_cast<int64_t>(first_row) * q_row_bytes);
        const char* base1 = uniform_ptr(base0 + 16 * static_cast<int64_t>(q_row_bytes));
#pragma unroll
        for (int j = 0; j < PITCH / 2; ++j)
            dma16_at(j < QJ ? base0 : base1, q_voff[j % QJ], q_lds_uni, std::integral_constant<int, 0>{}, j);
    };
    issue_q(row0);
    // Global -> LDS: instruction j of wavefront w fills slots [(w*NI + j)*64, +64) of a tile; slot ->
    // (row, physical chunk); the lane fetches the logical chunk that belongs there.  Every lane always
    // loads: rows past the end of the sequence re-read the last row (their scores are masked), chunks past
    // head_dim re-read chunk 0 (they meet zero-filled Q columns, or produce output columns that are never
    // stored).  The tile's first key enters through the scalar base, so the per-lane offsets are loop
    // invariant; only the tile that holds the end of the sequence needs the clamped set.
    uint32_t ld_voff[NI], ld_voff_tail[NI];
    const int tail_tile = (kv_seq - 1) / kBN;               // the tile that may run past the keys
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int slot = (w * NI + j) * kWave + lane;
        const int row = slot / PITCH;
        const int c = (slot % PITCH) ^ swz<PITCH>(row);
        const uint32_t cb = (c * 8 < a.head_dim) ? c * 16 : 0;
        ld_voff[j] = row * row_bytes + cb;
        ld_voff_tail[j] = (min(tail_tile * kBN + row, kv_seq - 1) - tail_tile * kBN) * row_bytes + cb;
    }
    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(
        static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds)) + w * NI * kWave * 16);
    auto issue_tile = [&](int kt, auto stage_c) {
        constexpr int st = decltype(stage_c)::value;
        // (wave-uniform by construction; made so explicitly because the load takes its base in scalar registers)
        const char* kb = uniform_ptr(reinterpret_cast<const char*>(kp) + static_cast<int64_t>(kt) * kBN * row_bytes);
        const char* vb = uniform_ptr(reinterpret_cast<const char*>(vp) + static_cast<int64_t>(kt) * kBN * row_bytes);
        const bool tail = kt == tail_tile;
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const uint32_t off = tail ? ld_voff_tail[j] : ld_voff[j];
            dma16_at(kb, off, lds_wave, std::integral_constant<int, st * TILEB>{}, j);
            dma16_at(vb, off, lds_wave, std::integral_constant<int, st * TILEB + VBASE>{}, j);
        }
    };

    // Start the pipeline: tile 0 (the ring runs one tile ahead of the one being consumed)
    issue_tile(0, std::integral_constant<int, 0>{});

    // Q^T as B operand: lane (col, half) holds Q[qi][16 s + 8 half .. +7] for every k-step s.
    bf16x8 qreg[KSTEPS];
    auto read_q = [&]() {
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) {
            const bf16x8 t = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(
                lds + q_lds + col * PITCHB + (((2 * s + half) ^ swz<PITCH>(col & 15)) << 4));
            qreg[s] = t;
        }
        if (a.head_dim != DP) {                               // a padded head: the columns past head_dim count as zero
            const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s) qreg[s] = (16 * s + 8 * half < a.head_dim) ? qreg[s] : zero;
        }
        // in registers before the area is written again
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (DP % 32 == 0 && a.q_cs != nullptr) {
            // Rotary embedding of the query row in registers: the lane holds elements 16 s + 8 half + j, and with
            // head_dim a multiple of 32 the partner of an element, head_dim / 2 further on, sits KSTEPS / 2
            // k-steps later in the same lane.  (cos, sin) of the row's 8 consecutive pairs come as four 16-byte loads.
            constexpr int HS = KSTEPS / 2;
            const float2* cs_row = a.q_cs + (static_cast<int64_t>(b) * seq + min(qi, seq - 1)) * (DP / 2) + 8 * half;
#pragma unroll
            for (int s = 0; s < HS; ++s) {
                float2 cs[8];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float4 t = reinterpret_cast<const float4*>(cs_row + 16 * s)[v];
                    cs[2 * v] = make_float2(t.x, t.y);
                    cs[2 * v + 1] = make_float2(t.z, t.w);
                }
                bf16x8 lo = qreg[s], hi = qreg[s + HS];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float x0 = static_cast<float>(lo[j]), x1 = static_cast<float>(hi[j]);
                    float r0, r1;
                    rope_pair(x0, x1, cs[j].x, cs[j].y, r0, r1);
                    lo[j] = static_cast<__bf16>(r0);
                    hi[j] = static_cast<__bf16>(r1);
                }
                qreg[s] = lo; qreg[s + HS] = hi;
            }
        }
    };
    // Loads retire in order and Q was issued first: wait until only the tile's loads are outstanding.
    wait_vmcnt<TLOADS>();
    read_q();

    // Per-lane LDS read addresses (bytes) inside stage 0; stage, t, u add compile-time immediates.
    lds_char* kaddr[KSTEPS];              // K: row col, logical chunk 2s + half
#pragma unroll
    for (int s = 0; s < KSTEPS; ++s) {
        kaddr[s] = lds + col * PITCHB + (((2 * s + half) ^ swz<PITCH>(col & 15)) << 4);
        // opaque to the optimiser: one register per address, every use is register + immediate
        asm volatile("" : "+v"(kaddr[s]));
    }
    const int l16 = lane & 15, g16 = (lane >> 4) & 1;
    lds_char* vaddr[2][DT];               // V: row 4 half + 8 hi + l16/4 (+ 32t + 16u), columns 32dt + 16 g16 + 4 (l16 % 4)
#pragma unroll
    for (int hi = 0; hi < 2; ++hi)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const int low4 = 4 * half + 8 * hi + (l16 >> 2);
            const int el = 32 * dt + 16 * g16 + 4 * (l16 & 3);
            vaddr[hi][dt] = lds + VBASE + low4 * PITCHB + (((el >> 3) ^ swz<PITCH>(low4)) << 4) + (el & 7) * 2;
            asm volatile("" : "+v"(vaddr[hi][dt]));
        }

    constexpr int kDist = CIVIC_ATTN_DIST;                  // LDS fragments are read this many MFMAs ahead of their use
    f32x16 acc_o[DT];
    float m_run;                           // offset subtracted from the raw logits (a recent row maximum)
    float l_run[2];                        // running row sum, two partial accumulators
    const bf16x2 ones = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};

    // The arithmetic of one tile (stage ST of the ring) for this wavefront: NT = 2 for the whole tile, 1 for
    // its first 32 keys only.
    auto tile = [&](int kt, auto stage_c, auto nt_c) {
        constexpr int ST = decltype(stage_c)::value;
        constexpr int NT = decltype(nt_c)::value;
        const int key0 = kt * kBN;
        if (a.causal && key0 > row0 + 31) return;             // no key of the tile is visible to this wavefront
        // S^T tile: rows = keys (two 32-key sub-tiles), columns = this wavefront's 32 queries
        f32x16 acc_s[NT];                                     // raw logits
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc_s[t][r] = 0.f;
        // (fragments are read two MFMAs ahead of their use, in the order written: a scheduling barrier per MFMA
        // keeps that order whatever the register pressure around it)
        {
            auto read_k = [&](int i) __attribute__((always_inline)) {     // MFMA i = (k-step i / NT, sub-tile i % NT)
                return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(
                    kaddr[i / NT] + ST * TILEB + 32 * (i % NT) * PITCHB);
            };
            bf16x8 kf[kDist + 1];
#pragma unroll
            for (int i = 0; i < kDist; ++i) kf[i] = read_k(i);
#pragma unroll
            for (int i = 0; i < NT * KSTEPS; ++i) {
                if (i + kDist < NT * KSTEPS) kf[(i + kDist) % (kDist + 1)] = read_k(i + kDist);
                acc_s[i % NT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i % (kDist + 1)], qreg[i / NT], acc_s[i % NT], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        // mask only where the tile crosses the diagonal or the end of the sequence (wave-uniform)
        if ((a.causal && key0 + kBN - 1 > row0) || key0 + kBN > kv_seq) {
            // The lane sees the tile's keys below `lim` (end of the sequence, and its own row under the causal
            // mask).  Register r of sub-tile t holds tile key 32 t + 8 (r / 4) + r % 4 + 4 half, so one
            // per-lane threshold against a constant per register decides: a compare and a select each.
            int lim = kv_seq - key0;
            if (a.causal) lim = min(lim, qi - key0 + 1);
            const int thr = lim - 4 * half;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    acc_s[t][r] = 32 * t + 8 * (r >> 2) + (r & 3) < thr ? acc_s[t][r] : -INFINITY;
        }
        // P = exp2((acc_s - m_run) * scale * log2 e), rounded to bf16, laid out as the B operands; lt = the
        // lane's two partial row sums of the rounded probabilities (what the PV product actually uses).
        bf16x8 pb[NT][2];
        float lt[2];
        auto probs = [&]() __attribute__((always_inline)) {
            const float off = -m_run * sl2;
            lt[0] = 0.f; lt[1] = 0.f;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    u32x4 packed;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float p0 = __builtin_amdgcn_exp2f(fmaf(acc_s[t][8 * u + 2 * e], sl2, off));
                        const float p1 = __builtin_amdgcn_exp2f(fmaf(acc_s[t][8 * u + 2 * e + 1], sl2, off));
                        const bf16x2 pp = {static_cast<__bf16>(p0), static_cast<__bf16>(p1)};
                        packed[e] = __builtin_bit_cast(uint32_t, pp);
                        lt[e & 1] = __builtin_amdgcn_fdot2_f32_bf16(pp, ones, lt[e & 1], false);
                    }
                    pb[t][u] = __builtin_bit_cast(bf16x8, packed);
                }
        };
        // The offset m_run is not the exact running maximum.  The first tile sets it to that tile's
        // row maximum; afterwards it moves (never down) only when a tile's probabilities come out
        // large, a row maximum 2^20 or so above it, which the row sums reveal without a separate
        // maximum pass.  Until then every term stays far inside the fp32 and bf16 ranges, and since P,
        // the row sum and the output accumulator all carry the same factor 2^-m_run the result does
        // not depend on it.
        const bool first = kt == 0;
        if (!first) probs();
        if (first || __any(lt[0] + lt[1] > 1048576.f)) {
            float mq[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
            for (int c4 = 0; c4 < 2 * NT; ++c4) {
                const f32x16& x = acc_s[c4 >> 1];
                const int o = 8 * (c4 & 1);
                mq[c4] = fmaxf(max3(max3(x[o], x[o + 1], x[o + 2]), x[o + 3], x[o + 4]), max3(x[o + 5], x[o + 6], x[o + 7]));
            }
            float mx = fmaxf(fmaxf(mq[0], mq[1]), fmaxf(mq[2], mq[3]));
            mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));        // finite on the first tile: key 0 is visible to every row
            const float m_new = first ? mx : fmaxf(mx, m_run);
            if (!first) {
                const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * sl2);
                l_run[0] *= alpha; l_run[1] *= alpha;
#pragma unroll
                for (int t = 0; t < DT; ++t)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc_o[t][r] *= alpha;
            }
            m_run = m_new;
            probs();
        }
        l_run[0] += lt[0]; l_run[1] += lt[1];
        // O^T += V^T P^T.  The k-slot (half, e) of step (t, u) is key 32t + 16u + 8(e/4) + 4 half + e%4.
        {
            auto read_v = [&](int i) __attribute__((always_inline)) {     // MFMA i = (key step i / DT, output tile i % DT)
                const int dt = i % DT, row = 16 * (i / DT);
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4*)(vaddr[0][dt] + ST * TILEB + row * PITCHB));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4*)(vaddr[1][dt] + ST * TILEB + row * PITCHB));
                const s16x8 v8 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                return __builtin_bit_cast(bf16x8, v8);
            };
            bf16x8 vf[kDist + 1];
#pragma unroll
            for (int i = 0; i < kDist; ++i) vf[i] = read_v(i);
#pragma unroll
            for (int i = 0; i < NT * 2 * DT; ++i) {
                if (i + kDist < NT * 2 * DT) vf[(i + kDist) % (kDist + 1)] = read_v(i + kDist);
                acc_o[i % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i % (kDist + 1)], pb[i / (2 * DT)][(i / DT) % 2], acc_o[i % DT], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // The same arithmetic for an inner tile (not the first, nothing masked), written out so that one wavefront's
    // matrix and vector instructions alternate: the logits of the tile's second 32 keys are multiplied while the
    // probabilities of its first 32 keys are exponentiated, a pair of scores behind every MFMA, and those enter the
    // PV product while the second half is exponentiated.  The order below is the order wanted: a scheduling barrier
    // after every unit keeps the compiler from regrouping it, and bounds the registers it needs.  (Measured against
    // the plain order with the same explicit fragment prefetch: 1-2 % on the 8B-shaped launch, 2-3 % on long
    // sequences - the vector work mostly does not hide behind the MFMAs, whatever the order.)  The offset check runs
    // per half, before that half's probabilities are used; a half whose row sums come out large raises the offset,
    // rescales what has been accumulated (the first half's PV product included, which carried the old offset like
    // everything else) and redoes that half's exponentials.
    auto tile_fast = [&](auto stage_c) {
        constexpr int ST = decltype(stage_c)::value;
        auto read_k = [&](int s, int t) __attribute__((always_inline)) {
            return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(kaddr[s] + ST * TILEB + 32 * t * PITCHB);
        };
        auto read_v = [&](int i, int t) __attribute__((always_inline)) {      // fragment i = (u, dt) of key half t
            const int u = i / DT, dt = i % DT;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) s16x4*)(vaddr[0][dt] + ST * TILEB + (32 * t + 16 * u) * PITCHB));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) s16x4*)(vaddr[1][dt] + ST * TILEB + (32 * t + 16 * u) * PITCHB));
            const s16x8 v8 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            return __builtin_bit_cast(bf16x8, v8);
        };
        // scores 2i, 2i + 1 of a half -> word i of its packed probabilities, and the lane's partial row sums
        auto soft_pair = [&](const f32x16& x, int i, float off, uint32_t (&packed)[8], float (&lt)[2]) __attribute__((always_inline)) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(x[2 * i], sl2, off));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(x[2 * i + 1], sl2, off));
            const bf16x2 pp = {static_cast<__bf16>(p0), static_cast<__bf16>(p1)};
            packed[i] = __builtin_bit_cast(uint32_t, pp);
            lt[i & 1] = __builtin_amdgcn_fdot2_f32_bf16(pp, ones, lt[i & 1], false);
        };
        auto operand = [&](const uint32_t (&packed)[8], int u) __attribute__((always_inline)) {
            const u32x4 w = {packed[4 * u], packed[4 * u + 1], packed[4 * u + 2], packed[4 * u + 3]};
            return __builtin_bit_cast(bf16x8, w);
        };
        auto raise_offset = [&](const f32x16& x, uint32_t (&packed)[8], float (&lt)[2]) __attribute__((always_inline)) {
            float mx = fmaxf(fmaxf(max3(x[0], x[1], x[2]), max3(x[3], x[4], x[5])),
                             fmaxf(max3(x[6], x[7], x[8]), max3(x[9], x[10], x[11])));
            mx = fmaxf(fmaxf(mx, max3(x[12], x[13], x[14])), x[15]);
            mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
            const float m_new = fmaxf(mx, m_run);
            float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * sl2);
            // (The compiler counts no wait states into or out of an asm statement: an exponential's result may be read one instruction
            // later at the earliest, a product may read what a vector instruction wrote two later, and a vector instruction what a
            // product of 8 passes wrote 12 later.  The products into acc_o were issued before the sums that led here, which took longer;
            // these 24 states, all products being in front of them, do not rely on it.)
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_nop 15\n\ts_nop 7" : "+v"(alpha));
            l_run[0] *= alpha; l_run[1] *= alpha;
            // (in place, tied operands: the accumulators stay in the registers they have on the common path)
#pragma unroll
            for (int t = 0; t < DT; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float y = acc_o[t][r];
                    asm volatile("v_mul_f32 %0, %0, %1\n\ts_nop 1" : "+v"(y) : "v"(alpha));
                    acc_o[t][r] = y;
                }
            m_run = m_new;
            const float off = -m_run * sl2;
            lt[0] = 0.f; lt[1] = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) soft_pair(x, i, off, packed, lt);
        };
        constexpr int NF = 2 * DT;                            // V fragments per key half
        f32x16 s0, s1;
#pragma unroll
        for (int r = 0; r < 16; ++r) { s0[r] = 0.f; s1[r] = 0.f; }
        uint32_t pk0[8], pk1[8];
        float lt0[2] = {0.f, 0.f}, lt1[2] = {0.f, 0.f};
        // K fragments as one sequence of 2 KSTEPS reads (first half, then second), kDist MFMAs ahead of their use
        auto read_kseq = [&](int i) __attribute__((always_inline)) { return read_k(i % KSTEPS, i / KSTEPS); };
        bf16x8 kf[kDist + 1];
#pragma unroll
        for (int i = 0; i < kDist; ++i) kf[i] = read_kseq(i);
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) {                    // logits of the first half
            kf[(s + kDist) % (kDist + 1)] = read_kseq(s + kDist);
            s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s % (kDist + 1)], qreg[s], s0, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        const float off0 = -m_run * sl2;
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) {                    // logits of the second half | exponentials of the first
            if (KSTEPS + s + kDist < 2 * KSTEPS) kf[(KSTEPS + s + kDist) % (kDist + 1)] = read_kseq(KSTEPS + s + kDist);
            s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[(KSTEPS + s) % (kDist + 1)], qreg[s], s1, 0, 0, 0);
#pragma unroll
            for (int i = s * 8 / KSTEPS; i < (s + 1) * 8 / KSTEPS; ++i) soft_pair(s0, i, off0, pk0, lt0);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (__builtin_expect(__any(lt0[0] + lt0[1] > 1048576.f), 0)) raise_offset(s0, pk0, lt0);
        l_run[0] += lt0[0]; l_run[1] += lt0[1];
        const float off1 = -m_run * sl2;
        auto read_vseq = [&](int i) __attribute__((always_inline)) { return read_v(i % NF, i / NF); };
        bf16x8 vf[kDist + 1];
#pragma unroll
        for (int i = 0; i < kDist; ++i) vf[i] = read_vseq(i);
#pragma unroll
        for (int i = 0; i < NF; ++i) {                        // PV of the first half | exponentials of the second
            vf[(i + kDist) % (kDist + 1)] = read_vseq(i + kDist);
            acc_o[i % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i % (kDist + 1)], operand(pk0, i / DT), acc_o[i % DT], 0, 0, 0);
#pragma unroll
            for (int j = i * 8 / NF; j < (i + 1) * 8 / NF; ++j) soft_pair(s1, j, off1, pk1, lt1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (__builtin_expect(__any(lt1[0] + lt1[1] > 1048576.f), 0)) raise_offset(s1, pk1, lt1);
        l_run[0] += lt1[0]; l_run[1] += lt1[1];
#pragma unroll
        for (int i = 0; i < NF; ++i) {                        // PV of the second half
            if (NF + i + kDist < 2 * NF) vf[(NF + i + kDist) % (kDist + 1)] = read_vseq(NF + i + kDist);
            acc_o[i % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[(NF + i) % (kDist + 1)], operand(pk1, i / DT), acc_o[i % DT], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // One step of the pipeline: wait until the tile has landed, release the previous one, refill the freed
    // stage, compute.  At step q_issue the Q rows of the workgroup's next row tile are requested as well (their
    // area has been free since Q moved into registers); they land with a later tile.
    int q_issue = -1, next_row0 = 0;
    auto advance = [&](int kt, auto stage_c) __attribute__((always_inline)) {
        constexpr int ST = decltype(stage_c)::value;
        wait_vmcnt<0>();
        block_barrier();                                      // landed for every wavefront; tile kt-1 is released
        if (kt + 1 < n_tiles) issue_tile(kt + 1, std::integral_constant<int, (ST + 1) % kStages>{});
        if (kt == q_issue) issue_q_next(next_row0);
    };
    // a tile that may be the first, cross the diagonal or hold the end of the sequence
    auto step = [&](int kt, auto stage_c) __attribute__((always_inline)) {
        advance(kt, stage_c);
        // On the diagonal a wavefront whose rows all precede the tile's second half computes the first half
        // only: half the MFMAs and exponentials of that tile for half of the wavefronts, which the other
        // wavefront of the SIMD turns into time.  The same holds for a last tile whose second half lies past
        // the end of the sequence.
        if ((a.causal && kt * kBN + 32 > row0 + 31) || kt * kBN + 32 >= kv_seq) tile(kt, stage_c, std::integral_constant<int, 1>{});
        else tile(kt, stage_c, std::integral_constant<int, 2>{});
    };
    // an inner tile: whole, visible to every row of the workgroup, not the first
    auto step_inner = [&](int kt, auto stage_c) __attribute__((always_inline)) {
        advance(kt, stage_c);
        tile_fast(stage_c);
    };

    constexpr int OROW = T::OROW;
    constexpr int CPR = DP / 8;
    constexpr int kKvJ = (DP / 8 + 7) / 8;                     // pieces per thread, row and tensor
    constexpr int kKvRows = WAVES * kWave / 8;                 // rows per pass of the workgroup (64 with 8 wavefronts)
    __bf16* const o_s = reinterpret_cast<__bf16*>(smem) + (T::IN_RINGS ? w * T::WAREA : q_lds) / 2;   // the wavefront's area, now its output tile

    for (;;) {
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc_o[t][r] = 0.f;
        m_run = 0.f; l_run[0] = 0.f; l_run[1] = 0.f;
        const bool has_next = !T::IN_RINGS && rt_next >= 0;
        q_issue = has_next ? max(n_tiles - 3, 0) : -1;
        next_row0 = rt_next * RB * 32 + wrow;

        // Tile 0, then the inner tiles in a loop of their own (one code path, so the accumulators keep their
        // registers across it), then whatever is left: the diagonal, the end of the sequence.
        const int inner_end = min(a.causal ? (block_row0 + 1) / kBN : kv_seq / kBN, n_tiles);
        step(0, std::integral_constant<int, 0>{});
        int kt = 1;
        for (; kt + 1 < inner_end; kt += kStages) {
            step_inner(kt, std::integral_constant<int, 1>{});
            step_inner(kt + 1, std::integral_constant<int, 0>{});
        }
        for (; kt < n_tiles; kt += kStages) {
            step(kt, std::integral_constant<int, 1>{});
            if (kt + 1 < n_tiles) step(kt + 1, std::integral_constant<int, 0>{});
        }
        if (has_next) wait_vmcnt<0>();                        // the next Q rows (a one-tile pass waits nowhere else)
        __syncthreads();                                      // every tile consumed: the rings are free

        // what the epilogue needs of the tile just computed
        const int e_row0 = row0, e_block_row0 = block_row0, e_rows_end = block_rows_end;
        float l_sum = l_run[0] + l_run[1];
        const float l_tot = l_sum + __shfl_xor(l_sum, 32, kWave);
        const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
        if (has_next) {
            // the next row tile starts here: its first K/V tile flies while this one's output is stored, and
            // its Q rows move into registers before the area takes the output tile
            set_rows(rt_next);
            issue_tile(0, std::integral_constant<int, 0>{});
            read_q();
        }

        // Fused KV-cache write: the workgroup of the first head block copies the K and V rows of its own
        // query rows (which it has just streamed through LDS, so the reads hit L2) into the cache; the loads
        // of the first 64 rows go out before the output rows are stored and their stores after; taller blocks
        // take the rest in a plain loop at the end.
        // Copy layout: 8 threads per row, thread t takes row t / 8 of a 64-row group and the 16-byte pieces
        // t % 8, t % 8 + 8, ... of it, the same piece of K and of V (one address computation for both).
        u32x4 kv_piece[2 * kKvJ];
        // opaque copies: they keep the address arithmetic of the epilogue down here, instead of in registers
        // (or spilled) across the main loop
        int tid_late = tid, lane_late = lane;
        asm volatile("" : "+v"(tid_late), "+v"(lane_late));
        const int col_late = lane_late & 31, half_late = lane_late >> 5;
        const bool kv_fused = a.k_cache != nullptr && hb == 0;
        const int kv_cpr = a.head_dim / 8;                     // 16-byte pieces per row
        const int kv_rows = e_rows_end - e_block_row0;
        const int kv_r = tid_late >> 3, kv_c = tid_late & 7;
        // element offsets of piece (row r, chunk kv_c) from kp / vp and from the cache bases
        auto kv_src_off = [&](int r) { return static_cast<int64_t>(e_block_row0 + r) * a.ks[1] + kv_c * 8; };
        auto kv_dst_off = [&](int r) {
            const int64_t cache_row = (static_cast<int64_t>(b) * a.n_kv_heads + g) * a.s_max + a.pos0 + e_block_row0 + r;
            return cache_row * a.head_dim + kv_c * 8;
        };
        // Stage the wavefront's 32 x DP output tile in LDS and write it out as whole 16-byte row segments.
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                bf16x4 o4;
#pragma unroll
                for (int e = 0; e < 4; ++e) o4[e] = static_cast<__bf16>(acc_o[dt][4 * rq + e] * inv);
                *reinterpret_cast<bf16x4*>(&o_s[col_late * OROW + 32 * dt + 8 * rq + 4 * half_late]) = o4;
            }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (kv_fused) {                                       // (the accumulators are dead by now: registers are free)
            const int64_t so = kv_src_off(kv_r);
#pragma unroll
            for (int j = 0; j < kKvJ; ++j) {
                kv_piece[2 * j] = kv_piece[2 * j + 1] = u32x4{0u, 0u, 0u, 0u};
                if (kv_r < kv_rows && kv_c + 8 * j < kv_cpr) {
                    kv_piece[2 * j] = *reinterpret_cast<const u32x4*>(kp + so + 64 * j);
                    kv_piece[2 * j + 1] = *reinterpret_cast<const u32x4*>(vp + so + 64 * j);
                }
            }
        }
        __bf16* ob = static_cast<__bf16*>(a.out) + o_first + h * a.os[2];
        if (kWave % CPR == 0 && e_row0 + 32 <= seq && a.head_dim == DP) {
            // whole tile, unpadded head: the lane keeps its column, rows advance by 64 / CPR per store.  The stores are non-temporal: next a
            // model runs a product over these rows, which takes no longer for it (path, a layer norm over the merged rows and that product,
            // 4 x 938 rows, 32 / 8 heads of 128 260.0 -> 257.5 us, 8 x 938 455 -> 452, 16 frames 324 -> 323; a layer norm over the output instead
            // 104.5 -> 105.9), and the path alone is faster where inputs change from pass to pass (72.4 -> 70.5, 153 -> 151).  Not for rows
            // that end inside a line of 128 bytes (heads of 72: two grids of 64 x 64 54.3 -> 55.9).
            constexpr int RPI = kWave / CPR > 0 ? kWave / CPR : 1;
            const int r0 = lane_late / CPR, dc = lane_late - r0 * CPR;
            __bf16* dst = ob + static_cast<int64_t>(e_row0 + r0) * a.os[1] + dc * 8;
            const __bf16* src = &o_s[r0 * OROW + dc * 8];
            const int64_t stride = static_cast<int64_t>(RPI) * a.os[1];
#pragma unroll
            for (int it = 0; it < 32 * CPR / kWave; ++it)
                store_streaming(reinterpret_cast<bf16x8*>(dst + it * stride), *reinterpret_cast<const bf16x8*>(src + it * RPI * OROW));
        } else {
#pragma unroll
            for (int it = 0; it < 32 * CPR / kWave; ++it) {
                const int id = it * kWave + lane_late;
                const int r = id / CPR, dc = id - r * CPR;
                if (e_row0 + r < seq && dc * 8 < a.head_dim)
                    *reinterpret_cast<bf16x8*>(ob + static_cast<int64_t>(e_row0 + r) * a.os[1] + dc * 8) =
                        *reinterpret_cast<const bf16x8*>(&o_s[r * OROW + dc * 8]);
            }
        }
        if (kv_fused) {
            __bf16* const kc = static_cast<__bf16*>(a.k_cache);
            __bf16* const vc = static_cast<__bf16*>(a.v_cache);
            const int64_t d0 = kv_dst_off(kv_r);
            // (whole lines non-temporally: the caches are read in a later step.  Path alone and with the layer norm and the product,
            // inputs that change: 4 x 938 rows 70.6 -> 69.8, 256.8 -> 255.7 us, eight ragged prompts 73.2 -> 71.5, 247.5 -> 246.2)
            const bool whole_lines = a.head_dim % 64 == 0;
            auto put = [&](__bf16* p, const u32x4& x) {
                if (whole_lines) store_streaming(reinterpret_cast<u32x4*>(p), x);
                else *reinterpret_cast<u32x4*>(p) = x;
            };
#pragma unroll
            for (int j = 0; j < kKvJ; ++j)
                if (kv_r < kv_rows && kv_c + 8 * j < kv_cpr) {
                    put(kc + d0 + 64 * j, kv_piece[2 * j]);
                    put(vc + d0 + 64 * j, kv_piece[2 * j + 1]);
                }
            for (int r = kv_r + kKvRows; r < kv_rows; r += kKvRows) {   // taller blocks (fewer than 4 heads per block)
                const int64_t so = kv_src_off(r), dd = kv_dst_off(r);
#pragma unroll
                for (int j = 0; j < kKvJ; ++j)
                    if (kv_c + 8 * j < kv_cpr) {
                        put(kc + dd + 64 * j, *reinterpret_cast<const u32x4*>(kp + so + 64 * j));
                        put(vc + dd + 64 * j, *reinterpret_cast<const u32x4*>(vp + so + 64 * j));
                    }
            }
        }
        if (!has_next) break;
        rt = rt_next;
        rt_next = -1;
    }
}

// Block shape and grid of the MFMA kernel for these sizes; false if the grid does not fit (more than 65535
// row tiles, or a block index too large for the multiply-high decoding: n * d < 2^32 for n < per_rt).
template <int WAVES>
static bool mfma_geometry(AttnArgs& a, int64_t* per_rt)
{
    const int group = a.n_q_heads / a.n_kv_heads;
    a.heads_per_block = (group % 4 == 0) ? 4 : (group % 2 == 0) ? 2 : 1;
    const int rows_per_block = 32 * (WAVES / a.heads_per_block);
    const int64_t row_tiles = (static_cast<int64_t>(a.seq) + rows_per_block - 1) / rows_per_block;
    a.row_tiles = static_cast<int32_t>(row_tiles);
    a.group = group;
    a.head_blocks = group / a.heads_per_block;
    a.hb_shift = a.heads_per_block == 4 ? 2 : a.heads_per_block == 2 ? 1 : 0;
    *per_rt = static_cast<int64_t>(a.head_blocks) * a.n_kv_heads * a.batch;
    const int64_t d_max = a.head_blocks > a.n_kv_heads ? a.head_blocks : a.n_kv_heads;
    return *per_rt * d_max < (int64_t{1} << 32) && row_tiles <= 65535;
}

constexpr int64_t kComputeUnits = 256;

// Time (in arbitrary units) until the last workgroup of a causal launch ends when every compute unit runs one
// workgroup at a time and takes the next in dispatch order.  `paired`: workgroup y walks row tiles n-1-y and
// its partner (see the kernel).  A key tile costs 1.9 and a workgroup 5.5 around its tiles, 2 more for a
// second row tile whose start hides under the first one's end (microseconds measured on the 8B-shaped
// launch).  Only the ratio of the two results is used.
static double causal_makespan(int n_row_tiles, int64_t per_rt, int rows_per_block, int seq, bool paired)
{
    auto tiles_of = [&](int rt) {
        const int64_t end = std::min<int64_t>(static_cast<int64_t>(rt + 1) * rows_per_block, seq);
        return static_cast<double>((end + kBN - 1) / kBN);
    };
    const int items = paired ? (n_row_tiles + 1) / 2 : n_row_tiles;
    std::array<double, kComputeUnits> free_at;                // a min-heap of the units' free times
    free_at.fill(0.0);
    auto cmp = [](double x, double y) { return x > y; };
    double last = 0.0;
    for (int y = 0; y < items; ++y) {
        double cost = 5.5 + 1.9 * tiles_of(n_row_tiles - 1 - y);
        if (paired) {
            const int light = y - (n_row_tiles & 1);
            if (light >= 0) cost += 2.0 + 1.9 * tiles_of(light);
        }
        for (int64_t x = 0; x < per_rt; ++x) {
            std::pop_heap(free_at.begin(), free_at.end(), cmp);
            const double t = free_at.back() + cost;
            free_at.back() = t;
            std::push_heap(free_at.begin(), free_at.end(), cmp);
            if (t > last) last = t;
        }
    }
    return last;
}

// Whether the launch gives every workgroup two row tiles.  It pays under the causal mask when the row tiles
// do not all run at once anyway: the pairs are equally heavy, there are half as many workgroup starts, and a
// pair's second start is hidden.  Decided with the model above for grids small enough that the answer depends
// on how the workgroups fall onto the compute units; larger grids always pair.  The last answer is kept per
// thread so that a loop over layers does not model the same launch again.
static bool choose_paired(const AttnArgs& a, int64_t per_rt, int rows_per_block)
{
#ifdef CIVIC_ATTN_FORCE_PAIRED
    return CIVIC_ATTN_FORCE_PAIRED && a.row_tiles >= 2;           // build-time override for A/B measurements
#endif
    if (!a.causal || a.row_tiles < 2) return false;
    const int64_t blocks = per_rt * a.row_tiles;
    if (blocks <= kComputeUnits) return false;                // one generation as it is
    if (blocks > 16 * kComputeUnits) return true;
    struct Memo { int32_t row_tiles, rows_per_block, seq; int64_t per_rt; bool paired; };
    static thread_local Memo memo = {0, 0, 0, 0, false};
    if (memo.row_tiles == a.row_tiles && memo.rows_per_block == rows_per_block && memo.seq == a.seq && memo.per_rt == per_rt)
        return memo.paired;
    const bool paired = causal_makespan(a.row_tiles, per_rt, rows_per_block, a.seq, true) <
                        causal_makespan(a.row_tiles, per_rt, rows_per_block, a.seq, false);
    memo = {a.row_tiles, rows_per_block, a.seq, per_rt, paired};
    return paired;
}

// Whether the launch takes workgroups of 8 wavefronts (256 query rows x heads); `a` holds their geometry.  Workgroups of 4 wavefronts,
// two to a unit, do not wait for each other at every key tile, start and end under each other's products and leave less idle at the
// end of a launch; those of 8 bring half as many K/V tiles into LDS and can pair causal row tiles.  8 is faster only for long rows of
// keys where its workgroups fill the units (us, 8 and 4 wavefronts; bf16 heads of 128 unless said):
//   - up to 128 workgroups of 8: 4.  1 x 469 rows causal, 16 / 8 heads 14.9, 11.2; 3 x 550, 16 / 8 17.9, 13.7
//   - no mask, one generation of 8: 8 from 8 key tiles on.  2 x 2048 over 512 and 4096 keys, 16 / 16 of 72 19.3, 20.5 and 98, 102; 1 x 4096
//     98, 102; 2 x 1365 over 4096 85, 87, over its own 35.9, 34.8; three items of 700 to 1100 rows over 512 keys 17.6, 17.6; but two
//     of 656 and 1637 rows over 64 keys, 16 / 16 7.9, 7.4
//   - no mask, more: 8 for wide heads from 24 key tiles on where the last generation is full.  8 x 4096, 32 / 8 1986, 2077; 3 x 2323,
//     16 / 8 138, 143; 2 x 4096, 16 / 16 of 72 191, 197, but over 1024 keys 60.1, 58.4; 4 x 1618, 32 / 8 192, 182; eight items of 85 to
//     1365 rows over 256 keys, 16 / 16 of 72 23.3, 18.3; 2 x 4096, 16 / 16 of 64 152, 144
//   - causal: 8 for heads wider than 64 where pairs of row tiles fill their generations.  4 x 938, 32 / 8 38.5, 40.0; 1 x 3584, 32 / 8 105.5,
//     109.6, of 72 84.0, 86.6; 8 x 900, 16 / 16 of 72 49.8, 51.0; but 4 x 600, 32 / 8 22.8, 21.1; 8 x 3000, 32 / 8 of 72 441, 429; 8 x 900,
//     16 / 16 of 64 30.0, 26.8
//   - causal, not paired (items of different length never are): 8 beyond 44 key tiles and one generation.  Eight items of 3000 rows,
//     28 / 4 544, 615 and 32 / 8 563, 573, of 72 433, 444, but 32 / 8 of 96 482, 457; eight of 101 to 938, 32 / 8 39.8, 35.9; four of 300
//     to 2700, 32 / 8 178, 169
static bool eight_wavefronts(const AttnArgs& a, int64_t per_rt, bool ragged)
{
    if (a.causal && a.head_dim <= 64) return false;           // (before the model of a launch that is not taken)
    const int rows_per_block = 32 * (8 / a.heads_per_block);
    int64_t blocks = per_rt * a.row_tiles;
    if (ragged) {
        blocks = 0;
        for (int i = 0; i < a.batch; ++i)
            blocks += (static_cast<int64_t>(a.item_row[i + 1]) - a.item_row[i] + rows_per_block - 1) / rows_per_block * (per_rt / a.batch);
    }
    const bool paired = !ragged && choose_paired(a, per_rt, rows_per_block);
    if (a.causal && !paired) return blocks > kComputeUnits && a.seq > 44 * kBN;
    if (paired) blocks = per_rt * ((a.row_tiles + 1) / 2);
    const int64_t generations = (blocks + kComputeUnits - 1) / kComputeUnits;
    const bool full = 100 * blocks >= 85 * generations * kComputeUnits;
    if (a.causal) return full;
    if (generations == 1) return 2 * blocks > kComputeUnits && a.kv_seq > 7 * kBN;
    return a.head_dim > 64 && full && a.kv_seq > 23 * kBN;
}

// Whether every fourth row tile of a ragged launch begins with the next item.  Items of different length leave workgroups without work
// in the grid, and as the hardware hands workgroup n to unit n mod 256 (to XCD n mod 8, to the XCD's 32 units in turn), the row tiles of
// a long item, a fixed number of workgroups apart, may meet on a few units again and again, several of the heaviest to a unit.  Shifted
// items spread them then, and bring them together where the plain order has them on units of their own.  So both orders' loads of the
// 256 units are counted, 3 for a workgroup and 1 for a key tile, and the items are shifted if that makes the largest load smaller, or an
// XCD's by 8 % and a unit's by no more than a fifth larger (24 items, 12 / 3 44, 39; 294, 1197, 384 and 157 rows, 16 / 4 of 72 25.2, 24.0).
// (us, plain and shifted, and the ratio of the largest loads; heads of 128 unless said: eight items of 60..2700 rows, 16 / 8 105, 63, 0.25,
// 16 / 4 169, 60, 0.40, 8 / 2 90, 49, 0.62; eight of 117 to 938, 32 / 8 52, 40, 0.66; eight of 85 to 1365 over 256 keys, 16 / 16 of 72 19.9, 18.6, 0.67;
// but items of 2000, 500 and 200, 16 / 4 38.7, 43.5, 2.08, 36 / 6 of 64 39, 49, 1.39; five of 117..1500, 28 / 4 of 64 31.6, 36.8, 1.66; eight of
// 60..2700, 12 / 3 of 64 49, 60, 1.98; four of 1400..1600 over 512 keys, 12 / 12 of 64 18.0, 19.2, 1.00: K and V change their XCD.)
static bool shift_items(const AttnArgs& a, int64_t per_rt, int rows_per_block)
{
    if (a.row_tiles <= 4 || per_rt * a.row_tiles <= kComputeUnits) return false;   // (nothing to shift; a unit for every workgroup)
    constexpr uint32_t kUnits = kComputeUnits, kMask = kUnits - 1;
    static_assert((kUnits & kMask) == 0, "unit numbers are taken by a mask");
    const uint32_t per_item = static_cast<uint32_t>(per_rt / a.batch);
    int32_t left = 4096;                                      // tiles to count: a few microseconds on the host; longer launches are shifted
    int64_t plain[kUnits] = {}, shifted[kUnits] = {};         // differences from unit to unit
    auto put = [&](int64_t* load, uint32_t y, int at, int64_t cost) {
        const uint32_t from = (y * static_cast<uint32_t>(per_rt) + static_cast<uint32_t>(at) * per_item) & kMask, to = from + (per_item & kMask);
        load[from] += cost;
        if (to < kUnits) load[to] -= cost;
        else { load[0] += cost; load[to - kUnits] -= cost; }
    };
    for (int it = 0; it < a.batch; ++it) {
        const int64_t rows = static_cast<int64_t>(a.item_row[it + 1]) - a.item_row[it];
        const int32_t tiles = static_cast<int32_t>((rows + rows_per_block - 1) / rows_per_block);
        if ((left -= tiles) < 0) return true;
        uint32_t y = static_cast<uint32_t>(a.row_tiles) - 1;  // of row tile 0
        int at = it - static_cast<int>((y >> 2) % static_cast<uint32_t>(a.batch));   // the shifted item's place among the items
        if (at < 0) at += a.batch;
        for (int32_t rt = 0; rt < tiles; ++rt, --y) {
            const int64_t keys = a.causal ? std::min((rt + 1) * static_cast<int64_t>(rows_per_block), rows) : a.kv_packed ? rows : a.kv_seq;
            const int64_t cost = 3 + (keys + kBN - 1) / kBN;
            put(plain, y, it, cost);
            put(shifted, y, at, cost);
            if ((y & 3) == 0 && ++at == a.batch) at = 0;
        }
    }
    int64_t most[2] = {0, 0}, sum[2] = {0, 0}, xcd[2][8] = {};
    for (uint32_t u = 0; u < kUnits; ++u) {
        most[0] = std::max(most[0], sum[0] += plain[u]);
        most[1] = std::max(most[1], sum[1] += shifted[u]);
        xcd[0][u & 7] += sum[0];
        xcd[1][u & 7] += sum[1];
    }
    const int64_t xcd0 = *std::max_element(xcd[0], xcd[0] + 8), xcd1 = *std::max_element(xcd[1], xcd[1] + 8);
    return most[1] < most[0] || (5 * most[1] <= 6 * most[0] && 100 * xcd1 <= 92 * xcd0);
}

// The choice of a launch whose geometry with 8 wavefronts fits; `a` holds it.
static bool takes_eight(const AttnArgs& a, int64_t per_rt, bool ragged)
{
    AttnArgs four = a;
    int64_t per_rt4 = 0;
    return eight_wavefronts(a, per_rt, ragged) || !mfma_geometry<4>(four, &per_rt4);
}

template <int DP, int WAVES, int STAGES, bool RAGGED>
static int launch_mfma(AttnArgs& a, hipStream_t s)
{
    using T = AttnTile<DP, WAVES, STAGES>;
    int64_t per_rt = 0;
    if (!mfma_geometry<WAVES>(a, &per_rt)) return CIVIC_ERR_UNSUPPORTED;      // (the caller has checked)
    auto magic = [](int64_t d) { return d <= 1 ? 0u : static_cast<uint32_t>(((int64_t{1} << 32) + d - 1) / d); };
    a.magic_head_blocks = magic(a.head_blocks);
    a.magic_kv_heads = magic(a.n_kv_heads);
    a.paired = !RAGGED && WAVES == 8 && choose_paired(a, per_rt, 32 * (WAVES / a.heads_per_block)) ? 1 : 0;   // (pairs assume one length)
    if constexpr (RAGGED) a.item_shift = shift_items(a, per_rt, 32 * (WAVES / a.heads_per_block)) ? 1 : 0;
    const unsigned grid_y = static_cast<unsigned>(a.paired ? (a.row_tiles + 1) / 2 : a.row_tiles);
    constexpr size_t lds = T::LDS_BYTES;
    if (lds > 64 * 1024) {
        static std::atomic<uint64_t> allowed{0};
        const int rc = allow_dynamic_lds(reinterpret_cast<const void*>(attn_mfma_kernel<DP, WAVES, STAGES, RAGGED>), lds, &allowed);
        if (rc != CIVIC_OK) return rc;
    }
    civic::launch((attn_mfma_kernel<DP, WAVES, STAGES, RAGGED>), dim3(static_cast<unsigned>(per_rt), grid_y),
                       dim3(T::THREADS), lds, s, a);
    return check_launch();
}

#ifndef CIVIC_ATTN_STAGES
#define CIVIC_ATTN_STAGES 2
#endif
template <int WAVES, bool RAGGED>
static int launch_mfma_for(AttnArgs& a, hipStream_t s)
{
    if (a.head_dim <= 64) return launch_mfma<64, WAVES, CIVIC_ATTN_STAGES, RAGGED>(a, s);
    if (a.head_dim <= 80) return launch_mfma<80, WAVES, CIVIC_ATTN_STAGES, RAGGED>(a, s);
    if (a.head_dim <= 96) return launch_mfma<96, WAVES, CIVIC_ATTN_STAGES, RAGGED>(a, s);
    return launch_mfma<128, WAVES, CIVIC_ATTN_STAGES, RAGGED>(a, s);
}

}  // namespace civic

namespace civic {

// Attention, and the KV-cache write when k_cache is not null (inside the attention kernel where the
// MFMA path runs, as a second launch otherwise).
// item_row (host, batch + 1 ascending row numbers, or null): the queries and outputs of the `batch` items are packed
// along the token axis, item b owning rows [item_row[b], item_row[b + 1]) of q and out, and `seq` is the longest item;
// at most kRaggedItems items, no rotary table.  kv_packed: k and v are packed the same way (self-attention of every
// item over its own rows, `kv_seq` = `seq`; the mask and the caches are allowed); otherwise they are [batch, kv_seq]
// and there is neither.  dry_run: every check and nothing launched.
static int prefill_attn(const void* q, const void* k, const void* v, void* out, int dtype, int32_t batch, int32_t seq,
                        int32_t kv_seq, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, const int64_t* q_strides,
                        const int64_t* kv_strides, const int64_t* o_strides, int32_t causal, float softmax_scale,
                        void* k_cache, void* v_cache, int64_t s_max, int64_t pos0, const float* q_cos_sin, void* stream,
                        const int32_t* item_row = nullptr, bool dry_run = false, bool kv_packed = false)
{
    const int esz = dtype_size(dtype);
    if (!esz || !q_strides || !kv_strides || !o_strides) return CIVIC_ERR_INVALID_ARG;
    if (batch < 0 || seq < 0 || kv_seq < 0 || n_q_heads <= 0 || n_kv_heads <= 0 || head_dim <= 0) return CIVIC_ERR_INVALID_ARG;
    if (causal && kv_seq != seq) return CIVIC_ERR_INVALID_ARG;
    if (seq > 0 && kv_seq == 0) return CIVIC_ERR_INVALID_ARG;                             // a softmax over no key has no value
    if (batch > 0 && seq > 0 && (!q || !k || !v || !out)) return CIVIC_ERR_INVALID_ARG;   // no tokens: no tensors
    if (n_q_heads % n_kv_heads) return CIVIC_ERR_INVALID_ARG;
    if (head_dim % 8) return CIVIC_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out)) return CIVIC_ERR_INVALID_ARG;
    for (int i = 0; i < 3; ++i) {
        if (q_strides[i] < 0 || kv_strides[i] < 0 || o_strides[i] < 0) return CIVIC_ERR_INVALID_ARG;
        if ((q_strides[i] * esz) % 16 || (kv_strides[i] * esz) % 16 || (o_strides[i] * esz) % 16) return CIVIC_ERR_INVALID_ARG;
    }
    if (!(softmax_scale >= 0.f) || std::isinf(softmax_scale)) return CIVIC_ERR_INVALID_ARG;
    if (k_cache) {
        if (!v_cache || !aligned16(k_cache) || !aligned16(v_cache)) return CIVIC_ERR_INVALID_ARG;
        if (pos0 < 0 || s_max < 0 || pos0 + seq > s_max) return CIVIC_ERR_INVALID_ARG;
        if (kv_strides[2] < head_dim && n_kv_heads > 1) return CIVIC_ERR_INVALID_ARG;
    }
    if (q_cos_sin && (!aligned16(q_cos_sin) || head_dim % 4)) return CIVIC_ERR_INVALID_ARG;
    if (head_dim > CIVIC_MAX_HEAD_DIM || batch > 65535 || n_q_heads > 65535) return CIVIC_ERR_UNSUPPORTED;
    if (item_row && (batch > kRaggedItems || q_cos_sin || (!kv_packed && (causal || k_cache)))) return CIVIC_ERR_INVALID_ARG;
    if (kv_packed && (!item_row || kv_seq != seq)) return CIVIC_ERR_INVALID_ARG;
    if (batch == 0 || seq == 0) return CIVIC_OK;

    AttnArgs a;
    a.q = q; a.k = k; a.v = v; a.out = out;
    for (int i = 0; i < 3; ++i) { a.qs[i] = q_strides[i]; a.ks[i] = kv_strides[i]; a.os[i] = o_strides[i]; }
    a.batch = batch; a.seq = seq; a.kv_seq = kv_seq; a.n_q_heads = n_q_heads; a.n_kv_heads = n_kv_heads; a.head_dim = head_dim;
    a.causal = causal ? 1 : 0;
    a.scale = softmax_scale > 0.f ? softmax_scale : 1.0f / std::sqrt(static_cast<float>(head_dim));
    a.heads_per_block = 1; a.row_tiles = 0; a.pass_tiles = 0; a.paired = 0; a.item_shift = 0;
    a.group = n_q_heads / n_kv_heads; a.head_blocks = 0; a.hb_shift = 0; a.magic_head_blocks = 0; a.magic_kv_heads = 0;
    a.k_cache = k_cache; a.v_cache = v_cache; a.s_max = s_max; a.pos0 = pos0;
    a.q_cs = reinterpret_cast<const float2*>(q_cos_sin);
    for (int i = 0; i <= kRaggedItems; ++i) a.item_row[i] = item_row && i <= batch ? item_row[i] : 0;
    a.kv_packed = kv_packed ? 1 : 0;
    hipStream_t s = static_cast<hipStream_t>(stream);

    // the MFMA path addresses a K/V tile, and a head's Q rows, with 32-bit per-lane byte offsets, and its grid
    // has limits of its own; whatever falls outside takes the plain kernel
    int64_t per_rt = 0;
    // (with a rotary table the MFMA kernel needs an unpadded head whose halves are whole k-step pairs)
    const bool rope_fits = !q_cos_sin || head_dim == 64 || head_dim == 96 || head_dim == 128;
    if (dtype == CIVIC_BF16 && head_dim <= 128 && rope_fits && kv_strides[1] * 2 < (1 << 25) &&
        static_cast<int64_t>(seq) * q_strides[1] * 2 < (int64_t{1} << 32) && mfma_geometry<8>(a, &per_rt)) {
        if (dry_run) return CIVIC_OK;
        const bool eight = takes_eight(a, per_rt, item_row != nullptr);
        if (item_row) return eight ? launch_mfma_for<8, true>(a, s) : launch_mfma_for<4, true>(a, s);
        return eight ? launch_mfma_for<8, false>(a, s) : launch_mfma_for<4, false>(a, s);
    }
    if (dry_run) return CIVIC_OK;
    // everything else: the fp32 kernel (which also writes the caches when asked to); ragged items one launch each
    for (int32_t it = 0; it < (item_row ? batch : 1); ++it) {
        AttnArgs ai = a;
        if (item_row) {
            ai.batch = 1; ai.seq = item_row[it + 1] - item_row[it];
            ai.q = static_cast<const char*>(q) + static_cast<int64_t>(item_row[it]) * q_strides[1] * esz;
            ai.out = static_cast<char*>(out) + static_cast<int64_t>(item_row[it]) * o_strides[1] * esz;
            const int64_t kv_at = kv_packed ? static_cast<int64_t>(item_row[it]) * kv_strides[1] : static_cast<int64_t>(it) * kv_strides[0];
            ai.k = static_cast<const char*>(k) + kv_at * esz;
            ai.v = static_cast<const char*>(v) + kv_at * esz;
            if (kv_packed) ai.kv_seq = ai.seq;
            if (k_cache) {
                const int64_t cache_at = static_cast<int64_t>(it) * n_kv_heads * s_max * head_dim * esz;
                ai.k_cache = static_cast<char*>(k_cache) + cache_at;
                ai.v_cache = static_cast<char*>(v_cache) + cache_at;
            }
        }
        const int rc = dtype == CIVIC_BF16 ? launch_f32_for<true>(ai, s) : launch_f32_for<false>(ai, s);
        if (rc != CIVIC_OK) return rc;
    }
    return CIVIC_OK;
}

}  // namespace civic

// For tests, on the host alone (no part of civic.h): whether a ragged launch of bf16 attention, of up to 64 items with rows
// [offsets[i], offsets[i + 1]), shifts its items.  kv_seq > 0: over so many keys each; 0: over the item's own rows.
extern "C" int civic_attn_item_shift(int32_t batch, const int32_t* offsets, int32_t kv_seq, int32_t n_q_heads, int32_t n_kv_heads,
                                     int32_t head_dim, int32_t causal)
{
    using namespace civic;
    if (batch <= 0 || batch > kRaggedItems || !offsets || n_kv_heads <= 0 || n_q_heads % n_kv_heads || head_dim > 128) return -1;
    AttnArgs a = {};
    a.batch = batch; a.n_q_heads = n_q_heads; a.n_kv_heads = n_kv_heads; a.head_dim = head_dim;
    a.causal = causal ? 1 : 0; a.kv_packed = kv_seq > 0 ? 0 : 1;
    for (int32_t i = 0; i <= batch; ++i) a.item_row[i] = offsets[i];
    for (int32_t i = 0; i < batch; ++i) a.seq = std::max(a.seq, offsets[i + 1] - offsets[i]);
    a.kv_seq = kv_seq > 0 ? kv_seq : a.seq;
    int64_t per_rt = 0;
    if (!mfma_geometry<8>(a, &per_rt)) return -1;
    const bool eight = takes_eight(a, per_rt, true);
    if (!eight && !mfma_geometry<4>(a, &per_rt)) return -1;
    return shift_items(a, per_rt, 32 * ((eight ? 8 : 4) / a.heads_per_block)) ? 1 : 0;
}

// For tests, on the host alone (no part of civic.h): how a launch of bf16 attention of these sizes, one length for all samples, is
// taken.  4 or 8: wavefronts of a workgroup of the MFMA kernel; 9: of 8, with two row tiles each; 0: another kernel.
extern "C" int civic_attn_workgroup(int32_t batch, int32_t seq, int32_t kv_seq, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                                    int32_t causal)
{
    using namespace civic;
    if (batch <= 0 || seq <= 0 || kv_seq <= 0 || n_kv_heads <= 0 || n_q_heads % n_kv_heads || head_dim > 128) return 0;
    AttnArgs a = {};
    a.batch = batch; a.seq = seq; a.kv_seq = kv_seq; a.n_q_heads = n_q_heads; a.n_kv_heads = n_kv_heads; a.head_dim = head_dim;
    a.causal = causal ? 1 : 0;
    int64_t per_rt = 0;
    if (!mfma_geometry<8>(a, &per_rt)) return 0;
    if (!takes_eight(a, per_rt, false)) return 4;
    return choose_paired(a, per_rt, 32 * (8 / a.heads_per_block)) ? 9 : 8;
}

extern "C" int civic_prefill_attn(const void* q, const void* k, const void* v, void* out, int dtype, int32_t batch,
                                  int32_t seq, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                                  const int64_t* q_strides, const int64_t* kv_strides, const int64_t* o_strides,
                                  int32_t causal, float softmax_scale, void* stream)
{
    return civic::prefill_attn(q, k, v, out, dtype, batch, seq, seq, n_q_heads, n_kv_heads, head_dim, q_strides, kv_strides,
                               o_strides, causal, softmax_scale, nullptr, nullptr, 0, 0, nullptr, stream);
}

extern "C" int civic_prefill_attn_rope(const void* q, const void* k, const void* v, void* out, int dtype, int32_t batch,
                                       int32_t seq, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                                       const int64_t* q_strides, const int64_t* kv_strides, const int64_t* o_strides,
                                       int32_t causal, float softmax_scale, const float* q_cos_sin, void* stream)
{
    if (!q_cos_sin && batch > 0 && seq > 0) return CIVIC_ERR_INVALID_ARG;
    return civic::prefill_attn(q, k, v, out, dtype, batch, seq, seq, n_q_heads, n_kv_heads, head_dim, q_strides, kv_strides,
                               o_strides, causal, softmax_scale, nullptr, nullptr, 0, 0, q_cos_sin, stream);
}

extern "C" int civic_prefill_attn_kv(const void* q, const void* k, const void* v, void* out, void* k_cache, void* v_cache,
                                     int dtype, int32_t batch, int32_t seq, int32_t n_q_heads, int32_t n_kv_heads,
                                     int32_t head_dim, const int64_t* q_strides, const int64_t* kv_strides,
                                     const int64_t* o_strides, int64_t s_max, int64_t pos0, int32_t causal,
                                     float softmax_scale, void* stream)
{
    if ((!k_cache || !v_cache) && batch > 0 && seq > 0) return CIVIC_ERR_INVALID_ARG;
    return civic::prefill_attn(q, k, v, out, dtype, batch, seq, seq, n_q_heads, n_kv_heads, head_dim, q_strides, kv_strides,
                               o_strides, causal, softmax_scale, k_cache, v_cache, s_max, pos0, nullptr, stream);
}

extern "C" int civic_cross_attn(const void* q, const void* k, const void* v, void* out, int dtype, int32_t batch, int32_t n_q,
                                int32_t n_kv, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, const int64_t* q_strides,
                                const int64_t* kv_strides, const int64_t* o_strides, float softmax_scale, void* stream)
{
    return civic::prefill_attn(q, k, v, out, dtype, batch, n_q, n_kv, n_q_heads, n_kv_heads, head_dim, q_strides, kv_strides,
                               o_strides, 0, softmax_scale, nullptr, nullptr, 0, 0, nullptr, stream);
}

extern "C" int civic_cross_attn_ragged(const void* q, const void* k, const void* v, void* out, int dtype, int32_t batch,
                                       const int64_t* q_offsets, int32_t n_kv, int32_t n_q_heads, int32_t n_kv_heads,
                                       int32_t head_dim, const int64_t* q_strides, const int64_t* kv_strides,
                                       const int64_t* o_strides, float softmax_scale, void* stream)
{
    const int esz = civic::dtype_size(dtype);
    if (!esz || batch < 0 || !q_strides || !kv_strides || !o_strides) return CIVIC_ERR_INVALID_ARG;
    if (batch == 0) return CIVIC_OK;
    if (!q_offsets || q_offsets[0] != 0 || !q || !k || !v || !out) return CIVIC_ERR_INVALID_ARG;
    for (int32_t b = 0; b < batch; ++b)
        if (q_offsets[b + 1] <= q_offsets[b] || q_offsets[b + 1] - q_offsets[b] > INT32_MAX) return CIVIC_ERR_INVALID_ARG;
    // q_strides[0] / o_strides[0] (the batch stride of the rectangular call) are not used: items are packed along the
    // token axis (a token stride that keeps rows 16-byte aligned keeps every item's first row aligned as well).  Up to
    // kRaggedItems items go out as ONE launch whose workgroups look their item's rows up in a table in the kernel
    // arguments; longer lists in several.  Every group is checked before the first one is launched.
    if (q_offsets[batch] > INT32_MAX) return CIVIC_ERR_UNSUPPORTED;
    for (int pass = 0; pass < 2; ++pass)
        for (int32_t b0 = 0; b0 < batch; b0 += civic::kRaggedItems) {
            const int32_t nb = batch - b0 < civic::kRaggedItems ? batch - b0 : civic::kRaggedItems;
            int32_t rows[civic::kRaggedItems + 1], longest = 0;
            for (int32_t i = 0; i <= nb; ++i) rows[i] = static_cast<int32_t>(q_offsets[b0 + i]);
            for (int32_t i = 0; i < nb; ++i) longest = rows[i + 1] - rows[i] > longest ? rows[i + 1] - rows[i] : longest;
            const int rc = civic::prefill_attn(q, static_cast<const char*>(k) + static_cast<int64_t>(b0) * kv_strides[0] * esz,
                                               static_cast<const char*>(v) + static_cast<int64_t>(b0) * kv_strides[0] * esz, out, dtype, nb,
                                               longest, n_kv, n_q_heads, n_kv_heads, head_dim, q_strides, kv_strides, o_strides, 0,
                                               softmax_scale, nullptr, nullptr, 0, 0, nullptr, stream, rows, pass == 0);
            if (rc != CIVIC_OK) return rc;
        }
    return CIVIC_OK;
}


extern "C" int civic_prefill_attn_ragged(const void* q, const void* k, const void* v, void* out, int dtype, int32_t batch,
                                         const int64_t* row_offsets, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                                         const int64_t* q_strides, const int64_t* kv_strides, const int64_t* o_strides,
                                         int32_t causal, float softmax_scale, void* k_cache, void* v_cache, int64_t s_max,
                                         int64_t pos0, void* stream)
{
    const int esz = civic::dtype_size(dtype);
    if (!esz || batch < 0 || !q_strides || !kv_strides || !o_strides) return CIVIC_ERR_INVALID_ARG;
    if ((k_cache == nullptr) != (v_cache == nullptr)) return CIVIC_ERR_INVALID_ARG;
    if (batch == 0) return CIVIC_OK;
    if (!row_offsets || row_offsets[0] != 0 || !q || !k || !v || !out) return CIVIC_ERR_INVALID_ARG;
    for (int32_t b = 0; b < batch; ++b)
        if (row_offsets[b + 1] <= row_offsets[b] || row_offsets[b + 1] - row_offsets[b] > INT32_MAX) return CIVIC_ERR_INVALID_ARG;
    if (row_offsets[batch] > INT32_MAX) return CIVIC_ERR_UNSUPPORTED;
    // Groups of up to kRaggedItems samples, ONE launch each: attention of every sample over its own rows (the mask counts
    // from the sample's first row) and, with caches, the write of its K and V rows into its own cache rows.  Every
    // group is checked before the first one is launched.
    for (int pass = 0; pass < 2; ++pass)
        for (int32_t b0 = 0; b0 < batch; b0 += civic::kRaggedItems) {
            const int32_t nb = batch - b0 < civic::kRaggedItems ? batch - b0 : civic::kRaggedItems;
            int32_t rows[civic::kRaggedItems + 1], longest = 0;
            for (int32_t i = 0; i <= nb; ++i) rows[i] = static_cast<int32_t>(row_offsets[b0 + i]);
            for (int32_t i = 0; i < nb; ++i) longest = rows[i + 1] - rows[i] > longest ? rows[i + 1] - rows[i] : longest;
            const int64_t cache_at = static_cast<int64_t>(b0) * n_kv_heads * s_max * head_dim * esz;
            const int rc = civic::prefill_attn(q, k, v, out, dtype, nb, longest, longest, n_q_heads, n_kv_heads, head_dim, q_strides,
                                               kv_strides, o_strides, causal, softmax_scale,
                                               k_cache ? static_cast<char*>(k_cache) + cache_at : nullptr,
                                               v_cache ? static_cast<char*>(v_cache) + cache_at : nullptr, s_max, pos0, nullptr, stream,
                                               rows, pass == 0, true);
            if (rc != CIVIC_OK) return rc;
        }
    return CIVIC_OK;
}
