// One decode step of the accumulated attention score (paper Eq. 2, taken incrementally;
// order of operations as in Fig. 2): append the new token's row, let its query attend
// over every cached row, add the attention weights to the rows' running scores.
//
// Two launches, no atomics, no fences:
//   logits  HBM-bound GEMV.  A (batch, head) unit is cut into chunks of kDecodeChunk rows, one
//           workgroup each, so that even a single sequence fills the chip.  Every K row is
//           read exactly once, 16 bytes per lane, a group of lanes per row, all of the
//           workgroup's loads in flight before the first is used.  The workgroup leaves its
//           logits (base-2 domain, t = c*log2(e)*<q,k>) and its chunk's (max, sum of 2^(t-max))
//           in the workspace, and the one that owns the new row appends k, v, |v|_1 and pos.
//           With an output pointer (vatp_decode_attend_step) it also reads the V rows and leaves
//           the chunk's unnormalised share of the attention output (Eq. 1) in the workspace.
//   finish  one row per thread: every wavefront merges the unit's few chunk statistics into
//           log2 sum 2^t and applies S += 2^(t - lse2); 12 bytes per row, a tiny launch
//           ordered after the first by the stream.  Further workgroups merge the attention outputs.
#include "vatp_device.h"

namespace vatp {

namespace {

template <typename T, int D, bool kAttend, bool kStream>
__global__ __launch_bounds__(256) void decode_logits_kernel(
    const T *__restrict__ q, const T *__restrict__ k_new, const T *__restrict__ v_new,
    T *__restrict__ K, T *__restrict__ V, float *__restrict__ nrm, int32_t *__restrict__ pos,
    float *__restrict__ ws_logit, float2 *__restrict__ ws_part, float *__restrict__ ws_out,
    BatchMeta meta, int n_heads, int cap, int chunks_alloc, float scale_log2, int norm)
{
    constexpr int kE = Elt<T>::kPer16B;
    constexpr int kLanesPerRow = D / kE;
    constexpr int kRowsPerPass = 256 / kLanesPerRow;
    constexpr int kPasses = kDecodeChunk / kRowsPerPass;
    constexpr int kGroup = kPasses < 16 ? kPasses : 16;        // loads issued back to back

    __shared__ float s_logit[kDecodeChunk];

    // unit in the fast grid dimension: workgroups go to the 8 XCDs round-robin by linear id, so (with a
    // unit count that is a multiple of 8) a head's chunks, and the launch that consumes their logits,
    // share one XCD's L2
    const size_t unit = blockIdx.x;
    const int b = static_cast<int>(unit / n_heads), chunk = blockIdx.y;
    const int n0 = meta.len[b];            // rows cached before this step = index of the new row
    const int n = n0 + 1;
    const int row0 = chunk * kDecodeChunk;
    if (row0 >= n) return;
    const uint4 *Ku = reinterpret_cast<const uint4 *>(K + unit * cap * D);
    const uint4 *knew = reinterpret_cast<const uint4 *>(k_new + unit * D);
    const int tid = threadIdx.x;
    const int sub = tid % kLanesPerRow;
    const int rloc = tid / kLanesPerRow;
    const int lane = tid & 63, wave = tid >> 6;

    // Every load of this phase is requested before the first result is used: the query, the new row (in the
    // workgroup that owns it), then all of the workgroup's K rows.
    const uint4 q_raw = reinterpret_cast<const uint4 *>(q + unit * D)[sub];
    const bool owns_new_row = n0 >= row0 && n0 < row0 + kDecodeChunk && tid < kLanesPerRow;
    uint4 kraw = make_uint4(0, 0, 0, 0), vraw = make_uint4(0, 0, 0, 0);
    if (owns_new_row) {
        kraw = knew[sub];
        vraw = reinterpret_cast<const uint4 *>(v_new + unit * D)[sub];
    }

    // logits of the chunk's rows; the new row is read from the step's input, not from the cache
#pragma unroll
    for (int p0 = 0; p0 < kPasses; p0 += kGroup) {
        uint4 raw[kGroup];
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            const int r = row0 + (p0 + u) * kRowsPerPass + rloc;
            const uint4 *src = (r == n0) ? knew + sub : Ku + static_cast<size_t>(r) * kLanesPerRow + sub;
            raw[u] = (r < n) ? load_rows<kStream>(src) : make_uint4(0, 0, 0, 0);
        }
        if (p0 == 0 && owns_new_row) {
            // the workgroup that owns the new row stores k, v, |v| and pos into the caches
            reinterpret_cast<uint4 *>(K + unit * cap * D)[static_cast<size_t>(n0) * kLanesPerRow + sub] = kraw;
            reinterpret_cast<uint4 *>(V + unit * cap * D)[static_cast<size_t>(n0) * kLanesPerRow + sub] = vraw;
            const float new_norm = row_norm<T, kLanesPerRow>(norm, vraw);
            if (sub == 0) {
                nrm[unit * cap + n0] = new_norm;
                if (pos) pos[unit * cap + n0] = meta.aux[b];
            }
        }
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            const int rl = (p0 + u) * kRowsPerPass + rloc;
            const float dot = group_all_reduce<kLanesPerRow>(dot_16_bytes<T>(raw[u], q_raw), OpSum{});
            if (sub == 0) s_logit[rl] = (row0 + rl < n) ? dot * scale_log2 : -INFINITY;
        }
    }
    __syncthreads();

    // the chunk's logits go to the workspace; its statistics (maximum, sum of 2^(t - max)) are formed by one
    // wavefront, two rows per lane, without any exchange between wavefronts
    if (tid < kDecodeChunk && row0 + tid < n) ws_logit[unit * cap + row0 + tid] = s_logit[tid];
    float2 st = make_float2(0.f, 0.f);
    if (wave == 0 || kAttend) {
        st = chunk_stats_64x2(s_logit[lane], s_logit[lane + 64]);
        if (tid == 0) ws_part[unit * chunks_alloc + chunk] = st;
    }

    if constexpr (kAttend) {
        // this chunk's share of the attention output (paper Eq. 1), unnormalised and relative to the
        // chunk maximum:  o_c = sum_r 2^(t_r - max_c) v_r ; the finish launch rescales and adds the chunks
        // (every wavefront has formed the chunk maximum for itself above)
        const float mx = st.x;
        __shared__ float s_o[kRowsPerPass][D];
        const uint4 *Vu = reinterpret_cast<const uint4 *>(V + unit * cap * D);
        const uint4 *vnew = reinterpret_cast<const uint4 *>(v_new + unit * D);
        float oacc[kE];
#pragma unroll
        for (int e = 0; e < kE; ++e) oacc[e] = 0.f;
#pragma unroll
        for (int p0 = 0; p0 < kPasses; p0 += kGroup) {
            uint4 raw[kGroup];
#pragma unroll
            for (int u = 0; u < kGroup; ++u) {
                const int r = row0 + (p0 + u) * kRowsPerPass + rloc;
                const uint4 *src = (r == n0) ? vnew + sub : Vu + static_cast<size_t>(r) * kLanesPerRow + sub;
                raw[u] = (r < n) ? load_rows<kStream>(src) : make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < kGroup; ++u) {
                const float p = exp2f(s_logit[(p0 + u) * kRowsPerPass + rloc] - mx);   // 0 past the end
                float vf[kE];
                Elt<T>::unpack(raw[u], vf);
#pragma unroll
                for (int e = 0; e < kE; ++e) oacc[e] = fmaf(p, vf[e], oacc[e]);
            }
        }
#pragma unroll
        for (int e = 0; e < kE; ++e) s_o[rloc][sub * kE + e] = oacc[e];
        __syncthreads();
        if (tid < D) {
            float o = 0.f;
#pragma unroll
            for (int g = 0; g < kRowsPerPass; ++g) o += s_o[g][tid];
            ws_out[(unit * chunks_alloc + chunk) * D + tid] = o;
        }
    }
}

static __device__ const uint4 zero_row[32] = {};          // the longest row, 128 fp32 elements

// What a thread of the group kernel holds of its chunk: row slots u * kRowsPerPass + tid / kLanesPerRow, 16 bytes each.
template <typename T, int D>
struct ChunkRows {
    static constexpr int kE = Elt<T>::kPer16B;
    static constexpr int kLanesPerRow = D / kE;
    static constexpr int kRowsPerPass = 256 / kLanesPerRow;
    static constexpr int kPasses = kDecodeChunk / kRowsPerPass;

    // Requests the chunk's rows of one cache; the new row (index n0) comes from the step's input.  Rows past it read `past`
    // (keys: anything, their logits are -inf; values: zeros, as a weight of 0 does not undo an infinity), so that no load is
    // conditional: a row merged with a default value would be waited for where it is requested.
    template <bool kStream>
    __device__ static __forceinline__ void request(uint4 (&raw)[kPasses], const uint4 *cache, const uint4 *fresh, const uint4 *past,
                                                   int row0, int n0)
    {
        const int sub = threadIdx.x % kLanesPerRow, rloc = threadIdx.x / kLanesPerRow;
#pragma unroll
        for (int u = 0; u < kPasses; ++u) {
            const int r = row0 + u * kRowsPerPass + rloc;
            const uint4 *beyond = r == n0 ? fresh : past;
            raw[u] = load_rows<kStream>((r >= n0 ? beyond : cache + static_cast<size_t>(r) * kLanesPerRow) + sub);
        }
    }

    // Stores the new row's k, v, norm and position: by the first kLanesPerRow threads of the workgroup that owns it.
    __device__ static __forceinline__ void append(T *K, T *V, float *nrm, int32_t *pos, size_t row, const uint4 &k, const uint4 &v,
                                                  int norm, int new_pos)
    {
        reinterpret_cast<uint4 *>(K)[row * kLanesPerRow + threadIdx.x] = k;
        reinterpret_cast<uint4 *>(V)[row * kLanesPerRow + threadIdx.x] = v;
        const float new_norm = row_norm<T, kLanesPerRow>(norm, v);
        if (threadIdx.x == 0) {
            nrm[row] = new_norm;
            if (pos) pos[row] = new_pos;
        }
    }
};

// Sum over the wavefront's lanes that hold the same columns (lane groups of kLanes) of kN values per lane, kN halving where
// a step can hand half of the values over: v_permlane32_swap and v_permlane16_swap exchange halves of two registers, so
// one swap and one addition serve two values.  Value i of the result is value i + (kN / 2) * (lane >= 32) + ... of the
// input, see group_value.
template <int kLanes, int kN>
__device__ __forceinline__ void lane_group_sum(float (&v)[kN])
{
    auto swap_add = [&](auto pair, int half) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < half; ++i) {
            const unsigned x = __float_as_uint(v[i]), y = __float_as_uint(v[i + half]);
            const auto r = pair(x, y);
            v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
    };
    swap_add([](unsigned x, unsigned y) { return __builtin_amdgcn_permlane32_swap(x, y, false, false); }, kN / 2);
    if constexpr (kLanes <= 16)
        swap_add([](unsigned x, unsigned y) { return __builtin_amdgcn_permlane16_swap(x, y, false, false); }, kN / 4);
    if constexpr (kLanes <= 8) {
#pragma unroll
        for (int i = 0; i < kN / 4; ++i) v[i] += dpp_move<0x128>(v[i]);       // row_ror:8
    }
}
template <int kLanes, int kN>
__device__ __forceinline__ int group_value(int lane, int i)
{
    return i + (lane >> 5) * (kN / 2) + (kLanes <= 16 ? ((lane >> 4) & 1) * (kN / 4) : 0);
}

// The same launch for grouped-query attention: the workgroup reads its chunk of K rows once and
// forms the logits of all g query heads of the group against it (the point of sharing a K/V head:
// the cache is read once per group, not once per query head).  Logits and chunk statistics are kept
// per query head ([g, cap] and [g, chunks] per unit); with an output pointer each head's share of
// its attention output as well.  Instantiated for groups of up to kMaxG = 2, 4, 8 and 16.  Of what a thread keeps per
// query head (its slice of the outputs, 8 registers in bf16) a smaller one saves the arithmetic, and registers, so wavefronts,
// where these are what is short: with outputs and bf16 rows of 128, 132 registers and three wavefronts per SIMD up to 8 query
// heads, 192 and two for 16; rows of 64, 84, 84, 108 and 176.  The V rows are requested once the K rows are used up (requested with them, 4 % slower: registers again).  Measured, with
// outputs, against one instantiation for every group and reductions across lanes through LDS: 16 sequences of 8 heads x 4
// query heads, 307..2457 rows, 64.5 -> 33.6 us per fused step; 4 x 4 heads x 8 query heads x 4096 rows 48.4 -> 26.9.
template <typename T, int D, int kMaxG, bool kAttend, bool kStream>
__global__ __launch_bounds__(256) void decode_logits_group_kernel(
    const T *__restrict__ q, const T *__restrict__ k_new, const T *__restrict__ v_new,
    T *__restrict__ K, T *__restrict__ V, float *__restrict__ nrm, int32_t *__restrict__ pos,
    float *__restrict__ ws_logit, float2 *__restrict__ ws_part, float *__restrict__ ws_out,
    BatchMeta meta, int n_heads, int cap, int chunks_alloc, float scale_log2, int norm, int group)
{
    using R = ChunkRows<T, D>;
    constexpr int kE = R::kE, kLanesPerRow = R::kLanesPerRow, kRowsPerPass = R::kRowsPerPass, kPasses = R::kPasses;
    // bf16: the logits of a group are a (rows x D) by (D x g) product and go to the matrix cores (the chunk's rows staged
    // in LDS, every wavefront one 32-row tile); fp32 uses FMAs
    constexpr bool kMfma = sizeof(T) == 2;
    constexpr int kSteps = D / 16;

    constexpr int kOutBytes = kAttend ? 4 * kMaxG * D * 4 : 16, kRowBytes = kMfma ? kDecodeChunk * D * 2 : 16;
    __shared__ __attribute__((aligned(16))) char s_buf[kOutBytes > kRowBytes ? kOutBytes : kRowBytes];   // K rows, then outputs
    __shared__ float s_logit[kMaxG][kDecodeChunk];
    __shared__ __attribute__((aligned(16))) float s_p[kAttend ? kDecodeChunk : 1][kMaxG];              // weights 2^(t - max)

    const size_t unit = blockIdx.x;                            // K/V head
    const int b = static_cast<int>(unit / n_heads), chunk = blockIdx.y;
    const int n0 = meta.len[b];
    const int n = n0 + 1;
    const int row0 = chunk * kDecodeChunk;
    if (row0 >= n) return;
    const uint4 *knew = reinterpret_cast<const uint4 *>(k_new + unit * D);
    const uint4 *vnew = reinterpret_cast<const uint4 *>(v_new + unit * D);
    const int tid = threadIdx.x;
    const int sub = tid % kLanesPerRow, rloc = tid / kLanesPerRow;
    const int lane = tid & 63, wave = tid >> 6;

    // per lane: kSteps MFMA steps' worth of one head (lanes beyond the group read the last head: columns nobody uses), or a
    // slice of every head
    uint4 q_raw[kMfma ? kSteps : kMaxG];
#pragma unroll
    for (int i = 0; i < (kMfma ? kSteps : kMaxG); ++i) {
        if constexpr (kMfma)
            q_raw[i] = reinterpret_cast<const uint4 *>(q + (unit * group + min(lane & 31, group - 1)) * D)[i + kSteps * (lane >> 5)];
        else
            q_raw[i] = reinterpret_cast<const uint4 *>(q + (unit * group + min(i, group - 1)) * D)[sub];
    }
    const uint4 k_own = knew[sub], v_own = vnew[sub];
    uint4 k_raw[kPasses], v_raw[kAttend ? kPasses : 1];
    R::template request<kStream>(k_raw, reinterpret_cast<const uint4 *>(K + unit * cap * D), knew, knew, row0, n0);
    if (n0 - row0 < kDecodeChunk && tid < kLanesPerRow)
        R::append(K, V, nrm, pos, unit * cap + n0, k_own, v_own, norm, meta.aux[b]);

    if constexpr (kMfma) {
        static_assert(kMaxG <= 32, "a head per column of the tile");
        uint4 *s_k = reinterpret_cast<uint4 *>(s_buf);
#pragma unroll
        for (int u = 0; u < kPasses; ++u) {
            const int rl = u * kRowsPerPass + rloc;
            s_k[rl * kLanesPerRow + tile_slot<kLanesPerRow>(rl, sub)] = k_raw[u];
        }
        lds_barrier();
        const int ln = lane & 31, gl = lane >> 5;
        const int ar = 32 * wave + ln;             // this lane's row of the wavefront's tile
        floatx16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
        for (int st = 0; st < kSteps; ++st)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                as_bf16x8(s_k[ar * kLanesPerRow + tile_slot<kLanesPerRow>(ar, st + kSteps * gl)]), as_bf16x8(q_raw[st]), acc, 0, 0, 0);
        if (ln < group) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int rl = 32 * wave + acc_row(v) + 4 * gl;
                s_logit[ln][rl] = (row0 + rl < n) ? acc[v] * scale_log2 : -INFINITY;
            }
        }
    } else {
        static_assert(kMfma || kPasses == kLanesPerRow / 2, "the butterfly below pairs rows with lanes");
        float kf[kPasses][kE];
#pragma unroll
        for (int u = 0; u < kPasses; ++u) Elt<T>::unpack(k_raw[u], kf[u]);
#pragma unroll
        for (int i = 0; i < kMaxG; ++i) {
            if (i >= group) continue;
            float qf[kE];
            Elt<T>::unpack(q_raw[i], qf);
            // this lane's share of the dot products of head i with its kPasses rows ...
            float part[kPasses];
#pragma unroll
            for (int u = 0; u < kPasses; ++u) {
                part[u] = 0.f;
#pragma unroll
                for (int e = 0; e < kE; ++e) part[u] = fmaf(qf[e], kf[u][e], part[u]);
            }
            // ... summed over the row's lanes by a butterfly that halves the number of rows a lane is
            // responsible for at every step (the lane with the offset bit set keeps the upper half and
            // hands over the lower one): kPasses - 1 exchanges instead of kPasses * log2(lanes per row).
            // The lane ends up with the whole sum of row sub / 2.
#pragma unroll
            for (int off = kLanesPerRow / 2; off >= 2; off >>= 1) {
                const int half = off / 2;
                const bool upper = (sub & off) != 0;
#pragma unroll
                for (int j = 0; j < half; ++j) {
                    const float send = upper ? part[j] : part[j + half];
                    const float keep = upper ? part[j + half] : part[j];
                    part[j] = keep + __shfl_xor(send, off);
                }
            }
            part[0] += __shfl_xor(part[0], 1);
            if ((sub & 1) == 0) {
                const int rl = (sub >> 1) * kRowsPerPass + rloc;
                s_logit[i][rl] = (row0 + rl < n) ? part[0] * scale_log2 : -INFINITY;
            }
        }
    }
    lds_barrier();

    if constexpr (kAttend) R::template request<kStream>(v_raw, reinterpret_cast<const uint4 *>(V + unit * cap * D), vnew, zero_row, row0, n0);
    // per query head, by one wavefront (two rows per lane, no exchange between wavefronts): chunk statistics, logits to
    // the workspace, weights relative to the chunk maximum
    for (int i = wave; i < group; i += 4) {
        const float t0 = s_logit[i][lane], t1 = s_logit[i][lane + 64];
        const float2 st = chunk_stats_64x2(t0, t1);
        if (lane == 0) ws_part[(unit * group + i) * chunks_alloc + chunk] = st;
        float *lu = ws_logit + (unit * group + i) * cap + row0 + lane;
        if (row0 + lane < n) lu[0] = t0;
        if (row0 + lane + 64 < n) lu[64] = t1;
        if constexpr (kAttend) {
            s_p[lane][i] = exp2f(t0 - st.x);                       // 0 past the end
            s_p[lane + 64][i] = exp2f(t1 - st.x);
        }
    }

    if constexpr (kAttend) {
        // every head's share of its attention output (Eq. 1) over this chunk, relative to the head's
        // chunk maximum; rows are summed inside the wavefront first, then across the four through LDS
        lds_barrier();
        constexpr int kN = kMaxG * kE;
        float oacc[kN];                                        // [head][element of this lane's 16 bytes]
#pragma unroll
        for (int f = 0; f < kN; ++f) oacc[f] = 0.f;
#pragma unroll
        for (int u = 0; u < kPasses; ++u) {
            const int rl = u * kRowsPerPass + rloc;
            float vf[kE], p[kMaxG];
            Elt<T>::unpack(v_raw[u], vf);
#pragma unroll
            for (int i = 0; i < kMaxG; ++i) p[i] = s_p[rl][i];          // (heads beyond the group: anything, not stored)
#pragma unroll
            for (int i = 0; i < kMaxG; ++i)
#pragma unroll
                for (int e = 0; e < kE; ++e) oacc[i * kE + e] = fmaf(p[i], vf[e], oacc[i * kE + e]);
        }
        lane_group_sum<kLanesPerRow, kN>(oacc);
        float *s_o = reinterpret_cast<float *>(s_buf) + wave * kMaxG * D;
        constexpr int kLeft = kLanesPerRow <= 16 ? kN / 4 : kN / 2;
        if (kLanesPerRow >= 16 || (lane & 8) == 0) {
#pragma unroll
            for (int f = 0; f < kLeft; ++f) {
                const int v = group_value<kLanesPerRow, kN>(lane, f);
                s_o[v / kE * D + sub * kE + v % kE] = oacc[f];
            }
        }
        lds_barrier();
        const float *o = reinterpret_cast<const float *>(s_buf);
        for (int idx = tid; idx < group * D; idx += 256) {
            const int i = idx / D, x = idx % D;
            ws_out[((unit * group + i) * chunks_alloc + chunk) * D + x] =
                (o[idx] + o[kMaxG * D + idx]) + (o[2 * kMaxG * D + idx] + o[3 * kMaxG * D + idx]);
        }
    }
}

// Workgroups of one unit: row_blocks of 256 rows each, then (with an output) one per query head of the group.
template <int kMaxG, int D>
__global__ __launch_bounds__(256) void decode_finish_kernel(float *__restrict__ S,
                                                            const float *__restrict__ ws_logit,
                                                            const float2 *__restrict__ ws_part,
                                                            const float *__restrict__ ws_out,
                                                            float *__restrict__ out, BatchMeta meta, int n_heads,
                                                            int cap, int chunks_alloc, int group, int row_blocks)
{
    const size_t unit = blockIdx.x;
    const int b = static_cast<int>(unit / n_heads);
    const int n0 = meta.len[b], n = n0 + 1;
    const int n_chunks = (n + kDecodeChunk - 1) / kDecodeChunk;
    const float2 *part = ws_part + unit * group * chunks_alloc;
    if (static_cast<int>(blockIdx.y) >= row_blocks) {
        const size_t i = blockIdx.y - row_blocks;
        merge_head_output<D>(out + (unit * group + i) * D, ws_out + (unit * group + i) * chunks_alloc * D, part + i * chunks_alloc,
                             n_chunks, 256);
        return;
    }
    const int row0 = static_cast<int>(blockIdx.y) * 256;
    const int r = row0 + static_cast<int>(threadIdx.x);          // one row per thread
    if (row0 >= n) return;
    float2 stats[kMaxG];
    load_group_stats<kMaxG>(part, chunks_alloc, group, n_chunks, stats);
    float logit[kMaxG], s_old = 0.f;
    load_group_logits<kMaxG>(logit, ws_logit + unit * group * cap, cap, group, r, r < n);
    if (r < n && r != n0) s_old = S[unit * cap + r];
    // the softmax denominators from the unit's chunk statistics (per wavefront, one round trip)
    float lse2[kMaxG];
    merge_group_stats<kMaxG>(part, chunks_alloc, group, n_chunks, stats, lse2);
    if (r < n) S[unit * cap + r] = s_old + group_weight<kMaxG>(logit, lse2, group);
}

}  // namespace

hipError_t launch_decode(int dtype, int head_dim, const void *q, const void *k, const void *v,
                         void *K, void *V, float *S, float *nrm, int32_t *pos, float *ws_logit,
                         float2 *ws_part, float *ws_out, float *out, bool finish, const BatchMeta &meta,
                         const Geometry &g, hipStream_t st)
{
    const int chunks_alloc = (g.cap + kDecodeChunk - 1) / kDecodeChunk;
    const unsigned units = static_cast<unsigned>(g.batch) * g.n_heads;
    dim3 grid(units, (g.max_len + kDecodeChunk - 1) / kDecodeChunk), block(256);
    const bool attend = ws_out != nullptr;
    // (the group kernel is instantiated for groups of up to 2, 4, 8 and 16: the smallest that fits)
#define VATP_DEC_L(KERNEL, T, ...)                                                                           \
    hipLaunchKernelGGL((KERNEL), grid, block, 0, st, static_cast<const T *>(q), static_cast<const T *>(k),     \
                       static_cast<const T *>(v), static_cast<T *>(K), static_cast<T *>(V), nrm, pos, ws_logit, ws_part, \
                       ws_out, meta, g.n_heads, g.cap, chunks_alloc, g.scale_log2, g.norm, ##__VA_ARGS__)
#define VATP_DEC_A(T, D, A, STREAM)                                                                          \
    do {                                                                                                     \
        if (g.group > 8) VATP_DEC_L((decode_logits_group_kernel<T, D, 16, A, STREAM>), T, g.group);          \
        else if (g.group > 4) VATP_DEC_L((decode_logits_group_kernel<T, D, 8, A, STREAM>), T, g.group);      \
        else if (g.group > 2) VATP_DEC_L((decode_logits_group_kernel<T, D, 4, A, STREAM>), T, g.group);      \
        else if (g.group > 1) VATP_DEC_L((decode_logits_group_kernel<T, D, 2, A, STREAM>), T, g.group);      \
        else VATP_DEC_L((decode_logits_kernel<T, D, A, STREAM>), T);                                         \
    } while (0)
#define VATP_DEC(T, D)                                                                                       \
    do {                                                                                                     \
        if (attend && g.stream) VATP_DEC_A(T, D, true, true);                                                \
        else if (attend) VATP_DEC_A(T, D, true, false);                                                      \
        else if (g.stream) VATP_DEC_A(T, D, false, true);                                                    \
        else VATP_DEC_A(T, D, false, false);                                                                 \
    } while (0)
    if (dtype == VATP_F32 && head_dim == 64) VATP_DEC(float, 64);
    else if (dtype == VATP_F32) VATP_DEC(float, 128);
    else if (head_dim == 64) VATP_DEC(bf16_t, 64);
    else VATP_DEC(bf16_t, 128);
#undef VATP_DEC
#undef VATP_DEC_A
#undef VATP_DEC_L
    if (finish) {   // (the fused decode-and-evict step has its own second launch)
        const int row_blocks = (g.max_len + 255) / 256;
        const dim3 fgrid(units, row_blocks + (out ? g.group : 0));
#define VATP_FIN_D(G, D)                                                                                          \
    hipLaunchKernelGGL((decode_finish_kernel<G, D>), fgrid, block, 0, st, S, ws_logit, ws_part, ws_out, out, meta, g.n_heads, \
                       g.cap, chunks_alloc, g.group, row_blocks)
#define VATP_FIN(G)                                \
    do {                                           \
        if (head_dim == 64) VATP_FIN_D(G, 64);     \
        else VATP_FIN_D(G, 128);                   \
    } while (0)
        if (g.group > 8) VATP_FIN(VATP_MAX_GROUP);
        else if (g.group > 4) VATP_FIN(8);
        else if (g.group > 2) VATP_FIN(4);
        else if (g.group > 1) VATP_FIN(2);
        else VATP_FIN(1);
#undef VATP_FIN
#undef VATP_FIN_D
    }
    return hipGetLastError();
}

}  // namespace vatp
