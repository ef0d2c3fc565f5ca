// Second launch of the fused decode-and-evict step: finishes the softmax of the new query,
// adds the attention weights to the running scores (paper Eq. 2, incrementally), finds the one
// row per head that has to leave (smallest S * nrm among the rows that are neither sink nor
// recent, Eq. 4; the highest index among equals) and brings the other cache set up to date.
//
// The two cache sets alternate as input and output.  After a step that removed input row e,
// the old input set still agrees with the new state in its rows 0 .. e-1, so the next step
// (which writes into it) only has to rewrite rows from min(synced, e') on, where e' is its own
// evicted row.  The per-head count `synced` travels in a small device array.  Rows that have
// just left the recent window carry the smallest accumulated scores, so in practice only about
// `recent` rows move per step instead of the whole cache; the scores themselves change in
// every row and are rewritten in full.
//
// Grid: (units, G), and with an attention output one more workgroup per query head, which merges the chunks' shares of
// it (vatp_device.h).  Each of a head's G workgroups repeats the cheap part (12 bytes per row from L2: logit, S, nrm) to
// learn the evicted row by itself, then takes a 1/G share of the stores, so the launch needs no exchange between workgroups.
//
// What bounds it is a chain of round trips to memory, not bytes, so everything that can be is requested at the start:
//   own rows    a workgroup owns a range of INPUT rows and scans the head from there on, round the end: what it scans
//               first is what it stores later, and it still holds those scores when the evicted row is known;
//   recent rows no row behind e* = n - recent - 1, the last one that may leave, can leave, so they move down by one
//               whichever row does: loaded with the scan, stored without waiting for the decision.
// Only rows between min(synced, evicted) and e* are copied afterwards; normally there are none.  This launch, before (scan,
// then scores, then rows, each with a round trip of its own) / now: 16 sequences of 8 heads x 4 query heads, 307..2457
// rows, 13.3 / 8.8 us, 32 heads x 2049 rows 6.5 / 6.0, 4 heads x 129 rows 5.5 / 4.7.
//
// Arithmetic is the same, operation for operation, as decode_finish_kernel followed by the
// evict-one gather, so both routes give identical bits.
#include "vatp_device.h"

namespace vatp {

namespace {

constexpr int kThreads = 512;

// What a row's new score is made of.
template <int kMaxG>
struct ScanRow {
    float t[kMaxG], s, w, gone, lo;        // logits, old score, norm; windowed: the weight that leaves, low-order part
    int col;                               // windowed: column of the ring
};

template <typename T, int D, int kMaxG, bool kWindowed>
__global__ __launch_bounds__(kThreads) void decode_prune_kernel(
    const T *__restrict__ K, const T *__restrict__ V, const float *__restrict__ S,
    const float *__restrict__ nrm, const int32_t *__restrict__ pos, T *__restrict__ K_out,
    T *__restrict__ V_out, float *__restrict__ S_out, float *__restrict__ nrm_out,
    int32_t *__restrict__ pos_out, int32_t *__restrict__ kept_idx, const int32_t *__restrict__ synced_in,
    int32_t *__restrict__ synced_out, const float *__restrict__ ws_logit, const float2 *__restrict__ ws_part,
    const float *__restrict__ ws_out, float *__restrict__ out, WindowArgs win, BatchMeta meta, int n_heads,
    int cap, int cap_out, int chunks_alloc, int n_sink, int recent, int group, int stream, int G)
{
    constexpr int kE = Elt<T>::kPer16B;
    constexpr int kLanesPerRow = D / kE;
    constexpr int kRowsPerPass = kThreads / kLanesPerRow;

    __shared__ unsigned long long s_min[kThreads / 64];

    // workgroups go to the 8 XCDs round-robin by linear id = unit + units * g: with the unit in the fast
    // dimension a head's G workgroups meet in one XCD's L2 (unit count a multiple of 8), where the rows
    // they all scan are fetched once
    const size_t unit = blockIdx.x;
    const int g = blockIdx.y;
    const int b = static_cast<int>(unit / n_heads);
    const int n0 = meta.len[b], n = n0 + 1, B = meta.aux[b];
    const int n_keep = n < B ? n : B;
    const int tid = threadIdx.x;
    const int n_chunks = (n + kDecodeChunk - 1) / kDecodeChunk;
    const float2 *part = ws_part + unit * group * chunks_alloc;
    if (g >= G) {
        const size_t i = g - G;
        merge_head_output<D>(out + (unit * group + i) * D, ws_out + (unit * group + i) * chunks_alloc * D, part + i * chunks_alloc,
                             n_chunks, kThreads);
        return;
    }
    const float *Su = S + unit * cap;
    const float *Nu = nrm + unit * cap;
    const float *Lu = ws_logit + unit * group * cap;       // the group's logits: query head i at Lu + i * cap
    const bool evicts = n > B;
    const int lo = n_sink, hi = n - recent;                // rows [lo, hi) may leave

    // this workgroup's rows, in whole 256-byte lines of a row array, and the rows it scans from the first of them on
    const int share = ((n + G - 1) / G + 63) & ~63;
    const int own0 = min(g * share, n);
    const int n_own = min(share, n - own0);
    const int n_scan = evicts ? n : n_own;
    auto scan_row = [&](int i) { const int r = own0 + i; return r < n ? r : r - n; };

    // history window (Eq. 3): the ring row this step writes, the one that leaves the window, and
    // the column of every row (the appended row takes the free column and has no past)
    const int step = kWindowed ? win.step[b] : 0;
    float *h_write = kWindowed ? win.hist + (unit * win.rows + step % win.rows) * static_cast<size_t>(win.cap_hist) : nullptr;
    const float *h_leave =
        kWindowed ? win.hist + (unit * win.rows + (step + 1) % win.rows) * static_cast<size_t>(win.cap_hist) : nullptr;
    const int new_col = kWindowed ? win.free_in[unit] : 0;
    auto column = [&](int r) { return r == n0 ? new_col : win.hid[unit * cap + r]; };

    // kScan rows per thread and round trip (each brings kMaxG logits).  No load is conditional, so that none is waited
    // for where it is requested: indexes past the end read the last row, and nobody uses what comes back.
    constexpr int kScan = kMaxG > 8 ? 1 : 4;
    auto request = [&](ScanRow<kMaxG> (&rows)[kScan], int i0) __attribute__((always_inline)) {
        if constexpr (kWindowed) {
#pragma unroll
            for (int u = 0; u < kScan; ++u) rows[u].col = win.hid[unit * cap + scan_row(min(i0 + u * kThreads, n - 1))];
        }
#pragma unroll
        for (int u = 0; u < kScan; ++u) {
            const int r = scan_row(min(i0 + u * kThreads, n - 1));
#pragma unroll
            for (int i = 0; i < kMaxG; ++i) rows[u].t[i] = Lu[static_cast<size_t>(min(i, group - 1)) * cap + r];
            rows[u].s = Su[r];
            rows[u].w = Nu[r];
            if constexpr (kWindowed) rows[u].lo = win.s_lo[unit * cap + r];
        }
        if constexpr (kWindowed) {
#pragma unroll
            for (int u = 0; u < kScan; ++u) {
                if (scan_row(min(i0 + u * kThreads, n - 1)) == n0) rows[u].col = new_col;
                rows[u].gone = h_leave[rows[u].col];
            }
        }
    };
    // new score from the old one, this step's attention weight and (windowed) the weight that leaves the
    // window: accumulated scores are one fp32 addition; windowed scores are carried in two floats (window_update),
    // so that adding a weight and subtracting the same float w+1 steps later leaves no residue behind
    auto combine = [&](const ScanRow<kMaxG> &row, int r, const float (&lse2)[kMaxG], float &p, float &lo_new) {
        p = group_weight<kMaxG>(row.t, lse2, group);
        lo_new = 0.f;
        float score = r == n0 ? 0.f : row.s;
        if constexpr (!kWindowed) return score + p;
        if (r != n0) lo_new = row.lo;
        window_update(score, lo_new, r == n0 ? 0.f : row.gone, p);
        return score;
    };

    // requested together: chunk statistics, the first rows of the scan, and the rows behind e* (K and V row, norm,
    // position, column; kMove passes of them, with G workgroups all there are in most calls)
    const int synced = synced_in[unit];
    float2 stats[kMaxG];
    load_group_stats<kMaxG>(part, chunks_alloc, group, n_chunks, stats);
    ScanRow<kMaxG> held[kScan];
    request(held, tid);

    const uint4 *Ku = reinterpret_cast<const uint4 *>(K + unit * cap * D);
    const uint4 *Vu = reinterpret_cast<const uint4 *>(V + unit * cap * D);
    uint4 *Ko = reinterpret_cast<uint4 *>(K_out + unit * cap_out * D);
    uint4 *Vo = reinterpret_cast<uint4 *>(V_out + unit * cap_out * D);
    const int sub = tid % kLanesPerRow;
    const int rloc = tid / kLanesPerRow;
    struct MovedRow { uint4 k, v; float w; int pos, col; };
    auto fetch = [&](MovedRow &m, int src) __attribute__((always_inline)) {
        const size_t at = static_cast<size_t>(src) * kLanesPerRow + sub;
        if (stream) { m.k = load_stream(Ku + at); m.v = load_stream(Vu + at); }       // (uniform)
        else { m.k = Ku[at]; m.v = Vu[at]; }
        m.w = Nu[src];
        m.pos = pos ? pos[unit * cap + src] : 0;
        m.col = kWindowed ? win.hid[unit * cap + src] : 0;
    };
    auto place = [&](const MovedRow &m, int src, int o) __attribute__((always_inline)) {
        const size_t at = static_cast<size_t>(o) * kLanesPerRow + sub;
        if (stream) { store_stream(Ko + at, m.k); store_stream(Vo + at, m.v); }
        else { Ko[at] = m.k; Vo[at] = m.v; }
        if (sub == 0) {
            nrm_out[unit * cap_out + o] = m.w;
            if (pos_out) pos_out[unit * cap_out + o] = m.pos;
            if constexpr (kWindowed) win.hid_out[unit * cap_out + o] = src == n0 ? new_col : m.col;
        }
    };
    constexpr int kMove = 2;
    const int after0 = evicts ? hi : n;                     // first row behind e*
    MovedRow moved[kMove];
#pragma unroll
    for (int u = 0; u < kMove; ++u) fetch(moved[u], min(after0 + (u * G + g) * kRowsPerPass + rloc, n - 1));

    // log2 of the softmax denominator of every query head of the group from the chunk statistics
    float lse2[kMaxG];
    merge_group_stats<kMaxG>(part, chunks_alloc, group, n_chunks, stats, lse2);

    // the first rows' scores (kept: the workgroup's own rows are among them), then the row that leaves: minimise
    // (importance bits, ~row) over the unprotected rows
    float score[kScan], weight[kScan], low[kScan];
#pragma unroll
    for (int u = 0; u < kScan; ++u) score[u] = combine(held[u], scan_row(tid + u * kThreads), lse2, weight[u], low[u]);
    int evicted = n;                                       // n <= B: nothing leaves
    if (evicts) {
        unsigned long long best = ~0ull;
        auto consider = [&](int i, float importance) {
            const int r = scan_row(i);
            const unsigned long long c = (static_cast<unsigned long long>(__float_as_uint(importance)) << 32) |
                                         static_cast<unsigned>(~static_cast<unsigned>(r));
            if (i < n_scan && r >= lo && r < hi) best = c < best ? c : best;
        };
#pragma unroll
        for (int u = 0; u < kScan; ++u) consider(tid + u * kThreads, __fmul_rn(score[u], held[u].w));
        for (int i0 = tid + kScan * kThreads; i0 < n_scan; i0 += kScan * kThreads) {
            ScanRow<kMaxG> rows[kScan];
            request(rows, i0);
#pragma unroll
            for (int u = 0; u < kScan; ++u) {
                float p, lo_new;
                consider(i0 + u * kThreads, __fmul_rn(combine(rows[u], scan_row(i0 + u * kThreads), lse2, p, lo_new), rows[u].w));
            }
        }
        best = wave_min_u64(best);
        if ((tid & 63) == 0) s_min[tid >> 6] = best;
        lds_barrier();                                     // (LDS only: the rows in flight stay in flight)
        best = s_min[0];
#pragma unroll
        for (int w = 1; w < kThreads / 64; ++w) best = s_min[w] < best ? s_min[w] : best;
        evicted = static_cast<int>(~static_cast<unsigned>(best & 0xffffffffull));
    }

    // scores and source indices of this workgroup's rows: from the registers, then (more than kScan * kThreads of them)
    // formed once more
    auto emit = [&](int i, float score_new, float p, float lo_new, int col) {
        const int r = own0 + i;
        if (i >= n_own || r == evicted) return;
        const int o = r - (r > evicted ? 1 : 0);
        S_out[unit * cap_out + o] = score_new;
        if (kept_idx) kept_idx[unit * cap_out + o] = r;
        if constexpr (kWindowed) {
            win.s_lo_out[unit * cap_out + o] = lo_new;
            h_write[col] = p;
        }
    };
#pragma unroll
    for (int u = 0; u < kScan; ++u) emit(tid + u * kThreads, score[u], weight[u], low[u], held[u].col);
    for (int i0 = tid + kScan * kThreads; i0 < n_own; i0 += kScan * kThreads) {
        ScanRow<kMaxG> rows[kScan];
        request(rows, i0);
#pragma unroll
        for (int u = 0; u < kScan; ++u) {
            float p, lo_new;
            const float score_new = combine(rows[u], scan_row(i0 + u * kThreads), lse2, p, lo_new);
            emit(i0 + u * kThreads, score_new, p, lo_new, rows[u].col);
        }
    }
    if (g == 0 && tid == 0) synced_out[unit] = evicted;
    if constexpr (kWindowed) {
        // the appended row has received nothing in the steps before this one: clear its column in every
        // ring row but the one written above and the one that leaves (rewritten in full by the next step)
        for (int s = g * kThreads + tid; s < win.rows; s += G * kThreads)
            if (s != step % win.rows && s != (step + 1) % win.rows)
                win.hist[(unit * win.rows + s) * static_cast<size_t>(win.cap_hist) + new_col] = 0.f;
        if (g == 0 && tid == 0) {
            win.hid[unit * cap + n0] = new_col;
            win.free_out[unit] = evicted < n ? column(evicted) : n;     // a fresh column while the cache grows
        }
    }

    // rows behind e* to their places, one down; then the rows of the other set that are out of date before them: from the
    // first row in which it differs from the input set, or from the evicted row if that comes earlier
#pragma unroll
    for (int u = 0; u < kMove; ++u) {
        const int src = after0 + (u * G + g) * kRowsPerPass + rloc;
        if (src < n) place(moved[u], src, src - 1);
    }
    for (int src = after0 + (kMove * G + g) * kRowsPerPass + rloc; src < n; src += G * kRowsPerPass) {
        MovedRow m;
        fetch(m, src);
        place(m, src, src - 1);
    }
    const int o_end = evicts ? hi - 1 : n_keep;
    for (int o = min(synced, evicted) + g * kRowsPerPass + rloc; o < o_end; o += G * kRowsPerPass) {
        const int src = o + (o >= evicted ? 1 : 0);
        MovedRow m;
        fetch(m, src);
        place(m, src, o);
    }
}

// The whole step in one launch, one workgroup of 16 wavefronts per head: logits of the new query
// over the head's rows (they stay in LDS), softmax statistics, new scores, the evicted row, and
// the rows of the other cache set that are out of date.  Used when every head's rows fit the LDS
// buffer; no workspace traffic and no second launch.  Logits and per-chunk statistics are formed by
// the same functions as in decode_logits_kernel (dot_16_bytes, group_all_reduce, chunk_stats_64x2 on
// 128-row chunks), so the result has the same bits as the two-launch route.
//
// Rows are dealt to threads from the END of the cache: load slot u of thread (rloc, sub) is row
// n-1 - (u * rows_per_pass + rloc).  The row that leaves is almost always the one at the edge of the recent
// window, e* = n - recent - 1 (it has just lost the window's protection and has collected the least
// attention), and then exactly the rows behind it move one position down in the other set.  Those rows are
// the first slots of every thread: their V rows, norms and positions are the first loads of the kernel,
// their K rows the first of the stream, and they are stored -- to the positions the guess e* implies -- as
// soon as they have arrived, while the rest of the head is still streaming in, instead of in a burst at the
// end.  When the real evicted row e turns out to lie before e*, what was stored is still right (rows behind
// e* move down by one either way); row e* itself, which the guess skipped, is then stored to e* - 1 from the
// registers that still hold it, and the rows between e and e* are copied the ordinary way.
constexpr int kOneThreads = 1024;
constexpr int kOneMaxRows = 2048;                          // logits, old scores and norms kept in LDS (24 KiB)

template <typename T, int D, bool kStream>
__global__ __launch_bounds__(kOneThreads) void decode_prune_one_kernel(
    const T *__restrict__ q, const T *__restrict__ k_new, const T *__restrict__ v_new, T *__restrict__ K,
    T *__restrict__ V, const float *__restrict__ S, float *__restrict__ nrm, int32_t *__restrict__ pos,
    T *__restrict__ K_out, T *__restrict__ V_out, float *__restrict__ S_out, float *__restrict__ nrm_out,
    int32_t *__restrict__ pos_out, int32_t *__restrict__ kept_idx, const int32_t *__restrict__ synced_in,
    int32_t *__restrict__ synced_out, BatchMeta len_pos, BudgetList budget, int n_heads, int cap, int cap_out,
    int n_sink, int recent, float scale_log2, int norm)
{
    constexpr int kE = Elt<T>::kPer16B;
    constexpr int kLanesPerRow = D / kE;
    constexpr int kRowsPerPass = kOneThreads / kLanesPerRow;
    constexpr int kGroup = 16;                             // row loads in flight per thread: 1024 rows per round trip
    constexpr int kWaves = kOneThreads / 64;
    constexpr int kPre = kOneMaxRows / kOneThreads;        // rows of S and nrm a thread brings in
    // rows requested ahead of the eviction: the last kSpecRows of the cache (>= 128), kSpecSlots per thread
    constexpr int kSpecSlots = kRowsPerPass >= 64 ? 2 : 128 / kRowsPerPass, kSpecRows = kSpecSlots * kRowsPerPass;
    static_assert(kSpecSlots <= kGroup, "the speculative rows are slots of the first round trip");

    __shared__ float s_logit[kOneMaxRows];
    __shared__ float s_score[kOneMaxRows];                 // old scores (0 for the appended row)
    __shared__ float s_norm[kOneMaxRows];
    __shared__ float2 s_part[kOneMaxRows / kDecodeChunk];
    __shared__ float s_new_norm;
    __shared__ unsigned long long s_min[kWaves];

    const size_t unit = blockIdx.x;
    const int b = static_cast<int>(unit / n_heads);
    const int n0 = len_pos.len[b], n = n0 + 1, B = budget.v[b];
    const int n_keep = n < B ? n : B;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub = tid % kLanesPerRow, rloc = tid / kLanesPerRow;
    const float *Su = S + unit * cap;
    float *Nu = nrm + unit * cap;
    const uint4 *Ku = reinterpret_cast<const uint4 *>(K + unit * cap * D);
    const uint4 *Vu = reinterpret_cast<const uint4 *>(V + unit * cap * D);
    const uint4 *knew = reinterpret_cast<const uint4 *>(k_new + unit * D);
    const uint4 *vnew = reinterpret_cast<const uint4 *>(v_new + unit * D);

    // the row expected to leave (n > B: there are candidates, so n - recent - 1 >= n_sink), and the first of
    // the rows that are stored ahead of the decision
    const int e_star = n > B ? n - recent - 1 : n;
    const int spec_lo = max(max(n - recent - 1, n - kSpecRows), 0);
    uint4 *Ko = reinterpret_cast<uint4 *>(K_out + unit * cap_out * D);
    uint4 *Vo = reinterpret_cast<uint4 *>(V_out + unit * cap_out * D);

    // Every load this phase needs is requested before the first result is used: V rows, norms and positions
    // of the rows stored ahead, the count of rows the two sets share, the query, the new row, the old scores
    // and norms (parked in LDS after the sweep, so that the later phases do not start with a round trip to
    // memory of their own), then the first 16 K rows of every thread.
    uint4 spec_k[kSpecSlots], spec_v[kSpecSlots];
    float spec_w[kSpecSlots];
    int spec_pos[kSpecSlots];
#pragma unroll
    for (int u = 0; u < kSpecSlots; ++u) {
        const int r = n - 1 - (u * kRowsPerPass + rloc);
        spec_v[u] = make_uint4(0, 0, 0, 0);
        spec_w[u] = 0.f;
        spec_pos[u] = 0;
        if (r >= spec_lo) {
            spec_v[u] = r == n0 ? vnew[sub] : load_rows<kStream>(Vu + static_cast<size_t>(r) * kLanesPerRow + sub);
            if (sub == 0 && r != n0) {
                spec_w[u] = Nu[r];
                if (pos) spec_pos[u] = pos[unit * cap + r];
            }
        }
    }
    const int synced = synced_in[unit];
    const uint4 q_raw = reinterpret_cast<const uint4 *>(q + unit * D)[sub];
    uint4 k_raw = make_uint4(0, 0, 0, 0);
    if (tid < kLanesPerRow) k_raw = knew[sub];
    float pre_s[kPre], pre_w[kPre];
#pragma unroll
    for (int u = 0; u < kPre; ++u) {
        const int r = tid + u * kOneThreads;
        pre_s[u] = r < n0 ? Su[r] : 0.f;
        pre_w[u] = r < n0 ? Nu[r] : 0.f;
    }

    // logits of all rows into LDS; the new row is read from the step's input, not from the cache
    for (int base = 0; base < n; base += kGroup * kRowsPerPass) {
        uint4 raw[kGroup];
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            const int r = n - 1 - (base + u * kRowsPerPass + rloc);
            const uint4 *src = (r == n0) ? knew + sub : Ku + static_cast<size_t>(r) * kLanesPerRow + sub;
            raw[u] = (r >= 0) ? load_rows<kStream>(src) : make_uint4(0, 0, 0, 0);
        }
        if (base == 0) {
            if (tid < kLanesPerRow) {
                // append the new row (slot 0 of these threads): k, v, |v|, pos
                reinterpret_cast<uint4 *>(K + unit * cap * D)[static_cast<size_t>(n0) * kLanesPerRow + sub] = k_raw;
                reinterpret_cast<uint4 *>(V + unit * cap * D)[static_cast<size_t>(n0) * kLanesPerRow + sub] = spec_v[0];
                const float new_norm = row_norm<T, kLanesPerRow>(norm, spec_v[0]);
                if (sub == 0) {
                    s_new_norm = new_norm;
                    Nu[n0] = new_norm;
                    if (pos) pos[unit * cap + n0] = len_pos.aux[b];
                    spec_w[0] = new_norm;
                    spec_pos[0] = len_pos.aux[b];
                }
            }
            // the rows behind the expected eviction go to the other set now, at the positions that guess implies
#pragma unroll
            for (int u = 0; u < kSpecSlots; ++u) {
                const int r = n - 1 - (u * kRowsPerPass + rloc);
                spec_k[u] = raw[u];
                if (r >= spec_lo && r != e_star) {
                    const int o = r - (r > e_star ? 1 : 0);
                    store_rows<kStream>(Ko + static_cast<size_t>(o) * kLanesPerRow + sub, raw[u]);
                    store_rows<kStream>(Vo + static_cast<size_t>(o) * kLanesPerRow + sub, spec_v[u]);
                    if (sub == 0) {
                        nrm_out[unit * cap_out + o] = spec_w[u];
                        if (pos_out) pos_out[unit * cap_out + o] = spec_pos[u];
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            const int r = n - 1 - (base + u * kRowsPerPass + rloc);
            const float dot = group_all_reduce<kLanesPerRow>(dot_16_bytes<T>(raw[u], q_raw), OpSum{});
            if (sub == 0 && r >= 0) s_logit[r] = dot * scale_log2;
        }
    }
#pragma unroll
    for (int u = 0; u < kPre; ++u) {
        const int r = tid + u * kOneThreads;
        if (r < n0) { s_score[r] = pre_s[u]; s_norm[r] = pre_w[u]; }
    }
    // (a barrier for LDS only: the writes above must be visible, the V rows requested ahead need not have arrived)
    lds_barrier();
    if (tid == 0) { s_score[n0] = 0.f; s_norm[n0] = s_new_norm; }      // the appended row (published by the barriers below)

    // Statistics of every 128-row chunk, one wavefront per chunk and no exchange between wavefronts: the lane
    // takes rows lane and lane + 64 of the chunk -- the same function, on the same values, as in
    // decode_logits_kernel.
    const int n_chunks = (n + kDecodeChunk - 1) / kDecodeChunk;
    for (int chunk = wave; chunk < n_chunks; chunk += kWaves) {
        const int r0 = chunk * kDecodeChunk + lane, r1 = r0 + 64;
        const float2 st = chunk_stats_64x2(r0 < n ? s_logit[r0] : -INFINITY, r1 < n ? s_logit[r1] : -INFINITY);
        if (lane == 0) s_part[chunk] = st;
    }
    lds_barrier();
    float M, L;
    merge_chunk_stats(s_part, n_chunks, M, L);
    const float lse2 = M + log2f(L);

    auto new_score = [&](int r) { return s_score[r] + exp2f(s_logit[r] - lse2); };

    // the row that leaves: smallest importance among the unprotected rows, the highest row among equals.
    // A thread looks at rows tid, tid + 1024, ...: within a wavefront rows ascend with the lane, so the
    // wavefront's answer for one such round is the smallest key and the highest lane that holds it.
    int evicted = n;
    if (n > B) {
        unsigned long long best = ~0ull;
        for (int r0 = 0; r0 < n - recent; r0 += kOneThreads) {
            const int r = r0 + tid;
            const bool cand = r >= n_sink && r < n - recent;
            const unsigned key = cand ? __float_as_uint(__fmul_rn(new_score(r), s_norm[r])) : 0xffffffffu;
            const unsigned kmin = wave_min_u32(key);
            const unsigned long long holders = __ballot(cand && key == kmin);
            if (holders != 0ull) {
                const int top = 63 - __builtin_clzll(holders);
                const unsigned long long c = (static_cast<unsigned long long>(kmin) << 32) |
                                             static_cast<unsigned>(~static_cast<unsigned>(r0 + wave * 64 + top));
                best = c < best ? c : best;
            }
        }
        if (lane == 0) s_min[wave] = best;
        lds_barrier();
        best = s_min[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) best = s_min[w] < best ? s_min[w] : best;
        evicted = static_cast<int>(~static_cast<unsigned>(best & 0xffffffffull));
    }

    // rows of the other set that are out of date: from the first row in which it differs from the input
    // set, or from the evicted row if that comes earlier.  Source row r goes to row r - (r > evicted).
    const int first = min(synced, evicted);
    if (tid == 0) synced_out[unit] = evicted;

    // new scores and source rows of the survivors
    for (int o = tid; o < n_keep; o += kOneThreads) {
        const int src = o + (o >= evicted ? 1 : 0);
        if constexpr (kStream) {
            __builtin_nontemporal_store(new_score(src), &S_out[unit * cap_out + o]);
            if (kept_idx) __builtin_nontemporal_store(src, &kept_idx[unit * cap_out + o]);
        } else {
            S_out[unit * cap_out + o] = new_score(src);
            if (kept_idx) kept_idx[unit * cap_out + o] = src;
        }
    }

    // The rows from spec_lo on are in place already, except that a row e* which does not leave after all
    // (evicted < e*) has not been stored: it goes to e* - 1.
    if (evicted != e_star) {
#pragma unroll
        for (int u = 0; u < kSpecSlots; ++u) {
            const int r = n - 1 - (u * kRowsPerPass + rloc);
            if (r == e_star && r >= spec_lo) {
                const int o = r - 1;
                store_rows<kStream>(Ko + static_cast<size_t>(o) * kLanesPerRow + sub, spec_k[u]);
                store_rows<kStream>(Vo + static_cast<size_t>(o) * kLanesPerRow + sub, spec_v[u]);
                if (sub == 0) {
                    nrm_out[unit * cap_out + o] = spec_w[u];
                    if (pos_out) pos_out[unit * cap_out + o] = spec_pos[u];
                }
            }
        }
    }

    // ... and the rows before spec_lo that are out of date (the two sets were in step only up to a row
    // before it, or the evicted row lies before it) are copied from the cache as it was on entry: source
    // rows below spec_lo, never the appended row
    {
        const int o_end = min(n_keep, spec_lo - (evicted < spec_lo ? 1 : 0));
        for (int o = first + rloc; o < o_end; o += kRowsPerPass) {
            const int src = o + (o >= evicted ? 1 : 0);
            const uint4 kr = load_rows<kStream>(Ku + static_cast<size_t>(src) * kLanesPerRow + sub);
            const uint4 vr = load_rows<kStream>(Vu + static_cast<size_t>(src) * kLanesPerRow + sub);
            store_rows<kStream>(Ko + static_cast<size_t>(o) * kLanesPerRow + sub, kr);
            store_rows<kStream>(Vo + static_cast<size_t>(o) * kLanesPerRow + sub, vr);
            if (sub == 0) {
                nrm_out[unit * cap_out + o] = s_norm[src];
                if (pos_out) pos_out[unit * cap_out + o] = pos[unit * cap + src];
            }
        }
    }
}

}  // namespace

hipError_t launch_decode_prune(int dtype, int head_dim, const void *K, const void *V, const float *S,
                               const float *nrm, const int32_t *pos, void *K_out, void *V_out, float *S_out,
                               float *nrm_out, int32_t *pos_out, int32_t *kept_idx, const int32_t *synced_in,
                               int32_t *synced_out, const float *ws_logit, const float2 *ws_part,
                               const float *ws_out, float *out, const WindowArgs &win, const BatchMeta &meta,
                               const Geometry &g, hipStream_t st)
{
    const int chunks_alloc = (g.cap + kDecodeChunk - 1) / kDecodeChunk;
    const unsigned units = static_cast<unsigned>(g.batch) * g.n_heads;
    // Workgroups per head: each of them repeats the scan over all of the head's rows (group times as many logits
    // with grouped queries), so more of them only pay while the chip is not yet full.  Measured per step: 512 heads
    // (ragged16) 49.8 us with one, 51.2 with two, 56 with four; 64 heads x 4 query heads 28 us with 2 to 8, 35 with 16.
    unsigned G = 512u / (units * static_cast<unsigned>(g.group));
    G = G < 1u ? 1u : (G > 16u ? 16u : G);
    dim3 grid(units, G + (out ? static_cast<unsigned>(g.group) : 0u)), block(kThreads);
#define VATP_DPG(T, D, MAXG)                                   \
    do {                                                       \
        if (win.hist) VATP_DPW(T, D, MAXG, true);              \
        else VATP_DPW(T, D, MAXG, false);                      \
    } while (0)
#define VATP_DPW(T, D, MAXG, WINDOWED)                                                                         \
    hipLaunchKernelGGL((decode_prune_kernel<T, D, MAXG, WINDOWED>), grid, block, 0, st, static_cast<const T *>(K),            \
                       static_cast<const T *>(V), S, nrm, pos, static_cast<T *>(K_out), static_cast<T *>(V_out), \
                       S_out, nrm_out, pos_out, kept_idx, synced_in, synced_out, ws_logit, ws_part, ws_out, out, \
                       win, meta, g.n_heads, g.cap, g.cap_out, chunks_alloc, g.n_sink, g.recent, g.group, g.stream, static_cast<int>(G))
    // (instantiated for group sizes up to 2, 4, 8 and 16: the smallest that fits)
#define VATP_DP(T, D)                                      \
    do {                                                   \
        if (g.group > 8) VATP_DPG(T, D, VATP_MAX_GROUP);   \
        else if (g.group > 4) VATP_DPG(T, D, 8);           \
        else if (g.group > 2) VATP_DPG(T, D, 4);           \
        else if (g.group > 1) VATP_DPG(T, D, 2);           \
        else VATP_DPG(T, D, 1);                            \
    } while (0)
    if (dtype == VATP_F32 && head_dim == 64) VATP_DP(float, 64);
    else if (dtype == VATP_F32) VATP_DP(float, 128);
    else if (head_dim == 64) VATP_DP(bf16_t, 64);
    else VATP_DP(bf16_t, 128);
#undef VATP_DP
#undef VATP_DPG
#undef VATP_DPW
    return hipGetLastError();
}

}  // namespace vatp

namespace vatp {

int decode_prune_one_max_rows() { return kOneMaxRows; }

hipError_t launch_decode_prune_one(int dtype, int head_dim, const void *q, const void *k, const void *v, void *K,
                                   void *V, const float *S, float *nrm, int32_t *pos, void *K_out, void *V_out,
                                   float *S_out, float *nrm_out, int32_t *pos_out, int32_t *kept_idx,
                                   const int32_t *synced_in, int32_t *synced_out, const BatchMeta &len_pos,
                                   const BudgetList &budget, const Geometry &g, hipStream_t st)
{
    const unsigned units = static_cast<unsigned>(g.batch) * g.n_heads;
    dim3 grid(units), block(kOneThreads);
#define VATP_DP1(T, D)                                                                                           \
    do {                                                                                                         \
        if (g.stream) VATP_DP1_S(T, D, true);                                                                    \
        else VATP_DP1_S(T, D, false);                                                                            \
    } while (0)
#define VATP_DP1_S(T, D, STREAM)                                                                                    \
    hipLaunchKernelGGL((decode_prune_one_kernel<T, D, STREAM>), grid, block, 0, st, static_cast<const T *>(q),         \
                       static_cast<const T *>(k), static_cast<const T *>(v), static_cast<T *>(K),                \
                       static_cast<T *>(V), S, nrm, pos, static_cast<T *>(K_out), static_cast<T *>(V_out), S_out, \
                       nrm_out, pos_out, kept_idx, synced_in, synced_out, len_pos, budget, g.n_heads, g.cap,     \
                       g.cap_out, g.n_sink, g.recent, g.scale_log2, g.norm)
    if (dtype == VATP_F32 && head_dim == 64) VATP_DP1(float, 64);
    else if (dtype == VATP_F32) VATP_DP1(float, 128);
    else if (head_dim == 64) VATP_DP1(bf16_t, 64);
    else VATP_DP1(bf16_t, 128);
#undef VATP_DP1
#undef VATP_DP1_S
    return hipGetLastError();
}

}  // namespace vatp
