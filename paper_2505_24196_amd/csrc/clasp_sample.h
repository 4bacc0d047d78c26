// Stochastic decoding (the paper's Temperature = 1 setting, Sec. 4; "still speculative sampling", Sec. 4.1): draws from
// softmax(logits / T) by inverting the cumulative distribution with a uniform number the caller supplies, and the
// speculative-sampling acceptance rule over one round of drafts.
// A row of 128k logits is half a megabyte: one workgroup pulls that at ~50 GB/s and needs it three times (maximum, sum,
// draw), 10 us each. So the rows are cut into chunks, a workgroup each:
//   chunk_stats_kernel     largest logit and sum of exp relative to it, per (row, chunk): the only pass over all rows
//   residual_sums_kernel   (acceptance) every workgroup merges the rows' pieces, finds the first rejected draft for
//                          itself (a few hundred words), and sums max(0, p - q) of its chunk of that row
//   draw_kernel            one workgroup: running sums over the chunks' totals name the chunk that the draw falls into,
//                          and only that chunk is read again
// Measured at 128256 entries, GPU time of a call on logits that were just read: one draw 170 us with one workgroup for
// everything, 6.7 us now; acceptance of four drafts 340 us (first one rejected) to 1360 us (all kept), 11.8 to 10.1 us; on
// logits that have left the caches 480 to 1700 us and about 1 us more than the above. Rows of at most 4096 entries take
// one or two launches (draw_mode).
// Every sum runs in a fixed order, so the same inputs give the same token on every run.
#pragma once
#include "clasp_common.h"

namespace clasp {

constexpr int kSampleThreads = 256;      // chunk_stats_kernel
constexpr int kDrawThreads = 1024;       // the kernels that merge rows: a wavefront per row, sixteen rows at a time
constexpr int kSampleChunks = 64;        // most chunks of a row: one lane each where they are merged
constexpr int kSampleChunkMin = 1024;    // entries below which a row is not cut further
constexpr int kSampleRows = 2 * kMaxRows - 1;  // p rows 0..n and q rows 0..n-1, n <= kMaxRows - 1

struct RowStat {
    float m, s;  // max logit, sum over v of exp((logit_v - m) * inv_t)
};

// Chunks of a row of V entries and entries per chunk (the last chunk may be shorter, none is empty).
struct SampleCut {
    int chunks, size;
};
__host__ __device__ inline SampleCut sample_cut(int V) {
    int size = (V + kSampleChunks - 1) / kSampleChunks;
    size = size < kSampleChunkMin ? kSampleChunkMin : size;
    return SampleCut{(V + size - 1) / size, size};
}
// Scratch: RowStat [kSampleRows][kSampleChunks], then the residual sums [kSampleChunks].
constexpr size_t kSampleScratchBytes = (size_t)kSampleRows * kSampleChunks * sizeof(RowStat) + kSampleChunks * sizeof(float);

struct SampleArgs {
    const float* p;       // full model's rows (or the one row to draw from)
    const float* q;       // draft model's rows, null for a plain draw
    size_t ld;            // elements between rows
    int n, V;             // drafts (0 for a plain draw), entries per row
    float inv_t;
    const int32_t* tokens;
    const float *u_accept, *u_final;
    int32_t *n_accepted_out, *token_out;
    RowStat* stats;       // rows 0..n of p, then rows 0..n-1 of q
    float* residual;
};

// A chunk's sum relative to the row's maximum m. A chunk without a finite maximum holds entries of weight 0 (sum 0) or NaN.
__device__ __forceinline__ float rescaled(const RowStat& st, float m, float inv_t) {
    return st.m == -INFINITY ? st.s : st.s * expf((st.m - m) * inv_t);
}

// Merged (max, sum) of a row from its chunks' pieces, by one whole wavefront, the same in every lane.
__device__ __forceinline__ RowStat merge_row(const RowStat* pieces, int chunks, float inv_t) {
    const int lane = threadIdx.x & 63;
    const RowStat st = lane < chunks ? pieces[lane] : RowStat{-INFINITY, 0.f};
    const float m = wave_max(st.m);
    return RowStat{m, wave_sum(rescaled(st, m, inv_t))};
}

// Grid (chunks, rows of p then rows of q).
__global__ __launch_bounds__(kSampleThreads) void chunk_stats_kernel(SampleArgs a) {
    __shared__ float red[kSampleThreads / 64], red2[kSampleThreads / 64];
    const SampleCut cut = sample_cut(a.V);
    const int row = blockIdx.y, lo = blockIdx.x * cut.size, hi = min(lo + cut.size, a.V);
    const float* lg = row <= a.n ? a.p + (size_t)row * a.ld : a.q + (size_t)(row - a.n - 1) * a.ld;
    // the first kKeep entries of a thread stay in registers (all of them up to 128k entries a row)
    constexpr int kKeep = 8;
    float keep[kKeep];
    float m = -INFINITY;
#pragma unroll
    for (int u = 0; u < kKeep; ++u) {
        const int v = lo + threadIdx.x + u * kSampleThreads;
        keep[u] = v < hi ? lg[v] : -INFINITY;
    }
#pragma unroll
    for (int u = 0; u < kKeep; ++u) m = fmaxf(m, keep[u]);
    for (int v = lo + threadIdx.x + kKeep * kSampleThreads; v < hi; v += kSampleThreads) m = fmaxf(m, lg[v]);
    m = wave_max(m);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) red[wave] = m;
    __syncthreads();
    m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    auto weight = [&](float x) { return x == -INFINITY ? 0.f : expf((x - m) * a.inv_t); };  // also where all are -inf
    float s = 0.f;
#pragma unroll
    for (int u = 0; u < kKeep; ++u) s += weight(keep[u]);
    for (int v = lo + threadIdx.x + kKeep * kSampleThreads; v < hi; v += kSampleThreads) s += weight(lg[v]);
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red2[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) a.stats[(size_t)row * kSampleChunks + blockIdx.x] = RowStat{m, (red2[0] + red2[1]) + (red2[2] + red2[3])};
}

// ---- rows short enough for one workgroup to hold ------------------------------------------------------------------------
// What a call over a small vocabulary costs is its launches and, in one workgroup, its exponentials (a CU gets through about
// 2.5 per cycle), so the acceptance of several drafts leaves the rows' statistics to chunk_stats_kernel as long rows do
// and only the draw stays in one workgroup: two launches instead of three. One launch is left where its exponentials
// are few: plain draws, and acceptances of few drafts over few entries.
// GPU time of a call in us, against one workgroup that walks the rows one after another / one that gives every row a
// wavefront: 2064 entries, a draw 7.1 / 10.6 -> 3.7, four drafts, first rejected 10.1 / 10.7 -> 7.1, all kept 24 / 10.0 -> 7.0;
// 4096 entries, a draw 8.6 / 15.9 -> 4.2, four drafts 13.4 / 16.8 -> 8.2 and 35 / 13.9 -> 7.6; 512 entries, a draw 6.1 / 6.6 ->
// 3.5, four drafts 8.8 / 6.6 -> 5.6 and 20 / 6.7 -> 5.8.
// 4096: with eight entries a thread instead of four every call here takes 1 us more, and 8192 entries take 7.5 us a draw
// and 13.7 us for four drafts against 6.3 and 10.4 in chunks. (Slower than row after row: rounds of some 31 drafts over
// 4112..6000 entries that reject the first, 12.6 -> 13.4 us; with all kept 173 -> 12.6.)
constexpr int kRegisterVocab = 4096;  // entries of a row whose weights one workgroup keeps in registers
constexpr int kOneLaunchVocab = 1024, kOneLaunchDrafts = 7;  // acceptance in one launch: a wavefront per row, sixteen entries a lane
constexpr int kDrawWaves = kDrawThreads / 64;
constexpr int kDrawChunks = 0, kDrawRow = 1, kDrawAll = 2;  // what draw_kernel does (see there)
static_assert(2 * kOneLaunchDrafts + 1 <= kDrawWaves, "a wavefront per row");

__host__ inline int draw_mode(int V, int n) {
    if (V > kRegisterVocab) return kDrawChunks;
    return n == 0 || (V <= kOneLaunchVocab && n <= kOneLaunchDrafts) ? kDrawAll : kDrawRow;
}

struct AcceptShared {
    RowStat row[kSampleRows];
    int first;
};

// Maximum and sum of one row of at most kOneLaunchVocab entries, by one wavefront.
__device__ __forceinline__ RowStat wave_row_stat(const float* lg, int V, float inv_t) {
    constexpr int kKeep = kOneLaunchVocab / 64;
    const int lane = threadIdx.x & 63;
    float x[kKeep], m = -INFINITY, s = 0.f;
#pragma unroll
    for (int u = 0; u < kKeep; ++u) x[u] = u * 64 + lane < V ? lg[u * 64 + lane] : -INFINITY;
#pragma unroll
    for (int u = 0; u < kKeep; ++u) m = fmaxf(m, x[u]);
    m = wave_max(m);
#pragma unroll
    for (int u = 0; u < kKeep; ++u)
        if (u * 64 < V) s += x[u] == -INFINITY ? 0.f : expf((x[u] - m) * inv_t);
    return RowStat{m, wave_sum(s)};
}

// The first rejected draft (n if none), by a whole workgroup; sh.row holds every row's (max, sum) afterwards. Draft i is
// kept when u_accept[i] * q_i(x) < p_i(x). MODE: the rows' (max, sum) from the rows themselves (kDrawAll) or their chunks.
template <int MODE>
__device__ __forceinline__ int accept_prefix(const SampleArgs& a, int chunks, AcceptShared& sh) {
    const int wave = threadIdx.x >> 6, i = threadIdx.x;
    float pl = 0.f, ql = 0.f, u = 0.f;  // this draft's logits and uniform number, requested beside the rows' pieces
    if (i < a.n) {
        const int x = min(max(a.tokens[i + 1], 0), a.V - 1);
        pl = a.p[(size_t)i * a.ld + x];
        ql = a.q[(size_t)i * a.ld + x];
        u = a.u_accept[i];
    }
    for (int r = wave; r < 2 * a.n + 1; r += kDrawWaves) {
        RowStat st;
        if constexpr (MODE == kDrawAll) st = wave_row_stat(r <= a.n ? a.p + (size_t)r * a.ld : a.q + (size_t)(r - a.n - 1) * a.ld, a.V, a.inv_t);
        else st = merge_row(a.stats + (size_t)r * kSampleChunks, chunks, a.inv_t);
        if ((threadIdx.x & 63) == 0) sh.row[r] = st;
    }
    __syncthreads();
    if (wave == 0) {  // a lane per draft
        bool rejected = false;
        if (i < a.n) {
            const RowStat ps = sh.row[i], qs = sh.row[a.n + 1 + i];
            const float px = expf((pl - ps.m) * a.inv_t) / ps.s, qx = expf((ql - qs.m) * a.inv_t) / qs.s;
            rejected = !(u * qx < px);
        }
        const unsigned long long any = __builtin_amdgcn_ballot_w64(rejected);
        if (i == 0) sh.first = any ? __builtin_ctzll(any) : a.n;
    }
    __syncthreads();
    return sh.first;
}

struct ResidualWeight {  // max(0, p - q) of the first rejected row
    const float *p, *q;
    RowStat ps, qs;
    float ip, iq, inv_t;
    __device__ ResidualWeight(const SampleArgs& a, int row, const AcceptShared& sh)
        : p(a.p + (size_t)row * a.ld), q(a.q + (size_t)row * a.ld), ps(sh.row[row]), qs(sh.row[a.n + 1 + row]),
          ip(1.0f / ps.s), iq(1.0f / qs.s), inv_t(a.inv_t) {}
    __device__ float operator()(int v) const {
#pragma clang fp contract(off)  // equal logits have to leave exactly nothing, not the rounding of one of the products
        const float pv = expf((p[v] - ps.m) * inv_t) * ip, qv = expf((q[v] - qs.m) * inv_t) * iq;
        return fmaxf(pv - qv, 0.f);
    }
};

// Grid (chunks). Leaves the chunk's residual mass at the first rejected draft.
__global__ __launch_bounds__(kDrawThreads) void residual_sums_kernel(SampleArgs a) {
    __shared__ AcceptShared sh;
    __shared__ float red[kDrawThreads / 64];
    const SampleCut cut = sample_cut(a.V);
    const int lo = blockIdx.x * cut.size, hi = min(lo + cut.size, a.V);
    const int first = accept_prefix<kDrawChunks>(a, cut.chunks, sh);
    if (first == a.n) return;
    const ResidualWeight w(a, first, sh);
    float s = 0.f;
#pragma unroll 2
    for (int v = lo + threadIdx.x; v < hi; v += kDrawThreads) s += w(v);
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.f;
        for (int k = 0; k < kDrawThreads / 64; ++k) t += red[k];
        a.residual[blockIdx.x] = t;
    }
}

struct DrawShared {
    float wave_max[kDrawWaves], wave_tot[kDrawWaves];
    int found[kDrawWaves], last[kDrawWaves];
};

// The entries [first, end) in index order, a contiguous piece lo .. hi-1 of at most `each` per thread.
struct DrawRange {
    int each, lo, hi;
    __device__ DrawRange(int first, int end) {
        each = (end - first + kDrawThreads - 1) / kDrawThreads;
        lo = min(first + (int)threadIdx.x * each, end);
        hi = min(lo + each, end);
    }
};

// The lowest index at which the running sums over a range, which start at `base`, exceed a target; the range's last index of
// positive weight where rounding leaves the target at or beyond the last sum. keep: the weights of the thread's first KEEP
// entries (0 beyond its piece), w(v): any weight. target_of(sum at the end): the target, negative for none (returns -1).
template <int KEEP, class WF, class TF>
__device__ __forceinline__ int draw_in_range(const DrawRange& own, const float (&keep)[KEEP], WF w, float base, TF target_of,
                                             DrawShared& sh) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    float local = 0.f;
#pragma unroll
    for (int e = 0; e < KEEP; ++e) local += keep[e];
    for (int v = own.lo + KEEP; v < own.hi; ++v) local += w(v);
    float run = local;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float x = __shfl_up(run, o);
        if (lane >= o) run += x;
    }
    const float prev = __shfl_up(run, 1);
    __syncthreads();  // sh may still be read from an earlier draw
    if (lane == 63) sh.wave_tot[wave] = run;
    __syncthreads();
    float c = base, end_sum = base;
#pragma unroll
    for (int k = 0; k < kDrawWaves; ++k) {
        if (k == wave) c = end_sum;
        end_sum += sh.wave_tot[k];
    }
    const float target = target_of(end_sum);
    if (target < 0.f) return -1;  // the same in every thread
    if (lane) c += prev;
    int last = -1, found = -1;
    auto visit = [&](int v, float wv) {
        c += wv;
        if (wv > 0.f) last = v;
        if (wv > 0.f && target < c && found < 0) found = v;
    };
#pragma unroll
    for (int e = 0; e < KEEP; ++e) visit(own.lo + e, keep[e]);
    for (int v = own.lo + KEEP; v < own.hi; ++v) visit(v, w(v));
    // lanes and wavefronts are in index order: the first that found one, the last that has weight
    const unsigned long long hit = __builtin_amdgcn_ballot_w64(found >= 0), some = __builtin_amdgcn_ballot_w64(last >= 0);
    const int wave_found = hit ? __shfl(found, __builtin_ctzll(hit)) : -1, wave_last = some ? __shfl(last, 63 - __builtin_clzll(some)) : -1;
    if (lane == 0) {
        sh.found[wave] = wave_found;
        sh.last[wave] = wave_last;
    }
    __syncthreads();
    int pick = -1, fallback = -1;
#pragma unroll
    for (int k = kDrawWaves - 1; k >= 0; --k) {
        if (sh.found[k] >= 0) pick = sh.found[k];
        fallback = max(fallback, sh.last[k]);
    }
    return pick >= 0 ? pick : fallback;
}

// Inverse-CDF draw: the index v with c_{v-1} <= u * c_last < c_v, c = running sums of the weights w in index order.
// `total` = this lane's chunk total (lane < chunks; the same in every wavefront). Returns the index to every thread, -1 when
// the weights do not add up to a positive number. Only the chunk that holds the index is read again.
template <class WF>
__device__ __forceinline__ int draw_from_chunks(WF w, float total, const SampleCut& cut, int V, float u, DrawShared& sh) {
    const int lane = threadIdx.x & 63;
    const float mine = lane < cut.chunks ? total : 0.f;
    float incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float x = __shfl_up(incl, o);
        if (lane >= o) incl += x;
    }
    const float all = __shfl(incl, 63);
    if (!(all > 0.f)) return -1;
    const float target = u * all;
    // the last chunk that has weight and starts at or below the target
    const float before = __shfl_up(incl, 1), excl = lane ? before : 0.f;
    const unsigned long long starts = __builtin_amdgcn_ballot_w64(mine > 0.f && excl <= target);
    const int chunk = starts ? 63 - __builtin_clzll(starts) : __builtin_ctzll(__builtin_amdgcn_ballot_w64(mine > 0.f));
    const float base = __shfl(excl, chunk);
    const int first = chunk * cut.size;
    const DrawRange own(first, min(first + cut.size, V));
    constexpr int kKeep = 2;  // weights that stay in registers: all of a thread's up to 128k entries a row
    float keep[kKeep];
#pragma unroll
    for (int e = 0; e < kKeep; ++e) keep[e] = own.lo + e < own.hi ? w(own.lo + e) : 0.f;
    return draw_in_range(own, keep, w, base, [&](float) { return fmaxf(target, 0.f); }, sh);
}

// The same over a row of at most kRegisterVocab entries, all weights in registers (keep: the thread's, see draw_in_range).
constexpr int kRowKeep = kRegisterVocab / kDrawThreads;
__device__ __forceinline__ int draw_from_row(const DrawRange& own, const float (&keep)[kRowKeep], float u, DrawShared& sh) {
    return draw_in_range(own, keep, [](int) { return 0.f; }, 0.f, [&](float all) { return all > 0.f ? fmaxf(u * all, 0.f) : -1.f; }, sh);
}
template <class WF>
__device__ __forceinline__ void row_weights(const DrawRange& own, WF w, float (&keep)[kRowKeep]) {
#pragma unroll
    for (int e = 0; e < kRowKeep; ++e) {
        keep[e] = 0.f;
        if (e < own.each && own.lo + e < own.hi) keep[e] = w(own.lo + e);
    }
}

// One workgroup. Plain draw (q null): token ~ softmax(p / T). Acceptance: the replacement of the first rejected draft from
// its residual, or from the full model's row where the residual is empty; the bonus token from row n when all are kept.
// MODE kDrawChunks: behind chunk_stats_kernel and (acceptance) residual_sums_kernel; kDrawRow: acceptance over at most
// kRegisterVocab entries behind chunk_stats_kernel; kDrawAll: the whole call (draw_mode).
template <int MODE>
__global__ __launch_bounds__(kDrawThreads) void draw_kernel(SampleArgs a) {
    __shared__ AcceptShared ac;
    __shared__ DrawShared sh;
    const SampleCut cut = sample_cut(a.V);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const DrawRange own(0, a.V);
    const float u = a.u_final[0];
    int row = 0, tok = -1;
    RowStat ps{};
    if (a.q) {
        float mass = 0.f;  // unwritten, and not used, when all drafts are kept
        if (MODE == kDrawChunks && lane < cut.chunks) mass = a.residual[lane];
        row = accept_prefix<MODE>(a, cut.chunks, ac);
        ps = ac.row[row];
        if (row < a.n) {
            const ResidualWeight w(a, row, ac);
            if constexpr (MODE == kDrawChunks) {
                tok = draw_from_chunks(w, mass, cut, a.V, u, sh);
            } else {
                float keep[kRowKeep];
                row_weights(own, w, keep);
                tok = draw_from_row(own, keep, u, sh);
            }
        }
    } else if constexpr (MODE == kDrawChunks) {
        ps = merge_row(a.stats, cut.chunks, a.inv_t);
    }
    if (tok < 0) {
        const float* p = a.p + (size_t)row * a.ld;
        if constexpr (MODE == kDrawChunks) {
            const RowStat st = lane < cut.chunks ? a.stats[(size_t)row * kSampleChunks + lane] : RowStat{-INFINITY, 0.f};
            tok = draw_from_chunks([&](int v) { return expf((p[v] - ps.m) * a.inv_t); }, rescaled(st, ps.m, a.inv_t), cut, a.V, u, sh);
        } else {
            float keep[kRowKeep], m = ps.m;
            row_weights(own, [&](int v) { return p[v]; }, keep);
            if (!a.q) {  // the row's maximum is not known yet
                m = -INFINITY;
#pragma unroll
                for (int e = 0; e < kRowKeep; ++e)
                    if (own.lo + e < own.hi) m = fmaxf(m, keep[e]);
                m = wave_max(m);
                if (lane == 0) sh.wave_max[wave] = m;
                __syncthreads();
#pragma unroll
                for (int k = 0; k < kDrawWaves; ++k) m = fmaxf(m, sh.wave_max[k]);
            }
#pragma unroll
            for (int e = 0; e < kRowKeep; ++e)
                if (e < own.each && own.lo + e < own.hi) keep[e] = expf((keep[e] - m) * a.inv_t);
            tok = draw_from_row(own, keep, u, sh);
        }
    }
    if (threadIdx.x == 0) {  // outputs last: every input of the call has been read by now
        if (a.q) a.n_accepted_out[0] = row;
        a.token_out[0] = tok;
    }
}

}  // namespace clasp
