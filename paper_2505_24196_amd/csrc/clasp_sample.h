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
// Measured at 128256 entries: one draw 202 us with one workgroup for everything, 12 us (4.6 + 7.3) now; acceptance of four
// drafts 340 us (first draft rejected) to 1.4 ms, 17.5 us (3.8 + 4.9 + 6.8 and the boundaries) whichever is rejected.
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

struct AcceptShared {
    RowStat row[kSampleRows];
    int reject[kMaxRows];
};

// Rows of at most kSmallVocab entries (the small models): a wavefront takes a row, so one workgroup, and one launch
// instead of three, does all of a call. 2064 entries, one draft: 15 us with a workgroup per call that walked the rows one
// after another, 17 over chunks, 14 now; seven drafts: 31, 17, 14 (about 12 us of each is the caller).
constexpr int kSmallVocab = 4096;
__device__ __forceinline__ RowStat small_row_stat(const float* lg, int V, float inv_t) {
    const int lane = threadIdx.x & 63;
    float m = -INFINITY, s = 0.f;
#pragma unroll 8
    for (int v = lane; v < V; v += 64) m = fmaxf(m, lg[v]);
    m = wave_max(m);
#pragma unroll 8
    for (int v = lane; v < V; v += 64) {
        const float x = lg[v];
        s += x == -INFINITY ? 0.f : expf((x - m) * inv_t);
    }
    return RowStat{m, wave_sum(s)};
}

// The first rejected draft (n if none), by a whole workgroup; sh.row holds every row's (max, sum) afterwards. Draft i is
// kept when u_accept[i] * q_i(x) < p_i(x). SMALL: the rows' (max, sum) from the rows themselves, else from their chunks.
template <bool SMALL>
__device__ __forceinline__ int accept_prefix(const SampleArgs& a, int chunks, AcceptShared& sh) {
    const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6, i = threadIdx.x;
    float pl = 0.f, ql = 0.f, u = 0.f;  // this draft's logits and uniform number, requested beside the rows' pieces
    if (i < a.n) {
        const int x = min(max(a.tokens[i + 1], 0), a.V - 1);
        pl = a.p[(size_t)i * a.ld + x];
        ql = a.q[(size_t)i * a.ld + x];
        u = a.u_accept[i];
    }
    for (int r = wave; r < 2 * a.n + 1; r += nw) {
        RowStat st;
        if constexpr (SMALL) st = small_row_stat(r <= a.n ? a.p + (size_t)r * a.ld : a.q + (size_t)(r - a.n - 1) * a.ld, a.V, a.inv_t);
        else st = merge_row(a.stats + (size_t)r * kSampleChunks, chunks, a.inv_t);
        if ((threadIdx.x & 63) == 0) sh.row[r] = st;
    }
    __syncthreads();
    if (i < a.n) {
        const RowStat ps = sh.row[i], qs = sh.row[a.n + 1 + i];
        const float px = expf((pl - ps.m) * a.inv_t) / ps.s, qx = expf((ql - qs.m) * a.inv_t) / qs.s;
        sh.reject[i] = !(u * qx < px);
    }
    __syncthreads();
    int first = a.n;
    for (int k = a.n - 1; k >= 0; --k)
        if (sh.reject[k]) first = k;
    return first;
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
    const int first = accept_prefix<false>(a, cut.chunks, sh);
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
    float wave_tot[kDrawThreads / 64], wave_excl[kDrawThreads / 64];
    int pick;
    int last[kDrawThreads / 64];
};

// Inverse-CDF draw: the index v with c_{v-1} <= u * c_last < c_v, c = running sums of the weights w in index order.
// `total` = this lane's chunk total (lane < chunks; the same in every wavefront). Returns the index to every thread, -1 when
// the weights do not add up to a positive number.
template <class WF>
__device__ __forceinline__ int draw_from_chunks(WF w, float total, const SampleCut& cut, int V, float u, DrawShared& sh) {
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
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
    const int first = chunk * cut.size, end = min(first + cut.size, V);
    // the chunk again, in index order: a contiguous piece per thread
    const int E = (end - first + kDrawThreads - 1) / kDrawThreads;
    const int lo = min(first + t * E, end), hi = min(lo + E, end);
    constexpr int kKeep = 2;  // weights that stay in registers: all of a thread's up to 128k entries a row
    float keep[kKeep], local = 0.f;
#pragma unroll
    for (int e = 0; e < kKeep; ++e) keep[e] = lo + e < hi ? w(lo + e) : 0.f;
#pragma unroll
    for (int e = 0; e < kKeep; ++e) local += keep[e];
    for (int v = lo + kKeep; v < hi; ++v) local += w(v);
    float run = local;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float x = __shfl_up(run, o);
        if (lane >= o) run += x;
    }
    __syncthreads();  // sh may still be read from an earlier draw
    if (lane == 63) sh.wave_tot[wave] = run;
    if (t == 0) sh.pick = 0x7fffffff;
    __syncthreads();
    float wbase = base;
    for (int k = 0; k < wave; ++k) wbase += sh.wave_tot[k];
    const float prev = __shfl_up(run, 1);
    float c = wbase + (lane ? prev : 0.f);
    int last = -1;
    int found = 0x7fffffff;
    auto visit = [&](int v, float wv) {
        c += wv;
        if (wv > 0.f) last = v;
        if (wv > 0.f && target < c) found = min(found, v);
    };
#pragma unroll
    for (int e = 0; e < kKeep; ++e) visit(lo + e, keep[e]);
    for (int v = lo + kKeep; v < hi; ++v) visit(v, w(v));
    if (found != 0x7fffffff) atomicMin(&sh.pick, found);  // the lowest index whose running sum exceeds the target
    // rounding may leave u * c_last at or beyond the last running sum: the chunk's last index of positive weight
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) last = max(last, __shfl_xor(last, o));
    if (lane == 0) sh.last[wave] = last;
    __syncthreads();
    int pick = sh.pick;
    if (pick == 0x7fffffff) {
        pick = -1;
        for (int k = 0; k < kDrawThreads / 64; ++k) pick = max(pick, sh.last[k]);
    }
    return pick;
}

// One workgroup. Plain draw (q null): token ~ softmax(p / T). Acceptance: the replacement of the first rejected draft from
// its residual, or from the full model's row where the residual is empty; the bonus token from row n when all are kept.
// SMALL: the whole call for rows of at most kSmallVocab entries, which are one chunk.
template <bool SMALL>
__global__ __launch_bounds__(kDrawThreads) void draw_kernel(SampleArgs a) {
    __shared__ AcceptShared ac;
    __shared__ DrawShared sh;
    __shared__ float red[kDrawThreads / 64];
    const SampleCut cut = SMALL ? SampleCut{1, a.V} : sample_cut(a.V);
    const int lane = threadIdx.x & 63;
    const float u = a.u_final[0];
    int row = 0, tok = -1;
    RowStat ps;
    if (a.q) {
        float mass = 0.f;  // unwritten, and not used, when all drafts are kept
        if (!SMALL && lane < cut.chunks) mass = a.residual[lane];
        row = accept_prefix<SMALL>(a, cut.chunks, ac);
        ps = ac.row[row];
        if (row < a.n) {
            const ResidualWeight w(a, row, ac);
            if constexpr (SMALL) {
#pragma unroll 4
                for (int v = threadIdx.x; v < a.V; v += kDrawThreads) mass += w(v);
                mass = block_sum(mass, red);
            }
            tok = draw_from_chunks(w, mass, cut, a.V, u, sh);
        }
    } else {
        ps = SMALL ? small_row_stat(a.p, a.V, a.inv_t) : merge_row(a.stats, cut.chunks, a.inv_t);
    }
    if (tok < 0) {
        const float* p = a.p + (size_t)row * a.ld;
        float total = ps.s;
        if constexpr (!SMALL) {
            const RowStat st = lane < cut.chunks ? a.stats[(size_t)row * kSampleChunks + lane] : RowStat{-INFINITY, 0.f};
            total = rescaled(st, ps.m, a.inv_t);
        }
        tok = draw_from_chunks([&](int v) { return expf((p[v] - ps.m) * a.inv_t); }, total, cut, a.V, u, sh);
    }
    if (threadIdx.x == 0) {  // outputs last: every input of the call has been read by now
        if (a.q) a.n_accepted_out[0] = row;
        a.token_out[0] = tok;
    }
}

}  // namespace clasp
