// Grouped-query attention of the candidate / verify / draft rows over the layer's shared KV cache.
//
// All rows of a launch read the cached prefix ONCE: the rows times the query heads of one KV group form the N
// dimension of S^T = K . Q^T, so a key fragment loaded from HBM serves every row (this is the paper's Sec. 3.6
// point: the DP's candidate states share one KV cache instead of duplicating it).
//   mode 0 (DP candidates): every row sits at position pos0 and sees cache positions 0..pos0-1 plus its own
//                           key/value, which live in a small per-launch self block; the cache is not touched.
//   mode 1 (verify / draft): row r sits at pos0 + r; its key/value is in the cache at that position already (the
//                           projection kernel wrote it) and it sees cache positions 0..pos0+r.
//
// bf16 kernel: flash-decoding on MFMA. Queries arrive rotated, scaled and in MFMA operand order from the q/k/v
// projection's epilogue. Keys are the M dimension of S^T (a lane then holds 4 keys x 1 query, and the two 16-key
// tiles of a 32-key block are interleaved so that the exponentiated scores of a lane are already the 8-key B
// fragment of O^T = V^T . P^T); V is cached transposed so that its fragments are 16-byte loads too. Wavefronts of a
// workgroup take 32-key blocks round-robin and are merged through LDS in a fixed order; several workgroups may split
// a long prefix (grid.z); attn_combine_kernel then merges their partial results in split order.
// fp32 kernel: vector arithmetic, exact softmax over all visible keys; the projection leaves q, k and v un-rotated, the kernel
// rotates them on their way into LDS.
#pragma once
#include "clasp_common.h"

namespace clasp {

struct AttnArgs {
    const float* qkv;  // fp32 path: [rows][ld_qkv]: q heads | k heads | v heads, un-rotated
    int ld_qkv;
    int n_rows, n_heads, n_kv_heads, head_dim;
    int pos0, mode;
    const float2* rope;  // [max_seq][head_dim/2] (cos, sin)
    void* Kc;            // this layer: fp32 [n_kv_heads][t_max][head_dim]; bf16: fragment order (kfrag_offset)
    void* Vt;            // this layer: fp32 [n_kv_heads][head_dim][t_max]; bf16: fragment order (vfrag_offset)
    int t_max;
    void* out_op;  // operand of the output projection (K = n_heads*head_dim)
    int R;
    int n_split;
    float* partial;      // [n_kv_heads][query groups][n_split][NT*16][head_dim+2] when n_split > 1
    float scale;         // 1/sqrt(head_dim)
    // bf16 path: written by the q/k/v projection's epilogue
    const void* q_frag;
    const void* k_self;  // [n_kv_heads] one 32-position block each: the DP candidates' own keys / values
    const void* v_self;
};

// The scalars that the attention kernels need first, preloaded like those of the GEMM kernels.
#define ATTN_LEAD_PARAMS                                                                                            \
    const void *lead_q, const void *lead_k, const void *lead_v, int lead_pos0, int lead_rows, int lead_heads,        \
        int lead_kv_heads, int lead_t_max, int lead_mode, int lead_split
#define ATTN_LEAD_ARGS(a) (a).q_frag, (a).Kc, (a).Vt, (a).pos0, (a).n_rows, (a).n_heads, (a).n_kv_heads, (a).t_max, (a).mode, (a).n_split
#define ATTN_F32_LEAD_PARAMS                                                                                        \
    const float *lead_qkv, const void *lead_k, const void *lead_v, const float2 *lead_rope, int lead_ld, int lead_hd, \
        int lead_pos0, int lead_t_max, int lead_heads, int lead_kv_heads
#define ATTN_F32_LEAD_ARGS(a) \
    (a).qkv, (a).Kc, (a).Vt, (a).rope, (a).ld_qkv, (a).head_dim, (a).pos0, (a).t_max, (a).n_heads, (a).n_kv_heads

#ifndef CLASP_ATTN_DOUBLE_NT
#define CLASP_ATTN_DOUBLE_NT 1  // query tiles up to which a workgroup keeps two whole fragment sets
#endif

// Keys and values of a long prefix are read once per launch and should not displace anything (streaming loads); a
// short prefix is read by the sibling workgroups of its KV head within microseconds and fits in L2 many times over,
// where plain loads let the siblings hit (measured: 1.5 us per layer at T = 512, the other way round from 8k tokens on).
template <bool STREAM>
__device__ __forceinline__ u32x4 load_kv(const u32x4* p) {
    if constexpr (STREAM) return load_stream(p);
    else return *p;
}

constexpr float kLog2e = 1.4426950408889634f;

template <int HD, int NT>
struct AttnState {
    float m[NT], l[NT];
    f32x4 o[NT][HD / 16];
};

// Fragments of one 32-key block: k[u][kk] = A fragment of key tile u (16 keys), k-step kk; v[c] = A fragment of V^T
// rows c*16..c*16+15.
template <int HD>
struct AttnFrags {
    kvx8 k[2][HD / 32], v[HD / 16];
};

// All of a block's key and value fragments are requested together (and, in the pipelined loop, one block ahead), so
// that neither the value loads nor the next block wait behind the softmax.
template <int HD, class KF, class VF>
__device__ __forceinline__ void attn_load(AttnFrags<HD>& f, KF kf, VF vf) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int kk = 0; kk < HD / 32; ++kk) f.k[u][kk] = kf(u, kk);
#pragma unroll
    for (int c = 0; c < HD / 16; ++c) f.v[c] = vf(c);
}

// One 32-key block in two steps, so that a pipelined loop can re-use the key registers for the next block's keys as
// soon as the scores exist, and the value registers as soon as the block is accumulated.
// attn_scores: S^T = K Q^T for NT query tiles, online softmax update (running max / sum, rescaling of O^T), leaves the
//              exponentiated scores as the B fragments pf[t] of the second product.
//   valid(u, r, t) -> whether key (lane/16)*8 + u*4 + r of the block is visible to query t*16 + lane%16
// attn_pv:     O^T += V^T P^T.
//   masked (wave-uniform) = false promises that valid() holds for every key of the block and every query of the
//   wavefront (a block below the diagonal of a causal pass), and the comparisons are left out.
// The exponentials are the hardware's 2^x (v_exp_f32: arguments are <= 0, results in [0, 1], tiny ones may flush to 0).
// O^T and the running sum are only rescaled in blocks where some query's running maximum grows (for the others the
// factor is exactly 1): after the first few blocks of a long prefix that is rare, and the rescaling is a third of the
// vector work of a block.
// attn_qk: the raw scores S^T = K Q^T of one block (MFMAs only); attn_softmax: everything between the two products.
template <int HD, int NT>
__device__ __forceinline__ void attn_qk(f32x4 (&s)[2][NT], const kvx8 (&qf)[NT][HD / 32], const kvx8 (&kfr)[2][HD / 32]) {
    constexpr int KK = HD / 32;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
        for (int t = 0; t < NT; ++t) s[u][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
                s[u][t] = mfma_kv(kfr[u][kk], qf[t][kk], s[u][t]);
        }
    }
}

template <int HD, int NT, class VALID>
__device__ __forceinline__ void attn_softmax(AttnState<HD, NT>& st, f32x4 (&s)[2][NT], VALID valid, kvx8 (&pf)[NT], bool masked) {
    constexpr int CT = HD / 16;
    if (masked) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (!valid(u, r, t)) s[u][t][r] = -INFINITY;
    }
    float m_safe[NT], m_new[NT];
    bool grew = false;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        float mx = -INFINITY;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) mx = fmaxf(mx, s[u][t][r]);
        mx = max32(max16(mx));
        m_new[t] = fmaxf(st.m[t], mx);
        m_safe[t] = (m_new[t] == -INFINITY) ? 0.f : m_new[t];
        grew = grew || m_new[t] > st.m[t];
    }
    if (__builtin_amdgcn_ballot_w64(grew) != 0) {  // wave-uniform: some query's maximum grew
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float alpha = __builtin_amdgcn_exp2f(st.m[t] - m_safe[t]);
            st.l[t] *= alpha;
            st.m[t] = m_new[t];
#pragma unroll
            for (int c = 0; c < CT; ++c) st.o[t][c] *= alpha;
        }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        float psum = 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float p = __builtin_amdgcn_exp2f(s[u][t][r] - m_safe[t]);
                psum += p;
                pf[t][u * 4 + r] = (kv_t)p;  // p in [0, 1]
            }
        st.l[t] += psum;
    }
}

template <int HD, int NT, class VALID>
__device__ __forceinline__ void attn_scores(AttnState<HD, NT>& st, const kvx8 (&qf)[NT][HD / 32],
                                            const kvx8 (&kfr)[2][HD / 32], VALID valid, kvx8 (&pf)[NT], bool masked = true) {
    f32x4 s[2][NT];
    attn_qk<HD, NT>(s, qf, kfr);
    attn_softmax<HD, NT>(st, s, valid, pf, masked);
}

template <int HD, int NT>
__device__ __forceinline__ void attn_pv(AttnState<HD, NT>& st, const kvx8 (&vfr)[HD / 16], const kvx8 (&pf)[NT]) {
#pragma unroll
    for (int c = 0; c < HD / 16; ++c) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
            st.o[t][c] = mfma_kv(vfr[c], pf[t], st.o[t][c]);
    }
}

template <int HD, int NT, class VALID>
__device__ __forceinline__ void attn_compute(AttnState<HD, NT>& st, const kvx8 (&qf)[NT][HD / 32],
                                             const AttnFrags<HD>& f, VALID valid, bool masked = true) {
    kvx8 pf[NT];
    attn_scores<HD, NT>(st, qf, f.k, valid, pf, masked);
    attn_pv<HD, NT>(st, f.v, pf);
}

// q_frag: queries of one KV head (query index qi = row*group + head%group) as MFMA B fragments,
// [kv_head][qi/16][x/32][lane = ((x%32)/8)*16 + qi%16][x%8], written by the q/k/v projection's epilogue.
template <int HD, int NT, int NW, bool STREAM>
__global__ __launch_bounds__(NW * 64) void attn_bf16_kernel(ATTN_LEAD_PARAMS, AttnArgs a) {
    constexpr int KK = HD / 32, CT = HD / 16;
    extern __shared__ float lds_dyn[];  // NW*HD*17 floats: per-wavefront O^T tiles (+1 column against bank conflicts)
    typedef float (*MgT)[HD][17];
    MgT mg_o = reinterpret_cast<MgT>(lds_dyn);
    __shared__ float mg_m[NW][16], mg_l[NW][16], mg_f[NW][16];
    const int kvh = blockIdx.x, qg = blockIdx.y, split = blockIdx.z;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int G = lead_heads / lead_kv_heads, nQ = lead_rows * G;
    const int q_base = qg * NT * 16;
    const int m16 = lane & 15, q4 = lane >> 4;
    const kv_t* Kc = reinterpret_cast<const kv_t*>(lead_k);
    const kv_t* Vt = reinterpret_cast<const kv_t*>(lead_v);

    // query fragments straight from HBM/L2 (already rotated, scaled and in B-operand order)
    kvx8 qf[NT][KK];
    {
        const u32x4* qp = reinterpret_cast<const u32x4*>(lead_q) + ((size_t)kvh * (2 * G) + qg * NT) * KK * 64 + lane;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) qf[t][kk] = as_kvx8(qp[(t * KK + kk) * 64]);
    }
    // visibility: query qi of row r sees cache keys <= limit (verify/draft: pos0 + r, its own position, whose
    // key/value the projection kernel has just written; DP candidates: pos0 - 1) and, for DP candidates, its own
    // entry of the self block
    int limit[NT], qrow[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int qi = q_base + t * 16 + m16;
        qrow[t] = qi < nQ ? qi / G : -1;
        limit[t] = qi < nQ ? (lead_mode ? lead_pos0 + qrow[t] : lead_pos0 - 1) : -1;
    }

    AttnState<HD, NT> st;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        st.m[t] = -INFINITY;
        st.l[t] = 0.f;
#pragma unroll
        for (int c = 0; c < CT; ++c) st.o[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    const int n_cache = lead_pos0 + (lead_mode ? lead_rows : 0);  // cache positions any row may see
    const int nblk = (n_cache + 31) >> 5;
    const int b0 = (int)(((long long)nblk * split) / lead_split), b1 = (int)(((long long)nblk * (split + 1)) / lead_split);
    const u32x4* Kh = reinterpret_cast<const u32x4*>(Kc + (size_t)kvh * lead_t_max * HD) + lane;
    const u32x4* Vh = reinterpret_cast<const u32x4*>(Vt + (size_t)kvh * lead_t_max * HD) + lane;
    auto load_blk = [&](AttnFrags<HD>& f, int blk) {
        const u32x4* kp = Kh + (size_t)blk * (2 * KK * 64);
        const u32x4* vp = Vh + (size_t)blk * (CT * 64);
        attn_load<HD>(f, [&](int u, int kk) { return as_kvx8(load_kv<STREAM>(kp + (u * KK + kk) * 64)); },
                      [&](int c) { return as_kvx8(load_kv<STREAM>(vp + c * 64)); });
    };
    auto compute_blk = [&](const AttnFrags<HD>& f, int blk) {
        const int kb = blk << 5;
        attn_compute<HD, NT>(st, qf, f, [&](int u, int r, int t) { return kb + q4 * 8 + u * 4 + r <= limit[t]; });
    };
    int blk = b0 + wave;
    if constexpr (NT <= CLASP_ATTN_DOUBLE_NT || (NW <= 4 && NT <= 3)) {  // registers allow a second fragment set (four wavefronts: one per SIMD, the whole register file each): the next block is in flight during the MFMAs
        AttnFrags<HD> f0, f1;
        if (blk < b1) load_blk(f0, blk);
        while (blk < b1) {
            if (blk + NW < b1) load_blk(f1, blk + NW);
            compute_blk(f0, blk);
            blk += NW;
            if (blk >= b1) break;
            if (blk + NW < b1) load_blk(f0, blk + NW);
            compute_blk(f1, blk);
            blk += NW;
        }
    } else {
        // one fragment set, re-used in flight: the next block's keys are requested as soon as this block's scores
        // exist (they land during the softmax and the second product), its values as soon as the block is accumulated
        AttnFrags<HD> f;
        auto load_k = [&](int b) {
            const u32x4* kp = Kh + (size_t)b * (2 * KK * 64);
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int kk = 0; kk < KK; ++kk) f.k[u][kk] = as_kvx8(load_kv<STREAM>(kp + (u * KK + kk) * 64));
        };
        auto load_v = [&](int b) {
            const u32x4* vp = Vh + (size_t)b * (CT * 64);
#pragma unroll
            for (int c = 0; c < CT; ++c) f.v[c] = as_kvx8(load_kv<STREAM>(vp + c * 64));
        };
        if (blk < b1) {
            load_k(blk);
            load_v(blk);
        }
        for (; blk < b1; blk += NW) {
            const int kb = blk << 5;
            kvx8 pf[NT];
            attn_scores<HD, NT>(st, qf, f.k, [&](int u, int r, int t) { return kb + q4 * 8 + u * 4 + r <= limit[t]; }, pf);
            if (blk + NW < b1) load_k(blk + NW);
            attn_pv<HD, NT>(st, f.v, pf);
            if (blk + NW < b1) load_v(blk + NW);
        }
    }
    if (!lead_mode && split == lead_split - 1 && wave == (b1 - b0) % NW) {  // DP candidates: own key/value only
        const u32x4* kp = reinterpret_cast<const u32x4*>(a.k_self) + (size_t)kvh * (2 * KK * 64) + lane;
        const u32x4* vp = reinterpret_cast<const u32x4*>(a.v_self) + (size_t)kvh * (CT * 64) + lane;
        AttnFrags<HD> f;
        attn_load<HD>(f, [&](int u, int kk) { return as_kvx8(kp[(u * KK + kk) * 64]); },
                      [&](int c) { return as_kvx8(vp[c * 64]); });
        attn_compute<HD, NT>(st, qf, f, [&](int u, int r, int t) { return q4 * 8 + u * 4 + r == qrow[t]; });
    }

    // merge the wavefronts' running (max, sum, O^T), one query tile at a time, fixed order
    float* part = a.partial + ((((size_t)kvh * gridDim.y + qg) * lead_split + split) * NT * 16) * (HD + 2);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        float l = st.l[t];
        l = add32(add16(l));
        if (lane < 16) {
            mg_m[wave][lane] = st.m[t];
            mg_l[wave][lane] = l;
        }
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) mg_o[wave][c * 16 + q4 * 4 + r][m16] = st.o[t][c][r];
        __syncthreads();
        if (tid < 16) {  // per query: global max, rescale factors, total sum
            float mstar = -INFINITY;
            for (int w = 0; w < NW; ++w) mstar = fmaxf(mstar, mg_m[w][tid]);
            float L = 0.f;
            for (int w = 0; w < NW; ++w) {
                const float mw = mg_m[w][tid];
                const float f = (mw == -INFINITY) ? 0.f : exp2f(mw - mstar);
                mg_f[w][tid] = f;
                L += f * mg_l[w][tid];
            }
            mg_m[0][tid] = mstar;
            mg_l[0][tid] = L;
        }
        __syncthreads();
        for (int idx = tid; idx < HD * 16; idx += NW * 64) {
            const int e = idx >> 4, j = idx & 15, qi = q_base + t * 16 + j;
            if (qi < nQ) {
                float O = 0.f;
                for (int w = 0; w < NW; ++w) O += mg_f[w][j] * mg_o[w][e][j];
                if (lead_split == 1) {
                    const int row = qi / G, h = kvh * G + qi % G;
                    store_operand<kDtBf16>(a.out_op, a.R, 0, row, h * HD + e, O / mg_l[0][j]);
                } else {
                    float* p = part + (size_t)(t * 16 + j) * (HD + 2);
                    p[e] = O;
                    if (e == 0) {
                        p[HD] = mg_m[0][j];
                        p[HD + 1] = mg_l[0][j];
                    }
                }
            }
        }
        __syncthreads();
    }
}

// Merges the n_split partial results of one query and writes the output-projection operand. Grid (kv heads, queries),
// kCombineWaves wavefronts: every thread first takes the largest of the splits' maxima (the same few words for the whole
// workgroup), then wavefront w adds the rescaled sums of splits w, w + kCombineWaves, .. for two head-dim elements per
// lane (all of a wavefront's loads in flight together), and the wavefronts' sums are added in order through LDS.
constexpr int kCombineWaves = 4;
__global__ __launch_bounds__(kCombineWaves * 64) void attn_combine_kernel(AttnArgs a, int nt, int qgroups) {
    __shared__ float sL[kCombineWaves];
    __shared__ float2 sO[kCombineWaves][64];
    const int kvh = blockIdx.x, qi = blockIdx.y, HD = a.head_dim;
    const int G = a.n_heads / a.n_kv_heads;
    const int qg = qi / (nt * 16), ql = qi % (nt * 16);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const size_t sstride = (size_t)nt * 16 * (HD + 2);
    const float* pq = a.partial + (((size_t)kvh * qgroups + qg) * a.n_split) * sstride + (size_t)ql * (HD + 2);
    float mstar = -INFINITY;
#pragma unroll 8
    for (int s = 0; s < a.n_split; ++s) mstar = fmaxf(mstar, pq[s * sstride + HD]);
    float L = 0.f;
    float2 O = make_float2(0.f, 0.f);
    const bool live = 2 * lane < HD;  // head_dim 64: half of the lanes carry elements
#pragma unroll 4
    for (int s = wave; s < a.n_split; s += kCombineWaves) {
        const float2 ml = *reinterpret_cast<const float2*>(pq + s * sstride + HD);
        const float2 ov = live ? *reinterpret_cast<const float2*>(pq + s * sstride + 2 * lane) : make_float2(0.f, 0.f);
        const float f = (ml.x == -INFINITY) ? 0.f : exp2f(ml.x - mstar);
        L += f * ml.y;
        O.x += f * ov.x;
        O.y += f * ov.y;
    }
    if (lane == 0) sL[wave] = L;
    sO[wave][lane] = O;
    __syncthreads();
    if (wave == 0 && live) {
        float Lt = sL[0];
        float2 Ot = sO[0][lane];
        for (int w = 1; w < kCombineWaves; ++w) {
            Lt += sL[w];
            Ot.x += sO[w][lane].x;
            Ot.y += sO[w][lane].y;
        }
        const int row = qi / G, h = kvh * G + qi % G;
        store_operand<kDtBf16>(a.out_op, a.R, 0, row, h * HD + 2 * lane, Ot.x / Lt);
        store_operand<kDtBf16>(a.out_op, a.R, 0, row, h * HD + 2 * lane + 1, Ot.y / Lt);
    }
}

// fp32 path: one workgroup per (query head, row), exact softmax over all visible keys. Bound by latency (the fp32 models
// are small), so everything a short prefix needs is requested in one trip to memory: the first 64 keys and values of the
// prefix into registers, the query and the launch's own visible keys (both rotated on the way) and values into LDS, from
// where the rest of the kernel, the cache write included, takes them. Four lanes share a key (16-byte pieces of its row),
// sixteen lanes a feature of V (stored transposed: 64 positions per load).
// Measured at 5 rows behind 64 tokens, head_dim 64: one thread per key and per feature, 4 bytes at a time, the own keys
// rotated by every query that sees them: 9.1 us; 7.9 us now. Behind 1000 tokens about 40 -> 25 us.
// head_dim not a multiple of 8 (VEC = false) takes the same steps element by element.
// Dynamic LDS: attn_f32_lds_floats() floats.
constexpr size_t attn_f32_lds_floats(int head_dim, int pos0, int n_rows) {
    return (size_t)head_dim * (2 + 2 * n_rows) + pos0 + 32 + 4;
}
template <bool VEC>
__global__ __launch_bounds__(256) void attn_f32_kernel(ATTN_F32_LEAD_PARAMS, AttnArgs a) {
    extern __shared__ __align__(16) float lds[];
    __shared__ float red[8];
    const int h = blockIdx.x, r = blockIdx.y, HD = lead_hd, HALF = HD / 2;
    const int G = lead_heads / lead_kv_heads, kvh = h / G;
    const int pos = lead_pos0 + (a.mode ? r : 0);
    const int n_self = a.mode ? r + 1 : 1;  // visible self keys: rows 0..r, or only row r
    const int self0 = a.mode ? 0 : r;
    const int n_keys = lead_pos0 + n_self;
    const int tid = threadIdx.x, lane = tid & 63, sub = tid & 3, l16 = tid & 15, g16 = tid >> 4, key = tid >> 2;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float* q = lds;                        // [HD], then the n_self own keys, then the n_self own values
    float* own_k = q + HD;
    float* own_v = own_k + n_self * HD;
    float* sc = lds + (HD * (1 + 2 * n_self) + 3) / 4 * 4;  // [n_keys]
    const float* Kc = reinterpret_cast<const float*>(lead_k) + (size_t)kvh * lead_t_max * HD;
    const float* Vt = reinterpret_cast<const float*>(lead_v) + (size_t)kvh * HD * lead_t_max;
    const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
    // rows 0 (query), 1..n_self (own keys), n_self+1.. (own values), a wavefront each, as rotary pairs (e, e + HALF)
    const int rows = 1 + 2 * n_self;
    struct Pair { float x, y; float2 cs; };
    auto fetch = [&](int row, int e) -> Pair {
        const int kind = row == 0 ? 0 : (row <= n_self ? 1 : 2);
        const int sr = kind == 0 ? r : self0 + (row - 1) - (kind == 2 ? n_self : 0);
        const int head = kind == 0 ? h : lead_heads + kvh + (kind == 2 ? lead_kv_heads : 0);
        const float* p = lead_qkv + (size_t)sr * lead_ld + head * HD + e;
        const float2 cs = lead_rope[(size_t)(lead_pos0 + (a.mode ? sr : 0)) * HALF + e];
        return Pair{p[0], p[HALF], kind < 2 ? cs : make_float2(1.f, 0.f)};
    };
    auto stash = [&](const Pair& p, int row, int e) {
        q[row * HD + e] = p.x * p.cs.x - p.y * p.cs.y;
        q[row * HD + e + HALF] = p.y * p.cs.x + p.x * p.cs.y;
    };
    // the first three rows of the wavefront and its pieces of the first 64 keys and values of the prefix: one trip
    constexpr int kRows = 3, kPre = 4;
    Pair pr[kRows];
    f32x4 kpre[kPre], vpre[kPre];
    const int e0 = min(lane, HALF - 1);
#pragma unroll
    for (int u = 0; u < kRows; ++u) pr[u] = fetch(min(wave + 4 * u, rows - 1), e0);
    auto load_v = [&](int e, int t) {  // positions t .. t+3; those at or beyond pos0 are not this call's to use
        f32x4 v = *reinterpret_cast<const f32x4*>(Vt + (size_t)e * lead_t_max + t);
#pragma unroll
        for (int u = 1; u < 4; ++u) v[u] = t + u < lead_pos0 ? v[u] : 0.f;
        return v;
    };
    if constexpr (VEC) {
#pragma unroll
        for (int i = 0; i < kPre; ++i) {
            const int e = (i * 4 + sub) * 4, ev = i * 16 + g16;
            kpre[i] = key < lead_pos0 && e < HD ? *reinterpret_cast<const f32x4*>(Kc + (size_t)key * HD + e) : zero;
            vpre[i] = l16 * 4 < lead_pos0 && ev < HD ? load_v(ev, l16 * 4) : zero;
        }
    }
#pragma unroll
    for (int u = 0; u < kRows; ++u)
        if (wave + 4 * u < rows && lane < HALF) stash(pr[u], wave + 4 * u, lane);
#pragma unroll 1
    for (int row = wave; row < rows; row += 4)  // what the first trip did not take
#pragma unroll 1
        for (int e = lane + (row < 4 * kRows ? 64 : 0); e < HALF; e += 64) stash(fetch(row, e), row, e);
    __syncthreads();
    float mx = -INFINITY;
    auto dot4 = [&](const f32x4& k, int e) {
        const f32x4 qv = *reinterpret_cast<const f32x4*>(q + e);
        return (qv[0] * k[0] + qv[1] * k[1]) + (qv[2] * k[2] + qv[3] * k[3]);
    };
    auto score = [&](float s, int t) {  // the four lanes of a key add up
        s += dpp<kDppXor1>(s);
        s += dpp<kDppXor2>(s);
        s *= a.scale;
        if (sub == 0) sc[t] = s;
        mx = fmaxf(mx, s);
    };
#pragma unroll 1
    for (int t = key; t < lead_pos0; t += 64) {
        float s = 0.f;
        const float* kp = Kc + (size_t)t * HD;
        if constexpr (VEC) {
            int e = sub * 4;
            if (t == key) {
#pragma unroll
                for (int i = 0; i < kPre; ++i)
                    if (e + i * 16 < HD) s += dot4(kpre[i], e + i * 16);
                e += kPre * 16;
            }
#pragma unroll 4
            for (; e < HD; e += 16) s += dot4(*reinterpret_cast<const f32x4*>(kp + e), e);
        } else {
            for (int e = sub; e < HD; e += 4) s = fmaf(q[e], kp[e], s);
        }
        score(s, t);
    }
    if (key < n_self) {  // at most 32
        float s = 0.f;
#pragma unroll 4
        for (int e = sub; e < HD; e += 4) s = fmaf(q[e], own_k[key * HD + e], s);
        score(s, lead_pos0 + key);
    }
    mx = wave_max(mx);
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    float den = 0.f;
#pragma unroll 1
    for (int t = tid; t < n_keys; t += 256) {
        const float p = expf(sc[t] - mx);
        sc[t] = p;
        den += p;
    }
    // The last piece of four positions below pos0 reads weights up to pos0 + 2, of which those from n_keys > pos0 on belong
    // to nobody: their values count as zero, but zero times a word that an earlier kernel left could be a NaN. (The barriers
    // of block_sum stand between these stores and the reads.)
    if (tid < 2) sc[n_keys + tid] = 0.f;
    den = block_sum(den, red + 4);
    // feature e of the output: sixteen lanes take positions l16*4 + 64*j .. +3 each, and own values l16, l16 + 16
    auto pv4 = [&](const f32x4& v, int t) {
        const f32x4 p = *reinterpret_cast<const f32x4*>(sc + t);
        return (p[0] * v[0] + p[1] * v[1]) + (p[2] * v[2] + p[3] * v[3]);
    };
    float first[kPre];
    if constexpr (VEC) {
#pragma unroll
        for (int i = 0; i < kPre; ++i) first[i] = l16 * 4 < lead_pos0 ? pv4(vpre[i], l16 * 4) : 0.f;
    }
#pragma unroll 1
    for (int i = 0; i * 16 < HD; ++i) {
        const int e = i * 16 + g16;
        float o = 0.f;
        if (e < HD) {
            if constexpr (VEC) {
                int t = l16 * 4;
                if (i < kPre) {
                    o = i == 0 ? first[0] : (i == 1 ? first[1] : (i == 2 ? first[2] : first[3]));
                    t += 64;
                }
#pragma unroll 4
                for (; t < lead_pos0; t += 64) o += pv4(load_v(e, t), t);
            } else {
                for (int t = l16; t < lead_pos0; t += 16) o = fmaf(sc[t], Vt[(size_t)e * lead_t_max + t], o);
            }
            for (int k = l16; k < n_self; k += 16) o = fmaf(sc[lead_pos0 + k], own_v[k * HD + e], o);
        }
        o = sum16(o);
        if (e < HD && l16 == 0) store_operand<kDtF32>(a.out_op, a.R, lead_heads * HD, r, h * HD + e, o / den);
    }
    if (a.mode && h % G == 0) {  // this row's key/value into the cache: the last of the own ones
        float* Kw = reinterpret_cast<float*>(a.Kc) + ((size_t)kvh * lead_t_max + pos) * HD;
        float* Vw = reinterpret_cast<float*>(a.Vt) + (size_t)kvh * HD * lead_t_max + pos;
        for (int e = tid; e < HD; e += 256) {
            Kw[e] = own_k[r * HD + e];
            Vw[(size_t)e * lead_t_max] = own_v[r * HD + e];
        }
    }
}

}  // namespace clasp
