// Softmax branch over the compacted keys to fp32 accuracy: the forward of fp32 arithmetic (with its merge epilogue), the
// branch's rows and log-sum-exps for the backward pass, and the backward pass itself (Section 4.2).
//   o_nla[t] = softmax_{c < cnt[t]}(scale q_t . Kc[c]) Vc        (Eq. 11 under the mask of Eq. 12: the keys visible to
//                                                                  query t are the first cnt[t] compacted rows)
//   O[t] = O_la[t] + o_nla[t], Eq. 21, or its ablation with one normalisation;  cnt[t] == 0 gives o_nla = 0, lse = -inf
// Backward, with P_ic = exp(scale q_i . Kc[c] - lse_i), dP_ic = do_i . Vc[c], D_i = do_i . o_nla_i:
//   dS_ic = P_ic (dP_ic - D_i)                 (Eq. 15: also the gradient of the mask entry)
//   dq_i  = scale sum_c dS_ic Kc[c],   dKc_c = scale sum_i dS_ic q_i,   dVc_c = sum_i P_ic do_i,   g_c = sum_i dS_ic
// and the rows of dKc, dVc, g go back to the token positions idx[c] they were gathered from.
// Routing per chunk: a query sees the compacted rows of earlier chunks and then, causally, its own chunk's rows of K
// and V (no mask stands on those: they add to dq, dk, dv and not to g).
//
// All products run on the bf16 matrix instruction with operands as sums of bf16 terms (softmax_terms.h): bf16 tensors
// are one term, fp32 tensors, the weights P, dS and fp32 gradients of the output rows three.  The kernels before this
// took the products of fp32 tensors on the vector units: at B 4, H 6, L 4096, d 128, routing per chunk, fp32, the branch's
// rows 710 -> 206 us, dQ 640 -> 271, dK / dV over the compacted keys 790 -> 314, inside the chunks 483 -> 114.  For bf16
// tensors they took two fp16 terms of P and dS (22 of 24 bits, and the range of fp16), with transposed fp16 copies of
// the tiles written to LDS: at B 2, H 16, L 8192, d 128 dQ 170 -> 146 us, dK / dV 185 -> 182.  What bounds them: per tile
// and wavefront about as much vector work (masks, exponentials, splitting) as matrix work, and as many LDS reads (every
// wavefront reads the whole tile for 16 rows of its own), which two blocks per CU overlap in part.
//
// Every kernel: a block of 4 wavefronts, wavefront w owns 16 rows of one side (queries, or keys) as the 16 columns of its
// result tiles; the other side's rows come as tiles of 64 through LDS.  Products over d read the tile's rows, products
// over the tile's rows read it transposed (ds_read_b64_tr_b16), and P and dS go from the first product's result tiles
// into the second product's operand in registers.  A tile's product starts from zero and is added to the running sum by
// a vector add: the matrix instruction's own accumulation does not round to nearest, and over a long walk (a first token
// seen by 8192 queries) its error showed (1.6e-4 of dV's RMS; 6e-5 this way).  It truncates towards minus infinity, and D,
// which dP is taken from, is summed by rounding adds: g and the chunk scores, sums of dS over all queries in which dP and D
// cancel, then collect that error with one sign (2e-6 .. 8e-6 of the chunk scores' norm at L 700 .. 1700, 64-bit arithmetic
// as the measure).  So every other step of dP's contraction is taken with one operand negated and subtracted: the errors
// have both signs and the scores are off by 3e-7 .. 1.1e-6, as with sums that round to nearest (4e-7 .. 1.8e-6).  No sum runs over blocks: results are deterministic.
#include <math.h>

#include "softmax_terms.h"

namespace nats {

constexpr float LOG2E = 1.44269504088896341f, LN2 = 0.69314718055994531f;

// e^x for x <= 0 and a little above.  x is a logit minus the row's maximum or log-sum-exp, taken in one rounding: it is small
// where the weight counts, so the factor's and the product's rounding are too.  (Logits, maxima and log-sum-exps in base 2
// would save this multiplication and round each of them at their own size: queries and keys of RMS norm 2, logits of up
// to 20, d 128: the branch's rows 7.5e-7 from 64 bits, dV 9e-7.)
__device__ __forceinline__ float exp_of(float x) { return __builtin_amdgcn_exp2f(LOG2E * x); }

// logits from the two sums of mfma_terms; bf16 tensors have one product and no rest
template <int NT>
__device__ __forceinline__ void add_rest(f32x4 (&s)[4], const f32x4 (&rest)[4]) {
    if constexpr (NT > 1) {
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) s[mt] += rest[mt];
    }
}

// Grid of the kernels whose blocks own queries: one-dimensional, tile-major over (batch, head) pairs padded to a multiple
// of 8.  The last tiles, which see the most keys, are dispatched first, and the blocks of a pair land on the same XCD
// and share its L2 for the compacted keys.
struct QueryBlock { int bh, q0; };
__device__ __forceinline__ QueryBlock query_block(int n_bh) {
    const int pad = (n_bh + 7) & ~7, n_tiles = gridDim.x / pad;
    return {(int)(blockIdx.x % pad), (n_tiles - 1 - (int)(blockIdx.x / pad)) * 64};
}
static dim3 query_grid(int n_bh, int L) { return dim3((unsigned)((size_t)((n_bh + 7) & ~7) * (L / 64))); }

template <typename T, int D>
struct SmFwdArgs {
    const T *Q, *Kc, *Vc, *K, *V;
    const int32_t* cnt;
    const float *O_la, *w_nla, *w_la;
    T* O;
    float *O_nla, *lse;
    int L, BH, chunk_routing;   // BH: output heads; chunk_routing: tokens per routing chunk (64 or 128), 0 with routing per token
    float scale, eps;
    int combine_mode, G, qk_per_out_head, own_chunk;
};

// ---- forward --------------------------------------------------------------------------------------------------------
// S^T [key][query] = K Q^T, online maximum and sum per query (a result column: 4 lanes), O^T [d][query] += V^T P^T.
template <typename T, int D>
__global__ __launch_bounds__(256, sizeof(T) == 2 ? 2 : 1) void softmax_terms_fwd_kernel(const SmFwdArgs<T, D> a) {
    constexpr int NT = terms_of<T>(), KS = D / 32, MD = D / 16, NPC = 64 * D / 8 / 256;
    using Tile = TermTile<D, NT>;
    extern __shared__ __align__(16) unsigned char st_smem[];
    const Tile Kt{reinterpret_cast<uint16_t*>(st_smem)}, Vt{reinterpret_cast<uint16_t*>(st_smem + Tile::BYTES)};
    const auto [bh, q0] = query_block(a.BH);
    if (bh >= a.BH) return;
    const int tid = threadIdx.x, L = a.L;
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, lq = lane >> 4;
    // bh counts output heads; the G heads of a group share the counts of linear head bh / G, and take their queries
    // (and the raw keys of their own chunk) from it unless the softmax heads have their own
    const size_t tokb = (size_t)bh * L, tokb_lin = (size_t)(bh / a.G) * L;
    const size_t tokb_qk = a.qk_per_out_head ? tokb : tokb_lin;
    const int t = q0 + 16 * w + l16;   // this lane's query

    u32x4 qf[KS][NT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        Raw8<T> r;
        r.load(a.Q + (tokb_qk + t) * D + 32 * ks + 8 * lq);
        r.terms(qf[ks]);
    }
    const int cs = a.chunk_routing ? (q0 & ~(a.chunk_routing - 1)) : 0;
    const int my_cnt = a.chunk_routing ? (cs > 0 ? a.cnt[tokb_lin + cs - 1] : 0) : a.cnt[tokb_lin + t];
    const int n_hi = a.chunk_routing ? my_cnt : a.cnt[tokb_lin + q0 + 63];   // cnt is non-decreasing: the block's bound
    const int n_comp = (n_hi + 63) >> 6, n_own = (a.chunk_routing && a.own_chunk) ? (q0 + 64 - cs) >> 6 : 0;

    f32x4 acc[MD];
#pragma unroll
    for (int md = 0; md < MD; ++md) acc[md] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;   // l_run: this lane's share of the sum

    // tile it: compacted rows 64 it .. , then the chunk's own rows; fetched while the tile before it is multiplied
    Raw8<T> rk[NPC], rv[NPC];
    auto fetch = [&](int it) {
        const bool own = it >= n_comp;
        const int row0 = own ? cs + 64 * (it - n_comp) : 64 * it, n_rows = own ? 64 : n_hi - row0;
        const T* kb = (own ? a.K + tokb_qk * D : a.Kc + tokb * D) + (size_t)row0 * D;
        const T* vb = (own ? a.V : a.Vc) + (tokb + row0) * D;
#pragma unroll
        for (int i = 0; i < NPC; ++i) {
            const int e = tid + 256 * i, row = e / (D / 8), c = (e % (D / 8)) * 8;
            rk[i].zero();
            rv[i].zero();
            if (row < n_rows) {   // rows past the bound are not initialised: they enter as zeros
                rk[i].load(kb + (size_t)row * D + c);
                rv[i].load(vb + (size_t)row * D + c);
            }
        }
    };
    if (n_comp + n_own > 0) fetch(0);
#pragma unroll 1
    for (int it = 0; it < n_comp + n_own; ++it) {
        const bool own = it >= n_comp;
        const int mine = own ? t + 1 - cs - 64 * (it - n_comp) : my_cnt - 64 * it;   // this query sees rows < mine of the tile
        __syncthreads();   // the previous tile has been read by everyone
#pragma unroll
        for (int i = 0; i < NPC; ++i) {
            const int e = tid + 256 * i, row = e / (D / 8), c = (e % (D / 8)) * 8;
            u32x4 x[NT];
            rk[i].terms(x);
            Kt.put(row, c, x);
            rv[i].terms(x);
            Vt.put(row, c, x);
        }
        __syncthreads();
        if (it + 1 < n_comp + n_own) fetch(it + 1);
        if (wave_extreme_i32<true>(mine) <= 0) continue;   // uniform: none of the wavefront's queries sees the tile
        f32x4 s[4], sr[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) s[mt] = sr[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                u32x4 k[NT];
                Kt.rows(16 * mt + l16, 32 * ks + 8 * lq, k);
                mfma_terms(k, qf[ks], s[mt], sr[mt]);   // rows: keys 16 mt + 4 lq + j, column: query l16
            }
        add_rest<NT>(s, sr);
        if (wave_extreme_i32<false>(mine) < 64) {   // uniform: some query does not see the whole tile
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int j = 0; j < 4; ++j) s[mt][j] = 16 * mt + 4 * lq + j < mine ? s[mt][j] : -INFINITY;
        }
        float tm = -INFINITY;
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int j = 0; j < 4; ++j) tm = fmaxf(tm, s[mt][j]);
        tm *= a.scale;   // > 0
        tm = fmaxf(tm, lane_xor16(tm, lane));
        tm = fmaxf(tm, lane_xor32(tm, lane));
        const float m_new = fmaxf(m_run, tm), m_use = m_new == -INFINITY ? 0.f : m_new;   // nothing visible yet: weights 0
        const float corr = exp_of(m_run - m_use);   // exp(-inf) = 0 on the first tile
        m_run = m_new;
        float ps = 0.f;
        u32x4 p[2][N_TERMS];
#pragma unroll
        for (int mp = 0; mp < 2; ++mp) {
            float x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                x[j] = exp_of(fmaf(a.scale, s[2 * mp + (j >> 2)][j & 3], -m_use));
                ps += x[j];
            }
            split_terms(x, p[mp]);
        }
        l_run = l_run * corr + ps;
#pragma unroll
        for (int md = 0; md < MD; ++md) {
            f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int mp = 0; mp < 2; ++mp) {
                u32x4 v[NT];
                Vt.cols(32 * mp, 16 * md, l16, lq, v);
                x = mfma_terms(v, p[mp], x);   // rows: d = 16 md + 4 lq + j, column: query l16
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[md][j] = fmaf(acc[md][j], corr, x[j]);
        }
    }
    // ---- epilogue: normalise, optional branch outputs, merge, store; the query's row lies in its 4 lanes
    l_run += lane_xor16(l_run, lane);
    l_run += lane_xor32(l_run, lane);
    // A weight 0 times a NaN or an infinity in a row of V that the query does not see is NaN (and an infinity's second term is one
    // by itself).  So a wavefront with a query that did not come out finite walks its queries' own rows once more, one row at a
    // time on the vector units, and what came out that way stands for those queries.
    float seen = 0.f * l_run;   // stays 0 while all is finite
#pragma unroll
    for (int md = 0; md < MD; ++md)
#pragma unroll
        for (int j = 0; j < 4; ++j) seen = fmaf(acc[md][j], 0.f, seen);
    seen += lane_xor16(seen, lane);
    seen += lane_xor32(seen, lane);
    if (__any(seen != 0.f)) {
        f32x4 acc2[MD];
#pragma unroll
        for (int md = 0; md < MD; ++md) acc2[md] = f32x4{0.f, 0.f, 0.f, 0.f};
        float m = -INFINITY, l = 0.f;
        const T* qr = a.Q + (tokb_qk + t) * D + 4 * lq;
        auto walk = [&](const T* kb, const T* vb, int n) {   // the query sees the first n rows
            const int n_max = wave_extreme_i32<true>(n);     // all lanes stay: the sums below run across them
#pragma unroll 1
            for (int c = 0; c < n_max; ++c) {
                const T *kr = kb + (size_t)c * D + 4 * lq, *vr = vb + (size_t)c * D + 4 * lq;
                float dot = 0.f;
#pragma unroll
                for (int md = 0; md < MD; ++md)
#pragma unroll
                    for (int j = 0; j < 4; ++j) dot = fmaf(to_float(qr[16 * md + j]), to_float(kr[16 * md + j]), dot);
                dot += lane_xor16(dot, lane);
                dot += lane_xor32(dot, lane);
                if (c >= n) continue;
                const float sc = a.scale * dot, m_new = fmaxf(m, sc), m_use = m_new == -INFINITY ? 0.f : m_new;
                const float corr = exp_of(m - m_use), pw = exp_of(sc - m_use);
                m = m_new;
                l = l * corr + pw;
#pragma unroll
                for (int md = 0; md < MD; ++md)
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc2[md][j] = fmaf(pw, to_float(vr[16 * md + j]), acc2[md][j] * corr);
            }
        };
        walk(a.Kc + tokb * D, a.Vc + tokb * D, my_cnt);
        if (n_own > 0) walk(a.K + (tokb_qk + cs) * D, a.V + (tokb + cs) * D, t + 1 - cs);
        if (seen != 0.f) {
            m_run = m;
            l_run = l;
#pragma unroll
            for (int md = 0; md < MD; ++md) acc[md] = acc2[md];
        }
    }
    const float inv_l = l_run > 0.f ? 1.f / l_run : 0.f;
    const size_t row = tokb + t;
    if (a.lse != nullptr && lq == 0) a.lse[row] = l_run > 0.f ? m_run + __builtin_amdgcn_logf(l_run) * LN2 : -INFINITY;
#pragma unroll
    for (int md = 0; md < MD; ++md) {
        acc[md][0] *= inv_l; acc[md][1] *= inv_l; acc[md][2] *= inv_l; acc[md][3] *= inv_l;
        if (a.O_nla != nullptr)
            *reinterpret_cast<float4*>(a.O_nla + row * D + 16 * md + 4 * lq) = make_float4(acc[md][0], acc[md][1], acc[md][2], acc[md][3]);
    }
    if (a.O == nullptr) return;   // the caller wanted the branch's rows and lse only (backward pass)
    f32x4 la[MD];
#pragma unroll
    for (int md = 0; md < MD; ++md) la[md] = *reinterpret_cast<const f32x4*>(a.O_la + row * D + 16 * md + 4 * lq);
    auto row_sum = [&](float x) { x += lane_xor16(x, lane); x += lane_xor32(x, lane); return x; };
    const float none = a.combine_mode == 1 ? 0.5f : 1.f;   // weights not given
    float wn = 1.f, wl = 1.f, after = 1.f;
    if (a.combine_mode != 0) {
        wn = a.w_nla ? a.w_nla[row] : none;
        wl = a.w_la ? a.w_la[row] : none;
    }
    if (a.combine_mode == 1) {          // Eq. 21: each branch normalised, then weighted
        float ss_la = 0.f, ss_nla = 0.f;
#pragma unroll
        for (int md = 0; md < MD; ++md)
#pragma unroll
            for (int j = 0; j < 4; ++j) { ss_la += la[md][j] * la[md][j]; ss_nla += acc[md][j] * acc[md][j]; }
        wn /= sqrtf(row_sum(ss_nla) / D + a.eps);
        wl /= sqrtf(row_sum(ss_la) / D + a.eps);
    } else if (a.combine_mode == 2) {   // one normalisation of the (weighted) sum
        float ss = 0.f;
#pragma unroll
        for (int md = 0; md < MD; ++md)
#pragma unroll
            for (int j = 0; j < 4; ++j) { const float x = wn * acc[md][j] + wl * la[md][j]; ss += x * x; }
        after = 1.f / sqrtf(row_sum(ss) / D + a.eps);
    }
#pragma unroll
    for (int md = 0; md < MD; ++md) {
        float o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = (wn * acc[md][j] + wl * la[md][j]) * after;
        T* dst = a.O + row * D + 16 * md + 4 * lq;
        if constexpr (sizeof(T) == 4)
            *reinterpret_cast<float4*>(dst) = make_float4(o[0], o[1], o[2], o[3]);
        else
            *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
    }
}

// ---- backward: dQ and D -------------------------------------------------------------------------------------------------
// The forward's walk over the key tiles once more: S^T = K Q^T, dP^T = V dO^T, dQ^T [d][query] += K^T dS^T.  The block's
// 64 queries are one chunk, so with routing per chunk its own chunk is one more tile.
template <typename T, typename TO>
struct SmDqArgs {
    const T *Q, *Kc, *Vc, *K, *V;
    const TO* dO;
    const int32_t* vis;   // compacted rows visible to a query (nondecreasing within a head)
    const float *O_nla, *lse;
    float *Dvec, *dQ;
    int L, BH, own_chunk;   // BH: output heads (of V, dO, the cache and the results); the G of a group share vis and,
    int G, qk_per_out_head; // unless the softmax heads have their own, Q and K
    float scale;
};
template <typename T, typename TO, int D>
__global__ __launch_bounds__(256, sizeof(T) == 2 ? 2 : 1) void softmax_terms_dq_kernel(const SmDqArgs<T, TO> a) {
    constexpr int NT = terms_of<T>(), NO = terms_of<TO>(), KS = D / 32, MD = D / 16, NPC = 64 * D / 8 / 256;
    using Tile = TermTile<D, NT>;
    extern __shared__ __align__(16) unsigned char st_smem[];
    const Tile Kt{reinterpret_cast<uint16_t*>(st_smem)}, Vt{reinterpret_cast<uint16_t*>(st_smem + Tile::BYTES)};
    const auto [bh, q0] = query_block(a.BH);
    if (bh >= a.BH) return;
    const int tid = threadIdx.x;
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, lq = lane >> 4;
    const size_t tokb = (size_t)bh * a.L, tokb_lin = (size_t)(bh / a.G) * a.L, tokb_qk = a.qk_per_out_head ? tokb : tokb_lin;
    const int t = q0 + 16 * w + l16;   // this lane's query

    u32x4 qf[KS][NT], of[KS][NO];
    float Dq = 0.f;   // D = do . o: the query's row lies in its 4 lanes
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const size_t off = (tokb + t) * D + 32 * ks + 8 * lq;
        Raw8<T> r;
        r.load(a.Q + (tokb_qk + t) * D + 32 * ks + 8 * lq);
        r.terms(qf[ks]);
        Raw8<TO> ro;
        ro.load(a.dO + off);
        ro.terms(of[ks]);
        if (ks & 1) negate(of[ks]);
        float x[8];
        ro.floats(x);
        const float4 o0 = ld4(a.O_nla + off), o1 = ld4(a.O_nla + off + 4);
        Dq += x[0] * o0.x + x[1] * o0.y + x[2] * o0.z + x[3] * o0.w + x[4] * o1.x + x[5] * o1.y + x[6] * o1.z + x[7] * o1.w;
    }
    Dq += lane_xor16(Dq, lane);
    Dq += lane_xor32(Dq, lane);
    if (lq == 0) a.Dvec[tokb + t] = Dq;
    const float lse = a.lse[tokb + t];
    const int my_cnt = a.vis[tokb_lin + t], n_hi = a.vis[tokb_lin + q0 + 63];
    const int n_comp = (n_hi + 63) >> 6, n_all = n_comp + (a.own_chunk ? 1 : 0);

    f32x4 acc[MD];
#pragma unroll
    for (int md = 0; md < MD; ++md) acc[md] = f32x4{0.f, 0.f, 0.f, 0.f};
    Raw8<T> rk[NPC], rv[NPC];
    auto fetch = [&](int it) {
        const bool own = it >= n_comp;
        const int row0 = own ? q0 : 64 * it, n_rows = own ? 64 : n_hi - row0;
        const T* kb = (own ? a.K + tokb_qk * D : a.Kc + tokb * D) + (size_t)row0 * D;
        const T* vb = (own ? a.V : a.Vc) + (tokb + row0) * D;
#pragma unroll
        for (int i = 0; i < NPC; ++i) {
            const int e = tid + 256 * i, row = e / (D / 8), c = (e % (D / 8)) * 8;
            rk[i].zero();
            rv[i].zero();
            if (row < n_rows) {
                rk[i].load(kb + (size_t)row * D + c);
                rv[i].load(vb + (size_t)row * D + c);
            }
        }
    };
    if (n_all > 0) fetch(0);
#pragma unroll 1
    for (int it = 0; it < n_all; ++it) {
        const int mine = it >= n_comp ? 16 * w + l16 + 1 : my_cnt - 64 * it;   // this query sees rows < mine of the tile
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NPC; ++i) {
            const int e = tid + 256 * i, row = e / (D / 8), c = (e % (D / 8)) * 8;
            u32x4 x[NT];
            rk[i].terms(x);
            Kt.put(row, c, x);
            rv[i].terms(x);
            Vt.put(row, c, x);
        }
        __syncthreads();
        if (it + 1 < n_all) fetch(it + 1);
        if (wave_extreme_i32<true>(mine) <= 0) continue;   // uniform
        f32x4 s[4], sr[4], dp[4], dn[4];   // dn: the steps with the negated operand
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) s[mt] = sr[mt] = dp[mt] = dn[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                u32x4 k[NT], v[NT];
                Kt.rows(16 * mt + l16, 32 * ks + 8 * lq, k);
                Vt.rows(16 * mt + l16, 32 * ks + 8 * lq, v);
                mfma_terms(k, qf[ks], s[mt], sr[mt]);
                if (ks & 1) dn[mt] = mfma_terms(v, of[ks], dn[mt]);
                else dp[mt] = mfma_terms(v, of[ks], dp[mt]);
            }
        add_rest<NT>(s, sr);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) dp[mt] -= dn[mt];
        u32x4 ds[2][N_TERMS];
#pragma unroll
        for (int mp = 0; mp < 2; ++mp) {
            float x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int mt = 2 * mp + (j >> 2), key = 16 * mt + 4 * lq + (j & 3);
                const float p = key < mine ? exp_of(fmaf(a.scale, s[mt][j & 3], -lse)) : 0.f;
                x[j] = p * (dp[mt][j & 3] - Dq);
            }
            split_terms(x, ds[mp]);
        }
#pragma unroll
        for (int md = 0; md < MD; ++md) {
            f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int mp = 0; mp < 2; ++mp) {
                u32x4 k[NT];
                Kt.cols(32 * mp, 16 * md, l16, lq, k);
                x = mfma_terms(k, ds[mp], x);
            }
            acc[md] += x;
        }
    }
#pragma unroll
    for (int md = 0; md < MD; ++md)
        *reinterpret_cast<float4*>(a.dQ + (tokb + t) * D + 16 * md + 4 * lq) =
            make_float4(a.scale * acc[md][0], a.scale * acc[md][1], a.scale * acc[md][2], a.scale * acc[md][3]);
}

// ---- backward: dK, dV, column sums of dS -------------------------------------------------------------------------------
// Wavefront w owns 16 keys and walks query tiles: S [query][key] = Q K^T, dP = dO V^T, dV^T [d][key] += dO^T P,
// dK^T [d][key] += Q^T dS.
//   OWN = false: 64 compacted keys per block, an n_seg-th share of the queries that see the first of them; the shares are
//       added up, in order, and scattered by a second kernel.
//   OWN = true (routing per chunk): the chunk's own 64 keys, its 64 queries, causal; added onto dK and dV.
template <typename T, typename TO>
struct SmDkvArgs {
    const T *Q, *K, *V;   // OWN: the tensors; otherwise Kc, Vc
    const TO* dO;
    const int32_t *vis, *idx, *n_s;
    const float *lse, *Dvec;
    float *dk, *dv, *g;   // OWN: dK, dV; otherwise the shares [n_seg][BH][L][..]
    int L, BH, n_seg;
    int G, qk_per_out_head;   // as above; the G of a group share idx and n_s too
    float scale;
};
template <typename T, typename TO, int D>
struct DkvLds {
    using QTile = TermTile<D, terms_of<T>()>;
    using OTile = TermTile<D, terms_of<TO>()>;
    static constexpr int bytes = QTile::BYTES + OTile::BYTES + 3 * 64 * 4;
    static constexpr int blocks = 2 * bytes <= 160 * 1024 ? 2 : 1;   // per CU
};
template <typename T, typename TO, int D, bool OWN>
__global__ __launch_bounds__(256, (DkvLds<T, TO, D>::blocks)) void softmax_terms_dkv_kernel(const SmDkvArgs<T, TO> a) {
    constexpr int NT = terms_of<T>(), NO = terms_of<TO>(), KS = D / 32, MD = D / 16, NPC = 64 * D / 8 / 256;
    using LY = DkvLds<T, TO, D>;
    extern __shared__ __align__(16) unsigned char st_smem[];
    const typename LY::QTile Qt{reinterpret_cast<uint16_t*>(st_smem)};
    const typename LY::OTile Ot{reinterpret_cast<uint16_t*>(st_smem + LY::QTile::BYTES)};
    float* s_lse = reinterpret_cast<float*>(st_smem + LY::QTile::BYTES + LY::OTile::BYTES);
    float* s_D = s_lse + 64;
    int* s_vis = reinterpret_cast<int*>(s_D + 64);
    // One-dimensional grid, the key tile slowest: the tiles that hold keys (the first ones) are dispatched first, the
    // heaviest of all (tile 0, seen by every query) at the very front; the empty ones follow and exit at once.  (With the
    // key tile as the fastest dimension the few working blocks sat between thousands of empty ones, each of which
    // claims a block's LDS and registers before it can exit: 1.2 ms instead of 0.35 in the kernel before this one.)
    const int seg = OWN ? 0 : blockIdx.x % a.n_seg, bh = (blockIdx.x / a.n_seg) % a.BH, c0 = (blockIdx.x / a.n_seg / a.BH) * 64;
    const int tid = threadIdx.x, L = a.L;
    const int n_keys = OWN ? L : a.n_s[bh / a.G];
    if (c0 >= n_keys) return;                          // uniform: this tile holds no key
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, lq = lane >> 4;
    const int c = c0 + 16 * w + l16;                   // this lane's key
    const bool valid = c < n_keys;
    const size_t tokb = (size_t)bh * L, tokb_lin = (size_t)(bh / a.G) * L, tokb_qk = a.qk_per_out_head ? tokb : tokb_lin;

    // the wavefront's rows of K and V (row of an invalid key: the tile's first, masked below)
    u32x4 kf[KS][NT], vf[KS][NT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const size_t off = (size_t)(valid ? c : c0) * D + 32 * ks + 8 * lq;
        Raw8<T> r;
        r.load(a.K + (OWN ? tokb_qk : tokb) * D + off);
        r.terms(kf[ks]);
        r.load(a.V + tokb * D + off);
        r.terms(vf[ks]);
        if (ks & 1) negate(vf[ks]);
    }
    f32x4 accK[MD], accV[MD];
#pragma unroll
    for (int md = 0; md < MD; ++md) { accK[md] = f32x4{0.f, 0.f, 0.f, 0.f}; accV[md] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    float g = 0.f;

    // the queries that see the tile's first key, in tiles; the blocks of the tile take equal shares of them
    const int i_first = OWN ? c0 : a.idx[tokb_lin + c0] & ~63;
    const int n_tiles = OWN ? 1 : (L - i_first) / 64;
    const int i_lo = i_first + (int)((long long)n_tiles * seg / a.n_seg) * 64;
    const int i_hi = i_first + (int)((long long)n_tiles * (seg + 1) / a.n_seg) * 64;
    Raw8<T> rq[NPC];
    Raw8<TO> ro[NPC];
    float rl = 0.f, rd = 0.f;
    int rc = 0;
    auto fetch = [&](int i0) {   // L is a multiple of the tile
#pragma unroll
        for (int i = 0; i < NPC; ++i) {
            const int e = tid + 256 * i, row = e / (D / 8), col = (e % (D / 8)) * 8;
            rq[i].load(a.Q + (tokb_qk + i0 + row) * D + col);
            ro[i].load(a.dO + (tokb + i0 + row) * D + col);
        }
        if (tid < 64) {
            rl = a.lse[tokb + i0 + tid];
            rd = a.Dvec[tokb + i0 + tid];
            if (!OWN) rc = a.vis[tokb_lin + i0 + tid];
        }
    };
    // the next tile is fetched while this one is multiplied, except where the gradients' two registers per value do not
    // fit beside the accumulators at two blocks per CU
    constexpr bool AHEAD = !(NT == 1 && NO == N_TERMS && D == 128);
    if (AHEAD && i_lo < i_hi) fetch(i_lo);
#pragma unroll 1
    for (int i0 = i_lo; i0 < i_hi; i0 += 64) {
        if (!AHEAD) fetch(i0);
        __syncthreads();   // the previous tile has been read by everyone
#pragma unroll
        for (int i = 0; i < NPC; ++i) {
            const int e = tid + 256 * i, row = e / (D / 8), col = (e % (D / 8)) * 8;
            u32x4 x[NT], y[NO];
            rq[i].terms(x);
            Qt.put(row, col, x);
            ro[i].terms(y);
            Ot.put(row, col, y);
        }
        if (tid < 64) { s_lse[tid] = rl; s_D[tid] = rd; s_vis[tid] = OWN ? c0 + tid + 1 : rc; }
        __syncthreads();
        if (AHEAD && i0 + 64 < i_hi) fetch(i0 + 64);
        f32x4 s[4], sr[4], dp[4], dn[4];   // dn: the steps with the negated operand
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) s[mt] = sr[mt] = dp[mt] = dn[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                u32x4 q[NT], o[NO];
                Qt.rows(16 * mt + l16, 32 * ks + 8 * lq, q);
                Ot.rows(16 * mt + l16, 32 * ks + 8 * lq, o);
                mfma_terms(q, kf[ks], s[mt], sr[mt]);   // rows: queries 16 mt + 4 lq + j, column: key l16
                if (ks & 1) dn[mt] = mfma_terms(o, vf[ks], dn[mt]);
                else dp[mt] = mfma_terms(o, vf[ks], dp[mt]);
            }
        add_rest<NT>(s, sr);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) dp[mt] -= dn[mt];
        u32x4 p[2][N_TERMS], ds[2][N_TERMS];
#pragma unroll
        for (int mp = 0; mp < 2; ++mp) {
            float x[8], y[8];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int mt = 2 * mp + h;
                const float4 l4 = *reinterpret_cast<const float4*>(s_lse + 16 * mt + 4 * lq);
                const float4 d4 = *reinterpret_cast<const float4*>(s_D + 16 * mt + 4 * lq);
                const int4 c4 = *reinterpret_cast<const int4*>(s_vis + 16 * mt + 4 * lq);
                const float ls[4] = {l4.x, l4.y, l4.z, l4.w}, dd[4] = {d4.x, d4.y, d4.z, d4.w};
                const int vs[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float pj = (valid && c < vs[j]) ? exp_of(fmaf(a.scale, s[mt][j], -ls[j])) : 0.f;
                    const float dj = pj * (dp[mt][j] - dd[j]);
                    g += dj;
                    x[4 * h + j] = pj;
                    y[4 * h + j] = dj;
                }
            }
            split_terms(x, p[mp]);
            split_terms(y, ds[mp]);
        }
#pragma unroll
        for (int md = 0; md < MD; ++md) {
            f32x4 xv = {0.f, 0.f, 0.f, 0.f}, xk = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int mp = 0; mp < 2; ++mp) {
                u32x4 q[NT], o[NO];
                Ot.cols(32 * mp, 16 * md, l16, lq, o);
                Qt.cols(32 * mp, 16 * md, l16, lq, q);
                xv = mfma_terms(o, p[mp], xv);   // rows: d = 16 md + 4 lq + j, column: key l16
                xk = mfma_terms(q, ds[mp], xk);
            }
            accV[md] += xv;
            accK[md] += xk;
        }
    }
    if (OWN) {
        float* dk = a.dk + (tokb + c) * D;
        float* dv = a.dv + (tokb + c) * D;
        float4 k0[MD], v0[MD];
#pragma unroll
        for (int md = 0; md < MD; ++md) { k0[md] = ld4(dk + 16 * md + 4 * lq); v0[md] = ld4(dv + 16 * md + 4 * lq); }
#pragma unroll
        for (int md = 0; md < MD; ++md) {
            *reinterpret_cast<float4*>(dk + 16 * md + 4 * lq) =
                make_float4(k0[md].x + a.scale * accK[md][0], k0[md].y + a.scale * accK[md][1],
                            k0[md].z + a.scale * accK[md][2], k0[md].w + a.scale * accK[md][3]);
            *reinterpret_cast<float4*>(dv + 16 * md + 4 * lq) =
                make_float4(v0[md].x + accV[md][0], v0[md].y + accV[md][1], v0[md].z + accV[md][2], v0[md].w + accV[md][3]);
        }
        return;
    }
    g += lane_xor16(g, lane);
    g += lane_xor32(g, lane);
    if (valid) {   // this block's share, by compacted key
        const size_t row = ((size_t)seg * a.BH + bh) * L + c;
#pragma unroll
        for (int md = 0; md < MD; ++md) {
            *reinterpret_cast<float4*>(a.dk + row * D + 16 * md + 4 * lq) = make_float4(accK[md][0], accK[md][1], accK[md][2], accK[md][3]);
            *reinterpret_cast<float4*>(a.dv + row * D + 16 * md + 4 * lq) = make_float4(accV[md][0], accV[md][1], accV[md][2], accV[md][3]);
        }
        if (lq == 0) a.g[row] = g;
    }
}

// Adds the segments' shares of a compacted key up, in order, and writes the rows of dK, dV (and g_nla) of the
// token the key was gathered from (its linear-branch gradient is zero).  One thread per key and 4 columns.
// dKb, dVb (both or neither; not with accumulate): the rows go there as bf16 instead.
template <int D>
__global__ __launch_bounds__(256) void softmax_bwd_dkv_combine_kernel(
    const float* __restrict__ dk_part, const float* __restrict__ dv_part, const float* __restrict__ g_part,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ n_s, float* __restrict__ dK, float* __restrict__ dV,
    float* __restrict__ g_nla, bf16_t* __restrict__ dKb, bf16_t* __restrict__ dVb, int L, int G, int n_seg, float scale,
    int accumulate) {
    constexpr int TPK = D / 4;                 // threads per key
    const int bh = blockIdx.y, c = blockIdx.x * (256 / TPK) + threadIdx.x / TPK, col = (threadIdx.x % TPK) * 4;
    if (c >= n_s[bh / G]) return;
    const size_t tokb = (size_t)bh * L;
    const int t = idx[(size_t)(bh / G) * L + c];   // the token the key was gathered from
    float4 k = make_float4(0.f, 0.f, 0.f, 0.f), v = k;
    float g = 0.f;
    for (int s = 0; s < n_seg; ++s) {
        const size_t row = ((size_t)s * gridDim.y + bh) * L + c;
        const float4 a = *reinterpret_cast<const float4*>(dk_part + row * D + col);
        const float4 b = *reinterpret_cast<const float4*>(dv_part + row * D + col);
        k.x += a.x; k.y += a.y; k.z += a.z; k.w += a.w;
        v.x += b.x; v.y += b.y; v.z += b.z; v.w += b.w;
        g += g_part[row];
    }
    const size_t dst = (tokb + t) * D + col;
    if (dKb != nullptr) {
        *reinterpret_cast<uint2*>(dKb + dst) = make_uint2(pack_bf16x2(scale * k.x, scale * k.y), pack_bf16x2(scale * k.z, scale * k.w));
        *reinterpret_cast<uint2*>(dVb + dst) = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
    } else if (accumulate) {   // routing per chunk: the token's rows already hold its shares from inside its chunk
        const float4 k0 = *reinterpret_cast<const float4*>(dK + dst), v0 = *reinterpret_cast<const float4*>(dV + dst);
        *reinterpret_cast<float4*>(dK + dst) = make_float4(k0.x + scale * k.x, k0.y + scale * k.y, k0.z + scale * k.z, k0.w + scale * k.w);
        *reinterpret_cast<float4*>(dV + dst) = make_float4(v0.x + v.x, v0.y + v.y, v0.z + v.z, v0.w + v.w);
    } else {
        *reinterpret_cast<float4*>(dK + dst) = make_float4(scale * k.x, scale * k.y, scale * k.z, scale * k.w);
        *reinterpret_cast<float4*>(dV + dst) = v;
    }
    if (col == 0 && g_nla != nullptr) g_nla[tokb + t] = g;
}

// Compacted rows a query sees: with routing per token the first cnt[t]; with routing per chunk those of earlier
// chunks, cnt at the last token before the query's chunk.  Written out once so that the backward kernels above, which
// take "rows visible to query t" as an array, serve both routings.
__global__ __launch_bounds__(256) void visible_rows_kernel(const int32_t* __restrict__ cnt, int32_t* __restrict__ vis, int L,
                                                          size_t n_tok) {
    const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= n_tok) return;
    const size_t cs = t - (t % L) % 64;          // first token of the query's chunk
    vis[t] = (cs % L) > 0 ? cnt[cs - 1] : 0;
}

// ---- launchers ----------------------------------------------------------------------------------------------------------
template <typename K>
static bool lds_limit(K kern, int bytes) {   // more than 64 KB of LDS: the limit is raised per kernel
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
}

template <typename T, int D>
static bool launch_fwd_t(const FwdPlan& pl, const void* Q, const void* Kc, const void* Vc, const void* K, const void* V,
                         const int32_t* cnt, const float* O_la, const float* w_nla, const float* w_la, void* O,
                         float* O_nla, float* lse, hipStream_t st) {
    auto kern = softmax_terms_fwd_kernel<T, D>;
    constexpr int lds = 2 * TermTile<D, terms_of<T>()>::BYTES;
    if (!lds_limit(kern, lds)) return false;
    const SmFwdArgs<T, D> a{(const T*)Q, (const T*)Kc, (const T*)Vc, (const T*)K, (const T*)V, cnt, O_la, w_nla, w_la, (T*)O,
                            O_nla, lse, pl.L, pl.BHG, pl.routing == NATS_ROUTE_CHUNK ? pl.RC : 0, pl.softmax_scale, pl.rms_eps,
                            pl.combine_mode, pl.G, pl.qk_per_out_head, pl.inner_chunk != 2};
    hipLaunchKernelGGL(kern, query_grid(pl.BHG, pl.L), dim3(256), lds, st, a);
    return true;
}

// O NULL: the branch's rows and lse only
nats_status launch_softmax_terms_fwd(const FwdPlan& pl, const void* Q, const void* Kc, const void* Vc, const void* K,
                                     const void* V, const int32_t* cnt, const float* O_la, const float* w_nla,
                                     const float* w_la, void* O, float* O_nla_out, float* lse_out, hipStream_t st) {
    bool ok;
#define NATS_SMF(TT, DD) launch_fwd_t<TT, DD>(pl, Q, Kc, Vc, K, V, cnt, O_la, w_nla, w_la, O, O_nla_out, lse_out, st)
    if (pl.dtype == NATS_BF16) ok = pl.d == 64 ? NATS_SMF(bf16_t, 64) : NATS_SMF(bf16_t, 128);
    else ok = pl.d == 64 ? NATS_SMF(float, 64) : NATS_SMF(float, 128);
#undef NATS_SMF
    if (!ok) { set_error("softmax_terms_fwd: the kernel's LDS size was refused"); return NATS_ERR_HIP; }
    return check_launch("softmax_terms_fwd");
}

template <typename T, typename TO, int D>
static bool launch_dq_t(const FwdPlan& pl, const void* Q, const void* Kc, const void* Vc, const void* K, const void* V,
                        const void* dO, const int32_t* vis, const float* O_nla, const float* lse, float* Dvec, float* dQ,
                        hipStream_t st) {
    auto kern = softmax_terms_dq_kernel<T, TO, D>;
    constexpr int lds = 2 * TermTile<D, terms_of<T>()>::BYTES;
    if (!lds_limit(kern, lds)) return false;
    const SmDqArgs<T, TO> a{(const T*)Q, (const T*)Kc, (const T*)Vc, (const T*)K, (const T*)V, (const TO*)dO, vis, O_nla, lse,
                            Dvec, dQ, pl.L, pl.BHG, pl.routing == NATS_ROUTE_CHUNK, pl.G, pl.qk_per_out_head, pl.softmax_scale};
    hipLaunchKernelGGL(kern, query_grid(pl.BHG, pl.L), dim3(256), lds, st, a);
    return true;
}

// (In this and the launchers below dQ, dK, dV, Dvec, the cache, lse, O_nla and the scratch have pl.BHG heads.)
// dQ [BHG,L,d] f32 is written (not accumulated), with routing per chunk including the queries' own chunks; also
// Dvec [BHG,L].  dO_f32: dO is fp32 whatever the tensors' type.
nats_status launch_softmax_bwd_dq(const FwdPlan& pl, const void* Q, const void* Kc, const void* Vc, const void* K, const void* V,
                                  const void* dO, bool dO_f32, const int32_t* vis, const float* O_nla, const float* lse,
                                  float* Dvec, float* dQ, hipStream_t st) {
    bool ok;
#define NATS_SMQ(TT, TO, DD) launch_dq_t<TT, TO, DD>(pl, Q, Kc, Vc, K, V, dO, vis, O_nla, lse, Dvec, dQ, st)
    if (pl.dtype == NATS_F32) ok = pl.d == 64 ? NATS_SMQ(float, float, 64) : NATS_SMQ(float, float, 128);
    else if (dO_f32) ok = pl.d == 64 ? NATS_SMQ(bf16_t, float, 64) : NATS_SMQ(bf16_t, float, 128);
    else ok = pl.d == 64 ? NATS_SMQ(bf16_t, bf16_t, 64) : NATS_SMQ(bf16_t, bf16_t, 128);
#undef NATS_SMQ
    if (!ok) { set_error("softmax_bwd_dq: the kernel's LDS size was refused"); return NATS_ERR_HIP; }
    return check_launch("softmax_bwd_dq");
}

template <typename T, typename TO, int D, bool OWN>
static bool launch_dkv_t(const FwdPlan& pl, const void* Q, const void* K, const void* V, const void* dO, const int32_t* vis,
                         const int32_t* idx, const int32_t* n_s, const float* lse, const float* Dvec, float* dk, float* dv,
                         float* g, hipStream_t st) {
    auto kern = softmax_terms_dkv_kernel<T, TO, D, OWN>;
    constexpr int lds = DkvLds<T, TO, D>::bytes;
    if (!lds_limit(kern, lds)) return false;
    const int n_seg = OWN ? 1 : BWD_DKV_SEGMENTS;
    const SmDkvArgs<T, TO> a{(const T*)Q, (const T*)K, (const T*)V, (const TO*)dO, vis, idx, n_s, lse, Dvec, dk, dv, g, pl.L,
                             pl.BHG, n_seg, pl.G, pl.qk_per_out_head, pl.softmax_scale};
    hipLaunchKernelGGL(kern, dim3((unsigned)((size_t)(pl.L / 64) * pl.BHG * n_seg)), dim3(256), lds, st, a);
    return true;
}
template <bool OWN>
static bool launch_dkv(const FwdPlan& pl, const void* Q, const void* K, const void* V, const void* dO, bool dO_f32,
                       const int32_t* vis, const int32_t* idx, const int32_t* n_s, const float* lse, const float* Dvec,
                       float* dk, float* dv, float* g, hipStream_t st) {
#define NATS_SMK(TT, TO, DD) launch_dkv_t<TT, TO, DD, OWN>(pl, Q, K, V, dO, vis, idx, n_s, lse, Dvec, dk, dv, g, st)
    if (pl.dtype == NATS_F32) return pl.d == 64 ? NATS_SMK(float, float, 64) : NATS_SMK(float, float, 128);
    if (dO_f32) return pl.d == 64 ? NATS_SMK(bf16_t, float, 64) : NATS_SMK(bf16_t, float, 128);
    return pl.d == 64 ? NATS_SMK(bf16_t, bf16_t, 64) : NATS_SMK(bf16_t, bf16_t, 128);
#undef NATS_SMK
}

// the rows idx[c] of dK, dV [BHG,L,d] f32 (and of g_nla [BHG,L], optional) are overwritten (routing per chunk: added to);
// other rows are left alone.  rounded (dK and dV, or neither; routing per token): they go there instead.  dk_part, dv_part: BWD_DKV_SEGMENTS * BHG * L * d floats, g_part: BWD_DKV_SEGMENTS * BHG * L (scratch)
nats_status launch_softmax_bwd_dkv(const FwdPlan& pl, const void* Q, const void* Kc, const void* Vc, const void* dO, bool dO_f32,
                                   const int32_t* vis, const int32_t* idx, const int32_t* n_s, const float* lse,
                                   const float* Dvec, float* dK, float* dV, float* g_nla, float* dk_part, float* dv_part,
                                   float* g_part, const RoundedGrads& rounded, hipStream_t st) {
    if (!launch_dkv<false>(pl, Q, Kc, Vc, dO, dO_f32, vis, idx, n_s, lse, Dvec, dk_part, dv_part, g_part, st)) {
        set_error("softmax_bwd_dkv: the kernel's LDS size was refused");
        return NATS_ERR_HIP;
    }
    nats_status rc = check_launch("softmax_bwd_dkv");
    if (rc != NATS_OK) return rc;
    if (pl.d == 64) {
        dim3 grid((pl.L + 15) / 16, pl.BHG);   // 256 / (64 / 4) keys per block
        hipLaunchKernelGGL((softmax_bwd_dkv_combine_kernel<64>), grid, dim3(256), 0, st, dk_part, dv_part, g_part, idx, n_s,
                           dK, dV, g_nla, (bf16_t*)rounded.dK, (bf16_t*)rounded.dV, pl.L, pl.G, BWD_DKV_SEGMENTS, pl.softmax_scale, pl.routing == NATS_ROUTE_CHUNK);
    } else {
        dim3 grid((pl.L + 7) / 8, pl.BHG);     // 256 / (128 / 4) keys per block
        hipLaunchKernelGGL((softmax_bwd_dkv_combine_kernel<128>), grid, dim3(256), 0, st, dk_part, dv_part, g_part, idx, n_s,
                           dK, dV, g_nla, (bf16_t*)rounded.dK, (bf16_t*)rounded.dV, pl.L, pl.G, BWD_DKV_SEGMENTS, pl.softmax_scale, pl.routing == NATS_ROUTE_CHUNK);
    }
    return check_launch("softmax_bwd_dkv_combine");
}

nats_status launch_visible_rows(const FwdPlan& pl, const int32_t* cnt, int32_t* vis, hipStream_t st) {
    const size_t n_tok = (size_t)pl.BH * pl.L;
    hipLaunchKernelGGL(visible_rows_kernel, dim3((unsigned)((n_tok + 255) / 256)), dim3(256), 0, st, cnt, vis, pl.L, n_tok);
    return check_launch("visible_rows");
}

// routing per chunk: the shares of dK, dV from inside every chunk, added onto the rows that are there
nats_status launch_softmax_bwd_own_chunk(const FwdPlan& pl, const void* Q, const void* K, const void* V, const void* dO,
                                         bool dO_f32, const float* lse, const float* Dvec, float* dK, float* dV, hipStream_t st) {
    if (!launch_dkv<true>(pl, Q, K, V, dO, dO_f32, nullptr, nullptr, nullptr, lse, Dvec, dK, dV, nullptr, st)) {
        set_error("softmax_bwd_own_chunk: the kernel's LDS size was refused");
        return NATS_ERR_HIP;
    }
    return check_launch("softmax_bwd_own_chunk");
}

}  // namespace nats
