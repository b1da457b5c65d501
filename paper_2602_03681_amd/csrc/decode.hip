// Single-token decode step (Section 4.1, per-token generation; per-token routing):
//   S <- alpha S ;  linear token: S <- S + beta (v - S k) k^T  (Eq. 19, Eq. 20)
//   softmax token: (k, v) appended to the KV cache of softmax tokens, and attended (Eq. 12, i >= j)
//   o = merge( la_scale * S q ,  softmax(scale * q . Kcache^T) Vcache )     (Section 4.1 / Eq. 21)
// One block per (batch, head).  HBM-bound: the fp32 state is streamed once (read +
// write, 8 d^2 bytes) and the live cache rows once (4 d len bytes for bf16).
#include <math.h>

#include "nats_common.h"

namespace nats {

constexpr int DEC_THREADS = 256;
constexpr int DEC_WIDE = 1024;   // threads of the form for few (batch, head) pairs
constexpr int DEC_WIDE_PAIRS = 256;

// A wavefront's groups of LPK lanes, each with a running maximum m, sum l and EPL columns of the accumulator per lane, into
// one (in every group), relative to the wavefront's maximum.  A group that saw no row has m = -inf.
template <int LPK, int EPL>
__device__ __forceinline__ void merge_groups(float& m, float& l, float (&acc)[EPL]) {
    const int lane = (int)(threadIdx.x & 63);
    auto across = [&](float x, auto op) {
        if (LPK <= 8) x = op(x, dpp_move<0x128>(x));   // lane ^ 8 (a rotation by 8 inside the 16-lane row)
        if (LPK <= 16) x = op(x, lane_xor16(x, lane));
        return op(x, lane_xor32(x, lane));
    };
    auto add = [](float x, float y) { return x + y; };
    const float m_w = across(m, [](float x, float y) { return fmaxf(x, y); });
    const float wgt = m_w > -INFINITY ? expf(m - m_w) : 0.f;
    l = across(wgt * l, add);
#pragma unroll
    for (int j = 0; j < EPL; ++j) acc[j] = across(wgt * acc[j], add);
    m = m_w;
}

// The block's wavefronts have one of two jobs, side by side: the first SW of them stream the state (LPR = D/4 lanes hold
// one row of S as a float4 each, all row passes of a thread loaded up front; S k and S q are reduced across the LPR
// lanes), the others the cache (LPK = D/(16/sizeof T) lanes share one row, 16 bytes per lane; every group of LPK lanes
// strides over the rows with its own running max / sum / accumulator, merged inside the wavefront and then through LDS).
// Rows are asked for one group ahead of their use, the first group before the cache's length is known (rows below
// cap exist whatever the length).  The new token is folded in from registers.
//
// What one CU streams is bound by the loads it has in flight: 16 wavefronts side by side against 4 that do one job after
// the other (decode_kernel below), us per step, bf16, d 128: 16 pairs, 64 / 256 / 1000 / 2048 rows 6.5 / 8.0 / 13.0 / 19.6
// against 7.1 / 10.5 / 22.7 / 39.4; 256 pairs 10.2 / 12.7 / 30 / 49 against 9.7 / 15.5 / 36.9 / 87.  With 512 pairs the
// blocks of four wavefronts, several to a CU, are ahead for short caches (32 rows 14.1 against 18.1) and level for long
// ones: up to DEC_WIDE_PAIRS pairs take this form.
//
// CHUNK = false: routing per token (mask: the token's type).
// CHUNK = true : routing per chunk, known only after the chunk (Section 4.1, per-token generation): every
//   token is written into the state and appended to the cache provisionally (row cache_len +
//   chunk_pos); at a chunk's first token the state is copied to state_start; chunk_decay collects the
//   chunk's decay; cache_len stays, chunk_pos advances.  decode_commit_kernel settles the chunk.
template <typename T, int D, bool CHUNK>
__global__ __launch_bounds__(DEC_WIDE) void decode_wide_kernel(
    float* __restrict__ state, float* __restrict__ state_start, float* __restrict__ chunk_decay,
    int32_t* __restrict__ chunk_pos, T* __restrict__ k_cache, T* __restrict__ v_cache,
    int32_t* __restrict__ cache_len, const T* __restrict__ q, const T* __restrict__ k,
    const T* __restrict__ v, const float* __restrict__ alpha, const float* __restrict__ beta,
    const uint8_t* __restrict__ mask, const float* __restrict__ w_nla, const float* __restrict__ w_la,
    T* __restrict__ o, int32_t* __restrict__ err_flags, int cap, float scale, float la_scale,
    int combine_mode, float eps, int linear_op, int freeze_on_softmax, const T* __restrict__ q_nla,
    const T* __restrict__ k_nla) {
    constexpr int SW = 4;                         // wavefronts on the state
    constexpr int CW = DEC_WIDE / 64 - SW;              // wavefronts on the cache
    constexpr int LPR = D / 4;                    // lanes per state row
    constexpr int ROWS_PER_PASS = 64 * SW / LPR;
    constexpr int PASSES = D / ROWS_PER_PASS;     // 16 (D = 128) or 4 (D = 64)
    constexpr int EPL = Vec16<T>::N;              // elements per lane of a cache row
    constexpr int LPK = D / EPL;                  // lanes per cache row
    constexpr int NSG = 64 * CW / LPK;            // groups of lanes on the cache
    constexpr int UNROLL = 4;

    __shared__ float s_ola[D];
    __shared__ float s_m[CW], s_l[CW];
    __shared__ float s_acc[CW][D];

    const int bh = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pos = CHUNK ? chunk_pos[bh] : 0;
    const bool is_softmax = CHUNK ? true : mask[bh] != 0;     // CHUNK: every token goes to the cache ...
    // variant without decay on softmax tokens: alpha counts as 1 there (routing per chunk: the commit decides)
    const float a = (!CHUNK && is_softmax && freeze_on_softmax) ? 1.f : alpha[bh];
    const float b = (!CHUNK && is_softmax) ? 0.f : beta[bh];  // ... and into the state
    bool append = false;   // (known to the wavefronts on the cache)
    int n_old = 0;

    if (wave < SW) {   // ---- state update and o_la = la_scale * S q ----
        const int lr = tid % LPR, r0 = tid / LPR;
        float* Sb = state + (size_t)bh * D * D;
        float kk[4], qq[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            kk[j] = to_float(k[(size_t)bh * D + lr * 4 + j]);
            qq[j] = to_float(q[(size_t)bh * D + lr * 4 + j]);
        }
        float4 S4[PASSES];
        float vv[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int row = p * ROWS_PER_PASS + r0;
            S4[p] = *reinterpret_cast<const float4*>(Sb + (size_t)row * D + lr * 4);
            vv[p] = to_float(v[(size_t)bh * D + row]);
        }
        if (CHUNK && pos == 0) {   // first token of a chunk: keep the state it starts from
            float* Sst = state_start + (size_t)bh * D * D;
#pragma unroll
            for (int p = 0; p < PASSES; ++p)
                *reinterpret_cast<float4*>(Sst + (size_t)(p * ROWS_PER_PASS + r0) * D + lr * 4) = S4[p];
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int row = p * ROWS_PER_PASS + r0;
            float4 s = S4[p];
            s.x *= a; s.y *= a; s.z *= a; s.w *= a;
            if (b != 0.f) {
                const float pred = lane_group_sum<LPR>(s.x * kk[0] + s.y * kk[1] + s.z * kk[2] + s.w * kk[3]);
                const float delta = b * (vv[p] - (linear_op == 0 ? pred : 0.f));   // no correction without the delta rule
                s.x += delta * kk[0]; s.y += delta * kk[1]; s.z += delta * kk[2]; s.w += delta * kk[3];
            }
            const float oq = lane_group_sum<LPR>(s.x * qq[0] + s.y * qq[1] + s.z * qq[2] + s.w * qq[3]);
            if (lr == 0) s_ola[row] = la_scale * oq;
            *reinterpret_cast<float4*>(Sb + (size_t)row * D + lr * 4) = s;
        }
    } else {           // ---- softmax over the cache (+ the new token) ----
        const int ct = tid - 64 * SW, lk = ct % LPK, sg = ct / LPK;
        const T* Kb = k_cache + (size_t)bh * cap * D + lk * EPL;
        const T* Vb = v_cache + (size_t)bh * cap * D + lk * EPL;
        auto load_rows = [&](int c0, int last, uint4 (&kr)[UNROLL], uint4 (&vr)[UNROLL]) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int c = min(c0 + u * NSG, last);   // rows past the end repeat the last one; masked below
                kr[u] = *reinterpret_cast<const uint4*>(Kb + (size_t)c * D);
                vr[u] = *reinterpret_cast<const uint4*>(Vb + (size_t)c * D);
            }
        };
        uint4 ka[UNROLL], va[UNROLL], kb2[UNROLL], vb2[UNROLL];
        load_rows(sg, cap - 1, ka, va);
        float qf[EPL], acc[EPL];
        const T* qs = (q_nla != nullptr ? q_nla : q) + (size_t)bh * D + lk * EPL;
        Vec16<T>::load(qs, qf);
#pragma unroll
        for (int j = 0; j < EPL; ++j) { qf[j] *= scale; acc[j] = 0.f; }
        // Rows present, provisional ones included.  Never beyond the cache: once an open chunk has filled it, or when
        // the caller's cache_len exceeds cap, the rows that exist are [0, cap) and later tokens are not stored.
        const int n_want = cache_len[bh] + pos;
        n_old = min(max(n_want, 0), cap);
        append = is_softmax && n_want >= 0 && n_want < cap;
        float m_run = -INFINITY, l_run = 0.f;
        auto use_rows = [&](int c0, const uint4 (&kr)[UNROLL], const uint4 (&vr)[UNROLL]) {
            float sc[UNROLL], bm = -INFINITY;
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                float kf[EPL];
                Vec16<T>::unpack(kr[u], kf);
                float dot = 0.f;
#pragma unroll
                for (int j = 0; j < EPL; ++j) dot += qf[j] * kf[j];
                dot = lane_group_sum<LPK>(dot);
                sc[u] = (c0 + u * NSG < n_old) ? dot : -INFINITY;
                bm = fmaxf(bm, sc[u]);
            }
            const float m_new = fmaxf(m_run, bm);   // finite: row c0 exists
            const float corr = expf(m_run - m_new);
            l_run *= corr;
#pragma unroll
            for (int j = 0; j < EPL; ++j) acc[j] *= corr;
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                // a row past the end may hold anything before it is first written: its weight is 0 and it does not enter
                if (c0 + u * NSG >= n_old) continue;
                const float p = expf(sc[u] - m_new);
                l_run += p;
                float vf[EPL];
                Vec16<T>::unpack(vr[u], vf);
#pragma unroll
                for (int j = 0; j < EPL; ++j) acc[j] += p * vf[j];
            }
            m_run = m_new;
        };
        constexpr int STEP = NSG * UNROLL;
        int c0 = sg;
        while (c0 < n_old) {
            if (c0 + STEP < n_old) load_rows(c0 + STEP, n_old - 1, kb2, vb2);
            use_rows(c0, ka, va);
            c0 += STEP;
            if (c0 >= n_old) break;
            if (c0 + STEP < n_old) load_rows(c0 + STEP, n_old - 1, ka, va);
            use_rows(c0, kb2, vb2);
            c0 += STEP;
        }
        if (append && sg == 0) {   // the new softmax token attends to itself, and goes into the cache
            const uint4 kw = *reinterpret_cast<const uint4*>((k_nla != nullptr ? k_nla : k) + (size_t)bh * D + lk * EPL);
            const uint4 vw = *reinterpret_cast<const uint4*>(v + (size_t)bh * D + lk * EPL);
            float kf[EPL], vf[EPL];
            Vec16<T>::unpack(kw, kf);
            Vec16<T>::unpack(vw, vf);
            float dot = 0.f;
#pragma unroll
            for (int j = 0; j < EPL; ++j) dot += qf[j] * kf[j];
            dot = lane_group_sum<LPK>(dot);
            const float m_new = fmaxf(m_run, dot);
            const float corr = expf(m_run - m_new);
            const float p = expf(dot - m_new);
            l_run = l_run * corr + p;
#pragma unroll
            for (int j = 0; j < EPL; ++j) acc[j] = acc[j] * corr + p * vf[j];
            m_run = m_new;
            *reinterpret_cast<uint4*>(k_cache + ((size_t)bh * cap + n_old) * D + lk * EPL) = kw;
            *reinterpret_cast<uint4*>(v_cache + ((size_t)bh * cap + n_old) * D + lk * EPL) = vw;
        }
        merge_groups<LPK, EPL>(m_run, l_run, acc);
        if (lane < LPK) {
#pragma unroll
            for (int j = 0; j < EPL; ++j) s_acc[wave - SW][lk * EPL + j] = acc[j];
            if (lane == 0) { s_m[wave - SW] = m_run; s_l[wave - SW] = l_run; }
        }
        if (ct == 0) {
            if (CHUNK) chunk_decay[bh] = (pos == 0 ? 1.f : chunk_decay[bh]) * a;
            if (err_flags != nullptr) err_flags[bh] = (is_softmax && !append) ? 1 : 0;
        }
    }
    __syncthreads();   // every thread has read chunk_pos and cache_len
    if (CHUNK && tid == 0) chunk_pos[bh] = pos + 1;
    if (!CHUNK && tid == 64 * SW && append) cache_len[bh] = n_old + 1;

    // ---- merge the wavefronts' results, then the two branches (threads 0..D-1, one output each) --------
    // D <= 128 <= 2 wavefronts; row statistics for Eq. 21 go through LDS.
    __shared__ float s_red[4];
    if (tid >= 128) return;   // (only wavefronts 0 and 1 meet at the barriers below)
    float o_nla = 0.f, o_la = 0.f;
    if (tid < D) {
        float M = -INFINITY;
#pragma unroll
        for (int g = 0; g < CW; ++g) M = fmaxf(M, s_m[g]);
        float num = 0.f, den = 0.f;
        if (M > -INFINITY) {
#pragma unroll
            for (int g = 0; g < CW; ++g) {
                const float wgt = expf(s_m[g] - M);   // wavefronts that saw no row have m = -inf -> 0
                num += wgt * s_acc[g][tid];
                den += wgt * s_l[g];
            }
            o_nla = num / den;
        }
        o_la = s_ola[tid];
    }
    if (combine_mode == 0) {
        if (tid < D) o[(size_t)bh * D + tid] = from_float<T>(o_la + o_nla);
    } else if (combine_mode == 2) {   // one normalisation of the (weighted) sum
        const float sum = (w_nla ? w_nla[bh] : 1.f) * o_nla + (w_la ? w_la[bh] : 1.f) * o_la;
        float x = (tid < D) ? sum * sum : 0.f;
        x = lane_group_sum<64>(x);
        if ((tid & 63) == 0 && tid < 128) s_red[tid >> 6] = x;
        __syncthreads();
        if (tid < D) {
            const float ss = s_red[0] + (D > 64 ? s_red[1] : 0.f);
            o[(size_t)bh * D + tid] = from_float<T>(sum / sqrtf(ss / D + eps));
        }
    } else {
        float x = (tid < D) ? o_la * o_la : 0.f, y = (tid < D) ? o_nla * o_nla : 0.f;
        x = lane_group_sum<64>(x); y = lane_group_sum<64>(y);
        if ((tid & 63) == 0 && tid < 128) { s_red[(tid >> 6) * 2] = x; s_red[(tid >> 6) * 2 + 1] = y; }
        __syncthreads();
        if (tid < D) {
            const float ss_la = s_red[0] + (D > 64 ? s_red[2] : 0.f);
            const float ss_nla = s_red[1] + (D > 64 ? s_red[3] : 0.f);
            const float wn = (w_nla ? w_nla[bh] : 0.5f) / sqrtf(ss_nla / D + eps);
            const float wl = (w_la ? w_la[bh] : 0.5f) / sqrtf(ss_la / D + eps);
            o[(size_t)bh * D + tid] = from_float<T>(wn * o_nla + wl * o_la);
        }
    }
}

// The same with 256 threads that do one job after the other: what many (batch, head) pairs take, several blocks to a CU.
template <typename T, int D, bool CHUNK>
__global__ __launch_bounds__(DEC_THREADS) void decode_kernel(
    float* __restrict__ state, float* __restrict__ state_start, float* __restrict__ chunk_decay,
    int32_t* __restrict__ chunk_pos, T* __restrict__ k_cache, T* __restrict__ v_cache,
    int32_t* __restrict__ cache_len, const T* __restrict__ q, const T* __restrict__ k,
    const T* __restrict__ v, const float* __restrict__ alpha, const float* __restrict__ beta,
    const uint8_t* __restrict__ mask, const float* __restrict__ w_nla, const float* __restrict__ w_la,
    T* __restrict__ o, int32_t* __restrict__ err_flags, int cap, float scale, float la_scale,
    int combine_mode, float eps, int linear_op, int freeze_on_softmax, const T* __restrict__ q_nla,
    const T* __restrict__ k_nla) {
    constexpr int LPR = D / 4;                    // lanes per state row
    constexpr int ROWS_PER_PASS = DEC_THREADS / LPR;
    constexpr int PASSES = D / ROWS_PER_PASS;     // 16 (D=128) or 4 (D=64)
    constexpr int EPL = Vec16<T>::N;              // elements per lane of a cache row
    constexpr int LPK = D / EPL;                  // lanes per key
    constexpr int NSG = DEC_THREADS / LPK;        // key groups in the block
    constexpr int UNROLL = 4;

    __shared__ float s_q[D], s_k[D], s_v[D], s_ola[D];
    __shared__ float s_qn[D], s_kn[D];            // query and key of the softmax branch (q, k unless given apart)
    __shared__ float s_m[NSG], s_l[NSG];
    __shared__ float s_acc[NSG][D];

    const int bh = blockIdx.x, tid = threadIdx.x;
    for (int c = tid; c < D; c += DEC_THREADS) {
        s_q[c] = to_float(q[(size_t)bh * D + c]);
        s_k[c] = to_float(k[(size_t)bh * D + c]);
        s_qn[c] = to_float((q_nla != nullptr ? q_nla : q)[(size_t)bh * D + c]);
        s_kn[c] = to_float((k_nla != nullptr ? k_nla : k)[(size_t)bh * D + c]);
        s_v[c] = to_float(v[(size_t)bh * D + c]);
    }
    const int pos = CHUNK ? chunk_pos[bh] : 0;
    const bool is_softmax = CHUNK ? true : mask[bh] != 0;     // CHUNK: every token goes to the cache ...
    // variant without decay on softmax tokens: alpha counts as 1 there (routing per chunk: the commit decides)
    const float a = (!CHUNK && is_softmax && freeze_on_softmax) ? 1.f : alpha[bh];
    const float b = (!CHUNK && is_softmax) ? 0.f : beta[bh];  // ... and into the state
    // Rows present, provisional ones included.  Never beyond the cache: once an open chunk has filled it, or when
    // the caller's cache_len exceeds cap, the rows that exist are [0, cap) and later tokens are not stored.
    const int n_want = cache_len[bh] + pos;
    const int n_old = min(max(n_want, 0), cap);
    const bool append = is_softmax && n_want >= 0 && n_want < cap;
    __syncthreads();

    // ---- phase A: state update and o_la = la_scale * S q --------------------------------
    {
        const int lr = tid % LPR, r0 = tid / LPR;
        float* Sb = state + (size_t)bh * D * D;
        float4 S4[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            S4[p] = *reinterpret_cast<const float4*>(Sb + (size_t)(p * ROWS_PER_PASS + r0) * D + lr * 4);
        const float4 k4 = *reinterpret_cast<const float4*>(&s_k[lr * 4]);
        const float4 q4 = *reinterpret_cast<const float4*>(&s_q[lr * 4]);
        if (CHUNK && pos == 0) {   // first token of a chunk: keep the state it starts from
            float* Sst = state_start + (size_t)bh * D * D;
#pragma unroll
            for (int p = 0; p < PASSES; ++p)
                *reinterpret_cast<float4*>(Sst + (size_t)(p * ROWS_PER_PASS + r0) * D + lr * 4) = S4[p];
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int row = p * ROWS_PER_PASS + r0;
            float4 s = S4[p];
            s.x *= a; s.y *= a; s.z *= a; s.w *= a;
            if (b != 0.f) {
                const float pred = lane_group_sum<LPR>(s.x * k4.x + s.y * k4.y + s.z * k4.z + s.w * k4.w);
                const float delta = b * (s_v[row] - (linear_op == 0 ? pred : 0.f));   // no correction without the delta rule
                s.x += delta * k4.x; s.y += delta * k4.y; s.z += delta * k4.z; s.w += delta * k4.w;
            }
            const float oq = lane_group_sum<LPR>(s.x * q4.x + s.y * q4.y + s.z * q4.z + s.w * q4.w);
            if (lr == 0) s_ola[row] = la_scale * oq;
            *reinterpret_cast<float4*>(Sb + (size_t)row * D + lr * 4) = s;
        }
    }

    // ---- phase B: softmax over the cache (+ the new token) ---------------------------------
    const int lk = tid % LPK, sg = tid / LPK;
    float qf[EPL], acc[EPL];
#pragma unroll
    for (int j = 0; j < EPL; ++j) { qf[j] = s_qn[lk * EPL + j] * scale; acc[j] = 0.f; }
    float m_run = -INFINITY, l_run = 0.f;
    const T* Kb = k_cache + (size_t)bh * cap * D + lk * EPL;
    const T* Vb = v_cache + (size_t)bh * cap * D + lk * EPL;

    for (int c0 = sg; c0 < n_old; c0 += NSG * UNROLL) {
        float kf[UNROLL][EPL], vf[UNROLL][EPL], s[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int c = c0 + u * NSG;
            if (c < n_old) {
                Vec16<T>::load(Kb + (size_t)c * D, kf[u]);
                Vec16<T>::load(Vb + (size_t)c * D, vf[u]);
            } else {
#pragma unroll
                for (int j = 0; j < EPL; ++j) { kf[u][j] = 0.f; vf[u][j] = 0.f; }
            }
        }
        float bm = -INFINITY;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            float dot = 0.f;
#pragma unroll
            for (int j = 0; j < EPL; ++j) dot += qf[j] * kf[u][j];
            dot = lane_group_sum<LPK>(dot);
            s[u] = (c0 + u * NSG < n_old) ? dot : -INFINITY;
            bm = fmaxf(bm, s[u]);
        }
        const float m_new = fmaxf(m_run, bm);   // finite: key c0 is live
        const float corr = expf(m_run - m_new);
        l_run *= corr;
#pragma unroll
        for (int j = 0; j < EPL; ++j) acc[j] *= corr;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const float p = expf(s[u] - m_new);
            l_run += p;
#pragma unroll
            for (int j = 0; j < EPL; ++j) acc[j] += p * vf[u][j];
        }
        m_run = m_new;
    }
    if (append && sg == 0) {   // the new softmax token attends to itself
        float dot = 0.f;
#pragma unroll
        for (int j = 0; j < EPL; ++j) dot += qf[j] * s_kn[lk * EPL + j];
        dot = lane_group_sum<LPK>(dot);
        const float m_new = fmaxf(m_run, dot);
        const float corr = expf(m_run - m_new);
        const float p = expf(dot - m_new);
        l_run = l_run * corr + p;
#pragma unroll
        for (int j = 0; j < EPL; ++j) acc[j] = acc[j] * corr + p * s_v[lk * EPL + j];
        m_run = m_new;
    }
    if (lk == 0) { s_m[sg] = m_run; s_l[sg] = l_run; }
#pragma unroll
    for (int j = 0; j < EPL; ++j) s_acc[sg][lk * EPL + j] = acc[j];
    __syncthreads();

    // ---- append the new token to the cache -------------------------------------------------
    if (append) {
        for (int c = tid; c < D; c += DEC_THREADS) {
            k_cache[((size_t)bh * cap + n_old) * D + c] = (k_nla != nullptr ? k_nla : k)[(size_t)bh * D + c];
            v_cache[((size_t)bh * cap + n_old) * D + c] = v[(size_t)bh * D + c];
        }
        if (tid == 0 && !CHUNK) cache_len[bh] = n_old + 1;
    }
    if (CHUNK && tid == 0) {
        chunk_pos[bh] = pos + 1;
        chunk_decay[bh] = (pos == 0 ? 1.f : chunk_decay[bh]) * a;
    }
    if (tid == 0 && err_flags != nullptr) err_flags[bh] = (is_softmax && !append) ? 1 : 0;

    // ---- merge the key groups, then the two branches (threads 0..D-1, one output each) --------
    // D <= 128 <= 2 wavefronts; row statistics for Eq. 21 go through LDS.
    __shared__ float s_red[4];
    float o_nla = 0.f, o_la = 0.f;
    if (tid < D) {
        float M = -INFINITY;
#pragma unroll
        for (int g = 0; g < NSG; ++g) M = fmaxf(M, s_m[g]);
        float num = 0.f, den = 0.f;
        if (M > -INFINITY) {
#pragma unroll
            for (int g = 0; g < NSG; ++g) {
                const float wgt = expf(s_m[g] - M);   // groups that saw no key have m = -inf -> 0
                num += wgt * s_acc[g][tid];
                den += wgt * s_l[g];
            }
            o_nla = num / den;
        }
        o_la = s_ola[tid];
    }
    if (combine_mode == 0) {
        if (tid < D) o[(size_t)bh * D + tid] = from_float<T>(o_la + o_nla);
    } else if (combine_mode == 2) {   // one normalisation of the (weighted) sum
        const float sum = (w_nla ? w_nla[bh] : 1.f) * o_nla + (w_la ? w_la[bh] : 1.f) * o_la;
        float x = (tid < D) ? sum * sum : 0.f;
        x = lane_group_sum<64>(x);
        if ((tid & 63) == 0 && tid < 128) s_red[tid >> 6] = x;
        __syncthreads();
        if (tid < D) {
            const float ss = s_red[0] + (D > 64 ? s_red[1] : 0.f);
            o[(size_t)bh * D + tid] = from_float<T>(sum / sqrtf(ss / D + eps));
        }
    } else {
        float x = (tid < D) ? o_la * o_la : 0.f, y = (tid < D) ? o_nla * o_nla : 0.f;
        x = lane_group_sum<64>(x); y = lane_group_sum<64>(y);
        if ((tid & 63) == 0 && tid < 128) { s_red[(tid >> 6) * 2] = x; s_red[(tid >> 6) * 2 + 1] = y; }
        __syncthreads();
        if (tid < D) {
            const float ss_la = s_red[0] + (D > 64 ? s_red[2] : 0.f);
            const float ss_nla = s_red[1] + (D > 64 ? s_red[3] : 0.f);
            const float wn = (w_nla ? w_nla[bh] : 0.5f) / sqrtf(ss_nla / D + eps);
            const float wl = (w_la ? w_la[bh] : 0.5f) / sqrtf(ss_la / D + eps);
            o[(size_t)bh * D + tid] = from_float<T>(wn * o_nla + wl * o_la);
        }
    }
}

// ------------------------------------------------------------------------------------------------------------
// The same step as many small blocks of equal size, for batches whose caches differ in length (with one block per (batch,
// head) the longest caches set the time of the step while most CUs idle) and for few (batch, head) pairs.
//   decode_split_kernel   grid (D / DSP_SROWS + n_split, B*H): the first D / DSP_SROWS blocks of a (batch, head)
//                         each update DSP_SROWS rows of the state (rows are independent) and leave their part
//                         of o_la in the workspace; block D / DSP_SROWS + s runs the online softmax over cache
//                         rows [s ROWS, (s + 1) ROWS) (exits at once if the cache ends before them) and
//                         leaves (acc[D], max, sum) in the workspace;
//   decode_combine_kernel one block per (batch, head): merges the partial softmax results and the new token
//                         (from registers), merges the branches, appends the token, stores o.
// ROWS = 64 is one trip of the block through memory; 256 rows are four, but need a quarter of the results (us per step,
// bf16, d 128, ROWS 64 / 256: 16 pairs of 1000 rows 7.2 / 8.0; 1024 pairs of 64 .. 2048 rows 138 / 142).
// Workspace per (batch, head): n_split x (D + 4) floats of partial results, then D floats of o_la.
// ------------------------------------------------------------------------------------------------------------
constexpr int DSP_ROWS = 256;       // cache rows per block: this many, or, where the workspace has room for as many results, ...
constexpr int DSP_ROWS_SMALL = 64;  // ... this many
constexpr int DSP_SROWS = 32;       // state rows per block

template <typename T, int D, bool CHUNK, int ROWS>
__global__ __launch_bounds__(DEC_THREADS) void decode_split_kernel(
    float* __restrict__ state, float* __restrict__ state_start, const int32_t* __restrict__ chunk_pos,
    const T* __restrict__ k_cache, const T* __restrict__ v_cache,
    const int32_t* __restrict__ cache_len, const T* __restrict__ q, const T* __restrict__ k,
    const T* __restrict__ v, const float* __restrict__ alpha, const float* __restrict__ beta,
    const uint8_t* __restrict__ mask, float* __restrict__ ws, int cap, int n_split, float scale, float la_scale,
    int linear_op, int freeze_on_softmax, const T* __restrict__ q_nla) {
    constexpr int NSP = D / DSP_SROWS;                // state blocks per (batch, head)
    constexpr int LPR = D / 4;                    // lanes per state row
    constexpr int ROWS_PER_PASS = DEC_THREADS / LPR;
    constexpr int PASSES = DSP_SROWS / ROWS_PER_PASS;
    constexpr int EPL = Vec16<T>::N;
    constexpr int LPK = D / EPL;
    constexpr int NSG = DEC_THREADS / LPK, NW = DEC_THREADS / 64;
    constexpr int UNROLL = ROWS / NSG < 4 ? ROWS / NSG : 4;
    const int bh = blockIdx.y, tid = threadIdx.x;
    float* wsb = ws + (size_t)bh * ((size_t)n_split * (D + 4) + D);
    const int pos = CHUNK ? chunk_pos[bh] : 0;

    if (blockIdx.x < NSP) {   // ---- state rows [part * DSP_SROWS, + DSP_SROWS) ----
        const int lr = tid % LPR, r0 = tid / LPR, row0 = blockIdx.x * DSP_SROWS;
        float* Sb = state + (size_t)bh * D * D;
        float4 S4[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            S4[p] = *reinterpret_cast<const float4*>(Sb + (size_t)(row0 + p * ROWS_PER_PASS + r0) * D + lr * 4);
        const bool is_softmax = !CHUNK && mask[bh] != 0;
        const float a = (is_softmax && freeze_on_softmax) ? 1.f : alpha[bh];
        const float b = is_softmax ? 0.f : beta[bh];
        if (CHUNK && pos == 0) {   // first token of a chunk: keep the state it starts from
            float* Sst = state_start + (size_t)bh * D * D;
#pragma unroll
            for (int p = 0; p < PASSES; ++p)
                *reinterpret_cast<float4*>(Sst + (size_t)(row0 + p * ROWS_PER_PASS + r0) * D + lr * 4) = S4[p];
        }
        float kk[4], qq[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            kk[j] = to_float(k[(size_t)bh * D + lr * 4 + j]);
            qq[j] = to_float(q[(size_t)bh * D + lr * 4 + j]);
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int row = row0 + p * ROWS_PER_PASS + r0;
            float4 s = S4[p];
            s.x *= a; s.y *= a; s.z *= a; s.w *= a;
            if (b != 0.f) {
                const float pred = lane_group_sum<LPR>(s.x * kk[0] + s.y * kk[1] + s.z * kk[2] + s.w * kk[3]);
                const float delta = b * (to_float(v[(size_t)bh * D + row]) - (linear_op == 0 ? pred : 0.f));
                s.x += delta * kk[0]; s.y += delta * kk[1]; s.z += delta * kk[2]; s.w += delta * kk[3];
            }
            const float oq = lane_group_sum<LPR>(s.x * qq[0] + s.y * qq[1] + s.z * qq[2] + s.w * qq[3]);
            if (lr == 0) wsb[(size_t)n_split * (D + 4) + row] = la_scale * oq;
            *reinterpret_cast<float4*>(Sb + (size_t)row * D + lr * 4) = s;
        }
        return;
    }

    // ---- cache rows [split * DSP_ROWS, ...) of the rows present ----
    const int split = blockIdx.x - NSP;
    const int n_old = min(max(cache_len[bh] + pos, 0), cap);
    const int c_lo = split * ROWS, c_hi = min(c_lo + ROWS, n_old);
    if (c_lo >= c_hi) return;   // uniform: the combine kernel knows which parts exist from the same length
    __shared__ float s_m[NW], s_l[NW];
    __shared__ float s_acc[NW][D];
    const int lk = tid % LPK, sg = tid / LPK;
    float qf[EPL], acc[EPL];
    {
        const T* qs = (q_nla != nullptr ? q_nla : q) + (size_t)bh * D + lk * EPL;
#pragma unroll
        for (int j = 0; j < EPL; ++j) { qf[j] = to_float(qs[j]) * scale; acc[j] = 0.f; }
    }
    float m_run = -INFINITY, l_run = 0.f;
    const T* Kb = k_cache + (size_t)bh * cap * D + lk * EPL;
    const T* Vb = v_cache + (size_t)bh * cap * D + lk * EPL;
    // Rows as they come from memory (16 bytes of a row per lane); the next group of rows is asked for before the
    // current one is used, so that a wavefront always has loads in flight.
    typedef uint4 raw_t;
    static_assert(sizeof(T) * EPL == 16, "one 16-byte word per lane and row");
    auto load_rows = [&](int c0, raw_t (&kr)[UNROLL], raw_t (&vr)[UNROLL]) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int c = min(c0 + u * NSG, c_hi - 1);   // rows past the end repeat the last one; masked below
            kr[u] = *reinterpret_cast<const raw_t*>(Kb + (size_t)c * D);
            vr[u] = *reinterpret_cast<const raw_t*>(Vb + (size_t)c * D);
        }
    };
    auto use_rows = [&](int c0, const raw_t (&kr)[UNROLL], const raw_t (&vr)[UNROLL]) {
        float sc[UNROLL], bm = -INFINITY;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            float kf[EPL];
            Vec16<T>::unpack(kr[u], kf);
            float dot = 0.f;
#pragma unroll
            for (int j = 0; j < EPL; ++j) dot += qf[j] * kf[j];
            dot = lane_group_sum<LPK>(dot);
            sc[u] = (c0 + u * NSG < c_hi) ? dot : -INFINITY;
            bm = fmaxf(bm, sc[u]);
        }
        const float m_new = fmaxf(m_run, bm);   // finite: row c0 exists
        const float corr = __builtin_amdgcn_exp2f((m_run - m_new) * 1.44269504088896341f);   // exp2(-inf) = 0
        l_run *= corr;
#pragma unroll
        for (int j = 0; j < EPL; ++j) acc[j] *= corr;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            if (c0 + u * NSG >= c_hi) continue;   // (a repeated row's weight is 0, but 0 x infinity is NaN)
            const float pw = __builtin_amdgcn_exp2f((sc[u] - m_new) * 1.44269504088896341f);
            l_run += pw;
            float vf[EPL];
            Vec16<T>::unpack(vr[u], vf);
#pragma unroll
            for (int j = 0; j < EPL; ++j) acc[j] += pw * vf[j];
        }
        m_run = m_new;
    };
    {
        raw_t ka[UNROLL], va[UNROLL], kb2[UNROLL], vb2[UNROLL];
        constexpr int STEP = NSG * UNROLL;
        int c0 = c_lo + sg;
        if (c0 < c_hi) load_rows(c0, ka, va);
        while (c0 < c_hi) {
            if (c0 + STEP < c_hi) load_rows(c0 + STEP, kb2, vb2);
            use_rows(c0, ka, va);
            c0 += STEP;
            if (c0 >= c_hi) break;
            if (c0 + STEP < c_hi) load_rows(c0 + STEP, ka, va);
            use_rows(c0, kb2, vb2);
            c0 += STEP;
        }
    }
    merge_groups<LPK, EPL>(m_run, l_run, acc);
    if ((tid & 63) < LPK) {
        const int w = tid >> 6;
#pragma unroll
        for (int j = 0; j < EPL; ++j) s_acc[w][lk * EPL + j] = acc[j];
        if (lk == 0) { s_m[w] = m_run; s_l[w] = l_run; }
    }
    __syncthreads();
    if (tid < D) {   // the block's wavefronts into one partial result, relative to the block's maximum
        float M = -INFINITY;
#pragma unroll
        for (int g = 0; g < NW; ++g) M = fmaxf(M, s_m[g]);
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int g = 0; g < NW; ++g) {
            const float wgt = expf(s_m[g] - M);   // wavefronts that saw no row have m = -inf -> 0
            num += wgt * s_acc[g][tid];
            den += wgt * s_l[g];
        }
        float* part = wsb + (size_t)split * (D + 4);
        part[tid] = num;
        if (tid == 0) { part[D] = M; part[D + 1] = den; }
    }
}

template <typename T, int D, bool CHUNK>
__global__ __launch_bounds__(DEC_THREADS) void decode_combine_kernel(
    const float* __restrict__ ws, float* __restrict__ chunk_decay, int32_t* __restrict__ chunk_pos,
    const float* __restrict__ alpha, T* __restrict__ k_cache, T* __restrict__ v_cache, int32_t* __restrict__ cache_len,
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, const uint8_t* __restrict__ mask,
    const float* __restrict__ w_nla, const float* __restrict__ w_la, T* __restrict__ o,
    int32_t* __restrict__ err_flags, int cap, int n_split, int rows, float scale, int combine_mode, float eps,
    const T* __restrict__ q_nla, const T* __restrict__ k_nla) {
    // NH groups of D threads share the parts, thread `col` of a group one column of the result
    constexpr int NH = DEC_THREADS / D, AHEAD = 8;
    const int bh = blockIdx.x, tid = threadIdx.x, lane = tid & 63, col = tid % D, h = tid / D;
    const float* wsb = ws + (size_t)bh * ((size_t)n_split * (D + 4) + D);
    __shared__ float s_red[4];
    __shared__ float s_m[NH], s_l[NH], s_num[NH][D];
    // Everything is asked for at the start, the group's first parts before it is known how many there are (a part's place
    // exists whatever the length; what it holds enters only if the part does): one trip to memory instead of three.
    float pa[AHEAD], pm[AHEAD], pl[AHEAD];
    auto load_parts = [&](int first) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const float* part = wsb + (size_t)min(first + h + i * NH, n_split - 1) * (D + 4);
            pa[i] = part[col];
            pm[i] = part[D];
            pl[i] = part[D + 1];
        }
    };
    load_parts(0);
    const T* qs = (q_nla != nullptr ? q_nla : q) + (size_t)bh * D;
    const T* ks = (k_nla != nullptr ? k_nla : k) + (size_t)bh * D;
    const T kn = ks[col], vn = v[(size_t)bh * D + col];
    float dot = to_float(qs[col]) * scale * to_float(kn);
    const float o_la = wsb[(size_t)n_split * (D + 4) + col];
    const int pos = CHUNK ? chunk_pos[bh] : 0;
    const bool is_softmax = CHUNK || mask[bh] != 0;   // CHUNK: every token goes to the cache
    const int n_want = cache_len[bh] + pos;
    const int n_old = min(max(n_want, 0), cap);
    const bool append = is_softmax && n_want >= 0 && n_want < cap;
    const int n_parts = (n_old + rows - 1) / rows;
    const bool live = tid < D;
    // logit of the new token (it attends to itself, Eq. 12 i >= j)
    dot = lane_group_sum<64>(dot);
    if (live && lane == 0) s_red[tid >> 6] = dot;
    // the group's parts
    float M = -INFINITY, num = 0.f, den = 0.f;
    for (int first = 0; first < n_parts; first += AHEAD * NH) {
        if (first > 0) load_parts(first);
        float M2 = M;
#pragma unroll
        for (int i = 0; i < AHEAD; ++i)
            if (first + h + i * NH < n_parts) M2 = fmaxf(M2, pm[i]);
        // (no part here, or none with a finite logit: weights 0, and a part that holds NaN still brings it)
        const float ref = M2 == -INFINITY ? 0.f : M2;
        const float was = expf(M - ref);
        num *= was;
        den *= was;
#pragma unroll
        for (int i = 0; i < AHEAD; ++i)
            if (first + h + i * NH < n_parts) {
                const float wgt = expf(pm[i] - ref);
                num += wgt * pa[i];
                den += wgt * pl[i];
            }
        M = M2;
    }
    s_num[h][col] = num;
    if (col == 0) { s_m[h] = M; s_l[h] = den; }
    __syncthreads();
    if (!live) return;   // the first D threads go on (the barriers below count the wavefronts that are left)
    dot = s_red[0] + (D > 64 ? s_red[1] : 0.f);
    float Mx = append ? dot : -INFINITY;
#pragma unroll
    for (int g = 0; g < NH; ++g) Mx = fmaxf(Mx, s_m[g]);
    float o_nla = 0.f;
    if (Mx > -INFINITY) {
        num = den = 0.f;
#pragma unroll
        for (int g = 0; g < NH; ++g) {
            const float wgt = expf(s_m[g] - Mx);   // a group without a part has m = -inf -> 0
            num += wgt * s_num[g][col];
            den += wgt * s_l[g];
        }
        if (append) {
            const float pw = expf(dot - Mx);
            num += pw * to_float(vn);
            den += pw;
        }
        o_nla = num / den;
    }
    __syncthreads();   // s_red is written again below
    // ---- append the new token, bookkeeping ----
    if (append) {
        k_cache[((size_t)bh * cap + n_old) * D + col] = kn;
        v_cache[((size_t)bh * cap + n_old) * D + col] = vn;
    }
    if (tid == 0) {   // (behind a barrier: every thread has read chunk_pos and cache_len)
        if (CHUNK) {
            chunk_pos[bh] = pos + 1;
            chunk_decay[bh] = (pos == 0 ? 1.f : chunk_decay[bh]) * alpha[bh];
        } else if (append) {
            cache_len[bh] = n_old + 1;
        }
        if (err_flags != nullptr) err_flags[bh] = (is_softmax && !append) ? 1 : 0;
    }
    // ---- merge of the branches ----
    if (combine_mode == 0) {
        if (live) o[(size_t)bh * D + tid] = from_float<T>(o_la + o_nla);
    } else if (combine_mode == 2) {   // one normalisation of the (weighted) sum
        const float sum = (w_nla ? w_nla[bh] : 1.f) * o_nla + (w_la ? w_la[bh] : 1.f) * o_la;
        float x = live ? sum * sum : 0.f;
        x = lane_group_sum<64>(x);
        if ((tid & 63) == 0) s_red[tid >> 6] = x;
        __syncthreads();
        if (live) {
            const float ss = s_red[0] + (D > 64 ? s_red[1] : 0.f);
            o[(size_t)bh * D + tid] = from_float<T>(sum / sqrtf(ss / D + eps));
        }
    } else {
        float x = live ? o_la * o_la : 0.f, y = live ? o_nla * o_nla : 0.f;
        x = lane_group_sum<64>(x); y = lane_group_sum<64>(y);
        if ((tid & 63) == 0) { s_red[(tid >> 6) * 2] = x; s_red[(tid >> 6) * 2 + 1] = y; }
        __syncthreads();
        if (live) {
            const float ss_la = s_red[0] + (D > 64 ? s_red[2] : 0.f);
            const float ss_nla = s_red[1] + (D > 64 ? s_red[3] : 0.f);
            const float wn = (w_nla ? w_nla[bh] : 0.5f) / sqrtf(ss_nla / D + eps);
            const float wl = (w_la ? w_la[bh] : 0.5f) / sqrtf(ss_la / D + eps);
            o[(size_t)bh * D + tid] = from_float<T>(wn * o_nla + wl * o_la);
        }
    }
}

// After a chunk has been seen and its type decided (mask_c[b,h] != 0: softmax chunk): a softmax chunk keeps
// its provisional cache rows and gives the state back as (chunk decay) x (chunk-start state); a linear
// chunk keeps the state and drops the rows.  chunk_pos returns to 0.  err_flags (optional) is set where
// rows of a softmax chunk did not fit into the cache (they were never stored).
template <int D>
__global__ __launch_bounds__(DEC_THREADS) void decode_commit_kernel(
    float* __restrict__ state, const float* __restrict__ state_start, const float* __restrict__ chunk_decay,
    int32_t* __restrict__ chunk_pos, int32_t* __restrict__ cache_len, const uint8_t* __restrict__ mask_c,
    int32_t* __restrict__ err_flags, int cap, int freeze_on_softmax) {
    const int bh = blockIdx.x, tid = threadIdx.x;
    const int pos = chunk_pos[bh];
    const bool soft = mask_c[bh] != 0;
    const int n = cache_len[bh];
    if (soft && pos > 0) {
        const float dec = freeze_on_softmax ? 1.f : chunk_decay[bh];   // variant: the state as the chunk found it
        float4* S = reinterpret_cast<float4*>(state + (size_t)bh * D * D);
        const float4* S0 = reinterpret_cast<const float4*>(state_start + (size_t)bh * D * D);
        for (int i = tid; i < D * D / 4; i += DEC_THREADS) {
            const float4 x = S0[i];
            S[i] = make_float4(dec * x.x, dec * x.y, dec * x.z, dec * x.w);
        }
    }
    __syncthreads();   // every thread has read pos and n
    if (tid == 0) {
        if (soft) cache_len[bh] = min(n + pos, cap);
        if (err_flags != nullptr) err_flags[bh] = (soft && n + pos > cap) ? 1 : 0;
        chunk_pos[bh] = 0;
    }
}

// device pointers of one step; state_start, chunk_decay, chunk_pos with routing per chunk only, mask without it only
struct DecCall {
    float *state, *state_start, *chunk_decay;
    int32_t *chunk_pos;
    void *k_cache, *v_cache;
    int32_t* cache_len;
    const void *q, *k, *v;
    const float *alpha, *beta;
    const uint8_t* mask;
    const float *w_nla, *w_la;
    void* o;
    int32_t* err_flags;
    float scale, la_scale, eps;
};

template <typename T, int D, bool CHUNK>
static void launch_dec(const nats_dec_params& p, const DecCall& c, hipStream_t st) {
    const bool wide = p.B * p.H <= DEC_WIDE_PAIRS;
    auto kern = wide ? decode_wide_kernel<T, D, CHUNK> : decode_kernel<T, D, CHUNK>;
    hipLaunchKernelGGL(kern, dim3(p.B * p.H), dim3(wide ? DEC_WIDE : DEC_THREADS), 0, st, c.state, c.state_start, c.chunk_decay,
                       c.chunk_pos, (T*)c.k_cache, (T*)c.v_cache, c.cache_len, (const T*)c.q, (const T*)c.k, (const T*)c.v,
                       c.alpha, c.beta, c.mask, c.w_nla, c.w_la, (T*)c.o, c.err_flags, p.cap, c.scale, c.la_scale,
                       p.combine_mode, c.eps, p.linear_op, p.freeze_on_softmax, (const T*)p.q_nla, (const T*)p.k_nla);
}

static size_t split_bytes(const nats_dec_params& p, int rows) {
    const size_t n_split = ((size_t)p.cap + rows - 1) / rows;
    return (size_t)p.B * p.H * (n_split * (p.d + 4) + p.d) * sizeof(float);
}
size_t decode_split_workspace_bytes(const nats_dec_params& p) { return split_bytes(p, DSP_ROWS); }

// Cache rows per block: the smaller number where the workspace holds that many partial results.
static int split_rows(const nats_dec_params& p) {
    return p.workspace_bytes >= split_bytes(p, DSP_ROWS_SMALL) ? DSP_ROWS_SMALL : DSP_ROWS;
}

template <typename T, int D, bool CHUNK>
static void launch_dec_split(const nats_dec_params& p, const DecCall& c, float* ws, hipStream_t st) {
    const int rows = split_rows(p), n_split = (p.cap + rows - 1) / rows;
    {
        ProfScope ps("decode_split", st);
        auto kern = rows == DSP_ROWS_SMALL ? decode_split_kernel<T, D, CHUNK, DSP_ROWS_SMALL> : decode_split_kernel<T, D, CHUNK, DSP_ROWS>;
        hipLaunchKernelGGL(kern, dim3(D / DSP_SROWS + n_split, p.B * p.H), dim3(DEC_THREADS), 0, st, c.state, c.state_start,
                           c.chunk_pos, (const T*)c.k_cache, (const T*)c.v_cache, c.cache_len, (const T*)c.q, (const T*)c.k,
                           (const T*)c.v, c.alpha, c.beta, c.mask, ws, p.cap, n_split, c.scale, c.la_scale, p.linear_op,
                           p.freeze_on_softmax, (const T*)p.q_nla);
    }
    ProfScope ps("decode_combine", st);
    hipLaunchKernelGGL((decode_combine_kernel<T, D, CHUNK>), dim3(p.B * p.H), dim3(DEC_THREADS), 0, st, ws, c.chunk_decay, c.chunk_pos,
                       c.alpha, (T*)c.k_cache, (T*)c.v_cache, c.cache_len, (const T*)c.q, (const T*)c.k, (const T*)c.v,
                       c.mask, c.w_nla, c.w_la, (T*)c.o, c.err_flags, p.cap, n_split, rows, c.scale, p.combine_mode,
                       c.eps, (const T*)p.q_nla, (const T*)p.k_nla);
}

// ws: NULL, or decode_split_workspace_bytes(p) bytes (the step as blocks of equal size)
template <typename T, bool CHUNK>
static void launch_dec_d(const nats_dec_params& p, const DecCall& c, float* ws, hipStream_t st) {
    if (p.d == 64) ws != nullptr ? launch_dec_split<T, 64, CHUNK>(p, c, ws, st) : launch_dec<T, 64, CHUNK>(p, c, st);
    else ws != nullptr ? launch_dec_split<T, 128, CHUNK>(p, c, ws, st) : launch_dec<T, 128, CHUNK>(p, c, st);
}

nats_status launch_decode(const nats_dec_params& p, float softmax_scale, float la_scale, float eps,
                          float* state, void* k_cache, void* v_cache, int32_t* cache_len, const void* q,
                          const void* k, const void* v, const float* alpha, const float* beta,
                          const uint8_t* mask, const float* w_nla, const float* w_la, void* o,
                          int32_t* err_flags, float* ws, hipStream_t st) {
    const DecCall c{state, nullptr, nullptr, nullptr, k_cache, v_cache, cache_len, q, k, v, alpha, beta, mask, w_nla, w_la, o,
                    err_flags, softmax_scale, la_scale, eps};
    if (p.dtype == NATS_BF16) launch_dec_d<bf16_t, false>(p, c, ws, st);
    else launch_dec_d<float, false>(p, c, ws, st);
    return check_launch("decode");
}

nats_status launch_decode_chunk(const nats_dec_params& p, float softmax_scale, float la_scale, float eps,
                                float* state, float* state_start, float* chunk_decay, int32_t* chunk_pos,
                                void* k_cache, void* v_cache, int32_t* cache_len, const void* q, const void* k,
                                const void* v, const float* alpha, const float* beta, const float* w_nla,
                                const float* w_la, void* o, int32_t* err_flags, float* ws, hipStream_t st) {
    const DecCall c{state, state_start, chunk_decay, chunk_pos, k_cache, v_cache, cache_len, q, k, v, alpha, beta, nullptr,
                    w_nla, w_la, o, err_flags, softmax_scale, la_scale, eps};
    if (p.dtype == NATS_BF16) launch_dec_d<bf16_t, true>(p, c, ws, st);
    else launch_dec_d<float, true>(p, c, ws, st);
    return check_launch("decode (routing per chunk)");
}

nats_status launch_decode_commit(const nats_dec_params& p, float* state, const float* state_start,
                                 const float* chunk_decay, int32_t* chunk_pos, int32_t* cache_len,
                                 const uint8_t* mask_c, int32_t* err_flags, hipStream_t st) {
    dim3 grid(p.B * p.H);
    if (p.d == 64)
        hipLaunchKernelGGL(decode_commit_kernel<64>, grid, dim3(DEC_THREADS), 0, st, state, state_start, chunk_decay,
                           chunk_pos, cache_len, mask_c, err_flags, p.cap, p.freeze_on_softmax);
    else
        hipLaunchKernelGGL(decode_commit_kernel<128>, grid, dim3(DEC_THREADS), 0, st, state, state_start, chunk_decay,
                           chunk_pos, cache_len, mask_c, err_flags, p.cap, p.freeze_on_softmax);
    return check_launch("decode_commit");
}

}  // namespace nats
