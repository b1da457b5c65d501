// Backward of the linear branch by chunks of 64 tokens, to fp32 accuracy on matrix instructions (Section 4.2; the recurrence is
// Eq. 19 with the decay of Eq. 20, written for linear tokens only, Eq. 14).
//
// One chunk, with the state S0 [d_v][d_k] at its start, b' = beta (0 for a softmax token), gamma_r the product of the
// chunk's alphas up to token r, Gamma_ri = gamma_r / gamma_i, kd_i = gamma_C / gamma_i:
//     At = strict lower (Gamma . K K^T),  P = lower (Gamma . Q K^T),  T = (I + At diag(b'))^-1
//     R = V - diag(gamma) K S0^T,   Uh = T R  (= v_t - Sd k_t, the residual of Eq. 19: Uh = R - At U),   U = diag(b') Uh,
//     O = la (diag(gamma) Q S0^T + P U),   S1 = gamma_C S0 + U^T diag(kd) K.
// Given dO' = la dO and dS1 (from the chunks behind):
//     dU = P^T dO' + diag(kd) K dS1^T,   dR = T^T diag(b') dU = dV,
//     dbeta_r = Uh_r . (dU - At^T dR)_r = sum_i (P_ir (dO' Uh^T)_ir - At_ir (dR Uh^T)_ir) + kd_r K_r . (Uh dS1)_r
//     dS0 = gamma_C dS1 + dO'^T diag(gamma) Q - dR^T diag(gamma) K
//     dP = lower (dO' U^T),   dAt = - strict lower (dR U^T)
//     dQ = diag(gamma) dO' S0 + (dP . Gamma) K
//     dK = (dP . Gamma)^T Q + ((dAt . Gamma) + (dAt . Gamma)^T) K + diag(kd) U dS1 - diag(gamma) dR S0
//     d ln gamma_r = sum_i (dAt_ri At_ri + dP_ri P_ri) - sum_r' (dAt_r'r At_r'r + dP_r'r P_r'r)
//                    + gamma_r (Q_r . (dO' S0)_r - K_r . (dR S0)_r) - E_r,      E_i = kd_i K_i . (U dS1)_i
//     d ln gamma_C += sum_i E_i + gamma_C <dS1, S0>;     dalpha_t = (sum over r >= t of d ln gamma_r) / alpha_t.
// (The gated operation without the delta rule has At = 0, T = I, R = V: the terms that come from K S0^T drop.)
//
// Four kinds of kernel: the operands of every chunk (parallel over chunks), the states at the chunk starts (forwards
// along the sequence), the state gradients (backwards along it), and the gradients of every chunk from those
// (parallel over chunks).  Columns of V (rows of the state) never mix along the sequence, so the two sequential
// kernels split every (batch, head) into slices of 16 value columns, one or two per block.
//
// The operands' and the output's products run on v_mfma_f32_16x16x4_f32 through mac16 (sixteen contraction indices in four
// instructions), everything else on the bf16 instruction with operands as sums of bf16 terms (softmax_terms.h).
#include <type_traits>

#include "nats_common.h"
#include "scan_compact_block.h"
#include "softmax_terms.h"

namespace nats {

constexpr int CB_C = 64;          // chunk
constexpr int CB_MS = CB_C + 4;   // row stride (floats) of a 64 x 64 operand in LDS
constexpr int CB_NV = 16;         // value columns per slice of the sequential kernels

// per chunk: Tm, At, Pm [64][64] f32 row-major;  per token: gam, kd, bp;  per chunk: gamC;  for the gradients, per token:
// log2 of gamma as the sum of two floats, g2 and g2l
struct ChunkOps {
    float *Tm, *At, *Pm, *g2, *g2l, *gam, *kd, *bp, *gamC;
};

// a 16-byte word of T as it came from memory -> floats (8 for bf16, 4 for fp32)
__device__ __forceinline__ void unpack16(const u32x4 w, float (&out)[8], bf16_t) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        out[2 * q] = __uint_as_float(w[q] << 16);
        out[2 * q + 1] = __uint_as_float(w[q] & 0xffff0000u);
    }
}
__device__ __forceinline__ void unpack16(const u32x4 w, float (&out)[4], float) {
#pragma unroll
    for (int q = 0; q < 4; ++q) out[q] = __uint_as_float(w[q]);
}

// c + the product over 16 contraction indices, its four instructions from zero and added pairwise
__device__ __forceinline__ f32x4 add16(const float4 a, const float4 b, const f32x4 c) {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    const f32x4 x = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, zero, 0, 0, 0) + __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, zero, 0, 0, 0);
    const f32x4 y = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, zero, 0, 0, 0) + __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, zero, 0, 0, 0);
    return c + (x + y);
}

// x of the lane that the DPP control names (rows of the mask only; 0 where there is no source), both halves of a double
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_move_f64(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xF, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// ---- operands of a chunk ---------------------------------------------------------------------------------------------
// One block per (chunk, batch*head).  K K^T and Q K^T from the inputs as given: bf16 tensors on the bf16 instruction (one
// exact product per step, tiles of 17 KB: four blocks per CU; widened to fp32 in LDS, two blocks per CU, B 2, H 16,
// L 8192, d 128 took 129 us, now 75 with the scan), fp32 tensors on the fp32 one.  The inverse by 16 x 16 blocks: forward substitution
// on the diagonal, fp32 matrix instructions below it.
// The grid starts with the blocks of the mask scan and compaction (as a launch of their own these few, latency-bound
// blocks stood on the stream for 3 us at L 256, 6 at L 704, 14 at the size above).
template <typename T>
struct PrepArgs {
    const T *Q, *K;
    const float *alpha, *beta;
    const uint8_t* mask;
    ChunkOps o;
    int L, BH, freeze_on_softmax, linear_op, chunk_mask;
};
template <typename T, int D>
struct PrepLds {
    static constexpr bool bf16 = sizeof(T) == 2;
    static constexpr int KS = D + 4;                            // row stride of an fp32 tile
    static constexpr int M_BYTES = CB_C * CB_MS * 4;            // T and At diag(b') take the tiles' places
    static constexpr int TILE = bf16 ? TermTile<D, 1>::BYTES : CB_C * KS * 4;
    static constexpr int REGION = TILE > M_BYTES ? TILE : M_BYTES;
    static constexpr int bytes = 2 * REGION + CB_C * (8 + 4);
    static_assert(bytes >= SCAN_LDS_INTS * 4, "the scan's blocks use the same bytes");
};

// FWD: for the forward (o.At and the gradients' logarithms are not asked for)
template <typename T, int D, bool FWD>
__device__ __forceinline__ void gdn_bwd_prep_block(const PrepArgs<T>& a, const int block, unsigned char* lds) {
    using LY = PrepLds<T, D>;
    constexpr int KS = LY::KS, E = Vec16<T>::N, NP = CB_C * D / E / 256;
    const T* __restrict__ Q = a.Q;
    const T* __restrict__ K = a.K;
    const float* __restrict__ alpha = a.alpha;
    const float* __restrict__ beta = a.beta;
    const uint8_t* __restrict__ mask = a.mask;
    const ChunkOps& o = a.o;
    const int L = a.L, BH = a.BH, freeze_on_softmax = a.freeze_on_softmax, linear_op = a.linear_op, chunk_mask = a.chunk_mask;
    float* Ks = reinterpret_cast<float*>(lds);
    float* Qs = reinterpret_cast<float*>(lds + LY::REGION);
    const TermTile<D, 1> Kt{reinterpret_cast<uint16_t*>(lds)}, Qt{reinterpret_cast<uint16_t*>(lds + LY::REGION)};
    float* As = Qs;                         // after the products: At diag(b'), [64][CB_MS]
    // log2 gamma: its prefix sums in double, so that a decay ratio gamma_r / gamma_i, the exponential of a difference of
    // two of them, keeps fp32 accuracy whatever stands in front of token i in the chunk (alphas near 0)
    double* s_g = reinterpret_cast<double*>(lds + 2 * LY::REGION);
    float* s_bp = reinterpret_cast<float*>(s_g + CB_C);
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int n_chunks = L / CB_C;
    const int bh = block % BH, chunk = block / BH;
    const size_t gc = (size_t)bh * n_chunks + chunk, tok0 = (size_t)bh * L + (size_t)chunk * CB_C;
    if constexpr (LY::bf16) {
        u32x4 kr[NP], qr[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            kr[i] = reinterpret_cast<const u32x4*>(K + tok0 * D)[tid + 256 * i];
            qr[i] = reinterpret_cast<const u32x4*>(Q + tok0 * D)[tid + 256 * i];
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int e = tid + 256 * i, row = e / (D / E), c = (e % (D / E)) * E;
            const u32x4 k1[1] = {kr[i]}, q1[1] = {qr[i]};
            Kt.put(row, c, k1);
            Qt.put(row, c, q1);
        }
    } else {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int e = tid + 256 * i, row = e / (D / E), c = (e % (D / E)) * E;
            *reinterpret_cast<float4*>(Ks + row * KS + c) = ld4(reinterpret_cast<const float*>(K) + (tok0 + row) * D + c);
            *reinterpret_cast<float4*>(Qs + row * KS + c) = ld4(reinterpret_cast<const float*>(Q) + (tok0 + row) * D + c);
        }
    }
    if (w == 0) {
        // Routing per token: a softmax token writes nothing (b' = 0) and, in the variant without decay there, its
        // alpha counts as 1.  Routing per chunk (mask: one byte per chunk): every token writes inside its chunk, and
        // a softmax chunk hands on only (its decay) x (the state at its start): kd = 0, and the carried decay is 1
        // in the variant without decay (inside the chunk the decays still act on the provisional state).
        const bool soft = !chunk_mask && mask[tok0 + lane] != 0;
        const bool soft_chunk = chunk_mask && mask[gc] != 0;
        const float a = (freeze_on_softmax && soft) ? 1.f : alpha[tok0 + lane];
        // An alpha of (nearly) 0 counts as 1e-37.  In the forward one that is no decay at all, negative or NaN, makes NaN here
        // and so in the rows behind it: their head is then done token by token (gdn_chunk_out_kernel).
        const float ac = !FWD ? fmaxf(a, 1e-37f) : (a >= 0.f && a < 1e-37f) ? 1e-37f : a;
        double gd = (double)__builtin_amdgcn_logf(ac);   // log2; inclusive scan over the 64 lanes
        gd += dpp_move_f64<0x111, 0xF>(gd);
        gd += dpp_move_f64<0x112, 0xF>(gd);
        gd += dpp_move_f64<0x114, 0xF>(gd);
        gd += dpp_move_f64<0x118, 0xF>(gd);
        gd += dpp_move_f64<0x142, 0xA>(gd);
        gd += dpp_move_f64<0x143, 0xC>(gd);
        const uint64_t gu = __builtin_bit_cast(uint64_t, gd);
        const double gC = __builtin_bit_cast(double, ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(gu >> 32), 63) << 32) |
                                                         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)gu, 63));
        const float g = (float)gd, gam = __builtin_amdgcn_exp2f(g);
        const float bp = soft ? 0.f : beta[tok0 + lane];
        s_g[lane] = gd;
        s_bp[lane] = bp;
        if (!FWD) {
            o.g2[tok0 + lane] = g;
            o.g2l[tok0 + lane] = (float)(gd - (double)g);
        }
        o.gam[tok0 + lane] = gam;
        o.kd[tok0 + lane] = soft_chunk ? 0.f : __builtin_amdgcn_exp2f((float)(gC - gd));
        o.bp[tok0 + lane] = bp;
        if (lane == 63) o.gamC[gc] = (freeze_on_softmax && soft_chunk) ? 1.f : gam;
    }
    __syncthreads();
    // the 10 lower tiles (a, b), b <= a, of K K^T and Q K^T: tile t of the list to wavefront t % 4
    float* Ato = FWD ? nullptr : o.At + gc * (CB_C * CB_C);
    float* Pmo = o.Pm + gc * (CB_C * CB_C);
    float* Tmo = o.Tm + gc * (CB_C * CB_C);
    f32x4 keepA[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        const int t = w + 4 * s;   // uniform
        keepA[s] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (t < 10) {
            const int a = (0x3333222110 >> (4 * t)) & 15, b = (0x3210210100 >> (4 * t)) & 15;
            f32x4 accK = {0.f, 0.f, 0.f, 0.f}, accQ = {0.f, 0.f, 0.f, 0.f};
            if constexpr (LY::bf16) {
                // (steps of 32 columns from zero, added by vector adds, which round to nearest)
#pragma unroll
                for (int ks = 0; ks < D / 32; ++ks) {
                    u32x4 kb[1], ka[1], qa[1];
                    Kt.rows(16 * b + l16, 32 * ks + 8 * lq, kb);
                    Kt.rows(16 * a + l16, 32 * ks + 8 * lq, ka);
                    Qt.rows(16 * a + l16, 32 * ks + 8 * lq, qa);
                    accK += mfma_bf16(ka[0], kb[0], f32x4{0.f, 0.f, 0.f, 0.f});
                    accQ += mfma_bf16(qa[0], kb[0], f32x4{0.f, 0.f, 0.f, 0.f});
                }
            } else {
                // The forward adds the instructions' results up pairwise: with q . k and k . k as one running sum of D products
                // O_la was 2.0e-7 of its norm from 64 bits, now 1.14e-7 (token by token 1.07e-7; B 1, H 2, L 256, d 64: this
                // kernel 8.6 -> 10.9 us).  The backward pass keeps the running sum: behind Eq. 21 a row of O_la that is
                // nearly zero, its q . k by chance nearly zero, is divided by its norm, and whichever last bits it has are
                // the gradient's.
                f32x4 sumK[2] = {accK, accK}, sumQ[2] = {accQ, accQ};
#pragma unroll 4
                for (int kt = 0; kt < D / 16; ++kt) {
                    const float4 bk = ld4(Ks + (16 * b + l16) * KS + 16 * kt + 4 * lq);
                    const float4 ak = ld4(Ks + (16 * a + l16) * KS + 16 * kt + 4 * lq), aq = ld4(Qs + (16 * a + l16) * KS + 16 * kt + 4 * lq);
                    if constexpr (FWD) {
                        sumK[kt & 1] = add16(ak, bk, sumK[kt & 1]);
                        sumQ[kt & 1] = add16(aq, bk, sumQ[kt & 1]);
                    } else {
                        accK = mac16(ak, bk, accK);
                        accQ = mac16(aq, bk, accQ);
                    }
                }
                if constexpr (FWD) {
                    accK = sumK[0] + sumK[1];
                    accQ = sumQ[0] + sumQ[1];
                }
            }
            const int i = 16 * b + l16;
            const double gi = s_g[i];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = 16 * a + 4 * lq + j;
                const float G = __builtin_amdgcn_exp2f((float)(s_g[r] - gi));
                const float at = (i < r && linear_op == 0) ? G * accK[j] : 0.f;
                if (!FWD) Ato[r * CB_C + i] = at;
                Pmo[r * CB_C + i] = (i <= r) ? G * accQ[j] : 0.f;
                keepA[s][j] = at * s_bp[i];
            }
        }
    }
    // the 6 tiles above the diagonal are zeros (T's come out of the substitution below)
    for (int z = w; z < 6; z += 4) {
        const int a = (0x211000 >> (4 * z)) & 15, b = (0x332321 >> (4 * z)) & 15;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int off = (16 * a + 4 * lq + j) * CB_C + 16 * b + l16;
            if (!FWD) Ato[off] = 0.f;
            Pmo[off] = 0.f;
        }
    }
    __syncthreads();   // the Q tile is dead: its region takes At diag(b')
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        const int t = w + 4 * s;
        if (t < 10) {
            const int a = (0x3333222110 >> (4 * t)) & 15, b = (0x3210210100 >> (4 * t)) & 15;
#pragma unroll
            for (int j = 0; j < 4; ++j) As[(16 * a + 4 * lq + j) * CB_MS + 16 * b + l16] = keepA[s][j];
        }
    }
    __syncthreads();
    // T = (I + A)^-1, unit lower triangular, by 16 x 16 blocks (K's region, dead since the products, holds T).
    // (a) Diagonal blocks: wavefront b inverts I + A_bb by forward substitution, lane j < 16 owns column j:
    //     T[r][j] = [r == j] - sum over i < r of A[r][i] T[i][j]  (entries above the diagonal come out as exact zeros).
    float* Ts = Ks;   // [64][CB_MS]
    if (lane < 16) {
        const float* Ab = As + (16 * w) * CB_MS + 16 * w;
        float col[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float acc = 0.f;
#pragma unroll
            for (int i4 = 0; i4 < (r + 3) / 4; ++i4) {
                const float4 a4 = ld4(Ab + r * CB_MS + 4 * i4);
                acc += a4.x * col[4 * i4];
                if (4 * i4 + 1 < r) acc += a4.y * col[4 * i4 + 1];
                if (4 * i4 + 2 < r) acc += a4.z * col[4 * i4 + 2];
                if (4 * i4 + 3 < r) acc += a4.w * col[4 * i4 + 3];
            }
            col[r] = ((r == lane) ? 1.f : 0.f) - acc;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) Ts[(16 * w + r) * CB_MS + 16 * w + lane] = col[r];
    }
    __syncthreads();
    // (b) Blocks below the diagonal: T_ab = - T_aa sum over b <= k < a of A_ak T_kb.  Wavefront b owns block column b
    //     and walks down it; the sum's result tile is the right operand of the product with T_aa as it sits in
    //     registers.
    for (int ta = w + 1; ta < 4; ++ta) {
        f32x4 X = {0.f, 0.f, 0.f, 0.f};
        for (int k = w; k < ta; ++k)
            X = mac16(ld4(As + (16 * ta + l16) * CB_MS + 16 * k + 4 * lq), ld4col(Ts + (16 * k + 4 * lq) * CB_MS + 16 * w + l16, CB_MS), X);
        const f32x4 Y = mac16(ld4(Ts + (16 * ta + l16) * CB_MS + 16 * ta + 4 * lq), make_float4(X[0], X[1], X[2], X[3]),
                              f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
        for (int j = 0; j < 4; ++j) Ts[(16 * ta + 4 * lq + j) * CB_MS + 16 * w + l16] = -Y[j];
        __builtin_amdgcn_wave_barrier();   // LDS operations of one wavefront complete in order
    }
    __syncthreads();
    // (c) out, 16 bytes per thread and step; the tiles above the diagonal were never written: zeros
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e = tid + 256 * i, r = e / 16, c4 = (e % 16) * 4;
        float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
        if ((c4 >> 4) <= (r >> 4)) t = ld4(Ts + r * CB_MS + c4);
        *reinterpret_cast<float4*>(Tmo + r * CB_C + c4) = t;
    }
}

template <typename T, int D, bool FWD>
__global__ __launch_bounds__(256) void gdn_bwd_prep_kernel(const PrepArgs<T> a, const ScanArgs<T> sc, const int scan_segs,
                                                           const int scan_blocks) {
    static_assert(SCAN_THREADS == 256, "both kinds of block");
    extern __shared__ __align__(16) float cb_smem[];
    if ((int)blockIdx.x < scan_blocks) {
        scan_compact_block<T>(sc, blockIdx.x % scan_segs, blockIdx.x / scan_segs, reinterpret_cast<int*>(cb_smem));
        return;
    }
    gdn_bwd_prep_block<T, D, FWD>(a, blockIdx.x - scan_blocks, reinterpret_cast<unsigned char*>(cb_smem));
}

// ---- the states along the sequence -------------------------------------------------------------------------------------
// DIR 0: forwards, the state S^T [d_k][16] of a slice's 16 value columns; leaves S0 of every chunk (ck) and Uh.
// DIR 1: backwards, the gradient of that state; leaves dS1 of every chunk (ck), <dS1, S0>, dV and the gradient of the
// initial state.  Wavefront w owns the chunk's tokens 16 w .. 16 w + 15 in everything that is one
// row per token, and D / 64 of the state's 16 x 16 tiles.
template <typename T, typename TX>
struct SeqArgs {
    const T *K, *Q;
    const TX* X;                   // V (DIR 0) or dO (DIR 1; fp32 beside bf16 tensors behind a merge's adjoint), [BH][L][D]
    ChunkOps o;
    const float* S_init;           // DIR 0: [BH][D][D] or NULL
    float* ck;                     // [BH][L/64][D][D]
    float* rows;                   // [BH][L][D]: Uh (DIR 0), dV (DIR 1)
    const float* S0;               // DIR 1: the states forwards, laid out as ck
    float* dot;                    // DIR 1: <dS1, S0> of every chunk in parts, [BH][L/64][D/16][D/32]
    float* S_end;                  // [BH][D][D] or NULL.  DIR 0: the state after the last token; DIR 1: the gradient of S_init
    int L, BH;                     // BH: heads of V (output heads)
    int G;                         // head grouping: K, Q and the operands are those of linear head bh / G
    float la_scale;
    int delta;                     // 1: delta rule; 0: gated linear attention
};

// Eight wavefronts per slice (fp32 tensors: twelve): four compute (as above), four only move the next chunks' operands from global memory to LDS and cut
// them into bf16 terms (softmax_terms.h), the products' operands: bf16 tensors are one term, everything else three.  A
// burst of loads of this size keeps a wavefront at the issue of its memory instructions for about as long as a whole
// phase of the chunk's products takes, and there is one block per CU with nothing else to fill the time: so the
// wavefronts that multiply issue no global loads at all.
// A chunk is a chain of three products (K S^T, the inverse, the state's update) with a barrier behind each; what stands
// beside the chain (DIR 1: P^T dO', Q^T diag(gamma) dO') is multiplied in the first phase.  So most operands are dead
// for a part of the chunk and have one place in LDS, replaced there:
//     Q, P, dO (DIR 1)   behind the first barrier        T   behind the second
// K (first and third phase) and the per-token vectors have two places.  With fp32 tensors (three terms) K has one where
// two do not fit: it is replaced between the third barrier and a fourth; and in DIR 1 at d = 128 Q and K take turns in
// one place, and P and T, with the products beside the chain in a phase of their own.
// The loads of a chunk are asked for three chunks ahead (two at fp32 d = 128, for registers), into sets that take turns.
// What leaves the chain for other kernels: U is not stored (b' Uh where it is needed), dbeta and the residuals' part of it
// come from sums the gradient kernel has anyway, and the states are stored by the moving wavefronts, in whole rows, from
// the terms they lie in.  On fp32 instructions, with all of that in the chain, at B 2, H 16, L 8192, d 128 bf16: forwards
// 398 us (3.1 us per chunk), backwards 560; now 243 and 357.  Still a chain of latencies: 393 MB written and 100-300 MB
// read from HBM would take 100-140 us.
// With fp32 tensors, whose K and Q are cut into three terms too, eight wavefronts move for one slice: forwards / backwards in us with
// four -> eight, d 64: 6 heads, L 704 19.0 / 35.2 -> 17.9 / 30.4; 64 heads, L 2048 61 / 111 -> 60 / 104; d 128: 8 heads, L 2048
// 83.6 / 141 -> 69.7 / 115; 32 heads, L 2048 95 / 159 -> 89 / 144.  (bf16, 32 heads, L 8192, d 128: 243 / 362 -> 258 / 368.)
// NSL 2: two slices per block, with what they share (K, Q, T, P, the vectors) moved once, by all eight moving wavefronts, and two
// chains on every SIMD, each in the gaps of the other.  In DIR 1 P and T then take turns in one place (T, cut into terms
// beforehand, is written while K S^T is multiplied) and K has one.  A chunk takes 1.3 (DIR 0) and 1.45 times as long as with one slice,
// which pays where one slice per block makes a second round of blocks: see launch_seq_t.
template <typename T, typename TX, int D, int DIR, int NSL>
struct SeqLds {
    static constexpr int NT = terms_of<T>(), NX = DIR ? terms_of<TX>() : 1;
    // Rows of 64: 8 elements longer, not LDS_PAD = 16, but for fp32 tensors and for DIR 0 at d = 128.  16 -> 8 in us: d 64, 3 heads, L 5376
    // forwards 102 -> 96.5, backwards 156 -> 153.5; d 128, 48 heads, L 4096 backwards 262 -> 250; the others 243 -> 248 (32 heads,
    // L 8192, d 128 forwards), 18.0 -> 18.4 and 30.2 -> 30.9 (6 heads, L 704, d 64 fp32).
    static constexpr int P64 = NT > 1 || (DIR == 0 && D == 128) ? LDS_PAD : 8, PD = D == 64 ? P64 : LDS_PAD;
    using KTile = TermTile<D, NT, 64, PD>;                 // K; (DIR 1) Q
    using MTile = TermTile<64, N_TERMS, 64, P64>;          // T; (DIR 1) P
    using STile = TermTile<D, N_TERMS, CB_NV, PD>;         // the state
    using BTile = TermTile<64, N_TERMS, CB_NV, P64>;       // 16 value columns of a chunk's tokens
    using XTile = TermTile<64, NX, CB_NV, P64>;            // ... of dO as given
    static constexpr int V_BYTES = ((DIR ? 0 : NSL * CB_NV * CB_MS) + 256) * 4;   // gam, kd, bp [64], gamC; (DIR 0) V [16 v][CB_MS]
    static constexpr int n_b = DIR ? 3 : 2;           // DIR 0: R, kd U;  DIR 1: b' dU, -diag(gamma) dR, diag(gamma) dO'
    static constexpr bool turns = DIR == 1 && NT > 1 && D == 128;
    static constexpr bool m_one = turns || (DIR == 1 && NSL > 1);
    static constexpr int fixed = (DIR && !m_one ? 2 : 1) * MTile::BYTES + 2 * V_BYTES + NSL * (STile::BYTES + n_b * BTile::BYTES) +
                                 (DIR ? (turns ? 0 : KTile::BYTES) + NSL * XTile::BYTES : 0);
    static constexpr bool k_one = turns || fixed + 2 * KTile::BYTES > 160 * 1024;
    static constexpr int o_k = 0;
    static constexpr int o_m1 = o_k + (k_one ? 1 : 2) * KTile::BYTES;
    static constexpr int o_m2 = DIR && !m_one ? o_m1 + MTile::BYTES : o_m1;
    static constexpr int o_v = o_m2 + MTile::BYTES;
    static constexpr int o_s = o_v + 2 * V_BYTES;
    static constexpr int o_b = o_s + NSL * STile::BYTES;
    static constexpr int o_x = o_b + NSL * n_b * BTile::BYTES;
    static constexpr int o_q = turns ? o_k : o_x + NSL * XTile::BYTES;
    static constexpr int bytes = o_k + fixed + (k_one ? 1 : 2) * KTile::BYTES;
    static constexpr int move = NSL > 1 || NT > 1 ? 512 : 256;   // threads that move
    static constexpr int sets = (NT > 1 && D == 128) || (DIR == 1 && NSL > 1) ? 1 : 2;
};

template <typename T, typename TX, int D, int DIR, int NSL>
__global__ __launch_bounds__((256 * NSL + SeqLds<T, TX, D, DIR, NSL>::move)) void gdn_chunk_seq_kernel(const SeqArgs<T, TX> a) {
    using LY = SeqLds<T, TX, D, DIR, NSL>;
    constexpr int NT = LY::NT, NX = LY::NX, KT = D / 64, MS = CB_MS, NS = LY::sets;
    constexpr int LT = LY::move, NPC = 64 * D / 8 / LT, NPM = 64 * 64 / 8 / LT;   // threads that move; 8-element pieces of K and of T per thread
    extern __shared__ __align__(16) float cb_smem[];
    unsigned char* lds = reinterpret_cast<unsigned char*>(cb_smem);
    auto at = [&](int off) { return reinterpret_cast<uint16_t*>(lds + off); };
    auto Kt = [&](int i) { return typename LY::KTile{at(LY::o_k + (LY::k_one ? 0 : i) * LY::KTile::BYTES)}; };
    const typename LY::MTile Tt{at(LY::o_m1)}, Pt{at(LY::o_m2)};
    auto Gf = [&](int i) { return reinterpret_cast<float*>(lds + LY::o_v + i * LY::V_BYTES); };   // gam, kd, bp, gamC
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool loader = wave >= 4 * NSL;
    const int w = wave & 3, lt = (LT > 256 * NSL ? tid - 256 * NSL : tid) & (LT - 1), sl = NSL > 1 ? (wave >> 2) & (NSL - 1) : 0;   // sl: the wavefront's slice
    const int l16 = lane & 15, lq = lane >> 4;
    const int bh = blockIdx.x % a.BH, slice = NSL * (blockIdx.x / a.BH) + sl, v0 = CB_NV * slice;
    auto Xf = [&](int i) { return Gf(i) + 256 + sl * CB_NV * MS; };                               // DIR 0: V [16 v][MS]
    const typename LY::STile St{at(LY::o_s + sl * LY::STile::BYTES)};
    auto Bt = [&](int i) { return typename LY::BTile{at(LY::o_b + (sl * LY::n_b + i) * LY::BTile::BYTES)}; };
    const typename LY::BTile B0 = Bt(0), B1 = Bt(1), B2 = Bt(2);
    const typename LY::KTile Qt{at(LY::o_q)};                              // DIR 1
    const typename LY::XTile Xt{at(LY::o_x + sl * LY::XTile::BYTES)};      // DIR 1
    const int lin = bh / a.G;   // linear head
    const int L = a.L, n_chunks = L / CB_C;
    const float delta = a.delta ? 1.f : 0.f;

    // The two kinds of wavefront run loops of their own with the same number of barriers (a barrier counts
    // arrivals, wherever in the code they come from): what one kind keeps in registers across a chunk then takes
    // no registers from the other.
    if (loader) {
        struct Set {
            Raw8<T> k[NPC], q[DIR ? NPC : 1];
            Raw8<float> m1[NPM], m2[DIR ? NPM : 1];
            float4 gate4, g4;
            TX x[4];
            float gC;
        } set[NS];
        // chunk number i of the walk; past the end: the last one once more (loads and writes stay unconditional: around
        // a branch the compiler waits for every load in flight).  As it comes from memory: a conversion here would wait.
        auto chunk_at = [&](int i) { i = i < n_chunks ? i : n_chunks - 1; return DIR ? n_chunks - 1 - i : i; };
        auto fetch_k = [&](Set& s, int i) {
            const size_t tok0 = (size_t)lin * L + (size_t)chunk_at(i) * CB_C;
#pragma unroll
            for (int p = 0; p < NPC; ++p) s.k[p].load(a.K + tok0 * D + 8 * (lt + LT * p));   // a chunk's rows are contiguous
        };
        auto fetch_m = [&](Raw8<float> (&m)[NPM], const float* M, int i) {
            M += ((size_t)lin * n_chunks + chunk_at(i)) * (CB_C * CB_C);
#pragma unroll
            for (int p = 0; p < NPM; ++p) m[p].load(M + 8 * (lt + LT * p));
        };
        auto fetch = [&](Set& s, int i) {   // all but K where it has one place and T where it takes turns
            const int c = chunk_at(i);
            const size_t gc = (size_t)lin * n_chunks + c, tok0 = (size_t)lin * L + (size_t)c * CB_C;
            if (!LY::k_one) fetch_k(s, i);
            if (DIR) {
#pragma unroll
                for (int p = 0; p < NPC; ++p) s.q[p].load(a.Q + tok0 * D + 8 * (lt + LT * p));
            }
            if (lt < 48) s.gate4 = ld4((lt < 16 ? a.o.gam : lt < 32 ? a.o.kd : a.o.bp) + tok0 + 4 * (lt & 15));
            if (lt == 48) s.gC = a.o.gamC[gc];
            if (DIR) s.g4 = ld4(a.o.gam + tok0 + 16 * w + 4 * lq);
            const size_t t4 = (size_t)bh * L + (size_t)c * CB_C + 16 * w + 4 * lq;
#pragma unroll
            for (int j = 0; j < 4; ++j) s.x[j] = a.X[(t4 + j) * D + v0 + l16];
            if constexpr (DIR) fetch_m(s.m2, a.o.Pm, i);
            if (!LY::m_one) fetch_m(s.m1, a.o.Tm, i);
        };
        auto put_k = [&](const typename LY::KTile& dst, const auto& r) {
#pragma unroll
            for (int p = 0; p < NPC; ++p) {
                const int e = 8 * (lt + LT * p);
                u32x4 t[NT];
                r[p].terms(t);
                dst.put(e / D, e % D, t);
            }
        };
        auto put_m = [&](const typename LY::MTile& dst, const auto& r) {
#pragma unroll
            for (int p = 0; p < NPM; ++p) {
                const int e = 8 * (lt + LT * p);
                u32x4 t[N_TERMS];
                r[p].terms(t);
                dst.put(e / 64, e % 64, t);
            }
        };
        const int ls = lt & 255, sv = ls / (D / 8), sk = 8 * (ls % (D / 8));
        const bool half = LT > 256 * NSL && wave >= 8;   // twice the wavefronts per slice: half of them store the state, the others cut X
        const bool has_state = !half && ls < CB_NV * D / 8, has_x = LT == 256 * NSL || half;   // uniform
        auto put_vectors = [&](const Set& s, int nb) {
            float* Gt = Gf(nb);
            if (lt < 48) *reinterpret_cast<float4*>(Gt + 4 * lt) = s.gate4;
            if (lt == 48) Gt[3 * CB_C] = s.gC;
            if (DIR == 0 && has_x)
                *reinterpret_cast<float4*>(Xf(nb) + l16 * MS + 16 * w + 4 * lq) =
                    make_float4(to_float(s.x[0]), to_float(s.x[1]), to_float(s.x[2]), to_float(s.x[3]));
        };
        // the state of chunk ci, in whole rows: 8 columns per thread, put together from their terms
        auto state_at = [&](int i) { return (((size_t)bh * n_chunks + chunk_at(i)) * D + v0 + (has_state ? sv : 0)) * D + sk; };
        Raw8<float> s0[DIR ? NS : 1];                // DIR 1: the same elements of S0
        auto store_state = [&](const Raw8<float>& s0r, int ci) {
            if (!has_state) return;
            u32x4 t[N_TERMS];
            St.rows(sv, sk, t);
            float x[8], dot = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                x[i] = 0.f;
#pragma unroll
                for (int n = N_TERMS - 1; n >= 0; --n)   // exact: the terms of one number
                    x[i] += __uint_as_float(i & 1 ? t[n][i / 2] & 0xffff0000u : t[n][i / 2] << 16);
                if (DIR) dot += x[i] * __uint_as_float(s0r.w[i / 4][i % 4]);
            }
            float* dst = a.ck + state_at(ci);
            *reinterpret_cast<float4*>(dst) = make_float4(x[0], x[1], x[2], x[3]);
            *reinterpret_cast<float4*>(dst + 4) = make_float4(x[4], x[5], x[6], x[7]);
            if (DIR) {
                dot = lane_group_sum<64>(dot);
                if (lane == 0)
                    a.dot[(((size_t)bh * n_chunks + chunk_at(ci)) * (D / CB_NV) + slice) * (D / 32) + w] = dot;
            }
        };
        auto put_first = [&](const Set& s) {   // DIR 1: what the first phase alone reads
            if (!LY::turns) put_k(Qt, s.q);
            if (!has_x) return;
            const float gg[4] = {s.g4.x, s.g4.y, s.g4.z, s.g4.w};
            float x[4], y[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                x[j] = to_float(s.x[j]);
                y[j] = gg[j] * (a.la_scale * x[j]);
            }
            uint2 t[N_TERMS];
            split_terms(y, t);
            B2.put(l16, 16 * w + 4 * lq, t);
            split_terms(x, t);
            uint2 tx[NX];
#pragma unroll
            for (int i = 0; i < NX; ++i) tx[i] = t[i];
            Xt.put(l16, 16 * w + 4 * lq, tx);
        };
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            fetch(set[i], i);
            if (LY::k_one) fetch_k(set[i], i);
            if (LY::m_one) fetch_m(set[i].m1, a.o.Tm, i);
            if constexpr (DIR == 1) s0[i].load(a.S0 + state_at(i));
        }
        put_k(LY::turns ? Qt : Kt(0), LY::turns ? set[0].q : set[0].k);
        put_vectors(set[0], 0);
        if constexpr (DIR == 1) {
            put_first(set[0]);
            put_m(Pt, set[0].m2);
        }
        if (!LY::m_one) put_m(Tt, set[0].m1);
        fetch(set[0], NS);
        if (LY::k_one && !LY::turns) fetch_k(set[0], NS);
        __syncthreads();
        auto step = [&](auto which, int ci) {   // chunk ci is multiplied, chunk ci + 1 written, chunk ci + 1 + NS asked for
            constexpr int S = decltype(which)::value;
            Set& s = set[S];
            const int nb = (ci + 1) & 1;
            if constexpr (DIR == 1) {
                constexpr int Z = (S + NS - 1) % NS;   // chunk ci
                store_state(s0[Z], ci);
                s0[Z].load(a.S0 + state_at(ci + NS));
            } else {
                store_state(s0[0], ci);
            }
            u32x4 tm[LY::m_one && !LY::turns ? NPM : 1][N_TERMS];
            if constexpr (LY::m_one && !LY::turns) {   // chunk ci's T, cut here so that only its writes stand between two barriers
                auto& m = set[(S + NS - 1) % NS].m1;
#pragma unroll
                for (int p = 0; p < NPM; ++p) m[p].terms(tm[p]);
                fetch_m(m, a.o.Tm, ci + NS);
            }
            __syncthreads();
            if constexpr (LY::m_one && !LY::turns) {   // in P's place
#pragma unroll
                for (int p = 0; p < NPM; ++p) {
                    const int e = 8 * (lt + LT * p);
                    Tt.put(e / 64, e % 64, tm[p]);
                }
                __syncthreads();
            }
            if (LY::turns) {   // chunk ci's K in Q's place, T in P's
                put_k(Kt(0), s.k);
                put_m(Tt, s.m1);
                fetch_k(s, ci + 1);
                fetch_m(s.m1, a.o.Tm, ci + 1);
                __syncthreads();
            }
            if constexpr (DIR == 1) put_first(s);
            put_vectors(s, nb);
            if (!LY::k_one) put_k(Kt(nb), s.k);
            if constexpr (DIR == 1 && !LY::m_one) put_m(Pt, s.m2);
            __syncthreads();
            if (LY::turns) __syncthreads();
            if constexpr (LY::m_one) put_m(Pt, s.m2);
            else put_m(Tt, s.m1);
            if (!LY::turns) fetch(s, ci + 1 + NS);
            __syncthreads();
            if constexpr (LY::turns) {
                put_k(Qt, s.q);
                fetch(s, ci + 1 + NS);
                __syncthreads();
            } else if (LY::k_one) {
                put_k(Kt(0), s.k);
                fetch_k(s, ci + 1 + NS);
                __syncthreads();
            }
        };
        for (int ci = 0; ci < n_chunks; ci += NS) {
            step(std::integral_constant<int, NS - 1>{}, ci);   // chunk ci + 1 is in set (ci + 1) % NS
            if (NS == 2 && ci + 1 < n_chunks) step(std::integral_constant<int, 0>{}, ci + 1);
        }
        return;
    }

    // the state: tiles kt = KT w + t, element [k = 16 kt + 4 lq + j][v = l16]
    f32x4 Sacc[KT];
    auto put_state = [&](int t) {
        const float x[4] = {Sacc[t][0], Sacc[t][1], Sacc[t][2], Sacc[t][3]};
        uint2 y[N_TERMS];
        split_terms(x, y);
        St.put(l16, 16 * (KT * w + t) + 4 * lq, y);
    };
#pragma unroll
    for (int t = 0; t < KT; ++t) {
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
        if (DIR == 0 && a.S_init != nullptr) s = ld4(a.S_init + ((size_t)bh * D + v0 + l16) * D + 16 * (KT * w + t) + 4 * lq);
        Sacc[t] = f32x4{s.x, s.y, s.z, s.w};
        put_state(t);
    }
    auto put_b = [&](const typename LY::BTile& dst, const float (&x)[4]) {   // this lane's four tokens of its value column
        uint2 t[N_TERMS];
        split_terms(x, t);
        dst.put(l16, 16 * w + 4 * lq, t);
    };
    __syncthreads();

    for (int ci = 0; ci < n_chunks; ++ci) {
        const int c = DIR ? n_chunks - 1 - ci : ci, cb = ci & 1;
        const size_t t4 = (size_t)bh * L + (size_t)c * CB_C + 16 * w + 4 * lq;   // the lane's first token
        const typename LY::KTile Ks = Kt(cb);
        const float* Gt = Gf(cb);
        float gg[4], kk[4], bb[4], xv[4];
        {
            const float4 g4 = ld4(Gt + 16 * w + 4 * lq), kd4 = ld4(Gt + CB_C + 16 * w + 4 * lq);
            const float4 bp4 = ld4(Gt + 2 * CB_C + 16 * w + 4 * lq), x4 = DIR ? g4 : ld4(Xf(cb) + l16 * MS + 16 * w + 4 * lq);
            gg[0] = g4.x; gg[1] = g4.y; gg[2] = g4.z; gg[3] = g4.w;
            kk[0] = kd4.x; kk[1] = kd4.y; kk[2] = kd4.z; kk[3] = kd4.w;
            bb[0] = bp4.x; bb[1] = bp4.y; bb[2] = bp4.z; bb[3] = bp4.w;
            xv[0] = x4.x; xv[1] = x4.y; xv[2] = x4.z; xv[3] = x4.w;
        }
        const float gC = Gt[3 * CB_C];
        f32x4 upd[KT];   // what the chunk adds to the state
#pragma unroll
        for (int t = 0; t < KT; ++t) upd[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        // DIR 1, beside the chain: P^T dO' (rows of P behind the wavefront's tokens), Q^T diag(gamma) dO'
        f32x4 accP = {0.f, 0.f, 0.f, 0.f};
        auto beside = [&]() {
            for (int ks = w >> 1; ks < 2; ++ks) {
                u32x4 p[N_TERMS], x[NX];
                Pt.cols_in_order(32 * ks, 16 * w, l16, lq, p);
                Xt.rows(l16, 32 * ks + 8 * lq, x);
                accP = mfma_terms(p, x, accP);
            }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                u32x4 b[N_TERMS];
                B2.rows(l16, 32 * ks + 8 * lq, b);
#pragma unroll
                for (int t = 0; t < KT; ++t) {
                    u32x4 q[NT];
                    Qt.cols_in_order(32 * ks, 16 * (KT * w + t), l16, lq, q);
                    upd[t] = mfma_terms(q, b, upd[t]);
                }
            }
        };
        if (LY::turns) {
            beside();
            __syncthreads();
            __syncthreads();   // K and T take Q's and P's places
        } else if (LY::m_one) {
            beside();
            __syncthreads();   // T takes P's place
        }
        // ---- 1: the state seen by the wavefront's tokens: K_w S^T --------------------------------------------
        {
            f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
#pragma unroll
            for (int ks = 0; ks < D / 32; ++ks) {
                u32x4 k[NT], s[N_TERMS];
                Ks.rows(16 * w + l16, 32 * ks + 8 * lq, k);
                St.rows(l16, 32 * ks + 8 * lq, s);
                if (ks & 1) acc1 = mfma_terms(k, s, acc1);
                else acc0 = mfma_terms(k, s, acc0);
            }
            acc0 += acc1;
            float y[4];
            if (DIR == 0) {
#pragma unroll
                for (int j = 0; j < 4; ++j) y[j] = xv[j] - delta * gg[j] * acc0[j];
            } else {   // dU = P^T dO' + diag(kd) K dS1^T
                if (!LY::m_one) beside();
#pragma unroll
                for (int j = 0; j < 4; ++j) y[j] = bb[j] * (kk[j] * acc0[j] + a.la_scale * accP[j]);
            }
            put_b(B0, y);
        }
        __syncthreads();
        // ---- 2: through the inverse ------------------------------------------------------------------------
        {
            f32x4 X = {0.f, 0.f, 0.f, 0.f};   // Uh (DIR 0), dR (DIR 1)
            auto half = [&](int ks) {         // 32 tokens of the contraction
                u32x4 m[N_TERMS], b[N_TERMS];
                if (DIR == 0) Tt.rows(16 * w + l16, 32 * ks + 8 * lq, m);
                else Tt.cols_in_order(32 * ks, 16 * w, l16, lq, m);
                B0.rows(l16, 32 * ks + 8 * lq, b);
                X = mfma_terms(m, b, X);
            };
            if (DIR == 0 || w < 2) half(0);   // T is lower triangular; uniform
            if (DIR == 1 || w >= 2) half(1);
            float y[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) y[j] = DIR == 0 ? kk[j] * (bb[j] * X[j]) : -delta * gg[j] * X[j];
            put_b(B1, y);
#pragma unroll
            for (int j = 0; j < 4; ++j) a.rows[(t4 + j) * D + v0 + l16] = X[j];
        }
        __syncthreads();
        // ---- 3: the chunk's contribution to the state ------------------------------------------------------------
        // (summed from zero and added by vector adds: the matrix instruction's own accumulation does not round to nearest)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {   // token tiles outside: their operands serve all of the wavefront's state tiles
            u32x4 b[N_TERMS];
            B1.rows(l16, 32 * ks + 8 * lq, b);
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                u32x4 k[NT];
                Ks.cols_in_order(32 * ks, 16 * (KT * w + t), l16, lq, k);
                upd[t] = mfma_terms(k, b, upd[t]);
            }
        }
        // the state for the next chunk's first phase (nothing reads it in between)
#pragma unroll
        for (int t = 0; t < KT; ++t) {
#pragma unroll
            for (int j = 0; j < 4; ++j) Sacc[t][j] = fmaf(gC, Sacc[t][j], upd[t][j]);
            put_state(t);
        }
        __syncthreads();   // every read of the chunk's operands is done, the new state is in place
        if (LY::k_one) __syncthreads();   // K is replaced in between
    }
    if (a.S_end != nullptr) {
#pragma unroll
        for (int t = 0; t < KT; ++t)
            *reinterpret_cast<float4*>(a.S_end + ((size_t)bh * D + v0 + l16) * D + 16 * (KT * w + t) + 4 * lq) =
                make_float4(Sacc[t][0], Sacc[t][1], Sacc[t][2], Sacc[t][3]);
    }
}

__device__ __forceinline__ void store_rounded(bf16_t* p, const float (&x)[2]) { *reinterpret_cast<uint32_t*>(p) = pack_bf16x2(x[0], x[1]); }
__device__ __forceinline__ void store_rounded(bf16_t* p, const float (&x)[1]) { p->bits = (uint16_t)pack_bf16x2(x[0], 0.f); }

// ---- the gradients of a chunk -------------------------------------------------------------------------------------------
// One block per (chunk, batch*head), 4 wavefronts; wavefront w owns a quarter of the columns of dQ and dK (all 64 rows)
// and of the three products with the states that feed them.  Every element of S0 and dS1 is then the operand of one
// wavefront alone and goes from memory to its registers; what all read (dO, dR, Uh in turn; then K, Q and the two
// 64 x 64 operands) goes through LDS.  At d = 128 a lane's two columns are neighbours (8-byte loads and stores, whole
// lines per 16 lanes): column 32 w + 2 l16 + ct; K and Q lie in LDS in that order.
// All products on bf16 terms (softmax_terms.h).  On the fp32 instruction they took as long as the bytes (1.5 GB at
// B 2, H 16, L 8192, d 128), one behind the other with one block of 139 KB of LDS per CU: 555 us; with two blocks per CU
// and the terms 377, 1.0 GB at 2.7 TB/s.  Sums over rows,
// columns or wavefronts go through small per-tile or per-wavefront arrays that one wavefront adds up in a fixed order.
template <typename T, typename TO>
struct GradArgs {
    const T *Q, *K;
    const TO* dO;
    ChunkOps o;
    const float *alpha;
    const uint8_t* mask;
    const float *ck, *dck, *Uh, *dR, *dot;
    float *dQ, *dK, *dalpha, *dbeta, *g_nla;
    float* dscore_la;   // optional, routing per chunk: Eq. 17 per chunk
    bf16_t *dQb, *dKb, *dVb;   // ROUNDED: the results rounded to bf16 instead (dKb, dVb optional; dQ then holds the softmax branch's share)
    int L, BH, G;       // BH: output heads; the G of a group share Q, K, alpha, the mask and the operands
    float la_scale;
    int delta, freeze_on_softmax, chunk_mask;
};

template <typename T, typename TO, int D>
struct GradLds {
    using RTile = TermTile<D, N_TERMS>;      // dO, dR, Uh, in turn
    using KTile = TermTile<D, terms_of<T>()>;
    static constexpr int o_q = KTile::BYTES, o_p = 2 * KTile::BYTES, o_a = o_p + CB_C * CB_MS * 4;
    static constexpr int last = o_a + CB_C * CB_MS * 4;
    static constexpr int first = RTile::BYTES + (terms_of<TO>() == 1 ? TermTile<D, 1>::BYTES : 0);
    static constexpr int o_small = first > last ? first : last;
    static constexpr int bytes = o_small + (5 + 8 + 8) * CB_C * 4 + 4 * 4;
    static constexpr int blocks = 2 * bytes <= 160 * 1024 ? 2 : 1;   // per CU
};

// ROUNDED: dQ (and, where nothing is added to them later but whole rows, dK and dV) go out as bf16, for a caller whose tensors are:
// a cast behind the pass reads the fp32 gradient once more and writes it a second time (three of 134 MB at the size
// above: 109 us).
template <typename T, typename TO, int D, bool ROUNDED>
__global__ __launch_bounds__(256, (GradLds<T, TO, D>::blocks)) void gdn_chunk_grads_kernel(const GradArgs<T, TO> a) {
    using LY = GradLds<T, TO, D>;
    constexpr int NT = terms_of<T>(), NO = terms_of<TO>(), NCT = D / 64, KS = D / 32, MS = CB_MS, NPC = D / 32;
    constexpr int NTL = 3;   // lower 16 x 16 tiles of a 64 x 64 operand per wavefront
    extern __shared__ __align__(16) float cb_smem[];
    unsigned char* lds = reinterpret_cast<unsigned char*>(cb_smem);
    const typename LY::RTile Rt{reinterpret_cast<uint16_t*>(lds)};
    const TermTile<D, NO> Ot{reinterpret_cast<uint16_t*>(lds + (NO == 1 ? LY::RTile::BYTES : 0))};
    const typename LY::KTile Kt{reinterpret_cast<uint16_t*>(lds)}, Qt{reinterpret_cast<uint16_t*>(lds + LY::o_q)};
    float* Pf = reinterpret_cast<float*>(lds + LY::o_p);       // dP . Gamma
    float* Af = reinterpret_cast<float*>(lds + LY::o_a);       // (dAt . Gamma) + (dAt . Gamma)^T
    float* s_g2 = reinterpret_cast<float*>(lds + LY::o_small);
    float* s_gam = s_g2 + CB_C;
    float* s_kd = s_gam + CB_C;
    float* s_bp = s_kd + CB_C;
    float* s_g2l = s_bp + CB_C;
    float* rs = s_g2l + CB_C;                  // [4 column tiles][64 rows]: row sums of dAt . At + dP . P per tile
    float* cs = rs + 4 * CB_C;                 // [4 row tiles][64 columns]: column sums of the same without the factor b'
    float* gk = cs + 4 * CB_C;                 // [4 wavefronts][64]: the state terms of d ln gamma, per wavefront's columns
    float* gu = gk + 4 * CB_C;                 // ...: kd K . (Uh dS1), likewise
    float* ge = gu + 4 * CB_C;                 // [4]: the sum of E_r over the chunk, likewise
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int n_chunks = a.L / CB_C;
    const int bh = blockIdx.x % a.BH, chunk = blockIdx.x / a.BH;
    const size_t gc = (size_t)bh * n_chunks + chunk, tok0 = (size_t)bh * a.L + (size_t)chunk * CB_C;
    const size_t gcl = (size_t)(bh / a.G) * n_chunks + chunk, tokl = (size_t)(bh / a.G) * a.L + (size_t)chunk * CB_C;
    const float delta = a.delta ? 1.f : 0.f;
    const int col0 = 16 * NCT * w + NCT * l16;   // the lane's NCT columns

    using Strip = float[KS][8][NCT];             // rows 32 ks + 8 lq + i of the lane's columns of a state
    auto load_strip = [&](float (&s)[8][NCT], const float* S, int ks) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float* p = S + (size_t)(32 * ks + 8 * lq + i) * D + col0;
            if constexpr (NCT == 2) {
                const float2 x = *reinterpret_cast<const float2*>(p);
                s[i][0] = x.x;
                s[i][1] = x.y;
            } else {
                s[i][0] = p[0];
            }
        }
    };
    auto strip_terms = [&](const float (&s)[8][NCT], u32x4 (&t)[NCT][N_TERMS]) {
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
            float x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = s[i][ct];
            split_terms(x, t[ct]);
        }
    };
    auto put_rows = [&](const auto& dst, const auto& r) {   // [64][D] -> terms
#pragma unroll
        for (int p = 0; p < NPC; ++p) {
            const int e = 8 * (tid + 256 * p);
            std::remove_const_t<std::remove_reference_t<decltype(r[0])>> x = r[p];
            typename std::remove_const_t<std::remove_reference_t<decltype(dst)>>::Terms t;
            x.terms(t);
            dst.put(e / D, e % D, t);
        }
    };
    const float* S0g = a.ck + gc * ((size_t)D * D);
    const float* dS1g = a.dck + gc * ((size_t)D * D);
    Strip S0;
    Raw8<TO> dOr[NPC];
    Raw8<float> Rr[NPC];
    // one of g2, gam, kd, b' of the chunk's tokens
    const float gate_in = (w == 0 ? a.o.g2 : w == 1 ? a.o.gam : w == 2 ? a.o.kd : a.o.bp)[tokl + lane];
    const float g2l_in = w == 0 ? a.o.g2l[tokl + lane] : 0.f;
#pragma unroll
    for (int p = 0; p < NPC; ++p) dOr[p].load(a.dO + tok0 * D + 8 * (tid + 256 * p));
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) load_strip(S0[ks], S0g, ks);
#pragma unroll
    for (int p = 0; p < NPC; ++p) Rr[p].load(a.dR + tok0 * D + 8 * (tid + 256 * p));
    // ---- stage 1: dO S0 and dR S0, with dO and dR in LDS together where dO is one term ------------------------------
    constexpr bool together = NO == 1;
    put_rows(Ot, dOr);
    if (ROUNDED && a.dVb != nullptr) {   // dV = dR
#pragma unroll
        for (int p = 0; p < NPC; ++p) {
            float x[8];
            Rr[p].floats(x);
            Vec16<bf16_t>::store(a.dVb + tok0 * D + 8 * (tid + 256 * p), x);
        }
    }
    if (together) put_rows(Rt, Rr);
    s_g2[tid] = gate_in;   // s_g2, s_gam, s_kd, s_bp lie one behind the other
    if (w == 0) s_g2l[lane] = g2l_in;
    for (int e = tid; e < 8 * CB_C; e += 256) rs[e] = 0.f;   // rs and cs
    __syncthreads();
    f32x4 Gdq[4][NCT], Gdk[4][NCT], Gu[4][NCT];
    auto clear = [&](f32x4 (&G)[4][NCT]) {
#pragma unroll
        for (int ta = 0; ta < 4; ++ta)
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) G[ta][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto add_product = [&](const auto& X, const u32x4 (&b)[NCT][N_TERMS], int ks, f32x4 (&G)[4][NCT]) {
#pragma unroll
        for (int ta = 0; ta < 4; ++ta) {
            typename std::remove_const_t<std::remove_reference_t<decltype(X)>>::Terms x;
            X.rows(16 * ta + l16, 32 * ks + 8 * lq, x);
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) G[ta][ct] = mfma_terms(x, b[ct], G[ta][ct]);
        }
    };
    // (the scheduling barriers keep the reads and the splitting of later steps from being drawn forward: ahead of their
    // place they cost registers that are not there)
    clear(Gdq);
    if (together) clear(Gdk);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        u32x4 b[NCT][N_TERMS];
        strip_terms(S0[ks], b);
        add_product(Ot, b, ks, Gdq);
        if (together) add_product(Rt, b, ks, Gdk);
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    if (!together) {
        put_rows(Rt, Rr);
        __syncthreads();
        clear(Gdk);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            u32x4 b[NCT][N_TERMS];
            strip_terms(S0[ks], b);
            add_product(Rt, b, ks, Gdk);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
    }
    // ---- stage 2: Uh dS1; dP and dAt, whose left operands (one tile of 16 rows each) come from memory -----------------
#pragma unroll
    for (int p = 0; p < NPC; ++p) Rr[p].load(a.Uh + tok0 * D + 8 * (tid + 256 * p));
    Strip dS1;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) load_strip(dS1[ks], dS1g, ks);
    put_rows(Rt, Rr);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    clear(Gu);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        u32x4 b[NCT][N_TERMS];
        strip_terms(dS1[ks], b);
        add_product(Rt, b, ks, Gu);
        __builtin_amdgcn_sched_barrier(0);
    }
    Raw8<T> Kr[NPC], Qr[NPC];
#pragma unroll
    for (int p = 0; p < NPC; ++p) {
        Kr[p].load(a.K + tokl * D + 8 * (tid + 256 * p));
        Qr[p].load(a.Q + tokl * D + 8 * (tid + 256 * p));
    }
    f32x4 DPv[NTL], DAv[NTL];   // tile t of the list to wavefront t % 4
#pragma unroll
    for (int s = 0; s < NTL; ++s) {
        const int t = w + 4 * s;   // uniform
        DPv[s] = DAv[s] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (t < 10) {
            const int ta = (0x3333222110 >> (4 * t)) & 15, tb = (0x3210210100 >> (4 * t)) & 15;
            const size_t row = (tok0 + 16 * ta + l16) * D + 8 * lq;
            Raw8<TO> xo[KS];
            Raw8<float> xr[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                xo[ks].load(a.dO + row + 32 * ks);
                xr[ks].load(a.dR + row + 32 * ks);
            }
            float atv[4], pmv[4];   // At and P where this lane holds dAt and dP
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const size_t off = gcl * (CB_C * CB_C) + (16 * ta + 4 * lq + j) * CB_C + 16 * tb + l16;
                atv[j] = a.o.At[off];
                pmv[j] = a.o.Pm[off];
            }
            f32x4 accP = {0.f, 0.f, 0.f, 0.f}, accA = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                u32x4 u[N_TERMS], o[NO], r[N_TERMS];
                Rt.rows(16 * tb + l16, 32 * ks + 8 * lq, u);
                xo[ks].terms(o);
                xr[ks].terms(r);
                accP = mfma_terms(o, u, accP);
                accA = mfma_terms(r, u, accA);
            }
            const int i = 16 * tb + l16;
            const float gi = s_g2[i], gil = s_g2l[i], bi = s_bp[i];
            float csum = 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = 16 * ta + 4 * lq + j;
                // as the operands' kernel has it: behind alphas near 0 log2 gamma reaches thousands, and a float of that
                // size holds no more than three digits of a ratio
                const float G = __builtin_amdgcn_exp2f((s_g2[r] - gi) + (s_g2l[r] - gil));
                const float dp = (i <= r) ? a.la_scale * accP[j] : 0.f, da = (i < r) ? -delta * accA[j] : 0.f;   // no At without the delta rule
                const float e = da * atv[j] + dp * pmv[j];   // dP = dO' U^T, dAt = - dR U^T: these times b'_i
                const float rsum = lane_group_sum<16>(bi * e);
                if (l16 == 0) rs[tb * CB_C + r] = rsum;
                csum += e;
                DPv[s][j] = (i <= r) ? bi * dp * G : 0.f;
                DAv[s][j] = (i < r) ? bi * da * G : 0.f;
            }
            csum += lane_xor16(csum, lane);
            csum += lane_xor32(csum, lane);
            if (lq == 0) cs[ta * CB_C + i] = csum;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    // ---- stage 3: K, Q and the two 64 x 64 operands ---------------------------------------------------------------
    auto put_paired = [&](const typename LY::KTile& dst, const Raw8<T> (&r)[NPC]) {
#pragma unroll
        for (int p = 0; p < NPC; ++p) {
            const int e = 8 * (tid + 256 * p), row = e / D, c = e % D;
            u32x4 t[NT];
            r[p].terms(t);
            if constexpr (NCT == 2) {   // columns 32 g + 2 m + ct to places 32 g + 16 ct + m
                uint2 even[NT], odd[NT];
#pragma unroll
                for (int i = 0; i < NT; ++i) {
                    even[i] = make_uint2(__builtin_amdgcn_perm(t[i][1], t[i][0], 0x05040100u), __builtin_amdgcn_perm(t[i][3], t[i][2], 0x05040100u));
                    odd[i] = make_uint2(__builtin_amdgcn_perm(t[i][1], t[i][0], 0x07060302u), __builtin_amdgcn_perm(t[i][3], t[i][2], 0x07060302u));
                }
                dst.put(row, (c & ~31) + (c & 31) / 2, even);
                dst.put(row, (c & ~31) + 16 + (c & 31) / 2, odd);
            } else {
                dst.put(row, c, t);
            }
        }
    };
    put_paired(Kt, Kr);
    put_paired(Qt, Qr);
#pragma unroll
    for (int s = 0; s < NTL; ++s) {
        const int t = w + 4 * s;   // tiles 10, 11 of the list: those above the diagonal that a product over 32 tokens meets
        const int ta = (int)((0x203333222110ull >> (4 * t)) & 15), tb = (int)((0x313210210100ull >> (4 * t)) & 15);
        const int i = 16 * tb + l16;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = 16 * ta + 4 * lq + j;
            Pf[r * MS + i] = DPv[s][j];
            if (i < r) {
                Af[r * MS + i] = DAv[s][j];
                Af[i * MS + r] = DAv[s][j];
            } else if (i == r) {
                Af[r * MS + i] = 0.f;
            }
        }
    }
    // the softmax branch's share of dQ, which the result is added to: asked for before the products below
    float oldq[4][4][NCT];
#pragma unroll
    for (int ta = 0; ta < 4; ++ta)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float* p = a.dQ + (tok0 + 16 * ta + 4 * lq + j) * D + col0;
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) oldq[ta][j][ct] = p[ct];
        }
    __syncthreads();
    f32x4 dQa[4][NCT], dKa[4][NCT];
    float esum = 0.f;   // E_r is needed only as its sum over the chunk
#pragma unroll
    for (int tp = 0; tp < 2; ++tp) {
        float kc[NCT][8], qc[NCT][8];   // K and Q: the lane's columns, rows 4 lq + j of token tiles 2 tp and 2 tp + 1
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
            u32x4 tk[NT], tq[NT];
            Kt.cols(32 * tp, 16 * (NCT * w + ct), l16, lq, tk);
            Qt.cols(32 * tp, 16 * (NCT * w + ct), l16, lq, tq);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                kc[ct][i] = qc[ct][i] = 0.f;
#pragma unroll
                for (int n = NT - 1; n >= 0; --n) {   // exact: the terms of one number
                    kc[ct][i] += __uint_as_float(i & 1 ? tk[n][i / 2] & 0xffff0000u : tk[n][i / 2] << 16);
                    qc[ct][i] += __uint_as_float(i & 1 ? tq[n][i / 2] & 0xffff0000u : tq[n][i / 2] << 16);
                }
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ta = 2 * tp + h;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = 16 * ta + 4 * lq + j;
                const float gam = s_gam[r], kd = s_kd[r], bp = s_bp[r];
                float x = 0.f, u = 0.f;
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct) {
                    const float k = kc[ct][4 * h + j], q = qc[ct][4 * h + j], gq = a.la_scale * Gdq[ta][ct][j];
                    const float ku = kd * Gu[ta][ct][j], eu = k * ku;
                    u += eu;
                    x += gam * (q * gq - delta * k * Gdk[ta][ct][j]) - bp * eu;
                    dQa[ta][ct][j] = gam * gq;
                    dKa[ta][ct][j] = bp * ku - delta * gam * Gdk[ta][ct][j];
                }
                esum += bp * u;
                const float xs = lane_group_sum<16>(x), us = lane_group_sum<16>(u);
                if (l16 == 0) {
                    gk[w * CB_C + r] = xs;
                    gu[w * CB_C + r] = us;
                }
            }
        }
    }
    esum = lane_group_sum<64>(esum);
    if (lane == 0) ge[w] = esum;
    auto row_terms = [&](const float* M, int row, int col, u32x4 (&t)[N_TERMS]) {   // 8 of a row
        const float4 lo = ld4(M + row * MS + col), hi = ld4(M + row * MS + col + 4);
        const float x[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        split_terms(x, t);
    };
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        u32x4 kb[NCT][NT], qb[NCT][NT];
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
            Kt.cols_in_order(32 * ks, 16 * (NCT * w + ct), l16, lq, kb[ct]);
            Qt.cols_in_order(32 * ks, 16 * (NCT * w + ct), l16, lq, qb[ct]);
        }
#pragma unroll
        for (int ta = 0; ta < 4; ++ta) {
            u32x4 m[N_TERMS];
            if (ks <= ta >> 1) {
                row_terms(Pf, 16 * ta + l16, 32 * ks + 8 * lq, m);
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct) dQa[ta][ct] = mfma_terms(m, kb[ct], dQa[ta][ct]);
            }
            row_terms(Af, 16 * ta + l16, 32 * ks + 8 * lq, m);
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) dKa[ta][ct] = mfma_terms(m, kb[ct], dKa[ta][ct]);
            if (ks >= ta >> 1) {   // (dP . Gamma)^T Q
                float x[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = Pf[(32 * ks + 8 * lq + i) * MS + 16 * ta + l16];
                split_terms(x, m);
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct) dKa[ta][ct] = mfma_terms(m, qb[ct], dKa[ta][ct]);
            }
        }
    }
#pragma unroll
    for (int ta = 0; ta < 4; ++ta)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const size_t off = (tok0 + 16 * ta + 4 * lq + j) * D + col0;
            if constexpr (ROUNDED) {
                float q[NCT], k[NCT];
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct) {
                    q[ct] = oldq[ta][j][ct] + dQa[ta][ct][j];
                    k[ct] = dKa[ta][ct][j];
                }
                store_rounded(a.dQb + off, q);
                if (a.dKb != nullptr) {
                    store_rounded(a.dKb + off, k);
                    continue;
                }
            }
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) {
                if (!ROUNDED) a.dQ[off + ct] = oldq[ta][j][ct] + dQa[ta][ct][j];
                a.dK[off + ct] = dKa[ta][ct][j];
            }
        }
    __syncthreads();
    // ---- the gates: d ln gamma of every token, its sum from the back, dalpha; dbeta ----------------------------
    if (w == 0) {
        const int r = 63 - lane;   // reversed, so that the inclusive scan below sums from the chunk's end
        float dl = 0.f, et = 0.f, db = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) { dl += rs[q * CB_C + r]; db += cs[q * CB_C + r]; }
        dl -= s_bp[r] * db;
#pragma unroll
        for (int q = 0; q < 4; ++q) { dl += gk[q * CB_C + r]; et += ge[q]; db += gu[q * CB_C + r]; }
        constexpr int ND = D / CB_NV * (D / 32);
        const float dt = lane_group_sum<64>(lane < ND ? a.dot[gc * ND + lane] : 0.f);   // <dS1, S0>
        // the decay carried over the chunk: not a function of the alphas for a softmax chunk in the variant without decay
        const bool carry_fixed = a.chunk_mask && a.freeze_on_softmax && a.mask[gcl] != 0;
        if (r == 63) dl += et + (carry_fixed ? 0.f : a.o.gamC[gcl] * dt);
        // Eq. 17 for a chunk: <dS1, what the chunk added to the carried state> = sum_i kd_i K_i . (U dS1)_i (kd = 0 for
        // a softmax chunk)
        if (lane == 0 && a.dscore_la != nullptr) a.dscore_la[gc] = et;
        dl += dpp_move<0x111>(dl);
        dl += dpp_move<0x112>(dl);
        dl += dpp_move<0x114>(dl);
        dl += dpp_move<0x118>(dl);
        dl += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(dl), 0x142, 0xA, 0xF, false));
        dl += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(dl), 0x143, 0xC, 0xF, false));
        const size_t t = tok0 + r, tl = tokl + r;
        const bool frozen = a.freeze_on_softmax && !a.chunk_mask && a.mask[tl] != 0;   // its alpha counted as 1
        // (an alpha below 1e-37 counted as that, whatever it was; what dl carries of the rounding of its sums would be all there is)
        const float al = a.alpha[tl];
        a.dalpha[t] = frozen || al < 1e-37f ? 0.f : dl / al;
        a.dbeta[t] = !a.chunk_mask && a.mask[tl] != 0 ? 0.f : db;   // routing per token: a softmax token does not write
        if (a.g_nla != nullptr) a.g_nla[t] = 0.f;
    }
}

// ---- the linear branch's output rows from what the forward-by-chunks leaves ---------------------------------------------
// O = la (diag(gamma) Q S0^T + P U) for every chunk at once, fp32: S0 the state at the chunk's start (ck), U the rows
// gdn_chunk_seq_kernel<.., 0> wrote, P and gamma from the chunk's operands.  Needed where the backward pass must know
// the branch's rows (the merges that normalise them, Eq. 21).  One block per (chunk, batch*head); wavefront w owns a
// quarter of the value columns for all 64 tokens, so every element of S0 and U is read once per block, straight
// from memory as the right operand; Q and P, which every wavefront reads whole, go through LDS (P with its columns times
// b': P U = P diag(b') Uh).
// FWD, redo: whether the chunk made anything that is not finite, redo[chunk].  A product over a chunk or a half of it takes in,
// with weight 0, tokens that a row does not see, and 0 x NaN is NaN: where a NaN or an infinity comes in (from the tensors, the
// gates or an overflow), rows before it are lost too, in this chunk.  The recurrence token by token has no such products; the
// launch behind this one redoes every head with a chunk marked here (gdn_recurrent.hip).  Whatever is not finite in a token's
// Uh meets the diagonal of P and is seen in that token's row; without the inner part Uh itself is looked at.
// O_la may be Uh itself: a wavefront has read all it needs of it before it writes, and both are its own columns.
// Head grouping: BH counts output heads, Q and the operands are those of linear head bh / G.  inner: 0 leaves P U out
// (the ablation whose linear branch reads the carried state only).
// FWD: 16 contraction indices at a time from zero, added up (see the operands' kernel); otherwise running sums.
template <typename T, int D, bool FWD>
__global__ __launch_bounds__(256) void gdn_chunk_out_kernel(const T* __restrict__ Q, const ChunkOps o,
                                                           const float* __restrict__ ck, const float* Uh,
                                                           float* O_la, const int L, const int BH, const int G,
                                                           const int inner, const float la_scale, int32_t* redo) {
    constexpr int KS = D + 4, MS = CB_MS, VW = D / 4, VT = VW / 16;   // value columns per wavefront, in tiles of 16
    auto mac = [](const float4 a, const float4 b, const f32x4 c) {
        if constexpr (FWD) return c + mac16(a, b, f32x4{0.f, 0.f, 0.f, 0.f});
        else return mac16(a, b, c);
    };
    __shared__ __align__(16) float Qs[CB_C * KS];
    __shared__ __align__(16) float Ps[CB_C * MS];
    __shared__ float s_gam[CB_C];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int n_chunks = L / CB_C;
    const int bh = blockIdx.x % BH, chunk = blockIdx.x / BH;
    const size_t gc = (size_t)bh * n_chunks + chunk, tok0 = (size_t)bh * L + (size_t)chunk * CB_C;
    const size_t gl = (size_t)(bh / G) * n_chunks + chunk, tokl = (size_t)(bh / G) * L + (size_t)chunk * CB_C;
    constexpr int E = Vec16<T>::N;
    float seen = 0.f;   // stays 0 while all that it is shown is finite
    auto look = [&](float x) { if constexpr (FWD) seen = fmaf(x, 0.f, seen); };
    for (int e = tid; e < CB_C * D / E; e += 256) {
        const int row = e / (D / E), c = (e % (D / E)) * E;
        float tmp[E];
        Vec16<T>::load(Q + (tokl + row) * D + c, tmp);
#pragma unroll
        for (int j = 0; j < E; j += 4)
            *reinterpret_cast<float4*>(Qs + row * KS + c + j) = make_float4(tmp[j], tmp[j + 1], tmp[j + 2], tmp[j + 3]);
    }
    for (int e = tid; e < CB_C * CB_C / 4; e += 256) {
        const int row = e / 16, c4 = (e % 16) * 4;
        const float4 p = ld4(o.Pm + gl * (CB_C * CB_C) + row * CB_C + c4), b = ld4(o.bp + tokl + c4);
        const float4 pb = make_float4(p.x * b.x, p.y * b.y, p.z * b.z, p.w * b.w);
        look(pb.x); look(pb.y); look(pb.z); look(pb.w);
        *reinterpret_cast<float4*>(Ps + row * MS + c4) = pb;
    }
    if (tid < CB_C) s_gam[tid] = o.gam[tokl + tid];
    __syncthreads();
    const float* S0 = ck + gc * (size_t)D * D;
    f32x4 acc[4][VT];
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
        for (int vt = 0; vt < VT; ++vt) acc[tt][vt] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Q S0^T: A = Q[token l16 of tile tt][k], B = S0[v = l16 of tile vt][k]
#pragma unroll 2
    for (int kt = 0; kt < D / 16; ++kt) {
        float4 b[VT];
#pragma unroll
        for (int vt = 0; vt < VT; ++vt) b[vt] = ld4(S0 + (size_t)(VW * w + 16 * vt + l16) * D + 16 * kt + 4 * lq);
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const float4 a = ld4(Qs + (16 * tt + l16) * KS + 16 * kt + 4 * lq);
#pragma unroll
            for (int vt = 0; vt < VT; ++vt) acc[tt][vt] = mac(a, b[vt], acc[tt][vt]);
        }
    }
    // rows scaled by gamma (a lane holds tokens 16 tt + 4 lq + j of value column l16)
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
        const float4 g4 = ld4(s_gam + 16 * tt + 4 * lq);
        const float g[4] = {g4.x, g4.y, g4.z, g4.w};
#pragma unroll
        for (int vt = 0; vt < VT; ++vt)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[tt][vt][j] *= g[j];
    }
    // + P U: A = P[token][i], B = U[i = 16 tb + 4 lq + j][v]; P is lower triangular: tiles tb <= tt
    if (inner) {
#pragma unroll
        for (int tb = 0; tb < 4; ++tb) {
            float4 b[VT];
#pragma unroll
            for (int vt = 0; vt < VT; ++vt)
                b[vt] = ld4col(Uh + (tok0 + 16 * tb + 4 * lq) * D + VW * w + 16 * vt + l16, D);
#pragma unroll
            for (int tt = tb; tt < 4; ++tt) {
                const float4 a = ld4(Ps + (16 * tt + l16) * MS + 16 * tb + 4 * lq);
#pragma unroll
                for (int vt = 0; vt < VT; ++vt) acc[tt][vt] = mac(a, b[vt], acc[tt][vt]);
            }
        }
    } else if constexpr (FWD) {
        for (int tb = 0; tb < 4; ++tb)
            for (int vt = 0; vt < VT; ++vt) {
                const float4 b = ld4col(Uh + (tok0 + 16 * tb + 4 * lq) * D + VW * w + 16 * vt + l16, D);
                look(b.x); look(b.y); look(b.z); look(b.w);
            }
    }
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
        for (int vt = 0; vt < VT; ++vt)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float x = la_scale * acc[tt][vt][j];
                look(x);
                O_la[(tok0 + 16 * tt + 4 * lq + j) * D + VW * w + 16 * vt + l16] = x;
            }
    if constexpr (FWD) {
        const int any = __syncthreads_or(seen != 0.f);   // NaN by now: unequal to everything
        if (tid == 0) redo[gc] = any;
    }
}

// with_at: room for At as well (the backward pass; the forward does without)
static ChunkOps chunk_ops(const FwdPlan& pl, float* base, bool with_at = true) {
    const size_t n_tok = (size_t)pl.BH * pl.L, n_ch = n_tok / CB_C;
    ChunkOps o;
    o.Tm = base;
    o.At = with_at ? o.Tm + n_ch * CB_C * CB_C : nullptr;
    o.Pm = o.Tm + (with_at ? 2 : 1) * n_ch * CB_C * CB_C;
    o.g2 = o.Pm + n_ch * CB_C * CB_C;
    o.g2l = o.g2 + (with_at ? n_tok : 0);
    o.gam = o.g2l + (with_at ? n_tok : 0);
    o.kd = o.gam + n_tok;
    o.bp = o.kd + n_tok;
    o.gamC = o.bp + n_tok;
    return o;
}
size_t chunk_ops_floats(const FwdPlan& pl, bool with_at) {
    const size_t n_tok = (size_t)pl.BH * pl.L, n_ch = n_tok / CB_C;
    return (with_at ? 3 : 2) * n_ch * CB_C * CB_C + (with_at ? 5 : 3) * n_tok + align_up(n_ch, 64);
}

template <typename T, int D, bool FWD>
static bool launch_prep_t(const FwdPlan& pl, const PrepArgs<T>& a, const ScanArgs<T>& sc, hipStream_t st) {
    auto kern = gdn_bwd_prep_kernel<T, D, FWD>;
    constexpr size_t lds = PrepLds<T, D>::bytes;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
        hipSuccess) return false;
    const int scan_segs = (pl.L + SCAN_SEG - 1) / SCAN_SEG, scan_blocks = scan_segs * pl.BHG;
    hipLaunchKernelGGL(kern, dim3((unsigned)(scan_blocks + pl.BH * (pl.L / CB_C))), dim3(256), lds, st, a, sc, scan_segs,
                       scan_blocks);
    return true;
}

// ops: chunk_ops_floats(pl) floats.  Either routing.  The same launch carries the mask scan and compaction (arguments as
// launch_scan_compact; Ks: the softmax branch's keys).
nats_status launch_gdn_bwd_prep(const FwdPlan& pl, const void* Q, const void* K, const float* alpha, const float* beta,
                                const uint8_t* mask, float* ops, bool with_at, const void* Ks, const void* V, int32_t* cnt,
                                int32_t* idx, int32_t* n_s, void* Kc, void* Vc, void* Kc_user, void* Vc_user, int cap_user,
                                void* Vh, hipStream_t st) {
    const int by_chunk = pl.routing == NATS_ROUTE_CHUNK;
    auto go = [&](auto t) {
        using T = decltype(t);
        const PrepArgs<T> a{(const T*)Q, (const T*)K, alpha, beta, mask, chunk_ops(pl, ops, with_at), pl.L, pl.BH,
                            pl.freeze_on_softmax, pl.linear_op, by_chunk};
        const ScanArgs<T> sc{mask, (const T*)Ks, (const T*)V, pl.L, pl.d, cnt, idx, n_s, (T*)Kc, (T*)Vc, (T*)Kc_user, (T*)Vc_user,
                             cap_user, (half_t*)Vh, by_chunk ? (pl.RC == 128 ? 7 : 6) : 0, pl.G, pl.qk_per_out_head, pl.zero_rest};
        if (pl.d == 64) return with_at ? launch_prep_t<T, 64, false>(pl, a, sc, st) : launch_prep_t<T, 64, true>(pl, a, sc, st);
        return with_at ? launch_prep_t<T, 128, false>(pl, a, sc, st) : launch_prep_t<T, 128, true>(pl, a, sc, st);
    };
    if (!(pl.dtype == NATS_BF16 ? go(bf16_t{}) : go(float{}))) {
        set_error("gdn_bwd_prep: the kernel's LDS size was refused");
        return NATS_ERR_HIP;
    }
    return check_launch("gdn_bwd_prep");
}

template <typename T, typename TX, int D, int DIR, int NSL>
static bool launch_seq_s(const SeqArgs<T, TX>& a, hipStream_t st) {
    auto kern = gdn_chunk_seq_kernel<T, TX, D, DIR, NSL>;
    constexpr size_t lds = SeqLds<T, TX, D, DIR, NSL>::bytes;
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
        hipSuccess) return false;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.BH * (D / CB_NV / NSL))), dim3(256 * NSL + SeqLds<T, TX, D, DIR, NSL>::move), lds, st, a);
    return true;
}
template <typename T, typename TX, int D, int DIR>
static bool launch_seq_t(const SeqArgs<T, TX>& a, hipStream_t st) {
    // A block takes a CU to itself.  One slice per block up to one block per CU; beyond, where it would take another round, two (n
    // against n / 2 blocks, never as many rounds).  Forwards / backwards in us, one slice -> two, d 128: 36 heads, L 2048
    // 107 / 171 -> 75 / 133; 48 heads, L 4096 234 / 362 -> 167 / 270; 80 heads, L 2048 178 / 279 -> 150 / 254; 128 heads, L 2048
    // 256 / 417 -> 177 / 298; d 64: 72 heads, L 2048 68 / 132 -> 60 / 97; 256 heads, L 2048 263 / 520 -> 191 / 277.  (32 heads,
    // L 2048, one round: 62 / 94 with one.)  fp32 tensors, three terms each, leave no room for a second slice.
    if constexpr (sizeof(T) == 2) {
        if (a.BH * (D / CB_NV) > 256) return launch_seq_s<T, TX, D, DIR, 2>(a, st);
    }
    return launch_seq_s<T, TX, D, DIR, 1>(a, st);
}
template <int DIR, typename T, typename TX>
static bool launch_seq_d(const FwdPlan& pl, const SeqArgs<T, TX>& a, hipStream_t st) {
    return pl.d == 64 ? launch_seq_t<T, TX, 64, DIR>(a, st) : launch_seq_t<T, TX, 128, DIR>(a, st);
}

// The states at the chunk starts, ck [BHG][L/64][d][d], with the residuals Uh [BHG][L][d] of every chunk; S_final (or
// NULL): the state after the last token.  ops as launch_gdn_bwd_prep left them (with_at as there).  Head grouping
// (pl.G > 1): V, the states and Uh have pl.BHG heads.
nats_status launch_gdn_chunk_states(const FwdPlan& pl, const void* K, const void* V, float* ops, bool with_at,
                                    const float* S_init, float* S_final, float* ck, float* Uh, hipStream_t st) {
    auto go = [&](auto t) {
        using T = decltype(t);
        const SeqArgs<T, T> a{(const T*)K, nullptr, (const T*)V, chunk_ops(pl, ops, with_at), S_init, ck, Uh, nullptr, nullptr, S_final, pl.L,
                              pl.BHG, pl.G, pl.la_scale, pl.linear_op == 0};
        return launch_seq_d<0>(pl, a, st);
    };
    if (!(pl.dtype == NATS_BF16 ? go(bf16_t{}) : go(float{}))) {
        set_error("gdn_chunk_states: the kernel's LDS size was refused");
        return NATS_ERR_HIP;
    }
    return check_launch("gdn_chunk_states");
}

// O_la [BHG][L][d] f32 from ops (after launch_gdn_bwd_prep), ck and Uh (after launch_gdn_chunk_states; O_la may be Uh).
// redo: the forward's marks of chunks that are not finite, [BHG][L/64], for launch_gdn_recurrent; NULL in the backward pass.
template <typename T, int D, bool FWD>
static void launch_out_t(const FwdPlan& pl, const void* Q, const ChunkOps& o, const float* ck, const float* Uh, float* O_la,
                         int32_t* redo, hipStream_t st) {
    hipLaunchKernelGGL((gdn_chunk_out_kernel<T, D, FWD>), dim3((unsigned)(pl.BHG * (pl.L / CB_C))), dim3(256), 0, st, (const T*)Q,
                       o, ck, Uh, O_la, pl.L, pl.BHG, pl.G, pl.inner_chunk != 1, pl.la_scale, redo);
}
template <typename T>
static void launch_out_d(const FwdPlan& pl, const void* Q, const ChunkOps& o, const float* ck, const float* Uh, float* O_la,
                         int32_t* redo, hipStream_t st) {
    const bool fwd = redo != nullptr;
    if (pl.d == 64) (fwd ? launch_out_t<T, 64, true> : launch_out_t<T, 64, false>)(pl, Q, o, ck, Uh, O_la, redo, st);
    else (fwd ? launch_out_t<T, 128, true> : launch_out_t<T, 128, false>)(pl, Q, o, ck, Uh, O_la, redo, st);
}
nats_status launch_gdn_chunk_out(const FwdPlan& pl, const void* Q, float* ops, bool with_at, const float* ck, const float* Uh,
                                 float* O_la, int32_t* redo, hipStream_t st) {
    const ChunkOps o = chunk_ops(pl, ops, with_at);
    if (pl.dtype == NATS_BF16) launch_out_d<bf16_t>(pl, Q, o, ck, Uh, O_la, redo, st);
    else launch_out_d<float>(pl, Q, o, ck, Uh, O_la, redo, st);
    return check_launch("gdn_chunk_out");
}

// The state gradients behind every chunk, dck [BHG][L/64][d][d], their products with the states ck (dot: at most d / 4 parts
// per chunk); dV (every row), dS0 (or NULL).  dO_f32: dO is fp32 whatever the tensors' type.
nats_status launch_gdn_chunk_state_grads(const FwdPlan& pl, const void* Q, const void* K, const void* dO, bool dO_f32,
                                         float* ops, const float* ck, float* dck, float* dot, float* dV, float* dS0,
                                         hipStream_t st) {
    auto go = [&](auto t, auto to) {
        using T = decltype(t);
        using TO = decltype(to);
        const SeqArgs<T, TO> a{(const T*)K, (const T*)Q, (const TO*)dO, chunk_ops(pl, ops), nullptr, dck, dV, ck, dot, dS0, pl.L,
                               pl.BHG, pl.G, pl.la_scale, pl.linear_op == 0};
        return launch_seq_d<1>(pl, a, st);
    };
    const bool ok = pl.dtype == NATS_F32 ? go(float{}, float{}) : dO_f32 ? go(bf16_t{}, float{}) : go(bf16_t{}, bf16_t{});
    if (!ok) { set_error("gdn_chunk_state_grads: the kernel's LDS size was refused"); return NATS_ERR_HIP; }
    return check_launch("gdn_chunk_state_grads");
}

template <typename T, typename TO, int D>
static bool launch_grads_t(const FwdPlan& pl, const GradArgs<T, TO>& a, hipStream_t st) {
    auto kern = gdn_chunk_grads_kernel<T, TO, D, false>;
    if constexpr (sizeof(T) == 2) {
        if (a.dQb != nullptr) kern = gdn_chunk_grads_kernel<T, TO, D, true>;
    }
    constexpr size_t lds = GradLds<T, TO, D>::bytes;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
        hipSuccess) return false;
    hipLaunchKernelGGL(kern, dim3((unsigned)(pl.BHG * (pl.L / CB_C))), dim3(256), lds, st, a);
    return true;
}

// dQ += the linear branch's share; dK, dalpha, dbeta = it; g_nla (optional) cleared.  ck, dck: the states and state
// gradients per chunk; Uh, dR (= the linear branch's dV) [BHG][L][d], and so everything written; dot as launch_gdn_chunk_state_grads left it.  dO_f32: dO is fp32 whatever the tensors' type.
// rounded (bf16 tensors): dQ goes there instead, and dK and dV (= dR) where given
nats_status launch_gdn_chunk_grads(const FwdPlan& pl, const void* Q, const void* K, const void* dO, bool dO_f32,
                                   const float* alpha, const uint8_t* mask, float* ops, const float* ck, const float* dck,
                                   const float* Uh, const float* dR, const float* dot, float* dQ, float* dK,
                                   float* dalpha, float* dbeta, float* g_nla, float* dscore_la, const RoundedGrads& rounded,
                                   hipStream_t st) {
    auto go = [&](auto t, auto to) {
        using T = decltype(t);
        using TO = decltype(to);
        const GradArgs<T, TO> a{(const T*)Q, (const T*)K, (const TO*)dO, chunk_ops(pl, ops), alpha, mask, ck, dck,
                                Uh, dR, dot, dQ, dK, dalpha, dbeta, g_nla, dscore_la, (bf16_t*)rounded.dQ, (bf16_t*)rounded.dK,
                                (bf16_t*)rounded.dV, pl.L, pl.BHG, pl.G, pl.la_scale,
                                pl.linear_op == 0, pl.freeze_on_softmax, pl.routing == NATS_ROUTE_CHUNK};
        return pl.d == 64 ? launch_grads_t<T, TO, 64>(pl, a, st) : launch_grads_t<T, TO, 128>(pl, a, st);
    };
    const bool ok = pl.dtype == NATS_F32 ? go(float{}, float{}) : dO_f32 ? go(bf16_t{}, float{}) : go(bf16_t{}, bf16_t{});
    if (!ok) { set_error("gdn_chunk_grads: the kernel's LDS size was refused"); return NATS_ERR_HIP; }
    return check_launch("gdn_chunk_grads");
}

}  // namespace nats
