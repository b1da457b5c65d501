// Chunkwise Gated DeltaNet, step 2 of 2, in one pass along the sequence (gdn_seg_scan.hip: the same in segments, two
// passes): on the raw K, Q, V and the per-chunk T'' = (I + A)^-1 diag(b'), P = (Q K^T) . D and gates of the inversion kernel
//   R  = V - diag(gam) K S0^T                 [C x d_v]
//   U  = T'' R                                [C x d_v]
//   O  = la_scale (diag(gam) Q S0^T + P U)    [C x d_v]   (linear-branch output, Eq. 7 / Eq. 10)
//   S1 = gam_C S0 + U^T diag(kd) K            [d_v x d_k]
//
// The rows of S (columns of V) never mix, so a (batch, head) falls into d / 16 SLICES of 16 value columns, each a chain of its
// own along the sequence.  The time is the number of chunks times that of a step, so a step has to be short: its chain
// S0 -> K S0^T -> R -> U -> S1 runs inside ONE wavefront with every link in its registers (a lane holds two 16-row
// accumulator tiles of a product as rows 4 lq .. 4 lq + 3 of each, and the contraction slots of the next product's operand
// are defined as exactly those 8 rows): at d = 128 38 matrix instructions, which a wavefront alone issues one per 16 cycles,
// and 226 others, one per 5.  Everything else is the work of other wavefronts of the block:
//   CHAIN     (one per slice)  the state, in fp32 accumulators, and the chain above;
//   OUTPUT    (one per slice)  S0 Q^T and U^T P^T from what the chain leaves in LDS, one chunk behind it; stores the rows
//                              (fp16, for the merge in the softmax kernel);
//   STAGING   (four)           the operands that the slices share, from memory to LDS a chunk ahead and in registers up to three
//                              chunks before that: K and Q (converted to fp16 once), T'', P, the gates, V transposed.
// One barrier per chunk; a block has NS slices, 1 or 2.  A step takes 0.96 us at d = 128 with one slice and 1.17 with two, 0.65 and
// 0.85 at d = 64, with 4-6 before the first, while the call's tensors fit the last cache (8 to 96 heads, L 512 against 2048); beyond
// (48 heads, L 4096, d 128) 1.29 with two.  (A CU has at most its 32 KB of L1 lines in flight, so 48 KB from HBM cost a step more
// than a memory latency.)  In segments a step takes 3.1 and 2.1 us, for all of a head's
// columns, and there are 2 / n_seg as many: see seg_form() in gdn_seg_scan.hip for where the line lies.
// Tried on the chain: four wavefronts per slice, a token tile and a quarter of the state each (three exchanges through LDS and
// three barriers per chunk: 1.15 us and more); its operands touched by the slices of a head in turn, some chunks ahead, so that
// the others' requests hit L2 (1.05 -> 1.15); a higher wave priority (nothing).
#include <type_traits>

#include "mfma_util.h"
#include "nats_common.h"

namespace nats {

constexpr int SL_C = 64;            // chunk size
constexpr int SL_STAGE = 256;       // staging threads of a block
constexpr int SL_SETS = 3;          // chunks in flight in the staging threads' registers
constexpr int slice_threads(int ns) { return SL_STAGE + 128 * ns; }

// LDS of a block: two operand sets; what the chains hand to the output wavefronts.
template <int D, int NS>
struct SliceLds {
    static constexpr int SS = D + 16;              // halves per row of the K, Q tiles: row-wise and transposing reads keep to different banks
    static constexpr int VS = SL_C + 4;            // floats per row of V transposed [v][token]
    // one operand set (halves)
    static constexpr int o_K = 0;
    static constexpr int o_Q = o_K + SL_C * SS;
    static constexpr int o_T = o_Q + SL_C * SS;        // T'' in fragment order (the 6 fragments on and below the diagonal)
    static constexpr int o_P = o_T + TRI_FRAG_HALFS;   // P in fragment order, times la_scale
    static constexpr int o_G = o_P + TRI_FRAG_HALFS;   // fp32: gam of K S0^T [64], gam la_scale [64], kd [64], gam_C
    static constexpr int o_V = o_G + 2 * 196;
    static constexpr int SET = o_V + 2 * NS * 16 * VS;
    // S0 and U of a slice as operand fragments, a buffer per chunk parity
    static constexpr int S_FR = D / 32 * 512, U_FR = 2 * 512;
    static constexpr int o_S = 2 * SET;                // [slice][parity][S_FR]
    static constexpr int o_U = o_S + NS * 2 * S_FR;    // [slice][parity][U_FR]
    static constexpr int bytes = (o_U + NS * 2 * U_FR) * 2;
    static_assert(bytes <= 160 * 1024, "one block per CU");
    static_assert(SET % 8 == 0 && o_G % 8 == 0 && o_V % 8 == 0, "16-byte aligned");
};

struct SliceArgs {
    const bf16_t *Q, *K, *V;
    const half_t *TF, *PF;
    const float *gamv, *kdv, *gamC;
    const float* S0;          // [BHG][D][D] initial state or nullptr
    float* S_final;           // [BHG][D][D] or nullptr
    half_t* O_la_h;           // fp16 linear-branch output, for the merge in the softmax kernel
    float* O_la_f32;          // optional fp32 copy of the linear-branch output
    int L, BH, gated;         // BH counts linear heads
    int G;                    // output heads per linear head (head grouping): K, Q, T'', P and the gates are the
                              // linear head's (index bh / G), V, the state and the outputs the output head's
    float la_scale;
};

// ---- CHAIN wavefronts.  Index conventions of a lane (l16 = lane % 16, lq = lane / 16):
//   accumulator tile      : rows 4 lq + j (j < 4), column l16
//   operand fragment      : row / column l16, contraction slots s < 8 of step ks: tokens 32 ks + 16 (s / 4) + 4 lq + s % 4,
//                           or d_k = 32 ks + 8 lq + s
// so that two accumulator tiles of tokens are the next operand, and so that K's and Q's fragments are 16 consecutive
// bytes of a row.  The state's tile (ks, p) holds d_k = 32 ks + 8 (row / 4) + 4 p + row % 4: its two tiles are the slots of
// step ks, and the update's operand, K^T with rows in that order, comes by transposing reads from the same K tile (each
// lane names where its four columns stand).
template <int D, int NS>
__device__ __forceinline__ void slice_chain(const SliceArgs& a, const int bh, const int slice, const int v0, half_t* lds) {
    using Lds = SliceLds<D, NS>;
    constexpr int SS = Lds::SS, VS = Lds::VS, KS_D = D / 32;
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
    const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
    const int n_chunks = a.L / SL_C;
    const size_t row = ((size_t)bh * D + v0 + l16) * D + 8 * lq;   // the lane's elements of a state in memory
    f32x4 S[KS_D][2];
#pragma unroll
    for (int ks = 0; ks < KS_D; ++ks)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
            if (a.S0 != nullptr) x = ld4(a.S0 + row + 32 * ks + 4 * p);
            S[ks][p] = f32x4{x.x, x.y, x.z, x.w};
        }
    half8 sf[KS_D];   // S[v = l16][d_k slots]: B operand of K S0^T, A operand of S0 Q^T
    half_t* Sb = lds + Lds::o_S + slice * 2 * Lds::S_FR;
    half_t* Ub = lds + Lds::o_U + slice * 2 * Lds::U_FR;
    auto operand_form = [&](int parity) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < KS_D; ++ks) {
            sf[ks] = pack_tiles(S[ks][0], S[ks][1]);
            *reinterpret_cast<half8*>(Sb + parity * Lds::S_FR + (ks * 64 + lane) * 8) = sf[ks];
        }
    };
    operand_form(0);
    __syncthreads();   // the first operand set is complete

    for (int c = 0; c < n_chunks; ++c) {
        const int par = c & 1;
        const half_t* set = lds + par * Lds::SET;
        const half_t* Kt = set + Lds::o_K;
        const half8* Tt = reinterpret_cast<const half8*>(set + Lds::o_T);
        const float* Gt = reinterpret_cast<const float*>(set + Lds::o_G);
        const float* Vt = reinterpret_cast<const float*>(set + Lds::o_V) + (16 * slice + l16) * VS;
        // ---- K S0^T, four independent chains of d / 32 instructions ----
        f32x4 acc[4];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) acc[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS_D; ++ks)
#pragma unroll
            for (int tt = 0; tt < 4; ++tt)
                acc[tt] = mfma16(lds_read8(Kt + (16 * tt + l16) * SS + 32 * ks + 8 * lq), sf[ks], acc[tt]);   // rows tok, col v
        const float gC = Gt[192];
#pragma unroll
        for (int ks = 0; ks < KS_D; ++ks)
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int j = 0; j < 4; ++j) S[ks][p][j] *= gC;
        // ---- R = V - gam (K S0^T) ----
        half8 rf[2];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const float4 g = ld4(Gt + 16 * tt + 4 * lq), x = ld4(Vt + 16 * tt + 4 * lq);
            acc[tt][0] = fmaf(-g.x, acc[tt][0], x.x);
            acc[tt][1] = fmaf(-g.y, acc[tt][1], x.y);
            acc[tt][2] = fmaf(-g.z, acc[tt][2], x.z);
            acc[tt][3] = fmaf(-g.w, acc[tt][3], x.w);
        }
#pragma unroll
        for (int kp = 0; kp < 2; ++kp) rf[kp] = pack_tiles(acc[2 * kp], acc[2 * kp + 1]);
        // ---- U = T'' R (T'' lower triangular: token tiles 0, 1 need the first contraction step only) ----
        half8 uf[2];   // kd U[token slots][v = l16]: B operand of K^T (kd U)
#pragma unroll
        for (int kp = 0; kp < 2; ++kp) {
            f32x4 u[2];
#pragma unroll
            for (int t2 = 0; t2 < 2; ++t2) {
                const int tt = 2 * kp + t2;
                u[t2] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks <= kp; ++ks) u[t2] = mfma16(Tt[tri_frag(tt, ks) * 64 + lane], rf[ks], u[t2]);   // rows r, col v
            }
            *reinterpret_cast<half8*>(Ub + par * Lds::U_FR + (kp * 64 + lane) * 8) = pack_tiles(u[0], u[1]);
#pragma unroll
            for (int t2 = 0; t2 < 2; ++t2) {
                const float4 k = ld4(Gt + 128 + 16 * (2 * kp + t2) + 4 * lq);
                u[t2][0] *= k.x;
                u[t2][1] *= k.y;
                u[t2][2] *= k.z;
                u[t2][3] *= k.w;
            }
            uf[kp] = pack_tiles(u[0], u[1]);
        }
        // ---- S1^T = gam_C S0^T + K^T (kd U) ----
#pragma unroll
        for (int kp = 0; kp < 2; ++kp)
#pragma unroll
            for (int ks = 0; ks < KS_D; ++ks)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const half_t* q = Kt + (32 * kp + 4 * lq + (l16 >> 2)) * SS + 32 * ks + 8 * (l16 & 3) + 4 * p;
                    const half4 lo = __builtin_bit_cast(half4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)q));
                    const half4 hi = __builtin_bit_cast(half4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(q + 16 * SS)));
                    S[ks][p] = mfma16(half8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]}, uf[kp], S[ks][p]);   // rows d_k, col v
                }
        operand_form(par ^ 1);
        __syncthreads();   // the next operand set is complete; this one and what was handed over for chunk c - 1 are free
    }
    if (a.S_final == nullptr) return;
#pragma unroll
    for (int ks = 0; ks < KS_D; ++ks)
#pragma unroll
        for (int p = 0; p < 2; ++p)
            *reinterpret_cast<float4*>(a.S_final + row + 32 * ks + 4 * p) = make_float4(S[ks][p][0], S[ks][p][1], S[ks][p][2], S[ks][p][3]);
}

// ---- OUTPUT wavefronts: S0 Q^T of the chunk at hand, U^T P^T of the one before, whose rows then go out.  Computed
// transposed, so that a lane holds four consecutive columns of a token.
template <int D, int NS, bool F32OUT>
__device__ __forceinline__ void slice_output(const SliceArgs& a, const int bh, const int slice, const int v0, half_t* lds) {
    using Lds = SliceLds<D, NS>;
    constexpr int SS = Lds::SS, KS_D = D / 32;
    const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
    const int n_chunks = a.L / SL_C;
    const half_t* Sb = lds + Lds::o_S + slice * 2 * Lds::S_FR;
    const half_t* Ub = lds + Lds::o_U + slice * 2 * Lds::U_FR;
    f32x4 acc[4];          // gam la_scale S0 Q^T of the previous chunk: rows v, col tok
    half8 pf[TRI_FRAGS];   // and its P
    auto finish = [&](int c) __attribute__((always_inline)) {
        half8 uf[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) uf[ks] = lds_read8(Ub + (c & 1) * Lds::U_FR + (ks * 64 + lane) * 8);
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
#pragma unroll
            for (int ks = 0; ks <= tt / 2; ++ks) acc[tt] = mfma16(uf[ks], pf[tri_frag(tt, ks)], acc[tt]);
            const size_t o = ((size_t)bh * a.L + (size_t)c * SL_C + 16 * tt + l16) * D + v0 + 4 * lq;
            *reinterpret_cast<half4*>(a.O_la_h + o) = to_half4_hw(acc[tt]);
            if (F32OUT) *reinterpret_cast<float4*>(a.O_la_f32 + o) = make_float4(acc[tt][0], acc[tt][1], acc[tt][2], acc[tt][3]);
        }
    };
    __syncthreads();
    for (int c = 0; c < n_chunks; ++c) {
        const int par = c & 1;
        const half_t* set = lds + par * Lds::SET;
        const half_t* Qt = set + Lds::o_Q;
        const half8* Pt = reinterpret_cast<const half8*>(set + Lds::o_P);
        const float* Gt = reinterpret_cast<const float*>(set + Lds::o_G);
        if (c > 0) finish(c - 1);
        half8 sf[KS_D];
#pragma unroll
        for (int ks = 0; ks < KS_D; ++ks) sf[ks] = lds_read8(Sb + par * Lds::S_FR + (ks * 64 + lane) * 8);
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) acc[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS_D; ++ks)
#pragma unroll
            for (int tt = 0; tt < 4; ++tt)
                acc[tt] = mfma16(sf[ks], lds_read8(Qt + (16 * tt + l16) * SS + 32 * ks + 8 * lq), acc[tt]);
#pragma unroll
        for (int f = 0; f < TRI_FRAGS; ++f) pf[f] = Pt[f * 64 + lane];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const float go = Gt[64 + 16 * tt + l16];
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[tt][j] *= go;
        }
        __syncthreads();
    }
    finish(n_chunks - 1);
}

// ---- STAGING wavefronts
template <int D, int NS>
__device__ __forceinline__ void slice_staging(const SliceArgs& a, const int bh, const int v0, half_t* lds) {
    using Lds = SliceLds<D, NS>;
    constexpr int SS = Lds::SS, VS = Lds::VS;
    constexpr int NPC = SL_C * D / 8 / SL_STAGE;       // 16-byte pieces of a [64][D] tile per thread
    constexpr int NFP = TRI_FRAG_HALFS / 8;            // pieces of a chunk's T'' or P
    constexpr int NV = NS * 2 * SL_C;                  // pieces of V
    static_assert(NV <= SL_STAGE, "one piece of V per thread");
    const int t = threadIdx.x - 128 * NS;
    const int n_chunks = a.L / SL_C;
    const size_t tokl = (size_t)(bh / a.G) * a.L, chl = (size_t)(bh / a.G) * n_chunks;   // the linear head's rows, chunks
    const bf16_t* Vp = a.V + ((size_t)bh * a.L + (t % NV) / (2 * NS)) * D + v0 + 8 * (t % (2 * NS));
    const half_t lah = (half_t)a.la_scale;
    const half8 la8 = {lah, lah, lah, lah, lah, lah, lah, lah};
    // Loads are unconditional, with clamped indices: around a branch the compiler waits for every load in flight.
    struct Regs {
        u32x4 k[NPC], q[NPC], v;
        half8 tp[2], pp[2];
        float g0, g1;
    } set[SL_SETS];
    auto fetch = [&](Regs& r, int c) __attribute__((always_inline)) {
        c = min(c, n_chunks - 1);   // the tail asks for the last chunk again
        const u32x4* K = reinterpret_cast<const u32x4*>(a.K + (tokl + (size_t)c * SL_C) * D);
        const u32x4* Q = reinterpret_cast<const u32x4*>(a.Q + (tokl + (size_t)c * SL_C) * D);
        const half8* T = reinterpret_cast<const half8*>(a.TF + (chl + c) * (size_t)TRI_FRAG_HALFS);
        const half8* P = reinterpret_cast<const half8*>(a.PF + (chl + c) * (size_t)TRI_FRAG_HALFS);
#pragma unroll
        for (int i = 0; i < NPC; ++i) r.k[i] = K[t + SL_STAGE * i];
#pragma unroll
        for (int i = 0; i < 2; ++i) r.tp[i] = T[min(t + SL_STAGE * i, NFP - 1)];
        r.v = *reinterpret_cast<const u32x4*>(Vp + (size_t)c * (SL_C * D));
        r.g0 = *(t < SL_C ? a.gamv + (chl + c) * SL_C + t : a.gamC + chl + c);
        r.g1 = a.kdv[(chl + c) * SL_C + (t & (SL_C - 1))];
#pragma unroll
        for (int i = 0; i < NPC; ++i) r.q[i] = Q[t + SL_STAGE * i];
#pragma unroll
        for (int i = 0; i < 2; ++i) r.pp[i] = P[min(t + SL_STAGE * i, NFP - 1)];
    };
    auto put = [&](const Regs& r, half_t* s) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NPC; ++i) {
            const int e = t + SL_STAGE * i, at = (e / (D / 8)) * SS + 8 * (e % (D / 8));
            *reinterpret_cast<half8*>(s + Lds::o_K + at) = cvt_bf16x8(r.k[i]);
            *reinterpret_cast<half8*>(s + Lds::o_Q + at) = cvt_bf16x8(r.q[i]);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (t + SL_STAGE * i >= NFP) continue;   // uniform per wavefront
            reinterpret_cast<half8*>(s + Lds::o_T)[t + SL_STAGE * i] = r.tp[i];
            reinterpret_cast<half8*>(s + Lds::o_P)[t + SL_STAGE * i] = r.pp[i] * la8;
        }
        float* G = reinterpret_cast<float*>(s + Lds::o_G);
        if (t < SL_C) {
            G[t] = a.gated ? 0.f : r.g0;   // without the delta rule the state does not enter R
            G[64 + t] = r.g0 * a.la_scale;
            G[128 + t] = r.g1;
        }
        if (t == SL_C) G[192] = r.g0;
        if (t < NV) {                      // uniform per wavefront
            float* Vt = reinterpret_cast<float*>(s + Lds::o_V) + 8 * (t % (2 * NS)) * VS + t / (2 * NS);
#pragma unroll
            for (int j = 0; j < 8; ++j) Vt[j * VS] = __uint_as_float(j & 1 ? r.v[j / 2] & 0xffff0000u : r.v[j / 2] << 16);
        }
    };
#pragma unroll
    for (int i = 0; i < SL_SETS; ++i) fetch(set[i], i);
    put(set[0], lds);
    fetch(set[0], SL_SETS);
    __syncthreads();   // the first operand set is complete
    auto step = [&](auto which, int c) __attribute__((always_inline)) {   // chunk c + 1 to LDS, chunk c + 1 + SL_SETS asked for
        Regs& r = set[decltype(which)::value];
        put(r, lds + ((c & 1) ^ 1) * Lds::SET);
        fetch(r, c + 1 + SL_SETS);
        __syncthreads();
    };
    // The register sets take turns without a copy: whole trips of SL_SETS steps, then the rest (a way out in the middle of the loop
    // would join at its head, where the compiler would then wait for every load in flight).
    static_assert(SL_SETS == 3, "the steps below");
    int c = 0;
    for (; c + 3 <= n_chunks; c += 3) {
        step(std::integral_constant<int, 1>{}, c);
        step(std::integral_constant<int, 2>{}, c + 1);
        step(std::integral_constant<int, 0>{}, c + 2);
    }
    if (c < n_chunks) step(std::integral_constant<int, 1>{}, c);
    if (c + 1 < n_chunks) step(std::integral_constant<int, 2>{}, c + 1);
}

template <int D, int NS, bool F32OUT>
__global__ __launch_bounds__(slice_threads(NS)) void gdn_slice_scan_kernel(const SliceArgs a) {
    extern __shared__ __align__(16) unsigned char slice_smem[];
    half_t* lds = reinterpret_cast<half_t*>(slice_smem);
    fp16_saturate_on();   // conversions to fp16 clamp to the fp16 range (see to_half4_hw)
    // Blocks with ids congruent modulo 8 share an XCD and its L2: the blocks of a linear head, which read the same K, Q,
    // T'' and P, are given such ids.
    constexpr int NB = D / 16 / NS;   // blocks per output head
    const int slot = blockIdx.x >> 3, hq = slot / NB, lin = (hq / a.G) * 8 + (blockIdx.x & 7);
    if (lin >= a.BH) return;
    const int bh = lin * a.G + hq % a.G, v0 = 16 * NS * (slot % NB);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), slice = wave % NS;
    if (wave < NS) slice_chain<D, NS>(a, bh, slice, v0 + 16 * slice, lds);
    else if (wave < 2 * NS) slice_output<D, NS, F32OUT>(a, bh, slice, v0 + 16 * slice, lds);
    else slice_staging<D, NS>(a, bh, v0, lds);
}

template <int D, int NS, bool F32OUT>
static nats_status launch_slice_k(const FwdPlan& pl, const SliceArgs& a, hipStream_t st) {
    static bool attr_done[64] = {};
    int dev = 0;
    (void)hipGetDevice(&dev);
    dev = (dev >= 0 && dev < 64) ? dev : 0;
    auto kern = gdn_slice_scan_kernel<D, NS, F32OUT>;
    constexpr int bytes = SliceLds<D, NS>::bytes;
    if (!attr_done[dev]) {   // the LDS-size attribute is per function and device
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess)
            return check_launch("gdn_slice_scan (LDS attribute)");
        attr_done[dev] = true;
    }
    ProfScope ps("gdn_slice_scan", st);
    hipLaunchKernelGGL(kern, dim3(8 * ((pl.BH + 7) / 8) * pl.G * (D / 16 / NS)), dim3(slice_threads(NS)), bytes, st, a);
    return check_launch("gdn_slice_scan");
}

template <int D>
static nats_status launch_slice_d(const FwdPlan& pl, int ns, const SliceArgs& a, hipStream_t st) {
    if (a.O_la_f32 != nullptr) return ns == 1 ? launch_slice_k<D, 1, true>(pl, a, st) : launch_slice_k<D, 2, true>(pl, a, st);
    return ns == 1 ? launch_slice_k<D, 1, false>(pl, a, st) : launch_slice_k<D, 2, false>(pl, a, st);
}

// ns: slices per block, 1 or 2.  Writes O_la_h (fp16) for the softmax kernel to merge, and O_la_f32 if given.
nats_status launch_gdn_slice_scan(const FwdPlan& pl, int ns, const void* Q, const void* K, const void* V, const void* TF, const void* PF,
                                  const float* gamv, const float* kdv, const float* gamC, const float* S0, float* S_final,
                                  void* O_la_h, float* O_la_f32, hipStream_t st) {
    const SliceArgs a{(const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, (const half_t*)TF, (const half_t*)PF, gamv, kdv, gamC,
                      S0, S_final, (half_t*)O_la_h, O_la_f32, pl.L, pl.BH, pl.linear_op == NATS_LINEAR_GATED, pl.G, pl.la_scale};
    return pl.d == 64 ? launch_slice_d<64>(pl, ns, a, st) : launch_slice_d<128>(pl, ns, a, st);
}

}  // namespace nats
