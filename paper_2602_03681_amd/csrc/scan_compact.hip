// Mask scan + K/V compaction (paper Section 4.1: the softmax branch loads only the
// tokens routed to it; Eq. 12 gives the column set).  For every (batch, head):
//   cnt[t] = #softmax tokens among 0..t,  idx[c] = position of the c-th one,
//   n_s = cnt[L-1],  Kc[c] = K[idx[c]],  Vc[c] = V[idx[c]].
// Integer work, exactly one correct answer.  HBM-bound.
//
// Grid (ceil(L / SEG), B*H).  A block owns SEG consecutive tokens.  Its base
// count is recomputed from the mask bytes in front of the segment (at most L
// bytes, read 16 at a time and served by L2), so blocks need no ordering and
// no inter-block communication.
#include "scan_compact_block.h"

namespace nats {

template <typename T>
__global__ __launch_bounds__(SCAN_THREADS) void scan_compact_kernel(const ScanArgs<T> a) {
    __shared__ int lds[SCAN_LDS_INTS];
    scan_compact_block<T>(a, blockIdx.x, blockIdx.y, lds);
}

nats_status launch_scan_compact(const FwdPlan& pl, const uint8_t* mask, const void* K, const void* V,
                                int32_t* cnt, int32_t* idx, int32_t* n_s, void* Kc, void* Vc,
                                void* Kc_user, void* Vc_user, int cap_user, void* Vh, hipStream_t st) {
    dim3 grid((pl.L + SCAN_SEG - 1) / SCAN_SEG, pl.BHG);
    if (pl.dtype == NATS_BF16) {
        const ScanArgs<bf16_t> a{mask, (const bf16_t*)K, (const bf16_t*)V, pl.L, pl.d, cnt, idx, n_s, (bf16_t*)Kc,
                                 (bf16_t*)Vc, (bf16_t*)Kc_user, (bf16_t*)Vc_user, cap_user, (half_t*)Vh,
                                 pl.routing == NATS_ROUTE_CHUNK ? (pl.RC == 128 ? 7 : 6) : 0, pl.G, pl.qk_per_out_head, pl.zero_rest};
        hipLaunchKernelGGL(scan_compact_kernel<bf16_t>, grid, dim3(SCAN_THREADS), 0, st, a);
    } else {
        const ScanArgs<float> a{mask, (const float*)K, (const float*)V, pl.L, pl.d, cnt, idx, n_s, (float*)Kc,
                                (float*)Vc, (float*)Kc_user, (float*)Vc_user, cap_user, (half_t*)Vh,
                                pl.routing == NATS_ROUTE_CHUNK ? (pl.RC == 128 ? 7 : 6) : 0, pl.G, pl.qk_per_out_head, pl.zero_rest};
        hipLaunchKernelGGL(scan_compact_kernel<float>, grid, dim3(SCAN_THREADS), 0, st, a);
    }
    return check_launch("scan_compact");
}

// n pieces of 16 bytes of Kc (blockIdx.y 0) and Vc.  One piece per thread: 2152 MB (64 heads, 32832 rows of 512 bytes) in 314 us, 6.8 TB/s;
// two pieces 346, four 360; head by head with the rows below L left out 174 instead of 159 (256 heads, 8256 rows of 256 bytes).
__global__ __launch_bounds__(SCAN_THREADS) void clear_cache_kernel(uint4* Kc, uint4* Vc, size_t n) {
    uint4* p = blockIdx.y ? Vc : Kc;
    for (size_t e = (size_t)blockIdx.x * SCAN_THREADS + threadIdx.x; e < n; e += (size_t)gridDim.x * SCAN_THREADS)
        p[e] = make_uint4(0u, 0u, 0u, 0u);
}

// The compaction's blocks, one per 1024 tokens of a head, clear what lies behind L on the side, at some 150 GB/s each: free up to 512 KB
// per block (2.8 us less than a launch of its own, over 68 sizes from 1 head and L 64 on), even with it at 1 MB (0.5 us), 5 us behind at 2 MB,
// 100 at 16 MB (16 heads, L 64, d 128, cap 32768 bf16: 144 us for the call, 59 with two fills beforehand).
bool clears_cache_apart(const FwdPlan& pl, int cap) {
    const size_t tail = cap > pl.L ? (size_t)(cap - pl.L) * pl.d * (pl.dtype == NATS_BF16 ? 4 : 8) : 0;   // of a head, both arrays
    return tail / ((pl.L + SCAN_SEG - 1) / SCAN_SEG) >= (size_t)1 << 20;
}

nats_status launch_clear_cache(const FwdPlan& pl, void* Kc_user, void* Vc_user, int cap, hipStream_t st) {
    const size_t n = (size_t)pl.BHG * cap * pl.d * (pl.dtype == NATS_BF16 ? 2 : 4) / 16, blocks = (n + SCAN_THREADS - 1) / SCAN_THREADS;
    const size_t most = (size_t)1 << 23;   // a launch has fewer than 2^32 threads along x
    hipLaunchKernelGGL(clear_cache_kernel, dim3((unsigned)(blocks < most ? blocks : most), 2), dim3(SCAN_THREADS), 0, st, (uint4*)Kc_user,
                       (uint4*)Vc_user, n);
    return check_launch("clear_cache");
}

}  // namespace nats
