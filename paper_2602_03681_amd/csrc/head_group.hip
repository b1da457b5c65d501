// Head grouping (Section 4.3) in the backward pass: G output heads (own V, own state) share the Q, K, alpha, beta
// and mask of one linear head, so the gradient of a shared input is the sum of what each of the G heads sends back.
// Where the pass runs over all output heads at once, their shares are added up here, all gradients in one launch.  Where
// it runs once per member of the groups on that member's heads, gathered into contiguous tensors, two kernels move a
// member's rows in and out of the [B, H G, ...] tensors and add a member's share onto the sums.  All only stream memory.  (Also here: the zero fill the pass needs when the softmax branch has queries
// and keys of its own, whose gradients are then tensors of their own.)
#include "nats_common.h"

namespace nats {

constexpr int HG_THREADS = 256;

// dst row r <- src row r (rows of row_vec 16-byte pieces, row strides in pieces)
__global__ __launch_bounds__(HG_THREADS) void copy_rows_kernel(const uint4* __restrict__ src, size_t src_stride,
                                                              uint4* __restrict__ dst, size_t dst_stride,
                                                              size_t row_vec, size_t n_rows) {
    const size_t n = row_vec * n_rows;
    for (size_t e = (size_t)blockIdx.x * HG_THREADS + threadIdx.x; e < n; e += (size_t)gridDim.x * HG_THREADS) {
        const size_t r = e / row_vec, c = e % row_vec;
        dst[r * dst_stride + c] = src[r * src_stride + c];
    }
}

// dst += src, n4 pieces of four floats
__global__ __launch_bounds__(HG_THREADS) void add_f32_kernel(float4* __restrict__ dst, const float4* __restrict__ src,
                                                            size_t n4) {
    for (size_t e = (size_t)blockIdx.x * HG_THREADS + threadIdx.x; e < n4; e += (size_t)gridDim.x * HG_THREADS) {
        float4 a = dst[e];
        const float4 b = src[e];
        a.x += b.x;
        a.y += b.y;
        a.z += b.z;
        a.w += b.w;
        dst[e] = a;
    }
}

// sum[h][i] = the G rows part[h G + g][i] in order; one gradient per blockIdx.y
constexpr int MAX_SUMS = 6;
struct GroupSums {
    GroupSum s[MAX_SUMS];
    int BH, G;
};
__global__ __launch_bounds__(HG_THREADS) void sum_groups_kernel(const GroupSums a) {
    const GroupSum s = a.s[blockIdx.y];
    const size_t at = (size_t)blockIdx.x * HG_THREADS + threadIdx.x, step = (size_t)gridDim.x * HG_THREADS;
    if (s.row % 4 == 0) {
        const size_t row = s.row / 4, n = row * a.BH;
        for (size_t e = at; e < n; e += step) {
            const float4* p = reinterpret_cast<const float4*>(s.part) + (e / row) * a.G * row + e % row;
            float4 x = p[0];
            for (int g = 1; g < a.G; ++g) {
                const float4 y = p[g * row];
                x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w;
            }
            if (s.rounded != nullptr) reinterpret_cast<uint2*>(s.rounded)[e] = make_uint2(pack_bf16x2(x.x, x.y), pack_bf16x2(x.z, x.w));
            else reinterpret_cast<float4*>(s.sum)[e] = x;
        }
    } else {   // a row per chunk, of any number of chunks
        const size_t n = s.row * a.BH;
        for (size_t e = at; e < n; e += step) {
            const float* p = s.part + (e / s.row) * a.G * s.row + e % s.row;
            float x = p[0];
            for (int g = 1; g < a.G; ++g) x += p[g * s.row];
            s.sum[e] = x;
        }
    }
}

constexpr int MAX_ROUNDINGS = 3;
struct Roundings {
    Rounding r[MAX_ROUNDINGS];
};
__global__ __launch_bounds__(HG_THREADS) void round_bf16_kernel(const Roundings a) {
    const Rounding r = a.r[blockIdx.y];
    const size_t n = r.n / 4;
    for (size_t e = (size_t)blockIdx.x * HG_THREADS + threadIdx.x; e < n; e += (size_t)gridDim.x * HG_THREADS) {
        const float4 x = reinterpret_cast<const float4*>(r.src)[e];
        reinterpret_cast<uint2*>(r.dst)[e] = make_uint2(pack_bf16x2(x.x, x.y), pack_bf16x2(x.z, x.w));
    }
}

// dst += src for any length and alignment
__global__ __launch_bounds__(HG_THREADS) void add_f32_scalar_kernel(float* __restrict__ dst, const float* __restrict__ src,
                                                                   size_t n) {
    for (size_t e = (size_t)blockIdx.x * HG_THREADS + threadIdx.x; e < n; e += (size_t)gridDim.x * HG_THREADS)
        dst[e] += src[e];
}

// dst[i] = 0 (a kernel, not a memset: the call may be part of a captured graph)
__global__ __launch_bounds__(HG_THREADS) void zero_f32_kernel(float* __restrict__ dst, size_t n) {
    for (size_t e = (size_t)blockIdx.x * HG_THREADS + threadIdx.x; e < n; e += (size_t)gridDim.x * HG_THREADS) dst[e] = 0.f;
}

static int hg_grid(size_t n) {
    const size_t blocks = (n + HG_THREADS - 1) / HG_THREADS;
    return (int)(blocks < 1 ? 1 : (blocks > 4096 ? 4096 : blocks));
}

// n_rows rows of row_bytes bytes (a multiple of 16; both buffers 16-byte aligned, strides in bytes, multiples of 16)
nats_status launch_copy_rows(const void* src, size_t src_stride_bytes, void* dst, size_t dst_stride_bytes,
                             size_t row_bytes, size_t n_rows, hipStream_t st) {
    if (row_bytes % 16 || src_stride_bytes % 16 || dst_stride_bytes % 16) {
        set_error("copy_rows: row size and strides must be multiples of 16 bytes");
        return NATS_ERR_SHAPE;
    }
    if (n_rows == 0 || row_bytes == 0) return NATS_OK;
    hipLaunchKernelGGL(copy_rows_kernel, dim3(hg_grid(row_bytes / 16 * n_rows)), dim3(HG_THREADS), 0, st,
                       (const uint4*)src, src_stride_bytes / 16, (uint4*)dst, dst_stride_bytes / 16, row_bytes / 16, n_rows);
    return check_launch("copy_rows");
}

// dst[i] += src[i], i < n
nats_status launch_add_f32(float* dst, const float* src, size_t n, hipStream_t st) {
    if (n == 0) return NATS_OK;
    const bool vec = n % 4 == 0 && (reinterpret_cast<uintptr_t>(dst) & 15u) == 0 && (reinterpret_cast<uintptr_t>(src) & 15u) == 0;
    if (vec)
        hipLaunchKernelGGL(add_f32_kernel, dim3(hg_grid(n / 4)), dim3(HG_THREADS), 0, st, (float4*)dst, (const float4*)src, n / 4);
    else
        hipLaunchKernelGGL(add_f32_scalar_kernel, dim3(hg_grid(n)), dim3(HG_THREADS), 0, st, dst, src, n);
    return check_launch("add_f32");
}

// part and sum 16-byte aligned (rows of a multiple of four floats are read and written 16 bytes at a time)
nats_status launch_sum_groups(int BH, int G, const GroupSum* sums, int n, hipStream_t st) {
    GroupSums a;
    a.BH = BH;
    a.G = G;
    int m = 0;
    size_t most = 0;
    for (int i = 0; i < n; ++i) {
        if (sums[i].sum == nullptr) continue;
        if (m == MAX_SUMS) { set_error("sum_groups: too many sums"); return NATS_ERR_SHAPE; }
        a.s[m++] = sums[i];
        if (sums[i].row > most) most = sums[i].row;
    }
    if (m == 0 || most == 0) return NATS_OK;
    hipLaunchKernelGGL(sum_groups_kernel, dim3(hg_grid(most * BH / 4), m), dim3(HG_THREADS), 0, st, a);
    return check_launch("sum_groups");
}

nats_status launch_round_bf16(const Rounding* r, int n, hipStream_t st) {
    Roundings a;
    int m = 0;
    size_t most = 0;
    for (int i = 0; i < n; ++i) {
        if (r[i].dst == nullptr || r[i].n == 0) continue;
        if (m == MAX_ROUNDINGS || r[i].n % 4 != 0) { set_error("round_bf16: too many arrays, or not of a multiple of four"); return NATS_ERR_SHAPE; }
        a.r[m++] = r[i];
        if (r[i].n > most) most = r[i].n;
    }
    if (m == 0) return NATS_OK;
    ProfScope ps("round_bf16", st);
    hipLaunchKernelGGL(round_bf16_kernel, dim3(hg_grid(most / 4), m), dim3(HG_THREADS), 0, st, a);
    return check_launch("round_bf16");
}

nats_status launch_zero_f32(float* dst, size_t n, hipStream_t st) {
    if (n == 0) return NATS_OK;
    hipLaunchKernelGGL(zero_f32_kernel, dim3(hg_grid(n)), dim3(HG_THREADS), 0, st, dst, n);
    return check_launch("zero_f32");
}

}  // namespace nats
