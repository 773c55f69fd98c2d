// attn_splitkv.h -- merge kernel of the split-KV forward launch.
//
// A split-KV launch runs the forward kernel once per key range; range s leaves a normalised partial
// output O_s (fp32) and its log-sum-exp LSE_s.  Softmax attention over the union of the ranges is
//     LSE = ln sum_s exp(LSE_s),    O = sum_s exp(LSE_s - LSE) O_s
// (the same rescaling that the online softmax applies tile by tile inside one workgroup).
#pragma once
#include "attn_common.h"

namespace attn {

constexpr int kMergeThreads = 256;

// lanes that share the ranges of one row: at least four ranges each (what one memory round trip brings)
inline int merge_lanes_log2(int D, int n_split)
{
    int l = 0;
    while ((8 << l) <= n_split && (2 << l) * (D / 4) <= kMergeThreads)
        ++l;
    return l;
}

// One row = D/4 threads (4 head-dimension elements each) times 2^lanes_log2 threads that take every 2^lanes_log2-th
// range, four at a time with their loads in flight together, and meet in LDS.  Reads n_split * (D + 1) floats per row:
// HBM-bound for many rows; for the few rows of a decode call the bound is latency, which is why the ranges of a row are
// not walked by one thread (D = 128: 16 rows of 64 ranges 36.8 -> 5.8 us, of 16 ranges 7.9 -> 4.1 us; 2048 rows of 32
// ranges 18.1 -> 10.2 us).
// OUT: bf16_t or _Float16, the element type of o.
template <int D, typename OUT>
__global__ __launch_bounds__(kMergeThreads) void attn_splitkv_merge_kernel(const float *__restrict__ o_part,
                                                                           const float *__restrict__ lse_part,
                                                                           OUT *__restrict__ o, float *__restrict__ lse,
                                                                           long long n_rows, int n_split, int lanes_log2)
{
    constexpr int TPR = D / 4, U = 4;
    __shared__ f32x4 s_acc[kMergeThreads];
    __shared__ f32x2 s_ml[kMergeThreads];
    const int sub = threadIdx.x % TPR;
    const int group = threadIdx.x / TPR;                 // (row of the block, lane of the row)
    const int lanes = 1 << lanes_log2, sl = group & (lanes - 1);
    const int rows_per_block = (kMergeThreads / TPR) >> lanes_log2;
    const long long n_blocks = (n_rows + rows_per_block - 1) / rows_per_block;
    for (long long b = blockIdx.x; b < n_blocks; b += gridDim.x) {
        const long long row = b * rows_per_block + (group >> lanes_log2);
        const long long r = row < n_rows ? row : n_rows - 1;
        // unnormalised weights against the lane's running maximum (lane sl < n_split has a range in its first step)
        float m = -INFINITY, sum = 0.f;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int s0 = sl; s0 < n_split; s0 += U * lanes) {
            float l[U];
            f32x4 x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int s = s0 + u * lanes;
                const long long i = (long long)(s < n_split ? s : n_split - 1) * n_rows + r;
                l[u] = lse_part[i];
                x[u] = *reinterpret_cast<const f32x4 *>(o_part + i * D + 4 * sub);
            }
            float m_new = m;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (s0 + u * lanes >= n_split)
                    l[u] = -INFINITY;
                m_new = fmaxf(m_new, l[u]);
            }
            const float keep = expf(m - m_new);
            sum *= keep;
            acc *= keep;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float w = expf(l[u] - m_new);
                sum += w;
                acc += w * x[u];
            }
            m = m_new;
        }
        if (lanes > 1) {
            s_acc[threadIdx.x] = acc;
            if (sub == 0)
                s_ml[group] = f32x2{m, sum};
            __syncthreads();
            if (sl == 0) {
                const float m_own = m;
                for (int j = 1; j < lanes; ++j)
                    m = fmaxf(m, s_ml[group + j][0]);
                const float keep = expf(m_own - m);
                sum *= keep;
                acc *= keep;
                for (int j = 1; j < lanes; ++j) {
                    const f32x2 ml = s_ml[group + j];
                    const float w = expf(ml[0] - m);
                    sum += w * ml[1];
                    acc += w * s_acc[threadIdx.x + j * TPR];
                }
            }
        }
        if (sl == 0 && row < n_rows) {
            acc *= 1.f / sum;
            const f32x2 lo = {acc[0], acc[1]}, hi = {acc[2], acc[3]};
            typedef OUT out2 __attribute__((ext_vector_type(2)));
            typedef OUT out4 __attribute__((ext_vector_type(4)));
            const out2 blo = __builtin_convertvector(lo, out2), bhi = __builtin_convertvector(hi, out2);  // RNE
            const out4 out = {blo[0], blo[1], bhi[0], bhi[1]};
            *reinterpret_cast<out4 *>(o + row * D + 4 * sub) = out;
            if (sub == 0)
                lse[row] = m + logf(sum);
        }
        if (lanes > 1)
            __syncthreads();   // the partials have been read
    }
}

}  // namespace attn
