// The graph layer around graph self-attention (Sec. 3.1 and Sec. 3.3, the update of the graph):
//   Z = norm(X + [head_1 .. head_H] Wo),   Y = norm(Z + max(0, Z W1 + b1) W2 + b2)
// for all 2n-1 nodes, forward and backward, and the loop over layers from the initial states
// (embeddings on the token rows, zero on the span rows) to the root or token rows of the last
// layer.  The dense maps are plain library GEMMs (hipBLASLt, rocBLAS for the weight gradients;
// bf16 operands, fp32 accumulation); attention is this library's own forward and backward on the
// [B][N][H][64] layout the projections produce (no transposes); residual + bias + layer
// normalisation, bias + ReLU, their backward counterparts and the fixed-order column sums are
// the small kernels below.
#include <hip/hip_runtime.h>
#include <hipblaslt/hipblaslt.h>
#include <rocblas/rocblas.h>

#include <algorithm>
#include <cstdlib>
#include <string>
#include <vector>

#include "bpt_internal.h"

namespace bpt {
namespace {

typedef uint16_t bf16_t;
constexpr int kLnMaxChunks = 4;   // 8-element chunks per lane: d <= 2048

__device__ __forceinline__ float bf16_to_f32(uint32_t bits16) { return __uint_as_float(bits16 << 16); }
__device__ __forceinline__ uint32_t f32_to_bf16(float f) { return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)f); }

// 8 consecutive fp32 parameters of a column chunk (any pointer: fp32 arrays of a multiple of 8 entries on a 16-byte
// boundary), zeros for a null array
__device__ __forceinline__ void load_params8(const float* __restrict__ p, int c, float* v) {
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    if (p) {
        a = *reinterpret_cast<const float4*>(p + c * 8);
        b = *reinterpret_cast<const float4*>(p + c * 8 + 4);
    }
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
// 8 bf16 of a 16-byte load as fp32
__device__ __forceinline__ void unpack8(const uint4& w, float* v) {
    const uint32_t x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[2 * e] = bf16_to_f32(x[e] & 0xFFFFu);
        v[2 * e + 1] = __uint_as_float(x[e] & 0xFFFF0000u);
    }
}

// y = norm(x + a + bias) * gain + beta, one wavefront per row; x bf16, a fp32 (the GEMM result of the
// sublayer), bias fp32 or null; the row stays in registers between the two passes (mean, then variance
// of the centred values: Ba et al., biased variance).  Bound by HBM (8 bytes per value).  A wavefront walks rows
// `wave, wave + waves, ...`, holds the parameters of its columns in registers and loads the next row before it
// works on the current one: with one row per wavefront the three parameter rows (6 KB at d = 512) were read from
// the caches for 4 KB of data (65 532 rows of 512: 61 -> 45 us, 6.0 TB/s; 15 000 rows: 16.9 -> 11.9 us).
template <int CHUNKS>   // 8-element chunks per lane: d <= 512 * CHUNKS
__global__ void __launch_bounds__(256) residual_layer_norm_kernel(const bf16_t* __restrict__ x, const float* __restrict__ a,
                                                                  const float* __restrict__ bias, const float* __restrict__ gain,
                                                                  const float* __restrict__ beta, bf16_t* __restrict__ y,
                                                                  float2* __restrict__ stats, int64_t rows, int d, float eps) {
    const int lane = threadIdx.x & 63;
    const int64_t stride = (int64_t)gridDim.x * 4;
    int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const int nchunk = d >> 3;
    constexpr bool kAhead = CHUNKS < kLnMaxChunks;   // (at 4 chunks a wavefront's row is 16 KB and its registers are full)
    float bi[CHUNKS][8], ga[CHUNKS][8], be[CHUNKS][8];
    uint4 xw[CHUNKS];
    float4 a0[CHUNKS], a1[CHUNKS];
    auto fetch = [&](int64_t r) {
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i) {
            const int c = lane + 64 * i;
            if (c < nchunk) {
                const int64_t at = r * d + c * 8;
                xw[i] = *reinterpret_cast<const uint4*>(x + at);
                a0[i] = *reinterpret_cast<const float4*>(a + at);
                a1[i] = *reinterpret_cast<const float4*>(a + at + 4);
            }
        }
    };
    if (kAhead) fetch(row);
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
        const int c = lane + 64 * i;
        if (c < nchunk) {
            load_params8(bias, c, bi[i]);
            load_params8(gain, c, ga[i]);
            load_params8(beta, c, be[i]);
        }
    }
    for (; row < rows; row += stride) {
        if (!kAhead) fetch(row);
        float v[CHUNKS][8];
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i)
            if (lane + 64 * i < nchunk) {
                const float av[8] = {a0[i].x, a0[i].y, a0[i].z, a0[i].w, a1[i].x, a1[i].y, a1[i].z, a1[i].w};
                unpack8(xw[i], v[i]);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    v[i][e] = v[i][e] + av[e] + bi[i][e];
                    sum += v[i][e];
                }
            }
        if (kAhead && row + stride < rows) fetch(row + stride);
#pragma unroll
        for (int s = 1; s < 64; s <<= 1) sum += __shfl_xor(sum, s);
        const float mean = sum / (float)d;
        float sq = 0.f;
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i)
            if (lane + 64 * i < nchunk)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    v[i][e] -= mean;
                    sq += v[i][e] * v[i][e];
                }
#pragma unroll
        for (int s = 1; s < 64; s <<= 1) sq += __shfl_xor(sq, s);
        const float inv = rsqrtf(sq / (float)d + eps);
        if (lane == 0) stats[row] = make_float2(mean, inv);   // what the backward normalises the row with
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i) {
            const int c = lane + 64 * i;
            if (c < nchunk) {
                uint32_t o[4];
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    const float y0 = v[i][e] * inv * ga[i][e] + be[i][e];
                    const float y1 = v[i][e + 1] * inv * ga[i][e + 1] + be[i][e + 1];
                    o[e >> 1] = f32_to_bf16(y0) | (f32_to_bf16(y1) << 16);
                }
                *reinterpret_cast<uint4*>(y + row * d + c * 8) = make_uint4(o[0], o[1], o[2], o[3]);
            }
        }
    }
}

// f = max(0, f + b) in place on [rows][cols] bf16, 8 values per thread (cols a multiple of 8)
__global__ void __launch_bounds__(256) bias_relu_kernel(bf16_t* __restrict__ f, const float* __restrict__ b, int64_t chunks,
                                                        int cols) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= chunks) return;
    const int col = (int)((i * 8) % cols);
    uint4 w = *reinterpret_cast<uint4*>(f + i * 8);
    uint32_t x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float lo = fmaxf(bf16_to_f32(x[e] & 0xFFFFu) + b[col + 2 * e], 0.f);
        const float hi = fmaxf(__uint_as_float(x[e] & 0xFFFF0000u) + b[col + 2 * e + 1], 0.f);
        x[e] = f32_to_bf16(lo) | (f32_to_bf16(hi) << 16);
    }
    *reinterpret_cast<uint4*>(f + i * 8) = make_uint4(x[0], x[1], x[2], x[3]);
}

// first token of a node of the tree over n = 2^lg tokens (ids are level-major)
__device__ __forceinline__ int first_token_of(int id, int lg) {
    const int x = (2 << lg) - id;
    const int level = lg - (31 - __clz(x - 1));
    return (((2 << lg) >> level) - x) << level;
}

// Backward of y = norm(s) * gain + beta with s = x + a + bias (as residual_layer_norm_kernel formed it;
// `stats` = its (mean, 1/deviation) per row):  dxh = dy * gain,
//   ds = (dxh - mean(dxh) - xh * mean(dxh * xh)) / deviation,   xh = (s - mean) / deviation,
// with dy = dy_b (bf16) + dy_f (fp32, may be null).  ds is written in bf16.  A wavefront walks rows
// `wave, wave + waves, ...` and keeps the column sums of dy * xh (gain), dy (beta) and ds (the bias
// inside s) of its rows in registers; the four wavefronts of a workgroup add theirs in a fixed order
// and the workgroup writes one row of `partials` [gridDim.x][3][d].  With seq_len, rows of nodes the
// sequence does not keep count as dy = 0.  Bound by HBM (10 bytes per value); the parameters of a lane's columns
// stay in registers and the next row is loaded before the current one's sums are exchanged; 1024 workgroups, as
// many as are resident, halve the partial rows (65 532 rows of 512: 113 -> 61 us, 5.5 TB/s; 15 000 rows: 34 -> 19 us).
template <int CHUNKS>   // 8-element chunks per lane: d <= 512 * CHUNKS
__global__ void __launch_bounds__(256) layer_norm_bwd_kernel(const bf16_t* __restrict__ dy_b, const float* __restrict__ dy_f,
                                                             const bf16_t* __restrict__ x, const float* __restrict__ a,
                                                             const float* __restrict__ bias, const float* __restrict__ gain,
                                                             const float2* __restrict__ stats, bf16_t* __restrict__ ds,
                                                             float* __restrict__ partials, int64_t rows, int d,
                                                             const int32_t* __restrict__ seq_len, int N, int lg) {
    extern __shared__ float red_s[];   // wavefronts 1..3: [wavefront - 1][sum][d columns]
    auto red = [&](int w, int which, int col) -> float& { return red_s[(w * 3 + which) * d + col]; };
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nchunk = d >> 3;
    float sg[CHUNKS][8], sb[CHUNKS][8], ss[CHUNKS][8];
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) sg[i][e] = sb[i][e] = ss[i][e] = 0.f;
    const int64_t stride = (int64_t)gridDim.x * 4;
    constexpr bool kAhead = CHUNKS < kLnMaxChunks;   // as in the forward
    float bi[CHUNKS][8], ga[CHUNKS][8];
    uint4 xw[CHUNKS], gw[CHUNKS];
    float4 a0[CHUNKS], a1[CHUNKS];
    float2 st_next = make_float2(0.f, 0.f);
    auto fetch = [&](int64_t r) {
        st_next = stats[r];
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i) {
            const int c = lane + 64 * i;
            if (c < nchunk) {
                const int64_t at = r * d + c * 8;
                xw[i] = *reinterpret_cast<const uint4*>(x + at);
                gw[i] = *reinterpret_cast<const uint4*>(dy_b + at);
                a0[i] = *reinterpret_cast<const float4*>(a + at);
                a1[i] = *reinterpret_cast<const float4*>(a + at + 4);
            }
        }
    };
    int64_t row = (int64_t)blockIdx.x * 4 + wave;
    if (kAhead && row < rows) fetch(row);
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
        const int c = lane + 64 * i;
        if (c < nchunk) {
            load_params8(bias, c, bi[i]);
            load_params8(gain, c, ga[i]);
        }
    }
    for (; row < rows; row += stride) {
        if (!kAhead) fetch(row);
        bool kept = true;
        if (seq_len) {
            const int b = (int)(row / N), node = (int)(row - (int64_t)b * N);
            kept = first_token_of(node, lg) < min(max(seq_len[b], 0), 1 << lg);
        }
        const float2 st = st_next;
        float xh[CHUNKS][8], dxh[CHUNKS][8];
        float m1 = 0.f, m2 = 0.f;
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i) {
            const int c = lane + 64 * i;
            if (c < nchunk) {
                float f[8], xv[8], gv[8];
                load_params8(dy_f ? dy_f + row * d : nullptr, c, f);
                unpack8(xw[i], xv);
                unpack8(gw[i], gv);
                const float av[8] = {a0[i].x, a0[i].y, a0[i].z, a0[i].w, a1[i].x, a1[i].y, a1[i].z, a1[i].w};
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float dye = kept ? gv[e] + f[e] : 0.f;
                    const float s = xv[e] + av[e] + bi[i][e];
                    xh[i][e] = (s - st.x) * st.y;
                    dxh[i][e] = dye * ga[i][e];
                    m1 += dxh[i][e];
                    m2 += dxh[i][e] * xh[i][e];
                    sg[i][e] += dye * xh[i][e];
                    sb[i][e] += dye;
                }
            }
        }
        if (kAhead && row + stride < rows) fetch(row + stride);
#pragma unroll
        for (int s = 1; s < 64; s <<= 1) {
            m1 += __shfl_xor(m1, s);
            m2 += __shfl_xor(m2, s);
        }
        m1 /= (float)d;
        m2 /= (float)d;
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i) {
            const int c = lane + 64 * i;
            if (c < nchunk) {
                uint32_t o[4];
                float r[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    r[e] = st.y * (dxh[i][e] - m1 - xh[i][e] * m2);
                    ss[i][e] += r[e];
                }
#pragma unroll
                for (int e = 0; e < 8; e += 2) o[e >> 1] = f32_to_bf16(r[e]) | (f32_to_bf16(r[e + 1]) << 16);
                *reinterpret_cast<uint4*>(ds + row * d + c * 8) = make_uint4(o[0], o[1], o[2], o[3]);
            }
        }
    }
    // wavefronts 1..3 hand their sums to wavefront 0, which adds them in order and writes the workgroup's row
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
        const int c = lane + 64 * i;
        if (c < nchunk && wave > 0)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                red(wave - 1, 0, c * 8 + e) = sg[i][e];
                red(wave - 1, 1, c * 8 + e) = sb[i][e];
                red(wave - 1, 2, c * 8 + e) = ss[i][e];
            }
    }
    __syncthreads();
    if (wave == 0) {
        float* out = partials + (int64_t)blockIdx.x * 3 * d;
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i) {
            const int c = lane + 64 * i;
            if (c < nchunk)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int col = c * 8 + e;
                    out[col] = ((sg[i][e] + red(0, 0, col)) + red(1, 0, col)) + red(2, 0, col);
                    out[d + col] = ((sb[i][e] + red(0, 1, col)) + red(1, 1, col)) + red(2, 1, col);
                    out[2 * d + col] = ((ss[i][e] + red(0, 2, col)) + red(1, 2, col)) + red(2, 2, col);
                }
        }
    }
}

// Backward of f = max(0, h): df *= (f > 0) in place on [rows][cols] bf16 (f is the stored output of
// bias_relu_kernel), and the column sums of the result (the gradient of the bias) of the rows
// `blockIdx.x, blockIdx.x + gridDim.x, ...` into partials[gridDim.x][cols].  A thread owns up to
// kReluChunks chunks of 8 columns.
constexpr int kReluChunks = 4;   // cols <= 8 * 256 * 4
__global__ void __launch_bounds__(256) relu_bwd_kernel(bf16_t* __restrict__ df, const bf16_t* __restrict__ f,
                                                       float* __restrict__ partials, int64_t rows, int cols) {
    const int nchunk = cols >> 3;
    float acc[kReluChunks][8];
#pragma unroll
    for (int i = 0; i < kReluChunks; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[i][e] = 0.f;
    for (int64_t row = blockIdx.x; row < rows; row += gridDim.x) {
#pragma unroll
        for (int i = 0; i < kReluChunks; ++i) {
            const int c = threadIdx.x + 256 * i;
            if (c < nchunk) {
                const int64_t at = row * cols + c * 8;
                const uint4 gw = *reinterpret_cast<const uint4*>(df + at);
                const uint4 fw = *reinterpret_cast<const uint4*>(f + at);
                uint32_t gv[4] = {gw.x, gw.y, gw.z, gw.w};
                const uint32_t fv[4] = {fw.x, fw.y, fw.z, fw.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // the stored activations are >= 0: positive iff the bits below the sign are not all zero
                    if ((fv[e] & 0x7FFFu) == 0u) gv[e] &= 0xFFFF0000u;
                    if ((fv[e] & 0x7FFF0000u) == 0u) gv[e] &= 0x0000FFFFu;
                    acc[i][2 * e] += bf16_to_f32(gv[e] & 0xFFFFu);
                    acc[i][2 * e + 1] += __uint_as_float(gv[e] & 0xFFFF0000u);
                }
                *reinterpret_cast<uint4*>(df + at) = make_uint4(gv[0], gv[1], gv[2], gv[3]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < kReluChunks; ++i) {
        const int c = threadIdx.x + 256 * i;
        if (c < nchunk) {
            float* out = partials + (int64_t)blockIdx.x * cols + c * 8;
            *reinterpret_cast<float4*>(out) = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
            *reinterpret_cast<float4*>(out + 4) = make_float4(acc[i][4], acc[i][5], acc[i][6], acc[i][7]);
        }
    }
}

// Column sums of partials[num_parts][cols] in a fixed order: a workgroup takes 32 columns (a cache line of every row),
// 8 lanes per row and 16 bytes per lane, each of its 128 groups of lanes with 8 rows in flight; the groups' sums are
// added across the lanes of a wavefront, then across the wavefronts, in a fixed tree.  (64 columns per workgroup, a
// row per wavefront, four 4-byte loads in flight: 24 workgroups and 12.5 us for 2048 x 1536; now 5.4 us for 1024 x
// 1536, the partial rows there are of a normalisation.)
// Column c goes to out[c / cols_each][c % cols_each] (up to three outputs whose partial sums sit side by side in a
// row; a null output is skipped); cols and cols_each are multiples of 4.
struct ColumnSumOut {
    float* out[3];
    int cols_each;
};
constexpr int kColumnSumCols = 32;
__global__ void __launch_bounds__(1024) column_sum_kernel(const float* __restrict__ partials, int num_parts, int cols,
                                                          const ColumnSumOut o) {
    __shared__ float s[16][kColumnSumCols];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = blockIdx.x * kColumnSumCols + (lane & 7) * 4;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    if (c < cols) {
        const float* src = partials + c;
        for (int p0 = threadIdx.x >> 3; p0 < num_parts; p0 += 8 * 128) {
            float4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int p = p0 + 128 * j;
                v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (p < num_parts) v[j] = *reinterpret_cast<const float4*>(src + (int64_t)p * cols);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                acc[0] += v[j].x;
                acc[1] += v[j].y;
                acc[2] += v[j].z;
                acc[3] += v[j].w;
            }
        }
    }
#pragma unroll
    for (int w = 8; w < 64; w <<= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], w);
    if (lane < 8)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[wave][lane * 4 + e] = acc[e];
    __syncthreads();
    for (int w = 8; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w * kColumnSumCols) {
            const int g = threadIdx.x / kColumnSumCols, e = threadIdx.x % kColumnSumCols;
            s[g][e] += s[g + w][e];
        }
        __syncthreads();
    }
    const int col = blockIdx.x * kColumnSumCols + threadIdx.x;
    if (threadIdx.x < kColumnSumCols && col < cols && o.out[col / o.cols_each])
        o.out[col / o.cols_each][col % o.cols_each] = s[0][threadIdx.x];
}

// out[i] = sum over s of slices[s][i] in slice order, 4 values per thread: the partial products of a
// GEMM C = A^T B whose contraction was cut into slices.  Element i belongs to row i / cols; its columns go to
// out[col / cols_each] (row pitch cols_each): up to three matrices computed side by side.  The `left` rows of the
// contraction that the equal slices leave over (fewer than there are slices) are multiplied here, into the first
// slice's sum: left_a, left_b are their rows of A and B (bf16, lda and ldb elements apart).  As a product of its own
// of depth 1..15 they cost a GEMM launch (5.6 - 7.7 us).
__global__ void __launch_bounds__(256) sum_slices_kernel(const float* __restrict__ slices, int num_slices, int64_t elems,
                                                         int cols, const ColumnSumOut o, const bf16_t* __restrict__ left_a,
                                                         const bf16_t* __restrict__ left_b, int left, int64_t lda, int64_t ldb) {
    const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (i >= elems) return;
    const int64_t row = i / cols;
    const int col = (int)(i - row * cols);
    float4 acc = *reinterpret_cast<const float4*>(slices + i);
    for (int r = 0; r < left; ++r) {
        const float av = bf16_to_f32(left_a[r * lda + row]);
        const uint2 b = *reinterpret_cast<const uint2*>(left_b + r * ldb + col);
        acc.x = fmaf(av, bf16_to_f32(b.x & 0xFFFFu), acc.x);
        acc.y = fmaf(av, __uint_as_float(b.x & 0xFFFF0000u), acc.y);
        acc.z = fmaf(av, bf16_to_f32(b.y & 0xFFFFu), acc.z);
        acc.w = fmaf(av, __uint_as_float(b.y & 0xFFFF0000u), acc.w);
    }
    for (int sl = 1; sl < num_slices; ++sl) {
        const float4 x = *reinterpret_cast<const float4*>(slices + (int64_t)sl * elems + i);
        acc.x += x.x; acc.y += x.y; acc.z += x.z; acc.w += x.w;
    }
    *reinterpret_cast<float4*>(o.out[col / o.cols_each] + row * o.cols_each + col % o.cols_each) = acc;
}

// dst (bf16) [d][3 d] = Wq | Wk | Wv ([d][d] each) side by side, 8 values per thread; blockIdx.y picks the matrix.
// One projection X [Wq | Wk | Wv] then reads X once and gives the three results side by side.
struct PackArgs {
    const bf16_t* src[3];
    bf16_t* dst;
};
__global__ void __launch_bounds__(256) pack_qkv_weights_kernel(const PackArgs t, int64_t chunks, int d) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= chunks) return;
    const int64_t row = (i * 8) / d;
    const int col = (int)(i * 8 - row * d);
    *reinterpret_cast<uint4*>(t.dst + row * 3 * d + (int64_t)blockIdx.y * d + col) =
        *reinterpret_cast<const uint4*>(t.src[blockIdx.y] + i * 8);
}

// y (bf16) = x (bf16) + a (fp32), 8 values per thread
__global__ void __launch_bounds__(256) add_cast_kernel(const bf16_t* __restrict__ x, const float* __restrict__ a,
                                                       bf16_t* __restrict__ y, int64_t chunks) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= chunks) return;
    const uint4 xw = *reinterpret_cast<const uint4*>(x + i * 8);
    const float4 a0 = *reinterpret_cast<const float4*>(a + i * 8), a1 = *reinterpret_cast<const float4*>(a + i * 8 + 4);
    const uint32_t w[4] = {xw.x, xw.y, xw.z, xw.w};
    const float av[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
    uint32_t o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
        o[e] = f32_to_bf16(bf16_to_f32(w[e] & 0xFFFFu) + av[2 * e]) |
               (f32_to_bf16(__uint_as_float(w[e] & 0xFFFF0000u) + av[2 * e + 1]) << 16);
    *reinterpret_cast<uint4*>(y + i * 8) = make_uint4(o[0], o[1], o[2], o[3]);
}

// Sec. 3.3, the states before the first layer: token nodes start from their embeddings, span nodes from
// zero.  e: [B][n][d], h: [B][N][d], 8 values per thread.
__global__ void __launch_bounds__(256) initial_states_kernel(const bf16_t* __restrict__ e, bf16_t* __restrict__ h, int64_t chunks,
                                                             int n, int N, int row_chunks) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= chunks) return;
    const int64_t row = i / row_chunks;
    const int c = (int)(i - row * row_chunks), v = (int)(row % N);
    const int64_t b = row / N;
    uint4 x = make_uint4(0u, 0u, 0u, 0u);
    if (v < n) x = *reinterpret_cast<const uint4*>(e + ((b * n + v) * row_chunks + c) * 8);
    *reinterpret_cast<uint4*>(h + i * 8) = x;
}

// Sec. 3.3, the output: the roots' rows and / or the token rows of h [B][N][d], to root [B][R][d] and tokens
// [B][n][d] (either may be null).  One thread per 8 values of the rows that are read.  A tree has one root, its
// last row (R = 1, root_row null); the graph of a packed batch has one per sequence, root_row[r] (-1: an empty
// sequence, whose output is zero).
__global__ void __launch_bounds__(256) readout_kernel(const bf16_t* __restrict__ h, bf16_t* __restrict__ root,
                                                      bf16_t* __restrict__ tokens, int64_t chunks, int n, int N, int row_chunks,
                                                      int R, const int32_t* __restrict__ root_row) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= chunks) return;
    const int64_t row = i / row_chunks;   // over [B][n + R]: the tokens, then the roots
    const int c = (int)(i - row * row_chunks), v = (int)(row % (n + R));
    const int64_t b = row / (n + R);
    bf16_t* dst = v < n ? tokens : root;
    if (!dst) return;
    const int src = v < n ? v : root_row ? root_row[v - n] : N - 1;
    uint4 x = make_uint4(0u, 0u, 0u, 0u);
    if (src >= 0) x = *reinterpret_cast<const uint4*>(h + ((b * N + src) * row_chunks + c) * 8);
    *reinterpret_cast<uint4*>(dst + ((v < n ? b * n + v : b * R + (v - n)) * row_chunks + c) * 8) = x;
}

// the reverse: the gradient with respect to the last states is d_tokens on the token rows, d_root on the
// root's row (a null one counts as zero) and zero on every other row
// (first_root: the first root row -- N - 1 for a tree; root_seq: for the graph of a packed batch, the sequence of
// every row from first_root on, else null)
__global__ void __launch_bounds__(256) readout_bwd_kernel(const bf16_t* __restrict__ d_root, const bf16_t* __restrict__ d_tokens,
                                                          bf16_t* __restrict__ dh, int64_t chunks, int n, int N, int row_chunks,
                                                          int R, int first_root, const int32_t* __restrict__ root_seq) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= chunks) return;
    const int64_t row = i / row_chunks;
    const int c = (int)(i - row * row_chunks), v = (int)(row % N);
    const int64_t b = row / N;
    uint4 x = make_uint4(0u, 0u, 0u, 0u);
    if (v < n && d_tokens) x = *reinterpret_cast<const uint4*>(d_tokens + ((b * n + v) * row_chunks + c) * 8);
    if (v >= first_root && d_root) {
        const int r = root_seq ? root_seq[v - first_root] : 0;
        x = *reinterpret_cast<const uint4*>(d_root + ((b * R + r) * row_chunks + c) * 8);
    }
    *reinterpret_cast<uint4*>(dh + i * 8) = x;
}

// one rocBLAS handle per host thread and device, created on first use and kept: a handle carries the
// stream of the call in progress, so two host threads must not share one
rocblas_handle blas_handle(int device) {
    thread_local rocblas_handle handles[64] = {};
    if (device < 0 || device >= 64) return nullptr;
    if (!handles[device] && rocblas_create_handle(&handles[device]) != rocblas_status_success) handles[device] = nullptr;
    return handles[device];
}

// C[M][N] = beta C + op(A) op(B), row-major, bf16 operands, fp32 accumulation; C bf16 or fp32.
// op(A) is [M][K]: A is stored [M][K], or [K][M] with ta; op(B) is [K][N]: B is stored [K][N], or [N][K]
// with tb.  rocBLAS is column-major: C^T = op(B)^T op(A)^T with the same buffers, a row-major
// [r][c] buffer being the column-major c x r matrix with leading dimension c.
int gemm_rm(rocblas_handle h, int64_t M, int64_t N, int64_t K, const void* A, bool ta, const void* B, bool tb, void* C,
            bool c_fp32, float beta = 0.f, int64_t lda = 0, int64_t ldc = 0) {   // lda, ldc: elements between rows of A, C as stored (0: dense)
    const float one = 1.f;
    const rocblas_datatype ct = c_fp32 ? rocblas_datatype_f32_r : rocblas_datatype_bf16_r;
    const rocblas_int ldc_ = (rocblas_int)(ldc ? ldc : N);
    const rocblas_status st = rocblas_gemm_ex(
        h, tb ? rocblas_operation_transpose : rocblas_operation_none, ta ? rocblas_operation_transpose : rocblas_operation_none,
        (rocblas_int)N, (rocblas_int)M, (rocblas_int)K, &one, B, rocblas_datatype_bf16_r, (rocblas_int)(tb ? K : N), A,
        rocblas_datatype_bf16_r, (rocblas_int)(lda ? lda : (ta ? M : K)), &beta, C, ct, ldc_, C, ct, ldc_,
        rocblas_datatype_f32_r, rocblas_gemm_algo_standard, 0, 0);
    return st == rocblas_status_success ? BPT_OK : BPT_ERR_LAUNCH;
}

// The same product through hipBLASLt, whose epilogue can add a bias row and apply the ReLU while the sums are
// still fp32 in registers (Sec. 3.1 eq. (3): max(0, Z W1 + b1) without a pass of its own), and whose kernel
// choice for the tall products of the layer (65 532 x 512..2048) is 5-15 % faster than the one behind
// rocblas_gemm_ex.  A plan (descriptor, layouts, algorithm) per distinct product, made on first use and kept,
// per host thread and device like the rocBLAS handle; the first use of a product must therefore lie outside a
// stream capture.  A product hipBLASLt has no algorithm for reports false and the caller takes the rocBLAS path.
struct LtPlan {
    int64_t M, N, K, lda, ldc;
    bool ta, tb, c_fp32, bias_relu, add;
    hipblasLtMatmulDesc_t desc;
    hipblasLtMatrixLayout_t la, lb, lc;
    hipblasLtMatmulAlgo_t algo;
    size_t ws_bytes;
};
struct LtContext {
    hipblasLtHandle_t handle = nullptr;
    void* ws = nullptr;               // the algorithms' scratch memory, kept until the process ends
    std::vector<LtPlan> plans;
    bool failed = false;
};
constexpr size_t kLtWorkspace = (size_t)32 << 20;
constexpr int kLtCandidates = 12, kLtTimedRuns = 3;
LtContext* lt_context(int device) {
    thread_local LtContext ctx[64];
    if (device < 0 || device >= 64) return nullptr;
    LtContext& c = ctx[device];
    if (c.failed) return nullptr;
    if (!c.handle) {
        if (hipblasLtCreate(&c.handle) != HIPBLAS_STATUS_SUCCESS || hipMalloc(&c.ws, kLtWorkspace) != hipSuccess) {
            c.failed = true;
            (void)hipGetLastError();
            return nullptr;
        }
    }
    return &c;
}
// C[M][N] = op(A) op(B) (+ bias[N], then max(0, .) with bias_relu; + add[M][N], of C's type and row stride, with add:
// the sum is formed in fp32 and rounded once), arguments as gemm_rm's with beta = 0
bool gemm_lt(int device, hipStream_t st, int64_t M, int64_t N, int64_t K, const void* A, bool ta, const void* B, bool tb, void* C,
             bool c_fp32, int64_t lda, int64_t ldc, const float* bias_relu, const void* add) {
    LtContext* c = lt_context(device);
    if (!c) return false;
    const int64_t lda_ = lda ? lda : (ta ? M : K), ldc_ = ldc ? ldc : N;
    LtPlan* plan = nullptr;
    for (LtPlan& q : c->plans)
        if (q.M == M && q.N == N && q.K == K && q.lda == lda_ && q.ldc == ldc_ && q.ta == ta && q.tb == tb && q.c_fp32 == c_fp32 &&
            q.bias_relu == (bias_relu != nullptr) && q.add == (add != nullptr)) {
            plan = &q;
            break;
        }
    if (!plan) {
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) return false;
        LtPlan q = {M, N, K, lda_, ldc_, ta, tb, c_fp32, bias_relu != nullptr, add != nullptr, nullptr, nullptr, nullptr, nullptr, {}, 0};
        // column-major view: C^T [N x M] = op(B)^T [N x K] op(A)^T [K x M] on the same buffers
        const hipblasOperation_t op_first = tb ? HIPBLAS_OP_T : HIPBLAS_OP_N, op_second = ta ? HIPBLAS_OP_T : HIPBLAS_OP_N;
        const hipDataType ctype = c_fp32 ? HIP_R_32F : HIP_R_16BF;
        bool ok = hipblasLtMatmulDescCreate(&q.desc, HIPBLAS_COMPUTE_32F, HIP_R_32F) == HIPBLAS_STATUS_SUCCESS;
        ok = ok && hipblasLtMatmulDescSetAttribute(q.desc, HIPBLASLT_MATMUL_DESC_TRANSA, &op_first, sizeof(op_first)) == HIPBLAS_STATUS_SUCCESS;
        ok = ok && hipblasLtMatmulDescSetAttribute(q.desc, HIPBLASLT_MATMUL_DESC_TRANSB, &op_second, sizeof(op_second)) == HIPBLAS_STATUS_SUCCESS;
        if (ok && bias_relu) {
            const hipblasLtEpilogue_t epi = HIPBLASLT_EPILOGUE_RELU_BIAS;
            const hipDataType btype = HIP_R_32F;
            ok = hipblasLtMatmulDescSetAttribute(q.desc, HIPBLASLT_MATMUL_DESC_EPILOGUE, &epi, sizeof(epi)) == HIPBLAS_STATUS_SUCCESS &&
                 hipblasLtMatmulDescSetAttribute(q.desc, HIPBLASLT_MATMUL_DESC_BIAS_DATA_TYPE, &btype, sizeof(btype)) == HIPBLAS_STATUS_SUCCESS &&
                 hipblasLtMatmulDescSetAttribute(q.desc, HIPBLASLT_MATMUL_DESC_BIAS_POINTER, &bias_relu, sizeof(bias_relu)) == HIPBLAS_STATUS_SUCCESS;
        }
        ok = ok && hipblasLtMatrixLayoutCreate(&q.la, HIP_R_16BF, tb ? K : N, tb ? N : K, tb ? K : N) == HIPBLAS_STATUS_SUCCESS;
        ok = ok && hipblasLtMatrixLayoutCreate(&q.lb, HIP_R_16BF, ta ? M : K, ta ? K : M, lda_) == HIPBLAS_STATUS_SUCCESS;
        ok = ok && hipblasLtMatrixLayoutCreate(&q.lc, ctype, N, M, ldc_) == HIPBLAS_STATUS_SUCCESS;
        hipblasLtMatmulPreference_t pref = nullptr;
        ok = ok && hipblasLtMatmulPreferenceCreate(&pref) == HIPBLAS_STATUS_SUCCESS;
        ok = ok && hipblasLtMatmulPreferenceSetAttribute(pref, HIPBLASLT_MATMUL_PREF_MAX_WORKSPACE_BYTES, &kLtWorkspace, sizeof(kLtWorkspace)) == HIPBLAS_STATUS_SUCCESS;
        hipblasLtMatmulHeuristicResult_t res[kLtCandidates];
        int found = 0;
        ok = ok && hipblasLtMatmulAlgoGetHeuristic(c->handle, q.desc, q.la, q.lb, q.lc, q.lc, pref, kLtCandidates, res, &found) ==
                       HIPBLAS_STATUS_SUCCESS;
        if (pref) hipblasLtMatmulPreferenceDestroy(pref);
        // the library's candidates, timed on the caller's own buffers (beta = 0: what they write is overwritten by
        // the product proper); the fastest is kept for this process
        int best = -1;
        float best_ms = 0.f;
        hipEvent_t e0 = nullptr, e1 = nullptr;
        if (ok && found > 1 && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)) found = 1;
        const float one = 1.f, beta = add ? 1.f : 0.f;
        const void* cin = add ? add : C;
        for (int i = 0; ok && i < found; ++i) {
            if (res[i].state != HIPBLAS_STATUS_SUCCESS || res[i].workspaceSize > kLtWorkspace) continue;
            if (found == 1) {
                best = i;
                break;
            }
            bool ran = true;
            for (int rep = 0; rep < kLtTimedRuns + 1 && ran; ++rep) {   // the first run is not timed
                if (rep == 1) ran = hipEventRecord(e0, st) == hipSuccess;
                ran = ran && hipblasLtMatmul(c->handle, q.desc, &one, B, q.la, A, q.lb, &beta, cin, q.lc, C, q.lc, &res[i].algo, c->ws,
                                             kLtWorkspace, st) == HIPBLAS_STATUS_SUCCESS;
            }
            float ms = 0.f;
            ran = ran && hipEventRecord(e1, st) == hipSuccess && hipEventSynchronize(e1) == hipSuccess &&
                  hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
            if (ran && (best < 0 || ms < best_ms)) {
                best = i;
                best_ms = ms;
            }
        }
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
        ok = ok && best >= 0;
        if (ok) {
            q.algo = res[best].algo;
            q.ws_bytes = res[best].workspaceSize;
        } else {   // remembered as a product to leave to rocBLAS
            if (q.lc) hipblasLtMatrixLayoutDestroy(q.lc);
            if (q.lb) hipblasLtMatrixLayoutDestroy(q.lb);
            if (q.la) hipblasLtMatrixLayoutDestroy(q.la);
            if (q.desc) hipblasLtMatmulDescDestroy(q.desc);
            q.desc = nullptr;
        }
        c->plans.push_back(q);
        plan = &c->plans.back();
    }
    if (!plan->desc) return false;
    if (bias_relu && hipblasLtMatmulDescSetAttribute(plan->desc, HIPBLASLT_MATMUL_DESC_BIAS_POINTER, &bias_relu, sizeof(bias_relu)) !=
                         HIPBLAS_STATUS_SUCCESS)
        return false;
    const float one = 1.f, beta = add ? 1.f : 0.f;
    return hipblasLtMatmul(c->handle, plan->desc, &one, B, plan->la, A, plan->lb, &beta, add ? add : C, plan->lc, C, plan->lc,
                           &plan->algo, c->ws, kLtWorkspace, st) == HIPBLAS_STATUS_SUCCESS;
}

// the dense products of the layer: hipBLASLt where it has an algorithm (always, with the bias + ReLU epilogue or
// without), else rocBLAS (and the caller's own bias + ReLU kernel: *fused says which).  BPT_LAYER_BLAS=rocblas in
// the environment keeps everything on rocBLAS (for comparisons).
struct Blas {
    rocblas_handle h;
    int device;
    hipStream_t st;
};
bool lt_enabled() {   // read at every call: a process can compare the two paths
    const char* e = getenv("BPT_LAYER_BLAS");
    return !(e && std::string(e) == "rocblas");
}
int gemm(const Blas& b, int64_t M, int64_t N, int64_t K, const void* A, bool ta, const void* B, bool tb, void* C, bool c_fp32,
         int64_t lda = 0, int64_t ldc = 0, const float* bias_relu = nullptr, bool* fused = nullptr) {
    if (fused) *fused = false;
    if (lt_enabled() && gemm_lt(b.device, b.st, M, N, K, A, ta, B, tb, C, c_fp32, lda, ldc, bias_relu, nullptr)) {
        if (fused) *fused = true;
        return BPT_OK;
    }
    return gemm_rm(b.h, M, N, K, A, ta, B, tb, C, c_fp32, 0.f, lda, ldc);
}
// C (bf16) = add (bf16) + op(A) op(B) in one product where hipBLASLt has it; else false and nothing is written
bool gemm_add(const Blas& b, int64_t M, int64_t N, int64_t K, const void* A, bool ta, const void* B, bool tb, void* C,
              const void* add, int64_t lda = 0) {
    return lt_enabled() && gemm_lt(b.device, b.st, M, N, K, A, ta, B, tb, C, false, lda, 0, nullptr, add);
}

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }
// the kernels here move 16 bytes per lane: every tensor has to start on a 16-byte boundary (null passes: optional
// arguments are checked where they are used)
template <typename... P>
bool any_misaligned(P... p) {
    const uintptr_t bits = (... | reinterpret_cast<uintptr_t>(static_cast<const void*>(p)));
    return (bits & 15u) != 0;
}

struct LayerBuffers {
    size_t qkvo, wqkv, lse, acc1, acc2, st1, st2, z, f1, attn, total;
};
LayerBuffers layer_buffers(const bpt_graph* g, int B, int H, int d_ff, size_t attn_ws) {
    const size_t rows = (size_t)B * g->num_nodes, d = (size_t)H * kD;
    LayerBuffers L;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align_up(bytes);
        return at;
    };
    L.qkvo = take(rows * 4 * d * 2);   // [rows][Q | K | V | O]: the projections side by side, then the attention's output
    L.wqkv = take(d * 3 * d * 2);      // [d][Wq | Wk | Wv]
    L.lse = take((size_t)B * H * g->num_nodes * 4);
    L.acc1 = take(rows * d * 4);     // W^O result, fp32
    L.acc2 = take(rows * d * 4);     // W_2 result, fp32
    L.st1 = take(rows * sizeof(float2));   // (mean, 1/deviation) of the two normalisations
    L.st2 = take(rows * sizeof(float2));
    L.z = take(rows * d * 2);
    L.f1 = take(rows * (size_t)d_ff * 2);
    L.attn = take(attn_ws);
    L.total = off;
    return L;
}

bpt_shape_t attn_shape(const bpt_graph* g, int B, int H, float scale, const int32_t* seq_len) {
    bpt_shape_t s = {};
    s.B = B;
    s.H = H;
    s.D = kD;
    s.dtype = BPT_BF16;
    // Q, K, V and the attention's output of a node sit side by side, [B][N][Q | K | V | O][H][64] (one projection
    // writes the first three); the gradients of the backward use the same layout with dO in the fourth place
    s.stride_n = (int64_t)4 * H * kD;
    s.stride_h = kD;
    s.stride_b = (int64_t)g->num_nodes * 4 * H * kD;
    s.grad_dtype = BPT_BF16;                   // dQ, dK, dV feed bf16 GEMMs
    s.scale = scale;
    s.seq_len = seq_len;
    return s;
}

// slices of the contraction over K for an M x N result: a power of two (the library's kernels for other counts are often
// slower ones; 65 532 rows, d = 512, [dWq | dWk | dWv]: 193 us in 11 slices, 121 us in 16), no more than give every compute
// unit two tiles, and at least 1000 rows each (trees of powers of two have just fewer rows than a power of two, which a
// bound of 1024 would halve the slices of).  Swept over the four products of a layer, d = 128, 256, 384, 512, 1024, 13 row
// counts from 1021 to 131 056 and 1, 2, 4, 8, 16 slices, sums of the slices included: this takes on average 1.046 times the
// best count's time (at least 512 rows 1.059, 900 or 1024 rows 1.048, 1400 rows 1.053, 1800 rows 1.084).
int pick_slices(int M, int N, int64_t K) {
    const int64_t tiles = (int64_t)((M + 127) / 128) * ((N + 127) / 128);
    int slices = 1;
    while (slices < 16 && slices * tiles < 512 && K / (2 * slices) >= 1000) slices *= 2;
    return slices;
}

// workgroups of the normalisations: what 256 compute units hold at once at the kernels' registers up to d = 512; wider ones
// walk the same grid (two calls each, before they held parameters and read ahead / now, us: d = 1024, 16 376 rows, forward
// 69.7 / 55.4, backward 160 / 85; d = 2048, 8188 rows, 76.9 / 65.2 and 268 / 154)
constexpr int kLnBlocks = 7 * 256, kLnBwdBlocks = 4 * 256;
constexpr int kColumnSumBlocks = 2048;   // workgroups (= partial rows) of the kernels that sum over rows

struct LayerBwdBuffers {
    size_t ds2, dh, t, ds1, dqkvo, part, gw, attn, total;
};
LayerBwdBuffers layer_bwd_buffers(const bpt_graph* g, int B, int H, int d_ff, size_t attn_ws) {
    const size_t rows = (size_t)B * g->num_nodes, d = (size_t)H * kD;
    LayerBwdBuffers L;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align_up(bytes);
        return at;
    };
    L.ds2 = take(rows * d * 2);              // gradient of the second pre-normalisation sum, bf16
    L.dh = take(rows * (size_t)d_ff * 2);    // gradient of the hidden FFN activations, bf16
    L.t = take(rows * d * 4);                // fp32 GEMM results: dH W1^T, later dQ Wq^T + dK Wk^T + dV Wv^T
    L.ds1 = take(rows * d * 2);
    L.dqkvo = take(rows * 4 * d * 2);        // [rows][dQ | dK | dV | dO] bf16: the attention's gradients, rounded to bf16 by its
                                             // backward, next to the gradient of its output -- the forward's layout
    L.part = take((size_t)kColumnSumBlocks * std::max<size_t>(3 * d, (size_t)d_ff) * 4);
    // partial products of the weight gradients (contraction over the rows, cut into slices)
    const size_t gw_qkv = (size_t)pick_slices((int)d, (int)(3 * d), (int64_t)rows) * d * 3 * d;
    const size_t gw_ffn = (size_t)pick_slices((int)d, d_ff, (int64_t)rows) * d * (size_t)d_ff;
    const size_t gw_o = (size_t)pick_slices((int)d, (int)d, (int64_t)rows) * d * d;
    L.gw = take(std::max(gw_qkv, std::max(gw_ffn, gw_o)) * 4);
    L.attn = take(attn_ws);
    L.total = off;
    return L;
}

// column sums of partials[parts][cols]; the columns are `cols / cols_each` outputs side by side
template <int CHUNKS>
int launch_ln_bwd_as(int blocks, hipStream_t st, const bf16_t* dy_b, const float* dy_f, const bf16_t* x, const float* a,
                     const float* bias, const float* gain, const float2* stats, bf16_t* ds, float* partials, int64_t rows, int d,
                     const int32_t* seq_len, int N, int lg) {
    const size_t lds = (size_t)9 * d * sizeof(float);
    if (lds > 65536)
        BPT_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(layer_norm_bwd_kernel<CHUNKS>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    BPT_LAUNCH("layer_norm_bwd_kernel", layer_norm_bwd_kernel<CHUNKS>, dim3(blocks), dim3(256), lds, st, dy_b, dy_f, x, a, bias,
               gain, stats, ds, partials, rows, d, seq_len, N, lg);
    BPT_HIP(hipGetLastError());
    return BPT_OK;
}
// forward normalisation: as many workgroups as the device holds at once (a row per wavefront and step)
int launch_ln(int d, hipStream_t st, const bf16_t* x, const float* a, const float* bias, const float* gain, const float* beta, bf16_t* y,
              float2* stats, int64_t rows, float eps) {
    const dim3 grid((unsigned)std::min<int64_t>(kLnBlocks, (rows + 3) / 4));
    if (d <= 512)
        BPT_LAUNCH("residual_layer_norm_kernel", residual_layer_norm_kernel<1>, grid, dim3(256), 0, st, x, a, bias, gain, beta, y, stats, rows, d, eps);
    else if (d <= 1024)
        BPT_LAUNCH("residual_layer_norm_kernel", residual_layer_norm_kernel<2>, grid, dim3(256), 0, st, x, a, bias, gain, beta, y, stats, rows, d, eps);
    else
        BPT_LAUNCH("residual_layer_norm_kernel", residual_layer_norm_kernel<kLnMaxChunks>, grid, dim3(256), 0, st, x, a, bias, gain, beta, y, stats, rows, d, eps);
    BPT_HIP(hipGetLastError());
    return BPT_OK;
}
template <typename... Args>
int launch_ln_bwd(int d, Args... args) {
    if (d <= 512) return launch_ln_bwd_as<1>(args...);
    if (d <= 1024) return launch_ln_bwd_as<2>(args...);
    return launch_ln_bwd_as<kLnMaxChunks>(args...);
}

int column_sum(const float* partials, int parts, int cols, int cols_each, float* o0, float* o1, float* o2, hipStream_t st) {
    const ColumnSumOut o = {{o0, o1, o2}, cols_each};
    BPT_LAUNCH("column_sum_kernel", column_sum_kernel, dim3((cols + kColumnSumCols - 1) / kColumnSumCols), dim3(1024), 0, st,
               partials, parts, cols, o);
    BPT_HIP(hipGetLastError());
    return BPT_OK;
}

// C[M][N] (fp32) = A^T B with A stored [K][M], B stored [K][N], bf16, K long and M x N small: the
// contraction is cut into `slices` equal parts that run as one strided-batched GEMM into
// `partials` [slices][M][N], and the parts are added in slice order, with the products of the few left-over rows of K,
// by sum_slices_kernel.  The N columns are N / n_each matrices side by
// side that go to out0..out2 (each [M][n_each]).
int gemm_at_b_sliced(rocblas_handle h, int M, int N, int64_t K, const void* A, const void* B, int ldb_cols, float* partials,
                     int slices, int n_each, float* out0, float* out1, float* out2, hipStream_t st, int lda_cols = 0) {
    const float one = 1.f, zero = 0.f;
    const int lda = lda_cols ? lda_cols : M;   // elements between rows of A as stored
    const int64_t ks = K / slices;
    if (ks < 1) return BPT_ERR_INVALID_ARG;
    // column-major view: C^T (N x M) = B^T-as-stored (N x K, ld = ldb_cols) times A (K x M) given as its transpose
    rocblas_status rs = rocblas_gemm_strided_batched_ex(
        h, rocblas_operation_none, rocblas_operation_transpose, N, M, (rocblas_int)ks, &one, B, rocblas_datatype_bf16_r, ldb_cols,
        ks * ldb_cols, A, rocblas_datatype_bf16_r, lda, ks * (int64_t)lda, &zero, partials, rocblas_datatype_f32_r, N, (int64_t)M * N,
        partials, rocblas_datatype_f32_r, N, (int64_t)M * N, slices, rocblas_datatype_f32_r, rocblas_gemm_algo_standard, 0, 0);
    if (rs != rocblas_status_success) return BPT_ERR_LAUNCH;
    const int64_t done = ks * slices;   // the rows behind are multiplied where the slices are added
    const ColumnSumOut o = {{out0, out1, out2}, n_each};
    const int64_t elems = (int64_t)M * N;
    BPT_LAUNCH("sum_slices_kernel", sum_slices_kernel, dim3((unsigned)((elems / 4 + 255) / 256)), dim3(256), 0, st, partials,
               slices, elems, N, o, static_cast<const bf16_t*>(A) + done * lda, static_cast<const bf16_t*>(B) + done * ldb_cols,
               (int)(K - done), (int64_t)lda, (int64_t)ldb_cols);
    BPT_HIP(hipGetLastError());
    return BPT_OK;
}

// Workspace of the stack's forward: the states H^0 .. H^layers, then one layer workspace per layer.
struct StackBuffers {
    size_t state_bytes, layer_bytes, layers_at, total;
};
StackBuffers stack_buffers(const bpt_graph* g, int B, int H, int d_ff, int num_layers) {
    const bpt_shape_t s = attn_shape(g, B, H, 0.f, nullptr);
    StackBuffers S;
    S.state_bytes = align_up((size_t)B * g->num_nodes * H * kD * 2);
    const size_t attn_ws = bpt_attn_fwd_workspace(g, &s);
    S.layer_bytes = align_up(layer_buffers(g, B, H, d_ff, attn_ws == SIZE_MAX ? 0 : attn_ws).total);
    S.layers_at = S.state_bytes * ((size_t)num_layers + 1);
    S.total = S.layers_at + S.layer_bytes * (size_t)num_layers;
    return S;
}
constexpr int kMaxStackLayers = 256;

}  // namespace
}  // namespace bpt

namespace bpt {
namespace {

// One layer, forward and backward, for the entry points below: a stack of layers is one call of the user's (UseOnReturn).
int layer_fwd(const bpt_graph_t* g, int32_t B, int32_t H, float scale, const int32_t* seq_len, const void* rel,
              const void* X, const bpt_layer_params_t* p, void* Y, void* workspace, size_t workspace_bytes, void* stream) {
    if (!g || !rel || !X || !p || !Y || B < 1 || H < 1) return BPT_ERR_INVALID_ARG;
    if (!p->Wq || !p->Wk || !p->Wv || !p->Wo || !p->W1 || !p->W2 || !p->b1 || !p->b2 || !p->g1 || !p->beta1 || !p->g2 || !p->beta2)
        return BPT_ERR_INVALID_ARG;
    if (any_misaligned(X, Y, workspace, p->Wq, p->Wk, p->Wv, p->Wo, p->W1, p->W2, p->b1, p->b2, p->g1, p->beta1, p->g2, p->beta2))
        return BPT_ERR_INVALID_ARG;
    const int d = H * kD, d_ff = p->d_ff;
    if (d > 8 * 64 * kLnMaxChunks || d_ff < 8 || (d_ff & 7)) return BPT_ERR_UNSUPPORTED;
    const int64_t rows = (int64_t)B * g->num_nodes;
    if (rows > INT32_MAX) return BPT_ERR_UNSUPPORTED;
    const bpt_shape_t s = attn_shape(g, B, H, scale, seq_len);
    const size_t attn_ws = bpt_attn_fwd_workspace(g, &s);
    if (attn_ws == SIZE_MAX) return BPT_ERR_UNSUPPORTED;
    const LayerBuffers L = layer_buffers(g, B, H, d_ff, attn_ws);
    if (L.total > workspace_bytes || (L.total && !workspace)) return BPT_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    rocblas_handle h = blas_handle(g->device);
    if (!h || rocblas_set_stream(h, st) != rocblas_status_success) return BPT_ERR_LAUNCH;
    const Blas bl = {h, g->device, st};
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    bf16_t* qkvo = reinterpret_cast<bf16_t*>(ws + L.qkvo);
    bf16_t* wqkv = reinterpret_cast<bf16_t*>(ws + L.wqkv);
    void *q = qkvo, *k = qkvo + d, *v = qkvo + 2 * d, *o = qkvo + 3 * d, *z = ws + L.z, *f1 = ws + L.f1;
    float* lse = reinterpret_cast<float*>(ws + L.lse);
    float* acc1 = reinterpret_cast<float*>(ws + L.acc1);
    float* acc2 = reinterpret_cast<float*>(ws + L.acc2);
    float2* st1 = reinterpret_cast<float2*>(ws + L.st1);
    float2* st2 = reinterpret_cast<float2*>(ws + L.st2);
    const float eps = p->eps > 0.f ? p->eps : 1e-5f;
    int rc;
    // [Q | K | V] = X [Wq | Wk | Wv] for all nodes in one product that reads X once: rows of [Q | K | V | O][H][64],
    // the layout the attention reads and writes through its strides (the packed weights stay in the workspace for
    // the backward)
    const PackArgs pa = {{static_cast<const bf16_t*>(p->Wq), static_cast<const bf16_t*>(p->Wk), static_cast<const bf16_t*>(p->Wv)}, wqkv};
    const int64_t wchunks = (int64_t)d * d / 8;
    BPT_LAUNCH("pack_qkv_weights_kernel", pack_qkv_weights_kernel, dim3((unsigned)((wchunks + 255) / 256), 3), dim3(256), 0, st, pa,
               wchunks, d);
    BPT_HIP(hipGetLastError());
    if ((rc = gemm(bl, rows, 3 * d, d, X, false, wqkv, false, qkvo, false, 0, 4 * d))) return rc;
    if ((rc = attn_fwd(g, &s, q, k, v, rel, o, lse, ws + L.attn, attn_ws, stream))) return rc;
    // Z = norm(X + O Wo)
    if ((rc = gemm(bl, rows, d, d, o, false, p->Wo, false, acc1, true, 4 * d))) return rc;
    if ((rc = launch_ln(d, st, static_cast<const bf16_t*>(X), acc1, nullptr, p->g1, p->beta1, static_cast<bf16_t*>(z), st1, rows, eps))) return rc;
    // Y = norm(Z + max(0, Z W1 + b1) W2 + b2)
    bool fused = false;   // bias + ReLU in the product's epilogue, on the fp32 sums
    if ((rc = gemm(bl, rows, d_ff, d, z, false, p->W1, false, f1, false, 0, 0, p->b1, &fused))) return rc;
    if (!fused) {
        const int64_t chunks = rows * d_ff / 8;
        BPT_LAUNCH("bias_relu_kernel", bias_relu_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, st,
                   static_cast<bf16_t*>(f1), p->b1, chunks, d_ff);
        BPT_HIP(hipGetLastError());
    }
    if ((rc = gemm(bl, rows, d, d_ff, f1, false, p->W2, false, acc2, true))) return rc;
    return launch_ln(d, st, static_cast<const bf16_t*>(z), acc2, p->b2, p->g2, p->beta2, static_cast<bf16_t*>(Y), st2, rows, eps);
}

int layer_bwd(const bpt_graph_t* g, int32_t B, int32_t H, float scale, const int32_t* seq_len, const void* rel,
              const void* X, const bpt_layer_params_t* p, const void* fwd_workspace, size_t fwd_workspace_bytes,
              const void* dY, void* dX, float* d_rel, const bpt_layer_grads_t* gr, void* workspace,
              size_t workspace_bytes, void* stream) {
    if (!g || !rel || !X || !p || !fwd_workspace || !dY || !dX || !d_rel || !gr || B < 1 || H < 1) return BPT_ERR_INVALID_ARG;
    if (!p->Wq || !p->Wk || !p->Wv || !p->Wo || !p->W1 || !p->W2 || !p->b1 || !p->b2 || !p->g1 || !p->beta1 || !p->g2 || !p->beta2)
        return BPT_ERR_INVALID_ARG;
    if (!gr->dWq || !gr->dWk || !gr->dWv || !gr->dWo || !gr->dW1 || !gr->db1 || !gr->dW2 || !gr->db2 || !gr->dg1 ||
        !gr->dbeta1 || !gr->dg2 || !gr->dbeta2)
        return BPT_ERR_INVALID_ARG;
    if (any_misaligned(X, fwd_workspace, dY, dX, d_rel, workspace, p->Wq, p->Wk, p->Wv, p->Wo, p->W1, p->W2, p->b1, p->b2, p->g1,
                       p->beta1, p->g2, p->beta2, gr->dWq, gr->dWk, gr->dWv, gr->dWo, gr->dW1, gr->db1, gr->dW2, gr->db2, gr->dg1,
                       gr->dbeta1, gr->dg2, gr->dbeta2))
        return BPT_ERR_INVALID_ARG;
    const int d = H * kD, d_ff = p->d_ff;
    if (d > 8 * 64 * kLnMaxChunks || d_ff < 8 || (d_ff & 7) || d_ff > 8 * 256 * kReluChunks) return BPT_ERR_UNSUPPORTED;
    const int64_t rows = (int64_t)B * g->num_nodes;
    if (rows > INT32_MAX) return BPT_ERR_UNSUPPORTED;
    const bpt_shape_t s = attn_shape(g, B, H, scale, seq_len);
    const size_t attn_fws = bpt_attn_fwd_workspace(g, &s);
    const size_t attn_ws = bpt_attn_bwd_workspace(g, &s);
    if (attn_fws == SIZE_MAX || attn_ws == SIZE_MAX) return BPT_ERR_UNSUPPORTED;
    const LayerBuffers F = layer_buffers(g, B, H, d_ff, attn_fws);
    if (F.total > fwd_workspace_bytes) return BPT_ERR_INVALID_ARG;
    const LayerBwdBuffers L = layer_bwd_buffers(g, B, H, d_ff, attn_ws);
    if (L.total > workspace_bytes || !workspace) return BPT_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    rocblas_handle h = blas_handle(g->device);
    if (!h || rocblas_set_stream(h, st) != rocblas_status_success) return BPT_ERR_LAUNCH;
    const Blas bl = {h, g->device, st};
    const unsigned char* fw = static_cast<const unsigned char*>(fwd_workspace);
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    const bf16_t* qkvo = reinterpret_cast<const bf16_t*>(fw + F.qkvo);
    const bf16_t* wqkv = reinterpret_cast<const bf16_t*>(fw + F.wqkv);
    const void *q = qkvo, *k = qkvo + d, *v = qkvo + 2 * d, *o = qkvo + 3 * d;
    const bf16_t* z = reinterpret_cast<const bf16_t*>(fw + F.z);
    const bf16_t* f1 = reinterpret_cast<const bf16_t*>(fw + F.f1);
    const float* lse = reinterpret_cast<const float*>(fw + F.lse);
    const float *acc1 = reinterpret_cast<const float*>(fw + F.acc1), *acc2 = reinterpret_cast<const float*>(fw + F.acc2);
    const float2 *st1 = reinterpret_cast<const float2*>(fw + F.st1), *st2 = reinterpret_cast<const float2*>(fw + F.st2);
    bf16_t *ds2 = reinterpret_cast<bf16_t*>(ws + L.ds2), *dh = reinterpret_cast<bf16_t*>(ws + L.dh);
    bf16_t *ds1 = reinterpret_cast<bf16_t*>(ws + L.ds1), *dqkvo = reinterpret_cast<bf16_t*>(ws + L.dqkvo);
    bf16_t* da = dqkvo + 3 * d;
    float *t = reinterpret_cast<float*>(ws + L.t), *part = reinterpret_cast<float*>(ws + L.part);
    float* gw = reinterpret_cast<float*>(ws + L.gw);
    const int lg = 31 - __builtin_clz((unsigned)g->n);
    const int ln_blocks = (int)std::min<int64_t>(kLnBwdBlocks, (rows + 3) / 4);
    const bf16_t* Xb = static_cast<const bf16_t*>(X);
    int rc;

    // second normalisation: dS2 (= the gradient of Z's residual branch, of the FFN output and of b2), dg2, dbeta2
    if ((rc = launch_ln_bwd(d, ln_blocks, st, static_cast<const bf16_t*>(dY), static_cast<const float*>(nullptr), z, acc2, p->b2,
                            p->g2, st2, ds2, part, rows, d, seq_len, g->num_nodes, lg)))
        return rc;
    if ((rc = column_sum(part, ln_blocks, 3 * d, d, gr->dg2, gr->dbeta2, gr->db2, st))) return rc;
    // FFN: dW2 = F^T dS2, dH = (dS2 W2^T) where the hidden unit was active, db1, dW1 = Z^T dH
    if ((rc = gemm_at_b_sliced(h, d_ff, d, rows, f1, ds2, d, gw, pick_slices(d, d_ff, rows), d, gr->dW2, nullptr, nullptr, st)))
        return rc;
    if ((rc = gemm(bl, rows, d_ff, d, ds2, false, p->W2, true, dh, false))) return rc;
    const int relu_blocks = (int)std::min<int64_t>(kColumnSumBlocks, rows);
    BPT_LAUNCH("relu_bwd_kernel", relu_bwd_kernel, dim3(relu_blocks), dim3(256), 0, st, dh, f1, part, rows, d_ff);
    BPT_HIP(hipGetLastError());
    if ((rc = column_sum(part, relu_blocks, d_ff, d_ff, gr->db1, nullptr, nullptr, st))) return rc;
    if ((rc = gemm_at_b_sliced(h, d, d_ff, rows, z, dh, d_ff, gw, pick_slices(d, d_ff, rows), d_ff, gr->dW1, nullptr, nullptr, st)))
        return rc;
    // first normalisation with dZ = dS2 + dH W1^T: dS1 (= the gradient of X's residual branch and of the
    // attention sublayer's output), dg1, dbeta1 (the third column sum, that of dS1, belongs to no parameter).
    // dZ is one product with dS2 as its addend (bf16, in the first half of t); without hipBLASLt the product
    // stays fp32 and the kernel adds
    bf16_t* dz = reinterpret_cast<bf16_t*>(t);
    const bool dz_joined = gemm_add(bl, rows, d, d_ff, dh, false, p->W1, true, dz, ds2);
    if (!dz_joined && (rc = gemm(bl, rows, d, d_ff, dh, false, p->W1, true, t, true))) return rc;
    if ((rc = launch_ln_bwd(d, ln_blocks, st, dz_joined ? static_cast<const bf16_t*>(dz) : static_cast<const bf16_t*>(ds2),
                            dz_joined ? static_cast<const float*>(nullptr) : static_cast<const float*>(t), Xb, acc1,
                            static_cast<const float*>(nullptr), p->g1, st1, ds1, part, rows, d,
                            static_cast<const int32_t*>(nullptr), g->num_nodes, lg)))
        return rc;
    if ((rc = column_sum(part, ln_blocks, 3 * d, d, gr->dg1, gr->dbeta1, nullptr, st))) return rc;
    // attention sublayer: dWo = O^T dS1, dO = dS1 Wo^T, then the attention's own backward
    if ((rc = gemm_at_b_sliced(h, d, d, rows, o, ds1, d, gw, pick_slices(d, d, rows), d, gr->dWo, nullptr, nullptr, st, 4 * d)))
        return rc;
    if ((rc = gemm(bl, rows, d, d, ds1, false, p->Wo, true, da, false, 0, 4 * d))) return rc;
    // dQ, dK, dV leave the attention's backward rounded to bf16, side by side next to dO: no cast pass
    if ((rc = attn_bwd(g, &s, q, k, v, rel, lse, da, dqkvo, dqkvo + d, dqkvo + 2 * d, d_rel, ws + L.attn, attn_ws, stream)))
        return rc;
    const int64_t chunks = rows * d / 8;
    // projections, one product each: [dWq | dWk | dWv] = X^T [dQ | dK | dV], dX = dS1 + [dQ | dK | dV] [Wq | Wk | Wv]^T
    if ((rc = gemm_at_b_sliced(h, d, 3 * d, rows, X, dqkvo, 4 * d, gw, pick_slices(d, 3 * d, rows), d, gr->dWq, gr->dWk, gr->dWv,
                               st)))
        return rc;
    // (the residual branch's gradient dS1 enters as the product's addend: one rounding, no pass of its own)
    if (gemm_add(bl, rows, d, 3 * d, dqkvo, false, wqkv, true, dX, ds1, 4 * d)) return BPT_OK;
    if ((rc = gemm(bl, rows, d, 3 * d, dqkvo, false, wqkv, true, t, true, 4 * d))) return rc;
    BPT_LAUNCH("add_cast_kernel", add_cast_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, st,
               static_cast<const bf16_t*>(ds1), static_cast<const float*>(t), static_cast<bf16_t*>(dX), chunks);
    BPT_HIP(hipGetLastError());
    return BPT_OK;
}

}  // namespace
}  // namespace bpt

using namespace bpt;

extern "C" {

size_t bpt_layer_fwd_workspace(const bpt_graph_t* g, int32_t B, int32_t H, int32_t d_ff) {
    if (!g || B < 1 || H < 1 || d_ff < 8) return 0;
    const bpt_shape_t s = attn_shape(g, B, H, 0.f, nullptr);
    const size_t attn_ws = bpt_attn_fwd_workspace(g, &s);
    if (attn_ws == SIZE_MAX) return SIZE_MAX;   // the attention calls refuse this graph and shape
    return layer_buffers(g, B, H, d_ff, attn_ws).total;
}

int bpt_layer_fwd(const bpt_graph_t* g, int32_t B, int32_t H, float scale, const int32_t* seq_len, const void* rel,
                  const void* X, const bpt_layer_params_t* p, void* Y, void* workspace, size_t workspace_bytes, void* stream) {
    const UseOnReturn use = {g, static_cast<hipStream_t>(stream)};
    return layer_fwd(g, B, H, scale, seq_len, rel, X, p, Y, workspace, workspace_bytes, stream);
}

size_t bpt_layer_bwd_workspace(const bpt_graph_t* g, int32_t B, int32_t H, int32_t d_ff) {
    if (!g || B < 1 || H < 1 || d_ff < 8) return 0;
    const bpt_shape_t s = attn_shape(g, B, H, 0.f, nullptr);
    const size_t attn_ws = bpt_attn_bwd_workspace(g, &s);
    if (attn_ws == SIZE_MAX) return SIZE_MAX;
    return layer_bwd_buffers(g, B, H, d_ff, attn_ws).total;
}

int bpt_layer_bwd(const bpt_graph_t* g, int32_t B, int32_t H, float scale, const int32_t* seq_len, const void* rel,
                  const void* X, const bpt_layer_params_t* p, const void* fwd_workspace, size_t fwd_workspace_bytes,
                  const void* dY, void* dX, float* d_rel, const bpt_layer_grads_t* gr, void* workspace,
                  size_t workspace_bytes, void* stream) {
    const UseOnReturn use = {g, static_cast<hipStream_t>(stream)};
    return layer_bwd(g, B, H, scale, seq_len, rel, X, p, fwd_workspace, fwd_workspace_bytes, dY, dX, d_rel, gr, workspace, workspace_bytes,
                     stream);
}

size_t bpt_stack_fwd_workspace(const bpt_graph_t* g, int32_t B, int32_t H, int32_t d_ff, int32_t num_layers) {
    if (!g || B < 1 || H < 1 || d_ff < 8 || num_layers < 1 || num_layers > kMaxStackLayers) return 0;
    if (g->batch > 0 && B != 1) return SIZE_MAX;   // the graph of a packed batch is the whole batch
    if (bpt_layer_fwd_workspace(g, B, H, d_ff) == SIZE_MAX) return SIZE_MAX;
    return stack_buffers(g, B, H, d_ff, num_layers).total;
}

int bpt_stack_fwd(const bpt_graph_t* g, int32_t B, int32_t H, int32_t num_layers, float scale, const int32_t* seq_len,
                  const void* const* rel, const void* E, const bpt_layer_params_t* p, void* root, void* tokens, void* workspace,
                  size_t workspace_bytes, void* stream) {
    if (!g || !rel || !E || !p || (!root && !tokens) || !workspace || B < 1 || H < 1 || num_layers < 1)
        return BPT_ERR_INVALID_ARG;
    if (num_layers > kMaxStackLayers) return BPT_ERR_UNSUPPORTED;
    if (g->batch > 0 && (B != 1 || seq_len)) return BPT_ERR_INVALID_ARG;   // the graph of a packed batch is the whole batch
    for (int l = 0; l < num_layers; ++l) {
        if (!rel[l]) return BPT_ERR_INVALID_ARG;
        if (p[l].d_ff != p[0].d_ff) return BPT_ERR_UNSUPPORTED;   // one workspace size serves every layer
    }
    if (p[0].d_ff < 8) return BPT_ERR_UNSUPPORTED;
    if (any_misaligned(E, root, tokens, workspace)) return BPT_ERR_INVALID_ARG;
    const StackBuffers S = stack_buffers(g, B, H, p[0].d_ff, num_layers);
    if (S.total > workspace_bytes) return BPT_ERR_INVALID_ARG;
    const int64_t rows = (int64_t)B * g->num_nodes;
    if (rows > INT32_MAX) return BPT_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const UseOnReturn use = {g, st};
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    const int row_chunks = H * kD / 8;
    const int64_t chunks = rows * row_chunks;
    BPT_LAUNCH("initial_states_kernel", initial_states_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, st,
               static_cast<const bf16_t*>(E), reinterpret_cast<bf16_t*>(ws), chunks, g->n_tokens, g->num_nodes, row_chunks);
    BPT_HIP(hipGetLastError());
    for (int l = 0; l < num_layers; ++l) {
        const int rc = layer_fwd(g, B, H, scale, seq_len, rel[l], ws + S.state_bytes * l, &p[l], ws + S.state_bytes * (l + 1),
                                 ws + S.layers_at + S.layer_bytes * l, S.layer_bytes, stream);
        if (rc) return rc;
    }
    // a tree has one root, its last row; the graph of a packed batch one per sequence
    const int roots = g->batch > 0 ? g->batch : 1;
    const int64_t out_chunks = (int64_t)B * (g->n_tokens + roots) * row_chunks;
    BPT_LAUNCH("readout_kernel", readout_kernel, dim3((unsigned)((out_chunks + 255) / 256)), dim3(256), 0, st,
               reinterpret_cast<const bf16_t*>(ws + S.state_bytes * num_layers), static_cast<bf16_t*>(root),
               static_cast<bf16_t*>(tokens), out_chunks, g->n_tokens, g->num_nodes, row_chunks, roots,
               static_cast<const int32_t*>(g->batch > 0 ? g->d_root_row : nullptr));
    BPT_HIP(hipGetLastError());
    return BPT_OK;
}

size_t bpt_stack_bwd_workspace(const bpt_graph_t* g, int32_t B, int32_t H, int32_t d_ff) {
    if (!g || B < 1 || H < 1 || d_ff < 8) return 0;
    if (g->batch > 0 && B != 1) return SIZE_MAX;
    const size_t layer = bpt_layer_bwd_workspace(g, B, H, d_ff);
    if (layer == SIZE_MAX) return SIZE_MAX;
    return layer ? 2 * align_up((size_t)B * g->num_nodes * H * kD * 2) + layer : 0;
}

int bpt_stack_bwd(const bpt_graph_t* g, int32_t B, int32_t H, int32_t num_layers, float scale, const int32_t* seq_len,
                  const void* const* rel, const bpt_layer_params_t* p, const void* fwd_workspace, size_t fwd_workspace_bytes,
                  const void* d_root, const void* d_tokens, void* dE, float* const* d_rel, const bpt_layer_grads_t* grads,
                  void* workspace, size_t workspace_bytes, void* stream) {
    if (!g || !rel || !p || !fwd_workspace || (!d_root && !d_tokens) || !dE || !d_rel || !grads || !workspace || B < 1 ||
        H < 1 || num_layers < 1)
        return BPT_ERR_INVALID_ARG;
    if (num_layers > kMaxStackLayers) return BPT_ERR_UNSUPPORTED;
    if (g->batch > 0 && (B != 1 || seq_len)) return BPT_ERR_INVALID_ARG;
    for (int l = 0; l < num_layers; ++l) {
        if (!rel[l] || !d_rel[l]) return BPT_ERR_INVALID_ARG;
        if (p[l].d_ff != p[0].d_ff) return BPT_ERR_UNSUPPORTED;
    }
    if (p[0].d_ff < 8) return BPT_ERR_UNSUPPORTED;
    if (any_misaligned(fwd_workspace, d_root, d_tokens, dE, workspace)) return BPT_ERR_INVALID_ARG;
    const StackBuffers S = stack_buffers(g, B, H, p[0].d_ff, num_layers);
    if (S.total > fwd_workspace_bytes) return BPT_ERR_INVALID_ARG;
    const size_t need = bpt_stack_bwd_workspace(g, B, H, p[0].d_ff);
    if (need == SIZE_MAX) return BPT_ERR_UNSUPPORTED;
    if (!need || need > workspace_bytes) return BPT_ERR_INVALID_ARG;
    const int64_t rows = (int64_t)B * g->num_nodes;
    if (rows > INT32_MAX) return BPT_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const UseOnReturn use = {g, st};
    const unsigned char* fw = static_cast<const unsigned char*>(fwd_workspace);
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    unsigned char* dh[2] = {ws, ws + S.state_bytes};   // gradients with respect to the states, alternating
    unsigned char* layer_ws = ws + 2 * S.state_bytes;
    const int row_chunks = H * kD / 8;
    const int64_t chunks = rows * row_chunks;
    BPT_LAUNCH("readout_bwd_kernel", readout_bwd_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, st,
               static_cast<const bf16_t*>(d_root), static_cast<const bf16_t*>(d_tokens), reinterpret_cast<bf16_t*>(dh[0]), chunks,
               g->n_tokens, g->num_nodes, row_chunks, g->batch > 0 ? g->batch : 1, g->batch > 0 ? g->first_root : g->num_nodes - 1,
               static_cast<const int32_t*>(g->batch > 0 ? g->d_root_seq : nullptr));
    BPT_HIP(hipGetLastError());
    int cur = 0;
    for (int l = num_layers - 1; l >= 0; --l, cur ^= 1) {
        const int rc = layer_bwd(g, B, H, scale, seq_len, rel[l], fw + S.state_bytes * l, &p[l],
                                 fw + S.layers_at + S.layer_bytes * l, S.layer_bytes, dh[cur], dh[cur ^ 1], d_rel[l], &grads[l],
                                 layer_ws, workspace_bytes - 2 * S.state_bytes, stream);
        if (rc) return rc;
    }
    // the embeddings are the token rows of the first states; the zero rows of the spans have no parameter behind them
    const int64_t out_chunks = (int64_t)B * (g->n_tokens + 1) * row_chunks;
    BPT_LAUNCH("readout_kernel", readout_kernel, dim3((unsigned)((out_chunks + 255) / 256)), dim3(256), 0, st,
               reinterpret_cast<const bf16_t*>(dh[cur]), static_cast<bf16_t*>(nullptr), static_cast<bf16_t*>(dE), out_chunks,
               g->n_tokens, g->num_nodes, row_chunks, 1, static_cast<const int32_t*>(nullptr));
    BPT_HIP(hipGetLastError());
    return BPT_OK;
}

}  // extern "C"
