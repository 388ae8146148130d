// fp32 tensors on the matrix cores: token rows and the key side over the dense tiles of the graph's metadata, span rows
// with the gather code, both in one launch.
//
// v_mfma_f32_16x16x4_f32 takes one value per lane and operand: A[m][k] and B[k][n] in lane m (n) + 16 k, and leaves C[m][n]
// in lane n + 16 (m / 4), register m % 4.  So nothing has to pass through LDS on its way to an operand: contracted over
// features, a lane reads 16-byte pieces of row m itself (feature 16q + 4g + e in step 4q + e, the same permutation for both
// operands); contracted over the rows of a chunk, a lane reads 16 bytes of row 4g + s, with features 4j .. 4j + 3 as the
// four A operands of step s -- whole rows of 256 bytes per 16 lanes -- and the score it holds in register s is the B operand.
// All products are single fp32 multiplications with fp32 sums, as in the gather kernels.
//
// An fp32 problem has few tiles (16 (batch, head)s at n = 2048: two per SIMD), so a workgroup of four wavefronts shares one
// tile: every wavefront takes a quarter of the chunks and the partial sums meet in LDS at the end.  The gather kernels
// spend about 70 vector instructions per 8 edges and side on dot products across lanes, online softmax per edge and index
// arithmetic, at half of the vector unit's time, the rest waiting.
// n = 2048, k = 8, causal, 16 (batch, head)s, gather kernels -> these (us): forward 71 -> 37, query side with d_rel 112 -> 73, key
// side 101 -> 40, step 315 -> 167; n = 512, k = 4, one head, forward 15.2 -> 7.8.  The matrix cores are busy for a fifth of
// that (7, 16 and 11 us); the rest is the chain ids -> rows -> products -> sums of a tile at two to four wavefronts per SIMD,
// and the span rows' vector code (15 and 19 us by themselves; in a launch of their own the step was no shorter).
#pragma once

#include "attn_gather.h"
#include "attn_token_tiles.h"

namespace bpt {
namespace {

constexpr int kF32Waves = 4;
constexpr int kF32Stride = kD + 4;   // floats per row of the partial sums in LDS
struct F32TileArgs {
    const int32_t *chunk_ptr, *cols, *cid_to_id;
    const int16_t* map;
    int32_t num_tiles, num_chunks, num_cids, cid_pad, bias_stride;
    int32_t token_blocks;   // workgroups of token tiles; then come those of the long, then those of the short segments
    int32_t long_blocks;
    int32_t first_long;     // segments of the span rows' schedule from here on are long
    float2* wp;             // backward: (p_e dP_e, p_e), [batch*head][token][wp_row]: column compact id of a token row's edge, and
                            // num_cids + l - 1 for the edge from the token's ancestor at level l
    int32_t wp_row;
};

// item i of `total` for a workgroup: workgroups run on XCD (index mod 8), and every XCD takes a contiguous share
__device__ __forceinline__ int xcd_item(int block, int total) {
    const int per = (total + 7) >> 3, i = (block & 7) * per + (block >> 3);
    return block >> 3 < per && i < total ? i : -1;
}

typedef float f32v4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32v4_t buf_f4(rsrc_t r, int byte_off) {
    return __builtin_bit_cast(f32v4_t, __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, 0, 0));
}
// sum over the 64 features of (row of lane j) x (row of lane j): C[m][n]
__device__ __forceinline__ f32x4_t dot_rows(const f32v4_t (&x)[4], const f32v4_t (&y)[4]) {
    f32x4_t c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
#pragma unroll
    for (int q = 0; q < 4; q += 2)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[q][e], y[q][e], c0, 0, 0, 0);
            c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[q + 1][e], y[q + 1][e], c1, 0, 0, 0);
        }
    return c0 + c1;
}
// Whether four values of a result are finite (a sum that overflows asks for nothing worse than the slow way below).
//
// A product takes every row of a chunk, with weight 0 where there is no edge, and 0 times an infinity or a NaN is not 0.  A
// finite result has met none, so the tiles look at their results on the way out, and what is not finite is computed
// once more over the row's own edges: such inputs reach the rows they have edges with and no others, in every fp32
// kernel (d_rel aside).  The look costs, at n = 2048, k = 8, causal, 16 heads (us, without / with): forward 36.5 / 36.9, query side
// 70.0 / 70.4, key side 39.5 / 40.4 (behind the key side's loop instead of in it: 41.5).
__device__ __forceinline__ bool all_finite(float x, float y, float z, float w) { return fabsf((x + y) + (z + w)) < INFINITY; }

// the 16 features of its row that a lane holds as an operand of dot_rows
__device__ __forceinline__ void load_operand(const float* row, int g, f32v4_t (&x)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = *reinterpret_cast<const f32v4_t*>(row + 16 * q + 4 * g);
}

// bias[token][id] * scale * log2(e) of the tile's tokens for all compact ids, a block of 16 ids per wavefront in turn
// (two blocks at a time: the rows of both are on their way together)
__device__ __forceinline__ int f32_rel_id(const F32TileArgs& t, int cid) { return t.cid_to_id[min(cid, t.num_cids - 1)]; }
__device__ __forceinline__ void form_bias_f32(const AttnArgs& a, const F32TileArgs& t, int id0, int id1, float* table,
                                              const f32v4_t (&q)[4], float qscale, int wave, int g, int j) {
    for (int b = wave; 16 * b < t.cid_pad; b += 2 * kF32Waves) {
        const bool two = 16 * (b + kF32Waves) < t.cid_pad;   // uniform
        f32v4_t r0[4], r1[4];
        load_operand(static_cast<const float*>(a.rel) + (int64_t)id0 * kD, g, r0);
        if (two) load_operand(static_cast<const float*>(a.rel) + (int64_t)id1 * kD, g, r1);
        if (16 * (b + 2 * kF32Waves) < t.cid_pad) {
            id0 = f32_rel_id(t, 16 * (b + 2 * kF32Waves) + j);
            id1 = f32_rel_id(t, 16 * (b + 3 * kF32Waves) + j);
        }
        float* at = table + j * t.bias_stride + 16 * b + 4 * g;
        *reinterpret_cast<f32x4_t*>(at) = dot_rows(r0, q) * qscale;
        if (two) *reinterpret_cast<f32x4_t*>(at + 16 * kF32Waves) = dot_rows(r1, q) * qscale;
    }
}

// segment s of the span rows' schedule: its row and its edges
struct SpanSeg {
    int u, e0, e1, slot;
};
__device__ __forceinline__ SpanSeg span_seg(const AttnArgs& a, int s) {
    SpanSeg x;
    x.u = uniform_i32(a.seg_row, s);
    x.e0 = uniform_i32(a.seg_begin, s);
    x.e1 = min(x.e0 + kSeg, uniform_i32(a.ptr, x.u + 1));
    x.slot = uniform_i32(a.seg_part, s);
    return x;
}
// the part of a long segment that falls to a wavefront: a quarter, in whole steps of 8 edges
__device__ __forceinline__ void quarter(const SpanSeg& x, int wave, int& b, int& e) {
    const int step = ((x.e1 - x.e0 + 8 * kF32Waves - 1) / (8 * kF32Waves)) * 8;
    b = min(x.e0 + wave * step, x.e1);
    e = min(b + step, x.e1);
}

// Span rows: workgroup `block` of those that take a long segment each, then a short segment per wavefront.
__device__ __forceinline__ void fwd_f32_spans(const AttnArgs& a, const F32TileArgs& t, float* f_s, int block, int wave, int lane) {
    const rsrc_t rIa = make_rsrc(a.ia, a.idx_bytes), rIb = make_rsrc(a.ib, a.idx_bytes);
    const bool is_long = block < t.long_blocks;
    const int segs = is_long ? a.num_segs - t.first_long : t.first_long;
    int item;
    if (is_long)
        item = xcd_item(block, a.BH * segs);
    else {
        const int per_block = xcd_item(block - t.long_blocks, (a.BH * segs + kF32Waves - 1) / kF32Waves);
        item = per_block < 0 || per_block * kF32Waves + wave >= a.BH * segs ? -1 : per_block * kF32Waves + wave;
    }
    if (item < 0) return;   // (long segments: the whole workgroup)
    const int bh = item / segs;
    const SpanSeg x = span_seg(a, (is_long ? t.first_long : 0) + item - bh * segs);
    const int64_t base = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh;
    const rsrc_t rK = make_rsrc(static_cast<const float*>(a.K) + base, a.slab_bytes);
    const rsrc_t rV = make_rsrc(static_cast<const float*>(a.V) + base, a.slab_bytes);
    float* part = x.slot < 0 ? nullptr : a.part + ((int64_t)bh * a.num_part + x.slot) * kPartStride;
    if (!is_long) {
        if (x.slot == kPartSpan8)
            fwd_span8<float>(a, rK, rV, bh, base, x.u, x.e0, a.ptr[x.u + 1] - x.e0, lane, a.n_tokens);
        else
            fwd_segment<float, false, true>(a, nullptr, rK, rV, rIa, rIb, bh, base, x.u, x.e0, x.e1, part, lane, a.n_tokens);
        return;
    }
    int b, e;
    quarter(x, wave, b, e);
    float* mine = f_s + wave * kPartStride;
    if (b < e)
        fwd_segment<float, false, true>(a, nullptr, rK, rV, rIa, rIb, bh, base, x.u, b, e, mine, lane, a.n_tokens);
    else {
        mine[lane] = 0.f;
        if (lane == 0) {
            mine[64] = kNegBig;
            mine[65] = 0.f;
        }
    }
    __syncthreads();
    if (wave == 0) {   // lane = feature
        float m = kNegBig, l = 0.f, acc = 0.f;
#pragma unroll
        for (int w = 0; w < kF32Waves; ++w) m = fmaxf(m, f_s[w * kPartStride + 64]);
#pragma unroll
        for (int w = 0; w < kF32Waves; ++w) {
            const float c = fast_exp2(f_s[w * kPartStride + 64] - m);
            l += c * f_s[w * kPartStride + 65];
            acc += c * f_s[w * kPartStride + lane];
        }
        if (part) {
            part[lane] = acc;
            if (lane == 0) {
                part[64] = m;
                part[65] = l;
            }
        } else {
            static_cast<float*>(a.out)[base + (int64_t)x.u * a.sn + lane] = acc / l;
            if (lane == 0) a.lse_w[(int64_t)bh * a.N + x.u] = (m + fast_log2(l)) * kLn2;
        }
    }
}
__device__ __forceinline__ void bwd_q_f32_spans(const AttnArgs& a, const F32TileArgs& t, float* f_s, int block, int wave, int lane) {
    const rsrc_t rIa = make_rsrc(a.ia, a.idx_bytes), rIb = make_rsrc(a.ib, a.idx_bytes);
    const bool is_long = block < t.long_blocks;
    const int segs = is_long ? a.num_segs - t.first_long : t.first_long;
    int item;
    if (is_long)
        item = xcd_item(block, a.BH * segs);
    else {
        const int per_block = xcd_item(block - t.long_blocks, (a.BH * segs + kF32Waves - 1) / kF32Waves);
        item = per_block < 0 || per_block * kF32Waves + wave >= a.BH * segs ? -1 : per_block * kF32Waves + wave;
    }
    if (item < 0) return;   // (long segments: the whole workgroup)
    const int bh = item / segs;
    const SpanSeg x = span_seg(a, (is_long ? t.first_long : 0) + item - bh * segs);
    const int64_t base = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh;
    const rsrc_t rK = make_rsrc(static_cast<const float*>(a.K) + base, a.slab_bytes);
    const rsrc_t rV = make_rsrc(static_cast<const float*>(a.V) + base, a.slab_bytes);
    float* part = x.slot < 0 ? nullptr : a.part + ((int64_t)bh * a.num_part + x.slot) * kQPartStride;
    float2* aff = t.wp + (int64_t)bh * a.n_tokens * t.wp_row + t.num_cids + node_level(x.u, a.lg) - 1;   // (eight rows of one segment are of one level)
    if (!is_long) {
        if (x.slot == kPartSpan8)
            bwd_q_span8<float>(a, rK, rV, bh, base, x.u, x.e0, a.ptr[x.u + 1] - x.e0, lane, a.n_tokens, aff, t.wp_row);
        else
            bwd_q_segment<float, false, true>(a, nullptr, rK, rV, rIa, rIb, bh, base, x.u, x.e0, x.e1, part, lane, a.n_tokens, aff,
                                              t.wp_row);
        return;
    }
    int b, e;
    quarter(x, wave, b, e);
    float* mine = f_s + wave * kQPartStride;
    if (b < e)
        bwd_q_segment<float, false, true>(a, nullptr, rK, rV, rIa, rIb, bh, base, x.u, b, e, mine, lane, a.n_tokens, aff, t.wp_row);
    else {
        mine[lane] = mine[kD + lane] = 0.f;
        if (lane == 0) mine[2 * kD] = 0.f;
    }
    __syncthreads();
    if (wave == 0) {   // lane = feature
        float A = 0.f, Bv = 0.f, dl = 0.f;
#pragma unroll
        for (int w = 0; w < kF32Waves; ++w) {
            A += f_s[w * kQPartStride + lane];
            Bv += f_s[w * kQPartStride + kD + lane];
            dl += f_s[w * kQPartStride + 2 * kD];
        }
        if (part) {
            part[lane] = A;
            part[kD + lane] = Bv;
            if (lane == 0) part[2 * kD] = dl;
        } else {
            a.dQ[base + (int64_t)x.u * a.sn + lane] = a.scale * (A - dl * Bv);
            if (lane == 0) a.stat[(int64_t)bh * a.N + x.u] = make_float2(a.lse_r[(int64_t)bh * a.N + x.u] * kLog2e, dl);
        }
    }
}
// Weighted sum of V rows, features f4 .. f4 + 3, of token t0 + tok with the softmax reference m: 16 lanes share a token.
__device__ __forceinline__ f32x4_t fwd_f32_again(const AttnArgs& a, const F32TileArgs& t, int64_t base, int t0, int tok, int f4, int c_begin,
                                                 int c_end, float m) {
    const float *K = static_cast<const float*>(a.K) + base + f4, *V = static_cast<const float*>(a.V) + base + f4;
    const f32x4_t q = *reinterpret_cast<const f32x4_t*>(static_cast<const float*>(a.Q) + base + (int64_t)(t0 + tok) * a.sn + f4);
    f32x4_t sum = {0.f, 0.f, 0.f, 0.f};
    for (int c = c_begin; c < c_end; ++c)
        for (int x = 0; x < 16; ++x) {
            const int cid = t.map[((int64_t)c * 16 + tok) * 16 + x];
            if (cid < 0) continue;   // (the same for the token's 16 lanes)
            const int64_t at = (int64_t)t.cols[c * 16 + x] * a.sn;
            const f32x4_t k = *reinterpret_cast<const f32x4_t*>(K + at) +
                              *reinterpret_cast<const f32x4_t*>(static_cast<const float*>(a.rel) + (int64_t)t.cid_to_id[cid] * kD + f4);
            float s = (q[0] * k[0] + q[1] * k[1]) + (q[2] * k[2] + q[3] * k[3]);
#pragma unroll
            for (int w = 1; w < 16; w <<= 1) s += __shfl_xor(s, w);
            sum += fast_exp2(fmaf(s, a.scale * kLog2e, -m)) * *reinterpret_cast<const f32x4_t*>(V + at);
        }
    return sum;
}

__global__ void __launch_bounds__(64 * kF32Waves, 4) fwd_f32_tile_kernel(const AttnArgs a, const F32TileArgs t) {
    extern __shared__ __align__(16) unsigned char smem[];
    float* f_s = reinterpret_cast<float*>(smem);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int block = blockIdx.x;
    if (block >= t.token_blocks) {
        fwd_f32_spans(a, t, f_s, block - t.token_blocks, wave, lane);
        return;
    }
    // ---- a tile of 16 token rows ----
    const int item = xcd_item(block, a.BH * t.num_tiles);
    if (item < 0) return;
    const int g = lane >> 4, j = lane & 15;
    const int bh = item / t.num_tiles, tile = item - bh * t.num_tiles, t0 = tile * 16;
    const int64_t base = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh;
    const rsrc_t rK = make_rsrc(static_cast<const float*>(a.K) + base, a.slab_bytes);
    const rsrc_t rV = make_rsrc(static_cast<const float*>(a.V) + base, a.slab_bytes);
    const rsrc_t rC = make_rsrc(t.cols, (uint32_t)t.num_chunks * 64u);
    const rsrc_t rM = make_rsrc(t.map, (uint32_t)t.num_chunks * 512u);
    const int c_begin = uniform_i32(t.chunk_ptr, tile), c_end = uniform_i32(t.chunk_ptr, tile + 1);
    const float qscale = a.scale * kLog2e;
    float* table = f_s;                                                             // [16 tokens][bias_stride]
    const int id0 = f32_rel_id(t, 16 * wave + j), id1 = f32_rel_id(t, 16 * (wave + kF32Waves) + j);
    // Rows are requested as soon as the registers of the chunk before are free, K rows behind its first product and V rows
    // behind its second; column ids and map words a chunk earlier.  (A chunk past the wavefront's last repeats the tile's
    // last: valid addresses, results unused.)
    int kcol;
    int4 vcol;
    uint2 mp;
    auto load_idx = [&](int c) {
        c = min(c, c_end - 1);
        kcol = buf_i32(rC, (c * 16 + j) * 4);
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rC, (c * 16 + 4 * g) * 4, 0, 0);
        vcol = make_int4((int)v.x, (int)v.y, (int)v.z, (int)v.w);
        const u32x2 m2 = __builtin_amdgcn_raw_buffer_load_b64(rM, (c * 16 + j) * 32 + 8 * g, 0, 0);
        mp = make_uint2(m2.x, m2.y);
    };
    f32v4_t k[4], v[4], q[4];
    auto load_k = [&]() {
        const int ko = (int)__umul24(kcol, a.row_bytes) + 16 * g;
#pragma unroll
        for (int x = 0; x < 4; ++x) k[x] = buf_f4(rK, ko + 64 * x);
    };
    auto load_v = [&](const int4& col) {
        const int vo[4] = {col.x, col.y, col.z, col.w};
#pragma unroll
        for (int s = 0; s < 4; ++s) v[s] = buf_f4(rV, (int)__umul24(vo[s], a.row_bytes) + 16 * j);
    };
    load_idx(c_begin + wave);
    load_operand(static_cast<const float*>(a.Q) + base + (int64_t)(t0 + j) * a.sn, g, q);
    load_k();
    load_v(vcol);
    uint2 mc = mp;
    load_idx(c_begin + wave + kF32Waves);
    form_bias_f32(a, t, id0, id1, table, q, qscale, wave, g, j);
    f32x4_t s = dot_rows(k, q);   // C[m = column 4g + r][n = token j]
    __syncthreads();

    float m_run = kNegBig, l_part = 0.f;
    f32x4_t o[4];   // out^T: lane (g, j), register r of o[f] = feature 16 g + 4 r + f of token j
#pragma unroll
    for (int f = 0; f < 4; ++f) o[f] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int c = c_begin + wave; c < c_end; c += kF32Waves) {
        load_k();
        const int4 vnext = vcol;
        const uint2 mnext = mp;
        load_idx(c + 2 * kF32Waves);
        const int cid[4] = {(int)(short)(mc.x & 0xFFFFu), (int)(short)(mc.x >> 16), (int)(short)(mc.y & 0xFFFFu), (int)(short)(mc.y >> 16)};
        float sc[4], p[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float bias = table[j * t.bias_stride + max(cid[r], 0)];
            sc[r] = cid[r] >= 0 ? fmaf(s[r], qscale, bias) : kNegBig;
        }
        float mx = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float mn = fmaxf(m_run, mx), corr = fast_exp2(m_run - mn);
        m_run = mn;
        l_part *= corr;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            p[r] = cid[r] >= 0 ? fast_exp2(sc[r] - mn) : 0.f;
            l_part += p[r];
        }
#pragma unroll
        for (int f = 0; f < 4; ++f) o[f] *= corr;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int f = 0; f < 4; ++f) o[f] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[r][f], p[r], o[f], 0, 0, 0);
        mc = mnext;
        if (c + kF32Waves < c_end) {   // uniform
            load_v(vnext);
            s = dot_rows(k, q);
        }
    }
    // the four wavefronts' sums
    l_part += __shfl_xor(l_part, 16);
    l_part += __shfl_xor(l_part, 32);
    __syncthreads();   // the table has been read
    float* o_s = f_s;                                              // [wavefront][16 tokens][kF32Stride]
    float* ml_s = f_s + kF32Waves * 16 * kF32Stride;               // [wavefront][16 tokens] max | sum
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const f32x4_t x = {o[0][r], o[1][r], o[2][r], o[3][r]};
        *reinterpret_cast<f32x4_t*>(o_s + (wave * 16 + j) * kF32Stride + 16 * g + 4 * r) = x;
    }
    if (g == 0) {
        ml_s[wave * 16 + j] = m_run;
        ml_s[kF32Waves * 16 + wave * 16 + j] = l_part;
    }
    __syncthreads();
    const int tok = threadIdx.x >> 4, f4 = (threadIdx.x & 15) * 4;
    float m = kNegBig, l = 0.f;
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) m = fmaxf(m, ml_s[w * 16 + tok]);
    f32x4_t sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) {
        const float c = fast_exp2(ml_s[w * 16 + tok] - m);
        l += c * ml_s[kF32Waves * 16 + w * 16 + tok];
        sum += c * *reinterpret_cast<const f32x4_t*>(o_s + (w * 16 + tok) * kF32Stride + f4);
    }
    if (__any(!all_finite(sum[0], sum[1], sum[2], sum[3]))) sum = fwd_f32_again(a, t, base, t0, tok, f4, c_begin, c_end, m);   // (four tokens)
    const float inv = 1.f / l;   // (a token row has its self edge)
    store_once(reinterpret_cast<float4*>(static_cast<float*>(a.out) + base + (int64_t)(t0 + tok) * a.sn + f4),
               make_float4(sum[0] * inv, sum[1] * inv, sum[2] * inv, sum[3] * inv));
    if (f4 == 0) a.lse_w[(int64_t)bh * a.N + t0 + tok] = (m + fast_log2(l)) * kLn2;
}

// Query side of the token rows and span rows.  delta is known when all chunks of a tile have been seen, so the tables in
// LDS hold what depends on it: table[token][id] the bias, replaced by w = p dP when the edge has been computed, and
// ptab[token][id] p, or -1 where the token has no such edge.  Then dS = w - delta p; it gives the relative-position part of
// dQ and the tile's share of d_rel, which a wavefront keeps for 16 of the features over all tiles of its workgroup.  The
// pairs (w, p) also go to memory, by token and id, for the key side.  NB: blocks of 16 ids.
// sum of dS (k + rel), features f4 .. f4 + 3, over the edges of token t0 + tok, from what the tile has left in memory
__device__ __forceinline__ f32x4_t bwd_q_f32_again(const AttnArgs& a, const F32TileArgs& t, int bh, int64_t base, int tile, int tok, int f4) {
    f32x4_t sum = {0.f, 0.f, 0.f, 0.f};
    const float2* wp = t.wp + ((int64_t)bh * a.n_tokens + tile * 16 + tok) * t.wp_row;
    const float delta = a.stat[(int64_t)bh * a.N + tile * 16 + tok].y;
    for (int i = 16 * t.chunk_ptr[tile]; i < 16 * t.chunk_ptr[tile + 1]; ++i) {
        const int cid = t.map[((int64_t)(i >> 4) * 16 + tok) * 16 + (i & 15)];
        if (cid >= 0)
            sum += (wp[cid].x - delta * wp[cid].y) *
                   (*reinterpret_cast<const f32x4_t*>(static_cast<const float*>(a.K) + base + (int64_t)t.cols[i] * a.sn + f4) +
                    *reinterpret_cast<const f32x4_t*>(static_cast<const float*>(a.rel) + (int64_t)t.cid_to_id[cid] * kD + f4));
    }
    return sum;
}
template <int NB>
__global__ void __launch_bounds__(64 * kF32Waves, 2) bwd_q_f32_tile_kernel(const AttnArgs a, const F32TileArgs t) {
    extern __shared__ __align__(16) unsigned char smem[];
    float* f_s = reinterpret_cast<float*>(smem);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int block = blockIdx.x;
    if (block >= t.token_blocks) {
        bwd_q_f32_spans(a, t, f_s, block - t.token_blocks, wave, lane);
        return;
    }
    // ---- tiles of 16 token rows ----
    const int g = lane >> 4, j = lane & 15;
    const rsrc_t rC = make_rsrc(t.cols, (uint32_t)t.num_chunks * 64u);
    const rsrc_t rM = make_rsrc(t.map, (uint32_t)t.num_chunks * 512u);
    const float qscale = a.scale * kLog2e;
    float* table = f_s;                                       // [16 tokens][bias_stride]: bias, then w, then dS
    float* ptab = table + 16 * t.bias_stride;                 // [16 tokens][bias_stride]: p or -1
    float* o_s = ptab + 16 * t.bias_stride;                   // [wavefront][16 tokens][kF32Stride]
    float* dl_s = o_s + kF32Waves * 16 * kF32Stride;          // [wavefront][16 tokens]
    int32_t* relid_s = reinterpret_cast<int32_t*>(dl_s + kF32Waves * 16);   // [cid_pad]
    for (int i = threadIdx.x; i < t.cid_pad; i += blockDim.x) relid_s[i] = f32_rel_id(t, i);
    const int id0 = f32_rel_id(t, 16 * wave + j), id1 = f32_rel_id(t, 16 * (wave + kF32Waves) + j);
    f32x4_t acc[NB];   // d_rel: register r = id 16 b + 4 g + r, feature 16 wave + j
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const int total = a.BH * t.num_tiles, per = (total + 7) >> 3, first = (block & 7) * per, last = min(first + per, total);
    // What a tile needs first -- its own rows, the ids of its first chunks and the rows of the first -- is requested when
    // the chunks of the tile before are through, so that it arrives behind that tile's last steps.
    int kcol;
    int4 vcol, vc;
    uint2 mp, mc;
    f32v4_t k[4], v[4], q[4], go[4];
    float lse2 = 0.f;
    int c_end = 0;
    bool bad = false;   // a dQ that this thread has stored was not finite
    auto load_idx = [&](int c) {
        c = min(c, c_end - 1);
        kcol = buf_i32(rC, (c * 16 + j) * 4);
        const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(rC, (c * 16 + 4 * g) * 4, 0, 0);
        vcol = make_int4((int)x.x, (int)x.y, (int)x.z, (int)x.w);
        const u32x2 m2 = __builtin_amdgcn_raw_buffer_load_b64(rM, (c * 16 + j) * 32 + 8 * g, 0, 0);
        mp = make_uint2(m2.x, m2.y);
    };
    auto load_rows = [&](rsrc_t rK, rsrc_t rV) {
        const int ko = (int)__umul24(kcol, a.row_bytes) + 16 * g;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            k[x] = buf_f4(rK, ko + 64 * x);
            v[x] = buf_f4(rV, ko + 64 * x);
        }
    };
    auto request_tile = [&](int item) {
        const int bh = item / t.num_tiles, tile = item - bh * t.num_tiles;
        const int64_t base = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh, row = base + (int64_t)(tile * 16 + j) * a.sn;
        const int c_begin = uniform_i32(t.chunk_ptr, tile);
        c_end = uniform_i32(t.chunk_ptr, tile + 1);
        load_idx(c_begin + wave);
        load_operand(static_cast<const float*>(a.Q) + row, g, q);
        load_operand(static_cast<const float*>(a.dout) + row, g, go);
        lse2 = a.lse_r[(int64_t)bh * a.N + tile * 16 + j] * kLog2e;
        load_rows(make_rsrc(static_cast<const float*>(a.K) + base, a.slab_bytes), make_rsrc(static_cast<const float*>(a.V) + base, a.slab_bytes));
        vc = vcol;
        mc = mp;
        load_idx(c_begin + wave + kF32Waves);
    };
    if (NB <= 12 && first + (block >> 3) < last) request_tile(first + (block >> 3));
    for (int item = first + (block >> 3); item < last; item += t.token_blocks >> 3) {
        const int bh = item / t.num_tiles, tile = item - bh * t.num_tiles, t0 = tile * 16;
        const int64_t base = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh;
        const rsrc_t rK = make_rsrc(static_cast<const float*>(a.K) + base, a.slab_bytes);
        const rsrc_t rV = make_rsrc(static_cast<const float*>(a.V) + base, a.slab_bytes);
        const int c_begin = uniform_i32(t.chunk_ptr, tile);
        const float* qrow = static_cast<const float*>(a.Q) + base + (int64_t)t0 * a.sn;
        if (NB > 12) request_tile(item);   // (the registers are taken)
        __syncthreads();   // the tile before has read table and o_s
        for (int x = threadIdx.x * 4; x < 16 * t.bias_stride; x += blockDim.x * 4)
            *reinterpret_cast<f32x4_t*>(ptab + x) = f32x4_t{-1.f, -1.f, -1.f, -1.f};
        form_bias_f32(a, t, id0, id1, table, q, qscale, wave, g, j);
        __syncthreads();

        float dl = 0.f;
        f32x4_t ow[4], op[4];   // sums of w k and p k, laid out as the forward's out
#pragma unroll
        for (int f = 0; f < 4; ++f) ow[f] = op[f] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        for (int c = c_begin + wave; c < c_end; c += kF32Waves) {
            const f32x4_t s = dot_rows(k, q), d = dot_rows(v, go);   // C[m = column 4g + r][n = token j]
            // the K rows once more, as operands over columns (they are in the caches), then the next chunk's rows
            f32v4_t kt[4];
            const int vo[4] = {vc.x, vc.y, vc.z, vc.w};
#pragma unroll
            for (int x = 0; x < 4; ++x) kt[x] = buf_f4(rK, (int)__umul24(vo[x], a.row_bytes) + 16 * j);
            load_rows(rK, rV);
            const int cid[4] = {(int)(short)(mc.x & 0xFFFFu), (int)(short)(mc.x >> 16), (int)(short)(mc.y & 0xFFFFu), (int)(short)(mc.y >> 16)};
            vc = vcol;
            mc = mp;
            load_idx(c + 2 * kF32Waves);
            float w[4], p[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float* at = table + j * t.bias_stride + max(cid[r], 0);
                const float x = fast_exp2(fmaf(s[r], qscale, *at) - lse2);
                p[r] = cid[r] >= 0 ? x : 0.f;
                w[r] = cid[r] >= 0 ? x * d[r] : 0.f;
                dl += w[r];
                if (cid[r] >= 0) {   // (an id stands for one edge of a token: no other lane uses the entry)
                    *at = w[r];
                    ptab[j * t.bias_stride + cid[r]] = p[r];
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int f = 0; f < 4; ++f) {
                    ow[f] = __builtin_amdgcn_mfma_f32_16x16x4f32(kt[r][f], w[r], ow[f], 0, 0, 0);
                    op[f] = __builtin_amdgcn_mfma_f32_16x16x4f32(kt[r][f], p[r], op[f], 0, 0, 0);
                }
        }
        // what the steps behind delta read, and the next tile
        const float lse_row = lse2;
        float qt[4];   // Q rows as operands over tokens: feature 16 wave + j of token 4 s + g
#pragma unroll
        for (int s = 0; s < 4; ++s) qt[s] = qrow[(int64_t)(4 * s + g) * a.sn + 16 * wave + j];
        constexpr int kAhead = NB > 6 ? 0 : NB;   // (more spill)
        f32v4_t rel[NB];   // table rows of the ids 4 (wave + 4 x) + g, features 4 j ..
        auto load_rel = [&](int x) {
            return *reinterpret_cast<const f32v4_t*>(static_cast<const float*>(a.rel) + (int64_t)relid_s[4 * (wave + kF32Waves * x) + g] * kD + 4 * j);
        };
#pragma unroll
        for (int x = 0; x < kAhead; ++x)
            if (16 * x < t.cid_pad) rel[x] = load_rel(x);   // uniform
        if (NB <= 12 && item + (t.token_blocks >> 3) < last) request_tile(item + (t.token_blocks >> 3));
        dl += __shfl_xor(dl, 16);
        dl += __shfl_xor(dl, 32);
        if (g == 0) dl_s[wave * 16 + j] = dl;
        __syncthreads();
        const float delta = (dl_s[j] + dl_s[16 + j]) + (dl_s[32 + j] + dl_s[48 + j]);
        if (wave == 0 && g == 0) a.stat[(int64_t)bh * a.N + t0 + j] = make_float2(lse_row, delta);
        {   // dS of the tile, and its (w, p) pairs by token and id
            const int tok = threadIdx.x >> 4;
            const float dt = (dl_s[tok] + dl_s[16 + tok]) + (dl_s[32 + tok] + dl_s[48 + tok]);
            float2* dst = t.wp + ((int64_t)bh * a.n_tokens + t0 + tok) * t.wp_row;
            for (int c = threadIdx.x & 15; c < t.cid_pad; c += 16) {
                const float w = table[tok * t.bias_stride + c], p = ptab[tok * t.bias_stride + c];
                const bool edge = p != -1.f;
                table[tok * t.bias_stride + c] = edge ? w - dt * p : 0.f;
                if (c < t.num_cids) dst[c] = make_float2(w, p);
            }
        }
        __syncthreads();
        f32x4_t dq[4];
#pragma unroll
        for (int f = 0; f < 4; ++f) dq[f] = ow[f] - delta * op[f];
        auto add_rel = [&](int x, const f32v4_t& r) {   // + dS x Rel, four ids at a time
            const float d = table[j * t.bias_stride + 4 * (wave + kF32Waves * x) + g];
#pragma unroll
            for (int f = 0; f < 4; ++f) dq[f] = __builtin_amdgcn_mfma_f32_16x16x4f32(r[f], d, dq[f], 0, 0, 0);
        };
#pragma unroll
        for (int x = 0; x < kAhead; ++x)
            if (16 * x < t.cid_pad) add_rel(x, rel[x]);
        for (int x = kAhead; 16 * x < t.cid_pad; ++x) add_rel(x, load_rel(x));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const f32x4_t x = {dq[0][r], dq[1][r], dq[2][r], dq[3][r]};
            *reinterpret_cast<f32x4_t*>(o_s + (wave * 16 + j) * kF32Stride + 16 * g + 4 * r) = x;
        }
#pragma unroll
        for (int b = 0; b < NB; ++b)
            if (16 * b < t.cid_pad)   // uniform
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(table[(4 * s + g) * t.bias_stride + 16 * b + j], qt[s], acc[b], 0, 0, 0);
        __syncthreads();
        {
            const int tok = threadIdx.x >> 4, f4 = (threadIdx.x & 15) * 4;
            f32x4_t sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < kF32Waves; ++w) sum += *reinterpret_cast<const f32x4_t*>(o_s + (w * 16 + tok) * kF32Stride + f4);
            bad |= !all_finite(sum[0], sum[1], sum[2], sum[3]);
            store_once(reinterpret_cast<float4*>(a.dQ + base + (int64_t)(t0 + tok) * a.sn + f4),
                       make_float4(a.scale * sum[0], a.scale * sum[1], a.scale * sum[2], a.scale * sum[3]));
        }
    }
    // this workgroup's copy of d_rel: [token_blocks][cid_pad][kD], compact-id order
    float* dst = a.drel_part + (int64_t)block * t.cid_pad * kD;
#pragma unroll
    for (int b = 0; b < NB; ++b)
        if (16 * b < t.cid_pad)
#pragma unroll
            for (int r = 0; r < 4; ++r) dst[(16 * b + 4 * g + r) * kD + 16 * wave + j] = acc[b][r] * a.scale;

    __syncthreads();   // (the tiles' deltas)
    if (!__any(bad)) return;
    // (behind the loop, where no registers are taken: inside it the kernel spills, 4 registers up to 192 ids and 26 more above)
    for (int item = first + (block >> 3); item < last; item += t.token_blocks >> 3) {
        const int bh = item / t.num_tiles, tile = item - bh * t.num_tiles, tok = threadIdx.x >> 4, f4 = (threadIdx.x & 15) * 4;
        const int64_t base = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh;
        f32x4_t* dq = reinterpret_cast<f32x4_t*>(a.dQ + base + (int64_t)(tile * 16 + tok) * a.sn + f4);
        const f32x4_t x = *dq;
        if (!all_finite(x[0], x[1], x[2], x[3])) *dq = a.scale * bwd_q_f32_again(a, t, bh, base, tile, tok, f4);
    }
}

// Key side: with (w, p) of every edge in memory nothing is left of it but dK^T += Q^T dS and dV^T += dO^T P over a tile of
// up to 16 keys; all operands come straight from memory.  A workgroup takes a task of the key tiles: chained tiles one per
// wavefront in turn, the chunks of a single tile a quarter per wavefront.
struct F32KeyArgs {
    const int32_t *tile_node0, *tile_info, *chunk_ptr, *cols, *task_tile, *task_c0, *task_nch, *task_part, *task_ntiles;
    const int16_t* map;
    const int32_t* id_to_cid;
    int32_t num_tasks, num_part, num_chunks, W, ctx_levels;
    const float2* wp;
    int32_t wp_row, num_cids;
};
__global__ void __launch_bounds__(64 * kF32Waves, 4) bwd_kv_f32_tile_kernel(const AttnArgs a, const F32KeyArgs t) {
    __shared__ __align__(16) float o_s[kF32Waves][16][2 * kD + 4];
    extern __shared__ __align__(16) unsigned char smem[];
    int32_t* cid_s = reinterpret_cast<int32_t*>(smem);   // [W] compact id of the level's orders
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, j = lane & 15;
    const int item = xcd_item(blockIdx.x, a.BH * t.num_tasks);
    if (item < 0) return;
    const int bh = item / t.num_tasks, task = item - bh * t.num_tasks;
    const int kt0 = uniform_i32(t.task_tile, task), ntiles = uniform_i32(t.task_ntiles, task), part = uniform_i32(t.task_part, task);
    const int level = uniform_i32(t.tile_info, kt0) & 255;
    for (int i = threadIdx.x; i < t.W; i += blockDim.x) cid_s[i] = level < t.ctx_levels ? max(t.id_to_cid[level * t.W + i], 0) : 0;
    __syncthreads();
    const int64_t base = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh;
    const rsrc_t rQ = make_rsrc(static_cast<const float*>(a.Q) + base, a.slab_bytes);
    const rsrc_t rG = make_rsrc(static_cast<const float*>(a.dout) + base, a.slab_bytes);
    const rsrc_t rS = make_rsrc(a.stat + (int64_t)bh * a.N, (uint32_t)a.N * 8u);
    const rsrc_t rW = make_rsrc(t.wp + (int64_t)bh * a.n_tokens * t.wp_row, (uint32_t)a.n_tokens * (uint32_t)t.wp_row * 8u);
    const rsrc_t rC = make_rsrc(t.cols, (uint32_t)t.num_chunks * 64u);
    const rsrc_t rM = make_rsrc(t.map, (uint32_t)t.num_chunks * 512u);
    const bool single = ntiles == 1;

    for (int kt = kt0 + (single ? 0 : wave); kt < kt0 + ntiles; kt += kF32Waves) {
        const int node0 = uniform_i32(t.tile_node0, kt), nkeys = uniform_i32(t.tile_info, kt) >> 8;
        int c = single ? uniform_i32(t.task_c0, task) + wave : uniform_i32(t.chunk_ptr, kt);
        const int c_end = single ? uniform_i32(t.task_c0, task) + uniform_i32(t.task_nch, task) : uniform_i32(t.chunk_ptr, kt + 1);
        const int c_step = single ? kF32Waves : 1;
        struct Idx {
            int u[4];
            u32x2 m;
            __device__ int bid(int s) const { return (int)(short)((s & 2 ? m.y : m.x) >> (s & 1 ? 16 : 0)); }
        };
        struct Rows {
            f32v4_t q[4], g[4];
            float2 wp[4];
            float delta[4];
        };
        // query 4g + s of the chunk is step s of the products: its map word and its rows belong to lane group g
        auto load_idx = [&](int cc, Idx& x) {
            cc = min(cc, c_end - 1);   // (a chunk past the end repeats the last one: valid addresses, results unused)
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rC, (cc * 16 + 4 * g) * 4, 0, 0);
            x.m = __builtin_amdgcn_raw_buffer_load_b64(rM, (cc * 16 + j) * 32 + 8 * g, 0, 0);
            x.u[0] = (int)v.x; x.u[1] = (int)v.y; x.u[2] = (int)v.z; x.u[3] = (int)v.w;
        };
        auto load_rows = [&](const Idx& x, Rows& r) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int off = (int)__umul24(x.u[s], a.row_bytes) + 16 * j;
                r.q[s] = buf_f4(rQ, off);
                r.g[s] = buf_f4(rG, off);
                // the pair of a token query by (query, its compact id), of an ancestor by (key token, its level)
                const int bid = x.bid(s);
                const bool by_query = bid < t.W;
                const int row = by_query ? x.u[s] : node0 + j, col = by_query ? cid_s[max(bid, 0)] : t.num_cids + bid - t.W;
                r.wp[s] = buf_f2(rW, bid < 0 ? 0 : (row * t.wp_row + col) * 8);
                r.delta[s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rS, x.u[s] * 8 + 4, 0, 0));
            }
        };
        f32x4_t dk[4], dv[4];   // lane (g, j), register r of dk[f] = feature 16 g + 4 r + f of key j
#pragma unroll
        for (int f = 0; f < 4; ++f) dk[f] = dv[f] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (c < c_end) {   // uniform
            Idx x;
            Rows r;
            load_idx(c, x);
            for (; c < c_end; c += c_step) {
                load_rows(x, r);
                bool on[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) on[s] = x.bid(s) >= 0;
                load_idx(c + c_step, x);
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const float p = on[s] ? r.wp[s].y : 0.f, ds = on[s] ? r.wp[s].x - r.delta[s] * r.wp[s].y : 0.f;
#pragma unroll
                    for (int f = 0; f < 4; ++f) {
                        dk[f] = __builtin_amdgcn_mfma_f32_16x16x4f32(r.q[s][f], ds, dk[f], 0, 0, 0);
                        dv[f] = __builtin_amdgcn_mfma_f32_16x16x4f32(r.g[s][f], p, dv[f], 0, 0, 0);
                    }
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const f32x4_t x = {a.scale * dk[0][r], a.scale * dk[1][r], a.scale * dk[2][r], a.scale * dk[3][r]};
            const f32x4_t y = {dv[0][r], dv[1][r], dv[2][r], dv[3][r]};
            *reinterpret_cast<f32x4_t*>(&o_s[wave][j][16 * g + 4 * r]) = x;
            *reinterpret_cast<f32x4_t*>(&o_s[wave][j][kD + 16 * g + 4 * r]) = y;
        }
        if (single)
            __syncthreads();
        else
            wave_lds_sync();
        // features q4 .. q4 + 3 of a key's dK | dV over its own edges in the chunks
        auto again = [&](int key, int q4) {
            const int c_first = single ? uniform_i32(t.task_c0, task) : uniform_i32(t.chunk_ptr, kt);
            f32x4_t sum = {0.f, 0.f, 0.f, 0.f};
            const float* rows = (q4 < kD ? static_cast<const float*>(a.Q) + q4 : static_cast<const float*>(a.dout) + (q4 - kD)) + base;
            for (int i = 16 * c_first; i < 16 * c_end; ++i) {
                const int bid = t.map[((int64_t)(i >> 4) * 16 + key) * 16 + (i & 15)], u = t.cols[i];
                if (bid < 0) continue;
                const int64_t at = bid < t.W ? (int64_t)u * t.wp_row + cid_s[bid] : (int64_t)(node0 + key) * t.wp_row + t.num_cids + bid - t.W;
                const float2 wp = t.wp[(int64_t)bh * a.n_tokens * t.wp_row + at];
                const float c = q4 < kD ? a.scale * (wp.x - a.stat[(int64_t)bh * a.N + u].y * wp.y) : wp.y;
                sum += c * *reinterpret_cast<const f32x4_t*>(rows + (int64_t)u * a.sn);
            }
            return sum;
        };
        // rows of 256 bytes: a thread per (key, 4 of its 64 dK | 64 dV)
        for (int i = single ? (int)threadIdx.x : lane; i < nkeys * 32; i += single ? 64 * kF32Waves : 64) {
            const int key = i >> 5, q4 = (i & 31) * 4;
            f32x4_t v = *reinterpret_cast<const f32x4_t*>(&o_s[single ? 0 : wave][key][q4]);
            if (single)
#pragma unroll
                for (int w = 1; w < kF32Waves; ++w) v += *reinterpret_cast<const f32x4_t*>(&o_s[w][key][q4]);
            if (!all_finite(v[0], v[1], v[2], v[3])) v = again(key, q4);
            if (part < 0)
                store_once(reinterpret_cast<float4*>((q4 < kD ? a.dK + q4 : a.dV + (q4 - kD)) + base + (int64_t)(node0 + key) * a.sn),
                           make_float4(v[0], v[1], v[2], v[3]));
            else   // kv_tile_merge_kernel reads the partial sums
                *reinterpret_cast<f32x4_t*>(a.part + (((int64_t)bh * t.num_part + part) * 16 + key) * (2 * kD) + q4) = v;
        }
        if (!single) wave_lds_sync();
    }
}

}  // namespace
}  // namespace bpt
