// Row-wise kernels of the decoder pass (embedding gather, RMSNorm, rotary
// embedding + cache scatter).
#include <math.h>

#include <algorithm>

#include "common.h"

namespace kvr {

namespace {

__device__ __forceinline__ float warp_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Sum over a block of up to 16 wavefronts, in wavefront order.
__device__ __forceinline__ float block_sum(float v, float *red) {
    v = warp_sum(v);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, nw = blockDim.x >> 6;
    if (l == 0) red[w] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int q = 0; q < 16; ++q) t += q < nw ? red[q] : 0.f;
    return t;
}

// h4 = H[r][4i..4i+3] + the split-K partial tiles part[q][r][4i..] in order
// (batches of eight independent loads).
__device__ __forceinline__ float4 add_partials(float4 h, const float *part, int nsplit, int R, int r, int d, int i) {
    constexpr int B = 8;
    int q = 0;
    for (; q + B <= nsplit; q += B) {
        float4 p[B];
#pragma unroll
        for (int u = 0; u < B; ++u) p[u] = *reinterpret_cast<const float4 *>(part + ((size_t)(q + u) * R + r) * d + 4 * i);
#pragma unroll
        for (int u = 0; u < B; ++u) { h.x += p[u].x; h.y += p[u].y; h.z += p[u].z; h.w += p[u].w; }
    }
    if (q < nsplit) {
        float4 p[B];
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (q + u < nsplit) p[u] = *reinterpret_cast<const float4 *>(part + ((size_t)(q + u) * R + r) * d + 4 * i);
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (q + u < nsplit) { h.x += p[u].x; h.y += p[u].y; h.z += p[u].z; h.w += p[u].w; }
    }
    return h;
}

// Four gains (8-byte or 16-byte aligned: d and the column are multiples of four).
__device__ __forceinline__ float4 load_gain4(const float *g) { return *reinterpret_cast<const float4 *>(g); }
__device__ __forceinline__ float4 load_gain4(const bf16_t *g) {
    const uint2 u = *reinterpret_cast<const uint2 *>(g);
    return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                       __uint_as_float(u.y & 0xffff0000u));
}

constexpr int NORM_V = 4;  // float4 per thread of the row kernels: d <= 16384

// Four consecutive outputs (columns c..c+3, c % 4 == 0) of an operand row;
// they are contiguous in both the row-major and the operand-order layout.
template <typename T>
__device__ __forceinline__ void store_operand4(T *hi, T *lo, size_t off, const float (&x)[4]) {
    if constexpr (sizeof(T) == 4) {
        *reinterpret_cast<float4 *>(hi + off) = make_float4(x[0], x[1], x[2], x[3]);
    } else {
        uint32_t h[2], l[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const bf16_t h0 = f32_to_bf16(x[2 * q]), h1 = f32_to_bf16(x[2 * q + 1]);
            h[q] = (uint32_t)h0 | ((uint32_t)h1 << 16);
            const bf16_t l0 = f32_to_bf16(x[2 * q] - bf16_to_f32(h0)), l1 = f32_to_bf16(x[2 * q + 1] - bf16_to_f32(h1));
            l[q] = (uint32_t)l0 | ((uint32_t)l1 << 16);
        }
        *reinterpret_cast<uint2 *>(hi + off) = make_uint2(h[0], h[1]);
        if (lo) *reinterpret_cast<uint2 *>(lo + off) = make_uint2(l[0], l[1]);
    }
}

// Where a normalised row goes: the next projection's operand (row-major or
// operand order), after which the residual row is needed again, or the
// caller's hidden row (null: nobody reads it), after the last layer.
template <typename TO, bool PERM>
struct OperandOut {
    static constexpr bool KEEP_H = true;
    TO *X, *X_lo;
    int ldx;
    __device__ __forceinline__ bool begin(int) { return true; }
    __device__ __forceinline__ void put(int r, int c, int d, const float (&x)[4]) const {
        store_operand4(X, X_lo, PERM ? perm_offset(r, c, d) : (size_t)r * ldx + c, x);
    }
};
struct HiddenOut {
    static constexpr bool KEEP_H = false;
    const RowInfo *rows;
    const DocInfo *docs;
    float *dst;
    __device__ __forceinline__ bool begin(int r) {
        const RowInfo ri = rows[r];
        dst = docs[ri.doc].hidden_out;
        out = ri.out;
        return dst != nullptr;
    }
    __device__ __forceinline__ void put(int, int c, int d, const float (&x)[4]) const {
        *reinterpret_cast<float4 *>(dst + (size_t)out * d + c) = make_float4(x[0], x[1], x[2], x[3]);
    }
    int out;
};

// H[r] += sum of the split-K partial tiles (fixed order; sum_first: added to
// each other before H), then H * rsqrt(mean(H^2) + eps) * gain to `o`.  One block per row, as many
// wavefronts as the row has 256-column pieces, at most 16; the row stays in
// registers between the two passes (four columns per thread per pass, d % 4
// == 0).  After the last layer H is not written back.
template <typename TG, typename OUT>
__global__ __launch_bounds__(1024) void rmsnorm_kernel(float *H, const float *part, int nsplit, bool sum_first, int R,
                                                       const TG *gain, int d, float eps, OUT o) {
    __shared__ float red[16];
    const int r = blockIdx.x;
    if (!o.begin(r)) return;
    float *h = H + (size_t)r * d;
    float4 v[NORM_V], gn[NORM_V];
    float ss = 0.f;
#pragma unroll
    for (int k = 0; k < NORM_V; ++k) {
        const int i = threadIdx.x + blockDim.x * k;
        if (4 * i >= d) break;
        gn[k] = load_gain4(gain + 4 * i);
        v[k] = *reinterpret_cast<const float4 *>(h + 4 * i);
        if (nsplit) {
            if (sum_first) {
                float4 p = *reinterpret_cast<const float4 *>(part + (size_t)r * d + 4 * i);
                p = add_partials(p, part + (size_t)R * d, nsplit - 1, R, r, d, i);
                v[k].x += p.x; v[k].y += p.y; v[k].z += p.z; v[k].w += p.w;
            } else {
                v[k] = add_partials(v[k], part, nsplit, R, r, d, i);
            }
            if (OUT::KEEP_H) *reinterpret_cast<float4 *>(h + 4 * i) = v[k];
        }
        ss += v[k].x * v[k].x + v[k].y * v[k].y + v[k].z * v[k].z + v[k].w * v[k].w;
    }
    ss = block_sum(ss, red);
    const float inv = rsqrtf(ss / (float)d + eps);
#pragma unroll
    for (int k = 0; k < NORM_V; ++k) {
        const int i = threadIdx.x + blockDim.x * k;
        if (4 * i >= d) break;
        const float x[4] = {v[k].x * inv * gn[k].x, v[k].y * inv * gn[k].y, v[k].z * inv * gn[k].z, v[k].w * inv * gn[k].w};
        o.put(r, 4 * i, d, x);
    }
}

// The same for many rows with few partial tiles (prefill, batched repair):
// one wavefront per row, each lane holding NV float4 of it, so that the row
// and a partial tile are loaded in one round (NV + NV loads in flight per
// lane) and no block barrier is needed.  A 1024-thread block per row keeps one
// load per thread in flight and waits at two barriers; at 5000 rows that
// kernel ran at 3.4 TB/s.  Results are bit-identical to it (d <= 4096, where
// it holds one float4 per thread).
template <typename TG, typename OUT, int NV>
__global__ __launch_bounds__(512) void rmsnorm_wave_kernel(float *H, const float *part, int nsplit, int R,
                                                           const TG *gain, int d, float eps, OUT o) {
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * 8 + (threadIdx.x >> 6);
    if (r >= R || !o.begin(r)) return;
    float *h = H + (size_t)r * d;
    float4 v[NV], p[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int c = 4 * (lane + 64 * k);
        v[k] = c < d ? *reinterpret_cast<const float4 *>(h + c) : make_float4(0.f, 0.f, 0.f, 0.f);
        if (nsplit > 0)
            p[k] = c < d ? *reinterpret_cast<const float4 *>(part + (size_t)r * d + c) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    for (int q = 0; q < nsplit; ++q) {  // partial tiles in order
        if (q > 0) {
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                const int c = 4 * (lane + 64 * k);
                p[k] = c < d ? *reinterpret_cast<const float4 *>(part + ((size_t)q * R + r) * d + c)
                             : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
#pragma unroll
        for (int k = 0; k < NV; ++k) { v[k].x += p[k].x; v[k].y += p[k].y; v[k].z += p[k].z; v[k].w += p[k].w; }
    }
    // the sum of squares in the row kernel's order (float4 k of lane l is the
    // row kernel's thread 64 k + l): a wavefront sum per k, then the sums in
    // k order, so that both kernels normalise a row bit for bit alike (a row
    // must not depend on how many rows the pass has)
    float ss = 0.f;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int c = 4 * (lane + 64 * k);
        float t = 0.f;
        if (c < d) {
            if (OUT::KEEP_H && nsplit) *reinterpret_cast<float4 *>(h + c) = v[k];
            t = v[k].x * v[k].x + v[k].y * v[k].y + v[k].z * v[k].z + v[k].w * v[k].w;
        }
        ss += warp_sum(t);
    }
    const float inv = rsqrtf(ss / (float)d + eps);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int c = 4 * (lane + 64 * k);
        if (c >= d) continue;
        const float x[4] = {v[k].x * inv * to_f32(gain[c]), v[k].y * inv * to_f32(gain[c + 1]),
                            v[k].z * inv * to_f32(gain[c + 2]), v[k].w * inv * to_f32(gain[c + 3])};
        o.put(r, c, d, x);
    }
}

// Adds the Q/K/V bias, rotates Q and K at the row's absolute position
// (rotate-half pairing) and scatters K and V into the row's cache slot; Q goes
// to the attention operand buffer [R][Hq*hd].
template <typename T>
__global__ __launch_bounds__(1024) void rope_scatter_kernel(const float *qkv, int nsplit, int R, const T *bq,
                                                           const T *bk, const T *bv, const RowInfo *rows,
                                                           const DocInfo *docs, int layer, int Hq, int Hkv, int hd,
                                                           const float *rcos, const float *rsin, T *Q, T *Q_lo) {
    const int r = blockIdx.x;
    const RowInfo ri = rows[r];
    const DocInfo dc = docs[ri.doc];
    const int half = hd >> 1;
    const int qd = Hq * hd, kd = Hkv * hd;
    const int N = qd + 2 * kd;
    // sum the split-K partial tiles of this row into LDS first
    extern __shared__ float row[];
    for (int i = threadIdx.x; 4 * i < N; i += 1024) {
        float4 v = *reinterpret_cast<const float4 *>(qkv + (size_t)r * N + 4 * i);
        if (nsplit > 1) v = add_partials(v, qkv + (size_t)R * N, nsplit - 1, R, r, N, i);
        *reinterpret_cast<float4 *>(row + 4 * i) = v;
    }
    __syncthreads();
    const float *cs = rcos + (size_t)ri.pos * half;
    const float *sn = rsin + (size_t)ri.pos * half;
    T *cache = (T *)dc.cache;
    const size_t head_stride = (size_t)dc.n_cap * hd;
    T *kbase = cache + ((size_t)layer * 2 + 0) * Hkv * head_stride + (size_t)ri.pos * hd;
    T *vbase = cache + ((size_t)layer * 2 + 1) * Hkv * head_stride + (size_t)ri.pos * hd;
    for (int idx = threadIdx.x; idx < (Hq + Hkv) * half; idx += 1024) {
        const int j = idx / half, i = idx - j * half;
        float a, b;
        if (j < Hq) {
            a = row[j * hd + i];
            b = row[j * hd + i + half];
            if (bq) { a += to_f32(bq[j * hd + i]); b += to_f32(bq[j * hd + i + half]); }
        } else {
            const int g = j - Hq;
            a = row[qd + g * hd + i];
            b = row[qd + g * hd + i + half];
            if (bk) { a += to_f32(bk[g * hd + i]); b += to_f32(bk[g * hd + i + half]); }
        }
        const float c = cs[i], s = sn[i];
        const float o1 = a * c - b * s, o2 = b * c + a * s;
        if (j < Hq) {
            store_operand(Q, Q_lo, (size_t)r * qd + j * hd + i, o1);
            store_operand(Q, Q_lo, (size_t)r * qd + j * hd + i + half, o2);
        } else {
            const int g = j - Hq;
            kbase[g * head_stride + i] = from_f32<T>(o1);
            kbase[g * head_stride + i + half] = from_f32<T>(o2);
        }
    }
    for (int idx = threadIdx.x; idx < kd; idx += 1024) {
        const int g = idx / hd, i = idx - g * hd;
        float v = row[qd + kd + idx];
        if (bv) v += to_f32(bv[idx]);
        vbase[g * head_stride + i] = from_f32<T>(v);
    }
}

// Residual update for a pass whose projections apply the RMS scale to their
// outputs (the skinny path): H[r] += the `nsplit` partial tiles (in order),
// X = H * gain as a compensated operand in operand order, and ssq[b][r] = the
// sum of H[r][c]^2 over the 1024 columns of column block b (fixed reduction
// order).  RMSNorm's scale is one factor per row and the projection is
// linear, so the projection that reads X multiplies its output row r by
// rsqrt((ssq[0][r] + ... ) / d + eps) instead; the work then spreads over
// (row, column block) blocks rather than one block per row.
template <typename G>
__global__ __launch_bounds__(256) void resid_gain_kernel(float *H, const float *part, int nsplit, int R, const G *gain,
                                                         int d, bf16_t *X, bf16_t *X_lo, float *ssq) {
    __shared__ float red[4];
    const int r = blockIdx.x, b = blockIdx.y;
    const int i = b * 256 + threadIdx.x;  // float4 index within the row
    float ss = 0.f;
    if (4 * i < d) {
        // the gain is loaded with the row: after the store of H it would be a
        // round trip of its own (the compiler cannot move it across the store)
        float *hp = H + (size_t)r * d + 4 * i;
        float4 h = *reinterpret_cast<const float4 *>(hp);
        const float4 gn = load_gain4(gain + 4 * i);
        if (nsplit) {
            h = add_partials(h, part, nsplit, R, r, d, i);
            *reinterpret_cast<float4 *>(hp) = h;
        }
        ss = h.x * h.x + h.y * h.y + h.z * h.z + h.w * h.w;
        const float4 x = {h.x * gn.x, h.y * gn.y, h.z * gn.z, h.w * gn.w};
        const bf16_t hi[4] = {f32_to_bf16(x.x), f32_to_bf16(x.y), f32_to_bf16(x.z), f32_to_bf16(x.w)};
        const bf16_t lo[4] = {f32_to_bf16(x.x - bf16_to_f32(hi[0])), f32_to_bf16(x.y - bf16_to_f32(hi[1])),
                              f32_to_bf16(x.z - bf16_to_f32(hi[2])), f32_to_bf16(x.w - bf16_to_f32(hi[3]))};
        const size_t o = perm_offset(r, 4 * i, d);  // four consecutive columns are adjacent in operand order
        *reinterpret_cast<uint2 *>(X + o) =
            make_uint2((uint32_t)hi[0] | ((uint32_t)hi[1] << 16), (uint32_t)hi[2] | ((uint32_t)hi[3] << 16));
        *reinterpret_cast<uint2 *>(X_lo + o) =
            make_uint2((uint32_t)lo[0] | ((uint32_t)lo[1] << 16), (uint32_t)lo[2] | ((uint32_t)lo[3] << 16));
    }
    ss = warp_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    if (threadIdx.x == 0) ssq[(size_t)b * R + r] = ((red[0] + red[1]) + red[2]) + red[3];
}

// The first kernel of a pass: H[r] = embed[token of row r] and, when the first
// projections apply the RMS scale (GAIN), layer 0's X = H * gain and sums of
// squares as resid_gain_kernel makes them, by (row, 1024-column block).  Token
// ids outside [0, vocab) are clamped into range rather than read out of
// bounds.
//
// The pass's tables may still be in pinned host memory: the blocks past
// `row_blocks` then copy them to the device while the others run, and the row
// kernels' blocks take their rows from the kernel argument (one document, up
// to EMBED_ROWS rows) or from host memory.  A copy, the embedding and the
// first norm were three launches of about 4 us and a boundary each.
template <typename TW, bool GAIN>
__global__ __launch_bounds__(256) void embed_kernel(EmbedArgs a, const TW *embed, const TW *gain, int d, int vocab,
                                                    float *H, bf16_t *X, bf16_t *X_lo, float *ssq) {
    if ((int)blockIdx.x >= a.row_blocks) {
        const int i = ((int)blockIdx.x - a.row_blocks) * 256 + (int)threadIdx.x;
        if (i < a.upload_16) a.upload_dst[i] = a.upload_src[i];
        return;
    }
    __shared__ float red[4];
    const int nb = (d + 1023) >> 10;
    const int r = blockIdx.x / nb, b = blockIdx.x - r * nb;
    const int32_t *tokens = a.tokens;
    int pos;
    if (tokens) {
        pos = a.pos[r];
    } else {
        const RowInfo ri = a.rows[r];
        pos = ri.pos;
        tokens = a.docs[ri.doc].tokens;
    }
    const int tok = min(max(tokens[pos], 0), vocab - 1);
    const int c = b * 1024 + 4 * (int)threadIdx.x;  // d is a multiple of four
    float ss = 0.f;
    if (c < d) {
        const TW *src = embed + (size_t)tok * d + c;
        float4 h;
        if constexpr (sizeof(TW) == 2) {
            const uint2 u = *reinterpret_cast<const uint2 *>(src);
            h = make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                            __uint_as_float(u.y & 0xffff0000u));
        } else {
            h = *reinterpret_cast<const float4 *>(src);
        }
        float4 gn = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (GAIN) gn = load_gain4(gain + c);
        *reinterpret_cast<float4 *>(H + (size_t)r * d + c) = h;
        if constexpr (GAIN) {
            ss = h.x * h.x + h.y * h.y + h.z * h.z + h.w * h.w;
            const float x[4] = {h.x * gn.x, h.y * gn.y, h.z * gn.z, h.w * gn.w};
            store_operand4(X, X_lo, perm_offset(r, c, d), x);
        }
    }
    if constexpr (GAIN) {
        ss = warp_sum(ss);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
        __syncthreads();
        if (threadIdx.x == 0) ssq[(size_t)b * a.R + r] = ((red[0] + red[1]) + red[2]) + red[3];
    }
}

__global__ __launch_bounds__(256) void table_chunk_kernel(TableChunk c, u32x4 *dst) {
    if ((int)threadIdx.x < c.n16) dst[threadIdx.x] = c.data[threadIdx.x];
}

// Four values of row-major type T at p (8-byte or 16-byte store).
template <typename T>
__device__ __forceinline__ void store4(T *p, float4 v) {
    if constexpr (sizeof(T) == 4) {
        *reinterpret_cast<float4 *>(p) = v;
    } else {
        const uint32_t a = (uint32_t)f32_to_bf16(v.x) | ((uint32_t)f32_to_bf16(v.y) << 16);
        const uint32_t b = (uint32_t)f32_to_bf16(v.z) | ((uint32_t)f32_to_bf16(v.w) << 16);
        *reinterpret_cast<uint2 *>(p) = make_uint2(a, b);
    }
}
// Four consecutive operand values (store_operand for each, vectorised).
template <typename T>
__device__ __forceinline__ void store4_operand(T *hi, T *lo, size_t i, float4 v) {
    if constexpr (sizeof(T) == 4) {
        store4(hi + i, v);
    } else {
        const bf16_t h[4] = {f32_to_bf16(v.x), f32_to_bf16(v.y), f32_to_bf16(v.z), f32_to_bf16(v.w)};
        *reinterpret_cast<uint2 *>(hi + i) =
            make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16));
        if (lo) {
            const float4 d = {v.x - bf16_to_f32(h[0]), v.y - bf16_to_f32(h[1]), v.z - bf16_to_f32(h[2]),
                              v.w - bf16_to_f32(h[3])};
            store4(lo + i, d);
        }
    }
}
template <typename T>
__device__ __forceinline__ float4 load4_f32(const T *p) {
    if constexpr (sizeof(T) == 4) return *reinterpret_cast<const float4 *>(p);
    else return float4{to_f32(p[0]), to_f32(p[1]), to_f32(p[2]), to_f32(p[3])};
}

// The same as rope_scatter_kernel with one thread per (row, head, four
// rotary pairs) and per (row, four value dimensions): nothing in it is
// reduced over a row, so the work spreads over all compute units instead of
// one block per row (head_dim a multiple of 8).
template <typename T>
__global__ __launch_bounds__(256) void rope_scatter_vec_kernel(const float *qkv, int nsplit, int R, const T *bq,
                                                               const T *bk, const T *bv, const RowInfo *rows,
                                                               const DocInfo *docs, int layer, int Hq, int Hkv, int hd,
                                                               const float *rcos, const float *rsin, T *Q, T *Q_lo) {
    const int r = blockIdx.x;
    const int idx = blockIdx.y * 256 + threadIdx.x;
    const int half = hd >> 1, hq4 = half >> 2;
    const int qd = Hq * hd, kd = Hkv * hd;
    const int N = qd + 2 * kd;
    const int nrot = (Hq + Hkv) * hq4;
    if (idx >= nrot + (kd >> 2)) return;
    // columns c..c+3 of this row, the split-K partial tiles summed in order
    auto load4 = [&](int c) {
        float4 v = *reinterpret_cast<const float4 *>(qkv + (size_t)r * N + c);
        for (int q = 1; q < nsplit; ++q) {
            const float4 p = *reinterpret_cast<const float4 *>(qkv + ((size_t)q * R + r) * N + c);
            v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
        }
        return v;
    };
    if (idx < nrot) {
        const int j = (hq4 & (hq4 - 1)) == 0 ? idx >> __builtin_ctz(hq4) : idx / hq4, i = (idx - j * hq4) * 4;
        const bool isq = j < Hq;
        const int g = j - Hq;
        const int ca = isq ? j * hd + i : qd + g * hd + i;
        // the partials do not wait for the row's position and document
        float4 a = load4(ca), b = load4(ca + half);
        const RowInfo ri = rows[r];
        const DocInfo dc = docs[ri.doc];
        T *cache = (T *)dc.cache;
        const size_t head_stride = (size_t)dc.n_cap * hd;
        const T *bias = isq ? bq : bk;
        if (bias) {
            const int bo = (isq ? j : g) * hd + i;
            const float4 ba = load4_f32(bias + bo), bb = load4_f32(bias + bo + half);
            a.x += ba.x; a.y += ba.y; a.z += ba.z; a.w += ba.w;
            b.x += bb.x; b.y += bb.y; b.z += bb.z; b.w += bb.w;
        }
        const float4 c = *reinterpret_cast<const float4 *>(rcos + (size_t)ri.pos * half + i);
        const float4 sn = *reinterpret_cast<const float4 *>(rsin + (size_t)ri.pos * half + i);
        const float4 o1 = {a.x * c.x - b.x * sn.x, a.y * c.y - b.y * sn.y, a.z * c.z - b.z * sn.z, a.w * c.w - b.w * sn.w};
        const float4 o2 = {b.x * c.x + a.x * sn.x, b.y * c.y + a.y * sn.y, b.z * c.z + a.z * sn.z, b.w * c.w + a.w * sn.w};
        if (isq) {
            store4_operand(Q, Q_lo, (size_t)r * qd + j * hd + i, o1);
            store4_operand(Q, Q_lo, (size_t)r * qd + j * hd + i + half, o2);
        } else {
            T *kb = cache + (((size_t)layer * 2 + 0) * Hkv + g) * head_stride + (size_t)ri.pos * hd;
            store4(kb + i, o1);
            store4(kb + i + half, o2);
        }
    } else {
        const int c4 = (idx - nrot) * 4;  // column of the value part [0, kd)
        float4 v = load4(qd + kd + c4);
        const RowInfo ri = rows[r];
        const DocInfo dc = docs[ri.doc];
        T *cache = (T *)dc.cache;
        const size_t head_stride = (size_t)dc.n_cap * hd;
        if (bv) {
            const float4 bb = load4_f32(bv + c4);
            v.x += bb.x; v.y += bb.y; v.z += bb.z; v.w += bb.w;
        }
        const int g = (hd & (hd - 1)) == 0 ? c4 >> __builtin_ctz(hd) : c4 / hd, i = c4 - g * hd;
        T *vb = cache + (((size_t)layer * 2 + 1) * Hkv + g) * head_stride + (size_t)ri.pos * hd;
        store4(vb + i, v);
    }
}

}  // namespace

hipError_t launch_embed(bool bf16, const EmbedArgs &args, const void *embed, const void *gain, int d, int vocab, float *H,
                        void *X, void *X_lo, float *ssq, hipStream_t s) {
    if (args.R <= 0) return hipSuccess;
    if (d % 4 != 0 || (gain && (!bf16 || d % 32 != 0 || !X || !X_lo || !ssq))) return hipErrorInvalidValue;
    EmbedArgs a = args;
    a.row_blocks = a.R * resid_gain_blocks(d);
    const dim3 grid(a.row_blocks + (a.upload_16 + 255) / 256);
    if (bf16 && gain)
        kvr_launch((embed_kernel<bf16_t, true>), grid, dim3(256), 0, s, a, (const bf16_t *)embed, (const bf16_t *)gain, d,
                   vocab, H, (bf16_t *)X, (bf16_t *)X_lo, ssq);
    else if (bf16)
        kvr_launch((embed_kernel<bf16_t, false>), grid, dim3(256), 0, s, a, (const bf16_t *)embed, (const bf16_t *)nullptr,
                   d, vocab, H, (bf16_t *)nullptr, (bf16_t *)nullptr, (float *)nullptr);
    else
        kvr_launch((embed_kernel<float, false>), grid, dim3(256), 0, s, a, (const float *)embed, (const float *)nullptr, d,
                   vocab, H, (bf16_t *)nullptr, (bf16_t *)nullptr, (float *)nullptr);
    return hipGetLastError();
}

hipError_t launch_table_chunk(const TableChunk &chunk, void *dst, hipStream_t s) {
    if (chunk.n16 < 1 || chunk.n16 > (int)(sizeof(chunk.data) / 16)) return hipErrorInvalidValue;
    kvr_launch(table_chunk_kernel, dim3(1), dim3(256), 0, s, chunk, (u32x4 *)dst);
    return hipGetLastError();
}

// Many rows and few partial tiles: a wavefront per row (d <= 4096).  Its blocks
// of eight rows leave units idle below a thousand rows (528 rows, three
// partial tiles: 21 us, 25 us in blocks of one row, against 17 us).  It adds
// several tiles to H one by one only.
template <typename TG, typename OUT>
static hipError_t launch_norm(float *H, const float *part, int nsplit, bool sum_first, const TG *gain, int R, int d,
                              float eps, OUT o, hipStream_t s) {
    if (R >= 1024 && nsplit <= (sum_first ? 1 : 3) && d <= 4096) {
        kvr_launch((rmsnorm_wave_kernel<TG, OUT, 16>), dim3((R + 7) / 8), dim3(512), 0, s, H, part, nsplit, R, gain, d, eps,
                   o);
    } else {
        const int threads = std::min(1024, (d / 4 + 63) / 64 * 64);
        kvr_launch((rmsnorm_kernel<TG, OUT>), dim3(R), dim3(threads), 0, s, H, part, nsplit, sum_first, R, gain, d, eps, o);
    }
    return hipGetLastError();
}

hipError_t launch_rmsnorm(bool bf16, float *H, const float *part, int nsplit, bool sum_first, const void *gain, int R, int d,
                          float eps, void *X, void *X_lo, int ldx, bool perm, hipStream_t s) {
    if (R <= 0) return hipSuccess;
    if (d % 4 != 0 || d > 4 * 1024 * NORM_V || (!perm && ldx % 4 != 0) || (!bf16 && perm)) return hipErrorInvalidValue;
    if (!bf16)
        return launch_norm(H, part, nsplit, sum_first, (const float *)gain, R, d, eps,
                           OperandOut<float, false>{(float *)X, nullptr, ldx}, s);
    if (perm)
        return launch_norm(H, part, nsplit, sum_first, (const bf16_t *)gain, R, d, eps,
                           OperandOut<bf16_t, true>{(bf16_t *)X, (bf16_t *)X_lo, ldx}, s);
    return launch_norm(H, part, nsplit, sum_first, (const bf16_t *)gain, R, d, eps,
                       OperandOut<bf16_t, false>{(bf16_t *)X, (bf16_t *)X_lo, ldx}, s);
}

int resid_gain_blocks(int d) { return (d + 1023) / 1024; }

hipError_t launch_resid_gain(bool bf16_gain, float *H, const float *part, int nsplit, const void *gain, int R, int d,
                             void *X, void *X_lo, float *ssq, hipStream_t s) {
    if (R <= 0) return hipSuccess;
    if (d % 32 != 0 || !X || !X_lo || !ssq) return hipErrorInvalidValue;
    const dim3 grid(R, resid_gain_blocks(d));
    if (bf16_gain)
        kvr_launch(resid_gain_kernel<bf16_t>, grid, dim3(256), 0, s, H, part, nsplit, R, (const bf16_t *)gain, d,
                   (bf16_t *)X, (bf16_t *)X_lo, ssq);
    else
        kvr_launch(resid_gain_kernel<float>, grid, dim3(256), 0, s, H, part, nsplit, R, (const float *)gain, d,
                   (bf16_t *)X, (bf16_t *)X_lo, ssq);
    return hipGetLastError();
}

hipError_t launch_final_norm(bool bf16_gain, float *H, const float *part, int nsplit, bool sum_first, const void *gain,
                             const RowInfo *rows, const DocInfo *docs, int R, int d, float eps, hipStream_t s) {
    if (R <= 0) return hipSuccess;
    if (d % 4 != 0 || d > 4 * 1024 * NORM_V) return hipErrorInvalidValue;
    const HiddenOut o{rows, docs, nullptr, 0};
    if (bf16_gain) return launch_norm(H, part, nsplit, sum_first, (const bf16_t *)gain, R, d, eps, o, s);
    return launch_norm(H, part, nsplit, sum_first, (const float *)gain, R, d, eps, o, s);
}

hipError_t launch_rope_scatter(bool bf16, const float *qkv, int nsplit, const void *bq, const void *bk,
                               const void *bv, const RowInfo *rows, const DocInfo *docs, int R, int layer, int Hq,
                               int Hkv, int hd, const float *rope_cos, const float *rope_sin, void *Q, void *Q_lo,
                               hipStream_t s) {
    if (R <= 0) return hipSuccess;
    if (hd % 8 == 0) {
        const int work = (Hq + Hkv) * (hd / 8) + Hkv * hd / 4;  // threads per row
        const dim3 grid(R, (work + 255) / 256);
        if (bf16)
            kvr_launch(rope_scatter_vec_kernel<bf16_t>, grid, dim3(256), 0, s, qkv, nsplit, R, (const bf16_t *)bq,
                       (const bf16_t *)bk, (const bf16_t *)bv, rows, docs, layer, Hq, Hkv, hd, rope_cos, rope_sin,
                       (bf16_t *)Q, (bf16_t *)Q_lo);
        else
            kvr_launch(rope_scatter_vec_kernel<float>, grid, dim3(256), 0, s, qkv, nsplit, R, (const float *)bq,
                       (const float *)bk, (const float *)bv, rows, docs, layer, Hq, Hkv, hd, rope_cos, rope_sin,
                       (float *)Q, (float *)nullptr);
        return hipGetLastError();
    }
    const size_t lds = (size_t)(Hq + 2 * Hkv) * hd * sizeof(float);
    if (lds > 160 * 1024 || ((Hq + 2 * Hkv) * hd) % 4 != 0) return hipErrorInvalidValue;
    if (bf16)
        kvr_launch(rope_scatter_kernel<bf16_t>, dim3(R), dim3(1024), lds, s, qkv, nsplit, R,
                           (const bf16_t *)bq, (const bf16_t *)bk, (const bf16_t *)bv, rows, docs, layer, Hq, Hkv, hd,
                           rope_cos, rope_sin, (bf16_t *)Q, (bf16_t *)Q_lo);
    else
        kvr_launch(rope_scatter_kernel<float>, dim3(R), dim3(1024), lds, s, qkv, nsplit, R,
                           (const float *)bq, (const float *)bk, (const float *)bv, rows, docs, layer, Hq, Hkv, hd,
                           rope_cos, rope_sin, (float *)Q, (float *)nullptr);
    return hipGetLastError();
}

}  // namespace kvr
