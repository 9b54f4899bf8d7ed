// Linear layer for fp32 models and for the bf16 shapes that the packed-weight
// kernels do not take (any R, N, K): row-major operands, products on
// v_mfma_f32_16x16x4_f32 with fp32 accumulation.
//
// Y[r][n] = sum_k X[r][k] * W[n][k].  A bf16 activation pair (hi + lo) is
// summed to fp32 on load.  A lane of an operand fragment holds row (column)
// l%16 and, as one float4, k = 16 s + 4 (l/16) .. +3: instruction c of a step
// multiplies component c of both sides (the sum over k does not mind the
// order).
//
// Up to 64 rows (linear_generic_kernel): a block owns all rows and one 16-wide
// column tile (SwiGLU: the gate and the up tile of 16 features), its four
// wavefronts split the K range and are summed in LDS in a fixed order; every
// wavefront reads its operands straight from memory with a ring of D steps of
// loads in flight.  More rows (linear_generic_tiled_kernel): 64 x 64 or
// 128 x 128 output tiles, four wavefronts of 32 x 32 (64 x 64) each, operands
// staged through two LDS stages of 32 k, whose rows are padded by four floats
// (a fragment's 16 rows then fall on distinct banks).  Reading 32 x 32
// wavefront tiles straight from memory was bound by the bytes a compute unit
// takes in (16 rows x 64 bytes per load: Q/K/V of
// 1501 rows 21 us, where the LDS tile takes 13).
//
// One K order for every row count.  K is cut into kslices slices of four
// quarters (part_start: at 32-wide k-steps, by K and the slice count alone,
// which generic_slices takes from N and K).  A quarter is one chain of
// products, a slice the sum of its quarters in order, an output the sum of its
// slices in order.  Up to 64 rows, a quarter is a wavefront and a slice a
// block (grid z) whose fp32 partial tile the next row kernel sums in slice
// order; the tiled kernel walks the same quarters and adds them up alike,
// either one slice per block or all of them (split 1).  A row's result
// therefore does not depend on the rows it shares a pass with: equal tokens at
// equal positions have bit-equal keys and values at layer 0, whether a prefill
// or a suffix computed them (CacheBlend's deviations there are exactly zero).
//
// What bounds it: latency for a few rows (a 256 x 256 projection of 40 rows is
// four steps per wavefront), the fp32 matrix rate and the fill of the chip for
// a prefill.  Tiny fp32 decoder, us per layer (Q/K/V, output, gate/up, down)
// against 64 x 64 tiles with scalar products: 40 rows 36, 94, 32, 41 -> 6, 6,
// 8, 7; 1501 rows 54, 44, 62, 101 -> 13, 9, 20, 13.
#include <math.h>

#include <algorithm>

#include "common.h"

namespace kvr {

namespace {

__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + expf(-z)); }

// Four consecutive elements of a row.  VEC: K is a multiple of four, so the
// row is aligned for one load.
template <bool VEC>
__device__ __forceinline__ f32x4 load4(const float *p) {
    if constexpr (VEC) return *reinterpret_cast<const f32x4 *>(p);
    return f32x4{p[0], p[1], p[2], p[3]};
}
template <bool VEC>
__device__ __forceinline__ f32x4 load4(const bf16_t *p) {
    if constexpr (VEC) {
        const uint2 u = *reinterpret_cast<const uint2 *>(p);
        return f32x4{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                     __uint_as_float(u.y & 0xffff0000u)};
    }
    return f32x4{bf16_to_f32(p[0]), bf16_to_f32(p[1]), bf16_to_f32(p[2]), bf16_to_f32(p[3])};
}
// Up to four elements, zeros past `left` of them.
template <typename T>
__device__ __forceinline__ f32x4 load_tail(const T *p, int left) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (e < left) v[e] = to_f32(p[e]);
    return v;
}

// First 32-wide k-step of part i of `parts` (quarters of a slice).
__device__ __forceinline__ int part_start(int steps, int i, int parts) { return steps * i / parts; }

// Row-major weight row of output column n (SwiGLU: part 0 gate, 1 up).
template <typename T, int EPI>
__device__ __forceinline__ const T *weight_row(const LinearArgs &a, int n, int part) {
    if (EPI == EPI_SWIGLU) return (const T *)a.w[part] + (size_t)n * a.K;
    const int q = n < a.seg_end[0] ? 0 : (n < a.seg_end[1] ? 1 : 2);
    return (const T *)a.w[q] + (size_t)(n - (q ? a.seg_end[q - 1] : 0)) * a.K;
}

// Rows r0 + 16 m + 4 (lane/16) + e, column n of an accumulator tile (the layout:
// lane l holds tile column l%16); add: to what this thread stored there before.
template <typename T, int EPI>
__device__ __forceinline__ void store_tile(const LinearArgs &a, int r, int n, f32x4 v, f32x4 up, bool add = false) {
    if (n >= a.N) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (r + e >= a.R) continue;
        if (EPI == EPI_SWIGLU)
            store_operand((T *)a.out, (T *)a.out_lo, (size_t)(r + e) * a.ldo + n, silu_f(v[e]) * up[e]);
        else {
            float *o = (float *)a.out + ((size_t)blockIdx.z * a.R + r + e) * a.ldo + n;
            *o = add ? *o + v[e] : v[e];
        }
    }
}

template <typename T, int EPI, int MT, bool VEC>
__global__ __launch_bounds__(256) void linear_generic_kernel(LinearArgs a) {
    constexpr int NT = EPI == EPI_SWIGLU ? 2 : 1, KW = 4;
    constexpr int D = 4;  // k-steps of loads in flight
    __shared__ __attribute__((aligned(16))) float red[(KW - 1) * MT * NT * 256];
    const int lane = threadIdx.x & 63, g = lane >> 4;
    const int kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c0 = blockIdx.x * 16;
    const int steps = a.K >> 4, pairs = (a.K + 31) >> 5;  // whole 16-wide k-steps; 32-wide ones, the last may be shorter
    const int part = blockIdx.z * KW + kw, parts = gridDim.z * KW;
    const int s0 = 2 * part_start(pairs, part, parts), s1 = min(steps, 2 * part_start(pairs, part + 1, parts));

    // rows and columns past the end re-read the last one; their results are not stored
    const T *xp[MT], *xl[MT], *wp[NT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const size_t o = (size_t)min(16 * m + (lane & 15), a.R - 1) * a.ldx + 4 * g;
        xp[m] = (const T *)a.x + o;
        xl[m] = (const T *)a.x_lo + o;  // bf16 only
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) wp[j] = weight_row<T, EPI>(a, min(c0 + (lane & 15), a.N - 1), j) + 4 * g;
    f32x4 acc[MT][NT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto mma = [&](const f32x4(&xs)[MT], const f32x4(&ws)[NT]) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[m][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[m][c], ws[j][c], acc[m][j], 0, 0, 0);
    };
    if (s0 < s1) {
        // the ring's loads are unconditional (steps past the slice re-read its
        // last one) and the scheduling barriers keep a slot's refill behind
        // its products, so that the other slots' loads stay in flight; with
        // predicated loads every step waited for all of them
        f32x4 xv[D][MT], wv[D][NT];
        auto load = [&](int b, int s) {
            const size_t k = 16 * (size_t)min(s, s1 - 1);
#pragma unroll
            for (int j = 0; j < NT; ++j) wv[b][j] = load4<VEC>(wp[j] + k);
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                xv[b][m] = load4<VEC>(xp[m] + k);
                if constexpr (sizeof(T) == 2) xv[b][m] += load4<VEC>(xl[m] + k);
            }
        };
#pragma unroll
        for (int b = 0; b < D; ++b) load(b, s0 + b);
        int s = s0;
        for (; s + D <= s1; s += D) {
#pragma unroll
            for (int b = 0; b < D; ++b) {
                mma(xv[b], wv[b]);
                __builtin_amdgcn_sched_barrier(0);
                load(b, s + b + D);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int b = 0; b < D; ++b)
            if (s + b < s1) mma(xv[b], wv[b]);
    }
    if ((a.K & 15) && part == parts - 1) {  // the last, shorter step
        const int k = 16 * steps, left = a.K - k - 4 * g;
        f32x4 xv[MT], wv[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) wv[j] = load_tail(wp[j] + k, left);
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            xv[m] = load_tail(xp[m] + k, left);
            if constexpr (sizeof(T) == 2) xv[m] += load_tail(xl[m] + k, left);
        }
        mma(xv, wv);
    }

    if (kw > 0) {
        float *q = red + ((kw - 1) * MT * NT * 64 + lane) * 4;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int j = 0; j < NT; ++j) *reinterpret_cast<f32x4 *>(q + (m * NT + j) * 256) = acc[m][j];
    }
    __syncthreads();
    if (kw > 0) return;
#pragma unroll
    for (int u = 0; u < KW - 1; ++u) {
        const float *q = red + (u * MT * NT * 64 + lane) * 4;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[m][j] += *reinterpret_cast<const f32x4 *>(q + (m * NT + j) * 256);
    }
#pragma unroll
    for (int m = 0; m < MT; ++m)
        store_tile<T, EPI>(a, 16 * m + 4 * g, c0 + (lane & 15), acc[m][0], acc[m][NT - 1]);
}

// WT x WT tiles of 16 x 16 per wavefront; block tile 32 WT x 32 WT (SwiGLU:
// 16 WT features, each wavefront's first WT / 2 column tiles gate, then up).
template <typename T, int EPI, int WT, bool VEC>
__global__ __launch_bounds__(256, 2) void linear_generic_tiled_kernel(LinearArgs a) {
    constexpr int B = 32 * WT, KB = 32, LD = KB + 4;
    constexpr int CH = B * KB / 4 / 256;                     // float4 chunks per thread and operand
    constexpr int CT = EPI == EPI_SWIGLU ? WT / 2 : WT;      // output column tiles of a wavefront
    __shared__ __attribute__((aligned(16))) float lds[2][2 * B * LD];  // [stage][X rows, then W rows]
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w >> 1, wn = w & 1;
    const int r0 = blockIdx.y * B, c0 = blockIdx.x * 32 * CT;
    // this block's quarters [p0, pend) of `parts`
    const int steps = (a.K + KB - 1) / KB, parts = 4 * (EPI == EPI_STORE ? max(1, a.kslices) : 1);
    const int p0 = parts / gridDim.z * blockIdx.z, pend = p0 + parts / gridDim.z;
    const int send = part_start(steps, pend, parts);

    // staging: chunk i of this thread is row (tid + 256 i) / 8, k 4 (tid % 8) .. +3
    size_t xo[CH];
    const T *wp[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int v = (tid + 256 * i) >> 3;
        xo[i] = (size_t)min(r0 + v, a.R - 1) * a.ldx;
        // W row v of the tile: wavefront column v / (16 WT), tile and column within it
        const int t = (v >> 4) % WT;
        const int n = c0 + (v / (16 * WT)) * 16 * CT + (t % CT) * 16 + (v & 15);
        wp[i] = weight_row<T, EPI>(a, min(n, a.N - 1), t / CT);
    }
    f32x4 xr[CH], wr[CH];
    const int kt = 4 * (tid & 7);
    auto load = [&](const T *p, int k) {  // zeros past K
        if (k + 4 <= a.K) return load4<VEC>(p + k);
        return load_tail(p + min(k, a.K), a.K - k);
    };
    auto fetch = [&](int s) {
        const int k = KB * s + kt;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            xr[i] = load((const T *)a.x + xo[i], k);
            if constexpr (sizeof(T) == 2) xr[i] += load((const T *)a.x_lo + xo[i], k);
            wr[i] = load(wp[i], k);
        }
    };
    // the running quarter, slice and output; the larger tile keeps its output in
    // memory between slices (a third set of sums in registers would leave one
    // block per unit)
    constexpr bool TOT = EPI == EPI_STORE && WT == 2;
    f32x4 acc[WT][WT], sum[WT][WT], tot[WT][WT];
#pragma unroll
    for (int m = 0; m < WT; ++m)
#pragma unroll
        for (int j = 0; j < WT; ++j) acc[m][j] = sum[m][j] = tot[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    int s = part_start(steps, p0, parts);
    if (s < send) fetch(s);
    for (int p = p0; p < pend; ++p) {
        for (const int e = part_start(steps, p + 1, parts); s < e; ++s) {
            float *st = lds[s & 1];
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const int o = ((tid + 256 * i) >> 3) * LD + kt;
                *reinterpret_cast<f32x4 *>(st + o) = xr[i];
                *reinterpret_cast<f32x4 *>(st + B * LD + o) = wr[i];
            }
            // one barrier per step: a stage is written again two steps later, when
            // every wavefront has passed the barrier after its last read
            __syncthreads();
            if (s + 1 < send) fetch(s + 1);
            const float *xs = st + (16 * WT * wm + (lane & 15)) * LD + 4 * g;
            const float *ws = st + (B + 16 * WT * wn + (lane & 15)) * LD + 4 * g;
#pragma unroll
            for (int q = 0; q < KB / 16; ++q) {
                if (WT == 4) __builtin_amdgcn_sched_barrier(0);  // registers: one half-step's fragments at a time
                f32x4 xv[WT], wv[WT];
#pragma unroll
                for (int m = 0; m < WT; ++m) {
                    xv[m] = *reinterpret_cast<const f32x4 *>(xs + 16 * m * LD + 16 * q);
                    wv[m] = *reinterpret_cast<const f32x4 *>(ws + 16 * m * LD + 16 * q);
                }
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int m = 0; m < WT; ++m)
#pragma unroll
                        for (int j = 0; j < WT; ++j)
                            acc[m][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[m][c], wv[j][c], acc[m][j], 0, 0, 0);
            }
        }
        const bool end = (p & 3) == 3;  // of a slice
#pragma unroll
        for (int m = 0; m < WT; ++m)
#pragma unroll
            for (int j = 0; j < WT; ++j) {
                sum[m][j] += acc[m][j];
                acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (TOT && end) {
                    tot[m][j] += sum[m][j];
                    sum[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
        if (TOT ? p + 1 < pend : !end) continue;
#pragma unroll
        for (int m = 0; m < WT; ++m)
#pragma unroll
            for (int j = 0; j < CT; ++j) {
                store_tile<T, EPI>(a, r0 + 16 * (WT * wm + m) + 4 * g, c0 + 16 * (CT * wn + j) + (lane & 15),
                                   TOT ? tot[m][j] : sum[m][j], sum[m][(j + CT) % WT], !TOT && p > p0 + 3);
                if (EPI == EPI_STORE) sum[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
    }
}

// Output tiles of a tiled launch: 128 x 128 when there are two for every
// compute unit, else 64 x 64.  fp32 prefills of one layer, with the line at
// 256, 512 and 1024 tiles: d_model 2048, 2500 tokens 3524, 3130, 3133 us;
// d_model 4096, 2000 tokens 7845, 7849, 8170 us.
int generic_tile(int R, int vcols) {
    return (long long)((R + 127) / 128) * ((vcols + 127) / 128) >= 512 ? 4 : 2;
}

template <typename T, int EPI, bool VEC>
hipError_t launch_vec(const LinearArgs &a, hipStream_t s) {
    // a row block of up to 64 rows runs a block per slice, a tile one or all
    const int slices = EPI == EPI_STORE ? std::max(1, (int)a.kslices) : 1;
    const int z = EPI == EPI_STORE ? std::max(1, (int)a.split) : 1;
    if (z != slices && (z != 1 || a.R <= 64)) return hipErrorInvalidValue;
    const int vcols = EPI == EPI_SWIGLU ? 2 * a.N : a.N;
    if (a.R <= 64) {
        const dim3 grid((a.N + 15) / 16, 1, z);
        switch ((a.R + 15) / 16) {
            case 1: kvr_launch((linear_generic_kernel<T, EPI, 1, VEC>), grid, dim3(256), 0, s, a); break;
            case 2: kvr_launch((linear_generic_kernel<T, EPI, 2, VEC>), grid, dim3(256), 0, s, a); break;
            case 3: kvr_launch((linear_generic_kernel<T, EPI, 3, VEC>), grid, dim3(256), 0, s, a); break;
            default: kvr_launch((linear_generic_kernel<T, EPI, 4, VEC>), grid, dim3(256), 0, s, a);
        }
    } else {
        const int b = 32 * generic_tile(a.R, vcols);
        const dim3 grid((vcols + b - 1) / b, (a.R + b - 1) / b, z);
        if (b == 128) kvr_launch((linear_generic_tiled_kernel<T, EPI, 4, VEC>), grid, dim3(256), 0, s, a);
        else kvr_launch((linear_generic_tiled_kernel<T, EPI, 2, VEC>), grid, dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

template <typename T, int EPI>
hipError_t launch_epi(const LinearArgs &a, hipStream_t s) {
    return a.K % 4 == 0 && a.ldx % 4 == 0 ? launch_vec<T, EPI, true>(a, s) : launch_vec<T, EPI, false>(a, s);
}

}  // namespace

// K slices of the sum of a STORE launch, whatever its rows: up to two blocks
// per compute unit for a row block of 64, and slices of 256 k, or of 128 while
// those are no more than four (tiny fp32 decoder, 600-token prefill: 136 us a
// call against 152 with slices of 256 only, which leave a 256-wide projection
// to 40 blocks; its 40-row repair takes 101-104 us either way).  At most eight:
// an 8192-wide projection to 1024 columns in a layer of 300 rows, 265 us with
// four, 246 with eight, 246 with sixteen; 40 rows 96, 98 and 98 us.
int generic_slices(int N, int K) {
    return std::max(1, std::min({512 / ((N + 15) / 16), std::max(std::min(K / 128, 4), K / 256), 8}));
}

// Partial tiles of a STORE launch (a.split): a block per slice up to 64 rows,
// and for more while that leaves at most two blocks per compute unit and the
// partial tiles fit; else a block adds up every slice itself.
int generic_split(int R, int N, int slices, size_t part_floats) {
    if (R <= 64) return slices;
    const int b = 32 * generic_tile(R, N);
    const long long blocks = (long long)((R + b - 1) / b) * ((N + b - 1) / b);
    return blocks * 2 <= 512 && (size_t)slices * R * N <= part_floats ? slices : 1;
}

hipError_t launch_linear_generic(bool bf16, int epi, const LinearArgs &a, hipStream_t s) {
    if (a.R <= 0) return hipSuccess;
    if ((epi != EPI_STORE && epi != EPI_SWIGLU) || (bf16 && !a.x_lo)) return hipErrorInvalidValue;
    if (bf16) return epi == EPI_STORE ? launch_epi<bf16_t, EPI_STORE>(a, s) : launch_epi<bf16_t, EPI_SWIGLU>(a, s);
    return epi == EPI_STORE ? launch_epi<float, EPI_STORE>(a, s) : launch_epi<float, EPI_SWIGLU>(a, s);
}

}  // namespace kvr
