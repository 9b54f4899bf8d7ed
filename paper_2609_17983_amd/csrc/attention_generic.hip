// Causal grouped-query attention of a set of rows over a KV cache for fp32
// models and for the bf16 shapes the bf16 MFMA kernel does not take: any
// head_dim up to 128, any number of query heads per kv head.
//
// The work items, partials and combine are the bf16 MFMA kernel's (an item is
// a document's rows, one kv head and a key range [k0, k1)).  Products run on
// v_mfma_f32_16x16x4_f32: fp32 operands with fp32 accumulation, so the fp32
// path keeps its precision and a bf16 pair (hi + lo) is summed exactly on
// load.  Scores are computed transposed, S^T = K Q^T, so a lane owns one query
// row (row lane%16, keys 4*(lane/16) + e of a 16-key tile), and the
// probabilities go from the accumulator straight into the B operand of
// O^T += V^T P^T: k-slot g of that instruction's step e is key 4g + e on both
// sides.  The score's k-slots are permuted alike (step 4q + c, slot g <->
// dimension 16q + 4g + c), so that a lane reads its key and query dimensions
// as one float4 per four steps.
//
// A block is four wavefronts over one 64-key tile in LDS (rows padded by four
// floats: a key fragment's 16 rows and a value fragment's four key groups then
// fall on distinct banks); the next tile is fetched into registers meanwhile.
// A wavefront works one (head, 16-row tile) pair; with fewer than four pairs
// per item the wavefronts split into KG key groups that take alternate 16-key
// tiles and merge their softmax states in LDS at the end.
//
// A row's result depends on the key ranges of its item, which follow from the
// rows of the whole pass, and on nothing else of the rows beside it.  It
// depends on no slot behind its position, whatever that slot holds: in
// the tiles that have a mask, values that are not finite are staged as zeros
// (a masked key's probability is zero, its product with them would not be) and
// added afterwards for the rows that see them.
//
// What bounds it: the fp32 matrix rate on long contexts (32 instructions of
// 32 cycles per 16 keys x 16 rows at head_dim 64), latency on short ones.  The
// blocks that share a compute unit hide each other's two barriers per key
// tile, so the registers are bounded for the att_generic_blocks that the
// planner counts on (146 at 64, 235 at 128; without the bound 174 and 270,
// which left two and one): 2500-token fp32 prefill, 32 heads of 128, 985 ->
// 714 us a layer, 1501 tokens, 4 heads of 64, 32 -> 26 us.  Four blocks at 64
// would spill.
// Tiny fp32 decoder (4 heads of 64), per layer against the kernel it replaced
// (one wavefront per row and head, one key per step): 1501-token prefill
// 1243 -> 36 us, 40-row repair at position 128 96 -> 8 us, plus a combine of
// 5 us each.
#include <math.h>

#include <algorithm>

#include "common.h"

namespace kvr {

namespace {

constexpr int KT = ATT_KT;
constexpr int WAVES = 4;
constexpr float RESCALE_SLACK = 8.0f;  // log2 headroom before the running max is raised

// Max / sum over the four lanes l, l^16, l^32, l^48 that hold one query row.
__device__ __forceinline__ float xmax4(float v) {
    v = fmaxf(v, __shfl_xor(v, 16));
    return fmaxf(v, __shfl_xor(v, 32));
}
__device__ __forceinline__ float xsum4(float v) {
    v += __shfl_xor(v, 16);
    return v + __shfl_xor(v, 32);
}

// Dimensions d .. d+3 of a row of hd values (zero past hd); vec: hd is a
// multiple of four, so the four are all inside or all outside and the row is
// aligned for one load.
__device__ __forceinline__ f32x4 load_dims(const float *p, int d, int hd, bool vec) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (vec) {
        if (d < hd) v = *reinterpret_cast<const f32x4 *>(p + d);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (d + e < hd) v[e] = p[d + e];
    }
    return v;
}
__device__ __forceinline__ f32x4 load_dims(const bf16_t *p, int d, int hd, bool vec) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (vec) {
        if (d < hd) {
            const uint2 u = *reinterpret_cast<const uint2 *>(p + d);
            v = f32x4{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                      __uint_as_float(u.y & 0xffff0000u)};
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (d + e < hd) v[e] = bf16_to_f32(p[d + e]);
    }
    return v;
}

// HDP: head_dim padded to 64 or 128; KG: key groups.
template <typename T, int HDP, int KG>
__global__ __launch_bounds__(64 * WAVES, att_generic_blocks(HDP)) void attention_generic_kernel(const T *Q, const T *Q_lo,
                                                                       const RowInfo *rows,
                                                                       const AttnItem *items, int layer, int Hq,
                                                                       int Hkv, int hd, int MT, float *part, T *O,
                                                                       T *O_lo, int o_perm, float *lse) {
    constexpr int DQ = HDP / 16;              // 16-wide dimension tiles
    constexpr int LD = HDP + 4;               // LDS row stride (floats)
    constexpr int CPR = HDP / 4;              // float4 chunks per row
    constexpr int NLD = KT * CPR / (64 * WAVES);
    constexpr int NSUB = KT / 16 / KG;        // 16-key tiles of an LDS tile each wavefront takes
    constexpr int PART_ROW = HDP + 4;
    __shared__ __attribute__((aligned(16))) float kv_lds[2 * KT * LD];
    float *Ks = kv_lds, *Vs = kv_lds + KT * LD;
    __shared__ int bad_tile;  // first key of the last staged tile that holds a value that is not finite

    const AttnItem it = items[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = Hq / Hkv, qd = Hq * hd;
    const int MTi = (it.nrows + 15) >> 4;
    const int kg = w % KG;
    const int p = blockIdx.y * (WAVES / KG) + w / KG;  // this wavefront's pair: head p / MTi, row tile p % MTi
    const bool pvalid = p < G * MTi;
    const int pt = pvalid ? p / MTi : 0, pm = pvalid ? p % MTi : 0;
    const int ri = pm * 16 + (lane & 15);              // this lane's query row within the item
    const int pos = (pvalid && ri < it.nrows) ? rows[it.row0 + ri].pos : -1;
    const int j = it.kvh * G + pt;
    const int minpos = rows[it.row0].pos;              // rows ascend: every row sees all keys <= minpos
    const bool vec = (hd & 3) == 0;
    const size_t head_stride = (size_t)it.n_cap * hd;
    const T *Kg = (const T *)it.cache + (((size_t)layer * 2 + 0) * Hkv + it.kvh) * head_stride;
    const T *Vg = (const T *)it.cache + (((size_t)layer * 2 + 1) * Hkv + it.kvh) * head_stride;

    f32x4 qf[DQ];
    {
        const size_t qo = (size_t)(it.row0 + min(ri, it.nrows - 1)) * qd + (size_t)j * hd;
        const bool qvec = vec && (qd & 3) == 0;
#pragma unroll
        for (int q = 0; q < DQ; ++q) {
            qf[q] = load_dims(Q + qo, 16 * q + 4 * g, hd, qvec);
            if (Q_lo) qf[q] += load_dims(Q_lo + qo, 16 * q + 4 * g, hd, qvec);
        }
    }
    f32x4 oacc[DQ];
#pragma unroll
    for (int q = 0; q < DQ; ++q) oacc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;  // l: this lane's share of the row's sum
    const float sc = 1.4426950408889634f / sqrtf((float)hd);

    f32x4 kreg[NLD], vreg[NLD];
    auto fetch = [&](int kb) {
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int c = tid + 64 * WAVES * i;
            const size_t o = (size_t)min(kb + c / CPR, it.k1 - 1) * hd;  // keys past the range re-read its last one
            kreg[i] = load_dims(Kg + o, 4 * (c % CPR), hd, vec);
            vreg[i] = load_dims(Vg + o, 4 * (c % CPR), hd, vec);
        }
    };
    fetch(it.k0);
    if (tid == 0) bad_tile = -1;
    for (int kb = it.k0; kb < it.k1; kb += KT) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int c = tid + 64 * WAVES * i;
            *reinterpret_cast<f32x4 *>(&Ks[(c / CPR) * LD + 4 * (c % CPR)]) = kreg[i];
            *reinterpret_cast<f32x4 *>(&Vs[(c / CPR) * LD + 4 * (c % CPR)]) = vreg[i];
        }
        const bool masked = kb + KT > it.k1 || kb + KT - 1 > minpos;
        if (masked) {
            // A masked key's probability is zero, and so is its product unless
            // its value is not finite: those are left out here and added below
            // for the rows that see them.
            float t = 0.f;
#pragma unroll
            for (int i = 0; i < NLD; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) t = fmaf(vreg[i][e], 0.f, t);
            if (t != 0.f) {
                bad_tile = kb;
#pragma unroll
                for (int i = 0; i < NLD; ++i) {
                    const int c = tid + 64 * WAVES * i;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (!isfinite(vreg[i][e])) Vs[(c / CPR) * LD + 4 * (c % CPR) + e] = 0.f;
                }
            }
        }
        __syncthreads();
        if (kb + KT < it.k1) fetch(kb + KT);

        f32x4 s[NSUB];
#pragma unroll
        for (int u = 0; u < NSUB; ++u) {
            const int t = kg + KG * u;  // 16-key tile of the LDS tile
            f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < DQ; ++q) {
                const f32x4 kf = *reinterpret_cast<const f32x4 *>(&Ks[(16 * t + (lane & 15)) * LD + 16 * q + 4 * g]);
                s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[0], qf[q][0], s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[1], qf[q][1], s1, 0, 0, 0);
                s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[2], qf[q][2], s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[3], qf[q][3], s1, 0, 0, 0);
            }
            s[u] = s0 + s1;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int u = 0; u < NSUB; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int key = kb + 16 * (kg + KG * u) + 4 * g + e;
                s[u][e] = (key < it.k1 && key <= pos) ? s[u][e] * sc : -INFINITY;
                mx = fmaxf(mx, s[u][e]);
            }
        mx = xmax4(mx);
        if (__any(mx > m + RESCALE_SLACK)) {
            const float mnew = mx > m + RESCALE_SLACK ? mx : m;  // the other rows of the tile keep theirs
            const float corr = m == -INFINITY ? 0.f : exp2f(m - mnew);
            m = mnew;
            l *= corr;
#pragma unroll
            for (int q = 0; q < DQ; ++q) oacc[q] *= corr;
        }
        const float muse = m == -INFINITY ? 0.f : m;
#pragma unroll
        for (int u = 0; u < NSUB; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float pr = exp2f(s[u][e] - muse);
                l += pr;
                const float *vr = &Vs[(16 * (kg + KG * u) + 4 * g + e) * LD + (lane & 15)];
#pragma unroll
                for (int q = 0; q < DQ; ++q)
                    oacc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[16 * q], pr, oacc[q], 0, 0, 0);
            }
        if (masked && bad_tile == kb) {
            const int nk = min(KT, it.k1 - kb);
#pragma unroll 1
            for (int k = 0; k < nk; ++k) {
                if ((k >> 4) % KG != kg) continue;
#pragma unroll
                for (int q = 0; q < DQ; ++q) {
                    const f32x4 v = load_dims(Vg + (size_t)(kb + k) * hd, 16 * q + 4 * g, hd, vec);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (!isfinite(v[e]) && kb + k <= pos) oacc[q][e] += v[e];
                }
            }
        }
    }
    l = xsum4(l);

    if constexpr (KG > 1) {
        // key groups 1 .. KG-1 hand their states to the group-0 wavefront of
        // their pair, which merges them in group order
        constexpr int ST = HDP / 4 + 2;
        static_assert(WAVES * 64 * ST <= 2 * KT * LD, "merge area");
        __syncthreads();  // every wavefront is done with the K/V tiles
        if (kg > 0) {
            float *q = kv_lds + (w * 64 + lane) * ST;
#pragma unroll
            for (int d = 0; d < DQ; ++d)
#pragma unroll
                for (int e = 0; e < 4; ++e) q[4 * d + e] = oacc[d][e];
            q[ST - 2] = m;
            q[ST - 1] = l;
        }
        __syncthreads();
        if (kg > 0) return;
#pragma unroll
        for (int u = 1; u < KG; ++u) {
            const float *q = kv_lds + ((w + u) * 64 + lane) * ST;
            const float m1 = q[ST - 2], l1 = q[ST - 1];
            const float M = fmaxf(m, m1);
            const float a0 = m == -INFINITY ? 0.f : exp2f(m - M), a1 = m1 == -INFINITY ? 0.f : exp2f(m1 - M);
            m = M;
            l = l * a0 + l1 * a1;
#pragma unroll
            for (int d = 0; d < DQ; ++d)
#pragma unroll
                for (int e = 0; e < 4; ++e) oacc[d][e] = oacc[d][e] * a0 + q[4 * d + e] * a1;
        }
    }
    if (!pvalid || ri >= it.nrows) return;
    if (it.part < 0) {
        const float inv = 1.0f / l;
        const int r = it.row0 + ri;
#pragma unroll
        for (int q = 0; q < DQ; ++q) {
            const int d = 16 * q + 4 * g;
            if (d < hd) store_attn4(O, O_lo, r, j * hd + d, min(4, hd - d), qd, o_perm, oacc[q] * inv);
        }
        if (lse && g == 0) lse[(size_t)r * Hq + j] = m + log2f(l);
    } else {
        float *o = part + ((size_t)(it.part * G + pt) * 16 * MT + ri) * PART_ROW;
#pragma unroll
        for (int q = 0; q < DQ; ++q) *reinterpret_cast<f32x4 *>(o + 16 * q + 4 * g) = oacc[q];
        if (g == 0) {
            o[HDP] = m;
            o[HDP + 1] = l;
        }
    }
}

template <typename T, int HDP>
hipError_t launch_hdp(const T *Q, const T *Q_lo, const RowInfo *rows, const AttnItem *items, int n_items, int MT,
                      int layer, int Hq, int Hkv, int hd, float *part, T *O, T *O_lo, bool o_perm, float *lse,
                      hipStream_t s) {
    const int npairs = (Hq / Hkv) * MT;
    const int kg = npairs >= 4 ? 1 : npairs >= 2 ? 2 : 4;
    const dim3 grid(n_items, (npairs * kg + WAVES - 1) / WAVES), block(64 * WAVES);
    if (kg == 1)
        kvr_launch((attention_generic_kernel<T, HDP, 1>), grid, block, 0, s, Q, Q_lo, rows, items, layer, Hq, Hkv, hd, MT,
                   part, O, O_lo, (int)o_perm, lse);
    else if (kg == 2)
        kvr_launch((attention_generic_kernel<T, HDP, 2>), grid, block, 0, s, Q, Q_lo, rows, items, layer, Hq, Hkv, hd, MT,
                   part, O, O_lo, (int)o_perm, lse);
    else
        kvr_launch((attention_generic_kernel<T, HDP, 4>), grid, block, 0, s, Q, Q_lo, rows, items, layer, Hq, Hkv, hd, MT,
                   part, O, O_lo, (int)o_perm, lse);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attention_generic(bool bf16, const void *Q, const void *Q_lo, const RowInfo *rows,
                                    const AttnItem *items, int n_items, int MT, int layer, int Hq, int Hkv, int hd,
                                    float *part, void *O, void *O_lo, bool o_perm, float *lse, hipStream_t s) {
    if (n_items <= 0) return hipSuccess;
    if (MT < 1 || MT > attention_max_row_tiles(Hq, Hkv) || hd < 1 || hd > 128 || (bf16 && (!Q_lo || !O_lo)))
        return hipErrorInvalidValue;
    if (bf16) {
        if (hd > 64)
            return launch_hdp<bf16_t, 128>((const bf16_t *)Q, (const bf16_t *)Q_lo, rows, items, n_items, MT, layer, Hq,
                                           Hkv, hd, part, (bf16_t *)O, (bf16_t *)O_lo, o_perm, lse, s);
        return launch_hdp<bf16_t, 64>((const bf16_t *)Q, (const bf16_t *)Q_lo, rows, items, n_items, MT, layer, Hq, Hkv,
                                      hd, part, (bf16_t *)O, (bf16_t *)O_lo, o_perm, lse, s);
    }
    if (hd > 64)
        return launch_hdp<float, 128>((const float *)Q, nullptr, rows, items, n_items, MT, layer, Hq, Hkv, hd, part,
                                      (float *)O, nullptr, o_perm, lse, s);
    return launch_hdp<float, 64>((const float *)Q, nullptr, rows, items, n_items, MT, layer, Hq, Hkv, hd, part,
                                 (float *)O, nullptr, o_perm, lse, s);
}

}  // namespace kvr
