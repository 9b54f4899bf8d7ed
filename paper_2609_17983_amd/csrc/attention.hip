// Attention of bf16 models with 128-wide heads (attention_mfma.h), the combine of
// split items, and the dispatch over head widths.
#include "attention_mfma.h"

namespace kvr {

namespace {

constexpr int COMBINE_NP = 16;  // partials per row loaded in one round by the combine

// One wavefront per (combine item, query head of the group, 256 / HDP rows): a
// lane takes four consecutive dimensions of one row (HDP is the partial rows'
// width: head_dim, or the width the generic kernel pads it to).  The split
// partials of the row are merged with log-sum-exp weights (exp2 domain), the
// parts summed in ascending order.  With at most NP parts every partial of
// the row is loaded in one round (clamped indexes, so the loads are
// unconditional and all in flight together); longer lists take batches of NP.
// `lse` as in the attention kernel.
template <typename T, int HDP, int NP>
__global__ __launch_bounds__(64) void attention_combine_kernel(const CombineItem *items, const float *part, int Hq,
                                                               int Hkv, int hd, int MT, T *O, T *O_lo, int o_perm,
                                                               float *lse) {
    constexpr int LPR = HDP / 4, PART_ROW = HDP + 4;  // lanes per row; floats per partial row
    const CombineItem it = items[blockIdx.x];
    const int t = blockIdx.y;
    const int lane = threadIdx.x;
    const int i = (64 / LPR) * blockIdx.z + lane / LPR;
    if (i >= it.nrows) return;
    const int G = Hq / Hkv;
    const int rows_item = 16 * MT;
    const int j = it.kvh * G + t;
    const int d = 4 * (lane % LPR);
    const size_t qstride = (size_t)G * rows_item * PART_ROW;
    const float *base = part + ((size_t)(it.part0 * G + t) * rows_item + i) * PART_ROW;
    const int np = it.nparts;
    float M = -INFINITY, L = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int q0 = 0; q0 < np; q0 += NP) {
        float mm[NP], ll[NP];
        f32x4 oo[NP];
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const float *p = base + (size_t)min(q0 + u, np - 1) * qstride;
            mm[u] = p[HDP];
            ll[u] = p[HDP + 1];
            oo[u] = *reinterpret_cast<const f32x4 *>(p + d);
        }
        float Mb = M;
#pragma unroll
        for (int u = 0; u < NP; ++u) Mb = fmaxf(Mb, mm[u]);  // clamped duplicates do not change the max
        const float r = M == -INFINITY ? 0.f : exp2f(M - Mb);  // rescale what earlier batches summed
        acc *= r;
        L *= r;
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const float wq = (q0 + u >= np || mm[u] == -INFINITY) ? 0.f : exp2f(mm[u] - Mb);
            acc += oo[u] * wq;
            L += ll[u] * wq;
        }
        M = Mb;
    }
    const int r = it.row0 + i, c = j * hd + d;
    if (lse && d == 0) lse[(size_t)r * Hq + j] = M + log2f(L);
    const f32x4 y = acc / L;
    store_attn4(O, O_lo, r, c, min(4, hd - d), Hq * hd, o_perm, y);
}

}  // namespace

int attention_max_row_tiles(int Hq, int Hkv) {
    const int G = Hq / Hkv;
    return G >= 16 ? 1 : std::min(4, std::max(1, 16 / G));
}

bool attention_mfma_ok(bool bf16, int Hq, int Hkv, int hd) {
    return bf16 && (hd == 64 || hd == 128) && Hq / Hkv <= 16;
}

hipError_t launch_attention_mfma(const bf16_t *Q, const bf16_t *Q_lo, const RowInfo *rows,
                                 const AttnItem *items, int n_items, int MT, int layer, int Hq, int Hkv, int hd,
                                 float *part, bf16_t *O, bf16_t *O_lo, bool o_perm, float *lse, hipStream_t s) {
    if (n_items <= 0) return hipSuccess;
    if (!Q_lo || !O_lo || MT < 1 || MT > attention_max_row_tiles(Hq, Hkv) || !attention_mfma_ok(true, Hq, Hkv, hd))
        return hipErrorInvalidValue;
    return hd == 128 ? launch_mfma_hd<128>(Q, Q_lo, rows, items, n_items, MT, layer, Hq, Hkv, part, O, O_lo, o_perm, lse, s)
                     : launch_attention_mfma64(Q, Q_lo, rows, items, n_items, MT, layer, Hq, Hkv, part, O, O_lo, o_perm, lse, s);
}

template <typename T>
static hipError_t launch_combine(const CombineItem *items, int n_items, int MT, const float *part, int Hq, int Hkv,
                                 int hd, T *O, T *O_lo, bool o_perm, float *lse, hipStream_t s) {
    if (hd > 64)
        kvr_launch((attention_combine_kernel<T, 128, COMBINE_NP>), dim3(n_items, Hq / Hkv, 8 * MT), dim3(64), 0, s, items,
                   part, Hq, Hkv, hd, MT, O, O_lo, (int)o_perm, lse);
    else
        kvr_launch((attention_combine_kernel<T, 64, COMBINE_NP>), dim3(n_items, Hq / Hkv, 4 * MT), dim3(64), 0, s, items,
                   part, Hq, Hkv, hd, MT, O, O_lo, (int)o_perm, lse);
    return hipGetLastError();
}

hipError_t launch_attention_combine(bool bf16, const CombineItem *items, int n_items, int MT, const float *part, int Hq,
                                    int Hkv, int hd, void *O, void *O_lo, bool o_perm, float *lse, hipStream_t s) {
    if (n_items <= 0) return hipSuccess;
    if (MT < 1 || MT > attention_max_row_tiles(Hq, Hkv) || hd > 128) return hipErrorInvalidValue;
    if (bf16) return launch_combine(items, n_items, MT, part, Hq, Hkv, hd, (bf16_t *)O, (bf16_t *)O_lo, o_perm, lse, s);
    return launch_combine(items, n_items, MT, part, Hq, Hkv, hd, (float *)O, (float *)nullptr, o_perm, lse, s);
}

}  // namespace kvr
