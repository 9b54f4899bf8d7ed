// Tiled bf16 MFMA linear layer for many rows (prefill, batched repair).
//
// Y[r][n] = sum_k X[r][k] * W[n][k].  Both operands arrive in MFMA operand
// order: the activations X (a compensated pair hi + lo, written so by their
// producers) and the packed weight W (pack.hip) are sequences of 1 KB
// fragments, one per 16-row tile and 32-wide k-step, that a wavefront loads
// with one 16-byte access per lane.  A block computes MT row tiles x 16 weight
// tiles (16 MT x 256 outputs, MT = 4 .. 8); each of its four wavefronts owns
// all the rows and four weight tiles (MT x 4 v_mfma_f32_16x16x32_bf16 tiles,
// two MFMAs per product for hi and lo).  A STORE launch may also cut K into
// `split` slices, each writing an fp32 partial tile that
// the consumer sums in a fixed order: the way a few hundred rows still fill
// the chip.
//
// Only the activations go through LDS.  A weight fragment is used by one
// wavefront, so it is loaded straight into registers, D k-steps ahead; the
// activation fragments all four wavefronts read are copied from memory into
// an LDS ring of D + 1 stages (global_load_lds_dwordx4: lane l's 16 bytes land
// at the destination + 16 l, so a fragment keeps its layout and no registers
// stage it).  Every iteration issues its stage's copies, multiplies, and
// refills the weight slot it used, in that order and always the same count
// (k-steps past the slice re-read its last one), so "the loads of the last
// D - 1 iterations may be in flight" is an exact wait that covers both (a
// slice of a single k-step issues fewer; its copies are still the oldest).  The
// barrier is a bare s_barrier: the compiler's workgroup fence would also wait
// for the loads still in flight.  Registers and LDS leave room for two blocks
// per compute unit, so that one block's MFMAs run while the other waits; a
// block alone (eight wavefronts, or 128 x 512 outputs in four) was slower.
//
// What bounds it: the chip's power under random operands (all-zero operands
// run 20-25 % faster at the same code), so bytes moved per product count: with
// the weights through LDS as well (four wavefronts of 64 x 128) every weight
// fragment was written to LDS once and read twice.  Same box, in turn, us
// against that kernel and its rule for the block shape (Q/K/V, output,
// gate/up, down): Llama-3-8B at 5000 rows 384, 279, 1850, 977 -> 367, 257,
// 1762, 926; at 3072 rows 272, 158, 1093, 524 -> 220, 159, 1038, 539 (the
// output and down projections without a K split now, so one partial tile less
// to write and read); Qwen2.5-7B at 528 rows 39, 32, 280, 139 (K splits 4, 5,
// 1, 5) -> 40, 33, 249, 129 (2, 2, 1, 3).
// Row tiles past the last one and weight tiles past the last one re-read the
// last tile; their results are not stored.
//
// Tile order.  Workgroups are handed to the eight XCDs in turn (workgroup b to
// XCD b % 8), and each XCD has its own L2.  The output tiles are therefore
// numbered in groups of row blocks (within a group: column block outer, row
// block inner), one K slice after the other, the numbering is cut into eight
// contiguous ranges that differ by at most one job, and XCD x runs range x in
// order, so the blocks that read one weight slab run at the
// same time on one XCD and share its L2.  Up to GROUP_ALL row blocks form one
// group (a repair of a few hundred rows: every weight slab is fetched from
// HBM about once; with groups of four, 528 rows fetched 3.6 times the
// gate/up weights); more (prefill, batches) are grouped by four.
#include <stdlib.h>

#include <algorithm>

#include "common.h"

namespace kvr {

namespace {

constexpr int NTW = 4;          // weight tiles per wavefront
constexpr int WT = 4 * NTW;     // weight tiles per block (256 output columns)
constexpr int FRAG = 512;       // bf16 elements of one 16 x 32 operand fragment
constexpr int D = 2;            // k-steps of loads in flight
constexpr int XCDS = 8;         // L2 domains the workgroups are dealt to in turn
constexpr int GROUP_M = 4;      // row blocks per group of the tile order (many row blocks)
constexpr int GROUP_ALL = 12;   // up to this many row blocks, one group holds them all
constexpr int MT_MIN = 4, MT_MAX = 8;

// Blocks of MT row tiles that share a compute unit (registers: 128 at MT 4,
// 168 at 5 and 6, 256 above; LDS 6 MT KB each).
constexpr int blocks_per_cu(int mt) { return mt <= 4 ? 4 : mt <= 6 ? 3 : 2; }

__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + __expf(-z)); }

// Block barrier that orders LDS accesses for the compiler without waiting for
// outstanding vector-memory loads.  The LDS wait is the builtin (not part of
// the asm) so that the compiler knows every earlier LDS read has completed.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); vmcnt and expcnt unconstrained
    asm volatile("s_barrier" ::: "memory");
}

// Wait until at most N of this wavefront's vector-memory loads are in flight
// (N below 16; expcnt and lgkmcnt left unconstrained).
template <int N>
__device__ __forceinline__ void wait_loads_upto() {
    static_assert(N >= 0 && N < 16, "vmcnt immediate");
    __builtin_amdgcn_s_waitcnt(0x70 | 0xF00 | N);
}

template <int EPI, int MT>
__global__ __launch_bounds__(256, blocks_per_cu(MT)) void linear_tiled_kernel(LinearArgs a) {
    constexpr int NX = 2 * MT;          // activation fragments per k-step: hi row tiles, then lo
    constexpr int FX = (NX + 3) / 4;    // fragments each wavefront copies per k-step
    constexpr int STAGE = NX * FRAG;
    static_assert(2 * (D + 1) * STAGE * 2 <= 160 * 1024, "LDS of two blocks");
    __shared__ __attribute__((aligned(16))) bf16_t lds[(D + 1) * STAGE];

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ksteps = a.K >> 5;   // k-steps of the whole row (operand strides)
    const int split = EPI == EPI_STORE ? max(1, a.split) : 1;
    const int ntiles = (a.N * (EPI == EPI_SWIGLU ? 2 : 1)) >> 4;
    const int rtiles = (a.R + 15) >> 4;
    // this workgroup's output tile (bm, bn) in the XCD-grouped order
    const int MB = (rtiles + MT - 1) / MT, NB = (ntiles + WT - 1) / WT;
    const int T = MB * NB, J = T * split;  // (K slice, tile) jobs, slice outer
    const int x = blockIdx.x % XCDS;
    const int job = (int)((long long)J * x / XCDS) + blockIdx.x / XCDS;
    if (job >= (int)((long long)J * (x + 1) / XCDS)) return;
    const int sp = job / T, tile = job - sp * T;
    const int k0 = ksteps * sp / split, nk = ksteps * (sp + 1) / split - k0;  // this job's k-steps [k0, k0 + nk)
    const int GM = MB <= a.group_all ? MB : GROUP_M;
    const int grp = tile / (GM * NB);
    const int gm = min(GM, MB - grp * GM);
    const int ti = tile - grp * GM * NB;
    const int bn = ti / gm, bm = grp * GM + ti % gm;

    // The arrays the lambdas capture have fixed sizes: local arrays whose size
    // depends on a template parameter made the host compiler drop the kernel's
    // launch stub.
    static_assert(FX <= 4 && MT <= 8, "array sizes");
    const bf16_t *xs[4];  // this wavefront's activation fragments (the last one repeated by those that have fewer)
    int xd[4];
#pragma unroll
    for (int i = 0; i < FX; ++i) {
        const int f = w + 4 * min(i, (NX - 1 - w) / 4);
        xd[i] = f * FRAG;
        const int t = min(bm * MT + (f < MT ? f : f - MT), rtiles - 1);
        xs[i] = (const bf16_t *)(f < MT ? a.x : a.x_lo) + ((size_t)t * ksteps + k0) * FRAG + lane * 8;
    }
    const bf16_t *wp[NTW];
    int ws[NTW];  // elements between a tile's k-steps
#pragma unroll
    for (int j = 0; j < NTW; ++j) {
        const int t = min(bn * WT + w * NTW + j, ntiles - 1);
        wp[j] = (const bf16_t *)a.wp + packed_tile_offset(t, ntiles, ksteps, a.grp, &ws[j]) + lane * 8;
        wp[j] += (size_t)k0 * ws[j];
    }
    // running pointers, advanced while a further k-step follows
    auto issue_x = [&](int slot, bool more) {
        bf16_t *st = lds + slot * STAGE;
#pragma unroll
        for (int i = 0; i < FX; ++i) {
            __builtin_amdgcn_global_load_lds(xs[i], st + xd[i], 16, 0, 0);
            xs[i] += more ? FRAG : 0;
        }
    };
    bf16x8 wv[D][NTW];
    auto load_w = [&](int b, bool more) {
#pragma unroll
        for (int j = 0; j < NTW; ++j) {
            wv[b][j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(wp[j]));
            wp[j] += more ? ws[j] : 0;
        }
    };
    f32x4 acc[8][NTW];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < NTW; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // stage 0's copies are the oldest loads: the first wait retires the oldest
    // FX + NTW, so the scheduler must not hoist weight loads in front of them
#pragma unroll
    for (int b = 0; b < D; ++b) {
        issue_x(b, b + 1 < nk);
        __builtin_amdgcn_sched_barrier(0);
        load_w(b, b + 1 < nk);
        __builtin_amdgcn_sched_barrier(0);
    }
    int rd = 0, wr = D;  // ring stages of k-step kk and of k-step kk + D
    auto step = [&](int b, int kk) {
        wait_loads_upto<(D - 1) * (FX + NTW)>();  // this wavefront's loads of k-step kk have landed
        lds_barrier();  // everyone's have; all reads of k-step kk - 1, whose stage is refilled now, are done
        issue_x(wr, kk + D + 1 < nk);
        wr = wr == D ? 0 : wr + 1;
        const bf16_t *st = lds + rd * STAGE + lane * 8;
        rd = rd == D ? 0 : rd + 1;
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 xh[2], xl[2];  // the next row tile's fragments are read during this one's MFMAs
        xh[0] = *reinterpret_cast<const bf16x8 *>(st);
        xl[0] = *reinterpret_cast<const bf16x8 *>(st + MT * FRAG);
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            if (m + 1 < MT) {
                xh[(m + 1) & 1] = *reinterpret_cast<const bf16x8 *>(st + (m + 1) * FRAG);
                xl[(m + 1) & 1] = *reinterpret_cast<const bf16x8 *>(st + (MT + m + 1) * FRAG);
            }
#pragma unroll
            for (int j = 0; j < NTW; ++j)
                acc[m][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh[m & 1], wv[b][j], acc[m][j], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < NTW; ++j)
                acc[m][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xl[m & 1], wv[b][j], acc[m][j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        load_w(b, kk + D + 1 < nk);
        __builtin_amdgcn_sched_barrier(0);
    };
    int kk = 0;
    for (; kk + D <= nk; kk += D) {
#pragma unroll
        for (int b = 0; b < D; ++b) step(b, kk + b);
    }
#pragma unroll
    for (int b = 0; b < D - 1; ++b)
        if (kk + b < nk) step(b, kk + b);

    // Epilogue through LDS.  The accumulators hold, per lane, one column and
    // four rows of each 16 x 16 tile, so stores straight from them write 2- or
    // 4-byte pieces scattered over rows (measured on the 5000-token prefill:
    // skipping every store of these kernels saved 8.5 of 126 ms).  Instead
    // each wavefront passes one row tile at a time through a region of its
    // own and copies it out in whole pieces: a SwiGLU output fragment (16 rows
    // x 32 features in operand order) as one contiguous 1 KB store of hi and
    // one of lo, fp32 partial rows in pieces of 256 bytes.  The 16-byte column
    // index is XORed with the row, so that the rows read by a fragment's
    // lanes fall on distinct banks.
    constexpr int SC = EPI == EPI_SWIGLU ? 32 : 64;  // staged columns
    static_assert(4 * 16 * SC * 4 <= (D + 1) * STAGE * 2, "epilogue staging fits in the LDS ring");
    wait_loads_upto<0>();  // the ring's last copies (k-steps past the slice) must not land on the staged rows
    __syncthreads();
    float *stg = reinterpret_cast<float *>(lds) + w * 16 * SC;
    auto sidx = [](int r, int c) { return r * SC + ((((c >> 2) ^ r) & (SC / 4 - 1)) << 2) + (c & 3); };
    const int lrow = 4 * (lane >> 4);  // accumulator layout: lane l holds tile column l%16, rows 4*(l/16)+e
    float *out = (float *)a.out + (size_t)sp * a.R * a.ldo;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int row0 = 16 * (bm * MT + m);
        if (row0 >= a.R) break;
        // the staged rows pass between lanes of one wavefront: its LDS
        // accesses complete in order, the fences keep the compiler from moving them
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (EPI == EPI_SWIGLU) {
            // gate/up interleaved: column j < 8 of weight tile t is the gate of
            // feature 8t+j, column j+8 its up (lane l+8 holds it); the output is
            // the down projection's operand, in operand order
#pragma unroll
            for (int j = 0; j < NTW; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float g = acc[m][j][e];
                    const float u = __shfl_xor(g, 8);
                    if ((lane & 8) == 0) stg[sidx(lrow + e, 8 * j + (lane & 7))] = silu_f(g) * u;
                }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const int lr = lane & 15, c = 8 * (lane >> 4);
            const int r = row0 + lr, f = 8 * (bn * WT + w * NTW) + c;  // the wavefront's features start a k-step
            const f32x4 v0 = *reinterpret_cast<const f32x4 *>(&stg[sidx(lr, c)]);
            const f32x4 v1 = *reinterpret_cast<const f32x4 *>(&stg[sidx(lr, c + 4)]);
            if (r >= a.R || f >= a.N) continue;
            const float y[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bf16_t h0 = f32_to_bf16(y[2 * q]), h1 = f32_to_bf16(y[2 * q + 1]);
                const bf16_t l0 = f32_to_bf16(y[2 * q] - bf16_to_f32(h0)), l1 = f32_to_bf16(y[2 * q + 1] - bf16_to_f32(h1));
                hi[q] = (uint32_t)h0 | ((uint32_t)h1 << 16);
                lo[q] = (uint32_t)l0 | ((uint32_t)l1 << 16);
            }
            const size_t off = perm_offset(r, f, a.N);
            *reinterpret_cast<u32x4 *>((bf16_t *)a.out + off) = u32x4{hi[0], hi[1], hi[2], hi[3]};
            *reinterpret_cast<u32x4 *>((bf16_t *)a.out_lo + off) = u32x4{lo[0], lo[1], lo[2], lo[3]};
        } else {
#pragma unroll
            for (int j = 0; j < NTW; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) stg[sidx(lrow + e, 16 * j + (lane & 15))] = acc[m][j][e];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const int c = 4 * (lane & 15);  // this lane's four columns
            const int t = bn * WT + w * NTW + c / 16;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int lr = 4 * q + (lane >> 4);
                const f32x4 v = *reinterpret_cast<const f32x4 *>(&stg[sidx(lr, c)]);
                if (row0 + lr < a.R && t < ntiles)
                    *reinterpret_cast<f32x4 *>(out + (size_t)(row0 + lr) * a.ldo + 16 * t + (c & 15)) = v;
            }
        }
    }
}

template <int MT>
void launch_mt(int epi, const LinearArgs &a, int jobs, hipStream_t s) {
    const dim3 grid((jobs + XCDS - 1) / XCDS * XCDS);
    if (epi == EPI_STORE) kvr_launch(linear_tiled_kernel<EPI_STORE, MT>, grid, dim3(256), 0, s, a);
    else kvr_launch(linear_tiled_kernel<EPI_SWIGLU, MT>, grid, dim3(256), 0, s, a);
}

int output_tiles(int R, int vrows, int mt) {
    return ((R + 15) / 16 + mt - 1) / mt * ((vrows / 16 + WT - 1) / WT);
}

}  // namespace

// Row tiles per block and K slices: the plan with the lowest estimated time
//   u K EFF[mt] mt (mean + most) / 2 / split + the partial tiles' traffic,
// where mean and most are the jobs per compute unit, u K is one row tile x 256
// columns x K at the rate a busy unit reaches (1.35 PFLOP/s for the chip) and
// a partial tile past the first is written and read back.  A last round that
// fills part of the units costs about half of what it would on paper (the
// chip is power bound and the units that have work clock higher), hence the
// average of the two.  EFF is the time per row tile against six of them:
// measured (Llama-3-8B gate/up at 5000 rows) 12.4, 12.3, 11.8, 12.8, 12.1 us
// per row tile and round for 4 .. 8, that is 1.05, 1.04, 1, 1.08, 1.03, and
// entered 0.01 to 0.02 lower, by which boxes differ; six leave room for three
// blocks per unit, seven and eight for two.  Measured against the former rule
// (256-, 128- or 64-row blocks by grid size; us, same box): batched repair
// (3072 rows) Q/K/V, six row tiles, one full round: 272 -> 220; Qwen2.5-7B down
// projection at 528 rows, six row tiles x split 3 instead of four x 5: 139 ->
// 129.
// KVR_TILED_RT (4 .. 8; larger values stand for 8) forces the row tiles.
TiledPlan plan_tiled(int R, int vrows, int K, bool split_ok, size_t p_floats) {
    static const double EFF[MT_MAX + 1] = {0, 0, 0, 0, 1.04, 1.03, 1.0, 1.06, 1.01};
    int lo = MT_MIN, hi = MT_MAX;
    if (const char *e = getenv("KVR_TILED_RT")) {
        const int v = std::min(atoi(e), MT_MAX);
        if (v >= MT_MIN) lo = hi = v;
    }
    const int ksteps = K / 32;
    const double unit = 16.0 * 256 * 4 * K / 5.3e6;            // us per row tile and column block
    const double part = (double)R * vrows * 4 * (1 / 4.8e6 + 1 / 3e6);  // us per further partial tile
    TiledPlan best{hi, 1};
    double cost = -1;
    for (int mt = hi; mt >= lo; --mt) {
        const int tiles = output_tiles(R, vrows, mt);
        for (int sp = 1; sp <= 16; ++sp) {
            if (sp > 1 && (!split_ok || ksteps / sp < 16 || (size_t)sp * R * vrows > p_floats)) break;
            const long long jobs = (long long)tiles * sp;
            const long long most = ((jobs + XCDS - 1) / XCDS + 31) / 32;  // on one of an XCD's 32 units
            const double t = unit * EFF[mt] * mt * (jobs / 256.0 + most) / 2 / sp + part * (sp - 1);
            if (cost < 0 || t < cost) {
                best = TiledPlan{mt, sp};
                cost = t;
            }
        }
    }
    return best;
}

hipError_t launch_linear_tiled(int epi, const LinearArgs &a, hipStream_t s) {
    if (a.R <= 0) return hipSuccess;
    if ((epi != EPI_STORE && epi != EPI_SWIGLU) || !a.x_lo || !a.wp || (epi == EPI_SWIGLU && !a.out_lo))
        return hipErrorInvalidValue;
    const int vrows = epi == EPI_SWIGLU ? 2 * a.N : a.N;
    if (a.K % 32 != 0 || a.K < 32 || vrows % 16 != 0 || (epi == EPI_SWIGLU && a.N % 32 != 0)) return hipErrorInvalidValue;
    if (a.rt < MT_MIN || a.rt > MT_MAX || (a.split > 1 && (epi != EPI_STORE || a.split > a.K / 32)))
        return hipErrorInvalidValue;
    const int jobs = output_tiles(a.R, vrows, a.rt) * std::max(1, (int)a.split);
    LinearArgs b = a;
    const char *ge = getenv("KVR_TILED_GROUP");  // tuning: row blocks that may form one group
    b.group_all = ge && *ge ? atoi(ge) : GROUP_ALL;
    switch (a.rt) {
        case 4: launch_mt<4>(epi, b, jobs, s); break;
        case 5: launch_mt<5>(epi, b, jobs, s); break;
        case 6: launch_mt<6>(epi, b, jobs, s); break;
        case 7: launch_mt<7>(epi, b, jobs, s); break;
        case 8: launch_mt<8>(epi, b, jobs, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace kvr
