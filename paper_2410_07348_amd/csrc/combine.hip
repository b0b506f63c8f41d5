// Weighted combine (paper Eq.1) with the zero, copy and constant experts
// (Eq.3-5) evaluated in place: tokens routed to those experts never enter a
// GEMM, their contribution is elementwise work on x and the constant vectors.
//
//   y_t = sum over slots s = 0..K-1, in that order, of g_s * E_s(x_t)
//     FFN expert      : E = yffn[row_of[t,s]]
//     zero expert     : E = 0                          (nothing is read)
//     copy expert     : E = x_t
//     constant expert : E = a1 x_t + (1 - a1) v_j
//     any expert, slot dropped by the expert capacity (row_of = -2): nothing
// fp32 accumulation, one rounding to the activation type.  HBM-bound: one wavefront streams one token with
// 16-byte accesses per lane.  (Few tokens of the weight-streaming FFN are combined by the kernel of their
// GEMM2, in the same order with the same roundings.)
#include "common.h"

#include <type_traits>

namespace moepp {

constexpr int kCombineWaves = 4;
// tokens up to which a wave takes a piece of a token, for Top-2 and for more slots
constexpr int kCombineSplitT = 2048, kCombineSplitTMany = 1024;

// KMAX: slots the kernel is unrolled for (2: the paper's Top-2 layers keep their
// per-slot plan in a handful of registers; 4; kMaxTopK: any k).
// A wave takes columns [span y, span (y + 1)) of one token, y = blockIdx.y.
template <typename AT, int KMAX>
__global__ __launch_bounds__(kCombineWaves *kWave) void k_combine(CombineArgs a, int span) {
    const int lane = threadIdx.x % kWave;
    const int t = __builtin_amdgcn_readfirstlane(blockIdx.x * kCombineWaves + threadIdx.x / kWave);
    if (t >= a.d.T) return;
    const int D = a.d.D, K = a.d.k;
    const int zero0 = a.d.n_ffn, copy0 = zero0 + a.d.n_zero, const0 = copy0 + a.d.n_copy;
    constexpr int V = ActVec<AT>::N;

    // Per-slot plan (wave-uniform): coefficient of a gathered row, of x, of v_j.
    float g_row[KMAX], g_x[KMAX], g_v[KMAX];
    const AT *p_row[KMAX];
    const AT *p_v[KMAX];
    bool need_x = false;
    // The token is the same for the whole wave, so its slots come as scalar loads, all of them at once, and
    // in a piece of a token of a layer with copy or constant experts x as well, whether or not a slot wants
    // it: one after the other, behind a branch each, they were a memory latency each.  T = 777, D = 4096
    // 7.0 -> 5.6 us; T = 16384, D = 2048 41.5 -> 38; T = 32768, D = 4096 138.5 -> 134; k = 4 (with an instance of its own),
    // T = 1024, D = 4096 14.7 -> 9.2, T = 16384, D = 1024 39.1 -> 25.4; k = 5 .. 8, whose scalars spill into lanes of vector
    // registers, 0.66 - 1.0 of the time of before in bf16, 0.69 - 1.05 in float32 (36 sizes).  Without copy and constant
    // experts nothing wants x: T = 2048, D = 4096 12.3 us when the slots came one by one, 11.9 with x, 9.7 now.
    int idx[KMAX], rows[KMAX];
    float gs[KMAX];
#pragma unroll
    for (int s = 0; s < KMAX; ++s) {
        idx[s] = rows[s] = 0;
        gs[s] = 0.f;
        if (s < K) {
            const size_t q = (size_t)t * K + s;
            idx[s] = a.topk_idx[q];
            gs[s] = a.topk_w[q];
            rows[s] = a.row_of[q];
        }
    }
    const AT *xt = static_cast<const AT *>(a.x) + (size_t)t * D;
    const int d0 = blockIdx.y * span, d1 = min(D, d0 + span);
    const bool early = gridDim.y > 1 && a.d.n_copy + a.d.n_const > 0;
    ActVec<AT> x0;
    if (early) x0 = load_vec_stream(xt + min(d0 + lane * V, D - V));
#pragma unroll
    for (int s = 0; s < KMAX; ++s) {
        g_row[s] = g_x[s] = g_v[s] = 0.f;
        p_row[s] = p_v[s] = nullptr;
        if (s < K) {
            const int i = idx[s], row = rows[s];
            const float g = gs[s];
            if (row == -2) {
                // over the expert's capacity: dropped
            } else if (i < zero0) {
                g_row[s] = g;
                p_row[s] = static_cast<const AT *>(a.yffn) + (size_t)row * D;
            } else if (i < copy0) {
                // zero expert: contributes nothing
            } else if (i < const0) {
                g_x[s] = g;
                need_x = true;
            } else {
                const int j = i - const0;
                const float a1 = a.alpha1[(size_t)t * a.d.n_const + j];
                g_x[s] = g * a1;
                g_v[s] = g * (1.f - a1);
                p_v[s] = static_cast<const AT *>(a.const_vecs) + (size_t)j * D;
                need_x = true;
            }
        }
    }
    AT *ot = static_cast<AT *>(a.out) + (size_t)t * D;
#pragma unroll 4
    for (int d = d0 + lane * V; d < d1; d += kWave * V) {
        float acc[V];
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] = 0.f;
        ActVec<AT> xv;
        if (early && d < d0 + kWave * V) xv = x0;
        else if (need_x) xv = load_vec_stream(xt + d);
#pragma unroll
        for (int s = 0; s < KMAX; ++s) {
            if (s < K) {
                if (p_row[s]) {
                    ActVec<AT> rv = load_vec_stream(p_row[s] + d);   // read once
#pragma unroll
                    for (int i = 0; i < V; ++i) acc[i] = fmaf(g_row[s], rv.get(i), acc[i]);
                } else if (p_v[s]) {
                    ActVec<AT> vv = load_vec(p_v[s] + d);
#pragma unroll
                    for (int i = 0; i < V; ++i)
                        acc[i] += g_x[s] * xv.get(i) + g_v[s] * vv.get(i);
                } else if (g_x[s] != 0.f) {
#pragma unroll
                    for (int i = 0; i < V; ++i) acc[i] = fmaf(g_x[s], xv.get(i), acc[i]);
                }
            }
        }
        ActVec<AT> ov;
#pragma unroll
        for (int i = 0; i < V; ++i) ov.set(i, acc[i]);
        store_vec_stream(ot + d, ov);
    }
}

hipError_t launch_combine(const CombineArgs &a, bool bf16, hipStream_t s) {
    if (a.d.T == 0) return hipSuccess;
    // With few tokens a wave per token leaves the chip empty and every column waits for the one
    // before it: pieces of one 16-byte access per lane (T = 64,
    // D = 4096: 9.4 -> 4.6 us; T = 777: 11.3 -> 7.0; T = 1500, D = 768: 5.8 -> 5.2).
    const int step = kWave * (bf16 ? ActVec<bf16_t>::N : ActVec<float>::N);
    // With more than two slots the plan is what a piece costs: T = 1999, k = 3, D = 1000 10.3 us in two
    // pieces, 8.0 whole; T = 1000, k = 4, D = 1536 7.7 in three, 9.0 whole.
    const int steps = (a.d.D + step - 1) / step;
    // (as many pieces as the grid's second dimension takes)
    const int span = step * (a.d.T <= (a.d.k <= 2 ? kCombineSplitT : kCombineSplitTMany) ? (steps + 65534) / 65535 : steps);
    const dim3 grid((a.d.T + kCombineWaves - 1) / kCombineWaves, (a.d.D + span - 1) / span);
    const dim3 block(kCombineWaves * kWave);
    auto go = [&](auto k_c) {
        constexpr int KMAX = decltype(k_c)::value;
        if (bf16) hipLaunchKernelGGL((k_combine<bf16_t, KMAX>), grid, block, 0, s, a, span);
        else hipLaunchKernelGGL((k_combine<float, KMAX>), grid, block, 0, s, a, span);
    };
    if (a.d.k <= 2) go(std::integral_constant<int, 2>());
    else if (a.d.k <= 4) go(std::integral_constant<int, 4>());
    else go(std::integral_constant<int, kMaxTopK>());
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// One-time repacking of the expert weights (not part of the forward pass).
template <typename AT>
__global__ __launch_bounds__(256) void k_pack(Dims d, const AT *w1, const AT *w3, const AT *w2,
                                              AT *w13, AT *w2o) {
    constexpr int V = ActVec<AT>::N;
    const size_t per = (size_t)d.F * d.D / V;            // vectors per matrix
    const size_t n = (size_t)d.n_ffn * per;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x) {
        const size_t e = i / per, v = i % per;
        {   // W1 / W3 row f, columns dv..: packed rows of the [2F, D] matrix, in panels
            const int f = (int)(v / (d.D / V));
            const int dv = (int)(v % (d.D / V)) * V;
            AT *dst = w13 + e * 2 * d.F * d.D;
            const int sl = dv / kSlab, in = dv % kSlab;
            store_vec(dst + panel_row(packed_row(f, 0, d.F), sl, 2 * d.F, d.D) + in, load_vec(w1 + i * V));
            store_vec(dst + panel_row(packed_row(f, 1, d.F), sl, 2 * d.F, d.D) + in, load_vec(w3 + i * V));
        }
        {   // W2 row dd, columns fv..: the [D, F] matrix, in panels
            const int dd = (int)(v / (d.F / V));
            const int fv = (int)(v % (d.F / V)) * V;
            AT *dst = w2o + e * d.D * d.F;
            store_vec(dst + panel_row(dd, fv / kSlab, d.D, d.F) + fv % kSlab, load_vec(w2 + i * V));
        }
    }
}

hipError_t launch_pack(const Dims &d, bool bf16, const void *w1, const void *w3, const void *w2,
                       void *w13_out, void *w2_out, hipStream_t s) {
    if (d.n_ffn == 0) return hipSuccess;
    dim3 grid(4096), block(256);
    if (bf16)
        hipLaunchKernelGGL(k_pack<bf16_t>, grid, block, 0, s, d, (const bf16_t *)w1,
                           (const bf16_t *)w3, (const bf16_t *)w2, (bf16_t *)w13_out,
                           (bf16_t *)w2_out);
    else
        hipLaunchKernelGGL(k_pack<float>, grid, block, 0, s, d, (const float *)w1,
                           (const float *)w3, (const float *)w2, (float *)w13_out,
                           (float *)w2_out);
    return hipGetLastError();
}

}  // namespace moepp
