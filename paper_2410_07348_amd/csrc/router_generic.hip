// Routers for any supported shape and activation type, plain fp32 FMA.
//
// k_router_generic: one wavefront per token computes, in one pass over x:
//   G(x) = W x (+ W_g G(x_prev)) (+ bias)            (paper Eq.2 / Eq.6)
//   Softmax over all N experts and Top-K of G(x)     (Eq.1)
//   a1 of every constant expert, Softmax(W_c x)_1    (Eq.5)
// Top-K runs on the float32 logits; ties go to the lower index and slots are
// written in descending order of logit.
#include "common.h"
#include "perm_device.h"
#include "router_device.h"

#include <type_traits>

namespace moepp {

constexpr int kRouterWaves = 4;
constexpr int kMaxRouterRows = kMaxExperts + 2 * kMaxConst;

// W_res into LDS with all threads of the workgroup (the caller synchronises).
__device__ inline void stage_wres(const RouterArgs &a, float *wres) {
    if (!a.prev_gate) return;
    for (int c = threadIdx.x; c < a.d.N * a.d.N; c += blockDim.x) wres[c] = a.W_res[c];
}

// Gating residual, bias, softmax, Top-K and a1 for token t by one wave; `dots`
// holds the token's N + 2 n_const dot products with x, `wres` W_res (both LDS).
__device__ inline void router_tail(const RouterArgs &a, int t, int lane, const float *dots,
                                   const float *wres) {
    const int N = a.d.N, K = a.d.k, nc = a.d.n_const;
    // logits: lane i owns expert i
    float L = -INFINITY;
    const bool mine = lane < N;
    float r = 0.f;
    if (a.prev_gate) {
        const float pg = mine ? a.prev_gate[(size_t)t * N + lane] : 0.f;
        for (int m = 0; m < N; ++m) {
            const float pm = __shfl(pg, m, kWave);
            if (mine) r = fmaf(wres[lane * N + m], pm, r);
        }
    }
    if (mine) {
        L = dots[lane] + r;
        if (a.bias) L += a.bias[lane];
        a.out_gate[(size_t)t * N + lane] = L;
    }
    const float mx = wave_max(L);
    const float e = lane < N ? expf(L - mx) : 0.f;
    const float p = e / wave_sum(e);

    // Top-K by K rounds of wave-wide argmax on (logit desc, index asc)
    // (a NaN is selected like -infinity; a lane without an expert, or whose expert is taken, holds
    // -infinity at an index that loses against every other)
    float cand = L == L ? L : -INFINITY;
    int cand_i = mine ? lane : 0x7fffffff;
    for (int s = 0; s < K; ++s) {
        float bv = cand;
        int bi = cand_i;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            float ov = __shfl_xor(bv, o, kWave);
            int oi = __shfl_xor(bi, o, kWave);
            if (ov > bv || (ov == bv && oi < bi)) {
                bv = ov;
                bi = oi;
            }
        }
        float pw = __shfl(p, bi, kWave);
        if (lane == bi) {
            cand = -INFINITY;
            cand_i = 0x7fffffff;
        }
        if (lane == 0) {
            a.topk_idx[(size_t)t * K + s] = bi;
            a.topk_w[(size_t)t * K + s] = pw;
        }
    }

    if (lane < nc) {
        float l1 = dots[N + 2 * lane], l2 = dots[N + 2 * lane + 1];
        a.alpha1[(size_t)t * nc + lane] = 1.f / (1.f + expf(l2 - l1));
    }
}

template <typename AT>
__global__ __launch_bounds__(kRouterWaves *kWave) void k_router_generic(RouterArgs a) {
    __shared__ float dots[kRouterWaves][kMaxRouterRows];
    __shared__ float wres[kMaxExperts * kMaxExperts];
    const int lane = threadIdx.x % kWave;
    const int w = threadIdx.x / kWave;
    const int t = blockIdx.x * kRouterWaves + w;
    const int D = a.d.D, N = a.d.N, nc = a.d.n_const;
    const bool active = t < a.d.T;
    const int rows = N + 2 * nc;
    constexpr int V = ActVec<AT>::N;
    stage_wres(a, wres);

    if (active) {
        const AT *xt = static_cast<const AT *>(a.x) + (size_t)t * D;
        for (int r = 0; r < rows; ++r) {
            const float *wr = r < N ? a.W_g + (size_t)r * D : a.W_c + (size_t)(r - N) * D;
            float acc = 0.f;
            for (int d = lane * V; d < D; d += kWave * V) {
                ActVec<AT> xv = load_vec(xt + d);
#pragma unroll
                for (int i = 0; i < V; ++i) acc = fmaf(wr[d + i], xv.get(i), acc);
            }
            acc = wave_sum(acc);
            if (lane == 0) dots[w][r] = acc;
        }
    }
    __syncthreads();
    if (active) router_tail(a, t, lane, dots[w], wres);
}

// ---- few tokens -------------------------------------------------------------
// With a few hundred tokens at most, one workgroup per block of tokens leaves
// the chip empty and the pass over x and the router weights runs at one CU's
// load rate.  Here the reduction over D is cut into up to kRsSplits slices:
// workgroup (slice, token block) writes the partial dot products of its slice,
// and a second kernel adds the slices of a token in slice order (the result is
// the same on every run) and finishes as above: one workgroup for up to 64 tokens, which
// goes on with the permutation, else k_router_final.  The float32 layers, and the bf16
// widths that the matrix-core router does not take, run the same way with more tokens:
// one wave per token reads every router weight once per token (22 us at T = 2048,
// D = 768, 24 rows; sliced 12.9).
constexpr int kRsTok = 64;      // tokens per workgroup
constexpr int kRsBK = 64;       // K elements per LDS tile
constexpr int kRsStr = kRsBK + 4;   // floats per LDS tile row: 16-byte reads of 16 consecutive rows cover all banks
constexpr int kRsSplits = kRouterSplits;   // slices at most

// RPT: weight rows per thread; the four waves share 4 RPT >= N + 2 n_const rows
// (rows past the last are zero in LDS, so the inner loop has no conditions).
template <typename AT, int RPT>
__global__ __launch_bounds__(4 * kWave) void k_router_small_partial(RouterArgs a, int slice,
                                                                    float *partial) {
    __shared__ __attribute__((aligned(16))) float sx[kRsTok][kRsStr];
    __shared__ __attribute__((aligned(16))) float sw[4 * RPT][kRsStr];
    const int tid = threadIdx.x, tok = tid % kWave, rg = tid / kWave;
    const int D = a.d.D, N = a.d.N, T = a.d.T, rows = N + 2 * a.d.n_const;
    const int t0 = blockIdx.y * kRsTok;
    const int k_begin = blockIdx.x * slice, k_end = min(k_begin + slice, D);
    constexpr int V = ActVec<AT>::N;
    const AT *x = static_cast<const AT *>(a.x);
    // Products are added up in chains of 8, four for half a tile, then the halves: chains over a
    // whole slice would be further from the exact sum than the one-kernel router's tree is.
    float tot[RPT];
#pragma unroll
    for (int j = 0; j < RPT; ++j) tot[j] = 0.f;
    for (int k0 = k_begin; k0 < k_end; k0 += kRsBK) {
        // x tile [64 tokens][64 k] and weight tile [4 RPT rows][64 k], zero past k_end and past the last row
        for (int c = tid; c < kRsTok * (kRsBK / V); c += 4 * kWave) {
            const int tt = c / (kRsBK / V), kk = (c % (kRsBK / V)) * V;
            const int t = min(t0 + tt, T - 1);
            ActVec<AT> xv;
#pragma unroll
            for (int i = 0; i < V; ++i) xv.set(i, 0.f);
            if (k0 + kk < k_end) xv = load_vec(x + (size_t)t * D + k0 + kk);
#pragma unroll
            for (int i = 0; i < V; i += 4)
                *reinterpret_cast<f32x4 *>(&sx[tt][kk + i]) =
                    f32x4{xv.get(i), xv.get(i + 1), xv.get(i + 2), xv.get(i + 3)};
        }
        for (int c = tid; c < 4 * RPT * (kRsBK / 4); c += 4 * kWave) {
            const int r = c / (kRsBK / 4), kk = (c % (kRsBK / 4)) * 4;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (r < rows && k0 + kk < k_end) {
                const float *wr = r < N ? a.W_g + (size_t)r * D : a.W_c + (size_t)(r - N) * D;
                v = *reinterpret_cast<const f32x4 *>(wr + k0 + kk);
            }
            *reinterpret_cast<f32x4 *>(&sw[r][kk]) = v;
        }
        __syncthreads();
        // wave rg owns rows rg, rg + 4, ...: the weight reads are broadcasts.
        // acc[j][i] collects the k with k % 4 == i of half a tile.
        for (int half = 0; half < kRsBK; half += kRsBK / 2) {
            f32x4 acc[RPT];
#pragma unroll
            for (int j = 0; j < RPT; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
            for (int kk = half; kk < half + kRsBK / 2; kk += 4) {
                const f32x4 xv = *reinterpret_cast<const f32x4 *>(&sx[tok][kk]);
#pragma unroll
                for (int j = 0; j < RPT; ++j) {
                    const f32x4 wv = *reinterpret_cast<const f32x4 *>(&sw[rg + 4 * j][kk]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[j][i] = fmaf(wv[i], xv[i], acc[j][i]);
                }
            }
#pragma unroll
            for (int j = 0; j < RPT; ++j) tot[j] += (acc[j][0] + acc[j][1]) + (acc[j][2] + acc[j][3]);
        }
        __syncthreads();
    }
    if (t0 + tok < T) {
        float *dst = partial + ((size_t)blockIdx.x * T + t0 + tok) * rows;
#pragma unroll
        for (int j = 0; j < RPT; ++j)
            if (rg + 4 * j < rows) dst[rg + 4 * j] = tot[j];
    }
}

// The second kernel and the permutation in one launch, for T <= kRouterFusedT: one
// workgroup adds the slices of every dot product (in slice order), finishes the
// logits (gating residual, bias) with all threads, does softmax / Top-K / a1 with
// four threads per token, and then groups the T*k selections, which it still
// holds in LDS, by expert like k_perm_small does.
// (PER: router_token_quad)
template <int PER>
__global__ __launch_bounds__(kPermSmallWaves *kWave) void k_router_small_final_perm(RouterArgs a, int n_splits,
                                                                                  const float *partial, Workspace w,
                                                                                  CapArgs cap) {
    constexpr int NT = kPermSmallWaves * kWave;
    constexpr int DSTR = kMaxRouterRows + 1, MAXN = 4 * PER;
    __shared__ float dots[kRouterFusedT * DSTR];
    __shared__ __attribute__((aligned(16))) float prevs[kRouterFusedT * residual_stride_max(MAXN)];
    __shared__ __attribute__((aligned(16))) float wres[MAXN * residual_stride_max(MAXN)];
    __shared__ float sbias[MAXN];
    __shared__ int s_idx[kRouterFusedT * kMaxTopK];
    __shared__ int s_rank[kPermSmallWaves][kMaxExperts];
    __shared__ int s_first[kMaxExperts], s_limit[kMaxExperts];
    const int tid = threadIdx.x;
    const int T = a.d.T, N = a.d.N, K = a.d.k, rows = N + 2 * a.d.n_const, rs = residual_stride(N);
    for (int c = tid; c < T * rows; c += NT) {
        // element c = (token c / rows, row c % rows) of every slice; all loads first, then the sum in slice order
        float v[kRsSplits];
#pragma unroll
        for (int sp = 0; sp < kRsSplits; ++sp) v[sp] = sp < n_splits ? partial[(size_t)sp * T * rows + c] : 0.f;
        float sum = 0.f;
#pragma unroll
        for (int sp = 0; sp < kRsSplits; ++sp) sum += v[sp];
        dots[(c / rows) * DSTR + c % rows] = sum;
    }
    if (a.prev_gate) {
        for (int c = tid; c < T * N; c += NT) prevs[(c / N) * rs + c % N] = a.prev_gate[c];
        for (int c = tid; c < N * N; c += NT) wres[(c / N) * rs + c % N] = a.W_res[c];
        zero_residual_pad(prevs, T, N, NT);
        zero_residual_pad(wres, N, N, NT);
    }
    if (tid < N) sbias[tid] = a.bias ? a.bias[tid] : 0.f;
    __syncthreads();
    // consecutive threads: consecutive tokens of one row of W_res, or, with fewer tokens than
    // that is worth, consecutive rows of one token; the padded rows keep both off one bank
    for (int c = tid; c < T * N; c += NT) {
        const int tt = T >= 16 ? c % T : c / N, i = T >= 16 ? c / T : c % N;
        float L = dots[tt * DSTR + i];
        if (a.prev_gate) {
            f32x4 pv[MAXN / 4];
#pragma unroll
            for (int m = 0; m < MAXN / 4; ++m)
                if (4 * m < N) pv[m] = *reinterpret_cast<const f32x4 *>(prevs + tt * rs + 4 * m);
            L += gating_residual<MAXN>(wres + i * rs, pv, N);
        }
        L += sbias[i];
        dots[tt * DSTR + i] = L;        // only this thread reads or writes the element
        a.out_gate[(size_t)tt * N + i] = L;
    }
    __syncthreads();
    if (tid / kWave * kWave < 4 * T) {
        // whole waves (the shuffles are wave-wide); threads past the last token compute on the
        // last token and store nothing
        const int tok = tid >> 2;
        const int tk = tok < T ? tok : T - 1;
        router_token_quad<PER>(a, (size_t)tk, tok < T, tid & 3, dots + tk * DSTR, nullptr, s_idx + tk * K);
    }
    __syncthreads();
    perm_small_body(a.d, w, cap, s_idx, s_rank, s_first, s_limit);
}

// The second kernel of a router that has split D, for blocks of 64 tokens: the slices of
// every dot product are added in slice order, then as in the one-kernel router.
constexpr int kRouterFinalTok = kRouterSlicedTok, kRouterFinalThreads = 512;
template <int ROWS>
__global__ __launch_bounds__(kRouterFinalThreads) void k_router_final(RouterArgs a, int splits) {
    constexpr int TOK = kRouterFinalTok, NT = kRouterFinalThreads;
    constexpr int MAXN = ROWS < kMaxExperts ? ROWS : kMaxExperts, DSTR = ROWS + 1;
    __shared__ __attribute__((aligned(16))) float prevs[TOK * residual_stride_max(MAXN)];
    __shared__ __attribute__((aligned(16))) float wres[MAXN * residual_stride_max(MAXN)];
    __shared__ float dots[TOK * DSTR];
    __shared__ float sbias[MAXN];
    __shared__ int s_hist[MAXN];
    const int tid = threadIdx.x, t0 = blockIdx.x * TOK;
    const int T = a.d.T, N = a.d.N, rows = N + 2 * a.d.n_const;
    const int n_tok = min(TOK, T - t0), rs = residual_stride(N);
    const float *part = a.partial + (size_t)t0 * rows;
    for (int c = tid; c < n_tok * rows; c += NT) {
        float sum = 0.f;
        for (int s0 = 0; s0 < splits; s0 += 8) {           // eight loads in flight, added up as a tree
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = s0 + u < splits ? part[(size_t)(s0 + u) * T * rows + c] : 0.f;
            sum += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
        }
        dots[(c / rows) * DSTR + c % rows] = sum;
    }
    if (a.prev_gate) {
        for (int c = tid; c < n_tok * N; c += NT) prevs[(c / N) * rs + c % N] = a.prev_gate[(size_t)t0 * N + c];
        for (int c = tid; c < N * N; c += NT) wres[(c / N) * rs + c % N] = a.W_res[c];
        zero_residual_pad(prevs, n_tok, N, NT);
        zero_residual_pad(wres, N, N, NT);
    }
    if (tid < N) {
        sbias[tid] = a.bias ? a.bias[tid] : 0.f;
        s_hist[tid] = 0;
    }
    __syncthreads();
    router_finish<TOK, NT, ROWS, 1>(a, t0, dots, prevs, wres, sbias, s_hist);
}

int router_split_max(const Dims &d) {
    const size_t slice = (size_t)d.T * (d.N + 2 * d.n_const) * sizeof(float);
    const size_t n = router_small_bytes() / slice;
    return (int)(n < kRouterSplits ? n : kRouterSplits);
}

hipError_t launch_router_final(const RouterArgs &a, int splits, hipStream_t s) {
    const int rows = a.d.N + 2 * a.d.n_const;
    const dim3 grid((a.d.T + kRouterFinalTok - 1) / kRouterFinalTok), block(kRouterFinalThreads);
    if (rows <= 32) hipLaunchKernelGGL(k_router_final<32>, grid, block, 0, s, a, splits);
    else if (rows <= 64) hipLaunchKernelGGL(k_router_final<64>, grid, block, 0, s, a, splits);
    else hipLaunchKernelGGL(k_router_final<kMaxRouterRows>, grid, block, 0, s, a, splits);
    return hipGetLastError();
}

size_t router_small_bytes() {
    return (size_t)kRsSplits * 256 * kMaxRouterRows * sizeof(float);     // all slices of 256 tokens with the most rows
}

// First kernel of the sliced routers: slices of whole K tiles, at most max_splits of them.
// Returns their number through *n_splits.
static hipError_t launch_router_partial(const RouterArgs &a, bool bf16, int max_splits, int *n_splits, hipStream_t s) {
    const int tiles = (a.d.D + kRsBK - 1) / kRsBK;
    const int per = (tiles + max_splits - 1) / max_splits;      // K tiles per slice
    const int slice = per * kRsBK;
    *n_splits = (a.d.D + slice - 1) / slice;                    // <= max_splits
    const dim3 grid(*n_splits, (a.d.T + kRsTok - 1) / kRsTok), block(4 * kWave);
    const int rows = a.d.N + 2 * a.d.n_const;
    auto go = [&](auto rpt) {
        constexpr int RPT = decltype(rpt)::value;
        if (bf16)
            hipLaunchKernelGGL((k_router_small_partial<bf16_t, RPT>), grid, block, 0, s, a, slice, a.partial);
        else
            hipLaunchKernelGGL((k_router_small_partial<float, RPT>), grid, block, 0, s, a, slice, a.partial);
    };
    static_assert(kMaxRouterRows <= 80, "rows per thread");
    if (rows <= 24) go(std::integral_constant<int, 6>());
    else if (rows <= 40) go(std::integral_constant<int, 10>());
    else go(std::integral_constant<int, 20>());
    return hipGetLastError();
}

hipError_t launch_router_small(const RouterArgs &a, bool bf16, hipStream_t s, const Workspace &perm_ws,
                               const CapArgs &perm_cap) {
    if (a.d.T == 0) return hipSuccess;
    if (a.d.T > kRouterFusedT) return hipErrorInvalidValue;
    int n_splits = 0;
    const hipError_t e = launch_router_partial(a, bf16, kRouterSplits, &n_splits, s);
    if (e != hipSuccess) return e;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(1), dim3(kPermSmallWaves * kWave), 0, s, a, n_splits, a.partial, perm_ws,
                           perm_cap);
    };
    if (a.d.N <= 20) go(k_router_small_final_perm<5>);
    else if (a.d.N <= 32) go(k_router_small_final_perm<8>);
    else go(k_router_small_final_perm<kMaxExperts / 4>);
    return hipGetLastError();
}

hipError_t launch_router_sliced(const RouterArgs &a, bool bf16, hipStream_t s) {
    if (a.d.T == 0) return hipSuccess;
    // slices until there are some 512 workgroups, as far as the partial sums fit
    const int blocks = (a.d.T + kRsTok - 1) / kRsTok, fit = router_split_max(a.d);
    if (fit < 1) return hipErrorInvalidValue;
    int want = (512 + blocks - 1) / blocks, n_splits = 0;
    want = want < fit ? want : fit;
    const hipError_t e = launch_router_partial(a, bf16, want, &n_splits, s);
    return e == hipSuccess ? launch_router_final(a, n_splits, s) : e;
}

hipError_t launch_router_generic(const RouterArgs &a, bool bf16, hipStream_t s) {
    if (a.d.T == 0) return hipSuccess;
    dim3 grid((a.d.T + kRouterWaves - 1) / kRouterWaves), block(kRouterWaves * kWave);
    if (bf16)
        hipLaunchKernelGGL(k_router_generic<bf16_t>, grid, block, 0, s, a);
    else
        hipLaunchKernelGGL(k_router_generic<float>, grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace moepp
