// Routers for any supported shape and activation type: k_router_generic, plain fp32 FMA, and those
// that cut the reduction over D into slices (below).
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

// ---- few tokens, float32 layers, widths the matrix-core router does not take or is slower at --------
// The reduction over D is cut into slices of 32 columns, a wave each, whose operands go straight
// from memory into the registers of the matrix instruction: for each of TB blocks of 16 tokens and RB
// blocks of 16 weight rows lane l holds row l % 16, columns 8 (l / 16) .. + 7.  bf16 layers: the
// float32 weights are split into three exact bf16 pieces, so all products are exact (weights that have no such
// pieces, and infinities and NaN on either side, go to the float32 instruction); float32 layers:
// v_mfma_f32_16x16x4_f32, column 8 (l / 16) + j in instruction j.  The waves of a
// workgroup meet in LDS.  (One thread per token with the tile in LDS, plain FMA: every thread read each
// weight from LDS, 5300 cycles for 64 columns, any number of tokens.)
//  * T <= 16 and few bytes: one workgroup does the whole router and the permutation.
//  * T <= 64: workgroups leave partial dot products, one adds them up in slice order, finishes as
//    above and goes on with the permutation.
//  * more tokens (where: do_route and router_sliced_wins): workgroups of a slice and 16 or 32 tokens, then k_router_final.
//    (One wave per token reads every router weight once per token: 22 us at T = 2048, D = 768, 24 rows.)
// The gating residual (Eq.6) is 32 and more columns of its own, W_res against the previous logits, which
// follow those of D: no kernel has to bring the two into LDS.
//
// Slices of the reduction: 32 columns of D each, then of the previous logits.
__host__ __device__ inline int router_slices(const Dims &d, bool residual) { return (d.D + 31) / 32 + (residual ? (d.N + 31) / 32 : 0); }

// The partial logits of slices first, first + stride, ...: acc[tb][rb][v]
// of lane l belongs to token t0 + 16 tb + l % 16 and weight row 16 rb + 4 (l / 16) + v (rows past the
// last repeat it, and are never read).
// SETS: 2 keeps every other slice of the wave in accumulators of its own: no chain of sums is longer than one slice
// while a wave has two.
template <typename AT, int TB, int RB, int SETS = 1>
__device__ inline void few_dots(const RouterArgs &a, int t0, int first, int stride, f32x4 (&acc)[TB][RB]) {
    constexpr bool BF16 = ActVec<AT>::N == 8;
    constexpr int XV = BF16 ? 1 : 2;                       // 16-byte loads of 8 columns of x
    const int lane = threadIdx.x % kWave, l16 = lane % 16, lq = lane / 16;
    const int D = a.d.D, N = a.d.N, rows = N + 2 * a.d.n_const, n = (D + 31) / 32;
    const AT *px[TB];
    const float *pw[RB];
#pragma unroll
    for (int i = 0; i < TB; ++i) px[i] = static_cast<const AT *>(a.x) + (size_t)min(t0 + 16 * i + l16, a.d.T - 1) * D;
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int r = min(16 * i + l16, rows - 1);
        pw[i] = r < N ? a.W_g + (size_t)r * D : a.W_c + (size_t)(r - N) * D;
    }
    struct Slice {
        ActVec<AT> x[TB][XV];
        f32x4 w[RB][2];
    };
    auto load = [&](int ks, Slice &s) {
        const int k = min(32 * min(ks, n - 1) + 8 * lq, D - 8);
#pragma unroll
        for (int i = 0; i < TB; ++i)
#pragma unroll
            for (int u = 0; u < XV; ++u) s.x[i][u] = load_vec(px[i] + k + 4 * u);
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int u = 0; u < 2; ++u) s.w[i][u] = *reinterpret_cast<const f32x4 *>(pw[i] + k + 4 * u);
    };
    // bf16: part 0 has the products of the hi pieces, part 1 all others; float32: part p the columns
    // with 8 (l / 16) + j, j % 4 = p (short chains of sums: a few of them are as exact as a tree)
    constexpr int NP = BF16 ? 2 : 4;
    f32x4 part[SETS * NP][TB][RB];
#pragma unroll
    for (int q = 0; q < SETS * NP; ++q)
#pragma unroll
        for (int i = 0; i < TB; ++i)
#pragma unroll
            for (int j = 0; j < RB; ++j) part[q][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    uint32_t lost = 0;
    auto mul = [&](auto set_c, int ks, Slice &s) {
        constexpr int P = SETS == 2 ? NP * decltype(set_c)::value : 0;
        if (ks >= n) return;                               // (the same for the whole wave)
        if (32 * ks + 8 * lq >= D) {                       // columns past the last: zero in both operands
#pragma unroll
            for (int i = 0; i < TB; ++i)
#pragma unroll
                for (int u = 0; u < XV; ++u) s.x[i][u].v = {};
#pragma unroll
            for (int i = 0; i < RB; ++i) s.w[i][0] = s.w[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int j = 0; j < RB; ++j) {
            if constexpr (BF16) {
                const Split4 p0 = split4(s.w[j][0], lost), p1 = split4(s.w[j][1], lost);
                auto join = [](u32x2 u, u32x2 v) {
                    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                    return __builtin_bit_cast(bf16x8, u32x4{u[0], u[1], v[0], v[1]});
                };
                const bf16x8 hi = join(p0.hi, p1.hi), mid = join(p0.mid, p1.mid), lo = join(p0.lo, p1.lo);
#pragma unroll
                for (int i = 0; i < TB; ++i) {
                    const bf16x8 xv = __builtin_bit_cast(bf16x8, s.x[i][0].v);
                    part[P][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, xv, part[P][i][j], 0, 0, 0);
                    part[P + 1][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mid, xv, part[P + 1][i][j], 0, 0, 0);
                    part[P + 1][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, xv, part[P + 1][i][j], 0, 0, 0);
                }
            } else {
#pragma unroll
                for (int c = 0; c < 8; ++c)
#pragma unroll
                    for (int i = 0; i < TB; ++i)
                        part[P + c % NP][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            s.w[j][c / 4][c % 4], s.x[i][c / 4].get(c % 4), part[P + c % NP][i][j], 0, 0, 0);
            }
        }
    };
    // previous logits: eight columns of the slice per lane, as above, float32 (16 bytes at a time where
    // rows are whole 16-byte pieces, which then are in the row or past it: T = 300, D = 768, 52 rows 15.5
    // -> 13.9 us, T = 64 17.6 -> 16.3)
    auto residual = [&](int m0) {
        float pv[TB][8], wv[RB][8];
        if (N % 4 == 0) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int m = m0 + 8 * lq + 4 * u, at = m < N ? m : 0;
                auto get = [&](const float *from, float *to) {
                    const f32x4 v = *reinterpret_cast<const f32x4 *>(from);
#pragma unroll
                    for (int c = 0; c < 4; ++c) to[c] = v[c];
                };
#pragma unroll
                for (int i = 0; i < TB; ++i) get(a.prev_gate + (size_t)min(t0 + 16 * i + l16, a.d.T - 1) * N + at, pv[i] + 4 * u);
#pragma unroll
                for (int j = 0; j < RB; ++j) get(a.W_res + (size_t)min(16 * j + l16, N - 1) * N + at, wv[j] + 4 * u);
            }
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int m = min(m0 + 8 * lq + c, N - 1);
#pragma unroll
                for (int i = 0; i < TB; ++i) pv[i][c] = a.prev_gate[(size_t)min(t0 + 16 * i + l16, a.d.T - 1) * N + m];
#pragma unroll
                for (int j = 0; j < RB; ++j) wv[j][c] = a.W_res[(size_t)min(16 * j + l16, N - 1) * N + m];
            }
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const bool in = m0 + 8 * lq + c < N;           // columns past the last: zero in both operands
#pragma unroll
            for (int j = 0; j < RB; ++j) wv[j][c] = in ? wv[j][c] : 0.f;
#pragma unroll
            for (int i = 0; i < TB; ++i) pv[i][c] = in ? pv[i][c] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < RB; ++j)
#pragma unroll
            for (int i = 0; i < TB; ++i) {
                f32x4 r[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                for (int c = 0; c < 8; ++c) r[c % 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[j][c], pv[i][c], r[c % 2], 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 4; ++v)                // (rows of W_c: none, whatever the previous logits hold)
                    if (16 * j + 4 * lq + v < N) acc[i][j][v] += r[0][v] + r[1][v];
            }
    };
    const int n_all = router_slices(a.d, a.prev_gate != nullptr);
    Slice s0, s1;
    load(first, s0);
    if (first + stride < n) load(first + stride, s1);
    for (int ks = first; ks < n; ks += 2 * stride) {
        mul(std::integral_constant<int, 0>{}, ks, s0);
        if (ks + 2 * stride < n) load(ks + 2 * stride, s0);
        mul(std::integral_constant<int, 1>{}, ks + stride, s1);
        if (ks + 3 * stride < n) load(ks + 3 * stride, s1);
    }
    bool odd = false;
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
        for (int j = 0; j < RB; ++j) {
            acc[i][j] = part[0][i][j] + part[1][i][j];
#pragma unroll
            for (int q = 2; q < SETS * NP; q += 2) acc[i][j] += part[q][i][j] + part[q + 1][i][j];
#pragma unroll
            for (int v = 0; v < 4; ++v) odd |= !__builtin_isfinite(acc[i][j][v]);
        }
    if constexpr (BF16) {
        // What the pieces do not give comes from the float32 instruction: sums that are not finite (the lower
        // pieces of an infinity are NaN, and hi of a NaN may be infinite), one by one, so that no token
        // depends on another; all of them when a weight was too small for its pieces.
        const bool small = __ballot(split_lost(lost)) != 0;
        if (small || __ballot(odd) != 0) {
            // (block by block: few registers, or fewer waves of the others fit a SIMD)
#pragma unroll
            for (int i = 0; i < TB; ++i)
#pragma unroll
                for (int j = 0; j < RB; ++j) {
                    f32x4 plain = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                    for (int ks = first; ks < n; ks += stride) {
                        const int k = 32 * ks + 8 * lq, at = min(k, D - 8);
                        const bool in = k < D;             // columns past the last: zero in both operands
                        const ActVec<AT> x = load_vec(px[i] + at);
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const f32x4 w = *reinterpret_cast<const f32x4 *>(pw[j] + at + 4 * u);
#pragma unroll
                            for (int c = 0; c < 4; ++c)
                                plain = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? w[c] : 0.f, in ? x.get(4 * u + c) : 0.f, plain, 0, 0, 0);
                        }
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (small || !__builtin_isfinite(acc[i][j][v])) acc[i][j][v] = plain[v];
                }
        }
    }
    // (the wave's first slice of them)
    for (int ks = first + (max(n - first, 0) + stride - 1) / stride * stride; ks < n_all; ks += stride) residual(32 * (ks - n));
}

// Floats from one slice of partial sums to the next, a multiple of four: slices are read 16 bytes at a time.
__host__ __device__ inline size_t slice_floats(const Dims &d) { return ((size_t)d.T * (d.N + 2 * d.n_const) + 3) & ~(size_t)3; }

// Element c of a block's [tokens][rows] array: token c / rows and row c % rows; inv = 2^32 / rows
// rounded up (0: one row), exact while c rows < 2^32.
struct RowOf {
    int tt, r;
    __device__ RowOf(int c, int rows, uint32_t inv) {
        tt = inv ? (int)__umulhi((uint32_t)c, inv) : c;
        r = c - tt * rows;
    }
};
static uint32_t inverse_rows(int rows) { return rows < 2 ? 0u : (uint32_t)((1ull << 32) / (unsigned)rows + 1); }

// The sums of W waves, red [W][TB * RB][64 lanes][4], for (token tt, weight row r) of the block: a tree.
template <int W, int TB, int RB>
__device__ inline float few_sum(const float (*red)[TB * RB][kWave][4], int tt, int r) {
    const int blk = tt / 16 * RB + r / 16, ln = r % 16 / 4 * 16 + tt % 16;
    float v[W];
#pragma unroll
    for (int w = 0; w < W; ++w) v[w] = red[w][blk][ln][r % 4];
#pragma unroll
    for (int h = W / 2; h >= 1; h /= 2)
#pragma unroll
        for (int w = 0; w < h; ++w) v[w] += v[w + h];
    return v[0];
}

// Workgroup (slice, block of 16 TB tokens) of W waves: the partial sums of its columns.
template <typename AT, int TB, int RB, int W>
__global__ __launch_bounds__(W *kWave) void k_router_small_partial(RouterArgs a, uint32_t inv, float *partial) {
    __shared__ __attribute__((aligned(16))) float red[W][TB * RB][kWave][4];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int T = a.d.T, rows = a.d.N + 2 * a.d.n_const, t0 = blockIdx.y * 16 * TB;
    f32x4 acc[TB][RB];
    few_dots<AT, TB, RB>(a, t0, blockIdx.x * W + wave, gridDim.x * W, acc);
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
        for (int j = 0; j < RB; ++j) *reinterpret_cast<f32x4 *>(red[wave][i * RB + j][tid % kWave]) = acc[i][j];
    __syncthreads();
    float *dst = partial + blockIdx.x * slice_floats(a.d) + (size_t)t0 * rows;
    const int n_el = min(16 * TB, T - t0) * rows;
#pragma unroll 1
    for (int c = tid; c < n_el; c += W * kWave) {
        const RowOf o(c, rows, inv);
        dst[c] = few_sum<W, TB, RB>(red, o.tt, o.r);
    }
}

// The sums of the slices of four elements, all loads before the first addition, as trees of four in slice
// order.  (One element per thread, the fewer bytes per load instruction: T = 777, 17 slices 10.6 - 12.9 us, 7.0 - 9.1 now;
// eight at a time, 12 - 17.)
template <int MAXS>
__device__ inline f32x4 add_slices(const float *part, size_t step, int splits) {
    f32x4 v[MAXS], sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < MAXS; ++u) v[u] = *reinterpret_cast<const f32x4 *>(part + min(u, splits - 1) * step);
    __builtin_amdgcn_sched_barrier(0);                     // (or the compiler trades loads in flight for registers)
    auto at = [&](int u) { return u < splits ? v[u] : f32x4{0.f, 0.f, 0.f, 0.f}; };
#pragma unroll
    for (int u = 0; u < MAXS; u += 4) sum += (at(u) + at(u + 1)) + (at(u + 2) + at(u + 3));
    return sum;
}

// Logits of n_tok tokens from t0 on, from their slices, with all NT threads: to dots (LDS) and to memory.
constexpr int kDotStride = kMaxRouterRows + 1;
template <int MAXS, int NT>
__device__ inline void finish_logits(const RouterArgs &a, int t0, int n_tok, int splits, uint32_t inv, float *dots) {
    const int N = a.d.N, rows = N + 2 * a.d.n_const, n_el = n_tok * rows;
    const float *part = a.partial + (size_t)t0 * rows;     // (t0 is a multiple of four)
    for (int c0 = threadIdx.x * 4; c0 < n_el; c0 += NT * 4) {
        const f32x4 sum = add_slices<MAXS>(part + c0, slice_floats(a.d), splits);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = c0 + i;
            if (c >= n_el) break;
            const RowOf o(c, rows, inv);
            float L = sum[i];
            if (a.bias && o.r < N) L += a.bias[o.r];
            dots[o.tt * kDotStride + o.r] = L;
            if (o.r < N) a.out_gate[(size_t)(t0 + o.tt) * N + o.r] = L;
        }
    }
}

// The ends of these routers are one chain of instructions in few waves, fetched once: they are written to
// be short, not unrolled.

// From the logits (in dots, [T][kDotStride], LDS) to the permutation, one workgroup of at least 16 T threads.
template <int MAXN>
__device__ inline void few_finish(const RouterArgs &a, const Workspace &w, const CapArgs &cap, const float *dots, int *idx,
                                  int *rank) {
    const int tid = threadIdx.x, T = a.d.T, K = a.d.k;
    __syncthreads();
    if (tid / kWave * 4 < T) {            // whole waves, four tokens each
        const int tok = tid >> 4, tk = min(tok, T - 1);
        router_token<MAXN, 16>(a, (size_t)tk, tok < T, tid & 15, dots + tk * kDotStride, nullptr, idx + tk * K);
    }
    __syncthreads();
    if (tid < kWave) perm_one_wave(a.d, w, cap, idx, rank);
}

// The second kernel and the permutation in one launch, for T <= kRouterFusedT: one
// workgroup adds the slices of every logit, does softmax / Top-K / a1 with
// sixteen threads per token, and then groups the T*k selections, which it still
// holds in LDS, by expert.
constexpr int kFewThreads = 1024;
template <int MAXN, int MAXS>
__global__ __launch_bounds__(kFewThreads) void k_router_small_final_perm(RouterArgs a, int n_splits, uint32_t inv,
                                                                         Workspace w, CapArgs cap) {
    __shared__ float dots[kRouterFusedT * kDotStride];
    __shared__ int idx[kRouterFusedT * kMaxTopK], rank[kRouterFusedT * kMaxTopK];
    finish_logits<MAXS, kFewThreads>(a, 0, a.d.T, n_splits, inv, dots);
    few_finish<MAXN>(a, w, cap, dots, idx, rank);
}

// The whole router and the permutation in one workgroup of W waves, T <= 16.
constexpr int kRouterOneT = 16;
template <typename AT, int RB, int MAXN, int W>
__global__ __launch_bounds__(W *kWave) void k_router_one(RouterArgs a, uint32_t inv, Workspace w, CapArgs cap) {
    __shared__ float dots[kRouterOneT * kDotStride];
    __shared__ int idx[kRouterOneT * kMaxTopK], rank[kRouterOneT * kMaxTopK];
    __shared__ __attribute__((aligned(16))) float red[W][RB][kWave][4];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int N = a.d.N, rows = N + 2 * a.d.n_const, n_el = a.d.T * rows;
    static_assert(W * 4 >= kRouterOneT, "sixteen threads per token");
    f32x4 acc[1][RB];
    few_dots<AT, 1, RB>(a, 0, wave, W, acc);
#pragma unroll
    for (int j = 0; j < RB; ++j) *reinterpret_cast<f32x4 *>(red[wave][j][tid % kWave]) = acc[0][j];
    __syncthreads();
#pragma unroll 1
    for (int c = tid; c < n_el; c += W * kWave) {
        const RowOf o(c, rows, inv);
        const float bias = a.bias && o.r < N ? a.bias[o.r] : 0.f;
        const float L = few_sum<W, 1, RB>(red, o.tt, o.r) + bias;
        dots[o.tt * kDotStride + o.r] = L;
        if (o.r < N) a.out_gate[(size_t)o.tt * N + o.r] = L;
    }
    few_finish<MAXN>(a, w, cap, dots, idx, rank);
}

// The second kernel for more tokens, in blocks of 64: logits, softmax, Top-K and a1, the selections per expert
// for the permutation, and the sums of the statistics, which also the one-kernel router leaves.
constexpr int kRouterFinalTok = kRouterSlicedTok, kRouterFinalThreads = 1024;
template <int MAXN, int MAXS>
__global__ __launch_bounds__(kRouterFinalThreads) void k_router_final(RouterArgs a, int splits, uint32_t inv) {
    constexpr int TOK = kRouterFinalTok, NT = kRouterFinalThreads;
    static_assert(NT == 16 * TOK, "sixteen threads per token");
    __shared__ float dots[TOK * kDotStride];
    __shared__ float probs[TOK * (MAXN + 1)];
    __shared__ int s_hist[MAXN];
    const int tid = threadIdx.x, t0 = blockIdx.x * TOK;
    const int N = a.d.N, n_tok = min(TOK, a.d.T - t0);
    if (tid < N) s_hist[tid] = 0;
    finish_logits<MAXS, NT>(a, t0, n_tok, splits, inv, dots);
    __syncthreads();
    // (tokens past the end compute on whatever their part of `dots` holds and store nothing)
    const int tok = tid >> 4;
    router_token<MAXN, 16>(a, (size_t)(t0 + tok), tok < n_tok, tid & 15, dots + tok * kDotStride,
                                       a.chunk_hist ? s_hist : nullptr, nullptr,
                                       a.bal_partial ? probs + tok * (N + 1) : nullptr);
    router_block_sums<TOK, NT>(a, s_hist, probs);
}

// The whole router for a block of 16 TB tokens in one workgroup of W waves, which take the slices of D in turn; what
// it leaves is what k_router_final leaves.  With narrow layers the workgroups are short chains of instructions and
// memory latencies that one launch pays for once; beside k_router_mfma they are two or four times as many, so that the
// chip is full (figures: router_block_tokens).  Weights are read once per block, from the caches.
template <typename AT, int TB, int RB, int MAXN, int W, int SETS>
__global__ __launch_bounds__(W *kWave) void k_router_block(RouterArgs a, uint32_t inv) {
    constexpr int TOK = 16 * TB, NT = W * kWave, L = 16;
    constexpr int RED = W * TB * RB * kWave * 4, PROBS = TOK * (MAXN + 1);
    static_assert(NT >= L * TOK && NT >= 4 * kMaxExperts, "sixteen threads per token, four per expert");
    __shared__ float dots[TOK * kDotStride];
    __shared__ int s_hist[MAXN];
    __shared__ __attribute__((aligned(16))) float red[RED > PROBS ? RED : PROBS];     // partial sums, then probabilities
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), t0 = blockIdx.x * TOK;
    const int N = a.d.N, rows = N + 2 * a.d.n_const, n_tok = min(TOK, a.d.T - t0), n_el = n_tok * rows;
    if (tid < N) s_hist[tid] = 0;
    f32x4 acc[TB][RB];
    few_dots<AT, TB, RB, SETS>(a, t0, wave, W, acc);
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
        for (int j = 0; j < RB; ++j)
            *reinterpret_cast<f32x4 *>(red + (((size_t)wave * TB * RB + i * RB + j) * kWave + tid % kWave) * 4) = acc[i][j];
    __syncthreads();
#pragma unroll 1
    for (int c = tid; c < n_el; c += NT) {
        const RowOf o(c, rows, inv);
        const float bias = a.bias && o.r < N ? a.bias[o.r] : 0.f;
        const float v = few_sum<W, TB, RB>(reinterpret_cast<const float(*)[TB * RB][kWave][4]>(red), o.tt, o.r) + bias;
        dots[o.tt * kDotStride + o.r] = v;
        if (o.r < N) a.out_gate[(size_t)(t0 + o.tt) * N + o.r] = v;
    }
    __syncthreads();
    // (whole waves; tokens past the end compute on whatever their part of `dots` holds and store nothing)
    if (tid < L * TOK) {
        const int tok = tid / L;
        router_token<MAXN, L>(a, (size_t)(t0 + tok), tok < n_tok, tid % L, dots + tok * kDotStride, a.chunk_hist ? s_hist : nullptr,
                              nullptr, a.bal_partial ? red + tok * (N + 1) : nullptr);
    }
    router_block_sums<TOK, NT>(a, s_hist, red);
}

// Slices of a call with more than kRouterFusedT tokens, at most `most`, whose workgroups take `blocks` blocks of
// tokens each.  bf16: four to eight of them.  Up to eight, all workgroups of an XCD have the same slice and
// keep its weights in their L2, and each further one is more for the second kernel to add; and what counts is how
// long the fullest CU works, rounds of 256 workgroups over slices.  us with 4 / 5 / 8 / as many as fit, D = 4096, 24 rows:
// T = 300 14.6 / 14.0 / 12.5 / 12.3 (24), T = 1500 17.3 / 15.8 / 16.0 / 17.3 (18), T = 2048 17.7 / 18.9 / 16.2 / 18.7 (13); 52
// rows: T = 1024 23.9 / 21.7 / 18.5 / 27.2 (12), T = 1500 24.9 / 22.8 / 27.9 / 27.9 (8), T = 2048 25.1 / 29.2 / - / 27.2 (6).
// Of two numbers with the same quotient the smaller one with many rows, whose workgroups do not share a CU well.  (Fewer
// than four: T = 4096, 52 rows 32.8 with two, 37.0 with three, but the logits are 1.36e-7 from float64, not 1.05e-7.)
// Wider layers go on to gain while the workgroups fit the chip: D = 8192, T = 300 with 8 / 20 slices 14.5 / 13.3, with 52
// rows 23.3 / 19.7.  float32 sums round at every fourth product, and short chains of them keep their error
// (T = 2048, D = 768 8.9e-8 with seven slices, 9.5e-8 with four): as many as fit, some 1024 / (T / 64) at most.
static int sliced_splits(const Dims &d, bool bf16, int blocks, int most) {
    if (!bf16) {
        const int fill = (1024 + (d.T + 63) / 64 - 1) / ((d.T + 63) / 64);
        return most < fill ? most : fill;
    }
    if (d.D > 4096 && 8 * blocks < 256) {
        const int fill = 256 / blocks;
        return most < fill ? most : fill;
    }
    int best = most < 4 ? most : 4;
    for (int n = 5; n <= most && n <= 8; ++n) {
        const int gain = (best * blocks + 255) / 256 * n - (n * blocks + 255) / 256 * best;
        if (gain > 0 || (gain == 0 && d.N + 2 * d.n_const <= 32)) best = n;
    }
    return best;
}

int router_split_max(const Dims &d) {
    const size_t slice = slice_floats(d) * sizeof(float);
    const size_t n = router_small_bytes() / slice;
    return (int)(n < kRouterSplits ? n : kRouterSplits);
}

// Instances for up to 8, 20 and 24 slices: a load is issued for each slice of the instance.  us with the smallest that
// fits / with 24: T = 700, D = 1536, 24 rows (7 slices) 10.7 / 12.7, 52 rows 16.4 / 19.4; float32, T = 700, D = 3072 (13 slices)
// 16.4 / 17.0.  The one-workgroup end below: T = 64, D = 768, 24 rows 10.8 / 12.7, D = 4096 (17 slices) 12.3 / 12.9; with more
// than 32 experts four slices take 17.5 in either.
static hipError_t launch_router_final(const RouterArgs &a, int splits, hipStream_t s) {
    const int rows = a.d.N + 2 * a.d.n_const;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((a.d.T + kRouterFinalTok - 1) / kRouterFinalTok), dim3(kRouterFinalThreads), 0, s, a,
                           splits, inverse_rows(rows));
        return hipGetLastError();
    };
    if (a.d.N <= 32)
        return splits <= 8 ? go(k_router_final<32, 8>) : splits <= 20 ? go(k_router_final<32, 20>) : go(k_router_final<32, kRouterSplits>);
    return splits <= 8 ? go(k_router_final<kMaxExperts, 8>) : go(k_router_final<kMaxExperts, kRouterSplits>);
}

size_t router_small_bytes() {
    return (size_t)32 * 256 * kMaxRouterRows * sizeof(float);     // (32 slices of 256 tokens with the most rows)
}

// First kernel of the sliced routers: at most max_splits slices of D.
static hipError_t launch_router_partial(const RouterArgs &a, bool bf16, int max_splits, int *n_splits, hipStream_t s) {
    const int rows = a.d.N + 2 * a.d.n_const, n = router_slices(a.d, a.prev_gate != nullptr);
    const uint32_t inv = inverse_rows(rows);
    auto go = [&](auto tb_c, auto rb_c, auto w_c) {
        constexpr int TB = decltype(tb_c)::value, RB = decltype(rb_c)::value, W = decltype(w_c)::value;
        const int most = (n + W - 1) / W < max_splits ? (n + W - 1) / W : max_splits, blocks = (a.d.T + 16 * TB - 1) / (16 * TB);
        *n_splits = a.d.T <= kRouterFusedT ? most : sliced_splits(a.d, bf16, blocks, most);
        const dim3 grid(*n_splits, blocks), block(W * kWave);
        if (bf16) hipLaunchKernelGGL((k_router_small_partial<bf16_t, TB, RB, W>), grid, block, 0, s, a, inv, a.partial);
        else hipLaunchKernelGGL((k_router_small_partial<float, TB, RB, W>), grid, block, 0, s, a, inv, a.partial);
    };
    typedef std::integral_constant<int, 1> c1;
    typedef std::integral_constant<int, 2> c2;
    typedef std::integral_constant<int, 4> c4;
    typedef std::integral_constant<int, 5> c5;
    typedef std::integral_constant<int, 8> c8;
    static_assert(kMaxRouterRows <= 80, "blocks of 16 weight rows");
    // Blocks of 16 tokens while there are few (short code, and many workgroups), of 32 then; four waves from
    // the point where the chip is full.  us with blocks of 16 x 8 waves / 32 x 8 / 32 x 4 / 64 x 4: T = 100, D = 1536,
    // 24 rows 10.4 / 10.4 / 13.9 / 15.6; T = 777, D = 4096 19.3 / 17.1 / 17.4 / 18.5; T = 2048, D = 4096, 52 rows
    // 34.0 / 28.9 / 27.2 / 26.8.
    auto by_rows = [&](auto tb_c, auto w_c) {
        if (rows <= 32) go(tb_c, c2(), w_c);
        else if (rows <= 64) go(tb_c, c4(), w_c);
        else go(tb_c, c5(), c4());
    };
    if (a.d.T <= 256) by_rows(c1(), c8());
    else if (a.d.T <= 1024) by_rows(c2(), c8());
    else by_rows(c2(), c4());
    return hipGetLastError();
}

hipError_t launch_router_small(const RouterArgs &a, bool bf16, hipStream_t s, const Workspace &perm_ws,
                               const CapArgs &perm_cap) {
    if (a.d.T == 0) return hipSuccess;
    if (a.d.T > kRouterFusedT) return hipErrorInvalidValue;
    const int rows = a.d.N + 2 * a.d.n_const;
    // One workgroup for all of it while one CU reads x and the weights in about the time of a second
    // launch and its first loads, us in one / two kernels, 24 rows: 26 KB (D = 256) 8.3 / 8.5, 75 KB (D = 768, one
    // token) 8.6 / 8.7, 106 KB (D = 1024) 10.0 / 8.6; 52 rows: 55 KB (D = 256) 11.3 / 12.4, 166 KB (D = 768) 14.6 / 12.7.
    // (A launch also costs the host some 2 us.)
    const long long bytes = (long long)a.d.D * (rows * 4 + a.d.T * (bf16 ? 2 : 4));
    if (a.d.T <= kRouterOneT && bytes <= 80 * 1024) {
        auto go = [&](auto kernel, int waves) {
            hipLaunchKernelGGL(kernel, dim3(1), dim3(waves * kWave), 0, s, a, inverse_rows(rows), perm_ws, perm_cap);
            return hipGetLastError();
        };
        if (rows <= 32) return bf16 ? go(k_router_one<bf16_t, 2, 32, 16>, 16) : go(k_router_one<float, 2, 32, 16>, 16);
        return bf16 ? go(k_router_one<bf16_t, 5, kMaxExperts, 8>, 8) : go(k_router_one<float, 5, kMaxExperts, 8>, 8);
    }
    int n_splits = 0;
    const hipError_t e = launch_router_partial(a, bf16, kRouterSplits, &n_splits, s);
    if (e != hipSuccess) return e;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(1), dim3(kFewThreads), 0, s, a, n_splits, inverse_rows(rows), perm_ws, perm_cap);
        return hipGetLastError();
    };
    if (a.d.N <= 32)
        return n_splits <= 8    ? go(k_router_small_final_perm<32, 8>)
               : n_splits <= 20 ? go(k_router_small_final_perm<32, 20>)
                                : go(k_router_small_final_perm<32, kRouterSplits>);
    return go(k_router_small_final_perm<kMaxExperts, kRouterSplits>);
}

// Where the sliced router is faster than the matrix-core router in one kernel, whose workgroups of 64
// tokens leave most of the chip empty and walk all of D: router and permutation, us sliced / in one, 24 rows: D = 512
// T = 80 14.5 / 14.1, T = 2048 16.4 / 15.5; D = 768 T = 2048 16.3 / 16.6, T = 2500 17.5 / 16.8; D = 1024 T = 2048 17.6 / 18.3,
// T = 4096 19.3 / 18.5; D = 1536 T = 4096 21.0 / 21.3, T = 6000 23.3 / 21.6; D = 2048 T = 2048 19.4 / 23.7, T = 4096 22.4 /
// 23.6, T = 6000 25.6 / 23.6; 52 rows: D = 512 T = 1024 21.2 / 20.5; D = 768 T = 2048 21.7 / 23.3, T = 2500 23.7 / 23.2;
// D = 1024 T = 4096 26.3 / 25.1; D = 2048 T = 4096 31.3 / 33.0, T = 6000 39.2 / 34.0.  (D = 640 and 896, an odd number of pairs
// of K tiles, where the other kernel has one group of waves, would gain as well, up to 4096 tokens: D = 640 T = 2048
// 16.4 / 19.2, D = 896 T = 4096 18.5 / 23.1.)
bool router_sliced_wins(const Dims &d) { return (d.D >= 768 && d.T <= 2048) || (d.D >= 1536 && d.T <= 4096); }

// Tokens of a workgroup where the one-kernel router on blocks is faster than the sliced or the matrix-core router
// and its logits no further from float64, else 0.  Router and permutation, us, and in brackets the logits' error
// against float64, 1e-8.  Blocks of 16 / the matrix-core router, where it is the other choice:
//   24 weight rows: D = 128 T = 65 8.3 [6.0] / 11.9 [6.6], T = 2048 9.1 / 13.6; D = 512 T = 300 9.8 [6.9] /
//   13.8 [7.9]; D = 1024 T = 4096 13.7 [8.1] / 17.2 [10]; 52 rows: D = 256 T = 2048 11.9 [6.8] / 17.9
//   [7.2]; D = 768 T = 4096 17.4 [7.6] / 22.1 [9.2].
// Against slices, which spread a wide layer's few tokens over more CUs: what a block takes grows with D times its
// 16, 32 or 64 weight rows and eight for x, what slices take with T.  bf16, block / slices:
//   D = 768, 24 rows T = 65 10.2 / 11.9, T = 2048 11.0 [7.1] / 14.2 [7.2]; D = 1024, 24 rows T = 65 11.4 /
//   12.1, T = 300 11.6 / 13.5; D = 1536, 24 rows T = 65 13.1 / 12.1, T = 300 13.4 / 13.4, T = 2048 14.0
//   [7.7] / 16.4 [7.7]; D = 2048, 24 rows T = 1024 15.7 / 14.1, T = 2048 16.3 / 17.7, T = 4096 17.4 / 20.4;
//   D = 4096, 24 rows T = 2048 24.0 / 20.1, T = 4096 24.6 / 25.3; D = 2048, 12 rows T = 300 12.0 / 13.0; D
//   = 4096, 12 rows T = 300 16.8 / 14.2, T = 3000 18.2 / 21.1; D = 768, 52 rows T = 65 14.8 / 15.4, T =
//   1024 15.4 [7.4] / 17.7 [7.3]; D = 1024, 52 rows T = 65 16.3 / 15.3, T = 2048 17.5 [7.5] / 19.6 [7.5].
// The width ends where slices are more exact (float32 sums round at every fourth product and get worse with
// longer chains).  bf16: D = 2048, 12 rows T = 700 12.2 [8.0] / 13.8 [7.6], T = 2048 13.1 [7.9] / 16.8
// [7.9]; D = 1536, 52 rows T = 2100 22.2 [8.1] / 23.0 [7.8].  float32: D = 1024, 24 rows T = 2048 13.7
// [9.1] / 18.9 [9.2], D = 1536 15.8 [10.1] / 20.6 [9.5]; D = 512, 52 rows T = 300 13.5 [8.9] / 16.0 [9.1],
// D = 768 16.1 [9.9] / 15.9 [9.0]; D = 128, 12 rows T = 256 8.8 / 12.4.
// One workgroup per CU: blocks of 16 up to T = 4096 (24 rows, D = 768 T = 4300 15.4 [7.5], of 32 13.4,
// matrix cores 16.2; float32, D = 1024, 24 rows T = 4096 14.6 / 19.5, T = 5000 22.9 / 21.6), of 32 up to
// 8192 (24 rows, D = 768 T = 8192 14.1 / 16.8, T = 9000 18.3 / 17.6; 52 rows, D = 4096 T = 4097 44.6 [14] /
// 46.2 [19], T = 8192 46.3 / 47.6, T = 9000 84 / 49; 12 rows, D = 512 T = 9000 12.4 / 14.2, but D = 2048
// 21.8 / 20.7).  Blocks of 32 are eight waves with one set of sums: widths that slices would take go up to
// 512 there (D = 520 T = 8192 12.0 [7.0] / 18.3 [7.0], D = 1000 13.9 [8.1] / 18.4 [7.4]).
// More than 64 weight rows (five blocks of the instruction): no instance.
constexpr int kRouterBlocks = 256;
static_assert(kRouterBlocks <= kPermDirectChunks, "the permutation's table of first ranks has no rows for these blocks");
int router_block_tokens(const Dims &d, bool bf16) {
    const int rows = d.N + 2 * d.n_const, padded = rows <= 16 ? 16 : rows <= 32 ? 32 : 64;
    if (d.T <= kRouterFusedT || rows > 64 || d.T > 32 * kRouterBlocks) return 0;
    const bool mfma = bf16 && router_mfma_supported(d);
    if (d.T > 16 * kRouterBlocks) return mfma || (bf16 && d.D <= 512) ? 32 : 0;
    if (mfma && !router_sliced_wins(d)) return 16;
    const int widest = bf16 ? (rows > 32 ? 1024 : d.T < 1536 ? 1536 : d.D) : rows > 32 ? 512 : 1024;
    if (d.D > widest) return 0;
    const int most = d.T < 256 ? 40000 : d.T < 1536 ? 60000 : d.T <= 2048 ? 96000 : 120000;
    return (long long)d.D * (padded + 8) <= most ? 16 : 0;
}

// Waves and sets of sums.  Eight waves have at most two slices each up to D = 512; wider layers take sixteen with two
// sets where they replace slices, so that chains of sums stay as short as there (eight of them with more than
// 32 rows, whose registers do not fit sixteen): bf16, 24 rows, D = 1024 T = 2048 12.0 us [7.3], eight waves with
// one set 11.9 [8.0].  The matrix-core router's chains are longer than either's, and eight waves with one set are
// the fastest beside it: 52 rows, D = 768 T = 4096 17.4 us [7.6], with two sets 17.7 [7.4], matrix cores [9.2]; 24 rows, D =
// 256 9.1 us, sixteen waves 10.0.  float32, 24 rows, D = 256 eight waves 9.1, sixteen 10.3 [8.2 both], D = 768 11.6
// [9.7] and 11.8 [8.9]; 12 rows, D = 768 sixteen 10.3 [8.9].
hipError_t launch_router_block(const RouterArgs &a, bool bf16, hipStream_t s) {
    const int tok = router_block_tokens(a.d, bf16), rows = a.d.N + 2 * a.d.n_const;
    if (tok == 0 || (size_t)kRouterBlocks * a.d.N * sizeof(int32_t) > router_small_bytes()) return hipErrorInvalidValue;
    auto go = [&](auto kernel, int waves) {
        hipLaunchKernelGGL(kernel, dim3((a.d.T + tok - 1) / tok), dim3(waves * kWave), 0, s, a, inverse_rows(rows));
        return hipGetLastError();
    };
    const bool few = a.d.D <= 512 || (bf16 && router_mfma_supported(a.d) && !router_sliced_wins(a.d));
    if (!bf16) {
        if (rows <= 16) return go(k_router_block<float, 1, 1, 16, 16, 2>, 16);
        if (rows <= 32) return few ? go(k_router_block<float, 1, 2, 32, 8, 2>, 8) : go(k_router_block<float, 1, 2, 32, 16, 2>, 16);
        return go(k_router_block<float, 1, 4, kMaxExperts, 8, 2>, 8);
    }
    if (tok == 32) {
        if (rows <= 16) return go(k_router_block<bf16_t, 2, 1, 16, 8, 1>, 8);
        if (rows <= 32) return go(k_router_block<bf16_t, 2, 2, 32, 8, 1>, 8);
        return go(k_router_block<bf16_t, 2, 4, kMaxExperts, 8, 1>, 8);
    }
    if (rows <= 16) return few ? go(k_router_block<bf16_t, 1, 1, 16, 8, 1>, 8) : go(k_router_block<bf16_t, 1, 1, 16, 16, 2>, 16);
    if (rows <= 32) return few ? go(k_router_block<bf16_t, 1, 2, 32, 8, 1>, 8) : go(k_router_block<bf16_t, 1, 2, 32, 16, 2>, 16);
    return few ? go(k_router_block<bf16_t, 1, 4, kMaxExperts, 8, 1>, 8) : go(k_router_block<bf16_t, 1, 4, kMaxExperts, 8, 2>, 8);
}

hipError_t launch_router_sliced(const RouterArgs &a, bool bf16, hipStream_t s) {
    if (a.d.T == 0) return hipSuccess;
    const int fit = router_split_max(a.d);
    if (fit < 1) return hipErrorInvalidValue;
    int n_splits = 0;
    const hipError_t e = launch_router_partial(a, bf16, fit, &n_splits, s);
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
