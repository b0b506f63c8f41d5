// Device-side piece of the router that more than one kernel uses.
#pragma once
#include "common.h"

namespace moepp {

// Softmax over all N experts, Top-K (paper Eq.1) and a1 of every constant expert
// (Eq.5) for token t by four neighbouring threads q = 0 .. 3 of a wave; thread q
// owns the experts i = q, q + 4, ... and shuffles combine the four.  Lr: the token's
// N + 2 n_const float32 logits (LDS).  Ties go to the lower index, slots are
// written in descending order of logit.  Every thread of the wave must call this
// (the shuffles are wave-wide); `valid` false: compute, store nothing.
// hist (LDS, may be null): selections per expert, counted with integer atomics.
// sel (LDS, may be null): sel[s] receives the expert of slot s.
// probs (LDS, may be null): probs[i] receives Softmax(G(x))_i, 0 when not valid.
// PER: at least ceil(N / 4); the thread's logits are held in registers.
// expf and a division, not the hardware exp2 of a rounded product and a reciprocal: those are
// off by 3e-6 at logits 77 apart, these by at most 6e-7.
template <int PER>
__device__ inline void router_token_quad(const RouterArgs &a, size_t t, bool valid, int q, const float *Lr,
                                         int *hist, int *sel, float *probs = nullptr) {
    const int N = a.d.N, K = a.d.k, nc = a.d.n_const;
    float v[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) v[j] = q + 4 * j < N ? Lr[q + 4 * j] : -INFINITY;
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < PER; ++j) mx = fmaxf(mx, v[j]);
    mx = fmaxf(mx, __shfl_xor(mx, 1, kWave));
    mx = fmaxf(mx, __shfl_xor(mx, 2, kWave));
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (q + 4 * j < N) sum += expf(v[j] - mx);
    sum += __shfl_xor(sum, 1, kWave);
    sum += __shfl_xor(sum, 2, kWave);
    if (probs) {
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (q + 4 * j < N) probs[q + 4 * j] = valid ? expf(v[j] - mx) / sum : 0.f;
    }
    // A NaN logit (which makes sum, and with it all weights of the token, NaN) is selected like
    // -infinity: all four threads have to agree on the winner, or each takes an expert of its own
    // out of the race and after a few rounds there is none left to select.
#pragma unroll
    for (int j = 0; j < PER; ++j) v[j] = v[j] == v[j] ? v[j] : -INFINITY;
    unsigned open = 0;                          // of this thread's experts: not selected yet
#pragma unroll
    for (int j = 0; j < PER; ++j) open |= (q + 4 * j < N ? 1u : 0u) << j;
    for (int s = 0; s < K; ++s) {
        float bv = -INFINITY;
        int bi = 0x7fffffff;                    // none yet
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if ((open >> j & 1u) && (bi == 0x7fffffff || v[j] > bv)) {
                bv = v[j];
                bi = q + 4 * j;
            }
#pragma unroll
        for (int o = 1; o <= 2; o <<= 1) {
            const float ov = __shfl_xor(bv, o, kWave);
            const int oi = __shfl_xor(bi, o, kWave);
            // larger logit wins, equal logits go to the lower index
            if (oi != 0x7fffffff && (bi == 0x7fffffff || ov > bv || (ov == bv && oi < bi))) {
                bv = ov;
                bi = oi;
            }
        }
        if ((bi & 3) == q) open &= ~(1u << (bi >> 2));
        if (valid && q == 0) {
            a.topk_idx[t * K + s] = bi;
            a.topk_w[t * K + s] = expf(bv - mx) / sum;
            if (hist) atomicAdd(&hist[bi], 1);   // integer counts: the same on every run
            if (sel) sel[s] = bi;
        }
    }
    if (valid)
        for (int j = q; j < nc; j += 4)
            a.alpha1[t * nc + j] = 1.f / (1.f + expf(Lr[N + 2 * j + 1] - Lr[N + 2 * j]));
}

// Rows of W_res and of the previous logits in LDS: a multiple of four floats, so that
// they are read 16 bytes at a time, and an odd multiple, so that 16 rows read at one
// column lie on different banks.
__host__ __device__ constexpr int residual_stride(int N) { return ((N + 3) / 4 | 1) * 4; }
// ... and of the arrays that hold them for any N up to max_n: the widest row.
constexpr int residual_stride_max(int max_n) {
    int w = 0;
    for (int n = 1; n <= max_n; ++n) w = residual_stride(n) > w ? residual_stride(n) : w;
    return w;
}
// Zeros behind the N columns of n rows, up to the next multiple of four, with all threads.
__device__ inline void zero_residual_pad(float *rows, int n, int N, int threads) {
    const int pad = -N & 3;
    for (int c = threadIdx.x; c < n * pad; c += threads) rows[(c / pad) * residual_stride(N) + N + c % pad] = 0.f;
}

// (W_g G(x_prev))_i of one token (Eq.6): row i of W_res (LDS, residual_stride(N)) times the
// token's previous logits.  Even and odd terms are added up apart.
template <int MAXN>
__device__ inline float gating_residual(const float *w, const f32x4 *p, int N) {
    float r[2] = {0.f, 0.f};
#pragma unroll
    for (int m = 0; m < MAXN / 4; ++m) {
        if (4 * m < N) {                       // (both operands are zero between N and the next four)
            const f32x4 wv = *reinterpret_cast<const f32x4 *>(w + 4 * m);
#pragma unroll
            for (int u = 0; u < 4; ++u) r[u & 1] = fmaf(wv[u], p[m][u], r[u & 1]);
        }
    }
    return r[0] + r[1];
}

// The end of a router kernel for the TOK tokens from t0 on, all NT threads: logits
// (gating residual, bias), softmax, Top-K and a1, the logits to memory, and what
// the permutation and the statistics want of the block.  LDS, complete and visible:
// dots [G][TOK][ROWS + 1] partial dot products (added in that order; dots[0] is
// overwritten), prevs and wres rows of residual_stride(N) with zero_residual_pad, sbias [N], s_hist
// [N] zero.
template <int TOK, int NT, int ROWS, int G>
__device__ inline void router_finish(const RouterArgs &a, int t0, float *dots, float *prevs, const float *wres,
                                     const float *sbias, int *s_hist) {
    constexpr int DSTR = ROWS + 1, MAXN = ROWS < kMaxExperts ? ROWS : kMaxExperts;
    const int tid = threadIdx.x, N = a.d.N, rows = N + 2 * a.d.n_const;
    const int n_tok = min(TOK, a.d.T - t0), rs = residual_stride(N);
    // Logits: lane = token, a wave takes every (NT / TOK)-th row, so that the row of W_res is
    // the same in all lanes (one LDS broadcast) and the previous logits stay in registers.
    // One thread per (token, row) in any order read both operands from LDS for every product.
    {
        const int tt = tid % TOK, i0 = tid / TOK;
        constexpr int STEP = NT / TOK;
        static_assert(TOK % kWave == 0 && NT % TOK == 0, "whole waves share a row");
        if (tt < n_tok) {
            f32x4 pv[MAXN / 4];
            if (a.prev_gate) {
#pragma unroll
                for (int m = 0; m < MAXN / 4; ++m)
                    if (4 * m < N) pv[m] = *reinterpret_cast<const f32x4 *>(prevs + tt * rs + 4 * m);
            }
            // all dot products first: the writes below would order the reads of the next row behind them
            constexpr int PER = (ROWS + STEP - 1) / STEP;
            float L[PER];
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int i = min(i0 + u * STEP, rows - 1);
                L[u] = dots[tt * DSTR + i];
#pragma unroll
                for (int g = 1; g < G; ++g) L[u] += dots[(g * TOK + tt) * DSTR + i];
            }
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int i = i0 + u * STEP;
                if (i < N) {
                    if (a.prev_gate) L[u] += gating_residual<MAXN>(wres + i * rs, pv, N);
                    L[u] += sbias[i];
                }
            }
#pragma unroll
            for (int u = 0; u < PER; ++u)
                if (i0 + u * STEP < rows) dots[tt * DSTR + i0 + u * STEP] = L[u];
        }
    }
    __syncthreads();
    // Softmax, Top-K, a1: threads 4 tok .. 4 tok + 3 share token tok (whole waves
    // run this, so the shuffles are whole; tokens past the end compute on whatever their
    // part of `dots` holds and store nothing)
    static_assert(4 * TOK <= NT, "four threads per token");
    static_assert(residual_stride_max(MAXN) > MAXN, "N + 1 probabilities of a token fit its row of prevs");
    if (tid < 4 * TOK) {
        const int tok = tid >> 2;
        // (prevs is free again: the probabilities of the load-balance statistics go there)
        router_token_quad<MAXN / 4>(a, (size_t)(t0 + tok), tok < n_tok, tid & 3, dots + tok * DSTR,
                                    a.chunk_hist ? s_hist : nullptr, nullptr,
                                    a.bal_partial ? prevs + tok * (N + 1) : nullptr);
    }
    // out_gate block [n_tok, N] is contiguous in memory: coalesced copy from LDS
    for (int c = tid; c < n_tok * N; c += NT)
        a.out_gate[(size_t)t0 * N + c] = dots[(c / N) * DSTR + c % N];
    if (a.chunk_hist || a.bal_partial) __syncthreads();
    if (a.chunk_hist)
        for (int c = tid; c < N; c += NT) a.chunk_hist[(size_t)blockIdx.x * N + c] = s_hist[c];
    if (a.bal_partial && tid < 4 * N) {
        // sum of Softmax(G(x))_e over the workgroup's tokens (P_e of Eq.7 is the mean over all
        // tokens): threads 4 e .. 4 e + 3 add a quarter of the tokens each, in token order, and
        // the four sums are added as (0 + 1) + (2 + 3): the same on every run
        const int e = tid >> 2, part = tid & 3;
        double sum = 0.0;
        for (int tt = part * (TOK / 4); tt < (part + 1) * (TOK / 4); ++tt)
            sum += (double)prevs[tt * (N + 1) + e];
        sum += __shfl_xor(sum, 1, kWave);
        sum += __shfl_xor(sum, 2, kWave);
        if (part == 0) a.bal_partial[(size_t)blockIdx.x * kMaxExperts + e] = sum;
    }
}

}  // namespace moepp
