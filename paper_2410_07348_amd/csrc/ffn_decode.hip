// Grouped SwiGLU FFN for calls with a handful of rows per expert (decoding,
// small batches): the FFN experts of the layer (paper Eq.2) reduce to streaming
// every selected expert's weights past at most a few 16-row blocks of tokens.
//
//   GEMM1: h[r,f]    = silu(W1_e[f,:] . x_r) * (W3_e[f,:] . x_r),  x_r = x[src_of[r] / k]
//   GEMM2: yffn[r,d] = W2_e[d,:] . h[r,:]
//
// The kernel is bound by the weight stream (2.2 GB at the T = 64 workload
// against a few MB of activations), so it is built around that stream:
//  * an expert without rows is never touched: zero-computation slots and
//    unselected experts remove whole weight reads here (paper Sec. 3.4);
//  * work unit = (expert, block of 16 of its rows, panel of 256 packed weight
//    rows); the units of all experts form one list in that order, every eight (or
//    sixteen) neighbouring workgroups take a consecutive piece of it and each of
//    them works on 32 (16) rows of the panel, so a workgroup stays with
//    one expert (and one set of token operands) as long as it can, and what they
//    read at about the same time is consecutive memory;
//  * the eight waves of a workgroup split the reduction over K: wave w owns K
//    steps [S w, S (w + 1)) of 32 and keeps its slice of the (at most 16) token
//    rows in registers as MFMA operands for as long as the row block stays the
//    same; per step it multiplies two (one) 16-row weight fragments with them
//    (v_mfma_f32_16x16x32_bf16, 16 token rows is all the matrix core needs);
//  * the packed weight layout (panels of 256 rows, slabs of 32 columns) makes a
//    16-row x 32-column fragment 1 KB of consecutive memory: every load is a
//    whole-line, wave-wide load, 16 KB per wave in flight (a ring of steps that runs
//    on across unit boundaries, so the stream does not stop while the partial sums of a
//    unit meet), with the non-temporal hint: every weight is read once;
//  * the eight partial sums of a unit meet in LDS (two buffers, one barrier per
//    unit) and are added in wave order by all threads (the same on every
//    run), which apply SwiGLU and store.
// For a few tokens a kernel whose workgroups own columns of the output takes GEMM2 and the combine together (below).
// Rows past the end of a row block are clamped on load and masked on store.
#include "common.h"

#include <math.h>

#include <type_traits>

namespace moepp {

struct DecodeArgs {
    const bf16_t *A;         // GEMM1: x [T, ld] row-major; GEMM2: h, K-slab-major over h_rows rows
    const bf16_t *B;         // [n_ffn] matrices [Nb, K] in panels of K slabs (panel_row)
    bf16_t *C;               // GEMM1: h, K-slab-major over h_rows rows; GEMM2: yffn [R, ld] row-major
    const int32_t *offsets;  // [n_ffn + 1]
    const int32_t *src_of;   // GEMM1 only
    int ld, h_rows, K, Nb, n_ffn, topk;
};

constexpr int kDecWaves = 8;
constexpr int kDecThreads = kDecWaves * kWave;
constexpr int kDecMaxSteps = 24;               // K steps per wave at most: K <= 8 * 24 * 32 = 6144

__device__ inline float decode_silu(float z) {
    return z * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.44269504088896340736f * z));
}

// S: K steps per wave (K = 256 S).  A unit takes S4 = S rounded up to a multiple
// of the ring depth positions of the stream; the positions S .. S4 - 1 are empty
// (no load, no MFMA), which keeps the ring slot of every step a compile-time
// constant across unit boundaries.  The loop over the units of one row block is
// free of branches around loads, so the compiler's wait counts stay exact
// (after a join of paths with different loads in flight it waits for all of them).
// FR: 16-row weight fragments of a workgroup's share of a panel (2 or, GEMM2 only, 1);
// 16 / FR neighbouring workgroups share a panel and 16 / FR steps are in flight per wave.
template <bool SWIGLU, int S, int FR>
__global__ __launch_bounds__(kDecThreads, 1) void k_ffn_decode(DecodeArgs a) {
    constexpr int kDecRing = 16 / FR;             // K steps of weights in flight per wave: 16 KB
    constexpr int PARTS = 16 / FR;                // workgroups that share a panel
    constexpr int S4 = (S + kDecRing - 1) / kDecRing * kDecRing;
    static_assert(S >= 1 && S <= kDecMaxSteps && (FR == 2 || (FR == 1 && !SWIGLU)), "steps per wave, fragments");
    __shared__ __attribute__((aligned(16))) float part[2][kDecWaves][FR][kWave][4];   // FR * 16 KB
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int l16 = lane % 16, lq = lane / 16;
    const int ppe = a.Nb / kPanel;                 // panels of 256 packed weight rows per expert (Nb % 256 == 0)
    // PARTS neighbouring workgroups share a list of (expert, row block, panel) and each takes its
    // fragments of the panel: what they read at about the same time is the 16 KB of consecutive
    // memory of one K slab of the panel, not pieces from all over the weights.
    const int sub = blockIdx.x % PARTS, set = blockIdx.x / PARTS, n_sets = gridDim.x / PARTS;
    // row, within the panel, of fragment b: for GEMM1 blocks of 32 rows of W1 and 32 of W3, of
    // which two fragments are 16 rows of one and the same 16 of the other
    auto frag_row = [&](int b) {
        if constexpr (SWIGLU) return (sub / 2) * 64 + (sub % 2) * 16 + b * 32;
        else return (sub * FR + b) * 16;
    };

    // ---- the unit list: lane q looks after expert q --------------------------
    const int eq = lane < a.n_ffn ? lane : a.n_ffn;
    const int o_lo = a.offsets[eq];
    const int o_hi = a.offsets[eq < a.n_ffn ? eq + 1 : eq];
    const int units_q = ((o_hi - o_lo + 15) / 16) * ppe;      // 0 for an expert without rows
    const int incl = wave_prefix_sum(units_q);
    const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
    const int u0 = (int)((long long)total * set / n_sets);
    const int u1 = (int)((long long)total * (set + 1) / n_sets);
    if (u0 >= u1) return;

    // unit u -> expert, first row of its row block, rows in it, panel
    struct Unit {
        int e, row0, nrows, panel;
    };
    auto locate = [&](int u) {
        const unsigned long long past = __ballot(incl > u);
        Unit r;
        r.e = __builtin_ctzll(past);
        const int local = u - __builtin_amdgcn_readlane(incl - units_q, r.e);
        const int lo = __builtin_amdgcn_readlane(o_lo, r.e), hi = __builtin_amdgcn_readlane(o_hi, r.e);
        const int rb = local / ppe;                            // row blocks outermost: the token operands stay
        r.panel = local - rb * ppe;
        r.row0 = lo + 16 * rb;
        r.nrows = hi - r.row0 < 16 ? hi - r.row0 : 16;
        return r;
    };

    // ---- weight fragments: a ring of kDecRing steps -----------------------------
    // fragment (unit, step s, block b): 16 rows x 32 columns = 1 KB; lane l holds row l % 16,
    // columns 8 (l / 16) .. + 7
    bf16x8 wf[kDecRing][FR];
    // (real: false for a unit that does not exist)
    auto load_weights = [&](const Unit &un, int s, bf16x8 *dst, bool real = true) {
        const size_t at = (size_t)un.e * a.Nb * a.K + (size_t)un.panel * kPanel * a.K +
                          (size_t)(wave * S + s) * kPanel * kSlab;
        const size_t off = real ? at : 0;
        const char *p = reinterpret_cast<const char *>(a.B + off) + l16 * 64 + lq * 16;
#pragma unroll
        for (int b = 0; b < FR; ++b)
            dst[b] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8 *>(p + frag_row(b) * (kSlab * 2)));
    };

    // ---- token operands of this wave's K slice -----------------------------------
    bf16x8 af[S];
    auto load_tokens = [&](const Unit &un) {
        int row = un.row0 + l16;
        const int last = un.row0 + un.nrows - 1;
        row = row < last ? row : last;
        const char *p;
        size_t step;
        if constexpr (SWIGLU) {
            const int tok = a.src_of[row] / a.topk;
            p = reinterpret_cast<const char *>(a.A + (size_t)tok * a.ld + (size_t)wave * S * 32) + lq * 16;
            step = 64;
        } else {
            p = reinterpret_cast<const char *>(a.A + (size_t)wave * S * a.h_rows * kSlab + (size_t)row * kSlab) + lq * 16;
            step = (size_t)a.h_rows * kSlab * 2;
        }
#pragma unroll
        for (int s = 0; s < S; ++s) af[s] = *reinterpret_cast<const bf16x8 *>(p + s * step);
    };

    f32x4 acc[FR];
    auto clear_acc = [&]() {
#pragma unroll
        for (int b = 0; b < FR; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    };

    // ---- a finished unit: partial sums -> LDS -> all threads add, finish, store -----
    auto finish_unit = [&](const Unit &un, int buf) {
#pragma unroll
        for (int b = 0; b < FR; ++b) *reinterpret_cast<f32x4 *>(part[buf][wave][b][lane]) = acc[b];
        lds_barrier();         // orders LDS only: the weight loads of the next unit stay in flight
        // thread -> (block, lane of the accumulator layout, half of its four values)
        const int b = tid / 128, pl = (tid % 128) / 2, vh = tid % 2;
        const int m = pl % 16, n = 4 * (pl / 16) + 2 * vh;     // token row of the block, weight row of the 16
        const int row = un.row0 + m;
        typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
        if constexpr (SWIGLU) {
            // the first half of the blocks: rows of W1; the second: the same columns f of W3
            constexpr int H = FR / 2;
            if (b < H) {
                float z0 = 0.f, z1 = 0.f, g0 = 0.f, g1 = 0.f;
#pragma unroll
                for (int w = 0; w < kDecWaves; ++w) {          // wave order: the same on every run
                    z0 += part[buf][w][b][pl][2 * vh];
                    z1 += part[buf][w][b][pl][2 * vh + 1];
                    g0 += part[buf][w][b + H][pl][2 * vh];
                    g1 += part[buf][w][b + H][pl][2 * vh + 1];
                }
                if (m < un.nrows) {
                    bf16x2 o;
                    o[0] = (bf16_t)(decode_silu(z0) * g0);
                    o[1] = (bf16_t)(decode_silu(z1) * g1);
                    // row r of W1 in the panel's 64-row block q is column 32 q + r % 32 of h, slab 4 panel + q
                    const int r = frag_row(b);
                    *reinterpret_cast<bf16x2 *>(a.C + (size_t)(4 * un.panel + r / 64) * a.h_rows * kSlab +
                                                (size_t)row * kSlab + r % 64 + n) = o;
                }
            }
        } else if (b < FR) {
            float y0 = 0.f, y1 = 0.f;
#pragma unroll
            for (int w = 0; w < kDecWaves; ++w) {
                y0 += part[buf][w][b][pl][2 * vh];
                y1 += part[buf][w][b][pl][2 * vh + 1];
            }
            if (m < un.nrows) {
                bf16x2 o;
                o[0] = (bf16_t)y0;
                o[1] = (bf16_t)y1;
                *reinterpret_cast<bf16x2 *>(a.C + (size_t)row * a.ld + kPanel * un.panel + frag_row(b) + n) = o;
            }
        }
    };

    // ---- the stream: unit after unit, S4 positions each --------------------------
    // While position s of a unit is multiplied, position s + kDecRing of the stream is loaded into the ring
    // slot that s just left: of this unit, or of the next one, also where that has other token rows.  Past
    // the last unit every load takes the first line of the weights, which the caches hold: the last unit's
    // own first steps, once more, were 33 MB from memory at the end of either GEMM (T = 16, D = 4096 GEMM2
    // 106 -> 101 us; T = 8, D = 1536 29 -> 24; T = 64, D = 768, 32 experts 25.5 -> 19.5, where most
    // workgroups have three units).
    int buf = 0;
    int u = u0;
    Unit cur = locate(u);
#pragma unroll
    for (int r = 0; r < kDecRing; ++r)
        if (r < S) load_weights(cur, r, wf[r]);
    while (u < u1) {
        const int seg_end = min(u1, u + (ppe - cur.panel));    // units that share cur's token operands
        load_tokens(cur);
        for (; u < seg_end; ++u) {
            const bool more = u + 1 < u1;
            const Unit nxt = locate(u + 1 < u1 ? u + 1 : u1 - 1);
            clear_acc();
#pragma unroll
            for (int s = 0; s < S4; ++s) {
                if (s < S) {
#pragma unroll
                    for (int b = 0; b < FR; ++b)
                        acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s % kDecRing][b], af[s], acc[b], 0, 0, 0);
                }
                const int pos = s + kDecRing;              // compile-time after unrolling
                if (pos < S4) {
                    if (pos < S) load_weights(cur, pos, wf[s % kDecRing]);
                } else if (pos - S4 < S) {
                    load_weights(nxt, pos - S4, wf[s % kDecRing], more);
                }
                // (left alone, the compiler moves a load down to its first use, a ring later)
                __builtin_amdgcn_sched_barrier(0);
            }
            finish_unit(cur, buf);
            buf ^= 1;
            cur = nxt;
        }
    }
}

// GEMM2 and the combine (combine.hip, the same operations in the same order) in one kernel, for at most
// kDecOutT tokens: a workgroup owns 16 columns of the output and takes them through all row blocks of all
// experts, so that nobody waits for another workgroup.  Weights and the token rows of h travel in one ring
// of 16 steps (h comes from the caches, 16 rows for every 16 of weights), so nothing drains it between row
// blocks.  Waves split K; sums and yffn are those of the kernel above, bit by bit.  The code runs once and
// waits for its instructions: one row block at a time (several in a pass of the ring, where K is short, put
// more loads in flight and took 8.5 us for one token at D = 768 where this takes 7.3).
struct DecodeOutArgs {
    DecodeArgs g;
    CombineArgs c;
};
constexpr int kDecOutT = 48, kDecOutSlots = kDecOutT * kMaxTopK;
template <int S>
__global__ __launch_bounds__(kDecThreads, 1) void k_ffn_decode_combine(DecodeOutArgs oa) {
    constexpr int RING = 16, S4 = (S + RING - 1) / RING * RING;
    const DecodeArgs &a = oa.g;
    const CombineArgs &c = oa.c;
    __shared__ __attribute__((aligned(16))) float part[2][kDecWaves][kWave][4];
    __shared__ __attribute__((aligned(16))) bf16_t y[kDecOutSlots][16];      // yffn's 16 columns
    __shared__ int s_idx[kDecOutSlots], s_row[kDecOutSlots];
    __shared__ float s_w[kDecOutSlots], s_a1[kDecOutT * kMaxConst];
    __shared__ __attribute__((aligned(16))) bf16_t s_cv[kMaxConst][16];
    static_assert(kDecOutSlots <= kDecThreads && kDecOutT * kMaxConst <= kDecThreads && 2 * kDecOutT <= kDecThreads, "one pass each");
    const int tid = threadIdx.x, lane = tid % kWave, l16 = lane % 16, lq = lane / 16;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int c0 = blockIdx.x * 16, panel = c0 / kPanel;

    // ---- row blocks: lane q looks after expert q
    const int eq = lane < a.n_ffn ? lane : a.n_ffn;
    const int o_lo = a.offsets[eq], o_hi = a.offsets[eq < a.n_ffn ? eq + 1 : eq];
    const int blocks_q = (o_hi - o_lo + 15) / 16, incl = wave_prefix_sum(blocks_q);
    const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
    struct Block {
        int e, row0, nrows;                        // nrows 0: no such block
    };
    auto locate = [&](int b) {
        Block r = {0, 0, 0};
        if (b < total) {
            r.e = __builtin_ctzll(__ballot(incl > b));
            const int lo = __builtin_amdgcn_readlane(o_lo, r.e), hi = __builtin_amdgcn_readlane(o_hi, r.e);
            r.row0 = lo + 16 * (b - __builtin_amdgcn_readlane(incl - blocks_q, r.e));
            r.nrows = hi - r.row0 < 16 ? hi - r.row0 : 16;
        }
        return r;
    };
    // step s of a block (of none: the first lines of the weights and of h)
    bf16x8 wf[RING], tf[RING];
    auto load = [&](const Block &b, int s) {
        const size_t at = b.nrows ? (size_t)b.e * a.Nb * a.K + (size_t)panel * kPanel * a.K +
                                        (size_t)(wave * S + s) * kPanel * kSlab + c0 % kPanel * kSlab : 0;
        wf[s % RING] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8 *>(a.B + at + l16 * kSlab + lq * 8));
        const int last = b.nrows ? b.row0 + b.nrows - 1 : 0, row = b.row0 + l16 < last ? b.row0 + l16 : last;
        tf[s % RING] = *reinterpret_cast<const bf16x8 *>(a.A + (size_t)(wave * S + s) * a.h_rows * kSlab + (size_t)row * kSlab + lq * 8);
    };
    Block cur = locate(0);
#pragma unroll
    for (int s = 0; s < RING; ++s)
        if (s < S) load(cur, s);

    // what the combine wants, asked for behind the first weights
    const int T = c.d.T, D = c.d.D, K = c.d.k, nc = c.d.n_const;
    const int q = min(tid, T * K - 1), item = min(tid, 2 * T - 1), cv = min(tid, 2 * nc - 1);
    const int idx = c.topk_idx[q], row_q = c.row_of[q];
    const float w_q = c.topk_w[q];
    const size_t out_at = (size_t)(item / 2) * D + c0 + item % 2 * 8;        // this thread's eight columns of a token
    const bf16x8 xv = *reinterpret_cast<const bf16x8 *>((const bf16_t *)c.x + out_at);
    float a1 = 0.f;
    bf16x8 cvv = {};
    if (nc > 0) {
        a1 = c.alpha1[min(tid, T * nc - 1)];
        cvv = *reinterpret_cast<const bf16x8 *>((const bf16_t *)c.const_vecs + (size_t)(cv / 2) * D + c0 + cv % 2 * 8);
    }

    for (int b = 0; b < total; ++b) {
        const Block nxt = locate(b + 1);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < S4; ++s) {
            if (s < S) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s % RING], tf[s % RING], acc, 0, 0, 0);
            const int pos = s + RING;
            if (pos < S4) {
                if (pos < S) load(cur, pos);
            } else if (pos - S4 < S) {
                load(nxt, pos - S4);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        const int buf = b & 1, pl = tid / 2, vh = tid % 2, m = pl % 16, n = 4 * (pl / 16) + 2 * vh;
        *reinterpret_cast<f32x4 *>(part[buf][wave][lane]) = acc;
        lds_barrier();
        if (tid < 128 && m < cur.nrows) {
            float y0 = 0.f, y1 = 0.f;
#pragma unroll
            for (int w = 0; w < kDecWaves; ++w) {
                y0 += part[buf][w][pl][2 * vh];
                y1 += part[buf][w][pl][2 * vh + 1];
            }
            typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
            bf16x2 o;
            o[0] = (bf16_t)y0;
            o[1] = (bf16_t)y1;
            *reinterpret_cast<bf16x2 *>(&y[cur.row0 + m][n]) = o;
            *reinterpret_cast<bf16x2 *>(a.C + (size_t)(cur.row0 + m) * a.ld + c0 + n) = o;
        }
        cur = nxt;
    }
    if (tid < T * K) {
        s_idx[tid] = idx;
        s_row[tid] = row_q;
        s_w[tid] = w_q;
    }
    if (tid < T * nc) s_a1[tid] = a1;
    if (tid < 2 * nc) *reinterpret_cast<bf16x8 *>(&s_cv[tid / 2][tid % 2 * 8]) = cvv;
    __syncthreads();

    // ---- the combine of this workgroup's columns
    if (tid >= 2 * T) return;
    const int t = tid / 2, h8 = tid % 2 * 8, zero0 = c.d.n_ffn, copy0 = zero0 + c.d.n_zero, const0 = copy0 + c.d.n_copy;
    float sum[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) sum[i] = 0.f;
    for (int s = 0; s < K; ++s) {
        const int e = s_idx[t * K + s], row = s_row[t * K + s];
        const float g = s_w[t * K + s];
        if (row == -2) continue;                               // over the expert's capacity: dropped
        if (e < zero0) {
            const bf16x8 v = *reinterpret_cast<const bf16x8 *>(&y[row][h8]);
#pragma unroll
            for (int i = 0; i < 8; ++i) sum[i] = fmaf(g, (float)v[i], sum[i]);
        } else if (e >= const0) {
            const float al = s_a1[t * nc + e - const0], g_x = g * al, g_v = g * (1.f - al);
            const bf16x8 v = *reinterpret_cast<const bf16x8 *>(&s_cv[e - const0][h8]);
#pragma unroll
            for (int i = 0; i < 8; ++i) sum[i] += g_x * (float)xv[i] + g_v * (float)v[i];
        } else if (e >= copy0 && g != 0.f) {
#pragma unroll
            for (int i = 0; i < 8; ++i) sum[i] = fmaf(g, (float)xv[i], sum[i]);
        }
    }
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (bf16_t)sum[i];
    __builtin_nontemporal_store(o, reinterpret_cast<bf16x8 *>((bf16_t *)c.out + out_at));
}

template <int SMAX>
static hipError_t dispatch_out(int S, const DecodeOutArgs &a, hipStream_t s) {
    if constexpr (SMAX < 1) {
        return hipErrorInvalidValue;
    } else {
        if (S != SMAX) return dispatch_out<SMAX - 1>(S, a, s);
        hipLaunchKernelGGL((k_ffn_decode_combine<SMAX>), dim3(a.c.d.D / 16), dim3(kDecThreads), 0, s, a);
        return hipGetLastError();
    }
}

// launch k_ffn_decode<., S, FR> for the run-time S
template <int SMAX>
static hipError_t dispatch_steps(int S, int which, int fr, int n_wg, const DecodeArgs &a, hipStream_t s) {
    if constexpr (SMAX < 1) {
        return hipErrorInvalidValue;
    } else {
        if (S != SMAX) return dispatch_steps<SMAX - 1>(S, which, fr, n_wg, a, s);
        const dim3 grid(n_wg), block(kDecThreads);
        if (which == 0) hipLaunchKernelGGL((k_ffn_decode<true, SMAX, 2>), grid, block, 0, s, a);
        else if (fr == 2) hipLaunchKernelGGL((k_ffn_decode<false, SMAX, 2>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_ffn_decode<false, SMAX, 1>), grid, block, 0, s, a);
        return hipGetLastError();
    }
}

// An expert with more than 16 rows streams its weights once per block of 16, and the tiled kernel,
// which reads them once for up to 128 rows, is faster once most experts do.  But few experts leave
// the tiled kernel a part-filled chip, and weights that the caches hold are cheap to read again.  So
// the limit is a number of rows per expert (if the router spreads its slots evenly; never more
// slots than 16 per FFN expert), by the number of FFN experts and the bytes of their weights.  Top-2
// layer here / tiled, us, D x F:
//   16 rows: 2 experts, 4096 x 5632 81 / 105; 3 117 / 138; 12, 768 x 1024 (57 MB) 37.6 / 41.5
//   14 rows: 8, 1536 x 4096 (302 MB) 88 / 97; 10 109 / 123; 8, 4096 x 5632 (1.1 GB) 245 / 232
//   12 rows: 8, 4096 x 5632 212 / 226; 12, 1536 x 4096 114 / 131
//   10 rows: 16, 768 x 1024 (75 MB) 39 / 42; 24 49 / 53; 16, 1024 x 2048 (201 MB) 70 / 64
//    8 rows and more: 16, 1536 x 4096 134 / 128 at 9; 32, 768 x 2048 91 / 81 at 12
// (with more experts how the tiles fill their last round decides: 24, 1536 x 4096 at 9 191 / 201)
bool ffn_decode_supported(const Dims &d) {
    const long long slots = (long long)d.T * d.k;
    const double mb = 6e-6 * d.n_ffn * d.D * d.F;
    const int rows = d.n_ffn <= 3 || mb <= 64.0 ? 16 : d.n_ffn <= 12 ? (mb <= 400.0 ? 14 : 12) : mb <= 128.0 ? 10 : 8;
    return d.n_ffn > 0 && d.n_ffn <= kWave && slots <= 16ll * d.n_ffn && slots <= (long long)rows * d.N &&
           d.D % 256 == 0 && d.F % 256 == 0 && d.D <= kDecMaxSteps * 256 && d.F <= kDecMaxSteps * 256;
}

static DecodeArgs decode_args(const FfnArgs &f, int which) {
    DecodeArgs a;
    a.offsets = f.offsets;
    a.src_of = f.src_of;
    a.n_ffn = f.d.n_ffn;
    a.topk = f.d.k;
    a.h_rows = f.h_rows;
    a.ld = f.d.D;
    if (which == 0) {
        a.A = (const bf16_t *)f.x;
        a.B = (const bf16_t *)f.w13;
        a.C = (bf16_t *)f.h;
        a.K = f.d.D;
        a.Nb = 2 * f.d.F;
    } else {
        a.A = (const bf16_t *)f.h;
        a.B = (const bf16_t *)f.w2;
        a.C = (bf16_t *)f.yffn;
        a.K = f.d.F;
        a.Nb = f.d.D;
    }
    return a;
}

// CUs of the device, a multiple of the 16 workgroups that share a panel.
static int decode_cus() {
    static int n_cu = 0;
    if (n_cu == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 16)
            v = 256;
        n_cu = v / 16 * 16;
    }
    return n_cu;
}

// A CU of the kernel that combines, too, reads 32 KB of weights a us, all of them together 6.4 MB, and each
// row block costs every workgroup 0.14 us: where fewer than 200 workgroups (D < 3200) share the weights the
// stream takes longer, and with many row blocks so do their ends, which is worth it up to the 3.0 us that a launch and
// the combine cost.  The constants fit 1358 timings (D = 256 .. 4096, F = 256 .. 5632, 2 to 32 experts, T = 1 .. 48, cold
// and cached weights, calls one by one and in a graph): of 1560 us that the better choices would save they find 1407,
// the streams alone (27 KB, 6.1 MB and 3.2 us) 1342.  Layers, us, apart / together: D = 4096, F = 5632, 16 experts T = 1
// 65.8 / 62.1, T = 16 327 / 321, T = 45 368 / 367, T = 64 370 / 372 (the token rows are read by every workgroup); D = 768,
// F = 2048 three layers of T = 1 59.6 / 58.5, T = 2 65.0 / 68.9; D = 3072, F = 2048 T = 8 89.8 / 86.6; D = 2048, F = 2048 T =
// 2 94.2 / 90.8, T = 8 187 / 193; D = 512, F = 512, 8 experts T = 4 66.4 / 58.1; D = 1024, F = 256 T = 18 (14 row
// blocks) 20.6 / 23.8; D = 3072, F = 512, 32 experts T = 39 67.5 / 68.6.
// More workgroups than CUs (D > 4096) are a second round with most CUs idle: a CU has one of them from F = 2816 on
// (over 128 registers).  16 experts: D = 4352, F = 5632 T = 1 73.0 / 78.1, T = 16 298 / 336, T = 40 385 / 446; D = 5120,
// F = 5632 T = 16 377 / 404; D = 6144, F = 4352 T = 1 76.6 / 83.0; D = 4352, F = 1024 T = 16 72.9 / 78.4; D = 6144, F =
// 2048 T = 1 46.9 / 46.7, T = 4 68.5 / 70.5.  Up to F = 512 two share a CU and the launch they save is more: D =
// 6144, F = 512 T = 1 31.6 / 30.5, T = 16 59.9 / 58.1; D = 4352, F = 512 T = 4 30.9 / 29.7, but T = 16 47.6 / 49.0.
bool ffn_decode_combines(const Dims &d) {
    if (!ffn_decode_supported(d) || d.T > kDecOutT) return false;
    const double wgs = d.D / 16, cus = decode_cus(), cu_rate = 32e3, all_rate = 6.4e6;     // (bytes a us)
    if (wgs > cus && d.F > 512) return false;
    const double stream = wgs > cus ? cus / all_rate + 0.5 / cu_rate : 1.0 / cu_rate;      // us a byte of a workgroup
    const double longer = fmax(0.0, stream - wgs / all_rate);
    const double blocks = d.n_ffn * (1.0 - pow(1.0 - 1.0 / d.N, (double)d.T * d.k));     // experts with rows
    return blocks * (0.14 + 32.0 * d.F * longer) < 3.0;
}

hipError_t launch_ffn_decode_combine(const FfnArgs &f, const CombineArgs &c, hipStream_t s) {
    if (f.d.T == 0 || !ffn_decode_combines(f.d)) return hipErrorInvalidValue;
    const DecodeOutArgs a{decode_args(f, 1), c};
    return dispatch_out<kDecMaxSteps>(a.g.K / (32 * kDecWaves), a, s);
}

hipError_t launch_ffn_decode(const FfnArgs &f, int which, hipStream_t s) {
    if (f.d.T == 0 || f.d.n_ffn == 0) return hipSuccess;
    const DecodeArgs a = decode_args(f, which);
    const int n_cu = decode_cus();
    const long long slots = (long long)f.d.T * f.d.k;
    const long long experts = slots < f.d.n_ffn ? slots : f.d.n_ffn;
    // Two fragments (32 rows of weights) per workgroup and panel, where there were four: the work
    // divides more evenly.  T = 64, D = 4096: GEMM1 242 -> 231 us; 14 experts (T = 16) 212 + 115 ->
    // 208 + 107; one token 37.8 + 30.8 -> 36 + 21.7.  One fragment for GEMM2 when even that fills
    // less than half of the chip: one token, D = 768: 6.8 -> 5.2 us (10.4 with four).
    const int fr = which == 1 && experts * (a.Nb / 64) <= 128 ? 1 : 2;
    // one workgroup per CU; a workgroup without units returns at once
    const int S = a.K / (32 * kDecWaves);
    return dispatch_steps<kDecMaxSteps>(S, which, fr, n_cu, a, s);
}

}  // namespace moepp
