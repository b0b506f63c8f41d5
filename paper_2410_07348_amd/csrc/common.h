// Internal declarations shared by the HIP sources of libmoepp (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace moepp {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kMaxExperts = 64;   // N
constexpr int kMaxTopK = 8;       // K
constexpr int kMaxConst = 8;      // constant experts
constexpr int kWave = 64;         // CDNA wavefront

// Calls with at most this many tokens take the router on slices of D whose last kernel also does
// the permutation.
constexpr int kRouterFusedT = 64;

// Permutation: one wave owns a chunk of consecutive slots: kPermChunk of them,
// or the slots of one block of tokens of the router when that has counted
// them: 64 and more, or 16 or 32 (router_block_tokens), whose few hundred histogram rows are
// in the router's partial sums and need no chunk_base.
constexpr int kPermChunk = 4 * kWave;
constexpr int kPermMinChunkTokens = 64;      // of the chunks that chunk_hist and chunk_base have rows for
// Up to this many chunks every scatter wave adds up the histogram rows itself
// (work grows with the square of the chunk count); beyond it a scan kernel does.
constexpr int kPermDirectChunks = 2048;

// Rows of W1 and W3 are interleaved in blocks of this many rows in the packed
// expert buffer: [kPackBlk rows of W1][kPackBlk rows of W3] ...
constexpr int kPackBlk = 32;

// Row of the packed W1/W3 matrix [2F, D] that holds row f of W1 (up = 0) or
// of W3 (up = 1).  The last block may be partial when F % kPackBlk != 0.
__host__ __device__ inline int packed_row(int f, int up, int F) {
    int b = f / kPackBlk;
    int rem = F - b * kPackBlk;
    int bs = rem < kPackBlk ? rem : kPackBlk;
    return b * 2 * kPackBlk + up * bs + (f - b * kPackBlk);
}

// K-slab-major storage of a matrix [N rows, K columns]: slab s holds columns
// [s*kSlab, (s+1)*kSlab) of every row, rows consecutive, so that the part of
// the matrix a GEMM tile needs for one K step (some consecutive rows x one
// slab) is one consecutive piece of memory.  The last slab is narrower when
// K % kSlab != 0.  Used for h.
constexpr int kSlab = 32;
__host__ __device__ inline int slab_width(int s, int K) {
    const int rem = K - s * kSlab;
    return rem < kSlab ? rem : kSlab;
}
// element offset of (row n, first column of slab s)
__host__ __device__ inline size_t slab_row(int n, int s, int N, int K) {
    return (size_t)s * N * kSlab + (size_t)n * slab_width(s, K);
}

// The packed expert weight matrices [N rows, K columns] are stored in panels
// of kPanel rows (the GEMM's tile height), each panel K-slab-major: all that
// one GEMM tile reads of the matrix, in the order it reads it, is one
// consecutive run of memory.  The last panel has fewer rows when
// N % kPanel != 0.  Element offset of (row n, first column of slab s):
constexpr int kPanel = 256;
__host__ __device__ inline size_t panel_row(int n, int s, int N, int K) {
    const int p = n / kPanel;
    const int rem = N - p * kPanel;
    const int rows = rem < kPanel ? rem : kPanel;
    return (size_t)p * kPanel * K + slab_row(n - p * kPanel, s, rows, K);
}

// Logical row L of the packed W1/W3 matrix (SWIGLU) or of W2, as the tiled kernels
// number them: for W1/W3 blocks of 64, 32 rows of W1 and the same 32 of W3, also where
// the last block has fewer, so that silu's argument and its multiplier always sit
// 32 rows apart.  Returns the packed row; a row that does not exist gives row 0 (its
// output columns are never stored).
template <bool SWIGLU>
__device__ inline int packed_of_logical(int L, int Nb) {
    if constexpr (SWIGLU) {
        const int b = L / (2 * kPackBlk), up = L % (2 * kPackBlk) / kPackBlk, r = L % kPackBlk;
        const int rem = Nb / 2 - kPackBlk * b, bs = rem < kPackBlk ? rem : kPackBlk;
        return r < bs ? 2 * kPackBlk * b + up * bs + r : 0;
    } else {
        return L < Nb ? L : 0;
    }
}

struct Dims {
    int T, D, F;
    int n_ffn, n_zero, n_copy, n_const, N;
    int k;
};

// Device pointers into the caller's workspace.
struct Workspace {
    int32_t *topk_idx;   // [T_max*k]
    float *topk_w;       // [T_max*k]
    float *alpha1;       // [T_max*n_const]
    int32_t *counts;     // [N] assignments per expert, before any drop
    int32_t *kept;       // [N] min(counts, capacity)
    int32_t *offsets;    // [n_ffn+1]
    int32_t *row_of;     // [T_max*k]
    int32_t *src_of;     // [T_max*k]
    int32_t *chunk_hist; // [n_chunks*N]
    int32_t *chunk_base; // [n_chunks*N]
    void *h;             // [T_max*k, F] act, K-slab-major
    void *yffn;          // [T_max*k, D] act
    double *bal_partial; // [kBalWaves][kMaxExperts] partial sums of Softmax(G(x))
    float *bal;          // f [N], P [N], L_b [1]  (Eq.7)
    float *router_partial; // router_small_bytes(): per-slice dot products of the routers that split D
};

// Expert capacities (Eq.8), by value in the kernel arguments.  on = false: unlimited.
struct CapArgs {
    bool on;
    int32_t cap[kMaxExperts];
};

constexpr int kBalWaves = 2048;   // waves of the load-balance reduction (its partial sums)

struct RouterArgs {
    Dims d;
    const void *x;
    const float *prev_gate, *W_g, *W_res, *bias, *W_c;
    float *out_gate;
    int32_t *topk_idx;
    float *topk_w;
    float *alpha1;
    int32_t *chunk_hist;  // [block of tokens][N] selections per expert, or null
    float *partial;       // router_small_bytes() of scratch for partial dot products
    double *bal_partial;  // [block of tokens][kMaxExperts] sums of Softmax(G(x))_i over the
                          // block's tokens (for P_i of Eq.7), or null
};

struct FfnArgs {
    Dims d;
    const void *x;        // [T,D]
    const void *w13;      // packed: [n_ffn] matrices [2F, D] in panels (panel_row), rows in packed_row order
    const void *w2;       // packed: [n_ffn] matrices [D, F] in panels (panel_row)
    const int32_t *offsets;
    const int32_t *src_of;
    void *h;              // [h_rows, F] K-slab-major; rows < R are written
    void *yffn;           // [R,D] row-major
    int h_rows;           // T_max * k
    bool no_tail;         // tests (variant 3): one tile geometry, no half tiles, cached weights
};

struct CombineArgs {
    Dims d;
    const void *x, *const_vecs, *yffn;
    const int32_t *topk_idx, *row_of;
    const float *topk_w, *alpha1;
    void *out;
};

// Launchers (each returns hipGetLastError() after its launches).
// `bf16` selects the activation type; `which` selects GEMM1 / GEMM2.
hipError_t launch_router_generic(const RouterArgs &a, bool bf16, hipStream_t s);
// T <= kRouterFusedT only.  The second kernel also does the permutation of the call's T*k
// slots (counts, kept, offsets, row_of, src_of of perm_ws, capacities perm_cap), as
// launch_perm_small would.
hipError_t launch_router_small(const RouterArgs &a, bool bf16, hipStream_t s, const Workspace &perm_ws,
                               const CapArgs &perm_cap);
// More tokens, any width and type, while router_split_max(d) >= 1; leaves the histogram of
// the permutation (chunks of kRouterSlicedTok tokens) and the statistics' sums like the
// matrix-core router.
constexpr int kRouterSlicedTok = 64;
bool router_sliced_wins(const Dims &d);
hipError_t launch_router_sliced(const RouterArgs &a, bool bf16, hipStream_t s);
// One kernel on blocks of 16 or 32 tokens, where it is faster and as exact; leaves the same, its histogram in blocks of
// that many tokens (more rows than the workspace's table has: those are in RouterArgs::partial, which this router does
// not use).
int router_block_tokens(const Dims &d, bool bf16);
hipError_t launch_router_block(const RouterArgs &a, bool bf16, hipStream_t s);
size_t router_small_bytes();
// Slices of D whose partial logits [slice][T][N + 2 n_const] fit RouterArgs::partial, at most
// kRouterSplits (a thread that adds them up holds four floats of each)
constexpr int kRouterSplits = 24;
int router_split_max(const Dims &d);
bool router_mfma_supported(const Dims &d);
hipError_t launch_router_mfma(const RouterArgs &a, hipStream_t s);
int router_mfma_block_tokens(const Dims &d);

// chunk_slots: slots per chunk (kPermChunk, or tokens per router workgroup x k)
int perm_chunks(const Dims &d, int chunk_slots);
hipError_t launch_perm_hist(const Dims &d, const Workspace &w, int chunk_slots, hipStream_t s);
hipError_t launch_perm_scan(const Dims &d, const Workspace &w, const CapArgs &cap, int chunk_slots,
                            hipStream_t s);
hipError_t launch_perm_scatter(const Dims &d, const Workspace &w, const CapArgs &cap, int chunk_slots,
                               hipStream_t s);
// scan + scatter in one kernel; at most kPermDirectChunks chunks
hipError_t launch_perm_scan_scatter(const Dims &d, const Workspace &w, const CapArgs &cap, int chunk_slots,
                                    hipStream_t s);
// all three steps in one workgroup, for 0 < T*k <= kPermSmallSlots
constexpr int kPermSmallWaves = 16;
constexpr int kPermSmallSlots = kPermSmallWaves * kPermChunk;
hipError_t launch_perm_small(const Dims &d, const Workspace &w, const CapArgs &cap, hipStream_t s);
// f_i, P_i and L_b of Eq.7 from the logits of the routed call and the counts of the permutation.
// router_rows > 0: the router kernel has already left that many rows of per-workgroup sums of
// Softmax(G(x)) in w.bal_partial (at most kBalWaves), and only the final reduction runs.
hipError_t launch_balance(const Dims &d, const Workspace &w, const float *out_gate, float tau,
                          hipStream_t s, int router_rows = 0);

// float32 layers, any supported shape: matrix cores, float32 products and sums
hipError_t launch_ffn_f32(const FfnArgs &a, int which, hipStream_t s);

hipError_t launch_ffn_generic(const FfnArgs &a, bool bf16, int which, hipStream_t s);
bool ffn_mfma_supported(const Dims &d);
hipError_t launch_ffn_mfma(const FfnArgs &a, int which, hipStream_t s);

// few rows per expert (at most 16, by a rule on experts and weights): weight-streaming kernels
bool ffn_decode_supported(const Dims &d);
hipError_t launch_ffn_decode(const FfnArgs &a, int which, hipStream_t s);
// GEMM2 and the combine in one kernel, where that is faster; leaves yffn and `out` as the two would
bool ffn_decode_combines(const Dims &d);
struct CombineArgs;
hipError_t launch_ffn_decode_combine(const FfnArgs &f, const CombineArgs &c, hipStream_t s);

hipError_t launch_combine(const CombineArgs &a, bool bf16, hipStream_t s);

hipError_t launch_pack(const Dims &d, bool bf16, const void *w1, const void *w3,
                       const void *w2, void *w13_out, void *w2_out, hipStream_t s);

hipError_t launch_mfma_ceiling(float *scratch, int iters, hipStream_t s);
double mfma_ceiling_flops(int iters);
size_t mfma_ceiling_scratch_bytes();
hipError_t launch_stream(void *buf, size_t bytes, int mode, hipStream_t s);

// ---- small device helpers -------------------------------------------------
// Workgroup barrier that orders LDS accesses only: global loads (including
// loads that write LDS directly, which the caller waits for with vmcnt) stay
// in flight across it, unlike __syncthreads().
__device__ inline void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Lane l of a wave: the sum over lanes 0 .. l.  Moves between lanes inside the vector ALU (rows of
// 16 lanes shifted, then the ends of the rows broadcast), a few cycles each; a shuffle goes through the
// LDS hardware, some 130 cycles, and the next one waits for it.
__device__ inline int wave_prefix_sum(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);    // from lane - 1 of the row
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);    // - 2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);    // - 4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);    // - 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);    // lane 15 of the row before, rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);    // lane 31, rows 2 and 3
    return v;
}

// The largest value and the sum of L = 4, 8 or 16 neighbouring lanes, in each of them (the same bits
// in all: every move pairs the same values in either order): lanes ^ 1 and ^ 2 of four, then the mirrored half
// row of eight, then the row of sixteen turned by eight.
template <int CTRL>
__device__ inline float lane_move(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int L>
__device__ inline float lanes_max(float v) {
    v = fmaxf(v, lane_move<0xB1>(v));
    v = fmaxf(v, lane_move<0x4E>(v));
    if constexpr (L >= 8) v = fmaxf(v, lane_move<0x141>(v));
    if constexpr (L >= 16) v = fmaxf(v, lane_move<0x128>(v));
    return v;
}
template <int L>
__device__ inline float lanes_sum(float v) {
    v += lane_move<0xB1>(v);
    v += lane_move<0x4E>(v);
    if constexpr (L >= 8) v += lane_move<0x141>(v);
    if constexpr (L >= 16) v += lane_move<0x128>(v);
    return v;
}

// Three bf16 pieces of four floats, w = hi + mid + lo: hi is w cut off after 8 significand bits (so that no
// finite w overflows), mid the rest rounded to 8 bits, lo what is left, at most 8 bits.  bf16 has none of the
// bits of a float32 below 2^-133: `lost` collects the words that lo is cut from, whose lower halves are zero
// unless a w was too small for its pieces.  (w infinite or NaN: mid and lo are NaN, hi may be infinite for either.)
// NOW: collected with the split; the compiler by itself keeps the words for later, which costs registers (routers
// on slices 114 -> 132, two workgroups per CU -> one).
typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
struct Split4 {
    u32x2 hi, mid, lo;
};
template <bool NOW = true>
__device__ inline Split4 split4(f32x4 w, uint32_t &lost) {
    constexpr uint32_t UPPER = 0x07060302;                            // the upper halves of two words
    Split4 s;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t a = __float_as_uint(w[2 * i]), b = __float_as_uint(w[2 * i + 1]);
        s.hi[i] = __builtin_amdgcn_perm(b, a, UPPER);
        const float ra = w[2 * i] - __uint_as_float(a & 0xffff0000u);
        const float rb = w[2 * i + 1] - __uint_as_float(b & 0xffff0000u);
        bf16x2 m;
        m[0] = (bf16_t)ra;
        m[1] = (bf16_t)rb;
        s.mid[i] = __builtin_bit_cast(uint32_t, m);
        const uint32_t la = __float_as_uint(ra - __uint_as_float(s.mid[i] << 16));
        const uint32_t lb = __float_as_uint(rb - __uint_as_float(s.mid[i] & 0xffff0000u));
        s.lo[i] = __builtin_amdgcn_perm(lb, la, UPPER);
        if constexpr (NOW) asm("v_or3_b32 %0, %1, %2, %0" : "+v"(lost) : "v"(la), "v"(lb));
        else lost |= la | lb;
    }
    return s;
}
__device__ inline bool split_lost(uint32_t lost) { return (lost & 0xffffu) != 0; }

__device__ inline float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}
__device__ inline float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
    return v;
}

__device__ inline float silu_f(float z) { return z / (1.f + expf(-z)); }

// The same function for |z| <= kSiluNear (and NaN) in two thirds of the instructions: nothing overflows
// there.  e^-z = 2^n 2^f by the reduction of Cody and Waite (Software Manual for the Elementary Functions,
// 1980): log2 e in two floats, the product's rounding error by an FMA (Dekker, 1971), the addition that rounds to
// n leaves it in its low bits, from where it goes straight into the exponent.  The quotient is a reciprocal and one
// correction by its residual (Markstein, 1990); the residual is taken as -(q d - z), so that zero keeps its sign.
// Over all 2.24e9 floats of |z| <= 87 the error against float64 is 3.1 x 2^-24 at most, like that of silu_f, and
// 15 results differ from silu_f's (f a rounding apart), by one or two ulps.  No contraction: f counts on t as rounded.
constexpr float kSiluNear = 87.f;            // e^87 < 2^126: the reciprocal is a normal number
__device__ inline float silu_near(float z) {
#pragma clang fp contract(off)
    constexpr double log2e = 1.44269504088896340736;
    constexpr float hi = (float)log2e, lo = (float)(log2e - (double)hi), whole = 12582912.f;   // 1.5 * 2^23
    const float t = -z * hi, m = t + whole, n = m - whole;
    const float f = (t - n) + fmaf(-z, lo, fmaf(-z, hi, -t));
    const float p = __uint_as_float((__float_as_uint(m) << 23) + __float_as_uint(__builtin_amdgcn_exp2f(f)));
    const float d = 1.f + p, inv = __builtin_amdgcn_rcpf(d), q = z * inv;
    return fmaf(-fmaf(q, d, -z), inv, q);
}
// By element, so that no row's bits depend on another's.
__device__ inline float silu_both(float z) { return fabsf(z) <= kSiluNear ? silu_near(z) : silu_f(z); }

__device__ inline float to_f32(float v) { return v; }
__device__ inline float to_f32(bf16_t v) { return (float)v; }

template <typename T> struct ActVec;   // 16 bytes of activations
template <> struct ActVec<float> {
    static constexpr int N = 4;
    f32x4 v;
    __device__ float get(int i) const { return v[i]; }
    __device__ void set(int i, float f) { v[i] = f; }
};
template <> struct ActVec<bf16_t> {
    static constexpr int N = 8;
    bf16x8 v;
    __device__ float get(int i) const { return (float)v[i]; }
    __device__ void set(int i, float f) { v[i] = (bf16_t)f; }
};

template <typename T>
__device__ inline ActVec<T> load_vec(const T *p) {
    ActVec<T> r;
    r.v = *reinterpret_cast<const decltype(r.v) *>(p);
    return r;
}
template <typename T>
__device__ inline void store_vec(T *p, const ActVec<T> &r) {
    *reinterpret_cast<decltype(r.v) *>(p) = r.v;
}
// The same with the non-temporal hint, for data this library does not touch
// again (a layer's output) or reads exactly once (a row of the FFN output):
// such lines then do not displace, or sit dirty in, the caches that the
// following kernels read through (measured: the router that follows a combine
// runs 20 % faster).
template <typename T>
__device__ inline ActVec<T> load_vec_stream(const T *p) {
    ActVec<T> r;
    r.v = __builtin_nontemporal_load(reinterpret_cast<const decltype(r.v) *>(p));
    return r;
}
template <typename T>
__device__ inline void store_vec_stream(T *p, const ActVec<T> &r) {
    __builtin_nontemporal_store(r.v, reinterpret_cast<decltype(r.v) *>(p));
}

}  // namespace moepp
