// Float attention on the CDNA4 matrix cores (v_mfma_f32_32x32x2_f32: float operands, float
// accumulation), forward and backward, for head dimensions up to 128.
//
// A workgroup of 4 wavefronts owns 32 rows of one (sequence, head) pair - 32 queries in the forward
// and in the dQ role of the backward, 32 keys in the dK/dV role - and its wavefronts deal the other
// side's 32-row tiles among themselves; their results meet in LDS at the end.  That gives work to
// the whole chip even for a few short sequences, and no wavefront ever waits for another one inside
// the loop: operands go straight from memory (L1, L2) to registers.  A 32x32x2 instruction takes 64
// clocks for 8 operand bytes per lane, so nothing needs staging: per tile of 32 x 32 scores and head
// dim 64 the forward has 64 of them (4096 clocks) and 40 loads.
//
// Operand layouts are those of the bf16 kernels: scores are computed with the moving side's rows as
// result rows, which leaves each lane with one row of the workgroup's own side and 16 rows of the
// other - the operand of the next product.  For that product instruction r contracts the pair of
// rows that register r of the two lane groups holds, {8(r/4) + r%4, 8(r/4) + 4 + r%4}; for products
// over the head dimension lane group g holds columns 8i + 4g .. 8i + 4g + 3 (one 16-byte load) and
// instruction j contracts columns 8i + j and 8i + 4 + j.
// Head dimensions below the compiled D: the own side's columns beyond d are zeros, the moving side's
// repeat columns of the same head (finite, times zero), results beyond d are not stored.
#include "device.h"

#include <algorithm>

namespace chimera {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NT = 256, NW = 4, TILE = 32;
constexpr float NEG_BIG = -1.0e30f;
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f, LN2_LOW = -1.9046543e-9f;     // the float and what it lacks

struct Shape { int S, heads, batch, d; };

// Workgroup -> (sequence, head) pair and tile rank.  All tiles of a pair on one XCD (id mod 8); with
// the causal mask the longest tiles of all pairs first (rank slowest).
template <bool CAUSAL>
__device__ __forceinline__ bool tile_of(int bid, const Shape& sh, int& rank, int& h, int& b) {
    const int T = (sh.S + TILE - 1) / TILE, pairs = sh.heads * sh.batch, padded = (pairs + 7) & ~7;
    int p;
    if constexpr (CAUSAL) {
        p = bid % padded;
        rank = bid / padded;
    } else {
        const int j = bid >> 3;
        rank = j % T;
        p = (j / T) * 8 + (bid & 7);
    }
    h = p % sh.heads; b = p / sh.heads;
    return p < pairs;
}

// One row's share of a lane, over the head dimension: columns 8i + 4g .. +3.
template <int D> struct RowFrag {
    f32x4 v[D / 8];
    __device__ __forceinline__ void load(const float* __restrict__ row, int d, int g, bool zero_beyond) {
#pragma unroll
        for (int i = 0; i < D / 8; ++i) {
            const int c = 8 * i + 4 * g;
            v[i] = *reinterpret_cast<const f32x4*>(row + min(c, d - 4));
            if (zero_beyond && c >= d) v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
};
// acc[row of a][row of b] += sum over the head dimension
template <int D> __device__ __forceinline__ f32x16 dot_rows(const RowFrag<D>& a, const RowFrag<D>& b) {
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
    for (int i = 0; i < D / 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[i][j], b.v[i][j], acc, 0, 0, 0);
    return acc;
}
// The transposed operand: lane's column c = 32t + l32 of the 16 rows that its lane group contracts.
template <int D> struct ColFrag {
    float v[D / 32][16];
    __device__ __forceinline__ void load(const float* __restrict__ base, int ld, int row0, int last, int d, int l32, int g) {
#pragma unroll
        for (int t = 0; t < D / 32; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                v[t][r] = base[(size_t)min(row0 + 8 * (r >> 2) + 4 * g + (r & 3), last) * ld + min(t * 32 + l32, d - 1)];
    }
};
template <int D> __device__ __forceinline__ void add_outer(f32x16 (&acc)[D / 32], const ColFrag<D>& a, const f32x16& p) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int t = 0; t < D / 32; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[t][r], p[r], acc[t], 0, 0, 0);
}

// Sum of the wavefronts' accumulators [D columns][32 rows], in wavefront order; wavefront w receives
// the 4 columns 32t + 8w + 4g .. +3 of row l32 in out[t].
template <int D>
__device__ __forceinline__ void combine(float* lds, const f32x16 (&acc)[D / 32], f32x4 (&out)[D / 32], int wave, int lane) {
    constexpr int OT = D / 32;
#pragma unroll
    for (int t = 0; t < OT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) lds[((wave * OT + t) * 16 + r) * WAVE + lane] = acc[t][r];
    __syncthreads();
#pragma unroll
    for (int t = 0; t < OT; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) s += lds[((w * OT + t) * 16 + wave * 4 + c) * WAVE + lane];
            out[t][c] = s;
        }
}
template <int D>
__device__ __forceinline__ void store_rows(float* __restrict__ row, const f32x4 (&v)[D / 32], float scale, int d, int wave, int g) {
#pragma unroll
    for (int t = 0; t < D / 32; ++t) {
        const int c = t * 32 + 8 * wave + 4 * g;
        if (c < d) *reinterpret_cast<f32x4*>(row + c) = v[t] * scale;
    }
}

// A probability of the backward, exp(score * scale - lse): the difference is rounded once, in natural units, and what the
// product with log2(e) rounds off comes back behind the hardware's exp2.  (From a log-sum-exp in log2 units, rounded on the way
// there, it would carry 1.2 to 1.5 times the error.)
__device__ __forceinline__ float prob(float score, float scale, float lse) {
    const float x = __builtin_fmaf(score, scale, -lse), t = x * LOG2E, e = __builtin_amdgcn_exp2f(t);
    return e == 0.f ? 0.f : __builtin_fmaf(e, __builtin_fmaf(-t, LN2, x), e);        // x may be -inf
}

template <int D, bool CAUSAL>
__global__ __launch_bounds__(NT) void attn_fwd_f32_kernel(const float* __restrict__ qkv, float* __restrict__ ctx,
                                                          float* __restrict__ lse, Shape sh, float scale_log2e) {
    constexpr int OT = D / 32;
    __shared__ float lds[NW * OT * 16 * WAVE];
    __shared__ float stat[2][NW][32];
    const int S = sh.S, d = sh.d, H = sh.heads * d, ld = 3 * H;
    int rank, h, b;
    if (!tile_of<CAUSAL>((int)blockIdx.x, sh, rank, h, b)) return;
    const int q0 = ((S + TILE - 1) / TILE - 1 - rank) * TILE;
    const float* base = qkv + (size_t)b * S * ld + h * d;
    const float* Kg = base + H;
    const float* Vg = base + 2 * H;
    const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int qrow = q0 + l32;
    RowFrag<D> q;
    q.load(base + (size_t)min(qrow, S - 1) * ld, d, g, true);
    f32x16 o[OT];
#pragma unroll
    for (int t = 0; t < OT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] = 0.f;
    float m = NEG_BIG, lsum = 0.f;
    const int kend = CAUSAL ? min(S, q0 + TILE) : S;
    for (int k0 = wave * TILE; k0 < kend; k0 += NW * TILE) {
        RowFrag<D> k;
        ColFrag<D> v;
        k.load(Kg + (size_t)min(k0 + l32, S - 1) * ld, d, g, false);
        v.load(Vg, ld, k0, S - 1, d, l32, g);
        f32x16 s = dot_rows<D>(k, q);
        if (k0 + TILE > S || (CAUSAL && k0 + TILE - 1 > q0)) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = k0 + 8 * (r >> 2) + 4 * g + (r & 3);
                if (key >= S || (CAUSAL && key > qrow)) s[r] = NEG_BIG;
            }
        }
        float mx = s[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
        mx = max32(mx) * scale_log2e;
        const float m_new = fmaxf(m, mx), alpha = __builtin_amdgcn_exp2f(m - m_new);
        float rs = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            s[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], scale_log2e, -m_new));
            rs += s[r];
        }
        lsum = lsum * alpha + sum32(rs);
        m = m_new;
#pragma unroll
        for (int t = 0; t < OT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[t][r] *= alpha;
        add_outer<D>(o, v, s);
    }
    // the wavefronts' partial softmaxes: common maximum, rescaled sums
    if (g == 0) { stat[0][wave][l32] = m; stat[1][wave][l32] = lsum; }
    __syncthreads();
    float M = stat[0][0][l32];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, stat[0][w][l32]);
    float total = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) total += stat[1][w][l32] * __builtin_amdgcn_exp2f(stat[0][w][l32] - M);
    const float mine = __builtin_amdgcn_exp2f(m - M);           // 0 for a wavefront that saw no key
#pragma unroll
    for (int t = 0; t < OT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] *= mine;
    f32x4 out[OT];
    combine<D>(lds, o, out, wave, lane);
    if (qrow < S) {
        store_rows<D>(ctx + ((size_t)b * S + qrow) * H + h * d, out, 1.0f / total, d, wave, g);
        if (wave == 0 && g == 0) lse[((size_t)b * sh.heads + h) * S + qrow] = __builtin_fmaf(M, LN2, __builtin_fmaf(M, LN2_LOW, logf(total)));
    }
}

// dQ of 32 queries; delta = rowsum(dO * O) of the queries on the way.
template <int D, bool CAUSAL>
__device__ __forceinline__ void dq_role(float* lds, int bid, const float* __restrict__ qkv, const float* __restrict__ dctx,
                                        const float* __restrict__ ctx, const float* __restrict__ lse, float* __restrict__ dqkv,
                                        const Shape& sh, float scale) {
    constexpr int OT = D / 32;
    const int S = sh.S, d = sh.d, H = sh.heads * d, ld = 3 * H;
    int rank, h, b;
    if (!tile_of<CAUSAL>(bid, sh, rank, h, b)) return;
    const int q0 = ((S + TILE - 1) / TILE - 1 - rank) * TILE;
    const float* base = qkv + (size_t)b * S * ld + h * d;
    const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int qrow = q0 + l32, qr = min(qrow, S - 1);
    RowFrag<D> q, dO, o;
    q.load(base + (size_t)qr * ld, d, g, true);
    dO.load(dctx + ((size_t)b * S + qr) * H + h * d, d, g, true);
    o.load(ctx + ((size_t)b * S + qr) * H + h * d, d, g, true);
    const float my_lse = lse[((size_t)b * sh.heads + h) * S + qr];
    float delta = 0.f;
#pragma unroll
    for (int i = 0; i < D / 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) delta += dO.v[i][j] * o.v[i][j];
    delta = sum32(delta);
    f32x16 dq[OT];
#pragma unroll
    for (int t = 0; t < OT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) dq[t][r] = 0.f;
    const int kend = CAUSAL ? min(S, q0 + TILE) : S;
    for (int k0 = wave * TILE; k0 < kend; k0 += NW * TILE) {
        RowFrag<D> k, v;
        ColFrag<D> kt;
        k.load(base + H + (size_t)min(k0 + l32, S - 1) * ld, d, g, false);
        v.load(base + 2 * H + (size_t)min(k0 + l32, S - 1) * ld, d, g, false);
        kt.load(base + H, ld, k0, S - 1, d, l32, g);
        f32x16 p = dot_rows<D>(k, q), dp = dot_rows<D>(v, dO);
#pragma unroll
        for (int r = 0; r < 16; ++r) p[r] = prob(p[r], scale, my_lse);
        if (k0 + TILE > S || (CAUSAL && k0 + TILE - 1 > q0)) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = k0 + 8 * (r >> 2) + 4 * g + (r & 3);
                if (key >= S || (CAUSAL && key > qrow)) p[r] = 0.f;
            }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) dp[r] = p[r] * (dp[r] - delta);
        add_outer<D>(dq, kt, dp);
    }
    f32x4 out[OT];
    combine<D>(lds, dq, out, wave, lane);
    if (qrow < S) store_rows<D>(dqkv + ((size_t)b * S + qrow) * ld + h * d, out, scale, d, wave, g);
}

// dK, dV of 32 keys.
template <int D, bool CAUSAL>
__device__ __forceinline__ void dkv_role(float* lds, int bid, const float* __restrict__ qkv, const float* __restrict__ dctx,
                                         const float* __restrict__ ctx, const float* __restrict__ lse, float* __restrict__ dqkv,
                                         const Shape& sh, float scale) {
    constexpr int OT = D / 32;
    const int S = sh.S, d = sh.d, H = sh.heads * d, ld = 3 * H;
    int rank, h, b;
    if (!tile_of<CAUSAL>(bid, sh, rank, h, b)) return;
    const int j0 = rank * TILE;                  // the first keys meet the most queries
    const float* base = qkv + (size_t)b * S * ld + h * d;
    const float* dOg = dctx + (size_t)b * S * H + h * d;
    const float* Og = ctx + (size_t)b * S * H + h * d;
    const float* lseg = lse + ((size_t)b * sh.heads + h) * S;
    const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int jrow = j0 + l32, jr = min(jrow, S - 1);
    RowFrag<D> k, v;
    k.load(base + H + (size_t)jr * ld, d, g, true);
    v.load(base + 2 * H + (size_t)jr * ld, d, g, true);
    f32x16 dk[OT], dv[OT];
#pragma unroll
    for (int t = 0; t < OT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) { dk[t][r] = 0.f; dv[t][r] = 0.f; }
    for (int i0 = (CAUSAL ? j0 : 0) + wave * TILE; i0 < S; i0 += NW * TILE) {
        const int ir = min(i0 + l32, S - 1);
        RowFrag<D> q, dO, o;
        ColFrag<D> qt, dOt;
        q.load(base + (size_t)ir * ld, d, g, false);
        dO.load(dOg + (size_t)ir * H, d, g, true);
        o.load(Og + (size_t)ir * H, d, g, true);
        dOt.load(dOg, H, i0, S - 1, d, l32, g);
        qt.load(base, ld, i0, S - 1, d, l32, g);
        const float my_lse = lseg[ir];
        float delta = 0.f;                       // of row l32; the rows of the score registers fetch theirs from its lane
#pragma unroll
        for (int i = 0; i < D / 8; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) delta += dO.v[i][j] * o.v[i][j];
        delta = sum32(delta);
        f32x16 p = dot_rows<D>(q, k), dp = dot_rows<D>(dO, v);
        const bool edge = i0 + TILE > S || (CAUSAL && i0 < j0 + TILE - 1);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int ii = 8 * (r >> 2) + 4 * g + (r & 3);
            p[r] = prob(p[r], scale, __shfl(my_lse, ii, WAVE));
            if (edge && (i0 + ii >= S || (CAUSAL && i0 + ii < jrow))) p[r] = 0.f;
            dp[r] = p[r] * (dp[r] - __shfl(delta, ii, WAVE));
        }
        add_outer<D>(dv, dOt, p);
        add_outer<D>(dk, qt, dp);
    }
    f32x4 out[OT];
    combine<D>(lds, dv, out, wave, lane);
    if (jrow < S) store_rows<D>(dqkv + ((size_t)b * S + jrow) * ld + 2 * H + h * d, out, 1.0f, d, wave, g);
    __syncthreads();                             // everyone has read the dV sums
    combine<D>(lds, dk, out, wave, lane);
    if (jrow < S) store_rows<D>(dqkv + ((size_t)b * S + jrow) * ld + H + h * d, out, scale, d, wave, g);
}

// Both roles in one launch, in groups of 8 workgroups (one per XCD); each forms the delta it needs.
template <int D, bool CAUSAL>
__global__ __launch_bounds__(NT) void attn_bwd_f32_kernel(const float* __restrict__ qkv, const float* __restrict__ dctx,
                                                          const float* __restrict__ ctx, const float* __restrict__ lse,
                                                          float* __restrict__ dqkv, Shape sh, float scale) {
    __shared__ float lds[NW * (D / 32) * 16 * WAVE];
    const int blk = (int)blockIdx.x, bid = ((blk >> 4) << 3) | (blk & 7);
    if ((blk >> 3) & 1) dq_role<D, CAUSAL>(lds, bid, qkv, dctx, ctx, lse, dqkv, sh, scale);
    else dkv_role<D, CAUSAL>(lds, bid, qkv, dctx, ctx, lse, dqkv, sh, scale);
}

unsigned grid_of(const AttnArgs& a) {
    return (unsigned)((a.seq + TILE - 1) / TILE) * (((unsigned)a.heads * a.batch + 7) & ~7u);
}

}  // namespace

bool attention_f32_supports(const AttnArgs& a) {
    if (a.head_dim < 4 || a.head_dim > 128 || a.head_dim % 4) return false;
    if (a.batch < 1 || a.seq < 1 || a.heads < 1) return false;
    if (((unsigned long long)a.heads * a.batch + 7) * ((a.seq + TILE - 1) / TILE) >= (1ull << 30)) return false;
    return !(((uintptr_t)a.qkv | (uintptr_t)a.ctx | (uintptr_t)a.dctx | (uintptr_t)a.dqkv) & 15);
}

#define ATTN_F32(KERNEL, GRID, ...)                                                                                 \
    do {                                                                                                            \
        if (a.head_dim <= 32) { if (a.causal) ATTN_F32_GO(KERNEL, 32, true, GRID, __VA_ARGS__); else ATTN_F32_GO(KERNEL, 32, false, GRID, __VA_ARGS__); } \
        else if (a.head_dim <= 64) { if (a.causal) ATTN_F32_GO(KERNEL, 64, true, GRID, __VA_ARGS__); else ATTN_F32_GO(KERNEL, 64, false, GRID, __VA_ARGS__); } \
        else { if (a.causal) ATTN_F32_GO(KERNEL, 128, true, GRID, __VA_ARGS__); else ATTN_F32_GO(KERNEL, 128, false, GRID, __VA_ARGS__); } \
    } while (0)
#define ATTN_F32_GO(KERNEL, D, C, GRID, ...) hipLaunchKernelGGL((KERNEL<D, C>), dim3(GRID), dim3(NT), 0, s, __VA_ARGS__)

int attention_fwd_f32(const AttnArgs& a, void* stream) {
    if (!attention_f32_supports(a)) return fail(CHIMERA_EINVAL, "float matrix-core attention: unsupported shape (head_dim %d)", a.head_dim);
    hipStream_t s = (hipStream_t)stream;
    const Shape sh{a.seq, a.heads, a.batch, a.head_dim};
    ATTN_F32(attn_fwd_f32_kernel, grid_of(a), (const float*)a.qkv, (float*)a.ctx, a.lse, sh, LOG2E / sqrtf((float)a.head_dim));
    CHIMERA_LAUNCH_CHECK("float attention forward");
    return CHIMERA_OK;
}

int attention_bwd_f32(const AttnArgs& a, void* stream) {
    if (!attention_f32_supports(a)) return fail(CHIMERA_EINVAL, "float matrix-core attention: unsupported shape (head_dim %d)", a.head_dim);
    hipStream_t s = (hipStream_t)stream;
    const Shape sh{a.seq, a.heads, a.batch, a.head_dim};
    ATTN_F32(attn_bwd_f32_kernel, 2 * grid_of(a), (const float*)a.qkv, (const float*)a.dctx, (const float*)a.ctx, a.lse, (float*)a.dqkv, sh,
             1.0f / sqrtf((float)a.head_dim));
    CHIMERA_LAUNCH_CHECK("float attention backward");
    return CHIMERA_OK;
}

}  // namespace chimera
