// Fused attention on the CDNA4 matrix cores (bf16 in, float softmax and
// accumulation), forward and backward, for head dimensions that are multiples of 8 up to
// 128 (compiled for D = 64 and 128; below them the fixed operand's columns beyond the head
// dimension are zeros, the others' repeat columns of the same head, and results beyond it
// are not stored: half the matrix work at worst, while the softmax sets the time).
//
//   forward   per (sequence, head, 128 queries): loop over 64-key tiles with an
//             online softmax; writes ctx and the log-sum-exp of every row.
//   backward  two roles that both rebuild P = exp(q k^T / sqrt(d) - lse) from
//             the saved log-sum-exp:
//             dQ    per (sequence, head, 128 queries) looping over 64-key tiles,
//             dK/dV per (sequence, head, 128 keys) looping over 64-query tiles.
//             With many (sequence, head) pairs they are two launches and the dQ
//             one forms delta = rowsum(dctx * ctx) of its queries on the way;
//             with few pairs a small kernel forms delta first and both roles
//             share one launch.  No atomics: every output element has one
//             owner, so results are reproducible bit for bit.
//
// Register/LDS choreography.  v_mfma_f32_32x32x16_bf16 takes, per lane l, 8
// contraction values of row (or column) l%32; which 8 contraction indices a
// lane group l/32 holds is free as long as both operands agree.  Its result
// gives lane l column l%32 and rows 8*(r/4) + 4*(l/32) + r%4 (r = register).
// So a score tile computed TRANSPOSED (keys x queries) leaves each lane with
// one query and 16 keys - exactly an operand of the next product (contraction
// over keys) with keys {4g..4g+3, 8+4g..8+4g+3} (g = l/32) per 16-key step.
// The other operand of that product (V^T, or Q^T, dO^T, K^T in the backward)
// comes from the same LDS tile the tensor arrived in, through the transposing
// LDS read; P never touches LDS, and no transposed tensor exists anywhere.
// The fixed operand of a wavefront (its 32 queries, or its 32 keys and values)
// is loaded straight from global memory into MFMA operand registers.
#include "device.h"

#include <type_traits>

namespace chimera {

namespace {

typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int NT = 256;
constexpr float NEG_BIG = -1.0e30f;
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

__device__ __forceinline__ bf16x8 load_frag(const bf16_t* p, bool ok) {
    bf16x8 z;
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] = (bf16_t)0.f;
    return ok ? *reinterpret_cast<const bf16x8*>(p) : z;
}

// LDS tiles: one copy [64 rows][D] per tensor serves BOTH operand forms - a straight
// 16-byte read gives a lane 8 consecutive columns of its row (contraction over columns), the
// transposing read gives it 4 consecutive rows of its column (contraction over rows).  The
// 16-byte chunk c of row r sits at c ^ usw(r); usw is chosen so that both read patterns are
// conflict-free on the 64 banks: a straight read touches 16 consecutive rows at one chunk
// index, a transposing read 4 consecutive rows at 4 consecutive chunks.
template <int D> __device__ __forceinline__ int usw(int r) {
    if (D == 64) { const int h = (r >> 1) & 7; return ((h & 1) << 2) | (h & 2) | (h >> 2); }   // 128-byte rows: bit reversal of r/2
    return ((r & 3) << 2) | ((r >> 2) & 3);                                                     // 256-byte rows
}
template <int D>
__device__ __forceinline__ void dma_utile(const bf16_t* __restrict__ g, int ld, int row0, int row_last, int d, unsigned lds_base,
                                          int wave, int lane) {
    constexpr int KB = 64 * D * 2 / 1024, CPR = D / 8;
#pragma unroll
    for (int n0 = 0; n0 < KB; n0 += NT / WAVE) {
        const int n = n0 + wave;
        const int row = n * (64 / CPR) + lane / CPR;
        const int col = min((lane % CPR) ^ usw<D>(row), d / 8 - 1) << 3;
        lds_dma16(g + (size_t)min(row0 + row, row_last) * ld + col, lds_base + n * 1024);
    }
}
// rows = `row`, contraction step kk over 16 columns
template <int D>
__device__ __forceinline__ bf16x8 frag_us(const bf16_t* tile, int row, int kk, int g) {
    return *reinterpret_cast<const bf16x8*>(tile + row * D + (((kk * 2 + g) ^ usw<D>(row)) << 3));
}
// rows = columns col0 + lane%32 of the tile, contraction over tile rows of 16-step J, in the
// slot order {4g..4g+3, 8+4g..8+4g+3} of a transposed score tile
template <int D>
__device__ __forceinline__ bf16x8 frag_ut(const bf16_t* tile, int col0, int J, int lane) {
    typedef bf16x4 __attribute__((address_space(3))) * lds_v4;
    const int i = lane & 15, g = lane >> 5;
    const int c = (((col0 >> 4) + ((lane >> 4) & 1)) << 1) + ((i >> 1) & 1);
    const int r = 16 * J + 4 * g + (i >> 2);
    const bf16_t* p0 = tile + r * D + ((c ^ usw<D>(r)) << 3) + ((i & 1) << 2);
    const bf16_t* p1 = tile + (r + 8) * D + ((c ^ usw<D>(r + 8)) << 3) + ((i & 1) << 2);
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_v4)p0);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_v4)p1);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

__device__ __forceinline__ bf16x8 pack8(const f32x16& v, int first) {
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (bf16_t)v[first + i];
    return o;
}

// sum over four neighbouring lanes
__device__ __forceinline__ float quad_sum(float v) {
    v += dpp<0xb1>(v);
    return v + dpp<0x4e>(v);
}

// ------------------------------------------------------------------- forward
// Which 128-row tile (by rank: 0 = the one with the most work under the causal mask), head and
// sequence a workgroup of the 1-D grid takes; false for the padding workgroups.  Workgroup ids
// go round-robin over the 8 XCDs, so the (sequence, head) pair is chosen by id mod 8 first (the
// pair count is padded to a multiple of 8): all tiles of a pair then run on one XCD and its K, V
// (or Q, dO) are fetched into one L2 instead of up to eight.  Without a mask a group of 8 pairs
// works through its tiles before the next group starts.  With the causal mask a tile's work grows
// with its position, so the longest tiles of ALL pairs are dispatched first (rank slowest).
template <bool CAUSAL>
__device__ __forceinline__ bool attn_tile_of(int bid, int S, int heads, int batch, int& rank, int& h, int& b) {
    const int T = (S + 127) / 128;
    const int pairs = heads * batch, padded = (pairs + 7) & ~7;
    int p;
    if constexpr (CAUSAL) {
        p = bid % padded;
        rank = bid / padded;
    } else {
        const int j = bid >> 3;
        rank = j % T;
        p = (j / T) * 8 + (bid & 7);
    }
    h = p % heads; b = p / heads;
    return p < pairs;
}
inline unsigned attn_grid(const AttnArgs& a) {
    const unsigned T = (a.seq + 127) / 128, pairs = (unsigned)a.heads * a.batch;
    return T * ((pairs + 7) & ~7u);
}

// The forward moves its K and V tiles global -> LDS directly (lds_dma16), one tile ahead of
// the matrix cores, with no staging registers and no transposition work: K is read straight
// (contraction over the head dimension), V with the transposing read (contraction over keys).
// Rows beyond the sequence are fetched from its last row (finite data): their scores are
// masked, so they contribute exact zeros.
//
// A step is a serial chain per wavefront (scores, row maximum, exponentials, P V) with four
// wavefronts per SIMD at most (two at head dim 128) to cover it, so its length bounds the kernel.
// The two halves of a row's keys lie in lanes l and l ^ 32: their maxima meet through max32 (a
// register swap, where a lane exchange through LDS waits for the LDS queue), and each half's sum
// stays in its lane until the keys are done (both halves rescale by the same factor).  Measured
// against two LDS exchanges per step: 2 x 1024 rows of 25 heads of 64 causal 19.8 -> 17.9 us, 632
// rows 12.3 -> 11.3 us, 2048 rows of 16 heads of 128 45.0 -> 41.8 us, 8 x 512 rows of 16 heads of
// 64 15.8 -> 15.3 us.
template <int D, bool CAUSAL>
__global__ __launch_bounds__(NT) void attn_fwd_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ ctx,
                                                      float* __restrict__ lse, int S, int heads, int batch,
                                                      int d, float scale_log2e) {
    constexpr int KS = D / 16, OT = D / 32;
    __shared__ __attribute__((aligned(16))) bf16_t Ks[2][64 * D];
    __shared__ __attribute__((aligned(16))) bf16_t Vs[2][64 * D];
    const int H = heads * d, ld = 3 * H, bid = (int)blockIdx.x;
    int rank, h, b;
    if (!attn_tile_of<CAUSAL>(bid, S, heads, batch, rank, h, b)) return;
    const int q0 = ((S + 127) / 128 - 1 - rank) * 128;       // longest (causal) tiles first
    const bf16_t* base = qkv + (size_t)b * S * ld + h * d;
    const bf16_t* Kg = base + H;
    const bf16_t* Vg = base + 2 * H;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wq0 = q0 + wave * 32, qrow = wq0 + l32;
    const unsigned ks0 = lds_address(Ks), vs0 = lds_address(Vs);
    constexpr unsigned TILE_BYTES = 64 * D * 2;

    const int kv_end = CAUSAL ? min(S, q0 + 128) : S;
    const int ntiles = (kv_end + 63) / 64;
    dma_utile<D>(Kg, ld, 0, S - 1, d, ks0, wave, lane);
    dma_utile<D>(Vg, ld, 0, S - 1, d, vs0, wave, lane);

    bf16x8 qf[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) qf[kk] = load_frag(base + (size_t)qrow * ld + kk * 16 + g * 8, qrow < S && kk * 16 + g * 8 < d);

    f32x16 o[OT];
#pragma unroll
    for (int t = 0; t < OT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] = 0.f;
    float m = NEG_BIG, lsum = 0.f;          // lsum: over this lane's half of the keys

    // one step of the key loop; the LDS buffer index is a compile-time constant so that every LDS
    // address is the lane's base plus an immediate
    auto step = [&](int t, auto buf_c) {
        constexpr int buf = decltype(buf_c)::value;
        const int k0 = t * 64;
        wait_vmcnt<0>();                   // this wavefront's share of tile t has landed
        __syncthreads();                   // everyone's has; and tile t-1 is consumed, so its buffer is free
        if (t + 1 < ntiles) {
            dma_utile<D>(Kg, ld, k0 + 64, S - 1, d, ks0 + (buf ^ 1) * TILE_BYTES, wave, lane);
            dma_utile<D>(Vg, ld, k0 + 64, S - 1, d, vs0 + (buf ^ 1) * TILE_BYTES, wave, lane);
        }
        const bool live = !CAUSAL || k0 <= wq0 + 31;          // wavefront-uniform: some key is visible
        if (live) {
            f32x16 s[2];
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[kt][r] = 0.f;
#pragma unroll
                for (int kk = 0; kk < KS; ++kk)
                    s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_us<D>(Ks[buf], kt * 32 + l32, kk, g), qf[kk],
                                                                    s[kt], 0, 0, 0);
            }
            // tiles that reach past the sequence or the diagonal mask key by key; the others skip it
            // (wavefront-uniform branch)
            if ((k0 + 63 >= S) || (CAUSAL && k0 + 63 > wq0)) {
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int key = k0 + kt * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
                        if (key >= S || (CAUSAL && key > qrow)) s[kt][r] = NEG_BIG;
                    }
            }
            // running maximum in the scaled (log2) domain; the scale is positive, so it commutes with max
            float mx = NEG_BIG;
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kt][r]);
            const float m_new = fmaxf(m, max32(mx) * scale_log2e);
            float rs = 0.f;
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    // hardware exp2: arguments are <= 0 here, and flushing tiny results to zero is harmless
                    const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kt][r], scale_log2e, -m_new));
                    s[kt][r] = p;
                    rs += p;
                }
            // the accumulators only need rescaling when some row's maximum moved
            if (__builtin_amdgcn_ballot_w64(m_new != m)) {
                const float alpha = __builtin_amdgcn_exp2f(m - m_new);
                lsum *= alpha;
#pragma unroll
                for (int t2 = 0; t2 < OT; ++t2)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[t2][r] *= alpha;
            }
            lsum += rs;
            m = m_new;
#pragma unroll
            for (int J = 0; J < 4; ++J) {
                const bf16x8 pf = pack8(s[J >> 1], (J & 1) * 8);
#pragma unroll
                for (int t2 = 0; t2 < OT; ++t2)
                    o[t2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_ut<D>(Vs[buf], t2 * 32, J, lane), pf, o[t2], 0, 0, 0);
            }
        }
    };
    for (int t = 0; t < ntiles; t += 2) {
        step(t, std::integral_constant<int, 0>{});
        if (t + 1 < ntiles) step(t + 1, std::integral_constant<int, 1>{});
    }

    lsum = sum32(lsum);
    if (qrow < S) {
        const float inv = 1.0f / lsum;
        bf16_t* out = ctx + ((size_t)b * S + qrow) * H + h * d;
#pragma unroll
        for (int t2 = 0; t2 < OT; ++t2)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                bf16x4 v;
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = (bf16_t)(o[t2][r4 * 4 + c] * inv);
                if (t2 * 32 + 8 * r4 < d) *reinterpret_cast<bf16x4*>(out + t2 * 32 + 8 * r4 + 4 * g) = v;
            }
        if (g == 0) lse[((size_t)b * heads + h) * S + qrow] = (m + log2f(lsum)) * LN2;
    }
}

// ------------------------------------------------------------------ backward
// dK, dV of 128 keys (32 per wavefront), looping over 64-query tiles.
//   S  = Q K^T (queries x keys)   P = exp2(S c - lse2)     dP = dO V^T
//   dS = P (dP - delta)           dV^T += dO^T P           dK^T += Q^T dS (then * 1/sqrt(d))
// The Q and dO tiles of the next step travel global -> LDS (lds_dma16) while the matrix cores
// work on the current one; each 32-query half of a tile is finished (scores to dK/dV) before
// the next starts, which keeps the live score registers at 32.  Rows beyond the sequence
// repeat its last row; their P is masked to zero.
// The dP products start at -delta (its LDS copy is negated) where they started at zero: that
// is the subtraction without an instruction per score, and at head dim 128, whose accumulators
// and fragments exceed the 256 registers that vector instructions reach, fewer copies to the
// others: both roles together 2048 rows of 16 heads of 128 causal 111.7 -> 98.4 us, 2 x 1024 of
// 16 105.4 -> 94.1, 4 x 333 of 6 26.4 -> 24.1; 8 x 512 of 16 of 64 47.9 -> 47.2.
// LDS of one backward workgroup: two tensors x two stages of [64][D] tiles, and (dK/dV role) the
// statistics of a tile's 64 queries.
template <int D> struct AttnBwdLds {
    bf16_t t0[2][64 * D], t1[2][64 * D];
    float lse2[2][64], dl[2][64];
};

template <int D, bool CAUSAL, bool FORM_DELTA>
__device__ __forceinline__ void attn_bwd_dkv_role(AttnBwdLds<D>& sm, int bid, const bf16_t* __restrict__ qkv,
                                                  const bf16_t* __restrict__ dctx, const bf16_t* __restrict__ ctx,
                                                  const float* __restrict__ lse,
                                                  const float* __restrict__ delta, bf16_t* __restrict__ dqkv, int S,
                                                  int heads, int batch, int d, float scale) {
    constexpr int KS = D / 16, OT = D / 32;
    constexpr unsigned TILE_BYTES = 64 * D * 2;
    bf16_t (&Qs)[2][64 * D] = sm.t0;
    bf16_t (&Os)[2][64 * D] = sm.t1;
    float (&lse2)[2][64] = sm.lse2;
    float (&dl)[2][64] = sm.dl;
    const int H = heads * d, ld = 3 * H;
    int rank, h, b;
    if (!attn_tile_of<CAUSAL>(bid, S, heads, batch, rank, h, b)) return;
    const int j0 = rank * 128;             // the first keys meet the most queries
    const bf16_t* base = qkv + (size_t)b * S * ld + h * d;
    const bf16_t* dOg = dctx + (size_t)b * S * H + h * d;
    const size_t stat0 = ((size_t)b * heads + h) * S;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wj0 = j0 + wave * 32, jrow = wj0 + l32;
    const float c2 = scale * LOG2E;
    const unsigned qs0 = lds_address(Qs), os0 = lds_address(Os);

    const int qt0 = CAUSAL ? j0 / 64 : 0;
    const int ntiles = (S + 63) / 64;
    float stat = 0.f;                      // lse (threads 0..63) or delta (threads 64..127) of the next tile
    // FORM_DELTA: a query's delta comes from four neighbouring threads, each with a quarter of its row of dO and O
    constexpr int DP = FORM_DELTA ? D / 32 : 1;
    const int dq_row = tid >> 2, dq_col = (tid & 3) * (D / 4);
    bf16x8 od[DP], oc[DP];
    auto fetch = [&](int t, int buf) {
        const int i0 = t * 64;
        dma_utile<D>(base, ld, i0, S - 1, d, qs0 + buf * TILE_BYTES, wave, lane);
        dma_utile<D>(dOg, H, i0, S - 1, d, os0 + buf * TILE_BYTES, wave, lane);
        if (tid < (FORM_DELTA ? 64 : 128)) {
            const int i = i0 + (tid & 63);
            stat = i < S ? (tid < 64 ? lse[stat0 + i] * LOG2E : -delta[stat0 + i]) : 0.f;
        }
        if constexpr (FORM_DELTA) {
            const size_t at = (size_t)(i0 + dq_row) * H + dq_col;
#pragma unroll
            for (int j = 0; j < DP; ++j) {
                const bool ok = i0 + dq_row < S && dq_col + 8 * j < d;
                od[j] = load_frag(dOg + at + 8 * j, ok);
                oc[j] = load_frag(ctx + ((size_t)b * S * H + h * d) + at + 8 * j, ok);
            }
        }
    };
    fetch(qt0, 0);

    bf16x8 kf[KS], vf[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
        kf[kk] = load_frag(base + H + (size_t)jrow * ld + kk * 16 + g * 8, jrow < S && kk * 16 + g * 8 < d);
        vf[kk] = load_frag(base + 2 * H + (size_t)jrow * ld + kk * 16 + g * 8, jrow < S && kk * 16 + g * 8 < d);
    }
    f32x16 dk[OT], dv[OT];
#pragma unroll
    for (int t = 0; t < OT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) { dk[t][r] = 0.f; dv[t][r] = 0.f; }

    auto step = [&](int t, auto buf_c) {        // LDS buffer index at compile time: addresses become base + immediate
        constexpr int buf = decltype(buf_c)::value;
        const int i0 = t * 64;
        wait_vmcnt<0>();                   // this wavefront's share of tile t (and its statistics) has arrived
        if (tid < 64) lse2[buf][tid] = stat;
        else if (!FORM_DELTA && tid < 128) dl[buf][tid - 64] = stat;
        if constexpr (FORM_DELTA) {
            float v = 0.f;
#pragma unroll
            for (int j = 0; j < DP; ++j)
#pragma unroll
                for (int e = 0; e < 8; ++e) v += (float)od[j][e] * (float)oc[j][e];
            v = quad_sum(v);
            if ((tid & 3) == 0) dl[buf][dq_row] = -v;
        }
        __syncthreads();                   // tile t complete in LDS; tile t-1 consumed by everyone
        if (t + 1 < ntiles) fetch(t + 1, buf ^ 1);
        const bf16_t* Qt = Qs[buf];
        const bf16_t* Ot = Os[buf];
        const bool live = !CAUSAL || i0 + 63 >= wj0;           // some query of the tile sees some key of this wavefront
        if (live) {
            const bool edge = (i0 + 63 >= S) || (CAUSAL && i0 < wj0 + 31);
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                f32x16 p, dp;
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {                       // 4 consecutive queries; dP starts at -delta
                    const float4 d4 = *reinterpret_cast<const float4*>(&dl[buf][it * 32 + 8 * r4 + 4 * g]);
                    const float dv4[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
                    for (int c = 0; c < 4; ++c) { p[r4 * 4 + c] = 0.f; dp[r4 * 4 + c] = dv4[c]; }
                }
#pragma unroll
                for (int kk = 0; kk < KS; ++kk) {
                    p = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_us<D>(Qt, it * 32 + l32, kk, g), kf[kk], p, 0, 0, 0);
                    dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_us<D>(Ot, it * 32 + l32, kk, g), vf[kk], dp, 0, 0, 0);
                }
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const int il = it * 32 + 8 * r4 + 4 * g;       // 4 consecutive queries
                    const float4 l4 = *reinterpret_cast<const float4*>(&lse2[buf][il]);
                    const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int r = r4 * 4 + c;
                        p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(p[r], c2, -lv[c]));     // hardware exp2
                    }
                }
                if (edge) {                               // wavefront-uniform: only tiles on an edge mask
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int i = i0 + it * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
                        if (i >= S || (CAUSAL && i < jrow)) p[r] = 0.f;
                    }
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) dp[r] *= p[r];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int J = it * 2 + j;
                    const bf16x8 pf = pack8(p, j * 8);
                    const bf16x8 dsf = pack8(dp, j * 8);
#pragma unroll
                    for (int t2 = 0; t2 < OT; ++t2) {
                        dv[t2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_ut<D>(Ot, t2 * 32, J, lane), pf, dv[t2], 0, 0, 0);
                        dk[t2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_ut<D>(Qt, t2 * 32, J, lane), dsf, dk[t2], 0, 0, 0);
                    }
                }
            }
        }
    };
    for (int t = qt0; t < ntiles; t += 2) {
        step(t, std::integral_constant<int, 0>{});
        if (t + 1 < ntiles) step(t + 1, std::integral_constant<int, 1>{});
    }
    if (jrow < S) {
        bf16_t* out = dqkv + ((size_t)b * S + jrow) * ld + h * d;
#pragma unroll
        for (int t2 = 0; t2 < OT; ++t2)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                bf16x4 a, c;
#pragma unroll
                for (int e = 0; e < 4; ++e) { a[e] = (bf16_t)(dk[t2][r4 * 4 + e] * scale); c[e] = (bf16_t)dv[t2][r4 * 4 + e]; }
                if (t2 * 32 + 8 * r4 >= d) continue;
                *reinterpret_cast<bf16x4*>(out + H + t2 * 32 + 8 * r4 + 4 * g) = a;
                *reinterpret_cast<bf16x4*>(out + 2 * H + t2 * 32 + 8 * r4 + 4 * g) = c;
            }
    }
}

// dQ of 128 queries (32 per wavefront), looping over 64-key tiles.
//   S^T = K Q^T (keys x queries)   P = exp2(S^T c - lse2)   dP^T = V dO^T
//   dS^T = P (dP^T - delta)        dQ^T += K^T dS^T (then * 1/sqrt(d))
// FORM_DELTA: delta = rowsum(dO * O) of the workgroup's queries is formed here (from the dO
// fragments the wavefront holds anyway and the same pieces of O) and written out for the dK/dV
// kernel that follows; otherwise it is read (attn_delta_kernel has run).
template <int D, bool CAUSAL, bool FORM_DELTA>
__device__ __forceinline__ void attn_bwd_dq_role(AttnBwdLds<D>& sm, int bid, const bf16_t* __restrict__ qkv,
                                                 const bf16_t* __restrict__ dctx, const bf16_t* __restrict__ ctx,
                                                 const float* __restrict__ lse, float* __restrict__ delta,
                                                 bf16_t* __restrict__ dqkv, int S, int heads, int batch, int d, float scale) {
    constexpr int KS = D / 16, OT = D / 32;
    constexpr unsigned TILE_BYTES = 64 * D * 2;
    bf16_t (&Ks)[2][64 * D] = sm.t0;
    bf16_t (&Vs)[2][64 * D] = sm.t1;
    const int H = heads * d, ld = 3 * H;
    int rank, h, b;
    if (!attn_tile_of<CAUSAL>(bid, S, heads, batch, rank, h, b)) return;
    const int q0 = ((S + 127) / 128 - 1 - rank) * 128;
    const bf16_t* base = qkv + (size_t)b * S * ld + h * d;
    const bf16_t* dOg = dctx + (size_t)b * S * H + h * d;
    const size_t stat0 = ((size_t)b * heads + h) * S;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wq0 = q0 + wave * 32, qrow = wq0 + l32;
    const float c2 = scale * LOG2E;
    const unsigned ks0 = lds_address(Ks), vs0 = lds_address(Vs);

    const int kv_end = CAUSAL ? min(S, q0 + 128) : S;
    const int ntiles = (kv_end + 63) / 64;
    auto fetch = [&](int t, int buf) {
        dma_utile<D>(base + H, ld, t * 64, S - 1, d, ks0 + buf * TILE_BYTES, wave, lane);
        dma_utile<D>(base + 2 * H, ld, t * 64, S - 1, d, vs0 + buf * TILE_BYTES, wave, lane);
    };
    fetch(0, 0);

    bf16x8 qf[KS], of[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
        qf[kk] = load_frag(base + (size_t)qrow * ld + kk * 16 + g * 8, qrow < S && kk * 16 + g * 8 < d);
        of[kk] = load_frag(dOg + (size_t)qrow * H + kk * 16 + g * 8, qrow < S && kk * 16 + g * 8 < d);
    }
    const float my_lse2 = qrow < S ? lse[stat0 + qrow] * LOG2E : 0.f;
    float my_dl = 0.f;
    if constexpr (FORM_DELTA) {
        // the lane pair (l, l^32) holds the whole row of dO
        const bf16_t* Og = ctx + (size_t)b * S * H + h * d;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            const bf16x8 cf = load_frag(Og + (size_t)qrow * H + kk * 16 + g * 8, qrow < S && kk * 16 + g * 8 < d);
#pragma unroll
            for (int e = 0; e < 8; ++e) my_dl += (float)of[kk][e] * (float)cf[e];
        }
        my_dl = sum32(my_dl);
        if (g == 0 && qrow < S) delta[stat0 + qrow] = my_dl;
    } else {
        my_dl = qrow < S ? delta[stat0 + qrow] : 0.f;
    }
    f32x16 dq[OT];
#pragma unroll
    for (int t = 0; t < OT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) dq[t][r] = 0.f;

    auto step = [&](int t, auto buf_c) {        // LDS buffer index at compile time
        constexpr int buf = decltype(buf_c)::value;
        const int k0 = t * 64;
        wait_vmcnt<0>();
        __syncthreads();
        if (t + 1 < ntiles) fetch(t + 1, buf ^ 1);
        const bf16_t* Kt = Ks[buf];
        const bf16_t* Vt = Vs[buf];
        const bool live = !CAUSAL || k0 <= wq0 + 31;
        if (live) {
            const bool edge = (k0 + 63 >= S) || (CAUSAL && k0 + 63 > wq0);
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                f32x16 p, dp;
                // at head dim 64 sixteen registers of -delta cost the third wavefront per SIMD (170 for 152)
#pragma unroll
                for (int r = 0; r < 16; ++r) { p[r] = 0.f; dp[r] = D > 64 ? -my_dl : 0.f; }
#pragma unroll
                for (int kk = 0; kk < KS; ++kk) {
                    p = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_us<D>(Kt, kt * 32 + l32, kk, g), qf[kk], p, 0, 0, 0);
                    dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_us<D>(Vt, kt * 32 + l32, kk, g), of[kk], dp, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(p[r], c2, -my_lse2));   // hardware exp2
                if (edge) {                               // wavefront-uniform: only tiles on an edge mask
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int key = k0 + kt * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
                        if (key >= S || (CAUSAL && key > qrow)) p[r] = 0.f;
                    }
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) dp[r] = p[r] * (D > 64 ? dp[r] : dp[r] - my_dl);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const bf16x8 dsf = pack8(dp, j * 8);
#pragma unroll
                    for (int t2 = 0; t2 < OT; ++t2)
                        dq[t2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_ut<D>(Kt, t2 * 32, kt * 2 + j, lane), dsf, dq[t2], 0, 0, 0);
                }
            }
        }
    };
    for (int t = 0; t < ntiles; t += 2) {
        step(t, std::integral_constant<int, 0>{});
        if (t + 1 < ntiles) step(t + 1, std::integral_constant<int, 1>{});
    }
    if (qrow < S) {
        bf16_t* out = dqkv + ((size_t)b * S + qrow) * ld + h * d;
#pragma unroll
        for (int t2 = 0; t2 < OT; ++t2)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                bf16x4 a;
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] = (bf16_t)(dq[t2][r4 * 4 + e] * scale);
                if (t2 * 32 + 8 * r4 < d) *reinterpret_cast<bf16x4*>(out + t2 * 32 + 8 * r4 + 4 * g) = a;
            }
    }
}

// delta[sequence, head, position] = sum over the head dimension of dO * O: one lane per 8 elements
// (16 bytes of each tensor), D / 8 lanes of a (token, head) pair side by side (those beyond d add 0).
template <int D>
__global__ __launch_bounds__(NT) void attn_delta_kernel(const bf16_t* __restrict__ dctx, const bf16_t* __restrict__ ctx,
                                                        float* __restrict__ delta, int S, int heads, int batch, int d) {
    constexpr int LPH = D / 8;                                   // lanes per (token, head)
    const size_t th = ((size_t)blockIdx.x * NT + threadIdx.x) / LPH;
    const int j = threadIdx.x % LPH;
    const bool live = th < (size_t)batch * S * heads;
    float v = 0.f;
    if (live && j * 8 < d) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(dctx + th * d + j * 8);
        const bf16x8 o = *reinterpret_cast<const bf16x8*>(ctx + th * d + j * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) v += (float)a[e] * (float)o[e];
    }
#pragma unroll
    for (int off = LPH / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, WAVE);
    if (live && j == 0) {
        const size_t token = th / heads, h = th % heads;         // token = sequence * S + position
        delta[((token / S) * heads + h) * S + token % S] = v;
    }
}

// Both backward kernels in one launch: workgroups come in groups of 8 (one per XCD), the groups
// alternate between the dK/dV role and the dQ role, and a workgroup's number within its role keeps
// its id mod 8, so that a (sequence, head) pair's tiles of both roles meet in one L2.  The two
// roles are independent (delta comes from attn_delta_kernel, or with FORM_DELTA each forms its
// own), so with few pairs - where one role alone leaves the chip half empty and its longest causal
// tile sets the time - each fills the other's gaps.
template <int D, bool CAUSAL, bool FORM_DELTA>
__global__ __launch_bounds__(NT) void attn_bwd_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ dctx,
                                                      const bf16_t* __restrict__ ctx, const float* __restrict__ lse, float* __restrict__ delta,
                                                      bf16_t* __restrict__ dqkv, int S, int heads, int batch, int d, float scale) {
    __shared__ __attribute__((aligned(16))) AttnBwdLds<D> sm;
    const int blk = (int)blockIdx.x;
    const int role = (blk >> 3) & 1, bid = ((blk >> 4) << 3) | (blk & 7);
    if (role == 0) attn_bwd_dkv_role<D, CAUSAL, FORM_DELTA>(sm, bid, qkv, dctx, ctx, lse, delta, dqkv, S, heads, batch, d, scale);
    else attn_bwd_dq_role<D, CAUSAL, FORM_DELTA>(sm, bid, qkv, dctx, ctx, lse, delta, dqkv, S, heads, batch, d, scale);
}

// The roles as launches of their own, dQ first (it forms delta): for many pairs, where each role
// fills the chip by itself and the merged kernel's register count (that of its larger role) would
// only cost the other role wavefronts per SIMD.
template <int D, bool CAUSAL>
__global__ __launch_bounds__(NT) void attn_bwd_dq_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ dctx,
                                                         const bf16_t* __restrict__ ctx, const float* __restrict__ lse,
                                                         float* __restrict__ delta, bf16_t* __restrict__ dqkv, int S,
                                                         int heads, int batch, int d, float scale) {
    __shared__ __attribute__((aligned(16))) AttnBwdLds<D> sm;
    attn_bwd_dq_role<D, CAUSAL, true>(sm, (int)blockIdx.x, qkv, dctx, ctx, lse, delta, dqkv, S, heads, batch, d, scale);
}
template <int D, bool CAUSAL>
__global__ __launch_bounds__(NT) void attn_bwd_dkv_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ dctx,
                                                          const float* __restrict__ lse, const float* __restrict__ delta,
                                                          bf16_t* __restrict__ dqkv, int S, int heads, int batch, int d,
                                                          float scale) {
    __shared__ __attribute__((aligned(16))) AttnBwdLds<D> sm;
    attn_bwd_dkv_role<D, CAUSAL, false>(sm, (int)blockIdx.x, qkv, dctx, nullptr, lse, delta, dqkv, S, heads, batch, d, scale);
}

// ctx in the forward (which has no dctx), ctx, dctx and dqkv in the backward
bool misaligned(const AttnArgs& a) {
    return a.dctx ? ((uintptr_t)a.ctx | (uintptr_t)a.dctx | (uintptr_t)a.dqkv) & 15 : (uintptr_t)a.ctx & 7;
}

int check(const AttnArgs& a) {
    if (!attention_mfma_supports(a)) return fail(CHIMERA_EINVAL, "matrix-core attention: unsupported shape (head_dim %d)", a.head_dim);
    return CHIMERA_OK;
}

}  // namespace

bool attention_mfma_supports(const AttnArgs& a) {
    if (a.head_dim < 8 || a.head_dim > 128 || a.head_dim % 8) return false;
    if (a.batch < 1 || a.seq < 1 || a.heads < 1 || a.batch > 65535 || a.heads > 65535) return false;
    if (((unsigned long long)a.heads * a.batch + 7) * ((a.seq + 127) / 128) >= (1ull << 30)) return false;   // 1-D grid
    if ((uintptr_t)a.qkv & 15) return false;
    // Other buffers that 8- and 16-byte accesses cannot take: at the compiled head dimensions the call is refused
    // (it would run many times slower without a word), at the others the plain kernels serve it.
    return a.head_dim == 64 || a.head_dim == 128 || !misaligned(a);
}

int attention_fwd_mfma(const AttnArgs& a, void* stream) {
    if (int rc = check(a)) return rc;
    if (misaligned(a)) return fail(CHIMERA_EINVAL, "ctx must be 8-byte aligned");
    const dim3 grid(attn_grid(a)), block(NT);
    const float sl2 = LOG2E / sqrtf((float)a.head_dim);
    hipStream_t s = (hipStream_t)stream;
#define ATTN_FWD(D, C)                                                                                            \
    hipLaunchKernelGGL((attn_fwd_kernel<D, C>), grid, block, 0, s, (const bf16_t*)a.qkv, (bf16_t*)a.ctx, a.lse, a.seq, \
                       a.heads, a.batch, a.head_dim, sl2)
    if (a.head_dim <= 64) { if (a.causal) ATTN_FWD(64, true); else ATTN_FWD(64, false); }
    else { if (a.causal) ATTN_FWD(128, true); else ATTN_FWD(128, false); }
#undef ATTN_FWD
    CHIMERA_LAUNCH_CHECK("attention forward");
    return CHIMERA_OK;
}

int attention_bwd_mfma(const AttnArgs& a, void* stream) {
    if (int rc = check(a)) return rc;
    if (misaligned(a)) return fail(CHIMERA_EINVAL, "attention buffers must be 16-byte aligned");
    hipStream_t s = (hipStream_t)stream;
    const dim3 block(NT);
    const dim3 grid(attn_grid(a)), grid2(2 * attn_grid(a));    // one role / both roles; attn_grid is a multiple of 8
    const size_t chunks = (size_t)a.batch * a.seq * a.heads * (a.head_dim <= 64 ? 8 : 16);
    const dim3 dgrid((unsigned)((chunks + NT - 1) / NT));
    const float scale = 1.0f / sqrtf((float)a.head_dim);
    // Few (sequence, head) pairs: one launch with both roles (measured: 448 workgroups per role
    // 58 -> 53 us, 256 per role at head dim 128 149 -> 119 us; 512 and more per role are faster apart).
    const bool merged = attn_grid(a) <= 480;
    // With both roles in one launch the dK/dV role can form the deltas it needs itself, once per tile of keys, where
    // attn_delta_kernel is a launch of its own and a wait for it.  That pays while the chip has room beside the
    // workgroups (one per CU and role) and a query meets few tiles: head dim 64, 2 x 128 rows of 4 heads 9.5 -> 7.6 us,
    // 2 x 200 of 5 13.0 -> 11.3, 896 of 25 (224 workgroups) 28.7 -> 28.2, with two such calls at a time 37.4 -> 36.4;
    // 2 x 632 of 25 (280) 26.6 -> 24.3 but 37.2 -> 38.8, 3 x 768 of 16 (288) 29.6 -> 28.1 but 41.4 -> 42.7, 2 x 1024 of
    // 25 (448) 72.8 -> 75.7.  At head dim 128, one wavefront per SIMD: 2 x 128 rows of 8 14.7 -> 13.2, 2 x 256 19.1 -> 18.0,
    // but 2 x 512 28.7 -> 29.4 us.
    const bool own = merged && (a.head_dim <= 64 ? attn_grid(a) <= 256 && a.seq <= 1024 : a.seq <= 256);
#define ATTN_BWD(D, C)                                                                                              \
    do {                                                                                                            \
        if (own) {                                                                                                  \
            hipLaunchKernelGGL((attn_bwd_kernel<D, C, true>), grid2, block, 0, s, (const bf16_t*)a.qkv, (const bf16_t*)a.dctx, \
                               (const bf16_t*)a.ctx, a.lse, a.delta, (bf16_t*)a.dqkv, a.seq, a.heads, a.batch, a.head_dim, scale); \
        } else if (merged) {                                                                                        \
            hipLaunchKernelGGL((attn_delta_kernel<D>), dgrid, block, 0, s, (const bf16_t*)a.dctx, (const bf16_t*)a.ctx, \
                               a.delta, a.seq, a.heads, a.batch, a.head_dim);                                                   \
            hipLaunchKernelGGL((attn_bwd_kernel<D, C, false>), grid2, block, 0, s, (const bf16_t*)a.qkv, (const bf16_t*)a.dctx, \
                               (const bf16_t*)a.ctx, a.lse, a.delta, (bf16_t*)a.dqkv, a.seq, a.heads, a.batch, a.head_dim, scale); \
        } else {                                                                                                    \
            hipLaunchKernelGGL((attn_bwd_dq_kernel<D, C>), grid, block, 0, s, (const bf16_t*)a.qkv, (const bf16_t*)a.dctx, \
                               (const bf16_t*)a.ctx, a.lse, a.delta, (bf16_t*)a.dqkv, a.seq, a.heads, a.batch, a.head_dim, scale); \
            hipLaunchKernelGGL((attn_bwd_dkv_kernel<D, C>), grid, block, 0, s, (const bf16_t*)a.qkv, (const bf16_t*)a.dctx, \
                               a.lse, a.delta, (bf16_t*)a.dqkv, a.seq, a.heads, a.batch, a.head_dim, scale);                    \
        }                                                                                                           \
    } while (0)
    if (a.head_dim <= 64) { if (a.causal) ATTN_BWD(64, true); else ATTN_BWD(64, false); }
    else { if (a.causal) ATTN_BWD(128, true); else ATTN_BWD(128, false); }
#undef ATTN_BWD
    CHIMERA_LAUNCH_CHECK("attention backward");
    return CHIMERA_OK;
}

}  // namespace chimera
