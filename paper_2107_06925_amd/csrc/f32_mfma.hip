// Float products on the CDNA4 matrix cores: v_mfma_f32_32x32x2_f32, full float operands and
// accumulation (the chip's float matrix rate is 157 TFLOP/s, twice what an LDS-fed vector loop
// reached of it and eight times the plain kernel).  Same three layouts and epilogues as the bf16
// products.
//
// Per lane l the instruction takes ONE contraction value of row (column) l%32; which contraction
// index lane group g = l/32 holds is free as long as both operands agree.  Here the k range goes in
// groups of 8: group g holds 4g..4g+3 and instruction j (0..3) contracts the pair (j, 4+j).  A
// k-contiguous operand then delivers four instructions' values with one 16-byte read; an operand
// whose other index is contiguous delivers them as four 4-byte reads of 32 neighbouring values.
//
// Three forms:
//  - tiles of 64x64, 8 wavefronts, k in steps of 32 through LDS.  A 64-clock instruction needs 8 bytes
//    from LDS per lane at most, so LDS and L2 are far from their limits and the matrix pipes set the
//    time, once the loads and LDS reads of the next steps are under way during the current one.
//  - small outputs: one 32x32 tile per workgroup, the k range dealt over 4 or 8 wavefronts, operands
//    straight from memory into registers, one exchange in LDS at the end.  Such a product is bound
//    by its chain of latencies (launch, load, exchange, store), which this keeps to one of each;
//  - the smallest outputs: the same with 16x16 tiles, which four times as many CUs read the operands of.
#include "device.h"

#include <algorithm>

namespace chimera {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NUM_CUS = 256;

// One product of a launch; a launch holds up to MAX_PRODUCTS of them, tiles laid end to end.
struct F32Product {
    const float* a; const float* b; const float* bias; const float* r; float* c; float* c2;
    float* bsum;                         // optional: bsum[j] += sum_k B(k, j)
    int m, n, k, lda, ldb, tiles_m, tiles_n, first;
};
constexpr int MAX_PRODUCTS = 4;
struct F32Launch { F32Product p[MAX_PRODUCTS]; int count, total, epi, flag; };     // flag: GeLU form, or overwrite of an accumulate

// Workgroup id -> product and tile: each XCD takes a contiguous range of the launch's tiles, walked
// in groups of 8 tile rows.
__device__ __forceinline__ const F32Product& tile_of(const F32Launch& L, int& tile_m, int& tile_n) {
    const int xcd = (int)blockIdx.x & 7, local = (int)blockIdx.x >> 3;
    const int gid = xcd * (L.total >> 3) + min(xcd, L.total & 7) + local;
    int i = 0;
#pragma unroll
    for (int q = 1; q < MAX_PRODUCTS; ++q)
        if (q < L.count && gid >= L.p[q].first) i = q;
    const F32Product& p = L.p[i];
    const int pid = gid - p.first, width = 8 * p.tiles_n, first_m = (pid / width) * 8, rows = min(p.tiles_m - first_m, 8);
    tile_m = first_m + (pid % width) % rows;
    tile_n = (pid % width) / rows;
    return p;
}

// N consecutive results of one row (columns col..col+N-1, inside the matrix)
template <int EPI, int N>
__device__ __forceinline__ void finish(const F32Product& p, int flag, int row, int col, const float* acc) {
    const size_t idx = (size_t)row * p.n + col;
    float v[N], w[N];
#pragma unroll
    for (int e = 0; e < N; ++e) {
        v[e] = acc[e];
        if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_RESIDUAL) v[e] += p.bias[col + e];
        if constexpr (EPI == EPI_BIAS_RESIDUAL) v[e] += p.r[idx + e];
        if constexpr (EPI == EPI_BIAS_GELU) w[e] = gelu_f(v[e], flag);
        if constexpr (EPI == EPI_DGELU) v[e] *= gelu_grad_f(p.r[idx + e], flag);
        if constexpr (EPI == EPI_ACCUM_F32) v[e] += flag ? 0.f : p.c[idx + e];
    }
#pragma unroll
    for (int e = 0; e < N; ++e) {
        p.c[idx + e] = v[e];
        if constexpr (EPI == EPI_BIAS_GELU) p.c2[idx + e] = w[e];
    }
}

// The same for four columns whose other operands are asked for before the k loop: a round trip less at the end of a short launch.
struct F32Ahead {
    f32x4 bias, r;
    template <int EPI> __device__ __forceinline__ void request(const F32Product& p, int flag, int row, int col) {
        const size_t idx = (size_t)row * p.n + col;
        // n is a multiple of 4, but C, R and the bias need not be aligned to 16 bytes
        typedef f32x4 __attribute__((aligned(4))) f32x4_u;
        if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_RESIDUAL) bias = *reinterpret_cast<const f32x4_u*>(p.bias + col);
        if constexpr (EPI == EPI_BIAS_RESIDUAL || EPI == EPI_DGELU) r = *reinterpret_cast<const f32x4_u*>(p.r + idx);
        if constexpr (EPI == EPI_ACCUM_F32) { r = f32x4{0.f, 0.f, 0.f, 0.f}; if (!flag) r = *reinterpret_cast<const f32x4_u*>(p.c + idx); }
    }
    template <int EPI> __device__ __forceinline__ void finish(const F32Product& p, int flag, int row, int col, const f32x4& acc) const {
        const size_t idx = (size_t)row * p.n + col;
        float v[4], w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = acc[e];
            if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_RESIDUAL) v[e] += bias[e];
            if constexpr (EPI == EPI_BIAS_RESIDUAL || EPI == EPI_ACCUM_F32) v[e] += r[e];
            if constexpr (EPI == EPI_BIAS_GELU) w[e] = gelu_f(v[e], flag);
            if constexpr (EPI == EPI_DGELU) v[e] *= gelu_grad_f(r[e], flag);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            p.c[idx + e] = v[e];
            if constexpr (EPI == EPI_BIAS_GELU) p.c2[idx + e] = w[e];
        }
    }
};

// ------------------------------------------------------------------ tile form
// LDS layout of an operand tile of ROWS rows: [ROWS][BK + 4] (k-contiguous) or [BK][ROWS + 8].  Both
// paddings make the fragment reads conflict-free on the 64 banks: 16 consecutive rows at a stride of
// 20 or 36 words cover all banks with 4 words each; the two lane groups' rows 4g+j lie
// 4 * (ROWS + 8) = 32 (mod 64) words apart.
template <int ROWS, int BK, int NT, bool KC> struct OpTile {
    static constexpr int STRIDE = KC ? BK + 4 : ROWS + 8, FLOATS = KC ? ROWS * STRIDE : BK * STRIDE;
    static constexpr int N = ROWS * BK / 4 / NT;               // 16-byte pieces per thread and step
    static_assert(N >= 1, "every thread moves a piece");
    f32x4 v[N];
    unsigned oks;                        // bit i: v[i] lies inside the matrix; the others become zeros only on
                                         // their way to LDS (a select right behind the load would wait for it)
    __device__ __forceinline__ void load(const float* __restrict__ base, int ld, int row0, int nrows, int k0, int K, int tid) {
        oks = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int c = tid + i * NT;
            const int row = row0 + (KC ? c / (BK / 4) : c % (ROWS / 4) * 4), k = k0 + (KC ? c % (BK / 4) * 4 : c / (ROWS / 4));
            const bool ok = row < nrows && k < K;
            v[i] = *reinterpret_cast<const f32x4*>(base + (ok ? (KC ? (size_t)row * ld + k : (size_t)k * ld + row) : 0));
            oks |= (ok ? 1u : 0u) << i;
        }
    }
    __device__ __forceinline__ void store(float* lds, int tid) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int c = tid + i * NT;
            const int off = KC ? c / (BK / 4) * STRIDE + c % (BK / 4) * 4 : c / (ROWS / 4) * STRIDE + c % (ROWS / 4) * 4;
            const bool ok = (oks >> i) & 1;
            *reinterpret_cast<f32x4*>(lds + off) = f32x4{ok ? v[i][0] : 0.f, ok ? v[i][1] : 0.f, ok ? v[i][2] : 0.f, ok ? v[i][3] : 0.f};
        }
    }
    // the four values of row `row` and k group `grp` (of 8) that lane group g holds
    static __device__ __forceinline__ f32x4 frag(const float* lds, int row, int grp, int g) {
        if constexpr (KC) return *reinterpret_cast<const f32x4*>(lds + row * STRIDE + grp * 8 + 4 * g);
        const float* q = lds + (grp * 8 + 4 * g) * STRIDE + row;
        return f32x4{q[0], q[STRIDE], q[2 * STRIDE], q[3 * STRIDE]};
    }
};

// Two wavefronts share a 32x32 block (TM = TN = 1), each with half of every k step: with one 64x64 tile per CU there
// is otherwise one wavefront per SIMD, and nothing runs while it waits for a barrier or LDS.
template <bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(8 * WAVE) void gemm_f32_tile_kernel(F32Launch L) {
    constexpr int BM = 64, BN = 64, BK = 32, WGK = 2, NT = 4 * WGK * WAVE, WM = BM / 2, WN = BN / 2, TM = WM / 32, TN = WN / 32, GRPS = BK / 8 / WGK;
    using TA = OpTile<BM, BK, NT, A_KC>;
    using TB = OpTile<BN, BK, NT, B_KC>;
    __shared__ __attribute__((aligned(16))) float lds[3][TA::FLOATS + TB::FLOATS];
    int tile_m, tile_n;
    const F32Product& p = tile_of(L, tile_m, tile_n);
    const int i0 = tile_m * BM, j0 = tile_n * BN, m = p.m, n = p.n, K = p.k, lda = p.lda, ldb = p.ldb;
    const float* __restrict__ A = p.a;
    const float* __restrict__ B = p.b;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave >> 2, wm0 = ((wave >> 1) & 1) * WM, wn0 = (wave & 1) * WN;

    f32x16 acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
    // column sums of B come from the fragments that the top wavefronts of the first tile row hold anyway
    const bool col_sums = EPI == EPI_ACCUM_F32 && p.bsum && tile_m == 0 && wm0 == 0;
    float cs[TN];
#pragma unroll
    for (int b = 0; b < TN; ++b) cs[b] = 0.f;

    // Loads run in register sets three steps ahead of LDS (a step is 0.4 us of matrix work, a load that
    // misses L2 takes twice that) and LDS two steps ahead of the matrix cores, in rings of three walked
    // by an unrolled loop.  With LDS that far ahead the first fragments of the next step are read
    // before the barrier that ends this one.
    constexpr int NB = 3;
    TA ra[NB];
    TB rb[NB];
    const int KT = (K + BK - 1) / BK;
    auto fetch = [&](int u, int kt) {
        ra[u].load(A, lda, i0, m, kt * BK, K, tid);
        rb[u].load(B, ldb, j0, n, kt * BK, K, tid);
    };
    auto stash = [&](int u) {
        ra[u].store(lds[u], tid);
        rb[u].store(lds[u] + TA::FLOATS, tid);
    };
    f32x4 fa[2][TM], fb[2][TN];
    auto read = [&](int s, int buf, int gi) {
        const int grp = wk * GRPS + gi;
#pragma unroll
        for (int a = 0; a < TM; ++a) fa[s][a] = TA::frag(lds[buf], wm0 + a * 32 + l32, grp, g);
#pragma unroll
        for (int b = 0; b < TN; ++b) fb[s][b] = TB::frag(lds[buf] + TA::FLOATS, wn0 + b * 32 + l32, grp, g);
    };
#pragma unroll
    for (int u = 0; u < NB; ++u)
        if (u < KT) fetch(u, u);
    stash(0);
    if (1 < KT) stash(1);
    if (3 < KT) fetch(0, 3);
    if (4 < KT) fetch(1, 4);
    __syncthreads();
    read(0, 0, 0);
    static_assert(GRPS % 2 == 0, "fragment set of a group at compile time");
    for (int kt0 = 0; kt0 < KT; kt0 += NB) {
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int kt = kt0 + u;
            if (kt >= KT) break;
            if (kt + 2 < KT) stash((u + 2) % NB);            // its buffer was last read in step kt - 1
            if (kt + 5 < KT) fetch((u + 2) % NB, kt + 5);
#pragma unroll
            for (int gi = 0; gi < GRPS; ++gi) {
                const int s = gi & 1;
                if (gi + 1 < GRPS) read(s ^ 1, u, gi + 1);
                else if (kt + 1 < KT) read(s ^ 1, (u + 1) % NB, 0);
                if constexpr (EPI == EPI_ACCUM_F32)
                    if (col_sums)
#pragma unroll
                        for (int b = 0; b < TN; ++b) cs[b] += (fb[s][b][0] + fb[s][b][1]) + (fb[s][b][2] + fb[s][b][3]);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int a = 0; a < TM; ++a)
#pragma unroll
                        for (int b = 0; b < TN; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[s][a][j], fb[s][b][j], acc[a][b], 0, 0, 0);
            }
            __syncthreads();                   // step kt + 2 is in LDS, and everyone is done with step kt
        }
    }
    // Two wavefronts with partial sums of one block: each hands over one half of its registers and
    // finishes the other (registers 0..7 or 8..15 of every 32x32 tile, i.e. 16 of its rows).
    constexpr int R = 16 / WGK;
    {
        static_assert(TM == 1 && TN == 1, "one tile per wavefront");
        static_assert(sizeof(lds) >= 8 * R * WAVE * sizeof(float) + BN * sizeof(float), "LDS too small for the exchange");
        float* xch = &lds[0][0];
        float* xcs = xch + 8 * R * WAVE;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) xch[(wave * R + r) * WAVE + lane] = wk ? acc[0][0][r] : acc[0][0][R + r];
        if (col_sums) {
            cs[0] = sum32(cs[0]);
            if (wk && g == 0) xcs[wn0 + l32] = cs[0];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float other = xch[((wave ^ 4) * R + r) * WAVE + lane];
            acc[0][0][r] = wk ? other + acc[0][0][R + r] : acc[0][0][r] + other;
        }
        if (col_sums && !wk) cs[0] += xcs[wn0 + l32];
    }
    // register r of lane l: row 8(r/4) + 4g + r%4, column l%32 - 128 contiguous bytes per half wavefront
#pragma unroll
    for (int b = 0; b < TN; ++b) {
        const int col = j0 + wn0 + b * 32 + l32;
        if (col >= n) continue;
        if constexpr (EPI == EPI_ACCUM_F32)
            if (col_sums && g == 0 && wk == 0) p.bsum[col] = L.flag ? cs[b] : p.bsum[col] + cs[b];
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int row = i0 + wm0 + a * 32 + wk * 16 + 8 * (r >> 2) + 4 * g + (r & 3);
                const float v = acc[a][b][r];
                if (row < m) finish<EPI, 1>(p, L.flag, row, col, &v);
            }
    }
}

// ----------------------------------------------------------------- small form
// The 32 k values a wavefront takes at a time, of one operand row per lane: 16 registers.  Rows
// beyond the matrix repeat its last one (their results are not stored); k beyond the range becomes
// zero at use.
template <bool KC>
__device__ __forceinline__ void load_slice(f32x4 (&v)[4], const float* __restrict__ base, int ld, int row, int k0, int K, int g) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = k0 + 8 * i + 4 * g;
        if constexpr (KC) v[i] = *reinterpret_cast<const f32x4*>(base + (size_t)row * ld + min(k, K - 4));
        else
#pragma unroll
            for (int j = 0; j < 4; ++j) v[i][j] = base[(size_t)min(k + j, K - 1) * ld + row];
    }
}
__device__ __forceinline__ void mask_slice(f32x4 (&v)[4], int k0, int K, int g) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) v[i][j] = k0 + 8 * i + 4 * g + j < K ? v[i][j] : 0.f;
}

template <int NW, bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(NW* WAVE) void gemm_f32_small_kernel(F32Launch L) {
    __shared__ __attribute__((aligned(16))) float red[NW][32 * 32];
    __shared__ float red_cs[NW][32];
    int tile_m, tile_n;
    const F32Product& p = tile_of(L, tile_m, tile_n);
    const int m = p.m, n = p.n, K = p.k, lda = p.lda, ldb = p.ldb;
    const float* __restrict__ A = p.a;
    const float* __restrict__ B = p.b;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = min(tile_m * 32 + l32, m - 1), col = min(tile_n * 32 + l32, n - 1);
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    float cs = 0.f;
    f32x4 fa[2][4], fb[2][4];
    const int k_first = wave * 32, k_step = NW * 32;
    auto fetch = [&](int s, int k0) {
        load_slice<A_KC>(fa[s], A, lda, row, k0, K, g);
        load_slice<B_KC>(fb[s], B, ldb, col, k0, K, g);
    };
    auto work = [&](int s, int k0) {
        if (k0 + 32 > K) { mask_slice(fa[s], k0, K, g); mask_slice(fb[s], k0, K, g); }     // uniform: the last slice only
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (EPI == EPI_ACCUM_F32) cs += (fb[s][i][0] + fb[s][i][1]) + (fb[s][i][2] + fb[s][i][3]);
#pragma unroll
            for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[s][i][j], fb[s][i][j], acc, 0, 0, 0);
        }
    };
    if (k_first < K) {
        fetch(0, k_first);
        for (int k0 = k_first; k0 < K; k0 += 2 * k_step) {
            if (k0 + k_step < K) fetch(1, k0 + k_step);
            work(0, k0);
            if (k0 + k_step >= K) break;
            if (k0 + 2 * k_step < K) fetch(0, k0 + 2 * k_step);
            work(1, k0 + k_step);
        }
    }
    // partial tiles meet in LDS; thread t finishes four columns of one row, adding in wavefront order
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wave][(8 * (r >> 2) + 4 * g + (r & 3)) * 32 + l32] = acc[r];
    const bool col_sums = EPI == EPI_ACCUM_F32 && p.bsum && tile_m == 0;
    if constexpr (EPI == EPI_ACCUM_F32)
        if (col_sums) {
            cs = sum32(cs);
            if (g == 0) red_cs[wave][l32] = cs;
        }
    __syncthreads();
    if (tid < 256) {
        const int rr = tid >> 3, cc = (tid & 7) * 4, orow = tile_m * 32 + rr, ocol = tile_n * 32 + cc;
        f32x4 s = *reinterpret_cast<const f32x4*>(&red[0][rr * 32 + cc]);
#pragma unroll
        for (int w = 1; w < NW; ++w) s += *reinterpret_cast<const f32x4*>(&red[w][rr * 32 + cc]);
        const float v[4] = {s[0], s[1], s[2], s[3]};
        if (orow < m && ocol < n) finish<EPI, 4>(p, L.flag, orow, ocol, v);       // n is a multiple of 8
        if constexpr (EPI == EPI_ACCUM_F32)
            if (col_sums && tid < 32 && tile_n * 32 + tid < n) {
                float t = red_cs[0][tid];
#pragma unroll
                for (int w = 1; w < NW; ++w) t += red_cs[w][tid];
                float* o = p.bsum + tile_n * 32 + tid;
                *o = L.flag ? t : *o + t;
            }
    }
}

// The smallest outputs: one 16x16 tile per workgroup on v_mfma_f32_16x16x4_f32 (lane group l/16 holds contraction values
// 4(l/16)..+3 of a group of 16, instruction j the j-th of each), k dealt over the wavefronts 32 at a time, operands straight
// from memory.  What such a launch waits for is what one CU reads (60 to 90 bytes a nanosecond) and a wavefront's chain of matrix
// instructions: both are half, or a quarter, of a 32x32 tile's.
template <int NW, bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(NW* WAVE) void gemm_f32_tiny_kernel(F32Launch L) {
    __shared__ __attribute__((aligned(16))) float red[NW][16 * 16];
    int tile_m, tile_n;
    const F32Product& p = tile_of(L, tile_m, tile_n);
    const int m = p.m, n = p.n, K = p.k, lda = p.lda, ldb = p.ldb;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = min(tile_m * 16 + l16, m - 1), col = min(tile_n * 16 + l16, n - 1);
    // thread t finishes four columns of one row
    const int orow = tile_m * 16 + (tid >> 2), ocol = tile_n * 16 + (tid & 3) * 4;
    const bool finishes = tid < 64 && orow < m && ocol < n;
    F32Ahead ahead;
    if (finishes) ahead.request<EPI>(p, L.flag, orow, ocol);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    f32x4 fa[2][2], fb[2][2];
    // values 16 i + 4 g .. + 3 of 32 from k0 on (beyond K: the last ones, masked later)
    auto load = [&](f32x4 (&v)[2], const float* __restrict__ base, bool kc, int ld, int r, int k0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int k = k0 + 16 * i + 4 * g;
            if (kc) v[i] = *reinterpret_cast<const f32x4*>(base + (size_t)r * ld + min(k, K - 4));
            else
#pragma unroll
                for (int j = 0; j < 4; ++j) v[i][j] = base[(size_t)min(k + j, K - 1) * ld + r];
        }
    };
    auto fetch = [&](int s, int k0) { load(fa[s], p.a, A_KC, lda, row, k0); load(fb[s], p.b, B_KC, ldb, col, k0); };
    auto work = [&](int s, int k0) {
        if (k0 + 32 > K)                                          // uniform: the last slice only
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (k0 + 16 * i + 4 * g + j >= K) { fa[s][i][j] = 0.f; fb[s][i][j] = 0.f; }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[s][i][j], fb[s][i][j], acc, 0, 0, 0);
    };
    const int k_first = wave * 32, k_step = NW * 32;
    if (k_first < K) {
        fetch(0, k_first);
        for (int k0 = k_first; k0 < K; k0 += 2 * k_step) {
            if (k0 + k_step < K) fetch(1, k0 + k_step);
            work(0, k0);
            if (k0 + k_step >= K) break;
            if (k0 + 2 * k_step < K) fetch(0, k0 + 2 * k_step);
            work(1, k0 + k_step);
        }
    }
    // partial tiles meet in LDS, added in wavefront order
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][(4 * g + r) * 16 + l16] = acc[r];
    __syncthreads();
    if (finishes) {
        f32x4 s = *reinterpret_cast<const f32x4*>(&red[0][tid * 4]);
#pragma unroll
        for (int w = 1; w < NW; ++w) s += *reinterpret_cast<const f32x4*>(&red[w][tid * 4]);
        ahead.finish<EPI>(p, L.flag, orow, ocol, s);
    }
}

enum Form { TILE64, SMALL, TINY };

// Up to two 16x16 tiles per CU take the tiny form.  32x32 -> 16x16: 128 x 384 x 128 3.2 -> 2.4 us, 128 x 128 x 512 (64 tiles) 5.8 -> 3.3 with
// residual, 6.6 -> 3.9 A B^T, 256 x 256 x 1024 (256) 10.5 -> 5.7, 300 x 320 x 1280 (380) 12.6 -> 10.7, 512 x 256 x 256 (512) 4.2 -> 3.4,
// x 1024 10.6 -> 9.2.
constexpr long TINY_TILES = 2 * NUM_CUS;

// Form of a launch.  Up to half a 64x64 tile per CU the small form's 32x32 tiles spread the work
// further (512 x 1024 x 1024, 128 tiles: 20 against 23 us; 300 x 640 x 640, 50 tiles: 9.6 against 16);
// beyond that the tile form's shared operands win (1000 x 640 x 2560, 160 tiles: 53 against 66 us;
// 1024 x 1024 x 4096, 256 tiles: 85 against 140 us, 101 TFLOP/s; 2048^3: 160 us, 107 TFLOP/s).  128x128
// tiles were 5 % faster at 4096 x 4096 x 1024 k-contiguous and slower everywhere else.
Form choose_form(int count, const GemmArgs* g) {
    long t64 = 0;
    for (int i = 0; i < count; ++i) t64 += (long)((g[i].m + 63) / 64) * ((g[i].n + 63) / 64);
    return t64 <= NUM_CUS / 2 ? SMALL : TILE64;
}

template <bool A_KC, bool B_KC, int EPI>
int launch_form(F32Launch& L, Form form, hipStream_t s) {
    if (!A_KC && form == TINY) return fail(CHIMERA_EINVAL, "no 16x16 tile for weight gradients");       // (those go in groups, which are larger)
    const int tile = form == TILE64 ? 64 : form == SMALL ? 32 : 16;
    L.total = 0;
    int kmax = 0;
    for (int i = 0; i < L.count; ++i) {
        F32Product& p = L.p[i];
        p.tiles_m = (p.m + tile - 1) / tile;
        p.tiles_n = (p.n + tile - 1) / tile;
        p.first = L.total;
        L.total += p.tiles_m * p.tiles_n;
        kmax = std::max(kmax, p.k);
    }
    const dim3 grid(L.total);
    if (form == TILE64) hipLaunchKernelGGL((gemm_f32_tile_kernel<A_KC, B_KC, EPI>), grid, dim3(8 * WAVE), 0, s, L);
    else if (form == TINY) {
        if constexpr (A_KC) {
            if (kmax <= 128) hipLaunchKernelGGL((gemm_f32_tiny_kernel<4, A_KC, B_KC, EPI>), grid, dim3(4 * WAVE), 0, s, L);
            else hipLaunchKernelGGL((gemm_f32_tiny_kernel<8, A_KC, B_KC, EPI>), grid, dim3(8 * WAVE), 0, s, L);
        }
    } else if (kmax <= 256) hipLaunchKernelGGL((gemm_f32_small_kernel<4, A_KC, B_KC, EPI>), grid, dim3(4 * WAVE), 0, s, L);
    else hipLaunchKernelGGL((gemm_f32_small_kernel<8, A_KC, B_KC, EPI>), grid, dim3(8 * WAVE), 0, s, L);
    CHIMERA_LAUNCH_CHECK("float gemm");
    return CHIMERA_OK;
}

template <bool A_KC, bool B_KC>
int launch_epi(F32Launch& L, Form form, hipStream_t s) {
    switch (L.epi) {
        case EPI_NONE: return launch_form<A_KC, B_KC, EPI_NONE>(L, form, s);
        case EPI_BIAS: return launch_form<A_KC, B_KC, EPI_BIAS>(L, form, s);
        case EPI_BIAS_GELU: return launch_form<A_KC, B_KC, EPI_BIAS_GELU>(L, form, s);
        case EPI_BIAS_RESIDUAL: return launch_form<A_KC, B_KC, EPI_BIAS_RESIDUAL>(L, form, s);
        case EPI_DGELU: return launch_form<A_KC, B_KC, EPI_DGELU>(L, form, s);
        default: return launch_form<A_KC, B_KC, EPI_ACCUM_F32>(L, form, s);
    }
}

F32Product product_of(const GemmArgs& g) {
    F32Product p{};
    p.a = (const float*)g.a; p.b = (const float*)g.b; p.bias = (const float*)g.bias; p.r = (const float*)g.r;
    p.c = (float*)g.c; p.c2 = (float*)g.c2;
    p.m = g.m; p.n = g.n; p.k = g.k; p.lda = g.lda; p.ldb = g.ldb;
    return p;
}

}  // namespace

// 16-byte pieces: aligned operands, leading dimensions (and a contiguous k, and the row count of an
// index-contiguous A) in multiples of 4; n in multiples of 4 for the small form's output pieces.
bool gemm_f32_supports(const GemmArgs& g) {
    if (!g.a_kc && g.b_kc) return false;                       // layout no linear layer needs
    if (g.m < 1 || g.n < 1 || g.k < 1 || (g.n % 4) || (g.lda % 4) || (g.ldb % 4)) return false;
    if ((g.a_kc || g.b_kc) && (g.k % 4)) return false;
    if (!g.a_kc && (g.m % 4)) return false;
    return !(((uintptr_t)g.a | (uintptr_t)g.b) & 15) && (long)((g.m + 31) / 32) * ((g.n + 31) / 32) < (1l << 30);
}

int gemm_f32(const GemmArgs& g, void* stream) {
    if (!gemm_f32_supports(g)) return fail(CHIMERA_EINVAL, "float matrix-core gemm: unsupported shape or layout");
    if (g.epilogue < EPI_NONE || g.epilogue > EPI_ACCUM_F32) return fail(CHIMERA_EINVAL, "unknown epilogue %d", g.epilogue);
    F32Launch L{};
    L.count = 1; L.epi = g.epilogue; L.flag = g.epilogue == EPI_ACCUM_F32 ? 0 : g.gelu_erf;
    L.p[0] = product_of(g);
    Form form = choose_form(1, &g);
    if (g.a_kc && (long)((g.m + 15) / 16) * ((g.n + 15) / 16) <= TINY_TILES) form = TINY;
    hipStream_t s = (hipStream_t)stream;
    if (!g.a_kc) return launch_epi<false, false>(L, form, s);
    return g.b_kc ? launch_epi<true, true>(L, form, s) : launch_epi<true, false>(L, form, s);
}

bool gemm_f32_group_supports(int count, const GemmArgs* g) {
    if (count < 1 || count > MAX_PRODUCTS) return false;
    for (int i = 0; i < count; ++i)
        if (g[i].a_kc || g[i].b_kc || g[i].epilogue != EPI_ACCUM_F32 || !gemm_f32_supports(g[i])) return false;
    return true;
}

int gemm_f32_group(int count, const GemmArgs* g, float* const* bsum, int overwrite, void* stream) {
    if (!gemm_f32_group_supports(count, g)) return fail(CHIMERA_EINVAL, "float gemm group: unsupported shapes or layouts");
    F32Launch L{};
    L.count = count; L.epi = EPI_ACCUM_F32; L.flag = overwrite ? 1 : 0;
    for (int i = 0; i < count; ++i) { L.p[i] = product_of(g[i]); L.p[i].bsum = bsum ? bsum[i] : nullptr; }
    return launch_form<false, false, EPI_ACCUM_F32>(L, choose_form(count, g), (hipStream_t)stream);
}

}  // namespace chimera
