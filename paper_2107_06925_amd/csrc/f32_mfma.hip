// Float products on the CDNA4 matrix cores, same three layouts and epilogues as the bf16 products.  Four forms:
//  - tiles of 128x128 and 64x64 on the bf16 instructions, each float split into three bf16 numbers: six products where the float
//    instruction makes one, at 16 times its rate;
//  - small outputs: one 32x32 tile per workgroup on v_mfma_f32_32x32x2_f32, the k range dealt over 4 or 8 wavefronts, operands
//    straight from memory into registers, one exchange in LDS at the end.  Such a product is bound
//    by its chain of latencies (launch, load, exchange, store), which this keeps to one of each;
//  - the smallest outputs: the same with 16x16 tiles, which four times as many CUs read the operands of.
//
// Per lane l the float instruction takes ONE contraction value of row (column) l%32; which contraction
// index lane group g = l/32 holds is free as long as both operands agree.  Here the k range goes in
// groups of 8: group g holds 4g..4g+3 and instruction j (0..3) contracts the pair (j, 4+j).  A
// k-contiguous operand then delivers four instructions' values with one 16-byte read; an operand
// whose other index is contiguous delivers them as four 4-byte reads of 32 neighbouring values.
#include "device.h"

#include <algorithm>
#include <type_traits>

namespace chimera {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));

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

// One result whose other operands are there: the bias, and the residual, the GeLU's input or what the result is added to
template <int EPI> __device__ __forceinline__ void finish_one(const F32Product& p, int flag, size_t idx, float v, float bias, float other) {
    if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_RESIDUAL) v += bias;
    if constexpr (EPI == EPI_BIAS_RESIDUAL || EPI == EPI_ACCUM_F32) v += other;
    if constexpr (EPI == EPI_DGELU) v *= gelu_grad_f(other, flag);
    p.c[idx] = v;
    if constexpr (EPI == EPI_BIAS_GELU) p.c2[idx] = gelu_f(v, flag);
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

// ------------------------------------------------------------------ tile forms
// On the bf16 matrix instructions.  A float is the sum of three bf16 numbers: itself to nearest, the rest to nearest, and what that leaves
// (8 + 8 + 8 bits), so a product of two floats is nine products of their parts.  The three smallest are left out: at most 2^-24 of it, one
// rounding (a first part cut off instead leaves up to 2^-22, all of one sign for some operands).  A bf16 instruction rounds once for 16
// products where the float one rounds for every second: against float64, relative 2-norm of random operands, k = 64, 256, 1024, 4096:
// 1.06e-7 -> 4.8e-8, 2.06e-7 -> 7.1e-8, 4.06e-7 -> 1.30e-7, 8.10e-7 -> 2.74e-7 (128x128 tiles, whose sums are not halved, from 256 on:
// 8.9e-8, 1.86e-7, 3.96e-7); all elements 1.0077362: 5.7e-9 at every k, 2.3e-7 with a first part cut off.  The sums of the large parts'
// products and of the others are kept apart until the end.
//
// What bounds it: with two wavefronts on a SIMD matrix and vector instructions overlap by a third at best (8 of the former alone 140 ns, 64
// of the latter 148, both 202), and a 64x64 step of 32 k is 12 and 100 of them; LDS is busy 44 % of the time, without conflicts.  Against
// tiles of v_mfma_f32_32x32x2_f32, which were bound by that instruction: 1024 x 1024 x 1024 A B 24.1 -> 20.0 us, A B^T 23.3 -> 18.5, A^T B
// 26.9 -> 19.1; 1024 x 3072 x 1024 62.0 -> 47.4; 704 x 2816 x 704 30.9 -> 22.7; two steps of k, 1024 x 1024 x 64, 5.17 either way.
// Splitting in registers, a wavefront per k slice of a whole tile, was slower (2048^3 118 -> 161 us: no registers are left to load ahead).
struct SplitBuf { bf16_t part[2][3][64][32]; };                // operand, part, row, k: one step
// 16-byte chunk c (8 k values) of row r sits at c ^ bits of r: 16 rows of one chunk, as many of four rows, all fall on different banks
__device__ __forceinline__ int split_chunk(int row, int c) { return c ^ ((row >> 2) & 3); }

// The chunks a thread moves: 8 k values of one operand row in every step of BK.  Buffer loads: an address is a uniform base, which moves on
// by a step, and an offset that stays the same; what lies beyond the operand's end reads as zero, as the k rows behind K of an
// index-contiguous operand do.  (In a row of a k-contiguous one, others follow.)
template <bool KC, int BK> struct SplitChunk {
    const char* at;                       // the tile's first row, this step's first k
    size_t step;
    int ld, rows, left;                   // left: k values from this step on
    unsigned off[KC ? 1 : 8];
    __device__ __forceinline__ SplitChunk(const float* from, int ld, int row0, int nrows, int max_rows, int K, int row, int oct)
        : at((const char*)(from + (KC ? (size_t)row0 * ld : row0))), step((KC ? (size_t)BK : (size_t)BK * ld) * 4), ld(ld), rows(min(nrows - row0, max_rows)), left(K) {
        row = min(row, rows - 1);         // rows beyond the matrix repeat its last one: their results are not stored
#pragma unroll
        for (int j = 0; j < (KC ? 1 : 8); ++j) off[j] = (KC ? (unsigned)row * (unsigned)ld + oct * 8 : (unsigned)(oct * 8 + j) * (unsigned)ld + row) * 4u;
    }
    __device__ __forceinline__ void load(float (&v)[8]) {
        const int elems = KC ? (rows - 1) * ld + left : min(left, BK) * ld;
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)at, 0, (int)(4u * max(elems, 0)), 0x00020000);
        if constexpr (KC) {
            const f32x4 lo = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off[0], 0, 0));
            const f32x4 hi = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off[0] + 16, 0, 0));
#pragma unroll
            for (int j = 0; j < 4; ++j) { v[j] = lo[j]; v[4 + j] = hi[j]; }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, off[j], 0, 0));
        }
        at += step; left -= BK;
    }
};
constexpr int MAX_LD = 1 << 22;                                // 128 rows, or 32 k, of them stay below 2^31 bytes

// Writes a chunk's parts, part p at `at` + p * PART.  `rest` takes in the third parts, whose lower halves are not stored: see loses.
template <int PART> __device__ __forceinline__ void split_store(const float (&v)[8], bf16_t* at, unsigned& rest) {
    typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
    unsigned w[3][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const unsigned top = __builtin_bit_cast(unsigned, bf16x2{(bf16_t)v[2 * j], (bf16_t)v[2 * j + 1]});
        const float rx = v[2 * j] - __uint_as_float(top << 16), ry = v[2 * j + 1] - __uint_as_float(top & 0xffff0000u);
        const unsigned mid = __builtin_bit_cast(unsigned, bf16x2{(bf16_t)rx, (bf16_t)ry});
        const unsigned lx = __float_as_uint(rx - __uint_as_float(mid << 16)), ly = __float_as_uint(ry - __uint_as_float(mid & 0xffff0000u));
        w[0][j] = top;
        w[1][j] = mid;
        w[2][j] = __builtin_amdgcn_perm(ly, lx, 0x07060302u);
        rest |= lx | ly;
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<uint4*>(at + p * PART) = make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]);
}
// A third part has no more than eight bits, which bf16 holds, unless some lie below its smallest step, 2^-133: parts of a float from 2^-110
// on are exact (the matrix instructions keep subnormal operands and sums), and one smaller number that is not is seen here, whatever lies
// beside it.  (Operands split as 2^16 times what they are would all be exact, but take a multiplication each: 2 to 10 % of every product.)
__device__ __forceinline__ bool loses(unsigned rest) { return rest & 0xffff; }
// Whether that can matter to a result: each of a product's k terms lost less than 2^-133 times its other factor, of which `a` and `b` are the
// largest of the result's row and column.  What is below a quarter of a rounding of the result is let pass: one GeLU of -10 among
// ordinary numbers would otherwise have its tiles formed again.  Such numbers in every tile, formed again -> looked at like this, 2048^3
// A B 283 -> 166 us, A B^T 246 -> 153, A^T B 257 -> 186 (none: 98, 97, 108); 1024^3 52 -> 25, 47 -> 24, 56 -> 25 (18.3, 17.9, 18.9).  A sum
// that comes to zero by chance has its tile formed again.
__device__ __forceinline__ bool matters(float result, float a, float b, int k) {
    return a > 0.f && b > 0.f && !(fabsf(result) >= fmaxf(a, b) * ((float)k * 0x1p-106f));
}
// The largest value of the chunks that a thread stages, into `to`, of the chunks' row.  Not unrolled: by four, 2048^3 with small numbers
// 166 -> 124 us, but the kernels' code is longer, and a worker of 192-wide float blocks, none of whose numbers are small, 14.2 -> 14.5 ms.
template <bool KC, int BK> __device__ __forceinline__ void largest(SplitChunk<KC, BK> chunk, int steps, unsigned* to) {
    float most = 0.f;
#pragma unroll 1
    for (int kt = 0; kt < steps; ++kt) {
        float v[8];
        chunk.load(v);
#pragma unroll
        for (int j = 0; j < 8; ++j) most = fmaxf(most, fabsf(v[j]));
    }
    atomicMax(to, __float_as_uint(most));                        // (not negative: ordered as integers too)
}

// Asks the scheduler for one order of a step's instructions: the LDS reads, FIRST matrix instructions, then one of them behind every VALUS
// vector instructions of the split.  Its own order has most matrix instructions first and the split behind them.  1024 x 1024 x 1024 A B
// 21.5 -> 20.1 us, A B^T 19.6 -> 18.3; 2048^3 103 -> 95, A B^T 105 -> 92, A^T B 112 -> 102.  (64x64 tiles of A^T B are faster in its own
// order: 19.5 against 19.9 to 21.0.)
template <int READS, int FIRST, int REST, int VALUS> __device__ __forceinline__ void interleave() {
    __builtin_amdgcn_sched_group_barrier(0x100, READS, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, FIRST, 0);
#pragma unroll
    for (int i = 0; i < REST; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x002, VALUS, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
}

// 8 wavefronts: two share a 32x32 block, each with half of every k step; four stage A's rows, four B's.
template <bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(8 * WAVE, 4) void gemm_f32_tile_kernel(F32Launch L) {
    constexpr int BM = 64, BN = 64, BK = 32;
    __shared__ __attribute__((aligned(16))) SplitBuf lds[2];
    int tile_m, tile_n;
    const F32Product& p = tile_of(L, tile_m, tile_n);
    const int i0 = tile_m * BM, j0 = tile_n * BN, m = p.m, n = p.n, K = p.k, lda = p.lda, ldb = p.ldb;
    const float* __restrict__ A = p.a;
    const float* __restrict__ B = p.b;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave >> 2, wm0 = ((wave >> 1) & 1) * 32, wn0 = (wave & 1) * 32;

    // Each thread stages one chunk a step.  Rows beyond the matrix repeat its last one (their results are not stored).
    const bool stages_a = wave < 4;
    constexpr bool GROUPED = EPI == EPI_ACCUM_F32 && !A_KC && !B_KC;        // only those have column sums
    const bool col_sums = GROUPED && p.bsum && tile_m == 0;
    constexpr int STEP = sizeof(SplitBuf) / sizeof(bf16_t), PART = 64 * BK;
    constexpr int D = 2;                                         // steps that loads run ahead (four, A^T B: 19.5 -> 20.4 us)
    const int KT = (K + BK - 1) / BK;
    float cs = 0.f;
    unsigned rest = 0;
    f32x16 acc, low;                                             // the large parts' products, and the others
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = low[r] = 0.f;
    const bf16_t* const get_a = &lds[0].part[0][0][wm0 + l32][split_chunk(wm0 + l32, 2 * wk + g) * 8];
    const bf16_t* const get_b = &lds[0].part[1][0][wn0 + l32][split_chunk(wn0 + l32, 2 * wk + g) * 8];
    // register r of lane l: row 8(r/4) + 4g + r%4, column l%32 - 128 contiguous bytes per half wavefront
    constexpr int R = 8;
    const int col = j0 + wn0 + l32;
    auto row_of = [&](int r) { return i0 + wm0 + wk * 16 + 8 * (r >> 2) + 4 * g + (r & 3); };
    // what the epilogue reads is asked for behind the last requests of the loop
    constexpr bool READS = EPI == EPI_BIAS_RESIDUAL || EPI == EPI_DGELU || EPI == EPI_ACCUM_F32;
    float bias = 0.f, other[R];
    auto ask = [&] {
        const int c = min(col, n - 1);
        if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_RESIDUAL) bias = p.bias[c];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            other[r] = 0.f;
            if (READS && !(EPI == EPI_ACCUM_F32 && L.flag)) other[r] = (EPI == EPI_ACCUM_F32 ? p.c : p.r)[(size_t)min(row_of(r), m - 1) * n + c];
        }
    };
    auto steps = [&](auto kc_c, auto sums_c, const float* __restrict__ from, int ld, int row0, int rows) {
        constexpr bool KC = decltype(kc_c)::value, SUMS = decltype(sums_c)::value;
        const int srow = KC ? (tid & 255) >> 2 : lane, oct = KC ? tid & 3 : wave & 3;
        SplitChunk<KC, BK> chunk(from, ld, row0, rows, BM, K, srow, oct);
        bf16_t* const put = &lds[0].part[stages_a ? 0 : 1][0][srow][split_chunk(srow, oct) * 8];
        float v[D][8];
        auto stash = [&](int u, int kt, auto last_c) {
            if (KC && decltype(last_c)::value && kt * BK + BK > K)
#pragma unroll
                for (int j = 0; j < 8; ++j) v[u][j] = kt * BK + oct * 8 + j < K ? v[u][j] : 0.f;
            if (SUMS) cs += ((v[u][0] + v[u][1]) + (v[u][2] + v[u][3])) + ((v[u][4] + v[u][5]) + (v[u][6] + v[u][7]));
            split_store<PART>(v[u], put + (u & 1) * STEP, rest);
        };
        auto multiply = [&](int buf) {
            bf16x8 fa[3], fb[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                fa[q] = *reinterpret_cast<const bf16x8*>(get_a + buf * STEP + q * PART);
                fb[q] = *reinterpret_cast<const bf16x8*>(get_b + buf * STEP + q * PART);
            }
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0], fb[0], acc, 0, 0, 0);
            low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0], fb[1], low, 0, 0, 0);
            low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[1], fb[0], low, 0, 0, 0);
            low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[1], fb[1], low, 0, 0, 0);
            low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0], fb[2], low, 0, 0, 0);
            low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[2], fb[0], low, 0, 0, 0);
        };
        static_assert(D % 2 == 0, "buffer of a step at compile time");
#pragma unroll
        for (int u = 0; u < D; ++u) chunk.load(v[u]);
        stash(0, 0, std::true_type{});
        chunk.load(v[0]);
        __syncthreads();
        // A step multiplies one buffer while the next step's chunks, loaded D steps ago, go to the other.
        int kt = 0;
        for (; kt + D + 1 < KT; kt += D)
#pragma unroll
            for (int u = 0; u < D; ++u) {
                multiply(u & 1);
                stash((u + 1) % D, kt + u + 1, std::false_type{});
                chunk.load(v[(u + 1) % D]);
                if constexpr (A_KC && B_KC) interleave<6, 1, 5, 8>();
                else if constexpr (A_KC && !KC) interleave<6, 2, 4, 13>();
                __syncthreads();
            }
        ask();
#pragma unroll
        for (int u = 0; u <= D; ++u) {
            if (kt + u >= KT) break;
            multiply(u & 1);
            if (kt + u + 1 < KT) stash((u + 1) % D, kt + u + 1, std::true_type{});
            __syncthreads();
        }
        if (SUMS && !stages_a) reinterpret_cast<float*>(lds)[8 * 8 * WAVE + oct * BN + srow] = cs;      // behind the exchange of sums
    };
    auto chunks_largest = [&](auto kc_c, const float* __restrict__ from, int ld, int row0, int rows, unsigned* to) {
        constexpr bool KC = decltype(kc_c)::value;
        const int srow = KC ? (tid & 255) >> 2 : lane, oct = KC ? tid & 3 : wave & 3;
        largest(SplitChunk<KC, BK>(from, ld, row0, rows, BM, K, srow, oct), KT, to + srow);
    };
    // Wavefronts of A and of B may take different arms, each with its own barriers: one before the loop and one behind each of the KT steps in both.
    auto roles = [&](auto sums_c) {
        if constexpr (A_KC == B_KC) steps(std::bool_constant<A_KC>{}, sums_c, stages_a ? A : B, stages_a ? lda : ldb, stages_a ? i0 : j0, stages_a ? m : n);
        else if (stages_a) steps(std::bool_constant<A_KC>{}, std::false_type{}, A, lda, i0, m);
        else steps(std::bool_constant<B_KC>{}, std::false_type{}, B, ldb, j0, n);
    };
    if constexpr (GROUPED) {
        if (col_sums) roles(std::true_type{});
        else roles(std::false_type{});
    } else roles(std::false_type{});
    // Two wavefronts with partial sums of one block: each hands over one half of its registers and
    // finishes the other (registers 0..7 or 8..15, i.e. 16 of its rows).
    static_assert(sizeof(lds) >= (8 * R * WAVE + 4 * BN + 8 + BM + BN) * sizeof(float), "LDS too small for the exchange");
    float* xch = reinterpret_cast<float*>(lds);
    float* xcs = xch + 8 * R * WAVE;
    int* redo = reinterpret_cast<int*>(xcs + 4 * BN);
    unsigned* most = reinterpret_cast<unsigned*>(redo + 8);      // of A's rows, then of B's
    float out[R];
    auto meet = [&] {
#pragma unroll
        for (int r = 0; r < R; ++r) xch[(wave * R + r) * WAVE + lane] = wk ? acc[r] : acc[R + r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float sum = xch[((wave ^ 4) * R + r) * WAVE + lane];
            out[r] = wk ? sum + acc[R + r] : acc[r] + sum;
        }
    };
    // Parts of an infinity give NaN.  Tiles with such sums, or whose parts lost bits that matter, are formed again on the float instructions.
    bool again = false;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        acc[r] += low[r];
        again |= !(fabsf(acc[r]) < INFINITY);
    }
    const bool odd = __any(again || loses(rest));
    if (lane == 0) redo[wave] = odd;
    meet();
    int any = 0;
#pragma unroll
    for (int w = 0; w < 8; ++w) any |= redo[w];
    auto either = [&](bool mine) {                               // of the workgroup's threads (__syncthreads_or has LDS of its own)
        __syncthreads();                       // everyone has read the last answer
        mine = __any(mine);
        if (lane == 0) redo[wave] = mine;
        __syncthreads();
        int all = 0;
#pragma unroll
        for (int w = 0; w < 8; ++w) all |= redo[w];
        return all;
    };
    if (any && !either(again)) [[unlikely]] {                    // lost bits only
        if (tid < BM + BN) most[tid] = 0;
        __syncthreads();
        if (stages_a) chunks_largest(std::bool_constant<A_KC>{}, A, lda, i0, m, most);
        else chunks_largest(std::bool_constant<B_KC>{}, B, ldb, j0, n, most + BM);
        __syncthreads();
        bool matter = false;
#pragma unroll
        for (int r = 0; r < R; ++r)
            matter |= matters(out[r], __uint_as_float(most[row_of(r) - i0]), __uint_as_float(most[BM + wn0 + l32]), K);
        any = either(matter);
    }
    if (any) [[unlikely]] {
        const int row = min(i0 + wm0 + l32, m - 1), col = min(j0 + wn0 + l32, n - 1);
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        for (int k0 = wk * 32; k0 < K; k0 += 64) {
            f32x4 fa[4], fb[4];
            load_slice<A_KC>(fa, A, lda, row, k0, K, g);
            load_slice<B_KC>(fb, B, ldb, col, k0, K, g);
            if (k0 + 32 > K) { mask_slice(fa, k0, K, g); mask_slice(fb, k0, K, g); }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][j], fb[i][j], acc, 0, 0, 0);
        }
        __syncthreads();                       // everyone has read what is written again
        meet();
    }
    if constexpr (GROUPED)
        if (col_sums && tid < BN && j0 + tid < n) {
            const float sum = (xcs[tid] + xcs[BN + tid]) + (xcs[2 * BN + tid] + xcs[3 * BN + tid]);
            float* o = p.bsum + j0 + tid;
            *o = L.flag ? sum : *o + sum;
        }
    if (col >= n) return;
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (row_of(r) < m) finish_one<EPI>(p, L.flag, (size_t)row_of(r) * n + col, out[r], bias, other[r]);
}

// Larger outputs: 128x128, 4 wavefronts of 64x64, two workgroups on a CU, each thread stages a chunk of either operand: half of the vector
// work and of the LDS reads per matrix instruction.  Float instructions -> 64x64 -> this, A B: 2048^3 155 -> 121 -> 98 us, 2048 x 16384 x
// 512 319 -> 246 -> 193 (before interleave), 4096 x 4096 x 1024 - -> 226 -> 178 (before it).  Loads four steps ahead need more registers
// than there are (2048^3 131).
template <bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(4 * WAVE, 2) void gemm_f32_wide_kernel(F32Launch L) {
    constexpr int BM = 128, BN = 128, BK = 16, NT = 4 * WAVE, TM = 2, TN = 2, CPR = BK / 8;
    constexpr int PART_A = BM * BK, PART_B = BN * BK, STEP = 3 * (PART_A + PART_B);
    __shared__ __attribute__((aligned(16))) bf16_t lds[2 * STEP];
    // 16-byte chunk c of row r sits at c ^ bits of r: 16 rows of one chunk, as many chunks of neighbouring rows, all fall on different banks
    auto chunk = [](int row, int c) { return c ^ ((row >> 3) & 1); };
    int tile_m, tile_n;
    const F32Product& p = tile_of(L, tile_m, tile_n);
    const int i0 = tile_m * BM, j0 = tile_n * BN, m = p.m, n = p.n, K = p.k;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave >> 1) * 64, wn0 = (wave & 1) * (BN / 2);
    const int KT = (K + BK - 1) / BK;
    unsigned rest = 0;
    float cs = 0.f;
    f32x16 acc[TM][TN], low[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = low[a][b][r] = 0.f;

    constexpr bool GROUPED = EPI == EPI_ACCUM_F32 && !A_KC && !B_KC;        // only those have column sums
    const bool col_sums = GROUPED && p.bsum && tile_m == 0;
    static_assert(BM * CPR == NT && BN * CPR == NT, "a chunk of either operand per thread");
    auto row_of = [&](bool kc) { return kc ? tid / CPR : tid % BM; };
    auto oct_of = [&](bool kc) { return kc ? tid % CPR : __builtin_amdgcn_readfirstlane(tid / BM); };
    SplitChunk<A_KC, BK> ca(p.a, p.lda, i0, m, BM, K, row_of(A_KC), oct_of(A_KC));
    SplitChunk<B_KC, BK> cb(p.b, p.ldb, j0, n, BN, K, row_of(B_KC), oct_of(B_KC));
    bf16_t* const put_a = lds + row_of(A_KC) * BK + chunk(row_of(A_KC), oct_of(A_KC)) * 8;
    bf16_t* const put_b = lds + 3 * PART_A + row_of(B_KC) * BK + chunk(row_of(B_KC), oct_of(B_KC)) * 8;
    constexpr int D = 2;                                         // steps that loads run ahead
    float va[D][8], vb[D][8];
    auto fetch = [&](int u) { ca.load(va[u]); cb.load(vb[u]); };
    auto stash = [&](int u, int kt, auto last_c) {
        if ((A_KC || B_KC) && decltype(last_c)::value && kt * BK + BK > K)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (A_KC && kt * BK + oct_of(true) * 8 + j >= K) va[u][j] = 0.f;
                if (B_KC && kt * BK + oct_of(true) * 8 + j >= K) vb[u][j] = 0.f;
            }
        split_store<PART_A>(va[u], put_a + (u & 1) * STEP, rest);
        split_store<PART_B>(vb[u], put_b + (u & 1) * STEP, rest);
        const float* v = vb[u];
        if (GROUPED) cs += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    };
    auto multiply = [&](int buf) {
        bf16x8 fa[TM][3], fb[TN][3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
#pragma unroll
            for (int a = 0; a < TM; ++a) {
                const int row = wm0 + a * 32 + l32;
                fa[a][q] = *reinterpret_cast<const bf16x8*>(lds + buf * STEP + q * PART_A + row * BK + chunk(row, g) * 8);
            }
#pragma unroll
            for (int b = 0; b < TN; ++b) {
                const int row = wn0 + b * 32 + l32;
                fb[b][q] = *reinterpret_cast<const bf16x8*>(lds + buf * STEP + 3 * PART_A + q * PART_B + row * BK + chunk(row, g) * 8);
            }
        }
        // B's rows first: a lane's sums are then four neighbouring columns of a row
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b) {
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[b][0], fa[a][0], acc[a][b], 0, 0, 0);
                low[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[b][1], fa[a][0], low[a][b], 0, 0, 0);
                low[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[b][0], fa[a][1], low[a][b], 0, 0, 0);
                low[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[b][1], fa[a][1], low[a][b], 0, 0, 0);
                low[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[b][2], fa[a][0], low[a][b], 0, 0, 0);
                low[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[b][0], fa[a][2], low[a][b], 0, 0, 0);
            }
    };
    static_assert(D % 2 == 0, "buffer of a step at compile time");
#pragma unroll
    for (int u = 0; u < D; ++u) fetch(u);
    stash(0, 0, std::true_type{});
    fetch(0);
    __syncthreads();
    int kt = 0;
    for (; kt + D + 1 < KT; kt += D)
#pragma unroll
        for (int u = 0; u < D; ++u) {
            multiply(u & 1);
            stash((u + 1) % D, kt + u + 1, std::false_type{});
            fetch((u + 1) % D);
            if constexpr (A_KC && B_KC) interleave<12, 1, 23, 5>();
            else interleave<12, 4, 20, 6>();
            __syncthreads();
        }
#pragma unroll
    for (int u = 0; u <= D; ++u) {
        if (kt + u >= KT) break;
        multiply(u & 1);
        if (kt + u + 1 < KT) stash((u + 1) % D, kt + u + 1, std::true_type{});
        __syncthreads();
    }
    bool again = false;                                          // as in gemm_f32_tile_kernel
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[a][b][r] += low[a][b][r];
                again |= !(fabsf(acc[a][b][r]) < INFINITY);
            }
    bool redo = __syncthreads_or(again || loses(rest));
    if (redo && !__syncthreads_or(again)) [[unlikely]] {         // lost bits only
        unsigned* most = reinterpret_cast<unsigned*>(lds);       // of A's rows, then of B's
        most[tid] = 0;
        __syncthreads();
        largest(SplitChunk<A_KC, BK>(p.a, p.lda, i0, m, BM, K, row_of(A_KC), oct_of(A_KC)), KT, most + row_of(A_KC));
        largest(SplitChunk<B_KC, BK>(p.b, p.ldb, j0, n, BN, K, row_of(B_KC), oct_of(B_KC)), KT, most + BM + row_of(B_KC));
        __syncthreads();
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    again |= matters(acc[a][b][r], __uint_as_float(most[wm0 + a * 32 + l32]),
                                     __uint_as_float(most[BM + wn0 + b * 32 + 8 * (r >> 2) + 4 * g + (r & 3)]), K);
        redo = __syncthreads_or(again);
    }
    // Both of a wavefront's rows against both of its columns: 2048^3 in tiles that are all formed again 386 -> 277 us (one 32x32 block
    // after the other).
    if (redo) [[unlikely]] {
        int rows[TM], cols[TN];
#pragma unroll
        for (int a = 0; a < TM; ++a) rows[a] = min(i0 + wm0 + a * 32 + l32, m - 1);
#pragma unroll
        for (int b = 0; b < TN; ++b) cols[b] = min(j0 + wn0 + b * 32 + l32, n - 1);
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
        for (int k0 = 0; k0 < K; k0 += 32) {
            f32x4 fa[TM][4], fb[TN][4];
#pragma unroll
            for (int a = 0; a < TM; ++a) load_slice<A_KC>(fa[a], p.a, p.lda, rows[a], k0, K, g);
#pragma unroll
            for (int b = 0; b < TN; ++b) load_slice<B_KC>(fb[b], p.b, p.ldb, cols[b], k0, K, g);
            if (k0 + 32 > K) {
#pragma unroll
                for (int a = 0; a < TM; ++a) mask_slice(fa[a], k0, K, g);
#pragma unroll
                for (int b = 0; b < TN; ++b) mask_slice(fb[b], k0, K, g);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int a = 0; a < TM; ++a)
#pragma unroll
                        for (int b = 0; b < TN; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[b][i][j], fa[a][i][j], acc[a][b], 0, 0, 0);
        }
    }
    if constexpr (GROUPED)
        if (col_sums) {                                          // a column's chunks lie in NT / BN threads
            float* xcs = reinterpret_cast<float*>(lds);
            xcs[tid] = cs;
            __syncthreads();
            if (tid < BN && j0 + tid < n) {
                float sum = xcs[B_KC ? tid * CPR : tid];
#pragma unroll
                for (int i = 1; i < NT / BN; ++i) sum += xcs[B_KC ? tid * CPR + i : tid + i * BN];
                float* o = p.bsum + j0 + tid;
                *o = L.flag ? sum : *o + sum;
            }
        }
#pragma unroll
    for (int a = 0; a < TM; ++a) {
        const int row = i0 + wm0 + a * 32 + l32;
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int col = j0 + wn0 + b * 32 + 8 * q + 4 * g;
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[a][b][4 * q + e];
                if (row < m && col < n) finish<EPI, 4>(p, L.flag, row, col, v);      // n is a multiple of 4
            }
    }
}

// ----------------------------------------------------------------- small form
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

enum Form { WIDE128, TILE64, SMALL, TINY };

// Up to two 16x16 tiles per CU take the tiny form.  32x32 -> 16x16: 128 x 384 x 128 3.2 -> 2.4 us, 128 x 128 x 512 (64 tiles) 5.8 -> 3.3 with
// residual, 6.6 -> 3.9 A B^T, 256 x 256 x 1024 (256) 10.5 -> 5.7, 300 x 320 x 1280 (380) 12.6 -> 10.7, 512 x 256 x 256 (512) 4.2 -> 3.4,
// x 1024 10.6 -> 9.2.
constexpr long TINY_TILES = 2 * NUM_CUS;

// Form of a launch.  Up to half a 64x64 tile per CU the small form's 32x32 tiles spread the work further (512 x 1024 x 1024, 128 tiles: 19
// to 21 us; 512 x 512 x 2048, 64 tiles: 19 against 30 to 47); beyond that the larger tiles' shared operands win (512 x 1536 x 512, 192
// tiles: 10.7 to 15.3 against 15.0 to 17.4; 1024 x 1024 x 4096, 256 tiles: 62 to 88 against 129 to 149).  A round of 128x128 tiles (one per
// CU) takes as long as 3.5 of 64x64, each of several 3.25, and begins and ends more slowly: 64x64 -> 128x128, A B and A^T B, 1024 x 4096 x
// 512 36.5 -> 33.6 and 38.0 -> 38.3 us, x 1024 65.0 -> 55.0 and 65.7 -> 61.3, x 256 21.6 -> 21.4 and 24.2 -> 27.1; 1280 x 3840 x 512 (300
// tiles) 43.1 -> 43.9 and 45.2 -> 53.5; 1280 x 5120 x 640 (400) 68.9 -> 56.9 and 70.9 -> 66.3; 4096 x 4096 x 256 76 -> 57 and 82 -> 77; A^T
// B 1024 x 4096 x 128 16.6 -> 20.7.
Form choose_form(int count, const GemmArgs* g) {
    long t64 = 0, t128 = 0;
    for (int i = 0; i < count; ++i) {
        t64 += (long)((g[i].m + 63) / 64) * ((g[i].n + 63) / 64);
        t128 += (long)((g[i].m + 127) / 128) * ((g[i].n + 127) / 128);
    }
    bool far = false;                                            // beyond a buffer load's offsets
    for (int i = 0; i < count; ++i) far |= g[i].lda > MAX_LD || g[i].ldb > MAX_LD;
    if (far || t64 <= NUM_CUS / 2) return SMALL;
    const long rounds64 = (t64 + NUM_CUS - 1) / NUM_CUS, rounds128 = (t128 + NUM_CUS - 1) / NUM_CUS;
    const bool sums = g[0].epilogue == EPI_ACCUM_F32;
    if (rounds128 == 1) return rounds64 == 4 && g[0].k >= (sums ? 768 : 512) ? WIDE128 : TILE64;
    return 3.25 * rounds128 < rounds64 && !(sums && g[0].k < 192) ? WIDE128 : TILE64;
}

template <bool A_KC, bool B_KC, int EPI>
int launch_form(F32Launch& L, Form form, hipStream_t s) {
    if (!A_KC && form == TINY) return fail(CHIMERA_EINVAL, "no 16x16 tile for weight gradients");       // (those go in groups, which are larger)
    const int tile = form == WIDE128 ? 128 : form == TILE64 ? 64 : form == SMALL ? 32 : 16;
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
    if (form == WIDE128) hipLaunchKernelGGL((gemm_f32_wide_kernel<A_KC, B_KC, EPI>), grid, dim3(4 * WAVE), 0, s, L);
    else if (form == TILE64) hipLaunchKernelGGL((gemm_f32_tile_kernel<A_KC, B_KC, EPI>), grid, dim3(8 * WAVE), 0, s, L);
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
