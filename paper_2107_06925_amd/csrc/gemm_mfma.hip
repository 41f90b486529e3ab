// bf16 GEMM on the CDNA4 matrix cores, float accumulation, for the three products of a linear layer:
//   forward  Y  = X W      A k-contiguous, B stored [k, n]
//   dgrad    dX = dY W^T   A k-contiguous, B k-contiguous
//   wgrad    dW += X^T dY  A stored [k, m], B stored [k, n]  (k = tokens)
//
// One workgroup computes a tile of the output; its wavefronts own parts of it as a grid of MFMA
// tiles whose accumulators never leave the registers.  Three kernels, by size (choose_tile):
//   gemm_ring_tile    256x256, 256x128 and 128x128 tiles on v_mfma_f32_16x16x32_bf16
//   gemm_async_tile   32x32 to 128x64 tiles on v_mfma_f32_32x32x16_bf16, a ring of k steps
//   gemm_bf16_kernel  the register-staged form: split-K and shapes on request
// The k loop moves BK = 64 at a time through LDS, the next steps in flight.  What follows on
// LDS layouts is the latter two's; gemm_ring_tile's own differ in their exchanges and are described there.
//
// An operand that is k-contiguous in memory (X in the forward, both operands of
// dgrad) sits in LDS as [row][k], 128 bytes per row, and lane l reads its MFMA
// operand - row l%32, the 8 consecutive k of chunk 2*kk + l/32 - with one
// 16-byte load.  Chunk c of row r is stored at c ^ (r & 7) ^ ((r >> 3) & 7), so the
// 8 rows a read touches per bank cycle fall on 8 different bank groups.
// An operand whose OTHER index is contiguous in memory (W in the forward, both
// operands of wgrad) is copied to LDS as it lies in memory, [k][row], and the
// transposition is done by the LDS hardware: ds_read_b64_tr_b16 hands lane i of
// each 16-lane group the i-th 16-bit element of the data addressed by lanes
// 4e + i/4 (e = 0..3), i.e. column i of a 4 x 16 block - four consecutive k of one
// row.  Two such reads give the same 8 k values the other flavour gets from one
// 16-byte load.  The 32-byte column blocks of row k are stored at block ^ 2(k & 3):
// one bank cycle serves 32 lanes = two adjacent column blocks x four rows, and this
// puts those eight 32-byte pieces on eight different bank groups (measured: without
// it half of the LDS cycles of the wgrad kernel were bank conflicts).  No transposed
// copy of any activation or weight exists in HBM, and no data is shuffled in
// registers.
//
// Workgroups are renumbered so that each of the 8 XCDs (own L2 each; the
// hardware deals consecutive workgroup ids round-robin over them) works on a
// contiguous range of tiles, and tiles are walked in groups of 8 tile rows so
// that the tiles in flight on one XCD share operand panels in its L2.
#include "device.h"

#include <algorithm>
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <type_traits>

namespace chimera {

namespace {

typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int BK = 64;
constexpr int GROUP_M = 8;       // tile rows per raster group
constexpr int NUM_CUS = 256;     // compute units of an MI355X
constexpr int XCDS = 8, PER_XCD = NUM_CUS / XCDS;
constexpr size_t SPLITK_COUNTER_BYTES = 4096;

__device__ __forceinline__ int swz(int row, int chunk) { return chunk ^ (row & 7) ^ ((row >> 3) & 7); }

typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));

// The XOR of k-row k's 32-byte column blocks in a [BK][ROWS] tile (rows of 128 bytes have only four; four rows of 64 bytes
// are all banks as they are).
template <int ROWS> __device__ __forceinline__ int kswz(int k) { return ROWS == 32 ? 0 : ROWS == 64 ? k & 2 : (k & 3) << 1; }
// LDS element offset of the 16-byte chunk `ic` (8 rows) of k-row `k` in a [BK][ROWS] tile
template <int ROWS> __device__ __forceinline__ int mc_off(int k, int ic) {
    return k * ROWS + (((ic >> 1) ^ kswz<ROWS>(k)) << 4) + ((ic & 1) << 3);
}

template <int ROWS, int NT, bool KC> struct Staged {
    static constexpr int N = ROWS * (BK / 8) / NT;     // 16-byte chunks per thread
    uint4 v[N];
    unsigned ok;     // bit i: v[i] lies inside the matrix (others are zeroed when written to LDS)
};

// global -> registers for one operand tile of ROWS rows x BK k values.
// KC: element (row, k) at base[row * ld + k].  !KC: at base[k * ld + row].
// Loads are unconditional (an out-of-range piece reads element 0 instead and is
// zeroed later), so no branch separates the loads of different k steps.
template <int ROWS, int NT, bool KC>
__device__ __forceinline__ void load_tile(Staged<ROWS, NT, KC>& st, const bf16_t* __restrict__ base, int ld, int row0,
                                          int nrows, int k0, int K, int tid) {
    constexpr int CPT = ROWS * (BK / 8) / NT;
    unsigned okm = 0;
#pragma unroll
    for (int it = 0; it < CPT; ++it) {
        const int c = tid + it * NT;
        bool ok;
        unsigned off;
        if constexpr (KC) {
            const int gr = row0 + (c >> 3), gk = k0 + (c & 7) * 8;
            ok = gr < nrows && gk < K;
            off = (unsigned)gr * (unsigned)ld + (unsigned)gk;
        } else {
            const int gk = k0 + c / (ROWS / 8), gi = row0 + (c % (ROWS / 8)) * 8;
            ok = gk < K && gi < nrows;
            off = (unsigned)gk * (unsigned)ld + (unsigned)gi;
        }
        st.v[it] = *reinterpret_cast<const uint4*>(base + (ok ? off : 0u));
        okm |= (ok ? 1u : 0u) << it;
    }
    st.ok = okm;
}

__device__ __forceinline__ uint4 keep_if(const uint4& q, unsigned mask, int bit) {
    const bool ok = (mask >> bit) & 1u;
    return make_uint4(ok ? q.x : 0u, ok ? q.y : 0u, ok ? q.z : 0u, ok ? q.w : 0u);
}

// registers -> LDS: [ROWS][BK] (KC) or [BK][ROWS] (!KC), swizzled as described above.
template <int ROWS, int NT, bool KC>
__device__ __forceinline__ void store_tile(const Staged<ROWS, NT, KC>& st, bf16_t* lds, int tid) {
    constexpr int CPT = ROWS * (BK / 8) / NT;
#pragma unroll
    for (int it = 0; it < CPT; ++it) {
        const int c = tid + it * NT;
        int off;
        if constexpr (KC) { const int row = c >> 3, kc = c & 7; off = row * BK + swz(row, kc) * 8; }
        else off = mc_off<ROWS>(c / (ROWS / 8), c % (ROWS / 8));
        *reinterpret_cast<uint4*>(lds + off) = keep_if(st.v[it], st.ok, it);
    }
}

// MFMA operand of lane `lane` for the 32 rows starting at r0 and the 16 k values of step kk.
template <int ROWS, bool KC>
__device__ __forceinline__ bf16x8 read_frag(const bf16_t* lds, int r0, int kk, int lane) {
    if constexpr (KC) {
        const int row = r0 + (lane & 31);
        return *reinterpret_cast<const bf16x8*>(lds + row * BK + swz(row, kk * 2 + (lane >> 5)) * 8);
    } else {
        const int i = lane & 15, blk = (r0 >> 4) + ((lane >> 4) & 1);      // 16-row column block of this lane group
        const int k = kk * 16 + (lane >> 5) * 8 + (i >> 2);                // row this lane addresses (first read)
        typedef bf16x4 __attribute__((address_space(3))) * lds_v4;
        const bf16_t* p0 = lds + k * ROWS + ((blk ^ kswz<ROWS>(k)) << 4) + ((i & 3) << 2);
        const bf16_t* p1 = p0 + 4 * ROWS;                                  // rows k+4..k+7: same swizzle
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_v4)p0);
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_v4)p1);
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
}

// Epilogue of one wavefront.  The matrix instructions get B's rows as their first operand, so a lane's accumulators are runs of
// four consecutive columns of one row of C (row l%32 of a 32x32 tile, columns 8q + 4(l/32) + 0..3; row l%16 of a 16x16 tile,
// columns 4(l/16) + 0..3).  Each 32-row band of the wavefront's tile goes through a wavefront-private LDS slab ([32][WN] floats)
// and comes back as 8 consecutive columns per lane; bias, residual, GeLU operands and the results then move in 16-byte pieces,
// 128 contiguous bytes per 8 lanes.  16-byte chunk c of row r sits at c ^ flip(r): both the writes (16 rows, one chunk each) and
// the reads (whole rows, every other chunk) put a pass of 16 lanes on all banks.  With A's rows first (one column per lane, written float
// by float) and rows padded by 32 bytes instead, half of the slabs' LDS cycles were conflicts, 4096 clocks of a 256x256 tile: 4096 x 3072 x 1024
// 28.4 -> 27.7 us, 2048 x 6400 x 1600 with GeLU 48.3 -> 47.3, 1264 x 4800 x 1600 24.6 -> 24.1, 400 x 1280 x 320 with GeLU 4.87 -> 4.70,
// 512 x 2048 x 512 5.68 -> 5.52; the float accumulate is bound by HBM and as fast as before.
template <int TN> struct EpiSlab {
    static constexpr int WN = TN * 32, FLOATS = 32 * WN;
    static_assert(TN == 1 || TN == 2, "rows of 32 or 64 floats");
    static __device__ __forceinline__ int flip(int row) { return TN == 1 ? (row >> 1) & 7 : row & 15; }
    static __device__ __forceinline__ float* at(float* slab, int row, int chunk) { return slab + row * WN + ((chunk ^ flip(row)) << 2); }
};
// Writers of one 32-row band of accumulators into a slab: 32x32 tiles, and 16x16 tiles.
template <int TM, int TN> struct Acc32 {
    const f32x16 (&acc)[TM][TN];
    template <int BAND> __device__ __forceinline__ void put(float* slab, int lane) const {
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x16& t = acc[BAND][b];
                *reinterpret_cast<f32x4*>(EpiSlab<TN>::at(slab, lane & 31, 8 * b + 2 * q + (lane >> 5))) = f32x4{t[4 * q], t[4 * q + 1], t[4 * q + 2], t[4 * q + 3]};
            }
    }
};
template <int TM, int TN> struct Acc16 {
    const f32x4 (&acc)[2 * TM][2 * TN];
    template <int BAND> __device__ __forceinline__ void put(float* slab, int lane) const {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2 * TN; ++b)
                *reinterpret_cast<f32x4*>(EpiSlab<TN>::at(slab, 16 * a + (lane & 15), 4 * b + (lane >> 4))) = acc[BAND * 2 + a][b];
    }
};

// `epi_flag` of the float accumulate: the result replaces C, which is not read; C passes the caches by.
enum { ACCUM_OVERWRITE = 1, ACCUM_ONCE = 2 };

__device__ __forceinline__ void load8(const bf16_t* p, float* o) { load_vec<bf16_t>(p, o); }
__device__ __forceinline__ void load8(const float* p, float* o) { load_vec<float>(p, o); load_vec<float>(p + 4, o + 4); }
__device__ __forceinline__ void store8(bf16_t* p, const float* v) { store_vec<bf16_t>(p, v); }
__device__ __forceinline__ void store8(float* p, const float* v) { store_vec<float>(p, v); store_vec<float>(p + 4, v + 4); }

// 8 consecutive elements as they come from memory (one or two 16-byte pieces), widened later:
// what the epilogue requests ahead of time.
template <typename T> struct Raw8;
template <> struct Raw8<bf16_t> {
    uint4 q;
    __device__ __forceinline__ void load(const bf16_t* p) { q = *reinterpret_cast<const uint4*>(p); }
    __device__ __forceinline__ void unpack(float* o) const {
        const unsigned w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) { o[2 * i] = __uint_as_float(w[i] << 16); o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u); }
    }
};
template <> struct Raw8<float> {
    float4 lo, hi;
    __device__ __forceinline__ void load(const float* p) {
        lo = *reinterpret_cast<const float4*>(p); hi = *reinterpret_cast<const float4*>(p + 4);
    }
    __device__ __forceinline__ void unpack(float* o) const {
        o[0] = lo.x; o[1] = lo.y; o[2] = lo.z; o[3] = lo.w; o[4] = hi.x; o[5] = hi.y; o[6] = hi.z; o[7] = hi.w;
    }
};

// The operand an epilogue reads from memory besides the bias: the residual, the GeLU input, or
// the old value of a float accumulator.  Each band of 32 rows needs 32 / RPP pieces per lane, and
// a piece that is only requested when its turn comes costs a full memory round trip per pass
// (16 in a row for a 128-row wavefront tile: as long as a short k loop).  So the pieces of the
// next DEPTH bands are requested before the current band is worked on: all bands when the
// elements have 2 bytes, two bands when they are floats (registers).
//
// The small tiles ask for all of it, bias included, before their k loop (EpiAhead): a round trip less at the
// end of a short launch.  With the residual, 256 x 256 x 1024 6.9 -> 6.35 us, 400 x 320 x 1280 7.7 -> 7.25; bias 256 x 768 x 256
// 4.4 -> 4.15.
template <int PIECES> struct EpiAhead {
    uint4 bias, q[PIECES][2];
    // 8 columns from col on of rows row, row + 16, ...
    __device__ __forceinline__ void request(int row, int col, int m, int n, const bf16_t* b, const bf16_t* r, const void* c, int epi,
                                            int epi_flag, int res_types) {
        const int lcol = min(col, n - 8);
        if (epi == EPI_BIAS || epi == EPI_BIAS_GELU || epi == EPI_BIAS_RESIDUAL) bias = *reinterpret_cast<const uint4*>(b + lcol);
        const bool f32 = epi == EPI_ACCUM_F32 || (epi == EPI_BIAS_RESIDUAL && (res_types & 1));
        if (epi != EPI_BIAS_RESIDUAL && epi != EPI_DGELU && !(epi == EPI_ACCUM_F32 && !(epi_flag & ACCUM_OVERWRITE))) return;
        const char* src = epi == EPI_ACCUM_F32 ? (const char*)c : (const char*)r;
#pragma unroll
        for (int j = 0; j < PIECES; ++j) {
            const size_t at = (size_t)min(row + j * 16, m - 1) * n + lcol;
            q[j][0] = *reinterpret_cast<const uint4*>(src + at * (f32 ? 4 : 2));
            if (f32) q[j][1] = *reinterpret_cast<const uint4*>(src + at * 4 + 16);
        }
    }
};

// Sums v of 8 consecutive elements of C from idx on, with their bias bv and what the epilogue reads besides (rv): finishes and stores them.
template <int EPI, bool CF32>
__device__ __forceinline__ void finish8(float* v, const float* bv, const float* rv, size_t idx, void* c, bf16_t* C2, int epi_flag) {
    bf16_t* C = (bf16_t*)c;
    float* Cf = (float*)c;
    if constexpr (EPI == EPI_NONE) {
        store8(C + idx, v);
    } else if constexpr (EPI == EPI_BIAS) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += bv[e];
        store8(C + idx, v);
    } else if constexpr (EPI == EPI_BIAS_GELU) {
        float g[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += bv[e];
        if (epi_flag) {                               // one wavefront-uniform branch per piece, not per element
#pragma unroll
            for (int e = 0; e < 8; ++e) g[e] = gelu_f(v[e], 1);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) g[e] = gelu_f(v[e], 0);
        }
        if (C) store8(C + idx, v);                    // null: nobody reads it
        store8(C2 + idx, g);
    } else if constexpr (EPI == EPI_BIAS_RESIDUAL) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += bv[e] + rv[e];
        if constexpr (CF32) store8(Cf + idx, v); else store8(C + idx, v);
    } else if constexpr (EPI == EPI_DGELU) {
        if (epi_flag) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] *= gelu_grad_f(rv[e], 1);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] *= gelu_grad_f(rv[e], 0);
        }
        store8(C + idx, v);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += rv[e];    // rv = 0 when the result replaces C
        store8(Cf + idx, v);
    }
}
// What a launch's epilogue is, as template arguments of `f`: f.operator()<EPI, R is float, C is float>()
template <typename F> __device__ __forceinline__ void with_epilogue(int epi, int res_types, F&& f) {
    switch (epi) {
        case EPI_NONE: f.template operator()<EPI_NONE, false, false>(); break;
        case EPI_BIAS: f.template operator()<EPI_BIAS, false, false>(); break;
        case EPI_BIAS_GELU: f.template operator()<EPI_BIAS_GELU, false, false>(); break;
        case EPI_BIAS_RESIDUAL:                    // res_types: bit 0 = R is float, bit 1 = C is float
            if (res_types == 0) f.template operator()<EPI_BIAS_RESIDUAL, false, false>();
            else if (res_types == 1) f.template operator()<EPI_BIAS_RESIDUAL, true, false>();
            else if (res_types == 2) f.template operator()<EPI_BIAS_RESIDUAL, false, true>();
            else f.template operator()<EPI_BIAS_RESIDUAL, true, true>();
            break;
        case EPI_DGELU: f.template operator()<EPI_DGELU, false, false>(); break;
        default: f.template operator()<EPI_ACCUM_F32, false, false>(); break;
    }
}
// The float accumulate of one wavefront.  A lane takes 4 columns, so that an instruction's pieces are whole rows of the wavefront's tile:
// with 8, in two instructions, each had every other 16 bytes of the lines, and C, where it passes the caches by, was written in parts of
// lines.  8 columns -> 4: blocks of 1344, 1792 and 2560 at 2048 tokens 95.6 -> 94.5, 172.6 -> 163.2 and 363 -> 355 us; six blocks of 1600
// and 2048, forward and backward, at 448 tokens 1501 -> 1466 and 2099 -> 1879, at 632 1689 -> 1667 and 2457 -> 2357.
template <bool ONCE, int TM, int TN, typename Acc>
__device__ __forceinline__ void accumulate(const Acc& acc, float* slab, int row_base, int col_base, int m, int n, float* __restrict__ C, int epi_flag, int lane) {
    constexpr int CPR = EpiSlab<TN>::WN / 4, RPP = 64 / CPR, NP = 32 / RPP;       // lanes per row, rows at once, passes per band of 32 rows
    constexpr int DEPTH = TM < 2 ? TM : 2;                                         // bands whose old values are asked for ahead
    const int pr = lane / CPR, piece = lane % CPR, gcol = col_base + piece * 4, lcol = min(gcol, n - 4);
    const bool reads = !(epi_flag & ACCUM_OVERWRITE);
    f32x4 old[DEPTH][NP];
    auto request = [&](int a, auto slot_c) {
        constexpr int SLOT = decltype(slot_c)::value;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            // pieces outside the matrix are requested from its last row / last piece (never used)
            const f32x4* from = reinterpret_cast<const f32x4*>(C + (size_t)min(row_base + a * 32 + j * RPP + pr, m - 1) * n + lcol);
            if constexpr (ONCE) old[SLOT][j] = __builtin_nontemporal_load(from);
            else old[SLOT][j] = *from;
        }
    };
    if (reads) {
        request(0, std::integral_constant<int, 0>{});
        if constexpr (TM > 1) request(1, std::integral_constant<int, 1>{});
    }
    auto band = [&](auto a_c) {
        constexpr int a = decltype(a_c)::value, SLOT = a % DEPTH;
        acc.template put<a>(slab, lane);
        __builtin_amdgcn_s_waitcnt(0xc07f);                   // lgkmcnt(0): the slab is written (wavefront-private)
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int lr = j * RPP + pr, grow = row_base + a * 32 + lr;
            f32x4 v = *reinterpret_cast<const f32x4*>(EpiSlab<TN>::at(slab, lr, piece));
            if (reads) v += old[SLOT][j];
            if (grow >= m || gcol >= n) continue;
            f32x4* to = reinterpret_cast<f32x4*>(C + (size_t)grow * n + gcol);
            if constexpr (ONCE) __builtin_nontemporal_store(v, to);
            else *to = v;
        }
        __builtin_amdgcn_wave_barrier();                      // all lanes have read the slab before it is rewritten
        if constexpr (a + DEPTH < TM)
            if (reads) request(a + DEPTH, std::integral_constant<int, SLOT>{});
    };
    band(std::integral_constant<int, 0>{});
    if constexpr (TM > 1) band(std::integral_constant<int, 1>{});
    if constexpr (TM > 2) band(std::integral_constant<int, 2>{});
    if constexpr (TM > 3) band(std::integral_constant<int, 3>{});
}
template <int EPI, bool RF32, bool CF32, int TM, int TN, typename Acc>
__device__ __forceinline__ void epilogue(const Acc& acc, float* slab, int row_base, int col_base, int m,
                                         int n, const bf16_t* __restrict__ bias, const bf16_t* __restrict__ R,
                                         void* __restrict__ c, bf16_t* __restrict__ C2, int epi_flag, int lane) {
    if constexpr (EPI == EPI_ACCUM_F32) {
        if (epi_flag & ACCUM_ONCE) accumulate<true, TM, TN>(acc, slab, row_base, col_base, m, n, (float*)c, epi_flag, lane);
        else accumulate<false, TM, TN>(acc, slab, row_base, col_base, m, n, (float*)c, epi_flag, lane);
        return;
    }
    constexpr int WN = EpiSlab<TN>::WN;
    constexpr int CPR = WN / 8;                // 8-column pieces per row
    constexpr int RPP = 64 / CPR;              // rows covered by the 64 lanes at once
    constexpr int NP = 32 / RPP;               // passes per band of 32 rows
    constexpr bool READS = EPI == EPI_BIAS_RESIDUAL || EPI == EPI_DGELU;
    using RT = std::conditional_t<EPI == EPI_BIAS_RESIDUAL && RF32, float, bf16_t>;
    constexpr int DEPTH = !READS ? 1 : (sizeof(RT) == 4 ? (TM < 2 ? TM : 2) : TM);
    const int pr = lane / CPR, pc = (lane % CPR) * 8;
    const int gcol = col_base + pc;
    const RT* Rsrc = reinterpret_cast<const RT*>(R);
    // pieces outside the matrix are requested from its last row / last piece (never used)
    const int lcol = min(gcol, n - 8);
    Raw8<RT> ahead[DEPTH][NP];
    auto request = [&](int a, auto slot_c) {
        constexpr int SLOT = decltype(slot_c)::value;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int grow = min(row_base + a * 32 + j * RPP + pr, m - 1);
            ahead[SLOT][j].load(Rsrc + (size_t)grow * n + lcol);
        }
    };
    float bv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) bv[e] = 0.f;
    if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_RESIDUAL) {
        if (gcol < n) load8(bias + gcol, bv);
    }
    if constexpr (READS) {
        request(0, std::integral_constant<int, 0>{});
        if constexpr (DEPTH > 1 && TM > 1) request(1, std::integral_constant<int, 1 % DEPTH>{});
        if constexpr (DEPTH > 2 && TM > 2) request(2, std::integral_constant<int, 2 % DEPTH>{});
        if constexpr (DEPTH > 3 && TM > 3) request(3, std::integral_constant<int, 3 % DEPTH>{});
    }
    static_assert(TM <= 4, "at most four bands per wavefront");
    auto band = [&](auto a_c) {
        constexpr int a = decltype(a_c)::value;
        constexpr int SLOT = a % DEPTH;
        acc.template put<a>(slab, lane);
        __builtin_amdgcn_s_waitcnt(0xc07f);                   // lgkmcnt(0): the slab is written (wavefront-private)
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int lr = j * RPP + pr;
            const int grow = row_base + a * 32 + lr;
            float v[8];
            load_vec<float>(EpiSlab<TN>::at(slab, lr, pc / 4), v);
            load_vec<float>(EpiSlab<TN>::at(slab, lr, pc / 4 + 1), v + 4);
            float rv[8];
            if constexpr (READS) ahead[SLOT][j].unpack(rv);
            if (grow >= m || gcol >= n) continue;
            finish8<EPI, CF32>(v, bv, rv, (size_t)grow * n + gcol, c, C2, epi_flag);
        }
        __builtin_amdgcn_wave_barrier();                      // all lanes have read the slab before it is rewritten
        if constexpr (READS && a + DEPTH < TM) request(a + DEPTH, std::integral_constant<int, SLOT>{});
    };
    band(std::integral_constant<int, 0>{});
    if constexpr (TM > 1) band(std::integral_constant<int, 1>{});
    if constexpr (TM > 2) band(std::integral_constant<int, 2>{});
    if constexpr (TM > 3) band(std::integral_constant<int, 3>{});
}

template <int BM, int BN, int WGM, int WGN, int PF, bool A_KC, bool B_KC>
__global__ __launch_bounds__(WGM* WGN * 64) void gemm_bf16_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, const bf16_t* __restrict__ bias,
    const bf16_t* __restrict__ R, void* __restrict__ C, bf16_t* __restrict__ C2, int m, int n, int k, int lda,
    int ldb, int epi, int epi_flag, int res_types, int tiles_m, int tiles_n, int splits, float* __restrict__ slabs,
    unsigned* __restrict__ arrivals) {
    constexpr int NT = WGM * WGN * 64;
    constexpr int WM = BM / WGM, WN = BN / WGN;    // wavefront tile
    constexpr int TM = WM / 32, TN = WN / 32;      // MFMA tiles per wavefront
    __shared__ __attribute__((aligned(16))) bf16_t lds[2][(BM + BN) * BK];

    // workgroup id -> tile, XCD-contiguous then grouped raster
    // With split-K the grid holds `splits` workgroups per tile: split = blockIdx / tiles.
    const int nblk = tiles_m * tiles_n;
    const int split = blockIdx.x / nblk, bid = blockIdx.x % nblk;
    const int xcd = bid & 7, local = bid >> 3;
    const int pid = xcd * (nblk >> 3) + min(xcd, nblk & 7) + local;
    const int width = GROUP_M * tiles_n;
    const int first_m = (pid / width) * GROUP_M;
    const int gsz = min(tiles_m - first_m, GROUP_M);
    const int tile_m = first_m + (pid % width) % gsz;
    const int tile_n = (pid % width) / gsz;
    const int i0 = tile_m * BM, j0 = tile_n * BN;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm0 = (wave / WGN) * WM, wn0 = (wave % WGN) * WN;

    f32x16 acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

    // one k step of MFMA work out of LDS buffer `buf`
    auto compute = [&](int buf) {
        const bf16_t* As = lds[buf];
        const bf16_t* Bs = lds[buf] + BM * BK;
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            bf16x8 af[TM], bfr[TN];
#pragma unroll
            for (int a = 0; a < TM; ++a) af[a] = read_frag<BM, A_KC>(As, wm0 + a * 32, kk, lane);
#pragma unroll
            for (int b = 0; b < TN; ++b) bfr[b] = read_frag<BN, B_KC>(Bs, wn0 + b * 32, kk, lane);
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[b], af[a], acc[a][b], 0, 0, 0);
        }
    };
    auto fetch = [&](Staged<BM, NT, A_KC>& ra, Staged<BN, NT, B_KC>& rb, int kt) {
        load_tile<BM, NT, A_KC>(ra, A, lda, i0, m, kt * BK, k, tid);
        load_tile<BN, NT, B_KC>(rb, B, ldb, j0, n, kt * BK, k, tid);
    };
    auto stash = [&](const Staged<BM, NT, A_KC>& ra, const Staged<BN, NT, B_KC>& rb, int buf) {
        store_tile<BM, NT, A_KC>(ra, lds[buf], tid);
        store_tile<BN, NT, B_KC>(rb, lds[buf] + BM * BK, tid);
    };

    // Software pipeline: global loads run PF k steps ahead of the matrix cores in PF
    // register sets (a ring walked by an unrolled loop, so every index is static),
    // LDS runs one step ahead in two buffers, one barrier per step.
    // This workgroup's share of the k steps: [K0, K1).
    const int KT_all = (k + BK - 1) / BK;
    const int K0 = (int)((long)KT_all * split / splits), K1 = (int)((long)KT_all * (split + 1) / splits);
    const int KT = K1 - K0;
    Staged<BM, NT, A_KC> ra[PF];
    Staged<BN, NT, B_KC> rb[PF];
#pragma unroll
    for (int u = 0; u < PF; ++u)
        if (u < KT) fetch(ra[u], rb[u], K0 + u);
    stash(ra[0], rb[0], 0);
    __syncthreads();
    for (int kt = 0; kt < KT; kt += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int step = kt + u;
            if (step >= KT) break;
            if (step + PF < KT) fetch(ra[u], rb[u], K0 + step + PF);      // set u was stashed one step ago
            compute(step & 1);
            if (step + 1 < KT) stash(ra[(u + 1) % PF], rb[(u + 1) % PF], (step + 1) & 1);
            __syncthreads();
        }
    }

    // Split-K: every workgroup of a tile writes its partial accumulators to its own slab
    // (thread-private order, 16-byte stores), then counts itself in.  Whoever arrives last
    // adds the slabs in split order - so the sum does not depend on who that is - and runs
    // the epilogue.  Nobody waits for anybody.
    if (splits > 1) {
        __shared__ int is_last;
        const size_t tile_elems = (size_t)BM * BN;
        float4* mine = reinterpret_cast<float4*>(slabs + ((size_t)split * nblk + pid) * tile_elems);
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    mine[((a * TN + b) * 4 + q) * NT + tid] =
                        make_float4(acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]);
        __threadfence();                       // slab visible device-wide before the arrival count
        __syncthreads();
        if (tid == 0) is_last = atomicAdd(&arrivals[pid], 1u) == (unsigned)(splits - 1);
        __syncthreads();
        if (!is_last) return;
        __threadfence();                       // see the other workgroups' slabs
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
        for (int sp = 0; sp < splits; ++sp) {
            const float4* other = reinterpret_cast<const float4*>(slabs + ((size_t)sp * nblk + pid) * tile_elems);
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float4 v = other[((a * TN + b) * 4 + q) * NT + tid];
                        acc[a][b][4 * q] += v.x; acc[a][b][4 * q + 1] += v.y;
                        acc[a][b][4 * q + 2] += v.z; acc[a][b][4 * q + 3] += v.w;
                    }
        }
        if (tid == 0) arrivals[pid] = 0u;      // ready for the next launch on this stream
    }

    const int rb0 = i0 + wm0, cb0 = j0 + wn0;
    // the operand tiles in LDS are dead once every wavefront has left the k loop; each
    // wavefront then stages its output through its own slab there
    static_assert(sizeof(lds) >= (size_t)WGM * WGN * EpiSlab<TN>::FLOATS * sizeof(float), "LDS too small for the epilogue");
    __syncthreads();
    float* slab = reinterpret_cast<float*>(lds) + (size_t)(tid >> 6) * EpiSlab<TN>::FLOATS;
    with_epilogue(epi, res_types, [&]<int E, bool RF, bool CF>() {
        epilogue<E, RF, CF, TM, TN>(Acc32<TM, TN>{acc}, slab, rb0, cb0, m, n, bias, R, C, C2, epi_flag, lane);
    });
}

template <int N, typename F> __device__ __forceinline__ void static_for(F&& f) {
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// ---------------------------------------------------------------- async variant
// Same tiles, same LDS layouts, same MFMA loop, but the tiles travel global -> LDS
// without passing through registers (global_load_lds_dwordx4: lane i of a wavefront
// writes 16 bytes at LDS base + 16 i), into a ring of NS stages, so the loads of the
// next NS-1 k steps are in flight while the matrix cores work.  Because the LDS side of
// such a load is fixed, the swizzle is applied on the global side: the lane that owns
// LDS slot (row, position p) fetches the chunk that belongs there.  The instruction is
// issued through inline assembly so that the waits can be counted by hand
// (s_waitcnt vmcnt(n) with the younger stages still outstanding).
// Nothing can be zero-filled on this path: rows beyond the matrix are redirected to a
// valid row (they only feed outputs that are never stored), and the k % BK values behind
// the last whole step come first, through registers and zero-filled, while the DMA of the
// first whole steps is under way.

// What the next product reads from HBM (the weights of the next linear layer) is touched by this one between its
// k loop and its epilogue: 64 lines of 128 bytes per wavefront and instruction, the range dealt over the launch, four
// bytes of each line into a strip of LDS that nobody reads.  The lines are then in the memory-side cache when
// the next launch asks for them.  A CU has some 60 KiB of requests under way at most (61 to 68 GB/s per CU from HBM with every
// tile here, 80 to 96 from the memory-side cache; requesting further ahead changes nothing), so a k loop that is short of
// operands waits for the latency of the slower one, and weights come from HBM in every pass.
// Measured, A in the memory-side cache, B untouched -> touched: A B^T 2048 x 1600 x 6400 57 -> 44 us on 128x128
// tiles, 82 -> 68 on 256x128 (on two streams 44.6 -> 37.9 each), 4096 x 1024 x 4096 48.6 -> 41.4, A B 2048 x 4800 x 1600
// 42.9 -> 40.6 (31.0 -> 28.0), 632 x 4800 x 1600 18.6 -> 16.7, 1264 x 1600 x 6400 50.5 -> 44.6; with A from HBM too
// nothing is won.  Inside the loop the touches cost more on two streams (2048 x 1600 x 6400 37.9 -> 42.5), behind the
// epilogue too (39.1; 2048 x 1600 x 1600 28.1 -> 30.3 on one).  Touching the backward's stashed operands as well was slower
// than not (gpt2-1p3b-n32 97.8 -> 99.4 ms, gpt2-deep 50.2 -> 51.2).
struct Ahead { const char* p; unsigned bytes; };
constexpr unsigned AHEAD_PIECE = 64 * 128, AHEAD_STRIP = 256;
__device__ __forceinline__ void touch_ahead(const Ahead& ahead, int wave, int waves, int lane) {
    __shared__ __attribute__((aligned(16))) char lines[AHEAD_STRIP];
    const unsigned strip = lds_address(lines);
    // pieces beyond the range repeat its last word
    for (size_t at = ((size_t)blockIdx.x * waves + wave) * AHEAD_PIECE; at < ahead.bytes; at += (size_t)gridDim.x * waves * AHEAD_PIECE) {
        const unsigned off = min((unsigned)at + (unsigned)lane * 128u, ahead.bytes - 4u);
        asm volatile("global_load_lds_dword %0, %1" ::"v"(off), "s"(ahead.p), "{m0}"(strip) : "memory");
    }
}

// One output tile; `block_id` numbers the tiles of this product.  ONLY_EPI >= 0 compiles
// that epilogue alone.
// SPS: ring stages per barrier (NS stages of BK each).
template <int BM, int BN, int WGM, int WGN, int WGK, int NS, int SPS, bool A_KC, bool B_KC, int ONLY_EPI>
__device__ __forceinline__ void gemm_async_tile(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, const bf16_t* __restrict__ bias,
    const bf16_t* __restrict__ R, void* __restrict__ C, bf16_t* __restrict__ C2, int m, int n, int k, int lda,
    int ldb, int epi, int epi_flag, int res_types, int tiles_m, int tiles_n, int group_m, int block_id,
    float* __restrict__ bsum = nullptr, bool xcd_remap = true, const Ahead& ahead = {nullptr, 0}) {
    constexpr int NT = WGM * WGN * WGK * 64;
    constexpr int KSUB = BK / 16 / WGK;                                   // 16-wide k slices per wavefront and step
    static_assert(KSUB >= 1 && KSUB * WGK * 16 == BK, "k split must divide the step");
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int TM = WM / 32;                                           // a wavefront's 32x32 blocks, below one another
    static_assert(WN == 32, "rows of 32 columns");
    constexpr int CA = BM * (BK / 8) / NT, CB = BN * (BK / 8) / NT;      // 16-byte pieces per thread and stage
    constexpr int STAGE = (BM + BN) * BK;                                 // elements
    __shared__ __attribute__((aligned(16))) bf16_t lds[NS * STAGE];

    const int nblk = tiles_m * tiles_n;
    // `block_id` as the hardware deals it (round-robin over the XCDs) or already renumbered
    const int xcd = block_id & 7, local = block_id >> 3;
    const int pid = xcd_remap ? xcd * (nblk >> 3) + min(xcd, nblk & 7) + local : block_id;
    const int width = group_m * tiles_n;
    const int first_m = (pid / width) * group_m;
    const int gsz = min(tiles_m - first_m, group_m);
    const int tile_m = first_m + (pid % width) % gsz;
    const int tile_n = (pid % width) / gsz;
    const int i0 = tile_m * BM, j0 = tile_n * BN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave / (WGM * WGN), wmn = wave % (WGM * WGN);       // k slice, position in the tile
    const int wm0 = (wmn / WGN) * WM, wn0 = (wmn % WGN) * WN;

    // Per-thread source pointers (advanced by one k step after every issue) for the LDS
    // slots this thread's lane position fills.
    const bf16_t* ga[CA];
    const bf16_t* gb[CB];
    auto source = [&](const bf16_t* base, int ld, int row0, int nrows, auto rows_c, bool kc, int slot) {
        constexpr int rows_in_tile = decltype(rows_c)::value;
        if (kc) {
            const int row = slot >> 3, p = slot & 7;
            const int c = p ^ (row & 7) ^ ((row >> 3) & 7);
            const int gr = min(row0 + row, nrows - 1);
            return base + (size_t)gr * ld + c * 8;
        }
        const int per_row = rows_in_tile / 8;
        const int kk = slot / per_row, pc = slot % per_row;
        const int ic = (((pc >> 1) ^ kswz<rows_in_tile>(kk)) << 1) | (pc & 1);
        int gi = row0 + ic * 8;
        if (gi >= nrows) gi = 0;
        return base + (size_t)kk * ld + gi;
    };
#pragma unroll
    for (int it = 0; it < CA; ++it) ga[it] = source(A, lda, i0, m, std::integral_constant<int, BM>{}, A_KC, it * NT + tid);
#pragma unroll
    for (int it = 0; it < CB; ++it) gb[it] = source(B, ldb, j0, n, std::integral_constant<int, BN>{}, B_KC, it * NT + tid);
    const size_t step_a = A_KC ? (size_t)BK : (size_t)BK * lda;
    const size_t step_b = B_KC ? (size_t)BK : (size_t)BK * ldb;
    // LDS byte address of stage 0 (32-bit pointer in the LDS address space)
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) const void*)lds;

    auto issue = [&](int stage) {
        const unsigned sa = lds0 + (unsigned)(stage * STAGE) * 2u + (unsigned)wave * 1024u;
#pragma unroll
        for (int it = 0; it < CA; ++it) { lds_dma16(ga[it], sa + it * NT * 16); ga[it] += step_a; }
        const unsigned sb = sa + BM * BK * 2;
#pragma unroll
        for (int it = 0; it < CB; ++it) { lds_dma16(gb[it], sb + it * NT * 16); gb[it] += step_b; }
    };

    // The wavefronts of a block of the tile hold partial sums of it, one per k slice; in the end each finishes its share of the rows, a lane
    // 8 columns of rows row0, row0 + 16, ...
    constexpr int SHARE = WM / WGK, PIECES = (SHARE + 15) / 16;
    const int row0 = wk * SHARE + lane / 4, gcol = j0 + wn0 + lane % 4 * 8;
    // With two workgroups on a CU each hides the other's last trip, and these requests hold back the first operands.  Without them A^T B
    // 1472 x 1280 x 512 7.56 -> 7.24 us, groups of 12 x 384^2 x 1024 10.36 -> 9.97, A B^T with the GeLU derivative 1088 x 1088 x 192 5.54
    // -> 5.39; but A B x 64 4.2 -> 4.4.
    constexpr bool EPI_AHEAD = SPS > 1 || (A_KC && !B_KC);
    EpiAhead<PIECES> pre;
    auto ask = [&] { pre.request(i0 + wm0 + row0, gcol, m, n, bias, R, C, ONLY_EPI >= 0 ? ONLY_EPI : epi, epi_flag, res_types); };
    if (EPI_AHEAD) ask();

    f32x16 acc[TM][1];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][0][r] = 0.f;

    // Optional by-product: bsum[j] += sum over the contraction index of B(k, j), i.e. an extra
    // all-ones row of A.  The wavefronts at the top edge of the first tile row compute it
    // with one more MFMA per step (every row of that accumulator is the column sum).
    const bool col_sums = bsum != nullptr && tile_m == 0 && wm0 == 0;
    f32x16 cs;
    bf16x8 ones;
#pragma unroll
    for (int q = 0; q < 8; ++q) ones[q] = (bf16_t)1.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) cs[r] = 0.f;

    const int KT = k / BK;
    auto compute = [&](int stage) {
        const bf16_t* As = lds + stage * STAGE;
        const bf16_t* Bs = As + BM * BK;
#pragma unroll
        for (int ks = 0; ks < KSUB; ++ks) {
            const int kk = wk * KSUB + ks;
            bf16x8 af[TM];
#pragma unroll
            for (int a = 0; a < TM; ++a) af[a] = read_frag<BM, A_KC>(As, wm0 + a * 32, kk, lane);
            const bf16x8 bfr = read_frag<BN, B_KC>(Bs, wn0, kk, lane);
#pragma unroll
            for (int a = 0; a < TM; ++a) acc[a][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr, af[a], acc[a][0], 0, 0, 0);
            if constexpr (ONLY_EPI == EPI_ACCUM_F32)
                if (col_sums) cs = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, bfr, cs, 0, 0, 0);
        }
    };
    if (k % BK) {
        Staged<BM, NT, A_KC> ra;
        Staged<BN, NT, B_KC> rb;
        load_tile<BM, NT, A_KC>(ra, A, lda, i0, m, KT * BK, k, tid);
        load_tile<BN, NT, B_KC>(rb, B, ldb, j0, n, KT * BK, k, tid);
#pragma unroll
        for (int st = 0; st < NS - SPS; ++st)
            if (st < KT) [[likely]] issue(st);
        bf16_t* last = lds + (NS - 1) * STAGE;             // the stage that the first issue of the loop fills
        store_tile<BM, NT, A_KC>(ra, last, tid);
        store_tile<BN, NT, B_KC>(rb, last + BM * BK, tid);
        __syncthreads();
        compute(NS - 1);
    } else {
#pragma unroll
        for (int st = 0; st < NS - SPS; ++st)
            if (st < KT) [[likely]] issue(st);
    }
    int cur = 0, nxt = NS - SPS;               // stage computed now / stage the next issue fills
    auto advance = [](int& st) { st = st + 1 == NS ? 0 : st + 1; };
    // Operands of SPS stages out of LDS first, then a request behind each MFMA: all wavefronts leave the barrier together, and
    // a CU takes 16 clocks for each of their 16 to 32 requests, which reads behind them would wait for.  Requests first -> reads
    // first, operands in the memory-side cache: 632 x 1600 x 6400 26.1 -> 22.5 us, 1024 x 640 x 2560 11.5 -> 10.7, 1264 x 1600 x 6400
    // (two workgroups per CU) 42.9 -> 41.7.  The last steps, which have nothing left to request, and all of a k loop shorter than the
    // ring, leave the order to the compiler: with it fixed there too, and every instruction behind a condition, k = 192 to 768 takes 3 to 5 %
    // longer (A B^T 1280 x 768 x 320 4.68 -> 4.50 us, A B 1088 x 1088 x 512 6.32 -> 6.05).
    auto iteration = [&] {
        bf16x8 af[SPS][KSUB][TM], bfr[SPS][KSUB];
        int st = cur;
#pragma unroll
        for (int u = 0; u < SPS; ++u) {
            const bf16_t* As = lds + st * STAGE;
            advance(st);
#pragma unroll
            for (int ks = 0; ks < KSUB; ++ks) {
#pragma unroll
                for (int a = 0; a < TM; ++a) af[u][ks][a] = read_frag<BM, A_KC>(As, wm0 + a * 32, wk * KSUB + ks, lane);
                bfr[u][ks] = read_frag<BN, B_KC>(As + BM * BK, wn0, wk * KSUB + ks, lane);
            }
        }
        cur = st;
        __builtin_amdgcn_sched_barrier(0);
        constexpr int REQ = SPS * (CA + CB), MM = SPS * KSUB * TM, PER = (REQ + MM - 1) / MM;
        static_for<MM>([&](auto i_c) {
            constexpr int i = decltype(i_c)::value, u = i / (KSUB * TM), ks = i / TM % KSUB, a = i % TM;
            acc[a][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[u][ks], af[u][ks][a], acc[a][0], 0, 0, 0);
            if constexpr (ONLY_EPI == EPI_ACCUM_F32 && a == 0)
                if (col_sums) cs = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, bfr[u][ks], cs, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            static_for<PER>([&](auto j_c) {
                constexpr int r = i * PER + decltype(j_c)::value, it = r % (CA + CB);
                if constexpr (r < REQ) {
                    const unsigned to = lds0 + (unsigned)(nxt * STAGE) * 2u + (unsigned)wave * 1024u;
                    if constexpr (it < CA) { lds_dma16(ga[it], to + it * NT * 16); ga[it] += step_a; }
                    else { lds_dma16(gb[it - CA], to + BM * BK * 2 + (it - CA) * NT * 16); gb[it - CA] += step_b; }
                    if constexpr (it == CA + CB - 1) advance(nxt);
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    int kt = 0;
    for (; kt + NS <= KT; kt += SPS) {
        // the SPS oldest outstanding stages must have landed; NS - 2 SPS younger ones may fly on
        wait_vmcnt<(NS - 2 * SPS) * (CA + CB)>();
        __syncthreads();                       // every wavefront's part of this step is in LDS; the previous one is consumed
        iteration();
    }
    for (; kt < KT; kt += SPS) {
        if (kt + NS - SPS <= KT) wait_vmcnt<(NS - 2 * SPS) * (CA + CB)>(); else wait_vmcnt<0>();
        __syncthreads();
#pragma unroll
        for (int u = 0; u < SPS - 1; ++u)
            if (kt + NS - SPS + u < KT) { issue(nxt); advance(nxt); }
#pragma unroll
        for (int u = 0; u < SPS; ++u)
            if (u == 0 || kt + u < KT) { compute(cur); advance(cur); }
    }
    if constexpr (ONLY_EPI < 0)
        if (ahead.bytes) [[unlikely]] touch_ahead(ahead, wave, NT / 64, lane);       // weight gradients and split products precede no product

    if (!EPI_AHEAD) ask();
    // The operand tiles in LDS are dead once every wavefront has left the k loop: each puts its sums there, and every one of a block adds, in
    // the order of the k slices, and finishes its share.  With one of them (or each its half of 64 rows) finishing what it had taken from
    // the others after a second trip through LDS -> so: 256 x 768 x 256 3.57 -> 3.37 us, 256 x 1024 x 256 with GeLU 4.02 -> 3.55, 400 x 320 x 1280
    // 5.73 -> 5.43, 512 x 2048 x 512 5.56 -> 5.37, 1264 x 1600 x 1600 13.2 -> 12.5.
    constexpr int BAND = EpiSlab<1>::FLOATS;
    static_assert(sizeof(lds) >= ((size_t)(NT / 64) * TM * BAND + WGK * BN) * sizeof(float), "LDS too small for the sums");
    __syncthreads();
    float* slabs = reinterpret_cast<float*>(lds);
    float* xcs = slabs + NT / 64 * TM * BAND + wn0 + lane;
    static_for<TM>([&](auto a_c) { Acc32<TM, 1>{acc}.template put<decltype(a_c)::value>(slabs + (wave * TM + decltype(a_c)::value) * BAND, lane); });
    if constexpr (ONLY_EPI == EPI_ACCUM_F32)               // row 0 of a column-sum accumulator: register 0 of lanes 0..31
        if (col_sums && lane < 32) xcs[wk * BN] = cs[0];
    __syncthreads();
    if constexpr (ONLY_EPI == EPI_ACCUM_F32)
        if (col_sums && wk == 0 && lane < 32) {
            float v = cs[0];
#pragma unroll
            for (int w = 1; w < WGK; ++w) v += xcs[w * BN];
            const int col = j0 + wn0 + lane;
            if (col < n) bsum[col] = (epi_flag & ACCUM_OVERWRITE) ? v : bsum[col] + v;
        }
    auto finish = [&]<int E, bool RF, bool CF>() {
        constexpr bool READS_F32 = E == EPI_ACCUM_F32 || (E == EPI_BIAS_RESIDUAL && RF), READS = E == EPI_BIAS_RESIDUAL || E == EPI_DGELU || E == EPI_ACCUM_F32;
        float bv[8];
        if constexpr (E == EPI_BIAS || E == EPI_BIAS_GELU || E == EPI_BIAS_RESIDUAL) Raw8<bf16_t>{pre.bias}.unpack(bv);
#pragma unroll
        for (int j = 0; j < PIECES; ++j) {
            const int r = row0 + j * 16, grow = i0 + wm0 + r;
            float v[8];
#pragma unroll
            for (int w = 0; w < WGK; ++w) {
                float* slab = slabs + ((w * WGM * WGN + wmn) * TM + r / 32) * BAND;
                float u[8];
                load_vec<float>(EpiSlab<1>::at(slab, r % 32, lane % 4 * 2), u);
                load_vec<float>(EpiSlab<1>::at(slab, r % 32, lane % 4 * 2 + 1), u + 4);
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = w ? v[e] + u[e] : u[e];
            }
            float rv[8];
            if constexpr (READS_F32) {
                const bool reads = !(E == EPI_ACCUM_F32 && (epi_flag & ACCUM_OVERWRITE));
                if (reads) Raw8<float>{__builtin_bit_cast(float4, pre.q[j][0]), __builtin_bit_cast(float4, pre.q[j][1])}.unpack(rv);
                else
#pragma unroll
                    for (int e = 0; e < 8; ++e) rv[e] = 0.f;
            } else if constexpr (READS) {
                Raw8<bf16_t>{pre.q[j][0]}.unpack(rv);
            }
            if (grow < m && gcol < n) finish8<E, CF>(v, bv, rv, (size_t)grow * n + gcol, C, C2, epi_flag);
        }
    };
    if (SHARE < 16 && lane >= SHARE * 4) return;
    if constexpr (ONLY_EPI == EPI_ACCUM_F32) finish.template operator()<EPI_ACCUM_F32, false, false>();
    else with_epilogue(epi, res_types, finish);
}

// ------------------------------------------------------------------ tiles of 128x128 and 256x256
// One output tile on v_mfma_f32_16x16x32_bf16, k in steps of 64 through LDS buffers, software
// pipelined across the barrier.  WGK = 1: wavefronts of 128x64 (256x256, 8 of them) or 64x64 (128x128,
// 4 of them, two workgroups per CU) and two buffers.  WGK = 2, for 128x128 with one workgroup per CU: 8
// wavefronts, two on each 64x64 block, each taking half of every step's k, over a ring of four buffers; for
// 256x128 the same with blocks of 128x64 and three buffers.
//
// What bounds it (256x256, counters of one round of 256 tiles, random operands): a step is 2048 clocks of MFMAs
// on each SIMD and takes 2220 to 2390, so the loop keeps the matrix pipes 86 to 92 % busy; launch, first tiles and
// the epilogue's HBM traffic cost another 18 000 clocks (51 000 with a float accumulate), as much as 8 (22) steps: over
// the whole kernel the pipes are busy 45 % at k = 512, 60 % at 1024, 79 % at 4096.  Power comes after that: the
// same launch on zeros is 14 % faster at 4096^3, 1 to 6 % at the sizes of the replays (2048 x 6400 x 1600 46.7 -> 45.7 us).
//   * Measured in a loop over register operands: 16x16x32 instructions 2046 TFLOP/s, 32x32x16 1816;
//     with every operand re-read from LDS at this tile's ratio 1706 and 1549.
//   * Requests of 128-byte rows (64 k) cost less than two of 64 bytes: 4096^3, A B^T, 102 -> 95.5 us.
// The schedule only has to keep the matrix pipes from waiting.  A wavefront's step is four phases,
// {its first 64 rows, its other 64} x {k 0..31, 32..63}; each reads the next phase's operands out of LDS.
//   * One memory instruction goes behind an MFMA at a time: requests in a burst fill the memory queue,
//     and the wavefront's own MFMAs would wait behind them.
//   * The requests of a step go out in the last phase of the step that frees its buffer and in the first
//     phase of the next: the wait ahead of the barrier finds them two phases old.
//   * No branch between the MFMAs of the steady state, buffer numbers known at compile time: both
//     wavefronts of a SIMD reach such a point together, and its matrix pipe idles.
// Measured against the five-slot 32-k ring on 32x32x16 before it, 4096^3: A B 120 -> 101 us, A B^T 110 -> 96,
// A^T B 126 -> 110; 2048 x 6400 x 1600 42 -> 38; the weight gradients of a block of 1600 at 2048 tokens
// with their column sums 154 -> 142.  128x128, two workgroups per CU: 4096 x 1600 x 6400 97 -> 77.
//
// With WGK = 2 a step of a wavefront is 16 MFMAs only, and two buffers would be requested a quarter of a
// microsecond ahead: less than memory answers in (4096 x 1024 x 50304 ran 16 % slower so).  Four buffers of
// 32 KiB let requests go out three steps ahead.  2048 x 1600 x 4800 41 -> 33 us, 4096 x 1024 x 4096 39 -> 33,
// 632 x 4800 x 1600 16.4 -> 14.1.
constexpr int RK = 64;
// [row][64 k] tile (128-byte rows): 16-byte chunk c of row r sits at c ^ rswz(r).  A 16-byte LDS read is served
// in four passes of 16 lanes, {0-3, 12-15, 20-23, 24-27} and so on; with lanes over rows l%16 and chunks l/16
// this order puts each pass on all 64 banks.  (The loop's reads meet no conflicts, in any layout: their counter does not
// grow with k.  The 7 to 30 % of LDS cycles it shows for a whole kernel are the epilogue's slabs, 4096 clocks a 256x256 tile.)
__device__ __forceinline__ int rswz(int r) { return (r >> 1) & 7; }
// [k][ROWS] tile: the 32-byte column block j of k-row k sits at j ^ rkswz(k): a transposing read touches one
// block in rows 8g..8g+3 of four lane groups g.
__device__ __forceinline__ int rkswz(int k) { return (k & 3) | ((k >> 1) & 4); }

// Buffers of a tile in LDS (its epilogue's slabs take their place): the kernel owns them, so that one kernel can hold several tile sizes.
template <int BM, int BN, int WGM, int WGN, int WGK> struct RingLds {
    static constexpr int STAGES = WGK == 1 ? 2 : BM * BN > 128 * 128 ? 3 : 4, STAGE = (BM + BN) * RK * 2;
    static constexpr int EPILOGUE = WGM * WGN * WGK * EpiSlab<BN / WGN / 32>::FLOATS * 4, RING = STAGES * STAGE;
    static constexpr int BYTES = RING > EPILOGUE ? RING : EPILOGUE;
    static constexpr int PER_CU = WGM * WGN * WGK == 4 ? 2 : 1;            // workgroups
};

// The tile of workgroup `id`, tiles numbered along the raster: of every round's an XCD takes a run of neighbours, so that the
// tiles in flight share operand panels in its L2 and, between the XCDs, in the memory-side cache.  With one run of the whole
// launch per XCD 4096 x 50304 x 1024 (twelve rounds) 421 -> 361 us, 8192 x 6144 x 2048 (three) 145.8 -> 143.1, two rounds up to 1 %.
template <int PER_CU> __device__ __forceinline__ int dealt(int id, int tiles) {
    constexpr int ROUND = NUM_CUS * PER_CU, PER = ROUND / XCDS;
    const int xcd = id % XCDS, at = id / XCDS, whole = tiles / ROUND, rest = tiles % ROUND;
    if (at < whole * PER) return at / PER * ROUND + xcd * PER + at % PER;
    return whole * ROUND + xcd * (rest / XCDS) + min(xcd, rest % XCDS) + at - whole * PER;
}

__device__ __forceinline__ void lds_dma16_s(const void* sbase, unsigned voff, unsigned lds_base) {
    asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "{m0}"(lds_base) : "memory");
}
template <int BM, int BN, int WGM, int WGN, int WGK, bool A_KC, bool B_KC, int ONLY_EPI>
__device__ __forceinline__ void gemm_ring_tile(
    char* lds, const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, const bf16_t* __restrict__ bias,
    const bf16_t* __restrict__ R, void* __restrict__ C, bf16_t* __restrict__ C2, int m, int n, int k, int lda,
    int ldb, int epi, int epi_flag, int res_types, int tiles_m, int tiles_n, int group_m, int block_id,
    float* __restrict__ bsum = nullptr, bool xcd_remap = true, int col0 = 0, const Ahead& ahead = {nullptr, 0}, int band = 0) {
    using Lds = RingLds<BM, BN, WGM, WGN, WGK>;
    constexpr int NT = WGM * WGN * WGK * 64, NS = Lds::STAGES;
    constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 16, TN = WN / 16, HM = TM / 2;      // 16x16 tiles per wavefront
    constexpr int CA = BM * (RK / 8) / NT, CB = BN * (RK / 8) / NT, CS = CA + CB;     // 16-byte pieces per thread and stage
    constexpr unsigned STAGE = Lds::STAGE, ABYTES = BM * RK * 2;

    const int nblk = tiles_m * tiles_n;
    int pid = xcd_remap ? dealt<Lds::PER_CU>(block_id, nblk) : block_id, first_n = 0, cols = tiles_n;
    if (band) {                                // see raster_band
        first_n = pid / (tiles_m * band) * band;
        pid -= first_n * tiles_m;
        cols = min(band, tiles_n - first_n);
    }
    const int width = group_m * cols;
    const int first_m = (pid / width) * group_m;
    const int gsz = min(tiles_m - first_m, group_m);
    const int tile_m = first_m + (pid % width) % gsz;
    const int tile_n = first_n + (pid % width) / gsz;
    const int i0 = tile_m * BM, j0 = col0 + tile_n * BN;

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave / (WGM * WGN), wmn = wave % (WGM * WGN);
    const int wm0 = (wmn / WGN) * WM, wn0 = (wmn % WGN) * WN;

    // Piece `slot` of a stage: its k inside the stage, and its byte offset from the tile's corner
    // (rows beyond the matrix repeat its last ones: their results are not stored).
    auto piece = [&](int ld, int row0, int nrows, auto rows_c, bool kc, int slot, int& kk) {
        constexpr int rows = decltype(rows_c)::value;
        if (kc) {
            const int row = slot >> 3;
            kk = ((slot & 7) ^ rswz(row)) * 8;
            return (unsigned)((min(row0 + row, nrows - 1) - row0) * ld + kk) * 2u;
        }
        kk = slot / (rows / 8);
        const int pc = slot % (rows / 8), ic = (((pc >> 1) ^ rkswz(kk)) << 1) | (pc & 1);
        return ((unsigned)kk * (unsigned)ld + (unsigned)(min(row0 + ic * 8, nrows - 8) - row0)) * 2u;     // kk < k: see far_operand
    };
    // Requests of an index-contiguous operand lie whole k rows apart: one lane offset and a pointer each.
    // Those of a k-contiguous one lie rows apart (clamped at the matrix's end): a lane offset each.
    constexpr int OA = A_KC ? CA : 1, OB = B_KC ? CB : 1, PA = A_KC ? 1 : CA, PB = B_KC ? 1 : CB;
    unsigned va[OA], vb[OB];
    int ka, kb;                                // k inside the step of a lane's pieces (request i adds i * KI of an index-contiguous operand)
    const char *sa[PA], *sb[PB];
    constexpr int KIA = NT / (BM / 8), KIB = NT / (BN / 8);
#pragma unroll
    for (int it = 0; it < OA; ++it) va[it] = piece(lda, i0, m, std::integral_constant<int, BM>{}, A_KC, it * NT + tid, ka);
#pragma unroll
    for (int it = 0; it < OB; ++it) vb[it] = piece(ldb, j0, n, std::integral_constant<int, BN>{}, B_KC, it * NT + tid, kb);
#pragma unroll
    for (int it = 0; it < PA; ++it) sa[it] = (const char*)(A + (A_KC ? (size_t)i0 * lda : (size_t)i0 + (size_t)it * KIA * lda));
#pragma unroll
    for (int it = 0; it < PB; ++it) sb[it] = (const char*)(B + (B_KC ? (size_t)j0 * ldb : (size_t)j0 + (size_t)it * KIB * ldb));
    static_assert(KIA % 16 == 0 && KIB % 16 == 0, "requests of one lane share a swizzle");
    const size_t step_a = (A_KC ? (size_t)RK : (size_t)RK * lda) * 2, step_b = (B_KC ? (size_t)RK : (size_t)RK * ldb) * 2;
    const unsigned lds0 = lds_address(lds), dma0 = lds0 + wave * 1024;

    // Operand reads: lane l holds k 8(l/16)..+7 of row (column) l%16 of a 16-row tile.
    typedef bf16x8 __attribute__((address_space(3))) * lds_v8;
    typedef bf16x4 __attribute__((address_space(3))) * lds_v4;
    // half h (32 k) of buffer q: the offset field of an LDS instruction reaches over one buffer (64 KiB)
    // Column block b of an index-contiguous operand sits at its first one's address with b exchanged in.
    constexpr int NPA = A_KC ? 2 : 1, NPB = B_KC ? 2 : 1;
    static_assert((TM & (TM - 1)) == 0 && TM <= 8 && (TN & (TN - 1)) == 0 && TN <= 8, "column blocks exchange within 256 bytes");
    unsigned pa[NPA], pb[NPB];
    auto read_base = [&](auto rows_c, bool kc, int row0, int h) {
        constexpr int rows = decltype(rows_c)::value;
        if (kc) return lds0 + (unsigned)((row0 + l16) * 128 + ((4 * h + g) ^ rswz(row0 + l16)) * 16);
        const int kk = 32 * h + 8 * g + (l16 >> 2);
        return lds0 + (unsigned)(kk * rows * 2 + ((row0 >> 4) ^ rkswz(kk)) * 32 + (l16 & 3) * 8);
    };
#pragma unroll
    for (int a = 0; a < NPA; ++a) pa[a] = read_base(std::integral_constant<int, BM>{}, A_KC, wm0, WGK == 2 ? wk : a);
#pragma unroll
    for (int b = 0; b < NPB; ++b) pb[b] = read_base(std::integral_constant<int, BN>{}, B_KC, wn0, WGK == 2 ? wk : b) + ABYTES;
    auto read_tr = [&](unsigned p, int rows) {                 // rows k and k + 4 share a swizzle
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_v4)(size_t)p);
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_v4)(size_t)(p + 8 * rows));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    bf16x8 fa[TM], fb[2][TN];
    // An address moves to the other buffer behind its last read from this one.
    auto read_a = [&](auto a_c, auto h_c, auto q_c) {
        constexpr int a = decltype(a_c)::value, h = decltype(h_c)::value, q = decltype(q_c)::value;
        constexpr unsigned move = q ? 0u - STAGE : STAGE, far = q / 2 * 2 * STAGE, near = q % 2 * STAGE;
        if constexpr (WGK == 2) {
            if constexpr (A_KC) fa[a] = *(lds_v8)(size_t)((pa[0] + far) + near + a * 2048);
            else fa[a] = read_tr(((pa[0] ^ (a * 32)) + far) + near, BM);
        } else if constexpr (A_KC) {
            fa[a] = *(lds_v8)(size_t)(pa[h] + a * 2048);
            if constexpr (a == TM - 1) pa[h] += move;
        } else {
            fa[a] = read_tr((pa[0] ^ (a * 32)) + h * 64 * BM, BM);
            if constexpr (h == 1 && a == TM - 1) pa[0] += move;
        }
    };
    auto read_b = [&](auto b_c, auto h_c, auto q_c) {
        constexpr int b = decltype(b_c)::value, h = decltype(h_c)::value, q = decltype(q_c)::value;
        constexpr unsigned move = q ? 0u - STAGE : STAGE, far = q / 2 * 2 * STAGE, near = q % 2 * STAGE;
        if constexpr (WGK == 2) {
            if constexpr (B_KC) fb[h][b] = *(lds_v8)(size_t)((pb[0] + far) + near + b * 2048);
            else fb[h][b] = read_tr(((pb[0] ^ (b * 32)) + far) + near, BN);
        } else if constexpr (B_KC) {
            fb[h][b] = *(lds_v8)(size_t)(pb[h] + b * 2048);
            if constexpr (b == TN - 1) pb[h] += move;
        } else {
            fb[h][b] = read_tr((pb[0] ^ (b * 32)) + h * 64 * BN, BN);
            if constexpr (h == 1 && b == TN - 1) pb[0] += move;
        }
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Optional by-product: bsum[j] += sum over the contraction index of B(k, j), one more MFMA per 16
    // columns with an all-ones A in the wavefronts at the top edge of the first tile row - in a loop of
    // their own: a choice per MFMA costs the others a third of their rate.
    const bool col_sums = ONLY_EPI == EPI_ACCUM_F32 && bsum != nullptr && tile_m == 0 && wm0 == 0;
    f32x4 cs[TN];
    bf16x8 ones;
#pragma unroll
    for (int q = 0; q < 8; ++q) ones[q] = (bf16_t)1.0f;
#pragma unroll
    for (int b = 0; b < TN; ++b) cs[b] = f32x4{0.f, 0.f, 0.f, 0.f};

    // HM x TN MFMAs of one phase, between(i) behind the i-th
    auto phase = [&](auto half_c, auto set_c, auto sums_c, auto&& between) {
        constexpr int half = decltype(half_c)::value, set = decltype(set_c)::value;
        constexpr bool sums = decltype(sums_c)::value;
        static_for<HM * TN>([&](auto i_c) {
            constexpr int i = decltype(i_c)::value, a = half * HM + i / TN, b = i % TN;
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][b], fa[a], acc[a][b], 0, 0, 0);
            if constexpr (sums && a == 0) cs[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, fb[set][b], cs[b], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            between(i_c);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    auto meet = [&] {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // lgkmcnt(0), and all but the N youngest requests have landed
    auto arrived = [](auto n_c) {
        constexpr int N = decltype(n_c)::value;
        __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
    };

    // The k values behind the last whole step come first, as step 0 (lanes beyond them store zeros in
    // place of their request); the whole steps follow.
    const int rest = k % RK, KT = k / RK + (rest ? 1 : 0);
    if (rest) {
        const size_t ea = (size_t)(k / RK) * step_a, eb = (size_t)(k / RK) * step_b;
        auto fill = [&](const char* base, unsigned off, int kk, unsigned to) {
            typedef f32x4 __attribute__((address_space(3))) * lds_f4;
            if (kk < rest) lds_dma16_s(base, off, to);
            else *(lds_f4)(size_t)(to + lane * 16) = f32x4{0.f, 0.f, 0.f, 0.f};
        };
#pragma unroll
        for (int it = 0; it < CA; ++it) fill(sa[A_KC ? 0 : it] + ea, va[A_KC ? it : 0], A_KC ? ka : ka + it * KIA, dma0 + it * NT * 16);
#pragma unroll
        for (int it = 0; it < CB; ++it) fill(sb[B_KC ? 0 : it] + eb, vb[B_KC ? it : 0], B_KC ? kb : kb + it * KIB, dma0 + ABYTES + it * NT * 16);
    }
    // Request i of a step into buffer q
    auto request = [&](auto i_c, auto q_c) {
        constexpr int i = decltype(i_c)::value, q = decltype(q_c)::value;
        if constexpr (i < CA) {
            lds_dma16_s(sa[A_KC ? 0 : i], va[A_KC ? i : 0], dma0 + q * STAGE + i * NT * 16);
            if constexpr (!A_KC || i == CA - 1) sa[A_KC ? 0 : i] += step_a;
        } else {
            constexpr int j = i - CA;
            lds_dma16_s(sb[B_KC ? 0 : j], vb[B_KC ? j : 0], dma0 + q * STAGE + ABYTES + j * NT * 16);
            if constexpr (!B_KC || j == CB - 1) sb[B_KC ? 0 : j] += step_b;
        }
    };
#define CHIMERA_C(V) std::integral_constant<int, (V)>{}
    auto steps = [&](auto sums_c) {
        if constexpr (WGK == 1) {
            constexpr int ROOM_B = HM * TN - TN - HM, ROOM_A = HM * TN - HM;
            constexpr int D3 = CS / 2 < ROOM_B ? CS / 2 : ROOM_B, D0 = CS - D3;       // a step's requests in their first and second phase
            if (!rest) static_for<CS>([&](auto i) { request(i, CHIMERA_C(0)); });
            if (KT > 1) { static_for<CS>([&](auto i) { if constexpr (decltype(i)::value < D3) request(i, CHIMERA_C(1)); }); arrived(CHIMERA_C(D3)); }
            else arrived(CHIMERA_C(0));
            meet();
            static_for<TN>([&](auto b) { read_b(b, CHIMERA_C(0), CHIMERA_C(0)); });
            static_for<HM>([&](auto a) { read_a(a, CHIMERA_C(0), CHIMERA_C(0)); });

            // Step t in buffer q = t mod 2.  ALWAYS: further requests are due (the steady state: no branch between the
            // MFMAs - both wavefronts of a SIMD reach it at the same time, and the matrix pipe idles).
            constexpr int G3 = ROOM_B / D3, G0 = ROOM_A / D0;
            static_assert(G3 >= 1 && G0 >= 1, "room for a step's requests");
            auto step = [&](auto q_c, auto always_c, int t) {
                constexpr int q = decltype(q_c)::value;
                constexpr bool always = decltype(always_c)::value;
                const bool more1 = always || t + 1 < KT, more2 = always || t + 2 < KT;
                phase(CHIMERA_C(0), CHIMERA_C(0), sums_c, [&](auto i_c) {
                    constexpr int i = decltype(i_c)::value;
                    if constexpr (i < HM) read_a(CHIMERA_C(HM + i), CHIMERA_C(0), q_c);
                    else if constexpr ((i - HM) % G0 == 0 && (i - HM) / G0 < D0) { if (more1) request(CHIMERA_C(D3 + (i - HM) / G0), CHIMERA_C(q ^ 1)); }
                });
                phase(CHIMERA_C(1), CHIMERA_C(0), sums_c, [&](auto i_c) {
                    constexpr int i = decltype(i_c)::value;
                    if constexpr (i < TN) read_b(i_c, CHIMERA_C(1), q_c);
                    else if constexpr (i < TN + HM) read_a(CHIMERA_C(i - TN), CHIMERA_C(1), q_c);
                });
                phase(CHIMERA_C(0), CHIMERA_C(1), sums_c, [&](auto i_c) {
                    constexpr int i = decltype(i_c)::value;
                    if constexpr (i < HM) read_a(CHIMERA_C(HM + i), CHIMERA_C(1), q_c);
                });
                arrived(CHIMERA_C(0));
                meet();
                phase(CHIMERA_C(1), CHIMERA_C(1), sums_c, [&](auto i_c) {
                    constexpr int i = decltype(i_c)::value;
                    if constexpr (i < TN) read_b(i_c, CHIMERA_C(0), CHIMERA_C(q ^ 1));
                    else if constexpr (i < TN + HM) read_a(CHIMERA_C(i - TN), CHIMERA_C(0), CHIMERA_C(q ^ 1));
                    else if constexpr ((i - TN - HM) % G3 == 0 && (i - TN - HM) / G3 < D3) { if (more2) request(CHIMERA_C((i - TN - HM) / G3), q_c); }
                });
            };
            int t = 0;
            for (; t + 3 < KT; t += 2) { step(CHIMERA_C(0), std::true_type{}, 0); step(CHIMERA_C(1), std::true_type{}, 0); }
            for (; t < KT; t += 2) {
                step(CHIMERA_C(0), std::false_type{}, t);
                if (t + 1 < KT) step(CHIMERA_C(1), std::false_type{}, t + 1);
            }
        } else {
            // Wavefronts of either k half share the stages of a ring of NS slots.  In step t they request stage
            // t + NS - 1 into the slot that step t - 1 was the last to read.
            if (!rest) static_for<CS>([&](auto i) { request(i, CHIMERA_C(0)); });
            static_for<NS - 2>([&](auto j) {
                constexpr int q = decltype(j)::value + 1;
                if (q < KT) static_for<CS>([&](auto i) { request(i, CHIMERA_C(q)); });
            });
            // all but the `younger` stages behind it have landed
            auto landed = [&](int younger) {
                if (younger >= NS - 2) arrived(CHIMERA_C((NS - 2) * CS));
                else if (NS == 4 && younger == 1) arrived(CHIMERA_C(CS));
                else arrived(CHIMERA_C(0));
            };
            static_assert(NS == 3 || NS == 4, "landed() counts up to two younger stages");
            landed(KT - 1);
            meet();
            static_for<TN>([&](auto b) { read_b(b, CHIMERA_C(0), CHIMERA_C(0)); });
            static_for<HM>([&](auto a) { read_a(a, CHIMERA_C(0), CHIMERA_C(0)); });
            // step u of an unrolled group: slot u mod NS, operand set u mod 2
            auto step = [&](auto u_c, auto always_c, int t) {
                constexpr int u = decltype(u_c)::value, q = u % NS, next = (q + 1) % NS, set = u & 1;
                constexpr bool always = decltype(always_c)::value;
                const bool more = always || t + NS - 1 < KT;
                phase(CHIMERA_C(0), CHIMERA_C(set), sums_c, [&](auto i_c) {
                    constexpr int i = decltype(i_c)::value;
                    if constexpr (i < HM) read_a(CHIMERA_C(HM + i), CHIMERA_C(0), CHIMERA_C(q));
                    else if constexpr (i < HM + CS) { if (more) request(CHIMERA_C(i - HM), CHIMERA_C((q + NS - 1) % NS)); }
                });
                static_assert(HM + CS <= HM * TN && TN + HM <= HM * TN, "room behind the MFMAs");
                if constexpr (always) arrived(CHIMERA_C((NS - 2) * CS));
                else landed(KT - 2 - t);
                meet();
                phase(CHIMERA_C(1), CHIMERA_C(set), sums_c, [&](auto i_c) {
                    constexpr int i = decltype(i_c)::value;
                    if constexpr (i < TN) read_b(i_c, CHIMERA_C(set ^ 1), CHIMERA_C(next));
                    else if constexpr (i < TN + HM) read_a(CHIMERA_C(i - TN), CHIMERA_C(0), CHIMERA_C(next));
                });
            };
            int t = 0;
            constexpr int U = NS % 2 ? 2 * NS : NS;
            for (; t + U + NS - 2 < KT; t += U) static_for<U>([&](auto u) { step(u, std::true_type{}, 0); });
            for (; t < KT; t += U) static_for<U>([&](auto u) { if (t + u < KT) step(u, std::false_type{}, t + u); });
        }
    };
    if constexpr (ONLY_EPI == EPI_ACCUM_F32) {
        if (col_sums) steps(std::true_type{});
        else steps(std::false_type{});
    } else {
        steps(std::false_type{});
    }
#undef CHIMERA_C
    if constexpr (ONLY_EPI < 0) touch_ahead(ahead, wave, NT / 64, lane);       // weight gradients and split products precede no product

    const int cb0 = j0 + wn0;
    auto put_col_sums = [&](const float* v) {
#pragma unroll
        for (int b = 0; b < TN; ++b) {
            const int col = cb0 + b * 16 + lane;
            if (lane < 16 && col < n) bsum[col] = (epi_flag & ACCUM_OVERWRITE) ? v[b] : bsum[col] + v[b];
        }
    };
    float* slab = reinterpret_cast<float*>(lds) + (size_t)wave * EpiSlab<TN / 2>::FLOATS;
    auto finish = [&](const auto& out, auto rows_c, int rb0) {
        constexpr int TO = decltype(rows_c)::value;              // 32-row bands of this wavefront
        auto run = [&]<int E, bool RF, bool CF>() { epilogue<E, RF, CF, TO, TN / 2>(out, slab, rb0, cb0, m, n, bias, R, C, C2, epi_flag, lane); };
        if constexpr (ONLY_EPI == EPI_ACCUM_F32) run.template operator()<EPI_ACCUM_F32, false, false>();
        else with_epilogue(epi, res_types, run);
    };
    __syncthreads();                           // the buffers become the wavefronts' slabs
    if constexpr (WGK == 1) {
        if constexpr (ONLY_EPI == EPI_ACCUM_F32)
            if (col_sums) {                    // every row of these accumulators is the column sum
                float v[TN];
#pragma unroll
                for (int b = 0; b < TN; ++b) v[b] = cs[b][0];
                put_col_sums(v);
            }
        finish(Acc16<TM / 2, TN / 2>{acc}, std::integral_constant<int, TM / 2>{}, i0 + wm0);
    } else {
        // Two wavefronts hold partial sums of the same block.  Each keeps the upper or lower half of its rows:
        // it hands the other half to its partner through LDS and adds what the partner hands over.
        static_assert(WGK == 2 && TM % 4 == 0, "bands of 32 rows");
        constexpr int PER_WAVE = HM * TN * 64;                   // 16 bytes each
        static_assert(Lds::BYTES >= NT / 64 * PER_WAVE * 16 + BN * (int)sizeof(float), "LDS too small for the exchange");
        f32x4* xch = reinterpret_cast<f32x4*>(lds);
        float* xcs = reinterpret_cast<float*>(xch + NT / 64 * PER_WAVE) + wn0;
        if constexpr (ONLY_EPI == EPI_ACCUM_F32)
            if (col_sums && wk == 1 && lane < 16)
#pragma unroll
                for (int b = 0; b < TN; ++b) xcs[b * 16 + lane] = cs[b][0];
        f32x4* send = xch + (size_t)wave * PER_WAVE + lane;
        const f32x4* recv = xch + (size_t)(wave ^ (WGM * WGN)) * PER_WAVE + lane;
        f32x4 own[HM][TN];
#pragma unroll
        for (int a = 0; a < HM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b) {
                send[(a * TN + b) * 64] = wk ? acc[a][b] : acc[HM + a][b];
                own[a][b] = wk ? acc[HM + a][b] : acc[a][b];
            }
        __syncthreads();
#pragma unroll
        for (int a = 0; a < HM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b) own[a][b] += recv[(a * TN + b) * 64];
        if constexpr (ONLY_EPI == EPI_ACCUM_F32)
            if (col_sums && wk == 0) {
                float v[TN];
#pragma unroll
                for (int b = 0; b < TN; ++b) v[b] = cs[b][0] + (lane < 16 ? xcs[b * 16 + lane] : 0.f);
                put_col_sums(v);
            }
        __syncthreads();                       // the exchange area becomes the slabs
        finish(Acc16<TM / 4, TN / 2>{own}, std::integral_constant<int, TM / 4>{}, i0 + wm0 + wk * HM * 16);
    }
}

template <int BM, int BN, int WGM, int WGN, int WGK, bool A_KC, bool B_KC>
__global__ __launch_bounds__(WGM* WGN * WGK * 64, 2) void gemm_bf16_ring_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, const bf16_t* __restrict__ bias,
    const bf16_t* __restrict__ R, void* __restrict__ C, bf16_t* __restrict__ C2, int m, int n, int k, int lda,
    int ldb, int epi, int epi_flag, int res_types, int tiles_m, int tiles_n, int group_m, int band, int col0, Ahead ahead) {
    __shared__ __attribute__((aligned(1024))) char lds[RingLds<BM, BN, WGM, WGN, WGK>::BYTES];
    gemm_ring_tile<BM, BN, WGM, WGN, WGK, A_KC, B_KC, -1>(lds, A, B, bias, R, C, C2, m, n, k, lda, ldb, epi, epi_flag, res_types,
                                                          tiles_m, tiles_n, group_m, (int)blockIdx.x, nullptr, true, col0, ahead, band);
}

// A long contraction with few output tiles, cut along k: workgroups [s * tiles, (s+1) * tiles) (numbered so
// that an XCD works on few splits) write the partial sums over k in [s * k_per, (s+1) * k_per) to float slab s;
// split_sum_kernel adds the slabs in their order.  No workgroup waits for another.
template <int BM, int BN, int WGM, int WGN, int WGK>
__global__ __launch_bounds__(WGM* WGN * WGK * 64, 2) void gemm_bf16_ring_split_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, float* __restrict__ slabs, int m, int n, int k, int lda, int ldb,
    int tiles_m, int tiles_n, int group_m, int splits, int k_per) {
    const int tiles = tiles_m * tiles_n, total = tiles * splits;
    const int xcd = (int)blockIdx.x & 7, local = (int)blockIdx.x >> 3;
    const int pid = xcd * (total >> 3) + min(xcd, total & 7) + local;
    const int split = pid / tiles, k0 = split * k_per;
    __shared__ __attribute__((aligned(1024))) char lds[RingLds<BM, BN, WGM, WGN, WGK>::BYTES];
    gemm_ring_tile<BM, BN, WGM, WGN, WGK, true, true, EPI_ACCUM_F32>(
        lds, A + k0, B + k0, nullptr, nullptr, slabs + (size_t)split * m * n, nullptr, m, n, min(k_per, k - k0), lda, ldb,
        EPI_ACCUM_F32, 1, 0, tiles_m, tiles_n, group_m, pid % tiles, nullptr, false);
}

__global__ __launch_bounds__(256) void split_sum_kernel(const float* __restrict__ slabs, size_t elems, int splits, bf16_t* __restrict__ c) {
    const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8;
    if (i >= elems) return;
    float v[8];
    load8(slabs + i, v);
    for (int s = 1; s < splits; ++s) {
        float u[8];
        load8(slabs + (size_t)s * elems + i, u);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += u[e];
    }
    store8(c + i, v);
}

template <int BM, int BN, int WGM, int WGN, int WGK, int NS, int SPS, bool A_KC, bool B_KC>
__global__ __launch_bounds__(WGM* WGN * WGK * 64) void gemm_bf16_async_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, const bf16_t* __restrict__ bias,
    const bf16_t* __restrict__ R, void* __restrict__ C, bf16_t* __restrict__ C2, int m, int n, int k, int lda,
    int ldb, int epi, int epi_flag, int res_types, int tiles_m, int tiles_n, int group_m, Ahead ahead) {
    gemm_async_tile<BM, BN, WGM, WGN, WGK, NS, SPS, A_KC, B_KC, -1>(A, B, bias, R, C, C2, m, n, k, lda, ldb, epi, epi_flag,
                                                                res_types, tiles_m, tiles_n, group_m, (int)blockIdx.x, nullptr,
                                                                true, ahead);
}

// Several products C_p (float) += A_p B_p of one launch: same contraction length and operand
// layout, each with its own shapes and pointers.  Workgroups [first[p], first[p+1]) work on
// product p, so small products no longer leave most of the chip idle for a launch of their
// own.  (The weight gradients of one Transformer block are such a group.)
constexpr int GROUP_MAX = 4;
struct GemmGroup {
    const bf16_t* a[GROUP_MAX];
    const bf16_t* b[GROUP_MAX];
    float* c[GROUP_MAX];
    float* bsum[GROUP_MAX];      // optional: bsum[j] += sum_k B(k, j)
    int m[GROUP_MAX], n[GROUP_MAX], lda[GROUP_MAX], ldb[GROUP_MAX], tiles_m[GROUP_MAX], tiles_n[GROUP_MAX];
    int group_m[GROUP_MAX];      // tile rows per raster group of each product
    int first[GROUP_MAX + 1];
    int count, k;
    int overwrite;               // results replace C and bsum instead of being added
};

// The product of a group launch that this workgroup belongs to, and its tile's number inside the
// group: each XCD takes a contiguous range of the group's tiles (products laid end to end), so that
// its L2 sees few operand panels: one product's tiles are not dealt over all eight XCDs.
__device__ __forceinline__ int group_product(const GemmGroup& grp, int& gid) {
    const int total = grp.first[grp.count];
    const int xcd = (int)blockIdx.x & 7, local = (int)blockIdx.x >> 3;
    gid = xcd * (total >> 3) + min(xcd, total & 7) + local;
    int p = 0;
#pragma unroll
    for (int i = 1; i < GROUP_MAX; ++i)
        if (i < grp.count && gid >= grp.first[i]) p = i;
    return p;
}

template <int BM, int BN, int WGM, int WGN, int WGK>
__global__ __launch_bounds__(WGM* WGN * WGK * 64, 2) void gemm_bf16_ring_group_kernel(GemmGroup grp) {
    int gid;
    const int p = group_product(grp, gid);
    __shared__ __attribute__((aligned(1024))) char lds[RingLds<BM, BN, WGM, WGN, WGK>::BYTES];
    gemm_ring_tile<BM, BN, WGM, WGN, WGK, false, false, EPI_ACCUM_F32>(
        lds, grp.a[p], grp.b[p], nullptr, nullptr, grp.c[p], nullptr, grp.m[p], grp.n[p], grp.k, grp.lda[p], grp.ldb[p],
        EPI_ACCUM_F32, grp.overwrite, 0, grp.tiles_m[p], grp.tiles_n[p], grp.group_m[p], gid - grp.first[p], grp.bsum[p],
        false);
}

template <int BM, int BN, int WGM, int WGN, int WGK, int NS, int SPS, bool A_KC, bool B_KC>
__global__ __launch_bounds__(WGM* WGN * WGK * 64) void gemm_bf16_async_group_kernel(GemmGroup grp) {
    int gid;
    const int p = group_product(grp, gid);
    gemm_async_tile<BM, BN, WGM, WGN, WGK, NS, SPS, A_KC, B_KC, EPI_ACCUM_F32>(
        grp.a[p], grp.b[p], nullptr, nullptr, grp.c[p], nullptr, grp.m[p], grp.n[p], grp.k, grp.lda[p], grp.ldb[p],
        EPI_ACCUM_F32, grp.overwrite, 0, grp.tiles_m[p], grp.tiles_n[p], grp.group_m[p], gid - grp.first[p], grp.bsum[p],
        false);
}

// The same on tiles of several sizes in one launch.  An entry is the tiles of one size of one product, a phase the entries of all products
// that are begun together.  Of every 256 tiles of a phase an XCD takes 32 neighbours, so that the tiles in flight share operand panels in
// its L2 and, between the XCDs, in the memory-side cache (one range of the whole phase per XCD: block of 2048 at k = 512 121 -> 128 us, of
// 1920 at 2048 204 -> 220; one range of each product's tiles: block of 1280 at 2048 104 -> 128).
enum TileForm { TILE_256, TILE_128x256, TILE_256x128, TILE_128 };
constexpr int MIXED_MAX = 5 * GROUP_MAX;
struct MixedEntry {
    const bf16_t *a, *b;
    float *c, *bsum;
    int m, n, lda, ldb, tiles_m, tiles_n, group_m, band, col0;
    int form;
};
constexpr int MIXED_PHASES = 3;
struct MixedPhase {
    int first, tiles;                // its tiles
    int local;                       // number, within an XCD, of its first workgroup
    int skew;                        // the XCD that takes the first of the tiles that eight do not divide
};
struct MixedGroup {
    MixedPhase phase[MIXED_PHASES];
    int first[MIXED_MAX];            // number of an entry's first tile, all laid end to end (INT_MAX behind the last entry)
    int count, k, flags;             // flags: ACCUM_*
    MixedEntry e[MIXED_MAX];
};

__global__ __launch_bounds__(512, 2) void gemm_bf16_mixed_group_kernel(MixedGroup grp) {
    __shared__ __attribute__((aligned(1024))) char lds[RingLds<256, 128, 2, 2, 2>::BYTES];
    static_assert(RingLds<256, 256, 2, 4, 1>::BYTES <= sizeof(lds) && RingLds<128, 256, 1, 4, 2>::BYTES <= sizeof(lds) &&
                  RingLds<128, 128, 2, 2, 2>::BYTES <= sizeof(lds), "the largest of them");
    const int local = (int)blockIdx.x >> 3, h = local >= grp.phase[2].local ? 2 : local >= grp.phase[1].local ? 1 : 0;
    const MixedPhase& p = grp.phase[h];
    const int slot = ((int)blockIdx.x - p.skew) & 7, at = local - p.local, rounds = p.tiles / NUM_CUS, rest = p.tiles % NUM_CUS;
    int gid = p.first + at / PER_XCD * NUM_CUS + slot * PER_XCD + at % PER_XCD;
    if (at >= rounds * PER_XCD) {
        const int last = at - rounds * PER_XCD;
        if (last >= rest / XCDS + (slot < rest % XCDS ? 1 : 0)) return;
        gid = p.first + rounds * NUM_CUS + slot * (rest / XCDS) + min(slot, rest % XCDS) + last;
    }
    int i = 0;
#pragma unroll
    for (int j = 1; j < MIXED_MAX; ++j)
        if (gid >= grp.first[j]) i = j;
    const MixedEntry& e = grp.e[i];
    const int tile = gid - grp.first[i];
#define CHIMERA_MIXED(...)                                                                                                  \
    gemm_ring_tile<__VA_ARGS__, false, false, EPI_ACCUM_F32>(lds, e.a, e.b, nullptr, nullptr, e.c, nullptr, e.m, e.n, grp.k, \
        e.lda, e.ldb, EPI_ACCUM_F32, grp.flags, 0, e.tiles_m, e.tiles_n, e.group_m, tile, e.bsum, false, e.col0, Ahead{nullptr, 0}, e.band)
    if (e.form == TILE_256) CHIMERA_MIXED(256, 256, 2, 4, 1);
    else if (e.form == TILE_128x256) CHIMERA_MIXED(128, 256, 1, 4, 2);
    else if (e.form == TILE_256x128) CHIMERA_MIXED(256, 128, 2, 2, 2);
    else CHIMERA_MIXED(128, 128, 2, 2, 2);
#undef CHIMERA_MIXED
}

// A launch of 256x256 tiles runs in rounds of NUM_CUS tiles, and a last round with few tiles
// costs as much as a full one.  The products here can be cut along m without touching the data
// (row bands of A and C are just pointer offsets), so the last `b` bands of 256 rows may go to a
// second launch with 128x128 tiles instead.  Cost estimate in units of one 256x256 round: a round
// of 128x128 tiles (a quarter of the flops) counts 0.45.  Measured, launch included: 0.36 to 0.39 of a 256x256
// round at one tile per CU (k = 1600: 18.4 against 49.5 us A B, 24.5 against 68 A^T B), 0.34 each of two rounds
// at two per CU; the rest stands for what an estimate in whole rounds leaves out.  Returns the b
// that minimises it (0: leave the product whole).  Columns are counted by the same rule with rows and columns exchanged.
int bands_to_peel(int tm, int tn, int n, double* cost) {
    const int tn128 = (n + 127) / 128;
    auto rounds = [](long tiles) { return (double)((tiles + NUM_CUS - 1) / NUM_CUS); };
    const double whole = rounds((long)tm * tn);
    int best_b = 0;
    double best = whole - 0.25;                                  // a split must pay for its second launch
    for (int b = 1; b < tm; ++b) {
        const double est = rounds((long)(tm - b) * tn) + 0.45 * rounds((long)b * 2 * tn128);
        if (est < best) { best = est; best_b = b; }
    }
    *cost = best;
    return best_b;
}

// Tile rows per raster group.  A launch's tiles are dealt to the 8 XCDs in contiguous ranges of
// `per_xcd` tiles, walked column by column inside groups of g tile rows, so an XCD works on
// about g rows x per_xcd / g columns of tiles and its L2 has to fetch g row panels of A and
// per_xcd / g column panels of B - everything an L2 misses arrives at HBM speed (about 7 TB/s
// for the whole chip, a quarter of what the L2s deliver), whether or not it is in the memory-
// side cache.  Returns the g that minimises the bytes fetched (tile heights bm, widths bn),
// counting the ragged last group at its share of the rows.
int raster_group(int tiles_m, int tiles_n, int per_xcd, int bm, int bn) {
    int best_g = 1;
    double best = 1e300;
    for (int g = 1; g <= std::min(tiles_m, 16); ++g) {
        double cost = 0;
        for (int r0 = 0; r0 < tiles_m; r0 += g) {
            const int rows = std::min(g, tiles_m - r0);
            const int cols = std::min(tiles_n, (per_xcd + rows - 1) / rows);
            cost += ((double)rows * bm + (double)cols * bn) * rows;       // weighted by the group's share of the tiles
        }
        if (cost < best * 0.999) { best = cost; best_g = g; }
    }
    return best_g;
}

// Launches of several rounds whose B (`bytes`) the memory-side cache does not keep beside what else they move: tile columns per band.  All tile
// rows of a band come before the next band, so that B comes from HBM once and not for every raster group, and the tiles of a round, which are
// in flight together, are about as many rows as columns.  0: one band.  Without -> with, final layer forward and backward, 3339 tokens of
// 1624, vocabulary 58632 (190 MB) 2308 -> 2282 us; 8192 of 2048, 65536 (268 MB) 5843 -> 5676; but 4096 of 1024, 50304 (103 MB) 1330 -> 1351, 4096 x
// 8192 x 2048 (34 MB) 98.5 -> 100.8.
constexpr size_t B_IN_CACHE = (size_t)128 << 20;
int raster_band(int tiles_m, int tiles_n, int round, size_t bytes) {
    if (tiles_m * tiles_n <= round || bytes <= B_IN_CACHE) return 0;
    int side = 1;
    while (side * side < round) ++side;
    const int band = std::max(side, round / tiles_m);
    return band < tiles_n ? band : 0;
}

struct TileChoice { int bm, bn, splits; };

// The kernels' `epi_flag` argument modifies the epilogue: for the GeLU epilogues 1 selects the
// erf form (0: tanh form); for the float-accumulate epilogue it holds ACCUM_* flags, none in a single product
// (ACCUM_OVERWRITE: the column sums replace bsum too).
inline int epilogue_flag(const GemmArgs& g) { return g.epilogue == EPI_ACCUM_F32 ? 0 : g.gelu_erf; }
// A forward that keeps nothing leaves out u, half of what the first product of an MLP writes: six blocks of 1600 at 1264 tokens
// 775 -> 761 us, bert48 with doubled forwards 52.1 -> 51.4 ms.
inline void* result(const GemmArgs& g) { return g.epilogue == EPI_BIAS_GELU && g.c_unused ? nullptr : g.c; }

inline Ahead ahead_of(const GemmArgs& g) { return {(const char*)g.ahead, (unsigned)g.ahead_bytes}; }

// Tuning aids, read from the environment once (first use) and changeable through
// chimera_gemm_tuning(): a forced tile ("256x256", "128x128" or "256x256x<splits>" in
// CHIMERA_GEMM_TILE) and the form of the LDS-DMA kernels (CHIMERA_GEMM_ASYNC: "0" = the
// register-staged kernels, "4k" = the k-sliced 128x128 form always, "2" = never).
enum AsyncMode { ASYNC_AUTO = 0, ASYNC_OFF = 1, ASYNC_KSLICED = 2, ASYNC_PLAIN = 3 };
struct Tuning { TileChoice forced{0, 0, 0}; int async_mode = ASYNC_AUTO; unsigned long long version = 0; };
Tuning& tuning() {
    static Tuning t = [] {
        Tuning v;
        if (const char* e = std::getenv("CHIMERA_GEMM_TILE")) std::sscanf(e, "%dx%dx%d", &v.forced.bm, &v.forced.bn, &v.forced.splits);
        if (const char* e = std::getenv("CHIMERA_GEMM_ASYNC"))
            v.async_mode = e[0] == '0' ? ASYNC_OFF : (!std::strcmp(e, "4k") ? ASYNC_KSLICED : ASYNC_PLAIN);
        return v;
    }();
    return t;
}
TileChoice forced_tile() { return tuning().forced; }

constexpr int MAX_SPLITS = 8;

// gemm_ring_tile addresses a lane's pieces by 32-bit byte offsets from the tile's corner: up to 255 rows away
// in a k-contiguous operand, up to 31 rows of k (as many as there are) and 255 elements in an index-contiguous one.
// Operands that reach further go to the register-staged kernel, whose element offsets reach 2^32.  (A group's never do
// where k is 64 or more: k * ld < 2^32 bounds ld; a stage's rows are at most 16384 elements long.)
bool far_operand(const GemmArgs& g) {
    const long k_rows = std::min(g.k, 32) - 1;
    auto far = [&](int k_contiguous, long ld) { return k_contiguous ? ld >= 1l << 23 : k_rows * ld + 256 >= 1l << 31; };
    return far(g.a_kc, g.lda) || far(g.b_kc, g.ldb);
}

// 64x64 tiles while they all fit on the chip at once, two per CU: a smaller product is bound by
// its chain of latencies and by how many CUs pull its operands, not by the bytes a small tile
// costs.  Measured, 128x128 -> 64x64: 632 x 1600 x 1600 (65 tiles of 128x128, 250 of 64x64) 13.7 -> 9.2 us,
// 632 x 1600 x 6400 55 -> 31, 1024 x 1280 x 5120 (80, 320) 48.6 -> 42.4, 1264 x 1600 x 6400 (130, 500) 55.0 -> 52.3,
// 1024 x 2048 x 2048 (128, 512) 16.2 -> 16.5; beyond it turns: 1024 x 2560 x 640 (160, 640) 9.8 -> 11.9,
// 632 x 4800 x 1600 (190, 750) 17.7 -> 23.9, 1264 x 2400 x 6400 (190, 760) 60.6 -> 82.9.
bool small_tiles(long tiles64) { return tiles64 <= 2 * NUM_CUS && tuning().async_mode == ASYNC_AUTO; }

// The tile of such a product: the largest with which it still has a tile for every CU or nearly so.  A CU takes 60 to 90 bytes a
// nanosecond, so what bounds a small output's k loop is what its few workgroups have to read, (bm + bn) a step each; once
// the chip is full a larger tile reads less in all.  Measured, 64x64 -> 32x32: 256 x 256 x 256 3.74 -> 3.30 us, x 1024 5.5 -> 3.9,
// 400 x 320 x 1280 6.2 -> 4.2, 128 x 1600 x 6400 (200 tiles) 20.1 -> 11.8, 512 x 512 x 2048 (256) 8.2 -> 5.0; 32x64: 1024 x 512 x 2048
// (256) 8.8 -> 7.1 (32x32 8.4), 333 x 776 x 3104 13.7 -> 10.9 (12.4), 400 x 960 x 320 3.9 -> 3.7 (4.0).
// 64x64, two per CU -> 128x64: 1264 x 1600 x 6400 (250) 46.7 -> 39.5, x 1600 13.9 -> 12.1, 1024 x 2048 x 2048 (256) 16.6 -> 14.2,
// 2048 x 768 x 3072 21.5 -> 17.2, 512 x 3072 x 1024 10.7 -> 9.3; beside another stage 10.6 -> 11.1 each at k = 1600, 13.3 -> 12.6 at 2048.
// From k = 128 on: at 64 and 96 it is 1 to 5 % slower (1152 x 1280 x 64 A B 4.21 -> 4.44 us, A B^T 4.27 -> 4.40), at 128 as fast, from 256 on 3 to
// 13 % faster.  With the GeLU derivative, whose epilogue is the longest, from 640 on: x 192 2 to 3 % slower, x 512 1 to 2, x 640 as fast, x 768
// 2 to 4 % faster.
// Beside another stage the tiles below 64x64 may take half of the CUs: they read more in all, and what one stage's tiles take the
// other's do without.  Replays of two stages with the limit at all CUs -> at half: two blocks of 512 at 1024 tokens 1409 -> 1371 us
// (64x64 tiles throughout: 1398), of 512 at 512 1259 -> 1238, of 1024 at 128 1483 -> 1443 and at 256 1728 -> 1684, of 1600 at 128 2610 -> 2538; of 256 at
// 256, whose products need 64 to 192 such tiles, 859 -> 857 (at three quarters of the CUs 853).
// (Weight gradients stay on 64x64 tiles, so that one alone has the bits of one in a group.)
TileChoice small_tile(const GemmArgs& g) {
    if (!g.a_kc) return {64, 64, 1};
    auto fits = [&](int bm, int bn, int cus) { return (long)((g.m + bm - 1) / bm) * ((g.n + bn - 1) / bn) <= cus; };
    const int few = g.beside ? NUM_CUS / 2 : NUM_CUS;
    if (fits(32, 32, few)) return {32, 32, 1};
    if (fits(32, 64, few)) return {32, 64, 1};
    const int long_k = g.beside ? 2048 : g.epilogue == EPI_DGELU ? 640 : 128;
    if (!fits(64, 64, NUM_CUS) && fits(128, 64, NUM_CUS) && g.k >= long_k) return {128, 64, 1};
    return {64, 64, 1};
}

// 256x128 tiles for a product that shares the chip with another stage's: it should then take little of the
// chip's time, not little time.  Alone it is slower than 128x128, whose tiles are twice as many (4096 x 1024 x
// 4096 40 -> 56 us, 2048 x 1600 x 6400 57 -> 82), but it spends a third fewer CU-microseconds, a quarter less
// traffic into LDS and a third less out of it, and the other stage has work for the CUs it leaves.  Replays of
// two stages, 128x128 -> 256x128: bert48 21.1 -> 20.6 ms, gpt2-1p3b-n32 103.4 -> 100.2, gpt2-deep 52.3 -> 50.5, three
// blocks of 2048 at 3000 tokens 13.2 -> 12.7.  With fewer than 100 tiles the two stages together leave the chip
// half empty (1024 wide at 3000 tokens, 96 tiles: 8.2 -> 8.4 ms; 768 at 4096, 96: 7.3 -> 7.5), with k below 1024 the larger
// epilogue weighs more than the loop saves (512 wide at 4096 tokens, 192 tiles: 4.69 -> 4.77).  The two-per-CU form of
// 64x64 tiles (257 to 512 of them) gives way earlier, from 60 tiles on, where k is long: four blocks of 2048 at 1024
// tokens 8.06 -> 7.53 ms, six of 1024 at 2048 tokens 6.71 -> 6.59; not at 512 wide, k up to 2048 (4.69 -> 4.74).
bool wide_tiles(const GemmArgs& g) {
    if (!g.beside || tuning().async_mode != ASYNC_AUTO) return false;
    const long t2 = (long)((g.m + 255) / 256) * ((g.n + 127) / 128), t64 = (long)((g.m + 63) / 64) * ((g.n + 63) / 64);
    if (t2 > NUM_CUS) return false;
    return (t2 >= 100 && g.k >= 1024) || (t2 >= 60 && t64 > NUM_CUS && small_tiles(t64) && g.k > 2048);
}

// 256x256 (8 wavefronts) once the output has enough such tiles for most of the 256 CUs,
// else 128x128 (4 wavefronts, two workgroups per CU); thresholds measured on MI355X.
// A CU fills LDS from L2 at roughly 64 bytes per clock, so a 128x128x64 step (32 KiB for
// 512 clocks of MFMA work) is fed at half the rate the matrix cores could use; 256x256
// halves the bytes per flop, which is why it wins whenever it can occupy the chip.
// Split-K (several workgroups per 256x256 tile, see the kernel) is available on request
// (CHIMERA_GEMM_TILE=256x256x<splits> plus a workspace) but not chosen by default: on
// MI355X the device-wide fences its hand-over needs cost more than the idle CUs.
TileChoice choose_tile(const GemmArgs& g) {
    TileChoice f = forced_tile();
    const long t256 = (long)((g.m + 255) / 256) * ((g.n + 255) / 256);
    if (f.bm) {
        if (f.splits < 1 || f.bm != 256) f.splits = 1;
        f.splits = std::min(f.splits, std::min(MAX_SPLITS, std::max(1, (g.k + BK - 1) / BK)));
        if (f.splits > 1 && (!g.ws || g.ws_bytes < gemm_mfma_workspace_bytes(g.m, g.n, f.splits))) f.splits = 1;
        return f;
    }
    // (measured at 2048 x 4800 x 1600: 152 tiles of 256x256 on 256 CUs take 42 us, 608 of 128x128 48 us)
    if (t256 >= 144) return {256, 256, 1};
    if (wide_tiles(g)) return {256, 128, 1};
    if (small_tiles((long)((g.m + 63) / 64) * ((g.n + 63) / 64))) return small_tile(g);
    return {128, 128, 1};
}

template <int BM, int BN, int WGM, int WGN, int PF>
int launch_layout(const GemmArgs& g, int splits, hipStream_t s) {
    const int tm = (g.m + BM - 1) / BM, tn = (g.n + BN - 1) / BN;
    const dim3 grid(tm * tn * splits), block(WGM * WGN * 64);
    unsigned* arrivals = (unsigned*)g.ws;                               // [tiles], zero between launches
    float* slabs = g.ws ? (float*)((char*)g.ws + SPLITK_COUNTER_BYTES) : nullptr;
#define CHIMERA_GEMM_LAUNCH(AKC, BKC)                                                                              \
    hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WGM, WGN, PF, AKC, BKC>), grid, block, 0, s, (const bf16_t*)g.a,  \
                       (const bf16_t*)g.b, (const bf16_t*)g.bias, (const bf16_t*)g.r, result(g), (bf16_t*)g.c2, g.m, g.n, \
                       g.k, g.lda, g.ldb, g.epilogue, epilogue_flag(g), (g.r_f32 ? 1 : 0) | (g.c_f32 ? 2 : 0), tm, tn,    \
                       splits, slabs, arrivals)
    if (g.a_kc && !g.b_kc) CHIMERA_GEMM_LAUNCH(true, false);
    else if (g.a_kc && g.b_kc) CHIMERA_GEMM_LAUNCH(true, true);
    else CHIMERA_GEMM_LAUNCH(false, false);
#undef CHIMERA_GEMM_LAUNCH
    CHIMERA_LAUNCH_CHECK("bf16 gemm");
    return CHIMERA_OK;
}

template <int BM, int BN, int WGM, int WGN, int WGK, int NS, int SPS = 1>
int launch_async(const GemmArgs& g, hipStream_t s) {
    const int tm = (g.m + BM - 1) / BM, tn = (g.n + BN - 1) / BN;
    const dim3 grid(tm * tn), block(WGM * WGN * WGK * 64);
    const int gm = raster_group(tm, tn, (tm * tn + 7) / 8, BM, BN);
#define CHIMERA_GEMM_LAUNCH(AKC, BKC)                                                                                \
    hipLaunchKernelGGL((gemm_bf16_async_kernel<BM, BN, WGM, WGN, WGK, NS, SPS, AKC, BKC>), grid, block, 0, s,                   \
                       (const bf16_t*)g.a, (const bf16_t*)g.b, (const bf16_t*)g.bias, (const bf16_t*)g.r, result(g), \
                       (bf16_t*)g.c2, g.m, g.n, g.k, g.lda, g.ldb, g.epilogue, epilogue_flag(g),                            \
                       (g.r_f32 ? 1 : 0) | (g.c_f32 ? 2 : 0), tm, tn, gm, ahead_of(g))
    if (g.a_kc && !g.b_kc) CHIMERA_GEMM_LAUNCH(true, false);
    else if (g.a_kc && g.b_kc) CHIMERA_GEMM_LAUNCH(true, true);
    else if constexpr (BM == 64 && BN == 64) CHIMERA_GEMM_LAUNCH(false, false);
    else return fail(CHIMERA_EINVAL, "no %dx%d tile for weight gradients", BM, BN);
#undef CHIMERA_GEMM_LAUNCH
    CHIMERA_LAUNCH_CHECK("bf16 gemm (async)");
    return CHIMERA_OK;
}

// Columns [col0, col0 + 256 * cols256) of the product, or from col0 on.
template <int BM, int BN, int WGM, int WGN, int WGK>
int launch_ring(const GemmArgs& g, hipStream_t s, int col0 = 0, int cols256 = 0) {
    const int tm = (g.m + BM - 1) / BM, tn = cols256 ? cols256 * (256 / BN) : (g.n - col0 + BN - 1) / BN;
    const dim3 grid(tm * tn), block(WGM * WGN * WGK * 64);
    constexpr int PER_CU = RingLds<BM, BN, WGM, WGN, WGK>::PER_CU;
    const int band = raster_band(tm, tn, NUM_CUS * PER_CU, (size_t)g.n * g.k * sizeof(bf16_t));
    const int gm = raster_group(tm, band ? band : tn, std::min((tm * tn + 7) / 8, PER_XCD * PER_CU), BM, BN);
#define CHIMERA_GEMM_LAUNCH(AKC, BKC)                                                                                \
    hipLaunchKernelGGL((gemm_bf16_ring_kernel<BM, BN, WGM, WGN, WGK, AKC, BKC>), grid, block, 0, s,                     \
                       (const bf16_t*)g.a, (const bf16_t*)g.b, (const bf16_t*)g.bias, (const bf16_t*)g.r, result(g), \
                       (bf16_t*)g.c2, g.m, g.n, g.k, g.lda, g.ldb, g.epilogue, epilogue_flag(g),                            \
                       (g.r_f32 ? 1 : 0) | (g.c_f32 ? 2 : 0), tm, tn, gm, band, col0, ahead_of(g))
    if (g.a_kc && !g.b_kc) CHIMERA_GEMM_LAUNCH(true, false);
    else if (g.a_kc && g.b_kc) CHIMERA_GEMM_LAUNCH(true, true);
    else CHIMERA_GEMM_LAUNCH(false, false);
#undef CHIMERA_GEMM_LAUNCH
    CHIMERA_LAUNCH_CHECK("bf16 gemm (ring)");
    return CHIMERA_OK;
}

// Name of the kernel instantiation the last grouped launch on this thread went to (for reports).
thread_local char g_last_group_kernel[96] = "";
void note_group_kernel(const char* name) { std::snprintf(g_last_group_kernel, sizeof g_last_group_kernel, "%s", name); }

template <int BM, int BN, int WGM, int WGN, int WGK>
int launch_group_ring(const GemmGroup& grp, hipStream_t s) {
    char name[96];
    std::snprintf(name, sizeof name, "gemm_bf16_ring_group_kernel<%d,%d,%d,%d,%d>", BM, BN, WGM, WGN, WGK);
    note_group_kernel(name);
    hipLaunchKernelGGL((gemm_bf16_ring_group_kernel<BM, BN, WGM, WGN, WGK>), dim3(grp.first[grp.count]), dim3(WGM * WGN * WGK * 64), 0, s, grp);
    CHIMERA_LAUNCH_CHECK("bf16 gemm group");
    return CHIMERA_OK;
}

template <int BM, int BN, int WGM, int WGN, int WGK, int NS, int SPS = 1>
int launch_group(const GemmGroup& grp, hipStream_t s) {
    char name[96];
    std::snprintf(name, sizeof name, "gemm_bf16_async_group_kernel<%d,%d,%d,%d,%d,%d,%d,false,false>", BM, BN, WGM, WGN, WGK, NS, SPS);
    note_group_kernel(name);
    const dim3 grid(grp.first[grp.count]), block(WGM * WGN * WGK * 64);
    hipLaunchKernelGGL((gemm_bf16_async_group_kernel<BM, BN, WGM, WGN, WGK, NS, SPS, false, false>), grid, block, 0, s, grp);
    CHIMERA_LAUNCH_CHECK("bf16 gemm group");
    return CHIMERA_OK;
}

// A group on tiles of 256x256, its remainders of up to 128 rows or columns on halves of them, begun first, and what full rounds leave
// over on quarters or halves, begun last.  Against 256x256 tiles throughout, with the last row bands of one product in a launch of
// 128x128 tiles of its own: blocks of 1280, 1344, 1408, 1600 and 1792 at 2048 tokens 106 -> 103, 132 -> 109, 137 -> 116, 169 -> 152 and 207 -> 188 us;
// of 1024, 1536 and 2048, which have neither remainders nor a rest, within 1 %.  gpt2-1p3b-n32 96.0 -> 93.6 ms.
// (1) A remainder costs a half tile, not a whole one: a block of 1600 needs 450 + 82 halves instead of 532.
// (2) All workgroups of a launch that starts with one size reach their epilogues together, and the chip then waits for HBM: 256 tiles of += x 64
// take 25.5 us, 16 take 10.7.  Halves first put CUs out of step, and give CUs to the other lane of a replay at other times than the
// rest: halves first -> last gpt2-1p3b-n32 94.2 -> 96.1 ms, six blocks of 1600 at 632 tokens, forward and backward, 1665 -> 1706 us.  Halving
// whole tiles for it does not pay: a half takes 0.6 of a tile's time (2048 wide, 128 of 768 halved 222 -> 235 us).
// (3) Up to 64 tiles beyond full rounds take a round of quarters, 0.38 of one of 256x256; more of them a round of halves where these and
// the remainders' fit into one.
int launch_group_mixed(int count, const GemmArgs* g, float* const* bsum, int overwrite, bool smaller, hipStream_t stream) {
    int fm[GROUP_MAX], fn[GROUP_MAX], cut_m[GROUP_MAX] = {}, cut_n[GROUP_MAX] = {};      // tile rows and columns of 256x256, how many of each are cut smaller
    long full = 0, half = 0;
    for (int i = 0; i < count; ++i) {
        const int rm = g[i].m % 256, rn = g[i].n % 256;
        fm[i] = g[i].m / 256 + (rm > (smaller ? 128 : 0));
        fn[i] = g[i].n / 256 + (rn > (smaller ? 128 : 0));
        full += (long)fm[i] * fn[i];
        if (fm[i] * 256 < g[i].m) half += (g[i].n + 255) / 256;
        if (fn[i] * 256 < g[i].n) half += fm[i];
    }
    const long over = smaller && full + half > NUM_CUS ? (full + half) % NUM_CUS : 0;
    const bool quarters = 4 * over <= NUM_CUS;
    const long left = full % NUM_CUS;                        // of the whole tiles alone
    const bool fill = smaller && !quarters && full > NUM_CUS && half + 2 * left <= NUM_CUS;
    const long todo = fill ? left : over <= full && (quarters || (over > half && 2 * over <= NUM_CUS)) ? over : 0;
    const long most = quarters ? NUM_CUS / 4 : (NUM_CUS - (fill ? half : 0)) / 2;
    // Whole bands of rows or columns of one product, or bands of two kinds where that does not do, that come to `todo` tiles or the fewest
    // more, and to a round of the smaller tiles at most; less than `todo` would leave the last round as it is.  With one kind only, which
    // may find nothing, -> so: a block of 2696 at 2048 tokens (117 tiles) 435 -> 420 us, 1496 x 13464 x 2048 (62: a row of 53, two columns
    // of 5) 111 -> 91; but with two kinds wherever they come nearer a block of 1152 (19 tiles in place of 20) 78 -> 88.
    auto tiles_of = [&](int i, bool rows) { return (long)(rows ? fn[i] - cut_n[i] : fm[i] - cut_m[i]); };
    auto bands_of = [&](int i, bool rows) { return (long)(rows ? fm[i] - cut_m[i] : fn[i] - cut_n[i]); };
    auto take = [&](int i, bool rows, long bands) { (rows ? cut_m : cut_n)[i] += (int)bands; };
    struct Bands { int i; bool rows; long count; } first{}, last{}, none{};
    long best = most + 1;
    auto finish = [&](const Bands& before, long got) {
        for (int i = 0; i < count; ++i)
            for (bool rows : {true, false}) {
                const long per = tiles_of(i, rows), bands = per > 0 ? (todo - got + per - 1) / per : 0;
                if (bands > 0 && bands <= bands_of(i, rows) && got + bands * per < best) { best = got + bands * per; first = before; last = {i, rows, bands}; }
            }
    };
    if (todo > 0) {
        finish(none, 0);
        if (best > most)
            for (int i = 0; i < count; ++i)
                for (bool rows : {true, false}) {
                    const long per = tiles_of(i, rows), bands = per > 0 ? std::min(todo / per, bands_of(i, rows)) : 0;
                    if (bands <= 0) continue;
                    take(i, rows, bands);
                    finish({i, rows, bands}, bands * per);
                    take(i, rows, -bands);
                }
        take(first.i, first.rows, first.count);
        take(last.i, last.rows, last.count);
    }
    MixedGroup grp{};
    grp.k = g[0].k; grp.flags = (overwrite ? ACCUM_OVERWRITE : 0) | (g[0].c_once ? ACCUM_ONCE : 0);
    std::fill(std::begin(grp.first), std::end(grp.first), INT_MAX);
    int tiles = 0;
    auto put = [&](int i, int form, int row0, int rows, int col0, int cols) {
        if (rows <= 0 || cols <= 0) return;
        const int bm = form == TILE_128x256 || form == TILE_128 ? 128 : 256, bn = form == TILE_256x128 || form == TILE_128 ? 128 : 256;
        MixedEntry& e = grp.e[grp.count++];
        e.a = (const bf16_t*)g[i].a + row0;                      // A is [k, m]
        e.b = (const bf16_t*)g[i].b;
        e.c = (float*)g[i].c + (size_t)row0 * g[i].n;
        e.bsum = bsum && row0 == 0 ? bsum[i] : nullptr;
        e.m = rows; e.n = g[i].n; e.lda = g[i].lda; e.ldb = g[i].ldb; e.col0 = col0;
        e.tiles_m = (rows + bm - 1) / bm; e.tiles_n = (cols + bn - 1) / bn;
        e.form = form; grp.first[&e - grp.e] = tiles;
        tiles += e.tiles_m * e.tiles_n;
    };
    int local = 0;
    auto close = [&](int h) {                                    // the entries put since the last call are phase h
        MixedPhase& p = grp.phase[h];
        p.first = h ? grp.phase[h - 1].first + grp.phase[h - 1].tiles : 0;
        p.tiles = tiles - p.first; p.local = local; p.skew = p.first % XCDS;
        local += (p.tiles + XCDS - 1) / XCDS;
        for (int i = 0; i < grp.count; ++i) {
            MixedEntry& e = grp.e[i];
            if (grp.first[i] < p.first) continue;
            const int bm = e.form == TILE_128x256 || e.form == TILE_128 ? 128 : 256, bn = e.form == TILE_256x128 || e.form == TILE_128 ? 128 : 256;
            e.band = raster_band(e.tiles_m, e.tiles_n, NUM_CUS, (size_t)e.n * grp.k * sizeof(bf16_t));
            e.group_m = raster_group(e.tiles_m, e.band ? e.band : e.tiles_n, std::min((p.tiles + XCDS - 1) / XCDS, PER_XCD), bm, bn);
        }
    };
    // rows [0, whole_m) of columns [0, whole_n) on 256x256 tiles, up to `rows` and `cols` cut smaller, then the remainders
    auto rows = [&](int i) { return std::min(fm[i] * 256, g[i].m); };
    auto cols = [&](int i) { return std::min(fn[i] * 256, g[i].n); };
    auto whole_m = [&](int i) { return std::min((fm[i] - cut_m[i]) * 256, g[i].m); };
    auto whole_n = [&](int i) { return std::min((fn[i] - cut_n[i]) * 256, g[i].n); };
    for (int i = 0; i < count; ++i) put(i, TILE_128x256, rows(i), g[i].m - rows(i), 0, g[i].n);
    for (int i = 0; i < count; ++i) put(i, TILE_256x128, 0, rows(i), cols(i), g[i].n - cols(i));
    close(0);
    for (int i = 0; i < count; ++i) put(i, TILE_256, 0, whole_m(i), 0, whole_n(i));
    close(1);
    for (int i = 0; i < count; ++i) {
        put(i, quarters ? TILE_128 : TILE_128x256, whole_m(i), rows(i) - whole_m(i), 0, whole_n(i));
        put(i, quarters ? TILE_128 : TILE_256x128, 0, rows(i), whole_n(i), cols(i) - whole_n(i));
    }
    close(2);
    hipLaunchKernelGGL(gemm_bf16_mixed_group_kernel, dim3(local * XCDS), dim3(512), 0, stream, grp);
    CHIMERA_LAUNCH_CHECK("bf16 gemm group");
    return CHIMERA_OK;
}

}  // namespace

bool gemm_mfma_supports(const GemmArgs& g) {
    if (!g.a_kc && g.b_kc) return false;                       // layout no linear layer needs
    if ((g.n % 8) || (g.lda % 8) || (g.ldb % 8)) return false;
    if ((g.a_kc || g.b_kc) && (g.k % 8)) return false;         // index-contiguous operands are masked row by row: any k
    if (!g.a_kc && (g.m % 8)) return false;
    if (((uintptr_t)g.a | (uintptr_t)g.b) & 15) return false;  // 16-byte vector loads
    // operand elements are addressed with 32-bit offsets
    const unsigned long long ea = (unsigned long long)(g.a_kc ? g.m : g.k) * g.lda, eb = (unsigned long long)(g.b_kc ? g.n : g.k) * g.ldb;
    if (ea >= (1ull << 32) || eb >= (1ull << 32)) return false;
    return g.m >= 1 && g.n >= 1 && g.k >= 1;
}

// Workspace of a split-K launch: arrival counters (zero before the first launch, left zero
// by every launch) followed by one float slab per (split, 256x256 tile).
size_t gemm_mfma_workspace_bytes(int m, int n, int splits) {
    const size_t tiles = (size_t)((m + 255) / 256) * ((n + 255) / 256);
    return SPLITK_COUNTER_BYTES + (size_t)splits * tiles * 256 * 256 * sizeof(float);
}
// Workspace that allows any split count up to MAX_SPLITS for an m x n output.
size_t gemm_mfma_workspace_need(int m, int n, int k) {
    if (m < 1 || n < 1 || k < 1) return 0;
    return gemm_mfma_workspace_bytes(m, n, MAX_SPLITS);
}

int gemm_mfma_bf16(const GemmArgs& g, void* stream) {
    if (!gemm_mfma_supports(g)) return fail(CHIMERA_EINVAL, "bf16 matrix-core gemm: unsupported shape or layout");
    if (g.epilogue < EPI_NONE || g.epilogue > EPI_ACCUM_F32) return fail(CHIMERA_EINVAL, "unknown epilogue %d", g.epilogue);
    hipStream_t s = (hipStream_t)stream;
    const bool far = far_operand(g);
    TileChoice t = choose_tile(g);
    if (far && (t.bm < 128 || t.bm != t.bn)) t = {128, 128, 1};
    if (t.splits > 1 && (size_t)((g.m + 255) / 256) * ((g.n + 255) / 256) * sizeof(unsigned) > SPLITK_COUNTER_BYTES)
        return fail(CHIMERA_EINVAL, "too many tiles for split-K");
    // 128x128 tiles: with one workgroup per CU, a workgroup of 4 wavefronts leaves one wavefront
    // per SIMD, and nothing covers its LDS latency and the barrier of every k step; then 8
    // wavefronts share the tile, two per 64x64 block (their partial sums meet in LDS at the end),
    // over a ring of 128 KiB - one such workgroup per CU, so more than NUM_CUS tiles would take it
    // two rounds.  Beyond that the 4-wavefront form with its two buffers (64 KiB of LDS, two
    // workgroups per CU) is faster.
    const int mode = tuning().async_mode;
    const bool can_async = t.splits == 1 && mode != ASYNC_OFF && !far;
    if (can_async) {
        if (t.bm == 256 && t.bn == 256) {
            if (!g.a_kc && g.epilogue == EPI_ACCUM_F32) return launch_group_mixed(1, &g, nullptr, 0, forced_tile().bm == 0, s);
            const int tm = (g.m + 255) / 256, tn = (g.n + 255) / 256;
            double by_rows = 0, by_columns = 0;
            const int b = forced_tile().bm ? 0 : bands_to_peel(tm, tn, g.n, &by_rows);
            const int bc = forced_tile().bm ? 0 : bands_to_peel(tn, tm, g.m, &by_columns);
            if (bc > 0 && by_columns < by_rows && g.n - (tn - bc) * 256 >= 8) {
                // columns in the same way: wide outputs of few tile rows (1024 x 50304 x 4096, 788 tiles:
                // three full rounds and 20 tiles: 386 -> 344 us)
                const int col0 = (tn - bc) * 256;
                GemmArgs head = g;
                head.ahead = nullptr; head.ahead_bytes = 0;
                if (int rc = launch_ring<256, 256, 2, 4, 1>(head, s, 0, tn - bc)) return rc;
                if ((long)((g.m + 127) / 128) * ((g.n - col0 + 127) / 128) <= NUM_CUS) return launch_ring<128, 128, 2, 2, 2>(g, s, col0);
                return launch_ring<128, 128, 2, 2, 1>(g, s, col0);
            }
            if (b > 0 && g.m - (tm - b) * 256 >= 8) {
                // rows [0, m0) with 256x256 tiles, rows [m0, m) with 128x128 tiles
                const size_t m0 = (size_t)(tm - b) * 256;
                const size_t csz = (g.epilogue == EPI_ACCUM_F32 || g.c_f32) ? 4 : 2;
                GemmArgs head = g, tail = g;
                head.ahead = nullptr; head.ahead_bytes = 0;
                head.m = (int)m0;
                tail.m = g.m - (int)m0;
                tail.a = (const char*)g.a + (g.a_kc ? m0 * g.lda : m0) * 2;
                tail.c = (char*)g.c + m0 * g.n * csz;
                if (g.c2) tail.c2 = (char*)g.c2 + m0 * g.n * 2;
                if (g.r) tail.r = (const char*)g.r + m0 * g.n * (g.r_f32 ? 4 : 2);
                if (int rc = launch_ring<256, 256, 2, 4, 1>(head, s)) return rc;
                const long t128 = (long)((tail.m + 127) / 128) * ((tail.n + 127) / 128);
                if (t128 <= NUM_CUS) return launch_ring<128, 128, 2, 2, 2>(tail, s);
                return launch_ring<128, 128, 2, 2, 1>(tail, s);
            }
            return launch_ring<256, 256, 2, 4, 1>(g, s);
        }
        if (t.bm == 256) return launch_ring<256, 128, 2, 2, 2>(g, s);
        if (t.bm == 128 && t.bn == 64) return launch_async<128, 64, 2, 2, 2, 6, 2>(g, s);
        if (t.bm == 32) return t.bn == 32 ? launch_async<32, 32, 1, 1, 4, 8, 2>(g, s) : launch_async<32, 64, 1, 2, 2, 8, 2>(g, s);
        if (t.bm == 64) {
            // one tile per CU at most: all of LDS for one workgroup, an eight-stage ring walked two stages per
            // barrier by two wavefronts per SIMD (256 x 256 x 1024: 6.7 -> 6.1 us; 632 x 1600 x 6400: 28.4 -> 25.4)
            if ((long)((g.m + 63) / 64) * ((g.n + 63) / 64) <= NUM_CUS) return launch_async<64, 64, 2, 2, 2, 8, 2>(g, s);
            return launch_async<64, 64, 1, 2, 2, 4>(g, s);
        }
        if (t.bm == 128 && t.bn == 128) {
            const long t128 = (long)((g.m + 127) / 128) * ((g.n + 127) / 128);
            const bool ksplit = mode != ASYNC_AUTO ? mode == ASYNC_KSLICED : t128 <= NUM_CUS;
            if (ksplit) return launch_ring<128, 128, 2, 2, 2>(g, s);
            return launch_ring<128, 128, 2, 2, 1>(g, s);
        }
    }
    if (t.bm == 256 && t.bn == 256) return launch_layout<256, 256, 2, 4, 1>(g, t.splits, s);
    if (t.bm == 128 && t.bn == 128) return launch_layout<128, 128, 2, 2, 1>(g, 1, s);
    return fail(CHIMERA_EINVAL, "no %dx%d gemm tile", t.bm, t.bn);
}

// How a product of k-contiguous operands is cut along k (splits = 1: not at all): fewer tiles than CUs leave
// CUs idle, and 256x256 tiles cost a third less energy and time per flop than the 128x128 tiles that an uncut
// product of 64 to 143 of them takes.  Model of the time in us, constants measured: a step of 64 k of a round of
// tiles (A B^T, k 1024 to 8192: 256x256 1.55 to 1.63 from random operands that miss the caches, 128x128 0.50 to 0.56, 64x64
// 0.18 to 0.30), against the float slabs written and read (at 4.5 TB/s) and the launch that adds them.
// 4096 x 1024 x 50304 462 -> 355 + 12 us; a head's whole pass over 1000 x 512 x 20000 164 -> 131, 128 x 128 x 65536
// 252 -> 87, 1111 x 776 x 50304 507 -> 443, 632 x 1600 x 50304 589 -> 515 us.
struct SplitPlan { int tile, splits, k_per; };
static SplitPlan split_plan(int m, int n, int k) {
    const long steps = (k + RK - 1) / RK, t256 = (long)((m + 255) / 256) * ((n + 255) / 256), t128 = (long)((m + 127) / 128) * ((n + 127) / 128);
    const long t64 = (long)((m + 63) / 64) * ((n + 63) / 64);
    SplitPlan best{0, 1, k};
    if (forced_tile().bm || tuning().async_mode != ASYNC_AUTO || t256 >= 144) return best;
    constexpr double STEP256 = 1.4, STEP128 = 0.5, STEP64 = 0.25, SLAB = 8 / 4.5e6, LAUNCH = 10;
    auto rounds = [](long tiles) { return (double)((tiles + NUM_CUS - 1) / NUM_CUS); };
    double cost = steps * (t64 <= 2 * NUM_CUS ? rounds(t64) * STEP64 : rounds(t128) * STEP128);
    cost *= 0.9;                                         // a split must pay clearly
    for (int s = 2; s <= 64 && steps / s >= 8; ++s) {
        const long per = (steps + s - 1) / s;
        if ((steps + per - 1) / per != s) continue;
        const double slabs = SLAB * s * m * n + LAUNCH;
        const double c256 = rounds(t256 * s) * per * STEP256 + slabs, c128 = rounds(t128 * s) * per * STEP128 + slabs;
        if (c256 < cost) { cost = c256; best = {256, s, (int)per * RK}; }
        if (c128 < cost) { cost = c128; best = {128, s, (int)per * RK}; }
    }
    return best;
}
size_t gemm_mfma_split_bytes(int m, int n, int k) {
    const SplitPlan p = split_plan(m, n, k);
    return p.splits > 1 ? (size_t)p.splits * m * n * sizeof(float) : 0;
}
int gemm_mfma_split(const GemmArgs& g, float* slabs, void* stream) {
    if (!gemm_mfma_supports(g) || !g.a_kc || !g.b_kc || g.epilogue != EPI_NONE || ((uintptr_t)g.c | (uintptr_t)slabs) & 15)
        return fail(CHIMERA_EINVAL, "split product: k-contiguous operands and a plain bf16 result");
    const SplitPlan p = split_plan(g.m, g.n, g.k);
    if (p.splits < 2 || far_operand(g)) return gemm_mfma_bf16(g, stream);
    hipStream_t s = (hipStream_t)stream;
    const int tm = (g.m + p.tile - 1) / p.tile, tn = (g.n + p.tile - 1) / p.tile;
    const int gm = raster_group(tm, tn, std::min(tm * tn, (tm * tn * p.splits + 7) / 8), p.tile, p.tile);
    const dim3 grid(tm * tn * p.splits), block(512);
#define CHIMERA_SPLIT_LAUNCH(...)                                                                                       \
    hipLaunchKernelGGL((gemm_bf16_ring_split_kernel<__VA_ARGS__>), grid, block, 0, s, (const bf16_t*)g.a, (const bf16_t*)g.b, \
                       slabs, g.m, g.n, g.k, g.lda, g.ldb, tm, tn, gm, p.splits, p.k_per)
    if (p.tile == 256) CHIMERA_SPLIT_LAUNCH(256, 256, 2, 4, 1);
    else CHIMERA_SPLIT_LAUNCH(128, 128, 2, 2, 2);
#undef CHIMERA_SPLIT_LAUNCH
    CHIMERA_LAUNCH_CHECK("bf16 gemm (split)");
    const size_t elems = (size_t)g.m * g.n;
    hipLaunchKernelGGL(split_sum_kernel, dim3((unsigned)((elems / 8 + 255) / 256)), dim3(256), 0, s, slabs, elems, p.splits, (bf16_t*)g.c);
    CHIMERA_LAUNCH_CHECK("split sum");
    return CHIMERA_OK;
}

bool gemm_mfma_group_supports(int count, const GemmArgs* g) {
    if (count < 1 || count > GROUP_MAX || !g) return false;
    for (int i = 0; i < count; ++i) {
        if (g[i].a_kc || g[i].b_kc || g[i].epilogue != EPI_ACCUM_F32 || !gemm_mfma_supports(g[i])) return false;
        if (g[i].k != g[0].k) return false;
        if ((uintptr_t)g[i].c & 15) return false;
    }
    return true;
}

namespace {
int launch_group_tiled(int count, const GemmArgs* g, float* const* bsum, int overwrite, int tile, hipStream_t stream) {
    GemmGroup grp{};
    grp.count = count; grp.k = g[0].k; grp.overwrite = overwrite ? 1 : 0;
    int tiles = 0;
    for (int i = 0; i < count; ++i) {
        grp.a[i] = (const bf16_t*)g[i].a; grp.b[i] = (const bf16_t*)g[i].b; grp.c[i] = (float*)g[i].c;
        grp.bsum[i] = bsum ? bsum[i] : nullptr;
        grp.m[i] = g[i].m; grp.n[i] = g[i].n; grp.lda[i] = g[i].lda; grp.ldb[i] = g[i].ldb;
        grp.tiles_m[i] = (g[i].m + tile - 1) / tile; grp.tiles_n[i] = (g[i].n + tile - 1) / tile;
        grp.first[i] = tiles;
        tiles += grp.tiles_m[i] * grp.tiles_n[i];
    }
    for (int i = 0; i < count; ++i) grp.group_m[i] = raster_group(grp.tiles_m[i], grp.tiles_n[i], (tiles + 7) / 8, tile, tile);
    for (int i = count; i <= GROUP_MAX; ++i) grp.first[i] = tiles;
    if (tile == 64) return tiles <= NUM_CUS ? launch_group<64, 64, 2, 2, 2, 8, 2>(grp, stream) : launch_group<64, 64, 1, 2, 2, 4>(grp, stream);
    // two workgroups per CU or the k-sliced 8-wavefront form
    const int mode = tuning().async_mode;
    const bool ksplit = mode != ASYNC_AUTO ? mode == ASYNC_KSLICED : tiles <= NUM_CUS;
    if (ksplit) return launch_group_ring<128, 128, 2, 2, 2>(grp, stream);
    return launch_group_ring<128, 128, 2, 2, 1>(grp, stream);
}
}  // namespace

int gemm_mfma_bf16_group(int count, const GemmArgs* g, float* const* bsum, int overwrite, void* stream) {
    if (!gemm_mfma_group_supports(count, g))
        return fail(CHIMERA_EINVAL, "bf16 gemm group: 1..%d float-accumulating products with index-contiguous operands, "
                    "one contraction length", GROUP_MAX);
    // tile choice as for single products: 256x256 once such tiles occupy most of the chip, else
    // 128x128.  (192 tiles of 256x256 on 256 CUs beat 768 tiles of 128x128: they pull half the
    // bytes from L2 into LDS, which is what limits these kernels, and the CUs they leave free
    // serve the launches of the other stream.)
    long t256 = 0, t64 = 0;
    for (int i = 0; i < count; ++i) {
        t256 += (long)((g[i].m + 255) / 256) * ((g[i].n + 255) / 256);
        t64 += (long)((g[i].m + 63) / 64) * ((g[i].n + 63) / 64);
    }
    const int forced = forced_tile().bm;
    const int tile = forced == 256 || forced == 128 ? forced : t256 >= 160 ? 256 : small_tiles(t64) ? 64 : 128;
    if (tile == 256) {
        note_group_kernel("gemm_bf16_mixed_group_kernel");
        return launch_group_mixed(count, g, bsum, overwrite, forced == 0, (hipStream_t)stream);
    }
    return launch_group_tiled(count, g, bsum, overwrite, tile, (hipStream_t)stream);
}

const char* gemm_mfma_last_group_kernel() { return g_last_group_kernel; }

int gemm_mfma_set_tuning(int bm, int bn, int splits, int async_mode) {
    if (!((bm == 0 && bn == 0) || (bm == 128 && bn == 128) || (bm == 256 && bn == 256)))
        return fail(CHIMERA_EINVAL, "forced tile %dx%d: 0x0 (automatic), 128x128 or 256x256", bm, bn);
    if (splits < 0 || splits > MAX_SPLITS) return fail(CHIMERA_EINVAL, "splits=%d outside [0,%d]", splits, MAX_SPLITS);
    if (async_mode < ASYNC_AUTO || async_mode > ASYNC_PLAIN) return fail(CHIMERA_EINVAL, "async_mode=%d outside [0,3]", async_mode);
    Tuning& t = tuning();
    t.forced = TileChoice{bm, bn, splits};
    t.async_mode = async_mode;
    ++t.version;
    return CHIMERA_OK;
}

unsigned long long gemm_mfma_tuning_version() { return tuning().version; }

}  // namespace chimera
