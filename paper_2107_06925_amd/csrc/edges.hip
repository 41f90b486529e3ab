// The two ends of the pipeline (section 4.1 of the paper notes that the first stage of a
// language model carries an extra embedding layer; the last stage turns hidden states into a
// loss).  GPT-2 reading:
//   embedding  x[t] = wte[token[t]] + wpe[t mod S]
//   head       h = LayerNorm(y),  z = h W (W stored [H, V]),
//              loss = scale * sum_t (logsumexp(z[t]) - z[t, target[t]])
// with the matching backward.  The matrix products and the LayerNorm are the stage's own
// kernels; this file adds the gather / scatter of the embedding and the fused
// softmax-cross-entropy over a vocabulary row.  No atomics: every sum has a fixed order.
#include "device.h"

#include <algorithm>

namespace chimera {
namespace {

constexpr int EDGE_THREADS = 256;

// ---- embedding forward: one wavefront per token
template <typename T>
__global__ __launch_bounds__(EDGE_THREADS) void embed_fwd_kernel(const int* __restrict__ tokens, const T* __restrict__ wte,
                                                                 const T* __restrict__ wpe, T* __restrict__ x, int M, int S,
                                                                 int H, int vocab) {
    constexpr int V = Elem<T>::VEC;
    const int t = blockIdx.x * (EDGE_THREADS / WAVE) + threadIdx.x / WAVE, lane = threadIdx.x % WAVE;
    if (t >= M) return;
    const int tok = min(max(tokens[t], 0), vocab - 1);         // ids outside the table are clamped, never followed
    const T* a = wte + (size_t)tok * H;
    const T* p = wpe + (size_t)(t % S) * H;
    for (int c = lane; c < H / V; c += WAVE) {
        float u[V], w[V];
        load_vec<T>(a + c * V, u);
        load_vec<T>(p + c * V, w);
#pragma unroll
        for (int e = 0; e < V; ++e) u[e] += w[e];
        store_vec<T>(x + (size_t)t * H + c * V, u);
    }
}

// ---- embedding backward: one launch, three kinds of workgroups.
//
// Position table, dwpe[p] += sum over the sequences of dx[b*S + p], b ascending: one 16-byte piece
// of a row per thread, eight sequences' pieces requested at a time.
//
// Token table, dwte[v] += sum of dx[t] over the positions t with token v.  Workgroup w owns the
// tokens v with v mod owners = w: every table row has one owner, so the sums need no atomics, and their
// order is fixed by the positions alone.  Frequent tokens (more than embed_hot_from positions hold v mod EMB_BUCKETS)
// have owners of their own: one CU reads some 64 bytes a nanosecond, and a frequent word's rows are many.  Workgroup (w, s) of those
// owns columns [s, s + 1) * EMB_LANES * V of the frequent tokens with v mod hot_classes = w.  A workgroup
//   1. lists its positions in ascending order (one ballot per 64 positions),
//   2. finds the first entry of every distinct token in the list (a "head"),
//   3. gives each head and 64 pieces of its row to one wavefront, which walks the list 64 entries at a time (ballot of
//      "same token") and adds the rows in ascending order, several in flight;
//   4. or, for frequent tokens, shares each among 32 groups of lanes, the k-th of which takes the k-th, (k + 32)-th, ...
//      position; the partial rows are added in a fixed tree.
// A list holds EMB_LIST entries; a workgroup that owns more goes through the positions in windows that about fill it.
// What bounds it is latency (list, row, table row: a few dependent round trips), so there are
// enough workgroups that a wavefront seldom has more than one or two tokens.  (One workgroup per
// position, each scanning all tokens through LDS, took 301 us at 4096 positions x 1024 columns.)  With frequent tokens shared by
// the wavefronts of their owner, whole rows each, and windows of 4096 positions, ids spread over the logarithm of the
// vocabulary: 4096 x 1024 of 50304 35.6 -> 16.9 us (float 67 -> 18.7), 16384 x 2048 of 65536 244 -> 90, 16384 x 256 of 30000
// 73 -> 57, 1000 x 776 of 5000 11.7 -> 9.3; every second position the same token, 4096 x 1024, 179 -> 35.
// owners: 1024 x 1024 and 512 x 512 of them at 2048 tokens of 1600 columns 14.5 -> 11.2 us, at 4096 x 1024 16.9 -> 18.4,
// at 8192 x 512 25.8 -> 34.  Classes of frequent tokens: 16 -> 32 at 16384 x 2048 112 -> 89, at 4096 x 1024 (float) 18.7 -> 20.6.
// Frequent beyond 16 positions and windows of EMB_LIST positions -> beyond one in 256, 16 to 32 at least, and full lists: uniform ids
// 4096 x 1024 of 256 21.7 -> 11.5, 16384 x 1024 of 1000 77 -> 45, 262144 x 256 of 30000 8430 -> 577; logarithmic ids 32768 x 1024 of 50304
// 344 -> 112, 131072 x 1024 2270 -> 530.  With one in 128 524288 x 512 takes 2610 us for 2100, with one in 512 131072 x 1024 593 for 530; with 32 for
// 16 384 x 1024 of 2000 10.0 for 8.9, with 16 for 32 4096 x 256 of 2000 16.6 for 13.7.
constexpr int EMB_THREADS = 512, EMB_WAVES = EMB_THREADS / WAVE;
constexpr int EMB_LIST = 2048;
constexpr int EMB_HOT_MIN = 16;
inline int embed_hot_from(int tokens) { return std::max(std::clamp(tokens / 64, EMB_HOT_MIN, 32), tokens / 256); }
constexpr int EMB_OWNERS_MIN = 64, EMB_OWNERS_MAX = 1024;       // workgroups that share the token table (powers of two)
constexpr int EMB_HOT_CLASSES_MIN = 8, EMB_HOT_CLASSES_MAX = 32, EMB_BUCKETS = 16384;       // powers of two
constexpr int EMB_LANES = 16, EMB_GROUPS = EMB_THREADS / EMB_LANES, EMB_FLY = 4;       // lanes of a group (256 bytes of a row); rows in flight
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));     // gradient tables need not be 16-byte aligned
struct EmbedLds {
    int tok[EMB_LIST];                    // owned tokens, in position order
    int pos[EMB_LIST];                    // their positions
    unsigned short head[EMB_LIST];        // list index of the first entry of every distinct token
    unsigned short same[EMB_LIST];        // list indices of one frequent token
    int seen[EMB_BUCKETS / EMB_HOT_CLASSES_MIN];       // positions of the class's tokens, by bucket
    float part[EMB_WAVES][EMB_LANES * 8]; // partial rows of a frequent token
    int counts[EMB_WAVES];
    int heads;
};

// Three workgroups per CU: at 81 registers (two) 8192 x 768 bf16 takes 34.8 us instead of 28.2.
template <typename T>
__global__ __launch_bounds__(EMB_THREADS, 6) void embed_bwd_kernel(const int* __restrict__ tokens, const T* __restrict__ dx,
                                                                float* __restrict__ dwte, float* __restrict__ dwpe, int M, int S,
                                                                int H, int vocab, int owners, int hot_classes, int slices, int hot_from) {
    constexpr int V = Elem<T>::VEC;
    __shared__ __attribute__((aligned(16))) EmbedLds sm;
    const int tid = threadIdx.x, lane = tid % WAVE, wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int nchunk = H / V;
    const int hot_wgs = hot_classes * slices;
    const bool hot = (int)blockIdx.x < hot_wgs;
    if ((int)blockIdx.x >= hot_wgs + owners) {                  // position table
        const size_t i = (size_t)(blockIdx.x - hot_wgs - owners) * EMB_THREADS + tid;
        if (i >= (size_t)S * nchunk) return;
        const T* src = dx + i * V;                              // position p = i / nchunk of sequence 0
        const size_t stride = (size_t)S * H;
        const int B = M / S;
        float acc[V];
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] = 0.f;
        for (int b0 = 0; b0 < B; b0 += 8) {
            uint4 q[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) q[u] = *reinterpret_cast<const uint4*>(src + (size_t)min(b0 + u, B - 1) * stride);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (b0 + u < B) {
                    float v[V];
                    load_vec<T>(reinterpret_cast<const T*>(&q[u]), v);
#pragma unroll
                    for (int e = 0; e < V; ++e) acc[e] += v[e];
                }
        }
        float* out = dwpe + i * V;
#pragma unroll
        for (int e = 0; e < V; e += 4) {
            f32x4_u t = *reinterpret_cast<const f32x4_u*>(out + e);
#pragma unroll
            for (int k = 0; k < 4; ++k) t[k] += acc[e + k];
            *reinterpret_cast<f32x4_u*>(out + e) = t;
        }
        return;
    }
    const int mine = hot ? (int)blockIdx.x / slices : (int)blockIdx.x - hot_wgs, classes = hot ? hot_classes : owners;      // (powers of two)
    // of a frequent token's row: this group's lanes, and the lane's 16-byte piece
    const int group = tid / EMB_LANES, slice = hot ? (int)blockIdx.x % slices : 0, piece = slice * EMB_LANES + lane % EMB_LANES;
    auto add_row = [](float (&a)[V], const uint4& q) {
        float x[V];
        load_vec<T>(reinterpret_cast<const T*>(&q), x);
#pragma unroll
        for (int e = 0; e < V; ++e) a[e] += x[e];
    };
    // 512 positions at a time, 64 per load; ids outside the table are clamped, never followed
    constexpr int LOADS = EMB_THREADS / WAVE;
    int tok[LOADS];
    auto load_tokens = [&](int from, int end) {
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int t = from + i * WAVE + lane;
            tok[i] = t < end ? min(max(tokens[t], 0), vocab - 1) : -1;
        }
    };
    auto bucket = [&](int v) { return (v & (EMB_BUCKETS - 1)) / classes; };
    auto in_class = [&](int v) { return v >= 0 && (v & (classes - 1)) == mine; };
    // Wavefront k looks at the k-th eighth of the positions in question.  Where that is one look (up to 4096 positions), the tokens that the
    // count by bucket has read are those that the list of frequent tokens is made of, and are asked for ahead of the counts' barrier: a
    // trip to memory less, which is an eighth of a small call.  With what is beyond the positions skipped 64
    // at a time: 463 x 192 float 8.1 -> 7.0 us, 648 x 184 8.75 -> 7.75, 1662 x 1136 bf16 13.7 -> 12.5; 11450 x 800 float 47.5 -> 48.9.
    auto eighth = [](int size) { return ((size + EMB_WAVES - 1) / EMB_WAVES + WAVE - 1) / WAVE * WAVE; };
    const int share = eighth(M);
    const bool kept = share <= EMB_THREADS;
    // positions of the class by bucket; whether one is frequent
    auto count_buckets = [&] {
        const int end = kept ? min((wave + 1) * share, M) : M;
        if (kept) load_tokens(wave * share, end);
        for (int i = tid; i < EMB_BUCKETS / classes; i += EMB_THREADS) sm.seen[i] = 0;
        __syncthreads();
        bool frequent = false;
        for (int from = wave * (kept ? share : EMB_THREADS); from < end; from += EMB_WAVES * EMB_THREADS) {
            if (!kept) load_tokens(from, end);
#pragma unroll
            for (int i = 0; i < LOADS; ++i)
                if (from + i * WAVE < end && in_class(tok[i])) frequent |= atomicAdd(&sm.seen[bucket(tok[i])], 1) >= hot_from;
        }
        return __syncthreads_or(frequent) != 0;
    };
    if (hot && !count_buckets()) return;
    bool by_bucket = hot;                                       // the list leaves out what the other kind owns
    auto owned = [&](int v) { return in_class(v) && (!by_bucket || (sm.seen[bucket(v)] > hot_from) == hot); };
    // Counts what is owned of positions [w0, w0 + size): in the wavefronts before this one, and in all (returned).
    int at = 0;
    auto count_owned = [&](int w0, int size, bool load = true) {
        const int each = eighth(size), end = min(w0 + min((wave + 1) * each, size), M);
        int n_wave = 0;
        for (int from = w0 + wave * each; from < end; from += EMB_THREADS) {
            if (load) load_tokens(from, end);
#pragma unroll
            for (int i = 0; i < LOADS; ++i)
                if (from + i * WAVE < end) n_wave += __popcll(__ballot(owned(tok[i])));
        }
        if (lane == 0) sm.counts[wave] = n_wave;
        __syncthreads();                                        // also: the previous window's list and number of heads are no longer read
        if (tid == 0) sm.heads = 0;                             // counted up behind the next barrier
        int n = 0;
        at = 0;
#pragma unroll
        for (int k = 0; k < EMB_WAVES; ++k) { const int c = sm.counts[k]; at += k < wave ? c : 0; n += c; }
        return __builtin_amdgcn_readfirstlane(n);
    };
    int window = M, n = count_owned(0, M, !(hot && kept));
    if (n > EMB_LIST && !hot) {                                 // too many even without the frequent tokens?
        (void)count_buckets();
        by_bucket = true;
        n = count_owned(0, M);
    }
    int w0 = 0;
    // a window of which the list should be nearly full, by what the last one had (EMB_LIST positions always fit)
    auto fitting = [&] {
        const float even = (float)window * (EMB_LIST * 0.875f) / (float)max(n, 1);
        return __builtin_amdgcn_readfirstlane(min(M - w0, max(EMB_LIST, (int)min(even, (float)M))));
    };
    auto next_window = [&] {
        w0 += window;
        if (w0 >= M) return;
        window = fitting();
        n = count_owned(w0, window);
    };
    for (; w0 < M; next_window()) {
        while (n > EMB_LIST) {                                  // (uniform)
            window = fitting();
            __syncthreads();                                    // the counts have been read
            n = count_owned(w0, window);
        }
        // 1. the window's owned positions, ascending
        {
            const int each = eighth(window), end = min(w0 + min((wave + 1) * each, window), M);
            for (int from = w0 + wave * each; from < end; from += EMB_THREADS) {
                if (each > EMB_THREADS) load_tokens(from, end);         // else they are still there
#pragma unroll
                for (int i = 0; i < LOADS; ++i) {
                    const bool own = owned(tok[i]);
                    const unsigned long long m = __ballot(own);
                    if (own) {
                        const int j = at + __popcll(m & ((1ull << lane) - 1));
                        sm.tok[j] = tok[i];
                        sm.pos[j] = from + i * WAVE + lane;
                    }
                    at += __popcll(m);
                }
            }
        }
        __syncthreads();
        if (n == 0) continue;
        // 2. heads: entries whose token does not occur earlier in the list (their order does not matter)
        for (int j0 = 0; j0 < n; j0 += EMB_THREADS) {
            const int j = j0 + tid;
            const int v = j < n ? sm.tok[j] : -1;
            bool seen = j >= n;
            for (int k = 0; k < n; k += 16) {                   // entries beyond n are compared by nobody (k < j < n)
#pragma unroll
                for (int u = 0; u < 16; u += 4) {
                    const int4 e = *reinterpret_cast<const int4*>(&sm.tok[k + u]);
                    seen |= (k + u < j && e.x == v) || (k + u + 1 < j && e.y == v) || (k + u + 2 < j && e.z == v) || (k + u + 3 < j && e.w == v);
                }
                if (__ballot(!seen && k + 16 < j) == 0) break;
            }
            if (!seen) sm.head[atomicAdd(&sm.heads, 1)] = (unsigned short)j;
        }
        __syncthreads();
        const int heads = __builtin_amdgcn_readfirstlane(sm.heads);
        auto matches = [&](int from, int v, int mask) { return __ballot(from + lane < n && ((sm.tok[min(from + lane, n - 1)] ^ v) & mask) == 0); };     // of 64 entries
        // 4. frequent tokens: all groups
        if (hot) {
            for (int hd = 0; hd < heads; ++hd) {
                const int first = __builtin_amdgcn_readfirstlane((int)sm.head[hd]), v = __builtin_amdgcn_readfirstlane(sm.tok[first]);
                int count = 0;
                for (int g = first & ~(WAVE - 1); g < n; g += WAVE) {
                    const unsigned long long m = matches(g, v, -1);
                    if (g / WAVE % EMB_WAVES == wave && ((m >> lane) & 1)) sm.same[count + __popcll(m & ((1ull << lane) - 1))] = (unsigned short)(g + lane);
                    count += __popcll(m);
                }
                __syncthreads();
                const T* src = dx + (size_t)min(piece, nchunk - 1) * V;
                float a[V];
#pragma unroll
                for (int e = 0; e < V; ++e) a[e] = 0.f;
                for (int i = group; i < count; i += EMB_GROUPS * EMB_FLY) {
                    uint4 q[EMB_FLY];
#pragma unroll
                    for (int u = 0; u < EMB_FLY; ++u)
                        q[u] = *reinterpret_cast<const uint4*>(src + (size_t)sm.pos[sm.same[min(i + u * EMB_GROUPS, count - 1)]] * H);
#pragma unroll
                    for (int u = 0; u < EMB_FLY; ++u)
                        if (i + u * EMB_GROUPS < count) add_row(a, q[u]);
                }
#pragma unroll
                for (int e = 0; e < V; ++e) {                   // the wavefront's four groups
                    a[e] += __shfl_xor(a[e], 16, WAVE);
                    a[e] += __shfl_xor(a[e], 32, WAVE);
                    if (lane < EMB_LANES) sm.part[wave][lane * V + e] = a[e];
                }
                __syncthreads();                                // also: this token's indices are no longer read
                const int col = slice * EMB_LANES * V + tid;
                if (tid < EMB_LANES * V && col < H) {
                    float sum = 0.f;
#pragma unroll
                    for (int k = 0; k < EMB_WAVES; ++k) sum += sm.part[k][tid];
                    dwte[(size_t)v * H + col] += sum;           // (partial rows are written anew behind the next token's first barrier)
                }
            }
            continue;
        }
        // 3. one wavefront per token and 64 pieces of its row
        const int parts = (nchunk + WAVE - 1) / WAVE;
        for (int task = wave; task < heads * parts; task += EMB_WAVES) {
            const int first = __builtin_amdgcn_readfirstlane((int)sm.head[task / parts]), v = __builtin_amdgcn_readfirstlane(sm.tok[first]);
            if (!by_bucket && n > hot_from) {                    // a frequent token?  (the list holds all of its bucket)
                int count = 0;
                for (int g = 0; g < n; g += WAVE) count += __popcll(matches(g, v, EMB_BUCKETS - 1));
                if (count > hot_from) continue;
            }
            const int at_piece = task % parts * WAVE + lane;
            const size_t col = (size_t)min(at_piece, nchunk - 1) * V;
            float* out = dwte + (size_t)v * H + col;
            f32x4_u sum[V / 4];
#pragma unroll
            for (int e = 0; e < V / 4; ++e) sum[e] = *reinterpret_cast<const f32x4_u*>(out + 4 * e);
            float a[V];
#pragma unroll
            for (int e = 0; e < V; ++e) a[e] = 0.f;
            for (int g = first & ~(WAVE - 1); g < n; g += WAVE) {
                unsigned long long m = matches(g, v, -1);
                while (m) {
                    uint4 q[EMB_FLY];
                    int rows = 0;
#pragma unroll
                    for (int u = 0; u < EMB_FLY; ++u)
                        if (m) {
                            q[u] = *reinterpret_cast<const uint4*>(dx + (size_t)sm.pos[g + __ffsll((long long)m) - 1] * H + col);
                            m &= m - 1;
                            rows = u + 1;
                        }
#pragma unroll
                    for (int u = 0; u < EMB_FLY; ++u)
                        if (u < rows) add_row(a, q[u]);
                }
            }
            if (at_piece < nchunk)
#pragma unroll
                for (int e = 0; e < V / 4; ++e) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) sum[e][k] += a[4 * e + k];
                    *reinterpret_cast<f32x4_u*>(out + 4 * e) = sum[e];
                }
        }
    }
}

// ---- softmax cross-entropy over one vocabulary row per workgroup, in place:
// z[t, :] <- scale * (softmax(z[t, :]) - onehot(target[t])),  loss_rows[t] = scale * (lse - z[t, target]).
// One online pass for the running maximum and sum, one pass to write.
template <typename T>
__global__ __launch_bounds__(EDGE_THREADS) void xent_kernel(T* __restrict__ z, const int* __restrict__ targets,
                                                            float* __restrict__ loss_rows, int vocab, float scale) {
    constexpr int V = Elem<T>::VEC;
    constexpr int NW = EDGE_THREADS / WAVE;
    __shared__ float red_m[NW], red_s[NW];
    const int t = blockIdx.x, tid = threadIdx.x, lane = tid % WAVE, wave = tid / WAVE;
    T* row = z + (size_t)t * vocab;
    const int tgt = min(max(targets[t], 0), vocab - 1);
    float m = -3.0e38f, s = 0.f;
    for (int c = tid; c < vocab / V; c += EDGE_THREADS) {
        float v[V];
        load_vec<T>(row + c * V, v);
        float cm = v[0];
#pragma unroll
        for (int e = 1; e < V; ++e) cm = fmaxf(cm, v[e]);
        const float nm = fmaxf(m, cm);
        float add = 0.f;
#pragma unroll
        for (int e = 0; e < V; ++e) add += expf(v[e] - nm);
        s = s * expf(m - nm) + add;
        m = nm;
    }
    // combine (max, sum) pairs: across the lanes, then across the wavefronts in fixed order
    const float wm = wave_max(m);
    const float ws = wave_sum(s * expf(m - wm));
    if (lane == 0) { red_m[wave] = wm; red_s[wave] = ws; }
    __syncthreads();
    float gm = red_m[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) gm = fmaxf(gm, red_m[w]);
    float gs = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) gs += red_s[w] * expf(red_m[w] - gm);
    const float lse = gm + logf(gs);
    const float inv = 1.0f / gs;
    if (tid == 0) loss_rows[t] = scale * (lse - Elem<T>::to_f(row[tgt]));
    __syncthreads();                                  // the target logit is read before anyone overwrites it
    for (int c = tid; c < vocab / V; c += EDGE_THREADS) {
        float v[V];
        load_vec<T>(row + c * V, v);
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const float p = expf(v[e] - gm) * inv;
            v[e] = scale * (p - ((c * V + e) == tgt ? 1.0f : 0.0f));
        }
        store_vec<T>(row + c * V, v);
    }
}

// The same for bf16 rows that fit a workgroup's registers (up to NT * NV pieces of 16 bytes, kept as they
// arrive): the row is read once and written once.  What bounds it is that traffic as long as the exponentials
// hide behind it, which the general kernel's do not (expf and a running maximum are some 50 vector instructions
// an element, and it reads the row twice): 4096 x 50304 231 -> 155 us.  So the maximum comes first, an exponential is the
// hardware's exp2 of (z - max) log2(e) - the difference of two bf16 values first, which leaves no common
// error in the sum - and 64 registers a lane keep two workgroups of 1024 on a CU, one loading while the other works.
// The rounded product costs a probability e^-x up to 6e-8 x relative, against a bf16 result's 2e-3.  Made good with two
// more operations an element the kernel is 10 % slower and its loss rows and gradients are no nearer to float64 (3.2e-8 and
// 1.17e-4 relative at 4096 x 50304).
template <int NT, int NV>
__global__ __launch_bounds__(NT, 8) void xent_row_kernel(bf16_t* __restrict__ z, const int* __restrict__ targets,
                                                         float* __restrict__ loss_rows, int vocab, float scale) {
    constexpr int NW = NT / WAVE;
    constexpr float LOG2E = 1.4426950408889634f;
    __shared__ float red_m[NW], red_s[NW];
    const int t = blockIdx.x, tid = threadIdx.x, lane = tid % WAVE, wave = tid / WAVE, nchunk = vocab / 8;
    bf16_t* row = z + (size_t)t * vocab;
    uint4 q[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = tid + i * NT;
        if (c < nchunk) q[i] = *reinterpret_cast<const uint4*>(row + c * 8);
        else q[i] = make_uint4(0xff80ff80u, 0xff80ff80u, 0xff80ff80u, 0xff80ff80u);      // -inf: adds nothing
    }
    const int tgt = min(max(targets[t], 0), vocab - 1);
    const float z_tgt = (float)row[tgt];
    auto unpack = [&](int i, float* v) {
        // widened anew in every pass: kept from pass to pass, the floats would take 64 registers more and spill
        asm volatile("" : "+v"(q[i].x), "+v"(q[i].y), "+v"(q[i].z), "+v"(q[i].w));
        load_vec<bf16_t>(reinterpret_cast<const bf16_t*>(&q[i]), v);
    };
    float m = -3.0e38f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        float v[8];
        unpack(i, v);
#pragma unroll
        for (int e = 0; e < 8; ++e) m = fmaxf(m, v[e]);
    }
    m = wave_max(m);
    if (lane == 0) red_m[wave] = m;
    __syncthreads();                                  // also: the target logit has been read
    m = wave_max(red_m[lane % NW]);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        float v[8];
        unpack(i, v);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = __builtin_amdgcn_exp2f((v[e] - m) * LOG2E);
        s += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    }
    s = wave_sum(s);
    if (lane == 0) red_s[wave] = s;
    __syncthreads();
    const float gs = wave_sum(lane < NW ? red_s[lane] : 0.f);
    const float inv = 1.0f / gs;
    if (tid == 0) loss_rows[t] = scale * (m + logf(gs) - z_tgt);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = tid + i * NT;
        if (c >= nchunk) continue;
        float v[8];
        unpack(i, v);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = __builtin_amdgcn_exp2f((v[e] - m) * LOG2E) * inv;
        if (c == tgt / 8)
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] -= e == tgt % 8 ? 1.0f : 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] *= scale;
        store_vec<bf16_t>(row + c * 8, v);
    }
}

// loss[0] += sum of loss_rows in a fixed order (one workgroup)
__global__ __launch_bounds__(EDGE_THREADS) void loss_sum_kernel(const float* __restrict__ loss_rows, int n, float* __restrict__ loss) {
    __shared__ float red[EDGE_THREADS];
    float s = 0.f;
    for (int i = threadIdx.x; i < n; i += EDGE_THREADS) s += loss_rows[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = EDGE_THREADS / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] += red[0];
}

int check_edge(int dtype, int tokens, int seq, int hidden, int vocab, bool vocab_rows_only) {
    if (dtype != CHIMERA_F32 && dtype != CHIMERA_BF16) return fail(CHIMERA_EINVAL, "unknown dtype %d", dtype);
    if (tokens < 1 || seq < 1 || hidden < 1 || vocab < 1) return fail(CHIMERA_EINVAL, "sizes must be positive");
    if (tokens % seq) return fail(CHIMERA_EINVAL, "tokens=%d is not a multiple of seq=%d", tokens, seq);
    // the vocabulary only indexes table rows in the embedding; in the head it is a matrix dimension
    if (hidden % 8 || (!vocab_rows_only && vocab % 8))
        return fail(CHIMERA_EINVAL, "hidden=%d%s must be a multiple of 8", hidden, vocab_rows_only ? "" : " and the vocabulary");
    return CHIMERA_OK;
}

size_t aligned(size_t b) { return (b + 255) / 256 * 256; }

struct HeadLayout { size_t h, mean, rstd, logits, loss_rows, dh, scratch, need, slabs, total; };
HeadLayout head_layout(int dtype, int M, int H, int V) {
    const size_t e = dtype == CHIMERA_F32 ? 4 : 2;
    HeadLayout l{};
    size_t b = 0;
    auto take = [&](size_t bytes) { size_t r = b; b += aligned(bytes); return r; };
    l.h = take((size_t)M * H * e);
    l.mean = take((size_t)M * 4);
    l.rstd = take((size_t)M * 4);
    l.logits = take((size_t)M * V * e);
    l.loss_rows = take((size_t)M * 4);
    l.dh = take((size_t)M * H * e);
    l.scratch = take(layernorm_bwd_scratch_floats(M, H) * 4);
    // the slabs of the data gradient's partial sums; a workspace that holds only what comes before them does too
    l.need = b;
    l.slabs = take(dtype == CHIMERA_BF16 ? gemm_mfma_split_bytes(M, H, V) : 0);
    l.total = b;
    return l;
}

}  // namespace
}  // namespace chimera

using namespace chimera;

#define EDGE_TRY(expr) do { int rc__ = (expr); if (rc__) return rc__; } while (0)

extern "C" {

int chimera_op_embedding_fwd(int dtype, int tokens, int seq, int hidden, int vocab, const int32_t* d_tokens,
                             const void* d_wte, const void* d_wpe, void* d_x, void* hip_stream) {
    EDGE_TRY(check_edge(dtype, tokens, seq, hidden, vocab, true));
    if (!d_tokens || !d_wte || !d_wpe || !d_x) return fail(CHIMERA_EINVAL, "NULL operand");
    if (((uintptr_t)d_wte | (uintptr_t)d_wpe | (uintptr_t)d_x) & 15) return fail(CHIMERA_EINVAL, "buffers must be 16-byte aligned");
    const dim3 grid((tokens + EDGE_THREADS / WAVE - 1) / (EDGE_THREADS / WAVE)), block(EDGE_THREADS);
    hipStream_t s = (hipStream_t)hip_stream;
    if (dtype == CHIMERA_F32)
        hipLaunchKernelGGL(embed_fwd_kernel<float>, grid, block, 0, s, d_tokens, (const float*)d_wte, (const float*)d_wpe,
                           (float*)d_x, tokens, seq, hidden, vocab);
    else
        hipLaunchKernelGGL(embed_fwd_kernel<bf16_t>, grid, block, 0, s, d_tokens, (const bf16_t*)d_wte, (const bf16_t*)d_wpe,
                           (bf16_t*)d_x, tokens, seq, hidden, vocab);
    CHIMERA_LAUNCH_CHECK("embedding forward");
    return CHIMERA_OK;
}

int chimera_op_embedding_bwd(int dtype, int tokens, int seq, int hidden, int vocab, const int32_t* d_tokens, const void* d_dx,
                             float* d_dwte, float* d_dwpe, void* hip_stream) {
    EDGE_TRY(check_edge(dtype, tokens, seq, hidden, vocab, true));
    if (!d_tokens || !d_dx || !d_dwte || !d_dwpe) return fail(CHIMERA_EINVAL, "NULL operand");
    if ((uintptr_t)d_dx & 15) return fail(CHIMERA_EINVAL, "dx must be 16-byte aligned");
    const int vec = dtype == CHIMERA_F32 ? 4 : 8;
    if (hidden / vec > 2 * EDGE_THREADS) return fail(CHIMERA_EINVAL, "hidden=%d too wide for the embedding backward (max %d)", hidden, 2 * EDGE_THREADS * vec);
    hipStream_t s = (hipStream_t)hip_stream;
    const size_t pieces = (size_t)seq * (hidden / vec);
    // the workgroups of frequent tokens, which may take longest, go first
    const int slices = (hidden / vec + EMB_LANES - 1) / EMB_LANES;
    const int hot_from = embed_hot_from(tokens);
    int hot_classes = tokens > hot_from ? EMB_HOT_CLASSES_MAX : 0;
    while (hot_classes > EMB_HOT_CLASSES_MIN && hot_classes * slices > (tokens > 4096 ? 512 : 256)) hot_classes /= 2;
    int owners = EMB_OWNERS_MAX;
    while (owners > EMB_OWNERS_MIN && owners * 4 > tokens) owners /= 2;          // four positions each
    const dim3 grid(hot_classes * slices + owners + (unsigned)((pieces + EMB_THREADS - 1) / EMB_THREADS)), block(EMB_THREADS);
    if (dtype == CHIMERA_F32)
        hipLaunchKernelGGL(embed_bwd_kernel<float>, grid, block, 0, s, d_tokens, (const float*)d_dx, d_dwte, d_dwpe, tokens, seq, hidden,
                           vocab, owners, hot_classes, slices, hot_from);
    else
        hipLaunchKernelGGL(embed_bwd_kernel<bf16_t>, grid, block, 0, s, d_tokens, (const bf16_t*)d_dx, d_dwte, d_dwpe, tokens, seq, hidden,
                           vocab, owners, hot_classes, slices, hot_from);
    CHIMERA_LAUNCH_CHECK("embedding backward");
    return CHIMERA_OK;
}

int chimera_op_softmax_xent(int dtype, int rows, int vocab, void* d_logits, const int32_t* d_targets, float scale,
                            float* d_loss_rows, float* d_loss, void* hip_stream) {
    if (dtype != CHIMERA_F32 && dtype != CHIMERA_BF16) return fail(CHIMERA_EINVAL, "unknown dtype %d", dtype);
    if (rows < 1 || vocab < 1 || vocab % 8) return fail(CHIMERA_EINVAL, "rows=%d must be positive, vocab=%d a positive multiple of 8", rows, vocab);
    if (!d_logits || !d_targets || !d_loss_rows || !d_loss) return fail(CHIMERA_EINVAL, "NULL operand");
    if ((uintptr_t)d_logits & 15) return fail(CHIMERA_EINVAL, "logits must be 16-byte aligned");
    hipStream_t s = (hipStream_t)hip_stream;
    if (dtype == CHIMERA_F32)
        hipLaunchKernelGGL(xent_kernel<float>, dim3(rows), dim3(EDGE_THREADS), 0, s, (float*)d_logits, d_targets, d_loss_rows, vocab, scale);
    else {
        // registers for the row: a small workgroup as long as four pieces a thread do, else 1024 threads; beyond
        // eight pieces a thread (65536 columns) the row stays in memory
        bf16_t* z = (bf16_t*)d_logits;
#define XENT_ROW(NT, NV) hipLaunchKernelGGL((xent_row_kernel<NT, NV>), dim3(rows), dim3(NT), 0, s, z, d_targets, d_loss_rows, vocab, scale)
        if (vocab <= 256 * 8) XENT_ROW(256, 1);
        else if (vocab <= 512 * 8) XENT_ROW(256, 2);
        else if (vocab <= 1024 * 8) XENT_ROW(256, 4);
        else if (vocab <= 2048 * 8) XENT_ROW(1024, 2);
        else if (vocab <= 4096 * 8) XENT_ROW(1024, 4);
        else if (vocab <= 8192 * 8) XENT_ROW(1024, 8);
        else hipLaunchKernelGGL(xent_kernel<bf16_t>, dim3(rows), dim3(EDGE_THREADS), 0, s, z, d_targets, d_loss_rows, vocab, scale);
#undef XENT_ROW
    }
    CHIMERA_LAUNCH_CHECK("softmax cross-entropy");
    hipLaunchKernelGGL(loss_sum_kernel, dim3(1), dim3(EDGE_THREADS), 0, s, d_loss_rows, rows, d_loss);
    CHIMERA_LAUNCH_CHECK("loss sum");
    return CHIMERA_OK;
}

size_t chimera_head_workspace_bytes(int dtype, int tokens, int hidden, int vocab) {
    if (tokens < 1 || hidden < 1 || vocab < 1) return 0;
    return head_layout(dtype, tokens, hidden, vocab).total;
}

int chimera_head_loss(int dtype, int tokens, int hidden, int vocab, const void* d_y, const int32_t* d_targets,
                      const void* d_lnf_g, const void* d_lnf_b, const void* d_w_head, float scale, void* d_dy,
                      float* d_dlnf_g, float* d_dlnf_b, float* d_dw_head, float* d_loss, void* d_workspace,
                      size_t workspace_bytes, void* hip_stream) {
    EDGE_TRY(check_edge(dtype, tokens, 1, hidden, vocab, false));
    if (!d_y || !d_targets || !d_lnf_g || !d_lnf_b || !d_w_head || !d_dy || !d_dlnf_g || !d_dlnf_b || !d_dw_head || !d_loss || !d_workspace)
        return fail(CHIMERA_EINVAL, "NULL operand");
    const HeadLayout l = head_layout(dtype, tokens, hidden, vocab);
    if (workspace_bytes < l.need) return fail(CHIMERA_ENOMEM, "workspace holds %zu bytes, need %zu", workspace_bytes, l.need);
    if (((uintptr_t)d_workspace & 255) || (((uintptr_t)d_y | (uintptr_t)d_dy | (uintptr_t)d_w_head | (uintptr_t)d_dw_head) & 15))
        return fail(CHIMERA_EINVAL, "workspace must be 256-byte aligned, tensors 16-byte aligned");
    const int M = tokens, H = hidden, V = vocab;
    char* ws = (char*)d_workspace;
    void* h = ws + l.h;
    float* mean = (float*)(ws + l.mean);
    float* rstd = (float*)(ws + l.rstd);
    void* logits = ws + l.logits;
    float* loss_rows = (float*)(ws + l.loss_rows);
    void* dh = ws + l.dh;
    float* scratch = (float*)(ws + l.scratch);
    auto gemm = [&](const GemmArgs& g) {
        if (dtype == CHIMERA_BF16 && gemm_mfma_supports(g)) return gemm_mfma_bf16(g, hip_stream);
        if (dtype == CHIMERA_F32 && gemm_f32_supports(g)) return gemm_f32(g, hip_stream);
        return gemm_reference(dtype, g, hip_stream);
    };
    // h = LayerNorm(y)
    EDGE_TRY(layernorm_fwd(dtype, M, H, d_y, 0, d_lnf_g, d_lnf_b, h, mean, rstd, hip_stream));
    // z = h W
    GemmArgs f{};
    f.m = M; f.n = V; f.k = H; f.a = h; f.lda = H; f.a_kc = 1; f.b = d_w_head; f.ldb = V; f.b_kc = 0; f.c = logits; f.epilogue = EPI_NONE;
    EDGE_TRY(gemm(f));
    // loss and dz (in place of z)
    EDGE_TRY(chimera_op_softmax_xent(dtype, M, V, logits, d_targets, scale, loss_rows, d_loss, hip_stream));
    // dh = dz W^T
    GemmArgs d{};
    d.m = M; d.n = H; d.k = V; d.a = logits; d.lda = V; d.a_kc = 1; d.b = d_w_head; d.ldb = V; d.b_kc = 1; d.c = dh; d.epilogue = EPI_NONE;
    if (dtype == CHIMERA_BF16 && l.total > l.need && workspace_bytes >= l.total && gemm_mfma_supports(d))
        EDGE_TRY(gemm_mfma_split(d, (float*)(ws + l.slabs), hip_stream));
    else
        EDGE_TRY(gemm(d));
    // dW += h^T dz
    GemmArgs w{};
    w.m = H; w.n = V; w.k = M; w.a = h; w.lda = H; w.a_kc = 0; w.b = logits; w.ldb = V; w.b_kc = 0; w.c = d_dw_head; w.epilogue = EPI_ACCUM_F32;
    EDGE_TRY(gemm(w));
    // dy, dg, db: LayerNorm backward without a residual path
    return layernorm_bwd(dtype, M, H, dh, d_y, 0, mean, rstd, d_lnf_g, nullptr, 0, d_dy, nullptr, d_dlnf_g, d_dlnf_b, scratch, 0, hip_stream);
}

}  // extern "C"
