// specvlm_accept: which drafted tokens survive the target's verification
// (Sec. 2.1; greedy target decoding as in App. A, or the rejection-sampling rule
// of speculative sampling that keeps the target's output distribution).
//
// Pass 1 (many workgroups): per (request, row, vocab chunk) partial statistics
//   -- argmax with lowest-index ties for greedy; running (max, sum exp) of
//   logit/T for the target rows and the draft rows for sampling.
// Pass 2, greedy (one workgroup per request): merge the partials and walk the gamma tests in order.
// Pass 2, sampling (many workgroups): every workgroup merges the partials and repeats the gamma
//   accept tests (a few loads), so all agree on the first rejected position n; each then sums the
//   mass of the residual max(p - q, 0) at row n (of p when every draft survived) over its chunk.
//   The workgroup of a request that finishes last goes on: inverse CDF over the chunks, then over
//   the owning chunk's segments, then over the owning segment's tokens.
// The drawn token lies where fp32 sums put the uniform, so it depends on their order wherever the uniform
// is within rounding of a step of the CDF.  The order is therefore fixed by the vocabulary alone -- never by
// the batch, the grid or who arrives when (tests/sampling_order.py has it in full).
#include "common.h"

namespace specvlm {

constexpr int kAccThreads = 1024;
constexpr int kAccWaves = kAccThreads / kWave;
constexpr int kAccChunk = 8192;        // vocab entries per pass-1 workgroup
constexpr int kAccSegs = kAccWaves;    // segments of a chunk, in token order, one per wave of the second sampling pass
constexpr int kAccShort = kAccThreads; // vocabularies of at most so many have sampling kernels of their own

struct AcceptParams {
    const float* target;      // [batch, gamma+1, vocab]
    const float* draft;       // [batch, gamma, vocab] or null
    const int32_t* tokens;    // [batch, gamma]
    const float* uniforms;    // [batch, gamma+1] or null
    int batch, gamma, vocab, n_chunks;
    float inv_t_log2;         // log2(e) / temperature
    int32_t* n_accepted;
    int32_t* out_tokens;
    float* part_val;          // [batch][rows][n_chunks]   max
    float* part_aux;          // [batch][rows][n_chunks]   sum exp (sampling) / argmax index bits (greedy)
    float* tok_logit;         // sampling: [batch][2 * gamma + 1] logit of the drafted token in target and draft rows
    float* chunk_mass;        // sampling: [batch][n_chunks] residual (or target) mass of row n per chunk
    float* seg_mass;          // sampling: [batch][n_chunks][kAccSegs] the same per segment, or null
    uint32_t* arrived;        // sampling: [batch] chunks that are done, cleared by pass 1
};

__device__ __forceinline__ void argmax_merge(float& bv, int& bi, float v, int i)
{
    // larger value wins; equal values: lower index wins.  (i < 0 = empty; no NaN gets here)
    if (i >= 0 && (bi < 0 || v > bv || (v == bv && i < bi))) { bv = v; bi = i; }
}

// Wave-wide reductions over lane ^ 32, ^ 16, ^ 8, ^ 4, ^ 2 and ^ 1, in this order: swaps of half waves and of rows, then DPP in
// rows of 16 (rotations by 8 and 4, which reach the partner once the higher bits no longer matter).  The same bits
// as six shuffles, each of which is an LDS round trip.
template <typename OP> __device__ __forceinline__ float wave_reduce(float x, OP op)
{
    auto half = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = op(__uint_as_float(half[0]), __uint_as_float(half[1]));
    auto row = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = op(__uint_as_float(row[0]), __uint_as_float(row[1]));
    x = op(x, row_move<0x128>(x));
    x = op(x, row_move<0x124>(x));
    x = op(x, row_move<0x4E>(x));
    return op(x, row_move<0xB1>(x));
}

__device__ __forceinline__ float wave_sum(float x) { return wave_reduce(x, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float wave_max(float x) { return wave_reduce(x, [](float a, float b) { return fmaxf(a, b); }); }
__device__ __forceinline__ float from_lane(float x, int lane) { return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), lane)); }

// Argmax over groups of 16 lanes, and with WAVE over the wave, the same way: every lane ends with the group's (the order of the exchanges
// does not matter, of equal values the lowest index is taken).  With shuffles, two LDS round trips a step, greedy acceptance of 152064
// tokens at gamma 5 took 6.72 us from a graph instead of 6.35, of 32000 at gamma 1 6.38 instead of 6.17, a tree of 25 nodes 9.6 instead of 9.2.
template <bool WAVE> __device__ __forceinline__ void argmax_reduce(float& bv, int& bi)
{
    if constexpr (WAVE) {
        const auto v = __builtin_amdgcn_permlane32_swap(__float_as_uint(bv), __float_as_uint(bv), false, false);
        const auto i = __builtin_amdgcn_permlane32_swap((uint32_t)bi, (uint32_t)bi, false, false);
        bv = __uint_as_float(v[0]); bi = (int)i[0];
        argmax_merge(bv, bi, __uint_as_float(v[1]), (int)i[1]);
        const auto v2 = __builtin_amdgcn_permlane16_swap(__float_as_uint(bv), __float_as_uint(bv), false, false);
        const auto i2 = __builtin_amdgcn_permlane16_swap((uint32_t)bi, (uint32_t)bi, false, false);
        bv = __uint_as_float(v2[0]); bi = (int)i2[0];
        argmax_merge(bv, bi, __uint_as_float(v2[1]), (int)i2[1]);
    }
    argmax_merge(bv, bi, row_move<0x128>(bv), __float_as_int(row_move<0x128>(__int_as_float(bi))));
    argmax_merge(bv, bi, row_move<0x124>(bv), __float_as_int(row_move<0x124>(__int_as_float(bi))));
    argmax_merge(bv, bi, row_move<0x4E>(bv), __float_as_int(row_move<0x4E>(__int_as_float(bi))));
    argmax_merge(bv, bi, row_move<0xB1>(bv), __float_as_int(row_move<0xB1>(__int_as_float(bi))));
}

// A thread's share of a chunk [lo, hi): logits lo + thread + 256 j, all requested before the first is looked at; past the end
// it reads the last one again, which the caller leaves out.  (With a test around each load sampling takes up to 3 % longer:
// 152064 tokens, gamma 7, 2 requests 17.1 instead of 16.7 us, 4 requests 20.9 instead of 20.2;  greedy 7.5 instead of 7.35.)
template <int N>
__device__ __forceinline__ void load_share(const float* x, int lo, int hi, float (&y)[N])
{
#pragma unroll
    for (int j = 0; j < N; ++j) y[j] = x[min(lo + j * 256 + (int)threadIdx.x, hi - 1)];
}

// ---------------------------------------------------------------- greedy ----
__global__ __launch_bounds__(256)
void accept_argmax_partial(const AcceptParams p)
{
    __shared__ float s_v[4];
    __shared__ int s_i[4];
    const int chunk = blockIdx.x, row = blockIdx.y, b = blockIdx.z;
    const float* x = p.target + ((int64_t)b * (p.gamma + 1) + row) * p.vocab;
    const int lo = chunk * kAccChunk, hi = min(p.vocab, lo + kAccChunk);
    constexpr int N = kAccChunk / 256;                           // tokens of a thread
    float y[N];
    load_share(x, lo, hi, y);
#pragma unroll
    for (int j = 0; j < N; ++j) y[j] = lo + j * 256 + (int)threadIdx.x < hi ? y[j] : -INFINITY;
    // A NaN is greater than nothing: it must not become a share's maximum, or it would hide the tokens that a merge
    // compares with it, so the search starts at -inf.  It starts at token 0, and a NaN there stays: nothing is greater.
    if (lo == 0 && threadIdx.x == 0 && y[0] != y[0]) y[0] = INFINITY;
    float bv = -INFINITY;
    int bi = lo + (int)threadIdx.x < hi ? lo + (int)threadIdx.x : -1;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if (j % 4 == 0 && lo + j * 256 >= hi) break;                       // (a short chunk: 1024 tokens are four steps)
        if (y[j] > bv) { bv = y[j]; bi = lo + j * 256 + threadIdx.x; }     // ascending tokens: the first maximum is kept
    }
    argmax_reduce<true>(bv, bi);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) { s_v[wave] = bv; s_i[wave] = bi; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) argmax_merge(bv, bi, s_v[w], s_i[w]);
        const int64_t slot = ((int64_t)b * (p.gamma + 1) + row) * p.n_chunks + chunk;
        p.part_val[slot] = bv;
        p.part_aux[slot] = __int_as_float(bi);
    }
}

// Argmax of every row from the pass-1 partials, into LDS.  Bound: round trips.  One lane per row takes eight chunks a
// trip and all rows at once (one wave); 16 lanes per row take 64 chunks a trip and 16 rows at once (four waves, and an
// exchange): accept_final_lanes takes the fewer trips.
constexpr int kFinalLanes = 16, kFinalThreads = 256;            // (argmax_reduce goes over 16 lanes)
constexpr int final_threads(int lanes) { return lanes == 1 ? kWave : kFinalThreads; }
template <int LANES> __device__ __forceinline__ void accept_merge_argmax(const AcceptParams& p, int b, int rows, int* s_t)
{
    constexpr int LOADS = LANES == 1 ? 8 : 4;                    // chunks in flight per lane
    const int l = threadIdx.x % LANES;
    for (int row = threadIdx.x / LANES; row < rows; row += final_threads(LANES) / LANES) {
        const int64_t slot = ((int64_t)b * rows + row) * p.n_chunks;
        float bv = 0.f; int bi = -1;
        for (int c0 = l; c0 < p.n_chunks; c0 += LANES * LOADS) {
            float pv[LOADS]; int pi[LOADS];
#pragma unroll
            for (int j = 0; j < LOADS; ++j) {
                const bool in = c0 + LANES * j < p.n_chunks;
                pv[j] = in ? p.part_val[slot + c0 + LANES * j] : 0.f;
                pi[j] = in ? __float_as_int(p.part_aux[slot + c0 + LANES * j]) : -1;
            }
#pragma unroll
            for (int j = 0; j < LOADS; ++j) argmax_merge(bv, bi, pv[j], pi[j]);
        }
        if constexpr (LANES == 16) argmax_reduce<false>(bv, bi);
        if (l == 0) s_t[row] = bi;
    }
}

template <int LANES>
__global__ __launch_bounds__(final_threads(LANES))
void accept_greedy_final(const AcceptParams p)
{
    // one workgroup per request; lane i of its first wave holds drafted token i (gamma <= 64), the first mismatch is
    // found by a ballot and every lane writes its own output
    const int b = blockIdx.x, lane = threadIdx.x;
    __shared__ int s_t[65];
    const int32_t* x = p.tokens + (int64_t)b * p.gamma;
    const int drafted = lane < p.gamma ? x[lane] : -1;           // (in flight while the partials are merged)
    accept_merge_argmax<LANES>(p, b, p.gamma + 1, s_t);
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    const uint64_t mismatch = __ballot(lane < p.gamma && drafted != s_t[lane]);
    const int n = mismatch ? __ffsll((long long)mismatch) - 1 : p.gamma;
    int32_t* out = p.out_tokens + (int64_t)b * (p.gamma + 1);
    for (int i = lane; i <= p.gamma; i += 64)
        out[i] = i < n ? drafted : (i == n ? s_t[n] : -1);       // (i < n implies i = lane < gamma)
    if (lane == 0) p.n_accepted[b] = n;
}

// -------------------------------------------------------------- sampling ----
// rows 0..gamma: target rows; rows gamma+1..2*gamma: draft rows 0..gamma-1
template <int CHUNK>
__global__ __launch_bounds__(256)
void accept_softmax_partial(const AcceptParams p)
{
    __shared__ float s_m[4], s_z[4];
    const int chunk = blockIdx.x, row = blockIdx.y, b = blockIdx.z;
    // (pass 2 would look the drafted token's logits up behind its tokens, two round trips that nothing there covers)
    const int draft = row <= p.gamma ? row : row - p.gamma - 1;
    const int tok = draft < p.gamma ? p.tokens[(int64_t)b * p.gamma + draft] : -1;
    if (chunk == 0 && row == 0 && threadIdx.x == 0) p.arrived[b] = 0u;
    const float* x = row <= p.gamma
        ? p.target + ((int64_t)b * (p.gamma + 1) + row) * p.vocab
        : p.draft + ((int64_t)b * p.gamma + (row - p.gamma - 1)) * p.vocab;
    const int lo = chunk * CHUNK, hi = min(p.vocab, lo + CHUNK);
    constexpr int N = CHUNK / 256;                               // tokens of a thread
    float y[N];                                      // (kept for the second pass over them)
    load_share(x, lo, hi, y);
#pragma unroll
    for (int j = 0; j < N; ++j) y[j] = lo + j * 256 + (int)threadIdx.x < hi ? y[j] * p.inv_t_log2 : -INFINITY;
    if (threadIdx.x == 0 && tok >= lo && tok < hi) p.tok_logit[(int64_t)b * (2 * p.gamma + 1) + row] = x[tok];
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < N; ++j) m = fmaxf(m, y[j]);
    m = wave_max(m);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) s_m[wave] = m;
    __syncthreads();
    m = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));
    float z = 0.f;
#pragma unroll
    for (int j = 0; j < N; ++j) z += fast_exp2(y[j] - m);       // (-inf padding adds 0)
    z = wave_sum(z);
    if (lane == 0) s_z[wave] = z;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int64_t slot = ((int64_t)b * (2 * p.gamma + 1) + row) * p.n_chunks + chunk;
        p.part_val[slot] = m;
        p.part_aux[slot] = (s_z[0] + s_z[1]) + (s_z[2] + s_z[3]);
    }
}

// Merged (max, sum exp) of every row from its pass-1 partials, into LDS.  The sum runs over the chunks in ascending order, rescaled
// to the maximum so far at every eighth, so eight lanes share a row, a chunk each, and only the additions are one after
// the other (done in the first four lanes, which see the other four mirrored).  kMergeAhead groups of eight are requested together.
constexpr int kMergeAhead = 4;
__device__ __forceinline__ void accept_merge_rows(const AcceptParams& p, int rows, const float* val, const float* aux,
                                                  float* s_m, float* s_z)
{
    const int j = threadIdx.x & 7;
    for (int row = threadIdx.x >> 3; row < rows; row += kAccThreads / 8) {
        const int64_t slot = (int64_t)row * p.n_chunks;
        float m = -INFINITY, z = 0.f;
        for (int c0 = 0; c0 < p.n_chunks; c0 += 8 * kMergeAhead) {
            float pm[kMergeAhead], pz[kMergeAhead];
#pragma unroll
            for (int g = 0; g < kMergeAhead; ++g) {
                const int c = min(c0 + 8 * g + j, p.n_chunks - 1);           // (as in load_share)
                pm[g] = val[slot + c]; pz[g] = aux[slot + c];
            }
#pragma unroll
            for (int g = 0; g < kMergeAhead; ++g) {
                if (c0 + 8 * g >= p.n_chunks) break;
                const bool in = c0 + 8 * g + j < p.n_chunks;
                const float top = in ? pm[g] : -INFINITY;
                float mc = fmaxf(top, row_move<0xB1>(top));
                mc = fmaxf(mc, row_move<0x4E>(mc));
                mc = fmaxf(fmaxf(mc, row_move<0x141>(mc)), m);
                const float a = in && pz[g] > 0.f ? pz[g] * fast_exp2(top - mc) : 0.f, b = row_move<0x141>(a);
                z = fmaf(z, mc == -INFINITY ? 0.f : fast_exp2(m - mc), row_move<0x00>(a));
                z += row_move<0x55>(a); z += row_move<0xAA>(a); z += row_move<0xFF>(a);
                z += row_move<0xFF>(b); z += row_move<0xAA>(b); z += row_move<0x55>(b); z += row_move<0x00>(b);
                m = mc;
            }
        }
        if (j == 0) { s_m[row] = m; s_z[row] = z; }
    }
}

// weight of token v at the first rejected position: residual max(p - q, 0), or p when nothing was rejected
struct AcceptWeight {
    const float* trow;
    const float* drow;        // null: no residual
    float inv_t_log2, mt, inv_zt, md, inv_zd;
    // Weights of the lane's tokens lo + lane + 64 j below hi (0 from there on).  Both rows' logits are requested before the
    // first is looked at: with the test for a residual inside, every token was a round trip or two of its own.
    template <int N> __device__ __forceinline__ void operator()(float (&w)[N], int lo, int hi) const
    {
        const int lane = threadIdx.x & 63;
        float t[N], d[N];
        if (lo + 64 * N <= hi) {
            const float* const tl = trow + lo;
            const float* const dl = (drow ? drow : trow) + lo;
#pragma unroll
            for (int j = 0; j < N; ++j) t[j] = tl[lane + 64 * j];
#pragma unroll
            for (int j = 0; j < N; ++j) d[j] = dl[lane + 64 * j];
        } else {                                                 // (as in load_share; hi >= 1)
#pragma unroll
            for (int j = 0; j < N; ++j) t[j] = trow[min(lo + lane + 64 * j, hi - 1)];
            if (drow) {
#pragma unroll
                for (int j = 0; j < N; ++j) d[j] = drow[min(lo + lane + 64 * j, hi - 1)];
            }
        }
#pragma unroll
        for (int j = 0; j < N; ++j) w[j] = fast_exp2(t[j] * inv_t_log2 - mt) * inv_zt;
        if (drow) {
#pragma unroll
            for (int j = 0; j < N; ++j) w[j] = fmaxf(w[j] - fast_exp2(d[j] * inv_t_log2 - md) * inv_zd, 0.f);
        }
#pragma unroll
        for (int j = 0; j < N; ++j) w[j] = lo + lane + 64 * j < hi ? w[j] : 0.f;
    }
};

__device__ __forceinline__ AcceptWeight accept_weight(const AcceptParams& p, int b, int n, float mt, float zt, float md, float zd)
{
    AcceptWeight w;
    const bool residual = n < p.gamma;
    w.trow = p.target + ((int64_t)b * (p.gamma + 1) + n) * p.vocab;
    w.drow = residual ? p.draft + ((int64_t)b * p.gamma + n) * p.vocab : nullptr;
    w.inv_t_log2 = p.inv_t_log2;
    w.mt = mt; w.inv_zt = 1.f / zt;
    w.md = residual ? md : 0.f; w.inv_zd = residual ? 1.f / zd : 0.f;
    return w;
}

// Bound: its chain of round trips -- the partials beside the accept tests' inputs, the rejected row, the masses beside the
// arrival, the owning segment -- and the launches.  As a launch of its own the inverse CDF cost another start, the
// statistics' way through memory and a gap between launches.
//
// gamma 7, 152064 tokens, rows from HBM, us a call from a graph: 1 request 14.9, 8 requests 27.4 (three launches, with the tests'
// logits looked up behind their tokens: 29.9 and 49.5).  Of that the chunk's mass in the order of pass 1 takes 0.7, its weights'
// way through LDS; the last scan by shuffles 0.3.  Chunks of 4096 for few requests and sums in whatever order is the
// shortest were 12.0, but a uniform within rounding of a step then drew another token, and not the same in every batch.
//
// kWhole: the last workgroup of a request goes on.  Pass 1 has cleared the arrival counter, so nothing is asked of the
// workspace's earlier contents, and nobody waits for anybody: every workgroup writes its masses and counts itself in (release),
// the one that finds all others counted (acquire) reads them, at device scope.
// kMasses, kDraw: two launches, without a counter (see accept_one_launch).
// CHUNK = kAccShort: the only chunk, nothing to exchange.
enum AcceptPart { kWhole, kMasses, kDraw };

__device__ __forceinline__ void store_device(float* at, float x) { __hip_atomic_store(at, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float load_device(const float* at) { return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

template <int CHUNK, int PART>
__global__ __launch_bounds__(kAccThreads)
void accept_sample_kernel(const AcceptParams p)
{
    constexpr bool SHORT = CHUNK == kAccShort;
    constexpr int STEPS = CHUNK / kAccThreads;  // of 64 tokens, a wave's segment
    constexpr int COLS = 256, COL_TOKENS = CHUNK / COLS;         // running sums of a chunk's mass, as in pass 1
    __shared__ float s_w[CHUNK];                // the chunk's weights
    __shared__ float s_m[129], s_z[129];        // merged (max, sum) of up to 2*gamma+1 rows
    __shared__ float s_seg[kAccSegs], s_part[COLS / kWave];
    __shared__ float s_top[kAccWaves];
    __shared__ int s_idx[kAccWaves];
    __shared__ float s_mass;
    __shared__ int s_last, s_own;
    const int chunk = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rows = 2 * p.gamma + 1;
    // The gamma accept tests, one per lane (gamma <= 64) and again in every wave, which saves a barrier: their inputs are
    // in flight beside the partials, the first failing test is found by a ballot.
    int tok = -1;
    float t_logit = 0.f, d_logit = 0.f, u = 0.f;
    if (lane < p.gamma) {
        tok = p.tokens[(int64_t)b * p.gamma + lane];
        t_logit = p.tok_logit[(int64_t)b * rows + lane];
        d_logit = p.tok_logit[(int64_t)b * rows + p.gamma + 1 + lane];
        u = p.uniforms[(int64_t)b * (p.gamma + 1) + lane];
    }
    const float u_last = p.uniforms[(int64_t)b * (p.gamma + 1) + p.gamma];
    const float* val = p.part_val + (int64_t)b * rows * p.n_chunks;
    const float* aux = p.part_aux + (int64_t)b * rows * p.n_chunks;
    accept_merge_rows(p, rows, val, aux, s_m, s_z);
    __syncthreads();
    bool ok = true;
    if (lane < p.gamma) {
        const float pt = fast_exp2(t_logit * p.inv_t_log2 - s_m[lane]) / s_z[lane];
        const float qd = fast_exp2(d_logit * p.inv_t_log2 - s_m[p.gamma + 1 + lane]) / s_z[p.gamma + 1 + lane];
        ok = tok >= 0 && tok < p.vocab && u * qd < pt;           // (not a token: cannot be accepted, and has no logits)
    }
    const uint64_t failed = __ballot(!ok);
    const int n = failed ? __ffsll((long long)failed) - 1 : p.gamma;
    const int dn = n < p.gamma ? p.gamma + 1 + n : 0;
    const AcceptWeight weight = accept_weight(p, b, n, s_m[n], s_z[n], s_m[dn], s_z[dn]);
    // a chunk's segments are as wide as it takes to deal it to the waves in token order
    auto segment = [&](int c, int s, int& lo, int& hi) __attribute__((always_inline)) {
        const int from = c * CHUNK, to = min(p.vocab, from + CHUNK);
        const int width = ((to - from + kAccSegs - 1) / kAccSegs + 63) & ~63;
        lo = min(to, from + s * width); hi = min(to, lo + width);
    };
    int lo, hi;
    float w[STEPS];
    // masses of the wave's segment of a chunk: every lane's running sum, then the lanes
    auto segment_mass = [&](int c) __attribute__((always_inline)) {
        segment(c, wave, lo, hi);
        weight(w, lo, hi);
        float mine = 0.f;
#pragma unroll
        for (int i = 0; i < STEPS; ++i) mine += w[i];
        mine = wave_sum(mine);
        if (lane == 0) s_seg[wave] = mine;
    };
    float* const masses = p.chunk_mass + (int64_t)b * p.n_chunks;
    float* const seg_masses = p.seg_mass ? p.seg_mass + (int64_t)b * p.n_chunks * kAccSegs : nullptr;
    float mass = 0.f;
    if (PART != kDraw) {
        segment_mass(chunk);
        const int from = chunk * CHUNK, size = min(p.vocab - from, CHUNK);
#pragma unroll
        for (int i = 0; i < STEPS; ++i) if (lo + 64 * i + lane < hi) s_w[lo - from + 64 * i + lane] = w[i];
        __syncthreads();
        if (tid < COLS) {
            float col[COL_TOKENS], mine = 0.f;
#pragma unroll
            for (int j = 0; j < COL_TOKENS; ++j) col[j] = s_w[min(tid + COLS * j, size - 1)];
#pragma unroll
            for (int j = 0; j < COL_TOKENS; ++j) mine += tid + COLS * j < size ? col[j] : 0.f;
            mine = wave_sum(mine);
            if (lane == 0) s_part[wave] = mine;
        }
        __syncthreads();
        mass = (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);
        if (!SHORT && wave == 0) {
            if (seg_masses && lane < kAccSegs) store_device(seg_masses + (int64_t)chunk * kAccSegs + lane, s_seg[lane]);
            if (lane == 0) store_device(masses + chunk, mass);
            if (PART == kWhole && lane == 0)
                s_last = __hip_atomic_fetch_add(p.arrived + b, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)p.n_chunks - 1u;
        }
        if (PART == kMasses) return;
        if (!SHORT) {
            __syncthreads();
            if (!s_last) return;
        }
    }
    // ---- one workgroup of the request: total mass and the owner of the goal among the chunks: the LAST chunk with mass whose
    // prefix does not exceed the goal -- exactly one chunk, whatever rounding did to the sums (a goal that rounding put at or
    // beyond the total lands on the last chunk with mass).  A lane per chunk, 64 at a time; the prefixes are running sums.
    float W = 0.f, goal = 0.f, pre1 = 0.f, own_seg[kAccSegs];
    int own1 = 0;                                                // (no chunk qualifies for a uniform below 0 or NaN)
    if (wave == 0) {
        float m = 0.f, before = 0.f, seg[kAccSegs];              // the lane's chunk, the sum in front of it, its segments
        auto walk = [&](int c0, float& sum) __attribute__((always_inline)) {
            const int c = min(c0 + lane, p.n_chunks - 1);
            m = SHORT ? mass : load_device(masses + c);
            if (!SHORT && seg_masses) {
#pragma unroll
                for (int i = 0; i < kAccSegs; ++i) seg[i] = load_device(seg_masses + (int64_t)c * kAccSegs + i);
            }
            const int chunks = SHORT ? 1 : min(kWave, p.n_chunks - c0);
            m = lane < chunks ? m : 0.f;
            before = sum;
            for (int i = 0; i < chunks; i += 8) {                // (chunks from `chunks` on add 0)
#pragma unroll
                for (int x = 0; x < 8; ++x) before += lane > i + x ? from_lane(m, i + x) : 0.f;
            }
            sum = from_lane(before + m, chunks - 1);
        };
        for (int c0 = 0; c0 < p.n_chunks; c0 += kWave) walk(c0, W);
        goal = u_last * W;
        float sum = 0.f;
        for (int c0 = 0; c0 < p.n_chunks; c0 += kWave) {
            if (p.n_chunks > kWave) walk(c0, sum);
            const uint64_t fits = __ballot(m > 0.f && before <= goal);
            const int l = fits ? 63 - __builtin_clzll(fits) : 0;
            if (fits) { own1 = c0 + l; pre1 = from_lane(before, l); }
            if (!SHORT && seg_masses && (fits || c0 == 0)) {
#pragma unroll
                for (int i = 0; i < kAccSegs; ++i) own_seg[i] = from_lane(seg[i], l);
            }
        }
        if (lane == 0) { s_mass = W; s_own = own1; }
    }
    __syncthreads();
    W = s_mass;
    int y = -1;
    if (!(W > 0.f)) {
        // no residual mass (p == q): fall back to the target's most likely token
        const int share = ((p.vocab + kAccWaves - 1) / kAccWaves + 63) & ~63;
        const int from = min(p.vocab, wave * share), to = min(p.vocab, from + share);
        float bv = -INFINITY;
        int bi = from + lane < to ? from + lane : -1;
        for (int v = from + lane; v < to; v += 64) {
            const float x = weight.trow[v];
            if (x > bv) { bv = x; bi = v; }                      // (never a NaN, as in accept_argmax_partial)
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const float ov = __shfl_xor(bv, off);
            const int oi = __shfl_xor(bi, off);
            argmax_merge(bv, bi, ov, oi);
        }
        if (lane == 0) { s_top[wave] = bv; s_idx[wave] = bi; }
        __syncthreads();
        if (wave != 0) return;
        for (int x = 1; x < kAccWaves; ++x) argmax_merge(bv, bi, s_top[x], s_idx[x]);
        y = __builtin_amdgcn_readfirstlane(bi);
    } else {
        if (!SHORT && !seg_masses) {                             // (nobody kept the owning chunk's segments)
            segment_mass(s_own);
            __syncthreads();
        }
        if (wave != 0) return;
        if (SHORT || !seg_masses) {
#pragma unroll
            for (int i = 0; i < kAccSegs; ++i) own_seg[i] = s_seg[i];
        }
        // the same rule picks a segment of the owning chunk, whose few hundred tokens are then walked 64 at a time for
        // the first one whose cumulative mass passes the goal, else its last token with mass (rounding can leave no segment
        // that fits although the chunk had mass: the first one then)
        int own2 = 0;
        float pre2 = pre1, acc2 = pre1;
#pragma unroll
        for (int s = 0; s < kAccSegs; ++s) {
            if (own_seg[s] > 0.f && acc2 <= goal) { own2 = s; pre2 = acc2; }
            acc2 += own_seg[s];
        }
        own2 = __builtin_amdgcn_readfirstlane(own2);
        segment(own1, own2, lo, hi);
        weight(w, lo, hi);
        // (the scans of the steps do not depend on each other: six shuffles deep, not six per step)
        float incl[STEPS];
#pragma unroll
        for (int i = 0; i < STEPS; ++i) incl[i] = w[i];
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
#pragma unroll
            for (int i = 0; i < STEPS; ++i) {
                const float t = __shfl_up(incl[i], off);
                if (lane >= off) incl[i] += t;
            }
        }
        float c = pre2;
        int last = -1;
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            const int base = lo + 64 * i;
            const uint64_t massive = __ballot(w[i] > 0.f);
            const uint64_t passed = __ballot(w[i] > 0.f && c + incl[i] > goal);
            if (massive) last = base + 63 - __builtin_clzll(massive);
            if (passed && y < 0) y = base + __ffsll((long long)passed) - 1;
            c += from_lane(incl[i], 63);
        }
        if (y < 0) y = last >= 0 ? last : own1 * CHUNK;
    }
    // (the first wave only from here on)
    for (int i = lane; i <= p.gamma; i += 64)
        p.out_tokens[(int64_t)b * (p.gamma + 1) + i] = i < n ? tok : (i == n ? y : -1);      // (i < n implies i = lane < gamma)
    if (lane == 0) p.n_accepted[b] = n;
}

// ------------------------------------------------------------------ tree ----
// Greedy walk over a static draft tree (App. B): rows of target_logits are tree
// nodes; node 0 is the last committed token, parent[i] < i.  One workgroup per
// request merges the per-chunk argmax partials of all nodes; lane i of its first
// wave holds node i's parent and drafted token, and that wave walks from the root,
// moving to the lowest-numbered child that drafted the target's token (found by a ballot).
template <int LANES>
__global__ __launch_bounds__(final_threads(LANES))
void accept_tree_final(const AcceptParams p, const int32_t* parent, int32_t* accepted_nodes)
{
    const int b = blockIdx.x, lane = threadIdx.x;
    const int n_nodes = p.gamma + 1;                             // <= 64: lane i holds node i
    __shared__ int s_t[64];
    const int32_t* x = p.tokens + (int64_t)b * n_nodes;
    const int my_tok = lane < n_nodes ? x[lane] : -1;            // (in flight while the partials are merged)
    const int my_par = lane < n_nodes ? parent[lane] : -1;       // parent[] is shared by the batch
    accept_merge_argmax<LANES>(p, b, n_nodes, s_t);
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    int32_t* out = p.out_tokens + (int64_t)b * n_nodes;
    int32_t* nodes = accepted_nodes + (int64_t)b * n_nodes;
    // the walk: every lane follows it; the children of the current node that drafted the target's
    // token answer a ballot, the lowest-numbered one is taken (at most n_nodes - 1 steps)
    int cur = 0, n = 0;
    int my_out = -1, my_node = -1;                               // lane i ends up holding out[i] and nodes[i]
    for (;;) {
        const int t = s_t[cur];
        const uint64_t match = __ballot(lane > cur && lane < n_nodes && my_par == cur && my_tok == t);
        if (!match) { if (lane == n) my_out = t; break; }
        const int next = __ffsll((long long)match) - 1;
        const int tok_next = __shfl(my_tok, next);
        if (lane == n) { my_node = next; my_out = tok_next; }
        ++n; cur = next;
    }
    if (lane < n_nodes) { out[lane] = my_out; nodes[lane] = my_node; }
    if (lane == 0) p.n_accepted[b] = n;
}

static int accept_chunks(int vocab) { return (vocab + kAccChunk - 1) / kAccChunk; }

// One launch behind pass 1, or two: a release and an acquire by every workgroup cost more than a launch once there are more
// workgroups than CUs.  Us a call from a graph, rows from HBM, one / two, workgroups in brackets:  152064 tokens, gamma 7, 1
// request [19] 15.0 / 17.0, 8 [152] 27.4 / 28.4, 12 [228] 34.4 / 34.8, 14 [266] 40.2 / 38.8, 16 [304] 43.7 / 41.8;  gamma 3, 64 [1216]
// 96.1 / 70.6;  gamma 1, 128 [2432] 133.5 / 73.3;  32000 tokens, gamma 3, 64 [256] 24.4 / 24.1, 72 [288] 29.1 / 26.3.
static bool accept_one_launch(int batch, int n_chunks) { return (int64_t)batch * n_chunks <= kNumCu; }

// Lanes per row of the greedy final kernels: 16 where that is fewer trips.  The whole call from a graph, us, one lane /
// 16 lanes:  152064 tokens (19 chunks): 6 rows 8.4 / 6.7, 21 rows 9.0 / 8.5, 65 rows 13.4 / 14.4;  65537 (9 chunks): 16 rows
// 7.8 / 7.0, 21 rows 7.8 / 8.0;  32000 (4 chunks): 6 rows 6.7 / 7.0, 21 rows 6.9 / 8.0, 65 rows 7.5 / 10.7.
static int accept_final_lanes(int rows, int n_chunks)
{
    const int rounds = (rows * kFinalLanes + kFinalThreads - 1) / kFinalThreads;
    const int trips = rounds * ((n_chunks + 4 * kFinalLanes - 1) / (4 * kFinalLanes));
    return trips < (n_chunks + 7) / 8 ? kFinalLanes : 1;
}

}  // namespace specvlm

using namespace specvlm;

// Sampling: what a call cannot do without, and what it is asked to bring, with the segments' masses.  (Without them the owning
// chunk's are summed again; the tokens are the same.)
static size_t accept_least_bytes(int batch, int gamma, int vocab, int sampling)
{
    const size_t rows = sampling ? 2 * (size_t)gamma + 1 : (size_t)gamma + 1;
    size_t bytes = 2 * align256((size_t)batch * rows * accept_chunks(vocab) * sizeof(float));
    if (sampling)       // the drafted tokens' logits (room for two of each), chunk masses of the rejected row, arrivals
        bytes += align256((size_t)batch * rows * 2 * sizeof(float)) +
                 align256((size_t)batch * accept_chunks(vocab) * sizeof(float)) +
                 align256((size_t)batch * sizeof(uint32_t));
    return bytes;
}

extern "C" size_t specvlm_accept_workspace_bytes(int batch, int gamma, int vocab, int sampling)
{
    if (batch <= 0 || gamma < 0 || vocab < 1) return 0;
    const size_t segs = sampling ? align256((size_t)batch * accept_chunks(vocab) * kAccSegs * sizeof(float)) : 0;
    return accept_least_bytes(batch, gamma, vocab, sampling) + segs;
}

extern "C" int specvlm_accept(
    const float* target_logits, const float* draft_logits,
    const int32_t* draft_tokens, const float* uniforms,
    int batch, int gamma, int vocab, float temperature,
    int32_t* n_accepted, int32_t* out_tokens,
    void* workspace, size_t workspace_bytes, void* stream)
{
    if (batch < 0 || gamma < 0 || vocab < 1) return SPECVLM_EINVAL;
    const bool sampling = uniforms != nullptr;
    if (!sampling && draft_logits) return SPECVLM_EINVAL;            // draft logits without uniforms
    if (sampling && gamma > 0 && !draft_logits) return SPECVLM_EINVAL;
    if (sampling && !(temperature > 0.f && temperature < INFINITY)) return SPECVLM_EINVAL;
    if (gamma > 64) return SPECVLM_EUNSUPPORTED;
    if (batch == 0) return SPECVLM_OK;
    if (!target_logits || !n_accepted || !out_tokens || (gamma > 0 && !draft_tokens)) return SPECVLM_EINVAL;
    if (batch > 65535) return SPECVLM_EUNSUPPORTED;
    const size_t need = accept_least_bytes(batch, gamma, vocab, sampling);
    if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < need) return SPECVLM_EWORKSPACE;

    AcceptParams p;
    p.target = target_logits; p.draft = draft_logits; p.tokens = draft_tokens; p.uniforms = uniforms;
    p.batch = batch; p.gamma = gamma; p.vocab = vocab; p.n_chunks = accept_chunks(vocab);
    p.inv_t_log2 = sampling ? kLog2e / temperature : kLog2e;
    p.n_accepted = n_accepted; p.out_tokens = out_tokens;
    const size_t rows = sampling ? 2 * (size_t)gamma + 1 : (size_t)gamma + 1;
    const size_t part_bytes = align256((size_t)batch * rows * p.n_chunks * sizeof(float));
    char* ws = (char*)workspace;
    p.part_val = (float*)ws;
    p.part_aux = (float*)(ws + part_bytes);
    p.tok_logit = (float*)(ws + 2 * part_bytes);                 // (sampling only, from here on)
    p.chunk_mass = (float*)((char*)p.tok_logit + align256((size_t)batch * rows * 2 * sizeof(float)));
    p.arrived = (uint32_t*)((char*)p.chunk_mass + align256((size_t)batch * p.n_chunks * sizeof(float)));
    p.seg_mass = workspace_bytes >= specvlm_accept_workspace_bytes(batch, gamma, vocab, sampling) ? (float*)(ws + need) : nullptr;
    hipStream_t s = (hipStream_t)stream;
    if (!sampling) {
        hipLaunchKernelGGL(accept_argmax_partial, dim3(p.n_chunks, gamma + 1, batch), dim3(256), 0, s, p);
        if (accept_final_lanes(gamma + 1, p.n_chunks) == 1)
            hipLaunchKernelGGL(accept_greedy_final<1>, dim3(batch), dim3(kWave), 0, s, p);
        else
            hipLaunchKernelGGL(accept_greedy_final<kFinalLanes>, dim3(batch), dim3(kFinalThreads), 0, s, p);
    } else {
        const dim3 rows_grid(p.n_chunks, 2 * gamma + 1, batch), grid(p.n_chunks, batch);
        if (vocab <= kAccShort) {
            hipLaunchKernelGGL(accept_softmax_partial<kAccShort>, rows_grid, dim3(256), 0, s, p);
            hipLaunchKernelGGL((accept_sample_kernel<kAccShort, kWhole>), grid, dim3(kAccThreads), 0, s, p);
        } else {
            hipLaunchKernelGGL(accept_softmax_partial<kAccChunk>, rows_grid, dim3(256), 0, s, p);
            if (accept_one_launch(batch, p.n_chunks)) {
                hipLaunchKernelGGL((accept_sample_kernel<kAccChunk, kWhole>), grid, dim3(kAccThreads), 0, s, p);
            } else {
                hipLaunchKernelGGL((accept_sample_kernel<kAccChunk, kMasses>), grid, dim3(kAccThreads), 0, s, p);
                hipLaunchKernelGGL((accept_sample_kernel<kAccChunk, kDraw>), dim3(1, batch), dim3(kAccThreads), 0, s, p);
            }
        }
    }
    return launch_status();
}

extern "C" size_t specvlm_accept_tree_workspace_bytes(int batch, int n_nodes, int vocab)
{
    return specvlm_accept_workspace_bytes(batch, n_nodes - 1, vocab, 0);
}

extern "C" int specvlm_accept_tree(
    const float* target_logits, const int32_t* node_tokens, const int32_t* parent,
    int batch, int n_nodes, int vocab,
    int32_t* n_accepted, int32_t* accepted_nodes, int32_t* out_tokens,
    void* workspace, size_t workspace_bytes, void* stream)
{
    if (batch < 0 || n_nodes < 1 || vocab < 1) return SPECVLM_EINVAL;
    if (n_nodes > 64) return SPECVLM_EUNSUPPORTED;
    if (batch == 0) return SPECVLM_OK;
    if (!target_logits || !node_tokens || !parent || !n_accepted || !accepted_nodes || !out_tokens)
        return SPECVLM_EINVAL;
    if (batch > 65535) return SPECVLM_EUNSUPPORTED;
    const size_t need = specvlm_accept_tree_workspace_bytes(batch, n_nodes, vocab);
    if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < need) return SPECVLM_EWORKSPACE;
    AcceptParams p;
    p.target = target_logits; p.draft = nullptr; p.tokens = node_tokens; p.uniforms = nullptr;
    p.batch = batch; p.gamma = n_nodes - 1; p.vocab = vocab; p.n_chunks = accept_chunks(vocab);
    p.inv_t_log2 = kLog2e;
    p.n_accepted = n_accepted; p.out_tokens = out_tokens;
    p.part_val = (float*)workspace;
    p.part_aux = (float*)((char*)workspace + need / 2);
    p.tok_logit = nullptr; p.chunk_mass = nullptr; p.seg_mass = nullptr; p.arrived = nullptr;
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(accept_argmax_partial, dim3(p.n_chunks, n_nodes, batch), dim3(256), 0, s, p);
    if (accept_final_lanes(n_nodes, p.n_chunks) == 1)
        hipLaunchKernelGGL(accept_tree_final<1>, dim3(batch), dim3(kWave), 0, s, p, parent, accepted_nodes);
    else
        hipLaunchKernelGGL(accept_tree_final<kFinalLanes>, dim3(batch), dim3(kFinalThreads), 0, s, p, parent, accepted_nodes);
    return launch_status();
}
