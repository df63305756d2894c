// specvlm_select: the two-stage retention set of Sec. 3.2.
//   Stage I  : V_R = the k highest-scoring video tokens (ties -> lower index),
//              by a most-significant-digit radix select on order-preserving
//              integer keys (digits of 11, 11 and 10 bits, histograms in LDS).
//   Stage II : V_U = tokens of V \ V_R at the fixed fractional interval
//              I = R/U in raster order: remainder ranks floor(t*R/U), exact
//              integer arithmetic (Eq. 7 with the budget as denominator).
//   Output   : sort(V_R u V_U) by a stable compaction.
// One workgroup of 1024 threads per request; thread t owns the contiguous run
// of tokens [t*per, (t+1)*per) and keeps their keys in registers, so every
// "how many before me" question is one block-wide exclusive scan of popcounts.
//
// Bound: latency and VALU issue of the one workgroup.  Sixteen waves share four SIMDs, so an instruction that all of
// them execute takes about 20 cycles; a barrier 100, and a wave scan by __shfl six LDS round trips (600).  Hence the
// scans by DPP, no test on a key that its position or the pass already decides, masks of 32 bits where a thread has at
// most 32 keys, and few, wide digits.
#include <type_traits>

#include "common.h"

namespace specvlm {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / kWave;
// The key is read in digits of 11, 11 and 10 bits, each with a histogram of its own, cleared while the scores are on their way.
// With four digits of 8 bits 24 bits took three passes and scores that share their upper bits the fourth; two passes of 11
// usually decide, the third ends it: 12544 tokens, a tenth kept, half of it by score, us in a graph, 8 bits / now: long-tailed
// 10.5 / 9.6, within 1e-3 11.8 / 10.4, within 1e-5 12.4 / 11.0, all equal 13.8 / 13.4; 32768 tokens 19.3 / 17.8, 22.2 / 18.7,
// 24.0 / 20.3, 28.2 / 27.7; 1568 tokens 5.76 / 5.55 and 6.33 / 6.13.  10 and 12 bits in front: 9.7 and 10.7 for the first two.
// Copies of a histogram, summed after its pass by all waves: an LDS atomic serialises over the lanes that hit one address, and
// digits do coincide (the leading one takes a handful of values), but every copy is also cleared and summed.  12544 tokens,
// long-tailed / within 1e-5 / all equal, by the copies of the three digits:  4, 4, 1: 10.6 / 12.5 / 23.8;  4, 4, 4: 10.6 / 12.4 /
// 16.0;  8, 8, 4: 9.7 / 11.1 / 13.6.  With up to 4 tokens a thread four are enough (1568 tokens 5.55 / 6.28 / 6.79; eight 5.74 /
// 6.43 / 6.75; two 5.68 / 6.48 / 7.66); with more than 32 the last digit, where equal scores meet, takes sixteen, in the
// place of the first one's (65536 tokens, all equal: 43.9, with four 53.7, before 45.2).
constexpr int kSelBits[3] = {11, 11, 10}, kSelShift[3] = {21, 10, 0};
// PAIR: two workgroups share a CU's LDS (see select_pairs), where three histograms of eight copies leave room for one.  With up to 4
// tokens a thread the last digit takes the first one's place; with more all three take one place in turn, cleared between them,
// which costs less than copies do:  four copies in two places were 15.9 us for 257 requests of 12544 tokens, eight in one 14.6.
template <int E, bool PAIR> struct SelHist {
    static constexpr int copies(int pass) { return E <= 4 ? 4 : pass < 2 ? 8 : E <= 32 ? 4 : 16; }
    static constexpr int stride(int pass) { return (1 << kSelBits[pass]) + (pass < 2 ? 4 : 2); }   // (copies of a digit lie in different banks)
    static constexpr int words(int pass) { return copies(pass) * stride(pass); }
    static constexpr bool kSingle = PAIR && E > 4;               // every pass takes the same place
    static constexpr bool kReuse = !kSingle && (E > 32 || PAIR); // the last pass takes the first one's place
    static constexpr int at(int pass) { return kSingle || pass == 0 || (pass == 2 && kReuse) ? 0 : at(pass - 1) + words(pass - 1); }
    static constexpr int kWords = kSingle ? words(0) : words(0) + words(1) + (kReuse ? 0 : words(2));
    static_assert(words(1) <= words(0));
    static_assert(!kReuse || words(2) <= words(0));
};

// Wave-wide inclusive prefix sum by DPP: rows of 16 lanes, then the rows' totals.
template <int CTRL, int ROWS> __device__ __forceinline__ int dpp_or_0(int x)
{
    return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xf, false);
}

__device__ __forceinline__ int row_incl_scan(int x)
{
    x += dpp_or_0<0x111, 0xf>(x);         // row_shr 1, 2, 4, 8
    x += dpp_or_0<0x112, 0xf>(x);
    x += dpp_or_0<0x114, 0xf>(x);
    return x + dpp_or_0<0x118, 0xf>(x);
}

__device__ __forceinline__ int wave_incl_scan(int x)
{
    x = row_incl_scan(x);
    x += dpp_or_0<0x142, 0xa>(x);         // row_bcast 15, into rows 1 and 3
    return x + dpp_or_0<0x143, 0xc>(x);   // row_bcast 31, into rows 2 and 3
}

template <int CTRL, int ROWS> __device__ __forceinline__ unsigned long long dpp_or_0(unsigned long long x)
{
    const unsigned lo = (unsigned)dpp_or_0<CTRL, ROWS>((int)(unsigned)x), hi = (unsigned)dpp_or_0<CTRL, ROWS>((int)(x >> 32));
    return ((unsigned long long)hi << 32) | lo;
}

__device__ __forceinline__ unsigned long long wave_incl_scan(unsigned long long x)
{
    x += dpp_or_0<0x111, 0xf>(x);
    x += dpp_or_0<0x112, 0xf>(x);
    x += dpp_or_0<0x114, 0xf>(x);
    x += dpp_or_0<0x118, 0xf>(x);
    x += dpp_or_0<0x142, 0xa>(x);
    return x + dpp_or_0<0x143, 0xc>(x);
}

__device__ __forceinline__ int count_bits(uint32_t m) { return __popc(m); }
__device__ __forceinline__ int count_bits(uint64_t m) { return __popcll(m); }
__device__ __forceinline__ int first_bit(uint32_t m) { return __ffs((int)m) - 1; }
__device__ __forceinline__ int first_bit(uint64_t m) { return __ffsll((long long)m) - 1; }

struct SelectParams {
    const float* scores;
    const int32_t* cu_video;
    const int32_t* k_top;
    const int32_t* keep_budget;
    const int32_t* cu_keep;
    int max_n_video;
    int32_t* keep_idx;
    uint8_t* from_topk;
    int32_t* status;
};

// Order-preserving key: larger score <=> larger key.  -0.0 is +0.0; NaN is the
// smallest key of all, and so is a slot without a token.  (Without branches: with the test around the
// conversion every key had two of its own.)
__device__ __forceinline__ uint32_t score_key(float x, bool token = true)
{
    const uint32_t u = __float_as_uint(x + 0.f);                 // (-0 + 0 is +0)
    const uint32_t key = u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
    return ((x == x) & token) ? key : 0u;
}

// A thread's run of scores [first, first + per) of a request of n scores, four at a time (dword-aligned
// 16-byte loads); slots past the run or past n read as 0.  With one score per load every instruction
// would touch 64 different cache lines, and the address path takes a cycle per line: 13 such loads per
// thread were the longest phase of the select kernel.
template <int E>
__device__ __forceinline__ void load_run(const float* sc, int first, int per, int n, float (&raw)[E])
{
    typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
    for (int e4 = 0; e4 < E; e4 += 4) {
        const int idx = first + e4;
        if (e4 + 3 < per && idx + 3 < n) {
            const float4u v = *reinterpret_cast<const float4u*>(sc + idx);
#pragma unroll
            for (int i = 0; i < 4; ++i) raw[e4 + i] = v[i];
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) raw[e4 + i] = (e4 + i < per && idx + i < n) ? sc[idx + i] : 0.f;
        }
    }
}

// Exclusive prefix sums of two counts per thread (at most 64 each: a wave's sums fit 16 bits) behind one barrier.
__device__ __forceinline__ void block_excl_scan2(int a, int b, int* s_wave, int* a_before, int* b_before)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mine = a | (b << 16);
    const int incl = wave_incl_scan(mine);
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    const int w = lane < kSelWaves ? s_wave[lane] : 0;
    const int wa = row_incl_scan(w & 0xffff) - (w & 0xffff), wb = row_incl_scan(w >> 16) - (w >> 16);
    const int excl = incl - mine;
    *a_before = __builtin_amdgcn_readlane(wa, wave) + (excl & 0xffff);
    *b_before = __builtin_amdgcn_readlane(wb, wave) + (excl >> 16);
}

template <int E, bool PAIR>
__global__ __launch_bounds__(kSelThreads)
void select_kernel(const SelectParams p)
{
    using mask_t = std::conditional_t<(E <= 32), uint32_t, uint64_t>;      // a bit per key of a thread
    static_assert(kSelWaves == 16, "the waves' sums are one DPP row");
    using H = SelHist<E, PAIR>;
    __shared__ __align__(16) int s_hist[H::kWords];         // a histogram for each digit
    __shared__ int s_wave[kSelWaves];
    __shared__ int s_pick[3];

    const int b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int v0 = p.cu_video ? p.cu_video[b] : 0;
    const int n = p.cu_video ? p.cu_video[b + 1] - v0 : p.max_n_video;
    // The scores are requested first (guarded by the token count alone, so always in bounds); the
    // request's sizes, one more memory round trip away, are fetched while those loads are in flight.
    const int per = n > 0 ? (n + kSelThreads - 1) / kSelThreads : 0;
    const int first = tid * per;
    const float* sc = p.scores + v0;
    float raw[E];
    load_run<E>(sc, first, per, n, raw);
    // the histograms are cleared while the scores are on their way
    auto clear = [&](int words) __attribute__((always_inline)) {
        for (int i = tid; i < words / 4; i += kSelThreads) reinterpret_cast<u32x4*>(s_hist)[i] = u32x4{0u, 0u, 0u, 0u};
    };
    clear(H::kWords);
    const int k = p.k_top[b], budget = p.keep_budget[b];
    const int out0 = p.cu_keep ? p.cu_keep[b] : 0;
    const bool bad = n < 0 || n > E * kSelThreads || n > p.max_n_video || k < 0 || k > budget || budget > n;
    if (p.status && tid == 0) p.status[b] = bad ? SPECVLM_EINVAL : SPECVLM_OK;
    if (bad || budget == 0) return;

    // Slots past the last token hold the smallest key.  They come after every token of equal key, and never more keys
    // are taken than there are tokens, so they need no test: none of them is ever among the first `need` equal keys.
    const int mine = first < n ? min(per, n - first) : 0;
    uint32_t key[E];
#pragma unroll
    for (int e = 0; e < E; ++e) key[e] = score_key(raw[e], e < mine);

    // ---- Stage I: radix select of the k-th largest key ----
    uint32_t prefix = 0, known = 0;
    int need = k;                       // how many still to take inside the current prefix
    // One digit: its histogram, and the digit of the k-th key.  False when the rest of the key decides nothing.
    auto digit = [&](auto pass_) __attribute__((always_inline)) {
        constexpr int PASS = decltype(pass_)::value;
        constexpr int SHIFT = kSelShift[PASS], BITS = kSelBits[PASS], BINS = 1 << BITS, COPIES = H::copies(PASS);
        constexpr int PER = BINS / kSelThreads, STRIDE = H::stride(PASS);
        int* const hist = s_hist + H::at(PASS);
        // (every thread has read the histogram of the digit before, in front of the last barrier)
        if (PASS > 0 && H::kSingle) { clear(H::words(PASS)); __syncthreads(); }
        // A lane may add to any copy: the lanes of an instruction are spread over the copies, the waves start at
        // different ones.  No aggregation over the wave or over a thread's keys: both were measured and cost more
        // than the additions they save.
        int* const my_hist = hist + ((4 * wave + lane) & (COPIES - 1)) * STRIDE;
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (e < per && (PASS == 0 || (key[e] & known) == prefix)) atomicAdd(&my_hist[(key[e] >> SHIFT) & (BINS - 1)], 1);
        // (the first histogram was read for the last time before the barrier above)
        if (PASS == 1 && H::kReuse) clear(H::words(2));
        __syncthreads();
        // thread t sums PER digits from the top over the copies; prefix sums over the threads run down from the top digit
        const int d0 = BINS - PER - PER * tid;
        int c[PER] = {};
#pragma unroll
        for (int w = 0; w < COPIES; ++w)
#pragma unroll
            for (int i = 0; i < PER; ++i) c[i] += hist[w * STRIDE + d0 + i];
        int sum = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) sum += c[i];
        const int incl = wave_incl_scan(sum);
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        const int total = lane < kSelWaves ? s_wave[lane] : 0;
        int above = __builtin_amdgcn_readlane(row_incl_scan(total) - total, __builtin_amdgcn_readfirstlane(wave)) + incl - sum;   // keys in higher digits
        if (above < need && need <= above + sum) {
#pragma unroll
            for (int i = PER - 1; i >= 0; --i) {
                if (above < need && need <= above + c[i]) {
                    s_pick[0] = d0 + i;
                    s_pick[1] = need - above;
                    s_pick[2] = (need - above == c[i]);     // the whole bucket is taken: nothing left to rank
                }
                above += c[i];
            }
        }
        __syncthreads();
        prefix |= (uint32_t)s_pick[0] << SHIFT;
        known |= (uint32_t)(BINS - 1) << SHIFT;
        need = s_pick[1];
        // When the keys that share the digits known so far are exactly as many as are still needed,
        // all of them are taken and the lower digits decide nothing: the remaining passes are skipped.
        return s_pick[2] == 0;
    };
    if (k > 0) {
        __syncthreads();                                // the cleared histograms are visible
        if (digit(std::integral_constant<int, 0>{}) && digit(std::integral_constant<int, 1>{})) digit(std::integral_constant<int, 2>{});
    }
    // now: prefix = the known digits of the k-th largest key (all of them, or fewer when a whole bucket
    // is taken); take every key above it and the first `need` keys that share it, in index order.
    mask_t gt = 0, eq = 0;
    if (k > 0) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (e >= per) continue;
            const uint32_t kk = key[e] & known;
            gt |= kk > prefix ? (mask_t)1 << e : 0;
            eq |= kk == prefix ? (mask_t)1 << e : 0;
        }
    }
    // One block scan gives every thread the numbers of larger and of equal keys before its
    // tokens; everything else that is "before me" follows in closed form: the tokens before mine
    // are min(first, n), those taken by Stage I are the larger ones plus the equal ones up to
    // `need`, the rest is my first remainder rank, and the stride picks below that rank are counted
    // by the stride formula itself.
    int gt_before, eq_before;
    block_excl_scan2(count_bits(gt), count_bits(eq), s_wave, &gt_before, &eq_before);
    int take = need - eq_before;
    const int top_before = gt_before + (eq_before < need ? eq_before : need);
    mask_t top = gt;
    for (mask_t m = eq; m && take > 0; --take) {
        const mask_t bit = m & (~m + 1);
        top |= bit;
        m ^= bit;
    }

    // ---- Stage II: uniform stride over the remainder ----
    const mask_t valid = mine > 0 ? (mask_t)(~(mask_t)0 >> (sizeof(mask_t) * 8 - mine)) : 0;
    const mask_t rem_mask = valid & ~top;
    const uint32_t rho_before = (uint32_t)((first < n ? first : n) - top_before);
    // Stride picks are the ranks floor(t*R/U), t < U.  t(rho) = ceil(rho*U/R) of them lie below rank rho, and with
    // slack(rho) = t(rho)*R - rho*U (in [0, R), at least U where t(rho) = U) rank rho is a pick exactly if slack < U;
    // then slack moves by R - U, else by -U.  n <= 65536: for rho < R, rho*U + R - 1 <= (R-1)*(R+1) < 2^32.
    const uint32_t R = (uint32_t)(n - k), U = (uint32_t)(budget - k);
    mask_t uni = 0;
    uint32_t uni_before = U;                                      // stride picks with a rank below mine
    if (U > 0 && rho_before < R) {
        uni_before = (rho_before * U + R - 1) / R;
        uint32_t slack = uni_before * R - rho_before * U;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (e >= per) continue;
            if ((rem_mask >> e) & 1) {
                const bool pick = slack < U;
                uni |= pick ? (mask_t)1 << e : 0;
                slack += pick ? R - U : 0u - U;
            }
        }
    }

    // ---- stable compaction of V_R u V_U: my first output position is what was kept before me ----
    const mask_t keep = top | uni;
    int pos = out0 + top_before + (int)uni_before;
    for (mask_t m = keep; m;) {
        const int e = first_bit(m);
        m &= m - 1;
        p.keep_idx[pos] = first + e;
        if (p.from_topk) p.from_topk[pos] = (uint8_t)((top >> e) & 1);
        ++pos;
    }
}


// ---------------------------------------------------------------------------
// Stage I's own size rule (Sec. 3.2, Eq. 6): the smallest c such that the c
// largest scores reach lambda of the total score mass.  A radix descent as the
// selection's, in four digits of 8 bits, whose histograms carry the MASS of the keys, not
// their number (the first pass's sums also give the total); the numbers of keys
// above and at the threshold are counted once, at the end.
// Sums are 64-bit fixed point (score * 2^40 / max score): integer adds commute,
// so the result does not depend on the order in which lanes reach the atomics.
// Scores are attention masses: a value that is not a finite positive number
// counts as 0 (and keeps its place in the descending order).
struct TopPParams {
    const float* scores;
    const int32_t* cu_video;
    int max_n_video;
    float lambda;
    const int32_t* max_count;
    int32_t* count;
};

constexpr int kTopPCopies = 8;
constexpr int kTopPCopyWords = 258;       // 256 sums, 16-byte aligned; the copies of one digit lie in different banks

template <int E>
__global__ __launch_bounds__(kSelThreads)
void top_p_kernel(const TopPParams p)
{
    // copies of the 256 per-digit mass sums, two sets in turn; counts are not kept per digit: only the
    // threshold key's are needed, at the end
    __shared__ __align__(16) unsigned long long s_mass[2][kTopPCopies * kTopPCopyWords];
    __shared__ float s_redf[kSelWaves];
    __shared__ int s_redc[2][kSelWaves];
    __shared__ unsigned long long s_pick_sum, s_goal;
    __shared__ int s_pick;

    const int b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int v0 = p.cu_video ? p.cu_video[b] : 0;
    const int n = p.cu_video ? p.cu_video[b + 1] - v0 : p.max_n_video;
    if (n <= 0 || n > E * kSelThreads) { if (tid == 0) p.count[b] = 0; return; }
    const int per = (n + kSelThreads - 1) / kSelThreads;
    const int first = tid * per;
    const float* sc = p.scores + v0;

    // a value that is not a finite positive number carries no mass; its key still ranks it
    auto mass_of = [](float x) { return (x > 0.f && x < INFINITY) ? x : 0.f; };
    float val[E];
    load_run<E>(sc, first, per, n, val);
    // the sums are cleared while the scores are on their way
    auto clear = [&](unsigned long long* from, int words) __attribute__((always_inline)) {
        for (int i = tid; i < words / 2; i += kSelThreads) reinterpret_cast<u32x4*>(from)[i] = u32x4{0u, 0u, 0u, 0u};
    };
    clear(s_mass[0], 2 * kTopPCopies * kTopPCopyWords);
    // (slots past the last token hold a NaN: the lowest key, without mass, so they need no test)
    const int mine = first < n ? min(per, n - first) : 0;
    float mx = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (e >= mine) val[e] = NAN;
        mx = fmaxf(mx, mass_of(val[e]));
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    if (lane == 0) s_redf[wave] = mx;
    __syncthreads();                                    // (also: the cleared sums are visible)
    mx = 0.f;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) mx = fmaxf(mx, s_redf[w]);
    if (!(mx > 0.f)) { if (tid == 0) p.count[b] = 0; return; }

    // fixed point by an exact power-of-two scaling: the largest score lands in [2^39, 2^40)
    int mx_exp;
    (void)frexpf(mx, &mx_exp);
    const int fix_shift = 40 - mx_exp;
    auto to_fix = [&](float x) { return (unsigned long long)ldexpf(mass_of(x), fix_shift); };

    uint32_t prefix = 0, known = 0;
    unsigned long long above_sum = 0;          // mass of the keys known to rank above the threshold
    unsigned long long goal = 0;               // ceil(lambda * total), known once the first pass has the total
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        unsigned long long* const mass = s_mass[pass & 1];
        unsigned long long* const my_mass = mass + ((4 * wave + lane) & (kTopPCopies - 1)) * kTopPCopyWords;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (e >= per) continue;
            float x = val[e];
            __asm__ volatile("" : "+v"(x));          // recompute key and mass per pass: keeps them out of registers
            const uint32_t key = score_key(x);
            if ((key & known) == prefix) {
                const unsigned long long m = to_fix(x);
                if (m) atomicAdd(&my_mass[(key >> shift) & 255], m);
            }
        }
        // (the other set was read for the last time before the barrier above)
        if (pass == 1 || pass == 2) clear(s_mass[(pass + 1) & 1], kTopPCopies * kTopPCopyWords);
        __syncthreads();
        if (wave == 0) {
            // lane l sums digits 252 - 4l .. 255 - 4l over the copies; prefix sums run down from the top digit
            const int d0 = 252 - 4 * lane;
            unsigned long long m4[4] = {0ull, 0ull, 0ull, 0ull};
#pragma unroll
            for (int w = 0; w < kTopPCopies; ++w) {
                typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
                const u64x2* src = reinterpret_cast<const u64x2*>(mass + w * kTopPCopyWords + d0);
                const u64x2 v0 = src[0], v1 = src[1];
                m4[0] += v0[0]; m4[1] += v0[1]; m4[2] += v1[0]; m4[3] += v1[1];
            }
            const unsigned long long mmine = m4[0] + m4[1] + m4[2] + m4[3];
            const unsigned long long mincl = wave_incl_scan(mmine);
            if (pass == 0) {
                // the first pass sees every key: the last lane's sum is the total mass.
                // goal = ceil(lambda * total); lambda is an fp32 in [0,1] and total < 2^56, so the double
                // product is within a few units of 2^-40 of the largest score: far below the parity margin
                const unsigned long long total = __shfl(mincl, 63);
                const double goal_d = ceil((double)p.lambda * (double)total);
                goal = goal_d <= 0.0 ? 0ull : (unsigned long long)goal_d;
                if (goal > total) goal = total;
                if (lane == 0) s_goal = goal;
            }
            // the threshold digit: first digit from the top where the running mass reaches the goal
            unsigned long long m_above = above_sum + (mincl - mmine);
            if (goal > 0 && m_above < goal && goal <= above_sum + mincl) {
#pragma unroll
                for (int i = 3; i >= 0; --i) {
                    if (m_above < goal && goal <= m_above + m4[i]) { s_pick = d0 + i; s_pick_sum = m_above; }
                    m_above += m4[i];
                }
            }
        }
        __syncthreads();
        if (pass == 0) {
            goal = s_goal;
            if (goal == 0) { if (tid == 0) p.count[b] = 0; return; }
        }
        prefix |= (uint32_t)s_pick << shift;
        known |= 255u << shift;
        above_sum = s_pick_sum;
    }
    // prefix is now the threshold key: count the keys above it and those equal to it
    int gt = 0, eq = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const uint32_t key = score_key(val[e]);
        if (e < per) { gt += key > prefix; eq += key == prefix; }      // (prefix has mass, so no NaN equals it)
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) { gt += __shfl_xor(gt, off); eq += __shfl_xor(eq, off); }
    if (lane == 0) { s_redc[0][wave] = gt; s_redc[1][wave] = eq; }
    __syncthreads();
    if (tid == 0) {
        int above_cnt = 0, eq_cnt = 0;
#pragma unroll
        for (int w = 0; w < kSelWaves; ++w) { above_cnt += s_redc[0][w]; eq_cnt += s_redc[1][w]; }
        // every key equal to the threshold carries the same mass: take as many as the goal needs
        const uint32_t u = (prefix & 0x80000000u) ? (prefix & 0x7fffffffu) : ~prefix;
        const float tval = __uint_as_float(u);
        const unsigned long long each = to_fix(tval);
        const unsigned long long need = goal - above_sum;
        long long take = each > 0 ? (long long)((need + each - 1) / each) : eq_cnt;
        if (take > eq_cnt) take = eq_cnt;
        if (take < 1) take = 1;
        int c = above_cnt + (int)take;
        if (p.max_count && c > p.max_count[b]) c = p.max_count[b];
        p.count[b] = c;
    }
}

// From one request per CU on two share one.  Us a call from a graph, a twentieth kept by score and as many by stride, one to a CU /
// two:  257 requests of 1568 tokens 9.3 / 7.4, of 12544 17.5 / 14.6, of 32768 36.9 / 36.6;  512 of 4096 12.0 / 9.5, of 12544 20.9 /
// 17.6;  1024 of 1568 18.9 / 13.7, of 12544 41.5 / 32.9.  (More than 32 tokens a thread take too many registers for two.)
static bool select_pairs(int batch) { return batch > kNumCu; }

template <int E>
static void launch_select(const SelectParams& p, int batch, bool pair, hipStream_t s)
{
    if (pair) hipLaunchKernelGGL((select_kernel<E, true>), dim3(batch), dim3(kSelThreads), 0, s, p);
    else      hipLaunchKernelGGL((select_kernel<E, false>), dim3(batch), dim3(kSelThreads), 0, s, p);
}

}  // namespace specvlm

using namespace specvlm;

extern "C" size_t specvlm_select_workspace_bytes(int batch, int max_n_video)
{
    (void)batch; (void)max_n_video;
    return 0;                           // everything lives in registers and LDS
}

extern "C" int specvlm_select(
    const float* scores, const int32_t* cu_video,
    const int32_t* k_top, const int32_t* keep_budget, const int32_t* cu_keep,
    int batch, int max_n_video, int total_keep,
    int32_t* keep_idx, uint8_t* from_topk, int32_t* status,
    void* workspace, size_t workspace_bytes, void* stream)
{
    (void)workspace; (void)workspace_bytes;
    if (batch < 0 || max_n_video < 0 || total_keep < 0) return SPECVLM_EINVAL;
    if (batch == 0) return SPECVLM_OK;
    if (!k_top || !keep_budget) return SPECVLM_EINVAL;
    if (batch > 1 && (!cu_video || !cu_keep)) return SPECVLM_EINVAL;
    if ((int64_t)total_keep > (int64_t)batch * max_n_video) return SPECVLM_EINVAL;
    if (max_n_video > 64 * kSelThreads) return SPECVLM_EUNSUPPORTED;
    if (max_n_video == 0 || total_keep == 0) {
        // nothing can be kept; still report per-request status
        if (!status) return SPECVLM_OK;
    }
    if (total_keep > 0 && (!scores || !keep_idx)) return SPECVLM_EINVAL;

    SelectParams p;
    p.scores = scores; p.cu_video = cu_video; p.k_top = k_top; p.keep_budget = keep_budget;
    p.cu_keep = cu_keep; p.max_n_video = max_n_video;
    p.keep_idx = keep_idx; p.from_topk = from_topk; p.status = status;
    hipStream_t s = (hipStream_t)stream;
    const int per = (max_n_video + kSelThreads - 1) / kSelThreads;
    const bool pair = select_pairs(batch);
    if (per <= 4)       launch_select<4>(p, batch, pair, s);
    else if (per <= 16) launch_select<16>(p, batch, pair, s);
    else if (per <= 32) launch_select<32>(p, batch, pair, s);
    else                hipLaunchKernelGGL((select_kernel<64, false>), dim3(batch), dim3(kSelThreads), 0, s, p);
    return launch_status();
}

extern "C" size_t specvlm_top_p_count_workspace_bytes(int batch, int max_n_video)
{
    (void)batch; (void)max_n_video;
    return 0;
}

extern "C" int specvlm_top_p_count(
    const float* scores, const int32_t* cu_video, int batch, int max_n_video,
    float lambda, const int32_t* max_count, int32_t* count,
    void* workspace, size_t workspace_bytes, void* stream)
{
    (void)workspace; (void)workspace_bytes;
    if (batch < 0 || max_n_video < 0) return SPECVLM_EINVAL;
    if (!(lambda >= 0.f && lambda <= 1.f)) return SPECVLM_EINVAL;
    if (batch == 0) return SPECVLM_OK;
    if (!count || (max_n_video > 0 && !scores)) return SPECVLM_EINVAL;
    if (batch > 1 && !cu_video) return SPECVLM_EINVAL;
    if (max_n_video > 64 * kSelThreads) return SPECVLM_EUNSUPPORTED;
    TopPParams p;
    p.scores = scores; p.cu_video = cu_video; p.max_n_video = max_n_video;
    p.lambda = lambda; p.max_count = max_count; p.count = count;
    hipStream_t s = (hipStream_t)stream;
    const int per = (max_n_video + kSelThreads - 1) / kSelThreads;
    if (per <= 4)       hipLaunchKernelGGL(top_p_kernel<4>, dim3(batch), dim3(kSelThreads), 0, s, p);
    else if (per <= 16) hipLaunchKernelGGL(top_p_kernel<16>, dim3(batch), dim3(kSelThreads), 0, s, p);
    else if (per <= 32) hipLaunchKernelGGL(top_p_kernel<32>, dim3(batch), dim3(kSelThreads), 0, s, p);
    else                hipLaunchKernelGGL(top_p_kernel<64>, dim3(batch), dim3(kSelThreads), 0, s, p);
    return launch_status();
}
