// specvlm_select: the two-stage retention set of Sec. 3.2.
//   Stage I  : V_R = the k highest-scoring video tokens (ties -> lower index),
//              by a most-significant-digit radix select on order-preserving
//              integer keys (4 passes of 8 bits, histograms in LDS).
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
// most 32 keys, and one wave that sums and scans a pass's histograms between two barriers.
#include <type_traits>

#include "common.h"

namespace specvlm {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / kWave;
// Copies of the digit histogram, summed after a pass by one wave.  An LDS atomic serialises over the lanes that hit one
// address, and digits do coincide (the leading one, sign and exponent, takes a handful of values; scores summed over many
// rows share their upper 16 bits), but every copy is also cleared, summed and moves the pass's end: cycles of the select
// kernel at 12544 tokens, long-tailed / clustered within 1e-3 / within 1e-5, by the copies of passes 1 to 3:  2: 20.0 /
// 26.1 / 31.7 thousand, 4: 19.8 / 22.7 / 25.5, 8: 20.3 / 21.4 / 22.2, 16: 25.3, 32: 28.7; 16 or 64 in pass 0 are equal.
// More keys to a thread mean more additions to every sum: the selection with 33 to 64 of them takes sixteen copies
// (65536 tokens, a twentieth kept, us with 8 / 16, the 64 copies of before in brackets: long-tailed 31.7 / 30.9 [38.5], within
// 1e-5 46.0 / 41.2 [45.3], all equal 55.1 / 44.8 [46.5]).  With 17 to 32 the eight stay the better ones wherever scores differ
// (32768 tokens: long-tailed 17.6 / 18.7 [24.6], within 1e-5 23.7 / 22.7 [26.2]); only where nearly all are equal they are not
// (28.0 / 23.4 [25.9]).  Copies chosen pass by pass, by the keys still in play, cost more than they save (19.2 and 25.1).
constexpr int kSelCopies = 8;
constexpr int kSelCopyWords = 260;        // 256 counters, 16-byte aligned; the copies of one digit lie in different banks

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
// smallest key of all.
__device__ __forceinline__ uint32_t score_key(float x)
{
    const uint32_t u = __float_as_uint(x + 0.f);                 // (-0 + 0 is +0)
    const uint32_t key = u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
    return x != x ? 0u : key;
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

template <int E>
__global__ __launch_bounds__(kSelThreads)
void select_kernel(const SelectParams p)
{
    constexpr int COPIES = E <= 32 ? kSelCopies : 2 * kSelCopies;
    using mask_t = std::conditional_t<(E <= 32), uint32_t, uint64_t>;      // a bit per key of a thread
    static_assert(kSelWaves == 16, "the waves' sums are one DPP row");
    __shared__ __align__(16) int s_hist[2][COPIES * kSelCopyWords];    // the passes alternate between two sets
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
    // the first two passes' histograms are cleared while the scores are on their way
    auto clear = [&](int* from, int words) __attribute__((always_inline)) {
        for (int i = tid; i < words / 4; i += kSelThreads) reinterpret_cast<u32x4*>(from)[i] = u32x4{0u, 0u, 0u, 0u};
    };
    clear(s_hist[0], 2 * COPIES * kSelCopyWords);
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
    for (int e = 0; e < E; ++e) key[e] = e < mine ? score_key(raw[e]) : 0u;

    // ---- Stage I: radix select of the k-th largest key ----
    uint32_t prefix = 0, known = 0;
    int need = k;                       // how many still to take inside the current prefix
    if (k > 0) {
        __syncthreads();                                // the cleared histograms are visible
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 24 - 8 * pass;
            int* const hist = s_hist[pass & 1];
            // A lane may add to any copy: the lanes of an instruction are spread over the copies, the waves start at
            // different ones.  No aggregation over the wave or over a thread's keys: both were measured and cost more
            // than the additions they save.
            int* const my_hist = hist + ((4 * wave + lane) & (COPIES - 1)) * kSelCopyWords;
            if (pass == 0) {
#pragma unroll
                for (int e = 0; e < E; ++e)
                    if (e < per) atomicAdd(&my_hist[key[e] >> 24], 1);
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e)
                    if (e < per && (key[e] & known) == prefix) atomicAdd(&my_hist[(key[e] >> shift) & 255], 1);
                // (the other set was read for the last time before the barrier above)
                if (pass < 3) clear(s_hist[(pass + 1) & 1], COPIES * kSelCopyWords);
            }
            __syncthreads();
            if (wave == 0) {
                // lane l sums digits 252 - 4l .. 255 - 4l over the copies; prefix sums over the lanes run down from the
                // top digit
                const int d0 = 252 - 4 * lane;
                int c4[4] = {0, 0, 0, 0};
#pragma unroll
                for (int w = 0; w < COPIES; ++w) {
                    const u32x4 v = *reinterpret_cast<const u32x4*>(hist + w * kSelCopyWords + d0);
#pragma unroll
                    for (int i = 0; i < 4; ++i) c4[i] += (int)v[i];
                }
                const int sum = c4[0] + c4[1] + c4[2] + c4[3];
                const int incl = wave_incl_scan(sum);
                int above = incl - sum;                 // keys in higher digits
                if (above < need && need <= incl) {
#pragma unroll
                    for (int i = 3; i >= 0; --i) {
                        if (above < need && need <= above + c4[i]) {
                            s_pick[0] = d0 + i;
                            s_pick[1] = need - above;
                            s_pick[2] = (need - above == c4[i]);    // the whole bucket is taken: nothing left to rank
                        }
                        above += c4[i];
                    }
                }
            }
            __syncthreads();
            prefix |= (uint32_t)s_pick[0] << shift;
            known |= 255u << shift;
            need = s_pick[1];
            // When the keys that share the digits known so far are exactly as many as are still needed,
            // all of them are taken and the lower digits decide nothing: the remaining passes are skipped
            // (with distinct scores this is the usual case after three passes).
            if (s_pick[2]) break;
        }
    }
    // now: prefix = the known digits of the k-th largest key (all four, or fewer when a whole bucket
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
// largest scores reach lambda of the total score mass.  Same radix descent as
// the selection, but the per-digit histograms carry the MASS of the keys, not
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

constexpr int kTopPCopyWords = 258;       // 256 sums, 16-byte aligned; the copies of one digit lie in different banks

template <int E>
__global__ __launch_bounds__(kSelThreads)
void top_p_kernel(const TopPParams p)
{
    // copies of the 256 per-digit mass sums, two sets as in the selection; counts are not kept per digit: only the
    // threshold key's are needed, at the end
    __shared__ __align__(16) unsigned long long s_mass[2][kSelCopies * kTopPCopyWords];
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
    clear(s_mass[0], 2 * kSelCopies * kTopPCopyWords);
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
        unsigned long long* const my_mass = mass + ((4 * wave + lane) & (kSelCopies - 1)) * kTopPCopyWords;
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
        if (pass == 1 || pass == 2) clear(s_mass[(pass + 1) & 1], kSelCopies * kTopPCopyWords);
        __syncthreads();
        if (wave == 0) {
            // lane l sums digits 252 - 4l .. 255 - 4l over the copies; prefix sums run down from the top digit
            const int d0 = 252 - 4 * lane;
            unsigned long long m4[4] = {0ull, 0ull, 0ull, 0ull};
#pragma unroll
            for (int w = 0; w < kSelCopies; ++w) {
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
    if (per <= 4)       hipLaunchKernelGGL(select_kernel<4>, dim3(batch), dim3(kSelThreads), 0, s, p);
    else if (per <= 16) hipLaunchKernelGGL(select_kernel<16>, dim3(batch), dim3(kSelThreads), 0, s, p);
    else if (per <= 32) hipLaunchKernelGGL(select_kernel<32>, dim3(batch), dim3(kSelThreads), 0, s, p);
    else                hipLaunchKernelGGL(select_kernel<64>, dim3(batch), dim3(kSelThreads), 0, s, p);
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
