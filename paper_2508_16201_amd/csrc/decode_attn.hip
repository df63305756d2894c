// specvlm_decode_attn: grouped-query softmax attention of a short query block
// (1 query for plain decode, gamma+1 for parallel verification; Sec. 2.1 of the
// paper) over a bf16 KV cache, for gfx950: long caches in split-K (flash-decode)
// form, which the rest of this comment describes, short ones in one launch
// without splits (attn_short_kernel; attn_direct_chunks has the line).
//
// Work decomposition
//   One workgroup owns one (request, kv head, key split).  All G*q_len query
//   rows that share the kv head are packed into MFMA row blocks of 16 (MB of
//   them, MB <= 4), so every K/V byte is read from HBM exactly once.  The
//   workgroup has MB*KS compute waves -- wave (mb, ks) owns row block mb and
//   every KS-th 32-key chunk of each tile, so a wave carries one 16-row
//   accumulator only -- and, in the multi-query shapes, two or four loader
//   waves that do nothing but issue the tile loads: a direct-to-LDS load of
//   1 KB holds its wave for about 70 cycles, eight of them per tile are a
//   quarter of a tile's time when the waves that compute have to issue them.
//   More than 64 rows per kv head are cut into row groups, one workgroup each.
//
// Data movement
//   K/V tiles of TK keys stream HBM -> LDS with direct-to-LDS loads
//   (global_load_lds_dwordx4: no registers in between) into a ring of NS
//   stages; NS-1 tiles are in flight while one is consumed.  A stage is
//   released by one s_barrier per tile, which all waves pass; before it the
//   loader waves wait on their own vmcnt for the tile about to be read, never
//   on the younger tiles.  K rows are
//   stored with their 16-byte chunks XOR-swizzled by the key index so that the
//   MFMA operand reads (16 keys x one chunk per 16 lanes) hit distinct banks;
//   the swizzle is applied on the global-address side, the LDS side of a
//   direct load being fixed (lane * 16 bytes).  The Q fragments take the same
//   road (HBM -> LDS -> registers): with no load returning into registers the
//   compiler has nothing to guard with a wait that would drain the ring, and
//   the waits the kernel places itself are the only ones in the sweep.  A cache
//   of 8 MB or more per launch is read with non-temporal loads.
//
// Placement
//   Workgroup ids run over the kv heads fastest; ids are dealt to the 8 XCDs
//   round-robin, so with 8 kv heads all splits of a head and the merge of that
//   head share one XCD and its L2, where the partials (bf16 outputs, fp32
//   maxima and sums) stay between the two kernels.  A single request is cut
//   into about 192 workgroups in one round (HBM saturates before every CU is
//   busy); ragged batches of up to 64 requests into balanced pieces (equal runs
//   of key tiles per group of workgroups, see below), larger ones into splits
//   of at most 2048 keys that the dispatcher can balance.
//
// MFMA formulation (v_mfma_f32_16x16x32_bf16, lane = 16*c + r)
//   S^T = K Q^T : A = K chunk (rows = 16 keys, contraction = d), B = Q^T.  Query
//     row r sits in lane column r, keys 4c..4c+3 in the four accumulators: the
//     softmax statistics of a row live in lanes r, r+16, r+32, r+48.
//   O^T = V^T P^T : B = P^T is what the lane already holds (row r, keys
//     {4c..4c+3} of both 16-key halves); A = V^T needs per lane 8 keys x 1 value
//     column, which the transposing LDS read of gfx950 (ds_read_b64_tr_b16)
//     delivers from row-major V directly: per PV step two reads (one per
//     16-key half), no in-register transpose.  V rows are chunk-swizzled for
//     that read pattern like K rows are for theirs.  Step j yields value
//     columns 16j..16j+15 (lane (r, c): columns 16j+4c..16j+4c+3 of row r).
//     O^T keeps row r in lane column r too, so the running-max rescale is a
//     per-lane multiply -- and away from the mask no maximum is tracked at all
//     (exponentials against the reference the earlier chunks left, with the
//     tracked form as fallback; see compute_tile).
#include <atomic>

#include "common.h"

namespace specvlm {

#define SPECVLM_AS1 __attribute__((address_space(1)))
#define SPECVLM_AS3 __attribute__((address_space(3)))

struct AttnParams {
    const __bf16* q;
    const __bf16* k;
    const __bf16* v;
    __bf16* out;
    float* lse;
    int64_t q_tok, q_head, kv_tok, kv_head;
    const int32_t* cu_q;
    const int32_t* cu_kv;
    int batch, q_len, kv_len, n_q_heads, n_kv_heads, group;
    uint32_t inv_heads, inv_all_heads, inv_group, inv_splits, inv_rgroups, inv_split_keys, inv_help;   // reciprocal() of n_kv_heads, batch * n_kv_heads, ...
    float scale_log2;        // softmax_scale * log2(e)
    int num_splits, split_keys;
    __bf16* part_o;          // [batch*H_kv][num_splits][rows_pad][D] unnormalised partial outputs (bf16: see the merge kernel)
    float* part_ml;          // [batch*H_kv][num_splits][rows_pad][2] (running max in log2 units, sum)
    int rows_pad;            // rows per partial slot: n_rgroups * (row blocks per workgroup) * 16
    int n_rgroups;           // groups of at most 4 row blocks that share a (head, split): one workgroup each
    int n_work;
    int n_main;              // attn_short_kernel without splits: workgroups that compute (the rest prefetch)
    const uint64_t* block_mask;  // [sum q_len] tree masks of the block's queries, or null (chain)
    int balanced;            // batch mode: balanced pieces (see attn_balance) instead of uniform splits
    int max_wg;              // workgroups launched in balanced mode
    int32_t* seg_table;      // balanced mode: per (request, head) {first partial slot, pieces}, written by workgroup 0
};

constexpr int kChunkKeys = 32;       // keys per PV contraction step
constexpr int kMaxBalancedBatch = 64;   // (every workgroup walks the request lengths once)

// Brings in what a kernel is about to need of its parameters, together: left alone, the compiler fetches each one where it
// is first used, and every such place is a wait of its own in front of the first load of a key.  With this and divide() for
// the ids (us a layer, before / with divide() / both): 14/2 heads of size 64, 5000 keys 7.7 / 7.45 / 7.2, 28/4 heads, 4 queries, 3000
// keys 9.9 / 9.7 / 9.3, the 72B verify 15.9 / 15.6 / 15.4, 1511 keys in one launch 6.46 / 6.36 / 6.36.
__device__ __forceinline__ void attn_fetch_params(const AttnParams& p)
{
    __asm__ volatile("" :: "s"(p.q), "s"(p.k), "s"(p.v), "s"(p.q_tok), "s"(p.q_head), "s"(p.kv_tok), "s"(p.kv_head), "s"(p.cu_q), "s"(p.cu_kv),
                     "s"(p.q_len), "s"(p.kv_len), "s"(p.n_kv_heads), "s"(p.group), "s"(p.inv_heads), "s"(p.inv_group), "s"(p.inv_splits),
                     "s"(p.inv_rgroups), "s"(p.num_splits), "s"(p.split_keys), "s"(p.n_rgroups), "s"(p.n_main), "s"(p.scale_log2),
                     "s"(p.balanced), "s"(p.rows_pad));
}

// Tiles of request b in balanced mode, of the unit's size (one or more of the kernel's own tiles); a request with nothing to
// do (no queries, or fewer keys than queries) has none.
__device__ __forceinline__ int attn_request_tiles(const AttnParams& p, int b, int tile_keys)
{
    const int ql = p.cu_q[b + 1] - p.cu_q[b], kvl = p.cu_kv[b + 1] - p.cu_kv[b];
    return (ql <= 0 || kvl < ql) ? 0 : (kvl + tile_keys - 1) / tile_keys;
}

struct AttnBalance { int64_t n_units; int n_groups; };

// Balanced mode deals TILES OF REQUESTS (all kv heads of a token range together) to groups of
// n_kv_heads workgroups, one workgroup per head: n_units = tiles over the batch, n_groups = groups
// that share them -- never more groups than units, so every group's run is non-empty and the groups
// that touch a request are consecutive.  The workgroups of a group walk the same token rows at the
// same time (one DRAM page serves all heads of a token-major cache), and with workgroup ids dealt to
// the XCDs round-robin a kv head stays on one XCD.
__device__ __forceinline__ AttnBalance attn_balance(const AttnParams& p, int tile_keys)
{
    int64_t n = 0;
    for (int b = 0; b < p.batch; ++b) n += attn_request_tiles(p, b, tile_keys);
    AttnBalance r;
    r.n_units = n;
    r.n_groups = (int)min((int64_t)divide(p.max_wg, p.n_kv_heads, p.inv_heads).q, n);
    return r;
}
constexpr int kMaxSplits = 256;
constexpr float kSumRedo = 0x1p100f;     // a lane's sum of one chunk at or above this (or NaN) is redone with the maximum tracked
constexpr int kMaxQueryBlock = 64;      // queries per request: a row's view of its block is one 64-bit mask
constexpr int kTargetWorkgroups = 192;  // workgroups of a single-request launch

// s_waitcnt immediate (gfx9 encoding) that waits for vmcnt <= n only.
constexpr int vmcnt_imm(int n)
{
    return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8);
}

template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(N));
}

// Workgroup barrier that does not drain the direct-to-LDS loads still in
// flight for younger stages (a fence would).  Ordering of this wave's own LDS
// traffic is handled by the s_waitcnt the compiler places before each use.
__device__ __forceinline__ void stage_barrier()
{
    __asm__ volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    __asm__ volatile("" ::: "memory");
}

// Reductions over the four lanes r, r+16, r+32, r+48 that share a query row,
// with the VALU lane-swap instructions of gfx950 (no LDS crossbar round trip):
// v_permlane32_swap exchanges the upper 32 lanes of one operand with the lower
// 32 of the other, v_permlane16_swap the odd 16-lane rows with the even ones.
__device__ __forceinline__ float quad_max(float x)
{
    auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

__device__ __forceinline__ float quad_sum(float x)
{
    auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

constexpr int largest_divisor_le(int n, int cap)
{
    int best = 1;
    for (int d = 1; d <= cap; ++d) if (n % d == 0) best = d;
    return best;
}

// XOR applied to the 16-byte chunk index of value row `key` inside a tile.  The transposing read of
// one PV step touches, per 32 lanes, 8 consecutive keys x 32 contiguous bytes (two chunks 2j, 2j+1):
// with the pair index XORed by the key (d = 128: key mod 8; d = 64, two rows per 256 bytes: key/2
// mod 4) those 8 x 32 bytes fall on 64 distinct banks.
template <int D> __device__ __forceinline__ constexpr int v_swizzle(int key)
{
    return (D == 128) ? ((key & 7) << 1) : (((key >> 1) & 3) << 1);
}

// ds_read_b64_tr_b16: every lane hands in the address of 8 bytes (four 16-bit elements); inside each
// group of 16 lanes, lanes 4x..4x+3 together hold "row" x (16 elements), and lane o receives element o
// of rows 0..3.  Issued as assembly, with the wait below: as a builtin the compiler cannot tell the
// read from one that aliases the direct-to-LDS loads still in flight and drains them (vmcnt 0) first.
template <int OFFSET>
__device__ __forceinline__ u32x2 lds_read_tr16(uint32_t lds_addr)
{
    u32x2 v;
    __asm__ volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=&v"(v) : "v"(lds_addr), "n"(OFFSET));
    return v;
}

// Waits for this wave's LDS reads; the fragments pass through so that their uses stay behind the wait.
template <int N>
__device__ __forceinline__ void lds_wait_fragments(bf16x8 (&f)[N])
{
    static_assert(N == 4 || N == 8, "one fragment per 16 value columns");
    if constexpr (N == 8)
        __asm__ volatile("s_waitcnt lgkmcnt(0)"
                         : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]), "+v"(f[4]), "+v"(f[5]), "+v"(f[6]), "+v"(f[7]));
    else
        __asm__ volatile("s_waitcnt lgkmcnt(0)" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]));
}

// NLD: waves of a workgroup that only issue the direct-to-LDS loads (0: the compute waves issue them)
template <int D, int MB, int KS, int TK, int NS, int NLD, bool STREAM>
__global__ __launch_bounds__((MB * KS + NLD) * kWave)
void attn_split_kernel(const AttnParams p)
{
    attn_fetch_params(p);
    constexpr int NW = MB * KS;                  // compute waves per workgroup (the loader waves come after them)
    constexpr bool SPLIT_ROLES = NLD > 0;
    constexpr int DJ = D / 16;                   // value columns per lane (8 or 4)
    constexpr int KK = D / 32;                   // MFMA steps over the head dimension
    constexpr int CH = D / 8;                    // 16-byte chunks per key row
    constexpr int ROW_BYTES = D * 2;
    constexpr int KEYS_PER_LOAD = kWave / CH;    // key rows one wave-wide load covers (4 or 8)
    constexpr int TILE_BYTES = TK * ROW_BYTES;   // one of K or V
    constexpr int LOADS_PER_MAT = TK / KEYS_PER_LOAD;
    constexpr int LOADS = 2 * LOADS_PER_MAT;     // wave-wide loads per stage (K then V)
    constexpr int LW = SPLIT_ROLES ? NLD : largest_divisor_le(LOADS, NW);   // waves that issue loads
    constexpr int LPW = LOADS / LW;              // loads per loader wave per stage
    static_assert(LOADS % LW == 0, "the loads of a stage must divide among the loader waves");
    constexpr int NCHUNK = TK / kChunkKeys;      // 32-key chunks per tile
    constexpr int LDS_STRIDE = D + 4;            // merge buffer row stride (floats)
    static_assert(NCHUNK % KS == 0, "chunks must divide among the key-split waves");
    static_assert(NS >= 2 && NS <= 5, "ring depth");

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool is_loader = SPLIT_ROLES ? wave >= NW : wave < LW;
    const bool computes = SPLIT_ROLES ? wave < NW : true;
    const int lw = SPLIT_ROLES ? wave - NW : wave;   // loader index
    const int mb = wave % MB, ks = wave / MB;    // (compute waves)
    const int r = lane & 15, c = lane >> 4;

    extern __shared__ __align__(16) unsigned char smem[];
    // stage s: K tile at s*2*TILE_BYTES, V tile right after it

    // One piece of work: keys [k_begin, k_end) of (request b, kv head g) for all its query rows;
    // the result goes to partial slot slot0 (in units of rows), or straight to the output.
    auto piece = [&](const int b, const int g, const int row0, const int k_begin, const int k_end,
                     const int64_t slot0, const bool direct) {
    int q0 = 0, ql = p.q_len, kv0 = 0, kvl = p.kv_len;
    if (p.cu_q) { q0 = p.cu_q[b]; ql = p.cu_q[b + 1] - q0; }
    if (p.cu_kv) { kv0 = p.cu_kv[b]; kvl = p.cu_kv[b + 1] - kv0; }
    const int n_rows = p.group * ql;                // live query rows of this kv head

    // ---- this wave's Q fragments (B operand of S^T) ----
    // They travel HBM -> LDS -> registers like the tiles do (through the ring's last stage, which
    // no tile uses before the first barrier).  A load that returns into registers would make the
    // compiler guard those registers with waits that also drain the younger tile loads.
    bf16x8 qf[KK];
    int t_blk;                  // this lane's query row is the block's t_blk-th query
    unsigned char* q_stage = smem + (NS - 1) * (2 * TILE_BYTES) + wave * (KK * 1024);
    static_assert(MB * KS * KK * 1024 <= 2 * TILE_BYTES, "Q staging must fit in one ring stage");
    if (computes) {
        const int row = row0 + mb * 16 + r;
        const bool live = row < n_rows;             // padding rows read row 0: finite, never stored
        const QuotRem at = divide(live ? row : 0, p.group, p.inv_group);
        const int t = at.q, h = g * p.group + at.r;
        t_blk = t;
        const __bf16* qp = p.q + (int64_t)(q0 + t) * p.q_tok + (int64_t)h * p.q_head + c * 8;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
            __builtin_amdgcn_global_load_lds((const SPECVLM_AS1 void*)(qp + kk * 32),
                                             (SPECVLM_AS3 void*)(q_stage + kk * 1024), 16, 0, 0);
    }

    const char* kbase = reinterpret_cast<const char*>(p.k + (int64_t)kv0 * p.kv_tok + (int64_t)g * p.kv_head);
    const char* vbase = reinterpret_cast<const char*>(p.v + (int64_t)kv0 * p.kv_tok + (int64_t)g * p.kv_head);
    const uint32_t tok_bytes = (uint32_t)p.kv_tok * 2u;

    // ---- loader: wave-wide direct-to-LDS loads; load n of a stage covers
    // KEYS_PER_LOAD consecutive key rows of K (n < LOADS_PER_MAT) or of V ----
    const int ld_key = lane / CH;                   // key row inside the load
    const int ld_chunk = lane % CH;                 // LDS chunk slot inside the row
    auto issue_tile = [&](int tile, int stage) {
        const int base = k_begin + tile * TK;
        unsigned char* st = smem + stage * (2 * TILE_BYTES);
#pragma unroll
        for (int j = 0; j < LPW; ++j) {
            const int n = lw + LW * j;
            const bool is_v = n >= LOADS_PER_MAT;
            const int kl = (is_v ? n - LOADS_PER_MAT : n) * KEYS_PER_LOAD + ld_key;   // key inside the tile
            // rows past the split's end are masked in the compute: re-read its last row
            // (a cache hit) instead of pulling the neighbour split's keys from HBM
            const uint32_t key = (uint32_t)min(base + kl, k_end - 1);
            // K and V rows are chunk-swizzled so the operand reads spread over the banks: K for 16 keys x
            // one chunk per 16 lanes, V for the transposing read (8 keys x two neighbouring chunks per
            // 32 lanes, see v_swizzle)
            const int swz = is_v ? v_swizzle<D>(kl) : ((D == 128) ? (kl & 15) : ((kl >> 1) & 7));
            const int chunk = ld_chunk ^ swz;
            const char* src = (is_v ? vbase : kbase) + (key * tok_bytes + (uint32_t)chunk * 16u);
            unsigned char* dst = st + n * 1024;     // + lane * 16 by the hardware
            // a large cache is read once per launch: non-temporal, so it does not displace what is reused;
            // a small one (the draft's pruned cache, re-read every decode step) stays cacheable
            __builtin_amdgcn_global_load_lds((const SPECVLM_AS1 void*)src, (SPECVLM_AS3 void*)dst, 16, 0, STREAM ? 2 : 0);
        }
    };

    float m_run = -INFINITY, l_run = 0.f;
    floatx4 o_acc[DJ];
#pragma unroll
    for (int j = 0; j < DJ; ++j) o_acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};

    // (a zero scale is taken as a vanishing one, so that a masked logit, -inf, times the scale stays -inf
    // instead of becoming NaN; every other logit still scales to 0)
    const float sc = fmaxf(p.scale_log2, 1e-30f);
    auto compute_tile = [&](int tile, int stage) {
        const unsigned char* kt_lds = smem + stage * (2 * TILE_BYTES);
        const unsigned char* vt_lds = kt_lds + TILE_BYTES;
#pragma unroll
        for (int cc = 0; cc < NCHUNK / KS; ++cc) {
            const int chunk = ks + cc * KS;
            const int base = k_begin + tile * TK + chunk * kChunkKeys;
            if (base >= k_end) break;
            const bool need_mask = (base + kChunkKeys > k_end) || (base + kChunkKeys > kvl - ql);
            // ---- S^T = K Q^T for 32 keys ----
            floatx4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                const int x = kk * 4 + c;
                const int key0 = chunk * kChunkKeys + r, key1 = key0 + 16;
                const int sw0 = (D == 128) ? (key0 & 15) : ((key0 >> 1) & 7);
                const int sw1 = (D == 128) ? (key1 & 15) : ((key1 >> 1) & 7);
                const u32x4 k0 = *reinterpret_cast<const u32x4*>(kt_lds + key0 * ROW_BYTES + ((x ^ sw0) * 16));
                const u32x4 k1 = *reinterpret_cast<const u32x4*>(kt_lds + key1 * ROW_BYTES + ((x ^ sw1) * 16));
                s0 = mfma16(__builtin_bit_cast(bf16x8, k0), qf[kk], s0);
                s1 = mfma16(__builtin_bit_cast(bf16x8, k1), qf[kk], s1);
            }
            // The logits stay unscaled: the scale (> 0) is applied to the maximum once and rides in the
            // fused multiply-add that forms each exponent.
            float s[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) { s[i] = s0[i]; s[4 + i] = s1[i]; }
            if (need_mask) {
                // Block keys this lane's query row may see (bit b = block key b).  Chain: the block is
                // causal, query t sees block keys 0..t; tree: the caller's ancestor mask, fetched here
                // (only the last chunks of a request get here) rather than held through the sweep.
                const uint64_t row_mask = p.block_mask ? p.block_mask[q0 + t_blk] : ((2ull << t_blk) - 1ull);
                const uint32_t mask_lo = (uint32_t)row_mask, mask_hi = (uint32_t)(row_mask >> 32);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int key = base + (i < 4 ? 4 * c + i : 16 + 4 * c + (i - 4));
                    const int bk = key - (kvl - ql);        // index inside the block (negative: context key)
                    const uint32_t word = (bk & 32) ? mask_hi : mask_lo;
                    const bool in_block_hidden = bk >= 0 && ((word >> (bk & 31)) & 1u) == 0u;
                    s[i] = (key >= k_end || in_block_hidden) ? -INFINITY : s[i];
                }
            }
            // V^T fragments of the lane's 8 keys (4c+i and 16+4c+i, i < 4) by the transposing LDS read:
            // the 16 lanes of quarter c hand in the rows of keys 4c + x (x = r/4; four lanes per key,
            // 8 bytes each, together columns 16j..16j+15) and lane r receives column 16j + r of the four
            // keys -- the A operand of step j with no in-register transpose.
            bf16x8 vf[DJ];
            {
                const int kl = chunk * kChunkKeys + 4 * c + (r >> 2);           // (the second half is 16 rows on)
                const int pair_swz = v_swizzle<D>(kl) >> 1;                     // same for kl + 16
                const uint32_t vrow = (uint32_t)(uintptr_t)(SPECVLM_AS3 const void*)(vt_lds + kl * ROW_BYTES + (r & 3) * 8);
#pragma unroll
                for (int j = 0; j < DJ; ++j) {
                    const uint32_t src = vrow + (uint32_t)((j ^ pair_swz) * 32);
                    const u32x2 lo = lds_read_tr16<0>(src);
                    const u32x2 hi = lds_read_tr16<16 * ROW_BYTES>(src);
                    vf[j] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3));
                }
            }
            // Away from the mask the running maximum is not tracked: the exponentials are taken against
            // the reference the earlier chunks left (a logit above it only makes its term larger than one),
            // which saves the maximum, its exchange over the quarter waves and the rescale test -- a
            // quarter of a chunk's VALU work.  A lane sum that is no longer a moderate finite number (a
            // logit 2^100 above the reference, or a reference not set yet) sends the wave through the
            // tracked form of the same chunk instead.
            floatx8 pv;
            bool settled = false;
            if (!need_mask && !__any(!(m_run > -INFINITY))) {
                float psum = 0.f;
#pragma unroll
                for (int i = 0; i < 8; ++i) { pv[i] = fast_exp2(fmaf(s[i], sc, -m_run)); psum += pv[i]; }
                if (!__any(!(psum < kSumRedo))) {
                    l_run += psum;
                    settled = true;
                }
            }
            if (!settled) {
                float mx = fmaxf(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])),
                                 fmaxf(fmaxf(s[4], s[5]), fmaxf(s[6], s[7])));
                mx = quad_max(mx) * sc;
                const float m_new = fmaxf(m_run, mx);
                const float m_ref = (m_new == -INFINITY) ? 0.f : m_new;
                const float alpha = fast_exp2(m_run - m_ref);
                const bool rescale = m_new != m_run;
                m_run = m_new;
                float psum = 0.f;
#pragma unroll
                for (int i = 0; i < 8; ++i) { pv[i] = fast_exp2(fmaf(s[i], sc, -m_ref)); psum += pv[i]; }
                l_run = l_run * alpha + psum;
                if (__any(rescale)) {
#pragma unroll
                    for (int j = 0; j < DJ; ++j) o_acc[j] *= alpha;
                }
            }
            const bf16x8 pf = __builtin_convertvector(pv, bf16x8);
            // ---- O^T += V^T P^T ----
            lds_wait_fragments(vf);
#pragma unroll
            for (int j = 0; j < DJ; ++j) o_acc[j] = mfma16(vf[j], pf, o_acc[j]);
        }
    };

    // ---- ring of NS stages: NS-1 tiles in flight while one is consumed ----
    // The loader waves always start NS-1 tiles (a split shorter than that loads its last tile
    // again into a stage nobody reads), then every wave waits for its Q fragments, which are older
    // than any tile load, and takes them into registers.
    const int n_tiles = (k_end - k_begin + TK - 1) / TK;            // >= 1
    const int n_load = n_tiles > NS - 1 ? n_tiles : NS - 1;          // tiles as the loader counts them
    if constexpr (SPLIT_ROLES) {
    // Two loops, one per role (their registers do not add up); both pass the same barrier once per tile.
    if (is_loader) {
#pragma unroll
        for (int s = 0; s < NS - 1; ++s) issue_tile(s < n_tiles ? s : n_tiles - 1, s);
        int i = 0;
        do {
            // tiles issued after tile i so far: min(NS-2, n_load-1-i); each is LPW loads of a loader wave
            const int younger = min(NS - 2, n_load - 1 - i);
            wait_vmcnt<(NS - 2) * LPW>();
            if constexpr (NS >= 5) { if (younger <= 2) wait_vmcnt<2 * LPW>(); }
            if constexpr (NS >= 4) { if (younger <= 1) wait_vmcnt<1 * LPW>(); }
            if constexpr (NS >= 3) { if (younger <= 0) wait_vmcnt<0>(); }
            stage_barrier();                         // tile i landed for everyone; stage (i-1)%NS is free
            if (i + NS - 1 < n_load) issue_tile(i + NS - 1, (i + NS - 1) % NS);
        } while (++i < n_tiles);
        wait_vmcnt<0>();                             // (a short split's spare copies may still be landing)
    } else {
        wait_vmcnt<0>();                             // a compute wave's only loads: its Q fragments
        __asm__ volatile("" ::: "memory");
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
            qf[kk] = *reinterpret_cast<const bf16x8*>(q_stage + kk * 1024 + lane * 16);
        __asm__ volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): read before the stage is handed to the loaders
        __asm__ volatile("" ::: "memory");
        int i = 0;
        do {
            stage_barrier();
            compute_tile(i, i % NS);
        } while (++i < n_tiles);
    }
    } else {
    // Every wave computes and the first LW of them also issue the loads.  The loader waves always start
    // NS-1 tiles, then every wave waits for its Q fragments, which are older than any tile load.
    if (is_loader) {
#pragma unroll
        for (int s = 0; s < NS - 1; ++s) issue_tile(s < n_tiles ? s : n_tiles - 1, s);
        wait_vmcnt<(NS - 1) * LPW>();                // the Q loads are older than every tile load
    } else {
        wait_vmcnt<0>();
    }
    __asm__ volatile("" ::: "memory");
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
        qf[kk] = *reinterpret_cast<const bf16x8*>(q_stage + kk * 1024 + lane * 16);
    __asm__ volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0): read before the stage is handed to the loader
    __asm__ volatile("" ::: "memory");
    int i = 0;
    do {
        // tiles issued after tile i so far: min(NS-2, n_load-1-i); each is LPW loads of a loader wave
        const int younger = min(NS - 2, n_load - 1 - i);
        wait_vmcnt<(NS - 2) * LPW>();
        if constexpr (NS >= 5) { if (younger <= 2) wait_vmcnt<2 * LPW>(); }
        if constexpr (NS >= 4) { if (younger <= 1) wait_vmcnt<1 * LPW>(); }
        if constexpr (NS >= 3) { if (younger <= 0) wait_vmcnt<0>(); }
        stage_barrier();                             // tile i landed for everyone; stage (i-1)%NS is free
        if (is_loader && i + NS - 1 < n_load) issue_tile(i + NS - 1, (i + NS - 1) % NS);
        compute_tile(i, i % NS);
    } while (++i < n_tiles);
    wait_vmcnt<0>();                                 // (a short split's spare copies may still be landing)
    }

    // ---- epilogue (the loader waves only keep the barriers of the exchange) ----
    l_run = quad_sum(l_run);
    const int row = row0 + mb * 16 + r;
    const QuotRem out_at = divide(row, p.group, p.inv_group);
    const int t_row = out_at.q, h_row = g * p.group + out_at.r;
    const int64_t slot = slot0 + row;
    // The KS waves of a row block exchange their accumulators through LDS;
    // afterwards wave ks owns the column slice [ks*D/KS, (ks+1)*D/KS) of all
    // 16 rows, so every wave takes part in the final add and store.
    constexpr int SLICE = D / KS;                // columns per wave after the exchange
    constexpr int CPL = SLICE / 4;               // columns per lane (lane (r, c): c-th quarter)
    __syncthreads();                             // every wave is done with the ring
    float* sm_m = reinterpret_cast<float*>(smem);            // [NW][16]
    float* sm_l = sm_m + NW * 16;                            // [NW][16]
    float* sm_o = sm_l + NW * 16;                            // [NW][16][LDS_STRIDE]
    if (computes) {
        if (c == 0) { sm_m[wave * 16 + r] = m_run; sm_l[wave * 16 + r] = l_run; }
        float* buf = sm_o + (wave * 16 + r) * LDS_STRIDE + 4 * c;
#pragma unroll
        for (int j = 0; j < DJ; ++j) *reinterpret_cast<floatx4*>(buf + 16 * j) = o_acc[j];
    }
    __syncthreads();
    if (!computes) return;
    // (brought to one reference here and not before they are written: that was a barrier and a round trip more:  us a layer, before / now:
    // 64/8 heads, 12806 keys, 6 queries 14.97 / 14.71, one 13.79 / 13.63, 12 nodes 16.86 / 16.58;  14/2 heads of size 64, 12806 keys 8.87 / 8.66)
    float m_x[KS], m_all = -INFINITY, l_all = 0.f;
#pragma unroll
    for (int kx = 0; kx < KS; ++kx) { m_x[kx] = sm_m[(kx * MB + mb) * 16 + r]; m_all = fmaxf(m_all, m_x[kx]); }
    const float m_ref = (m_all == -INFINITY) ? 0.f : m_all;
#pragma unroll
    for (int kx = 0; kx < KS; ++kx) { m_x[kx] = fast_exp2(m_x[kx] - m_ref); l_all += m_x[kx] * sm_l[(kx * MB + mb) * 16 + r]; }
    const int col0 = ks * SLICE + c * CPL;
    floatx4 acc[CPL / 4];
#pragma unroll
    for (int qd = 0; qd < CPL / 4; ++qd) acc[qd] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kx = 0; kx < KS; ++kx) {
        const float* buf = sm_o + ((kx * MB + mb) * 16 + r) * LDS_STRIDE + col0;
#pragma unroll
        for (int qd = 0; qd < CPL / 4; ++qd) acc[qd] += m_x[kx] * *reinterpret_cast<const floatx4*>(buf + 4 * qd);
    }
    if (direct) {
        if (row >= n_rows) return;
        const float inv = 1.f / l_all;
        __bf16* op = p.out + (int64_t)(q0 + t_row) * p.q_tok + (int64_t)h_row * p.q_head + col0;
#pragma unroll
        for (int qd = 0; qd < CPL / 4; ++qd)
            *reinterpret_cast<bf16x4*>(op + 4 * qd) = __builtin_convertvector(acc[qd] * inv, bf16x4);
        if (p.lse && c == 0 && ks == 0)
            p.lse[(int64_t)(q0 + t_row) * p.n_q_heads + h_row] = (m_all + fast_log2(l_all)) * kLn2;
    } else {
        __bf16* po = p.part_o + slot * D + col0;
#pragma unroll
        for (int qd = 0; qd < CPL / 4; ++qd) *reinterpret_cast<bf16x4*>(po + 4 * qd) = __builtin_convertvector(acc[qd], bf16x4);
        if (c == 0 && ks == 0) { p.part_ml[slot * 2] = m_all; p.part_ml[slot * 2 + 1] = l_all; }
    }
    };   // piece

    if (!p.balanced) {
        // Uniform splits.  Dispatch order: the kv heads of one (request, row group, split) are neighbours.
        // Workgroups are dealt to the XCDs round-robin by id, so with 8 kv heads every split of head
        // g runs on XCD g: its partial results stay near that XCD, where the merge kernel (same
        // head-to-XCD order) finds them.  Token-major caches interleave the heads inside every token
        // row, so neighbours also walk the same DRAM pages at the same time.
        const QuotRem head = divide(blockIdx.x, p.n_kv_heads, p.inv_heads), part = divide(head.q, p.num_splits, p.inv_splits);
        const int g = head.r, split = part.r;
        // more than 64 query rows per kv head: groups of MB row blocks, one workgroup each; the groups of
        // a (head, split) re-read its keys, as neighbours in time on one XCD (mostly from its L2)
        const QuotRem group = divide(part.q, p.n_rgroups, p.inv_rgroups);
        const int rg = group.r, b = group.q;
        int ql = p.q_len, kvl = p.kv_len;
        if (p.cu_q) ql = p.cu_q[b + 1] - p.cu_q[b];
        if (p.cu_kv) kvl = p.cu_kv[b + 1] - p.cu_kv[b];
        if (ql <= 0 || kvl < ql) return;
        const int k_begin = split * p.split_keys;
        if (k_begin >= kvl) return;                     // the merge reads only the live splits
        const int bh = b * p.n_kv_heads + g;
        piece(b, g, rg * (MB * 16), k_begin, min(kvl, k_begin + p.split_keys),
              ((int64_t)bh * p.num_splits + split) * p.rows_pad, p.num_splits == 1);
        return;
    }

    // Balanced pieces for a batch.  The unit of work is UNIT keys of one request (all kv heads); the
    // units are numbered request-major, then tile, and group j -- workgroups j*H .. j*H+H-1, one per
    // kv head -- takes the contiguous run [j*T/G, (j+1)*T/G).  A run that crosses from one request
    // into the next is cut into pieces there; piece (group j, request b) of head g owns partial slot
    // (j + b)*H + g, unique because from one piece to the next exactly one of j and b grows.  Every
    // workgroup derives the same numbers from the request lengths, as the merge kernel does.
    // One row block is dealt by 128 keys whatever the tile: of 64 keys a piece is little work for what it costs to start and to merge, and with
    // few requests a row has twice as many pieces, eight to a trip of the merge (us a layer, units of 64 / 128 keys, size 128:  2 requests of 2500
    // keys, 28/4 heads 12.9 / 11.6;  4 of up to 6000, 7/1 heads 19.2 / 14.9;  8 of up to 600, 40/8 heads 13.1 / 10.8;  16 of 600, 12/3 heads 14.5 /
    // 13.0;  where a group has three to six units of 64 keys the finer ones are up to 7 % faster: 2 of up to 6000, 40/8 heads 16.2 / 16.8).
    constexpr int UNIT = MB == 1 ? 128 : TK;
    static_assert(UNIT % TK == 0, "a unit is whole tiles");
    const AttnBalance bal = attn_balance(p, UNIT);
    const int H = p.n_kv_heads;
    const int w = blockIdx.x;
    if (w == 0) {
        // the merge kernel's view of the decomposition: for every (request, head) its first partial
        // slot and the number of pieces (the groups that touch a request are consecutive; the group
        // that owns unit x is the largest j with j*T/G <= x)
        for (int seg = threadIdx.x; seg < p.batch * H; seg += (MB * KS + NLD) * kWave) {
            const int sb = seg / H, sg = seg % H;
            int64_t first = 0;
            for (int bb = 0; bb < sb; ++bb) first += attn_request_tiles(p, bb, UNIT);
            const int tiles = attn_request_tiles(p, sb, UNIT);
            int j_first = 0, live = 0;
            if (tiles > 0) {
                j_first = (int)(((first + 1) * bal.n_groups - 1) / bal.n_units);
                live = (int)(((first + tiles) * bal.n_groups - 1) / bal.n_units) - j_first + 1;
            }
            p.seg_table[2 * seg] = (j_first + sb) * H + sg;
            p.seg_table[2 * seg + 1] = live;
        }
    }
    const QuotRem run = divide(w, H, p.inv_heads);
    const int j = run.q, g = run.r;
    if (j >= bal.n_groups) return;
    int64_t x = (int64_t)j * bal.n_units / bal.n_groups;
    const int64_t x_end = (int64_t)(j + 1) * bal.n_units / bal.n_groups;
    int b = 0;
    int64_t base = 0;                                   // first unit of request b
    while (x < x_end) {
        int tiles = attn_request_tiles(p, b, UNIT);
        while (x >= base + tiles) {
            base += tiles;
            ++b;
            tiles = attn_request_tiles(p, b, UNIT);
        }
        const int t = (int)(x - base);
        const int n = (int)min((int64_t)(tiles - t), x_end - x);
        const int kvl = p.cu_kv[b + 1] - p.cu_kv[b];
        piece(b, g, 0, t * UNIT, min(kvl, (t + n) * UNIT), (int64_t)((j + b) * H + g) * p.rows_pad, false);
        x += n;
        __syncthreads();                                // the next piece reuses the ring and the exchange buffer
    }
}

// Merge of the split partials: o = sum_s 2^(m_s - m) o_s / sum_s 2^(m_s - m) l_s.
// The partial outputs travel as bf16 (the running maxima and sums stay fp32): each is rounded once, by
// at most 2^-9 of its own size, and the merged row is a convex combination of them, so the detour adds
// at most one more rounding of the size the bf16 output carries anyway, and it halves the bytes that
// the two kernels exchange.
// One workgroup per (kv head, query row); thread (grp, col) folds the splits grp, grp + GROUPS, ...
// for 4 output columns.  PRE covers all of a thread's splits, or they go in ROUNDS of PRE (launch_merge picks it), and every load of a
// round is issued up front, so the kernel costs one memory round trip; each group folds its splits against its own maximum and behind a single barrier
// four lanes a piece combine the GROUPS partial results.  (Splits beyond a thread's first three were a round trip each: 192 splits of
// 30000 keys, 4/1 heads of size 64, 11.9 us a layer, now 8.45;  96 splits of 12000, 14/2 heads, 8.4, now 6.95.)
// Twelve groups (two loads per thread at the usual 24 splits per head) measured best: 16.3 us per 72B
// layer against 16.7 with 8 groups, 16.35 with 16, 16.85 with 24 and 17.5 with 32; several rows per
// workgroup are slower as well (16.9 with two, 17.2 with four).
template <int D, int PRE, int THREADS, bool ROUNDS>
__global__ __launch_bounds__(THREADS)
void attn_merge_kernel(const AttnParams p)
{
    __asm__ volatile("" :: "s"(p.part_o), "s"(p.part_ml), "s"(p.cu_q), "s"(p.cu_kv), "s"(p.q_len), "s"(p.kv_len), "s"(p.batch), "s"(p.n_kv_heads),
                     "s"(p.group), "s"(p.inv_all_heads), "s"(p.inv_heads), "s"(p.inv_group), "s"(p.inv_split_keys), "s"(p.num_splits),
                     "s"(p.split_keys), "s"(p.rows_pad), "s"(p.out), "s"(p.lse), "s"(p.q_tok), "s"(p.q_head), "s"(p.n_q_heads));   // (see attn_fetch_params)
    constexpr int TPR = D / 4;                       // threads that cover one row of D columns
    constexpr int GROUPS = THREADS / TPR;            // split groups working in parallel
    __shared__ float s_m[GROUPS], s_l[GROUPS];
    __shared__ __align__(16) float s_acc[GROUPS][D + 4];           // (the groups' rows start on different banks)
    // (request, kv head) fastest: workgroup id modulo the XCD count follows the kv head, as in the split kernel
    const int nbh = p.batch * p.n_kv_heads;
    const QuotRem at = divide(blockIdx.x, nbh, p.inv_all_heads), head = divide(at.r, p.n_kv_heads, p.inv_heads);
    const int bh = at.r, row = at.q, b = head.q, g = head.r;
    int q0 = 0, ql = p.q_len, kvl = p.kv_len;
    if (p.cu_q) { q0 = p.cu_q[b]; ql = p.cu_q[b + 1] - q0; }
    if (p.cu_kv) { kvl = p.cu_kv[b + 1] - p.cu_kv[b]; }
    if (ql <= 0 || kvl < ql || row >= p.group * ql) return;
    // the partial slots of this (request, head) are consecutive: splits 0..live-1
    const int live = min(p.num_splits, divide(kvl + p.split_keys - 1, p.split_keys, p.inv_split_keys).q);
    const int64_t slot0 = (int64_t)bh * p.num_splits * p.rows_pad + row;
    // (a scalar base and 32-bit offsets: attn_merges_by_row leaves no larger (request, head) to this kernel)
    const char* const ml_base = reinterpret_cast<const char*>(p.part_ml + slot0 * 2);
    const char* const o_base = reinterpret_cast<const char*>(p.part_o + slot0 * D);
    const int tid = threadIdx.x;
    const int grp = tid / TPR, col = (tid % TPR) * 4;

    // (past the last split a group reads its first one again and leaves it out: no branch between the loads;  with a branch around
    // each and 64-bit addresses, 14/2 heads of size 64, 5000 keys were 7.2 us a layer instead of 6.7, 12000 keys 9.5 instead of 8.9.
    // Beyond the first eight a branch between fours, the same for the whole workgroup, and in rounds one between any two.)
    float m_loc = -INFINITY, l_loc = 0.f;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    int s0 = 0;
    do {
        const auto none_left = [&](int i) { return ROUNDS ? i > 0 && s0 + GROUPS * i >= live : i >= 8 && GROUPS * (i & ~3) >= live; };
        float2 ml_i[PRE];
        bf16x4 raw[PRE];
#pragma unroll
        for (int i = 0; i < PRE; ++i) {
            if (none_left(i)) break;
            const int s = s0 + grp + GROUPS * i;
            const uint32_t at = (uint32_t)((s < live ? s : min(grp, live - 1)) * p.rows_pad);
            ml_i[i] = *reinterpret_cast<const float2*>(ml_base + at * 8u);       // the same address across the group: one transaction
            raw[i] = *reinterpret_cast<const bf16x4*>(o_base + (at * (uint32_t)D + (uint32_t)col) * 2u);
        }
        float m_i[PRE], l_i[PRE];
        floatx4 ov[PRE];
#pragma unroll
        for (int i = 0; i < PRE; ++i) {
            const bool in = s0 + grp + GROUPS * i < live;
            m_i[i] = in ? ml_i[i].x : -INFINITY;
            l_i[i] = in ? ml_i[i].y : 0.f;
            const floatx4 o = __builtin_convertvector(raw[i], floatx4);
            ov[i] = in ? o : floatx4{0.f, 0.f, 0.f, 0.f};
        }
        float m_new = m_loc;
#pragma unroll
        for (int i = 0; i < PRE; ++i) m_new = fmaxf(m_new, m_i[i]);
        const float ref = (m_new == -INFINITY) ? 0.f : m_new;
        if constexpr (ROUNDS) {
            const float f_old = fast_exp2(m_loc - ref);
            acc *= f_old; l_loc *= f_old;
        }
#pragma unroll
        for (int i = 0; i < PRE; ++i) {
            if (none_left(i)) break;
            const float w = fast_exp2(m_i[i] - ref);             // 0 for an absent or empty split
            acc += w * ov[i];
            l_loc += w * l_i[i];
        }
        m_loc = m_new;
        s0 += GROUPS * PRE;
    } while (ROUNDS && s0 < live);
    *reinterpret_cast<floatx4*>(&s_acc[grp][col]) = acc;
    if (col == 0) { s_m[grp] = m_loc; s_l[grp] = l_loc; }
    __syncthreads();
    // four lanes a piece of four columns: three groups each, then by DPP.  (Group 0 alone walking over all twelve was 0.1 to 0.2 us longer, eight
    // lanes were no faster than four and, where a CU has several workgroups, slower:  us a layer, group 0 / four lanes:  14/2 heads of size 64, 3000 keys, one
    // query 6.28 / 6.12, six 7.68 / 7.49;  size 128, 12806 keys:  28/4 heads, six 11.9 / 11.74, 40/8 14.36 / 14.21, 64/8, one 13.75 / 13.64, but six the same
    // within the noise.)
    constexpr int LANES = 4, EACH = GROUPS / LANES;
    static_assert(GROUPS % LANES == 0 && TPR * LANES <= THREADS);
    if (tid >= TPR * LANES) return;
    const int w = tid % LANES, out_col = tid / LANES * 4;
    float m_g[EACH];
#pragma unroll
    for (int i = 0; i < EACH; ++i) m_g[i] = s_m[w + LANES * i];
    float m = m_g[0];
#pragma unroll
    for (int i = 1; i < EACH; ++i) m = fmaxf(m, m_g[i]);
    m = fmaxf(m, row_move<0xB1>(m)); m = fmaxf(m, row_move<0x4E>(m));
    const float m_ref = (m == -INFINITY) ? 0.f : m;
    floatx4 tot = {0.f, 0.f, 0.f, 0.f};
    float l = 0.f;
#pragma unroll
    for (int i = 0; i < EACH; ++i) {
        const float f = fast_exp2(m_g[i] - m_ref);               // 0 for a group without splits
        tot += f * *reinterpret_cast<const floatx4*>(&s_acc[w + LANES * i][out_col]);
        l += f * s_l[w + LANES * i];
    }
    l += row_move<0xB1>(l); l += row_move<0x4E>(l);
#pragma unroll
    for (int i = 0; i < 4; ++i) { tot[i] += row_move<0xB1>(tot[i]); tot[i] += row_move<0x4E>(tot[i]); }
    if (w != 0) return;
    tot *= 1.f / l;
    const QuotRem out_at = divide(row, p.group, p.inv_group);
    const int t = out_at.q, h = g * p.group + out_at.r;
    __bf16* op = p.out + (int64_t)(q0 + t) * p.q_tok + (int64_t)h * p.q_head + out_col;
    *reinterpret_cast<bf16x4*>(op) = __builtin_convertvector(tot, bf16x4);
    if (p.lse && out_col == 0)
        p.lse[(int64_t)(q0 + t) * p.n_q_heads + h] = (m + fast_log2(l)) * kLn2;
}

// Merge where a (request, head) has only a handful of pieces (the balanced decomposition, and uniform splits by
// attn_merges_by_row): each group of D/4 threads merges one query row on its own, with the loads of up to PRE pieces in
// flight together, so a workgroup finishes 256 / (D/4) rows and no cross-thread combine is needed.
template <int D, int PRE>
__global__ __launch_bounds__(256)
void attn_merge_rows_kernel(const AttnParams p)
{
    __asm__ volatile("" :: "s"(p.part_o), "s"(p.part_ml), "s"(p.cu_q), "s"(p.cu_kv), "s"(p.q_len), "s"(p.kv_len), "s"(p.batch), "s"(p.n_kv_heads),
                     "s"(p.group), "s"(p.inv_all_heads), "s"(p.inv_heads), "s"(p.inv_group), "s"(p.inv_split_keys), "s"(p.num_splits),
                     "s"(p.split_keys), "s"(p.rows_pad), "s"(p.out), "s"(p.lse), "s"(p.q_tok), "s"(p.q_head), "s"(p.n_q_heads));   // (see attn_fetch_params)
    constexpr int TPR = D / 4;
    constexpr int GROUPS = 256 / TPR;
    const int nbh = p.batch * p.n_kv_heads;
    const QuotRem at = divide(blockIdx.x, nbh, p.inv_all_heads), head = divide(at.r, p.n_kv_heads, p.inv_heads);
    const int bh = at.r, b = head.q, g = head.r;
    const int tid = threadIdx.x;
    const int row = at.q * GROUPS + tid / TPR, col = (tid % TPR) * 4;
    int q0 = 0, ql = p.q_len, kvl = p.kv_len;
    if (p.cu_q) { q0 = p.cu_q[b]; ql = p.cu_q[b + 1] - q0; }
    if (p.cu_kv) { kvl = p.cu_kv[b + 1] - p.cu_kv[b]; }
    if (ql <= 0 || kvl < ql || row >= p.group * ql) return;
    int live;
    int64_t slot0, step;                             // pieces, the row's slot in the first one, slots from one to the next
    if (p.balanced) {
        live = p.seg_table[2 * bh + 1];
        slot0 = (int64_t)p.seg_table[2 * bh] * p.rows_pad + row;
        step = (int64_t)p.n_kv_heads * p.rows_pad;   // the next group's piece
    } else {
        live = min(p.num_splits, divide(kvl + p.split_keys - 1, p.split_keys, p.inv_split_keys).q);
        slot0 = (int64_t)bh * p.num_splits * p.rows_pad + row;
        step = p.rows_pad;
    }
    float m = -INFINITY, l = 0.f;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < live; s0 += PRE) {
        // (past the last piece that one is read again and left out: branches only between fours of loads; a branch around each
        // was 25.3 instead of 24.8 us for the 26-node tree, none at all 16.9 instead of 16.6 for 64 nodes over 3000 keys)
        float2 ml_i[PRE];
        bf16x4 raw[PRE];
#pragma unroll
        for (int i = 0; i < PRE; ++i) {
            if (s0 + (i & ~3) >= live) break;
            const int64_t slot = slot0 + min(s0 + i, live - 1) * step;
            ml_i[i] = *reinterpret_cast<const float2*>(p.part_ml + slot * 2);
            raw[i] = *reinterpret_cast<const bf16x4*>(p.part_o + slot * D + col);
        }
        float m_i[PRE], l_i[PRE];
        floatx4 ov[PRE];
#pragma unroll
        for (int i = 0; i < PRE; ++i) {
            const bool in = s0 + i < live;
            m_i[i] = in ? ml_i[i].x : -INFINITY;
            l_i[i] = in ? ml_i[i].y : 0.f;
            const floatx4 o = __builtin_convertvector(raw[i], floatx4);
            ov[i] = in ? o : floatx4{0.f, 0.f, 0.f, 0.f};
        }
        float m_new = m;
#pragma unroll
        for (int i = 0; i < PRE; ++i) m_new = fmaxf(m_new, m_i[i]);
        const float m_ref = (m_new == -INFINITY) ? 0.f : m_new;
        const float f_old = fast_exp2(m - m_ref);
        acc *= f_old; l *= f_old;
#pragma unroll
        for (int i = 0; i < PRE; ++i) {
            const float w = fast_exp2(m_i[i] - m_ref);       // 0 for an absent or empty piece
            acc += w * ov[i];
            l += w * l_i[i];
        }
        m = m_new;
    }
    acc *= 1.f / l;
    const QuotRem out_at = divide(row, p.group, p.inv_group);
    const int t = out_at.q, h = g * p.group + out_at.r;
    __bf16* op = p.out + (int64_t)(q0 + t) * p.q_tok + (int64_t)h * p.q_head + col;
    *reinterpret_cast<bf16x4*>(op) = __builtin_convertvector(acc, bf16x4);
    if (p.lse && col == 0)
        p.lse[(int64_t)(q0 + t) * p.n_q_heads + h] = (m + fast_log2(l)) * kLn2;
}

// Short key ranges (bound: launches and round trips).  No ring and no barrier in the sweep: every wave owns 32 * CH
// keys of the workgroup's range and issues all its loads before it waits for the first.  K and V come through
// registers (the bytes in flight are then not bound by the LDS) into a private LDS buffer, one 32-key chunk at a
// time, and from there in operand layout: loaded in that layout directly a quad of lanes would touch four cache
// lines, and the address path takes one line a cycle (10.3 against 7.6 us at 1511 keys).  All logits of a wave are
// there before its maximum is taken, so nothing is rescaled; the waves meet once, at the end.
//   COLS < D: a workgroup computes a slice of 16 VALUE COLUMNS over ALL keys of its rows and writes output.  The
//     slices recompute the logits, and in return there are no partial results and no merge launch, which costs
//     2.8 us behind a first kernel of 3.6.  Every workgroup pulls all of K and the cache lines of V through one CU,
//     so this is for short caches only: attn_direct_chunks has the line and both sides' times.
//   COLS = D: a workgroup computes a key split and writes a partial result for the merge (head size 64, one block of
//     query rows: launch_attn_d has both sides' times; at head size 128 it equals the ring kernel).
//
// Helper workgroups.  The few workgroups that compute bring in about 100 bytes/ns each, bound by their CU's
// outstanding misses; helpers on the same XCD touch the head's rows at the same time, so that most of those misses
// find the line in that XCD's L2 already (7.4 -> 6.3 us at 1511 keys of head size 64, 9.0 -> 7.4 us at 1024 keys of
// head size 128; the caches of 80 to 120 layers in turn, so that they come from beyond the L2).
template <int D, int THREADS>
__device__ __forceinline__ void attn_prefetch_rows(const AttnParams& p, int id)
{
    // ids are dealt to the XCDs round-robin: helper `id` shares the XCD of workgroup id % kNumXcd and reads a share of
    // that workgroup's head (with fewer workgroups than XCDs some XCDs compute nothing)
    const int x = id % kNumXcd, n_help = (p.n_work - p.n_main) / kNumXcd, k = (id - p.n_main) / kNumXcd;
    if (x >= p.n_main) return;
    int ql = p.q_len, kv0 = 0, kvl = p.kv_len;
    if (p.cu_q) { ql = p.cu_q[1] - p.cu_q[0]; kv0 = p.cu_kv[0]; kvl = p.cu_kv[1] - kv0; }
    const int g = divide(x, p.n_kv_heads, p.inv_heads).r;
    const RowRange rows = helper_rows(ql, kvl, k, n_help, p.inv_help);
    const int first = rows.first, n = rows.n * (D / 8);
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (int i = threadIdx.x; i < n; i += THREADS) {
        const int64_t off = (int64_t)(kv0 + first + i / (D / 8)) * p.kv_tok + (int64_t)g * p.kv_head + (i % (D / 8)) * 8;
        acc ^= *reinterpret_cast<const u32x4*>(p.k + off) ^ *reinterpret_cast<const u32x4*>(p.v + off);
    }
    __asm__ volatile("" :: "v"(acc));
}

template <int D, int NW, int CH, int COLS>
__global__ __launch_bounds__(NW * kWave)
void attn_short_kernel(const AttnParams p)
{
    attn_fetch_params(p);
    constexpr bool DIRECT = COLS < D;
    constexpr int KK = D / 32;                       // MFMA steps over the head dimension
    constexpr int SLICES = D / COLS;
    constexpr int DJ = COLS / 16;
    constexpr int WAVE_KEYS = CH * kChunkKeys;
    constexpr int KP = D / 8, VP = COLS / 8;         // 16-byte pieces per key row and per row of the value slice
    constexpr int KPL = kWave / KP, VPL = kWave / VP;   // rows that one wave-wide load covers
    constexpr int KL = kChunkKeys / KPL, VL = kChunkKeys / VPL;   // loads per chunk
    constexpr int K_BYTES = kChunkKeys * D * 2;
    constexpr int WAVE_LDS = K_BYTES + kChunkKeys * COLS * 2;
    static_assert(16 * COLS * 4 + NW * 64 <= WAVE_LDS, "a wave's result takes the place of its buffers");
    // LDS: a private part per wave (its [row][column] fp32 result afterwards), then the waves' maxima and sums
    extern __shared__ __align__(16) unsigned char smem[];
    float (*s_m)[NW] = reinterpret_cast<float (*)[NW]>(smem + NW * WAVE_LDS);
    float (*s_l)[NW] = s_m + 16;

    if (DIRECT && (int)blockIdx.x >= p.n_main) { attn_prefetch_rows<D, NW * kWave>(p, blockIdx.x); return; }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, c = lane >> 4;
    // kv heads fastest, as in the split kernel: with 8 kv heads a head's workgroups share an XCD and its L2
    const QuotRem head = divide(blockIdx.x, p.n_kv_heads, p.inv_heads);
    const QuotRem cut = DIRECT ? QuotRem{head.q / SLICES, head.q % SLICES} : divide(head.q, p.num_splits, p.inv_splits);
    const QuotRem block = divide(cut.q, p.n_rgroups, p.inv_rgroups);
    const int g = head.r, part = cut.r;              // (part: column slice or key split)
    const int rb = block.r, b = block.q;             // block of 16 query rows, request
    int q0 = 0, ql = p.q_len, kv0 = 0, kvl = p.kv_len;
    if (p.cu_q) { q0 = p.cu_q[b]; ql = p.cu_q[b + 1] - q0; kv0 = p.cu_kv[b]; kvl = p.cu_kv[b + 1] - kv0; }
    const int n_rows = p.group * ql;
    if (ql <= 0 || kvl < ql || rb * 16 >= n_rows) return;
    const int k_begin = DIRECT ? 0 : part * p.split_keys;
    const int k_end = DIRECT ? kvl : min(kvl, k_begin + p.split_keys);
    if (k_begin >= kvl) return;                      // (the merge reads only the live splits)

    const int row = rb * 16 + r;
    const bool live = row < n_rows;                  // padding rows read row 0: finite, never stored
    const QuotRem at = divide(live ? row : 0, p.group, p.inv_group);
    const int t = at.q, h = g * p.group + at.r;
    const int k_wave = k_begin + wave * WAVE_KEYS;   // this wave's first key
    const char* kbase = reinterpret_cast<const char*>(p.k + (int64_t)kv0 * p.kv_tok + (int64_t)g * p.kv_head);
    const char* vbase = reinterpret_cast<const char*>(p.v + (int64_t)kv0 * p.kv_tok + (int64_t)g * p.kv_head +
                                                      (DIRECT ? part * COLS : 0));
    const uint32_t tok_bytes = (uint32_t)p.kv_tok * 2u;
    unsigned char* const k_lds = smem + wave * WAVE_LDS;
    unsigned char* const v_lds = k_lds + K_BYTES;

    float m = -INFINITY, l = 0.f;
    floatx4 o_acc[DJ];
#pragma unroll
    for (int j = 0; j < DJ; ++j) o_acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (k_wave < k_end) {
        bf16x8 qf[KK];
        u32x4 kraw[CH][KL], vraw[CH][VL];
        const __bf16* qp = p.q + (int64_t)(q0 + t) * p.q_tok + (int64_t)h * p.q_head + c * 8;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qp + kk * 32);
        // (keys past the end are masked below: the last key is read again)
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) {
#pragma unroll
            for (int n = 0; n < KL; ++n) {
                const uint32_t key = (uint32_t)min(k_wave + ch * kChunkKeys + n * KPL + lane / KP, k_end - 1);
                kraw[ch][n] = *reinterpret_cast<const u32x4*>(kbase + (key * tok_bytes + (uint32_t)(lane % KP) * 16u));
            }
        }
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) {
#pragma unroll
            for (int n = 0; n < VL; ++n) {
                const uint32_t key = (uint32_t)min(k_wave + ch * kChunkKeys + n * VPL + lane / VP, k_end - 1);
                vraw[ch][n] = *reinterpret_cast<const u32x4*>(vbase + (key * tok_bytes + (uint32_t)(lane % VP) * 16u));
            }
        }
        // ---- logits of all keys of the wave (S^T = K Q^T, as in the split kernel) ----
        const float sc = fmaxf(p.scale_log2, 1e-30f);      // (see attn_split_kernel)
        float s[CH][8];
        float mx = -INFINITY;
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) {
            // (LDS executes a wave's accesses in order: the buffer is rewritten behind the reads of the last chunk)
#pragma unroll
            for (int n = 0; n < KL; ++n) {
                const int kl = n * KPL + lane / KP;
                const int swz = (D == 128) ? (kl & 15) : ((kl >> 1) & 7);
                *reinterpret_cast<u32x4*>(k_lds + kl * (D * 2) + (((lane % KP) ^ swz) * 16)) = kraw[ch][n];
            }
            floatx4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                const int x = kk * 4 + c;
                const int sw = (D == 128) ? (r & 15) : ((r >> 1) & 7);      // (the same for row r + 16)
                const u32x4 k0 = *reinterpret_cast<const u32x4*>(k_lds + r * (D * 2) + ((x ^ sw) * 16));
                const u32x4 k1 = *reinterpret_cast<const u32x4*>(k_lds + (r + 16) * (D * 2) + ((x ^ sw) * 16));
                s0 = mfma16(__builtin_bit_cast(bf16x8, k0), qf[kk], s0);
                s1 = mfma16(__builtin_bit_cast(bf16x8, k1), qf[kk], s1);
            }
            const int base = k_wave + ch * kChunkKeys;
#pragma unroll
            for (int i = 0; i < 4; ++i) { s[ch][i] = s0[i]; s[ch][4 + i] = s1[i]; }
            if (base + kChunkKeys > k_end || base + kChunkKeys > kvl - ql) {
                // (no logit of a chunk past the last key is looked at: their masks, which nothing overlaps, were the launch's
                // end where a wave begins with few keys: head size 64, 1352 keys 7.6 us, now 6.5; 128, 904 keys 8.0, now 7.4)
                if (base >= k_end) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) s[ch][i] = -INFINITY;
                } else {
                    const uint64_t row_mask = p.block_mask ? p.block_mask[q0 + t] : ((2ull << t) - 1ull);
                    const uint32_t mask_lo = (uint32_t)row_mask, mask_hi = (uint32_t)(row_mask >> 32);
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int key = base + (i < 4 ? 4 * c + i : 16 + 4 * c + (i - 4));
                        const int bk = key - (kvl - ql);
                        const uint32_t word = (bk & 32) ? mask_hi : mask_lo;
                        const bool in_block_hidden = bk >= 0 && ((word >> (bk & 31)) & 1u) == 0u;
                        s[ch][i] = (key >= k_end || in_block_hidden) ? -INFINITY : s[ch][i];
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) mx = fmaxf(mx, s[ch][i]);
        }
        m = quad_max(mx) * sc;
        const float m_ref = (m == -INFINITY) ? 0.f : m;
        bf16x8 pf[CH];
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) {
            floatx8 pv;
#pragma unroll
            for (int i = 0; i < 8; ++i) { pv[i] = fast_exp2(fmaf(s[ch][i], sc, -m_ref)); l += pv[i]; }
            pf[ch] = __builtin_convertvector(pv, bf16x8);
        }
        l = quad_sum(l);
        // ---- O^T = V^T P^T ----
        const int vk = 4 * c + (r >> 2);                             // (the second half of a chunk is 16 rows on)
        const int pair_swz = DIRECT ? 0 : v_swizzle<D>(vk) >> 1;     // a 16-column slice needs none: 8 rows are 256 bytes
        const uint32_t v_addr = (uint32_t)(uintptr_t)(SPECVLM_AS3 const void*)(v_lds + vk * (COLS * 2) + (r & 3) * 8);
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) {
#pragma unroll
            for (int n = 0; n < VL; ++n) {
                const int kl = n * VPL + lane / VP;
                const int swz = DIRECT ? 0 : v_swizzle<D>(kl);
                *reinterpret_cast<u32x4*>(v_lds + kl * (COLS * 2) + (((lane % VP) ^ swz) * 16)) = vraw[ch][n];
            }
            __asm__ volatile("" ::: "memory");
            u32x2 lo[DJ], hi[DJ];
#pragma unroll
            for (int j = 0; j < DJ; ++j) {
                const uint32_t src = v_addr + (uint32_t)((j ^ pair_swz) * 32);
                lo[j] = lds_read_tr16<0>(src);
                hi[j] = lds_read_tr16<16 * COLS * 2>(src);
            }
            __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int j = 0; j < DJ; ++j) {
                __asm__ volatile("" : "+v"(lo[j]), "+v"(hi[j]));     // (their uses stay behind the wait)
                o_acc[j] = mfma16(__builtin_bit_cast(bf16x8, __builtin_shufflevector(lo[j], hi[j], 0, 1, 2, 3)), pf[ch], o_acc[j]);
            }
        }
    }
    // ---- the waves meet: lane (r, c) holds columns 16j + 4c .. 16j + 4c + 3 of row r ----
    // 16-byte piece q of a row goes to place q ^ r: the 16 rows of a store or a load fall on different banks
    constexpr int PIECES = COLS / 4;
    constexpr int LANES = 4, EACH = NW / LANES;      // (DIRECT: lanes that sum a piece, waves' results to each)
    constexpr int SKEW = DIRECT ? 256 / LANES : 0;   // (the waves' results start on different banks where lanes of one load go over the waves)
#pragma unroll
    for (int j = 0; j < DJ; ++j)
        reinterpret_cast<floatx4*>(k_lds + wave * SKEW)[r * PIECES + ((4 * j + c) ^ (r & (PIECES - 1)))] = o_acc[j];
    if (c == 0) { s_m[r][wave] = m; s_l[r][wave] = l; }
    if constexpr (DIRECT) {
        // four lanes a piece sum the waves' results, a quarter of them each, then by DPP: one wave of each SIMD has work.  A thread per piece is one
        // wave's walk over all the results, and was the launch's last 0.5 us;  a lane per wave and piece has every wave reduce, which loses from eight
        // query rows on.  Us a layer, thread / lane per wave / four lanes:  14/2 heads of size 64, 1511 keys, one query 6.37 / 6.18 / 6.04, six 6.68 /
        // 6.90 / 6.46;  4/1 heads, 250 keys, six 3.43 / 3.48 / 3.33;  size 128, 28/4 heads, 500 keys, four 5.68 / 5.82 / 5.56;  40/8 heads, 1010 keys, twelve
        // 8.07 / 8.25 / 7.79.  (Over 492 shapes four lanes are 3.0 % less than a thread, two as many, eight 1.6 %.)
        static_assert(16 * PIECES == kWave && NW % LANES == 0 && NW > LANES);
        const int w = threadIdx.x % LANES, orow = threadIdx.x / LANES / PIECES, piece = threadIdx.x / LANES % PIECES, grow = rb * 16 + orow;
        const QuotRem out_at = divide(grow, p.group, p.inv_group);
        const int to = out_at.q, ho = g * p.group + out_at.r;
        __syncthreads();
        if (grow >= n_rows || threadIdx.x >= kWave * LANES) return;
        float m_w[EACH], l_w[EACH];
        floatx4 o_w[EACH];
#pragma unroll
        for (int i = 0; i < EACH; ++i) {
            m_w[i] = s_m[orow][w + LANES * i];
            l_w[i] = s_l[orow][w + LANES * i];
            o_w[i] = reinterpret_cast<const floatx4*>(smem + (w + LANES * i) * (WAVE_LDS + SKEW))[orow * PIECES + (piece ^ (orow & (PIECES - 1)))];
        }
        const auto over_lanes = [](float x, auto op) {
            x = op(x, row_move<0xB1>(x));
            return op(x, row_move<0x4E>(x));
        };
        const auto sum = [](float a, float b) { return a + b; };
        float m_all = m_w[0], l_all = 0.f;
#pragma unroll
        for (int i = 1; i < EACH; ++i) m_all = fmaxf(m_all, m_w[i]);
        m_all = over_lanes(m_all, [](float a, float b) { return fmaxf(a, b); });
        const float ref = (m_all == -INFINITY) ? 0.f : m_all;
        floatx4 tot = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < EACH; ++i) {
            const float f = fast_exp2(m_w[i] - ref);             // 0 for a wave without keys
            tot += f * o_w[i];
            l_all += f * l_w[i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) tot[i] = over_lanes(tot[i], sum);
        l_all = over_lanes(l_all, sum);
        if (w != 0) return;
        tot *= 1.f / l_all;
        *reinterpret_cast<bf16x4*>(p.out + (int64_t)(q0 + to) * p.q_tok + (int64_t)ho * p.q_head + part * COLS + 4 * piece) =
            __builtin_convertvector(tot, bf16x4);
        if (p.lse && part == 0 && piece == 0)
            p.lse[(int64_t)(q0 + to) * p.n_q_heads + ho] = (m_all + fast_log2(l_all)) * kLn2;
        return;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 16 * PIECES; e += NW * kWave) {
        const int orow = e / PIECES, piece = e % PIECES, grow = rb * 16 + orow;
        if (grow >= n_rows) continue;
        float m_all = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) m_all = fmaxf(m_all, s_m[orow][w]);
        const float ref = (m_all == -INFINITY) ? 0.f : m_all;
        floatx4 tot = {0.f, 0.f, 0.f, 0.f};
        float l_all = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float f = fast_exp2(s_m[orow][w] - ref);           // 0 for a wave without keys
            tot += f * reinterpret_cast<const floatx4*>(smem + w * WAVE_LDS)[orow * PIECES + (piece ^ (orow & (PIECES - 1)))];
            l_all += f * s_l[orow][w];
        }
        const int64_t slot = ((int64_t)(b * p.n_kv_heads + g) * p.num_splits + part) * p.rows_pad + grow;
        *reinterpret_cast<bf16x4*>(p.part_o + slot * D + 4 * piece) = __builtin_convertvector(tot, bf16x4);
        if (piece == 0) { p.part_ml[slot * 2] = m_all; p.part_ml[slot * 2 + 1] = l_all; }
    }
}

// ---------------------------------------------------------------- host side ----
// A batch whose split count is left to the library is cut into balanced pieces by the kernels
// themselves (they know the request lengths; the host only knows their maximum).
static bool attn_is_balanced(int batch, int num_splits, int n_kv_heads, int rows)
{
    return batch > 1 && batch <= kMaxBalancedBatch && num_splits == 0 && n_kv_heads <= kNumCu && rows <= 64;
}

// Query rows of a kv head beyond 64 (long chains, draft trees) are cut into groups of equal size,
// at most 4 row blocks of 16 each: n groups, mb row blocks per group.
static void attn_row_groups(int rows, int* n_groups, int* mb)
{
    const int blocks = (rows + 15) / 16;
    *n_groups = (blocks + 3) / 4;
    *mb = (blocks + *n_groups - 1) / *n_groups;
}

// Launch shapes of attn_short_kernel.  Chunks per wave of a launch without splits; 0: the shape takes splits.
// Where the line lies (us a layer, splits and merge against this, one to four row blocks per kv head, caches of 40 to
// 160 layers in turn):  head size 64:  512 keys 6.5-7.9 / 3.9-4.3, 1024: 6.7-8.0 / 5.0-5.4, 1536: 6.7-8.1 / 6.1-6.5,
// 1790: 6.9-8.3 / 6.7-7.1;  head size 128:  512 keys 7.5-9.6 / 5.1-5.9, 1024: 7.7-9.6 / 7.1-8.7, 1280: 7.7-9.8 / 8.0-10.1.
// With five row blocks and more (up to 64) the splits' side grows faster: 1536 keys of size 64 8.3-8.8 / 6.6-8.0, 1024 of
// size 128 9.6-10.1 / 7.9-9.3.  More workgroups than CUs would take a second round.
// Less than that where the helpers miss heads or there are none:
//   one request whose heads do not divide the XCDs (a helper reads one head an XCD): 3, 5 or 6 heads, size 64, 1400 keys,
//     token-major 6.9-7.2 / 7.6-8.1, 1280 keys 0 to 10 % faster than splits; 10 and more heads lose from 1100 keys on (32 heads,
//     1200 keys 8.5 / 9.3) and win 8 % at 1000; size 128, 16 heads, 1024 keys 8.5 / 9.7, 768 keys 8.5 / 7.5;
//   a batch of more than 16 heads in all with more than four each, size 64: 4 requests of 8 heads, token-major, 1536 keys
//     10.7 / 12.0, 1280 keys 10.6 / 9.3; more than 16 heads each, 2 requests of 24 heads, 1280 keys 10.7 / 11.1;
//   a batch that fetches too much.  A head's slices lie on as many XCDs as its ids are dealt to, and each of these fetches
//     the head's rows (MB over all XCDs; the balanced pieces cost more with more requests):  32 requests of 2 heads, size
//     64, 1500 keys, 98 MB 16.8 / 18.2, 1280 keys, 84 MB 16.6 / 15.9;  size 128:  8 of 3 heads, 900 keys, 88 MB 12.5 / 14.8;
//     6 of 5, 768 keys, 94 MB 12.0 / 13.5;  5 of 6, 900 keys, 55 MB 12.4 / 13.1;  16 of 2, 900 keys, 59 MB 14.0 / 13.5.
// Other batches (2 to 64 requests, against the balanced pieces and their merge): size 64, 14/2 heads, 2 requests of 1536
// keys 10.7 / 7.5, 8 requests 12.5 / 8.1; size 128, 64/8 heads, 2 requests of 1024 keys 10.1 / 8.7, 4 requests 11.6 / 10.2.
constexpr int kDirectWaves = 8, kShortWaves = 4;
constexpr int kPrefetchers = 15;       // helper workgroups per XCD, at most (1511 keys: 7: 6.5 us, 15: 6.3, 28: 6.4)
static int attn_direct_chunks(int batch, int kv_len, int n_kv_heads, int head_dim, int rows, int num_splits)
{
    if (num_splits != 0) return 0;                            // (a caller that names a split count gets it)
    const int64_t wgs = (int64_t)batch * n_kv_heads * ((rows + 15) / 16) * (head_dim / 16);
    if (wgs > kNumCu) return 0;
    int most = head_dim == 64 ? 6 : 4;
    if (batch == 1) {
        if (kNumXcd % n_kv_heads != 0) most = head_dim == 64 && n_kv_heads < kNumXcd ? 5 : head_dim == 64 ? 4 : 3;
    } else {
        const int shared = n_kv_heads & -n_kv_heads;          // (ids run over the heads first: a head's step by n_kv_heads)
        int spread = shared < kNumXcd ? kNumXcd / shared : 1;
        if (spread > head_dim / 16) spread = head_dim / 16;
        if (4ll * batch * n_kv_heads * kv_len * head_dim * spread > ((44ll + batch) << 20)) return 0;
        if (head_dim == 64 && n_kv_heads > 4 && batch * n_kv_heads > 16) most = n_kv_heads > 16 ? 4 : 5;
    }
    const int ch = (kv_len + kDirectWaves * kChunkKeys - 1) / (kDirectWaves * kChunkKeys);
    return ch <= most ? ch : 0;
}

static int choose_splits(int batch, int kv_len, int n_kv_heads, int n_rgroups, int num_splits)
{
    const int max_by_len = (kv_len + 127) / 128;              // at least two tiles per split
    int s = num_splits;
    if (s <= 0) {
        const int heads = batch * n_kv_heads * n_rgroups;
        // One request: a single round of workgroups, about three per four CUs.  Every workgroup then
        // streams the same share from start to end and HBM is saturated well before all CUs are
        // busy; more, smaller splits only add partial results and rounds (measured on 8 kv heads:
        // 131K keys run at 6.2 TB/s with 24 or 32 splits per head, 4.7 TB/s with 128; 33K keys at
        // 4.9 TB/s with 24, 4.2 TB/s with 32).
        s = (kTargetWorkgroups + heads - 1) / heads;
        // (with several row groups per head the sweep is bound by arithmetic, not HBM: as many workgroups
        // as fit in one round on the 256 CUs, never one more)
        if (n_rgroups > 1) s = kNumCu / heads;
        if (batch > 1) {
            // Batches too large for the balanced decomposition: cap a split at 2048 keys so that
            // long and short requests decompose into similar pieces the dispatcher can balance,
            // and make a launch of several rounds a whole number of rounds of 2 x 256 workgroups.
            const int by_len = (kv_len + 2047) / 2048;
            if (by_len > s) s = by_len;
            const int slots = 2 * kNumCu;
            if (heads * s > slots && slots % heads == 0) {
                const int unit = slots / heads;
                s = ((s + unit / 2) / unit) * unit;
                if (s < unit) s = unit;
            }
        }
    }
    if (s > max_by_len) s = max_by_len;
    if (s > kMaxSplits) s = kMaxSplits;
    if (s < 1) s = 1;
    return s;
}

// Which merge uniform splits take.  A workgroup of attn_merge_kernel finishes one row with twelve groups of threads, so
// with eight splits or fewer a third of it has nothing to do, and when there are several such workgroups to a CU a group
// per row, which has all its loads in flight as well, does it in an eighth (head size 64: a sixteenth) of the workgroups.
// Us a layer, one row per workgroup against this (2 to 8 splits; keys in brackets):
//   size 128, 8 heads:  512 rows [1600] 11.0-15.6 / 11.6-15.6, 768 [3000] 0 to 3 % faster, 1664 [12826] 28.9-66.0 / 27.6-64.0,
//     4096 [3000] 22.4 / 18.2;  10 heads:  800 [3000] 13.2-15.2 / 14.3-15.6;  1 or 2 heads:  1280 [3000] 7 % slower to 3 % faster,
//     1536 3 % slower to 6 % faster, 2048 2 to 9 % faster;
//   size 64, 8 heads:  1024 [1600] 9.8-12.8 / 10.4-12.9, 1536 [3000] 1 % slower to 2 % faster, 4096 [1600] 13.6-17.8 / 11.6-16.1;
//     10 heads:  2560 [3000], 8 splits 18.3 / 19.0;  2 heads:  2048 [3000] 7 % slower to 3 % faster, 3072 0 to 9 % faster.
// Where the kv heads are a multiple of the XCDs a head's partials lie in the L2 of the XCD that merges them; elsewhere more
// rows are needed to hide the way.  With more splits the second trip costs more (16 splits 18.7 / 20.1).
// The kernel of one row per workgroup reaches its splits by 32-bit byte offsets.  Where those do not get that far (480000 rows of
// size 128 in 36 splits: 64 queries of a kv head's 7500 q heads) a group per row, with 64 bits, does it.
constexpr int kMergeRowPieces = 8, kMergeGroups = 12;
static bool attn_merges_by_row(int n_kv_heads, int64_t total_rows, int rows_pad, int head_dim, int num_splits)
{
    if ((int64_t)num_splits * rows_pad * head_dim * 2 > 0xffffffffll) return true;
    return num_splits <= kMergeRowPieces && total_rows * head_dim >= (n_kv_heads % kNumXcd == 0 ? 3 : 7) * kNumCu * 128ll;
}

// A thread's splits, all requested together: the fewest of these sizes that cover them.  (A split that is not there is a load
// of a line that is, yet eight where four do cost 0.2 us: 48 splits of 6000 keys, 28/4 heads 8.95 us a layer instead of 8.75.)
// With several workgroups to a CU it is their work that counts and not one's round trip: rounds of four, and no load for a split that is not
// there, of which the short requests of a batch have most (us a layer, all together / this:  64/8 heads, 8 queries, 8 requests of which one has 12800
// keys in 100 splits and the others 200 66.2 / 54.9, 8192 in 64 45.7 / 40.6, 5120 in 40 31.4 / 30.8;  28/4 heads, 12800 39.8 / 34.9;  equal requests the same).
template <int D>
static int launch_merge(const AttnParams& p, dim3 grid, hipStream_t stream)
{
    constexpr int THREADS = kMergeGroups * (D / 4), MOST = (kMaxSplits + kMergeGroups - 1) / kMergeGroups;
    const int each = (p.num_splits + kMergeGroups - 1) / kMergeGroups;
    if (each <= 3)                         hipLaunchKernelGGL((attn_merge_kernel<D, 3, THREADS, false>), grid, dim3(THREADS), 0, stream, p);
    else if (grid.x > 2u * kNumCu)         hipLaunchKernelGGL((attn_merge_kernel<D, 4, THREADS, true>), grid, dim3(THREADS), 0, stream, p);
    else if (each <= 4)                    hipLaunchKernelGGL((attn_merge_kernel<D, 4, THREADS, false>), grid, dim3(THREADS), 0, stream, p);
    else if (each <= 8)                    hipLaunchKernelGGL((attn_merge_kernel<D, 8, THREADS, false>), grid, dim3(THREADS), 0, stream, p);
    else if (each <= 16)                   hipLaunchKernelGGL((attn_merge_kernel<D, 16, THREADS, false>), grid, dim3(THREADS), 0, stream, p);
    else                                   hipLaunchKernelGGL((attn_merge_kernel<D, MOST, THREADS, false>), grid, dim3(THREADS), 0, stream, p);
    return launch_status();
}

template <int D, int MB, int KS, int TK, int NS, int NLD, bool STREAM>
static int launch_attn_s(const AttnParams& p, hipStream_t stream)
{
    constexpr int NW = MB * KS;
    constexpr size_t ring = (size_t)NS * 2 * TK * D * 2;
    constexpr size_t merge = sizeof(float) * (size_t)(2 * NW * 16 + NW * 16 * (D + 4));
    constexpr size_t lds = ring > merge ? ring : merge;
    if (lds > 64 * 1024)
        if (const int rc = allow_lds<&attn_split_kernel<D, MB, KS, TK, NS, NLD, STREAM>>((int)lds)) return rc;
    hipLaunchKernelGGL((attn_split_kernel<D, MB, KS, TK, NS, NLD, STREAM>), dim3(p.n_work), dim3((NW + NLD) * kWave),
                       lds, stream, p);
    return launch_status();
}

template <int D, int NW, int CH, int COLS>
static int launch_short(const AttnParams& p, hipStream_t stream)
{
    constexpr size_t lds = (size_t)NW * (kChunkKeys * (D + COLS) * 2 + 2 * 16 * sizeof(float));
    if (lds > 64 * 1024)
        if (const int rc = allow_lds<&attn_short_kernel<D, NW, CH, COLS>>((int)lds)) return rc;
    hipLaunchKernelGGL((attn_short_kernel<D, NW, CH, COLS>), dim3(p.n_work), dim3(NW * kWave), lds, stream, p);
    return launch_status();
}

// Waves of a workgroup without splits: eight, or sixteen with half the keys each where a wave of eight would have many.  The
// loads take as long either way, but less is left to do behind the last of them (us a layer, eight / sixteen).  Size 64: 14/2
// heads, 1400 keys 6.34 / 6.12, 26 nodes 7.07 / 6.82, 1500 keys 6.35 / 6.23, 26 nodes 6.60 / 6.65, 1281 keys 6.07 / 6.04, but 1200
// keys 5.69 / 5.99 (half a wave's keys are past the end), 1000 keys 5.27 / 5.40;  size 128, 64/8 heads, 6 queries: 672 keys
// 6.14 / 6.49, 700 6.68 / 6.56, 768 6.65 / 6.69, 800 7.25 / 7.16, 850 7.13 / 7.29, 900 8.03 / 7.54, 1024 8.16 / 7.71;  40/8, 1 query:
// 641 keys 5.65 / 6.01, 768 6.04 / 6.12, 800 6.68 / 6.56, 900 7.01 / 6.76;  28/4, 16 queries: 672 6.40 / 6.57, 800 7.55 / 7.23.
static bool attn_direct_16_waves(int head_dim, int kv_len) { return kv_len > (head_dim == 64 ? 1280 : 768); }

static int launch_attn_direct(const AttnParams& p, int head_dim, int chunks, hipStream_t stream)
{
    if (attn_direct_16_waves(head_dim, p.kv_len))
        return head_dim == 64 ? launch_short<64, 2 * kDirectWaves, 3, 16>(p, stream) : launch_short<128, 2 * kDirectWaves, 2, 16>(p, stream);
    if (head_dim == 64) {
        switch (chunks) {
            case 1: return launch_short<64, kDirectWaves, 1, 16>(p, stream);
            case 2: return launch_short<64, kDirectWaves, 2, 16>(p, stream);
            case 3: return launch_short<64, kDirectWaves, 3, 16>(p, stream);
            case 4: return launch_short<64, kDirectWaves, 4, 16>(p, stream);
            case 5: return launch_short<64, kDirectWaves, 5, 16>(p, stream);
        }
    } else {
        switch (chunks) {
            case 1: return launch_short<128, kDirectWaves, 1, 16>(p, stream);
            case 2: return launch_short<128, kDirectWaves, 2, 16>(p, stream);
            case 3: return launch_short<128, kDirectWaves, 3, 16>(p, stream);
        }
    }
    return SPECVLM_EUNSUPPORTED;
}

// From this size per launch on, the cache is streamed with non-temporal loads: its lines would
// only push the split partials (which the merge re-reads) and other reusable data out of the L2.
// Smaller caches (a draft's pruned cache, re-read at every decode step) stay cacheable.
constexpr int64_t kStreamBytes = 8ll << 20;
static bool attn_streams(const AttnParams& p, int head_dim) { return 4ll * p.batch * p.n_kv_heads * p.kv_len * head_dim >= kStreamBytes; }

template <int D, int MB, int KS, int TK, int NS, int NLD>
static int launch_attn(const AttnParams& p, hipStream_t stream)
{
    return attn_streams(p, D) ? launch_attn_s<D, MB, KS, TK, NS, NLD, true>(p, stream)
                                    : launch_attn_s<D, MB, KS, TK, NS, NLD, false>(p, stream);
}

// One block of query rows: two waves that compute and two that load, or four that do both.  The first keep more bytes in flight and win
// where the memory is what splits of 128 keys and more wait for (us a layer, four waves / roles):  size 128:  28/4 heads 6000 keys (splits of
// 128) 8.55 / 8.35, 8000 10.3 / 9.55, 30000 17.05 / 15.35, 120000 48.1 / 42.4;  64/8 heads 6000 10.45 / 10.0, 12000 14.55 / 13.35, 30000 26.9 / 23.85,
// 120000 87.6 / 77.3;  size 64:  14/2 heads 30000 9.65 / 8.6, 120000 18.9 / 15.45;  balanced pieces of size 128, 16 requests of up to 2500 keys, 40/8
// heads 26.3 / 25.1, 28/4 of up to 6000, 4 of them 18.0 / 17.3.  Left out is what loses:
//   splits of fewer keys (28/4 heads, 3000 keys, splits of 125 7.6 / 7.95) and caches below the streamed size, which stay near and whose launches are
//     bound by their start and their steps:  size 128, 7/1 heads, 1024 keys in 8 splits 6.45 / 7.0, 4096 in 32 7.15 / 7.5 (but 16384 in 32, 8 MB, 11.65 /
//     10.5);  size 64, 4/1 heads, 3072 in 8 6.7 / 7.2, 14/2 heads 12288 in 32 7.5 / 7.8 (16384, 8 MB, 9.2 / 8.7).  Splits of 700 keys of size 128 and
//     more, which a caller can name, are no start any more: 7/1 heads, 3590 in 3 14.9 / 14.0, 15719 in 5 43.8 / 34.3, from near caches 2 to 5 %
//     faster;  of size 64 they are from far ones (4/1 heads, 30637 in 20 17.9 / 13.9) and 11 to 16 % slower from near ones, and stay with four waves;
//   more workgroups of size 64 than CUs in one round, where two of the four waves' workgroups share a CU:  8/4 heads, 65 requests of 1500 keys 25.4 / 26.5,
//     8 of 3200 in 16 splits 10.5 / 10.7 (in several rounds a third workgroup shares it: 16/8 heads, 40 of 1280 in 8 35.7 / 30.3, 65 of 600 23.5 / 21.1);
//   splits of 256 keys, eight heads and more, in two rounds and more: the four waves have all of a split in flight at once, and lines of 512 KB strides:
//     64/8 heads, 32768 keys in 128 34.3 / 35.8, 65 requests of 256 23.6 / 24.0 (splits of 250 34.4 / 33.2 and of 272 38.6 / 35.5);
//   balanced pieces of size 64 (4/1 heads 12.6 / 13.7).
static bool attn_has_loaders(const AttnParams& p, int head_dim)
{
    if (!attn_streams(p, head_dim)) return head_dim == 128 && !p.balanced && p.split_keys >= 700;
    if (p.balanced) return head_dim == 128;
    if (p.split_keys < 128) return false;
    if (head_dim == 64) return p.n_work <= kNumCu || p.n_work > 2 * kNumCu;
    return !(p.split_keys == 256 && p.n_kv_heads % kNumXcd == 0 && p.n_work >= 2 * kNumCu);
}

// Ring depth of head size 64, whose tiles are half as large: a fourth stage keeps 16 KB more in flight where a workgroup has its CU to itself
// and tiles to come (us a layer, three stages / four, by query rows of a kv head):  14/2 heads, 100000 keys, 7 rows 14.3 / 14.1, 21 rows 14.9 / 14.5,
// 42 rows 15.45 / 14.9, 56 rows 15.65 / 15.2;  10/5 heads, 8 rows 26.9 / 25.3.  It leaves a CU two workgroups instead of three, and it is no gain where
// the memory is busy anyway:
//   balanced pieces:  8/4 heads, 48 rows, 5 requests of up to 20000 keys 22.7 / 23.1;  16/8, 40 rows, 8 of up to 3000 16.1 / 16.4;
//   eight heads in one round whose keys lie side by side for all of them, where the heads' workgroups walk the same pages at once:  16/8 heads, 2 rows, 20012
//     keys 13.2 / 13.6, 42214 22.4 / 23.1 (a head's keys side by side: 17329 11.7 / 11.3, 37883 18.6 / 17.8, 50652 in 6 splits 56.3 / 47.6;  row groups,
//     which share their keys, either way: 100 rows 23.0 / 22.6);
//   short splits in nearly as many workgroups as CUs:  trees of 14/2 heads, 280 rows, 12000 keys (splits of 286) 11.3 / 11.5, 30000 keys 18.4 / 17.8;
//   more workgroups than CUs:  14/2 heads, 42 rows, 65 requests of 1500 keys 18.7 / 19.6, 8 of 8000 in 32 splits 13.2 / 13.8;  8/4, 48 rows, 65 of 300
//     9.5 / 10.4.  In several rounds of long splits it wins again: 8/4, 16 rows, 128 of up to 3000 keys 61.0 / 54.3, 64 rows 67.7 / 65.3.
static bool attn_has_deep_ring(const AttnParams& p)
{
    const bool rounds = p.n_work > 2 * kNumCu;
    if (p.balanced || (p.n_work > kNumCu && !rounds)) return false;
    if (!rounds && p.n_kv_heads % kNumXcd == 0 && p.n_rgroups == 1 && p.kv_head < p.kv_tok) return false;
    return 5 * p.n_work <= 4 * kNumCu || p.split_keys >= 640;
}

template <int D>
static int launch_attn_d(const AttnParams& p, int mb, hipStream_t stream)
{

    // (key-split waves, tile keys, ring depth, loader waves) per row-block count; the ring holds NS * 2 * TK * D * 2 bytes of LDS
    constexpr int DEEP = D == 64 ? 4 : 3;
    const bool deep = D == 64 && attn_has_deep_ring(p);
    switch (mb) {
        case 1:
            // Splits of at most 128 keys: one chunk of 32 keys for each of four waves, results for the merge (a single split
            // writes output).  Us a layer, ring / this:  14/2 heads 2000 keys 7.2 / 6.9, 12000 10.0 / 9.6;  7/1 heads 24000 keys
            // 12.8 / 12.5;  named splits 12/4 heads, 256 of 32768 keys 20.2 / 18.6, 4 requests of 14/2 heads, 128 splits of 16384
            // keys 18.2 / 15.5.  Left out is what loses: one request of eight heads, a head an XCD, with 128 splits and more
            // (16384 keys token-major 15.0 / 15.5, 24000 in 256 splits 19.1 / 19.9; 96 splits of 12288 keys win 10 %).
            if constexpr (D == 64) {
                const bool loses = p.batch == 1 && p.n_kv_heads == kNumXcd && p.num_splits >= 128;
                if (p.num_splits > 1 && p.split_keys <= kShortWaves * kChunkKeys && !p.balanced && !loses)
                    return launch_short<D, kShortWaves, 1, D>(p, stream);
            }
            if (attn_has_loaders(p, D)) {
                if constexpr (D == 128) return launch_attn<D, 1, 2, 64, 3, 2>(p, stream);
                return deep ? launch_attn_s<D, 1, 2, 64, DEEP, 2, true>(p, stream) : launch_attn_s<D, 1, 2, 64, 3, 2, true>(p, stream);
            }
            return launch_attn<D, 1, 4, 128, 2, 0>(p, stream);
        case 2: return deep ? launch_attn<D, 2, 2, 64, DEEP, 4>(p, stream) : launch_attn<D, 2, 2, 64, 3, 4>(p, stream);
        // (two loaders: 16.7 against 17.0 us with four)
        case 3: return deep ? launch_attn<D, 3, 2, 64, DEEP, 2>(p, stream) : launch_attn<D, 3, 2, 64, 3, 2>(p, stream);
        // (four loaders: 64 rows, 12000 keys, 64/8 heads 15.2, with two 15.8)
        case 4: return deep ? launch_attn<D, 4, 2, 64, DEEP, 4>(p, stream) : launch_attn<D, 4, 2, 64, 3, 4>(p, stream);
    }
    return SPECVLM_EUNSUPPORTED;
}

}  // namespace specvlm

using namespace specvlm;

extern "C" size_t specvlm_decode_attn_workspace_bytes(int batch, int q_len, int kv_len,
                                                      int n_q_heads, int n_kv_heads, int head_dim,
                                                      int num_splits)
{
    if (batch <= 0 || q_len <= 0 || kv_len <= 0 || n_kv_heads <= 0 || n_q_heads <= 0 ||
        n_q_heads % n_kv_heads || (head_dim != 64 && head_dim != 128))
        return 0;
    const int rows = (n_q_heads / n_kv_heads) * q_len;
    if (q_len > kMaxQueryBlock) return 0;
    // (a launch without splits uses none of it, but asks for it all the same: what is enough for a shape stays enough for
    // every smaller one, whichever launch that takes)
    int n_rgroups, mb;
    attn_row_groups(rows, &n_rgroups, &mb);
    const int rows_pad = n_rgroups * mb * 16;
    size_t slots;
    if (attn_is_balanced(batch, num_splits, n_kv_heads, rows)) {
        slots = (size_t)(kNumCu + batch * n_kv_heads) * rows_pad;
        return align256(slots * head_dim * sizeof(__bf16)) + align256(slots * 2 * sizeof(float)) +
               align256((size_t)batch * n_kv_heads * 2 * sizeof(int32_t));
    } else {
        const int splits = choose_splits(batch, kv_len, n_kv_heads, n_rgroups, num_splits);
        if (splits == 1) return 256;
        slots = (size_t)batch * n_kv_heads * splits * rows_pad;
    }
    return align256(slots * head_dim * sizeof(__bf16)) + align256(slots * 2 * sizeof(float));
}

static int attn_impl(
    const void* q, int64_t q_tok_stride, int64_t q_head_stride,
    const void* k, const void* v, int64_t kv_tok_stride, int64_t kv_head_stride,
    const int32_t* cu_q, const int32_t* cu_kv, int batch, int q_len, int kv_len,
    int n_q_heads, int n_kv_heads, int head_dim, float softmax_scale,
    const uint64_t* block_mask, void* out, float* lse, int num_splits,
    void* workspace, size_t workspace_bytes, void* stream)
{
    if (batch < 0 || q_len < 0 || kv_len < 0 || n_q_heads <= 0 || n_kv_heads <= 0) return SPECVLM_EINVAL;
    if (n_q_heads % n_kv_heads) return SPECVLM_EINVAL;
    if ((cu_q == nullptr) != (cu_kv == nullptr)) return SPECVLM_EINVAL;
    if (!cu_q && batch > 1) return SPECVLM_EINVAL;
    if (!(softmax_scale >= 0.f) || !(softmax_scale < INFINITY)) return SPECVLM_EINVAL;
    if (num_splits < 0) return SPECVLM_EINVAL;
    if (head_dim != 64 && head_dim != 128) return SPECVLM_EUNSUPPORTED;
    if (batch == 0 || q_len == 0) return SPECVLM_OK;
    if (q_len > kv_len) return SPECVLM_EINVAL;
    if (!q || !k || !v || !out) return SPECVLM_EINVAL;
    if ((q_tok_stride | q_head_stride | kv_tok_stride | kv_head_stride) & 7) return SPECVLM_EUNSUPPORTED;
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)out) & 15) return SPECVLM_EUNSUPPORTED;
    const int group = n_q_heads / n_kv_heads;
    const int rows = group * q_len;
    if (q_len > kMaxQueryBlock) return SPECVLM_EUNSUPPORTED;
    // per-lane key offsets are 32-bit byte offsets from the request's first row
    if (kv_tok_stride <= 0 || (int64_t)kv_len * kv_tok_stride * 2 >= ((int64_t)1 << 32))
        return SPECVLM_EUNSUPPORTED;
    int n_rgroups, mb;
    attn_row_groups(rows, &n_rgroups, &mb);

    AttnParams p;
    p.q = (const __bf16*)q; p.k = (const __bf16*)k; p.v = (const __bf16*)v;
    p.out = (__bf16*)out; p.lse = lse;
    p.q_tok = q_tok_stride; p.q_head = q_head_stride;
    p.kv_tok = kv_tok_stride; p.kv_head = kv_head_stride;
    p.cu_q = cu_q; p.cu_kv = cu_kv; p.block_mask = block_mask;
    p.batch = batch; p.q_len = q_len; p.kv_len = kv_len;
    p.n_q_heads = n_q_heads; p.n_kv_heads = n_kv_heads; p.group = group;
    p.scale_log2 = softmax_scale * kLog2e;
    p.inv_heads = reciprocal(n_kv_heads); p.inv_all_heads = reciprocal(batch * n_kv_heads); p.inv_group = reciprocal(group);
    p.balanced = attn_is_balanced(batch, num_splits, n_kv_heads, rows) ? 1 : 0;
    p.max_wg = kNumCu;
    p.num_splits = p.balanced ? 2 : choose_splits(batch, kv_len, n_kv_heads, n_rgroups, num_splits);
    p.split_keys = (kv_len + p.num_splits - 1) / p.num_splits;
    p.rows_pad = n_rgroups * mb * 16;
    p.n_rgroups = n_rgroups;
    p.n_work = p.balanced ? p.max_wg : batch * n_kv_heads * p.num_splits * n_rgroups;
    p.inv_splits = reciprocal(p.num_splits); p.inv_split_keys = reciprocal(p.split_keys); p.inv_help = 0; p.inv_rgroups = reciprocal(n_rgroups);
    p.part_o = nullptr; p.part_ml = nullptr; p.seg_table = nullptr;
    if (p.num_splits > 1) {
        const size_t need = specvlm_decode_attn_workspace_bytes(batch, q_len, kv_len, n_q_heads,
                                                                n_kv_heads, head_dim, num_splits);
        if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < need) return SPECVLM_EWORKSPACE;
        const size_t slots = p.balanced ? (size_t)(p.max_wg + batch * n_kv_heads) * p.rows_pad
                                        : (size_t)batch * n_kv_heads * p.num_splits * p.rows_pad;
        p.part_o = (__bf16*)workspace;
        p.part_ml = (float*)((char*)workspace + align256(slots * head_dim * sizeof(__bf16)));
        p.seg_table = (int32_t*)((char*)p.part_ml + align256(slots * 2 * sizeof(float)));   // (used in balanced mode)
    }
    hipStream_t s = (hipStream_t)stream;
    if (const int chunks = attn_direct_chunks(batch, kv_len, n_kv_heads, head_dim, rows, num_splits)) {
        p.n_rgroups = (rows + 15) / 16;
        p.inv_rgroups = reciprocal(p.n_rgroups);
        p.n_main = batch * n_kv_heads * p.n_rgroups * (head_dim / 16);
        const int threads = (attn_direct_16_waves(head_dim, kv_len) ? 2 : 1) * kDirectWaves * kWave;
        int helpers = (kv_len * (head_dim / 8) + threads - 1) / threads;
        if (helpers > kPrefetchers) helpers = kPrefetchers;
        // (sixteen waves' LDS leaves a CU no second workgroup: a helper that finds none free would run when all is over; 64/8 heads, 8
        // queries, 700 keys 7.43 us a layer with all 120 of them, 6.93 with none, 7.02 with eight waves and 120)
        if (threads > kDirectWaves * kWave && helpers > (kNumCu - p.n_main) / kNumXcd) helpers = (kNumCu - p.n_main) / kNumXcd;
        p.n_work = p.n_main + (batch == 1 ? kNumXcd * helpers : 0);
        if (p.n_work > p.n_main) p.inv_help = reciprocal((p.n_work - p.n_main) / kNumXcd);
        return launch_attn_direct(p, head_dim, chunks, s);
    }
    int rc = head_dim == 128 ? launch_attn_d<128>(p, mb, s) : launch_attn_d<64>(p, mb, s);
    if (rc != SPECVLM_OK) return rc;
    if (p.balanced || (p.num_splits > 1 &&
                       attn_merges_by_row(n_kv_heads, batch * n_kv_heads * (int64_t)rows, p.rows_pad, head_dim, p.num_splits))) {
        const int per_wg = 256 / (head_dim / 4);
        dim3 grid((rows + per_wg - 1) / per_wg * batch * n_kv_heads);
        if (head_dim == 128) hipLaunchKernelGGL((attn_merge_rows_kernel<128, kMergeRowPieces>), grid, dim3(256), 0, s, p);
        else                 hipLaunchKernelGGL((attn_merge_rows_kernel<64, kMergeRowPieces>), grid, dim3(256), 0, s, p);
        rc = launch_status();
    } else if (p.num_splits > 1) {
        dim3 grid(rows * batch * n_kv_heads);
        rc = head_dim == 128 ? launch_merge<128>(p, grid, s) : launch_merge<64>(p, grid, s);
    }
    return rc;
}

extern "C" int specvlm_decode_attn(
    const void* q, int64_t q_tok_stride, int64_t q_head_stride,
    const void* k, const void* v, int64_t kv_tok_stride, int64_t kv_head_stride,
    const int32_t* cu_q, const int32_t* cu_kv, int batch, int q_len, int kv_len,
    int n_q_heads, int n_kv_heads, int head_dim, float softmax_scale,
    void* out, float* lse, int num_splits,
    void* workspace, size_t workspace_bytes, void* stream)
{
    return attn_impl(q, q_tok_stride, q_head_stride, k, v, kv_tok_stride, kv_head_stride, cu_q, cu_kv,
                     batch, q_len, kv_len, n_q_heads, n_kv_heads, head_dim, softmax_scale, nullptr,
                     out, lse, num_splits, workspace, workspace_bytes, stream);
}

// ---- the variant that takes no workspace ----
// Scratch for callers that cannot allocate or pass one (code under HIP graph capture, serving loops
// that own no spare device memory).  Every device that loads the library holds its own copy of this
// array until the process ends; the name below is a host-side handle, the device address is looked
// up once per device.
constexpr size_t kStaticScratchBytes = 16u << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

static std::atomic<void*> g_scratch_ptr[kMaxDevices];

static int static_scratch(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SPECVLM_ELAUNCH;
    void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!ptr) {
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return SPECVLM_ELAUNCH;
        g_scratch_ptr[dev].store(ptr, std::memory_order_release);   // (every thread looks up the same address)
    }
    *out = ptr;
    return SPECVLM_OK;
}

extern "C" size_t specvlm_decode_attn_static_scratch_bytes(void) { return kStaticScratchBytes; }

extern "C" int specvlm_decode_attn_static(
    const void* q, int64_t q_tok_stride, int64_t q_head_stride,
    const void* k, const void* v, int64_t kv_tok_stride, int64_t kv_head_stride,
    const int32_t* cu_q, const int32_t* cu_kv, int batch, int q_len, int kv_len,
    int n_q_heads, int n_kv_heads, int head_dim, float softmax_scale,
    void* out, float* lse, int num_splits, void* stream)
{
    // the shape decides how much scratch the kernels use; a shape the array cannot hold is refused
    // (a shape the workspace query itself rejects, size 0, is left to the argument checks below)
    const size_t need = specvlm_decode_attn_workspace_bytes(batch, q_len, kv_len, n_q_heads, n_kv_heads,
                                                            head_dim, num_splits);
    if (need > kStaticScratchBytes) return SPECVLM_EWORKSPACE;
    void* ptr = nullptr;
    const int rc = static_scratch(&ptr);
    if (rc != SPECVLM_OK) return rc;
    return attn_impl(q, q_tok_stride, q_head_stride, k, v, kv_tok_stride, kv_head_stride, cu_q, cu_kv,
                     batch, q_len, kv_len, n_q_heads, n_kv_heads, head_dim, softmax_scale, nullptr,
                     out, lse, num_splits, ptr, kStaticScratchBytes, stream);
}

extern "C" int specvlm_tree_attn(
    const void* q, int64_t q_tok_stride, int64_t q_head_stride,
    const void* k, const void* v, int64_t kv_tok_stride, int64_t kv_head_stride,
    const int32_t* cu_q, const int32_t* cu_kv, int batch, int q_len, int kv_len,
    int n_q_heads, int n_kv_heads, int head_dim, float softmax_scale,
    const uint64_t* ancestor_mask, void* out, float* lse, int num_splits,
    void* workspace, size_t workspace_bytes, void* stream)
{
    if (!ancestor_mask && batch > 0 && q_len > 0) return SPECVLM_EINVAL;
    if (q_len > 64) return SPECVLM_EUNSUPPORTED;
    return attn_impl(q, q_tok_stride, q_head_stride, k, v, kv_tok_stride, kv_head_stride, cu_q, cu_kv,
                     batch, q_len, kv_len, n_q_heads, n_kv_heads, head_dim, softmax_scale, ancestor_mask,
                     out, lse, num_splits, workspace, workspace_bytes, stream);
}
