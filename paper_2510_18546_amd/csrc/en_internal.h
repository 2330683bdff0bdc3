// Internal declarations shared by the host planner and the HIP kernels of
// libefficientnav.so. Not part of the public ABI (that is include/efficientnav.h).
#pragma once

#include <cstddef>
#include <cstdint>
#include <new>
#include <utility>
#include <vector>

#include <hip/hip_runtime_api.h>

#include "efficientnav.h"

constexpr size_t EN_LAST_LEVEL_CACHE_BYTES = size_t(256) << 20;
constexpr size_t EN_GATHER_HUGE_BYTES = 3 * EN_LAST_LEVEL_CACHE_BYTES;      // of a context's keys and values
constexpr int EN_XCDS = 8;         // dies of the chip, each with an L2 of its own; workgroups are dealt out over them in turn
constexpr size_t EN_GRID_MAX = ((size_t(1) << 32) - 1) / 256;      // workgroups of 256 along x: a launch counts threads in 32 bits
constexpr int EN_KEY_TILE = 64;    // keys per attention tile; context rows are padded to it
constexpr int EN_ROWS_PER_WAVE = 32;
constexpr int EN_WAVES = 8;          // waves per attention workgroup
constexpr int EN_F32_ROWS = 16;      // query rows per workgroup of the fp32 attention kernel
constexpr int EN_ONCE_ROWS = 16;     // query rows per KV head of attn_once_kernel at most
constexpr int EN_ONCE_TILES = 5;     // key tiles of a split there at most (32 KB of LDS each with D = 128)

struct en_pool {
    en_pool_desc d;
    void *k_dev = nullptr;
    void *v_dev = nullptr;
    float *k_scale = nullptr;     // EN_I8 pools: one scale per (group, head, token)
    float *v_scale = nullptr;
    std::vector<int32_t> len;     // current lengths [G]
    int r = 1;                    // Hq / Hkv
    // device side, created on first GPU use
    float *d_cos = nullptr;       // [max_ctx, D/2]
    float *d_sin = nullptr;
    int n_cu = 256;               // compute units, from the pool's creation on
    // descriptor blocks of destroyed plans, kept for reuse (bytes, pointer)
    mutable std::vector<std::pair<size_t, int32_t *>> desc_cache;
    // plans made on this pool and not yet destroyed: a pool that is destroyed
    // first cuts them loose, so that destroying them later stays safe
    mutable std::vector<struct en_plan *> plans;
    // measurement aid (en_timing_*): event pairs around the attention kernel of the calls on this pool
    std::vector<hipEvent_t> ev_start, ev_stop;
    int ev_used = 0;
};

struct en_plan {
    const en_pool *pool = nullptr;
    int B = 0, Nq = 0, Smax = 0;
    int ctx_stride = 0, max_ctx_len = 0, n_splits = 1;
    bool splits_set = false;      // by en_plan_set_splits
    int64_t total_pairs = 0, total_cached = 0;
    int64_t selected = 0, distinct = 0;      // groups that at least one agent selects, their tokens
    // host descriptors (uniform stride per agent)
    std::vector<int32_t> nseg;    // [B]
    std::vector<int32_t> sel;     // [B, Smax]   (-1 padded)
    std::vector<int32_t> bnd;     // [B, Smax+2] bucket bounds: offset[0..S], then L_c+N_q
    std::vector<int32_t> hdr;     // [B, 4] S, L_c, L_c+N_q, 0: what a workgroup needs first, in one load
    // length of EnGatherArgs::order, or 0; its entries are up to 1 << order_shift tiles
    size_t order_ints = 0;
    int order_shift = 0;
    // device block: nseg | sel | bnd | hdr | order, created on first GPU use
    int32_t *d_desc = nullptr;
    size_t d_desc_bytes = 0;
    std::vector<int32_t> h_desc;  // staging copy, alive as long as the plan
    bool uploaded = false;
    // behind the tables in the device block: B * (Smax + 1) 64-bit accumulators of the reduced masses
    // that the prefill attention kernel adds up itself (EnAttnArgs::red_direct). Zero when the block is
    // filled; whoever completes a sum sets its word back to zero.
    size_t acc_off = 0;           // in ints from d_desc
    // en_plan_values_from_pool: the gather leaves the values where they are (EnGatherArgs::v_rows)
    bool values_from_pool = false;
    int gathered_values_from_pool = -1;      // mode of the last gather on this plan, -1: none yet
};

// Arguments of the device kernels (plain data, passed by value).
struct EnGatherArgs {
    const void *k_pool, *v_pool, *k_new, *v_new;
    void *kc, *vt;
    const float *cos_tab, *sin_tab;
    const int32_t *nseg, *sel, *bnd;
    int B, Hkv, C, Nq, Smax, T;
    const float *k_scale, *v_scale;    // EN_I8 pools only
    // queries to prepare in the same launch, or null: q [B, Nq, Hq, D] unrotated ->
    // q_prep, rotated at L_c + i, scaled by scale_log2e, bf16
    const void *q;
    void *q_prep;
    int Hq;
    // units (along grid y) that share an agent's query rows with the 64-token tiles along x: a
    // workgroup takes its rows 16 at a time, one dependent round of loads each, so few rows per
    // workgroup keep the query units from outlasting the key and value streams of a small step
    int n_q_units;
    float scale_log2e;
    // 1 (bf16, D = 128): the values stay where they are. vt receives, per (agent, KV head, context
    // row up to the end of the last 64-row tile), the 8-byte address of the row's values in the
    // pool or the new tokens, [B, Hkv, T], and behind that table one row of zeros, which the
    // padding rows of an agent's last tile point at.
    int v_rows;
    // Order in which the tiles are gathered, or null (tile by tile along x, agent by agent along z): entries
    // {agent, first tile << 2 | tiles - 1} (agent -1: none) in lists per XCD, list X at X, X + EN_XCDS, ...
    const int32_t *order;
    int order_shift;
    int rope_unit;         // en_rope_unit
    // 1: the context is written past the caches (non-temporal stores). Contexts beyond the 256 MB of the
    // last-level cache are not there any more when the attention kernel comes to read them, and its lines
    // in the way cost the gather 3 % (64 agents x 16 K tokens, 4.3 GB: 1473 -> 1438 us); a smaller one is
    // read back from the cache (16 agents x 2 K tokens, 133 MB: the gather gains 13 us that way, the
    // attention kernel loses 12; one agent's 36 MB: the step gets 2.5 us longer). With rows of 64 values the
    // gather itself loses (64 agents x 16 K tokens, 8 heads 648 -> 674 us, 2 heads 188 -> 194), the attention
    // behind it gains more (together 1063 -> 1028, 358 -> 314). Plans that leave their values in the pool write
    // half as much, but the attention kernel then reads the pool's values beside the keys: the line is the same
    // one, twice the keys (9 agents x 8 K tokens, keys of 146 MB, gather and attention: 247 us kept in the caches,
    // 241 past them; 12 agents 195 MB: 305, 297; 15 agents 243 MB: 337, 329). From 8-bit pools, one head a workgroup:
    // 32 agents x 6 K tokens 501 -> 417, 16 x 14 K 582 -> 516, 64 x 16 K 2319 -> 2280, rows of 64 values 1220 -> 943.
    int stream;
};

// Bytes of the row-address table of EnGatherArgs::v_rows (the row of zeros follows it).
constexpr size_t en_v_rows_table_bytes(int B, int Hkv, int T)
{
    return ((size_t)B * Hkv * T * 8 + 255) / 256 * 256;
}

// The gather launch can carry a small plan's descriptor block inside its kernel
// arguments: the kernel reads the descriptors from there and one workgroup
// stores them to the plan's device block for the kernels that follow, which
// saves the separate host-to-device copy.
constexpr int EN_INLINE_DESC_MAX = 960;      // ints; keeps the argument block under 4 KB
struct EnGatherLaunch {
    EnGatherArgs a;
    int n_inline;           // ints of `desc` in use, 0: read the device block
    int n_zero;             // ints to set to zero behind them in the device block (the plan's accumulators)
    int32_t *desc_out;      // device block to fill when n_inline > 0
    int32_t desc[EN_INLINE_DESC_MAX];
};
// What every workgroup reads before its tables lies in the first three lines (of 64 bytes) of the arguments: a field in
// the fourth is one more trip before the tables' own (the gather of 64 fp32 rows 3.22 -> 3.32 us, of one agent's ragged
// map 5.59 -> 5.71). So what the host alone needs is not among them.
static_assert(offsetof(EnGatherLaunch, desc_out) <= 192, "a field that every workgroup reads is in the fourth line");

// A divisor of the attention kernels' workgroup and split numbers. An integer division by a run-time value is some thirty
// instructions one after the other, and eight of them stood in front of a workgroup's first load; this is three:
// x / n = x mul >> (31 + shift) for all x < 2^31, with shift = ceil(log2 n) and mul = ceil(2^(31 + shift) / n) < 2^32: mul n
// is less than n <= 2^shift above 2^(31 + shift), so the product is less than 1 / n of 2^(31 + shift) above x / n.
struct EnDivisor {
    unsigned n, mul, shift;      // (shift: 31 + ..)
};
inline EnDivisor en_divisor(unsigned n)
{
    unsigned s = 0;
    while ((1ull << s) < n)
        ++s;
    return {n, unsigned(((1ull << (31 + s)) + n - 1) / n), 31 + s};
}

struct EnAttnArgs {
    const void *q, *kc, *vt;
    void *out;
    const float *cos_tab, *sin_tab;
    const int32_t *nseg, *bnd, *hdr;
    float *ws_ml;      // [n_splits, B*Hq*Nq, 2]  (reference max in log2 units, sum)
    float *ws_seg;     // [n_splits, B*Hq, Smax+1, Nq, 2] (partial sum, its reference max)
    void *ws_opart;    // [n_splits, B*Hq*Nq, D] per-split softmax outputs (pool dtype)
    float *ws_mlfin;   // [B*Hq*Nq, 2] merged (reference, sum), written by the combine kernel
    int B, Hq, Hkv, Nq, Smax, T;
    int q_first;       // the Nq query rows are new tokens q_first .. q_first+Nq-1 of the plan: every key
                       // before L_c + q_first is visible to all of them (0 for a whole prefill)
    int n_splits, n_ptiles, total_wgs;
    // attention kernels: n_ptiles, n_splits (of workgroup numbers and of split boundaries), Hkv, Hq / Hkv
    EnDivisor by_ptiles, by_splits, by_hkv, by_r;
    EnDivisor by_nq, by_hq;      // merge, attn_once_kernel: Nq, Hq
    // the header {S, L_c} of the only agent (B == 1): one trip to memory less in front of its first load
    int one_S, one_Lc;
    int decode;        // 1: all r*Nq query rows of a KV head fit one wave (attn_decode kernel)
    int sub;           // decode kernel: waves per (agent, KV head, split); wave w takes every sub-th 32-key
                       // block of the split's tiles and leaves its own partial results at index
                       // sp * sub + w of n_splits * sub
    float scale_log2e;
    // fp32 kernel: waves per workgroup, 8 or 2. Eight share the keys of few workgroups, which wait for memory; where
    // two and more workgroups per compute unit and at most 1 K keys per split come together, most of the eight
    // have little or nothing to do and starting and merging them is what the launch takes (16 heads, a row each:
    // 256 agents x 33 keys 64.6 us with eight, 31.9 with two; x 513 keys 227, 208; 64 agents x 1025 keys 103, 98;
    // x 4097 keys 371, 372; 16 agents x 129 keys 8.1, 11.0).
    int f32_waves;
    // decode steps, or 0: the most 64-key tiles of a split, all of them in LDS at once (attn_once_kernel)
    int once_tiles;
    int q_prepared;    // prefill kernel: q holds prepared queries (rotated, scaled, bf16: see EnGatherArgs)
    int v_rows;        // prefill kernel: vt holds no values but the address of every context row's values
                       // (see EnGatherArgs::v_rows)
    // prefill and fp32 kernels, or null: n_red_zero accumulator words that their first workgroup sets to
    // zero (EnMassArgs::red_acc, which the launches after it add to)
    unsigned long long *red_zero;
    int n_red_zero;
    // prefill kernel with one KV split, or null: the reduced masses [B, Smax+1] without any further
    // launch. Every workgroup adds, per bucket, the masses of its rows to red_direct (fixed point,
    // 2^-red_shift, above a 10-bit count of arrivals, as in EnMassArgs); the one that sees
    // red_target arrivals writes the sum to red_direct_out and sets the word back to zero.
    unsigned long long *red_direct;
    float *red_direct_out;
    int red_shift, red_target;
    // decode kernel only, or null: the rows' own keys / values [B, Nq, Hkv, D], which the kernel
    // writes into the context (kc, vt) at positions L_c + q_first + t before it reads them
    const void *app_k, *app_v;
};

struct EnMassArgs {
    EnDivisor by_splits, by_groups, by_target, by_chunks;      // n_splits; of the reduced masses' workgroup numbers
    const float *ws_ml, *ws_seg, *ws_mlfin;
    // Reduced masses [B, Smax+1], or null. Unless the step has few rows (`few`, see mass_few_rows in en_host.cpp)
    // red_target workgroups, of EN_MASS_UNITS units of 64 rows of a head each, sum a bucket's rows in fp32.
    // Their sums meet in one of two ways. With `parts` null, as part of an attention call and without a
    // launch behind it: as fixed-point integers (2^-red_shift; integer sums do not depend on the order of
    // the additions) in red_acc [B, Smax+1], whose low red_count_bits bits count the arrivals; the last one
    // writes the sum and sets the word back to zero. Else in parts [B, Smax+1, red_target], which a second
    // launch adds up, fp32 all the way: in steps of 2^-40 a sum of 1e-9 has ten bits. (32 heads x 512 rows
    // over 8 K tokens: 8.1 us, 6.7 in fixed point; x 2048 rows: 11.2, 10.8; x 4096: 12.6, 14.7. One launch
    // whose last workgroup adds up the parts, behind a release of each: 11.8, 28.5 and 31.5.)
    float *red_out;
    float *parts;
    unsigned long long *red_acc;
    int red_shift, red_count_bits, red_target;
    const int32_t *nseg, *bnd;
    const int32_t *hdr;     // as in EnAttnArgs
    float *out;
    int B, Hq, Nq, Smax, n_splits;
    int sub;                // as in EnAttnArgs: n_splits * sub partial results per row, the sub of a split side by side
    int q_first;            // as in EnAttnArgs
    int few;                // 1: the reduced masses go through the kernel for few rows per head
};

struct EnAppendArgs {
    const void *k_rows, *v_rows;   // [n, Hkv, D]
    void *k_pool, *v_pool;         // [G, Hkv, C, D]
    int n, Hkv, C, group, first;   // rows go to tokens first .. first+n-1 of the group
    int row_chunks;                // 16-byte chunks per (token, head) row
};
struct EnAppendQ8Args {
    const void *k_rows, *v_rows;   // bf16 [n, Hkv, D]
    int8_t *k_pool, *v_pool;       // [G, Hkv, C, D]
    float *k_scale, *v_scale;      // [G, Hkv, C]
    int n, Hkv, C, group, first;
};


constexpr int EN_RED_DIRECT_MAX_BUCKETS = 256;   // EnAttnArgs::red_direct: buckets whose sums a workgroup keeps in LDS
// Reduced masses in an attention call: below this many query rows per head a launch behind the merge adds them up in
// fp32, from here on the merge launch does, in fixed point (56 heads, 4 K tokens, behind / beside the merge: 7 rows
// 25.1 / 23.2 us, 8 rows 25.3 / 23.4, 24 rows 32.3 / 26.0).
constexpr int EN_MASS_FEW_ROWS = 8;
// Reduced masses in a call of their own: up to this many (head, row) pairs one launch with a workgroup per bucket,
// beyond it the parts of many workgroups and a second launch (17 buckets: 1024 pairs 5.0 / 7.7 us, 2048 7.1 / 7.7,
// 3072 9.3 / 7.7; 16 agents x 25 buckets: 4.7 / 8.2, 6.2 / 8.2, 7.8 / 10.0).
constexpr int EN_MASS_FEW_PAIRS = 2048;
constexpr int EN_MASS_BG = 8;           // buckets per workgroup of the reduced masses
constexpr int EN_MASS_UNITS = 4;        // units of 64 query rows of a head per workgroup of the reduced masses, one per wave
constexpr int EN_MASS_ARRIVALS = 1023;  // workgroups that may meet in one accumulator of the reduced masses (10 bits)
constexpr int EN_MAX_SPLITS = 64;       // KV splits of a plan: the mass kernels hold one split per lane
constexpr int EN_MAX_OBJECTS = 255;    // per segment_cluster_assign call (spans travel in the kernel arguments)
struct EnClusterArgs {
    EnMassArgs m;                  // the scratch of the attention call (m.out unused)
    float *score;                  // [B, n_obj, Smax+1]
    int32_t *assign;               // [B, n_obj] or null
    int n_obj, per_key, accumulate;
    float scale, threshold;
    int32_t spans[EN_MAX_OBJECTS + 1];   // object o = new tokens [spans[o], spans[o+1])
};

// One launch loads up to EN_TIER_LOAD_MAX blocks from the pinned host store into device slots.
constexpr int EN_TIER_LOAD_MAX = 128;
struct EnTierLoadArgs {
    const char *k_store, *v_store;   // device-visible addresses of the store, blocks [G, Hkv, C, D]
    char *k_slots, *v_slots;         // device, blocks [slots, Hkv, C, D]
    unsigned long long block_bytes;  // Hkv * C * D * elem
    int head_bytes;                  // C * D * elem
    int row_bytes;                   // D * elem
    int Hkv, n;
    int32_t desc[EN_TIER_LOAD_MAX * 3];   // per block: group, slot, tokens
};

struct EnCtxAppendArgs {
    const void *k_rows, *v_rows;   // [B, n, Hkv, D], keys unrotated
    void *kc, *vt;                 // the context buffers
    const float *cos_tab, *sin_tab;
    const int32_t *hdr;            // per agent {S, L_c, ...}
    int B, Hkv, n, T, q_first;
};

// Workspace layout helper (bytes, every part 256-byte aligned).
struct EnWsLayout {
    size_t ml_off, seg_off, redacc_off, mlfin_off, opart_off, parts_off, total;
};
EnWsLayout en_ws_layout(const en_pool *pool, const en_plan *plan);
EnWsLayout en_ws_layout_for(const en_pool *pool, const en_plan *plan, int n_rows, int n_splits);
int en_attn_sub(const en_pool *pool, const en_plan *plan, int n_rows, int n_splits);
int en_attn_once_tiles(const en_pool *pool, const en_plan *plan, int n_rows, int n_splits);
// The order of a plan's gather, to the end of en_plan::h_desc.
void en_gather_order(en_plan *plan, int64_t queries);
size_t en_plan_block_bytes(const en_plan *plan, size_t bytes);

// Kernel launchers (the .hip files). Return hipError_t as int.
int en_launch_gather(const en_plan *plan, EnGatherLaunch &g, void *stream);
int en_launch_attention(const en_pool *pool, const EnAttnArgs &a, void *stream);
int en_launch_attention_prefill(const en_pool *pool, const EnAttnArgs &a, void *stream);   // called by the former
int en_launch_combine(const en_pool *pool, const EnAttnArgs &a, const EnMassArgs &m, void *stream);
int en_launch_append(const en_pool *pool, const EnAppendArgs &a, void *stream);
int en_launch_append_q8(const en_pool *pool, const EnAppendQ8Args &a, void *stream);
int en_launch_cluster(const en_pool *pool, const EnClusterArgs &a, void *stream);
int en_launch_ctx_append(const en_pool *pool, const EnCtxAppendArgs &a, void *stream);
int en_launch_mass(const en_pool *pool, const EnMassArgs &a, int reduce, void *stream);
int en_launch_tier_load(const EnTierLoadArgs &a, int max_tokens, void *stream);

// The static device scratch of segmented_decode_step_static (en_static_scratch.hip,
// EN_STATIC_SCRATCH_BYTES of the public header): the device address of the current device's copy
// (returns 0 or a hipError_t).
int en_static_scratch(void **ptr_out, size_t *bytes_out);

int en_launch_ceiling_mfma(float *sink_dev, int n_workgroups, int iters, int constant, void *stream);
int en_launch_ceiling_read(const void *src_dev, size_t bytes, void *sink_dev, int n_workgroups, void *stream);

void en_set_error(const char *fmt, ...);

// Every extern "C" entry point that returns a status runs its body through this: no C++
// exception (std::bad_alloc from a container sized by caller input, above all) crosses the C ABI.
int en_fail_exception(const char *who, bool out_of_memory);
#define EN_GUARDED(who, call)                      \
    try {                                          \
        return (call);                             \
    } catch (const std::bad_alloc &) {             \
        return en_fail_exception(who, true);       \
    } catch (...) {                                \
        return en_fail_exception(who, false);      \
    }

// Retrieval knapsack of Eq. (1) over `G` candidates with lengths `len` (tokens); ids ascending.
// Returns an en_status: INVALID_ARG for a score or threshold that is not finite, CAPACITY when the
// table of the dynamic programme would exceed EN_KNAPSACK_MAX_BYTES.
constexpr size_t EN_KNAPSACK_MAX_BYTES = size_t(1) << 30;
int en_knapsack(const float *p_host, const int32_t *len, int G, float threshold, int64_t budget_tokens,
                std::vector<int32_t> &chosen);
