// Merge of the KV splits (log-sum-exp), per-segment attention mass and the
// clustering scores and decision of Section 3.3 of arXiv 2510.18546.
#include "en_device.h"

// ---------------------------------------------------------------------------
// combine: out = sum_sp w_sp y_sp / sum_sp w_sp with y_sp the split's own
// softmax output and w_sp = l_sp 2^(m_sp - m). One thread per 16 bytes of an
// output row. grid: ceil(rows * D / V / 256), V = elements in 16 bytes.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void mass_partial_block(const EnMassArgs &a, int blk, float *red);

// A workgroup's part of the reduced mass of (agent, bucket) `idx`; the words were set to zero by the attention
// launch before.
__device__ __forceinline__ void add_reduced_mass(const EnMassArgs &a, size_t idx, float part)
{
    arrive_fixed_point(a.red_acc + idx, part, not_a_number(part), a.red_shift, a.red_count_bits, a.red_target,
                       a.red_out + idx);
}

// A workgroup of the reduced masses takes EN_MASS_BG consecutive buckets of one agent over EN_MASS_UNITS
// units of 64 query rows (see mass_partial_block).
__host__ __device__ inline int mass_bucket_groups(const EnMassArgs &m)
{
    return (m.Smax + 1 + EN_MASS_BG - 1) / EN_MASS_BG;
}
__host__ inline int mass_partial_blocks(const EnMassArgs &m)
{
    return mass_bucket_groups(m) * m.red_target * m.B;       // red_target: workgroups per agent and bucket group
}

// With many splits (decode over a long context by few agents) G = 4, 16 or 32 neighbouring lanes
// share a (row, 16-byte chunk): lane g takes the splits g, g + G, ... and the G partial results
// are merged among the lanes, so that the chain of dependent loads is 1/G as long (with 16
// lanes, up to 64 splits are one batch of loads) and the few rows of such a step make G times
// as many workgroups. NB: splits per lane and batch, no more than there are (eight of which six are the
// first one again: a decode step over 0.4 K tokens, 7 splits, 9.4 us with the merge, 8.2 with two; 26 splits 12.7, 11.8).
template <typename T, int D, int G, int NB>
__global__ __launch_bounds__(256) void combine_kernel(EnAttnArgs a, EnMassArgs m, int n_comb)
{
    // The arguments in one batch and no integer divisions, as in attn_bf16_kernel, sums over lanes in the vector ALU: the
    // launch without masses is 2.5 us of start and end and three trips to memory, with them these and what the set-up of
    // the buckets takes. With masses, one agent's ragged map 7.6 -> 6.2 us, 8 K tokens 9.5 -> 8.4; a decode step's 26
    // partial results 3.7 -> 3.4.
    asm volatile("" ::"s"(a.out), "s"(a.ws_ml), "s"(a.ws_opart), "s"(a.ws_mlfin), "s"(a.B), "s"(a.by_nq.mul), "s"(a.by_hq.mul),
                 "s"(m.by_splits.mul), "s"(m.ws_seg), "s"(m.red_acc), "s"(m.bnd), "s"(m.hdr), "s"(m.B), "s"(m.q_first), "s"(n_comb));
    // head of the grid (these workgroups take longest: they start first): the reduced masses, where
    // the attention call was asked for them (without: 10.1 -> 6.1 us on the 8K-context step)
    const int n_part = (int)gridDim.x - n_comb;
    if ((int)blockIdx.x < n_part) {
        __shared__ float red[4 * EN_MASS_BG];
        mass_partial_block(m, blockIdx.x, red);
        return;
    }
    constexpr int V = 16 / sizeof(T);
    typedef T tvec __attribute__((ext_vector_type(V)));
    typedef float fvec __attribute__((ext_vector_type(V)));
    const size_t rows = (size_t)a.B * a.Hq * a.Nq;
    size_t idx = (size_t)(blockIdx.x - n_part) * 256 + threadIdx.x;
    const int g = (int)(idx % G);
    idx /= G;
    if (idx >= rows * (D / V))
        return;
    const size_t row = idx / (D / V);
    const int d0 = (int)(idx % (D / V)) * V;
    // The splits are read in batches of independent loads, (reference, sum) pairs and outputs
    // together, and merged batch by batch with a running reference: read one after the other,
    // the latencies of 2 * n_splits dependent loads are what this kernel would take.
    float M = EN_NEG_INF, l = 0.f;
    fvec acc = 0.f;
    for (int sp0 = g; sp0 < a.n_splits; sp0 += NB * G) {
        f32x2 ml[NB];
        tvec v[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const bool on = sp0 + j * G < a.n_splits;
            const size_t r = (size_t)(on ? sp0 + j * G : 0) * rows + row;
            ml[j] = *reinterpret_cast<const f32x2 *>(a.ws_ml + r * 2);
            v[j] = *reinterpret_cast<const tvec *>((const T *)a.ws_opart + r * D + d0);
            if (!on)
                ml[j][0] = EN_NEG_INF;
        }
        float Mb = M;
#pragma unroll
        for (int j = 0; j < NB; ++j)
            Mb = fmaxf(Mb, ml[j][0]);
        if (Mb == EN_NEG_INF)
            continue;
        const float keep = M == EN_NEG_INF ? 0.f : fast_exp2(M - Mb);
        l *= keep;
        acc *= keep;
        M = Mb;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            // a split that saw no key of this row left (-inf, 0) and an output that is not to be used
            const float w = ml[j][0] == EN_NEG_INF ? 0.f : ml[j][1] * fast_exp2(ml[j][0] - M);
            l += w;
            acc += w == 0.f ? (fvec)0.f : __builtin_convertvector(v[j], fvec) * w;
        }
    }
    if constexpr (G > 1) {
        // (in the vector ALU: data-parallel primitives; through the LDS crossbar the 40 exchanges of 16 lanes are a chain
        // of four trips)
        const float Mall = lanes_reduce<G>(M, [](float x, float y) { return fmaxf(x, y); });
        const float keep = M == EN_NEG_INF ? 0.f : fast_exp2(M - Mall);
        l *= keep;
        acc *= keep;
        M = Mall;
        const auto plus = [](float x, float y) { return x + y; };
        l = lanes_reduce<G>(l, plus);
#pragma unroll
        for (int e = 0; e < V; ++e)
            acc[e] = lanes_reduce<G>(acc[e], plus);
        if (g != 0)
            return;
    }
    const float inv = 1.f / l;
    if (d0 == 0 && a.ws_mlfin) {
        f32x2 ml = {M, l};
        *reinterpret_cast<f32x2 *>(a.ws_mlfin + row * 2) = ml;
    }
    // (the host refuses 2^31 rows and more)
    const unsigned bh = divided((unsigned)row, a.by_nq);
    const unsigned i = (unsigned)row - bh * (unsigned)a.Nq;
    const unsigned b = divided(bh, a.by_hq);
    const unsigned hq = bh - b * (unsigned)a.Hq;
    T *op = (T *)a.out + (((size_t)b * a.Nq + i) * a.Hq + hq) * D + d0;
    *reinterpret_cast<tvec *>(op) = __builtin_convertvector(acc * inv, tvec);
}

// ---------------------------------------------------------------------------
// mass: probability mass per (row, bucket) from the raw partial sums.
//   mass = sum over splits touching the bucket of seg * 2^(m_seg - M) / L
// with (M, L) the row's final reference maximum and sum.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void row_final_ml(const EnMassArgs &a, size_t rows, size_t row, float &M,
                                             float &L)
{
    // one split: its own (reference, sum); several: the pair the combine kernel merged
    const float *p = (a.n_splits * a.sub > 1 ? a.ws_mlfin : a.ws_ml) + row * 2;
    (void)rows;
    M = p[0];
    L = p[1];
}

// The row's reference maximum and sum merged from the splits' pairs (what the combine kernel
// writes to ws_mlfin, for code that runs beside it). Independent loads in batches of four.
__device__ __forceinline__ void merged_ml(const EnMassArgs &a, size_t rows, size_t row, float &M, float &L)
{
    constexpr int NB = 4;
    M = EN_NEG_INF;
    L = 0.f;
    const int n_part = a.n_splits * a.sub;      // partial results per row
    for (int sp0 = 0; sp0 < n_part; sp0 += NB) {
        f32x2 ml[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            ml[j] = *reinterpret_cast<const f32x2 *>(a.ws_ml + ((size_t)(sp0 + j < n_part ? sp0 + j : 0) * rows + row) * 2);
            if (sp0 + j >= n_part)
                ml[j][0] = EN_NEG_INF;
        }
        float Mb = M;
#pragma unroll
        for (int j = 0; j < NB; ++j)
            Mb = fmaxf(Mb, ml[j][0]);
        if (Mb == EN_NEG_INF)
            continue;
        L *= M == EN_NEG_INF ? 0.f : fast_exp2(M - Mb);
        M = Mb;
#pragma unroll
        for (int j = 0; j < NB; ++j)
            L += ml[j][0] == EN_NEG_INF ? 0.f : ml[j][1] * fast_exp2(ml[j][0] - M);
    }
}

// Tiles of the KV splits, one split per lane (a plan has at most 64 splits): the attention
// kernels give split sp the tiles [split_first_tile(sp), split_first_tile(sp + 1)). Code that
// has to know which splits cover a bucket asks this map with two wave votes instead of doing
// integer divisions per bucket (a division by a run-time value is some thirty instructions, and
// these kernels are bound by their instruction count).
struct EnSplitMap {
    int end_tile;                  // first tile after this lane's split; lanes >= n_splits: INT_MAX
    unsigned long long keys;       // bit sp: split sp holds at least one tile
};
// whole wave, uniform arguments
__device__ __forceinline__ EnSplitMap split_map(const EnDivisor &by_splits, int ntiles)
{
    const int n_splits = by_splits.n;
    const unsigned q = threadIdx.x % 64;
    const unsigned bgn = divided(q * ntiles + n_splits - 1, by_splits);           // split_first_tile
    const unsigned end = divided((q + 1) * ntiles + n_splits - 1, by_splits);
    EnSplitMap m;
    m.end_tile = (int)q < n_splits ? (int)end : 0x7fffffff;
    m.keys = __ballot((int)q < n_splits && end != bgn);
    return m;
}
// Splits whose key range meets bucket [blo, bhi): a contiguous range [lo, hi]. Whole wave, uniform
// arguments: the split that holds tile t is the number of splits that end at or before t.
__device__ __forceinline__ void bucket_splits(const EnSplitMap &m, int n_splits, int Ltot, int blo, int bhi,
                                              int &lo, int &hi)
{
    bhi = min(bhi, Ltot);          // a decode step's rows see less than the plan's whole new block
    const int t_lo = blo / EN_KEY_TILE, t_hi = (bhi - 1) / EN_KEY_TILE;
    const int l = (int)__popcll(__ballot(m.end_tile <= t_lo));
    const int h = (int)__popcll(__ballot(m.end_tile <= t_hi));
    lo = bhi <= blo ? n_splits : l;
    hi = bhi <= blo ? -1 : h;
}
// The same for one thread on its own (32-bit arithmetic: t * n_splits <= Ltot): the split
// that holds tile t is the largest sp whose first tile is <= t, t * n_splits / ntiles.
// Also returns the mask of the splits in [lo, hi] that hold keys.
__device__ __forceinline__ void bucket_splits_thread(int n_splits, int ntiles, int Ltot, int blo, int bhi,
                                                     int &lo, int &hi, unsigned long long &keys)
{
    bhi = min(bhi, Ltot);
    keys = 0;
    if (bhi <= blo) {
        lo = n_splits;
        hi = -1;
        return;
    }
    const unsigned t_lo = blo / EN_KEY_TILE, t_hi = (bhi - 1) / EN_KEY_TILE;
    lo = (int)(t_lo * (unsigned)n_splits / (unsigned)ntiles);
    hi = (int)(t_hi * (unsigned)n_splits / (unsigned)ntiles);
    for (int sp = lo; sp <= hi; ++sp)
        if (split_first_tile(sp, ntiles, n_splits) != split_first_tile(sp + 1, ntiles, n_splits))
            keys |= 1ull << sp;
}

__device__ __forceinline__ float row_bucket_mass(const EnMassArgs &a, int b, int hq, int i, int bucket,
                                                 int sp_lo, int sp_hi, float M, float L,
                                                 unsigned long long keys)
{
    float acc = 0.f;
    for (int sp = sp_lo; sp <= sp_hi; ++sp) {
        // an agent with fewer key tiles than the plan has splits leaves some splits without
        // keys: nothing was written for them
        if (!((keys >> sp) & 1))
            continue;
        // the waves that shared the split's tiles each left a pair of their own
        for (int w = 0; w < a.sub; ++w) {
            const f32x2 v = *reinterpret_cast<const f32x2 *>(
                a.ws_seg +
                (((((size_t)(sp * a.sub + w) * a.B + b) * a.Hq + hq) * (a.Smax + 1) + bucket) * a.Nq + i) * 2);
            if (v[1] != EN_NEG_INF)
                acc += v[0] * fast_exp2(v[1] - M);
        }
    }
    return acc / L;
}

// reduce = 0. grid: (ceil(Nq/64) * chunks of EN_MASS_RB buckets, Hq, B), 256 threads: the block takes 64
// queries of one head and one chunk of buckets (both in x: the other dimensions of a grid end at 65535). The scratch is laid out query-fastest, the result
// bucket-fastest: each wave computes the masses of four buckets for the 64 queries (coalesced reads), the
// block transposes them through LDS and writes runs of 64 bytes per query. A trip to memory takes about a
// microsecond and each wave makes one for its four buckets: a block that walked all buckets of its rows
// made nine (4 agents x 129 rows x 32 heads x 33 buckets: 10.4 us against 5.9).
constexpr int EN_MASS_RB = 16;
__global__ __launch_bounds__(256) void mass_rows_kernel(EnMassArgs a)
{
    constexpr int PER = EN_MASS_RB / 4;          // buckets per wave
    __shared__ float tile[64][EN_MASS_RB + 1];
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    asm volatile("" ::"s"(a.ws_ml), "s"(a.ws_mlfin), "s"(a.bnd), "s"(a.out), "s"(a.B), "s"(a.by_splits.mul), "s"(a.q_first));
    const int n_chunks = (a.Smax + EN_MASS_RB) / EN_MASS_RB;
    const int rows64 = __builtin_amdgcn_readfirstlane(small_quotient(blockIdx.x, n_chunks));
    const int i0 = rows64 * 64, i = i0 + lane;
    const int hq = blockIdx.y, b = blockIdx.z;
    const int s0 = (blockIdx.x - rows64 * n_chunks) * EN_MASS_RB;
    const bool valid = i < a.Nq;
    const size_t rows = (size_t)a.B * a.Hq * a.Nq;
    const size_t row = ((size_t)b * a.Hq + hq) * a.Nq + (valid ? i : 0);
    float M, L;
    row_final_ml(a, rows, row, M, L);
    const en_table_ptr hdr = as_table(a.hdr + 4 * (size_t)b);
    const int S = hdr[0];
    const int Ltot = hdr[1] + a.q_first + a.Nq;     // end of what the rows could see
    const int ntiles = (Ltot + EN_KEY_TILE - 1) / EN_KEY_TILE;
    const EnSplitMap map = split_map(a.by_splits, ntiles);
    const int32_t *bnd = a.bnd + (size_t)b * (a.Smax + 2);
    int lo[PER], hi[PER];
    bool live[PER], simple = a.sub == 1;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int s = min(s0 + wave * PER + j, a.Smax);              // the same for the whole wave
        const int blo = bnd[s], bhi = bnd[s + 1];
        live[j] = s0 + wave * PER + j <= S && bhi > blo;
        bucket_splits(map, a.n_splits, Ltot, blo, bhi, lo[j], hi[j]);
        live[j] = live[j] && hi[j] >= lo[j];
        simple = simple && (!live[j] || hi[j] - lo[j] <= 1);
    }
    float v[PER];
    if (simple) {
        // one split covers the bucket or two neighbours do: both entries of every bucket in one batch of loads
        f32x2 e0[PER], e1[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int s = min(s0 + wave * PER + j, a.Smax);
            const int sp = live[j] ? lo[j] : 0, sp1 = live[j] ? hi[j] : 0;
            const f32x2 *p = reinterpret_cast<const f32x2 *>(a.ws_seg) +
                             (((size_t)b * a.Hq + hq) * (a.Smax + 1) + s) * a.Nq + (valid ? i : 0);
            const size_t per_split = (size_t)a.B * a.Hq * (a.Smax + 1) * a.Nq;
            e0[j] = p[sp * per_split];
            e1[j] = p[sp1 * per_split];
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            float acc = 0.f;
            // (an agent with fewer key tiles than the plan has splits leaves some splits without keys: nothing was
            // written for them)
            if (live[j] && ((map.keys >> lo[j]) & 1) && e0[j][1] != EN_NEG_INF)
                acc += e0[j][0] * fast_exp2(e0[j][1] - M);
            if (live[j] && hi[j] > lo[j] && ((map.keys >> hi[j]) & 1) && e1[j][1] != EN_NEG_INF)
                acc += e1[j][0] * fast_exp2(e1[j][1] - M);
            v[j] = acc / L;              // (as row_bucket_mass: one rounding, not two)
        }
    } else {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            v[j] = 0.f;
            if (live[j] && valid)
                v[j] = row_bucket_mass(a, b, hq, i, s0 + wave * PER + j, lo[j], hi[j], M, L, map.keys);
        }
    }
#pragma unroll
    for (int j = 0; j < PER; ++j)
        tile[lane][wave * PER + j] = v[j];
    __syncthreads();
    const int c = threadIdx.x % EN_MASS_RB;
#pragma unroll
    for (int k = 0; k < 64 * EN_MASS_RB / 256; ++k) {
        const int r = threadIdx.x / EN_MASS_RB + k * (256 / EN_MASS_RB);
        const int ir = i0 + r;
        if (ir < a.Nq && s0 + c <= a.Smax)
            a.out[(((size_t)b * a.Nq + ir) * a.Hq + hq) * (a.Smax + 1) + s0 + c] = tile[r][c];
    }
}

// reduce = 0 for few rows per head (decode steps): a thread per result, buckets fastest. grid: (ceil(Hq (Smax+1)
// / 256), Nq, B). One row of 64 queries' width per (agent, head) left 63 lanes of 64 idle in each of a
// bucket's trips to memory (64 agents x 32 heads x 65 buckets, one token: 25.8 us against 4.8).
__global__ __launch_bounds__(256) void mass_rows_few_kernel(EnMassArgs a)
{
    const unsigned nb = a.Smax + 1;
    const unsigned idx = blockIdx.x * 256u + threadIdx.x;
    if (idx >= a.Hq * nb)
        return;
    const int hq = idx / nb, s = idx - hq * nb;
    const int i = blockIdx.y, b = blockIdx.z;
    const size_t rows = (size_t)a.B * a.Hq * a.Nq;
    float M, L;
    row_final_ml(a, rows, ((size_t)b * a.Hq + hq) * a.Nq + i, M, L);
    const int32_t *bnd = a.bnd + (size_t)b * (a.Smax + 2);
    const int blo = bnd[s], bhi = bnd[s + 1];
    const en_table_ptr hdr = as_table(a.hdr + 4 * (size_t)b);
    const int S = hdr[0];
    const int Ltot = hdr[1] + a.q_first + a.Nq;
    const int ntiles = (Ltot + EN_KEY_TILE - 1) / EN_KEY_TILE;
    float v = 0.f;
    if (s <= S && bhi > blo) {
        int lo, hi;
        unsigned long long keys;
        bucket_splits_thread(a.n_splits, ntiles, Ltot, blo, bhi, lo, hi, keys);
        v = row_bucket_mass(a, b, hq, i, s, lo, hi, M, L, keys);
    }
    a.out[((size_t)b * a.Nq + i) * a.Hq * nb + idx] = v;
}

// The reduced masses: workgroup blk sums EN_MASS_BG buckets over EN_MASS_UNITS units, one per wave, a unit
// being 64 query rows of one head: a step of few rows per head fills its workgroups with heads (32 heads x 48
// rows over 1.6 K tokens, attention call: 29.3 us with a launch behind the merge that walked the rows of a
// bucket one trip to memory after the other, 22.8 like this; without masses 20.7). As part of an attention call with several KV splits this runs in the first
// workgroups of the combine launch and merges the splits' (reference, sum) pairs itself; otherwise it is a
// launch of its own.
//
// What this costs is instructions per (row, bucket) and dependent trips to memory (about a
// microsecond each), not bytes. So lanes are rows: a row's merged (reference,
// sum) pair is made once for the group's buckets; everything that is the same for all rows (which splits
// cover a bucket, whether they hold keys) is decided from the agent's header and bounds before the rows
// start; and a row's loads for all buckets go out together: a bucket
// is covered by one split or by two neighbours unless it is longer than a split, so two entries
// per bucket are fetched whether or not the second one counts (it lies inside the scratch either
// way). A group with a bucket over more than two splits takes them one after the other.
// (Other forms, measured on 16 agents x 25 buckets x 32 heads x 128 rows and on the tail of the
// 8K-context merge: one workgroup per (bucket, head), all of the above per row: 23 us / 6 us;
// the same buckets in one workgroup with loads as they are needed: 27 us / 13 us; one launch that
// lets the last workgroup finish (a device-scope release per workgroup, which writes the L2
// back): 25 us; one workgroup per bucket: 14 us; two units per wave and four buckets, four and four, which
// halve and quarter the arrivals at an accumulator: 0.3 and 4 us more than one and eight.)
__device__ __forceinline__ void mass_partial_block(const EnMassArgs &a, int blk, float *red)
{
    constexpr int BG = EN_MASS_BG;
    const int wgs = divided(blk, a.by_groups);
    const int s0 = (blk - wgs * a.by_groups.n) * BG;
    const int b = divided(wgs, a.by_target);
    const int wg = wgs - b * a.red_target;             // workgroup among those of the agent's bucket group
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const int n_chunks = (a.Nq + 63) / 64;
    const int n_units = a.Hq * n_chunks;
    const int unit = wg * EN_MASS_UNITS + wave;
    float acc[BG];
#pragma unroll
    for (int j = 0; j < BG; ++j)
        acc[j] = 0.f;
    if (unit < n_units) {                         // a wave without rows has nothing to set up
        const size_t rows = (size_t)a.B * a.Hq * a.Nq;
        const en_table_ptr hdr = as_table(a.hdr + 4 * (size_t)b);
        const int S = hdr[0];
        const int Ltot = hdr[1] + a.q_first + a.Nq;     // end of what the rows could see
        const unsigned ntiles = (Ltot + EN_KEY_TILE - 1) / EN_KEY_TILE;
        const unsigned n = a.n_splits;
        // Bucket s0 + j is worked out by the lanes j, j + BG, ... (all of them alike), every bucket
        // of the group at once: the first split that covers it and whether that split and the one
        // after it count. Done bucket by bucket in scalar registers, this set-up was most of the
        // kernel's time: the scalar unit is shared by all waves of a compute unit.
        int lo_v, hi_v;
        bool live_v, use0_v, use1_v, next_v;
        size_t off0_v, off1_v;                          // byte offsets of the bucket's two entries of row 0, head 0
        const size_t per_split = (size_t)a.B * a.Hq * (a.Smax + 1) * a.Nq * 8;      // bytes
        const size_t per_head = (size_t)(a.Smax + 1) * a.Nq * 8;
        {
            const int jl = lane % BG;
            const int s = min(s0 + jl, a.Smax);
            const int32_t *bnd = a.bnd + (size_t)b * (a.Smax + 2);
            const int blo = bnd[s];
            const int bhi = min(bnd[s + 1], Ltot);      // a decode step's rows see less than the whole new block
            live_v = s0 + jl <= S && bhi > blo;
            const unsigned t_lo = live_v ? blo / EN_KEY_TILE : 0, t_hi = live_v ? (bhi - 1) / EN_KEY_TILE : 0;
            // the split that holds tile t is the largest sp whose first tile is <= t
            const unsigned l = small_quotient(t_lo * n, ntiles), h = small_quotient(t_hi * n, ntiles);
            const auto first_tile = [&](unsigned sp) { return divided(sp * ntiles + n - 1, a.by_splits); };
            const unsigned e0 = first_tile(l), e1 = first_tile(l + 1), e2 = first_tile(l + 2);
            next_v = l + 1 < n;
            use0_v = live_v && e0 != e1;                // an agent with fewer tiles than splits leaves some empty
            use1_v = live_v && h > l && next_v && e1 != e2;
            lo_v = (int)l;
            hi_v = (int)h;
            off0_v = l * per_split + (size_t)b * a.Hq * per_head + (size_t)s * a.Nq * 8;
            off1_v = off0_v + (next_v ? per_split : 0);
        }
        const unsigned use0 = (unsigned)__ballot(use0_v), use1 = (unsigned)__ballot(use1_v);
        const unsigned live = (unsigned)__ballot(live_v);
        const bool simple = a.sub == 1 && __ballot(live_v && hi_v - lo_v > 1) == 0;
        const int hq = divided(unit, a.by_chunks);
        const int row_i = (unit - hq * n_chunks) * 64 + lane;
        const bool on = row_i < a.Nq;
        const int i = on ? row_i : 0;
        float M, L;
        if (simple) {
            f32x2 v0[BG], v1[BG];
#pragma unroll
            for (int j = 0; j < BG; ++j) {
                const char *p0 = (const char *)a.ws_seg + readlane64(off0_v, j) + hq * per_head;
                const char *p1 = (const char *)a.ws_seg + readlane64(off1_v, j) + hq * per_head;
                v0[j] = *reinterpret_cast<const f32x2 *>(p0 + (unsigned)i * 8u);
                v1[j] = *reinterpret_cast<const f32x2 *>(p1 + (unsigned)i * 8u);
            }
            merged_ml(a, rows, ((size_t)b * a.Hq + hq) * a.Nq + i, M, L);
            const float inv = on ? 1.f / L : 0.f;
#pragma unroll
            for (int j = 0; j < BG; ++j) {
                float part = 0.f;
                if (((use0 >> j) & 1) && v0[j][1] != EN_NEG_INF)
                    part += v0[j][0] * fast_exp2(v0[j][1] - M);
                if (((use1 >> j) & 1) && v1[j][1] != EN_NEG_INF)
                    part += v1[j][0] * fast_exp2(v1[j][1] - M);
                acc[j] = part * inv;
            }
        } else {
            const EnSplitMap map = split_map(a.by_splits, (int)ntiles);
            int lo[BG], hi[BG];
#pragma unroll
            for (int j = 0; j < BG; ++j) {
                lo[j] = __builtin_amdgcn_readlane(lo_v, j);
                hi[j] = __builtin_amdgcn_readlane(hi_v, j);
            }
            if (on) {
                merged_ml(a, rows, ((size_t)b * a.Hq + hq) * a.Nq + i, M, L);
#pragma unroll
                for (int j = 0; j < BG; ++j)
                    if ((live >> j) & 1)
                        acc[j] = row_bucket_mass(a, b, hq, i, s0 + j, lo[j], hi[j], M, L, map.keys);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < BG; ++j) {
        const float t = wave_sum(acc[j]);
        if (lane == 0)
            red[wave * BG + j] = t;
    }
    __syncthreads();
    if (threadIdx.x < BG && s0 + (int)threadIdx.x <= a.Smax) {
        const int j = threadIdx.x;
        const size_t idx = (size_t)b * (a.Smax + 1) + s0 + j;
        const float part = red[j] + red[BG + j] + red[2 * BG + j] + red[3 * BG + j];
        if (a.parts)
            a.parts[idx * a.red_target + wg] = part;
        else
            add_reduced_mass(a, idx, part);
    }
}

__global__ __launch_bounds__(256) void mass_partial_kernel(EnMassArgs a)
{
    __shared__ float red[4 * EN_MASS_BG];
    asm volatile("" ::"s"(a.by_splits.mul), "s"(a.ws_ml), "s"(a.parts), "s"(a.bnd), "s"(a.B), "s"(a.q_first));
    mass_partial_block(a, blockIdx.x, red);
}

// The parts of a sum, added up by one wave per (agent, bucket) in an order of its own: fp32 all the way.
__global__ __launch_bounds__(256) void mass_final_kernel(EnMassArgs a)
{
    const int pair = blockIdx.x * 4 + threadIdx.x / 64;
    if (pair >= a.B * (a.Smax + 1))
        return;
    const float *p = a.parts + (size_t)pair * a.red_target;
    float acc = 0.f;
    for (int k = threadIdx.x % 64; k < a.red_target; k += 64)
        acc += p[k];
    acc = wave_sum(acc);
    if (threadIdx.x % 64 == 0)
        a.red_out[pair] = acc;
}

// The reduced masses of few (head, row) pairs (decode steps, small layers): a workgroup of G threads per (agent,
// bucket) walks the bucket's (head, row) pairs and writes the sum, nothing to meet and no second launch.
template <int G>
__global__ __launch_bounds__(256) void mass_few_rows_kernel(EnMassArgs a)
{
    __shared__ float red[4];
    const int pair = blockIdx.x * (256 / G) + threadIdx.x / G;
    const bool on = pair < a.B * (a.Smax + 1);
    const int s = on ? pair % (a.Smax + 1) : 0;
    const int b = on ? pair / (a.Smax + 1) : 0;
    const size_t rows = (size_t)a.B * a.Hq * a.Nq;
    const int S = a.nseg[b];
    const int32_t *bnd = a.bnd + (size_t)b * (a.Smax + 2);
    const int Ltot = bnd[S] + a.q_first + a.Nq;
    const int ntiles = (Ltot + EN_KEY_TILE - 1) / EN_KEY_TILE;
    float acc = 0.f;
    if (on && s <= S && bnd[s + 1] > bnd[s]) {
        int lo, hi;
        unsigned long long keys;
        bucket_splits_thread(a.n_splits, ntiles, Ltot, bnd[s], bnd[s + 1], lo, hi, keys);
        for (int idx = threadIdx.x % G; idx < a.Hq * a.Nq; idx += G) {
            const int hq = idx / a.Nq, i = idx - hq * a.Nq;
            float M, L;
            row_final_ml(a, rows, (size_t)b * a.Hq * a.Nq + idx, M, L);      // runs after the combine launch
            acc += row_bucket_mass(a, b, hq, i, s, lo, hi, M, L, keys);
        }
    }
    acc = wave_sum(acc);
    if constexpr (G > 64) {
        if (threadIdx.x % 64 == 0)
            red[threadIdx.x / 64] = acc;
        __syncthreads();
        acc = red[0] + red[1] + red[2] + red[3];
    }
    if (on && threadIdx.x % G == 0)
        a.red_out[pair] = acc;
}

// ---------------------------------------------------------------------------
// cluster: score of every (object, segment) pair and the join / new-group
// decision of Section 3.3. Scores: grid (Smax+1, n_obj, B), 256 threads, the
// block sums the masses that the object's (token, head) pairs put on one bucket.
// Decision: one wave per (agent, object), its lanes take that object's scores in turn.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void cluster_score_kernel(EnClusterArgs a)
{
    __shared__ float red[4];
    const EnMassArgs &m = a.m;
    const int s = blockIdx.x, o = blockIdx.y, b = blockIdx.z;
    // the spans are read from the argument segment itself (a run-time index into a
    // by-value argument would make a private copy of the whole array)
    const int32_t *spans = reinterpret_cast<const int32_t *>(
        reinterpret_cast<uintptr_t>(__builtin_amdgcn_kernarg_segment_ptr()) + offsetof(EnClusterArgs, spans));
    const int lo = spans[o], hi = spans[o + 1];
    asm volatile("" ::"s"(m.ws_ml), "s"(m.ws_mlfin), "s"(m.bnd), "s"(m.B), "s"(m.by_splits.mul), "s"(m.q_first), "s"(a.score), "s"(a.scale));
    const int n_pairs = (hi - lo) * m.Hq;
    const size_t rows = (size_t)m.B * m.Hq * m.Nq;
    const en_table_ptr hdr = as_table(m.hdr + 4 * (size_t)b);
    const int S = hdr[0];
    const en_table_ptr bnd = as_table(m.bnd + (size_t)b * (m.Smax + 2));
    const int Ltot = hdr[1] + m.q_first + m.Nq;     // end of what the rows could see
    const int ntiles = (Ltot + EN_KEY_TILE - 1) / EN_KEY_TILE;
    const int len = s <= S ? bnd[s + 1] - bnd[s] : 0;
    float acc = 0.f;
    const EnSplitMap map = split_map(m.by_splits, ntiles);
    if (len > 0) {
        int slo, shi;
        bucket_splits(map, m.n_splits, Ltot, bnd[s], bnd[s + 1], slo, shi);
        for (int idx = threadIdx.x; idx < n_pairs; idx += 256) {
            // token fastest: neighbouring lanes read neighbouring scratch entries
            const int hq = small_quotient(idx, hi - lo), i = lo + idx - hq * (hi - lo);
            const size_t row = ((size_t)b * m.Hq + hq) * m.Nq + i;
            float M, L;
            row_final_ml(m, rows, row, M, L);
            acc += row_bucket_mass(m, b, hq, i, s, slo, shi, M, L, map.keys);
        }
    }
    acc = wave_sum(acc);
    if (threadIdx.x % 64 == 0)
        red[threadIdx.x / 64] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        float *score = a.score + ((size_t)b * a.n_obj + o) * (m.Smax + 1) + s;
        float v = (red[0] + red[1] + red[2] + red[3]) / (float)n_pairs;
        if (a.per_key && s < S && len > 0)       // the new tokens' own bucket stays a mass
            v /= (float)len;
        if (a.accumulate)
            v += *score;
        *score = v;
    }
}

// A wave per (agent, object), the lanes take the segments in turn.
__global__ __launch_bounds__(256) void cluster_decide_kernel(EnClusterArgs a)
{
    const EnMassArgs &m = a.m;
    const int idx = blockIdx.x * 4 + threadIdx.x / 64, lane = threadIdx.x % 64;
    if (idx >= m.B * a.n_obj)
        return;
    const int b = idx / a.n_obj;
    const int S = m.nseg[b];
    const int32_t *bnd = m.bnd + (size_t)b * (m.Smax + 2);
    const float *score = a.score + (size_t)idx * (m.Smax + 1);
    float best = EN_NEG_INF;
    int best_s = -1;
    for (int s = lane; s < S; s += 64) {
        const float v = score[s] * a.scale;
        if (bnd[s + 1] > bnd[s] && v > best) {   // empty segments never win; the lowest s among equals
            best = v;
            best_s = s;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float v = __shfl_xor(best, o, 64);
        const int s = __shfl_xor(best_s, o, 64);
        // (a lane without a segment has the largest number of all)
        if (v > best || (v == best && (unsigned)s < (unsigned)best_s)) {
            best = v;
            best_s = s;
        }
    }
    if (lane == 0)
        a.assign[idx] = (best_s >= 0 && best >= a.threshold) ? best_s : -1;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
int en_launch_combine(const en_pool *pool, const EnAttnArgs &a, const EnMassArgs &m, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    const int D = pool->d.head_dim;
    const int vec = pool->d.dtype == EN_F32 ? 4 : 8;      // elements in 16 bytes
    // Lanes that share a (row, chunk). What the merge of a step of few rows costs is the partial
    // results per lane (each a dependent step of the running merge), not the number of workgroups:
    // about four per lane is best. Per decoded token, same box: 128 partial results by 16 / 32 / 64
    // lanes 18.0 / 17.5 / 17.9 us; 74 by 16 / 32 / 64 lanes 12.1 / 11.5 / 11.6; 32 (four agents) by
    // 4 / 16 lanes 14.0 / 13.1. A prefill's many rows fill the chip without that. What a lane asks for at once beyond the
    // splits there are is the last split's again, so the batch is the one that holds them: plans of two splits by batches
    // of two and of four, passes of a ragged map 30.98 / 31.3 us, of an int8 map 75.1 / 75.6.
    int G = a.n_splits > 32 ? 16 : (a.n_splits > 8 ? 4 : 1);
    if ((size_t)a.B * a.Hq * a.Nq * (D / vec) <= 16384)
        G = a.n_splits > 64 ? 32 : (a.n_splits > 16 ? 16 : (a.n_splits > 4 ? 4 : 1));
    const size_t n = (size_t)a.B * a.Hq * a.Nq * (D / vec) * G;
    const int n_comb = (int)((n + 255) / 256);
    const int n_part = m.red_out && !m.few ? mass_partial_blocks(m) : 0;
    const dim3 grid((unsigned)(n_comb + n_part)), blk(256);
#define EN_COMBINE(T, DD)                                                                                    \
    do {                                                                                                     \
        if (G == 1 && a.n_splits == 2)                                                                       \
            hipLaunchKernelGGL((combine_kernel<T, DD, 1, 2>), grid, blk, 0, st, a, m, n_comb);               \
        else if (G == 1)                                                                                     \
            hipLaunchKernelGGL((combine_kernel<T, DD, 1, 4>), grid, blk, 0, st, a, m, n_comb);               \
        else if (G == 4 && a.n_splits <= 8)                                                                  \
            hipLaunchKernelGGL((combine_kernel<T, DD, 4, 2>), grid, blk, 0, st, a, m, n_comb);               \
        else if (G == 4 && a.n_splits <= 16)                                                                 \
            hipLaunchKernelGGL((combine_kernel<T, DD, 4, 4>), grid, blk, 0, st, a, m, n_comb);               \
        else if (G == 4)                                                                                     \
            hipLaunchKernelGGL((combine_kernel<T, DD, 4, 8>), grid, blk, 0, st, a, m, n_comb);               \
        else if (G == 16 && a.n_splits <= 32)                                                                \
            hipLaunchKernelGGL((combine_kernel<T, DD, 16, 2>), grid, blk, 0, st, a, m, n_comb);              \
        else if (G == 16)                                                                                    \
            hipLaunchKernelGGL((combine_kernel<T, DD, 16, 4>), grid, blk, 0, st, a, m, n_comb);              \
        else                                                                                                 \
            hipLaunchKernelGGL((combine_kernel<T, DD, 32, 4>), grid, blk, 0, st, a, m, n_comb);              \
    } while (0)
    if (pool->d.dtype == EN_F32) {
        if (D == 64)
            EN_COMBINE(float, 64);
        else
            EN_COMBINE(float, 128);
    } else {
        if (D == 64)
            EN_COMBINE(bf16_t, 64);
        else
            EN_COMBINE(bf16_t, 128);
    }
#undef EN_COMBINE
    return (int)hipGetLastError();
}

int en_launch_cluster(const en_pool *pool, const EnClusterArgs &a, void *stream)
{
    (void)pool;
    const dim3 grid(a.m.Smax + 1, a.n_obj, a.m.B), blk(256);
    hipLaunchKernelGGL(cluster_score_kernel, grid, blk, 0, (hipStream_t)stream, a);
    if (a.assign) {
        const dim3 grid2((a.m.B * a.n_obj + 3) / 4);
        hipLaunchKernelGGL(cluster_decide_kernel, grid2, blk, 0, (hipStream_t)stream, a);
    }
    return (int)hipGetLastError();
}

int en_launch_mass(const en_pool *pool, const EnMassArgs &a, int reduce, void *stream)
{
    (void)pool;
    hipStream_t st = (hipStream_t)stream;
    if (reduce == 0) {
        const dim3 blk(256);
        // The line: 64 agents x 32 heads x 65 buckets, a thread per result / 64 rows' width: 12 rows 17.7 / 27.5 us,
        // 15 21.0 / 28.0, 16 22.1 / 27.6, 20 26.8 / 29.3, 32 40.6 / 30.5; a few agents 4.0 either way.
        if (a.Nq < 16) {
            const dim3 grid((a.Hq * (a.Smax + 1) + 255) / 256, a.Nq, a.B);
            hipLaunchKernelGGL(mass_rows_few_kernel, grid, blk, 0, st, a);
        } else {
            const dim3 grid((a.Nq + 63) / 64 * ((a.Smax + EN_MASS_RB) / EN_MASS_RB), a.Hq, a.B);
            hipLaunchKernelGGL(mass_rows_kernel, grid, blk, 0, st, a);
        }
    } else {
        const dim3 blk(256);
        const int pairs = a.B * (a.Smax + 1);
        if (!a.few) {
            hipLaunchKernelGGL(mass_partial_kernel, dim3(mass_partial_blocks(a)), blk, 0, st, a);
            if (a.parts)
                hipLaunchKernelGGL(mass_final_kernel, dim3((pairs + 3) / 4), blk, 0, st, a);
        // A wave or a workgroup per bucket: 64 agents x 65 buckets, 128 (head, row) pairs 5.1 / 9.2 us, 256 6.4 / 10.4;
        // one agent, 33 buckets 4.0 / 3.9 and 4.4 / 3.9.
        } else if (a.Hq * a.Nq <= 128)
            hipLaunchKernelGGL((mass_few_rows_kernel<64>), dim3((pairs + 3) / 4), blk, 0, st, a);
        else
            hipLaunchKernelGGL((mass_few_rows_kernel<256>), dim3(pairs), blk, 0, st, a);
    }
    return (int)hipGetLastError();
}
