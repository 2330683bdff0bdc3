// Data movement kernels of libefficientnav.so.
//
//   gather_k / gather_vt   index-driven gather of the selected K/V blocks into
//                          one contiguous context per agent; keys receive the
//                          rotary encoding of their concatenated position
//                          (Section 3.2 of arXiv 2510.18546: select, then load
//                          each group's KV once per planning step); the same
//                          from a pool of 8-bit codes
//   ctx_append             a decode step's own K/V rows join the context
//   tier_load              blocks of the host store go to device slots
//   append / append_q8     new objects' K/V rows join their group's block
#include "en_device.h"

// The bucket bounds and the selected groups of an agent. Up to 62 segments, every wave holds both tables in its lanes
// and finds its tokens' groups without a memory access (see context_row). More are staged in LDS: a binary search over the
// table in global memory is six dependent trips to memory per row, the group number a seventh (about 3 us before a block
// that moves 16 KB can issue its first load); over LDS it is a few hundred cycles. Tables that do not fit there either are
// read where they are. All threads of the block call open_tables. Tables in lanes and the arguments asked for together,
// against tables in LDS and arguments one by one: one agent's 4 K tokens 5.96 / 6.22 us, its 8.7 K 15.6 / 16.1, from 8-bit
// codes 4 x 3.2 K 16.9 / 18.4.
constexpr int EN_GATHER_TAB_LDS = 256;          // entries of either table
struct EnGatherTables {
    const int32_t *bnd, *sel;                   // the agent's bounds [Smax + 2] and groups [Smax]
    int S, Lc, Ltot;                            // segments, gathered tokens, all tokens
    int my_bnd, my_sel;                         // entry `lane` of either
    bool in_lanes, staged;
};
__device__ __forceinline__ EnGatherTables open_tables(const EnGatherArgs &a, int b, int32_t *lds)
{
    const int nb = a.Smax + 2;
    const int sstr = a.Smax > 0 ? a.Smax : 1;
    EnGatherTables t;
    t.bnd = a.bnd + (size_t)b * nb;
    t.sel = a.sel + (size_t)b * sstr;
    t.in_lanes = nb <= 64;
    t.staged = nb <= EN_GATHER_TAB_LDS;
    t.my_bnd = t.my_sel = 0;
    if (t.in_lanes) {
        const int lane = threadIdx.x % 64;
        if (lane < nb)
            t.my_bnd = t.bnd[lane];
        if (lane < a.Smax)
            t.my_sel = t.sel[lane];
        t.S = as_table(a.nseg)[b];
        t.Lc = __builtin_amdgcn_readlane(t.my_bnd, t.S);
        t.Ltot = __builtin_amdgcn_readlane(t.my_bnd, t.S + 1);
        return t;
    }
    t.S = as_table(a.nseg)[b];
    t.Lc = as_table(t.bnd)[t.S];
    t.Ltot = as_table(t.bnd)[t.S + 1];
    if (t.staged) {
        for (int i = threadIdx.x; i < nb; i += 256)
            lds[i] = t.bnd[i];
        for (int i = threadIdx.x; i < a.Smax; i += 256)
            lds[EN_GATHER_TAB_LDS + i] = t.sel[i];
        __syncthreads();
    }
    return t;
}

// Group and row in its block of context token `tok` (below L_c; anything for others). The whole wave calls, its tokens
// ascending from lane to lane: the segments of the first and the last one are two counts of bounds, and a lane goes
// through the few between them.
__device__ __forceinline__ void context_row(const EnGatherTables &t, const int32_t *lds, int tok, int &group, int &row)
{
    if (t.in_lanes) {
        const int lane = threadIdx.x % 64;
        auto bucket = [&](int x) { return (int)__popcll(__ballot(lane <= t.S && t.my_bnd <= x)) - 1; };
        const int s0 = bucket(__builtin_amdgcn_readfirstlane(tok));
        const int s1 = bucket(min(__builtin_amdgcn_readlane(tok, 63), t.Lc - 1));
        int start = __builtin_amdgcn_readlane(t.my_bnd, s0);
        group = __builtin_amdgcn_readlane(t.my_sel, s0);
        for (int s = s0 + 1; s <= s1; ++s) {
            const int from = __builtin_amdgcn_readlane(t.my_bnd, s), g = __builtin_amdgcn_readlane(t.my_sel, s);
            start = tok >= from ? from : start;
            group = tok >= from ? g : group;
        }
        row = tok - start;
        return;
    }
    group = row = 0;
    if (tok >= t.Lc)
        return;
    if (t.staged) {
        const int s = find_bucket(lds, t.S, tok);
        group = lds[EN_GATHER_TAB_LDS + s];
        row = tok - lds[s];
    } else {
        const int s = find_bucket(t.bnd, t.S, tok);
        group = t.sel[s];
        row = tok - t.bnd[s];
    }
}

// The tables of a descriptor block, one behind the other.
__device__ __forceinline__ void tables_in(EnGatherArgs &a, const int32_t *block)
{
    a.nseg = block;
    a.sel = a.nseg + a.B;
    a.bnd = a.sel + a.B * (a.Smax > 0 ? a.Smax : 1);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A piece of the context goes out. STREAM: past the caches, for contexts that the last-level cache
// cannot hold until the attention kernel reads them (see EnGatherArgs::stream; a template parameter: the
// choice made at run time between two kinds of store cost 150 us of 1440).
template <bool STREAM, typename P, typename V>
__device__ __forceinline__ void store_context(P *dst, V v)
{
    V *p = reinterpret_cast<V *>(dst);
    if constexpr (STREAM)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// Units of heads whose keys, all but the last one's, are turned in the form X1_ROUNDED of rope_key_pair, or 0; `many`:
// heads per key unit by gather_heads_many.
__host__ __device__ constexpr int en_rope_unit(int elem, int d, int many)
{
    return elem == 2 && (many == 4 || (many == 8 && d == 64)) ? many : 0;
}
// Source row of context token `tok` for (agent b, KV head kvh), in `group` at `row` if it is a gathered one; nullptr for
// padding rows at or beyond L_c + N_q.
template <typename T, int D>
__device__ __forceinline__ const T *context_src(const EnGatherArgs &a, const EnGatherTables &t, const void *pool,
                                               const void *fresh, int b, int kvh, int tok, int group, int row)
{
    if (tok >= t.Ltot)
        return nullptr;
    if (tok >= t.Lc)
        return (const T *)fresh + (((size_t)b * a.Nq + (tok - t.Lc)) * a.Hkv + kvh) * D;
    return (const T *)pool + (((size_t)group * a.Hkv + kvh) * a.C + row) * D;
}

// ---------------------------------------------------------------------------
// gather_k: 8 lanes per token row. Lane c owns elements [c*E, c*E+E) of the
// first half and their rotary partners in the second half (E = D/16).
// With COPY_V (fp32 path) the value row is copied alongside.
// A block takes 32 token rows of HPB consecutive KV heads, kv0 onwards: where a
// row comes from and its cosines and sines (two fp32 table rows, twice the bytes
// of a bf16 key row) are the same for every head, so they are fetched once for
// the HPB heads (64 agents x 16 K tokens, keys only: 1.14 ms with the table read
// per head, 0.73 ms without the table, which is what the value half takes).
// 256 threads, 32 rows per pass.
// ---------------------------------------------------------------------------
template <typename T, int D, bool COPY_V, int HPB, bool STREAM, bool AHEAD>
__device__ __forceinline__ void gather_k_rows(const EnGatherArgs &a, const EnGatherTables &t, const int32_t *lds, int b,
                                              int tok, int kv0)
{
    constexpr int E = D / 16;
    const int c = threadIdx.x % 8;
    int group, row;
    context_row(t, lds, tok, group, row);
    const int Lpad = (t.Ltot + EN_KEY_TILE - 1) / EN_KEY_TILE * EN_KEY_TILE;
    if (tok >= Lpad)
        return;
    typedef T tvec __attribute__((ext_vector_type(E)));
    typedef float fvec __attribute__((ext_vector_type(E)));
    // the rows of head kv0; head kv0 + h is h * hstride elements further, keys and values alike
    const T *ksrc = context_src<T, D>(a, t, a.k_pool, a.k_new, b, kv0, tok, group, row);
    const T *vsrc = nullptr;
    if constexpr (COPY_V)
        vsrc = context_src<T, D>(a, t, a.v_pool, a.v_new, b, kv0, tok, group, row);
    const size_t hstride = tok >= t.Lc ? (size_t)D : (size_t)a.C * D;      // new tokens [.., Hkv, D], pool [.., Hkv, C, D]
    fvec cs = 0.f, sn = 0.f;
    if (ksrc) {
        cs = *reinterpret_cast<const fvec *>(a.cos_tab + (size_t)tok * (D / 2) + c * E);
        sn = *reinterpret_cast<const fvec *>(a.sin_tab + (size_t)tok * (D / 2) + c * E);
    }
    // HU heads at a time. AHEAD (see gather_ahead): the loads of the next ones go out before these are
    // turned and stored, so that a workgroup of several heads waits for memory once and not once per HU heads.
    // Four of eight at a time then (two: the ordered gather of 64 agents x 16 K tokens takes 1 % longer, that of 32
    // agents 3 %).
    constexpr int HU = AHEAD && HPB == 8 ? 4 : HPB < 2 ? HPB : 2;
    // (without AHEAD the heads of a unit are those that en_rope_unit goes by)
    const int rope_unit = AHEAD ? a.rope_unit : en_rope_unit(sizeof(T), D, HPB);
    tvec x1[HU], x2[HU];
    auto load = [&](int h0) {
        if (ksrc) {
#pragma unroll
            for (int h = 0; h < HU; ++h) {
                x1[h] = *reinterpret_cast<const tvec *>(ksrc + (h0 + h) * hstride + c * E);
                x2[h] = *reinterpret_cast<const tvec *>(ksrc + (h0 + h) * hstride + D / 2 + c * E);
            }
        }
    };
    if constexpr (AHEAD)
        load(0);
#pragma unroll 1
    for (int h0 = 0; h0 < HPB; h0 += HU) {
        if constexpr (!AHEAD)
            load(h0);
        tvec w1[HU], w2[HU];
#pragma unroll
        for (int h = 0; h < HU; ++h) {
            w1[h] = x1[h];
            w2[h] = x2[h];
        }
        if constexpr (AHEAD) {
            asm volatile("" ::: "memory");         // (not behind the stores)
            if (h0 + HU < HPB)
                load(h0 + HU);
        }
#pragma unroll
        for (int h = 0; h < HU; ++h) {
            const int kvh = kv0 + h0 + h;
            const fvec f1 = __builtin_convertvector(w1[h], fvec), f2 = __builtin_convertvector(w2[h], fvec);
            T *dst = (T *)a.kc + (((size_t)b * a.Hkv + kvh) * a.T + tok) * D;
            fvec y1 = 0.f, y2 = 0.f;
            if (ksrc) {
                if (rope_unit && (kvh + 1) % rope_unit != 0)
                    rope_key_pair<true>(f1, f2, cs, sn, y1, y2);
                else
                    rope_key_pair(f1, f2, cs, sn, y1, y2);
            }
            store_context<STREAM>(dst + c * E, __builtin_convertvector(y1, tvec));
            store_context<STREAM>(dst + D / 2 + c * E, __builtin_convertvector(y2, tvec));
        }
    }
    if constexpr (COPY_V) {
#pragma unroll
        for (int h = 0; h < HPB; ++h) {
            T *vdst = (T *)a.vt + (((size_t)b * a.Hkv + kv0 + h) * a.T + tok) * D;
            tvec v1 = (T)0.f, v2 = (T)0.f;
            if (vsrc) {
                v1 = *reinterpret_cast<const tvec *>(vsrc + h * hstride + c * E);
                v2 = *reinterpret_cast<const tvec *>(vsrc + h * hstride + D / 2 + c * E);
            }
            *reinterpret_cast<tvec *>(vdst + c * E) = v1;
            *reinterpret_cast<tvec *>(vdst + D / 2 + c * E) = v2;
        }
    }
}

// The key rows of 64-token tile `tile` for the heads kv0 .. kv0 + HPB - 1, 32 rows at a time:
// the halves first .. last of the tile.
template <typename T, int D, bool COPY_V, int HPB, bool STREAM, bool AHEAD>
__device__ __forceinline__ void gather_k_block(const EnGatherArgs &a, int b, int tile, int first, int last, int kv0,
                                               int32_t *lbnd)
{
    const EnGatherTables t = open_tables(a, b, lbnd);
#pragma unroll 1
    for (int half = first; half <= last; ++half)
        gather_k_rows<T, D, COPY_V, HPB, STREAM, AHEAD>(a, t, lbnd, b, tile * EN_KEY_TILE + half * 32 + threadIdx.x / 8, kv0);
}

// ---------------------------------------------------------------------------
// gather_vt (bf16): values of a 64-token tile are staged in LDS and written
// transposed, vt[d][column], where token j sits at column j with bits 2 and 3
// exchanged; the heads kv0 .. kv0 + HPB - 1 one after the other, the next head's
// loads on their way meanwhile. 256 threads; bx = number of the 64-token tile.
// ---------------------------------------------------------------------------
template <int D, int HPB, bool STREAM, bool AHEAD>
__device__ __forceinline__ void gather_vt_block(const EnGatherArgs &a, int b, int bx, int kv0, int32_t *lbnd)
{
    constexpr int STR = D + 2;                 // LDS row stride in elements
    __shared__ uint16_t tile[EN_KEY_TILE * STR];
    __shared__ const uint16_t *srcs[EN_KEY_TILE];
    const int t0 = bx * EN_KEY_TILE;
    const EnGatherTables t = open_tables(a, b, lbnd);
    const int Lc = t.Lc;
    if (t0 >= t.Ltot)                            // the same for the whole block
        return;
    // head kv0 + h is h * stride elements further: new tokens [.., Hkv, D], pool [.., Hkv, C, D]
    auto head_stride = [&](bool fresh) { return fresh ? (size_t)D : (size_t)a.C * D; };
    const uint16_t *src = nullptr;
    if (threadIdx.x < EN_KEY_TILE) {
        int group, row;
        context_row(t, lbnd, t0 + threadIdx.x, group, row);
        src = context_src<uint16_t, D>(a, t, a.v_pool, a.v_new, b, kv0, t0 + threadIdx.x, group, row);
    }
    if (a.v_rows) {
        // the values stay where they are: the tile's 64 row addresses instead (padding rows: the row of zeros)
        char *zero_row = (char *)a.vt + en_v_rows_table_bytes(a.B, a.Hkv, a.T);
        if (threadIdx.x < EN_KEY_TILE) {
            unsigned long long *tab = (unsigned long long *)a.vt + ((size_t)b * a.Hkv + kv0) * (size_t)a.T + t0;
            for (int h = 0; h < HPB; ++h)
                tab[(size_t)h * a.T + threadIdx.x] = (unsigned long long)(uintptr_t)(
                    src ? (const void *)(src + h * head_stride(t0 + (int)threadIdx.x >= Lc)) : (const void *)zero_row);
        } else if (bx == 0 && kv0 == 0 && b == 0 && threadIdx.x < EN_KEY_TILE + D * 2 / 16) {
            reinterpret_cast<uint4 *>(zero_row)[threadIdx.x - EN_KEY_TILE] = make_uint4(0, 0, 0, 0);
        }
        return;
    }
    if (threadIdx.x < EN_KEY_TILE)
        srcs[threadIdx.x] = src;
    __syncthreads();
    // D/8 chunks of 16 bytes per token, NC of them per thread
    constexpr int CH = D / 8, NC = EN_KEY_TILE * CH / 256;
    const int tk0 = threadIdx.x / CH, ch0 = threadIdx.x % CH;
    // DIRECT: chunk by chunk into LDS, not all of them through registers: for contexts gathered agent by agent past the
    // caches (64 agents x 8 K tokens 833 / 820 us, 16 x 13 K 295 / 291); rows of 64 values as fast either way
    constexpr bool DIRECT = !AHEAD && D == 128;
    auto stage = [&](int tk, uint4 c) {
        uint16_t *d = &tile[tk * STR + ch0 * 8];
        // STR is even but not a multiple of 8: store as 4 dwords
        reinterpret_cast<uint32_t *>(d)[0] = c.x;
        reinterpret_cast<uint32_t *>(d)[1] = c.y;
        reinterpret_cast<uint32_t *>(d)[2] = c.z;
        reinterpret_cast<uint32_t *>(d)[3] = c.w;
    };
    const uint16_t *from[NC];
    bool fresh[NC];                              // a row of the new tokens
    uint4 v[NC];
    if constexpr (!DIRECT) {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const int tk = tk0 + i * (256 / CH);
            from[i] = srcs[tk];
            fresh[i] = t0 + tk >= Lc;
            v[i] = make_uint4(0, 0, 0, 0);
            if (from[i])
                v[i] = *reinterpret_cast<const uint4 *>(from[i] += ch0 * 8);
        }
    }
    uint16_t *vt = (uint16_t *)a.vt + ((size_t)b * a.Hkv + kv0) * D * (size_t)a.T + t0;
#pragma unroll 1
    for (int h = 0; h < HPB; ++h, vt += D * (size_t)a.T) {
        if constexpr (DIRECT) {
            static_assert(!DIRECT || HPB == 1);
            for (int tk = tk0; tk < EN_KEY_TILE; tk += 256 / CH) {
                uint4 c = make_uint4(0, 0, 0, 0);
                if (srcs[tk])
                    c = *reinterpret_cast<const uint4 *>(srcs[tk] + ch0 * 8);
                stage(tk, c);
            }
        } else {
#pragma unroll
            for (int i = 0; i < NC; ++i)
                stage(tk0 + i * (256 / CH), v[i]);
        }
        if (h + 1 < HPB) {
#pragma unroll
            for (int i = 0; i < NC; ++i)
                if (from[i])
                    v[i] = *reinterpret_cast<const uint4 *>(from[i] += head_stride(fresh[i]));
        }
        __syncthreads();
        // store: for every d, 8 chunks of 8 columns
        for (int idx = threadIdx.x; idx < D * 8; idx += 256) {
            const int d = idx / 8, ch = idx % 8;      // columns ch*8 .. ch*8+7
            const int g16 = ch / 2, hf = ch % 2;
            uint16_t v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int tk = 16 * g16 + 8 * (e >> 2) + 4 * hf + (e & 3);
                v[e] = tile[tk * STR + d];
            }
            u32x4 o;
            o[0] = v[0] | ((uint32_t)v[1] << 16);
            o[1] = v[2] | ((uint32_t)v[3] << 16);
            o[2] = v[4] | ((uint32_t)v[5] << 16);
            o[3] = v[6] | ((uint32_t)v[7] << 16);
            store_context<STREAM>(reinterpret_cast<u32x4 *>(vt + (size_t)d * a.T + ch * 8), o);
        }
        if (h + 1 < HPB)
            __syncthreads();
    }
}

// The first three lines of the arguments at once: a trip to memory each when the code asks for them one by one.
__device__ __forceinline__ void ask_arguments(const EnGatherLaunch &g)
{
    const EnGatherArgs &a = g.a;
    asm volatile("" ::"s"(a.k_pool), "s"(a.k_new), "s"(a.kc), "s"(a.cos_tab), "s"(a.nseg), "s"(a.bnd), "s"(a.C), "s"(a.q),
                 "s"(a.n_q_units), "s"(a.order), "s"(g.n_inline), "s"(g.n_zero));
}

// One launch for the whole gather. Grid (64-token tiles, units, agents); the units, head group
// by head group: the key units (the tile's key rows of HPB heads, which also copy fp32 values),
// then, for bf16, the value units (the same heads' transposed tiles: one unit with AHEAD, else one each). Workgroups are dispatched
// tile by tile along one unit, then the next unit: each unit is a sequential stream through
// memory (with the units of one tile side by side instead, the 8K-context gather took 18.8 us
// against 13.5), and key and value units of several heads are in flight together: they load
// different parts of a compute unit (vector memory and ALU against LDS), and a launch that ran
// all key units before all value units took the sum of the two instead of little more than the
// larger.
// When the launch carries the plan's descriptor block in its arguments, the
// tables are read from the argument segment and the first workgroup stores the
// block to device memory for the kernels that follow on the stream.
// Key units per head group: with one head per unit a 64-token tile is two units of 32 rows
// (more, shorter workgroups: what a small gather wants), with several heads one unit of two passes.
__host__ __device__ constexpr int en_gather_key_units(int hpb)
{
    return hpb == 1 ? 2 : 1;
}

// Queries prepared for the attention kernel (rows i of agent b, every head): rotated at L_c + i,
// scaled for the log2-domain softmax, rounded to bf16 once, exactly what a workgroup of the
// attention kernel would otherwise do for its own rows, once per KV split. The rows of an agent are
// dealt out over the gridDim.x workgroups of this unit; D/8 threads share a row, each takes four
// rotary pairs (k .. k+3, k + D/2 ..).
template <int D>
__device__ __forceinline__ void prepare_queries(const EnGatherArgs &a, int part, int n_parts, int b)
{
    constexpr int TPR = D / 8;                     // threads per row
    const int S = as_table(a.nseg)[b];
    const int Lc = as_table(a.bnd)[b * (a.Smax + 2) + S];
    const int rows = a.Nq * a.Hq;
    const int per = (rows + n_parts - 1) / n_parts;
    const int r1 = min(rows, (part + 1) * per);
    const int t = threadIdx.x % TPR;
    for (int row = part * per + threadIdx.x / TPR; row < r1; row += 256 / TPR) {
        const int i = row / a.Hq;
        const size_t base = ((size_t)b * rows + row) * D;
        const bf16_t *src = (const bf16_t *)a.q + base;
        const bf16x4 x1 = *reinterpret_cast<const bf16x4 *>(src + 4 * t);
        const bf16x4 x2 = *reinterpret_cast<const bf16x4 *>(src + D / 2 + 4 * t);
        const size_t trow = (size_t)(Lc + i) * (D / 2) + 4 * t;
        const f32x4 c = *reinterpret_cast<const f32x4 *>(a.cos_tab + trow);
        const f32x4 sn = *reinterpret_cast<const f32x4 *>(a.sin_tab + trow);
        bf16x4 y1, y2;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float r1f, r2f;
            rope_scale_pair((float)x1[e], (float)x2[e], c[e], sn[e], a.scale_log2e, r1f, r2f);
            y1[e] = (bf16_t)r1f;
            y2[e] = (bf16_t)r2f;
        }
        bf16_t *dst = (bf16_t *)a.q_prep + base;
        *reinterpret_cast<bf16x4 *>(dst + 4 * t) = y1;
        *reinterpret_cast<bf16x4 *>(dst + D / 2 + 4 * t) = y2;
    }
}

// n_q_units more units along y, in front of the key and value units (dispatched first, so that their short
// chains of loads run beside the streams and not behind them): the queries to prepare. True: this was one;
// else `unit` is the number of the key or value unit.
template <int D, bool ORDERED>
__device__ __forceinline__ bool query_unit(const EnGatherArgs &a, int &unit)
{
    if (unit >= a.n_q_units) {
        unit -= a.n_q_units;
        return false;
    }
    const int w = unit * gridDim.x + blockIdx.x, n = a.n_q_units * gridDim.x;
    if (!ORDERED || !a.order)
        prepare_queries<D>(a, w, n, blockIdx.z);
    else if (w < n / a.B * a.B)              // one grid for all agents, one after the other (n >= B: each has a tile)
        prepare_queries<D>(a, w % (n / a.B), n / a.B, w / (n / a.B));
    return true;
}

// Which agent's 64-token tile a workgroup of a key or value unit takes (false: none). Without an order the grid
// says it. With one (EnGatherArgs::order) the workgroups of an XCD, every eighth of the grid, go through that XCD's
// list of entries; an entry is up to 1 << order_shift neighbouring tiles of an agent.
template <bool ORDERED>
__device__ __forceinline__ bool gather_where(const EnGatherArgs &a, int &tile, int &b)
{
    tile = blockIdx.x;
    b = blockIdx.z;
    if (ORDERED && a.order) {
        const unsigned q = blockIdx.x / EN_XCDS;
        const en_table_ptr e = as_table(a.order) + 2 * ((size_t)(q >> a.order_shift) * EN_XCDS + blockIdx.x % EN_XCDS);
        const int j = q & ((1 << a.order_shift) - 1);
        b = e[0];
        tile = (e[1] >> 2) + j;
        return j <= (e[1] & 3) && b >= 0;
    }
    return true;
}

// Workgroups of eight heads ahead: three on a compute unit, not the four that their registers allow. The streams of a
// fourth cost more than its loads hide: 64 agents x 16 K tokens 1054 / 1065 us (two: 1093), 16 x 14 K 264 / 270 (268),
// 32 x 4 K 171 / 174 (167).
constexpr int en_gather_waves(int hpb, bool ahead)
{
    return ahead && hpb == 8 ? 3 : 8;
}

template <typename T, int D, int HPB, bool STREAM, bool AHEAD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, en_gather_waves(HPB, AHEAD)))) void gather_kernel(EnGatherLaunch g)
{
    ask_arguments(g);
    EnGatherArgs a = g.a;
    if (g.n_inline > 0) {
        const int32_t *img = reinterpret_cast<const int32_t *>(
            reinterpret_cast<uintptr_t>(__builtin_amdgcn_kernarg_segment_ptr()) + offsetof(EnGatherLaunch, desc));
        tables_in(a, img);
        if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0)
        {
            for (int i = threadIdx.x; i < g.n_inline; i += 256)
                g.desc_out[i] = img[i];
            for (int i = threadIdx.x; i < g.n_zero; i += 256)
                g.desc_out[g.n_inline + i] = 0;
        }
    }
    __shared__ int32_t lbnd[2 * EN_GATHER_TAB_LDS];       // bucket bounds, then selected groups
    constexpr bool ORDERED = STREAM && AHEAD;                 // may come in an order
    constexpr int KU = en_gather_key_units(HPB);
    constexpr int VPB = AHEAD ? HPB : 1;                      // heads per value unit
    constexpr int PER = KU + (sizeof(T) == 2 ? HPB / VPB : 0);      // units per head group
    int unit = blockIdx.y;
    if constexpr (sizeof(T) == 2) {
        if (a.q && query_unit<D, ORDERED>(a, unit))
            return;
    }
    int tile, b;
    if (!gather_where<ORDERED>(a, tile, b))
        return;
    const int hg = unit / PER, r = unit % PER;
    if (r < KU)
        gather_k_block<T, D, sizeof(T) == 4, HPB, STREAM, AHEAD>(a, b, tile, KU == 2 ? r : 0, KU == 2 ? r : 1, hg * HPB, lbnd);
    else if constexpr (sizeof(T) == 2)
        gather_vt_block<D, VPB, STREAM, AHEAD>(a, b, tile, hg * HPB + (r - KU) * VPB, lbnd);
}

// ---------------------------------------------------------------------------
// gather from an 8-bit pool: the same bf16 contexts as above from rows of int8
// codes with one float scale per (group, head, token): value = code * scale in
// float32, keys rotated, everything rounded to bf16 once. New tokens arrive in
// bf16 as ever. grid as for the bf16 gather, the units by gather_heads_q8.
// ---------------------------------------------------------------------------
struct EnCtxLoc {
    int kind;        // 0 padding, 1 row of the pool, 2 row of the new tokens
    size_t row;      // index of the row, in rows of D elements
};
__device__ __forceinline__ EnCtxLoc context_loc(const EnGatherArgs &a, const EnGatherTables &t, const int32_t *lds,
                                               int b, int kvh, int tok)
{
    int group, row;
    context_row(t, lds, tok, group, row);
    if (tok >= t.Ltot)
        return {0, 0};
    if (tok >= t.Lc)
        return {2, ((size_t)b * a.Nq + (tok - t.Lc)) * a.Hkv + kvh};
    return {1, ((size_t)group * a.Hkv + kvh) * a.C + row};
}

// The key rows of HPB heads, kv0 onwards: where the row comes from, its cosines and sines once for all of them, and
// the codes of all of them on their way before the first are turned and stored. The codes are asked for first, the cosines
// and sines behind them (with nothing in the caches 24 agents x 2 K tokens of 2 heads of 64 values 14.0 / 13.7 us, 8 x 6 K
// 17.1 / 16.8), of a single head of 128 values when its codes have come: 3 agents x 2 K tokens 12.2 / 11.7, one agent's
// 24 K of 2 heads 15.1 / 14.9, 6 K of 8 heads 13.2 / 13.0, but its 0.5 K of 2 heads 4.24 / 4.36.
template <int D, int HPB, bool STREAM>
__device__ __forceinline__ void gather_q8_k_rows(const EnGatherArgs &a, const EnGatherTables &tabs, int b, int tok,
                                                 int kv0, int32_t *lds)
{
    constexpr int E = D / 16;
    const int c = threadIdx.x % 8;
    const EnCtxLoc loc = context_loc(a, tabs, lds, b, kv0, tok);
    const int Lpad = (tabs.Ltot + EN_KEY_TILE - 1) / EN_KEY_TILE * EN_KEY_TILE;
    if (tok >= Lpad)
        return;
    typedef bf16_t tvec __attribute__((ext_vector_type(E)));
    typedef float fvec __attribute__((ext_vector_type(E)));
    auto store = [&](int h, fvec y1, fvec y2) {
        bf16_t *dst = (bf16_t *)a.kc + (((size_t)b * a.Hkv + kv0 + h) * a.T + tok) * D;
        store_context<STREAM>(dst + c * E, __builtin_convertvector(y1, tvec));
        store_context<STREAM>(dst + D / 2 + c * E, __builtin_convertvector(y2, tvec));
    };
    if (loc.kind == 0) {
#pragma unroll
        for (int h = 0; h < HPB; ++h)
            store(h, 0.f, 0.f);
        return;
    }
    fvec cs, sn;
    auto angles = [&] {
        cs = *reinterpret_cast<const fvec *>(a.cos_tab + (size_t)tok * (D / 2) + c * E);
        sn = *reinterpret_cast<const fvec *>(a.sin_tab + (size_t)tok * (D / 2) + c * E);
    };
    auto turn = [&](int h, fvec x1, fvec x2) {
        fvec y1, y2;
        rope_key_pair<true>(x1, x2, cs, sn, y1, y2);
        store(h, y1, y2);
    };
    int8_t c1[HPB][E], c2[HPB][E];
    float sc[HPB];
    auto codes = [&] {
#pragma unroll
        for (int h = 0; h < HPB; ++h) {
            const size_t row = loc.row + (size_t)h * a.C;
            const int8_t *src = (const int8_t *)a.k_pool + row * D;
            __builtin_memcpy(c1[h], src + c * E, E);
            __builtin_memcpy(c2[h], src + D / 2 + c * E, E);
            sc[h] = a.k_scale[row];
        }
    };
    auto scaled = [&](int h, fvec &x1, fvec &x2) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            x1[e] = (float)c1[h][e] * sc[h];
            x2[e] = (float)c2[h][e] * sc[h];
        }
    };
    auto fresh = [&](int h, fvec &x1, fvec &x2) {
        const bf16_t *src = (const bf16_t *)a.k_new + (loc.row + h) * D;
        x1 = __builtin_convertvector(*reinterpret_cast<const tvec *>(src + c * E), fvec);
        x2 = __builtin_convertvector(*reinterpret_cast<const tvec *>(src + D / 2 + c * E), fvec);
    };
    if constexpr (HPB == 1 && D == 128) {
        fvec x1, x2;
        if (loc.kind == 1) {
            codes();
            scaled(0, x1, x2);
        } else {
            fresh(0, x1, x2);
        }
        asm volatile("" : "+v"(x1), "+v"(x2)::"memory");          // (before the angles)
        angles();
        turn(0, x1, x2);
    } else if (loc.kind == 1) {
        codes();
        angles();
        if constexpr (HPB > 1)
            asm volatile("" ::: "memory");             // (not behind the stores)
#pragma unroll
        for (int h = 0; h < HPB; ++h) {
            fvec x1, x2;
            scaled(h, x1, x2);
            turn(h, x1, x2);
        }
    } else {
        angles();
#pragma unroll
        for (int h = 0; h < HPB; ++h) {
            fvec x1, x2;
            fresh(h, x1, x2);
            turn(h, x1, x2);
        }
    }
}

template <int D, int HPB, bool STREAM>
__device__ __forceinline__ void gather_q8_k_block(const EnGatherArgs &a, int b, int tile, int kv0, int32_t *lds)
{
    const EnGatherTables tabs = open_tables(a, b, lds);
#pragma unroll 1
    for (int half = 0; half < 2; ++half)
        gather_q8_k_rows<D, HPB, STREAM>(a, tabs, b, tile * EN_KEY_TILE + half * 32 + threadIdx.x / 8, kv0, lds);
}

// The transposed values of a tile for HPB heads, kv0 onwards, one after the other, the next head's loads on their way
// meanwhile.
template <int D, int HPB, bool STREAM>
__device__ __forceinline__ void gather_q8_vt_block(const EnGatherArgs &a, int b, int bx, int kv0, int32_t *lds)
{
    constexpr int STR = D + 2;                 // LDS row stride in elements
    __shared__ uint16_t tile[EN_KEY_TILE * STR];
    __shared__ size_t rows[EN_KEY_TILE];
    __shared__ int kinds[EN_KEY_TILE];
    const int t0 = bx * EN_KEY_TILE;
    const EnGatherTables tabs = open_tables(a, b, lds);
    if (t0 >= tabs.Ltot)                            // the same for the whole block
        return;
    if (threadIdx.x < EN_KEY_TILE) {
        const EnCtxLoc loc = context_loc(a, tabs, lds, b, kv0, t0 + threadIdx.x);
        rows[threadIdx.x] = loc.row;
        kinds[threadIdx.x] = loc.kind;
    }
    __syncthreads();
    typedef bf16_t bvec __attribute__((ext_vector_type(8)));
    typedef float fvec8 __attribute__((ext_vector_type(8)));
    // D/8 chunks of 8 elements per token, NC of them per thread
    constexpr int CH = D / 8, NC = EN_KEY_TILE * CH / 256;
    const int tk0 = threadIdx.x / CH, ch0 = threadIdx.x % CH;
    int kind[NC];
    size_t row[NC];
    uint4 raw[NC];                             // 8 codes, or 8 values of a new token
    float sc[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        kind[i] = kinds[tk0 + i * (256 / CH)];
        row[i] = rows[tk0 + i * (256 / CH)];
    }
    auto load = [&] {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            if (kind[i] == 1) {
                __builtin_memcpy(&raw[i], (const int8_t *)a.v_pool + row[i] * D + ch0 * 8, 8);
                sc[i] = a.v_scale[row[i]];
                row[i] += a.C;
            } else if (kind[i] == 2) {
                raw[i] = *reinterpret_cast<const uint4 *>((const bf16_t *)a.v_new + row[i] * D + ch0 * 8);
                row[i] += 1;
            }
        }
    };
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        raw[i] = make_uint4(0, 0, 0, 0);
        sc[i] = 0.f;
    }
    load();
    uint16_t *vt = (uint16_t *)a.vt + ((size_t)b * a.Hkv + kv0) * D * (size_t)a.T + t0;
#pragma unroll 1
    for (int h = 0; h < HPB; ++h, vt += D * (size_t)a.T) {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            uint4 w = raw[i];
            if (kind[i] == 1) {
                int8_t cd[8];
                __builtin_memcpy(cd, &raw[i], 8);
                fvec8 f;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    f[e] = (float)cd[e] * sc[i];
                const bvec v = __builtin_convertvector(f, bvec);
                __builtin_memcpy(&w, &v, 16);
            }
            uint16_t *d = &tile[(tk0 + i * (256 / CH)) * STR + ch0 * 8];
            // STR is even but not a multiple of 8: store as 4 dwords
            reinterpret_cast<uint32_t *>(d)[0] = w.x;
            reinterpret_cast<uint32_t *>(d)[1] = w.y;
            reinterpret_cast<uint32_t *>(d)[2] = w.z;
            reinterpret_cast<uint32_t *>(d)[3] = w.w;
        }
        if (h + 1 < HPB)
            load();
        __syncthreads();
        // store: for every d, 8 chunks of 8 columns (the same order as the bf16 gather)
        for (int idx = threadIdx.x; idx < D * 8; idx += 256) {
            const int d = idx / 8, ch = idx % 8;      // columns ch*8 .. ch*8+7
            const int g16 = ch / 2, hf = ch % 2;
            uint16_t v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int tk = 16 * g16 + 8 * (e >> 2) + 4 * hf + (e & 3);
                v[e] = tile[tk * STR + d];
            }
            u32x4 o;
            o[0] = v[0] | ((uint32_t)v[1] << 16);
            o[1] = v[2] | ((uint32_t)v[3] << 16);
            o[2] = v[4] | ((uint32_t)v[5] << 16);
            o[3] = v[6] | ((uint32_t)v[7] << 16);
            store_context<STREAM>(reinterpret_cast<u32x4 *>(vt + (size_t)d * a.T + ch * 8), o);
        }
        if (h + 1 < HPB)
            __syncthreads();
    }
}

template <int D, int HPB, bool STREAM>
__global__ __launch_bounds__(256) void gather_q8_kernel(EnGatherLaunch g)
{
    ask_arguments(g);
    EnGatherArgs a = g.a;
    if (g.n_inline > 0) {
        const int32_t *img = reinterpret_cast<const int32_t *>(
            reinterpret_cast<uintptr_t>(__builtin_amdgcn_kernarg_segment_ptr()) + offsetof(EnGatherLaunch, desc));
        tables_in(a, img);
        if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0)
        {
            for (int i = threadIdx.x; i < g.n_inline; i += 256)
                g.desc_out[i] = img[i];
            for (int i = threadIdx.x; i < g.n_zero; i += 256)
                g.desc_out[g.n_inline + i] = 0;
        }
    }
    __shared__ int32_t ltab[2 * EN_GATHER_TAB_LDS];       // bucket bounds, then selected groups
    // per HPB heads one key unit, one value unit
    int unit = blockIdx.y;
    if (a.q && query_unit<D, false>(a, unit))
        return;
    const int tile = blockIdx.x, b = blockIdx.z;
    const int kv0 = unit / 2 * HPB;
    if (unit % 2 == 0)
        gather_q8_k_block<D, HPB, STREAM>(a, b, tile, kv0, ltab);
    else
        gather_q8_vt_block<D, HPB, STREAM>(a, b, tile, kv0, ltab);
}

// ---------------------------------------------------------------------------
// ctx_append: the keys and values of a decode step's new tokens join the
// gathered context at positions L_c + q_first + t (keys rotated there; values
// in the context's layout). grid: (n, Hkv, B), D/2 threads: thread c owns the
// rotary pair (c, c + D/2).
// ---------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(D / 2) void ctx_append_kernel(EnCtxAppendArgs a)
{
    const int t = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int c = threadIdx.x;
    const int pos = a.hdr[4 * b + 1] + a.q_first + t;
    const T *kr = (const T *)a.k_rows + (((size_t)b * a.n + t) * a.Hkv + h) * D;
    const T *vr = (const T *)a.v_rows + (((size_t)b * a.n + t) * a.Hkv + h) * D;
    const float cs = a.cos_tab[(size_t)pos * (D / 2) + c], sn = a.sin_tab[(size_t)pos * (D / 2) + c];
    const float x1 = (float)kr[c], x2 = (float)kr[c + D / 2];
    T *kd = (T *)a.kc + (((size_t)b * a.Hkv + h) * a.T + pos) * D;
    float y1, y2;
    rope_key_pair(x1, x2, cs, sn, y1, y2);
    kd[c] = (T)y1;
    kd[c + D / 2] = (T)y2;
    if constexpr (sizeof(T) == 4) {
        T *vd = (T *)a.vt + (((size_t)b * a.Hkv + h) * a.T + pos) * D;
        vd[c] = vr[c];
        vd[c + D / 2] = vr[c + D / 2];
    } else {
        // transposed layout [D][T], token j in column j with bits 2 and 3 exchanged
        const int col = (pos & ~0xC) | ((pos & 4) << 1) | ((pos & 8) >> 1);
        T *vd = (T *)a.vt + ((size_t)b * a.Hkv + h) * (size_t)D * a.T + col;
        vd[(size_t)c * a.T] = vr[c];
        vd[(size_t)(c + D / 2) * a.T] = vr[c + D / 2];
    }
}

// ---------------------------------------------------------------------------
// tier load: blocks of the pinned host store go to device slots (Section 3.2:
// the selected groups' KV is loaded from the slow store, once). The kernel
// reads host memory directly, 16 bytes per lane and four loads in flight per
// lane, so one launch moves every missing block of a step and, unlike a chain
// of copy commands, queues behind an event without holding up the host.
// grid: (chunks of 16 KB along a head's used rows, 2 * Hkv, blocks), 256 threads.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void tier_load_kernel(EnTierLoadArgs a)
{
    const int32_t *desc = reinterpret_cast<const int32_t *>(
        reinterpret_cast<uintptr_t>(__builtin_amdgcn_kernarg_segment_ptr()) + offsetof(EnTierLoadArgs, desc));
    const int m = blockIdx.z;
    const int group = desc[3 * m], slot = desc[3 * m + 1], tokens = desc[3 * m + 2];
    const int h = blockIdx.y >> 1, is_v = blockIdx.y & 1;
    const int units = tokens * (a.row_bytes / 16);           // 16-byte units of this head in use
    const int first = blockIdx.x * 1024 + threadIdx.x;
    if (blockIdx.x * 1024 >= units)
        return;
    const size_t head_off = (size_t)h * a.head_bytes;
    const uint4 *src = reinterpret_cast<const uint4 *>((is_v ? a.v_store : a.k_store) +
                                                       (size_t)group * a.block_bytes + head_off);
    uint4 *dst = reinterpret_cast<uint4 *>((is_v ? a.v_slots : a.k_slots) + (size_t)slot * a.block_bytes + head_off);
    uint4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (first + 256 * j < units)
            v[j] = src[first + 256 * j];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (first + 256 * j < units)
            dst[first + 256 * j] = v[j];
}

// ---------------------------------------------------------------------------
// append: rows [n, Hkv, D] go to tokens first .. first+n-1 of one group's block
// [Hkv, C, D] in both pool arrays (Section 3.2: new objects' KV is saved at the
// end of the group's cache). One thread per 16 bytes; grid.y: 0 keys, 1 values.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void append_kernel(EnAppendArgs a)
{
    // n rows of one group: n <= C, so the chunk count fits 32 bits with room to spare
    const unsigned idx = blockIdx.x * 256u + threadIdx.x;
    const unsigned total = (unsigned)a.n * a.Hkv * a.row_chunks;
    if (idx >= total)
        return;
    const unsigned rowi = idx / (unsigned)a.row_chunks;          // tok * Hkv + h
    const unsigned c = idx - rowi * (unsigned)a.row_chunks;
    const unsigned tok = rowi / (unsigned)a.Hkv;
    const unsigned h = rowi - tok * (unsigned)a.Hkv;
    const uint4 *src = reinterpret_cast<const uint4 *>(blockIdx.y == 0 ? a.k_rows : a.v_rows);
    uint4 *dst = reinterpret_cast<uint4 *>(blockIdx.y == 0 ? a.k_pool : a.v_pool);
    const size_t drow = ((size_t)a.group * a.Hkv + h) * a.C + a.first + tok;
    dst[drow * a.row_chunks + c] = src[(size_t)rowi * a.row_chunks + c];
}

// ---------------------------------------------------------------------------
// append to an 8-bit pool: one wave per (token, head) row and array. The row's
// largest magnitude fixes the scale (max|x| / 127), the codes are x / scale
// rounded to the nearest integer, ties to even, all in float32; a zero row has
// scale 0. grid: (n, Hkv, 2), 64 threads.
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(64) void append_q8_kernel(EnAppendQ8Args a)
{
    constexpr int EPL = D / 64;               // elements per lane
    const int tok = blockIdx.x, h = blockIdx.y, lane = threadIdx.x;
    const bf16_t *src = (const bf16_t *)(blockIdx.z == 0 ? a.k_rows : a.v_rows) + ((size_t)tok * a.Hkv + h) * D;
    float x[EPL];
    float amax = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
        x[e] = (float)src[lane * EPL + e];
        amax = fmaxf(amax, fabsf(x[e]));
    }
    amax = wave_max(amax);
    const float scale = amax / 127.0f;
    const size_t row = ((size_t)a.group * a.Hkv + h) * a.C + a.first + tok;
    int8_t *dst = (blockIdx.z == 0 ? a.k_pool : a.v_pool) + row * D;
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
        float q = scale > 0.f ? rintf(x[e] / scale) : 0.f;
        q = fminf(fmaxf(q, -127.f), 127.f);
        dst[lane * EPL + e] = (int8_t)(int)q;
    }
    if (lane == 0)
        (blockIdx.z == 0 ? a.k_scale : a.v_scale)[row] = scale;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// Heads per key unit of the forms without AHEAD: as many (8, 4, 2 that divide Hkv) as still leave 32 workgroups per
// compute unit (counted with a value unit per head).
static int gather_heads_many(const en_pool *pool, const EnGatherArgs &a, int n_tiles, bool with_value_units)
{
    for (int hpb = 8; hpb > 1; hpb /= 2) {
        const long units = (long)(a.Hkv / hpb) * (en_gather_key_units(hpb) + (with_value_units ? hpb : 0));
        if (a.Hkv % hpb == 0 && units * n_tiles * a.B >= 32L * pool->n_cu)
            return hpb;
    }
    return 1;
}

// Rows of a gather: query rows to prepare, rows of keys and values.
struct EnGatherRows {
    long queries, keys_values;
};

// Heads per unit with AHEAD: at most as many as leave 1.25 workgroups per compute unit, and
// - past the caches, where many rounds of workgroups follow each other, eight: gather and attention, us, with one / two /
//   four / eight heads, 1300 tiles (of 8 heads) 233 / 228 / 217 / 214, 6200: 965 / 840 / 823 / 805;
// - two where eight would be more than four workgroups per compute unit (three, of eight heads, to five fit one), the last
//   round of them alone: 528 tiles 129.2 / 125.7 / 127.3 / 129.7, 784: 130.2 / 130.7 / 133.0 / 135.2;
// - else one for contexts of under 24 tiles, two of six agents and more with under 60, four of three agents and more:
//   many short runs through memory gain by neither. The gather with nothing in the caches, one / two / four / eight heads:
//   24 agents x 3 runs (9 tiles) 20.2 / 20.3 / 20.4 / 22.3, 24 x 18 tiles of 2 heads 12.4 / 14.5, of 4 heads 20.4 / 21.1 /
//   23.3, 6 x 33 tiles 21.7 / 22.9 / 23.9 / 24.8, 12 x 32 34.8 / 32.8 / 34.3 / 34.1 (but 12 x 16 21.1 / 21.8 / 20.1 / 19.9),
//   4 x 104: 0.96 / 0.93 / 0.97 / 1.03 of the time without loads ahead, 8 x 107 of 4 heads 49.8 / 42.7 / 41.1, one agent's
//   201 28.1 / 24.7 / 25.0 / 24.6; in them, with the attention, 2 x 97 56.7 / 55.5 / 53.0 / 50.9, one agent's 137 88.8 / 88.6
//   / 88.9 / 90.3.
// With one query row to six of keys and values and more, at most four: eight heads are 132 registers, three workgroups to
// a compute unit, four are 96 and five, and queries prepared beside them want the more. The gather, us, with eight / four:
// 64 agents with 512 new tokens of 2.3 K, keys only (0.44 to 1) 228 / 209, with values (0.22) 318 / 310, 16 of 4.1 K, keys
// only (0.25) 78 / 72; but 2 with 512 of 7.7 K (0.13) 26.3 / 26.7, 24 with 130 of 11 K, keys only (0.05) 139 / 144, though
// 130 with 64 of 2 K (0.06) 252 / 243.
static int gather_heads_ahead(const en_pool *pool, const EnGatherArgs &a, const EnGatherRows &rows, int n_tiles)
{
    int hpb = 6 * rows.queries < rows.keys_values ? 8 : 4;
    const long work = (a.v_rows ? 1L : 2L) * a.Hkv * n_tiles * a.B;                  // (tile, head), keys and values
    if (!a.stream) {
        if (work > 8 * 4L * pool->n_cu)
            hpb = 2;
        else if (n_tiles < 24)
            hpb = 1;
        else if (a.B >= 6 && n_tiles < 60)
            hpb = 2;
        else if (a.B > 2)
            hpb = 4;
    }
    while (hpb > 1 && (a.Hkv % hpb || 4 * work < 5L * hpb * pool->n_cu))
        hpb /= 2;
    return hpb;
}

// AHEAD: a workgroup takes the keys, or the values, of several heads with the next heads' loads on their way (bf16 rows
// of 128 values). Gather and attention, us, without / with: 194 tiles of 8 heads 57.7 / 51.8, 390: 86.8 / 78.5, 528:
// 133 / 128. Not where a context of three times the last-level cache and more is gathered agent by agent: 16
// agents x 12 K tokens 433 / 445, 64 x 6 K 832 / 850, 64 x 16 K 2173 / 2217 (in order, see en_gather_order: 1806).
// Rows of 64 values: 64 agents x 16 K tokens 797 / 817.
// Nor where queries to prepare are most of a launch of several heads a workgroup, whose registers leave them fewer waves:
// from three query rows to two of keys and values on, in the caches from as many on. The gather, us: 16 agents with 512
// new tokens of 1 K (1.1 to 1) 45.8 / 48.9, with 1 K of 1.4 K (1.5) 86.5 / 87.2, keys only 16 with 512 of 1 K (2.1)
// 38.7 / 44.9 and 128 with 512 of 0.9 K (2.3) 291 / 321; but past the caches 128 with 512 of 0.9 K (1.1) 363 / 344, 64 with
// 512 of 1.4 K, keys only (1.5), 186 / 175. Of one head: 2 agents with 512 of 1 K (1.1) 7.98 / 7.58.
static bool gather_ahead(const en_plan *plan, const EnGatherArgs &a, const EnGatherRows &rows, int heads)
{
    const en_pool *pool = plan->pool;
    if (pool->d.dtype != EN_BF16 || pool->d.head_dim != 128 ||
        (!a.order && 2 * en_context_bytes(pool, plan) >= EN_GATHER_HUGE_BYTES))
        return false;
    return heads == 1 || 2 * rows.queries < (a.stream ? 3 : 2) * rows.keys_values;
}

template <typename T, int D, bool STREAM, bool AHEAD>
static void launch_gather_hpb(int hpb, dim3 grid, hipStream_t st, const EnGatherLaunch &g)
{
    const dim3 blk(256);
    if (hpb == 8)
        hipLaunchKernelGGL((gather_kernel<T, D, 8, STREAM, AHEAD>), grid, blk, 0, st, g);
    else if (hpb == 4)
        hipLaunchKernelGGL((gather_kernel<T, D, 4, STREAM, AHEAD>), grid, blk, 0, st, g);
    else if (hpb == 2)
        hipLaunchKernelGGL((gather_kernel<T, D, 2, STREAM, AHEAD>), grid, blk, 0, st, g);
    else
        hipLaunchKernelGGL((gather_kernel<T, D, 1, STREAM, AHEAD>), grid, blk, 0, st, g);
}

template <typename T, int D>
static void launch_gather_kernel(bool ahead, int hpb, dim3 grid, hipStream_t st, const EnGatherLaunch &g)
{
    if constexpr (sizeof(T) == 2 && D == 128)
        if (ahead) {
            if (g.a.stream)
                launch_gather_hpb<T, D, true, true>(hpb, grid, st, g);
            else
                launch_gather_hpb<T, D, false, true>(hpb, grid, st, g);
            return;
        }
    if (g.a.stream)
        launch_gather_hpb<T, D, true, false>(hpb, grid, st, g);
    else
        launch_gather_hpb<T, D, false, false>(hpb, grid, st, g);
}

// Heads per unit of the gather from 8-bit pools: four where the context goes past the caches and the launch is many
// rounds of workgroups, two from 16 or 18 (tile, head) units per compute unit on (about two rounds), one below. Gather and
// attention, us, with one / two / four / eight heads: 64 agents x 16 K tokens 2316 / 2116 / 1984 / 1976, rows of 64
// values 1233 / 1101 / 1044 / 1011, 32 x 6 K 430 / 406 / 399 / 409, 16 x 14 K 532 / 502 / 486 / 491; kept in the
// caches 16 x 2 K (9000 units) 138.4 / 136.1 / 138.2 / 145.0, rows of 64 values 84.0 / 80.9 / 82.5 / 83.9; 3600 units
// 56.5 / 57.5 / 56.7 / 61.0, 2200: 90.4 / 90.7 / 92.9 / 98.9, 450: 38.1 / 39.1 / 42.6 / 49.4. Rows of 128 values from 18
// units on: the gather with nothing in the caches, one / two heads, 4096 units 25.9 / 27.2, 4800: 31.6 / 30.3; rows of
// 64, 4096 units: 0.93 of the time with two.
static int gather_heads_q8(const en_pool *pool, const EnGatherArgs &a, int n_tiles)
{
    const long line = pool->d.head_dim == 128 ? 18 : 16;
    int hpb = a.stream ? 4 : 2L * a.Hkv * n_tiles * a.B >= line * pool->n_cu ? 2 : 1;
    while (a.Hkv % hpb)
        hpb /= 2;
    return hpb;
}

template <int D, bool STREAM>
static void launch_gather_q8(int hpb, dim3 grid, hipStream_t st, const EnGatherLaunch &g)
{
    const dim3 blk(256);
    if constexpr (STREAM)
        if (hpb == 4) {                              // (past the caches only)
            hipLaunchKernelGGL((gather_q8_kernel<D, 4, STREAM>), grid, blk, 0, st, g);
            return;
        }
    if (hpb == 2)
        hipLaunchKernelGGL((gather_q8_kernel<D, 2, STREAM>), grid, blk, 0, st, g);
    else
        hipLaunchKernelGGL((gather_q8_kernel<D, 1, STREAM>), grid, blk, 0, st, g);
}

int en_launch_gather(const en_plan *plan, EnGatherLaunch &g, void *stream)
{
    const en_pool *pool = plan->pool;
    const EnGatherArgs &a = g.a;
    hipStream_t st = (hipStream_t)stream;
    const int n_tiles = (plan->max_ctx_len + EN_KEY_TILE - 1) / EN_KEY_TILE;
    const int D = pool->d.head_dim;
    if (pool->d.dtype == EN_I8) {
        const int hpb = gather_heads_q8(pool, a, n_tiles);
        const dim3 grid(n_tiles, 2 * (a.Hkv / hpb) + (a.q ? a.n_q_units : 0), a.B);
        if (D == 64 && a.stream)
            launch_gather_q8<64, true>(hpb, grid, st, g);
        else if (D == 64)
            launch_gather_q8<64, false>(hpb, grid, st, g);
        else if (a.stream)
            launch_gather_q8<128, true>(hpb, grid, st, g);
        else
            launch_gather_q8<128, false>(hpb, grid, st, g);
        return (int)hipGetLastError();
    }
    const bool bf16 = pool->d.dtype != EN_F32;
    const int many = gather_heads_many(pool, a, n_tiles, bf16);
    // which heads' keys are turned in which form (rope_key_pair) goes by the number of heads that this rule gives
    g.a.rope_unit = en_rope_unit(bf16 ? 2 : 4, D, many);
    const long tokens = plan->total_cached + long(plan->B) * plan->Nq;
    const EnGatherRows rows = {a.q ? long(plan->B) * plan->Nq * a.Hq : 0, (a.v_rows ? 1 : 2) * tokens * a.Hkv};
    const int heads = gather_heads_ahead(pool, a, rows, n_tiles);
    const bool ahead = gather_ahead(plan, a, rows, heads);
    if (!ahead)
        g.a.order = nullptr;                                     // (the order is for that form)
    const int hpb = ahead ? heads : many;
    const int value_units = !bf16 ? 0 : ahead ? 1 : hpb;         // per key unit's heads
    // (n_q_units more units along y when the launch also prepares the queries: bf16 contexts only)
    const dim3 grid(a.order ? int(plan->order_ints / 2) << plan->order_shift : n_tiles,
                    (a.Hkv / hpb) * (en_gather_key_units(hpb) + value_units) + (bf16 && a.q ? a.n_q_units : 0),
                    a.order ? 1 : a.B);
    if (!bf16) {
        if (D == 64)
            launch_gather_kernel<float, 64>(ahead, hpb, grid, st, g);
        else
            launch_gather_kernel<float, 128>(ahead, hpb, grid, st, g);
    } else {
        if (D == 64)
            launch_gather_kernel<bf16_t, 64>(ahead, hpb, grid, st, g);
        else
            launch_gather_kernel<bf16_t, 128>(ahead, hpb, grid, st, g);
    }
    return (int)hipGetLastError();
}

int en_launch_ctx_append(const en_pool *pool, const EnCtxAppendArgs &a, void *stream)
{
    const int D = pool->d.head_dim;
    const dim3 grid(a.n, a.Hkv, a.B), blk(D / 2);
    hipStream_t st = (hipStream_t)stream;
    if (pool->d.dtype == EN_F32) {
        if (D == 64)
            hipLaunchKernelGGL((ctx_append_kernel<float, 64>), grid, blk, 0, st, a);
        else
            hipLaunchKernelGGL((ctx_append_kernel<float, 128>), grid, blk, 0, st, a);
    } else {
        if (D == 64)
            hipLaunchKernelGGL((ctx_append_kernel<bf16_t, 64>), grid, blk, 0, st, a);
        else
            hipLaunchKernelGGL((ctx_append_kernel<bf16_t, 128>), grid, blk, 0, st, a);
    }
    return (int)hipGetLastError();
}

int en_launch_tier_load(const EnTierLoadArgs &a, int max_tokens, void *stream)
{
    const int units = max_tokens * (a.row_bytes / 16);
    const dim3 grid((units + 1023) / 1024, 2 * a.Hkv, a.n), blk(256);
    hipLaunchKernelGGL(tier_load_kernel, grid, blk, 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

int en_launch_append_q8(const en_pool *pool, const EnAppendQ8Args &a, void *stream)
{
    const dim3 grid(a.n, a.Hkv, 2), blk(64);
    if (pool->d.head_dim == 64)
        hipLaunchKernelGGL((append_q8_kernel<64>), grid, blk, 0, (hipStream_t)stream, a);
    else
        hipLaunchKernelGGL((append_q8_kernel<128>), grid, blk, 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

int en_launch_append(const en_pool *pool, const EnAppendArgs &a, void *stream)
{
    (void)pool;
    const size_t total = (size_t)a.n * a.Hkv * a.row_chunks;
    const dim3 grid((unsigned)((total + 255) / 256), 2), blk(256);
    hipLaunchKernelGGL(append_kernel, grid, blk, 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}
