// attn_decode, attn_once: the same attention for steps of few query rows (the decode phase
// of a planning step, Section 3.2): contexts streamed through, bound by reading them once, and
// those that fit the chip's LDS in a round or a few, bound by latency; and attn_f32, the fp32 matrix-core path of small configurations.
#include "en_device.h"

// ---------------------------------------------------------------------------
// attn_decode (bf16): few query rows per KV head (r * N_q <= 32, e.g. one new
// token per agent in the decode phase of a planning step, Section 3.2: about 40
// tokens are decoded per plan over the KV that was loaded once).
//
// This case is bound by reading the gathered K / V^T once from HBM, not by the
// matrix cores, so the work is cut for bandwidth: one wave per (agent, KV head,
// KV split), no workgroup barrier at all. All r * N_q query rows of the KV head
// are columns of the wave's one 32-column Q^T block (column c = head_local *
// N_q + i). The wave streams its key range in 64-key load tiles through its own
// two LDS stages (the loads of tile j+1 run while tile j is computed): 64 keys
// are one whole 128-byte line of every V^T row, and reading V^T in half lines
// costs a fifth of the bandwidth. A tile is two 32-key blocks whose score
// chains, exponentials and products are independent of each other, which is
// all the instruction-level parallelism a wave that is alone on its SIMD has:
// S^T = K Q^T, the exponentials and O^T += V^T P^T as in the prefill kernel. Partial results of the splits are merged by the same combine
// and mass kernels.
// ---------------------------------------------------------------------------
template <int D, int SUB>
__global__ __launch_bounds__(64 * SUB) void attn_decode_kernel(EnAttnArgs a)
{
    // SUB = 2: two waves share the unit's tiles (each issues half of a tile's loads and takes one
    // of its two 32-key blocks, with softmax state, partial output and segment sums of its own,
    // stored at partial-result index sp * 2 + wave). For steps that leave compute units idle: a
    // wave alone on its SIMD takes about 2 us per tile, and the tiles' LDS stages allow two
    // workgroups per compute unit, so this puts all four SIMDs to work.
    static_assert(SUB == 1 || SUB == 2, "one or two waves per unit");
    // two LDS stages; a third (two tiles in flight per wave) was tried for grids of at most one
    // wave per compute unit and changed nothing: a lone wave is bound by issuing its own
    // instructions (about 2 us per tile), not by waiting for its loads
    constexpr int NST = 2;
    constexpr int KB = 32;                       // keys per matrix-instruction block
    constexpr int LB = EN_KEY_TILE;              // keys per tile
    constexpr int NU = LB / KB;                  // blocks per tile
    constexpr int NKS = D / 16;
    constexpr int NDB = D / 32;
    constexpr int ROWB = 2 * D;
    constexpr int KSTR = ROWB + 16;              // padded K row in LDS
    constexpr int KCPR = KSTR / 16;
    constexpr int KCHUNKS = LB * KCPR;           // 16-byte chunks of a K tile
    constexpr int NBK = KCHUNKS / 64;            // loader blocks
    constexpr int KBYTES = NBK * 1024;
    constexpr int VSTR = LB * 2 + 16;            // padded V^T row in LDS (144 bytes)
    constexpr int VCPR = VSTR / 16;
    constexpr int VCHUNKS = D * VCPR;
    constexpr int NBV = VCHUNKS / 64;
    constexpr int VBYTES = NBV * 1024;
    constexpr int STAGE = KBYTES + VBYTES;
    static_assert(KCHUNKS % 64 == 0 && VCHUNKS % 64 == 0, "tiles must be whole loader blocks");
    static_assert(NBK + NBV < 64, "the loads of one tile must fit the counter of outstanding loads");
    __shared__ __attribute__((aligned(1024))) char smem[NST * STAGE];

    // no tile is shared between waves here, so consecutive workgroups (which go
    // to different XCDs) simply take consecutive (agent, KV head, split) units
    const int logical = blockIdx.x;
    if (logical >= a.total_wgs)
        return;
    int t = logical;
    const int sp = t % a.n_splits;
    t /= a.n_splits;
    const int kvh = t % a.Hkv;
    const int b = t / a.Hkv;

    const int wave = SUB == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int lane = threadIdx.x % 64;
    const int spw = sp * SUB + wave;             // index of this wave's partial results
    const int col = lane % 32, half = lane / 32;
    const int r = a.Hq / a.Hkv;
    const bool row_valid = col < r * a.Nq;
    const int hl = row_valid ? col / a.Nq : 0;
    const int i_row = row_valid ? col % a.Nq : 0;
    const int hq = kvh * r + hl;

    // the agent's header {S, L_c, ..} in one scalar load and, when they fit the wave, all bucket
    // bounds at once, one per lane: no chain of dependent trips to memory before the first tile
    const int32_t *bnd_g = a.bnd + (size_t)b * (a.Smax + 2);
    const bool bnd_in_lanes = a.Smax + 2 <= 64;
    int my_bnd = 0x7fffffff;
    if (bnd_in_lanes && lane <= a.Smax + 1)
        my_bnd = bnd_g[lane];
    const en_table_ptr hdr = as_table(a.hdr + 4 * (size_t)b);
    const int S = hdr[0];
    const en_table_ptr bnd = as_table(bnd_g);
    auto bound_at = [&](int s) {          // s is wave-uniform
        return bnd_in_lanes ? __builtin_amdgcn_readlane(my_bnd, s) : bnd[s];
    };
    const int Lc = hdr[1] + a.q_first;       // rows are new tokens q_first .. q_first+Nq-1
    const int Ltot = Lc + a.Nq;
    const int ntiles64 = (Ltot + EN_KEY_TILE - 1) / EN_KEY_TILE;
    // split boundaries are whole 64-key tiles, as everywhere else
    const int split_key_begin = (int)split_first_tile(sp, ntiles64, a.n_splits) * EN_KEY_TILE;
    const int split_key_end = min((int)split_first_tile(sp + 1, ntiles64, a.n_splits) * EN_KEY_TILE, Ltot);
    const int t_begin = split_key_begin, t_end = split_key_end;
    const int lt_begin = split_key_begin / LB;           // load tiles; splits begin on them
    const int lt_end = (split_key_end + LB - 1) / LB;    // context rows are zero up to a multiple of 64

    // ---- loader set-up ----
    const char *kg = (const char *)a.kc + ((size_t)b * a.Hkv + kvh) * (size_t)a.T * ROWB;
    const char *vg = (const char *)a.vt + ((size_t)b * a.Hkv + kvh) * (size_t)D * a.T * 2;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    // the waves take the loader blocks in turn; a wave that would run out repeats the last one
    constexpr int NKW = (NBK + SUB - 1) / SUB, NVW = (NBV + SUB - 1) / SUB;
    uint32_t koff[NKW], voff[NVW], kblk[NKW], vblk[NVW];
#pragma unroll
    for (int jj = 0; jj < NKW; ++jj) {
        const int j = min(wave + SUB * jj, NBK - 1);
        const int q = j * 64 + lane;
        const int row = q / KCPR, c = q % KCPR;
        koff[jj] = (uint32_t)(row * ROWB + (c < KCPR - 1 ? c : 0) * 16);      // the pad chunk re-reads chunk 0
        kblk[jj] = (uint32_t)j * 1024;
    }
#pragma unroll
    for (int jj = 0; jj < NVW; ++jj) {
        const int j = min(wave + SUB * jj, NBV - 1);
        const int q = j * 64 + lane;
        const int d = q / VCPR, c = q % VCPR;
        voff[jj] = (uint32_t)((size_t)d * a.T * 2 + (c < VCPR - 1 ? c : 0) * 16);
        vblk[jj] = (uint32_t)(KBYTES + j * 1024);
    }
    auto issue = [&](int tile, int stage) {
        const char *kt = kg + (size_t)tile * (LB * ROWB);
        const char *vtile = vg + (size_t)tile * (LB * 2);
        const uint32_t dst = lds0 + stage * STAGE;
#pragma unroll
        for (int jj = 0; jj < NKW; ++jj)
            dma16(kt, koff[jj], dst + kblk[jj]);
#pragma unroll
        for (int jj = 0; jj < NVW; ++jj)
            dma16(vtile, voff[jj], dst + vblk[jj]);
    };

    const int klane = col * KSTR + half * 16;
    const int vlane = KBYTES + col * VSTR + half * 16;

    // ---- the step's own keys and values join the context (decode steps): new token t sits at
    // position L_c + t, and the one wave whose key range holds that position writes it: the key
    // rotated there, the value as a column of V^T, exactly as ctx_append_kernel does. Nobody else
    // reads those lines in this launch (a 64-key tile belongs to one split, a KV head to one wave),
    // and the wave itself waits for its stores to be acknowledged before it loads a tile that
    // holds a new token. The first tile is on its way meanwhile if it holds none. ----
    const int first_new = max(Lc, split_key_begin);
    const bool owns_new = a.app_k != nullptr && first_new < split_key_end;
    const bool first_tile_old = first_new >= (lt_begin + 1) * LB;
    if (t_begin < t_end && !(owns_new && !first_tile_old))
        issue(lt_begin, 0);
    // Lane c owns the rotary pairs (c, c + D/2), c + 64, ... of a token. The first new token's
    // row is fetched here, together with the queries below; the stores follow the queries.
    constexpr int APP_J = (D / 2 + 63) / 64;
    float app_x1[APP_J], app_x2[APP_J], app_cs[APP_J], app_sn[APP_J];
    bf16_t app_v1[APP_J], app_v2[APP_J];
    auto app_load = [&](int t) {
        const int pos = Lc + t;
        const bf16_t *kr = (const bf16_t *)a.app_k + (((size_t)b * a.Nq + t) * a.Hkv + kvh) * D;
        const bf16_t *vr = (const bf16_t *)a.app_v + (((size_t)b * a.Nq + t) * a.Hkv + kvh) * D;
#pragma unroll
        for (int j = 0; j < APP_J; ++j) {
            const int c = min(lane + 64 * j, D / 2 - 1);
            app_cs[j] = a.cos_tab[(size_t)pos * (D / 2) + c];
            app_sn[j] = a.sin_tab[(size_t)pos * (D / 2) + c];
            app_x1[j] = (float)kr[c];
            app_x2[j] = (float)kr[c + D / 2];
            app_v1[j] = vr[c];
            app_v2[j] = vr[c + D / 2];
        }
    };
    auto app_store = [&](auto first_tag, int t) {
        const int pos = Lc + t;
        bf16_t *kd = (bf16_t *)a.kc + (((size_t)b * a.Hkv + kvh) * a.T + pos) * D;
        // token j in column j with bits 2 and 3 exchanged
        const int vcol = (pos & ~0xC) | ((pos & 4) << 1) | ((pos & 8) >> 1);
        bf16_t *vd = (bf16_t *)a.vt + ((size_t)b * a.Hkv + kvh) * (size_t)D * a.T + vcol;
#pragma unroll
        for (int j = 0; j < APP_J; ++j) {
            const int c = lane + 64 * j;
            if (c < D / 2) {
                float y1, y2;
                rope_key_pair<decltype(first_tag)::value>(app_x1[j], app_x2[j], app_cs[j], app_sn[j], y1, y2);
                kd[c] = (bf16_t)y1;
                kd[c + D / 2] = (bf16_t)y2;
                vd[(size_t)c * a.T] = app_v1[j];
                vd[(size_t)(c + D / 2) * a.T] = app_v2[j];
            }
        }
    };
    const bool appends = owns_new && wave == 0;          // one wave writes, all wait for it
    if (appends)
        app_load(first_new - Lc);

    // ---- Q: load, rotate at L_c + i, scale, round to bf16 ----
    bf16x8 qf[NKS];
    {
        bf16x8 qraw[NKS];
        const bf16_t *qp = (const bf16_t *)a.q + (((size_t)b * a.Nq + i_row) * a.Hq + hq) * D + 8 * half;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            qraw[ks] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
            if (row_valid)
                qraw[ks] = *reinterpret_cast<const bf16x8 *>(qp + 16 * ks);
        }
        const int pos = row_valid ? Lc + i_row : 0;
        const float *ct = a.cos_tab + (size_t)pos * (D / 2) + 8 * half;
        const float *st = a.sin_tab + (size_t)pos * (D / 2) + 8 * half;
        float cs[NKS / 2][8], sn[NKS / 2][8];
#pragma unroll
        for (int ks = 0; ks < NKS / 2; ++ks)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                cs[ks][j] = ct[16 * ks + j];
                sn[ks][j] = st[16 * ks + j];
            }
        // the new tokens' stores go out between the loads of the queries and the arithmetic on
        // them, so that their acknowledgement is under way while the queries are rotated
        if (appends) {
            int t = first_new - Lc;
            app_store(std::true_type{}, t);
            for (++t; t < a.Nq && Lc + t < split_key_end; ++t) {
                app_load(t);
                app_store(std::false_type{}, t);
            }
        }
        if (owns_new && !first_tile_old) {
            if (appends)
                wait_all_memory();                   // stores included
            if (SUB > 1)
                __syncthreads();
            issue(lt_begin, 0);
        }
        float qx[NKS][8];
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
            for (int j = 0; j < 8; ++j)
                qx[ks][j] = (float)qraw[ks][j];
#pragma unroll
        for (int ks = 0; ks < NKS / 2; ++ks) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float x1 = qx[ks][j], x2 = qx[ks + NKS / 2][j];
                qx[ks][j] = (x1 * cs[ks][j] - x2 * sn[ks][j]) * a.scale_log2e;
                qx[ks + NKS / 2][j] = (x2 * cs[ks][j] + x1 * sn[ks][j]) * a.scale_log2e;
            }
        }
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
            for (int j = 0; j < 8; ++j)
                qf[ks][j] = (bf16_t)qx[ks][j];
    }

    // ---- state (see the prefill kernel for the softmax reference scheme) ----
    f32x16 o[NDB];
#pragma unroll
    for (int d = 0; d < NDB; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            o[d][e] = 0.f;
    float m_ref = 0.f;
    bool has_ref = false;
    bool pending = row_valid && Lc + i_row >= split_key_begin;
    f32x16 negm;
#pragma unroll
    for (int e = 0; e < 16; ++e)
        negm[e] = 0.f;
    float l_part = 0.f, seg_part = 0.f;

    const int tok0 = min(split_key_begin, Ltot - 1);
    int cur = bnd_in_lanes ? (int)__popcll(__ballot(lane <= S && my_bnd <= tok0)) - 1 : find_bucket(bnd, S, tok0);
    int cur_begin = bound_at(cur);
    int cur_end = bound_at(cur + 1);
    int nxt_end = (cur + 1 <= S) ? bound_at(cur + 2) : 0x7fffffff;
    const size_t row_hq = (size_t)b * a.Hq + hq;
    float *seg_base = a.ws_seg
                          ? a.ws_seg + (((size_t)spw * a.B * a.Hq + row_hq) * (a.Smax + 1)) * a.Nq * 2
                          : nullptr;
    auto close_bucket = [&]() {
        if (cur_end > cur_begin) {
            const float tot = seg_part + xor32(seg_part);
            if (seg_base && row_valid && half == 0) {
                f32x2 v = {tot, has_ref ? m_ref : EN_NEG_INF};
                *reinterpret_cast<f32x2 *>(seg_base + ((size_t)cur * a.Nq + i_row) * 2) = v;
            }
        }
        seg_part = 0.f;
        ++cur;
        cur_begin = cur_end;
        cur_end = (cur <= S) ? nxt_end : 0x7fffffff;
        nxt_end = (cur + 1 <= S) ? bound_at(cur + 2) : 0x7fffffff;
    };

    // the stores of new tokens are acknowledged before the loop loads the tile that holds them
    // (the loads of the queries went out in the meantime)
    if (owns_new && first_tile_old) {
        if (appends)
            wait_all_memory();
        if (SUB > 1)
            __syncthreads();
    }
    constexpr int NUW = NU / SUB;                // 32-key blocks of a tile per wave
    const int u0 = wave * NUW;                   // this wave's first
    int stage = 0;                               // of tile lt
    for (int lt = lt_begin; lt < lt_end; ++lt) {
        const char *stg = smem + stage * STAGE;
        // every LDS read of the previous tile has returned (its matrix
        // instructions consumed them), so its stage may be overwritten
        __builtin_amdgcn_s_waitcnt(0xc07f);                  // lgkmcnt(0)
        if (SUB == 1) {
            constexpr int PER_TILE = NBK + NBV;
            if (lt + 1 < lt_end) {
                issue(lt + 1, stage ^ 1);
                // this tile's loads have landed when at most the next tile's are outstanding
                __builtin_amdgcn_s_waitcnt((PER_TILE & 15) | ((PER_TILE >> 4) << 14) | 0x0f70);
            } else {
                __builtin_amdgcn_s_waitcnt(0x0f70);              // vmcnt(0)
            }
        } else {
            // this wave's share of the tile has landed, and past the barrier the other's too, and
            // nobody reads the previous tile any more: the next one may overwrite it. It was a
            // whole tile's arithmetic ahead of its wait, as with one wave.
            __builtin_amdgcn_s_waitcnt(0x0f70);                  // vmcnt(0)
            __builtin_amdgcn_s_barrier();
            if (lt + 1 < lt_end)
                issue(lt + 1, stage ^ 1);
        }
        lds_data_ready();
        const int kb = lt * LB;
        const int kbw = kb + KB * u0;                // this wave's keys of the tile: [kbw, kbw + KB * NUW)
        // ---- S^T = K Q^T - m_ref, the two 32-key blocks as independent chains ----
        f32x16 sv[NUW];
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
            for (int u = 0; u < NUW; ++u) {
                const bf16x8 fr = *reinterpret_cast<const bf16x8 *>(stg + (u0 + u) * (KB * KSTR) + klane + ks * 32);
                sv[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr, qf[ks], ks == 0 ? negm : sv[u], 0, 0, 0);
            }
        // causal / padding mask; columns differ in i, so every tile that reaches
        // past L_c is checked. Element e of block u is key 32 u + 8 (e / 4) + e % 4 + 4 half, counted from kbw.
        if (kbw + KB * NUW - 1 > Lc) {
            const int rel = Lc + i_row - kbw - 4 * half;
#pragma unroll
            for (int u = 0; u < NUW; ++u)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (KB * u + 8 * (e / 4) + (e % 4) > rel)
                        sv[u][e] = EN_NEG_INF;
        }
        // ---- reference (first visible tile, or near overflow) ----
        constexpr float BIG = 1.0e18f;
        bf16x8 pf[NUW][2];
        float rs = 0.f;
        {
            float p[NUW][16];
#pragma unroll
            for (int u = 0; u < NUW; ++u)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    p[u][e] = fast_exp2(sv[u][e]);
                    rs += p[u][e];
                }
            if (__any(pending || !(rs < BIG))) {
                float mx = sv[0][0];
#pragma unroll
                for (int u = 0; u < NUW; ++u)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        mx = fmaxf(mx, sv[u][e]);
                mx = pair_max(mx);
                const float want = (pending || !(rs < BIG)) ? 1.f : 0.f;
                const bool fix = pair_max(want) > 0.f && mx > EN_NEG_INF;
                const float delta = fix ? mx : 0.f;
                const float alpha = fix ? (has_ref ? fast_exp2(-delta) : 0.f) : 1.f;
#pragma unroll
                for (int d = 0; d < NDB; ++d)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        o[d][e] *= alpha;
                l_part *= alpha;
                seg_part *= alpha;
                m_ref += delta;
                has_ref = has_ref || fix;
                pending = pending && !fix;
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    negm[e] = -m_ref;
#pragma unroll
                for (int u = 0; u < NUW; ++u)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        p[u][e] = fast_exp2(sv[u][e] - delta);
            }
            // the sums use the rounded probabilities, like the products
            rs = 0.f;
#pragma unroll
            for (int u = 0; u < NUW; ++u)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const bf16_t pb = (bf16_t)p[u][e];
                    pf[u][e / 8][e % 8] = pb;
                    rs += (float)pb;
                }
        }
        l_part += rs;
        // ---- per-bucket partial sums ----
        // (a wave that takes every other block closes the buckets that lie between its blocks
        // with what it had of them, possibly nothing: ranges below kbw select no element)
        const int ke = min(kbw + KB * NUW, split_key_end);
        if (cur_end > ke) {
            seg_part += rs;
        } else if (kbw < split_key_end) {
            int lo = kbw;
            while (true) {
                const int hi = min(cur_end, ke);
                float part = 0.f;
                const int rlo = lo - kbw - 4 * half, rhi = hi - kbw - 4 * half;
#pragma unroll
                for (int u = 0; u < NUW; ++u)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int kr = KB * u + 8 * (e / 4) + (e % 4);
                        part += (kr >= rlo && kr < rhi) ? (float)pf[u][e / 8][e % 8] : 0.f;
                    }
                seg_part += part;
                if (cur_end > ke || cur > S)
                    break;
                close_bucket();
                lo = hi;
            }
        }
        // ---- O^T += V^T P^T ----
#pragma unroll
        for (int u = 0; u < NUW; ++u)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int d = 0; d < NDB; ++d) {
                    const bf16x8 av = *reinterpret_cast<const bf16x8 *>(stg + (u0 + u) * (KB * 2) + vlane + kk * 32 + d * 32 * VSTR);
                    o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, pf[u][kk], o[d], 0, 0, 0);
                }
        stage ^= 1;
    }

    if (seg_base)
        while (cur <= S && cur_begin < split_key_end)
            close_bucket();

    const float l_tot = l_part + xor32(l_part);
    const size_t row = row_hq * a.Nq + i_row;
    if (a.ws_ml && row_valid && half == 0) {
        f32x2 v = {has_ref ? m_ref : EN_NEG_INF, l_tot};
        *reinterpret_cast<f32x2 *>(a.ws_ml + ((size_t)spw * a.B * a.Hq * a.Nq + row) * 2) = v;
    }
    if (!row_valid)
        return;
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    bf16_t *op = (a.n_splits * SUB == 1)
                     ? (bf16_t *)a.out + (((size_t)b * a.Nq + i_row) * a.Hq + hq) * D
                     : (bf16_t *)a.ws_opart + ((size_t)spw * a.B * a.Hq * a.Nq + row) * D;
#pragma unroll
    for (int d = 0; d < NDB; ++d)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[e] = (bf16_t)(o[d][4 * g + e] * inv);
            *reinterpret_cast<bf16x4 *>(op + 32 * d + 8 * g + 4 * half) = v;
        }
}

// ---------------------------------------------------------------------------
// attn_once (bf16): the same for steps of at most 16 query rows per KV head whose (agent, KV head) pairs are so few that
// the kernel above is bound by its start-up and its tiles one after the other (a step of one agent over 8 K tokens: 12.3
// us for 34 MB, of which a plain read of them takes 4: what an earlier step left in the L2s is still there). Here nothing
// comes one after the other: a workgroup is a whole split of up to five tiles, two waves a tile and 32 keys a wave, all of
// its loads out before anything is waited for, one barrier before the products with the values, one before the waves'
// results meet in LDS. The chain that is left is argument, header, load, two products, exchange, store: 5.7 us on average
// for five tiles (7.1 the slowest workgroup), 3.2 for two, of which the loads' way through the vector memory path of a
// compute unit (64 bytes a clock) is 1.5 and 0.5. Per decoded token with the merge, streaming kernel / this one, in
// parentheses over a context from HBM: 8 K tokens 15.4 / 10.3 us (18.5 / 14.1), 1.5 K 11.6 / 7.9 (13.8 / 9.6), 0.25 K, with
// one split and no merge, 12.1 / 6.5 (14.1 / 8.2). See once_fits for more, and for which steps it takes.
//
// Products are 16 x 16 x 32: the 16 columns are the r * N_q rows, half the width of the kernel above, and a score product's
// chain of dependent instructions is D / 32 long instead of D / 16. A wave takes the maximum of its own 32 keys as its rows'
// reference, so that no row ever lacks one; the references meet with the results.
// ---------------------------------------------------------------------------
// The operands of a wave's score products, when all but the last NEWER of its loads have come: of k-step ks the bytes at
// addr ^ 64 ks, and STEP further.
template <int STEP, int NEWER>
__device__ __forceinline__ void read_keys(bf16x8 (&fr)[4][2], uint32_t addr, std::integral_constant<int, STEP>, std::integral_constant<int, NEWER>)
{
    asm volatile("s_waitcnt vmcnt(%12)\n\t"
                 "ds_read_b128 %0, %8\n\tds_read_b128 %1, %8 offset:%13\n\t"
                 "ds_read_b128 %2, %9\n\tds_read_b128 %3, %9 offset:%13\n\t"
                 "ds_read_b128 %4, %10\n\tds_read_b128 %5, %10 offset:%13\n\t"
                 "ds_read_b128 %6, %11\n\tds_read_b128 %7, %11 offset:%13\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(fr[0][0]), "=&v"(fr[0][1]), "=&v"(fr[1][0]), "=&v"(fr[1][1]), "=&v"(fr[2][0]), "=&v"(fr[2][1]),
                   "=&v"(fr[3][0]), "=&v"(fr[3][1])
                 : "v"(addr), "v"(addr ^ 64), "v"(addr ^ 128), "v"(addr ^ 192), "n"(NEWER), "n"(STEP)
                 : "memory");
}
template <int STEP, int NEWER>
__device__ __forceinline__ void read_keys(bf16x8 (&fr)[2][2], uint32_t addr, std::integral_constant<int, STEP>, std::integral_constant<int, NEWER>)
{
    asm volatile("s_waitcnt vmcnt(%6)\n\t"
                 "ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:%7\n\t"
                 "ds_read_b128 %2, %5\n\tds_read_b128 %3, %5 offset:%7\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(fr[0][0]), "=&v"(fr[0][1]), "=&v"(fr[1][0]), "=&v"(fr[1][1])
                 : "v"(addr), "v"(addr ^ 64), "n"(NEWER), "n"(STEP)
                 : "memory");
}

template <int D, int TPS>
__global__ __launch_bounds__(128 * TPS) void attn_once_kernel(EnAttnArgs a)
{
    constexpr int KB = 32;                       // keys per wave
    constexpr int NKS = D / 32;                  // k-steps of a 16 x 16 score product
    constexpr int NDT = D / 16;                  // 16-row blocks of O^T
    constexpr int W = 2 * TPS;                   // waves
    constexpr int ROWB = 2 * D;                  // bytes per K row
    constexpr int KCPR = ROWB / 16;              // 16-byte chunks per K row
    constexpr int KRPB = 1024 / ROWB;            // K rows per loader block
    constexpr int KHALF = KB * ROWB;             // a wave's K rows
    constexpr int KBYTES = 2 * KHALF;
    constexpr int VROWB = EN_KEY_TILE * 2;       // bytes per V^T row of a tile
    constexpr int VBYTES = D * VROWB;
    constexpr int STAGE = KBYTES + VBYTES;
    constexpr int NBK = KHALF / 1024, NBV = VBYTES / 2048;   // loader blocks per wave
    __shared__ __attribute__((aligned(1024))) char smem[TPS * STAGE];

    // (arguments and divisions: see attn_bf16_kernel)
    asm volatile("" ::"s"(a.q), "s"(a.cos_tab), "s"(a.kc), "s"(a.bnd), "s"(a.ws_ml), "s"(a.app_k), "s"(a.app_v), "s"(a.hdr), "s"(a.B),
                 "s"(a.by_splits.mul), "s"(a.by_r.n), "s"(a.by_nq.mul), "s"(a.one_Lc), "s"(a.scale_log2e));
    const int sp = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int lane = tid % 64;
    const int col = lane % 16, g = lane / 16;
    const int r = a.by_r.n;
    const int rows = r * a.Nq;                   // at most 16
    const bool row_valid = col < rows;           // (the other columns compute on zero queries, for nobody)
    const int hl = row_valid ? divided(col, a.by_nq) : 0;
    const int i_row = row_valid ? col - hl * a.Nq : 0;
    const int hq = kvh * r + hl;

    const int32_t *bnd_g = a.bnd + (size_t)b * (a.Smax + 2);
    const bool bnd_in_lanes = a.Smax + 2 <= 64;
    int my_bnd = 0x7fffffff;
    if (a.ws_seg && bnd_in_lanes && lane <= a.Smax + 1)
        my_bnd = bnd_g[lane];
    const en_table_ptr hdr = as_table(a.hdr + 4 * (size_t)b);
    int S = a.one_S, Lc = a.one_Lc;
    if (a.B > 1) {
        S = hdr[0];
        Lc = hdr[1];
    }
    Lc += a.q_first;                             // rows are new tokens q_first .. q_first+Nq-1
    const int Ltot = Lc + a.Nq;
    const int ntiles = (Ltot + EN_KEY_TILE - 1) / EN_KEY_TILE;
    const int t_begin = divided(sp * ntiles + a.n_splits - 1, a.by_splits);        // split_first_tile
    const int t_end = divided((sp + 1) * ntiles + a.n_splits - 1, a.by_splits);
    const int key_begin = t_begin * EN_KEY_TILE, key_end = min(t_end * EN_KEY_TILE, Ltot);
    const unsigned rows_all = (unsigned)a.B * a.Hq * a.Nq;
    if (t_begin >= t_end) {                      // an agent with fewer tiles than splits
        if (a.ws_ml && tid < rows) {
            f32x2 v = {EN_NEG_INF, 0.f};
            *reinterpret_cast<f32x2 *>(a.ws_ml + ((size_t)sp * rows_all + ((size_t)b * a.Hq + kvh * r) * a.Nq + tid) * 2) = v;
        }
        return;
    }
    const int u = wave & 1;                      // half of the tile
    const int tile = t_begin + wave / 2;
    const bool active = tile < t_end;            // the same for the whole wave
    const int kb = tile * EN_KEY_TILE + u * KB;  // first key
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    char *const kst = smem + (wave / 2) * STAGE + u * KHALF;         // the wave's K rows
    char *const vst = smem + (wave / 2) * STAGE + KBYTES;            // the pair's V^T tile

    // ---- queries and their angles, asked for first ----
    bf16x8 qraw[NKS];
    f32x8 cs[NKS / 2], sn[NKS / 2];
    if (row_valid) {                             // (lanes without a row ask for nothing: their way through the vector memory path is not free)
        const bf16_t *qp = (const bf16_t *)a.q + (((size_t)b * a.Nq + i_row) * a.Hq + hq) * D + 8 * g;
        const size_t pos = Lc + i_row;
        const float *ct = a.cos_tab + pos * (D / 2) + 8 * g, *st = a.sin_tab + pos * (D / 2) + 8 * g;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
            qraw[ks] = *reinterpret_cast<const bf16x8 *>(qp + 32 * ks);
#pragma unroll
        for (int ks = 0; ks < NKS / 2; ++ks) {
            cs[ks] = *reinterpret_cast<const f32x8 *>(ct + 32 * ks);
            sn[ks] = *reinterpret_cast<const f32x8 *>(st + 32 * ks);
        }
    }
    // ---- the step's own keys and values (see attn_decode_kernel): the wave whose keys they are writes them into the
    // context and, when the tile has landed, over what this holds in their place ----
    constexpr int APP_L = D / 2;                 // lanes that own a rotary pair
    const int first_new = max(Lc, key_begin);
    const int own_first = max(first_new, kb), own_end = min(key_end, kb + KB);
    const bool owns_new = a.app_k != nullptr && active && own_first < own_end;
    float app_cs = 0.f, app_sn = 0.f;
    bf16_t app_k1 = (bf16_t)0.f, app_k2 = (bf16_t)0.f, app_v1 = (bf16_t)0.f, app_v2 = (bf16_t)0.f;
    auto app_load = [&](int t) {
        const int c = min(lane, APP_L - 1);
        const bf16_t *kr = (const bf16_t *)a.app_k + (((size_t)b * a.Nq + t) * a.Hkv + kvh) * D;
        const bf16_t *vr = (const bf16_t *)a.app_v + (((size_t)b * a.Nq + t) * a.Hkv + kvh) * D;
        app_cs = a.cos_tab[(size_t)(Lc + t) * (D / 2) + c];
        app_sn = a.sin_tab[(size_t)(Lc + t) * (D / 2) + c];
        app_k1 = kr[c];
        app_k2 = kr[c + D / 2];
        app_v1 = vr[c];
        app_v2 = vr[c + D / 2];
    };
    if (owns_new)
        app_load(own_first - Lc);

    // ---- the tile's loads: the wave's own K rows, half of the pair's V^T rows. Inside a row the 16-byte chunks are
    // exchanged (XOR) so that the operand reads of 16 consecutive lanes meet distinct banks.
    // (a wave without a tile asks for bytes past the end, which is no trip to memory: with a branch here the waits for the
    // queries would have to be waits for everything. Its vector offset alone puts them there: a scalar offset beyond the
    // buffer may be taken from the buffer's length before the comparison) ----
    {
        typedef __attribute__((address_space(3))) char *lptr;
        constexpr int RSRC = 0x00027000;
        const auto kr = __builtin_amdgcn_make_buffer_rsrc((char *)const_cast<void *>(a.kc) + ((size_t)b * a.Hkv + kvh) * a.T * ROWB, 0,
                                                          a.T * ROWB, RSRC);
        const auto vr = __builtin_amdgcn_make_buffer_rsrc((char *)const_cast<void *>(a.vt) + ((size_t)b * a.Hkv + kvh) * a.T * ROWB, 0,
                                                          a.T * ROWB, RSRC);
        const int krow = lane / KCPR;            // row inside a loader block
        const int kpat = D == 128 ? krow : (krow >> 1) & 3;
        const uint32_t past = active ? 0u : 1u << 31;
        const int kat = active ? kb * ROWB : 0, vat = active ? tile * VROWB : 0;
        const uint32_t koff = (uint32_t)(krow * ROWB + ((lane % KCPR) ^ kpat) * 16) | past;
        static_for<NBK>([&](auto j_tag) {
            constexpr int j = decltype(j_tag)::value;
            constexpr int bits = D == 128 ? (j & 1) | ((j >> 1) & 2) : j >> 1;        // bits 2, 3 of the row's pattern
            __builtin_amdgcn_raw_ptr_buffer_load_lds(kr, (lptr)(kst + j * 1024), 16, koff ^ (bits << 6), kat + j * 1024, 0, 0);
        });
        // loader block 2 j + u is the V^T rows 16 j + 8 u ..
        const uint32_t voff = (uint32_t)((8 * u + lane / 8) * a.T * 2 + ((lane % 8) ^ (4 * u + lane / 16)) * 16) | past;
#pragma unroll
        for (int j = 0; j < NBV; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, (lptr)(vst + (2 * j + u) * 1024), 16, voff,
                                                     vat + 16 * j * a.T * 2, 0, 0);
    }

    // ---- Q: rotate at L_c + i, scale, round to bf16 ----
    bf16x8 qf[NKS];
    if (row_valid) {
#pragma unroll
        for (int ks = 0; ks < NKS / 2; ++ks)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float x1 = (float)qraw[ks][j], x2 = (float)qraw[ks + NKS / 2][j];
                qf[ks][j] = (bf16_t)((x1 * cs[ks][j] - x2 * sn[ks][j]) * a.scale_log2e);
                qf[ks + NKS / 2][j] = (bf16_t)((x2 * cs[ks][j] + x1 * sn[ks][j]) * a.scale_log2e);
            }
    } else {
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
            qf[ks] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
    }
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
        asm volatile("" : "+v"(qf[ks]));         // (here, while the tile is on its way)
    // addresses of what is read behind the barrier.
    // S^T: row 4 g' + e of block 0 is key 16 (g' / 2) + 4 (g' % 2) + e, of block 1 that key + 8, so that a lane's
    // eight scores are the keys of its chunk of a V^T row (bits 2 and 3 exchanged)
    auto k_pattern = [](int row) {
        return D == 128 ? (row & 3) | ((row >> 2) & 1) << 2 | ((row >> 4) & 1) << 3 : ((row >> 1) & 3) | ((row >> 4) & 1) << 2;
    };
    const int key0 = 16 * (col >> 3) + (col & 7);
    uint32_t kaddr = (uint32_t)(kst - smem) + (uint32_t)(key0 * ROWB + (g ^ k_pattern(key0)) * 16);
    uint32_t vaddr = (uint32_t)(vst - smem) + (uint32_t)(col * VROWB + ((4 * u + g) ^ (col / 2)) * 16);
    asm volatile("" : "+v"(kaddr), "+v"(vaddr));
    const int key_g = 16 * (g >> 1) + 4 * (g & 1);               // the lane's first key

    auto app_turn = [&](int pos, float &y1, float &y2) {
        // (the rows whose products are rounded the other way: see rope_key_pair)
        if (pos == first_new)
            rope_key_pair<true>((float)app_k1, (float)app_k2, app_cs, app_sn, y1, y2);
        else
            rope_key_pair((float)app_k1, (float)app_k2, app_cs, app_sn, y1, y2);
    };
    if (owns_new) {
        __builtin_amdgcn_s_waitcnt(0x0f70 | NBV);                // vmcnt(NBV): the wave's K rows have landed
        for (int pos = own_first; pos < own_end; ++pos) {
            if (pos > own_first)
                app_load(pos - Lc);
            float y1, y2;
            app_turn(pos, y1, y2);
            if (lane < APP_L) {
                char *kd = kst + (pos - kb) * ROWB + lane % 8 * 2;
                const int pat = k_pattern(pos - kb);
                *reinterpret_cast<bf16_t *>(kd + ((lane / 8) ^ pat) * 16) = (bf16_t)y1;
                *reinterpret_cast<bf16_t *>(kd + ((lane / 8 + D / 16) ^ pat) * 16) = (bf16_t)y2;
            }
        }
    }
    // ---- scores and probabilities, while the V^T tile is on its way. (The K operands are read in one piece of assembly:
    // the compiler would wait for everything in flight to LDS before any of its own reads.) ----
    float m = EN_NEG_INF, l = 0.f;
    bf16x8 pf;
    f32x4 pr[2];
    if (active) {
        f32x4 sv[2];
        bf16x8 fr[NKS][2];
        read_keys(fr, lds0 + kaddr, std::integral_constant<int, 8 * ROWB>{}, std::integral_constant<int, NBV>{});
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                sv[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[ks][h], qf[ks], ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sv[h], 0, 0, 0);
        if (kb + KB - 1 > Lc) {
            const int rel = Lc + i_row - kb - key_g;             // last visible key, counted from it
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (8 * h + e > rel)
                        sv[h][e] = EN_NEG_INF;
        }
        auto over_groups = [&](float v, auto op) {               // over the four lanes of a column
            typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
            u32x2 x = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
            v = op(__uint_as_float(x[0]), __uint_as_float(x[1]));
            x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
            return op(__uint_as_float(x[0]), __uint_as_float(x[1]));
        };
        m = sv[0][0];
#pragma unroll
        for (int e = 1; e < 8; ++e)
            m = fmaxf(m, sv[e / 4][e % 4]);
        m = over_groups(m, [](float x, float y) { return fmaxf(x, y); });
        const float ref = m == EN_NEG_INF ? 0.f : m;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            pf[e] = (bf16_t)fast_exp2(sv[e / 4][e % 4] - ref);
            pr[e / 4][e % 4] = (float)pf[e];                     // (the sums use what the products use)
            l += pr[e / 4][e % 4];
        }
        l = over_groups(l, [](float x, float y) { return x + y; });
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0)
    __builtin_amdgcn_s_barrier();
    lds_data_ready();
    if (owns_new)                                // (the partner's loads of these rows have landed, too)
        for (int pos = own_first; pos < own_end; ++pos) {
            if (own_end - own_first > 1)
                app_load(pos - Lc);
            float y1, y2;
            app_turn(pos, y1, y2);
            const int vcol = (pos & ~0xC) | ((pos & 4) << 1) | ((pos & 8) >> 1);      // bits 2 and 3 exchanged
            if (lane < APP_L) {
                auto vput = [&](int d, bf16_t v) {
                    *reinterpret_cast<bf16_t *>(vst + d * VROWB + (((vcol % EN_KEY_TILE) / 8) ^ ((d / 2) & 7)) * 16 + (vcol % 8) * 2) = v;
                };
                vput(lane, app_v1);
                vput(lane + D / 2, app_v2);
                bf16_t *kd = (bf16_t *)a.kc + (((size_t)b * a.Hkv + kvh) * a.T + pos) * D;
                bf16_t *vd = (bf16_t *)a.vt + ((size_t)b * a.Hkv + kvh) * (size_t)D * a.T + vcol;
                kd[lane] = (bf16_t)y1;
                kd[lane + D / 2] = (bf16_t)y2;
                vd[(size_t)lane * a.T] = app_v1;
                vd[(size_t)(lane + D / 2) * a.T] = app_v2;
            }
        }

    // P of the wave's block, [col][32 keys] floats, and (reference, sum) per column: over the wave's own columns of
    // the V^T tile, when its products have read them
    auto p_at = [&](int w, int c, int key) {
        const int row = 2 * c + key / 16;
        return smem + (w / 2) * STAGE + KBYTES + row * VROWB + ((4 * (w & 1) + (key % 16) / 4) ^ (c & 7)) * 16 + key % 4 * 4;
    };
    auto ml_at = [&](int w, int c) {
        return smem + (w / 2) * STAGE + KBYTES + (32 + c / 8) * VROWB + (w & 1) * 64 + c % 8 * 8;
    };
    // O of the wave's block, [col][D] floats, the chunks of a row rotated by the column: over its K rows
    auto o_at = [&](int w, int c, int chunk) {
        return smem + (w / 2) * STAGE + (w & 1) * KHALF + c * (4 * D) + ((chunk + c) & (D / 4 - 1)) * 16;
    };
    if (active) {
        // ---- O^T = V^T P^T ----
        f32x4 o[NDT];
#pragma unroll
        for (int d = 0; d < NDT; ++d) {
            const bf16x8 fr = *reinterpret_cast<const bf16x8 *>(smem + vaddr + d * 16 * VROWB);
            o[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr, pf, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        }
        if (row_valid) {
#pragma unroll
            for (int d = 0; d < NDT; ++d)
                *reinterpret_cast<f32x4 *>(o_at(wave, col, 4 * d + g)) = o[d];
#pragma unroll
            for (int h = 0; h < 2; ++h)
                *reinterpret_cast<f32x4 *>(p_at(wave, col, key_g + 8 * h)) = pr[h];
            if (g == 0) {
                f32x2 v = {m, l};
                *reinterpret_cast<f32x2 *>(ml_at(wave, col)) = v;
            }
        }
    } else if (lane < 16) {
        f32x2 v = {EN_NEG_INF, 0.f};
        *reinterpret_cast<f32x2 *>(ml_at(wave, lane)) = v;
    }
    // (LDS only: nobody waits for the stores of new tokens)
    __builtin_amdgcn_s_waitcnt(0xc07f);          // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    lds_data_ready();

    // the weights of the waves' results for row c; `none`: the wave has no key that the row sees (its sum is 0, with any key
    // it is 1 at least or NaN). By the bits: without NaN compares a row of NaN could pass for one without keys.
    auto weights = [&](int c, float (&wt)[W], bool (&none)[W], float &M, float &L) {
        f32x2 ml[W];
        M = EN_NEG_INF;
        L = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w)
            ml[w] = *reinterpret_cast<const f32x2 *>(ml_at(w, c));
#pragma unroll
        for (int w = 0; w < W; ++w)
            M = fmaxf(M, ml[w][0]);
#pragma unroll
        for (int w = 0; w < W; ++w) {
            none[w] = __float_as_uint(ml[w][1]) == 0u;
            wt[w] = none[w] ? 0.f : fast_exp2(ml[w][0] - M);
            L += wt[w] * ml[w][1];
        }
    };
    // ---- the waves' results meet: a thread takes four values of a row ----
    for (int it = tid; it < rows * (D / 4); it += 64 * W) {
        const int c = it / (D / 4), ch = it % (D / 4);
        float wt[W], M, L;
        bool none[W];
        f32x4 x[W];
#pragma unroll
        for (int w = 0; w < W; ++w)
            x[w] = *reinterpret_cast<const f32x4 *>(o_at(w, c, ch));
        weights(c, wt, none, M, L);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < W; ++w)
            acc += none[w] ? f32x4{0.f, 0.f, 0.f, 0.f} : x[w] * wt[w];      // (a wave without a tile left nothing)
        const float inv = L > 0.f ? 1.f / L : 0.f;
        const int ho = divided(c, a.by_nq), h = kvh * r + ho, i = c - ho * a.Nq;
        const size_t row = ((size_t)b * a.Hq + h) * a.Nq + i;
        bf16_t *op = (a.n_splits == 1) ? (bf16_t *)a.out + (((size_t)b * a.Nq + i) * a.Hq + h) * D
                                       : (bf16_t *)a.ws_opart + ((size_t)sp * rows_all + row) * D;
        *reinterpret_cast<bf16x4 *>(op + 4 * ch) = __builtin_convertvector(acc * inv, bf16x4);
        if (a.ws_ml && ch == 0) {
            f32x2 v = {M, L};
            *reinterpret_cast<f32x2 *>(a.ws_ml + ((size_t)sp * rows_all + row) * 2) = v;
        }
    }
    // ---- the buckets' sums: 16 lanes take a (bucket, row), from the last wave on (the first have rows to merge) ----
    if (!a.ws_seg)
        return;
    auto bucket_of = [&](int tok) {
        return bnd_in_lanes ? (int)__popcll(__ballot(lane <= S && my_bnd <= tok)) - 1 : find_bucket(as_table(bnd_g), S, tok);
    };
    const int s_first = bucket_of(key_begin), n_pairs = (bucket_of(key_end - 1) - s_first + 1) * rows;
    for (int p0 = 4 * (W - 1 - wave); p0 < n_pairs; p0 += 4 * W) {
        const int p = min(p0 + g, n_pairs - 1);
        const int sb = small_quotient(p, rows), c = p - sb * rows;
        const int s = s_first + sb;
        float x[2 * W];                          // this lane's keys col, col + 16, ..
#pragma unroll
        for (int k = 0; k < 2 * W; ++k)
            x[k] = *reinterpret_cast<const float *>(p_at(k / 2, c, col + 16 * (k & 1)));
        int blo, bhi;
        if (bnd_in_lanes) {
            blo = __shfl(my_bnd, s, 64);
            bhi = __shfl(my_bnd, s + 1, 64);
        } else {
            blo = bnd_g[s];
            bhi = bnd_g[s + 1];
        }
        const int lo = max(blo, key_begin) - key_begin, hi = min(bhi, key_end) - key_begin;
        float wt[W], M, L;
        bool none[W];
        weights(c, wt, none, M, L);
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const int k0 = w * KB + col, k1 = k0 + 16;
            sum += ((k0 >= lo && k0 < hi ? x[2 * w] : 0.f) + (k1 >= lo && k1 < hi ? x[2 * w + 1] : 0.f)) * wt[w];
        }
        sum = lanes_reduce<16>(sum, [](float x, float y) { return x + y; });
        if (col == 0 && p0 + g < n_pairs && bhi > blo) {
            const int ho = divided(c, a.by_nq), h = kvh * r + ho, i = c - ho * a.Nq;
            f32x2 v = {sum, M};
            *reinterpret_cast<f32x2 *>(a.ws_seg + ((((size_t)sp * a.B * a.Hq + (size_t)b * a.Hq + h) * (a.Smax + 1) + s) * a.Nq + i) * 2) = v;
        }
    }
}

// ---------------------------------------------------------------------------
// attn_f32: attention in single precision on the fp32 matrix instruction (16 x 16 x 4, exact products,
// fp32 sums), for small layers and short steps, which are bound by latency: the chain of a wave's trips
// to memory and of its dependent products, not by bytes or operations.
//
// A workgroup takes 16 of the r * N_q query rows of a KV head and one KV split, and its eight waves (two where
// short splits fill the chip: see EnAttnArgs::f32_waves) share the split's keys: each a contiguous run of
// 16-key blocks, with a softmax state of its own; they merge through LDS, so a step of few keys needs no
// launch behind this one. (One wave per row, the lanes 64 keys apart with a row of K and of V each, took
// 34 us for 4 heads x 64 rows over 192 keys.)
//
// S^T = K Q^T: lane l holds key l % 16, dimensions 4 (l / 16) .. + 3 of every 16: one 16-byte load each, and
// its four numbers are the operands of four instructions (K and Q agree on which dimension is which k). The
// result, keys 4 (l / 16) + e of query l % 16, is the B operand of O^T += V^T P^T as it is: instruction e
// takes the keys 4 k + e. Row l % 16 of V^T block d is dimension (l % 16) * D / 16 + d, so that a lane's
// values of a key are contiguous. No operand goes through LDS.
//
// Probabilities below 2^-126 of the row's largest count as 0 (fast_exp2).
// ---------------------------------------------------------------------------
constexpr int F32_ROWS = EN_F32_ROWS;
constexpr int F32_KEYS = 16;

template <int D, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void attn_f32_kernel(EnAttnArgs a)
{
    constexpr int NJ = D / 16;                   // 16-byte loads per key row and lane; blocks of O^T
    constexpr int NV = D / 64;                   // 16-byte loads per value row and lane
    constexpr int OSTR = D + 4;                  // floats per merged row in LDS
    __shared__ __attribute__((aligned(16))) float so[WAVES][F32_ROWS][OSTR];
    __shared__ f32x2 sml[WAVES][F32_ROWS];           // (reference, sum) of a wave's rows
    __shared__ f32x2 sfirst[WAVES][F32_ROWS];        // (sum, reference) of the bucket that a wave entered midway
    __shared__ int sspan[WAVES];                     // 1: ... and that it did not leave

    // (arguments and divisions: see attn_bf16_kernel)
    asm volatile("" ::"s"(a.q), "s"(a.cos_tab), "s"(a.bnd), "s"(a.ws_ml), "s"(a.B), "s"(a.Smax), "s"(a.by_ptiles.mul),
                 "s"(a.by_nq.mul), "s"(a.one_Lc), "s"(a.red_zero));
    if (blockIdx.x == 0 && a.red_zero)
        for (int i = threadIdx.x; i < a.n_red_zero; i += 64 * WAVES)
            a.red_zero[i] = 0ull;
    const unsigned t = divided(blockIdx.x, a.by_ptiles);
    const int rg = blockIdx.x - t * a.n_ptiles;
    const unsigned t2 = divided(t, a.by_splits);
    const int sp = t - t2 * a.n_splits;
    const int b = divided(t2, a.by_hkv);
    const int kvh = t2 - b * a.Hkv;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int lane = tid % 64;
    const int col = lane % 16, grp = lane / 16;
    const int r = a.by_r.n;

    // all bucket bounds at once, one per lane, when they fit: a search through the table is a trip to memory per step
    const int32_t *bnd_g = a.bnd + (size_t)b * (a.Smax + 2);
    const bool bnd_in_lanes = a.Smax + 2 <= 64;
    const int my_bnd = bnd_g[min(lane, a.Smax + 1)];
    const en_table_ptr hdr = as_table(a.hdr + 4 * (size_t)b);
    const en_table_ptr bnd = as_table(bnd_g);
    auto bound_at = [&](int s) {             // s is wave-uniform
        return bnd_in_lanes ? __builtin_amdgcn_readlane(my_bnd, s) : bnd[s];
    };
    int S = a.one_S, Lc = a.one_Lc;
    if (a.B > 1) {
        S = hdr[0];
        Lc = hdr[1];
    }
    Lc += a.q_first;                         // rows are new tokens q_first .. q_first+Nq-1
    const int Ltot = Lc + a.Nq;
    const int ntiles = (Ltot + EN_KEY_TILE - 1) / EN_KEY_TILE;
    const int kbeg = (int)divided(sp * ntiles + a.n_splits - 1, a.by_splits) * EN_KEY_TILE;           // split_first_tile
    const int kend = min((int)divided((sp + 1) * ntiles + a.n_splits - 1, a.by_splits) * EN_KEY_TILE, Ltot);

    // the workgroup's rows, head by head: row rr is new token rr % Nq of head rr / Nq
    const int n_rows = r * a.Nq;
    const int r0 = rg * F32_ROWS, r1 = min(r0 + F32_ROWS, n_rows) - 1;
    const int h1 = divided(r1, a.by_nq);
    const int i_hi = (int)divided(r0, a.by_nq) == h1 ? r1 - h1 * a.Nq : a.Nq - 1;
    const bool row_valid = r0 + col <= r1;
    const int rr = min(r0 + col, r1);
    const int hr = divided(rr, a.by_nq);
    const int hq = kvh * r + hr, i_row = rr - hr * a.Nq;
    const int kvis = min(kend, Lc + i_hi + 1);           // keys that any of the rows may see
    const int n_blk = kvis > kbeg ? (kvis - kbeg + F32_KEYS - 1) / F32_KEYS : 0;
    const int per = (n_blk + WAVES - 1) / WAVES;
    const int n_used = per > 0 ? __builtin_amdgcn_readfirstlane(small_quotient(n_blk + per - 1, per)) : 0;      // waves with keys
    const int wb = kbeg + min(wave * per, n_blk) * F32_KEYS;           // this wave's keys
    const int we = min(kbeg + min((wave + 1) * per, n_blk) * F32_KEYS, kvis);

    const float *K = (const float *)a.kc + ((size_t)b * a.Hkv + kvh) * (size_t)a.T * D;
    const float *V = (const float *)a.vt + ((size_t)b * a.Hkv + kvh) * (size_t)a.T * D;
    // (context rows are zero up to a multiple of 64 keys: whole blocks can be read)
    f32x4 kf[NJ], vf[4][NV];
    auto load_block = [&](int kb) {
        const float *kr = K + (size_t)(kb + col) * D + 4 * grp;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            kf[j] = *reinterpret_cast<const f32x4 *>(kr + 16 * j);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float *vr = V + (size_t)(kb + 4 * grp + e) * D + col * NJ;
#pragma unroll
            for (int v = 0; v < NV; ++v)
                vf[e][v] = *reinterpret_cast<const f32x4 *>(vr + 4 * v);
        }
    };
    if (wb < we)
        load_block(wb);

    // ---- the query, rotated at L_c + i and scaled ----
    f32x4 qf[NJ];
    {
        const float *qp = (const float *)a.q + (((size_t)b * a.Nq + i_row) * a.Hq + hq) * D + 4 * grp;
        const size_t trow = (size_t)(Lc + i_row) * (D / 2) + 4 * grp;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            qf[j] = *reinterpret_cast<const f32x4 *>(qp + 16 * j);
#pragma unroll
        for (int j = 0; j < NJ / 2; ++j) {
            const f32x4 cs = *reinterpret_cast<const f32x4 *>(a.cos_tab + trow + 16 * j);
            const f32x4 sn = *reinterpret_cast<const f32x4 *>(a.sin_tab + trow + 16 * j);
            const f32x4 x1 = qf[j], x2 = qf[j + NJ / 2];
            qf[j] = (x1 * cs - x2 * sn) * a.scale_log2e;
            qf[j + NJ / 2] = (x2 * cs + x1 * sn) * a.scale_log2e;
        }
    }

    f32x4 o[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
        o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = EN_NEG_INF, l = 0.f, seg = 0.f;            // l, seg: this lane's share
    auto row_sum = [](float v) {                         // over the four lanes of a row
        v += __shfl_xor(v, 16, 64);
        return v + xor32(v);
    };
    float *seg_row = a.ws_seg ? a.ws_seg + ((((size_t)sp * a.B + b) * a.Hq + hq) * (a.Smax + 1)) * a.Nq * 2
                              : nullptr;
    auto write_bucket = [&](int s, float tot, float ref) {
        if (seg_row && row_valid && grp == 0) {
            f32x2 v = {tot, ref};
            *reinterpret_cast<f32x2 *>(seg_row + ((size_t)s * a.Nq + i_row) * 2) = v;
        }
    };
    // The bucket the wave is in. One that an earlier wave began is handed over through sfirst, one that a
    // later wave goes on with stays open; the others are complete here.
    int cur = wb >= we ? 0 : bnd_in_lanes ? (int)__popcll(__ballot(lane <= S && my_bnd <= wb)) - 1 : find_bucket(bnd, S, wb);
    int cur_end = wb < we ? bound_at(cur + 1) : 0;
    const bool entered = wb < we && wb > kbeg && bound_at(cur) < wb;
    bool first = entered, open = false;
    auto leave_bucket = [&]() {
        const float tot = row_sum(seg);
        if (first)
            sfirst[wave][col] = f32x2{tot, m};
        else
            write_bucket(cur, tot, m);
        first = false;
        seg = 0.f;
    };

    for (int kb = wb; kb < we; kb += F32_KEYS) {
        // ---- scores; eight chains of products, whose sums meet in a tree: long chains round more often (error
        // against 64 bits, 64-dimensional heads: 2.1e-7 with two chains, 1.7e-7 with eight) ----
        f32x4 s[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            s[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int i = (e * NJ + j) % 8;
                s[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][e], qf[j][e], s[i], 0, 0, 0);
            }
        f32x4 vc[4][NV];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int v = 0; v < NV; ++v)
                vc[e][v] = vf[e][v];
        if (kb + F32_KEYS < we)
            load_block(kb + F32_KEYS);
        f32x4 p = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
        // causal mask; keys of a later wave or split do not occur: ranges are whole blocks up to kvis
        const int rel = min(Lc + i_row, we - 1) - kb - 4 * grp;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e > rel)
                p[e] = EN_NEG_INF;
        float mn = fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3]));
        mn = fmaxf(mn, __shfl_xor(mn, 16, 64));
        mn = fmaxf(m, pair_max(mn));
        const float ref = mn == EN_NEG_INF ? 0.f : mn;   // nothing seen yet: all exponentials are 0
        const float alpha = fast_exp2(m - ref);
        m = mn;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            p[e] = fast_exp2(p[e] - ref);
        l = l * alpha + ((p[0] + p[1]) + (p[2] + p[3]));
        // ---- per-bucket sums ----
        seg *= alpha;
        const int ke = min(kb + F32_KEYS, we);
        if (cur_end > ke) {
            seg += (p[0] + p[1]) + (p[2] + p[3]);
        } else {
            int lo = kb;
            while (true) {
                const int hi = min(cur_end, ke);
                const int rlo = lo - kb - 4 * grp, rhi = hi - kb - 4 * grp;
                f32x4 in;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    in[e] = (e >= rlo && e < rhi) ? p[e] : 0.f;
                seg += (in[0] + in[1]) + (in[2] + in[3]);
                if (cur_end > ke || cur > S)
                    break;
                if (cur_end > bound_at(cur)) // (an empty bucket has no entry)
                    leave_bucket();
                ++cur;
                cur_end = cur <= S ? bound_at(cur + 1) : 0x7fffffff;
                lo = hi;
            }
        }
        // ---- O^T += V^T P^T ----
        // (the block's products by themselves: one rounding per block of a sum that grows, not one per key)
        f32x4 ob[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            ob[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        // A product sums over the block's keys, the hidden ones with probability 0. That is no contribution
        // unless such a key's value is infinite or NaN, which a row that does not see the key must not take:
        // then the keys go one by one, and a row keeps its sums where it does not see the key.
        bool by_key = false;
        if (kb + F32_KEYS - 1 > min(Lc, we - 1)) {           // some key may be hidden from some row
            uint32_t top = 0;                                // (by the bits: this library is built without NaN compares)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    top = max(top, __float_as_uint(vc[e][j / 4][j % 4]) & 0x7f800000u);
            by_key = __any(top == 0x7f800000u);
        }
        if (!by_key) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    ob[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vc[e][j / 4][j % 4], p[e], ob[j], 0, 0, 0);
        } else {
            const int last = min(Lc + i_row, we - 1) - kb;   // the row's last visible key of the block
#pragma unroll 1
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        const f32x4 with = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            grp == g ? vc[e][j / 4][j % 4] : 0.f, grp == g ? p[e] : 0.f, ob[j], 0, 0, 0);
                        ob[j] = 4 * g + e <= last ? with : ob[j];
                    }
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            o[j] = o[j] * alpha + ob[j];
    }

    // ---- the waves meet ----
    float open_sum = 0.f;
    if (wb < we) {
        open = cur <= S && cur_end > we && bound_at(cur) < we && we < kvis;
        if (open) {
            open_sum = row_sum(seg);
            if (first && grp == 0)
                sfirst[wave][col] = f32x2{open_sum, m};
        } else if (cur <= S && bound_at(cur) < we && cur_end > we) {
            leave_bucket();                  // the split, or what the rows may see, ends in it
        }
        const float lt = row_sum(l);
        if (grp == 0)
            sml[wave][col] = f32x2{m, lt};
        if (lane == 0)
            sspan[wave] = open && first;
    } else if (n_used == 0 && wave == 0) {
        write_bucket(S, 0.f, EN_NEG_INF);    // a split beyond the rows' causal limit: only new tokens
    }
    __syncthreads();
    float M = EN_NEG_INF;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {        // (all read at once; what waves without keys left is not used)
        const float x = sml[w][col][0];
        M = w < n_used ? fmaxf(M, x) : M;
    }
    if (wb < we) {
        const float keep = m == EN_NEG_INF ? 0.f : fast_exp2(m - M);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                f32x4 x;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    x[j] = o[4 * v + j][e] * keep;
                *reinterpret_cast<f32x4 *>(&so[wave][col][(4 * grp + e) * NJ + 4 * v]) = x;
            }
        if (open && !first) {
            // the bucket began here and goes on in the next waves: their shares join, as far as it reaches
            float tot = open_sum, ref = m;
            for (int w = wave + 1; w < n_used; ++w) {
                const f32x2 x = sfirst[w][col];
                const float both = fmaxf(ref, x[1]);
                const float to = both == EN_NEG_INF ? 0.f : both;
                tot = tot * fast_exp2(ref - to) + x[0] * fast_exp2(x[1] - to);
                ref = both;
                if (!sspan[w])
                    break;
            }
            write_bucket(cur, tot, ref);
        }
    }
    __syncthreads();
    // ---- the output, a 16-byte piece per thread at a time ----
    constexpr int CPR = D / 4;
    const size_t rows = (size_t)a.B * a.Hq * a.Nq;
#pragma unroll
    for (int k = 0; k < (F32_ROWS * CPR + 64 * WAVES - 1) / (64 * WAVES); ++k) {
        const int row = (k * 64 * WAVES + tid) / CPR, c4 = tid % CPR * 4;
        if (row >= F32_ROWS || r0 + row > r1)
            return;
        float Mr = EN_NEG_INF, L = 0.f;
        f32x2 ml[WAVES];
        f32x4 part[WAVES];
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            ml[w] = sml[w][row];
            part[w] = *reinterpret_cast<const f32x4 *>(&so[w][row][c4]);
        }
#pragma unroll
        for (int w = 0; w < WAVES; ++w)
            Mr = w < n_used ? fmaxf(Mr, ml[w][0]) : Mr;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < WAVES; ++w)
            if (w < n_used) {
                L += ml[w][0] == EN_NEG_INF ? 0.f : ml[w][1] * fast_exp2(ml[w][0] - Mr);
                acc += part[w];
            }
        const int ho = divided(r0 + row, a.by_nq);
        const int h = kvh * r + ho, i = r0 + row - ho * a.Nq;
        const size_t out_row = ((size_t)b * a.Hq + h) * a.Nq + i;
        const float inv = L > 0.f ? 1.f / L : 0.f;
        if (a.ws_ml && c4 == 0) {
            f32x2 v = {Mr, L};
            *reinterpret_cast<f32x2 *>(a.ws_ml + ((size_t)sp * rows + out_row) * 2) = v;
        }
        float *op = (a.n_splits == 1) ? (float *)a.out + (((size_t)b * a.Nq + i) * a.Hq + h) * D
                                      : (float *)a.ws_opart + ((size_t)sp * rows + out_row) * D;
        *reinterpret_cast<f32x4 *>(op + c4) = acc * inv;
    }
}

template <int WAVES>
static void launch_f32_waves(int D, const EnAttnArgs &a, hipStream_t st)
{
    const dim3 grid(a.total_wgs), blk(64 * WAVES);
    if (D == 64)
        hipLaunchKernelGGL((attn_f32_kernel<64, WAVES>), grid, blk, 0, st, a);
    else
        hipLaunchKernelGGL((attn_f32_kernel<128, WAVES>), grid, blk, 0, st, a);
}

template <int D>
static void launch_once(const EnAttnArgs &a, hipStream_t st)
{
    const dim3 grid(a.n_splits, a.Hkv, a.B), blk(128 * a.once_tiles);
    switch (a.once_tiles) {
    case 1: hipLaunchKernelGGL((attn_once_kernel<D, 1>), grid, blk, 0, st, a); break;
    case 2: hipLaunchKernelGGL((attn_once_kernel<D, 2>), grid, blk, 0, st, a); break;
    case 3: hipLaunchKernelGGL((attn_once_kernel<D, 3>), grid, blk, 0, st, a); break;
    case 4: hipLaunchKernelGGL((attn_once_kernel<D, 4>), grid, blk, 0, st, a); break;
    default: hipLaunchKernelGGL((attn_once_kernel<D, 5>), grid, blk, 0, st, a); break;
    }
}

// ---------------------------------------------------------------------------
// launcher: fp32 pools, steps that fit the decode kernel, everything else
// ---------------------------------------------------------------------------
int en_launch_attention(const en_pool *pool, const EnAttnArgs &a, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    const int D = pool->d.head_dim;
    if (pool->d.dtype == EN_F32) {
        if (a.f32_waves == 8)
            launch_f32_waves<8>(D, a, st);
        else if (a.f32_waves == 2)
            launch_f32_waves<2>(D, a, st);
        else
            return (int)hipErrorInvalidValue;
    } else if (a.decode && a.once_tiles) {
        if (D == 64)
            launch_once<64>(a, st);
        else
            launch_once<128>(a, st);
    } else if (a.decode) {
        const dim3 grid((a.total_wgs + 7) / 8 * 8), blk(64 * a.sub);
        if (a.sub != 1 && a.sub != 2)
            return (int)hipErrorInvalidValue;
        if (D == 64) {
            if (a.sub == 1)
                hipLaunchKernelGGL((attn_decode_kernel<64, 1>), grid, blk, 0, st, a);
            else
                hipLaunchKernelGGL((attn_decode_kernel<64, 2>), grid, blk, 0, st, a);
        } else {
            if (a.sub == 1)
                hipLaunchKernelGGL((attn_decode_kernel<128, 1>), grid, blk, 0, st, a);
            else
                hipLaunchKernelGGL((attn_decode_kernel<128, 2>), grid, blk, 0, st, a);
        }
    } else {
        return en_launch_attention_prefill(pool, a, stream);
    }
    return (int)hipGetLastError();
}
