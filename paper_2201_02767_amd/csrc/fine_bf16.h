// The gathered fine attention for bf16 maps (steps 3-5 at the finer levels; Sec. 3.2, Fig. 1; QuadTree-A
// scores Eq. 4, QuadTree-B softmax Eq. 6; the finest level's combination, Eqs. 2 and 5), included by
// fine.hip. fine_item.h holds the fp32 form.
//
// Work item = one parent query at level l+1 and one head (ROW: two neighbouring parents of a one-row
// map); one wave owns it. Candidate slot s = 4r + c is child c of kept key r (ROW: s = 2(half*K + r) + c).
// The slots are taken in NT tiles of 16, NT = 1, 2, 4, 8 or 16 (a power of two that covers 4K; slots past
// 4K read slot 0's row and weigh nothing).
//   1. lane 4n + t works out the address of slot 16t + n (and of the slots 64 on) once and hands it to its
//      quad, which gathers that slot's row: the key rows into registers, the value rows straight into the
//      wave's LDS (bf16_tiles.h);
//   2. logits on the 16x16x32 MFMA, the key chunks passed through LDS into operand lanes; operand rows
//      4g .. 4g+3 are query g, so lane
//      16g + n holds query g's logits of slots 16t + n for every t;
//   3. weights: B a softmax over the row's 16 lanes and the lane's tiles (unnormalised, so that the largest
//      weight, 1, is exact in bf16; the message is scaled by 1/sum), A over each lane quad (the children of
//      one kept key) times the parent's score. They go to LDS as bf16 [query][n][t]: the lane's NT weights
//      are contiguous;
//   4. levels above 0: the ranking keys move to one slot per lane and each query keeps its K best;
//   5. messages m = P V on the same MFMA: the slots are contracted in the order of the stored weights, and
//      the value operand is read from LDS transposed (ds_read_b64_tr_b16). Operand rows 4g .. 4g+3 are query
//      g's weights, so lane 16g + n ends with query g's message at channels n, 16 + n, ...;
//   6. level 0 adds the ancestors' messages times their weights, a product on the fp32 MFMA, and stores.
//
// What bounds it, and what was measured (the finest level, before -> now): the L1's line rate in the gathers,
// then the fixed work per wave. The previous form gathered with a lane per row (lane 16g + n: chunk g of row
// n). Cycles of a CU an instruction of 16 64-byte rows, a lane per row against four neighbouring lanes on one: from
// the L1 46 and 19; from the L2, whose lines are 128 bytes, one row a line 64 and 38 to 39, runs of four rows side by
// side 34 and 21; past the L2, one row a line, 155 to 165 either way, such runs 78. It also moved the
// values through 2-byte LDS writes, worked out every slot's address in four lanes, loaded w and the ancestors
// lane by lane (64 * 4 scattered words for w alone, 16 of its 77 us) and stored 2 bytes a lane. VALU
// instructions a wave 400 -> 171, LDS 52 -> 19. One launch among others like it: 200x336 maps, 2 heads x 32,
// K = 16, batch 2: 77.0 -> 50.7 us; 120x160, 8 x 32, K = 8, batch 2: 53.0 -> 42.3; 200x334, 1 x 32, K = 32, batch 2:
// 45.1 -> 30.8; 32 maps of 56x56, 1 x 64, K = 8: 29.8 -> 16.0. In a whole layer they take 1 to 4 us more.
#ifndef QTA_FINE_BF16_H
#define QTA_FINE_BF16_H

#include "bf16_tiles.h"
#include "qta_internal.h"

namespace qta {
namespace fine16 {

using namespace tiles;

// One wave's region: the value tiles, then 1 KB through which the key chunks pass one instruction's worth at
// a time, and the weights after them.
template <int D, int NT>
constexpr int wave_bytes() { return NT * tile_bytes<D>() + (NT > 8 ? 128 * NT : 1024); }

// LIVE: the tiles that can hold a slot; those after them are not gathered (zeros in LDS, masked logits).
template <int D, int NT, int LIVE, bool VA, bool FINEST, bool ROW>
__device__ __forceinline__ void item(const FineArgs& a, const int it, unsigned char* const base)
{
    constexpr int RB = D * 2;                        // bytes of one head's row
    constexpr int NJ = RB / 64;                      // 16-byte chunks per lane and row
    constexpr int SPL = NT > 4 ? NT / 4 : 1;         // candidate slots per lane: lane + 64u
    constexpr int CT = D / 16;                       // 16-channel tiles of the message
    constexpr int TS = tile_bytes<D>();

    const int lane = threadIdx.x & 63, n16 = lane & 15, g = lane >> 4;
    lds_byte* const vlds = (lds_byte*)base;          // [tile][D / 32][16 slots][4] 16-byte chunks
    lds_byte* const plds = vlds + NT * TS;           // [query][n][t] bf16
    lds_byte* const slds = plds;                     // before the weights: the key chunks in passing

    // ---- the item's coordinates (scalar) ----
    const int Np = a.Hp * a.Wp;
    const int bp = fast_div(it, a.div_heads);
    const int h = it - bp * a.heads;
    const int NI = ROW ? (Np + 1) / 2 : Np;          // items per (batch, head)
    const int b = fast_div(bp, a.div_items);
    const int P = ROW ? 2 * (bp - b * NI) : bp - b * NI;
    const int Py = ROW ? 0 : fast_div(P, a.div_Wp), Px = ROW ? P : P - Py * a.Wp;
    const bool pair2 = ROW && P + 1 < Np;
    const int H = a.H, W = a.W, C = a.C, K = a.Kp, Ks = a.Ks;
    const int N = H * W;
    const uint32_t tok_bytes = static_cast<uint32_t>(C * 2);
    auto query_yx = [&](int r, int& qy, int& qx) {
        if constexpr (ROW) {
            qy = 0;
            qx = 2 * P + r;
        } else {
            qy = 2 * Py + (r >> 1);
            qx = 2 * Px + (r & 1);
        }
    };

    // ---- 1. kept keys (own slots) and query rows, then the gathers ----
    // Every load is unconditional at a clamped in-bounds address, with validity applied to the logits. Per
    // batch element a 64-bit base, within it 32-bit offsets (a map is below 2^31 bytes by the host's checks).
    constexpr int kShift = ROW ? 1 : 2;              // children per kept key
    const int last_sel = (ROW && pair2 ? 2 * K : K) - 1;
    const int nslot = (last_sel + 1) << kShift;
    const int32_t* prow = a.parent_idx + static_cast<size_t>(b) * static_cast<uint32_t>(a.heads * Np * K) +
                          static_cast<uint32_t>((h * Np + P) * K);
    const int own = 16 * (lane & 3) + (lane >> 2);   // this lane addresses slots own + 64u
    int J[SPL];
#pragma unroll
    for (int u = 0; u < SPL; ++u)
        J[u] = load_at<int32_t>(prow, static_cast<uint32_t>(min((64 * u + own) >> kShift, last_sel)) * 4u);
    float sigma[VA ? NT : 1];                        // A: the parents' scores of slots 16t + n16
    if constexpr (VA) {
        const float* pk = a.parent_key + static_cast<size_t>(b) * static_cast<uint32_t>(a.heads * Np * K) +
                          static_cast<uint32_t>((h * Np + P) * K);
#pragma unroll
        for (int t = 0; t < NT; ++t)
            sigma[t] = load_at<float>(pk, static_cast<uint32_t>(min((16 * t + n16) >> kShift, last_sel)) * 4u);
    }
    uint4 qa[NJ];                                    // MFMA operand row n16 holds query n16 >> 2
    {
        const int qi = n16 >> 2;
        int qy, qx;
        query_yx(qi, qy, qx);
        const bool on = qy < H && qx < W;
        const bool qb = !FINEST && a.q_blocked;      // level 0 is NHWC
        const unsigned char* qbase = static_cast<const unsigned char*>(a.q) +
            (qb ? ((static_cast<size_t>(b) * a.heads + h) * Np + P) * 4 * RB
                : (static_cast<size_t>(b) * N * C + h * D) * 2);
        // (ROW, blocked: query 4p + qi is child qi & 1 of parent 2p + (qi >> 1), which may not exist)
        const int qblk = ROW ? (on ? (qi >> 1) * 4 + (qi & 1) : 0) : qi;
        const uint32_t qoff = qb ? static_cast<uint32_t>(qblk * RB)
                                 : __umul24(static_cast<uint32_t>(__mul24(min(qy, H - 1), W) + min(qx, W - 1)), tok_bytes);
#pragma unroll
        for (int j = 0; j < NJ; ++j) qa[j] = load_at<uint4>(qbase, qoff + static_cast<uint32_t>((g + 4 * j) * 16));
    }

    const bool kvb = !FINEST && a.kv_blocked;
    const size_t kv_base = kvb ? (static_cast<size_t>(b) * a.heads + h) * Np * 4 * RB
                               : (static_cast<size_t>(b) * N * C + h * D) * 2;
    const unsigned char* kg = static_cast<const unsigned char*>(a.k) + kv_base;
    const unsigned char* vg = static_cast<const unsigned char*>(a.v) + kv_base;
    int flat[SPL];                                   // the slot's flat index at level l; negative: none
    uint64_t okm[SPL];                               // bit 4n + t: slot 64u + 16t + n is a candidate
    uint32_t off[NT];                                // tile t: this lane's chunk of slot 16t + (lane >> 2)
    const uint32_t chunk16 = gather_chunk(lane);
    uint32_t first = 0u;                             // slot 0's row, always a candidate's
#pragma unroll
    for (int u = 0; u < SPL; ++u) {
        const int s = 64 * u + own;
        const int Jc = max(J[u], 0);
        uint32_t o;
        bool ok;
        if constexpr (ROW) {
            flat[u] = 2 * Jc + (s & 1);
            ok = s < nslot && J[u] >= 0 && flat[u] < W;
            o = kvb ? static_cast<uint32_t>(Jc * 4 + (s & 1)) * RB : __umul24(static_cast<uint32_t>(flat[u]), tok_bytes);
        } else {
            const int Jy = fast_div(Jc, a.div_Wp), Jx = Jc - __mul24(Jy, a.Wp);
            const int cy = 2 * Jy + ((s >> 1) & 1), cx = 2 * Jx + (s & 1);
            flat[u] = __mul24(cy, W) + cx;
            ok = s < nslot && J[u] >= 0 && cy < H && cx < W;
            o = kvb ? static_cast<uint32_t>(Jc * 4 + (s & 3)) * RB : __umul24(static_cast<uint32_t>(flat[u]), tok_bytes);
        }
        // a missing candidate reads slot 0's row: its weight is zero, and zero times a row that the queries attend
        // anyway takes an infinity or a NaN nowhere else
        if (u == 0) first = __builtin_amdgcn_readfirstlane(o);
        o = ok ? o : first;
        flat[u] = ok ? flat[u] : -1;
        okm[u] = __ballot(ok);
        quad_offsets<(NT < 4 ? NT : 4)>(o, chunk16, off + 4 * u);
    }
    // key rows in registers, at most four tiles at a time (more would cost occupancy)
    constexpr int kTB = NT < 4 ? NT : 4;
    uint4 kc[kTB][NJ];
    auto load_keys = [&](int t0) {
#pragma unroll
        for (int i = 0; i < kTB; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                if (t0 + i < LIVE) kc[i][j] = load_at<uint4>(kg, off[t0 + i] + 64 * j);
    };
    load_keys(0);
    const __amdgpu_buffer_rsrc_t vres = map_resource(vg);
    // value rows into LDS: one instruction lands its lanes' chunks in lane order
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            if (t < LIVE) load_lds16(vres, off[t], 64 * j, vlds + t * TS + j * 1024);
            else *(lds_ptr<u32x4_t>)(vlds + t * TS + j * 1024 + lane * 16) = u32x4_t{0u, 0u, 0u, 0u};
        }

    // ---- the finest level's combination inputs. Lane 16g + n ends with query g's message at channels
    //      16 ct + n. out = w_0 m + sum over the ancestors e of w_e anc_e is a product of a 4 x E by an E x D
    //      matrix: MFMA operands with lane 16g + n holding w of query n >> 2 for ancestor g, and channel
    //      16 ct + n of ancestor g's message: one load each for four levels. ----
    int oy, ox;
    query_yx(g, oy, ox);
    const bool o_ok = oy < H && ox < W;
    const uint32_t opos = static_cast<uint32_t>(__mul24(min(oy, H - 1), W) + min(ox, W - 1));
    float w0 = 1.f, wa = 0.f, an[FINEST ? CT : 1];
    const float* const an_dummy = a.anc[1].msg;
    // ancestors: levels 1 .. L-1; a pair of parents (ROW) has two at level 1, first
    const int nanc = a.levels - 1 + (ROW ? 1 : 0);
    auto load_ancestors = [&](int e0) {
        if constexpr (FINEST) {
            const int e = min(e0 + g, nanc - 1);                 // past the last: repeats it, weight 0
            const int lev = ROW ? max(e, 1) : e + 1;
            const auto& t = a.anc[lev];
            const uint32_t ay = static_cast<uint32_t>((2 * Py) >> lev);
            const uint32_t ax = static_cast<uint32_t>((ROW ? 2 * P + (e == 1 ? 2 : 0) : 2 * Px) >> lev);
            const uint32_t at = __umul24(ay, static_cast<uint32_t>(t.W)) + min(ax, static_cast<uint32_t>(t.W - 1));
            const float* mr = t.msg + static_cast<size_t>(b) * t.map_floats + (at * static_cast<uint32_t>(C) + static_cast<uint32_t>(h * D + n16));
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) an[ct] = mr[16 * ct];
            const int qi = n16 >> 2;
            float w = VA ? 1.f : a.inv_levels;
            if constexpr (!VA) {
                int wy, wx;
                query_yx(qi, wy, wx);
                // without w a coarser message is read in its place (not used)
                const float* wb = a.w ? a.w + (static_cast<size_t>(b) * N * a.heads + h) * a.levels : an_dummy;
                const uint32_t wq = __umul24(static_cast<uint32_t>(__mul24(min(wy, H - 1), W) + min(wx, W - 1)),
                                             static_cast<uint32_t>(a.heads * a.levels));
                const float wr = load_at<float>(wb, a.w ? (wq + lev) * 4u : 0u);
                w = a.w ? wr : w;
                if (e0 == 0) {
                    const float w0r = load_at<float>(wb, a.w ? __umul24(opos, static_cast<uint32_t>(a.heads * a.levels)) * 4u : 0u);
                    w0 = a.w ? w0r : a.inv_levels;
                }
            }
            // (ROW: level 1's first entry is the first parent's, for queries 0 and 1, the second the other's)
            const bool mine = e0 + g < nanc && (!ROW || e > 1 || (qi >> 1) == e);
            wa = mine ? w : 0.f;
        }
    };
    load_ancestors(0);

    // ---- 2. logits (unscaled: the scale is positive and enters with the exponential) ----
    float xt[NT];
#pragma unroll
    for (int t0 = 0; t0 < NT; t0 += kTB) {
        if (t0 > 0) load_keys(t0);
#pragma unroll
        for (int i = 0; i < kTB; ++i) {
            if (t0 + i >= LIVE) {
                xt[t0 + i] = 0.f;                                // (masked below)
                continue;
            }
            float4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, qa[j]),
                                                              pass_operand(kc[i][j], slds, lane), acc, 0, 0, 0);
            xt[t0 + i] = acc[0];                                 // rows 4g .. 4g+3 are all query g
        }
    }
    // candidates that do not exist (ROW: or belong to the other parent of the pair). Mostly every slot
    // holds a candidate, and the masks are skipped
    bool full = !ROW;
#pragma unroll
    for (int u = 0; u < SPL; ++u)
        full = full && okm[u] == (NT >= 4 ? ~0ull : NT == 2 ? 0x3333333333333333ull : 0x1111111111111111ull);
    if (!full) {                                                 // uniform
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            bool okt = ((okm[t >> 2] >> (4 * n16 + (t & 3))) & 1ull) != 0ull;
            if constexpr (ROW) okt = okt && (16 * t + n16 >= 2 * K) == (g >= 2);
            xt[t] = okt ? xt[t] : -INFINITY;
        }
    }

    // ---- 3. weights ----
    const float c_exp = a.scale * 1.44269504088896341f;          // exp(scale * x) = exp2(c_exp * x)
    float wt[NT];
    float inv = 1.f;                                             // B: 1/sum of query g
    if constexpr (!VA) {
        float m = xt[0];
#pragma unroll
        for (int t = 1; t < NT; ++t) m = fmaxf(m, xt[t]);
        m = row_allreduce(m, [](float u, float v) { return fmaxf(u, v); });
        float se = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            wt[t] = __builtin_amdgcn_exp2f((xt[t] - m) * c_exp);
            se += wt[t];
        }
        inv = fast_rcp(row_allreduce(se, [](float u, float v) { return u + v; }));   // sum >= 1
    } else {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            // a softmax over the children of one kept key (a lane quad; ROW: a lane pair); a key whose
            // first child is missing has none
            float m = fmaxf(xt[t], xchg_f32<1>(xt[t]));
            if constexpr (!ROW) m = fmaxf(m, xchg_f32<2>(m));
            const bool live = xt[t] > -INFINITY;
            const float e = live ? __builtin_amdgcn_exp2f((xt[t] - m) * c_exp) : 0.f;
            float se = e + xchg_f32<1>(e);
            if constexpr (!ROW) se += xchg_f32<2>(se);
            wt[t] = live ? sigma[t] * e * fast_rcp(se) : 0.f;    // se >= 1
        }
    }

    // ---- 5a. the weights into LDS: [query g][place of n16][t] ----
    store_weights<NT>(plds, wt, lane);
    // (A's selection below clears single weights among them through another type, which alone would not keep the
    // compiler from moving these stores past those)
    if constexpr (VA && !FINEST) asm volatile("" ::: "memory");

    // ---- 4. this level's selection (levels above the finest): each query keeps its Ks best candidates ----
    if constexpr (!FINEST) {
        // ranking keys (B: the logit, ordered as the probability; A: the score) and scores, one slot per lane
        float kvs[SPL][4], scs[VA ? 1 : SPL][4];
#pragma unroll
        for (int u = 0; u < SPL; ++u) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = 4 * u + j;
                kvs[u][j] = t < NT ? (VA ? wt[t] : xt[t]) : 0.f;
                if constexpr (!VA) scs[u][j] = t < NT ? wt[t] * inv : 0.f;
            }
            rows_transpose4(kvs[u]);
            if constexpr (!VA) rows_transpose4(scs[u]);
        }
        // the candidates' names, one slot per lane too: slot 64u + lane was addressed by lane
        // 4 (lane & 15) + (lane >> 4)
        int nm[SPL];
#pragma unroll
        for (int u = 0; u < SPL; ++u) nm[u] = __builtin_amdgcn_ds_bpermute((4 * n16 + g) * 4, flat[u]);
        const size_t sel_base = (static_cast<size_t>(b) * a.heads + h) * N;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int qy, qx;
            query_yx(r, qy, qx);
            if (qy >= H || qx >= W) continue;                    // uniform
            bool okr[SPL];
            uint32_t key[SPL], name[SPL];
            int nvalid = 0;
#pragma unroll
            for (int u = 0; u < SPL; ++u) {
                const int s = 64 * u + lane;
                okr[u] = nm[u] >= 0 && (!ROW || (s >= 2 * K) == (r >= 2));
                nvalid += __popcll(__ballot(okr[u]));
                key[u] = okr[u] ? ordered_bits(kvs[u][r]) : 0u;
                name[u] = static_cast<uint32_t>(nm[u]);
            }
            const int keff = Ks < nvalid ? Ks : nvalid;
            bool kept[SPL];
            wave_select_top<SPL>(key, name, keff, kept);
            int32_t* const so = a.sel_idx + (sel_base + static_cast<uint32_t>(qy * W + qx)) * Ks;
            float* const ko = a.sel_key + (sel_base + static_cast<uint32_t>(qy * W + qx)) * Ks;
            int before = 0;
#pragma unroll
            for (int u = 0; u < SPL; ++u) {
                const uint64_t mask = __ballot(kept[u]);
                if (kept[u]) {
                    const uint32_t at = static_cast<uint32_t>(before + lanes_below(mask)) * 4u;
                    store_at<int32_t>(so, at, nm[u]);
                    store_at<float>(ko, at, VA ? kvs[u][r] : scs[VA ? 0 : u][r]);
                    // A: refined at the next level (Omega)
                    if constexpr (VA)
                        *(lds_ptr<uint16_t>)(plds + ((r * 16 + weight_place<NT>(n16)) * NT + 4 * u + g) * 2) = 0;
                }
                before += __popcll(mask);
            }
            if (lane >= keff && lane < Ks) {
                store_at<int32_t>(so, static_cast<uint32_t>(lane) * 4u, -1);
                store_at<float>(ko, static_cast<uint32_t>(lane) * 4u, 0.f);
            }
        }
    }
    wait_lds_loads();
    wave_lds_sync();

    // ---- 5b. messages ----
    float4_t m4[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) m4[ct] = float4_t{0.f, 0.f, 0.f, 0.f};
    mma_rows<D, NT, 1>(m4, plds, 0, vlds, lane);
    // rows 4g .. 4g+3 of the product are all query g
    float m[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) m[ct] = VA ? m4[ct][0] : m4[ct][0] * inv;

    // ---- 6. outputs ----
    if constexpr (!FINEST) {
        if (o_ok) {
            float* mb = a.msg + (static_cast<size_t>(b) * N * a.heads + h) * D;
            const uint32_t at = (opos * static_cast<uint32_t>(a.heads * D) + n16) * 4u;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) store_at<float>(mb, at + 64 * ct, m[ct]);
        }
    } else {
        if (a.pe0) {                                             // uniform: a separately computed encoding
            const float* pb = a.pe0 + (static_cast<size_t>(b) * N * a.heads + h) * D;
            const uint32_t at = (opos * static_cast<uint32_t>(a.heads * D) + n16) * 4u;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) m[ct] += load_at<float>(pb, at + 64 * ct);
        }
        float4_t o[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            o[ct] = float4_t{w0 * m[ct], 0.f, 0.f, 0.f};
            o[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(wa, an[ct], o[ct], 0, 0, 0);
        }
        for (int e0 = 4; e0 < nanc; e0 += 4) {                   // uniform: more than four ancestors
            load_ancestors(e0);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) o[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(wa, an[ct], o[ct], 0, 0, 0);
        }
        // neighbouring lanes trade a channel per two tiles: even lanes end with channels n, n + 1 of the first
        // tile, odd ones with n - 1, n of the second, a four-byte store each
        void* ob = static_cast<unsigned char*>(a.out) + (static_cast<size_t>(b) * N * C + h * D) * 2;
        const bool odd = (lane & 1) != 0;
        const uint32_t at = (opos * static_cast<uint32_t>(C) + (odd ? n16 + 15 : n16)) * 2u;
#pragma unroll
        for (int ct = 0; ct < CT; ct += 2) {
            const float x = o[ct][0], y = o[ct + 1][0];
            const float r = xchg_f32<1>(odd ? x : y);
            const uint32_t v = pack2(odd ? r : x, odd ? y : r);
            if (o_ok) store_at<uint32_t>(ob, at + 32 * ct, v);
        }
    }
}

}  // namespace fine16
}  // namespace qta

#endif
