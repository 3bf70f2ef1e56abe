// The finer levels' backward passes for bf16 maps (step 2 of backward.hip), on the row tiles of bf16_tiles.h:
// the combination's backward, and the finer levels' query and key passes. backward.hip holds the fp32 forms,
// with the derivation.
//
// Both passes contract fp32 weights (the logit gradients, the value weights) with bf16 rows. The weights are
// split exactly into three bf16 terms (8 + 8 + 8 bits), whose products with a bf16 row are exact in the
// MFMA's fp32 accumulator, so the sums are as accurate as on the fp32 MFMA at a sixth of its time.
//
// What bounds them, before -> now: the previous forms gathered with a lane per row (46 to 64 cycles of a CU
// an instruction, see bf16_tiles.h) and read the rows back from LDS two bytes at a time, one fp32 4x4 MFMA per
// slot. Finest level in a training step, 200x336 maps, 2 x 32 channels, K = 16, batch 2: query pass 125 us with
// the combination's backward -> 69 and 22 for that, key pass with its reduction 172 -> 111; 32 maps of 56x56,
// 1 x 64, K = 8: query pass 50 -> 25 and 14, key pass 76 -> 45.
#ifndef QTA_BWD_BF16_H
#define QTA_BWD_BF16_H

#include <type_traits>

#include "bf16_tiles.h"
#include "qta_internal.h"

namespace qta {
namespace bwd16 {

using namespace tiles;

// Lane 16g + n's fp32 weights of vector g as three planes of mma_rows' weights, 128 NT bytes apart.
template <int NT>
__device__ __forceinline__ void store_split(lds_byte* w, const float (&x)[NT], int lane)
{
    lds_byte* const p = w + ((lane >> 4) * 16 + weight_place<NT>(lane & 15)) * NT * 2;
    constexpr int PB = 128 * NT;
    if constexpr (NT == 1) {
        const Split2 s = split2(x[0], 0.f);
        *(lds_ptr<uint16_t>)p = static_cast<uint16_t>(s.hi);
        *(lds_ptr<uint16_t>)(p + PB) = static_cast<uint16_t>(s.mid);
        *(lds_ptr<uint16_t>)(p + 2 * PB) = static_cast<uint16_t>(s.lo);
    } else if constexpr (NT == 2) {
        const Split2 s = split2(x[0], x[1]);
        *(lds_ptr<uint32_t>)p = s.hi;
        *(lds_ptr<uint32_t>)(p + PB) = s.mid;
        *(lds_ptr<uint32_t>)(p + 2 * PB) = s.lo;
    } else {
        const Split2 s = split2(x[0], x[1]), r = split2(x[2], x[3]);
        *(lds_ptr<u32x2_t>)p = u32x2_t{s.hi, r.hi};
        *(lds_ptr<u32x2_t>)(p + PB) = u32x2_t{s.mid, r.mid};
        *(lds_ptr<u32x2_t>)(p + 2 * PB) = u32x2_t{s.lo, r.lo};
    }
}

// Lane 16g + n's row values at channels 16 ct + n to element `at` of the map at `base`, in fp32 or (MAY16 and
// `half`, uniform) bf16: neighbouring lanes then trade a channel per two tiles for four-byte stores.
template <int D, bool MAY16>
__device__ __forceinline__ void store_row(float* map, bool half, size_t base, uint32_t at, const float (&x)[D / 16], bool on, int lane)
{
    const int n16 = lane & 15;
    if (MAY16 && half) {                                      // uniform
        unsigned char* const b = reinterpret_cast<unsigned char*>(map) + base * 2;
        const bool odd = (lane & 1) != 0;
        const uint32_t to = (at + (odd ? n16 + 15 : n16)) * 2u;
#pragma unroll
        for (int ct = 0; ct < D / 16; ct += 2) {
            const float r = xchg_f32<1>(odd ? x[ct] : x[ct + 1]);
            const uint32_t v = pack2(odd ? r : x[ct], odd ? x[ct + 1] : r);
            if (on) store_at<uint32_t>(b, to + 32 * ct, v);
        }
    } else if (on) {
        float* const b = map + base;
#pragma unroll
        for (int ct = 0; ct < D / 16; ++ct) store_at<float>(b, (at + n16) * 4u + 64 * ct, x[ct]);
    }
}

// One wave's LDS: the row tiles, then 1 KB for chunks in passing and, after them, the three weight planes.
template <int D, int NT>
constexpr int wave_bytes() { return NT * tile_bytes<D>() + (NT == 4 ? 1536 : 1024); }

// ---------------------------------------------------------------------------------------------
// query pass
// ---------------------------------------------------------------------------------------------

// One work item: parent query P at level l+1 and head h (it = (b*Np + P)*heads + h); its four children at
// level l share the candidate slots 4r + c (child c of the parent's kept key r), in NT tiles of 16. Lane
// 16g + n works on query g and slots 16t + n.
template <int D, int NT, bool VA, bool FINEST>
__device__ __forceinline__ void query_item(const BwdLevelArgs& a, const int it, unsigned char* const base)
{
    constexpr int RB = D * 2;              // bytes of one head's row
    constexpr int NJ = RB / 64;            // chunks per lane and row
    constexpr int CT = D / 16;             // 16-channel tiles
    constexpr int TS = tile_bytes<D>();
    static_assert(NT == 1 || NT == 2 || NT == 4, "at most 64 candidate slots");

    const int lane = threadIdx.x & 63, n16 = lane & 15, g = lane >> 4;
    lds_byte* const klds = (lds_byte*)base;
    lds_byte* const work = klds + NT * TS;
    const int Np = a.Hp * a.Wp;
    const int bp = fast_div(it, a.div_heads);
    const int h = it - bp * a.heads;
    const int b = fast_div(bp, a.div_Np);
    const int P = bp - b * Np;
    const int Py = fast_div(P, a.div_Wp), Px = P - Py * a.Wp;
    const int H = a.H, W = a.W, C = a.C, K = a.Kp;
    const int N = H * W;
    const uint32_t tok_bytes = static_cast<uint32_t>(C * 2);
    const size_t prow_off = (static_cast<size_t>(b) * a.heads + h) * Np + P;
    const int32_t* prow = a.parent_idx + prow_off * K;

    // ---- kept keys, query rows and message gradients, then the gathers (every load unconditional, at a
    //      clamped in-bounds address) ----
    const int own = 16 * (lane & 3) + (lane >> 2);            // the slot this lane addresses
    const int J = load_at<int32_t>(prow, static_cast<uint32_t>(min(own >> 2, K - 1)) * 4u);
    const int Jk = load_at<int32_t>(prow, static_cast<uint32_t>(min(lane, K - 1)) * 4u);
    float sigma[VA ? NT : 1];                                 // A: the parents' scores of slots 16t + n16
    if constexpr (VA) {
        const float* pk = a.parent_key + prow_off * K;
#pragma unroll
        for (int t = 0; t < NT; ++t) sigma[t] = load_at<float>(pk, static_cast<uint32_t>(min(4 * t + (n16 >> 2), K - 1)) * 4u);
    }
    // MFMA operand row n16 holds query n16 >> 2
    const int qi = n16 >> 2;
    const int qy = 2 * Py + (qi >> 1), qx = 2 * Px + (qi & 1);
    const uint32_t qtok = static_cast<uint32_t>(__mul24(min(qy, H - 1), W) + min(qx, W - 1));
    bf16x8_t qa[NJ];
    {
        const unsigned char* qbase = static_cast<const unsigned char*>(a.q) +
            (a.blocked ? prow_off * 4 * RB : (static_cast<size_t>(b) * N * C + h * D) * 2);
        const uint32_t qoff = a.blocked ? static_cast<uint32_t>(qi * RB) : __umul24(qtok, tok_bytes);
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            qa[j] = __builtin_bit_cast(bf16x8_t, load_at<uint4>(qbase, qoff + static_cast<uint32_t>((g + 4 * j) * 16)));
    }
    // the gradient of the queries' messages as the operand of <dm, v>: at level 0 dout (times w_0 in the
    // weights), at the others dm in three bf16 terms
    constexpr int DP = FINEST ? 1 : 3;
    bf16x8_t da[DP][NJ];
    if constexpr (FINEST) {
        const unsigned char* db = static_cast<const unsigned char*>(a.dout) + (static_cast<size_t>(b) * N * C + h * D) * 2;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            da[0][j] = __builtin_bit_cast(bf16x8_t, load_at<uint4>(db, __umul24(qtok, tok_bytes) + static_cast<uint32_t>((g + 4 * j) * 16)));
    } else {
        const float* mb = a.dm + static_cast<size_t>(b) * N * C + h * D;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t at = (qtok * static_cast<uint32_t>(C) + static_cast<uint32_t>((g + 4 * j) * 8)) * 4u;
            const float4_t x = load_at<float4_t>(mb, at), y = load_at<float4_t>(mb, at + 16);
            const Split2 s0 = split2(x[0], x[1]), s1 = split2(x[2], x[3]), s2 = split2(y[0], y[1]), s3 = split2(y[2], y[3]);
            da[0][j] = __builtin_bit_cast(bf16x8_t, u32x4_t{s0.hi, s1.hi, s2.hi, s3.hi});
            da[DP > 1 ? 1 : 0][j] = __builtin_bit_cast(bf16x8_t, u32x4_t{s0.mid, s1.mid, s2.mid, s3.mid});
            da[DP > 1 ? 2 : 0][j] = __builtin_bit_cast(bf16x8_t, u32x4_t{s0.lo, s1.lo, s2.lo, s3.lo});
        }
    }
    // this lane's query g
    const int oy = 2 * Py + (g >> 1), ox = 2 * Px + (g & 1);
    const bool qv = oy < H && ox < W;
    const uint32_t qpos = static_cast<uint32_t>(__mul24(min(oy, H - 1), W) + min(ox, W - 1));
    const size_t wq_off = static_cast<size_t>(b) * static_cast<uint32_t>(N * a.heads * a.levels);
    const uint32_t wrow = (qpos * static_cast<uint32_t>(a.heads) + h) * static_cast<uint32_t>(a.levels);
    float w0 = 1.f;
    if constexpr (FINEST && !VA) w0 = a.w ? load_at<float>(a.w + wq_off, wrow * 4u) : 1.0f / a.levels;

    const bool kvb = a.blocked;
    const size_t kv_base = kvb ? (static_cast<size_t>(b) * a.heads + h) * Np * 4 * RB
                               : (static_cast<size_t>(b) * N * C + h * D) * 2;
    const unsigned char* vg = static_cast<const unsigned char*>(a.v) + kv_base;
    const __amdgpu_buffer_rsrc_t kres = map_resource(static_cast<const unsigned char*>(a.k) + kv_base);
    uint32_t off[NT];
    int flat;                                                 // the slot's flat index at level l
    uint64_t okm;                                             // bit 4n + t: slot 16t + n is a candidate
    {
        const int Jc = max(J, 0);
        const int Jy = fast_div(Jc, a.div_Wp), Jx = Jc - __mul24(Jy, a.Wp);
        const int cy = 2 * Jy + ((own >> 1) & 1), cx = 2 * Jx + (own & 1);
        flat = __mul24(cy, W) + cx;
        const bool ok = own < 4 * K && J >= 0 && cy < H && cx < W;
        uint32_t o = kvb ? static_cast<uint32_t>(Jc * 4 + (own & 3)) * RB : __umul24(static_cast<uint32_t>(flat), tok_bytes);
        // a missing candidate reads the row of slot 0, always a candidate's (see fine_bf16.h)
        const uint32_t first = __builtin_amdgcn_readfirstlane(o);
        o = ok ? o : first;
        flat = ok ? flat : -1;
        okm = __ballot(ok);
        quad_offsets<NT>(o, gather_chunk(lane), off);
    }
    // the parent's total gradient of q (without one, the first kept key is read in its place, unused)
    float up[CT];
    const float share = child_share(Py, Px, H, W);
    {
        const float* ub = a.up_q ? a.up_q + (static_cast<size_t>(b) * Np + P) * C + h * D : reinterpret_cast<const float*>(a.parent_idx);
        const uint32_t at = a.up_q ? static_cast<uint32_t>(n16 * 4) : 0u;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) up[ct] = load_at<float>(ub, at + (a.up_q ? 64u * ct : 0u));
    }
    uint4 vc[NT][NJ];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < NJ; ++j) vc[t][j] = load_at<uint4>(vg, off[t] + 64 * j);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < NJ; ++j) load_lds16(kres, off[t], 64 * j, klds + t * TS + j * 1024);
    // how many parents kept each key of level l+1 (for the key pass's counting sort); the count a pair finds
    // is its place in the key's list
    if (lane < K && Jk >= 0)
        a.slot[prow_off * K + lane] = atomicAdd(a.count + (static_cast<size_t>(b) * a.heads + h) * Np + Jk, 1);

    // ---- logits and <dm, v> ----
    float x[NT], gs[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        float4_t ag = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const bf16x8_t vv = pass_operand(vc[t][j], work, lane);
#pragma unroll
            for (int p = 0; p < DP; ++p) ag = __builtin_amdgcn_mfma_f32_16x16x32_bf16(da[p][j], vv, ag, 0, 0, 0);
        }
        gs[t] = ag[0];                                        // rows 4g .. 4g+3 are all query g
    }
    wait_lds_loads();                                         // the key rows
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        float4_t ax = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            ax = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[j], tile_operand(klds + t * TS + j * 1024, lane), ax, 0, 0, 0);
        x[t] = ((okm >> (4 * n16 + t)) & 1ull) != 0ull ? ax[0] * a.scale : -INFINITY;
    }

    // ---- softmax gradients ----
    // The sum over the query's slots of one value per tile, in the order of a butterfly over the 64 slots
    // (each tile over its 16-lane row, then tiles (0 + 1) + (2 + 3))
    auto slots_sum = [&](const float (&v)[NT]) -> float {
        float r[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < NT; ++t) r[t] = row_allreduce(v[t], [](float p, float q) { return p + q; });
        return (r[0] + r[1]) + (r[2] + r[3]);
    };
    float* const st_b = a.stats + static_cast<size_t>(b * a.heads + h) * static_cast<uint32_t>(N * 2 * (VA ? K : 1));
    float dx[NT];
    float dw0 = 0.f;
    if constexpr (!VA) {
        float m = x[0];
#pragma unroll
        for (int t = 1; t < NT; ++t) m = fmaxf(m, x[t]);
        m = row_allreduce(m, [](float p, float q) { return fmaxf(p, q); });
        float e[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) e[t] = __expf(x[t] - m);           // 0 for a missing candidate
        const float sum = slots_sum(e);
        const float inv = fast_rcp(sum);                      // sum >= 1 (the maximum's term)
        float pg[NT], pa[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            e[t] *= inv;
            pa[t] = e[t] * gs[t];
            gs[t] = FINEST ? w0 * gs[t] : gs[t];
            pg[t] = e[t] * gs[t];
        }
        const float Dr = slots_sum(pg);
#pragma unroll
        for (int t = 0; t < NT; ++t) dx[t] = qv ? e[t] * (gs[t] - Dr) : 0.f;
        // the key pass recomputes p = exp(x - lse) and needs D
        if (n16 == 0 && qv) store_at<float2_t>(st_b, qpos * 8u, float2_t{m + fast_ln(sum), Dr});
        if constexpr (FINEST) {
            if (a.w && a.dw) dw0 = slots_sum(pa);             // uniform
        }
    } else {
        // d sigma of each slot's key: a key this lane's query keeps is refined at level l-1, and its
        // score's gradient comes from there
        float ds[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) ds[t] = gs[t];
        if constexpr (!FINEST) {
            int name[NT];                                     // slot 16t + n16 was addressed by lane 4 n16 + t
#pragma unroll
            for (int t = 0; t < NT; ++t) name[t] = __builtin_amdgcn_ds_bpermute(16 * n16 + 4 * t, flat);
            const size_t srow = ((static_cast<size_t>(b) * a.heads + h) * N + qpos) * a.Ks;
            for (int mm = 0; mm < a.Ks; ++mm) {
                const int kept = a.sel_idx[srow + mm];
                const float dv = a.dsig_in[srow + mm];
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    if (name[t] >= 0 && kept == name[t]) ds[t] = dv;
            }
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            // a softmax over the children of one kept key (a lane quad)
            float m = fmaxf(x[t], xchg_f32<1>(x[t]));
            m = fmaxf(m, xchg_f32<2>(m));
            const bool live = x[t] > -INFINITY;
            const float e = live ? __expf(x[t] - m) : 0.f;
            float sum = e + xchg_f32<1>(e);
            sum += xchg_f32<2>(sum);
            const float tt = live ? e * fast_rcp(sum) : 0.f;  // sum >= 1
            const float sc = sigma[t] * tt;
            float dsq = tt * ds[t];                           // this query's d sigma of the kept key
            dsq += xchg_f32<1>(dsq);
            dsq += xchg_f32<2>(dsq);
            dx[t] = qv ? sc * (ds[t] - dsq) : 0.f;
            // the key pass recomputes t = exp(x - lse) per kept parent key and needs sum t ds
            const int key = 4 * t + (n16 >> 2);
            if ((n16 & 3) == 0 && key < K && qv)
                store_at<float2_t>(st_b, static_cast<uint32_t>(qpos * K + key) * 8u, float2_t{m + fast_ln(sum), dsq});
            // the four queries' sum, across the wave's rows
            float dsig = qv ? dsq : 0.f;
            dsig += xchg_f32<16>(dsig);
            dsig += xchg_f32<32>(dsig);
            if (g == 0 && (n16 & 3) == 0 && key < K) a.dsig_out[prow_off * K + key] = dsig;
        }
    }

    // ---- dq = scale * sum_s dx_s k_s, plus the parent's share ----
    store_split<NT>(work, dx, lane);
    wave_lds_sync();
    {
        float4_t o[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) o[ct] = float4_t{0.f, 0.f, 0.f, 0.f};
        mma_rows<D, NT, 3>(o, work, 128 * NT, klds, lane);
        float dq[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) dq[ct] = a.up_q ? a.scale * o[ct][0] + share * up[ct] : a.scale * o[ct][0];
        store_row<D, FINEST>(a.dq, FINEST && a.out_bf16, static_cast<size_t>(b) * N * C + h * D, qpos * static_cast<uint32_t>(C), dq,
                             qv, lane);
    }

    // (the rest of dw, and the coarser levels' message gradients: combine_item)
    if constexpr (FINEST && !VA) {
        if (a.w && a.dw && n16 == 0 && qv) store_at<float>(a.dw + wq_off, wrow * 4u, dw0);
    }
}

// ---------------------------------------------------------------------------------------------
// the combination's backward
// ---------------------------------------------------------------------------------------------

// x plus the other lane's x, for the lane at distance 8, 16 or 32.
template <int M>
__device__ __forceinline__ float add_across(float x)
{
    const uint32_t u = __float_as_uint(x);
    if constexpr (M == 8) {
        return x + __uint_as_float(__builtin_amdgcn_update_dpp(0u, u, kDppRowRor8, 0xF, 0xF, false));
    } else if constexpr (M == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else {
        static_assert(M == 32, "distance");
        const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
}

// dm^l of every level l >= 1 sums w_{i,l} dout_i over a token's level-0 descendants i, and dw_{i,l} =
// <dout_i, m^l of the ancestor>. One wave takes one head of a block of neighbouring parents (level-1 tokens;
// 4x2 with d = 32, 2x2 with d = 64, a run on one-row maps): lane Q i + e has channels 4e .. 4e+3 of parent i's
// four tokens. A level's sums go over the block in registers, and are stored where the block holds all of a
// token's descendants (levels 1 and 2; 1 to 4 on one-row maps) and added with atomics above. Bound by the
// latency of one wave's loads (few waves). Inside the query pass, a wave per parent, it took 31 of that pass's
// 98 us (200x336, 2 x 32, batch 2) and 13 of 38 (32 x 56x56, 1 x 64), with eight times the atomics; alone 21
// and 12, and the coarser levels no longer wait for the finest.
struct CombineGrid {
    FastDiv div_map, div_row;           // blocks of parents per map and per row of blocks
};

template <int D, bool VA, bool ROW>
__device__ __forceinline__ void combine_item(const BwdLevelArgs& a, const CombineGrid& cg, const int it)
{
    constexpr int Q = D / 4;                                  // lanes per parent
    constexpr int NP = 64 / Q;                                // parents per wave
    constexpr int RX = ROW ? NP : NP == 8 ? 4 : 2, RY = NP / RX;
    const int lane = threadIdx.x & 63;
    const int e = lane & (Q - 1), i = lane / Q;
    const int blk = fast_div(it, a.div_heads), h = it - blk * a.heads;
    const int b = fast_div(blk, cg.div_map), br = blk - b * cg.div_map.d;
    const int y0 = fast_div(br, cg.div_row), x0 = br - y0 * cg.div_row.d;
    // the bits of i: x, then y, then x again, so that 2x2 parents are four neighbours
    const int Px = x0 * RX + (ROW ? i : (i & 1) | ((i >> 1) & 2)), Py = ROW ? 0 : y0 * RY + ((i >> 1) & 1);
    const bool pv = Px < a.Wp && Py < a.Hp;
    const int H = a.H, W = a.W, C = a.C, L = a.levels;
    const int N = H * W;
    const bool want_dw = !VA && a.w && a.dw;                  // uniform
    const unsigned char* db = static_cast<const unsigned char*>(a.dout) + (static_cast<size_t>(b) * N * C + h * D) * 2;
    const float* const wb = a.w ? a.w + (static_cast<size_t>(b) * N * a.heads + h) * L : nullptr;
    float g[4][4];                                            // dout of token q, zero off the map
    uint32_t wrow[4];
    bool qv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int y = 2 * Py + (q >> 1), x = 2 * Px + (q & 1);
        qv[q] = pv && y < H && x < W;
        const uint32_t tok = static_cast<uint32_t>(__mul24(min(y, H - 1), W) + min(x, W - 1));
        wrow[q] = tok * static_cast<uint32_t>(a.heads * L);
        const unsigned m = opaque_mask(qv[q]);
        const uint2 r = load_at<uint2>(db, __umul24(tok, static_cast<uint32_t>(C * 2)) + static_cast<uint32_t>(e * 8));
        g[q][0] = low_half(r.x & m);
        g[q][1] = high_half(r.x & m);
        g[q][2] = low_half(r.y & m);
        g[q][3] = high_half(r.y & m);
    }
    for (int l0 = 1; l0 < L; l0 += 4) {                       // uniform: four levels at a time
        // w of the four levels by token: 16 bytes at a level that leaves them inside the row (rows of two or
        // three levels: 8 bytes)
        float w[4][4];
        if (!VA && a.w) {                                     // uniform
            typedef float float4u_t __attribute__((ext_vector_type(4), aligned(4)));
            typedef float float2u_t __attribute__((ext_vector_type(2), aligned(4)));
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (L >= 4) {                                 // uniform
                    const int from = min(l0, L - 4), sh = l0 - from;
                    const float4u_t v = load_at<float4u_t>(wb, (wrow[q] + from) * 4u);
                    w[q][0] = sh == 0 ? v[0] : sh == 1 ? v[1] : sh == 2 ? v[2] : v[3];
                    w[q][1] = sh == 0 ? v[1] : sh == 1 ? v[2] : v[3];
                    w[q][2] = sh == 0 ? v[2] : v[3];
                    w[q][3] = v[3];
                } else {
                    const float2u_t v = load_at<float2u_t>(wb, (wrow[q] + L - 2) * 4u);    // levels L-2, L-1
                    w[q][0] = L == 3 ? v[0] : v[1];
                    w[q][1] = w[q][2] = w[q][3] = v[1];
                }
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int j = 0; j < 4; ++j) w[q][j] = VA ? 1.f : 1.0f / L;
        }
        float4_t m[4];
        uint32_t row[4];                                      // bytes within a batch element's messages (below 2^32)
        size_t map[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int l = min(l0 + j, L - 1);                 // uniform; clamped: unused past L-1
            const int y = min(Py, a.Hp - 1) >> (l - 1), x = min(Px, a.Wp - 1) >> (l - 1);
            row[j] = (static_cast<uint32_t>(__mul24(y, a.lvl_W[l]) + x) * static_cast<uint32_t>(C) +
                      static_cast<uint32_t>(h * D + 4 * e)) * 4u;
            map[j] = static_cast<size_t>(b) * static_cast<uint32_t>(a.lvl_N[l]) * static_cast<uint32_t>(C);
            if (want_dw) m[j] = load_at<float4_t>(a.msg_fwd[l] + map[j], row[j]);
        }
        float part[4][4];                                     // dw of token q, level l0 + j
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int l = min(l0 + j, L - 1);                 // uniform; past L-1 nothing is stored
            float4_t s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int c = 0; c < 4; ++c) s[c] += w[q][j] * g[q][c];
            if (want_dw) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    part[q][j] = group_sum<Q>(g[q][0] * m[j][0] + g[q][1] * m[j][1] + g[q][2] * m[j][2] + g[q][3] * m[j][3]);
            }
            // over the block's parents that share the level-l ancestor
            int bits = 0;                                     // of i, summed over
            if (l >= 2) {                                     // uniform
#pragma unroll
                for (int c = 0; c < 4; ++c) s[c] = add_across<Q>(s[c]);
                bits = 1;
                if (!ROW || l >= 3) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) s[c] = add_across<2 * Q>(s[c]);
                    bits = 3;
                }
                if (NP == 8 && l >= (ROW ? 4 : 3)) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) s[c] = add_across<32>(s[c]);
                    bits = 7;
                }
            }
            // (a group's first parent exists whenever any does)
            if (l0 + j < L && pv && (i & bits) == 0) {
                float* const dst = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(a.dm_out[l] + map[j]) + row[j]);
                if (l == 1 || (ROW ? (1 << (l - 1)) <= NP : l == 2)) {      // uniform
                    *reinterpret_cast<float4_t*>(dst) = s;
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) unsafeAtomicAdd(dst + c, s[c]);
                }
            }
        }
        if (want_dw) {
            // lane e stores token e >> 1's levels l0 + 2 (e & 1) and the next
            const int q = (e >> 1) & 3;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float v = q == 0 ? part[0][j] : q == 1 ? part[1][j] : q == 2 ? part[2][j] : part[3][j];
                const uint32_t wr = q == 0 ? wrow[0] : q == 1 ? wrow[1] : q == 2 ? wrow[2] : wrow[3];
                const bool on = q == 0 ? qv[0] : q == 1 ? qv[1] : q == 2 ? qv[2] : qv[3];
                if (e < 8 && (e & 1) == (j >> 1) && l0 + j < L && on)
                    store_at<float>(a.dw + (static_cast<size_t>(b) * N * a.heads + h) * L, (wr + l0 + j) * 4u, v);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// key pass
// ---------------------------------------------------------------------------------------------

// A kept key J and this head: its four children (the keys) as MFMA operands, row n16 holding key n16 >> 2 (rows
// clamped onto the map).
template <int D>
struct KeyRows {
    int bh, b, h, Jy, Jx;
    bf16x8_t k[D / 32], v[D / 32];
};

template <int D, bool FINEST>
__device__ __forceinline__ void key_rows(const BwdLevelArgs& a, const int key, KeyRows<D>& r)
{
    const int lane = threadIdx.x & 63, n16 = lane & 15, g = lane >> 4;
    const int Np = a.Hp * a.Wp;
    r.bh = fast_div(key, a.div_Np);
    const int J = key - r.bh * Np;
    r.b = fast_div(r.bh, a.div_heads);
    r.h = r.bh - r.b * a.heads;
    r.Jy = fast_div(J, a.div_Wp);
    r.Jx = J - r.Jy * a.Wp;
    const bool blocked = !FINEST && a.blocked;
    const size_t map0 = blocked ? static_cast<size_t>(key) * 4 * D * 2
                                : (static_cast<size_t>(r.b) * a.H * a.W * a.C + r.h * D) * 2;
    const int c = n16 >> 2;
    const uint32_t tok = static_cast<uint32_t>(__mul24(min(2 * r.Jy + (c >> 1), a.H - 1), a.W) + min(2 * r.Jx + (c & 1), a.W - 1));
    // (a child off the map reads a clamped row, or in blocked storage the first child: its products are not used)
    const bool on = 2 * r.Jy + (c >> 1) < a.H && 2 * r.Jx + (c & 1) < a.W;
    const uint32_t roff = blocked ? static_cast<uint32_t>((on ? c : 0) * D * 2) : __umul24(tok, static_cast<uint32_t>(a.C * 2));
#pragma unroll
    for (int j = 0; j < D / 32; ++j) {
        const uint32_t at = roff + static_cast<uint32_t>((g + 4 * j) * 16);
        r.k[j] = __builtin_bit_cast(bf16x8_t, load_at<uint4>(static_cast<const unsigned char*>(a.k) + map0, at));
        r.v[j] = __builtin_bit_cast(bf16x8_t, load_at<uint4>(static_cast<const unsigned char*>(a.v) + map0, at));
    }
}

// Up to 16 of the parents that kept the key (entries beg .., NT = 1, 2 or 4 tiles of four): slot s = 4e + child
// is a child of parent e, and vector g one of the four keys. Roles as in the query pass with queries and
// keys exchanged: logits and <dout, v> from the gathered query and dout rows, then ok += dx^T Q and
// ov += vw^T dout with the rows in LDS, the query rows first. At the coarser levels dm stands in dout's place,
// fp32 rows as three bf16 terms (of the nine products of terms with vw's the three below 2^-26 are left out).
template <int D, int NT, bool VA, bool FINEST>
__device__ __forceinline__ void key_part(const BwdLevelArgs& a, const KeyRows<D>& kr, const int beg, const int nent,
                                         unsigned char* const base, float4_t (&ok)[D / 16], float4_t (&ov)[D / 16])
{
    constexpr int RB = D * 2;
    constexpr int NJ = RB / 64;
    constexpr int TS = tile_bytes<D>();
    // (opaque: what follows from the lane is worked out again for each part rather than held in registers
    // across the parts, for every number of tiles: 116 registers, and half the waves)
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    const int n16 = lane & 15, g = lane >> 4;
    lds_byte* const rows = (lds_byte*)base;
    lds_byte* const work = rows + NT * TS;
    const int Np = a.Hp * a.Wp;
    const int bh = kr.bh, b = kr.b, h = kr.h, Jy = kr.Jy, Jx = kr.Jx;
    const int H = a.H, W = a.W, C = a.C, N = H * W, K = a.Kp;
    const uint32_t tok_bytes = static_cast<uint32_t>(C * 2);
    const size_t map0 = static_cast<size_t>(b) * N * C + h * D;           // elements
    const bool blocked = !FINEST && a.blocked;

    // ---- the slot this lane addresses: child (own & 3) of parent own >> 2 of the part (the children of a
    //      parent on neighbouring quads), its row, its query's statistics and w_0 ----
    const int own = 16 * (lane & 3) + (lane >> 2);
    const int ent = load_at<int32_t>(a.entries + beg, static_cast<uint32_t>(min(own >> 2, nent - 1)) * 4u);
    const int P = fast_div(ent, a.div_Kp), r = ent - P * K;
    const int Py = fast_div(P, a.div_Wp), Px = P - Py * a.Wp;
    const int qy = 2 * Py + ((own >> 1) & 1), qx = 2 * Px + (own & 1);
    const bool qv = (own >> 2) < nent && qy < H && qx < W;
    const uint32_t qtok = static_cast<uint32_t>(__mul24(min(qy, H - 1), W) + min(qx, W - 1));
    const uint64_t okm = __ballot(qv);                        // bit 4n + t: slot 16t + n holds a query
    const uint32_t chunk = gather_chunk(lane);
    uint32_t off[NT];
    // (a child off the map reads its parent's first: in blocked storage its own place is unwritten padding, and
    // a row of weight 0 must still be finite)
    const int child = qy < H && qx < W ? own & 3 : 0;
    quad_offsets<NT>(blocked ? static_cast<uint32_t>((P * 4 + child) * RB) : __umul24(qtok, tok_bytes), chunk, off);
    const __amdgpu_buffer_rsrc_t qres = map_resource(static_cast<const unsigned char*>(a.q) +
        (blocked ? static_cast<size_t>(bh) * Np * 4 * RB : map0 * 2));
    // this lane's chunk of each slot's dout row, or the eight floats of it of each dm row
    uint4 dc[FINEST ? NT : 1][NJ];
    float4_t dmf[FINEST ? 1 : NT][NJ][2];
    if constexpr (FINEST) {
        const unsigned char* const dbase = static_cast<const unsigned char*>(a.dout) + map0 * 2;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < NJ; ++j) dc[t][j] = load_at<uint4>(dbase, off[t] + 64 * j);
    } else {
        uint32_t moff[NT];
        quad_offsets<NT>(qtok * static_cast<uint32_t>(C) * 4u, 2 * chunk, moff);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int i = 0; i < 2; ++i) dmf[t][j][i] = load_at<float4_t>(a.dm + map0, moff[t] + 128 * j + 16 * i);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < NJ; ++j) load_lds16(qres, off[t], 64 * j, rows + t * TS + j * 1024);
    const float* const st_b = a.stats + static_cast<size_t>(bh) * static_cast<uint32_t>(N * 2 * (VA ? K : 1));
    const float2_t st = load_at<float2_t>(st_b, (VA ? qtok * static_cast<uint32_t>(K) + r : qtok) * 8u);
    float scale_w = 1.0f;                                     // level 0 of B: w_0 of the slot's query; A: the parent's score
    if constexpr (VA) {
        scale_w = a.parent_key[(static_cast<size_t>(bh) * Np + P) * K + r];
    } else if constexpr (FINEST) {
        scale_w = a.w ? load_at<float>(a.w + static_cast<size_t>(b) * static_cast<uint32_t>(N * a.heads * a.levels),
                                       (qtok * static_cast<uint32_t>(a.heads) + h) * static_cast<uint32_t>(a.levels) * 4u)
                      : 1.0f / a.levels;
    }
    // the p-th bf16 term of this lane's chunk of slot 16t + (lane >> 2)
    auto term = [&](int t, int j, int p) -> uint4 {
        if constexpr (FINEST) {
            return dc[t][j];
        } else {
            uint32_t w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const Split2 s = split2(dmf[t][j][i >> 1][2 * (i & 1)], dmf[t][j][i >> 1][2 * (i & 1) + 1]);
                w[i] = p == 0 ? s.hi : p == 1 ? s.mid : s.lo;
            }
            return make_uint4(w[0], w[1], w[2], w[3]);
        }
    };
    constexpr int DP = FINEST ? 1 : 3;

    // ---- <dout, v> and logits: lane 16g + n holds key g's of slots 16t + n ----
    float gs[NT], x[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        float4_t ag = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int p = 0; p < DP; ++p)
                ag = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kr.v[j], pass_operand(term(t, j, p), work, lane), ag, 0, 0, 0);
        gs[t] = ag[0];
    }
    wait_lds_loads();                                         // the query rows
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        float4_t ax = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            ax = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kr.k[j], tile_operand(rows + t * TS + j * 1024, lane), ax, 0, 0, 0);
        x[t] = ax[0];
    }
    const int ky = 2 * Jy + (g >> 1), kx = 2 * Jx + (g & 1);
    const bool key_ok = ky < H && kx < W;
    float dx[NT], vw[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        // slot 16t + n16 was addressed by lane 4 n16 + t
        const int src = 16 * n16 + 4 * t;
        const float lse = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(st[0])));
        const float Dq = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(st[1])));
        const bool valid = key_ok && ((okm >> (4 * n16 + t)) & 1ull) != 0ull;
        const float pr = valid ? __expf(x[t] * a.scale - lse) : 0.f;      // B: p; A: t
        if constexpr (!VA && !FINEST) {
            vw[t] = pr;
            dx[t] = pr * (gs[t] - Dq);
        } else {
            const float sw = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(scale_w)));
            vw[t] = sw * pr;                                  // B: w_0 p (the dout rows come without w_0); A: s
            if constexpr (VA && !FINEST) {
                // a key that the query keeps is refined at level l-1: its score's gradient comes from there, and
                // it has no weight in this level's message
                const int tok = ky * W + kx;
                const size_t srow = (static_cast<size_t>(bh) * N + static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(src, static_cast<int>(qtok)))) * a.Ks;
                bool kept = false;
                float ds = gs[t];
                for (int mm = 0; mm < a.Ks; ++mm) {
                    if (valid && a.sel_idx[srow + mm] == tok) {
                        kept = true;
                        ds = a.dsig_in[srow + mm];
                    }
                }
                dx[t] = vw[t] * (ds - Dq);
                vw[t] = kept ? 0.f : vw[t];
            } else {
                dx[t] = VA ? vw[t] * (gs[t] - Dq) : pr * (sw * gs[t] - Dq);
            }
        }
    }

    // ---- dk from the query rows, then dv from the dout (dm) rows in their place ----
    store_split<NT>(work, dx, lane);
    wave_lds_sync();
    mma_rows<D, NT, 3>(ok, work, 128 * NT, rows, lane);
    wave_lds_sync();
    store_split<NT>(work, vw, lane);
#pragma unroll
    for (int p = 0; p < DP; ++p) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                *(lds_ptr<u32x4_t>)(rows + t * TS + j * 1024 + lane * 16) = __builtin_bit_cast(u32x4_t, term(t, j, p));
        wave_lds_sync();
        if (p == 0) mma_rows<D, NT, 3>(ov, work, 128 * NT, rows, lane);
        else if (p == 1) mma_rows<D, NT, 2>(ov, work, 128 * NT, rows, lane);
        else mma_rows<D, NT, 1>(ov, work, 128 * NT, rows, lane);
        wave_lds_sync();                 // the rows are read before the next ones replace them
    }
}

// One chunk of a kept key's list: up to kKeyGroup parents, 16 at a time, only the tiles that hold parents (lists
// of a few are common). Longer chunks write fewer partial rows for bwd_key_reduce_kernel to add up, and spread
// long lists over fewer waves: chunks of 16, 32 and 64 parents measured 421, 397 and 410 us a backward
// (200x336, 2 x 32, K = 16, batch 2) and 200 to 201 (32 maps of 56x56, 1 x 64, K = 8).
template <int D, bool VA, bool FINEST>
__device__ __forceinline__ void key_chunk(const BwdLevelArgs& a, const int chunk, const int key, const int nch, int beg,
                                          int left, unsigned char* const base)
{
    constexpr int CT = D / 16;
    const int lane = threadIdx.x & 63, n16 = lane & 15, g = lane >> 4;
    KeyRows<D> kr;
    key_rows<D, FINEST>(a, key, kr);
    float4_t ok[CT], ov[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) ok[ct] = ov[ct] = float4_t{0.f, 0.f, 0.f, 0.f};
    while (left > 0) {                                        // uniform
        const int nent = min(left, kKeyChunk);
        if (nent > 8) key_part<D, 4, VA, FINEST>(a, kr, beg, nent, base, ok, ov);
        else if (nent > 4) key_part<D, 2, VA, FINEST>(a, kr, beg, nent, base, ok, ov);
        else key_part<D, 1, VA, FINEST>(a, kr, beg, nent, base, ok, ov);
        beg += kKeyChunk;
        left -= kKeyChunk;
    }
    const int ky = 2 * kr.Jy + (g >> 1), kx = 2 * kr.Jx + (g & 1);
    if (nch > 1) {
        // this chunk's rows; bwd_key_reduce_kernel adds up the key's chunks
        float* const pk = a.partial + ((static_cast<size_t>(chunk) * 4 + g) * 2) * D + n16;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            pk[16 * ct] = ok[ct][0];
            pk[D + 16 * ct] = ov[ct][0];
        }
        return;
    }
    const bool on = ky < a.H && kx < a.W;
    const size_t map0 = static_cast<size_t>(kr.b) * a.H * a.W * a.C + kr.h * D;
    const uint32_t at = static_cast<uint32_t>((min(ky, a.H - 1) * a.W + min(kx, a.W - 1)) * a.C);
    float rk[CT], rv[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        rk[ct] = a.scale * ok[ct][0];
        rv[ct] = ov[ct][0];
    }
    // J's own totals, level l+1's, go to its children in equal shares
    const float share = child_share(kr.Jy, kr.Jx, a.H, a.W);
    const size_t up = (static_cast<size_t>(kr.b) * a.Hp * a.Wp + kr.Jy * a.Wp + kr.Jx) * a.C + kr.h * D + n16;
    if (a.up_k) {                                             // uniform
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) rk[ct] += share * a.up_k[up + 16 * ct];
    }
    if (a.up_v) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) rv[ct] += share * a.up_v[up + 16 * ct];
    }
    store_row<D, FINEST>(a.dk, FINEST && a.out_bf16, map0, at, rk, on, lane);
    store_row<D, FINEST>(a.dv, FINEST && a.out_bf16, map0, at, rv, on, lane);
}

}  // namespace bwd16
}  // namespace qta

#endif
