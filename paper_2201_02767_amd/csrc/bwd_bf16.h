// The finer levels' backward passes for bf16 maps (step 2 of backward.hip), on the row tiles of bf16_tiles.h:
// the query pass of every finer level, and the finest level's key pass. backward.hip holds the fp32 forms and
// the coarser levels' key pass, with the derivation.
//
// Both passes contract fp32 weights (the logit gradients, the value weights) with bf16 rows. The weights are
// split exactly into three bf16 terms (8 + 8 + 8 bits), whose products with a bf16 row are exact in the
// MFMA's fp32 accumulator, so the sums are as accurate as on the fp32 MFMA at a sixth of its time.
//
// What bounds them, before -> now: the previous forms gathered with a lane per row (46 cycles of the L1 an
// instruction, see bf16_tiles.h) and read the rows back from LDS two bytes at a time, one fp32 4x4 MFMA per
// slot. Finest level, 200x336 maps, 2 x 32 channels, K = 16, batch 2: query pass 125 -> 98 us, key pass 147 -> 99;
// 32 maps of 56x56, 1 x 64, K = 8: query pass 50 -> 38, key pass 69 -> 35.
#ifndef QTA_BWD_BF16_H
#define QTA_BWD_BF16_H

#include "bf16_tiles.h"
#include "qta_internal.h"

namespace qta {
namespace bwd16 {

using namespace tiles;

// x split into three bf16 terms: x = hi + mid + lo exactly (24 significant bits), two values a word.
struct Split2 {
    uint32_t hi, mid, lo;
};
__device__ __forceinline__ float low_half(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float high_half(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }
__device__ __forceinline__ Split2 split2(float x, float y)
{
    Split2 s;
    s.hi = pack2(x, y);
    x -= low_half(s.hi);
    y -= high_half(s.hi);
    s.mid = pack2(x, y);
    s.lo = pack2(x - low_half(s.mid), y - high_half(s.mid));
    return s;
}

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
        o = ok ? o : 0u;                                      // a missing candidate reads the map's first row
        flat = ok ? flat : -1;
        okm = __ballot(ok);
        quad_offsets<NT>(o, gather_chunk(lane), off);
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

    // ---- dq = scale * sum_s dx_s k_s ----
    store_split<NT>(work, dx, lane);
    wave_lds_sync();
    {
        float4_t o[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) o[ct] = float4_t{0.f, 0.f, 0.f, 0.f};
        mma_rows<D, NT, 3>(o, work, 128 * NT, klds, lane);
        if (qv) {
            float* const dq_b = a.dq + static_cast<size_t>(b) * N * C + h * D;
            const uint32_t at = (qpos * static_cast<uint32_t>(C) + n16) * 4u;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) store_at<float>(dq_b, at + 64 * ct, a.scale * o[ct][0]);
        }
    }

    // ---- level 0: the combination's backward. The four queries share one ancestor at every level j >= 1 (at
    //      j = 1 it is P itself): dm^j receives sum_r w_{r,j} dout_r, written at j = 1 and added with atomics
    //      above, and dw_{r,j} = <dout_r, m^j>. Four levels at a time: the fp32 MFMA sums over the queries
    //      (operand lane 16g + n: w of query g at level n >> 2, and dout of query g at channel n), so that
    //      lane group g ends with its level's sums; for dw, lane group g's messages go to all groups. ----
    if constexpr (FINEST) {
        const int L = a.levels;
        const bool want_dw = !VA && a.w && a.dw;              // uniform
        float dv[CT];                                         // dout of query g, zero off the map
        {
            const unsigned char* db = static_cast<const unsigned char*>(a.dout) + (static_cast<size_t>(b) * N * C + h * D) * 2;
            const uint32_t at = __umul24(qpos, tok_bytes) + static_cast<uint32_t>(n16 * 2);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) dv[ct] = qv ? bf16_bits_to_f32(load_at<uint16_t>(db, at + 32 * ct)) : 0.f;
        }
        if (want_dw && n16 == 0 && qv) store_at<float>(a.dw + wq_off, wrow * 4u, dw0);
        for (int l0 = 1; l0 < L; l0 += 4) {                   // uniform
            const int wlev = l0 + (n16 >> 2);                 // this lane's level as an operand row
            float wl = VA ? 1.f : 1.0f / L;
            if constexpr (!VA) {
                if (a.w) wl = load_at<float>(a.w + wq_off, (wrow + min(wlev, L - 1)) * 4u);   // uniform
            }
            // lane group g's level: the ancestor's row in its dm and in the forward's message
            const int lev = min(l0 + g, L - 1);
            const size_t arow = static_cast<size_t>(b) * a.lvl_N[lev] +
                                static_cast<size_t>((2 * Py) >> lev) * a.lvl_W[lev] + ((2 * Px) >> lev);
            const size_t at = (arow * a.heads + h) * D + n16;
            float mm[CT];
            if (want_dw) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) mm[ct] = a.msg_fwd[lev][at + 16 * ct];
            }
            float4_t s[CT];
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                s[ct] = float4_t{0.f, 0.f, 0.f, 0.f};
                s[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(wl, dv[ct], s[ct], 0, 0, 0);
            }
            if (l0 + g < L) {
                float* const dst = a.dm_out[lev] + at;
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    if (lev == 1) dst[16 * ct] = s[ct][0];
                    else unsafeAtomicAdd(dst + 16 * ct, s[ct][0]);
                }
            }
            if (want_dw) {
                float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const auto hf = __builtin_amdgcn_permlane32_swap(__float_as_uint(mm[ct]), __float_as_uint(mm[ct]), false, false);
                    const auto lo = __builtin_amdgcn_permlane16_swap(hf[0], hf[0], false, false);
                    const auto hi = __builtin_amdgcn_permlane16_swap(hf[1], hf[1], false, false);
                    part[0] += dv[ct] * __uint_as_float(lo[0]);
                    part[1] += dv[ct] * __uint_as_float(lo[1]);
                    part[2] += dv[ct] * __uint_as_float(hi[0]);
                    part[3] += dv[ct] * __uint_as_float(hi[1]);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) part[j] = row_allreduce(part[j], [](float p, float q) { return p + q; });
                const float mine = n16 == 0 ? part[0] : n16 == 1 ? part[1] : n16 == 2 ? part[2] : part[3];
                if (n16 < 4 && l0 + n16 < L && qv) store_at<float>(a.dw + wq_off, (wrow + l0 + n16) * 4u, mine);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// key pass of the finest level
// ---------------------------------------------------------------------------------------------

// One chunk of one kept key J's parent list (up to kKeyChunk = 16 parents, NT = 1, 2 or 4 tiles of four):
// slot s = 4e + child is a child of parent e, and vector g one of J's four children (the keys). Roles as in
// the query pass with queries and keys exchanged: logits and <dout, v> from the gathered query and dout rows,
// then dk = scale dx^T Q and dv = vw^T dout with the rows in LDS, the query rows first.
template <int D, int NT, bool VA>
__device__ __forceinline__ void key_chunk(const BwdLevelArgs& a, const int chunk, const int key, const int first, const int nch,
                                          const int beg, const int nent, unsigned char* const base)
{
    constexpr int RB = D * 2;
    constexpr int NJ = RB / 64;
    constexpr int CT = D / 16;
    constexpr int TS = tile_bytes<D>();
    const int lane = threadIdx.x & 63, n16 = lane & 15, g = lane >> 4;
    lds_byte* const rows = (lds_byte*)base;
    lds_byte* const work = rows + NT * TS;
    const int Np = a.Hp * a.Wp;
    const int bh = fast_div(key, a.div_Np), J = key - bh * Np;
    const int b = fast_div(bh, a.div_heads), h = bh - b * a.heads;
    const int H = a.H, W = a.W, C = a.C, N = H * W, K = a.Kp;
    const int Jy = fast_div(J, a.div_Wp), Jx = J - Jy * a.Wp;
    const uint32_t tok_bytes = static_cast<uint32_t>(C * 2);
    const size_t map0 = (static_cast<size_t>(b) * N * C + h * D) * 2;

    // ---- the slot this lane addresses: child (own & 3) of parent own >> 2 of the chunk (the children of a
    //      parent on neighbouring quads), its row, its query's statistics and w_0 ----
    const int own = 16 * (lane & 3) + (lane >> 2);
    const int ent = load_at<int32_t>(a.entries + beg, static_cast<uint32_t>(min(own >> 2, max(nent - 1, 0))) * 4u);
    // the four keys: MFMA operand row n16 holds key n16 >> 2, rows clamped onto the map
    bf16x8_t ka[NJ], va[NJ];
    {
        const int c = n16 >> 2;
        const uint32_t tok = static_cast<uint32_t>(__mul24(min(2 * Jy + (c >> 1), H - 1), W) + min(2 * Jx + (c & 1), W - 1));
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t at = __umul24(tok, tok_bytes) + static_cast<uint32_t>((g + 4 * j) * 16);
            ka[j] = __builtin_bit_cast(bf16x8_t, load_at<uint4>(static_cast<const unsigned char*>(a.k) + map0, at));
            va[j] = __builtin_bit_cast(bf16x8_t, load_at<uint4>(static_cast<const unsigned char*>(a.v) + map0, at));
        }
    }
    const int Pc = nent > 0 ? ent : 0;
    const int P = fast_div(Pc, a.div_Kp), r = Pc - P * K;
    const int Py = fast_div(P, a.div_Wp), Px = P - Py * a.Wp;
    const int qy = 2 * Py + ((own >> 1) & 1), qx = 2 * Px + (own & 1);
    const bool qv = (own >> 2) < nent && qy < H && qx < W;
    const uint32_t qtok = static_cast<uint32_t>(__mul24(min(qy, H - 1), W) + min(qx, W - 1));
    const uint64_t okm = __ballot(qv);                        // bit 4n + t: slot 16t + n holds a query
    uint32_t off[NT];
    quad_offsets<NT>(__umul24(qtok, tok_bytes), gather_chunk(lane), off);
    const unsigned char* const dbase = static_cast<const unsigned char*>(a.dout) + map0;
    const __amdgpu_buffer_rsrc_t qres = map_resource(static_cast<const unsigned char*>(a.q) + map0);
    uint4 dc[NT][NJ];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < NJ; ++j) dc[t][j] = load_at<uint4>(dbase, off[t] + 64 * j);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < NJ; ++j) load_lds16(qres, off[t], 64 * j, rows + t * TS + j * 1024);
    const float* const st_b = a.stats + static_cast<size_t>(bh) * static_cast<uint32_t>(N * 2 * (VA ? K : 1));
    const float2_t st = load_at<float2_t>(st_b, (VA ? qtok * static_cast<uint32_t>(K) + r : qtok) * 8u);
    float scale_w = 1.0f;                                     // B: w_0 of the slot's query; A: the parent's score
    if constexpr (VA) scale_w = a.parent_key[(static_cast<size_t>(bh) * Np + P) * K + r];
    else scale_w = a.w ? load_at<float>(a.w + static_cast<size_t>(b) * static_cast<uint32_t>(N * a.heads * a.levels),
                                        (qtok * static_cast<uint32_t>(a.heads) + h) * static_cast<uint32_t>(a.levels) * 4u)
                       : 1.0f / a.levels;

    // ---- <dout, v> and logits: lane 16g + n holds key g's of slots 16t + n ----
    float gs[NT], x[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        float4_t ag = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            ag = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[j], pass_operand(dc[t][j], work, lane), ag, 0, 0, 0);
        gs[t] = ag[0];
    }
    wait_lds_loads();                                         // the query rows
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        float4_t ax = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            ax = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[j], tile_operand(rows + t * TS + j * 1024, lane), ax, 0, 0, 0);
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
        const float sw = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(scale_w)));
        const bool valid = key_ok && ((okm >> (4 * n16 + t)) & 1ull) != 0ull;
        const float pr = valid ? __expf(x[t] * a.scale - lse) : 0.f;      // B: p; A: t
        vw[t] = sw * pr;                                                  // B: w_0 p (the dout rows come without w_0); A: s
        dx[t] = VA ? vw[t] * (gs[t] - Dq) : pr * (sw * gs[t] - Dq);
    }

    // ---- dk from the query rows, then dv from the dout rows in their place ----
    float4_t ok[CT], ov[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) ok[ct] = ov[ct] = float4_t{0.f, 0.f, 0.f, 0.f};
    store_split<NT>(work, dx, lane);
    wave_lds_sync();
    mma_rows<D, NT, 3>(ok, work, 128 * NT, rows, lane);
    wave_lds_sync();
    store_split<NT>(work, vw, lane);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            *(lds_ptr<u32x4_t>)(rows + t * TS + j * 1024 + lane * 16) = __builtin_bit_cast(u32x4_t, dc[t][j]);
    wave_lds_sync();
    mma_rows<D, NT, 3>(ov, work, 128 * NT, rows, lane);

    if (nch > 1) {
        // this chunk's rows; bwd_key_reduce_kernel adds up the key's chunks
        float* const pk = a.partial + ((static_cast<size_t>(chunk) * 4 + g) * 2) * D + n16;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            pk[16 * ct] = ok[ct][0];
            pk[D + 16 * ct] = ov[ct][0];
        }
    } else if (key_ok) {
        const size_t row = (static_cast<size_t>(b) * N + ky * W + kx) * C + h * D + n16;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            a.dk[row + 16 * ct] = a.scale * ok[ct][0];
            a.dv[row + 16 * ct] = ov[ct][0];
        }
    }
}

}  // namespace bwd16
}  // namespace qta

#endif
