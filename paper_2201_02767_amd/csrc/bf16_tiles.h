// Row tiles of bf16 maps in LDS, shared by the fine kernels' forward and backward forms.
//
// A wave works on slots in NT tiles of 16 (NT = 1, 2, 4, 8 or 16), each slot a row of D channels somewhere in
// a map. Rows come in by gathers in which lanes 4n .. 4n+3 take the four 16-byte chunks (per 64 bytes) of
// tile row n, lane l chunk (l & 3) ^ (n >> 2): four neighbouring lanes on one row cost a CU 19 (L1) to 39 (L2)
// cycles an instruction, a lane per row 46 to 64. They land in LDS (straight from memory, or from registers) in lane
// order, as [tile][D / 32][16 rows][4 places] chunks, place p of row n holding chunk p ^ (n >> 2). From there
//   - tile_operand reads MFMA operand lanes (16g + n: chunk g of row n) without bank conflicts,
//   - mma_rows contracts over the slots: weights [4 vectors][16][NT] times the rows, read transposed.
#ifndef QTA_BF16_TILES_H
#define QTA_BF16_TILES_H

#include "qta_device.h"

namespace qta {
namespace tiles {

typedef float float4_t __attribute__((ext_vector_type(4)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef short short8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) unsigned char lds_byte;
template <typename T> using lds_ptr = __attribute__((address_space(3))) T*;

// Bytes from one tile's rows to the next in LDS: 32 past a multiple of the 256 bytes of the banks, so that the
// 64 eight-byte pieces of a transposed read (four 16-lane groups, 64 bytes apart; four slots, mostly of four
// tiles) fall on every bank twice, the least for 512 bytes.
template <int D>
constexpr int tile_bytes() { return 32 * D + 32; }

// Two floats as packed bf16 (round to nearest, ties to even).
__device__ __forceinline__ uint32_t pack2(float lo, float hi)
{
    const float2_t f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
}

// x split into three bf16 terms: x = hi + mid + lo exactly (24 significant bits), two values a word. x finite, as
// the entry points ask: an infinity, or a value that rounds to one in bf16 (3.39e38 on), gives NaN in the sums.
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

// The value that lane T of each lane quad holds, in all four lanes.
template <int T>
__device__ __forceinline__ uint32_t quad_broadcast(uint32_t x)
{
    return __builtin_amdgcn_update_dpp(0u, x, T * 0x55, 0xF, 0xF, false);
}

// Lane 4n + t of each quad holds tile t's slot n: out[t] gets it in the quad's four lanes, plus `add`.
template <int N>
__device__ __forceinline__ void quad_offsets(uint32_t x, uint32_t add, uint32_t* out)
{
    out[0] = quad_broadcast<0>(x) + add;
    if constexpr (N > 1) out[1] = quad_broadcast<1>(x) + add;
    if constexpr (N > 2) {
        out[2] = quad_broadcast<2>(x) + add;
        out[3] = quad_broadcast<3>(x) + add;
    }
}

// This lane's chunk of its quad's row, in bytes.
__device__ __forceinline__ uint32_t gather_chunk(int lane) { return static_cast<uint32_t>(((lane & 3) ^ (lane >> 4)) * 16); }

// A buffer descriptor of a map from `base` (wave-uniform) on: raw bytes, offsets below 2^31.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t map_resource(const unsigned char* base)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(base), 0, 0x7FFFFFFF, 0x00020000);
}

// 16 bytes a lane from the map to LDS, lane i's at dst + 16 i (dst wave-uniform). The buffer form: with a
// global one in flight the compiler waits for every load wherever it needs any of them. See wait_lds_loads.
__device__ __forceinline__ void load_lds16(__amdgpu_buffer_rsrc_t map, uint32_t off, int more, lds_byte* dst)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(map, (__attribute__((address_space(3))) void*)dst, 16,
                                             static_cast<int>(off) + more, 0, 0, 0);
}

// Waits until every load_lds16 of this wave has landed: to stand before the first read of what they bring (the
// compiler counts the loads, but does not hold plain LDS reads back for them).
__device__ __forceinline__ void wait_lds_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The operand lanes of 1 KB of gathered chunks at `rows`: lane 16g + n gets chunk g of row n.
__device__ __forceinline__ bf16x8_t tile_operand(lds_byte* rows, int lane)
{
    const int n = lane & 15, g = lane >> 4;
    return __builtin_bit_cast(bf16x8_t, *(lds_ptr<u32x4_t>)(rows + n * 64 + ((g ^ (n >> 2)) * 16)));
}

// The same for chunks in registers, passed through 1 KB of LDS. A wave's LDS accesses complete in order, so
// the next chunks may overwrite these at once: only the compiler has to keep the order.
__device__ __forceinline__ bf16x8_t pass_operand(const uint4& chunk, lds_byte* stage, int lane)
{
    *(lds_ptr<u32x4_t>)(stage + lane * 16) = __builtin_bit_cast(u32x4_t, chunk);
    asm volatile("" ::: "memory");
    const bf16x8_t r = tile_operand(stage, lane);
    asm volatile("" ::: "memory");
    return r;
}

// Where lane 16g + n's NT weights (of vector g, slots 16t + n) go, in units of NT: the order of the
// contraction. It makes the lane groups of a transposed read take rows 64 bytes apart.
template <int NT>
__device__ __forceinline__ int weight_place(int n)
{
    return NT == 4 ? ((n & 8) | ((n & 3) << 1) | ((n >> 2) & 1))
         : NT == 2 ? (((n & 3) << 2) | ((n >> 3) << 1) | ((n >> 2) & 1)) : n;
}

// Stores lane 16g + n's weights of vector g as bf16 at `w` ([4][16][NT]).
template <int NT>
__device__ __forceinline__ void store_weights(lds_byte* w, const float (&x)[NT], int lane)
{
    lds_byte* const p = w + ((lane >> 4) * 16 + weight_place<NT>(lane & 15)) * NT * 2;
    if constexpr (NT == 1) {
        *(lds_ptr<uint16_t>)p = static_cast<uint16_t>(pack2(x[0], 0.f));
    } else if constexpr (NT == 2) {
        *(lds_ptr<uint32_t>)p = pack2(x[0], x[1]);
    } else {
#pragma unroll
        for (int t = 0; t < NT; t += 4)
            *(lds_ptr<u32x2_t>)(p + t * 2) = u32x2_t{pack2(x[t], x[t + 1]), pack2(x[t + 2], x[t + 3])};
    }
}

// Four tiles (64 slots) read transposed: channel tile ct of the eight slots of lane group g at step u (0 or 1),
// n = g + 4 (2u + r), t = 0 .. 3 for r = 0, 1 (see mma_rows), as an MFMA operand.
template <int D>
__device__ __forceinline__ bf16x8_t rows_transposed4(lds_byte* rows, int u, int ct, int lane)
{
    constexpr int TS = tile_bytes<D>();
    const int n16 = lane & 15, g = lane >> 4, k = n16 >> 2, c2 = (n16 >> 1) & 1;
    lds_byte* const r0 = rows + k * TS + g * 64 + (n16 & 1) * 8;
    short4_t v[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int x = 2 * u + r;
        v[r] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            reinterpret_cast<lds_ptr<short4_t>>(r0 + ((c2 ^ x ^ (2 * (ct & 1))) * 16) + (ct >> 1) * 1024 + 256 * x));
    }
    return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(v[0], v[1], 0, 1, 2, 3, 4, 5, 6, 7));
}

// acc[ct] += weights x rows on the 16x16 MFMA, contracted over the 16 NT slots: operand rows 4g .. 4g+3 are
// vector g's weights, column n of channel tile ct is channel 16 ct + n, so lane 16g + n ends with vector g's
// product at its channel in every element of acc[ct]. PLANES weight arrays, plane_bytes apart, are summed
// (fp32 weights as exact sums of three bf16 ones).
template <int D, int NT, int PLANES>
__device__ __forceinline__ void mma_rows(float4_t (&acc)[D / 16], lds_byte* weights, int plane_bytes, lds_byte* rows, int lane)
{
    constexpr int TS = tile_bytes<D>();
    const int n16 = lane & 15, g = lane >> 4;
    // Contraction index i = place(n) * NT + t, 32 per MFMA (16 with one tile); lane group g takes the eight
    // (four) from 32u + 8g (4g), a transposed read four of them: lane i of the group reads eight bytes of row
    // (index) k = i >> 2, half i & 1 of chunk 2ct + (i >> 1 & 1). The slots of a read:
    //   NT = 1:  n = 4g + k                          NT = 2:  n = g + 4 (k >> 1) + 8r, t = k & 1
    //   NT = 4:  n = g + 4 (2u + r), t = k           NT = 8:  n = g + 4u, t = k + 4r
    //   NT = 16: n = 2u + (g >> 1), t = 8 (g & 1) + k + 4r
    const int k = n16 >> 2, c2 = (n16 >> 1) & 1;
    const int row_at = NT == 1 ? (4 * g + k) * 64 : NT == 2 ? (k & 1) * TS + (g + 4 * (k >> 1)) * 64
                     : NT == 16 ? (8 * (g & 1) + k) * TS + (g >> 1) * 64 : k * TS + g * 64;
    const int swz = NT == 1 ? c2 ^ g : NT == 2 ? c2 ^ (k >> 1) : c2;     // the lane's part of the place
    lds_byte* const r0 = rows + row_at + (n16 & 1) * 8;
    // channel tile ct of rows `at` bytes on, where the rest of the place's n >> 2 is x (a constant)
    auto read = [&](int ct, int x, int at) -> short4_t {
        lds_byte* p = r0 + ((swz ^ x ^ (2 * (ct & 1))) * 16) + (ct >> 1) * 1024 + at;
        return __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_ptr<short4_t>>(p));
    };
    lds_byte* const w0 = weights + ((n16 >> 2) * 16 * NT + (NT == 1 ? 4 : 8) * g) * 2;
    if constexpr (NT == 1) {
        short4_t w[PLANES];
#pragma unroll
        for (int p = 0; p < PLANES; ++p) w[p] = *(lds_ptr<short4_t>)(w0 + p * plane_bytes);
#pragma unroll
        for (int ct = 0; ct < D / 16; ++ct) {
            const short4_t v = read(ct, 0, 0);
#pragma unroll
            for (int p = 0; p < PLANES; ++p) acc[ct] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w[p], v, acc[ct], 0, 0, 0);
        }
    } else {
#pragma unroll
        for (int u = 0; u < NT / 2; ++u) {
            short8_t w[PLANES];
#pragma unroll
            for (int p = 0; p < PLANES; ++p) w[p] = *(lds_ptr<short8_t>)(w0 + p * plane_bytes + u * 64);
#pragma unroll
            for (int ct = 0; ct < D / 16; ++ct) {
                short4_t v[2];
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    if constexpr (NT == 2) v[r] = read(ct, 2 * r, 512 * r);
                    else if constexpr (NT == 4) v[r] = read(ct, 2 * u + r, 256 * (2 * u + r));
                    else if constexpr (NT == 8) v[r] = read(ct, u, 256 * u + 4 * r * TS);
                    else v[r] = read(ct, u >> 1, 128 * u + 4 * r * TS);
                }
                const short8_t vv = __builtin_shufflevector(v[0], v[1], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                for (int p = 0; p < PLANES; ++p)
                    acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w[p]),
                                                                      __builtin_bit_cast(bf16x8_t, vv), acc[ct], 0, 0, 0);
            }
        }
    }
}

}  // namespace tiles
}  // namespace qta

#endif
