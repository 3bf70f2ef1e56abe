// Steps 2-3 at the coarsest level: full softmax attention, Eq. (1), plus each query's top-K keys.
//
// One workgroup of Q waves (Q = 8 or 16) owns a tile of Q queries of one (batch, head):
//   phase 1  logits S = tau * Q_tile K^T on MFMA (16x16 output tiles whose rows repeat the Q
//            queries when Q < 16; waves take key tiles in turn, a batch of loads at a time), kept
//            in LDS as fp32 [Q][N];
//   phase 2  wave r owns query row r: max, exp and sum over the row (register butterflies), then
//            the K best keys by a bitwise radix select on wave ballots among the few keys that reach
//            a bound on the K-th (ties at the cut go to the lower index), listed in index order;
//            QuadTree-A zeroes the kept keys' weights (their mass is refined at the next level);
//   phase 3  m = P V on MFMA. fp32: two batches of loads in flight, waves split the d columns into
//            16-wide tiles and the keys into chunks. bf16: a wave takes 64 keys, brought to LDS
//            during phase 2, with the weights as three bf16 terms. Partial tiles are summed
//            through LDS and written as fp32 messages (or, for a single-level problem, straight
//            to the output in the storage type).
// What bounds it: instruction issue of phase 2 at these sizes (a row is 1 KB to 4 KB of LDS, a map's
// keys and values stay in L2). Measured on MI355X, bf16 unless said: 8 heads x 1023 keys, d = 32, K = 16:
// 84 us with the selection over all values of a lane, the values widened one by one and 8 rows, now 49; 8 x 4
// maps of 300 keys 12.6 to 10.4; d = 64, 196 keys: 13.3 to 12.4; fp32, 300 keys: 11.8 to 11.1.
// The coarsest map holds at most QTA_MAX_COARSE tokens, so a row fits in 16 registers per lane.
// Maps of at most 64 tokens take coarse_small_kernel instead (one wave per query row).
#include <type_traits>
#include <utility>

#include "bf16_tiles.h"
#include "qta_internal.h"

namespace qta {

namespace {

using tiles::bf16x8_t;
using tiles::float4_t;


// LDS pitch of a logit row: whole 64-element groups plus 4 floats, so the 16 rows that one MFMA
// operand read touches fall in different banks.
__host__ __device__ inline int coarse_pitch(int N) { return (N + 63) / 64 * 64 + 4; }

// Row elements per lane: ceil(N / 64) rounded up to the next instantiated count (a template
// parameter, so the selection loops carry no bounds checks and no empty slots for common sizes).
inline int coarse_per_lane(int N)
{
    const int need = (N + kWave - 1) / kWave;
    static const int counts[] = {1, 2, 3, 4, 5, 6, 8, 12, 16};
    for (int c : counts)
        if (need <= c) return c;
    return 0;
}

// bf16, behind the logit rows: 1 KB per wave for key chunks in passing; after the logits, a buffer for each wave
// that has keys in the message product (64 at a time, 32 channels of their value rows), then its partial
// messages [D / 16][16][16].
constexpr int kCoarseBuffer = 4 * tiles::tile_bytes<32>();
__host__ __device__ inline int coarse_behind(int N, int Q)
{
    const int chunks = (N + kWave - 1) / kWave, bufs = (chunks < Q ? chunks : Q) * kCoarseBuffer;
    return bufs > Q * 1024 ? bufs : Q * 1024;
}

// Waves per SIMD the kernel's registers must leave room for, so that two workgroups of 16 rows share a CU: up to
// six values a lane everything fits 64 vector registers without a spill, and the figure also holds the scalar
// registers under their limit, which the selection's masks would pass (bf16, d = 64, 400 workgroups of 196 keys:
// 15.6 us without it, 12.4 with it). Not fp32 with d = 64 and five or six values, where 64 would spill, nor with
// four, which fit without and are 2% slower with it, nor more.
template <typename T, int D, int kPerLane>
constexpr int coarse_waves()
{
    return kPerLane <= (sizeof(T) == 4 && D == 64 ? 3 : 6) ? 8 : 4;
}

// The largest K for which phase 2 searches among the survivors of a bound (0: never). The bound costs a search of one
// value a lane, and keeps out the less the larger K is: of 64 groups' maxima the K-th is reached by 18 keys for
// K = 16, 44 for 32, 63 for 40, and more than 64 survivors fall back on all values. QuadTree-A also clears the
// kept weights by a second pass over the values. Measured with the bound over without (16 and 64 maps, bf16; fp32
// lies closer to 1): B, 15x17 keys: K = 8 0.97, 16 1.01; 18x21: 16 0.98, 24 1.02; 21x23: 16 0.89, 32 0.95, 44 1.03;
// 28x27: 16 0.83, 40 0.98, 44 1.05; 29x31: 16 0.77, 32 0.93, 40 1.05. A: 15x17 K = 8 1.04; 18x21 K = 4 0.98;
// 21x23 K = 8 0.97, 16 1.02; 28x27 K = 32 0.96; 31x33 K = 24 0.92, 32 1.02.
template <typename T, int D, bool VA, int kPerLane>
constexpr int bound_max_k()
{
    if (VA) return kPerLane >= 12 ? 32 : kPerLane == 8 ? 16 : kPerLane >= 5 ? 8 : 0;
    // (fp32 with d = 64 and four values: the survivors' code takes it past the 64 registers of two workgroups)
    if (kPerLane == 4) return sizeof(T) == 4 && D == 64 ? 0 : 12;
    return kPerLane == 12 ? 40 : kPerLane >= 8 ? 32 : kPerLane >= 5 ? 20 : 0;
}

// x of another lane of the 16-lane row, R lanes on.
template <int R>
__device__ __forceinline__ uint32_t row_rotated(uint32_t x)
{
    if constexpr (R == 0) return x;
    else return __builtin_amdgcn_update_dpp(0u, x, kDppRowRor + R, 0xF, 0xF, false);
}

// Whether a map's keys 64 on are its neighbours (at most two tokens away: maps 32 and 63 to 65 wide). A lane's keys
// are then alike in a smooth image, the best ones lie in few lanes, and a bound of the lanes' maxima is too low
// (64 and 32 wide: 1.06 and 1.04 of the time without it at K = 20 and 28; with the groups below 1.0 and 0.99).
inline bool lane_keys_near(int W)
{
    const int dy = (kWave + W / 2) / W, dx = kWave - dy * W;
    return dx * dx + dy * dy <= 4;
}

// The largest key of each of 64 groups, one a lane: key e of every lane belongs to the group of another lane of its
// row, which parts a map's columns where lane_keys_near.
template <int... E>
__device__ __forceinline__ uint32_t group_maxima(const uint32_t (&key)[sizeof...(E)], std::integer_sequence<int, E...>)
{
    constexpr int kRotation[16] = {0, 7, 3, 12, 9, 1, 14, 6, 11, 4, 15, 8, 2, 13, 5, 10};    // no common step
    uint32_t top = 0u;
    ((top = max(top, row_rotated<kRotation[E]>(key[E]))), ...);
    return top;
}

template <typename T, int D, bool VA, int kPerLane, int Q>
__global__ __launch_bounds__(Q * kWave) __attribute__((amdgpu_waves_per_eu(coarse_waves<T, D, kPerLane>()))) void coarse_attn_kernel(CoarseArgs a)
{
    using S = Storage<T>;
    constexpr bool kBf16 = sizeof(T) == 2;
    constexpr int kWaves = Q;                      // one wave per query row in phase 2
    static_assert(Q == 8 || Q == 16, "8 or 16 query rows per workgroup");
    extern __shared__ __align__(16) float smem[];
    const int N = a.N, C = a.C, pitch = coarse_pitch(N);
    float* Sm = smem;                              // [Q][pitch]
    float* red = smem + Q * pitch;                 // fp32: [waves][16][16]
    tiles::lds_byte* const stage = (tiles::lds_byte*)red + (threadIdx.x >> 6) * 1024;             // bf16
    tiles::lds_byte* const buf = (tiles::lds_byte*)red + (threadIdx.x >> 6) * kCoarseBuffer;
    const int qtiles = (N + Q - 1) / Q;            // query tiles of this map
    const int ktiles = (N + 15) / 16;              // 16-key tiles
    int blk = blockIdx.x;
    const int tile = blk % qtiles;
    blk /= qtiles;
    const int h = blk % a.heads;
    const int b = blk / a.heads;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const size_t tok0 = static_cast<size_t>(b) * N;           // first token of this batch element
    const size_t hoff = static_cast<size_t>(h) * D;
    // this map's rows as wave-uniform bases; a row's offset from them, below N * C elements
    // (N <= 1024 and C <= 2^20, so under 2^32 bytes), is a 32-bit lane offset
    const size_t map0 = tok0 * C + hoff;
    const unsigned char* qmap = static_cast<const unsigned char*>(a.q) + map0 * sizeof(T);
    const unsigned char* kmap = static_cast<const unsigned char*>(a.k) + map0 * sizeof(T);
    const unsigned char* vmap = static_cast<const unsigned char*>(a.v) + map0 * sizeof(T);
    const uint32_t row_bytes = static_cast<uint32_t>(C) * sizeof(T);   // <= 2^22

    // V operands of phase 3's first two key batches, requested after the logits' operands so that
    // their latency overlaps the logits and the selection (phase 3 layout: lane (kgrp, col) holds
    // V[4*step + kgrp][16*ct + col])
    constexpr int NCT = D / 16;          // 16-wide column tiles of the messages
    constexpr int NKS = kWaves / NCT;    // key chunks
    static_assert(NKS >= 1, "at least one wave per column tile");
    constexpr int kVBatch = 8;           // key steps per V batch
    const int p3_ct = wave % NCT, p3_ks = wave / NCT;
    const int p3_ch = p3_ct * 16 + (lane & 15);
    const int steps = (N + 3) / 4;
    float vb[kBf16 ? 1 : kVBatch], vb2[kBf16 ? 1 : kVBatch];
    auto load_v = [&](int st0, float (&dst)[kBf16 ? 1 : kVBatch]) {
#pragma unroll
        for (int u = 0; u < (kBf16 ? 0 : kVBatch); ++u) {
            const int cand = min((st0 + u * NKS) * 4 + (lane >> 4), N - 1);    // clamped; weight 0 beyond N
            dst[u] = S::load1_at(vmap, __umul24(static_cast<uint32_t>(cand), static_cast<uint32_t>(C)) + p3_ch);
        }
    };

    // ---- phase 1: logits on MFMA; a wave takes key tiles wave, wave + waves, ..., a batch at a time ----
    // The 16 rows of an MFMA tile hold the workgroup's Q query rows (repeated when Q < 16; only the
    // first Q are kept). The contraction over the d channels is taken in a permuted order so that each
    // lane loads whole 16-byte chunks of its query or key row: lane (kgrp, r) loads chunks kgrp,
    // kgrp+4, ... of row r and feeds their elements to consecutive k-steps; Q and K use the same
    // permutation.
    {
        const int arow = lane & 15, kgrp = lane >> 4;
        const int qi = min(tile * Q + (arow & (Q - 1)), N - 1);   // rows past N are computed and ignored
        constexpr int NJ = D * static_cast<int>(sizeof(T)) / 64;   // 16-byte chunks per lane and row
        // key tiles a wave takes (N <= 64 * kPerLane, so at most 4 * kPerLane tiles over Q waves),
        // loaded as one batch where that is at most four: no registers held for tiles no wave has
        constexpr int kTileBatch = (4 * kPerLane + Q - 1) / Q < 4 ? (4 * kPerLane + Q - 1) / Q : 4;
        uint4 qa[NJ];
        const uint32_t qoff = __umul24(static_cast<uint32_t>(qi), row_bytes) + kgrp * 16;
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) qa[jj] = load_at<uint4>(qmap, qoff + 64 * jj);
        bool first = true;
        for (int t0 = wave; t0 < ktiles; t0 += kWaves * kTileBatch) {             // uniform
            uint4 kb[kTileBatch][NJ];
#pragma unroll
            for (int it = 0; it < kTileBatch; ++it) {
                if (t0 + kWaves * it >= ktiles) break;                            // uniform
                // columns past N are set to -inf. bf16: four lanes per row (see bf16_tiles.h), moved to the
                // operand's lanes below
                const int n = min((t0 + kWaves * it) * 16 + (kBf16 ? lane >> 2 : arow), N - 1);
                const uint32_t koff = __umul24(static_cast<uint32_t>(n), row_bytes) +
                                      (kBf16 ? tiles::gather_chunk(lane) : static_cast<uint32_t>(kgrp * 16));
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj) kb[it][jj] = load_at<uint4>(kmap, koff + 64 * jj);
            }
            if (!kBf16 && first) {
                load_v(p3_ks, vb);
                load_v(p3_ks + NKS * kVBatch, vb2);
                first = false;
            }
#pragma unroll
            for (int it = 0; it < kTileBatch; ++it) {
                const int kt = t0 + kWaves * it;
                if (kt >= ktiles) break;
                float4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj) {
                    if constexpr (kBf16) {
                        // 8 bf16 per chunk: one k-step of 32 (eight channels per lane)
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, qa[jj]),
                                                                      tiles::pass_operand(kb[it][jj], stage, lane), acc, 0, 0, 0);
                    } else {
                        // 4 floats per chunk: four k-steps
                        const uint4 qq = qa[jj], kk = kb[it][jj];
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(qq.x), __uint_as_float(kk.x), acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(qq.y), __uint_as_float(kk.y), acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(qq.z), __uint_as_float(kk.z), acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(qq.w), __uint_as_float(kk.w), acc, 0, 0, 0);
                    }
                }
                const int n = kt * 16 + (lane & 15);
#pragma unroll
                for (int jr = 0; jr < 4; ++jr)
                    if (4 * kgrp + jr < Q) Sm[(4 * kgrp + jr) * pitch + n] = n < N ? acc[jr] * a.scale : -INFINITY;
            }
        }
        if (!kBf16 && first) {           // a wave with no key tile (more waves than tiles)
            load_v(p3_ks, vb);
            load_v(p3_ks + NKS * kVBatch, vb2);
        }
    }
    __syncthreads();

    // bf16: channels 32 jj .. of the value rows of 64 keys into the wave's buffer, the first of them now, so that
    // they arrive during the selection. Tile t's row n is key 32 (n >> 3) + 8 (n & 3) + 4 (n >> 2 & 1) + t:
    // the order in which a transposed read (bf16_tiles.h) hands lane group g keys 32u + 8g .. 32u + 8g + 7,
    // which are consecutive in a logit row.
    const int nchunk = (N + kWave - 1) / kWave;
    auto load_values = [&](int jj) {
        if constexpr (kBf16) {
            const __amdgpu_buffer_rsrc_t vres = tiles::map_resource(vmap);
            const int n = lane >> 2, key0 = wave * kWave + 32 * (n >> 3) + 8 * (n & 3) + 4 * ((n >> 2) & 1);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                tiles::load_lds16(vres, __umul24(static_cast<uint32_t>(min(key0 + t, N - 1)), row_bytes) + tiles::gather_chunk(lane) + 64 * jj,
                                  0, buf + t * tiles::tile_bytes<32>());
        }
    };
    if (kBf16 && wave < nchunk) load_values(0);

    // ---- phase 2: softmax and selection, one wave per query row ----
    {
        const int r = wave;
        const int qi = tile * Q + r;
        float* row = Sm + r * pitch;
        float x[kPerLane];
        float mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < kPerLane; ++e) {
            const int j = lane + kWave * e;
            x[e] = j < N ? row[j] : -INFINITY;
            mx = fmaxf(mx, x[e]);
        }
        mx = wave_max_fast(mx);
        float p[kPerLane];
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < kPerLane; ++e) {
            const int j = lane + kWave * e;
            p[e] = j < N ? __expf(x[e] - mx) : 0.f;
            sum += p[e];
        }
        const float inv = 1.0f / wave_sum_fast(sum);
#pragma unroll
        for (int e = 0; e < kPerLane; ++e) p[e] *= inv;

        if (a.K > 0 && qi < N) {
            // the K best keys by logit (ties to the lower index), listed in index order
            uint32_t key[kPerLane];
#pragma unroll
            for (int e = 0; e < kPerLane; ++e) key[e] = lane + kWave * e < N ? ordered_bits(x[e]) : 0u;
            const int keff = a.K < N ? a.K : N;
            int32_t* const so = a.sel_idx + ((static_cast<size_t>(b) * a.heads + h) * N + qi) * a.K;
            float* const ko = a.sel_key + ((static_cast<size_t>(b) * a.heads + h) * N + qi) * a.K;
            // Up to kBoundK (less where a lane's keys are alike; N > 64, so every group has a key): the K-th
            // largest of 64 groups' maxima bounds the K-th largest key from below, and the few keys at or above
            // it go to LDS (the row's logits are in registers) in index order, one a lane. The searches then test
            // one value a lane and bit, and the listing runs once instead of kPerLane times.
            constexpr int kBoundK = bound_max_k<T, D, VA, kPerLane>();
            int nsurv = kWave + 1;
            uint32_t low = 0u;
            if (kBoundK > 0 && keff <= (a.near ? kBoundK * 3 / 4 : kBoundK)) {       // uniform
                uint32_t top[1] = {0u};
                if (a.near) {
                    top[0] = group_maxima(key, std::make_integer_sequence<int, kPerLane>());
                } else {
#pragma unroll
                    for (int e = 0; e < kPerLane; ++e) top[0] = max(top[0], key[e]);
                }
                low = wave_cut<1>(top, keff);
                nsurv = 0;
#pragma unroll
                for (int e = 0; e < kPerLane; ++e) nsurv += __popcll(__ballot(key[e] >= low));
                nsurv = __builtin_amdgcn_readfirstlane(nsurv);
            }
            if (kBoundK > 0 && nsurv <= kWave) {             // uniform
                int before = 0;
#pragma unroll
                for (int e = 0; e < kPerLane; ++e) {
                    const uint64_t mask = __ballot(key[e] >= low);
                    if (key[e] >= low) {
                        const int pos = before + lanes_below(mask);
                        row[pos] = __uint_as_float(key[e]);
                        row[kWave + pos] = __uint_as_float(static_cast<uint32_t>(lane + kWave * e));
                    }
                    before += __popcll(mask);
                }
                wave_lds_sync();
                const uint32_t s[1] = {lane < nsurv ? __float_as_uint(row[lane]) : 0u};
                const uint32_t name = __float_as_uint(row[kWave + lane]);
                // (the search stops at any value that parts the keff best survivors from the rest; keys below the
                // bound must stay below the cut too)
                const uint32_t cut = max(wave_cut<1>(s, keff), low);
                const uint64_t above = __ballot(s[0] > cut), at = __ballot(s[0] == cut);
                const int need = keff - __popcll(above);     // places for keys at the cut, lowest index first
                const bool mine = s[0] > cut || (s[0] == cut && lanes_below(at) < need);
                const uint64_t mask = __ballot(mine);
                if (mine) {
                    const uint32_t pos = static_cast<uint32_t>(lanes_below(mask)) * 4u;
                    store_at<int32_t>(so, pos, static_cast<int32_t>(name));
                    store_at<float>(ko, pos, __expf(from_ordered_bits(s[0]) - mx) * inv);
                }
                if constexpr (VA) {                          // the kept keys are refined at the next level (Omega)
                    int ties = 0;
#pragma unroll
                    for (int e = 0; e < kPerLane; ++e) {
                        const uint64_t eq = __ballot(key[e] == cut);
                        if (key[e] > cut || (key[e] == cut && ties + lanes_below(eq) < need)) p[e] = 0.f;
                        ties += __popcll(eq);
                    }
                }
            } else {
                uint32_t name[kPerLane];
                bool kept[kPerLane];
#pragma unroll
                for (int e = 0; e < kPerLane; ++e) name[e] = static_cast<uint32_t>(lane + kWave * e);
                wave_select_top<kPerLane>(key, name, keff, kept);
                int before = 0;
#pragma unroll
                for (int e = 0; e < kPerLane; ++e) {
                    const uint64_t mask = __ballot(kept[e]);
                    if (kept[e]) {
                        const int pos = before + lanes_below(mask);
                        so[pos] = lane + kWave * e;
                        ko[pos] = p[e];
                        if constexpr (VA) p[e] = 0.f;        // refined at the next level (Omega)
                    }
                    before += __popcll(mask);
                }
            }
            if (lane >= keff && lane < a.K) {
                so[lane] = -1;
                ko[lane] = 0.f;
            }
        }
#pragma unroll
        for (int e = 0; e < kPerLane; ++e) {
            const int j = lane + kWave * e;
            if (j < pitch) row[j] = (j < N && qi < N) ? p[e] : 0.f;
        }
    }
    __syncthreads();

    // ---- phase 3: messages m = P V. fp32: on the fp32 MFMA; a wave takes key steps p3_ks, p3_ks + NKS, ... in
    // batches of kVBatch, two batches in flight. bf16: a wave takes 64 keys, or none; the weights are split
    // exactly into three bf16 terms as they are read, whose products with the values are exact, so the sums
    // are as accurate as fp32's. ----
    if constexpr (kBf16) {
        using namespace tiles;
        constexpr int CT = D / 16;
        const int n16 = lane & 15, g = lane >> 4;
        float4_t acc[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[ct] = float4_t{0.f, 0.f, 0.f, 0.f};
        const float* prow = Sm + (n16 & (Q - 1)) * pitch;            // P rows past Q repeat (ignored)
        static_assert(kPerLane <= kWaves, "a wave has at most one chunk of 64 keys");
        if (wave < nchunk) {                                         // uniform
#pragma unroll
            for (int jj = 0; jj < D / 32; ++jj) {
                if (jj > 0) {
                    wave_lds_sync();                                 // the last rows' reads
                    load_values(jj);
                }
                wait_lds_loads();
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const float* pk = prow + wave * kWave + 32 * u + 8 * g;
                    const float4_t x = *reinterpret_cast<const float4_t*>(pk), y = *reinterpret_cast<const float4_t*>(pk + 4);
                    const Split2 s0 = split2(x[0], x[1]), s1 = split2(x[2], x[3]), s2 = split2(y[0], y[1]), s3 = split2(y[2], y[3]);
                    const bf16x8_t w[3] = {__builtin_bit_cast(bf16x8_t, u32x4_t{s0.hi, s1.hi, s2.hi, s3.hi}),
                                           __builtin_bit_cast(bf16x8_t, u32x4_t{s0.mid, s1.mid, s2.mid, s3.mid}),
                                           __builtin_bit_cast(bf16x8_t, u32x4_t{s0.lo, s1.lo, s2.lo, s3.lo})};
#pragma unroll
                    for (int ct = 0; ct < 2; ++ct) {
                        const bf16x8_t v = rows_transposed4<32>(buf, u, ct, lane);
#pragma unroll
                        for (int p = 0; p < 3; ++p)
                            acc[2 * jj + ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[p], v, acc[2 * jj + ct], 0, 0, 0);
                    }
                }
            }
        }
        wave_lds_sync();
        if (wave < nchunk) {                                         // uniform
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int j = 0; j < 4; ++j) ((lds_ptr<float>)buf)[(ct * 16 + 4 * g + j) * 16 + n16] = acc[ct][j];
        }
    } else {
        const int prow = (lane & 15) & (Q - 1), kgrp = lane >> 4;   // P rows past Q repeat (ignored)
        const float* prw = Sm + prow * pitch + kgrp;
        float4_t acc = {0.f, 0.f, 0.f, 0.f};
        auto mma_batch = [&](int st0, const float (&vv)[kVBatch]) {
#pragma unroll
            for (int u = 0; u < kVBatch; ++u) {
                const int st = st0 + u * NKS;
                if (st >= steps) break;
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(prw[st * 4], vv[u], acc, 0, 0, 0);
            }
        };
        constexpr int kStride = NKS * kVBatch;
        for (int st0 = p3_ks; st0 < steps; st0 += 2 * kStride) {
            mma_batch(st0, vb);
            if (st0 + 2 * kStride < steps) load_v(st0 + 2 * kStride, vb);
            if (st0 + kStride >= steps) break;
            mma_batch(st0 + kStride, vb2);
            if (st0 + 3 * kStride < steps) load_v(st0 + 3 * kStride, vb2);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) red[(wave * 16 + 4 * kgrp + j) * 16 + (lane & 15)] = acc[j];
    }
    // The output element of this thread in the epilogue (Q*D <= the Q*64 threads: one each, or none),
    // and for the fused position encoding its operands, requested now that the selection and the
    // message product need their registers no more (held from before the softmax they took d = 64 past the 64
    // registers that two workgroups of 16 waves leave each other): the 3x3 window of v around the query token
    // (clamped addresses, zero outside the map through opaque masks), this channel's kernel and its bias.
    static_assert(D <= kWave, "one output element per thread");
    const int er = static_cast<int>(threadIdx.x) / D, ech = static_cast<int>(threadIdx.x) - er * D;
    const int eqi = tile * Q + er;
    float pev[9], pew[9], peb = 0.f;
    if (a.pe_w) {                                    // uniform
        const int Wc = a.Wc, Hc = N / Wc;
        const int qc = min(eqi, N - 1);
        const int qy = qc / Wc, qx = qc - qy * Wc;
        const float* wk = a.pe_w + (static_cast<size_t>(h) * D + ech) * 9;
#pragma unroll
        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                const int yy = qy + ky - 1, xx = qx + kx - 1;
                const int yc = min(max(yy, 0), Hc - 1), xc = min(max(xx, 0), Wc - 1);
                const unsigned ok = opaque_mask(yy >= 0 && yy < Hc && xx >= 0 && xx < Wc);
                pev[ky * 3 + kx] = masked(S::load1_at(vmap, __umul24(static_cast<uint32_t>(yc * Wc + xc), static_cast<uint32_t>(C)) + ech), ok);
                pew[ky * 3 + kx] = wk[ky * 3 + kx];
            }
        peb = a.pe_b ? a.pe_b[h * D + ech] : 0.f;
    }
    __syncthreads();
    if (er < Q && eqi < N) {
        const int r = er, ch = ech;
        const int ct = ch / 16, col = ch % 16;
        float s = 0.f;
        if constexpr (kBf16) {
            for (int ks = 0; ks < min(nchunk, kWaves); ++ks)         // uniform
                s += red[ks * (kCoarseBuffer / 4) + (ct * 16 + r) * 16 + col];
        } else {
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) s += red[((ks * NCT + ct) * 16 + r) * 16 + col];
        }
        const int qi = eqi;
        if (a.pe_w) {                                    // uniform: the fused position encoding
            // 3x3 depth-wise cross-correlation of v around token qi, zero outside the map, plus the bias
            float pe = peb;
#pragma unroll
            for (int k = 0; k < 9; ++k) pe = fmaf(pew[k], pev[k], pe);
            s += pe;
        }
        if (a.out) {
            float wl = 1.0f;
            if (!VA) wl = a.w ? a.w[((tok0 + qi) * a.heads + h) * a.levels] : 1.0f / a.levels;
            const float pe = a.pe0 ? a.pe0[((tok0 + qi) * a.heads + h) * D + ch] : 0.f;
            S::store1_at(static_cast<unsigned char*>(a.out) + map0 * sizeof(T), __umul24(static_cast<uint32_t>(qi), static_cast<uint32_t>(C)) + ch, wl * (s + pe));
        } else {
            store_at<float>(a.msg + map0, (__umul24(static_cast<uint32_t>(qi), static_cast<uint32_t>(C)) + ch) * 4u, s);
        }
    }
}

// a.lo * b.lo + a.hi * b.hi + c for two packed bf16 pairs, fp32 accumulation
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c, false);
}

// Small coarsest maps (N <= 64, e.g. the many short maps of attention along epipolar lines): a wave
// takes `qpw` consecutive query rows of one (batch, head) map, lane j holding key j. Key row j and
// the value chunks a lane needs are loaded once per wave; per query row the logits are per-lane dot
// products, the softmax and the selection are wave reductions and a ballot radix select, and the
// message is formed from the weights in LDS: lane (c, g) sums chunk c of value rows g, g + G, ...
// and DPP sums over the G lanes of a chunk add the groups.
template <typename T, int D, bool VA>
__global__ __launch_bounds__(256) void coarse_small_kernel(CoarseArgs a, int qpw)
{
    using S = Storage<T>;
    constexpr int E = S::kPer16B;
    constexpr int CH = D / E;                                 // chunks of a head row
    constexpr int G = kWave / CH;                             // key groups of the message, >= E (D <= 64)
    constexpr int NV = kWave / G;                             // value rows a lane covers (N <= 64)
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int N = a.N, C = a.C;
    const int wpm = (N + qpw - 1) / qpw;                      // waves per map
    const int gw = static_cast<int>(blockIdx.x) * 4 + wave;   // < 2^31, checked by the launcher
    if (gw >= a.B * a.heads * wpm) return;                    // whole wave
    const int bh = gw / wpm;
    const int q0 = (gw - bh * wpm) * qpw, qend = min(q0 + qpw, N);
    const int h = bh % a.heads, b = bh / a.heads;
    const size_t tok0 = static_cast<size_t>(b) * N;
    const size_t hoff = static_cast<size_t>(h) * D;
    const bool valid = lane < N;
    const unsigned char* qb = static_cast<const unsigned char*>(a.q) + (tok0 * C + hoff) * sizeof(T);
    // key row j (clamped onto the map) and value chunk c of rows g, g + G, ...
    const int c = lane / G, g = lane % G;
    // bf16 keys stay packed (products of pairs with the query's packed pairs); fp32 keys as floats
    constexpr bool kDot2 = std::is_same<T, bf16>::value;
    uint4 kraw[CH];
    float kf[kDot2 ? 1 : D];
    uint4 vraw[NV];
    {
        const uint4* kp = reinterpret_cast<const uint4*>(static_cast<const unsigned char*>(a.k) +
                                                         ((tok0 + min(lane, N - 1)) * C + hoff) * sizeof(T));
        const unsigned char* vb = static_cast<const unsigned char*>(a.v) + (tok0 * C + hoff) * sizeof(T) + c * 16;
#pragma unroll
        for (int cc = 0; cc < CH; ++cc) kraw[cc] = kp[cc];
#pragma unroll
        for (int u = 0; u < NV; ++u)
            vraw[u] = *reinterpret_cast<const uint4*>(vb + static_cast<size_t>(min(g + u * G, N - 1)) * C * sizeof(T));
        if constexpr (!kDot2) {
#pragma unroll
            for (int cc = 0; cc < CH; ++cc) S::unpack(kraw[cc], kf + cc * E);
        }
    }
    __shared__ float pw[4][kWave];
    __shared__ int sidx[4][kWave];
    __shared__ float skey[4][kWave];
    // the query row: lanes c * G, ... hold its chunk c, read by every lane with readlane; the next
    // row is in flight while this one is used
    auto qchunk = [&](int qi) {
        return reinterpret_cast<const uint4*>(qb + static_cast<size_t>(qi) * C * sizeof(T))[c];
    };
    uint4 qv = qchunk(q0);
    // the previous row's selection and message, stored once this row's query has arrived so that
    // the wait for the query never waits for them
    size_t sel_at = 0, msg_at = 0;
    int sel_i = 0;
    float sel_k = 0.f, msg_v = 0.f;
    bool sel_pending = false, msg_pending = false;
    for (int qi = q0; qi < qend; ++qi) {
        float x = 0.f;
#pragma unroll
        for (int cc = 0; cc < CH; ++cc) {
            uint4 t;
            t.x = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(qv.x), cc * G));
            t.y = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(qv.y), cc * G));
            t.z = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(qv.z), cc * G));
            t.w = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(qv.w), cc * G));
            if constexpr (kDot2) {
                x = dot2_bf16(t.x, kraw[cc].x, x);
                x = dot2_bf16(t.y, kraw[cc].y, x);
                x = dot2_bf16(t.z, kraw[cc].z, x);
                x = dot2_bf16(t.w, kraw[cc].w, x);
            } else {
                float qf[E];
                S::unpack(t, qf);
#pragma unroll
                for (int e = 0; e < E; ++e) x += qf[e] * kf[cc * E + e];
            }
        }
        qv = qchunk(min(qi + 1, qend - 1));
        if (sel_pending) {
            a.sel_idx[sel_at] = sel_i;
            a.sel_key[sel_at] = sel_k;
        }
        if (msg_pending) a.msg[msg_at] = msg_v;
        x = valid ? x * a.scale : -INFINITY;
        const float mx = wave_max_fast(x);
        float p = valid ? __expf(x - mx) : 0.f;
        p *= fast_rcp(wave_sum_fast(p));
        if (a.K > 0) {
            const uint32_t key[1] = {valid ? ordered_bits(x) : 0u};
            const uint32_t name[1] = {static_cast<uint32_t>(lane)};
            bool sel[1];
            const int keff = a.K < N ? a.K : N;
            wave_select_top<1>(key, name, keff, sel);
            const bool kept = sel[0];
            // listed in index order through LDS, then slot o = min(lane, K - 1) written by every lane
            // (lanes past K repeat slot K - 1 with its own values)
            if (kept) {
                const int pos = lanes_below(__ballot(kept));
                sidx[wave][pos] = lane;
                skey[wave][pos] = p;
                if constexpr (VA) p = 0.f;                    // refined at the next level (Omega)
            }
            wave_lds_sync();
            const int o = min(lane, a.K - 1);
            const size_t orow = (static_cast<size_t>(bh) * N + qi) * a.K;
            const int oi = sidx[wave][min(o, kWave - 1)];
            const float ok = skey[wave][min(o, kWave - 1)];
            sel_at = orow + o;
            sel_i = o < keff ? oi : -1;
            sel_k = o < keff ? ok : 0.f;
            sel_pending = true;
        }
        pw[wave][lane] = p;
        wave_lds_sync();
        float acc[E];
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = 0.f;
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int jj = g + u * G;
            float pj = pw[wave][jj];
            pj = jj < N ? pj : 0.f;
            float vf[E];
            S::unpack(vraw[u], vf);
#pragma unroll
            for (int e = 0; e < E; ++e) acc[e] += pj * vf[e];
        }
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = group_sum<G>(acc[e]);
        // every lane holds its chunk's sums: lane (g, c) writes channel c * E + g % E (lanes with
        // g >= E repeat a channel with the same value)
        const int ge = g % E;
        float m = acc[0];
#pragma unroll
        for (int e = 1; e < E; ++e) m = ge == e ? acc[e] : m;
        const int ch = c * E + ge;
        if (a.out) {
            float wl = 1.0f;
            if (!VA) wl = a.w ? a.w[((tok0 + qi) * a.heads + h) * a.levels] : 1.0f / a.levels;
            const float pe = a.pe0 ? a.pe0[((tok0 + qi) * a.heads + h) * D + ch] : 0.f;
            S::store1(a.out, (tok0 + qi) * C + hoff + ch, wl * (m + pe));
        } else {
            msg_at = ((tok0 + qi) * a.heads + h) * D + ch;
            msg_v = m;
            msg_pending = true;
        }
    }
    if (sel_pending) {
        a.sel_idx[sel_at] = sel_i;
        a.sel_key[sel_at] = sel_k;
    }
    if (msg_pending) a.msg[msg_at] = msg_v;
}

template <typename T, int D, bool VA>
hipError_t launch_small(const CoarseArgs& a, hipStream_t stream)
{
    // enough query rows per wave that the waves fit the chip's wave slots (at the kernel's
    // occupancy) about once
    // (the occupancy depends on the kernel and the architecture only; racing threads store the same value)
    static std::atomic<int> occupancy{0};
    int blocks_per_cu = occupancy.load(std::memory_order_relaxed);
    if (blocks_per_cu == 0) {
        int n = 0;
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &n, reinterpret_cast<const void*>(&coarse_small_kernel<T, D, VA>), 4 * kWave, 0);
        if (e != hipSuccess) return e;
        blocks_per_cu = n > 0 ? n : 1;
        occupancy.store(blocks_per_cu, std::memory_order_relaxed);
    }
    const long long maps = static_cast<long long>(a.B) * a.heads;
    const long long slots = static_cast<long long>(device_cu_count()) * blocks_per_cu * 4;
    long long qpw = std::min<long long>(a.N, std::max<long long>(1, (maps * a.N + slots - 1) / slots));
    while (qpw < a.N && maps * ((a.N + qpw - 1) / qpw) > slots) ++qpw;   // no partial second round
    const long long wpm = (a.N + qpw - 1) / qpw;
    qpw = (a.N + wpm - 1) / wpm;                                          // the rows spread evenly
    const long long waves = maps * wpm;
    if (waves > 0x7FFFFFFFLL - 3) return hipErrorInvalidValue;
    const long long blocks = (waves + 3) / 4;
    hipLaunchKernelGGL((coarse_small_kernel<T, D, VA>), dim3(static_cast<unsigned>(blocks)), dim3(4 * kWave), 0, stream, a,
                       static_cast<int>(qpw));
    return hipGetLastError();
}

// Query rows per workgroup of the coarse kernel (its waves, one per row in the softmax and selection
// phase). Fewer rows per workgroup spread a small map's rows over more compute units, so that the
// selection's scalar work and each phase's latency are shared by fewer rows, at the price of more
// passes over the map's keys and values (from L2) and of MFMA tiles only half filled. Measured on
// MI355X, a call of the stage, bf16, d = 32, K = 16, 8 against 16 rows: 16 maps of 300 keys 11.6 and 12.6 us, 128 of
// them 46.1 and 48.7 (both without the ordering launch); 4, 16, 64 and 128 maps of 440 keys 10.3 and 11.5, 20.2 and
// 20.4, 55 and 61, 95 and 117; of 512 11.1 and 11.8, 22.2 and 22.3, 66 and 73, 118 and 140; of 672 14.3 and 13.3, 36.1
// and 33.4, 113 and 110, 218 and 209; of 1023 17.6 and 15.8, 56 and 51, 200 and 194, 394 and 383 (8 rows are ahead
// there for K = 64 alone). d = 64, 32 maps of 196 keys: 13.3 and 12.3. So 8 rows for bf16 with d = 32 (one 16-byte
// chunk per key row and k-step pair) up to 512 keys, 16 elsewhere: fp32, d = 64, and more keys, where the passes over
// them count for more.
template <typename T, int D, int kPerLane>
constexpr int coarse_rows()
{
    return (sizeof(T) == 2 && D == 32 && kPerLane <= 8) ? 8 : 16;
}

template <typename T, int D, bool VA, int kPerLane, int Q>
hipError_t launch_rows(const CoarseArgs& a, hipStream_t stream)
{
    const size_t behind = sizeof(T) == 2 ? static_cast<size_t>(coarse_behind(a.N, Q)) : static_cast<size_t>(Q) * 16 * 16 * sizeof(float);
    const size_t lds = static_cast<size_t>(Q) * coarse_pitch(a.N) * sizeof(float) + behind;
    if (lds > device_max_lds()) return hipErrorInvalidValue;
    static std::atomic<unsigned long long> configured{0};     // devices whose LDS limit is raised
    if (hipError_t e = set_max_lds_once(reinterpret_cast<const void*>(&coarse_attn_kernel<T, D, VA, kPerLane, Q>), configured);
        e != hipSuccess)
        return e;
    const int tiles = (a.N + Q - 1) / Q;
    const long long blocks = static_cast<long long>(a.B) * a.heads * tiles;
    if (blocks > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((coarse_attn_kernel<T, D, VA, kPerLane, Q>), dim3(static_cast<unsigned>(blocks)), dim3(Q * kWave),
                       lds, stream, a);
    return hipGetLastError();
}

template <typename T, int D, bool VA, int kPerLane>
hipError_t launch_one(const CoarseArgs& a, hipStream_t stream)
{
    return launch_rows<T, D, VA, kPerLane, coarse_rows<T, D, kPerLane>()>(a, stream);
}

template <typename T, int D, bool VA>
hipError_t launch_per_lane(const CoarseArgs& a, hipStream_t stream)
{
    if (a.N <= kWave) {
        if (a.pe_w) return hipErrorInvalidValue;       // the small-map kernel has no fused position encoding
        return launch_small<T, D, VA>(a, stream);
    }
    switch (coarse_per_lane(a.N)) {
    case 1: return launch_one<T, D, VA, 1>(a, stream);
    case 2: return launch_one<T, D, VA, 2>(a, stream);
    case 3: return launch_one<T, D, VA, 3>(a, stream);
    case 4: return launch_one<T, D, VA, 4>(a, stream);
    case 5: return launch_one<T, D, VA, 5>(a, stream);
    case 6: return launch_one<T, D, VA, 6>(a, stream);
    case 8: return launch_one<T, D, VA, 8>(a, stream);
    case 12: return launch_one<T, D, VA, 12>(a, stream);
    case 16: return launch_one<T, D, VA, 16>(a, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_coarse_attn(const CoarseArgs& args, int d, bool variant_a, bool bf16_in, hipStream_t stream)
{
    CoarseArgs a = args;
    a.near = a.Wc > 0 && lane_keys_near(a.Wc);
#define QTA_COARSE_CASE(T, D)                                                                     \
    if (d == D) return variant_a ? launch_per_lane<T, D, true>(a, stream) : launch_per_lane<T, D, false>(a, stream);
    if (bf16_in) {
        QTA_COARSE_CASE(bf16, 32)
        QTA_COARSE_CASE(bf16, 64)
    } else {
        QTA_COARSE_CASE(float, 32)
        QTA_COARSE_CASE(float, 64)
    }
#undef QTA_COARSE_CASE
    return hipErrorInvalidValue;
}

}  // namespace qta
