// Step 3 as a standalone row-wise top-K (Sec. 3.2: each query keeps the K keys with the highest
// attention scores).
//
// One wave per row, read once. Each lane holds NPER candidates of the row as 32-bit ranking keys (larger is
// better, 0 = not a candidate):
//   1. a lower bound of the K-th largest key: the K-th largest of the wave's group maxima (a lane's
//      candidates form G groups; K groups have a member at or above it). A bitwise search on ballots over G
//      values a lane instead of NPER;
//   2. the candidates at or above the bound (about K of them for K <= 16, 44 for K = 32 of one group a
//      lane, 74 for K = 64 of four) go to LDS with their names. More than fit there (equal scores) are first
//      cut to exactly K by the same search over all the wave's candidates;
//   3. more than 64 survivors are cut to exactly K by the search over four a lane;
//   4. at most 64 survivors, one a lane: each counts the words (score, inverted name) above its own and,
//      when fewer than K are, writes itself to that place. So the order is (score descending, name
//      ascending), and repeated names stay separate candidates.
// Bound by the row's read (3.3 of 5.1 TB/s at that size). The previous form took K rounds of a wave-wide 64-bit maximum over 1, 4, 16 or
// 64 slots a lane: 9600 rows of 1200, K = 16: 226 -> 14.4 us.
#include "qta_device.h"
#include "qta_internal.h"

namespace qta {

namespace {

constexpr int kSurvivors = 256;         // survivors of a row kept in LDS

// Lists in LDS every one of the wave's keys above `thr`, with its name; returns how many.
template <int NPER, typename Name>
__device__ __forceinline__ int list_above(const uint32_t (&key)[NPER], Name name, uint32_t thr, uint32_t* lk, int32_t* ln)
{
    int n = 0;
#pragma unroll
    for (int e = 0; e < NPER; ++e) {
        const bool in = key[e] > thr;
        const uint64_t mask = __ballot(in);
        if (in) {
            const int pos = n + lanes_below(mask);
            lk[pos] = key[e];
            ln[pos] = name(e);
        }
        n += __popcll(mask);
    }
    return n;
}

// Lists exactly keff of the wave's keys: every key above the cut, and at the cut the lowest names first (of a
// repeated name, the lowest place in the row), a wave-wide minimum for each.
template <int NPER, typename Name>
__device__ __forceinline__ void list_top(const uint32_t (&key)[NPER], Name name, int keff, uint32_t* lk, int32_t* ln)
{
    const uint32_t cut = wave_cut<NPER>(key, keff);
    int n = 0;
#pragma unroll
    for (int e = 0; e < NPER; ++e) n += __popcll(__ballot(key[e] >= cut));
    n = list_above<NPER>(key, name, n == keff ? cut - 1u : cut, lk, ln);
    const uint32_t lane = threadIdx.x & 63;
    uint64_t last = 0;                                   // (name, place in the row) + 1 of the last one taken
    for (int r = n; r < keff; ++r) {                     // uniform
        uint64_t mine = ~0ull;
#pragma unroll
        for (int e = 0; e < NPER; ++e) {
            const uint64_t w = (static_cast<uint64_t>(static_cast<uint32_t>(name(e))) << 32) | (lane + kWave * e);
            if (key[e] == cut && w >= last && w < mine) mine = w;
        }
        uint64_t low = mine;
        for (int m = 32; m >= 1; m >>= 1) {
            const uint64_t o = shfl_xor_u64(low, m);
            low = o < low ? o : low;
        }
        if (lane == 0) {
            lk[r] = cut;
            ln[r] = static_cast<int32_t>(low >> 32);
        }
        last = low + 1;
    }
}

// NAMED: candidates are named by cand_idx (negative: not a candidate), else by their column.
template <int NPER, bool NAMED>
__global__ __launch_bounds__(256) void topk_kernel(TopkArgs a)
{
    __shared__ uint32_t lkey[4][kSurvivors];
    __shared__ int32_t lname[4][kSurvivors];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int row = blockIdx.x * 4 + wave;
    if (row >= a.rows) return;                  // whole wave leaves; no workgroup barriers below
    const float* keys = a.keys + static_cast<size_t>(row) * a.n;
    const int32_t* names = NAMED ? a.cand_idx + static_cast<size_t>(row) * a.n : nullptr;
    const int K = a.K;
    auto name = [&](int e) -> int32_t {
        const int j = lane + kWave * e;
        return NAMED ? names[min(j, a.n - 1)] : j;
    };
    // every load unconditional (clamped into the row) so that all are in flight at once; slots past the row
    // and negative names are masked to 0 (no candidate)
    uint32_t key[NPER];
    {
        int32_t nm[NAMED ? NPER : 1];
#pragma unroll
        for (int e = 0; e < NPER; ++e) {
            key[e] = __float_as_uint(keys[min(lane + kWave * e, a.n - 1)]);
            if constexpr (NAMED) nm[e] = name(e);
        }
#pragma unroll
        for (int e = 0; e < NPER; ++e) {
            const bool live = lane + kWave * e < a.n && (!NAMED || nm[NAMED ? e : 0] >= 0);
            key[e] = live ? ordered_bits(__uint_as_float(key[e])) : 0u;
        }
    }
    asm volatile("" ::: "memory");       // names are read again where they are listed, not kept in registers

    // 1. the bound (0 keeps nothing out; a key of a candidate is never 0)
    constexpr int G = NPER < 4 ? NPER : 4;
    uint32_t low = 1u;
    {
        uint32_t gm[G];
#pragma unroll
        for (int g = 0; g < G; ++g) gm[g] = 0u;
#pragma unroll
        for (int e = 0; e < NPER; ++e) gm[e % G] = max(gm[e % G], key[e]);
        if (K > 32) {                                    // uniform
            int n = 0;
#pragma unroll
            for (int g = 0; g < G; ++g) n += __popcll(__ballot(gm[g] != 0u));
            if (n >= K) low = wave_cut<G>(gm, K);
        } else {
            uint32_t m[1] = {gm[0]};
#pragma unroll
            for (int g = 1; g < G; ++g) m[0] = max(m[0], gm[g]);
            if (__popcll(__ballot(m[0] != 0u)) >= K) low = wave_cut<1>(m, K);
        }
        low = max(low, 1u);
    }
    // 2. the survivors
    int n = 0;
#pragma unroll
    for (int e = 0; e < NPER; ++e) n += __popcll(__ballot(key[e] >= low));
    n = __builtin_amdgcn_readfirstlane(n);
    if (n > kSurvivors) {                                // uniform; then n > K
        list_top<NPER>(key, name, K, lkey[wave], lname[wave]);
        n = K;
    } else {
        list_above<NPER>(key, name, low - 1u, lkey[wave], lname[wave]);
    }
    wave_lds_sync();
    // 3. at most 64 of them
    if (n > kWave) {                                     // uniform
        constexpr int S = kSurvivors / kWave;
        uint32_t k4[S];
        int32_t n4[S];
#pragma unroll
        for (int e = 0; e < S; ++e) {
            const int i = lane + kWave * e;
            k4[e] = i < n ? lkey[wave][i] : 0u;
            n4[e] = i < n ? lname[wave][i] : -1;
        }
        wave_lds_sync();
        list_top<S>(k4, [&](int e) { return n4[e]; }, K, lkey[wave], lname[wave]);
        wave_lds_sync();
        n = K;
    }
    // 4. each survivor's place (equal words, of a repeated name, in lane order)
    const bool have = lane < n;
    const uint32_t wk = have ? lkey[wave][lane] : 0u;
    const int32_t wn = have ? lname[wave][lane] : -1;
    const uint64_t word = have ? (static_cast<uint64_t>(wk) << 32) | static_cast<uint32_t>(~static_cast<uint32_t>(wn)) : 0ull;
    int place = 0;
    for (int i = 0; i < n; ++i) {                        // uniform trip count
        const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(word), i);
        const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(word >> 32), i);
        const uint64_t wi = (static_cast<uint64_t>(hi) << 32) | lo;
        place += (wi > word || (wi == word && i < lane)) ? 1 : 0;
    }
    const size_t orow = static_cast<size_t>(row) * K;
    if (have && place < K) {
        a.idx_out[orow + place] = wn;
        if (a.key_out) a.key_out[orow + place] = from_ordered_bits(wk);
    }
    if (lane >= n && lane < K) {                         // fewer than K candidates: pad
        a.idx_out[orow + lane] = -1;
        if (a.key_out) a.key_out[orow + lane] = 0.f;
    }
}

// In-place ordering of selection rows of K <= 64 entries (the stage calls' output contract): one
// wave per row, lane i holds entry i as a ranking word (0 for an empty slot, index -1), counts the
// entries ranked before it by reading every other lane's word, and writes itself to that place.
// Empty slots follow the kept keys. Every load of the row completes before any store (the ranks
// need all of them).
__global__ __launch_bounds__(256) void sort_rows_kernel(int32_t* idx, float* key, int rows, int K)
{
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;                    // whole wave leaves; no workgroup barriers below
    const size_t base = static_cast<size_t>(row) * K;
    const int e = min(lane, K - 1);
    const int32_t my_idx = idx[base + e];
    const float my_key = key[base + e];
    const bool live = lane < K && my_idx >= 0;
    const uint64_t word = live ? rank_word(my_key, my_idx) : 0ull;
    int before = 0;
    for (int j = 0; j < K; ++j) {               // uniform trip count
        const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(word), j);
        const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(word >> 32), j);
        const uint64_t wj = (static_cast<uint64_t>(hi) << 32) | lo;
        before += wj > word ? 1 : 0;
    }
    const uint64_t live_mask = __ballot(live);
    const uint64_t dead_mask = __ballot(lane < K && !live);
    const int nlive = __popcll(live_mask);
    const int pos = live ? before : nlive + lanes_below(dead_mask);
    if (lane < K) {
        idx[base + pos] = live ? my_idx : -1;
        key[base + pos] = live ? my_key : 0.f;
    }
}

}  // namespace

hipError_t launch_sort_rows(int32_t* idx, float* key, long long rows, int K, hipStream_t stream)
{
    if (rows <= 0) return hipSuccess;
    if (K < 1 || K > kWave || rows > 0x7FFFFFFFLL - 3) return hipErrorInvalidValue;
    hipLaunchKernelGGL(sort_rows_kernel, dim3(static_cast<unsigned>((rows + 3) / 4)), dim3(256), 0, stream, idx, key,
                       static_cast<int>(rows), K);
    return hipGetLastError();
}

template <int NPER>
hipError_t launch_topk_row(const TopkArgs& a, hipStream_t stream)
{
    const unsigned blocks = static_cast<unsigned>((static_cast<long long>(a.rows) + 3) / 4);
    if (a.cand_idx) hipLaunchKernelGGL((topk_kernel<NPER, true>), dim3(blocks), dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((topk_kernel<NPER, false>), dim3(blocks), dim3(256), 0, stream, a);
    return hipGetLastError();
}

// Slots a lane holds: as many as the row needs, rounded up to the next instantiated count (at most a third
// idle; a row of 1200 in 64 slots a lane instead of 20 would do three times the work).
hipError_t launch_topk(const TopkArgs& a, hipStream_t stream)
{
    const int need = (a.n + kWave - 1) / kWave;
    if (need <= 1) return launch_topk_row<1>(a, stream);
    if (need <= 2) return launch_topk_row<2>(a, stream);
    if (need <= 4) return launch_topk_row<4>(a, stream);
    if (need <= 6) return launch_topk_row<6>(a, stream);
    if (need <= 8) return launch_topk_row<8>(a, stream);
    if (need <= 12) return launch_topk_row<12>(a, stream);
    if (need <= 16) return launch_topk_row<16>(a, stream);
    if (need <= 20) return launch_topk_row<20>(a, stream);
    if (need <= 24) return launch_topk_row<24>(a, stream);
    if (need <= 32) return launch_topk_row<32>(a, stream);
    if (need <= 48) return launch_topk_row<48>(a, stream);
    if (need <= 64) return launch_topk_row<64>(a, stream);
    return hipErrorInvalidValue;
}

}  // namespace qta
