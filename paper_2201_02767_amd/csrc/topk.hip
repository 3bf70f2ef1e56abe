// Step 3 as a standalone row-wise top-K (Sec. 3.2: each query keeps the K keys with the highest
// attention scores).
//
// One wave per row, read once. Each lane holds NPER candidates of the row as 32-bit ranking keys (larger is
// better, 0 = not a candidate):
//   1. a lower bound of the K-th largest key: the K-th largest of the wave's group maxima (a lane's
//      candidates form G groups; K groups have a member at or above it). Up to K = 8 by wave-wide maxima,
//      else a bitwise search on ballots over G values a lane instead of NPER;
//   2. the candidates at or above the bound (about K of them for K <= 16, 44 for K = 32 of one group a
//      lane, 74 for K = 64 of four) go to LDS with their names. More than fit there (equal scores) are first
//      cut to exactly K by the same search over all the wave's candidates, the lowest names at the cut first:
//      those of the lowest columns, or with drawn names the lowest of those seen so far, a few chunks at a time;
//   3. survivors are cut to exactly K where that costs less than placing them all;
//   4. at most 64 survivors, one a lane: each counts the words (score, inverted name) above its own and,
//      when fewer than K are, writes itself to that place. So the order is (score descending, name
//      ascending), and repeated names stay separate candidates.
// What its time goes to: for long rows mostly their read (9600 rows of 1200, K = 16: 14.4 us, 3.3 TB/s or 65% of
// the rate of a copy), for short ones instruction issue. Rows of one score throughout, us a call (the host takes
// 10): 1e4 rows of 100, K = 4 10 and K = 33 15; 5e3 of 200, K = 16 10; 244 of 4096, K = 4 10, with drawn names 22.
// With one wave-wide 64-bit minimum for each place at the cut they took 24, 57, 22, 43 and 44; with K rounds of a
// maximum over the whole row 10, 53, 17, 22 and 22 (and the long rows 226).
#include "qta_device.h"
#include "qta_internal.h"

namespace qta {

namespace {

constexpr int kSurvivors = 256;         // survivors of a row kept in LDS
constexpr int kFew = 8;                 // K up to which the bound is found by maxima

// A candidate's ranking key: never 0, which the NaN of all one bits alone would get.
__device__ __forceinline__ uint32_t rank_key(float f) { return max(ordered_bits(f), 1u); }

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

// wave_cut for a small keff: the largest value, the next, ... until keff keys reach it, a wave-wide maximum each.
// Equal keys end it early, where the search by bits goes to the last bit.
template <int NPER>
__device__ __forceinline__ uint32_t wave_cut_few(const uint32_t (&key)[NPER], int keff)
{
    uint32_t cut = ~0u;
    int n = 0;
    do {                                                 // uniform
        uint32_t top = 0u;
#pragma unroll
        for (int e = 0; e < NPER; ++e) top = max(top, key[e] < cut ? key[e] : 0u);
        cut = wave_max_u32(top);
        n = 0;
#pragma unroll
        for (int e = 0; e < NPER; ++e) n += __popcll(__ballot(key[e] >= cut));
    } while (n < keff);
    return cut;
}

// Leaves the `need` lowest of the m names at `ln` (need < m <= 64 S) there, in any order, and returns a bound: a
// name whose complement is below it is none of them.
template <int S>
__device__ __forceinline__ uint32_t lowest_names(int32_t* ln, int m, int need)
{
    const int lane = threadIdx.x & 63;
    uint32_t k[S];                                       // complements: the lowest names are the largest
#pragma unroll
    for (int e = 0; e < S; ++e) {
        const int i = lane + kWave * e;
        k[e] = i < m ? ~static_cast<uint32_t>(ln[i]) : 0u;
    }
    wave_lds_sync();
    const uint32_t cut = need <= kFew ? wave_cut_few<S>(k, need) : wave_cut<S>(k, need);
    int t = 0;
#pragma unroll
    for (int e = 0; e < 2 * S; ++e) {                    // those above the cut, then as many at it as are missing
        const bool in = e < S ? k[e % S] > cut : k[e % S] == cut;
        const uint64_t mask = __ballot(in);
        const int pos = t + lanes_below(mask);
        if (in && pos < need) ln[pos] = static_cast<int32_t>(~k[e % S]);
        t += __popcll(mask);
    }
    wave_lds_sync();
    return cut;
}

// Lists exactly keff of the wave's keys, of which at least keff reach `low`: every key above the cut, and at the cut
// the lowest names first. Returns how many lie above the cut; the rest are for the caller where TIES is false.
// ORDERED: names ascend with (e, lane), so those are the first in that order; else (at most kSurvivors keys in
// all) the lowest names are found among the ties.
template <int NPER, bool ORDERED, bool TIES, typename Name>
__device__ __forceinline__ int list_top(const uint32_t (&key)[NPER], Name name, int keff, uint32_t low, uint32_t* lk,
                                        int32_t* ln, uint32_t& cut)
{
    // mostly the bound itself is the cut: it was reached by too many keys because they are equal
    int n = 0;
#pragma unroll
    for (int e = 0; e < NPER; ++e) n += __popcll(__ballot(key[e] > low));
    cut = __builtin_amdgcn_readfirstlane(n) < keff ? low : wave_cut<NPER>(key, keff);
    const int above = list_above<NPER>(key, name, cut, lk, ln), need = keff - above;
    if constexpr (TIES) {
        const int limit = ORDERED ? need : kSurvivors - above;
        int m = 0;
#pragma unroll
        for (int e = 0; e < NPER; ++e) {
            if (m < limit) {                             // uniform
                const uint64_t mask = __ballot(key[e] == cut);
                const int pos = m + lanes_below(mask);
                if (key[e] == cut && pos < limit) ln[above + pos] = name(e);
                m += __popcll(mask);
            }
        }
        wave_lds_sync();
        if (!ORDERED && m > need && need > 0) lowest_names<NPER>(ln + above, m, need);        // uniform
        if (static_cast<int>(threadIdx.x & 63) < need) lk[above + (threadIdx.x & 63)] = cut;
    }
    return above;
}

// The `need` (at least 1) lowest names of the row's candidates with this ranking key to `ln`, which has room for
// `cap` (at least 64 more than need) names. Keys and names are read again, a few chunks in flight, and names past the
// `need` lowest so far are left out.
__device__ __forceinline__ void list_ties(const float* keys, const int32_t* names, int n, uint32_t cut, int need, int cap,
                                          int32_t* ln)
{
    constexpr int kBatch = 4;
    const int lane = threadIdx.x & 63;
    uint32_t floor = 0u;
    int m = 0;
    for (int j0 = 0; j0 < n; j0 += kBatch * kWave) {     // uniform
        float k[kBatch];
        int32_t nm[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int j = min(j0 + kWave * u + lane, n - 1);
            k[u] = keys[j];
            nm[u] = names[j];
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const bool in = j0 + kWave * u + lane < n && nm[u] >= 0 && rank_key(k[u]) == cut &&
                            ~static_cast<uint32_t>(nm[u]) >= floor;
            const uint64_t mask = __ballot(in);
            if (m + __popcll(mask) > cap) {              // uniform
                wave_lds_sync();
                floor = lowest_names<kSurvivors / kWave>(ln, m, need);
                m = need;
            }
            if (in) ln[m + lanes_below(mask)] = nm[u];
            m += __popcll(mask);
        }
    }
    wave_lds_sync();
    if (m > need) lowest_names<kSurvivors / kWave>(ln, m, need);      // uniform
}

// Cuts the n listed survivors (at most 64 S, K < n) to exactly K, in place. ORDERED: listed by ascending name.
template <int S, bool ORDERED>
__device__ __forceinline__ void top_survivors(int n, int K, uint32_t low, uint32_t* lk, int32_t* ln)
{
    const int lane = threadIdx.x & 63;
    uint32_t k[S], cut;
    int32_t nm[S];
#pragma unroll
    for (int e = 0; e < S; ++e) {
        const int i = lane + kWave * e;
        k[e] = i < n ? lk[i] : 0u;
        nm[e] = i < n ? ln[i] : -1;
    }
    wave_lds_sync();
    list_top<S, ORDERED, true>(k, [&](int e) { return nm[e]; }, K, low, lk, ln, cut);
    wave_lds_sync();
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
            key[e] = live ? rank_key(__uint_as_float(key[e])) : 0u;
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
            if (__popcll(__ballot(m[0] != 0u)) >= K) low = K <= kFew ? wave_cut_few<1>(m, K) : wave_cut<1>(m, K);
        }
        low = max(low, 1u);
    }
    // 2. the survivors
    int n = 0;
#pragma unroll
    for (int e = 0; e < NPER; ++e) n += __popcll(__ballot(key[e] >= low));
    n = __builtin_amdgcn_readfirstlane(n);
    if (NPER * kWave > kSurvivors && n > kSurvivors) {   // uniform; then n > K
        uint32_t cut;
        const int above = list_top<NPER, true, !NAMED>(key, name, K, low, lkey[wave], lname[wave], cut);
        if (NAMED && above < K) {
            list_ties(keys, names, a.n, cut, K - above, kSurvivors - above, lname[wave] + above);
            if (lane < K - above) lkey[wave][above + lane] = cut;
        }
        n = K;
    } else {
        list_above<NPER>(key, name, low - 1u, lkey[wave], lname[wave]);
    }
    wave_lds_sync();
    // 3. at most 64 of them, and not many more than K: placing one costs 8 instructions, cutting one a lane some 130,
    // or 250 with drawn names and K > kFew (rows of 64 equal scores, K = 16: 31 us with that cut, 23 without)
    if (n > K + 16) {                                    // uniform
        bool cut = true;
        if (NPER > 2 && n > 2 * kWave) top_survivors<kSurvivors / kWave, !NAMED>(n, K, low, lkey[wave], lname[wave]);
        else if (NPER > 1 && n > kWave) top_survivors<2, !NAMED>(n, K, low, lkey[wave], lname[wave]);
        else if (!NAMED || K <= kFew) top_survivors<1, !NAMED>(n, K, low, lkey[wave], lname[wave]);
        else cut = false;
        n = cut ? K : n;
    } else if (n > kWave) {
        top_survivors<2, !NAMED>(n, K, low, lkey[wave], lname[wave]);
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
