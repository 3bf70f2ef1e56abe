// Kernels and launchers of the backward passes for bf16 maps (bwd_bf16.h).
#include "bwd_bf16.h"

namespace qta {

namespace {

template <int D, int NT, bool VA, bool FINEST>
__global__ __launch_bounds__(256) void bwd_query_bf16_kernel(BwdLevelArgs a)
{
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int nitems = a.B * a.heads * a.Hp * a.Wp;           // below 2^31 (checked by the launcher)
    const int it = xcd_remap(blockIdx.x, gridDim.x) * 4 + wave;
    if (it >= nitems) return;              // whole wave leaves; only wave-level syncs follow
    extern __shared__ __align__(16) unsigned char smem[];
    bwd16::query_item<D, NT, VA, FINEST>(a, it, smem + wave * bwd16::wave_bytes<D, NT>());
}

template <int D, int NT, bool VA, bool FINEST>
hipError_t launch_query(const BwdLevelArgs& a, hipStream_t stream)
{
    constexpr size_t lds = 4 * bwd16::wave_bytes<D, NT>();
    static_assert(lds <= 64 * 1024, "within the default LDS limit");
    const long long items = static_cast<long long>(a.B) * a.heads * a.Hp * a.Wp;
    const long long blocks = (items + 3) / 4;
    if (blocks * 4 >= 0x7FFFFFFFLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((bwd_query_bf16_kernel<D, NT, VA, FINEST>), dim3(static_cast<unsigned>(blocks)), dim3(4 * kWave),
                       lds, stream, a);
    return hipGetLastError();
}

template <int D, bool VA, bool FINEST>
hipError_t launch_query_tiles(const BwdLevelArgs& a, hipStream_t stream)
{
    const int nslot = 4 * a.Kp;
    if (nslot <= 16) return launch_query<D, 1, VA, FINEST>(a, stream);
    if (nslot <= 32) return launch_query<D, 2, VA, FINEST>(a, stream);
    if (nslot <= 64) return launch_query<D, 4, VA, FINEST>(a, stream);
    return hipErrorInvalidValue;
}

template <int D>
hipError_t launch_query_d(const BwdLevelArgs& a, bool variant_a, bool finest, hipStream_t stream)
{
    if (variant_a) return finest ? launch_query_tiles<D, true, true>(a, stream) : launch_query_tiles<D, true, false>(a, stream);
    return finest ? launch_query_tiles<D, false, true>(a, stream) : launch_query_tiles<D, false, false>(a, stream);
}

template <int D, bool VA, bool ROW>
__global__ __launch_bounds__(256) void bwd_combine_bf16_kernel(BwdLevelArgs a, bwd16::CombineGrid cg, int nitems)
{
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int it = xcd_remap(blockIdx.x, gridDim.x) * 4 + wave;
    if (it >= nitems) return;              // whole wave
    bwd16::combine_item<D, VA, ROW>(a, cg, it);
}

template <int D, bool VA, bool ROW>
hipError_t launch_combine(const BwdLevelArgs& a, hipStream_t stream)
{
    constexpr int NP = 256 / D;            // parents per wave, RX x RY of them (combine_item)
    constexpr int RX = ROW ? NP : NP == 8 ? 4 : 2, RY = NP / RX;
    const int bx = (a.Wp + RX - 1) / RX, by = (a.Hp + RY - 1) / RY;
    const long long items = static_cast<long long>(a.B) * bx * by * a.heads;
    if (items + 3 >= 0x7FFFFFFFLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((bwd_combine_bf16_kernel<D, VA, ROW>), dim3(static_cast<unsigned>((items + 3) / 4)), dim3(4 * kWave), 0,
                       stream, a, bwd16::CombineGrid{make_fastdiv(bx * by), make_fastdiv(bx)}, static_cast<int>(items));
    return hipGetLastError();
}

template <int D>
hipError_t launch_combine_d(const BwdLevelArgs& a, bool variant_a, hipStream_t stream)
{
    if (a.H == 1) return variant_a ? launch_combine<D, true, true>(a, stream) : launch_combine<D, false, true>(a, stream);
    return variant_a ? launch_combine<D, true, false>(a, stream) : launch_combine<D, false, false>(a, stream);
}

// One wave per chunk; the grid is an upper bound of the chunks.
template <int D, bool VA, bool FINEST>
__global__ __launch_bounds__(64) void bwd_key_bf16_kernel(BwdLevelArgs a)
{
    const int n = a.B * a.heads * a.Hp * a.Wp;
    // chunks of neighbouring keys (whose parents overlap) run on one XCD and share its L2: the workgroups that
    // have a chunk are remapped onto contiguous ranges
    const int nchunks = a.coff[n];
    if (static_cast<int>(blockIdx.x) >= nchunks) return;      // whole wave
    const int chunk = __builtin_amdgcn_readfirstlane(xcd_remap(static_cast<int>(blockIdx.x), nchunks));
    extern __shared__ __align__(16) unsigned char smem[];
    const int key = a.chunk_key[chunk];                       // bh * Np + J
    const int first = a.coff[key], nch = a.coff[key + 1] - first;
    const int beg = a.off[key] + (chunk - first) * kKeyGroup;
    bwd16::key_chunk<D, VA, FINEST>(a, chunk, key, nch, beg, min(a.off[key + 1] - beg, kKeyGroup), smem);
}

template <int D, bool VA, bool FINEST>
hipError_t launch_key(const BwdLevelArgs& a, long long max_chunks, hipStream_t stream)
{
    if (max_chunks >= 0x7FFFFFFFLL) return hipErrorInvalidValue;
    constexpr size_t lds = bwd16::wave_bytes<D, 4>();
    hipLaunchKernelGGL((bwd_key_bf16_kernel<D, VA, FINEST>), dim3(static_cast<unsigned>(max_chunks)), dim3(kWave), lds, stream, a);
    return hipGetLastError();
}

template <int D>
hipError_t launch_key_d(const BwdLevelArgs& a, bool variant_a, bool finest, long long max_chunks, hipStream_t stream)
{
    if (variant_a) return finest ? launch_key<D, true, true>(a, max_chunks, stream) : launch_key<D, true, false>(a, max_chunks, stream);
    return finest ? launch_key<D, false, true>(a, max_chunks, stream) : launch_key<D, false, false>(a, max_chunks, stream);
}

}  // namespace

hipError_t launch_bwd_query_bf16(const BwdLevelArgs& a, int d, bool variant_a, bool finest, hipStream_t stream)
{
    if (d == 32) return launch_query_d<32>(a, variant_a, finest, stream);
    if (d == 64) return launch_query_d<64>(a, variant_a, finest, stream);
    return hipErrorInvalidValue;
}

hipError_t launch_bwd_combine_bf16(const BwdLevelArgs& a, int d, bool variant_a, hipStream_t stream)
{
    if (d == 32) return launch_combine_d<32>(a, variant_a, stream);
    if (d == 64) return launch_combine_d<64>(a, variant_a, stream);
    return hipErrorInvalidValue;
}

hipError_t launch_bwd_key_bf16(const BwdLevelArgs& a, int d, bool variant_a, bool finest, long long max_chunks, hipStream_t stream)
{
    if (d == 32) return launch_key_d<32>(a, variant_a, finest, max_chunks, stream);
    if (d == 64) return launch_key_d<64>(a, variant_a, finest, max_chunks, stream);
    return hipErrorInvalidValue;
}

}  // namespace qta
