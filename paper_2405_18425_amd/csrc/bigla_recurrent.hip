// Exact fp32 evaluation of the BiGLA recurrences (Section 4.2.1, Eq. (BiGLA)), token by token.
//
// This is the fp32 path of the library and the path for every head shape the chunkwise MFMA
// kernels do not cover.  A pair of waves owns a strip of columns of one (batch, head) slab's state and
// walks the two directions at the same time from the two ends (exact_sweep.hpp); each parks its partial
// outputs of the first half as fp32 and writes (o_fwd + o_bwd)/2 for the other half.
#include "exact_sweep.hpp"
#include "vig_common.hpp"
#include "vig_kernels.hpp"
#include "vig_timing.hpp"

#include <type_traits>

namespace vig {

namespace {

// kPairs: column strips of one slab per workgroup, so that they find the slab's rows in the compute
// unit's own cache.
template <typename T, int DK, int DV, int kPairs>
__global__ __launch_bounds__(128 * kPairs, 1) void bigla_recurrent_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ g_fwd,
    const T *__restrict__ g_bwd, T *out, float *o_part /* may alias out (fp32) */, int L,
    int heads_token_major /* 0: [B,H,L,d]; H: [B,L,H,d] */, unsigned n_slabs, bool part_in_out)
{
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x)) >> 6, lane = int(threadIdx.x) & 63;
    const unsigned slab = blockIdx.x % n_slabs;
    const int col_block = int(blockIdx.x / n_slabs) * kPairs + (wave >> 1);
    const bool descending = (wave & 1) != 0;
    // first row of the slab and distance between its tokens, in rows of the tensor
    const size_t row0 = slab_first_row(slab, L, heads_token_major);
    const size_t step = heads_token_major ? heads_token_major : 1;
    // the fp32 side buffer is dense [slab][L][DV]; when the partial sums live in `out` they follow it
    float *park = o_part + (part_in_out ? row0 : size_t(slab) * L) * DV;
    column_sweep<T, DK, DV, false>(k + row0 * DK, q + row0 * DK, (descending ? g_bwd : g_fwd) + row0 * DK, v + row0 * DV,
                                   park, out + row0 * DV, step, part_in_out ? step : 1, L, descending, col_block, 1.f,
                                   0.5f, lane);
}

template <typename T, int DK, int DV>
hipError_t launch(const void *q, const void *k, const void *v, const void *gf, const void *gb, void *out,
                  float *o_part, int BH, int L, int heads_token_major, hipStream_t stream)
{
    constexpr int kBlocks = DV / (kStrip * (64 / DK));  // column strips of a slab
    const bool part_in_out = static_cast<void *>(o_part) == out;
    auto run = [&](auto pairs) -> hipError_t {
        constexpr int kPairs = decltype(pairs)::value;
        const long blocks = long(BH) * (kBlocks / kPairs);
        if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
        LaunchTimer timer(kKernelRecurrent, stream);
        hipLaunchKernelGGL((bigla_recurrent_kernel<T, DK, DV, kPairs>), dim3((unsigned)blocks), dim3(128 * kPairs), 0,
                           stream, static_cast<const T *>(q), static_cast<const T *>(k), static_cast<const T *>(v),
                           static_cast<const T *>(gf), static_cast<const T *>(gb), static_cast<T *>(out), o_part, L,
                           heads_token_major, unsigned(BH), part_in_out);
        return hipGetLastError();
    };
    // Few strips: one pair per workgroup, so that they spread over the compute units.  More than one pair
    // for every unit: two per workgroup, which read the slab's rows from memory once.
    if constexpr (kBlocks % 2 == 0)
        if (long(BH) * kBlocks > 256) return run(std::integral_constant<int, 2>{});
    return run(std::integral_constant<int, 1>{});
}

template <typename T, int DK>
hipError_t launch_dv(int dv, const void *q, const void *k, const void *v, const void *gf, const void *gb,
                     void *out, float *o_fwd, int BH, int L, int heads_token_major, hipStream_t stream)
{
    switch (dv) {
        case 16: return launch<T, DK, 16>(q, k, v, gf, gb, out, o_fwd, BH, L, heads_token_major, stream);
        case 32: return launch<T, DK, 32>(q, k, v, gf, gb, out, o_fwd, BH, L, heads_token_major, stream);
        case 64: return launch<T, DK, 64>(q, k, v, gf, gb, out, o_fwd, BH, L, heads_token_major, stream);
    }
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_dk(int dk, int dv, const void *q, const void *k, const void *v, const void *gf,
                     const void *gb, void *out, float *o_fwd, int BH, int L, int heads_token_major, hipStream_t stream)
{
    switch (dk) {
        case 16: return launch_dv<T, 16>(dv, q, k, v, gf, gb, out, o_fwd, BH, L, heads_token_major, stream);
        case 32: return launch_dv<T, 32>(dv, q, k, v, gf, gb, out, o_fwd, BH, L, heads_token_major, stream);
        case 64: return launch_dv<T, 64>(dv, q, k, v, gf, gb, out, o_fwd, BH, L, heads_token_major, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace

size_t bigla_recurrent_workspace_bytes(long BH, int L, int dv, bool is_bf16)
{
    // fp32 runs keep the partial outputs in `out` itself; bf16 runs need an fp32 side buffer
    return is_bf16 ? size_t(BH) * L * dv * sizeof(float) : 0;
}

hipError_t bigla_recurrent_launch(const void *q, const void *k, const void *v, const void *g_fwd,
                                  const void *g_bwd, void *out, long BH, int L, int dk, int dv, bool is_bf16,
                                  int heads_token_major, void *workspace, hipStream_t stream)
{
    if (is_bf16)
        return launch_dk<bf16_t>(dk, dv, q, k, v, g_fwd, g_bwd, out, static_cast<float *>(workspace), int(BH), L,
                                 heads_token_major, stream);
    return launch_dk<float>(dk, dv, q, k, v, g_fwd, g_bwd, out, static_cast<float *>(out), int(BH), L,
                            heads_token_major, stream);
}

}  // namespace vig
