// Gradient of the BiGLA token mixer (Section 4.2.1, Eq. (BiGLA); the paper trains through it,
// Section 5, and prints no gradient formulas), evaluated token by token in fp32 arithmetic.
//
// With do_t = d_out_t / 2 and, per direction, the state S_t = diag(alpha_t) S_{t-/+1} + k_t^T v_t
// and its adjoint A_t = q_t^T do_t + diag(alpha_{t+/-1}) A_{t+/-1} (running against the state),
//     dq_t = S_t do_t^T ,   dk_t = A_t v_t^T ,   dv_t = k_t A_t ,
// each summed over the two directions, and the log-gates of a direction enter the output only
// through differences of their cumulative sums b, so that dLoss/db_t = q_t * dq_t - k_t * dk_t
// (that direction's parts, elementwise) and
//     dg_fwd_s = sum_{t >= s} (q_t * dq^f_t - k_t * dk^f_t) ,
//     dg_bwd_s = sum_{t <= s} (q_t * dq^b_t - k_t * dk^b_t) .
// One launch (exact_sweep.hpp): a pair of waves walks the two directions at the same time, from the two ends.
//   dq, dk, dg : a strip of rows; a wave has the state of one direction and the adjoint of the other, which
//                run the same way, and the gate gradients are running sums of what the pair leaves behind;
//   dv         : a strip of columns of the adjoint.
// This is the exact-arithmetic path for every head shape and both dtypes (bf16 storage, fp32
// arithmetic).  For bf16 with 64-wide values the chunkwise matrix-core kernels run instead, and evaluate the slabs
// whose gates are beyond their range with the same sweeps.
#include "exact_sweep.hpp"
#include "vig_common.hpp"
#include "vig_kernels.hpp"
#include "vig_timing.hpp"

#include <type_traits>

namespace vig {

namespace {

// 12 slabs of 196 tokens, 64 x 64, fp32: 34.8 us (in one part per strip 39.7; a workgroup per 16 rows or columns, tokens through
// LDS, two launches: 54 + 61); 1024 slabs 1.65 ms (2.97), 8192 slabs of 20 tokens in bf16 2.1 ms (12.7).  Bound by its instructions, about 90 a token and wave.
// kPairs: strips of one slab per workgroup.  A slab's strips are first the DK / kRows of dq, dk and dg, then the
// DV / kCols of dv; a workgroup has strips of one kind only, so that its waves meet the same barriers.
template <typename T, int DK, int DV, int kPairs, typename Off, int kParts>
__global__ __launch_bounds__(128 * kPairs * kParts, 1) void bigla_bwd_exact_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ gf,
    const T *__restrict__ gb, const T *__restrict__ d_out, T *__restrict__ dq, T *__restrict__ dk, T *__restrict__ dv,
    T *__restrict__ dgf, T *__restrict__ dgb, float *part_f /* [slabs][L][DK] */, float *part_b /* same */,
    float *part_v /* [slabs][L][DV] */, int L, int heads_token_major /* 0: [B,H,L,d]; H: [B,L,H,d] */, unsigned first_slab,
    unsigned n_slabs /* of this launch */)
{
    constexpr int kRowWork = DK / (kStrip * (64 / DV)) / kPairs;  // workgroups of a slab that take rows
    static_assert(kPairs == 1 || kParts == 1, "one strip's parts per workgroup");
    __shared__ RowStage<DV> stage[2 * kPairs * kParts];
    __shared__ PartStage<kParts, 2> parts;
    const unsigned slab = first_slab + blockIdx.x % n_slabs;
    const int work = int(blockIdx.x / n_slabs);
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x)) >> 6, lane = int(threadIdx.x) & 63;
    const bool descending = (wave & 1) != 0;
    const int pair = kPairs > 1 ? wave >> 1 : 0, part = kParts > 1 ? wave >> 1 : 0;
    const size_t row0 = slab_first_row(slab, L, heads_token_major);
    const size_t step = heads_token_major ? heads_token_major : 1;
    if (work < kRowWork)
        row_sweep<T, DK, DV, Off, kParts>(q + row0 * DK, k + row0 * DK, v + row0 * DV, gf + row0 * DK, gb + row0 * DK, d_out + row0 * DV,
                             dq + row0 * DK, dk + row0 * DK, dgf + row0 * DK, dgb + row0 * DK, part_f + size_t(slab) * L * DK,
                             part_b + size_t(slab) * L * DK, stage[wave], step, L, descending, part, parts, work * kPairs + pair, lane);
    else
        // the adjoint that runs with the wave belongs to the other direction
        column_sweep<T, DK, DV, true, Off, kParts>(q + row0 * DK, k + row0 * DK, (descending ? gf : gb) + row0 * DK, d_out + row0 * DV,
                                      part_v + size_t(slab) * L * DV, dv + row0 * DV, step, 1, L, descending,
                                      part, parts, (work - kRowWork) * kPairs + pair, 0.5f, 1.f, lane);
}

template <typename T, int DK, int DV>
hipError_t launch(const void *q, const void *k, const void *v, const void *gf, const void *gb, const void *d_out,
                  void *dq, void *dk, void *dv, void *dgf, void *dgb, long BH, int L, int heads_token_major,
                  float *ws, hipStream_t stream)
{
    constexpr int kRowStrips = DK / (kStrip * (64 / DV)), kColStrips = DV / (kStrip * (64 / DK));
    float *part_f = ws, *part_b = ws + size_t(BH) * L * DK, *part_v = part_b + size_t(BH) * L * DK;
    auto run = [&](auto pairs, auto offset, auto parts) -> hipError_t {
        constexpr int kPairs = decltype(pairs)::value, kParts = decltype(parts)::value;
        // a launch has fewer than 2^32 work-items (one of more goes wrong without an error): further slabs in another one
        constexpr long kMost = 0xffffffffL / (128 * kParts * (kRowStrips + kColStrips));
        for (long first = 0; first < BH; first += kMost) {
            const long slabs = BH - first < kMost ? BH - first : kMost;
            const long blocks = slabs * ((kRowStrips + kColStrips) / kPairs);
            hipLaunchKernelGGL((bigla_bwd_exact_kernel<T, DK, DV, kPairs, decltype(offset), kParts>), dim3((unsigned)blocks), dim3(128 * kPairs * kParts), 0, stream,
                               static_cast<const T *>(q), static_cast<const T *>(k), static_cast<const T *>(v),
                               static_cast<const T *>(gf), static_cast<const T *>(gb), static_cast<const T *>(d_out),
                               static_cast<T *>(dq), static_cast<T *>(dk), static_cast<T *>(dv), static_cast<T *>(dgf),
                               static_cast<T *>(dgb), part_f, part_b, part_v, L, heads_token_major, unsigned(first),
                               unsigned(slabs));
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    };
    using std::integral_constant;
    if (!tile_fits_32_bits(heads_token_major ? heads_token_major : 1, DK > DV ? DK : DV, sizeof(T)))
        return run(integral_constant<int, 1>{}, size_t{}, integral_constant<int, 1>{});
    // Parts of a strip's tokens (exact_sweep.hpp) while a compute unit has one strip, or two of two parts each.  fp32, us for 1 / 2 /
    // 4 parts: 8 slabs (256 strips, 64 x 64) of 196 tokens 37.8 / 32.9 / 25.8, of 98 22.0 / 20.1 / 15.6, of 56 13.7 / 12.6 / 10.0, of 32
    // 8.4 / 8.0 / 8.3; 12 slabs of 196 39.7 / 34.8 / 44.8, of 17 8.7 / 8.4 / 12.7; 20 (640 strips) of 196 41.9 / 54.7 / 63.5; 128 slabs of
    // 196, 16 x 16, 54.6 / 48.9 / 36.1.  A second part starts to pay at three tiles, 0.90 to 0.98 of one part's time for 17 to 48 tokens (two
    // tiles: 1.04 to 1.25); with 64-wide values, whose sums over the lanes are the longest, at seven (17 to 24 tokens 0.96 to 0.99, 25 to
    // 48 0.96 to 1.04, 49 to 80 0.92 to 1.00).
    const long strips = BH * (kRowStrips + kColStrips);
    if (strips <= 256 && L >= 40) return run(integral_constant<int, 1>{}, 0u, integral_constant<int, 4>{});
    if (strips <= 512 && L > (DV == 64 ? 6 : 2) * kTile) return run(integral_constant<int, 1>{}, 0u, integral_constant<int, 2>{});
    // as in the forward: one pair per workgroup until every compute unit has one
    if constexpr (kRowStrips % 2 == 0 && kColStrips % 2 == 0)
        if (BH * (kRowStrips + kColStrips) > 512) return run(integral_constant<int, 2>{}, 0u, integral_constant<int, 1>{});
    return run(integral_constant<int, 1>{}, 0u, integral_constant<int, 1>{});
}

template <typename T, int DK>
hipError_t launch_dv(int dv_, const void *q, const void *k, const void *v, const void *gf, const void *gb,
                     const void *d_out, void *dq, void *dk, void *dv, void *dgf, void *dgb, long BH, int L,
                     int heads_token_major, float *ws, hipStream_t stream)
{
    switch (dv_) {
        case 16: return launch<T, DK, 16>(q, k, v, gf, gb, d_out, dq, dk, dv, dgf, dgb, BH, L, heads_token_major, ws, stream);
        case 32: return launch<T, DK, 32>(q, k, v, gf, gb, d_out, dq, dk, dv, dgf, dgb, BH, L, heads_token_major, ws, stream);
        case 64: return launch<T, DK, 64>(q, k, v, gf, gb, d_out, dq, dk, dv, dgf, dgb, BH, L, heads_token_major, ws, stream);
    }
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_dk(int dk_, int dv_, const void *q, const void *k, const void *v, const void *gf, const void *gb,
                     const void *d_out, void *dq, void *dk, void *dv, void *dgf, void *dgb, long BH, int L,
                     int heads_token_major, float *ws, hipStream_t stream)
{
    switch (dk_) {
        case 16: return launch_dv<T, 16>(dv_, q, k, v, gf, gb, d_out, dq, dk, dv, dgf, dgb, BH, L, heads_token_major, ws, stream);
        case 32: return launch_dv<T, 32>(dv_, q, k, v, gf, gb, d_out, dq, dk, dv, dgf, dgb, BH, L, heads_token_major, ws, stream);
        case 64: return launch_dv<T, 64>(dv_, q, k, v, gf, gb, d_out, dq, dk, dv, dgf, dgb, BH, L, heads_token_major, ws, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace

size_t bigla_bwd_workspace_bytes(long BH, int L, int dk, int dv, bool is_bf16)
{
    // (part_f, part_b and part_v are 2 dk + dv of these: what callers have asked for and may have written down stays)
    const size_t exact = size_t(BH) * L * (size_t(3) * dk + dv) * sizeof(float);
    return exact + (bigla_bwd_chunk_supported(dk, dv, is_bf16) ? bigla_bwd_chunk_workspace_bytes(BH, L) : 0);
}

constexpr int kChunkwiseMinTokens = 32;

hipError_t bigla_bwd_launch(const void *q, const void *k, const void *v, const void *g_fwd, const void *g_bwd,
                            const void *d_out, void *dq, void *dk, void *dv, void *dg_fwd, void *dg_bwd, long BH, int L,
                            int dk_, int dv_, bool is_bf16, int heads_token_major, bool recurrent_only, void *workspace,
                            hipStream_t stream)
{
    LaunchTimer timer(kKernelBackward, stream);
    char *base = static_cast<char *>(workspace);
    if (bigla_bwd_chunk_supported(dk_, dv_, is_bf16)) {
        float *exact = reinterpret_cast<float *>(base + bigla_bwd_chunk_workspace_bytes(BH, L));
        // The chunkwise kernels evaluate a slab whose gates they cannot carry with the exact form themselves.  Sequences
        // shorter than half a chunk go to the exact kernels altogether: a slab of a few tokens has only a
        // handful of score entries, all of which can be small at once, and the bf16 rounding of the scaled
        // queries and keys (relative to the summands of those entries) is then large against the slab's own
        // gradients -- reproduced on the CPU from the operand roundings alone.
        if (!recurrent_only && L >= kChunkwiseMinTokens)
            return bigla_bwd_chunk_launch(q, k, v, g_fwd, g_bwd, d_out, dq, dk, dv, dg_fwd, dg_bwd, BH, L, dk_,
                                          heads_token_major, base, exact, stream);
        base = reinterpret_cast<char *>(exact);
    }
    float *ws = reinterpret_cast<float *>(base);
    if (is_bf16)
        return launch_dk<bf16_t>(dk_, dv_, q, k, v, g_fwd, g_bwd, d_out, dq, dk, dv, dg_fwd, dg_bwd, BH, L,
                                 heads_token_major, ws, stream);
    return launch_dk<float>(dk_, dv_, q, k, v, g_fwd, g_bwd, d_out, dq, dk, dv, dg_fwd, dg_bwd, BH, L,
                            heads_token_major, ws, stream);
}

}  // namespace vig
