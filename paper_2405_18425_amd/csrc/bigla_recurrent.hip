// Exact fp32 evaluation of the BiGLA recurrences (Section 4.2.1, Eq. (BiGLA)), token by token.
//
// This is the fp32 path of the library and the path for every head shape the chunkwise MFMA
// kernels do not cover.  For few slabs a pair of waves owns a strip of columns of one (batch, head)
// slab's state and walks the two directions at the same time from the two ends (exact_sweep.hpp); each parks its partial
// outputs of the first half as fp32 and writes (o_fwd + o_bwd)/2 for the other half.  For many, a workgroup owns a slab.
#include "exact_sweep.hpp"
#include "vig_common.hpp"
#include "vig_kernels.hpp"
#include "vig_timing.hpp"

#include <type_traits>

namespace vig {

namespace {

// ---- many slabs: a workgroup per slab --------------------------------------------------------------
// One direction after the other; thread (j, s) holds rows [s*DK/4, (s+1)*DK/4) of column j, so a token costs DK/4 fused
// decay-update-readout steps per thread plus a 4-lane reduction, and a token's rows are loaded, and its gates
// exponentiated, once per slab (a pair of waves does that for every strip of four columns again).  Tokens are staged
// through LDS 16 at a time.
namespace staged {

constexpr int kSplit = 4;   // threads sharing one state column
constexpr int kTile = 16;   // tokens staged per LDS tile

template <typename T, int DK, int DV>
__global__ __launch_bounds__(DV *kSplit) void bigla_recurrent_staged_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ g_fwd,
    const T *__restrict__ g_bwd, T *out, float *o_fwd /* may alias out (fp32) */, int L,
    int heads_token_major /* 0: [B,H,L,d]; H: [B,L,H,d] */, bool o_fwd_in_out)
{
    constexpr int R = DK / kSplit;
    constexpr int NT = DV * kSplit;
    __shared__ float sq[kTile][DK], sk[kTile][DK], sa[kTile][DK], sv[kTile][DV];

    const int tid = threadIdx.x;
    const int j = tid / kSplit, s = tid % kSplit, c0 = s * R;
    const size_t slab = blockIdx.x;
    // first row of the slab and distance between its tokens, in rows of the tensor
    const size_t row0 = slab_first_row(unsigned(slab), L, heads_token_major);
    const size_t step = heads_token_major ? heads_token_major : 1;
    q += row0 * DK;
    k += row0 * DK;
    g_fwd += row0 * DK;
    g_bwd += row0 * DK;
    v += row0 * DV;
    out += row0 * DV;
    // the fp32 side buffer is dense [slab][L][DV]; when the partial sums live in `out` they follow it
    o_fwd += (o_fwd_in_out ? row0 : slab * size_t(L)) * DV;
    const size_t fwd_step = o_fwd_in_out ? step : 1;

    float S[R];

    for (int dir = 0; dir < 2; ++dir) {
        const T *g = dir == 0 ? g_fwd : g_bwd;
#pragma unroll
        for (int r = 0; r < R; ++r) S[r] = 0.f;
        const int ntiles = (L + kTile - 1) / kTile;
        for (int it = 0; it < ntiles; ++it) {
            const int tile = dir == 0 ? it : ntiles - 1 - it;
            const int t0 = tile * kTile;
            const int n = min(kTile, L - t0);
            __syncthreads();
            for (int e = tid; e < n * DK; e += NT) {
                const int tt = e / DK, c = e % DK;
                const size_t off = size_t(t0 + tt) * step * DK + c;
                sq[tt][c] = io<T>::load(q + off);
                sk[tt][c] = io<T>::load(k + off);
                sa[tt][c] = expf(io<T>::load(g + off));
            }
            for (int e = tid; e < n * DV; e += NT) {
                const int tt = e / DV, c = e % DV;
                sv[tt][c] = io<T>::load(v + size_t(t0 + tt) * step * DV + c);
            }
            __syncthreads();
            for (int i = 0; i < n; ++i) {
                const int tt = dir == 0 ? i : n - 1 - i;
                const float vj = sv[tt][j];
                float acc = 0.f;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    // S_t = diag(alpha_t) S_{t -/+ 1} + k_t^T v_t ;  o_t = q_t S_t
                    S[r] = fmaf(sa[tt][c0 + r], S[r], sk[tt][c0 + r] * vj);
                    acc = fmaf(sq[tt][c0 + r], S[r], acc);
                }
                acc += __shfl_xor(acc, 1);
                acc += __shfl_xor(acc, 2);
                if (s == 0) {
                    const size_t o = size_t(t0 + tt) * step * DV + j, of = size_t(t0 + tt) * fwd_step * DV + j;
                    if (dir == 0)
                        o_fwd[of] = acc;
                    else
                        io<T>::store(out + o, 0.5f * (o_fwd[of] + acc));
                }
            }
        }
    }
}

}  // namespace staged

// ---- few slabs: a pair of waves per strip of columns -------------------------------------------------
// kPairs: column strips of one slab per workgroup, so that they find the slab's rows in the compute
// unit's own cache.
template <typename T, int DK, int DV, int kPairs, int kParts>
__global__ __launch_bounds__(128 * kPairs * kParts, 1) void bigla_recurrent_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ g_fwd,
    const T *__restrict__ g_bwd, T *out, float *o_part /* may alias out (fp32) */, int L,
    int heads_token_major /* 0: [B,H,L,d]; H: [B,L,H,d] */, unsigned n_slabs, bool part_in_out)
{
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x)) >> 6, lane = int(threadIdx.x) & 63;
    static_assert(kPairs == 1 || kParts == 1, "one strip's parts per workgroup");
    __shared__ PartStage<kParts, 1> parts;
    const unsigned slab = blockIdx.x % n_slabs;
    const int col_block = int(blockIdx.x / n_slabs) * kPairs + (kPairs > 1 ? wave >> 1 : 0);
    const bool descending = (wave & 1) != 0;
    // first row of the slab and distance between its tokens, in rows of the tensor
    const size_t row0 = slab_first_row(slab, L, heads_token_major);
    const size_t step = heads_token_major ? heads_token_major : 1;
    // the fp32 side buffer is dense [slab][L][DV]; when the partial sums live in `out` they follow it
    float *park = o_part + (part_in_out ? row0 : size_t(slab) * L) * DV;
    column_sweep<T, DK, DV, false, unsigned, kParts>(k + row0 * DK, q + row0 * DK, (descending ? g_bwd : g_fwd) + row0 * DK,
                                                     v + row0 * DV, park, out + row0 * DV, step, part_in_out ? step : 1, L,
                                                     descending, kParts > 1 ? wave >> 1 : 0, parts, col_block, 1.f, 0.5f, lane);
}

// A pair of waves per strip does about 1.7 times the work of the workgroup per slab, in a sixth of the time while the chip
// is not full of strips: 16 slabs of 196 tokens, 64 x 64, fp32: 25 us against 191; 192: 109 / 241; 256: 137 / 246; 1024 (16384
// strips): 550 / 323.  Short sequences fill it less well.  The limits are where the pairs are still no slower in any of the
// nine head shapes, in fp32 and bf16 (time of the pairs over that of the workgroups, mean and largest of the shapes): 5120 strips of 400,
// 196, 128, 100, 64 tokens 0.63 / 0.82, 0.72 / 1.00, 0.74 / 1.00, 0.84 / 1.15, 0.91 / 1.23; 4096 of 100, 80, 64: 0.71 / 0.97, 0.68 / 0.90,
// 0.79 / 1.11; 3072 of 64: 0.66 / 0.96; 2048 of 49, 20, 16, 8: 0.65 / 0.93, 0.82 / 1.02, 0.83 / 0.94, 1.10 / 1.34; 1024 of 8: 0.68 / 0.84.
inline bool take_pairs(long strips, int L)
{
    return strips <= (L >= 128 ? 5120 : L >= 80 ? 4096 : L >= 64 ? 3072 : L >= 16 ? 2048 : 1024);
}

template <typename T, int DK, int DV>
hipError_t launch(const void *q, const void *k, const void *v, const void *gf, const void *gb, void *out,
                  float *o_part, int BH, int L, int heads_token_major, hipStream_t stream)
{
    constexpr int kBlocks = DV / (kStrip * (64 / DK));  // column strips of a slab
    if (!take_pairs(long(BH) * kBlocks, L)) {
        LaunchTimer timer(kKernelRecurrent, stream);
        hipLaunchKernelGGL((staged::bigla_recurrent_staged_kernel<T, DK, DV>), dim3(BH), dim3(DV * staged::kSplit), 0, stream,
                           static_cast<const T *>(q), static_cast<const T *>(k), static_cast<const T *>(v),
                           static_cast<const T *>(gf), static_cast<const T *>(gb), static_cast<T *>(out), o_part, L,
                           heads_token_major, static_cast<void *>(o_part) == out);
        return hipGetLastError();
    }
    const bool part_in_out = static_cast<void *>(o_part) == out;
    auto run = [&](auto pairs, auto parts) -> hipError_t {
        constexpr int kPairs = decltype(pairs)::value, kParts = decltype(parts)::value;
        const long blocks = long(BH) * (kBlocks / kPairs);
        if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
        LaunchTimer timer(kKernelRecurrent, stream);
        hipLaunchKernelGGL((bigla_recurrent_kernel<T, DK, DV, kPairs, kParts>), dim3((unsigned)blocks), dim3(128 * kPairs * kParts), 0,
                           stream, static_cast<const T *>(q), static_cast<const T *>(k), static_cast<const T *>(v),
                           static_cast<const T *>(gf), static_cast<const T *>(gb), static_cast<T *>(out), o_part, L,
                           heads_token_major, unsigned(BH), part_in_out);
        return hipGetLastError();
    };
    using std::integral_constant;
    // A strip per compute unit at most, of sequences long enough for a walk over a quarter of them to pay for the one that
    // finds what enters it: four parts.  The walks are bound by the instructions their SIMD can issue, so with two strips on
    // a compute unit the extra ones cost more than the shorter way gains.  fp32, us for 1 / 2 / 4 parts: 12 slabs (192 strips, 64 x 64) of
    // 196 tokens 23.3 / 23.2 / 20.5, of 98 14.3 / 14.6 / 13.3, of 56 9.7 / 9.5 / 8.1, of 32 5.8 / 6.0 / 6.1; 20 slabs (320 strips) of 196
    // 26.2 / 30.9 / 37.5; one slab of 1024 104 / 88 / 68.  Not for ten tiles, which are parts of two, three, two and three: 15
    // slabs of 72 / 80 / 88 tokens 11.0 / 11.2 / 12.6 in one part, 10.4 / 12.0 / 12.1 in four.
    if (long(BH) * kBlocks <= 256 && L >= 40 && (L + kTile - 1) / kTile != 10) return run(integral_constant<int, 1>{}, integral_constant<int, 4>{});
    // Few strips: one pair per workgroup, so that they spread over the compute units.  More than one pair
    // for every unit: two per workgroup, which read the slab's rows from memory once.
    if constexpr (kBlocks % 2 == 0)
        if (long(BH) * kBlocks > 256) return run(integral_constant<int, 2>{}, integral_constant<int, 1>{});
    return run(integral_constant<int, 1>{}, integral_constant<int, 1>{});
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
