// Building blocks of the exact (token by token, fp32 arithmetic) kernels of the token mixer and its
// gradient (Section 4.2.1, Eq. (BiGLA)).
//
// Every quantity they produce is a readout of a dk x dv matrix that follows a recurrence over the
// tokens: M_t = diag(decay_t) M_prev + (outer product), then a contraction of M_t with a vector over
// one of its dimensions.  The chain from token to token is one fused multiply-add per element, so
// what bounds these kernels is the instructions and the latencies around it.  The mapping keeps both
// out of the chain: a WAVE owns a strip of the matrix, its lanes lie along the contracted dimension
// (64 lanes, or 64 / W strips side by side where that dimension is W = 32 or 16), and a lane holds
// kStrip = 4 elements of the other dimension.  Operands along the lanes are then plain coalesced
// loads into registers, kDepth tiles ahead, with no trip through LDS and no barrier; the products of
// kTile tokens x 4 elements are summed over the lanes together, in a tree that halves the values a lane
// keeps at every level (70 instructions for 32 values over 64 lanes).
// The two directions are walked at the same time by two waves, from the two ends: each parks its
// results for the first half of its way (split at a tile boundary), one barrier, then each adds what the
// other has parked to its own.  For 12 slabs of 196 tokens, 64 x 64, fp32 (a workgroup per slab and one
// direction after the other, tokens through LDS, took 236 us for the forward; a workgroup per 16 rows,
// tokens through LDS, 54 + 61 us for the gradient) see the measurements at the kernels.
// Where the strips leave most of the chip idle, a strip's tokens are cut into kParts parts with a pair of waves
// each.  The matrix is linear in what enters a part, so a wave first walks its part from zero for the matrix it
// leaves and its total decay alone (about half the instructions of the walk with readouts), the waves of a direction
// exchange the two through LDS, and each then walks its part from what the parts before it leave.  The same products
// and sums as in one walk, in fewer steps: the error against fp64 stays what it was.
#pragma once

#include <type_traits>

#include "vig_common.hpp"

namespace vig {

namespace {

constexpr int kStrip = 4;   // matrix elements per lane
constexpr int kTile = 8;    // tokens whose readouts are summed over the lanes together
// Tiles whose operands are in registers or on their way there.  Offsets inside a tile are 32 bits wide (Off = unsigned)
// unless its eight tokens span more than that, which takes millions of token-major heads: with 64 bits they are twice the
// registers, and the chip is full of strips whatever a wave has in flight.
template <typename Off, int kParts>
constexpr int kDepth = sizeof(Off) == 4 ? (kParts > 1 ? 2 : 3) : 1;
inline bool tile_fits_32_bits(size_t step, int width, size_t value_bytes)
{
    return size_t(kTile) * step * width * value_bytes <= 0xffffffffu;
}
constexpr int kVals = kTile * kStrip;

// the partner's value under a DPP permutation that exchanges the two halves of a lane group
template <int CTRL>
__device__ __forceinline__ float dpp_swap(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}

template <int CTRL, int N>
__device__ __forceinline__ void halve_dpp(float (&x)[kVals], bool upper)
{
#pragma unroll
    for (int n = 0; n < N / 2; ++n) {
        const float keep = upper ? x[n + N / 2] : x[n];
        const float send = upper ? x[n] : x[n + N / 2];
        x[n] = keep + dpp_swap<CTRL>(send);
    }
}

// Sums of kVals values over groups of W lanes.  Afterwards lane l holds in x[0] (x[0], x[1] for W = 16)
// the totals of value number lane_value<W>(l) (and the next).
template <int W>
__device__ __forceinline__ void sum_over_lanes(float (&x)[kVals], int lane)
{
    static_assert(kVals == 32 && (W == 64 || W == 32 || W == 16), "levels of the tree");
    if constexpr (W == 64) {
        // v_permlane32_swap: the upper half of the first register against the lower half of the second
#pragma unroll
        for (int n = 0; n < 16; ++n) {
            const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[n]), __float_as_uint(x[n + 16]), false, false);
            x[n] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
        }
    }
    constexpr int kA = W == 64 ? 16 : 32;
    if constexpr (W >= 32) {
        // v_permlane16_swap: odd rows of 16 lanes of the first against even rows of the second
#pragma unroll
        for (int n = 0; n < kA / 2; ++n) {
            const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[n]), __float_as_uint(x[n + kA / 2]), false, false);
            x[n] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
        }
    }
    constexpr int kB = W >= 32 ? kA / 2 : kA;
    halve_dpp<0x140, kB>(x, (lane & 8) != 0);      // row_mirror
    halve_dpp<0x141, kB / 2>(x, (lane & 4) != 0);  // row_half_mirror
    halve_dpp<0x4e, kB / 4>(x, (lane & 2) != 0);   // quad_perm [2,3,0,1]
    if constexpr (kB / 8 >= 2)
        halve_dpp<0xb1, kB / 8>(x, (lane & 1) != 0);  // quad_perm [1,0,3,2]
    else
        x[0] += dpp_swap<0xb1>(x[0]);  // (both lanes of a pair end up with the total)
}

// first value whose total a lane holds, values it holds, and whether it is the one that stores them
template <int W>
__device__ __forceinline__ int lane_value(int lane)
{
    return W == 64 ? lane >> 1 : W == 32 ? (lane & 31) : 2 * (lane & 15);
}
template <int W>
constexpr int kHeld = W == 16 ? 2 : 1;
template <int W>
__device__ __forceinline__ bool lane_stores(int lane)
{
    return W != 64 || (lane & 1) == 0;
}

template <typename T>
__device__ __forceinline__ void load_strip(const T *p, float (&f)[kStrip])
{
    if constexpr (sizeof(T) == 2) {
        const uint2 u = *reinterpret_cast<const uint2 *>(p);
        f[0] = bf16_lo_to_f32(u.x); f[1] = bf16_hi_to_f32(u.x);
        f[2] = bf16_lo_to_f32(u.y); f[3] = bf16_hi_to_f32(u.y);
    } else {
        const float4 u = *reinterpret_cast<const float4 *>(p);
        f[0] = u.x; f[1] = u.y; f[2] = u.z; f[3] = u.w;
    }
}

// byte offset (inside a tile) of element `n` of a row tensor, and what lies there
template <typename T, typename Off>
__device__ __forceinline__ Off at_byte(Off n)
{
    return n * Off(sizeof(T));
}
template <typename T, typename Off>
__device__ __forceinline__ const T *at(const T *base, Off bytes)
{
    return reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + bytes);
}

// Orders this wave's LDS writes before its later LDS reads of what other lanes of the wave wrote (the LDS
// executes one wave's accesses in order; this keeps the compiler from moving them across each other)
__device__ __forceinline__ void lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// alpha = e^g to within an ulp in nine instructions (expf: fifteen): 2^(g log2 e) on the hardware's instruction, with
// the rounding of the product put back to first order.  A log-gate is <= 0; below -150 alpha is zero in fp32.
__device__ __forceinline__ float gate_factor(float g)
{
    const float kHi = 1.44269502162933349609375f, kLo = 1.92596299112661746887e-8f;  // log2 e in two parts
    g = g < -150.f ? -150.f : g;  // (NaN stays)
    const float x = g * kHi;
    const float rest = fmaf(g, kLo, fmaf(g, kHi, -x));
    const float e = __builtin_amdgcn_exp2f(x);
    return fmaf(e, 0.693147182464599609375f * rest, e);
}

// The way of one direction over the tokens of a part (whole tiles of the sequence): tile number n of it covers the tokens
// token(n, 0..kTile-1) in visiting order.  Both directions share the tile boundaries; a ragged last tile belongs to the
// sequence's end.
template <bool kWhole>
struct Way {
    int L, start, tiles;  // first tile of the part and how many it has
    bool descending;
    __device__ __forceinline__ int low(int n) const { return (start + (descending ? tiles - 1 - n : n)) * kTile; }
    // (the same number either way; what the compiler makes of it differs: over the whole sequence the first form takes 0.96 to 0.98 of
    // the second one's time in 257 to 512 strips, in parts 1.00 to 1.04)
    __device__ __forceinline__ int token(int n, int i) const
    {
        if constexpr (kWhole) return descending ? (tiles - 1 - n) * kTile + (kTile - 1 - i) : n * kTile + i;
        return low(n) + (descending ? kTile - 1 - i : i);
    }
    __device__ __forceinline__ bool ragged(int n) const { return low(n) + kTile > L; }
    // offset in a tile of its last token
    __device__ __forceinline__ unsigned last_offset(int n) const { return unsigned(min(kTile - 1, L - 1 - low(n))); }
    // token(n, i) - low(n), clamped to the sequence (always a valid address)
    __device__ __forceinline__ unsigned offset(int n, int i) const
    {
        return unsigned(min(descending ? kTile - 1 - i : i, L - 1 - low(n)));
    }
    // tiles of the first half: what the other direction meets in its second half
    __device__ __forceinline__ int first_half() const { return descending ? tiles - tiles / 2 : tiles / 2; }
};

template <int kParts>
__device__ __forceinline__ Way<kParts == 1> make_way(int L, bool descending, int part)
{
    const int tiles = (L + kTile - 1) / kTile;
    Way<kParts == 1> w;
    w.L = L;
    w.start = tiles * part / kParts;
    w.tiles = tiles * (part + 1) / kParts - w.start;
    w.descending = descending;
    return w;
}

// Calls walk(operands, n) for the tiles first .. last - 1 of a way, with the operands of kDepth tiles requested ahead by fetch
template <typename Operands, int kAhead, typename Fetch, typename Walk>
__device__ __forceinline__ void over_tiles(int first, int last, Fetch fetch, Walk walk)
{
    if (first >= last) return;
    Operands o[kAhead];
#pragma unroll
    for (int d = 0; d < kAhead; ++d) fetch(o[d], first + d);
    int n = first;
    for (; n + kAhead <= last; n += kAhead) {
#pragma unroll
        for (int d = 0; d < kAhead; ++d) {
            walk(o[d], n + d);
            fetch(o[d], n + d + kAhead);
        }
    }
#pragma unroll
    for (int d = 0; d < kAhead - 1; ++d)
        if (n + d < last) walk(o[d], n + d);
}

// What the waves of a strip exchange between its parts: a lane's elements of the matrices a part leaves when nothing enters
// it, and the decay over the part, per direction and part.  kMatrices: 1 for column sweeps alone, 2 where row sweeps use it too.
template <int kParts, int kMatrices>
struct PartStage {
    float4 end[2][kParts][kMatrices][64], decay[2][kParts][kMatrices][64];
};
template <int kMatrices>
struct PartStage<1, kMatrices> {};

// A decay over several tokens, as a product of their factors that is zero only where a factor is: an infinite element of the
// matrix then stays infinite over a part, as it does from token to token.  (The smallest positive number for a product below
// it: the largest finite element adds less than 5e-7.)
constexpr float kLeastFactor = 1.401298464324817e-45f;
__device__ __forceinline__ float joint_factor(float a, float b) { return fmaxf(a * b, fminf(fminf(a, b), kLeastFactor)); }

// M: what enters the wave's part, from what the parts before it on its way leave
template <int kParts, int kMatrices>
__device__ __forceinline__ void enter_part(const PartStage<kParts, kMatrices> &ex, int matrix, bool descending, int part, int lane, float (&M)[kStrip])
{
    const int before = descending ? kParts - 1 - part : part;
    for (int u = 0; u < before; ++u) {
        const int from = descending ? kParts - 1 - u : u;
        const float4 e = ex.end[descending][from][matrix][lane], d = ex.decay[descending][from][matrix][lane];
        M[0] = fmaf(d.x, M[0], e.x);
        M[1] = fmaf(d.y, M[1], e.y);
        M[2] = fmaf(d.z, M[2], e.z);
        M[3] = fmaf(d.w, M[3], e.w);
    }
}

// Readouts over the rows of the matrix: M_t = diag(alpha) M_prev + u_t^T (b_scale * b_t), result_t = r_t M_t, for the
// strip of columns col0 .. (64 / DK strips of four side by side in a wave).  kDelayed false: alpha is the gate of
// the token itself (a state: u = k, b = v, r = q); true: the gate of the token visited before (an adjoint: u = q,
// b = d_out, r = k).  `park`: fp32, dense or strided like the result; result = result_scale * (own + parked).
// One barrier, and one more with several parts, executed by every wave that calls this.  `park` and `result` may be one
// buffer (fp32).
template <typename T, int DK, int DV, bool kDelayed, typename Off = unsigned, int kParts = 1, int kMatrices>
__device__ __forceinline__ void column_sweep(const T *u_rows, const T *r_rows, const T *g_rows, const T *b_rows,
                                             float *park, T *result, size_t step, size_t park_step, int L,
                                             bool descending, int part, PartStage<kParts, kMatrices> &parts, int col_block,
                                             float b_scale, float result_scale, int lane)
{
    constexpr int kGroups = 64 / DK;
    constexpr int kH = kHeld<DK>;
    const auto way = make_way<kParts>(L, descending, part);
    const int ch = lane % DK;
    int col0 = (col_block * kGroups + lane / DK) * kStrip;
    // kept out of the scalar unit where a wave has one strip: scalar loads of the strip's operands, three
    // tiles of them, overflow the scalar registers
    asm("" : "+v"(col0));
    const int held = lane_value<DK>(lane);
    const int held_i = held / kStrip, held_col = col0 + held % kStrip;
    const bool storing = lane_stores<DK>(lane);

    struct Operands {
        float u[kTile], r[kTile], g[kTile], b[kTile][kStrip], other[kH];
    };
    // (delayed: `before` is the gate of the token visited before; what enters a part has it applied already)
    float M[kStrip] = {0.f, 0.f, 0.f, 0.f}, before = 1.f;
    // a whole tile's offsets, the same in every tile (a wave alone on its SIMD pays for scalar address
    // arithmetic as much as for any other instruction)
    Off off_k[kTile], off_v[kTile];
#pragma unroll
    for (int i = 0; i < kTile; ++i) {
        const Off t = Off(descending ? kTile - 1 - i : i) * Off(step);
        off_k[i] = at_byte<T>(t * DK + unsigned(ch));
        off_v[i] = at_byte<T>(t * DV + unsigned(col0));
    }

    // the rows of tile n, readout operands too where kRead
    auto fetch_rows = [&](Operands &o, int n, auto read) __attribute__((always_inline)) {
        const size_t low = size_t(way.low(n));
        const T *u = u_rows + low * step * DK, *r = r_rows + low * step * DK, *g = g_rows + low * step * DK;
        const T *b = b_rows + low * step * DV;
        // (a token past the sequence repeats the last one's offset, so every address is valid)
        const Off last_token = Off(way.last_offset(n)) * Off(step);
        const Off end_k = at_byte<T>(last_token * DK + unsigned(ch)), end_v = at_byte<T>(last_token * DV + unsigned(col0));
#pragma unroll
        for (int i = 0; i < kTile; ++i) {
            const Off tk = min(off_k[i], end_k), tv = min(off_v[i], end_v);
            o.u[i] = io<T>::load(at(u, tk));
            if constexpr (decltype(read)::value) o.r[i] = io<T>::load(at(r, tk));
            o.g[i] = io<T>::load(at(g, tk));
            load_strip(at(b, tv), o.b[i]);
        }
    };
    // tokens past the sequence: nothing enters the matrix (ascending they come last, descending first, when it is still zero)
    auto clear_past_end = [&](Operands &o, int n) __attribute__((always_inline)) {
        if (way.ragged(n)) {
#pragma unroll
            for (int i = 0; i < kTile; ++i) {
                if (way.token(n, i) < L) continue;
                o.u[i] = 0.f;
                o.g[i] = 0.f;
#pragma unroll
                for (int c = 0; c < kStrip; ++c) o.b[i][c] = 0.f;
            }
        }
    };
    auto advance = [&](const Operands &o, int i) __attribute__((always_inline)) {
        const float alpha = gate_factor(o.g[i]);
        const float decay = kDelayed ? before : alpha;
#pragma unroll
        for (int c = 0; c < kStrip; ++c)
            M[c] = fmaf(decay, M[c], o.u[i] * (kDelayed ? b_scale * o.b[i][c] : o.b[i][c]));
        before = alpha;
        return alpha;
    };
    if constexpr (kParts > 1) {
        if (part != (descending ? 0 : kParts - 1)) {  // (nobody enters anything after the last part)
            float total = 1.f, least = 1.f;  // joint_factor of the part's factors, their minimum taken apart
            auto fetch = [&](Operands &o, int n) __attribute__((always_inline)) { fetch_rows(o, min(n, way.tiles - 1), std::false_type{}); };
            auto walk = [&](Operands &o, int n) __attribute__((always_inline)) {
                clear_past_end(o, n);
#pragma unroll
                for (int i = 0; i < kTile; ++i) {
                    const float alpha = advance(o, i);
                    total *= alpha;
                    least = fminf(least, alpha);
                }
            };
            over_tiles<Operands, kDepth<Off, kParts>>(0, way.tiles, fetch, walk);
            total = fmaxf(total, fminf(least, kLeastFactor));
            const float f = kDelayed ? before : 1.f;
            parts.end[descending][part][0][lane] = make_float4(f * M[0], f * M[1], f * M[2], f * M[3]);
            parts.decay[descending][part][0][lane] = make_float4(total, total, total, total);
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kStrip; ++c) M[c] = 0.f;
        before = 1.f;
        enter_part(parts, 0, descending, part, lane, M);
    }

    auto half = [&](int first, int last, bool second) __attribute__((always_inline)) {
        auto fetch = [&](Operands &o, int n) __attribute__((always_inline)) {
            n = min(n, last - 1);  // (past the end: loaded, never used; a branch would make every wait a full one)
            fetch_rows(o, n, std::true_type{});
            if (second) {
                const size_t t = size_t(min(way.token(n, held_i), L - 1));
#pragma unroll
                for (int h = 0; h < kH; ++h) o.other[h] = park[t * park_step * DV + held_col + h];
            }
        };
        auto walk = [&](Operands &o, int n) __attribute__((always_inline)) {
            clear_past_end(o, n);
            float x[kVals];
#pragma unroll
            for (int i = 0; i < kTile; ++i) {
                advance(o, i);
#pragma unroll
                for (int c = 0; c < kStrip; ++c) x[kStrip * i + c] = o.r[i] * M[c];
            }
            sum_over_lanes<DK>(x, lane);
            const int t = way.token(n, held_i);
            if (storing && t < L) {
#pragma unroll
                for (int h = 0; h < kH; ++h) {
                    if (second)
                        io<T>::store(result + size_t(t) * step * DV + held_col + h, result_scale * (o.other[h] + x[h]));
                    else
                        park[size_t(t) * park_step * DV + held_col + h] = x[h];
                }
            }
        };
        over_tiles<Operands, kDepth<Off, kParts>>(first, last, fetch, walk);
    };
    half(0, way.first_half(), false);
    __threadfence_block();
    __syncthreads();
    half(way.first_half(), way.tiles, true);
}

// Inclusive prefix sum over the wave's 64 lanes
__device__ __forceinline__ float wave_scan(float x, int lane)
{
    x = row_scan<0>(x);
#pragma unroll
    for (int row = 1; row < 4; ++row) {
        const float total = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 16 * row - 1));
        x += lane >> 4 == row ? total : 0.f;
    }
    return x;
}

// Gradients that are readouts over the columns: for the strip of rows row0 .. (64 / DV strips of four in a wave) the state
// S of the wave's own direction (dq_t = S_t do_t^T) and the adjoint A that runs the same way, the other
// direction's (dk_t = A_t v_t^T), together: they share every operand.  The ascending wave of a pair has S of the
// forward direction and A of the backward one, the descending wave the other two; where they have
// met, dq and dk are sums of both, and
//   e^f = q * dq^f - k * dk^f ,  e^b = q * dq^b - k * dk^b
// take the place of the parked partial results (part_f, part_b: dense fp32 [L][DK]); their running sums over
// the tokens, descending and ascending, are dg_fwd and dg_bwd.
// Two barriers, and one more with several parts, executed by every wave that calls this.  `stage` is the wave's own LDS.
template <int DV>
struct RowStage {
    // per token of the tile: both gates' factors, k and q of the wave's rows
    float x[kTile][4][kStrip * (64 / DV)];
};

template <typename T, int DK, int DV, typename Off = unsigned, int kParts = 1>
__device__ __forceinline__ void row_sweep(const T *q_rows, const T *k_rows, const T *v_rows, const T *gf_rows,
                                          const T *gb_rows, const T *do_rows, T *dq_rows, T *dk_rows, T *dgf_rows,
                                          T *dgb_rows, float *part_f, float *part_b, RowStage<DV> &stage, size_t step,
                                          int L, bool descending, int part, PartStage<kParts, 2> &parts, int row_block, int lane)
{
    constexpr int kGroups = 64 / DV;
    constexpr int kRows = kStrip * kGroups;   // rows of the wave
    constexpr int kLoads = 2 * kGroups;       // staged values a lane loads per tile
    constexpr int kH = kHeld<DV>;
    const auto way = make_way<kParts>(L, descending, part);
    const int col = lane % DV, grp = lane / DV, first_row = row_block * kRows;
    const int held = lane_value<DV>(lane);
    const int held_i = held / kStrip, held_c = kStrip * grp + held % kStrip;  // token and row (of the wave's) of the totals held
    const bool storing = lane_stores<DV>(lane);
    // the lane's staged values: array (0: gate of S, 1: gate of A, 2: k, 3: q), token and row
    auto staged = [&](int j, int &array, int &i, int &row) __attribute__((always_inline)) {
        const int n = lane + 64 * j;
        array = n / (kTile * kRows);
        i = n / kRows % kTile;
        row = n % kRows;
    };
    const T *staged_rows[kLoads];  // where a lane's staged values come from (row included)
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
        int array, i, row;
        staged(j, array, i, row);
        const T *rows = descending ? gb_rows : gf_rows;
        if (array == 1) rows = descending ? gf_rows : gb_rows;
        if (array == 2) rows = k_rows;
        if (array == 3) rows = q_rows;
        staged_rows[j] = rows + first_row + row;
    }

    struct Operands {
        float v[kTile], d[kTile], s[kLoads], other_f[kH], other_b[kH];
    };
    Off off_v[kTile];  // a whole tile's offsets
#pragma unroll
    for (int i = 0; i < kTile; ++i)
        off_v[i] = at_byte<T>(Off(descending ? kTile - 1 - i : i) * Off(step) * DV + unsigned(col));
    // (`before`: gates of the token visited before; what enters a part has them applied already)
    float S[kStrip] = {0.f, 0.f, 0.f, 0.f}, A[kStrip] = {0.f, 0.f, 0.f, 0.f}, before[kStrip] = {1.f, 1.f, 1.f, 1.f};

    auto fetch_rows = [&](Operands &o, int n) __attribute__((always_inline)) {
        const size_t low = size_t(way.low(n));
        const T *v = v_rows + low * step * DV, *d = do_rows + low * step * DV;
        const Off end_v = at_byte<T>(Off(way.last_offset(n)) * Off(step) * DV + unsigned(col));
#pragma unroll
        for (int i = 0; i < kTile; ++i) {
            const Off t = min(off_v[i], end_v);
            o.v[i] = io<T>::load(at(v, t));
            o.d[i] = io<T>::load(at(d, t));
        }
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            int array, i, row;
            staged(j, array, i, row);
            o.s[j] = io<T>::load(staged_rows[j] + (low + way.offset(n, i)) * step * DK);
        }
    };
    // the staged values of tile n, gates as factors, into the wave's stage (and in o.s); tokens past the sequence: nothing
    // enters the matrices
    auto put_stage = [&](Operands &o, int n) __attribute__((always_inline)) {
        const bool ragged = way.ragged(n);
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            int array, i, row;
            staged(j, array, i, row);
            float x = array < 2 ? gate_factor(o.s[j]) : o.s[j];
            if (ragged && way.token(n, i) >= L) x = array < 2 ? 1.f : 0.f;
            stage.x[i][array][row] = o.s[j] = x;
        }
        if (ragged) {
#pragma unroll
            for (int i = 0; i < kTile; ++i)
                if (way.token(n, i) >= L) o.v[i] = o.d[i] = 0.f;
        }
        lds_order();
    };
    // both matrices through token i of the tile in the stage; d: d_out / 2
    auto advance = [&](float v, float d, int i) __attribute__((always_inline)) {
        float gs[kStrip], ga[kStrip], kr[kStrip], qr[kStrip];
        load_strip(&stage.x[i][0][kStrip * grp], gs);
        load_strip(&stage.x[i][1][kStrip * grp], ga);
        load_strip(&stage.x[i][2][kStrip * grp], kr);
        load_strip(&stage.x[i][3][kStrip * grp], qr);
#pragma unroll
        for (int c = 0; c < kStrip; ++c) {
            S[c] = fmaf(gs[c], S[c], kr[c] * v);
            A[c] = fmaf(before[c], A[c], qr[c] * d);
            before[c] = ga[c];
        }
    };
    if constexpr (kParts > 1) {
        if (part != (descending ? 0 : kParts - 1)) {  // (nobody enters anything after the last part)
            // the decay over the part: a lane multiplies the factors it stages (the first half of its values), then every
            // lane those of its rows
            float total[kLoads / 2];
#pragma unroll
            for (int j = 0; j < kLoads / 2; ++j) total[j] = 1.f;
            auto fetch = [&](Operands &o, int n) __attribute__((always_inline)) { fetch_rows(o, min(n, way.tiles - 1)); };
            auto walk = [&](Operands &o, int n) __attribute__((always_inline)) {
                put_stage(o, n);
#pragma unroll
                for (int j = 0; j < kLoads / 2; ++j) total[j] = joint_factor(total[j], o.s[j]);
#pragma unroll
                for (int i = 0; i < kTile; ++i) advance(o.v[i], 0.5f * o.d[i], i);
                lds_order();
            };
            // (one value a lane in a stage of 64-wide columns: the upper half of the wave stages the second gate)
            static_assert(kLoads / 2 * 64 == 2 * kTile * kRows, "the first half of the staged values are the gates");
            over_tiles<Operands, kDepth<Off, kParts>>(0, way.tiles, fetch, walk);
#pragma unroll
            for (int j = 0; j < kLoads / 2; ++j) {
                int array, i, row;
                staged(j, array, i, row);
                stage.x[i][array][row] = total[j];
            }
            lds_order();
            float decay[2][kStrip];
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                load_strip(&stage.x[0][m][kStrip * grp], decay[m]);
#pragma unroll
                for (int i = 1; i < kTile; ++i) {
                    float f[kStrip];
                    load_strip(&stage.x[i][m][kStrip * grp], f);
#pragma unroll
                    for (int c = 0; c < kStrip; ++c) decay[m][c] = joint_factor(decay[m][c], f[c]);
                }
                parts.decay[descending][part][m][lane] = make_float4(decay[m][0], decay[m][1], decay[m][2], decay[m][3]);
            }
            parts.end[descending][part][0][lane] = make_float4(S[0], S[1], S[2], S[3]);
            parts.end[descending][part][1][lane] = make_float4(before[0] * A[0], before[1] * A[1], before[2] * A[2], before[3] * A[3]);
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kStrip; ++c) {
            S[c] = A[c] = 0.f;
            before[c] = 1.f;
        }
        enter_part(parts, 0, descending, part, lane, S);
        enter_part(parts, 1, descending, part, lane, A);
    }

    auto half = [&](int first, int last, bool second) __attribute__((always_inline)) {
        auto fetch = [&](Operands &o, int n) __attribute__((always_inline)) {
            n = min(n, last - 1);  // (past the end: loaded, never used; a branch would make every wait a full one)
            fetch_rows(o, n);
            if (second) {
                const size_t t = size_t(way.low(n)) + way.offset(n, held_i);
#pragma unroll
                for (int h = 0; h < kH; ++h) {
                    o.other_f[h] = part_f[t * DK + first_row + held_c + h];
                    o.other_b[h] = part_b[t * DK + first_row + held_c + h];
                }
            }
        };
        auto walk = [&](Operands &o, int n) __attribute__((always_inline)) {
            put_stage(o, n);
            float xq[kVals], xk[kVals];
#pragma unroll
            for (int i = 0; i < kTile; ++i) {
                const float d = 0.5f * o.d[i], v = o.v[i];
                advance(v, d, i);
#pragma unroll
                for (int c = 0; c < kStrip; ++c) {
                    xq[kStrip * i + c] = S[c] * d;
                    xk[kStrip * i + c] = A[c] * v;
                }
            }
            sum_over_lanes<DV>(xq, lane);
            sum_over_lanes<DV>(xk, lane);
            const int t = way.token(n, held_i);
            if (storing && t < L) {
#pragma unroll
                for (int h = 0; h < kH; ++h) {
                    const size_t dense = size_t(t) * DK + first_row + held_c + h;
                    // the parked halves lie where the other wave finds them by direction: the state's in
                    // part_f, the adjoint's in part_b
                    if (!second) {
                        part_f[dense] = xq[h];
                        part_b[dense] = xk[h];
                        continue;
                    }
                    const float kk = stage.x[held_i][2][held_c + h], qq = stage.x[held_i][3][held_c + h];
                    const size_t o_row = size_t(t) * step * DK + first_row + held_c + h;
                    io<T>::store(dq_rows + o_row, o.other_f[h] + xq[h]);
                    io<T>::store(dk_rows + o_row, o.other_b[h] + xk[h]);
                    // own state with the other wave's adjoint: the own state's direction, and the reverse
                    const float e_state = qq * xq[h] - kk * o.other_b[h];
                    const float e_adjoint = qq * o.other_f[h] - kk * xk[h];
                    part_f[dense] = descending ? e_adjoint : e_state;
                    part_b[dense] = descending ? e_state : e_adjoint;
                }
            }
            lds_order();  // the totals' reads of the stage before the next tile's writes
        };
        over_tiles<Operands, kDepth<Off, kParts>>(first, last, fetch, walk);
    };
    half(0, way.first_half(), false);
    __threadfence_block();
    __syncthreads();
    half(way.first_half(), way.tiles, true);
    __threadfence_block();
    __syncthreads();

    // running sums, a lane per token: dg_fwd from the last token on (descending wave), dg_bwd from the first
    const float *part_sums = descending ? part_f : part_b;
    T *dg = descending ? dgf_rows : dgb_rows;
    // (several parts: a wave takes its share of each strip's rows)
    constexpr int kMine = kStrip / kParts;
    static_assert(kStrip % kParts == 0, "rows of a strip shared out to the parts");
    for (int r0 = part * kMine; r0 < kRows; r0 += kStrip) {
        float run[kMine];
#pragma unroll
        for (int c = 0; c < kMine; ++c) run[c] = 0.f;
        for (int n = 0; n < L; n += 64) {
            const int t = descending ? L - 1 - n - lane : n + lane;
            const bool live = n + lane < L;
            float e[kStrip] = {0.f, 0.f, 0.f, 0.f};
            if (live) {
                const float *p = part_sums + size_t(t) * DK + first_row + r0;
                if constexpr (kMine == kStrip)
                    load_strip(p, e);
                else
#pragma unroll
                    for (int c = 0; c < kMine; ++c) e[c] = p[c];
            }
#pragma unroll
            for (int c = 0; c < kMine; ++c) {
                e[c] = run[c] + wave_scan(e[c], lane);
                run[c] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(e[c]), 63));
                if (live) io<T>::store(dg + size_t(t) * step * DK + first_row + r0 + c, e[c]);
            }
        }
    }
}

}  // namespace

}  // namespace vig
