// The gradients of one chunk of 64 tokens (Section 4.2.1, Eq. (BiGLA); the formulas are at the head of bigla_bwd_chunk.hip), both
// directions together.  A workgroup takes a chunk, a wave a tile of 16 tokens.
//
// For a wave's own tokens the other tokens of the chunk lie on two sides, and each side belongs to one direction: as keys of
// the own queries the tokens before them are the forward direction's and those after them the backward one's, as
// queries of the own keys the other way round.  So a strip of d_out v^T is formed, split into bf16 halves and contracted
// once for both directions, on either side with that side's scaled keys (or queries); only the wave's own pair of tiles
// meets both, its split scores masked as packed words.  The scores P of the two directions add up to one strip in the same
// way.  X, Y and dv follow one another, so that a wave holds one of them at a time.
//
// Lane (r, g) of the wave of tile w holds 16 channels (or columns) of token 16w + r in operand order, channel 32 (n / 8) + 8 g +
// n % 8 in slot n: two 16-byte pieces of the row.  The rows of an MFMA's A operand are assigned to channels so that accumulator
// row 4g + e of tile ct is slot 4ct + e: what a wave contracts against the other tokens is in its registers as an operand, and results
// leave from the registers.  What other waves contract over lies in LDS as whole rows, 128 (64 for 32-wide keys) bytes without
// padding, their pieces permuted by row (grad_place).
//
// With Y = dP^T q~ + v A'^T the gate gradient is dg_u = sum_{t >= u} (q~ * X - k~ * Y)_t + sum_t k~_t * (v A'^T)_t + rowsum(S_in * A')
// (mirrored backward): one running sum, and a term that is the same for every token.  Its summands take q~ and k~ as the contractions saw
// them (rounded to bf16): term by term they are then sums over pairs of tokens that the rounding perturbs once, instead of long
// sums whose differences no longer cancel.
//
// What bounds it: the memory traffic (1920 bytes a head and token, 377 MB at 48 slabs of 4096 tokens, 70 us at the rate of a copy) and the
// instructions (156 MFMAs and about 1500 vector instructions a wave, two waves a SIMD) take about as long as each other.  A kernel that
// took one direction after the other, every strip masked to half its tiles, issued 208 and 2320 with eleven barriers for
// these five, and a gradient call took 185 us against 159 here (48 slabs of 4096 tokens), 93 / 79 (384 of 196), 48.5 / 43 (15 of
// 1961), 39 / 32.5 (48 of 1024, 32-wide keys).  Measured on the way: state matrices read from memory as operands, row by row,
// instead of through LDS 196 us; three workgroups a compute unit at 168 registers, some of them spilled, 175 against 162.
#pragma once

namespace vig {

namespace {

constexpr int kTiles = kC / 16;
constexpr unsigned kTileBytes = 2048;  // 16 rows of 128 bytes

// the chunk kernel's LDS: rows of values and output gradients; scaled queries (first the states entering the chunk) and keys (first the
// gates); adjoint matrices; sums.  70 KB, two workgroups a compute unit (45 KB and three for 32-wide keys).
template <int kCt>
struct GradLds {
    static constexpr unsigned kKeyTile = 512u * kCt;  // 16 rows of keys, queries or gates
    static constexpr unsigned v = 0, d = v + kTiles * kTileBytes, qf = d + kTiles * kTileBytes, qb = qf + kTiles * kKeyTile;
    static constexpr unsigned kf = qb + kTiles * kKeyTile, kb = kf + kTiles * kKeyTile, kMatrix = 2048u * kCt;
    static constexpr unsigned af = kb + kTiles * kKeyTile, ab = af + kMatrix, scans = ab + kMatrix;
    // fp32 [direction][..][64]: per wave the total of the dg summands that are summed up over the chunk, and of those that every token
    // takes; the last row of a block of the second kind is rowsum(S_in * A')
    static constexpr unsigned kRow = 4 * kD, every = scans + 2 * kTiles * kRow, bytes = every + 2 * (kTiles + 1) * kRow;
};

extern __shared__ __align__(16) unsigned char g_grad_lds[];

// byte offset of 16-byte piece `piece` of row `row` in a 16-row tile of kBytes-byte rows (see bigla_short.hpp, which uses the same
// placement): the 16 rows of a tile read by piece, and the 4 x 4 pieces of a transposing read, fall into different banks
template <int kBytes>
__device__ __forceinline__ unsigned grad_place(int row, int piece)
{
    const int f = kBytes == 128 ? ((row & 6) | ((row >> 3) & 1)) : (((row >> 1) & 2) | ((row >> 3) & 1));
    return unsigned(row * kBytes + ((piece ^ f) << 4));
}

__device__ __forceinline__ bf16x8 grad_b128(unsigned off) { return *reinterpret_cast<const bf16x8 *>(g_grad_lds + off); }
__device__ __forceinline__ s16x4 grad_tr(unsigned off) { return lds_read_tr(reinterpret_cast<const uint16_t *>(g_grad_lds + off)); }
__device__ __forceinline__ float *grad_sums(unsigned off) { return reinterpret_cast<float *>(g_grad_lds + off); }
__device__ __forceinline__ bf16x8 as_operand(const u32x4 &x) { return __builtin_bit_cast(bf16x8, x); }
__device__ __forceinline__ bf16x8 as_operand(const uint2 &a, const uint2 &b) { return __builtin_bit_cast(bf16x8, make_uint4(a.x, a.y, b.x, b.y)); }

// c + a.lo * b.lo + a.hi * b.hi on bf16 pairs
__device__ __forceinline__ float grad_dot2(uint32_t a, uint32_t b, float c)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
}

// Sums over the 16 lanes r of N values per lane (16 or 8): lane r ends up with the total of value r (of r / 2 for 8)
template <int N>
__device__ __forceinline__ float sum_over_tokens(float (&x)[N], int r)
{
    auto halve = [&](auto ctrl, int n, bool upper) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < n / 2; ++i) {
            const float keep = upper ? x[i + n / 2] : x[i], send = upper ? x[i] : x[i + n / 2];
            x[i] = keep + dpp_swap<decltype(ctrl)::value>(send);
        }
    };
    using std::integral_constant;
    halve(integral_constant<int, 0x140>{}, N, (r & 8) != 0);      // row_mirror
    halve(integral_constant<int, 0x141>{}, N / 2, (r & 4) != 0);  // row_half_mirror
    halve(integral_constant<int, 0x4e>{}, N / 4, (r & 2) != 0);   // quad_perm [2,3,0,1]
    if constexpr (N == 16)
        halve(integral_constant<int, 0xb1>{}, 2, (r & 1) != 0);   // quad_perm [1,0,3,2]
    else
        x[0] += dpp_swap<0xb1>(x[0]);
    return x[0];
}

// x = h + l on bf16 pairs
__device__ __forceinline__ void split_scores(const f32x4 &x, uint2 &h, uint2 &l)
{
    h = pack4(x);
    const f32x4 u = unpack4(h);
    l = pack4(f32x4{x[0] - u[0], x[1] - u[1], x[2] - u[2], x[3] - u[3]});
}
__device__ __forceinline__ uint2 operator&(const uint2 &a, const uint2 &b) { return make_uint2(a.x & b.x, a.y & b.y); }

struct GradRows {  // the tensors of the whole call; a slab's rows are put behind a buffer resource where they are used
    const void *q, *k, *v, *gf, *gb, *dout;
    void *dq, *dk, *dv, *dgf, *dgb;
    size_t first;
    int L, heads_token_major;
};

// mats: the chunk's four state matrices; nothing enters the first chunk from the left and the last one from the right, and those
// matrices are not read.  Every wave of the workgroup calls this (barriers).
template <int kCt>
__device__ __forceinline__ void chunk_gradients(const GradRows &io, const uint16_t *mats, unsigned t0, bool first_chunk, bool last_chunk,
                                                int w, int lane, int tid)
{
    constexpr int kKs = kCt / 2;         // K-steps of a contraction over channels
    constexpr int kKeyBytes = 32 * kCt;  // row of keys, queries or gates
    typedef GradLds<kCt> at;
    const int r = lane & 15, g = lane >> 4;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};

    // ---- lane offsets in a tile: whole pieces of row r, and the 4 x 4 patches of the transposing reads (rows 4g .. 4g + 3)
    const unsigned row_v[2] = {grad_place<128>(r, g), grad_place<128>(r, 4 + g)};
    const unsigned row_k[2] = {grad_place<kKeyBytes>(r, g), kKs > 1 ? grad_place<kKeyBytes>(r, 4 + g) : 0u};
    const unsigned patch_v[2] = {grad_place<128>(4 * g + (r >> 2), r & 3), grad_place<128>(4 * g + (r >> 2), 4 + (r & 3))};
    const unsigned patch_k[2] = {grad_place<kKeyBytes>(4 * g + (r >> 2), r & 3), kKs > 1 ? grad_place<kKeyBytes>(4 * g + (r >> 2), 4 + (r & 3)) : 0u};
    const unsigned own_v_rows = unsigned(w) * kTileBytes, own_k_rows = unsigned(w) * at::kKeyTile;

    // A operand over the tokens of tiles a and a + 1: channel tile ct of the key-wide rows (columns, of the 64-wide ones)
    auto tokens_k = [&](unsigned region, int a, int ct) __attribute__((always_inline)) {
        const unsigned off = patch_k[ct >> 1] + unsigned(a) * at::kKeyTile + (region + 8u * unsigned(ct & 1));
        return join(grad_tr(off), grad_tr(off + at::kKeyTile));
    };
    auto tokens_v = [&](unsigned region, int a, int ct) __attribute__((always_inline)) {
        const unsigned off = patch_v[ct >> 1] + unsigned(a) * kTileBytes + (region + 8u * unsigned(ct & 1));
        return join(grad_tr(off), grad_tr(off + kTileBytes));
    };
    // A state matrix lies in LDS as rows of 128 bytes, placed like the 64-wide rows.  Its rows as the A operand of a contraction over
    // its columns: accumulator row r of channel tile ct is matrix row 32 (ct / 2) + 8 (r / 4) + 4 (ct % 2) + r % 4.
    auto matrix_rows = [&](unsigned region, int ct, int kk) __attribute__((always_inline)) {
        const int row = 8 * (r >> 2) + 4 * (ct & 1) + (r & 3);
        return grad_b128(region + unsigned(ct >> 1) * 2u * kTileBytes + unsigned(row >> 4) * kTileBytes + grad_place<128>(row & 15, 4 * kk + g));
    };
    // pieces of a state matrix that this thread carries from memory to LDS: number tid and, of 64 rows, tid + 256
    constexpr int kPieces = kCt / 2;
    const __amdgpu_buffer_rsrc_t mats_rows = slab_resource(mats, unsigned(4 * kMat * sizeof(uint16_t)));
    auto matrix_piece = [&](int kind, int i) __attribute__((always_inline)) {
        const bool zeros = kind == 0 || kind == 3 ? first_chunk : last_chunk;
        return __builtin_amdgcn_raw_buffer_load_b128(mats_rows, zeros ? kBeyond : unsigned(kind * 2 * int(kMat) + (tid + i * kThreads) * 16), 0, 0);
    };
    auto put_matrix_piece = [&](unsigned region, int i, const u32x4 &x) __attribute__((always_inline)) {
        const int row = (tid >> 3) & 15;
        *reinterpret_cast<u32x4 *>(g_grad_lds + region + unsigned(tid >> 7) * kTileBytes + unsigned(i) * 2u * kTileBytes + grad_place<128>(row, tid & 7)) = x;
    };
    auto keys = [&](const void *p) __attribute__((always_inline)) { return slab_rows(p, io.first, io.L, io.heads_token_major, 16 * kCt); };
    auto values = [&](const void *p) __attribute__((always_inline)) { return slab_rows(p, io.first, io.L, io.heads_token_major); };
    const unsigned row_off = (t0 + 16u * unsigned(w) + unsigned(r));
    auto load_piece = [&](const SlabRows &rows, int kk) __attribute__((always_inline)) {
        return __builtin_amdgcn_raw_buffer_load_b128(rows.rsrc, row_off * rows.pitch + 16u * unsigned(g) + 64u * unsigned(kk), 0, 0);
    };
    auto store_pieces = [&](const SlabRows &rows, const f32x4 *x, int tiles) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < tiles / 2; ++kk) {
            const uint2 a = pack4(x[2 * kk]), b = pack4(x[2 * kk + 1]);
            __builtin_amdgcn_raw_buffer_store_b128(u32x4{a.x, a.y, b.x, b.y}, rows.rsrc, row_off * rows.pitch + 16u * unsigned(g) + 64u * unsigned(kk), 0, 0);
        }
    };

    // whole rows of the wave's tile, 8 rows of 128 (16 of 64) bytes per instruction, to LDS
    const int vrow = lane >> 3, vpiece = lane & 7, krow = kKs > 1 ? lane >> 3 : lane >> 2, kpiece = kKs > 1 ? lane & 7 : lane & 3;
    auto load_rows = [&](const SlabRows &rows, int i, int row, int piece) __attribute__((always_inline)) {
        return __builtin_amdgcn_raw_buffer_load_b128(rows.rsrc, (t0 + 16u * unsigned(w) + 8u * unsigned(i) + unsigned(row)) * rows.pitch + 16u * unsigned(piece), 0, 0);
    };

    // ---- rows in: gates to where the scaled keys will be, the states entering the chunk to where the scaled queries will be
    u32x4 rq[kKs], rk[kKs], own_v[2], own_d[2];
    {
        u32x4 rgf[kKs], rgb[kKs], rv[2], rd[2], st[2][kPieces], ad[2][kPieces];
#pragma unroll
        for (int i = 0; i < kKs; ++i) {
            rgf[i] = load_rows(keys(io.gf), i, krow, kpiece);
            rgb[i] = load_rows(keys(io.gb), i, krow, kpiece);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            rv[i] = load_rows(values(io.v), i, vrow, vpiece);
            rd[i] = load_rows(values(io.dout), i, vrow, vpiece);
        }
#pragma unroll
        for (int dir = 0; dir < 2; ++dir)
#pragma unroll
            for (int i = 0; i < kPieces; ++i) {
                st[dir][i] = matrix_piece(2 * dir, i);
                ad[dir][i] = matrix_piece(2 * dir + 1, i);
            }
#pragma unroll
        for (int kk = 0; kk < kKs; ++kk) {
            rq[kk] = load_piece(keys(io.q), kk);
            rk[kk] = load_piece(keys(io.k), kk);
        }
#pragma unroll
        for (int i = 0; i < kKs; ++i) {
            const unsigned off = own_k_rows + grad_place<kKeyBytes>(8 * i + krow, kpiece);
            *reinterpret_cast<u32x4 *>(g_grad_lds + at::kf + off) = rgf[i];
            *reinterpret_cast<u32x4 *>(g_grad_lds + at::kb + off) = rgb[i];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const unsigned off = own_v_rows + grad_place<128>(8 * i + vrow, vpiece);
            *reinterpret_cast<u32x4 *>(g_grad_lds + at::v + off) = rv[i];
            *reinterpret_cast<u32x4 *>(g_grad_lds + at::d + off) = rd[i];
        }
#pragma unroll
        for (int dir = 0; dir < 2; ++dir)
#pragma unroll
            for (int i = 0; i < kPieces; ++i) {
                put_matrix_piece(dir == 0 ? at::qf : at::qb, i, st[dir][i]);
                put_matrix_piece(dir == 0 ? at::af : at::ab, i, ad[dir][i]);
                // rowsum(S_in * A'): a dot product of pieces, then over the eight lanes of a row
                float sum = 0.f;
#pragma unroll
                for (int j = 0; j < 4; ++j) sum = grad_dot2(st[dir][i][j], ad[dir][i][j], sum);
                sum += dpp_swap<0x141>(sum);  // row_half_mirror
                sum += dpp_swap<0x4e>(sum);
                sum += dpp_swap<0xb1>(sum);
                if ((lane & 7) == 0) grad_sums(at::every)[(dir * (kTiles + 1) + kTiles) * kD + (tid >> 3) + 32 * i] = sum;
            }
    }
    __syncthreads();  // gates, values, output gradients, states visible

    // masks of packed values, rows 4g + e (token of a tile) against column r (the own token): those up to the own token, and from it on
    uint2 upto, from;
    {
        uint32_t lo[4], up[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            lo[e] = 4 * g + e <= r ? 0xffffu : 0u;
            up[e] = 4 * g + e >= r ? 0xffffu : 0u;
        }
        upto = make_uint2(lo[0] | lo[1] << 16, lo[2] | lo[3] << 16);
        from = make_uint2(up[0] | up[1] << 16, up[2] | up[3] << 16);
    }
    // the same for tile i of the chunk: tokens before the own one and itself, and after it and itself (w is the same in every lane)
    auto word = [](bool all, bool diagonal, uint32_t m) { return all ? 0xffffffffu : diagonal ? m : 0u; };
    auto before = [&](int i) __attribute__((always_inline)) { return make_uint2(word(i < w, i == w, upto.x), word(i < w, i == w, upto.y)); };
    auto after = [&](int i) __attribute__((always_inline)) { return make_uint2(word(i > w, i == w, from.x), word(i > w, i == w, from.y)); };

    f32x4 Ef[kCt], Eb[kCt];  // 1/2 exp(b): the queries carry the 1/2 of d_out / 2 (as the adjoint matrices do)
    f32x4 Xf[kCt], Xb[kCt];
    u32x4 pqf[kKs], pqb[kKs], own_kf[kKs], own_kb[kKs];
    {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            own_v[kk] = *reinterpret_cast<const u32x4 *>(g_grad_lds + at::v + own_v_rows + row_v[kk]);
            own_d[kk] = *reinterpret_cast<const u32x4 *>(g_grad_lds + at::d + own_v_rows + row_v[kk]);
        }
        // ---- cumulative gates: a product with a 0/1 triangle
        const uint2 one = make_uint2(0x3F803F80u, 0x3F803F80u);
        bf16x8 tri_f[2], tri_b[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            tri_f[p] = as_operand(before(2 * p) & one, before(2 * p + 1) & one);
            tri_b[p] = as_operand(after(2 * p) & one, after(2 * p + 1) & one);
        }
#pragma unroll
        for (int kk = 0; kk < kKs; ++kk) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int ct = 2 * kk + h;
                const f32x4 Bf = mfma(tokens_k(at::kf, 2, ct), tri_f[1], mfma(tokens_k(at::kf, 0, ct), tri_f[0], zero));
                const f32x4 Bb = mfma(tokens_k(at::kb, 2, ct), tri_b[1], mfma(tokens_k(at::kb, 0, ct), tri_b[0], zero));
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    const float q0 = bf16_lo_to_f32(rq[kk][2 * h + d]), q1 = bf16_hi_to_f32(rq[kk][2 * h + d]);
                    const float k0 = bf16_lo_to_f32(rk[kk][2 * h + d]), k1 = bf16_hi_to_f32(rk[kk][2 * h + d]);
                    const float f0 = Bf[2 * d] * kLog2e, f1 = Bf[2 * d + 1] * kLog2e, b0 = Bb[2 * d] * kLog2e, b1 = Bb[2 * d + 1] * kLog2e;
                    Ef[ct][2 * d] = fast_exp2(f0 - 1.f);
                    Ef[ct][2 * d + 1] = fast_exp2(f1 - 1.f);
                    Eb[ct][2 * d] = fast_exp2(b0 - 1.f);
                    Eb[ct][2 * d + 1] = fast_exp2(b1 - 1.f);
                    pqf[kk][2 * h + d] = pack2(q0 * Ef[ct][2 * d], q1 * Ef[ct][2 * d + 1]);
                    pqb[kk][2 * h + d] = pack2(q0 * Eb[ct][2 * d], q1 * Eb[ct][2 * d + 1]);
                    own_kf[kk][2 * h + d] = pack2(k0 * fast_exp2(-f0), k1 * fast_exp2(-f1));
                    own_kb[kk][2 * h + d] = pack2(k0 * fast_exp2(-b0), k1 * fast_exp2(-b1));
                }
            }
        }
        // what the states contribute to X: do S_in^T
#pragma unroll
        for (int ct = 0; ct < kCt; ++ct) {
            Xf[ct] = mfma(matrix_rows(at::qf, ct, 1), as_operand(own_d[1]), mfma(matrix_rows(at::qf, ct, 0), as_operand(own_d[0]), zero));
            Xb[ct] = mfma(matrix_rows(at::qb, ct, 1), as_operand(own_d[1]), mfma(matrix_rows(at::qb, ct, 0), as_operand(own_d[0]), zero));
        }
    }
    __syncthreads();  // every wave is through with the gates and the states
    {
#pragma unroll
        for (int kk = 0; kk < kKs; ++kk) {
            const unsigned off = own_k_rows + row_k[kk];
            *reinterpret_cast<u32x4 *>(g_grad_lds + at::qf + off) = pqf[kk];
            *reinterpret_cast<u32x4 *>(g_grad_lds + at::qb + off) = pqb[kk];
            *reinterpret_cast<u32x4 *>(g_grad_lds + at::kf + off) = own_kf[kk];
            *reinterpret_cast<u32x4 *>(g_grad_lds + at::kb + off) = own_kb[kk];
        }
    }
    __syncthreads();  // scaled queries and keys visible

    // scores of tiles a and a + 1 against the own tokens, rows from `region` (64 wide), as two bf16 halves
    struct Split {
        uint2 h[2], l[2];
    };
    auto strip = [&](unsigned region, int a, const u32x4 (&own)[2]) __attribute__((always_inline)) {
        Split s;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const unsigned off = unsigned(a) * kTileBytes + (region + unsigned(half) * kTileBytes);
            const f32x4 x = mfma(grad_b128(row_v[1] + off), as_operand(own[1]), mfma(grad_b128(row_v[0] + off), as_operand(own[0]), zero));
            split_scores(x, s.h[half], s.l[half]);
        }
        return s;
    };
    auto add_strip = [&](unsigned region, int a, const Split &s, f32x4 (&acc)[kCt]) __attribute__((always_inline)) {
        const bf16x8 h = as_operand(s.h[0], s.h[1]), l = as_operand(s.l[0], s.l[1]);
#pragma unroll
        for (int ct = 0; ct < kCt; ++ct) {
            const bf16x8 x = tokens_k(region, a, ct);
            acc[ct] = mfma(x, h, mfma(x, l, acc[ct]));
        }
    };
    // The strip of `rows` against `own`, contracted on the side before the own tokens with `below`, into acc_below, which `turn` then takes,
    // and on the side after them with `above`, into acc_above.  The own pair of tiles meets both sides, the other pair one.
    const int own_pair = w & 2;
    const uint2 mask_before[2] = {before(own_pair), before(own_pair + 1)}, mask_after[2] = {after(own_pair), after(own_pair + 1)};
    auto both_sides = [&](unsigned rows, const u32x4 (&own)[2], unsigned below, unsigned above, f32x4 (&acc_below)[kCt], f32x4 (&acc_above)[kCt],
                          auto turn) __attribute__((always_inline)) {
        if (own_pair != 0) add_strip(below, 0, strip(rows, 0, own), acc_below);
        {
            const Split s = strip(rows, own_pair, own);
            auto masked = [&](const uint2 (&m)[2]) { return Split{{s.h[0] & m[0], s.h[1] & m[1]}, {s.l[0] & m[0], s.l[1] & m[1]}}; };
            add_strip(below, own_pair, masked(mask_before), acc_below);
            add_strip(above, own_pair, masked(mask_after), acc_above);
        }
        turn();
        if (own_pair == 0) add_strip(above, 2, strip(rows, 2, own), acc_above);
    };

    // slots 4ct .. 4ct + 3 of the own scaled query
    auto own_query = [&](unsigned region, int ct) __attribute__((always_inline)) {
        return unpack4(*reinterpret_cast<const uint2 *>(g_grad_lds + region + own_k_rows + row_k[ct >> 1] + 8u * unsigned(ct & 1)));
    };
    f32x4 ef[kCt], eb[kCt];  // dg summands: q~ * X - k~ * Y
    {
        f32x4 dq[kCt];
        // X: dP k~ + do S_in^T, the own tokens as queries
        both_sides(at::v, own_d, at::kf, at::kb, Xf, Xb, [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int ct = 0; ct < kCt; ++ct) {
                const f32x4 qs = own_query(at::qf, ct);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    ef[ct][e] = qs[e] * Xf[ct][e];
                    dq[ct][e] = Ef[ct][e] * Xf[ct][e];
                }
            }
        });
#pragma unroll
        for (int ct = 0; ct < kCt; ++ct) {
            const f32x4 qs = own_query(at::qb, ct);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                eb[ct][e] = qs[e] * Xb[ct][e];
                dq[ct][e] = fmaf(Eb[ct][e], Xb[ct][e], dq[ct][e]);
            }
        }
        store_pieces(keys(io.dq), dq, kCt);


        // Y: v A'^T + dP^T q~, the own tokens as keys.  The first part alone goes into the sums that every token takes.
        f32x4 dk[kCt], Yf[kCt], Yb[kCt];
        auto adjoint_part = [&](int dir, const u32x4 (&ks)[kKs], f32x4 (&Y)[kCt]) __attribute__((always_inline)) {
            float x[4 * kCt];
#pragma unroll
            for (int ct = 0; ct < kCt; ++ct) {
                Y[ct] = mfma(matrix_rows(dir == 0 ? at::af : at::ab, ct, 1), as_operand(own_v[1]), mfma(matrix_rows(dir == 0 ? at::af : at::ab, ct, 0), as_operand(own_v[0]), zero));
                const f32x4 kv = unpack4(make_uint2(ks[ct >> 1][2 * (ct & 1)], ks[ct >> 1][2 * (ct & 1) + 1]));
#pragma unroll
                for (int e = 0; e < 4; ++e) x[4 * ct + e] = kv[e] * Y[ct][e];
            }
            const float total = sum_over_tokens<4 * kCt>(x, r);
            const int n = kCt == 4 ? r : r >> 1, ct = n >> 2;
            grad_sums(at::every)[(dir * (kTiles + 1) + w) * kD + 32 * (ct >> 1) + 8 * g + 4 * (ct & 1) + (n & 3)] = total;
        };
        adjoint_part(1, own_kb, Yb);
        adjoint_part(0, own_kf, Yf);
        both_sides(at::d, own_v, at::qb, at::qf, Yb, Yf, [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int ct = 0; ct < kCt; ++ct) {
                const f32x4 ks = unpack4(make_uint2(own_kb[ct >> 1][2 * (ct & 1)], own_kb[ct >> 1][2 * (ct & 1) + 1]));
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    eb[ct][e] = fmaf(-ks[e], Yb[ct][e], eb[ct][e]);
                    dk[ct][e] = __builtin_amdgcn_rcpf(Eb[ct][e]) * Yb[ct][e];
                }
            }
        });
#pragma unroll
        for (int ct = 0; ct < kCt; ++ct) {
            const f32x4 ks = unpack4(make_uint2(own_kf[ct >> 1][2 * (ct & 1)], own_kf[ct >> 1][2 * (ct & 1) + 1]));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ef[ct][e] = fmaf(-ks[e], Yf[ct][e], ef[ct][e]);
                dk[ct][e] = 0.5f * fmaf(__builtin_amdgcn_rcpf(Ef[ct][e]), Yf[ct][e], dk[ct][e]);
            }
        }
        store_pieces(keys(io.dk), dk, kCt);

        // running sums of the summands over the wave's 16 tokens, from the far side of each direction
#pragma unroll
        for (int ct = 0; ct < kCt; ++ct) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ef[ct][e] = row_scan<1>(ef[ct][e]);
                eb[ct][e] = row_scan<0>(eb[ct][e]);
            }
            float *sum = grad_sums(at::scans) + w * kD + 32 * (ct >> 1) + 8 * g + 4 * (ct & 1);
            if (r == 0) *reinterpret_cast<f32x4 *>(sum) = ef[ct];
            if (r == 15) *reinterpret_cast<f32x4 *>(sum + kTiles * kD) = eb[ct];
        }
    }
    // dv = P^T do + k~ A': the scores of the own keys, both directions in one strip
    f32x4 V[4];
    {
        // over the matrix's rows (channels in operand order): rows 32kk + 8g .. + 7, two patches
        const unsigned patch_m[2] = {grad_place<128>(8 * (g & 1) + (r >> 2), r & 3), grad_place<128>(8 * (g & 1) + 4 + (r >> 2), r & 3)};
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
            V[ct] = zero;
#pragma unroll
            for (int kk = 0; kk < kKs; ++kk)
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const unsigned base = (m == 0 ? at::af : at::ab) + unsigned(2 * kk + (g >> 1)) * kTileBytes + 8u * unsigned(ct & 1);
                    const unsigned flip = 64u * unsigned(ct >> 1);
                    const bf16x8 a = join(grad_tr(base + (patch_m[0] ^ flip)), grad_tr(base + (patch_m[1] ^ flip)));
                    V[ct] = mfma(a, as_operand(m == 0 ? own_kf[kk] : own_kb[kk]), V[ct]);
                }
        }
    }
    auto scores = [&](unsigned region, int tile, const u32x4 (&own)[kKs]) __attribute__((always_inline)) {
        const unsigned off = unsigned(tile) * at::kKeyTile + region;
        f32x4 p = mfma(grad_b128(off + row_k[0]), as_operand(own[0]), zero);
        if (kKs > 1) p = mfma(grad_b128(off + row_k[kKs - 1]), as_operand(own[kKs - 1]), p);
        return p;
    };
    auto add_values = [&](int a, const f32x4 &pa, const f32x4 &pb) __attribute__((always_inline)) {
        Split s;
        split_scores(pa, s.h[0], s.l[0]);
        split_scores(pb, s.h[1], s.l[1]);
        const bf16x8 h = as_operand(s.h[0], s.h[1]), l = as_operand(s.l[0], s.l[1]);
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
            const bf16x8 x = tokens_v(at::d, a, ct);
            V[ct] = mfma(x, h, mfma(x, l, V[ct]));
        }
    };
    if (own_pair != 0)
        add_values(0, scores(at::qb, 0, own_kb), scores(at::qb, 1, own_kb));
    else
        add_values(2, scores(at::qf, 2, own_kf), scores(at::qf, 3, own_kf));
    {
        f32x4 s[2];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int tile = own_pair + half;
            const f32x4 x = scores(at::qb, tile, own_kb), y = scores(at::qf, tile, own_kf);
            const int own = 16 * (w - tile) + r;  // the own token, counted from the tile's first
#pragma unroll
            for (int e = 0; e < 4; ++e) s[half][e] = (4 * g + e <= own ? x[e] : 0.f) + (4 * g + e >= own ? y[e] : 0.f);
        }
        add_values(own_pair, s[0], s[1]);
    }
    store_pieces(values(io.dv), V, 4);

    __syncthreads();  // the waves' sums are visible
    // what the running sums of each wave start from, in place
    if (tid < 2 * 16 * kCt) {
        const int dir = tid / (16 * kCt), ch = tid % (16 * kCt);
        const float *every = grad_sums(at::every) + dir * (kTiles + 1) * kD + ch;
        float *scan = grad_sums(at::scans) + dir * kTiles * kD + ch;
        float run = every[kTiles * kD], own[kTiles];
#pragma unroll
        for (int u = 0; u < kTiles; ++u) {
            run += every[u * kD];
            own[u] = scan[(dir == 0 ? kTiles - 1 - u : u) * kD];
        }
#pragma unroll
        for (int u = 0; u < kTiles; ++u) {
            scan[(dir == 0 ? kTiles - 1 - u : u) * kD] = run;
            run += own[u];
        }
    }
    __syncthreads();  // starting values visible
#pragma unroll
    for (int ct = 0; ct < kCt; ++ct) {
        const float *sum = grad_sums(at::scans) + w * kD + 32 * (ct >> 1) + 8 * g + 4 * (ct & 1);
        const f32x4 sf = *reinterpret_cast<const f32x4 *>(sum), sb = *reinterpret_cast<const f32x4 *>(sum + kTiles * kD);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            ef[ct][e] += sf[e];
            eb[ct][e] += sb[e];
        }
    }
    store_pieces(keys(io.dgf), ef, kCt);
    store_pieces(keys(io.dgb), eb, kCt);
}

}  // namespace

}  // namespace vig
