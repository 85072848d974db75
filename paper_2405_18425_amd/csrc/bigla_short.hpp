// BiGLA forward (Section 4.2.1, Eq. (BiGLA)) for sequences of up to 256 tokens, bf16, dv = 64, dk = 64 or 32: the
// whole sequence is one chunk.  The kernel with two 16-token tiles to a wave, which is given 65 to 256 tokens in at least 128 slabs
// (bigla_tile.hpp has the one with a tile to a wave; wave_per_tile says which runs).  With b_t (c_t) the forward (backward) cumulative log-gate of the sequence, referred to
// the middle of the sequence,
//   out_t = 1/2 sum_{i <= t} (q_t exp(b_t) . k_i exp(-b_i)) v_i + 1/2 sum_{i >= t} (q_t exp(c_t) . k_i exp(-c_i)) v_i ,
// so there are no states at all: no second pass over k, v and the gates, no workspace traffic, no walk from chunk to
// chunk.  What the longer products cost in matrix instructions (all 16 x 16 tiles of the L x L score matrix) is what
// the states of the chunked form cost (readouts, updates): at L = 196 about 1070 against 1056 MFMAs per slab.
//
// One workgroup holds one slab (or two short ones): keys scaled for both directions and values in LDS, 3 x 128
// bytes per token, two workgroups per CU up to L = 208.  A wave owns 32 tokens (two 16-token tiles): their cumulative
// gates (products with a 0/1 triangle, as in the chunked kernels; the waves' totals are exchanged through LDS and enter
// as the accumulators' initial values), exponentials, scaled queries (registers) and keys (LDS), then their rows of the
// score matrix, two key tiles at a time: scores, mask on the diagonal tiles, hi + lo split, P.V.  Every key tile and
// value tile read from LDS serves two query tiles.  q and k come straight into operand layout (lane (r, g): two 16-byte
// pieces of token r), the value columns are assigned to matrix rows so that a lane ends up with 16 consecutive columns
// of its token, and nothing is bounced through LDS.  LDS rows are 128 (64) bytes without padding, their 16-byte pieces
// permuted by row so that the accesses of 16 lanes fall into different banks.
//
// A slab in which some 64-token stretch decays by more than kMildRange in a channel takes the range-safe form of
// bigla_chunk.hip, tile by tile (short_slab_safe), inside the same launch.
//
// Measured (kernel trace): 384 slabs of 196 tokens, 57.8 MB: 23.0 us (the chunked kernel that walks a slab twice in one
// launch: 32.0 us); 192 slabs: 14.7 us (23.2).
// What bounds it: with two workgroups per CU the phases of one overlap those of the other, and a SIMD then spends about
// equal times on the exponentials and scalings (24 vector instructions and 4 exponentials per 64 elements of q and k)
// and on matrix instructions; a lone workgroup is a chain of 25 000 cycles: 6000 until the rows arrive, 5000 for the
// totals and their exchange, 4000 - 7000 for the scalings, 7500 for the products.
//
// This file is part of the translation unit of bigla_chunk.hip.
#pragma once

namespace vig {

namespace {

constexpr int kShortTokens = 256;  // longest sequence
constexpr int kShortTiles = kShortTokens / 16;
constexpr int kShortWaves = 8;     // waves per workgroup at most

extern __shared__ __align__(16) unsigned char g_short_lds[];

// Placement of 16-byte piece `piece` of row `row` in a tile of kBytes-byte rows: rows whose 16-byte accesses meet in
// one instruction (16 rows, same piece) and rows of a transposing read (4 or 8 rows, 32 bytes each) use distinct banks.
template <int kBytes>
__device__ __forceinline__ unsigned key_place(int row, int piece)
{
    const int f = kBytes == 128 ? ((row & 6) | ((row >> 3) & 1)) : (((row >> 1) & 2) | ((row >> 3) & 1));
    return unsigned(row * kBytes + ((piece ^ f) << 4));
}
__device__ __forceinline__ unsigned value_place(int row, int piece) { return unsigned(row * 128 + ((piece ^ ((row >> 1) & 7)) << 4)); }

__device__ __forceinline__ s16x4 short_tr(unsigned off) { return lds_read_tr(reinterpret_cast<const uint16_t *>(g_short_lds + off)); }
__device__ __forceinline__ bf16x8 short_b128(unsigned off) { return *reinterpret_cast<const bf16x8 *>(g_short_lds + off); }

// LDS of one slab: keys scaled forward, keys scaled backward, values.  The per-wave gate totals, and the offsets made
// from them, live in the value rows until those are written.
template <int kDk>
struct ShortSlab {
    static constexpr int kKeyBytes = 2 * kDk;
    unsigned kf, kb, v;
    __host__ __device__ static constexpr unsigned bytes(int n_tiles) { return unsigned(n_tiles) * 16u * (2u * kKeyBytes + 128u); }
    __device__ __forceinline__ ShortSlab(int slot, int n_tiles)
    {
        kf = unsigned(slot) * bytes(n_tiles);
        kb = kf + unsigned(n_tiles) * 16u * kKeyBytes;
        v = kb + unsigned(n_tiles) * 16u * kKeyBytes;
    }
};

// values of tile `tile` (16 whole rows) into LDS
__device__ __forceinline__ void short_put_values(unsigned v_base, int tile, int lane, const StagedRows &s)
{
#pragma unroll
    for (int t = 0; t < 2; ++t)
        *reinterpret_cast<uint4 *>(g_short_lds + v_base + tile * 2048 + value_place(8 * t + (lane >> 3), lane & 7)) = s.p[t];
}

// the lane's pieces of 16-token tile `tile` of a query or key tensor, in operand order
template <int kDk>
__device__ __forceinline__ Row16 short_operand_rows(__amdgpu_buffer_rsrc_t rows, unsigned pitch, int tile, int r, int g)
{
    const unsigned off = unsigned(16 * tile + r) * pitch + 16u * unsigned(g);
    Row16 x;
    const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(rows, off, 0, 0);
    x.p[0] = make_uint4(a.x, a.y, a.z, a.w);
    x.p[1] = make_uint4(0u, 0u, 0u, 0u);
    if (kDk == kD) {
        const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(rows, off + 64u, 0, 0);
        x.p[1] = make_uint4(b.x, b.y, b.z, b.w);
    }
    return x;
}

// O[jt][e]: column 16g + 4jt + e of the lane's token
__device__ __forceinline__ void short_store(__amdgpu_buffer_rsrc_t out, unsigned pitch, int tile, int r, int g, const f32x4 (&O)[4])
{
    const unsigned off = unsigned(16 * tile + r) * pitch + 32u * unsigned(g);
    const uint2 a = pack4(O[0]), b = pack4(O[1]), c = pack4(O[2]), d = pack4(O[3]);
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{a.x, a.y, b.x, b.y}, out, off, 0, 0);
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{c.x, c.y, d.x, d.y}, out, off + 16u, 0, 0);
}

// lane's offset of value column group jt in a tile: patch position 4j + e' is column 16j + 4jt + e'
__device__ __forceinline__ unsigned short_value_off(int jt, int r, int g)
{
    return value_place(4 * g + (r >> 2), 2 * (r & 3) + (jt >> 1)) + 8u * unsigned(jt & 1);
}

// The range-safe form of one slab (the algebra is in bigla_chunk.hip: cumulative gates local to a 16-token tile, keys
// decayed to the edge of their own tile, queries from the start of theirs, whole-tile factors in between, diagonal
// operands referred to the middle of the tile and split into bf16 pairs).  Takes the place of everything after the
// second barrier of the kernel, with the same one barrier left to pass.  eb: the slab's whole-tile decay factors,
// [direction][tile][channel], in the workspace.
template <int kDk, bool kTm>
__device__ __attribute__((noinline)) void short_slab_safe(
    const uint16_t *q_all, const uint16_t *k_all, const uint16_t *v_all, const uint16_t *gf_all, const uint16_t *gb_all,
    uint16_t *out_all, float *eb, long slab, int slot, int w, int n_waves, int L, int n_tiles, int heads)
{
    constexpr int kKs = kDk / 32;
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const SlabIo<kTm, kDk> io(q_all, k_all, v_all, gf_all, gb_all, out_all, slab, L, heads);
    const ShortSlab<kDk> at(slot, n_tiles);
    // (as global memory: a generic pointer's loads count with those of LDS, and every wait for LDS would wait for them)
    typedef __attribute__((address_space(1))) f32x4 Factors;
    auto factors = [&](int dir, int tile) { return (Factors *)(eb + (dir * kShortTiles + tile) * kD) + 2 * g; };
    auto load_factors = [&](int dir, int tile, f32x4 (&f)[4]) {
        const Factors *p = factors(dir, tile);
        f[0] = p[0]; f[1] = p[1]; f[2] = p[8]; f[3] = p[9];
    };
#pragma unroll 1
    for (int tile = w; tile < n_tiles; tile += n_waves) {
        float kf[16], F[16], EB[16];
        unpack16(short_operand_rows<kDk>(io.k, io.key_pitch, tile, r, g), kf);
#pragma unroll
        for (int dir = 0; dir < 2; ++dir) {
            if (dir == 0)
                gate_factors_state<0>(short_operand_rows<kDk>(io.gf, io.key_pitch, tile, r, g), F, EB);
            else
                gate_factors_state<1>(short_operand_rows<kDk>(io.gb, io.key_pitch, tile, r, g), F, EB);
            if (r == 0) {
                Factors *p = factors(dir, tile);
#pragma unroll
                for (int h = 0; h < 4; ++h) p[8 * (h >> 1) + (h & 1)] = f32x4{EB[4 * h], EB[4 * h + 1], EB[4 * h + 2], EB[4 * h + 3]};
            }
#pragma unroll
            for (int n = 0; n < 16; ++n) F[n] *= kf[n];
            const unsigned base = (dir == 0 ? at.kf : at.kb) + tile * 16 * ShortSlab<kDk>::kKeyBytes;
#pragma unroll
            for (int kk = 0; kk < kKs; ++kk)
                *reinterpret_cast<bf16x8 *>(g_short_lds + base + key_place<2 * kDk>(r, 4 * kk + g)) = pack8(F + 8 * kk);
        }
    }
#pragma unroll 1
    for (int tile = w; tile < n_tiles; tile += n_waves)
        short_put_values(at.v, tile, lane, load_rows(io.v, lane_rows<kD>(0, lane, io.pitch), 16u * tile));
    __syncthreads();  // keys, values and factors visible
#pragma unroll 1
    for (int tile = w; tile < n_tiles; tile += n_waves) {
        float qf[16], kf[16], cum[2][16], tmp[16];
        unpack16(short_operand_rows<kDk>(io.q, io.key_pitch, tile, r, g), qf);
        unpack16(short_operand_rows<kDk>(io.k, io.key_pitch, tile, r, g), kf);
#pragma unroll
        for (int n = 0; n < 16; ++n) qf[n] *= 0.5f;
        f32x4 diag[2];
#pragma unroll
        for (int dir = 0; dir < 2; ++dir) {
            float X[16], Y[16], F[16], Emid[16], EB[16];
            if (dir == 0)
                gate_factors<0>(short_operand_rows<kDk>(io.gf, io.key_pitch, tile, r, g), r, X, Y, F, Emid, EB);
            else
                gate_factors<1>(short_operand_rows<kDk>(io.gb, io.key_pitch, tile, r, g), r, X, Y, F, Emid, EB);
            f32x4 p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < kKs; ++kk) {
                bf16x8 kh, kl, qh, ql;
#pragma unroll
                for (int n = 0; n < 8; ++n) tmp[n] = kf[8 * kk + n] * Y[8 * kk + n];
                pack8_split(tmp, kh, kl);
#pragma unroll
                for (int n = 0; n < 8; ++n) tmp[n] = qf[8 * kk + n] * X[8 * kk + n];
                pack8_split(tmp, qh, ql);
                p = mfma(kh, qh, mfma(kl, qh, mfma(kh, ql, p)));
            }
            diag[dir] = p;
#pragma unroll
            for (int n = 0; n < 16; ++n) cum[dir][n] = qf[n] * X[n] * Emid[n];  // decay since the tile's near edge
        }
        f32x4 O[4];
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) O[jt] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto add_tile = [&](const f32x4 &p, int I) {  // O += V^T P^T for key tile I, P as hi + lo
            uint2 h, l;
            split4(p, h, l);
#pragma unroll
            for (int jt = 0; jt < 4; ++jt) {
                const s16x4 a = short_tr(at.v + I * 2048 + short_value_off(jt, r, g));
                O[jt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, __builtin_bit_cast(s16x4, l), O[jt], 0, 0, 0);
                O[jt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, __builtin_bit_cast(s16x4, h), O[jt], 0, 0, 0);
            }
        };
        {
            f32x4 p;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = 4 * g + e;
                p[e] = (i <= r ? diag[0][e] : 0.f) + (i >= r ? diag[1][e] : 0.f);
            }
            add_tile(p, tile);
        }
#pragma unroll
        for (int dir = 0; dir < 2; ++dir) {
            const unsigned base = dir == 0 ? at.kf : at.kb;
            const int step = dir == 0 ? -1 : 1, last = dir == 0 ? 0 : n_tiles - 1;
            f32x4 ahead[4];  // the next tile's factors, requested a tile ahead
            load_factors(dir, dir == 0 ? max(tile - 1, 0) : min(tile + 1, last), ahead);
#pragma unroll 1
            for (int I = tile + step; I >= 0 && I < n_tiles; I += step) {
                f32x4 now[4];
#pragma unroll
                for (int h = 0; h < 4; ++h) now[h] = ahead[h];
                load_factors(dir, I == last ? I : I + step, ahead);
                f32x4 p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < kKs; ++kk)
                    p = mfma(short_b128(base + I * 16 * ShortSlab<kDk>::kKeyBytes + key_place<2 * kDk>(r, 4 * kk + g)),
                             pack8(cum[dir] + 8 * kk), p);
                add_tile(p, I);
#pragma unroll
                for (int n = 0; n < 16; ++n) cum[dir][n] *= now[n >> 2][n & 3];
            }
        }
        short_store(io.out, io.pitch, tile, r, g, O);
    }
}

// kGates: g_fwd and g_bwd are OUTPUTS, made from the gate producer's low-rank half as in bigla_ws_state_kernel (lane
// (r, g) the 16 channels 16g..16g+15 of token r, the arithmetic of gate_producer_bf16_kernel bit for bit).
template <int kDk, bool kTm, bool kGates>
__global__ __launch_bounds__(64 * kShortWaves, 4) void bigla_short_kernel(
    const uint16_t *__restrict__ q_all, const uint16_t *__restrict__ k_all, const uint16_t *__restrict__ v_all,
    const uint16_t *gf_all, const uint16_t *gb_all, uint16_t *__restrict__ out_all, float *__restrict__ eb_all, int L,
    int n_tiles, int slab_waves, int slots, long n_slabs, int heads, GateSource gs)
{
    constexpr int kKs = kDk / 32;        // K-steps of a contraction over channels
    constexpr int kCt = kDk / 16;        // 16-channel tiles
    constexpr int kKeyBytes = 2 * kDk;
    constexpr int kGateLoads = kDk / 32;  // 16-byte loads per lane for the 16 whole rows of a gate tile
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int slot = wave / slab_waves, w = wave - slot * slab_waves;
    // (past the last slab: the last one once more, same values)
    const long mine = long(blockIdx.x) * slots + slot, slab = mine < n_slabs ? mine : n_slabs - 1;
    const SlabIo<kTm, kDk> io(q_all, k_all, v_all, gf_all, gb_all, out_all, slab, L, heads);
    const ShortSlab<kDk> at(slot, n_tiles);
    int *strong = reinterpret_cast<int *>(g_short_lds + unsigned(slots) * ShortSlab<kDk>::bytes(n_tiles)) + slot;
    const bool two = 2 * w + 1 < n_tiles;  // the wave's second tile exists
    const int tile0 = 2 * w;

    if (w == 0 && lane == 0) *strong = 0;
    if constexpr (!kGates) {
        // ---- the gates of the wave's 32 tokens
        uint4 rg[2][2][kGateLoads];
        const int grow = kDk == kD ? lane >> 3 : lane >> 2, gpiece = kDk == kD ? lane & 7 : lane & 3;
#pragma unroll
        for (int T = 0; T < 2; ++T)
#pragma unroll
            for (int dir = 0; dir < 2; ++dir)
#pragma unroll
                for (int h = 0; h < kGateLoads; ++h) {
                    const unsigned off = unsigned(16 * (tile0 + T) + 8 * h + grow) * io.key_pitch + 16u * gpiece;
                    const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(dir == 0 ? io.gf : io.gb, off, 0, 0);
                    rg[T][dir][h] = make_uint4(x.x, x.y, x.z, x.w);
                }
        // ---- gates into the wave's own rows of the key tiles (columns permuted as by stage_gates, so that accumulator
        // row 4g + e of channel tile ct is the lane's slot 4ct + e)
#pragma unroll
        for (int T = 0; T < 2; ++T) {
            if (T == 1 && !two) break;
#pragma unroll
            for (int dir = 0; dir < 2; ++dir)
#pragma unroll
                for (int h = 0; h < kGateLoads; ++h) {
                    const unsigned base = (dir == 0 ? at.kf : at.kb) + unsigned(tile0 + T) * 16u * kKeyBytes;
                    const int row = 8 * h + grow, kk = gpiece >> 2, j = gpiece & 3;
                    const uint4 x = rg[T][dir][h];
                    *reinterpret_cast<uint2 *>(g_short_lds + base + key_place<kKeyBytes>(row, 4 * kk + (j >> 1)) + 8 * (j & 1)) = make_uint2(x.x, x.y);
                    *reinterpret_cast<uint2 *>(g_short_lds + base + key_place<kKeyBytes>(row, 4 * kk + 2 + (j >> 1)) + 8 * (j & 1)) = make_uint2(x.z, x.w);
                }
        }
    } else {
        const int head = int(unsigned(slab) % unsigned(gs.n_heads));
        const uint16_t *lowrank = gs.lowrank + size_t(unsigned(slab) / unsigned(gs.n_heads)) * L * 16;
        uint2 low[2];
#pragma unroll
        for (int T = 0; T < 2; ++T) {
            const int t = 16 * (tile0 + T) + r;
            low[T] = t < L ? *reinterpret_cast<const uint2 *>(lowrank + size_t(t) * 16 + 4 * g) : make_uint2(0u, 0u);
        }
        // (a 32-wide head has channels for the lanes g = 0, 1 only; the others repeat those rows and store nowhere)
        const bool has_channels = 16 * g < kDk;
        const int arow = (16 * (r >> 2)) % kDk + (r & 3);
#pragma unroll
        for (int dir = 0; dir < 2; ++dir) {
            const int base = (dir * gs.n_heads + head) * kDk;
            s16x4 a[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                a[i] = __builtin_bit_cast(s16x4, *reinterpret_cast<const uint2 *>(gs.w2 + size_t(base + arow + 4 * i) * 16 + 4 * g));
            uint4 braw[2];
#pragma unroll
            for (int h = 0; h < 2; ++h)
                braw[h] = gs.bias ? *reinterpret_cast<const uint4 *>(gs.bias + base + (16 * g) % kDk + 8 * h) : make_uint4(0u, 0u, 0u, 0u);
            const uint32_t b[8] = {braw[0].x, braw[0].y, braw[0].z, braw[0].w, braw[1].x, braw[1].y, braw[1].z, braw[1].w};
#pragma unroll
            for (int T = 0; T < 2; ++T) {
                const int t = 16 * (tile0 + T) + r;
                uint32_t packed[8];
#pragma unroll
                for (int i = 0; i < 4; ++i) {  // channels 16g + 4i .. + 3
                    const f32x4 bias = {bf16_lo_to_f32(b[2 * i]), bf16_hi_to_f32(b[2 * i]), bf16_lo_to_f32(b[2 * i + 1]), bf16_hi_to_f32(b[2 * i + 1])};
                    const f32x4 z = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[i], __builtin_bit_cast(s16x4, low[T]), bias, 0, 0, 0);
                    const float o0 = log_sigmoid(z[0]) * gs.inv_tau, o1 = log_sigmoid(z[1]) * gs.inv_tau;
                    const float o2 = log_sigmoid(z[2]) * gs.inv_tau, o3 = log_sigmoid(z[3]) * gs.inv_tau;
                    // (rows past the sequence: log-gate 0 in LDS, and their stores are dropped by the bounds check)
                    packed[2 * i] = t < L ? pack2(o0, o1) : 0u;
                    packed[2 * i + 1] = t < L ? pack2(o2, o3) : 0u;
                }
                if (has_channels && (T == 0 || two)) {
                    const unsigned row = (dir == 0 ? at.kf : at.kb) + unsigned(tile0 + T) * 16u * kKeyBytes;
                    const int piece = 4 * (g >> 1) + (g & 1);
                    *reinterpret_cast<uint2 *>(g_short_lds + row + key_place<kKeyBytes>(r, piece)) = make_uint2(packed[0], packed[1]);
                    *reinterpret_cast<uint2 *>(g_short_lds + row + key_place<kKeyBytes>(r, piece + 2)) = make_uint2(packed[2], packed[3]);
                    *reinterpret_cast<uint2 *>(g_short_lds + row + key_place<kKeyBytes>(r, piece) + 8) = make_uint2(packed[4], packed[5]);
                    *reinterpret_cast<uint2 *>(g_short_lds + row + key_place<kKeyBytes>(r, piece + 2) + 8) = make_uint2(packed[6], packed[7]);
                }
                const __amdgpu_buffer_rsrc_t dst = dir == 0 ? io.gf : io.gb;
                const unsigned off = has_channels ? unsigned(t) * io.key_pitch + 32u * unsigned(g) : 0xf0000000u;
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{packed[0], packed[1], packed[2], packed[3]}, dst, off, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{packed[4], packed[5], packed[6], packed[7]}, dst, off + 16u, 0, 0);
            }
        }
    }
    wave_lds_fence();
    // the other rows, requested here: they travel while the totals are formed, in the registers that held the gates
    Row16 rq[2], rk[2];
    StagedRows rv[2];
    const LaneRows vr = lane_rows<kD>(0, lane, io.pitch);
#pragma unroll
    for (int T = 0; T < 2; ++T) {
        rk[T] = short_operand_rows<kDk>(io.k, io.key_pitch, tile0 + T, r, g);
        rq[T] = short_operand_rows<kDk>(io.q, io.key_pitch, tile0 + T, r, g);
    }
#pragma unroll
    for (int T = 0; T < 2; ++T) rv[T] = load_rows(io.v, vr, unsigned(16 * (tile0 + T)));

    // A operand of a gate scan: channels of tile ct, k-slots = tokens 4g + e of the wave's first and second tile
    unsigned goff[kCt];
#pragma unroll
    for (int ct = 0; ct < kCt; ++ct)
        goff[ct] = unsigned(tile0) * 16u * kKeyBytes + key_place<kKeyBytes>(4 * g + (r >> 2), 2 * ct + ((r & 3) >> 1)) + 8u * (r & 1);
    // (without a second tile the slots of its tokens repeat the first one's and meet zeros in the other operand)
    const unsigned second_tile = two ? 16u * kKeyBytes : 0u;
    auto gate_operand = [&](int dir, int ct) {
        const unsigned off = (dir == 0 ? at.kf : at.kb) + goff[ct];
        return join(short_tr(off), short_tr(off + second_tile));
    };
    const uint2 none = make_uint2(0u, 0u), all = make_uint2(0x3F803F80u, 0x3F803F80u);
    const uint2 all2 = two ? all : none;
    // the wave's total log-gates per channel
    float *tot = reinterpret_cast<float *>(g_short_lds + at.v);  // [direction][wave][channel: slot order, 16ct + 4g + e]
    {
        const bf16x8 ones = operand(all, all2);
#pragma unroll
        for (int dir = 0; dir < 2; ++dir)
#pragma unroll
            for (int ct = 0; ct < kCt; ++ct) {
                const f32x4 t = mfma(gate_operand(dir, ct), ones, f32x4{0.f, 0.f, 0.f, 0.f});
                if (r == 0) *reinterpret_cast<f32x4 *>(&tot[(dir * slab_waves + w) * kDk + 16 * ct + 4 * g]) = t;
            }
    }
    __syncthreads();  // totals visible
    // What enters the wave's scans: the other waves' totals between it and the middle of the sequence, forward
    // (u < w minus u < mid) and backward (u > w minus u >= mid).  Lane = channel; the sums come back in accumulator
    // layout through the wave's own slots.
    float *own_offs = tot + (2 * slab_waves + 2 * w) * kDk;
    {
        const int c = lane & (kDk - 1), mid = slab_waves / 2;
        const unsigned below_w = (1u << w) - 1u, below_mid = (1u << mid) - 1u, upto_w = 2u * below_w + 1u;
        const unsigned take_f = below_w ^ below_mid;                        // one of the two contains the other
        const unsigned take_b = w < mid ? below_mid & ~upto_w : upto_w & ~below_mid;
        float t[2][kShortWaves];
#pragma unroll
        for (int dir = 0; dir < 2; ++dir)
#pragma unroll
            for (int u = 0; u < kShortWaves; ++u) t[dir][u] = tot[(dir * slab_waves + min(u, slab_waves - 1)) * kDk + c];
        // the 64-token stretch this wave lies in (the last one may be 32 tokens)
        const int u0 = w & ~1;
        float stretch[2];
#pragma unroll
        for (int dir = 0; dir < 2; ++dir) {
            stretch[dir] = tot[(dir * slab_waves + u0) * kDk + c];
            if (u0 + 1 < slab_waves) stretch[dir] += tot[(dir * slab_waves + u0 + 1) * kDk + c];
        }
        float of = 0.f, ob = 0.f;
#pragma unroll
        for (int u = 0; u < kShortWaves; ++u) {
            of += __int_as_float(__float_as_int(t[0][u]) & -int((take_f >> u) & 1u));
            ob += __int_as_float(__float_as_int(t[1][u]) & -int((take_b >> u) & 1u));
        }
        own_offs[c] = w < mid ? -of : of;
        own_offs[kDk + c] = w < mid ? ob : -ob;
        // (a NaN counts as too fast; a last stretch of a few tokens has the whole range: see bigla_tile.hpp)
        if (!(stretch[0] >= -kMildRange && stretch[1] >= -kMildRange)) *strong = 1;
        wave_lds_fence();
    }
    f32x4 offs[2][kCt];
#pragma unroll
    for (int dir = 0; dir < 2; ++dir)
#pragma unroll
        for (int ct = 0; ct < kCt; ++ct)
            offs[dir][ct] = *reinterpret_cast<const f32x4 *>(&own_offs[dir * kDk + 16 * ct + 4 * g]);
    __syncthreads();  // every wave has its offsets: the value rows may be written; the slab's flag is visible
    int flag = __builtin_amdgcn_readfirstlane(*strong);
    if (flag == 0) {
#pragma unroll
    for (int T = 0; T < 2; ++T)
        if (T == 0 || two) short_put_values(at.v, tile0 + T, lane, rv[T]);

    // ---- scaled queries (kept) and keys (into the rows the gates were in)
    // B operands of the scans: k-slots 0..3 = tokens 4g + e of the first tile, 4..7 of the second; 1 where the token
    // contributes to the lane's own token (token r of tile T)
    uint2 lower, upper;
    {
        uint32_t lo[4], up[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            lo[e] = 4 * g + e <= r ? 0x3F80u : 0u;
            up[e] = 4 * g + e >= r ? 0x3F80u : 0u;
        }
        lower = make_uint2(lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16));
        upper = make_uint2(up[0] | (up[1] << 16), up[2] | (up[3] << 16));
    }
    const bf16x8 tri_f[2] = {operand(lower, none), operand(all, lower)};
    const bf16x8 tri_b[2] = {operand(upper, all2), operand(none, upper)};
    bf16x8 qf[2][kKs], qb[2][kKs];
#pragma unroll
    for (int kk = 0; kk < kKs; ++kk) {
        uint32_t pqf[2][4], pqb[2][4], pkf[2][4], pkb[2][4];  // [tile][dword of the K-step's eight slots]
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ct = 2 * kk + h;
            const bf16x8 af = gate_operand(0, ct), ab = gate_operand(1, ct);
#pragma unroll
            for (int T = 0; T < 2; ++T) {
                const f32x4 Bf = mfma(af, tri_f[T], offs[0][ct]), Bb = mfma(ab, tri_b[T], offs[1][ct]);
                const uint4 &rqp = rq[T].p[kk], &rkp = rk[T].p[kk];
                const uint32_t dq[2] = {h == 0 ? rqp.x : rqp.z, h == 0 ? rqp.y : rqp.w};
                const uint32_t dk[2] = {h == 0 ? rkp.x : rkp.z, h == 0 ? rkp.y : rkp.w};
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    const float q0 = bf16_lo_to_f32(dq[d]), q1 = bf16_hi_to_f32(dq[d]);
                    const float k0 = bf16_lo_to_f32(dk[d]), k1 = bf16_hi_to_f32(dk[d]);
                    const float f0 = Bf[2 * d] * kLog2e, f1 = Bf[2 * d + 1] * kLog2e;
                    const float b0 = Bb[2 * d] * kLog2e, b1 = Bb[2 * d + 1] * kLog2e;
                    pqf[T][2 * h + d] = pack2(q0 * fast_exp2(f0), q1 * fast_exp2(f1));    // q exp(b_t)
                    pqb[T][2 * h + d] = pack2(q0 * fast_exp2(b0), q1 * fast_exp2(b1));
                    pkf[T][2 * h + d] = pack2(k0 * fast_exp2(-f0), k1 * fast_exp2(-f1));  // k exp(-b_i)
                    pkb[T][2 * h + d] = pack2(k0 * fast_exp2(-b0), k1 * fast_exp2(-b1));
                }
            }
        }
        // (the K-step's pieces of the key rows are where the gates of its two channel tiles were)
#pragma unroll
        for (int T = 0; T < 2; ++T) {
            qf[T][kk] = __builtin_bit_cast(bf16x8, make_uint4(pqf[T][0], pqf[T][1], pqf[T][2], pqf[T][3]));
            qb[T][kk] = __builtin_bit_cast(bf16x8, make_uint4(pqb[T][0], pqb[T][1], pqb[T][2], pqb[T][3]));
            // (materialised here: left to itself the compiler sinks the backward exponentials past the first key tiles)
            asm volatile("" : "+v"(qf[T][kk]), "+v"(qb[T][kk]));
            if (T == 0 || two) {
                const unsigned off = unsigned(tile0 + T) * 16u * kKeyBytes + key_place<kKeyBytes>(r, 4 * kk + g);
                *reinterpret_cast<uint4 *>(g_short_lds + at.kf + off) = make_uint4(pkf[T][0], pkf[T][1], pkf[T][2], pkf[T][3]);
                *reinterpret_cast<uint4 *>(g_short_lds + at.kb + off) = make_uint4(pkb[T][0], pkb[T][1], pkb[T][2], pkb[T][3]);
            }
        }
    }
    __syncthreads();  // scaled keys and values visible

    // ---- the wave's 32 rows of the score matrix, 32 keys at a time
    unsigned koff[kKs], voff[4];
#pragma unroll
    for (int kk = 0; kk < kKs; ++kk) koff[kk] = key_place<kKeyBytes>(r, 4 * kk + g);
#pragma unroll
    for (int jt = 0; jt < 4; ++jt) voff[jt] = at.v + short_value_off(jt, r, g);
    f32x4 O[2][4];
#pragma unroll
    for (int T = 0; T < 2; ++T)
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) O[T][jt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    struct Keys {
        bf16x8 a[kKs];
    };
    auto key_rows = [&](unsigned region, int tile) {
        Keys k;
#pragma unroll
        for (int kk = 0; kk < kKs; ++kk) k.a[kk] = short_b128(region + unsigned(tile) * 16u * kKeyBytes + koff[kk]);
        return k;
    };
    auto scores = [&](const Keys &k, const bf16x8 (&qx)[2][kKs], f32x4 (&p)[2]) {
#pragma unroll
        for (int T = 0; T < 2; ++T) {
            p[T] = mfma(k.a[0], qx[T][0], zero);
            if (kKs > 1) p[T] = mfma(k.a[kKs - 1], qx[T][kKs - 1], p[T]);
        }
    };
    // O += V^T P^T for key tiles t0 and t1 (t1 = t0 where there is no second one: its scores are then zero)
    auto add_pair = [&](int t0, int t1, const f32x4 (&p0)[2], const f32x4 (&p1)[2]) {
        bf16x8 h[2], l[2];
#pragma unroll
        for (int T = 0; T < 2; ++T) {
            uint2 h0, h1, l0, l1;
            split4(p0[T], h0, l0);
            split4(p1[T], h1, l1);
            h[T] = operand(h0, h1);
            l[T] = operand(l0, l1);
        }
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) {
            const bf16x8 vv = join(short_tr(voff[jt] + unsigned(t0) * 2048u), short_tr(voff[jt] + unsigned(t1) * 2048u));
#pragma unroll
            for (int T = 0; T < 2; ++T) O[T][jt] = mfma(vv, h[T], mfma(vv, l[T], O[T][jt]));
        }
    };
    // (each step's keys are read from LDS a step ahead)
    const int own1 = two ? tile0 + 1 : tile0;
    Keys k0 = key_rows(at.kf, 0), k1 = key_rows(at.kf, w > 0 ? 1 : own1);
    for (int p = 0; p < w; ++p) {
        f32x4 p0[2], p1[2];
        scores(k0, qf, p0);
        scores(k1, qf, p1);
        k0 = key_rows(at.kf, 2 * p + 2);
        k1 = key_rows(at.kf, p + 1 < w ? 2 * p + 3 : own1);
        add_pair(2 * p, 2 * p + 1, p0, p1);
    }
    {
        // keys of the first tile: own diagonal, and forward for the second tile; of the second tile: own diagonal,
        // and backward for the first tile
        f32x4 f0[2], f1[2], b0[2], b1[2];
        const Keys c0 = key_rows(at.kb, tile0), c1 = key_rows(at.kb, own1);
        scores(k0, qf, f0);
        scores(k1, qf, f1);
        scores(c0, qb, b0);
        scores(c1, qb, b1);
        const int next = min(w + 1, slab_waves - 1);
        k0 = key_rows(at.kb, 2 * next);
        k1 = key_rows(at.kb, min(2 * next + 1, n_tiles - 1));
        f32x4 p0[2], p1[2];
        p0[1] = f0[1];
        p1[0] = two ? b1[0] : zero;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 4 * g + e;
            p0[0][e] = (i <= r ? f0[0][e] : 0.f) + (i >= r ? b0[0][e] : 0.f);
            p1[1][e] = (i <= r ? f1[1][e] : 0.f) + (i >= r ? b1[1][e] : 0.f);
        }
        if (!two) p1[1] = zero;
        add_pair(tile0, own1, p0, p1);
    }
    for (int p = w + 1; p < slab_waves; ++p) {
        f32x4 p0[2], p1[2];
        const bool second = 2 * p + 1 < n_tiles;
        scores(k0, qb, p0);
        scores(k1, qb, p1);
        k0 = key_rows(at.kb, min(2 * p + 2, n_tiles - 1));
        k1 = key_rows(at.kb, min(2 * p + 3, n_tiles - 1));
        if (!second) p1[0] = p1[1] = zero;
        add_pair(2 * p, second ? 2 * p + 1 : 2 * p, p0, p1);
    }
#pragma unroll
    for (int T = 0; T < 2; ++T) {
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
#pragma unroll
            for (int e = 0; e < 4; ++e) O[T][jt][e] *= 0.5f;  // the average of the two directions
        short_store(io.out, io.pitch, tile0 + T, r, g, O[T]);
    }
    }
    // (tested anew: as the other branch of the test above the call would be placed before the fast form, with everything
    // that form holds in registers spilled around it)
    asm volatile("" : "+s"(flag));
    if (flag != 0)
        short_slab_safe<kDk, kTm>(q_all, k_all, v_all, gf_all, gb_all, out_all, eb_all + slab * (2 * kShortTiles * kD), slab, slot, w,
                                  slab_waves, L, n_tiles, heads);
}

}  // namespace

}  // namespace vig

#include "bigla_tile.hpp"

namespace vig {

// A sequence in one chunk, in one launch: a wave per tile (bigla_tile.hpp) or per two tiles (bigla_short_kernel), see below.
// With gates that decay by up to 16 nats in 64 tokens one chunk is the faster way at nearly every length up to 256 and number of
// slabs; beyond that the kernel with two tiles to a wave takes the range-safe form (at -0.3 a step, 192 and 384 slabs of 196
// tokens 34 and 55 us against 67 and 96 of the four-wave kernels), the one with a tile to a wave and the eight-wave kernels stay
// in the fast form.  Whose gates those are is known on the device only.  From 193 tokens on in fewer than 128 slabs the
// eight-wave kernels are kept: 6 and 48 slabs of 225 tokens 12.9 us with mild gates and 13.2 at -0.3 a step against 13.7 and 15.4.
// The score matrix grows with the square of the length: beyond 256 tokens the sequence is chunked.
bool bigla_short_applicable(long BH, int L) { return L <= kShortTokens && (BH >= 128 || L <= 192); }

// A wave per tile, or per two tiles (which reads half as much LDS and keeps two slabs on a compute unit).  us per call, two tiles to a wave /
// one, mild gates, 64-wide keys: 256 slabs of 80 tokens 10.1 / 8.4, 768 of 80 18.0 / 16.1, 1024 of 80 19.8 / 22.0, 1024 of 112 28.3 / 22.9, 2048 of 128
// 59.7 / 45.1, 192 of 130 10.7 / 11.1, 192 of 196 14.0 / 15.5, 384 of 196 23.8 / 28.7; 32-wide: 256 of 100 8.7 / 6.9, 512 10.4 / 10.6, 1024 of 80
// 13.9 / 17.3; up to 64 tokens 0.73 to 1.04 of it at any number of slabs.
inline bool wave_per_tile(long BH, int L, int dk)
{
    if (L <= kC || BH < 128) return true;
    if (L > 2 * kC) return false;
    return dk == kD ? BH <= 768 || L > 96 : BH <= 384;
}

// bytes of workspace: the range-safe form's whole-tile decay factors
size_t bigla_short_workspace_bytes(long BH) { return size_t(BH) * 2 * kShortTiles * kD * sizeof(float); }

hipError_t bigla_short_launch(const void *q, const void *k, const void *v, const void *g_fwd, const void *g_bwd, void *out,
                              long BH, int L, int dk, int heads_token_major, void *workspace, hipStream_t stream,
                              const GateSource *gates = nullptr)
{
    const int n_tiles = (L + 15) / 16, slab_waves = (n_tiles + 1) / 2;
    const bool per_tile = wave_per_tile(BH, L, dk);
    const int slots = per_tile ? 1 : kShortWaves / slab_waves;  // slabs per workgroup
    const long blocks = (BH + slots - 1) / slots;
    if (blocks > 0x7fffffffL || (per_tile && n_tiles > kTileMost)) return hipErrorInvalidValue;
    LaunchTimer timer(kKernelSlab, stream);
    const GateSource none = {};
    auto go = [&](auto dk_c, auto tm_c, auto gates_c) {
        constexpr int kDk = decltype(dk_c)::value;
        constexpr bool kTm = decltype(tm_c)::value, kGates = decltype(gates_c)::value;
        auto tile_launch = [&](auto halves_c) {
            constexpr bool kHalves = decltype(halves_c)::value;
            const unsigned lds = tile_lds_bytes<kDk, kHalves>(n_tiles);
            hipLaunchKernelGGL((bigla_tile_kernel<kDk, kTm, kGates, kHalves>), dim3((unsigned)BH), dim3(unsigned(64 * n_tiles)), lds, stream,
                               static_cast<const uint16_t *>(q), static_cast<const uint16_t *>(k), static_cast<const uint16_t *>(v),
                               static_cast<const uint16_t *>(g_fwd), static_cast<const uint16_t *>(g_bwd), static_cast<uint16_t *>(out),
                               static_cast<float *>(workspace), L, n_tiles, heads_token_major > 0 ? heads_token_major : 1, gates ? *gates : none);
        };
        if (per_tile) {
            if (tile_halves(n_tiles)) tile_launch(std::true_type{}); else tile_launch(std::false_type{});
            return;
        }
        const unsigned lds = unsigned(slots) * (ShortSlab<kDk>::bytes(n_tiles) + unsigned(sizeof(int)));
        hipLaunchKernelGGL((bigla_short_kernel<kDk, kTm, kGates>), dim3((unsigned)blocks), dim3(unsigned(64 * slab_waves * slots)), lds, stream,
                           static_cast<const uint16_t *>(q), static_cast<const uint16_t *>(k), static_cast<const uint16_t *>(v),
                           static_cast<const uint16_t *>(g_fwd), static_cast<const uint16_t *>(g_bwd), static_cast<uint16_t *>(out),
                           static_cast<float *>(workspace), L, n_tiles, slab_waves, slots, BH, heads_token_major > 0 ? heads_token_major : 1,
                           gates ? *gates : none);
    };
    using std::integral_constant;
    auto go_layout = [&](auto dk_c, auto gates_c) {
        if (heads_token_major > 0) go(dk_c, std::true_type{}, gates_c); else go(dk_c, std::false_type{}, gates_c);
    };
    auto go_gates = [&](auto dk_c) {
        if (gates) go_layout(dk_c, std::true_type{}); else go_layout(dk_c, std::false_type{});
    };
    if (dk == kD) go_gates(integral_constant<int, kD>{}); else go_gates(integral_constant<int, kD / 2>{});
    return hipGetLastError();
}

}  // namespace vig
