// BiGLA forward (Section 4.2.1, Eq. (BiGLA)) for sequences of up to 192 tokens (12 tiles) in one chunk, as in bigla_short.hpp (the
// algebra is there), with a wave per 16-token tile and a slab per workgroup: for few slabs, where the chain of one workgroup is what takes
// the time and most of the chip's wave slots are empty, and for up to 64 tokens in any number of slabs.
//
// A wave scans the gates of its own tile only (its rows never leave it, so there is no barrier before the scan); the tiles'
// totals are exchanged through LDS and enter as offsets of the exponents.  Its own diagonal tile of the scores comes from its
// registers.  Three barriers.
//
// A slab in which some 64-token stretch decays by more than kMildRange (a sequence of fewer tokens: by more than its share of that) has the operands of the diagonal tiles split into bf16 pairs,
// as in the eight-wave kernels.  All exponents are referred to one point in the middle of the sequence as long as neither half decays
// by more than kFastRange.  Up to 128 tokens a slab beyond that takes the range-safe form (short_slab_safe), a tile a wave; there
// that is the limit of the eight-wave kernels, 60 nats in 64 tokens.  From 129 tokens on (kHalves) each half is then referred to
// its own middle, with a second set of scaled queries for the keys of the other half, and the range-safe form is left to
// slabs with a quarter beyond kFastRange.  At -0.8 a step, 64-wide keys, one point and the range-safe form / two points / the eight-wave
// kernels: 6 slabs of 144 tokens 19.3 / 11.2 / 11.2 us, of 192 22.5 / 12.3 / 11.1, 127 slabs of 192 26.2 / 12.8 / 16.9; at -0.3 one point holds
// and two would take 0.6 us more.
//
// Per call in a captured graph, us, 64-wide keys, mild gates and -0.3 a step (the kernels before it: up to 64 tokens and from 128 slabs on
// bigla_short_kernel, else the eight-wave kernels): 6 slabs of 65 tokens 6.7 / 7.4 (11.7 / 12.0), 48 of 100 7.5 / 8.3 (12.2 / 12.5), 48
// of 192 10.7 / 11.7 (13.0 / 13.4), 127 of 192 12.0 / 13.0 (18.3 / 19.1), 192 of 100 7.9 / 8.9 (11.0 / 26.0), 1024 of 49 11.8 / 13.4 (13.1 /
// 33.6), 4096 of 40 27.6 / 32.9 (34.1 / 87.8).  What bounds it: the instructions of the waves on a SIMD; they grow with the
// square of the length, and beyond 12 tiles some SIMD has four waves (6 slabs: 192 tokens 10.4, 196 tokens 12.7).
//
// This file is part of the translation unit of bigla_chunk.hip.
#pragma once

namespace vig {

namespace {

constexpr int kTileMost = 12;  // tiles of the longest sequence (192 tokens)
constexpr int kTileWhole = 8;  // up to so many, halves of at most 64 tokens: one reference point
inline bool tile_halves(int n_tiles) { return n_tiles > kTileWhole; }

template <int kDk, bool kHalves>
constexpr unsigned tile_lds_bytes(int n_tiles)
{
    return ShortSlab<kDk>::bytes(n_tiles) + 4 * unsigned(sizeof(int)) + unsigned(n_tiles) * (kHalves ? 5 : 4) * kDk * unsigned(sizeof(float));
}

template <int kDk, bool kTm, bool kGates, bool kHalves /* 9 to 12 tiles */>
__global__ __launch_bounds__(64 * (kHalves ? kTileMost : kTileWhole), kHalves ? 3 : 4) void bigla_tile_kernel(
    const uint16_t *__restrict__ q_all, const uint16_t *__restrict__ k_all, const uint16_t *__restrict__ v_all,
    const uint16_t *gf_all, const uint16_t *gb_all, uint16_t *__restrict__ out_all, float *__restrict__ eb_all, int L,
    int n_tiles, int heads, GateSource gs)
{
    constexpr int kKs = kDk / 32;  // K-steps of a contraction over channels
    constexpr int kCt = kDk / 16;  // 16-channel tiles
    constexpr int kKeyBytes = 2 * kDk;
    constexpr unsigned kKeyTile = 16u * kKeyBytes, kValueTile = 2048u;
    const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const long slab = blockIdx.x;
    const SlabIo<kTm, kDk> io(q_all, k_all, v_all, gf_all, gb_all, out_all, slab, L, heads);
    const ShortSlab<kDk> at(0, n_tiles);
    // strong: some 64-token stretch beyond kMildRange; far: half the sequence beyond kFastRange; beyond: a quarter of it
    int *strong = reinterpret_cast<int *>(g_short_lds + ShortSlab<kDk>::bytes(n_tiles)), *far = strong + 1, *beyond = kHalves ? strong + 2 : far;
    float *tot = reinterpret_cast<float *>(strong + 4);  // totals [direction][tile][channel], then what enters each tile, likewise
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    const unsigned own_keys = unsigned(w) * kKeyTile;
    if (w == 0 && lane == 0) *strong = *far = *beyond = 0;

    // ---- rows of the tile; its gates into its rows of the key tiles
    Row16 rq, rk;
    StagedRows rv;
    auto load_others = [&]() __attribute__((always_inline)) {
        rk = short_operand_rows<kDk>(io.k, io.key_pitch, w, r, g);
        rq = short_operand_rows<kDk>(io.q, io.key_pitch, w, r, g);
        rv = load_rows(io.v, lane_rows<kD>(0, lane, io.pitch), unsigned(16 * w));
    };
    if constexpr (!kGates) {
        const int grow = kKs > 1 ? lane >> 3 : lane >> 2, gpiece = kKs > 1 ? lane & 7 : lane & 3;
        u32x4 rg[2][kKs];
#pragma unroll
        for (int dir = 0; dir < 2; ++dir)
#pragma unroll
            for (int h = 0; h < kKs; ++h)
                rg[dir][h] = __builtin_amdgcn_raw_buffer_load_b128(dir == 0 ? io.gf : io.gb, unsigned(16 * w + 8 * h + grow) * io.key_pitch + 16u * unsigned(gpiece), 0, 0);
        load_others();
#pragma unroll
        for (int dir = 0; dir < 2; ++dir)
#pragma unroll
            for (int h = 0; h < kKs; ++h)
                *reinterpret_cast<u32x4 *>(g_short_lds + (dir == 0 ? at.kf : at.kb) + own_keys + key_place<kKeyBytes>(8 * h + grow, gpiece)) = rg[dir][h];
    } else {
        // as in bigla_short_kernel: lane (r, g) the 16 channels 16g .. 16g + 15 of token r (a 32-wide head has channels for the
        // lanes g = 0, 1 only; the others repeat those rows and store nowhere)
        const int head = int(unsigned(slab) % unsigned(gs.n_heads)), t = 16 * w + r;
        const uint16_t *lowrank = gs.lowrank + size_t(unsigned(slab) / unsigned(gs.n_heads)) * L * 16;
        const uint2 low = t < L ? *reinterpret_cast<const uint2 *>(lowrank + size_t(t) * 16 + 4 * g) : make_uint2(0u, 0u);
        const bool has_channels = 16 * g < kDk;
        const int arow = (16 * (r >> 2)) % kDk + (r & 3);
        s16x4 a[2][4];
        uint4 braw[2][2];
#pragma unroll
        for (int dir = 0; dir < 2; ++dir) {
            const int base = (dir * gs.n_heads + head) * kDk;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                a[dir][i] = __builtin_bit_cast(s16x4, *reinterpret_cast<const uint2 *>(gs.w2 + size_t(base + arow + 4 * i) * 16 + 4 * g));
#pragma unroll
            for (int h = 0; h < 2; ++h)
                braw[dir][h] = gs.bias ? *reinterpret_cast<const uint4 *>(gs.bias + base + (16 * g) % kDk + 8 * h) : make_uint4(0u, 0u, 0u, 0u);
        }
        load_others();
#pragma unroll
        for (int dir = 0; dir < 2; ++dir) {
            const uint32_t b[8] = {braw[dir][0].x, braw[dir][0].y, braw[dir][0].z, braw[dir][0].w, braw[dir][1].x, braw[dir][1].y, braw[dir][1].z, braw[dir][1].w};
            uint32_t packed[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {  // channels 16g + 4i .. + 3
                const f32x4 bias = {bf16_lo_to_f32(b[2 * i]), bf16_hi_to_f32(b[2 * i]), bf16_lo_to_f32(b[2 * i + 1]), bf16_hi_to_f32(b[2 * i + 1])};
                const f32x4 z = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[dir][i], __builtin_bit_cast(s16x4, low), bias, 0, 0, 0);
                const float o0 = log_sigmoid(z[0]) * gs.inv_tau, o1 = log_sigmoid(z[1]) * gs.inv_tau;
                const float o2 = log_sigmoid(z[2]) * gs.inv_tau, o3 = log_sigmoid(z[3]) * gs.inv_tau;
                // (rows past the sequence: log-gate 0 in LDS, and their stores are dropped by the bounds check)
                packed[2 * i] = t < L ? pack2(o0, o1) : 0u;
                packed[2 * i + 1] = t < L ? pack2(o2, o3) : 0u;
            }
            const u32x4 lo = {packed[0], packed[1], packed[2], packed[3]}, hi = {packed[4], packed[5], packed[6], packed[7]};
            if (has_channels) {
                const unsigned base = (dir == 0 ? at.kf : at.kb) + own_keys;
                *reinterpret_cast<u32x4 *>(g_short_lds + base + key_place<kKeyBytes>(r, 2 * g)) = lo;
                *reinterpret_cast<u32x4 *>(g_short_lds + base + key_place<kKeyBytes>(r, 2 * g + 1)) = hi;
            }
            const __amdgpu_buffer_rsrc_t dst = dir == 0 ? io.gf : io.gb;
            const unsigned off = has_channels ? unsigned(t) * io.key_pitch + 32u * unsigned(g) : 0xf0000000u;
            __builtin_amdgcn_raw_buffer_store_b128(lo, dst, off, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b128(hi, dst, off + 16u, 0, 0);
        }
    }
    short_put_values(at.v, w, lane, rv);
    wave_lds_fence();

    // ---- cumulative gates of the tile, a product with a 0/1 triangle.  Patches of the transposing reads: tile rows 4g .. 4g + 3, columns such
    // that accumulator row 4g + e of channel tile ct is slot 4ct + e of the lane's operand order, channel 32 (ct / 2) + 8g + 4 (ct % 2) + e
    const unsigned patch = own_keys + key_place<kKeyBytes>(4 * g + (r >> 2), r & 3);
    auto gate_patch = [&](int dir, int ct) __attribute__((always_inline)) {
        return short_tr(((dir == 0 ? at.kf : at.kb) + patch + 8u * unsigned(ct & 1)) ^ (ct >= 2 ? 64u : 0u));
    };
    uint2 upto, from;  // 1.0 where token 4g + e comes no later (no earlier) than token r
    {
        uint32_t lo[4], up[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            lo[e] = 4 * g + e <= r ? 0x3F80u : 0u;
            up[e] = 4 * g + e >= r ? 0x3F80u : 0u;
        }
        upto = make_uint2(lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16));
        from = make_uint2(up[0] | (up[1] << 16), up[2] | (up[3] << 16));
    }
    f32x4 B[2][kCt];
#pragma unroll
    for (int dir = 0; dir < 2; ++dir)
#pragma unroll
        for (int ct = 0; ct < kCt; ++ct) {
            B[dir][ct] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(gate_patch(dir, ct), __builtin_bit_cast(s16x4, dir == 0 ? upto : from), zero, 0, 0, 0);
            if (r == (dir == 0 ? 15 : 0)) *reinterpret_cast<f32x4 *>(&tot[(dir * n_tiles + w) * kDk + 32 * (ct >> 1) + 8 * g + 4 * (ct & 1)]) = B[dir][ct];
        }
    __syncthreads();  // totals visible

    // ---- what enters the tile's scans, referred to the first token of tile `mid`; lane = channel
    const int mid = kHalves ? (n_tiles + 2) / 4 * 2 : n_tiles >> 1;  // (halves of whole pairs of tiles)
    const bool low = w < mid;
    float *own_offs = tot + (2 * n_tiles + (kHalves ? 3 : 2) * w) * kDk;
    const int c = lane & (kDk - 1);
    auto sum = [&](auto most, int dir, int first, int last) __attribute__((always_inline)) {  // of the totals of tiles first .. last - 1
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < decltype(most)::value; ++i) {
            const float t = tot[(dir * n_tiles + min(first + i, n_tiles - 1)) * kDk + c];
            s += __int_as_float(__float_as_int(t) & (first + i < last ? -1 : 0));
        }
        return s;
    };
    const std::integral_constant<int, (kHalves ? kTileMost : kTileWhole) / 2> half;
    const std::integral_constant<int, kTileMost / 4> quarter;
    const int ref[2] = {mid / 2, (mid + n_tiles) / 2};  // kHalves: the halves' own reference points, likewise
    {
        const float of = sum(half, 0, low ? w : mid, low ? mid : w), ob = sum(half, 1, low ? w + 1 : mid, low ? mid : w + 1);
        const float xf = low ? -of : of, xb = low ? ob : -ob;
        own_offs[c] = xf * kLog2e;
        own_offs[kDk + c] = xb * kLog2e;
        // The 64-token stretch that begins here.  (A NaN counts as too fast; a sequence of under 64 tokens has its share of the range: the
        // decay per token is what leaves an output few tokens to sum over.  A last stretch of a few tokens keeps all of it: the slab's
        // scale is that of the others, and few gates of such a stretch are an ordinary draw away from a share.)
        if ((w & 3) == 0) {
            float s[2] = {0.f, 0.f};
#pragma unroll
            for (int dir = 0; dir < 2; ++dir)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (w + i < n_tiles) s[dir] += tot[(dir * n_tiles + w + i) * kDk + c];
            const float range = kMildRange / kC * float(min(L, kC));
            if (!(s[0] >= -range && s[1] >= -range)) *strong = 1;
        }
        // exponents reach furthest at the two ends; with a reference point to each half, at the ends of the quarters
        auto is_far = [&](bool upper) __attribute__((always_inline)) {
            *far = 1;
            if constexpr (kHalves) {
                const int first = upper ? mid : 0, own = ref[upper], last = upper ? n_tiles : mid;
                const bool near = sum(quarter, 0, first, own) >= -kFastRange && sum(quarter, 0, own, last) >= -kFastRange &&
                                  sum(quarter, 1, first, own) >= -kFastRange && sum(quarter, 1, own, last) >= -kFastRange;
                if (!near) *beyond = 1;
            }
        };
        if (w == 0 && !(xf <= kFastRange && xb + tot[n_tiles * kDk + c] >= -kFastRange)) is_far(false);
        if (w == n_tiles - 1 && !(xb <= kFastRange && xf + tot[w * kDk + c] >= -kFastRange)) is_far(true);
        wave_lds_fence();
    }
    // exponents (of 2) of the lane's token
#pragma unroll
    for (int dir = 0; dir < 2; ++dir)
#pragma unroll
        for (int ct = 0; ct < kCt; ++ct) {
            const f32x4 off = *reinterpret_cast<const f32x4 *>(&own_offs[dir * kDk + 32 * (ct >> 1) + 8 * g + 4 * (ct & 1)]);
#pragma unroll
            for (int e = 0; e < 4; ++e) B[dir][ct][e] = fmaf(B[dir][ct][e], kLog2e, off[e]);
        }
    __syncthreads();  // the slab's flags are visible
    const bool split = __builtin_amdgcn_readfirstlane(*strong) != 0;
    const bool apart = kHalves && split && __builtin_amdgcn_readfirstlane(*far) != 0;  // each half has a reference point of its own
    int safe = __builtin_amdgcn_readfirstlane(*strong & *beyond);
    if (safe == 0) {
        // ---- scaled queries (kept; they carry the 1/2 of the average) and keys (into the rows the gates were in), and the own
        // diagonal tile of the scores
        bf16x8 qx[2][kKs];
        bf16x8 qc[kHalves ? kKs : 1] = {};  // the queries for the other half's keys, referred to that half's point
        f32x4 diag[2] = {zero, zero};
        auto scale = [&](auto split_c) __attribute__((always_inline)) {
            constexpr bool kSplit = decltype(split_c)::value;
            // (values of its own for this copy: shared with the other one, all 64 products would be live across the branch)
            if constexpr (kSplit) {
#pragma unroll
                for (int ct = 0; ct < kCt; ++ct) asm volatile("" : "+v"(B[0][ct]), "+v"(B[1][ct]));
            }
            if constexpr (kSplit && kHalves) {
                if (apart) {
                    // from the middle to the own half's reference point, and for the queries that meet the other half's keys to
                    // that half's (those are the backward direction's in the lower half, the forward one's in the upper)
                    const int h0 = low ? ref[0] : mid, h1 = low ? mid : ref[1], o0 = low ? mid : ref[0], o1 = low ? ref[1] : mid;
                    const float sf = sum(quarter, 0, h0, h1), sb = sum(quarter, 1, h0, h1), so = sum(quarter, low ? 1 : 0, o0, o1);
                    own_offs[c] = (low ? sf : -sf) * kLog2e;
                    own_offs[kDk + c] = (low ? -sb : sb) * kLog2e;
                    own_offs[2 * kDk + c] = so * kLog2e;
                    wave_lds_fence();
#pragma unroll
                    for (int kk = 0; kk < kKs; ++kk) {
                        float qv[8];
                        unpack8(rq.p[kk], qv);
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const int ct = 2 * kk + h;
                            const float *off = &own_offs[32 * kk + 8 * g + 4 * h];
                            const f32x4 x = (low ? B[1][ct] : B[0][ct]) + *reinterpret_cast<const f32x4 *>(off + 2 * kDk);
                            B[0][ct] += *reinterpret_cast<const f32x4 *>(off);
                            B[1][ct] += *reinterpret_cast<const f32x4 *>(off + kDk);
#pragma unroll
                            for (int e = 0; e < 4; ++e) qv[4 * h + e] *= fast_exp2(x[e] - 1.f);
                        }
                        qc[kk] = pack8(qv);
                    }
                }
            }
#pragma unroll
            for (int kk = 0; kk < kKs; ++kk) {
                float qv[8], kv[8];
                unpack8(rq.p[kk], qv);
                unpack8(rk.p[kk], kv);
#pragma unroll
                for (int dir = 0; dir < 2; ++dir) {
                    float qs[8], ks[8];
#pragma unroll
                    for (int n = 0; n < 8; ++n) {
                        const int ct = 2 * kk + (n >> 2);
                        const float x = B[dir][ct][n & 3];
                        qs[n] = qv[n] * fast_exp2(x - 1.f);
                        ks[n] = kv[n] * fast_exp2(-x);
                    }
                    bf16x8 kh;
                    if constexpr (kSplit) {
                        bf16x8 kl, ql;
                        pack8_split(ks, kh, kl);
                        pack8_split(qs, qx[dir][kk], ql);
                        diag[dir] = mfma(kl, qx[dir][kk], mfma(kh, ql, diag[dir]));
                    } else {
                        kh = pack8(ks);
                        qx[dir][kk] = pack8(qs);
                    }
                    diag[dir] = mfma(kh, qx[dir][kk], diag[dir]);
                    *reinterpret_cast<bf16x8 *>(g_short_lds + (dir == 0 ? at.kf : at.kb) + own_keys + key_place<kKeyBytes>(r, 4 * kk + g)) = kh;
                }
            }
        };
        if (split) scale(std::true_type{}); else scale(std::false_type{});
        f32x4 own;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 4 * g + e;
            own[e] = (i <= r ? diag[0][e] : 0.f) + (i >= r ? diag[1][e] : 0.f);
        }
        __syncthreads();  // scaled keys and values visible

        // ---- the tile's rows of the score matrix, 32 keys at a time (each step's keys are read from LDS a step ahead)
        const unsigned koff = key_place<kKeyBytes>(r, g);
        const unsigned voff = at.v + value_place(4 * g + (r >> 2), r & 3);
        f32x4 O[4] = {zero, zero, zero, zero};
        struct Keys {
            bf16x8 a[kKs];
        };
        auto key_rows = [&](unsigned region, int tile) __attribute__((always_inline)) {
            Keys k;
#pragma unroll
            for (int kk = 0; kk < kKs; ++kk) k.a[kk] = short_b128((region + unsigned(tile) * kKeyTile + koff) ^ (64u * unsigned(kk)));
            return k;
        };
        auto scores = [&](const Keys &k, const bf16x8 *q) __attribute__((always_inline)) {
            f32x4 p = mfma(k.a[0], q[0], zero);
            if (kKs > 1) p = mfma(k.a[kKs - 1], q[kKs - 1], p);
            return p;
        };
        auto add_pair = [&](int t0, int t1, const f32x4 &p0, const f32x4 &p1) __attribute__((always_inline)) {
            uint2 h0, h1, l0, l1;
            split4(p0, h0, l0);
            split4(p1, h1, l1);
            const bf16x8 h = operand(h0, h1), l = operand(l0, l1);
#pragma unroll
            for (int jt = 0; jt < 4; ++jt) {
                const unsigned off = (voff + 8u * unsigned(jt & 1)) ^ (jt >= 2 ? 64u : 0u);
                const bf16x8 vv = join(short_tr(off + unsigned(t0) * kValueTile), short_tr(off + unsigned(t1) * kValueTile));
                O[jt] = mfma(vv, h, mfma(vv, l, O[jt]));
            }
        };
        const int own_pair = w >> 1, pairs = (n_tiles + 1) >> 1, sibling = min(w ^ 1, n_tiles - 1);
        const bool odd = (w & 1) != 0;
        Keys k0 = key_rows(at.kf, 0), k1 = key_rows(at.kf, min(1, n_tiles - 1));
        auto forward = [&](int first, int last, const bf16x8 *q) __attribute__((always_inline)) {
            for (int p = first; p < last; ++p) {
                const f32x4 p0 = scores(k0, q), p1 = scores(k1, q);
                k0 = key_rows(at.kf, 2 * p + 2);
                k1 = key_rows(at.kf, min(2 * p + 3, n_tiles - 1));
                add_pair(2 * p, 2 * p + 1, p0, p1);
            }
        };
        auto backward = [&](int first, int last, const bf16x8 *q) __attribute__((always_inline)) {
            for (int p = first; p < last; ++p) {
                const f32x4 p0 = scores(k0, q);
                f32x4 p1 = scores(k1, q);
                const int second = min(2 * p + 1, n_tiles - 1);
                if (second == 2 * p) p1 = zero;
                k0 = key_rows(at.kb, min(2 * p + 2, n_tiles - 1));
                k1 = key_rows(at.kb, min(2 * p + 3, n_tiles - 1));
                add_pair(2 * p, second, p0, p1);
            }
        };
        // (apart: the pairs of the other half, before the upper one and after the lower one)
        const int other_before = apart && !low ? mid >> 1 : 0, own_last = apart && low ? mid >> 1 : pairs;
        if constexpr (kHalves) forward(0, other_before, qc);
        forward(other_before, own_pair, qx[0]);
        {
            // the own tile, and beside it the one before it (forward) or after it (backward; there may be none)
            const Keys c = key_rows(at.kb, sibling);
            const int next = 2 * min(own_pair + 1, pairs - 1);
            f32x4 other = odd ? scores(k0, qx[0]) : scores(c, qx[1]);
            if (sibling == w) other = zero;
            k0 = key_rows(at.kb, next);
            k1 = key_rows(at.kb, min(next + 1, n_tiles - 1));
            add_pair(w, sibling, own, other);
        }
        backward(own_pair + 1, own_last, qx[1]);
        if constexpr (kHalves) backward(own_last, pairs, qc);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const uint2 a = pack4(O[2 * kk]), b = pack4(O[2 * kk + 1]);
            __builtin_amdgcn_raw_buffer_store_b128(u32x4{a.x, a.y, b.x, b.y}, io.out, unsigned(16 * w + r) * io.pitch + 16u * unsigned(g) + 64u * unsigned(kk), 0, 0);
        }
    }
    // (tested anew: see bigla_short_kernel)
    asm volatile("" : "+s"(safe));
    if (safe != 0)
        short_slab_safe<kDk, kTm>(q_all, k_all, v_all, gf_all, gb_all, out_all, eb_all + slab * (2 * kShortTiles * kD), slab, 0, w,
                                  n_tiles, L, n_tiles, heads);
}

}  // namespace

}  // namespace vig
