// Chunkwise bf16 MFMA evaluation of the gradient of the BiGLA token mixer (Section 4.2.1,
// Eq. (BiGLA); the paper trains through it, Section 5, and prints no gradient formulas) for
// dv = 64 and dk = 64 (or 32, widened to 64 with zero channels) in bf16: the counterpart of the
// chunkwise forward kernels.
//
// One direction, forward (the backward one is its mirror image: suffix sums, keys to the right).
// Inside a chunk of 64 tokens let b_t be the inclusive cumulative log-gate since the chunk's left
// edge, E+ = exp(b), E- = exp(-b), q~ = q * E+, k~ = k * E-, do' = d_out / 2.  With
//   S_in : the state entering the chunk (after the previous chunk's last token), [dk][dv]
//   A'   : diag(exp(b_end)) times the adjoint of the chunk's end state due to all later chunks
// the regrouped chain rule is, with the masks s <= t,
//   P  = mask(q~ k~^T)             dP = mask(do' v^T)                          [t][s]
//   X  = dP k~ + do' S_in^T        dq = E+ * X
//   Yi = dP^T q~   Ye = v A'^T     dk = E- * (Yi + Ye)
//   dv = P^T do' + k~ A'
//   dg_u = sum_{t >= u} (q~ * X - k~ * Yi)_t + sum_{t < u} (k~ * Ye)_t + rowsum(S_in * A')
// (the three parts of dg are the token pairs (s, t), s < u <= t, that straddle u: both inside the
// chunk or s before it; s inside and t after it; s before and t after).  Every sum of dg runs over
// at most one chunk, so no long-range cancellation enters it; its two prefix/suffix sums are fp32
// scans over the wave's tokens (DPP row operations) plus the other waves' totals.
// The four state matrices of every chunk (the state entering it and A', both directions) come from
//   bigla_bwd_chunk_walk_kernel (a workgroup per slab and matrix, walking the slab's chunks with the running
//   matrix in registers), where there are enough slabs to fill the chip that way or few chunks to walk;
// otherwise from two small launches:
//   1. bigla_bwd_chunk_local_kernel (workgroup per chunk): the chunk's own contributions
//      U = (k * exp(b_end - b))^T v and W = q~^T do' for both directions, and the chunk totals of
//      the log-gates;
//   2. bigla_bwd_chunk_scan_kernel (elementwise over the 64x64 matrices, sequential over the
//      chunks of a slab): S_in(c+1) = d_c S_in(c) + U_c and A'_c = d_c (W_{c+1} + A'_{c+1}), in
//      place, fp32 running values, bf16 storage.
// Either leaves marks of the slabs in which some chunk's total log-decay exceeds 60 nats in some channel.  Then
//   bigla_bwd_chunk_main_kernel (workgroup per chunk): everything above for both directions at once (bigla_bwd_main.hpp).
// exp(-b) grows with the decay accumulated over a chunk, so marked slabs are evaluated token by token (exact_sweep.hpp) by
// the workgroups of the main launch; gates of the paper's form,
// sigmoid(z)^(1/16), reach 60 nats in 64 steps only for z < -15 throughout.
//
// Wavefront mapping of the passes that make the states (256 threads = 4 waves): wave w owns tokens 16w..16w+15 of the chunk; lane
// (r = lane%16, g = lane/16) holds, for token 16w + r, channels 16ct + 4g + e (ct, e = 0..3) -- four 8-byte pieces of the
// token's row.  All tiles are row-major bf16 in LDS; an operand whose contraction index runs along the tile's rows is read
// with ds_read_b64_tr_b16.  Tokens past the sequence are read as zeros (q = k = v = do = 0, log-gate 0: a no-op) and their
// stores are dropped, both by the bounds check of the buffer resource that spans the slab.
#include <algorithm>
#include <type_traits>

#include "exact_sweep.hpp"
#include "vig_common.hpp"
#include "vig_kernels.hpp"
#include "vig_timing.hpp"

namespace vig {

namespace {

constexpr int kC = 64;       // chunk length (tokens)
constexpr int kD = 64;       // dk = dv
constexpr int kPitch = 72;   // LDS row pitch in bf16 elements
constexpr int kThreads = 256;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kFastRange = 60.0f;  // largest chunk log-decay (nats, any channel) this path accepts
constexpr size_t kMat = size_t(kD) * kD;  // elements of one state matrix

typedef uint16_t Tile[kC][kPitch];

// MFMA operand whose 16 rows (A) or columns (B) are tile columns col0..col0+15 and whose contraction
// index runs along the tile's rows: k-slot j of K-step kk is row 32kk + 8g + j.
__device__ __forceinline__ bf16x8 col_frag(const Tile &tile, int col0, int kk, int r, int g)
{
    const int row = 32 * kk + 8 * g + (r >> 2), col = col0 + 4 * (r & 3);
    return join(lds_read_tr(&tile[row][col]), lds_read_tr(&tile[row + 4][col]));
}

// B operand of a contraction over the chunk's tokens with a 0/1 triangle: k-slot j of K-step kk is
// token s = 32kk + 8g + j, the lane's column is token u; 1 where s REL u holds.
enum Rel { kLe = 0, kGe = 1 };
template <int REL>
__device__ __forceinline__ bf16x8 tri_frag(int kk, int g, int u)
{
    uint32_t word[4];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        uint32_t bits = 0;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int s = 32 * kk + 8 * g + 2 * jj + half;
            const bool one = REL == kLe ? s <= u : s >= u;
            bits |= (one ? 0x3F80u : 0u) << (16 * half);
        }
        word[jj] = bits;
    }
    return __builtin_bit_cast(bf16x8, make_uint4(word[0], word[1], word[2], word[3]));
}

// One slab's rows of a [.., width] bf16 tensor (width 64, or 32 for the queries, keys and gates of
// a 32-wide head) behind a buffer resource that ends with the slab's last token (loads beyond it
// return zeros, stores beyond it are dropped).  Rows of 32 are widened to the kernels' 64 channels
// with zeros: channels 32..63 then carry q = k = 0 and log-gate 0 through every step and their
// results are not stored; the pieces of the missing half are requested, and stored, at an offset
// beyond the extent.
struct SlabRows {
    __amdgpu_buffer_rsrc_t rsrc;
    unsigned pitch;   // bytes between consecutive tokens
    unsigned pieces;  // 16-byte pieces per row: 8 or 4
};
constexpr unsigned kBeyond = 0xfffffff0u;

__device__ __forceinline__ SlabRows slab_rows(const void *base, size_t first, int L, int heads_token_major, int width = kD)
{
    const unsigned pitch = 2u * unsigned(width) * unsigned(heads_token_major ? heads_token_major : 1);
    const unsigned extent = unsigned(L - 1) * pitch + 2u * unsigned(width);
    SlabRows s;
    s.rsrc = slab_resource(static_cast<const char *>(base) + first * (2 * size_t(width)), extent);
    s.pitch = pitch;
    s.pieces = unsigned(width) / 8u;
    return s;
}

// Whole rows of a chunk: lane i of wave w takes 16-byte piece i%8 of rows 16w + i/8 and 16w + 8 + i/8.
// Requested first (all of a phase's tensors together), put into a tile when they are needed.
struct ChunkRows {
    u32x4 p[2];
};

// wanted: false reads zeros, without going to memory
__device__ __forceinline__ ChunkRows fetch_rows(const SlabRows &rows, unsigned t0, int w, int lane, bool wanted = true)
{
    ChunkRows c;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const unsigned off = (t0 + 16 * w + 8 * h + (lane >> 3)) * rows.pitch + 16u * (lane & 7);
        c.p[h] = __builtin_amdgcn_raw_buffer_load_b128(rows.rsrc, wanted && unsigned(lane & 7) < rows.pieces ? off : kBeyond, 0, 0);
    }
    return c;
}

// kHalf: the values are halved on the way (exact in bf16).
template <bool kHalf>
__device__ __forceinline__ void put_rows(Tile &tile, const ChunkRows &c, int w, int lane)
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        u32x4 x = c.p[h];
        if (kHalf) {
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = pack2(0.5f * bf16_lo_to_f32(x[i]), 0.5f * bf16_hi_to_f32(x[i]));
        }
        *reinterpret_cast<uint4 *>(&tile[16 * w + 8 * h + (lane >> 3)][8 * (lane & 7)]) = make_uint4(x[0], x[1], x[2], x[3]);
    }
}

// Orders this wave's earlier LDS writes before its later LDS reads of what other lanes of the
// same wave wrote (the LDS executes one wave's accesses in order; this keeps the compiler from
// moving them across each other).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The lane's own four pieces of a token row (channels 16ct + 4g .. + 3 of token 16w + r) out of
// rows the wave has staged itself: rows 16w..16w+15 of a tile belong to wave w alone.
__device__ __forceinline__ void take_own(const Tile &tile, int w, int r, int g, uint2 (&x)[4])
{
    wave_lds_fence();
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) x[ct] = *reinterpret_cast<const uint2 *>(&tile[16 * w + r][16 * ct + 4 * g]);
}

// the lane's piece of tile row 16w + r
__device__ __forceinline__ void put_own(Tile &tile, int w, int r, int g, int ct, const f32x4 &x)
{
    *reinterpret_cast<uint2 *>(&tile[16 * w + r][16 * ct + 4 * g]) = pack4(x);
}

// Inclusive cumulative log-gates of the chunk on the matrix cores (a product with a 0/1 triangle is
// exact in bf16 x bf16 -> fp32): b[ct][e] for the lane's token and channel 16ct + 4g + e, prefix
// sums for DIR 0, suffix sums for DIR 1.
template <int DIR, int kCt>
__device__ __forceinline__ void gate_scan(const Tile &gates, int w, int r, int g, f32x4 (&b)[4])
{
    const bf16x8 t0 = tri_frag<DIR == 0 ? kLe : kGe>(0, g, 16 * w + r);
    const bf16x8 t1 = tri_frag<DIR == 0 ? kLe : kGe>(1, g, 16 * w + r);
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        b[ct] = zero;
        if (ct < kCt) b[ct] = mfma(col_frag(gates, 16 * ct, 1, r, g), t1, mfma(col_frag(gates, 16 * ct, 0, r, g), t0, zero));
    }
}

// ---- workspace ---------------------------------------------------------------------------------
// [states][log-decays][slab marks]
//   states, per (slab, chunk): four bf16 64x64 matrices, row-major [key channel][value column]:
//     0: forward  state entering the chunk from the left      (pass 1 leaves U there)
//     1: forward  A' of the chunk (decayed adjoint from the right)     (pass 1: W)
//     2: backward state entering the chunk from the right
//     3: backward A' of the chunk (decayed adjoint from the left)
//     (0 and 3 of a slab's first chunk and 1 and 2 of its last are zero; the main pass does not read them, the walks do not write them)
//   log-decays, per (slab, chunk, direction): the chunk's total log-gate per channel, fp32
//   slab marks: two bytes per slab (walks: one of each direction), not both zero when the slab takes the exact form; with
//     zeros up to a multiple of kShareSlabs slabs
constexpr unsigned kShareSlabs = 16;  // slabs whose workgroups share out the exact form of the marked ones among them
__device__ __forceinline__ void end_marks(uint16_t *marks, unsigned n_slabs, unsigned lane)  // the zeros, a wave's work
{
    if (lane < (0u - n_slabs) % kShareSlabs) marks[size_t(n_slabs) + lane] = 0;
}

struct Workspace {
    uint16_t *states;
    float *logdec;
    uint16_t *marks;
};

inline size_t align256(size_t n) { return (n + 255) / 256 * 256; }

inline int chunks_of(int L) { return (L + kC - 1) / kC; }

inline size_t states_bytes(long BH, int L) { return align256(size_t(BH) * chunks_of(L) * 4 * kMat * sizeof(uint16_t)); }
inline size_t logdec_bytes(long BH, int L) { return align256(size_t(BH) * chunks_of(L) * 2 * kD * sizeof(float)); }
inline size_t marks_bytes(long BH) { return align256((size_t(BH) + kShareSlabs - 1) / kShareSlabs * kShareSlabs * 2); }

struct LocalLds {
    Tile v, dout, gates, qt, kh;
};

// ---- pass 1: the chunk's own contributions to the states ----------------------------------------
// kCt: channel tiles of 16 that carry data (4; 2 for a 32-wide head, whose channels 32..63 are zero
// in q, k and the gates: their rows of the matrices are neither computed, stored nor read anywhere).
template <int kCt>
__global__ __launch_bounds__(kThreads, 2) void bigla_bwd_chunk_local_kernel(
    const void *__restrict__ q_all, const void *__restrict__ k_all, const void *__restrict__ v_all,
    const void *__restrict__ gf_all, const void *__restrict__ gb_all, const void *__restrict__ do_all,
    uint16_t *__restrict__ states, float *__restrict__ logdec, uint16_t *__restrict__ marks, int L, int heads_token_major, int n_chunks,
    int dk)
{
    __shared__ __align__(16) LocalLds sm;
    const unsigned unit = blockIdx.x, slab = unit / unsigned(n_chunks);
    const unsigned t0 = (unit - slab * unsigned(n_chunks)) * kC;
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, r = lane & 15, g = lane >> 4;
    if (unit == 0 && w == 0) end_marks(marks, gridDim.x / unsigned(n_chunks), unsigned(lane));

    const size_t first = slab_first_row(slab, L, heads_token_major);
    const SlabRows q = slab_rows(q_all, first, L, heads_token_major, dk), k = slab_rows(k_all, first, L, heads_token_major, dk);
    const SlabRows v = slab_rows(v_all, first, L, heads_token_major), dout = slab_rows(do_all, first, L, heads_token_major);
    const SlabRows gf = slab_rows(gf_all, first, L, heads_token_major, dk), gb = slab_rows(gb_all, first, L, heads_token_major, dk);

    uint2 qr[4], kr[4];
    {
        const ChunkRows cq = fetch_rows(q, t0, w, lane), ck = fetch_rows(k, t0, w, lane);
        const ChunkRows cv = fetch_rows(v, t0, w, lane), cd = fetch_rows(dout, t0, w, lane);
        put_rows<false>(sm.qt, cq, w, lane);
        put_rows<false>(sm.kh, ck, w, lane);
        put_rows<false>(sm.v, cv, w, lane);
        put_rows<true>(sm.dout, cd, w, lane);
    }
    ChunkRows cg[2] = {fetch_rows(gf, t0, w, lane), fetch_rows(gb, t0, w, lane)};
    take_own(sm.qt, w, r, g, qr);
    take_own(sm.kh, w, r, g, kr);

    uint16_t *mats = states + size_t(unit) * 4 * kMat;
    const bf16x8 ones = __builtin_bit_cast(bf16x8, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));

#pragma unroll
    for (int dir = 0; dir < 2; ++dir) {
        if (dir == 1) __syncthreads();  // the first direction's products have read the tiles
        put_rows<false>(sm.gates, cg[dir], w, lane);
        __syncthreads();
        f32x4 b[4], T[4];
        if (dir == 0)
            gate_scan<0, kCt>(sm.gates, w, r, g, b);
        else
            gate_scan<1, kCt>(sm.gates, w, r, g, b);
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            if (ct >= kCt) {  // no data: total log-gate 0 (the scan of the marks reads every channel)
                if (w == 0 && r == 0) *reinterpret_cast<f32x4 *>(&logdec[(size_t(unit) * 2 + dir) * kD + 16 * ct + 4 * g]) = zero;
                continue;
            }
            T[ct] = mfma(col_frag(sm.gates, 16 * ct, 1, r, g), ones, mfma(col_frag(sm.gates, 16 * ct, 0, r, g), ones, zero));
            const f32x4 qv = unpack4(qr[ct]), kv = unpack4(kr[ct]);
            f32x4 qs, ks;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                qs[e] = qv[e] * fast_exp2(b[ct][e] * kLog2e);
                ks[e] = kv[e] * fast_exp2((T[ct][e] - b[ct][e]) * kLog2e);
            }
            put_own(sm.qt, w, r, g, ct, qs);
            put_own(sm.kh, w, r, g, ct, ks);
            if (w == 0 && r == 0)
                *reinterpret_cast<f32x4 *>(&logdec[(size_t(unit) * 2 + dir) * kD + 16 * ct + 4 * g]) = T[ct];
        }
        __syncthreads();
        // U^T[j][i] = sum_t v[t][j] kh[t][i],  W^T[j][i] = sum_t do'[t][j] q~[t][i]: a wave takes 16 rows
        // i (and, with two row tiles only, half of the column tiles), the lane ends up with four
        // consecutive columns j of its row
        uint16_t *U = mats + size_t(2 * dir) * kMat, *W = U + kMat;
        const int it = kCt == 4 ? w : (w & 1);          // row tile
        const int mt0 = kCt == 4 ? 0 : 2 * (w >> 1);    // first column tile
#pragma unroll
        for (int mi = 0; mi < kCt; ++mi) {
            const int mt = mt0 + mi;
            f32x4 u = {0.f, 0.f, 0.f, 0.f}, x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                u = mfma(col_frag(sm.v, 16 * mt, kk, r, g), col_frag(sm.kh, 16 * it, kk, r, g), u);
                x = mfma(col_frag(sm.dout, 16 * mt, kk, r, g), col_frag(sm.qt, 16 * it, kk, r, g), x);
            }
            *reinterpret_cast<uint2 *>(&U[(16 * it + r) * kD + 16 * mt + 4 * g]) = pack4(u);
            *reinterpret_cast<uint2 *>(&W[(16 * it + r) * kD + 16 * mt + 4 * g]) = pack4(x);
        }
    }
}

// ---- pass 2: the chunk-to-chunk recurrences, elementwise ------------------------------------------
// grid: 16 workgroups per slab = 4 matrices x 4 quarters; a thread owns 4 consecutive elements of a
// row and walks the slab's chunks in the matrix's direction, its loads requested kScanAhead chunks
// ahead (the walk is a chain of dependent fp32 operations, but the addresses are known; measured at
// 64 chunks per slab: 69 / 66 / 62 / 56 us for 4 / 8 / 16 / 32 chunks ahead; with 4 chunks per slab
// the deep version only pays for its longer prologue, 25 us against 17 us).
constexpr int kScanThreads = 256;

template <int kScanAhead, int kCt>
__global__ __launch_bounds__(kScanThreads) void bigla_bwd_chunk_scan_kernel(uint16_t *__restrict__ states,
                                                                       const float *__restrict__ logdec,
                                                                       uint16_t *__restrict__ marks, int n_chunks)
{
    constexpr int kScanParts = kCt * 256 / kScanThreads;  // workgroups per matrix: 16 * kCt rows of 16 pieces
    const unsigned slab = blockIdx.x / (4 * kScanParts);
    const int kind = (blockIdx.x / kScanParts) & 3, part = blockIdx.x % kScanParts;
    const int tid = threadIdx.x;
    const int piece = part * kScanThreads + tid;  // 0 .. 256 * kCt - 1
    const int row = piece >> 4;
    const int dir = kind >> 1;
    const bool adjoint = (kind & 1) != 0;
    const bool ascending = kind == 0 || kind == 3;

    if (kind == 0 && part == 0) {
        // mark the slab when some chunk decays by more than the fast form can carry
        __shared__ float lowest[kScanThreads];
        float m = 0.f;
        const float *ld = logdec + size_t(slab) * n_chunks * 2 * kD;
        for (long i = tid; i < long(n_chunks) * 2 * kD; i += kScanThreads) m = fminf(m, ld[i]);
        lowest[tid] = m;
        __syncthreads();
        for (int s = kScanThreads / 2; s > 0; s >>= 1) {
            if (tid < s) lowest[tid] = fminf(lowest[tid], lowest[tid + s]);
            __syncthreads();
        }
        // (a NaN gate total compares false and leaves the slab to this path, whose outputs are then NaN too)
        if (tid == 0) marks[slab] = (-lowest[0] > kFastRange) ? 1 : 0;
    }

    uint16_t *mat = states + (size_t(slab) * n_chunks * 4 + kind) * kMat + size_t(piece) * 4;
    const float *ld = logdec + (size_t(slab) * n_chunks * 2 + dir) * kD + row;
    struct Item {
        uint2 x;
        float logd;
    };
    auto fetch = [&](int n) {
        Item it;
        it.x = make_uint2(0u, 0u);
        it.logd = 0.f;
        if (n < n_chunks) {
            const int c = ascending ? n : n_chunks - 1 - n;
            it.x = *reinterpret_cast<const uint2 *>(mat + size_t(c) * 4 * kMat);
            it.logd = ld[size_t(c) * 2 * kD];
        }
        return it;
    };
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    Item ahead[kScanAhead];
#pragma unroll
    for (int j = 0; j < kScanAhead; ++j) ahead[j] = fetch(j);
    for (int n0 = 0; n0 < n_chunks; n0 += kScanAhead) {
#pragma unroll
        for (int j = 0; j < kScanAhead; ++j) {
            const int n = n0 + j;
            if (n < n_chunks) {
                const Item cur = ahead[j];
                ahead[j] = fetch(n + kScanAhead);
                const int c = ascending ? n : n_chunks - 1 - n;
                const float d = fast_exp2(cur.logd * kLog2e);
                const f32x4 u = unpack4(cur.x);
                f32x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (adjoint) {
                        o[e] = d * s[e];     // A' of this chunk
                        s[e] = u[e] + o[e];  // adjoint of the previous chunk's end state
                    } else {
                        o[e] = s[e];         // state entering this chunk
                        s[e] = d * s[e] + u[e];
                    }
                }
                *reinterpret_cast<uint2 *>(mat + size_t(c) * 4 * kMat) = pack4(o);
            }
        }
    }
}

// ---- passes 1 and 2 in one: a workgroup walks a slab for one of its four matrices --------------------
// The running matrix stays in registers (fp32) and what enters each chunk is written once; a tensor is read by the two
// walks that need it, which are at opposite ends of the slab: with the matrices 385 MB at 48 slabs of 4096 tokens, 70 us at the rate of a
// copy, which is what bounds the walks there (preparing two chunks at a time with eight waves: 156 us a call against 156).  Leaving out
// the rows of the last chunk and the zero matrices of the first: 75.4 -> 72.4 us a call at 384 slabs of 196 tokens, 158 -> 152 at 192 of 1024.  A chunk is a chain of a gate scan, exponentials and
// scalings and then the products; four waves do the first half of chunk n + 1 while four do the second half of chunk n, one
// barrier per chunk, on tiles that alternate.  Rows are requested two chunks before their turn.
constexpr int kWalkThreads = 2 * kThreads;
// The time of the walks goes with the chunks to walk, 1 us each, until about half the compute units have one; the two passes
// take the same time per chunk at any shape.  A gradient call with the walks against the passes (event times): 48 heads of 4096
// tokens 181 us against 198, 36: 150 / 158, 30: 138 / 140, 24: 119 / 117, 6: 82 / 60; 30 heads of 1961 tokens 73 / 76, 15: 56 / 50;
// 48 heads of 1024 tokens 53 / 62, 12: 37 / 37; 384 heads of 196 tokens 94 / 104, 24: 24 / 28, 6: 22 / 25.
constexpr long kWalkWorkgroups = 112;
constexpr int kWalkShort = 8;

struct WalkLds {
    Tile gates[2], x[2], y[2];
    float total[2][kD];  // the chunk's total log-gate per channel
};

template <int kCt>
__global__ __launch_bounds__(kWalkThreads, 4) void bigla_bwd_chunk_walk_kernel(
    const void *__restrict__ q_all, const void *__restrict__ k_all, const void *__restrict__ v_all,
    const void *__restrict__ gf_all, const void *__restrict__ gb_all, const void *__restrict__ do_all,
    uint16_t *__restrict__ states, uint16_t *__restrict__ marks, int L, int heads_token_major,
    int n_chunks, unsigned n_slabs)
{
    constexpr int dk = 16 * kCt;
    __shared__ __align__(16) WalkLds sm;
    // a slab's four walks on one XCD (workgroups go round-robin over the eight) and next to each other in time, where
    // the slabs divide by eight
    unsigned slab, kind_no;
    if (n_slabs % 8 == 0) {
        kind_no = blockIdx.x / 8 % 4;
        slab = blockIdx.x / 32 * 8 + blockIdx.x % 8;
    } else {
        kind_no = blockIdx.x % 4;
        slab = blockIdx.x / 4;
    }
    const int kind = int(kind_no), dir = kind >> 1;
    const bool adjoint = (kind & 1) != 0, ascending = kind == 0 || kind == 3;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x)) >> 6;
    const int w = wave & 3, lane = int(threadIdx.x) & 63, r = lane & 15, g = lane >> 4;
    // (past the end: the last one once more, loaded and not used; without a branch, which would make every wait a full one)
    const int chunk0 = ascending ? 0 : n_chunks - 1, chunk_step = ascending ? 1 : -1;
    auto chunk_of = [&](int n) { return chunk0 + chunk_step * min(n, n_chunks - 1); };

    if (wave < 4) {
        const size_t first = slab_first_row(slab, L, heads_token_major);
        const SlabRows xs = slab_rows(adjoint ? q_all : k_all, first, L, heads_token_major, dk);
        const SlabRows ys = slab_rows(adjoint ? do_all : v_all, first, L, heads_token_major);
        const SlabRows gs = slab_rows(dir == 0 ? gf_all : gb_all, first, L, heads_token_major, dk);
        // (what the last chunk would add to the matrix enters no chunk: its rows are not read, only its gates)
        auto fetch_gates = [&](int n) { return fetch_rows(gs, unsigned(chunk_of(n)) * kC, w, lane); };
        auto fetch = [&](const SlabRows &rows, int n) { return fetch_rows(rows, unsigned(chunk_of(n)) * kC, w, lane, n < n_chunks - 1); };
        bf16x8 tri[2];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) tri[kk] = dir == 0 ? tri_frag<kLe>(kk, g, 16 * w + r) : tri_frag<kGe>(kk, g, 16 * w + r);
        const bf16x8 ones = __builtin_bit_cast(bf16x8, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));
        // keys of a state decay to the chunk's far edge, exp(total - b); queries of an adjoint from its near edge, exp(b),
        // and carry the 1/2 of d_out / 2
        const float of_scan = adjoint ? kLog2e : -kLog2e, of_total = adjoint ? 0.f : kLog2e, bias = adjoint ? -1.f : 0.f;
        // gates in tile gates[buf], the wave's own rows of x in tile x[buf] -> scaled x and the totals in tiles [buf]
        auto scale_rows = [&](int buf) __attribute__((always_inline)) {
            uint2 own[4];
            take_own(sm.x[buf], w, r, g, own);
#pragma unroll
            for (int ct = 0; ct < kCt; ++ct) {
                const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                const bf16x8 a0 = col_frag(sm.gates[buf], 16 * ct, 0, r, g), a1 = col_frag(sm.gates[buf], 16 * ct, 1, r, g);
                const f32x4 b = mfma(a1, tri[1], mfma(a0, tri[0], zero)), T = mfma(a1, ones, mfma(a0, ones, zero));
                f32x4 x = unpack4(own[ct]);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] *= fast_exp2(fmaf(of_scan, b[e], fmaf(of_total, T[e], bias)));
                put_own(sm.x[buf], w, r, g, ct, x);
                if (w == 0 && r == 0) *reinterpret_cast<f32x4 *>(&sm.total[buf][16 * ct + 4 * g]) = T;
            }
        };
        ChunkRows cg[2], cx[2], cy[2];
        cg[0] = fetch_gates(0);
        put_rows<false>(sm.gates[0], cg[0], w, lane);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            cx[j] = fetch(xs, j);
            cy[j] = fetch(ys, j);
            cg[j ^ 1] = fetch_gates(j + 1);
        }
        // chunk n + 1 into the tiles of parity j ^ 1, the gates of chunk n + 2 into those of parity j, and the next requests
        auto advance = [&](int j, int n) __attribute__((always_inline)) {
            put_rows<false>(sm.x[j ^ 1], cx[j ^ 1], w, lane);
            put_rows<false>(sm.y[j ^ 1], cy[j ^ 1], w, lane);
            put_rows<false>(sm.gates[j], cg[j], w, lane);
            cx[j ^ 1] = fetch(xs, n + 3);
            cy[j ^ 1] = fetch(ys, n + 3);
            cg[j] = fetch_gates(n + 4);
            scale_rows(j ^ 1);
        };
        __syncthreads();
        advance(1, -1);
        // (what is prepared past the last chunk is a repetition of it, unused; two chunks per turn without a way out in
        // between, which would make the waits of the first half full ones)
        for (int n = 0; n + 1 < n_chunks; n += 2) {
            __syncthreads();
            advance(0, n);
            __syncthreads();
            advance(1, n + 1);
        }
        if (n_chunks & 1) __syncthreads();
        return;
    }

    const int it = kCt == 4 ? w : (w & 1);        // the wave's row tile of the matrix
    const int mt0 = kCt == 4 ? 0 : 2 * (w >> 1);  // its first column tile
    const int row = 16 * it + r;
    uint16_t *mats = states + (size_t(slab) * unsigned(n_chunks) * 4 + kind_no) * kMat + row * kD + 4 * g;
    bool beyond = false;
    f32x4 s[kCt];
#pragma unroll
    for (int mi = 0; mi < kCt; ++mi) s[mi] = f32x4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();
    auto step = [&](int j, int n) __attribute__((always_inline)) {
        const float d = fast_exp2(sm.total[j][row] * kLog2e);
        beyond = beyond || -sm.total[j][lane % dk] > kFastRange;  // (every wave: all channels)
        uint16_t *mat = mats + size_t(chunk_of(n)) * 4 * kMat;
        bf16x8 xf[2];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) xf[kk] = col_frag(sm.x[j], 16 * it, kk, r, g);
#pragma unroll
        for (int mi = 0; mi < kCt; ++mi) {
            const int mt = mt0 + mi;
            f32x4 t, o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                t[e] = d * s[mi][e];
                o[e] = adjoint ? t[e] : s[mi][e];
            }
            if (n > 0) *reinterpret_cast<uint2 *>(mat + 16 * mt) = pack4(o);  // (nothing enters the first chunk, and nobody reads it)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) t = mfma(col_frag(sm.y[j], 16 * mt, kk, r, g), xf[kk], t);
            s[mi] = t;
        }
    };
    int n = 0;
    for (; n + 1 < n_chunks; n += 2) {
        __syncthreads();
        step(0, n);
        __syncthreads();
        step(1, n + 1);
    }
    if (n < n_chunks) {
        __syncthreads();
        step(0, n);
    }
    // mark the slab when some chunk decays by more than the fast form can carry (a NaN gate total compares false and
    // leaves the slab to this path, whose outputs are then NaN too)
    if (!adjoint && w == 0) {
        const bool any = __any(beyond);
        if (lane == 0) reinterpret_cast<uint8_t *>(marks)[2 * size_t(slab) + dir] = any ? 1 : 0;
        if (slab == n_slabs - 1 && dir == 0) end_marks(marks, n_slabs, unsigned(lane));
    }
}

}  // namespace

}  // namespace vig

#include "bigla_bwd_main.hpp"

namespace vig {

namespace {

// ---- pass 3: the gradients of one chunk ------------------------------------------------------------

// Marked slabs: the workgroups of every sixteen slabs share out the strips of the exact form, two pairs of waves at a time,
// of those that are marked among them.  Inside this launch and not in one of its own: a launch that finds no marked
// slab still took 4.7 us (and two of them, 9.5 us, were 7 % of a call at 384 slabs of 196 tokens).  A gradient call with one
// marked slab, and with all marked: 48 slabs of 64 tokens 27 and 50 us (a slab's strips dealt to the workgroups of its own
// chunks, from a function that spilled: 410 and 476; the token-by-token kernels before these, in launches of their own: 65 and
// 107), 384 of 196 tokens 113 and 634 us (298 / 1494; 218 / 1052), 48 of 4096 tokens 0.84 and 1.60 ms (0.94 / 3.42; 2.35 / 2.41).
// What the exact form needs is a kernel argument of its own, read where it is used: the chunkwise code's copies of the same
// pointers, kept for it, cost that code scalar registers.
struct ExactArgs {
    const bf16_t *q, *k, *v, *gf, *gb, *d_out;
    bf16_t *dq, *dk, *dv, *dgf, *dgb;
    float *parts;
    int L, heads_token_major;
    unsigned n_slabs, workers_per_slab;
};

template <int DK>
__device__ __forceinline__ void exact_strips(const ExactArgs &a, RowStage<kD> (&stage)[4], unsigned first_slab,
                                             unsigned marked /* a bit per slab from there on */, unsigned worker, unsigned workers)
{
    constexpr unsigned kRowItems = DK / kStrip / 2, kColItems = kD / (kStrip * (kD / DK)) / 2;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x)) >> 6;
    const bool descending = (wave & 1) != 0;
    const size_t step = a.heads_token_major ? a.heads_token_major : 1, keys = size_t(a.L) * DK, all_keys = keys * a.n_slabs;
    const unsigned n_marked = unsigned(__popc(marked));
    PartStage<1, 2> whole;
#pragma unroll 1
    for (unsigned i = worker; i < n_marked * (kRowItems + kColItems); i += workers) {
        // (what depends on the lane is formed anew for every strip: hoisted out of this loop, the offsets of both kinds of
        // strips together spilled 2 KB a lane, and a strip took three times as long)
        int lane = int(threadIdx.x) & 63;
        asm volatile("" : "+v"(lane));
        const unsigned item = i / n_marked;
        unsigned bits = marked;
        for (unsigned skip = i - item * n_marked; skip > 0; --skip) bits &= bits - 1;
        const unsigned slab = first_slab + unsigned(__ffs(int(bits)) - 1);
        const size_t row0 = slab_first_row(slab, a.L, a.heads_token_major), k0 = row0 * DK, v0 = row0 * kD;
        float *parts = a.parts + slab * keys;
        if (item < kRowItems)
            row_sweep<bf16_t, DK, kD>(a.q + k0, a.k + k0, a.v + v0, a.gf + k0, a.gb + k0, a.d_out + v0, a.dq + k0, a.dk + k0,
                                      a.dgf + k0, a.dgb + k0, parts, parts + all_keys, stage[wave], step, a.L, descending, 0, whole,
                                      int(2 * item) + (wave >> 1), lane);
        else
            column_sweep<bf16_t, DK, kD, true>(a.q + k0, a.k + k0, (descending ? a.gf : a.gb) + k0, a.d_out + v0,
                                               a.parts + 2 * all_keys + size_t(slab) * a.L * kD, a.dv + v0, step, 1, a.L,
                                               descending, 0, whole, int(2 * (item - kRowItems)) + (wave >> 1), 0.5f, 1.f, lane);
    }
}

template <int kCt>
__global__ __launch_bounds__(kThreads, 2) void bigla_bwd_chunk_main_kernel(
    const void *__restrict__ q_all, const void *__restrict__ k_all, const void *__restrict__ v_all,
    const void *__restrict__ gf_all, const void *__restrict__ gb_all, const void *__restrict__ do_all,
    void *__restrict__ dq_all, void *__restrict__ dk_all, void *__restrict__ dv_all, void *__restrict__ dgf_all,
    void *__restrict__ dgb_all, const uint16_t *__restrict__ states, const uint16_t *__restrict__ marks, int L,
    int heads_token_major, int n_chunks, unsigned n_slabs, unsigned extra /* workgroups per slab without a chunk */,
    ExactArgs exact)
{
    constexpr int dk = 16 * kCt;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid) >> 6;
    const unsigned unit = blockIdx.x, units = n_slabs * unsigned(n_chunks);
    const bool has_chunk = unit < units;
    const unsigned slab = has_chunk ? unit / unsigned(n_chunks) : (unit - units) / extra;
    const unsigned chunk = unit - slab * unsigned(n_chunks);
    // the slabs that share out the exact form, and which of them take it (their marks are one scalar load, and as a rule all
    // zero; a lane each for the first look at them made calls on a few slabs 0.2 us longer)
    const unsigned first_slab = slab & ~(kShareSlabs - 1), sharing = min(kShareSlabs, n_slabs - first_slab);
    unsigned marked;
    const uint4 *group = reinterpret_cast<const uint4 *>(marks + first_slab);
    const uint4 m0 = group[0], m1 = group[1];
    marked = (m0.x | m0.y | m0.z | m0.w) | (m1.x | m1.y | m1.z | m1.w);
    if (marked != 0) marked = unsigned(__ballot(marks[first_slab + unsigned(lane) % kShareSlabs] != 0)) & ((1u << kShareSlabs) - 1u);
    const bool own_marked = (marked >> (slab - first_slab) & 1u) != 0;
    if (has_chunk && !own_marked) {
        const size_t first = slab_first_row(slab, L, heads_token_major);
        const GradRows io = {q_all, k_all, v_all, gf_all, gb_all, do_all, dq_all, dk_all, dv_all, dgf_all, dgb_all, first, L, heads_token_major};
        chunk_gradients<kCt>(io, states + size_t(unit) * 4 * kMat, chunk * kC, chunk == 0, chunk + 1 == unsigned(n_chunks), wave, lane, tid);
    }
    if (marked == 0) return;
    __syncthreads();  // the chunk's LDS is used anew
    // gates beyond the range of this form; workgroups without a chunk to do come first
    const unsigned below = unsigned(__popc(marked & ((1u << (slab - first_slab)) - 1u))), free_units = unsigned(__popc(marked)) * unsigned(n_chunks);
    unsigned worker;
    if (!has_chunk)
        worker = free_units + (unit - units - first_slab * extra);
    else if (own_marked)
        worker = below * unsigned(n_chunks) + chunk;
    else
        worker = free_units + sharing * extra + (slab - first_slab - below) * unsigned(n_chunks) + chunk;
    exact_strips<dk>(exact, *reinterpret_cast<RowStage<kD>(*)[4]>(g_grad_lds), first_slab, marked, worker, sharing * exact.workers_per_slab);
}

}  // namespace

bool bigla_bwd_chunk_supported(int dk, int dv, bool is_bf16) { return is_bf16 && (dk == kD || dk == kD / 2) && dv == kD; }

size_t bigla_bwd_chunk_workspace_bytes(long BH, int L)
{
    return states_bytes(BH, L) + logdec_bytes(BH, L) + marks_bytes(BH);
}

hipError_t bigla_bwd_chunk_launch(const void *q, const void *k, const void *v, const void *g_fwd, const void *g_bwd,
                                  const void *d_out, void *dq, void *dk, void *dv, void *dg_fwd, void *dg_bwd, long BH,
                                  int L, int dk_, int heads_token_major, void *workspace,
                                  float *exact_workspace, hipStream_t stream)
{
    const int n_chunks = chunks_of(L);
    const long units = BH * n_chunks;
    if (units > 0x7fffffffL || BH * 16 > 0x7fffffffL) return hipErrorInvalidValue;
    Workspace ws;
    char *base = static_cast<char *>(workspace);
    ws.states = reinterpret_cast<uint16_t *>(base);
    ws.logdec = reinterpret_cast<float *>(base + states_bytes(BH, L));
    ws.marks = reinterpret_cast<uint16_t *>(base + states_bytes(BH, L) + logdec_bytes(BH, L));
    auto launch = [&](auto ct) -> hipError_t {
        constexpr int kCt = decltype(ct)::value;
        // Walks as long as there are enough of them, or few chunks to walk; else a workgroup per chunk and a pass over the
        // matrices.
        const bool walk = BH * 4 >= kWalkWorkgroups || n_chunks <= kWalkShort;
        if (walk) {
            hipLaunchKernelGGL(bigla_bwd_chunk_walk_kernel<kCt>, dim3((unsigned)(BH * 4)), dim3(kWalkThreads), 0, stream, q, k, v,
                               g_fwd, g_bwd, d_out, ws.states, ws.marks, L, heads_token_major, n_chunks, unsigned(BH));
        } else {
            const dim3 scan_grid((unsigned)(BH * 4 * (kCt * 256 / kScanThreads)));
            hipLaunchKernelGGL(bigla_bwd_chunk_local_kernel<kCt>, dim3((unsigned)units), dim3(kThreads), 0, stream, q, k, v,
                               g_fwd, g_bwd, d_out, ws.states, ws.logdec, ws.marks, L, heads_token_major, n_chunks, dk_);
            if (n_chunks > 16)
                hipLaunchKernelGGL((bigla_bwd_chunk_scan_kernel<32, kCt>), scan_grid, dim3(kScanThreads), 0, stream, ws.states,
                                   ws.logdec, ws.marks, n_chunks);
            else
                hipLaunchKernelGGL((bigla_bwd_chunk_scan_kernel<8, kCt>), scan_grid, dim3(kScanThreads), 0, stream, ws.states,
                                   ws.logdec, ws.marks, n_chunks);
        }
        // Where the chunks leave compute units idle, workgroups without a chunk take strips of marked slabs (a slab
        // has 16 for a workgroup each, 12 with 32-wide keys), up to two workgroups a unit.
        const long extra = units < 512 ? std::min((512 - units) / BH, std::max(16L - n_chunks, 0L)) : 0;
        auto in = [](const void *p) { return static_cast<const bf16_t *>(p); };
        auto out = [](void *p) { return static_cast<bf16_t *>(p); };
        const ExactArgs exact = {in(q), in(k), in(v), in(g_fwd), in(g_bwd), in(d_out), out(dq), out(dk), out(dv), out(dg_fwd), out(dg_bwd),
                                 exact_workspace, L, heads_token_major, unsigned(BH), unsigned(n_chunks + extra)};
        hipLaunchKernelGGL(bigla_bwd_chunk_main_kernel<kCt>, dim3((unsigned)(units + BH * extra)), dim3(kThreads), GradLds<kCt>::bytes,
                           stream, q, k, v, g_fwd, g_bwd, d_out, dq, dk, dv, dg_fwd, dg_bwd, ws.states, ws.marks, L, heads_token_major, n_chunks,
                           unsigned(BH), unsigned(extra), exact);
        return hipGetLastError();
    };
    return dk_ == kD ? launch(std::integral_constant<int, 4>{}) : launch(std::integral_constant<int, 2>{});
}

}  // namespace vig
