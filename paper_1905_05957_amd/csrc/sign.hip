// 1-bit compressor kernels (Section 3.2 "1-Bit Quantization", Section 5.1 "1-bit
// compression" of the DoubleSqueeze paper) for the three calls of Algorithm 1.
//
// A message is a sign plane (bit = v < 0) plus one scale per group, scale = mean |v| of
// the group, so that the decoded group has the l1 magnitude of v.
//
// Three routes:
//  * fused (groups are chunks of 512..2048 elements, a multiple of 128): one workgroup holds
//    a whole chunk in registers, so v = g + delta, sum |v|, the sign bits and
//    delta' = v - Q[v] happen in ONE pass over HBM.
//  * held (one group, the whole vector, where the device holds a row on chip; held.h): the workgroups
//    of a row keep v until the row's scale is known, so this is ONE pass over HBM too.
//  * general (whole vectors beyond that, arbitrary segments, other chunk sizes): the scale needs a sum
//    over more than one workgroup, so pass 1 writes v into the delta buffer together with
//    the sign bits and fp64 partial sums, a small kernel reduces them in a fixed order,
//    and pass 2 turns v into delta' = v - Q[v].
//
// Sums of |v| are accumulated in fp64 and rounded once, in an order that depends only on
// the shape, so results are bit-reproducible run to run.
#include "ds_device.h"
#include "ds_internal.h"
#include "held.h"

#include <mutex>
#include <type_traits>
#include <vector>

using namespace ds;

namespace {

// ---------------------------------------------------------------------------------------
// sources of the vector v that is being compressed
// ---------------------------------------------------------------------------------------

// Worker: v = g + delta  (Algorithm 1, worker block, first step; Section 3.1).
template <bool BF16>
struct WorkerSrc {
    const void *g;
    int64_t g_stride;
    const float *delta;
    int64_t delta_stride;

    __device__ __forceinline__ const void *grow(int row) const
    {
        if constexpr (BF16) return static_cast<const uint16_t *>(g) + row * g_stride;
        else return static_cast<const float *>(g) + row * g_stride;
    }
};

// Server with one scale per chunk: v = delta_s + (1/n) sum_i Q[v_i], taken as the chain
// acc = fma(q_i, 1/n, acc) over workers in ascending order (Algorithm 1, parameter-server
// block, first step).
struct ServerArgs {
    const uint64_t *words_in;  // [n, W]
    const float *scales_in;    // [n, S]
    int32_t n;
    int64_t W, S;
    float inv_n;
};

// What a group sums to find its scale: |v| (scale = mean |v|, the l1 reading of "the same
// magnitude", Section 5.1) or v^2 (scale = root mean square, the l2 reading of Section 3.2's
// norm).  The product of two fp32 values is exact in fp64.
// (A compile-time switch: as a run-time one it cost the 124 M-element step 4 %.)
template <bool RMS>
__device__ __forceinline__ double measure(float x)
{
    if constexpr (RMS) return static_cast<double>(x) * static_cast<double>(x);
    else return static_cast<double>(fabsf(x));
}

// (s0, s1, s2, s3) with the sign flipped where the element's bit of `nib` is set.
__device__ __forceinline__ f32x4 signed4(float s0, float s1, float s2, float s3, uint32_t nib)
{
    return f32x4{__uint_as_float(__float_as_uint(s0) ^ ((nib << 31) & 0x80000000u)),
                 __uint_as_float(__float_as_uint(s1) ^ ((nib << 30) & 0x80000000u)),
                 __uint_as_float(__float_as_uint(s2) ^ ((nib << 29) & 0x80000000u)),
                 __uint_as_float(__float_as_uint(s3) ^ ((nib << 28) & 0x80000000u))};
}

// The same chain step with the lane's four sign bits in bits 28..31 of `top` (element 0 in bit
// 28): the sign bit of the scale is flipped where the element's bit is set, which is what
// "bit ? -scale : scale" does for every float.  Shift, mask, exclusive-or instead of test,
// compare and select: no condition-code hazards in a loop that runs n times per element.
__device__ __forceinline__ f32x4 chain4_top(f32x4 a, uint32_t top, float s, float inv_n)
{
    const uint32_t sb = __float_as_uint(s);
    a.x = __fmaf_rn(__uint_as_float(sb ^ ((top << 3) & 0x80000000u)), inv_n, a.x);
    a.y = __fmaf_rn(__uint_as_float(sb ^ ((top << 2) & 0x80000000u)), inv_n, a.y);
    a.z = __fmaf_rn(__uint_as_float(sb ^ ((top << 1) & 0x80000000u)), inv_n, a.z);
    a.w = __fmaf_rn(__uint_as_float(sb ^ (top & 0x80000000u)), inv_n, a.w);
    return a;
}

template <bool RMS>
__device__ __forceinline__ double abs_sum4(f32x4 v)
{
    return ((measure<RMS>(v.x) + measure<RMS>(v.y)) + measure<RMS>(v.z)) + measure<RMS>(v.w);
}

__device__ __forceinline__ float group_scale(double total, double len, bool rms)
{
    return rms ? static_cast<float>(sqrt(total / len)) : static_cast<float>(total / len);
}

// delta' = v - Q[v] with Q[v]_j = (v_j < 0) ? -scale : +scale
__device__ __forceinline__ f32x4 sign_error4(f32x4 v, float s)
{
    f32x4 o;
    o.x = v.x - ((v.x < 0.f) ? -s : s);
    o.y = v.y - ((v.y < 0.f) ? -s : s);
    o.z = v.z - ((v.z < 0.f) ? -s : s);
    o.w = v.w - ((v.w < 0.f) ? -s : s);
    return o;
}

// ---------------------------------------------------------------------------------------
// fused route: one workgroup per chunk
// ---------------------------------------------------------------------------------------
// Common tail: scale from the held values, sign plane, error, stores.  keep: the error is stored with ordinary
// accesses.
template <bool RMS>
__device__ __forceinline__ float fused_finish(f32x4 v, int64_t base, int64_t lim,
                                             float *__restrict__ err_row,
                                             uint64_t *__restrict__ words_row, int64_t bit_lim,
                                             float *__restrict__ scale_out, double *lds, uint32_t *sw_lds, bool keep = false)
{
    // sign words: gathered in LDS, one store per workgroup after the barrier of the reduction
    stash_sign_words(sw_lds, wave_sign_word(v.x < 0.f, v.y < 0.f, v.z < 0.f, v.w < 0.f));
    const double total = block_sum(abs_sum4<RMS>(v), lds, false);
    const float scale = group_scale(total, static_cast<double>(lim - base), RMS);
    if (threadIdx.x == 0) *scale_out = scale;
    flush_sign_words(sw_lds, words_row, base, bit_lim);
    const int64_t e = base + threadIdx.x * 4;
    if (err_row && e < lim) {                                   // no buffer: no compensation
        if (keep) st4(err_row, e, lim, sign_error4(v, scale));  // uniform
        else st4_stream(err_row, e, lim, sign_error4(v, scale));
    }
    return scale;
}

// NOFB: Algorithm 1 without compensation, v = g; no error buffer is touched.
// CPW chunks per workgroup, all loads issued before the first is used: two with compensation; without
// it a chunk is only 4 to 8 KiB of traffic and a workgroup per chunk is bound by the rate at which
// workgroups can be dispatched (486 k workgroups took 0.88 ms for 2.1 GB on the 124 M-element
// workload), so that variant takes four.
// keep_odd: every other row's error is stored with ordinary accesses.
template <bool BF16, bool RMS, bool NOFB, int CPW>
__global__ __launch_bounds__(kBlock) void k_sign_chunk_worker(WorkerSrc<BF16> src, float *delta,
                                                              int64_t d, int64_t chunk,
                                                              uint64_t *words, int64_t W,
                                                              float *scales, int64_t S, bool keep_odd)
{
    __shared__ double lds[CPW][kWaves];
    __shared__ __attribute__((aligned(16))) uint32_t sw_lds[CPW][kWaves * 8];
    const int row = blockIdx.y;
    const void *grow = src.grow(row);
    float *drow = NOFB ? nullptr : delta + row * src.delta_stride;
    f32x4 v[CPW];
    int64_t base[CPW], lim[CPW];
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
        const int64_t ci = static_cast<int64_t>(blockIdx.x) * CPW + c;
        base[c] = ci * chunk;
        lim[c] = (base[c] + chunk < d) ? base[c] + chunk : d;     // base >= d: empty chunk, lim < base
        const int64_t e = base[c] + threadIdx.x * 4;
        v[c] = ld4_grad<BF16>(grow, e, lim[c]);
        if constexpr (!NOFB) v[c] = v[c] + ld4_stream(drow, e, lim[c]);
    }
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
        const int64_t ci = static_cast<int64_t>(blockIdx.x) * CPW + c;
        if (base[c] < d)    // uniform over the workgroup
            fused_finish<RMS>(v[c], base[c], lim[c], drow, words + row * W, (lim[c] == d) ? W * 64 : lim[c],
                              scales + row * S + ci, lds[c], sw_lds[c], keep_odd && (row & 1));
    }
}

// UPD: 0 = the parameter-server block alone; 1, 2 = followed by the model update of Algorithm 1
// for the same elements (2: through the momentum buffer), from the registers that hold the
// server's sign bits and scale: x and m stream through once and the server's message is not
// read back.
template <int CPW, bool RMS, int UPD>   // CPW chunks per workgroup: independent chunks, more bytes in flight per thread
__global__ __launch_bounds__(kBlock) void k_sign_chunk_server(ServerArgs a, float *delta_s, int64_t d,
                                                              int64_t chunk, uint64_t *words_out,
                                                              float *scales_out, float *x, float *m, float gamma,
                                                              float beta)
{
    __shared__ double lds[CPW][kWaves];
    __shared__ __attribute__((aligned(16))) uint32_t sw_lds[CPW][kWaves * 8];
    const int lane = lane_id();
    f32x4 v[CPW];
    int64_t base[CPW], lim[CPW];
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
        const int64_t ci = static_cast<int64_t>(blockIdx.x) * CPW + c;
        base[c] = ci * chunk;
        lim[c] = (base[c] + chunk < d) ? base[c] + chunk : d;     // base >= d: empty chunk, lim < base
        v[c] = delta_s ? ld4_stream(delta_s, base[c] + threadIdx.x * 4, lim[c]) : f32x4{0.f, 0.f, 0.f, 0.f};   // no buffer: no server error
    }
    // the update's operands are fetched up front, beside the error: more bytes in flight
    f32x4 xv[CPW], mv[CPW];
    if constexpr (UPD != 0) {
#pragma unroll
        for (int c = 0; c < CPW; ++c) {
            xv[c] = ld4_stream(x, base[c] + threadIdx.x * 4, lim[c]);
            if constexpr (UPD == 2) mv[c] = ld4_stream(m, base[c] + threadIdx.x * 4, lim[c]);
        }
    }
    // The wavefront's 256 elements are 32 bytes of each worker's sign plane.  Eight workers at
    // a time: lane L loads 32-bit word (L & 7) of worker (L >> 3), one load instruction for
    // all of them; the nibble a lane needs for worker i then sits in lane 8 i + (L >> 3).
    for (int i0 = 0; i0 < a.n; i0 += 8) {
        const int nb = (a.n - i0 < 8) ? a.n - i0 : 8;
        const int wi = lane >> 3;
        uint32_t word[CPW];
        float sc[CPW];
#pragma unroll
        for (int c = 0; c < CPW; ++c) {
            const int64_t ci = static_cast<int64_t>(blockIdx.x) * CPW + c;
            const int64_t wave_first = base[c] + wave_id() * 256;
            word[c] = 0u;
            if (wi < nb && wave_first + 32 * (lane & 7) < a.W * 64)
                word[c] = reinterpret_cast<const uint32_t *>(a.words_in + (i0 + wi) * a.W)[(wave_first >> 5) + (lane & 7)];
            sc[c] = (lane < nb && base[c] < d) ? a.scales_in[(i0 + lane) * a.S + ci] : 0.f;
        }
        // Lanes past the end of their chunk run the chain too (their values are cleared below):
        // no branch inside the loop.  A full batch of eight workers is unrolled, so that the
        // eight cross-lane fetches are in flight together instead of one wait per worker.
        const int top_shift = 28 - 4 * (lane & 7);
        if (nb == 8) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
#pragma unroll
                for (int c = 0; c < CPW; ++c) {
                    const uint32_t w = __shfl(word[c], i * 8 + (lane >> 3), 64);
                    const float s = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sc[c]), i));
                    v[c] = chain4_top(v[c], w << top_shift, s, a.inv_n);
                }
            }
        } else {
            for (int i = 0; i < nb; ++i) {
#pragma unroll
                for (int c = 0; c < CPW; ++c) {
                    const uint32_t w = __shfl(word[c], i * 8 + (lane >> 3), 64);
                    const float s = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sc[c]), i));
                    v[c] = chain4_top(v[c], w << top_shift, s, a.inv_n);
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
        const int64_t ci = static_cast<int64_t>(blockIdx.x) * CPW + c;
        // components past lim must stay zero: they count in the sum of |v|
        v[c] = zero_past(v[c], base[c] + threadIdx.x * 4, lim[c]);
        if (base[c] < d) {   // uniform over the workgroup
            const float s = fused_finish<RMS>(v[c], base[c], lim[c], delta_s, words_out,
                                              (lim[c] == d) ? a.W * 64 : lim[c], scales_out + ci, lds[c], sw_lds[c]);
            if constexpr (UPD != 0) {
                // q = decode of the message just written: bit ? -scale : +scale, bit = (v < 0)
                const int64_t e = base[c] + threadIdx.x * 4;
                if (e < lim[c]) {
                    f32x4 q = {(v[c].x < 0.f) ? -s : s, (v[c].y < 0.f) ? -s : s, (v[c].z < 0.f) ? -s : s, (v[c].w < 0.f) ? -s : s};
                    if constexpr (UPD == 2) {
                        q = fma4(beta, mv[c], q);
                        st4_stream(m, e, lim[c], q);
                    }
                    st4_stream(x, e, lim[c], fma4(-gamma, q, xv[c]));
                }
            }
        }
    }
}

// One thread per 4 elements.
template <bool MOM, bool DECODE_ONLY>
__global__ __launch_bounds__(kBlock) void k_sign_chunk_update(const uint64_t *__restrict__ words,
                                                              const float *__restrict__ scales,
                                                              int64_t chunk, float *x, float *m,
                                                              int64_t d, float gamma, float beta)
{
    const int64_t e = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) * 4;
    if (e >= d) return;
    // chunk is a multiple of 4 on this route, so the four elements share a chunk;
    // e < 2^31, so the chunk index is a 32-bit division
    const float s = scales[static_cast<uint32_t>(e) / static_cast<uint32_t>(chunk)];
    const uint32_t nib = load_sign_nibble(words, e);
    apply_q4<MOM, DECODE_ONLY>(signed4(s, s, s, s, nib), e, d, x, m, gamma, beta);
}

// ---------------------------------------------------------------------------------------
// general route: tiles x pieces
// ---------------------------------------------------------------------------------------
// Pieces [p0, p1) of a tile; seg0 = its group when it has one piece, else -1.
struct TilePieces {
    int32_t p0, p1, seg0;
};

__device__ __forceinline__ TilePieces tile_pieces(const ds_sign_tables &tb, int64_t tile)
{
    if (tb.whole_d > 0) return TilePieces{static_cast<int32_t>(tile), static_cast<int32_t>(tile) + 1, 0};
    const int2 ti = tb.tile_info[tile];
    return (ti.y >= 0) ? TilePieces{ti.x, ti.x + 1, ti.y} : TilePieces{ti.x, ti.x - ti.y, -1};
}

// Group of element e, given the pieces [p0, p1) of its tile.
__device__ __forceinline__ int32_t seg_of(const ds_sign_tables &tb, int32_t p0, int32_t p1, int64_t e)
{
    int32_t p = p0;
    while (p + 1 < p1 && tb.piece_start[p + 1] <= e) ++p;
    return tb.piece_seg[p];
}

template <bool RMS>
__device__ __forceinline__ double masked_abs(float x, int64_t e, int64_t lo, int64_t hi)
{
    return (e >= lo && e < hi) ? measure<RMS>(x) : 0.0;
}

// v - Q[v] for the four elements of a thread, with the group scales of its tile's pieces.
__device__ __forceinline__ f32x4 sign_error_tile(f32x4 v, int64_t e, int64_t d, const float *__restrict__ srow,
                                                 const ds_sign_tables &tb, int32_t p0, int32_t p1, int32_t seg0)
{
    if (seg0 >= 0) return sign_error4(v, srow[seg0]);
    float s[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) s[c] = (e + c < d) ? srow[seg_of(tb, p0, p1, e + c)] : 0.f;
    v.x = v.x - ((v.x < 0.f) ? -s[0] : s[0]);
    v.y = v.y - ((v.y < 0.f) ? -s[1] : s[1]);
    v.z = v.z - ((v.z < 0.f) ? -s[2] : s[2]);
    v.w = v.w - ((v.w < 0.f) ? -s[3] : s[3]);
    return v;
}

// Pass-1 tail: store v, sign bits, per-piece partial sums of |v| (or v^2).  STREAM: v is not
// read again in this call (deferred error form), so it leaves non-temporally.
template <bool RMS, bool STREAM, bool KEEP = true>   // KEEP = false: v is not stored (no compensation: it is not needed again)
__device__ __forceinline__ void pass1_finish(f32x4 v, int64_t base, int64_t d,
                                             float *__restrict__ vrow,
                                             uint64_t *__restrict__ words_row, int64_t bit_lim,
                                             const ds_sign_tables &tb, int32_t p0, int32_t p1,
                                             double *__restrict__ partial_row, double *lds, uint32_t *sw_lds)
{
    const int64_t e = base + threadIdx.x * 4;
    if (KEEP && vrow && e < d) {             // no buffer: no compensation either
        if constexpr (STREAM) st4_stream(vrow, e, d, v);
        else st4(vrow, e, d, v);
    }
    stash_sign_words(sw_lds, wave_sign_word(v.x < 0.f, v.y < 0.f, v.z < 0.f, v.w < 0.f));
    if (p1 - p0 == 1) {
        const double total = block_sum(abs_sum4<RMS>(v), lds, false);   // elements past d are zero
        if (threadIdx.x == 0) partial_row[p0] = total;
        flush_sign_words(sw_lds, words_row, base, bit_lim);
    } else {
        __syncthreads();
        flush_sign_words(sw_lds, words_row, base, bit_lim);
        for (int32_t p = p0; p < p1; ++p) {
            const int64_t lo = tb.piece_start[p], hi = tb.piece_start[p + 1];
            const double part = ((masked_abs<RMS>(v.x, e, lo, hi) + masked_abs<RMS>(v.y, e + 1, lo, hi)) +
                                 masked_abs<RMS>(v.z, e + 2, lo, hi)) + masked_abs<RMS>(v.w, e + 3, lo, hi);
            const double total = block_sum(part, lds, true);
            if (threadIdx.x == 0) partial_row[p] = total;
        }
    }
}

// DEFERRED: the error buffer holds the previous call's v and `prev_scales` that call's group
// scales; the error delta = v_prev - Q[v_prev] is formed on the fly (the same subtraction
// pass 2 would have stored), so the buffer is looked at once per call.
// MODE 0: plain.  1 (deferred): as described above.  2: Algorithm 1 without compensation, v = g,
// no error buffer is touched.
template <bool BF16, int MODE, bool RMS>
__global__ __launch_bounds__(kBlock) void k_sign_pass1_worker(WorkerSrc<BF16> src, float *delta,
                                                              int64_t d, uint64_t *words, int64_t W,
                                                              ds_sign_tables tb, double *partials,
                                                              const float *__restrict__ prev_scales, int64_t S)
{
    __shared__ double lds[kWaves];
    __shared__ __attribute__((aligned(16))) uint32_t sw_lds[kWaves * 8];
    const int row = blockIdx.y;
    const int64_t tile = blockIdx.x;
    const int64_t base = tile * kTile;
    const void *grow = src.grow(row);
    constexpr bool DEFERRED = MODE == 1, NOFB = MODE == 2;
    float *drow = NOFB ? nullptr : delta + row * src.delta_stride;
    const int64_t e = base + threadIdx.x * 4;
    const TilePieces tp = tile_pieces(tb, tile);
    const int32_t p0 = tp.p0, p1 = tp.p1;
    f32x4 v = ld4_grad<BF16>(grow, e, d);
    if constexpr (!NOFB) {
        f32x4 dl = DEFERRED ? ld4_stream(drow, e, d) : ld4(drow, e, d);
        if (DEFERRED && e < d) dl = zero_past(sign_error_tile(dl, e, d, prev_scales + row * S, tb, p0, p1, tp.seg0), e, d);
        v = v + dl;
    }
    pass1_finish<RMS, DEFERRED, !NOFB>(v, base, d, drow, words + row * W, W * 64, tb, p0, p1,
                      partials + static_cast<int64_t>(row) * tb.n_pieces, lds, sw_lds);
}

// STREAM: the error buffer is read and written non-temporally (see ds_sign_server).
template <bool DEFERRED, bool RMS, bool STREAM>
__global__ __launch_bounds__(kBlock) void k_sign_pass1_server(ServerArgs a, float *delta_s, int64_t d,
                                                              uint64_t *words_out, ds_sign_tables tb,
                                                              double *partials, const float *__restrict__ prev_scales)
{
    __shared__ double lds[kWaves];
    __shared__ __attribute__((aligned(16))) uint32_t sw_lds[kWaves * 8];
    const int64_t tile = blockIdx.x;
    const int64_t base = tile * kTile;
    const TilePieces tp = tile_pieces(tb, tile);
    const int32_t p0 = tp.p0, p1 = tp.p1;
    const int64_t e = base + threadIdx.x * 4;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};                                      // no buffer: no server error
    if (delta_s) v = STREAM ? ld4_stream(delta_s, e, d) : ld4(delta_s, e, d);
    const int lane = lane_id();
    const int64_t wave_first = base + wave_id() * 256;
    // sign words of the first eight workers (lane L: word L & 7 of worker L >> 3): their
    // addresses do not depend on the tile's pieces, so they leave together with the table
    // entry and the error instead of after the scales that the entry leads to
    const bool word_in = wave_first + 32 * (lane & 7) < a.W * 64;
    uint32_t word0 = 0u;
    if ((lane >> 3) < a.n && word_in)
        word0 = reinterpret_cast<const uint32_t *>(a.words_in + (lane >> 3) * a.W)[(wave_first >> 5) + (lane & 7)];
    // scales of the first eight workers (lane i: worker i), asked for before the previous
    // call's scale below is waited for: both hang on the table entry alone
    float sc0 = 0.f;
    if (tp.seg0 >= 0 && lane < a.n && lane < 8) sc0 = a.scales_in[lane * a.S + tp.seg0];
    if (DEFERRED && e < d) v = sign_error_tile(v, e, d, prev_scales, tb, p0, p1, tp.seg0);   // past d: cleared below
    if (p1 - p0 == 1) {
        // the whole tile lies in one scale group: same batched loads as the chunk route
        const int32_t sg = tp.seg0;
        for (int i0 = 0; i0 < a.n; i0 += 8) {
            const int nb = (a.n - i0 < 8) ? a.n - i0 : 8;
            uint32_t word = word0;
            float sc = sc0;
            if (i0 > 0) {
                word = 0u;
                if ((lane >> 3) < nb && word_in)
                    word = reinterpret_cast<const uint32_t *>(a.words_in + (i0 + (lane >> 3)) * a.W)[(wave_first >> 5) + (lane & 7)];
                sc = (lane < nb) ? a.scales_in[(i0 + lane) * a.S + sg] : 0.f;
            }
            // lanes past d run the chain too (cleared below); a full batch is unrolled so that
            // its eight cross-lane fetches are in flight together
            const int top_shift = 28 - 4 * (lane & 7);
            if (nb == 8) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint32_t w = __shfl(word, i * 8 + (lane >> 3), 64);
                    const float sv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sc), i));
                    v = chain4_top(v, w << top_shift, sv, a.inv_n);
                }
            } else {
                for (int i = 0; i < nb; ++i) {
                    const uint32_t w = __shfl(word, i * 8 + (lane >> 3), 64);
                    const float sv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sc), i));
                    v = chain4_top(v, w << top_shift, sv, a.inv_n);
                }
            }
        }
    } else if (e < d) {
        int32_t seg[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) seg[c] = (e + c < d) ? seg_of(tb, p0, p1, e + c) : 0;
        for (int i = 0; i < a.n; ++i) {
            const float *srow = a.scales_in + i * a.S;
            const uint32_t nib = load_sign_nibble(a.words_in + i * a.W, e);
            const float s0 = srow[seg[0]], s1 = srow[seg[1]], s2 = srow[seg[2]], s3 = srow[seg[3]];
            v = fma4(a.inv_n, signed4(s0, s1, s2, s3, nib), v);
        }
    }
    v = zero_past(v, e, d);
    pass1_finish<RMS, STREAM>(v, base, d, delta_s, words_out, a.W * 64, tb, p0, p1, partials, lds, sw_lds);
}

// scale[row][s] = (float)( sum of the group's partials / |group| ), fixed order.
// `keep` (may be null): the context's own copy of the scales, for the deferred error form.
__global__ __launch_bounds__(kBlock) void k_sign_reduce(const double *__restrict__ partials,
                                                        ds_sign_tables tb, float *scales, int64_t S, float *keep)
{
    __shared__ double lds[kWaves];
    const int32_t s = blockIdx.x;
    const int row = blockIdx.y;
    const double *prow = partials + static_cast<int64_t>(row) * tb.n_pieces;
    const bool whole = tb.whole_d > 0;
    const int32_t p0 = whole ? 0 : tb.seg_piece_first[s], p1 = whole ? tb.n_pieces : tb.seg_piece_first[s + 1];
    double acc = 0.0;
    for (int32_t p = p0 + threadIdx.x; p < p1; p += kBlock) acc += prow[p];
    const double total = block_sum(acc, lds, false);
    if (threadIdx.x == 0) {
        const double len = static_cast<double>(whole ? tb.whole_d : tb.seg_off[s + 1] - tb.seg_off[s]);
        const float sc = group_scale(total, len, tb.rms);
        scales[row * S + s] = sc;
        if (keep) keep[row * S + s] = sc;
    }
}

// Pass 2: the buffer holds v; overwrite with delta' = v - Q[v].  STREAM: non-temporal stores.
template <bool STREAM>
__global__ __launch_bounds__(kBlock) void k_sign_pass2(float *buf, int64_t stride, int64_t d,
                                                       const float *__restrict__ scales, int64_t S,
                                                       ds_sign_tables tb)
{
    // Pass 2 walks the rows and tiles in the opposite order to pass 1: what pass 1 wrote last
    // is still in the 256 MB memory-side cache, so those reads (and the v lines they
    // overwrite) never reach HBM.
    const int row = gridDim.y - 1 - blockIdx.y;
    const int64_t tile = gridDim.x - 1 - blockIdx.x;
    float *brow = buf + row * stride;
    const float *srow = scales + row * S;
    const TilePieces tp = tile_pieces(tb, tile);
    const int64_t e = tile * kTile + threadIdx.x * 4;
    if (e >= d) return;
    const f32x4 v = ld4_stream(brow, e, d);
    const f32x4 o = sign_error_tile(v, e, d, srow, tb, tp.p0, tp.p1, tp.seg0);
    if constexpr (STREAM) st4_stream(brow, e, d, o);
    else st4(brow, e, d, o);
}

// ---------------------------------------------------------------------------------------
// held route: one look at a row whose scale spans workgroups
// ---------------------------------------------------------------------------------------
// A workgroup keeps v of T consecutive tiles in registers and LDS, hands their sums over, waits for
// the row's scale and stores delta' = v - Q[v]: the row is read once and written once, where pass 1
// / reduce / pass 2 move v through memory twice more.  The workgroup whose arrival completes the
// row adds the sums up and publishes the scale.  The sums are of tiles and are added in the order of k_sign_reduce: a
// scale does not depend on the route, nor on how many tiles a workgroup holds.
//
// The host takes this route when the device holds all workgroups of a row at once, and they are
// dispatched in row order, so a wait normally lasts as long as the rest of the row takes to load.
// Nothing depends on that: a wait is bounded by the clock, and a workgroup that gives up leaves
// v in the buffer and sets its flag for k_sign_held_finish, which forms the error from there.
//
// What bounds it is the traffic (12 bytes per element) and, where the rows do not all fit the
// device at once, that a row's loads have to overlap the barrier and the stores of the row before:
// the worker call at 8 x 11,173,962 took 243 us with 1.5 rows resident (T = 8), 222 us with 2.0
// (T = 14), 213 us with 2.25 (T = 24), at 171 us for its bytes at the copy kernel's rate and 286 us
// in two looks.  7 x 2,345,679, all rows resident: 35 us against 62 us in two looks (31 us for its
// bytes; both with the finish launch, 4.8 us).  With all errors of a workgroup loaded up front and the gradients in groups of three the
// first took 220 us, with D = 4 and 6 tiles in flight instead of 3 213 and 214 us.
// The tiles' sums cost issue.  Worker call at 8 x 11,173,962 in bf16, at 8 x 24,000,000 in f32 and in bf16, and server and update of
// 24,000,000: a wave_sum for every tile 200, 461, 412 and 72.9 us; four tiles together (HeldSums), and the last workgroup adding
// up twelve at a time instead of eight in the largest size, 196, 459, 405 and 69.8 us; eight together nothing more.  One
// sum per thread over all its tiles, whose order would depend on their number, 191, 444, 389 and 66.7 us.
//
// What a workgroup of the held route shares: per tile the wavefronts' sums and the sign words.
template <int T>
struct HeldShared {
    double sums[T][kWaves], red[kWaves];
    __attribute__((aligned(16))) uint32_t words[T][kWaves * 8];
    uint32_t sh[2];
};

// Two tiles' values of a step of wave_sum in one: lanes with `second` go on with y, the others with x, each with the two
// numbers that wave_sum adds.  CTRL leads to a lane with the other choice.
template <int CTRL>
__device__ __forceinline__ double two_sums(double x, double y, bool second)
{
    return (second ? y : x) + dpp_f64<CTRL>(second ? x : y);
}

// wave_sum of up to four tiles together.  After two steps lane i has that of tile (bit 0 ^ bit 2) + 2 (bit 1 ^ bit 2) of i, which the
// lanes that the mirrors pair have in common, and lanes 0 .. 3 have the four in order.
struct HeldSums {
    double one, pair;
};

template <bool RMS, int Q, int L, int T>
__device__ __forceinline__ void held_look(f32x4 v, int t, HeldShared<T> &m, HeldSums &h)
{
    stash_sign_words(m.words[t], wave_sign_word(v.x < 0.f, v.y < 0.f, v.z < 0.f, v.w < 0.f));
    const int lane = lane_id();
    const bool odd = ((lane ^ (lane >> 2)) & 1) != 0, upper = ((lane ^ (lane >> 1)) & 2) != 0;
    double s = abs_sum4<RMS>(v);
    constexpr int at = Q & 3, count = (Q == T - 1 && at != 3) ? at + 1 : 4;       // of the group that is complete with this tile
    static_assert(count != 3, "no size leaves three");
    if constexpr (at == 0 && count != 1) {
        h.one = s;
        asm volatile("" : "+v"(h.one));       // now: put off, the sums of all tiles would keep their values in registers
    } else if constexpr (at == 1 && count != 2) {
        h.pair = two_sums<kDppXor1>(h.one, s, odd);
        asm volatile("" : "+v"(h.pair));
    } else if constexpr (at == 2) {
        h.one = s;
        asm volatile("" : "+v"(h.one));
    } else {
        if constexpr (count == 1) {
            s += dpp_f64<kDppXor1>(s);
            s += dpp_f64<kDppXor2>(s);
        } else if constexpr (count == 2) {
            s = two_sums<kDppXor1>(h.one, s, odd);
            s += dpp_f64<kDppXor2>(s);
        } else {
            s = two_sums<kDppXor2>(h.pair, two_sums<kDppXor1>(h.one, s, odd), upper);
        }
        s += dpp_f64<kDppHalfMirror>(s);
        s += dpp_f64<kDppRowMirror>(s);
        s = pair_row_sum<16>(s);
        s = pair_row_sum<32>(s);
        if (lane < count) {
            const int q = Q - at + lane;
            m.sums[q < L ? T - L + q : q - L][wave_id()] = s;
        }
    }
}

// After every tile was looked at: sign words and sums out, the arrival, the row's scale (true) or
// no scale in time (false).
template <bool RMS, int T>
__device__ __forceinline__ bool held_scale(HeldShared<T> &m, int64_t tile0, int row, uint64_t *__restrict__ words_row,
                                           const ds_sign_tables &tb, double *partial_row, float *scale_out, HeldRow *rows,
                                           uint32_t patience, float *s)
{
    __syncthreads();
    const int64_t bit_lim = ((tb.whole_d + 63) / 64) * 64;
    const double len = static_cast<double>(tb.whole_d);
    // lane t < T of every wavefront: sum of tile t (zero past the end of the row)
    double tile_sum = 0.0;
    if (lane_id() < T) {
        tile_sum = m.sums[lane_id()][0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) tile_sum += m.sums[lane_id()][w];
    }
    if (gridDim.x != 1 && wave_id() == 0) {
        if (lane_id() < T && tile0 + lane_id() < tb.n_pieces)
            as_shared(reinterpret_cast<uint64_t *>(partial_row))[tile0 + lane_id()].store(__double_as_longlong(tile_sum));
        // the sums are in memory before the arrival is announced
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane_id() == 0) m.sh[0] = (rows[row].arrived.fetch_add(1u) + 1u == gridDim.x) ? 1u : 0u;
    }
    // the tiles' sign words, 16 threads and 256 bytes each
    const int t16 = threadIdx.x >> 4;
    if (t16 < T) flush_sign_words_at(m.words[t16], words_row, (tile0 + t16) * kTile, bit_lim, threadIdx.x & 15);
    if (gridDim.x == 1) {                                    // the row is this workgroup's
        *s = group_scale(wave_sum(tile_sum), len, RMS);
        if (threadIdx.x == 0) *scale_out = *s;
        return true;
    }
    __syncthreads();
    const bool last = m.sh[0] != 0u;
    __syncthreads();
    if (!last) return held_wait(rows, row, patience, m.sh, s);
    constexpr int B = T > 16 ? 12 : 8;                       // in flight; what the registers beside the held tiles allow
    double acc = 0.0;
    for (int32_t p0 = threadIdx.x; p0 < tb.n_pieces; p0 += B * kBlock) {
        uint64_t b[B];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const int32_t p = p0 + j * kBlock;
            b[j] = (p < tb.n_pieces) ? as_shared(reinterpret_cast<uint64_t *>(partial_row))[p].load() : 0ull;
        }
#pragma unroll
        for (int j = 0; j < B; ++j) acc += __longlong_as_double(static_cast<long long>(b[j]));   // + 0.0 past the end
    }
    const double total = block_sum(acc, m.red, false);
    *s = group_scale(total, len, RMS);
    if (threadIdx.x == 0) {
        rows[row].pub.store(kHeldValue | __float_as_uint(*s));
        *scale_out = *s;
    }
    return true;
}

// One lane's group of four that the end of the row cuts, and where it lies in the stretch (-1: nowhere).
struct HeldCut {
    f32x4 v;
    int at;
};

template <bool BF16>
__device__ __forceinline__ HeldCut held_cut(const void *grow, const float *drow, int64_t first, int left)
{
    HeldCut c{{0.f, 0.f, 0.f, 0.f}, -1};
    if (left & 3) {                               // uniform
        c.at = left & ~3;
        c.v = ld4_grad<BF16>(grow, first + c.at, first + left) + ld4_stream(drow, first + c.at, first + left);
    }
    return c;
}

// v of tile t, zero past the end of the row.  The selects run in every workgroup: under a branch
// the compiler copies all of the held values around it.
__device__ __forceinline__ f32x4 held_sum4(f32x4 g, f32x4 dl, const HeldCut &c, int t)
{
    f32x4 v = g + dl;
    const bool mine = static_cast<int>(threadIdx.x) * 4 + t * kTile == c.at;
    v.x = mine ? c.v.x : v.x;
    v.y = mine ? c.v.y : v.y;
    v.z = mine ? c.v.z : v.z;
    return v;
}

// delta' of tile t, or v itself when the scale is not there.
__device__ __forceinline__ void held_store(f32x4 v, int t, float *out, int left, bool ok, float s)
{
    const f32x4 o = ok ? sign_error4(v, s) : v;
    held_st4(out, left, t, o);
    const int e = static_cast<int>(threadIdx.x) * 4 + t * kTile;
    if ((left & 3) && e == (left & ~3)) st4_tail(out, e, left, o);
}

struct HeldUpdate {
    float *x, *m;
    float gamma, beta;
};

// x (and m) of elements e..e+3 of the row from the held v: q = the decoded message.
template <int UPD>
__device__ __forceinline__ void held_update4(f32x4 v, f32x4 &x, f32x4 &m, float s, const HeldUpdate &u)
{
    f32x4 q = {(v.x < 0.f) ? -s : s, (v.y < 0.f) ? -s : s, (v.z < 0.f) ? -s : s, (v.w < 0.f) ? -s : s};
    if constexpr (UPD == 2) q = m = fma4(u.beta, m, q);
    x = fma4(-u.gamma, q, x);
}

// What a workgroup that gave up left: its error, and where u.x is set the update, from the stored v.
__device__ __forceinline__ void held_finish_part(float *brow, int64_t d, int part, int T, float s, const HeldUpdate &u)
{
    const int64_t e0 = static_cast<int64_t>(part) * T * kTile + threadIdx.x * 4;
    constexpr int D = 4;                                      // loads in flight
    for (int t0 = 0; t0 < T; t0 += D) {
        f32x4 v[D];
#pragma unroll
        for (int j = 0; j < D; ++j)
            v[j] = (t0 + j < T) ? ld4_stream(brow, e0 + (t0 + j) * kTile, d) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const int64_t e = e0 + (t0 + j) * kTile;
            if (t0 + j >= T || e >= d) continue;
            st4_stream(brow, e, d, sign_error4(v[j], s));
            if (u.x) {
                f32x4 x4 = ld4_stream(u.x, e, d), m4 = x4;
                if (u.m) {
                    m4 = ld4_stream(u.m, e, d);
                    held_update4<2>(v[j], x4, m4, s, u);
                    st4_stream(u.m, e, d, m4);
                } else {
                    held_update4<1>(v[j], x4, m4, s, u);
                }
                st4_stream(u.x, e, d, x4);
            }
        }
    }
}

// The end of a workgroup in a row that finishes itself.
__device__ __forceinline__ void held_self_finish(float *brow, int64_t d, int T, bool ok, uint32_t *gave_up_row, HeldRow *rows, int row,
                                                 uint32_t *sh, const HeldUpdate &u)
{
    uint32_t unused;
    if (!held_depart(rows + row, gridDim.x, ok, 0u, sh, &unused)) return;
    if (rows[row].late.load() != 0u) {                        // uniform: all have departed
        __threadfence();
        const float s = __uint_as_float(static_cast<uint32_t>(rows[row].pub.load()));
        for (uint32_t p = 0; p < gridDim.x; ++p)
            if (as_shared(gave_up_row)[p].load() != 0u) held_finish_part(brow, d, static_cast<int>(p), T, s, u);
        __syncthreads();
    }
    if (threadIdx.x == 0) rows[row].next_call(row == 0);
}

// R tiles of a workgroup are held in registers and L more in LDS (every thread reads back its own
// elements).
constexpr int kHeldDepth = 3;

template <bool BF16, bool RMS, int R, int L>
__global__ __launch_bounds__(kBlock, held_waves(R)) void k_sign_held_worker(WorkerSrc<BF16> src, float *delta, int64_t d,
                                                                            uint64_t *words, int64_t W, ds_sign_tables tb,
                                                                            double *partials, float *scales, HeldRow *rows,
                                                                            uint32_t *gave_up, uint32_t patience, bool self)
{
    constexpr int T = R + L;
    __shared__ HeldShared<T> m;
    __shared__ f32x4 far[L ? L : 1][kBlock];
    const int row = blockIdx.y;
    const int64_t tile0 = static_cast<int64_t>(blockIdx.x) * T, first = tile0 * kTile;
    const void *grow = src.grow(row);
    float *drow = delta + row * src.delta_stride;
    int left = held_left<T>(tile0, d);
    const HeldCut cut = held_cut<BF16>(grow, drow, first, left);
    // The tiles one after the other, those for LDS first, with the loads of D tiles in flight.
    constexpr int D = kHeldDepth < T ? kHeldDepth : T;
    f32x4 v[R], g[D], dl[L ? D : 1];
    HeldSums sums;
    auto fetch = [&](auto qc) {
        constexpr int q = decltype(qc)::value, t = q < L ? R + q : q - L;
        if constexpr (q < L) dl[q % D] = held_ld4(drow + first, left, t);
        else v[t] = held_ld4(drow + first, left, t);
        g[q % D] = held_g4<BF16>(grow, first, left, t);
    };
    static_for<0, D>(fetch);
    static_for<0, T>([&](auto qc) {
        constexpr int q = decltype(qc)::value, t = q < L ? R + q : q - L;
        __builtin_amdgcn_sched_barrier(0);
        f32x4 w;
        if constexpr (q < L) w = held_sum4(g[q % D], dl[q % D], cut, t);
        else w = held_sum4(g[q % D], v[t], cut, t);
        asm volatile("" : "+v"(w));       // nothing is carried from here to the store of the errors but w
        if constexpr (q + D < T) fetch(std::integral_constant<int, q + D>{});
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (q < L) far[q][threadIdx.x] = w;
        else v[t] = w;
        held_look<RMS, q, L, T>(w, t, m, sums);
    });
    held_fence(v, left);
    float s;
    const bool ok = held_scale<RMS, T>(m, tile0, row, words + row * W, tb, partials + static_cast<int64_t>(row) * tb.n_pieces,
                                       scales + row, rows, patience, &s);
    uint32_t *gave_up_row = gave_up + row * static_cast<int64_t>(gridDim.x);
    if (threadIdx.x == 0 && gridDim.x != 1) as_shared(gave_up_row)[blockIdx.x].store(ok ? 0u : 1u);
#pragma unroll
    for (int t = 0; t < R; ++t) {
        held_store(v[t], t, drow + first, left, ok, s);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int t = R; t < T; ++t) held_store(far[t - R][threadIdx.x], t, drow + first, left, ok, s);
    if constexpr (kHeldSelf<R, L>)
        if (self) held_self_finish(drow, d, T, ok, gave_up_row, rows, row, m.sh, HeldUpdate{nullptr, nullptr, 0.f, 0.f});
}

// The parameter-server block the same way, and with UPD the model update of Algorithm 1 (2: through
// the momentum buffer) from the values that the workgroup holds: the average is formed once, the
// error is read and written once, the server's message is not read back.  Compressor, reduce,
// second look and update as launches of their own took 59 us at 8 x 11,173,962, one launch and its
// finish take 45 us (30 us for their bytes at the copy kernel's rate; the barrier is not hidden, there
// is one row).  Ordinary accesses beat non-temporal ones at every size that is held, above 64 MB too: whole
// steps at 8 x 11,173,962 260 against 265 us, with momentum 271 and 282 us; 2 x 24,000,000 189 and 204 us, with
// momentum 225 and 240 us; 1 x 5,000,003 with momentum 50 and 52 us.  With 14 and 24 tiles per workgroup instead of
// the smallest size that holds the row, server and update take 58 and 60 us.
// One tile's average: v = delta_s + (1/n) sum_i Q[v_i] by the chain over workers.  word0, sc0: sign
// words and scales of the first eight workers (layout as in k_sign_pass1_server).
__device__ __forceinline__ f32x4 held_chain(f32x4 v, uint32_t word0, float sc0, const ServerArgs &a, int64_t wave_first)
{
    const int lane = lane_id();
    const int top_shift = 28 - 4 * (lane & 7);
    for (int i0 = 0; i0 < a.n; i0 += 8) {
        const int nb = (a.n - i0 < 8) ? a.n - i0 : 8;
        uint32_t word = word0;
        float sc = sc0;
        if (i0 > 0) {
            word = 0u;
            if ((lane >> 3) < nb && wave_first + 32 * (lane & 7) < a.W * 64)
                word = reinterpret_cast<const uint32_t *>(a.words_in + (i0 + (lane >> 3)) * a.W)[(wave_first >> 5) + (lane & 7)];
            sc = (lane < nb) ? a.scales_in[i0 + lane] : 0.f;
        }
        if (nb == 8) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t w = __shfl(word, i * 8 + (lane >> 3), 64);
                v = chain4_top(v, w << top_shift, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sc), i)), a.inv_n);
            }
        } else {
            for (int i = 0; i < nb; ++i) {
                const uint32_t w = __shfl(word, i * 8 + (lane >> 3), 64);
                v = chain4_top(v, w << top_shift, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sc), i)), a.inv_n);
            }
        }
    }
    return v;
}

template <bool RMS, int UPD, int R, int L>
__global__ __launch_bounds__(kBlock, held_waves(R)) void k_sign_held_server(ServerArgs a, float *delta_s, int64_t d, uint64_t *words_out,
                                                                            ds_sign_tables tb, double *partials, float *scale_out,
                                                                            HeldUpdate u, HeldRow *rows, uint32_t *gave_up,
                                                                            uint32_t patience, bool self)
{
    constexpr int T = R + L;
    __shared__ HeldShared<T> m;
    __shared__ f32x4 far[L ? L : 1][kBlock];
    const int lane = lane_id();
    const int64_t tile0 = static_cast<int64_t>(blockIdx.x) * T, first = tile0 * kTile;
    int left = held_left<T>(tile0, d);
    f32x4 cut = {0.f, 0.f, 0.f, 0.f};
    int cut_at = -1;
    if (left & 3) {
        cut_at = left & ~3;
        cut = ld4_tail(delta_s, first + cut_at, first + left);
    }
    const float sc0 = (lane < a.n && lane < 8) ? a.scales_in[lane] : 0.f;
    constexpr int D = 4 < T ? 4 : T;
    f32x4 v[R], ring[L ? D : 1];
    uint32_t word[D];
    HeldSums sums;
    auto fetch = [&](auto qc) {
        constexpr int q = decltype(qc)::value, t = q < L ? R + q : q - L;
        if constexpr (q < L) ring[q % D] = held_ld4<0>(delta_s + first, left, t);
        else v[t] = held_ld4<0>(delta_s + first, left, t);
        const int64_t wave_first = first + t * kTile + wave_id() * 256;
        word[q % D] = 0u;
        if ((lane >> 3) < a.n && wave_first + 32 * (lane & 7) < a.W * 64)
            word[q % D] = reinterpret_cast<const uint32_t *>(a.words_in + (lane >> 3) * a.W)[(wave_first >> 5) + (lane & 7)];
    };
    static_for<0, D>(fetch);
    static_for<0, T>([&](auto qc) {
        constexpr int q = decltype(qc)::value, t = q < L ? R + q : q - L;
        __builtin_amdgcn_sched_barrier(0);
        f32x4 w;
        if constexpr (q < L) w = ring[q % D];
        else w = v[t];
        const int e = static_cast<int>(threadIdx.x) * 4 + t * kTile;
        const bool mine = e == cut_at;
        w.x = mine ? cut.x : w.x;
        w.y = mine ? cut.y : w.y;
        w.z = mine ? cut.z : w.z;
        w = held_chain(w, word[q % D], sc0, a, first + t * kTile + wave_id() * 256);
        w = zero_past(w, e, left);
        asm volatile("" : "+v"(w));
        cut.x = mine ? w.x : cut.x;
        cut.y = mine ? w.y : cut.y;
        cut.z = mine ? w.z : cut.z;
        if constexpr (q + D < T) fetch(std::integral_constant<int, q + D>{});
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (q < L) far[q][threadIdx.x] = w;
        else v[t] = w;
        held_look<RMS, q, L, T>(w, t, m, sums);
    });
    held_fence(v, left);
    const bool mine_cut = cut_at >= 0 && (cut_at & (kTile - 1)) == static_cast<int>(threadIdx.x) * 4;   // `cut` holds its v
    // the update's operands of the first tiles are asked for before the wait
    constexpr int P = UPD == 0 ? 0 : R <= 2 ? R : R <= 4 ? (UPD == 2 ? 1 : 2) : 0;
    f32x4 xv[P ? P : 1], mv[P ? P : 1];
#pragma unroll
    for (int t = 0; t < P; ++t) {
        xv[t] = held_ld4<0>(u.x + first, left, t);
        if constexpr (UPD == 2) mv[t] = held_ld4<0>(u.m + first, left, t);
    }
    float s;
    const bool ok = held_scale<RMS, T>(m, tile0, 0, words_out, tb, partials, scale_out, rows, patience, &s);
    if (threadIdx.x == 0 && gridDim.x != 1) as_shared(gave_up)[blockIdx.x].store(ok ? 0u : 1u);
    if (!ok) {                                                // uniform
#pragma unroll
        for (int t = 0; t < T; ++t) held_st4<0>(delta_s + first, left, t, t < R ? v[t < R ? t : 0] : far[t < R ? 0 : t - R][threadIdx.x]);
        if (mine_cut) st4_tail(delta_s + first, cut_at, left, cut);
        if constexpr (kHeldSelf<R, L>)
            if (self) held_self_finish(delta_s, d, T, false, gave_up, rows, 0, m.sh, u);
        return;
    }
    // tiles in groups whose operands of the update are asked for together
    constexpr int G = P ? P : 2;
#pragma unroll
    for (int t0 = 0; t0 < T; t0 += G) {
        f32x4 xg[G], mg[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if constexpr (UPD != 0) {
                if (t0 + j < P) {
                    xg[j] = xv[j];
                    if constexpr (UPD == 2) mg[j] = mv[j];
                } else if (t0 + j < T) {
                    xg[j] = held_ld4<0>(u.x + first, left, t0 + j);
                    if constexpr (UPD == 2) mg[j] = held_ld4<0>(u.m + first, left, t0 + j);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const int t = t0 + j;
            if (t < T) {
                const f32x4 w = t < R ? v[t < R ? t : 0] : far[(t < R || t >= T) ? 0 : t - R][threadIdx.x];
                held_st4<0>(delta_s + first, left, t, sign_error4(w, s));
                if constexpr (UPD != 0) {
                    held_update4<UPD>(w, xg[j], mg[j], s, u);
                    held_st4<0>(u.x + first, left, t, xg[j]);
                    if constexpr (UPD == 2) held_st4<0>(u.m + first, left, t, mg[j]);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if (mine_cut) {
        st4_tail(delta_s + first, cut_at, left, sign_error4(cut, s));
        if constexpr (UPD != 0) {
            float *xr = u.x + first, *mr = UPD == 2 ? u.m + first : nullptr;
            f32x4 xc = ld4_tail(xr, cut_at, left), mc = UPD == 2 ? ld4_tail(mr, cut_at, left) : xc;
            held_update4<UPD>(cut, xc, mc, s, u);
            st4_tail(xr, cut_at, left, xc);
            if constexpr (UPD == 2) st4_tail(mr, cut_at, left, mc);
        }
    }
    if constexpr (kHeldSelf<R, L>)
        if (self) held_self_finish(delta_s, d, T, true, gave_up, rows, 0, m.sh, u);
}

// After a held launch (rows that finish themselves go without): forms the error (and, where u.x is set, the
// update) where a workgroup gave up,
// normally nowhere, and readies the synchronisation words for the next call.  One workgroup for every
// workgroup of the held launch.  Calls in which all waits are given up, 8 x 11,173,962: worker 375 us
// (two looks 289 us, held 213 us), server and update 66 us; 1203 and 521 us with one finishing workgroup for
// 64 of the held launch, which left 32 workgroups to go through all elements.
__global__ __launch_bounds__(kBlock) void k_sign_held_finish(float *buf, int64_t stride, int64_t d, const float *__restrict__ scales,
                                                             int T, const uint32_t *__restrict__ gave_up, HeldRow *rows,
                                                             HeldUpdate u)
{
    // from the end, as k_sign_pass2: what was written last is still in the memory-side cache
    const int row = gridDim.y - 1 - blockIdx.y, part = gridDim.x - 1 - blockIdx.x;
    if (part == 0 && threadIdx.x == 0) rows[row].next_call(row == 0);
    if (gave_up[row * static_cast<int64_t>(gridDim.x) + part] == 0u) return;
    held_finish_part(buf + row * stride, d, part, T, scales[row], u);
}

template <bool MOM, bool DECODE_ONLY, bool STREAM>
__global__ __launch_bounds__(kBlock) void k_sign_update(const uint64_t *__restrict__ words,
                                                        const float *__restrict__ scales,
                                                        ds_sign_tables tb, float *x, float *m,
                                                        int64_t d, float gamma, float beta)
{
    const int64_t tile = blockIdx.x;
    const TilePieces tp = tile_pieces(tb, tile);
    const int64_t e = tile * kTile + threadIdx.x * 4;
    if (e >= d) return;
    // the model (and momentum) words leave before the scale that the table entry leads to is
    // waited for
    f32x4 xv = {0.f, 0.f, 0.f, 0.f}, mv = xv;
    if constexpr (!DECODE_ONLY) {
        xv = STREAM ? ld4_stream(x, e, d) : ld4(x, e, d);
        if constexpr (MOM) mv = STREAM ? ld4_stream(m, e, d) : ld4(m, e, d);
    }
    const uint32_t nib = load_sign_nibble(words, e);
    float q[4];
    if (tp.seg0 >= 0) {
        const float s = scales[tp.seg0];
#pragma unroll
        for (int c = 0; c < 4; ++c) q[c] = (e + c < d) ? s : 0.f;
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) q[c] = (e + c < d) ? scales[seg_of(tb, tp.p0, tp.p1, e + c)] : 0.f;
    }
    f32x4 qv = signed4(q[0], q[1], q[2], q[3], nib);
    if constexpr (DECODE_ONLY) {
        st4_stream(x, e, d, qv);             // a decoded message: written once, read by the caller
    } else {
        if constexpr (MOM) {                       // m <- beta m + q ; x <- x - gamma m
            qv = fma4(beta, mv, qv);
            if constexpr (STREAM) st4_stream(m, e, d, qv);
            else st4(m, e, d, qv);
        }
        if constexpr (STREAM) st4_stream(x, e, d, fma4(-gamma, qv, xv));
        else st4(x, e, d, fma4(-gamma, qv, xv));
    }
}

// Server that does not compress (Section 5.1 "MEM-SGD"): a = (1/n) sum_i Q[v_i] by the chain
// from +0, per element: the element's bit and the scale of its group from every worker's
// message.  CHUNKS: the groups are chunks of `chunk` elements (a multiple of 4), else they come
// from the tile tables.
template <bool CHUNKS>
__global__ __launch_bounds__(kBlock) void k_sign_server_identity(ServerArgs a, int64_t d, int64_t chunk, ds_sign_tables tb,
                                                                 float *dense_out, ds_update_args u)
{
    const int64_t tile = blockIdx.x;
    const int64_t e = tile * kTile + threadIdx.x * 4;
    if (e >= d) return;
    int32_t seg[4];
    if constexpr (CHUNKS) {
        seg[0] = seg[1] = seg[2] = seg[3] = static_cast<int32_t>(static_cast<uint32_t>(e) / static_cast<uint32_t>(chunk));
    } else {
        const TilePieces tp = tile_pieces(tb, tile);
#pragma unroll
        for (int c = 0; c < 4; ++c) seg[c] = (tp.seg0 >= 0) ? tp.seg0 : ((e + c < d) ? seg_of(tb, tp.p0, tp.p1, e + c) : 0);
    }
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    for (int i = 0; i < a.n; ++i) {
        const float *srow = a.scales_in + i * a.S;
        const uint32_t nib = load_sign_nibble(a.words_in + i * a.W, e);
        v = fma4(a.inv_n, signed4(srow[seg[0]], srow[seg[1]], srow[seg[2]], srow[seg[3]], nib), v);
    }
    put_average4(zero_past(v, e, d), e, d, dense_out, u.x, u.m, u.gamma, u.beta);
}

}  // namespace

// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------
ds_status_t ds_sign_server_identity(ds_ctx *c, const ds_payload_t *in, float *dense_out, ds_update_args u, hipStream_t st)
{
    const ds_config_t &cfg = c->cfg;
    ServerArgs a{in->sign_words, in->scales, cfg.n, c->W, c->S, c->inv_n};
    const unsigned blocks = static_cast<unsigned>(c->n_tiles);
    if (c->sign_fused) k_sign_server_identity<true><<<blocks, kBlock, 0, st>>>(a, cfg.d, cfg.chunk, c->sign_tb, dense_out, u);
    else k_sign_server_identity<false><<<blocks, kBlock, 0, st>>>(a, cfg.d, 0, c->sign_tb, dense_out, u);
    return ds_launch_status();
}

ds_status_t ds_sign_init(ds_ctx *c)
{
    const ds_config_t &cfg = c->cfg;
    const int64_t d = cfg.d;
    c->sign_fused = false;
    c->sign_defer = c->sign_w_deferred = c->sign_s_deferred = false;
    c->sign_prev_w = c->sign_prev_s = nullptr;
    c->sign_tb_mem = nullptr;
    c->sign_partials = nullptr;
    c->held = c->held_s = ds_held_sync{};
    std::vector<int64_t> seg_off;
    if (cfg.scale_mode == DS_SCALE_WHOLE) {
        seg_off = {0, d};
    } else if (cfg.scale_mode == DS_SCALE_SEGMENTS) {
        seg_off.assign(cfg.seg_offsets, cfg.seg_offsets + cfg.n_seg + 1);
    } else {
        if (cfg.chunk % 128 == 0 && cfg.chunk >= 512 && cfg.chunk <= kTile) {
            c->sign_fused = true;
            c->S = (d + cfg.chunk - 1) / cfg.chunk;
            return DS_OK;
        }
        for (int64_t o = 0; o < d; o += cfg.chunk) seg_off.push_back(o);
        seg_off.push_back(d);
    }
    const int64_t S = static_cast<int64_t>(seg_off.size()) - 1;
    c->S = S;
    const int64_t n_tiles = c->n_tiles;
    // One group for the whole vector: a piece is a tile, and the kernels read none of the tables.  Uploading them
    // was most of the time to create such a context.
    int64_t n_pieces = n_tiles;
    if (S > 1) {
        std::vector<int32_t> tile_piece_first(n_tiles + 1), piece_seg, seg_piece_first(S + 1);
        std::vector<int2> tile_info(n_tiles);
        std::vector<int64_t> piece_start;
        int64_t s = 0;
        for (int64_t t = 0; t < n_tiles; ++t) {
            const int64_t lo = t * kTile, hi = (lo + kTile < d) ? lo + kTile : d;
            tile_piece_first[t] = static_cast<int32_t>(piece_start.size());
            int64_t pos = lo;
            while (pos < hi) {
                while (seg_off[s + 1] <= pos) ++s;
                if (pos == seg_off[s]) seg_piece_first[s] = static_cast<int32_t>(piece_start.size());
                piece_start.push_back(pos);
                piece_seg.push_back(static_cast<int32_t>(s));
                pos = (seg_off[s + 1] < hi) ? seg_off[s + 1] : hi;
            }
        }
        n_pieces = static_cast<int64_t>(piece_seg.size());
        if (n_pieces > 0x7FFFFFFF) return DS_ERR_SHAPE;
        tile_piece_first[n_tiles] = static_cast<int32_t>(n_pieces);
        seg_piece_first[S] = static_cast<int32_t>(n_pieces);
        piece_start.push_back(d);
        for (int64_t t = 0; t < n_tiles; ++t) {
            const int32_t p0 = tile_piece_first[t], cnt = tile_piece_first[t + 1] - p0;
            tile_info[t] = int2{p0, cnt == 1 ? piece_seg[p0] : -cnt};
        }

        // one allocation: int64 arrays first (8-byte aligned), then the int32 arrays
        const size_t b_ps = sizeof(int64_t) * (n_pieces + 1), b_so = sizeof(int64_t) * (S + 1);
        const size_t b_tpf = sizeof(int32_t) * (n_tiles + 1), b_pseg = sizeof(int32_t) * n_pieces;
        const size_t b_spf = sizeof(int32_t) * (S + 1), b_ti = sizeof(int2) * n_tiles;
        char *mem = nullptr;
        DS_HIP_TRY(hipMalloc(&mem, b_ps + b_so + b_ti + b_tpf + b_pseg + b_spf));
        c->sign_tb_mem = mem;
        char *p = mem;
        auto put = [&](const void *src, size_t bytes) -> const void * {
            const void *at = p;
            if (bytes) (void)hipMemcpy(p, src, bytes, hipMemcpyHostToDevice);
            p += bytes;
            return at;
        };
        c->sign_tb.piece_start = static_cast<const int64_t *>(put(piece_start.data(), b_ps));
        c->sign_tb.seg_off = static_cast<const int64_t *>(put(seg_off.data(), b_so));
        c->sign_tb.tile_info = static_cast<const int2 *>(put(tile_info.data(), b_ti));
        c->sign_tb.tile_piece_first = static_cast<const int32_t *>(put(tile_piece_first.data(), b_tpf));
        c->sign_tb.piece_seg = static_cast<const int32_t *>(put(piece_seg.data(), b_pseg));
        c->sign_tb.seg_piece_first = static_cast<const int32_t *>(put(seg_piece_first.data(), b_spf));
    }
    c->sign_tb.n_pieces = static_cast<int32_t>(n_pieces);
    c->sign_tb.n_seg = static_cast<int32_t>(S);
    c->sign_tb.rms = (cfg.flags & DS_FLAG_SIGN_RMS) != 0;
    c->sign_tb.whole_d = (S == 1) ? d : 0;
    if (hipGetLastError() != hipSuccess) return DS_ERR_DEVICE;
    DS_HIP_TRY(hipMalloc(&c->sign_partials, sizeof(double) * n_pieces * static_cast<size_t>(cfg.n)));
    if (S == 1 && !c->nofb && !(cfg.flags & DS_FLAG_DEFERRED_ERROR)) {
        // Worker.  GPU time of a call, n = 1 .. 16, against two looks as separate launches and one tile per workgroup:
        //  * one workgroup, 8 tiles in 8: 5.5 .. 6.1 us (bf16 6.3 .. 7.3), 7.1 .. 9.0 and 6.4 .. 7.8 us; 12 tiles in 14: 7.4 .. 8.2 us
        //    (bf16 9.0 .. 9.9), 7.7 .. 9.5 and 6.6 .. 7.4 us; 24 tiles in 24: 11.3 .. 12.1 us (bf16 13.9 .. 15.2), 7.3 .. 11.2 and
        //    6.5 .. 8.3 us;
        //  * 1 x 1,000,003: 12.8, 10.3, 9.1 and 9.7 us with 1, 2, 4 and 8 tiles, 10.1 us in two looks; 4 x 300,001: 9.8, 8.8
        //    and 9.2 us with 1, 2 and 4;
        //  * 7 x 2,345,679: 72, 42, 35, 38 us with 2, 4, 8, 14 tiles, of which 8 is the first that holds all rows;
        //  * 8 x 5,000,003: 88 us with 14, 93 us with 24 tiles; 8 x 16,000,000: 352 and 333 us, 541 us in two looks;
        //    8 x 24,000,000: 454 us with 24, 619 us in two looks.
        static constexpr HeldStep worker[] = {{1, 0, 128}, {2, 0, 128}, {4, 0, 0}, {8, 0, 0}, {14, 4, 0}, {24, 1, 0}};
        const ds_status_t rc = held_size(c, cfg.n, 8, worker, [](auto r, auto l) {
            constexpr int R = decltype(r)::value, L = decltype(l)::value;
            int per_cu = 0;
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_sign_held_worker<false, false, R, L>, kBlock, 0) ==
                           hipSuccess ? per_cu : -1;
        }, &c->held);
        if (rc != DS_OK) return rc;
        if (c->held.T) {
            const ds_status_t ra = held_alloc(c, cfg.n, &c->held);
            if (ra != DS_OK) return ra;
        }
        // The server's block handles one row, and the chain over the workers comes once per tile, so that the more
        // workers there are, the more workgroups are wanted.  GPU time of server and update against
        // separate launches:
        //  * one workgroup: 4 tiles in 4: 5.7 us (n = 1), 6.8 us (n = 8), 8.9 us (n = 16), 9.2 .. 9.9 us, one tile per
        //    workgroup 6.6 .. 7.5 us; 8 tiles in 8: 8.7 .. 15.5 us, 9.0 .. 10.0 us; 24 tiles in 24: 22 .. 42 us, 9.1 .. 10.1 us,
        //    one tile per workgroup 6.9 .. 7.8 us; n = 64: 2 tiles in 2 12.0 us, 12.7 us, in two workgroups 10.3 us;
        //  * d = 1,000,003, n = 1: 13.7, 11.4 and 11.4 us with 1, 2 and 4 tiles, 13.1 us; n = 16: 14.7, 13.2 and 14.7, 14.6 us;
        //  * d = 8,000,002: 35 us with 4 tiles, 47 us (n = 8), 53 and 61 us (n = 32), 77.6 and 80.8 us (n = 64), 185 and 174 us
        //    (n = 200); d = 16,000,001, 8 tiles: 57 and 80 us (n = 8), 95 and 107 us (n = 32); 11,173,962 and n = 64: 113 and
        //    106 us; d = 2,500,001, 2 tiles: 35.0 and 35.6 us (n = 64), 77 and 68 us (n = 200);
        //  * d = 18,000,001 with momentum, 14 tiles: 132 and 134 us (n = 20), 155 and 147 us (n = 32); d = 24,000,000, 24 tiles:
        //    171 and 172 us (n = 20), 200 and 188 us (n = 32).
        static constexpr HeldStep few[] = {{1, 0, 256}, {2, 0, 256}, {4, 0, 0}, {8, 0, 0}, {14, 0, 0}, {24, 0, 0}};
        static constexpr HeldStep upto24[] = {{1, 0, 256}, {2, 0, 0}, {4, 0, 0}, {8, 0, 0}, {14, 0, 0}, {24, 0, 0}};
        static constexpr HeldStep upto32[] = {{1, 0, 256}, {2, 0, 0}, {4, 0, 0}, {8, 0, 0}, {0, 0, 0}, {0, 0, 0}};
        static constexpr HeldStep upto64[] = {{1, 0, 0}, {2, 0, 0}, {0, 0, 0}, {0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
        static constexpr HeldStep many[] = {{1, 0, 0}, {0, 0, 0}, {0, 0, 0}, {0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
        const int n = cfg.n, one = n <= 8 ? 4 : n <= 32 ? 2 : 1;
        const auto &server = n <= 8 ? few : n <= 24 ? upto24 : n <= 32 ? upto32 : n <= 64 ? upto64 : many;
        const ds_status_t rs = c->sid ? DS_OK : held_size(c, 1, one, server, [](auto r, auto l) {
            constexpr int R = decltype(r)::value, L = decltype(l)::value;
            int per_cu = 0;
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_sign_held_server<false, 2, R, L>, kBlock, 0) ==
                           hipSuccess ? per_cu : -1;
        }, &c->held_s);
        if (rs != DS_OK) return rs;
        if (c->held_s.T) {
            const ds_status_t ra = held_alloc(c, 1, &c->held_s);
            if (ra != DS_OK) return ra;
        }
    }
    if ((cfg.flags & DS_FLAG_DEFERRED_ERROR) && !c->nofb) {
        c->sign_defer = true;
        DS_HIP_TRY(hipMalloc(&c->sign_prev_w, sizeof(float) * static_cast<size_t>(S) * cfg.n));
        DS_HIP_TRY(hipMalloc(&c->sign_prev_s, sizeof(float) * static_cast<size_t>(S)));
    }
    return DS_OK;
}

void ds_sign_fini(ds_ctx *c)
{
    if (c->sign_tb_mem) (void)hipFree(c->sign_tb_mem);
    if (c->sign_partials) (void)hipFree(c->sign_partials);
    held_free(&c->held);
    held_free(&c->held_s);
    if (c->sign_prev_w) (void)hipFree(c->sign_prev_w);
    if (c->sign_prev_s) (void)hipFree(c->sign_prev_s);
    c->sign_prev_w = c->sign_prev_s = nullptr;
    c->sign_tb_mem = nullptr;
    c->sign_partials = nullptr;
}

// Calls f with the run-time flags turned into compile-time constants (std::bool_constant).
template <class F>
static void with_flags(bool a, bool b, bool c, F f)
{
    auto l2 = [&](auto ta, auto tb) { if (c) f(ta, tb, std::true_type{}); else f(ta, tb, std::false_type{}); };
    auto l1 = [&](auto ta) { if (b) l2(ta, std::true_type{}); else l2(ta, std::false_type{}); };
    if (a) l1(std::true_type{}); else l1(std::false_type{});
}

// Pass 2 over `rows` rows.  Its stores are ordinary ones where the buffer is more than what the eight L2s take in
// beside the rest and fits the 256 MB memory-side cache, which then still holds it for the next call.  Whole
// steps with groups of 16,384, ordinary against non-temporal: 8 x 800,000 (26 MB) 43.5 and 48.0 us, 8 x 1,000,002
// 48.8 and 52.4 us, 8 x 4,000,002 137 and 143 us, 1 x 25,557,032 (102 MB) 193 and 202 us, 16 x 3,900,002 (250 MB) 229
// and 234 us; but 16 x 200,002 (13 MB) 38 and 33 us, 8 x 25,557,030 (818 MB) 870 and 839 us, and, where the worker's and
// the server's buffer do not fit together, 1 x 60,000,002 431 and 418 us.
static void sign_pass2(float *buf, int64_t stride, int64_t d, int64_t rows, const float *scales, int64_t S, const ds_sign_tables &tb, hipStream_t st)
{
    const dim3 grid(static_cast<unsigned>((d + kTile - 1) / kTile), static_cast<unsigned>(rows));
    const int64_t mb = (rows * d * 4) >> 20;
    if (mb >= 20 && mb < 256 && (d * 4) >> 20 < 192) k_sign_pass2<false><<<grid, kBlock, 0, st>>>(buf, stride, d, scales, S, tb);
    else k_sign_pass2<true><<<grid, kBlock, 0, st>>>(buf, stride, d, scales, S, tb);
}

ds_status_t ds_sign_worker(ds_ctx *c, const void *g, int64_t gs, float *delta, int64_t dstr,
                           const ds_payload_t *out, hipStream_t st)
{
    const ds_config_t &cfg = c->cfg;
    const bool bf16 = cfg.grad_dtype == DS_BF16;
    const bool rms = (cfg.flags & DS_FLAG_SIGN_RMS) != 0;
    if (c->sign_fused) {
        // With every other row's errors stored with ordinary accesses the next call finds those rows in a cache,
        // where the buffer as a whole would not stay: half of it in the eight L2s (32 MB) or, beside the gradients, in
        // the 256 MB memory-side cache.  Whole steps, chunks of 2048, ordinary accesses for no, every other and every row:
        //  * fp32: 8 x 400,000 (13 MB) 14.6, 13.4 and 13.9 us; 16 x 2,000,000 (128 MB) 73.8, 72.0 and 73.5 us; 16 x 3,900,000
        //    (250 MB) 139, 131 and 135 us; 8 x 11,173,960 (357 MB) 212, 200 and 235 us; 2 x 60,000,002 (480 MB) 400, 382 and
        //    437 us; in between 4 x 4,000,000 (64 MB) 46.2, 47.1 and 47.1 us; beyond, 8 x 25,557,032 (818 MB) 490 and 516 us;
        //  * bf16: 8 x 11,173,960 183 and 180 us, 8 x 16,000,002 259 and 254 us, but 16 x 1,000,002 36.8 and 38.0 us;
        //  * chunks of 512, 4 x 11,173,962: 209 and 216 us.
        const int64_t mb = (cfg.n * cfg.d * 4) >> 20, half_mb = ((cfg.n / 2) * cfg.d * 4) >> 20;
        const bool keep_odd = cfg.chunk == kTile && half_mb < 256 && (bf16 ? mb >= 256 : mb <= 32 || mb >= 96);
        with_flags(bf16, rms, c->nofb, [&](auto bf, auto rm, auto nf) {
            constexpr bool BF = decltype(bf)::value, RM = decltype(rm)::value, NF = decltype(nf)::value;
            constexpr int CPW = NF ? 4 : 2;
            const dim3 grid(static_cast<unsigned>((c->S + CPW - 1) / CPW), static_cast<unsigned>(cfg.n));
            WorkerSrc<BF> src{g, gs, delta, dstr};
            k_sign_chunk_worker<BF, RM, NF, CPW><<<grid, kBlock, 0, st>>>(src, delta, cfg.d, cfg.chunk, out->sign_words, c->W,
                                                                          out->scales, c->S, keep_odd);
        });
        return ds_launch_status();
    }
    if (c->held.T) {
        const ds_held_sync &h = c->held;
        const unsigned rows_n = static_cast<unsigned>(cfg.n);
        HeldRow *rows = static_cast<HeldRow *>(h.rows);
        with_held(h.T, [&](auto rr, auto ll) {
            constexpr int R = decltype(rr)::value, L = decltype(ll)::value;
            with_flags(bf16, rms, false, [&](auto bf, auto rm, auto) {
                constexpr bool BF = decltype(bf)::value, RM = decltype(rm)::value;
                WorkerSrc<BF> src{g, gs, delta, dstr};
                k_sign_held_worker<BF, RM, R, L><<<dim3(static_cast<unsigned>(h.parts), rows_n), kBlock, 0, st>>>(
                    src, delta, cfg.d, out->sign_words, c->W, c->sign_tb, c->sign_partials, out->scales, rows, h.gave_up, h.patience, h.self);
            });
        });
        if (h.parts > 1 && !h.self)
            k_sign_held_finish<<<dim3(static_cast<unsigned>(h.parts), rows_n), kBlock, 0, st>>>(
                delta, dstr, cfg.d, out->scales, h.T, h.gave_up, rows, HeldUpdate{nullptr, nullptr, 0.f, 0.f});
        return ds_launch_status();
    }
    dim3 grid(static_cast<unsigned>(c->n_tiles), static_cast<unsigned>(cfg.n));
    const bool deferred = c->sign_defer && c->sign_w_deferred;     // never set without compensation
    with_flags(bf16, deferred || c->nofb, rms, [&](auto bf, auto md, auto rm) {
        constexpr bool BF = decltype(bf)::value, MD = decltype(md)::value, RM = decltype(rm)::value;
        WorkerSrc<BF> src{g, gs, delta, dstr};
        if (!MD)
            k_sign_pass1_worker<BF, 0, RM><<<grid, kBlock, 0, st>>>(src, delta, cfg.d, out->sign_words, c->W, c->sign_tb,
                                                                    c->sign_partials, c->sign_prev_w, c->S);
        else if (deferred)
            k_sign_pass1_worker<BF, 1, RM><<<grid, kBlock, 0, st>>>(src, delta, cfg.d, out->sign_words, c->W, c->sign_tb,
                                                                    c->sign_partials, c->sign_prev_w, c->S);
        else
            k_sign_pass1_worker<BF, 2, RM><<<grid, kBlock, 0, st>>>(src, delta, cfg.d, out->sign_words, c->W, c->sign_tb,
                                                                    c->sign_partials, c->sign_prev_w, c->S);
    });
    k_sign_reduce<<<dim3(static_cast<unsigned>(c->S), static_cast<unsigned>(cfg.n)), kBlock, 0, st>>>(
        c->sign_partials, c->sign_tb, out->scales, c->S, c->sign_defer ? c->sign_prev_w : nullptr);
    if (!c->sign_defer && delta) sign_pass2(delta, dstr, cfg.d, cfg.n, out->scales, c->S, c->sign_tb, st);
    const ds_status_t rc = ds_launch_status();
    if (rc == DS_OK && c->sign_defer) c->sign_w_deferred = true;   // the buffer now holds v; delta = v - Q[v] is applied by the next load
    return rc;
}

// x != nullptr (chunk and held routes only): the model update for the same elements in the same kernel.
ds_status_t ds_sign_server(ds_ctx *c, const ds_payload_t *in, float *delta_s, const ds_payload_t *out,
                           hipStream_t st, float *x, float *m, float gamma, float beta)
{
    const ds_config_t &cfg = c->cfg;
    ServerArgs a{in->sign_words, in->scales, cfg.n, c->W, c->S, c->inv_n};
    const bool rms = (cfg.flags & DS_FLAG_SIGN_RMS) != 0;
    if (c->sign_fused) {
        // two chunks per workgroup: more bytes in flight per thread (measured 271 us against
        // 292 us with one and 285 us with four on the 124 M-element workload)
        const dim3 grid(static_cast<unsigned>((c->S + 1) / 2));
        auto launch = [&](auto rm, auto upd) {
            constexpr bool RM = decltype(rm)::value;
            constexpr int UPD = decltype(upd)::value;
            k_sign_chunk_server<2, RM, UPD><<<grid, kBlock, 0, st>>>(a, delta_s, cfg.d, cfg.chunk, out->sign_words, out->scales,
                                                                      x, m, gamma, beta);
        };
        auto with_upd = [&](auto rm) {
            if (!x) launch(rm, std::integral_constant<int, 0>{});
            else if (!m) launch(rm, std::integral_constant<int, 1>{});
            else launch(rm, std::integral_constant<int, 2>{});
        };
        if (rms) with_upd(std::true_type{}); else with_upd(std::false_type{});
        return ds_launch_status();
    }
    if (c->held_s.T) {
        const ds_held_sync &h = c->held_s;
        HeldRow *rows = static_cast<HeldRow *>(h.rows);
        const HeldUpdate u{x, m, gamma, beta};
        with_held(h.T, [&](auto rr, auto ll) {
            constexpr int R = decltype(rr)::value, L = decltype(ll)::value;
            with_flags(rms, x != nullptr, m != nullptr, [&](auto rm, auto up, auto mo) {
                constexpr bool RM = decltype(rm)::value;
                constexpr int UPD = decltype(up)::value ? (decltype(mo)::value ? 2 : 1) : 0;
                k_sign_held_server<RM, UPD, R, L><<<static_cast<unsigned>(h.parts), kBlock, 0, st>>>(
                    a, delta_s, cfg.d, out->sign_words, c->sign_tb, c->sign_partials, out->scales, u, rows, h.gave_up, h.patience, h.self);
            });
        });
        if (h.parts > 1 && !h.self)
            k_sign_held_finish<<<static_cast<unsigned>(h.parts), kBlock, 0, st>>>(
                delta_s, cfg.d, cfg.d, out->scales, h.T, h.gave_up, rows, u);
        return ds_launch_status();
    }
    if (x) return DS_ERR_UNSUPPORTED;   // the caller asks for the fused form on the routes that have it
    dim3 grid(static_cast<unsigned>(c->n_tiles));
    const bool deferred = c->sign_defer && c->sign_s_deferred && delta_s;
    // Deferred form: the buffer is looked at once per call, so it may stream past the caches.
    // Measured on the 11 M-element workload (45 MB per buffer) that costs more than it saves:
    // server call 35.0 us streamed, 33.7 us with ordinary accesses, the next worker pass 1 us
    // slower; the 124 M-element measurements that led to streaming stand for large buffers.
    const bool stream = deferred && ds_stream_worthwhile(cfg.d);
    with_flags(deferred, rms, stream, [&](auto df, auto rm, auto sm) {
        constexpr bool DF = decltype(df)::value, RM = decltype(rm)::value, SM = decltype(sm)::value;
        k_sign_pass1_server<DF, RM, SM><<<grid, kBlock, 0, st>>>(a, delta_s, cfg.d, out->sign_words, c->sign_tb, c->sign_partials,
                                                             deferred ? c->sign_prev_s : nullptr);
    });
    k_sign_reduce<<<dim3(static_cast<unsigned>(c->S), 1), kBlock, 0, st>>>(c->sign_partials, c->sign_tb, out->scales, c->S,
                                                                          c->sign_defer ? c->sign_prev_s : nullptr);
    if (!c->sign_defer && delta_s) sign_pass2(delta_s, cfg.d, cfg.d, 1, out->scales, c->S, c->sign_tb, st);
    const ds_status_t rc = ds_launch_status();
    if (rc == DS_OK && c->sign_defer) c->sign_s_deferred = true;
    return rc;
}

// Deferred error form -> plain form, in place; a no-op for buffers that are in plain form.
ds_status_t ds_sign_materialize(ds_ctx *c, float *delta, int64_t dstr, float *delta_s, hipStream_t st)
{
    const ds_config_t &cfg = c->cfg;
    if (!c->sign_defer) return DS_OK;
    if (delta && c->sign_w_deferred) {
        sign_pass2(delta, dstr, cfg.d, cfg.n, c->sign_prev_w, c->S, c->sign_tb, st);
        c->sign_w_deferred = false;
    }
    if (delta_s && c->sign_s_deferred) {
        sign_pass2(delta_s, cfg.d, cfg.d, 1, c->sign_prev_s, c->S, c->sign_tb, st);
        c->sign_s_deferred = false;
    }
    return ds_launch_status();
}

template <bool DECODE_ONLY>
static ds_status_t sign_update_impl(ds_ctx *c, const uint64_t *words, const float *scales, float *x, float *m,
                                    float gamma, float beta, hipStream_t st)
{
    const ds_config_t &cfg = c->cfg;
    if (c->sign_fused) {
        const unsigned blocks = static_cast<unsigned>((cfg.d + kBlock * 4 - 1) / (kBlock * 4));
        if (m && !DECODE_ONLY)
            k_sign_chunk_update<true, false><<<blocks, kBlock, 0, st>>>(words, scales, cfg.chunk, x, m, cfg.d, gamma, beta);
        else
            k_sign_chunk_update<false, DECODE_ONLY><<<blocks, kBlock, 0, st>>>(words, scales, cfg.chunk, x, m, cfg.d, gamma, beta);
    } else {
        const unsigned blocks = static_cast<unsigned>(c->n_tiles);
        // ordinary accesses to a small model: 20.4 us -> 18.8 us on the 11 M-element workload
        const bool stream = DECODE_ONLY || ds_stream_worthwhile(cfg.d);
        if (m && !DECODE_ONLY) {
            if (stream) k_sign_update<true, false, true><<<blocks, kBlock, 0, st>>>(words, scales, c->sign_tb, x, m, cfg.d, gamma, beta);
            else k_sign_update<true, false, false><<<blocks, kBlock, 0, st>>>(words, scales, c->sign_tb, x, m, cfg.d, gamma, beta);
        } else {
            if (stream) k_sign_update<false, DECODE_ONLY, true><<<blocks, kBlock, 0, st>>>(words, scales, c->sign_tb, x, m, cfg.d, gamma, beta);
            else k_sign_update<false, DECODE_ONLY, false><<<blocks, kBlock, 0, st>>>(words, scales, c->sign_tb, x, m, cfg.d, gamma, beta);
        }
    }
    return ds_launch_status();
}

ds_status_t ds_sign_update(ds_ctx *c, const ds_payload_t *srv, float *x, float *m, float gamma, float beta,
                           hipStream_t st)
{
    return sign_update_impl<false>(c, srv->sign_words, srv->scales, x, m, gamma, beta, st);
}

ds_status_t ds_sign_decode(ds_ctx *c, const ds_payload_t *p, int32_t row, float *out, hipStream_t st)
{
    return sign_update_impl<true>(c, p->sign_words + row * c->W, p->scales + row * c->S, out, nullptr, 0.f, 0.f, st);
}

// ---------------------------------------------------------------------------------------
// the worker block without a context and without any allocation
// ---------------------------------------------------------------------------------------
// The general route needs the fp64 partial sums of every tile between its first pass and the
// reduce.  ds_create allocates them; callers that cannot allocate get them from this fixed
// array instead (one copy per device, held until the process ends).
#define DS_NOALLOC_MAX_PARTIALS 65536
static __device__ __align__(256) double scratch[DS_NOALLOC_MAX_PARTIALS];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
double *g_scratch_ptr[kMaxDevices];   // device address of `scratch` on each device, looked up once
}  // namespace

extern "C" ds_status_t ds_worker_compress_sign_noalloc(int32_t n, int64_t d, int32_t grad_dtype, int32_t flags,
                                                       const void *g, int64_t g_row_stride, float *delta,
                                                       int64_t delta_row_stride, uint64_t *sign_words, float *scales,
                                                       void *hip_stream)
{
    if (!g || !delta || !sign_words || !scales) return DS_ERR_NULL;
    if (n < 1 || n > 65535 || d < 1 || d > 0x7FFFFFFFLL) return DS_ERR_SHAPE;
    if (g_row_stride < d || delta_row_stride < d) return DS_ERR_SHAPE;
    if (grad_dtype != DS_F32 && grad_dtype != DS_BF16) return DS_ERR_CONFIG;
    if (flags & ~static_cast<int32_t>(DS_FLAG_SIGN_RMS)) return DS_ERR_CONFIG;
    const int64_t n_tiles = (d + kTile - 1) / kTile;
    if (n_tiles * n > DS_NOALLOC_MAX_PARTIALS) return DS_ERR_SHAPE;
    auto misaligned = [](const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; };
    if (misaligned(g) || misaligned(delta) || misaligned(sign_words) || misaligned(scales)) return DS_ERR_ALIGN;
    int dev = -1;
    DS_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return DS_ERR_DEVICE;
    double *partials = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[dev]) {
            // every device holds its own copy of the array at its own address
            void *p = nullptr;
            DS_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
            g_scratch_ptr[dev] = static_cast<double *>(p);
        }
        partials = g_scratch_ptr[dev];
    }
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    ds_sign_tables tb{};
    tb.n_pieces = static_cast<int32_t>(n_tiles);
    tb.n_seg = 1;
    tb.rms = (flags & DS_FLAG_SIGN_RMS) != 0;
    tb.whole_d = d;
    const int64_t W = (d + 63) / 64;
    const dim3 grid(static_cast<unsigned>(n_tiles), static_cast<unsigned>(n));
    with_flags(grad_dtype == DS_BF16, tb.rms, false, [&](auto bf, auto rm, auto) {
        constexpr bool BF = decltype(bf)::value, RM = decltype(rm)::value;
        WorkerSrc<BF> src{g, g_row_stride, delta, delta_row_stride};
        k_sign_pass1_worker<BF, 0, RM><<<grid, kBlock, 0, st>>>(src, delta, d, sign_words, W, tb, partials, nullptr, 1);
    });
    k_sign_reduce<<<dim3(1, static_cast<unsigned>(n)), kBlock, 0, st>>>(partials, tb, scales, 1, nullptr);
    sign_pass2(delta, delta_row_stride, d, n, scales, 1, tb, st);
    return ds_launch_status();
}
