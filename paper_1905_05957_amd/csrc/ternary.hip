// Ternary quantiser (Section 5.1 of the DoubleSqueeze paper, the compressor of its "QSGD"
// comparison system): every element becomes a code in {-1, 0, +1}.  With m the largest
// absolute value of the row, element e becomes sign(e) with probability |e| / m, decided by
// u < |e| / m with the element's 24-bit uniform (Philox4x32-10, counter (j >> 2, 0, stream,
// lo32(step)), key (lo32(seed), hi32(seed) ^ hi32(step)), word j & 3), and 0 otherwise.  One
// scale per row, sum |v| / number of non-zero codes ("magnitude of original gradient over
// magnitude of compressed gradient", read as l1), so that code * scale has the l1 magnitude of v.
//
// The comparison system runs without compensation and with a server that does not compress,
// and that is the mode built here: v = g, no error buffer.  The row-wide maximum has to be
// known before the first code.  Rows that the device can hold on chip are read once (k_tern_held, where
// that was measured to pay): the workgroups of a row keep its elements until the maximum is known.
// Other worker calls look at g twice:
//   stats    per 2048-element tile: max |v| and sum |v| (fp64)
//   rowstat  per row: the maximum, and the sum in a fixed order
//   encode   codes from the second look: two bit planes packed like the sign words, kept count per tile
//   scale    per row: sum / count, rounded once
// The message is 2 bits per element: plane `levels` (bit j = code_j is not 0), plane
// `sign_words` (bit j = code_j is -1), one fp32 scale.
#include "ds_device.h"
#include "ds_internal.h"
#include "held.h"

#include <new>

using namespace ds;

struct ds_tern_scratch {
    float *pmax;       // [n][n_tiles]
    double *psum;      // [n][n_tiles]
    uint32_t *pcnt;    // [n][n_tiles]
    float *rowmax;     // [n]
    double *rowsum;    // [n]
    ds_held_sync held;
};

namespace {

template <bool BF16>
__device__ __forceinline__ const void *grad_row(const void *g, int64_t gs, int row)
{
    if constexpr (BF16) return static_cast<const uint16_t *>(g) + row * gs;
    else return static_cast<const float *>(g) + row * gs;
}

template <bool BF16>
__global__ __launch_bounds__(kBlock) void k_tern_stats(const void *g, int64_t gs, int64_t d, float *pmax, double *psum)
{
    __shared__ double lds[kWaves];
    __shared__ float mx[kWaves];
    const int row = blockIdx.y;
    const int64_t e = static_cast<int64_t>(blockIdx.x) * kTile + threadIdx.x * 4;
    const void *grow = grad_row<BF16>(g, gs, row);
    const f32x4 v = ld4_grad<BF16>(grow, e, d);   // zero past d
    const float a0 = fabsf(v.x), a1 = fabsf(v.y), a2 = fabsf(v.z), a3 = fabsf(v.w);
    float m = fmaxf(fmaxf(a0, a1), fmaxf(a2, a3));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if (lane_id() == 0) mx[wave_id()] = m;
    const double total = block_sum(((static_cast<double>(a0) + static_cast<double>(a1)) + static_cast<double>(a2)) +
                                       static_cast<double>(a3), lds, false);   // its barrier also covers mx
    if (threadIdx.x == 0) {
        float t = mx[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) t = fmaxf(t, mx[w]);
        pmax[row * gridDim.x + blockIdx.x] = t;
        psum[row * gridDim.x + blockIdx.x] = total;
    }
}

// One workgroup per row: maximum and, in a fixed order, the sum over the row's tiles.
__global__ __launch_bounds__(kBlock) void k_tern_rowstat(const float *pmax, const double *psum, int64_t n_tiles,
                                                         float *rowmax, double *rowsum)
{
    __shared__ double lds[kWaves];
    __shared__ float mx[kWaves];
    const int row = blockIdx.x;
    double acc = 0.0;
    float m = 0.f;
    for (int64_t t = threadIdx.x; t < n_tiles; t += kBlock) {
        acc += psum[row * n_tiles + t];
        m = fmaxf(m, pmax[row * n_tiles + t]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if (lane_id() == 0) mx[wave_id()] = m;
    const double total = block_sum(acc, lds, false);          // its barrier also covers mx
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 0; w < kWaves; ++w) m = fmaxf(m, mx[w]);
        rowmax[row] = m;
        rowsum[row] = total;
    }
}

struct TernKey {
    uint32_t key0, key1, step_lo;
};

// What the encoding of a row needs to know of its maximum m: r = fl(2^32 / m), 0 where m leaves the range of the
// products below.
struct TernMax {
    float m, r;
};
__device__ __forceinline__ TernMax tern_max(float m)
{
    return TernMax{m, (m >= 0x1p-90f && m <= 0x1p90f) ? __fdiv_rn(0x1p32f, m) : 0.f};
}

// acc * 2 + the sign bit of x, in one instruction
__device__ __forceinline__ uint32_t push_sign(uint32_t acc, float x)
{
    return __builtin_amdgcn_alignbit(acc, __float_as_uint(x), 31);
}

// Codes of the four elements of group `quad` of the row (elements 4 quad .., zero past its end): bits of the codes
// that are not 0, and << 16 of those that are -1.  The encoding is bound by vector instructions.  Element |v| is kept
// iff U < 2^24 fl(|v| / m) for the upper 24 bits U of its random word R.  F = fl(R) is within 256 + 2^-24 R of 2^8 U, and
// D = F - |v| r, one rounding, within (2^-20 |v| r + 512) of 2^8 U - 2^32 fl(|v| / m): outside of that its sign is the decision,
// without the quotient, a shift or a comparison per bit.  Where one of the four lies inside, or is a NaN, and in rows whose
// maximum leaves the range, the quotients decide.
__device__ __forceinline__ uint32_t tern_codes4(f32x4 v, TernMax M, uint32_t quad, int row, TernKey K)
{
    const u32x4 rnd = philox4x32_10(u32x4{quad, 0u, static_cast<uint32_t>(row), K.step_lo}, K.key0, K.key1);
    const float tol = M.r * 0x1p-20f;
    uint32_t nz = 0u, neg = 0u;
    bool open = !(M.r > 0.f);                                   // uniform
#pragma unroll
    for (int c = 3; c >= 0; --c) {
        const float a = fabsf(v[c]);
        const float D = __fmaf_rn(a, -M.r, static_cast<float>(rnd[c]));
        open = open || !(fabsf(D) > __fmaf_rn(a, tol, 512.f));
        nz = push_sign(nz, D);
        neg = push_sign(neg, v[c]);
    }
    if (open) {
        nz = 0u;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            // not where m = 0: the quotient is a NaN
            const bool keep = static_cast<float>(rnd[c] >> 8) * 0x1p-24f < __fdiv_rn(fabsf(v[c]), M.m);
            nz |= keep ? 1u << c : 0u;
        }
    }
    return nz | ((nz & neg) << 16);                             // what is kept is not 0
}

// The 32-bit words that lane's group of eight lanes contributes to the two planes, from the codes of its lanes.
__device__ __forceinline__ void tern_words(uint32_t code, uint32_t &nz, uint32_t &neg)
{
    uint32_t w = code << (4 * (lane_id() & 3));                 // four lanes: 16 bits of either plane
    w |= dpp_u32<kDppXor1>(w);
    w |= dpp_u32<kDppXor2>(w);
    const uint32_t o = dpp_u32<kDppHalfMirror>(w);              // of the other four
    const bool upper = (lane_id() & 4) != 0;
    const uint32_t lo = upper ? o : w, hi = upper ? w : o;
    nz = (lo & 0xFFFFu) | (hi << 16);
    neg = (lo >> 16) | (hi & 0xFFFF0000u);
}

template <bool BF16>
__global__ __launch_bounds__(kBlock) void k_tern_encode(const void *g, int64_t gs, int64_t d, const float *rowmax,
                                                        uint32_t key0, uint32_t key1, uint32_t step_lo, uint64_t *neg,
                                                        uint64_t *nz, int64_t W, uint32_t *pcnt)
{
    __shared__ __attribute__((aligned(16))) uint32_t sw_neg[kWaves * 8], sw_nz[kWaves * 8];
    __shared__ uint32_t cnt[kWaves];
    const int row = blockIdx.y;
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kTile;
    const int64_t e = base + threadIdx.x * 4;
    const void *grow = grad_row<BF16>(g, gs, row);
    const f32x4 v = ld4_grad<BF16>(grow, e, d);
    const uint32_t code = tern_codes4(v, tern_max(rowmax[row]), static_cast<uint32_t>(e >> 2), row, TernKey{key0, key1, step_lo});
    uint32_t w_nz, w_neg;
    tern_words(code, w_nz, w_neg);
    stash_sign_words(sw_nz, w_nz);
    stash_sign_words(sw_neg, w_neg);
    const uint32_t kept = wave_sum_u32(static_cast<uint32_t>(__popc(code & 0xFFFFu)));
    if (lane_id() == 0) cnt[wave_id()] = kept;
    __syncthreads();
    flush_sign_words(sw_nz, nz + row * W, base, W * 64);
    flush_sign_words(sw_neg, neg + row * W, base, W * 64);
    if (threadIdx.x == 0) {
        uint32_t t = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) t += cnt[w];
        pcnt[row * gridDim.x + blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(kBlock) void k_tern_scale(const uint32_t *pcnt, const double *rowsum, int64_t n_tiles, float *scales)
{
    __shared__ unsigned long long sm[kBlock];
    const int row = blockIdx.x;
    unsigned long long acc = 0;
    for (int64_t t = threadIdx.x; t < n_tiles; t += kBlock) acc += pcnt[row * n_tiles + t];
    sm[threadIdx.x] = acc;
    __syncthreads();
    for (int o = kBlock / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o) sm[threadIdx.x] += sm[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) scales[row] = sm[0] ? static_cast<float>(rowsum[row] / static_cast<double>(sm[0])) : 0.f;
}

// ---------------------------------------------------------------------------------------
// held route: rows that are read once
// ---------------------------------------------------------------------------------------
// A workgroup keeps T consecutive tiles in registers and LDS, hands over their sums and maximum,
// waits for the row's maximum, which the workgroup that arrives last publishes, encodes what it holds
// and leaves its count of kept codes for the finish launch, which writes the scale.  Waits are bounded,
// and what a workgroup that gave up did not encode the finish launch does (held.h).  The arrival is the
// only word that all workgroups of a row add to: such additions come one after the other, about 11 ns
// each, and with the maximum and the count as two more of them a call at 1 x 1,000,003 took 24.9, 16.9 and
// 13.8 us with 1, 2 and 4 tiles per workgroup (16.0, 12.9 and 12.1 us without).
//
// What bounds it is vector instructions, 38 of Philox among about 150 per four elements (57 us for its bytes at the copy
// kernel's rate).  Worker call at 8 x 11,173,962: 159 us in two looks; 149 .. 154 us here with three comparisons per
// element in the encoding and a sum over the wavefront for every tile, 139 us with the encoding as it is (tern_codes4), 124 us
// with sums that stay with their thread until the end.  Tried without effect: drawing while the tiles are loaded and keeping
// |v| / U (145 us), and starting the second row later by a row's load, so that one would load while the other is
// encoded (138 .. 141 us for 0 .. 1.5 loads).
__device__ __forceinline__ float tern_scale(double sum, uint32_t kept)
{
    return kept ? static_cast<float>(sum / static_cast<double>(kept)) : 0.f;
}

struct TernShared {
    double sums[kWaves], red[kWaves];
    float mx[kWaves];
    uint32_t cnt[kWaves], sh[2];
};

// The wavefront's words of one tile to both planes: word of an 8-lane group, by its first lane.  Rows have
// fewer than 2^31 elements and a stretch reaches less than 2^31 past their end: 32 bits number the groups of
// four and their bits.
__device__ __forceinline__ void tern_put_words(uint32_t code, uint32_t quad, uint64_t *neg_row, uint64_t *nz_row, uint32_t words)
{
    const uint32_t w = quad >> 3;
    uint32_t a, b;
    tern_words(code, a, b);
    if ((lane_id() & 7) == 0 && w < words) {
        reinterpret_cast<uint32_t *>(nz_row)[w] = a;
        reinterpret_cast<uint32_t *>(neg_row)[w] = b;
    }
}

// Non-zero codes of the workgroup.  Every thread calls, with its own.
__device__ __forceinline__ uint32_t tern_kept(uint32_t kept, uint32_t *cnt)
{
    kept = wave_sum_u32(kept);
    if (lane_id() == 0) cnt[wave_id()] = kept;
    __syncthreads();
    uint32_t total = cnt[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) total += cnt[w];
    return total;
}

// Encodes what a workgroup that gave up did not; the thread's non-zero codes.
template <bool BF16>
__device__ __forceinline__ uint32_t tern_finish_part(const void *grow, int64_t d, int part, int T, TernMax M, int row, TernKey K,
                                                     uint64_t *neg_row, uint64_t *nz_row, uint32_t words)
{
    uint32_t kept = 0;
    f32x4 next = ld4_grad<BF16>(grow, static_cast<int64_t>(part) * T * kTile + threadIdx.x * 4, d);
    for (int t = 0; t < T; ++t) {
        const int64_t e = (static_cast<int64_t>(part) * T + t) * kTile + threadIdx.x * 4;
        const uint32_t quad = static_cast<uint32_t>(e >> 2);
        const f32x4 v = next;
        if (t + 1 < T) next = ld4_grad<BF16>(grow, e + kTile, d);       // zero past the end of the row
        const uint32_t code = tern_codes4(v, M, quad, row, K);
        tern_put_words(code, quad, neg_row, nz_row, words);
        kept += __popc(code & 0xFFFFu);
    }
    return kept;
}

template <bool BF16, int R, int L>
__global__ __launch_bounds__(kBlock, held_waves(R)) void k_tern_held(const void *g, int64_t gs, int64_t d, int32_t n_tiles, double *psum,
                                                                     float *pmax, uint32_t *pcnt, float *rowmax, double *rowsum, TernKey K,
                                                                     uint64_t *neg, uint64_t *nz, int64_t W, float *scales, HeldRow *rows,
                                                                     uint32_t *gave_up, uint32_t patience, bool self)
{
    constexpr int T = R + L;
    __shared__ TernShared sm;
    __shared__ f32x4 far[L ? L : 1][kBlock];
    const int row = blockIdx.y;
    const int64_t tile0 = static_cast<int64_t>(blockIdx.x) * T, first = tile0 * kTile;
    const void *grow = grad_row<BF16>(g, gs, row);
    int left = held_left<T>(tile0, d);
    f32x4 cut = {0.f, 0.f, 0.f, 0.f};
    int cut_at = -1;
    if (left & 3) {                                           // the row ends inside a group of four
        cut_at = left & ~3;
        cut = ld4_grad<BF16>(grow, first + cut_at, first + left);
    }
    constexpr int D = 6 < T ? 6 : T;                          // tiles in flight
    f32x4 v[R], ring[L ? D : 1];
    auto fetch = [&](auto qc) {
        constexpr int q = decltype(qc)::value;
        if constexpr (q < L) ring[q % D] = held_g4<BF16>(grow, first, left, R + q);
        else v[q - L] = held_g4<BF16>(grow, first, left, q - L);
    };
    float mx = 0.f;
    double sum = 0.0;                                         // of the thread's elements
    static_for<0, D>(fetch);
    static_for<0, T>([&](auto qc) {
        constexpr int q = decltype(qc)::value, t = q < L ? R + q : q - L;
        __builtin_amdgcn_sched_barrier(0);
        f32x4 w;
        if constexpr (q < L) w = ring[q % D];
        else w = v[t];
        const bool mine = static_cast<int>(threadIdx.x) * 4 + t * kTile == cut_at;
        w.x = mine ? cut.x : w.x;
        w.y = mine ? cut.y : w.y;
        w.z = mine ? cut.z : w.z;
        asm volatile("" : "+v"(w));
        if constexpr (q + D < T) fetch(std::integral_constant<int, q + D>{});
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (q < L) far[q][threadIdx.x] = w;
        else v[t] = w;
        const float a0 = fabsf(w.x), a1 = fabsf(w.y), a2 = fabsf(w.z), a3 = fabsf(w.w);
        mx = fmaxf(mx, fmaxf(fmaxf(a0, a1), fmaxf(a2, a3)));
        asm volatile("" : "+v"(mx));      // now: put off to the end, the maximum keeps |v| of all tiles in registers
        sum += ((static_cast<double>(a0) + static_cast<double>(a1)) + static_cast<double>(a2)) + static_cast<double>(a3);
        asm volatile("" : "+v"(sum));
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    sum = wave_sum(sum);
    if (lane_id() == 0) { sm.mx[wave_id()] = mx; sm.sums[wave_id()] = sum; }
    held_fence(v, left);
    __syncthreads();
    sum = sm.sums[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) sum += sm.sums[w];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) mx = fmaxf(mx, sm.mx[w]);
    const bool alone = gridDim.x == 1;
    bool ok = true;
    if (!alone) {
        uint64_t *psum_row = reinterpret_cast<uint64_t *>(psum) + static_cast<int64_t>(row) * n_tiles;
        uint32_t *pmax_row = reinterpret_cast<uint32_t *>(pmax) + static_cast<int64_t>(row) * n_tiles;   // both one per workgroup
        if (wave_id() == 0) {
            if (lane_id() == 0) {
                as_shared(psum_row)[blockIdx.x].store(__double_as_longlong(sum));
                as_shared(pmax_row)[blockIdx.x].store(__float_as_uint(mx));
            }
            // both are in memory before the arrival is announced
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (lane_id() == 0) sm.sh[0] = (rows[row].arrived.fetch_add(1u) + 1u == gridDim.x) ? 1u : 0u;
        }
        __syncthreads();
        const bool last = sm.sh[0] != 0u;
        __syncthreads();
        if (!last) {
            ok = held_wait(rows, row, patience, sm.sh, &mx);
        } else {
            double acc = 0.0;
            for (uint32_t p = threadIdx.x; p < gridDim.x; p += kBlock)
                acc += __longlong_as_double(static_cast<long long>(as_shared(psum_row)[p].load()));
            const double total = block_sum(acc, sm.red, false);
            if (wave_id() == 0) {
                for (uint32_t p = lane_id(); p < gridDim.x; p += 64) mx = fmaxf(mx, __uint_as_float(as_shared(pmax_row)[p].load()));
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
                if (lane_id() == 0) {
                    rowmax[row] = mx;                         // for the finish launch
                    as_shared(reinterpret_cast<uint64_t *>(rowsum))[row].store(__double_as_longlong(total));
                    rows[row].pub.store(kHeldValue | __float_as_uint(mx));
                    sm.sh[1] = __float_as_uint(mx);
                }
            }
            __syncthreads();
            mx = __uint_as_float(sm.sh[1]);
        }
        if (threadIdx.x == 0) {
            as_shared(gave_up + row * static_cast<int64_t>(gridDim.x))[blockIdx.x].store(ok ? 0u : 1u);
            if (!ok) rows[row].late.store(1u);
        }
        if (!ok && !(kHeldSelf<R, L> && self)) return;        // uniform
    }
    held_fence(v, left);
    const uint32_t words = static_cast<uint32_t>(W) * 2u, quad0 = static_cast<uint32_t>(first >> 2) + threadIdx.x;
    uint64_t *neg_row = neg + row * W, *nz_row = nz + row * W;
    uint32_t kept = 0;
    const TernMax M = tern_max(mx);
    auto encode = [&](f32x4 w, int t) {
        const uint32_t quad = quad0 + t * (kTile / 4);
        const uint32_t code = tern_codes4(w, M, quad, row, K);
        tern_put_words(code, quad, neg_row, nz_row, words);
        kept += __popc(code & 0xFFFFu);
    };
    if (!kHeldSelf<R, L> || ok) {                             // uniform
#pragma unroll
        for (int t = 0; t < R; ++t) {
            encode(v[t], t);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll 1
        for (int t = R; t < T; ++t) encode(far[t - R][threadIdx.x], t);
    }
    kept = tern_kept(kept, sm.cnt);
    if constexpr (kHeldSelf<R, L>)
        if (self) {
            uint32_t all;
            if (!held_depart(rows + row, gridDim.x, ok, kept, sm.sh, &all)) return;
            if (rows[row].late.load() != 0u) {                // uniform: all have departed
                const float m = __uint_as_float(static_cast<uint32_t>(rows[row].pub.load()));
                uint32_t more = 0;
                for (uint32_t p = 0; p < gridDim.x; ++p)
                    if (as_shared(gave_up + row * static_cast<int64_t>(gridDim.x))[p].load() != 0u)
                        more += tern_finish_part<BF16>(grow, d, static_cast<int>(p), T, tern_max(m), row, K, neg_row, nz_row, words);
                __syncthreads();                              // sm.cnt is used again
                all += tern_kept(more, sm.cnt);
            }
            if (threadIdx.x != 0) return;
            scales[row] = tern_scale(__longlong_as_double(static_cast<long long>(as_shared(reinterpret_cast<uint64_t *>(rowsum))[row].load())), all);
            rows[row].next_call(row == 0);
            return;
        }
    if (threadIdx.x != 0) return;
    if (alone) scales[row] = tern_scale(sum, kept);
    else pcnt[static_cast<int64_t>(row) * n_tiles + blockIdx.x] = kept;    // added up by the finish launch
}

// After a held launch: writes the scale of every row from the counts of its workgroups and readies the
// synchronisation words for the next call.  In a row in which a workgroup gave up (normally none) one
// workgroup for each of them encodes what it held, and the one that is through last adds up.
// 8 x 11,173,962 with all waits given up: 169 us; with one finishing workgroup for 64 of the held launch it was seven
// times that.
template <bool BF16>
__global__ __launch_bounds__(kBlock) void k_tern_held_finish(const void *g, int64_t gs, int64_t d, int32_t n_tiles, uint32_t *pcnt,
                                                             const float *rowmax, const double *rowsum, TernKey K, uint64_t *neg,
                                                             uint64_t *nz, int64_t W, float *scales, int T,
                                                             const uint32_t *gave_up, HeldRow *rows)
{
    __shared__ uint32_t cnt[kWaves], last;
    const int row = blockIdx.y, part = blockIdx.x;
    DevWord *cnt_row = as_shared(pcnt + static_cast<int64_t>(row) * n_tiles);
    const bool late = rows[row].late.load() != 0u;            // uniform: nobody clears it before all have come by here
    if (!late && part != 0) return;
    if (late) {
        uint32_t kept = 0;
        const bool mine = gave_up[row * static_cast<int64_t>(gridDim.x) + part] != 0u;
        if (mine)
            kept = tern_finish_part<BF16>(grad_row<BF16>(g, gs, row), d, part, T, tern_max(rowmax[row]), row, K, neg + row * W, nz + row * W,
                                          static_cast<uint32_t>(W) * 2u);
        kept = tern_kept(kept, cnt);
        if (threadIdx.x == 0) {
            if (mine) cnt_row[part].store(kept);
            // the count is in memory before it is announced
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            last = (rows[row].done.fetch_add(1u) + 1u == gridDim.x) ? 1u : 0u;
        }
        __syncthreads();
        if (last == 0u) return;                               // uniform
    }
    uint32_t kept = 0;
    for (uint32_t p = threadIdx.x; p < gridDim.x; p += kBlock) kept += cnt_row[p].load();
    kept = tern_kept(kept, cnt);                              // not more than d: 32 bits hold it
    if (threadIdx.x != 0) return;
    scales[row] = tern_scale(rowsum[row], kept);
    rows[row].next_call(row == 0);
}

// code * scale of four elements of one message from their bits of the planes
__device__ __forceinline__ f32x4 tern_decode4(uint32_t nz, uint32_t neg, float s)
{
    f32x4 q;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint32_t keep = static_cast<uint32_t>(static_cast<int32_t>(nz << (31 - c)) >> 31);
        q[c] = __uint_as_float((__float_as_uint(s) ^ ((neg << (31 - c)) & 0x80000000u)) & keep);
    }
    return q;
}

// Server that does not compress: a = (1/n) sum_i Q[v_i] by the chain from +0.  The bits of eight messages are asked
// for before the first is used: one message after the other was a chain of memory latencies.  Batches that are not full go
// one by one: with a test of the count before every load the compiler waits for each, and the tests cost more than the
// rest where there are few workers.  Server and update, one by one : eights with tests : as it is, 1 x 2,500,001 5.2 : 6.5 :
// 5.2 us; 9 x 60,000 3.7 : 4.4 : 3.1 us; 8 x 11,173,962 38.0 : 37.3 : 28.1 us; 16 x 11,173,962 59.0 : 57.2 : 36.0 us.
__global__ __launch_bounds__(kBlock) void k_tern_server_identity(const uint64_t *neg, const uint64_t *nz, const float *scales,
                                                                 int n, float inv_n, int64_t d, int64_t W, float *dense_out,
                                                                 ds_update_args u)
{
    const int64_t e = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) * 4;
    if (e >= d) return;
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
    int i = 0;
    for (; i + 8 <= n; i += 8) {
        uint32_t kb[8], nb[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            kb[j] = load_sign_nibble(nz + (i + j) * W, e);
            nb[j] = load_sign_nibble(neg + (i + j) * W, e);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) a = fma4(inv_n, tern_decode4(kb[j], nb[j], scales[i + j]), a);
    }
    for (; i < n; ++i) a = fma4(inv_n, tern_decode4(load_sign_nibble(nz + i * W, e), load_sign_nibble(neg + i * W, e), scales[i]), a);
    put_average4(zero_past(a, e, d), e, d, dense_out, u.x, u.m, u.gamma, u.beta);
}

__global__ __launch_bounds__(kBlock) void k_tern_decode(const uint64_t *neg_row, const uint64_t *nz_row, const float *scale,
                                                        int64_t d, float *out)
{
    const int64_t e = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) * 4;
    if (e >= d) return;
    st4(out, e, d, tern_decode4(load_sign_nibble(nz_row, e), load_sign_nibble(neg_row, e), scale[0]));
}

unsigned blocks4(int64_t d) { return static_cast<unsigned>((d + kBlock * 4 - 1) / (kBlock * 4)); }

}  // namespace

ds_status_t ds_ternary_init(ds_ctx *c)
{
    ds_tern_scratch *t = new (std::nothrow) ds_tern_scratch();
    if (!t) return DS_ERR_DEVICE;
    *t = ds_tern_scratch{};
    c->tern = t;
    const size_t n = static_cast<size_t>(c->cfg.n), tiles = static_cast<size_t>(c->n_tiles);
    DS_HIP_TRY(hipMalloc(&t->pmax, n * tiles * sizeof(float)));
    DS_HIP_TRY(hipMalloc(&t->psum, n * tiles * sizeof(double)));
    DS_HIP_TRY(hipMalloc(&t->pcnt, n * tiles * sizeof(uint32_t)));
    DS_HIP_TRY(hipMalloc(&t->rowmax, n * sizeof(float)));
    DS_HIP_TRY(hipMalloc(&t->rowsum, n * sizeof(double)));
    // GPU time of a worker call, two looks as separate launches against sizes of the held route (two looks are four
    // launches, this route is two, and one for a row that finishes itself or that one workgroup holds, which counts for
    // the host).
    //  * one workgroup, 4 tiles in 4: 5.2 .. 5.5 us (bf16 5.8 .. 6.2), two looks 8.8 .. 10.3 us; one tile per workgroup 5 to 24
    //    tiles 7.8 .. 8.4 us, two looks 9.1 .. 10.6 us;
    //  * one row gains on the host's side only up to 5 M elements: d = 300,001 9.9 us, two looks 9.6 us; 1,000,003 11.4 and
    //    10.6 us; 2,500,001 8 tiles 14.6 us, 13.0 us; 5,000,003 14 tiles 18.0 us, 17.5 us; 11,173,962 14 and 24 tiles 25.8 and
    //    24.7 us, 30.9 us; 20,000,000 37.5 and 35.7 us, 49.5 us;
    //  * n = 8: 300,001 13.4 us, 1, 2 and 4 tiles 19.2, 12.2 and 12.2 us; 1,000,003 22.7 us, 4 and 8 tiles 17.0 and 16.6 us;
    //    2,500,001 44 us, 8, 14 and 24 tiles 34.5, 30.6 and 33.5 us; 5,000,003 80 us, 62, 55 and 59 us;
    //  * rounds of fewer rows, two looks : 14 : 24 tiles, and how much of the device the rounds keep busy with 14 : 24:
    //    8 x 8,000,002 115 : 94 : 91 us (73 : 85 %); 8 x 11,173,962 159 : 153 : 123 us (51 : 89 %); 3 x 9,000,001 56 : 47 : 55 us
    //    (61 : 54 %); 5 x 9,000,001 86 : 73 : 79 us (68 : 60 %); 3 x 11,173,962 67 : 64 : 58 us (51 : 67 %); 8 x 16,000,001
    //    225 : 199 : 214 us (73 : 64 %); 8 x 20,000,000 287 : 236 : 242 us (91 : 79 %); 8 x 24,000,000 24 tiles only, 326 : 265 us;
    //  * bf16 the same, with 24 tiles a little behind: 8 x 8,000,002 120 : 101 : 109 us; 8 x 11,173,962 164 : 171 : 144 us; 5 x
    //    9,000,001 89 : 78 : 93 us; 8 x 20,000,000 285 : 257 : 292 us; 8 x 24,000,000 340 : 304 us.  Rounds of two rows with 8 tiles:
    //    8 x 8,000,002 104 us, 6 x 6,000,000 62 us (two looks 72 us);
    //  * below: a step at 13 M elements with 24 tiles, 52 % busy, two rows 87 us (bf16 97), two looks 85 us (87); one row of
    //    8,000,001, 36 % busy with 14 tiles, 43.1 us (45.6), 42.6 us (42.3).
    static constexpr HeldStep one_row[8] = {{1, 0, 64}, {2, 0, 128}, {4, 0, 256}, {14, 1, 0, 50}, {24, 1, 0, 50}};
    static constexpr HeldStep f32[8] = {{1, 0, 64}, {2, 0, 128}, {4, 0, 256}, {8, 0, 0}, {14, 4, 0}, {24, 1, 0, 85}, {14, 1, 0, 58}, {24, 1, 0, 65}};
    static constexpr HeldStep bf16[8] = {{1, 0, 64}, {2, 0, 128}, {4, 0, 256}, {8, 0, 0}, {14, 4, 0}, {8, 2, 0, 70}, {14, 1, 0, 58}, {24, 1, 0, 65}};
    const auto &steps = c->cfg.n == 1 ? one_row : c->cfg.grad_dtype == DS_BF16 ? bf16 : f32;
    const ds_status_t rc = held_size(c, c->cfg.n, 4, steps, [](auto r, auto l) {
        constexpr int R = decltype(r)::value, L = decltype(l)::value;
        int per_cu = 0;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_tern_held<false, R, L>, kBlock, 0) == hipSuccess ? per_cu : -1;
    }, &t->held);
    if (rc != DS_OK) return rc;
    return t->held.T ? held_alloc(c, c->cfg.n, &t->held) : DS_OK;
}

void ds_ternary_fini(ds_ctx *c)
{
    ds_tern_scratch *t = c->tern;
    if (!t) return;
    void *ptrs[5] = {t->pmax, t->psum, t->pcnt, t->rowmax, t->rowsum};
    for (void *p : ptrs)
        if (p) (void)hipFree(p);
    held_free(&t->held);
    delete t;
    c->tern = nullptr;
}

ds_status_t ds_ternary_worker(ds_ctx *c, uint64_t step, const void *g, int64_t gs, const ds_payload_t *out, hipStream_t st)
{
    ds_tern_scratch *t = c->tern;
    const int64_t d = c->cfg.d, n_tiles = c->n_tiles;
    const unsigned n = static_cast<unsigned>(c->cfg.n);
    const dim3 grid(static_cast<unsigned>(n_tiles), n);
    const uint32_t key0 = static_cast<uint32_t>(c->cfg.seed);
    const uint32_t key1 = static_cast<uint32_t>(c->cfg.seed >> 32) ^ static_cast<uint32_t>(step >> 32);
    uint64_t *nz = reinterpret_cast<uint64_t *>(out->levels);
    const bool bf16 = c->cfg.grad_dtype == DS_BF16;
    if (t->held.T) {
        const ds_held_sync &h = t->held;
        HeldRow *rows = static_cast<HeldRow *>(h.rows);
        const TernKey K{key0, key1, static_cast<uint32_t>(step)};
        const dim3 hgrid(static_cast<unsigned>(h.parts), n);
        auto go = [&](auto bf) {
            constexpr bool BF = decltype(bf)::value;
            with_held(h.T, [&](auto rr, auto ll) {
                constexpr int R = decltype(rr)::value, L = decltype(ll)::value;
                k_tern_held<BF, R, L><<<hgrid, kBlock, 0, st>>>(g, gs, d, static_cast<int32_t>(n_tiles), t->psum, t->pmax, t->pcnt, t->rowmax,
                                                                t->rowsum, K,
                                                                out->sign_words, nz, c->W, out->scales, rows, h.gave_up, h.patience, h.self);
            });
            if (h.parts > 1 && !h.self)
                k_tern_held_finish<BF><<<hgrid, kBlock, 0, st>>>(g, gs, d, static_cast<int32_t>(n_tiles), t->pcnt, t->rowmax, t->rowsum, K,
                                                                 out->sign_words, nz, c->W, out->scales, h.T, h.gave_up, rows);
        };
        if (bf16) go(std::true_type{}); else go(std::false_type{});
        return ds_launch_status();
    }
    if (bf16) k_tern_stats<true><<<grid, kBlock, 0, st>>>(g, gs, d, t->pmax, t->psum);
    else k_tern_stats<false><<<grid, kBlock, 0, st>>>(g, gs, d, t->pmax, t->psum);
    k_tern_rowstat<<<n, kBlock, 0, st>>>(t->pmax, t->psum, n_tiles, t->rowmax, t->rowsum);
    if (bf16)
        k_tern_encode<true><<<grid, kBlock, 0, st>>>(g, gs, d, t->rowmax, key0, key1, static_cast<uint32_t>(step),
                                                     out->sign_words, nz, c->W, t->pcnt);
    else
        k_tern_encode<false><<<grid, kBlock, 0, st>>>(g, gs, d, t->rowmax, key0, key1, static_cast<uint32_t>(step),
                                                      out->sign_words, nz, c->W, t->pcnt);
    k_tern_scale<<<n, kBlock, 0, st>>>(t->pcnt, t->rowsum, n_tiles, out->scales);
    return ds_launch_status();
}

ds_status_t ds_ternary_server_identity(ds_ctx *c, const ds_payload_t *in, float *dense_out, ds_update_args u, hipStream_t st)
{
    k_tern_server_identity<<<blocks4(c->cfg.d), kBlock, 0, st>>>(in->sign_words, reinterpret_cast<const uint64_t *>(in->levels),
                                                                in->scales, c->cfg.n, c->inv_n, c->cfg.d, c->W, dense_out, u);
    return ds_launch_status();
}

ds_status_t ds_ternary_decode(ds_ctx *c, const ds_payload_t *p, int32_t row, float *out, hipStream_t st)
{
    k_tern_decode<<<blocks4(c->cfg.d), kBlock, 0, st>>>(p->sign_words + row * c->W,
                                                       reinterpret_cast<const uint64_t *>(p->levels) + row * c->W,
                                                       p->scales + row, c->cfg.d, out);
    return ds_launch_status();
}
