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

// Codes of the four elements of group `quad` of the row (elements 4 quad ..), of which `left` (at most 4) belong
// to it: bit c = code is not 0, bit 4 + c = code is -1.  The encoding is bound by
// vector instructions, and four IEEE divisions were a third of them.  With U = 2^24 u a whole
// number and q = |v| * fl(2^24 / m), which is within 2^-22 of 2^24 fl(|v| / m), U outside
// q (1 -+ 2^-20) (and, for U = 0, q above 2^-20) decides u < fl(|v| / m) without the quotient; what
// lies inside, NaN included, and rows whose maximum leaves the range of that product divide.
__device__ __forceinline__ uint32_t tern_codes4(f32x4 v, float m, uint32_t quad, int left, int row, TernKey K)
{
    const u32x4 rnd = philox4x32_10(u32x4{quad, 0u, static_cast<uint32_t>(row), K.step_lo}, K.key0, K.key1);
    const float vv[4] = {v.x, v.y, v.z, v.w};
    const uint32_t rr[4] = {rnd.x, rnd.y, rnd.z, rnd.w};
    const bool in_range = m >= 0x1p-100f && m <= 0x1p100f;      // uniform
    const float r = __fdiv_rn(0x1p24f, m);
    uint32_t nz = 0u, open = 0u;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float U = static_cast<float>(rr[c] >> 8), q = fabsf(vv[c]) * r;
        const bool below = U < __fmaf_rn(q, 1.f - 0x1p-20f, -0x1p-20f), above = U > q * (1.f + 0x1p-20f);
        nz |= below ? 1u << c : 0u;
        open |= (below || above) ? 0u : 1u << c;
    }
    if (!in_range) { nz = 0u; open = (m > 0.f) ? 15u : 0u; }
    if (open) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bool keep = static_cast<float>(rr[c] >> 8) * 0x1p-24f < __fdiv_rn(fabsf(vv[c]), m);
            nz |= ((open >> c) & 1u) && keep ? 1u << c : 0u;
        }
    }
    nz &= (left >= 4) ? 15u : (left > 0) ? (1u << left) - 1u : 0u;
    const uint32_t neg = (vv[0] < 0.f ? 1u : 0u) | (vv[1] < 0.f ? 2u : 0u) | (vv[2] < 0.f ? 4u : 0u) | (vv[3] < 0.f ? 8u : 0u);
    return nz | ((nz & neg) << 4);
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
    const float m = rowmax[row];
    const uint32_t code = tern_codes4(v, m, static_cast<uint32_t>(e >> 2), static_cast<int>(d - e), row, TernKey{key0, key1, step_lo});
    stash_sign_words(sw_nz, wave_nibble_word(code & 15u));
    stash_sign_words(sw_neg, wave_nibble_word(code >> 4));
    const uint32_t kept = wave_sum_u32(static_cast<uint32_t>(__popc(code & 15u)));
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
// What bounds it is the encoding: vector instructions, most of them Philox.  Worker call at
// 8 x 11,173,962: 189 us in two looks with four divisions per thread, 164 us in two looks without
// them, 149 .. 154 us here with the finish launch (57 us for its bytes at the copy kernel's rate).
__device__ __forceinline__ float tern_scale(double sum, uint32_t kept)
{
    return kept ? static_cast<float>(sum / static_cast<double>(kept)) : 0.f;
}

template <int T>
struct TernShared {
    double sums[T][kWaves], red[kWaves];
    float mx[kWaves];
    uint32_t cnt[kWaves], sh[2];
};

// The wavefront's words of one tile to both planes: word of an 8-lane group, by its first lane.  Rows have
// fewer than 2^31 elements and a stretch reaches less than 2^31 past their end: 32 bits number the groups of
// four and their bits.
__device__ __forceinline__ void tern_put_words(uint32_t code, uint32_t quad, uint64_t *neg_row, uint64_t *nz_row, uint32_t words)
{
    const uint32_t a = wave_nibble_word(code & 15u), b = wave_nibble_word(code >> 4), w = quad >> 3;
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
__device__ __forceinline__ uint32_t tern_finish_part(const void *grow, int64_t d, int part, int T, float m, int row, TernKey K,
                                                     uint64_t *neg_row, uint64_t *nz_row, uint32_t words)
{
    uint32_t kept = 0;
    f32x4 next = ld4_grad<BF16>(grow, static_cast<int64_t>(part) * T * kTile + threadIdx.x * 4, d);
    for (int t = 0; t < T; ++t) {
        const int64_t e = (static_cast<int64_t>(part) * T + t) * kTile + threadIdx.x * 4;
        const uint32_t quad = static_cast<uint32_t>(e >> 2);
        const f32x4 v = next;
        if (t + 1 < T) next = ld4_grad<BF16>(grow, e + kTile, d);       // zero past the end of the row
        const uint32_t code = tern_codes4(v, m, quad, static_cast<int>(d - e), row, K);
        tern_put_words(code, quad, neg_row, nz_row, words);
        kept += __popc(code & 15u);
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
    __shared__ TernShared<T> sm;
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
        const double s = wave_sum(((static_cast<double>(a0) + static_cast<double>(a1)) + static_cast<double>(a2)) + static_cast<double>(a3));
        if (lane_id() == 0) sm.sums[t][wave_id()] = s;
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    if (lane_id() == 0) sm.mx[wave_id()] = mx;
    held_fence(v, left);
    __syncthreads();
    double tile_sum = 0.0;                                    // lane t < T of every wavefront: tile t
    if (lane_id() < T) {
        tile_sum = sm.sums[lane_id()][0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) tile_sum += sm.sums[lane_id()][w];
    }
#pragma unroll
    for (int w = 0; w < kWaves; ++w) mx = fmaxf(mx, sm.mx[w]);
    const bool alone = gridDim.x == 1;
    double row_sum_alone = 0.0;
    bool ok = true;
    if (alone) {
        row_sum_alone = wave_sum(tile_sum);
    } else {
        uint64_t *psum_row = reinterpret_cast<uint64_t *>(psum) + static_cast<int64_t>(row) * n_tiles;
        uint32_t *pmax_row = reinterpret_cast<uint32_t *>(pmax) + static_cast<int64_t>(row) * n_tiles;   // one per workgroup
        if (wave_id() == 0) {
            if (lane_id() < T && tile0 + lane_id() < n_tiles)
                as_shared(psum_row)[tile0 + lane_id()].store(__double_as_longlong(tile_sum));
            if (lane_id() == 0) as_shared(pmax_row)[blockIdx.x].store(__float_as_uint(mx));
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
            for (int32_t p = threadIdx.x; p < n_tiles; p += kBlock)
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
    auto encode = [&](f32x4 w, int t) {
        const uint32_t quad = quad0 + t * (kTile / 4);
        const uint32_t code = tern_codes4(w, mx, quad, left - t * kTile - static_cast<int>(threadIdx.x) * 4, row, K);
        tern_put_words(code, quad, neg_row, nz_row, words);
        kept += __popc(code & 15u);
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
                        more += tern_finish_part<BF16>(grow, d, static_cast<int>(p), T, m, row, K, neg_row, nz_row, words);
                __syncthreads();                              // sm.cnt is used again
                all += tern_kept(more, sm.cnt);
            }
            if (threadIdx.x != 0) return;
            scales[row] = tern_scale(__longlong_as_double(static_cast<long long>(as_shared(reinterpret_cast<uint64_t *>(rowsum))[row].load())), all);
            rows[row].next_call(row == 0);
            return;
        }
    if (threadIdx.x != 0) return;
    if (alone) scales[row] = tern_scale(row_sum_alone, kept);
    else pcnt[static_cast<int64_t>(row) * n_tiles + blockIdx.x] = kept;    // added up by the finish launch
}

// After a held launch: writes the scale of every row from the counts of its workgroups and readies the
// synchronisation words for the next call.  In a row in which a workgroup gave up (normally none) one
// workgroup for each of them encodes what it held, and the one that is through last adds up.
// 8 x 11,173,962 with all waits given up: 172 us, 1259 us with one finishing workgroup for 64 of
// the held launch.
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
            kept = tern_finish_part<BF16>(grad_row<BF16>(g, gs, row), d, part, T, rowmax[row], row, K, neg + row * W, nz + row * W,
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

// code * scale of elements e..e+3 of one message
__device__ __forceinline__ f32x4 tern_decode4(const uint64_t *neg_row, const uint64_t *nz_row, float s, int64_t e)
{
    const uint32_t kb = load_sign_nibble(nz_row, e), nb = load_sign_nibble(neg_row, e);
    f32x4 q;
    q.x = (kb & 1u) ? ((nb & 1u) ? -s : s) : 0.f;
    q.y = (kb & 2u) ? ((nb & 2u) ? -s : s) : 0.f;
    q.z = (kb & 4u) ? ((nb & 4u) ? -s : s) : 0.f;
    q.w = (kb & 8u) ? ((nb & 8u) ? -s : s) : 0.f;
    return q;
}

// Server that does not compress: a = (1/n) sum_i Q[v_i] by the chain from +0.
__global__ __launch_bounds__(kBlock) void k_tern_server_identity(const uint64_t *neg, const uint64_t *nz, const float *scales,
                                                                 int n, float inv_n, int64_t d, int64_t W, float *dense_out,
                                                                 ds_update_args u)
{
    const int64_t e = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) * 4;
    if (e >= d) return;
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
    for (int i = 0; i < n; ++i) a = fma4(inv_n, tern_decode4(neg + i * W, nz + i * W, scales[i], e), a);
    put_average4(zero_past(a, e, d), e, d, dense_out, u.x, u.m, u.gamma, u.beta);
}

__global__ __launch_bounds__(kBlock) void k_tern_decode(const uint64_t *neg_row, const uint64_t *nz_row, const float *scale,
                                                        int64_t d, float *out)
{
    const int64_t e = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) * 4;
    if (e >= d) return;
    st4(out, e, d, tern_decode4(neg_row, nz_row, scale[0], e));
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
    // GPU time of a worker call, two looks as separate launches against sizes of the held route.  In a stream of
    // calls the four launches of two looks also cost the host 17 us, the two of this route 12 us, and the one of a
    // row that finishes itself or that one workgroup holds 10 us.
    //  * one workgroup, 4 tiles in 4: 5.2 .. 5.5 us (bf16 5.8 .. 6.2), two looks 8.8 .. 10.3 us; 8 tiles in 8: 7.8 .. 8.1 us (bf16
    //    8.9 .. 9.4), 8.9 .. 10.6 us; 12 tiles in 14: 11.5 .. 11.9 us (bf16 13.1 .. 13.5), 9.0 .. 10.6 us; one tile per workgroup
    //    5 to 24 tiles 7.7 .. 8.6 us;
    //  * one row gains on the host's side only: d = 300,001 9.1 us, with 2 tiles 10.1 us; 1,000,003 10.1 us, with 1, 2, 4
    //    and 8 tiles 16.0, 12.9, 12.1 and 13.7 us; 2,500,001 13.3 us, with 4 and 8 tiles 16.6 and 16.2 us;
    //  * n = 8: 300,001 13.1 us, 1, 2 and 4 tiles 18.7, 12.2 and 12.7 us; 1,000,003 23.3 us, 4 and 8 tiles 18.0 and 17.9 us;
    //    2,500,001 44 us, 8, 14 and 24 tiles 39, 35 and 37 us; 5,000,003 78, 69, 63 and 69 us;
    //  * 8,000,002, two and more rows on chip: n = 8 121 us, 8 and 24 tiles 113 and 109 us; bf16 125, 119 and 133 us;
    //    8 x 11,173,962 164 us, 24 tiles (two rows) 149 us, 8 tiles (a row and a half) 197 us; bf16 171 and 173 us;
    //    8 x 16,000,001, not two rows with any size: 231 us, 24 tiles 273 us;
    //  * rounds of two rows, n = 3 .. 16, two looks : held by how much of the device the rounds keep busy.  24 tiles: 0.87 at 54 %
    //    (3 x 9,000,001, 57.6 and 66.3 us), 0.91 .. 0.98 at 60 .. 68 %, 0.98 .. 1.04 at 70 .. 75 %, 1.05 .. 1.14 above.  8 tiles of
    //    bf16: 0.91 .. 0.98 at 60 .. 70 %, 0.98 .. 1.01 at 72 .. 80 %, 1.00 .. 1.06 above.
    static constexpr HeldStep one_row[] = {{1, 0, 64}, {2, 0, 128}, {4, 0, 256}, {0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
    static constexpr HeldStep f32[] = {{1, 0, 64}, {2, 0, 128}, {4, 0, 256}, {8, 0, 0}, {14, 4, 0}, {24, 2, 0, 70}};
    static constexpr HeldStep bf16[] = {{1, 0, 64}, {2, 0, 128}, {4, 0, 256}, {8, 0, 0}, {14, 4, 0}, {8, 2, 0, 80}};
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
