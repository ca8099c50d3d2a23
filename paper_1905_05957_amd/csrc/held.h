// Held route: kernels that need one value per row (a scale, a maximum) before they can finish its
// elements keep a row in registers and LDS across the workgroups of one launch instead of
// reading it twice.  Shared pieces: the synchronisation words and the bounded wait, the addressing
// of the held tiles, and the choice of how many tiles a workgroup holds.
#pragma once
#include "ds_device.h"
#include "ds_internal.h"

#include <type_traits>

namespace ds {

// Synchronisation words of one row; published word and counter on cache lines of their own.
constexpr size_t kHeldRowBytes = 256;
// A wait that was not answered in time (part of a row had no room beside another stream's workgroups) ends
// all waits of its call, and nobody waits in the next one either.  If the wait after that is in vain
// too, two calls go by without one, then four, up to kHeldShy, until a call has all its waits answered:
// the price of waiting in vain is not paid over and over, and a single late call is soon forgotten.
// 1-bit worker block at 8 x 11,173,962 with a matrix product running on another stream: 323 .. 338 us a call,
// 478 .. 496 us when every late call was followed by kHeldShy calls without a wait.
constexpr uint32_t kHeldShy = 256, kHeldLate = ~0u;
struct HeldRow {
    DevShared<uint64_t> pub;      // kHeldValue | bits of the row's value, 0 = not there yet
    DevShared<uint32_t> quit;     // row 0 only: nobody waits in this call: kHeldLate, or calls left for which that holds
    uint32_t span;                // row 0 only: calls without a wait after the last late one
    uint32_t pad0[28];
    DevShared<uint32_t> arrived;
    DevShared<uint32_t> late;     // a workgroup of the row gave up (ternary, and rows that finish themselves)
    DevShared<uint32_t> done;     // ternary: workgroups of the finish launch that are through with the row
    uint32_t pad1;
    DevShared<uint64_t> departed; // rows that finish themselves: workgroups << 40 | what they counted
    uint32_t pad2[26];

    // in the finish launch or by the last workgroup of the row, by one thread per row
    __device__ __forceinline__ void next_call(bool first_row)
    {
        pub.clear_for_next_launch();
        arrived.clear_for_next_launch();
        late.clear_for_next_launch();
        done.clear_for_next_launch();
        departed.clear_for_next_launch();
        if (!first_row) return;
        const uint32_t q = quit.load();
        if (q == kHeldLate) {
            span = (span == 0u) ? 1u : (span < kHeldShy) ? 2u * span : kHeldShy;
            quit.store(span);
        } else if (q != 0u) {
            quit.store(q - 1u);
        } else {
            span = 0u;
        }
    }
};
static_assert(sizeof(HeldRow) == kHeldRowBytes, "as allocated by the host");
constexpr uint64_t kHeldValue = 1ull << 32;

// The row's published value, false if it did not come in time.  Every thread of the workgroup calls.
__device__ __forceinline__ bool held_wait(HeldRow *rows, int row, uint32_t patience, uint32_t *sh, float *s)
{
    if (threadIdx.x == 0) {
        const long long t0 = wall_clock64();
        uint64_t v;
        for (uint32_t polls = 0;; ++polls) {
            v = rows[row].pub.load();
            if (v & kHeldValue) break;
            if ((polls & 7u) == 0u) {
                if (rows[0].quit.load() != 0u) break;
                if (wall_clock64() - t0 >= static_cast<long long>(patience)) { rows[0].quit.store(kHeldLate); break; }
            }
            __builtin_amdgcn_s_sleep(8);
        }
        sh[0] = (v & kHeldValue) ? 1u : 0u;
        sh[1] = static_cast<uint32_t>(v);
    }
    __syncthreads();
    *s = __uint_as_float(sh[1]);
    return sh[0] != 0u;
}

// Rows of few tiles finish themselves: the workgroup that departs last does what the finish launch does for longer
// rows (which would leave it too much in a late call).  It saves a launch, 2 to 3 us of the host's time for a call and
// about as much of the device's: server and update at n = 8 and 24 tiles 7.1 us, 11 us a call in a stream of calls (7.4 and 13.4
// us with a finish launch).  A call in which all waits are given up takes 33 us then, the worker block's 67 us
// (two looks 8 us), but with at most 32 workgroups a row finds room, and the wait may be long.
constexpr int kHeldSelfTiles = 32;
template <int R, int L>
constexpr bool kHeldSelf = L == 0 && R <= 2;       // the sizes that such rows take

// Departure of a workgroup that adds `count`; true in the last one, with the sum of all counts.  Every thread
// calls.  What a workgroup that gave up has stored is in memory for the others before it departs.
__device__ __forceinline__ bool held_depart(HeldRow *row, uint32_t parts, bool ok, uint32_t count, uint32_t *sh, uint32_t *sum)
{
    if (!ok) __threadfence();                                  // uniform
    __syncthreads();
    if (threadIdx.x == 0) {
        if (!ok) row->late.store(1u);
        // the published value, the sum and the flags too
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const uint64_t all = row->departed.fetch_add((1ull << 40) | count) + ((1ull << 40) | count);
        sh[0] = (all >> 40) == parts ? 1u : 0u;
        sh[1] = static_cast<uint32_t>(all);
    }
    __syncthreads();
    *sum = sh[1];
    return sh[0] != 0u;
}

// Tile t of a workgroup's stretch of an fp32 row as a buffer: a descriptor in scalar registers and
// one 32-bit offset per lane, the same for every tile, where 64-bit addresses would take the
// registers that v needs.  Only the whole groups of four elements of the row lie inside the
// buffer: a lane past them reads zero and stores nothing, and the one to three elements of a
// last cut group are the caller's.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t held_tile(const float *first, int left, int t)
{
    const int whole = (left & ~3) - t * kTile;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(first + t * kTile), 0, (whole > 0 ? whole : 0) * 4, 0x00027000);
}

constexpr int kNonTemporal = 2;   // cache policy operand of the buffer instructions

template <int POLICY = kNonTemporal>
__device__ __forceinline__ f32x4 held_ld4(const float *first, int left, int t)
{
    const u32x4 u = __builtin_amdgcn_raw_buffer_load_b128(held_tile(first, left, t), static_cast<int>(threadIdx.x) * 16, 0, POLICY);
    return f32x4{__uint_as_float(u.x), __uint_as_float(u.y), __uint_as_float(u.z), __uint_as_float(u.w)};
}

template <int POLICY = kNonTemporal>
__device__ __forceinline__ void held_st4(float *first, int left, int t, f32x4 v)
{
    const u32x4 u = {__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)};
    __builtin_amdgcn_raw_buffer_store_b128(u, held_tile(first, left, t), static_cast<int>(threadIdx.x) * 16, 0, POLICY);
}

// Four gradients of tile t, zero past the row's last whole group of four.
template <bool BF16>
__device__ __forceinline__ f32x4 held_g4(const void *grow, int64_t first, int left, int t)
{
    if constexpr (BF16) return ld4_bf16(static_cast<const uint16_t *>(grow), first + t * kTile + threadIdx.x * 4, first + (left & ~3));
    else return held_ld4(static_cast<const float *>(grow) + first, left, t);
}

// Between the phases of a held kernel: the compiler must not carry what it derived from v in one
// phase (sign masks, addresses) into the next in registers that v itself needs.
template <int T>
__device__ __forceinline__ void held_fence(f32x4 (&v)[T], int &left)
{
    asm volatile("" : "+s"(left));
#pragma unroll
    for (int t = 0; t < T; ++t) asm volatile("" : "+v"(v[t]));
}

// Elements of the row from the first one of the workgroup on, as far as they matter to it.
template <int T>
__device__ __forceinline__ int held_left(int64_t tile0, int64_t d)
{
    const int64_t left = d - tile0 * kTile;
    return left < T * kTile ? static_cast<int>(left) : T * kTile;
}

// f(0), f(1), ... with the index as a compile-time constant
template <int A, int B, class F>
__device__ __forceinline__ void static_for(F f)
{
    if constexpr (A < B) {
        f(std::integral_constant<int, A>{});
        static_for<A + 1, B>(f);
    }
}

// wavefronts per SIMD that the register count of a kernel holding R tiles in registers allows
constexpr int held_waves(int R) { return R <= 4 ? 8 : R <= 8 ? 6 : 4; }

// The built sizes: calls f with the tiles that a workgroup keeps in registers and in LDS as
// compile-time constants.  512 threads with up to 64, 80 and 128 registers leave room for 4, 3
// and 2 workgroups per compute unit, and the LDS tiles fill that number's share of 160 KB.
constexpr int kHeldT[] = {1, 2, 4, 8, 14, 24};

template <class F>
static void with_held(int T, F f)
{
    using std::integral_constant;
    switch (T) {
    case 1: f(integral_constant<int, 1>{}, integral_constant<int, 0>{}); break;
    case 2: f(integral_constant<int, 2>{}, integral_constant<int, 0>{}); break;
    case 4: f(integral_constant<int, 4>{}, integral_constant<int, 0>{}); break;
    case 8: f(integral_constant<int, 4>{}, integral_constant<int, 4>{}); break;
    case 14: f(integral_constant<int, 8>{}, integral_constant<int, 6>{}); break;
    case 24: f(integral_constant<int, 15>{}, integral_constant<int, 9>{}); break;
    }
}

// One line of a kernel's choice of size: `T` tiles per workgroup if the device holds `rows` rows at once
// (all, if they are fewer or 0 stands here), a row is not more than `parts` workgroups (0: any number) and
// rounds of whole rows keep at least `full` per cent of the device's workgroups busy.
struct HeldStep {
    int T, rows, parts, full = 0;
};

// Tiles per workgroup for `rows` rows, 0 = the kernel's way in separate launches; per_cu(R, L): resident
// workgroups of that kernel per compute unit, negative on failure.  A row of at most `one` tiles is left to
// one workgroup, of the smallest size that holds it: nobody waits and the finish launch falls away, but
// the tiles come one after the other, and a size pays for all the tiles that it is built for.  For
// longer rows the first step that holds is taken.  What speaks for a size:
//  * more workgroups have more loads in flight, and a row that is on chip as a whole does not wait for
//    room: the smallest size with which all rows are there at once, or else a few rows, so that one row's loads
//    overlap another's barrier and stores;
//  * the arrivals of a row's workgroups are additions to one word, which come one after the other (11 ns
//    each), so short rows take fewer workgroups than the device would hold;
//  * rows that are not all there at once go in rounds: what the last round leaves free, and the room that one more row
//    would not fit into, is idle.
// The lines lie where the kernels were measured to cross over; the figures stand with each kernel's steps.
template <class F, int N>
static ds_status_t held_size(const ds_ctx *c, int64_t rows, int one, const HeldStep (&steps)[N], F per_cu, ds_held_sync *sync)
{
    int cus = 0;
    DS_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device));
    const int64_t tiles = c->n_tiles;
    sync->T = 0;
    auto take = [&](int T, int64_t at_once, int64_t most, int full) {
        int held = 0;
        with_held(T, [&](auto r, auto l) { held = per_cu(r, l); });
        if (held < 0) return DS_ERR_DEVICE;
        const int64_t slots = static_cast<int64_t>(held) * cus, parts = (tiles + T - 1) / T;
        if (at_once * parts > slots || parts > most) return DS_OK;
        const int64_t together = slots / parts, rounds = (rows + together - 1) / together;
        if (100 * rows * parts >= full * rounds * slots) { sync->T = T; sync->slots = slots; }
        return DS_OK;
    };
    if (tiles <= one) {
        for (int T : kHeldT)
            if (tiles <= T) return take(T, 1, 1, 0);
    }
    for (const HeldStep &s : steps) {
        if (s.T == 0) break;
        const ds_status_t rc = take(s.T, (s.rows && s.rows < rows) ? s.rows : rows, s.parts ? s.parts : tiles, s.full);
        if (rc != DS_OK || sync->T) return rc;
    }
    return DS_OK;
}

// The synchronisation words and flags of a context that takes the route with `sync->T` tiles.
static ds_status_t held_alloc(const ds_ctx *c, int32_t rows, ds_held_sync *sync)
{
    const size_t n = static_cast<size_t>(rows);
    sync->parts = static_cast<int>((c->n_tiles + sync->T - 1) / sync->T);
    // A wait, in ticks of the 100 MHz clock: 20 us, and 10 ps (eight bytes at 0.8 TB/s) for every element of
    // the rows that are loaded at the same time, which share the bandwidth: those that the device
    // holds and the one whose workgroups come in as others leave.
    // Rows that finish themselves keep few workgroups from anything else and wait up to 2 ms.
    sync->self = sync->parts > 1 && sync->T <= 2 && c->n_tiles <= kHeldSelfTiles;
    const int64_t together = sync->slots / sync->parts + 1;
    sync->patience = (c->cfg.topk_spin_limit < 0) ? 0u : sync->self ? 200000u :
                     static_cast<uint32_t>(2000 + (rows < together ? rows : together) * c->cfg.d / 1000);
    DS_HIP_TRY(hipMalloc(&sync->rows, kHeldRowBytes * n + sizeof(uint32_t) * n * static_cast<size_t>(sync->parts)));
    DS_HIP_TRY(hipMemset(sync->rows, 0, kHeldRowBytes * n));
    sync->gave_up = reinterpret_cast<uint32_t *>(static_cast<char *>(sync->rows) + kHeldRowBytes * n);
    return DS_OK;
}

static void held_free(ds_held_sync *sync)
{
    if (sync->rows) (void)hipFree(sync->rows);
    *sync = ds_held_sync{};
}

}  // namespace ds
