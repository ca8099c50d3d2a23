// Clipping compressor (Section 3.2 "Clipping" of the DoubleSqueeze paper): the lower b bits
// of every number's binary representation are set to zero.  The message keeps the upper 32-b
// bits of every element in the smallest of 1, 2 or 4 bytes that holds them (b >= 24,
// b >= 16, otherwise), little endian; b = 16 is the truncation of fp32 to the bf16 grid.
// The error v - Q[v] is the value of the cleared bits and is exact in fp32.
//
// Everything is element-wise, so each of the three calls is one streaming pass with one
// 128-bit load per thread and input stream; the message leaves as one 4*NB-byte store per
// thread.
#include "ds_device.h"
#include "ds_internal.h"

#include <type_traits>

using namespace ds;

namespace {

// Message rows of an odd length start at any byte: the four elements of a thread are one access
// of 4 * NB bytes all the same (global accesses need no alignment).
typedef uint32_t u32_byte __attribute__((aligned(1)));
typedef uint32_t u32x2_byte __attribute__((ext_vector_type(2), aligned(1)));
typedef uint32_t u32x4_byte __attribute__((ext_vector_type(4), aligned(1)));

template <int NB>
__device__ __forceinline__ void store_msg4(uint8_t *__restrict__ row, int64_t e, int64_t d, const uint32_t top[4])
{
    uint8_t *p = row + e * NB;
    if (e + 4 <= d) {
        if constexpr (NB == 1) {
            *reinterpret_cast<u32_byte *>(p) = top[0] | (top[1] << 8) | (top[2] << 16) | (top[3] << 24);
        } else if constexpr (NB == 2) {
            *reinterpret_cast<u32x2_byte *>(p) = u32x2{top[0] | (top[1] << 16), top[2] | (top[3] << 16)};
        } else {
            *reinterpret_cast<u32x4_byte *>(p) = u32x4{top[0], top[1], top[2], top[3]};
        }
        return;
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        if (e + c >= d) break;
        if constexpr (NB == 1) p[c] = static_cast<uint8_t>(top[c]);
        else if constexpr (NB == 2) {
            p[2 * c] = static_cast<uint8_t>(top[c]);
            p[2 * c + 1] = static_cast<uint8_t>(top[c] >> 8);
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) p[4 * c + t] = static_cast<uint8_t>(top[c] >> (8 * t));
        }
    }
}

// Four elements of a message as they are stored, and decoded.  Apart, so that loads of several messages can be in
// flight before the first is decoded.
template <int NB>
struct ClipRaw {
    uint32_t w[NB];
};

template <int NB>
__device__ __forceinline__ ClipRaw<NB> load_raw4(const uint8_t *p)
{
    if constexpr (NB == 1) return {{*reinterpret_cast<const u32_byte *>(p)}};
    else if constexpr (NB == 2) {
        const u32x2 w = *reinterpret_cast<const u32x2_byte *>(p);
        return {{w.x, w.y}};
    } else {
        const u32x4 w = *reinterpret_cast<const u32x4_byte *>(p);
        return {{w.x, w.y, w.z, w.w}};
    }
}

template <int NB>
__device__ __forceinline__ f32x4 decode_raw4(const ClipRaw<NB> &r)
{
    uint32_t u[4];
    if constexpr (NB == 1) { u[0] = r.w[0] << 24; u[1] = (r.w[0] << 16) & 0xFF000000u; u[2] = (r.w[0] << 8) & 0xFF000000u; u[3] = r.w[0] & 0xFF000000u; }
    else if constexpr (NB == 2) { u[0] = r.w[0] << 16; u[1] = r.w[0] & 0xFFFF0000u; u[2] = r.w[1] << 16; u[3] = r.w[1] & 0xFFFF0000u; }
    else { u[0] = r.w[0]; u[1] = r.w[1]; u[2] = r.w[2]; u[3] = r.w[3]; }
    return f32x4{__uint_as_float(u[0]), __uint_as_float(u[1]), __uint_as_float(u[2]), __uint_as_float(u[3])};
}

// decoded values of four elements; elements past d decode to 0
template <int NB>
__device__ __forceinline__ f32x4 load_msg4(const uint8_t *__restrict__ row, int64_t e, int64_t d)
{
    const uint8_t *p = row + e * NB;
    if (e + 4 <= d) return decode_raw4<NB>(load_raw4<NB>(p));
    uint32_t top[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        if (e + c >= d) break;
#pragma unroll
        for (int t = 0; t < NB; ++t) top[c] |= static_cast<uint32_t>(p[NB * c + t]) << (8 * t);
    }
    constexpr int sh = 32 - 8 * NB;
    return f32x4{__uint_as_float(top[0] << sh), __uint_as_float(top[1] << sh), __uint_as_float(top[2] << sh),
                 __uint_as_float(top[3] << sh)};
}

// Q[v], which it returns, the message and the error for the four elements of a thread
template <int NB>
__device__ __forceinline__ f32x4 clip_store4(f32x4 v, uint32_t mask, int64_t e, int64_t d, uint8_t *__restrict__ msg_row,
                                            float *__restrict__ err_row)
{
    const uint32_t u[4] = {__float_as_uint(v.x) & mask, __float_as_uint(v.y) & mask, __float_as_uint(v.z) & mask,
                           __float_as_uint(v.w) & mask};
    constexpr int sh = 32 - 8 * NB;
    const uint32_t top[4] = {u[0] >> sh, u[1] >> sh, u[2] >> sh, u[3] >> sh};
    store_msg4<NB>(msg_row, e, d, top);
    const f32x4 q = {__uint_as_float(u[0]), __uint_as_float(u[1]), __uint_as_float(u[2]), __uint_as_float(u[3])};
    if (err_row) st4_stream(err_row, e, d, v - q);     // no buffer: no compensation
    return q;
}

// Algorithm 1, worker block: v = g + delta ; message = Q[v] ; delta <- v - Q[v].
template <bool BF16, int NB>
__global__ __launch_bounds__(kBlock) void k_clip_worker(const void *g, int64_t gs, float *delta, int64_t dstr,
                                                        uint8_t *msg, int64_t d, uint32_t mask)
{
    const int row = blockIdx.y;
    const int64_t e = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) * 4;
    if (e >= d) return;
    const void *grow = BF16 ? static_cast<const void *>(static_cast<const uint16_t *>(g) + row * gs)
                            : static_cast<const void *>(static_cast<const float *>(g) + row * gs);
    float *drow = delta ? delta + row * dstr : nullptr;         // null: no compensation, v = g
    f32x4 v = ld4_grad<BF16>(grow, e, d);
    if (drow) v = v + ld4_stream(drow, e, d);
    clip_store4<NB>(v, mask, e, d, msg + static_cast<int64_t>(row) * d * NB, drow);
}

// a + (1/n) sum_i Q[v_i] as the chain acc = fma(q_i, 1/n, acc) over workers in ascending order.  The messages of up to
// eight workers are asked for before the first is used: one after the other they were a chain of memory latencies.  Batches
// of 8, 4, 2 and 1 without a test of the count before every load, which with few workers cost more than the batch gains.
// Server block alone, one by one : eights with tests : as it is: 16 bits, 1 x 1,000,003 3.2 : 3.4 : 3.2 us, 9 x 5000 3.2 : 2.8 :
// 2.4 us, 16 x 1,000,003 9.9 : 7.6 : 7.3 us; 24 bits, 8 x 3,000,001 11.6 : 8.8 : 8.7 us, 8 x 25.6 M 74.7 : 65.7 : 65.7 us.
// ONE: one by one after all, where it is ahead (clip_one_by_one).
// The update in the server's pass spares a launch and reading the message again: server and update repeated, two launches :
// one pass, 8 x 1,000,003 7.8 : 5.2 us, 1 x 10 M 35 : 31 us, 16 x 10 M of 8 bits 153 : 153 us; within whole steps at 8 x 25.6 M,
// where nothing is left in a cache, 140 + 42 and 186 us.
// (Eight elements per thread, for 16 bytes of a message in one access, made steps of 8 x 25.6 M 746 us instead of 635, the stores
// of 16 bytes in every 32 being what costs.)
template <int NB, bool ONE>
__device__ __forceinline__ f32x4 clip_chain(f32x4 a, const uint8_t *msg_in, int n, float inv_n, int64_t e, int64_t d)
{
    if (!ONE && e + 4 <= d) {
        const uint8_t *p = msg_in + e * NB;
        const int64_t row = d * NB;
        auto batch = [&](auto count) {
            constexpr int C = decltype(count)::value;
            ClipRaw<NB> q[C];
#pragma unroll
            for (int i = 0; i < C; ++i) q[i] = load_raw4<NB>(p + i * row);
#pragma unroll
            for (int i = 0; i < C; ++i) a = fma4(inv_n, decode_raw4<NB>(q[i]), a);
            p += C * row;
        };
        int left = n;
        for (; left >= 8; left -= 8) batch(std::integral_constant<int, 8>{});
        if (left >= 4) { batch(std::integral_constant<int, 4>{}); left -= 4; }
        if (left >= 2) { batch(std::integral_constant<int, 2>{}); left -= 2; }
        if (left) batch(std::integral_constant<int, 1>{});
    } else {
        for (int i = 0; i < n; ++i) a = fma4(inv_n, load_msg4<NB>(msg_in + static_cast<int64_t>(i) * d * NB, e, d), a);
    }
    return a;
}

// Parameter-server block: v = delta_s + (1/n) sum_i Q[v_i], then the same compression.
// UPD: 0 = that block alone; 1, 2 = followed by the model update for the same elements (2: through the momentum
// buffer) from the registers that hold the message.
template <int NB, int UPD, bool ONE>
__global__ __launch_bounds__(kBlock) void k_clip_server(const uint8_t *msg_in, int n, float inv_n, float *delta_s,
                                                        uint8_t *msg_out, int64_t d, uint32_t mask, float *x, float *m,
                                                        float gamma, float beta)
{
    const int64_t e = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) * 4;
    if (e >= d) return;
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
    if (delta_s) a = ld4_stream(delta_s, e, d);           // null: no server error
    f32x4 xv = {0.f, 0.f, 0.f, 0.f}, mv = {0.f, 0.f, 0.f, 0.f};
    if constexpr (UPD != 0) xv = ld4_stream(x, e, d);
    if constexpr (UPD == 2) mv = ld4_stream(m, e, d);
    f32x4 q = clip_store4<NB>(clip_chain<NB, ONE>(a, msg_in, n, inv_n, e, d), mask, e, d, msg_out, delta_s);
    if constexpr (UPD != 0) {
        if constexpr (UPD == 2) {
            q = fma4(beta, mv, q);
            st4_stream(m, e, d, q);
        }
        st4_stream(x, e, d, fma4(-gamma, q, xv));
    }
}

// Server that does not compress: the average is the message (written and / or applied).
template <int NB, bool ONE>
__global__ __launch_bounds__(kBlock) void k_clip_server_identity(const uint8_t *msg_in, int n, float inv_n, int64_t d,
                                                                 float *dense_out, ds_update_args u)
{
    const int64_t e = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) * 4;
    if (e >= d) return;
    const f32x4 a = clip_chain<NB, ONE>(f32x4{0.f, 0.f, 0.f, 0.f}, msg_in, n, inv_n, e, d);
    put_average4(a, e, d, dense_out, u.x, u.m, u.gamma, u.beta);
}

template <int NB, bool MOM, bool DECODE_ONLY>
__global__ __launch_bounds__(kBlock) void k_clip_update(const uint8_t *msg, float *x, float *m, int64_t d, float gamma,
                                                        float beta)
{
    const int64_t e = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) * 4;
    if (e >= d) return;
    apply_q4<MOM, DECODE_ONLY>(load_msg4<NB>(msg, e, d), e, d, x, m, gamma, beta);
}

unsigned blocks4(int64_t d) { return static_cast<unsigned>((d + kBlock * 4 - 1) / (kBlock * 4)); }

uint32_t clip_mask(int bits) { return ~static_cast<uint32_t>((1ull << bits) - 1ull); }

// f(std::integral_constant<int, NB>) for the configured width
template <class F>
void with_bytes(int bits, F f)
{
    if (bits >= 24) f(std::integral_constant<int, 1>{});
    else if (bits >= 16) f(std::integral_constant<int, 2>{});
    else f(std::integral_constant<int, 4>{});
}

// Whether the server takes the messages one by one.  Messages of four bytes an element that come from memory keep it
// busy without batches, which then only cost wavefronts.  Server block, one by one : batches, 12 x 10 M 107 : 110 us, 24 x 5 M
// 97 : 101, 16 x 10 M 136 : 141, 32 x 10 M 251 : 271, 64 x 5 M 245 : 256 us; with the update it starts later, 12 x 25.6 M 311 : 301, 16 x
// 25.6 M 427 : 416, 24 x 10 M 213 : 218, 32 x 10 M 268 : 288, 64 x 3 M 151 : 160 us.  8 x 10 M 90 : 86 us, 64 x 1,000,003, from the
// cache, 48.5 : 45.6 us; shorter messages, 16 bits 0.95 .. 1.20 and 24 bits 1.03 .. 1.30 times as long one by one.
bool clip_one_by_one(const ds_ctx *c, bool update)
{
    return c->cfg.n >= (update ? 24 : 12) && c->cfg.n * c->cfg.d >= 100'000'000;
}

// f(bytes of an element of the message, whether the messages are taken one by one)
template <class F>
void with_chain(const ds_ctx *c, bool update, F f)
{
    with_bytes(c->cfg.levels, [&](auto nb) {
        constexpr int NB = decltype(nb)::value;
        if constexpr (NB == 4) {
            if (clip_one_by_one(c, update)) return f(nb, std::true_type{});
        }
        f(nb, std::false_type{});
    });
}

}  // namespace

int ds_clip_bytes(int bits) { return bits >= 24 ? 1 : bits >= 16 ? 2 : 4; }

ds_status_t ds_clip_worker(ds_ctx *c, const void *g, int64_t gs, float *delta, int64_t dstr, const ds_payload_t *out,
                           hipStream_t st)
{
    const int bits = c->cfg.levels;
    const dim3 grid(blocks4(c->cfg.d), static_cast<unsigned>(c->cfg.n));
    with_bytes(bits, [&](auto nb) {
        constexpr int NB = decltype(nb)::value;
        if (c->cfg.grad_dtype == DS_BF16)
            k_clip_worker<true, NB><<<grid, kBlock, 0, st>>>(g, gs, delta, dstr, out->levels, c->cfg.d, clip_mask(bits));
        else
            k_clip_worker<false, NB><<<grid, kBlock, 0, st>>>(g, gs, delta, dstr, out->levels, c->cfg.d, clip_mask(bits));
    });
    return ds_launch_status();
}

// x != nullptr: the model update for the same elements in the same kernel.
ds_status_t ds_clip_server(ds_ctx *c, const ds_payload_t *in, float *delta_s, const ds_payload_t *out, hipStream_t st, float *x,
                           float *m, float gamma, float beta)
{
    const int bits = c->cfg.levels;
    with_chain(c, x != nullptr, [&](auto nb, auto one) {
        auto go = [&](auto upd) {
            k_clip_server<decltype(nb)::value, decltype(upd)::value, decltype(one)::value><<<blocks4(c->cfg.d), kBlock, 0, st>>>(
                in->levels, c->cfg.n, c->inv_n, delta_s, out->levels, c->cfg.d, clip_mask(bits), x, m, gamma, beta);
        };
        if (!x) go(std::integral_constant<int, 0>{});
        else if (!m) go(std::integral_constant<int, 1>{});
        else go(std::integral_constant<int, 2>{});
    });
    return ds_launch_status();
}

ds_status_t ds_clip_server_identity(ds_ctx *c, const ds_payload_t *in, float *dense_out, ds_update_args u, hipStream_t st)
{
    with_chain(c, u.x != nullptr, [&](auto nb, auto one) {
        k_clip_server_identity<decltype(nb)::value, decltype(one)::value><<<blocks4(c->cfg.d), kBlock, 0, st>>>(
            in->levels, c->cfg.n, c->inv_n, c->cfg.d, dense_out, u);
    });
    return ds_launch_status();
}

ds_status_t ds_clip_update(ds_ctx *c, const ds_payload_t *srv, float *x, float *m, float gamma, float beta, hipStream_t st)
{
    with_bytes(c->cfg.levels, [&](auto nb) {
        constexpr int NB = decltype(nb)::value;
        if (m) k_clip_update<NB, true, false><<<blocks4(c->cfg.d), kBlock, 0, st>>>(srv->levels, x, m, c->cfg.d, gamma, beta);
        else k_clip_update<NB, false, false><<<blocks4(c->cfg.d), kBlock, 0, st>>>(srv->levels, x, m, c->cfg.d, gamma, beta);
    });
    return ds_launch_status();
}

ds_status_t ds_clip_decode(ds_ctx *c, const ds_payload_t *p, int32_t row, float *out, hipStream_t st)
{
    with_bytes(c->cfg.levels, [&](auto nb) {
        constexpr int NB = decltype(nb)::value;
        k_clip_update<NB, false, true><<<blocks4(c->cfg.d), kBlock, 0, st>>>(
            p->levels + static_cast<int64_t>(row) * c->cfg.d * NB, out, nullptr, c->cfg.d, 0.f, 0.f);
    });
    return ds_launch_status();
}
