// Philox4x32-10 stream sets (Salmon, Moraes, Dror & Shaw, SC 2011): the
// counter-based generator family the paper embeds beside MRG32k3a.  A stream's
// six state words are (position lo, hi, stream id lo, hi, key lo, hi); output
// number `position` is word position % 4 of the block whose 128-bit counter is
// (position / 4, stream id).  No jump tables: a jump adds to the position.
//
//   philox_init_kernel    stream g = g0 + s: position 0, id g, the set's key
//   philox_jump_kernel    position += e (per stream from device memory, or
//                         one e for the range)
//   philox_rows_kernel    stream-major fill of short rows: a workgroup's rows
//                         are one block of memory, staged in LDS and written
//                         as 16-byte stores
//   philox_runs_kernel    stream-major fill of longer rows: a wave per run of
//                         a row, one 16-byte aligned unit of 4 values per lane
//                         and step
//   philox_il_kernel      interleaved fill: one stream (or a segment of one)
//                         per lane, consecutive lanes write consecutive
//                         elements
// A fill moves the positions itself: the workgroup or lane that holds a whole
// row, or the last to read it of several (arrive(), gen_device.hpp); rows of
// very many parts (parts_move, kernels.h) leave it to a jump launch after the
// fill.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gen_device.hpp"
#include "kernels.h"
#include "philox_device.h"  // philox10, philox_block, conversions

namespace mrg {
namespace {

// Conversions of a word: (2*(w>>9)+1)*2^-24 as binary32 (1 + k*2^-23 minus
// 1 - 2^-24, exact), (2w+1)*2^-33 as binary64 (one exact FMA).
template <int DT> struct PhiloxOut;
template <> struct PhiloxOut<0> {
    using T = uint32_t;
    __device__ static T conv(uint32_t w) { return w; }
};
template <> struct PhiloxOut<1> {
    using T = float;
    __device__ static T conv(uint32_t w) { return philox_to_f32(w); }
};
template <> struct PhiloxOut<2> {
    using T = double;
    __device__ static T conv(uint32_t w) { return philox_to_f64(w); }
};

__device__ __forceinline__ uint64_t position(const uint32_t *w)
{
    return (uint64_t)w[0] | (uint64_t)w[1] << 32;
}

__global__ void __launch_bounds__(256)
philox_init_kernel(uint32_t *__restrict__ planes, uint64_t plane_stride, uint64_t count,
                   uint64_t g0, uint64_t key)
{
    const uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= count) return;
    const uint64_t g = g0 + s;
    const uint32_t w[6] = {0u, 0u, (uint32_t)g, (uint32_t)(g >> 32), (uint32_t)key,
                           (uint32_t)(key >> 32)};
    store_state(planes, plane_stride, s, w);
    if (ticket_pitch(plane_stride)) planes[ticket_of(plane_stride, s)] = 0u;
}

__global__ void __launch_bounds__(256)
philox_jump_kernel(uint32_t *__restrict__ planes, uint64_t plane_stride, uint64_t first,
                   uint64_t count, const uint64_t *__restrict__ exps, uint64_t e_uniform)
{
    const uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= count) return;
    const uint64_t idx = first + s;
    const uint64_t e = exps ? exps[3 * s] : e_uniform;  // position wraps at 2^64
    const uint64_t pos = ((uint64_t)planes[idx] | (uint64_t)planes[plane_stride + idx] << 32) + e;
    planes[idx] = (uint32_t)pos;
    planes[plane_stride + idx] = (uint32_t)(pos >> 32);
}

// Position p + n of a row into its state words.
__device__ __forceinline__ void store_position(uint32_t *planes, uint64_t plane_stride, uint64_t idx,
                                               uint64_t pos)
{
    planes[idx] = (uint32_t)pos;
    planes[plane_stride + idx] = (uint32_t)(pos >> 32);
}

// Four words, values of a row from element p on, as 16-byte stores (p on a
// 16-byte boundary).
template <int DT>
__device__ __forceinline__ void store_unit(typename PhiloxOut<DT>::T *p, const uint32_t *v)
{
    if constexpr (DT == 2) {
        *(double2 *)p = make_double2(PhiloxOut<2>::conv(v[0]), PhiloxOut<2>::conv(v[1]));
        *(double2 *)(p + 2) = make_double2(PhiloxOut<2>::conv(v[2]), PhiloxOut<2>::conv(v[3]));
    } else {
        uint4 q;
        q.x = __builtin_bit_cast(uint32_t, PhiloxOut<DT>::conv(v[0]));
        q.y = __builtin_bit_cast(uint32_t, PhiloxOut<DT>::conv(v[1]));
        q.z = __builtin_bit_cast(uint32_t, PhiloxOut<DT>::conv(v[2]));
        q.w = __builtin_bit_cast(uint32_t, PhiloxOut<DT>::conv(v[3]));
        *(uint4 *)p = q;
    }
}

// Stream-major, short rows: a workgroup owns rpw adjacent rows, one piece of
// memory; MANY (its own instance: the loop over pieces costs the others 5-10 %):
// rows_wg rows, several such pieces, in the chunked XCD order, so that rows whose
// states share a line meet in one L2 and an XCD's workgroups write one front.
// Item i is block i % mb of row i / mb (mb: the most blocks a row can touch;
// magic = ceil(2^32 / mb), exact for the few thousand items here).  With `quads`
// (rows of whole 16-byte units on 16-byte boundaries; mb is then n / 4) and every
// position at a block's start (and one key), the items are the piece's units in
// order and go straight to memory; else the rows are staged rpw at a time (at
// most kPhiloxLds bytes, 4 blocks per thread): an item's values go to LDS at
// their byte in the piece (off by the piece's own place in 16 bytes) and the
// piece is then written as 16-byte stores.
constexpr int kPhiloxLds = 16384;

template <int DT, bool MANY>
__global__ void __launch_bounds__(256)
philox_rows_kernel(uint32_t *__restrict__ planes, uint64_t plane_stride, uint64_t first,
                   uint64_t count, uint32_t n, uint32_t rows_wg, uint32_t rpw, uint32_t mb,
                   uint32_t magic, int quads, unsigned char *__restrict__ out)
{
    using T = typename PhiloxOut<DT>::T;
    __shared__ __attribute__((aligned(16))) unsigned char lds[kPhiloxLds + 16];
    __shared__ uint32_t st[6][256];
    if (!MANY) rows_wg = rpw;
    const uint64_t wg = MANY ? xcd_chunk(gridDim.x).first : blockIdx.x;
    for (uint64_t s0 = wg * rows_wg; s0 < count; s0 += (uint64_t)gridDim.x * rows_wg) {
        const uint32_t all = count - s0 < rows_wg ? (uint32_t)(count - s0) : rows_wg;
        // this thread's row starts within a block, or has another key than the
        // first row (sets are made under one key, but any states can be set)
        int within = 0, odd_key = 0;
        if (threadIdx.x < all) {
            uint32_t w[6];
            load_state(planes, plane_stride, first + s0 + threadIdx.x, w);
#pragma unroll
            for (int c = 0; c < 6; ++c) st[c][threadIdx.x] = w[c];
            store_position(planes, plane_stride, first + s0 + threadIdx.x, position(w) + n);
            within = w[0] & 3u;
        }
        const bool lined = !__syncthreads_or(within) && quads;
        if (threadIdx.x < all)
            odd_key = st[4][threadIdx.x] != st[4][0] || st[5][threadIdx.x] != st[5][0];
        const bool one_key = !__syncthreads_or(odd_key);
        // the round keys stay in scalar registers
        const uint32_t key0 = __builtin_amdgcn_readfirstlane(st[4][0]);
        const uint32_t key1 = __builtin_amdgcn_readfirstlane(st[5][0]);
        unsigned char *base = out + s0 * n * sizeof(T);
        if (lined && one_key) {
            for (uint32_t i = threadIdx.x; i < all * mb; i += 256) {
                const uint32_t r = mb == 1 ? i : __umulhi(i, magic), b = i - r * mb;
                const uint32_t w[6] = {st[0][r], st[1][r], st[2][r], st[3][r], key0, key1};
                uint32_t v[4];
                philox_block(w, (position(w) >> 2) + b, v);
                store_unit<DT>((T *)base + 4 * i, v);
            }
            __syncthreads();  // st is free again
            continue;
        }
        // a row of whole units that starts within a block touches one block more
        const uint32_t nb = mb + (quads ? 1u : 0u);
        for (uint32_t q = 0; q < all; q += rpw, base += rpw * n * sizeof(T)) {
            const uint32_t rows = !MANY ? all : all - q < rpw ? all - q : rpw;
            const uint32_t o = (uint32_t)((uintptr_t)base & 15u);
            for (uint32_t i = threadIdx.x; i < rows * nb; i += 256) {
                const uint32_t r = quads ? i / nb : mb == 1 ? i : __umulhi(i, magic), b = i - r * nb;
                const uint32_t t = q + r;
                uint32_t w[6] = {st[0][t], st[1][t], st[2][t], st[3][t], key0, key1};
                const uint64_t pos = position(w);
                uint32_t v[4];
                if (one_key) {
                    philox_block(w, (pos >> 2) + b, v);
                } else {
                    w[4] = st[4][t];
                    w[5] = st[5][t];
                    philox_block(w, (pos >> 2) + b, v);
                }
                const uint32_t k0 = 4 * b - ((uint32_t)pos & 3u);  // wraps below 0 for b = 0
                const uint32_t at = o + (r * n + k0) * (uint32_t)sizeof(T);
                if (k0 < n && k0 + 4 <= n && at % 16 == 0) {
                    store_unit<DT>((T *)(lds + at), v);
                    continue;
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t k = k0 + j;
                    if (k < n) ((T *)(lds + o))[r * n + k] = PhiloxOut<DT>::conv(v[j]);
                }
            }
            __syncthreads();
            // bytes [o, end) of lds belong at base - o
            const uint32_t end = o + rows * n * (uint32_t)sizeof(T);
            unsigned char *dst = base - o;
            for (uint32_t i = threadIdx.x * 16; i < end; i += 256 * 16) {
                if (i >= o && i + 16 <= end) {
                    *(uint4 *)(dst + i) = *(const uint4 *)(lds + i);
                } else {
#pragma unroll
                    for (uint32_t d = i; d < i + 16; d += 4)
                        if (d >= o && d < end) *(uint32_t *)(dst + d) = *(const uint32_t *)(lds + d);
                }
            }
            __syncthreads();  // lds, and after the last rows st, are free again
            if (!MANY) break;
        }
    }
}

// Stream-major, longer rows: each row is cut into nrun runs of `units` units
// of 4 values, a wave each, one unit per lane and step; unit u holds the row's
// values [4u - neg, 4u - neg + 4), neg values from the 128-byte line on which
// the row starts, so that every store of a step is whole lines.  A unit's
// words start at word sh = (position - neg) % 4 of a block, so with sh > 0
// each lane takes the rest from the next lane's block (a wave shift), the last
// lane from the first one of the next step, which is why a step's units are
// stored after the next step's blocks are drawn.  A wave takes rw rows (one
// when they are cut), lane r loading row r's state, so that short rows share
// the wait for it.  With `chunked` the workgroups take the rows in the chunked
// XCD order.
__device__ __forceinline__ uint32_t from_next_lane(uint32_t v, uint32_t last)
{
    // wave_shl:1, lane 63 keeps `last`
    return (uint32_t)__builtin_amdgcn_update_dpp((int)last, (int)v, 0x130, 0xf, 0xf, false);
}

template <int DT>
__global__ void __launch_bounds__(256)
philox_runs_kernel(uint32_t *__restrict__ planes, uint64_t plane_stride, uint64_t first,
                   uint64_t count, uint64_t n, uint32_t rw, uint32_t nrun, uint32_t units, int move,
                   int chunked, unsigned char *__restrict__ out)
{
    using T = typename PhiloxOut<DT>::T;
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t items = (count + rw - 1) / rw * nrun;
    const uint64_t wg = chunked ? xcd_chunk(gridDim.x).first : blockIdx.x;
    for (uint64_t item = wg * 4 +
                         (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
         item < items; item += (uint64_t)gridDim.x * 4) {
        const uint64_t s0 = item / nrun * rw, q = item % nrun;
        const uint32_t rows = count - s0 < rw ? (uint32_t)(count - s0) : rw;
        // lane r holds row s0 + r's state
        uint32_t w[6] = {0u, 0u, 0u, 0u, 0u, 0u};
        if (lane < rows) load_state(planes, plane_stride, first + s0 + lane, w);
        uint32_t arrived = 0;
        if (move && lane < rows && nrun > 1)
            arrived = arrive(planes + ticket_of(plane_stride, first + s0 + lane), nrun, w);
        for (uint32_t r = 0; r < rows; ++r) {
            uint32_t x[6];
#pragma unroll
            for (int i = 0; i < 6; ++i)
                x[i] = (uint32_t)__builtin_amdgcn_readlane((int)w[i], (int)r);
            const uint64_t pos = position(x);
            T *row = (T *)out + (s0 + r) * n;
            const uint32_t neg = (uint32_t)((uintptr_t)row & 127u) / (uint32_t)sizeof(T);
            const uint32_t sh = ((uint32_t)pos - neg) & 3u;
            const uint64_t nu = (n + neg + 3) / 4;
            const uint64_t u0 = q * units, u1 = u0 + units < nu ? u0 + units : nu;
            // unit u's first block (mod 2^62, as the positions wrap)
            uint64_t blk = ((pos - neg) >> 2) + u0 + lane;
            uint32_t c[4], d[4];
            auto put = [&](uint64_t u, const uint32_t *v) {
                const uint64_t k = 4 * u - neg;  // before the row: wraps to a huge value
                if (u >= u1) return;
                if (k < n && k + 4 <= n) {
                    store_unit<DT>(row + k, v);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (k + j < n) row[k + j] = PhiloxOut<DT>::conv(v[j]);
                }
            };
            if (sh == 0) {
                for (uint64_t u = u0; u < u1; u += 64, blk += 64) {
                    philox_block(x, blk, c);
                    put(u + lane, c);
                }
                continue;
            }
            philox_block(x, blk, c);
            for (uint64_t u = u0; u < u1; u += 64) {
                blk += 64;
                philox_block(x, blk, d);
                uint32_t t[7] = {c[0], c[1], c[2], c[3], 0u, 0u, 0u};
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    t[4 + j] = from_next_lane(c[j], __builtin_amdgcn_readfirstlane(d[j]));
                if (sh & 1u) {
#pragma unroll
                    for (int j = 0; j < 6; ++j) t[j] = t[j + 1];
                }
                if (sh & 2u) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) t[j] = t[j + 2];
                }
                put(u + lane, t);
#pragma unroll
                for (int j = 0; j < 4; ++j) c[j] = d[j];
            }
        }
        if (move && lane < rows && last_arrival(arrived, nrun))
            store_position(planes, plane_stride, first + s0 + lane, position(w) + n);
    }
}

// Interleaved: out[k * count + s]; lane t draws segment t / count (sb blocks,
// nseg segments per stream) of stream t % count.
template <int DT>
__global__ void __launch_bounds__(256)
philox_il_kernel(uint32_t *__restrict__ planes, uint64_t plane_stride, uint64_t first,
                 uint64_t count, uint64_t n, uint32_t nseg, uint64_t sb, int move,
                 unsigned char *__restrict__ out)
{
    using T = typename PhiloxOut<DT>::T;
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t s = t, q = 0;
    if (nseg > 1) {  // count * nseg < 2^31
        q = (uint32_t)t / (uint32_t)count;
        s = (uint32_t)t % (uint32_t)count;
    }
    if (s >= count || q >= nseg) return;
    uint32_t w[6];
    load_state(planes, plane_stride, first + s, w);
    uint32_t arrived = 0;
    if (move && nseg > 1) arrived = arrive(planes + ticket_of(plane_stride, first + s), nseg, w);
    const uint64_t pos = position(w);
    const uint64_t off = pos & 3, b0 = pos >> 2;
    const uint64_t nb = (off + n + 3) / 4;
    const uint64_t b1 = q + 1 < nseg && (q + 1) * sb < nb ? (q + 1) * sb : nb;
    T *col = (T *)out + s;
    for (uint64_t b = q * sb; b < b1; ++b) {
        uint32_t v[4];
        philox_block(w, b0 + b, v);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t k = 4 * b + j - off;
            if (k < n) col[k * count] = PhiloxOut<DT>::conv(v[j]);
        }
    }
    if (move && last_arrival(arrived, nseg)) store_position(planes, plane_stride, first + s, pos + n);
}

unsigned grid256(uint64_t items) { return (unsigned)((items + 255) / 256); }

}  // namespace

hipError_t launch_philox_init(uint32_t *planes, uint64_t plane_stride, uint64_t count,
                              uint64_t g0, uint64_t key, hipStream_t st)
{
    hipLaunchKernelGGL(philox_init_kernel, dim3(grid256(count)), dim3(256), 0, st, planes,
                       plane_stride, count, g0, key);
    return hipGetLastError();
}

hipError_t launch_philox_jump(uint32_t *planes, uint64_t plane_stride, uint64_t first,
                              uint64_t count, const uint64_t *d_exp, uint64_t e, hipStream_t st)
{
    hipLaunchKernelGGL(philox_jump_kernel, dim3(grid256(count)), dim3(256), 0, st, planes,
                       plane_stride, first, count, d_exp, e);
    return hipGetLastError();
}

template <int DT>
static hipError_t launch_philox_fill_t(uint32_t *planes, uint64_t plane_stride, uint64_t first,
                                       uint64_t count, uint64_t n, int layout, int cus, void *out,
                                       hipStream_t st)
{
    unsigned char *o = (unsigned char *)out;
    constexpr uint64_t ES = sizeof(typename PhiloxOut<DT>::T);
    const uint64_t cap = 1 << 22;  // workgroups (the kernels loop; 2^32 threads to a launch)
    if (layout == 1 && count > 1) {
        // segments of at least 16 blocks, up to four waves per SIMD (one for
        // binary64: 65536 x 1000 in four segments 89 -> 110 us)
        const uint64_t lanes = (uint64_t)cus * (ES == 8 ? 256 : 1024), nb = (n + 6) / 4;
        uint64_t nseg = lanes / count < nb / 16 ? lanes / count : nb / 16;
        if (nseg > 256) nseg = 256;  // arrivals per ticket
        if (nseg < 1) nseg = 1;
        const uint64_t sb = (nb + nseg - 1) / nseg;
        nseg = (nb + sb - 1) / sb;
        const int move = parts_move(plane_stride, count, nseg, true);
        hipLaunchKernelGGL((philox_il_kernel<DT>), dim3(grid256(count * nseg)), dim3(256), 0, st,
                           planes, plane_stride, first, count, n, (uint32_t)nseg, sb, move, o);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess && !move)
            e = launch_philox_jump(planes, plane_stride, first, count, nullptr, n, st);
        return e;
    }
    // short rows a workgroup at a time (rows of 600 and 1000 float32 off 16
    // bytes or blocks are faster in runs: 65536 x 600 42 against 39 us)
    const int quads = n % 4 == 0 && (uintptr_t)out % 16 == 0;
    if (n * ES < (quads || ES == 8 ? 4096 : 2048)) {
        // pieces of as many rows as fit (four blocks per thread), fewer while
        // that leaves under four workgroups per CU; fills of 512 MiB and more two
        // pieces to a workgroup, of a GiB in binary64 four, in the chunked order
        // (2^20 x 384 uint32 403 us in single pieces, 298 in pairs, at position 1
        // 407 and 359; 2^20 x 384 binary64 690, in pairs 650, in fours 601; below
        // 512 MiB pairs lose: 262144 x 128 uint32 25.2 us in single pieces and 28)
        const uint32_t mb = quads ? (uint32_t)n / 4 : (uint32_t)(n + 6) / 4;
        uint64_t rpw = kPhiloxLds / (n * ES) < 1024 / mb ? kPhiloxLds / (n * ES) : 1024 / mb;
        if (rpw > 256) rpw = 256;
        const uint64_t spread = count / ((uint64_t)cus * 4);
        if (rpw > spread) rpw = spread < 1 ? 1 : spread;
        const uint64_t bytes = count * n * ES;
        const bool many = bytes >= (uint64_t)512 << 20;
        const uint64_t pieces = !many ? 1 : ES == 8 && bytes >= (uint64_t)1 << 30 ? 4 : 2;
        const uint64_t rows_wg = rpw * pieces <= 256 ? rpw * pieces : 256 / rpw * rpw;
        const uint64_t wgs = (count + rows_wg - 1) / rows_wg;
        const uint32_t magic = (uint32_t)((((uint64_t)1 << 32) + mb - 1) / mb);  // mb = 1: not used
        const dim3 grid((unsigned)(wgs < cap ? wgs : cap)), block(256);
#define MRG_ROWS(MANY)                                                                          \
    hipLaunchKernelGGL((philox_rows_kernel<DT, MANY>), grid, block, 0, st, planes, plane_stride,  \
                       first, count, (uint32_t)n, (uint32_t)rows_wg, (uint32_t)rpw, mb, magic,    \
                       quads, o)
        if (many) MRG_ROWS(true);
        else MRG_ROWS(false);
#undef MRG_ROWS
        return hipGetLastError();
    }
    // runs of up to 16 KiB (16 steps of 64 units, 8 of binary64: 131072 x 4096
    // binary64 748 us, in runs of 16 steps 777, x 5120 881 and 999), fewer steps
    // while that leaves under eight waves per SIMD
    const uint64_t neg = (uintptr_t)out % 128 || (n * ES) % 128 ? 128 / ES - 1 : 0;
    const uint64_t steps = ((n + neg + 3) / 4 + 63) / 64;
    uint64_t per = steps * count / ((uint64_t)cus * 32);
    const uint64_t most = ES == 8 ? 8 : 16;
    per = per < 1 ? 1 : per > most ? most : per;
    while (per < steps && (steps + per - 1) / per >= (uint64_t)1 << 31) per *= 2;
    uint64_t nrun = (steps + per - 1) / per;
    per = (steps + nrun - 1) / nrun;
    nrun = (steps + per - 1) / per;
    // rows under 6 KiB: several to a wave while eight waves per SIMD are left
    // (65536 x 1024 float32 56 -> 49 us); longer ones lose by it (262144 x
    // 1024 binary64 382 -> 456)
    uint64_t rw = nrun > 1 || n * ES >= 6144 ? 1 : count / ((uint64_t)cus * 32);
    rw = rw < 1 ? 1 : rw > 8 ? 8 : rw;
    const uint64_t wgs = ((count + rw - 1) / rw * nrun + 3) / 4;
    // rows of one run in the chunked order, so that rows whose states share a
    // line meet in one L2 (131072 x 3072 uint32 290 us, in dispatch order 305;
    // x 4096 368 and 379), but for 8 KiB (2^19 x 1024 binary64 932 and 730, 2048
    // uint32 804 and 677) and cut rows (131072 x 5120 uint32 690 and 448)
    const int chunked = nrun == 1 && n * ES > 8192;
    const int move = parts_move(plane_stride, count, nrun, false);
    hipLaunchKernelGGL((philox_runs_kernel<DT>), dim3((unsigned)(wgs < cap ? wgs : cap)), dim3(256), 0, st,
                       planes, plane_stride, first, count, n, (uint32_t)rw,
                       (uint32_t)nrun, (uint32_t)(per * 64), move, chunked, o);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && !move)
        e = launch_philox_jump(planes, plane_stride, first, count, nullptr, n, st);
    return e;
}

hipError_t launch_philox_fill(uint32_t *planes, uint64_t plane_stride, uint64_t first,
                              uint64_t count, uint64_t n, int dtype, int layout, int cus,
                              void *out, hipStream_t st)
{
    switch (dtype) {
    case 0: return launch_philox_fill_t<0>(planes, plane_stride, first, count, n, layout, cus, out, st);
    case 1: return launch_philox_fill_t<1>(planes, plane_stride, first, count, n, layout, cus, out, st);
    default: return launch_philox_fill_t<2>(planes, plane_stride, first, count, n, layout, cus, out, st);
    }
}

}  // namespace mrg
