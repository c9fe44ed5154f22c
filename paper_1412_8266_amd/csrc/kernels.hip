// HIP kernels of the MRG32k3a stream library (gfx950, wave64).
//
//   init_kernel      stream-set creation: state_g = A^(g * 2^127) seed     (sec. 4.1, 5.1)
//   jump_kernel      per-stream jump ahead with 4-bit windowed tables of
//                    A^(d * 16^w) mod m staged in LDS                    (sec. 2.3)
//   jumpu_kernel     one jump matrix (formed on the host) for every stream
//   fill_sm_kernel   bulk generation, stream-major output, one stream per
//                    lane, state in registers, LDS transpose to 16-byte
//                    row-segment stores                                  (sec. 5.2, Listing 1)
//   fill_il_kernel   bulk generation, interleaved output (lane = stream,
//                    consecutive lanes write consecutive elements);
//                    fill_il_seg_kernel the same in segments of each stream
//   fill_coop_kernel bulk generation, stream-major output, GL lanes per
//                    stream (sequence splitting inside each stream)
//   random_init_kernel  random spacing: each stream from its own expanded
//                    SplitMix64 draw                                     (sec. 2.3)
//   fill_split_kernel   rows of few streams (or one stream in order), split
//                       into blocks of a wave each                     (sec. 2.3)
//   fill_leap_kernel    leapfrog: one stream dealt to P players, each
//                    player's cards in a row                            (sec. 2.3)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gen_device.hpp"
#include "kernels.h"

namespace mrg {

// 16-byte units of a window's 16 matrices, and how many of `windows` windows'
// units a thread of a workgroup of 256 stages.
constexpr int kJumpUnits = kTableWindowWords / 4;
constexpr int jump_per(int windows) { return (windows * kJumpUnits + 255) / 256; }

// One component (blockIdx.y) of 256 streams per workgroup, a stream per lane:
// half the serial chain and twice the waves of a lane with both.  The windows
// [w_lo, the highest one that any exponent of the workgroup reaches) are
// staged in LDS with all of a thread's loads in flight, then applied; a matrix
// is 9 words, so lanes on different digits read different banks.  What bounds
// it is the chain of products.  Staging all 48 windows of both components a
// word at a time took most of 19 us for 65536 streams with 77-bit exponents.
// Every thread loads and stores each of its PER units (jump_per of the windows
// the launch can reach), those past the windows in use from the first one into
// room that nothing reads: under a condition of their own the units went
// through scratch memory one by one (192-bit jumps of 262144 streams 56.7 us,
// 43.8 now, 52.3 with both components in a lane).
// BOTH: the lane has both components, one after the other, for set creation on
// a full chip, where the chain is hidden and the exponents are shared (2^24
// streams 353 us, 420 with a component per lane; 2^18 9.7 and 9.9, 2^17 6.3 and
// 6.1).
template <int PER, bool BOTH = false>
__global__ void __launch_bounds__(256)
jump_kernel(uint32_t *__restrict__ planes, uint64_t plane_stride, uint64_t first,
            uint64_t count, const uint64_t *__restrict__ exps, uint64_t g0,
            InitSeed seed, const uint32_t *__restrict__ table, int w_lo, int w_hi)
{
    constexpr int NC = BOTH ? 2 : 1;
    __shared__ __attribute__((aligned(16))) uint32_t tab[NC][PER * 256 * 4];
    __shared__ int top_all;
    const int c0 = BOTH ? 0 : blockIdx.y;
    const uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool active = s < count;
    const uint64_t idx = first + s;
    uint32_t a[NC][3] = {};
    uint64_t e0 = 0, e1 = 0, e2 = 0;
    if (threadIdx.x == 0) top_all = w_lo;
    if (active) {
        if (exps) {  // jump the current state by its own exponent
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int i = 0; i < 3; ++i) a[c][i] = planes[(3 * (c0 + c) + i) * plane_stride + idx];
            e0 = exps[3 * s + 0];
            e1 = exps[3 * s + 1];
            e2 = exps[3 * s + 2];
        } else {     // create: start of global stream g = g0 + s is A^(g 2^127) seed
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int i = 0; i < 3; ++i) a[c][i] = seed.w[3 * (c0 + c) + i];
            const uint64_t g = g0 + s;
            e0 = 0;
            e1 = (g & 1u) << 63;
            e2 = g >> 1;
        }
    }
    int top = top_window(e0, e1, e2);
#pragma unroll
    for (int d = 32; d; d >>= 1) {
        const int o = __shfl_xor(top, d);
        top = o > top ? o : top;
    }
    __syncthreads();
    if (threadIdx.x % 64 == 0) atomicMax(&top_all, top);
    __syncthreads();
    const int end = top_all < w_hi ? top_all : w_hi;
    {
        const int units = (end - w_lo) * kJumpUnits;
        uint4 v[NC][PER];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint4 *src =
                (const uint4 *)(table + ((c0 + c) * kTableWindows + w_lo) * kTableWindowWords);
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int u = k * 256 + (int)threadIdx.x;
                v[c][k] = src[u < units ? u : 0];
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < PER; ++k) ((uint4 *)tab[c])[k * 256 + threadIdx.x] = v[c][k];
    }
    __syncthreads();
    for (int w = w_lo; w < end; ++w) {
        const uint32_t d = exp_digit(e0, e1, e2, w);
        if (!__any(d != 0u)) continue;  // wave-uniform skip of empty windows
        const uint32_t at = ((w - w_lo) * 16 + d) * 9;
        if (c0 == 0) matvec3<C1>(tab[0] + at, a[0][0], a[0][1], a[0][2]);
        else matvec3<C2>(tab[0] + at, a[0][0], a[0][1], a[0][2]);
        if (BOTH) matvec3<C2>(tab[NC - 1] + at, a[NC - 1][0], a[NC - 1][1], a[NC - 1][2]);
    }
    if (active) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int i = 0; i < 3; ++i)
                planes[(3 * (c0 + c) + i) * plane_stride + idx] =
                    c0 + c == 0 ? canon1(a[c][i]) : canon2(a[c][i]);
        if (!exps && c0 == 0 && ticket_pitch(plane_stride)) planes[ticket_of(plane_stride, idx)] = 0u;
    }
}

__global__ void __launch_bounds__(256)
jumpu_kernel(uint32_t *__restrict__ planes, uint64_t plane_stride, uint64_t first,
             uint64_t count, JumpMatrices J)
{
    const uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= count) return;
    const uint64_t idx = first + s;
    uint32_t a0 = planes[0 * plane_stride + idx];
    uint32_t a1 = planes[1 * plane_stride + idx];
    uint32_t a2 = planes[2 * plane_stride + idx];
    uint32_t b0 = planes[3 * plane_stride + idx];
    uint32_t b1 = planes[4 * plane_stride + idx];
    uint32_t b2 = planes[5 * plane_stride + idx];
    matvec3<C1>(J.m, a0, a1, a2);
    matvec3<C2>(J.m + 9, b0, b1, b2);
    planes[0 * plane_stride + idx] = a0;
    planes[1 * plane_stride + idx] = a1;
    planes[2 * plane_stride + idx] = a2;
    planes[3 * plane_stride + idx] = b0;
    planes[4 * plane_stride + idx] = b1;
    planes[5 * plane_stride + idx] = b2;
}

// Random spacing (sec. 2.3): stream g = g0 + s starts at the state expanded
// from SplitMix64 output g of the master seed.
__global__ void __launch_bounds__(256)
random_init_kernel(uint32_t *__restrict__ planes, uint64_t plane_stride, uint64_t count,
                   uint64_t g0, uint64_t master)
{
    const uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= count) return;
    uint32_t w[6];
    expand_seed(splitmix64_mix(master + (g0 + s + 1) * kSplitMixGamma), w);
    store_state(planes, plane_stride, s, w);
    if (ticket_pitch(plane_stride)) planes[ticket_of(plane_stride, s)] = 0u;
}

__global__ void __launch_bounds__(256)
ticket_reset_kernel(uint32_t *__restrict__ planes, uint64_t n, uint64_t first, uint64_t count)
{
    const uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s < count) planes[ticket_of(n, first + s)] = 0u;
}

// ---------------------------------------------------------------------------
// generation
// ---------------------------------------------------------------------------
// Lane-per-stream stream-major fill: one wave per 64 streams, each lane
// generating its stream's n values through the LDS tile writer rows_fill.
// HALVES: every stream is two lanes, the odd one drawing the second half of
// its row from J = A^(n/2) on (n even; rows and halves on 128-byte lines), so
// the wave's rows are 64 halves.  For rows of whole 4 KiB: a step of the
// wave then writes tiles 2 KiB apart instead of 4, which memory takes at 4.5
// instead of 3.4 TB/s (65536 x 1024 float32, buffers in turn: 80 -> 59 us).
template <int DT, int TB, class G, bool HALVES = false>
__global__ void __launch_bounds__(64)
fill_sm_kernel(uint32_t *__restrict__ planes, uint64_t plane_stride, uint64_t first,
               uint64_t count, uint64_t n, unsigned char *__restrict__ out, JumpMatrices J)
{
    constexpr int ES = Elem<DT>::size;
    // TB = 0: rows off their lines, written by rows_fill_carry in 128-byte windows
    __shared__ __attribute__((aligned(16))) unsigned char lds[64 * (TB ? TB + 16 : 128 + 160)];
    const int lane = threadIdx.x;
    const uint64_t rows = HALVES ? 2 * count : count;
    const uint64_t rn = HALVES ? n / 2 : n;  // values per row of the wave
    const uint64_t s0 = (uint64_t)blockIdx.x * 64;
    const uint64_t nrows = rows - s0 < 64 ? rows - s0 : 64;
    const bool active = (uint64_t)lane < nrows;
    const uint64_t idx = first + (HALVES ? (s0 + lane) / 2 : s0 + lane);

    uint32_t w[6] = {1u, 1u, 1u, 1u, 1u, 1u};
    if (active) load_state(planes, plane_stride, idx, w);
    if constexpr (HALVES) {
        if (lane & 1) {
            matvec3<C1>(J.m, w[0], w[1], w[2]);
            matvec3<C2>(J.m + 9, w[3], w[4], w[5]);
        }
    }
    G g;
    g.load(w);
    if (n * ES < 128) {  // the wave's rows are one block shorter than 64 lines
        rows_fill_short<DT, G>(g, lds, lane, nrows, out + s0 * n * ES, n);
    } else {
        if constexpr (TB == 0)
            rows_fill_carry<DT, 128, G>(g, lds, lane, nrows, out + s0 * n * ES, n);
        else
            rows_fill<DT, TB, G>(g, lds, lane, nrows, out + s0 * rn * ES, rn * ES, rn);
    }
    // the second half ends where the stream goes on (both lanes have read it)
    if (active && (!HALVES || (lane & 1))) {
        g.store(w);
        store_state(planes, plane_stride, idx, w);
    }
}

// Interleaved output out[k * count + s]: consecutive lanes are consecutive
// streams, so each step is one coalesced store per wave.  Written with the
// per-thread stream object of the public device header, as a user kernel
// would draw: one stream per thread, next() per value.
template <int DT, class G>
__global__ void __launch_bounds__(256)
fill_il_kernel(uint32_t *__restrict__ planes, uint64_t plane_stride, uint64_t first,
               uint64_t count, uint64_t n, unsigned char *__restrict__ out)
{
    constexpr int ES = Elem<DT>::size;
    const uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= count) return;
    Stream<G> rng;
    rng.load(planes, plane_stride, first + s);
    unsigned char *p = out + s * ES;
    const uint64_t step = count * ES;
    uint64_t k = 0;
    for (; k + 4 <= n; k += 4) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            put1<DT>(p, rng.g);
            p += step;
        }
    }
    for (; k < n; ++k) {
        put1<DT>(p, rng.g);
        p += step;
    }
    rng.store(planes, plane_stride, first + s);
}

// Interleaved fill of fewer streams than fill the chip one lane each: each
// stream's n steps are cut into nseg segments of S, lane t taking segment
// t / count of stream t % count (consecutive lanes still write consecutive
// elements), started by a jump of q * S; with `move` a stream's last segment to read
// its state moves it by n (J = A^n; arrive()).  Without segments a lane draws its
// whole stream in series, about 42 ns a step: 4096 x 16384 binary64 took
// 677 us on 64 waves.
template <int DT, class G>
__global__ void __launch_bounds__(256)
fill_il_seg_kernel(uint32_t *__restrict__ planes, uint64_t plane_stride, uint64_t first,
                   uint32_t count, uint64_t n, uint32_t nseg, uint64_t S,
                   unsigned char *__restrict__ out, int move, JumpMatrices J,
                   const uint32_t *__restrict__ table)
{
    constexpr int ES = Elem<DT>::size;
    const uint32_t t = blockIdx.x * 256 + threadIdx.x;  // count * nseg < 2^31
    const uint32_t q = t / count, s = t % count;
    if (q >= nseg) return;
    uint32_t w[6];
    load_state(planes, plane_stride, first + s, w);
    uint32_t arrived = 0;
    if (move) arrived = arrive(planes + ticket_of(plane_stride, first + s), nseg, w);
    uint32_t b[6] = {w[0], w[1], w[2], w[3], w[4], w[5]};
    const uint32_t q0 = __builtin_amdgcn_readfirstlane(q);
    if (__all(q == q0)) jump_uniform(table, (uint64_t)q0 * S, b);
    else jump_global(table, (uint64_t)q * S, 0, 0, 0, 16, b);
    G g;
    g.load(b);
    const uint64_t k0 = (uint64_t)q * S, k1 = k0 + S < n ? k0 + S : n;
    const uint64_t step = (uint64_t)count * ES;
    unsigned char *p = out + k0 * step + (uint64_t)s * ES;
    uint64_t k = k0;
    for (; k + 4 <= k1; k += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            put1<DT>(p, g);
            p += step;
        }
    }
    for (; k < k1; ++k) {
        put1<DT>(p, g);
        p += step;
    }
    if (move && last_arrival(arrived, nseg)) {
        matvec3<C1>(J.m, w[0], w[1], w[2]);
        matvec3<C2>(J.m + 9, w[3], w[4], w[5]);
        store_state(planes, plane_stride, first + s, w);
    }
}

// Wave-per-stream stream-major fill: workgroups (one wave each) stride over
// groups of 64/GL streams, GL lanes per stream; each group is written by
// wave_fill, so that every flush writes whole 128-byte lines and the streams
// in flight stay adjacent.  Lanes of a group past the last stream run on a
// dummy state and write nothing.  Groups go to XCDs by xcd_chunk (or
// xcd_range), gen_device.hpp.  Members stage two pieces per flush when their
// chunk segment holds an even number of them (runs of two lines per member
// per store instruction: 4 % faster on 2^20 x 4096 uint32 than one piece, at
// 17 KiB of LDS per wave, two waves per SIMD); else one (9 KiB, four waves
// per SIMD).  The bound keeps the register count inside that occupancy.
template <int DT, int L>
constexpr int coop_pieces() { return (L / (128 / Elem<DT>::size)) % 2 == 0 ? 2 : 1; }

template <int DT, int L, int GL, class G>
__global__ void __launch_bounds__(64, (coop_pieces<DT, L>() == 2 ? 2 : 4))
fill_coop_kernel(uint32_t *__restrict__ planes, uint64_t plane_stride, uint64_t first,
                 uint64_t count, uint64_t n, unsigned char *__restrict__ out,
                 const uint32_t *__restrict__ lane_tab, const uint32_t *__restrict__ tabs,
                 const uint32_t *__restrict__ table, int order, int whole)
{
    constexpr int ES = Elem<DT>::size;
    constexpr int SPW = 64 / GL;
    constexpr int NP = coop_pieces<DT, L>();
    __shared__ __attribute__((aligned(16))) unsigned char lds[64 * (NP * 128 + 16)];
    const int lane = threadIdx.x;
    const int t = lane / GL;  // this lane's stream within the group

    const uint64_t groups = (count + SPW - 1) / SPW;
    const XcdRange R = order == 0 && gridDim.x == groups ? xcd_chunk(groups) : xcd_range(groups);
    for (uint64_t grp = R.first; grp < R.end; grp += R.step) {
        const uint64_t s0 = grp * SPW;
        const int nsv = count - s0 < (uint64_t)SPW ? (int)(count - s0) : SPW;
        const uint64_t idx = first + s0 + t;
        uint32_t w[6] = {1u, 1u, 1u, 1u, 1u, 1u};
        if (t < nsv) load_state(planes, plane_stride, idx, w);
        // this member's lane matrix, loaded per group (L2-resident) so that it
        // holds no registers while the group's values are drawn
        uint32_t m[18];
#pragma unroll
        for (int i = 0; i < 18; ++i) m[i] = lane_tab[(lane % GL) * 18 + i];
        if (whole && nsv == SPW)  // every chunk whole, rows on lines (checked on the host)
            wave_fill_whole<DT, L, G, GL, NP>(w, m, lds, lane, out + s0 * n * ES, n, table);
        else
            wave_fill<DT, L, G, true, GL, 0, NP>(w, m, lds, lane, out + s0 * n * ES, n * ES, nsv, 0,
                                                 n, table, tabs, true);
        if (lane % GL == 0 && t < nsv) store_state(planes, plane_stride, idx, w);
    }
}

// Sequence splitting inside each stream (sec. 2.3), for fewer streams than
// the chip has wave slots (and one stream dealt in order): row s, n values at
// out + s * n * ES, is cut into nblk blocks, block q > 0 starting B values per
// block past the row's first 128-byte line, so that blocks meet on lines.  One
// wave per block jumps the stream's state to it (A^v0, windowed) and writes it
// with wave_fill (64 lanes, L values per lane per chunk).  With `move` the
// last wave to read a stream's state moves it by n (J = A^n; arrive()), else
// the states are left to a launch after this one.  Each XCD takes one
// contiguous range of blocks (one stream in order: 4 % faster than the
// chunked order of the stream-major fill).
//
// NP: pieces that members stage per flush; with one, four waves per SIMD, with
// two, longer runs of lines (FillLaunch::pieces).
template <int DT, int L, class G, int NP>
__global__ void __launch_bounds__(64, (NP == 2 ? 2 : 4))
fill_split_kernel(uint32_t *__restrict__ planes, uint64_t plane_stride, uint64_t first,
                  uint64_t count, uint64_t n, uint64_t B, uint32_t nblk,
                  unsigned char *__restrict__ out, int move, JumpMatrices J,
                  const uint32_t *__restrict__ lane_tab, const uint32_t *__restrict__ tabs,
                  const uint32_t *__restrict__ table)
{
    constexpr int ES = Elem<DT>::size;
    __shared__ __attribute__((aligned(16))) unsigned char lds[64 * (NP * 128 + 16)];
    const int lane = threadIdx.x;
    uint32_t m[18];
#pragma unroll
    for (int i = 0; i < 18; ++i) m[i] = lane_tab[lane * 18 + i];
    const XcdRange R = xcd_range(count * nblk);
    for (uint64_t r = R.first; r < R.end; r += R.step) {
        const uint64_t s = r / nblk, q = r % nblk;
        uint32_t w[6];
        load_state(planes, plane_stride, first + s, w);
        uint32_t arrived = 0;
        if (move && nblk > 1 && lane == 0)
            arrived = arrive(planes + ticket_of(plane_stride, first + s), nblk, w);
        unsigned char *row = out + s * n * ES;
        const uint64_t hv = head_values<ES>(row, n);
        const uint64_t v0 = q ? hv + q * B : 0;
        const uint64_t v1 = q + 1 < nblk && hv + (q + 1) * B < n ? hv + (q + 1) * B : n;
        if (v0 < v1) {  // the last block of a row with a head may be empty
            uint32_t b[6] = {w[0], w[1], w[2], w[3], w[4], w[5]};
            jump_uniform(table, v0, b);
            wave_fill<DT, L, G, true, 64, 0, NP>(b, m, lds, lane, row, 0, 1, v0, v1, table, tabs,
                                                 false);
        }
        if (move && lane == 0 && last_arrival(arrived, nblk)) {
            matvec3<C1>(J.m, w[0], w[1], w[2]);
            matvec3<C2>(J.m + 9, w[3], w[4], w[5]);
            store_state(planes, plane_stride, first + s, w);
        }
    }
}

// Leapfrog (sec. 2.3) with each player's cards in a row: card k of player t
// is output t + k*P of the stream (stream sidx of the planes) and goes to
// out[t*K + k].  A column block is KB = min(K, 64) card columns; lane
// l < R*KB (R = 64 / KB) takes column k = KB*kb + l % KB and sub-segment
// r = l / KB of each segment of T = R*Ts players, i.e. the stream's outputs
// [k*P + t0 + r*Ts, ... + Ts) in order, written down its column: a store
// instruction covers R runs of KB adjacent cards (64 adjacent cards when
// K >= 64).  Work items are (column block kb, segment); each wave takes a
// contiguous run of the nkb * nseg items, jumps its lanes once (A^(k*P +
// t0 + r*Ts)) and from then on only continues: to the next segment by
// A^(T - Ts) (Jseg; stepping on when R = 1), to the next column block by
// A^(63*P) (J63; only with R = 1, since K < 64 leaves one column block).  The
// waves of a workgroup (up to 16, for at most 256 workgroups) arrive together
// at the stream's ticket: 4096 arrivals one by one would queue for 80 us.  With
// `move` the last workgroup to read the state moves it by P*K, else a launch
// after this one.
template <int DT, class G>
__global__ void __launch_bounds__(1024)
fill_leap_kernel(uint32_t *__restrict__ planes, uint64_t plane_stride, uint64_t sidx,
                 LeapArgs A, unsigned char *__restrict__ out, const uint32_t *__restrict__ table)
{
    constexpr int ES = Elem<DT>::size;
    const uint64_t lane = threadIdx.x % 64;
    uint32_t w[6];
    load_state(planes, plane_stride, sidx, w);
    // this wave's state words are in registers, then the workgroup's
    asm volatile("" : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(w[4]), "+v"(w[5])::"memory");
    __syncthreads();
    if (A.move && threadIdx.x == 0 &&
        last_arrival(arrive(planes + ticket_of(plane_stride, sidx), gridDim.x, w), gridDim.x)) {
        uint32_t e[6] = {w[0], w[1], w[2], w[3], w[4], w[5]};
        matvec3<C1>(A.end.m, e[0], e[1], e[2]);
        matvec3<C2>(A.end.m + 9, e[3], e[4], e[5]);
        store_state(planes, plane_stride, sidx, e);
    }
    const uint64_t nb = (uint64_t)gridDim.x * (blockDim.x / 64);
    const uint64_t b = (uint64_t)blockIdx.x * (blockDim.x / 64) +
                       (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const uint64_t q = A.items / nb, rr = A.items % nb;
    const uint64_t i0 = b * q + (b < rr ? b : rr);
    const uint64_t i1 = i0 + q + (b < rr ? 1 : 0);
    if (i0 >= i1 || lane >= (uint64_t)A.R * A.KB) return;
    const uint64_t kl = lane % A.KB, r = lane / A.KB;
    uint64_t kb = i0 / A.nseg, seg = i0 % A.nseg;
    {
        // lanes past the last column start anywhere in range and write nothing
        const uint64_t k = kb * A.KB + kl < A.K ? kb * A.KB + kl : A.K - 1;
        if (A.R == 1) {  // the same segment start in every lane
            jump_uniform(table, seg * A.T, w);
            jump_global(table, k * A.P, 0, 0, 0, 16, w);
        } else {
            const uint64_t t = seg * A.T + r * A.Ts < A.P ? seg * A.T + r * A.Ts : A.P - 1;
            jump_global(table, k * A.P + t, 0, 0, 0, 16, w);
        }
    }
    G g;
    g.load(w);
    const uint64_t row = A.K * ES;
    for (uint64_t it = i0; it < i1; ++it) {
        if (it != i0) {
            if (seg == 0) {
                // column k ended at output (k+1)*P; column k+64 starts at (k+64)*P
                g.store(w);
                matvec3<C1>(A.J63.m, w[0], w[1], w[2]);
                matvec3<C2>(A.J63.m + 9, w[3], w[4], w[5]);
                g.load(w);
            } else if (A.R > 1) {
                // sub-segment r ended at t0 + (r+1)*Ts; the next one starts T - Ts on
                g.store(w);
                matvec3<C1>(A.Jseg.m, w[0], w[1], w[2]);
                matvec3<C2>(A.Jseg.m + 9, w[3], w[4], w[5]);
                g.load(w);
            }
        }
        const uint64_t k = kb * A.KB + kl;
        const uint64_t t0 = seg * A.T + r * A.Ts;
        const uint64_t t1 = t0 + A.Ts < A.P ? t0 + A.Ts : A.P;
        if (k < A.K && t0 < t1) {
            unsigned char *p = out + (t0 * A.K + k) * ES;
            uint64_t t = t0;
            for (; t + 4 <= t1; t += 4) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    put1<DT>(p, g);
                    p += row;
                }
            }
            for (; t < t1; ++t) {
                put1<DT>(p, g);
                p += row;
            }
        }
        if (++seg == A.nseg) {
            seg = 0;
            ++kb;
        }
    }
}

// ---------------------------------------------------------------------------
// launchers (host side)
// ---------------------------------------------------------------------------
static unsigned grid_of(uint64_t items, unsigned block)
{
    return (unsigned)((items + block - 1) / block);
}

hipError_t launch_init(uint32_t *planes, uint64_t plane_stride, uint64_t count,
                       uint64_t g0, const InitSeed &seed, const uint32_t *table,
                       int w_lo, int w_hi, hipStream_t st)
{
    const dim3 grid(grid_of(count, 256), 2), block(256);
    const uint64_t *none = nullptr;
#define MRG_INIT(PER)                                                                           \
    hipLaunchKernelGGL(jump_kernel<PER>, grid, block, 0, st, planes, plane_stride, (uint64_t)0,  \
                       count, none, g0, seed, table, w_lo, w_hi)
    // start states use 7 windows up to stream 2^24, 17 up to 2^64
    if (jump_per(w_hi - w_lo) <= 1 && count >= ((uint64_t)1 << 18))
        hipLaunchKernelGGL((jump_kernel<1, true>), dim3(grid_of(count, 256)), block, 0, st, planes,
                           plane_stride, (uint64_t)0, count, none, g0, seed, table, w_lo, w_hi);
    else if (jump_per(w_hi - w_lo) <= 1) MRG_INIT(1);
    else if (jump_per(w_hi - w_lo) <= 3) MRG_INIT(3);
    else MRG_INIT(jump_per(kTableWindows));
#undef MRG_INIT
    return hipGetLastError();
}

hipError_t launch_jump(uint32_t *planes, uint64_t plane_stride, uint64_t first,
                       uint64_t count, const uint64_t *d_exp, const uint32_t *table,
                       hipStream_t st)
{
    InitSeed none = {};
    hipLaunchKernelGGL(jump_kernel<jump_per(kTableWindows)>, dim3(grid_of(count, 256), 2),
                       dim3(256), 0, st, planes, plane_stride, first, count, d_exp, (uint64_t)0,
                       none, table, 0, kTableWindows);
    return hipGetLastError();
}

hipError_t launch_jump_uniform(uint32_t *planes, uint64_t plane_stride, uint64_t first,
                               uint64_t count, const JumpMatrices &J, hipStream_t st)
{
    hipLaunchKernelGGL(jumpu_kernel, dim3(grid_of(count, 256)), dim3(256), 0, st, planes,
                       plane_stride, first, count, J);
    return hipGetLastError();
}

template <int DT, class G>
static hipError_t launch_fill_g(uint32_t *planes, uint64_t plane_stride, uint64_t first,
                                uint64_t count, uint64_t n, int layout, void *out,
                                const FillLaunch &fl, int tile_bytes, hipStream_t st)
{
    unsigned char *o = (unsigned char *)out;
    if (layout == 1 && fl.kernel == 3) {
        hipLaunchKernelGGL((fill_il_seg_kernel<DT, G>), dim3(grid_of(count * fl.nblk, 256)),
                           dim3(256), 0, st, planes, plane_stride, first, (uint32_t)count, n,
                           fl.nblk, fl.B, o, fl.move, fl.end, fl.table);
    } else if (layout == 1) {
        hipLaunchKernelGGL((fill_il_kernel<DT, G>), dim3(grid_of(count, 256)), dim3(256), 0, st,
                           planes, plane_stride, first, count, n, o);
    } else if (fl.kernel == 1) {
        constexpr int TV = 128 / Elem<DT>::size;  // values per 128-byte piece
        const dim3 grid(fl.grid), block(64);
        const int nh = fl.L / TV;
#define MRG_COOP(GL, NH)                                                                        \
    hipLaunchKernelGGL((fill_coop_kernel<DT, (NH) * TV, GL, G>), grid, block, 0, st, planes,     \
                       plane_stride, first, count, n, o, fl.lane_tab, fl.tabs, fl.table,   \
                       fl.order, fl.whole)
        if (fl.L % TV) return hipErrorInvalidValue;
        else if (fl.lanes == 64 && nh == 1) MRG_COOP(64, 1);
        else if (fl.lanes == 64 && nh == 2) MRG_COOP(64, 2);
        else if (fl.lanes == 32 && nh == 2) MRG_COOP(32, 2);
        else if (fl.lanes == 32 && nh == 4) MRG_COOP(32, 4);
        else if (fl.lanes == 16 && nh == 4) MRG_COOP(16, 4);
        else if (fl.lanes == 16 && nh == 8) MRG_COOP(16, 8);
        else if (fl.lanes == 8 && nh == 8) MRG_COOP(8, 8);
        else if (fl.lanes == 8 && nh == 16) MRG_COOP(8, 16);
        else return hipErrorInvalidValue;
#undef MRG_COOP
    } else if (fl.kernel == 2) {
        constexpr int TV = 128 / Elem<DT>::size;
        const dim3 grid(fl.grid), block(64);
#define MRG_SPLIT(L, NP)                                                                        \
    hipLaunchKernelGGL((fill_split_kernel<DT, L, G, NP>), grid, block, 0, st, planes,            \
                       plane_stride, first, count, n, fl.B, fl.nblk, o, fl.move, fl.end,         \
                       fl.lane_tab, fl.tabs, fl.table)
        if (fl.L == TV && fl.pieces == 1) MRG_SPLIT(TV, 1);
        else if (fl.L == 2 * TV && fl.pieces == 1) MRG_SPLIT(2 * TV, 1);
        else if (fl.L == 8 * TV && fl.pieces == 1 && DT != 2) MRG_SPLIT(8 * TV, (DT == 2 ? 2 : 1));
        else if (fl.L == 8 * TV && fl.pieces == 2) MRG_SPLIT(8 * TV, 2);
        else return hipErrorInvalidValue;
#undef MRG_SPLIT
    } else if (fl.kernel == 4) {
        hipLaunchKernelGGL((fill_sm_kernel<DT, 256, G, true>), dim3(grid_of(2 * count, 64)), dim3(64),
                           0, st, planes, plane_stride, first, count, n, o, fl.end);
    } else if (tile_bytes == 0 && ((uintptr_t)out % 128 || (n * Elem<DT>::size) % 128)) {
        // rows off their lines: one write per shared line (rows_fill_carry)
        hipLaunchKernelGGL((fill_sm_kernel<DT, 0, G>), dim3(grid_of(count, 64)), dim3(64), 0, st,
                           planes, plane_stride, first, count, n, o, fl.end);
    } else if (tile_bytes == 256 || (tile_bytes == 0 && n * Elem<DT>::size >= 1024)) {
        hipLaunchKernelGGL((fill_sm_kernel<DT, 256, G>), dim3(grid_of(count, 64)), dim3(64), 0, st,
                           planes, plane_stride, first, count, n, o, fl.end);
    } else {
        hipLaunchKernelGGL((fill_sm_kernel<DT, 128, G>), dim3(grid_of(count, 64)), dim3(64), 0, st,
                           planes, plane_stride, first, count, n, o, fl.end);
    }
    return hipGetLastError();
}

template <class G>
static hipError_t launch_fill_d(uint32_t *planes, uint64_t plane_stride, uint64_t first,
                                uint64_t count, uint64_t n, int dtype, int layout, void *out,
                                const FillLaunch &fl, int tile_bytes, hipStream_t st)
{
    switch (dtype) {
    case 0: return launch_fill_g<0, G>(planes, plane_stride, first, count, n, layout, out, fl, tile_bytes, st);
    case 1: return launch_fill_g<1, G>(planes, plane_stride, first, count, n, layout, out, fl, tile_bytes, st);
    default: return launch_fill_g<2, G>(planes, plane_stride, first, count, n, layout, out, fl, tile_bytes, st);
    }
}

hipError_t launch_fill(uint32_t *planes, uint64_t plane_stride, uint64_t first, uint64_t count,
                       uint64_t n, int dtype, int layout, void *out,
                       const FillLaunch &fl, const FillTuning &tune, hipStream_t st)
{
    if (tune.engine == 1)
        return launch_fill_d<GenF>(planes, plane_stride, first, count, n, dtype, layout, out, fl,
                                   tune.tile_bytes, st);
    return launch_fill_d<GenI>(planes, plane_stride, first, count, n, dtype, layout, out, fl,
                               tune.tile_bytes, st);
}

hipError_t launch_random_init(uint32_t *planes, uint64_t plane_stride, uint64_t count,
                              uint64_t g0, uint64_t master, hipStream_t st)
{
    hipLaunchKernelGGL(random_init_kernel, dim3(grid_of(count, 256)), dim3(256), 0, st, planes,
                       plane_stride, count, g0, master);
    return hipGetLastError();
}

hipError_t launch_ticket_reset(uint32_t *planes, uint64_t n, uint64_t first, uint64_t count,
                               hipStream_t st)
{
    if (!ticket_pitch(n)) return hipSuccess;
    hipLaunchKernelGGL(ticket_reset_kernel, dim3(grid_of(count, 256)), dim3(256), 0, st, planes, n,
                       first, count);
    return hipGetLastError();
}

template <class G>
static hipError_t launch_leap_g(uint32_t *planes, uint64_t plane_stride, uint64_t sidx,
                                int dtype, const LeapArgs &A, const uint32_t *table,
                                unsigned char *o, hipStream_t st)
{
    const dim3 g((A.waves + A.per_group - 1) / A.per_group), b(A.per_group * 64);
    if (dtype == 0)
        hipLaunchKernelGGL((fill_leap_kernel<0, G>), g, b, 0, st, planes, plane_stride, sidx, A, o, table);
    else if (dtype == 1)
        hipLaunchKernelGGL((fill_leap_kernel<1, G>), g, b, 0, st, planes, plane_stride, sidx, A, o, table);
    else
        hipLaunchKernelGGL((fill_leap_kernel<2, G>), g, b, 0, st, planes, plane_stride, sidx, A, o, table);
    return hipGetLastError();
}

hipError_t launch_leap(uint32_t *planes, uint64_t plane_stride, uint64_t sidx, int dtype,
                       const LeapArgs &A, const uint32_t *table, void *out, int engine,
                       hipStream_t st)
{
    unsigned char *o = (unsigned char *)out;
    if (engine == 1) return launch_leap_g<GenF>(planes, plane_stride, sidx, dtype, A, table, o, st);
    return launch_leap_g<GenI>(planes, plane_stride, sidx, dtype, A, table, o, st);
}

}  // namespace mrg
