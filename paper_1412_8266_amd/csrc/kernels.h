// Internal interface between the C-ABI host code and the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mrg32k3a_device.h"  // table layout (kTableWindows, kTableWindowWords)

namespace mrg {

constexpr int kTableWords = 2 * kTableWindows * kTableWindowWords;

// A set's device memory: the six state planes, then in sets of up to 2^20 streams
// one ticket word per stream (arrive() in gen_device.hpp), 0 between launches and
// set by the kernels that create the streams and by mrg_set_states: fills of one
// stream that a caller failed to order can leave its ticket in between, and every
// later fill would then move the stream before all its parts have read the state.
// Arrivals at one 128-byte line queue up, 20 ns each over the eight XCDs, so sets
// of up to 4096 streams give each ticket its own line. Larger sets than 2^20
// streams have no tickets: few of their fills are cut into parts, a launch moves
// those, and every set would pay a sixth more memory and time to create (2^24
// streams: 64 of 448 MiB).
__host__ __device__ constexpr uint64_t ticket_pitch(uint64_t n)
{
    return n <= 4096 ? 32 : n <= ((uint64_t)1 << 20) ? 1 : 0;
}
__host__ __device__ constexpr uint64_t ticket_of(uint64_t n, uint64_t i)
{
    return 6 * n + i * ticket_pitch(n);
}
// Whether the parts of a fill of `count` streams of a set of n count themselves
// in, and the last one moves its stream (a single part does so without a ticket);
// else a launch follows (1.5-4 us).  The arrivals at one line must not take
// longer.  One per wave: 256 a line (5 us in a row).  One per lane, up to 32 of
// them in a step of a wave: 256 a ticket, and 2048 a line, 4096 where the fill is
// long enough to hide them (segments of 16 x 16384 uint32 of a set with packed
// tickets 15.8 us at 4096 a line, 9.7 with a launch; 32 x 4096 7.9 at 2048 and
// 7.9-8.4; 1024 x 16384 20.3 at 4096 and 21.4).
constexpr bool parts_move(uint64_t n, uint64_t count, uint64_t parts, bool per_lane)
{
    const uint64_t line = ticket_pitch(n) > 1 || count == 1 ? 1 : count < 32 ? count : 32;
    const uint64_t most = per_lane && line > 1 ? (count < 512 ? 2048 : 4096) : 256;
    return parts == 1 || (ticket_pitch(n) && parts <= 256 && parts * line <= most);
}
constexpr uint64_t set_words(uint64_t n) { return 6 * n + n * ticket_pitch(n); }

struct InitSeed { uint32_t w[6]; };
struct JumpMatrices { uint32_t m[18]; };  // component 1 then component 2

hipError_t launch_init(uint32_t *planes, uint64_t plane_stride, uint64_t count, uint64_t g0,
                       const InitSeed &seed, const uint32_t *table, int w_lo, int w_hi,
                       hipStream_t st);
hipError_t launch_jump(uint32_t *planes, uint64_t plane_stride, uint64_t first, uint64_t count,
                       const uint64_t *d_exp, const uint32_t *table, hipStream_t st);
hipError_t launch_jump_uniform(uint32_t *planes, uint64_t plane_stride, uint64_t first,
                               uint64_t count, const JumpMatrices &J, hipStream_t st);
// Generation engine (0: integer lazy words, 1: binary64 near-canonical words),
// bytes per row per LDS tile (128 or 256) of the lane-per-stream fill, and
// the stream-major strategy (0: automatic, 1: lane per stream, 2: wave per
// stream).
struct FillTuning {
    int engine = 1;
    int tile_bytes = 0;       // lane per stream: 0 = 128 for rows under 1 KiB, else 256
    int strategy = 0;
    int coop_wgs_per_cu = 0;  // wave per stream: 0 = one workgroup per stream group
    int coop_lanes = 0;       // wave per stream: lanes per stream (64, 32, 16, 8; 0 automatic)
    int coop_order = 0;       // wave per stream: 0 chunked (one front), 1 one range per XCD
};

// Lane tables of the wave-per-stream writer: table lane_table(L) holds
// A^(l*L) for l < 64 and each lane-segment length L = 16, 32, ..., 512 values
// (a chunk's members, and the shorter members of a chunk where rows end);
// table kHeadTable holds A^l (the values before a row's first 128-byte line
// boundary).
constexpr int kNumLaneTabs = 33;
constexpr int kHeadTable = 32;
__host__ __device__ constexpr int lane_table(int L) { return L / 16 - 1; }

// How one stream-major fill is launched (chosen on the host).
struct FillLaunch {
    // 0 lane per stream, 1 wave per stream, 2 rows in blocks; 3 interleaved in
    // segments (nblk segments of B steps per stream); 4 two lanes per stream
    // (end = A^(n/2))
    int kernel = 0;
    int L = 0;                          // values per lane per chunk (wave per stream)
    int lanes = 64;                     // lanes per stream (wave per stream)
    const uint32_t *lane_tab = nullptr; // [64][18]: A^(l*L), component 1 then 2 (lane l % lanes)
    const uint32_t *tabs = nullptr;     // all lane tables ([kNumLaneTabs][64][18])
    const uint32_t *table = nullptr;    // windowed jump tables (end state of a partial chunk)
    unsigned grid = 0;                  // workgroups (wave per stream)
    int order = 0;                      // group order (FillTuning::coop_order)
    int whole = 0;                      // rows on 128-byte lines, whole chunks only (fast writer)
    // rows in blocks: each row cut into nblk blocks of B values from its first
    // 128-byte line on, a wave each; the streams then move by n (end = A^n)
    uint64_t B = 0;
    uint32_t nblk = 0;
    int pieces = 1;                     // 128-byte pieces a lane stages per flush
    int move = 0;                       // the last block to read a state moves it (tickets)
    JumpMatrices end = {};
};

hipError_t launch_fill(uint32_t *planes, uint64_t plane_stride, uint64_t first, uint64_t count,
                       uint64_t n, int dtype, int layout, void *out,
                       const FillLaunch &fl, const FillTuning &tune, hipStream_t st);

// Random spacing: stream g0 + s of a set starts at the state expanded from
// SplitMix64 output g0 + s of the master seed.
// Tickets of streams [first, first + count) of a set of n streams back to 0.
hipError_t launch_ticket_reset(uint32_t *planes, uint64_t n, uint64_t first, uint64_t count,
                               hipStream_t st);

hipError_t launch_random_init(uint32_t *planes, uint64_t plane_stride, uint64_t count,
                              uint64_t g0, uint64_t master, hipStream_t st);

// Leapfrog with each player's cards in a row: P players, K cards each; work
// items of KB = min(K, 64) card columns x T = R*Ts players (R = 64 / KB lanes
// per column), nseg segments per column block, items = column blocks x nseg.
struct LeapArgs {
    uint64_t P = 0, K = 0, T = 0, Ts = 0, nseg = 0, items = 0;
    int KB = 64, R = 1;
    JumpMatrices J63 = {};   // A^(63*P): to the next column block (R = 1)
    JumpMatrices Jseg = {};  // A^(T - Ts): to the next segment (R > 1)
    unsigned waves = 0, per_group = 1;  // waves, and how many to a workgroup
    int move = 1;            // the last workgroup to read the state moves it (ticket)
    JumpMatrices end = {};   // A^(P*K): the stream's state after the deal
};

// One stream (plane index sidx) dealt to players, each player's cards in a row.
hipError_t launch_leap(uint32_t *planes, uint64_t plane_stride, uint64_t sidx, int dtype,
                       const LeapArgs &A, const uint32_t *table, void *out, int engine,
                       hipStream_t st);

// Philox4x32-10 stream sets (philox.hip): states (position, id, key).
hipError_t launch_philox_init(uint32_t *planes, uint64_t plane_stride, uint64_t count,
                              uint64_t g0, uint64_t key, hipStream_t st);
hipError_t launch_philox_jump(uint32_t *planes, uint64_t plane_stride, uint64_t first,
                              uint64_t count, const uint64_t *d_exp, uint64_t e, hipStream_t st);
hipError_t launch_philox_fill(uint32_t *planes, uint64_t plane_stride, uint64_t first,
                              uint64_t count, uint64_t n, int dtype, int layout, int cus,
                              void *out, hipStream_t st);

// TinyMT32 stream sets (tinymt.hip): states (s0, s1, s2, s3, q, 0), one
// record of tmt::kRecordWords words per parameter set (sets q0, q0 + 1, ...).
// Candidates: flags[i] = L | accepted << 16 for candidate c0 + i, phis
// (optional) its characteristic polynomial.  Records: ok[i] = 1 when set i
// is accepted.
hipError_t launch_tmt_candidates(uint64_t master, uint64_t c0, uint64_t n, uint32_t *flags,
                                 uint32_t *phis, hipStream_t st);
hipError_t launch_tmt_records(const uint32_t *params, uint64_t n, uint32_t *records, uint32_t *ok,
                              hipStream_t st);
hipError_t launch_tmt_init(uint32_t *planes, uint64_t plane_stride, uint64_t count, uint64_t g0,
                           uint64_t per_param, uint64_t q0, uint64_t master,
                           const uint32_t *records, hipStream_t st);
hipError_t launch_tmt_jump(uint32_t *planes, uint64_t plane_stride, uint64_t first, uint64_t count,
                           const uint64_t *d_exp, const uint64_t e[3], const uint32_t *records,
                           uint64_t q0, hipStream_t st);
hipError_t launch_tmt_fill(uint32_t *planes, uint64_t plane_stride, uint64_t first, uint64_t count,
                           uint64_t n, int dtype, int layout, void *out, const uint32_t *records,
                           uint64_t q0, int tile_bytes, hipStream_t st);

// Store-only bandwidth probes (probe.hip): pattern 0 streaming, 1 the
// wave-per-stream fill's line geometry.
hipError_t launch_write_probe(void *out, uint64_t bytes, int pattern, hipStream_t st);

}  // namespace mrg
