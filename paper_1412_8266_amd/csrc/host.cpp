// C ABI of the MRG32k3a stream library: argument validation, host-side jump
// matrices and tables, device memory of stream sets, kernel launches.
//
// Host initialisation before any kernel (sec. 5.1): creating a stream set
// allocates its device state and computes every stream's starting state on
// the device; release frees it.  Streams and substreams follow sec. 4.1 and
// the jump ahead of sec. 2.3 (matrix powers mod m).
#include <hip/hip_runtime.h>

#include <array>
#include <cstdarg>
#include <cstdio>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "internal.h"
#include "mrg_arith.hpp"

namespace {
thread_local std::string g_last_error;
}

namespace mrg {

mrg_status set_error(mrg_status s, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return s;
}

mrg_status hip_error(hipError_t e, const char *what)
{
    return set_error(MRG_EHIP, "%s: %s", what, hipGetErrorString(e));
}

}  // namespace mrg

namespace {

using mrg::set_error;
using mrg::hip_error;

// ---- host jump matrices (sec. 2.3) ---------------------------------------
using Mat = std::array<uint32_t, 9>;

Mat identity() { return {1, 0, 0, 0, 1, 0, 0, 0, 1}; }

uint64_t modulus(int c) { return c == 0 ? mrg::M1 : mrg::M2; }

// Companion matrix of component c on the column (x[n-3], x[n-2], x[n-1]).
Mat companion(int c)
{
    Mat A = {0, 1, 0, 0, 0, 1, 0, 0, 0};
    if (c == 0) {
        A[6] = mrg::M1 - mrg::A13N;
        A[7] = mrg::A12;
    } else {
        A[6] = mrg::M2 - mrg::A23N;
        A[8] = mrg::A21;
    }
    return A;
}

Mat mul(const Mat &X, const Mat &Y, uint64_t m)
{
    Mat R;
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            unsigned __int128 acc = 0;
            for (int k = 0; k < 3; ++k) acc += (unsigned __int128)X[3 * i + k] * Y[3 * k + j];
            R[3 * i + j] = (uint32_t)(acc % m);
        }
    return R;
}

Mat power(int c, const uint64_t e[3])
{
    const uint64_t m = modulus(c);
    Mat R = identity(), B = companion(c);
    int top = 191;
    while (top >= 0 && !((e[top / 64] >> (top % 64)) & 1u)) --top;
    for (int b = 0; b <= top; ++b) {
        if ((e[b / 64] >> (b % 64)) & 1u) R = mul(R, B, m);
        if (b < top) B = mul(B, B, m);
    }
    return R;
}

// T[c][w][d] = A_c^(d * 16^w), d = 0 the identity.
std::vector<uint32_t> build_tables()
{
    std::vector<uint32_t> t(mrg::kTableWords);
    for (int c = 0; c < 2; ++c) {
        const uint64_t m = modulus(c);
        Mat base = companion(c);  // A^(16^w)
        for (int w = 0; w < mrg::kTableWindows; ++w) {
            Mat cur = identity();
            for (int d = 0; d < 16; ++d) {
                std::memcpy(&t[((c * mrg::kTableWindows + w) * 16 + d) * 9], cur.data(), 36);
                cur = mul(cur, base, m);
            }
            // cur = base^16 = A^(16^(w+1))
            base = cur;
        }
    }
    return t;
}

const std::vector<uint32_t> &host_tables()
{
    static const std::vector<uint32_t> t = build_tables();
    return t;
}

// ---- per-device context ----------------------------------------------------
struct DevCtx {
    uint32_t *d_table = nullptr;     // windowed jump tables
    uint32_t *d_lane_tab = nullptr;  // [kNumLaneSegs][64][18]: A^(l*L) for L in kLaneSegs
    int cus = 256;                   // compute units of the device
};

// A^(l*L) for l in [0, 64) and each lane-segment length L, both components.
std::vector<uint32_t> build_lane_tables()
{
    std::vector<uint32_t> t(mrg::kNumLaneTabs * 64 * 18);
    for (int k = 0; k < mrg::kNumLaneTabs; ++k) {
        const uint64_t L = k == mrg::kHeadTable ? 1 : (uint64_t)(16 * (k + 1));
        for (int l = 0; l < 64; ++l) {
            const uint64_t e[3] = {L * (uint64_t)l, 0, 0};
            for (int c = 0; c < 2; ++c) {
                const Mat P = power(c, e);
                std::memcpy(&t[(k * 64 + l) * 18 + 9 * c], P.data(), 36);
            }
        }
    }
    return t;
}

std::mutex g_mu;
std::map<int, DevCtx> g_dev;
mrg::FillTuning g_tune;  // process-wide kernel tuning (guarded by g_mu)

mrg::FillTuning tuning()
{
    std::lock_guard<std::mutex> lk(g_mu);
    return g_tune;
}

mrg_status current_device(int *dev)
{
    int count = 0;
    hipError_t e = hipGetDeviceCount(&count);
    if (e != hipSuccess || count <= 0) return set_error(MRG_ENODEV, "no HIP device available");
    e = hipGetDevice(dev);
    if (e != hipSuccess) return hip_error(e, "hipGetDevice");
    return MRG_OK;
}

mrg_status device_ctx(int dev, DevCtx **out)
{
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_dev.find(dev);
    if (it != g_dev.end()) {
        *out = &it->second;
        return MRG_OK;
    }
    const std::vector<uint32_t> &t = host_tables();
    DevCtx ctx;
    hipError_t e = hipMalloc(&ctx.d_table, t.size() * sizeof(uint32_t));
    if (e != hipSuccess) return set_error(MRG_ENOMEM, "hipMalloc(jump tables): %s", hipGetErrorString(e));
    e = hipMemcpy(ctx.d_table, t.data(), t.size() * sizeof(uint32_t), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        (void)hipFree(ctx.d_table);
        return hip_error(e, "hipMemcpy(jump tables)");
    }
    const std::vector<uint32_t> lt = build_lane_tables();
    e = hipMalloc(&ctx.d_lane_tab, lt.size() * sizeof(uint32_t));
    if (e != hipSuccess) {
        (void)hipFree(ctx.d_table);
        return set_error(MRG_ENOMEM, "hipMalloc(lane tables): %s", hipGetErrorString(e));
    }
    e = hipMemcpy(ctx.d_lane_tab, lt.data(), lt.size() * sizeof(uint32_t), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        (void)hipFree(ctx.d_table);
        (void)hipFree(ctx.d_lane_tab);
        return hip_error(e, "hipMemcpy(lane tables)");
    }
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
        ctx.cus = cus;
    auto res = g_dev.emplace(dev, ctx);
    *out = &res.first->second;
    return MRG_OK;
}

bool state_ok(const uint32_t *s)
{
    if (s[0] >= mrg::M1 || s[1] >= mrg::M1 || s[2] >= mrg::M1) return false;
    if (s[3] >= mrg::M2 || s[4] >= mrg::M2 || s[5] >= mrg::M2) return false;
    if ((s[0] | s[1] | s[2]) == 0u || (s[3] | s[4] | s[5]) == 0u) return false;
    return true;
}

}  // namespace

namespace mrg {

FillTuning current_tuning() { return tuning(); }

mrg_status current_device_id(int *dev) { return current_device(dev); }

mrg_status device_tables(int dev, DeviceTables *out)
{
    DevCtx *ctx;
    mrg_status st = device_ctx(dev, &ctx);
    if (st) return st;
    out->table = ctx->d_table;
    out->lane_tab = ctx->d_lane_tab;
    out->cus = ctx->cus;
    return MRG_OK;
}

mrg_status check_streamset(mrg_streamset ss)
{
    if (!ss || !ss->d_planes) return set_error(MRG_EINVAL, "null stream set");
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != ss->device)
        return set_error(MRG_EINVAL, "stream set lives on device %d, current device is %d", ss->device, dev);
    return MRG_OK;
}

mrg_status check_device_span(const void *p, uint64_t bytes, int dev, const char *what)
{
    hipPointerAttribute_t a;
    hipError_t e = hipPointerGetAttributes(&a, p);
    if (e != hipSuccess) {
        (void)hipGetLastError();  // keep the failed lookup from reaching a later launch check
        return set_error(MRG_EINVAL, "%s (%p) is not memory known to HIP: %s", what, p,
                         hipGetErrorString(e));
    }
    const bool managed = a.type == hipMemoryTypeManaged || a.isManaged;
    if (!managed && !(a.type == hipMemoryTypeDevice && a.device == dev))
        return set_error(MRG_EINVAL, "%s (%p) is not device memory of device %d (memory type %d, "
                         "device %d)", what, p, dev, (int)a.type, a.device);
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    e = hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)p);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return MRG_OK;  // no extent known: the type check above is all there is
    }
    const uint64_t off = (uint64_t)((uintptr_t)p - (uintptr_t)base);
    if (off > size || bytes > size - off)
        return set_error(MRG_ERANGE, "%s (%p, %llu bytes) extends past the end of its allocation "
                         "(%llu bytes at %p)", what, p, (unsigned long long)bytes,
                         (unsigned long long)size, (void *)base);
    return MRG_OK;
}

mrg_status check_range(mrg_streamset ss, uint64_t first, uint64_t count)
{
    if (first > ss->n || count > ss->n - first)
        return set_error(MRG_ERANGE, "streams [%llu, %llu+%llu) outside the set of %llu",
                    (unsigned long long)first, (unsigned long long)first,
                    (unsigned long long)count, (unsigned long long)ss->n);
    // one lane per stream, gridDim.x < 2^31 blocks of 64
    if (count > ((uint64_t)1 << 36))
        return set_error(MRG_ERANGE, "count %llu above the per-call limit 2^36", (unsigned long long)count);
    return MRG_OK;
}

}  // namespace mrg

namespace {

using mrg::check_range;
mrg_status check_set(mrg_streamset ss) { return mrg::check_streamset(ss); }

int bit_length(uint64_t v)
{
    int b = 0;
    while (v) { ++b; v >>= 1; }
    return b;
}

// Validated size, device context and state planes of a new stream set.
mrg_status new_streamset(uint64_t n_streams, uint64_t first_stream, mrg_streamset *out,
                         DevCtx **ctx_out)
{
    if (n_streams == 0) return set_error(MRG_ERANGE, "n_streams must be >= 1");
    if (n_streams - 1 > UINT64_MAX - first_stream)
        return set_error(MRG_ERANGE, "first_stream + n_streams exceeds 2^64");
    if (n_streams > ((uint64_t)1 << 36))
        return set_error(MRG_ERANGE, "n_streams above the limit 2^36");
    int dev;
    mrg_status st = current_device(&dev);
    if (st) return st;
    if ((st = device_ctx(dev, ctx_out))) return st;
    auto *ss = new (std::nothrow) mrg_streamset_s;
    if (!ss) return set_error(MRG_ENOMEM, "host allocation");
    ss->device = dev;
    ss->n = n_streams;
    ss->first = first_stream;
    hipError_t e = hipMalloc(&ss->d_planes, mrg::set_words(n_streams) * sizeof(uint32_t));
    if (e != hipSuccess) {
        delete ss;
        return set_error(MRG_ENOMEM, "hipMalloc(%llu states): %s", (unsigned long long)n_streams,
                         hipGetErrorString(e));
    }
    *out = ss;
    return MRG_OK;
}

// Shortest row (bytes) that the automatic stream-major fill gives to several
// lanes per stream.  A lane draws its stream in series, 60 ns a uint32 and
// 90 ns a binary64 when its wave has the SIMD to itself, so a launch of few
// streams takes that time its row length whatever it writes (64 x 1000
// uint32: 58 us; 9 us with 64 lanes per stream, the time of the call itself).
// Several lanes cost a jump per lane instead, which grows with the streams,
// and cut rows; the lane writer is at its best on lines and per byte with
// binary64.  The line (several lanes against one, us): on lines, uint32 600
// bytes for 8192 streams (512 bytes 8.5 and 7.8, 768 8.1 and 9.9), 1450 for
// 16384 (1280 17.8 and 17.1, 1536 17.9 and 19.5), 5600 for 32768 (5120 59.2 and
// 54.9, 6144 60.6 and 65.7); binary64 768, 2900 and 8192 (32768 x 256 28.4 and
// 18.9); off lines 512, 1024 and 2730 (32768 x 2052 bytes 40.0 and 35.8, 3076 47.9
// and 49.5).  From half a wave per SIMD on a whole chunk of 64 lines (49152 x
// 1000: 64 against 69 us).
uint64_t coop_min_bytes(uint64_t count, uint64_t es, bool rows_aligned, int cus)
{
    if (count > (uint64_t)cus * 128) return 64 * 128;
    const double c = (double)count / (32.0 * cus);  // 1 for 8192 streams
    double line = c <= 2 ? 512 * c : 683 * c;
    if (rows_aligned && es == 8) line = (c <= 1 ? 768 : 1024) * c * std::sqrt(c);
    else if (rows_aligned) line = c > 3.5 ? 1408 * c : (c <= 1 ? 600 : 512) * c * std::sqrt(c);
    const double least = !rows_aligned ? 384 : es == 8 ? 512 : 448;
    return (uint64_t)(line > least ? line : least);
}

// Lanes per stream of the automatic stream-major fill: as many as bring the
// launch to two waves per SIMD (64 for up to 2048 streams on 256 CUs, 32 for
// 4096, 16 for 8192; 1024 x 10000 uint32 with 64 / 32 / 16 lanes: 16.5 / 23.8
// / 38.0 us, 4096 x 3000 with 32 / 16: 21.4 / 26.6, 8192 x 1000 with 32 / 16
// / 8: 21.4 / 18.4 / 23.1).  With more streams 64 for rows of 64 KiB and
// more, 16 for shorter ones (8 when they are cut: rows under 16 KiB off
// their lines, 32768 x 1000 49 against 53 us, 49152 x 3000 160 against 175).
int coop_auto_lanes(uint64_t count, uint64_t row_bytes, bool rows_aligned, int cus)
{
    if (row_bytes >= 65536) return 64;
    const uint64_t slots = (uint64_t)cus * 8 * 64;  // lanes of two waves per SIMD
    if (count * 64 <= slots) return 64;
    if (count * 32 <= slots) return 32;
    return !rows_aligned && row_bytes < 16 * 1024 && count * 8 >= slots ? 8 : 16;
}

// A^e for both components as kernel arguments: the product of the windowed
// tables' matrices at the nonzero hexadecimal digits of e.
mrg::JumpMatrices jump_matrices(const uint64_t e[3])
{
    mrg::JumpMatrices J;
    const std::vector<uint32_t> &t = host_tables();
    for (int c = 0; c < 2; ++c) {
        Mat R = identity();
        bool any = false;
        for (int w = 0; w < mrg::kTableWindows; ++w) {
            const int d = (int)(e[w / 16] >> (4 * (w % 16))) & 15;
            if (!d) continue;
            Mat T;
            std::memcpy(T.data(), &t[((c * mrg::kTableWindows + w) * 16 + d) * 9], 36);
            R = any ? mul(R, T, modulus(c)) : T;
            any = true;
        }
        std::memcpy(J.m + 9 * c, R.data(), 36);
    }
    return J;
}

// Rows in blocks of a wave each (fill_split_kernel), by the bytes of the fill;
// the figures are of one stream in order, uint32 unless said.  Blocks are to be
// short enough to reach all SIMDs evenly, several to each, and long enough for
// their jump:
//   up to 12 MiB   8 KiB, one chunk (8 MiB 9.3 us, 16 KiB blocks 9.6)
//   up to 48 MiB   16 KiB, one chunk (27 MiB 13.7 us, 8 KiB 16.7, 32 KiB 14.0)
//   up to 192 MiB  32 KiB, two chunks (72 MB 22.9 us, 16 KiB 23.6, 64 KiB, just
//                  over one to a SIMD, 28.9; 128 MiB 29.4, 32.5 and 28.2);
//                  binary64 up to 320 MiB (260 MB 44.8 us, 64 KiB 45.2)
//   up to 320 MiB  48 KiB, three chunks (270 MB 62.5 us, 32 KiB 63.9, 64 KiB 67.3,
//                  in one chunk 68.7; 220 MB 54.3, 48.6, 54.9 and 57.9), or where
//                  the busiest SIMD then has less to draw 64 KiB in one chunk: 256
//                  uint32 per lane and start state (64 rows of 4 MiB 59.5 us, 48
//                  KiB 60.7)
//   beyond         64 KiB in one chunk, with two pieces staged per flush, half
//                  the waves and longer runs of lines (1.1 GB 204 us, with one
//                  piece 214); 128 KiB from 2 GiB on (4 GiB 763, 64 KiB 786, 2
//                  MiB 2 % more)
void split_rows(mrg::FillLaunch *fl, int cus, uint64_t set_n, uint64_t count, uint64_t n, uint64_t es)
{
    const uint64_t row = n * es, want = row / 16 * count / (uint64_t)cus;  // 16 per CU
    // bytes of the SIMD that draws most
    auto most = [&](uint64_t b) {
        const uint64_t simds = (uint64_t)cus * 4, blocks = count * ((row + b - 1) / b);
        return (blocks + simds - 1) / simds * b;
    };
    const bool large = want >= 81920;
    const uint64_t mid = es == 8 || want < 49152 ? 32768 : most(49152) < most(65536) ? 49152 : 65536;
    uint64_t bb = want < 3072 ? 8192 : want < 12288 ? 16384 : !large ? mid : want < 524288 ? 65536 : 131072;
    const uint64_t unit = want < 3072 ? 8192 : bb >= 65536 ? 65536 : 16384;  // a chunk of 64 lanes
    // fewer blocks than 2^32 per row, and than 2^31 workgroups in all
    while (row / bb >= ((uint64_t)1 << 31) / count) bb *= 2;
    fl->kernel = 2;
    fl->L = (int)(unit / 64 / es);
    fl->pieces = large ? 2 : 1;
    fl->B = bb / es;
    // a remainder under an eighth of a block goes to the last block
    fl->nblk = (uint32_t)(n / fl->B + (n % fl->B > fl->B / 8 || n < fl->B));
    fl->grid = (unsigned)(count * fl->nblk);
    const uint64_t e[3] = {n, 0, 0};
    fl->end = jump_matrices(e);
    fl->move = mrg::parts_move(set_n, count, fl->nblk, false);
}

// Interleaved fill in segments of each stream (fill_il_seg_kernel): as many as
// bring the launch to two waves of lanes per SIMD (one for binary64, whose
// stores fill the memory with half the lanes), of at least 64 steps.  A lane
// draws 42-50 ns a step in series, so few streams take that time their steps
// whatever they write (64 x 1000 float32 50 -> 9.5 us, 4096 x 16384 795 -> 62,
// 32768 x 4096 206 -> 116); four waves per SIMD were slower for 1024 to 4096
// streams (4096 x 4096 26.6 against 23.0 us, eight 33.6), segments of 32
// steps no faster, and 65536 binary64 streams in two segments slower (x 1000
// 98.6 -> 105 us).
//
// Segments write as many places at once, which the memory takes worse the more
// streams there are and the more their rows share lines, so with many streams
// the segments have to pay for it.  uint32, up to half a wave of streams per
// SIMD they do (32768 x 4096 184 -> 100 us on lines, 168 -> 155 off them); up
// to 40960 on lines and from 192 steps on (36000 x 1000 46 -> 34; off lines
// x 4096 171 -> 197, x 128 9.2 -> 9.9), off lines up to 38912 for 192 to 800
// steps (38900 x 800 0.92 times, x 1000 1.10) and up to 43008 for 192 to 600
// (42788 x 512 28.1 -> 21.2, 45000 x 512 0.99 times); beyond, only near a wave
// per SIMD, on lines and for long fills (65536 x 1000 53 -> 51, off lines 72 ->
// 76; 52000 x 4096 1.04 times).  binary64: up to 18432 always (18001 x 4096 off lines 0.92
// times, 20001 1.02, 24000 x 1000 47 -> 52), up to 28672 on lines (28000 x 4096
// 0.97 times, 30000 1.04), up to 32768 for short fills (x 512 0.90 times).
bool steps_cut(int cus, uint64_t count, uint64_t n, uint64_t es, bool lined)
{
    const uint64_t c = (uint64_t)cus;
    if (es == 4)
        return count <= c * 128 || (n >= 192 && n <= 600 && count <= c * 168) ||
               (n >= 192 && (lined ? count <= c * 160 : n <= 800 && count <= c * 152)) ||
               (lined && n >= 1000 && count >= c * 224);
    return count <= c * 72 || (count <= c * 128 && (n <= 512 || (lined && (n < 1000 || count <= c * 112))));
}

void split_steps(mrg::FillLaunch *fl, int cus, uint64_t set_n, uint64_t count, uint64_t n, uint64_t es,
                 bool lined)
{
    if (!steps_cut(cus, count, n, es, lined)) return;
    const uint64_t lanes = (uint64_t)cus * 2048 / es;
    uint64_t nseg = lanes / count;
    if (nseg > n / 64) nseg = n / 64;
    if (nseg < 2) return;
    fl->B = ((n + nseg - 1) / nseg + 15) / 16 * 16;
    fl->nblk = (uint32_t)((n + fl->B - 1) / fl->B);
    if (fl->nblk < 2) return;
    fl->kernel = 3;
    const uint64_t e[3] = {n, 0, 0};
    fl->end = jump_matrices(e);
    fl->move = mrg::parts_move(set_n, count, fl->nblk, true);
}

// How an MRG32k3a fill is launched under `tune` on a device of `cus` compute
// units (the tables' addresses apart).  *layout becomes stream-major where one
// stream is drawn in order.
mrg::FillLaunch plan_fill(const mrg::FillTuning &tune, int cus, uint64_t set_n, uint64_t count,
                          uint64_t n_per_stream, uint64_t es, mrg_layout *layout, uintptr_t out)
{
    mrg::FillLaunch fl;
    // one stream: both layouts are its values in a row
    if (count == 1 && tune.strategy == 0) *layout = MRG_STREAM_MAJOR;
    if (*layout == MRG_STREAM_MAJOR) {
        // several lanes per stream (or when forced) for rows from coop_min_bytes
        // on (see below for rows under 16 KiB); lane per stream for the others
        const bool rows_aligned = out % 128 == 0 && (n_per_stream * es) % 128 == 0;
        const bool coop =
            tune.strategy == 2 || (tune.strategy == 0 && n_per_stream * es >=
                                                             coop_min_bytes(count, es, rows_aligned, cus));
        if (coop) {
            // GL lanes per stream, 64/GL streams per wave; each lane takes
            // 64/GL or 2*64/GL pieces of 128 bytes per chunk (a chunk is then
            // 64 or 128 lines), whichever generates fewer values past the end
            // of a row (the longer chunk on a tie).  A row's line-aligned
            // part is n values, or about n - tv/2 when rows start anywhere.
            const int GL = tune.coop_lanes ? tune.coop_lanes
                                           : coop_auto_lanes(count, n_per_stream * es, rows_aligned, cus);
            const uint64_t tv = 128 / es;
            const uint64_t nh_min = 64 / GL, nh_max = 2 * nh_min;
            const uint64_t body = rows_aligned || n_per_stream <= tv ? n_per_stream : n_per_stream - tv / 2;
            const uint64_t ch_min = (uint64_t)GL * nh_min * tv, ch_max = 2 * ch_min;
            const uint64_t gen_min = (body + ch_min - 1) / ch_min * ch_min;
            const uint64_t gen_max = (body + ch_max - 1) / ch_max * ch_max;
            const uint64_t nh = gen_max <= gen_min ? nh_max : nh_min;
            const int L = (int)(nh * tv);
            fl.kernel = 1;
            fl.L = L;
            fl.lanes = GL;
            // resident workgroups stride over the stream groups, or one per group
            const uint64_t groups = (count + (64 / GL) - 1) / (64 / GL);
            const uint64_t cap = tune.coop_wgs_per_cu ? (uint64_t)cus * tune.coop_wgs_per_cu
                                                      : ((uint64_t)1 << 31) - 1;
            fl.grid = (unsigned)(groups < cap ? groups : cap);
            fl.order = tune.coop_order;
            // the bulk case: rows on lines, whole chunks, a group's rows
            // addressable with 32-bit offsets
            fl.whole = rows_aligned && n_per_stream % ((uint64_t)GL * L) == 0 &&
                       (uint64_t)(64 / GL) * n_per_stream * es < ((uint64_t)1 << 32);
            // automatic choice: a row under 16 KiB that is not whole chunks on
            // lines is one cut chunk for this writer (values drawn past the
            // row's end, one piece per flush), and with enough streams for one
            // wave of them on every SIMD (2^16 on 256 CUs) the lane-per-stream
            // writer is the faster one (uint32 rows of 3000: 190 us against
            // 210-235 for 2^16 streams, 4.0-4.5 against 3.4 TB/s for 2^17 and
            // more; of 4000: 228 against 264-276 us, 4.2-4.4 against 3.6-3.7
            // TB/s; from 4500 values this writer leads, 4.7-4.8 against
            // 4.0-4.5).  With fewer streams this writer keeps the launch short
            // (49152 x 3000: 160 against 177 us).
            if (tune.strategy == 0 && !fl.whole && n_per_stream * es < 16 * 1024 &&
                count >= (uint64_t)cus * 256)
                fl = mrg::FillLaunch();
        }
        // lane per stream, rows of whole 4 KiB on lines: two lanes per stream
        // (fill_sm_kernel's HALVES: float32 rows of 4 KiB 65536 80 -> 59 us, 262144
        // 306 -> 226; of 12 KiB, from 65536 on in lanes, 240 -> 171 and 730 -> 682,
        // at 131072 367 and 365, binary64 187 -> 157 and 637 -> 615; rows of 8 KiB
        // are whole chunks of the wave writer.  Other row lengths lose by it:
        // 131072 x 1536 float32 171 -> 189 us, x 512 59 -> 62)
        if (tune.strategy == 0 && fl.kernel == 0 && tune.tile_bytes == 0 &&
            out % 128 == 0 && n_per_stream * es % 4096 == 0) {
            fl.kernel = 4;
            const uint64_t e[3] = {n_per_stream / 2, 0, 0};
            fl.end = jump_matrices(e);
        }
        // few streams: a wave per stream leaves the chip idle and takes 2.3 us
        // per 4096 uint32 of a row whatever the launch writes, so rows are cut
        // into blocks (256 x 16384 uint32 13.8 -> 8.9 us, 64 x 2^20 730 -> 58).
        // With two waves or more per CU the rows have to be long enough for the
        // blocks' jumps (512 x 10000 15.7 -> 16.9, 512 x 40000 33.7 -> 23.1),
        // and with a wave per SIMD the rows alone fill the chip (1000 x 65536
        // 50 -> 56).  A key of the wave-per-stream writer that is set keeps it.
        const bool asked = tune.coop_lanes || tune.coop_wgs_per_cu || tune.coop_order;
        if (tune.strategy == 0 && !asked &&
            ((count <= (uint64_t)cus && n_per_stream * es >= 16 * 1024) ||
             (count <= (uint64_t)cus * 2 && n_per_stream * es >= 64 * 1024))) {
            fl = mrg::FillLaunch();
            split_rows(&fl, cus, set_n, count, n_per_stream, es);
        }
    }
    if (*layout == MRG_INTERLEAVED && tune.strategy == 0)
        split_steps(&fl, cus, set_n, count, n_per_stream, es,
                    out % 128 == 0 && count * es % 128 == 0);
    return fl;
}

// How a deal is launched: true for one drawn in order (fl: the stream as one
// row in blocks), else A.
bool plan_leap(int cus, uint64_t set_n, uint64_t players, uint64_t per_player, uint64_t es,
               mrg_layout layout, mrg::FillLaunch *fl, mrg::LeapArgs *leap)
{
    const uint64_t N = players * per_player;
    const uint64_t en[3] = {N, 0, 0};
    // with one player or one card per player both layouts are the stream in order
    if (layout == MRG_INTERLEAVED || players == 1 || per_player == 1) {
        split_rows(fl, cus, set_n, 1, N, es);
        return true;
    }
    mrg::LeapArgs &A = *leap;
    // each player's cards in a row: items of KB = min(K, 64) card columns
    // x T players (R = 64 / KB lanes per column, Ts = T / R players
    // each), T chosen for about 4 items per resident wave, with at least 64
    // players per lane, 32 where that leaves four waves per CU or fewer (65536 x
    // 52: with 256 18.4 us, with 64, a wave on each SIMD, 11.5, with 32 10.3, with
    // 16 14.0; 70400 x 52 has more, 32 loses 2 %).  While the items at 64
    // players do not fill the chip, and for up to 4096 cards, up to 16 waves to a
    // workgroup, which count themselves in together, and the stream moved in the
    // kernel (4096 x 4096 float64 31.7 us against 39.9 with a wave to a workgroup
    // and a launch; 8192 x 2048 26.6 and 32.3; 65536 x 1024 52.6 and 55.3); beyond,
    // a wave to a workgroup, since the waves of one share a CU and write far
    // apart, and a launch for the stream (65536 x 8000 uint32 439 us, in groups of
    // 16 475; 8192 x 6000 43.4 and 45.8).  Over 218 deals of 1 MB to 2 GB these
    // rules take 1.03 times the best of 32 to 256 players per lane in groups of
    // 1, 4 and 16 waves, 32 players and 16 waves for all 1.04.
    const uint64_t slots = (uint64_t)cus * 16;  // resident waves
    A.P = players;
    A.K = per_player;
    A.KB = (int)(per_player < 64 ? per_player : 64);
    A.R = 64 / A.KB;
    const uint64_t nkb = (per_player + A.KB - 1) / A.KB;
    const uint64_t target = 4 * slots;
    const uint64_t ts_max = (players + A.R - 1) / A.R;
    const uint64_t at64 = nkb * ((ts_max + 63) / 64);
    const bool grouped = at64 < (uint64_t)cus * 15 || per_player <= 4096;
    const uint64_t ts_min = at64 <= (uint64_t)cus * 4 ? 32 : 64;
    uint64_t Ts = ts_max;
    if (nkb < target) {
        const uint64_t segs = (target + nkb - 1) / nkb;
        Ts = (players + segs * A.R - 1) / (segs * A.R);
        if (Ts < ts_min) Ts = ts_min;
    }
    if (Ts > ts_max) Ts = ts_max;
    // few segments are even ones, no shorter than 64 (76 players as 64 and 12 took
    // 17.9 us, whole 16.0) and no longer than 32 (114 as 3 x 38 10.3 us, 4 x 29 8.5)
    if (const uint64_t nseg = ts_min == 64 ? ts_max / Ts : (ts_max + Ts - 1) / Ts; nseg < 8)
        Ts = (ts_max + nseg - 1) / nseg;
    A.Ts = Ts;
    A.T = Ts * A.R;
    A.nseg = (players + A.T - 1) / A.T;
    A.items = nkb * A.nseg;
    // 63 * players and T - Ts as 192-bit exponents
    const unsigned __int128 e63 = (unsigned __int128)players * 63u;
    const uint64_t ew[3] = {(uint64_t)e63, (uint64_t)(e63 >> 64), 0};
    A.J63 = jump_matrices(ew);
    const uint64_t es_[3] = {A.T - A.Ts, 0, 0};
    A.Jseg = jump_matrices(es_);
    A.end = jump_matrices(en);  // the stream moves past the N outputs dealt
    // up to 16 waves a workgroup, for at most 256 arrivals at the ticket
    A.waves = (unsigned)(A.items < slots ? A.items : slots);
    A.per_group = !grouped || A.waves <= 256 ? 1 : A.waves >= 4096 ? 16 : (A.waves + 255) / 256;
    A.move = grouped && mrg::ticket_pitch(set_n);
    return false;
}

// The fill planned in fl and, when it cuts streams into parts that do not move
// them, their jump.
hipError_t run_fill(mrg_streamset ss, const DevCtx *ctx, mrg::FillLaunch fl,
                    const mrg::FillTuning &tune, uint64_t first, uint64_t count, uint64_t n,
                    mrg_dtype dtype, mrg_layout layout, void *d_out, hipStream_t st)
{
    fl.tabs = ctx->d_lane_tab;
    fl.lane_tab = ctx->d_lane_tab + (fl.L ? mrg::lane_table(fl.L) * 64 * 18 : 0);
    fl.table = ctx->d_table;
    hipError_t e = mrg::launch_fill(ss->d_planes, ss->n, first, count, n, (int)dtype, (int)layout,
                                    d_out, fl, tune, st);
    if (e == hipSuccess && (fl.kernel == 2 || fl.kernel == 3) && !fl.move)
        e = mrg::launch_jump_uniform(ss->d_planes, ss->n, first, count, fl.end, st);
    return e;
}

}  // namespace

extern "C" {

mrg_status mrg_seed_from_master(uint64_t master_seed, uint32_t out6[6])
{
    if (!out6) return set_error(MRG_EINVAL, "null output");
    mrg::expand_seed(master_seed, out6);
    return MRG_OK;
}

mrg_status mrg_jump_matrix(int component, const uint64_t h_exp[3], uint32_t out9[9])
{
    if (!h_exp || !out9) return set_error(MRG_EINVAL, "null argument");
    if (component != 0 && component != 1) return set_error(MRG_EINVAL, "component must be 0 or 1");
    const Mat R = power(component, h_exp);
    std::memcpy(out9, R.data(), 36);
    return MRG_OK;
}

mrg_status mrg_state_check(const uint32_t state6[6])
{
    if (!state6) return set_error(MRG_EINVAL, "null state");
    if (!state_ok(state6)) return set_error(MRG_EINVAL, "invalid MRG32k3a state");
    return MRG_OK;
}

mrg_status mrg_streamset_create(mrg_streamset *out, uint64_t n_streams, uint64_t first_stream,
                                const uint32_t seed6[6], void *stream)
{
    if (!out || !seed6) return set_error(MRG_EINVAL, "null argument");
    *out = nullptr;
    if (!state_ok(seed6)) return set_error(MRG_EINVAL, "invalid seed state");
    mrg_streamset ss;
    DevCtx *ctx;
    mrg_status st = new_streamset(n_streams, first_stream, &ss, &ctx);
    if (st) return st;
    std::memcpy(ss->seed, seed6, sizeof ss->seed);
    // exponent g * 2^127 uses bits 127 .. 126 + bit_length(g): windows 31 ..
    const uint64_t g_max = first_stream + (n_streams - 1);
    const int top_bit = 126 + bit_length(g_max);  // highest set bit of g_max * 2^127
    const int w_lo = 31, w_hi = g_max ? top_bit / 4 + 1 : 31;
    mrg::InitSeed sd;
    std::memcpy(sd.w, seed6, sizeof sd.w);
    hipError_t e = mrg::launch_init(ss->d_planes, n_streams, n_streams, first_stream, sd,
                                    ctx->d_table, w_lo, w_hi, (hipStream_t)stream);
    if (e != hipSuccess) {
        (void)hipFree(ss->d_planes);
        delete ss;
        return hip_error(e, "init kernel launch");
    }
    *out = ss;
    return MRG_OK;
}

mrg_status mrg_streamset_create_seed64(mrg_streamset *out, uint64_t n_streams,
                                       uint64_t first_stream, uint64_t master_seed, void *stream)
{
    uint32_t s[6];
    mrg_status st = mrg_seed_from_master(master_seed, s);
    if (st) return st;
    return mrg_streamset_create(out, n_streams, first_stream, s, stream);
}

mrg_status mrg_streamset_create_random(mrg_streamset *out, uint64_t n_streams,
                                       uint64_t first_stream, uint64_t master_seed, void *stream)
{
    if (!out) return set_error(MRG_EINVAL, "null argument");
    *out = nullptr;
    mrg_streamset ss;
    DevCtx *ctx;
    mrg_status st = new_streamset(n_streams, first_stream, &ss, &ctx);
    if (st) return st;
    // no common base state: info reports all zeros
    hipError_t e = mrg::launch_random_init(ss->d_planes, n_streams, n_streams, first_stream,
                                           master_seed, (hipStream_t)stream);
    if (e != hipSuccess) {
        (void)hipFree(ss->d_planes);
        delete ss;
        return hip_error(e, "random init kernel launch");
    }
    *out = ss;
    return MRG_OK;
}

mrg_status mrg_streamset_create_philox(mrg_streamset *out, uint64_t n_streams,
                                       uint64_t first_stream, uint64_t key, void *stream)
{
    if (!out) return set_error(MRG_EINVAL, "null argument");
    *out = nullptr;
    mrg_streamset ss;
    DevCtx *ctx;
    mrg_status st = new_streamset(n_streams, first_stream, &ss, &ctx);
    if (st) return st;
    ss->gen = 1;
    hipError_t e = mrg::launch_philox_init(ss->d_planes, n_streams, n_streams, first_stream, key,
                                           (hipStream_t)stream);
    if (e != hipSuccess) {
        (void)hipFree(ss->d_planes);
        delete ss;
        return hip_error(e, "philox init kernel launch");
    }
    *out = ss;
    return MRG_OK;
}

mrg_status mrg_streamset_destroy(mrg_streamset ss)
{
    if (!ss) return MRG_OK;
    mrg_status st = MRG_OK;
    if (ss->d_planes) {
        int prev = -1;
        (void)hipGetDevice(&prev);
        if (prev != ss->device) (void)hipSetDevice(ss->device);
        hipError_t e = hipDeviceSynchronize();
        if (e != hipSuccess) st = hip_error(e, "hipDeviceSynchronize before free");
        e = hipFree(ss->d_planes);
        if (e != hipSuccess && st == MRG_OK) st = hip_error(e, "hipFree(states)");
        if (ss->d_records) {
            e = hipFree(ss->d_records);
            if (e != hipSuccess && st == MRG_OK) st = hip_error(e, "hipFree(parameter records)");
        }
        if (prev != ss->device && prev >= 0) (void)hipSetDevice(prev);
    }
    delete ss;
    return st;
}

mrg_status mrg_streamset_info(mrg_streamset ss, uint64_t *n_streams, uint64_t *first_stream,
                              uint32_t seed6[6])
{
    if (!ss) return set_error(MRG_EINVAL, "null stream set");
    if (n_streams) *n_streams = ss->n;
    if (first_stream) *first_stream = ss->first;
    if (seed6) std::memcpy(seed6, ss->seed, sizeof ss->seed);
    return MRG_OK;
}

mrg_status mrg_streamset_states_ptr(mrg_streamset ss, void **d_states)
{
    if (!ss || !d_states) return set_error(MRG_EINVAL, "null argument");
    *d_states = ss->d_planes;
    return MRG_OK;
}

mrg_status mrg_streamset_tables_ptr(mrg_streamset ss, const void **d_tables)
{
    mrg_status st = check_set(ss);
    if (st) return st;
    if (!d_tables) return set_error(MRG_EINVAL, "null argument");
    DevCtx *ctx;
    if ((st = device_ctx(ss->device, &ctx))) return st;
    *d_tables = ctx->d_table;
    return MRG_OK;
}

mrg_status mrg_jump(mrg_streamset ss, uint64_t first, uint64_t count, const uint64_t *d_exp,
                    void *stream)
{
    mrg_status st = check_set(ss);
    if (st) return st;
    if ((st = check_range(ss, first, count))) return st;
    if (count == 0) return MRG_OK;
    if (!d_exp) return set_error(MRG_EINVAL, "null exponent array");
    if ((st = mrg::check_device_span(d_exp, 24 * count, ss->device, "exponent array"))) return st;
    if (ss->gen == mrg::kGenPhilox) {  // the position moves by e mod 2^64
        hipError_t e = mrg::launch_philox_jump(ss->d_planes, ss->n, first, count, d_exp, 0,
                                               (hipStream_t)stream);
        return e == hipSuccess ? MRG_OK : hip_error(e, "jump kernel launch");
    }
    if (ss->gen == mrg::kGenTinyMT) {
        const uint64_t none[3] = {0, 0, 0};
        hipError_t e = mrg::launch_tmt_jump(ss->d_planes, ss->n, first, count, d_exp, none,
                                            ss->d_records, ss->q0, (hipStream_t)stream);
        return e == hipSuccess ? MRG_OK : hip_error(e, "jump kernel launch");
    }
    DevCtx *ctx;
    if ((st = device_ctx(ss->device, &ctx))) return st;
    hipError_t e = mrg::launch_jump(ss->d_planes, ss->n, first, count, d_exp, ctx->d_table,
                                    (hipStream_t)stream);
    return e == hipSuccess ? MRG_OK : hip_error(e, "jump kernel launch");
}

mrg_status mrg_jump_uniform(mrg_streamset ss, uint64_t first, uint64_t count,
                            const uint64_t h_exp[3], void *stream)
{
    mrg_status st = check_set(ss);
    if (st) return st;
    if ((st = check_range(ss, first, count))) return st;
    if (!h_exp) return set_error(MRG_EINVAL, "null exponent");
    if (count == 0) return MRG_OK;
    if (ss->gen == mrg::kGenPhilox) {
        hipError_t e = mrg::launch_philox_jump(ss->d_planes, ss->n, first, count, nullptr,
                                               h_exp[0], (hipStream_t)stream);
        return e == hipSuccess ? MRG_OK : hip_error(e, "jump kernel launch");
    }
    if (ss->gen == mrg::kGenTinyMT) {
        hipError_t e = mrg::launch_tmt_jump(ss->d_planes, ss->n, first, count, nullptr, h_exp,
                                            ss->d_records, ss->q0, (hipStream_t)stream);
        return e == hipSuccess ? MRG_OK : hip_error(e, "jump kernel launch");
    }
    hipError_t e = mrg::launch_jump_uniform(ss->d_planes, ss->n, first, count,
                                            jump_matrices(h_exp), (hipStream_t)stream);
    return e == hipSuccess ? MRG_OK : hip_error(e, "jump kernel launch");
}

mrg_status mrg_jump_substreams(mrg_streamset ss, uint64_t first, uint64_t count, uint64_t k,
                               void *stream)
{
    if (ss && ss->gen != mrg::kGenMRG)
        return set_error(MRG_EINVAL, "substreams are defined for MRG32k3a stream sets only");
    // k * 2^76 = (k << 12) * 2^64 + (k >> 52) * 2^128
    const uint64_t e[3] = {0, k << 12, k >> 52};
    return mrg_jump_uniform(ss, first, count, e, stream);
}

mrg_status mrg_fill(mrg_streamset ss, uint64_t first, uint64_t count, uint64_t n_per_stream,
                    mrg_dtype dtype, mrg_layout layout, void *d_out, void *stream)
{
    mrg_status st = check_set(ss);
    if (st) return st;
    if ((st = check_range(ss, first, count))) return st;
    if (dtype != MRG_U32 && dtype != MRG_F32 && dtype != MRG_F64)
        return set_error(MRG_EINVAL, "unknown dtype %d", (int)dtype);
    if (layout != MRG_STREAM_MAJOR && layout != MRG_INTERLEAVED)
        return set_error(MRG_EINVAL, "unknown layout %d", (int)layout);
    if (count == 0 || n_per_stream == 0) return MRG_OK;
    if (!d_out) return set_error(MRG_EINVAL, "null output");
    const uint64_t es = dtype == MRG_F64 ? 8 : 4;
    if ((uintptr_t)d_out % es) return set_error(MRG_EINVAL, "output not aligned to its element size");
    if (n_per_stream > UINT64_MAX / es / count)
        return set_error(MRG_ERANGE, "output size overflows 64 bits");
    if ((st = mrg::check_device_span(d_out, count * n_per_stream * es, ss->device, "output")))
        return st;
    if (ss->gen == mrg::kGenPhilox) {
        DevCtx *ctx;
        if ((st = device_ctx(ss->device, &ctx))) return st;
        hipError_t e = mrg::launch_philox_fill(ss->d_planes, ss->n, first, count, n_per_stream,
                                               (int)dtype, (int)layout, ctx->cus, d_out,
                                               (hipStream_t)stream);
        return e == hipSuccess ? MRG_OK : hip_error(e, "philox fill kernel launch");
    }
    const mrg::FillTuning tune = tuning();
    if (ss->gen == mrg::kGenTinyMT) {
        hipError_t e = mrg::launch_tmt_fill(ss->d_planes, ss->n, first, count, n_per_stream,
                                            (int)dtype, (int)layout, d_out, ss->d_records, ss->q0,
                                            tune.tile_bytes, (hipStream_t)stream);
        return e == hipSuccess ? MRG_OK : hip_error(e, "tinymt fill kernel launch");
    }
    DevCtx *ctx;
    if ((st = device_ctx(ss->device, &ctx))) return st;
    const mrg::FillLaunch fl = plan_fill(tune, ctx->cus, ss->n, count, n_per_stream, es, &layout,
                                         (uintptr_t)d_out);
    hipError_t e = run_fill(ss, ctx, fl, tune, first, count, n_per_stream, dtype, layout, d_out,
                            (hipStream_t)stream);
    return e == hipSuccess ? MRG_OK : hip_error(e, "fill kernel launch");
}

mrg_status mrg_fill_leapfrog(mrg_streamset ss, uint64_t s, uint64_t players,
                             uint64_t per_player, mrg_dtype dtype, mrg_layout layout,
                             void *d_out, void *stream)
{
    mrg_status st = check_set(ss);
    if (st) return st;
    if ((st = check_range(ss, s, 1))) return st;
    if (dtype != MRG_U32 && dtype != MRG_F32 && dtype != MRG_F64)
        return set_error(MRG_EINVAL, "unknown dtype %d", (int)dtype);
    if (layout != MRG_STREAM_MAJOR && layout != MRG_INTERLEAVED)
        return set_error(MRG_EINVAL, "unknown layout %d", (int)layout);
    if (ss->gen != mrg::kGenMRG)
        return set_error(MRG_EINVAL, "leapfrog is defined for MRG32k3a stream sets only");
    if (players == 0 || per_player == 0) return MRG_OK;
    if (!d_out) return set_error(MRG_EINVAL, "null output");
    const uint64_t es = dtype == MRG_F64 ? 8 : 4;
    if ((uintptr_t)d_out % es) return set_error(MRG_EINVAL, "output not aligned to its element size");
    if (players > UINT64_MAX / per_player || players * per_player > UINT64_MAX / es)
        return set_error(MRG_ERANGE, "players * per_player * element size overflows 64 bits");
    const uint64_t N = players * per_player;
    if ((st = mrg::check_device_span(d_out, N * es, ss->device, "output"))) return st;
    DevCtx *ctx;
    if ((st = device_ctx(ss->device, &ctx))) return st;
    const mrg::FillTuning tune = tuning();
    mrg::LeapArgs A;
    mrg::FillLaunch fl;
    if (plan_leap(ctx->cus, ss->n, players, per_player, es, layout, &fl, &A)) {
        // the stream's outputs in order: one row in blocks
        hipError_t e = run_fill(ss, ctx, fl, tune, s, 1, N, dtype, MRG_STREAM_MAJOR, d_out,
                                (hipStream_t)stream);
        return e == hipSuccess ? MRG_OK : hip_error(e, "leapfrog kernel launch");
    }
    hipError_t e = mrg::launch_leap(ss->d_planes, ss->n, s, (int)dtype, A, ctx->d_table, d_out,
                                    tune.engine, (hipStream_t)stream);
    if (e == hipSuccess && !A.move)
        e = mrg::launch_jump_uniform(ss->d_planes, ss->n, s, 1, A.end, (hipStream_t)stream);
    return e == hipSuccess ? MRG_OK : hip_error(e, "leapfrog kernel launch");
}

mrg_status mrg_fill_route(uint64_t set_streams, uint64_t count, uint64_t n_per_stream,
                          mrg_dtype dtype, mrg_layout layout, uint64_t out_offset, int32_t cus,
                          mrg_route *route)
{
    if (!route) return set_error(MRG_EINVAL, "null argument");
    if (!count || !n_per_stream || count > set_streams || cus < 1)
        return set_error(MRG_ERANGE, "no such fill");
    const uint64_t es = dtype == MRG_F64 ? 8 : 4;
    const mrg::FillLaunch fl = plan_fill(tuning(), cus, set_streams, count, n_per_stream, es,
                                         &layout, (uintptr_t)out_offset);
    *route = mrg_route();
    route->kernel = layout == MRG_INTERLEAVED && fl.kernel != 3 ? MRG_ROUTE_STEPS : fl.kernel;
    const bool parts = fl.kernel == 2 || fl.kernel == 3;
    route->lanes = fl.kernel == 1 ? fl.lanes : fl.kernel == 2 ? 64 : fl.kernel == 4 ? 2 : 1;
    route->parts = parts ? fl.nblk : 1;
    route->part_values = parts ? fl.B : n_per_stream;
    route->chunk_values = fl.kernel == 1 || fl.kernel == 2 ? (uint32_t)(fl.L * route->lanes) : 0;
    route->moves = !parts || fl.move;
    return MRG_OK;
}

mrg_status mrg_leapfrog_route(uint64_t set_streams, uint64_t players, uint64_t per_player,
                              mrg_dtype dtype, mrg_layout layout, int32_t cus, mrg_route *route)
{
    if (!route) return set_error(MRG_EINVAL, "null argument");
    if (!players || !per_player || !set_streams || cus < 1) return set_error(MRG_ERANGE, "no such deal");
    mrg::LeapArgs A;
    mrg::FillLaunch fl;
    *route = mrg_route();
    if (plan_leap(cus, set_streams, players, per_player, dtype == MRG_F64 ? 8 : 4, layout, &fl, &A)) {
        route->kernel = fl.kernel;
        route->lanes = 64;
        route->parts = fl.nblk;
        route->part_values = fl.B;
        route->chunk_values = (uint32_t)(fl.L * 64);
        route->moves = fl.move;
    } else {
        route->kernel = MRG_ROUTE_DEAL;
        route->lanes = A.KB * A.R;
        route->parts = A.items;
        route->part_values = A.Ts;
        route->waves = A.waves;
        route->waves_per_group = A.per_group;
        route->moves = A.move;
    }
    return MRG_OK;
}

mrg_status mrg_get_states(mrg_streamset ss, uint64_t first, uint64_t count, uint32_t *h_out,
                          void *stream)
{
    mrg_status st = check_set(ss);
    if (st) return st;
    if ((st = check_range(ss, first, count))) return st;
    if (count == 0) return MRG_OK;
    if (!h_out) return set_error(MRG_EINVAL, "null output");
    std::vector<uint32_t> tmp(6 * count);
    for (int c = 0; c < 6; ++c) {
        hipError_t e = hipMemcpyAsync(tmp.data() + c * count, ss->d_planes + c * ss->n + first,
                                      count * 4, hipMemcpyDeviceToHost, (hipStream_t)stream);
        if (e != hipSuccess) return hip_error(e, "hipMemcpyAsync(states)");
    }
    hipError_t e = hipStreamSynchronize((hipStream_t)stream);
    if (e != hipSuccess) return hip_error(e, "hipStreamSynchronize");
    for (uint64_t i = 0; i < count; ++i)
        for (int c = 0; c < 6; ++c) h_out[6 * i + c] = tmp[c * count + i];
    return MRG_OK;
}

mrg_status mrg_set_states(mrg_streamset ss, uint64_t first, uint64_t count, const uint32_t *h_in,
                          void *stream)
{
    mrg_status st = check_set(ss);
    if (st) return st;
    if ((st = check_range(ss, first, count))) return st;
    if (count == 0) return MRG_OK;
    if (!h_in) return set_error(MRG_EINVAL, "null input");
    for (uint64_t i = 0; ss->gen == mrg::kGenMRG && i < count; ++i)  // any 6 words are a Philox state
        if (!state_ok(h_in + 6 * i))
            return set_error(MRG_EINVAL, "state %llu is not a valid MRG32k3a state",
                        (unsigned long long)i);
    for (uint64_t i = 0; ss->gen == mrg::kGenTinyMT && i < count; ++i) {
        // a TinyMT state: nonzero 127-bit part, a parameter set of this set
        // (the one its stream was created with), word 5 zero
        const uint32_t *w = h_in + 6 * i;
        const uint64_t q_want = (ss->first + first + i) / ss->per_param;
        if (((w[0] & 0x7fffffffu) | w[1] | w[2] | w[3]) == 0u || w[4] != q_want || w[5] != 0u)
            return set_error(MRG_EINVAL, "state %llu is not a TinyMT32 state of its stream "
                             "(nonzero state, parameter set %llu, last word 0)",
                             (unsigned long long)i, (unsigned long long)q_want);
    }
    std::vector<uint32_t> tmp(6 * count);
    for (uint64_t i = 0; i < count; ++i)
        for (int c = 0; c < 6; ++c) tmp[c * count + i] = h_in[6 * i + c];
    for (int c = 0; c < 6; ++c) {
        hipError_t e = hipMemcpyAsync(ss->d_planes + c * ss->n + first, tmp.data() + c * count,
                                      count * 4, hipMemcpyHostToDevice, (hipStream_t)stream);
        if (e != hipSuccess) return hip_error(e, "hipMemcpyAsync(states)");
    }
    hipError_t e = hipSuccess;
    if (ss->gen != mrg::kGenTinyMT)  // its fills have no parts
        e = mrg::launch_ticket_reset(ss->d_planes, ss->n, first, count, (hipStream_t)stream);
    if (e != hipSuccess) return hip_error(e, "ticket reset launch");
    e = hipStreamSynchronize((hipStream_t)stream);
    return e == hipSuccess ? MRG_OK : hip_error(e, "hipStreamSynchronize");
}

mrg_status mrg_config_set(const char *key, int64_t value)
{
    if (!key) return set_error(MRG_EINVAL, "null key");
    std::lock_guard<std::mutex> lk(g_mu);
    if (!std::strcmp(key, "engine")) {
        if (value != 0 && value != 1) return set_error(MRG_EINVAL, "engine must be 0 or 1");
        g_tune.engine = (int)value;
    } else if (!std::strcmp(key, "coop_order")) {
        if (value != 0 && value != 1) return set_error(MRG_EINVAL, "coop_order must be 0 or 1");
        g_tune.coop_order = (int)value;
    } else if (!std::strcmp(key, "coop_wgs_per_cu")) {
        if (value < 0 || value > 1024) return set_error(MRG_EINVAL, "coop_wgs_per_cu must be in [0, 1024]");
        g_tune.coop_wgs_per_cu = (int)value;
    } else if (!std::strcmp(key, "coop_lanes")) {
        if (value != 64 && value != 32 && value != 16 && value != 8 && value != 0)
            return set_error(MRG_EINVAL, "coop_lanes must be 0, 64, 32, 16 or 8");
        g_tune.coop_lanes = (int)value;
    } else if (!std::strcmp(key, "strategy")) {
        if (value < 0 || value > 2) return set_error(MRG_EINVAL, "strategy must be 0, 1 or 2");
        g_tune.strategy = (int)value;
    } else if (!std::strcmp(key, "tile_bytes")) {
        if (value != 0 && value != 128 && value != 256)
            return set_error(MRG_EINVAL, "tile_bytes must be 0 (automatic), 128 or 256");
        g_tune.tile_bytes = (int)value;
    } else {
        return set_error(MRG_EINVAL, "unknown key '%s'", key);
    }
    return MRG_OK;
}

mrg_status mrg_config_get(const char *key, int64_t *value)
{
    if (!key || !value) return set_error(MRG_EINVAL, "null argument");
    std::lock_guard<std::mutex> lk(g_mu);
    if (!std::strcmp(key, "engine")) *value = g_tune.engine;
    else if (!std::strcmp(key, "tile_bytes")) *value = g_tune.tile_bytes;
    else if (!std::strcmp(key, "strategy")) *value = g_tune.strategy;
    else if (!std::strcmp(key, "coop_wgs_per_cu")) *value = g_tune.coop_wgs_per_cu;
    else if (!std::strcmp(key, "coop_order")) *value = g_tune.coop_order;
    else if (!std::strcmp(key, "coop_lanes")) *value = g_tune.coop_lanes;
    else return set_error(MRG_EINVAL, "unknown key '%s'", key);
    return MRG_OK;
}

const char *mrg_status_string(mrg_status s)
{
    switch (s) {
    case MRG_OK: return "MRG_OK";
    case MRG_EINVAL: return "MRG_EINVAL: invalid argument";
    case MRG_ENOMEM: return "MRG_ENOMEM: allocation failed";
    case MRG_EHIP: return "MRG_EHIP: HIP runtime error";
    case MRG_ERANGE: return "MRG_ERANGE: out of range";
    case MRG_ENODEV: return "MRG_ENODEV: no HIP device";
    case MRG_EBUSY: return "MRG_EBUSY: waiting on memory or time";
    default: return "unknown mrg_status";
    }
}

const char *mrg_last_error(void) { return g_last_error.c_str(); }

mrg_status mrg_write_probe(void *d_out, uint64_t bytes, int32_t pattern, void *stream)
{
    if (pattern < 0 || pattern > 3) return set_error(MRG_EINVAL, "unknown probe pattern %d", pattern);
    if (!d_out) return set_error(MRG_EINVAL, "null output");
    const uint64_t unit = pattern == 0 ? 16 : 65536, align = pattern == 0 ? 16 : 128;
    if (bytes % unit) return set_error(MRG_EINVAL, "probe size must be a multiple of %llu bytes",
                                       (unsigned long long)unit);
    if ((uintptr_t)d_out % align) return set_error(MRG_EINVAL, "probe output must be %llu-byte aligned",
                                                   (unsigned long long)align);
    if (!bytes) return MRG_OK;
    int dev;
    mrg_status st = current_device(&dev);
    if (st) return st;
    if ((st = mrg::check_device_span(d_out, bytes, dev, "probe output"))) return st;
    hipError_t e = mrg::launch_write_probe(d_out, bytes, pattern, (hipStream_t)stream);
    return e == hipSuccess ? MRG_OK : hip_error(e, "probe launch");
}

int32_t mrg_version(void) { return 100; }

}  // extern "C"
