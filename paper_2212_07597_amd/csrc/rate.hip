// rate.hip - rate-based sampling (section 3.2), the scheme the threshold
// sampler is compared with: every byte allocated or freed counts towards the
// next sample, one sample per T bytes, whatever the bytes do to the footprint.
// Deterministic reading: the countdown starts at T instead of a random draw,
// so event i takes floor(V_i / T) - floor(V_(i-1) / T) samples, V being the
// cumulative bytes allocated plus bytes freed by memory events; the samples
// are attributed to the event's line.
//
// One kernel over the records: a workgroup holds a tile of them in registers,
// publishes the tile's volume, takes the volume before it from a look-back
// over the tiles before and counts each event's samples from the registers,
// per line through an LDS cache.  A small kernel before it clears the counts
// and the look-back's words.
#include <hip/hip_runtime.h>

#include <mutex>

#include "scalene_sampler.h"
#include "sampler_device.h"

namespace smp {
namespace {

constexpr uint32_t NO_LINE = 0xFFFFFFFFu;
constexpr uint64_t VOL_LIMIT = 1ull << 62;  // volumes at or above it: SMP_EOVERFLOW

// Workspace: a header of 64-bit words, then one look-back word per tile
// (2-bit state: 1 the tile's own volume, 2 the volume through it; 62-bit
// volume).
constexpr uint64_t RATE_HDR = 256;
constexpr uint64_t RATE_BIG = 512ull << 10;  // events above which tiles are large
enum { RH_FLAGS = 0, RH_DONE, RH_TOTAL, RH_TICKET, RH_WORDS };  // flags, workgroups finished, volume, next tile
enum { RF_BAD = 1, RF_OVERFLOW = 2, RF_FAULT = 4 };

struct RateRec {
    int64_t delta;
    uint32_t line;
    uint32_t fw;
};

typedef const __attribute__((address_space(1))) uint8_t ru8_t;
typedef const __attribute__((address_space(1))) uint64_t ru64_t;
typedef const __attribute__((address_space(1))) uint32_t ru32_t;

// Lane l's record of window w of the segment at base with nv >= 1 records
// (lanes past nv re-read the last one; their volume is masked).
__device__ __forceinline__ RateRec rate_load(ru8_t* base, int nv, int w) {
    const int k = w * 64 + lane_id();
    ru8_t* p = base + (uint32_t)((k < nv ? k : nv - 1) * 24);
    RateRec r;
    r.delta = (int64_t)*(ru64_t*)p;
    r.line = *(ru32_t*)(p + 12);
    r.fw = *(ru32_t*)(p + 16);
    return r;
}

// |delta| of a well-formed memory record (else 0); bad: a malformed record
// (the checks of the threshold sampler: kind 3, line >= L, delta out of its
// kind's range).
__device__ __forceinline__ uint64_t rate_volume(const RateRec& r, bool valid, uint32_t L, bool& bad) {
    const uint64_t d = (uint64_t)r.delta;
    const uint32_t kind = (r.fw >> 1) & 3;
    const bool okm = d + (uint64_t)(MAX_ABS_DELTA - 1) < (uint64_t)(2 * MAX_ABS_DELTA - 1);
    const bool okc = d < (uint64_t)MAX_ABS_DELTA;
    const bool okt = (d >> 32) == 0;
    const bool good = (r.line < L) & (((kind == 0) & okm) | ((kind == 1) & okc) | ((kind == 2) & okt));
    bad = valid & !good;
    const bool mem = valid & good & (kind == 0);
    return mem ? (r.delta < 0 ? (uint64_t)(-r.delta) : d) : 0;
}

__global__ void k_rate_clear(int64_t* counts, uint32_t L, uint64_t* result, uint64_t* hdr, uint64_t ntile) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < L) gp(counts)[i] = 0;
    if (i < 2) gp(result)[i] = 0;
    if (i < RH_WORDS) gp(hdr)[i] = 0;
    if (i < ntile) gp(hdr)[RATE_HDR / 8 + i] = 0;
}

constexpr uint64_t VOL_MASK = (1ull << 62) - 1;
constexpr uint32_t RATE_SPINS = 1u << 24;

// Volume before tile t (one wave): 64 tiles per probe, nearest first, up to
// the nearest one that knows the volume through it.  (Volumes whose sum
// reaches 2^62 are flagged by the first tile that sees them, a tile's own
// volume included: every sum up to there is exact.)  Probes of 256 or 512 tiles measured 3 to 10 % slower.
__device__ bool rate_lookback(const uint64_t* st, int64_t t, uint64_t& excl) {
    const int l = lane_id();
    uint64_t acc = 0;
    int64_t base = t - 1;
    for (uint32_t spins = 0; spins < RATE_SPINS;) {
        const int64_t j = base - l;
        const uint64_t w = j >= 0 ? ld_status(st + j) : 2ull << 62;  // before the first tile: nothing
        const uint64_t inc = ballot((w >> 62) == 2);
        const int lim = inc ? ctz64(inc) : 63;
        if (ballot(l <= lim && (w >> 62) == 0)) {  // one of them is not there yet
            ++spins;
            __builtin_amdgcn_s_sleep(4);
            continue;
        }
        acc += (uint64_t)wave_sum((int64_t)(l <= lim ? w & VOL_MASK : 0));
        if (inc) {
            excl = acc;
            return true;
        }
        base -= 64;
    }
    return false;
}

// A workgroup's counts per line in LDS; a line whose slot holds another goes to
// global atomics.  64 slots per wave, and flushed with the held ones side by side
// (a flush of few lines scattered over many waves queues at the same addresses).
// One call with 256 slots for 16 waves and like this: 3e6 events at T = 1,000 on
// 1e5 lines 200 and 85 us (before tiles, with 256 for four waves: 180), 5e7 at T
// = 1 3.9 and 1.25 ms (3.4), 1e6 on 64 lines at T = 1 MiB 24.6 and 17.4 us, on
// 10,000 lines 17.1 and 17.8.
template <int SLOTS>
struct RateCache {
    uint32_t key[SLOTS];
    unsigned long long cnt[SLOTS];
    uint16_t held[SLOTS];  // (at the flush)
    int n;
};

template <int SLOTS>
__device__ __forceinline__ void rate_add(RateCache<SLOTS>& c, int64_t* counts, uint32_t line, uint64_t v) {
    const int slot = (int)((line * 2654435761u) >> (32 - __builtin_ctz(SLOTS)));
    uint32_t k = c.key[slot];
    if (k == NO_LINE) k = atomicCAS(&c.key[slot], NO_LINE, line);
    if (k == NO_LINE || k == line)
        atomicAdd(&c.cnt[slot], (unsigned long long)v);
    else
        g_add((uint64_t*)&counts[line], v);
}

// floor(u / T) for u < 2^62 with m = floor((2^64 - 1) / T): the high product
// is the quotient or one less.  rem receives u mod T.
__device__ __forceinline__ uint64_t rate_div(uint64_t u, uint64_t T, uint64_t m, uint64_t& rem) {
    uint64_t q = __umul64hi(u, m);
    uint64_t r = u - q * T;
    const bool up = r >= T;
    q += up ? 1 : 0;
    r -= up ? T : 0;
    rem = r;
    return q;
}

// Persistent workgroups take tiles by ticket, so every tile that a look-back
// waits on belongs to a running workgroup, which depends on earlier tiles
// only.  Lane
// l's count is floor(b_l / T) - floor(b_(l-1) / T), b_l the volume through
// its record, taken modulo T at each window's start; a window whose volume
// does not reach the next multiple of T is passed over, and the divisions of
// the others are products with a reciprocal.
// Bound: HBM reads (24 bytes per event, once) and the look-back's latency (the
// same kernel without its waits: 0.48 ms).  One call on 1e8 events at T = 10
// MiB: 0.57 ms, 4.2 TB/s; as two passes over the records with a scan between
// them it took 0.92 ms.  1e5 events: 17.5 -> 11 to
// 13 us (two launches, not four).
template <int WV>
__global__ __launch_bounds__(64 * WV) __attribute__((amdgpu_waves_per_eu(4))) void k_rate(const uint8_t* __restrict__ ev, uint64_t n, uint64_t ntile,
                                                     uint32_t L, int64_t T, uint64_t m, uint64_t* hdr,
                                                     int64_t* counts, uint64_t* result) {
    constexpr int BLK = 64 * WV, TILE_EV = SEG * WV;  // one segment per wave
    constexpr int SLOTS = 64 * WV;
    __shared__ RateCache<SLOTS> c;
    __shared__ uint64_t s_sum[WV];
    __shared__ uint64_t s_excl, s_tk, s_last;
    const int tid = threadIdx.x, l = lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    c.key[tid] = NO_LINE;  // (a slot per thread)
    c.cnt[tid] = 0;
    if (tid == 0) c.n = 0;
    uint64_t* st = hdr + RATE_HDR / 8;
    const uint64_t uT = (uint64_t)T;
    // The tile in hand: its records' volumes and lines, the sum of the waves'
    // volumes before this wave.  The next one: its records, loading.
    uint64_t vol[NW], before = 0, agg = 0;
    uint32_t line[NW];
    RateRec r[NW];
    auto valid_of = [&](uint64_t t) {
        const uint64_t a = t * TILE_EV + (uint64_t)wv * SEG;
        return t >= ntile || a >= n ? 0 : (int)(n - a < (uint64_t)SEG ? n - a : (uint64_t)SEG);
    };
    auto take_ticket = [&]() -> uint64_t {
        __syncthreads();
        if (tid == 0) s_tk = g_add_rtn(hdr + RH_TICKET, 1ull);
        __syncthreads();
        return readlaneu64(s_tk, 0);
    };
    auto load_tile = [&](uint64_t t) {
        const int nv = valid_of(t);
        // (a wave past the end re-reads the last record, whose volume is masked)
        const uint64_t a = t * TILE_EV + (uint64_t)wv * SEG;
        ru8_t* base = (ru8_t*)(ev + (nv ? a : n - 1) * 24);
#pragma unroll
        for (int w = 0; w < NW; ++w) r[w] = rate_load(base, nv ? nv : 1, w);
    };
    // the loaded tile becomes the one in hand, its volume published
    auto take_tile = [&](uint64_t t) {
        const int nv = valid_of(t);
        uint64_t acc = 0, badm = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            bool bad;
            vol[w] = rate_volume(r[w], w * 64 + l < nv, L, bad);
            line[w] = r[w].line;
            acc += vol[w];  // < 8 x 2^52 per lane
            badm |= ballot(bad);
        }
        const uint64_t mine = (uint64_t)wave_sum((int64_t)acc);  // < 2^61
        if (l == 0) s_sum[wv] = mine;
        if (badm && l == 0) g_or(hdr + RH_FLAGS, RF_BAD);
        __syncthreads();
        // (each eight waves' sum stays below 2^64; 16 would wrap, and one that
        // reaches VOL_LIMIT stands for the tile's, which its look-back flags.  A
        // limit after every wave's addition cost 4 % of the call)
        uint64_t half[2] = {0, 0};
#pragma unroll
        for (int w = 0; w < WV; ++w) {
            if (w == wv) before = half[0] + half[1];
            half[w >> 3] += s_sum[w];
        }
        agg = ((half[0] | half[1]) >> 62) ? VOL_LIMIT : half[0] + half[1];
        if (tid == 0) st_status(st + t, (agg < VOL_MASK ? agg : VOL_MASK) | (t == 0 ? 2ull : 1ull) << 62);
    };
    uint64_t t = take_ticket();
    if (t < ntile) {
        load_tile(t);
        take_tile(t);
    }
    while (t < ntile) {
        // (no more tiles than workgroups: each has its one)
        const uint64_t tn = ntile > gridDim.x ? take_ticket() : ntile;
        if (tn < ntile) load_tile(tn);
        if (wv == 0) {
            uint64_t excl = 0;
            const bool ok = t == 0 || rate_lookback(st, (int64_t)t, excl);
            const uint64_t incl = excl + agg;
            if (l == 0) {
                st_status(st + t, (incl & VOL_MASK) | 2ull << 62);
                s_excl = excl;
                const uint32_t f = (agg >= VOL_LIMIT || excl >= VOL_LIMIT || incl >= VOL_LIMIT ? RF_OVERFLOW : 0) |
                                   (ok ? 0 : RF_FAULT);
                if (f) g_or(hdr + RH_FLAGS, f);
                if (t == ntile - 1) st_status(hdr + RH_TOTAL, incl);
            }
        }
        __syncthreads();
        uint64_t rem;
        (void)rate_div(readlaneu64(s_excl + before, 0) & VOL_MASK, uT, m, rem);
        rem = readlaneu64(rem, 0);
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const uint64_t u = (uint64_t)wave_incl_sum((int64_t)vol[w]) + rem;
            const uint64_t last = readlaneu64(u, 63);
            if (last >= uT) {
                uint64_t q_rem;
                const uint64_t q = rate_div(u, uT, m, q_rem);
                const uint64_t cnt = q - (uint64_t)wave_shr1((int64_t)q, 0);
                if (cnt) rate_add(c, counts, line[w], cnt);
                rem = readlaneu64(q_rem, 63);
            } else {
                rem = last;
            }
        }
        if (tn < ntile) take_tile(tn);
        t = tn;
    }
    __syncthreads();
    {
        const bool held = c.key[tid] != NO_LINE;
        const uint64_t m64 = ballot(held);
        int at = 0;
        if (m64 && l == 0) at = atomicAdd(&c.n, __popcll(m64));
        at = __builtin_amdgcn_readfirstlane(at);
        if (held) c.held[at + __popcll(m64 & lanemask_lt())] = (uint16_t)tid;
    }
    __syncthreads();
    if (tid < c.n) g_add((uint64_t*)&counts[c.key[c.held[tid]]], c.cnt[c.held[tid]]);
    // The last workgroup to finish writes the status and the total.  (What the
    // others wrote went to memory by agent-scope atomics, with no cache to
    // write back: each wave waits for its own before the barrier.)
    stores_done();
    __syncthreads();
    if (tid == 0) s_last = g_add_rtn(hdr + RH_DONE, 1ull);
    __syncthreads();
    if (s_last != (uint64_t)gridDim.x - 1) return;
    const uint64_t f = ld_status(hdr + RH_FLAGS), total = ld_status(hdr + RH_TOTAL);
    if (f) {  // nothing to count for a malformed or overflowing trace
        for (uint64_t i = tid; i < L; i += BLK) gp(counts)[i] = 0;
    }
    if (tid == 0) {
        const bool ovf = (f & RF_OVERFLOW) != 0;
        gp(result)[1] = (f & RF_BAD) ? (uint64_t)SMP_EINVAL
                                     : ((f & RF_FAULT) ? (uint64_t)SMP_EDEVICE
                                                       : (ovf ? (uint64_t)SMP_EOVERFLOW : (uint64_t)SMP_OK));
        gp(result)[0] = ovf ? 0 : total / uT;
    }
}

bool rate_args_ok(const smp_event_t* ev, uint64_t n, int64_t threshold, uint32_t num_lines, int64_t* line_counts,
                  uint64_t* result) {
    return threshold >= 1 && threshold < ((int64_t)1 << 60) && num_lines != 0 && n < 0xFFFFFFFFull && (!n || ev) &&
           line_counts && result;
}

// The launch sequence of one call, with its scratch at ws (RATE_HDR bytes of
// header, then 8 bytes per segment).
int rate_launch(const smp_event_t* ev, uint64_t n, int64_t threshold, uint32_t num_lines, void* ws,
                int64_t* line_counts, uint64_t* result, hipStream_t s) {
    // Tiles of 8 segments up to RATE_BIG events, of 16 above: the large ones
    // halve the look-back's steps and the line caches that are flushed, the
    // small ones give short traces more workgroups.  Small against large: 1e5
    // events 13.6 / 15.6 us, 4e5 14.2 / 16.4, 1e6 17.5 / 18.2, 3e6 36.5 / 33.5 (64
    // lines; on 10,000 lines within 1.5 us of these), 1e8 719 / 604.
    const bool big = n > RATE_BIG;
    const uint64_t te = (uint64_t)SEG * (big ? 16 : 8);
    const uint64_t ntile = (n + te - 1) / te;
    uint64_t* hdr = (uint64_t*)ws;
    uint64_t cl = num_lines > RH_WORDS ? num_lines : RH_WORDS;
    if (cl < ntile) cl = ntile;
    // a kernel, not a memset, clears the counts, the result and the words of the look-back
    k_rate_clear<<<dim3((unsigned)((cl + 255) / 256)), dim3(256), 0, s>>>(line_counts, num_lines, result, hdr, ntile);
    if (hipGetLastError() != hipSuccess) return SMP_EDEVICE;
    if (ntile == 0) {
        // no events: K = 0, status OK (the clear wrote both)
        return SMP_OK;
    }
    // as many workgroups as a device of 256 CUs holds at once (two of 16 waves
    // do not fit one CU); more tiles are taken by the same workgroups
    const uint64_t lim = big ? 256 : 512;
    const unsigned grid = (unsigned)(ntile < lim ? ntile : lim);
    const uint64_t m = ~0ull / (uint64_t)threshold;
    if (big)
        k_rate<16><<<dim3(grid), dim3(1024), 0, s>>>((const uint8_t*)ev, n, ntile, num_lines, threshold, m, hdr,
                                                     line_counts, result);
    else
        k_rate<8><<<dim3(grid), dim3(512), 0, s>>>((const uint8_t*)ev, n, ntile, num_lines, threshold, m, hdr,
                                                   line_counts, result);
    return hipGetLastError() == hipSuccess ? SMP_OK : SMP_EDEVICE;
}

}  // namespace
}  // namespace smp

// Scratch of the no-allocation entry point: one copy per GPU, held until the
// process ends, shared by every call on that GPU.  Host code never uses this
// name as an address (on the host it only names the symbol); the device
// address comes from hipGetSymbolAddress, once per device.
constexpr uint64_t RATE_SCRATCH_BYTES = smp::RATE_HDR + 8 * (SMP_RATE_NOALLOC_MAX_EVENTS / smp::SEG);
static __device__ __align__(256) uint8_t scratch[RATE_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[MAX_DEVICES] = {};

// Device address of this device's scratch (looked up on the device's first
// call, with that device current).
int scratch_address(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return SMP_EDEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return SMP_EDEVICE;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return SMP_OK;
}
}  // namespace

using namespace smp;

extern "C" {

SMP_API uint64_t rate_workspace_bytes(uint64_t n_events) {
    return RATE_HDR + 8 * ((n_events + SEG - 1) / SEG);
}

SMP_API int rate_run(const smp_event_t* ev, uint64_t n, int64_t threshold, uint32_t num_lines, void* workspace,
                     uint64_t workspace_bytes, int64_t* line_counts, uint64_t* result, void* hip_stream) {
    if (!rate_args_ok(ev, n, threshold, num_lines, line_counts, result) || !workspace ||
        workspace_bytes < rate_workspace_bytes(n))
        return SMP_EINVAL;
    return rate_launch(ev, n, threshold, num_lines, workspace, line_counts, result, (hipStream_t)hip_stream);
}

SMP_API int rate_run_noalloc(const smp_event_t* ev, uint64_t n, int64_t threshold, uint32_t num_lines,
                             int64_t* line_counts, uint64_t* result, void* hip_stream) {
    if (!rate_args_ok(ev, n, threshold, num_lines, line_counts, result)) return SMP_EINVAL;
    if (n > SMP_RATE_NOALLOC_MAX_EVENTS) return SMP_ETOOBIG;
    void* ws = nullptr;
    if (int rc = scratch_address(&ws)) return rc;
    return rate_launch(ev, n, threshold, num_lines, ws, line_counts, result, (hipStream_t)hip_stream);
}

}  // extern "C"
