// gfx950 kernels of the threshold sampler.
//
// Method (paper sections cited per step):
//  * The footprint F is the running sum of memory-event deltas (section 3.1:
//    every allocation and free is intercepted once, tagged Python or native).
//  * Threshold sampling (section 3.2): after a sample at node r the next one is
//    the first later node j with |F_j - F_r| >= T.  Restated per segment of
//    events: the chain state entering a segment is the reference footprint
//    relative to the segment start, rho in (-T, T); the segment maps it to the
//    state entering the next segment.
//  * Each segment computes that map for all entries at once ("all-entry
//    analysis"): entries that never reach the threshold inside the segment
//    form one interval and are shifted by the segment's footprint change; every
//    other entry starts a chain at a running-maximum or running-minimum node,
//    and chains that sample at the same node coincide from there on.  When all
//    of them coincide the segment's exit is known before its entry is.
//  * Attribution (section 3.3): each sample goes to the triggering event's
//    line with the net Python and native bytes since the previous sample.
//  * Leak rule (section 3.4): a growth sample above the high-water mark of the
//    earlier tracked samples is tracked; frees of its ptr_id before the next
//    tracked sample mark it reclaimed.  The high-water mark and the active
//    tracked object flow between segments as a running "argmax" (the largest
//    growth footprint, earliest on ties).
//  * Copy volume (section 3.5) and the timer split (section 2.1) are
//    per-event histogram updates.
//
// Passes of one launch (no pass over the records waits on another segment):
//   summarize  per segment: sums, prefix extremes, chain map        (records)
//   resolve    per tile:    exclusive sums, entry offset of each segment
//   chain      per segment: samples, best growth sample, last sample (records)
//   scan       per tile:    rank base, high-water mark, last sample before
//   emit       per segment: samples, per-line histograms, leak bits (records)
#include "sampler_device.h"

namespace smp {

constexpr unsigned long long EMPTY_KEY = ~0ull;

// ---- line caches
//
// One workgroup's counters in LDS, a table per kind of event, so that a slot
// holds only the counters its kind adds to: samples (Python bytes, growth and
// shrink bytes, growth count | shrink count << 32, a trace having fewer than
// 2^32 events; the native bytes are growth - shrink - Python), copies (exact
// and sampled bytes) with timers (delays and events), tracked samples
// (mallocs, frees).  Keys are (trace << 32) | line; K is a power of two below
// 2^16.  A line may sit in either slot of a pair (one 16-byte read), and one
// that finds both taken goes to global atomics.  Those are what the emit pass
// waits on: of its 4.2 ms over 500 M events on 1 M lines, 1.9 went to the
// copy and timer counters (a tenth of the events), most of which missed a
// cache of 128 slots of 12 counters.
template <int K, int V>
struct LineTable {
    alignas(16) unsigned long long key[K];
    unsigned long long v[V][K];
    __device__ __forceinline__ void init() {
        for (int i = threadIdx.x; i < K; i += blockDim.x) {
            key[i] = EMPTY_KEY;
            for (int c = 0; c < V; ++c) v[c][i] = 0;
        }
    }
    // the slot of a line, -1 if both of its slots hold others (a first slot
    // once taken stays so: a line never comes to hold both)
    __device__ __forceinline__ int find(uint32_t t, uint32_t line) {
        const unsigned long long want = ((unsigned long long)t << 32) | line;
        const uint32_t h = (line * 2654435761u) ^ (t * 0x9E3779B9u);
        // (the topmost bits, which a multiplicative hash spreads evenly over
        // consecutive lines and which put a line's timers half a table from its
        // copies: with bits 16 up, 64 lines' copies and timers overflowed 128
        // pairs, and the emit pass on nine copies in ten events took 58 us
        // instead of 22)
        const int s0 = (int)(h >> (32 - __builtin_ctz(K))) & (K - 2);
        const ulonglong2 k = *(const ulonglong2*)&key[s0];
        if (k.x == want) return s0;
        if (k.y == want) return s0 + 1;
        if (k.x == EMPTY_KEY) {
            const unsigned long long o = atomicCAS(&key[s0], EMPTY_KEY, want);
            if (o == EMPTY_KEY || o == want) return s0;
        }
        if (k.y == EMPTY_KEY) {
            const unsigned long long o = atomicCAS(&key[s0 + 1], EMPTY_KEY, want);
            if (o == EMPTY_KEY || o == want) return s0 + 1;
        }
        return -1;
    }
    __device__ __forceinline__ void add(int slot, int c, uint64_t x) {
        if (x) atomicAdd(&v[c][slot], (unsigned long long)x);
    }
};
enum { LS_PY = 0, LS_GB, LS_SB, LS_N, LA_BYTES = 0, LA_N, LK_M = 0, LK_F };
constexpr uint32_t TIMER_LINE = 1u << 31;  // added to the trace in a timer's key

template <class C>
struct LineCaches {
    LineTable<C::SAMPLES, 4> smp;
    LineTable<C::AUX, 2> aux;
};

__device__ __forceinline__ void hist_global(const Desc& D, int h, uint32_t line, uint64_t x) {
    if (x) g_add((uint64_t*)&D.hist[(size_t)h * D.L + line], x);
}

// A sample of py and nat bytes at line (their sum is not 0).
template <class C>
__device__ __forceinline__ void count_sample(C& c, const Desc& D, uint32_t t, uint32_t line, int64_t py, int64_t nat) {
    const int64_t dl = py + nat;
    const bool gr = dl > 0;
    const uint64_t bytes = (uint64_t)(gr ? dl : -dl);
    const int s = c.smp.find(t, line);
    if (s >= 0) {
        c.smp.add(s, LS_PY, (uint64_t)py);
        c.smp.add(s, gr ? LS_GB : LS_SB, bytes);
        c.smp.add(s, LS_N, gr ? 1ull : 1ull << 32);
    } else {
        hist_global(D, H_PY, line, (uint64_t)py);
        hist_global(D, H_NAT, line, (uint64_t)nat);
        hist_global(D, gr ? H_GN : H_SN, line, 1);
        hist_global(D, gr ? H_GB : H_SB, line, bytes);
    }
}

// A copy of x bytes that triggers copy samples of `sampled` bytes in all, or a
// timer event of delay x.
template <class C>
__device__ __forceinline__ void count_aux(C& c, const Desc& D, uint32_t t, uint32_t line, bool timer, uint64_t x,
                                          uint64_t sampled) {
    const int s = c.aux.find(timer ? t | TIMER_LINE : t, line);
    if (s >= 0) {
        c.aux.add(s, LA_BYTES, x);
        c.aux.add(s, LA_N, timer ? 1 : sampled);
    } else {
        hist_global(D, timer ? H_NT : H_CE, line, x);
        hist_global(D, timer ? H_PT : H_CS, line, timer ? (uint64_t)D.q : sampled);
    }
}

// Copy samples of x bytes in all.
template <class C>
__device__ __forceinline__ void count_copy_sample(C& c, const Desc& D, uint32_t t, uint32_t line, uint64_t x) {
    const int s = c.aux.find(t, line);
    if (s >= 0)
        c.aux.add(s, LA_N, x);
    else
        hist_global(D, H_CS, line, x);
}

__device__ __forceinline__ void count_tracked(LineTable<TRACK_SLOTS, 2>& c, const Desc& D, uint32_t t, uint32_t line,
                                              uint32_t freed) {
    const int s = c.find(t, line);
    if (s >= 0) {
        c.add(s, LK_M, 1);
        c.add(s, LK_F, freed);
    } else {
        hist_global(D, H_LEAK_M, line, 1);
        hist_global(D, H_LEAK_F, line, freed);
    }
}

// Move a table to the per-line histograms (whole workgroup, after a barrier):
// add(trace, line, slot) for each slot held.
template <int K, int V, class A>
__device__ __forceinline__ void flush_table(const LineTable<K, V>& c, A add) {
    for (int i = threadIdx.x; i < K; i += blockDim.x) {
        const unsigned long long k = c.key[i];
        if (k != EMPTY_KEY) add((uint32_t)(k >> 32), (uint32_t)k, i);
    }
}

// The same with the held slots gathered first (list: room for K in LDS, n: a
// word of LDS), so that a wave's 64 atomics of one counter go to 64 lines.  A
// table of few lines sends its counters in the fewest requests then, and those
// of all workgroups queue at the same few addresses: the emit pass on 12 M
// events on 64 lines took 138 us slot by slot (512 workgroups of 512 slots)
// and takes 68.
template <int K, int V, class A>
__device__ __forceinline__ void flush_gathered(const LineTable<K, V>& c, uint16_t* list, int* n, A add) {
    __syncthreads();  // (list and n are free)
    if (threadIdx.x == 0) *n = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < K; i += blockDim.x) {
        const bool held = c.key[i] != EMPTY_KEY;
        const uint64_t m = ballot(held);
        int at = 0;
        if (m && lane_id() == 0) at = atomicAdd(n, __popcll(m));
        at = __builtin_amdgcn_readfirstlane(at);
        if (held) list[at + __popcll(m & lanemask_lt())] = (uint16_t)i;
    }
    __syncthreads();
    for (int x = threadIdx.x; x < *n; x += blockDim.x) {
        const int i = list[x];
        const unsigned long long k = c.key[i];
        add((uint32_t)(k >> 32), (uint32_t)k, i);
    }
}

template <class C>
__device__ __forceinline__ void flush_lines(const C& c, const Desc* desc, uint16_t* list, int* n) {
    flush_gathered(c.smp, list, n, [&](uint32_t t, uint32_t line, int i) {
        const Desc& D = desc[t];
        const uint64_t py = c.smp.v[LS_PY][i], gb = c.smp.v[LS_GB][i], sb = c.smp.v[LS_SB][i], n = c.smp.v[LS_N][i];
        hist_global(D, H_PY, line, py);
        hist_global(D, H_NAT, line, gb - sb - py);
        hist_global(D, H_GN, line, n & 0xFFFFFFFFull);
        hist_global(D, H_SN, line, n >> 32);
        hist_global(D, H_GB, line, gb);
        hist_global(D, H_SB, line, sb);
    });
    flush_gathered(c.aux, list, n, [&](uint32_t t, uint32_t line, int i) {
        const Desc& D = desc[t & ~TIMER_LINE];
        const bool timer = (t & TIMER_LINE) != 0;
        const uint64_t x = c.aux.v[LA_BYTES][i], n = c.aux.v[LA_N][i];
        hist_global(D, timer ? H_NT : H_CE, line, x);
        hist_global(D, timer ? H_PT : H_CS, line, timer ? n * (uint64_t)D.q : n);
    });
}

// last trace whose first segment index is <= x
__device__ __forceinline__ int find_trace_seg(const Desc* desc, int lo, int ntraces, uint64_t x) {
    int hi = ntraces - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (desc[mid].seg_begin <= x) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// last trace whose first tile index is <= x
__device__ __forceinline__ int find_trace_tile(const Desc* desc, int ntraces, uint64_t x) {
    int lo = 0, hi = ntraces - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (desc[mid].tile_begin <= x) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// -------------------------------------------------------------- time stamps

// The device clock when a pass starts, for the host's pass timing (ts: the
// word in pinned host memory, null when the pass is not timed).  Kernels of a
// stream do not overlap, so a pass lasts from its own stamp to the next
// one's.  A HIP event between two kernels left the GPU idle for 5.7 us.
__device__ __forceinline__ void stamp(uint64_t* ts) {
    if (ts && blockIdx.x == 0 && threadIdx.x == 0) *gp(ts) = (uint64_t)wall_clock64();
}

// ------------------------------------------------------------ event records

// One decoded record (24 bytes: delta i64, ptr u32, line u32, flags u8).
// Flags: bit 0 native (else Python), bits 1-2 kind (0 memory, 1 copy,
// 2 timer).  Memory deltas satisfy |delta| < 2^52, copies 0 <= delta < 2^52,
// timer delays 0 <= delta < 2^32, and line < L; anything else is malformed
// and contributes nothing.
struct Ev {
    int64_t delta;
    int64_t dm;    // footprint delta
    int64_t dp;    // Python footprint delta
    bool mem_ok;   // well-formed memory event
    bool cp;       // well-formed copy event (its bytes: delta)
    bool bad;
    bool aux;      // well-formed copy or timer event
};

// Each kind's range test is made for every lane and the results combined as
// lane masks: cheaper than choosing per-lane bounds by kind.
__device__ __forceinline__ Ev decode(uint64_t r0, uint32_t line, uint32_t fw, bool valid, uint32_t L) {
    Ev e;
    e.delta = (int64_t)r0;
    const uint32_t kind = (fw >> 1) & 3;
    const bool okm = r0 + (uint64_t)(MAX_ABS_DELTA - 1) < (uint64_t)(2 * MAX_ABS_DELTA - 1);
    const bool okc = r0 < (uint64_t)MAX_ABS_DELTA;
    const bool okt = (r0 >> 32) == 0;
    const bool mem = kind == 0, cpy = kind == 1;
    // bitwise, not short-circuit: no branches
    const bool good = valid & (line < L) & ((mem & okm) | (cpy & okc) | ((kind == 2) & okt));
    e.bad = valid & !good;
    e.mem_ok = good & mem;
    e.dm = e.mem_ok ? e.delta : 0;
    e.dp = (fw & 1u) ? 0 : e.dm;
    e.cp = good & cpy;
    e.aux = good & !mem;
    return e;
}

// Global-memory view of the records (the descriptor's generic pointer would
// otherwise compile to flat loads).
typedef const __attribute__((address_space(1))) uint64_t gu64_t;
typedef const __attribute__((address_space(1))) uint8_t gu8_t;

typedef const __attribute__((address_space(1))) int64_t gi64_t;

__device__ __forceinline__ gu64_t* record(const Desc& D, int64_t i) { return (gu64_t*)(D.ev + (size_t)i * 24); }

// Value p of segment j (any lane-varying p; global loads, never flat).
__device__ __forceinline__ int64_t seg_val(const Desc& D, int p, int64_t j) {
    return ((gi64_t*)D.seg)[(int64_t)p * (int64_t)D.nseg + j];
}

// What the summary pass takes from a segment's records.
struct SegScan {
    int64_t sumF, sumP, sumC;
    int64_t mxF, mnF, mxP, mnP;  // extremes of the relative prefixes
    bool any_aux;
    uint32_t err;
};

// A segment's records in registers: lane l holds records 64w + l.  Only the
// words a pass uses are loaded (PTR: the pointer word, LINE: the line word;
// the delta and the flags word always): a loaded word that is never read
// lets the compiler reuse its register while the load is still in flight,
// which makes it wait for every load of the segment before the first window.
struct SegRecs {
    uint64_t d[NW];      // delta
    uint32_t ptr[NW];    // pointer tag
    uint32_t line[NW];
    uint32_t fw[NW];     // flags word (flags in the low byte)
};

typedef const __attribute__((address_space(1))) uint32_t gu32_t;

// Load the words of one record at p into slot w of r.
template <bool PTR, bool LINE>
__device__ __forceinline__ void load_record(gu8_t* p, int w, SegRecs& r) {
    r.d[w] = *(gu64_t*)p;
    if (PTR) r.ptr[w] = *(gu32_t*)(p + 8);
    if (LINE) r.line[w] = *(gu32_t*)(p + 12);
    r.fw[w] = *(gu32_t*)(p + 16);
}

// Address of lane l's record in window w of a segment at base with nv >= 1
// records (lanes past nv re-read record nv-1, a line already fetched).
__device__ __forceinline__ gu8_t* record_addr(gu8_t* base, int nv, int w) {
    const int k = w * 64 + lane_id();
    return base + (uint32_t)((k < nv ? k : nv - 1) * 24);
}

// Issue the loads of one segment's first nv (>= 1) records.  All addresses
// are formed before the first load so that the loads leave back to back.
// Plain loads: the nontemporal hint measured 5-7 % slower on this pattern.
template <bool PTR, bool LINE>
__device__ __forceinline__ void fetch_segment(const Desc& D, int64_t a, int nv, SegRecs& r) {
    gu8_t* base = (gu8_t*)(D.ev + (size_t)a * 24);  // wave-uniform
    gu8_t* ptrs[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) ptrs[w] = record_addr(base, nv, w);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int w = 0; w < NW; ++w) load_record<PTR, LINE>(ptrs[w], w, r);
    __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ int seg_events(const Desc& D, int64_t j) {
    const uint64_t a = (uint64_t)j * SEG;
    return (int)((D.n - a) < (uint64_t)SEG ? (D.n - a) : (uint64_t)SEG);
}

// ------------------------------------------------------------------- chains

// a > b for wave-uniform values below 2^62 in magnitude, as the sign of
// b - a in scalar arithmetic (the scalar unit has no 64-bit ordered compare,
// so a plain comparison would run on the vector unit).
__device__ __forceinline__ bool sgt64(int64_t a, int64_t b) {
    // the high word's sign (readfirstlane, free on a scalar value, keeps the
    // compiler from turning this back into a 64-bit compare)
    return __builtin_amdgcn_readfirstlane((int)(uint32_t)(((uint64_t)b - (uint64_t)a) >> 32)) < 0;
}

// Lanes whose prefix f is at least T away from ref, from fT = f + (T - 1)
// (formed once per window): |f - ref| >= T as one unsigned compare,
// fT - ref >= 2T - 1 modulo 2^64.  Exact here: prefixes and references stay
// below 2^61 in magnitude and T below 2^61, so the true value of fT - ref lies
// in (-2^63, 2^63) and a negative one wraps above 2^63.
__device__ __forceinline__ uint64_t crossing(int64_t fT, int64_t ref, uint64_t span) {
    return ballot((uint64_t)fT - (uint64_t)ref >= span);
}

// One chain followed through a segment: its reference, sample masks (lane w
// holds window w's mask), the largest growth-sample footprint (earliest on
// ties), the largest sampled footprint and the last sample's index.
struct ChainRun {
    int64_t ref;
    uint64_t mvec;
    int64_t gbest;
    int gnode;
    int64_t smax;
    int lastS;
    int cnt;  // samples recorded
};

// Advance cr through one window whose footprint prefixes f (and Python
// footprint prefixes p) are in registers, after lane st.  FULL also records
// the window's sample mask (lane w), the best growth sample, the largest
// sampled footprint, the last sample node and, in lsp, the Python footprint
// at the last sample.
template <bool FULL>
__device__ __forceinline__ void chain_window(int64_t f, int64_t p, int64_t T, ChainRun& cr, int64_t& lsp, int w,
                                             int st) {
    const int l = lane_id();
    uint64_t m = 0;
    const int64_t fT = (int64_t)((uint64_t)f + (uint64_t)(T - 1));
    const uint64_t span = (uint64_t)(2 * T - 1);
    while (st < 63) {  // (lanes above st: ~0 << (st + 1))
        const uint64_t ex = crossing(fT, cr.ref, span) & (~0ull << (st + 1));
        if (!ex) break;
        const int jj = ctz64(ex);
        const int64_t fj = readlane64(f, jj);
        if (FULL) {
            // (prefixes and references stay below 2^61 in magnitude; smax
            // starts at INT64_MIN)
            if (sgt64(fj, cr.ref) && (cr.gnode < 0 || sgt64(fj, cr.gbest))) {
                cr.gbest = fj;
                cr.gnode = w * 64 + jj;
            }
            if (cr.smax == INT64_MIN || sgt64(fj, cr.smax)) cr.smax = fj;
            m |= 1ull << jj;
            cr.lastS = w * 64 + jj;
        }
        cr.ref = fj;
        st = jj;
    }
    if (FULL && m) {
        lsp = readlane64(p, top64(m));
        if (l == w) cr.mvec |= m;
        cr.cnt += __popcll(m);
    }
}

// Follow one chain through the window held in f (one node per lane), starting
// after lane st.  U holds the lanes where an earlier chain of this window
// sampled; reaching one of them means the chains coincide (returns false).
__device__ __forceinline__ bool follow(int64_t f, int64_t T, int64_t& ref, int st, uint64_t& U) {
    const int64_t fT = (int64_t)((uint64_t)f + (uint64_t)(T - 1));
    const uint64_t span = (uint64_t)(2 * T - 1);
    for (;;) {
        if (st >= 63) return true;
        const uint64_t m = crossing(fT, ref, span) & (~0ull << (st + 1));
        if (!m) return true;
        const int j = ctz64(m);
        if ((U >> j) & 1) return false;
        U |= 1ull << j;
        ref = readlane64(f, j);
        st = j;
    }
}

struct SegMap {
    int64_t lo, hi, kf;
    int kind;
    int fnode;  // first forced event (-1 if none)
};

// All-entry analysis of a segment without forced events (F: relative
// prefixes in LDS), following at most cap distinct chains at once (cap <= 64,
// one per lane; more make the map SIM).
__device__ SegMap analyse_segment(const int64_t* F, int64_t T, int64_t sumF, int cap) {
    const int l = lane_id();
    SegMap m;
    // Entries in [Lo, Hi] have not sampled yet; chain c (lane c < nch) holds
    // the reference of one distinct chain of the entries that have.
    int64_t Lo = -T + 1, Hi = T - 1;
    int nch = 0;
    bool ovf = false;
    int64_t chref = 0;
    for (int w = 0; w < NW; ++w) {
        const int64_t f = F[w * 64 + l];
        if (ovf) {
            if (Lo <= Hi) {
                const int64_t wmx = wave_max(f), wmn = wave_min(f);
                Lo = (wmx - T + 1) > Lo ? (wmx - T + 1) : Lo;
                Hi = (wmn + T - 1) < Hi ? (wmn + T - 1) : Hi;
            }
            continue;
        }
        uint64_t U = 0;
        int nal = 0;
        for (int c = 0; c < nch; ++c) {
            int64_t ref = readlane64(chref, c);
            if (follow(f, T, ref, -1, U)) {
                if (l == nal) chref = ref;
                ++nal;
            }
        }
        if (Lo <= Hi) {
            const int64_t im = wave_incl_max(f), in = wave_incl_min(f);
            const int64_t em = wave_shr1(im, INT64_MIN), en = wave_shr1(in, INT64_MAX);
            // entries still unsampled just before node l
            int64_t lob = Lo, hib = Hi;
            if (l > 0) {
                lob = (em - T + 1) > Lo ? (em - T + 1) : Lo;
                hib = (en + T - 1) < Hi ? (en + T - 1) : Hi;
            }
            const bool ne = lob <= hib;
            const bool up = ne && (f - T >= lob);
            const bool dn = ne && (f + T <= hib);
            // node c is the first sample of some entries: a chain starts there
            uint64_t cm = ballot(up || dn);
            while (cm) {
                const int c = ctz64(cm);
                cm &= cm - 1;
                if ((U >> c) & 1) continue;
                U |= 1ull << c;
                int64_t ref = readlane64(f, c);
                if (follow(f, T, ref, c, U)) {
                    if (nal >= cap) {
                        ovf = true;
                        break;
                    }
                    if (l == nal) chref = ref;
                    ++nal;
                }
            }
            const int64_t wmx = readlane64(im, 63), wmn = readlane64(in, 63);
            Lo = (wmx - T + 1) > Lo ? (wmx - T + 1) : Lo;
            Hi = (wmn + T - 1) < Hi ? (wmn + T - 1) : Hi;
        }
        nch = ovf ? 0 : nal;
    }
    if (Lo > T) Lo = T;
    if (Hi < -T) Hi = -T;
    const bool has_const = !ovf && nch == 1;
    m.fnode = -1;
    m.lo = Lo;
    m.hi = Hi;
    m.kf = has_const ? readlane64(chref, 0) - sumF : 0;
    m.kind = has_const ? (Lo > Hi ? MAP_TOTAL : MAP_CONST) : MAP_SIM;
    return m;
}

// The same for a segment that moves less than T, from its extremes: an entry
// samples at most once in it, at the first node beyond all earlier ones that
// is T away, and every node beyond all earlier ones is that for some entry.
// So the segment has one chain (a constant exit) only if there is one such
// node: if the first node away from 0 is an extreme already and the other
// side has none.  Summary pass, against following the chains: 2e7 events at
// T = 64 MiB 150 -> 118 us, 1,024 traces at T up to 10 MiB 1.07 -> 0.98 ms
// (5e8 events, bound by memory: unchanged at 3.26 ms).
__device__ __forceinline__ bool still_segment(const int64_t* F, int64_t T, int64_t sumF, int64_t mx, int64_t mn,
                                              SegMap& m) {
    const int64_t hi = sgt64(mx, 0) ? mx : 0, lo = sgt64(0, mn) ? mn : 0;
    if (!sgt64(T, hi - lo)) return false;
    m.fnode = -1;
    m.lo = hi - T + 1;
    m.hi = lo + T - 1;
    m.kf = 0;
    m.kind = MAP_SIM;
    if ((hi == 0) != (lo == 0)) {
        const int64_t x = hi - lo == hi ? hi : lo;  // the one extreme
        int64_t first = 0;
        for (int w = 0; w < NW; ++w) {
            const int64_t f = F[w * 64 + lane_id()];
            const uint64_t a = ballot(f != 0);
            if (a) {
                first = readlane64(f, ctz64(a));
                break;
            }
        }
        if (first == x) {
            m.kind = MAP_CONST;
            m.kf = x - sumF;
        }
    }
    return true;
}

// ---------------------------------------------------------------- look-backs

// Every wait on another tile's status polls with a budget and an exponential
// back-off.  Running out of budget (only possible through an internal fault)
// raises the launch-wide abort word, after which every wait returns at once,
// so all waves always exit.
constexpr uint32_t SPIN_BUDGET = 1u << 24;

struct Spin {
    uint32_t budget = SPIN_BUDGET;
    uint32_t reps = 1;
};

__device__ __forceinline__ bool spin_abort(unsigned long long* ctl, Spin& sp) {
    if (ld_status((const uint64_t*)&ctl[1])) return true;
    for (uint32_t i = 0; i < sp.reps; ++i) __builtin_amdgcn_s_sleep(4);
    if (sp.reps < 8) sp.reps <<= 1;
    if (--sp.budget == 0) {
        st_status((uint64_t*)&ctl[1], 1);
        return true;
    }
    return false;
}

// A wait on a flag in LDS (set by another wave of the same workgroup) polls
// with a short sleep and checks the abort word and the budget only every 64
// polls: the exponential back-off above would add up to a microsecond to
// every hand-off.
struct LocalSpin {
    Spin sp;
    uint32_t n = 0;
};

__device__ __forceinline__ bool local_spin_abort(unsigned long long* ctl, LocalSpin& s) {
    __builtin_amdgcn_s_sleep(1);
    if ((++s.n & 63) != 0) return false;
    return spin_abort(ctl, s.sp);
}

// Wait until a status word is published (wave-uniform address).
__device__ bool wait_word(const uint64_t* p, int64_t& v, unsigned long long* ctl) {
    Spin sp;
    for (;;) {
        const uint64_t w = ld_status(p);
        if (wstate(w)) {
            v = unpack(w);
            return true;
        }
        if (spin_abort(ctl, sp)) return false;
    }
}

// Decoupled look-backs over tiles.  Tile g looks at its predecessors g-1-l
// (lane l, nearest first): it needs the nearest one that has published an
// inclusive value and the aggregates of all tiles after it.  Having them, it
// also publishes the inclusive values of those intermediate tiles
// ("helping").  Identical values may be written by several waves.

// Exclusive (F, P, C) prefix of tile g.
__device__ bool scan_sums(const StatusView& sv, int64_t g, int64_t& oF, int64_t& oP, int64_t& oC,
                          unsigned long long* ctl) {
    const int l = lane_id();
    {
        uint64_t v = 0;
        if (l < 3) v = ld_status(sv.at(W_IF + l, g - 1));
        if ((ballot(l < 3 && wstate(v)) & 7ull) == 7ull) {
            oF = unpack(readlaneu64(v, 0));
            oP = unpack(readlaneu64(v, 1));
            oC = unpack(readlaneu64(v, 2));
            return true;
        }
    }
    int64_t accF = 0, accP = 0, accC = 0;
    int64_t base = g - 1;
    bool first = true;
    Spin sp;
    while (base >= 0) {
        const int64_t jj = base - l;
        const bool in = jj >= 0;
        const int64_t js = in ? jj : 0;
        const uint64_t iF = in ? ld_status(sv.at(W_IF, js)) : 0;
        const uint64_t im = ballot(in && wstate(iF));
        const int lim = im ? ctz64(im) : __popcll(ballot(in));
        const bool need = in && l < lim;
        const bool at = im && l == lim;
        uint64_t x0 = 0, x1 = 0, x2 = 0;  // aggregate (need) or inclusive (at) words
        bool have = !(need || at);
        for (;;) {
            if (!have) {
                if (need) {
                    x0 = ld_status(sv.at(W_AF, js));
                    x1 = ld_status(sv.at(W_AP, js));
                    x2 = ld_status(sv.at(W_AC, js));
                } else {
                    x0 = iF;
                    x1 = ld_status(sv.at(W_IP, js));
                    x2 = ld_status(sv.at(W_IC, js));
                }
                have = wstate(x0) && wstate(x1) && wstate(x2);
            }
            if (!ballot(!have)) break;
            if (spin_abort(ctl, sp)) return false;
        }
        const int64_t vF = (need || at) ? unpack(x0) : 0;
        const int64_t vP = (need || at) ? unpack(x1) : 0;
        const int64_t vC = (need || at) ? unpack(x2) : 0;
        // suffix sums toward older tiles: S_l = sum over lanes >= l
        int64_t xF = vF, xP = vP, xC = vC;
        wave_incl_sum3(xF, xP, xC);
        const int64_t tF = readlane64(xF, 63), tP = readlane64(xP, 63), tC = readlane64(xC, 63);
        if (first && im && need) {
            st_status(sv.at(W_IF, js), pack(tF - xF + vF, 1));
            st_status(sv.at(W_IP, js), pack(tP - xP + vP, 1));
            st_status(sv.at(W_IC, js), pack(tC - xC + vC, 1));
        }
        accF += tF;
        accP += tP;
        accC += tC;
        if (im) break;
        base -= 64;
        first = false;
    }
    oF = accF;
    oP = accP;
    oC = accC;
    return true;
}

// (count, best growth record) items, combined in segment order: counts add;
// the record with the larger footprint wins, the earlier one on ties.  The
// state before a trace is a high-water mark of 0 with nothing tracked.
struct Best {
    int64_t cnt;
    bool has;
    int64_t val;
    uint32_t idx, ptr;
};

__device__ __forceinline__ Best with_baseline(Best b) {
    if (b.has && b.val <= 0) b.has = false;  // a high-water mark of 0 beats it
    if (!b.has) b.val = 0;
    return b;
}

// a, then b
__device__ __forceinline__ Best combine(const Best& a, const Best& b) {
    Best r = a;
    r.cnt = a.cnt + b.cnt;
    if (b.has && (!a.has || b.val > a.val)) {
        r.has = true;
        r.val = b.val;
        r.idx = b.idx;
        r.ptr = b.ptr;
    }
    return r;
}

// value of lane l + d (lanes past 63 get `fill`)
__device__ __forceinline__ int64_t lane_down(int64_t x, int d, int64_t fill) {
    const int l = lane_id();
    const int64_t y = shfl64(x, l + d < 64 ? l + d : l);
    return l + d < 64 ? y : fill;
}

// Exclusive Best prefix of tile g (baseline applied), loading as scan_sums.
__device__ bool scan_best(const StatusView& sv, int64_t g, Best& out, unsigned long long* ctl) {
    const int l = lane_id();
    {
        uint64_t v = 0;
        if (l < 4) v = ld_status(sv.at(W_ICNT + l, g - 1));
        if ((ballot(l < 4 && wstate(v)) & 15ull) == 15ull) {
            const uint64_t wg = readlaneu64(v, 1);
            out.cnt = unpack(readlaneu64(v, 0));
            out.has = wstate(wg) == 2;
            out.val = unpack(wg);
            out.idx = (uint32_t)unpack(readlaneu64(v, 2));
            out.ptr = (uint32_t)unpack(readlaneu64(v, 3));
            out = with_baseline(out);
            return true;
        }
    }
    Best acc{0, false, 0, 0, 0};  // later tiles combined so far
    int64_t base = g - 1;
    bool first = true;
    Spin sp;
    while (base >= 0) {
        const int64_t jj = base - l;
        const bool in = jj >= 0;
        const int64_t js = in ? jj : 0;
        const uint64_t ic = in ? ld_status(sv.at(W_ICNT, js)) : 0;
        const uint64_t im = ballot(in && wstate(ic));
        const int lim = im ? ctz64(im) : __popcll(ballot(in));
        const bool need = in && l < lim;
        const bool at = im && l == lim;
        uint64_t c = 0, gm = 0, gr = 0, gp = 0;
        bool have = !(need || at);
        for (;;) {
            if (!have) {
                if (need) {
                    c = ld_status(sv.at(W_BCNT, js));
                    gm = ld_status(sv.at(W_BGM, js));
                    gr = ld_status(sv.at(W_BGR, js));
                    gp = ld_status(sv.at(W_BGP, js));
                } else {
                    c = ic;
                    gm = ld_status(sv.at(W_IGM, js));
                    gr = ld_status(sv.at(W_IGR, js));
                    gp = ld_status(sv.at(W_IGP, js));
                }
                have = wstate(c) && wstate(gm) && wstate(gr) && wstate(gp);
            }
            if (!ballot(!have)) break;
            if (spin_abort(ctl, sp)) return false;
        }
        const bool use = need || at;
        const int64_t cnt = use ? unpack(c) : 0;
        const bool has = use && wstate(gm) == 2;
        const int64_t val = has ? unpack(gm) : INT64_MIN;
        const uint32_t idx = (uint32_t)unpack(gr), ptr = (uint32_t)unpack(gp);
        // suffix (toward older) counts and maxima
        const int64_t xc = wave_incl_sum(cnt);
        const int64_t tc = readlane64(xc, 63);
        const int64_t rev = shfl64(val, 63 - l);
        const int64_t M = shfl64(wave_incl_max(rev), 63 - l);  // max over lanes >= l
        // the earliest holder of M for lane l is the first lane >= l where the
        // suffix maximum drops (or the last lane)
        const int64_t Mn = lane_down(M, 1, INT64_MIN);
        const uint64_t bnd = ballot(M != INT64_MIN && M > Mn);
        const uint64_t ge = bnd & ~lanemask_lt();
        const int src = ge ? ctz64(ge) : l;
        const uint32_t sidx = (uint32_t)shfl32((int)idx, src), sptr = (uint32_t)shfl32((int)ptr, src);
        if (first && im && need) {
            Best inc{tc - xc + cnt, M != INT64_MIN, M, sidx, sptr};
            inc = with_baseline(inc);
            st_status(sv.at(W_ICNT, js), pack(inc.cnt, 1));
            st_status(sv.at(W_IGM, js), pack(inc.val, inc.has ? 2 : 1));
            st_status(sv.at(W_IGR, js), pack((int64_t)inc.idx, 1));
            st_status(sv.at(W_IGP, js), pack((int64_t)inc.ptr, 1));
        }
        // the whole window (lane 0's suffix) comes before everything in acc
        Best win;
        win.cnt = tc;
        const int64_t M0 = readlane64(M, 0);
        win.has = M0 != INT64_MIN;
        win.val = M0;
        win.idx = (uint32_t)readlane32((int)sidx, 0);
        win.ptr = (uint32_t)readlane32((int)sptr, 0);
        acc = combine(win, acc);
        if (im) break;
        base -= 64;
        first = false;
    }
    out = with_baseline(acc);
    return true;
}

// Python footprint at the last sample before tile g (0 if none).
__device__ bool scan_last_sample(const StatusView& sv, int64_t g, int64_t& oP, unsigned long long* ctl) {
    const int l = lane_id();
    int64_t base = g - 1;
    bool first = true;
    Spin sp;
    while (base >= 0) {
        const int64_t jj = base - l;
        const bool in = jj >= 0;
        const int64_t js = in ? jj : 0;
        uint64_t li = 0, la = 0;
        if (in) {
            li = ld_status(sv.at(W_LSI, js));
            la = ld_status(sv.at(W_LSA, js));
        }
        // a lane resolves the search if its tile has a sample or a known exit value
        const bool hit = in && (wstate(la) == 2 || wstate(li) != 0);
        const uint64_t hm = ballot(hit);
        const int lim = hm ? ctz64(hm) : __popcll(ballot(in));
        if (ballot(in && l < lim && wstate(la) == 0)) {
            if (spin_abort(ctl, sp)) return false;
            continue;
        }
        if (hm) {
            const uint64_t src_w = wstate(readlaneu64(la, lim)) == 2 ? readlaneu64(la, lim) : readlaneu64(li, lim);
            const int64_t v = unpack(src_w);
            if (first && in && l < lim && wstate(li) == 0) st_status(sv.at(W_LSI, js), pack(v, 1));
            oP = v;
            return true;
        }
        base -= 64;
        first = false;
    }
    oP = 0;
    return true;
}

// ------------------------------------------------------------ summary pass

// Sums, extremes of the relative prefixes and the chain map of segment g.
// An event with |delta| >= 2T-1 samples for every entry state, so from the
// first such event on the chain is the same for all entries: it is followed
// here, window by window while scanning, with its samples recorded for the
// chain and emit passes.  Segments without one get the all-entry analysis
// over the prefixes kept in LDS.
// The footprint prefixes of SIM segments, kept for the resolve pass in the
// sample area (written only later, by the emit pass): segment j at
// samples + 4 KB * j.  A trace of fewer than 127 events has too small an
// area; the resolve pass then scans such segments from their records.
// A segment whose prefixes all lie in (-2^30, 2^30) keeps them as 32-bit
// values (flag FLG_FIT): lane l's eight windows side by side, so that a
// segment is two 16-byte words per lane each way, half the bytes of the
// 64-bit form (window by window) that the others keep.
__device__ __forceinline__ bool prefixes_kept(const Desc& D) {
    return (D.n + 1) * sizeof(Sample) >= (uint64_t)D.nseg * SEG * sizeof(int64_t);
}
__device__ __forceinline__ SMP_GLOBAL int64_t* kept_prefixes(const Desc& D, int64_t j) {
    return gp((int64_t*)D.samples) + j * SEG;
}

typedef int32_t v4i32 __attribute__((ext_vector_type(4)));

// The 32-bit kept prefixes of segment j into registers, f[w] = node 64w + l
// (the loads are issued here; the first use of f waits for them).
__device__ __forceinline__ void load_kept32(const Desc& D, int64_t j, int32_t (&f)[NW]) {
    const SMP_GLOBAL v4i32* p = (const SMP_GLOBAL v4i32*)kept_prefixes(D, j) + 2 * lane_id();
    const v4i32 a = p[0], b = p[1];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        f[w] = a[w];
        f[4 + w] = b[w];
    }
}

__device__ __forceinline__ void summarize_segment(const Desc& D, uint64_t g, int64_t* lF_) {
    const int l = lane_id();
    const int64_t j = (int64_t)(g - D.seg_begin);
    const int64_t a = j * SEG;
    const int nv = seg_events(D, j);
    SegRecs rr;
    fetch_segment<false, true>(D, a, nv, rr);
    const int64_t T = D.T;
    const int64_t two_t = 2 * T - 1;
    int64_t cF = 0, cP = 0, accC = 0;
    int64_t mxF = INT64_MIN, mnF = INT64_MAX, mxP = INT64_MIN, mnP = INT64_MAX;
    uint64_t bad_m = 0, aux_m = 0, cp_m = 0;  // lanes that saw such a record
    int fnode = -1;
    int64_t plo = -T + 1, phi = T - 1, ffn = 0, pfn = 0;
    ChainRun r{0, 0, 0, -1, INT64_MIN, -1, 0};
    int64_t alp = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int k = w * 64 + l;
        const bool valid = k < nv;
        const Ev e = decode(rr.d[w], rr.line[w], rr.fw[w], valid, D.L);
        // malformed, copy and timer records are rare: one test per window
        if (ballot(valid & !e.mem_ok)) {
            bad_m |= ballot(e.bad);
            aux_m |= ballot(e.aux);
            const uint64_t cpw = ballot(e.cp);
            cp_m |= cpw;
            if (cpw) accC += e.cp ? e.delta : 0;
        }
        // forced: |dm| >= 2T - 1, as one unsigned compare (as in crossing)
        const uint64_t fm = ballot((uint64_t)e.dm + (uint64_t)(two_t - 1) >= (uint64_t)(2 * two_t - 1));
        int64_t f = e.dm, p = e.dp;
        wave_incl_sum2(f, p);
        f += cF;
        p += cP;
        cF = readlane64(f, 63);
        cP = readlane64(p, 63);
        if (fnode < 0) lF_[k] = f;  // (only the all-entry analysis reads them)
        if (fnode < 0 && fm) {
            // The first forced event: entries in [plo, phi] take no sample
            // before it (the prefix's extremes: earlier windows, then the
            // lanes before it in this one).
            const int fl = ctz64(fm);
            fnode = w * 64 + fl;
            if (fnode > 0) {
                int64_t pmx, pmn;
                if (w == 0 && !ballot(l < fl && (f > INT32_MAX || f < INT32_MIN))) {
                    // the usual case: a first-window prefix of 32-bit values
                    pmx = wave_ext32<true>(l < fl ? (int32_t)f : INT32_MIN);
                    pmn = wave_ext32<false>(l < fl ? (int32_t)f : INT32_MAX);
                } else {
                    pmx = wave_max(l < fl && f > mxF ? f : mxF);
                    pmn = wave_min(l < fl && f < mnF ? f : mnF);
                }
                plo = pmx > 0 ? pmx - T + 1 : -T + 1;
                phi = pmn < 0 ? pmn + T - 1 : T - 1;
            }
            ffn = readlane64(f, fl);
            pfn = readlane64(p, fl);
            r.ref = ffn;
        }
        // lanes past the segment end hold its last prefixes, which are
        // prefixes too: no lane mask needed
        mxF = f > mxF ? f : mxF;
        mnF = f < mnF ? f : mnF;
        mxP = p > mxP ? p : mxP;
        mnP = p < mnP ? p : mnP;
        if (fnode >= w * 64) {
            // the chain from the forced event (the same for every entry)
            chain_window<true>(f, p, T, r, alp, w, fnode - w * 64);
        } else if (fnode >= 0) {
            chain_window<true>(f, p, T, r, alp, w, -1);
        }
    }
    SegScan sc;
    sc.sumF = cF;
    sc.sumP = cP;
    sc.sumC = cp_m ? wave_sum(accC) : 0;
    sc.mxF = wave_max(mxF);
    sc.mnF = wave_min(mnF);
    sc.mxP = wave_max(mxP);
    sc.mnP = wave_min(mnP);
    sc.any_aux = aux_m != 0;
    sc.err = bad_m ? 1u : 0u;
    SegMap m;
    int fit = 0;
    if (fnode >= 0) {
        m.lo = 1;
        m.hi = 0;
        m.kf = r.ref - cF;
        m.kind = MAP_TOTAL;
        m.fnode = fnode;
    } else {
        if (!still_segment(lF_, T, cF, sc.mxF, sc.mnF, m)) m = analyse_segment(lF_, T, cF, (int)D.chain_cap);
        if (m.kind == MAP_SIM && prefixes_kept(D)) {
            if (sgt64(KEPT32, sc.mxF) && sgt64(sc.mnF, -KEPT32)) {
                fit = FLG_FIT;
                v4i32 a, b;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    a[w] = (int32_t)lF_[w * 64 + l];
                    b[w] = (int32_t)lF_[(4 + w) * 64 + l];
                }
                SMP_GLOBAL v4i32* o = (SMP_GLOBAL v4i32*)kept_prefixes(D, j) + 2 * l;
                o[0] = a;
                o[1] = b;
            } else {
                SMP_GLOBAL int64_t* o = kept_prefixes(D, j);
#pragma unroll
                for (int w = 0; w < NW; ++w) o[w * 64 + l] = lF_[w * 64 + l];
            }
        }
    }
    const int64_t acnt = r.cnt;
    const int64_t amf = fnode >= 0 ? (int64_t)readlaneu64(r.mvec, fnode >> 6) : 0;
    // the plane values (all wave-uniform) into lanes 0..SP_PFN, one store
    int64_t v = 0;
    v = writelane64<SP_AF>(v, sc.sumF);
    v = writelane64<SP_AP>(v, sc.sumP);
    v = writelane64<SP_AC>(v, sc.sumC);
    v = writelane64<SP_MXF>(v, sc.mxF);
    v = writelane64<SP_MNF>(v, sc.mnF);
    v = writelane64<SP_MXP>(v, sc.mxP);
    v = writelane64<SP_MNP>(v, sc.mnP);
    v = writelane64<SP_LO>(v, m.lo);
    v = writelane64<SP_HI>(v, m.hi);
    v = writelane64<SP_KF>(v, m.kf);
    v = writelane64<SP_FLG>(v, m.kind | (sc.any_aux ? FLG_AUX : 0) | fit);
    v = writelane64<SP_FN>(v, m.fnode);
    v = writelane64<SP_ACNT>(v, acnt);
    v = writelane64<SP_AGV>(v, r.gbest);
    v = writelane64<SP_AGN>(v, r.gnode);
    v = writelane64<SP_ASMX>(v, r.smax);
    v = writelane64<SP_ALS>(v, r.lastS);
    v = writelane64<SP_ALP>(v, r.lastS >= 0 ? alp : 0);
    v = writelane64<SP_AMF>(v, amf);
    v = writelane64<SP_PLO>(v, plo);
    v = writelane64<SP_PHI>(v, phi);
    v = writelane64<SP_FFN>(v, ffn);
    v = writelane64<SP_PFN>(v, pfn);
    if (l <= SP_PFN) gp(D.seg)[(int64_t)l * (int64_t)D.nseg + j] = v;
    if (fnode >= 0 && l < NW) gp(D.mask)[j * NW + l] = r.mvec;
    if (sc.err && l == 0) g_or32(&D.scal->err, sc.err);
}

// The work of workgroup b when each XCD takes runs of XCD_RUN consecutive
// workgroups' work (workgroups are dealt to the 8 XCDs in turn; the last,
// incomplete round stays in order).
constexpr uint64_t XCDS = 8, XCD_RUN = 16;
__device__ __forceinline__ uint64_t xcd_block(uint64_t b, uint64_t n) {
    const uint64_t first = b / (XCDS * XCD_RUN) * (XCDS * XCD_RUN), r = b - first;
    return first + XCDS * XCD_RUN <= n ? first + r % XCDS * XCD_RUN + r / XCDS : b;
}

// One wave per segment, one launch wave per segment (measured faster here
// than a grid-stride loop: the hardware starts a new wave's loads while
// others compute).  Runs of 16 workgroups per XCD: a segment writes 8 bytes to
// each of 23 planes, and the 128-byte lines of 16 segments then fill up in one
// XCD's L2 instead of going out in pieces from eight.  1e8 events 518 -> 460 us
// (5.2 TB/s of records), 5e8 events 3.0 -> 2.76 ms; runs of 2 and 4: 510 and
// 499 us, of 8 to 64: 448 to 470.
__global__ __launch_bounds__(BLOCK) void k_summarize(const Desc* __restrict__ desc, int ntraces,
                                                     uint64_t nseg_total, uint64_t* ts) {
    __shared__ int64_t lF[WAVES][SEG];
    stamp(ts);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
    const uint64_t g = xcd_block(blockIdx.x, gridDim.x) * WAVES + wv;
    if (g >= nseg_total) return;
    summarize_segment(desc[__builtin_amdgcn_readfirstlane(find_trace_seg(desc, 0, ntraces, g))], g, lF[wv]);
}

// ------------------------------------------------------------ resolve pass

constexpr int RING = 12;  // SIM segments pre-scanned ahead of the walker

// Relative footprint prefixes of segment j into F (one wave; lanes past the
// segment end hold its last prefix).
// Two halves of four windows each, to keep the register footprint small.
__device__ __forceinline__ void prescan_segment(const Desc& D, int64_t j, int64_t* F) {
    const int l = lane_id();
    const int nv = seg_events(D, j);
    gu8_t* base = (gu8_t*)(D.ev + (size_t)j * SEG * 24);
    int64_t cF = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint64_t q0[NW / 2];
        uint32_t q2[NW / 2];
#pragma unroll
        for (int w = 0; w < NW / 2; ++w) {
            gu8_t* p = record_addr(base, nv, h * NW / 2 + w);
            q0[w] = *(gu64_t*)p;
            q2[w] = *(gu32_t*)(p + 16);
        }
#pragma unroll
        for (int w = 0; w < NW / 2; ++w) {
            const int k = (h * NW / 2 + w) * 64 + l;
            const uint32_t fl = q2[w];
            const int64_t dm = (k < nv && (fl & 6u) == 0) ? (int64_t)q0[w] : 0;
            const int64_t f = wave_incl_sum(dm) + cF;
            cF = readlane64(f, 63);
            F[k] = f;
        }
    }
}

// The kept prefixes of segment j (fit: in 32 bits) into registers (one round trip).
__device__ __forceinline__ void load_kept(const Desc& D, int64_t j, bool fit, int64_t (&f)[NW]) {
    const int l = lane_id();
    if (fit) {
        int32_t v[NW];
        load_kept32(D, j, v);
#pragma unroll
        for (int w = 0; w < NW; ++w) f[w] = v[w];
    } else {
        const SMP_GLOBAL int64_t* F = kept_prefixes(D, j);
#pragma unroll
        for (int w = 0; w < NW; ++w) f[w] = F[w * 64 + l];
    }
}

// The same into F (one wave).
__device__ __forceinline__ void copy_prefixes(const Desc& D, int64_t j, bool fit, int64_t* F) {
    int64_t v[NW];
    load_kept(D, j, fit, v);
#pragma unroll
    for (int w = 0; w < NW; ++w) F[w * 64 + lane_id()] = v[w];
}

// Exit offset of a segment from entry offset x, following its prefixes F
// window by window (read four windows at a time, so that the LDS reads
// overlap).  A round-based search over all windows at once measured slower:
// walked segments often hold many samples.
__device__ __forceinline__ int64_t walk_prefixes(const int64_t* F, int64_t T, int64_t x) {
    const int l = lane_id();
    const int64_t fend = F[SEG - 1];
    int64_t lsp = 0;
    ChainRun cr{x, 0, 0, -1, INT64_MIN, -1, 0};
#pragma unroll
    for (int h = 0; h < NW; h += 4) {
        int64_t f[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) f[w] = F[(h + w) * 64 + l];
#pragma unroll
        for (int w = 0; w < 4; ++w) chain_window<false>(f[w], 0, T, cr, lsp, h + w, -1);
    }
    return cr.ref - fend;
}

// The ends of the 32-bit range stand for anything beyond it: no kept 32-bit
// prefix reaches them.
// (compares of 32-bit words: a wave-uniform x stays in scalar registers)
__device__ __forceinline__ int32_t clamp32(int64_t x) {
    const int32_t lo = (int32_t)(uint32_t)(uint64_t)x, hi = (int32_t)((uint64_t)x >> 32);
    return hi == (lo >> 31) ? lo : (hi < 0 ? INT32_MIN : INT32_MAX);
}
__device__ __forceinline__ int64_t rl(int64_t v, int l) { return readlane64(v, l); }
__device__ __forceinline__ int64_t rl(int32_t v, int l) { return (int64_t)readlane32(v, l); }
template <class FT>
__device__ __forceinline__ FT threshold_of(int64_t x);
template <>
__device__ __forceinline__ int64_t threshold_of<int64_t>(int64_t x) { return x; }
template <>
__device__ __forceinline__ int32_t threshold_of<int32_t>(int64_t x) { return clamp32(x); }

// Exit offset from entry offset x, following prefixes held in registers.
__device__ __forceinline__ int64_t walk_regs(const int64_t (&f)[NW], int64_t T, int64_t x) {
    int64_t lsp = 0;
    ChainRun cr{x, 0, 0, -1, INT64_MIN, -1, 0};
#pragma unroll
    for (int w = 0; w < NW; ++w) chain_window<false>(f[w], 0, T, cr, lsp, w, -1);
    return cr.ref - readlane64(f[NW - 1], 63);
}

// Exit offset from entry offset x of a segment that moves less than T (its
// prefixes f in registers) when x lies outside its no-sample interval: the
// chain samples once, at the first node at least T above x (x below the
// interval) or at least T below it (above), and never again in the segment.
// The eight windows are tested at once, not one after another.
template <class FT>
__device__ __forceinline__ int64_t exit_one_sample(const FT (&f)[NW], int64_t T, int64_t x, bool up) {
    uint64_t m[NW];
    if (up) {  // (wave-uniform: one set of compares, not both and a select)
        const FT thr = threshold_of<FT>(x + T);
#pragma unroll
        for (int w = 0; w < NW; ++w) m[w] = ballot(f[w] >= thr);
    } else {
        const FT thr = threshold_of<FT>(x - T);
#pragma unroll
        for (int w = 0; w < NW; ++w) m[w] = ballot(f[w] <= thr);
    }
    int64_t fu = x;  // (unreachable for a stop: some node crosses)
#pragma unroll
    for (int w = NW - 1; w >= 0; --w)
        if (m[w]) fu = rl(f[w], ctz64(m[w]));
    return fu - rl(f[NW - 1], 63);
}

// The exit from the kept prefixes in HBM (all windows loaded at once).
__device__ __forceinline__ int64_t walk_kept(const Desc& D, int64_t j, bool fit, int64_t T, int64_t x) {
    int64_t f[NW];
    load_kept(D, j, fit, f);
    return walk_regs(f, T, x);
}

// Index of the r-th set bit (r < popcount(m)).
__device__ __forceinline__ int nth_bit(uint64_t m, int r) {
    for (; r > 0; --r) m &= m - 1;
    return ctz64(m);
}

// Lanes [lo, hi) of wave w as a mask (tile-wide lane indices).
__device__ __forceinline__ uint64_t range_mask(int w, int lo, int hi) {
    const int a = lo - w * 64, b = hi - w * 64;
    const uint64_t ma = a <= 0 ? ~0ull : (a >= 64 ? 0ull : (~0ull << a));
    const uint64_t mb = b >= 64 ? ~0ull : (b <= 0 ? 0ull : ((1ull << b) - 1));
    return ma & mb;
}

// The first node of a segment at least T from each lane's reference xr (a
// lane that crosses nowhere gets some node): f holds the prefixes, lane g of
// cgx and cgn the largest and smallest prefix up to the end of the eight-node
// group g: a binary search over the groups, then the nodes of one.  (Two
// levels of eight groups with their reads in flight together: 8 % slower.)
__device__ __forceinline__ int first_samples(const int32_t* f, int32_t cgx, int32_t cgn, int32_t T, int32_t xr,
                                             int32_t& v) {
    const int32_t hi = xr + T, lo = xr - T;
    int g = 0;
#pragma unroll
    for (int d = 32; d; d >>= 1) {
        const int32_t mx = shfl32(cgx, g + d - 1), mn = shfl32(cgn, g + d - 1);
        g += mx >= hi || mn <= lo ? 0 : d;
    }
    g &= 63;
    const v4i32 a = *(const v4i32*)&f[8 * g], b = *(const v4i32*)&f[8 * g + 4];
    int e = 7;
    v = b[3];
#pragma unroll
    for (int i = 6; i >= 0; --i) {
        const int32_t y = i < 4 ? a[i & 3] : b[i & 3];
        const bool c = beyond32(y, xr, T);
        e = c ? i : e;
        v = c ? y : v;
    }
    return 8 * g + e;
}

// ------------------------------------------------------------ tile maps
//
// A tile whose segments each move less than T (every SIM map holds at least
// T entries in its no-sample interval) lets an entry sample at most once per
// segment.  For such a tile the chain map over all entry offsets of the whole
// tile is computed before the resolve pass (section 3.2's rule, restated over
// entries as in the segment analysis): each of eight waves follows a block of
// 64 segments, segment by segment, and the eight maps are composed:
//  * entries that have not sampled yet form one interval U, which shrinks as
//    the tile's running maximum and minimum footprint grow apart;
//  * at each new running maximum (minimum) node while U is not empty, the
//    entries of U at least T below (above) that node sample there: they form
//    one source interval and start a chain whose reference is that node's
//    footprint;
//  * a chain outside a segment's no-sample interval samples once in it, at
//    the first node at least T above (below) its reference;
//  * chains that sample at the same node coincide from there on and are
//    merged (their sources are joined in a union-find forest).
// Source intervals started at maxima lie below U and grow upward in start
// order; those started at minima lie above it and grow downward.  Runs of
// consecutive sources that end at the same reference are written as (bound,
// exit) pairs, so that the tile's exit for any entry is one search.  Waves
// that have finished a tile chain the trace's tile entries through the maps in
// tile order and publish every tile's exit, so that the resolve pass does not
// wait for the previous tile's walk.  A tile that
// does not qualify, or whose chains or runs exceed the capacities below, gets
// no map; the resolve pass chains the tiles from it on, by a map lookup where
// a tile has one and by its walk where not.

constexpr int TM_CAP = 1024;   // chains followed at once (64-bit path)
constexpr int TM_SRC = 2048;   // source intervals per tile (64-bit path)
constexpr int TM_SIDE = 128;   // runs per side (below and above U)
constexpr int64_t TM_WORDS = (int64_t)(TILE_MAP_BYTES / 8);
// Run r of side s (0: below U, 1: above) has its bound at run_word(s, 0, r)
// and its exit at run_word(s, 1, r).  Runs l < 64 of both sides lie in words
// 4l..4l+3 (bound and exit below U, bound and exit above: one lane's words,
// two 16-byte loads), followed by the header (state, runs below, runs above,
// tile change) at word 256; runs 64-127 follow at word 512 the same way.
constexpr int TM_HDR = 256;
constexpr int TM_RUN_HI = 512;
__device__ __forceinline__ int run_word(int side, int which, int r) {
    return (r < 64 ? 0 : TM_RUN_HI) + 4 * (r & 63) + 2 * side + which;
}
constexpr int TM_SB = 1024;    // source bounds (scratch while the map is built)
constexpr int TM_SD = 3072;    // source sides, one byte each: 1 = below U (scratch)
enum { TM_MAPPED = 1, TM_NONE = 2 };
// causes of a tile without a map (control words 7-10 count them)
enum { TMF_QUALIFY = 1, TMF_SOURCES, TMF_CHAINS, TMF_RUNS };

// The map area of tile k: the tracked-list area, unused until the tracked
// list is built at the end of the launch (16 bytes per event against 4 bytes
// per event needed here).
__device__ __forceinline__ SMP_GLOBAL int64_t* tile_map(const Desc& D, int64_t k) {
    return gp((int64_t*)D.tracked) + k * TM_WORDS;
}
// A word of a map that another wave reads in the same launch: stored through
// to memory, as the look-back words are.
__device__ __forceinline__ void st_map(SMP_GLOBAL int64_t* p, int64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// First node of a segment (relative prefixes f) whose prefix is >= thr (GE)
// or <= thr (LE); SEG if none.  Branch-free: one compare per window, then a
// select per window from the last one down.
template <bool GE>
__device__ __forceinline__ int first_node(const int64_t (&f)[NW], int64_t thr) {
    uint64_t m[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) m[w] = ballot(GE ? f[w] >= thr : f[w] <= thr);
    int k = SEG;
#pragma unroll
    for (int w = NW - 1; w >= 0; --w) k = m[w] ? w * 64 + ctz64(m[w]) : k;
    return k;
}
// The same for two thresholds at once (independent, so their instructions interleave).
template <bool GE>
__device__ __forceinline__ void first_node2(const int64_t (&f)[NW], int64_t t1, int64_t t2, int& k1, int& k2) {
    uint64_t m1[NW], m2[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        m1[w] = ballot(GE ? f[w] >= t1 : f[w] <= t1);
        m2[w] = ballot(GE ? f[w] >= t2 : f[w] <= t2);
    }
    k1 = SEG;
    k2 = SEG;
#pragma unroll
    for (int w = NW - 1; w >= 0; --w) {
        k1 = m1[w] ? w * 64 + ctz64(m1[w]) : k1;
        k2 = m2[w] ? w * 64 + ctz64(m2[w]) : k2;
    }
}

// The exit of a tile from entry e, from its map's runs (two per lane and
// side: runs l and 64 + l, bound and exit) and header values.
static_assert(TM_SIDE == 128, "map_exit takes two runs per lane and side");
__device__ __forceinline__ int64_t map_exit(int64_t e, int nup, int ndn, int64_t tF, int64_t ub0, int64_t ub1,
                                            int64_t ue0, int64_t ue1, int64_t db0, int64_t db1, int64_t de0,
                                            int64_t de1) {
    const int l = lane_id();
    // below U: the first run whose (upper) bound is >= e
    const uint64_t u0 = ballot(l < nup && ub0 >= e), u1 = ballot(64 + l < nup && ub1 >= e);
    if (u0) return readlane64(ue0, ctz64(u0));
    if (u1) return readlane64(ue1, ctz64(u1));
    // above U: the first run whose (lower) bound is <= e
    const uint64_t d0 = ballot(l < ndn && db0 <= e), d1 = ballot(64 + l < ndn && db1 <= e);
    if (d0) return readlane64(de0, ctz64(d0));
    if (d1) return readlane64(de1, ctz64(d1));
    return e - tF;  // in U: no sample in the tile
}

// The same for a map of at most 64 runs per side (one per lane; vu, vd:
// the lanes that hold one), without branches: both searches, then selects.
__device__ __forceinline__ int64_t map_exit64(int64_t e, uint64_t vu, uint64_t vd, int64_t tF, int64_t ub, int64_t ue,
                                              int64_t db, int64_t de) {
    const uint64_t u = vu & ballot(ub >= e), d = vd & ballot(db <= e);
    const int64_t xu = readlane64(ue, u ? ctz64(u) : 0), xd = readlane64(de, d ? ctz64(d) : 0);
    return u ? xu : (d ? xd : e - tF);
}

// The tile entries of a trace, chained through the maps of tiles t0 to nt - 1
// by one wave: each tile's exit is published as the word the resolve pass
// waits for.  It stops at the first tile without a map; returns the tiles
// chained.  Tiles are taken TC_CB at a time, the next ones' words loading
// while these are looked up.
constexpr int TC_CB = 8;
__device__ int chain_maps(const Desc& D, int t0, int nt, unsigned long long* ctl) {
    const int l = lane_id();
    const StatusView ts{D.tstat, (int64_t)D.ntile};
    // lane l: runs l of both sides (bound, exit below U; bound, exit above);
    // lanes 0-3: the header
    auto load = [&](int at, int64_t (&w)[TC_CB][4], int64_t (&h)[TC_CB]) {
#pragma unroll
        for (int b = 0; b < TC_CB; ++b) {
            const SMP_GLOBAL int64_t* m = tile_map(D, at + b < nt ? at + b : nt - 1);
#pragma unroll
            for (int q = 0; q < 4; ++q) w[b][q] = m[4 * l + q];
            h[b] = m[TM_HDR + (l & 3)];
        }
    };
    int64_t nw[TC_CB][4], nh[TC_CB];
    load(t0, nw, nh);
    // tile 0's entry is 0, every other's the exit published before it
    // (always there: the chain is freed after its exits are in memory)
    const uint64_t before = t0 ? readlaneu64(ld_status(ts.at(W_XF, t0 - 1)), 0) : 0;
    if (t0 && !wstate(before)) return 0;
    int64_t e = t0 ? unpack(before) : 0;
    int t = t0;
    for (; t < nt;) {
        int64_t cw[TC_CB][4], ch[TC_CB];
#pragma unroll
        for (int b = 0; b < TC_CB; ++b) {
            ch[b] = nh[b];
#pragma unroll
            for (int q = 0; q < 4; ++q) cw[b][q] = nw[b][q];
        }
        if (t + TC_CB < nt) load(t + TC_CB, nw, nh);
        const int nb = (nt - t) < TC_CB ? (nt - t) : TC_CB;
        // everything that does not depend on the entry first: the tiles that
        // can be chained, their runs and tile changes
        int nm = 0;
        int64_t nup[TC_CB], ndn[TC_CB], tFs[TC_CB];
        uint64_t vu[TC_CB], vd[TC_CB];
#pragma unroll
        for (int b = 0; b < TC_CB; ++b) {
            nm += (b == nm && b < nb && readlane64(ch[b], 0) == TM_MAPPED) ? 1 : 0;
            nup[b] = readlane64(ch[b], 1);
            ndn[b] = readlane64(ch[b], 2);
            tFs[b] = readlane64(ch[b], 3);
            vu[b] = ballot(l < nup[b]);
            vd[b] = ballot(l < ndn[b]);
        }
        int done = 0;
        int64_t xs = 0;  // lane b: the exit of tile t + b
#pragma unroll
        for (int b = 0; b < TC_CB; ++b) {
            if (b >= nm) break;
            int64_t x;
            if (nup[b] <= 64 && ndn[b] <= 64) {
                x = map_exit64(e, vu[b], vd[b], tFs[b], cw[b][0], cw[b][1], cw[b][2], cw[b][3]);
            } else {  // more than 64 runs on a side: the rest from the map itself
                const SMP_GLOBAL int64_t* m = tile_map(D, t + b) + TM_RUN_HI + 4 * l;
                x = map_exit(e, (int)nup[b], (int)ndn[b], tFs[b], cw[b][0], m[0], cw[b][1], m[1], cw[b][2], m[2],
                             cw[b][3], m[3]);
            }
            xs = l == b ? x : xs;
            e = x;
            ++done;
        }
        if (l < done) st_status(ts.at(W_XF, t + l), pack(xs, 1));
        t += done;
        if (done < nb) break;  // a tile without a map
    }
    if (l == 0 && t > t0) g_add((uint64_t*)&ctl[6], (uint64_t)(t - t0));
    return t - t0;
}

// Chain what can be chained, by the wave that has just written a tile's map:
// it marks the tile (D.blk, cleared again by the resolve pass), and whichever
// wave finds the chain free takes it on from where it stands over the marked
// tiles.  A wave that finds it held leaves: the holder looks again after it has
// freed the chain.  A tile without a map is never marked and ends the chain.
// So the chain runs beside the builds (5e8 events, 1,908 tiles: 0.7 ms of it),
// not after them, and no wave waits for another.
__device__ void chain_mapped_tiles(const Desc& D, int64_t k, unsigned long long* ctl) {
    const int l = lane_id();
    const int nt = __builtin_amdgcn_readfirstlane((int)D.ntile);
    auto marked = [&](int pos) {  // tiles marked from pos on, without a gap
        const int t = pos + l;
        const uint64_t m = ballot(t < nt && ld_status(D.blk + (t < nt ? t : 0)) != 0);
        return ~m ? ctz64(~m) : 64;
    };
    stores_done();  // the map is in memory before the mark
    if (l == 0) st_status(D.blk + k, 1);
    int pos;
    do {
        stores_done();  // the mark (the freed chain) before the chain is asked for
        uint64_t held = 0;
        if (l == 0)
            held = __hip_atomic_exchange(gp(&D.scal->tmap_held), 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (readlaneu64(held, 0)) return;
        pos = readlane32((int)__hip_atomic_load(gp(&D.scal->tmap_pos), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), 0);
        for (int n; pos < nt && (n = marked(pos)) > 0;) {
            // drop stale copies of the tiles' words before they are read
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            pos = chain_maps(D, pos, pos + n, ctl) < n ? nt : pos + n;
        }
        if (l == 0)
            __hip_atomic_store(gp(&D.scal->tmap_pos), (uint32_t)pos, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        stores_done();  // the exits and the position before the chain is free
        if (l == 0) __hip_atomic_store(gp(&D.scal->tmap_held), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        stores_done();  // free before the marks are looked at again
    } while (pos < nt && marked(pos) > 0);
}

// The map of a tile past the 32-bit range, by one wave over all its segments
// (64-bit references, prefixes loaded as they are used).  Returns the cause
// if it fails, 0 if the runs are written.
struct TmapWide {
    int64_t cx[TM_CAP];       // live chains: reference (tile coordinates)
    uint16_t cr[TM_CAP];      // and the root source of their set
    uint16_t par[TM_SRC];     // union-find parent of each source
    // per segment: its prefixes, and per node the chain that sampled there
    // first (see claim below); at the end: the live chain of each root
    int64_t u[(SEG * 8 + SEG * 4 > TM_SRC * 2 ? SEG * 8 + SEG * 4 : TM_SRC * 2) / 8];
};
__device__ int tmap_wide(const Desc& D, int64_t k, int nval, TmapWide& W, SMP_GLOBAL int64_t* map) {
    int64_t (&cx)[TM_CAP] = W.cx;
    uint16_t (&cr)[TM_CAP] = W.cr;
    uint16_t (&par)[TM_SRC] = W.par;
    int64_t* fl = W.u;
    uint32_t* claim = (uint32_t*)(W.u + SEG);
    uint16_t* cidx = (uint16_t*)W.u;
    const int l = lane_id();
    const int64_t ns = (int64_t)D.nseg;
    const int64_t T = D.T;
    SMP_GLOBAL uint8_t* sside = (SMP_GLOBAL uint8_t*)(map + TM_SD);
    const SMP_GLOBAL int64_t* sp = gp(D.seg) + k * TILE;
    for (int i = l; i < SEG; i += 64) claim[i] = 0;
    int nch = 0, nsrc = 0;
    int fail = 0;  // cause, 0 while the map holds
    int64_t Umax = 0, Umin = 0, carry = 0;  // running extremes (from the tile start), footprint change so far
    // segments g..g+63, one per lane: offset, no-sample bounds and extremes in tile coordinates
    int64_t gR = 0, gL = 0, gH = 0, gX = 0, gN = 0;
    auto step = [&](int s, const int64_t (&f)[NW]) {
        if ((s & 63) == 0) {
            const int j = s + l;
            const bool v = j < nval;
            const int64_t af = v ? sp[SP_AF * ns + j] : 0;
            const int64_t lo = v ? sp[SP_LO * ns + j] : 0, hi = v ? sp[SP_HI * ns + j] : 0;
            const int64_t mx = v ? sp[SP_MXF * ns + j] : 0, mn = v ? sp[SP_MNF * ns + j] : 0;
            const int64_t inc = wave_incl_sum(af);
            gR = carry + inc - af;
            carry += readlane64(inc, 63);
            gL = gR + lo;
            gH = gR + hi;
            gX = gR + mx;
            gN = gR + mn;
        }
        const int i = s & 63;
        const int64_t R = readlane64(gR, i), Ls = readlane64(gL, i), Hs = readlane64(gH, i);
        const int64_t Sx = readlane64(gX, i), Sn = readlane64(gN, i);
        // the prefixes in LDS: the value at a sampled node is read from there
#pragma unroll
        for (int w = 0; w < NW; ++w) fl[w * 64 + l] = f[w];
        // Chains that sample at one node merge into the first of them.
        // claim[node] (step numbers from 1): step << 16 | 0x7FFF - chain
        // while chains compete for it (the largest wins: the earliest
        // chain), then step << 16 | 0x8000 | root of the winner's set.
        const uint32_t stag = (uint32_t)(s + 1) << 16;
        // live chains: those outside the no-sample interval sample once here
        // (each group's words load while the one before it is processed:
        // the compaction below never writes past the group it processes)
        int out = 0;
        int64_t Xn = l < nch ? cx[l] : 0;
        int rtn = l < nch ? (int)cr[l] : 0;
        for (int c0 = 0; c0 < nch; c0 += 64) {
            const int c = c0 + l;
            const bool v = c < nch;
            int64_t X = Xn;
            const int rt = rtn;
            if (c0 + 64 < nch) {
                const int cn = c + 64;
                Xn = cn < nch ? cx[cn] : 0;
                rtn = cn < nch ? (int)cr[cn] : 0;
            }
            const uint64_t vm = ballot(v);
            uint64_t alive = vm;
            bool moved = false;  // sampled here and keeps its chain
            const bool up = v && X < Ls;
            const uint64_t sm0 = ballot(up || (v && X > Hs));
            if (sm0) {
                // each sampling chain's node: two chains of one direction at a time
                const uint64_t um = ballot(up), dm = sm0 & ~um;
                const int64_t thr = up ? X - R + T : X - R - T;
                int xnode = SEG;
#define SMP_TM_SEARCH(MASK, GE)                                                 \
    for (uint64_t m_ = (MASK); m_;) {                                           \
        const int q1 = ctz64(m_);                                               \
        m_ &= m_ - 1;                                                           \
        const int64_t th1 = readlane64(thr, q1);                                \
        if (m_) {                                                               \
            const int q2 = ctz64(m_);                                           \
            m_ &= m_ - 1;                                                       \
            int n1, n2;                                                         \
            first_node2<GE>(f, th1, readlane64(thr, q2), n1, n2);               \
            xnode = l == q1 ? n1 : (l == q2 ? n2 : xnode);                      \
        } else {                                                                \
            const int n1 = first_node<GE>(f, th1);                              \
            xnode = l == q1 ? n1 : xnode;                                       \
        }                                                                       \
    }
                SMP_TM_SEARCH(um, true)
                SMP_TM_SEARCH(dm, false)
#undef SMP_TM_SEARCH
                const bool mine = (sm0 >> l) & 1;
                if (ballot(mine && xnode >= SEG)) {  // (unreachable: a chain outside the interval crosses)
                    fail = TMF_QUALIFY;
                    break;
                }
                // merges, for the whole group at once
                const uint32_t key = stag | (uint32_t)(0x7FFF - c);
                if (mine) __hip_atomic_fetch_max(&claim[xnode], key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                const uint32_t got =
                    mine ? __hip_atomic_load(&claim[xnode], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : 0;
                const bool win = mine && got == key;
                if (win)
                    __hip_atomic_store(&claim[xnode], stag | 0x8000u | (uint32_t)rt, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
                const bool lose = mine && !win;
                // the winner's root: in the claim once resolved (an earlier
                // group), else held by the winner's lane in this group
                const int wl = (int)(0x7FFFu - (got & 0x7FFFu)) - c0;
                const int wr = shfl32(rt, (got & 0x8000u) ? l : (wl & 63));
                if (lose) par[rt] = (uint16_t)((got & 0x8000u) ? (got & 0x7FFFu) : (uint32_t)wr);
                alive &= ~ballot(lose);
                if (win) X = R + fl[xnode];
                moved = win;
            }
            // compact in place (survivors never move up); while no chain of
            // this step has merged, only the sampled references change
            if (out == c0 && alive == vm) {
                if (moved) cx[c] = X;
            } else if ((alive >> l) & 1) {
                const int o = out + __popcll(alive & lanemask_lt());
                cx[o] = X;
                cr[o] = (uint16_t)rt;
            }
            out += __popcll(alive);
        }
        nch = out;
        // New running extremes while U is not empty start chains.  A window
        // with no node beyond the extremes so far leaves them unchanged; in
        // the others, the extremes before each node come from a scan.
        if (!fail && Umax - Umin <= 2 * T - 2 && (Sx > Umax || Sn < Umin)) {
            int64_t cm = Umax, cn = Umin;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                if (cm - cn > 2 * T - 2 || fail) break;
                const int64_t gv = R + f[w];
                if (!ballot(gv > cm || gv < cn)) continue;
                int64_t im = wave_incl_max(gv), in = wave_incl_min(gv);
                im = im > cm ? im : cm;
                in = in < cn ? in : cn;
                const int64_t pm = wave_shr1(im, cm), pn = wave_shr1(in, cn);  // before the node
                const bool open = pm - pn <= 2 * T - 2;
                const bool up = open && gv > pm, dn = open && gv < pn;
                const uint64_t spm = ballot(up || dn);
                cm = readlane64(im, 63);
                cn = readlane64(in, 63);
                if (!spm) continue;
                const int cnt = __popcll(spm);
                if (nsrc + cnt > TM_SRC) {
                    fail = TMF_SOURCES;
                    break;
                }
                // sources in node order; the entries of U = [pm - T + 1,
                // pn + T - 1] that sample at this node
                const bool sp_ = (spm >> l) & 1;
                const int src = nsrc + __popcll(spm & lanemask_lt());
                const int64_t bound = up ? ((pn + T - 1) < (gv - T) ? (pn + T - 1) : (gv - T))
                                         : ((pm - T + 1) > (gv + T) ? (pm - T + 1) : (gv + T));
                // a chain that sampled at the same node takes the source into its set
                const uint32_t cl =
                    sp_ ? __hip_atomic_load(&claim[w * 64 + l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : 0;
                const bool hit = sp_ && (cl >> 16) == (stag >> 16);
                const uint64_t nm = spm & ~ballot(hit);  // new chains
                if (nch + __popcll(nm) > TM_CAP) {
                    fail = TMF_CHAINS;
                    break;
                }
                if (sp_) {
                    map[TM_SB + src] = bound;
                    sside[src] = up ? 1 : 0;
                    par[src] = (uint16_t)(hit ? (cl & 0x7FFFu) : (uint32_t)src);
                }
                if ((nm >> l) & 1) {
                    const int o = nch + __popcll(nm & lanemask_lt());
                    cx[o] = gv;
                    cr[o] = (uint16_t)src;
                }
                nsrc += cnt;
                nch += __popcll(nm);
            }
        }
        Umax = Sx > Umax ? Sx : Umax;
        Umin = Sn < Umin ? Sn : Umin;
    };
    const int64_t j0 = k * TILE;
    for (int s = 0; s < nval && !fail; ++s) {
        int64_t f[NW];
        load_kept(D, j0 + s, (sp[SP_FLG * ns + s] & FLG_FIT) != 0, f);
        step(s, f);
    }
    // runs: consecutive sources of one side that end at the same reference
    int nup = 0, ndn = 0;
    if (!fail) {
        const int64_t tF = carry;
        for (int i = l; i < nsrc; i += 64) cidx[i] = 0;
        for (int c0 = 0; c0 < nch; c0 += 64)
            if (c0 + l < nch) cidx[cr[c0 + l]] = (uint16_t)(c0 + l);
        // the source bounds and sides stored above (by this wave), before they are read back
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        int64_t lastU = 0, lastD = 0;  // exit of the previous source of each side
        for (int s0 = 0; s0 < nsrc; s0 += 64) {
            const int s = s0 + l;
            const bool v = s < nsrc;
            int r = s;
            for (int d = 0; v && d < TM_SRC && par[r] != r; ++d) r = par[r];
            const int64_t ex = v ? cx[cidx[r]] - tF : 0;
            const int64_t bnd = v ? map[TM_SB + s] : 0;
            const bool isup = v && sside[s] != 0;
            const bool isdn = v && !isup;
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const bool mine = side == 0 ? isup : isdn;
                const uint64_t sm = ballot(mine);
                if (!sm) continue;
                int& cnt = side == 0 ? nup : ndn;
                int64_t& last = side == 0 ? lastU : lastD;
                // the previous source of this side: an earlier lane, else the carried one
                const uint64_t before = sm & lanemask_lt();
                const int64_t pe = shfl64(ex, before ? top64(before) : 0);
                const bool has_prev = before != 0 || cnt > 0;
                const int64_t prev = before ? pe : last;
                const bool start = mine && (!has_prev || ex != prev);
                const uint64_t stm = ballot(start);
                const int run = cnt + __popcll(stm & (lanemask_lt() | (1ull << l))) - 1;
                // a source whose next source of this side (in this group)
                // starts a new run, or that is the group's last, writes its
                // bound; a later group may still extend its run
                const uint64_t after = sm & ~(lanemask_lt() | (1ull << l));
                const bool ends = mine && (!after || ((stm >> ctz64(after)) & 1));
                const int nr = cnt + __popcll(stm);
                if (nr > TM_SIDE) {
                    fail = TMF_RUNS;
                    break;
                }
                if (start) st_map(map + run_word(side, 1, run), ex);
                if (ends) st_map(map + run_word(side, 0, run), bnd);
                cnt = nr;
                last = readlane64(ex, top64(sm));
            }
            if (fail) break;
        }
        if (!fail && l == 0) {
            st_map(map + TM_HDR + 1, nup);
            st_map(map + TM_HDR + 2, ndn);
            st_map(map + TM_HDR + 3, tF);
        }
    }
    return fail;
}

// A 32-bit tile: eight waves, each following the chains of its 64 segments,
// then the eight maps composed.  Chains that stop in a segment are searched
// side by side (64 at a time).  Bound: the serial steps of 64 segments (one
// wave over all 512 took 0.88 ms whatever the number of tiles).
constexpr int TS_SRC = 2048;  // sources per block, pieces per tile
constexpr int TS_CAP = 1088;  // chains followed at once
constexpr int TS_UNROLL = 4;
constexpr int TS_FRESH = 43;  // segments with new extremes a tile may have
constexpr int32_t TS_DEAD = INT32_MIN;
struct TmapBuild {
    int32_t cx[TS_CAP];       // live chains: reference (block coordinates), TS_DEAD once merged
    uint16_t cr[TS_CAP];      // and the root source of their set
    uint16_t par[TS_SRC];     // union-find parent of each source
    union {
        struct {
            int32_t f[SEG];       // the current segment's prefixes
            uint32_t claim[SEG];  // the chain that sampled at each node: (segment + 1) << 16 | root
            uint16_t lst[TS_CAP]; // the chains that stop in it
        } s;
        uint16_t cidx[TS_SRC];    // at the end: the live chain of each root
    } u;
};
// A map as runs: those below the unsampled interval from the front (bounds
// growing: the largest entry of each), those above it from the back (bounds
// falling: the smallest).
struct TmapRuns {
    int32_t b[TS_SRC], e[TS_SRC];
};
union alignas(16) TmapLds {
    TmapBuild build;
    TmapRuns runs;
};
struct TmapBlock {
    int nup, ndn;
    int32_t lo, hi;  // unsampled entries (none: lo > hi)
    int64_t rend;    // the block's footprint change
    int fail;
};
// Scratch of block b of tile k (sources' bounds and exits), behind the tiles' maps.
__device__ __forceinline__ SMP_GLOBAL int32_t* tmap_scratch(const Desc& D, int64_t k, int b) {
    return (SMP_GLOBAL int32_t*)((SMP_GLOBAL uint8_t*)gp((uint8_t*)D.tracked) + (uint64_t)D.ntile * TILE_MAP_BYTES) +
           (k * TWAVES + b) * (2 * TS_SRC);
}
static_assert(TILE_MAP_BYTES + TWAVES * 2 * TS_SRC * 4 <= TILE_MAP_ROOM, "scratch of a tile");

// Runs of one side among 64 lanes in order (mine: lanes of that side, ex:
// their exits, bnd: their bounds): store(run, which, value) writes a run's
// bound (0) and exit (1).  cnt: runs so far, last: the exit of the latest.
template <class F>
__device__ __forceinline__ void add_runs(bool mine, int64_t ex, int64_t bnd, int& cnt, int64_t& last, F store) {
    const uint64_t sm = ballot(mine);
    if (!sm) return;
    // the previous one of this side: an earlier lane, else the carried one
    const uint64_t before = sm & lanemask_lt();
    const int64_t pe = shfl64(ex, before ? top64(before) : 0);
    const bool start = mine && ((before == 0 && cnt == 0) || ex != (before ? pe : last));
    const uint64_t stm = ballot(start), le = lanemask_lt() | (1ull << lane_id());
    const int run = cnt + __popcll(stm & le) - 1;
    // one whose next of this side starts a new run, or that is the last of
    // these lanes, writes the bound (a later call may still extend its run)
    const uint64_t after = sm & ~le;
    const bool ends = mine && (!after || ((stm >> ctz64(after)) & 1));
    if (start) store(run, 1, ex);
    if (ends) store(run, 0, bnd);
    cnt += __popcll(stm);
    last = readlane64(ex, top64(sm));
}

// Follow all entries through the block of nb segments at j0 (lane i: segment
// i's offset and extremes, block coordinates) and leave its runs in X.
__device__ TmapBlock tmap_block(const Desc& D, int64_t k, int64_t j0, int b, int nb, int32_t T, int32_t Rv, int32_t Sxv,
                                int32_t Snv, int32_t rend, TmapLds& X) {
    const int l = lane_id();
    TmapBuild& B = X.build;
    SMP_GLOBAL int32_t* sb = tmap_scratch(D, k, b);  // 2 * bound + (below the interval ? 1 : 0)
    SMP_GLOBAL int32_t* se = sb + TS_SRC;            // exit
    int nch = 0, nsrc = 0, dead = 0, fail = 0;
    int32_t Umax = 0, Umin = 0;
    bool open = true;
    for (int i = l; i < SEG; i += 64) B.u.s.claim[i] = 0;
    int32_t pf[NW];  // the next segment's prefixes, loading
    if (nb > 0) load_kept32(D, j0, pf);
    for (int s = 0; s < nb && !fail; ++s) {
        const int32_t R = readlane32(Rv, s), Sx = readlane32(Sxv, s), Sn = readlane32(Snv, s);
        int nst = 0;
        for (int c0 = 0; c0 < nch; c0 += 64 * TS_UNROLL) {  // (the groups' reads overlap)
            int32_t x[TS_UNROLL];
#pragma unroll
            for (int q = 0; q < TS_UNROLL; ++q) {
                const int c = c0 + 64 * q + l;
                x[q] = c < nch ? B.cx[c] : TS_DEAD;
            }
#pragma unroll
            for (int q = 0; q < TS_UNROLL; ++q) {
                const bool st = x[q] != TS_DEAD && (x[q] <= Sx - T || x[q] >= Sn + T);
                const uint64_t m = ballot(st);
                if (st) B.u.s.lst[nst + __popcll(m & lanemask_lt())] = (uint16_t)(c0 + 64 * q + l);
                nst += __popcll(m);
            }
        }
        const bool fresh = open && (Sx > Umax || Sn < Umin);
        int32_t cur[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) cur[w] = pf[w];
        load_kept32(D, j0 + (s + 1 < nb ? s + 1 : s), pf);
        if (nst) {
#pragma unroll
            for (int w = 0; w < NW; ++w) B.u.s.f[w * 64 + l] = cur[w];
        }
        if (nst) {
            // the running extremes of the eight-node groups
            const v4i32 a = *(const v4i32*)&B.u.s.f[8 * l], c4 = *(const v4i32*)&B.u.s.f[8 * l + 4];
            int32_t gx = a[0], gn = a[0];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                gx = a[i] > gx ? a[i] : gx;
                gx = c4[i] > gx ? c4[i] : gx;
                gn = a[i] < gn ? a[i] : gn;
                gn = c4[i] < gn ? c4[i] : gn;
            }
            gx = wave_incl_ext32<true>(gx);
            gn = wave_incl_ext32<false>(gn);
            for (int i0 = 0; i0 < nst; i0 += 64) {
                const bool mine = i0 + l < nst;
                const int c = mine ? B.u.s.lst[i0 + l] : 0;
                const int32_t x = B.cx[c], xr = mine ? x - R : 0;
                const int root = B.cr[c];
                int32_t v;
                const int node = first_samples(B.u.s.f, gx, gn, T, xr, v);
                // chains that sample at one node merge into the one that claims it
                // (an LDS exchange in place of these three accesses: 4 % slower)
                const uint32_t key = (uint32_t)(s + 1) << 16 | (uint32_t)root;
                uint32_t got = mine ? B.u.s.claim[node] : 0;
                const bool taken = (got >> 16) == (uint32_t)(s + 1);
                if (mine && !taken) B.u.s.claim[node] = key;
                asm volatile("" ::: "memory");  // (several lanes may write one claim: what it holds is read back)
                if (mine && !taken) got = B.u.s.claim[node];
                const bool win = mine && got == key;
                if (mine) B.cx[c] = win ? R + v : TS_DEAD;
                if (mine && !win) B.par[root] = (uint16_t)(got & 0xFFFFu);
                dead += __popcll(ballot(mine && !win));
            }
        }
        if (fresh) {
            // nodes beyond the extremes so far: first samples of unsampled entries
            int32_t cm = Umax, cn = Umin;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                if (fail || cm - cn > 2 * T - 2) break;
                const int32_t gv = R + cur[w];
                if (!ballot(gv > cm || gv < cn)) continue;
                int32_t im = wave_incl_ext32<true>(gv), in = wave_incl_ext32<false>(gv);
                im = im > cm ? im : cm;
                in = in < cn ? in : cn;
                const int32_t pm = wave_shr1_32(im, cm), pn = wave_shr1_32(in, cn);  // before the node
                const bool op = pm - pn <= 2 * T - 2;
                const bool up = op && gv > pm, dn = op && gv < pn;
                const uint64_t spm = ballot(up || dn);
                cm = readlane32(im, 63);
                cn = readlane32(in, 63);
                const int cnt = __popcll(spm);
                if (nsrc + cnt > TS_SRC) {
                    fail = TMF_SOURCES;
                    break;
                }
                const bool mine = (spm >> l) & 1;
                const int src = nsrc + __popcll(spm & lanemask_lt());
                const uint32_t cl = mine ? B.u.s.claim[w * 64 + l] : 0;
                const bool hit = (cl >> 16) == (uint32_t)(s + 1);
                const uint64_t nm = spm & ~ballot(hit);  // new chains
                if (nch + __popcll(nm) > TS_CAP) {
                    fail = TMF_CHAINS;
                    break;
                }
                if (mine) {
                    sb[src] = up ? 2 * (pn + T - 1 < gv - T ? pn + T - 1 : gv - T) + 1
                                 : 2 * (pm - T + 1 > gv + T ? pm - T + 1 : gv + T);
                    B.par[src] = (uint16_t)(hit ? (cl & 0xFFFFu) : (uint32_t)src);
                }
                if ((nm >> l) & 1) {
                    const int o = nch + __popcll(nm & lanemask_lt());
                    B.cx[o] = gv;
                    B.cr[o] = (uint16_t)src;
                }
                nsrc += cnt;
                nch += __popcll(nm);
            }
        }
        Umax = Sx > Umax ? Sx : Umax;
        Umin = Sn < Umin ? Sn : Umin;
        open = open && Umax - Umin <= 2 * T - 2;
        if (dead >= 64 || (dead && nch > TS_CAP - 192)) {  // drop the merged chains (survivors never move up)
            int out = 0;
            for (int c0 = 0; c0 < nch; c0 += 64) {
                const int c = c0 + l;
                const int32_t x = c < nch ? B.cx[c] : TS_DEAD;
                const uint16_t r = c < nch ? B.cr[c] : 0;
                const uint64_t m = ballot(x != TS_DEAD);
                asm volatile("" ::: "memory");
                if (x != TS_DEAD) {
                    const int o = out + __popcll(m & lanemask_lt());
                    B.cx[o] = x;
                    B.cr[o] = r;
                }
                out += __popcll(m);
            }
            nch = out;
            dead = 0;
        }
    }
    TmapBlock r{0, 0, 1, 0, rend, fail};
    if (fail) return r;
    if (open) {
        r.lo = Umax - T + 1;
        r.hi = Umin + T - 1;
    }
    // each source's exit: its root's chain
    asm volatile("" ::: "memory");
    for (int c0 = 0; c0 < nch; c0 += 64)
        if (c0 + l < nch && B.cx[c0 + l] != TS_DEAD) B.u.cidx[B.cr[c0 + l]] = (uint16_t)(c0 + l);
    asm volatile("" ::: "memory");
    for (int s0 = 0; s0 < nsrc; s0 += 64) {
        const int src = s0 + l;
        if (src < nsrc) {
            int id = src;
            for (int d = 0; d < TS_SRC && B.par[id] != id; ++d) id = B.par[id];
            se[src] = B.cx[B.u.cidx[id]] - rend;
        }
    }
    // the runs of both sides (what this wave stored above is read back, and
    // the words of the build are done with)
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    int64_t lastU = 0, lastD = 0;
    for (int s0 = 0; s0 < nsrc; s0 += 64) {
        const int src = s0 + l;
        const bool v = src < nsrc;
        const int32_t b2 = v ? sb[src] : 0, ex = v ? se[src] : 0;
        add_runs(v && (b2 & 1), ex, b2 >> 1, r.nup, lastU,
                 [&](int run, int which, int64_t x) { (which ? X.runs.e : X.runs.b)[run] = (int32_t)x; });
        add_runs(v && !(b2 & 1), ex, b2 >> 1, r.ndn, lastD,
                 [&](int run, int which, int64_t x) { (which ? X.runs.e : X.runs.b)[TS_SRC - 1 - run] = (int32_t)x; });
    }
    return r;
}

// First of n bounds at p (step d: 1 upward, -1 from the back) that is >= e (GE) or <= e.
template <bool GE>
__device__ __forceinline__ int first_bound(const int32_t* p, int d, int n, int32_t e) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        const int32_t b = p[d * mid];
        if (GE ? b >= e : b <= e) hi = mid; else lo = mid + 1;
    }
    return lo;
}
__device__ __forceinline__ int32_t runs_exit(const TmapRuns& M, const TmapBlock& m, int32_t e) {
    if (e >= m.lo && e <= m.hi) return e - (int32_t)m.rend;
    const int u = first_bound<true>(M.b, 1, m.nup, e);
    if (u < m.nup) return M.e[u];
    const int d = first_bound<false>(M.b + TS_SRC - 1, -1, m.ndn, e);
    return M.e[TS_SRC - 1 - (d < m.ndn ? d : 0)];
}

// One workgroup per tile (grid: every tile of the launch; tiles of traces
// without maps return at once).  2e7 events at T = 64 MiB (77 tiles): 0.21 ms
// (a tile: 134 us of block builds, 19 us waiting for the slowest, 8 us of
// composing; chaining the tiles 0.4 us each), 0.88 ms with one wave per tile.
// 5e8 events (1,908 tiles, one workgroup per CU at a time): 1.50 ms with the
// chaining beside the builds, 2.2 ms with it after them, 1.97 ms with one wave
// per tile.
__global__ __launch_bounds__(TILE) void k_tmap(const Desc* __restrict__ desc, int ntraces, unsigned long long* ctl,
                                               uint64_t* ts) {
    stamp(ts);
    __shared__ union {
        TmapLds blk[TWAVES];
        TmapWide wide;
    } u_;
    __shared__ TmapRuns pieces;  // the tile's map so far (runs not yet joined)
    __shared__ TmapBlock s_blk[TWAVES];
    __shared__ int s_bad[TWAVES];  // not 0: the tile does not qualify, then: it needs the wide path
    __shared__ int64_t s_ext[3][TWAVES];  // each block's footprint change, largest and smallest footprint
    __shared__ int s_new[TWAVES];  // segments with a new extreme while entries are unsampled
    const int tid = threadIdx.x, l = lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint64_t tk = blockIdx.x;
    const Desc& D = desc[find_trace_tile(desc, ntraces, tk)];
    if (!D.tmap) return;
    const int64_t k = (int64_t)(tk - D.tile_begin);
    const int64_t ns = (int64_t)D.nseg;
    const int nval = (int)((ns - k * TILE) < TILE ? (ns - k * TILE) : TILE);
    const int64_t T = D.T;
    SMP_GLOBAL int64_t* map = tile_map(D, k);
    const bool valid = tid < nval;
    const SMP_GLOBAL int64_t* sp = gp(D.seg) + k * TILE + (valid ? tid : 0);
    // every segment SIM, with a no-sample interval of at least T entries
    // (then max - min < T over its prefixes and the entry); a tile where one is
    // not leaves after this one look (resolve pass of 1.2e7 events at T = 128 KiB
    // without tile maps 18 us, with every tile of it marked and chained like a
    // mapped one 27, like this 20)
    const int64_t fl = sp[SP_FLG * ns];
    {
        const int64_t lo = sp[SP_LO * ns], hi = sp[SP_HI * ns];
        const bool no = valid && ((fl & 3) != MAP_SIM || hi < lo || hi - lo < T - 1);
        const int no_w = ballot(no) || !prefixes_kept(D) ? 1 : 0;
        if (l == 0) s_bad[wv] = no_w;
        __syncthreads();
        int no_map = 0;
        for (int w = 0; w < TWAVES; ++w) no_map |= s_bad[w];
        if (no_map) {
            if (tid == 0) {
                map[TM_HDR] = TM_NONE;
                g_add((uint64_t*)&ctl[6 + TMF_QUALIFY], 1ull);
            }
            return;
        }
        __syncthreads();  // (s_bad is written again)
    }
    int64_t af = 0, mx = 0, mn = 0;
    int32_t Rv, Sxv, Snv;
    {
        if (valid) {
            af = sp[SP_AF * ns];
            mx = sp[SP_MXF * ns];
            mn = sp[SP_MNF * ns];
        }
        const int64_t R = wave_incl_sum(af) - af;
        const bool in = R + mx < KEPT32 && R + mn > -KEPT32 && (fl & FLG_FIT);
        const int bad = ballot(valid && !in) || T >= KEPT32 ? 2 : 0;
        const int64_t im = wave_incl_max(R + mx), in_ = wave_incl_min(R + mn);
        if (l == 63) {
            s_bad[wv] = bad;
            s_ext[0][wv] = R + af;
            s_ext[1][wv] = im;
            s_ext[2][wv] = in_;
        }
        Rv = (int32_t)R;
        Sxv = (int32_t)(R + mx);
        Snv = (int32_t)(R + mn);
        __syncthreads();
        // the tile's extremes before this block, then before each segment
        int64_t base = 0, x = 0, n = 0;
        for (int w = 0; w < wv; ++w) {
            x = base + s_ext[1][w] > x ? base + s_ext[1][w] : x;
            n = base + s_ext[2][w] < n ? base + s_ext[2][w] : n;
            base += s_ext[0][w];
        }
        const int64_t pm = wave_shr1(im, INT64_MIN), pn = wave_shr1(in_, INT64_MAX);
        const int64_t bx = l && base + pm > x ? base + pm : x, bn = l && base + pn < n ? base + pn : n;
        const int c = __popcll(
            ballot(valid && bx - bn <= 2 * T - 2 && (base + R + mx > bx || base + R + mn < bn)));
        if (l == 0) s_new[wv] = c;
    }
    __syncthreads();
    int bad = 0, fresh_segs = 0;
    for (int w = 0; w < TWAVES; ++w) {
        bad |= s_bad[w];
        fresh_segs += s_new[w];
    }
    int fail = 0;
    // A tile whose entries take too long to sample would start more chains
    // than a map holds (~31 sources per segment with a new extreme on the
    // log-uniform mixes, and then too many runs): found out here, not after
    // a build of 0.2 to 0.4 ms.  Footprints that grow by single steps have one or
    // two sources in each such segment, but chains that do not meet, so that
    // they too come to too many runs: 70 tiles with a step in every fifth or in
    // every segment, T = 64 MiB, 421 to 490 us for the resolve pass, and 440 to
    // 635 where the sources were estimated first and the maps then tried.
    if (fresh_segs > TS_FRESH) {
        fail = TMF_SOURCES;
    } else if (bad) {
        if (wv) return;
        fail = tmap_wide(D, k, nval, u_.wide, map);
    } else {
        const int nb = block_segments(nval, wv);
        const int32_t rend = readlane32(Rv + (int32_t)af, 63);
        const TmapBlock mine = tmap_block(D, k, k * TILE + wv * 64, wv, nb, (int32_t)T, Rv, Sxv, Snv, rend, u_.blk[wv]);
        if (l == 0) s_blk[wv] = mine;
        __syncthreads();
        for (int w = 0; w < TWAVES; ++w) fail = fail ? fail : s_blk[w].fail;
        // Compose: every piece's exit through the next block's map, and what
        // is left unsampled cut by that block's runs.
        int nup = 0, ndn = 0;
        int64_t Ulo = -T + 1, Uhi = T - 1, tF = 0;
        for (int w = 0; w < TWAVES && !fail; ++w) {
            const TmapBlock m = s_blk[w];
            const TmapRuns& M = u_.blk[w].runs;
            for (int i = tid; i < nup + ndn; i += TILE) {
                const int at = i < nup ? i : TS_SRC - 1 - (i - nup);
                pieces.e[at] = runs_exit(M, m, pieces.e[at]);
            }
            if (Ulo <= Uhi) {
                // (an unsampled entry stays inside (-T, T) of every segment's start)
                const int32_t a = (int32_t)(Ulo - tF), z = (int32_t)(Uhi - tF);
                const int u0 = first_bound<true>(M.b, 1, m.nup, a), u1 = first_bound<true>(M.b, 1, m.nup, z);
                const int nu = u0 < m.nup ? (u1 < m.nup ? u1 : m.nup - 1) - u0 + 1 : 0;
                const int32_t* db = M.b + TS_SRC - 1;
                const int d0 = first_bound<false>(db, -1, m.ndn, z), d1 = first_bound<false>(db, -1, m.ndn, a);
                const int nd = d0 < m.ndn ? (d1 < m.ndn ? d1 : m.ndn - 1) - d0 + 1 : 0;
                if (nup + ndn + nu + nd > TS_SRC) {
                    fail = TMF_SOURCES;
                    break;
                }
                for (int i = tid; i < nu; i += TILE) {
                    const int32_t b = M.b[u0 + i];
                    pieces.b[nup + i] = (int32_t)((b < z ? b : z) + tF);
                    pieces.e[nup + i] = M.e[u0 + i];
                }
                for (int i = tid; i < nd; i += TILE) {
                    const int32_t b = db[-(d0 + i)];
                    pieces.b[TS_SRC - 1 - (ndn + i)] = (int32_t)((b > a ? b : a) + tF);
                    pieces.e[TS_SRC - 1 - (ndn + i)] = M.e[TS_SRC - 1 - (d0 + i)];
                }
                nup += nu;
                ndn += nd;
                if (m.lo > m.hi) {
                    Uhi = Ulo - 1;
                } else {
                    Ulo = m.lo + tF > Ulo ? m.lo + tF : Ulo;
                    Uhi = m.hi + tF < Uhi ? m.hi + tF : Uhi;
                }
            }
            tF += m.rend;
            __syncthreads();
        }
        if (wv) return;
        // the tile's runs, stored through to memory (another wave reads them in this launch)
        int ru = 0, rd = 0;
        int64_t lastU = 0, lastD = 0;
        for (int g = 0; g < nup && !fail && ru <= TM_SIDE; g += 64) {
            const bool v = g + l < nup;
            add_runs(v, v ? pieces.e[g + l] : 0, v ? pieces.b[g + l] : 0, ru, lastU, [&](int run, int which, int64_t x) {
                if (run < TM_SIDE) st_map(map + run_word(0, which, run), x);
            });
        }
        for (int g = 0; g < ndn && !fail && rd <= TM_SIDE; g += 64) {
            const bool v = g + l < ndn;
            const int at = TS_SRC - 1 - (v ? g + l : 0);
            add_runs(v, v ? pieces.e[at] : 0, v ? pieces.b[at] : 0, rd, lastD, [&](int run, int which, int64_t x) {
                if (run < TM_SIDE) st_map(map + run_word(1, which, run), x);
            });
        }
        if (ru > TM_SIDE || rd > TM_SIDE) fail = fail ? fail : TMF_RUNS;
        if (!fail && l == 0) {
            st_map(map + TM_HDR + 1, ru);
            st_map(map + TM_HDR + 2, rd);
            st_map(map + TM_HDR + 3, tF);
        }
    }
    if (wv) return;
    if (l == 0) {
        st_map(map + TM_HDR, fail ? TM_NONE : TM_MAPPED);
        g_add((uint64_t*)&ctl[fail ? 6 + fail : 5], 1ull);
    }
    if (!fail) chain_mapped_tiles(D, k, ctl);
}

// ------------------------------------------------------------ block maps
//
// The chain map of a block of 64 consecutive segments over all entry offsets
// (section 3.2, by the steps of the tile maps above, but for segments of any
// map kind that may sample several times): one wave follows the block's
// distinct chains segment by segment, the 8 waves of a tile at once, so that
// a tile costs the time of 64 segments instead of 512 and its entry is needed
// only for eight lookups.  Chains live in lanes (two per lane); a chain is
// named by the source that started it, and a chain that reaches a node where
// another has sampled ends there and points to that one.  Every chain's
// reference after every segment is written to the sample area, so that the
// exits of all segments follow from the block's entry by reading one column
// per stretch of the entry's path.
//
// Coordinates are footprints relative to the block start, as 32-bit values:
// T and all of them must stay below 2^30 in magnitude, the SIM segments must
// keep 32-bit prefixes, and the block's entries must all have sampled within
// its first BM_OPEN segments (a threshold far above what a segment moves
// would start more chains than fit); a tile that does not qualify, or whose
// blocks start more, is walked instead.
// Bound: the serial chain of one wave through 64 segments (a sample of a lone
// chain costs ~150 ns of dependent ballots and LDS reads; the first samples of
// many chains are searched side by side).  Measured, resolve pass: 1,024
// traces of 1e3-1e6 events at T = 256 KiB / 1 MiB / 10 MiB 1.12 -> 0.28 ms; a
// trace of 777,777 events at T = 3 MiB (three tiles) 1.53 -> 0.15 ms; one of
// 1.2e7 events at T = 10 MiB 9.5 -> 0.2 ms.  (Prefixes two segments ahead
// instead of one: 25 spilled registers and 0.16 / 0.29 ms.)
constexpr int BM_SRC = 512;   // sources per block
constexpr int BM_OPEN = 14;   // ~31 sources per segment on the log-uniform mixes while entries are left
constexpr int BM_MIN_SIM = 8; // SIM segments from which a waiting tile builds its maps
constexpr int BM_PAR = 4;     // chains that stop in a segment from which they are searched side by side

// Whether a tile takes them.  One that has to wait for its entry builds them
// meanwhile (from BM_MIN_SIM SIM segments on: 700 segments, the last 188 of them
// a tile of their own, T = 10 MiB, 140 us, and 242 with the second tile walked).
// One whose entry is there compares the walk's time with the slowest block's, in
// 1/20 us.  The walk stops in a SIM segment for the share of entries outside
// its no-sample interval (expected stops, in 1/256), 1.25 us each, or 0.85 in a
// sparse tile (see the resolve pass).  A block takes about 10 us, 1.55 per SIM
// segment up to its first segment with a total map (its chains are many until
// there) and 1.5 per stop after it.  Walked and mapped, us: traces of 64 / 128 /
// 256 / 512 segments at T = 10 MiB 41 / 75 / 143 / 292 and 109 / 110 / 128 /
// 138, at T = 3 MiB 73 / 142 / 280 / 550 and 104 / 105 / 108 / 129, at T = 1 MiB
// 11 / 14 / 26 / 52 and 12 / 14 / 22 / 32; half copies at T = 1 MiB 36 / 73 /
// 140 / 257 and 49 / 54 / 58 / 64, at T = 10 MiB (sparse) 19 / 31 / 57 / 106 and
// 82 / 89 / 93 / 101.  At T = 30 MiB the walk takes 15 / 24 / 43 / 78, and a map
// tried in vain 20 more.
__device__ __forceinline__ int block_cost(int many, int after) { return 200 + 31 * many + 30 * after / 256; }
__device__ __forceinline__ bool block_maps_pay(bool sparse, int stops, int slowest) {
    return (sparse ? 17 : 25) * stops / 256 > slowest;
}

struct alignas(16) BlockLds {
    int32_t f[SEG];          // the current SIM segment's prefixes
    int32_t sb[BM_SRC];      // source bounds (entry offsets at the block start): 2 * bound, + 1 for a source of the
                             // entries below the unsampled interval (its largest; + 0: above, its smallest)
    int32_t ex[128];         // exit offset of each column's chain
    uint16_t claim[SEG];     // chain that sampled at each node: (segment + 1) << 9 | chain
    uint16_t init[BM_SRC];   // the chain the source joins
    uint16_t par[BM_SRC];    // chain a chain has merged into (itself: none)
    uint8_t cseg[BM_SRC];    // the segment where the source joins it
    uint8_t mseg[BM_SRC];    // the segment where the chain merged
    uint8_t slot[BM_SRC];    // a chain's column
};
constexpr uint32_t BM_ID = BM_SRC - 1;
static_assert(BM_SRC == 1 << 9, "a claim holds the segment and the chain");
// value pushed to lane dst (lanes that none is pushed to receive 0)
__device__ __forceinline__ int32_t push32(int32_t v, int dst) { return __builtin_amdgcn_ds_permute(dst << 2, v); }

// The references after each segment: 128 columns of 32-bit values per
// segment, in the sample area behind the kept prefixes.
__device__ __forceinline__ bool block_rows_fit(const Desc& D) {
    return (D.n + 1) * sizeof(Sample) >= (uint64_t)D.nseg * (SEG * sizeof(int64_t) + 512);
}
__device__ __forceinline__ SMP_GLOBAL int32_t* block_row(const Desc& D, int64_t j) {
    return (SMP_GLOBAL int32_t*)((SMP_GLOBAL uint8_t*)gp((uint8_t*)D.samples) + (uint64_t)D.nseg * (SEG * 8) +
                                 (uint64_t)j * 512);
}

// A block's map as the wave that built it holds it (uniform values, but for
// ref: lane i's is the one reference after segment i, from segment one_from on).
struct BlockMap {
    int ok;
    int nsrc;
    int32_t umax, umin;  // unsampled entries: [umax - T + 1, umin + T - 1]
    int32_t rend;        // the block's footprint change
    int one_from;        // from this segment's end on every entry has one reference (64: never)
    int32_t ref;
};

// Follow a chain from reference xr (relative to the segment) from node st on
// through a segment whose prefixes lie in B.f and whose eight-node groups
// (lane g: nodes 8g .. 8g + 7) reach from gn to gx: each sample takes two
// ballots over the groups and one over the nodes of the first group that
// crosses.  CLAIM: every sampled node is claimed (tag: the segment's bits of
// a claim, id: the chain); returns the chain that had claimed one, or -1 at
// the segment end.  one: stop after a sample (a segment that moves less than
// T holds one of a chain).
template <bool CLAIM>
__device__ __forceinline__ int follow_groups(BlockLds& B, int32_t gx, int32_t gn, int32_t T, int32_t& xr, int st,
                                             uint32_t tag, uint32_t id, bool one) {
    const int l = lane_id();
    if (st >= SEG) return -1;
    int gfrom = st >> 3;
    uint64_t emask = (0xFFull << (st & 7)) & 0xFFull, gmask = ~0ull << gfrom;
    for (;;) {
        uint64_t gm = (ballot(gx >= xr + T) | ballot(gn <= xr - T)) & gmask, m;
        int g;
        int32_t v;
        uint32_t c = 0;
        for (;;) {
            if (!gm) return -1;
            g = ctz64(gm);
            v = B.f[8 * g + (l & 7)];
            if (CLAIM) c = B.claim[8 * g + (l & 7)];
            asm volatile("" : "+v"(v), "+v"(c));  // (both reads in flight together)
            m = ballot(beyond32(v, xr, T)) & (g == gfrom ? emask : 0xFFull);
            if (m) break;
            gm &= gm - 1;  // (the first group's crossings lie before st)
        }
        const int j = ctz64(m);
        if (CLAIM) {
            const uint32_t cj = (uint32_t)readlane32((int)c, j);
            if ((cj & ~BM_ID) == tag) return (int)(cj & BM_ID);
            B.claim[8 * g + j] = (uint16_t)(tag | id);
        }
        xr = readlane32(v, j);
        if (one) return -1;
        gfrom = g;
        gmask = ~0ull << g;
        emask = (0xFEull << j) & 0xFFull;
    }
}

// Build the map of the block at segment j0 of nb segments; lane i holds
// segment i's kind, offset Rv, extremes Sxv, Snv and constant exit kxv (block
// coordinates).
__device__ __forceinline__ BlockMap build_block(const Desc& D, int64_t j0, int nb, int32_t T, int kindv, int32_t Rv,
                                                int32_t Sxv, int32_t Snv, int32_t kxv, int32_t rend, BlockLds& B) {
    // (a block past the trace's end has no prefixes to load: every entry passes)
    if (nb == 0) return BlockMap{1, 0, 0, 0, 0, 64, 0};
    const int l = lane_id();
    int32_t XA = 0, XB = 0;     // lane l: chains in columns l and 64 + l
    int idA = 0, idB = 0;
    uint64_t alA = 0, alB = 0;  // columns in use
    int nsrc = 0;
    int32_t Umax = 0, Umin = 0;
    bool open = true, ok = true;
    const uint64_t simm = ballot(l < nb && kindv == MAP_SIM);
    for (int i = l; i < SEG; i += 64) B.claim[i] = 0;
    // the next SIM segment's prefixes load while one is processed
    int32_t pf[NW];
    auto prefetch = [&](int s) {
        const uint64_t m = s < 64 ? simm & (~0ull << s) : 0;
        load_kept32(D, next_kept(j0, m), pf);
    };
    // segment s's prefixes (just prefetched) into LDS, and their group extremes
    int32_t gx = 0, gn = 0;
    auto group_extremes = [&]() {
        const v4i32 a = *(const v4i32*)&B.f[8 * l], b = *(const v4i32*)&B.f[8 * l + 4];
        gx = a[0];
        gn = a[0];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            gx = a[i] > gx ? a[i] : gx;
            gx = b[i] > gx ? b[i] : gx;
            gn = a[i] < gn ? a[i] : gn;
            gn = b[i] < gn ? b[i] : gn;
        }
    };
    auto take = [&](int s) {
#pragma unroll
        for (int w = 0; w < NW; ++w) B.f[w * 64 + l] = pf[w];
        prefetch(s + 1);
        group_extremes();
    };
    // Follow chain id from reference xr (relative to segment s) from node st
    // on; the chain it meets, or -1 at the segment end.
    auto follow = [&](int32_t& xr, int st, int id, int s, bool single) -> int {
        return follow_groups<true>(B, gx, gn, T, xr, st, (uint32_t)(s + 1) << 9, (uint32_t)id, single);
    };
    // Columns for the new chains of the lanes in nm (reference X, name id).
    auto new_columns = [&](uint64_t nm, int32_t X, int id) {
        const int n = __popcll(nm), na = __popcll(~alA);
        if (n > na + __popcll(~alB)) {
            ok = false;
            return;
        }
        const int rank = __popcll(nm & lanemask_lt());
        // the chains in rank order, one per lane (lanes outside nm push past them)
        const bool mine = (nm >> l) & 1;
        const int dst = mine ? rank : n + (l - rank);
        const int32_t px = push32(X, dst), pid = push32(id, dst);
        const int ra = __popcll(~alA & lanemask_lt()), rb = na + __popcll(~alB & lanemask_lt());
        const bool ta = !((alA >> l) & 1) && ra < n, tb = !((alB >> l) & 1) && rb < n;
        const int32_t xa = shfl32(px, ra & 63), ia = shfl32(pid, ra & 63);
        XA = ta ? xa : XA;
        idA = ta ? ia : idA;
        if (ta) B.slot[ia] = (uint8_t)l;
        alA |= ballot(ta);
        if (n > na) {
            const int32_t xb = shfl32(px, rb & 63), ib = shfl32(pid, rb & 63);
            XB = tb ? xb : XB;
            idB = tb ? ib : idB;
            if (tb) B.slot[ib] = (uint8_t)(64 + l);
            alB |= ballot(tb);
        }
    };
    // The stopping chains st of one group of columns through the segment in
    // B.f: their first samples side by side (a search over the running
    // extremes of the groups, then over the eight nodes of one), the ones at
    // one node merged, the rest of the segment one chain after another.
    auto stop_group = [&](uint64_t& al, uint64_t st, int32_t& X, int id, int32_t R, int s, bool single, int32_t cgx,
                          int32_t cgn) {
        const bool mine = (st >> l) & 1;
        const int32_t xr = mine ? X - R : 0;
        int32_t v;
        const int node = first_samples(B.f, cgx, cgn, T, xr, v);
        const uint32_t tag = (uint32_t)(s + 1) << 9, key = tag | (uint32_t)id;
        uint32_t got = mine ? B.claim[node] : 0;
        const bool taken = (got >> 9) == (uint32_t)(s + 1);
        if (mine && !taken) B.claim[node] = (uint16_t)key;
        asm volatile("" ::: "memory");  // (several lanes may write one claim: what it holds is read back)
        if (mine && !taken) got = B.claim[node];
        const bool win = mine && got == key;
        if (mine && !win) {
            B.par[id] = (uint16_t)(got & BM_ID);
            B.mseg[id] = (uint8_t)s;
        }
        const uint64_t wm = ballot(win);
        al = (al & ~st) | wm;
        X = win ? R + v : X;
        if (single) return;
        for (uint64_t m = wm; m; m &= m - 1) {
            const int c = ctz64(m), cid = readlane32(id, c);
            int32_t x = readlane32(v, c);
            const int to = follow(x, readlane32(node, c) + 1, cid, s, false);
            if (to >= 0) {
                B.par[cid] = (uint16_t)to;
                B.mseg[cid] = (uint8_t)s;
                al &= ~(1ull << c);
            }
            X = l == c ? R + x : X;
        }
    };
    // The same, one chain after another.
    auto stop_each = [&](uint64_t& al, uint64_t st, int32_t& X, int id, int32_t R, int s, bool single) {
        for (uint64_t m = st; m; m &= m - 1) {
            const int c = ctz64(m), cid = readlane32(id, c);
            int32_t x = readlane32(X, c) - R;
            const int to = follow(x, 0, cid, s, single);
            if (to >= 0) {
                B.par[cid] = (uint16_t)to;
                B.mseg[cid] = (uint8_t)s;
                al &= ~(1ull << c);
            }
            X = l == c ? R + x : X;
        }
    };
    prefetch(0);
    int s = 0;
    // every chain, until one is left and no entry is unsampled
    for (; s < nb && ok; ++s) {
        if (!open && __popcll(alA) + __popcll(alB) == 1) break;
        const int kind = readlane32(kindv, s);
        const int32_t R = readlane32(Rv, s), Sx = readlane32(Sxv, s), Sn = readlane32(Snv, s);
        uint64_t stA = alA & ballot(XA <= Sx - T || XA >= Sn + T), stB = alB & ballot(XB <= Sx - T || XB >= Sn + T);
        bool fresh = open && (Sx > Umax || Sn < Umin);
        if (kind == MAP_TOTAL) {
            stA = alA;
            stB = alB;
            fresh = open;
        }
        if (kind != MAP_SIM) {
            if (stA | stB | (fresh ? 1ull : 0ull)) {
                // every chain and entry that samples leaves at one reference:
                // the first source's new chain, or the first chain's
                const int32_t kx = readlane32(kxv, s);
                int id = nsrc;
                if (stA) id = readlane32(idA, ctz64(stA));
                else if (stB) id = readlane32(idB, ctz64(stB));
                if (fresh) {
                    const int32_t mx = Sx > Umax ? Sx : Umax, uhi = Umin + T - 1;
                    const bool all = kind == MAP_TOTAL;
                    const bool up = all || Sx > Umax;
                    const bool dn = !all && Sn < Umin && mx - Umin <= 2 * T - 2;
                    const int add = (up ? 1 : 0) + (dn ? 1 : 0);
                    if (nsrc + add > BM_SRC) {
                        ok = false;
                        break;
                    }
                    if (l < add) {
                        const bool u = up && l == 0;
                        const int src = nsrc + l;
                        B.sb[src] = u ? 2 * (all || uhi < Sx - T ? uhi : Sx - T) + 1
                                      : 2 * (mx - T + 1 > Sn + T ? mx - T + 1 : Sn + T);
                        B.init[src] = (uint16_t)id;
                        B.cseg[src] = (uint8_t)s;
                        B.par[src] = (uint16_t)id;
                        B.mseg[src] = (uint8_t)s;
                    }
                    if (!(stA | stB)) new_columns(1ull, kx, id);
                    nsrc += add;
                }
                // the others end in it
                if (((stA >> l) & 1) && idA != id) {
                    B.par[idA] = (uint16_t)id;
                    B.mseg[idA] = (uint8_t)s;
                }
                if (((stB >> l) & 1) && idB != id) {
                    B.par[idB] = (uint16_t)id;
                    B.mseg[idB] = (uint8_t)s;
                }
                if (stA) {
                    const uint64_t first = stA & (~stA + 1);
                    alA = (alA & ~stA) | first;
                    alB &= ~stB;
                    XA = (first >> l) & 1 ? kx : XA;
                } else if (stB) {
                    const uint64_t first = stB & (~stB + 1);
                    alB = (alB & ~stB) | first;
                    XB = (first >> l) & 1 ? kx : XB;
                }
            }
        } else if (stA | stB | (fresh ? 1ull : 0ull)) {
            take(s);
            const bool single = Sx - Sn < T;
            if (__popcll(stA) + __popcll(stB) >= BM_PAR) {
                const int32_t cgx = wave_incl_ext32<true>(gx), cgn = wave_incl_ext32<false>(gn);
                if (stA) stop_group(alA, stA, XA, idA, R, s, single, cgx, cgn);
                if (stB) stop_group(alB, stB, XB, idB, R, s, single, cgx, cgn);
            } else {
                stop_each(alA, stA, XA, idA, R, s, single);
                stop_each(alB, stB, XB, idB, R, s, single);
            }
            if (fresh) {
                // nodes beyond the extremes so far: first samples of unsampled entries
                int32_t cm = Umax, cn = Umin;
                for (int w = 0; w < NW && ok && cm - cn <= 2 * T - 2; ++w) {
                    const int32_t fv = B.f[w * 64 + l], gv = R + fv;
                    if (!ballot(gv > cm || gv < cn)) continue;
                    int32_t im = wave_incl_ext32<true>(gv), in = wave_incl_ext32<false>(gv);
                    im = im > cm ? im : cm;
                    in = in < cn ? in : cn;
                    const int32_t pm = wave_shr1_32(im, cm), pn = wave_shr1_32(in, cn);  // before the node
                    const bool op = pm - pn <= 2 * T - 2;
                    const bool up = op && gv > pm, dn = op && gv < pn;
                    const uint64_t spm = ballot(up || dn);
                    cm = readlane32(im, 63);
                    cn = readlane32(in, 63);
                    if (nsrc + __popcll(spm) > BM_SRC) {
                        ok = false;
                        break;
                    }
                    // the sources, in node order; each starts a chain at its
                    // node or joins the one that sampled there
                    const bool mine = (spm >> l) & 1;
                    const int src = nsrc + __popcll(spm & lanemask_lt());
                    if (mine) {
                        B.sb[src] = up ? 2 * (pn + T - 1 < gv - T ? pn + T - 1 : gv - T) + 1
                                       : 2 * (pm - T + 1 > gv + T ? pm - T + 1 : gv + T);
                        B.cseg[src] = (uint8_t)s;
                        B.par[src] = (uint16_t)src;
                    }
                    const uint32_t cl = mine ? B.claim[w * 64 + l] : 0;
                    const bool hit = (cl >> 9) == (uint32_t)(s + 1);
                    if (mine) {
                        B.init[src] = (uint16_t)(hit ? (int)(cl & BM_ID) : src);
                        if (!hit) B.claim[w * 64 + l] = (uint16_t)((s + 1) << 9 | src);
                    }
                    const uint64_t nm = spm & ~ballot(hit);
                    new_columns(nm, gv, src);
                    nsrc += __popcll(spm);
                    if (single) continue;  // (no chain samples again)
                    for (uint64_t m = nm; m && ok; m &= m - 1) {
                        const int c = ctz64(m), id = readlane32(src, c);
                        int32_t xr = readlane32(fv, c);
                        const int32_t x0 = xr;
                        const int to = follow(xr, w * 64 + c + 1, id, s, false);
                        if (to < 0 && xr == x0) continue;
                        const int col = readlane32((int)B.slot[id], 0);
                        if (to >= 0) {
                            B.par[id] = (uint16_t)to;
                            B.mseg[id] = (uint8_t)s;
                            alA &= col < 64 ? ~(1ull << col) : ~0ull;
                            alB &= col < 64 ? ~0ull : ~(1ull << (col - 64));
                        } else {
                            XA = l == col ? R + xr : XA;
                            XB = 64 + l == col ? R + xr : XB;
                        }
                    }
                }
            }
        } else {
            prefetch(s + 1);
        }
        Umax = Sx > Umax ? Sx : Umax;
        Umin = Sn < Umin ? Sn : Umin;
        open = open && kind != MAP_TOTAL && Umax - Umin <= 2 * T - 2;
        SMP_GLOBAL int32_t* row = block_row(D, j0 + s);
        row[l] = XA;
        if (alB) row[64 + l] = XB;
    }
    BlockMap r{ok ? 1 : 0, nsrc, Umax, Umin, rend, 64, 0};
    if (!ok) return r;
    if (!open) {  // (a closed interval stays closed whatever the extremes do later)
        r.umax = T;
        r.umin = -T;
    }
    if (!open && __popcll(alA) + __popcll(alB) == 1) {
        // One reference is left: followed alone to the block end, all
        // segments up to its next stop at once, and a run of segments that
        // each take their predecessor's one exit to their own at once too.
        r.one_from = s > 0 ? s - 1 : 0;
        int32_t X = alA ? readlane32(XA, ctz64(alA)) : readlane32(XB, ctz64(alB));
        const int32_t kp = wave_shr1_32(kxv, 0);
        const uint64_t runm =
            ballot(l > 0 && l < nb && kindv != MAP_SIM && (kindv == MAP_TOTAL || kp <= Sxv - T || kp >= Snv + T));
        r.ref = X;
        auto next_sim = [&](int from) {
            const uint64_t m = from < 64 ? simm & (~0ull << from) : 0;
            return m ? ctz64(m) : 64;
        };
        int ia = next_sim(s);  // the segment whose prefixes are in pf
        while (s < nb) {
            const uint64_t stop =
                ballot(l >= s && l < nb && (kindv == MAP_TOTAL || X <= Sxv - T || X >= Snv + T));
            if (l >= s) r.ref = X;
            if (!stop) break;
            const int i = ctz64(stop);
            if ((simm >> i) & 1) {
                if (i != ia) prefetch(i);
                take(i);
                ia = next_sim(i + 1);
                const int32_t R = readlane32(Rv, i);
                const bool single = readlane32(Sxv, i) - readlane32(Snv, i) < T;
                int32_t xr = X - R;
                (void)follow_groups<false>(B, gx, gn, T, xr, 0, 0, 0, single);
                X = R + xr;
                if (l >= i) r.ref = X;
                s = i + 1;
            } else {
                // i and the run after it
                const uint64_t nr = ~runm & ~(i < 63 ? ((2ull << i) - 1) : ~0ull);
                const int e = nr ? ctz64(nr) : 64;  // first segment past the run
                if (l >= i && l < e) r.ref = kxv;
                X = readlane32(kxv, e - 1);
                s = e;
            }
        }
        B.ex[0] = X - rend;
        return r;
    }
    B.ex[l] = XA - rend;
    B.ex[64 + l] = XB - rend;
    return r;
}

// The source that holds entry e of a block (-1: e has not sampled at the block end).
__device__ __forceinline__ int block_source(const BlockLds& B, int nsrc, int32_t umax, int32_t umin, int32_t T,
                                            int32_t e) {
    const int l = lane_id();
    if (e >= umax - T + 1 && e <= umin + T - 1) return -1;
    int dn = -1;
    for (int g = 0; g < nsrc; g += 64) {
        const int s = g + l;
        const bool v = s < nsrc;
        const int32_t b2 = v ? B.sb[s] : 0, b = b2 >> 1;
        const bool up = (b2 & 1) != 0;
        const uint64_t u = ballot(v && up && b >= e), d = ballot(v && !up && b <= e);
        if (u) return g + ctz64(u);
        if (d && dn < 0) dn = g + ctz64(d);
    }
    return dn;  // (every entry outside the interval has one)
}

// A block's exit offset of the entries of source src.
__device__ __forceinline__ int32_t block_exit(const BlockLds& B, const BlockMap& m, int src) {
    if (m.one_from < 64) return __builtin_amdgcn_readfirstlane(B.ex[0]);
    int id = readlane32((int)B.init[src], 0);
    for (int d = 0; d < BM_SRC; ++d) {
        const int to = readlane32((int)B.par[id], 0);
        if (to == id) break;
        id = to;
    }
    return __builtin_amdgcn_readfirstlane(B.ex[readlane32((int)B.slot[id], 0)]);
}

// The reference after each segment of the block (lane i: segment i) of the
// chain from entry e, whose source is src (one_from, ref: the block's map).
__device__ __forceinline__ int32_t block_refs(const Desc& D, int64_t j0, int nb, const BlockLds& B, int one_from,
                                              int32_t ref, int32_t e, int src) {
    const int l = lane_id();
    int col = -1;
    if (src >= 0 && one_from > 0) {
        int from = readlane32((int)B.cseg[src], 0), id = readlane32((int)B.init[src], 0);
        for (int d = 0; d < BM_SRC; ++d) {
            const int to = readlane32((int)B.par[id], 0);
            const int until = to == id ? 64 : readlane32((int)B.mseg[id], 0);
            const int sl = readlane32((int)B.slot[id], 0);
            if (l >= from && l < until) col = sl;
            if (to == id) break;
            from = until > from ? until : from;
            id = to;
        }
    }
    if (l >= one_from) return ref;
    return col >= 0 && l < nb ? block_row(D, j0 + l)[col] : e;
}

// One workgroup per tile of TILE segments (tiles taken in ticket order, so a
// tile's predecessors are always running or done): exclusive prefix sums and
// the chain's entry and exit offset of every segment.
//
// Exits of segments with a total map are known at once.  The other segments
// are resolved in order by one wave (the walker), from the segment after the
// tile's first total map to the tile end first (their exits do not depend on
// the tile's entry, so the tile's exit is published before its entry is
// awaited), then from the tile start; the walker takes 64 segments per step
// and stops only at segments whose entry lies outside their no-sample
// interval.  A SIM segment where it stops is followed through its records;
// the other waves scan the SIM segments' footprint prefixes into an LDS ring
// ahead of the walker (skipping those it has already passed), so each one
// costs the walker only a pass over LDS.  Tiles of several SIM segments whose
// blocks qualify take block maps (above) instead of the walk.
__global__ __launch_bounds__(TILE) __attribute__((amdgpu_waves_per_eu(4))) void k_resolve(const Desc* __restrict__ desc, int ntraces, uint64_t ntile_total,
                                                  unsigned long long* ctl, uint64_t* ts_) {
    stamp(ts_);
    __shared__ unsigned long long s_tk;
    __shared__ int64_t w_sum[3][TWAVES];
    __shared__ int64_t s_pre[3];
    __shared__ int64_t w_peak[TWAVES], w_peakS[TWAVES];
    __shared__ int w_left[TWAVES];
    __shared__ int64_t m_ex[TILE];
    __shared__ uint64_t w_tot[TWAVES], w_sim[TWAVES];  // valid lanes with TOTAL / SIM maps
    __shared__ uint64_t w_fit[TWAVES];                 // lanes whose kept prefixes are 32-bit values
    __shared__ union {
        struct {
            int64_t ring[RING][SEG];
            int64_t lo[TILE], hi[TILE], af[TILE], kf[TILE];
            int64_t R[TILE];  // sparse tiles: the footprint change before each segment
        } w;
        BlockLds blk[TWAVES];  // (a tile uses one or the other)
    } u_;
    int64_t (&ring)[RING][SEG] = u_.w.ring;
    int64_t (&m_lo)[TILE] = u_.w.lo, (&m_hi)[TILE] = u_.w.hi, (&m_af)[TILE] = u_.w.af, (&m_kf)[TILE] = u_.w.kf;
    int64_t (&m_R)[TILE] = u_.w.R;
    __shared__ BlockMap s_bm[TWAVES];
    __shared__ int s_bok[TWAVES], s_bsrc[TWAVES];
    __shared__ int32_t s_bent[TWAVES + 1];
    __shared__ int r_ready[RING];  // walk-order SIM index held by each slot
    __shared__ int s_prod, s_cons, s_abort;
    __shared__ int s_known;  // 1: the tile's entry is there already
    __shared__ int w_wide[TWAVES];
    __shared__ int w_stops[TWAVES], w_cost[TWAVES];  // expected stops of the walk, cost of the block's map
    __shared__ int64_t s_entry;
    const int tid = threadIdx.x, wv = tid >> 6, l = lane_id();
    if (tid == 0) {
        s_tk = g_add_rtn((uint64_t*)&ctl[2], 1ull);
        s_known = 1;
        s_prod = 0;
        s_cons = 0;
        s_abort = 0;
    }
    if (tid < RING) r_ready[tid] = -1;
    __syncthreads();
    const uint64_t tk = s_tk;
    if (tk >= ntile_total) return;
    const Desc& D = desc[find_trace_tile(desc, ntraces, tk)];
    const int64_t k = (int64_t)(tk - D.tile_begin);
    const int64_t ns = (int64_t)D.nseg;
    const int64_t j = k * TILE + tid;
    const bool valid = j < ns;
    const int nval = (int)((ns - k * TILE) < TILE ? (ns - k * TILE) : TILE);  // valid lanes
    const StatusView ts{D.tstat, (int64_t)D.ntile};
    if (D.tmap && tid == 0) D.blk[k] = 0;  // (the mark of a tile map)
    // (published by a tile map or by a tile that is done already: decides how this
    // tile is followed, not what comes out)
    if (k > 0 && tid == 0) s_known = wstate(ld_status(ts.at(W_XF, k - 1))) != 0;
    const SMP_GLOBAL int64_t* sp = gp(D.seg) + (valid ? j : 0);
    int64_t af = 0, ap = 0, ac = 0, kf = 0, lo = 0, hi = 0, mxf = 0, mnf = 0;
    int kind = MAP_CONST, flg = 0;
    if (valid) {
        af = sp[SP_AF * ns];
        ap = sp[SP_AP * ns];
        ac = sp[SP_AC * ns];
        lo = sp[SP_LO * ns];
        hi = sp[SP_HI * ns];
        kf = sp[SP_KF * ns];
        mxf = sp[SP_MXF * ns];
        mnf = sp[SP_MNF * ns];
        flg = (int)sp[SP_FLG * ns];
        kind = flg & 3;
    }
    m_lo[tid] = lo;
    m_hi[tid] = hi;
    m_af[tid] = af;
    m_kf[tid] = kf;
    m_ex[tid] = kf;  // final for total maps; the walker overwrites the others
    const uint64_t tot = ballot(valid && kind == MAP_TOTAL), sim = ballot(valid && kind == MAP_SIM);
    const uint64_t fitm = ballot((flg & FLG_FIT) != 0);
    const int64_t T = D.T;
    const bool kept = prefixes_kept(D);
    // sums inside the wave
    int64_t iF = af, iP = ap, iC = ac;
    wave_incl_sum3(iF, iP, iC);
    if (l == 63) {
        w_sum[0][wv] = iF;
        w_sum[1][wv] = iP;
        w_sum[2][wv] = iC;
    }
    // SIM maps whose no-sample interval holds at least half of the entries
    const int nwide_w = __popcll(ballot(valid && kind == MAP_SIM && hi - lo >= D.T));
    // (see block_maps_pay)
    const int first_tot = tot ? ctz64(tot) : 64;
    const float inside = hi < lo ? 0.0f : (float)(hi - lo + 1) / (float)(2 * T - 1);
    const int stop = valid && kind == MAP_SIM ? (int)(256.0f * (1.0f - (inside < 1.0f ? inside : 1.0f))) : 0;
    const uint64_t stops = (uint64_t)wave_sum((int64_t)((uint64_t)stop << 32 | (uint64_t)(l > first_tot ? stop : 0)));
    if (l == 0) {
        w_stops[wv] = (int)(stops >> 32);
        w_cost[wv] = block_cost(__popcll(sim & range_mask(0, 0, first_tot)), (int)(uint32_t)stops);
        w_tot[wv] = tot;
        w_sim[wv] = sim;
        w_fit[wv] = fitm;
        w_wide[wv] = nwide_w;
    }
    // whether this wave's 64 segments may get a block map (see there)
    const int nb = block_segments(nval, wv);
    const int64_t bR = iF - af;
    int32_t bSx = 0, bSn = 0;
    {
        const bool in = bR + mxf < KEPT32 && bR + mnf > -KEPT32 && bR + af < KEPT32 && bR + af > -KEPT32 &&
                        (kind != MAP_SIM || (flg & FLG_FIT));
        bool q = T < KEPT32 && kept && block_rows_fit(D) && !ballot(valid && !in);
        if (q) {
            bSx = (int32_t)(bR + mxf);
            bSn = (int32_t)(bR + mnf);
            const int32_t x = wave_ext32<true>(l < BM_OPEN && valid ? bSx : 0);
            const int32_t n = wave_ext32<false>(l < BM_OPEN && valid ? bSn : 0);
            q = nb <= BM_OPEN || (int64_t)x - n > 2 * T - 2 || (tot & ((1ull << BM_OPEN) - 1)) != 0;
        }
        if (l == 0) s_bok[wv] = q ? 1 : 0;
    }
    __syncthreads();
    int64_t oF = 0, oP = 0, oC = 0, tF = 0, tP = 0, tC = 0;
    int ft = nval;  // first lane with a total map
    for (int w = TWAVES - 1; w >= 0; --w)
        if (w_tot[w]) ft = w * 64 + ctz64(w_tot[w]);
    for (int w = 0; w < TWAVES; ++w) {
        if (w == wv) {
            oF = tF;
            oP = tP;
            oC = tC;
        }
        tF += w_sum[0][w];
        tP += w_sum[1][w];
        tC += w_sum[2][w];
    }
    tF = readlane64(tF, 0);  // (wave-uniform: scalar registers)
    tP = readlane64(tP, 0);
    tC = readlane64(tC, 0);
    // prefixes relative to the tile start (the tile's own prefix is added at the end)
    const int64_t rF = oF + iF - af, rP = oP + iP - ap, rC = oC + iC - ac;
    // SIM segments in walk order: (ft, nval) first, then [0, ft)
    int nA = 0, nsim = 0, nwide = 0;
    for (int w = 0; w < TWAVES; ++w) {
        nA += __popcll(w_sim[w] & range_mask(w, ft + 1, nval));
        nsim += __popcll(w_sim[w]);
        nwide += w_wide[w];
    }
    // publish the tile's sums (inclusive right away for the first tile)
    if (tid < 3) st_status(ts.at(W_AF + tid, k), pack(tid == 0 ? tF : (tid == 1 ? tP : tC), 1));
    if (k == 0 && tid < 3) st_status(ts.at(W_IF + tid, k), pack(tid == 0 ? tF : (tid == 1 ? tP : tC), 1));
    // Sparse tile: most SIM maps leave at least half of the entries without a
    // sample, so the walker stops at few of them (T far above what a segment
    // moves).  Producers pre-scanning every SIM segment would fall behind the
    // walker, and their loads would queue in the CU's memory pipeline ahead
    // of the walker's own (each stop of the walker waits for one): here the
    // other waves stay idle and the walker reads the kept prefixes itself.
    const bool sparse = kept && nsim > 0 && 4 * nwide >= 3 * nsim;
    // The tile's prefix sums (one wave).
    auto tile_sums = [&]() {
        int64_t pF = 0, pP = 0, pC = 0;
        bool ok = true;
        if (k > 0) {
            ok = scan_sums(ts, k, pF, pP, pC, ctl);
            if (l < 3) st_status(ts.at(W_IF + l, k), pack(l == 0 ? pF + tF : (l == 1 ? pP + tP : pC + tC), 1));
        }
        if (l == 0) {
            s_pre[0] = pF;
            s_pre[1] = pP;
            s_pre[2] = pC;
            if (!ok) g_or32(&D.scal->err, 8u);
        }
    };
    // Block maps: the tile's eight blocks are followed for all entries at
    // once, one wave each; the tile's entry then costs eight lookups and the
    // segments' exits are read from the rows its chain left.
    int nstops = 0, slowest = 0;
    for (int w = 0; w < TWAVES; ++w) {
        nstops += w_stops[w];
        slowest = w_cost[w] > slowest ? w_cost[w] : slowest;
    }
    bool blocks = s_known ? block_maps_pay(sparse, nstops, slowest) : nsim >= BM_MIN_SIM;
    for (int w = 0; w < TWAVES; ++w) blocks = blocks && s_bok[w] != 0;
    const bool tried = blocks;
    int32_t bref = 0;  // (BlockMap::ref)
    if (blocks) {
        const BlockMap bm = build_block(D, k * TILE + wv * 64, nb, (int32_t)T, kind, (int32_t)bR, bSx, bSn,
                                        (int32_t)(bR + af + kf), readlane32((int32_t)(bR + af), 63), u_.blk[wv]);
        bref = bm.ref;
        if (l == 0) s_bm[wv] = bm;
        __syncthreads();
        for (int w = 0; w < TWAVES; ++w) blocks = blocks && s_bm[w].ok != 0;
    }
    if (blocks) {
        if (wv == 0) {
            const int32_t t32 = (int32_t)T;
            auto follow_block = [&](int b, int32_t e) {
                const BlockMap& m = s_bm[b];
                const int src = __builtin_amdgcn_readfirstlane(
                    block_source(u_.blk[b], m.nsrc, m.umax, m.umin, t32, e));
                s_bsrc[b] = src;
                return src < 0 ? e - m.rend : block_exit(u_.blk[b], m, src);
            };
            // from the last block that every entry leaves at one exit, the
            // tile's exit does not depend on its entry: published first
            int c = -1;
            for (int b = 0; b < TWAVES; ++b)
                if (s_bm[b].one_from < 64) c = b;
            bool out = false;
            if (c >= 0) {
                // a tile map may have published the exit already: it must agree
                const uint64_t pw = D.tmap ? ld_status(ts.at(W_XF, k)) : 0;
                int32_t x = __builtin_amdgcn_readfirstlane(u_.blk[c].ex[0]);
                for (int b = c + 1; b < TWAVES; ++b) x = follow_block(b, x);
                if (wstate(pw) && unpack(pw) != x && l == 0) g_or32(&D.scal->err, 4u);
                st_status(ts.at(W_XF, k), pack(x, 1));
                out = true;
            }
            int64_t e = 0;
            bool ok = true;
            if (k > 0) ok = wait_word(ts.at(W_XF, k - 1), e, ctl);
            int32_t x = (int32_t)e;
            for (int b = 0; b < TWAVES; ++b) {
                s_bent[b] = x;
                x = follow_block(b, x);
            }
            if (!out && ok) {
                // a tile map may have published the exit already: it must agree
                const uint64_t pw = ld_status(ts.at(W_XF, k));
                if (wstate(pw) && unpack(pw) != x && l == 0) g_or32(&D.scal->err, 4u);
                st_status(ts.at(W_XF, k), pack(x, 1));
            }
            if (l == 0) {
                s_entry = e;
                if (!ok) g_or32(&D.scal->err, 8u);
            }
        } else if (wv == 1) {
            tile_sums();
        }
        __syncthreads();
        const int32_t ref = block_refs(D, k * TILE + wv * 64, nb, u_.blk[wv], s_bm[wv].one_from, bref,
                                       __builtin_amdgcn_readfirstlane(s_bent[wv]),
                                       __builtin_amdgcn_readfirstlane(s_bsrc[wv]));
        m_ex[tid] = (int64_t)ref - (bR + af);
    } else {
    if (tried) {  // block maps that did not fit have taken the words' place
        __syncthreads();
        m_lo[tid] = valid ? sp[SP_LO * ns] : 0;
        m_hi[tid] = valid ? sp[SP_HI * ns] : 0;
        m_af[tid] = valid ? sp[SP_AF * ns] : 0;
        m_kf[tid] = valid ? sp[SP_KF * ns] : 0;
    }
    // sparse tiles: the walker reads footprint offsets inside the tile from
    // LDS instead of scanning each group of 64 segments it enters
    if (sparse) m_R[tid] = rF;
    if (sparse || tried) __syncthreads();
    if (wv == 0) {
        // ---- the walker ----
        int q = 0;  // SIM segments passed, in walk order
        bool ok = true;
        // Sparse tiles: the kept prefixes of the predicted next stop, loaded
        // into pf while the current stop is resolved (pf_lane: its tile lane,
        // -1 if none).  At a stop they are written to ring slot 0 (unused in
        // sparse tiles; the write waits only for loads the stop needs) and
        // the registers take the next prediction's loads at once.  (32-bit
        // prefixes only: a stop in another segment loads its own.)
        int32_t pf[NW];
        int pf_lane = -1;
        auto walk = [&](int b, int e, int64_t x) -> int64_t {
            x = readlane64(x, 0);  // (wave-uniform: scalar registers)
            for (int g0 = b & ~63; g0 < e && ok; g0 += 64) {
                const int i = g0 + l;
                const int64_t lo = m_lo[i], hi = m_hi[i], af = m_af[i], kf = m_kf[i];
                const uint64_t sim = w_sim[g0 >> 6], tot = w_tot[g0 >> 6], fits = w_fit[g0 >> 6];
                const bool is_tot = (tot >> l) & 1;
                const int64_t S = sparse ? (int64_t)((uint64_t)m_R[i] - (uint64_t)m_R[g0])
                                         : (int64_t)((uint64_t)wave_incl_sum(af) - (uint64_t)af);
                // the last total-map lane before this one, and the entry it gives
                const uint64_t tb = tot & lanemask_lt();
                const int jl = tb ? top64(tb) : -1;
                const int64_t rj = (int64_t)((uint64_t)kf + (uint64_t)S + (uint64_t)af);  // kf_j + S_(j+1) on lane j
                const int64_t xt = (int64_t)((uint64_t)shfl64(rj, jl < 0 ? l : jl) - (uint64_t)S);
                const int ge = e - g0 < 64 ? e - g0 : 64;
                int i0 = b > g0 ? b - g0 : 0;
                while (i0 < ge) {
                    const int64_t xi = jl >= i0 ? xt : (int64_t)((uint64_t)x - ((uint64_t)S - (uint64_t)readlane64(S, i0)));
                    const uint64_t fire = ballot(l >= i0 && l < ge && !is_tot && !(xi >= lo && xi <= hi));
                    const int stop = fire ? ctz64(fire) : ge;
                    const int64_t xo = is_tot ? kf : (int64_t)((uint64_t)xi - (uint64_t)af);
                    if (l >= i0 && l < stop && !is_tot) m_ex[i] = xo;
                    if (!sparse) q += __popcll(sim & range_mask(0, i0, stop));
                    // release the slots passed over before any wait below (a
                    // producer may be waiting for them); every lane stores the
                    // same value (no lane-0-only region inside the loop).  A
                    // sparse tile has no producers, and the release would wait
                    // for every load in flight (the prefetch of the next stop).
                    if (!sparse) __hip_atomic_store(&s_cons, q, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (stop > i0) x = readlane64(xo, stop - 1);
                    if (stop < ge) {
                        const int64_t xs = readlane64(xi, stop);
                        int64_t r = readlane64(kf, stop);
                        if ((sim >> stop) & 1 && sparse) {
                            // The exit lies in [xs + T, max] - af for an
                            // entry below lo (one sample at the first node
                            // reaching xs + T; more only where the segment
                            // moves T or more), in [min, xs - T] - af above hi
                            // (max = lo + T - 1, min = hi - T + 1).  The next
                            // stop is predicted as the first later segment
                            // whose no-sample interval does not hold that
                            // whole range, shifted by the footprint changes in
                            // between (this group, else the next one).  A
                            // prediction only decides what is loaded early.
                            const int64_t lo_c = readlane64(lo, stop), hi_c = readlane64(hi, stop);
                            const int64_t af_c = readlane64(af, stop);
                            uint64_t A, B;
                            if (xs < lo_c) {
                                A = (uint64_t)xs + (uint64_t)T - (uint64_t)af_c;
                                B = (uint64_t)lo_c + (uint64_t)(T - 1) - (uint64_t)af_c;
                            } else {
                                A = (uint64_t)hi_c - (uint64_t)(T - 1) - (uint64_t)af_c;
                                B = (uint64_t)xs - (uint64_t)T - (uint64_t)af_c;
                            }
                            const uint64_t base = (uint64_t)readlane64(S, stop) + (uint64_t)af_c;
                            int p = -1;
                            {
                                const uint64_t d = (uint64_t)S - base;
                                const bool cand = l > stop && l < ge &&
                                                  (is_tot || !((int64_t)(A - d) >= lo && (int64_t)(B - d) <= hi));
                                const uint64_t cm = ballot(cand);
                                if (cm) {
                                    const int pl = ctz64(cm);
                                    if ((sim >> pl) & 1) p = g0 + pl;
                                } else if (g0 + 64 < e) {
                                    const int i2 = g0 + 64 + l;
                                    const bool v2 = i2 < e;
                                    const int64_t lo2 = m_lo[v2 ? i2 : 0], hi2 = m_hi[v2 ? i2 : 0];
                                    const uint64_t tot2 = w_tot[(g0 >> 6) + 1], sim2 = w_sim[(g0 >> 6) + 1];
                                    const uint64_t d2 = (uint64_t)m_R[v2 ? i2 : 0] - (uint64_t)m_R[g0] - base;
                                    const bool cand2 = v2 && (((tot2 >> l) & 1) ||
                                                              !((int64_t)(A - d2) >= lo2 && (int64_t)(B - d2) <= hi2));
                                    const uint64_t cm2 = ballot(cand2);
                                    if (cm2 && ((sim2 >> ctz64(cm2)) & 1)) p = g0 + 64 + ctz64(cm2);
                                }
                            }
                            // pf is defined once per stop (the compiler would
                            // otherwise copy it between registers, and a copy
                            // waits for the loads in flight): a miss loads
                            // into a temporary, and the next prefetch is
                            // always issued (of this segment again when there
                            // is no prediction)
                            // A segment that moves less than T samples once
                            // (hi - lo >= T - 1 implies max - min < T): its
                            // exit comes straight from the registers.  Others
                            // are walked from ring slot 0.
                            const int c = g0 + stop;
                            const bool one = (uint64_t)hi_c - (uint64_t)lo_c >= (uint64_t)(T - 1) && hi_c >= lo_c;
                            const bool up = xs < lo_c;
                            const bool fit = (fits >> stop) & 1;
                            if (pf_lane == c && fit) {
                                if (one) {
                                    r = exit_one_sample(pf, T, xs, up);
                                } else {
#pragma unroll
                                    for (int w = 0; w < NW; ++w) ring[0][w * 64 + l] = pf[w];
                                }
                            } else {
                                int64_t tmp[NW];
                                load_kept(D, k * TILE + c, fit, tmp);
                                if (one) {
                                    r = exit_one_sample(tmp, T, xs, up);
                                } else {
#pragma unroll
                                    for (int w = 0; w < NW; ++w) ring[0][w * 64 + l] = tmp[w];
                                }
                            }
                            pf_lane = p;
                            load_kept32(D, k * TILE + (p >= 0 ? p : c), pf);
                            if (!one) r = walk_prefixes(ring[0], T, xs);
                        } else if ((sim >> stop) & 1) {
                            const int slot = q % RING;
                            if (kept && __hip_atomic_load(&r_ready[slot], __ATOMIC_ACQUIRE,
                                                          __HIP_MEMORY_SCOPE_WORKGROUP) != q) {
                                // its producer is behind: read the kept prefixes instead of waiting
                                r = walk_kept(D, k * TILE + g0 + stop, (fits >> stop) & 1, T, xs);
                            } else {
                                LocalSpin sp_;
                                while (__hip_atomic_load(&r_ready[slot], __ATOMIC_ACQUIRE,
                                                         __HIP_MEMORY_SCOPE_WORKGROUP) != q) {
                                    if (local_spin_abort(ctl, sp_)) {
                                        ok = false;
                                        break;
                                    }
                                }
                                r = ok ? walk_prefixes(ring[slot], T, xs) : 0;
                            }
                            ++q;
                            __hip_atomic_store(&s_cons, q, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                        }
                        if (l == stop) m_ex[i] = r;
                        x = r;
                    }
                    i0 = stop + 1;
                    if (!ok) break;
                }
            }
            return x;
        };
        // (ft, nval): entry-independent
        if (ft < nval) {
            const int64_t xa = walk(ft + 1, nval, m_kf[ft]);
            st_status(ts.at(W_XF, k), pack(xa, 1));
        }
        // the tile's entry, then [0, ft)
        int64_t e = 0;
        // A tile with a map whose exit the map chain has not published (a
        // tile before it has no map): the exit follows from the entry by one
        // lookup and is published before the walk, so that the next tile
        // need not wait for the walk.  The map loads while the entry is
        // awaited.
        const bool use_map = D.tmap && ft >= nval && k > 0;
        int64_t mh = 0, mr[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        if (use_map) {
            const SMP_GLOBAL int64_t* mp = tile_map(D, k);
            if (l < 4) mh = mp[TM_HDR + l];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                mr[w] = mp[4 * l + w];
                mr[4 + w] = mp[TM_RUN_HI + 4 * l + w];
            }
        }
        if (k > 0 && ok) ok = wait_word(ts.at(W_XF, k - 1), e, ctl);
        if (use_map && ok && readlane64(mh, 0) == TM_MAPPED && !wstate(ld_status(ts.at(W_XF, k)))) {
            const int64_t x = map_exit(e, (int)readlane64(mh, 1), (int)readlane64(mh, 2), readlane64(mh, 3), mr[0],
                                       mr[4], mr[1], mr[5], mr[2], mr[6], mr[3], mr[7]);
            st_status(ts.at(W_XF, k), pack(x, 1));
        }
        const int64_t xb = ok ? walk(0, ft, e) : 0;
        if (ft >= nval) {
            // a tile map may have published the exit already: it must agree
            const uint64_t pw = ld_status(ts.at(W_XF, k));
            if (wstate(pw) && unpack(pw) != xb && l == 0) g_or32(&D.scal->err, 4u);
            st_status(ts.at(W_XF, k), pack(xb, 1));
        }
        if (l == 0) {
            s_entry = e;
            if (!ok) {
                g_or32(&D.scal->err, 8u);
                __hip_atomic_store(&s_abort, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
    } else {
        if (wv == 1) tile_sums();
        // ---- producers: pre-scan SIM segments in walk order (dense tiles only) ----
        if (!sparse) for (;;) {
            // every lane takes part (lane 0 adds 1, the others 0): a lane-0-only
            // region here lets the compiler split the wave across loop trips
            const int pidx = __builtin_amdgcn_readfirstlane(
                __hip_atomic_fetch_add(&s_prod, l == 0 ? 1 : 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
            if (pidx >= nsim) break;
            // its lane: the pidx-th SIM lane of (ft, nval), else of [0, ft)
            int r = pidx < nA ? pidx : pidx - nA;
            const int rlo = pidx < nA ? ft + 1 : 0, rhi = pidx < nA ? nval : ft;
            int lane = -1;
            for (int w = 0; w < TWAVES && lane < 0; ++w) {
                const uint64_t m = w_sim[w] & range_mask(w, rlo, rhi);
                const int c = __popcll(m);
                if (r < c) lane = w * 64 + nth_bit(m, r);
                else r -= c;
            }
            // Wait until the slot is free: the walker has passed its previous
            // occupant (it may pass one without reading it) and that
            // occupant's producer has finished writing.
            const int slot = pidx % RING;
            LocalSpin sp_;
            bool ok = true;
            while (__hip_atomic_load(&s_cons, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) <= pidx - RING ||
                   (pidx >= RING &&
                    __hip_atomic_load(&r_ready[slot], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) != pidx - RING)) {
                if (__hip_atomic_load(&s_abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) ||
                    local_spin_abort(ctl, sp_)) {
                    ok = false;
                    break;
                }
            }
            if (!ok) break;
            // a segment the walker has already passed is not scanned
            if (lane >= 0 && __hip_atomic_load(&s_cons, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) <= pidx) {
                if (kept) copy_prefixes(D, k * TILE + lane, (w_fit[lane >> 6] >> (lane & 63)) & 1, ring[slot]);
                else prescan_segment(D, k * TILE + lane, ring[slot]);
            }
            __hip_atomic_store(&r_ready[slot], pidx, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    }
    __syncthreads();
    const int64_t ef = tid == 0 ? s_entry : m_ex[tid - 1];
    const int64_t ex = m_ex[tid];
    const int64_t F0 = s_pre[0] + rF;
    const int64_t P0 = s_pre[1] + rP;
    const int64_t C0 = s_pre[2] + rC;
    uint32_t err = 0;
    int64_t pk = 0, pks = 0;
    bool left = false;  // left to the chain pass
    if (valid) {
        const int64_t af = sp[SP_AF * ns], ac = sp[SP_AC * ns];
        // (read again: kept in registers across the block maps they would spill)
        const int64_t mxf = sp[SP_MXF * ns], mnf = sp[SP_MNF * ns], mxp = sp[SP_MXP * ns], mnp = sp[SP_MNP * ns];
        const int64_t lo = sp[SP_LO * ns], hi = sp[SP_HI * ns];
        SMP_GLOBAL int64_t* o = gp(D.seg) + j;
        o[SP_F0 * ns] = F0;
        o[SP_P0 * ns] = P0;
        o[SP_C0 * ns] = C0;
        o[SP_EF * ns] = ef;
        o[SP_XF * ns] = ex;
        if (F0 + mxf >= MAX_ABS_F || F0 + mnf <= -MAX_ABS_F || P0 + mxp >= MAX_ABS_F || P0 + mnp <= -MAX_ABS_F ||
            C0 + ac >= MAX_ABS_F || F0 >= MAX_ABS_F || F0 <= -MAX_ABS_F)
            err = 2u;
        pk = F0 + mxf;
        if (j == ns - 1) *gp(&D.scal->final_F) = F0 + af;
        // The chain pass's results, here, for a segment whose entry takes no
        // sample before its first forced event (the prefix's only sample is
        // that event's, and from it on the chain is the summary pass's) or,
        // without a forced event, no sample at all.  Every other segment is
        // left to the chain pass.  (Copy and timer events are counted by the
        // emit pass.)
        const int fn = (int)sp[SP_FN * ns];
        if (fn < 0 && ef >= lo && ef <= hi) {
            // no forced event and an entry inside the no-sample interval:
            // the segment takes no sample
            o[SP_BCNT * ns] = 0;
            o[SP_BGV * ns] = 0;
            o[SP_BGI * ns] = 0;
            o[SP_BGP * ns] = 0;
            o[SP_LSV * ns] = 0;
            o[SP_BFL * ns] = 0;
            SMP_GLOBAL uint64_t* mk = gp(D.mask) + j * NW;
#pragma unroll
            for (int w = 0; w < NW; ++w) mk[w] = 0;
        } else if (fn >= 0 && ef >= sp[SP_PLO * ns] && ef <= sp[SP_PHI * ns]) {
            const int64_t ffn = sp[SP_FFN * ns];
            int64_t gbest = 0, smax = ffn, lsrel;
            int gnode = -1;
            if (ffn > ef) {
                gbest = ffn;
                gnode = fn;
            }
            const int64_t agv = sp[SP_AGV * ns], asmx = sp[SP_ASMX * ns];
            const int agn = (int)sp[SP_AGN * ns], als = (int)sp[SP_ALS * ns];
            if (agn >= 0 && (gnode < 0 || agv > gbest)) {
                gbest = agv;
                gnode = agn;
            }
            if (asmx > smax) smax = asmx;
            lsrel = als >= 0 ? sp[SP_ALP * ns] : sp[SP_PFN * ns];
            pks = F0 + smax;
            const int64_t a = j * SEG;
            const bool hg = gnode >= 0 && gnode < seg_events(D, j);
            o[SP_BCNT * ns] = 1 + sp[SP_ACNT * ns];
            o[SP_BGV * ns] = hg ? F0 + gbest : 0;
            o[SP_BGI * ns] = hg ? a + gnode : 0;
            o[SP_BGP * ns] = hg ? (int64_t)(uint32_t)record(D, a + gnode)[1] : 0;
            o[SP_LSV * ns] = P0 + lsrel;
            o[SP_BFL * ns] = (hg ? 1 : 0) | 2;
            // windows before the forced one hold no sample (as the summary
            // pass wrote); the forced window gains the forced sample
            gp(D.mask)[j * NW + (fn >> 6)] = (1ull << (fn & 63)) | (uint64_t)sp[SP_AMF * ns];
        } else {
            o[SP_BFL * ns] = BFL_CHAIN;
            left = true;
        }
    }
    if (ballot(err != 0) && l == 0) g_or32(&D.scal->err, 2u);
    const int nleft = __popcll(ballot(left));
    pk = wave_max(pk);
    pks = wave_max(pks);
    if (l == 0) {
        w_peak[wv] = pk;
        w_peakS[wv] = pks;
        w_left[wv] = nleft;
    }
    __syncthreads();
    if (tid == 0) {
        int64_t p = 0, q = 0;
        uint64_t c = 0;
        for (int w = 0; w < TWAVES; ++w) {
            p = w_peak[w] > p ? w_peak[w] : p;
            q = w_peakS[w] > q ? w_peakS[w] : q;
            c += (uint64_t)w_left[w];
        }
        if (p > 0) g_max(&D.scal->peak_F, (int64_t)p);
        if (q > 0) g_max(&D.scal->peak_S, (int64_t)q);
        if (c) g_add((uint64_t*)&ctl[4], c);
        if (tried) g_add((uint64_t*)&ctl[blocks ? 11 : 12], 1ull);
    }
}

// -------------------------------------------------------------- chain pass

// The first two windows of a segment's records (delta, pointer, flags), which
// the chain pass loads one marked segment ahead: in most segments the first
// forced event lies in them, so the walk needs no other record.
constexpr int HEAD_W = 2;  // (the pointer lookup below assumes two)
struct ChainHead {
    uint64_t d[HEAD_W];
    uint32_t ptr[HEAD_W];
    uint32_t fw[HEAD_W];
};

__device__ __forceinline__ void load_head(const Desc& D, int64_t j, ChainHead& h) {
    gu8_t* base = (gu8_t*)(D.ev + (size_t)(j * SEG) * 24);  // wave-uniform
    const int nv = seg_events(D, j);
#pragma unroll
    for (int w = 0; w < HEAD_W; ++w) {
        gu8_t* p = record_addr(base, nv, w);
        h.d[w] = *(gu64_t*)p;
        h.ptr[w] = *(gu32_t*)(p + 8);
        h.fw[w] = *(gu32_t*)(p + 16);
    }
}

// One wave per segment (grid-stride): follow the chain from the segment's
// entry offset; record its samples, count, best growth sample and the Python
// footprint at its last sample.  (Copy and timer events are the emit pass's.)
__global__ __launch_bounds__(BLOCK) void k_chain(const Desc* __restrict__ desc, int ntraces, uint64_t nseg_total,
                                                 uint64_t* ts) {
    stamp(ts);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
    const int l = lane_id();
    int cur_t = 0;
    // lanes 0-4: prefixes, entry and exit from the resolve pass; lanes 5-17:
    // flags, the chain after the first forced sample and the entries that
    // take no sample before it, from the summary pass.  Each wave reads them
    // one segment ahead.
    const int pl_ = l < 5 ? SP_F0 + l : (l == 5 ? SP_FLG : (l < 18 ? SP_FN + (l - 6) : SP_F0));
    // Only the segments the resolve pass left to this pass, grid-stride:
    // each wave reads the flags of its next 64 segments in one load (lane i:
    // the i-th) and visits the marked ones.
    const uint64_t stride = (uint64_t)gridDim.x * WAVES;
    uint64_t gb = (uint64_t)blockIdx.x * WAVES + wv, cur_gb = 0;
    uint64_t pend = 0;  // marked segments among the last 64 read, not yet taken
    int hint = 0;       // a trace at or before the wave's next segment
    auto next_marked = [&]() -> uint64_t {
        while (!pend) {
            if (gb >= nseg_total) return nseg_total;
            hint = __builtin_amdgcn_readfirstlane(find_trace_seg(desc, hint, ntraces, gb));
            const uint64_t x = gb + (uint64_t)l * stride;
            bool mk = false;
            if (x < nseg_total) {
                const Desc& Dx = desc[find_trace_seg(desc, hint, ntraces, x)];
                mk = seg_val(Dx, SP_BFL, (int64_t)(x - Dx.seg_begin)) == BFL_CHAIN;
            }
            pend = ballot(mk);
            cur_gb = gb;
            gb += 64 * stride;
        }
        const int i = ctz64(pend);
        pend &= pend - 1;
        return cur_gb + (uint64_t)i * stride;
    };
    uint64_t g = next_marked();
    int64_t pv_next = 0;
    ChainHead hd;  // the head of the wave's next segment
    if (g < nseg_total) {
        const Desc& D0 = desc[__builtin_amdgcn_readfirstlane(find_trace_seg(desc, 0, ntraces, g))];
        pv_next = seg_val(D0, pl_, (int64_t)(g - D0.seg_begin));
        load_head(D0, (int64_t)(g - D0.seg_begin), hd);
    }
    for (uint64_t gn; g < nseg_total; g = gn) {
        gn = next_marked();
        const int t = __builtin_amdgcn_readfirstlane(find_trace_seg(desc, cur_t, ntraces, g));
        cur_t = t;
        const Desc& D = desc[t];
        const int64_t j = (int64_t)(g - D.seg_begin);
        const int64_t ns = (int64_t)D.nseg;
        const int64_t a = j * SEG;
        const int nv = seg_events(D, j);
        const int64_t T = D.T;
        const int64_t pv = pv_next;
        const ChainHead cur = hd;
        {
            // past the last segment, this one's again (no branch)
            const uint64_t gq = gn < nseg_total ? gn : g;
            const Desc& Dn = desc[__builtin_amdgcn_readfirstlane(find_trace_seg(desc, t, ntraces, gq))];
            pv_next = seg_val(Dn, pl_, (int64_t)(gq - Dn.seg_begin));
            load_head(Dn, (int64_t)(gq - Dn.seg_begin), hd);
        }
        const int64_t F0 = readlane64(pv, 0), P0 = readlane64(pv, 1);
        const int64_t eF = readlane64(pv, 3), xF = readlane64(pv, 4);
        const int fn = (int)readlane64(pv, 6);
        // The pointer of the summary pass's best growth sample after the forced
        // event, loaded now (it is the segment's best unless the walk below
        // finds a larger one before the forced event).
        const int agn0 = (int)readlane64(pv, 9);
        uint32_t aptr = 0;
        if (fn >= 0 && agn0 >= 0 && agn0 < nv) aptr = (uint32_t)record(D, a + agn0)[1];
        // From a forced sample on the chain is the one the summary pass followed,
        // so only the events up to it are read again.
        const int fwin = fn >= 0 ? fn >> 6 : NW - 1;
        const int nlim = fn >= 0 ? fn + 1 : nv;
        uint32_t err = 0;
        ChainRun cr{eF, 0, 0, -1, INT64_MIN, -1, 0};
        int64_t lsp = 0, cF = 0, cP = 0;
        const int64_t plo = readlane64(pv, 14), phi = readlane64(pv, 15);
        if (fn >= 0 && eF >= plo && eF <= phi) {
            // No sample before the forced event: the prefix's chain is that
            // event's sample alone, known from the summary pass.
            const int64_t ffn = readlane64(pv, 16);
            if (ffn > eF) {
                cr.gbest = ffn;
                cr.gnode = fn;
            }
            cr.smax = ffn;
            cr.lastS = fn;
            cr.ref = ffn;
            if (l == fwin) cr.mvec = 1ull << (fn & 63);
            cr.cnt = 1;
            lsp = readlane64(pv, 17);
        } else {
            // the chain from the entry, window by window while scanning
            // (prefixes in registers): the head from the prefetch, later
            // windows loaded here
            uint64_t rd[NW - HEAD_W];
            uint32_t rfw[NW - HEAD_W];
            if (fwin >= HEAD_W) {
                gu8_t* base = (gu8_t*)(D.ev + (size_t)a * 24);  // wave-uniform
#pragma unroll
                for (int w = HEAD_W; w < NW; ++w) {
                    gu8_t* p = record_addr(base, nlim, w);
                    rd[w - HEAD_W] = *(gu64_t*)p;
                    rfw[w - HEAD_W] = *(gu32_t*)(p + 16);
                }
            }
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                if (w > fwin) break;
                const int k = w * 64 + l;
                const uint32_t fl = w < HEAD_W ? cur.fw[w] : rfw[w - HEAD_W];
                const uint64_t rdw = w < HEAD_W ? cur.d[w] : rd[w - HEAD_W];
                const int64_t dm = (k < nlim && (fl & 6u) == 0) ? (int64_t)rdw : 0;
                const int64_t dp = (fl & 1u) ? 0 : dm;
                int64_t f = dm, p = dp;
                wave_incl_sum2(f, p);
                f += cF;
                p += cP;
                cF = readlane64(f, 63);
                cP = readlane64(p, 63);
                chain_window<true>(f, p, T, cr, lsp, w, -1);
            }
        }

        int64_t count = cr.cnt;
        int64_t gbest = cr.gbest, smax = cr.smax, lsrel = 0;
        int gnode = cr.gnode, lastS = cr.lastS;
        if (fn >= 0) {
            if (lastS != fn) err |= 4u;  // internal: every entry samples at a forced event
            count += readlane64(pv, 7);
            const int64_t agv = readlane64(pv, 8), asmx = readlane64(pv, 10);
            const int agn = (int)readlane64(pv, 9), als = (int)readlane64(pv, 11);
            if (agn >= 0 && (gnode < 0 || agv > gbest)) {
                gbest = agv;
                gnode = agn;
            }
            if (asmx > smax) smax = asmx;
            if (als >= 0) {
                lastS = als;
                lsrel = readlane64(pv, 12);
            } else {
                lsrel = lsp;  // the forced sample is the prefix's last
            }
        } else {
            if (cr.ref - cF != xF) err |= 4u;  // internal: the resolved exit disagrees with the chain
            if (lastS >= 0) lsrel = lsp;
        }
        const bool hg = gnode >= 0 && gnode < nv;  // nodes past the trace end never sample
        uint32_t gptr = 0;
        if (hg) {
            if (fn >= 0 && gnode > fn)
                gptr = aptr;  // the summary pass's sample (gnode == agn0)
            else if (gnode < HEAD_W * 64)
                gptr = (uint32_t)readlane32((int)((gnode >> 6) == 0 ? cur.ptr[0] : cur.ptr[1]), gnode & 63);
            else
                gptr = (uint32_t)record(D, a + gnode)[1];
        }
        const int64_t lsv = lastS >= 0 ? P0 + lsrel : 0;
        // The segment's largest sample goes to the scan pass, which updates the
        // trace's peak once per tile: updates by every wave queued behind one
        // another.  The pass on one trace of 1e8 events 115 -> 65 us, of 2e7
        // 163 -> 113, of 3e6 78 -> 21; two of 1e7 166 -> 95.
        if (l < 7) {
            int64_t v;
            switch (l) {
                case 0: v = count; break;
                case 1: v = hg ? F0 + gbest : 0; break;
                case 2: v = hg ? a + gnode : 0; break;
                case 3: v = gptr; break;
                case 4: v = lsv; break;
                case 5: v = (hg ? 1 : 0) | (lastS >= 0 ? 2 : 0) | (smax != INT64_MIN ? BFL_PEAK : 0); break;
                default: v = smax != INT64_MIN ? F0 + smax : 0; break;
            }
            gp(D.seg)[(SP_BCNT + l) * ns + j] = v;
        }
        // windows after the forced sample's keep the summary pass's masks
        const uint64_t amf = fn >= 0 ? (uint64_t)readlane64(pv, 13) : 0ull;
        if (l < NW && l <= fwin) gp(D.mask)[j * NW + l] = cr.mvec | (l == fwin ? amf : 0ull);
        if (err && l == 0) g_or32(&D.scal->err, err);
    }
}

// --------------------------------------------------------------- scan pass

// (count, best growth record, last-sample Python footprint) of a run of segments.
struct BItem {
    Best b;
    bool lsh;
    int64_t ls;
};

__device__ __forceinline__ BItem bcombine(const BItem& a, const BItem& b) {
    BItem r;
    r.b = combine(a.b, b.b);
    r.lsh = a.lsh || b.lsh;
    r.ls = b.lsh ? b.ls : a.ls;
    return r;
}

// One workgroup per tile (ticket order): the state before every segment.
__global__ __launch_bounds__(TILE) void k_bscan(const Desc* __restrict__ desc, int ntraces, uint64_t ntile_total,
                                                unsigned long long* ctl, uint64_t* ts_) {
    stamp(ts_);
    __shared__ unsigned long long s_tk;
    __shared__ int64_t w_cnt[TWAVES], w_val[TWAVES], w_ls[TWAVES], w_peak[TWAVES];
    __shared__ uint32_t w_idx[TWAVES], w_ptr[TWAVES];
    __shared__ int w_flags[TWAVES];
    __shared__ int64_t s_pre_cnt, s_pre_val, s_pre_ls;
    __shared__ uint32_t s_pre_idx, s_pre_ptr;
    __shared__ int s_pre_has;
    const int tid = threadIdx.x, wv = tid >> 6, l = lane_id();
    if (tid == 0) s_tk = g_add_rtn((uint64_t*)&ctl[3], 1ull);
    __syncthreads();
    const uint64_t tk = s_tk;
    if (tk >= ntile_total) return;
    const Desc& D = desc[find_trace_tile(desc, ntraces, tk)];
    const int64_t k = (int64_t)(tk - D.tile_begin);
    const int64_t ns = (int64_t)D.nseg;
    const int64_t j = k * TILE + tid;
    const bool valid = j < ns;
    const StatusView ts{D.tstat, (int64_t)D.ntile};
    int64_t cnt = 0, gv = 0, gi = 0, gpt = 0, lsv = 0, fl = 0, pk = 0;
    if (valid) {
        const SMP_GLOBAL int64_t* sp = gp(D.seg) + j;
        cnt = sp[SP_BCNT * ns];
        gv = sp[SP_BGV * ns];
        gi = sp[SP_BGI * ns];
        gpt = sp[SP_BGP * ns];
        lsv = sp[SP_LSV * ns];
        fl = sp[SP_BFL * ns];
        pk = sp[SP_BPK * ns];
    }
    const int64_t peak = wave_max((fl & BFL_PEAK) ? pk : 0);  // largest sample of the chain pass's segments
    const bool hg = (fl & 1) != 0, hs = (fl & 2) != 0;
    // inclusive within the wave
    const int64_t icnt = wave_incl_sum(cnt);
    const int64_t M = wave_incl_max(hg ? gv : INT64_MIN);
    const int64_t Mp = wave_shr1(M, INT64_MIN);
    const uint64_t le = lanemask_lt() | (1ull << l);
    const uint64_t bnd = ballot(M != INT64_MIN && M > Mp) & le;  // where the running maximum rises
    const int src = bnd ? top64(bnd) : l;
    const uint32_t iidx = (uint32_t)shfl32((int)(uint32_t)gi, src), iptr = (uint32_t)shfl32((int)(uint32_t)gpt, src);
    const uint64_t lsm = ballot(hs) & le;
    const int lsrc = lsm ? top64(lsm) : l;
    const int64_t ils = shfl64(lsv, lsrc);
    if (l == 63) {
        w_cnt[wv] = icnt;
        w_val[wv] = M;
        w_idx[wv] = iidx;
        w_ptr[wv] = iptr;
        w_ls[wv] = ils;
        w_peak[wv] = peak;
        w_flags[wv] = (M != INT64_MIN ? 1 : 0) | (lsm ? 2 : 0);
    }
    __syncthreads();
    BItem wpre{{0, false, 0, 0, 0}, false, 0}, agg{{0, false, 0, 0, 0}, false, 0};
    for (int w = 0; w < TWAVES; ++w) {
        if (w == wv) wpre = agg;
        const BItem it{{w_cnt[w], (w_flags[w] & 1) != 0, w_val[w], w_idx[w], w_ptr[w]}, (w_flags[w] & 2) != 0, w_ls[w]};
        agg = bcombine(agg, it);
    }
    if (tid == 0) {
        int64_t p = 0;
        for (int w = 0; w < TWAVES; ++w) p = sgt64(w_peak[w], p) ? w_peak[w] : p;
        if (p > 0) g_max(&D.scal->peak_S, p);
        st_status(ts.at(W_BCNT, k), pack(agg.b.cnt, 1));
        st_status(ts.at(W_BGM, k), pack(agg.b.has ? agg.b.val : 0, agg.b.has ? 2 : 1));
        st_status(ts.at(W_BGR, k), pack((int64_t)agg.b.idx, 1));
        st_status(ts.at(W_BGP, k), pack((int64_t)agg.b.ptr, 1));
        st_status(ts.at(W_LSA, k), pack(agg.ls, agg.lsh ? 2 : 1));
    }
    if (wv == 0) {
        Best pre{0, false, 0, 0, 0};
        int64_t eP = 0;
        bool ok = true;
        if (k > 0) {
            ok = scan_best(ts, k, pre, ctl);
            if (ok) ok = scan_last_sample(ts, k, eP, ctl);
        }
        const Best inc = with_baseline(combine(pre, agg.b));
        if (l == 0) {
            st_status(ts.at(W_ICNT, k), pack(inc.cnt, 1));
            st_status(ts.at(W_IGM, k), pack(inc.val, inc.has ? 2 : 1));
            st_status(ts.at(W_IGR, k), pack((int64_t)inc.idx, 1));
            st_status(ts.at(W_IGP, k), pack((int64_t)inc.ptr, 1));
            st_status(ts.at(W_LSI, k), pack(agg.lsh ? agg.ls : eP, 1));
            s_pre_cnt = pre.cnt;
            s_pre_has = pre.has ? 1 : 0;
            s_pre_val = pre.val;
            s_pre_idx = pre.idx;
            s_pre_ptr = pre.ptr;
            s_pre_ls = eP;
            if (!ok) g_or32(&D.scal->err, 8u);
        }
    }
    __syncthreads();
    // state before this segment: tile prefix, waves before, lanes before
    const BItem tpre{{s_pre_cnt, s_pre_has != 0, s_pre_val, s_pre_idx, s_pre_ptr}, true, s_pre_ls};
    const int pl = l > 0 ? l - 1 : 0;
    const int64_t pcnt = shfl64(icnt, pl);
    const uint32_t pidx = (uint32_t)shfl32((int)iidx, pl), pptr = (uint32_t)shfl32((int)iptr, pl);
    const int64_t pls = shfl64(ils, pl);
    const bool plsh = l > 0 && (lsm & ~(1ull << l)) != 0;
    BItem lpre{{l > 0 ? pcnt : 0, l > 0 && Mp != INT64_MIN, Mp, pidx, pptr}, plsh, pls};
    const BItem st = bcombine(bcombine(tpre, wpre), lpre);
    const Best b = with_baseline(st.b);
    if (valid) {
        SMP_GLOBAL int64_t* o = gp(D.seg) + j;
        o[SP_XCNT * ns] = b.cnt;
        o[SP_XHV * ns] = b.val;
        o[SP_XHI * ns] = b.idx;
        o[SP_XHP * ns] = b.ptr;
        o[SP_XFL * ns] = b.has ? 1 : 0;
        o[SP_XLS * ns] = st.ls;
        if (j == ns - 1) *gp(&D.scal->K) = (uint64_t)(b.cnt + cnt);
    }
}

// --------------------------------------------------------------- emit pass

// One wave per segment (grid-stride): write the segment's samples with their
// attribution, per-line counters, tracked samples and the frees that reclaim
// them.
// What a wave collects before it writes it out or adds it to the line tables,
// up to 64 at a time: a window holds a few samples, copies and timers, and one
// by one they would keep a few lanes busy each time.
struct Staging {
    Sample smp[64];
    uint64_t ax[64];  // copies and timers: bytes or delay, bit 63: timer
    uint32_t aline[64];
};

// Write staged samples [0, cnt) (cnt <= 64) to ranks r0.. and add them to
// their lines' counters, one sample per lane.
template <class C>
__device__ __forceinline__ void flush_stage(const Desc& D, uint32_t t, const Sample* stg, int cnt, int64_t r0, C& hc) {
    const int l = lane_id();
    if (l < cnt && r0 + l < (int64_t)D.n) {
        const Sample smp = stg[l];
        store_sample(D.samples + r0 + l, smp);
        if (smp.line < D.L) count_sample(hc, D, t, smp.line, smp.py, smp.nat);
    }
}

// Add staged copies and timers [0, cnt) (cnt <= 64) to their lines' counters.
template <class C>
__device__ __forceinline__ void flush_aux(const Desc& D, uint32_t t, const Staging& sg, int cnt, C& hc) {
    const int l = lane_id();
    if (l < cnt) {
        const uint64_t x = sg.ax[l];
        count_aux(hc, D, t, sg.aline[l], (x >> 63) != 0, x & ~(1ull << 63), 0);
    }
}

// What the emit pass loads for a segment: its records, its plane values
// (lanes 0-3: F0, P0, C0, entry offset; lanes 4-9: the scan state before
// the segment; lane 18: its copy bytes; lane 19: its summary flags) and its
// sample masks (lane w: window w).
// The emit pass carries each window's records from one segment to the next
// as one 16-byte vector (delta, pointer, line) and the flags word: the
// registers a refill load writes are then the ones the next segment reads,
// with no copy (a copy would wait for the load).  pv holds, on lanes 0-3,
// F0, P0, C0 and the entry offset, on lanes 4-9 the scan state before the
// segment, on lanes 10-17 the sample masks of windows 0-7, on lane 18 the
// segment's copy bytes and on lane 19 its summary flags.
typedef uint32_t v4u32 __attribute__((ext_vector_type(4), aligned(8)));
typedef const __attribute__((address_space(1))) v4u32 gv4u32_t;

struct EmitIn {
    v4u32 q[NW];
    uint32_t fw[NW];
    int64_t pv;
};

__device__ __forceinline__ void emit_load_record(gu8_t* p, int w, EmitIn& in) {
    in.q[w] = *(gv4u32_t*)p;
    in.fw[w] = *(gu32_t*)(p + 16);
}

// A segment of the emit pass: trace t, index j in the trace, nv records.
struct EmitSeg {
    int t;
    int64_t j;
    int nv;
};

__device__ __forceinline__ void emit_fetch_meta(const Desc& D, int64_t j, EmitIn& in) {
    const int l = lane_id();
    const int pl = l < 4 ? SP_F0 + (l == 3 ? SP_EF - SP_F0 : l) : (l == 18 ? SP_AC : (l == 19 ? SP_FLG : SP_XCNT + (l - 4)));
    gi64_t* src = (l < 10 || l == 18 || l == 19) ? (gi64_t*)D.seg + (int64_t)pl * (int64_t)D.nseg + j
                                                 : (gi64_t*)D.mask + j * NW + ((l - 10) & (NW - 1));
    in.pv = *src;
}

// Emit segment s from in: its samples (staged in stg), the tracked and freed
// bits of its growth samples and its lines' counters.  When hn, the wave's
// next segment sn is loaded into in as this one is consumed: its planes at
// the start, its records window by window as each window's registers free up
// (so the next segment's loads are in flight while this one computes).
template <class C>
__device__ __forceinline__ void emit_segment(const Desc* __restrict__ desc, const EmitSeg& s, C& hc, Staging& sg,
                                             EmitIn& in, bool hn, const EmitSeg& sn) {
    const int l = lane_id();
    const int t = s.t;
    const Desc& D = desc[t];
    const int64_t a = s.j * SEG;
    const int nv = s.nv;
    const int64_t pv = in.pv;
    const Desc& Dn = desc[sn.t];
    gu8_t* nbase = (gu8_t*)(Dn.ev + (size_t)(sn.j * SEG) * 24);  // wave-uniform
    const int64_t F0 = readlane64(pv, 0), P0 = readlane64(pv, 1), eF = readlane64(pv, 3);
    // Copy volume (section 3.5: one Tc sample per multiple of Tc crossed by
    // the cumulative copy bytes) and the timer split (section 2.1: Python
    // time += quantum, native time += delay) go to the lines' counters here.
    // Only a segment that holds such events (FLG_AUX) looks for
    // them, and only one whose copy bytes cross a multiple of Tc holds a copy
    // sample and scans its copy bytes.
    const bool has_aux = (readlane64(pv, 19) & FLG_AUX) != 0;
    int64_t cc = 0;
    bool csmp = false;
    if (has_aux) {
        cc = readlane64(pv, 2);
        const uint64_t c0u = (uint64_t)cc, c1u = c0u + (uint64_t)readlane64(pv, 18);
        csmp = D.tc_shift >= 0 ? (c1u >> D.tc_shift) != (c0u >> D.tc_shift)
                               : c1u / (uint64_t)D.Tc != c0u / (uint64_t)D.Tc;
    }
    int64_t base = readlane64(pv, 4);
    const int64_t hv = readlane64(pv, 5);
    const uint32_t hidx = (uint32_t)readlane64(pv, 6), hptr = (uint32_t)readlane64(pv, 7);
    const bool hh = (readlane64(pv, 8) & 1) != 0;
    const int64_t eP = readlane64(pv, 9);
    uint64_t wm[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) wm[w] = readlaneu64((uint64_t)pv, 10 + w);
    if (hn) emit_fetch_meta(Dn, sn.j, in);
    uint32_t err = 0;
    if (base < 0 || base > (int64_t)D.n) {  // only reachable after an internal fault
        err |= 8u;
        base = 0;
    }
    int64_t refF = eF, refP = eP - P0;
    int64_t cnt = 0;
    bool cur_has = hh;
    uint32_t cur_ptr = hptr, cur_idx = hidx;
    int64_t hwm = hh ? hv : 0;
    int64_t cF = 0, cP = 0;
    // Sample records are staged in LDS in rank order and written (with their
    // per-line counters) up to 64 at a time; copies and timers likewise.
    Sample* stg = sg.smp;
    int staged = 0, aux = 0;
    int64_t stage_rank = base;
    // Window by window: decode and scan (prefixes stay in registers), then
    // the window's samples and frees.
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int k = w * 64 + l;
        const uint32_t fl = in.fw[w];
        const int64_t dm = (k < nv && (fl & 6u) == 0) ? (int64_t)(((uint64_t)in.q[w].y << 32) | in.q[w].x) : 0;
        const int64_t dp = (fl & 1u) ? 0 : dm;
        int64_t f = dm, p = dp;
        wave_incl_sum2(f, p);
        f += cF;
        p += cP;
        cF = readlane64(f, 63);
        cP = readlane64(p, 63);
        const uint64_t fm = ballot(dm < 0);
        const uint64_t m = wm[w];
        if (staged + __popcll(m) > 64) {
            flush_stage(D, (uint32_t)t, stg, staged, stage_rank, hc);
            stage_rank += staged;
            staged = 0;
        }
        if (m != 0 || (fm != 0 && cur_has)) {
            const uint32_t pt = in.q[w].z, wline = in.q[w].w;
            const uint64_t below = m & lanemask_lt();
            uint64_t tmask = 0;
            if (m) {
                const int pl = below ? top64(below) : l;
                int64_t fprev = shfl64(f, pl), pprev = shfl64(p, pl);
                if (!below) {
                    fprev = refF;
                    pprev = refP;
                }
                const bool is_s = ((m >> l) & 1) && k < nv;
                const int64_t dl = f - fprev;
                const int64_t pyb = p - pprev;
                const int64_t nat = dl - pyb;
                const int64_t Fabs = F0 + f;
                const int64_t rank = base + cnt + __popcll(below);
                if (is_s) {
                    Sample smp;
                    smp.event_idx = (uint32_t)(a + k);
                    smp.line = wline;
                    smp.F = Fabs;
                    smp.py = pyb;
                    smp.nat = nat;
                    stg[staged + __popcll(below)] = smp;
                }
                uint64_t cand = ballot(is_s && dl > 0 && Fabs > hwm);
                while (cand) {
                    const int c = ctz64(cand);
                    cand &= cand - 1;
                    const int64_t Fc = readlane64(Fabs, c);
                    if (Fc > hwm) {
                        hwm = Fc;
                        tmask |= 1ull << c;
                    }
                }
                if (((tmask >> l) & 1) && rank < (int64_t)D.n) {
                    g_or(&D.tracked_bits[rank >> 6], 1ull << (rank & 63));
                    gp(D.sample_ptr)[rank] = pt;
                }
                const int ls = top64(m);
                refF = readlane64(f, ls);
                refP = readlane64(p, ls);
            }
            if (fm && tmask) {
                // a new tracked object in this window: each free compares
                // with the last one tracked before it
                const uint64_t tb = tmask & lanemask_lt();
                const int al = tb ? top64(tb) : l;
                const uint32_t spt = (uint32_t)shfl32((int)pt, al);
                const uint32_t aptr = tb ? spt : cur_ptr;
                const uint32_t aidx = tb ? (uint32_t)(a + w * 64 + al) : cur_idx;
                const bool ahas = tb != 0 || cur_has;
                if (((fm >> l) & 1) && ahas && pt == aptr && aidx < D.n)
                    g_or(&D.freed_bits[aidx >> 6], 1ull << (aidx & 63));
            } else if (fm && cur_has) {
                // (the usual case) every free compares with the active object
                if (((fm >> l) & 1) && pt == cur_ptr && cur_idx < D.n)
                    g_or(&D.freed_bits[cur_idx >> 6], 1ull << (cur_idx & 63));
            }
            if (tmask) {
                const int tl = top64(tmask);
                cur_ptr = (uint32_t)readlane32((int)pt, tl);
                cur_idx = (uint32_t)(a + w * 64 + tl);
                cur_has = true;
            }
            cnt += __popcll(m);
            staged += __popcll(m);
        }
        // the window's copy and timer events (validated as in the summary pass)
        if (has_aux) {
            const uint32_t kind = (fl >> 1) & 3u;
            const uint64_t r0 = ((uint64_t)in.q[w].y << 32) | in.q[w].x;
            const uint32_t line = in.q[w].w;
            const bool lok = k < nv && line < D.L;
            const bool cp = lok && kind == 1u && r0 < (uint64_t)MAX_ABS_DELTA;
            const bool tm = lok && kind == 2u && (r0 >> 32) == 0;
            uint64_t sampled = 0;  // bytes of the copy samples this event triggers
            if (csmp) {
                const int64_t dc = cp ? (int64_t)r0 : 0;
                const int64_t sc_ = wave_incl_sum(dc) + cc;
                cc = readlane64(sc_, 63);
                const uint64_t cout = (uint64_t)sc_, cin = cout - (uint64_t)dc;
                const uint64_t nsmp = D.tc_shift >= 0 ? (cout >> D.tc_shift) - (cin >> D.tc_shift)
                                                      : cout / (uint64_t)D.Tc - cin / (uint64_t)D.Tc;
                sampled = cp ? nsmp * (uint64_t)D.Tc : 0;
            }
            const uint64_t am = ballot(cp || tm);
            const int na = __popcll(am);
            if (na >= 32) {
                // a window of mostly such events keeps the lanes busy by
                // itself (300,000 events, nine copies in ten: 21.7 us staged,
                // 20.6 directly; 12 M: 142 and 138)
                if (cp || tm) count_aux(hc, D, (uint32_t)t, line, tm, r0, sampled);
            } else {
                if (sampled) count_copy_sample(hc, D, (uint32_t)t, line, sampled);
                if (aux + na > 64) {
                    flush_aux(D, (uint32_t)t, sg, aux, hc);
                    aux = 0;
                }
                if (cp || tm) {
                    const int at = aux + __popcll(am & lanemask_lt());
                    sg.ax[at] = tm ? r0 | 1ull << 63 : r0;
                    sg.aline[at] = line;
                }
                aux += na;
            }
        }
        // this window's registers take the next segment's window w (after
        // their last use here, so no copies and no early wait)
        if (hn) emit_load_record(record_addr(nbase, sn.nv, w), w, in);
    }
    if (staged) flush_stage(D, (uint32_t)t, stg, staged, stage_rank, hc);
    if (aux) flush_aux(D, (uint32_t)t, sg, aux, hc);
    if (err && l == 0) g_or32(&D.scal->err, err);
}

// The emit pass's two shapes: waves per workgroup, waves per SIMD, slots of
// the line tables.
//
// Wide, two workgroups per CU: a long single trace.  Its segments go to all
// workgroups alike, so each of them meets every line, and the tables want to
// be large.  Measured against four waves around one table of 128 slots with
// 12 counters, five workgroups per CU: 500 M events with copies and timers on
// 1 M lines 2.7-2.9 ms (4.1-4.3), 20 M on 100,000 lines 0.125 (0.25), 10 M
// without them 0.074 (0.075), 100 M without 0.55-0.57 (0.54-0.57, bound by
// the records).  16 waves, one workgroup per CU: 0.116 at 20 M, but
// 0.56-0.58 at 100 M and 3.05 ms at 500 M.  Ten waves (five per SIMD): 0.142
// and 0.62.
// Narrow, five workgroups per CU: batches, whose workgroups meet the lines of
// one or two traces, and short traces (see emit_wide).  1,024 traces of 1e3 to
// 1e6 events 1.35 ms (1.44) in one round of workgroups; 16 traces of 2 M events
// with copies on 100 lines 0.26, the wide shape 0.28; 2 of 10 M 0.18 and 0.19.
// Four workgroups per CU with 512 slots for samples: 1.2 ms for the 1,024
// traces, but 0.28-0.33 for the 16.
struct EmitWide { static constexpr int WAVES = 8, PER_SIMD = 4, SAMPLES = 512, AUX = 1024; };
struct EmitNarrow { static constexpr int WAVES = 4, PER_SIMD = 5, SAMPLES = 256, AUX = 256; };

template <class SHAPE>
__global__ __launch_bounds__(64 * SHAPE::WAVES) __attribute__((amdgpu_waves_per_eu(SHAPE::PER_SIMD))) void k_emit(
    const Desc* __restrict__ desc, int ntraces, uint64_t nseg_total, uint64_t* ts) {
    stamp(ts);
    constexpr int EMIT_WAVES = SHAPE::WAVES;
    __shared__ LineCaches<SHAPE> hc;
    __shared__ Staging stage[EMIT_WAVES];
    hc.smp.init();
    hc.aux.init();
    __syncthreads();
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
    // A batch of several traces: each workgroup takes one contiguous run of
    // segments (its waves interleaved in it), so that it sees the lines of
    // one or two traces and its line cache holds their hot lines; spread over
    // the grid, it would fill the cache with the first keys seen and send
    // nearly every later update to global atomics.  A single trace: segments
    // grid-stride (consecutive waves, consecutive segments), which streams
    // HBM faster than one run per workgroup.  Each wave loads its next
    // segment while it emits the current.
    uint64_t g, g_end, stride;
    if (ntraces > 1) {
        const uint64_t per = (nseg_total + (uint64_t)gridDim.x * EMIT_WAVES - 1) / ((uint64_t)gridDim.x * EMIT_WAVES);
        const uint64_t e0 = ((uint64_t)blockIdx.x + 1) * per * EMIT_WAVES;
        g = (uint64_t)blockIdx.x * per * EMIT_WAVES + wv;
        g_end = e0 < nseg_total ? e0 : nseg_total;
        stride = EMIT_WAVES;
    } else {
        g = (uint64_t)blockIdx.x * EMIT_WAVES + wv;
        g_end = nseg_total;
        stride = (uint64_t)gridDim.x * EMIT_WAVES;
    }
    if (g < g_end) {
        auto locate = [&](uint64_t x, int from) {
            EmitSeg r;
            r.t = __builtin_amdgcn_readfirstlane(find_trace_seg(desc, from, ntraces, x));
            r.j = (int64_t)(x - desc[r.t].seg_begin);
            r.nv = seg_events(desc[r.t], r.j);
            return r;
        };
        EmitSeg s = locate(g, 0);
        EmitIn in;
        emit_fetch_meta(desc[s.t], s.j, in);
        {
            gu8_t* base = (gu8_t*)(desc[s.t].ev + (size_t)(s.j * SEG) * 24);
#pragma unroll
            for (int w = 0; w < NW; ++w) emit_load_record(record_addr(base, s.nv, w), w, in);
        }
        for (;;) {
            const uint64_t gn = g + stride;
            const bool hn = gn < g_end;
            const EmitSeg sn = hn ? locate(gn, s.t) : s;
            emit_segment(desc, s, hc, stage[wv], in, hn, sn);
            if (!hn) break;
            g = gn;
            s = sn;
        }
    }
    __shared__ int held;
    static_assert(sizeof(stage) >= 2 * SHAPE::SAMPLES && sizeof(stage) >= 2 * SHAPE::AUX, "a list of slots");
    flush_lines(hc, desc, (uint16_t*)stage, &held);
}

// ----------------------------------------------------------------- clearing

__global__ void k_clear(const Desc* __restrict__ desc, int ntraces, uint64_t total_bytes, unsigned long long* ctl) {
    const uint64_t chunk = 1ull << 16;
    const uint64_t begin = (uint64_t)blockIdx.x * chunk;
    if (blockIdx.x == 0 && threadIdx.x < 32) gp(ctl)[threadIdx.x] = 0;
    if (begin >= total_bytes) return;
    const uint64_t end = begin + chunk < total_bytes ? begin + chunk : total_bytes;
    // traces overlapping [begin, end)
    int lo = 0, hi = ntraces - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (desc[mid].zero_begin <= begin) lo = mid; else hi = mid - 1;
    }
    for (int t = lo; t < ntraces; ++t) {
        const Desc& D = desc[t];
        if (D.zero_begin >= end) break;
        const uint64_t s = D.zero_begin > begin ? D.zero_begin : begin;
        const uint64_t e = (D.zero_begin + D.zero_bytes) < end ? (D.zero_begin + D.zero_bytes) : end;
        if (s >= e) continue;
        SMP_GLOBAL uint64_t* p = gp((uint64_t*)(D.zero_ptr + (s - D.zero_begin)));
        const uint64_t nw = (e - s) >> 3;
        for (uint64_t i = threadIdx.x; i < nw; i += blockDim.x) p[i] = 0;
    }
}

// ------------------------------------------------ tracked-list compaction

constexpr int CBLK_WORDS = 256;    // bitmap words per compaction block (one per thread)
constexpr int TRACK_UNROLL = 4;    // tracked entries per thread and trip of the fill

__device__ __forceinline__ int find_trace_blk(const Desc* desc, int ntraces, uint64_t x) {
    int lo = 0, hi = ntraces - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (desc[mid].blk_begin <= x) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Count before compaction block b of a trace's tracked bitmap, by a
// decoupled look-back over its earlier blocks (one wave; status words st:
// state 1 = a block's own count, 2 = the count through it).
__device__ bool count_lookback(const uint64_t* st, int64_t b, uint64_t& excl, unsigned long long* ctl) {
    const int l = lane_id();
    uint64_t acc = 0;
    int64_t base = b - 1;
    Spin sp;
    while (base >= 0) {
        const int64_t jj = base - l;
        const bool in = jj >= 0;
        const uint64_t w = in ? ld_status(st + (in ? jj : 0)) : 0;
        const uint32_t stt = wstate(w);
        const uint64_t incl = ballot(in && stt == 2);
        // lanes before the nearest inclusive word need their blocks' own counts
        const int lim = incl ? ctz64(incl) : 64;
        const uint64_t need = ballot(in && l < lim);
        if ((ballot(in && stt != 0) & need) != need) {
            if (spin_abort(ctl, sp)) return false;
            continue;
        }
        acc += (uint64_t)wave_sum(in && l <= lim && (l < lim || incl) ? unpack(w) : 0);
        if (incl) break;
        base -= 64;
    }
    excl = acc;
    return true;
}

// Ordered tracked list (the samples that set a new high-water mark, section
// 3.4) in one pass: the entries in rank order, each with the event, line and
// ptr_id of its sample and whether a free reclaimed it, and the per-line
// (mallocs, frees) counts.  Grid-stride over the compaction blocks of every
// trace's tracked bitmap (only the blocks that hold words below the trace's
// sample count do work), each workgroup taking its blocks in increasing
// order.  A block counts its set bits, publishes that count (status words in
// D.blk, cleared per launch), takes the count before it from a look-back
// over the trace's earlier blocks and writes its entries; the block holding
// the bitmap's last word writes H.  The grid never exceeds what the device
// holds at once, so every block a look-back waits on belongs to a running
// workgroup that reaches it in order.  Every reclaimed object is counted
// here; the last one of a trace (unresolved unless RESOLVE_AT_END) is taken
// back out by k_finish.
__global__ __launch_bounds__(256) void k_track(const Desc* __restrict__ desc, int ntraces, uint64_t nblk_total,
                                               unsigned long long* ctl, uint64_t* ts) {
    stamp(ts);
    __shared__ LineTable<TRACK_SLOTS, 2> hc;
    __shared__ uint64_t s_excl;
    __shared__ uint64_t w_cnt[4];
    hc.init();
    __syncthreads();
    const int tid = threadIdx.x, l = lane_id(), wv = tid >> 6;
    constexpr int PER = CBLK_WORDS / 256;  // each thread owns PER consecutive words
    for (uint64_t b = blockIdx.x; b < nblk_total; b += gridDim.x) {
        const uint32_t t = (uint32_t)find_trace_blk(desc, ntraces, b);
        const Desc& D = desc[t];
        const uint64_t lb = b - D.blk_begin;
        const uint64_t Kr = *gp(&D.scal->K);
        const uint64_t K = Kr < D.n ? Kr : D.n;
        const uint64_t nwords = (K + 63) >> 6;
        const uint64_t w0 = lb * CBLK_WORDS;
        if (w0 >= nwords) continue;  // (workgroup-uniform) no sample of this trace in the block
        uint64_t words[PER];
        uint64_t c = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const uint64_t wi = w0 + (uint64_t)tid * PER + i;
            words[i] = wi < nwords ? gp(D.tracked_bits)[wi] : 0;
            c += __popcll(words[i]);
        }
        const uint64_t ci = (uint64_t)wave_incl_sum((int64_t)c);
        if (l == 63) w_cnt[wv] = ci;
        __syncthreads();
        uint64_t woff = 0, total = 0;
        for (int w = 0; w < 4; ++w) {
            if (w < wv) woff += w_cnt[w];
            total += w_cnt[w];
        }
        uint64_t* st = D.blk;
        if (wv == 0) {
            uint64_t excl = 0;
            bool ok = true;
            if (lb == 0) {
                if (l == 0) st_status(st, pack((int64_t)total, 2));
            } else {
                if (l == 0) st_status(st + lb, pack((int64_t)total, 1));
                ok = count_lookback(st, (int64_t)lb, excl, ctl);
                if (l == 0) st_status(st + lb, pack((int64_t)(excl + total), 2));
            }
            if (l == 0) {
                s_excl = excl;
                if (!ok) g_or32(&D.scal->err, 8u);
            }
        }
        __syncthreads();
        const uint64_t h0 = s_excl, h1 = s_excl + total;
        if (tid == 0 && w0 + CBLK_WORDS >= nwords) *gp(&D.scal->H) = h1;
        // First the sample rank of each entry (tracked samples cluster, so a
        // thread may own many), then the entries, spread over all threads.
        uint64_t h = h0 + woff + ci - c;
        SMP_GLOBAL uint32_t* tq = (SMP_GLOBAL uint32_t*)D.tracked;
        for (int i = 0; i < PER; ++i) {
            uint64_t m = words[i];
            const uint64_t wi = w0 + (uint64_t)tid * PER + i;
            while (m) {
                const int bit = __builtin_ctzll(m);
                m &= m - 1;
                const uint64_t r = wi * 64 + bit;
                tq[4 * h] = r < K ? (uint32_t)r : 0xFFFFFFFFu;  // (r >= K only after an internal fault)
                ++h;
            }
        }
        __syncthreads();
        // TRACK_UNROLL entries per thread and trip, each step's loads issued
        // for all of them before the first is used: a block may hold many
        // thousands of entries, and one at a time its three dependent loads
        // (rank, sample, freed bit) would each cost a full round trip.
        for (uint64_t hb = h0 + tid; hb < h1; hb += 256 * TRACK_UNROLL) {
            uint32_t r[TRACK_UNROLL], ptr[TRACK_UNROLL];
            uint64_t sw[TRACK_UNROLL], fw[TRACK_UNROLL];
#pragma unroll
            for (int u = 0; u < TRACK_UNROLL; ++u) {
                const uint64_t hh = hb + 256 * (uint64_t)u;
                r[u] = hh < h1 ? tq[4 * hh] : 0xFFFFFFFFu;
            }
#pragma unroll
            for (int u = 0; u < TRACK_UNROLL; ++u) {
                const uint32_t rr = r[u] < K ? r[u] : 0u;
                sw[u] = *(const SMP_GLOBAL uint64_t*)(D.samples + rr);  // event index, line
                ptr[u] = gp(D.sample_ptr)[rr];
            }
#pragma unroll
            for (int u = 0; u < TRACK_UNROLL; ++u) {
                const uint32_t ev = (uint32_t)sw[u];
                fw[u] = r[u] < K && ev < D.n ? gp(D.freed_bits)[ev >> 6] : 0;
            }
#pragma unroll
            for (int u = 0; u < TRACK_UNROLL; ++u) {
                if (r[u] >= K) continue;  // (past the block's entries, or after an internal fault)
                const uint64_t hh = hb + 256 * (uint64_t)u;
                const uint32_t ev = (uint32_t)sw[u], line = (uint32_t)(sw[u] >> 32);
                const uint32_t freed = (uint32_t)((fw[u] >> (ev & 63)) & 1);
                tq[4 * hh] = ev;
                tq[4 * hh + 1] = line;
                tq[4 * hh + 2] = ptr[u];
                tq[4 * hh + 3] = freed;
                if (line < D.L) count_tracked(hc, D, t, line, freed);
            }
        }
        __syncthreads();  // w_cnt and s_excl are reused by the next block
    }
    __syncthreads();
    flush_table(hc, [&](uint32_t t, uint32_t line, int i) {
        const Desc& D = desc[t];
        hist_global(D, H_LEAK_M, line, hc.v[LK_M][i]);
        hist_global(D, H_LEAK_F, line, hc.v[LK_F][i]);
    });
}

// ------------------------------------------------ leak likelihood per line

__device__ int64_t gcd64(int64_t x, int64_t y) {
    if (x < 0) x = -x;
    while (y) {
        const int64_t r = x % y;
        x = y;
        y = r;
    }
    return x;
}

// After the tracked list: per line, exact reduced rationals of the leak
// likelihood (section 3.4) - Laplace's rule of succession (m-f+1)/(m+2) and
// the formula as printed (m-2f+1)/(m-f+2) - and their gates, likelihood >
// 0.95.  The last tracked object of a trace stays unresolved (its free does
// not count) unless RESOLVE_AT_END, so the thread of its line takes it back
// out of that line's frees.  Threads below 8 x ntraces also gather every
// trace's scalars (final from here on) into one array, which may live in
// pinned host memory (the host reads it once the launch has completed).
__global__ void k_finish(const Desc* __restrict__ desc, int ntraces, uint64_t total_lines, Scalars* gather,
                         uint64_t* ts) {
    stamp(ts);
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < (uint64_t)ntraces * 8) {
        const uint64_t t = i >> 3, w = i & 7;  // 8 words per Scalars
        gp((uint64_t*)(gather + t))[w] = gp((const uint64_t*)desc[t].scal)[w];
    }
    if (i >= total_lines) return;
    int lo = 0, hi = ntraces - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (desc[mid].line_begin <= i) lo = mid; else hi = mid - 1;
    }
    const Desc& D = desc[lo];
    const uint64_t line = i - D.line_begin;
    if (line >= D.L) return;
    SMP_GLOBAL int64_t* hist = gp(D.hist);
    const int64_t m = hist[(size_t)H_LEAK_M * D.L + line];
    int64_t f = hist[(size_t)H_LEAK_F * D.L + line];
    if (m > 0 && (D.options & 2u) == 0) {
        const uint64_t H = *gp(&D.scal->H);
        if (H > 0) {
            const SMP_GLOBAL uint32_t* last = (const SMP_GLOBAL uint32_t*)(D.tracked + (H - 1));
            if (last[1] == (uint32_t)line && last[3] != 0) {
                f -= 1;
                hist[(size_t)H_LEAK_F * D.L + line] = f;
            }
        }
    }
    SMP_GLOBAL int64_t* out = gp(D.leak);
    SMP_GLOBAL uint8_t* gates = gp(D.gates);
    if (m <= 0) {
        out[line] = 0;
        out[D.L + line] = 0;
        out[2 * (size_t)D.L + line] = 0;
        out[3 * (size_t)D.L + line] = 0;
        gates[line] = 0;
        gates[D.L + line] = 0;
        return;
    }
    int64_t n1 = m - f + 1, d1 = m + 2;
    int64_t n2 = m - 2 * f + 1, d2 = m - f + 2;
    const uint8_t g1 = 20 * n1 > 19 * d1;
    const uint8_t g2 = 20 * n2 > 19 * d2;
    if (n1 == 0) { d1 = 1; } else { const int64_t g = gcd64(n1, d1); n1 /= g; d1 /= g; }
    if (n2 == 0) { d2 = 1; } else { const int64_t g = gcd64(n2, d2); n2 /= g; d2 /= g; }
    out[line] = n1;
    out[D.L + line] = d1;
    out[2 * (size_t)D.L + line] = n2;
    out[3 * (size_t)D.L + line] = d2;
    gates[line] = g1;
    gates[D.L + line] = g2;
}

// ---------------------------------------------------------------- copy out

// A finished trace's results into pinned host memory, up to three ranges one
// behind another (offsets and lengths in 8-byte words): one launch and one
// wait in place of a blocking copy per array.
__global__ __launch_bounds__(256) void k_copy_out(CopyOut c, uint64_t* dst) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
#pragma unroll
    for (int r = 0; r < 3; ++r)
        for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < c.words[r]; i += stride)
            gp(dst)[c.at[r] + i] = gp(c.src[r])[i];
}

// ------------------------------------------------------------ launchers

static int occupancy_grid(const void* fn, int block) {
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, block, 0) != hipSuccess) return 0;
    return cus * (per > 0 ? per : 1);
}

int chain_grid_limit() { return occupancy_grid((const void*)k_chain, BLOCK); }
int emit_grid_limit(bool wide) {
    return wide ? occupancy_grid((const void*)k_emit<EmitWide>, 64 * EmitWide::WAVES)
                : occupancy_grid((const void*)k_emit<EmitNarrow>, 64 * EmitNarrow::WAVES);
}
// workgroups of k_track the device holds at once (its look-back needs all of them resident)
int track_grid_limit() { return occupancy_grid((const void*)k_track, 256); }

hipError_t launch_copy_out(const CopyOut& c, uint64_t* dst, hipStream_t s) {
    uint64_t most = 1;
    for (uint64_t w : c.words) most = w > most ? w : most;
    const uint64_t blocks = (most + 511) / 512;
    k_copy_out<<<dim3((unsigned)(blocks < 256 ? blocks : 256)), dim3(256), 0, s>>>(c, dst);
    return hipGetLastError();
}

hipError_t launch_clear(const Desc* desc, int ntraces, uint64_t total_bytes, unsigned long long* ctl, hipStream_t s) {
    const uint64_t blocks = (total_bytes + (1ull << 16) - 1) >> 16;
    k_clear<<<dim3((unsigned)(blocks ? blocks : 1)), dim3(256), 0, s>>>(desc, ntraces, total_bytes, ctl);
    return hipGetLastError();
}

hipError_t launch_tmap(const Desc* desc, int ntraces, uint64_t ntile_total, unsigned long long* ctl, uint64_t* ts,
                       hipStream_t s) {
    if (ntile_total == 0) return hipSuccess;
    k_tmap<<<dim3((unsigned)ntile_total), dim3(TILE), 0, s>>>(desc, ntraces, ctl, ts);
    return hipGetLastError();
}

hipError_t launch_pass(int pass, const Desc* desc, int ntraces, uint64_t nseg_total, uint64_t ntile_total,
                       unsigned long long* ctl, int grid_limit, uint64_t* ts, hipStream_t s) {
    if (nseg_total == 0) return hipSuccess;
    const uint64_t wgs = (nseg_total + WAVES - 1) / WAVES;
    const unsigned pgrid = (unsigned)(wgs < (uint64_t)grid_limit ? wgs : (uint64_t)grid_limit);
    switch (pass) {
        case 0: k_summarize<<<dim3((unsigned)wgs), dim3(BLOCK), 0, s>>>(desc, ntraces, nseg_total, ts); break;
        case 1: k_resolve<<<dim3((unsigned)ntile_total), dim3(TILE), 0, s>>>(desc, ntraces, ntile_total, ctl, ts); break;
        case 2: k_chain<<<dim3(pgrid), dim3(BLOCK), 0, s>>>(desc, ntraces, nseg_total, ts); break;
        case 3: k_bscan<<<dim3((unsigned)ntile_total), dim3(TILE), 0, s>>>(desc, ntraces, ntile_total, ctl, ts); break;
        default: {
            const bool wide = emit_wide(ntraces, nseg_total);
            const uint64_t ew = wide ? EmitWide::WAVES : EmitNarrow::WAVES;
            const uint64_t ewgs = (nseg_total + ew - 1) / ew;
            const dim3 egrid((unsigned)(ewgs < (uint64_t)grid_limit ? ewgs : (uint64_t)grid_limit)), eblock(64 * (unsigned)ew);
            if (wide)
                k_emit<EmitWide><<<egrid, eblock, 0, s>>>(desc, ntraces, nseg_total, ts);
            else
                k_emit<EmitNarrow><<<egrid, eblock, 0, s>>>(desc, ntraces, nseg_total, ts);
            break;
        }
    }
    return hipGetLastError();
}

hipError_t launch_finish(const Desc* desc, int ntraces, uint64_t nblk_total, uint64_t total_lines,
                         unsigned long long* ctl, int track_grid, Scalars* gather, uint64_t* ts, hipStream_t s) {
    if (nblk_total) {
        const unsigned g = (unsigned)(nblk_total < (uint64_t)track_grid ? nblk_total : (uint64_t)track_grid);
        k_track<<<dim3(g), dim3(256), 0, s>>>(desc, ntraces, nblk_total, ctl, ts);
        ts = nullptr;
    }
    const uint64_t items = total_lines > (uint64_t)ntraces * 8 ? total_lines : (uint64_t)ntraces * 8;
    k_finish<<<dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s>>>(desc, ntraces, total_lines, gather, ts);
    return hipGetLastError();
}

}  // namespace smp
