// Load-aware request router (Sec. 3.4.3): score every instance for each request of a micro-batch and
// dispatch to the smallest score,
//     100 L_i = 100 (queued_p_i + P + current_d_i + D) + beta * max(0, 100 peak_i - T_pct M_i),
// peak_i = the largest value, over the next `window` iterations, of instance i's look-ahead map with
// the request virtually added (P + t tokens at iteration t < D).  Decisions are sequential by
// definition (a dispatched request changes its instance's queue and map for the next one), so one
// workgroup walks the micro-batch with all state on chip.  Integer arithmetic throughout: the
// decisions are exact.
//
// The walk is a chain of dependent decisions, so what counts is the latency of one of them.  Scanning an
// instance's window for every request is most of that, and is not needed: with D' = min(D, window),
//     peak = max(P + max_{t < D'} (w[t] + t),  max_{t >= D'} w[t]),
// a prefix maximum and a suffix maximum that change only for the instance a request is dispatched to.
// They are kept per block of the window (at most 32 blocks: at window 100 the blocks are 4 slots), so a score
// reads one prefix, one suffix and the one block that D' falls into (8 or 16 slots where the tables of smaller ones would
// not fit).  One thread per instance scores it; the wavefront that owns the chosen instance adds the request to its
// window with one lane per piece of four slots (per block, where the window has more than 32 pieces: 2048 requests over
// 256 instances of 128 slots 3.17 ms by blocks and with scores in 64 bits, 1.25 by pieces and in one register) and rebuilds
// both rows of maxima with one scan (prefixes in lanes 0..31, suffixes, in reverse order, in lanes 32..63),
// while the other wavefronts are already at the next request.  An instance's state is touched by its own
// wavefront only, so the exchange of the wavefronts' minima is the one barrier of a request; up to 64
// instances need none.
// A decision is some 150 instructions of one wavefront after the other (no more than one to a SIMD is at work), so their
// number counts as well: where a bound on queues and windows allows, scores are made in one register (walk_narrow).
// 4096 requests over 256 instances with windows of 100: 13.0 ms when four threads per instance scanned the
// window in registers for every request, 3.09 ms from the tables with scores in 64 bits, 2.05 in one register (1.27 by one
// wavefront over windows that fall towards their end, solo_walk); 64 instances 2.06 and 1.46.  Scoring a request ahead and putting
// the last chosen instance's score right afterwards: 3.67.
#include <type_traits>

#include "device_util.h"
#include "internal.h"

namespace {

const int kRouteThreads = 1024;
const int kRouteLdsBytes = 160 * 1024;       // all of a compute unit's LDS
const int kRouteMaxBlocks = 32;              // blocks of a window: one lane each in either half of the update's scan

// How the windows lie in LDS: 16-byte pieces of four consecutive slots, [piece][instance], `pitch` instances apart
// (odd where that fits, so that one instance's pieces fall in different banks); behind them the two tables of
// block maxima, [block][instance].
struct RoutePlan {
    int block;                               // slots per block, a multiple of 4
    int n_blocks, pitch;
    size_t lds_bytes;
};

RoutePlan plan_route(int n_inst, int window) {
    RoutePlan p;
    const int whole = (window + 3) / 4 * 4;
    for (int block = 4 * ((window + 4 * kRouteMaxBlocks - 1) / (4 * kRouteMaxBlocks));; block *= 2) {
        if (block > whole) block = whole;
        p.block = block;
        p.n_blocks = window > 0 ? (window + block - 1) / block : 0;
        // small blocks make the cheapest scores; larger ones, and at last the plain pitch and a single block, are
        // for maps that fill the LDS
        for (int odd = 1; odd >= 0; --odd) {
            p.pitch = odd ? n_inst | 1 : n_inst;
            p.lds_bytes = 512 + (size_t)p.pitch * 4 * ((size_t)p.n_blocks * block + 2 * (size_t)(p.n_blocks + 1));
            if (p.lds_bytes <= (size_t)kRouteLdsBytes) return p;
        }
        if (block == whole) return p;
    }
}

// DPP moves with the operation's identity where no lane is read, so that they fold into the operation.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_max(int v) {
    return max(v, __builtin_amdgcn_update_dpp((int)0x80000000, v, CTRL, ROWS, 0xf, false));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_min(int v) {
    return min(v, __builtin_amdgcn_update_dpp(0x7fffffff, v, CTRL, ROWS, 0xf, false));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ long long dpp_min64(long long v) {
    const int lo = (int)v, hi = (int)(v >> 32);
    const int olo = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false);
    const int ohi = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false);
    const long long o = ((long long)ohi << 32) | (unsigned)olo;
    return o < v ? o : v;
}
// Minimum of v over the wavefront (lanes that take no part hold 2^63 - 1) and the lowest lane that has it.  Scores
// hardly ever leave 32 bits (that takes 2^31 / 100 tokens on one instance): then the minimum is taken in one
// register, else in two.
__device__ __forceinline__ long long wave_min(long long v, bool part, int& src) {
    const int lo = (int)v;
    if (!__any(part && (int)(v >> 32) != (lo >> 31))) {
        const int x = part ? lo : 0x7fffffff;
        int m = dpp_min<0x111, 0xf>(x);          // row_shr 1, 2, 4, 8: lane 15 of a row has the row's minimum
        m = dpp_min<0x112, 0xf>(m);
        m = dpp_min<0x114, 0xf>(m);
        m = dpp_min<0x118, 0xf>(m);
        m = dpp_min<0x142, 0xa>(m);              // row_bcast 15 into rows 1 and 3
        m = dpp_min<0x143, 0xc>(m);              // row_bcast 31 into rows 2 and 3: lane 63 has it
        m = __builtin_amdgcn_readlane(m, 63);
        src = __builtin_ctzll(__ballot(x == m)); // (some lane holds it)
        return m;
    }
    long long m = dpp_min64<0x111, 0xf>(v);
    m = dpp_min64<0x112, 0xf>(m);
    m = dpp_min64<0x114, 0xf>(m);
    m = dpp_min64<0x118, 0xf>(m);
    m = dpp_min64<0x142, 0xa>(m);
    m = dpp_min64<0x143, 0xc>(m);
    const unsigned mlo = (unsigned)__builtin_amdgcn_readlane((int)m, 63);
    m = ((long long)__builtin_amdgcn_readlane((int)(m >> 32), 63) << 32) | mlo;
    src = __builtin_ctzll(__ballot(v == m));
    return m;
}

// ---- one wavefront walks the requests -----------------------------------------------------------------------------
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned dpp_umax(unsigned v) {
    return max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ unsigned wave_umax(unsigned m) {
    m = dpp_umax<0x111, 0xf>(m);
    m = dpp_umax<0x112, 0xf>(m);
    m = dpp_umax<0x114, 0xf>(m);
    m = dpp_umax<0x118, 0xf>(m);
    m = dpp_umax<0x142, 0xa>(m);
    m = dpp_umax<0x143, 0xc>(m);
    return (unsigned)__builtin_amdgcn_readlane((int)m, 63);
}
__device__ __forceinline__ int wave_total(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return __builtin_amdgcn_readlane(v, 63);
}

// What the walk needs to know: peaks below 2^24, penalties and the rest of a score below 2^29.
__device__ __forceinline__ bool peaks_fit(long long peak, int beta) { return peak < 1 << 24 && peak * 100 * max(beta, 1) < 1 << 29; }

// The exchange between wavefronts costs a request as much as its scores do, and the tables are made for requests that end
// anywhere in any window.  So wavefront 0 walks the requests, R instances a lane, with an instance's window in a few numbers:
// F = max (w[t] + t), the first slot t* that has it, and the largest w.  A request whose ramp reaches beyond t* has the
// peak P + F exactly (no slot behind the ramp is above F), and with p = beta (100 F - limit) a score is
//     s + max(p + 100 beta P, 0),  s the queue a hundredfold.
// For a ramp that ends before, the largest w gives a lower bound, and where an instance with such a bound has the smallest
// score its window is read, once, for this request.  The other wavefronts add the requests of a batch to the windows and make
// the numbers afresh while the next batch is walked; until then an instance's old numbers are a lower bound (windows only grow),
// and F is less than P + D' above the old one, which keeps most instances below their limit: only where it does not, and the
// instance is the choice again already, the walk waits for them.  A decision is some 110 instructions of one wavefront and no
// exchange.
//
// What it gains is for the windows to say.  Microseconds, the tables alone / with this walk in front of them, 4096 requests over
// instances x slots, windows that fall by half towards their end (as requests finish) | all slots near the limit | slots each on
// their own, around the limits | windows that rise to their limits:
//   65 x 100    2035 / 1146 | 2050 / 2050 | 2036 / 2036 | 2006 / 1864        256 x 100  2048 / 1272 | 2050 / 2050 | 2047 / 2054 | 2049 / 2055
//   128 x 64    2031 /  977 | 2035 / 2034 | 2028 / 1893 | 2032 / 1499        256 x 128  2513 / 1307 | 2517 / 2498 | 2512 / 2498 | 2512 / 2496
//   300 x 60    2202 / 1806 | 2239 / 2238 | 2198 / 2207 | 2237 / 2244        500 x 60   2890 / 1750 | 2892 / 2864 | 2886 / 2853 | 2886 / 2859
// Windows whose largest w[t] + t lies at t* anywhere are the bad ones: most ramps end before, and each such request looks at windows
// one after the other (256 x 100: 2800 us near the limit, 2680 on their own, as long as nothing stopped it).  So where most instances
// are at their limits behind their first slot the walk does not begin, and it keeps account of its costs (solo_saves).  Short calls:
// 32 requests over 256 x 100 34.8 / 29.5 falling, 35.0 near the limit, 36.1 on their own; 64 50.2 / 38.8, 50.5, 51.0; 256 x 100 of
// 12, where nothing is gained, 25.1 / 25.2 to 26.5.  257 to 384 instances, whose tables cost less: 64 requests over 300 48.2 / 42.1
// falling, but 57.3 on their own, 256 151 / 122 and 160.  Up to 64 instances a walk with the tables has no exchange either, and waits
// would be frequent (20 instances 739 -> 820, 64 1470 -> 1280 to 1440): left to it.
const int kSoloInstances = 512;              // eight a lane
inline int solo_least_requests(int n_inst) { return n_inst > 256 && n_inst <= 384 ? 256 : 32; }
const int kSoloTokens = 1 << 20;             // prompts and predictions from here on are not walked
const int kSoloWaves = 8;
const int kSoloBatch = 16;
// Which requests leave the short way is for the windows and the requests to say, so the walk keeps account of what it saves
// against the tables and of what it pays, and leaves the rest of the call to them where the costs pass the savings.  Cycles by
// regression over groups of 64 requests, two / four / eight instances a lane: a request 570 / 700 / 970, by the tables 1190 / 1200 /
// 1290 to 1690; one off the short way 705 / 850 / 1220 more, a window read 690 / 870 / 1110, a wait 2400 / 2700 / 3400.  In eighths
// of a window read: what a request saves, what a read or a request off the short way costs and a wait, how far costs may run ahead
// of savings, and savings count on.
template <int R>
__device__ __forceinline__ int solo_saves(int n_inst) { return R == 2 ? 6 : R == 4 ? 4 : n_inst <= 384 ? 2 : 3; }
const int kSoloUnit = 8, kSoloWait = 26, kSoloSlack = 32, kSoloMost = 128;
struct SoloWalk {
    const int32_t* prompt_tokens;
    const int32_t* pred_tokens;
    int n_req, n_inst, window, pitch, beta;
    int* win;                                // s_win
    int lanes_log2;                          // of R: instance i is number i % R of lane i / R
    int4* state;                             // [R][64] p; t*; p with the largest w for F; limit.  At the end, x: s
    int* added;                              // [n_inst] s, then prompt tokens added
    unsigned char* lists;                    // [2] of kSoloList: a batch's choices, and whether it was the last
    int32_t* assigned;
    int64_t* score100;
    ps_status* st;
};
const int kSoloList = 64 * 8 + 16;           // int2 a request: instance + ramp * 2^16 (or -1), prompt
size_t solo_lds_bytes(int n_inst) {
    int lanes = 1;                           // R
    while (64 * lanes < n_inst) lanes *= 2;
    return (size_t)lanes * 1024 + 16 + 2 * kSoloList + (size_t)n_inst * 4;
}

// beta v, from -2^29 on: no request walked makes more than that of it.
__device__ __forceinline__ int solo_penalty(int v, int beta) { return beta * max(v, -(1 << 29) / max(beta, 1)); }

__device__ __forceinline__ int solo_at_state(const SoloWalk& a, int i) { return (i & ((1 << a.lanes_log2) - 1)) * 64 + (i >> a.lanes_log2); }

// An instance's numbers: the largest w[t] + t, the first t that has it, the largest w; the largest ones from 0 on.
__device__ __forceinline__ int4 solo_numbers(int f, int t, int most, int lim, int beta) {
    return make_int4(solo_penalty(100 * f - lim, beta), t, solo_penalty(100 * most - lim, beta), lim);
}

struct SoloSlots {                           // a lane's two slots of a window
    int t0, t1;
    bool live0, live1;
    int *w0, *w1;
    __device__ __forceinline__ SoloSlots(const SoloWalk& a, int lane) {
        t0 = lane;
        t1 = lane + 64;
        live0 = t0 < a.window;
        live1 = t1 < a.window;
        w0 = a.win + ((live0 ? t0 >> 2 : 0) * a.pitch * 4 + (t0 & 3));
        w1 = a.win + ((live1 ? t1 >> 2 : 0) * a.pitch * 4 + (t1 & 3));
    }
};

// The requests of a list go to their windows, and the instances' numbers are made afresh: wavefronts 1 to 7, an instance always
// by the same one.
__device__ __forceinline__ void solo_apply(const SoloWalk& a, const SoloSlots& sl, const unsigned char* list, int wave) {
    const int lane = threadIdx.x & 63;
    const int2 d = ((const int2*)list)[lane];
    for (unsigned long long mask = __ballot(d.x >= 0 && (d.x & 0xffff) % (kSoloWaves - 1) == wave - 1); mask; mask &= mask - 1) {
        const int q = __builtin_ctzll(mask), x = __builtin_amdgcn_readlane(d.x, q), P = __builtin_amdgcn_readlane(d.y, q);
        const int i = x & 0xffff, Dc = x >> 16;
        int4* const state = a.state + solo_at_state(a, i);
        const int lim = state->w;
        const int v0 = sl.w0[4 * i] + (sl.t0 < Dc ? P + sl.t0 : 0), v1 = sl.w1[4 * i] + (sl.t1 < Dc ? P + sl.t1 : 0);
        if (sl.t0 < Dc) sl.w0[4 * i] = v0;
        if (sl.t1 < Dc) sl.w1[4 * i] = v1;
        // F * 256 + 255 - t: the largest has the first slot of the largest sum; 0 where all sums are below 0
        const unsigned k0 = sl.live0 && v0 + sl.t0 >= 0 ? ((unsigned)(v0 + sl.t0) << 8) + 255 - sl.t0 : 0;
        const unsigned k1 = sl.live1 && v1 + sl.t1 >= 0 ? ((unsigned)(v1 + sl.t1) << 8) + 255 - sl.t1 : 0;
        const unsigned k = wave_umax(max(k0, k1));
        const int most = (int)wave_umax((unsigned)max(max(sl.live0 ? v0 : 0, sl.live1 ? v1 : 0), 0));
        if (lane == 0) *state = solo_numbers((int)(k >> 8), k ? 255 - (int)(k & 255) : a.window, most, lim, a.beta);
        asm volatile("" ::: "memory");                           // (in order: the next one may be of the same instance)
    }
}

// Wavefront 0's part; the others are in solo_follow.  Returns the first request not walked.
template <int R>
__device__ __forceinline__ int solo_walk(const SoloWalk& a, long long bound, long long load_bound) {
    const int lane = threadIdx.x, window = a.window, beta = a.beta, beta100 = 100 * beta, saves = solo_saves<R>(a.n_inst);
    const SoloSlots sl(a, lane);
    // score; its penalty at P = 0; an upper bound of that, above it where the penalty is an old one; t*; as its name
    int s[R], p[R], u[R], top[R], low[R], id[R];
    int cur = 0;                             // bit j: the list being made has instance j
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int i = lane * R + j;
        id[j] = i;
        s[j] = 1 << 30;
        p[j] = u[j] = -(1 << 29);
        top[j] = low[j] = 0;
        if (i < a.n_inst) {
            s[j] = a.added[i];
            a.added[i] = 0;
        }
    }
    int base = 0, nP = 0, nD = 0;
    if (lane < a.n_req) { nP = a.prompt_tokens[lane]; nD = a.pred_tokens[lane]; }
    bool quit = false, drain = false, last = false;
    int vP = 0, vDc = 0, v_add = 0, cnt = 0, most = 0, credit = 0, out_i = -1, out_s = 0, buffer = 0;
    unsigned long long todo = 0, part = 0;   // of the group: requests to walk; the batch at hand
    bool open = false;                       // a group is being walked
    for (;;) {
        // ---- the numbers as the lists before the last one left them ----
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int i = lane * R + j;
            if (i < a.n_inst && !drain && !(cur >> j & 1)) {     // (not while it only waits)
                const int4 v = a.state[64 * j + lane];
                p[j] = u[j] = v.x;
                top[j] = v.y;
                low[j] = v.z;
            }
        }
        cur = 0;
        // ---- the next group ----
        if (!open && base < a.n_req && !quit) {
            cnt = min(64, a.n_req - base);
            vP = nP;
            int vD = nD;
            if (base + 64 + lane < a.n_req) { nP = a.prompt_tokens[base + 64 + lane]; nD = a.pred_tokens[base + 64 + lane]; }
            const bool good = lane < cnt && vP >= 0 && vD >= 0;
            if (!__ballot(good && (vP >= kSoloTokens || vD >= kSoloTokens))) {
                const int sum_p = wave_total(good ? vP : 0), sum_d = wave_total(good ? vD : 0);
                const long long rise = sum_p + 64ll * window, load_rise = 100ll * ((long long)sum_p + sum_d);
                if (peaks_fit(bound + rise, beta) && load_bound + load_rise < 1 << 29) {
                    bound += rise;
                    load_bound += load_rise;
                    if (lane < cnt && !good) report_fault(a.st, PS_ST_BAD_RECORD, base + lane);
                    vDc = min(vD, window);
                    v_add = 100 * (vP + vD);
                    most = (int)wave_umax(good ? (unsigned)vP : 0);
                    out_i = -1;
                    out_s = 0;
                    todo = __ballot(good);
                    part = (1ull << kSoloBatch) - 1;
                    open = true;
                }
            }
        }
        last = !open;
        const unsigned long long before = todo;
        if (!drain && todo) {
            // ramps beyond `reach` pass t* of every instance that may be above its limit
            int reach = 0;
#pragma unroll
            for (int j = 0; j < R; ++j) reach = p[j] + beta100 * most > 0 ? max(reach, top[j]) : reach;
            reach = (int)wave_umax((unsigned)reach);
            while (!(todo & part)) part <<= kSoloBatch;
            unsigned long long now = todo & part;
            const unsigned long long all = now;
            int L[R], best, src, at, sure;                       // smallest score, its lane (the lowest), its place there
            auto smallest = [&](int pb) {
                int own = L[0];
#pragma unroll
                for (int j = 1; j < R; ++j) own = min(own, L[j]);
                int m = dpp_min<0x111, 0xf>(own);                // as in wave_min
                m = dpp_min<0x112, 0xf>(m);
                m = dpp_min<0x114, 0xf>(m);
                m = dpp_min<0x118, 0xf>(m);
                m = dpp_min<0x142, 0xa>(m);
                m = dpp_min<0x143, 0xc>(m);
                int place = R - 1, up = u[R - 1], pen = p[R - 1];
#pragma unroll
                for (int j = R - 2; j >= 0; --j) {
                    const bool here = L[j] == own;
                    place = here ? j : place;
                    up = here ? u[j] : up;
                    pen = here ? p[j] : pen;
                }
                // an old penalty is a new one as long as neither passes the limit; bit 0: to be trusted, above it: place
                place = place * 2 + (up == pen || up + pb <= 0);
                best = __builtin_amdgcn_readlane(m, 63);
                src = __builtin_ctzll(__ballot(own == best));
                at = __builtin_amdgcn_readlane(place, src);
                sure = at & 1;
                at >>= 1;
            };
            auto commit = [&](int q, int add, int lift) {
                const int i = src * R + at;
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    const bool hit = id[j] == i;
                    s[j] += hit ? add : 0;
                    u[j] += hit ? lift : 0;
                }
                cur |= lane == src ? 1 << at : 0;
                const bool rec = lane == q;
                out_i = rec ? i : out_i;
                out_s = rec ? best + add : out_s;
            };
            do {
                int q;
                // one way through, with one branch out of it: a taken branch costs as much as five instructions
                for (;;) {
                    q = __builtin_ctzll(now);
                    const int P = __builtin_amdgcn_readlane(vP, q), Dc = __builtin_amdgcn_readlane(vDc, q);
                    const int add = __builtin_amdgcn_readlane(v_add, q), pb = beta100 * P;
#pragma unroll
                    for (int j = 0; j < R; ++j) L[j] = s[j] + max(p[j] + pb, 0);
                    smallest(pb);
                    if (__builtin_expect((Dc <= reach) | (sure == 0), 0)) break;
                    commit(q, add, pb + beta100 * Dc);
                    now &= now - 1;
                    if (!now) break;
                }
                if (!now) break;
                // a ramp that ends before some t*, or an instance whose numbers are not made yet
                const int P = __builtin_amdgcn_readlane(vP, q), Dc = __builtin_amdgcn_readlane(vDc, q);
                const int add = __builtin_amdgcn_readlane(v_add, q), pb = beta100 * P;
                credit -= kSoloUnit;
#pragma unroll
                for (int j = 0; j < R; ++j) L[j] = s[j] + max(top[j] < Dc ? p[j] + pb : low[j], 0);
                unsigned seen = 0;                               // the lane's instances whose window has been read
                for (;;) {
                    smallest(pb);
                    const int i = src * R + at;
                    bool bound_only = false;
#pragma unroll
                    for (int j = 0; j < R; ++j)
                        bound_only |= id[j] == i && top[j] >= Dc && p[j] + pb > 0 && !(seen >> j & 1);
                    if (!sure || !__ballot(bound_only)) break;
                    int pk = 0;                                  // (a peak below 0 is no more over a limit than one of 0)
                    if (sl.live0) pk = max(pk, sl.w0[4 * i] + (sl.t0 < Dc ? P + sl.t0 : 0));
                    if (sl.live1) pk = max(pk, sl.w1[4 * i] + (sl.t1 < Dc ? P + sl.t1 : 0));
                    pk = (int)wave_umax((unsigned)pk);
                    const int over = beta * max(100 * pk - a.state[64 * at + src].w, 0);
#pragma unroll
                    for (int j = 0; j < R; ++j) {
                        L[j] = id[j] == i ? s[j] + over : L[j];
                        seen |= id[j] == i ? 1u << j : 0u;
                    }
                    credit -= kSoloUnit;
                }
                if (!sure) {
                    drain = true;
                    credit -= kSoloWait;
                    break;
                }
                commit(q, add, pb + beta100 * Dc);
                now &= now - 1;
                quit = credit + saves * (int)__popcll(all ^ now) < -kSoloSlack;
            } while (now && !quit);
            credit = min(credit + saves * (int)__popcll(all ^ now), kSoloMost);
            quit |= credit < -kSoloSlack;
            todo = (todo & ~part) | now;
        } else {
            drain = false;
        }
        // ---- the batch's choices to the other wavefronts ----
        unsigned char* const list = a.lists + buffer * kSoloList;
        const bool done = (before & ~todo) >> lane & 1;
        ((int2*)list)[lane] = make_int2(done && vDc > 0 ? out_i | vDc << 16 : -1, vP);
        if (lane == 0) *(int*)(list + 64 * 8) = last;
        buffer ^= 1;
        if (open && (!todo || quit)) {                           // (a group left half walked goes on with the tables)
            if (todo) cnt = __builtin_ctzll(todo);
            if (out_i >= 0) atomicAdd(a.added + out_i, vP);
            if (lane < cnt) {
                a.assigned[base + lane] = out_i;
                a.score100[base + lane] = out_s;
            }
            base += cnt;
            todo = 0;
            open = false;
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (last) break;
    }
    // (the last list is empty, the one before it has been applied)
#pragma unroll
    for (int j = 0; j < R; ++j)
        if (lane * R + j < a.n_inst) a.state[64 * j + lane].x = s[j];
    return base;
}
__device__ __forceinline__ void solo_follow(const SoloWalk& a, int wave) {
    const SoloSlots sl(a, threadIdx.x & 63);
    for (int buffer = 0;; buffer ^= 1) {
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        const unsigned char* list = a.lists + buffer * kSoloList;
        if (__builtin_amdgcn_readfirstlane(*(const int*)(list + 64 * 8))) break;
        solo_apply(a, sl, list, wave);
    }
}

// Launched with 1024 threads: all of them bring the windows in, then the wavefronts without instances leave.
// CH: 16-byte pieces of a block (1, 2 or 4: windows of at most 32 pieces, which an update takes a lane each; 0: any
// plan, a lane takes a block).  NARROW: with walk_narrow, for calls of 12 requests and more, where it saves over a
// microsecond of a call by itself; its bounds cost a call of few (256 instances of 100 slots, 3 requests 27.5 us without,
// 27.6 with, 8 30.9 and 29.8, 12 34.1 and 31.8; 64 instances 23.7 and 24.2, 26.3 and 25.9, 28.2 and 27.5).
// SOLO: with one wavefront's walk in front of the tables' one (NARROW too); eight wavefronts stay for it.
template <int CH, bool NARROW, bool SOLO>
__global__ __launch_bounds__(kRouteThreads) void route_kernel(
    const int32_t* __restrict__ prompt_tokens, const int32_t* __restrict__ pred_tokens, int n_req, int n_inst,
    int window, int block, int n_blocks, int pitch, int32_t* __restrict__ window_tokens,
    const int32_t* __restrict__ capacity, int64_t* __restrict__ queued_p, int64_t* __restrict__ current_d, int t_mem_pct,
    int beta, int32_t* __restrict__ assigned, int64_t* __restrict__ score100, ps_status* st, int solo_at) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    int4* s_best = (int4*)lds_raw;                               // [2][16] a wavefront's minimum: score, instance
    int4* s_win = (int4*)(lds_raw + 512);                        // [pieces][pitch]
    const int pieces = n_blocks * (block >> 2);
    // maxima by block, with a row of minima for "no block": row b of s_pre is over the blocks below b, of w[t] + t;
    // row b of s_suf over the blocks from b on, of w[t]
    int* s_pre = (int*)(s_win + (size_t)pieces * pitch);         // [n_blocks + 1][pitch]
    int* s_suf = s_pre + (n_blocks + 1) * pitch;                 // [n_blocks + 1][pitch]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kMin = (int)0x80000000;
    const int nw = (n_inst + 63) >> 6;                           // wavefronts that own instances
    // windows in: a wavefront takes whole rows; the slots that fill the last piece hold the minimum, to which
    // nothing is ever added
    for (int t0 = 0; t0 < 4 * pieces; t0 += 64) {
        const int t = t0 + lane;
        for (int i0 = wave; i0 < n_inst; i0 += 16 * 8) {
            int v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + 16 * u;
                v[u] = i < n_inst && t < window ? window_tokens[(int64_t)i * window + t] : kMin;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + 16 * u;
                if (i < n_inst && t < 4 * pieces) ((int*)(s_win + (t >> 2) * pitch + i))[t & 3] = v[u];
            }
        }
    }
    const int inst = tid;
    const bool mine = inst < n_inst;
    long long qp = 0, cd = 0, s100 = 0, thr = 0;
    if (mine) {
        qp = queued_p[inst];
        cd = current_d[inst];
        s100 = 100 * (qp + cd);
        thr = (long long)t_mem_pct * capacity[inst];
        s_pre[inst] = kMin;
        s_suf[n_blocks * pitch + inst] = kMin;
    }
    if (tid < 32) s_best[tid] = make_int4(0x7fffffff, 0, 0, 0);
    if (SOLO && tid == 0) *(int*)(lds_raw + solo_at) = 0;
    __syncthreads();
    // (all eight wavefronts of the one wavefront's walk meet the barriers up to its end)
    if (wave >= (SOLO ? kSoloWaves : nw)) return;

    // One instance's window with a request's ramp added on its first Dc slots, and its two rows of block maxima:
    // all lanes of its wavefront, lane j and lane 32 + n_parts - 1 - j for part j (a piece or a block) of the window.
    const int chunks = CH ? CH : block >> 2;                     // pieces of a block
    const int n_parts = CH ? pieces : n_blocks, part_chunks = CH ? 1 : block >> 2, part_slots = CH ? 4 : block;
    const bool u_low = lane < 32, u_live = (lane & 31) < n_parts;
    const int u_part = u_live ? (u_low ? lane & 31 : n_parts - 1 - (lane & 31)) : 0;
    int4* const u_win = s_win + u_part * part_chunks * pitch;
    const int u_blk = CH ? u_part / max(CH, 1) : u_part;
    int* const u_out = u_low ? s_pre + (u_blk + 1) * pitch : s_suf + u_blk * pitch;
    // the last piece of a block has the prefix, the first the suffix
    const bool u_put = u_live && (CH < 2 || u_part % max(CH, 1) == (u_low ? CH - 1 : 0));
    bool range_fault = false;                                    // a stored value has left int32
    auto update = [&](auto far, int i, int P, int Dc) {
        int m = kMin;
        for (int c = 0; c < part_chunks; ++c) {
            int4* at = u_win + c * pitch + i;
            const int4 v4 = *at;
            int v[4] = {v4.x, v4.y, v4.z, v4.w};
            const int t0 = u_part * part_slots + 4 * c;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int t = t0 + e;
                if (far.value && t < Dc && (long long)v[e] + P + t > 2147483647ll) range_fault = true;
                v[e] = (int)((unsigned)v[e] + (t < Dc ? (unsigned)P + (unsigned)t : 0u));
                m = max(m, (int)((unsigned)v[e] + (u_low && t < window ? (unsigned)t : 0u)));
            }
            if (u_low && u_live) *at = make_int4(v[0], v[1], v[2], v[3]);
        }
        m = u_live ? m : kMin;
        m = dpp_max<0x111, 0xf>(m);
        m = dpp_max<0x112, 0xf>(m);
        m = dpp_max<0x114, 0xf>(m);
        m = dpp_max<0x118, 0xf>(m);
        m = dpp_max<0x142, 0xa>(m);                              // the halves stay apart: lane 15 to row 1, 47 to row 3
        if (u_put) u_out[i] = m;
        // the next score reads what other lanes have written: LDS serves a wavefront in order, the compiler has to
        // keep that order
        asm volatile("" ::: "memory");
    };
    int last = 0;                                                // SOLO: the block that has the first largest w[t] + t
    auto make_tables = [&]() {
        if (CH > 0) {
            // every thread its own instance's rows
            if (mine) {
                int m = kMin;
                for (int b = 0; b < n_blocks; ++b) {
                    const int was = m;
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        const int4 v = s_win[(b * CH + c) * pitch + inst];
                        const int t = 4 * (b * CH + c);
                        // (one piece a block: its first slot is inside.  Not said to the NARROW kernel, whose walk comes out
                        // 0.4 % slower: 4096 requests over 256 instances 2035 us, 2044)
                        if ((CH == 1 && !NARROW) || t < window) m = max(m, (int)((unsigned)v.x + (unsigned)t));
                        if (t + 1 < window) m = max(m, (int)((unsigned)v.y + (unsigned)(t + 1)));
                        if (t + 2 < window) m = max(m, (int)((unsigned)v.z + (unsigned)(t + 2)));
                        if (t + 3 < window) m = max(m, (int)((unsigned)v.w + (unsigned)(t + 3)));
                    }
                    s_pre[(b + 1) * pitch + inst] = m;
                    if (SOLO && m > was) last = b;
                }
                m = kMin;
                for (int b = n_blocks - 1; b >= 0; --b) {
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        const int4 v = s_win[(b * CH + c) * pitch + inst];
                        m = max(m, max(max(v.x, v.y), max(v.z, v.w)));
                    }
                    s_suf[b * pitch + inst] = m;
                }
            }
            asm volatile("" ::: "memory");
        } else if (n_blocks > 0) {
            for (int i = 64 * wave; i < min(64 * wave + 64, n_inst); ++i) update(std::false_type{}, i, 0, 0);
        }
    };
    make_tables();
    // exchange slots alternate: one is rewritten two requests later, after the barrier of the one in between
    int par = 0;
    // The largest of the lanes' values (0 at the least), uniform over the workgroup.
    auto largest = [&](int top) {
        for (int o = 32; o > 0; o >>= 1) top = max(top, __shfl_xor(top, o, 64));
        if (nw > 1) {
            if (lane == 0 && (!SOLO || wave < nw)) s_best[par + wave].x = top;   // (the slots that are written next)
            __syncthreads();
            for (int w = 0; w < nw; ++w) top = max(top, s_best[par + w].x);
            __syncthreads();
        }
        return __builtin_amdgcn_readfirstlane(max(top, 0));
    };

    const long long kNone = 0x7fffffffffffffffll;
    const int ic = mine ? inst : 0;
    const int row4 = pitch * 4, row16 = pitch * 16;              // bytes from a row of the tables to the next
    int nP = 0, nD = 0;                                          // lane l: request l of the next 64
    if (lane < n_req) { nP = prompt_tokens[lane]; nD = pred_tokens[lane]; }
    // The requests of one group of 64.  FAR: their tokens could take a sum, or one of the tables' w[t] + t, to 2^31, so
    // they are scored slot by slot in 64 bits.
    auto walk = [&](auto far, int base, int cnt, int vP, int vD) {
        // blocks below b lie under the request's ramp whole, block b is looked at slot by slot (where the ramp ends on
        // a block boundary that only repeats what the tables say), blocks from the next one on keep their values
        const int vDc = min(max(vD, 0), window), vb = n_blocks > 0 ? vDc / block : 0;
        const int vs = n_blocks > 0 ? (vDc + block - 1) / block : 0;
        const int v_pre = vb * row4, v_suf = vs * row4, v_win = max(min(vb, n_blocks - 1), 0);
        int out_i = -1, out_lo = 0, out_hi = 0;
        for (int q = 0; q < cnt; ++q) {
            const int P = __builtin_amdgcn_readlane(vP, q), D = __builtin_amdgcn_readlane(vD, q);
            if (P < 0 || D < 0) {
                if (tid == 0) report_fault(st, PS_ST_BAD_RECORD, base + q);
                continue;
            }
            const int Dc = __builtin_amdgcn_readlane(vDc, q), blk = __builtin_amdgcn_readlane(v_win, q);
            long long pen = -thr;
            if (far.value) {
                long long pk = kMin;
                for (int t = 0; t < window; ++t)
                    pk = max(pk, (long long)((const int*)(s_win + (t >> 2) * pitch + ic))[t & 3] + (t < Dc ? (long long)P + t : 0ll));
                pen += 100 * pk;
            } else {
                const int pre = *(const int*)((const char*)(s_pre + ic) + __builtin_amdgcn_readlane(v_pre, q));
                const int suf = *(const int*)((const char*)(s_suf + ic) + __builtin_amdgcn_readlane(v_suf, q));
                int pk = kMin;
                for (int c = 0; c < chunks; ++c) {
                    const int4 v = *(const int4*)((const char*)(s_win + ic) + (blk * chunks + c) * row16);
                    const int t = blk * (CH ? 4 * CH : block) + 4 * c;
                    pk = max(max(pk, v.x + (t < Dc ? P + t : 0)), v.y + (t + 1 < Dc ? P + t + 1 : 0));
                    pk = max(max(pk, v.z + (t + 2 < Dc ? P + t + 2 : 0)), v.w + (t + 3 < Dc ? P + t + 3 : 0));
                }
                pen += 100 * (long long)max(max(pk, pre + P), suf);
            }
            pen = pen > 0 && (CH > 0 || window > 0) ? pen : 0;
            if (beta != 1) pen *= beta;
            const long long add100 = 100 * ((long long)P + D);
            const long long L = mine ? s100 + (pen + add100) : kNone;
            // minimum over the wavefront, lowest instance on ties
            int src;
            long long best = wave_min(L, mine, src);
            int best_i = 64 * wave + src;
            if (nw > 1) {
                if (lane == 0) s_best[par + wave] = make_int4((int)best, (int)(best >> 32), best_i, 0);
                // (LDS only: __syncthreads would also wait for the results' global stores)
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                const int4 o = s_best[par + (lane & 15)];        // (slots no wavefront writes are not looked at)
                const int o_lo = o.x, o_hi = o.y, o_i = o.z;
                // (wavefronts are in the order of their instances)
                best = wave_min(lane < nw ? ((long long)o_hi << 32) | (unsigned)o_lo : kNone, lane < nw, src);
                best_i = __builtin_amdgcn_readlane(o_i, src);
                par ^= 16;
            }
            if (lane == q) { out_i = best_i; out_lo = (int)best; out_hi = (int)(best >> 32); }
            if (inst == best_i) { qp += P; cd += D; s100 += add100; }
            if ((best_i >> 6) == wave && Dc > 0) update(far, best_i, P, Dc);
        }
        if (wave == 0 && lane < cnt) {
            assigned[base + lane] = out_i;
            score100[base + lane] = ((long long)out_hi << 32) | (unsigned)out_lo;
        }
    };
    // The same with less to do for a request: blocks of 4, 8 or 16 slots (CH), and scores, peaks and limits that a bound shows
    // to lie in [0, 2^30), peaks below 2^24, so that one register holds a score and a full-rate multiply makes it.  What a
    // request's ramp adds to the block it ends in is worked out for 64 requests at once; what it adds to a lane's slots of
    // the chosen window, while the exchange is under way.
    auto walk_narrow = [&](auto many, int base, int cnt, int vP, int vD) {
        constexpr int B = CH ? 4 * CH : 4;                       // slots of a block
        const int vDc = min(max(vD, 0), window), vb = vDc / B, vw = min(vb, n_blocks - 1);
        const int v_pre = vb * row4, v_suf = (vDc + B - 1) / B * row4, v_win = vw * (B / 4) * row16;
        const int v_add = (int)(100u * ((unsigned)vP + (unsigned)vD));
        int v_ramp[B];
#pragma unroll
        for (int e = 0; e < B; ++e) v_ramp[e] = B * vw + e < vDc ? vP + B * vw + e : 0;
        const bool good = lane < cnt && vP >= 0 && vD >= 0;
        if (wave == 0 && lane < cnt && !good) report_fault(st, PS_ST_BAD_RECORD, base + lane);
        int out_i = -1, out_s = 0, dP = 0;
        // lanes without an instance stay above every score
        const int lim = mine ? (int)min(thr, 0x7fffffffll) : 0x7fffffff, s0 = mine ? (int)s100 : 1 << 30;
        int s32 = s0;
        // Where the loop starts within 32 bytes of instructions is worth up to 5 % of it.  In the kernels with one wavefront's walk
        // it would start in a poor place; all eight measured, 4096 requests that go to the tables at once: 256 instances of 100 slots
        // 2052 us here, 2060 to 2153 elsewhere; of 112 (CH 2) 2196, 2187 to 2284; of 128 (CH 4) 2500, 2508 to 2600.  (What stands
        // in front of the loop moves it: to be measured again with it.)
        if constexpr (SOLO) asm volatile(".p2align 5\n\t.rept %0\n\ts_nop 0\n\t.endr" ::"n"(CH == 1 ? 6 : 4));
        for (unsigned long long todo = __ballot(good); todo; todo &= todo - 1) {
            const int q = __builtin_ctzll(todo);
            const int at = __builtin_amdgcn_readlane(v_win, q);
            int4 w[B / 4];
#pragma unroll
            for (int c = 0; c < B / 4; ++c) w[c] = *(const int4*)((const char*)(s_win + ic) + at + c * row16);
            const int pre = *(const int*)((const char*)(s_pre + ic) + __builtin_amdgcn_readlane(v_pre, q));
            const int suf = *(const int*)((const char*)(s_suf + ic) + __builtin_amdgcn_readlane(v_suf, q));
            const int P = __builtin_amdgcn_readlane(vP, q), Dc = __builtin_amdgcn_readlane(vDc, q);
            const int add = __builtin_amdgcn_readlane(v_add, q);
            int e[B];
#pragma unroll
            for (int c = 0; c < B / 4; ++c) {
                e[4 * c] = w[c].x + __builtin_amdgcn_readlane(v_ramp[4 * c], q);
                e[4 * c + 1] = w[c].y + __builtin_amdgcn_readlane(v_ramp[4 * c + 1], q);
                e[4 * c + 2] = w[c].z + __builtin_amdgcn_readlane(v_ramp[4 * c + 2], q);
                e[4 * c + 3] = w[c].w + __builtin_amdgcn_readlane(v_ramp[4 * c + 3], q);
            }
            int pk = e[0];
#pragma unroll
            for (int c = 1; c + 1 < B; c += 2) pk = max(max(pk, e[c]), e[c + 1]);
            pk = max(max(pk, e[B - 1]), pre + P);
            pk = max(max(pk, suf), 0);                           // (a peak below 0 is no more over a limit than one of 0)
            int pen = max((int)__umul24(pk, 100) - lim, 0);
            if (beta != 1) pen *= beta;
            const int L = s32 + pen + add;
            int m = dpp_min<0x111, 0xf>(L);                      // as in wave_min
            m = dpp_min<0x112, 0xf>(m);
            m = dpp_min<0x114, 0xf>(m);
            m = dpp_min<0x118, 0xf>(m);
            m = dpp_min<0x142, 0xa>(m);
            m = dpp_min<0x143, 0xc>(m);
            int best = __builtin_amdgcn_readlane(m, 63);
            int best_i = 64 * wave + __builtin_ctzll(__ballot(L == best));
            int2 o = make_int2(0, 0);
            if (many.value) {
                if (lane == 0) *(int2*)(s_best + par + wave) = make_int2(best, best_i);
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                o = *(const int2*)(s_best + par + (lane & 15));  // (slots no wavefront writes hold 2^31 - 1)
                par ^= 16;
            }
            int r[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = 4 * u_part + e < Dc ? P + 4 * u_part + e : 0;
            if (many.value) {
                m = dpp_min<0x111, 0xf>(o.x);
                m = dpp_min<0x112, 0xf>(m);                      // lane 3 has the first four
                if (nw > 4) {
                    m = dpp_min<0x114, 0xf>(m);
                    m = dpp_min<0x118, 0xf>(m);
                }
                best = __builtin_amdgcn_readlane(m, nw > 4 ? 15 : 3);
                best_i = __builtin_amdgcn_readlane(o.y, __builtin_ctzll(__ballot(o.x == best)));
            }
            if (lane == q) { out_i = best_i; out_s = best; }
            if (inst == best_i) { s32 += add; dP += P; }
            if ((best_i >> 6) == wave && Dc > 0) {               // as in update
                int4 v = u_win[best_i];
                v.x += r[0];
                v.y += r[1];
                v.z += r[2];
                v.w += r[3];
                if (u_low && u_live) u_win[best_i] = v;
                const int t = 4 * u_part;
                m = max(v.x + (u_low && t < window ? t : 0), v.y + (u_low && t + 1 < window ? t + 1 : 0));
                m = max(max(m, v.z + (u_low && t + 2 < window ? t + 2 : 0)), v.w + (u_low && t + 3 < window ? t + 3 : 0));
                m = u_live ? m : kMin;
                m = dpp_max<0x111, 0xf>(m);
                m = dpp_max<0x112, 0xf>(m);
                m = dpp_max<0x114, 0xf>(m);
                m = dpp_max<0x118, 0xf>(m);
                m = dpp_max<0x142, 0xa>(m);
                if (u_put) u_out[best_i] = m;
                asm volatile("" ::: "memory");
            }
        }
        const int rise = s32 - s0;
        s100 += rise;
        qp += dP;
        cd += rise / 100 - dP;
        if (wave == 0 && lane < cnt) {
            assigned[base + lane] = out_i;
            score100[base + lane] = out_s;
        }
    };
    // bound: no window value is above it, load_bound: no instance's queue, a hundredfold, is (a request raises them by its
    // tokens and the window; taken afresh when that has added up).  A queue or limit below 0 counts as one without bound.
    long long bound = largest(mine ? s_suf[ic] : kMin);
    auto load100 = [&]() { return mine ? (s100 < 0 || thr < 0 || s100 >= 1 << 30 ? 1 << 30 : (int)s100) : 0; };
    bool narrow = NARROW;
    long long load_bound = narrow ? largest(load100()) : 0;
    int walked = 0;                                              // requests that one wavefront's walk has done
    if constexpr (SOLO) {
        const int lanes_log2 = 32 - __builtin_clz(nw - 1);
        int* const words = (int*)(lds_raw + solo_at);            // [4] instances at their limits, requests walked
        int4* const state = (int4*)(words + 4);
        unsigned char* const lists = (unsigned char*)(state + (64 << lanes_log2));
        const SoloWalk a = {prompt_tokens, pred_tokens, n_req, n_inst, window, pitch, beta, (int*)s_win, lanes_log2, state,
                            (int*)(lists + 2 * kSoloList), lists, assigned, score100, st};
        int4* const own = state + solo_at_state(a, ic);
        bool late = false;                                       // at its limit, but not from the first slot on
        if (mine) {
            // (where no sum reaches 0, no ramp reaches beyond t*)
            const int f = s_pre[n_blocks * pitch + inst], most = max(s_suf[inst], 0), lim = (int)min(thr, 0x7fffffffll);
            int t_f = window;
#pragma unroll
            for (int c = CH - 1; c >= 0; --c) {
                const int t = 4 * (last * CH + c);
                const int4 v = s_win[(last * CH + c) * pitch + inst];
                if (t + 3 < window && (int)((unsigned)v.w + (unsigned)(t + 3)) == f) t_f = t + 3;
                if (t + 2 < window && (int)((unsigned)v.z + (unsigned)(t + 2)) == f) t_f = t + 2;
                if (t + 1 < window && (int)((unsigned)v.y + (unsigned)(t + 1)) == f) t_f = t + 1;
                if (t < window && (int)((unsigned)v.x + (unsigned)t) == f) t_f = t;
            }
            if (f < 0) t_f = window;
            late = t_f > 0 && 100ll * f > lim;
            *own = solo_numbers(max(f, 0), t_f, most, lim, beta);
            a.added[inst] = (int)s100;
        }
        const int n_late = __popcll(__ballot(late));
        if (lane == 0 && wave < nw) atomicAdd(words, n_late);
        __syncthreads();
        if (peaks_fit(bound, beta) && load_bound < 1 << 29 && 2 * words[0] <= n_inst) {
            if (wave == 0) {
                const int to = nw == 2   ? solo_walk<2>(a, bound, load_bound)
                               : nw <= 4 ? solo_walk<4>(a, bound, load_bound)
                                         : solo_walk<8>(a, bound, load_bound);
                if (lane == 0) words[1] = to;
            } else {
                solo_follow(a, wave);
            }
            __syncthreads();
            walked = __builtin_amdgcn_readfirstlane(words[1]);
        }
        if (wave >= nw) return;
        if (walked > 0) {
            if (mine) {
                const int rise = own->x - (int)s100, dP = a.added[inst];
                s100 += rise;
                qp += dP;
                cd += rise / 100 - dP;
            }
            if (walked < n_req) {
                make_tables();
                bound = largest(mine ? s_suf[ic] : kMin);
                load_bound = largest(load100());
                if (walked + lane < n_req) { nP = prompt_tokens[walked + lane]; nD = pred_tokens[walked + lane]; }
            }
        }
    }
    for (int base = walked; base < n_req; base += 64) {
        const int cnt = min(64, n_req - base), vP = nP, vD = nD;
        if (base + 64 + lane < n_req) { nP = prompt_tokens[base + 64 + lane]; nD = pred_tokens[base + 64 + lane]; }
        // largest prompt and prediction of the group
        int most = lane < cnt ? max(vP, 0) : 0, most_d = lane < cnt ? max(vD, 0) : 0;
        for (int o = 32; o > 0; o >>= 1) {
            most = max(most, __shfl_xor(most, o, 64));
            if (narrow) most_d = max(most_d, __shfl_xor(most_d, o, 64));
        }
        most = __builtin_amdgcn_readfirstlane(most);
        const long long rise = 64ll * ((long long)most + window);
        const long long load_rise = 6400ll * ((long long)most + __builtin_amdgcn_readfirstlane(most_d));
        auto fits = [&]() { return peaks_fit(bound + rise, beta) && load_bound + load_rise < 1 << 29; };
        if ((narrow && !fits()) || bound + rise >= 2147483647ll) {
            bound = largest(mine ? s_suf[ic] : kMin);
            if (narrow) {
                load_bound = largest(load100());
                narrow = peaks_fit(bound, beta) && load_bound < 1 << 29;     // (neither ever falls)
            }
        }
        if (NARROW && narrow && fits()) {
            if (SOLO || nw > 1) walk_narrow(std::true_type{}, base, cnt, vP, vD);
            else walk_narrow(std::false_type{}, base, cnt, vP, vD);
        } else if (bound + rise >= 2147483647ll) walk(std::true_type{}, base, cnt, vP, vD);
        else walk(std::false_type{}, base, cnt, vP, vD);
        bound += rise;
        load_bound += load_rise;
    }
    if (range_fault) report_fault(st, PS_ST_RANGE, -1);
    if (mine) { queued_p[inst] = qp; current_d[inst] = cd; }
    for (int i = 64 * wave; i < min(64 * wave + 64, n_inst); ++i)
        for (int t = lane; t < window; t += 64) window_tokens[(int64_t)i * window + t] = ((const int*)(s_win + (t >> 2) * pitch + i))[t & 3];
}

// ---- a few requests, or long windows ----------------------------------------------------------------------
// The tables have to be made before the first request is scored, and long blocks make dear scores.  Where that costs more
// than it saves, TPI threads per instance scan its whole window for every request.  The windows lie in LDS:
__device__ __forceinline__ void scan_walk(
    unsigned char* lds_raw, const int32_t* prompt_tokens, const int32_t* pred_tokens, int first_index, int n_req, int n_inst,
    int window, int tpi, int32_t* window_tokens, const int32_t* capacity, int64_t* queued_p, int64_t* current_d,
    int t_mem_pct, int beta, int32_t* assigned, int64_t* score100, ps_status* st) {
    long long* s_qp = (long long*)lds_raw;                       // [n_inst]
    long long* s_cd = s_qp + n_inst;                             // [n_inst]
    long long* s_best = s_cd + n_inst;                           // [2][16] per-wavefront minimum score
    int* s_best_i = (int*)(s_best + 32);                         // [2][16] and its instance
    int* s_cap = s_best_i + 32;                                  // [n_inst]
    int2* s_req = (int2*)(s_cap + n_inst + (n_inst & 1));         // [1024] (P, D) of the requests being walked
    long long* s_out_s = (long long*)(s_req + kRouteThreads);    // [1024] their scores
    int* s_out_i = (int*)(s_out_s + kRouteThreads);              // [1024] and instances, written out per chunk: a
                                                                 // global store per request would be waited for at
                                                                 // every barrier
    int* s_win = s_out_i + kRouteThreads;                        // [n_inst][window]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < n_inst; i += kRouteThreads) { s_qp[i] = queued_p[i]; s_cd[i] = current_d[i]; s_cap[i] = capacity[i]; }
    for (int i = tid; i < n_inst * window; i += kRouteThreads) s_win[i] = window_tokens[i];
    __syncthreads();
    const int inst = tid / tpi, sub = tid % tpi;
    const bool mine = inst < n_inst;
    int* row = s_win + (mine ? inst : 0) * window;
    const long long kNone = 0x7fffffffffffffffll;
    bool range_fault = false;
    for (int r = 0; r < n_req; ++r) {
        if ((r & (kRouteThreads - 1)) == 0) {
            // results of the last 1024 requests out, the next 1024 requests in
            __syncthreads();
            if (r > 0) { assigned[r - kRouteThreads + tid] = s_out_i[tid]; score100[r - kRouteThreads + tid] = s_out_s[tid]; }
            if (r + tid < n_req) s_req[tid] = make_int2(prompt_tokens[r + tid], pred_tokens[r + tid]);
            __syncthreads();
        }
        const int slot = r & (kRouteThreads - 1);
        const int2 pd = s_req[slot];
        const int P = pd.x, D = pd.y;                           // uniform
        if (P < 0 || D < 0) {
            if (tid == 0) { s_out_i[slot] = -1; s_out_s[slot] = 0; report_fault(st, PS_ST_BAD_RECORD, first_index + r); }
            __syncthreads();                                    // keeps the one-barrier-per-request rhythm of the exchange slots
            continue;
        }
        long long peak = -kNone;
        if (mine)
            for (int t = sub; t < window; t += tpi) peak = max(peak, (long long)row[t] + (t < D ? (long long)P + t : 0ll));
        for (int o = tpi >> 1; o > 0; o >>= 1) peak = max(peak, __shfl_xor(peak, o, 64));
        long long L = kNone;
        if (mine && sub == 0) {
            const long long pen = window > 0 ? max(0ll, 100 * peak - (long long)t_mem_pct * s_cap[inst]) : 0ll;
            L = 100 * (s_qp[inst] + P + s_cd[inst] + D) + (long long)beta * pen;
        }
        int bi = mine ? inst : 0x7fffffff;
        // minimum over the wavefront, lowest instance on ties
        for (int o = 32; o > 0; o >>= 1) {
            const long long oL = __shfl_xor(L, o, 64);
            const int oi = __shfl_xor(bi, o, 64);
            if (oL < L || (oL == L && oi < bi)) { L = oL; bi = oi; }
        }
        // the exchange slots alternate between requests, so one barrier per request is enough: a slot
        // is rewritten two requests later, after the barrier of the request in between
        const int par = (r & 1) * 16;
        if (lane == 0) { s_best[par + wave] = L; s_best_i[par + wave] = bi; }
        __syncthreads();
        long long bL = s_best[par];
        int bI = s_best_i[par];
        for (int w = 1; w < kRouteThreads / 64; ++w) {
            const long long oL = s_best[par + w];
            const int oi = s_best_i[par + w];
            if (oL < bL || (oL == bL && oi < bI)) { bL = oL; bI = oi; }
        }
        if (tid == 0) { s_out_i[slot] = bI; s_out_s[slot] = bL; }
        if (mine && inst == bI) {
            const int stop = min(D, window);
            for (int t = sub; t < stop; t += tpi) {
                const long long v = (long long)row[t] + P + t;
                if (v > 2147483647ll) range_fault = true;
                row[t] = (int)v;
            }
            if (sub == 0) { s_qp[inst] += P; s_cd[inst] += D; }
        }
        // no barrier here: an instance's window and counters are only ever touched by its own threads
    }
    __syncthreads();
    {   // results of the last, possibly partial, chunk
        const int done = n_req & ~(kRouteThreads - 1), first = done == n_req ? n_req - kRouteThreads : done;
        if (first + tid < n_req) { assigned[first + tid] = s_out_i[tid]; score100[first + tid] = s_out_s[tid]; }
    }
    if (range_fault) report_fault(st, PS_ST_RANGE, -1);
    for (int i = tid; i < n_inst; i += kRouteThreads) { queued_p[i] = s_qp[i]; current_d[i] = s_cd[i]; }
    for (int i = tid; i < n_inst * window; i += kRouteThreads) window_tokens[i] = s_win[i];
}

__global__ __launch_bounds__(kRouteThreads) void route_scan_kernel(
    const int32_t* __restrict__ prompt_tokens, const int32_t* __restrict__ pred_tokens, int n_req, int n_inst,
    int window, int tpi, int32_t* __restrict__ window_tokens, const int32_t* __restrict__ capacity,
    int64_t* __restrict__ queued_p, int64_t* __restrict__ current_d, int t_mem_pct, int beta,
    int32_t* __restrict__ assigned, int64_t* __restrict__ score100, ps_status* st) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    scan_walk(lds_raw, prompt_tokens, pred_tokens, 0, n_req, n_inst, window, tpi, window_tokens, capacity, queued_p, current_d,
              t_mem_pct, beta, assigned, score100, st);
}

// The same walk with every instance's window in the registers of its TPI threads (thread `sub` of an instance
// owns iterations sub, sub + TPI, ...; at most kRegSlots each).  32-bit arithmetic: a running bound B on every
// window value is kept, and from the first request on that could take a sum to 2^31 (B + P + window) the walk goes on
// in LDS with 64-bit peaks (the registers have no room for them).  The sixteen wavefronts' minima are combined by every wavefront in parallel (one
// entry per lane, shuffles) instead of a serial scan.
const int kRegSlots = 32;

__global__ __launch_bounds__(kRouteThreads) void route_reg_kernel(
    const int32_t* __restrict__ prompt_tokens, const int32_t* __restrict__ pred_tokens, int n_req, int n_inst,
    int window, int tpi, int32_t* __restrict__ window_tokens, const int32_t* __restrict__ capacity,
    int64_t* __restrict__ queued_p, int64_t* __restrict__ current_d, int t_mem_pct, int beta,
    int32_t* __restrict__ assigned, int64_t* __restrict__ score100, ps_status* st) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    long long(*s_best)[16] = (long long(*)[16])lds_raw;         // [2]
    long long* s_out_s = (long long*)lds_raw + 32;              // [1024]
    int2* s_req = (int2*)(s_out_s + kRouteThreads);             // [1024]
    int* s_out_i = (int*)(s_req + kRouteThreads);               // [1024]
    int(*s_best_i)[16] = (int(*)[16])(s_out_i + kRouteThreads); // [2]
    int* s_max = s_out_i + kRouteThreads + 32;                  // [16]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int inst = tid / tpi, sub = tid % tpi;
    const bool mine = inst < n_inst;
    const int kMin = (int)0x80000000;
    int r[kRegSlots];                            // dead slots (beyond the window, or no instance) hold the minimum
    int top = kMin;
#pragma unroll
    for (int i = 0; i < kRegSlots; ++i) {
        const int t = sub + tpi * i;
        r[i] = mine && t < window ? window_tokens[(int64_t)inst * window + t] : kMin;
        top = max(top, r[i]);
    }
    long long qp = 0, cd = 0, cap = 0;
    if (mine && sub == 0) { qp = queued_p[inst]; cd = current_d[inst]; cap = capacity[inst]; }
    // B: an upper bound on every window value, uniform over the workgroup
    for (int o = 32; o > 0; o >>= 1) top = max(top, __shfl_xor(top, o, 64));
    if (lane == 0) s_max[wave] = top;
    __syncthreads();
    long long B = 1 << 30;
    for (int w = 0; w < 16; ++w) B = max(B, (long long)s_max[w]);
    const long long kNone = 0x7fffffffffffffffll;
    int done = n_req;                                           // requests walked here
    for (int q = 0; q < n_req; ++q) {
        if ((q & (kRouteThreads - 1)) == 0) {
            // results of the last 1024 requests out, the next 1024 requests in
            __syncthreads();
            if (q > 0) { assigned[q - kRouteThreads + tid] = s_out_i[tid]; score100[q - kRouteThreads + tid] = s_out_s[tid]; }
            if (q + tid < n_req) s_req[tid] = make_int2(prompt_tokens[q + tid], pred_tokens[q + tid]);
            __syncthreads();
        }
        const int slot = q & (kRouteThreads - 1);
        const int2 pd = s_req[slot];
        const int P = pd.x, D = pd.y;                           // uniform
        if (P < 0 || D < 0) {
            if (tid == 0) { s_out_i[slot] = -1; s_out_s[slot] = 0; report_fault(st, PS_ST_BAD_RECORD, q); }
            __syncthreads();                                    // keeps the one-barrier-per-request rhythm of the exchange slots
            continue;
        }
        if (B + P + window >= 2147483647ll) { done = q; break; }    // a sum below may leave the int32 range
        int pk = kMin;
        const int Pt = P + sub;                                 // P + t of this thread's first iteration
#pragma unroll
        for (int i = 0; i < kRegSlots; ++i) {
            const int t = sub + tpi * i;
            const unsigned add = t < D ? (unsigned)(Pt + tpi * i) : 0u;
            pk = max(pk, (int)((unsigned)r[i] + add));          // (a dead slot stays far below any live one)
        }
        for (int o = tpi >> 1; o > 0; o >>= 1) pk = max(pk, __shfl_xor(pk, o, 64));
        long long L = kNone;
        if (mine && sub == 0) {
            const long long pen = max(0ll, 100 * (long long)pk - (long long)t_mem_pct * cap);
            L = 100 * (qp + P + cd + D) + (long long)beta * pen;
        }
        int bi = mine ? inst : 0x7fffffff;
        // minimum over the wavefront, lowest instance on ties
        for (int o = 32; o > 0; o >>= 1) {
            const long long oL = __shfl_xor(L, o, 64);
            const int oi = __shfl_xor(bi, o, 64);
            if (oL < L || (oL == L && oi < bi)) { L = oL; bi = oi; }
        }
        // the exchange slots alternate between requests, so one barrier per request is enough: a slot
        // is rewritten two requests later, after the barrier of the request in between
        const int par = q & 1;
        if (lane == 0) { s_best[par][wave] = L; s_best_i[par][wave] = bi; }
        __syncthreads();
        long long bL = lane < 16 ? s_best[par][lane] : kNone;
        int bI = lane < 16 ? s_best_i[par][lane] : 0x7fffffff;
        for (int o = 8; o > 0; o >>= 1) {
            const long long oL = __shfl_xor(bL, o, 64);
            const int oi = __shfl_xor(bI, o, 64);
            if (oL < bL || (oL == bL && oi < bI)) { bL = oL; bI = oi; }
        }
        bL = __shfl(bL, 0, 64);
        bI = __shfl(bI, 0, 64);
        if (tid == 0) { s_out_i[slot] = bI; s_out_s[slot] = bL; }
        if (mine && inst == bI) {
#pragma unroll
            for (int i = 0; i < kRegSlots; ++i) {
                const int t = sub + tpi * i;
                if (t < D && t < window) r[i] = (int)((unsigned)r[i] + (unsigned)(Pt + tpi * i));
            }
            if (sub == 0) { qp += P; cd += D; }
        }
        B += (long long)P + window;                             // every new value is at most an old one + P + window
    }
    __syncthreads();
    for (int q = (max(done, 1) - 1) / kRouteThreads * kRouteThreads + tid; q < done; q += kRouteThreads) {   // the last chunk
        assigned[q] = s_out_i[q & (kRouteThreads - 1)];
        score100[q] = s_out_s[q & (kRouteThreads - 1)];
    }
    if (mine && sub == 0) { queued_p[inst] = qp; current_d[inst] = cd; }
#pragma unroll
    for (int i = 0; i < kRegSlots; ++i) {
        const int t = sub + tpi * i;
        if (mine && t < window) window_tokens[(int64_t)inst * window + t] = r[i];
    }
    if (done == n_req) return;
    __threadfence_block();                                      // the state as it stands is the scan's input
    __syncthreads();
    scan_walk(lds_raw, prompt_tokens + done, pred_tokens + done, done, n_req - done, n_inst, window, tpi, window_tokens, capacity,
              queued_p, current_d, t_mem_pct, beta, assigned + done, score100 + done, st);
}

// An update can take a window's pieces a lane each.
bool by_piece(const RoutePlan& p) {
    return (p.block == 4 || p.block == 8 || p.block == 16) && (int64_t)p.n_blocks * p.block <= 4 * kRouteMaxBlocks;
}

// Microseconds a call for n requests, scanned / with the tables, calls back to back (a call by itself takes 10 to 11 more
// either way); the tables take 4 us to make where updates go by pieces, 20 to 60 where the wavefronts make them block by block:
//   by pieces: 256 instances of 100 slots (blocks of 4), n = 1 13.5 / 17.4, 2 17.0 / 18.1, 3 20.3 / 18.9, 64 224 / 49;  256 of 120
//   (of 8) 2 17.6 / 19.5, 3 20.9 / 20.4, 31 115 / 36;  256 of 128 (of 16) 2 18.9 / 19.9, 3 22.2 / 20.8, 31 116 / 37
//   blocks of 8 and 16, not by pieces: 90 of 256, n = 8 33 / 50, 24 83 / 67, 31 106 / 74, 64 209 / 108;  64 of 500, n = 1
//   11.5 / 72, 24 91 / 101, 31 116 / 110, 64 230 / 152, 2048 7107 / 2673
//   blocks of 32 and 48: 1024 of 29 (one block), n = 64 233 / 82, 128 441 / 147, 2048 6624 / 2043;  16 of 1500, n = 64 237 / 252,
//   128 467 / 439, 2048 7340 / 6033
//   longer ones: 1 of 2000, n = 2048 6512 / 8457;  8 of 3000 11409 / 11409;  256 of 134 (one block each) 13903 / 15861
bool tables_pay(int n_req, int window, const RoutePlan& p) {
    if (window == 0) return true;
    return by_piece(p) ? n_req >= 3 : p.block <= 16 ? n_req >= 32 : p.block <= 48 && n_req >= 128;
}

}  // namespace

extern "C" int ps_route(const int32_t* prompt_tokens, const int32_t* pred_tokens, int32_t n_req, int32_t n_inst,
                        int32_t window, int32_t* window_tokens, const int32_t* capacity, int64_t* queued_p,
                        int64_t* current_d, int32_t t_mem_pct, int32_t beta, int32_t* assigned, int64_t* score100,
                        ps_status* status, void* hip_stream) {
    if (n_req < 0 || n_inst < 1 || window < 0 || t_mem_pct < 0 || beta < 0) return PS_EINVAL;
    if (!capacity || !queued_p || !current_d || (window > 0 && !window_tokens)) return PS_EINVAL;
    if (n_req == 0) return PS_OK;
    if (!prompt_tokens || !pred_tokens || !assigned || !score100) return PS_EINVAL;
    if (n_inst > kRouteThreads) return PS_EUNSUPPORTED;
    // the limit the header states (what the scan keeps in LDS); every map within it has a plan that fits (plan_route's
    // last one, a single block per window, takes less)
    const size_t map_bytes = (size_t)n_inst * 20 + (size_t)n_inst * window * 4 + 20928;
    if (map_bytes > (size_t)kRouteLdsBytes) return PS_EUNSUPPORTED;
    RoutePlan p = plan_route(n_inst, window);
    if (p.lds_bytes > (size_t)kRouteLdsBytes) return PS_EUNSUPPORTED;
    hipStream_t s = (hipStream_t)hip_stream;
    (void)hipGetLastError();
    static bool lds_attr_set = false;     // raising the limit twice is harmless, so no lock
    if (!lds_attr_set) {
        if (hipFuncSetAttribute((const void*)route_scan_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kRouteLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void*)route_reg_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kRouteLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void*)route_kernel<0, false, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kRouteLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void*)route_kernel<1, false, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kRouteLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void*)route_kernel<1, true, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kRouteLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void*)route_kernel<1, true, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kRouteLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void*)route_kernel<2, false, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kRouteLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void*)route_kernel<2, true, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kRouteLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void*)route_kernel<2, true, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kRouteLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void*)route_kernel<4, false, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kRouteLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void*)route_kernel<4, true, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kRouteLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void*)route_kernel<4, true, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kRouteLdsBytes) != hipSuccess)
            return PS_EHIP;
        lds_attr_set = true;
    }
#define PS_ROUTE(CH, NARROW, SOLO)                                                                                       \
    hipLaunchKernelGGL((route_kernel<CH, NARROW, SOLO>), dim3(1), dim3(kRouteThreads), p.lds_bytes, s,    \
                       prompt_tokens, pred_tokens, n_req, n_inst, window, p.block, p.n_blocks, p.pitch, window_tokens,   \
                       capacity, queued_p, current_d, t_mem_pct, beta, assigned, score100, status, solo_at)
#define PS_ROUTE_CH(CH)                                \
    do {                                               \
        if (solo_at) PS_ROUTE(CH, true, true);         \
        else if (narrow) PS_ROUTE(CH, true, false);    \
        else PS_ROUTE(CH, false, false);               \
    } while (0)
    int solo_at = 0;
    if (tables_pay(n_req, window, p)) {
        const bool narrow = n_req >= 12;
        // one wavefront's walk, where there is room for it beside the tables
        const size_t at = (p.lds_bytes + 15) / 16 * 16, more = solo_lds_bytes(n_inst);
        if (n_req >= solo_least_requests(n_inst) && by_piece(p) && n_inst > 64 && n_inst <= kSoloInstances && at + more <= (size_t)kRouteLdsBytes) {
            solo_at = (int)at;
            p.lds_bytes = at + more;
        }
        if (!by_piece(p)) PS_ROUTE(0, false, false);
        else if (p.block == 4) PS_ROUTE_CH(1);
        else if (p.block == 8) PS_ROUTE_CH(2);
        else PS_ROUTE_CH(4);
        return hipGetLastError() == hipSuccess ? PS_OK : PS_EHIP;
    }
#undef PS_ROUTE_CH
#undef PS_ROUTE
    int tpi = 64;                                               // threads per instance: a power of two, <= 64
    while (tpi > 1 && (int64_t)tpi * n_inst > kRouteThreads) tpi >>= 1;
    if ((window + tpi - 1) / tpi <= kRegSlots)
        hipLaunchKernelGGL(route_reg_kernel, dim3(1), dim3(kRouteThreads), map_bytes, s, prompt_tokens, pred_tokens, n_req, n_inst,
                           window, tpi, window_tokens, capacity, queued_p, current_d, t_mem_pct, beta, assigned,
                           score100, status);
    else
        hipLaunchKernelGGL(route_scan_kernel, dim3(1), dim3(kRouteThreads), map_bytes, s, prompt_tokens, pred_tokens, n_req,
                           n_inst, window, tpi, window_tokens, capacity, queued_p, current_d, t_mem_pct, beta, assigned,
                           score100, status);
    return hipGetLastError() == hipSuccess ? PS_OK : PS_EHIP;
}
