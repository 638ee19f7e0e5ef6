// Load anticipator (paper Sec. 3.4.1): fold per-request predicted response lengths into the
// per-instance future-load curves load[instance][one-second bucket].
//
// A request is two range additions on its instance's row: buckets [a, a + rem) take q + 1 tokens
// and [a + rem, a + dur) take q, with q = D / dur, rem = D % dur.  Range additions are point
// updates of the row's difference array (+q+1 at a, -1 at a+rem, -q at a+dur), so a record costs
// three integer updates however long it decodes; the curve is the prefix sum of the differences.
//
// Kernel 1 (scatter): the map's rows are split into groups that fit one compute unit's LDS as
// difference arrays; the records are split into slices.  Workgroup (group, slice) streams its
// slice with coalesced 16-byte loads (four records per lane).  Each wavefront compacts the records
// whose instance is in its group into a small LDS queue (ballot + prefix count, no atomics) and,
// whenever 64 are queued, applies them with every lane busy: two exact divisions by float
// reciprocal and three LDS adds into the workgroup's private rows.  At the end the rows go to a
// partial buffer.  The groups of one slice are placed on the same XCD so the slice is fetched from
// HBM once and shared through that XCD's L2.
// Kernel 2 (reduce): one workgroup per instance sums the partial difference rows, takes the prefix
// sum over buckets and accumulates into load[]; overflow[] likewise.  No global atomics: every
// global word has exactly one writer; the only atomic operations are the LDS adds of kernel 1.  All arithmetic is
// integer, so the result is exact and independent of record order.
//
// Records in arrival order (a request log, the order requests are admitted in) allow a cheaper first
// kernel, tried first on long streams: a slice of such a stream touches few buckets, so its workgroup
// keeps a window of buckets for ALL instances in LDS (256 x 152 counters) instead of all buckets for a
// quarter of them.  Every record then belongs to the one workgroup that reads it: no second, third
// and fourth inspection by other groups, no compaction queue.  A workgroup that meets a record
// outside its window says so in place of its result; that makes a kernel for any order run after it
// (otherwise its workgroups leave at once) and tells the reduction which partial results to use, so
// the outcome is the same for any order.  That kernel works as above or, for long streams of many rows, with 16-bit
// counters (halves_body), unless a sample that the windowed kernel takes shows loads too crowded for those.
#include <string.h>

#include <mutex>
#include <type_traits>

#include "device_util.h"
#include "internal.h"

namespace {

const int kLdsBytes = 160 * 1024;        // LDS of one gfx950 compute unit
const int kWaves = 16;                   // wavefronts per scatter workgroup
const int kScatterThreads = kWaves * 64;
const int kQueue = 128;                  // entries of a wavefront's compaction queue
const int kQueueBytes = kWaves * kQueue * 4;
const int64_t kMinSlice = 16384;         // records per slice below which more slices do not pay
const int kTargetWorkgroups = 256;       // one scatter workgroup per compute unit

const int64_t kWindowMinRecords = 262144;   // shorter streams do not pay for the extra launches
// Looks at records (records x groups) that 16-bit counters must save to pay for the sample and the prefix sums: fewer where
// the general form's workgroups do not fit the chip at once, or a workgroup of its reduction has many words to add up.
// Microseconds a call, general / halves: 256 instances of 600 buckets (4 groups / 2) 2 M records 39.9 / 44.5, 5 M 53.3 / 52.6,
// 10 M 72 / 65, 44 M 222 / 175; 100 of 600 (2 / 1) 5 M 48.4 / 50.2, 10 M 61.4 / 58.9; 256 of 1200 (8 / 4) 2 M 45.5 / 47.3, 3 M
// 53.1 / 50.8, 25 M 201 / 141.  The others: 200 of 1100 (6 / 3) 1 M 47.5 / 44.4, 25 M 302 / 211; 1000 of 200 2 M 75 / 59; 66 of
// 1023 (2 / 1) 3 M 61 / 47; 30 of 4096 2 M 66 / 54.
const int64_t kHalvesMinSaved = 8000000, kHalvesMinSavedOthers = 3000000, kHalvesReduceWords = 100000;
const int kWindowMaxHorizon = 4096;         // the reduction keeps one 64-bit row of the map in LDS
// What a windowed workgroup leaves: the first bucket of its window, and
const int kGaveUp = 1 << 16;                // a record fell outside it
const int kCrowded = 1 << 17;               // the rows it weighed are too crowded for 16-bit counters
const int kNothing = 1 << 18;               // no records in its slice

struct AntPlan {
    int rows_per_group, groups, slices;
    int64_t slice_len;
    size_t lds_bytes, partial_bytes, ovf_bytes, total_bytes;
    // windowed first kernel (records in arrival order); w_slices == 0: not used
    int w_slices, w_buckets;
    int64_t w_slice_len;
    size_t w_lds_bytes, w_partial_bytes, w_ovf_bytes, w_origin_bytes, w_partial_at, w_ovf_at, w_origin_at;
    // halves form (records in any order, twice as many rows a workgroup); h_slices == 0: not used
    int h_rows, h_groups, h_slices, h_stride, h_row_bits, h_bucket_bits, h_weighed;
    int64_t h_slice_len;
    size_t h_lds_bytes, h_high_at, h_ovf_at, h_flag_at;
    bool ok;
};

AntPlan make_plan(int64_t n, int n_inst, int horizon) {
    AntPlan p;
    memset(&p, 0, sizeof(p));
    if (horizon > 65535) return p;
    const int64_t per_row = 4 * (int64_t)horizon + 8 + 8;      // difference row + overflow + (rate, 1/rate)
    int64_t fit = (kLdsBytes - kQueueBytes - 64) / per_row;
    if (fit < 1) return p;
    // a queued record names its difference cell (row * horizon + bucket) in 16 bits; LDS capacity
    // already keeps a group below 2^16 cells
    p.groups = (int)((n_inst + fit - 1) / fit);
    p.rows_per_group = (n_inst + p.groups - 1) / p.groups;
    int64_t s = (n + kMinSlice - 1) / kMinSlice;
    const int64_t cap = kTargetWorkgroups / p.groups > 0 ? kTargetWorkgroups / p.groups : 1;
    if (s > cap) s = cap;
    if (s < 1) s = 1;
    p.slices = (int)s;
    p.slice_len = (n + s - 1) / s;
    p.slice_len = (p.slice_len + 3) / 4 * 4;                    // slices start on 16-byte boundaries
    p.lds_bytes = (size_t)(p.rows_per_group * per_row + kQueueBytes + 64);
    p.partial_bytes = align_up((size_t)p.slices * n_inst * horizon * 4, 256);
    p.ovf_bytes = align_up((size_t)p.slices * n_inst * 8, 256);
    p.total_bytes = p.partial_bytes + p.ovf_bytes;
    p.ok = true;
    return p;
}

// Adds the windowed kernel's buffers behind the general ones when the call qualifies for it.
void plan_window(AntPlan& p, int64_t n, int n_inst, int horizon, bool with_rate) {
    p.w_slices = 0;
    if (!p.ok || !with_rate || n < kWindowMinRecords || horizon > kWindowMaxHorizon) return;
    const int64_t fixed = 64 + (int64_t)n_inst * 16;             // flag + overflow + (rate, 1/rate)
    int64_t wb = (kLdsBytes - fixed) / ((int64_t)n_inst * 4);
    if (wb > horizon) wb = horizon;
    if (wb < horizon) wb &= ~(int64_t)3;                          // whole 16-byte groups for the reduction's loads
    if (wb < 32) return;
    int64_t s = (n + kMinSlice - 1) / kMinSlice;
    if (s > kTargetWorkgroups) s = kTargetWorkgroups;
    p.w_slices = (int)s;
    p.w_buckets = (int)wb;
    p.w_slice_len = ((n + s - 1) / s + 3) / 4 * 4;
    p.w_lds_bytes = (size_t)(fixed + (int64_t)n_inst * wb * 4);
    p.w_partial_bytes = align_up((size_t)s * n_inst * wb * 4, 256);
    p.w_ovf_bytes = align_up((size_t)s * n_inst * 8, 256);
    p.w_origin_bytes = align_up((size_t)s * 4, 256);
    p.w_partial_at = p.total_bytes;
    p.w_ovf_at = p.w_partial_at + p.w_partial_bytes;
    p.w_origin_at = p.w_ovf_at + p.w_ovf_bytes;
    p.total_bytes = p.w_origin_at + p.w_origin_bytes;
}

// Bits that hold any index below n.
int bits_for(int n) {
    int bits = 0;
    while ((1 << bits) < n) ++bits;
    return bits;
}

// Lays the halves form's results over the general and the windowed buffers (they are needed only where the windowed
// kernel gave up), as many slices as fit; not used where a workgroup would not hold more rows than the general one's.
void plan_halves(AntPlan& p, int64_t n, int n_inst, int horizon) {
    p.h_slices = 0;
    if (p.w_slices == 0) return;
    const int64_t per_pair = 4 * (int64_t)horizon + 2 * (8 + 4);  // counters, overflow and 1/rate of two rows
    int64_t fit = (kLdsBytes - kQueueBytes - 64) / per_pair * 2;
    if (fit > 256) fit = 256;                                     // (measured up to here)
    p.h_groups = fit > 0 ? (int)((n_inst + fit - 1) / fit) : p.groups;
    const bool others = 8 * p.groups * ((p.slices + 7) / 8) > kTargetWorkgroups || (int64_t)p.slices * horizon > kHalvesReduceWords;
    if (p.h_groups >= p.groups || n * (p.groups - p.h_groups) < (others ? kHalvesMinSavedOthers : kHalvesMinSaved)) return;
    // rows that a windowed workgroup weighs beforehand, a wavefront each
    p.h_weighed = (n_inst + p.w_slices - 1) / p.w_slices;
    if (p.h_weighed > kWaves || 64 + (int64_t)n_inst * 16 + 4 * (int64_t)p.h_weighed * horizon > (int64_t)p.w_lds_bytes) return;
    p.h_rows = ((n_inst + p.h_groups - 1) / p.h_groups + 1) / 2 * 2;
    // fields of a queued record; what LDS holds keeps the two below 19 bits together
    p.h_row_bits = bits_for(p.h_rows);
    p.h_bucket_bits = bits_for(horizon);
    p.h_stride = (horizon + 7) / 8 * 8;
    const int64_t slice_bytes = (int64_t)n_inst * (4 * (int64_t)p.h_stride + 8) + 4 * (int64_t)p.h_groups;
    int64_t s = (n + kMinSlice / 2 - 1) / (kMinSlice / 2);
    const int64_t cap = kTargetWorkgroups / p.h_groups, room = ((int64_t)p.w_origin_at - 1024) / slice_bytes;
    s = s < cap ? s : cap;
    s = s < room ? s : room;
    if (s < 1) return;
    // (beyond some hundred records a cell, of some hundred tokens each, loads would leave 16 bits as a rule)
    if (n / s > 128 * (int64_t)n_inst * horizon) return;
    p.h_slices = (int)s;
    p.h_slice_len = ((n + s - 1) / s + 3) / 4 * 4;
    p.h_lds_bytes = (size_t)(p.h_rows / 2 * per_pair + kQueueBytes + 64);
    p.h_high_at = align_up((size_t)s * n_inst * p.h_stride * 2, 256);
    p.h_ovf_at = 2 * p.h_high_at;
    p.h_flag_at = align_up(p.h_ovf_at + (size_t)s * n_inst * 8, 256);
}

// Exact integer division by float reciprocals.  All numerators here are below 2^20
// (pred_tokens <= PS_MAX_PRED < 2^16, rates clamped to PS_MAX_PRED, which changes no result because a
// rate above the prediction already gives a duration of one bucket; cell indices below 2^16).  For a numerator N < 2^20 and a
// divisor d, let x = N / d.  An estimate e with x < x (1 + 2.5 * 2^-23) <= e <= x (1 + 1.3 * 2^-20) has
// floor(e) = floor(x): e is never below x, and x is either an integer or at least 1/d below the
// next one, while e - x <= N * 1.3 * 2^-20 / d < 1/d.  Both estimates below stay inside that band:
//   - row reciprocal: fl(fl(1/r) * (1 + 2^-21)), then one multiply: factors (1 + 2^-21)(1 +- 2^-24)^3;
//   - v_rcp_f32 (1 ulp) times N times (1 + 2^-20): factors (1 + 2^-20)(1 +- 2^-23)(1 +- 2^-24)^2.
__device__ __forceinline__ unsigned div_by_row(unsigned num, float biased_rcp) {
    return (unsigned)((float)num * biased_rcp);
}
__device__ __forceinline__ unsigned div_exact(unsigned num, unsigned den) {
    return (unsigned)(((float)num * __builtin_amdgcn_rcpf((float)den)) * (1.0f + 0x1p-20f));
}

// What the workgroups of the windowed kernel say together.  Every wavefront looks through all of it itself, so the answer
// is the same across the workgroup without a barrier or LDS.
__device__ __forceinline__ int origin_bits(const int32_t* __restrict__ worigin, int w_slices) {
    int mine = 0;
    for (int s = threadIdx.x & 63; s < w_slices; s += 64) mine |= worigin[s];
    return (__any(mine & kGaveUp) ? kGaveUp : 0) | (__any(mine & kCrowded) ? kCrowded : 0);
}

struct GeneralArgs {
    const int32_t *pred_tokens, *instance_id, *arrival_bucket, *rate;
    int64_t n, slice_len;
    int n_inst, horizon, rows_per_group, groups, slices;
    int32_t* partial;
    int64_t* partial_ovf;
};

__device__ __forceinline__ void general_body(const GeneralArgs& p, unsigned char* lds_raw, ps_status* st) {
    const int32_t *__restrict__ pred_tokens = p.pred_tokens, *__restrict__ instance_id = p.instance_id;
    const int32_t *__restrict__ arrival_bucket = p.arrival_bucket, *__restrict__ rate = p.rate;
    const int64_t n = p.n, slice_len = p.slice_len;
    const int n_inst = p.n_inst, horizon = p.horizon, rows_per_group = p.rows_per_group, groups = p.groups;
    // blocks are dealt to the 8 XCDs round-robin: keep the groups of one slice on one XCD
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int g = j % groups;
    const int slice = (j / groups) * 8 + xcd;
    if (slice >= p.slices) return;
    const int k0 = g * rows_per_group;
    const int rows = min(rows_per_group, n_inst - k0);
    if (rows <= 0) return;
    uint32_t* s_queue = (uint32_t*)lds_raw;                                    // [kWaves][kQueue]
    int* s_flag = (int*)(lds_raw + kQueueBytes);                               // [1] some row has rate < 1
    unsigned long long* s_ovf = (unsigned long long*)(lds_raw + kQueueBytes + 64);  // [rows_per_group]
    int2* s_rr = (int2*)(s_ovf + rows_per_group);                              // (rate, biased 1/rate)
    int* s_diff = (int*)(s_rr + rows_per_group);                               // [rows_per_group][horizon]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) *s_flag = 0;
    __syncthreads();
    for (int i = tid; i < rows * horizon; i += kScatterThreads) s_diff[i] = 0;
    for (int i = tid; i < rows; i += kScatterThreads) {
        s_ovf[i] = 0;
        int r = rate ? rate[k0 + i] : 1;
        if (r < 1) { *s_flag = 1; r = 0; }
        r = min(r, PS_MAX_PRED);
        const float rcp = r > 0 ? (1.0f / (float)r) * (1.0f + 0x1p-21f) : 0.f;
        s_rr[i] = make_int2(r, __float_as_int(rcp));
    }
    __syncthreads();
    const bool bad_rate_rows = *s_flag != 0;                 // uniform; rare

    uint32_t* q = s_queue + wave * kQueue;
    const float rcp_horizon = (1.0f / (float)horizon) * (1.0f + 0x1p-21f);
    unsigned head = 0, tail = 0;                                // wave-uniform ring indices
    unsigned long long mass = 0;       // bound on the magnitude any difference cell can have reached

    // Apply up to 64 queued records (lane i takes entry head + i): all lanes busy on the divisions.
    auto consume = [&](unsigned count) {
        if ((unsigned)lane < count) {
            // entry: difference cell of the arrival bucket (row * horizon + bucket) | prediction
            const uint32_t e = q[(head + lane) & (kQueue - 1)];
            const unsigned D = e & 0xffffu, cell = e >> 16;
            const unsigned kk = div_by_row(cell, rcp_horizon), a = cell - kk * (unsigned)horizon;
            const int2 rr = s_rr[kk];
            unsigned dur;
            if (rate) dur = div_by_row(D + (unsigned)rr.x - 1u, __int_as_float(rr.y));
            else dur = (unsigned)horizon - a;
            const unsigned qq = div_exact(D, dur);
            const unsigned rem = D - qq * dur;
            int* row = s_diff + cell;
            const unsigned room = (unsigned)horizon - a;        // buckets from a to the end of the row
            atomicAdd(row, (int)(qq + 1));
            if (rem < room) atomicAdd(row + rem, -1);
            if (dur < room) {
                atomicAdd(row + dur, -(int)qq);
            } else if (dur > room) {
                const unsigned long long inside = (unsigned long long)room * qq + min(room, rem);
                atomicAdd(&s_ovf[kk], (unsigned long long)D - inside);
            }
            mass += qq + 1;
        }
    };

    const int64_t begin = (int64_t)slice * slice_len;
    const int64_t end = min(begin + slice_len, n);

    // Four consecutive records per lane, 256 per wavefront and block.  Loads run two blocks ahead of
    // the block being processed, so six 16-byte loads per lane are in flight while the wavefront works.
    // The last, partial block of a slice is read record by record.
    struct Block {
        int k[4], d[4], a[4];
        bool ragged;                                            // lane crosses the end of the slice
    };
    // Full blocks are loaded unconditionally (straight-line code keeps the memory counter exact, so
    // a block can be used while the two after it are still in flight); a prefetch past the last
    // full block is redirected to it and never used.
    const int64_t n_full = (end - begin) / 256;
    const int64_t last_full = begin + (n_full - 1) * 256;
    auto load_full = [&](int64_t blk) {
        Block b;
        const int64_t idx = min(blk, last_full) + lane * 4;
        // plain loads: the four row groups of a slice run on one XCD and share the slice through its L2 (with
        // the non-temporal hint the other three groups fetch it again: 0.258 against 0.225 ms on 44.1 M records)
        const int4 kv = *(const int4*)(instance_id + idx);
        const int4 dv = *(const int4*)(pred_tokens + idx);
        const int4 av = *(const int4*)(arrival_bucket + idx);
        b.k[0] = kv.x; b.k[1] = kv.y; b.k[2] = kv.z; b.k[3] = kv.w;
        b.d[0] = dv.x; b.d[1] = dv.y; b.d[2] = dv.z; b.d[3] = dv.w;
        b.a[0] = av.x; b.a[1] = av.y; b.a[2] = av.z; b.a[3] = av.w;
        b.ragged = false;
        return b;
    };
    auto load_ragged = [&](int64_t blk) {
        Block b;
        const int64_t idx = blk + lane * 4;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bool in = idx + c < end;
            b.k[c] = in ? instance_id[idx + c] : -1;            // -1 never matches a group
            b.d[c] = in ? pred_tokens[idx + c] : 0;
            b.a[c] = in ? arrival_bucket[idx + c] : 0;
        }
        b.ragged = idx < end;
        return b;
    };
    auto process_block = [&](const Block& b, int64_t blk) {
        const int64_t idx = blk + lane * 4;
        // validity of all four records at once; a block with a faulty record, or the ragged tail,
        // is checked record by record
        const unsigned dmax = max(max((unsigned)b.d[0], (unsigned)b.d[1]), max((unsigned)b.d[2], (unsigned)b.d[3]));
        const unsigned amax = max(max((unsigned)b.a[0], (unsigned)b.a[1]), max((unsigned)b.a[2], (unsigned)b.a[3]));
        const unsigned kmax = max(max((unsigned)b.k[0], (unsigned)b.k[1]), max((unsigned)b.k[2], (unsigned)b.k[3]));
        const bool suspect = b.ragged || dmax > (unsigned)PS_MAX_PRED || amax >= (unsigned)horizon ||
                             kmax >= (unsigned)n_inst;
        const bool slow = __any(suspect) || bad_rate_rows;      // uniform
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const unsigned kk = (unsigned)(b.k[c] - k0);
            bool m = kk < (unsigned)rows && b.d[c] != 0;
            if (slow) {
                const bool in = idx + c < end;
                const bool k_ok = (unsigned)b.k[c] < (unsigned)n_inst;
                bool ok = (unsigned)b.d[c] <= (unsigned)PS_MAX_PRED && (unsigned)b.a[c] < (unsigned)horizon;
                if (kk < (unsigned)rows && ok && s_rr[kk].x < 1) ok = false;
                // a record outside every group is reported by group 0, others by their own group
                if (in && ((!k_ok && g == 0) || (kk < (unsigned)rows && !ok))) report_fault(st, PS_ST_BAD_RECORD, idx + c);
                m = m && in && ok;
            }
            const unsigned long long mask = __ballot(m);
            if (mask) {
                const unsigned pos = tail + __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                                   __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
                if (m) q[pos & (kQueue - 1)] = ((kk * (unsigned)horizon + (unsigned)b.a[c]) << 16) | (unsigned)b.d[c];
                tail += (unsigned)__popcll(mask);
                if (tail - head >= 64u) {
                    consume(64u);
                    head += 64u;
                }
            }
        }
    };

    const int64_t stride = (int64_t)kWaves * 256;
    const int64_t blk0 = begin + (int64_t)wave * 256;
    const int64_t full_end = begin + n_full * 256;
    if (blk0 < full_end) {
        // three register sets used in rotation (unrolled, so no set is ever copied: a copy would
        // have to wait for the load it copies)
        Block b0 = load_full(blk0);
        Block b1 = load_full(blk0 + stride);
        Block b2 = load_full(blk0 + 2 * stride);
        for (int64_t blk = blk0;;) {
            process_block(b0, blk);
            b0 = load_full(blk + 3 * stride);
            if ((blk += stride) >= full_end) break;
            process_block(b1, blk);
            b1 = load_full(blk + 3 * stride);
            if ((blk += stride) >= full_end) break;
            process_block(b2, blk);
            b2 = load_full(blk + 3 * stride);
            if ((blk += stride) >= full_end) break;
        }
    }
    if (full_end < end && wave == (int)(n_full % kWaves)) process_block(load_ragged(full_end), full_end);
    if (tail != head) consume(tail - head);

    // a cell can only have wrapped if the updates of this workgroup's wavefronts add up to 2^31 or
    // more, i.e. if some wavefront contributed at least 2^31 / kWaves
    for (int o = 32; o > 0; o >>= 1) mass += __shfl_xor(mass, o, 64);
    if (lane == 0 && mass >= (1ull << 31) / kWaves) report_fault(st, PS_ST_RANGE, begin);
    __syncthreads();
    int32_t* out = p.partial + ((int64_t)slice * n_inst + k0) * horizon;
    for (int i = tid; i < rows * horizon; i += kScatterThreads) out[i] = s_diff[i];
    for (int i = tid; i < rows; i += kScatterThreads) p.partial_ovf[(int64_t)slice * n_inst + k0 + i] = (int64_t)s_ovf[i];
}

// Scatter for long streams in any order: 16-bit counters, two rows to a word, so that a workgroup holds twice the rows
// and a record is looked at by half as many workgroups.  The general form is bound by instruction issue, most of it
// looking at records of other groups (118 wavefront instructions per 64 records over four groups of 64 rows).
//
// Word [w][b] holds the difference of row w in its low half and of row w + R in its high half: adding signed amounts,
// shifted for the high half, keeps word = low + 2^16 high modulo 2^32, and the same holds for the prefix sums over b, whose
// halves are the two rows' loads.  Loads are never negative, so if both are below 2^16 the halves are exactly they; a load
// that is not makes the halves add up to less than the true loads (65535 less for every wrap of the low half, which
// carries into the high one, 65536 for the high half).  Compared over the whole workgroup, what the halves add up to is
// therefore equal to the tokens put in exactly if no load has wrapped.  Where one has, the workgroup goes through its slice
// a second time with the rows of a word exchanged: word' = high + 2^16 low.  The low halves of the two are the loads'
// lower 16 bits; word's upper half less the lower 16 bits of the high row is what the low row carried into it, its upper 16
// bits, and the other way round.  The upper bits go to a second plane.
// Results are loads, not differences: the reduction adds them up and needs no scan.
//
// 44.1 M records over 256 instances of 600 buckets: 200 us in the general form, 148 here, of which about 105 are vector
// instructions (19 a look, 48 a record); a queue entry names row, bucket and tokens in fields, so neither side multiplies
// or divides by the row length.  The fields are as wide as the call's rows and buckets ask for, which leaves 14 bits and
// more to the tokens (12 as a fixed width: with 5 % of the predictions above 4096 284 us, the general form 220).
//
// A second pass costs what the first does.  Crowds that a sample shows are left to the general form (anticipate_window_kernel
// takes the sample in 2 us); 5 % of those records in one cell 229 us so, 467 with two more passes in place of a sample,
// general 221; instances drawn by Zipf's law and a rush hour 296, 501 and 287.  What it does not show: 2756 records for one
// cell that follow each other in the stream 290 us, general 217.
struct HalvesArgs {
    const int32_t *pred, *inst, *arrival, *rate;
    int64_t n, slice_len;
    int n_inst, horizon, rows, groups, slices, stride;
    int row_shift, d_bits;               // a queued record: row << row_shift | arrival bucket << d_bits | prediction less one
    uint16_t *low, *high;                // [instance][slice][stride]: the reduction of an instance reads one block
    int64_t* ovf;                        // [slice][instance]
    int32_t* wide;                       // [slice][group]: the upper halves are there too
};

// Difference of both halves, each modulo 2^16.
__device__ __forceinline__ uint32_t sub_halves(uint32_t a, uint32_t b) {
    return ((a - b) & 0xffffu) | ((a & 0xffff0000u) - (b & 0xffff0000u));
}

// One pass over a slice for the group's rows.  SWAP: the second one, with the rows of a word exchanged.
template <bool SWAP>
__device__ __forceinline__ void halves_pass(const HalvesArgs& p, int slice, int g, int k0, int rows, unsigned char* lds_raw,
                                            unsigned long long* s_sum, ps_status* st) {
    const int horizon = p.horizon, R = p.rows / 2;
    uint32_t* s_queue = (uint32_t*)lds_raw;                                    // [kWaves][kQueue]
    int* s_flag = (int*)(lds_raw + kQueueBytes);                               // some row has rate < 1
    unsigned long long* s_ovf = (unsigned long long*)(lds_raw + kQueueBytes + 64);  // [p.rows]
    float* s_rcp = (float*)(s_ovf + p.rows);                                   // biased 1 / rate; 0: no usable rate
    int* s_word = (int*)(s_rcp + p.rows);                                      // [R][horizon]
    // (the wavefront index is uniform: what is derived from it stays in scalar registers)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    __syncthreads();
    if (tid == 0) *s_flag = 0;
    __syncthreads();
    for (int i = tid; i < R * horizon; i += kScatterThreads) s_word[i] = 0;
    for (int i = tid; i < rows; i += kScatterThreads) {
        s_ovf[i] = 0;
        const int r = min(p.rate[k0 + i], PS_MAX_PRED);
        if (r < 1) *s_flag = 1;
        s_rcp[i] = r > 0 ? (1.0f / (float)r) * (1.0f + 0x1p-21f) : 0.f;
    }
    __syncthreads();
    const bool bad_rate_rows = *s_flag != 0;                  // uniform; rare

    uint32_t* q = s_queue + wave * kQueue;
    unsigned head = 0, tail = 0;                                // wave-uniform ring indices
    unsigned long long inside_sum = 0;                          // tokens this lane has put into buckets
    unsigned long long mass = 0;                                // SWAP: bound on what any counter can have reached

    // one record of row `row`: D1 = its tokens less one
    auto apply = [&](unsigned row, unsigned a, unsigned D1) __attribute__((always_inline)) {
        const bool upper = row >= (unsigned)R;
        const unsigned D = D1 + 1u, w = min(row, row - (unsigned)R), sh = upper != SWAP ? 16u : 0u;
        const unsigned dur = div_by_row(D1, s_rcp[row]) + 1u;                   // ceil(D / rate)
        const unsigned qq = div_exact(D, dur);
        const unsigned rem = D - __umul24(qq, dur);
        const unsigned room = (unsigned)horizon - a;            // buckets from a to the end of the row
        int* cell = s_word + __umul24(w, (unsigned)horizon) + a;
        atomicAdd(cell, (int)((qq + (rem != 0)) << sh));        // rem == 0: the +1 and the -1 fall on the same cell
        if (rem != 0 && rem < room) atomicAdd(cell + rem, (int)(0xffffffffu << sh));
        if (dur < room) atomicAdd(cell + dur, (int)(0u - (qq << sh)));
        inside_sum += D;
        if (SWAP) mass += qq + 1;
        if (dur > room) {
            const unsigned long long over = (unsigned long long)D - ((unsigned long long)room * qq + min(room, rem));
            atomicAdd(&s_ovf[row], over);
            inside_sum -= over;
        }
    };
    const unsigned d_most = 1u << p.d_bits, a_mask = (1u << (p.row_shift - p.d_bits)) - 1u;
    // up to 64 queued records, lane i entry head + i
    auto consume = [&](unsigned count) __attribute__((always_inline)) {
        if ((unsigned)lane < count) {
            const uint32_t e = q[(head + lane) & (kQueue - 1)];
            apply(e >> p.row_shift, (e >> p.d_bits) & a_mask, e & (d_most - 1u));
        }
    };
    const int64_t begin = (int64_t)slice * p.slice_len, end = min(begin + p.slice_len, p.n);
    // four consecutive records per lane, 256 per wavefront and block, loads two blocks ahead (plain loads: the groups
    // of a slice share it through their XCD's L2)
    struct Block { int k[4], d[4], a[4]; };
    const int64_t n_full = max(end - begin, (int64_t)0) / 256;
    const int64_t last_full = begin + (n_full - 1) * 256;
    auto load_full = [&](int64_t blk) {
        Block b;
        const int64_t at = min(blk, last_full);                // uniform: scalar addresses
        const int4 kv = ((const int4*)(p.inst + at))[lane];
        const int4 dv = ((const int4*)(p.pred + at))[lane];
        const int4 av = ((const int4*)(p.arrival + at))[lane];
        b.k[0] = kv.x; b.k[1] = kv.y; b.k[2] = kv.z; b.k[3] = kv.w;
        b.d[0] = dv.x; b.d[1] = dv.y; b.d[2] = dv.z; b.d[3] = dv.w;
        b.a[0] = av.x; b.a[1] = av.y; b.a[2] = av.z; b.a[3] = av.w;
        return b;
    };
    auto process = [&](Block b, int64_t blk, bool ragged) __attribute__((always_inline)) {
        // validity of all four records at once; a block with a faulty record, or the ragged tail, is looked at record by
        // record first: what is not to be queued loses its tokens
        const unsigned dmax = max(max((unsigned)b.d[0], (unsigned)b.d[1]), max((unsigned)b.d[2], (unsigned)b.d[3]));
        const unsigned amax = max(max((unsigned)b.a[0], (unsigned)b.a[1]), max((unsigned)b.a[2], (unsigned)b.a[3]));
        const unsigned kmax = max(max((unsigned)b.k[0], (unsigned)b.k[1]), max((unsigned)b.k[2], (unsigned)b.k[3]));
        const bool suspect = ragged || dmax > (unsigned)PS_MAX_PRED || amax >= (unsigned)horizon || kmax >= (unsigned)p.n_inst;
        if (__any(suspect) || bad_rate_rows) {                 // uniform
            const int64_t idx = blk + lane * 4;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const unsigned kk = (unsigned)(b.k[c] - k0);
                const bool in = idx + c < end, k_ok = (unsigned)b.k[c] < (unsigned)p.n_inst, mine = k_ok && kk < (unsigned)rows;
                bool ok = (unsigned)b.d[c] <= (unsigned)PS_MAX_PRED && (unsigned)b.a[c] < (unsigned)horizon;
                if (mine && ok && s_rcp[kk] == 0.f) ok = false;
                // a record outside every group is reported by group 0, others by their own group
                if (in && ((!k_ok && g == 0) || (mine && !ok))) report_fault(st, PS_ST_BAD_RECORD, idx + c);
                if (!(in && mine && ok)) b.d[c] = 0;
            }
        }
        if (__any(dmax > d_most)) {                            // records that no entry holds: applied at once, one a lane and turn
            unsigned left = 0;
            for (int c = 0; c < 4; ++c)
                if ((unsigned)b.d[c] > d_most && (unsigned)(b.k[c] - k0) < (unsigned)rows) left |= 1u << c;
            const unsigned taken = left;
            while (__any(left != 0)) {
                const int k = left & 1 ? b.k[0] : left & 2 ? b.k[1] : left & 4 ? b.k[2] : b.k[3];
                const int d = left & 1 ? b.d[0] : left & 2 ? b.d[1] : left & 4 ? b.d[2] : b.d[3];
                const int a = left & 1 ? b.a[0] : left & 2 ? b.a[1] : left & 4 ? b.a[2] : b.a[3];
                if (left != 0) apply((unsigned)(k - k0), (unsigned)a, (unsigned)d - 1u);
                left &= left - 1;
            }
            for (int c = 0; c < 4; ++c) b.d[c] = taken >> c & 1 ? 0 : b.d[c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const unsigned kk = (unsigned)(b.k[c] - k0), d1 = (unsigned)b.d[c] - 1u;
            const bool m = (kk | (d1 & 0x80000000u)) < (unsigned)rows;          // (no tokens: d1 wraps)
            const unsigned long long mask = __builtin_amdgcn_ballot_w64(m);
            const unsigned pos = __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, tail));
            if (m) q[pos & (kQueue - 1)] = (kk << p.row_shift) | ((unsigned)b.a[c] << p.d_bits) | d1;
            tail += (unsigned)__popcll(mask);
            if (tail - head >= 64u) {
                consume(64u);
                head += 64u;
            }
        }
    };
    const int64_t stride = (int64_t)kWaves * 256;
    const int64_t blk0 = begin + (int64_t)wave * 256;
    const int64_t full_end = begin + n_full * 256;
    if (blk0 < full_end) {
        Block b0 = load_full(blk0);
        Block b1 = load_full(blk0 + stride);
        Block b2 = load_full(blk0 + 2 * stride);
        for (int64_t blk = blk0;;) {
            process(b0, blk, false);
            b0 = load_full(blk + 3 * stride);
            if ((blk += stride) >= full_end) break;
            process(b1, blk, false);
            b1 = load_full(blk + 3 * stride);
            if ((blk += stride) >= full_end) break;
            process(b2, blk, false);
            b2 = load_full(blk + 3 * stride);
            if ((blk += stride) >= full_end) break;
        }
    }
    if (full_end < end && wave == (int)(n_full % kWaves)) {
        Block b;
        const int64_t idx = full_end + lane * 4;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bool in = idx + c < end;
            b.k[c] = in ? p.inst[idx + c] : -1;                // -1 matches no row
            b.d[c] = in ? p.pred[idx + c] : 0;
            b.a[c] = in ? p.arrival[idx + c] : 0;
        }
        process(b, full_end, true);
    }
    if (tail != head) consume(tail - head);
    if (SWAP) {
        for (int o = 32; o > 0; o >>= 1) mass += __shfl_xor(mass, o, 64);
        if (lane == 0 && mass >= (1ull << 31) / kWaves) report_fault(st, PS_ST_RANGE, begin);
    }
    __syncthreads();

    // prefix sums, a wavefront per row of words, two words a lane; the loads of both rows go out as they are
    unsigned long long halves_sum = 0;
    for (int w = wave; w < min(R, rows); w += kWaves) {
        const int64_t at = ((int64_t)(k0 + w) * p.slices + slice) * p.stride, at2 = at + (int64_t)R * p.slices * p.stride;
        const bool two = w + R < rows;
        if (SWAP && !two) continue;                             // (alone in its words: nothing is missing)
        unsigned carry = 0;
        for (int b0 = 0; b0 < horizon; b0 += 128) {
            const int b = b0 + 2 * lane;
            const unsigned x = b < horizon ? (unsigned)s_word[w * horizon + b] : 0u;
            const unsigned y = b + 1 < horizon ? (unsigned)s_word[w * horizon + b + 1] : 0u;
            unsigned incl = x + y;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const unsigned t = __shfl_up(incl, o, 64);
                if (lane >= o) incl += t;
            }
            const unsigned s1 = carry + incl, s0 = s1 - y;     // loads of buckets b and b + 1
            const unsigned lo = (s0 & 0xffffu) | (s1 << 16), up = (s0 >> 16) | (s1 & 0xffff0000u);
            if (b < p.stride) {                                 // (stride is even; cells beyond the horizon are not read)
                if (SWAP) {
                    const unsigned lo1 = *(const uint32_t*)(p.low + at + b), up1 = *(const uint32_t*)(p.low + at2 + b);
                    *(uint32_t*)(p.high + at + b) = sub_halves(up1, lo);
                    *(uint32_t*)(p.low + at2 + b) = lo;
                    *(uint32_t*)(p.high + at2 + b) = sub_halves(up, lo1);
                } else {
                    *(uint32_t*)(p.low + at + b) = lo;
                    *(uint32_t*)((two ? p.low + at2 : p.high + at) + b) = up;
                }
            }
            if (!SWAP) {
                if (b < horizon) halves_sum += (s0 & 0xffffu) + (s0 >> 16);
                if (b + 1 < horizon) halves_sum += (s1 & 0xffffu) + (s1 >> 16);
            }
            carry += __shfl(incl, 63, 64);
        }
    }
    for (int i = tid; i < rows; i += kScatterThreads) p.ovf[(int64_t)slice * p.n_inst + k0 + i] = (int64_t)s_ovf[i];
    if (!SWAP) {
        unsigned long long diff = inside_sum - halves_sum;
        for (int o = 32; o > 0; o >>= 1) diff += __shfl_xor(diff, o, 64);
        if (lane == 0) atomicAdd(s_sum, diff);
    }
}

__device__ __forceinline__ void halves_body(const HalvesArgs& p, unsigned char* lds_raw, ps_status* st) {
    unsigned long long* s_sum = (unsigned long long*)(lds_raw + kQueueBytes + 8);   // tokens put in less what the halves show
    // blocks are dealt to the 8 XCDs round-robin: keep the groups of one slice on one XCD
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int g = j % p.groups, slice = (j / p.groups) * 8 + xcd;
    if (slice >= p.slices) return;
    const int k0 = g * p.rows, rows = min(p.rows, p.n_inst - k0);
    if (rows <= 0) return;
    if (threadIdx.x == 0) *s_sum = 0;
    halves_pass<false>(p, slice, g, k0, rows, lds_raw, s_sum, st);
    __syncthreads();
    const bool wrapped = *s_sum != 0;                          // uniform
    if (threadIdx.x == 0) p.wide[slice * p.groups + g] = wrapped;
    if (wrapped) halves_pass<true>(p, slice, g, k0, rows, lds_raw, s_sum, st);
}

// The scatter for any order, launched behind the windowed one where that is tried: needed only if it gave up somewhere.
__global__ __launch_bounds__(kScatterThreads) void anticipate_scatter_kernel(GeneralArgs p, HalvesArgs hv,
                                                                             const int32_t* __restrict__ worigin,
                                                                             int w_slices, ps_status* st) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int bits = worigin ? origin_bits(worigin, w_slices) : kGaveUp;
    if (!(bits & kGaveUp)) return;
    if (hv.slices > 0 && !(bits & kCrowded)) halves_body(hv, lds_raw, st);
    else general_body(p, lds_raw, st);
}

// Windowed scatter for records in arrival order: workgroup = slice of the records; LDS holds, for
// every instance, the difference counters of the buckets [a0, a0 + w_buckets), a0 = the arrival bucket
// of the slice's first record.  Each lane takes its own records straight through the two divisions and
// the three LDS adds.  A record that reaches outside the window (or before it) makes the workgroup
// leave kGaveUp in place of its origin; the scatter for any order then redoes the whole call.
__global__ __launch_bounds__(kScatterThreads) void anticipate_window_kernel(
    const int32_t* __restrict__ pred_tokens, const int32_t* __restrict__ instance_id,
    const int32_t* __restrict__ arrival_bucket, const int32_t* __restrict__ rate, int64_t n, int n_inst,
    int horizon, int w_buckets, int64_t slice_len, int weighed, int64_t h_slice_len, int32_t* __restrict__ wpartial,
    int64_t* __restrict__ wovf, int32_t* __restrict__ worigin, ps_status* st) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    int* s_flag = (int*)lds_raw;                                              // [0] a row has rate < 1, [1] gave up
    unsigned long long* s_ovf = (unsigned long long*)(lds_raw + 64);          // [n_inst]
    int2* s_rr = (int2*)(s_ovf + n_inst);                                      // (rate, biased 1/rate)
    int* s_diff = (int*)(s_rr + n_inst);                                       // [n_inst][w_buckets]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int slice = blockIdx.x;
    const int64_t begin = (int64_t)slice * slice_len;
    const int64_t end = min(begin + slice_len, n);
    // window origin: the slice's first arrival bucket; a faulty (negative) one must not shift the window the
    // slice's valid records are placed in, so the origin is never below bucket 0 (a first bucket at or beyond
    // the horizon leaves every valid record before the window: the workgroup gives up and the scatter for any order runs)
    const int a0 = begin < end ? max(arrival_bucket[begin], 0) : 0;
    const int64_t probe = begin + (int64_t)tid * 4;
    int4 probed = make_int4(-1, -1, -1, -1);
    if (probe + 4 <= end) probed = *(const int4*)(arrival_bucket + probe);
    unsigned* s_top = (unsigned*)(lds_raw + 8);               // of the sample: largest load; tokens; tokens times what a
    unsigned long long *s_tokens = (unsigned long long*)(lds_raw + 16), *s_weighted = s_tokens + 1;   // bucket gets of them
    if (tid < 2) { s_flag[tid] = 0; *s_top = 0; s_tokens[tid] = 0; }
    if (begin >= end) {
        if (tid == 0) worigin[slice] = kNothing;
        return;
    }
    __syncthreads();
    {
        // A look at the slice's first records before anything is set up: a stream in no particular order shows a
        // valid arrival bucket outside the window at once, and the workgroup leaves without clearing its counters.
        // (Invalid buckets are not counted: such records are skipped, not folded.)
        const int aa[4] = {probed.x, probed.y, probed.z, probed.w};
        bool far = false;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            far |= (unsigned)aa[c] < (unsigned)horizon && (unsigned)(aa[c] - a0) >= (unsigned)w_buckets;
        if (__any(far) && lane == 0) s_flag[1] = 1;
        __syncthreads();
    }
    if (s_flag[1]) {                                          // uniform
        // A sample of the whole stream, 16 records from each of 256 places (four from each of 1024: 4 us more a call), for
        // `weighed` rows a workgroup.  Loaded here and not ahead of the look above: 0.3 us more for streams in any order,
        // 0.9 less for a log of 44.1 M.
        const int k0 = slice * weighed, rows = max(min(weighed, n_inst - k0), 0);
        int4 kv = {}, dv = {}, av = {};
        int rates = 0;                                         // of row `lane`
        if (rows > 0) {
            const int64_t at = (int64_t)(tid >> 2) * (n / 4096 * 16) + 4 * (tid & 3);
            kv = *(const int4*)(instance_id + at);
            dv = *(const int4*)(pred_tokens + at);
            av = *(const int4*)(arrival_bucket + at);
            rates = rate[min(k0 + (lane & (kWaves - 1)), n_inst - 1)];
            for (int i = tid; i < rows * horizon; i += kScatterThreads) s_diff[i] = 0;
        }
        __syncthreads();
        // Are its rows too crowded for 16-bit counters?  The sample's largest load, scaled up to a slice of halves_body.  A
        // load m of records that give a bucket q each varies by sqrt(q m) from sample to sample (q: the mean over
        // tokens): two of those are taken off, so that a few large records that met by chance are no crowd.
        const int kk[4] = {kv.x, kv.y, kv.z, kv.w}, dd[4] = {dv.x, dv.y, dv.z, dv.w}, aa[4] = {av.x, av.y, av.z, av.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int row = kk[c] - k0, D = dd[c], r = min(__shfl(rates, row & (kWaves - 1), 64), PS_MAX_PRED);
            if ((unsigned)kk[c] >= (unsigned)n_inst || (unsigned)row >= (unsigned)rows) continue;
            if (D < 1 || D > PS_MAX_PRED || (unsigned)aa[c] >= (unsigned)horizon || r < 1) continue;
            const int dur = (int)div_exact((unsigned)(D + r - 1), (unsigned)r), q = (int)div_exact((unsigned)D, (unsigned)dur);
            atomicAdd(s_diff + row * horizon + aa[c], q);
            if (dur < horizon - aa[c]) atomicAdd(s_diff + row * horizon + aa[c] + dur, -q);
            atomicAdd(s_tokens, (unsigned long long)D);
            atomicAdd(s_weighted, (unsigned long long)D * q);
        }
        __syncthreads();
        if (wave < rows) {                                     // a wavefront a row, sixteen neighbouring buckets a lane
            int carry = 0, top = 0;
            for (int b0 = 0; b0 < horizon; b0 += 1024) {
                const int b = b0 + 16 * lane;
                int v[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] = b + i < horizon ? s_diff[wave * horizon + b + i] : 0;
                int most = v[0];
#pragma unroll
                for (int i = 1; i < 16; ++i) {
                    v[i] += v[i - 1];
                    most = max(most, v[i]);
                }
                int run = v[15];
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int t = __shfl_up(run, o, 64);
                    if (lane >= o) run += t;
                }
                top = max(top, carry + run - v[15] + most);
                carry += __shfl(run, 63, 64);
            }
            for (int o = 32; o > 0; o >>= 1) top = max(top, __shfl_xor(top, o, 64));
            if (lane == 0) atomicMax(s_top, (unsigned)top);
        }
        if (rows > 1) __syncthreads();                         // (one row: its wavefront is the one that goes on)
        if (tid == 0) {
            const float m = (float)*s_top, q = (float)*s_weighted / fmaxf((float)*s_tokens, 1.0f);
            const bool crowded = (m - 2.0f * sqrtf(q * m)) * (float)h_slice_len > 65535.0f * 4096.0f;
            worigin[slice] = kGaveUp | (crowded ? kCrowded : 0);
        }
        return;
    }
    for (int i = tid; i < n_inst * w_buckets; i += kScatterThreads) s_diff[i] = 0;
    for (int i = tid; i < n_inst; i += kScatterThreads) {
        s_ovf[i] = 0;
        int r = rate[i];
        if (r < 1) { s_flag[0] = 1; r = 0; }
        r = min(r, PS_MAX_PRED);
        const float rcp = r > 0 ? (1.0f / (float)r) * (1.0f + 0x1p-21f) : 0.f;
        s_rr[i] = make_int2(r, __float_as_int(rcp));
    }
    __syncthreads();
    const bool bad_rate_rows = s_flag[0] != 0;               // uniform; rare
    unsigned long long mass = 0;       // bound on the magnitude any difference cell can have reached
    unsigned mass32 = 0;               //   (a block's share, folded into it after the block)
    bool outside = false;

    // One record: (validity,) the two divisions, window test, three adds.  CHECKED is only used for
    // blocks that hold a record failing the cheap range test, rows without a usable rate, and the tail.
    // (rr = the instance's (rate, 1 / rate), read by the caller for all of a lane's records before the
    // first add, so that no read queues up behind another record's adds)
    auto take = [&](int k, int D, int a, int2 rr, int64_t idx, bool in, auto checked_tag) {
        constexpr bool CHECKED = decltype(checked_tag)::value;
        if (CHECKED) {
            bool ok = (unsigned)k < (unsigned)n_inst && (unsigned)D <= (unsigned)PS_MAX_PRED && (unsigned)a < (unsigned)horizon;
            if (ok && rr.x < 1) ok = false;
            if (in && !ok) report_fault(st, PS_ST_BAD_RECORD, idx);
            if (!(in && ok)) return;
        }
        const unsigned dur = div_by_row((unsigned)D + (unsigned)rr.x - 1u, __int_as_float(rr.y));
        const unsigned qq = div_exact((unsigned)D, max(dur, 1u));         // D == 0: dur == 0, nothing is added
        const unsigned rem = (unsigned)D - __umul24(qq, dur);        // both below 2^16
        const unsigned room = (unsigned)horizon - (unsigned)a;     // buckets from a to the end of the row
        const unsigned rel = (unsigned)(a - a0);                    // wraps to a huge value before the window
        const unsigned reach = min(dur, room - 1u);                 // furthest bucket touched, from a
        const bool out = rel >= (unsigned)w_buckets || rel + reach >= (unsigned)w_buckets;
        outside |= out && D != 0;
        if (!out && D != 0) {
            int* cell = s_diff + __umul24((unsigned)k, (unsigned)w_buckets) + rel;   // (LDS holds the rows: both small)
            atomicAdd(cell, (int)(qq + (rem != 0)));                // rem == 0: the +1 and the -1 fall on the same cell
            if (rem != 0 && rem < room) atomicAdd(cell + rem, -1);
            if (dur < room) {
                atomicAdd(cell + dur, -(int)qq);
            } else if (dur > room) {
                const unsigned long long inside = (unsigned long long)room * qq + min(room, rem);
                atomicAdd(&s_ovf[k], (unsigned long long)D - inside);
            }
            mass32 += qq + 1;
        }
    };
    using Checked = std::true_type;
    using Unchecked = std::false_type;

    // four consecutive records per lane, 256 per wavefront and block, loads two blocks ahead
    const int64_t n_full = (end - begin) / 256;
    const int64_t last_full = begin + (n_full - 1) * 256;
    struct Blk { int4 k, d, a; };
    auto load_full = [&](int64_t blk) {
        Blk b;
        const int64_t idx = min(blk, last_full) + lane * 4;
        b.k = load_stream_int4(instance_id + idx);
        b.d = load_stream_int4(pred_tokens + idx);
        b.a = load_stream_int4(arrival_bucket + idx);
        return b;
    };
    auto process = [&](const Blk& b, int64_t blk) {
        const int64_t idx = blk + lane * 4;
        // range test of all four records at once; a block with a suspect record is checked record by record
        const unsigned dmax = max(max((unsigned)b.d.x, (unsigned)b.d.y), max((unsigned)b.d.z, (unsigned)b.d.w));
        const unsigned amax = max(max((unsigned)b.a.x, (unsigned)b.a.y), max((unsigned)b.a.z, (unsigned)b.a.w));
        const unsigned kmax = max(max((unsigned)b.k.x, (unsigned)b.k.y), max((unsigned)b.k.z, (unsigned)b.k.w));
        const bool suspect = dmax > (unsigned)PS_MAX_PRED || amax >= (unsigned)horizon || kmax >= (unsigned)n_inst;
        const int kk[4] = {b.k.x, b.k.y, b.k.z, b.k.w}, dd[4] = {b.d.x, b.d.y, b.d.z, b.d.w}, aa[4] = {b.a.x, b.a.y, b.a.z, b.a.w};
        int2 rr[4];
        if (__any(suspect) || bad_rate_rows) {
#pragma unroll
            for (int c = 0; c < 4; ++c) rr[c] = (unsigned)kk[c] < (unsigned)n_inst ? s_rr[kk[c]] : make_int2(0, 0);
#pragma unroll
            for (int c = 0; c < 4; ++c) take(kk[c], dd[c], aa[c], rr[c], idx + c, true, Checked{});
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) rr[c] = s_rr[kk[c]];
#pragma unroll
            for (int c = 0; c < 4; ++c) take(kk[c], dd[c], aa[c], rr[c], idx + c, true, Unchecked{});
        }
        mass += mass32;
        mass32 = 0;
    };
    const int64_t stride = (int64_t)kWaves * 256;
    const int64_t blk0 = begin + (int64_t)wave * 256;
    const int64_t full_end = begin + n_full * 256;
    if (blk0 < full_end) {
        Blk b0 = load_full(blk0);
        Blk b1 = load_full(blk0 + stride);
        Blk b2 = load_full(blk0 + 2 * stride);
        for (int64_t blk = blk0;;) {
            process(b0, blk);
            b0 = load_full(blk + 3 * stride);
            if ((blk += stride) >= full_end || __any(outside)) break;
            process(b1, blk);
            b1 = load_full(blk + 3 * stride);
            if ((blk += stride) >= full_end || __any(outside)) break;
            process(b2, blk);
            b2 = load_full(blk + 3 * stride);
            if ((blk += stride) >= full_end || __any(outside)) break;
        }
    }
    if (full_end < end && wave == (int)(n_full % kWaves)) {
        const int64_t idx = full_end + lane * 4;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bool in = idx + c < end;
            const int k = in ? instance_id[idx + c] : 0;
            take(k, in ? pred_tokens[idx + c] : 0, in ? arrival_bucket[idx + c] : 0,
                 (unsigned)k < (unsigned)n_inst ? s_rr[k] : make_int2(0, 0), idx + c, in, Checked{});
        }
    }
    mass += mass32;
    if (__any(outside) && lane == 0) s_flag[1] = 1;
    for (int o = 32; o > 0; o >>= 1) mass += __shfl_xor(mass, o, 64);
    if (lane == 0 && mass >= (1ull << 31) / kWaves) report_fault(st, PS_ST_RANGE, begin);
    __syncthreads();
    if (s_flag[1]) {                                          // uniform: the scatter for any order takes over
        if (tid == 0) worigin[slice] = kGaveUp;
        return;
    }
    // instance-major: wpartial[instance][slice][bucket of the window], so that the reduction of an
    // instance reads one contiguous block
    const float inv_wb = 1.0f / (float)w_buckets;
    for (int i = tid; i < n_inst * w_buckets; i += kScatterThreads) {
        int k = (int)(((float)i + 0.5f) * inv_wb);
        int r = i - k * w_buckets;
        if (r < 0) { r += w_buckets; --k; }
        if (r >= w_buckets) { r -= w_buckets; ++k; }
        wpartial[((int64_t)k * gridDim.x + slice) * w_buckets + r] = s_diff[i];
    }
    for (int i = tid; i < n_inst; i += kScatterThreads) wovf[(int64_t)slice * n_inst + i] = (int64_t)s_ovf[i];
    if (tid == 0) worigin[slice] = a0;
}

// One workgroup per instance.  Where the horizon is short enough for a 64-bit row of the map in LDS, all
// 1024 threads first stream this instance's partial rows (one per slice: the whole horizon from the
// general form, a window at its origin from the windowed one) and add them into that row: the
// (slice, cell) pairs are dealt to the threads in order, so loads are contiguous runs, 16 in flight per
// thread, and the lanes of an LDS add hit different cells.  Longer horizons sum the general form's
// rows bucket by bucket.  Then buckets are taken 1024 at a time, thread t < 256 owning the four
// consecutive buckets 4 t .. 4 t + 3: it prefix-sums its four values, the 256 thread totals are scanned
// with wavefront shuffles, and the curve is accumulated into load[].  64-bit sums, so a bucket leaving
// the int32 range is seen exactly.
const int kReduceThreads = 1024;

__global__ __launch_bounds__(kReduceThreads) void anticipate_reduce_kernel(
    const int32_t* __restrict__ partial, const int64_t* __restrict__ partial_ovf, int slices, int n_inst, int horizon,
    const int32_t* __restrict__ wpartial, const int64_t* __restrict__ wovf, const int32_t* __restrict__ worigin,
    int w_slices, int w_buckets, HalvesArgs hv, int32_t* __restrict__ load, int64_t* __restrict__ overflow, ps_status* st) {
    __shared__ long long s_wave[4];
    __shared__ unsigned long long s_over;
    __shared__ int s_origin[kTargetWorkgroups];              // first bucket of every slice's row
    __shared__ unsigned long long s_row[kWindowMaxHorizon];  // this instance's difference row, 64-bit
    const int k = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // which first kernel produced the partial results: the windowed one unless it gave up
    const int bits = worigin ? origin_bits(worigin, w_slices) : kGaveUp;
    const bool windowed = !(bits & kGaveUp);
    const bool in_lds = horizon <= kWindowMaxHorizon;         // (the windowed kernel is only used then)
    if (tid == 0) s_over = 0;                                 // (a barrier follows before its first use)
    if (hv.slices > 0 && bits == kGaveUp) {
        // the halves form's loads: a thread adds up eight neighbouring buckets of every T-th slice
        for (int i = tid; i < horizon; i += kReduceThreads) s_row[i] = 0;
        const int wg = k / hv.rows;
        bool some = false;
        for (int i = tid; i < hv.slices; i += kReduceThreads) {
            s_origin[i] = hv.wide[i * hv.groups + wg];         // (this slice's upper halves are there)
            some |= s_origin[i] != 0;
        }
        const bool wide = __syncthreads_or(some) != 0;        // rare
        const int groups = hv.stride >> 3, T = kReduceThreads / groups;       // (at most 512 groups)
        const int sl0 = tid / groups, g8 = tid - sl0 * groups;
        const int64_t step = hv.stride, at0 = (int64_t)k * hv.slices * hv.stride + 8 * g8;
        auto add_plane = [&](const uint16_t* plane, bool upper) {
            unsigned sum[8] = {0, 0, 0, 0, 0, 0, 0, 0};       // at most 256 slices of 16 bits
            constexpr int NB = 10;
            for (int s0 = sl0; s0 < hv.slices; s0 += T * NB) {
                uint4 v[NB];
#pragma unroll
                for (int u = 0; u < NB; ++u) v[u] = *(const uint4*)(plane + min(s0 + T * u, hv.slices - 1) * step + at0);
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const int sl = s0 + T * u;
                    if (sl >= hv.slices || (upper && s_origin[sl] == 0)) continue;
                    const unsigned x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                    for (int c = 0; c < 4; ++c) { sum[2 * c] += x[c] & 0xffffu; sum[2 * c + 1] += x[c] >> 16; }
                }
            }
#pragma unroll
            for (int c = 0; c < 8; ++c)
                if (8 * g8 + c < horizon && sum[c]) atomicAdd(&s_row[8 * g8 + c], (unsigned long long)sum[c] << (upper ? 16 : 0));
        };
        if (sl0 < T) {
            add_plane(hv.low, false);
            if (wide) add_plane(hv.high, true);
        }
        __syncthreads();
        for (int b = tid; b < horizon; b += kReduceThreads) {
            int32_t* cell = load + (int64_t)k * horizon + b;
            const long long nv = (long long)*cell + (long long)s_row[b];
            if (nv > 2147483647ll || nv < -2147483648ll) report_fault(st, PS_ST_RANGE, -1);
            *cell = (int32_t)(uint32_t)(unsigned long long)nv;
        }
        if (overflow) {
            for (int s2 = tid; s2 < hv.slices; s2 += kReduceThreads) {
                const long long o = hv.ovf[(int64_t)s2 * n_inst + k];
                if (o) atomicAdd(&s_over, (unsigned long long)o);
            }
            __syncthreads();
            if (tid == 0 && s_over) overflow[k] += (long long)s_over;
        }
        return;
    }
    if (in_lds) {
        const int n_rows = windowed ? w_slices : slices, row_len = windowed ? w_buckets : horizon;
        for (int s = tid; s < n_rows; s += kReduceThreads) s_origin[s] = !windowed ? 0 : worigin[s] & kNothing ? -1 : worigin[s] & 0xffff;
        for (int i = tid; i < horizon; i += kReduceThreads) s_row[i] = 0;
        __syncthreads();
        // general partials are [slice][instance][bucket], windowed ones [instance][slice][bucket of the window]
        const int32_t* rk = windowed ? wpartial + (int64_t)k * n_rows * row_len : partial + (int64_t)k * row_len;
        const int64_t rstride = windowed ? (int64_t)row_len : (int64_t)n_inst * row_len;
        const int total = n_rows * row_len;                   // at most 256 * 4096
        const float inv_len = 1.0f / (float)row_len;
        if ((row_len & 3) == 0) {
            // rows of whole 16-byte groups (every row then starts on a 16-byte boundary): four cells a load,
            // all of a thread's loads requested before the first is used
            const int groups = row_len >> 2, total4 = n_rows * groups;
            const float inv_groups = 1.0f / (float)groups;
            constexpr int NB = 12;
            for (int e0 = tid; e0 < total4; e0 += kReduceThreads * NB) {
                int4 v[NB];
                int cell[NB];
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const int e = min(e0 + kReduceThreads * u, total4 - 1);
                    int sl = (int)(((float)e + 0.5f) * inv_groups);
                    int g4 = e - sl * groups;
                    if (g4 < 0) { g4 += groups; --sl; }
                    if (g4 >= groups) { g4 -= groups; ++sl; }
                    v[u] = *(const int4*)(rk + sl * rstride + 4 * g4);
                    const int a0 = s_origin[sl];              // -1: a slice that added nothing
                    cell[u] = (e0 + kReduceThreads * u < total4 && a0 >= 0) ? a0 + 4 * g4 : -1;
                }
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    if (cell[u] < 0) continue;
                    const int x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (x[c] != 0 && cell[u] + c < horizon) atomicAdd(&s_row[cell[u] + c], (unsigned long long)(long long)x[c]);
                }
            }
        } else {
            constexpr int NB = 16;                            // loads requested before the first is used
            for (int e0 = tid; e0 < total; e0 += kReduceThreads * NB) {
                int32_t v[NB];
                int cell[NB];
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const int e = min(e0 + kReduceThreads * u, total - 1);
                    int sl = (int)(((float)e + 0.5f) * inv_len);
                    int i = e - sl * row_len;
                    if (i < 0) { i += row_len; --sl; }
                    if (i >= row_len) { i -= row_len; ++sl; }
                    v[u] = rk[sl * rstride + i];
                    const int a0 = s_origin[sl];              // -1: a slice that added nothing
                    cell[u] = (e0 + kReduceThreads * u < total && a0 >= 0 && a0 + i < horizon) ? a0 + i : -1;
                }
#pragma unroll
                for (int u = 0; u < NB; ++u)
                    if (cell[u] >= 0 && v[u] != 0) atomicAdd(&s_row[cell[u]], (unsigned long long)(long long)v[u]);
            }
        }
        __syncthreads();
    }
    const int64_t stride = (int64_t)n_inst * horizon;
    const int32_t* prow = partial + (int64_t)k * horizon;
    int32_t* lrow = load + (int64_t)k * horizon;
    const bool worker = tid < 256;                            // the scan is the first four wavefronts' work
    long long carry = 0;
    for (int b0 = 0; b0 < horizon; b0 += 1024) {
        const int b = b0 + 4 * (tid & 255);
        long long v[4] = {0, 0, 0, 0};
        if (worker) {
            if (in_lds) {
#pragma unroll
                for (int c = 0; c < 4; ++c) if (b + c < horizon) v[c] = (long long)s_row[b + c];
            } else {
                int s = 0;
                for (; s + 4 <= slices; s += 4) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int32_t* p = prow + (s + u) * stride;
#pragma unroll
                        for (int c = 0; c < 4; ++c) if (b + c < horizon) v[c] += p[b + c];
                    }
                }
                for (; s < slices; ++s) {
                    const int32_t* p = prow + s * stride;
#pragma unroll
                    for (int c = 0; c < 4; ++c) if (b + c < horizon) v[c] += p[b + c];
                }
            }
        }
        v[1] += v[0]; v[2] += v[1]; v[3] += v[2];
        // inclusive scan of the thread totals: within a wavefront by shuffles, then across the four
        long long incl = v[3];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const long long t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        if (worker && lane == 63) s_wave[wave] = incl;
        __syncthreads();
        long long before = carry + incl - v[3];
        for (int w = 0; w < (wave & 3); ++w) before += s_wave[w];
        const long long total = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
        if (worker) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (b + c < horizon) {
                    const long long nv = (long long)lrow[b + c] + before + v[c];
                    if (nv > 2147483647ll || nv < -2147483648ll) report_fault(st, PS_ST_RANGE, -1);
                    lrow[b + c] = (int32_t)(uint32_t)(unsigned long long)nv;
                }
            }
        }
        carry += total;
        __syncthreads();
    }
    // tokens past the horizon: one slice per thread, added up in LDS
    if (overflow) {
        const int n_rows = windowed ? w_slices : slices;
        for (int s2 = tid; s2 < n_rows; s2 += kReduceThreads) {
            long long o = 0;
            if (windowed) {
                if (!(worigin[s2] & kNothing)) o = wovf[(int64_t)s2 * n_inst + k];
            } else {
                o = partial_ovf[(int64_t)s2 * n_inst + k];
            }
            if (o) atomicAdd(&s_over, (unsigned long long)o);
        }
        __syncthreads();
        if (tid == 0 && s_over) overflow[k] += (long long)s_over;
    }
}

// ---- short calls ------------------------------------------------------------------------------------------
// A management period's batch is a few thousand records: one launch and no partial curves.  A workgroup per instance
// looks through the batch's instances (eight ids a thread requested together), applies its own records to an LDS row
// of differences and adds the row's prefix sums to the map.  At most 2^14 records of at most 2^16 tokens: no cell can
// leave 32 bits.  The slices of the general form keep LDS rows for 65 instances each and hand 256 x 600 counters
// over through memory: 8 us and 6 us for 4096 records.  The map's row and the first ids are requested ahead of all else, sums go
// by lane moves: 4096 records over 256 x 600 5.9 -> 4.8 us a call.
//
// Microseconds, the general form / this one: 16384 records over 8 and 64 instances of 600 buckets 19 / 14 and 21 / 12,
// 4096 over 1024 30 / 12, 64 over 65536 instances of 48 buckets 1105 / 340.  Where hundreds of records meet in one cell
// the atomics of its only copy queue up: 16384 records over 1 instance of 16, 48 and 100 buckets 21 / 32, 17 / 19 and
// 17 / 17, over 4 of 4 buckets 20 / 25, over 8 of 48 19 / 16.
const int64_t kDirectMaxRecords = 16384;
const int64_t kDirectMaxLooks = (int64_t)1 << 23;            // records * instances
const int kDirectMaxHorizon = 16000;                         // the row and the rest fit 64 KB of LDS
bool direct_pays(int64_t n_req, int n_inst, int horizon) {
    return n_req <= kDirectMaxRecords && n_req * n_inst <= kDirectMaxLooks && horizon <= kDirectMaxHorizon &&
           n_req <= 256 * (int64_t)n_inst * horizon;
}
__global__ __launch_bounds__(1024) void anticipate_direct_kernel(
    const int32_t* __restrict__ pred_tokens, const int32_t* __restrict__ instance_id,
    const int32_t* __restrict__ arrival_bucket, const int32_t* __restrict__ rate, int n, int n_inst, int horizon,
    int32_t* __restrict__ load, int64_t* __restrict__ overflow, ps_status* st) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    int* s_diff = (int*)lds_raw;                                // [horizon]
    __shared__ long long s_wave[16];
    __shared__ unsigned long long s_ovf;
    const int k = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the first ids, and the map's row, ahead of all else
    constexpr int U = 8;
    int kk[U];
    auto look = [&](int r0) {
#pragma unroll
        for (int u = 0; u < U; ++u) kk[u] = instance_id[min(r0 + 1024 * u, n - 1)];
    };
    if (n > 0) look(tid);
    const int r_k = rate ? rate[k] : 1;
    int32_t* row = load + (int64_t)k * horizon;
    const int row_first = tid < horizon ? row[tid] : 0;
    asm volatile("" ::: "memory");
    for (int i = tid; i < horizon; i += 1024) s_diff[i] = 0;
    if (tid == 0) s_ovf = 0;
    __syncthreads();
    for (int r0 = tid; r0 < n; r0 += 1024 * U) {
        if (r0 != tid) look(r0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + 1024 * u;
            if (r >= n) continue;
            // an instance outside the map is nobody's: reported by the first workgroup
            if ((unsigned)kk[u] >= (unsigned)n_inst && k == 0) report_fault(st, PS_ST_BAD_RECORD, r);
            if (kk[u] != k) continue;
            const unsigned D = (unsigned)pred_tokens[r], a = (unsigned)arrival_bucket[r];
            if (D > (unsigned)PS_MAX_PRED || a >= (unsigned)horizon || r_k < 1) {
                report_fault(st, PS_ST_BAD_RECORD, r);
                continue;
            }
            if (D == 0) continue;
            const unsigned room = (unsigned)horizon - a;        // buckets from a to the end of the row
            const unsigned rc = (unsigned)min(r_k, PS_MAX_PRED);
            const unsigned dur = rate ? (D + rc - 1u) / rc : room;
            const unsigned q = D / dur, rem = D - q * dur;
            atomicAdd(&s_diff[a], (int)(q + 1));
            if (rem < room) atomicAdd(&s_diff[a + rem], -1);
            if (dur < room) {
                atomicAdd(&s_diff[a + dur], -(int)q);
            } else if (dur > room) {
                atomicAdd(&s_ovf, (unsigned long long)D - ((unsigned long long)room * q + min(room, rem)));
            }
        }
    }
    __syncthreads();
    if (tid == 0 && overflow && s_ovf) overflow[k] += (int64_t)s_ovf;
    long long carry = 0;
    for (int b0 = 0; b0 < horizon; b0 += 1024) {                // a bucket per thread: neighbours read neighbouring words
        const int b = b0 + tid;
        const int was = b0 == 0 ? row_first : b < horizon ? row[b] : 0;
        const long long incl = prefix_sum64(b < horizon ? s_diff[b] : 0);
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        long long total;
        const long long before = carry + sum_in_front(s_wave, wave, total);
        if (b < horizon) {
            const long long nv = was + before + incl;
            if (nv > 2147483647ll || nv < -2147483648ll) report_fault(st, PS_ST_RANGE, -1);
            row[b] = (int32_t)(uint32_t)(unsigned long long)nv;
        }
        carry += total;
        __syncthreads();
    }
}

}  // namespace

extern "C" size_t ps_anticipate_workspace_bytes(int64_t n_req, int32_t n_inst, int32_t horizon) {
    if (n_req < 0 || n_inst < 1 || horizon < 1) return 0;
    AntPlan p = make_plan(n_req, n_inst, horizon);
    plan_window(p, n_req, n_inst, horizon, true);
    return p.ok ? p.total_bytes : 0;
}

namespace {

// Validates the arguments and enqueues the kernels of one call on `s`, with `workspace` (device memory of at
// least `workspace_bytes` bytes) for the partial curves.
int anticipate_enqueue(const int32_t* pred_tokens, const int32_t* instance_id, const int32_t* arrival_bucket,
                       const int32_t* rate, int64_t n_req, int32_t n_inst, int32_t horizon, int32_t* load,
                       int64_t* overflow, void* workspace, size_t workspace_bytes, ps_status* status, hipStream_t s) {
    if (n_req < 0 || n_inst < 1 || horizon < 1 || !load) return PS_EINVAL;
    if (rate && !overflow) return PS_EINVAL;
    if (n_req == 0) return PS_OK;
    if (!pred_tokens || !instance_id || !arrival_bucket || !workspace) return PS_EINVAL;
    if ((((uintptr_t)pred_tokens | (uintptr_t)instance_id | (uintptr_t)arrival_bucket) & 15) != 0) return PS_EINVAL;
    if ((int64_t)n_inst * horizon > (int64_t)0x7fffffff) return PS_EUNSUPPORTED;
    AntPlan p = make_plan(n_req, n_inst, horizon);
    if (!p.ok) return PS_EUNSUPPORTED;
    {
        // the workspace is sized for the windowed path whether or not this call takes it
        AntPlan sized = p;
        plan_window(sized, n_req, n_inst, horizon, true);
        if (((uintptr_t)workspace & 255) != 0 || workspace_bytes < sized.total_bytes) return PS_EWORKSPACE;
    }
    plan_window(p, n_req, n_inst, horizon, rate != nullptr);
    if (((uintptr_t)workspace & 255) != 0 || workspace_bytes < p.total_bytes) return PS_EWORKSPACE;
    (void)hipGetLastError();
    if (direct_pays(n_req, n_inst, horizon)) {
        hipLaunchKernelGGL(anticipate_direct_kernel, dim3((unsigned)n_inst), dim3(1024), (size_t)horizon * 4, s, pred_tokens,
                           instance_id, arrival_bucket, rate, (int)n_req, n_inst, horizon, load, overflow, status);
        return hipGetLastError() == hipSuccess ? PS_OK : PS_EHIP;
    }
    static bool lds_attr_set = false;     // raising the limit twice is harmless, so no lock
    if (!lds_attr_set) {
        if (hipFuncSetAttribute((const void*)anticipate_scatter_kernel,
                                hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void*)anticipate_window_kernel,
                                hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes) != hipSuccess)
            return PS_EHIP;
        lds_attr_set = true;
    }
    plan_halves(p, n_req, n_inst, horizon);
    uint8_t* wsb = (uint8_t*)workspace;
    int32_t* partial = (int32_t*)wsb;
    int64_t* partial_ovf = (int64_t*)(wsb + p.partial_bytes);
    int32_t* wpartial = nullptr;
    int64_t* wovf = nullptr;
    int32_t* worigin = nullptr;
    if (p.w_slices > 0) {
        wpartial = (int32_t*)(wsb + p.w_partial_at);
        wovf = (int64_t*)(wsb + p.w_ovf_at);
        worigin = (int32_t*)(wsb + p.w_origin_at);
        hipLaunchKernelGGL(anticipate_window_kernel, dim3((unsigned)p.w_slices), dim3(kScatterThreads), p.w_lds_bytes, s,
                           pred_tokens, instance_id, arrival_bucket, rate, n_req, n_inst, horizon, p.w_buckets,
                           p.w_slice_len, p.h_slices > 0 ? p.h_weighed : 0, p.h_slice_len, wpartial, wovf, worigin, status);
    }
    HalvesArgs hv = {pred_tokens, instance_id, arrival_bucket, rate, n_req, p.h_slice_len, n_inst, horizon, p.h_rows, p.h_groups,
                     p.h_slices, p.h_stride, 32 - p.h_row_bits, 32 - p.h_row_bits - p.h_bucket_bits, (uint16_t*)wsb,
                     (uint16_t*)(wsb + p.h_high_at), (int64_t*)(wsb + p.h_ovf_at), (int32_t*)(wsb + p.h_flag_at)};
    const GeneralArgs ga = {pred_tokens, instance_id, arrival_bucket, rate, n_req, p.slice_len, n_inst, horizon,
                            p.rows_per_group, p.groups, p.slices, partial, partial_ovf};
    // (which of the two runs is known on the device)
    const unsigned blocks = 8u * (unsigned)p.groups * (unsigned)((p.slices + 7) / 8);
    const unsigned h_blocks = 8u * (unsigned)p.h_groups * (unsigned)((p.h_slices + 7) / 8);
    const bool halves = p.h_slices > 0;
    hipLaunchKernelGGL(anticipate_scatter_kernel, dim3(halves && h_blocks > blocks ? h_blocks : blocks), dim3(kScatterThreads),
                       halves && p.h_lds_bytes > p.lds_bytes ? p.h_lds_bytes : p.lds_bytes, s, ga, hv, worigin, p.w_slices, status);
    hipLaunchKernelGGL(anticipate_reduce_kernel, dim3((unsigned)n_inst), dim3(kReduceThreads), 0, s, partial, partial_ovf, p.slices,
                       n_inst, horizon, wpartial, wovf, worigin, p.w_slices, p.w_buckets, hv, load, overflow, status);
    return hipGetLastError() == hipSuccess ? PS_OK : PS_EHIP;
}

}  // namespace

extern "C" int ps_anticipate(const int32_t* pred_tokens, const int32_t* instance_id,
                             const int32_t* arrival_bucket, const int32_t* rate, int64_t n_req,
                             int32_t n_inst, int32_t horizon, int32_t* load, int64_t* overflow,
                             void* workspace, size_t workspace_bytes, ps_status* status, void* hip_stream) {
    return anticipate_enqueue(pred_tokens, instance_id, arrival_bucket, rate, n_req, n_inst, horizon, load, overflow,
                              workspace, workspace_bytes, status, (hipStream_t)hip_stream);
}

// ---- the variant for callers that cannot allocate ---------------------------------------------------------
// Its partial curves live in a file-scope device array instead of a caller-provided workspace.  Every GPU the
// library runs on holds its own copy of the array at its own address: the address is looked up once per
// device and kept; host code only ever uses that address, never the array's name.
static __device__ __align__(256) unsigned char scratch[PS_ANTICIPATE_STATIC_BYTES];

namespace {
const int kMaxDevices = 64;
std::mutex g_scratch_lock;
void* g_scratch_ptr[kMaxDevices];       // per device: device address of `scratch`, null until looked up
}  // namespace

extern "C" int ps_anticipate_static(const int32_t* pred_tokens, const int32_t* instance_id,
                                    const int32_t* arrival_bucket, const int32_t* rate, int64_t n_req,
                                    int32_t n_inst, int32_t horizon, int32_t* load, int64_t* overflow,
                                    ps_status* status, void* hip_stream) {
    if (n_req < 0 || n_inst < 1 || horizon < 1) return PS_EINVAL;
    // sizes beyond the array are refused before anything else is looked at
    const size_t need = ps_anticipate_workspace_bytes(n_req, n_inst, horizon);
    if (need == 0) return PS_EUNSUPPORTED;
    if (need > (size_t)PS_ANTICIPATE_STATIC_BYTES) return PS_EWORKSPACE;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return PS_EHIP;
    if (dev < 0 || dev >= kMaxDevices) return PS_EUNSUPPORTED;
    void* ptr;
    {
        std::lock_guard<std::mutex> hold(g_scratch_lock);
        if (!g_scratch_ptr[dev]) {
            void* p = nullptr;
            if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return PS_EHIP;
            g_scratch_ptr[dev] = p;
        }
        ptr = g_scratch_ptr[dev];
    }
    // the kernels write every partial cell they later read, so the last call's contents need no clearing
    return anticipate_enqueue(pred_tokens, instance_id, arrival_bucket, rate, n_req, n_inst, horizon, load, overflow,
                              ptr, (size_t)PS_ANTICIPATE_STATIC_BYTES, status, (hipStream_t)hip_stream);
}
