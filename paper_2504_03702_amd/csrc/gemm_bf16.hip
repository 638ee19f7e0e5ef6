// bf16 GEMM on the gfx950 matrix cores with fused epilogues.
//
//   C[m, n] = sum_k A[m, k] * W[n, k]   (A: activations [rows][K], W: weights [N][K], both bf16,
//                                        contraction index contiguous; fp32 accumulation)
//   epilogue: + bias[n], then one of: store | erf-GELU, store | + residual stream, store as hi + lo |
//             QKV split (query and key columns to [rows][2H], value columns transposed to
//             Vt[H][max_rows] so the attention kernel reads keys-contiguous value tiles), also as
//             keys and values only | erf-GELU, store as hi + lo, for an operand that is hi + lo too.
//   A LayerNorm in front of a map is folded into it: the operand is the row before normalisation,
//   W carries the LayerNorm's scale, and the epilogue finishes with the row's (mean, 1/std):
//   rstd * (acc - mean * colsum[n]) + d[n].  The residual epilogues produce such operands: they write
//   the new sums as two bf16 values hi + lo (hi is the operand) and leave per-row partial sums for the
//   statistics.
//
// One workgroup computes a BM x BN tile.  Per 64-deep k slice the A and W sub-tiles are brought
// straight from global memory into LDS (global_load_lds, 16 bytes per lane, no register staging),
// double buffered; each wavefront then reads 32 x 16 fragments with ds_read_b128 and issues
// v_mfma_f32_32x32x16_bf16.  LDS rows are 128 bytes (64 bf16); the 16-byte chunks of a row are
// XOR-swizzled with the row index so that the 8 or 16 rows one ds_read_b128 phase touches fall in
// different banks.  The swizzle is applied on the global side of the DMA (each lane picks which
// chunk it fetches), since the LDS side of a DMA is always lane-linear.
//
// The kernel is persistent: one workgroup per compute unit walks a list of tiles, prefetching the
// first k slices of its next tile while the current one finishes, so only the very first tile pays
// the latency of filling LDS.  The number of rows is only known on the device (padded inputs are
// compacted); each workgroup derives its tile list from it.  Workgroups are dealt to the 8 XCDs
// round-robin by the hardware; the tile list is built so that the tiles in flight on one XCD are
// neighbours that share activation row panels and weight column panels through that XCD's L2.
#include <type_traits>

#include "device_util.h"
#include "internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

#define GLOBAL_AS __attribute__((address_space(1)))
#define LDS_AS __attribute__((address_space(3)))

template <int BM, int BN, int WM, int WN>
struct Tile {
    static_assert(WM == 2, "two rows of wavefronts: the lower one may have fewer blocks");
    static constexpr int NW = WM * WN;               // wavefronts per workgroup
    static constexpr int THREADS = NW * 64;
    static constexpr int TM = BM / WM / 32;          // 32 x 32 accumulator blocks of a wavefront, at most
    static constexpr int TN = BN / WN / 32;
    static constexpr int A_BYTES = BM * 128;         // one 64-deep slice
    static constexpr int B_BYTES = BN * 128;
    static constexpr int STAGE = A_BYTES + B_BYTES;  // an A slice followed by a W slice
    static constexpr int EPI_BYTES = 4096;           // per-wavefront transpose region of the epilogue
    static constexpr int LDS = 2 * STAGE + NW * EPI_BYTES;
    static_assert(NW % 2 == 0 && BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "tile / wave split");
    static_assert(LDS <= 160 * 1024, "LDS budget");
};

// Every DMA of this wavefront has landed, and every wavefront is past its LDS reads.
__device__ __forceinline__ void dma_barrier() {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

struct GemmArgs {
    const bf16_t *A, *W;
    const float* bias;
    ResidualSrc res;
    void* C;
    bf16_t* Vt;
    int64_t max_rows;            // rows of every activation buffer; also the row stride of Vt
    int N, K, hidden;
};

// One region of the output: the rows from row_begin on, in tiles of bm rows (32 for each of the 2 x TM blocks of the two
// rows of wavefronts; wavefront row 0 has tm0 of them, this wavefront TM).
struct Region {
    int row_begin, bm, tm0, m_tiles;
    int rows;                    // rows of the whole problem
};

// The tiles of a region that this workgroup computes.  The grid is persistent.  The hardware deals workgroups to the 8 XCDs
// round-robin, so workgroup b runs on XCD b % 8 as its slot b / 8.  Each XCD has its own L2: the tiles in flight on one XCD
// should share operand panels.  Tiles are numbered in bands of 8 tile rows, column by column within a band (up to 3 columns
// row by row), and in every round of the grid an XCD takes a run of `slots` consecutive numbers.  Columns in P groups of 4
// make a run of 32 an 8 x 4 block, the fewest distinct panels for 32 tiles.  Which run:
//  * P divides 8: the XCDs' runs follow each other, so an XCD keeps its column group for the whole region (4 x 256 rows of
//    W stay in its L2) and the P XCDs that need a band work on it at the same time: it comes from HBM once and from the
//    memory-side cache for the others.
//  * P does not: an XCD takes bands x, x + 8, ... and the P column groups of each in turn.
//  * other column counts: every XCD goes through a range of its own (hidden 768, query-key-value map, 250 k rows: 895 us,
//    row by row 935).
// The tiles of the last round are dealt to the XCDs evenly, so every workgroup gets the same number of tiles to one (P = 3
// in whole bands per XCD, as it used to be: the first feed-forward map of 100 k rows of hidden 768 549 us, 523 so).
// Without BANDS, row by row and a range to each XCD: small tiles, mostly one to a workgroup, where a launch of 27 us shows the
// arithmetic (18 to 26 requests, maps of hidden 768 27.4 us with bands, 26.6 so; keys and values 17.6, 17.1).  4096 requests'
// first feed-forward map of hidden 1024, 1024 of those tiles: 90 us with bands, 101 without.
template <bool BANDS>
struct Walk {
    int n_tiles, m_tiles, slots, xcd, slot, full, rest, n_my;
    __device__ __forceinline__ Walk(int m, int n) : n_tiles(n), m_tiles(m) {
        xcd = blockIdx.x & 7; slot = blockIdx.x >> 3; slots = gridDim.x >> 3;
        const int tiles = m * n;
        full = tiles / (int)gridDim.x;
        rest = tiles - full * (int)gridDim.x;
        const int per = (rest + 7) >> 3;
        n_my = full + (slot < per && xcd * per + slot < rest ? 1 : 0);
    }
    // row and column of this workgroup's tile `round`
    __device__ __forceinline__ void tile(int round, int& tm, int& tn) const {
        int run = xcd * full + round;
        if (BANDS && (n_tiles & 3) == 0) {
            const int P = n_tiles >> 2, done = 8 % P == 0 ? 0 : full / P * P;
            run = round < done ? (round / P * 8 + xcd) * P + round % P : round * 8 + xcd;
        }
        const int id = round < full ? run * slots + slot : full * (int)gridDim.x + xcd * ((rest + 7) >> 3) + slot;
        if constexpr (BANDS) {
            const int high = n_tiles < 4 ? 1 : 8;
            const int band = id / (high * n_tiles), in = id - band * high * n_tiles, rb = min(high, m_tiles - high * band);
            tn = in / rb;
            tm = high * band + in - tn * rb;
        } else {
            tm = id / n_tiles;
            tn = id - tm * n_tiles;
        }
    }
};

// All tiles of a region that belong to this workgroup, by one of its wavefronts; TM: the wavefront's 32-row blocks.
template <typename T, int WN, int TM, int EPI, bool PLANNED>
__device__ __forceinline__ void region_tiles(const GemmArgs& g, const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                             const float* __restrict__ bias, void* __restrict__ Cv, bf16_t* __restrict__ Vt,
                                             const Region& rg_, unsigned char* smem) {
    constexpr int STAGE = T::STAGE, EPI_BYTES = T::EPI_BYTES, BN = 32 * T::TN * WN;
    const ResidualSrc& res = g.res;
    const int64_t vt_ld = g.max_rows;
    const int N = g.N, K = g.K, hidden = g.hidden, rows = rg_.rows;

    // (a copy the compiler takes for new: nothing derived from it is kept across the regions)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    // the wavefront index is uniform; saying so keeps everything derived from it in scalar registers
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int wave_row = wm * rg_.tm0 * 32;                  // the wavefront's first row in a tile

    // (EPI_GELU_SPLIT: small tiles, but many of them for many requests)
    constexpr bool BANDS = PLANNED || EPI == EPI_GELU_SPLIT;
    const Walk<BANDS> walk(rg_.m_tiles, N / BN);
    const int n_my = walk.n_my;
    if (n_my == 0) return;
    // first row of a tile; the last tile is moved up where it would pass the end of the buffers (rows of two tiles are
    // written twice with the same values)
    const int last_m0 = (int)g.max_rows - rg_.bm;
    auto row_of = [&](int tm) { return min(rg_.row_begin + tm * rg_.bm, last_m0); };

    // ---- DMA sources: lane i of a wavefront fetches chunk (i%8)^swz of row i/8 of its group ----
    const int dma_row = wave * 8 + (lane >> 3);
    const int dma_chunk = (lane & 7) ^ lds_swz(dma_row);
    const unsigned lane_off = (unsigned)(dma_row * K + dma_chunk * 8) * 2u;
    const int64_t ld_bytes = (int64_t)K * 2;
    // EPI_GELU_SPLIT: a row of A is hi | lo, both halves meet the same W, whose rows have K / 2 elements.  The halves'
    // sums are kept apart until the last addition (the bits of the small tiles, so a request's prediction does not
    // depend on how many others are in the call); 64 more accumulators, which the 128 x 128 tiles have room for.
    constexpr bool SPLIT = EPI == EPI_GELU_SPLIT;
    const int ldw = SPLIT ? K / 2 : K;
    const unsigned lane_off_w = SPLIT ? (unsigned)(dma_row * ldw + dma_chunk * 8) * 2u : lane_off;
    const int64_t ldw_bytes = SPLIT ? (int64_t)ldw * 2 : ld_bytes;

    // ---- fragment addresses: row (lane%32) of a 32-row tile, chunks 2*ks + lane/32 ----------
    const int frow = lane & 31, fhalf = lane >> 5;
    const int a_off = (wave_row + frow) * 128;
    const int b_off = (wn * (BN / WN) + frow) * 128;
    int koff[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) koff[ks] = ((2 * ks + fhalf) ^ lds_swz(frow)) * 16;

    f32x16 acc[TM][T::TN];
    auto clear_acc = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < T::TN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    };

    // Fragment double buffer: while the MFMAs of k-step s run, the ds_reads of step s+1 are in
    // flight.  The 64-deep slices of all this workgroup's tiles form one stream, slice g living in
    // stage g & 1.  Schedule per slice g:
    //   steps 0..2 : read fragments of the next step of this slice | MFMAs of the current step
    //   then       : wait for this wavefront's DMA of slice g+1, workgroup barrier (now every
    //                wavefront has read its last fragments of slice g and slice g+1 is visible),
    //                start the DMA of slice g+2 into the stage slice g occupied
    //   step 3     : read step-0 fragments of slice g+1 | MFMAs of step 3
    // Slices g+1 and g+2 may belong to the next tile: its first two slices land while this tile
    // finishes and runs its epilogue (which has an LDS region of its own), so a tile starts with
    // its operands already in LDS.
    bf16x8 fa0[TM], fb0[T::TN], fa1[TM], fb1[T::TN];
    auto read_frags = [&](bf16x8* fa, bf16x8* fb, const unsigned char* stage, int ks) {
        const unsigned char* sA = stage + a_off + koff[ks];
        const unsigned char* sB = stage + T::A_BYTES + b_off + koff[ks];
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[i] = *(const bf16x8*)(sA + i * 4096);
#pragma unroll
        for (int j = 0; j < T::TN; ++j) fb[j] = *(const bf16x8*)(sB + j * 4096);
    };
    const int nk = K / 64;
    // Prefetch cursor: the next slice to fetch is slice pf_kt of the tile at (pf_a, pf_w).  It runs up to two slices ahead of
    // the products, so it enters the next tile, at (nx_a, nx_w), while they finish this one.  Once the workgroup's tiles are
    // used up it parks on the region's first tile: the DMAs stay unconditional (straight-line code the scheduler can
    // interleave with the MFMAs) and the parked ones refill LDS stages nobody reads any more.
    int pf_kt = 0, pf_stage = 0, tm, tn;
    walk.tile(0, tm, tn);
    auto a_of = [&](int m) { return (const unsigned char*)(A + (int64_t)row_of(m) * K); };
    auto w_of = [&](int n) { return (const unsigned char*)(W + (int64_t)n * BN * ldw); };
    const unsigned char *pf_a = a_of(tm), *pf_w = w_of(tn), *nx_a = pf_a, *nx_w = pf_w;
    // The DMA of a slice is issued in two halves, A rows then W rows, each spread among the MFMAs of
    // one k-step: a wavefront that queues all of a slice's DMA instructions at once waits at the
    // memory pipeline's issue queue and issues no MFMA meanwhile.
    auto prefetch_a = [&](int j) {        // DMA j of the slice's A rows
        const unsigned char* ub = pf_a + pf_kt * 128 + (int64_t)j * (T::NW * 8) * ld_bytes;    // wave-uniform
        __builtin_amdgcn_global_load_lds((const GLOBAL_AS void*)(ub + lane_off),
                                         (LDS_AS void*)(smem + pf_stage * STAGE + (j * T::NW + wave) * 1024), 16, 0, 0);
    };
    auto prefetch_w = [&](int j) {        // DMA j of the slice's W rows
        int kt = pf_kt;
        if constexpr (SPLIT) kt -= pf_kt < nk / 2 ? 0 : nk / 2;
        const unsigned char* ub = pf_w + kt * 128 + (int64_t)j * (T::NW * 8) * ldw_bytes;
        __builtin_amdgcn_global_load_lds((const GLOBAL_AS void*)(ub + lane_off_w),
                                         (LDS_AS void*)(smem + pf_stage * STAGE + T::A_BYTES + (j * T::NW + wave) * 1024), 16, 0, 0);
    };
    auto advance_cursor = [&]() {         // after the W rows: on to the next slice
        pf_stage ^= 1;
        const bool last = ++pf_kt == nk;
        pf_kt = last ? 0 : pf_kt;
        pf_a = last ? nx_a : pf_a;
        pf_w = last ? nx_w : pf_w;
    };
    // wavefronts of the upper row move as many 8-row groups more as they have blocks more
    constexpr int NDMA_A = TM * 8 / T::NW, NDMA_W = BN / 8 / T::NW;

    // One k-step in exact issue order (the scheduler may not move anything across the fences): in
    // each of TM + TN rounds one fragment read for the next step, at most one DMA, and a share of this
    // step's MFMAs.  dma_tag: 0 none, 1 the slice's A rows, 2 its W rows.
    auto k_step = [&](const bf16x8* fa, const bf16x8* fb, bf16x8* na, bf16x8* nb, const unsigned char* rd_stage,
                      int rd_ks, auto dma_tag) {
        constexpr int DMA = decltype(dma_tag)::value;
        constexpr int nR = TM + T::TN, nM = TM * T::TN;
        static_assert(NDMA_A <= nR && NDMA_W <= nR, "one DMA per round");
        const unsigned char* sA = rd_stage + a_off + koff[rd_ks];
        const unsigned char* sB = rd_stage + T::A_BYTES + b_off + koff[rd_ks];
#pragma unroll
        for (int r = 0; r < nR; ++r) {
            if (r < TM) na[r] = *(const bf16x8*)(sA + r * 4096);
            else nb[r - TM] = *(const bf16x8*)(sB + (r - TM) * 4096);
            if (DMA == 1 && r < NDMA_A) prefetch_a(r);
            if (DMA == 2 && r < NDMA_W) prefetch_w(r);
            // MFMAs [r * nM / nR, (r + 1) * nM / nR) of the step, in row-major order of the wavefront's tiles
#pragma unroll
            for (int m = r * nM / nR; m < (r + 1) * nM / nR; ++m)
                acc[m / T::TN][m % T::TN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[m / T::TN], fb[m % T::TN],
                                                                                   acc[m / T::TN][m % T::TN], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using NoDma = std::integral_constant<int, 0>;
    using ADma = std::integral_constant<int, 1>;
    using WDma = std::integral_constant<int, 2>;

#pragma unroll
    for (int j = 0; j < NDMA_A; ++j) prefetch_a(j);
#pragma unroll
    for (int j = 0; j < NDMA_W; ++j) prefetch_w(j);
    advance_cursor();
    dma_barrier();
#pragma unroll
    for (int j = 0; j < NDMA_A; ++j) prefetch_a(j);
    read_frags(fa0, fb0, smem, 0);
    int stage = 0;
    float* stg = (float*)(smem + 2 * STAGE + wave * EPI_BYTES);
    constexpr int WTN = BN / WN;

    for (int it = 0; it < n_my; ++it) {
        const int m_base = row_of(tm) + wave_row, n0 = tn * BN, n_base = n0 + wn * WTN;
        int tm2, tn2;
        if constexpr (BANDS) {
            walk.tile(it + 1 < n_my ? it + 1 : 0, tm2, tn2);
        } else {                                               // mostly the only one
            tm2 = tm; tn2 = tn;
            if (it + 1 < n_my) walk.tile(it + 1, tm2, tn2);
        }
        nx_a = a_of(tm2);
        nx_w = w_of(tn2);
        tm = tm2;
        tn = tn2;
        auto contract = [&](int slices) {
            clear_acc();
            for (int kt = 0; kt < slices; ++kt) {
                unsigned char* cur = smem + stage * STAGE;
                unsigned char* nxt = smem + (stage ^ 1) * STAGE;
                stage ^= 1;
                k_step(fa0, fb0, fa1, fb1, cur, 1, WDma{});       // + W half of the slice after this one
                advance_cursor();
                k_step(fa1, fb1, fa0, fb0, cur, 2, NoDma{});
                k_step(fa0, fb0, fa1, fb1, cur, 3, NoDma{});
                dma_barrier();
                // reads the step-0 fragments of the next slice, of this tile or of the next one (after the
                // last slice of all: of a stage nobody needs); + A half of the slice two after this one
                k_step(fa1, fb1, fa0, fb0, nxt, 0, ADma{});
            }
        };
        if constexpr (SPLIT) {
            f32x16 hi[TM][T::TN];
            contract(nk / 2);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < T::TN; ++j) hi[i][j] = acc[i][j];
            contract(nk / 2);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < T::TN; ++j) acc[i][j] = hi[i][j] + acc[i][j];
        } else {
            contract(nk);
        }

        // ---- epilogue -----------------------------------------------------------------------------
        // Accumulator element e of tile (i, j) is C[row, col] with row = 32 i + 8 (e / 4) + 4 (lane / 32)
        // + e % 4, col = 32 j + lane % 32: a lane holds one column.  Each wavefront transposes through
        // its private 4 KB of LDS: it writes a strip of accumulators, reads it back with 16 bytes of
        // consecutive output per lane, applies the epilogue there and issues 16-byte global accesses.

        // (a copy of the lane index that the compiler takes for new: what is derived from it is worked out here for every
        // tile, and no register holds it through the contraction)
        int el = lane;
        asm volatile("" : "+v"(el));
        const int ecol = el & 31, ehalf = el >> 5;

        // first value column of this launch's W: after the query and key columns, or after the key columns
        const int v_col0 = EPI == EPI_KV ? hidden : 2 * hidden;
        if ((EPI == EPI_QKV || EPI == EPI_KV) && n0 >= v_col0) {
            // Value columns go to Vt[feature][row].  One 32 x 32 accumulator tile at a time is staged as
            // [32 features][32 rows]; the 16-byte chunks of a feature's rows are XOR-swizzled with the
            // feature index so the 128-byte-strided writes of the 32 lanes spread over the banks.  Read
            // back, a lane holds 8 consecutive rows of one feature: the folded LayerNorm is finished there.
            const int rg = el & 3;
            float cc[T::TN][2], dd[T::TN][2];
#pragma unroll
            for (int j = 0; j < T::TN; ++j)
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const int c = n_base + 32 * j + (el >> 2) + 16 * it;
                    cc[j][it] = res.colsum[c];
                    dd[j][it] = bias[c];
                }
            float2 sv[8];                            // statistics of the lane's 8 rows of block i
            auto fetch_sv = [&](int i) {
#pragma unroll
                for (int r = 0; r < 8; ++r) sv[r] = res.stats[m_base + 32 * i + 8 * rg + r];
            };
            fetch_sv(0);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                float rs[8], nm[8];
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    rs[r] = sv[r].y;
                    nm[r] = -sv[r].x * sv[r].y;
                }
                if (i + 1 < TM) fetch_sv(i + 1);
#pragma unroll
                for (int j = 0; j < T::TN; ++j) {
#pragma unroll
                    for (int e4 = 0; e4 < 4; ++e4) {
                        const f32x16& a = acc[i][j];
                        *(float4*)(stg + ecol * 32 + 4 * ((2 * e4 + ehalf) ^ (ecol & 7))) =
                            make_float4(a[4 * e4], a[4 * e4 + 1], a[4 * e4 + 2], a[4 * e4 + 3]);
                    }
#pragma unroll
                    for (int it = 0; it < 2; ++it) {
                        const int c = (el >> 2) + 16 * it;
                        const float4 lo = *(const float4*)(stg + c * 32 + 4 * ((2 * rg) ^ (c & 7)));
                        const float4 hi = *(const float4*)(stg + c * 32 + 4 * ((2 * rg + 1) ^ (c & 7)));
                        const float a8[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                        float v[8];
#pragma unroll
                        for (int r = 0; r < 8; ++r) v[r] = fmaf(a8[r], rs[r], fmaf(nm[r], cc[j][it], dd[j][it]));
                        const uint4 o = make_uint4(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]),
                                                   cvt_pk_bf16(v[4], v[5]), cvt_pk_bf16(v[6], v[7]));
                        *(uint4*)(Vt + (int64_t)(n_base - v_col0 + 32 * j + c) * vt_ld + m_base + 32 * i + 8 * rg) = o;
                    }
                }
            }
            continue;
        }

        // other epilogues: strips of 8 rows x WTN columns, row-major, padded rows
        constexpr int SW = WTN + 4;
        static_assert(8 * SW * 4 <= EPI_BYTES && 32 * 32 * 4 <= EPI_BYTES, "epilogue staging region");
        auto stage_strip = [&](int i, int e4) {      // rows 32 i + 8 e4 + 0..7 of the wavefront's tile
#pragma unroll
            for (int j = 0; j < T::TN; ++j)
#pragma unroll
                for (int t = 0; t < 4; ++t) stg[(4 * ehalf + t) * SW + 32 * j + ecol] = acc[i][j][4 * e4 + t];
        };

        if (EPI == EPI_BIAS_RESIDUAL) {
            // New sums of the residual stream: v = acc + bias + LayerNorm(y_prev) recomputed from the
            // previous sums (kept as two bf16, hi + lo) and the row statistics, so the stream is never
            // rounded to 8 bits.  v goes out as hi + lo again: hi is what the next map reads.  A lane
            // handles 8 consecutive columns (16-byte accesses), 8 lanes a row of the strip.
            constexpr int LPR = WTN / 8, RPI = 64 / LPR, NIT = 8 / RPI, NS = 4 * TM;
            static_assert(LPR == 8 && NIT == 1, "8 lanes per 64-column row piece");
            const int cg = el % LPR, r_in = el / LPR;
            const int col = n_base + 8 * cg;
            float bv[8], rg[8], rb[8];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float4 b4 = *(const float4*)(bias + col + 4 * h);
                const float4 g4 = *(const float4*)(res.gamma + col + 4 * h);
                const float4 e4 = *(const float4*)(res.beta + col + 4 * h);
                bv[4 * h] = b4.x; bv[4 * h + 1] = b4.y; bv[4 * h + 2] = b4.z; bv[4 * h + 3] = b4.w;
                rg[4 * h] = g4.x; rg[4 * h + 1] = g4.y; rg[4 * h + 2] = g4.z; rg[4 * h + 3] = g4.w;
                rb[4 * h] = e4.x; rb[4 * h + 1] = e4.y; rb[4 * h + 2] = e4.z; rb[4 * h + 3] = e4.w;
            }
            bf16_t* Cl = (bf16_t*)Cv;
            const int piece = n_base >> 6, pieces = N >> 6;
            // one row of a strip: combine, store hi and lo, and (where asked for) leave the 64-column
            // piece's sum and sum of squares, added up over the row's 8 lanes
            auto finish_row = [&](int r, const uint4& h, const uint4& l, const float2& st, int64_t row, bool live) {
                const float4 a0 = *(const float4*)(stg + r * SW + 8 * cg);
                const float4 a1 = *(const float4*)(stg + r * SW + 8 * cg + 4);
                const float a[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
                const uint32_t hw[4] = {h.x, h.y, h.z, h.w}, lw[4] = {l.x, l.y, l.z, l.w};
                float o[8];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float y0 = __uint_as_float(hw[t] << 16) + __uint_as_float(lw[t] << 16);
                    const float y1 = __uint_as_float(hw[t] & 0xffff0000u) + __uint_as_float(lw[t] & 0xffff0000u);
                    o[2 * t] = a[2 * t] + bv[2 * t] + ((y0 - st.x) * st.y * rg[2 * t] + rb[2 * t]);
                    o[2 * t + 1] = a[2 * t + 1] + bv[2 * t + 1] + ((y1 - st.x) * st.y * rg[2 * t + 1] + rb[2 * t + 1]);
                }
                float sm = 0.f, sq = 0.f;
                if (res.pstats) {
                    sm = ((o[0] + o[1]) + (o[2] + o[3])) + ((o[4] + o[5]) + (o[6] + o[7]));
                    sq = (fmaf(o[0], o[0], o[1] * o[1]) + fmaf(o[2], o[2], o[3] * o[3])) +
                         (fmaf(o[4], o[4], o[5] * o[5]) + fmaf(o[6], o[6], o[7] * o[7]));
                    sm = row8_sum(sm);
                    sq = row8_sum(sq);
                }
                if (live) {
                    uint32_t ho[4], lo[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        ho[t] = cvt_pk_bf16(o[2 * t], o[2 * t + 1]);
                        lo[t] = cvt_pk_bf16(o[2 * t] - __uint_as_float(ho[t] << 16),
                                            o[2 * t + 1] - __uint_as_float(ho[t] & 0xffff0000u));
                    }
                    *(uint4*)(res.x_out + row * N + col) = make_uint4(ho[0], ho[1], ho[2], ho[3]);
                    *(uint4*)(Cl + row * N + col) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
                    if (res.pstats && cg == 0) res.pstats[row * pieces + piece] = make_float2(sm, sq);
                }
            };
            // The previous sums and statistics of strip s + D are requested before strip s is worked
            // on, so the strips do not each wait out a trip to memory.  Strip s covers rows
            // 8 s .. 8 s + 7 of the wavefront's tile.
            constexpr int D = 3;
            const int64_t row0 = m_base + r_in;
            const bf16_t* yh = res.y_hi + row0 * N + col;
            const bf16_t* yl = res.y_lo + row0 * N + col;
            const float2* sb = res.stats + row0;
            uint4 ph[D + 1], pl[D + 1];
            float2 st[D + 1];
            auto fetch = [&](int s) {
                ph[s % (D + 1)] = *(const uint4*)(yh + (int64_t)(8 * s) * N);
                pl[s % (D + 1)] = *(const uint4*)(yl + (int64_t)(8 * s) * N);
                st[s % (D + 1)] = sb[8 * s];
            };
#pragma unroll
            for (int s = 0; s < D; ++s) fetch(s);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                if (s + D < NS) fetch(s + D);
                stage_strip(s / 4, s % 4);
                const int64_t row = row0 + 8 * s;
                finish_row(r_in, ph[s % (D + 1)], pl[s % (D + 1)], st[s % (D + 1)], row, row < rows);
            }
            continue;
        }

        {
            // bf16 out (plain, GELU, or the query / key columns of the QKV projection): 8 columns per lane
            constexpr int LPR = WTN / 8, RPI = 64 / LPR, NIT = 8 / RPI;
            const int cg = el % LPR, r_in = el / LPR;
            const int col = n_base + 8 * cg;
            const float4 b0 = *(const float4*)(bias + col), b1 = *(const float4*)(bias + col + 4);
            // maps with a LayerNorm folded in: column sums, and the statistics of every row this lane
            // will touch, requested before the first strip
            constexpr bool FOLD = EPI == EPI_QKV || EPI == EPI_KV || EPI == EPI_BIAS_GELU;
            float4 c0 = make_float4(0.f, 0.f, 0.f, 0.f), c1 = c0;
            float2 rst[FOLD ? TM * 4 * NIT : 1];
            if (FOLD) {
                c0 = *(const float4*)(res.colsum + col);
                c1 = *(const float4*)(res.colsum + col + 4);
#pragma unroll
                for (int s = 0; s < TM * 4; ++s)
#pragma unroll
                    for (int it = 0; it < NIT; ++it) {
                        const int64_t row = m_base + 8 * s + r_in + RPI * it;
                        rst[s * NIT + it] = res.stats[row];
                    }
            }
            const int64_t ldc = (EPI == EPI_QKV || EPI == EPI_KV) ? 2 * (int64_t)hidden
                                : SPLIT ? 2 * (int64_t)N : (int64_t)N;
            const int c_col = col + (EPI == EPI_KV ? hidden : 0);   // key columns sit after the query columns
            bf16_t* C = (bf16_t*)Cv;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int e4 = 0; e4 < 4; ++e4) {
                    stage_strip(i, e4);
#pragma unroll
                    for (int it = 0; it < NIT; ++it) {
                        const int r = r_in + RPI * it;
                        const int64_t row = m_base + 32 * i + 8 * e4 + r;
                        const float4 lo = *(const float4*)(stg + r * SW + 8 * cg);
                        const float4 hi = *(const float4*)(stg + r * SW + 8 * cg + 4);
                        float v[8];
                        if (FOLD) {
                            const float2 st = rst[(4 * i + e4) * NIT + it];
                            const float nm = -st.x * st.y;
                            v[0] = fmaf(lo.x, st.y, fmaf(nm, c0.x, b0.x)); v[1] = fmaf(lo.y, st.y, fmaf(nm, c0.y, b0.y));
                            v[2] = fmaf(lo.z, st.y, fmaf(nm, c0.z, b0.z)); v[3] = fmaf(lo.w, st.y, fmaf(nm, c0.w, b0.w));
                            v[4] = fmaf(hi.x, st.y, fmaf(nm, c1.x, b1.x)); v[5] = fmaf(hi.y, st.y, fmaf(nm, c1.y, b1.y));
                            v[6] = fmaf(hi.z, st.y, fmaf(nm, c1.z, b1.z)); v[7] = fmaf(hi.w, st.y, fmaf(nm, c1.w, b1.w));
                        } else {
                            v[0] = lo.x + b0.x; v[1] = lo.y + b0.y; v[2] = lo.z + b0.z; v[3] = lo.w + b0.w;
                            v[4] = hi.x + b1.x; v[5] = hi.y + b1.y; v[6] = hi.z + b1.z; v[7] = hi.w + b1.w;
                        }
                        if (EPI == EPI_BIAS_GELU || SPLIT) {
#pragma unroll
                            for (int e = 0; e < 8; ++e) v[e] = gelu_erf(v[e]);
                        }
                        const uint4 o = make_uint4(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]),
                                                   cvt_pk_bf16(v[4], v[5]), cvt_pk_bf16(v[6], v[7]));
                        *(uint4*)(C + row * ldc + c_col) = o;
                        if constexpr (SPLIT) {
                            // second half of the row: what the first rounding lost, as bf16 again
                            const uint32_t h[4] = {o.x, o.y, o.z, o.w};
                            uint32_t l[4];
#pragma unroll
                            for (int t = 0; t < 4; ++t)
                                l[t] = cvt_pk_bf16(v[2 * t] - __uint_as_float(h[t] << 16),
                                                   v[2 * t + 1] - __uint_as_float(h[t] & 0xffff0000u));
                            *(uint4*)(C + row * ldc + N + c_col) = make_uint4(l[0], l[1], l[2], l[3]);
                        }
                    }
                }
        }
    }
    // parked DMAs may still be in flight: they must land before the workgroup gives up its LDS
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Rows in two regions: plan->m_tiles tiles of BM rows, then the others in tiles of 32 (tm0 + tm1) rows, as prep chose them
// (PLANNED); without a plan all in tiles of BM rows.
template <int BM, int BN, int WM, int WN, int EPI, bool PLANNED>
__global__ __launch_bounds__(WM * WN * 64) void gemm_bf16_kernel(GemmArgs g, const int32_t* __restrict__ total_rows,
                                                                 const GemmPlan* __restrict__ plan, int64_t* __restrict__ clk) {
    using T = Tile<BM, BN, WM, WN>;
    __shared__ __align__(1024) unsigned char smem[T::LDS];
    // clock probe (profiling only): core cycles and constant-rate ticks over this workgroup's life
    const int64_t clk_c0 = clk ? (int64_t)clock64() : 0, clk_w0 = clk ? (int64_t)wall_clock64() : 0;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Region rg;
    rg.rows = *total_rows;
    if constexpr (!PLANNED) {
        rg.row_begin = 0; rg.bm = BM; rg.tm0 = T::TM;
        rg.m_tiles = (rg.rows + BM - 1) / BM;
        region_tiles<T, WN, T::TM, EPI, false>(g, g.A, g.W, g.bias, g.C, g.Vt, rg, smem);
    } else {
        static_assert(T::TM == 4, "regions of 2 to 4 blocks a wavefront");
        const GemmPlan pl = *plan;
        for (int r = pl.m_tiles > 0 ? 0 : 1; r < 2; ++r) {
            const int tm0 = r == 0 ? T::TM : pl.tm0, tm1 = r == 0 ? T::TM : pl.tm1;
            rg.row_begin = r == 0 ? 0 : pl.m_tiles * BM;
            rg.bm = 32 * (tm0 + tm1); rg.tm0 = tm0;
            rg.m_tiles = r == 0 ? pl.m_tiles : (rg.rows - rg.row_begin + rg.bm - 1) / rg.bm;
            if (rg.m_tiles <= 0) break;
            if (r == 1 && pl.m_tiles > 0) dma_barrier();     // every wavefront's parked DMAs have landed
            const int tm = wave / WN == 0 ? tm0 : tm1;       // both paths meet the same barriers
            if (tm == 4) region_tiles<T, WN, 4, EPI, true>(g, g.A, g.W, g.bias, g.C, g.Vt, rg, smem);
            else if (tm == 3) region_tiles<T, WN, 3, EPI, true>(g, g.A, g.W, g.bias, g.C, g.Vt, rg, smem);
            else region_tiles<T, WN, 2, EPI, true>(g, g.A, g.W, g.bias, g.C, g.Vt, rg, smem);
        }
    }
    if (clk && blockIdx.x == 0 && threadIdx.x == 0) {
        clk[0] = (int64_t)clock64() - clk_c0;
        clk[1] = (int64_t)wall_clock64() - clk_w0;
    }
}

template <int BM, int BN, int WM, int WN, bool PLANNED>
void launch_cfg(GemmEpilogue epi, const GemmArgs& g, const int32_t* total_rows, const GemmPlan* plan, int64_t* clk,
                hipStream_t s) {
    // persistent: one workgroup per compute unit; the small tiles leave room for two (LDS and registers), which then hide
    // each other's waits, and take fewer workgroups if there cannot be that many tiles
    const int64_t tiles = (g.max_rows + BM - 1) / BM * (g.N / BN);
    const int64_t wgs = PLANNED ? 256 : tiles < 512 ? (tiles + 7) / 8 * 8 : 512;
    const dim3 grid((unsigned)wgs), block(WM * WN * 64);
#define PS_LAUNCH(E) hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WM, WN, E, PLANNED>), grid, block, 0, s, g, total_rows, plan, clk)
    switch (epi) {
        case EPI_BIAS: PS_LAUNCH(EPI_BIAS); break;
        case EPI_BIAS_GELU: PS_LAUNCH(EPI_BIAS_GELU); break;
        case EPI_BIAS_RESIDUAL: PS_LAUNCH(EPI_BIAS_RESIDUAL); break;
        case EPI_QKV: PS_LAUNCH(EPI_QKV); break;
        case EPI_KV: PS_LAUNCH(EPI_KV); break;
        case EPI_GELU_SPLIT:
            if constexpr (!PLANNED) PS_LAUNCH(EPI_GELU_SPLIT);
            break;
        default: break;                                  // the mapped forms are small_gemm.hip's and skinny_gemm.hip's
    }
#undef PS_LAUNCH
}

}  // namespace

// Requirements (checked when the model is loaded): N % 256 == 0, K % 64 == 0; every buffer holds max_rows rows with
// max_rows % 256 == 0.  Tiles of 128 and 256 rows are then always in bounds; those of other heights may reach past the end
// and are moved up (row_of).
void launch_gemm_bf16(GemmEpilogue epi, const bf16_t* A, const bf16_t* W, const float* bias,
                      ResidualSrc residual, void* C, bf16_t* vt, int64_t max_rows, int N, int K,
                      int hidden, const int32_t* total_rows, const GemmPlan* plan, int64_t* clk, hipStream_t s) {
    // Problems with few 256 x 256 tiles (whole calls on a micro-batch of a few requests) would leave most compute
    // units idle: 128 x 128 tiles give four times as many workgroups to spread them over.  EPI_GELU_SPLIT has only these
    // (its second set of accumulators): 4096 requests of hidden 768 in 57 us, 20000 in 234.
    const int64_t big_tiles = (max_rows + 255) / 256 * (N / 256);
    const GemmArgs g = {A, W, bias, residual, C, vt, max_rows, N, K, hidden};
    if (epi == EPI_GELU_SPLIT || big_tiles < 128)
        launch_cfg<128, 128, 2, 2, false>(epi, g, total_rows, nullptr, clk, s);
    else
        launch_cfg<256, 256, 2, 4, true>(epi, g, total_rows, plan, clk, s);
}
