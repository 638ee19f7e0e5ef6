// bf16 GEMM on the gfx950 matrix cores with fused epilogues.
//
//   C[m, n] = sum_k A[m, k] * W[n, k]   (A: activations [rows][K], W: weights [N][K], both bf16,
//                                        contraction index contiguous; fp32 accumulation)
//   epilogue: + bias[n], then one of: erf-GELU, store | + residual stream, store in two halves |
//             QKV split (query and key columns to [rows][2H], value columns transposed to
//             Vt[H][max_rows] so the attention kernel reads keys-contiguous value tiles), also as
//             keys and values only | erf-GELU, store as hi + lo, for an operand that is hi + lo too.
//   A LayerNorm in front of a map is folded into it: the operand is the row before normalisation,
//   W carries the LayerNorm's scale, and the epilogue finishes with the row's (mean, 1/std):
//   rstd * (acc - mean * colsum[n]) + d[n].  The residual epilogues produce such operands: they write
//   the new sums in two halves (hi, rounded to bf16, is the operand) and leave per-row partial sums for the
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
#include <limits.h>

#include <type_traits>

#include "device_util.h"
#include "internal.h"
#include "skinny_gemm.h"
#include "small_gemm.h"

namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

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
    // what the epilogue needs of a tile's columns (three arrays of floats) and rows (their statistics)
    static constexpr int COLS = 2 * STAGE, ROWS = COLS + 3 * BN * 4;
    static constexpr int STRIPS = ROWS + BM * 8;
    // residual epilogue: a wavefront's strip of 8 rows x 64 columns of floats, rows padded
    static constexpr int STRIP_LD = 68, LDS = STRIPS + NW * 8 * STRIP_LD * 4;
    static_assert(2 * BN <= 512 && BM <= 128 * (NW - 3), "a wavefront fetches an array of the columns, or 128 rows' statistics");
    static_assert(NW % 2 == 0 && BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "tile / wave split");
    static_assert(LDS <= 160 * 1024, "LDS budget");
};

// Every DMA of this wavefront has landed, and every wavefront is past its LDS reads.
__device__ __forceinline__ void dma_barrier() {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The 16-row groups of both operands are stored in LDS with row bits 2 and 3 exchanged, so that an accumulator's lane and
// register indexes stand for these rows and columns: see `epilogue`.
__device__ __forceinline__ int swap23(int r) { return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1); }

struct GemmArgs {
    const bf16_t *A, *W;
    const float* bias;
    ResidualSrc res;
    void* C;
    bf16_t* Vt;
    int64_t max_rows;            // rows of every activation buffer; also the row stride of Vt
    int N, K, hidden;
    int wgs;                     // workgroups of the map itself
    int ahead;                   // workgroups of a side map in front of them in the grid, a multiple of 8
    const uint8_t* first_row;    // rows that a side map writes (1), for the kernels that carry one
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
    int n_tiles, m_tiles, wgs, slots, xcd, slot, full, rest, n_my;
    __device__ __forceinline__ Walk(int m, int n, int wgs_, int wg) : n_tiles(n), m_tiles(m), wgs(wgs_) {
        xcd = wg & 7; slot = wg >> 3; slots = wgs >> 3;
        const int tiles = m * n;
        full = tiles / wgs;
        rest = tiles - full * wgs;
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
        const int id = round < full ? run * slots + slot : full * wgs + xcd * ((rest + 7) >> 3) + slot;
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
template <typename T, int WN, int TM, int EPI, bool PLANNED, bool SKIP, bool AHEAD>
__device__ __forceinline__ void region_tiles(const GemmArgs& g, const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                             const float* __restrict__ bias, void* __restrict__ Cv, bf16_t* __restrict__ Vt,
                                             const Region& rg_, unsigned char* smem) {
    constexpr int STAGE = T::STAGE, BN = 32 * T::TN * WN;
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
    const Walk<BANDS> walk(rg_.m_tiles, N / BN, g.wgs, blockIdx.x - (AHEAD ? g.ahead : 0));
    const int n_my = walk.n_my;
    if (n_my == 0) return;
    // first row of a tile; the last tile is moved up where it would pass the end of the buffers (rows of two tiles are
    // written twice with the same values)
    const int last_m0 = (int)g.max_rows - rg_.bm;
    auto row_of = [&](int tm) { return min(rg_.row_begin + tm * rg_.bm, last_m0); };

    // ---- DMA sources: lane i of a wavefront fetches chunk (i%8)^swz of row i/8 of its group ----
    const int dma_row = wave * 8 + (lane >> 3);
    const int dma_chunk = (lane & 7) ^ lds_swz(dma_row);
    const int src_row = swap23(dma_row);                     // (the DMAs of a slice are multiples of 32 rows apart)
    const unsigned dma_off = (unsigned)(src_row * K + dma_chunk * 8) * 2u;
    const int64_t ld_bytes = (int64_t)K * 2;
    // EPI_GELU_SPLIT: a row of A is hi | lo, both halves meet the same W, whose rows have K / 2 elements.  The halves'
    // sums are kept apart until the last addition (the bits of the small tiles, so a request's prediction does not
    // depend on how many others are in the call); 64 more accumulators, which the 128 x 128 tiles have room for.
    constexpr bool SPLIT = EPI == EPI_GELU_SPLIT;
    const int ldw = SPLIT ? K / 2 : K;
    const unsigned dma_off_w = SPLIT ? (unsigned)(src_row * ldw + dma_chunk * 8) * 2u : dma_off;
    const int64_t ldw_bytes = SPLIT ? (int64_t)ldw * 2 : ld_bytes;

    // ---- fragment addresses: row (lane%32) of a 32-row tile, chunks 2*ks + lane/32 ----------
    const int frow = lane & 31, fhalf = lane >> 5;
    const int a_off = (wave_row + frow) * 128;
    const int b_off = (wn * (BN / WN) + frow) * 128;
    int koff[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) koff[ks] = ((2 * ks + fhalf) ^ lds_swz(frow)) * 16;

    // SWAP: the product transposed, C^T = W A^T: a lane holds one row and, in its registers, columns
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
        __builtin_amdgcn_global_load_lds((const GLOBAL_AS void*)(ub + dma_off),
                                         (LDS_AS void*)(smem + pf_stage * STAGE + (j * T::NW + wave) * 1024), 16, 0, 0);
    };
    auto prefetch_w = [&](int j) {        // DMA j of the slice's W rows
        int kt = pf_kt;
        if constexpr (SPLIT) kt -= pf_kt < nk / 2 ? 0 : nk / 2;
        const unsigned char* ub = pf_w + kt * 128 + (int64_t)j * (T::NW * 8) * ldw_bytes;
        __builtin_amdgcn_global_load_lds((const GLOBAL_AS void*)(ub + dma_off_w),
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
                      int rd_ks, auto dma_tag, auto swap_tag) {
        constexpr int DMA = decltype(dma_tag)::value;
        constexpr bool SWAP = decltype(swap_tag)::value;
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
                acc[m / T::TN][m % T::TN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    SWAP ? fb[m % T::TN] : fa[m / T::TN], SWAP ? fa[m / T::TN] : fb[m % T::TN], acc[m / T::TN][m % T::TN], 0, 0, 0);
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
    constexpr int WTN = BN / WN;
    static_assert(WTN == 64 && T::TN == 2, "64 columns to a wavefront: one piece of the partial row sums");
    // maps with a LayerNorm folded in: column sums of the weights and statistics of the rows
    constexpr bool FOLD = EPI == EPI_QKV || EPI == EPI_KV || EPI == EPI_BIAS_GELU;
    constexpr bool RESIDUAL = EPI == EPI_BIAS_RESIDUAL;
    const float* col_bias = (const float*)(smem + T::COLS);
    const float *col_1 = col_bias + BN, *col_2 = col_bias + 2 * BN;        // column sums, or gamma and beta
    const float2* row_stats = (const float2*)(smem + T::ROWS);

    for (int it = 0; it < n_my; ++it) {
        const int m0 = row_of(tm), m_base = m0 + wave_row, n0 = tn * BN, n_base = n0 + wn * WTN;
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
        // What the epilogue needs of the tile's columns and rows goes to LDS by DMA behind the tile's first barrier (every
        // wavefront is past the last tile's epilogue) and has landed at the second one, two slices or more before it is read
        // (hidden 256 has four): read from memory there it came behind the DMAs of the next tile's slices, which the memory counter keeps in order.
        auto fetch_params = [&]() {
            const float* src = wave == 0 ? bias : wave == 1 ? (FOLD ? res.colsum : res.gamma) : res.beta;
            if (wave == 0 || (wave == 1 && (FOLD || RESIDUAL)) || (wave == 2 && RESIDUAL)) {
                if (lane < BN / 4)
                    __builtin_amdgcn_global_load_lds((const GLOBAL_AS void*)(src + n0 + 4 * lane),
                                                     (LDS_AS void*)(smem + T::COLS + wave * BN * 4), 16, 0, 0);
            } else if ((FOLD || RESIDUAL) && wave >= 3 && wave < 3 + (32 * T::TM * 2) / 128) {
                // two rows a lane; a lower tile's rows end earlier
                const int r = min((wave - 3) * 128 + 2 * lane, rg_.bm - 2);
                __builtin_amdgcn_global_load_lds((const GLOBAL_AS void*)(res.stats + m0 + r),
                                                 (LDS_AS void*)(smem + T::ROWS + (wave - 3) * 1024), 16, 0, 0);
            }
        };
        // Residual epilogue: strip s covers rows 16 (s / 2) + 4 (s % 2) + {0..3, 8..11} of the wavefront's tile; lane l handles
        // 8 columns from 8 (l % 8) of row l / 8 of a strip.  The previous sums of the first D strips are requested a slice
        // ahead of the epilogue, those of strip s + D before strip s is worked on.
        constexpr int D = RESIDUAL ? 3 : 1, NS = 4 * TM;
        auto row_in = [](int s) { return 16 * (s >> 1) + 4 * (s & 1); };
        auto lane_row = [](int l) { return ((l >> 3) & 3) + 8 * (l >> 5); };
        u32x4 ph[D + 1], pl[D + 1];
        int first_a = 0, first_b = 0;                             // SKIP: whether rows lane, 64 + lane are a side map's
        auto fetch_sums = [&](int s, int in_tile) {               // in_tile: of the lane's first element in the wavefront's tile
            const int64_t at = (int64_t)(m_base + row_in(s)) * N + n_base;
            ph[s % (D + 1)] = *(const u32x4*)(res.y_hi + at + in_tile);
            pl[s % (D + 1)] = *(const u32x4*)(res.y_lo + at + in_tile);
        };
        auto contract = [&](int slices, auto swap_tag) {
            clear_acc();
            auto slice = [&](int kt) {
                unsigned char* cur = smem + stage * STAGE;
                unsigned char* nxt = smem + (stage ^ 1) * STAGE;
                stage ^= 1;
                k_step(fa0, fb0, fa1, fb1, cur, 1, WDma{}, swap_tag);       // + W half of the slice after this one
                advance_cursor();
                k_step(fa1, fb1, fa0, fb0, cur, 2, NoDma{}, swap_tag);
                k_step(fa0, fb0, fa1, fb1, cur, 3, NoDma{}, swap_tag);
                dma_barrier();
                if (kt == 0) fetch_params();
                // (the first groups' sums have landed too: said here, where it costs nothing)
                if constexpr (RESIDUAL)
                    if (kt < 0) asm volatile("" : "+v"(ph[0]), "+v"(pl[0]), "+v"(ph[1]), "+v"(pl[1]), "+v"(ph[2]), "+v"(pl[2]));
                // reads the step-0 fragments of the next slice, of this tile or of the next one (after the
                // last slice of all: of a stage nobody needs); + A half of the slice two after this one
                k_step(fa1, fb1, fa0, fb0, nxt, 0, ADma{}, swap_tag);
            };
            for (int kt = 0; kt < slices - (RESIDUAL ? 1 : 0); ++kt) slice(kt);
            if constexpr (RESIDUAL) {
                if constexpr (SKIP) {
                    first_a = g.first_row[m_base + lane];         // (the buffers' last rows at most: tiles are inside)
                    if (TM > 2) first_b = g.first_row[min(m_base + 64 + lane, (int)g.max_rows - 1)];
                }
                const int off = lane_row(lane) * N + 8 * (lane & 7);
#pragma unroll
                for (int s = 0; s < D; ++s) fetch_sums(s, off);
                slice(-1);
            }
        };
        // first value column of this launch's W: after the query and key columns, or after the key columns
        const int v_col0 = EPI == EPI_KV ? hidden : 2 * hidden;
        const bool values = (EPI == EPI_QKV || EPI == EPI_KV) && n0 >= v_col0;
        if constexpr (SPLIT) {
            f32x16 hi[TM][T::TN];
            contract(nk / 2, std::true_type{});
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < T::TN; ++j) hi[i][j] = acc[i][j];
            contract(nk / 2, std::true_type{});
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < T::TN; ++j) acc[i][j] = hi[i][j] + acc[i][j];
        } else if (values || RESIDUAL) {
            contract(nk, std::false_type{});
        } else {
            contract(nk, std::true_type{});
        }

        // ---- epilogue -----------------------------------------------------------------------------
        // The product is transposed: accumulator element e of tile (i, j) is C[row, col] with row = 32 i + swap23(lane % 32),
        // col = 32 j + 16 (e / 8) + 8 (lane / 32) + e % 8, so a lane holds one row and runs of 8 columns.  Exchanges between
        // lanes (gather_runs) then give every access whole lines of memory, 8 rows of 128 bytes, with no trip through LDS:
        // lines written in halves (16 rows of 64 bytes) cost 90 clocks an instruction against 30, and a map's
        // launch 850 us against 805.  248 k rows of hidden 768, staged through LDS as floats / so: query-key-value map 891 /
        // 872 us, keys and values 620 / 570, first feed-forward map 1330 / 1284.  Value tiles are contracted
        // the other way round: a lane holds one feature and runs of 8 rows, and the same exchanges give lines of Vt.

        // (a copy of the lane index that the compiler takes for new: what is derived from it is worked out here for every
        // tile, and no register holds it through the contraction)
        int el = lane;
        asm volatile("" : "+v"(el));
        const int line = swap23(el & 31), half = el >> 5;
        const int out_run = 32 * ((el >> 3) & 1) + 16 * ((el >> 4) & 1) + 8 * half;   // after the exchanges
        const int out_line = 8 * ((el >> 2) & 1) + (el & 3);                          // + 16 b + 4 a of set (a, b)

        if (values) {
            bf16_t* vrow = Vt + (int64_t)(n_base - v_col0 + out_line) * vt_ld + m_base + out_run;
            float cc[2], dd[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                cc[j] = col_1[wn * WTN + 32 * j + line];
                dd[j] = col_bias[wn * WTN + 32 * j + line];
            }
            uint32_t u[2][2][2][4];                            // [j][i % 2][e / 8]: 64 rows of a feature in two blocks
#pragma unroll
            for (int i = 0; i < TM; ++i) {
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    float rs[8], nm[8];
#pragma unroll
                    for (int t = 0; t < 8; t += 2) {
                        const float4 s2 = *(const float4*)(row_stats + wave_row + 32 * i + 16 * b + 8 * half + t);
                        rs[t] = s2.y; nm[t] = -s2.x * s2.y;
                        rs[t + 1] = s2.w; nm[t + 1] = -s2.z * s2.w;
                    }
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int t = 0; t < 8; t += 2)
                            u[j][i & 1][b][t / 2] =
                                cvt_pk_bf16(fmaf(acc[i][j][8 * b + t], rs[t], fmaf(nm[t], cc[j], dd[j])),
                                            fmaf(acc[i][j][8 * b + t + 1], rs[t + 1], fmaf(nm[t + 1], cc[j], dd[j])));
                }
                if ((i & 1) == 0 && i + 1 < TM) continue;
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    if ((i & 1) == 0) {                        // an odd block at the end: lines in halves, as they are
                        bf16_t* f = Vt + (int64_t)(n_base - v_col0 + 32 * j + line) * vt_ld + m_base + 32 * i + 8 * half;
#pragma unroll
                        for (int b = 0; b < 2; ++b)
                            *(uint4*)(f + 16 * b) = make_uint4(u[j][0][b][0], u[j][0][b][1], u[j][0][b][2], u[j][0][b][3]);
                        continue;
                    }
                    gather_runs<4>(u[j]);
#pragma unroll
                    for (int a = 0; a < 2; ++a)
#pragma unroll
                        for (int b = 0; b < 2; ++b)
                            *(uint4*)(vrow + (int64_t)(32 * j + 16 * b + 4 * a) * vt_ld + 32 * (i - 1)) =
                                make_uint4(u[j][a][b][0], u[j][a][b][1], u[j][a][b][2], u[j][a][b][3]);
                }
            }
            continue;
        }

        if constexpr (RESIDUAL) {
            // New sums of the residual stream: acc + bias + LayerNorm(y_prev) recomputed from the previous sums and the row
            // statistics.  Bound by vector arithmetic, which nothing overlaps (one instruction an element is 1000 clocks a
            // tile): the product, not transposed, is brought into whole rows through LDS strip by strip, not by exchanges
            // between lanes, and the stream's two arrays are taken apart and put together by two instructions an element.
            // 1400 vector instructions a wavefront and tile, 2400 with sums of two bf16 values, exchanges and guarded stores:
            // output projection of 248 k rows of hidden 768 504 -> 488 us, of 1.8 M rows of hidden 1024 5012 -> 4910 (what
            // is left is 512 KB in and out a tile, by all units at about the same time), second feed-forward maps even.
            const int cg = el & 7, in_tile = lane_row(el) * N + 8 * cg;
            float gm[8], sh[8];
#pragma unroll
            for (int t = 0; t < 8; t += 4) {
                const int c = wn * WTN + 8 * cg + t;
                const float4 b4 = *(const float4*)(col_bias + c), g4 = *(const float4*)(col_1 + c), e4 = *(const float4*)(col_2 + c);
                gm[t] = g4.x; gm[t + 1] = g4.y; gm[t + 2] = g4.z; gm[t + 3] = g4.w;
                sh[t] = e4.x + b4.x; sh[t + 1] = e4.y + b4.y; sh[t + 2] = e4.z + b4.z; sh[t + 3] = e4.w + b4.w;
            }
            // Stores by buffer instructions whose range ends with the last live row: no lane is masked and no branch taken,
            // so the compiler counts them and a strip waits for its own sums only (guarded by the row, every strip waited
            // for the stores before it).
            const int pieces = N >> 6;
            const int live = __builtin_amdgcn_readfirstlane(max(0, min(rows - m_base, 32 * TM)));
            auto range = [&](void* base, int ld, int last) {
                const uint64_t a = (uint64_t)base;            // (wave-uniform, which the compiler has to be told)
                const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) << 32 |
                                   (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a);
                return __builtin_amdgcn_make_buffer_rsrc((void*)u, 0, live > 0 ? (live - 1) * ld + last : 0, 0x27000);
            };
            const int64_t at0 = (int64_t)m_base * N + n_base;
            const auto hi_out = range(res.x_out + at0, 2 * N, 128), lo_out = range((bf16_t*)Cv + at0, 2 * N, 128);
            const auto ps_out = range(res.pstats + (int64_t)m_base * pieces + (n_base >> 6), 8 * pieces, 8);
            const int ps_off = cg == 0 ? lane_row(el) * pieces * 8 : INT_MIN;          // one lane a row, the others out of range
            float* strip = (float*)(smem + T::STRIPS) + wave * 8 * T::STRIP_LD;
            const unsigned long long skip_a = SKIP ? __ballot(first_a != 0) : 0, skip_b = SKIP ? __ballot(first_b != 0) : 0;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                // The next slice's DMAs, while nothing is behind them: with one on its way the compiler takes every wait for
                // a load as a wait for all memory instructions.
                if (s == 0) __builtin_amdgcn_s_waitcnt(0x0f70);               // vmcnt(0)
                if (s + D < NS) fetch_sums(s + D, in_tile);
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int t = 0; t < 4; ++t) strip[(4 * half + t) * T::STRIP_LD + 32 * j + line] = acc[s >> 2][j][4 * (s & 3) + t];
                const float2 st = row_stats[wave_row + row_in(s) + lane_row(el)];
                const float4 a0 = *(const float4*)(strip + (el >> 3) * T::STRIP_LD + 8 * cg);
                const float4 a1 = *(const float4*)(strip + (el >> 3) * T::STRIP_LD + 8 * cg + 4);
                const float a[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
                float o[8];
                u32x4 ho, lo;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float2 y = stream_join2(ph[s % (D + 1)][t], pl[s % (D + 1)][t]);
                    o[2 * t] = residual_sum(a[2 * t], y.x, st, gm[2 * t], sh[2 * t]);
                    o[2 * t + 1] = residual_sum(a[2 * t + 1], y.y, st, gm[2 * t + 1], sh[2 * t + 1]);
                    uint32_t h, l;
                    stream_split2(o[2 * t], o[2 * t + 1], h, l);
                    ho[t] = h;
                    lo[t] = l;
                }
                // the 64-column piece's sum and sum of squares
                const float sm = row8_sum(((o[0] + o[1]) + (o[2] + o[3])) + ((o[4] + o[5]) + (o[6] + o[7])));
                const float sq = row8_sum((fmaf(o[0], o[0], o[1] * o[1]) + fmaf(o[2], o[2], o[3] * o[3])) +
                                          (fmaf(o[4], o[4], o[5] * o[5]) + fmaf(o[6], o[6], o[7] * o[7])));
                const u32x2 ps = {__float_as_uint(sm), __float_as_uint(sq)};
                // (offsets in the vector operand: the scalar one takes no part in the range check)
                int at = 2 * (in_tile + row_in(s) * N), ps_at = ps_off + 8 * row_in(s) * pieces;
                if constexpr (SKIP) {
                    // (bits 0-3 and 8-11: the strip's rows; most strips have none, and only stores that are dropped differ)
                    const unsigned mine = (unsigned)((s < 8 ? skip_a : skip_b) >> (row_in(s) & 63)) & 0xf0fu;
                    if (__builtin_expect(mine != 0, 0)) {
                        const bool drop = mine >> lane_row(el) & 1;
                        at = drop ? INT_MIN : at;
                        ps_at = drop ? INT_MIN : ps_at;
                    }
                }
                __builtin_amdgcn_raw_buffer_store_b128(ho, hi_out, at, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b128(lo, lo_out, at, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b64(ps, ps_out, ps_at, 0, 0);
            }
            continue;
        }

        {
            // bf16 out (GELU, or the query / key columns of the QKV projection): the left 32 columns of all rows are
            // finished first, then block by block the right ones, the exchanges and the stores
            const int64_t ldc = (EPI == EPI_QKV || EPI == EPI_KV) ? 2 * (int64_t)hidden
                                : SPLIT ? 2 * (int64_t)N : (int64_t)N;
            const int c_col = n_base + out_run + (EPI == EPI_KV ? hidden : 0);   // key columns sit after the query columns
            bf16_t* C = (bf16_t*)Cv + (int64_t)(m_base + out_line) * ldc + c_col;
            float rs[TM], nm[TM];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const float2 st = FOLD ? row_stats[wave_row + 32 * i + line] : make_float2(0.f, 0.f);
                rs[i] = st.y; nm[i] = -st.x * st.y;
            }
            auto store = [&](uint32_t (&u)[2][2][4], int i, int64_t off) {
                gather_runs<4>(u);
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        *(uint4*)(C + (int64_t)(32 * i + 16 * b + 4 * a) * ldc + off) =
                            make_uint4(u[a][b][0], u[a][b][1], u[a][b][2], u[a][b][3]);
            };
            uint32_t u[TM][2][2][4], l[SPLIT ? TM : 1][2][2][4];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                float cc[16], dd[16];                          // of the lane's columns 16 (e / 8) + 8 half + e % 8
#pragma unroll
                for (int e = 0; e < 16; e += 4) {
                    const int c = wn * WTN + 32 * j + 16 * (e >> 3) + 8 * half + (e & 7);
                    const float4 d4 = *(const float4*)(col_bias + c);
                    dd[e] = d4.x; dd[e + 1] = d4.y; dd[e + 2] = d4.z; dd[e + 3] = d4.w;
                    if (FOLD) {
                        const float4 c4 = *(const float4*)(col_1 + c);
                        cc[e] = c4.x; cc[e + 1] = c4.y; cc[e + 2] = c4.z; cc[e + 3] = c4.w;
                    }
                }
#pragma unroll
                for (int i = 0; i < TM; ++i) {
#pragma unroll
                    for (int e = 0; e < 16; e += 2) {
                        float v[2];
#pragma unroll
                        for (int t = 0; t < 2; ++t) {
                            const float a = acc[i][j][e + t];
                            v[t] = FOLD ? fmaf(a, rs[i], fmaf(nm[i], cc[e + t], dd[e + t])) : a + dd[e + t];
                            if (EPI == EPI_BIAS_GELU || SPLIT) v[t] = gelu_erf(v[t]);
                        }
                        const uint32_t h = cvt_pk_bf16(v[0], v[1]);
                        u[i][j][e >> 3][(e & 7) >> 1] = h;
                        // second half of the row: what the first rounding lost, as bf16 again
                        if constexpr (SPLIT)
                            l[i][j][e >> 3][(e & 7) >> 1] =
                                cvt_pk_bf16(v[0] - __uint_as_float(h << 16), v[1] - __uint_as_float(h & 0xffff0000u));
                    }
                    if (j == 0) continue;
                    store(u[i], i, 0);
                    if constexpr (SPLIT) store(l[i], i, N);
                }
            }
        }
    }
    // parked DMAs may still be in flight: they must land before the workgroup gives up its LDS
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// The per-request map that a launch can carry (see launch_gemm_bf16): blocks of the skinny form up to PS_SKINNY_ROWS requests
// (FEW), else 64 x 64 tiles for the maps back to the hidden width, 128 x 64 for the first feed-forward map, with as many slices on
// their way as the launch's LDS has room for.
constexpr int kNoSide = -1;
template <int EPI>
constexpr int side_of = EPI == EPI_BIAS_RESIDUAL ? (int)EPI_RESIDUAL_MAPPED : (int)EPI_GELU_SPLIT;
template <int SIDE, int BM, bool FEW>
struct SideTile {
    using Args = std::conditional_t<FEW, SkinnyArgs, SmallGemm>;
    static constexpr int TM = SIDE == EPI_GELU_SPLIT ? 2 : 1;
    static constexpr int STAGES = SIDE == EPI_GELU_SPLIT ? (BM == 256 ? 6 : 3) : (BM == 256 ? 8 : 4);
    static constexpr int BYTES = SIDE == kNoSide ? 0 : FEW ? kSkinnyLds : STAGES * 64 * (TM + 1) * 128;
};

// Rows in two regions: plan->m_tiles tiles of BM rows, then the others in tiles of 32 (tm0 + tm1) rows, as prep chose them
// (PLANNED); without a plan all in tiles of BM rows.  SIDE: further workgroups do a per-request map.  Behind the map's own a unit
// that has no tile in the launch's last round takes them.  Blocks of a few requests' map beside 128 x 128 tiles (AHEAD), which take
// as long as a tile, come first: the tiles are then dealt to the other units as long as there are any, and share one beyond.
// Two wavefronts a SIMD: for 128 x 128 tiles two workgroups a unit, which the compiler misses by itself with a few requests' map
// (202 + 64 registers; 216 so).  Padded calls of hidden 768, twelve layers, slots all filled, one workgroup a unit / two: 12 requests
// 2482 / 2110 us, 16 2648 / 2314; filled to a half, where all tiles have a unit each, 1524 / 1512 and 1641 / 1621, but 5 % more
// than the first with the side blocks behind the tiles.  12 prompts of the production encoder 3578 -> 3154 us, 8 3428 -> 2797.
template <int BM, int BN, int WM, int WN, int EPI, bool PLANNED, int SIDE, bool FEW>
__global__ __launch_bounds__(WM * WN * 64, 2) void gemm_bf16_kernel(GemmArgs g, const int32_t* __restrict__ total_rows,
                                                                 const GemmPlan* __restrict__ plan, int64_t* __restrict__ clk,
                                                                 typename SideTile<SIDE, BM, FEW>::Args side) {
    using T = Tile<BM, BN, WM, WN>;
    using S = SideTile<SIDE, BM, FEW>;
    constexpr int kBytes = EPI == EPI_BIAS_RESIDUAL ? T::LDS : T::STRIPS;
    constexpr bool SKIP = SIDE == EPI_RESIDUAL_MAPPED, AHEAD = FEW && !PLANNED;
    __shared__ __align__(1024) unsigned char smem[kBytes > S::BYTES ? kBytes : S::BYTES];
    if constexpr (SIDE != kNoSide) {
        const int b = AHEAD ? (int)blockIdx.x : (int)blockIdx.x - g.wgs;
        if (AHEAD ? b < g.ahead : b >= 0) {
            if constexpr (FEW) {
                if (b * kSkinnyCols < side.N) skinny_block<SIDE, WM * WN, SIDE != EPI_RESIDUAL_MAPPED>(side, b, smem);
            } else {
                if (threadIdx.x < 256) small_tile<SIDE, S::TM, 1, S::STAGES>(side, b, smem, nullptr);
            }
            return;
        }
    }
    // clock probe (profiling only): core cycles and constant-rate ticks over this workgroup's life
    const int64_t clk_c0 = clk ? (int64_t)clock64() : 0, clk_w0 = clk ? (int64_t)wall_clock64() : 0;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Region rg;
    rg.rows = *total_rows;
    if constexpr (!PLANNED) {
        rg.row_begin = 0; rg.bm = BM; rg.tm0 = T::TM;
        rg.m_tiles = (rg.rows + BM - 1) / BM;
        region_tiles<T, WN, T::TM, EPI, false, SKIP, AHEAD>(g, g.A, g.W, g.bias, g.C, g.Vt, rg, smem);
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
            if (tm == 4) region_tiles<T, WN, 4, EPI, true, SKIP, AHEAD>(g, g.A, g.W, g.bias, g.C, g.Vt, rg, smem);
            else if (tm == 3) region_tiles<T, WN, 3, EPI, true, SKIP, AHEAD>(g, g.A, g.W, g.bias, g.C, g.Vt, rg, smem);
            else region_tiles<T, WN, 2, EPI, true, SKIP, AHEAD>(g, g.A, g.W, g.bias, g.C, g.Vt, rg, smem);
        }
    }
    if (clk && blockIdx.x == (AHEAD ? g.ahead : 0) && threadIdx.x == 0) {
        clk[0] = (int64_t)clock64() - clk_c0;
        clk[1] = (int64_t)wall_clock64() - clk_w0;
    }
}

template <int BM, int BN, int WM, int WN, bool PLANNED>
void launch_cfg(GemmEpilogue epi, GemmArgs g, const int32_t* total_rows, const GemmPlan* plan, int64_t* clk,
                const SmallGemm* side, const SkinnyArgs* few, hipStream_t s) {
    // persistent: one workgroup per compute unit; the small tiles leave room for two (LDS and registers), which then hide
    // each other's waits, and take fewer workgroups if there cannot be that many tiles
    const int64_t tiles = (g.max_rows + BM - 1) / BM * (g.N / BN);
    g.wgs = (int)(PLANNED ? 256 : tiles < 512 ? (tiles + 7) / 8 * 8 : 512);
    const dim3 block(WM * WN * 64);
    // a side map's tiles, hi and lo part of a request in one
    auto side_wgs = [&](int tm) {
        const int64_t n = (side->max_rows * 2 + 64 * tm - 1) / (64 * tm) * (side->N / 64);
        return (unsigned)((n + 7) / 8 * 8);
    };
#define PS_LAUNCH(E)                                                                                                     \
    hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WM, WN, E, PLANNED, kNoSide, false>), dim3((unsigned)g.wgs), block, 0, s, g, total_rows, plan, clk, SmallGemm{})
#define PS_LAUNCH_SIDE(E)                                                                                                \
    do {                                                                                                                 \
        constexpr int kSide = side_of<E>;                                                                                \
        if (few) {                                                                                                       \
            g.ahead = (int)align_up((size_t)(few->N / kSkinnyCols), 8);                                                  \
            hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WM, WN, E, PLANNED, kSide, true>),                              \
                               dim3((unsigned)(g.wgs + g.ahead)), block, 0, s, g, total_rows, plan, clk, *few);          \
        } else if (side)                                                                                                   \
            hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WM, WN, E, PLANNED, kSide, false>),                             \
                               dim3((unsigned)g.wgs + side_wgs(SideTile<kSide, BM, false>::TM)), block, 0, s, g, total_rows, plan, \
                               clk, *side);                                                                              \
        else                                                                                                             \
            PS_LAUNCH(E);                                                                                                \
    } while (0)
    switch (epi) {
        case EPI_BIAS_GELU: PS_LAUNCH_SIDE(EPI_BIAS_GELU); break;
        case EPI_BIAS_RESIDUAL: PS_LAUNCH_SIDE(EPI_BIAS_RESIDUAL); break;
        case EPI_QKV: PS_LAUNCH(EPI_QKV); break;
        case EPI_KV: PS_LAUNCH(EPI_KV); break;
        case EPI_GELU_SPLIT:
            if constexpr (!PLANNED) PS_LAUNCH(EPI_GELU_SPLIT);
            break;
        default: break;                                  // the mapped forms are small_gemm.hip's and skinny_gemm.hip's
    }
#undef PS_LAUNCH
#undef PS_LAUNCH_SIDE
}

}  // namespace

// Requirements (hidden and feed-forward width are multiples of 256, checked when the model is loaded): N % 256 == 0,
// K % 64 == 0 and K >= 128, 256 for EPI_GELU_SPLIT's two halves (a tile's biases and statistics are fetched behind the first slice of
// a contraction, its previous sums ahead of the last); every buffer holds max_rows rows with
// max_rows % 256 == 0.  Tiles of 128 and 256 rows are then always in bounds; those of other heights may reach past the end
// and are moved up (row_of).
void launch_gemm_bf16(GemmEpilogue epi, const bf16_t* A, const bf16_t* W, const float* bias,
                      ResidualSrc residual, void* C, bf16_t* vt, int64_t max_rows, int N, int K,
                      int hidden, const int32_t* total_rows, const GemmPlan* plan, int64_t* clk, hipStream_t s,
                      const uint8_t* first_row, const SmallGemm* side, const SkinnyArgs* few) {
    // Problems with few 256 x 256 tiles (whole calls on a micro-batch of a few requests) would leave most compute
    // units idle: 128 x 128 tiles give four times as many workgroups to spread them over.  EPI_GELU_SPLIT has only these
    // (its second set of accumulators): 4096 requests of hidden 768 in 57 us, 20000 in 234.
    const GemmArgs g = {A, W, bias, residual, C, vt, max_rows, N, K, hidden, 0, 0, first_row};
    if (epi == EPI_GELU_SPLIT || !large_tiles(max_rows, N))
        launch_cfg<128, 128, 2, 2, false>(epi, g, total_rows, nullptr, clk, side, few, s);
    else
        launch_cfg<256, 256, 2, 4, true>(epi, g, total_rows, plan, clk, side, few, s);
}
