// Decode-size linears (M <= 64): y[M,N] = x[M,K] * W[K,N] with W either fp16 or the 4-bit
// record, bound by the rate at which the weights stream out of HBM.  The streaming multiply
// itself is tile_partial() of decode_core.h; this file adds what one launch per linear needs:
//   * K is split over the waves of a workgroup and over S workgroups per column tile.  Waves are
//     summed out of LDS in a fixed order; workgroups write fp32 partials (written through to
//     memory) and the last one to arrive, found with an atomic counter, adds them in index order,
//     so results do not depend on timing.  A workgroup takes a slice of 16 or 32 rows; further
//     rows are handled by further slices of the grid running the same code.
#include "decode_core.h"
#include "kernels.h"

namespace morph {

namespace {

constexpr int kScatterBase = 8192;                       // the polled counters sit behind the plain ones, 32 ints apart
constexpr int kScatterTiles = 256;                       // as many tiles as have a line there
constexpr int kScatterPolls = 4096;                      // bound of the wait for the other workgroups of a tile

// What a workgroup needs before its first load comes as scalar arguments, first in the list: the
// compiler has them preloaded into scalar registers at wave launch (kernarg preload), so the start
// does not wait for a load of the argument block from memory.  The rest (used at the hand-over)
// follows in a structure that is fetched when it is needed.
struct DecodeTail {
    void*  y;
    float* partial;
    int*   counters;
    int    rows, stream_loads, scatter, polls, cstride;
};

// BF: x, y (and the weights of the fp16 kind) are bfloat16 instead of fp16.
template <int Q, int MT, int kWaves, bool NT, bool BF>
__global__ __launch_bounds__(kWaves * 64, kWaves == 4 ? 2 : 1) void decode_kernel(
    const void* w, const void* x, const void* scales, const void* qzeros, int Ktot, int Ntot, int Mtot, int Stot,
    int tiles, int slices, DecodeTail t)
{
    DecodeArgs p;
    p.w = w; p.x = x; p.scales = scales; p.qzeros = qzeros; p.K = Ktot; p.N = Ntot; p.M = Mtot; p.S = Stot;
    p.tiles = tiles; p.slices = slices;
    p.y = t.y; p.partial = t.partial; p.counters = t.counters; p.rows = t.rows; p.stream_loads = t.stream_loads;
    p.scatter = t.scatter; p.polls = t.polls; p.cstride = t.cstride;
    MORPH_TICK(6);                                       // kernel entry
    typedef TileGeom<Q, MT, kWaves> G;
    constexpr int CPL = G::CPL, TN = G::TN, TNB = G::TNB, NV = G::NV, ITEMS = G::ITEMS;
    extern __shared__ __align__(16) f32x4 yl[];

    const int tid = threadIdx.x;
    const int S = p.S;
    // Which (column tile, part of K, row slice) this workgroup takes.  With several row slices the
    // slices of one (tile, part) are dealt to consecutive workgroups OF ONE XCD (workgroup g runs
    // on XCD g % 8), so that they run at the same time on the same L2 and the weights leave
    // memory once instead of once per slice.
    int unit = blockIdx.x, slice = 0;
    if (p.slices > 1) {
        const int units = p.tiles * S, whole = (units >> 3) * 8 * p.slices;   // workgroups of whole rounds of 8 units
        if ((int)blockIdx.x < whole) {
            const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
            slice = j % p.slices;
            unit  = (j / p.slices) * 8 + xcd;
        } else {                                         // the last units (fewer than 8): slice by slice
            const int r = blockIdx.x - whole, left = units & 7;
            slice = r / left;
            unit  = (units >> 3) * 8 + (r - slice * left);
        }
    }
    const int nt = unit / S, sp = unit - nt * S;
    const int n0 = nt * TNB;                             // first column of the workgroup tile
    const int mbase = slice * (MT * 16);                 // first row of this slice
    const int M = (p.M - mbase) < MT * 16 ? (p.M - mbase) : MT * 16;   // rows of this slice
    const int N = p.N;

    TileJob job;
    job.x = (const half_t*)p.x + (size_t)mbase * p.K;
    job.w = p.w; job.scales = p.scales; job.qzeros = p.qzeros;
    job.M = M; job.K = p.K; job.N = N; job.n0 = n0; job.S = S; job.sp = sp;
    tile_partial<Q, MT, kWaves, false, NT, BF>(job, yl);

    // ---- sum the waves that share columns (in the order of their k parts) and write out ----
    uint16_t* y = (uint16_t*)p.y + (size_t)mbase * N;
    auto item_sum = [&](int it) { return G::item_sum(yl, it); };
    auto item_store_y = [&](int it, f32x4 acc) {
        const int pn = it / (NV * 64), rem = it - pn * (NV * 64);
        const int v = rem >> 6, ln = rem & 63;
        const int mt = v / CPL, j = v - mt * CPL;
        const int col = n0 + pn * TN + CPL * (ln & 15) + j;
        const int row = 16 * mt + 4 * (ln >> 4);
        if (col < N) {
#pragma unroll
            for (int r = 0; r < 4; r++)
                if (row + r < M) y[(size_t)(row + r) * N + col] = narrow16<BF>(acc[r]);
        }
    };
    auto item_rows_live = [&](int it) {                  // does the vector hold any row below M?
        const int rem = it % (NV * 64), v = rem >> 6, ln = rem & 63;
        return 16 * (v / CPL) + 4 * (ln >> 4) < M;
    };
    // With at most four rows only lanes 0..15 of a vector hold rows that exist: those vectors are
    // numbered 0 .. LIVE-1 so that every thread gets one, instead of a quarter of the threads four.
    constexpr int LIVE = (ITEMS / 64) * 16;
    auto live_item = [](int L) { return (L >> 4) * 64 + (L & 15); };
    const bool few = M <= 4;
    if (S == 1) {
        if (few) {
            for (int L = tid; L < LIVE; L += kWaves * 64) item_store_y(live_item(L), item_sum(live_item(L)));
        } else {
            for (int it = tid; it < ITEMS; it += kWaves * 64)
                if (item_rows_live(it)) item_store_y(it, item_sum(it));
        }
        return;
    }
    // Partials cross workgroups that may sit on different XCDs (separate L2s).  They are written
    // through to memory and read past the caches (scope bits on the instructions), which is all the
    // ordering needs: wait for the stores, count the arrival, and the last arriver reads.  No
    // whole-cache write-back or invalidate is issued.  Layout: [tile][split][item] f32x4.
    const int tile_id = slice * p.tiles + nt;                        // slices keep separate counters and partials
    constexpr uint32_t kPartBytes = (uint32_t)ITEMS * 16u;           // one workgroup's partial
    const float* tile_base = p.partial + (size_t)tile_id * S * ITEMS * 4;
    const __amdgpu_buffer_rsrc_t rp = make_rsrc(tile_base, (uint32_t)S * kPartBytes);
    if (few) {
        for (int L = tid; L < LIVE; L += kWaves * 64)
            buf_store_through(rp, (uint32_t)sp * kPartBytes + (uint32_t)live_item(L) * 16u, item_sum(live_item(L)));
    } else {
        for (int it = tid; it < ITEMS; it += kWaves * 64)
            if (item_rows_live(it)) buf_store_through(rp, (uint32_t)sp * kPartBytes + (uint32_t)it * 16u, item_sum(it));
    }
    wait_stores();
    MORPH_TICK(3);
    __syncthreads();                                     // every wave is done reading yl
    int* flag = reinterpret_cast<int*>(yl);
    if (p.scatter) {
        // The sum over the splits is shared out: every workgroup of the tile waits (a bounded number
        // of polls) until all S partials are there and then adds up its own S-th of the tile, instead
        // of the last arriver adding up all of it alone.  Correctness never depends on the wait: every
        // workgroup ends by adding its "done" bit to a second counter, and the last one to do so adds
        // up whatever parts are still missing (a workgroup that gave up waiting leaves its part) and
        // puts both counters back to zero; by then nobody polls any more.  Sums run over the splits in
        // index order whoever computes them.
        int* arrive = p.counters + kScatterBase + tile_id * 32;   // a 128-byte line of its own per tile: up to 16 workgroups poll it
        int* depart = arrive + 16;
        if (tid == 0) {
            const int c = __hip_atomic_fetch_add(arrive, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            int complete = c == S - 1;
            for (int i = 0; !complete && i < p.polls; i++) {
                complete = __hip_atomic_load(arrive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) >= S;
                __builtin_amdgcn_s_sleep(4);
            }
            *flag = complete;
        }
        __syncthreads();
        const int complete = *flag;
        __syncthreads();                                 // the flag word is written again below
        constexpr int NVEC = ITEMS / 64;                 // vectors of 64 lanes in the tile
        auto reduce_part = [&](int j) {
            const int v0 = (j * NVEC) / S, v1 = ((j + 1) * NVEC) / S;
            for (int it = v0 * 64 + tid; it < v1 * 64; it += kWaves * 64) {
                if (!item_rows_live(it)) continue;
                f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
                for (int s2 = 0; s2 < S; s2 += 8) {
                    f32x4 v[8];
#pragma unroll
                    for (int q = 0; q < 8; q++)            // splits beyond S read past the buffer and come back as zeros
                        v[q] = bit_cast<f32x4>(__builtin_amdgcn_raw_buffer_load_b128(rp, (uint32_t)it * 16u, (uint32_t)(s2 + q) * kPartBytes, kAuxSystemScope));
#pragma unroll
                    for (int q = 0; q < 8; q++) a += v[q];
                }
                item_store_y(it, a);
            }
        };
        if (complete) reduce_part(sp);
        if (tid == 0) {
            const int old = __hip_atomic_fetch_add(depart, 1 | (complete << (8 + sp)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *flag = (old & 0xFF) == S - 1 ? (0x10000 | (((old >> 8) | (complete << sp)) & 0xFFFF)) : 0;
        }
        __syncthreads();
        const int last = *flag;
        if (last) {
            for (int j = 0; j < S; j++)
                if (!((last >> j) & 1)) reduce_part(j);  // parts whose owner gave up waiting: normally none
            if (tid == 0) { atomicExch(arrive, 0); atomicExch(depart, 0); }
        }
        return;
    }
    if (tid == 0) *flag = (atomicAdd(p.counters + tile_id * p.cstride, 1) == S - 1) ? 1 : 0;
    __syncthreads();
    MORPH_TICK(4);
    if (!*flag) return;
    // All loads of a thread's items are independent: they are issued together and summed in index
    // order (split 0 first), so the result does not depend on which workgroup arrived last.
    if (few) {
        // one live vector per thread and all splits in flight at once (a deep split is then fetched
        // in one round trip instead of two)
        constexpr int CH4 = 16;
        for (int L = tid; L < LIVE; L += kWaves * 64) {
            const int it = live_item(L);
            f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int s2 = 0; s2 < S; s2 += CH4) {
                f32x4 v[CH4];
#pragma unroll
                for (int q = 0; q < CH4; q++)              // splits beyond S read past the buffer and come back as zeros
                    v[q] = bit_cast<f32x4>(__builtin_amdgcn_raw_buffer_load_b128(rp, (uint32_t)it * 16u, (uint32_t)(s2 + q) * kPartBytes, kAuxSystemScope));
#pragma unroll
                for (int q = 0; q < CH4; q++) a += v[q];
            }
            item_store_y(it, a);
        }
        if (tid == 0) atomicExch(p.counters + tile_id * p.cstride, 0);
        MORPH_TICK(5);
        return;
    }
    constexpr int IPT = ITEMS / (kWaves * 64);           // items per thread
    f32x4 acc[IPT];
#pragma unroll
    for (int i = 0; i < IPT; i++) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int CH = IPT <= 4 ? 8 : 4;                 // splits fetched together (registers are free here)
    uint32_t item_off[IPT];
#pragma unroll
    for (int i = 0; i < IPT; i++) {                      // vectors made of rows that do not exist are not fetched
        const int it = tid + i * kWaves * 64;
        item_off[i] = item_rows_live(it) ? (uint32_t)it * 16u : 0xFFFFFFF0u;
    }
    for (int s2 = 0; s2 < S; s2 += CH) {
        f32x4 v[CH][IPT];
#pragma unroll
        for (int q = 0; q < CH; q++)
#pragma unroll
            for (int i = 0; i < IPT; i++) {
                // splits beyond S read past the buffer and come back as zeros
                v[q][i] = bit_cast<f32x4>(__builtin_amdgcn_raw_buffer_load_b128(rp, item_off[i], (uint32_t)(s2 + q) * kPartBytes, kAuxSystemScope));
            }
#pragma unroll
        for (int q = 0; q < CH; q++)
#pragma unroll
            for (int i = 0; i < IPT; i++) acc[i] += v[q][i];
    }
#pragma unroll
    for (int i = 0; i < IPT; i++) {
        const int it = tid + i * kWaves * 64;
        if (item_rows_live(it)) item_store_y(it, acc[i]);
    }
    if (tid == 0) atomicExch(p.counters + tile_id * p.cstride, 0);
    MORPH_TICK(5);
}

// Waves per workgroup: two M tiles halve the bytes a wave keeps in flight, so eight waves per
// compute unit in one workgroup do better there; one M tile runs best as two workgroups of four.
inline int decode_waves(int rows)
{
    const int t = tuning_get(TUNE_DECODE_WAVES);
    if (t == 4 || t == 8) return t;
    return rows > 16 ? 8 : 4;
}

template <int Q, int MT, int kWaves, bool NT, bool BF>
hipError_t launch_waves(const DecodeArgs& a, int slices, hipStream_t st)
{
    constexpr int tnb = Tile<Q, MT>::TN * Tile<Q, MT>::WN;
    constexpr size_t lds = TileGeom<Q, MT, kWaves>::kLdsBytes;
    static_assert(lds <= 128 * 1024, "LDS of one compute unit");
    if (lds > 64 * 1024) {
        static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&decode_kernel<Q, MT, kWaves, NT, BF>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (attr != hipSuccess) return attr;
    }
    DecodeArgs b = a;
    b.tiles  = (a.N + tnb - 1) / tnb;
    b.slices = slices;
    b.cstride = b.tiles * slices <= 256 ? 32 : b.tiles * slices <= 512 ? 16 : 1;   // a cache line per arrival counter while they fit
    const int units = b.tiles * a.S;
    const int grid  = units * slices;
    DecodeTail t;
    t.y = b.y; t.partial = b.partial; t.counters = b.counters; t.rows = b.rows; t.stream_loads = b.stream_loads;
    t.scatter = b.scatter; t.polls = b.polls; t.cstride = b.cstride;
    hipLaunchKernelGGL((decode_kernel<Q, MT, kWaves, NT, BF>), dim3(grid), dim3(kWaves * 64), lds, st, b.w, b.x, b.scales,
                       b.qzeros, b.K, b.N, b.M, b.S, b.tiles, b.slices, t);
    return hipGetLastError();
}

template <int Q, int MT, bool BF>
hipError_t launch_one(const DecodeArgs& a, int slices, hipStream_t st)
{
    const bool w8 = decode_waves(MT * 16) == 8;
    if constexpr (MT == 1 || Q != 1) {                   // not the 4-bit two-tile kernel: its two column halves share cache lines
        if (a.stream_loads) return w8 ? launch_waves<Q, MT, 8, true, BF>(a, slices, st) : launch_waves<Q, MT, 4, true, BF>(a, slices, st);
    }
    return w8 ? launch_waves<Q, MT, 8, false, BF>(a, slices, st) : launch_waves<Q, MT, 4, false, BF>(a, slices, st);
}

template <bool BF>
hipError_t launch_format(int q, bool one, const DecodeArgs& a, int slices, hipStream_t st)
{
    if (q == 1) return one ? launch_one<1, 1, BF>(a, slices, st) : launch_one<1, 2, BF>(a, slices, st);
    if (q == 2) return one ? launch_one<2, 1, BF>(a, slices, st) : launch_one<2, 2, BF>(a, slices, st);
    return one ? launch_one<0, 1, BF>(a, slices, st) : launch_one<0, 2, BF>(a, slices, st);
}

}  // namespace

MORPH_TICK_EXPORTS(ticks)

namespace {

// The plan for slices of `rows` rows (16: one MFMA row tile per workgroup, 32: two), with an
// estimate of the launch time net of what does not depend on the choice.
DecodePlan plan_rows(int q, int M, int K, int N, int rows)
{
    DecodePlan pl{};
    pl.rows   = rows;
    const bool is_w4 = q == 1;                          // q: 0 = fp16, 1 = 4-bit, 2 = 8-bit codes
    pl.tile_n = !is_w4 ? Tile<0, 1>::TN : 256;          // workgroup tile (W4: 1 x 256 or 2 x 128 columns)
    const int kWaves = decode_waves(rows);
    const int wk = (is_w4 && rows > 16) ? kWaves / Tile<1, 2>::WN : kWaves;   // waves of a workgroup along K
    pl.tiles  = (N + pl.tile_n - 1) / pl.tile_n;
    pl.slices = (M + rows - 1) / rows;
    const int T = K / 32;
    int target = tuning_get(TUNE_DECODE_WGS);
    if (target <= 0) target = 256;                       // one workgroup per compute unit
    const int units = pl.tiles * pl.slices;
    int S = target / units;                              // never more workgroups than are resident at once
    // at least one group of four k-steps per wave; with at most four rows the hand-over is short and
    // more workgroups pay even if half their waves stay empty (o-proj 4096 x 4096 at M = 1: 7.7 -> 7.2 us)
    int smax = T / (wk * (M <= 4 ? 2 : 4));
    if (S > smax) S = smax;
    if (S > 64) S = 64;
    const int forced = tuning_get(TUNE_DECODE_SPLIT);
    if (forced > 0) S = forced > T / wk ? T / wk : forced;
    const long long lim = ((1LL << 31) / T) - 1;          // the kernels form (part + 1) * T in 32 bits
    if (S > lim) S = (int)lim;
    if (S < 1) S = 1;
    pl.S = S;
    // items of one workgroup tile: rows x tile columns, as fp32
    const size_t tile_floats = (size_t)rows * pl.tile_n;
    pl.partial_bytes = S > 1 ? (size_t)units * S * tile_floats * sizeof(float) : 0;
    // Estimate (microseconds, W4 constants measured on MI355X): the rows of K one workgroup walks at
    // the rate its waves unpack them, or the weights at the rate strips of them leave memory when
    // that is slower; then the hand-over.
    const double wgs = (double)units * S, fill = wgs < 256.0 ? wgs / 256.0 : 1.0;
    const double walk = ((double)K / S) * (rows > 16 ? 6.7e-3 : 3.24e-3) * (double)(((long long)wgs + 255) / 256);
    const double hbm  = ((double)K * N * 0.5) / (4.6e6 * fill);
    // Sharing the sum over the splits out among the workgroups of a tile pays where that sum is long
    // (measured: 4 .. 14 % at 16 to 64 rows, a loss of 3 % at 8): from 16 rows on and with at least
    // three splits (16 at most: one bit per split in a counter; 256 tiles at most: a line each).
    const int sc = tuning_get(TUNE_DECODE_SCATTER);
    pl.scatter = S >= 2 && S <= 16 && units <= kScatterTiles && (sc == 1 || sc == 3 || (sc == 0 && S >= 3 && M >= 16));
    pl.polls   = sc == 3 ? 0 : kScatterPolls;          // 3: nobody waits, so that the last one out has every part left to do (test hook)
    // hand-over: the last arriver reads S partial tiles on its own, or every workgroup one tile's worth
    const double handover = S <= 1 ? 0.0 : pl.scatter ? 2.3 + (double)tile_floats * 4.0 / 2.0e5
                                                       : 1.5 + (double)S * tile_floats * 4.0 / 2.0e5;
    pl.est_us = (walk > hbm ? walk : hbm) + handover;
    // Non-temporal weight loads where one workgroup alone reads its rows, once: measured on graphs
    // that cycle through 1.26 GB of 7B layers, fp16 5.6 % and W4 2 % faster.  Never where slices,
    // or the two column halves of the 4-bit two-tile kernel, meet in the caches (up to 17 % slower).
    const int nt = tuning_get(TUNE_DECODE_STREAM);
    pl.stream_loads = nt ? (nt == 1 && (rows == 16 || q != 1)) : (pl.slices == 1 && (rows == 16 || q != 1));
    return pl;
}

}  // namespace

// Slices of 32 rows share the unpacking of a weight between two MFMA row tiles; slices of 16 rows
// put twice the workgroups along M instead of along K, which halves both the split and the
// partial tile the last arriver has to add up.  For the 4-bit kernels between 17 and 64 rows the
// estimate decides, as long as all workgroups of the 16-row plan run at the same time.
// At most 16 rows of 4-bit weights: the kernel of decode_small.hip.  One workgroup per compute unit;
// K is shared out over S <= 16 workgroups per column tile of 256 (one "share done" bit each in the
// tile's counter), every workgroup keeping at least four k-steps, one per wave.
// narrow: dense weights in column tiles of 128, beyond 32 rows all rows in one workgroup (plan_narrow).
static DecodePlan plan_small(int q, int M, int K, int N, int native, bool narrow = false)
{
    DecodePlan pl{};
    pl.small  = 1;
    pl.rows   = 16;
    pl.slices = 1;
    pl.tile_n = q == 2 || narrow ? 128 : 256;             // 8-bit codes: a wave's 8 bytes per row are 8 columns
    pl.tiles  = (N + pl.tile_n - 1) / pl.tile_n;
    const int T = K / 32;
    // Never more workgroups than compute units: the workgroups of a tile wait for each other's partial
    // sums, which is quick only while all of them run at the same time (one per compute unit: the kernel
    // uses more than half the registers and the LDS of one).
    int target = tuning_get(TUNE_DECODE_WGS);
    if (target <= 0) target = prefill_compute_units();
    const int slices = M > 32 && !narrow ? 2 : 1;         // beyond 32 rows slices of 32 rows, a workgroup each
    // `most`: every workgroup keeps a quantization group (decode_small_kernel), or each half of its waves one
    auto split_for = [&](int most) {
        int S = target / (pl.tiles * slices);
        // ... and never more on one XCD than it has compute units: the workgroups of a tile share an XCD, tile t goes to
        // XCD t % 8, so an XCD runs ceil(tiles / 8) tiles (20 tiles of a 5120-wide matrix: 3, not 2.5 -- with 12 splits
        // that made 36 workgroups for 32 compute units, and the four that had to wait for a free one found the others
        // gone, waited the bound out and recomputed everything: 49 us instead of 7)
        const int per_xcd = (target / 8) / (((pl.tiles + 7) / 8) * slices);
        if (S > per_xcd) S = per_xcd;
        if (S > most) S = most;
        if (S > 16) S = 16;
        const int forced = tuning_get(TUNE_DECODE_SPLIT);
        if (forced > 0) S = forced > 16 ? 16 : forced;
        if (S > T / 4) S = T / 4;
        return S < 1 ? 1 : S;
    };
    const int halves = T / 8 > 0 ? T / 8 : 1;
    int S;
    if (q == 0) {
        // Dense weights can be shared out in k-steps (dense_by_steps): four per workgroup are enough (7 rows, us, with eight -> four: 2048 x 2048 7.32 -> 5.95,
        // 1024 x 4096 6.91 -> 6.01, 3072 x 3072 8.20 -> 7.84); where eight would leave one workgroup, one it stays (no workspace needed).
        S = split_for(halves > 1 ? T / 4 : 1);
        // Splits that all start a multiple of 1 MB apart read the same channels at the same time.  One fewer makes their parts uneven; at 128
        // k-steps and fewer three fewer, as the hand-over over many splits is a larger part there.  us at 7 / 32 rows, even splits -> fewer: 4096 x 4096 16 splits
        // 10.6 / 13.0, 13 9.6 / 12.1; 2048 x 4096 7.3 / 9.4, 6.9 / 9.1; 1536 .. 1920 x 4096 12 .. 15 splits 6.6 .. 7.0 / 8.7 .. 9.2, 9 .. 12 6.4 .. 6.7 / 8.4 .. 8.8;
        // 4096 x 2048 8.9 / 10.8, 7.9 / 10.1 (64 rows 11.8, 10.5); 8192 x 2048 16 splits 11.2 / 13.35, 15 10.8 / 13.35 (64 rows 14.7, 13.8); 8192 x 1024 10.3, 9.95
        // (32 rows 12.35, 12.55: fewer than 128 workgroups); 8192 x 4096 15.4 / 17.7, 14.7 / 17.3; 14336 x 4096 23.3 / 25.6, 22.7 / 25.0.
        //   A workgroup's part grows by a sixteenth with it.  Beyond 16 k-steps to a part, and at multiples of 1 MB that are no power of two, that costs more
        // (12288 x 2048 14.0 / 16.4, 14.2 / 17.4; 16384 x 1024 15.3 / 17.9, 15.7 / 19.1; 8192 x 3072 13.4 / 15.65, 13.3 / 16.0), but where the workgroups of 4096 columns take
        // every compute unit and memory is the bound whatever the part.  512 KB do not show (4096 x 1024 7.3, 15 splits 7.3; 2048 x 2048 6.0, 5.95), nor odd multiples of
        // them (11008 x 4096 16.7, 16.9).  Below twelve splits one fewer costs more (5120 x 5120 10 splits 13.95, 9 14.2; 1024 x 4096 8 splits 6.0, 7 6.2).
        const long long apart = (long long)(T / S) * N * 64;
        if (S >= 12 && T % S == 0 && apart % (1 << 20) == 0 && tuning_get(TUNE_DECODE_SPLIT) <= 0) {
            const bool takes_all = pl.tiles * S >= target;
            const bool short_part = T / S <= 16 && (apart & (apart - 1)) == 0 && (M <= 16 || pl.tiles * slices * S >= 128);
            if (takes_all || short_part) S -= T <= 128 ? 3 : 1;
        }
        // The sum over up to four splits is read four wide, over five to eight eight wide (finish_over_splits), which shows a little beyond 16 rows: four instead of five where
        // the slowest share of the waves has no more to walk then and parts are short (us, 5 -> 4: 768 x 12288 at 17 / 32 rows 9.4 / 9.55 -> 9.25 / 9.3, 1024 x 12288 11.0 / 10.95 -> 10.95 / 10.85; tiles of
        // 128, 896 x 5248 at 17 / 64 rows 7.2 / 9.7 -> 7.05 / 9.45, 1408 x 5248 7.9 / 10.6 -> 7.8 / 10.4, but 2048 x 6144 at 17 rows 10.25 -> 10.6).  Not in slices of 32 rows
        // (768 x 6144 at 33 / 64 rows 8.45 / 8.6 either way, 1024 x 6144 9.55 / 9.7 -> 9.8 / 9.85).
        const int shares = narrow ? 4 : 2;                // of a part among the waves
        auto slowest = [&](int s) { return ((T + s - 1) / s + shares - 1) / shares; };
        if (S == 5 && M > 16 && slices == 1 && T <= 48 && slowest(4) == slowest(5) && tuning_get(TUNE_DECODE_SPLIT) <= 0) S = 4;
    } else {
        S = split_for((M <= 16 && q != 0) ? T / 4 : halves);
    }
    // The native code order has the eight-wave kernel (decode_wide_kernel) from 9 to 32 rows, and below nine rows where a
    // workgroup is left with few groups to walk, which eight waves share out better than four (measured on the 7B shapes
    // at M = 1 and 4: o-proj, 2 groups per workgroup, 5.7 -> 5.4 us, down, 5.4 groups, 8.1 -> 7.7; qkv, 6.4 groups, 8.0 -> 8.4,
    // gate_up, 16 groups, 11.1 -> 12.4).
    bool wide = false;
    if (native && q == 1 && tuning_get(TUNE_SMALL) != 4) {
        wide = M > 8 || (T / 4) <= 6 * S || tuning_get(TUNE_SMALL) == 5;
        if (wide) S = split_for(halves);
    }
    pl.S = S;
    // vectors of four rows per tile: up to 16 rows only the groups of four that exist, beyond whole tiles of 16 rows
    const size_t nvec = (size_t)pl.tile_n * (M <= 16 ? (M + 3) / 4 : M > 32 && narrow ? 16 : 8);
    pl.wide = wide;
    pl.slices = slices;
    pl.partial_bytes = S > 1 ? (size_t)pl.tiles * slices * S * nvec * 16 : 0;
    // A look is one trip to the L2, 0.15 .. 0.3 us; the others of a unit normally follow within a few of them.  A workgroup
    // that starts after another one of its unit has already finished (compute units held up by other work) cannot tell
    // and waits the bound out before it recomputes: the bound is what such a launch costs, about 25 us (seen in
    // about one launch in a thousand when the grid takes every compute unit of the chip).
    pl.polls = tuning_get(TUNE_DECODE_SCATTER) == 3 ? 0 : 128;    // 3: nobody looks, every workgroup recomputes what it needs (test hook)
    pl.stream_loads = 1;
    pl.scatter = S > 1;
    return pl;
}

DecodePlan plan_decode(int q, int M, int K, int N, int native)
{
    const int t = tuning_get(TUNE_DECODE_SLICE);        // a forced slice height means the general streaming kernels
    const int small_rows = tuning_get(TUNE_SMALL) == 3 ? 16 : 64;       // 3: the register-tiled kernel only up to 16 rows
    if ((q == 0 || q == 1 || (q == 2 && M <= 16)) && M <= small_rows && tuning_get(TUNE_SMALL) != 2 && t != 16 && t != 32) {
        const DecodePlan ps = plan_small(q, M, K, N, native);
        // (tile and group counts travel in 16 bits each)
        if (ps.partial_bytes <= kSlotBytes && (ps.S == 1 || ps.tiles * ps.slices <= 256) && ps.tiles <= 65535 && K / kGroup <= 65535) return ps;
    }
    if (t == 16 || t == 32) return plan_rows(q, M, K, N, t);
    if (M <= 16) return plan_rows(q, M, K, N, 16);
    const DecodePlan p32 = plan_rows(q, M, K, N, 32);
    if (q != 1 || M > 64) return p32;
    const DecodePlan p16 = plan_rows(q, M, K, N, 16);
    if (p16.tiles * p16.slices * p16.S > 256) return p32;
    return p16.est_us < p32.est_us ? p16 : p32;
}

// Dense weights in column tiles of 128 instead of 256 (small = 0: not here).  Up to 32 rows a workgroup loads half as many columns, which for the same number of
// workgroups takes half the splits, and a tile count that fits the chip better or, for matrices of few columns (at most 16 splits), up to twice the workgroups; but
// its reads are pieces of 256 bytes of a row.  us, tiles of 256 -> of 128:
//   - more workgroups, at 1 / 7 / 24 rows: 8192 x 1024 (60 -> 120) 9.9 / 10.1 / 12.4 -> 8.1 / 8.0 / 9.55; 4096 x 1024 7.0 / 7.2 / 8.9 -> 5.8 / 5.8 / 7.1; 8192 x 2048 (120 -> 240)
//     11.3 / 11.5 / 14.2 -> 9.9 / 9.7 / 11.4; 14336 x 5120 (200 -> 240) 31.9 / 32.4 / 36.2 -> 29.6 / 28.8 / 31.2; 5120 x 5120 14.5 -> 12.7 at 7; 1024 x 1024 (32 -> 64) 5.0 / 5.1 / 6.6 ->
//     4.7 / 4.8 / 5.9; 2048 x 2048 5.8 / 5.9 / 7.5 -> 5.5 / 5.6 / 7.0; not where the few splits start whole megabytes apart (see above: 4096 x 4096 9.75 / 9.9 -> 10.0 / 9.8);
//   - about as many: beyond 16 rows, where the hand-over is the larger, with up to 48 k-steps to a part (3584 x 3584 at 24 rows 11.0 -> 10.3, 6144 x 6144 19.8 -> 19.3; 74 steps
//     of 18944 x 3584 29.75 -> 30.2, 80 of 5120 x 13824 31.3 -> 33.8); below, 0.96 .. 1.05;
//   - fewer: 1.03 .. 1.10 (4096 x 12288, 240 -> 192, 20.8 -> 22.7 at 7 rows).
// Beyond 32 rows the plan above has slices of 32 rows, each of which reads the matrix; here all rows are in one workgroup, and it is read once.  us at 33 / 64 rows, slices (or the LDS ring,
// which took most matrices from 26e6 weights on) -> one pass: 4096 x 11008 30.5 / 31.0 -> 26.4 / 27.0, 4096 x 22016 54.8 / 55.9 -> 44.9 / 47.4, 5120 x 5120 23.7 / 24.5 -> 18.2 / 18.7,
// 5120 x 27648 71.3 / 72.0 -> 58.0 / 61.3, 13824 x 5120 45.6 / 46.7 -> 34.9 / 36.3, 11008 x 4096 26.6 / 27.2 -> 24.2 / 25.3, 6144 x 4096 17.1 / 17.7 -> 16.8 / 17.3.  But a workgroup loads
// and hands on twice the rows: where a part has up to 16 k-steps (4096 x 4096 13.6 -> 14.2, 1024 x 4096 8.2 -> 9.0, 512 x 2048 7.1 -> 7.9) that gains only by more workgroups
// (2048 x 5120, 200 -> 240: 12.8 -> 11.9; 4096 x 3072, 192 -> 240: 13.7 -> 13.1; 3072 x 3072 the same, 11.7 -> 11.4), and where split parts on a full chip (240 workgroups and more) have up to 22
// (33 / 64 rows: 2816 x 8192 16.05 / 15.7 -> 16.5 / 16.25, 5632 x 4096 15.1 / 15.3 -> 15.8 / 16.0, 8192 x 2048 13.5 / 13.7 -> 14.2 / 14.15; but 24, 3072 x 8192, 17.2 / 17.0 -> 16.8 / 16.7, and on 198 workgroups
// 18, 1664 x 8448 at 48, 14.1 -> 13.8).  Where rows do not start on cache lines, a piece of 256 bytes touches
// three lines instead of two, which a chip two thirds full does not hide (4224 x 11016, 174 workgroups, 31.2 / 32.2 -> 31.7 / 34.2; 5120 x 13832, 218, 41.9 / 42.3 -> 38.0 / 40.5;
// 8064 x 12192, 192, 51.3 / 52.1 -> 49.1 / 55.0; 7296 x 20488, 161 with 228 k-steps each, 91.7 / 92.8 -> 83.0 / 95.5, 4096 x 20488, 128 k-steps, 54.6 / 55.7 -> 47.9 / 52.2).  And up to 160 workgroups leave matrices that the ring takes
// to it: tiles of 256 columns still come three to a tile there (4096 x 18432, 144 workgroups against 216, 42.9 / 43.8 -> 44.2 / 48.0; 7296 x 18432 67.9 / 67.9 -> 76.8 / 84.2; 2048 x 17000, 133, 26.2 / 27.5
// -> 27.4 / 28.5; 4096 x 20488, 161 against 162, above; 1280 x 16792, which the ring does not take, 26.8 / 26.6 -> 18.8 / 19.6).
// Beyond 256 tiles (32768 columns, K in one part) what counts is the rounds in which the compute units take the tiles, two of 128 columns to one of 256.  Up to 32 rows: fewer rounds pay
// from 21 k-steps on (70000 columns, 3 halves against 4, at 1 / 24 rows: 1024 rows of K 36.2 / 42.4 -> 32.2 / 38.2, 512 18.9 / 22.4 -> 18.5 / 23.4; 151936 columns, 5 against 6: 4096 208.9 / 221.9 ->
// 194.7 / 211.4, 640 37.3 / 43.2 -> 37.5 / 45.7), as many do not (5120 x 33024 72.0 / 80.0 -> 78.7 / 86.7, 1024 x 50304 18.7 / 21.1 -> 21.6 / 25.5, 4096 x 128256 24 rows 170.5 -> 183.5).  At 33 .. 64 rows
// the ring reads the matrix once as well, in tiles of 256 (the slices twice).  Fewer rounds pay there too (33 / 64 rows: 4096 x 70000 176.0 / 179.9 -> 133.7 / 142.1, 768 x 98304 41.3 / 41.9 -> 37.1 / 39.3); as
// many do from 48 k-steps on and on cache lines, if the last round of tiles of 256 leaves compute units idle (4096 x 33024 84.7 / 85.9 -> 71.1 / 74.7, 5120 x 64256 125.3 / 127.1 -> 111.5 / 119.4, 4096 x 128256
// 208.3 / 213.9 -> 184.6 / 200.8, 1536 x 57344 41.2 / 41.8 -> 40.6 / 42.0; but 4096 x 131072 205.6 / 209.6 -> 202.7 / 217.8, 1024 x 33024 23.7 / 24.5 -> 24.9 / 26.0, 3072 x 33032 65.4 / 65.3 -> 65.6 / 69.7).
DecodePlan plan_narrow(int M, int K, int N)
{
    if (M > 64) return DecodePlan{};
    const DecodePlan wide = plan_decode(0, M, K, N);
    if (!wide.small) return DecodePlan{};
    const DecodePlan pl = plan_small(0, M, K, N, 0, true);
    if (pl.partial_bytes > kSlotBytes || (pl.S > 1 && (pl.tiles > 256 || wide.S == 1)) || pl.tiles > 65535) return DecodePlan{};   // (no workspace where none was asked for)
    if (tuning_get(TUNE_SMALL) == 6) return pl;
    const int  T = K / 32, steps = (T + pl.S - 1) / pl.S, wgs = pl.tiles * pl.S, wgs_wide = wide.tiles * wide.slices * wide.S;
    const int  cus = prefill_compute_units();
    const bool more = 8 * wgs >= 9 * wgs_wide;
    bool take;
    if (wgs > cus) {
        auto rounds = [&](int n) { return (n + cus - 1) / cus; };
        const bool ring  = M > 32 && (double)K * N >= 26e6;
        const bool fewer = rounds(wgs) < 2 * rounds(ring ? wide.tiles : wgs_wide);
        take = fewer ? steps > (M > 32 ? 16 : 20) : ring && steps >= 48 && N % 64 == 0 && wide.tiles % cus != 0;
    } else if (M > 32) take = (steps > (pl.S > 1 && 16 * wgs >= 15 * cus ? 22 : 16) || (steps > 8 && more)) && !(N % 64 != 0 && wgs <= 192 && (pl.S > 1 || steps > 128)) && !(wgs <= 160 && (double)K * N >= 26e6);
    else if (more) take = M > 16 || pl.S >= 12 || steps < 16 || T % pl.S != 0 || (long long)steps * N * 64 % (1 << 20) != 0;
    else take = M > 16 && 16 * wgs >= 15 * wgs_wide && steps <= 48;
    return take ? pl : DecodePlan{};
}

hipError_t launch_decode(int q, const DecodeArgs& a, hipStream_t st)
{
    const int rows = a.rows;
    if (rows != 16 && rows != 32) return hipErrorInvalidValue;
    const int slices = (a.M + rows - 1) / rows;
    const bool one   = rows == 16;                       // a single 16-row MFMA tile
    return a.bf ? launch_format<true>(q, one, a, slices, st) : launch_format<false>(q, one, a, slices, st);
}

}  // namespace morph
