// What the two LDS-ring kernels (tiled.hip, tiled_exact.hip) share: asynchronous loads into LDS and the waits for
// them, the place of a workgroup, the sum over the parts of K inside a workgroup, and the hand-over between the
// workgroups that split K.
//
// Both kernels keep everything they read from memory -- x and the weights as they are stored -- in a ring of stages in
// LDS that is filled by buffer_load ... lds (no staging registers, several microseconds' worth in flight) and read
// back as matrix-core operands: x rows as A of v_mfma_f32_16x16x32, the weights unpacked in registers as B.  A wave
// owns 64 columns of the workgroup's tile and MT tiles of 16 rows, so a weight is unpacked once per wave that needs
// it and never written back to LDS.
#pragma once
#include "dev_common.h"
#include "kernels.h"
#include "ticks.h"

namespace morph {

// What the hand-over at the end needs (fetched when it is reached).
struct TiledTail {
    void*     y;
    uint32_t* slots;                                     // [unit][split][vector] f32x4 partial sums (no content between launches)
    int*      ctl;                                       // kSmallCtlInts per unit
    int       polls;                                     // looks at the flags before a workgroup stops waiting
    int       far;                                       // write the hand-over through to memory instead of leaving it in the L2
};

// One asynchronous load of 16 (4) bytes per lane straight into LDS: lane l's bytes land at lds + 16 l (4 l); lanes whose
// offset lies past the buffer write zeros.  (Measured on the device: any LDS offset up to 160 KB, any source address
// that is a multiple of 4.)  Assembly, because the compiler would wait for all of them before any read of LDS; it does
// not see these loads, and the waits are wait_vm() below, counted by hand.  A load or a reload from scratch memory that the
// compiler adds only makes those waits longer.
// s_nop 4: a vector instruction that writes a scalar register and a memory instruction that reads it need five wait states between them.  The
// compiler keeps them for its own loads and does not look in here, and it brings descriptor words and offsets that it has parked in vector lanes back with
// v_readlane right before the block.  The five states also cover the one that m0 needs.  m0, where the LDS address goes, is an operand,
// so that the compiler writes it and knows what it holds (as a clobber it is a reserved register and draws a warning).
template <bool NT>
__device__ __forceinline__ void dma16(uint32_t lds, uint32_t voff, u32x4 rsrc, uint32_t soff)
{
    if constexpr (NT) asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds" ::"{m0}"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
    else              asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"{m0}"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
__device__ __forceinline__ void dma4(uint32_t lds, uint32_t voff, u32x4 rsrc, uint32_t soff)
{
    asm volatile("s_nop 4\n\tbuffer_load_dword %1, %2, %3 offen lds" ::"{m0}"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
// until at most N of this wave's loads are outstanding (they return in order)
template <int N>
__device__ __forceinline__ void wait_vm()
{
    static_assert(N >= 0 && N <= 63, "the counter holds six bits");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// barrier of the workgroup; this wave's reads and writes of LDS are done, its loads from memory may go on
__device__ __forceinline__ void wg_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// the words of a raw buffer descriptor (as make_rsrc), in scalar registers
__device__ __forceinline__ u32x4 rsrc_words(const void* base, uint32_t bytes)
{
    const uint64_t a = (uint64_t)base;
    return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a), (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xFFFFu)),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes), 0x00020000u};
}
// the same, or a buffer of no bytes (every lane of a load then writes zeros)
__device__ __forceinline__ u32x4 rsrc_if(u32x4 r, bool live) { return u32x4{r[0], r[1], live ? r[2] : 0u, r[3]}; }

template <bool BF>
__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c)
{
    if constexpr (BF) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(bit_cast<bf16x8_t>(a), bit_cast<bf16x8_t>(b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_f16(bit_cast<half8_t>(a), bit_cast<half8_t>(b), c, 0, 0, 0);
}

// Which (column tile, slice of rows, part of K) a workgroup is.  Workgroup L runs on XCD L % 8.  The units (tile, slice),
// slices of a tile next to each other, are dealt to the XCDs in runs of `per` = ceil(units / 8): the XCDs carry the
// same number of units whatever their count, the workgroups of a unit share an L2, and so do most slices of a tile.
// Units that do not exist have tile >= tiles.
struct TiledPlace { int tile, slice, sp, unit; };
__device__ __forceinline__ TiledPlace tiled_place(int S, int slices, int per)
{
    const int L = blockIdx.x, xcd = L & 7, jj = L >> 3;
    TiledPlace p;
    const int j = jj / S;
    p.sp = jj - j * S;
    p.unit = xcd * per + j;
    p.tile = p.unit / slices;
    p.slice = p.unit - p.tile * slices;
    return p;
}

// Groups of 128 rows of K of a split, cut into KW parts; g0, g1 of part kg; returns how many groups are walked.
struct TiledRange { int gb, ng; };
__device__ __forceinline__ TiledRange tiled_range(int qr, int split)
{
    const int q = qr & 0xFFFF, r = qr >> 16;
    return TiledRange{split * q + (split < r ? split : r), q + (split < r ? 1 : 0)};
}

// A wave's results: yr[mt][e] = rows 16 (rw MT + mt) + 4 b .. + 3 of the lane's column e (of four).  Wave (kg, rw, cw).
// Vector number of (rw, cw, mt, e, lane) = (((rw CW + cw) MT + mt) 4 + e) 64 + lane.
template <int MT, int RW, int CW, int KW>
struct TiledGeom {
    static constexpr int kThreads = RW * CW * KW * 64;
    static constexpr int kVecs = RW * CW * MT * 4 * 64;
    static constexpr int kKept = MT * 4 / KW;            // (mt, e) pairs a wave keeps after the parts of K have met
    static_assert(MT * 4 % (2 * KW) == 0, "pairs of columns stay together");
    static constexpr int kRedBytes = RW * CW * KW * MT * 4 * 1024 * (KW - 1) / KW;
    static __device__ __forceinline__ bool kept(int p, int kg) { return KW == 1 || p / kKept == kg; }
};

// The KW parts of K meet: the waves of part kg keep the kg-th share of the (mt, e) pairs and add the others', in the order of the
// parts.  `red`: kRedBytes of LDS that nothing else uses any more.
template <int MT, int RW, int CW, int KW>
__device__ __forceinline__ void tiled_meet(f32x4 (&yr)[MT][4], f32x4* red, int kg, int rc, int lane)
{
    if constexpr (KW > 1) {
        constexpr int PK = TiledGeom<MT, RW, CW, KW>::kKept;
        auto at = [&](int owner, int from, int p) -> f32x4& {
            return red[((((owner * (KW - 1) + (from < owner ? from : from - 1)) * PK + p % PK) * (RW * CW)) + rc) * 64 + lane];
        };
#pragma unroll
        for (int p = 0; p < MT * 4; p++)
            if (p / PK != kg) at(p / PK, kg, p) = yr[p >> 2][p & 3];
        wg_barrier();
#pragma unroll
        for (int p = 0; p < MT * 4; p++) {
            if (p / PK != kg) continue;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < KW; i++) {
                if (i == kg) acc += yr[p >> 2][p & 3];
                else acc += at(kg, i, p);
            }
            yr[p >> 2][p & 3] = acc;
        }
    }
}

// The unit's flags as they stand when the workgroup starts (first wave, lane q: split q).
__device__ __forceinline__ uint32_t tiled_flags(const TiledTail& t, int S, int unit, int wave, int lane)
{
    if (S > 1 && wave == 0 && lane < S) {
        const __amdgpu_buffer_rsrc_t rc = make_rsrc(t.ctl + (size_t)unit * kSmallCtlInts, kSmallCtlInts * 4u);
        return __builtin_amdgcn_raw_buffer_load_b32(rc, (uint32_t)lane * 4u, 0, kAuxSystemScope);
    }
    return 0;
}

// Runs the workgroup's pass and writes y (rows from this slice's first on, M rows).  With K split over S workgroups this is
// the hand-over of decode_small.hip (see finish_over_splits there: flags that only move, bounded wait, a workgroup
// whose wait runs out works the missing parts out itself, sums in split order whoever adds them), on this file's
// vectors.  col0(cw, c): first of the four columns of lane group c of column wave cw.
template <bool BF, int MT, int RW, int CW, int KW, class Begin, class Pass, class Col0>
__device__ __forceinline__ void tiled_finish(const TiledTail& t, int S, const TiledPlace& p, int M, int N, uint16_t* y, uint32_t base,
                                             uint32_t* fresh_word, f32x4 (&yr)[MT][4], Begin&& begin, Pass&& pass, Col0&& col0)
{
    typedef TiledGeom<MT, RW, CW, KW> G;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave / (RW * CW), rw = (wave / CW) % RW, cw = wave % CW;
    auto pack2 = [](float a, float b) { return (uint32_t)narrow16<BF>(a) | ((uint32_t)narrow16<BF>(b) << 16); };
    if (S == 1) {
        pass();
        const int col = col0(cw, lane & 15);
        if (col < N) {
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const int row = 16 * (rw * MT + mt) + 4 * (lane >> 4) + r;
                    if (row >= M) continue;
                    uint16_t* yp = y + (size_t)row * N + col;
                    if (G::kept(4 * mt, kg) && G::kept(4 * mt + 2, kg))
                        *reinterpret_cast<u32x2*>(yp) = u32x2{pack2(yr[mt][0][r], yr[mt][1][r]), pack2(yr[mt][2][r], yr[mt][3][r])};
                    else if (G::kept(4 * mt, kg)) *reinterpret_cast<uint32_t*>(yp) = pack2(yr[mt][0][r], yr[mt][1][r]);
                    else if (G::kept(4 * mt + 2, kg)) *reinterpret_cast<uint32_t*>(yp + 2) = pack2(yr[mt][2][r], yr[mt][3][r]);
                }
        }
        return;
    }
    constexpr uint32_t slot_bytes = (uint32_t)G::kVecs * 16u;
    const __amdgpu_buffer_rsrc_t rc = make_rsrc(t.ctl + (size_t)p.unit * kSmallCtlInts, kSmallCtlInts * 4u);
    const __amdgpu_buffer_rsrc_t rp = make_rsrc(t.slots + (size_t)p.unit * S * G::kVecs * 4, (uint32_t)S * slot_bytes);
    uint32_t my_xcc;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(my_xcc));
    const uint32_t where = t.far ? 0u : (my_xcc & 0xFu) + 1u;
    // My share: with up to four splits, quads (the four columns of a lane) v0 .. v1 - 1; beyond, vectors: every thread
    // then has about one vector of every split to fetch, all of them in flight at once, instead of a quarter of
    // the threads four.
    const bool quads = S <= 4;
    const int nv = quads ? G::kVecs / 4 : G::kVecs;
    const int v0 = (p.sp * nv) / S, v1 = ((p.sp + 1) * nv) / S;
    auto put_all = [&](int split, int q0, int q1) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < MT * 4; i++) {
            const int mt = i >> 2, e = i & 3;
            if (!G::kept(i, kg) || 16 * (rw * MT + mt) >= M) continue;
            const int blk = (rw * CW + cw) * MT + mt, vec = (blk * 4 + e) * 64 + lane, mine = quads ? blk * 64 + lane : vec;
            if (mine < q0 || mine >= q1) continue;
            const uint32_t off = (uint32_t)split * slot_bytes + (uint32_t)vec * 16u;
            if (where) __builtin_amdgcn_raw_buffer_store_b128(bit_cast<u32x4>(yr[mt][e]), rp, off, 0, 0);
            else __builtin_amdgcn_raw_buffer_store_b128(bit_cast<u32x4>(yr[mt][e]), rp, off, 0, kAuxSystemScope);
        }
    };
    pass();
    put_all(p.sp, 0, G::kVecs);
    MORPH_TICK(4);
    wait_stores();
    __syncthreads();
    MORPH_TICK(5);
    const uint32_t want = (1u << S) - 1u;
    if (wave == 0) {
        if (lane == p.sp) {
            const uint32_t up = (((base >> 4) + 1u) << 4) | where;
            if (where) __builtin_amdgcn_raw_buffer_store_b32(up, rc, (uint32_t)p.sp * 4u, 0, 0);
            else __builtin_amdgcn_raw_buffer_store_b32(up, rc, (uint32_t)p.sp * 4u, 0, kAuxSystemScope);
        }
        uint32_t moved = 1u << p.sp, usable = 1u << p.sp;
        for (int look = 0; look < t.polls && moved != want; look++) {
            asm volatile("" ::: "memory");
            uint32_t f = base;
            if (lane < S) f = __builtin_amdgcn_raw_buffer_load_b32(rc, (uint32_t)lane * 4u, 0, kAuxSystemScope);
            asm volatile("" ::: "memory");
            moved  = ((uint32_t)__builtin_amdgcn_ballot_w64((f >> 4) != (base >> 4)) & want) | (1u << p.sp);
            usable = ((uint32_t)__builtin_amdgcn_ballot_w64((f >> 4) != (base >> 4) && ((f & 15u) == 0u || (f & 15u) == (my_xcc & 0xFu) + 1u)) & want) | (1u << p.sp);
        }
        if (lane == 0) *fresh_word = usable;
    }
    __syncthreads();
    const uint32_t fresh = *fresh_word;
    MORPH_TICK(6);
    if (fresh != want) {                                 // the slow way, for every split that is not there
        for (int q = 0; q < S; q++) {
            if ((fresh >> q) & 1) continue;
            __syncthreads();
            begin(q);
            pass();
            put_all(q, v0, v1);
        }
        wait_stores();
        __syncthreads();
    }
    auto get = [&](int q, int vec) __attribute__((always_inline)) {  // (splits that do not exist lie past the buffer: zeros)
        return __builtin_amdgcn_raw_buffer_load_b128(rp, q < S ? (uint32_t)q * slot_bytes + (uint32_t)vec * 16u : 0xFFFFFFF0u, 0, kAuxSystemScope);
    };
    for (int v = v0 + tid; v < v1; v += G::kThreads) {
        const int blk = quads ? v >> 6 : v >> 8, ln = v & 63;
        const int mt = blk % MT, cw_ = (blk / MT) % CW, rw_ = blk / (MT * CW);
        const int row = 16 * (rw_ * MT + mt) + 4 * (ln >> 4), col = col0(cw_, ln & 15);
        asm volatile("" ::: "memory");
        if (quads) {
            u32x4 f[4][4];
#pragma unroll
            for (int q = 0; q < 4; q++)
#pragma unroll
                for (int e = 0; e < 4; e++) f[q][e] = get(q, (blk * 4 + e) * 64 + ln);
            f32x4 acc[4] = {};
#pragma unroll
            for (int q = 0; q < 4; q++)
#pragma unroll
                for (int e = 0; e < 4; e++)
                    if (q < S) acc[e] += bit_cast<f32x4>(f[q][e]);
            if (col < N) {
#pragma unroll
                for (int r = 0; r < 4; r++)
                    if (row + r < M) *reinterpret_cast<u32x2*>(y + (size_t)(row + r) * N + col) = u32x2{pack2(acc[0][r], acc[1][r]), pack2(acc[2][r], acc[3][r])};
            }
        } else {
            u32x4 f[16];
#pragma unroll
            for (int q = 0; q < 16; q++) f[q] = get(q, v);
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 16; q++)
                if (q < S) acc += bit_cast<f32x4>(f[q]);
            const int e = (v >> 6) & 3;
            if (col < N) {
#pragma unroll
                for (int r = 0; r < 4; r++)
                    if (row + r < M) y[(size_t)(row + r) * N + col + e] = narrow16<BF>(acc[r]);
            }
        }
    }
    MORPH_TICK(7);
}

}  // namespace morph
