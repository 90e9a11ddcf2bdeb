// Quantizer (fp32/fp16/bf16 weights -> 4-bit or 8-bit layer record) and the verification dequantizer.
// Format and arithmetic: see include/morph.h.  Both are exact procedures with one right answer;
// neither sits on the per-token path.  Both work on units of 8 columns x 8 rows per thread.
#include "dev_common.h"
#include "kernels.h"

namespace morph {

// ---- quantizer ----
// Bound: memory at fp32 sources (5.3 TB/s); at 16-bit ones the bytes and about eight vector instructions per weight, which overlap as
// far as independent workgroups share a compute unit.  A thread keeps 8 columns of 8 consecutive rows in registers from the load to
// the codes, 16-bit sources as stored, so that three workgroups of 512 threads fit a compute unit (two with widened values);
// what crosses threads are the column ranges of a workgroup's 16 row octets (one exchange through LDS) and the scales
// and zero points on their way back (a second one).  Workgroup = one group of 128 rows x kQU column units of 8.
// Measured (cold, to the 4-bit record, us; before = widened values, ranges in fp32, words near a half-integer divided): bfloat16 4096 x 22016 51.5 -> 39.5
// (5.7 TB/s), 4096 x 4096 14.5 -> 10.8, 1024 x 1288 7.3 -> 4.7; fp16 48.3 -> 41.0, 13.3 -> 11.9, 7.2 -> 4.7; 8 bits from bfloat16 51.6 -> 46.4, 15.1 -> 11.6,
// 8.0 -> 4.9; fp32 the same (78.0 -> 77.7, 16.5 -> 16.2, 7.0 -> 6.7); the native order within 3 % of these.
//
// The code of a weight is rint(v / s) + z clamped to 0 .. L, the division correctly rounded.  A scale has 11 significant bits, so
// that three instructions divide: r = 1 / s correctly rounded, q = v r, e = v - q s, and q + e r, rounded once, is the rounded quotient.
// q is off by at most 2^-23 of itself, hence e has at most 13 bits and is exact; q + e r is then within 2^-47 of v / s, relatively, before its
// rounding.  A quotient of a 24-bit by an 11-bit number that is no 25-bit number stays 2^-36 away from all of them, and it never is one with an odd last
// bit (v would have 25 bits): no rounding boundary lies between the two.  (Quotients so small that e underflows are 0 rounded either way; no
// finite quotient overflows, as s is at least 2^-14 and a group's range / L, or 65504.)  Adding 1.5 * 2^23 rounds to an integer, halves
// to even; clamped to [1.5 * 2^23 - z, + L] the codes of a word are the bits' differences from the lower bounds.  Infinities and NaN make e NaN: a
// thread that has one among its 64 weights works all of them out by dividing.
// Before, v r alone was rounded and the words in which some lane came close to a half-integer were divided again; bfloat16 weights, which have 8 bits,
// meet half-integers so often that this was a quarter of the instructions.
constexpr float kMagic = 12582912.0f;                     // 1.5 * 2^23, bit pattern 0x4B400000

template <int BITS>
__device__ __forceinline__ uint32_t code_divided(float v, float s, float z)
{
    constexpr float L = (float)((1 << BITS) - 1);
    const float t = rintf(__fdiv_rn(v, s));
    // in floating point to the end: an integer holds neither infinities nor quotients beyond 2^31 plus z (t + z is exact where it matters; NaN: the code of 0)
    return (uint32_t)__builtin_amdgcn_fmed3f(t == t ? t + z : z, 0.0f, L);
}

// the 8 columns of a row, widened
template <typename WT> struct RowOf8;
template <> struct RowOf8<float> {
    f32x4 v[2];
    __device__ __forceinline__ void load(const float* p)
    {
        v[0] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
        v[1] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p) + 1);
    }
    __device__ __forceinline__ void zero() { v[0] = v[1] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    __device__ __forceinline__ void apart() {}
    __device__ __forceinline__ float at(int j) const { return v[j >> 2][j & 3]; }
};
template <bool BF> struct Row16 {
    u32x4 v;
    template <typename T> __device__ __forceinline__ void load(const T* p) { v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)); }
    __device__ __forceinline__ void zero() { v = u32x4{0u, 0u, 0u, 0u}; }
    // what is widened from here on is not shared with what was before (64 widened values would take twice the registers)
    __device__ __forceinline__ void apart() { asm volatile("" : "+v"(v)); }
    __device__ __forceinline__ float at(int j) const
    {
        if constexpr (BF) return bit_cast<float>((j & 1) ? v[j >> 1] & 0xFFFF0000u : v[j >> 1] << 16);
        else return (float)bit_cast<half8_t>(v)[j];
    }
};
template <> struct RowOf8<half_t> : Row16<false> {};
template <> struct RowOf8<bf16_t> : Row16<true> {};

// Smallest and largest of 0 and the values of 8 rows, column by column, NaN passed over.
// 16-bit values are compared as the integers of their bits, two to an instruction and without widening them (which would be
// a third of the kernel's instructions and, kept for the codes, half of its registers): as signed integers the largest is the largest
// positive value, as unsigned ones with -0 among them the most negative.  Only NaN lies beyond the infinities there: with one, all
// NaN become 0 first.
template <typename WT> struct ColumnRanges {
    typedef uint16_t Part;
    typedef int16_t  i16x8 __attribute__((ext_vector_type(8)));
    typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
    static constexpr bool     kBf  = __is_same(WT, bf16_t);
    static constexpr uint16_t kInf = kBf ? 0x7F80 : 0x7C00;
    u32x4 lo, hi;
    __device__ __forceinline__ void take(const u32x4& w)
    {
        lo = bit_cast<u32x4>(__builtin_elementwise_max(bit_cast<u16x8>(lo), bit_cast<u16x8>(w)));
        hi = bit_cast<u32x4>(__builtin_elementwise_max(bit_cast<i16x8>(hi), bit_cast<i16x8>(w)));
    }
    __device__ __forceinline__ bool over(const RowOf8<WT> (&v)[8])   // true: an infinity or NaN is among them
    {
        lo = u32x4{0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
        hi = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < 8; i++) take(v[i].v);
        const u16x8 out = bit_cast<u16x8>((bit_cast<i16x8>(hi) >= (int16_t)kInf) | (bit_cast<u16x8>(lo) >= (uint16_t)(kInf | 0x8000u)));
        const u32x4 any = bit_cast<u32x4>(out);
        const bool odd = (any[0] | any[1] | any[2] | any[3]) != 0u;
        if (__builtin_expect(odd, 0)) {
            lo = u32x4{0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
            hi = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int i = 0; i < 8; i++) {
                const u16x8 w = bit_cast<u16x8>(v[i].v);
                take(bit_cast<u32x4>(w & bit_cast<u16x8>((w & (uint16_t)0x7FFF) <= kInf)));
            }
        }
        return odd;
    }
    __device__ __forceinline__ void join_lane(int d)
    {
        u32x4 l, h;
#pragma unroll
        for (int k = 0; k < 4; k++) { l[k] = __shfl_xor(lo[k], d, 64); h[k] = __shfl_xor(hi[k], d, 64); }
        lo = bit_cast<u32x4>(__builtin_elementwise_max(bit_cast<u16x8>(lo), bit_cast<u16x8>(l)));
        hi = bit_cast<u32x4>(__builtin_elementwise_max(bit_cast<i16x8>(hi), bit_cast<i16x8>(h)));
    }
    __device__ __forceinline__ void park(Part* pl, Part* ph) const
    {
        *reinterpret_cast<u32x4*>(pl) = lo;
        *reinterpret_cast<u32x4*>(ph) = hi;
    }
    static __device__ __forceinline__ float widen(Part b) { return widen16<kBf>(b); }
};
template <> struct ColumnRanges<float> {
    typedef float Part;
    float lo[8], hi[8];
    __device__ __forceinline__ bool over(const RowOf8<float> (&v)[8])
    {
        float far = 0.f;
#pragma unroll
        for (int j = 0; j < 8; j++) {
            lo[j] = hi[j] = 0.f;
#pragma unroll
            for (int i = 0; i < 8; i++) {
                lo[j] = __builtin_fminf(lo[j], v[i].at(j));
                hi[j] = __builtin_elementwise_maximum(hi[j], v[i].at(j));     // NaN stays
            }
            far = __builtin_elementwise_maximum(far, __builtin_elementwise_maximum(hi[j], -lo[j]));
        }
        const bool odd = !(far < __builtin_inff());
        if (__builtin_expect(odd, 0)) {
#pragma unroll
            for (int j = 0; j < 8; j++) {
                hi[j] = 0.f;
#pragma unroll
                for (int i = 0; i < 8; i++) hi[j] = __builtin_fmaxf(hi[j], v[i].at(j));
            }
        }
        return odd;
    }
    __device__ __forceinline__ void join_lane(int d)
    {
#pragma unroll
        for (int j = 0; j < 8; j++) {
            lo[j] = __builtin_fminf(lo[j], __shfl_xor(lo[j], d, 64));
            hi[j] = __builtin_fmaxf(hi[j], __shfl_xor(hi[j], d, 64));
        }
    }
    __device__ __forceinline__ void park(Part* pl, Part* ph) const
    {
        f32x4* const l = reinterpret_cast<f32x4*>(pl);
        f32x4* const h = reinterpret_cast<f32x4*>(ph);
        l[0] = f32x4{lo[0], lo[1], lo[2], lo[3]}; l[1] = f32x4{lo[4], lo[5], lo[6], lo[7]};
        h[0] = f32x4{hi[0], hi[1], hi[2], hi[3]}; h[1] = f32x4{hi[4], hi[5], hi[6], hi[7]};
    }
    static __device__ __forceinline__ float widen(Part v) { return v; }
};

// BITS = 4: 15 steps, eight codes per word; BITS = 8: 255 steps, four codes per word.
// WT: float, or a 16-bit type (half_t, bf16_t) whose values are widened exactly.
// native: also (qweight given) or only (qweight NULL) write the 4-bit codes in the native order, see below.
template <typename WT, int BITS, int kQU>
__global__ __launch_bounds__(kQU * 16, sizeof(WT) == 2 ? 6 : 4) void quantize_kernel(const WT* __restrict__ w, uint32_t* __restrict__ qweight,
                                                            half_t* __restrict__ scales, uint32_t* __restrict__ qzeros,
                                                            u32x4* __restrict__ native, int K, int N)
{
    constexpr int   L = (1 << BITS) - 1;                    // largest code
    constexpr int   CPW = 32 / BITS, WPU = 8 / CPW;         // codes per word, words per unit of 8 columns
    constexpr int   kQC = 8 * kQU, kThreads = 16 * kQU, kWaves = kThreads / 64;
    __shared__ __align__(16) typename ColumnRanges<WT>::Part part[2][kWaves][kQC];
    __shared__ __align__(16) float col[3][kQC];             // s, 1 / s and 1.5 * 2^23 - z of a column
    const int tid = threadIdx.x, wave = tid >> 6;
    const int u = tid & (kQU - 1), oct = tid / kQU;
    const int NW = N / CPW;
    // Workgroup L runs on XCD L % 8.  Where the number of column tiles is a power of two, an XCD would see the same few columns of every group, and with
    // the rows' pitch a power of two the same channels of its L2: the tiles of a group move on by one from group to group there (fp32, 4096 x 4096
    // 21.6 -> 16.4 us, 14336 x 4096 60.4 -> 50.2; elsewhere it would cost the division by an odd number, 1 %).
    const int bx = (gridDim.x & (gridDim.x - 1)) == 0 ? (int)((blockIdx.x + blockIdx.y) & (gridDim.x - 1)) : (int)blockIdx.x;
    const int n0 = bx * kQC, n = n0 + 8 * u;
    const int g  = blockIdx.y;
    const bool live = n < N;
    const size_t row0 = (size_t)g * kGroup + 8 * oct;

    RowOf8<WT> v[8];
    if (live) {
#pragma unroll
        for (int i = 0; i < 8; i++) v[i].load(w + (row0 + i) * N + n);
    } else {
#pragma unroll
        for (int i = 0; i < 8; i++) v[i].zero();
    }

    // ---- column ranges, widened to contain 0: 8 rows, the octets of the wave, the waves ----
    ColumnRanges<WT> cr;
    const bool odd = cr.over(v);
#pragma unroll
    for (int d = kQU; d < 64; d *= 2) cr.join_lane(d);
    if ((tid & 63) < kQU) cr.park(&part[0][wave][8 * u], &part[1][wave][8 * u]);
    __syncthreads();
    int zz = 0;
    if (tid < kQC) {                                        // one thread per column (kQC <= kThreads)
        float l = ColumnRanges<WT>::widen(part[0][0][tid]), h = ColumnRanges<WT>::widen(part[1][0][tid]);
#pragma unroll
        for (int q = 1; q < kWaves; q++) {
            l = __builtin_fminf(l, ColumnRanges<WT>::widen(part[0][q][tid]));
            h = __builtin_fmaxf(h, ColumnRanges<WT>::widen(part[1][q][tid]));
        }
        const float s32 = __fdiv_rn(h - l, (float)L);
        half_t   s    = (half_t)s32;                        // round to nearest even
        uint16_t bits = bit_cast<uint16_t>(s);
        if ((float)s < s32) bits = (uint16_t)(bits + 1);    // round the step size up
        if (bits < 0x0400u) bits = 0x0400u;                 // at least 2^-14 (stay normal)
        if (bits > 0x7BFFu) bits = 0x7BFFu;                 // at most 65504
        s = bit_cast<half_t>(bits);
        const float sf = (float)s;
        zz = (int)__builtin_amdgcn_fmed3f(rintf(__fdiv_rn(-l, sf)), 0.0f, (float)L);
        col[0][tid] = sf;
        col[1][tid] = __fdiv_rn(1.0f, sf);
        col[2][tid] = kMagic - (float)zz;
        if (n0 + tid < N) scales[(size_t)g * N + n0 + tid] = s;
    }
    if (tid < kQC) {                                        // zero points: CPW neighbouring lanes make a word
        uint32_t zw = (uint32_t)zz << (BITS * (tid & (CPW - 1)));
#pragma unroll
        for (int d = 1; d < CPW; d *= 2) zw |= __shfl_xor(zw, d, 64);
        if ((tid & (CPW - 1)) == 0 && n0 + tid < N) qzeros[(size_t)g * NW + (n0 + tid) / CPW] = zw;
    }
    __syncthreads();

    // ---- codes ----
    float sc[8], r[8], m[8];
    {
        const f32x4* const ps = reinterpret_cast<const f32x4*>(&col[0][8 * u]);
        const f32x4* const pr = reinterpret_cast<const f32x4*>(&col[1][8 * u]);
        const f32x4* const pm = reinterpret_cast<const f32x4*>(&col[2][8 * u]);
#pragma unroll
        for (int j = 0; j < 8; j++) { sc[j] = ps[j >> 2][j & 3]; r[j] = pr[j >> 2][j & 3]; m[j] = pm[j >> 2][j & 3]; }
    }
    uint32_t word[8][WPU];
    if (__builtin_expect(odd, 0)) {
#pragma unroll
        for (int i = 0; i < 8; i++) {
            v[i].apart();
#pragma unroll
            for (int k = 0; k < WPU; k++) word[i][k] = 0;
#pragma unroll
            for (int j = 0; j < 8; j++)
                word[i][j / CPW] |= code_divided<BITS>(v[i].at(j), sc[j], kMagic - m[j]) << (BITS * (j % CPW));
        }
    } else {
        uint32_t base[WPU];                                  // minus what the lower bounds of a word's codes add up to
#pragma unroll
        for (int k = 0; k < WPU; k++) base[k] = 0;
#pragma unroll
        for (int j = 0; j < 8; j++) base[j / CPW] -= bit_cast<uint32_t>(m[j]) << (BITS * (j % CPW));
#pragma unroll
        for (int i = 0; i < 8; i++) {
#pragma unroll
            for (int k = 0; k < WPU; k++) word[i][k] = base[k];
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const float x = v[i].at(j);
                const float q = x * r[j];
                const float t = __builtin_fmaf(__builtin_fmaf(-q, sc[j], x), r[j], q) + kMagic;
                const float c = __builtin_amdgcn_fmed3f(t, m[j], m[j] + (float)L);
                word[i][j / CPW] += bit_cast<uint32_t>(c) << (BITS * (j % CPW));
            }
        }
    }
    if (qweight && live) {
        uint32_t* dst = qweight + row0 * NW + (size_t)(n / CPW);
#pragma unroll
        for (int i = 0; i < 8; i++) {
            if constexpr (BITS == 4) dst[(size_t)i * NW] = word[i][0];
            else *reinterpret_cast<u32x2*>(dst + (size_t)i * NW) = u32x2{word[i][0], word[i][1]};
        }
    }
    if constexpr (BITS == 4) {
        if (native) {
            // unit = column half h of lane (c, b): loads 2 h and 2 h + 1 of the block, the padding of the last tile holds zeros
            const int T = (N + 255) >> 8, tile = n >> 8, c = (n >> 4) & 15, h = (n >> 3) & 1;
            const int ks = (int)(row0 >> 5), b = oct & 3;
            u32x4* const blk = native + ((size_t)ks * T + tile) * 256 + 16 * b + c;
            if (tile < T) {
#pragma unroll
                for (int p = 0; p < 2; p++) {
                    u32x4 o;
#pragma unroll
                    for (int q = 0; q < 4; q++)
                        o[q] = live ? __builtin_amdgcn_perm(word[2 * q + 1][0], word[2 * q][0], p ? 0x07060302u : 0x05040100u) : 0u;
                    blk[(2 * h + p) * 64] = o;
                }
            }
        }
    }
}

// ---- the native storage order of the 4-bit codes (what decode_small.hip's lanes consume) ----
// A block = one column tile of 256 and one k-step of 32 rows, 4096 bytes, blocks in (k-step, tile)
// order (the workgroups of a launch walk k together, each in its own tile: what they read at the same
// time lies together; with whole tiles one after the other the kernels measured 3 to 9 % slower).  Lane (c, b) of the decode kernel (lane number 16 b + c) owns columns 16 c .. 16 c + 15 of
// the tile and rows 8 b .. 8 b + 7 of the k-step: four 16-byte loads, load i = 2 h + p for column half
// h and byte pair p of the canonical word of that half; a load's 1024 bytes hold the 64 lanes' 16
// bytes in lane order; a lane's 16 bytes are four words, word q for rows 2 q, 2 q + 1 of its 8; byte
// 2 r + e of a word is byte 2 p + e of the canonical word (columns 8 h + 4 p + 2 e, + 1) of row 2 q + r.
//
// Canonical word wd (columns 8 wd ..) of row k, gathered from the native array.
__device__ __forceinline__ uint32_t native_word(const uint8_t* __restrict__ nat, int T, int k, int wd)
{
    const int tile = wd >> 5, c = (wd & 31) >> 1, h = wd & 1;
    const int ks = k >> 5, kr = k & 31, b = kr >> 3, q = (kr & 7) >> 1, r = kr & 1;
    const uint8_t* blk = nat + ((size_t)ks * T + tile) * 4096 + (size_t)(16 * b + c) * 16 + 4 * q + 2 * r;
    uint32_t out = 0;
#pragma unroll
    for (int y = 0; y < 4; y++) out |= (uint32_t)blk[(2 * h + (y >> 1)) * 1024 + (y & 1)] << (8 * y);
    return out;
}

// One thread per word of the native array: its four bytes come from two canonical words (rows 2 q,
// 2 q + 1); words of columns at or beyond N (the padding of the last tile) are zero.
__global__ __launch_bounds__(256) void repack_native_kernel(const uint32_t* __restrict__ qweight, uint32_t* __restrict__ nat,
                                                            int K, int N, size_t words)
{
    const size_t wi = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (wi >= words) return;
    const int T = (N + 255) >> 8, NW = N >> 3;
    const int q = (int)(wi & 3), lane = (int)((wi >> 2) & 63), i = (int)((wi >> 8) & 3);
    const size_t blk = wi >> 10;
    const int tile = (int)(blk % T), ks = (int)(blk / T);
    const int c = lane & 15, b = lane >> 4, h = i >> 1, p = i & 1;
    const int wd = tile * 32 + 2 * c + h, k = ks * 32 + 8 * b + 2 * q;
    uint32_t out = 0;
    if (wd < NW) {
        const uint32_t w0 = qweight[(size_t)k * NW + wd], w1 = qweight[(size_t)(k + 1) * NW + wd];
        out = ((w0 >> (16 * p)) & 0xFFFFu) | (((w1 >> (16 * p)) & 0xFFFFu) << 16);
    }
    nat[wi] = out;
}

// One thread per canonical word.
__global__ __launch_bounds__(256) void unpack_native_kernel(const uint8_t* __restrict__ nat, uint32_t* __restrict__ qweight, int K, int N)
{
    const int NW = N >> 3;
    const int wd = blockIdx.x * 256 + threadIdx.x, k = blockIdx.y;
    if (wd < NW) qweight[(size_t)k * NW + wd] = native_word(nat, (N + 255) >> 8, k, wd);
}

// ---- dequantizer export ----
// Bound: the bytes written.  A thread takes a piece of 8 columns (4 for fp32, so that neighbouring lanes write
// neighbouring 16 bytes either way; pieces of 32 bytes made half-written lines and 142 us below) of 8 consecutive rows:
// its scales and zero points are loaded once, the eight rows' codes are in flight together, and in the native order
// they are two 16-byte loads (one for fp32).
// NAT: qweight is the native array of 4-bit codes.
// Measured (4096 x 22016, cold): to fp16 58.3 -> 40.4 us from canonical 4-bit codes, 80.6 -> 40.4 from the native order,
// 57.4 -> 46.4 from 8-bit codes; to fp32 103.8 -> 80.2 us.
constexpr int kDU = 32;                                    // pieces side by side per workgroup
constexpr int kDO = 8;                                     // row octets per workgroup
template <typename OT, int BITS, bool NAT = false>
__global__ __launch_bounds__(kDU * kDO) void dequantize_kernel(const uint32_t* __restrict__ qweight,
                                                               const half_t* __restrict__ scales,
                                                               const uint32_t* __restrict__ qzeros,
                                                               OT* __restrict__ out, int K, int N)
{
    constexpr int CPT = 16 / (int)sizeof(OT);               // columns of a piece
    constexpr int BPP = CPT * BITS;                         // bits of a row's piece: 16, 32 or 64
    constexpr int WPP = BPP > 32 ? 2 : 1;
    constexpr uint32_t kMask = (1u << BITS) - 1u;
    const int NW = N * BITS / 32;
    const int piece = blockIdx.x * kDU + (threadIdx.x & (kDU - 1)), col = piece * CPT;
    const int k0 = (blockIdx.y * kDO + threadIdx.x / kDU) * 8;   // K is a multiple of 128: every octet of the grid exists
    if (col >= N) return;
    const int g = k0 / kGroup;
    const int wi = col * BITS / 32;                         // its word of a row
    const int sh = BPP == 16 ? 16 * (piece & 1) : 0;        // and where it starts there
    uint32_t qp[8][WPP];
    if constexpr (NAT) {
        // columns 8 h ..  of lane (c, b): loads 2 h (first four columns) and 2 h + 1; word q of a load holds rows 2 q, 2 q + 1
        const int T = (N + 255) >> 8, tile = col >> 8, c = (col >> 4) & 15, h = (col >> 3) & 1, b = (k0 >> 3) & 3;
        const u32x4* const blk = reinterpret_cast<const u32x4*>(qweight) + ((size_t)(k0 >> 5) * T + tile) * 256 + 16 * b + c;
        if constexpr (BPP == 16) {
            const u32x4 w = __builtin_nontemporal_load(blk + (2 * h + (piece & 1)) * 64);
#pragma unroll
            for (int q = 0; q < 4; q++) { qp[2 * q][0] = w[q] & 0xFFFFu; qp[2 * q + 1][0] = w[q] >> 16; }
        } else {
            const u32x4 w0 = __builtin_nontemporal_load(blk + (2 * h) * 64), w1 = __builtin_nontemporal_load(blk + (2 * h + 1) * 64);
#pragma unroll
            for (int q = 0; q < 4; q++) {
                qp[2 * q][0]     = __builtin_amdgcn_perm(w1[q], w0[q], 0x05040100u);
                qp[2 * q + 1][0] = __builtin_amdgcn_perm(w1[q], w0[q], 0x07060302u);
            }
        }
    } else {
        const uint32_t* src = qweight + (size_t)k0 * NW + wi;
#pragma unroll
        for (int i = 0; i < 8; i++) {
            if constexpr (WPP == 1) qp[i][0] = __builtin_nontemporal_load(src + (size_t)i * NW) >> sh;
            else {
                const u32x2 v = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(src + (size_t)i * NW));
                qp[i][0] = v[0];
                qp[i][1] = v[1];
            }
        }
    }
    float s[CPT];
    int   z[CPT];
    {
        const uint32_t* zp = qzeros + (size_t)g * NW + wi;
        const half_t*   sp = scales + (size_t)g * N + col;
        half_t s16[CPT];
        if constexpr (CPT == 8) {
            const half8_t v = *reinterpret_cast<const half8_t*>(sp);
#pragma unroll
            for (int j = 0; j < CPT; j++) s16[j] = v[j];
        } else {
            const half4_t v = *reinterpret_cast<const half4_t*>(sp);
#pragma unroll
            for (int j = 0; j < CPT; j++) s16[j] = v[j];
        }
#pragma unroll
        for (int j = 0; j < CPT; j++) {
            s[j] = (float)s16[j];
            z[j] = (int)((zp[BITS * j / 32] >> (sh + (BITS * j) % 32)) & kMask);
        }
    }
    OT* o = out + (size_t)k0 * N + col;
#pragma unroll
    for (int i = 0; i < 8; i++, o += N) {
        float d[CPT];
#pragma unroll
        for (int j = 0; j < CPT; j++)                       // exact: at most 9 x 11 significant bits
            d[j] = (float)((int)((qp[i][BITS * j / 32] >> ((BITS * j) % 32)) & kMask) - z[j]) * s[j];
        u32x4 v;
        if constexpr (sizeof(OT) == 4) v = bit_cast<u32x4>(f32x4{d[0], d[1], d[2], d[3]});
        else {
            constexpr bool BF = !__is_same(OT, half_t);
#pragma unroll
            for (int j = 0; j < 4; j++)                     // one rounding, to nearest even
                v[j] = (uint32_t)narrow16<BF>(d[2 * j]) | ((uint32_t)narrow16<BF>(d[2 * j + 1]) << 16);
        }
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(o));
    }
}

template <typename OT>
static dim3 dequantize_grid(int K, int N)
{
    const int pieces = N / (16 / (int)sizeof(OT));
    return dim3((pieces + kDU - 1) / kDU, K / (8 * kDO));
}

// Wide workgroups (32 units, 512 threads) read whole kilobytes of a row of fp32; below two of them per compute unit
// the narrow ones (16 units) spread the matrix over twice as many.  Narrow / wide, us to 4 bits: bfloat16 1024 x 1288 4.7 / 5.4 (48 wide tiles),
// 4096 x 22016 44.0 / 39.5 (2752); fp16 4.7 / 5.9, 42.8 / 41.0; fp32 6.7 / 8.7, 87.7 / 77.7.  The line is the one of wide matrices: of at most 4096 columns and 512 tiles
// and more, fp16 would be 1 to 8 % faster on narrow ones (8192 x 2048 11.4 / 12.0, 11008 x 4096 22.8 / 23.4), bfloat16 from 6 % slower to 1 % faster (4096 x 4096
// 11.5 / 10.8, 11008 x 4096 21.9 / 22.1) and fp32 up to 3 % faster (8192 x 2048 16.9 / 17.2).
template <int BITS, int QU>
static void quantize_units(const void* w, int dtype, uint32_t* qweight, half_t* sc, uint32_t* qzeros, void* native, int K, int N, hipStream_t st)
{
    const int cols = native ? (N + 255) & ~255 : N;         // the native order pads the last tile of 256 columns
    dim3 grid((cols + 8 * QU - 1) / (8 * QU), K / kGroup), block(16 * QU);
    u32x4* nat = (u32x4*)native;
    if (dtype == 1)      hipLaunchKernelGGL((quantize_kernel<half_t, BITS, QU>), grid, block, 0, st, (const half_t*)w, qweight, sc, qzeros, nat, K, N);
    else if (dtype == 2) hipLaunchKernelGGL((quantize_kernel<bf16_t, BITS, QU>), grid, block, 0, st, (const bf16_t*)w, qweight, sc, qzeros, nat, K, N);
    else                 hipLaunchKernelGGL((quantize_kernel<float, BITS, QU>), grid, block, 0, st, (const float*)w, qweight, sc, qzeros, nat, K, N);
}

// dtype: 0 = fp32, 1 = fp16, 2 = bf16 (the MORPH_DTYPE_* values); native: NULL, or the native array of 4-bit codes
template <int BITS>
static void quantize_bits(const void* w, int dtype, uint32_t* qweight, half_t* sc, uint32_t* qzeros, void* native, int K, int N, hipStream_t st)
{
    if ((long long)((N + 255) / 256) * (K / kGroup) < 512) quantize_units<BITS, 16>(w, dtype, qweight, sc, qzeros, native, K, N, st);
    else quantize_units<BITS, 32>(w, dtype, qweight, sc, qzeros, native, K, N, st);
}

hipError_t launch_quantize(int bits, const void* w, int w_dtype, uint32_t* qweight, void* scales,
                           uint32_t* qzeros, void* native, int K, int N, hipStream_t st)
{
    if (bits == 4) quantize_bits<4>(w, w_dtype, qweight, (half_t*)scales, qzeros, native, K, N, st);
    else           quantize_bits<8>(w, w_dtype, qweight, (half_t*)scales, qzeros, nullptr, K, N, st);
    return hipGetLastError();
}

template <typename OT, int BITS, bool NAT>
static void dequantize_to(const void* codes, const void* sc, const uint32_t* qzeros, void* out, int K, int N, hipStream_t st)
{
    hipLaunchKernelGGL((dequantize_kernel<OT, BITS, NAT>), dequantize_grid<OT>(K, N), dim3(kDU * kDO), 0, st,
                       (const uint32_t*)codes, (const half_t*)sc, qzeros, (OT*)out, K, N);
}

template <int BITS, bool NAT>
static void dequantize_bits(const void* codes, const void* sc, const uint32_t* qzeros, void* out, int dtype, int K, int N, hipStream_t st)
{
    if (dtype == 1)      dequantize_to<half_t, BITS, NAT>(codes, sc, qzeros, out, K, N, st);
    else if (dtype == 2) dequantize_to<bf16_t, BITS, NAT>(codes, sc, qzeros, out, K, N, st);
    else                 dequantize_to<float, BITS, NAT>(codes, sc, qzeros, out, K, N, st);
}

hipError_t launch_repack_native(const uint32_t* qweight, void* native, int K, int N, hipStream_t st)
{
    const size_t words = (size_t)((N + 255) / 256) * (K / 32) * 1024;
    hipLaunchKernelGGL(repack_native_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st, qweight, (uint32_t*)native, K, N, words);
    return hipGetLastError();
}

hipError_t launch_unpack_native(const void* native, uint32_t* qweight, int K, int N, hipStream_t st)
{
    hipLaunchKernelGGL(unpack_native_kernel, dim3(((N >> 3) + 255) / 256, K), dim3(256), 0, st, (const uint8_t*)native, qweight, K, N);
    return hipGetLastError();
}

hipError_t launch_dequantize_native(const void* native, const void* scales, const uint32_t* qzeros,
                                    void* out, int out_dtype, int K, int N, hipStream_t st)
{
    dequantize_bits<4, true>(native, scales, qzeros, out, out_dtype, K, N, st);
    return hipGetLastError();
}

hipError_t launch_dequantize(int bits, const uint32_t* qweight, const void* scales, const uint32_t* qzeros,
                             void* out, int out_dtype, int K, int N, hipStream_t st)
{
    if (bits == 4) dequantize_bits<4, false>(qweight, scales, qzeros, out, out_dtype, K, N, st);
    else           dequantize_bits<8, false>(qweight, scales, qzeros, out, out_dtype, K, N, st);
    return hipGetLastError();
}

}  // namespace morph
