// Offline quantizer / packer (ZeroQuant(4+2) Section 4 Eq. 3, Section 5.1) and the two
// plane-reading test utilities, for gfx950.
#include "fp6_common.hpp"
#include "fp6_internal.hpp"

namespace fp6 {

// ------------------------------------------------------------------ quantizer
// S = RNE_fp16(max |w| / 28) over one block of `block` consecutive elements of a row
// (Section 4, Eq. 3; block == K is the row-wise scheme, smaller blocks the fine-grained
// one of Section 3).  Scale (n, g) is stored at scales[g * N + n]: block-major, so that the
// scales of neighbouring output channels are neighbours in memory.
// |w| of finite fp16 orders like its 15 magnitude bits, so the maximum is taken on
// integers.  The quotient is one IEEE fp32 division followed by one fp32->fp16 rounding;
// a double rounding cannot occur because amax/28 is either exact in fp16 or at least
// 2^-14 (relative) away from every fp16 midpoint.
__device__ __forceinline__ _Float16 scale_of(uint32_t amax, float fmax)
{
    return (_Float16)((float)__builtin_bit_cast(_Float16, (uint16_t)amax) / fmax);
}

// the larger 15-bit magnitude of each half of two dwords of fp16 pairs (a holds magnitudes already)
__device__ __forceinline__ uint32_t max_magnitudes(uint32_t a, uint32_t w)
{
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a),
                                                                  __builtin_bit_cast(u16x2, w & 0x7FFF7FFFu)));
}

// What dividing by one scale needs: the scale and minus its reciprocal, with the 2^12 of the bias shift (Section 5.2)
// folded in, so that quotients come out 2^-12 times the FP6 value.  A zero scale gives zero quotients.
struct Divisor {
    float s, neg_r;
};
__device__ __forceinline__ Divisor divisor_of(_Float16 S)
{
    const float s = (float)S * 4096.0f;
    return Divisor{s, s == 0.0f ? -0.0f : -1.0f / s};
}

// w / (S * 2^12), saturated at the format's largest magnitude: q0 = w * r is corrected by its exact remainder, two
// fused operations instead of the eight of an IEEE division.  Where the quotient is a midpoint of the code grid (few
// bits) the corrected quotient is that midpoint; any other quotient is at least 2^-17 (relative) away from every
// midpoint, far more than the 2^-24 that q can be off - so rounding q decides exactly as rounding the real quotient
// would.  The signs are arranged so that -0 stays -0: the remainder of an exact quotient is +0 and -r < 0.
template <int FMT>
__device__ __forceinline__ float quotient(float w, Divisor d)
{
    constexpr float kMax = (FMT == kE3M1 ? 24.0f : 28.0f) / 4096.0f;
    const float q0 = w * -d.neg_r;
    const float rem = __builtin_fmaf(d.s, q0, -w);
    return __builtin_amdgcn_fmed3f(__builtin_fmaf(rem, d.neg_r, q0), -kMax, kMax);
}

// E3M1: the quotient rounded to one mantissa bit (to nearest even) while it is still fp32; the conversion below is then
// exact.  From 2^-14 up (0.25 before the shift) half a unit minus one, plus the last kept bit, is added below the kept
// bits (a carry runs into the exponent as it should); below, the values are multiples of 2^-15, the spacing of fp32
// numbers around 384.
__device__ __forceinline__ float round_e3m1(float q)
{
    const uint32_t b = __builtin_bit_cast(uint32_t, q);
    const uint32_t normal = (b + 0x1FFFFFu + ((b >> 22) & 1u)) & 0xFFC00000u;
    const float sub = __builtin_copysignf((fabsf(q) + 384.0f) - 384.0f, q);
    return fabsf(q) < 0x1p-14f ? sub : __builtin_bit_cast(float, normal);
}

__device__ __forceinline__ float low_half(uint32_t d) { return (float)__builtin_bit_cast(_Float16, (uint16_t)d); }
__device__ __forceinline__ float high_half(uint32_t d) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(d >> 16)); }

// Four weights to the bytes  s 0 0 e e e m m : the E5M2 number nearest to w / (S * 2^12) (to nearest even).  With the
// 2^12 taken out, E3M2's values are exactly E5M2's up to 28 * 2^-12, subnormals included (Eq. 5 read in eight bits), so
// the hardware conversion to E5M2 is the quantizer's rounding.  The bytes hold, in order, the weights a, b, c, d.
template <int FMT>
__device__ __forceinline__ uint32_t code_bytes(float a, float b, float c, float d, Divisor dv)
{
    float q[4] = {quotient<FMT>(a, dv), quotient<FMT>(b, dv), quotient<FMT>(c, dv), quotient<FMT>(d, dv)};
    if (FMT == kE3M1) {
#pragma unroll
        for (int e = 0; e < 4; e++) q[e] = round_e3m1(q[e]);
    }
    int u = __builtin_amdgcn_cvt_pk_bf8_f32(q[0], q[1], 0, false);
    return (uint32_t)__builtin_amdgcn_cvt_pk_bf8_f32(q[2], q[3], u, true);
}

// One lane slot of one tile (64 weights): v[f] = the eight consecutive weights of fragment f = 2t + q, i.e. of channel
// 16t + i at k block q; d[t] = the channel's divisor.  Writes the slot's 32 + 16 (FP5: 8) bytes of the two planes.
template <int FMT>
__device__ __forceinline__ void pack_slot(const u32x4 (&v)[8], const Divisor (&d)[4], u32x4* __restrict__ hi,
                                          u32x4* __restrict__ lo, size_t tile, int slot)
{
    uint32_t hiw[8], low[4] = {0, 0, 0, 0};
    if (FMT == kE3M2H) {
#pragma unroll
        for (int q = 0; q < 2; q++) {
            // the unit's codes as a string of 192 bits, 48 per fragment
            uint32_t T[6], head[4], tail[4];
#pragma unroll
            for (int t = 0; t < 4; t++) {
                const u32x4 w = v[2 * t + q];
                uint32_t x[2];
#pragma unroll
                for (int p = 0; p < 2; p++) {
                    const uint32_t u = code_bytes<FMT>(low_half(w[2 * p]), high_half(w[2 * p]), low_half(w[2 * p + 1]),
                                                       high_half(w[2 * p + 1]), d[t]);
                    const uint32_t c = ((u >> 2) & 0x20202020u) | (u & 0x1F1F1F1Fu);          // four codes, a byte each
                    const uint32_t y = (c & 0x003F003Fu) | ((c & 0x3F003F00u) >> 2);          // two pairs of 12 bits
                    x[p] = (y & 0xFFFu) | ((y >> 4) & 0xFFF000u);                             // 24 bits
                }
                head[t] = x[0] | (x[1] << 24);
                tail[t] = x[1] >> 8;
            }
            T[0] = head[0];
            T[1] = tail[0] | (head[1] << 16);
            T[2] = (head[1] >> 16) | (tail[1] << 16);
            T[3] = head[2];
            T[4] = tail[2] | (head[3] << 16);
            T[5] = (head[3] >> 16) | (tail[3] << 16);
            // split the string by kind of bit (the inverse of merge_unit)
            low[2 * q] = (T[0] & ~kSE0) | (T[1] & ~kSE1) | (T[2] & ~kSE2);
            low[2 * q + 1] = (T[3] & ~kSE0) | (T[4] & ~kSE1) | (T[5] & ~kSE2);
            hiw[4 * q + 0] = (T[0] & kSE0) | (T[4] & ~kSE0);
            hiw[4 * q + 1] = (T[1] & kSE1) | ((T[4] & 0x0C30C30Cu) << 2);
            hiw[4 * q + 2] = (T[2] & kSE2) | ((T[5] & 0x030C30C3u) << 2);
            const uint32_t r5 = T[5] & kFromA3;
            hiw[4 * q + 3] = (T[3] & kSE0) | (r5 << 2) | (r5 >> 30);
        }
    } else {
#pragma unroll
        for (int f = 0; f < 8; f++) {
            // bytes 0..3 of a plane dword carry elements 0, 2, 1, 3 of their group of four
            uint32_t u[2];
#pragma unroll
            for (int p = 0; p < 2; p++)
                u[p] = code_bytes<FMT>(low_half(v[f][2 * p]), low_half(v[f][2 * p + 1]), high_half(v[f][2 * p]),
                                       high_half(v[f][2 * p + 1]), d[f >> 1]);
            hiw[f] = (u[0] & 0x1C1C1C1Cu) | ((u[1] & 0x1C1C1C1Cu) << 3) | ((u[0] >> 7) & 0x01010101u) |
                     ((u[1] >> 6) & 0x02020202u);
            if (FMT == kE3M2)
                low[f >> 1] |= ((u[0] & 0x03030303u) | ((u[1] & 0x03030303u) << 2)) << (4 * (f & 1));
            else
                low[f >> 2] |= (((u[0] >> 1) & 0x01010101u) | (u[1] & 0x02020202u)) << (2 * (f & 3));
        }
    }
    u32x4* hp = hi + tile * kHiTileVec + slot;
    hp[0] = u32x4{hiw[0], hiw[1], hiw[2], hiw[3]};
    hp[64] = u32x4{hiw[4], hiw[5], hiw[6], hiw[7]};
    if (FMT != kE3M1) lo[tile * kLoTileVec + slot] = u32x4{low[0], low[1], low[2], low[3]};
    else reinterpret_cast<u32x2*>(lo)[tile * 64 + slot] = u32x2{low[0], low[1]};
}

// Bound by HBM: W is read and 0.75 byte per weight written.  A work item is 4 * I rows (channels 16t + I * part + 0..I-1
// of a 64-channel block, t = 0..3) of one scale block along K.  A lane holds a whole lane slot of a tile (8 x 16 bytes:
// four rows, both k blocks); a wavefront covers 16 / I tiles at a time, and a round of the workgroup W times that.  The
// first R rounds stay in registers between the maximum and the rounding, so that W is read from memory once; what lies
// beyond them is read a second time.  Fewer rows (I = 2: eight) let longer rows fit, at the price of shorter pieces of
// the planes (32 bytes) per store.  Workgroups stay and walk over the items: as soon as a round is packed its registers
// are refilled for the next item, so that the rounding of one item runs while the next one is being fetched (28672 x 8192
// with I = 4, W = 8, R = 4: 157 us without, 142 with).  The rounding takes about 9 vector operations a weight (an IEEE
// division and integer rounding took about 30, which alone cost 160 us on that shape).
template <int FMT, int I, int W, int R>
__global__ __launch_bounds__(W * 64) void quantize_kernel(const uint16_t* __restrict__ Wt, int N, int K, int block,
                                                          uint16_t* __restrict__ scales, u32x4* __restrict__ hi,
                                                          u32x4* __restrict__ lo)
{
    constexpr float kMax = FMT == kE3M1 ? 24.0f : 28.0f;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int Q = 16 / I;                 // parts of a unit = tiles side by side in a wavefront
    constexpr int kRound = W * Q;             // tiles per round
    const int g = (lane / I) & 3, kq = lane / (4 * I);
    const int tiles = block / kTile, groups = K / block, units = (N / kTile) * groups;
    const int tk0 = wave * Q + kq;
    // the four quads of a unit get ids 8 apart: one die, whose L2 merges their 64-byte pieces of each line
    const int i = (int)((blockIdx.x >> 3) % Q) * I + lane % I;
    const int stride = (int)(gridDim.x / (8 * Q)) * 8;
    int unit = (int)(blockIdx.x / (8 * Q)) * 8 + (int)(blockIdx.x & 7);

    auto row0 = [&](int u) {      // this lane's first weight of the unit, in channel i of the block
        return Wt + ((size_t)(u / groups) * kTile + i) * K + (size_t)(u % groups) * block + g * 8;
    };
    auto load = [&](u32x4 (&v)[8], const uint16_t* base, int tk) {
        const uint16_t* p = base + (size_t)min(tk, tiles - 1) * kTile;
#pragma unroll
        for (int f = 0; f < 8; f++) v[f] = *reinterpret_cast<const u32x4*>(p + (size_t)(f >> 1) * 16 * K + (f & 1) * 32);
    };
    __shared__ uint32_t smax[2][W][4][I];
    u32x4 keep[R][8];
    if (unit < units) {
#pragma unroll
        for (int r = 0; r < R; r++) load(keep[r], row0(unit), tk0 + r * kRound);
    }
    for (int turn = 0; unit < units; unit += stride, turn ^= 1) {
        const uint16_t* base = row0(unit);
        const int nb = unit / groups, gb = unit % groups;
        uint32_t mx[4] = {0, 0, 0, 0};
        auto fold = [&](const u32x4 (&v)[8]) {
#pragma unroll
            for (int f = 0; f < 8; f++)
#pragma unroll
                for (int c = 0; c < 4; c++) mx[f >> 1] = max_magnitudes(mx[f >> 1], v[f][c]);
        };
        for (int tk = tk0 + R * kRound; tk - kq < tiles; tk += kRound) {
            u32x4 v[8];
            load(v, base, tk);
            fold(v);
        }
#pragma unroll
        for (int r = 0; r < R; r++) fold(keep[r]);
#pragma unroll
        for (int t = 0; t < 4; t++) {
            uint32_t m = max(mx[t] & 0xFFFFu, mx[t] >> 16);
#pragma unroll
            for (int off = I; off < 64; off <<= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
            if (lane < I) smax[turn][wave][t][lane] = m;
        }
        __syncthreads();          // (two buffers: the next item's maxima go to the other one)
        Divisor d[4];
#pragma unroll
        for (int t = 0; t < 4; t++) {
            uint32_t m = 0;
#pragma unroll
            for (int w = 0; w < W; w++) m = max(m, smax[turn][w][t][lane % I]);
            const _Float16 S = scale_of(m, kMax);
            if (threadIdx.x < I) scales[(size_t)gb * N + nb * kTile + t * 16 + i] = __builtin_bit_cast(uint16_t, S);
            d[t] = divisor_of(S);
        }
        const size_t tile0 = (size_t)nb * (K / kTile) + (size_t)gb * tiles;
        const int slot = 16 * g + i;
        for (int tk = tk0 + R * kRound; tk - kq < tiles; tk += kRound) {
            u32x4 v[8];
            load(v, base, tk);
            if (tk < tiles) pack_slot<FMT>(v, d, hi, lo, tile0 + tk, slot);
        }
        const bool more = unit + stride < units;
        const uint16_t* next = more ? row0(unit + stride) : base;
#pragma unroll
        for (int r = 0; r < R; r++) {
            if (tk0 + r * kRound < tiles) pack_slot<FMT>(keep[r], d, hi, lo, tile0 + tk0 + r * kRound, slot);
            if (more) load(keep[r], next, tk0 + r * kRound);
        }
    }
}

// Scale blocks of one, two or four tiles: a wavefront holds 16 rows of four tiles and finds the maxima with shuffles.
template <int FMT>
__global__ __launch_bounds__(256) void quantize_small_block_kernel(const uint16_t* __restrict__ Wt, int N, int K,
                                                                   int block, uint16_t* __restrict__ scales,
                                                                   u32x4* __restrict__ hi, u32x4* __restrict__ lo)
{
    constexpr float kMax = FMT == kE3M1 ? 24.0f : 28.0f;
    const int ktiles = K / kTile, chunks = (ktiles + 15) / 16;      // a workgroup: 16 rows x 16 tiles
    const unsigned rest = blockIdx.x >> 3;
    const int quad = rest & 3;
    const int unit = (int)(rest >> 2) * 8 + (int)(blockIdx.x & 7);
    if (unit >= (N / kTile) * chunks) return;
    const int nb = unit / chunks;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = quad * 4 + (lane & 3), g = (lane >> 2) & 3, kq = lane >> 4;
    const int tk = (unit % chunks) * 16 + wave * 4 + kq;
    const bool valid = tk < ktiles;
    const uint16_t* p = Wt + ((size_t)nb * kTile + i) * K + g * 8 + (valid ? tk : ktiles - 1) * kTile;
    u32x4 v[8];
#pragma unroll
    for (int f = 0; f < 8; f++) v[f] = *reinterpret_cast<const u32x4*>(p + (size_t)(f >> 1) * 16 * K + (f & 1) * 32);
    Divisor d[4];
#pragma unroll
    for (int t = 0; t < 4; t++) {
        uint32_t mx = 0;
#pragma unroll
        for (int c = 0; c < 8; c++) mx = max_magnitudes(mx, v[2 * t + (c >> 2)][c & 3]);
        uint32_t m = max(mx & 0xFFFFu, mx >> 16);
        m = max(m, (uint32_t)__shfl_xor((int)m, 4, 64));
        m = max(m, (uint32_t)__shfl_xor((int)m, 8, 64));
        // (blocks divide K, so a block never mixes valid tiles with the lanes past the end)
        if (block >= 2 * kTile) m = max(m, (uint32_t)__shfl_xor((int)m, 16, 64));
        if (block >= 4 * kTile) m = max(m, (uint32_t)__shfl_xor((int)m, 32, 64));
        const _Float16 S = scale_of(m, kMax);
        if (valid && g == 0 && tk % (block / kTile) == 0)
            scales[(size_t)(tk * kTile / block) * N + nb * kTile + t * 16 + i] = __builtin_bit_cast(uint16_t, S);
        d[t] = divisor_of(S);
    }
    if (valid) pack_slot<FMT>(v, d, hi, lo, (size_t)nb * ktiles + tk, 16 * g + i);
}

// Few, long scale blocks: quantize_kernel would give eight rows of them to one compute unit and leave most of the chip idle.
// There the maxima are taken by a launch of their own, one workgroup per scale, and a second launch rounds one tile per
// wavefront and reads W again (a W this small comes from the last-level cache).  Bound by the two launches and the length
// of a row in one workgroup: 64 x 28672 takes 7.7 us (23.8 in quantize_kernel), 512 x 28672 14.2 (24.3), 64 x 262144 23 (201).
template <int FMT>
__global__ __launch_bounds__(256) void block_scale_kernel(const uint16_t* __restrict__ Wt, int N, int K, int block,
                                                          uint16_t* __restrict__ scales)
{
    constexpr float kMax = FMT == kE3M1 ? 24.0f : 28.0f;
    const unsigned groups = (unsigned)(K / block);
    const unsigned n = blockIdx.x / groups, gb = blockIdx.x % groups;
    const u32x4* row = reinterpret_cast<const u32x4*>(Wt + (size_t)n * K + (size_t)gb * block);
    uint32_t mx = 0;
#pragma unroll 4
    for (int v = threadIdx.x; v < block / 8; v += 256) {
        const u32x4 d = row[v];
#pragma unroll
        for (int c = 0; c < 4; c++) mx = max_magnitudes(mx, d[c]);
    }
    uint32_t m = max(mx & 0xFFFFu, mx >> 16);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
    __shared__ uint32_t smax[4];
    if ((threadIdx.x & 63) == 0) smax[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0)
        scales[(size_t)gb * N + n] = __builtin_bit_cast(uint16_t, scale_of(max(max(smax[0], smax[1]), max(smax[2], smax[3])), kMax));
}

template <int FMT>
__global__ __launch_bounds__(256) void pack_kernel(const uint16_t* __restrict__ Wt, int N, int K, int block,
                                                   const uint16_t* __restrict__ scales, u32x4* __restrict__ hi,
                                                   u32x4* __restrict__ lo)
{
    const unsigned ktiles = (unsigned)(K / kTile);
    const unsigned tile = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (tile >= (unsigned)(N / kTile) * ktiles) return;
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int nb = (int)(tile / ktiles), tk = (int)(tile % ktiles);
    const uint16_t* p = Wt + ((size_t)nb * kTile + i) * K + (size_t)tk * kTile + g * 8;
    u32x4 v[8];
#pragma unroll
    for (int f = 0; f < 8; f++) v[f] = *reinterpret_cast<const u32x4*>(p + (size_t)(f >> 1) * 16 * K + (f & 1) * 32);
    Divisor d[4];
#pragma unroll
    for (int t = 0; t < 4; t++)
        d[t] = divisor_of(__builtin_bit_cast(_Float16, scales[(size_t)(tk / (block / kTile)) * N + nb * kTile + t * 16 + i]));
    pack_slot<FMT>(v, d, hi, lo, tile, lane);
}

// ------------------------------------------------------------------ plane readers
// code of element e (0..7) of a fragment, from its two dwords (L already shifted by 4*(f&1))
// MB = 2: L = the fragment's dword of the 2-bit plane shifted right by 4*(f&1); code s eee mm.
// MB = 1: L = its dword of the 1-bit plane shifted right by 2*(f&3); code s eee m.
template <int MB = 2>
__device__ __forceinline__ uint32_t fragment_code(uint32_t H, uint32_t L, int e)
{
    const int grp = e >> 2, j = e & 3;
    const int b = 2 * (j & 1) + (j >> 1);
    const uint32_t hb = (H >> (8 * b)) & 0xFF, lb = (L >> (8 * b)) & 0xFF;
    const uint32_t s = (hb >> grp) & 1, ex = (hb >> (2 + 3 * grp)) & 7, m = (lb >> (MB * grp)) & ((1u << MB) - 1u);
    return s << (3 + MB) | ex << MB | m;
}

// the fragment's plane dwords as fragment_code wants them
template <int FMT>
__device__ __forceinline__ uint32_t fragment_lo(const TileRaw& r, int f)
{
    return FMT == kE3M2 ? tile_lo_dword(r, f) >> (4 * (f & 1)) : r.lo[f >> 2] >> (2 * (f & 3));
}

// code of element e of fragment f of a tile, any layout (f, e compile-time constants after unrolling)
template <int FMT>
__device__ __forceinline__ uint32_t tile_code(const TileRaw& r, int f, int e)
{
    if (FMT == kE3M2H) {
        const int q = f & 1, bit = 6 * (8 * (f >> 1) + e);
        const u32x6 T = merge_unit(q ? r.hi1 : r.hi0, r.lo[2 * q], r.lo[2 * q + 1]);
        uint32_t c = T[bit >> 5] >> (bit & 31);
        if ((bit & 31) > 26) c |= T[(bit >> 5) + 1] << (32 - (bit & 31));
        return c & 63u;
    }
    return fragment_code<FMT == kE3M1 ? 1 : 2>(tile_hi_dword(r, f), fragment_lo<FMT>(r, f), e);
}

template <int FMT>
__global__ __launch_bounds__(256) void unpack_codes_kernel(const u32x4* __restrict__ hi, const u32x4* __restrict__ lo,
                                                            int64_t N, int64_t K, uint8_t* __restrict__ codes)
{
    const int64_t slot = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t tile = slot >> 6;
    const int lane = (int)(slot & 63);
    const int64_t ktiles = K / kTile;
    if (tile >= (N / kTile) * ktiles) return;
    const int64_t nb = tile / ktiles, kb = tile % ktiles;
    const int i = lane & 15, g = lane >> 4;
    TileRaw r = load_tile<FMT>(hi, lo, (size_t)tile, lane);
#pragma unroll
    for (int f = 0; f < 8; f++) {
        const int64_t n = nb * kTile + (f >> 1) * 16 + i;
        const int64_t k = kb * kTile + (f & 1) * 32 + g * 8;
        uint32_t c0 = 0, c1 = 0;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            c0 |= tile_code<FMT>(r, f, e) << (8 * e);
            c1 |= tile_code<FMT>(r, f, 4 + e) << (8 * e);
        }
        *reinterpret_cast<uint2*>(codes + n * K + k) = make_uint2(c0, c1);
    }
}

// W_hat = RNE_fp16(S * value(code)): the fp32 product of an 11-bit and a 3-bit
// significand is exact, so the only rounding is the conversion to fp16.
// A wavefront takes a tile.  Its fragments hold 64-byte pieces of a row; the two of a row are put together in the wavefront's own LDS
// (16-byte chunk c of row r at chunk position c ^ (r & 7): no bank conflicts), so that eight lanes write a line of W_hat.  Bound by the copy: 13824 x 5120 43.8 ->
// 36.7 us (5.3 TB/s, read and written), 28672 x 8192 145 -> 121; the lines, and the tile's index divided once and in 32
// bits, where each of eight fragments had divided its column by the block in 64.
template <int FMT>
__global__ __launch_bounds__(256) void dequantize_kernel(const u32x4* __restrict__ hi, const u32x4* __restrict__ lo,
                                                          const uint16_t* __restrict__ scales, int64_t N, int64_t K,
                                                          int64_t block, uint16_t* __restrict__ W_hat)
{
    __shared__ __align__(16) unsigned char lines[4][2048];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), tile = blockIdx.x * 4 + wave;     // (at most 2^28 tiles)
    const int lane = threadIdx.x & 63;
    const uint32_t ktiles = (uint32_t)(K / kTile);
    if (tile >= (uint32_t)(N / kTile) * ktiles) return;
    const uint32_t nb = tile / ktiles, kb = tile % ktiles;
    const int i = lane & 15, g = lane >> 4;
    constexpr int MB = FMT == kE3M1 ? 1 : 2;
    TileRaw r = load_tile<FMT>(hi, lo, (size_t)tile, lane);
    // (a block of scales is whole tiles)
    const uint16_t* srow = scales + (size_t)(kb * (uint32_t)kTile / (uint32_t)block) * N + (size_t)nb * kTile + i;
    uint16_t* out_row = W_hat + ((size_t)nb * kTile + (lane >> 3)) * K + (size_t)kb * kTile + (lane & 7) * 8;
    unsigned char* own = lines[wave];
#pragma unroll
    for (int t = 0; t < 4; t++) {
        const float S = (float)__builtin_bit_cast(_Float16, srow[t * 16]);
        uint4 v[2];
#pragma unroll
        for (int q = 0; q < 2; q++) {
            uint32_t out[4];
#pragma unroll
            for (int e = 0; e < 8; e++) {
                const uint32_t c = tile_code<FMT>(r, 2 * t + q, e);
                const uint32_t ex = (c >> MB) & 7, m = (c & ((1u << MB) - 1u)) << (2 - MB);   // mantissa as quarters
                // value = m/16 (subnormal) or (4+m) * 2^(ex-5)
                float mag = ex ? (float)((4 + m) << (ex - 1)) * 0.0625f : (float)m * 0.0625f;
                _Float16 hval = (_Float16)(S * mag);
                uint32_t hb = __builtin_bit_cast(uint16_t, hval) | ((c >> (3 + MB)) << 15);
                if (e & 1) out[e >> 1] |= hb << 16; else out[e >> 1] = hb;
            }
            v[q] = make_uint4(out[0], out[1], out[2], out[3]);
        }
        // (DS instructions of a wavefront are carried out in order)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < 2; q++) *reinterpret_cast<uint4*>(own + i * 128 + ((4 * q + g) ^ (i & 7)) * 16) = v[q];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int p = 0; p < 2; p++)
            *reinterpret_cast<uint4*>(out_row + (size_t)(t * 16 + p * 8) * K) =
                *reinterpret_cast<const uint4*>(own + p * 1024 + (lane >> 3) * 128 + ((lane & 7) ^ (lane >> 3)) * 16);
    }
}

// ------------------------------------------------------------------ launchers
static inline unsigned slot_blocks(int64_t N, int64_t K) { return (unsigned)(((N / kTile) * (K / kTile) * 64 + 255) / 256); }

template <int FMT, int I, int W, int R>
static void launch_quantize_t(const uint16_t* Wt, int64_t N, int64_t K, int64_t block, void* hi, void* lo, uint16_t* scales,
                              int per_unit, hipStream_t stream)
{
    const int64_t units = (N / kTile) * (K / block), need = (units + 7) / 8 * (8 * 16 / I), most = 256 * per_unit;
    hipLaunchKernelGGL((quantize_kernel<FMT, I, W, R>), dim3((unsigned)(need < most ? need : most)), dim3(W * 64), 0, stream, Wt,
                       (int)N, (int)K, (int)block, scales, (u32x4*)hi, (u32x4*)lo);
}

// Up to 16 units (64 channels x one scale block; quantize_kernel cuts them into 128 work items at most, one to a compute
// unit) two launches are ahead from 7168 columns on, in every format.  Measured, us (one launch / two): 1024 x 5632 8.4 / 8.8,
// 1024 x 8192 10.1 / 10.1, 1024 x 11008 13.8 / 11.9, 1024 x 65536 59 / 49, 1536 x 11008 15.7 / 16.2, 2048 x 16384 23.1 / 26.1;
// five bits: 1024 x 7168 12.6 / 11.1, 1536 x 8192 14.5 / 14.5, 2048 x 11008 21.9 / 22.2.
static bool few_long_blocks(int64_t units, int64_t block) { return units <= 16 && block > 7168; }

template <int FMT>
static hipError_t launch_quantize_format(const uint16_t* Wt, int64_t N, int64_t K, int64_t block, void* hi, void* lo,
                                         uint16_t* scales, hipStream_t stream)
{
    // Rows per workgroup, wavefronts and rounds kept in registers, by the length of a scale block (= K for row scales).
    // Where a row fits the registers W is read once.  Measured, us (two-kernel version before / now; 2.75 bytes a weight
    // at the 5.1 TB/s of a plain copy): 1024 x 1024 10.8 / 4.7; 8192 x 2048 26 / 12.4 (9.0); 4096 x 4096 26 / 13.1 (9.0);
    // 13824 x 5120 84 / 48 (38); 28672 x 8192 263 / 147 (126); 5120 x 13824 85 / 52 (38); 8192 x 28672 270 / 186 (126).
    // The lines between the instances lie where their measured times cross: two rounds of (8 rows, 8 wavefronts) need
    // half-empty registers below about 5600 (13824 x 5120: one round and a short second read 48, two rounds 54), and four
    // rounds leave one workgroup per unit (28672 x 8192: 163 against 147; 4096 x 11008: 32 against 34).
    if (block <= 4 * kTile && (block & (block - 1)) == 0) {
        const int64_t units = (N / kTile) * ((K / kTile + 15) / 16);
        hipLaunchKernelGGL((quantize_small_block_kernel<FMT>), dim3((unsigned)((units + 7) / 8 * 32)), dim3(256), 0, stream,
                           Wt, (int)N, (int)K, (int)block, scales, (u32x4*)hi, (u32x4*)lo);
    } else if (few_long_blocks((N / kTile) * (K / block), block)) {
        hipLaunchKernelGGL((block_scale_kernel<FMT>), dim3((unsigned)(N * (K / block))), dim3(256), 0, stream, Wt, (int)N, (int)K,
                           (int)block, scales);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((pack_kernel<FMT>), dim3((unsigned)(((N / kTile) * (K / kTile) + 3) / 4)), dim3(256), 0, stream, Wt,
                           (int)N, (int)K, (int)block, (const uint16_t*)scales, (u32x4*)hi, (u32x4*)lo);
    } else if (block <= 1024) {
        launch_quantize_t<FMT, 4, 4, 1>(Wt, N, K, block, hi, lo, scales, 4, stream);
    } else if (block <= 2048) {
        launch_quantize_t<FMT, 2, 4, 1>(Wt, N, K, block, hi, lo, scales, 4, stream);
    } else if (block <= 5632) {
        launch_quantize_t<FMT, 2, 8, 1>(Wt, N, K, block, hi, lo, scales, 2, stream);
    } else if (block <= 9216) {
        launch_quantize_t<FMT, 2, 8, 2>(Wt, N, K, block, hi, lo, scales, 2, stream);
    } else {
        launch_quantize_t<FMT, 2, 8, 4>(Wt, N, K, block, hi, lo, scales, 1, stream);
    }
    return hipGetLastError();
}

hipError_t launch_quantize_pack(int format, const uint16_t* W, int64_t N, int64_t K, int64_t block, void* hi, void* lo,
                                uint16_t* scales, hipStream_t stream)
{
    if (format == kE3M2) return launch_quantize_format<kE3M2>(W, N, K, block, hi, lo, scales, stream);
    if (format == kE3M2H) return launch_quantize_format<kE3M2H>(W, N, K, block, hi, lo, scales, stream);
    return launch_quantize_format<kE3M1>(W, N, K, block, hi, lo, scales, stream);
}

hipError_t launch_unpack_codes(int format, const void* hi, const void* lo, int64_t N, int64_t K, uint8_t* codes,
                               hipStream_t stream)
{
    if (format == kE3M2)
        hipLaunchKernelGGL(unpack_codes_kernel<kE3M2>, dim3(slot_blocks(N, K)), dim3(256), 0, stream, (const u32x4*)hi,
                           (const u32x4*)lo, N, K, codes);
    else if (format == kE3M2H)
        hipLaunchKernelGGL(unpack_codes_kernel<kE3M2H>, dim3(slot_blocks(N, K)), dim3(256), 0, stream, (const u32x4*)hi,
                           (const u32x4*)lo, N, K, codes);
    else
        hipLaunchKernelGGL(unpack_codes_kernel<kE3M1>, dim3(slot_blocks(N, K)), dim3(256), 0, stream, (const u32x4*)hi,
                           (const u32x4*)lo, N, K, codes);
    return hipGetLastError();
}

hipError_t launch_dequantize(int format, const void* hi, const void* lo, const uint16_t* scales, int64_t N, int64_t K,
                             int64_t block, uint16_t* W_hat, hipStream_t stream)
{
    if (format == kE3M2)
        hipLaunchKernelGGL(dequantize_kernel<kE3M2>, dim3(slot_blocks(N, K)), dim3(256), 0, stream, (const u32x4*)hi,
                           (const u32x4*)lo, scales, N, K, block, W_hat);
    else if (format == kE3M2H)
        hipLaunchKernelGGL(dequantize_kernel<kE3M2H>, dim3(slot_blocks(N, K)), dim3(256), 0, stream, (const u32x4*)hi,
                           (const u32x4*)lo, scales, N, K, block, W_hat);
    else
        hipLaunchKernelGGL(dequantize_kernel<kE3M1>, dim3(slot_blocks(N, K)), dim3(256), 0, stream, (const u32x4*)hi,
                           (const u32x4*)lo, scales, N, K, block, W_hat);
    return hipGetLastError();
}

}  // namespace fp6
