// Tiled kernel (any M) of the W6A16 linear layer for gfx950: the kernel template and its launcher.
// Included by the translation units that instantiate it (fp6_gemm.hip: the FP6 bias-shift kernels;
// fp6_gemm_variants.hip: ablations, fine-grained scales, FP5; fp6_gemm_heights*.hip: heights between the powers of two).
//
// A workgroup computes a BM x (64 * GBN) block of Y, BM = 32 to 128 in steps of 16, GBN = 8 or 4.  Its wavefronts stand side by
// side along N, one per 64 output channels (two per SIMD at GBN = 8).  Every packed
// weight is fetched and padded to fp16 (bias shift, Section 5.2) by exactly one
// wavefront and goes straight into MFMA operand registers - the dequantized weight never
// exists in memory.  Only the activations are shared.
//
// All global traffic of the main loop is asynchronous DMA into LDS (global_load_lds,
// 16 bytes per lane, no register staging), into a ring of D stages per workgroup:
//   - the BM x 64 slice of X for a k tile (read by every wavefront as MFMA operands).
//     Rows are not padded; the 16-byte chunk c of row r is stored at chunk position
//     c ^ (r & 7), which keeps the DMA writes and the 128-bit operand reads free of bank
//     conflicts;
//   - each wavefront's own 3 KB of packed planes per block of output channels
//     (lane-linear, exactly the order the planes have in memory).
// The DMA is issued from inline assembly and waited for with explicit s_waitcnt vmcnt:
// every step but the last ones issues the same number of loads per wavefront, so "at most (D-2)
// groups still in flight" is a constant, and the compiler (which cannot see these loads) has
// no reason to drain the queue.  One barrier per k tile publishes the next step's activations and
// frees this step's, which are in registers by then; planes are a wavefront's own and need none (see step()).
//
// LDS traffic per k tile: every wavefront reads the whole X slice (wavefronts x BM x 128 B) plus its
// planes - at BM = 128 about 152 KB per 2048 MFMA cycles of a SIMD, some 60 % of the 128 B/clk port.
// What bounds it (cycle counter and wall clock read in the kernel, random data): with every compute unit busy the clock.  A
// step at 128 x 512 takes 2430 cycles of the 2048 its MFMAs need, at 1.84 GHz: 170 us for the 128 steps of 2048 x 8192 x 8192, 162 to
// 175 by unit, in a call of 186 (1.48 PFLOP/s; 198 on a slower machine); the rest is 2.2 us of prologue, 3.8 of epilogue and 5 between
// launches.  Without the LDS reads of X a step takes 40 cycles less, without the DMA or without the unpack 220, without all three 380 - and
// the clock stays at 1.8 to 2.0, where an MFMA-only loop on random operands settles too (1.98 PFLOP/s, 2.44 on zeros).  What costs energy
// costs time there: 5, 11 and 12 %.  With 172 units busy (512 x 22016 x 8192) the clock is 2.3 GHz, 2407 cycles a step and 135 us of 153.
// The vector operations of the unpack hide behind the MFMAs of a SIMD's two wavefronts as long as there are no more than two of them to
// each, evenly spread: in bursts they cost a quarter (a loop of nothing else: 2640 cycles against 2140).
// Four-wavefront workgroups with a compute unit to themselves are bound by the instructions one wavefront can issue, one
// in five cycles or so: 1190 cycles a step at 64 rows (210 instructions, 512 cycles of MFMAs), 1325 at 112 rows in bf16 (896).
// Where K is split, the meeting of the slices costs another 5-12 % at M = 512.
//
// The row scale is applied once, after the accumulation (Section 5.2).  K may be split
// over workgroups; the slices meet in an fp32 workspace and are added by the workgroup that arrives last, as in
// the decode kernel, or by a second launch.
#pragma once

#include "fp6_common.hpp"
#include "fp6_internal.hpp"
#include "fp6_reduce.hpp"

#include <type_traits>

namespace fp6 {

constexpr int kWaveTileBytes = kHiTileBytes + kLoTileBytes;   // 3072: the planes of one 64x64 tile

// 16 bytes per lane from (base + lane_offset) to LDS address lds + 16 * lane (lds is wave-uniform).
// M0 carries the LDS address; nothing else in these kernels uses M0 (gfx9 DS instructions do not),
// and the compiler does not accept it in a clobber list.
__device__ __forceinline__ void dma16(const void* base, uint32_t lane_offset, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(lane_offset), "s"(base), "s"(lds)
                 : "memory");
}

// 4 bytes per lane from (base + lane_offset) to LDS address lds + 4 * lane.
__device__ __forceinline__ void dma4(const void* base, uint32_t lane_offset, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
                 :
                 : "v"(lane_offset), "s"(base), "s"(lds)
                 : "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// FGQ: one scale per `64 << gshift` elements along K (Section 3, fine-grained quantization).
// The product sums of the k tiles of one such block are formed in a second accumulator; at
// the end of the block they are multiplied by the block's scales and added to the running
// sum: the scale is applied to each block's finished product sum, and only then do the blocks
// accumulate (the fine-grained rule of Section 5.2).  The scales of
// a wavefront's 64 channels (128 bytes per block) ride along with every stage of the DMA ring.
// GBN = 64-wide blocks of output channels per workgroup: 8 (512 channels), or 4 for launches that would
// otherwise have too few workgroups.
// KW = K-ways inside the workgroup.  KW = 2 doubles the wavefronts: the second set (kh = 1) works on the same
// BM x (64 * GBN) block of Y one k tile further along, so a step covers two k tiles, and the two sets' sums are
// added in LDS after the main loop.  It is what two workgroups of a two-way K-split would do, with the meeting moved
// from the workspace into LDS: where K has to be split to fill the chip, half of the partial sums never leave the
// compute unit.
template <int BM, int D, int DQ, bool FGQ, int FMT, int GBN, int KW>
__global__ __launch_bounds__(GBN * KW * 64, GBN == 4 && KW == 1 ? 2 : 1) void gemm_kernel(
    const uint16_t* __restrict__ X, int M, const u32x4* __restrict__ hi, const u32x4* __restrict__ lo,
    const uint16_t* __restrict__ scales, int N, int K, uint16_t* __restrict__ Y,
    float4v* __restrict__ partials, uint32_t* __restrict__ counters, int split_k, int gshift, int second_launch)
{
    static_assert(!FGQ || BM <= 64, "fine-grained scales: two accumulators must fit the register file");
    static_assert(KW == 1 || KW == 2 || KW == 4, "K-ways inside the workgroup");
    constexpr int WAVES = GBN * KW;
    constexpr int OUT_THREADS = GBN * 64;               // threads that hold the block of Y after the main loop
    constexpr int MT = BM / 16;                         // 16-row blocks of X per workgroup
    constexpr int NT = 4;                               // 16-channel blocks per wavefront
    constexpr int XG = KW * BM / 8;                     // 8-row groups (1 KB of DMA each) per stage: BM / 8 per k tile
    constexpr int XL = (XG + WAVES - 1) / WAVES;        // X groups moved per wavefront and step
    constexpr int PL = 3 + (FGQ ? 1 : 0);               // DMA instructions for a wavefront's planes (and scales) and step
    constexpr int kLoads = XL + PL;
    constexpr int kXBytes = KW * BM * kTile * 2;
    constexpr int kPlaneBytes = GBN * KW * kWaveTileBytes + (FGQ ? WAVES * 256 : 0);   // per stage of the plane ring
    constexpr int kScaleOff = GBN * KW * kWaveTileBytes;          // FGQ: 256 bytes per wavefront, inside the plane stage
    constexpr int kPlaneBase = D * kXBytes;                       // the plane ring follows the activation ring
    constexpr int kRingBytes = D * (kXBytes + kPlaneBytes);
    constexpr int kTileRegs = MT * NT * OUT_THREADS;    // float4 per output tile
    constexpr int kSumBytes = (KW - 1) * kTileRegs * 16;          // LDS for adding the K-ways
    constexpr int kSmemBytes = kRingBytes > kSumBytes ? kRingBytes : kSumBytes;
    // activations are read kAhead groups of MFMAs ahead, into a ring of kXRegs operands (see step() below)
    constexpr bool kWhole = MT <= 2;                    // all of a step's operands are read a step ahead
    constexpr int kXRegs = MT % 2 ? (MT == 3 ? 6 : MT) : 4, kAhead = kWhole ? 4 : (FGQ ? 2 : 3);
    // the groups in which the next step's planes and activations are read for the first time
    constexpr int kPlanesAt = MT - 1, kXAt = 2 * MT - kAhead;
    constexpr int kPlanesEvery = (kXAt - kPlanesAt) / PL > 0 ? (kXAt - kPlanesAt) / PL : 1;
    constexpr int kValu = layout2(FMT) ? 3 : ((DQ == kIntRebias ? 8 : 2) * 8 + MT - 1) / MT;      // vector operations behind an MFMA
    static_assert((2 * MT) % kXRegs == 0 && kAhead < kXRegs + (kWhole ? 1 : 0), "a step starts at entry 0 of the operand ring");
    __shared__ __align__(16) unsigned char smem[kSmemBytes];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kh = KW > 1 ? wave / GBN : 0;             // which of the K-ways this wavefront works on
    const int nw = KW > 1 ? wave % GBN : wave;          // its position along N
    const int ktiles = K / kTile, nblocks = N / kTile;
    const int mblk = (M + BM - 1) / BM;
    const int nblk = (nblocks + GBN - 1) / GBN;
    // Workgroups are dealt round-robin to the eight compute dies, each with its own L2.  The
    // workgroups that read the same planes (same block of weights and K-slice, different rows of
    // X) get ids that are congruent mod 8, so they run on one die and the planes are fetched
    // into one L2 once.  It is the (weight block, K-slice) pairs that are dealt to the dies, so
    // that every die gets the same number of them, give or take one (dealing whole blocks left
    // two dies with twice the work at 10 blocks: 512 x 5120 x 13824 in three K-slices took 136 us, now 87).
    const int xcd = blockIdx.x & 7;
    int id = blockIdx.x >> 3;
    const int mb = id % mblk;
    id /= mblk;
    const int pair = id * 8 + xcd;
    if (pair >= nblk * split_k) return;      // the grid is padded to a multiple of eight pairs
    const int nbw = pair / split_k, s = pair % split_k;
    // slices are whole steps; k tiles that fill none go to the last slice
    const int kt_begin = slice_begin(ktiles / KW, split_k, s) * KW;
    const int kt_end = s + 1 < split_k ? slice_begin(ktiles / KW, split_k, s + 1) * KW : ktiles;
    const int m0 = mb * BM;
    const int nb0 = nbw * GBN + nw;            // block of output channels of this wavefront
    const int i = lane & 15, g = lane >> 4;
    const uint32_t smem_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

    // X DMA: this wavefront moves the 8-row groups j = (wave*XL + p) % XG; group j belongs to k tile j / (BM/8)
    // of the step and holds rows 8 * (j % (BM/8)) .. +7; lane l of a group fetches row l/8 of them, chunk
    // (l%8) ^ (l/8), and lands at chunk position l%8.
    uint32_t xlane[XL], xlds[XL];
#pragma unroll
    for (int p = 0; p < XL; p++) {
        const int j = (wave * XL + p) % XG;
        int row = m0 + (j % (BM / 8)) * 8 + (lane >> 3);
        row = row < M ? row : M - 1;      // rows past M are computed on valid data and dropped
        xlane[p] = (uint32_t)row * (uint32_t)K * 2u + (uint32_t)(((lane & 7) ^ (lane >> 3)) * 16) +
                   (uint32_t)((j / (BM / 8)) * kTile * 2);
        xlds[p] = j * 1024;
    }
    const uint32_t wlane = lane * 16;
    const uint32_t wlds = wave * kWaveTileBytes;            // inside a stage of the plane ring
    // blocks of channels past N are computed on the last valid block and dropped
    const size_t tile0 = (size_t)min(nb0, nblocks - 1) * ktiles;

    // DMA instruction p of XL: this wavefront's part of the activations of the step that starts at k tile `kt`, into stage sx
    auto issue_x = [&](int kt, int sx, int p) {
        const unsigned char* xb = reinterpret_cast<const unsigned char*>(X) + (size_t)kt * (kTile * 2);
        dma16(xb, xlane[p], smem_base + sx * kXBytes + xlds[p]);
    };
    // DMA instruction p of PL: its own planes of the step that starts at `ktw`, into stage sw
    auto issue_planes = [&](int ktw, int sw, int p) {
        const uint32_t sb = smem_base + kPlaneBase + sw * kPlaneBytes;
        const int kt = ktw + kh;          // this wavefront's k tile of the step
        if (p < 2) {
            const unsigned char* hb = reinterpret_cast<const unsigned char*>(hi) + (tile0 + kt) * kHiTileBytes;
            dma16(hb + p * 1024, wlane, sb + wlds + p * 1024);
        } else if (p == 2) {
            // FP5: the 1-bit plane has 512 bytes per tile; the upper lanes fetch them a second time
            // (into the unused half of the stage's 1 KB) rather than bytes of the next tile
            const unsigned char* lb = reinterpret_cast<const unsigned char*>(lo) + (tile0 + kt) * kLoBytesOf<FMT>;
            dma16(lb, FMT != kE3M1 ? wlane : (wlane & 511u), sb + wlds + 2048);
        } else {
            // fine-grained scales of this tile's block for the wavefront's 64 channels: 128 bytes, fetched by lanes
            // 0..31 (the upper lanes fetch the same bytes again rather than bytes past the array)
            const unsigned char* sp = reinterpret_cast<const unsigned char*>(scales) +
                                      ((size_t)(kt >> gshift) * N + (size_t)min(nb0, nblocks - 1) * kTile) * 2;
            dma4(sp, (lane & 31) * 4, sb + kScaleOff + wave * 256);
        }
    };
    // Steps past the end fetch the last KW k tiles again; so does the last one where the k tiles of the slice fill no whole
    // number of steps, and a wavefront whose tile the step before has worked on gets zeros for its activations (`x_of`).
    const int kt_last = kt_end - KW;

    // operand reads: row r = 16a + i, chunk 4q + g, at position (4q + g) ^ (i & 7), in this wavefront's k tile of the stage
    const int xoff0 = kh * (BM * kTile * 2) + i * (kTile * 2) + ((g ^ (i & 7)) * 16);
    const int xoff1 = kh * (BM * kTile * 2) + i * (kTile * 2) + (((4 + g) ^ (i & 7)) * 16);

    float4v acc[MT][NT];
    float4v part[FGQ ? MT : 1][FGQ ? NT : 1];      // FGQ: product sums of the current block of K
#pragma unroll
    for (int a = 0; a < MT; a++)
#pragma unroll
        for (int t = 0; t < NT; t++) {
            acc[a][t] = float4v{0.f, 0.f, 0.f, 0.f};
            if (FGQ) part[a][t] = float4v{0.f, 0.f, 0.f, 0.f};
        }

    // all of a step's, in the order in which the loop below issues them
    auto issue = [&](int kt, int u) {
#pragma unroll
        for (int p = 0; p < XL; p++)
            if (kWhole) issue_x(min(kt, kt_last), u, p);
#pragma unroll
        for (int p = 0; p < PL; p++) issue_planes(min(kt, kt_last), u, p);
#pragma unroll
        for (int p = 0; p < XL; p++)
            if (!kWhole) issue_x(min(kt, kt_last), u, p);
    };

    // prologue: the steps 0 .. D-1
#pragma unroll
    for (int u = 0; u < D; u++) issue(kt_begin + u * KW, u);

    // operand reads from a stage of the ring
    auto read_x = [&](int ux, int q, int a) {
        return *reinterpret_cast<const half8*>(smem + ux * kXBytes + (q ? xoff1 : xoff0) + a * 16 * (kTile * 2));
    };
    auto read_planes = [&](TileRaw& r, int uw) {
        const unsigned char* wt = smem + kPlaneBase + uw * kPlaneBytes + wlds;
        r.hi0 = *reinterpret_cast<const u32x4*>(wt + wlane);
        r.hi1 = *reinterpret_cast<const u32x4*>(wt + 1024 + wlane);
        if (FMT != kE3M1) {
            r.lo = *reinterpret_cast<const u32x4*>(wt + 2048 + wlane);
        } else {
            const u32x2 l = *reinterpret_cast<const u32x2*>(wt + 2048 + lane * 8);
            r.lo = u32x4{l.x, l.y, 0u, 0u};
        }
    };

    // One step (KW k tiles) is 2 * MT groups of four MFMAs: group j multiplies the 16 rows a = j % MT of X with the
    // wavefront's 64 channels over the 32-wide k block q = j / MT.  Everything else rides between those MFMAs (which the
    // compiler is told to keep so): in group j the operand of X for group j + kAhead is read, one MT-th of the next k block's
    // weights is unpacked, and no two DMA instructions follow each other, which would keep the wavefront waiting.
    // The planes are a wavefront's own: it waits for its own DMA, and refills a stage once the next one has been read.  The
    // activations are everyone's: the barrier comes where the next step's are read first.
    // Against reading a step's operands together behind its barrier, and unpacking each fragment in front of its MFMAs (us, planes of
    // random bits, in turn): 333 x 13824 x 5120 in bf16 66.5 / 61.9 (blocks of 128 rows both), 512 x 8192 x 22016 159 / 144, 512 x 22016 x
    // 8192 165 / 157, 2048 x 8192 x 8192 199 / 192; 198 random plans 4-5 % at 128 x 256, 2-3 % at 128 x 512 and 64 x 256.  At 32 rows (kWhole) a group has 29 vector operations to 4 MFMAs and nothing to hide; there
    // all operands are read a step ahead, behind the barrier at the step's head, and each fragment is unpacked where it is used.
    // tail < 0: a step of the steady state.  Otherwise the tail-th of the last steps, for which everything has been issued: the
    // loads that may be in flight are those of the steps after the next, and the D-th of them has no next step.
    TileRaw raw;                      // planes of the current step
    u32x4 w[4];                       // unpacked weights of the current k block
    half8 x[kXRegs];                  // activations of the next groups
    wait_vmcnt<(D - 1) * kLoads>();
    __syncthreads();
    read_planes(raw, 0);
#pragma unroll
    for (int j = 0; j < kAhead; j++) x[j] = read_x(0, j / MT, j % MT);
    auto read_scales = [&](half4 (&h)[4], int u) {
        const unsigned char* sct = smem + kPlaneBase + u * kPlaneBytes + kScaleOff + wave * 256;
#pragma unroll
        for (int t = 0; t < 4; t++) h[t] = *reinterpret_cast<const half4*>(sct + (t * 16 + g * 4) * 2);
    };
    half4 sc4[4];                     // FGQ, kWhole: the current step's scales
    if (kWhole) {
        if (FGQ) read_scales(sc4, 0);
    } else {
        half8 h[4];
        unpack_kblock<DQ, FMT>(raw, 0, h);
#pragma unroll
        for (int t = 0; t < 4; t++) w[t] = __builtin_bit_cast(u32x4, h[t]);
    }
    auto mac = [&](int a, int t, half8 weights, half8 activations) {
        if (FGQ) part[a][t] = mfma16x16x32_of<FMT>(weights, activations, part[a][t]);
        else acc[a][t] = mfma16x16x32_of<FMT>(weights, activations, acc[a][t]);
    };

    // FGQ, this wavefront's last tile of a block of K (or of the workgroup's K-slice): scale and accumulate
    auto fold = [&](int tile, bool last, const half4 (&sc)[4]) {
        if (!FGQ) return;
        if (((tile + KW) >> gshift) == (tile >> gshift) && !last) return;
#pragma unroll
        for (int t = 0; t < NT; t++) {
#pragma unroll
            for (int a = 0; a < MT; a++) {
#pragma unroll
                for (int r = 0; r < 4; r++) acc[a][t][r] += part[a][t][r] * (float)sc[t][r];
                part[a][t] = float4v{0.f, 0.f, 0.f, 0.f};
            }
        }
    };

    auto step = [&](int kt, int u, auto tail) {
        constexpr int T = decltype(tail)::value;
        constexpr bool more = T < D - 1;          // the tail's last possible step has no successor
        const int tile = (T < 0 ? kt : min(kt, kt_last)) + kh;          // this wavefront's k tile
        const uint32_t live = KW == 1 || T < 0 || tile >= kt ? ~0u : 0u;
        auto x_of = [&](half8 v) {
            return KW == 1 || T < 0 ? v : __builtin_bit_cast(half8, __builtin_bit_cast(u32x4, v) & live);
        };
        TileRaw raw_n;
        if constexpr (kWhole) {
            half8 xn[4];
            half4 sc_n[4];
            if constexpr (more) {
                wait_vmcnt<(T < 0 ? D - 2 : D - 2 - T) * kLoads>();
                __syncthreads();
                if (T < 0) issue(kt + D * KW, u);
                read_planes(raw_n, (u + 1) % D);
#pragma unroll
                for (int j = 0; j < 4; j++) xn[j] = read_x((u + 1) % D, j / MT, j % MT);
                if (FGQ) read_scales(sc_n, (u + 1) % D);
            }
#pragma unroll
            for (int q = 0; q < 2; q++) {
                half8 w4[4];
                if (layout2(FMT)) unpack_kblock<DQ, FMT>(raw, q, w4);
#pragma unroll
                for (int t = 0; t < 4; t++) {
                    if (!layout2(FMT)) w4[t] = unpack_tile_fragment<DQ, FMT>(raw, 2 * t + q);
#pragma unroll
                    for (int a = 0; a < MT; a++) mac(a, t, w4[t], x_of(x[q * MT + a]));
                }
            }
            fold(tile, kt + KW >= kt_end, sc4);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (more) {
                raw = raw_n;
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    x[j] = xn[j];
                    if (FGQ) sc4[j] = sc_n[j];
                }
            }
            return;
        }
        half4 sc[4];
        if (FGQ) read_scales(sc, u);
#pragma unroll
        for (int q = 0; q < 2; q++) {
            u32x4 wn[4];
            u32x6 merged;
            uint32_t em, signed_em;
#pragma unroll
            for (int a = 0; a < MT; a++) {
                const int j = q * MT + a, ja = j + kAhead;
                if constexpr (more) {
                    if (j == kPlanesAt) {
                        wait_vmcnt<XL + (T < 0 ? D - 2 : D - 2 - T) * kLoads>();
                        read_planes(raw_n, (u + 1) % D);
                    }
                    if (T < 0) {
#pragma unroll
                        for (int p = 0; p < PL; p++) {
                            if (j != min(kPlanesAt + p * kPlanesEvery, kXAt)) continue;
                            if (p == 3) asm volatile("" : "+v"(sc[0]), "+v"(sc[1]), "+v"(sc[2]), "+v"(sc[3]));    // (they have been read)
                            issue_planes(min(kt + D * KW, kt_last), u, p);
                        }
                    }
                    if (j == kXAt) {
                        wait_vmcnt<T < 0 ? (D - 2) * kLoads + PL : (D - 2 - T) * kLoads>();
                        __syncthreads();
                    }
                    if (T < 0) {
#pragma unroll
                        for (int p = 0; p < XL; p++)
                            if (j == kXAt + p * kAhead / XL) issue_x(min(kt + D * KW, kt_last), u, p);
                    }
                }
                if (ja < 2 * MT) x[ja % kXRegs] = read_x(u, ja / MT, ja % MT);
                else if (more) x[ja % kXRegs] = read_x((u + 1) % D, (ja - 2 * MT) / MT, (ja - 2 * MT) % MT);
                const half8 xa = x_of(x[j % kXRegs]);
#pragma unroll
                for (int t = 0; t < 4; t++) {
                    mac(a, t, __builtin_bit_cast(half8, w[t]), xa);
                    if (q == 0 || more) {
                        const TileRaw& r = q ? raw_n : raw;
                        if (layout2(FMT)) {
                            if (a == 0 && t == 0) merged = merge_kblock(r, 1 - q);
                            if (a == MT / 2 && t == 0) convert_kblock<FMT>(merged, wn);
                        } else {
                            // 32 steps over the 4 * MT MFMAs of the k block
#pragma unroll
                            for (int c = 0; c < 32; c++) {
                                if (c * MT / 8 != 4 * a + t) continue;
                                unpack_step<DQ, FMT>(r, 1 - q, c, em, signed_em, wn);
                                // (a fragment is finished here, and not where it is used first)
                                if ((c & 7) == 7) asm volatile("" : "+v"(wn[c >> 3]));
                            }
                        }
                    }
                }
                // issue order of the group: each MFMA with its share of the vector operations behind it
                if (ja < 2 * MT || more) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
#pragma unroll
                for (int t = 0; t < 4; t++) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (q == 0 || more) {
#pragma unroll
                for (int t = 0; t < 4; t++) w[t] = wn[t];
            }
        }
        fold(tile, kt + KW >= kt_end, sc);
        if (FGQ) __builtin_amdgcn_sched_barrier(0);
        if constexpr (more) raw = raw_n;
    };

    constexpr auto steady = std::integral_constant<int, -1>();
    int kt = kt_begin;
    for (; kt + D * KW < kt_end; kt += D * KW) {         // steady state: branch-free trips of D steps
#pragma unroll
        for (int u = 0; u < D; u++) step(kt + u * KW, u, steady);
    }
    // One to D steps are left; their stages have all been issued by then, so they fetch nothing, and a slice of few k tiles
    // pays for no more stages than its ring has.
    static_assert(D <= 4, "one line below per step");
    auto last = [&](auto nth) {
        constexpr int u = decltype(nth)::value;
        if constexpr (u < D) {
            if (kt + u * KW < kt_end) step(kt + u * KW, u, nth);
        }
    };
    last(std::integral_constant<int, 0>());
    last(std::integral_constant<int, 1>());
    last(std::integral_constant<int, 2>());
    last(std::integral_constant<int, 3>());
    wait_vmcnt<0>();     // the over-fetched ring slots must land before LDS is given back
    __syncthreads();

    // ---- the K-ways of the workgroup: all sets of wavefronts but the first hand their sums over in LDS and are done
    if (KW > 1) {
        float4v* sums = reinterpret_cast<float4v*>(smem);
        if (kh) {
#pragma unroll
            for (int a = 0; a < MT; a++)
#pragma unroll
                for (int t = 0; t < NT; t++) sums[((kh - 1) * MT * NT + a * NT + t) * OUT_THREADS + nw * 64 + lane] = acc[a][t];
        }
        __syncthreads();
        if (kh) return;            // (barriers from here on wait for the wavefronts that are left)
#pragma unroll
        for (int k = 0; k < KW - 1; k++)
#pragma unroll
            for (int a = 0; a < MT; a++)
#pragma unroll
                for (int t = 0; t < NT; t++) acc[a][t] += sums[(k * MT * NT + a * NT + t) * OUT_THREADS + nw * 64 + lane];
    }

    // Everything below is addressed through a copy of the thread index that the compiler cannot
    // see through, so that none of its address arithmetic is hoisted above the main loop, where it
    // would take registers the loop needs (and a spilled value reloaded inside the loop makes the
    // compiler drain the DMA queue).
    int tid2 = tid;
    asm volatile("" : "+v"(tid2));
    const int i2 = tid2 & 15, g2 = (tid2 >> 4) & 3;

    // ---- K-slices of other workgroups
    if (split_k > 1) {
        const int tile = nbw * mblk + mb, ntiles = mblk * nblk;
        __amdgpu_buffer_rsrc_t mine = partial_window(partials + ((size_t)s * ntiles + tile) * kTileRegs, kTileRegs * 16);
        auto store = [&](int a) {
#pragma unroll
            for (int t = 0; t < NT; t++) store_partial(mine, tid2, acc[a][t], (a * NT + t) * OUT_THREADS);
        };
        if (m0 + BM <= M) {
#pragma unroll
            for (int a = 0; a < MT; a++) store(a);
        } else {
#pragma unroll
            for (int a = 0; a < MT; a++) {
                if (m0 + a * 16 >= M) break;          // rows past M: nobody reads them
                store(a);
            }
        }
        if (second_launch) return;                        // add_slices_kernel does the rest
        if (!arrive_last(&counters[tile * kCounterStride], (uint32_t)split_k)) return;
        // Two slices: the one that arrives last adds the other's sums to its own, which it still holds - a + b
        // does not depend on who that is.  More slices: all of them are read back and added in slice order.
        const bool two = split_k == 2;
        if (!two) {
#pragma unroll
            for (int a = 0; a < MT; a++)
#pragma unroll
                for (int t = 0; t < NT; t++) acc[a][t] = float4v{0.f, 0.f, 0.f, 0.f};
        }
        for (int ss = two ? 1 - s : 0; ss < (two ? 2 - s : split_k); ss++) {
            __amdgpu_buffer_rsrc_t win = partial_window(partials + ((size_t)ss * ntiles + tile) * kTileRegs, kTileRegs * 16);
            // up to AG * 4 16-byte loads in flight at a time: more would need registers the main loop
            // cannot spare
            constexpr int AG = MT < 4 ? MT : (MT % 4 == 0 ? 4 : (MT % 3 == 0 ? 3 : (MT == 5 ? 5 : 4)));
#pragma unroll
            for (int a0 = 0; a0 < MT; a0 += AG) {
                float4v v[AG][NT];
#pragma unroll
                for (int a = 0; a < AG; a++)
#pragma unroll
                    for (int t = 0; t < NT; t++)
                        if (a0 + a < MT) v[a][t] = load_partial(win, tid2, ((a0 + a) * NT + t) * OUT_THREADS);
#pragma unroll
                for (int a = 0; a < AG; a++)
#pragma unroll
                    for (int t = 0; t < NT; t++)
                        if (a0 + a < MT) acc[a0 + a][t] += v[a][t];
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // ---- epilogue: lane holds channels n = 16t + 4g + r of row m = 16a + i  (i2, g2 = i, g)
    if (nb0 >= nblocks) return;
    float sc[4][4];
#pragma unroll
    for (int t = 0; t < 4; t++) {
        half4 h = half4{1, 1, 1, 1};       // fine-grained scales were applied block by block
        if (!FGQ) h = *reinterpret_cast<const half4*>(scales + (size_t)nb0 * kTile + t * 16 + g2 * 4);
#pragma unroll
        for (int r = 0; r < 4; r++) sc[t][r] = (float)h[r] * kUnshift<DQ, FMT>;
    }
#pragma unroll
    for (int a = 0; a < MT; a++) {
        const int m = m0 + a * 16 + i2;
        if (m < M) {
#pragma unroll
            for (int t = 0; t < 4; t++) {
                float yv[4];
#pragma unroll
                for (int r = 0; r < 4; r++) yv[r] = acc[a][t][r] * sc[t][r];
                *reinterpret_cast<half4*>(Y + (size_t)m * N + (size_t)nb0 * kTile + t * 16 + g2 * 4) = to_out4<FMT>(yv);
            }
        }
    }
}

// The second launch of a split layer: adds the slices (in slice order) and applies the epilogue.  A workgroup takes 16 rows of one
// 64-channel block: the partial sums of four rows are pieces of 64 bytes, so its four wavefronts share whole cache lines (four
// neighbouring blocks of the same four rows fetched every line twice: of 1320 plans with 192 KB of partial sums per block of Y
// and more 88 were slower than with the last arriver, now 36).  A wavefront takes four rows, 16 lanes a row, and writes
// 128-byte pieces of Y.  GBN and BM are those of the launch that wrote the partial sums (a block of Y holds them as
// [row block a][16-channel block t][thread]).
template <bool FGQ, int FMT, int DQ>
__global__ __launch_bounds__(256) void add_slices_kernel(const float4v* __restrict__ partials, const uint16_t* __restrict__ scales,
                                                         int M, int N, int bm, int gbn, int split_k, uint16_t* __restrict__ Y)
{
    const int lane = threadIdx.x & 63;
    const int nblocks = N / kTile;
    const int nb = (int)(blockIdx.x % (unsigned)nblocks);
    const int m = (int)(blockIdx.x / (unsigned)nblocks) * 16 + (threadIdx.x >> 6) * 4 + (lane >> 4);
    if (m >= M) return;
    const int t = (lane >> 2) & 3, g = lane & 3;
    const int mblk = (M + bm - 1) / bm, nblk = (nblocks + gbn - 1) / gbn;
    const int mb = m / bm, a = (m % bm) >> 4, i = m & 15;
    const size_t tile_regs = (size_t)bm * gbn * 16;
    const size_t slice = tile_regs * mblk * nblk;
    const float4v* p = partials + ((size_t)(nb / gbn) * mblk + mb) * tile_regs + (size_t)(a * 4 + t) * (gbn * 64) + (nb % gbn) * 64 + g * 16 + i;
    const int n = nb * kTile + t * 16 + g * 4;
    half4 sc = half4{1, 1, 1, 1};          // fine-grained scales were applied block by block
    if (!FGQ) sc = *reinterpret_cast<const half4*>(scales + n);
    float4v sum = float4v{0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < split_k; s0 += 8) {          // eight loads in flight
        float4v v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) v[u] = p[(size_t)min(s0 + u, split_k - 1) * slice];
#pragma unroll
        for (int u = 0; u < 8; u++)
            if (s0 + u < split_k) sum += v[u];
    }
    float yv[4];
#pragma unroll
    for (int r = 0; r < 4; r++) yv[r] = sum[r] * ((float)sc[r] * kUnshift<DQ, FMT>);
    *reinterpret_cast<half4*>(Y + (size_t)m * N + n) = to_out4<FMT>(yv);
}

template <int BM, int DQ = kBiasShift, bool FGQ = false, int FMT = kE3M2, int GBN = 8, int KW = 1>
static hipError_t launch_gemm_t(const LinearPlan& p, const uint16_t* X, int64_t M, const void* hi, const void* lo,
                                const uint16_t* scales, int64_t N, int64_t K, uint16_t* Y, void* workspace,
                                hipStream_t stream)
{
    uint32_t* counters = reinterpret_cast<uint32_t*>(workspace);
    float4v* partials = reinterpret_cast<float4v*>(reinterpret_cast<char*>(workspace) + kZeroBytes);
    const int64_t mblk = (M + BM - 1) / BM, nblk = (N / kTile + GBN - 1) / GBN;
    const unsigned grid = (unsigned)(mblk * ((nblk * p.split_k + 7) / 8 * 8));   // padded: see the id mapping
    constexpr int D = ring_stages(BM, GBN, KW);
    hipLaunchKernelGGL((gemm_kernel<BM, D, DQ, FGQ, FMT, GBN, KW>), dim3(grid), dim3(GBN * KW * 64), 0, stream, X, (int)M,
                       (const u32x4*)hi, (const u32x4*)lo, scales, (int)N, (int)K, Y, partials, counters, p.split_k, p.gshift, p.second_launch);
    if (p.second_launch) {
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((add_slices_kernel<FGQ, FMT, DQ>), dim3((unsigned)((M + 15) / 16 * (N / kTile))), dim3(256), 0, stream, partials, scales,
                           (int)M, (int)N, BM, GBN, p.split_k, Y);
    }
    return hipGetLastError();
}

}  // namespace fp6
