// Backprojection of a fused chunk (paper, Sections 2.2 and 3, "LineRec"): the
// filtered rows that the normalise + filter kernels wrote in blocks of 8
// slices, summed over angles on the matrix cores.  Rows in sinogram order go
// through k_backproject.hip.
//
// Detector coordinate of voxel (ix, iy) at angle a, for tile (bx, by) =
// (ix / 32, iy / 32) and in-tile offset (dx, dy) = (ix % 32, iy % 32):
//   s = bi + fma(dx, cos_a, fma(dy, sin_a, bf)),
//   bi + bf = (bx*32 - N/2) cos_a + (by*32 - N/2) sin_a + center   (FP64 on the host,
//   split into integers xi + yi and FP32 fractions xf + yf),
// the expression of k_backproject.hip and k_radon.hip.
//
// The sum over angles is a matrix product:
//   slice[voxel][z] += sum over (angle, bin) W[voxel][(angle, bin)] rows[(angle, bin)][z],
// where W holds a voxel's two weights per angle.  The 16 voxels of a 4x4 block
// see at most 7 consecutive bins of an angle (3 (|cos| + |sin|) <= 4.25 bins
// apart, plus the second tap), so one 16x16x32 instruction adds 4 angles x 8
// bins for 16 voxels and 16 slices:
//   A operand: lane l holds voxel l % 16, angle l / 16: its 8 weights;
//   B operand: lane l holds slice l % 16, angle l / 16: 8 consecutive samples;
//   result:    lane l holds slice l % 16, voxels (0..3, l / 16) of the block.
// The weights cost about 20 VALU instructions per (block, 4 angles) and serve
// every slice of the work-group (up to 64).
//
// Precision (16-bit operands, FP32 sums):
//   FP16 rows:  weights (1 - w, w) rounded to FP16 (the 16-bit mode), products exact;
//   BF16 rows:  the BF16 values as FP16 (times 2^12: the filtered rows of 16-bit
//               counts stay below 7), weights as two FP16 values;
//   FP32 rows:  rows and weights as two FP16 values each (22 bits and the sign
//               of the second); three products, the dropped one is below 2^-22
//               of its term.  The rows' second values are kept 2^11 times as
//               large and have sums of their own, joined at the end: unscaled
//               they are subnormal for faint objects (at a largest line integral
//               of 0.0001 the error was 2.8e-6, now as at 1, 8.9e-7).
// Each voxel's sum depends only on its block and on the angles taken 4 at a
// time, so results do not depend on the tiling, the chunk or the row count.
// Rows here are always finite (counts are clamped before the logarithm), so a
// zero weight never meets a NaN.
//
// Work-group: one tile of 32x32 (or 16x16) voxels x 16 NT slices, one or two waves
// per row of 4x4 blocks.  A block of A angles stages, per angle, the window of bins
// that the tile can reach, straight from global memory into one of two LDS
// buffers while the other one is summed; LDS holds [16-slice tile][bin][slice],
// and the transposing read (ds_read_b64_tr_b16) takes 4 bins from any start.
// (Rows kept sample by sample, as in sinogram order, need 16-byte reads at any
// 4-byte address, which ran at a fraction of the LDS rate: 69 ms where the
// transposing reads take 21.)
//
// What bounds it (counters of 256 slices of the 2048-cubed scan; a CU issues one
// vector instruction a cycle at the half rate of conversions, permutes and
// comparisons, two at the full one): FP16 rows 44.7 ms (a kernel with one dot
// product per voxel, slice and angle: 115.6), per 4x4 block, 4 angles and 64
// slices 20.8 vector instructions (0.48 a cycle and CU), 9.9 LDS reads (the LDS
// busy 0.52 of the time) and 4 matrix instructions (0.37), in turn; BF16 rows 58.7
// ms (150.9); FP32 rows 114 ms (162.6), per 32 slices 35.8 vector instructions
// (0.63), 9.9 LDS reads (0.39) and 6 matrix instructions (0.42).
#include <type_traits>

#include "blocked_rows.h"
#include "mfma_lds.h"

namespace tp {
namespace {

template <int ST, int TB, int NT> struct Tile {
    static constexpr int kBlocks = TB / 4;             // 4x4 blocks per side
    static constexpr int kSplit = TB == 32 && NT * Blocked<ST>::PB == 4 ? 2 : 1;  // waves per row of blocks
    static constexpr int kWaves = kBlocks * kSplit, kThreads = 64 * kWaves;
    // bins per staged window: blocks start at most 1.4143 (TB - 4) + 1 bins
    // past the tile's first one and read 8 (40 + 8 = 48, 17 + 8 < 32)
    static constexpr int kWinB = TB == 32 ? 48 : 32;
    static constexpr int kBytes = 64 * kWinB;          // of a tile of 16 slices for two angles
};

// LDS layout: [plane][angle pair][16-slice tile][bin][angle of the pair][slice] (mfma_lds.h).
constexpr int kRing = 4;
template <int ST, int TB, int NT>
constexpr size_t bb_lds() {
    return size_t{2} * Blocked<ST>::PB * (Blocked<ST>::A / 2) * NT * Tile<ST, TB, NT>::kBytes + kRing * Blocked<ST>::A * 24 +
           7 * 16;
}

// Tile of work-group `wg` among nb x nb tiles.  Work-groups are dispatched
// round-robin over the 8 XCDs, so wg % 8 names the XCD; each XCD gets one
// eighth of the grid (nb/2 x nb/4 tiles) and walks it in Morton order, so the
// work-groups resident on an XCD at a time form a compact cluster whose
// detector windows overlap in that XCD's L2.  Bijective for power-of-two
// nb >= 8; other sizes give each XCD a contiguous range of tiles, walked in
// strips 8 tiles high.
__device__ __forceinline__ void tile_of(int wg, int nb, int& bx, int& by) {
    if (nb >= 8 && (nb & (nb - 1)) == 0) {
        const int part = wg & 7, q = wg >> 3;
        const int hr = nb >> 2;                      // part is (2 hr) x hr tiles
        const int sq = hr * hr;
        const int half_x = q / sq;                   // left or right square of the part
        int r = q - half_x * sq, sx = 0, sy = 0;
        for (int bit = 0; (1 << (2 * bit)) < sq; ++bit) {
            sx |= ((r >> (2 * bit)) & 1) << bit;
            sy |= ((r >> (2 * bit + 1)) & 1) << bit;
        }
        bx = (part & 1) * (2 * hr) + half_x * hr + sx;
        by = (part >> 1) * hr + sy;
    } else {
        const int total = nb * nb, q = total >> 3, rem = total & 7, x = wg & 7;
        const int item = x * q + min(x, rem) + (wg >> 3);
        const int strip = item / (8 * nb), in = item - strip * 8 * nb;
        const int high = min(8, nb - 8 * strip);
        bx = in / high;
        by = 8 * strip + in - bx * high;
    }
}

// The pair p = (1 - w, w) at 16-bit slots d and d + 1 (d in 0..6) of an 8-slot
// operand: four byte permutes with the selectors of row d of a table in LDS.
__device__ __forceinline__ void place_table(uint32_t* tab, int tid) {
    if (tid < 28) {
        const int e = (tid >> 2) - 2 * (tid & 3);  // slot d relative to register tid % 4
        tab[tid] = e == 0 ? 0x03020100u : e == 1 ? 0x01000c0cu : e == -1 ? 0x0c0c0302u : 0x0c0c0c0cu;
    }
}
__device__ __forceinline__ u4_t place_pair(uint32_t p, u4_t sel) {
    u4_t r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __builtin_amdgcn_perm(p, p, sel[i]);
    return r;
}


// 32-voxel tiles are held to 128 registers, 4 waves per SIMD: two work-groups
// of 8 waves per CU, or one of 16.
//
// NARROW: fewer than 8 slices in blocks as wide as there are, where the workspace
// has no room for whole blocks.  A lane picks its bin's samples one by one and
// pads them with zeros (one slice of 1024 x 1024 from 900 angles, FP32: 1.04 ms
// against 0.90 of whole blocks; 5 slices 1.24 against 0.92).
template <int ST, typename OutT, int TB, int NT, bool NARROW>
__global__ void __launch_bounds__((Tile<ST, TB, NT>::kThreads)) __attribute__((amdgpu_waves_per_eu(TB == 32 ? 4 : 1)))
k_backproject_blocked(GeoTables g, const uint16_t* __restrict__ rows, int n_rows, float scale,
                      OutT* __restrict__ vol) {
    constexpr int A = Blocked<ST>::A, PA = Blocked<ST>::PA, PB = Blocked<ST>::PB;
    constexpr int W = Tile<ST, TB, NT>::kWaves, BW = Tile<ST, TB, NT>::kBlocks / Tile<ST, TB, NT>::kSplit;  // waves, blocks of each
    constexpr int KS = 16 * NT;                            // slices
    constexpr int kTile = Tile<ST, TB, NT>::kBytes, kPair = NT * kTile, kPlane = (A / 2) * kPair, kBuf = PB * kPlane;
    constexpr int kParts = kTile / 1024;                   // 1 KiB pieces of a tile: one load of a wave each
    constexpr int kLoads = PB * (A / 2) * NT * kParts;
    static_assert(kLoads * 1024 == kBuf, "whole pieces");
    extern __shared__ __align__(16) unsigned char smem[];
    // ring of the angles' geometry: {bf, cos, sin, 64 (bi - j0)}; bf plus the
    // offset of a block's minimising corner, less 2^-10; j0, the first staged bin
    float4* sGeo = reinterpret_cast<float4*>(smem + 2 * kBuf);            // [kRing][A]
    float* sCor = reinterpret_cast<float*>(sGeo + kRing * A);             // [kRing][A]
    int* sJ0 = reinterpret_cast<int*>(sCor + kRing * A);                  // [kRing][A]
    uint32_t* sSel = reinterpret_cast<uint32_t*>(sJ0 + kRing * A);        // [7][4] place_pair's selectors

    const int na = g.na, n = g.n, nbt = (g.N + TB - 1) / TB;
    int tx, ty;
    tile_of(blockIdx.x, nbt, tx, ty);
    const int bx = tx * TB / kGeoTile, by = ty * TB / kGeoTile;            // table tile
    const int ex = tx * TB % kGeoTile, ey = ty * TB % kGeoTile;            // this tile's offset in it
    const int z0 = blockIdx.y * KS;
    const int kz = min(KS, n_rows - z0);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nblk = (na + A - 1) / A;

    // sums, and those of the products with the rows' second values
    f4_t acc[BW][NT], low[PB == 2 ? BW : 1][NT];
#pragma unroll
    for (int i = 0; i < BW; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            acc[i][t] = f4_t{0.0f, 0.0f, 0.0f, 0.0f};
            if (PB == 2) low[i][t] = f4_t{0.0f, 0.0f, 0.0f, 0.0f};
        }

    // Geometry of block k's angles (one lane each): table entries as loaded, a
    // block before they are summed and written, so no wait follows the loads.
    struct Entry {
        float cs, sn, xf, yf;
        int xi, yi;
    };
    auto geo_load = [&](int k) {
        Entry e{1.0f, 0.0f, 0.0f, 0.0f, 0, 0};
        const int a = k * A + tid;
        if (tid < A && a < na) {
            e.cs = g.cs[a];
            e.sn = g.sn[a];
            e.xi = g.xi[bx * na + a];
            e.yi = g.yi[by * na + a];
            e.xf = g.xf[bx * na + a];
            e.yf = g.yf[by * na + a];
        }
        return e;
    };
    auto geo_write = [&](int k, const Entry& e) {
        if (tid < A) {
            // every voxel's floor is at least that of the tile's minimising
            // corner; the blocks' starts below are within 1e-4 of theirs, less 2^-10
            const float bf = e.xf + e.yf;
            const int bi = e.xi + e.yi;
            const float smin = tile_offset(static_cast<float>(e.cs >= 0.0f ? ex : ex + TB - 1),
                                           static_cast<float>(e.sn >= 0.0f ? ey : ey + TB - 1), e.cs, e.sn, bf);
            const int first = coord_floor(smin - 0.001953125f);
            const int at = (k & (kRing - 1)) * A + tid;
            sGeo[at] = make_float4(bf, e.cs, e.sn, __int_as_float(-64 * first));
            sCor[at] = bf + (3.0f * fminf(e.cs, 0.0f) + (3.0f * fminf(e.sn, 0.0f) - 0.0009765625f));
            // past the last angle: a start off every detector, so that zeros are staged
            sJ0[at] = k * A + tid < na ? bi + first : 1 << 30;
        }
    };

    // Staging: each load of a wave moves 1 KiB of LDS: 16 bins of a 16-slice
    // tile for a pair of angles, 16 bytes (8 slices of one bin) per lane.
    const int lpar = (lane >> 1) & 1;
    const int last8 = (n_rows - 1) >> 3;
    const int64_t slab = static_cast<int64_t>(na) * PB * n;  // 16-byte units of 8 slices' rows
    const uint32_t lds0 = lds_address(smem);
    const u4_t* units = reinterpret_cast<const u4_t*>(rows);
    const int64_t odd = (lane & 1) ? slab : 0;                // the tile's second 8 slices
    const u4_t* lane_units = units + static_cast<int64_t>(lpar * PB) * n;
    auto stage = [&](int k) {
#pragma unroll
        for (int s = 0; s < (kLoads + W - 1) / W; ++s) {
            const int i = s * W + wv;
            if (kLoads % W != 0 && i >= kLoads) break;
            const int part = i % kParts, t = i / kParts % NT, pair = i / (kParts * NT) % (A / 2),
                      pl = i / (kParts * NT * (A / 2));
            const int j = sJ0[(k & (kRing - 1)) * A + 2 * pair + lpar] + (16 * part + (lane >> 2));
            // slices past the last are read from its group again; their sums are never stored
            const int g8 = min((z0 >> 3) + 2 * t, last8);
            const int64_t at = g8 * slab + static_cast<int64_t>((k * A + 2 * pair) * PB + pl) * n;  // uniform
            const u4_t* src = lane_units + (g8 < last8 ? odd : int64_t{0}) + (at + static_cast<uint32_t>(j));
            load_lds16(static_cast<unsigned>(j) < static_cast<unsigned>(n) ? src : reinterpret_cast<const u4_t*>(g_zero),
                       lds0 + (k & 1) * kBuf + i * 1024);
        }
    };

    // The same of NARROW blocks, through registers: loaded before a block is
    // summed, written after it.
    constexpr int kPieces = (kLoads + W - 1) / W;
    u4_t piece[NARROW ? kPieces : 1];
    auto take = [&](int k) {
#pragma unroll
        for (int s = 0; s < kPieces; ++s) {
            const int i = s * W + wv;
            if (kLoads % W != 0 && i >= kLoads) break;
            const int part = i % kParts, pair = i / kParts % (A / 2), pl = i / (kParts * (A / 2));
            const int j = sJ0[(k & (kRing - 1)) * A + 2 * pair + lpar] + (16 * part + (lane >> 2));
            piece[s] = u4_t{0, 0, 0, 0};
            if ((lane & 1) == 0 && static_cast<unsigned>(j) < static_cast<unsigned>(n)) {
                const uint16_t* p = rows + (static_cast<int64_t>((k * A + 2 * pair + lpar) * PB + pl) * n + j) * n_rows;
#pragma unroll
                for (int z = 0; z < 7; ++z)
                    if (z < n_rows) piece[s][z >> 1] |= static_cast<uint32_t>(p[z]) << (16 * (z & 1));
            }
        }
    };
    auto put = [&](int k) {
#pragma unroll
        for (int s = 0; s < kPieces; ++s) {
            const int i = s * W + wv;
            if (kLoads % W != 0 && i >= kLoads) break;
            *reinterpret_cast<u4_t*>(smem + (k & 1) * kBuf + i * 1024 + 16 * lane) = piece[s];
        }
    };

    place_table(sSel, tid);
    geo_write(0, geo_load(0));
    geo_write(1, geo_load(1));
    Entry ent = geo_load(2);
    __syncthreads();
    if constexpr (NARROW) {
        take(0);
        put(0);
    } else {
        stage(0);
        wait_loads();
    }
    __syncthreads();

    const int vx = lane & 3, vy = (lane >> 2) & 3, ag = lane >> 4;  // A operand: the lane's voxel and angle
    const int wrow = 4 * (wv / Tile<ST, TB, NT>::kSplit), wcol = 4 * BW * (wv % Tile<ST, TB, NT>::kSplit);  // first block
    const float dyv = static_cast<float>(ey + wrow + vy);
    const float dxv = static_cast<float>(ex + wcol + vx);
    const float dx0 = static_cast<float>(ex + wcol), dy0 = static_cast<float>(ey + wrow);
    const unsigned char* lane_buf = smem + (ag >> 1) * kPair + (ag & 1) * 32 + 8 * (lane & 3) + 64 * vy;
    for (int k = 0; k < nblk; ++k) {
        // the geometry first: the loads into LDS that follow complete in order,
        // and nothing before the end of the block waits for them
        geo_write(k + 2, ent);
        ent = geo_load(k + 3);
        if (k + 1 < nblk) {
            if constexpr (NARROW) take(k + 1);
            else stage(k + 1);
        }
        const int nA = min(A, na - k * A);
        const float4* geo = sGeo + (k & (kRing - 1)) * A;
#pragma unroll
        for (int gq = 0; gq < A / 4; ++gq) {
            if (4 * gq >= nA) break;
            const float4 ge = geo[4 * gq + ag];  // angles past the last: zero rows, finite weights
            const float cs = ge.y, sn = ge.z;
            const float inner = __builtin_fmaf(dyv, sn, ge.x);
            // estimated start of the first block's window: a little low, and a
            // window one bin early still holds the 7 bins of its block
            const float first = tile_offset(dx0, dy0, cs, sn, sCor[(k & (kRing - 1)) * A + 4 * gq + ag]);
            // the transposing read takes row (lane / 4) % 4 of 4 from this lane's address
            const unsigned char* rowp = lane_buf + (k & 1) * kBuf + 2 * gq * kPair + __float_as_int(ge.w);
            // block i's weights as pairs, their places and its samples
            struct Block {
                uint32_t p[PA];
                u4_t sel, q[NT][PB];
            };
            auto fetch = [&](int i, Block& o) {
                const float s = __builtin_fmaf(dxv + 4.0f * i, cs, inner);
                const int f0 = coord_floor(__builtin_fmaf(cs, 4.0f * i, first));  // first bin of the window
                const int d = coord_floor(s) - f0;                                 // lower tap, 0..6
                o.sel = *reinterpret_cast<const u4_t*>(sSel + 4 * d);
                const unsigned char* src = rowp + 64 * f0;
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int b = 0; b < PB; ++b) o.q[t][b] = read_slots(src + b * kPlane + t * kTile);
                const float w = coord_frac(s), omw = 1.0f - w;
                if constexpr (PA == 1) {
                    o.p[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2_t{omw, w}), half2_t));
                } else {
                    split_pair(omw, w, o.p[0], o.p[1]);
                }
            };
            auto add = [&](int i, const Block& o) {
                u4_t wt[PA];
#pragma unroll
                for (int c = 0; c < PA; ++c) wt[c] = place_pair(o.p[c], o.sel);
                // The matrix cores round after every product they add: with two per tap,
                // FP32 rows take the 4 angles' sum from zero, the smaller product first,
                // and add it once, which keeps the error below that of two FP32 FMAs per
                // angle.  Their second values' products, 2^11 times as large as they
                // count, have a sum of their own; the low parts' product is dropped.
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    f4_t sum = ST == kStF32 ? f4_t{0.0f, 0.0f, 0.0f, 0.0f} : acc[i][t];
#pragma unroll
                    for (int c = PA - 1; c >= 0; --c) sum = mfma16(wt[c], o.q[t][0], sum);
                    acc[i][t] = ST == kStF32 ? acc[i][t] + sum : sum;
                    if constexpr (PB == 2) low[i][t] = mfma16(wt[0], o.q[t][1], low[i][t]);
                }
            };
            // (unrolled: the compiler moves reads of later blocks ahead of products as
            // far as registers allow)
#pragma unroll
            for (int i = 0; i < BW; ++i) {
                Block cur;
                fetch(i, cur);
                add(i, cur);
            }
        }
        if constexpr (NARROW) {
            if (k + 1 < nblk) put(k + 1);
        } else {
            wait_loads();  // this wave's part of block k + 1 is in LDS
        }
        __syncthreads();
    }

    const int N = g.N;
    // whole groups of 4 voxels stored at once: x is a multiple of 4
    const bool wide = (N & 3) == 0 && (reinterpret_cast<uintptr_t>(vol) & (4 * sizeof(OutT) - 1)) == 0;
    const int y = ty * TB + wrow + ag;
    if (y >= N) return;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int z = 16 * t + (lane & 15);
        if (z >= kz) continue;
        OutT* line = vol + (static_cast<int64_t>(z0 + z) * N + y) * N;
#pragma unroll
        for (int i = 0; i < BW; ++i) {
            const int x = tx * TB + wcol + 4 * i;
            f4_t v = (PB == 2 ? acc[i][t] + low[PB == 2 ? i : 0][t] * (1.0f / kLowScale) : acc[i][t]) * scale;
            // FP16 slices: the FP32 result rounded once to nearest.  The value is
            // formed before the conversion: contracted with it, the product that
            // forms it would be rounded to FP16 without the FP32 step.
            asm volatile("" : "+v"(v));
            if (wide) {
                if (x >= N) continue;
                if constexpr (std::is_same<OutT, float>::value)
                    *reinterpret_cast<f4_t*>(line + x) = v;
                else
                    *reinterpret_cast<half4_t*>(line + x) = __builtin_convertvector(v, half4_t);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (x + r < N) store_from_float(line, x + r, v[r]);
            }
        }
    }
}

template <int ST, typename OutT, int TB, int NT, bool NARROW = false>
hipError_t launch_bb_t(const GeoTables& g, const uint16_t* rows, int n_rows, float scale, void* vol, hipStream_t st) {
    constexpr size_t lds = bb_lds<ST, TB, NT>();
    static_assert(lds <= (NARROW ? 64 : 160) * 1024, "LDS of a CU; the default limit");
    if constexpr (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_backproject_blocked<ST, OutT, TB, NT, NARROW>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
        if (e != hipSuccess) return e;
    }
    if (vol == nullptr) return hipSuccess;  // only the attribute
    const unsigned nbt = static_cast<unsigned>((g.N + TB - 1) / TB);
    const dim3 grid(nbt * nbt, static_cast<unsigned>((n_rows + 16 * NT - 1) / (16 * NT)));
    hipLaunchKernelGGL((k_backproject_blocked<ST, OutT, TB, NT, NARROW>), grid, dim3((Tile<ST, TB, NT>::kThreads)), lds, st, g, rows,
                       n_rows, scale, static_cast<OutT*>(vol));
    return hipGetLastError();
}

template <int ST, typename OutT, int TB>
hipError_t launch_bb_n(const GeoTables& g, const uint16_t* rows, int n_rows, float scale, void* vol, int nt,
                       hipStream_t st) {
    switch (nt) {
        case 0: return launch_bb_t<ST, OutT, TB, 1, true>(g, rows, n_rows, scale, vol, st);
        case 1: return launch_bb_t<ST, OutT, TB, 1>(g, rows, n_rows, scale, vol, st);
        case 2: return launch_bb_t<ST, OutT, TB, 2>(g, rows, n_rows, scale, vol, st);
        default:
            if constexpr (ST != kStF32) return launch_bb_t<ST, OutT, TB, 4>(g, rows, n_rows, scale, vol, st);
            return hipErrorInvalidValue;
    }
}

template <int ST, typename OutT>
hipError_t launch_bb(const GeoTables& g, const uint16_t* rows, int n_rows, int wide, float scale, void* vol,
                     hipStream_t st) {
    if (vol == nullptr) {  // every instance a later launch can choose
        for (int nt = 1; nt <= (ST == kStF32 ? 2 : 4); nt *= 2) {
            hipError_t e = launch_bb_n<ST, OutT, 32>(g, rows, n_rows, scale, vol, nt, st);
            if (e == hipSuccess) e = launch_bb_n<ST, OutT, 16>(g, rows, n_rows, scale, vol, nt, st);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    // As many slices per work-group as there are, up to 64 (32 for FP32 rows):
    // they share the weights.  FP32 rows at 64 (two planes of samples and sums
    // from zero) no longer fit 128 registers: 9.3 ms against 7.3 at 32, 128 rows
    // of 1024 x 1024 from 1024 angles.
    const int nt = n_rows > 32 && ST != kStF32 ? 4 : n_rows > 16 ? 2 : 1;
    // 16-voxel tiles where 32-voxel ones give fewer than two work-groups per CU
    // (16 slices of 256 x 256 from 180 angles: 0.044 ms, a quarter of the chip
    // idle with 64 tiles); 32-voxel ones stage half the bins per voxel (one
    // slice of 1024 x 1024 from 900 angles: 1.05 against 1.30 ms).
    const int64_t side = (g.N + 31) / 32;
    const int64_t groups = side * side * ((n_rows + 16 * nt - 1) / (16 * nt));
    const int form = wide < 8 ? 0 : nt;
    if (groups < 512) return launch_bb_n<ST, OutT, 16>(g, rows, n_rows, scale, vol, form, st);
    return launch_bb_n<ST, OutT, 32>(g, rows, n_rows, scale, vol, form, st);
}

}  // namespace

size_t blocked_rows_bytes(int n_rows, int wide, int na, int n, tp_dtype dt) {
    return static_cast<size_t>((n_rows + wide - 1) / wide) * wide * na * n * (dt == TP_F32 ? 4 : 2);
}

// A null `vol` only sets the instances' dynamic-LDS limits, so that later
// launches, possibly graph-captured, make no attribute call that matters (those
// of narrow blocks stay below the default limit).
hipError_t launch_backproject_blocked(const GeoTables& g, const void* rows, tp_dtype dt, int n_rows, int wide,
                                      float scale, void* vol, tp_dtype vol_dt, hipStream_t st) {
    const uint16_t* r = static_cast<const uint16_t*>(rows);
    if (vol_dt == TP_F16)
        return dt == TP_F16 ? launch_bb<kStF16, __half>(g, r, n_rows, wide, scale, vol, st) : hipErrorInvalidValue;
    if (vol_dt != TP_F32) return hipErrorInvalidValue;
    switch (dt) {
        case TP_F32: return launch_bb<kStF32, float>(g, r, n_rows, wide, scale / kRowScale, vol, st);
        case TP_F16: return launch_bb<kStF16, float>(g, r, n_rows, wide, scale, vol, st);
        case TP_BF16: return launch_bb<kStBF16, float>(g, r, n_rows, wide, scale / kRowScale, vol, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace tp
