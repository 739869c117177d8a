// Fourier-domain filtered backprojection (paper, Section 2.2: backprojection
// evaluated with exponential interpolation kernels in the frequency domain;
// Section 3 uses it as the reference method).
//
// By the Fourier slice theorem the spectrum of the projection at angle theta
// is the line of the 2-D image spectrum through the origin in direction
// theta.  Filtered backprojection with band-limited interpolation along each
// ray is therefore a non-uniform inverse DFT from these polar samples to the
// voxel grid:
//   f(x) = sum_{a,k} c_{a,k} exp(2 pi i (k / L) theta_a . x),
//   c_{a,k} = (pi / na) / L * w_k * H[k] * U_a[k] * exp(2 pi i k pos0 / L),
// where U_a is the DFT of the padded row, H the filter response, w_k = 1/2 at
// the two Nyquist terms and pos0 the padded-row position of the axis.  It is
// evaluated as an unequally spaced FFT: every polar sample is spread with a
// Gaussian phi(u) = exp(-|u|^2 / (4 tau)) onto a Cartesian grid of M points
// per side (oversampling >= 2), the grid is inverse-transformed, and each
// voxel is divided by the Gaussian's Fourier transform.
//
// Two slices travel as the real and imaginary parts of one complex row, so
// every transform and the spreading are complex and the two reconstructions
// come back as the real and imaginary parts of the image.
//
// Stages (one launch each):
//   k_fr_spectra  normalise two rows, pad, FFT, multiply by the E table and
//                 store the L + 1 signed-frequency samples of the angle;
//   k_fr_grid     for every grid point, sum the Gaussian-weighted samples of
//                 every angle whose ray passes within the truncation radius
//                 (a gather on the matrix cores: no atomics, a fixed
//                 summation order);
//   k_fr_rows     inverse FFT along the grid's fast axis, keeping the N
//                 output rows, stored in 16-wide column groups;
//   k_fr_cols     inverse FFT along the other axis, deconvolution, split of
//                 the two slices, store.
#include <type_traits>

#include "fft_device.h"
#include "mfma_lds.h"

namespace tp {
namespace {

__device__ __forceinline__ float2 cconj(float2 a) { return make_float2(a.x, 0.0f - a.y); }

// Store one voxel: FP32, or the FP32 value rounded once to FP16.  The value is
// fenced into a register first: otherwise the compiler contracts the product
// that forms it with the conversion (one mixed-precision multiply rounding the
// exact product to FP16), which differs from the FP32 slice rounded at ties.
__device__ __forceinline__ void fr_store(float* p, int64_t i, float v) { p[i] = v; }
__device__ __forceinline__ void fr_store(__half* p, int64_t i, float v) {
    asm volatile("" : "+v"(v));
    p[i] = __float2half_rn(v);
}

// A value all lanes agree on, in a scalar register.
__device__ __forceinline__ float uniform(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

int fr_block(int L) {
    int b = L / 16;
    if (b < 64) b = 64;
    if (b > 1024) b = 1024;
    return b;
}

template <typename K>
hipError_t fr_lds(K kernel, size_t bytes) {
    if (bytes <= 65536) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes));
}

// ---------------------------------------------------------------------------
// Spectra rows: groups of four pairs of slices side by side, so that one
// 16-byte piece holds a sample of four pairs, in two FP16 planes; entry 0 of a
// row is zero (what the gather reads off either end), frequency k is entry
// k + L/2 + 1.  Without room for four pairs, one at a time: rows of one pair
// (t.wide = 1) without the zero (t.first = 0).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t* spectra_row(uint32_t* spec, int p, int slot, const FourierTables& t) {
    return spec + ((static_cast<int64_t>(p / kFrPairGroup) * t.na + slot) * 2 * t.SL) * t.wide + p % kFrPairGroup;
}
// The sample of entry k (counted from frequency -L/2).
__device__ __forceinline__ void spectra_store(uint32_t* row, int k, const FourierTables& t, float2 v) {
    uint32_t hi, lo;
    split_data(v.x, v.y, hi, lo);
    const int at = __mul24(k + t.first, t.wide);
    row[at] = hi;
    row[t.SL * t.wide + at] = lo;
}
__device__ __forceinline__ void spectra_zero(uint32_t* row, const FourierTables& t) {
    if (t.first == 0) return;
    row[0] = 0;
    row[t.SL * t.wide] = 0;
}
// Work-group -> (pair, piece of the angles): work-groups go to the 8 XCDs in
// turn, and the four pairs of a group run back to back on one XCD for the same
// piece, so their 4-byte stores of a line meet in that XCD's L2.
__device__ __forceinline__ void spectra_work(int pairs, int pieces, int& p, int& piece) {
    const int id = blockIdx.x, xcd = id & 7, s = id >> 3, high = min(pairs, kFrPairGroup);
    const int item = s / high * 8 + xcd;
    piece = item % pieces;
    p = item / pieces * kFrPairGroup + s % high;
}
unsigned spectra_grid(int pairs, int pieces) {
    const int64_t items = static_cast<int64_t>((pairs + kFrPairGroup - 1) / kFrPairGroup) * pieces;
    return static_cast<unsigned>((items + 7) / 8 * 8 * (pairs < kFrPairGroup ? pairs : kFrPairGroup));
}

// ---------------------------------------------------------------------------
// Spectra: one work-group per (pair of slices, angle).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(1024)
k_fr_spectra(RawInput in, int rows, const float* __restrict__ dmean, const float* __restrict__ rden,
             const float2* __restrict__ tw, FourierTables t, uint32_t* __restrict__ spec) {
    extern __shared__ float2 buf[];
    const int tid = threadIdx.x, B = blockDim.x;
    const int L = t.L, n = t.n, off = (L - n) / 2, h = L / 2;
    int p, a;
    spectra_work((rows + 1) / 2, t.na, p, a);
    if (2 * p >= rows) return;  // whole work-group
    const int z0 = 2 * p;
    const bool has1 = z0 + 1 < rows;
    const uint16_t* p0 = in.proj + a * in.proj_stride + static_cast<int64_t>(z0) * n;
    const uint16_t* p1 = has1 ? p0 + n : p0;
    const float* d0 = dmean + static_cast<int64_t>(z0) * n;
    const float* e0 = rden + static_cast<int64_t>(z0) * n;
    const float* d1 = has1 ? d0 + n : d0;
    const float* e1 = has1 ? e0 + n : e0;
    // clamping the column onto the detector gives the edge-replicated padding
    for (int m = tid; m < L; m += B) {
        const int c = min(max(m - off, 0), n - 1);
        const float v0 = neglog_counts(static_cast<float>(p0[c]), d0[c], e0[c]);
        const float v1 = has1 ? neglog_counts(static_cast<float>(p1[c]), d1[c], e1[c]) : 0.0f;
        buf[m] = make_float2(v0, v1);
    }
    __syncthreads();
    fft_forward_lds(buf, L, t.log2L, tw);
    const int sl = t.slot[a];
    const bool rev = (sl & 1) != 0;
    uint32_t* row = spectra_row(spec, p, sl >> 1, t);
    if (tid == 0) spectra_zero(row, t);
    for (int m = tid; m < L; m += B) {
        const float2 X = buf[m];
        const int k = m < h ? m : m - L;  // m = L/2 is the -L/2 term
        spectra_store(row, (rev ? -k : k) + h, t, cmul(X, t.E[k + h]));
        if (m == h) spectra_store(row, (rev ? -h : h) + h, t, cmul(X, t.E[L]));  // and its +L/2 copy
    }
}

// ---------------------------------------------------------------------------
// Gather onto the Cartesian frequency grid.
//
// The Gaussian's weights depend on the grid point and the sample only, not on
// the slices, so the sum over the polar samples is a matrix product:
//   grid[point][column] = sum over (angle, sample) W[point][(angle, sample)] spec[(angle, sample)][column],
// a column being the real or imaginary part of a pair.  Each slice's spectrum is
// Hermitian, so the point -u has the weights of u on the mirrored samples: 16
// columns are the two parts of four pairs at sample k and the same at -k.  One
// 16x16x32 instruction adds 4 angles x 8 samples for a 4x4 block of points and
// 16 columns; the weights are formed once for up to 16 pairs.  A block reaches
// 8.1 samples either way of its centre (half_width 6, one grid point per
// sample): three such groups of 8 per angle.
//
// Precision: weights and samples are two FP16 values each (the rounded value
// and what it misses, the samples' kept 2^11 times as large: see split_data) and
// three products are summed, the dropped one below 2^-22 of the whole.  The
// samples' scale is set by the largest row there can be, a line integral of
// 13.8, so those of a faint object lie far down FP16's range; with the second
// value unscaled, and so subnormal, the error was 1.7e-5 at a largest line
// integral of 0.001, now 4.6e-7 as at 1 (100 angles, 160 columns).
// 4 angles at a time are summed from zero and added once, and
// where more than 128 angles meet (tiles around the origin) FP64 totals take
// up the FP32 sums every 64 angles.  The weights are not cut off at the
// truncation radius: every sample that a window holds counts.
//
// Work-group: 32x32 points of a tile (or a 16x16 quarter of one that many
// angles reach) for 4 NT pairs, 16 waves; wave w owns 4 neighbouring blocks (or
// one).  The grid is periodic (M points per side): the host lists, per tile, the
// sorted angles that reach it or an image of it shifted by +-M.  Four angles at
// a time, the samples from 32 before the tile centre's to 31 after (24 and 23)
// go straight from global memory into one of two LDS buffers while the other is
// summed; a wave skips the blocks that none of the four angles reaches.  The
// tile centre's along-ray position and perpendicular offset are formed in FP64
// (integer + FP32 fraction), lanes add only their in-tile offsets, so the
// coordinates keep FP32 precision at any grid size.
//
// Bound: vector work on the weights and their split (7.5 vector instructions per
// matrix product in all, 0.42 a cycle and CU, the matrix cores busy 0.23 of the
// time); waves wait half of their cycles, 16 of them taking a tile's blocks of
// angles (8 at 2048 angles) in step, each waiting for the busiest.  2048 angles, 32
// pairs, 4096^2 grid: 9.5 ms as a gather per grid point and pair, 3.3 ms so; 721
// angles, 5 pairs, 2048^2: 0.57 -> 0.29 ms, the longest chain of blocks around the
// origin.  Tried and not better: wave priorities, all LDS reads of a product group
// ahead of its weights.
// ---------------------------------------------------------------------------
constexpr int kFrWaves = 16;
constexpr int kFrAngles = 4;  // per staged block: one per 16 lanes of an operand
constexpr int kFrChunk = 16;  // blocks whose geometry is formed at a time, one angle per lane

template <int TB> constexpr int fr_slots() { return TB == 32 ? 64 : 48; }
template <int TB, int NT> constexpr int fr_buffer() { return 2 * (kFrAngles / 2) * NT * kSlotBytes * fr_slots<TB>(); }
// Image of a tile of one pair while it is stored: rows and images start in other banks.
template <int TB> constexpr int fr_row() { return 8 * TB + 16; }
template <int TB> constexpr int fr_image() { return TB * fr_row<TB>() + 64; }
template <int NT> constexpr size_t fr_grid_lds() {
    constexpr int stage = 2 * fr_buffer<32, NT>() + 2 * kFrChunk * kFrAngles * 24, store = 2 * kFrPairGroup * fr_image<32>();
    return stage > store ? stage : store;
}

// S1: one grid point per frequency sample (the weights then follow from two
// exponentials per 8 samples); otherwise one exponential per sample.
// NARROW: rows of one pair.  A lane picks its sample alone and pads it with zeros
// (the sums of the other three pairs are never stored).
template <int TB, int NT, bool S1, bool NARROW>
__device__ __forceinline__ void gather_tile(const FourierTables& t, const u4_t* __restrict__ spec, int4 item, int group0,
                                            int pairs, float2* __restrict__ grid, unsigned char* smem) {
    constexpr int BW = TB == 32 ? 4 : 1;                  // blocks per wave
    constexpr bool kWide = TB == 16;                       // FP64 totals, every 16 blocks of angles
    constexpr int WN = fr_slots<TB>(), kBack = WN / 2;
    constexpr int kTile = kSlotBytes * WN, kPair = NT * kTile, kPlane = (kFrAngles / 2) * kPair;
    constexpr int kBuf = fr_buffer<TB, NT>(), kParts = kTile / 1024, kLoads = kBuf / 1024;
    // two chunks of the item's blocks: fraction, offset, cos, sin; frequency of slot 0, angle
    float4* sGeo = reinterpret_cast<float4*>(smem + 2 * fr_buffer<32, NT>());
    int2* sRow = reinterpret_cast<int2*>(sGeo + 2 * kFrChunk * kFrAngles);
    constexpr int kRing = 2 * kFrChunk - 1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = t.M, hM = M / 2, h = t.L / 2;
    const float mid = 0.5f * (TB - 1);

    f4_t acc[BW][NT];
    double wide[kWide ? NT : 1][4];
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int i = 0; i < BW; ++i) acc[i][n][r] = 0.0f;
            if (kWide) wide[n][r] = 0.0;
        }
    // FP64 totals: what has been summed in FP32 since the last time
    auto carry = [&]() {
#pragma unroll
        for (int n = 0; n < (kWide ? NT : 0); ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                wide[n][r] += static_cast<double>(acc[0][n][r]);
                acc[0][n][r] = 0.0f;
            }
    };

    const int nblk = item.w;
    // Geometry of the angles of a chunk of blocks, one per lane of wave 0.
    auto geometry = [&](int chunk) {
        const int b = chunk * kFrChunk + (lane >> 2), j = lane & 3;
        if (b >= nblk) return;
        const int4 blk = t.blocks[item.z + b];
        const bool on = j < blk.y;
        const int a = blk.x + (on ? j : 0);
        const double Cx = static_cast<double>(__int_as_float(blk.z)), Cy = static_cast<double>(__int_as_float(blk.w));
        const double c = t.cbd[a], sn = t.sbd[a];
        const double tc = (Cx * c + Cy * sn) * static_cast<double>(t.inv_s);
        const double kc = floor(tc);
        const int e = (chunk & 1) * kFrChunk * kFrAngles + lane;
        // no angle: an offset that every weight vanishes at, samples off every row
        sGeo[e] = make_float4(static_cast<float>(tc - kc), on ? static_cast<float>(Cy * c - Cx * sn) : 1e9f,
                              static_cast<float>(c), static_cast<float>(sn));
        sRow[e] = make_int2(on ? static_cast<int>(kc) - kBack : 1 << 28, a);
    };
    // Staging: each load of a wave moves 1 KiB of LDS, 16 samples of four pairs
    // (16 bytes of sample k, 16 of sample -k) for two angles: a uniform base
    // (row of the first angle) and a 32-bit offset per lane, 0 off the row's ends.
    const int flip = lane & 1 ? -1 : 0;
    const uint32_t pair_off = (lane & 2 ? 2u * static_cast<uint32_t>(t.SL) : 0u) * 16u + 16u * static_cast<uint32_t>(h + 1);
    const uint32_t lds0 = lds_address(smem);
    const int last_group = (pairs - 1) / kFrPairGroup;
    auto stage = [&](int k) {
        const int2* rows = sRow + (k & kRing) * kFrAngles;
#pragma unroll
        for (int s = 0; s < (kLoads + kFrWaves - 1) / kFrWaves; ++s) {
            const int i = s * kFrWaves + wv;
            if (kLoads % kFrWaves != 0 && i >= kLoads) break;
            const int part = i % kParts, n = i / kParts % NT, pr = i / (kParts * NT) % (kFrAngles / 2),
                      pl = i / (kParts * NT * (kFrAngles / 2));
            const int a = __builtin_amdgcn_readfirstlane(rows[2 * pr].y);
            const int kk = rows[2 * pr + ((lane >> 1) & 1)].x + 16 * part + (lane >> 2);
            const bool in = static_cast<uint32_t>(kk + h) <= static_cast<uint32_t>(2 * h);
            const uint32_t off = static_cast<uint32_t>((kk ^ flip) - flip) * 16u + pair_off;
            // pairs past the last are read from its group again; their sums are never stored
            const int g = min(group0 + n, last_group);
            load_lds16(spec + ((static_cast<int64_t>(g) * t.na + a) * 2 + pl) * t.SL, in ? off : 0u,
                       lds0 + (k & 1) * kBuf + i * 1024);
        }
    };

    // The same of NARROW rows, through registers: loaded before a block is
    // summed, written after it.
    constexpr int kPieces = (kLoads + kFrWaves - 1) / kFrWaves;
    uint32_t sample[NARROW ? kPieces : 1];
    auto take = [&](int k) {
        const int2* rows = sRow + (k & kRing) * kFrAngles;
        const uint32_t* rows32 = reinterpret_cast<const uint32_t*>(spec);
#pragma unroll
        for (int s = 0; s < kPieces; ++s) {
            const int i = s * kFrWaves + wv;
            if (kLoads % kFrWaves != 0 && i >= kLoads) break;
            const int part = i % kParts, pr = i / kParts % (kFrAngles / 2), pl = i / (kParts * (kFrAngles / 2));
            const int2 row = rows[2 * pr + ((lane >> 1) & 1)];
            const int kk = row.x + 16 * part + (lane >> 2);
            sample[s] = 0;
            if (static_cast<uint32_t>(kk + h) <= static_cast<uint32_t>(2 * h))
                sample[s] = rows32[(static_cast<int64_t>(row.y) * 2 + pl) * t.SL + ((kk ^ flip) - flip) + h];
        }
    };
    auto put = [&](int k) {
#pragma unroll
        for (int s = 0; s < kPieces; ++s) {
            const int i = s * kFrWaves + wv;
            if (kLoads % kFrWaves != 0 && i >= kLoads) break;
            *reinterpret_cast<u4_t*>(smem + (k & 1) * kBuf + i * 1024 + 16 * lane) = u4_t{sample[s], 0, 0, 0};
        }
    };

    // points of the wave's blocks: operand row m = lane % 16 is point (m / 4, m % 4) of a block
    const int px = (lane >> 2) & 3, py = lane & 3, ag = lane >> 4;
    // block i of the wave starts at (bx + 16 (i / 2), by + 16 (i % 2)): any strip
    // of a ray's width meets about half the blocks of every wave
    const int bx = 4 * (wv >> 2), by = TB == 32 ? 4 * ((wv + (wv >> 2)) & 3) : 4 * (wv & 3);
    const float dx = static_cast<float>(bx + px) - mid, dy = static_cast<float>(by + py) - mid;
    const float cx = uniform(static_cast<float>(bx) + 1.5f - mid), cy = uniform(static_cast<float>(by) + 1.5f - mid);
    const float half = uniform(4.0f * static_cast<float>(t.units)), reach = uniform(t.msp + 2.1313f);
    const float kap = t.kappa, kap2 = uniform(2.0f * kap), s1 = t.s, step = uniform(8.0f * s1);
    // the transposing read takes slot (lane / 4) % 4 of 4 from this lane's address
    const uint32_t lane_buf = lds0 + (ag >> 1) * kPair + (ag & 1) * 32 + 8 * (lane & 3) +
                                    kSlotBytes * (kBack + ((lane >> 2) & 3));

    if (wv == 0) geometry(0);
    __syncthreads();
    if (nblk > 0) {
        if constexpr (NARROW) {
            take(0);
            put(0);
        } else {
            stage(0);
        }
    }
    wait_loads();
    __syncthreads();
    for (int k = 0; k < nblk; ++k) {
        // the geometry first: the loads into LDS that follow complete in order,
        // and nothing before the end of the block waits for them
        if (wv == 0 && k % kFrChunk == 0) geometry(k / kFrChunk + 1);
        if (k + 1 < nblk) {
            if constexpr (NARROW) take(k + 1);
            else stage(k + 1);
        }
        const float4 ge = sGeo[(k & kRing) * kFrAngles + ag];
        const float cb = ge.z, sb = ge.w;
        // block 0 of the wave: its centre's offset from the ray and position on
        // it, and the same for this lane's point
        const float oc = ge.y + cy * cb - cx * sb;
        const float tc = __builtin_fmaf(__builtin_fmaf(cx, cb, cy * sb), t.inv_s, ge.x);
        const float op = ge.y + dy * cb - dx * sb;
        const float tp = __builtin_fmaf(__builtin_fmaf(dx, cb, dy * sb), t.inv_s, ge.x);
#pragma unroll
        for (int i = 0; i < BW; ++i) {
            const float ex = 16.0f * (i >> 1), ey = 16.0f * (i & 1);
            const float across = ey * cb - ex * sb, along = __builtin_fmaf(ex, cb, ey * sb);
            // does any of the four rays pass within the radius of a point of the block?
            if (!__any(fabsf(oc + across) <= reach)) continue;
            const int st = coord_floor(__builtin_fmaf(along, t.inv_s, tc) - half);  // first sample of the window, from the centre's
            const float tr = __builtin_fmaf(along, t.inv_s, tp), dp = op + across;
            const float q0 = (tr - static_cast<float>(st)) * s1;        // distance to the first sample, grid points
            const float e0 = -kap * dp * dp;
            uint32_t rowp = opaque(lane_buf + (k & 1) * kBuf + kSlotBytes * st);
            f4_t sum[NT];
            // 8 samples from distance q: weights in two FP16 values, then NT products of three
            auto unit = [&](auto first, float q, uint32_t src) {
                float w[8];
                if constexpr (S1) {
                    // the recurrence starts anew every 8 samples.  kappa is 3.2 /
                    // half_width: a start underflows from 6.26 sqrt(half_width) grid
                    // points away, so its samples, at most 7 nearer, weigh at most
                    // 2^-15.9 at half_width 3, 2^-24.5 at 4 and 2^-31 above, all
                    // beyond the radius (that setting's own error is 2^-9.5, 2^-12.7,
                    // 2^-15.9 and less)
                    float v = __builtin_amdgcn_exp2f(__builtin_fmaf(-kap * q, q, e0));
                    float ratio = __builtin_amdgcn_exp2f(__builtin_fmaf(kap2, q, -kap));
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        w[j] = v;
                        v *= ratio;
                        ratio *= t.ratio2;
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const float qj = __builtin_fmaf(-static_cast<float>(j), s1, q);
                        w[j] = __builtin_amdgcn_exp2f(__builtin_fmaf(-kap * qj, qj, e0));
                    }
                }
                u4_t hi, lo, hiy;  // hiy: the first values for the samples' second ones
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    uint32_t a, b;
                    split_pair(w[2 * j], w[2 * j + 1], a, b);
                    hi[j] = a;
                    lo[j] = b;
                    hiy[j] = low_weights(a);
                }
#pragma unroll
                for (int n = 0; n < NT; ++n) {
                    const u4_t x = read_slots(src + n * kTile), y = read_slots(src + n * kTile + kPlane);
                    if constexpr (first.value) sum[n] = f4_t{0.0f, 0.0f, 0.0f, 0.0f};
                    sum[n] = mfma16(lo, x, sum[n]);  // smallest products first
                    sum[n] = mfma16(hiy, y, sum[n]);
                    sum[n] = mfma16(hi, x, sum[n]);
                }
            };
            unit(std::true_type{}, q0, rowp);
            float q = q0;
#pragma unroll 1
            for (int u = 1; u < t.units; ++u) {
                q -= step;
                rowp = opaque(rowp + 8 * kSlotBytes);
                unit(std::false_type{}, q, rowp);
            }
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][n][r] += sum[n][r];
        }
        if (kWide && k % 16 == 15) carry();
        if (NARROW && k + 1 < nblk) put(k + 1);
        wait_loads();  // this wave's part of block k + 1 is in LDS
        __syncthreads();
    }

    // Result: lane l holds column l % 16 (part l & 1 of pair (l / 2) % 4, mirrored
    // for l & 8) of points (l / 16, 0 .. 3) of each block.  Neighbouring lanes
    // exchange parts (the even one keeps points 0 and 1, the odd one 2 and 3), and
    // the four pairs of a group go through LDS to be stored a tile row at a time.
    // A mirrored row is kept from its end, in the order of its addresses.
    carry();
    constexpr int kRow = fr_row<TB>(), kImage = fr_image<TB>();
    const bool odd = lane & 1, mirror = lane & 8;
    const bool nyq = item.y == -hM;  // this tile row only supplies the grid row uy = -M/2, which no mirror reaches
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        if ((group0 + n) * kFrPairGroup >= pairs) break;
        if (n > 0) __syncthreads();
#pragma unroll
        for (int i = 0; i < BW; ++i) {
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = kWide ? static_cast<float>(wide[kWide ? n : 0][r]) : acc[i][n][r];
            const float x0 = __shfl_xor(odd ? v[0] : v[2], 1), x1 = __shfl_xor(odd ? v[1] : v[3], 1);
            const float2 c0 = odd ? make_float2(x0, v[2]) : make_float2(v[0], x0);
            const float2 c1 = odd ? make_float2(x1, v[3]) : make_float2(v[1], x1);
            const int y = by + 16 * (i & 1) + (odd ? 2 : 0);  // even
            unsigned char* row = smem + (((lane >> 1) & 3) + (mirror ? 4 : 0)) * kImage + (bx + 16 * (i >> 1) + ag) * kRow;
            *reinterpret_cast<float4*>(row + 8 * (mirror ? TB - 2 - y : y)) =
                mirror ? make_float4(c1.x, c1.y, c0.x, c0.y) : make_float4(c0.x, c0.y, c1.x, c1.y);
        }
        __syncthreads();
        constexpr int kPer = TB / 2;  // threads per row of TB points
#pragma unroll
        for (int q = tid; q < 8 * TB * kPer; q += 64 * kFrWaves) {
            const int y = 2 * (q % kPer), x = q / kPer % TB, img = q / (kPer * TB);
            const int p = (group0 + n) * kFrPairGroup + (img & 3);
            if (p >= pairs) continue;
            const float4 v = *reinterpret_cast<const float4*>(smem + img * kImage + x * kRow + 8 * y);
            const int ux = item.x + x;
            float2* plane = grid + static_cast<int64_t>(p) * M * M;
            if (img < 4) {
                float2* g = plane + static_cast<int64_t>(ux & (M - 1)) * M + ((item.y + y) & (M - 1));
                if (!nyq) *reinterpret_cast<float4*>(g) = v;
                else if (item.y + y == -hM) *g = make_float2(v.x, v.y);
            } else if (!nyq) {
                // points uy = item.y + TB - 1 - y and the one below it, mirrored
                const int uy = -(item.y + TB - 1 - y);
                float2* g = plane + static_cast<int64_t>((-ux) & (M - 1)) * M;
                g[uy & (M - 1)] = make_float2(v.x, v.y);
                if (uy + 1 < 0) g[(uy + 1) & (M - 1)] = make_float2(v.z, v.w);  // the row uy = 0 is its own mirror
            }
        }
    }
}

template <int NT, bool S1, bool NARROW>
__global__ void __launch_bounds__(64 * kFrWaves)
k_fr_grid(FourierTables t, const u4_t* __restrict__ spec, int pairs, int groups, float2* __restrict__ grid) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int it = blockIdx.x / groups, group0 = (blockIdx.x - it * groups) * NT;
    const int4 item = t.items[it];
    if (it < t.n_small)
        gather_tile<16, NT, S1, NARROW>(t, spec, item, group0, pairs, grid, smem);
    else
        gather_tile<32, NT, S1, NARROW>(t, spec, item, group0, pairs, grid, smem);
}

// ---------------------------------------------------------------------------
// Inverse FFT along the grid's fast axis (frequency uy -> image y) for one
// (pair, ux) row; the inverse transform is conj(FFT(conj(.))).  Outputs
// y = iy - N/2 for iy in [0, N) go to cols[p][iy / 16][ux][iy % 16], so the
// column pass reads 16 neighbouring image rows from one 128-byte line.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(1024)
k_fr_rows(const float2* __restrict__ grid, const float2* __restrict__ tw, FourierTables t,
          float2* __restrict__ cols) {
    extern __shared__ float2 buf[];
    const int tid = threadIdx.x, B = blockDim.x;
    const int M = t.M, N = t.N, hN = N / 2;
    const int64_t rid = blockIdx.x;
    const int p = static_cast<int>(rid / M);
    const int ux = static_cast<int>(rid - static_cast<int64_t>(p) * M);
    const float2* g = grid + rid * M;
    for (int m = tid; m < M; m += B) buf[m] = cconj(g[m]);
    __syncthreads();
    fft_forward_lds(buf, M, t.log2M, tw);
    const int ng = (N + 15) / 16;
    float2* cp = cols + static_cast<int64_t>(p) * ng * M * 16;
    for (int m = tid; m < M; m += B) {
        const int y = m < M / 2 ? m : m - M;
        const int iy = y + hN;
        if (iy >= 0 && iy < N) cp[(static_cast<int64_t>(iy >> 4) * M + ux) * 16 + (iy & 15)] = cconj(buf[m]);
    }
}

// ---------------------------------------------------------------------------
// Inverse FFT along ux for one (pair, image row iy), deconvolution by the
// Gaussian's transform, and the split into the pair's two slices.  The 16
// work-groups of one column group run back to back on one XCD (work-groups
// are dealt to the 8 XCDs in turn), so their shared 128-byte lines are read
// from that XCD's L2.
// ---------------------------------------------------------------------------
template <typename OutT>
__global__ void __launch_bounds__(1024)
k_fr_cols(const float2* __restrict__ cols, const float2* __restrict__ tw, FourierTables t, int pairs, int rows,
          OutT* __restrict__ vol) {
    extern __shared__ float2 buf[];
    const int tid = threadIdx.x, B = blockDim.x;
    const int M = t.M, N = t.N, hN = N / 2;
    const int ng = (N + 15) / 16;
    const int b = blockIdx.x;
    const int xcd = b & 7, r = b >> 3;
    const int gidx = (r >> 4) * 8 + xcd;
    const int p = gidx / ng, gi = gidx - p * ng;
    const int iy = gi * 16 + (r & 15);
    if (p >= pairs || iy >= N) return;  // whole work-group
    const float2* src = cols + (static_cast<int64_t>(p) * ng + gi) * M * 16 + (iy & 15);
    for (int m = tid; m < M; m += B) buf[m] = cconj(src[static_cast<int64_t>(m) * 16]);
    __syncthreads();
    fft_forward_lds(buf, M, t.log2M, tw);
    const float fy = t.D[iy];
    const int z0 = 2 * p;
    const bool has1 = z0 + 1 < rows;
    OutT* o0 = vol + (static_cast<int64_t>(z0) * N + iy) * N;
    OutT* o1 = o0 + static_cast<int64_t>(N) * N;
    for (int m = tid; m < M; m += B) {
        const int x = m < M / 2 ? m : m - M;
        const int ix = x + hN;
        if (ix >= 0 && ix < N) {
            const float2 v = buf[m];  // conj of the inverse transform: (re, -im)
            const float f = t.D[ix] * fy;
            fr_store(o0, ix, v.x * f);  // FP16 slices: the FP32 value rounded once
            if (has1) fr_store(o1, ix, (0.0f - v.y) * f);
        }
    }
}

// ---------------------------------------------------------------------------
// Register-resident variants of the three transform kernels for lengths
// 1024..8192: thread t holds elements t + B s (B = length / 16) and the
// radix-16 passes exchange only their outputs through LDS; after the last
// pass slot s holds output index t + B s in natural order.
// ---------------------------------------------------------------------------
// A work-group takes `run` angles (run_length): each angle's raw counts are
// prefetched while the previous angle is transformed.
template <int L>
__global__ void __launch_bounds__(L / kRegPts)
k_fr_spectra_reg(RawInput in, int rows, const float* __restrict__ dmean, const float* __restrict__ rden,
                 const float2* __restrict__ tw, FourierTables t, int run, uint32_t* __restrict__ spec) {
    extern __shared__ float2 lds[];
    constexpr int B = L / kRegPts, h = L / 2;
    const int n = t.n, off = (L - n) / 2;
    int p, a0;
    spectra_work((rows + 1) / 2, (t.na + run - 1) / run, p, a0);
    if (2 * p >= rows) return;  // whole work-group
    a0 *= run;
    const int a1 = min(t.na, a0 + run);
    const int z0 = 2 * p;
    const bool has1 = z0 + 1 < rows;
    const int64_t r0 = static_cast<int64_t>(z0) * n;
    const int64_t r1 = has1 ? r0 + n : r0;
    // slot s holds padded position t + B s; the column clamped onto the
    // detector gives the edge-replicated padding
    auto load_raw = [&](int a, int tid, uint32_t (&raw)[kRegPts]) {
        const uint16_t* q0 = in.proj + a * in.proj_stride + r0;
        const uint16_t* q1 = in.proj + a * in.proj_stride + r1;
#pragma unroll
        for (int s = 0; s < kRegPts; ++s) {
            const int c = min(max(tid + B * s - off, 0), n - 1);
            raw[s] = static_cast<uint32_t>(q0[c]) | (static_cast<uint32_t>(q1[c]) << 16);
        }
    };
    uint32_t cur[kRegPts], nxt[kRegPts];
    load_raw(a0, threadIdx.x, cur);
#pragma unroll 1
    for (int a = a0; a < a1; ++a) {
        // an opaque thread index per angle keeps per-thread offsets from being
        // hoisted into registers held across the loop
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        if (a + 1 < a1) load_raw(a + 1, tid, nxt);
        float2 x[kRegPts];
#pragma unroll
        for (int s = 0; s < kRegPts; ++s) {
            const int c = min(max(tid + B * s - off, 0), n - 1);
            x[s] = make_float2(neglog_counts(static_cast<float>(cur[s] & 0xffffu), dmean[r0 + c], rden[r0 + c]),
                               has1 ? neglog_counts(static_cast<float>(cur[s] >> 16), dmean[r1 + c], rden[r1 + c])
                                    : 0.0f);
        }
        reg_fft<L>(x, lds, tw, tid);
        const int sl = t.slot[a];
        const bool rev = (sl & 1) != 0;
        uint32_t* row = spectra_row(spec, p, sl >> 1, t);
        if (tid == 0) spectra_zero(row, t);
#pragma unroll
        for (int s = 0; s < kRegPts; ++s) {
            const int m = tid + B * s;
            const int k = m < h ? m : m - L;
            spectra_store(row, (rev ? -k : k) + h, t, cmul(x[s], t.E[k + h]));
            if (m == h) spectra_store(row, (rev ? -h : h) + h, t, cmul(x[s], t.E[L]));
        }
#pragma unroll
        for (int s = 0; s < kRegPts; ++s) cur[s] = nxt[s];
    }
}

template <int M>
__global__ void __launch_bounds__(M / kRegPts)
k_fr_rows_reg(const float2* __restrict__ grid, const float2* __restrict__ tw, FourierTables t,
              float2* __restrict__ cols) {
    extern __shared__ float2 lds[];
    constexpr int B = M / kRegPts;
    const int tid = threadIdx.x;
    const int N = t.N, hN = N / 2;
    const int64_t rid = blockIdx.x;
    const int p = static_cast<int>(rid / M);
    const int ux = static_cast<int>(rid - static_cast<int64_t>(p) * M);
    const float2* g = grid + rid * M;
    float2 x[kRegPts];
#pragma unroll
    for (int s = 0; s < kRegPts; ++s) x[s] = cconj(g[tid + B * s]);
    reg_fft<M>(x, lds, tw, tid);
    const int ng = (N + 15) / 16;
    float2* cp = cols + static_cast<int64_t>(p) * ng * M * 16;
#pragma unroll
    for (int s = 0; s < kRegPts; ++s) {
        const int m = tid + B * s;
        const int y = m < M / 2 ? m : m - M;
        const int iy = y + hN;
        if (iy >= 0 && iy < N) cp[(static_cast<int64_t>(iy >> 4) * M + ux) * 16 + (iy & 15)] = cconj(x[s]);
    }
}

template <int M, typename OutT>
__global__ void __launch_bounds__(M / kRegPts)
k_fr_cols_reg(const float2* __restrict__ cols, const float2* __restrict__ tw, FourierTables t, int pairs, int rows,
              OutT* __restrict__ vol) {
    // two neighbouring image rows (iy, iy + 1) per work-group: 16-byte loads
    extern __shared__ float2 lds[];
    constexpr int B = M / kRegPts;
    const int tid = threadIdx.x;
    const int N = t.N, hN = N / 2;
    const int ng = (N + 15) / 16;
    const int b = blockIdx.x;
    const int xcd = b & 7, r = b >> 3;
    const int gidx = (r >> 3) * 8 + xcd;
    const int p = gidx / ng, gi = gidx - p * ng;
    const int iy = gi * 16 + 2 * (r & 7);
    if (p >= pairs || iy >= N) return;  // whole work-group
    const float4* src = reinterpret_cast<const float4*>(cols + (static_cast<int64_t>(p) * ng + gi) * M * 16 + (iy & 15));
    float2 x[kRegPts], y[kRegPts];
#pragma unroll
    for (int s = 0; s < kRegPts; ++s) {
        const float4 v = src[static_cast<int64_t>(tid + B * s) * 8];
        x[s] = make_float2(v.x, 0.0f - v.y);
        y[s] = make_float2(v.z, 0.0f - v.w);
    }
    const int z0 = 2 * p;
    const bool has1 = z0 + 1 < rows;
    OutT* o0 = vol + (static_cast<int64_t>(z0) * N + iy) * N;
    OutT* o1 = o0 + static_cast<int64_t>(N) * N;
    // each row is transformed and stored before the next one is transformed
    auto finish = [&](float2 (&v)[kRegPts], int row) {
        reg_fft<M>(v, lds, tw, tid);
        const float fy = t.D[iy + row];
#pragma unroll
        for (int s = 0; s < kRegPts; ++s) {
            const int m = tid + B * s;
            const int x0 = m < M / 2 ? m : m - M;
            const int ix = x0 + hN;
            if (ix >= 0 && ix < N) {
                const float f = t.D[ix] * fy;
                fr_store(o0, row * N + ix, v[s].x * f);
                if (has1) fr_store(o1, row * N + ix, (0.0f - v[s].y) * f);
            }
        }
    };
    finish(x, 0);
    if (iy + 1 < N) finish(y, 1);
}

size_t reg_lds(int L) { return static_cast<size_t>(L + L / 16) * sizeof(float2); }

template <int NT, bool S1, bool NARROW>
hipError_t launch_grid_t(const FourierTables& t, const uint32_t* spec, int pairs, float2* grid, hipStream_t st) {
    constexpr size_t lds = fr_grid_lds<NT>();
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    hipError_t e = fr_lds(k_fr_grid<NT, S1, NARROW>, lds);
    if (e != hipSuccess) return e;
    const int groups = (pairs + kFrPairGroup * NT - 1) / (kFrPairGroup * NT);
    const dim3 g(static_cast<unsigned>(static_cast<int64_t>(t.n_items) * groups));
    hipLaunchKernelGGL((k_fr_grid<NT, S1, NARROW>), g, dim3(64 * kFrWaves), lds, st, t, reinterpret_cast<const u4_t*>(spec), pairs,
                       groups, grid);
    return hipGetLastError();
}

template <int NT, bool NARROW = false>
hipError_t launch_grid_nt(const FourierTables& t, const uint32_t* spec, int pairs, float2* grid, hipStream_t st) {
    return t.s == 1.0f ? launch_grid_t<NT, true, NARROW>(t, spec, pairs, grid, st)
                       : launch_grid_t<NT, false, NARROW>(t, spec, pairs, grid, st);
}

}  // namespace

hipError_t launch_fourier_spectra(const RawInput& in, int rows, const float* dmean, const float* rden,
                                  const float2* tw_L, const FourierTables& t, uint32_t* spec, hipStream_t st) {
    const int pairs = (rows + 1) / 2;
    const int run = run_length(pairs, t.na);
#define TP_FR_REG(LL)                                                                                      \
    case LL: {                                                                                            \
        const dim3 g(spectra_grid(pairs, (t.na + run - 1) / run));                                        \
        const hipError_t e = fr_lds(k_fr_spectra_reg<LL>, reg_lds(LL));                                   \
        if (e != hipSuccess) return e;                                                                    \
        hipLaunchKernelGGL((k_fr_spectra_reg<LL>), g, dim3(LL / kRegPts), reg_lds(LL), st, in, rows, dmean, rden, \
                           tw_L, t, run, spec);                                                          \
        return hipGetLastError();                                                                         \
    }
    switch (t.L) {
        TP_FR_REG(1024)
        TP_FR_REG(2048)
        TP_FR_REG(4096)
        TP_FR_REG(8192)
        default: break;
    }
#undef TP_FR_REG
    const size_t lds = static_cast<size_t>(t.L) * sizeof(float2);
    hipError_t e = fr_lds(k_fr_spectra, lds);
    if (e != hipSuccess) return e;
    const dim3 grid(spectra_grid(pairs, t.na));
    hipLaunchKernelGGL(k_fr_spectra, grid, dim3(fr_block(t.L)), lds, st, in, rows, dmean, rden, tw_L, t, spec);
    return hipGetLastError();
}

// As many pairs per work-group as there are, up to 16: they share the weights.
hipError_t launch_fourier_grid(const FourierTables& t, const uint32_t* spec, int pairs, float2* grid, hipStream_t st) {
    if (t.wide == 1) return launch_grid_nt<1, true>(t, spec, pairs, grid, st);
    if (pairs > 2 * kFrPairGroup) return launch_grid_nt<4>(t, spec, pairs, grid, st);
    return pairs > kFrPairGroup ? launch_grid_nt<2>(t, spec, pairs, grid, st)
                                : launch_grid_nt<1>(t, spec, pairs, grid, st);
}

hipError_t launch_fourier_rows(const FourierTables& t, const float2* tw_M, const float2* grid, int pairs,
                               float2* cols, hipStream_t st) {
#define TP_FR_REG(MM)                                                                                      \
    case MM: {                                                                                            \
        const dim3 g(static_cast<unsigned>(static_cast<int64_t>(pairs) * MM));                            \
        const hipError_t e = fr_lds(k_fr_rows_reg<MM>, reg_lds(MM));                                      \
        if (e != hipSuccess) return e;                                                                    \
        hipLaunchKernelGGL((k_fr_rows_reg<MM>), g, dim3(MM / kRegPts), reg_lds(MM), st, grid, tw_M, t, cols); \
        return hipGetLastError();                                                                         \
    }
    switch (t.M) {
        TP_FR_REG(1024)
        TP_FR_REG(2048)
        TP_FR_REG(4096)
        TP_FR_REG(8192)
        default: break;
    }
#undef TP_FR_REG
    const size_t lds = static_cast<size_t>(t.M) * sizeof(float2);
    hipError_t e = fr_lds(k_fr_rows, lds);
    if (e != hipSuccess) return e;
    const dim3 g(static_cast<unsigned>(static_cast<int64_t>(pairs) * t.M));
    hipLaunchKernelGGL(k_fr_rows, g, dim3(fr_block(t.M)), lds, st, grid, tw_M, t, cols);
    return hipGetLastError();
}

namespace {
template <typename OutT>
hipError_t launch_fourier_cols_t(const FourierTables& t, const float2* tw_M, const float2* cols, int pairs, int rows,
                                 OutT* vol, hipStream_t st) {
    const int64_t groups = static_cast<int64_t>(pairs) * ((t.N + 15) / 16);
    const dim3 g(static_cast<unsigned>(((groups + 7) / 8) * 8 * 16));
    const dim3 g2(static_cast<unsigned>(((groups + 7) / 8) * 8 * 8));  // two rows per work-group
#define TP_FR_REG(MM)                                                                                      \
    case MM: {                                                                                            \
        const hipError_t e = fr_lds(k_fr_cols_reg<MM, OutT>, reg_lds(MM));                                \
        if (e != hipSuccess) return e;                                                                    \
        hipLaunchKernelGGL((k_fr_cols_reg<MM, OutT>), g2, dim3(MM / kRegPts), reg_lds(MM), st, cols, tw_M, t, pairs, \
                           rows, vol);                                                                    \
        return hipGetLastError();                                                                         \
    }
    switch (t.M) {
        TP_FR_REG(1024)
        TP_FR_REG(2048)
        TP_FR_REG(4096)
        TP_FR_REG(8192)
        default: break;
    }
#undef TP_FR_REG
    const size_t lds = static_cast<size_t>(t.M) * sizeof(float2);
    hipError_t e = fr_lds(k_fr_cols<OutT>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_fr_cols<OutT>, g, dim3(fr_block(t.M)), lds, st, cols, tw_M, t, pairs, rows, vol);
    return hipGetLastError();
}
}  // namespace

// vol: FP32 slices, or FP16 (`half_out`: each voxel's FP32 value rounded once).
hipError_t launch_fourier_cols(const FourierTables& t, const float2* tw_M, const float2* cols, int pairs, int rows,
                               void* vol, bool half_out, hipStream_t st) {
    if (half_out) return launch_fourier_cols_t(t, tw_M, cols, pairs, rows, static_cast<__half*>(vol), st);
    return launch_fourier_cols_t(t, tw_M, cols, pairs, rows, static_cast<float*>(vol), st);
}

}  // namespace tp
