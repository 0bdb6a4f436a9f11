// Kernels of the learned CGLS warm start: a small 3D U-Net with 3x3x3
// convolutions, BF16 activations and weights, FP32 accumulation.
//
// Layout: channels last, [D][H][W][C] BF16, with an explicit channel stride
// (so a tensor can be a channel slice of a wider one: concatenation costs
// nothing) and channel counts that are multiples of 8.
//
// conv3d (forward and backward-data) is an implicit GEMM on the MFMA unit:
//   out[v][co] = sum_k A[v][k] B[k][co],  k = tap * Cin + ci,  27 taps,
// with v_mfma_f32_16x16x32_bf16.  Lane l of a wave holds, for the 16x32 A
// tile, row l%16 and the 8 consecutive k of group l/16 -- 8 consecutive input
// channels of one tap, i.e. one 16-byte load in channels-last layout; the B
// tile likewise holds 8 consecutive input channels of one output channel
// (weights stored [tap][co][ci]).  The 16x16 FP32 result has row 4*(l/16)+e,
// column l%16 in element e of lane l.
// conv3d backward-weight reduces over voxels: D[co][ci] = sum_v dY[v][co] X[v+off][ci],
// with dY and X staged in LDS as they lie in memory and the voxels of a lane
// gathered by the transposing LDS read.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

namespace cvpnn {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

struct Act {             // a channels-last BF16 tensor (or channel slice)
    __bf16 *p;
    int D, H, W;
    int C;               // channels used
    int stride;          // channels between consecutive voxels (>= C)
};

__device__ __forceinline__ bf16x8 zero8()
{
    bf16x8 z;
#pragma unroll
    for (int e = 0; e < 8; ++e) z[e] = (__bf16)0.0f;
    return z;
}

// ------------------------------------------------------------------ conv3d

// One wave computes 64 consecutive voxels of one (d, h) row (4 row tiles of
// 16) for all output channels (CO/16 column tiles).  Weights wt: [27][Co][Ci].
// flip = 1 mirrors the taps (used by backward-data with the transposed
// weights).  relu = 1 applies max(., 0) before the BF16 store.
template <int CO>
__global__ void __launch_bounds__(256)
conv3d_kernel(const Act in, const __bf16 *__restrict__ wt, const float *__restrict__ bias,
              Act out, int relu, int flip)
{
    constexpr int NT = CO / 16;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int segs = (in.W + 63) / 64;
    const int row = blockIdx.x * 4 + wave;           // (d, h, segment)
    if (row >= in.D * in.H * segs) return;
    const int seg = row % segs;
    const int dh = row / segs;
    const int d = dh / in.H, h = dh % in.H;
    const int w0 = seg * 64;
    const int Ci = in.C;
    const int K = 27 * Ci;
    const int ksteps = (K + 31) / 32;

    f32x4 acc[4][NT];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[r][n] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int i16 = lane & 15;
    const int kg = lane >> 4;        // which group of 8 k within the 32
    for (int ks = 0; ks < ksteps; ++ks) {
        const int k = ks * 32 + kg * 8;
        const int tap = k / Ci;
        const int ci = k - tap * Ci;
        const bool tv = tap < 27;
        const int tp = flip ? 26 - tap : tap;
        const int dz = tp / 9 - 1, dy = (tp / 3) % 3 - 1, dx = tp % 3 - 1;
        const int z = d + dz, y = h + dy;
        const bool zy = tv && z >= 0 && z < in.D && y >= 0 && y < in.H;
        bf16x8 a[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int x = w0 + r * 16 + i16 + dx;
            if (zy && x >= 0 && x < in.W)
                a[r] = *reinterpret_cast<const bf16x8 *>(in.p + (((size_t)z * in.H + y) * in.W + x) * in.stride + ci);
            else
                a[r] = zero8();
        }
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            const int co = n * 16 + i16;
            bf16x8 b = tv ? *reinterpret_cast<const bf16x8 *>(wt + ((size_t)tap * CO + co) * Ci + ci) : zero8();
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[r], b, acc[r][n], 0, 0, 0);
        }
    }
    // epilogue: lane holds rows 4*(l/16)+e, column l%16 of each tile
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const int co = n * 16 + i16;
        const float bv = bias ? bias[co] : 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int x = w0 + r * 16 + (lane >> 4) * 4 + e;
                if (x < out.W) {
                    float v = acc[r][n][e] + bv;
                    if (relu) v = fmaxf(v, 0.0f);
                    out.p[(((size_t)d * out.H + h) * out.W + x) * out.stride + co] = (__bf16)v;
                }
            }
        }
    }
}

// The same convolution for 16, 32 or 64 input channels and volumes whose
// element count fits 32 bits.  A workgroup marches tiles of up to 8 x 32
// voxels along d: the LDS holds three slices of the input with their halo
// (zeros outside the volume), each step loads one new slice while the last is
// computed, and the weights of 16 NT output channels stay in a wave's
// registers for the whole march, so the inner loop is LDS reads at constant
// offsets and MFMAs.  A wave computes two rows (four tiles of 16 voxels) at a
// time; with more than 16 NT output channels the waves split the channels and
// then the rows.  The weights are the first MFMA operand, which puts four
// consecutive output channels of a voxel in a lane: one 8-byte store.  MASK:
// the result becomes 0 where `keep` (a post-ReLU output) is not positive.  The
// k order and the MFMA sequence of an element are those of conv3d_kernel: the
// results are the same bits.  The LDS bandwidth (one fragment per NT MFMAs)
// bounds the inner loop with 64 input channels, with 16 output channels memory
// nearly does: 16 -> 16, 32 -> 16 at 128^3, 64 -> 32 at 64^3 and 64 -> 64 at
// 32^3 take 43, 71, 44 and 19 us; with a workgroup per tile of 4 x 64 voxels,
// all three slices staged by each and the weights fetched at each k step, 85,
// 184, 141 and 35 us.  (Sharing the fragments between four output rows halves
// the LDS reads, but the shorter chains of independent MFMAs and the registers
// cost more: 66, 51 and 20 us for the last three.)
constexpr int kMarchRows = 8, kMarchX = 34;
constexpr unsigned kOutside = 0xFFFFFF00u;      // beyond a buffer of at most kMarchElems elements, 255 bytes further too
constexpr int64_t kMarchElems = (int64_t(1) << 31) - 256;

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

template <int CI>
constexpr int march_lds_bytes() { return 3 * (kMarchRows + 2) * kMarchX * CI * 2; }

struct MarchPlan {
    int units;           // tile columns x runs of slices
    int run;             // slices per unit
    int rows;            // rows per tile: 2, 4 or 8
    int ytiles, segs;    // tiles along y and x
};

template <int CO, int CI, int NT, bool FLIP, bool MASK>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CI * NT == 16 ? 3 : CI * NT == 32 ? 2 : 1)))
conv3d_march_kernel(const Act in, const __bf16 *__restrict__ wt, const float *__restrict__ bias, const Act out,
                    const Act keep, int relu, const MarchPlan P)
{
    constexpr int KSTEPS = (27 * CI + 31) / 32;
    constexpr int WN = CO / (16 * NT), WR = 4 / WN;        // waves over channels and over rows
    constexpr int C8 = CI / 8;
    constexpr int XV = (kMarchRows + 2) * kMarchX;         // voxels of a staged slice
    constexpr int SLICE = XV * CI * 2;
    constexpr int NX = (XV * C8 + 255) / 256;
    extern __shared__ __align__(16) unsigned char tile[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i16 = lane & 15, kg = lane >> 4;
    const int cow = wave % WN * NT * 16;                   // first output channel of this wave

    // weights of k step ks: k = 32 ks + 8 kg .. + 7 of channel cow + 16 n + i16
    bf16x8 w[KSTEPS][NT];
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
        const int k = ks * 32 + kg * 8, tap = k / CI, ci = k % CI;
#pragma unroll
        for (int n = 0; n < NT; ++n)
            w[ks][n] = tap < 27 ? *reinterpret_cast<const bf16x8 *>(wt + (tap * CO + cow + 16 * n + i16) * CI + ci) : zero8();
    }
    f32x4 bv[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int e = 0; e < 4; ++e) bv[n][e] = bias ? bias[cow + 16 * n + 4 * kg + e] : 0.0f;

    // Buffer accesses: an offset outside reads zeros and stores nothing, so
    // the loads and stores need no branches (a branch makes the compiler wait
    // for all of them at once).  The results of a pass are stored when the
    // next begins: the wait for a slice's loads, in order of issue, would
    // otherwise wait for the stores just issued as well.
    const int nvox = in.D * in.H * in.W;
    const __amdgpu_buffer_rsrc_t src_buf =
        __builtin_amdgcn_make_buffer_rsrc(in.p, 0, (unsigned)((nvox - 1) * in.stride + CI) * 2u, 0x00027000);
    const __amdgpu_buffer_rsrc_t dst_buf =
        __builtin_amdgcn_make_buffer_rsrc(out.p, 0, (unsigned)((nvox - 1) * out.stride + CO) * 2u, 0x00027000);
    const __amdgpu_buffer_rsrc_t keep_buf = __builtin_amdgcn_make_buffer_rsrc(
        MASK ? keep.p : out.p, 0, MASK ? (unsigned)((nvox - 1) * keep.stride + CO) * 2u : 0u, 0x00027000);
    u32x2 res[4][NT];
    unsigned res_at[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        res_at[t] = kOutside;
#pragma unroll
        for (int n = 0; n < NT; ++n) res[t][n] = u32x2{0, 0};
    }
    auto flush = [&] {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int n = 0; n < NT; ++n)
                __builtin_amdgcn_raw_buffer_store_b64(res[t][n], dst_buf, res_at[t], n * 32, 0);
    };

    for (int unit = blockIdx.x; unit < P.units; unit += gridDim.x) {
        const int seg = unit % P.segs, ty = unit / P.segs % P.ytiles, run = unit / P.segs / P.ytiles;
        const int w0 = seg * 32, h0 = ty * P.rows;
        const int d0 = run * P.run, d1 = min(d0 + P.run, in.D);
        const int rows = min(P.rows, in.H - h0);

        // a slice: 16-byte slots [8-channel chunk][voxel], so that the 16
        // lanes of a fragment read consecutive slots
        u32x4 px[NX];
        unsigned at[NX];                                   // of the thread's slots in slice 0
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int idx = threadIdx.x + 256 * i;
            const int v = idx / C8, c8 = idx % C8;
            const int r = v / kMarchX, x = w0 - 1 + v % kMarchX, y = h0 - 1 + r;
            const bool ok = r < P.rows + 2 && (unsigned)x < (unsigned)in.W && (unsigned)y < (unsigned)in.H;
            at[i] = ok ? (unsigned)((y * in.W + x) * in.stride + c8 * 8) * 2u : kOutside;
        }
        auto load = [&](int z) {
            const unsigned zo = (unsigned)(z * in.H * in.W) * (unsigned)in.stride * 2u;
#pragma unroll
            for (int i = 0; i < NX; ++i)
                px[i] = __builtin_amdgcn_raw_buffer_load_b128(
                    src_buf, (unsigned)z < (unsigned)in.D && at[i] != kOutside ? at[i] + zo : kOutside, 0, 0);
        };
        auto store = [&](int slot) {
#pragma unroll
            for (int i = 0; i < NX; ++i) {
                const int idx = threadIdx.x + 256 * i;
                if (idx < XV * C8)
                    *reinterpret_cast<u32x4 *>(tile + slot * SLICE + (idx % C8 * XV + idx / C8) * 16) = px[i];
            }
        };

        __syncthreads();                                   // the unit before is done with the tiles
        load(d0 - 1);
        store(0);
        load(d0);
        store(1);
        load(d0 + 1);
        int b = 0;                                         // slot of slice d - 1
        for (int d = d0; d < d1; ++d) {
            __syncthreads();
            store(b == 0 ? 2 : b - 1);
            __syncthreads();
            if (d + 1 < d1) load(d + 2);

            // lane's offsets of the three slices; with 16 input channels two
            // taps share a k step and the offset is that of the lane's tap
            int slot[3];
#pragma unroll
            for (int z = 0; z < 3; ++z) slot[z] = (b + z >= 3 ? b + z - 3 : b + z) * SLICE;
            constexpr int NO = CI == 16 ? KSTEPS : 3;
            int off[NO];
#pragma unroll
            for (int o = 0; o < NO; ++o) {
                if (CI == 16) {
                    const int t0 = FLIP ? 26 - 2 * o : 2 * o, t1 = o == 13 ? t0 : FLIP ? t0 - 1 : t0 + 1;
                    const int o0 = slot[t0 / 9] + (t0 / 3 % 3 * kMarchX + t0 % 3) * 16;
                    const int o1 = slot[t1 / 9] + (t1 / 3 % 3 * kMarchX + t1 % 3) * 16;
                    off[o] = (kg & 2 ? o1 : o0) + ((kg & 1) * XV + i16) * 16;
                } else {
                    off[o] = slot[o] + (kg * XV + i16) * 16;
                }
            }
            for (int r = wave / WN * 2; r < rows; r += 2 * WR) {
                flush();
                u32x2 kept[4][NT];                         // read ahead of the pass
                if constexpr (MASK) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const int x = w0 + t % 2 * 16 + i16, y = h0 + r + t / 2;
                        const unsigned at = x < out.W && r + t / 2 < rows
                                                ? (unsigned)(((d * out.H + y) * out.W + x) * keep.stride + cow + 4 * kg) * 2u
                                                : kOutside;
#pragma unroll
                        for (int n = 0; n < NT; ++n)
                            kept[t][n] = __builtin_amdgcn_raw_buffer_load_b64(keep_buf, at, n * 32, 0);
                    }
                }
                f32x4 acc[4][NT];
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int n = 0; n < NT; ++n) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
                const unsigned char *row = tile + r * kMarchX * 16;
#pragma unroll
                for (int ks = 0; ks < KSTEPS; ++ks) {
                    const unsigned char *src;
                    if (CI == 16) {
                        src = row + off[ks];
                    } else {
                        const int tap = ks * 32 / CI, tp = FLIP ? 26 - tap : tap;
                        src = row + off[tp / 9] + (tp / 3 % 3 * kMarchX + tp % 3) * 16 + ks * 32 % CI / 8 * XV * 16;
                    }
#pragma unroll
                    for (int t = 0; t < 4; ++t) {          // tile t: row t / 2, voxels 16 (t % 2) ..
                        bf16x8 a = *reinterpret_cast<const bf16x8 *>(src + (t / 2 * kMarchX + t % 2 * 16) * 16);
                        if (CI == 16 && ks == KSTEPS - 1 && (kg & 2)) a = zero8();     // no 28th tap
#pragma unroll
                        for (int n = 0; n < NT; ++n)
                            acc[t][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][n], a, acc[t][n], 0, 0, 0);
                    }
                }
                // lane: voxel i16 of the tile, channels 4 kg .. + 3
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int x = w0 + t % 2 * 16 + i16, y = h0 + r + t / 2;
                    res_at[t] = x < out.W && r + t / 2 < rows
                                    ? (unsigned)(((d * out.H + y) * out.W + x) * out.stride + cow + 4 * kg) * 2u
                                    : kOutside;
#pragma unroll
                    for (int n = 0; n < NT; ++n) {
                        bf16x4 o;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            float v = acc[t][n][e] + bv[n][e];
                            if (relu) v = fmaxf(v, 0.0f);
                            o[e] = (__bf16)v;
                        }
                        if constexpr (MASK) {
                            const bf16x4 m = __builtin_bit_cast(bf16x4, kept[t][n]);
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (!((float)m[e] > 0.0f)) o[e] = (__bf16)0.0f;
                        }
                        res[t][n] = __builtin_bit_cast(u32x2, o);
                    }
                }
            }
            b = b == 2 ? 0 : b + 1;
        }
    }
    flush();
}

// Backward-weight partials: part[chunk][tap][co][ci] = sum over the chunk's
// voxels v of dY[v][co] X[v + off(tap)][ci].  A chunk is a set of units, a unit
// a column of tiles of TY x 32 voxels marched along d: the LDS holds three
// slices of X with their halo and one of dY, both as they lie in memory (16
// channels of a voxel are 32 bytes), so every step of the march loads one new
// slice for all 27 taps, and loads it while the taps of the last are summed.
// The contraction runs over voxels, that is across the rows of that layout:
// the transposing LDS read gives each lane 4 consecutive voxels of one
// channel, and with voxels 16 j + 4 g + e in element e of lane group g the 64
// lanes of a read touch 512 consecutive bytes whatever the tap, so a shift by
// a tap is an offset and no bank conflicts arise.  The 27 taps are split over
// the waves (7, 7, 7, 6); 64 output channels are two workgroups.  With `bias`
// a partial sum ends with the CO sums of dY, added as it is staged.
// With 16 output channels an X fragment feeds one MFMA and the LDS bandwidth
// bounds the inner loop; with 64 input channels (one wave per SIMD, 480
// registers) the latency of staging does.  With the reduction 25 us at 16 ->
// 16 channels, 64 x 72 x 88 (134 with 64 rows per workgroup, one (dz, dy) each
// and voxel pairs transposed by hand on the way into the LDS), 58 us at 64 ->
// 32, 48 x 50 x 66 (262).
template <int CI>
constexpr int wgrad_rows() { return CI == 16 ? 8 : CI == 32 ? 4 : 2; }

template <int CO, int CI>
constexpr int wgrad_lds_bytes()
{
    return (3 * (wgrad_rows<CI>() + 2) * 34 * CI + wgrad_rows<CI>() * 32 * (CO < 32 ? CO : 32)) * 2;
}

struct WgradPlan {
    int chunks;          // partial sums, one workgroup each (two for 64 output channels)
    int units;           // tile columns x runs of slices
    int run;             // slices per unit
    int ytiles, segs;    // tiles along y and x
};

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

__device__ __forceinline__ s16x4 read_voxels4(const unsigned char *p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p);
}

__device__ __forceinline__ bf16x8 join(s16x4 lo, s16x4 hi)
{
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// The q-th tap of a wave: two of the nine (dz, dy) with their three dx, and
// one dx of the ninth (the fourth wave repeats one and drops it).
__device__ __forceinline__ int wgrad_tap(int wave, int q)
{
    return q < 6 ? (2 * wave + q / 3) * 3 + q % 3 : 24 + min(wave, 2);
}

template <int CO, int CI>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((CO < 32 ? 1 : 2) * CI / 16 > 4 ? 1 : 2)))
conv3d_wgrad_kernel(const Act x, const Act dy, const WgradPlan P, int bias, float *__restrict__ part)
{
    constexpr int COB = CO < 32 ? CO : 32;         // output channels of this workgroup
    constexpr int MT = COB / 16, NT = CI / 16;
    constexpr int TY = wgrad_rows<CI>(), XW = 34;
    constexpr int TAPS = 7;                        // per wave
    constexpr int XV = (TY + 2) * XW, DV = TY * 32;        // voxels of a staged slice
    constexpr int XT = XV * (CI / 8), DT = DV * (COB / 8); // 16-byte loads of a staged slice
    constexpr int NX = (XT + 255) / 256, ND = (DT + 255) / 256;
    constexpr int SLICE = XV * CI * 2;             // bytes
    extern __shared__ __align__(16) unsigned char tile[];
    unsigned char *const sdy = tile + 3 * SLICE;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int co0 = blockIdx.y * COB;

    f32x4 acc[TAPS][MT][NT];
#pragma unroll
    for (int q = 0; q < TAPS; ++q)
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n) acc[q][m][n] = f32x4{0.f, 0.f, 0.f, 0.f};

    float bsum[8];                                 // channels 8 (thread % (COB / 8)) ..
#pragma unroll
    for (int e = 0; e < 8; ++e) bsum[e] = 0.0f;

    for (int unit = blockIdx.x; unit < P.units; unit += P.chunks) {
        const int seg = unit % P.segs, ty = unit / P.segs % P.ytiles, run = unit / P.segs / P.ytiles;
        const int w0 = seg * 32, h0 = ty * TY;
        const int d0 = run * P.run, d1 = min(d0 + P.run, x.D);
        const int rows = min(TY, x.H - h0);

        bf16x8 px[NX], pd[ND];
        auto load_x = [&](int z) {
#pragma unroll
            for (int i = 0; i < NX; ++i) {
                const int idx = threadIdx.x + 256 * i;
                const int v = idx / (CI / 8), c8 = idx % (CI / 8);
                const int xx = w0 - 1 + v % XW, y = h0 - 1 + v / XW;
                px[i] = zero8();
                if (idx < XT && (unsigned)xx < (unsigned)x.W && (unsigned)y < (unsigned)x.H && (unsigned)z < (unsigned)x.D)
                    px[i] = *reinterpret_cast<const bf16x8 *>(x.p + (((size_t)z * x.H + y) * x.W + xx) * x.stride + c8 * 8);
            }
        };
        auto store_x = [&](int slot) {
#pragma unroll
            for (int i = 0; i < NX; ++i) {
                const int idx = threadIdx.x + 256 * i;
                const int v = idx / (CI / 8), c8 = idx % (CI / 8);
                if (idx < XT)
                    *reinterpret_cast<bf16x8 *>(tile + slot * SLICE + ((c8 / 2) * XV + v) * 32 + (c8 & 1) * 16) = px[i];
            }
        };
        auto load_dy = [&](int d) {
#pragma unroll
            for (int i = 0; i < ND; ++i) {
                const int idx = threadIdx.x + 256 * i;
                const int v = idx / (COB / 8), c8 = idx % (COB / 8);
                const int xx = w0 + v % 32, r = v / 32;
                pd[i] = zero8();
                if (idx < DT && r < rows && xx < dy.W)
                    pd[i] = *reinterpret_cast<const bf16x8 *>(dy.p + (((size_t)d * dy.H + h0 + r) * dy.W + xx) * dy.stride +
                                                              co0 + c8 * 8);
            }
        };
        auto store_dy = [&]() {
#pragma unroll
            for (int i = 0; i < ND; ++i) {
                const int idx = threadIdx.x + 256 * i;
                const int v = idx / (COB / 8), c8 = idx % (COB / 8);
                if (idx < DT) *reinterpret_cast<bf16x8 *>(sdy + ((c8 / 2) * DV + v) * 32 + (c8 & 1) * 16) = pd[i];
#pragma unroll
                for (int e = 0; e < 8; ++e) bsum[e] += (float)pd[i][e];
            }
        };

        // voxels 16 j + 4 g + e past the end of the row: X[v - 1] of the first
        // of them is a voxel of the row and must not meet the zero dY beyond
        // it (an infinite X would give NaN); the other taps read zeros there
        s16x4 keep[2], keep6[2];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                keep[j][e] = 16 * j + 4 * (lane >> 4) + e < x.W - w0 ? -1 : 0;
                keep6[j][e] = wave == 0 ? keep[j][e] : -1;
            }

        // the taps of one slice, whose X slices d - 1, d, d + 1 are in slots
        // b, b + 1, b + 2 (mod 3)
        auto sum = [&](int b) {
            const unsigned char *src[TAPS];
#pragma unroll
            for (int q = 0; q < TAPS; ++q) {
                const int tap = wgrad_tap(wave, q);
                int slot = b + tap / 9;
                slot = slot >= 3 ? slot - 3 : slot;
                src[q] = tile + slot * SLICE + ((tap / 3 % 3) * XW + tap % 3) * 32 + lane * 8;
            }
#pragma unroll 1
            for (int r = 0; r < rows; ++r) {
                bf16x8 a[MT];
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    const unsigned char *p = sdy + (m * DV + r * 32) * 32 + lane * 8;
                    a[m] = join(read_voxels4(p), read_voxels4(p + 512));
                }
#pragma unroll
                for (int q = 0; q < TAPS; ++q)
#pragma unroll
                    for (int n = 0; n < NT; ++n) {
                        const unsigned char *p = src[q] + (n * XV + r * XW) * 32;
                        s16x4 lo = read_voxels4(p), hi = read_voxels4(p + 512);
                        if (q == 0 || q == 3) {
                            lo &= keep[0];
                            hi &= keep[1];
                        } else if (q == 6) {
                            lo &= keep6[0];
                            hi &= keep6[1];
                        }
                        const bf16x8 c = join(lo, hi);
#pragma unroll
                        for (int m = 0; m < MT; ++m)
                            acc[q][m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], c, acc[q][m][n], 0, 0, 0);
                    }
            }
        };

        __syncthreads();                           // the unit before is done with the tiles
        load_x(d0 - 1);
        store_x(0);
        load_x(d0);
        store_x(1);
        load_x(d0 + 1);
        load_dy(d0);
        int b = 0;
        for (int d = d0; d < d1; ++d) {
            __syncthreads();
            store_x(b == 0 ? 2 : b - 1);
            store_dy();
            __syncthreads();
            if (d + 1 < d1) {
                load_x(d + 2);
                load_dy(d + 1);
            }
            sum(b);
            b = b == 2 ? 0 : b + 1;
        }
    }
    const size_t stride = (size_t)27 * CO * CI + (bias ? CO : 0);
    if (bias) {
        __syncthreads();
        float *red = reinterpret_cast<float *>(tile);
#pragma unroll
        for (int e = 0; e < 8; ++e) red[threadIdx.x * 8 + e] = bsum[e];
        __syncthreads();
        if (threadIdx.x < COB) {
            float t = 0.0f;
            for (int k = threadIdx.x / 8; k < 256; k += COB / 8) t += red[k * 8 + threadIdx.x % 8];
            part[blockIdx.x * stride + (size_t)27 * CO * CI + co0 + threadIdx.x] = t;
        }
    }
#pragma unroll
    for (int q = 0; q < TAPS; ++q) {
        if (q == 6 && wave == 3) continue;
        const int tap = wgrad_tap(wave, q);
        float *dst = part + blockIdx.x * stride + (size_t)tap * CO * CI;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    dst[(co0 + m * 16 + (lane >> 4) * 4 + e) * CI + n * 16 + (lane & 15)] = acc[q][m][n][e];
    }
}

// out[i] = sum over chunks of part[chunk][i], i < n.  A block takes 64
// consecutive i; wave w of its 16 sums the chunks c = w, w + 16, ... in order
// and the wave sums are added in a fixed order (deterministic).  The sums from
// index n1 on go to out2.
__global__ void __launch_bounds__(1024) reduce_chunks(const float *__restrict__ part, int chunks, int64_t n,
                                                      float *__restrict__ out, int64_t n1, float *__restrict__ out2)
{
    __shared__ float red[16][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int64_t base = (int64_t)blockIdx.x * 64; base < n; base += (int64_t)gridDim.x * 64) {
        const int64_t i = base + lane;
        float s = 0.0f;
        if (i < n) {
#pragma unroll 8
            for (int c = wave; c < chunks; c += 16) s += part[(size_t)c * n + i];
        }
        red[wave][lane] = s;
        __syncthreads();
        if (wave == 0 && i < n) {
            float t = red[0][lane];
#pragma unroll
            for (int w = 1; w < 16; ++w) t += red[w][lane];
            (i < n1 ? out[i] : out2[i - n1]) = t;
        }
        __syncthreads();
    }
}

// Per-channel sums over voxels (bias gradient), partials per block row chunk.
// Thread t takes channel group t % (C/8) of every (256/(C/8))-th voxel with
// 16-byte loads; the block then adds the per-thread sums of each channel in
// a fixed order.
__global__ void channel_sum_partials(const Act a, int rows_per_chunk, float *__restrict__ part)
{
    __shared__ float red[256 * 8];
    const int chunk = blockIdx.x;
    const int nvox = a.D * a.H * a.W;
    const int v0 = chunk * rows_per_chunk * a.W;
    const int v1 = min(v0 + rows_per_chunk * a.W, nvox);
    const int groups = a.C / 8;
    const int g = threadIdx.x % groups, lanes = 256 / groups;
    const int vt = threadIdx.x / groups;
    float s[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] = 0.0f;
    if (vt < lanes) {
        for (int v = v0 + vt; v < v1; v += lanes) {
            const bf16x8 q = *reinterpret_cast<const bf16x8 *>(a.p + (size_t)v * a.stride + 8 * g);
#pragma unroll
            for (int e = 0; e < 8; ++e) s[e] += (float)q[e];
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) red[threadIdx.x * 8 + e] = s[e];
    __syncthreads();
    for (int c = threadIdx.x; c < a.C; c += 256) {
        const int gg = c / 8, e = c % 8;
        float t = 0.0f;
        for (int k = 0; k < lanes; ++k) t += red[(k * groups + gg) * 8 + e];
        part[(size_t)chunk * a.C + c] = t;
    }
}

// Elementwise kernels: one thread per 8-channel chunk of a voxel (16-byte
// loads and stores), index I = int when the chunk count fits 31 bits.  Each
// value is computed as in a per-channel loop, in the same order.
template <typename I>
__device__ __forceinline__ void chunk_coords(I i, int C8, int W, int H, int &c, int &x, int &y, int &z)
{
    c = (int)(i % C8) * 8;
    I v = i / C8;
    x = (int)(v % W);
    v /= W;
    y = (int)(v % H);
    z = (int)(v / H);
}

__device__ __forceinline__ size_t voxel_at(const Act &t, int z, int y, int x)
{
    return (((size_t)z * t.H + y) * t.W + x) * t.stride;
}

// g where y > 0, else 0
__device__ __forceinline__ bf16x8 mask8(bf16x8 g, const bf16x8 y)
{
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (!((float)y[e] > 0.0f)) g[e] = (__bf16)0.0f;
    return g;
}

// dY *= (Y > 0) in place (ReLU backward; Y is the post-ReLU output)
template <typename I>
__global__ void relu_mask(Act dy, const Act y)
{
    const int C8 = dy.C / 8;
    const I n = (I)dy.D * dy.H * dy.W * C8;
    for (I i = (I)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (I)gridDim.x * blockDim.x) {
        const I v = i / C8;
        const int c = (int)(i % C8) * 8;
        const bf16x8 g = *reinterpret_cast<const bf16x8 *>(dy.p + (size_t)v * dy.stride + c);
        const bf16x8 q = *reinterpret_cast<const bf16x8 *>(y.p + (size_t)v * y.stride + c);
        *reinterpret_cast<bf16x8 *>(dy.p + (size_t)v * dy.stride + c) = mask8(g, q);
    }
}

// 2x2x2 average pooling: out (D/2,H/2,W/2) from in
template <typename I>
__global__ void avgpool2(const Act in, Act out)
{
    const int C8 = out.C / 8;
    const I n = (I)out.D * out.H * out.W * C8;
    for (I i = (I)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (I)gridDim.x * blockDim.x) {
        int c, x, y, z;
        chunk_coords<I>(i, C8, out.W, out.H, c, x, y, z);
        float s[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] = 0.0f;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const bf16x8 t = *reinterpret_cast<const bf16x8 *>(
                in.p + voxel_at(in, 2 * z + (q >> 2), 2 * y + ((q >> 1) & 1), 2 * x + (q & 1)) + c);
#pragma unroll
            for (int e = 0; e < 8; ++e) s[e] += (float)t[e];
        }
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (__bf16)(0.125f * s[e]);
        *reinterpret_cast<bf16x8 *>(out.p + voxel_at(out, z, y, x) + c) = o;
    }
}

// backward of avgpool2: din = dout(parent) / 8
template <typename I>
__global__ void avgpool2_bwd(const Act dout, Act din)
{
    const int C8 = din.C / 8;
    const I n = (I)din.D * din.H * din.W * C8;
    for (I i = (I)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (I)gridDim.x * blockDim.x) {
        int c, x, y, z;
        chunk_coords<I>(i, C8, din.W, din.H, c, x, y, z);
        const bf16x8 g = *reinterpret_cast<const bf16x8 *>(dout.p + voxel_at(dout, z / 2, y / 2, x / 2) + c);
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (__bf16)(0.125f * (float)g[e]);
        *reinterpret_cast<bf16x8 *>(din.p + voxel_at(din, z, y, x) + c) = o;
    }
}

// Where a tensor feeds a pooling and a skip connection: g = (g + dout(parent)
// / 8) where keep > 0, else 0; each addend and the sum rounded to BF16 as by
// avgpool2_bwd and add_kernel.
template <typename I>
__global__ void avgpool2_bwd_add(const Act dout, const Act keep, Act g)
{
    const int C8 = g.C / 8;
    const I n = (I)g.D * g.H * g.W * C8;
    for (I i = (I)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (I)gridDim.x * blockDim.x) {
        int c, x, y, z;
        chunk_coords<I>(i, C8, g.W, g.H, c, x, y, z);
        const bf16x8 p = *reinterpret_cast<const bf16x8 *>(dout.p + voxel_at(dout, z / 2, y / 2, x / 2) + c);
        bf16x8 *const at = reinterpret_cast<bf16x8 *>(g.p + voxel_at(g, z, y, x) + c);
        const bf16x8 q = *at;
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (__bf16)((float)q[e] + (float)(__bf16)(0.125f * (float)p[e]));
        *at = mask8(o, *reinterpret_cast<const bf16x8 *>(keep.p + voxel_at(keep, z, y, x) + c));
    }
}

// nearest 2x upsampling: out (2D,2H,2W) from in
template <typename I>
__global__ void upsample2(const Act in, Act out)
{
    const int C8 = out.C / 8;
    const I n = (I)out.D * out.H * out.W * C8;
    for (I i = (I)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (I)gridDim.x * blockDim.x) {
        int c, x, y, z;
        chunk_coords<I>(i, C8, out.W, out.H, c, x, y, z);
        *reinterpret_cast<bf16x8 *>(out.p + voxel_at(out, z, y, x) + c) =
            *reinterpret_cast<const bf16x8 *>(in.p + voxel_at(in, z / 2, y / 2, x / 2) + c);
    }
}

// backward of upsample2: din = sum of the 8 children of dout, 0 where keep (if
// given) is not positive
template <typename I>
__global__ void upsample2_bwd(const Act dout, Act din, const Act keep)
{
    const int C8 = din.C / 8;
    const I n = (I)din.D * din.H * din.W * C8;
    for (I i = (I)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (I)gridDim.x * blockDim.x) {
        int c, x, y, z;
        chunk_coords<I>(i, C8, din.W, din.H, c, x, y, z);
        float s[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] = 0.0f;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const bf16x8 t = *reinterpret_cast<const bf16x8 *>(
                dout.p + voxel_at(dout, 2 * z + (q >> 2), 2 * y + ((q >> 1) & 1), 2 * x + (q & 1)) + c);
#pragma unroll
            for (int e = 0; e < 8; ++e) s[e] += (float)t[e];
        }
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (__bf16)s[e];
        if (keep.p) o = mask8(o, *reinterpret_cast<const bf16x8 *>(keep.p + voxel_at(keep, z, y, x) + c));
        *reinterpret_cast<bf16x8 *>(din.p + voxel_at(din, z, y, x) + c) = o;
    }
}

// out = a + b (BF16 tensors of the same shape; slices allowed)
template <typename I>
__global__ void add_kernel(const Act a, const Act b, Act out)
{
    const int C8 = out.C / 8;
    const I n = (I)out.D * out.H * out.W * C8;
    for (I i = (I)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (I)gridDim.x * blockDim.x) {
        const I v = i / C8;
        const int c = (int)(i % C8) * 8;
        const bf16x8 p = *reinterpret_cast<const bf16x8 *>(a.p + (size_t)v * a.stride + c);
        const bf16x8 q = *reinterpret_cast<const bf16x8 *>(b.p + (size_t)v * b.stride + c);
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (__bf16)((float)p[e] + (float)q[e]);
        *reinterpret_cast<bf16x8 *>(out.p + (size_t)v * out.stride + c) = o;
    }
}

// Pack two FP32 volumes into channels 0 and 1 of a 16-channel BF16 tensor
// (channels 2..15 zero), scaled by `scale`.
__global__ void pack_input(const float *__restrict__ x1, const float *__restrict__ x2, int64_t nvox,
                           float scale, Act out)
{
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < nvox; v += (int64_t)gridDim.x * blockDim.x) {
        __bf16 *o = out.p + v * out.stride;
        bf16x8 a = zero8(), b = zero8();
        a[0] = (__bf16)(scale * x1[v]);
        a[1] = (__bf16)(scale * x2[v]);
        *reinterpret_cast<bf16x8 *>(o) = a;
        *reinterpret_cast<bf16x8 *>(o + 8) = b;
    }
}

// Output head (1x1x1 convolution 16 -> 1, in FP32) with the residual on x2:
//   x0 = x2 + (sum_c w[c] h[v][c] + b) / scale
__global__ void head_fwd(const Act h, const float *__restrict__ w, const float *__restrict__ b,
                         const float *__restrict__ x2, float inv_scale, float *__restrict__ x0)
{
    const int64_t n = (int64_t)h.D * h.H * h.W;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        float s = b[0];
        for (int c8 = 0; c8 < h.C; c8 += 8) {
            const bf16x8 q = *reinterpret_cast<const bf16x8 *>(h.p + v * h.stride + c8);
#pragma unroll
            for (int e = 0; e < 8; ++e) s = fmaf(w[c8 + e], (float)q[e], s);
        }
        x0[v] = x2[v] + s * inv_scale;
    }
}

// Head backward: dh[v][c] = w[c] g[v] / scale (BF16), with `relu` 0 where
// h[v][c] is not positive; partial sums for dw, db
__global__ void head_bwd(const Act h, const float *__restrict__ w, const float *__restrict__ g,
                         float inv_scale, Act dh, int64_t per_block, int relu, float *__restrict__ part)
{
    __shared__ float sh[17][256];
    const int64_t n = (int64_t)h.D * h.H * h.W;
    const int64_t v0 = (int64_t)blockIdx.x * per_block;
    const int64_t v1 = v0 + per_block < n ? v0 + per_block : n;
    float acc[17];
    for (int c = 0; c < 17; ++c) acc[c] = 0.0f;
    for (int64_t v = v0 + threadIdx.x; v < v1; v += blockDim.x) {
        const float gv = g[v] * inv_scale;
#pragma unroll
        for (int c8 = 0; c8 < 16; c8 += 8) {
            if (c8 >= h.C) break;
            const bf16x8 q = *reinterpret_cast<const bf16x8 *>(h.p + v * h.stride + c8);
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                acc[c8 + e] = fmaf((float)q[e], gv, acc[c8 + e]);
                o[e] = (__bf16)(w[c8 + e] * gv);
            }
            *reinterpret_cast<bf16x8 *>(dh.p + v * dh.stride + c8) = relu ? mask8(o, q) : o;
        }
        acc[16] += gv;
    }
    for (int c = 0; c < 17; ++c) sh[c][threadIdx.x] = acc[c];
    __syncthreads();
    // 15 threads a channel, then their sums
    const int c = threadIdx.x / 15, k = threadIdx.x % 15;
    float s = 0.0f;
    if (threadIdx.x < 255)
        for (int t = k; t < 256; t += 15) s += sh[c][t];
    __syncthreads();
    if (threadIdx.x < 255) sh[c][k] = s;
    __syncthreads();
    if (threadIdx.x < 17) {
        float s = 0.0f;
        for (int t = 0; t < 15; ++t) s += sh[threadIdx.x][t];
        part[(size_t)blockIdx.x * 17 + threadIdx.x] = s;
    }
}

// Weights [27][Co][Ci] -> [27][Ci][Co] (backward-data uses the mirrored taps)
__global__ void transpose_weights(const __bf16 *__restrict__ w, __bf16 *__restrict__ wt, int co, int ci)
{
    const int n = 27 * co * ci;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const int t = i / (co * ci), r = i % (co * ci);
        const int o = r / ci, c = r % ci;
        wt[((size_t)t * ci + c) * co + o] = w[i];
    }
}

// sh[0] = the sum of v over the 256 threads of a block, in a fixed order
__device__ __forceinline__ void block_sum_f64(double *sh, double v)
{
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
        __syncthreads();
    }
}

// MSE: grad = 2 (a - b) / n, partial sums of (a - b)^2 (FP64)
__global__ void mse_kernel(const float *__restrict__ a, const float *__restrict__ b, int64_t n,
                           float *__restrict__ grad, double *__restrict__ part)
{
    __shared__ double sh[256];
    double acc = 0.0;
    const float sc = 2.0f / (float)n;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float dlt = a[i] - b[i];
        grad[i] = sc * dlt;
        acc += (double)dlt * dlt;
    }
    block_sum_f64(sh, acc);
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ void sum_partials_f64(const double *__restrict__ part, int n, double scale, double *__restrict__ out)
{
    __shared__ double sh[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) s += part[i];
    block_sum_f64(sh, s);
    if (threadIdx.x == 0) *out = sh[0] * scale;
}

// Adam on FP32 master weights, with a BF16 copy for the kernels (optional)
__global__ void adam_kernel(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                            float *__restrict__ v, int64_t n, float lr, float b1, float b2, float eps,
                            float c1, float c2, __bf16 *__restrict__ pb)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.0f - b1) * gi;
        const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        const float upd = lr * (mi * c1) / (sqrtf(vi * c2) + eps);
        const float np = p[i] - upd;
        p[i] = np;
        if (pb) pb[i] = (__bf16)np;
    }
}

}  // namespace cvpnn

// ------------------------------------------------------------------ C ABI
#include "cvp.h"

namespace {

cvpnn::Act act(const cvp_nn_tensor *t)
{
    cvpnn::Act a;
    a.p = reinterpret_cast<__bf16 *>(t->data);
    a.D = t->d; a.H = t->h; a.W = t->w; a.C = t->channels; a.stride = t->stride;
    return a;
}

bool valid(const cvp_nn_tensor *t)
{
    return t && t->data && t->d > 0 && t->h > 0 && t->w > 0 && t->channels > 0 &&
           t->stride >= t->channels && (t->channels % 8) == 0 && (t->stride % 8) == 0 &&
           (reinterpret_cast<uintptr_t>(t->data) & 15) == 0;
}

cvp_status st(hipError_t e) { return e == hipSuccess ? CVP_OK : CVP_E_DEVICE; }

// Bounds of the weight gradient's partial sums: two workgroups per CU, and 57
// MB.  Measured with the reduction, microseconds at (16 -> 16, 64 x 72 x 88),
// (32 -> 16, the same) and (64 -> 32, 48 x 50 x 66): 25, 42, 58; with at most
// 256 chunks 34, 58, 58; with 28 MB 25, 42, 89; with 113 MB 25, 42, 71.
constexpr int64_t kWgradChunks = 512;
constexpr int64_t kWgradFloats = int64_t(2) * 64 * 64 * 27 * 64;

int grid_for(int64_t n) { return (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096); }

// The next longer run of a march along d slices that takes fewer runs (the ones
// between cost more for as many units, so a plan need not try them); d + 1 after
// the last.  About 2 sqrt(d) candidates: a call on 200 000 slices takes 27 us of
// the host, trying every run 1450.
int next_run(int d, int run)
{
    const int n = (d + run - 1) / run;
    return n == 1 ? d + 1 : (d + n - 2) / (n - 1);
}

// A convolution marched along d: the tile height and the run length whose
// busiest workgroup is done first.  A unit takes the weights' load, its slices
// and the two more that its first needs; a slice takes its matrix work or its
// loads, whichever is longer (cycles of a CU).
template <int CO, int CI, int NT>
cvpnn::MarchPlan march_plan(const cvpnn::Act &a, int &blocks)
{
    constexpr int per_cu = CI * NT == 16 ? 3 : CI * NT == 32 ? 2 : 1;
    constexpr int steps = (27 * CI + 31) / 32, WR = 4 / (CO / (16 * NT));
    cvpnn::MarchPlan best{};
    double least = 0.0;
    for (int rows = 2; rows <= cvpnn::kMarchRows; rows *= 2) {
        cvpnn::MarchPlan p;
        p.rows = rows;
        p.ytiles = (a.H + rows - 1) / rows;
        p.segs = (a.W + 31) / 32;
        const int passes = (rows / 2 + WR - 1) / WR;
        const double work = passes * steps * 4 * NT * 16.0 * (NT == 1 ? 2 : 1) * (per_cu > 1 ? per_cu / 1.5 : 1.0) + 600;
        const double load = (rows + 2) * 34.0 * CI * 2 / 24 * per_cu + 800;
        for (int run = 1; run <= a.D; run = next_run(a.D, run)) {
            const int64_t units = (int64_t)p.ytiles * p.segs * ((a.D + run - 1) / run);
            if (units > INT32_MAX / 2) continue;
            const int64_t slots = std::min<int64_t>(units, 256 * per_cu);
            const double cost = (double)((units + slots - 1) / slots) * (run * std::max(work, load) + 2 * load) +
                                steps * NT * 16.0 * 4 * per_cu;
            if (least == 0.0 || cost < least) {
                least = cost;
                p.run = run;
                p.units = (int)units;
                best = p;
                blocks = (int)slots;
            }
        }
    }
    return best;
}

template <int CO, int CI, int NT, bool FLIP, bool MASK>
hipError_t launch_march(const cvpnn::Act &a, const __bf16 *w, const float *bias, const cvpnn::Act &o, const cvpnn::Act &keep,
                        int relu, hipStream_t s)
{
    static const hipError_t ready =
        hipFuncSetAttribute(reinterpret_cast<const void *>(cvpnn::conv3d_march_kernel<CO, CI, NT, FLIP, MASK>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, cvpnn::march_lds_bytes<CI>());
    if (ready != hipSuccess) return ready;
    int blocks = 0;
    const cvpnn::MarchPlan p = march_plan<CO, CI, NT>(a, blocks);
    hipLaunchKernelGGL((cvpnn::conv3d_march_kernel<CO, CI, NT, FLIP, MASK>), dim3(blocks), dim3(256),
                       (cvpnn::march_lds_bytes<CI>()), s, a, w, bias, o, keep, relu, p);
    return hipGetLastError();
}

bool same_grid(const cvp_nn_tensor *a, const cvp_nn_tensor *b) { return a->d == b->d && a->h == b->h && a->w == b->w; }

// keep: 0, or the post-ReLU tensor that masks the result (flip set, then)
cvp_status convolve(const cvp_nn_tensor *in, const void *weight, const float *bias, const cvp_nn_tensor *out,
                    const cvp_nn_tensor *keep, int relu, int flip, void *stream)
{
    const cvpnn::Act a = act(in), o = act(out), k = keep ? act(keep) : cvpnn::Act{};
    hipStream_t s = (hipStream_t)stream;
    const __bf16 *w = reinterpret_cast<const __bf16 *>(weight);
    // channel counts 16, 32, 64 and 32-bit byte offsets: the marching kernel,
    // with the weights of 32 output channels in a wave where they fit its
    // registers (with 64 input channels 432 of 512 would be taken)
    const int64_t elems = (int64_t)in->d * in->h * in->w * std::max(std::max(in->stride, out->stride), k.stride);
    const int ci = in->channels, co = out->channels;
    const bool spec = elems <= cvpnn::kMarchElems && (ci == 16 || ci == 32 || ci == 64);
#define MARCH(CO_, CI_, NT_)                                                                       \
    if (spec && co == CO_ && ci == CI_)                                                            \
        return st(keep   ? launch_march<CO_, CI_, NT_, true, true>(a, w, bias, o, k, relu, s)      \
                  : flip ? launch_march<CO_, CI_, NT_, true, false>(a, w, bias, o, k, relu, s)     \
                         : launch_march<CO_, CI_, NT_, false, false>(a, w, bias, o, k, relu, s));
    MARCH(16, 16, 1) MARCH(16, 32, 1) MARCH(16, 64, 1)
    MARCH(32, 16, 2) MARCH(32, 32, 2) MARCH(32, 64, 1)
    MARCH(64, 16, 2) MARCH(64, 32, 2) MARCH(64, 64, 1)
#undef MARCH
    const int rows = in->d * in->h * ((in->w + 63) / 64);
    const dim3 grid((rows + 3) / 4), block(256);
    switch (co) {
    case 16: hipLaunchKernelGGL(cvpnn::conv3d_kernel<16>, grid, block, 0, s, a, w, bias, o, relu, flip); break;
    case 32: hipLaunchKernelGGL(cvpnn::conv3d_kernel<32>, grid, block, 0, s, a, w, bias, o, relu, flip); break;
    case 64: hipLaunchKernelGGL(cvpnn::conv3d_kernel<64>, grid, block, 0, s, a, w, bias, o, relu, flip); break;
    default: return CVP_E_UNSUPPORTED;
    }
    const hipError_t e = hipGetLastError();
    return e != hipSuccess || !keep ? st(e) : cvp_nn_relu_mask(out, keep, stream);
}

}  // namespace

extern "C" {

cvp_status cvp_nn_conv3d(const cvp_nn_tensor *in, const void *weight, const float *bias,
                         const cvp_nn_tensor *out, int32_t relu, int32_t flip, void *stream)
{
    if (!valid(in) || !valid(out) || !weight) return CVP_E_INVALID;
    if (in->d != out->d || in->h != out->h || in->w != out->w) return CVP_E_INVALID;
    return convolve(in, weight, bias, out, nullptr, relu, flip, stream);
}

cvp_status cvp_nn_conv3d_bwd_masked(const cvp_nn_tensor *dy, const void *weight_t, const cvp_nn_tensor *keep,
                                    const cvp_nn_tensor *dx, void *stream)
{
    if (!valid(dy) || !valid(dx) || !valid(keep) || !weight_t) return CVP_E_INVALID;
    if (!same_grid(dy, dx) || !same_grid(dx, keep) || keep->channels != dx->channels) return CVP_E_INVALID;
    return convolve(dy, weight_t, nullptr, dx, keep, 0, 1, stream);
}

// Partial sums of the weight gradient that fill the GPU (nw floats each).
static int64_t wgrad_chunks_wanted(int64_t nw)
{
    return std::max<int64_t>(1, std::min<int64_t>(kWgradChunks, kWgradFloats / nw));
}

// the smallest workspace taken: one partial sum per 64 rows
static int64_t wgrad_chunks_least(const cvp_nn_tensor *x) { return ((int64_t)x->d * x->h + 63) / 64; }

// rows of a tile and tiles of a slice
static int wgrad_tile_rows(int ci) { return ci == 16 ? cvpnn::wgrad_rows<16>() : ci == 32 ? cvpnn::wgrad_rows<32>() : cvpnn::wgrad_rows<64>(); }
static int64_t wgrad_columns(const cvp_nn_tensor *x)
{
    const int ty = wgrad_tile_rows(x->channels);
    return (int64_t)((x->h + ty - 1) / ty) * ((x->w + 31) / 32);
}

cvp_status cvp_nn_wgrad_workspace(const cvp_nn_tensor *x, const cvp_nn_tensor *dy, int64_t *floats)
{
    if (!x || !dy || !floats) return CVP_E_INVALID;
    const int64_t nw = (int64_t)27 * dy->channels * x->channels;
    const int64_t least = wgrad_chunks_least(x);
    // no more partial sums than there are tiles; each with the bias gradient's
    const int64_t chunks = nw > 0 ? std::max(least, std::min(wgrad_chunks_wanted(nw), wgrad_columns(x) * x->d)) : least;
    *floats = chunks * (nw + dy->channels);
    return CVP_OK;
}

// db: 0, or the bias gradient as well
static cvp_status wgrad(const cvp_nn_tensor *x, const cvp_nn_tensor *dy, float *dw, float *db, float *work,
                        int64_t work_floats, void *stream)
{
    if (!valid(x) || !valid(dy) || !dw || !work) return CVP_E_INVALID;
    const int co = dy->channels, ci = x->channels;
    const int64_t nw = (int64_t)27 * co * ci, n = nw + (db ? co : 0);
    if (work_floats < wgrad_chunks_least(x) * n) return CVP_E_INVALID;
    const cvpnn::Act a = act(x), g = act(dy);
    hipStream_t s = (hipStream_t)stream;
    // the run length whose longest chunk is shortest: a unit costs its slices
    // and the two more that its first needs
    const int64_t cap = std::min(work_floats / n, wgrad_chunks_wanted(nw));
    cvpnn::WgradPlan p;
    p.ytiles = (x->h + wgrad_tile_rows(ci) - 1) / wgrad_tile_rows(ci);
    p.segs = (x->w + 31) / 32;
    const int64_t columns = wgrad_columns(x);
    if (columns * x->d > INT32_MAX / 2) return CVP_E_UNSUPPORTED;
    int64_t best = INT64_MAX;
    for (int run = 1; run <= x->d; run = next_run(x->d, run)) {
        const int64_t units = columns * ((x->d + run - 1) / run), chunks = std::min(cap, units);
        const int64_t cost = (units + chunks - 1) / chunks * (run + 2);
        if (cost < best) {
            best = cost;
            p.run = run;
            p.units = (int)units;
            p.chunks = (int)chunks;
        }
    }
#define WG(CO_, CI_)                                                                                            \
    do {                                                                                                        \
        static const hipError_t ready = hipFuncSetAttribute(                                                    \
            reinterpret_cast<const void *>(cvpnn::conv3d_wgrad_kernel<CO_, CI_>),                               \
            hipFuncAttributeMaxDynamicSharedMemorySize, cvpnn::wgrad_lds_bytes<CO_, CI_>());                    \
        if (ready != hipSuccess) return st(ready);                                                              \
        hipLaunchKernelGGL((cvpnn::conv3d_wgrad_kernel<CO_, CI_>), dim3(p.chunks, CO_ > 32 ? CO_ / 32 : 1),     \
                           dim3(256), (cvpnn::wgrad_lds_bytes<CO_, CI_>()), s, a, g, p, db ? 1 : 0, work);                  \
    } while (0)
    if (co == 16 && ci == 16) WG(16, 16);
    else if (co == 16 && ci == 32) WG(16, 32);
    else if (co == 32 && ci == 16) WG(32, 16);
    else if (co == 32 && ci == 32) WG(32, 32);
    else if (co == 32 && ci == 64) WG(32, 64);
    else if (co == 64 && ci == 32) WG(64, 32);
    else if (co == 64 && ci == 64) WG(64, 64);
    else if (co == 16 && ci == 64) WG(16, 64);
    else return CVP_E_UNSUPPORTED;
#undef WG
    hipLaunchKernelGGL(cvpnn::reduce_chunks, dim3(grid_for(4 * n)), dim3(1024), 0, s, work, p.chunks, n, dw, nw, db);
    return st(hipGetLastError());
}

cvp_status cvp_nn_conv3d_wgrad(const cvp_nn_tensor *x, const cvp_nn_tensor *dy, float *dw, float *work,
                               int64_t work_floats, void *stream)
{
    return wgrad(x, dy, dw, nullptr, work, work_floats, stream);
}

cvp_status cvp_nn_conv3d_wgrad_bias(const cvp_nn_tensor *x, const cvp_nn_tensor *dy, float *dw, float *db, float *work,
                                    int64_t work_floats, void *stream)
{
    if (!db) return CVP_E_INVALID;
    return wgrad(x, dy, dw, db, work, work_floats, stream);
}

cvp_status cvp_nn_channel_sum(const cvp_nn_tensor *a, float *out, float *work, int64_t work_floats,
                              void *stream)
{
    if (!valid(a) || !out || !work) return CVP_E_INVALID;
    if (a->channels > 2048) return CVP_E_UNSUPPORTED;
    const int rows = a->d * a->h, rpc = 16, chunks = (rows + rpc - 1) / rpc;
    if (work_floats < (int64_t)chunks * a->channels) return CVP_E_INVALID;
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(cvpnn::channel_sum_partials, dim3(chunks), dim3(256), 0, s, act(a), rpc, work);
    hipLaunchKernelGGL(cvpnn::reduce_chunks, dim3(1), dim3(1024), 0, s, work, chunks, (int64_t)a->channels, out,
                       (int64_t)a->channels, nullptr);
    return st(hipGetLastError());
}

cvp_status cvp_nn_relu_mask(const cvp_nn_tensor *dy, const cvp_nn_tensor *y, void *stream)
{
    if (!valid(dy) || !valid(y)) return CVP_E_INVALID;
    const int64_t n = (int64_t)dy->d * dy->h * dy->w * dy->channels / 8;
    if (n < (int64_t(1) << 31))
        hipLaunchKernelGGL(cvpnn::relu_mask<int>, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)stream, act(dy), act(y));
    else
        hipLaunchKernelGGL(cvpnn::relu_mask<int64_t>, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)stream, act(dy),
                           act(y));
    return st(hipGetLastError());
}

static cvp_status resample(int kind, const cvp_nn_tensor *a, const cvp_nn_tensor *b, void *stream,
                           const cvp_nn_tensor *keep = nullptr)
{
    if (!valid(a) || !valid(b) || a->channels != b->channels) return CVP_E_INVALID;
    hipStream_t s = (hipStream_t)stream;
    const cvp_nn_tensor *big = (kind == 0 || kind == 3) ? a : b;    // fine-resolution operand
    const cvp_nn_tensor *small = big == a ? b : a;
    if (big->d != 2 * small->d || big->h != 2 * small->h || big->w != 2 * small->w) return CVP_E_INVALID;
    // 8-channel chunks of the fine and the coarse operand
    const int64_t nb = (int64_t)big->d * big->h * big->w * big->channels / 8;
    const int64_t ns = nb / 8;
    const bool i32 = nb < (int64_t(1) << 31);
#define RS(K, N, ...)                                                                                       \
    do {                                                                                                    \
        if (i32) hipLaunchKernelGGL(cvpnn::K<int>, dim3(grid_for(N)), dim3(256), 0, s, act(a), __VA_ARGS__); \
        else hipLaunchKernelGGL(cvpnn::K<int64_t>, dim3(grid_for(N)), dim3(256), 0, s, act(a), __VA_ARGS__); \
    } while (0)
    switch (kind) {
    case 0: RS(avgpool2, ns, act(b)); break;
    case 1:
        if (keep) RS(avgpool2_bwd_add, nb, act(keep), act(b));
        else RS(avgpool2_bwd, nb, act(b));
        break;
    case 2: RS(upsample2, nb, act(b)); break;
    default: RS(upsample2_bwd, ns, act(b), keep ? act(keep) : cvpnn::Act{}); break;
    }
#undef RS
    return st(hipGetLastError());
}

cvp_status cvp_nn_avgpool2(const cvp_nn_tensor *in, const cvp_nn_tensor *out, void *stream) { return resample(0, in, out, stream); }
cvp_status cvp_nn_avgpool2_bwd(const cvp_nn_tensor *dout, const cvp_nn_tensor *din, void *stream) { return resample(1, dout, din, stream); }
cvp_status cvp_nn_upsample2(const cvp_nn_tensor *in, const cvp_nn_tensor *out, void *stream) { return resample(2, in, out, stream); }
cvp_status cvp_nn_upsample2_bwd(const cvp_nn_tensor *dout, const cvp_nn_tensor *din, void *stream) { return resample(3, dout, din, stream); }

cvp_status cvp_nn_avgpool2_bwd_add(const cvp_nn_tensor *dout, const cvp_nn_tensor *keep, const cvp_nn_tensor *g, void *stream)
{
    if (!valid(keep) || !valid(g) || !same_grid(keep, g) || keep->channels != g->channels) return CVP_E_INVALID;
    return resample(1, dout, g, stream, keep);
}

cvp_status cvp_nn_upsample2_bwd_masked(const cvp_nn_tensor *dout, const cvp_nn_tensor *keep, const cvp_nn_tensor *din,
                                       void *stream)
{
    if (!valid(keep) || !valid(din) || !same_grid(keep, din) || keep->channels != din->channels) return CVP_E_INVALID;
    return resample(3, dout, din, stream, keep);
}

cvp_status cvp_nn_add(const cvp_nn_tensor *a, const cvp_nn_tensor *b, const cvp_nn_tensor *out, void *stream)
{
    if (!valid(a) || !valid(b) || !valid(out) || a->channels != out->channels || b->channels != out->channels ||
        a->d != out->d || a->h != out->h || a->w != out->w || b->d != out->d || b->h != out->h || b->w != out->w)
        return CVP_E_INVALID;
    const int64_t n = (int64_t)out->d * out->h * out->w * out->channels / 8;
    if (n < (int64_t(1) << 31))
        hipLaunchKernelGGL(cvpnn::add_kernel<int>, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)stream, act(a), act(b),
                           act(out));
    else
        hipLaunchKernelGGL(cvpnn::add_kernel<int64_t>, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)stream, act(a),
                           act(b), act(out));
    return st(hipGetLastError());
}

cvp_status cvp_nn_transpose_weights(const void *w, void *wt, int32_t co, int32_t ci, void *stream)
{
    if (!w || !wt || co <= 0 || ci <= 0) return CVP_E_INVALID;
    const int64_t n = (int64_t)27 * co * ci;
    hipLaunchKernelGGL(cvpnn::transpose_weights, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)stream,
                       reinterpret_cast<const __bf16 *>(w), reinterpret_cast<__bf16 *>(wt), co, ci);
    return st(hipGetLastError());
}

cvp_status cvp_nn_pack_input(const float *x1, const float *x2, float scale, const cvp_nn_tensor *out, void *stream)
{
    if (!x1 || !x2 || !valid(out) || out->channels != 16) return CVP_E_INVALID;
    const int64_t n = (int64_t)out->d * out->h * out->w;
    hipLaunchKernelGGL(cvpnn::pack_input, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)stream, x1, x2, n, scale, act(out));
    return st(hipGetLastError());
}

cvp_status cvp_nn_head(const cvp_nn_tensor *h, const float *w, const float *b, const float *x2, float scale,
                       float *x0, void *stream)
{
    if (!valid(h) || h->channels > 16 || !w || !b || !x2 || !x0 || !(scale > 0)) return CVP_E_INVALID;
    const int64_t n = (int64_t)h->d * h->h * h->w;
    hipLaunchKernelGGL(cvpnn::head_fwd, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)stream, act(h), w, b, x2,
                       1.0f / scale, x0);
    return st(hipGetLastError());
}

static cvp_status head_bwd(const cvp_nn_tensor *h, const float *w, const float *g, float scale,
                           const cvp_nn_tensor *dh, float *dwb /*17*/, float *work, int64_t work_floats, int relu,
                           void *stream)
{
    if (!valid(h) || !valid(dh) || h->channels > 16 || !w || !g || !dwb || !work || !(scale > 0)) return CVP_E_INVALID;
    const int64_t n = (int64_t)h->d * h->h * h->w;
    const int64_t per = 4096;
    const int blocks = (int)((n + per - 1) / per);
    if (work_floats < (int64_t)blocks * 17) return CVP_E_INVALID;
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(cvpnn::head_bwd, dim3(blocks), dim3(256), 0, s, act(h), w, g, 1.0f / scale, act(dh), per, relu,
                       work);
    hipLaunchKernelGGL(cvpnn::reduce_chunks, dim3(1), dim3(1024), 0, s, work, blocks, (int64_t)17, dwb, (int64_t)17, nullptr);
    return st(hipGetLastError());
}

cvp_status cvp_nn_head_bwd(const cvp_nn_tensor *h, const float *w, const float *g, float scale,
                           const cvp_nn_tensor *dh, float *dwb, float *work, int64_t work_floats, void *stream)
{
    return head_bwd(h, w, g, scale, dh, dwb, work, work_floats, 0, stream);
}

cvp_status cvp_nn_head_bwd_masked(const cvp_nn_tensor *h, const float *w, const float *g, float scale,
                                  const cvp_nn_tensor *dh, float *dwb, float *work, int64_t work_floats, void *stream)
{
    return head_bwd(h, w, g, scale, dh, dwb, work, work_floats, 1, stream);
}

cvp_status cvp_nn_mse(const float *a, const float *b, int64_t n, float *grad, double *loss, double *work,
                      int64_t work_doubles, void *stream)
{
    if (!a || !b || !grad || !loss || !work || n <= 0 || work_doubles < 1024) return CVP_E_INVALID;
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(cvpnn::mse_kernel, dim3(1024), dim3(256), 0, s, a, b, n, grad, work);
    hipLaunchKernelGGL(cvpnn::sum_partials_f64, dim3(1), dim3(256), 0, s, work, 1024, 1.0 / (double)n, loss);
    return st(hipGetLastError());
}

cvp_status cvp_nn_adam(float *p, const float *g, float *m, float *v, int64_t n, float lr, float beta1,
                       float beta2, float eps, int32_t step, void *p_bf16, void *stream)
{
    if (!p || !g || !m || !v || n <= 0 || step < 1) return CVP_E_INVALID;
    const float c1 = 1.0f / (1.0f - powf(beta1, (float)step));
    const float c2 = 1.0f / (1.0f - powf(beta2, (float)step));
    hipLaunchKernelGGL(cvpnn::adam_kernel, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)stream, p, g, m, v, n, lr,
                       beta1, beta2, eps, c1, c2, reinterpret_cast<__bf16 *>(p_bf16));
    return st(hipGetLastError());
}

}  // extern "C"
