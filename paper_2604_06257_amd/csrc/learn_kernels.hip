// gfx950 kernels of the learned-compounding network (3D U-Net): BF16 MFMA
// convolutions with FP32 accumulation, and the small element-wise steps of
// training.  Volumes are channels-last [D][H][W][C]; a tensor may be a slice of
// a wider buffer (row stride `*_stride` channels, first channel `*_coff`).
//
// Convolution (3 x 3 x 3, zero padding, stride 1) as an implicit GEMM on
// v_mfma_f32_16x16x32_bf16: voxels and output channels are the tile's two sides,
// K = 27 * Cin in steps of 32, ordered by channel chunk, in-plane tap and depth
// tap.  A workgroup stages a brick of the input with its one-voxel halo in LDS,
// one channel chunk at a time (conv3d_brick_kernel for aligned tensors,
// conv3d_kernel for the others; the same bits).  With `flip`, the taps are
// mirrored: this is the input gradient of a convolution when the weights are
// passed transposed ([Cin][27][Cout]).
#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <type_traits>

#include "das_learn.h"

// The loads straight to LDS are inline assembly that sets m0, the compiler's own register for that place; it warns of it in a
// clobber list, which is where it has to stand so that no value is kept there across one.
#pragma clang diagnostic ignored "-Winline-asm"

namespace learn {

typedef __attribute__((__vector_size__(8 * sizeof(short)))) short bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

__device__ __forceinline__ float bf2f(uint16_t u) { return __uint_as_float((uint32_t)u << 16); }
__device__ __forceinline__ uint16_t f2bf(float x) {  // round to nearest even (finite inputs)
    const uint32_t u = __float_as_uint(x);
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

struct Vol {
    int D, H, W;
};

constexpr int kMaxNT = 8;  // up to 128 output channels per launch

// General convolution (calls that conv3d_brick_kernel below does not take), on a brick of 8 (W) x 8 (H) x MT (D) output
// voxels per workgroup of 4 waves, for NT x 16 of the
// output channels (grid.y = channel groups).  Wave w owns the 4 x 4 (W x H) patch w of every depth slice (one
// 16-voxel MFMA row tile per slice) and the workgroup's output channels.  The input brick with its one-voxel
// halo, 10 x 10 x (MT + 2) voxels, is staged in LDS one channel chunk (CC channels) at a time, so each input
// value is read from global memory once per chunk instead of once per tap.
//
// K is ordered by in-plane offset (dx, dy) first: a K step of 32 holds 32 / CC in-plane taps of one depth offset
// dz (CC channels each).  The operand-A fragment of an in-plane offset at halo slice z (one 16-byte LDS read per
// lane) is the same for the three depth offsets, so it feeds three MFMAs: output slice z - 1 - dz for dz = -1, 0,
// 1 (the slices that exist).  Per chunk a wave reads (MT + 2) ceil(9 CC / 32) fragments for 3 MT ceil(9 CC / 32)
// MFMAs per channel tile, instead of one fragment per MFMA.  Weights (operand B) of the three depth offsets
// come from global memory (shared by all waves through the caches), one in-plane group ahead.
//
// With several channel chunks and DB the halo is double-buffered: the next chunk's loads are issued before the
// current chunk's MFMAs and written to the other buffer after them, one barrier per chunk (used for launches with
// few workgroups, in the 1 x 1 shape; elsewhere the second buffer's LDS costs more occupancy than it hides).
//
// Epilogue: bias, ReLU, then the tile goes through LDS as float [voxel][channel], and each thread writes 8
// channels of a voxel (one 16-byte store, two for float output) after the optional mask; with `vec` = 0
// (unaligned slices) the same values are stored one element at a time.
constexpr int kHaloW = 10, kHaloH = 10;

template <int MT, int NT, int CC, bool DB>
__global__ __launch_bounds__(256) void conv3d_kernel(const uint16_t* __restrict__ in, int in_stride, int in_coff,
                                                     const uint16_t* __restrict__ wk, const float* __restrict__ bias,
                                                     void* __restrict__ out, int out_stride, int out_coff, int out_f32,
                                                     const uint16_t* __restrict__ mask, int mask_stride, int mask_coff,
                                                     Vol vol, int Cin, int flip, int relu, int vec) {
    constexpr int HD = MT + 2;
    constexpr int NHALO = kHaloW * kHaloH * HD;
    constexpr int VP = CC + 8;             // LDS elements per halo voxel (padding spreads the banks)
    constexpr int TPK = 32 / CC;           // in-plane taps per K step: 1 (CC = 32), 2 (16), 4 (8)
    constexpr int NG = (9 + TPK - 1) / TPK;  // K steps per depth offset and chunk
    constexpr int CH = 16 * NT + 4;        // epilogue row (floats; the pad spreads the banks)
    constexpr int HALO_BYTES = NHALO * VP * 2 * (DB ? 2 : 1), OUT_BYTES = 64 * MT * CH * 4;
    constexpr int NITEMS = NHALO * (CC / 8), IPT = (NITEMS + 255) / 256;  // 16-byte halo items (per thread)
    __shared__ __attribute__((aligned(16))) char smem[HALO_BYTES > OUT_BYTES ? HALO_BYTES : OUT_BYTES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nbw = (vol.W + 7) / 8, nbh = (vol.H + 7) / 8;
    const int bx = blockIdx.x % nbw, by = (blockIdx.x / nbw) % nbh, bz = blockIdx.x / (nbw * nbh);
    // output channels [n0, n0 + 16 NT) of this workgroup (grid.y = channel groups)
    const int n0 = blockIdx.y * NT * 16;
    const int w0 = 8 * bx, h0 = 8 * by, d0 = MT * bz;
    const int K = 27 * Cin;
    const int s = flip ? -1 : 1;
    // this lane's operand-A voxel within its wave's patch (row lane & 15 of the MFMA tile)
    const int pw = 4 * (wave & 1), ph = 4 * (wave >> 1);
    const int rw = pw + (lane & 3), rh = ph + ((lane >> 2) & 3);
    // this lane's 8 elements of a K step: in-plane tap slot and channel offset within the chunk
    const int g = lane >> 4, slot = g / (CC / 8), cg = 8 * (g % (CC / 8));
    f32x4 acc[MT][NT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[m][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // this thread's halo items: global offset (without the chunk's first channel; -1 outside the volume) and LDS
    // offset, the same for every chunk
    int64_t goff[IPT];
    int loff[IPT];
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int it = threadIdx.x + 256 * i;
        const int hv = it / (CC / 8), c8 = it - hv * (CC / 8);
        const int hx = hv % kHaloW, hy = (hv / kHaloW) % kHaloH, hz = hv / (kHaloW * kHaloH);
        const int zw = w0 - 1 + hx, zh = h0 - 1 + hy, zd = d0 - 1 + hz;
        const bool inside = it < NITEMS && (unsigned)zw < (unsigned)vol.W && (unsigned)zh < (unsigned)vol.H &&
                            (unsigned)zd < (unsigned)vol.D;
        goff[i] = inside ? (((int64_t)zd * vol.H + zh) * vol.W + zw) * in_stride + in_coff + 8 * c8 : -1;
        loff[i] = it < NITEMS ? hv * VP + 8 * c8 : -1;
    }
    bf16x8 pre[IPT];
    auto fetch = [&](int cc0) {
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            pre[i] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
            if (goff[i] >= 0) pre[i] = *reinterpret_cast<const bf16x8*>(in + goff[i] + cc0);
        }
    };
    auto put = [&](uint16_t* buf) {
#pragma unroll
        for (int i = 0; i < IPT; ++i)
            if (loff[i] >= 0) *reinterpret_cast<bf16x8*>(&buf[loff[i]]) = pre[i];
    };
    uint16_t* const hbuf0 = reinterpret_cast<uint16_t*>(smem);
    uint16_t* const hbuf1 = hbuf0 + (DB ? NHALO * VP : 0);
    fetch(0);
    put(hbuf0);
    __syncthreads();
    for (int cc0 = 0, ci = 0; cc0 < Cin; cc0 += CC, ++ci) {
        const uint16_t* halo = (ci & 1) ? hbuf1 : hbuf0;
        const bool more = cc0 + CC < Cin;
        if (DB && more) fetch(cc0 + CC);  // in flight during this chunk's MFMAs
        // B of in-plane group q: slot dzi holds the weights of depth offset dz with s dz = dzi - 1 (so that halo
        // slice z feeds output slice z - dzi); taps past the ninth are zero
        bf16x8 b[3][NT], bn[3][NT];
        auto load_b = [&](int q, bf16x8(&dst)[3][NT]) {
            const int idx = q * TPK + slot;
            const int dx = idx % 3 - 1, dy = idx / 3 - 1;
#pragma unroll
            for (int dzi = 0; dzi < 3; ++dzi) {
                const int dz = s * (dzi - 1);
                const int tap = (dz + 1) * 9 + (dy + 1) * 3 + (dx + 1);
                const uint16_t* wp = wk + (int64_t)(n0 + (lane & 15)) * K + tap * Cin + cc0 + cg;
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    dst[dzi][t] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
                    if (idx < 9) dst[dzi][t] = *reinterpret_cast<const bf16x8*>(wp + (int64_t)t * 16 * K);
                }
            }
        };
        load_b(0, b);
        for (int q = 0; q < NG; ++q) {
            if (q + 1 < NG) load_b(q + 1, bn);
            // operand A: this lane's voxel shifted in-plane by s (dx, dy); padding slots read the centre (their
            // weights are zero)
            const int idx = q * TPK + slot, ii = idx < 9 ? idx : 4;
            const int dx = ii % 3 - 1, dy = ii / 3 - 1;
            const uint16_t* ap = &halo[((rh + 1 + s * dy) * kHaloW + (rw + 1 + s * dx)) * VP + cg];
#pragma unroll
            for (int z = 0; z < HD; ++z) {
                const bf16x8 a = *reinterpret_cast<const bf16x8*>(ap + z * kHaloW * kHaloH * VP);
#pragma unroll
                for (int dzi = 0; dzi < 3; ++dzi) {
                    const int m = z - dzi;
                    if (m >= 0 && m < MT) {
#pragma unroll
                        for (int t = 0; t < NT; ++t)
                            acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[dzi][t], acc[m][t], 0, 0, 0);
                    }
                }
            }
#pragma unroll
            for (int dzi = 0; dzi < 3; ++dzi)
#pragma unroll
                for (int t = 0; t < NT; ++t) b[dzi][t] = bn[dzi][t];
        }
        if (more) {
            if (DB) {
                put((ci & 1) ? hbuf0 : hbuf1);  // the other buffer: every wave finished reading it a chunk ago
            } else {
                __syncthreads();  // single buffer: all waves done with this chunk before it is overwritten
                fetch(cc0 + CC);
                put(hbuf0);
            }
        }
        __syncthreads();
    }
    // epilogue: result row 4 (lane / 16) + r of tile (m, t) is voxel (pw + r, ph + lane / 16) of slice m, channel
    // t * 16 + lane % 16; bias and ReLU here, the tile into LDS as [voxel][channel] (the loop ended on a barrier)
    float* ot = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int ch = t * 16 + (lane & 15);
        const float bn_ = bias ? bias[n0 + ch] : 0.0f;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float y = acc[m][t][r] + bn_;
                if (relu) y = fmaxf(y, 0.0f);
                ot[((m * 8 + ph + (lane >> 4)) * 8 + pw + r) * CH + ch] = y;
            }
    }
    __syncthreads();
    for (int it = threadIdx.x; it < 64 * MT * 2 * NT; it += 256) {
        const int vl = it / (2 * NT), c8 = it - vl * (2 * NT);
        const int zw = w0 + (vl & 7), zh = h0 + ((vl >> 3) & 7), zd = d0 + (vl >> 6);
        if (zw >= vol.W || zh >= vol.H || zd >= vol.D) continue;
        const int64_t v = ((int64_t)zd * vol.H + zh) * vol.W + zw;
        const int n = n0 + 8 * c8;
        const float4 lo = *reinterpret_cast<const float4*>(&ot[vl * CH + 8 * c8]);
        const float4 hi = *reinterpret_cast<const float4*>(&ot[vl * CH + 8 * c8 + 4]);
        float y[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        if (mask) {
            const uint16_t* mp = mask + v * mask_stride + mask_coff + n;
            if (vec) {
                const bf16x8 mk = *reinterpret_cast<const bf16x8*>(mp);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (!(bf2f((uint16_t)mk[e]) > 0.0f)) y[e] = 0.0f;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (!(bf2f(mp[e]) > 0.0f)) y[e] = 0.0f;
            }
        }
        if (out_f32) {
            float* op = reinterpret_cast<float*>(out) + v * out_stride + out_coff + n;
            if (vec) {
                *reinterpret_cast<float4*>(op) = make_float4(y[0], y[1], y[2], y[3]);
                *reinterpret_cast<float4*>(op + 4) = make_float4(y[4], y[5], y[6], y[7]);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) op[e] = y[e];
            }
        } else {
            uint16_t* op = reinterpret_cast<uint16_t*>(out) + v * out_stride + out_coff + n;
            if (vec) {
                bf16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (short)f2bf(y[e]);
                *reinterpret_cast<bf16x8*>(op) = o;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) op[e] = f2bf(y[e]);
            }
        }
    }
}

// Weight gradient: partial sums over parts of the volume,
//   part[b][n][tap][c] = sum_{v in part b} dy[v][n] * in[v + off(tap)][c],  part_db[b][n] = sum_v dy[v][n]
//
// One workgroup (8 waves) owns one part and one pair of 16 output and 16 input channels, for all 27 taps.  It walks
// depth slices of a block of BH rows x WB columns: dy's slice and the input's three slices around it are staged in LDS
// as they lie in memory, 32 bytes (16 channels) per voxel, rows `pitch` = WB + 2 voxels apart.  Slices come by loads
// straight to LDS (no registers), the next step's during this step's MFMAs (a ring of four input slices, two of dy; one
// barrier per step); pads and what lies outside the volume or the channels are lanes out of range, which write zeros.
// The reduction index runs over the block's voxels, pads included, 32 consecutive ones a step.  Both MFMA operands need
// 8 voxels of one channel per lane: the transposing LDS read gives four voxels of 16 channels per 16 lanes (which voxel
// takes which place in K does not matter as long as both operands agree: the first read takes voxels 0-15, the second
// 16-31, each 512 contiguous bytes, free of bank conflicts).  A tap's depth and row offset move the input's address, its
// column offset dy's (by the opposite amount): 9 input and 3 dy fragments per step for 27 MFMAs, where one shifted input
// per tap would be 28.  The input's pad columns are zeros, and so are dy's at the volume's sides.  Waves w and w + 4 (one
// SIMD) take every fourth step of 32 voxels, w for 15 of the taps, w + 4 for the other 12 and the bias gradient (dy
// times a fragment of ones), so that a wave needs little more than the 128 registers that let two workgroups share a CU: 5
// are spilled (29 in the 64-bit form, 15 and 27 with permuted axes), read back where slices are asked for, not between MFMAs.
//
// MFMA-bound in the steps (27 x 16 cycles per 32 voxels and SIMD), with staging and the final sums on top.  A wave per
// (chunk, tap) staging transposed copies of its own had re-read both tensors 27 times:
// 133 -> 21 us for 16 -> 16 channels at 96^3, 265 -> 56 us for 48 -> 16, 51 -> 16 us for 32 -> 32 at 48^3, 54 -> 13 us
// for 64 -> 64 at 12^3.  (Of 45000 cycles at 16 -> 16: steps 19000, waits for slices 7000, asking for them 3600, the first
// slices of a block 5000, final sums 4400, set-up 1800.)
constexpr int kWgThreads = 512, kWgWaves = 8, kWgSplit = 4;  // kWgSplit: waves that share the reduction
constexpr int kWgX = 6, kWgY = 5;               // KiB of an input and of a dy slice that a wave loads, at most
constexpr int kWgTiles = 15;                    // accumulator tiles of a wave: 5 (depth, row) offsets x 3, or 4 x 3
                                                // and the bias gradient
constexpr int kWgPhase = 8;                     // tiles of a wave summed at a time (3 i and 3 i + 1 together)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef __bf16 bf16v4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4s lds_v4s;
typedef __attribute__((address_space(3))) char lds_char;

struct WgradShape {
    int bh, wb;        // rows and columns of a block
    int nyb, nwb;      // blocks along H and W
    int parts;
    int lds;           // bytes
    int64_t slice, row, col;  // voxels from a slice, a row, a column to the next, and the taps' (kPerm)
    int tap_slice, tap_row, tap_col;
};

// KiB of LDS that n voxels take, in whole loads of a wave.
__host__ __device__ constexpr int wgrad_kib(int n) { return (n * 32 + 1023) / 1024; }

__device__ __forceinline__ bf16x8 tr_read(uint32_t at) {
    const v4s a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(size_t)at);
    const v4s b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(size_t)(at + 512));
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

__device__ __attribute__((aligned(16))) const uint32_t kZeros[4] = {0, 0, 0, 0};

// k64: a block's rows span 2 GiB or more: per-lane 64-bit addresses (of a constant zero where a lane is out of range)
// instead of 32-bit offsets into a buffer resource.  kPerm: `vol` is the volume with its axes in another order (sh says how;
// a form of its own, since strides held in registers cost the plain one up to a third).
template <bool k64, bool kPerm>
__global__ __launch_bounds__(kWgThreads, 4) void wgrad_kernel(const uint16_t* __restrict__ in, int in_stride, int in_coff,
                                                              const uint16_t* __restrict__ dy, int dy_stride,
                                                              int dy_coff, float* __restrict__ part,
                                                              float* __restrict__ part_db, Vol vol, int Cin, int Cout,
                                                              WgradShape sh) {
    using off_t = std::conditional_t<k64, int64_t, uint32_t>;
    constexpr off_t kOut = k64 ? (off_t)-1 : (off_t)0x80000000u;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ctiles = (Cin + 15) / 16;
    // workgroup -> (part, pair of channel tiles): consecutive ones, which share slices, on one XCD
    const int pairs = Cout / 16 * ctiles, run = (int)gridDim.x / 8;
    const int unit = (int)(blockIdx.x % 8) * run + (int)(blockIdx.x / 8);
    if (unit >= sh.parts * pairs) return;
    const int my_part = unit / pairs, pair = unit - my_part * pairs;
    const int n0 = pair / ctiles * 16, c0 = pair % ctiles * 16;
    const int pitch = sh.wb + 2, nk = sh.bh * pitch, nks = (nk + 31) / 32;
    const int nbx = wgrad_kib((sh.bh + 2) * pitch + 32), nby = wgrad_kib(nks * 32 + 2);  // KiB of a slice
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)lds, ys = lds0 + 4 * nbx * 1024, ones = ys + 2 * nby * 1024;

    // Lane -> (voxel, 8-channel half) of KiB k of a slice, as a byte offset from the block's first row.
    const int half = lane & 1;
    off_t xo[kWgX], yo[kWgY];
    const char *xbase = nullptr, *ybase = nullptr;
    auto block = [&](int h0, int w0) {
        const int hx = max(h0 - 1, 0);
        xbase = reinterpret_cast<const char*>(in + in_coff + (kPerm ? hx * sh.row : (int64_t)hx * vol.W) * in_stride);
        ybase = reinterpret_cast<const char*>(dy + dy_coff + n0 + (kPerm ? h0 * sh.row : (int64_t)h0 * vol.W) * dy_stride);
#pragma unroll
        for (int k = 0; k < kWgX; ++k) {
            const int v = ((wave + kWgWaves * k) * 64 + lane) >> 1, r = v / pitch, h = h0 - 1 + r, w = w0 + (v - r * pitch);
            const bool ok = r < sh.bh + 2 && v - r * pitch < sh.wb && c0 + 8 * half < Cin && (unsigned)h < (unsigned)vol.H &&
                            w < vol.W;
            if constexpr (kPerm) xo[k] = ok ? (((off_t)(h - hx) * (off_t)sh.row + w * (off_t)sh.col) * in_stride + c0 + 8 * half) * 2 : kOut;
            else xo[k] = ok ? (((off_t)(h - hx) * vol.W + w) * in_stride + c0 + 8 * half) * 2 : kOut;
        }
#pragma unroll
        for (int k = 0; k < kWgY; ++k) {
            const int v = ((wave + kWgWaves * k) * 64 + lane) >> 1, r = v / pitch, h = h0 + r, w = w0 - 1 + (v - r * pitch);
            const bool ok = r < sh.bh && h < vol.H && (unsigned)w < (unsigned)vol.W;
            if constexpr (kPerm) yo[k] = ok ? (((off_t)r * (off_t)sh.row + w * (off_t)sh.col) * dy_stride + 8 * half) * 2 : kOut;
            else yo[k] = ok ? (((off_t)r * vol.W + w) * dy_stride + 8 * half) * 2 : kOut;
        }
    };
    // One KiB: 16 bytes per lane, to consecutive LDS places from `at` on (wave-uniform).
    auto load = [&](const char* src, off_t off, uint32_t at, bool none) {
        if constexpr (k64) {
            const char* a = off < 0 || none ? reinterpret_cast<const char*>(kZeros) : src + off;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(at), "v"(a) : "memory", "m0");
        } else {
            const uint64_t a = reinterpret_cast<uint64_t>(src);
            const u32x4 rs = {(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, none ? 0u : 0x80000000u, 0x00020000u};
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(at), "v"(off), "s"(rs)
                         : "memory", "m0");
        }
    };
    const int64_t xslice = (kPerm ? sh.slice : (int64_t)vol.H * vol.W) * in_stride * 2,
                  yslice = (kPerm ? sh.slice : (int64_t)vol.H * vol.W) * dy_stride * 2;
    auto load_x = [&](int z) {
        const bool none = (unsigned)z >= (unsigned)vol.D;
        const char* const src = xbase + (none ? 0 : z) * xslice;
#pragma unroll
        for (int k = 0; k < kWgX; ++k)
            if (wave + kWgWaves * k < nbx) load(src, xo[k], lds0 + (uint32_t)(((z + 4) % 4 * nbx + wave + kWgWaves * k) * 1024), none);
    };
    auto load_y = [&](int z) {
        const char* const src = ybase + z * yslice;
#pragma unroll
        for (int k = 0; k < kWgY; ++k)
            if (wave + kWgWaves * k < nby) load(src, yo[k], ys + (uint32_t)((z % 2 * nby + wave + kWgWaves * k) * 1024), false);
    };

    f32x4 acc[kWgTiles];
#pragma unroll
    for (int t = 0; t < kWgTiles; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // this lane's byte within a step's first 16 voxels: voxel 4 (lane / 16) + (lane % 16) / 4, channels 4 (lane % 4)
    const uint32_t lane_at = (uint32_t)((4 * (lane >> 4) + ((lane & 15) >> 2)) * 32 + (lane & 3) * 8);
    const int share = wave & (kWgSplit - 1), upper = wave / kWgSplit;  // upper: the last 12 taps
    // Ones, for the bias gradient.  In a volume cut along W, dy's pad columns hold its neighbours' values: a plane of
    // ones with zeros there counts each of the block's own once; else one step's worth serves all.
    const bool cut = sh.nwb > 1;
    for (int i = tid; i < (cut ? nks : 1) * 256; i += kWgThreads)
        reinterpret_cast<uint32_t*>(lds + (ones - lds0))[i] = !cut || (i / 8 < nk && i / 8 % pitch < sh.wb) ? 0x3f803f80u : 0u;
    const bool fifth = !upper || c0 == 0;
    const uint32_t fifth_step = upper && !cut ? 0u : ~0u;

    const int64_t total = (int64_t)sh.nyb * sh.nwb * vol.D;
    const int64_t s0 = total * my_part / sh.parts, s1 = total * (my_part + 1) / sh.parts;
    int z = (int)(s0 % vol.D);
    int blk = (int)(s0 / vol.D);
    bool fresh = true;
    for (int64_t s = s0; s < s1; ++s) {
        if (fresh) {
            __syncthreads();  // the previous block's reads are done
            block(blk % sh.nyb * sh.bh, blk / sh.nyb * sh.wb);
            load_x(z - 1);
            load_x(z);
            load_x(z + 1);
            load_y(z);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's share of the step's slices has landed
        __syncthreads();                                   // and everyone's; the previous step's reads are done too
        fresh = z + 1 == vol.D;
        if (s + 1 < s1 && !fresh) {  // the next step's, into the ring places that no wave reads now
            load_x(z + 2);
            load_y(z + 1);
        }
        uint32_t xb[5];  // this wave's (depth, row) offsets: 0-4, or 5-8
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const int q = upper ? (5 + i) / 3 : i / 3, r = upper ? (5 + i) % 3 : i % 3;
            xb[i] = lds0 + lane_at + (uint32_t)((z + q + 3) % 4 * nbx * 1024 + r * pitch * 32);
        }
        if (upper) xb[4] = ones + lane_at;
        const uint32_t yb = ys + lane_at + 32u + (uint32_t)(z % 2 * nby * 1024);
        for (int ks = share; ks < nks; ks += kWgSplit) {
            const uint32_t o = (uint32_t)ks * 1024u;
            bf16x8 a[3], b[5];
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) a[dx] = tr_read(yb + o - (uint32_t)(dx - 1) * 32u);
#pragma unroll
            for (int i = 0; i < 4; ++i) b[i] = tr_read(xb[i] + o);
            b[4] = tr_read(xb[4] + (o & fifth_step));
            __builtin_amdgcn_sched_barrier(0);  // all reads in flight before the first MFMA waits for its own
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
                    acc[i * 3 + dx] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[dx], b[i], acc[i * 3 + dx], 0, 0, 0);
            if (fifth)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
                    acc[12 + dx] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[dx], b[4], acc[12 + dx], 0, 0, 0);
        }
        if (++z == vol.D) {
            z = 0;
            ++blk;
        }
    }
    // The four waves of a tap half: all tiles through LDS, kWgPhase at a time, each wave sums every fourth tile in the
    // waves' order and stores it.
    //
    // In a block's first row nothing pairs dy's first column with the input's pad before it.  The first wave's sum of the tap
    // beside (the same gradient times the first column) is added times zero instead, so that an infinity or NaN shows.
    float* const red = reinterpret_cast<float*>(lds);  // [upper][tile][share][64 lanes] x 4
    const int c = c0 + (lane & 15), ntiles = upper ? (c0 == 0 ? 14 : 12) : 15;
    float* const pb = part + ((int64_t)my_part * Cout + n0 + 4 * (lane >> 4)) * 27 * Cin + c;
#pragma unroll
    for (int p0 = 0; p0 < kWgTiles; p0 += kWgPhase) {
        __syncthreads();
#pragma unroll
        for (int t = p0; t < p0 + kWgPhase && t < kWgTiles; ++t)
            *reinterpret_cast<f32x4*>(&red[(((upper * kWgPhase + t - p0) * kWgSplit + share) * 64 + lane) * 4]) = acc[t];
        __syncthreads();
        for (int t = p0 + share; t < min(p0 + kWgPhase, ntiles); t += kWgSplit) {
            f32x4 v[kWgSplit];
#pragma unroll
            for (int w = 0; w < kWgSplit; ++w)
                v[w] = *reinterpret_cast<const f32x4*>(&red[(((upper * kWgPhase + t - p0) * kWgSplit + w) * 64 + lane) * 4]);
            const f32x4 b = *reinterpret_cast<const f32x4*>(
                &red[((upper * kWgPhase + t + (t % 3 == 0 ? 1 : 0) - p0) * kWgSplit * 64 + lane) * 4]);
            f32x4 y = ((v[0] + v[1]) + v[2]) + v[3];
#pragma unroll
            for (int r = 0; r < 4; ++r) y[r] = fmaf(0.0f, b[r], y[r]);
            if (upper && t >= 12) {  // dy (unshifted: tile 13) times ones: every column holds the bias gradient's rows
                if (t == 13 && (lane & 15) == 0)
#pragma unroll
                    for (int r = 0; r < 4; ++r) part_db[(int64_t)my_part * Cout + n0 + 4 * (lane >> 4) + r] = y[r];
            } else if (c < Cin) {
                const int i = upper * 5 + t / 3;
                const int tap = kPerm ? i / 3 * sh.tap_slice + i % 3 * sh.tap_row + t % 3 * sh.tap_col : upper * 15 + t;
#pragma unroll
                for (int r = 0; r < 4; ++r) pb[((int64_t)r * 27 + tap) * Cin] = y[r];
            }
        }
    }
}

// The convolution for aligned tensors (launch_brick says which): K steps, operand values and order of accumulation as in
// conv3d_kernel, so the results are the same bits.
//
// A workgroup (WV waves) owns 16 output channels and walks bricks of 16 (W) x WV (H) x MT (D) voxels, depth first.  Its
// weights, all taps and channels, are laid out in LDS once as the MFMA fragments they are read as (kHold: one chunk of
// channels, kept in registers).  A brick's halo, 18 x (WV + 2) x (MT + 2) voxels of one channel chunk, comes by loads
// straight to LDS, in memory order; lanes outside the volume are out of range and write zeros.  kDB: into one of two
// buffers during the previous stage's MFMAs; else into one, hidden by the CU's other workgroups.  Wave w owns row w: its
// operand is 16 voxels along W, read without bank conflicts (32-channel voxels swap their halves every four voxels).  The
// weights are operand A, so that a lane ends with 4 channels of one voxel: bias, ReLU, mask, BF16 and an 8-byte store
// need no LDS.
//
// What bounds it: MFMA issue and LDS reads in the same order of magnitude, loads of 32 of a voxel's bytes at a time with
// many chunks (48 -> 16: MFMAs and LDS alone 32 us, loads alone 33 us), fixed costs on small volumes (launch, weights and
// first halo: about 4 us).  Instructions count as much as MFMAs: addresses advance by scalar adds, places in the halo are
// worked out once.  conv3d_kernel, whose waves fetch every weight fragment through the vector cache, took, and this takes:
// 96^3: 8 -> 16 channels 23.5 and 12.0 us, 16 -> 16 32 and 15.4, 48 -> 16 76 and 43, masked 16 -> 48 125 and 47; 48^3:
// 32 -> 32 16.7 and 9.7, 80 -> 32 41 and 20.2, masked 32 -> 80 66 and 22; 24^3: 112 -> 48 29 and 11.2, masked 48 -> 112 24.5
// and 9.2; 12^3: 64 -> 64 10.0 and 7.5.
struct BrickShape {
    int nx, ny, nz;      // bricks along W, H, D
    int workers;         // workgroups per group of 16 output channels
    int per, extra;      // bricks of each, and how many have one more
};

constexpr int kBrickX = 18;

template <int CC, int WV, int MT>
struct BrickGeom {
    static constexpr int kTaps = 32 / CC, kSteps = (9 + kTaps - 1) / kTaps, kPieces = CC / 8;
    static constexpr int kSlice = (kBrickX * (WV + 2) + 7) / 8 * 8, kHalo = kSlice * (MT + 2);
    static constexpr int kKib = (kHalo * kPieces * 16 + 1023) / 1024;
    static constexpr int kBuf = kKib * 1024;
};

template <int CC, int WV, int MT, bool kHold, bool kDB, bool kMask, bool kF32>
__global__ __launch_bounds__(64 * WV, WV == 4 && kHold ? 3 : 4) void conv3d_brick_kernel(
    const uint16_t* __restrict__ in, int in_stride, const uint16_t* __restrict__ wk, const float* __restrict__ bias,
    char* __restrict__ out, int out_stride, const uint16_t* __restrict__ mask, int mask_stride, Vol vol, int Cin, int ngroups,
    int flip, int relu, BrickShape sh) {
    using G = BrickGeom<CC, WV, MT>;
    constexpr int TPK = G::kTaps, NG = G::kSteps, NP = G::kPieces, KPW = (G::kKib + WV - 1) / WV, HD = MT + 2;
    constexpr int kEs = kF32 ? 4 : 2;
    typedef const __attribute__((address_space(3))) bf16x8 lds_frag;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int unit = (int)((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3));
    if (unit >= sh.workers * ngroups) return;
    const int worker = unit / ngroups, n0 = (unit - worker * ngroups) * 16;
    const int nchunks = kHold ? 1 : Cin / CC;
    const int u0 = worker * sh.per + min(worker, sh.extra);
    int left = sh.per + (worker < sh.extra ? 1 : 0);  // bricks still to be staged
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)lds;
    const uint32_t wlds = lds0 + (uint32_t)((kDB ? 2 : 1) * G::kBuf);
    const int s = flip ? -1 : 1;
    const int g = lane >> 4, slot = g / NP, piece = g % NP;

    auto load = [&](uint64_t src, uint32_t off, uint32_t to) {
        const u32x4 rs = {(uint32_t)__builtin_amdgcn_readfirstlane((int)src),
                          (uint32_t)__builtin_amdgcn_readfirstlane((int)(src >> 32)) & 0xffffu, 0x80000000u, 0x00020000u};
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(to), "v"(off), "s"(rs)
                     : "memory", "m0");
    };
    // this lane's halo pieces: place in the halo (x, y, z; bit 31: outside the volume's rows or columns) and byte offset
    // from the halo's first voxel
    const uint32_t voxel = (uint32_t)in_stride * 2u, row = (uint32_t)vol.W * voxel, slice = row * (uint32_t)vol.H;
    uint32_t at[KPW], off[KPW];
    {
        constexpr int kStep = WV * 64 / NP;  // voxels between a lane's pieces
        const int p = wave * 64 + lane, v = p / NP;
        const int pc = NP == 4 ? (p % NP) ^ (2 * ((v >> 2) & 1)) : p % NP;
        int hz = v / G::kSlice, r = v - hz * G::kSlice;
#pragma unroll
        for (int k = 0; k < KPW; ++k) {
            const int hy = (int)(__umul24((unsigned)r, 3641u) >> 16), hx = r - hy * kBrickX;
            at[k] = (uint32_t)(hx | hy << 8 | (hy < WV + 2 ? hz : 127) << 16);
            off[k] = (uint32_t)hz * slice + (uint32_t)hy * row + (uint32_t)hx * voxel + 16u * pc;
            hz += kStep / G::kSlice;
            r += kStep % G::kSlice;
            if (r >= G::kSlice) {
                r -= G::kSlice;
                ++hz;
            }
        }
    }
    // the brick being staged, and its halo's first voxel (it may lie before the tensor: lanes there are out of range)
    const int c0 = u0 / sh.nz;
    int sz = u0 - c0 * sh.nz, sy = c0 / sh.nx, sx = c0 - sy * sh.nx;
    uint64_t src;
    auto column = [&] {
        src = reinterpret_cast<uint64_t>(in) + (uint64_t)((int64_t)(MT * sz - 1) * slice + (int64_t)(WV * sy - 1) * row +
                                                          (int64_t)(16 * sx - 1) * voxel);
#pragma unroll
        for (int k = 0; k < KPW; ++k) {
            const uint32_t x = (at[k] & 255u) + (uint32_t)(16 * sx - 1), y = (at[k] >> 8 & 255u) + (uint32_t)(WV * sy - 1);
            const bool ok = (x < (uint32_t)vol.W) & (y < (uint32_t)vol.H);
            at[k] = (at[k] & 0x7fffffffu) | (ok ? 0u : 0x80000000u);
        }
    };
    auto stage = [&](int chunk, uint32_t to) {
        const uint32_t lo = sz == 0 ? 65536u : 0u, n = ((uint32_t)min(vol.D - MT * sz + 1, 100) << 16) - lo;
        const uint64_t from = src + (uint64_t)(uint32_t)(chunk * CC * 2);
#pragma unroll
        for (int k = 0; k < KPW; ++k)
            if ((k + 1) * WV <= G::kKib || wave + WV * k < G::kKib)
                load(from, at[k] - lo < n ? off[k] : 0x80000000u, to + (uint32_t)((wave + WV * k) * 1024));
    };
    column();
    // weights, once: fragment (chunk NG + q) 3 + dzi, 16 bytes per lane
    {
        const uint32_t wl = (uint32_t)((lane & 15) * 27 * Cin + slot * Cin + 8 * piece) * 2u;
        for (int f = wave; f < nchunks * NG * 3; f += WV) {
            const int cq = f / 3, dzi = f - 3 * cq, ch = cq / NG, q = cq - ch * NG;
            const int tap = (s * (dzi - 1) + 1) * 9 + q * TPK;
            load(reinterpret_cast<uint64_t>(wk), q * TPK + slot < 9 ? wl + (uint32_t)((n0 * 27 + tap) * Cin + ch * CC) * 2u : 0x80000000u,
                 wlds + (uint32_t)f * 1024u);
        }
    }
    uint32_t aoff[NG];
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        const int idx = q * TPK + slot, ii = idx < 9 ? idx : 4, t3 = (int)(__umul24((unsigned)ii, 86u) >> 8);
        const int v = (wave + 1 + s * (t3 - 1)) * kBrickX + (lane & 15) + 1 + s * (ii - 3 * t3 - 1);
        aoff[q] = lds0 + (uint32_t)((v * NP + (NP == 4 ? piece ^ (2 * ((v >> 2) & 1)) : piece)) * 16);
    }
    f32x4 bs = {0.0f, 0.0f, 0.0f, 0.0f};
    if (bias) bs = f32x4{bias[n0 + 4 * g], bias[n0 + 4 * g + 1], bias[n0 + 4 * g + 2], bias[n0 + 4 * g + 3]};
    const uint32_t olane = (uint32_t)((lane & 15) * out_stride + 4 * g) * kEs, mlane = (uint32_t)((lane & 15) * mask_stride + 4 * g) * 2u;
    const int64_t HW = (int64_t)vol.H * vol.W, oslice = HW * out_stride * kEs, mslice = HW * mask_stride * 2;

    bf16x8 hold[kHold ? NG * 3 : 1];
    f32x4 acc[MT];
    v4s mk[MT];
    int chunk = 0, nc = 0;       // the chunk at work, the next
    int d0 = 0, oy = 0, ox = 0;  // the brick at work
    uint32_t buf = lds0;
    bool have = false;
    char* op = nullptr;
    const char* mp = nullptr;
    bool inside = false;
    auto compute = [&] {
        if (kMask && chunk + 1 == nchunks) {
            const char* a = mp;
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                if (inside) mk[m] = *reinterpret_cast<const v4s*>(a + mlane);
                if (d0 + m + 1 < vol.D) a += mslice;
            }
        }
        if (chunk == 0) {
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        const uint32_t wb = wlds + (uint32_t)(chunk * NG * 3 * 1024 + lane * 16);
#pragma unroll
        for (int q = 0; q < NG; ++q) {
            bf16x8 b[3], a[HD];
            const uint32_t aq = aoff[q] + (kDB ? buf - lds0 : 0u);
#pragma unroll
            for (int dzi = 0; dzi < 3; ++dzi) b[dzi] = kHold ? hold[kHold ? q * 3 + dzi : 0] : *(lds_frag*)(size_t)(wb + (uint32_t)((q * 3 + dzi) * 1024));
#pragma unroll
            for (int z = 0; z < HD; ++z) a[z] = *(lds_frag*)(size_t)(aq + (uint32_t)(z * G::kSlice * NP * 16));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int z = 0; z < HD; ++z)
#pragma unroll
                for (int dzi = 0; dzi < 3; ++dzi) {
                    const int m = z - dzi;
                    if (m >= 0 && m < MT) acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[dzi], a[z], acc[m], 0, 0, 0);
                }
        }
    };
    auto store = [&] {
        if (inside) {
            char* a = op;
            if (relu) {
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[m][e] = fmaxf(acc[m][e] + bs[e], 0.0f);
            } else {
#pragma unroll
                for (int m = 0; m < MT; ++m) acc[m] += bs;
            }
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                f32x4 r = acc[m];
                if (kMask)
#pragma unroll
                    for (int e = 0; e < 4; ++e) r[e] = bf2f((uint16_t)mk[m][e]) > 0.0f ? r[e] : 0.0f;
                if (d0 + m < vol.D) {
                    if constexpr (kF32)
                        *reinterpret_cast<f32x4*>(a + olane) = r;
                    else
                        *reinterpret_cast<v4s*>(a + olane) = __builtin_bit_cast(v4s, __builtin_convertvector(r, bf16v4));
                }
                a += oslice;
            }
        }
    };
    // what was staged becomes what is at work; the next stage's place
    auto advance = [&] {
        chunk = nc;
        if (chunk == 0) {
            d0 = MT * sz;
            oy = WV * sy + wave;
            ox = 16 * sx + (lane & 15);
            inside = (oy < vol.H) & (ox < vol.W);
            const int64_t v0 = ((int64_t)d0 * vol.H + oy) * vol.W + 16 * sx;
            op = out + (v0 * out_stride + n0) * kEs;
            if (kMask) mp = reinterpret_cast<const char*>(mask + v0 * mask_stride + n0);
        }
        if (++nc == nchunks) {
            nc = 0;
            --left;
            src += (uint64_t)slice * MT;
            if (++sz == sh.nz) {
                sz = 0;
                if (++sx == sh.nx) {
                    sx = 0;
                    ++sy;
                }
                column();
            }
        }
        have = true;
    };
    if constexpr (kDB) {
        uint32_t nbuf = lds0;  // where the next stage goes
        for (;;) {
            const bool more = left > 0;
            if (more) stage(nc, nbuf);
            if (have) compute();
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (have && chunk + 1 == nchunks) store();
            if (!more) break;
            __syncthreads();
            if constexpr (kHold)
                if (!have)
#pragma unroll
                    for (int i = 0; i < NG * 3; ++i) hold[i] = *(lds_frag*)(size_t)(wlds + (uint32_t)(i * 1024 + lane * 16));
            buf = nbuf;
            nbuf = lds0 + lds0 + G::kBuf - nbuf;
            advance();
        }
    } else {
        for (;;) {
            const bool more = left > 0;
            if (more) stage(nc, lds0);
            if (have && chunk + 1 == nchunks) store();
            if (!more) break;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if constexpr (kHold)
                if (!have)
#pragma unroll
                    for (int i = 0; i < NG * 3; ++i) hold[i] = *(lds_frag*)(size_t)(wlds + (uint32_t)(i * 1024 + lane * 16));
            advance();
            compute();
            __syncthreads();
        }
    }
}

// What the weight gradient was formed from, as it was walked (tap_* and the strides of `sh` set in either order of axes).
struct WgradTensors {
    const uint16_t* in;
    const uint16_t* dy;
    int in_stride, dy_stride, Cin;
    Vol vol;
    WgradShape sh;
};

// A part's sum that is not finite, again from its terms in float64: with its zero pads wgrad_kernel multiplies an infinity or
// NaN of a block's side columns by a zero that is no term.  The terms are dy[v][n] * in[v + off(tap)][c], with zeros outside
// the volume; tap < 0: dy[v][n].  Every second row, from `row` on, until the sum is a NaN.
//
// A block's terms are those whose input column it holds; the one past the volume's side goes with the side's own.
__device__ __forceinline__ double wgrad_terms(const WgradTensors& x, int part, int n, int tap, int c, int row) {
    const WgradShape& sh = x.sh;
    const Vol& vol = x.vol;
    const int oz = tap < 0 ? 0 : tap / sh.tap_slice % 3 - 1, oy = tap < 0 ? 0 : tap / sh.tap_row % 3 - 1,
              u = tap < 0 ? 0 : tap / sh.tap_col % 3 - 1;
    const int64_t total = (int64_t)sh.nyb * sh.nwb * vol.D;
    const int64_t s0 = total * part / sh.parts, s1 = total * (part + 1) / sh.parts;
    double sum = 0.0;
    for (int64_t s = s0; s < s1; ++s) {
        const int z = (int)(s % vol.D), blk = (int)(s / vol.D);
        const int h0 = blk % sh.nyb * sh.bh, h1 = min(h0 + sh.bh, vol.H), w0 = blk / sh.nyb * sh.wb, w1 = min(w0 + sh.wb, vol.W);
        const int from = w0 == 0 ? 0 : w0 - u, to = w1 == vol.W ? vol.W : w1 - u;
        for (int h = h0 + ((row ^ (int)s) & 1); h < h1; h += 2) {
            const bool inside = (unsigned)(z + oz) < (unsigned)vol.D && (unsigned)(h + oy) < (unsigned)vol.H;
            const int64_t at = z * sh.slice + h * sh.row;
            const uint16_t* const yp = x.dy + at * x.dy_stride + n;
            const uint16_t* const xp = x.in + (at + oz * sh.slice + oy * sh.row + u * sh.col) * x.in_stride + c;
            for (int w = from; w < to && sum == sum; w += 4) {
                float g[4], q[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int64_t wk = min(w + k, to - 1);
                    g[k] = bf2f(yp[wk * sh.col * x.dy_stride]);
                    q[k] = tap < 0 ? 1.0f : inside && (unsigned)((int)wk + u) < (unsigned)vol.W ? bf2f(xp[wk * sh.col * x.in_stride]) : 0.0f;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (w + k < to) sum += (double)g[k] * q[k];
            }
        }
    }
    return sum;
}

// dw[i] = sum_b part[b][i], i over Cout * K, and the same for db (the blocks past the first nwb): 32 outputs per
// workgroup, the parts split over 8 thread rows (row r sums parts r, r + 8, ... in order), the 8 row sums added in row
// order: deterministic.  Sums that are not finite: the parts that are not, again from their terms (16 -> 16 channels at 96^3
// with one infinity: 0.3 to 0.7 ms; 376 when one thread formed a whole sum, 0.035 without the infinity).
__global__ __launch_bounds__(256) void reduce_parts_kernel(const float* __restrict__ part, const float* __restrict__ part_db,
                                                           int nparts, int64_t nw, int nwb, int nb,
                                                           float* __restrict__ dw, float* __restrict__ db, WgradTensors x) {
    __shared__ float red[8][32];
    const int col = threadIdx.x & 31, row = threadIdx.x >> 5;
    const bool is_db = (int)blockIdx.x >= nwb;
    const float* src = is_db ? part_db : part;
    const int64_t n = is_db ? nb : nw;
    const int64_t i = (int64_t)(blockIdx.x - (is_db ? nwb : 0)) * 32 + col;
    float s = 0.0f;
    if (i < n) {
        // eight loads in flight (one at a time, 256 parts of 6912 sums took 10.8 us, all latency)
        const float* p = src + (int64_t)row * n + i;
        int b = row;
        for (; b + 56 < nparts; b += 64, p += 64 * n) {
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = p[8 * j * n];
#pragma unroll
            for (int j = 0; j < 8; ++j) s += v[j];
        }
        for (; b < nparts; b += 8, p += 8 * n) s += *p;
    }
    red[row][col] = s;
    __syncthreads();
    if (row > 1) return;
    float t = red[0][col];
#pragma unroll
    for (int r = 1; r < 8; ++r) t += red[r][col];
    if (i < n && !(fabsf(t) < __builtin_inff())) {
        double sum = 0.0;
        const int k = (int)(i % (27 * x.Cin));
        const int ch = is_db ? (int)i : (int)(i / (27 * x.Cin)), tap = is_db ? -1 : k / x.Cin, c = is_db ? 0 : k % x.Cin;
        for (int b0 = 0; b0 < nparts && sum == sum; b0 += 8) {
            unsigned bad = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float v = src[(int64_t)min(b0 + j, nparts - 1) * n + i];
                const bool finite = fabsf(v) < __builtin_inff();
                if (b0 + j < nparts) sum += finite && row == 0 ? v : 0.0f, bad |= finite ? 0u : 1u << j;
            }
            for (; bad; bad &= bad - 1) sum += wgrad_terms(x, b0 + __builtin_ctz(bad), ch, tap, c, row);
        }
        t = (float)(sum + __shfl_xor(sum, 32));
    }
    if (row == 0 && i < n) (is_db ? db : dw)[i] = t;
}

// wt[ci][tap][co] = w[co][tap][ci] (bf16), the weights of the input-gradient convolution.
// Weights of up to kTransposes layers in one launch: a layer's blocks follow the previous layer's.
constexpr int kTransposes = 16;
struct TransposeList {
    const uint16_t* w[kTransposes];
    uint16_t* wt[kTransposes];
    int cin[kTransposes], cout[kTransposes];
    unsigned end[kTransposes];  // first block past the layer's
};
__global__ void transpose_w_kernel(TransposeList l) {
    int k = 0;
    while (blockIdx.x >= l.end[k]) ++k;
    const int Cin = l.cin[k], Cout = l.cout[k];
    const int64_t i = (int64_t)(blockIdx.x - (k ? l.end[k - 1] : 0u)) * blockDim.x + threadIdx.x;
    const int64_t n = (int64_t)Cout * 27 * Cin;
    if (i >= n) return;
    const int co = (int)(i / (27 * Cin)), rem = (int)(i % (27 * Cin)), tap = rem / Cin, ci = rem % Cin;
    l.wt[k][((int64_t)ci * 27 + tap) * Cout + co] = l.w[k][i];
}

// 2x average pooling: out[d][h][w][c] = mean of the 8 children.
__global__ void avgpool2_kernel(const uint16_t* __restrict__ in, int in_stride, int in_coff, uint16_t* __restrict__ out,
                                int out_stride, int out_coff, Vol vo, int C) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n = (int64_t)vo.D * vo.H * vo.W * C;
    if (i >= n) return;
    const int c = (int)(i % C);
    const int64_t v = i / C;
    const int w = (int)(v % vo.W), h = (int)((v / vo.W) % vo.H), d = (int)(v / ((int64_t)vo.W * vo.H));
    const int Hi = 2 * vo.H, Wi = 2 * vo.W;
    float s = 0.0f;
    for (int q = 0; q < 8; ++q) {
        const int64_t vi = ((int64_t)(2 * d + (q >> 2)) * Hi + (2 * h + ((q >> 1) & 1))) * Wi + (2 * w + (q & 1));
        s += bf2f(in[vi * in_stride + in_coff + c]);
    }
    out[v * out_stride + out_coff + c] = f2bf(0.125f * s);
}

// Gradient of the 2x average pooling: each child gets 1/8 of its parent's gradient, optionally added.
__global__ void avgpool2_bwd_kernel(const uint16_t* __restrict__ gout, int gout_stride, int gout_coff,
                                    uint16_t* __restrict__ gin, int gin_stride, int gin_coff, Vol vi, int C,
                                    int accumulate) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n = (int64_t)vi.D * vi.H * vi.W * C;
    if (i >= n) return;
    const int c = (int)(i % C);
    const int64_t v = i / C;
    const int w = (int)(v % vi.W), h = (int)((v / vi.W) % vi.H), d = (int)(v / ((int64_t)vi.W * vi.H));
    const int64_t vp = ((int64_t)(d >> 1) * (vi.H >> 1) + (h >> 1)) * (vi.W >> 1) + (w >> 1);
    float g = 0.125f * bf2f(gout[vp * gout_stride + gout_coff + c]);
    uint16_t* dst = gin + v * gin_stride + gin_coff + c;
    if (accumulate) g += bf2f(*dst);
    *dst = f2bf(g);
}

// 2x nearest upsampling (forward) into a channel slice.
__global__ void upsample2_kernel(const uint16_t* __restrict__ in, int in_stride, int in_coff, uint16_t* __restrict__ out,
                                 int out_stride, int out_coff, Vol vo, int C) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n = (int64_t)vo.D * vo.H * vo.W * C;
    if (i >= n) return;
    const int c = (int)(i % C);
    const int64_t v = i / C;
    const int w = (int)(v % vo.W), h = (int)((v / vo.W) % vo.H), d = (int)(v / ((int64_t)vo.W * vo.H));
    const int64_t vp = ((int64_t)(d >> 1) * (vo.H >> 1) + (h >> 1)) * (vo.W >> 1) + (w >> 1);
    out[v * out_stride + out_coff + c] = in[vp * in_stride + in_coff + c];
}

// Gradient of the 2x nearest upsampling: sum over the 8 children (fixed order), optionally masked by a ReLU output.
__global__ void upsample2_bwd_kernel(const uint16_t* __restrict__ gout, int gout_stride, int gout_coff,
                                     uint16_t* __restrict__ gin, int gin_stride, int gin_coff,
                                     const uint16_t* __restrict__ mask, int mask_stride, int mask_coff, Vol vi, int C) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n = (int64_t)vi.D * vi.H * vi.W * C;
    if (i >= n) return;
    const int c = (int)(i % C);
    const int64_t v = i / C;
    const int w = (int)(v % vi.W), h = (int)((v / vi.W) % vi.H), d = (int)(v / ((int64_t)vi.W * vi.H));
    const int Ho = 2 * vi.H, Wo = 2 * vi.W;
    float s = 0.0f;
    for (int q = 0; q < 8; ++q) {
        const int64_t vo = ((int64_t)(2 * d + (q >> 2)) * Ho + (2 * h + ((q >> 1) & 1))) * Wo + (2 * w + (q & 1));
        s += bf2f(gout[vo * gout_stride + gout_coff + c]);
    }
    if (mask && !(bf2f(mask[v * mask_stride + mask_coff + c]) > 0.0f)) s = 0.0f;
    gin[v * gin_stride + gin_coff + c] = f2bf(s);
}

// Vector forms of the upsampling, the pooling gradient and add_mask: 8 BF16 channels (16 bytes) per thread, for
// slices whose channel count, stride and offset are multiples of 8.  Same arithmetic in the same order per
// element, so the results are bitwise those of the scalar kernels.  Thread (x, y) of block (bx, by, d): x over
// (w, channel group), h = 4 by + y, d = depth of the volume the thread writes.
__device__ __forceinline__ void unpack8(const uint4& r, float (&f)[8]) {
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f[2 * j] = __uint_as_float(w[j] << 16);
        f[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
    }
}

__device__ __forceinline__ uint4 pack8(const float (&f)[8]) {
    uint32_t w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = (uint32_t)f2bf(f[2 * j]) | ((uint32_t)f2bf(f[2 * j + 1]) << 16);
    return make_uint4(w[0], w[1], w[2], w[3]);
}

struct V8Pos {
    int d, h, w, c;
    bool ok;
};

__device__ __forceinline__ V8Pos v8_pos(const Vol& v, int C8) {
    V8Pos p;
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    p.h = blockIdx.y * blockDim.y + threadIdx.y;
    p.d = blockIdx.z;
    p.w = x / C8;
    p.c = (x - p.w * C8) * 8;
    p.ok = x < v.W * C8 && p.h < v.H;
    return p;
}

__global__ void avgpool2_bwd_v8_kernel(const uint16_t* __restrict__ gout, int gout_stride, int gout_coff,
                                       uint16_t* __restrict__ gin, int gin_stride, int gin_coff, Vol vi, int C8,
                                       int accumulate) {
    const V8Pos p = v8_pos(vi, C8);
    if (!p.ok) return;
    const int64_t v = ((int64_t)p.d * vi.H + p.h) * vi.W + p.w;
    const int64_t vp = ((int64_t)(p.d >> 1) * (vi.H >> 1) + (p.h >> 1)) * (vi.W >> 1) + (p.w >> 1);
    float g[8];
    unpack8(*reinterpret_cast<const uint4*>(gout + vp * gout_stride + gout_coff + p.c), g);
#pragma unroll
    for (int j = 0; j < 8; ++j) g[j] = 0.125f * g[j];
    uint4* dst = reinterpret_cast<uint4*>(gin + v * gin_stride + gin_coff + p.c);
    if (accumulate) {
        float a[8];
        unpack8(*dst, a);
#pragma unroll
        for (int j = 0; j < 8; ++j) g[j] += a[j];
    }
    *dst = pack8(g);
}

__global__ void upsample2_v8_kernel(const uint16_t* __restrict__ in, int in_stride, int in_coff,
                                    uint16_t* __restrict__ out, int out_stride, int out_coff, Vol vo, int C8) {
    const V8Pos p = v8_pos(vo, C8);
    if (!p.ok) return;
    const int64_t v = ((int64_t)p.d * vo.H + p.h) * vo.W + p.w;
    const int64_t vp = ((int64_t)(p.d >> 1) * (vo.H >> 1) + (p.h >> 1)) * (vo.W >> 1) + (p.w >> 1);
    *reinterpret_cast<uint4*>(out + v * out_stride + out_coff + p.c) =
        *reinterpret_cast<const uint4*>(in + vp * in_stride + in_coff + p.c);
}

__global__ void upsample2_bwd_v8_kernel(const uint16_t* __restrict__ gout, int gout_stride, int gout_coff,
                                        uint16_t* __restrict__ gin, int gin_stride, int gin_coff,
                                        const uint16_t* __restrict__ mask, int mask_stride, int mask_coff, Vol vi,
                                        int C8) {
    const V8Pos p = v8_pos(vi, C8);
    if (!p.ok) return;
    const int Ho = 2 * vi.H, Wo = 2 * vi.W;
    float s[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) s[j] = 0.0f;
    for (int q = 0; q < 8; ++q) {
        const int64_t vo = ((int64_t)(2 * p.d + (q >> 2)) * Ho + (2 * p.h + ((q >> 1) & 1))) * Wo + (2 * p.w + (q & 1));
        float f[8];
        unpack8(*reinterpret_cast<const uint4*>(gout + vo * gout_stride + gout_coff + p.c), f);
#pragma unroll
        for (int j = 0; j < 8; ++j) s[j] += f[j];
    }
    const int64_t v = ((int64_t)p.d * vi.H + p.h) * vi.W + p.w;
    if (mask) {
        float m[8];
        unpack8(*reinterpret_cast<const uint4*>(mask + v * mask_stride + mask_coff + p.c), m);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (!(m[j] > 0.0f)) s[j] = 0.0f;
    }
    *reinterpret_cast<uint4*>(gin + v * gin_stride + gin_coff + p.c) = pack8(s);
}

// add_mask over V voxels x C8 channel groups (V * C8 < 2^31, so the index split is a 32-bit division)
__global__ void add_mask_v8_kernel(const uint16_t* __restrict__ a, int a_stride, int a_coff,
                                   const uint16_t* __restrict__ b, int b_stride, int b_coff,
                                   const uint16_t* __restrict__ mask, int m_stride, int m_coff,
                                   uint16_t* __restrict__ g, int g_stride, int g_coff, int n, int C8) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int v32 = i / C8;
    const int c = (i - v32 * C8) * 8;
    const int64_t v = v32;
    float x[8], y[8];
    unpack8(*reinterpret_cast<const uint4*>(a + v * a_stride + a_coff + c), x);
    unpack8(*reinterpret_cast<const uint4*>(b + v * b_stride + b_coff + c), y);
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] += y[j];
    if (mask) {
        float m[8];
        unpack8(*reinterpret_cast<const uint4*>(mask + v * m_stride + m_coff + c), m);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (!(m[j] > 0.0f)) x[j] = 0.0f;
    }
    *reinterpret_cast<uint4*>(g + v * g_stride + g_coff + c) = pack8(x);
}

// g[v][c] = (a[v][c] + b[v][c]) * (mask[v][c] > 0)   (bf16 slices)
__global__ void add_mask_kernel(const uint16_t* __restrict__ a, int a_stride, int a_coff, const uint16_t* __restrict__ b,
                                int b_stride, int b_coff, const uint16_t* __restrict__ mask, int m_stride, int m_coff,
                                uint16_t* __restrict__ g, int g_stride, int g_coff, int64_t V, int C) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= V * C) return;
    const int c = (int)(i % C);
    const int64_t v = i / C;
    float s = bf2f(a[v * a_stride + a_coff + c]) + bf2f(b[v * b_stride + b_coff + c]);
    if (mask && !(bf2f(mask[v * m_stride + m_coff + c]) > 0.0f)) s = 0.0f;
    g[v * g_stride + g_coff + c] = f2bf(s);
}

// Residual prediction and MSE: pred = base + net (FP32 [V][2]); loss parts per block; grad = 2 (pred - target) / n
// written as BF16 into a [V][gstride] buffer (first 2 channels; the padded channels get 0).  kVec: pairs are 8-byte
// accesses and gstride is a multiple of 8: a wave writes its 64 rows as consecutive 16-byte pieces, those with the two
// channels from the lane that has them (96^3 voxels, 16 channels: 44 us with a 2-byte store per channel, 18 us so; bound by
// the 64-byte rows of net).
template <bool kVec>
__global__ void mse_kernel(const float* __restrict__ net, int net_stride, const float* __restrict__ base,
                           const float* __restrict__ target, int64_t V, uint16_t* __restrict__ grad, int gstride,
                           float* __restrict__ pred, float* __restrict__ loss_part) {
    __shared__ float red[256];
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const float scale = 2.0f / (float)(2 * V);
    float l = 0.0f;
    if constexpr (kVec) {
        uint32_t g = 0;
        if (v < V) {
            const float2 n = *reinterpret_cast<const float2*>(net + v * net_stride);
            const float2 b = reinterpret_cast<const float2*>(base)[v], t = reinterpret_cast<const float2*>(target)[v];
            const float2 p = make_float2(b.x + n.x, b.y + n.y), e = make_float2(p.x - t.x, p.y - t.y);
            if (pred) reinterpret_cast<float2*>(pred)[v] = p;
            l += e.x * e.x;
            l += e.y * e.y;
            g = (uint32_t)f2bf(scale * e.x) | (uint32_t)f2bf(scale * e.y) << 16;
        }
        if (grad) {
            const int lane = threadIdx.x & 63, np = gstride / 8;  // pieces of a row
            const int64_t v0 = v - lane;
            uint4* dst = reinterpret_cast<uint4*>(grad + v0 * gstride);
            for (int i = lane; i < 64 * np; i += 64) {
                const int from = i / np;
                const uint32_t x = __shfl(g, from);
                if (v0 + from < V) dst[i] = make_uint4(from * np == i ? x : 0u, 0u, 0u, 0u);
            }
        }
    } else if (v < V) {
        for (int c = 0; c < gstride || c < 2; ++c) {
            if (c < 2) {
                const float p = base[2 * v + c] + net[v * net_stride + c];
                const float e = p - target[2 * v + c];
                if (pred) pred[2 * v + c] = p;
                l += e * e;
                if (grad) grad[v * gstride + c] = f2bf(scale * e);
            } else if (grad) {
                grad[v * gstride + c] = 0;
            }
        }
    }
    red[threadIdx.x] = l;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss_part[blockIdx.x] = red[0];
}

// Adam with bias correction on FP32 master weights; refreshes the BF16 copy.
__global__ void adam_kernel(float* __restrict__ w, float* __restrict__ m, float* __restrict__ vv,
                            const float* __restrict__ g, uint16_t* __restrict__ wbf, int64_t n, float lr, float b1,
                            float b2, float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * vv[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    vv[i] = vi;
    const float wi = w[i] - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
    w[i] = wi;
    if (wbf) wbf[i] = f2bf(wi);
}

__global__ void f32_to_bf16_kernel(const float* __restrict__ x, uint16_t* __restrict__ y, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = f2bf(x[i]);
}


// ---- compounding features
// part[b] = sum over the block's voxels of |sum_a y_a[v]|^2   (y complex64 [A][V])
__global__ __launch_bounds__(256) void sumsq_kernel(const float2* __restrict__ y, int A, int64_t V,
                                                    float* __restrict__ part) {
    __shared__ float red[256];
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    float l = 0.0f;
    if (v < V) {
        float re = 0.0f, im = 0.0f;
        for (int a = 0; a < A; ++a) {
            const float2 z = y[(int64_t)a * V + v];
            re += z.x;
            im += z.y;
        }
        l = re * re + im * im;
    }
    red[threadIdx.x] = l;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// scale[0] = sqrt(sum(part) / V) (the RMS), scale[1] = 1 / scale[0] (0 for an all-zero input); one block.
__global__ __launch_bounds__(256) void rms_kernel(const float* __restrict__ part, int nparts, int64_t V,
                                                  float* __restrict__ scale) {
    __shared__ double red[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < nparts; i += 256) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const float rms = (float)sqrt(red[0] / (double)V);
        scale[0] = rms;
        scale[1] = rms > 0.0f ? 1.0f / rms : 0.0f;
    }
}

// x[v][2a + {0,1}] = bf16(y_a[v] / rms), x[v][c >= 2A] = 0; base[v] = gain * sum_a y_a[v] / rms
__global__ __launch_bounds__(256) void features_kernel(const float2* __restrict__ y, int A, int64_t V, float gain,
                                                       const float* __restrict__ scale, uint16_t* __restrict__ x,
                                                       int cin, float* __restrict__ base) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= V) return;
    const float inv = scale[1];
    float re = 0.0f, im = 0.0f;
    for (int a = 0; a < A; ++a) {
        const float2 z = y[(int64_t)a * V + v];
        re += z.x;
        im += z.y;
        x[v * cin + 2 * a] = f2bf(z.x * inv);
        x[v * cin + 2 * a + 1] = f2bf(z.y * inv);
    }
    for (int c = 2 * A; c < cin; ++c) x[v * cin + c] = 0;
    if (base) {
        base[2 * v] = gain * re * inv;
        base[2 * v + 1] = gain * im * inv;
    }
}

// out[v] = y[v] * scale[k]: k = 1 normalises a complex64 volume, k = 0 restores physical units
__global__ void rescale_kernel(const float2* __restrict__ y, int64_t V, const float* __restrict__ scale, int k,
                               float2* __restrict__ out) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= V) return;
    const float s = scale[k];
    const float2 z = y[v];
    out[v] = make_float2(z.x * s, z.y * s);
}

// out[v] = (base[v] + net[v][0:2]) * rms: the network's estimate in the beamformer's units (complex64)
__global__ void compound_output_kernel(const float* __restrict__ net, int net_stride, const float* __restrict__ base,
                                       int64_t V, const float* __restrict__ scale, float2* __restrict__ out) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= V) return;
    const float s = scale[0];
    out[v] = make_float2((base[2 * v] + net[v * net_stride]) * s, (base[2 * v + 1] + net[v * net_stride + 1]) * s);
}

}  // namespace learn

// ------------------------------------------------------------------ C ABI
namespace {
thread_local const char* g_learn_err = "";
int lfail(int st, const char* msg) {
    g_learn_err = msg;
    return st;
}
bool al(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }
unsigned blocks_for(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

// The 8-channel vector kernels apply when every slice is 16-byte aligned (pointer, stride and offset) and the
// volume fits their grid (x = W * C / 8 in 64-thread blocks, y = H in blocks of 4, z = D).
bool v8_slice(const void* p, int stride, int coff) {
    return p == nullptr || (reinterpret_cast<uintptr_t>(p) % 16 == 0 && stride % 8 == 0 && coff % 8 == 0);
}

bool v8_volume(int D, int H, int W, int c) {
    return c % 8 == 0 && (int64_t)W * (c / 8) < (int64_t)1 << 30 && D <= 65535 && (H + 3) / 4 <= 65535;
}

dim3 v8_grid(int D, int H, int W, int c) {
    return dim3((unsigned)(((int64_t)W * (c / 8) + 63) / 64), (unsigned)((H + 3) / 4), (unsigned)D);
}

const dim3 kV8Block(64, 4, 1);
bool slices_ok(int s1, int o1, int s2, int o2, int c) { return c >= 1 && o1 >= 0 && o2 >= 0 && s1 >= o1 + c && s2 >= o2 + c; }
bool even_dims(int D, int H, int W) { return D >= 2 && H >= 2 && W >= 2 && D % 2 == 0 && H % 2 == 0 && W % 2 == 0; }
int launch_status(const char* what) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return lfail(DAS_EHIP, what);
    return DAS_OK;
}

// Workgroup shape: MT depth slices and NT channel tiles (NT divides Cout / 16).  Candidates in order of
// decreasing work per workgroup; the first with at least 512 workgroups (two per CU) is used, else the one
// with the most workgroups (small volumes).  The input chunk is the largest of 32, 16, 8 channels dividing Cin.
template <int MT, int NT, int CC>
void launch_conv_t(int ngroups, int out_f32, const learn::Vol& vol, hipStream_t s, const uint16_t* x, int in_stride,
                   int in_coff, const uint16_t* w, const float* bias, void* out, int out_stride, int out_coff,
                   const uint16_t* mk, int mask_stride, int mask_coff, int cin, int flip, int relu) {
    const unsigned nb = (unsigned)(((vol.W + 7) / 8) * ((vol.H + 7) / 8) * ((vol.D + MT - 1) / MT));
    // 16-byte output (and mask) accesses: 8 channels of a voxel start on a 16-byte boundary
    const int ea = out_f32 ? 4 : 8;
    const bool vec = reinterpret_cast<uintptr_t>(out) % 16 == 0 && out_stride % ea == 0 && out_coff % ea == 0 &&
                     (!mk || (reinterpret_cast<uintptr_t>(mk) % 16 == 0 && mask_stride % 8 == 0 && mask_coff % 8 == 0));
    // double-buffered halo only for small launches (few workgroups: latency-bound), which take the 1 x 1 shape;
    // on large ones the second buffer costs occupancy (d0a at 96^3: 84 -> 94 us; the 24^3 and 12^3 layers gain
    // ~1 us each).  Other shapes are not instantiated double-buffered (compile time).
    if constexpr (MT == 1 && NT == 1) {
        if (cin > CC && (int64_t)nb * ngroups <= 768) {
            hipLaunchKernelGGL((learn::conv3d_kernel<MT, NT, CC, true>), dim3(nb, ngroups), dim3(256), 0, s, x,
                               in_stride, in_coff, w, bias, out, out_stride, out_coff, out_f32, mk, mask_stride,
                               mask_coff, vol, cin, flip, relu, (int)vec);
            return;
        }
    }
    hipLaunchKernelGGL((learn::conv3d_kernel<MT, NT, CC, false>), dim3(nb, ngroups), dim3(256), 0, s, x, in_stride,
                       in_coff, w, bias, out, out_stride, out_coff, out_f32, mk, mask_stride, mask_coff, vol, cin,
                       flip, relu, (int)vec);
}

template <int MT, int NT>
void launch_conv_cc(int ngroups, int out_f32, const learn::Vol& vol, hipStream_t s, const uint16_t* x,
                    int in_stride, int in_coff, const uint16_t* w, const float* bias, void* out, int out_stride,
                    int out_coff, const uint16_t* mk, int mask_stride, int mask_coff, int cin, int flip, int relu) {
    if (cin % 32 == 0)
        launch_conv_t<MT, NT, 32>(ngroups, out_f32, vol, s, x, in_stride, in_coff, w, bias, out, out_stride, out_coff,
                                  mk, mask_stride, mask_coff, cin, flip, relu);
    else if (cin % 16 == 0)
        launch_conv_t<MT, NT, 16>(ngroups, out_f32, vol, s, x, in_stride, in_coff, w, bias, out, out_stride, out_coff,
                                  mk, mask_stride, mask_coff, cin, flip, relu);
    else
        launch_conv_t<MT, NT, 8>(ngroups, out_f32, vol, s, x, in_stride, in_coff, w, bias, out, out_stride, out_coff,
                                 mk, mask_stride, mask_coff, cin, flip, relu);
}

struct ConvShape {
    int mt, nt;
};

ConvShape pick_conv_shape(int nt_total, const learn::Vol& vol) {
    // (MT, NT) instantiated below, by decreasing MT * NT
    static const ConvShape cands[] = {{1, 8}, {1, 7}, {1, 6}, {1, 5}, {2, 4}, {2, 3}, {4, 2}, {4, 1},
                                      {1, 4}, {1, 3}, {1, 2}, {1, 1}};
    auto blocks = [&](const ConvShape& c) {
        return (int64_t)((vol.W + 7) / 8) * ((vol.H + 7) / 8) * ((vol.D + c.mt - 1) / c.mt) * (nt_total / c.nt);
    };
    ConvShape best{1, 1};
    int64_t best_blocks = -1;
    int best_work = 0;
    for (const ConvShape& c : cands) {
        if (nt_total % c.nt) continue;
        const int64_t b = blocks(c);
        if (b >= 512 && c.mt * c.nt > best_work) {
            best = c;
            best_work = c.mt * c.nt;
            best_blocks = b;
        }
    }
    if (best_work > 0) return best;
    for (const ConvShape& c : cands) {
        if (nt_total % c.nt) continue;
        if (blocks(c) > best_blocks) {
            best = c;
            best_blocks = blocks(c);
        }
    }
    return best;
}

void launch_conv(int nt_total, int out_f32, const learn::Vol& vol, hipStream_t s, const uint16_t* x, int in_stride,
                 int in_coff, const uint16_t* w, const float* bias, void* out, int out_stride, int out_coff,
                 const uint16_t* mk, int mask_stride, int mask_coff, int cin, int flip, int relu) {
    const ConvShape c = pick_conv_shape(nt_total, vol);
    const int ng = nt_total / c.nt;
#define LC(M, N)                                                                                                  \
    if (c.mt == M && c.nt == N) {                                                                                 \
        launch_conv_cc<M, N>(ng, out_f32, vol, s, x, in_stride, in_coff, w, bias, out, out_stride, out_coff, mk,  \
                             mask_stride, mask_coff, cin, flip, relu);                                            \
        return;                                                                                                   \
    }
    LC(1, 8) LC(1, 7) LC(1, 6) LC(1, 5) LC(2, 4) LC(2, 3) LC(4, 2) LC(4, 1) LC(1, 4) LC(1, 3) LC(1, 2) LC(1, 1)
#undef LC
}

constexpr int kLdsBytes = 160 * 1024;

// Raises a kernel's dynamic LDS limit on the current device, once per device (`done`: a bit each; setting it twice does
// no harm).  A launch past the limit fails by itself.
std::atomic<uint64_t> g_wgrad_devices[4];
void allow_lds(const void* kernel, std::atomic<uint64_t>& done) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return;
    const uint64_t bit = (uint64_t)1 << (dev & 63);
    if (dev < 64 && (done.load() & bit)) return;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes) == hipSuccess && dev < 64)
        done.fetch_or(bit);
}

// Blocks and parts of the weight gradient.  Columns: the whole width, or equal parts of at most 128.  Parts: one or two
// workgroups per CU in all, at most the caller's voxel chunks (whose number the work buffer is sized for).  Rows and
// workgroups per CU: the least time of the longest part, each of its steps costing the MFMAs of the busiest wave pair
// (480 cycles per 32 voxels) and about 1000 cycles more (two workgroups on a CU hide half of that); within what the
// waves' loads and their share of the LDS hold.  (32 -> 32 channels at 48^3: 18.9 us as two workgroups per CU, 16.3 us
// as one of 12-row blocks; 112 -> 48 at 24^3: 16.6 and 15.0 us.)
learn::WgradShape wgrad_shape(const learn::Vol& vol, int pairs, int nparts, double& best_cost) {
    learn::WgradShape best{};
    best_cost = 0.0;
    const int nwb = (vol.W + 127) / 128, wb = (vol.W + nwb - 1) / nwb, pitch = wb + 2;
    const int red = 2 * learn::kWgPhase * learn::kWgSplit * 1024;  // the waves' sums
    for (int per_cu = 1; per_cu <= 2; ++per_cu) {
        int64_t parts = pairs < 256 * per_cu ? 256 * per_cu / pairs : 1;
        if (parts > nparts) parts = nparts;
        if (per_cu == 2 && parts * pairs <= 256) break;
        for (int bh = 1; bh <= vol.H; ++bh) {
            const int nks = (bh * pitch + 31) / 32;
            const int nbx = learn::wgrad_kib((bh + 2) * pitch + 32), nby = learn::wgrad_kib(nks * 32 + 2);
            int lds = (4 * nbx + 2 * nby + (nwb > 1 ? nks : 1)) * 1024;
            if (lds < red) lds = red;
            if ((bh > 1 || per_cu == 2) && (lds > kLdsBytes / per_cu || nbx > learn::kWgX * learn::kWgWaves ||
                                            nby > learn::kWgY * learn::kWgWaves))
                break;
            const int nyb = (vol.H + bh - 1) / bh;
            const int64_t steps = (int64_t)nyb * nwb * vol.D, p = parts < steps ? parts : steps;
            const double rounds = (nks + learn::kWgSplit - 1) / learn::kWgSplit;
            const double cost = (double)((steps + p - 1) / p) * (rounds * 480.0 * per_cu + 1000.0);
            if (best.bh == 0 || cost < best_cost) {
                best_cost = cost;
                best = learn::WgradShape{bh, wb, nyb, nwb, (int)p, lds, 0, 0, 0, 0, 0, 0};
            }
        }
    }
    return best;
}

learn::WgradTensors launch_wgrad(int nparts, hipStream_t s, const uint16_t* in, int in_stride, int in_coff, const uint16_t* dy,
                                 int dy_stride, int dy_coff, float* part, float* part_db, learn::Vol vol, int cin, int cout) {
    const int pairs = cout / 16 * ((cin + 15) / 16);
    double cost = 0.0;
    learn::WgradShape sh = wgrad_shape(vol, pairs, nparts, cost);
    sh.slice = (int64_t)vol.H * vol.W, sh.row = vol.W, sh.col = 1;
    sh.tap_slice = 9, sh.tap_row = 3, sh.tap_col = 1;
    // A volume of few short rows in few parts is a chain of short steps, or of padding; with its axes in another order it may
    // be few long ones (16 -> 16 channels in one part: 64 x 3 x 3 52 and 12, 31 x 48 x 1 38 and 17 us).  Voxels then come
    // one by one from afar, so the other order has to promise a third less (and is not looked for where no order can).
    bool perm = false;
    const int n[3] = {vol.D, vol.H, vol.W}, tap[3] = {9, 3, 1}, order[5][3] = {{1, 0, 2}, {0, 2, 1}, {2, 1, 0}, {1, 2, 0}, {2, 0, 1}};
    const int64_t far[3] = {(int64_t)vol.H * vol.W, vol.W, 1};
    double least = cost / 1.5;
    const double voxels = (double)vol.D * vol.H * vol.W / (pairs < 256 ? std::min(256 / pairs, nparts) : 1);
    for (const auto& o : order) {
        if (least < voxels / (32 * learn::kWgSplit) * 480.0 + 1480.0) break;
        double c = 0.0;
        const learn::Vol v{n[o[0]], n[o[1]], n[o[2]]};
        learn::WgradShape p = wgrad_shape(v, pairs, nparts, c);
        if (c >= least) continue;
        least = c;
        sh = p;
        sh.slice = far[o[0]], sh.row = far[o[1]], sh.col = far[o[2]];
        sh.tap_slice = tap[o[0]], sh.tap_row = tap[o[1]], sh.tap_col = tap[o[2]];
        vol = v;
        perm = true;
    }
    const int64_t stride = in_stride > dy_stride ? in_stride : dy_stride;
    const int64_t span = perm ? (sh.bh + 2) * sh.row + vol.W * sh.col : (int64_t)(sh.bh + 2) * vol.W;
    const bool big = span * stride * 2 >= (int64_t)1 << 31;
    const auto kernel = big ? perm ? learn::wgrad_kernel<true, true> : learn::wgrad_kernel<true, false>
                            : perm ? learn::wgrad_kernel<false, true> : learn::wgrad_kernel<false, false>;
    allow_lds((const void*)kernel, g_wgrad_devices[2 * big + perm]);
    hipLaunchKernelGGL(kernel, dim3((sh.parts * pairs + 7) / 8 * 8), dim3(learn::kWgThreads), sh.lds, s, in, in_stride,
                       in_coff, dy, dy_stride, dy_coff, part, part_db, vol, cin, cout, sh);
    return {in + in_coff, dy + dy_coff, in_stride, dy_stride, cin, vol, sh};
}
constexpr int kBrickD = 4;
struct ConvArgs {
    const uint16_t* in;
    int in_stride, in_coff;
    const uint16_t* w;
    const float* bias;
    void* out;
    int out_stride, out_coff, out_f32;
    const uint16_t* mask;
    int mask_stride, mask_coff;
    learn::Vol vol;
    int cin, cout, flip, relu;
};

template <int CC, int WV, bool kHold, bool kDB>
int brick_lds(const ConvArgs& a) {
    using G = learn::BrickGeom<CC, WV, kBrickD>;
    return (kDB ? 2 : 1) * G::kBuf + a.cin / CC * G::kSteps * 3 * 1024;
}

learn::BrickShape brick_shape(const learn::Vol& vol, int wv) {
    return learn::BrickShape{(vol.W + 15) / 16, (vol.H + wv - 1) / wv, (vol.D + kBrickD - 1) / kBrickD, 0, 0, 0};
}

// One launch: as many workgroups per CU as LDS and registers hold, all resident, each with bricks in a row.
template <int CC, int WV, bool kHold, bool kDB>
bool launch_brick(const ConvArgs& a, hipStream_t s) {
    const int lds = brick_lds<CC, WV, kHold, kDB>(a), groups = a.cout / 16;
    if (lds > kLdsBytes) return false;
    learn::BrickShape sh = brick_shape(a.vol, WV);
    const int64_t bricks = (int64_t)sh.nx * sh.ny * sh.nz;
    const int most = WV == 8 ? 2 : kHold ? 3 : 4, fit = kLdsBytes / lds < most ? kLdsBytes / lds : most;
    const int64_t room = 256 * fit / groups > 0 ? 256 * fit / groups : 1, per = (bricks + room - 1) / room;
    sh.workers = (int)((bricks + per - 1) / per);
    sh.per = (int)(bricks / sh.workers);
    sh.extra = (int)(bricks % sh.workers);
    const auto kernel = a.mask      ? learn::conv3d_brick_kernel<CC, WV, kBrickD, kHold, kDB, true, false>
                        : a.out_f32 ? learn::conv3d_brick_kernel<CC, WV, kBrickD, kHold, kDB, false, true>
                                    : learn::conv3d_brick_kernel<CC, WV, kBrickD, kHold, kDB, false, false>;
    static std::atomic<uint64_t> done[3];
    allow_lds((const void*)kernel, done[a.mask ? 2 : a.out_f32]);
    hipLaunchKernelGGL(kernel, dim3((unsigned)((sh.workers * groups + 7) / 8 * 8)), dim3(64 * WV), lds, s, a.in + a.in_coff,
                       a.in_stride, a.w, a.bias, reinterpret_cast<char*>(a.out) + (int64_t)a.out_coff * (a.out_f32 ? 4 : 2),
                       a.out_stride, a.mask ? a.mask + a.mask_coff : nullptr, a.mask_stride, a.vol, a.cin, groups, a.flip,
                       a.relu, sh);
    return true;
}

// Calls that conv3d_brick_kernel takes: output (and mask) such that 4 channels of a voxel are one access, no mask on a
// float32 output, every voxel of a halo within 2 GiB of its first (which may lie a slice, a row and a voxel before the
// tensor) and rows of less than 2^24 channels (32-bit offsets), weights and halo within a CU's LDS (up to 128 channels).
// Rows up to 8 voxels fill at most half of its 16: there it takes only what gains all the same, one held chunk or 64
// channels and more (8^3: 64 -> 64 channels 10.0 us by conv3d_kernel and 7.4 us by this, 32 -> 32 5.3 and 5.5 us); of these
// not what conv3d_kernel walks 4 slices at a time, except 64 and 128 channels (96 x 96 x 3: 64 -> 32 0.85 of its time, 96 -> 32
// 1.10, 120 -> 32 1.53; at 8 columns 0.87, 1.05, 1.07).
// One chunk of 8 or 16 channels: held in registers, 4 waves, two buffers (16 -> 16 at 96^3: 15.4 us; 18.0 us with the
// weights in LDS).  32-channel chunks: one buffer where two workgroups then fit on a CU (32 -> 32 at 48^3: 9.7 us, with two
// buffers 11.4 us), else two if they fit (64 -> 64 at 96 x 96 x 8: 39 and 37 us).  Several chunks of 8 or 16: two buffers,
// and 8 waves if those give most CUs a workgroup (48 -> 16 at 96^3: 50 us with 4 waves, 43 us with 8; 48 -> 48 at 24^3,
// 54 workgroups of 8: 6.6 and 7.8 us).
bool try_brick(const ConvArgs& a, hipStream_t s) {
    const int64_t voxel = (int64_t)a.in_stride * 2, row = a.vol.W * voxel, slice = a.vol.H * row;
    const int64_t halo = (kBrickD + 1) * slice + (a.vol.H < 9 ? a.vol.H : 9) * row + (a.vol.W < 17 ? a.vol.W : 17) * voxel + 64;
    const bool held = a.cin == 8 || a.cin == 16;
    if (!al(a.out, a.out_f32 ? 16 : 8) || a.out_stride % 4 || a.out_coff % 4 || (a.mask && a.out_f32) ||
        (a.mask && (!al(a.mask, 8) || a.mask_stride % 4 || a.mask_coff % 4 || a.mask_stride >= 1 << 24)) ||
        a.out_stride >= 1 << 24 || halo > (int64_t)1 << 31 ||
        (a.vol.W <= 8 && !held && (a.cin < 64 || (a.cin % 64 && pick_conv_shape(a.cout / 16, a.vol).mt == 4))))
        return false;
    const learn::BrickShape rows8 = brick_shape(a.vol, 8);
    const bool tall = (int64_t)rows8.nx * rows8.ny * rows8.nz * (a.cout / 16) >= 192;
    if (a.cin == 8) return launch_brick<8, 4, true, true>(a, s);
    if (a.cin == 16) return launch_brick<16, 4, true, true>(a, s);
    if (a.cin % 32 == 0) {
        if (2 * brick_lds<32, 4, false, false>(a) > kLdsBytes && launch_brick<32, 4, false, true>(a, s)) return true;
        return launch_brick<32, 4, false, false>(a, s);
    }
    if (a.cin % 16 == 0) return (tall && launch_brick<16, 8, false, true>(a, s)) || launch_brick<16, 4, false, true>(a, s);
    return (tall && launch_brick<8, 8, false, true>(a, s)) || launch_brick<8, 4, false, true>(a, s);
}
}  // namespace

extern "C" {

const char* das_learn_last_error(void) { return g_learn_err; }

int das_conv3d(const void* in, int in_stride, int in_coff, const void* weight, const float* bias, void* out,
               int out_stride, int out_coff, int out_f32, const void* mask, int mask_stride, int mask_coff, int D,
               int H, int W, int cin, int cout, int flip, int relu, void* stream) {
    if (!in || !weight || !out) return lfail(DAS_EINVAL, "conv3d: null pointer");
    if (D < 1 || H < 1 || W < 1 || cin < 8 || cin % 8 || cout < 16 || cout % 16 || cout > 16 * learn::kMaxNT)
        return lfail(DAS_ESHAPE, "conv3d: need D,H,W >= 1, Cin a multiple of 8, Cout a multiple of 16 up to 128");
    if (in_stride < in_coff + cin || in_stride % 8 || in_coff % 8 || in_coff < 0 || out_stride < out_coff + cout ||
        out_coff < 0 || (mask && (mask_stride < mask_coff + cout || mask_coff < 0)))
        return lfail(DAS_ESHAPE, "conv3d: channel slice outside its buffer or not a multiple of 8");
    if (!al(in, 16) || !al(weight, 16)) return lfail(DAS_EALIGN, "conv3d: input and weights must be 16-byte aligned");
    const int64_t V = (int64_t)D * H * W;
    const learn::Vol vol{D, H, W};
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const uint16_t* x = reinterpret_cast<const uint16_t*>(in);
    const uint16_t* w = reinterpret_cast<const uint16_t*>(weight);
    const uint16_t* mk = reinterpret_cast<const uint16_t*>(mask);
    (void)V;
    const ConvArgs args{x, in_stride, in_coff, w, bias, out, out_stride, out_coff, out_f32 != 0, mk, mask_stride, mask_coff, vol,
                        cin, cout, flip, relu};
    if (!try_brick(args, s))
        launch_conv(cout / 16, out_f32 != 0, vol, s, x, in_stride, in_coff, w, bias, out, out_stride, out_coff, mk,
                    mask_stride, mask_coff, cin, flip, relu);
    return launch_status("conv3d launch failed");
}

int das_conv3d_wgrad(const void* in, int in_stride, int in_coff, const void* dy, int dy_stride, int dy_coff,
                     float* dw, float* db, float* work, int64_t work_floats, int D, int H, int W, int cin, int cout,
                     int chunk, void* stream) {
    if (!in || !dy || !dw || !db || !work) return lfail(DAS_EINVAL, "wgrad: null pointer");
    if (D < 1 || H < 1 || W < 1 || cin < 8 || cin % 8 || cout < 16 || cout % 16 || chunk < 32 || chunk % 32)
        return lfail(DAS_ESHAPE, "wgrad: bad sizes (chunk a positive multiple of 32)");
    const int64_t V = (int64_t)D * H * W;
    const int nparts = (int)((V + chunk - 1) / chunk);
    const int64_t K = 27LL * cin, nw = (int64_t)cout * K;
    if (in_stride < in_coff + cin || in_coff < 0 || dy_stride < dy_coff + cout || dy_coff < 0 || in_stride % 8 ||
        in_coff % 8 || dy_stride % 8 || dy_coff % 8)
        return lfail(DAS_ESHAPE, "wgrad: channel slices outside their buffers or not multiples of 8");
    if ((int64_t)D * H * W >= (int64_t)1 << 31) return lfail(DAS_ESHAPE, "wgrad: volume above 2^31 voxels");
    if (!al(in, 16) || !al(dy, 16)) return lfail(DAS_EALIGN, "wgrad: input and dy must be 16-byte aligned");
    if (work_floats < (int64_t)nparts * (nw + cout)) return lfail(DAS_ESHAPE, "wgrad: work buffer too small");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    float* part = work;
    float* part_db = work + (int64_t)nparts * nw;
    const learn::WgradTensors tensors = launch_wgrad(nparts, s, reinterpret_cast<const uint16_t*>(in), in_stride, in_coff,
                                                     reinterpret_cast<const uint16_t*>(dy), dy_stride, dy_coff, part, part_db,
                                                     learn::Vol{D, H, W}, cin, cout);
    hipLaunchKernelGGL(learn::reduce_parts_kernel, dim3(blocks_for(nw, 32) + blocks_for(cout, 32)), dim3(256), 0, s, part,
                       part_db, tensors.sh.parts, nw, (int)blocks_for(nw, 32), cout, dw, db, tensors);
    return launch_status("wgrad launch failed");
}

int64_t das_conv3d_wgrad_work(int D, int H, int W, int cin, int cout, int chunk) {
    if (chunk < 1) return -1;
    const int64_t V = (int64_t)D * H * W;
    return ((V + chunk - 1) / chunk) * ((int64_t)cout * 27 * cin + cout);
}

int das_transpose_weights_many(int n, const void* const* w, void* const* wt, const int* cin, const int* cout, void* stream) {
    if (n < 0 || (n > 0 && (!w || !wt || !cin || !cout))) return lfail(DAS_EINVAL, "transpose: null pointer");
    for (int i = 0; i < n; ++i)
        if (!w[i] || !wt[i]) return lfail(DAS_EINVAL, "transpose: null pointer");
    for (int first = 0; first < n; first += learn::kTransposes) {
        const int m = n - first < learn::kTransposes ? n - first : learn::kTransposes;
        learn::TransposeList l{};
        unsigned blocks = 0;
        for (int i = 0; i < m; ++i) {
            l.w[i] = reinterpret_cast<const uint16_t*>(w[first + i]);
            l.wt[i] = reinterpret_cast<uint16_t*>(wt[first + i]);
            l.cin[i] = cin[first + i];
            l.cout[i] = cout[first + i];
            l.end[i] = blocks += blocks_for((int64_t)l.cout[i] * 27 * l.cin[i], 256);
        }
        hipLaunchKernelGGL(learn::transpose_w_kernel, dim3(blocks), dim3(256), 0, reinterpret_cast<hipStream_t>(stream), l);
    }
    return launch_status("transpose launch failed");
}

int das_transpose_weights(const void* w, void* wt, int cin, int cout, void* stream) {
    return das_transpose_weights_many(1, &w, &wt, &cin, &cout, stream);
}

int das_avgpool2(const void* in, int in_stride, int in_coff, void* out, int out_stride, int out_coff, int Do, int Ho,
                 int Wo, int c, void* stream) {
    if (!in || !out) return lfail(DAS_EINVAL, "avgpool2: null pointer");
    if (!slices_ok(in_stride, in_coff, out_stride, out_coff, c) || Do < 1 || Ho < 1 || Wo < 1)
        return lfail(DAS_ESHAPE, "avgpool2: bad sizes or channel slices");
    // one channel per thread: the 8-channel form (8x fewer threads, eight 16-byte gathers each) measured slower
    const int64_t n = (int64_t)Do * Ho * Wo * c;
    hipLaunchKernelGGL(learn::avgpool2_kernel, dim3(blocks_for(n, 256)), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), reinterpret_cast<const uint16_t*>(in), in_stride, in_coff,
                       reinterpret_cast<uint16_t*>(out), out_stride, out_coff, learn::Vol{Do, Ho, Wo}, c);
    return launch_status("avgpool2 launch failed");
}

int das_avgpool2_bwd(const void* gout, int gout_stride, int gout_coff, void* gin, int gin_stride, int gin_coff, int Di,
                     int Hi, int Wi, int c, int accumulate, void* stream) {
    if (!gout || !gin) return lfail(DAS_EINVAL, "avgpool2_bwd: null pointer");
    if (!slices_ok(gout_stride, gout_coff, gin_stride, gin_coff, c) || !even_dims(Di, Hi, Wi))
        return lfail(DAS_ESHAPE, "avgpool2_bwd: input dimensions must be even and positive; bad channel slices");
    if (v8_volume(Di, Hi, Wi, c) && v8_slice(gout, gout_stride, gout_coff) && v8_slice(gin, gin_stride, gin_coff)) {
        hipLaunchKernelGGL(learn::avgpool2_bwd_v8_kernel, v8_grid(Di, Hi, Wi, c), kV8Block, 0,
                           reinterpret_cast<hipStream_t>(stream), reinterpret_cast<const uint16_t*>(gout), gout_stride,
                           gout_coff, reinterpret_cast<uint16_t*>(gin), gin_stride, gin_coff, learn::Vol{Di, Hi, Wi},
                           c / 8, accumulate);
        return launch_status("avgpool2_bwd launch failed");
    }
    const int64_t n = (int64_t)Di * Hi * Wi * c;
    hipLaunchKernelGGL(learn::avgpool2_bwd_kernel, dim3(blocks_for(n, 256)), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), reinterpret_cast<const uint16_t*>(gout), gout_stride,
                       gout_coff, reinterpret_cast<uint16_t*>(gin), gin_stride, gin_coff, learn::Vol{Di, Hi, Wi}, c,
                       accumulate);
    return launch_status("avgpool2_bwd launch failed");
}

int das_upsample2(const void* in, int in_stride, int in_coff, void* out, int out_stride, int out_coff, int Do, int Ho,
                  int Wo, int c, void* stream) {
    if (!in || !out) return lfail(DAS_EINVAL, "upsample2: null pointer");
    if (!slices_ok(in_stride, in_coff, out_stride, out_coff, c) || !even_dims(Do, Ho, Wo))
        return lfail(DAS_ESHAPE, "upsample2: output dimensions must be even and positive; bad channel slices");
    if (v8_volume(Do, Ho, Wo, c) && v8_slice(in, in_stride, in_coff) && v8_slice(out, out_stride, out_coff)) {
        hipLaunchKernelGGL(learn::upsample2_v8_kernel, v8_grid(Do, Ho, Wo, c), kV8Block, 0,
                           reinterpret_cast<hipStream_t>(stream), reinterpret_cast<const uint16_t*>(in), in_stride,
                           in_coff, reinterpret_cast<uint16_t*>(out), out_stride, out_coff, learn::Vol{Do, Ho, Wo},
                           c / 8);
        return launch_status("upsample2 launch failed");
    }
    const int64_t n = (int64_t)Do * Ho * Wo * c;
    hipLaunchKernelGGL(learn::upsample2_kernel, dim3(blocks_for(n, 256)), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), reinterpret_cast<const uint16_t*>(in), in_stride, in_coff,
                       reinterpret_cast<uint16_t*>(out), out_stride, out_coff, learn::Vol{Do, Ho, Wo}, c);
    return launch_status("upsample2 launch failed");
}

int das_upsample2_bwd(const void* gout, int gout_stride, int gout_coff, void* gin, int gin_stride, int gin_coff,
                      const void* mask, int mask_stride, int mask_coff, int Di, int Hi, int Wi, int c, void* stream) {
    if (!gout || !gin) return lfail(DAS_EINVAL, "upsample2_bwd: null pointer");
    if (!slices_ok(gout_stride, gout_coff, gin_stride, gin_coff, c) || Di < 1 || Hi < 1 || Wi < 1 ||
        (mask && (mask_stride < mask_coff + c || mask_coff < 0)))
        return lfail(DAS_ESHAPE, "upsample2_bwd: bad sizes or channel slices");
    if (v8_volume(Di, Hi, Wi, c) && v8_slice(gout, gout_stride, gout_coff) && v8_slice(gin, gin_stride, gin_coff) &&
        v8_slice(mask, mask_stride, mask_coff)) {
        hipLaunchKernelGGL(learn::upsample2_bwd_v8_kernel, v8_grid(Di, Hi, Wi, c), kV8Block, 0,
                           reinterpret_cast<hipStream_t>(stream), reinterpret_cast<const uint16_t*>(gout), gout_stride,
                           gout_coff, reinterpret_cast<uint16_t*>(gin), gin_stride, gin_coff,
                           reinterpret_cast<const uint16_t*>(mask), mask_stride, mask_coff, learn::Vol{Di, Hi, Wi},
                           c / 8);
        return launch_status("upsample2_bwd launch failed");
    }
    const int64_t n = (int64_t)Di * Hi * Wi * c;
    hipLaunchKernelGGL(learn::upsample2_bwd_kernel, dim3(blocks_for(n, 256)), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), reinterpret_cast<const uint16_t*>(gout), gout_stride,
                       gout_coff, reinterpret_cast<uint16_t*>(gin), gin_stride, gin_coff,
                       reinterpret_cast<const uint16_t*>(mask), mask_stride, mask_coff, learn::Vol{Di, Hi, Wi}, c);
    return launch_status("upsample2_bwd launch failed");
}

int das_add_mask(const void* a, int a_stride, int a_coff, const void* b, int b_stride, int b_coff, const void* mask,
                 int m_stride, int m_coff, void* g, int g_stride, int g_coff, int64_t V, int c, void* stream) {
    if (!a || !b || !g) return lfail(DAS_EINVAL, "add_mask: null pointer");
    if (V < 0 || !slices_ok(a_stride, a_coff, g_stride, g_coff, c) || b_stride < b_coff + c || b_coff < 0 ||
        (mask && (m_stride < m_coff + c || m_coff < 0)))
        return lfail(DAS_ESHAPE, "add_mask: bad sizes or channel slices");
    if (c % 8 == 0 && V * (c / 8) < ((int64_t)1 << 31) && v8_slice(a, a_stride, a_coff) &&
        v8_slice(b, b_stride, b_coff) && v8_slice(mask, m_stride, m_coff) && v8_slice(g, g_stride, g_coff)) {
        const int n = (int)(V * (c / 8));
        if (n == 0) return DAS_OK;
        hipLaunchKernelGGL(learn::add_mask_v8_kernel, dim3(blocks_for(n, 256)), dim3(256), 0,
                           reinterpret_cast<hipStream_t>(stream), reinterpret_cast<const uint16_t*>(a), a_stride,
                           a_coff, reinterpret_cast<const uint16_t*>(b), b_stride, b_coff,
                           reinterpret_cast<const uint16_t*>(mask), m_stride, m_coff, reinterpret_cast<uint16_t*>(g),
                           g_stride, g_coff, n, c / 8);
        return launch_status("add_mask launch failed");
    }
    hipLaunchKernelGGL(learn::add_mask_kernel, dim3(blocks_for(V * c, 256)), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), reinterpret_cast<const uint16_t*>(a), a_stride, a_coff,
                       reinterpret_cast<const uint16_t*>(b), b_stride, b_coff, reinterpret_cast<const uint16_t*>(mask),
                       m_stride, m_coff, reinterpret_cast<uint16_t*>(g), g_stride, g_coff, V, c);
    return launch_status("add_mask launch failed");
}

int das_mse_residual(const float* net, int net_stride, const float* base, const float* target, int64_t V, void* grad,
                     int grad_stride, float* pred, float* loss_parts, void* stream) {
    if (!net || !base || !target || !loss_parts) return lfail(DAS_EINVAL, "mse: null pointer");
    if (net_stride < 2 || (grad && grad_stride < 2)) return lfail(DAS_ESHAPE, "mse: strides");
    const bool vec = al(net, 8) && net_stride % 2 == 0 && al(base, 8) && al(target, 8) && (!pred || al(pred, 8)) &&
                     (!grad || (al(grad, 16) && grad_stride % 8 == 0));
    hipLaunchKernelGGL(vec ? learn::mse_kernel<true> : learn::mse_kernel<false>, dim3(blocks_for(V, 256)), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), net, net_stride, base, target, V,
                       reinterpret_cast<uint16_t*>(grad), grad_stride, pred, loss_parts);
    return launch_status("mse launch failed");
}

int das_adam(float* w, float* m, float* v, const float* g, void* w_bf16, int64_t n, float lr, float beta1, float beta2,
             float eps, int step, void* stream) {
    if (!w || !m || !v || !g) return lfail(DAS_EINVAL, "adam: null pointer");
    if (step < 1) return lfail(DAS_EINVAL, "adam: step counts from 1");
    const float c1 = 1.0f / (1.0f - powf(beta1, (float)step)), c2 = 1.0f / (1.0f - powf(beta2, (float)step));
    hipLaunchKernelGGL(learn::adam_kernel, dim3(blocks_for(n, 256)), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), w, m, v, g, reinterpret_cast<uint16_t*>(w_bf16), n, lr,
                       beta1, beta2, eps, c1, c2);
    return launch_status("adam launch failed");
}

int das_f32_to_bf16(const float* x, void* y, int64_t n, void* stream) {
    if (!x || !y) return lfail(DAS_EINVAL, "cast: null pointer");
    hipLaunchKernelGGL(learn::f32_to_bf16_kernel, dim3(blocks_for(n, 256)), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), x, reinterpret_cast<uint16_t*>(y), n);
    return launch_status("cast launch failed");
}


int das_compound_features(const void* y, int n_in, int64_t V, float gain, void* x, int cin, float* base, float* work,
                          float* scale, void* stream) {
    if (!y || !x || !work || !scale) return lfail(DAS_EINVAL, "compound_features: null pointer");
    if (n_in < 1 || V < 1 || cin < 2 * n_in) return lfail(DAS_ESHAPE, "compound_features: need V >= 1, cin >= 2 n_in");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const float2* yy = reinterpret_cast<const float2*>(y);
    const unsigned nb = blocks_for(V, 256);
    hipLaunchKernelGGL(learn::sumsq_kernel, dim3(nb), dim3(256), 0, s, yy, n_in, V, work);
    hipLaunchKernelGGL(learn::rms_kernel, dim3(1), dim3(256), 0, s, work, (int)nb, V, scale);
    hipLaunchKernelGGL(learn::features_kernel, dim3(nb), dim3(256), 0, s, yy, n_in, V, gain, scale,
                       reinterpret_cast<uint16_t*>(x), cin, base);
    return launch_status("compound_features launch failed");
}

int64_t das_compound_work(int64_t V) { return V < 1 ? 0 : (V + 255) / 256; }

int das_compound_rescale(const void* y, int64_t V, const float* scale, int restore, void* out, void* stream) {
    if (!y || !scale || !out) return lfail(DAS_EINVAL, "compound_rescale: null pointer");
    if (V < 0) return lfail(DAS_ESHAPE, "compound_rescale: V < 0");
    if (V == 0) return DAS_OK;
    hipLaunchKernelGGL(learn::rescale_kernel, dim3(blocks_for(V, 256)), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), reinterpret_cast<const float2*>(y), V, scale,
                       restore ? 0 : 1, reinterpret_cast<float2*>(out));
    return launch_status("compound_rescale launch failed");
}

int das_compound_output(const float* net, int net_stride, const float* base, int64_t V, const float* scale, void* out,
                        void* stream) {
    if (!net || !base || !scale || !out) return lfail(DAS_EINVAL, "compound_output: null pointer");
    if (V < 0 || net_stride < 2) return lfail(DAS_ESHAPE, "compound_output: V < 0 or net_stride < 2");
    if (V == 0) return DAS_OK;
    hipLaunchKernelGGL(learn::compound_output_kernel, dim3(blocks_for(V, 256)), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), net, net_stride, base, V, scale,
                       reinterpret_cast<float2*>(out));
    return launch_status("compound_output launch failed");
}

}  // extern "C"
