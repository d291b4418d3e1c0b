// gfx950 kernels of the delay-and-sum beamformer.
//
// Work decomposition (one wave = 64 voxels of a tile, one lane = one voxel slot,
// FC frames per wave; a workgroup holds one or more such wave tiles, each split
// over one or more element groups):
//
//   for each element e, transmit t that the wave's 64 voxels see (its items):
//     every lane forms its coefficients (fixed-point delay and phase, FP32 result):
//       sample row i0, weight beta, complex C = w exp(+j 2 pi fd tau)
//     the wave stages its sample window of channel data into its own part of LDS
//       as FP32 rows of FC frames, zero outside the record
//     every lane, for each frame f:
//       q0, q1 = row i0, row i0 + 1
//       acc[f] += C * (q0 + beta (q1 - q0))
//   write acc to out[voxel][f]
//
// A wave stages for itself alone: LDS serves one wave's writes and reads in order,
// so there is one buffer per wave and no barrier in the loop, waves drift apart
// and hide each other's latencies, and a wave visits only the elements that its
// own 64 voxels see.  (Workgroup-wide windows, double-buffered with a barrier per
// stage, left the VALU 38 % busy on a 256 x 256 x 32 frame ensemble of 128
// elements: 0.072 ms there.)
//
// The channel data is frame-innermost ([T][E][S][F]), so staging reads are
// contiguous across lanes.  The sum over elements and transmits of each (voxel,
// frame) is taken in a fixed order: results are deterministic (no atomics).
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <type_traits>

#include "das.h"
#include "das_device.h"
#include "das_internal.h"

namespace das {

// ---------------------------------------------------------------- IQ loads
// Complex samples are read in groups of FPT consecutive frames of one sample
// row: one 16-, 8- or 4-byte load, kept raw in registers until the LDS write.
template <int BYTES>
struct RawT;
template <>
struct RawT<16> {
    using type = uint4;
};
template <>
struct RawT<8> {
    using type = uint2;
};
template <>
struct RawT<4> {
    using type = uint32_t;
};

template <int DT>
struct IQType {
    static constexpr int kBytes = (DT == DAS_IQ_C64) ? 8 : 4;  // bytes per complex sample
    static constexpr int kVec = 16 / kBytes;                    // complex samples per 16 bytes
};

// Frame j of a raw group, as FP32 (re, im).
template <int DT, typename R>
__device__ __forceinline__ float2 decode(const R& raw, int j) {
    const uint32_t* w = reinterpret_cast<const uint32_t*>(&raw);
    if constexpr (DT == DAS_IQ_C64) {
        return make_float2(__uint_as_float(w[2 * j]), __uint_as_float(w[2 * j + 1]));
    } else if constexpr (DT == DAS_IQ_C16F) {
        const uint32_t u = w[j];
        return make_float2(__half2float(__ushort_as_half((unsigned short)(u & 0xffffu))),
                           __half2float(__ushort_as_half((unsigned short)(u >> 16))));
    } else {
        const uint32_t u = w[j];
        return make_float2(__uint_as_float(u << 16), __uint_as_float(u & 0xffff0000u));
    }
}

// ------------------------------------------------------- window pre-pass
// For every (wave tile, element, transmit): first sample row and row count used by any active lane ((0, 0) when
// none is).  One wave per wave tile, element-major; 64 results are kept one per lane and stored together.
template <bool kWide>
__global__ __launch_bounds__(kSlots) void window_kernel(PlanDev p, int tile0, int2* __restrict__ win, unsigned long long* counts) {
    const das_kparams& kp = p.kp;
    const int lane = threadIdx.x & 63;
    const int wi = (tile0 + blockIdx.x) * kWaves + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t slot = (int64_t)wi * kLanes + lane;
    const bool valid = p.slot_vox[slot] >= 0;
    const das_lane vl = das_lane_setup(p.vx[slot], p.vy[slot], p.vz[slot], kp);
    const int n = kp.E * kp.T;
    int2* const dst = win + (int64_t)(wi - tile0 * kWaves) * n;
    unsigned long long active = 0, rows = 0;
    int i = 0, longest = 0, used = 0;
    int2 mine = make_int2(0, 0);
    for (int e = 0; e < kp.E; ++e) {
        const das_rx rx = das_rx_setup(vl, p.elemd[4 * e], p.elemd[4 * e + 1], p.elemd[4 * e + 2], kp);
        for (int t = 0; t < kp.T; ++t, ++i) {
            const float txv = p.tx[((int64_t)wi * kp.T + t) * kLanes + lane];
            das_coef c;
            if constexpr (kWide) c = das_wide_setup(rx, txv, kp);
            else c = das_tx_setup(rx, das_tx_const(txv, kp.fix_t0, kp.fix_ph, kp), kp);
            const bool act = valid && das_active(rx, c, kp);
            const unsigned long long ball = __ballot(act);
            int2 w = make_int2(0, 0);
            if (ball != 0) {
                const int i0 = c.hi - kp.row_fix;
                int lo = act ? i0 : INT_MAX, hi = act ? i0 : INT_MIN;
                for (int o = 32; o > 0; o >>= 1) {
                    lo = min(lo, __shfl_xor(lo, o));
                    hi = max(hi, __shfl_xor(hi, o));
                }
                w = make_int2(lo, hi - lo + 1);
                active += (unsigned long long)__popcll(ball);
                longest = max(longest, w.y);
                rows += (unsigned)w.y;
                ++used;
            }
            if ((i & 63) == lane) mine = w;
            if ((i & 63) == 63) dst[i - 63 + lane] = mine;
        }
    }
    if ((n & 63) > lane) dst[(n & ~63) + lane] = mine;
    if (lane == 0) {
        atomicAdd(&counts[0], active);
        atomicMax(&counts[3], (unsigned long long)longest);
        atomicAdd(&counts[4], rows);
        atomicAdd(&counts[5], (unsigned long long)used);
    }
}

// Tile-granular figures: the (slot, e, t) triples of tiles whose window is not empty, and the longest tile window.
__global__ __launch_bounds__(kSlots) void window_stats_kernel(PlanDev p, int tile0, const int2* __restrict__ win,
                                                              unsigned long long* counts) {
    __shared__ unsigned long long s_n;
    __shared__ int s_valid, s_max;
    if (threadIdx.x == 0) {
        s_n = 0;
        s_valid = s_max = 0;
    }
    __syncthreads();
    const int64_t tile = blockIdx.x;
    if (p.slot_vox[(tile0 + tile) * kSlots + threadIdx.x] >= 0) atomicAdd(&s_valid, 1);
    const int n = p.kp.E * p.kp.T;
    unsigned long long used = 0;
    int longest = 0;
    for (int i = threadIdx.x; i < n; i += kSlots) {
        int lo = INT_MAX, hi = INT_MIN;
        for (int w = 0; w < kWaves; ++w) {
            const int2 x = win[(tile * kWaves + w) * n + i];
            if (x.y > 0) {
                lo = min(lo, x.x);
                hi = max(hi, x.x + x.y);
            }
        }
        if (hi > lo) {
            ++used;
            longest = max(longest, hi - lo);
        }
    }
    atomicAdd(&s_n, used);
    atomicMax(&s_max, longest);
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicAdd(&counts[1], s_n * (unsigned long long)s_valid);
        atomicMax(&counts[2], (unsigned long long)s_max);
    }
}

// Items of each wave tile: its non-empty windows cut into pieces of at most `cap` rows, element-major.  Without
// `items`, only their number; one wave per wave tile.
__global__ __launch_bounds__(kLanes) void items_kernel(das_kparams kp, int tile0, const int2* __restrict__ win,
                                                       int cap, const uint32_t* __restrict__ off,
                                                       int4* __restrict__ items, int32_t* __restrict__ n_items) {
    const int wi = tile0 * kWaves + blockIdx.x, lane = threadIdx.x, T = kp.T, E = kp.E, n = E * T;
    const int2* const w = win + (int64_t)blockIdx.x * n;
    const int64_t first = items ? 2 * (int64_t)off[wi] : 0;
    int64_t at = first;
    for (int i0 = 0; i0 < n; i0 += kLanes) {
        const int i = i0 + lane;
        const int2 x = i < n ? w[i] : make_int2(0, 0);
        const int pieces = cap == kGather ? (x.y > 0 ? 1 : 0) : (x.y + cap - 1) / cap;
        int before = pieces;  // inclusive scan
        for (int o = 1; o < kLanes; o <<= 1) {
            const int y = __shfl_up(before, o);
            if (lane >= o) before += y;
        }
        if (items) {
            const int e = i / T, t = i - e * T;
            int4* dst = items + at + (before - pieces);
            if (cap == kGather) {
                if (x.y > 0) *dst = pack_item(e, t, 0, 1, E, kp.S, kp.F, kp.row_fix);
            } else {
                for (int r = 0; r < x.y; r += cap)
                    *dst++ = pack_item(e, t, x.x + r, min(cap, x.y - r), E, kp.S, kp.F, kp.row_fix);
            }
        }
        at += __shfl(before, kLanes - 1);
    }
    if (!items && lane == 0) n_items[wi] = (int32_t)min(at + (at & 1), (int64_t)INT_MAX - 1);
    // an even number of items: the last may have no rows
    if (items && lane == 0 && ((at - first) & 1)) items[at] = make_int4(0, 0, 0, items[at - 1].w);
    // what a wave reads ahead past the last item loads nothing (no rows)
    if (items && wi == kp.n_tiles * kWaves - 1 && lane < kItemPad) items[2 * (int64_t)off[wi + 1] + lane] = make_int4(0, 0, 0, 0);
}

hipError_t launch_windows(const PlanDev& p, int tile0, int n, int2* win, unsigned long long* counts, hipStream_t s) {
    if (p.kp.wide) hipLaunchKernelGGL(window_kernel<true>, dim3(n), dim3(kSlots), 0, s, p, tile0, win, counts);
    else hipLaunchKernelGGL(window_kernel<false>, dim3(n), dim3(kSlots), 0, s, p, tile0, win, counts);
    hipLaunchKernelGGL(window_stats_kernel, dim3(n), dim3(kSlots), 0, s, p, tile0, win, counts);
    return hipGetLastError();
}

hipError_t launch_items(const PlanDev& p, int tile0, int n, const int2* win, const uint32_t* off, int4* items,
                        int32_t* n_items, hipStream_t s) {
    hipLaunchKernelGGL(items_kernel, dim3(n * kWaves), dim3(kLanes), 0, s, p.kp, tile0, win, p.cap_rows, off, items,
                       n_items);
    return hipGetLastError();
}

// ------------------------------------------------------------- main kernel
// How a wave stages window rows of FC frames: FPT consecutive frames of a row per lane and load (16 bytes where
// there are enough), LPR lanes per row, RPI rows per load instruction; the first NL loads of a window are issued an
// item ahead and wait in registers, rows past them (windows longer than NL * RPI - 1 rows) are fetched on the spot.
// LDS rows are FP32, PB bytes apart: an odd number of 16-byte units, so that lanes on 16 consecutive rows read
// from distinct banks (one row per 8 or 16 bytes needs no padding for that).
template <int FC, int DT>
struct Stage {
    static constexpr int kEB = IQType<DT>::kBytes;
    static constexpr int FPT = FC < IQType<DT>::kVec ? FC : IQType<DT>::kVec;
    static constexpr int LPR = FC / FPT;
    static constexpr int RPI = kLanes / LPR;
    static constexpr int NL = RPI >= 32 ? 1 : RPI >= 16 ? 2 : 3;
    static constexpr int PB = lds_row_bytes(FC);
};

// A plan's arrays through the constant address space, so that wave-uniform reads are scalar loads.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* constant(const T* p) {
    return (const __attribute__((address_space(4))) T*)(uintptr_t)p;
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) f32x2 lds_f32x2;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
typedef __attribute__((address_space(3))) char lds_char;

// Waves per SIMD the registers are cut for.
constexpr int das_waves(int fc, int ntx, bool planar) {
    return fc >= 16 ? 4 : fc >= 8 ? 6 : ((fc == 2 && ntx > 1) || !planar) ? 7 : 8;
}
constexpr int das_gather_waves(int fc, int ntx) { return fc >= 8 ? (ntx > 1 ? 4 : 5) : 8; }
constexpr int kMaxThreads = 1024;

// Sums the groups' accumulators in a fixed order, ((g0 + g1) + g2) + ..., and writes them.  With several groups all of
// them pass through LDS, and group g sums and writes frames g * nf ... (nf = frames / groups, rounded up).
template <int N, int FC>
__device__ __forceinline__ void das_finish(char* lds, const float (&ar)[N], const float (&ai)[N], int col, int row,
                                           int grp, int lg_groups, int vox, int f0, int F, int T, int64_t tx_stride,
                                           float2* __restrict__ out) {
    const int groups = 1 << lg_groups;
    if (groups == 1) {
        if (vox < 0) return;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            if (N > FC && k / FC >= T) break;
            float2* o = out + (k / FC) * tx_stride + (size_t)vox * F;
            if (f0 + k % FC < F) o[f0 + k % FC] = make_float2(ar[k], ai[k]);
        }
        return;
    }
    float2* red = reinterpret_cast<float2*>(lds);  // [groups][N][row]
    __syncthreads();  // every wave is done with its window
#pragma unroll
    for (int k = 0; k < N; ++k) red[(grp * N + k) * row + col] = make_float2(ar[k], ai[k]);
    __syncthreads();
    if (vox < 0) return;
    const int nf = (N + groups - 1) >> lg_groups, k1 = min(N, (grp + 1) * nf);
    for (int k = grp * nf; k < k1; ++k) {
        float2 s = red[k * row + col];
        for (int g = 1; g < groups; ++g) {
            const float2 v = red[(g * N + k) * row + col];
            s.x += v.x;
            s.y += v.y;
        }
        const int t = k / FC, f = f0 + k % FC;
        if (f < F && (N == FC || t < T)) out[t * tx_stride + (size_t)vox * F + f] = s;
    }
}

// kOne: one transmit; otherwise the receive part is kept across an element's transmits.  NTX > 1: per-transmit output; each lane keeps NTX
// sets of FC accumulators and adds an item into the set of its transmit (wave-uniform, so the choice is a scalar
// branch); out is [T][V][F] (tx_stride = V * F), T <= NTX.
template <int FC, int DT, int NTX, bool kOne, bool kPlanar>
__global__ __launch_bounds__(kMaxThreads) __attribute__((amdgpu_waves_per_eu(das_waves(FC, NTX, kPlanar),
                                                                              das_waves(FC, NTX, kPlanar))))
void das_kernel(PlanDev p, const void* __restrict__ iq, float2* __restrict__ out, int lg_wt, int lg_halves, int lg_groups,
                int wave_bytes, int64_t tx_stride) {
    using St = Stage<FC, DT>;
    constexpr int kEB = St::kEB, FPT = St::FPT, LPR = St::LPR, RPI = St::RPI, NL = St::NL, PB = St::PB;
    using Raw = typename RawT<FPT * kEB>::type;
    extern __shared__ __attribute__((aligned(16))) char lds[];  // one window and two zero rows per wave
    const das_kparams& kp = p.kp;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // Wave tiles, halves and groups of a workgroup are powers of two, and what depends on the workgroup comes in one load:
    // integer divisions and one load waiting for another had been half a microsecond of every wave's start.
    const int lg_cols = lg_wt + lg_halves, cols = 1 << lg_cols, groups = 1 << lg_groups;
    const int col = wave & (cols - 1), grp = wave >> lg_cols;  // (wave tile, frame half), element group
    const int4 unit = p.wg_unit[blockIdx.x];  // all chunks of the heaviest wave tiles are dispatched first
    const int wi = unit.x + (col & ((1 << lg_wt) - 1));
    const int f0 = ((unit.y << lg_halves) + (col >> lg_wt)) * FC;
    const int64_t slot = (int64_t)wi * kLanes + lane;
    const int vox = p.slot_vox[slot];
    const das_lane L = das_lane_setup(p.vx[slot], p.vy[slot], p.vz[slot], kp);

    float acc_r[NTX * FC], acc_i[NTX * FC];
#pragma unroll
    for (int f = 0; f < NTX * FC; ++f) {
        acc_r[f] = 0.0f;
        acc_i[f] = 0.0f;
    }
    // this group's share of the wave tile's items
    uint32_t first = (uint32_t)unit.z;
    int pairs = unit.w;
    if (lg_wt) {
        first = p.item_off[wi];
        pairs = (int)(p.item_off[wi + 1] - first);
    }
    const int share = pairs >> lg_groups, left = pairs & (groups - 1);
    const int k0 = share * grp + min(grp, left), k1 = k0 + share + (grp < left ? 1 : 0);
    const auto* next = constant(reinterpret_cast<const uint64_t*>(p.items + 2 * (size_t)(first + (uint32_t)k0)));
    const auto* const elem = constant(p.elemd);

    const int rl = lane / LPR, fg = lane % LPR;  // this lane's row and frame group of a load
    const int row_bytes = kp.F * kEB;
    // A lane whose frames are all past F stays out of every record (offsets are 32 bits, records below 2 GiB).
    const uint32_t lane_off =
        f0 + fg * FPT < kp.F ? (uint32_t)(rl * row_bytes + (f0 + fg * FPT) * kEB) : 0x80000000u;
    char* const win = lds + wave * wave_bytes;
    const uint32_t win_at = (uint32_t)(uintptr_t)(lds_char*)win;  // LDS address
    uint32_t zero_row = (uint32_t)(wave_bytes / PB - 2);  // two rows of zeros behind the window
    asm volatile("" : "+v"(zero_row));
    char* const wdst = win + rl * PB + fg * FPT * 8;
    for (int i = lane; i < 2 * PB / 8; i += kLanes)
        *reinterpret_cast<float2*>(win + zero_row * PB + 8 * i) = make_float2(0.0f, 0.0f);
    __builtin_amdgcn_wave_barrier();  // the wave's own rows: no wait for the others, nor for the loads so far

    struct Item {
        uint64_t at;  // sample offset and row counts
        int row;      // first row + row_fix
        uint32_t et;  // element and transmit
        // (spelled out: the compiler would compare all 64 bits on the vector unit instead)
        __device__ int rows() const {
            uint32_t r;
            asm("s_lshr_b32 %0, %1, 24" : "=s"(r) : "s"((uint32_t)(at >> 32)) : "scc");
            return (int)r;
        }
        __device__ int loaded() const { return (int)__builtin_amdgcn_ubfe((uint32_t)(at >> 32), 16, 8); }
        __device__ int e() const { return (int)(et >> kTxBits); }
        __device__ int t() const { return (int)(et & (kMaxTx - 1)); }
    };
    auto item = [&] {
        const uint64_t a = next[0], b = next[1];
        next += 2;
        return Item{a, (int)(uint32_t)b, (uint32_t)(b >> 32)};
    };
    // Reads go through a buffer resource over the rows to load, whose range check returns zero outside it: for the
    // rows past the record's end, and for row -1 (whose offset wraps to one past the end), the record's zero
    // padding; and for the lanes past the window, which then fetch nothing.  Frames past F read the next row's and
    // feed no output.  (Where rows are not counted from 0, no window begins before the row they are counted from.)
    auto window = [&](const Item& it) {
        const uint64_t a = reinterpret_cast<uint64_t>(iq) + it.at * kEB;  // the low 48 bits count
        return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(a), (short)0, it.loaded() * row_bytes,
                                                 0x00020000);
    };
    auto first_off = [&](const Item& it) { return lane_off - (it.row < kDasFixHigh ? (uint32_t)row_bytes : 0u); };
    auto load = [&](const __amdgpu_buffer_rsrc_t& rs, uint32_t off) {
        if constexpr (sizeof(Raw) == 16) return __builtin_bit_cast(Raw, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
        else if constexpr (sizeof(Raw) == 8) return __builtin_bit_cast(Raw, __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0));
        else return __builtin_bit_cast(Raw, __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
    };
    // The rows of an item's window and the row after it, RPI at a time.
    auto issue = [&](const Item& it, Raw (&raw)[NL]) {
        const __amdgpu_buffer_rsrc_t rs = window(it);
        const uint32_t off = first_off(it);
#pragma unroll
        for (int j = 0; j < NL; ++j)
            if (j == 0 || it.rows() >= j * RPI) raw[j] = load(rs, off + (uint32_t)(j * RPI * row_bytes));
    };
    auto put = [&](const Raw& raw, char* dst) {
        if constexpr (FPT == 1) {
            const float2 a = decode<DT>(raw, 0);
            *reinterpret_cast<f32x2*>(dst) = f32x2{a.x, a.y};
        } else {
#pragma unroll
            for (int q = 0; q < FPT; q += 2) {
                const float2 a = decode<DT>(raw, q), b = decode<DT>(raw, q + 1);
                *reinterpret_cast<f32x4*>(dst + 8 * q) = f32x4{a.x, a.y, b.x, b.y};
            }
        }
    };
    auto stage = [&](const Item& it, const Raw (&raw)[NL]) {
#pragma unroll
        for (int j = 0; j < NL; ++j)
            if (j == 0 || it.rows() >= j * RPI) put(raw[j], wdst + j * RPI * PB);
        const int rows = it.rows();
        if (__builtin_expect(rows >= NL * RPI, 0)) {
            const __amdgpu_buffer_rsrc_t rs = window(it);
            const uint32_t off = first_off(it);
            // (two loads at a time; at 8 frames the second one's registers spill)
#pragma unroll FC == 8 ? 1 : 2
            for (int j = NL; j <= rows / RPI; ++j)
                put(load(rs, off + (uint32_t)(j * RPI * row_bytes)), wdst + j * RPI * PB);
        }
    };

    // Coefficients of an item for this lane.  A lane whose sample row is outside the item's window reads the zero
    // rows: it adds exact zeros whatever the window holds.  A row inside the window is inside the record (windows
    // span the rows of active lanes only); lanes outside the aperture carry w = 0; empty slots compute a valid
    // voxel's sums that are never stored.
    struct Coef {
        uint32_t src;  // LDS address of the lane's first row
        float beta, cr, ci;
    };
    int last_e = -1;
    das_rx rx;
    double fix_t0 = kp.fix_t0, fix_ph = kp.fix_ph;
    asm volatile("" : "+v"(fix_t0), "+v"(fix_ph));  // an FMA takes one scalar operand: kept in vector registers
    const das_txc tc0 = das_tx_const(p.tx[(int64_t)wi * kp.T * kLanes + lane], fix_t0, fix_ph, kp);  // transmit 0
    struct Xyz {
        double x, y, z;
    };
    auto coords = [&](const Item& it) {
        // (a 32-bit offset that the compiler cannot see through goes into the load; it would add 64 bits otherwise: three
        // transmits apart at 96^3 x 1024 elements 1079 -> 1049 us, scalar instructions bounding them)
        uint32_t off = it.et >> kTxBits << 5;
        asm("" : "+s"(off));
        const auto* e = (const __attribute__((address_space(4))) f64x2*)((const __attribute__((address_space(4))) char*)elem + off);
        const f64x2 xy = e[0];
        return Xyz{xy.x, xy.y, kPlanar ? 0.0 : e[1].x};
    };
    auto coef = [&](const Item& it, const Xyz& e, float txv) {
        das_coef c;
        if constexpr (kOne) {
            c = das_tx_setup(das_rx_setup_t<kPlanar>(L, e.x, e.y, e.z, kp), tc0, kp);
        } else {
            // marked unlikely (it is taken once per element, every T-th item), so that the compiler keeps
            // the branch rather than forming the receive part for every item
            if (__builtin_expect(it.e() != last_e, 0)) {
                rx = das_rx_setup_t<kPlanar>(L, e.x, e.y, e.z, kp);
                last_e = it.e();
            }
            c = das_tx_setup(rx, das_tx_const(txv, fix_t0, fix_ph, kp), kp);
        }
        const unsigned d = (unsigned)c.hi - (unsigned)it.row;
        const unsigned r = d < (unsigned)it.rows() ? d : zero_row;
        return Coef{win_at + (PB < 16 ? r * PB : __umul24(r, PB)), c.beta, c.cr, c.ci};
    };
    auto point = [&](const Coef& c, float qx, float qy, float nx, float ny, int k) {
        const float tr = fmaf(c.beta, nx - qx, qx);
        const float ti = fmaf(c.beta, ny - qy, qy);
        acc_r[k] = fmaf(c.cr, tr, acc_r[k]);
        acc_r[k] = fmaf(-c.ci, ti, acc_r[k]);
        acc_i[k] = fmaf(c.cr, ti, acc_i[k]);
        acc_i[k] = fmaf(c.ci, tr, acc_i[k]);
    };
    auto mac_into = [&](const Coef& c, int a0) {
        if constexpr (FC == 1) {
            const f32x2 a = *(const lds_f32x2*)(size_t)c.src, b = *(const lds_f32x2*)(size_t)(c.src + PB);
            point(c, a.x, a.y, b.x, b.y, a0);
        } else {
#pragma unroll
            for (int f = 0; f < FC; f += 2) {
                const f32x4 a = *(const lds_f32x4*)(size_t)(c.src + 8 * f);
                const f32x4 b = *(const lds_f32x4*)(size_t)(c.src + PB + 8 * f);
                point(c, a.x, a.y, b.x, b.y, a0 + f);
                point(c, a.z, a.w, b.z, b.w, a0 + f + 1);
            }
        }
    };
    auto mac = [&](const Coef& c, int t) {
        if constexpr (NTX == 1) {
            mac_into(c, 0);
        } else {
#pragma unroll
            for (int j = 0; j < NTX; ++j)
                if (t == j) mac_into(c, j * FC);
        }
    };

    if (k0 < k1) {
        const __amdgpu_buffer_rsrc_t txs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>(p.tx + (int64_t)wi * kp.T * kLanes), (short)0, kp.T * kLanes * 4, 0x00020000);
        auto tx_of = [&](const Item& x) {
            if constexpr (kOne) return 0.0f;
            else return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(txs, lane * 4, x.t() * (kLanes * 4), 0));
        };
        // Step k: write item k's window (loaded during step k - 1) to LDS; load item k + 1's window and item k + 2's
        // transmit times; multiply-accumulate item k while forming item k + 1's coefficients.  Scalar loads (item
        // k + 3, item k + 2's element) start the step, so that they have landed when its LDS reads are waited for (an
        // outstanding scalar load turns that wait into a wait for everything).  Two steps alternate between register
        // sets: a copy at the loop's end would wait for the loads just issued.  (Every group has an even
        // number of items: the lists are padded with items of no rows, which every lane reads zeros for.)  Items past the group's last (the next
        // group's, the next tile's or padding) are loaded and formed but not accumulated.
        Raw raw[NL];
        Item it = item(), nx = item(), af = item();
        float txa = tx_of(it), txb = tx_of(nx);
        issue(it, raw);
        Xyz ea = coords(it), eb = coords(nx);
        Coef ca = coef(it, ea, txa), cb;
        auto step = [&](const Coef& c, Coef& cn, Xyz& e, const Xyz& en, float& tx, float txn) {
            const Item far = item();
            e = coords(af);
            stage(it, raw);
            __builtin_amdgcn_wave_barrier();  // lanes read what other lanes of the wave wrote
            issue(nx, raw);
            tx = tx_of(af);
            cn = coef(nx, en, txn);
            mac(c, it.t());
            // The step's results belong to the step: otherwise the compiler moves part of the sums and coefficients
            // behind the next step's branches, where two steps' values are live at once and spill.
#pragma unroll
            for (int f = 0; f < NTX * FC; ++f) asm volatile("" : "+v"(acc_r[f]), "+v"(acc_i[f]));
            asm volatile("" : "+v"(cn.beta), "+v"(cn.cr), "+v"(cn.ci), "+v"(cn.src));
            __builtin_amdgcn_sched_barrier(0);
            it = nx;
            nx = af;
            af = far;
        };
        for (int k = k0; k < k1; ++k) {
            step(ca, cb, ea, eb, txa, txb);
            step(cb, ca, eb, ea, txb, txa);
        }
    }
    das_finish<NTX * FC, FC>(lds, acc_r, acc_i, col * kLanes + lane, cols * kLanes, grp, lg_groups, vox, f0, kp.F, kp.T,
                             tx_stride, out);
}

// Long windows: a lane reads its own two rows of every item straight from the record, FC frames of each, with no LDS but for
// the groups' sums.  choose_gather says when.
// Bound by the cache's rate on 64 places at a time; the rows of an item are all asked for before the first is used, and many
// waves hide the wait.
template <int FC, int DT, int NTX>
__global__ __launch_bounds__(kMaxThreads) __attribute__((amdgpu_waves_per_eu(das_gather_waves(FC, NTX), das_gather_waves(FC, NTX))))
void das_gather_kernel(PlanDev p, const void* __restrict__ iq, float2* __restrict__ out, int lg_wt, int lg_halves, int lg_groups,
                       int64_t tx_stride) {
    constexpr int kEB = IQType<DT>::kBytes, FPT = FC < IQType<DT>::kVec ? FC : IQType<DT>::kVec;
    using Raw = typename RawT<FPT * kEB>::type;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const das_kparams& kp = p.kp;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lg_cols = lg_wt + lg_halves, cols = 1 << lg_cols, groups = 1 << lg_groups;
    const int col = wave & (cols - 1), grp = wave >> lg_cols;
    const int4 unit = p.wg_unit[blockIdx.x];
    const int wi = unit.x + (col & ((1 << lg_wt) - 1));
    const int f0 = ((unit.y << lg_halves) + (col >> lg_wt)) * FC;
    const int64_t slot = (int64_t)wi * kLanes + lane;
    const int vox = p.slot_vox[slot];
    const das_lane L = das_lane_setup(p.vx[slot], p.vy[slot], p.vz[slot], kp);
    float acc_r[NTX * FC], acc_i[NTX * FC];
#pragma unroll
    for (int f = 0; f < NTX * FC; ++f) acc_r[f] = acc_i[f] = 0.0f;
    const uint32_t first = p.item_off[wi];
    const int pairs = (int)(p.item_off[wi + 1] - first), share = pairs >> lg_groups, left = pairs & (groups - 1);
    const int k0 = share * grp + min(grp, left), k1 = k0 + share + (grp < left ? 1 : 0);
    const auto* next = constant(reinterpret_cast<const uint64_t*>(p.items + 2 * (size_t)(first + (uint32_t)k0)));
    const auto* const elem = constant(p.elemd);
    const float* const txs = p.tx + (int64_t)wi * kp.T * kLanes + lane;
    const int row_bytes = kp.F * kEB, rec_bytes = kp.S * row_bytes;
    int last_e = -1;
    das_rx rx;
    for (int k = 2 * k0; k < 2 * k1; ++k) {
        const uint64_t at = next[0];
        const uint32_t et = (uint32_t)(next[1] >> 32);
        next += 2;
        const int e = (int)(et >> kTxBits), t = (int)(et & (kMaxTx - 1));
        if (e != last_e) {
            rx = das_rx_setup(L, elem[4 * e], elem[4 * e + 1], elem[4 * e + 2], kp);
            last_e = e;
        }
        const das_coef c = das_tx_setup(rx, das_tx_const(txs[t * kLanes], kp.fix_t0, kp.fix_ph, kp), kp);
        // (an item of no rows pads the list; a lane that has no part in the item reads zeros)
        const bool on = das_active(rx, c, kp) & ((at >> 56) != 0);
        const uint32_t off = on ? (uint32_t)((c.hi - kp.row_fix) * row_bytes + f0 * kEB) : 0x80000000u;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            reinterpret_cast<void*>(reinterpret_cast<uint64_t>(iq) + at * kEB), (short)0, rec_bytes, 0x00020000);
        auto load = [&](uint32_t o) {
            if constexpr (sizeof(Raw) == 16) return __builtin_bit_cast(Raw, __builtin_amdgcn_raw_buffer_load_b128(rs, o, 0, 0));
            else if constexpr (sizeof(Raw) == 8) return __builtin_bit_cast(Raw, __builtin_amdgcn_raw_buffer_load_b64(rs, o, 0, 0));
            else return __builtin_bit_cast(Raw, __builtin_amdgcn_raw_buffer_load_b32(rs, o, 0, 0));
        };
        Raw q0[FC / FPT], q1[FC / FPT];
#pragma unroll
        for (int g = 0; g < FC / FPT; ++g) {
            q0[g] = load(off + g * FPT * kEB);
            q1[g] = load(off + g * FPT * kEB + (on ? row_bytes : 0));
        }
        auto mac = [&](int a0) {
#pragma unroll
            for (int f = 0; f < FC; ++f) {
                const float2 a = decode<DT>(q0[f / FPT], f % FPT), b = decode<DT>(q1[f / FPT], f % FPT);
                const float tr = fmaf(c.beta, b.x - a.x, a.x), ti = fmaf(c.beta, b.y - a.y, a.y);
                acc_r[a0 + f] = fmaf(-c.ci, ti, fmaf(c.cr, tr, acc_r[a0 + f]));
                acc_i[a0 + f] = fmaf(c.ci, tr, fmaf(c.cr, ti, acc_i[a0 + f]));
            }
        };
        if constexpr (NTX == 1) {
            mac(0);
        } else {
#pragma unroll
            for (int j = 0; j < NTX; ++j)
                if (t == j) mac(j * FC);
        }
    }
    das_finish<NTX * FC, FC>(lds, acc_r, acc_i, col * kLanes + lane, cols * kLanes, grp, lg_groups, vox, f0, kp.F, kp.T,
                             tx_stride, out);
}

// Any finite geometry: FP64 delays and phases, samples gathered from the record, every (element, transmit) visited.
// Serves only plans whose own rows span 2^19 and more, whose phases over the record do not fit 2^19 cycles, whose sizes do
// not fit an item (more than 16384 transmits or 262144 elements, records of more than 2^45 samples), or whose items fit neither
// 2^32 pairs nor the memory.
template <int DT>
__global__ __launch_bounds__(kSlots) void das_wide_kernel(PlanDev p, const void* __restrict__ iq,
                                                          float2* __restrict__ out, int per_tx, int64_t tx_stride) {
    const das_kparams& kp = p.kp;
    const int64_t slot = (int64_t)blockIdx.x * kSlots + threadIdx.x;
    const int vox = p.slot_vox[slot];
    if (vox < 0) return;
    const das_lane L = das_lane_setup(p.vx[slot], p.vy[slot], p.vz[slot], kp);
    using S = std::conditional_t<DT == DAS_IQ_C64, uint2, uint32_t>;
    for (int f = blockIdx.y; f < kp.F; f += gridDim.y) {
        float re = 0.0f, im = 0.0f;
        for (int t = 0; t < kp.T; ++t) {
            const float txv = p.tx[(slot / kLanes * kp.T + t) * kLanes + slot % kLanes];
            for (int e = 0; e < kp.E; ++e) {
                const das_rx rx = das_rx_setup(L, p.elemd[4 * e], p.elemd[4 * e + 1], p.elemd[4 * e + 2], kp);
                const das_coef c = das_wide_setup(rx, txv, kp);
                if (!das_active(rx, c, kp)) continue;
                const S* rec = reinterpret_cast<const S*>(iq) + ((int64_t)t * kp.E + e) * kp.S * kp.F + f;
                float2 a = make_float2(0.0f, 0.0f), b = a;
                const int i0 = c.hi - kp.row_fix;
                if (i0 >= 0) a = decode<DT>(rec[(int64_t)i0 * kp.F], 0);
                if (i0 + 1 < kp.S) b = decode<DT>(rec[(int64_t)(i0 + 1) * kp.F], 0);
                const float tr = fmaf(c.beta, b.x - a.x, a.x);
                const float ti = fmaf(c.beta, b.y - a.y, a.y);
                re = fmaf(-c.ci, ti, fmaf(c.cr, tr, re));
                im = fmaf(c.ci, tr, fmaf(c.cr, ti, im));
            }
            if (per_tx) {
                out[t * tx_stride + (int64_t)vox * kp.F + f] = make_float2(re, im);
                re = im = 0.0f;
            }
        }
        if (!per_tx) out[(int64_t)vox * kp.F + f] = make_float2(re, im);
    }
}

// ---------------------------------------------------------------- launches
constexpr int kPerTx = 4;  // transmits of per-transmit output (variants of at most 2 frames per workgroup)
constexpr int kGatherFrames = 8;  // frames that gathering waves take of more than 8

template <int FC, int DT>
static int wave_bytes(const PlanDev& p) {
    using St = Stage<FC, DT>;
    return ((p.cap_rows + St::RPI) / St::RPI * St::RPI + 2) * St::PB;  // cap_rows + 1 rows in whole loads, two of zeros
}

// The plan's workgroups in launches of at most launch_units.
template <typename Launch>
static hipError_t launch_all(const PlanDev& p, int64_t units, Launch&& launch) {
    if (units <= p.launch_units) {
        launch(p, units);
    } else {
        PlanDev q = p;
        for (int64_t u = 0; u < units; u += p.launch_units) {
            q.wg_unit = p.wg_unit + u;
            launch(q, std::min(p.launch_units, units - u));
        }
    }
    return hipGetLastError();
}

template <int FC, int DT, int NTX>
static hipError_t launch_gather(const PlanDev& p, const void* iq, void* out, hipStream_t s) {
    const int halves = p.fc / FC, nchunk = (p.kp.F + p.fc - 1) / p.fc, waves = p.n_wt * halves * p.split;
    const size_t sh = p.split > 1 ? (size_t)waves * NTX * FC * kLanes * sizeof(float2) : 0;
    return launch_all(p, (int64_t)p.kp.n_tiles * (kWaves / p.n_wt) * nchunk, [&](const PlanDev& q, int64_t n) {
        hipLaunchKernelGGL((das_gather_kernel<FC, DT, NTX>), dim3((unsigned)n), dim3(waves * kLanes), sh, s, q, iq,
                           reinterpret_cast<float2*>(out), __builtin_ctz(p.n_wt), __builtin_ctz(halves), __builtin_ctz(p.split),
                           p.n_vox * p.kp.F);
    });
}

template <int FC, int DT, int NTX, bool kOne, bool kPlanar>
static hipError_t launch_k(const PlanDev& p, const void* iq, void* out, hipStream_t s) {
    const int halves = p.fc / FC, nchunk = (p.kp.F + p.fc - 1) / p.fc, waves = p.n_wt * halves * p.split;
    const int wb = wave_bytes<FC, DT>(p);
    const size_t win = (size_t)waves * wb;
    const size_t red = p.split > 1 ? (size_t)waves * NTX * FC * kLanes * sizeof(float2) : 0;
    const size_t sh = win > red ? win : red;
    return launch_all(p, (int64_t)p.kp.n_tiles * (kWaves / p.n_wt) * nchunk, [&](const PlanDev& q, int64_t n) {
        hipLaunchKernelGGL((das_kernel<FC, DT, NTX, kOne, kPlanar>), dim3((unsigned)n), dim3(waves * kLanes), sh, s, q, iq,
                           reinterpret_cast<float2*>(out), __builtin_ctz(p.n_wt), __builtin_ctz(halves), __builtin_ctz(p.split), wb,
                           p.n_vox * p.kp.F);
    });
}

template <int FC, int DT, int NTX, bool kOne, bool kPlanar>
static hipError_t lds_limit() {
    return hipFuncSetAttribute((const void*)das_kernel<FC, DT, NTX, kOne, kPlanar>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               kLdsBytes);
}

template <int FC, int DT, int NTX, bool kOne>
static hipError_t dispatch_ntx(const PlanDev& p, const void* iq, void* out, bool prepare, hipStream_t s) {
    if (p.kp.planar)
        return prepare ? lds_limit<FC, DT, NTX, kOne, true>() : launch_k<FC, DT, NTX, kOne, true>(p, iq, out, s);
    return prepare ? lds_limit<FC, DT, NTX, kOne, false>() : launch_k<FC, DT, NTX, kOne, false>(p, iq, out, s);
}

template <int FC, int DT, int NTX>
static hipError_t dispatch_gather(const PlanDev& p, const void* iq, void* out, bool prepare, hipStream_t s) {
    if (prepare)
        return hipFuncSetAttribute((const void*)das_gather_kernel<FC, DT, NTX>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    return launch_gather<FC, DT, NTX>(p, iq, out, s);
}

template <int FC, int DT>
static hipError_t dispatch(const PlanDev& p, const void* iq, void* out, bool per_tx, bool prepare, hipStream_t s) {
    if (p.cap_rows == kGather) {
        if constexpr (FC <= kGatherFrames) {
            if (p.per_tx && (prepare || per_tx)) {
                const hipError_t e = dispatch_gather<FC, DT, kPerTx>(p, iq, out, prepare, s);
                if (e != hipSuccess || per_tx) return e;
            }
        }
        if constexpr (FC <= kGatherFrames) return dispatch_gather<FC, DT, 1>(p, iq, out, prepare, s);
    }
    if constexpr (FC <= 2) {
        if (p.per_tx && (prepare || per_tx)) {
            const hipError_t e = dispatch_ntx<FC, DT, kPerTx, false>(p, iq, out, prepare, s);
            if (e != hipSuccess || per_tx) return e;
        }
    }
    if (p.kp.T > 1) return dispatch_ntx<FC, DT, 1, false>(p, iq, out, prepare, s);
    return dispatch_ntx<FC, DT, 1, true>(p, iq, out, prepare, s);
}

template <int DT>
static hipError_t dispatch_fc(const PlanDev& p, const void* iq, void* out, bool per_tx, bool prepare, hipStream_t s) {
    if (p.kp.wide) {
        if (!prepare)
            hipLaunchKernelGGL(das_wide_kernel<DT>, dim3(p.kp.n_tiles, p.kp.F < 65535 ? p.kp.F : 65535), dim3(kSlots), 0,
                               s, p, iq, reinterpret_cast<float2*>(out), per_tx ? 1 : 0, p.n_vox * p.kp.F);
        return hipGetLastError();
    }
    switch (p.fc) {
        case 1: return dispatch<1, DT>(p, iq, out, per_tx, prepare, s);
        case 2: return dispatch<2, DT>(p, iq, out, per_tx, prepare, s);
        case 4: return dispatch<4, DT>(p, iq, out, per_tx, prepare, s);
        case 8: return dispatch<8, DT>(p, iq, out, per_tx, prepare, s);
        case 16:
        case 32:  // two halves of 16 frames, each by waves of its own (32 accumulator pairs per lane: 248 against 217 us
                  // for 512 x 512 x 32 frames, three waves per SIMD instead of five)
            return dispatch<16, DT>(p, iq, out, per_tx, prepare, s);
        default: return hipErrorInvalidValue;
    }
}

static hipError_t dispatch_dt(const PlanDev& p, const void* iq, int dtype, void* out, bool per_tx, bool prepare,
                              hipStream_t s) {
    switch (dtype) {
        case DAS_IQ_C64: return dispatch_fc<DAS_IQ_C64>(p, iq, out, per_tx, prepare, s);
        case DAS_IQ_C16F: return dispatch_fc<DAS_IQ_C16F>(p, iq, out, per_tx, prepare, s);
        default: return dispatch_fc<DAS_IQ_C16BF>(p, iq, out, per_tx, prepare, s);
    }
}

hipError_t prepare_variant(const PlanDev& p) {
    for (int dt : {DAS_IQ_C64, DAS_IQ_C16F, DAS_IQ_C16BF}) {
        const hipError_t e = dispatch_dt(p, nullptr, dt, nullptr, false, true, nullptr);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_das(const PlanDev& p, const void* iq, int dtype, void* out, hipStream_t s) {
    if (p.kp.n_tiles == 0) return hipSuccess;
    return dispatch_dt(p, iq, dtype, out, false, false, s);
}

bool per_tx_supported(const PlanDev& p) { return p.per_tx; }

hipError_t launch_das_per_tx(const PlanDev& p, const void* iq, int dtype, void* out, hipStream_t s) {
    if (p.kp.n_tiles == 0) return hipSuccess;
    return dispatch_dt(p, iq, dtype, out, true, false, s);
}

// ------------------------------------------------------------ variant rule
// A variant says how a plan cuts its work: FC frames per workgroup (waves of up to 16 frames; 32 in two halves), items
// of at most P - 1 window rows (P = 0: only the LDS bounds them), and whether (G > 1) element groups share a wave tile's
// items; it is kernel code for FC only.
#define DAS_VARIANTS(X)                                                                              \
    X(32, 41, 3) X(32, 49, 3) X(32, 33, 2) X(32, 65, 2) X(16, 33, 2) X(16, 65, 2) X(16, 129, 2) X(8, 33, 1) X(8, 65, 1)       \
    X(8, 129, 1) X(8, 257, 1) X(4, 33, 1) X(4, 65, 1) X(4, 129, 1) X(4, 257, 1) X(4, 513, 1) X(2, 129, 1)      \
    X(2, 257, 1) X(2, 513, 1) X(2, 1025, 1) X(1, 65, 1) X(1, 129, 1) X(1, 257, 1) X(1, 513, 1) X(1, 1025, 1) X(1, 2049, 1) \
    X(1, 65, 4) X(1, 129, 4) X(1, 257, 4) X(2, 129, 4) X(2, 257, 4) X(4, 65, 4) X(4, 129, 4) X(8, 65, 2) X(8, 65, 4) X(8, 33, 2) X(8, 129, 2) X(16, 65, 4) X(4, 65, 2) \
    X(1, 65, 2) X(1, 129, 2) X(1, 257, 2) X(2, 129, 2) X(2, 257, 2) X(4, 129, 2) X(8, 129, 4)                  \
    X(8, 257, 2) X(8, 257, 4) X(4, 257, 2) X(4, 257, 4) X(4, 513, 2) X(4, 513, 4) X(2, 513, 2) X(2, 513, 4) X(2, 1025, 2) \
    X(2, 1025, 4) X(1, 513, 2) X(1, 513, 4) X(1, 1025, 2) X(1, 1025, 4) X(1, 2049, 2) X(1, 2049, 4) \
    X(1, 0, 1) X(1, 0, 2) X(1, 0, 4) X(2, 0, 1) X(2, 0, 2) X(2, 0, 4)

// Variant choice, from the frame count, the longest tile window, the tile count and the items per tile:
//  - frames are cut into chunks of FC: 1, 2, 4, 8 or 16 by their number (the coefficients are formed once per chunk:
//    96^3 voxels x 8 frames 3.79 ms in one chunk, 4.69 in two of four; 256 x 256 x 32 frames 54 us in 16-frame chunks,
//    63 in 8-frame ones), 32 in two halves from 512 tiles on;
//  - with fewer workgroups than CUs (256), the frame chunk is halved until there are enough (84 x 263 x 4 frames:
//    22.7 us in one chunk of 8, 12.1 in two of 2);
//  - the pitch is the smallest that holds the longest tile window in one piece; one or two frames per workgroup on
//    tiles of fewer than 1200 items leave it open (P = 0);
//  - a launch should hold about 6144 waves (FC <= 4) or 2560 waves (FC >= 8), or 8192 when tiles carry 1024 or more
//    items on average: element groups are added until it does, up to 4.  For the launch they say whether a wave tile's items
//    are split at all (more than 1); how far, choose_split sets.
static bool variant_exists(int fc, int pitch, int g) {
#define DAS_HAS(FC_, P_, G_) \
    if (FC_ == fc && P_ == pitch && G_ == g) return true;
    DAS_VARIANTS(DAS_HAS)
#undef DAS_HAS
    return false;
}

// smallest pitch >= min_pitch with a (fc, pitch, g) variant, or -1
static int pitch_at_least(int fc, int min_pitch, int g) {
    int best = -1;
#define DAS_PIT(FC_, P_, G_) \
    if (FC_ == fc && G_ == g && P_ >= min_pitch && (best < 0 || P_ < best)) best = P_;
    DAS_VARIANTS(DAS_PIT)
#undef DAS_PIT
    return best;
}

Variant choose_variant(int frames, int max_window, int64_t n_tiles, double items_per_tile) {
    int fc;
    if (frames >= 32) fc = (n_tiles < 512) ? 16 : 32;
    else if (frames > 8) fc = 16;
    else if (frames > 4) fc = 8;
    else fc = frames > 2 ? 4 : frames > 1 ? 2 : 1;
    if (const char* env = std::getenv("DAS_VARIANT")) {  // tuning override: "fc,pitch,groups"
        int f = 0, pp = 0, g = 0;
        if (std::sscanf(env, "%d,%d,%d", &f, &pp, &g) == 3 && f <= (frames >= 32 ? 32 : fc * 2) &&
            variant_exists(f, pp, g))
            return Variant{f, pp, g};
    }
    if (fc == 32 && max_window <= 40) return Variant{32, 41, 3};
    if (fc == 32 && max_window <= 48) return Variant{32, 49, 3};
    auto chunks = [&](int f) { return (int64_t)((frames + f - 1) / f); };
    if (fc <= 16)
        while (fc > 1 && n_tiles * chunks(fc) < 256) fc /= 2;
    const int base_g = fc >= 16 ? 2 : 1;
    const int min_pitch = fc >= 8 ? 65 : 0;
    Variant best{0, 0, 0};
    const bool open = fc <= 2 && items_per_tile < 1200.0 && variant_exists(fc, 0, base_g);
    if (open) best = {fc, 0, base_g};
#define DAS_PICK(FC_, P_, G_)                                                                       \
    if (!open && FC_ == fc && G_ == base_g && P_ >= min_pitch && P_ > 0) {                        \
        if (best.fc == 0 || (best.pitch - 1 < max_window && P_ > best.pitch)) best = {FC_, P_, G_}; \
    }
    DAS_VARIANTS(DAS_PICK)
#undef DAS_PICK
    if (best.fc == 0 || best.fc > 16) return best;
    const int64_t target = items_per_tile >= 1024.0 ? 8192 : (best.fc <= 4 ? 6144 : 2560);
    for (int g = base_g; g <= 4; g *= 2) {
        const int p = pitch_at_least(best.fc, best.pitch, g);
        if (p >= 0 && (n_tiles * chunks(best.fc) * 4 * g >= target || g == 4)) return Variant{best.fc, p, g};
    }
    return best;
}

// Whether lanes gather their samples: where a wave's windows hold many rows on average (scattered points, grids of steps of
// many samples), staging them costs more than 64 lanes' own rows.  Staged and gathered, complex64, us by mean rows:
//   1 frame a chunk    58 rows 7.2, 8.9 (128 x 128, 64 elements); 68 rows 8.1, 5.2; 82 rows 25.8, 18.1 (20,000 points, 256
//                      elements); 131 rows 63, 46 (5000 points, 256 x 4 pairs); 196 rows 13.1, 5.2;
//   2                  68 rows 13.9, 14.9; 82 rows 239, 207; 131 rows 1538, 751;
//   4                  82 rows 471, 548; 113 rows 175, 157; 135 rows 36.9, 32.7;
//   8                  82 rows 287, 305; 116 rows 74, 64; 173 rows 80, 69;
//   16                 116 rows 113, 135; 173 rows 148, 155: always staged.
// Small launches cut their frames into small chunks; gathering ones of some tiles take more frames (the rows are read once
// instead of once a chunk, and groups make up for the workgroups): 16 frames, 5000 points (20 tiles) and 4 transmits 506 us in
// chunks of 1, 262 of 8; 8 frames, 8000 points (32 tiles) 56 of 1, 39 of 2, 28 of 4; but 1000 points (4 tiles) 20, 22, 33.
void choose_gather(PlanDev& p, double mean_rows) {
    p.per_tx = p.fc <= 2 && p.kp.T <= kPerTx;
    if (std::getenv("DAS_VARIANT") || p.fc >= 16 || mean_rows < (p.fc == 1 ? 64.0 : p.fc == 2 ? 80.0 : 100.0)) return;
    p.cap_rows = kGather;
    const int frames = p.kp.F, tiles = p.kp.n_tiles;
    const int least = tiles < 12 ? 1 : frames > 8 ? kGatherFrames : frames > 4 && tiles >= 16 ? 4 : frames > 2 ? 2 : 1;
    p.fc = std::max(p.fc, least);
}

// Workgroup shape and item length.
//
// Items: a window is cut only where its rows would take more than 10 KB of LDS (16 waves per CU), since every piece
// is a whole multiply-accumulate pass more.
//
// Groups: one wave tile per workgroup and four groups (4 waves) is the best or within 2 % of it on 18 of 21 measured
// shapes (256 x 256 x 32 frames: 1 / 2 / 4 / 8 groups 72 / 58 / 55 / 60 us; a 96^3 volume of 8 frames 4.00 / 3.89 /
// 3.79 / 3.84 ms; four wave tiles of four groups 62 us and 3.95 ms): small workgroups fill the tail of a launch.
// More groups pay where the launch stays short of 20000 waves and a group keeps 12 items (193 x 311, 3 transmits,
// 7 frames: 46.5 -> 44.7 us; 16 groups from 32 items on: 63 x 32 x 32, 6 transmits, 1 frame 56.9 -> 50.7 us), or
// where a group keeps 400 (96^3, 11 transmits: 3.27 -> 3.13 ms).  One group stays one where a wave tile has few items
// (under 256) and the launch holds many: splitting gains nothing there (223 x 368 x 72 frames 171.5 / 171.7 us).  Gathering
// waves take no LDS but for their sums: 16 groups up to 8192 waves (3000 points, 1 frame 17.1 -> 11.7 us).
void choose_split(PlanDev& p, int chunks, int max_wave_window, double items_per_tile) {
    const int fc = std::min(p.fc, 16), halves = p.fc / fc;  // frames per wave
    const int row = lds_row_bytes(fc);
    const int limit = p.pitch > 0 ? p.pitch - 1 : kMaxRows;
    int cap = std::max(1, std::min(max_wave_window, std::min(limit, kMaxRows)));
    cap = std::min(cap, 10 * 1024 / row - 1);
    const bool gather = p.cap_rows == kGather;
    if (!gather) p.cap_rows = cap;
    const int64_t units = (int64_t)p.kp.n_tiles * kWaves * chunks;
    int g = p.groups;
    if (gather) {
        g = units * 16 <= 8192 ? 16 : units * 8 <= 20000 ? 8 : 4;
    } else if (g > 1 || items_per_tile >= 256.0) {
        g = 4 / halves;
        if ((units * 8 <= 20000 && items_per_tile >= 8 * 12.0) || items_per_tile >= 8 * 400.0) g = 8;
        if (p.fc <= 4 && units * 16 <= 20000 && items_per_tile >= 16 * 32.0) g = 16;
    }
    p.split = g;
    p.n_wt = std::max(1, kWaves / (g * halves));
    int want[2] = {0, 0};
    if (const char* env = std::getenv("DAS_SPLIT"))  // tuning override: "groups,wave tiles", powers of two
        if (std::sscanf(env, "%d,%d", &want[0], &want[1]) == 2 && want[0] >= 1 && want[0] <= 16 && !(want[0] & (want[0] - 1)) &&
            (want[1] == 1 || want[1] == 2 || want[1] == 4)) {
            p.split = want[0];
            p.n_wt = want[1];
        }
    // the most that any IQ type's launch asks for
    const int rpi = fc <= 4 ? kLanes : kLanes / (fc / 4);
    auto waves = [&] { return (int64_t)p.n_wt * halves * p.split; };
    auto lds = [&] {
        const int64_t ntx = p.per_tx ? kPerTx : 1;
        return std::max(gather ? 0 : waves() * (((cap + rpi) / rpi * rpi + 2) * row), waves() * ntx * fc * kLanes * 8);
    };
    // (wave tiles and groups stay powers of two)
    while (waves() * kLanes > kMaxThreads || lds() > kLdsBytes) (p.n_wt > 1 ? p.n_wt : p.split) /= 2;
    // A launch of 2^32 threads and more wraps around.
    p.launch_units = (((int64_t)1 << 32) - 1) / (waves() * kLanes) / 8 * 8;
    if (const char* env = std::getenv("DAS_LAUNCH"))  // tuning override
        if (const long n = std::atol(env); n > 0) p.launch_units = std::min<int64_t>(n, p.launch_units);
}

int list_variants(int32_t* out, int capacity) {
    int n = 0;
#define DAS_LIST(FC_, P_, G_)                 \
    {                                         \
        if (out != nullptr && n < capacity) { \
            out[3 * n] = FC_;                 \
            out[3 * n + 1] = P_;              \
            out[3 * n + 2] = G_;              \
        }                                     \
        ++n;                                  \
    }
    DAS_VARIANTS(DAS_LIST)
#undef DAS_LIST
    return n;
}

// ------------------------------------------------- plane-wave arrival table
struct Normals {
    double n[16][3];
};

__global__ void tx_plane_wave_kernel(float* tx, const float* __restrict__ vox, int64_t n_vox, Normals nrm, int32_t t0,
                                     int32_t nt, double inv_c) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n_vox) return;
    const double x = vox[3 * v], y = vox[3 * v + 1], z = vox[3 * v + 2];
    for (int t = 0; t < nt; ++t) {
        const double a = nrm.n[t][0] * x + nrm.n[t][1] * y + nrm.n[t][2] * z;
        tx[(int64_t)(t0 + t) * n_vox + v] = (float)(a * inv_c);
    }
}

hipError_t launch_tx_plane_wave(float* tx_out, const float* vox_xyz, int64_t n_vox, const double* normals_host,
                                int32_t n_tx, double inv_c, hipStream_t s) {
    if (n_vox == 0) return hipSuccess;
    const int threads = 256;
    const int64_t blocks = (n_vox + threads - 1) / threads;
    for (int32_t t0 = 0; t0 < n_tx; t0 += 16) {
        Normals nr;
        const int nt = (n_tx - t0) < 16 ? (n_tx - t0) : 16;
        for (int t = 0; t < nt; ++t)
            for (int k = 0; k < 3; ++k) nr.n[t][k] = normals_host[3 * (t0 + t) + k];
        hipLaunchKernelGGL(tx_plane_wave_kernel, dim3((unsigned)blocks), dim3(threads), 0, s, tx_out, vox_xyz, n_vox, nr,
                           t0, nt, inv_c);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace das
