// Internal interfaces between the C ABI (das_api.cpp) and the kernels
// (das_kernels.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime_api.h>
#include <hip/hip_vector_types.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "das_device_params.h"

namespace das {

constexpr int kWaves = 4;               // waves per workgroup tile
constexpr int kLanes = 64;              // gfx950 wavefront
constexpr int kSlots = kWaves * kLanes; // voxel slots per tile

// Host-side voxel tiling: slot -> voxel index (-1 = empty slot).
struct Tiling {
    int32_t tile_dims[3] = {0, 0, 0};   // lattice points per tile (0: not a lattice)
    int32_t wave_dims[3] = {0, 0, 0};   // lattice points per wave
    int64_t n_tiles = 0;
    std::vector<int32_t> slot_to_vox;   // n_tiles * kSlots
    std::vector<int32_t> tile_xyz;      // n_tiles * 3 tile coordinates (lattice), else (index, 0, 0)
};

// Returns 0 or a negative das_status; err receives a message.
int tile_points(const float* xyz, int64_t n, const char* override_spec, Tiling& out, std::string& err);

constexpr int kLdsBytes = 160 * 1024;   // LDS of a CU, the most a workgroup can have

// LDS bytes of one staged row of FC frames.
constexpr int lds_row_bytes(int fc) { return fc <= 2 ? 8 * fc : 8 * fc + 16; }

// A work item of a wave tile, laid out so that the kernel's scalar work per item is short (scalar instructions issue
// once per four cycles and SIMD: at one frame they bound the kernel):
//   x, y  offset of its first loaded sample (frame 0) in the channel data, in samples: 48 bits, bits 16-31 of y left
//         to the rows loaded (bits 16-23: the window's rows and the one after them, less what lies past the record)
//         and the window's rows (bits 24-31)
//   z     the window's first row + row_fix (the high word of a fixed-point sample coordinate in that row);
//         a window that begins at row -1 loads from row 0
//   w     element << kTxBits | transmit (a split that depends on the plan took two more scalar registers and 2 % of the time
//         of three transmits apart at 96^3 x 1024 elements, 1009 -> 1034 us)
constexpr int kTxBits = 14, kMaxTx = 1 << kTxBits, kMaxElem = 1 << (32 - kTxBits), kMaxRows = 254;
constexpr int kGather = 1 << 30;  // cap_rows of plans whose lanes gather their samples: whole windows, rows left out
constexpr int kItemPad = 4;  // items past the end that a wave may read ahead
#ifdef __HIPCC__
__host__ __device__
#endif
inline int4 pack_item(int e, int t, int row, int rows, int E, int S, int F, int row_fix) {
    const int from = row < 0 ? 0 : row, end = row + rows + 1 < S ? row + rows + 1 : S, loaded = end - from;
    const int64_t off = (((int64_t)t * E + e) * S + from) * F;
    return int4{(int)(uint32_t)off, (int)((uint32_t)(off >> 32) | (uint32_t)loaded << 16 | (uint32_t)rows << 24),
                row + row_fix, (int)((uint32_t)e << kTxBits | (uint32_t)t)};
}

struct PlanDev {
    das_kparams kp;
    float* vx = nullptr;       // [n_slots]
    float* vy = nullptr;
    float* vz = nullptr;
    float* tx = nullptr;       // [n_slots / 64][T][64]
    int32_t* slot_vox = nullptr;  // [n_slots]
    double* elemd = nullptr;   // [E][4] element coordinates (float32 inputs held in FP64), x y z 0
    int4* items = nullptr;     // per wave tile, its work items, element-major (and kItemPad more at the end)
    uint32_t* item_off = nullptr;  // [n_tiles * kWaves + 1] offsets into items, in pairs of them
    int4* wg_unit = nullptr;      // workgroup -> first wave tile, frame chunk, and that tile's first pair of items and pairs
    int32_t fc = 0, pitch = 0, groups = 1;  // kernel variant: frames per workgroup, most rows per item + 1, element groups
    int32_t n_wt = kWaves, split = 1;       // wave tiles and element groups of a workgroup
    int32_t cap_rows = 0;                   // most rows of an item
    bool per_tx = false;                    // per-transmit output is served
    int64_t launch_units = 0;               // most workgroups of a launch
    int64_t n_vox = 0;                      // voxels (per-transmit output stride: n_vox * F)
};

// Workgroup -> unit order: each of the 8 XCDs gets a lateral region of tile columns (all depths), heaviest units
// first inside a region, regions interleaved so that workgroup w runs on XCD w % 8.  A unit is a run of n_wt wave
// tiles of one tile, times the frame chunk.
std::vector<int32_t> order_units(const Tiling& tl, const std::vector<uint32_t>& item_off, int n_wt, int chunks);

// Kernel variant for F frames, the largest tile window (rows), the tile count and the average number of
// (transmit, element) items per tile.
struct Variant {
    int fc, pitch, groups;
};
Variant choose_variant(int frames, int max_window, int64_t n_tiles, double items_per_tile);

// Sets what the plan's variant says of its kernel: per_tx, and for windows of many rows on average that lanes gather their
// samples (cap_rows = kGather, possibly more frames per workgroup).
void choose_gather(PlanDev& p, double mean_rows);

// Sets the plan's workgroup shape (n_wt, split) and item length (cap_rows) for its variant, the frame chunks, the
// longest wave window and the items per tile.
void choose_split(PlanDev& p, int chunks, int max_wave_window, double items_per_tile);

// The compiled variants as (fc, pitch, groups) triples: writes min(count, capacity) of them to out (when not
// null) and returns the count.
int list_variants(int32_t* out, int capacity);

// Computes per (wave tile, element, transmit) sample windows (first row, rows) of n tiles from tile0 on, and counts:
// counts[0] = active (slot, e, t) triples (w > 0, inside the record);
// counts[1] = processed triples (valid slots of tiles whose window is not
// empty); counts[2] = longest tile window; counts[3] = longest wave window;
// counts[4], counts[5] = rows and number of the wave windows that are not empty.
hipError_t launch_windows(const PlanDev& p, int tile0, int n, int2* win, unsigned long long* counts, hipStream_t s);

// Items of those tiles' wave tiles (pieces of at most cap_rows rows): their numbers, even and at most INT32_MAX - 1 (items =
// null), or the items at off (in pairs).
hipError_t launch_items(const PlanDev& p, int tile0, int n, const int2* win, const uint32_t* off, int4* items,
                        int32_t* n_items, hipStream_t s);

// Raises the dynamic LDS limit of the plan's kernels (all IQ types).
hipError_t prepare_variant(const PlanDev& p);

hipError_t launch_das(const PlanDev& p, const void* iq, int dtype, void* out, hipStream_t s);
// Per-transmit output [T][V][F] (variants with at most 2 frames per workgroup, T <= 4).
bool per_tx_supported(const PlanDev& p);
hipError_t launch_das_per_tx(const PlanDev& p, const void* iq, int dtype, void* out, hipStream_t s);

hipError_t launch_tx_plane_wave(float* tx_out, const float* vox_xyz, int64_t n_vox, const double* normals_host,
                                int32_t n_tx, double inv_c, hipStream_t s);

}  // namespace das
