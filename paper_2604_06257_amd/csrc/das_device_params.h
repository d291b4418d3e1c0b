// Kernel parameter block (plain data shared by host and device code).
#pragma once

#include <stdint.h>

constexpr double kDasFix = 1572864.0;  // 1.5 * 2^20: added to a delay or phase, leaves 32 fraction bits (das_device.h)
constexpr int kDasFixHigh = 0x41380000;  // high word of kDasFix

struct das_kparams {
    int32_t T, E, S, F;
    int64_t n_slots;     // tiles * slots per tile
    int32_t n_tiles;
    int32_t use_apod;    // f# > 0
    double fs_c;         // fs / c: samples per metre of receive path
    double fd_c;         // fd / c: carrier cycles per metre of receive path
    double fs;
    double fd;
    double t0fs;         // t0 * fs
    double fix_t0;       // the fixed-point offset less t0 * fs and the rows that sample coordinates are counted from
    double fix_ph;       // the fixed-point offset less a whole number of carrier cycles
    int32_t row_fix;     // high word of a sample coordinate less this: the sample row
    float two_fnum;      // 2 f#
    float alpha;         // Tukey taper fraction
    float inv_2alpha;    // 1 / (2 alpha), 0 when alpha = 0
    float edge_2alpha;   // (1 - alpha) / (2 alpha), 0 when alpha = 0
    int32_t planar;      // every element lies in the plane z = z0
    double z0;           // that plane's depth (when planar)
    int32_t wide;        // rows or phases outside the fixed point's range: the general kernel
};
