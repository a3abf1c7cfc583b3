// Internal declarations of the resident CPM kernel.  Not part of the C ABI.
#pragma once
#include "spinmc_internal.hpp"

namespace spinmc {

// LDS bytes of the resident kernel: thresholds, five per-cell arrays of
// cell_cap entries, the waves' queues, and the ids with their halo (max_padded
// sites for the largest replica).
size_t cpm_resident_lds_bytes(int range, int tab_lds_bytes, int cell_cap, int max_sites,
                              int max_padded);

// n_steps Monte Carlo steps of every replica in one launch, one workgroup per
// replica (rows: range 1 with every Lx % 8 == 0); the device step counter is
// not advanced.  The launch holds steps sw0 .. sw0 + n_steps - 1 of
// a call; with re > 0, step k re of the call stores its statistics (the whole
// row) in stats row k - 1.
hipError_t launch_cpm_resident(const CpmArgs& a, bool rows, int n_steps, int sw0, int re,
                               int tab_lds_bytes, int cell_cap, int max_sites, int max_padded,
                               hipStream_t s);

// A tile of the streamed two-phase pass: rows y0 .. y0 + rows - 1 (even), columns
// x0 .. x0 + cols - 1 (multiples of 8) of the replica whose record it carries
// (one dependent load less than a tile and then its replica).
struct CpmTile {
    RepDev R;
    int32_t y0, rows, x0, cols;
};
size_t cpm_tile_lds_bytes(int tab_lds_bytes, int cell_cap, int threads, int rows, int cols);
hipError_t cpm_tile_reserve_lds(int cell_cap, size_t lds_bytes);
// One colour pass (range 1, every Lx % 8 == 0; cell_cap a multiple of 16, or 0: the
// cells' tables stay in global memory; threads
// a multiple of 64 up to 512; lds_bytes for the largest tile).
hipError_t launch_cpm_pass_tile(const CpmArgs& a, const CpmTile* tiles, int n_tiles, int c,
                                int sweep_off, int threads, int tab_lds_bytes, int cell_cap,
                                size_t lds_bytes, hipStream_t s);

// The same over bands of whole rows: x0 0, cols Lx, y0 and rows multiples of 3
// (range 2) or 2.  cell_cap 0 (always with
// range 2): the cells' tables stay in global memory.
size_t cpm_band_lds_bytes(int range, int tab_lds_bytes, int cell_cap, int threads, int rows,
                          int Lx);
hipError_t cpm_band_reserve_lds(int range, int cell_cap, size_t lds_bytes);
hipError_t launch_cpm_pass_band(const CpmArgs& a, const CpmTile* tiles, int n_tiles, int c,
                                int sweep_off, int threads, int tab_lds_bytes, int cell_cap,
                                size_t lds_bytes, hipStream_t s);

// Tiled persistent passes (range 1, Lx % 8 == 0, TH | Ly, TW | Lx, TH even,
// TW % 8 == 0): n_steps unrecorded Monte Carlo steps, one 256-thread
// workgroup per tile of every replica (n_blocks = R x tiles per replica, the
// same tile count for every replica); bar: one uint32 per replica, zero at
// launch; the device step counter is not advanced.
size_t cpm_tiled_lds_bytes(int tab_lds_bytes, int cell_cap, int TH, int TW);
hipError_t cpm_tiled_occupancy(int tab_lds_bytes, int cell_cap, int TH, int TW, int* per_cu);
hipError_t launch_cpm_tiled(const CpmArgs& a, int n_steps, int TH, int TW, int tab_lds_bytes,
                            int cell_cap, int n_blocks, uint32_t* bar, uint32_t* abort_flag,
                            hipStream_t s);

}  // namespace spinmc
