// Internal declarations of the multispin-coded Ising kernels (32 replicas
// per uint32 word).  Not part of the C ABI.
#pragma once
#include "spinmc_internal.hpp"

namespace spinmc {

constexpr int kModelIsingMsc = 5;
constexpr int kMscClasses = 18;  // 9 [s > 0] + 3 (Sx/2 + 1) + (Sy/2 + 1)

// What the thresholds of every group of a context have in common.
enum { kMscIso = 0, kMscSym = 1, kMscAny = 2 };

struct MscArgs {
    const RepDev* reps;       // per group: Lx, Ly, rid, lat_off (bytes)
    uint32_t* lat;            // packed words, two colour planes per group
    const uint64_t* tab;      // [G][18] thresholds (2^32 = always)
    const uint64_t* t_base;   // device sweep counter
    int32_t* stats;           // [rows][32 G][width]
    uint32_t key0, key1;
    int32_t G, width;         // groups; stats rows hold 32 G replicas
    int32_t max_blocks;       // max over groups of Lx Ly / 8
    int32_t max_sites;
    int32_t mode;             // kMscIso, kMscSym or kMscAny
};

hipError_t launch_msc_init(const MscArgs& a, hipStream_t s);
hipError_t launch_msc_pass(const MscArgs& a, int c, int sweep_off, hipStream_t s);
// Adds [M, Bx, By] of replica 32 g + b to stats row rec_row (zeroed first).
hipError_t launch_msc_stats(const MscArgs& a, int rec_row, hipStream_t s);
// LDS bytes of a resident workgroup of `lanes` lanes (a multiple of 64), `rows`
// (2, 4 or 8) rows of four words of each plane a lane.
inline size_t msc_resident_lds(int rows, int lanes) {
    return (size_t)lanes * 32 * (2 + (rows + 3) / 4) + 384;
}
// n_sweeps sweeps of every group in one launch, one workgroup a group: every
// group has Ly >= rows and (Lx / 8) ceil(Ly / rows) <= lanes <= 1024.  The
// launch holds sweeps sw0 .. sw0 + n_sweeps - 1 of a call; with re > 0, sweep
// k re of the call stores its statistics in stats row k - 1.
hipError_t launch_msc_resident(const MscArgs& a, int rows, int lanes, int n_sweeps, int sw0, int re,
                               hipStream_t s);

}  // namespace spinmc
