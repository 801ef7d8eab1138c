// rtc.hpp -- generated saturated generic kernels (hipRTC), see rtc.cpp.
#pragma once

#include <string>
#include <utility>
#include <vector>

#include "internal.hpp"

namespace stn {

// One coefficient group of one z slot: coefficient and its taps (dx, dy),
// in ascending address order.
struct RtcGroup {
    double coef;
    std::vector<std::pair<int, int>> taps;
};

// What a generated kernel depends on besides its tile.
struct RtcSpec {
    int R = 1, eb = 8;
    bool corners = false;
    long long row_bytes = 0;  // row pitch in bytes
    std::vector<std::vector<RtcGroup>> slots;  // 2R+1 slots, slot s holds dz = s - R
    // The plan's compiled kernels, by tile: a launch takes its kernel from
    // here.  (Emitting and hashing the source on each launch cost 90 us and
    // more, longer than most sweeps.)
    // ... and the text that identifies the stencil among the process's plans
    // (made by the first use)
    std::string key;
    struct Kernel {
        int tx, ty;
        hipFunction_t fn;
    };
    std::vector<Kernel> kernels;
};

// Thread rows (by) and rows per thread (ry) of a generated kernel's tile;
// by * ry = tile rows.
struct GenRows {
    int by, ry;
};
GenRows gen_rows(int tx, int ty);

// Compile (or fetch from the in-process and STENCIL_RTC_CACHE caches) kernel
// `kernel` of `src` for the current device; nullptr (error text set) on failure.
hipFunction_t rtc_function(const std::string &src, const char *kernel);

// The tile a plan takes when its descriptor leaves it open (FIXED tuning).
Tile rtc_default_tile(RtcSpec &sp, const Geom &g);
std::string rtc_generic_source(RtcSpec &sp, int TX, int TY);
// Stencils the process holds emission plans and kernels of.
size_t rtc_stencils();
// Compile the generated kernels of the given tiles (concurrently) and keep
// them in sp.kernels; false if any failed.
bool rtc_prepare(RtcSpec &sp, const std::vector<Tile> &tiles);
hipError_t rtc_generic_launch(const RtcSpec &sp, Tile t, const SweepArgs &a, hipStream_t s);

}  // namespace stn
