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

// Thread rows (by) and rows per thread (ry) of a generated kernel's tile;
// by * ry = tile rows.
struct GenRows {
    int by, ry;
};

// What a generated kernel depends on besides its tile.
struct RtcSpec {
    int R = 1, eb = 8;
    bool corners = false;
    long long row_bytes = 0;  // row pitch in bytes
    std::vector<std::vector<RtcGroup>> slots;  // 2R+1 slots, slot s holds dz = s - R
    // the text that identifies the stencil among the process's plans (made by
    // the first use)
    std::string key;
    // The plan's compiled kernels, by tile: a launch takes its kernel from
    // here.  (Emitting and hashing the source on each launch cost 90 us and
    // more, longer than most sweeps.)
    struct Kernel {
        Tile t;
        GenRows rows;
        hipFunction_t fn;
    };
    std::vector<Kernel> kernels;
    const Kernel *kernel(const Tile &t) const {
        for (const Kernel &k : kernels)
            if (k.t.tx == t.tx && k.t.ty == t.ty && k.t.tz == t.tz) return &k;
        return nullptr;
    }
    Tile fitted{};  // what rtc_default_tile chose for the plan
};

// The rows of a tile's own.
GenRows gen_rows(int tx, int ty);

// Compile (or fetch from the in-process and STENCIL_RTC_CACHE caches) kernel
// `kernel` of `src` for the current device; nullptr (error text set) on failure.
hipFunction_t rtc_function(const std::string &src, const char *kernel);

// The tile a plan takes when its descriptor leaves it open (FIXED tuning).
Tile rtc_default_tile(RtcSpec &sp, const Geom &g);
// Rows per thread of a plan's launches at tile t.
GenRows rtc_rows(RtcSpec &sp, Tile t, const Geom &g);
std::string rtc_generic_source(RtcSpec &sp, int TX, int TY, GenRows gr);
// A generated kernel's work at tile t over grids g, for the cost model.
struct RtcWork {
    GenRows rows;
    double fp64;       // FP64 instructions per output
    int lds_eb;        // bytes per LDS cell
    double registers;  // estimate: accumulators, plane sums, a column of cells
};
RtcWork rtc_work(RtcSpec &sp, Tile t, const Geom &g);
// Stencils the process holds emission plans and kernels of.
size_t rtc_stencils();
// Drop sp's entry if no kernel was made for it.
void rtc_forget(RtcSpec &sp);
// Compile the generated kernels of the given tiles over grids g (concurrently)
// and keep them in sp.kernels; false if any failed.
bool rtc_prepare(RtcSpec &sp, const std::vector<Tile> &tiles, const Geom &g);
hipError_t rtc_generic_launch(const RtcSpec &sp, Tile t, const SweepArgs &a, hipStream_t s);

}  // namespace stn
