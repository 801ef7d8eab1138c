// tune.hpp -- autotuner interface (exhaustive search and its cache).
#pragma once

#include <string>
#include <utility>
#include <vector>

#include "../../include/stencil.h"

#include "internal.hpp"

struct stencil_plan_s;

namespace stn {

struct RtcSpec;

// What the descriptor leaves open: variant STENCIL_AUTO and 0-valued fields
// are searched; other values restrict the candidates.
struct TuneRequest {
    int variant, tile_x, tile_y, zblock, tile_map;
    int bc = STENCIL_BC_DIRICHLET;  // fused HEAT2D5 sweeps are offered for Dirichlet plans only
};

// Sweeps one launch of (kind, variant, tile) performs: the two-sweep form
// does two; HEAT2D5 PLAIN with tile.tz > 1 fuses tile.tz sweeps per launch.
inline int launch_sweeps(int kind, int variant, const Tile &t) {
    if (variant == V_MARCH) return t.tx;
    if (kind == STENCIL_HEAT2D5 && variant == V_PLAIN && t.tz > 1) return t.tz;
    return sweeps_per_launch(variant);
}

struct TuneEntry {
    int variant;  // V_PLAIN, V_SATURATED, V_SAT2 or V_SAT3
    Tile tile;
    int remap;    // 0 natural, 1 XCD-chunked
    double us;    // median time per sweep of (variant, tile)
    // what the plan launches instead where that is faster still with the same
    // results (settle_run); run_variant < 0: nothing
    int run_variant = -1;
    Tile run_tile{};
};

// One launch candidate: form, shape and tile map (remap 1 = XCD-chunked).
struct Cand {
    int variant;
    Tile tile;
    int remap;
};

// Static description of a stencil used by the cost model's features.
struct StencilInfo {
    int kind, dtype, eb, r;
    Geom g;
    int n_taps;        // points read per update from the state grid
    int n_coef;        // distinct coefficients (coefficient arrays for POISSON19)
    int n_groups;      // saturated tap groups (GENERIC), else distinct coefficients
    double box_frac;   // fraction of taps with two or more nonzero offsets
    RtcSpec *rtc;      // GENERIC: what its saturated kernels are generated from
};

StencilInfo stencil_info(const stencil_desc *d, const Geom &g);
// Candidates the tuners consider for a plan's kind and geometry, restricted
// by the request's fixed fields.
std::vector<Cand> tune_candidates(const KindOps *ops, int kind, const Geom &g, const TuneRequest &rq);
// Launches the tuners time beside the candidates of a request that leaves the
// shape open (see TuneEntry::run_variant).
std::vector<Cand> run_candidates(int kind, const Geom &g, const TuneRequest &rq);
// Whether launches of form `run` leave the grids of reported form `form` bit
// for bit: HEAT2D5 PLAIN runs may march, the saturated HEAT3D7 forms stand for
// each other; PLAIN adds in another order than those.
bool same_grids(int kind, int form, int run);
// Let the fastest of the timed launches (us, index into runs) replace what
// `best` launches if it is faster.  A pick of another result gives way to the
// fastest timed candidate (sorted by us) of the launch's result, so that the
// plan reports a form whose grids it produces.
void settle_run(int kind, const std::vector<Cand> &cands, const std::vector<std::pair<double, size_t>> &timed,
                const std::vector<Cand> &runs, const std::vector<double> &run_us, TuneEntry *best);
void cost_features(const StencilInfo &si, const Cand &c, float out[24]);
stencil_status tune_model(stencil_plan_s *p, const TuneRequest &rq, TuneEntry *best);

std::string tune_key(const stencil_plan_s *p, const TuneRequest &rq);
// The cached pick of a request, if there is one and what it names is offered
// (entries may come from a file).
bool tune_lookup(const std::string &key, const KindOps *ops, int kind, const TuneRequest &rq, TuneEntry *out);
void tune_store(const std::string &key, const TuneEntry &e);
stencil_status tune_exhaustive(stencil_plan_s *p, const TuneRequest &rq, TuneEntry *best);

}  // namespace stn
