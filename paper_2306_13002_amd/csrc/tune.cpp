// tune.cpp -- exhaustive autotuner for stencil plans.
//
// For a plan's kind, dtype, boundary and geometry it enumerates every
// offered (variant, tile, zblock, tile map) that the descriptor leaves open,
// runs each on private buffers of the same layout (filled with benign
// constants) on a private stream, and keeps the candidate with the lowest
// median time per sweep.  Results are cached per geometry in-process and,
// when STENCIL_TUNE_CACHE names a file, in that file as JSON lines that a
// later process reloads verbatim.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/stencil.h"
#include "internal.hpp"
#include "plan.hpp"
#include "tune.hpp"
#include "rtc.hpp"

namespace stn {

stencil_status fail(stencil_status st, const char *fmt, ...);
void logf(const char *fmt, ...);
stencil_status hip_fail(hipError_t e, const char *what);
int elem_bytes(int dtype);

namespace {

std::mutex g_mu;
std::map<std::string, TuneEntry> g_cache;
bool g_file_loaded = false;

const char *cache_path() {
    const char *e = std::getenv("STENCIL_TUNE_CACHE");
    return (e && *e) ? e : nullptr;
}

void load_file_locked() {
    if (g_file_loaded) return;
    g_file_loaded = true;
    const char *path = cache_path();
    if (!path) return;
    FILE *f = std::fopen(path, "r");
    if (!f) return;
    char line[1024], key[512];
    while (std::fgets(line, sizeof line, f)) {
        TuneEntry e{};
        // {"key": "...", "variant": V, "tx": X, "ty": Y, "zb": Z, "map": M, "us": U[, "run": [V, X, Y, Z]]}
        if (std::sscanf(line, " {\"key\": \"%511[^\"]\", \"variant\": %d, \"tx\": %d, \"ty\": %d, \"zb\": %d, "
                              "\"map\": %d, \"us\": %lf}",
                        key, &e.variant, &e.tile.tx, &e.tile.ty, &e.tile.tz, &e.remap, &e.us) == 7) {
            const char *run = std::strstr(line, "\"run\": [");
            if (run && std::sscanf(run, "\"run\": [%d, %d, %d, %d]", &e.run_variant, &e.run_tile.tx, &e.run_tile.ty,
                                   &e.run_tile.tz) != 4)
                e.run_variant = -1;
            g_cache[key] = e;
        }
    }
    std::fclose(f);
}

void append_file_locked(const std::string &key, const TuneEntry &e) {
    const char *path = cache_path();
    if (!path) return;
    FILE *f = std::fopen(path, "a");
    if (!f) return;
    std::fprintf(f, "{\"key\": \"%s\", \"variant\": %d, \"tx\": %d, \"ty\": %d, \"zb\": %d, \"map\": %d, \"us\": %.4f",
                 key.c_str(), e.variant, e.tile.tx, e.tile.ty, e.tile.tz, e.remap, e.us);
    if (e.run_variant >= 0)
        std::fprintf(f, ", \"run\": [%d, %d, %d, %d]", e.run_variant, e.run_tile.tx, e.run_tile.ty, e.run_tile.tz);
    std::fprintf(f, "}\n");
    std::fclose(f);
}

const Tile kPlainTiles[] = {{64, 4, 1},  {64, 2, 2},  {128, 2, 1}, {256, 1, 1}, {32, 8, 1},
                            {64, 8, 1},  {128, 4, 1}, {128, 8, 1}, {256, 2, 1}};
const int kZblocks[] = {4, 8, 16, 32, 64, 128, 256};

}  // namespace

std::vector<Cand> tune_candidates(const KindOps *ops, int kind, const Geom &g, const TuneRequest &rq) {
    std::vector<Cand> out;
    auto want_v = [&](int v) { return rq.variant == STENCIL_AUTO || rq.variant == v; };
    auto tile_fits = [&](const Tile &t) {
        return (!rq.tile_x || rq.tile_x == t.tx) && (!rq.tile_y || rq.tile_y == t.ty) &&
               (!rq.zblock || rq.zblock == t.tz);
    };
    if (want_v(V_PLAIN))
        for (const Tile &t : kPlainTiles)
            if (ops->tile_ok(V_PLAIN, t) && tile_fits(t)) out.push_back({V_PLAIN, t, 0});
    // HEAT2D5 PLAIN with fused sweeps (Dirichlet): square output tiles, 2..16
    // sweeps per launch; the last six fill a 32 x 32 region exactly
    if (want_v(V_PLAIN) && kind == STENCIL_HEAT2D5 && rq.bc == STENCIL_BC_DIRICHLET) {
        std::vector<Tile> ft;
        for (int ot : {16, 32})
            for (int k : {2, 4, 5, 8, 10, 16}) ft.push_back(Tile{ot, ot, k});
        for (int k : {2, 4, 5, 6, 10, 12}) ft.push_back(Tile{32 - 2 * k, 32 - 2 * k, k});
        for (const Tile &t : ft)
            if (ops->tile_ok(V_PLAIN, t) && tile_fits(t)) out.push_back({V_PLAIN, t, 0});
    }
    // two sweeps per pass hold the boundary fixed between them; the Poisson
    // kernel addresses a plane with 32-bit byte offsets
    const bool sat2_fits = rq.bc == STENCIL_BC_DIRICHLET &&
                           (kind != STENCIL_POISSON19 || g.pz * (long long)sizeof(float) <= kMaxPlaneBytes32);
    if ((rq.variant == V_SAT2 || rq.variant == STENCIL_AUTO) && ops->sat2_tiles && sat2_fits) {
        Tile st[64];
        const int ns = ops->sat2_tiles(st, 64);
        std::vector<int> zbs;
        for (int zb : kZblocks)
            if (zb < g.nz) zbs.push_back(zb);
        zbs.push_back(g.nz);
        for (int s = 0; s < ns; ++s)
            for (int zb : zbs) {
                Tile t{st[s].tx, st[s].ty, zb};
                if (!ops->tile_ok(V_SAT2, t) || !tile_fits(t)) continue;
                for (int m = 1; m <= 2; ++m)
                    if (!rq.tile_map || rq.tile_map == m) out.push_back({V_SAT2, t, m == 2 ? 1 : 0});
            }
    }
    // the three-sweep form (HEAT3D7, Dirichlet); its z-blocks also between the
    // powers of two: with one or two blocks per CU, how evenly the blocks fill
    // the chip moves a pass by several per cent
    if ((rq.variant == V_SAT3 || rq.variant == STENCIL_AUTO) && ops->sat3_tiles && rq.bc == STENCIL_BC_DIRICHLET) {
        Tile st[16];
        const int ns = ops->sat3_tiles(st, 16);
        std::vector<int> zbs;
        for (int zb : {4, 8, 12, 16, 20, 24, 32, 40, 48, 64, 128, 256})
            if (zb < g.nz) zbs.push_back(zb);
        zbs.push_back(g.nz);
        for (int s = 0; s < ns; ++s)
            for (int zb : zbs) {
                Tile t{st[s].tx, st[s].ty, zb};
                if (!ops->tile_ok(V_SAT3, t) || !tile_fits(t)) continue;
                for (int m = 1; m <= 2; ++m)
                    if (!rq.tile_map || rq.tile_map == m) out.push_back({V_SAT3, t, m == 2 ? 1 : 0});
            }
    }
    if (want_v(V_SATURATED) && ops->sat_tiles) {
        Tile st[64];
        const int ns = ops->sat_tiles(st, 64);
        std::vector<int> zbs;
        if (kind == STENCIL_GENERIC) {
            // z depth trades planes loaded for their neighbours only against
            // block count
            for (int zb : {4, 8, 16, 32, 64})
                if (zb < g.nz) zbs.push_back(zb);
        } else {
            for (int zb : kZblocks)
                if (zb < g.nz) zbs.push_back(zb);
        }
        zbs.push_back(g.nz);
        for (int s = 0; s < ns; ++s)
            for (int zb : zbs) {
                Tile t{st[s].tx, st[s].ty, zb};
                if (!ops->tile_ok(V_SATURATED, t) || !tile_fits(t)) continue;
                for (int m = 1; m <= 2; ++m)
                    if (!rq.tile_map || rq.tile_map == m) out.push_back({V_SATURATED, t, m == 2 ? 1 : 0});
            }
    }
    return out;
}

std::vector<Cand> run_candidates(int kind, const Geom &g, const TuneRequest &rq) {
    std::vector<Cand> out;
    if (rq.tile_x || rq.tile_y || rq.zblock) return out;
    if (kind == STENCIL_HEAT2D5 && rq.bc == STENCIL_BC_DIRICHLET)
        for (int k : {4, 5, 8}) out.push_back({V_MARCH, h2_march_tile(k, g), 0});
    if (kind != STENCIL_HEAT3D7) return out;
    for (int v : {(int)V_SATURATED, (int)V_SAT2, (int)V_SAT3}) {
        if (rq.variant != STENCIL_AUTO && rq.variant != v) continue;
        if (v != V_SATURATED && rq.bc != STENCIL_BC_DIRICHLET) continue;
        Tile rt[8];
        const int n = h3_rt_tiles(v, rt);
        for (int i = 0; i < n; ++i)
            for (int zb : {2, 4, 8, 16, 32})
                if (zb == 2 || zb < 2 * g.nz) out.push_back({v, Tile{rt[i].tx, rt[i].ty, zb}, 1});
    }
    return out;
}

bool same_grids(int kind, int form, int run) {
    if (kind == STENCIL_HEAT2D5) return form == V_PLAIN && run == V_MARCH;
    auto sat = [](int v) { return v == V_SATURATED || v == V_SAT2 || v == V_SAT3; };
    return kind == STENCIL_HEAT3D7 && sat(form) && sat(run);
}

void settle_run(int kind, const std::vector<Cand> &cands, const std::vector<std::pair<double, size_t>> &timed,
                const std::vector<Cand> &runs, const std::vector<double> &run_us, TuneEntry *best) {
    if (runs.empty()) return;
    const size_t r = std::min_element(run_us.begin(), run_us.end()) - run_us.begin();
    if (run_us[r] >= best->us) return;
    if (!same_grids(kind, best->variant, runs[r].variant)) {
        size_t i = 0;
        while (i < timed.size() && !same_grids(kind, cands[timed[i].second].variant, runs[r].variant)) ++i;
        if (i == timed.size()) return;
        const Cand &c = cands[timed[i].second];
        best->variant = c.variant;
        best->tile = c.tile;
        best->remap = c.remap;
        best->us = timed[i].first;
    }
    best->run_variant = runs[r].variant;
    best->run_tile = runs[r].tile;
}

namespace {

struct Buffers {
    void *f[2] = {nullptr, nullptr};
    void *c[12] = {};
    int nc = 0;
    ~Buffers() {
        for (void *q : f)
            if (q) (void)hipFree(q);
        for (void *q : c)
            if (q) (void)hipFree(q);
    }
};

}  // namespace

std::string tune_key(const stencil_plan_s *p, const TuneRequest &rq) {
    char buf[512];
    // "/c10": candidate set 10 (AUTO includes the two- and three-sweep forms
    // where boundaries are fixed, the latter with intermediate z-blocks;
    // HEAT2D5 the fused plain sweeps with one-cell-per-thread tiles; GENERIC
    // tiles of 16 and 32 rows and z-blocks from 4; the closest candidates
    // re-timed; launches only of the reported form's result); entries of
    // earlier sets are not reused
    std::snprintf(buf, sizeof buf, "k%d/d%d/bc%d/n%dx%dx%d/r%d/py%lld/pz%lld/v%d/t%d,%d,%d,%d/h%08x/c10", p->kind,
                  p->dtype, p->bc, p->g.nx, p->g.ny, p->g.nz, p->g.r, p->g.py, p->g.pz, rq.variant, rq.tile_x,
                  rq.tile_y, rq.zblock, rq.tile_map, p->taps_hash);
    return buf;
}

// Whether a tuner could have made this entry for the request: a launch shape
// that is not offered would divide by zero or fail at every launch.
static bool entry_offered(const KindOps *ops, int kind, const TuneRequest &rq, const TuneEntry &e) {
    const bool fixed = rq.bc == STENCIL_BC_DIRICHLET;
    auto form_ok = [&](int v) {
        switch (v) {
        case V_PLAIN: return true;
        case V_SATURATED: return ops->sat_tiles != nullptr;
        case V_SAT2: return ops->sat2_tiles && fixed;
        case V_SAT3: return ops->sat3_tiles && fixed;
        default: return false;
        }
    };
    const Tile &t = e.tile;
    if (!form_ok(e.variant) || (rq.variant != STENCIL_AUTO && rq.variant != e.variant) || !ops->tile_ok(e.variant, t) ||
        (rq.tile_x && rq.tile_x != t.tx) || (rq.tile_y && rq.tile_y != t.ty) || (rq.zblock && rq.zblock != t.tz) ||
        (launch_sweeps(kind, e.variant, t) > 1 && !fixed))
        return false;
    if (e.run_variant < 0) return true;
    if (rq.tile_x || rq.tile_y || rq.zblock || !same_grids(kind, e.variant, e.run_variant)) return false;
    if (e.run_variant == V_MARCH) return fixed;
    return form_ok(e.run_variant) && ops->tile_ok(e.run_variant, e.run_tile);
}

bool tune_lookup(const std::string &key, const KindOps *ops, int kind, const TuneRequest &rq, TuneEntry *out) {
    std::lock_guard<std::mutex> lk(g_mu);
    load_file_locked();
    auto it = g_cache.find(key);
    if (it == g_cache.end()) return false;
    if (!entry_offered(ops, kind, rq, it->second)) {
        logf("tune cache: entry of %s is not offered; tuning again", key.c_str());
        return false;
    }
    *out = it->second;
    return true;
}

void tune_store(const std::string &key, const TuneEntry &e) {
    std::lock_guard<std::mutex> lk(g_mu);
    load_file_locked();
    g_cache[key] = e;
    append_file_locked(key, e);
}

// Time one candidate: T sweeps back to back, `reps` times; median per sweep (us).
static double time_one(const stencil_plan_s *p, const Cand &c, Buffers &b, hipStream_t s, hipEvent_t e0,
                       hipEvent_t e1, int T, int reps, hipError_t *err) {
    SweepArgs a = p->base_args;
    a.remap = c.remap;
    a.part = nullptr;
    const int per = launch_sweeps(p->kind, c.variant, c.tile);
    a.sweeps = per;
    for (int i = 0; i < b.nc; ++i) a.coefs[i] = b.c[i];
    std::vector<double> ts;
    const bool wave = p->kind == STENCIL_WAVE25;
    for (int r = 0; r < reps + 1; ++r) {  // first repetition warms up
        void *src = wave ? b.f[1] : b.f[0], *dst = wave ? b.f[0] : b.f[1];
        if ((*err = hipEventRecord(e0, s)) != hipSuccess) return 0;
        for (int t = 0; t < T; ++t) {
            a.src = src;
            a.dst = dst;
            if ((*err = p->ops->launch(c.variant, c.tile, a, s)) != hipSuccess) return 0;
            std::swap(src, dst);
        }
        if ((*err = hipEventRecord(e1, s)) != hipSuccess) return 0;
        if ((*err = hipEventSynchronize(e1)) != hipSuccess) return 0;
        float ms = 0;
        if ((*err = hipEventElapsedTime(&ms, e0, e1)) != hipSuccess) return 0;
        if (r > 0) ts.push_back(1e3 * ms / (T * per));
    }
    std::sort(ts.begin(), ts.end());
    return ts[ts.size() / 2];
}

stencil_status tune_exhaustive(stencil_plan_s *p, const TuneRequest &rq, TuneEntry *best) {
    const std::vector<Cand> cands = tune_candidates(p->ops, p->kind, p->g, rq);
    if (cands.empty()) return fail(STENCIL_E_UNSUPPORTED, "no launch shape matches the requested tile fields");
    if (p->kind == STENCIL_GENERIC && p->base_args.rtc) {  // compile the generated kernels up front, in parallel
        std::vector<Tile> tiles;
        for (const Cand &c : cands)
            if (c.variant == V_SATURATED) tiles.push_back(c.tile);
        if (!tiles.empty() && !rtc_prepare(*p->rtc, tiles, p->g)) {
            logf("%s; tuning the table-driven generic kernel", stencil_last_error());
            p->base_args.rtc = nullptr;
        }
    }
    const int eb = elem_bytes(p->dtype);
    const long long span = (long long)(p->g.PZ() - 1) * p->g.pz * (p->rz ? 1 : 0) +
                           (long long)(p->g.PY() - 1) * p->g.py + p->g.PX();
    const size_t bytes = (size_t)span * eb;
    Buffers b;
    hipError_t e;
    for (int i = 0; i < 2; ++i)
        if ((e = hipMalloc(&b.f[i], bytes)) != hipSuccess) return fail(STENCIL_E_NOMEM, "tuner buffers: %s", hipGetErrorString(e));
    b.nc = p->kind == STENCIL_POISSON19 ? 12 : (p->kind == STENCIL_WAVE25 ? 1 : 0);  // GENERIC: none
    const size_t cb = p->kind == STENCIL_POISSON19 ? (size_t)span * 4 : bytes;
    for (int i = 0; i < b.nc; ++i)
        if ((e = hipMalloc(&b.c[i], cb)) != hipSuccess) return fail(STENCIL_E_NOMEM, "tuner buffers: %s", hipGetErrorString(e));
    hipStream_t s = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if ((e = hipStreamCreate(&s)) != hipSuccess) return hip_fail(e, "hipStreamCreate");
    struct Cleanup {
        hipStream_t s;
        hipEvent_t *a, *b;
        ~Cleanup() {
            if (*a) (void)hipEventDestroy(*a);
            if (*b) (void)hipEventDestroy(*b);
            if (s) (void)hipStreamDestroy(s);
        }
    } cleanup{s, &e0, &e1};
    if ((e = hipEventCreate(&e0)) != hipSuccess || (e = hipEventCreate(&e1)) != hipSuccess)
        return hip_fail(e, "hipEventCreate");
    // benign values: the state stays bounded under every kind's update
    const double fv = 1.0;
    for (int i = 0; i < 2; ++i)
        if ((e = launch_fill(b.f[i], span, eb, fv, s)) != hipSuccess) return hip_fail(e, "fill");
    for (int i = 0; i < b.nc; ++i) {
        const double cv = p->kind == STENCIL_WAVE25 ? 0.01 : 0.1;
        if ((e = launch_fill(b.c[i], span, p->kind == STENCIL_POISSON19 ? 4 : eb, cv, s)) != hipSuccess)
            return hip_fail(e, "fill");
    }
    // sweeps per timing: about 1 ms of work per repetition, 2..50 sweeps
    hipError_t te = hipSuccess;
    double probe = time_one(p, cands[0], b, s, e0, e1, 2, 1, &te);
    if (te != hipSuccess) return hip_fail(te, "tuner launch");
    int T = (int)std::min(50.0, std::max(2.0, 1000.0 / std::max(probe, 1.0)));
    TuneEntry bestv{};
    bestv.us = 1e300;
    std::vector<std::pair<double, size_t>> timed;
    for (size_t i = 0; i < cands.size(); ++i) {
        const Cand &c = cands[i];
        const double us = time_one(p, c, b, s, e0, e1, T, 3, &te);
        if (te != hipSuccess) return hip_fail(te, "tuner launch");
        logf("tune kind=%d v=%d tile=(%d,%d,%d) map=%d: %.2f us/sweep", p->kind, c.variant, c.tile.tx, c.tile.ty,
             c.tile.tz, c.remap ? 2 : 1, us);
        timed.push_back({us, i});
    }
    // candidates within 5 % of the fastest (at most eight) are timed again
    // with more repetitions, so that the pick does not rest on one noisy median
    std::sort(timed.begin(), timed.end());
    for (size_t r = 0; r < timed.size() && r < 8 && timed[r].first <= 1.05 * timed[0].first; ++r) {
        const Cand &c = cands[timed[r].second];
        const double us = time_one(p, c, b, s, e0, e1, T, 9, &te);
        if (te != hipSuccess) return hip_fail(te, "tuner launch");
        if (us < bestv.us) {
            bestv.us = us;
            bestv.variant = c.variant;
            bestv.tile = c.tile;
            bestv.remap = c.remap;
        }
    }
    const std::vector<Cand> runs = run_candidates(p->kind, p->g, rq);
    std::vector<double> run_us;
    for (const Cand &c : runs) {
        run_us.push_back(time_one(p, c, b, s, e0, e1, T, 3, &te));
        if (te != hipSuccess) return hip_fail(te, "tuner launch");
        logf("tune kind=%d launches v=%d tile=(%d,%d,%d): %.2f us/sweep", p->kind, c.variant, c.tile.tx, c.tile.ty,
             c.tile.tz, run_us.back());
    }
    settle_run(p->kind, cands, timed, runs, run_us, &bestv);
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    *best = bestv;
    return STENCIL_OK;
}

}  // namespace stn
