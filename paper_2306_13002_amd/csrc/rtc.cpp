// rtc.cpp -- saturated generic stencils generated for one stencil and
// compiled at plan time with hipRTC.
//
// This is the paper's code-generation step (Sec. Code Generation) done at
// run time for the taps a plan was given: the saturated expression -- taps
// grouped by coefficient id and z offset, each group summed before it is
// multiplied, the sums shared among rows and planes, or one FMA per tap where
// sharing saves little (SlotEmitter, emit_plan) -- is emitted as straight-line
// HIP with compile-time LDS offsets and exact coefficient literals, wrapped
// around the streaming body every generic kernel shares (generic_body.hpp), and
// compiled for the device.  Modules are cached per source text in-process and,
// when STENCIL_RTC_CACHE names a directory, as code-object files there.
// rtc_function serves every generated kernel of the library (also the
// saturator's programs).
#include <hip/hip_runtime.h>
#include <hip/hiprtc.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "../../include/stencil.h"
#include "internal.hpp"
#include "rtc.hpp"
#include "rtc_headers.inc"  // kCommonHppText, kGenericBodyHppText (written by the build)

namespace stn {

stencil_status fail(stencil_status st, const char *fmt, ...);
void logf(const char *fmt, ...);

namespace {

std::mutex g_mu;
std::map<std::string, hipFunction_t> g_fn;  // hash of source and kernel name + device -> kernel

unsigned long long fnv64(const std::string &s) {
    unsigned long long h = 1469598103934665603ull;
    for (unsigned char c : s) h = (h ^ c) * 1099511628211ull;
    return h;
}

// Whether by_planes keeps a sum for slot s: it pays for two taps or more (of the
// centre column: where the plane has others too).
bool plane_sum(const RtcSpec &sp, int s, bool centre) {
    int mid = 0, n = 0;
    for (const RtcGroup &gr : sp.slots[s])
        for (const auto &t : gr.taps) {
            ++n;
            mid += t.first == 0;
        }
    return centre ? mid > 1 && n > mid : n > 1;
}

// Emits one plane's contributions to the accumulator queue for every row of
// a thread.  Values are named once and shared (the paper's common
// subexpressions): a cell of the window is read from LDS once, a mirrored
// pair u(-dx) + u(+dx) of a window row once for all the output rows that use
// it, a pair of such rows (dy, -dy) and a whole group's sum once for all the
// z slots whose groups have the same in-plane shape.
struct SlotEmitter {
    const RtcSpec &sp;
    const int RY, W, phase;  // phase: see generic_rows_body
    std::string o;
    std::map<std::string, std::string> memo;  // expression -> name
    int n_add = 0, n_fma = 0, n_cell = 0, n_name = 0;
    std::set<std::string> sums;  // by_sums: what it holds at once

    SlotEmitter(const RtcSpec &sp_, int ry, int w, int ph) : sp(sp_), RY(ry), W(w), phase(ph) {}

    std::string named(const std::string &expr) {
        auto it = memo.find(expr);
        if (it != memo.end()) return it->second;
        const std::string nm = "v" + std::to_string(n_name++);
        o += "        const double " + nm + " = " + expr + ";\n";
        return memo[expr] = nm;
    }
    std::string add(const std::string &a, const std::string &b) {
        const std::string expr = a + " + " + b;
        if (!memo.count(expr)) ++n_add;
        return named(expr);
    }
    // cell dx of window row wy (row m of the thread is window row m + R)
    std::string cell(int dx, int wy) {
        const std::string expr = "t[me + " + std::to_string((wy - sp.R) * W + dx) + "]";
        if (!memo.count(expr)) ++n_cell;
        return named(expr);
    }
    std::string tree(const std::vector<std::string> &v, size_t a, size_t b) {
        if (b - a == 1) return v[a];
        const size_t m = a + (b - a + 1) / 2;
        const std::string l = tree(v, a, m);
        return add(l, tree(v, m, b));
    }
    // the sum of a group's taps for output row m
    std::string sum(const RtcGroup &gr, int m) {
        const int R = sp.R, w = 2 * R + 1;
        std::vector<int> has(w * w, 0);
        for (const auto &t : gr.taps) has[(t.second + R) * w + t.first + R]++;
        // per row dy: mirrored pairs, then single cells (a tap named twice counts twice)
        std::vector<std::string> terms;
        auto item = [&](int kind, int dx, int dy) {  // kind 1: the pair of |dx|, 0: one cell
            const int wy = m + R + dy;
            if (!kind) return cell(dx, wy);
            const std::string l = cell(-dx, wy);
            return add(l, cell(dx, wy));
        };
        std::vector<std::pair<int, int>> rows[9];  // dy + R -> (kind, dx)
        for (int dy = -R; dy <= R; ++dy) {
            int *h = &has[(dy + R) * w];
            for (int dx = R; dx >= 1; --dx)
                while (h[R + dx] > 0 && h[R - dx] > 0) {
                    rows[dy + R].push_back({1, dx});
                    --h[R + dx];
                    --h[R - dx];
                }
            for (int dx = -R; dx <= R; ++dx)
                for (; h[R + dx] > 0; --h[R + dx]) rows[dy + R].push_back({0, dx});
        }
        for (int dy = 0; dy <= R; ++dy) {
            std::vector<std::pair<int, int>> up = rows[R + dy], dn = dy ? rows[R - dy] : std::vector<std::pair<int, int>>();
            for (const auto &it : up) {
                auto f = std::find(dn.begin(), dn.end(), it);
                if (f != dn.end()) {
                    dn.erase(f);
                    const std::string l = item(it.first, it.second, -dy);
                    terms.push_back(add(l, item(it.first, it.second, dy)));
                } else {
                    terms.push_back(item(it.first, it.second, dy));
                }
            }
            for (const auto &it : dn) terms.push_back(item(it.first, it.second, -dy));
        }
        return tree(terms, 0, terms.size());
    }
    static std::string lit(double c) {
        char buf[48];
        std::snprintf(buf, sizeof buf, "%a", c);
        return buf;
    }
    // acc of slot s += c * v for row m (the queue starts each slot at 0)
    std::string acc_name(int s, int m) const {
        const int w = 2 * sp.R + 1;
        return "acc[" + std::to_string((s - phase + w) % w) + "][" + std::to_string(m) + "]";
    }
    void fma_into(int s, int m, double c, const std::string &v) {
        const std::string dst = acc_name(s, m);
        o += "        " + dst + " = fma(" + lit(c) + ", " + v + ", " + dst + ");\n";
        ++n_fma;
    }
    bool guarded = false;  // skip the slots that are not live
    void guard(int s) { o += guarded ? "        if (live >> " + std::to_string(s) + " & 1) {\n" : std::string("        {\n"); }
    // The sums of every row first, shared among the slots, then slot by slot
    // one FMA per group and row: for patterns whose sums repeat (a symmetric
    // box adds and multiplies several times fewer values than it has taps).
    void by_sums() {
        const int NQ = 2 * sp.R + 1;
        std::vector<std::vector<std::vector<std::string>>> v(NQ, std::vector<std::vector<std::string>>(RY));
        for (int m = 0; m < RY; ++m)
            for (int s = 0; s < NQ; ++s)
                for (const RtcGroup &gr : sp.slots[s]) {
                    v[s][m].push_back(sum(gr, m));
                    sums.insert(v[s][m].back());
                }
        for (int s = 0; s < NQ; ++s) {
            if (sp.slots[s].empty()) continue;
            guard(s);
            for (size_t g = 0; g < sp.slots[s].size(); ++g)
                for (int m = 0; m < RY; ++m) fma_into(s, m, sp.slots[s][g].coef, v[s][m][g]);
            o += "        }\n";
        }
    }
    // The taps for which `takes` holds, column by column of the window, so that
    // a column's cells are all that is held; each coefficient is used for all
    // the thread's rows at once, one FMA per tap and row by fma(slot, row, dx, ...).
    template <class Takes, class Fma>
    void by_columns(Takes takes, Fma fma) {
        const int R = sp.R, w = 2 * R + 1, NQ = 2 * R + 1;
        std::vector<std::vector<std::vector<double>>> c(NQ, std::vector<std::vector<double>>(w * w));
        for (int s = 0; s < NQ; ++s)
            for (const RtcGroup &gr : sp.slots[s])
                for (const auto &t : gr.taps)
                    if (takes(gr)) c[s][(t.second + R) * w + t.first + R].push_back(gr.coef);
        for (int dx = 0; dx < w; ++dx) {
            for (int dy = 0; dy < w; ++dy)
                for (int s = 0; s < NQ; ++s)
                    for (int m = 0; m < RY && !c[s][dy * w + dx].empty(); ++m) cell(dx - R, m + dy);
            for (int s = 0; s < NQ; ++s) {
                bool any = false;
                for (int dy = 0; dy < w; ++dy)
                    for (double v : c[s][dy * w + dx]) {
                        if (!any) guard(s);
                        any = true;
                        for (int m = 0; m < RY; ++m) fma(s, m, dx - R, v, cell(dx - R, m + dy));
                    }
                if (any) o += "        }\n";
            }
        }
    }
    // For patterns whose sums do not repeat: one FMA per tap into its slot.
    void by_taps() {
        by_columns([](const RtcGroup &) { return true; },
                   [this](int s, int m, int, double c, const std::string &v) { fma_into(s, m, c, v); });
    }
    // ... in the written order of rounding: the groups of one tap by columns,
    // then row by row and slot by slot the groups of several, each a tree and
    // one FMA.
    void by_groups() {
        const int R = sp.R, NQ = 2 * R + 1;
        by_columns([](const RtcGroup &gr) { return gr.taps.size() == 1; },
                   [this](int s, int m, int, double c, const std::string &v) { fma_into(s, m, c, v); });
        for (int m = 0; m < RY; ++m)
            for (int s = 0; s < NQ; ++s) {
                bool any = false;
                for (const RtcGroup &gr : sp.slots[s])
                    for (const auto &t : gr.taps)
                        if (gr.taps.size() > 1) {
                            cell(t.first, m + R + t.second);
                            any = true;
                        }
                if (!any) continue;
                guard(s);
                const std::map<std::string, std::string> outer = memo;  // names made inside the guard end with it
                for (const RtcGroup &gr : sp.slots[s])
                    if (gr.taps.size() > 1) fma_into(s, m, gr.coef, sum(gr, m));
                memo = outer;
                o += "        }\n";
            }
    }
    // ... and with one sum per plane, or (centre) one for the taps of a plane's
    // centre column: an FMA per tap into a sum that starts at 0 with the plane
    // and is added to the slot once; the other taps straight into the slot.
    // Holds a column's cells where trees hold the window's.
    void by_planes(bool centre) {
        const int NQ = 2 * sp.R + 1;
        std::vector<char> sums(NQ);
        for (int s = 0; s < NQ; ++s) sums[s] = plane_sum(sp, s, centre);
        auto part = [](int s, int m) { return "p" + std::to_string(s) + "_" + std::to_string(m); };
        for (int s = 0; s < NQ; ++s)
            for (int m = 0; m < RY && sums[s]; ++m) o += "        double " + part(s, m) + " = 0.0;\n";
        by_columns([](const RtcGroup &) { return true; },
                   [&](int s, int m, int dx, double c, const std::string &v) {
                       if (!sums[s] || (centre && dx)) return fma_into(s, m, c, v);
                       o += "        " + part(s, m) + " = fma(" + lit(c) + ", " + v + ", " + part(s, m) + ");\n";
                   });
        for (int s = 0; s < NQ; ++s) {
            if (!sums[s]) continue;
            guard(s);
            for (int m = 0; m < RY; ++m) o += "        " + acc_name(s, m) + " += " + part(s, m) + ";\n";
            o += "        }\n";
        }
    }
};

}  // namespace

namespace {

// How a stencil's plane arithmetic is emitted for RY rows per thread.
struct EmitPlan {
    int ry;
    enum { SUMS, TAPS, PLANES, CENTRES, GROUPS } order;  // by_sums, by_taps, by_planes, by_groups
    int per_plane;  // FP64 instructions per thread and plane
    bool rotate;    // the accumulator queue moves on by name
    bool guarded;   // slots that are not live are skipped
    bool narrow;    // F32 storage: the LDS tile holds F32, widened at each read
};

// What a kernel's source depends on besides its tile and wide_rows, as text.
const std::string &spec_key(RtcSpec &sp) {
    if (!sp.key.empty()) return sp.key;
    std::string k;
    auto put = [&k](const void *v, size_t n) { k.append((const char *)v, n); };
    const int head[3] = {sp.R, sp.eb, sp.corners};
    put(head, sizeof head);
    for (const auto &sl : sp.slots) {
        const int n = (int)sl.size();
        put(&n, sizeof n);
        for (const RtcGroup &g : sl) {
            const int m = (int)g.taps.size();
            put(&g.coef, sizeof g.coef);
            put(&m, sizeof m);
            for (const auto &t : g.taps) {
                put(&t.first, sizeof t.first);
                put(&t.second, sizeof t.second);
            }
        }
    }
    return sp.key = k;
}

// Whether a tile's rows span too much for 32-bit lane offsets.
bool wide_rows(const RtcSpec &sp, int TY) { return (TY + 2 * sp.R) * sp.row_bytes >= 0xFFFFFFF0LL; }

// Per stencil of the process: how it is emitted, and its kernels per tile and
// device.  A plan of a stencil that another plan has compiled takes both from
// here instead of emitting the source again (0.3 to 3 ms).  Entries stay as
// long as the modules do, and there are no more of them: grids of other
// extents and pitches share them.
struct SpecEntry {
    std::vector<EmitPlan> emit;
    std::map<std::vector<int>, hipFunction_t> fn;  // tx, ty, rows per thread, device, wide_rows
};
std::map<std::string, SpecEntry> g_specs;  // guarded by g_mu

// Squares of the rounded values' magnitudes, summed over the roundings of one
// output, with every cell at 1 (the mean square of the error up to a factor):
// the tap sums as written -- per plane and coefficient a balanced tree and one
// FMA -- and by_planes' two orders.
struct Rounding {
    double groups = 0, planes = 0, centres = 0;
};
double tree_rounding(double c, size_t n) {
    if (n < 2) return 0;
    const size_t m = (n + 1) / 2;
    return c * c * n * n + tree_rounding(c, m) + tree_rounding(c, n - m);
}
double plane_rounding(const RtcSpec &sp, bool centre) {
    double e = 0, acc = 0;
    for (int s = 0; s < (int)sp.slots.size(); ++s) {
        const bool sums = plane_sum(sp, s, centre);
        double part = 0;
        for (int dx = -sp.R; dx <= sp.R; ++dx)  // a column at a time
            for (const RtcGroup &gr : sp.slots[s])
                for (const auto &t : gr.taps) {
                    if (t.first != dx) continue;
                    double &h = sums && !(centre && dx) ? part : acc;
                    h += std::fabs(gr.coef);
                    e += h * h;
                }
        acc += part;
        if (sums) e += acc * acc;
    }
    return e;
}
Rounding rounding(const RtcSpec &sp) {
    Rounding e;
    double acc = 0;
    for (const auto &sl : sp.slots)
        for (const RtcGroup &gr : sl) {
            const double c = std::fabs(gr.coef);
            acc += c * gr.taps.size();
            e.groups += acc * acc + tree_rounding(c, gr.taps.size());
        }
    e.planes = plane_rounding(sp, false);
    e.centres = plane_rounding(sp, true);
    return e;
}

EmitPlan emit_plan(RtcSpec &sp, int ry) {
    const std::string &key = spec_key(sp);
    {
        std::lock_guard<std::mutex> lk(g_mu);
        auto it = g_specs.find(key);
        if (it != g_specs.end())
            for (const EmitPlan &e : it->second.emit)
                if (e.ry == ry) return e;
    }
    int taps = 0;
    for (const auto &sl : sp.slots)
        for (const RtcGroup &g : sl) taps += (int)g.taps.size();
    SlotEmitter er(sp, ry, 1024, 0);
    er.by_sums();
    EmitPlan p;
    p.ry = ry;
    // The shared sums win where they save at least a tenth of one FMA per tap
    // (a symmetric box of radius 3: 100 instead of 343 instructions per point)
    // and fit the registers (40 sums there; box r = 4 with ten coefficients has
    // 360, in scratch 30 % slower than sums per plane).
    // One FMA per tap where that is the written order too (no coefficient
    // repeats in a plane) and for F32 storage, whose rounding of the result (at
    // 2^-24) hides the sums'.  Otherwise the order that rounds no more than the
    // written one: rms error against it, 10 coefficients drawn for a box, sums
    // per plane 0.52 at r = 2 and 0.49 at r = 4 (one FMA per tap 1.8 and 2.8),
    // a star r = 4 with a sum for its centre column 0.99.  us per sweep, one
    // FMA per tap, trees and this: those boxes at 256 x 200 x 160 54, 53, 55 and
    // 239, 319, 251; the star at 321 x 190 x 257 80, 82, 79.
    const Rounding err = rounding(sp);
    bool single = true;
    for (const auto &sl : sp.slots)
        for (const RtcGroup &g : sl) single &= g.taps.size() == 1;
    const bool shared = 10 * (er.n_add + er.n_fma) <= 9 * ry * taps && er.sums.size() <= 128;
    // (Decided at four rows per thread for every tile, so that all of a
    // stencil's kernels round alike.)
    p.order = ry != 4                                     ? emit_plan(sp, 4).order
              : shared                                    ? EmitPlan::SUMS
              : single || sp.eb == 4                      ? EmitPlan::TAPS
              : err.planes <= err.groups                  ? EmitPlan::PLANES
              : err.centres <= err.groups                 ? EmitPlan::CENTRES
                                                          : EmitPlan::GROUPS;
    p.per_plane = p.order == EmitPlan::SUMS ? er.n_add + er.n_fma : ry * taps;
    // The rotating queue repeats the plane's arithmetic 2R+1 times: taken up
    // to 4096 FP64 instructions (32 KB of the 64 KB instruction cache).
    p.rotate = p.per_plane * (2 * sp.R + 1) <= 4096;
    // Skipping pays from about 64 instructions per point on (box r = 2, 125
    // coefficients: 81 -> 64 us a sweep at 201 x 233 x 160); the branches cost
    // small stencils more (star r = 1 at 64^3: 8.4 -> 10.4 us).
    p.guarded = p.per_plane >= 64 * ry;
    // Widening F32 cells once, as they are staged, doubles the LDS bytes of
    // every read: worth it unless the stencil does little arithmetic per cell
    // (star r = 4 321 x 190 x 257: F32 in LDS 56.0 us a sweep, FP64 58.1; box r
    // = 2 201 x 233 x 160: 61.6 against 57.4).
    p.narrow = sp.eb == 4 && p.per_plane < 4 * er.n_cell;
    std::lock_guard<std::mutex> lk(g_mu);
    g_specs[key].emit.push_back(p);
    return p;
}

}  // namespace

// Grids that stream from memory: F64 of radius 1, beyond the Infinity Cache, or
// beyond 96 MB where a cell costs at most 16 instructions.  The time is then the
// rate of the loads and stores, which 64 x 4 tiles with one row per thread keep
// highest (many small blocks, rows of whole lines).  us per sweep, such tiles
// and the fitted ones: star r = 1 256 x 200 x 160 23.3 and 26.4, 321 x 190 x 257
// 42.7 and 51, 400^3 252 and 306, 500 x 300 x 260 159 and 159; box r = 1 of 27
// coefficients 350^3 181 and 204, but 256 x 256 x 128 27.8 and 27.5.
bool streams(RtcSpec &sp, const Geom &g) {
    const double mb = 2.0 * g.nx * g.ny * g.nz * sp.eb / (1 << 20);
    return sp.eb == 8 && sp.R == 1 && g.nx >= 64 && (mb > 320 || (mb > 96 && emit_plan(sp, 4).per_plane <= 4 * 16));
}

// Default tile of a generated kernel: the tile and z-block with the lowest
// estimate, in cycles, of
//   [live planes * 7 FP64 + planes * (150 + 250 cells staged per thread)
//    + 60 outputs per thread] * (waves per SIMD + 0.7).
// The constants are a fit to 109 random stencils and grids (edges 65..321) at
// six tiles and six z-blocks each: the pick is within 3.1 % of the best of
// those in the geometric mean (within 28 % in the worst case); 32 or 64 x 16
// tiles alone, with the z-block from a simpler estimate, were 7 % off (45 %).
// Where the two grids exceed the L2s (8 x 4 MB), a stencil of little
// arithmetic takes no z-block shorter than its halo: the planes that blocks
// load again then come from memory (star r = 3 f64 288 x 92 x 148 after other
// work: a call of one sweep 60.9 us with z-blocks of 4, 55.3 with 8).  Small
// z-blocks and tiles give more waves, large ones fewer planes and rings that are
// loaded only for their neighbours.  Measured us per sweep at that rule -> now:
// star r = 4 f64 118 x 86 x 177 22.7 -> 15.8, f32 134 x 267 x 73 25.4 -> 19.6;
// box r = 3 symmetric f64 127 x 164 x 252 53.0 -> 45.4; box r = 3 f64
// 65 x 101 x 177 53.9 -> 44.0.
Tile rtc_default_tile(RtcSpec &sp, const Geom &g) {
    const double mb = 2.0 * g.nx * g.ny * g.nz * sp.eb / (1 << 20);
    const Tile large{64, 4, 16};
    auto blocks = [&g](Tile t) { return cdiv(g.nx, t.tx) * cdiv(g.ny, t.ty) * cdiv(g.nz, t.tz); };
    if (streams(sp, g)) return mb > 320 || blocks({64, 4, 8}) > kNoallocPartials ? large : Tile{64, 4, 8};
    static const Tile tiles[] = {{64, 16, 0}, {32, 32, 0}, {32, 16, 0}, {32, 8, 0}, {64, 4, 0}, {32, 4, 0}};
    const bool beyond_l2 = 2.0 * g.nx * g.ny * g.nz * sp.eb > (32 << 20);
    Tile best{0, 0, 0};
    double cost = 0;
    for (Tile t : tiles) {
        const GenRows gr = gen_rows(t.tx, t.ty);
        const EmitPlan ep = emit_plan(sp, gr.ry);
        const double waves = t.tx * gr.by / 64.0;
        const double staged = (double)(t.tx + 2 * sp.R) * (t.ty + 2 * sp.R) / (t.tx * gr.by);
        for (int zb : {2, 4, 8, 16, 32, 64}) {
            if (zb > 2 && zb >= 2 * g.nz) break;
            if (zb < 2 * sp.R && !ep.guarded && beyond_l2 && zb < g.nz) continue;
            const double per_cu = (double)cdiv(cdiv(g.nx, t.tx) * cdiv(g.ny, t.ty) * cdiv(g.nz, zb), 256);
            const double out = std::min(zb, g.nz), planes = out + 2 * sp.R, live = ep.guarded && ep.order != EmitPlan::SUMS ? out : planes;
            const double block = live * 7 * ep.per_plane + planes * (150 + 250 * staged) + out * gr.ry * 60;
            const double est = block * (per_cu * waves / 4 + 0.7);
            if (cost == 0 || est < cost) {
                cost = est;
                best = Tile{t.tx, t.ty, zb};
            }
        }
    }
    // streaming stars of radius 2 take tall tiles: 400^3 328 -> 276 us a sweep,
    // 321 x 190 x 257 58 -> 52, 288 x 250 x 250 84 -> 80
    if (sp.eb == 8 && sp.R == 2 && mb > 200 && emit_plan(sp, 4).per_plane <= 4 * 16) best = Tile{64, 16, 8};
    // flat and thin grids whose partials only longer blocks keep within the
    // allocation-free run's scratch (the table-driven kernel's) take those
    if (blocks(best) > kNoallocPartials && blocks(large) <= kNoallocPartials) best = large;
    sp.fitted = best;
    return best;
}

// Rows per thread of a tile that a caller or a tuner asks for: the tile's own,
// unless these leave few waves per SIMD (less than one, or 1.75 in long
// z-blocks).  The chip then waits for each wave's chain, which one row per
// thread makes shortest.  us per sweep, own rows and one: box r = 2
// 140 x 184 x 20 at 32x8x16 36.4 and 17.8, star r = 4 20 x 30 x 110 at 32x8x64
// 48.7 and 27.3, box r = 2 18 x 163 x 97 at 128x2x32 (one wave) 65 and 39;
// beyond, box r = 2 167 x 181 x 213 at 32x4x32 (two waves) 62.9 and 71.7, box
// r = 3 42 x 99 x 229 at 32x8x4 (1.5) 40 and 57.  Of 150 stencils, grids and
// tiles the rule loses 12 % once and 3 % at most otherwise.  (The default tile
// is fitted with its own rows.)  Streaming grids: one row (streams).
GenRows rtc_rows(RtcSpec &sp, Tile t, const Geom &g) {
    const GenRows own = gen_rows(t.tx, t.ty);
    if (t.tx == sp.fitted.tx && t.ty == sp.fitted.ty && t.tz == sp.fitted.tz) return own;
    const long long per_cu = cdiv(cdiv(g.nx, t.tx) * cdiv(g.ny, t.ty) * cdiv(g.nz, t.tz), 256);
    const bool few = per_cu * t.tx * own.by < (std::min(t.tz, g.nz) < 16 ? 256 : 448);  // threads per CU
    return t.tx * t.ty <= 256 && (few || streams(sp, g)) ? GenRows{t.ty, 1} : own;
}

std::string rtc_generic_source(RtcSpec &sp, int TX, int TY, GenRows gr) {
    const int R = sp.R, W = TX + 2 * R;
    const EmitPlan ep = emit_plan(sp, gr.ry);
    std::string o;
    char buf[320];
    o += "#include \"generic_body.hpp\"\n\nnamespace {\nstruct GenSlots {\n    static constexpr bool rotate = ";
    o += ep.rotate ? "true;\n" : "false;\n";
    std::snprintf(buf, sizeof buf,
                  "    template <int PH>\n    __device__ __forceinline__ void add(const %s *__restrict__ t, int me, "
                  "unsigned live, double (*acc)[%d]) const {\n",
                  ep.narrow ? "float" : "double", gr.ry);
    o += buf;
    for (int ph = 0; ph < (ep.rotate ? 2 * R + 1 : 1); ++ph) {
        SlotEmitter em(sp, gr.ry, W, ph);
        em.guarded = ep.guarded;
        if (ep.order == EmitPlan::SUMS) em.by_sums();
        else if (ep.order == EmitPlan::TAPS) em.by_taps();
        else if (ep.order == EmitPlan::GROUPS) em.by_groups();
        else em.by_planes(ep.order == EmitPlan::CENTRES);
        std::snprintf(buf, sizeof buf, "        if constexpr (PH == %d) {\n", ph);
        o += buf + em.o + "        }\n";
    }
    o += "    }\n};\n}  // namespace\n\n";
    const char *T = sp.eb == 4 ? "float" : "double";
    std::snprintf(buf, sizeof buf,
                  "extern \"C\" __global__ __launch_bounds__(%d) void stencil_generic_gen(const %s *__restrict__ src, "
                  "%s *__restrict__ dst, stn::Geom g, int zb, int remap, double *__restrict__ part) {\n",
                  TX * gr.by, T, T);
    o += buf;
    std::snprintf(buf, sizeof buf, "    __shared__ %s tile[2][%d];\n    __shared__ double red[16];\n",
                  ep.narrow ? "float" : "double", (TY + 2 * R) * W);
    o += buf;
    o += "    int bx, by, bz;\n    stn::tile_coords(remap, bx, by, bz);\n";
    std::snprintf(buf, sizeof buf,
                  "    const double sacc = stn::generic_rows_body<%s, %d, %d, %d, %d, %s, %s>(src, dst, g, zb, bx, by, bz, "
                  "part != nullptr, GenSlots{}, tile);\n",
                  T, R, TX, gr.by, gr.ry, sp.corners ? "true" : "false",
                  wide_rows(sp, TY) ? "unsigned long long" : "unsigned");
    o += buf;
    o += "    if (part) {\n        const double s = stn::block_sum_f64(sacc, red);\n";
    o += "        if (threadIdx.x == 0 && threadIdx.y == 0) part[stn::block_linear_id()] = s;\n    }\n}\n";
    return o;
}

RtcWork rtc_work(RtcSpec &sp, Tile t, const Geom &g) {
    RtcWork w;
    w.rows = rtc_rows(sp, t, g);
    const EmitPlan ep = emit_plan(sp, w.rows.ry);
    const int ry = w.rows.ry, q = 2 * sp.R + 1, out = std::min(t.tz, g.nz);
    // slots that are not live cost nothing where they are skipped
    const double planes = ep.guarded && ep.order != EmitPlan::SUMS ? 1.0 : (out + 2.0 * sp.R) / out;
    w.fp64 = (double)ep.per_plane / ry * planes;
    w.lds_eb = ep.narrow ? 4 : 8;
    w.registers = 40 + 2.0 * q * ry * (ep.order == EmitPlan::PLANES ? 2 : 1) + 2.0 * (ry + 2 * sp.R);
    return w;
}

void rtc_forget(RtcSpec &sp) {
    const std::string &key = spec_key(sp);
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_specs.find(key);
    if (it != g_specs.end() && it->second.fn.empty()) g_specs.erase(it);
}

size_t rtc_stencils() {
    std::lock_guard<std::mutex> lk(g_mu);
    return g_specs.size();
}

// Compile (or fetch from the caches) kernel `kernel` of source `src`;
// returns nullptr and sets the error text on failure.
hipFunction_t rtc_function(const std::string &src, const char *kernel) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    char key[96];
    std::snprintf(key, sizeof key, "%016llx-%d", fnv64(src + '\n' + kernel), dev);
    {
        std::lock_guard<std::mutex> lk(g_mu);
        auto it = g_fn.find(key);
        if (it != g_fn.end()) return it->second;
    }
    std::vector<char> code;
    const char *cache = std::getenv("STENCIL_RTC_CACHE");
    std::string path;
    if (cache && *cache) {
        path = std::string(cache) + "/" + key + ".co";
        if (FILE *f = std::fopen(path.c_str(), "rb")) {
            std::fseek(f, 0, SEEK_END);
            const long n = std::ftell(f);
            std::fseek(f, 0, SEEK_SET);
            code.resize(n > 0 ? n : 0);
            if (n <= 0 || std::fread(code.data(), 1, n, f) != (size_t)n) code.clear();
            std::fclose(f);
        }
    }
    if (code.empty()) {
        hiprtcProgram prog;
        const char *hdrs[] = {kCommonHppText, kGenericBodyHppText};
        const char *names[] = {"common.hpp", "generic_body.hpp"};
        if (hiprtcCreateProgram(&prog, src.c_str(), "generated.hip", 2, hdrs, names) != HIPRTC_SUCCESS) {
            fail(STENCIL_E_DEVICE, "hiprtcCreateProgram failed");
            return nullptr;
        }
        const char *opts[] = {"--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off",
                              "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"};
        const hiprtcResult r = hiprtcCompileProgram(prog, 8, opts);
        if (r != HIPRTC_SUCCESS) {
            size_t ln = 0;
            hiprtcGetProgramLogSize(prog, &ln);
            std::string log(ln + 1, '\0');
            hiprtcGetProgramLog(prog, &log[0]);
            fail(STENCIL_E_DEVICE, "hipRTC compile of generated kernel %s failed: %.400s", kernel, log.c_str());
            hiprtcDestroyProgram(&prog);
            return nullptr;
        }
        size_t n = 0;
        hiprtcGetCodeSize(prog, &n);
        code.resize(n);
        hiprtcGetCode(prog, code.data());
        hiprtcDestroyProgram(&prog);
        if (!path.empty())
            if (FILE *f = std::fopen(path.c_str(), "wb")) {
                std::fwrite(code.data(), 1, code.size(), f);
                std::fclose(f);
            }
    }
    hipModule_t mod = nullptr;
    hipFunction_t fn = nullptr;
    hipError_t e = hipModuleLoadData(&mod, code.data());
    if (e == hipSuccess) e = hipModuleGetFunction(&fn, mod, kernel);
    if (e != hipSuccess) {
        fail(STENCIL_E_DEVICE, "loading generated kernel %s: %s", kernel, hipGetErrorString(e));
        return nullptr;
    }
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_fn.find(key);
    if (it != g_fn.end()) return it->second;  // another thread won; its module stays loaded too
    g_fn[key] = fn;
    return fn;
}

bool rtc_prepare(RtcSpec &sp, const std::vector<Tile> &tiles, const Geom &g) {
    struct Shape {
        int tx, ty, ry;
        hipFunction_t fn = nullptr;
    };
    std::vector<Shape> uniq;
    std::vector<size_t> of;  // per tile, its shape's index
    for (const Tile &t : tiles) {
        const int ry = rtc_rows(sp, t, g).ry;
        size_t i = 0;
        while (i < uniq.size() && (uniq[i].tx != t.tx || uniq[i].ty != t.ty || uniq[i].ry != ry)) ++i;
        if (i == uniq.size()) uniq.push_back(Shape{t.tx, t.ty, ry});
        of.push_back(i);
    }
    int dev = 0;
    (void)hipGetDevice(&dev);
    const std::string &key = spec_key(sp);
    auto at = [&](const Shape &k) { return std::vector<int>{k.tx, k.ty, k.ry, dev, wide_rows(sp, k.ty)}; };
    std::vector<Shape *> todo;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        const SpecEntry &e = g_specs[key];
        for (Shape &k : uniq) {
            auto it = e.fn.find(at(k));
            if (it != e.fn.end()) k.fn = it->second;
            else todo.push_back(&k);
        }
    }
    // compile what is not there yet, concurrently
    auto compile = [&](Shape &k) {
        k.fn = rtc_function(rtc_generic_source(sp, k.tx, k.ty, {k.ty / k.ry, k.ry}), "stencil_generic_gen");
    };
    std::vector<std::thread> th;
    for (size_t i = 1; i < todo.size(); ++i)
        th.emplace_back([&, i] {
            (void)hipSetDevice(dev);
            compile(*todo[i]);
        });
    if (!todo.empty()) compile(*todo[0]);
    for (auto &t : th) t.join();
    bool ok = true;
    std::lock_guard<std::mutex> lk(g_mu);
    for (const Shape &k : uniq) {
        ok &= k.fn != nullptr;
        if (k.fn) g_specs[key].fn[at(k)] = k.fn;
    }
    for (size_t i = 0; i < tiles.size(); ++i) {
        const Shape &k = uniq[of[i]];
        if (k.fn && !sp.kernel(tiles[i])) sp.kernels.push_back({tiles[i], {k.ty / k.ry, k.ry}, k.fn});
    }
    return ok;
}

hipError_t rtc_generic_launch(const RtcSpec &sp, Tile t, const SweepArgs &a, hipStream_t s) {
    const RtcSpec::Kernel *k = sp.kernel(t);
    if (!k) return hipErrorInvalidImage;
    const void *src = a.src;
    void *dst = a.dst;
    Geom g = a.g;
    int zb = t.tz, remap = a.remap;
    double *part = a.part;
    void *args[] = {&src, &dst, &g, &zb, &remap, &part};
    return hipModuleLaunchKernel(k->fn, (unsigned)cdiv(a.g.nx, t.tx), (unsigned)cdiv(a.g.ny, t.ty),
                                 (unsigned)cdiv(a.g.nz, t.tz), t.tx, k->rows.by, 1, 0, s, args, nullptr);
}

}  // namespace stn
