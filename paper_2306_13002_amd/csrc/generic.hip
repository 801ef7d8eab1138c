// generic.hip -- generic 3-D linear stencils (star or box, radius 1..4).
//
//   u'(x) = sum_t coef[cid_t] * u(x + delta_t)
//
// F32 or F64 storage; arithmetic is FP64 in both (operands widened on load,
// the result rounded to the storage type on store).
//
// PLAIN: one thread per point; taps in the caller's order, each operand
// loaded from memory, products rounded and added left to right.  The tap
// table (linear offset, coefficient per tap) is uniform across the launch,
// so it is read through the scalar cache.
//
// SATURATED: the paper's rewrites on the tap sum.  Loads: a block owns a
// column tile and streams input planes; each plane is staged once in LDS (with
// its r-wide ring, corners included where a tap needs them) and contributes
// to the 2r+1 output planes it touches, which wait in a register queue of FP64
// accumulators (plane accumulation), so every input value is read from memory
// once per block.  The next plane's loads are issued before the current
// plane's arithmetic.  The kernels generated for one stencil (rtc.cpp) choose
// between sums shared among the slots, one sum per plane, a tree per coefficient
// and one FMA per tap.  The table-driven kernel here (the fallback, and the allocation-free run) sums the taps that
// share a coefficient id AND a z offset (COMM/ASSOC, ascending address) and
// multiplies once with an FMA (FMA1).
#include "generic_body.hpp"
#include "internal.hpp"
#include "rtc.hpp"

namespace stn {
namespace {

constexpr int kMaxWaves = 16;

template <typename T>
__global__ void generic_plain(const T *__restrict__ src, T *__restrict__ dst, Geom g, GenTab tab,
                             double *__restrict__ part) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const int k = blockIdx.z * blockDim.z + threadIdx.z;
    double d2 = 0.0;
    if (i < g.nx && j < g.ny && k < g.nz) {
        const long long q = (long long)(k + g.r) * g.pz + (long long)(j + g.r) * g.py + (i + g.r);
        double v = tab.c[0] * (double)src[q + tab.off[0]];
        for (int t = 1; t < tab.n; ++t) v = v + tab.c[t] * (double)src[q + tab.off[t]];
        const T out = (T)v;
        dst[q] = out;
        const double d = (double)out - (double)src[q];
        d2 = d * d;
    }
    if (part) {
        __shared__ double lds[kMaxWaves];
        const double s = block_sum_f64(d2, lds);
        if (threadIdx.x == 0 && threadIdx.y == 0 && threadIdx.z == 0) part[block_linear_id()] = s;
    }
}

// Table-driven tap sums: slot s's groups are read from the plan's tables.
template <int R, int W, int RY>
struct TableSlots {
    static constexpr bool rotate = false;
    GenTab tab;
    template <int>
    __device__ __forceinline__ void add(const double *__restrict__ t, int me, unsigned live, double (*acc)[RY]) const {
#pragma unroll
        for (int s = 0; s < 2 * R + 1; ++s) {
            if (!(live >> s & 1)) continue;
            const int g0 = tab.slot_g[s], g1 = tab.slot_g[s + 1];
            double a[RY];
#pragma unroll
            for (int m = 0; m < RY; ++m) a[m] = acc[s][m];
            for (int gi = g0; gi < g1; ++gi) {
                const int t0 = tab.g_t[gi], t1 = tab.g_t[gi + 1];
                // the group's taps (ascending address), eight at a time, into
                // four partial sums per row, then one FMA
                double p[4][RY];
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int m = 0; m < RY; ++m) p[q][m] = 0.0;
                auto at = [&](int ti) {
                    const int xy = tab.t_xy[ti];
                    return t + me + (xy >> 16) * W + (short)(xy & 0xFFFF);
                };
                int ti = t0;
                for (; ti + 8 <= t1; ti += 8) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const double *pa = at(ti + q), *pb = at(ti + q + 4);
#pragma unroll
                        for (int m = 0; m < RY; ++m) p[q][m] += pa[m * W] + pb[m * W];
                    }
                }
                for (; ti < t1; ++ti) {
                    const double *pa = at(ti);
#pragma unroll
                    for (int m = 0; m < RY; ++m) p[0][m] += pa[m * W];
                }
#pragma unroll
                for (int m = 0; m < RY; ++m)
                    a[m] = fma(tab.g_c[gi], (p[0][m] + p[1][m]) + (p[2][m] + p[3][m]), a[m]);
            }
#pragma unroll
            for (int m = 0; m < RY; ++m) acc[s][m] = a[m];
        }
    }
};

template <typename T, int R, int TX, int BY, int RY, bool CORNERS>
__global__ __launch_bounds__(TX *BY) void generic_sat(const T *__restrict__ src, T *__restrict__ dst, Geom g,
                                                      GenTab tab, int zb, int remap, double *__restrict__ part) {
    constexpr int W = TX + 2 * R;
    __shared__ double tile[2][(BY * RY + 2 * R) * W];
    __shared__ double red[kMaxWaves];
    int bx, by, bz;
    tile_coords(remap, bx, by, bz);
    const double sacc = generic_rows_body<T, R, TX, BY, RY, CORNERS, unsigned long long>(
        src, dst, g, zb, bx, by, bz, part != nullptr, TableSlots<R, W, RY>{tab}, tile);
    if (part) {
        const double s = block_sum_f64(sacc, red);
        if (threadIdx.x == 0 && threadIdx.y == 0) part[block_linear_id()] = s;
    }
}

bool plain_tile_ok(Tile t) {
    const long long n = (long long)t.tx * t.ty * t.tz;
    return t.tx >= 1 && t.ty >= 1 && t.tz >= 1 && n % 64 == 0 && n <= 1024;
}

// Saturated tiles: (TX, tile rows) -> thread rows BY, rows per thread RY
#define GEN_SAT_TILES(X) X(32, 4, 2, 2) X(32, 8, 2, 4) X(64, 2, 1, 2) X(64, 4, 2, 2) X(128, 2, 1, 2) X(32, 16, 4, 4) \
    X(32, 32, 8, 4) X(64, 16, 4, 4)

bool gen_tile_ok(int v, Tile t) {
    if (v == V_PLAIN) return plain_tile_ok(t);
    if (t.tz < 1) return false;
#define X(a, b, by, ry) if (t.tx == a && t.ty == b) return true;
    GEN_SAT_TILES(X)
#undef X
    return false;
}

int gen_sat_tiles(Tile *out, int max) {
    int n = 0;
#define X(a, b, by, ry) if (n < max) out[n++] = Tile{a, b, 0};
    GEN_SAT_TILES(X)
#undef X
    return n;
}

}  // namespace

GenRows gen_rows(int tx, int ty) {
#define X(a, b, by, ry) if (tx == a && ty == b) return {by, ry};
    GEN_SAT_TILES(X)
#undef X
    return {0, 0};
}

namespace {

long long gen_nblocks(int, Tile t, const Geom &g) { return cdiv(g.nx, t.tx) * cdiv(g.ny, t.ty) * cdiv(g.nz, t.tz); }

template <typename T>
hipError_t gen_launch_t(int v, Tile t, const SweepArgs &a, hipStream_t s) {
    const T *src = (const T *)a.src;
    T *dst = (T *)a.dst;
    dim3 grid(cdiv(a.g.nx, t.tx), cdiv(a.g.ny, t.ty), cdiv(a.g.nz, t.tz));
    if (v == V_PLAIN) {
        hipLaunchKernelGGL(generic_plain<T>, grid, dim3(t.tx, t.ty, t.tz), 0, s, src, dst, a.g, a.gen, a.part);
        return hipGetLastError();
    }
#define GEN_LAUNCH(A_, B_, R_, C_)                                                                          \
    hipLaunchKernelGGL((generic_sat<T, R_, A_, BY_, RY_, C_>), grid, dim3(A_, BY_, 1), 0, s, src, dst, a.g, a.gen, \
                       t.tz, a.remap, a.part)
#define X(A, B, BY, RY)                                                                                          \
    if (t.tx == A && t.ty == B) {                                                                           \
        constexpr int BY_ = BY, RY_ = RY;                                                                   \
        const bool c = a.gen.corners;                                                                       \
        switch (a.g.r) {                                                                                    \
        case 1: if (c) GEN_LAUNCH(A, B, 1, true); else GEN_LAUNCH(A, B, 1, false); break;                               \
        case 2: if (c) GEN_LAUNCH(A, B, 2, true); else GEN_LAUNCH(A, B, 2, false); break;                               \
        case 3: if (c) GEN_LAUNCH(A, B, 3, true); else GEN_LAUNCH(A, B, 3, false); break;                               \
        case 4: if (c) GEN_LAUNCH(A, B, 4, true); else GEN_LAUNCH(A, B, 4, false); break;                               \
        default: return hipErrorInvalidValue;                                                               \
        }                                                                                                   \
        return hipGetLastError();                                                                           \
    }
    GEN_SAT_TILES(X)
#undef X
#undef GEN_LAUNCH
    return hipErrorInvalidValue;
}

hipError_t gen_launch(int v, Tile t, const SweepArgs &a, hipStream_t s) {
    if (v == V_SATURATED && a.rtc) return rtc_generic_launch(*a.rtc, t, a, s);
    return a.elem_bytes == 4 ? gen_launch_t<float>(v, t, a, s) : gen_launch_t<double>(v, t, a, s);
}

}  // namespace

KindOps generic_ops = {gen_tile_ok, gen_sat_tiles, nullptr, gen_nblocks, gen_launch, nullptr};

}  // namespace stn
