// generic_body.hpp -- the saturated generic stencil's streaming body, shared
// by the table-driven kernel (generic.hip) and the kernels generated for one
// stencil at plan time (rtc.cpp).
//
// A block owns a TX x TY column tile and streams input planes
// zp = bz*zb .. bz*zb + zb - 1 + 2R (padded z).  Each plane is staged once in
// LDS with its R-wide ring (corners when CORNERS) and contributes to the 2R+1
// output planes it touches; their FP64 accumulators wait in a register queue
// (slot s holds output plane m + R - s after input plane m).
// `slots.add<PH>(t, me, live, acc)` adds the plane's taps to the slots whose
// bit is set in `live` (the others hold outputs of the next block in z): slot
// s takes the taps with dz = s - R.  The next plane's loads are issued before this plane's
// arithmetic.  Returns the thread's sum of squared changes.
#pragma once

#include "common.hpp"

namespace stn {

// RY rows per thread: a block of TX x BY threads owns a TX x (BY*RY) tile, and
// a thread's RY outputs of a column share the values it reads from LDS: a box
// of radius R costs (2R+1)(RY+2R)/RY LDS reads per point instead of
// (2R+1)^2, and a coefficient (an SGPR pair written by two scalar moves) is
// used RY times in a row.  The queue moves on either by name (Slots::rotate:
// the plane loop is unrolled over the 2R+1 positions, so a slot never moves
// between registers; moving it makes the compiler hold the queue twice) or by
// 2R*RY register moves per plane, where 2R+1 copies of the plane's arithmetic
// would not stay in the instruction cache.  Loads are
// unconditional: a cell outside the padded array is read at the nearest cell
// of it and used by no output that is stored.  Addresses are a uniform
// pointer per plane plus a byte offset per lane, of type OFF: 32 bits (and
// buffer accesses) where the tile's rows span less than 4 GiB.  The old value of an output is wanted
// for the residual only (the last sweep of a run), and is then read again
// (from L2) instead of waiting in registers.
// Access to a plane: a uniform base and a byte offset per lane.  32-bit
// offsets go through a scalar buffer resource, which leaves no address
// arithmetic to the vector unit.
template <typename T>
__device__ __forceinline__ T plane_ld(const char *base, unsigned off) {
    if constexpr (sizeof(T) == 8) return buf_ld_f64(plane_rsrc(base), off);
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(plane_rsrc(base), off, 0, 0));
}
template <typename T>
__device__ __forceinline__ T plane_ld(const char *base, unsigned long long off) {
    return *(const T *)(base + off);
}
template <typename T>
__device__ __forceinline__ void plane_st(char *base, unsigned off, T v) {
    if constexpr (sizeof(T) == 8) buf_st_f64(plane_rsrc(base), off, v);
    else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), plane_rsrc(base), off, 0, 0);
}
template <typename T>
__device__ __forceinline__ void plane_st(char *base, unsigned long long off, T v) {
    *(T *)(base + off) = v;
}

template <int N>
struct Phase {
    static constexpr int value = N;
};

template <typename T, int R, int TX, int BY, int RY, bool CORNERS, typename OFF, class Slots, typename L>
__device__ __forceinline__ double generic_rows_body(const T *__restrict__ src, T *__restrict__ dst, const Geom &g,
                                                    int zb, int bx, int by, int bz, bool want_res, const Slots &slots,
                                                    L (*tile)[(BY * RY + 2 * R) * (TX + 2 * R)]) {
    constexpr int TY = BY * RY, W = TX + 2 * R, NT = TX * BY, NQ = 2 * R + 1;
    constexpr int BW = CORNERS ? W : TX, X0 = CORNERS ? 0 : R;
    constexpr int NH = 2 * R * BW + 2 * R * TY, HR = (NH + NT - 1) / NT;
    const int tx = threadIdx.x, ty = threadIdx.y, tid = ty * TX + tx;
    const int PX = g.nx + 2 * R, PY = g.ny + 2 * R;
    const int xp0 = bx * TX, yp0 = by * TY;  // padded coordinates of LDS cell (0, 0)
    const int k0 = bz * zb, k1 = min(k0 + zb, g.nz);
    const int me = (ty * RY + R) * W + (tx + R);
    auto at = [&](int lx, int ly) -> OFF {
        const int x = min(xp0 + lx, PX - 1), y = min(yp0 + ly, PY - 1) - yp0;
        return (OFF)(((long long)y * g.py + x) * (long long)sizeof(T));
    };
    OFF co[RY], ho[HR];
    int hl[HR];
#pragma unroll
    for (int m = 0; m < RY; ++m) co[m] = at(tx + R, ty * RY + m + R);
#pragma unroll
    for (int s = 0; s < HR; ++s) {
        int h = tid + s * NT, lx, ly;
        if (h < 2 * R * BW) {
            const int row = h / BW;
            ly = row < R ? row : TY + row;
            lx = h % BW + X0;
        } else {
            h = min(h, NH - 1) - 2 * R * BW;  // lanes past the ring repeat its last cell
            const int c = h % (2 * R);
            ly = R + h / (2 * R);
            lx = c < R ? c : TX + c;
        }
        hl[s] = ly * W + lx;
        ho[s] = at(lx, ly);
    }
    const int rows = min(RY, g.ny - (yp0 + ty * RY));  // rows of this thread inside the grid (may be <= 0)
    const bool inx = xp0 + tx < g.nx;
    const char *pl = (const char *)(src + (long long)k0 * g.pz + (long long)yp0 * g.py);
    char *out = (char *)(dst + (long long)(k0 + R) * g.pz + (long long)yp0 * g.py);
    const long long pzb = g.pz * (long long)sizeof(T);

    T cv[RY], hv[HR];
    auto load = [&]() {
#pragma unroll
        for (int m = 0; m < RY; ++m) cv[m] = plane_ld<T>(pl, co[m]);
#pragma unroll
        for (int s = 0; s < HR; ++s) hv[s] = plane_ld<T>(pl, ho[s]);
    };
    load();
    double acc[NQ][RY];
#pragma unroll
    for (int s = 0; s < NQ; ++s)
#pragma unroll
        for (int m = 0; m < RY; ++m) acc[s][m] = 0.0;
    double sacc = 0.0;
    const int zend = k1 - 1 + 2 * R;
    int zp = k0, b = 0;
    // One input plane.  PH: the planes before it, mod the queue's length when
    // the queue rotates (slot s then sits in acc[(s - PH) mod NQ]).
    auto step = [&](auto phase) -> bool {
        constexpr int PH = decltype(phase)::value, LAST = (2 * R - PH + NQ) % NQ;
        if (zp > zend) return false;
        L *t = tile[b];
#pragma unroll
        for (int m = 0; m < RY; ++m) t[me + m * W] = (L)cv[m];
#pragma unroll
        for (int s = 0; s < HR; ++s) t[hl[s]] = (L)hv[s];
        if (zp < zend) {  // the next plane
            pl += pzb;
            load();
        }
        __syncthreads();
        // slot s adds to output zp - s, if that is one of this block's
        const int lo = max(zp - k1 + 1, 0), hi = min(zp - k0, 2 * R);
        const unsigned live = ((2u << hi) - 1u) & ~((1u << lo) - 1u);
        slots.template add<PH>(t, me, live, acc);
        // the sums end here: moved past the branch below, they would keep every
        // value read from LDS in registers
#pragma unroll
        for (int s = 0; s < NQ; ++s)
#pragma unroll
            for (int m = 0; m < RY; ++m) asm volatile("" : "+v"(acc[s][m]));
        const int kout = zp - 2 * R;  // input plane zp completes output kout (slot 2R)
        if (kout >= k0) {
            T v[RY];
#pragma unroll
            for (int m = 0; m < RY; ++m) {
                v[m] = (T)acc[LAST][m];
                if (inx && m < rows) plane_st<T>(out, co[m], v[m]);
            }
            if (want_res) {
                const char *old = (const char *)src + (out - (char *)dst);
                T ov[RY];
#pragma unroll
                for (int m = 0; m < RY; ++m) ov[m] = plane_ld<T>(old, co[m]);
#pragma unroll
                for (int m = 0; m < RY; ++m)
                    if (inx && m < rows) {
                        const double d = (double)v[m] - (double)ov[m];
                        sacc = fma(d, d, sacc);
                    }
            }
            out += pzb;
        }
        if constexpr (Slots::rotate) {
#pragma unroll
            for (int m = 0; m < RY; ++m) acc[LAST][m] = 0.0;
        } else {
#pragma unroll
            for (int s = NQ - 1; s >= 0; --s)
#pragma unroll
                for (int m = 0; m < RY; ++m) acc[s][m] = s > 0 ? acc[s > 0 ? s - 1 : 0][m] : 0.0;
        }
        ++zp;
        b ^= 1;
        return true;
    };
    if constexpr (!Slots::rotate) {
        while (step(Phase<0>{})) {
        }
    } else if constexpr (R == 1) {
        while (step(Phase<0>{}) && step(Phase<1>{}) && step(Phase<2>{})) {
        }
    } else if constexpr (R == 2) {
        while (step(Phase<0>{}) && step(Phase<1>{}) && step(Phase<2>{}) && step(Phase<3>{}) && step(Phase<4>{})) {
        }
    } else if constexpr (R == 3) {
        while (step(Phase<0>{}) && step(Phase<1>{}) && step(Phase<2>{}) && step(Phase<3>{}) && step(Phase<4>{}) &&
               step(Phase<5>{}) && step(Phase<6>{})) {
        }
    } else {
        while (step(Phase<0>{}) && step(Phase<1>{}) && step(Phase<2>{}) && step(Phase<3>{}) && step(Phase<4>{}) &&
               step(Phase<5>{}) && step(Phase<6>{}) && step(Phase<7>{}) && step(Phase<8>{})) {
        }
    }
    return sacc;
}

}  // namespace stn
