// support.hip -- halo copy, periodic halo fill, the residual's final pass and
// the device scratch of the allocation-free run.
#include <algorithm>
#include <mutex>

#include "internal.hpp"

namespace stn {
namespace {

// Enumerate the halo cells of a padded grid (x/y halo width r, z halo width
// rz; rz = 0 and nz = 1 for 2-D grids) as three segments: the z-halo planes,
// then the y-halo rows of interior planes, then the x-halo cells of interior
// rows.  Writes the padded (x, y, z) of halo cell t.
__device__ __forceinline__ void halo_cell(long long t, const Geom &g, int rz, long long &x, long long &y,
                                          long long &z) {
    const long long PX = g.nx + 2 * g.r, PY = g.ny + 2 * g.r;
    const long long cA = 2LL * rz * PY * PX, cB = (long long)g.nz * 2 * g.r * PX;
    if (t < cA) {
        const long long zz = t / (PY * PX), rem = t % (PY * PX);
        z = zz < rz ? zz : g.nz + zz;
        y = rem / PX;
        x = rem % PX;
    } else if (t < cA + cB) {
        t -= cA;
        const long long per = 2LL * g.r * PX;
        z = rz + t / per;
        const long long rem = t % per, yy = rem / PX;
        y = yy < g.r ? yy : g.ny + yy;
        x = rem % PX;
    } else {
        t -= cA + cB;
        const long long zy = t / (2 * g.r), xx = t % (2 * g.r);
        z = rz + zy / g.ny;
        y = g.r + zy % g.ny;
        x = xx < g.r ? xx : g.nx + xx;
    }
}

__host__ __device__ inline long long halo_count(const Geom &g, int rz) {
    const long long PX = g.nx + 2 * g.r, PY = g.ny + 2 * g.r;
    return 2LL * rz * PY * PX + (long long)g.nz * 2 * g.r * PX + (long long)g.nz * g.ny * 2 * g.r;
}

// The halo as rows: whole rows of the padded grid (the z-halo planes, then the
// y-halo rows of interior planes), one wave per row of up to 1024 cells or per
// 256 cells of a longer one, then the two x-halo pieces of every interior row,
// one thread per cell.  (A 2-D grid has two such rows, however long: one wave
// each took 10 us longer at 4000 x 4000.)  One division per row or thread, of
// type I (32 bits unless the grid has more rows), instead of four 64-bit ones
// per cell (400^3: 22 -> 18 us; the two part-written lines of every row are
// what is left).
constexpr int kRowWhole = 1024, kRowPiece = 256;
__host__ __device__ inline int row_pieces(const Geom &g) {
    const int PX = g.nx + 2 * g.r;
    return PX <= kRowWhole ? 1 : (PX + kRowPiece - 1) / kRowPiece;
}

template <typename T, typename I>
__device__ __forceinline__ void halo_rows(const T *__restrict__ src, T *__restrict__ dst, const Geom &g, int rz,
                                          I full_rows, I wave, I waves) {
    const int PX = g.nx + 2 * g.r, PY = g.ny + 2 * g.r, pieces = row_pieces(g);
    const I top = (I)2 * rz * PY;
    for (I item = wave; item < full_rows * pieces; item += waves) {
        const I t = pieces == 1 ? item : item / pieces;
        const int x1 = (int)(item - t * pieces) * kRowPiece, x2 = pieces == 1 ? PX : min(PX, x1 + kRowPiece);
        const I per = t < top ? (I)PY : (I)2 * g.r, u = t < top ? t : t - top;
        const I zz = u / per;
        const int yy = (int)(u - zz * per);
        const long long z = t >= top ? (long long)zz + rz : zz < (I)rz ? (long long)zz : (long long)g.nz + (long long)zz;
        const int y = t < top || yy < g.r ? yy : g.ny + yy;
        const long long q = z * g.pz + y * g.py;
        for (int x0 = x1 + (threadIdx.x & 63); x0 < x2; x0 += 256) {  // four loads in flight
            T v[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = src[q + min(x0 + 64 * c, PX - 1)];
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (x0 + 64 * c < PX) dst[q + x0 + 64 * c] = v[c];
        }
    }
}

// a row's 2r side cells: threads per row, as a power of two
__host__ __device__ inline int side_shift(int r) { return r == 1 ? 1 : r == 2 ? 2 : 3; }

template <typename T, typename I>
__device__ __forceinline__ void halo_sides(const T *__restrict__ src, T *__restrict__ dst, const Geom &g, int rz,
                                           I side_threads, I thread, I threads) {
    const int sh = side_shift(g.r), c = (int)(thread & ((1 << sh) - 1));  // threads: a multiple of 8
    if (c >= 2 * g.r) return;
    const int x = c < g.r ? c : g.nx + c;
    for (I t = thread; t < side_threads; t += threads) {
        const I row = t >> sh, k = row / (I)g.ny;
        const long long q = ((long long)k + rz) * g.pz + ((long long)(row - k * g.ny) + g.r) * g.py + x;
        dst[q] = src[q];
    }
}

template <typename T, typename I>
__global__ __launch_bounds__(256) void halo_copy_kernel(const T *__restrict__ src, T *__restrict__ dst, Geom g, int rz,
                                                        I full_rows, I side_threads, unsigned full_blocks) {
    if (blockIdx.x < full_blocks)
        halo_rows<T, I>(src, dst, g, rz, full_rows, (I)blockIdx.x * 4 + (threadIdx.x >> 6), (I)full_blocks * 4);
    else
        halo_sides<T, I>(src, dst, g, rz, side_threads, (I)(blockIdx.x - full_blocks) * 256 + threadIdx.x,
                         (I)(gridDim.x - full_blocks) * 256);
}

// The halo copies and the interior copies (scratch grid back to state) of the
// grids of a batch class in one launch each; gridDim.x = grids * chunks.  One
// launch per grid, one after the other, took 0.5 of 5.75 ms for 64 grids and
// 50 sweeps.
template <typename I>
__global__ __launch_bounds__(256) void batch_halo_kernel(const BatchProb *__restrict__ probs,
                                                         const int *__restrict__ members, int chunks) {
    const BatchProb &P = probs[members[blockIdx.x / chunks]];
    const int c = blockIdx.x % chunks;
    const Geom g = P.g;
    const I full = (I)2 * (g.ny + 2) + (I)g.nz * 2, side = ((I)g.nz * g.ny) << side_shift(1);
    halo_rows<double, I>(P.f[0], P.f[1], g, 1, full, (I)c * 4 + (threadIdx.x >> 6), (I)chunks * 4);
    halo_sides<double, I>(P.f[0], P.f[1], g, 1, side, (I)c * 256 + threadIdx.x, (I)chunks * 256);
}

__device__ __forceinline__ long long wrap_into(long long c, int r, int n) {
    // padded coordinate -> padded coordinate of the interior cell it images
    long long i = (c - r) % n;
    if (i < 0) i += n;
    return i + r;
}

template <typename T>
__global__ void periodic_fill_kernel(T *__restrict__ buf, Geom g, int rz, long long n) {
    for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < n;
         t += (long long)gridDim.x * blockDim.x) {
        long long x, y, z;
        halo_cell(t, g, rz, x, y, z);
        const long long sx = wrap_into(x, g.r, g.nx), sy = wrap_into(y, g.r, g.ny);
        const long long sz = rz ? wrap_into(z, rz, g.nz) : z;
        buf[z * g.pz + y * g.py + x] = buf[sz * g.pz + sy * g.py + sx];
    }
}

// I: the index type (32 bits unless the grid has more cells)
template <typename T, typename I>
__device__ __forceinline__ void interior_cells(const T *__restrict__ src, T *__restrict__ dst, const Geom &g, I n,
                                               I thread, I threads) {
    for (I t = thread; t < n; t += threads) {
        const I jk = t / (I)g.nx, i = t - jk * g.nx, k = jk / (I)g.ny, j = jk - k * g.ny;
        const long long q = ((long long)k + g.r) * g.pz + ((long long)j + g.r) * g.py + ((long long)i + g.r);  // 2-D: pz = 0
        dst[q] = src[q];
    }
}

template <typename T, typename I>
__global__ __launch_bounds__(256) void interior_copy_kernel(const T *__restrict__ src, T *__restrict__ dst, Geom g, I n) {
    interior_cells<T, I>(src, dst, g, n, (I)blockIdx.x * 256 + threadIdx.x, (I)gridDim.x * 256);
}

template <typename I>
__global__ __launch_bounds__(256) void batch_tail_kernel(const BatchProb *__restrict__ probs,
                                                         const int *__restrict__ members, int chunks) {
    const BatchProb &P = probs[members[blockIdx.x / chunks]];
    const Geom g = P.g;
    interior_cells<double, I>(P.f[1], P.f[0], g, (I)g.nx * g.ny * g.nz, (I)(blockIdx.x % chunks) * 256 + threadIdx.x,
                              (I)chunks * 256);
}

// Pass 1: block b sums the contiguous chunk [b*chunk, min((b+1)*chunk, n))
// (thread-strided, then the block sum); pass 2 (one block) sums the pass-1
// results.  The split depends only on n, so the total is reproducible.
__global__ void reduce_pass1_kernel(const double *__restrict__ part, long long n, long long chunk,
                                    double *__restrict__ out) {
    __shared__ double lds[4];
    const long long b0 = blockIdx.x * chunk, b1 = min(b0 + chunk, n);
    double s = 0.0;
    for (long long i = b0 + threadIdx.x; i < b1; i += 256) s += part[i];
    s = block_sum_f64(s, lds);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

template <typename T>
__global__ void fill_kernel(T *__restrict__ buf, long long n, T v) {
    for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < n; t += (long long)gridDim.x * blockDim.x)
        buf[t] = v;
}

// seg holds count begins, then count ends.
__global__ void segment_sums_kernel(const double *__restrict__ part, const int *__restrict__ seg, int count,
                                    double *__restrict__ out) {
    __shared__ double lds[4];
    const int b0 = seg[blockIdx.x], b1 = seg[count + blockIdx.x];
    double s = 0.0;
    for (int i = b0 + threadIdx.x; i < b1; i += 256) s += part[i];
    s = block_sum_f64(s, lds);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

dim3 grid_for(long long n) {
    long long b = cdiv(n, 256);
    if (b > 65536) b = 65536;
    if (b < 1) b = 1;
    return dim3((unsigned)b);
}

}  // namespace

namespace {
template <typename T, typename I>
hipError_t halo_copy(const T *src, T *dst, const Geom &g, int rz, long long full, long long side, hipStream_t s) {
    const unsigned fb = (unsigned)std::min(cdiv(full * row_pieces(g), 4), 32768LL);
    const unsigned sb = (unsigned)std::min(cdiv(side, 256), 32768LL);
    hipLaunchKernelGGL((halo_copy_kernel<T, I>), dim3(fb + sb), dim3(256), 0, s, src, dst, g, rz, (I)full, (I)side, fb);
    return hipGetLastError();
}
constexpr long long kIndex32 = 0x7F000000LL;  // counts below this, plus a grid's stride, stay below 2^32
}  // namespace

hipError_t launch_halo_copy(const void *src, void *dst, int eb, const Geom &g, int rz, hipStream_t s) {
    const long long PY = g.ny + 2 * g.r;
    const long long full = 2LL * rz * PY + (long long)g.nz * 2 * g.r,
                    side = ((long long)g.nz * g.ny) << side_shift(g.r);
    const bool w = full * row_pieces(g) + side < kIndex32;
    if (eb == 8)
        return w ? halo_copy<double, unsigned>((const double *)src, (double *)dst, g, rz, full, side, s)
                 : halo_copy<double, unsigned long long>((const double *)src, (double *)dst, g, rz, full, side, s);
    return w ? halo_copy<float, unsigned>((const float *)src, (float *)dst, g, rz, full, side, s)
             : halo_copy<float, unsigned long long>((const float *)src, (float *)dst, g, rz, full, side, s);
}

hipError_t launch_periodic_fill(void *buf, int eb, const Geom &g, int rz, hipStream_t s) {
    const long long n = halo_count(g, rz);
    if (n == 0) return hipSuccess;
    if (eb == 8)
        hipLaunchKernelGGL(periodic_fill_kernel<double>, grid_for(n), dim3(256), 0, s, (double *)buf, g, rz, n);
    else
        hipLaunchKernelGGL(periodic_fill_kernel<float>, grid_for(n), dim3(256), 0, s, (float *)buf, g, rz, n);
    return hipGetLastError();
}

hipError_t launch_fill(void *buf, long long n, int eb, double v, hipStream_t s) {
    if (eb == 8)
        hipLaunchKernelGGL(fill_kernel<double>, grid_for(n), dim3(256), 0, s, (double *)buf, n, v);
    else
        hipLaunchKernelGGL(fill_kernel<float>, grid_for(n), dim3(256), 0, s, (float *)buf, n, (float)v);
    return hipGetLastError();
}

hipError_t launch_interior_copy(const void *src, void *dst, int eb, const Geom &g, int rz, hipStream_t s) {
    const long long n = (long long)g.nx * g.ny * g.nz;
    Geom h = g;
    if (rz == 0) h.pz = 0;  // 2-D: a single plane
    const bool w = n < kIndex32;
#define GO(T, I) \
    hipLaunchKernelGGL((interior_copy_kernel<T, I>), grid_for(n), dim3(256), 0, s, (const T *)src, (T *)dst, h, (I)n)
    if (eb == 8) {
        if (w) GO(double, unsigned);
        else GO(double, unsigned long long);
    } else {
        if (w) GO(float, unsigned);
        else GO(float, unsigned long long);
    }
#undef GO
    return hipGetLastError();
}

// Threads of a batch problem's copy at one piece each: the tail's cells; the
// halo's rows, a wave each, or its side cells, which the same threads copy.
long long batch_copy_work(bool tail, const Geom &g) {
    if (tail) return (long long)g.nx * g.ny * g.nz;
    const long long rows = 2LL * (g.ny + 2) + 2LL * g.nz, side = ((long long)g.nz * g.ny) << side_shift(1);
    return std::max(rows * row_pieces(g) * 64, side);
}

hipError_t launch_batch_copy(bool tail, const BatchProb *probs, const int *members, int n, long long work,
                             hipStream_t s) {
    const int chunks = batch_copy_chunks(n, work);
    const dim3 grid((unsigned)n * (unsigned)chunks);
    const bool w = work < kIndex32;
    if (tail) {
        if (w) hipLaunchKernelGGL(batch_tail_kernel<unsigned>, grid, dim3(256), 0, s, probs, members, chunks);
        else hipLaunchKernelGGL(batch_tail_kernel<unsigned long long>, grid, dim3(256), 0, s, probs, members, chunks);
    } else {
        if (w) hipLaunchKernelGGL(batch_halo_kernel<unsigned>, grid, dim3(256), 0, s, probs, members, chunks);
        else hipLaunchKernelGGL(batch_halo_kernel<unsigned long long>, grid, dim3(256), 0, s, probs, members, chunks);
    }
    return hipGetLastError();
}

hipError_t launch_segment_sums(const double *part, const int *seg, int count, double *out, hipStream_t s) {
    hipLaunchKernelGGL(segment_sums_kernel, dim3(count), dim3(256), 0, s, part, seg, count, out);
    return hipGetLastError();
}

hipError_t launch_reduce_partials(const double *part, long long n, double *scratch, double *out, hipStream_t s) {
    long long chunk = cdiv(n, kReduceBlocks);
    if (chunk < 1024) chunk = 1024;
    const long long nb = cdiv(n, chunk);
    if (nb == 1) {
        // One chunk: a second pass would add zeros to this sum and return it
        // unchanged (residuals are sums of squares, never -0), so the single
        // block writes the total itself and one launch is saved.
        hipLaunchKernelGGL(reduce_pass1_kernel, dim3(1), dim3(256), 0, s, part, n, chunk, out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(reduce_pass1_kernel, dim3((unsigned)nb), dim3(256), 0, s, part, n, chunk, scratch);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_pass1_kernel, dim3(1), dim3(256), 0, s, (const double *)scratch, nb, nb, out);
    return hipGetLastError();
}

// Scratch of the allocation-free run: kNoallocPartials per-block residual
// partials, then kReduceBlocks first-pass sums of their reduction.  One copy
// per GPU, resident until the process ends.  In host code the array's name
// is not a device address: only the address hipGetSymbolAddress returns for
// the current device is passed to kernels.
static __device__ __align__(256) double scratch[kNoallocPartials + kReduceBlocks];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t noalloc_scratch(double **out) {
    *out = nullptr;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        double *ptr = nullptr;
        if ((e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch))) != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace stn
