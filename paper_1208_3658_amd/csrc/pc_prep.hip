// pc_prep.hip -- per-launch preparation kernels: spatial ordering of the
// catalogues, tile bounding spheres, and exact whole-tile-pair binning.
//
// Counts do not depend on the order of a catalogue, so each index range a job
// uses is copied in a spatial order (counting sort on a cube-face Hilbert key
// of the unit vector; the order inside a key bucket is arbitrary).  Consecutive
// tiles of 256 points are then compact, each gets a bounding sphere (centre,
// radius), and a tile pair whose squared-chord interval lies inside one bin
// is binned as a whole without visiting its pairs (the paper, Sec. 2.2: time
// is saved by not computing separations outside the binned range).
#include <algorithm>
#include <cstring>

#include "pc_internal.hpp"
#include "pc_math.h"

namespace pc {

#if PC_R == 4
// ------------------- tile-independent part (compiled once, 256-point build)


// Every step runs once over all sources and views of a launch (a block finds
// its own by a search over the first blocks): a batch of many small catalogues
// is then bound by its points and not by its launches.  For 64 mocks of 10,000
// to 80,000 points and 300,000 randoms the time outside the counting kernel
// is 2.5 ms, against 4.4 ms with each view's eight launches of its own.

// The last of n descriptors whose first block is at or before b.
template <typename D>
__device__ __forceinline__ int find_block(const D *d, int n, int64_t b) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (d[mid].blk0 <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// ---------------------------------------------------------- ordering keys
// Cube-face Hilbert key: the face of the cube the unit vector points through
// (axis and sign of its largest component), then the 2-D Hilbert index of the
// two other components divided by the largest one, in a square grid laid over
// the part of the face that the catalogue occupies.  Points close on the
// sphere get close keys, without the long jumps of a Morton order.  The grid
// follows the catalogue's extent because most catalogues are patches: a grid
// over whole faces, sized by the number of points, left 10,000 points on 10 x
// 10 degrees in a handful of cells, in no order inside them.  With the grid on
// the extent the counting step takes 503 us there against 634, 23.4 ms against
// 28.3 for the 64 mocks on 50 x 50 degrees, and the 1M workload's kernel (100 x
// 100 degrees, well ordered before) 42.7 ms against 45.2.

struct FacePoint {
    uint32_t face;
    float u, w;  // in [-1, 1]
};

__device__ __forceinline__ FacePoint face_point(double x, double y, double z) {
    const double ax = fabs(x), ay = fabs(y), az = fabs(z);
    uint32_t face;
    double major, u, w;
    if (ax >= ay && ax >= az) { face = 0; major = x; u = y; w = z; }
    else if (ay >= az) { face = 2; major = y; u = x; w = z; }
    else { face = 4; major = z; u = x; w = y; }
    if (major < 0.0) face += 1;
    const double inv = 1.0 / fmax(fabs(major), 1e-300);
    return {face, static_cast<float>(u * inv), static_cast<float>(w * inv)};
}

// Order-preserving code of a float, above 0 for every value, and its inverse.
__device__ __forceinline__ uint32_t ordered_bits(float f) {
    const uint32_t b = __float_as_uint(f);
    return (b >> 31) ? ~b : b | 0x80000000u;
}
__device__ __forceinline__ float from_ordered_bits(uint32_t o) {
    return __uint_as_float((o >> 31) ? o & 0x7FFFFFFFu : ~o);
}

// The wave's maximum in its last lane (0 below every value).
__device__ __forceinline__ uint32_t wave_max_last(uint32_t x) {
#define PC_DPP_MAX(ctrl, rows) \
    x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), ctrl, rows, 0xF, false)))
    PC_DPP_MAX(0x111, 0xF);  // row_shr 1, 2, 4, 8
    PC_DPP_MAX(0x112, 0xF);
    PC_DPP_MAX(0x114, 0xF);
    PC_DPP_MAX(0x118, 0xF);
    PC_DPP_MAX(0x142, 0xA);  // row_bcast 15, 31
    PC_DPP_MAX(0x143, 0xC);
#undef PC_DPP_MAX
    return x;
}

// -------------------------------------------------------------- conversion

// Points per thread: several where there are points enough to fill the device,
// so that a workgroup's extent goes out once for all of them.
constexpr int kConvPer = 4;
__host__ __device__ inline int convert_per(int64_t n) { return n >= 65536 ? kConvPer : 1; }

// RA/Dec (degrees, binary64) -> unit vectors, binary64 (x, y, z, 0), and the
// source's extent: per face the largest ordered_bits of u, -u, w and -w over its
// points (0: no point).  Invalid inputs (non-finite, |Dec| > 90) set *err and
// produce the vector of (0, 0).
// The extent's maxima are taken in registers over a wave, in LDS over the
// workgroup, and go out with an atomic only where they exceed what is there.
// (With every wave looking at the extent in memory 1M points took 73 us, now
// 27; without the extent 17.)
__global__ void __launch_bounds__(256) k_convert(const SrcDesc *__restrict__ srcs, int n_srcs) {
#pragma clang fp contract(off)
    __shared__ uint32_t most[kExtWords];
    const int tid = static_cast<int>(threadIdx.x);
    if (tid < kExtWords) most[tid] = 0u;
    __syncthreads();
    const SrcDesc s = srcs[find_block(srcs, n_srcs, blockIdx.x)];
    const int per = convert_per(s.n);
    const int64_t i0 = (static_cast<int64_t>(blockIdx.x) - s.blk0) * (256 * per) + tid;
    FacePoint p[kConvPer];
    uint32_t faces = 0u;  // of the thread's points
#pragma unroll
    for (int q = 0; q < kConvPer; ++q) {
        const int64_t i = i0 + q * 256;
        p[q] = {6u, 0.0f, 0.0f};
        if (q >= per || i >= s.n) continue;
        double r = s.ra[i], d = s.dec[i];
        const bool ok = isfinite(r) && isfinite(d) && d >= -90.0 && d <= 90.0;
        if (!ok) {
            atomicOr(s.err, 1);
            r = 0.0;
            d = 0.0;
        }
        double sa, ca, sd, cd;
        sincosd(r, &sa, &ca);
        sincosd(d, &sd, &cd);
        const double x = cd * ca;
        const double y = cd * sa;
        const double z = sd;
        s.a64[i] = make_double4(x, y, z, 0.0);
        p[q] = face_point(x, y, z);
        faces |= 1u << p[q].face;
    }
    for (uint32_t f = 0; f < 6u; ++f) {
        if (__ballot((faces >> f) & 1u) == 0) continue;
        uint32_t v[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int q = 0; q < kConvPer; ++q) {
            const bool mine = p[q].face == f;
            v[0] = max(v[0], mine ? ordered_bits(p[q].u) : 0u);
            v[1] = max(v[1], mine ? ordered_bits(-p[q].u) : 0u);
            v[2] = max(v[2], mine ? ordered_bits(p[q].w) : 0u);
            v[3] = max(v[3], mine ? ordered_bits(-p[q].w) : 0u);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = wave_max_last(v[k]);
            if ((tid & (kWave - 1)) == kWave - 1) atomicMax(most + 4 * f + k, v[k]);
        }
    }
    __syncthreads();
    if (tid < kExtWords && most[tid] > *static_cast<volatile uint32_t *>(s.ext + tid)) atomicMax(s.ext + tid, most[tid]);
}

// ------------------------------------------------------------------- keys

// The key grid of a view: per face 4^bits cells over the extent, the first
// key of the face.  The cell size is chosen for about two points per cell and
// the faces' grids are coarsened together while they have more cells than the
// view has counters.
struct KeyFrame {
    float lo_u[6], lo_w[6], scale[6];
    uint32_t bits[6], base[6];
};

__device__ void key_frame(const uint32_t *ext, int64_t n, uint32_t budget, KeyFrame &k) {
    float eu[6], ew[6];
    float area = 0.0f;
    for (int f = 0; f < 6; ++f) {
        const uint32_t a = ext[4 * f], b = ext[4 * f + 1], c = ext[4 * f + 2], d = ext[4 * f + 3];
        k.lo_u[f] = a ? -from_ordered_bits(b) : 0.0f;
        k.lo_w[f] = a ? -from_ordered_bits(d) : 0.0f;
        eu[f] = a ? fmaxf(from_ordered_bits(a) - k.lo_u[f], 1e-12f) : 0.0f;
        ew[f] = a ? fmaxf(from_ordered_bits(c) - k.lo_w[f], 1e-12f) : 0.0f;
        area += eu[f] * ew[f];
    }
    const float s = sqrtf(fmaxf(area, 1e-30f) * 2.0f / static_cast<float>(n));
    int32_t bits[6];
    for (int f = 0; f < 6; ++f) {
        const float e = fmaxf(eu[f], ew[f]);
        bits[f] = e > 0.0f ? max(0, min(14, static_cast<int32_t>(ceilf(log2f(fmaxf(e / s, 1.0f)))))) : 0;
    }
    for (;;) {
        uint64_t cells = 0;
        int32_t most = 0;
        for (int f = 0; f < 6; ++f) {
            cells += uint64_t(1) << (2 * bits[f]);
            most = max(most, bits[f]);
        }
        if (cells <= budget || most == 0) break;
        for (int f = 0; f < 6; ++f) bits[f] = max(0, bits[f] - 1);
    }
    uint32_t base = 0;
    for (int f = 0; f < 6; ++f) {
        k.bits[f] = static_cast<uint32_t>(bits[f]);
        k.base[f] = base;
        base += 1u << (2 * bits[f]);
        k.scale[f] = static_cast<float>(1u << bits[f]) / fmaxf(fmaxf(eu[f], ew[f]), 1e-12f);
    }
}

__device__ __forceinline__ uint32_t hilbert2d(uint32_t bits, uint32_t x, uint32_t y) {
    const uint32_t n = 1u << bits;
    uint32_t d = 0;
    for (uint32_t s = n >> 1; s > 0; s >>= 1) {
        const uint32_t rx = (x & s) ? 1u : 0u;
        const uint32_t ry = (y & s) ? 1u : 0u;
        d += s * s * ((3u * rx) ^ ry);
        if (ry == 0u) {
            if (rx == 1u) {
                x = n - 1u - x;
                y = n - 1u - y;
            }
            const uint32_t t = x;
            x = y;
            y = t;
        }
    }
    return d;
}

constexpr int kKeysPer = 4;  // points per thread: the key grid is worked out once per block

__global__ void __launch_bounds__(256) k_keys(const ViewDesc *__restrict__ views, int n_views) {
    __shared__ KeyFrame fr;
    const ViewDesc v = views[find_block(views, n_views, blockIdx.x)];
    if (threadIdx.x == 0) key_frame(v.ext, v.n, v.buckets, fr);
    __syncthreads();
    const int64_t i0 = (static_cast<int64_t>(blockIdx.x) - v.blk0) * (256 * kKeysPer) + threadIdx.x;
#pragma unroll
    for (int q = 0; q < kKeysPer; ++q) {
        const int64_t i = i0 + q * 256;
        if (i >= v.n) return;
        const double4 a = v.src[i];
        const FacePoint p = face_point(a.x, a.y, a.z);
        const uint32_t bits = fr.bits[p.face], m = (1u << bits) - 1u;
        const float x = fmaxf((p.u - fr.lo_u[p.face]) * fr.scale[p.face], 0.0f);
        const float y = fmaxf((p.w - fr.lo_w[p.face]) * fr.scale[p.face], 0.0f);
        const uint32_t k = fr.base[p.face] + hilbert2d(bits, min(static_cast<uint32_t>(x), m), min(static_cast<uint32_t>(y), m));
        v.keys[i] = k;
        if (v.slots) v.slots[i] = atomicAdd(v.hist + k, 1u);
        else atomicAdd(v.hist + k, 1u);
    }
}

// ------------------------------------------------------------------ scan
// Exclusive prefix sum of m uint32 counters: per-block scans of kScanChunk
// values with block totals, then a scan of the totals by one workgroup (up to
// eight million counters in one step).  The blocks' offsets are added where
// the counters are used, or by a third pass (launch_exclusive_scan).

constexpr int kScanBlock = 256;
constexpr int kScanPer = 8;
constexpr int kScanChunk = kScanBlock * kScanPer;
constexpr int kSumsBlock = 1024;
constexpr int kSumsPer = 4;

// exclusive scan of one value per thread; sh: a word per wave
template <int THREADS>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *sh, uint32_t *total) {
    const int lane = static_cast<int>(threadIdx.x) & (kWave - 1), wave = static_cast<int>(threadIdx.x) / kWave;
    uint32_t s = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t x = __shfl_up(s, o, kWave);
        if (lane >= o) s += x;
    }
    if (lane == kWave - 1) sh[wave] = s;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < THREADS / kWave; ++w) {
        const uint32_t x = sh[w];
        before += w < wave ? x : 0u;
        all += x;
    }
    __syncthreads();
    *total = all;
    return before + s - v;
}

__global__ void __launch_bounds__(kScanBlock) k_scan_local(uint32_t *__restrict__ a, int64_t m,
                                                           uint32_t *__restrict__ block_sums) {
    __shared__ uint32_t sh[kScanBlock / kWave];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanChunk + threadIdx.x * kScanPer;
    uint32_t v[kScanPer];
    uint32_t s = 0;
    const bool whole = base + kScanPer <= m;
    if (whole) {
#pragma unroll
        for (int k = 0; k < kScanPer; k += 4) {
            const uint4 q = *reinterpret_cast<const uint4 *>(a + base + k);
            v[k] = q.x;
            v[k + 1] = q.y;
            v[k + 2] = q.z;
            v[k + 3] = q.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < kScanPer; ++k) v[k] = base + k < m ? a[base + k] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        const uint32_t x = v[k];
        v[k] = s;
        s += x;
    }
    uint32_t total;
    const uint32_t run = block_exclusive_scan<kScanBlock>(s, sh, &total);
    if (whole) {
#pragma unroll
        for (int k = 0; k < kScanPer; k += 4)
            *reinterpret_cast<uint4 *>(a + base + k) =
                make_uint4(run + v[k], run + v[k + 1], run + v[k + 2], run + v[k + 3]);
    } else {
#pragma unroll
        for (int k = 0; k < kScanPer; ++k)
            if (base + k < m) a[base + k] = run + v[k];
    }
    if (threadIdx.x == 0) block_sums[blockIdx.x] = total;
}

__global__ void __launch_bounds__(kSumsBlock) k_scan_sums(uint32_t *__restrict__ s, int64_t nb) {
    __shared__ uint32_t sh[kSumsBlock / kWave];
    uint32_t carry = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += kSumsBlock * kSumsPer) {
        const int64_t i = b0 + threadIdx.x * kSumsPer;
        uint32_t v[kSumsPer], t = 0;
#pragma unroll
        for (int k = 0; k < kSumsPer; ++k) {
            v[k] = i + k < nb ? s[i + k] : 0u;
            t += v[k];
        }
        uint32_t total;
        uint32_t run = block_exclusive_scan<kSumsBlock>(t, sh, &total) + carry;
#pragma unroll
        for (int k = 0; k < kSumsPer; ++k) {
            if (i + k < nb) s[i + k] = run;
            run += v[k];
        }
        carry += total;
    }
}

__global__ void __launch_bounds__(kScanBlock) k_scan_add(uint32_t *__restrict__ a, int64_t m,
                                                         const uint32_t *__restrict__ block_sums) {
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanChunk + threadIdx.x;
    const uint32_t add = block_sums[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanPer; ++k)
        if (base + k * kScanBlock < m) a[base + k * kScanBlock] += add;
}

// --------------------------------------------------------------- scatter

// The counters of all views are scanned as one array, so a point's slot is
// its counter plus its block's offset less the points of the views before, plus
// its place among the points of its cell: kept from the counting (47 us for 1M
// points), or where there is no room for it drawn from the counter again (70).
__global__ void __launch_bounds__(256) k_scatter(const ViewDesc *__restrict__ views, int n_views,
                                                 const uint32_t *__restrict__ sums) {
    const ViewDesc v = views[find_block(views, n_views, blockIdx.x)];
    const int64_t i0 = (static_cast<int64_t>(blockIdx.x) - v.blk0) * (256 * kKeysPer) + threadIdx.x;
#pragma unroll
    for (int q = 0; q < kKeysPer; ++q) {
        const int64_t i = i0 + q * 256;
        if (i >= v.n) return;
        const uint32_t k = v.keys[i];
        const uint32_t pos = (v.slots ? v.hist[k] + v.slots[i] : atomicAdd(v.hist + k, 1u)) + sums[(v.hist0 + k) / kScanChunk] - v.points0;
        const double4 a = v.src[i];
        v.a64s[pos] = a;
        if (v.a32s)
            v.a32s[pos] = make_float4(static_cast<float>(a.x), static_cast<float>(a.y), static_cast<float>(a.z), 0.0f);
    }
}

// --------------------------------------------------------------- launchers

__global__ void __launch_bounds__(256) k_zero_u32(uint32_t *p, int64_t n) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// 16 bytes per thread and step; p is 16-byte aligned and n a multiple of 4
__global__ void __launch_bounds__(256) k_zero_u128(uint4 *p, int64_t n4) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n4;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// The same, and the descriptors of a small call by value: a copy from the host's
// memory takes a transfer of its own (about 10 us of a call of 113 us).
struct PutData {
    uint4 v[kPutBytes / 16];
};
__global__ void __launch_bounds__(256) k_zero_put(uint4 *p, int64_t n4, uint4 *dst, int n_put, const PutData d) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n4;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        p[i] = make_uint4(0u, 0u, 0u, 0u);
    if (blockIdx.x == 0 && static_cast<int>(threadIdx.x) < n_put) dst[threadIdx.x] = d.v[threadIdx.x];
}

// Ordering counters of a view of n points (a multiple of 4; at least one per
// face of the cube).
uint32_t order_buckets(int64_t n, int per_point) {
    const int64_t m = std::min<int64_t>(std::max<int64_t>(per_point * n, kMinBuckets), int64_t(1) << 26);
    return static_cast<uint32_t>((m + 3) & ~int64_t(3));
}

size_t scan_sums_words(int64_t m) { return static_cast<size_t>((m + kScanChunk - 1) / kScanChunk); }

hipError_t launch_zero_u32(uint32_t *p, int64_t m, hipStream_t st) {
    if (m <= 0) return hipSuccess;
    k_zero_u32<<<dim3(static_cast<uint32_t>((m + 255) / 256)), dim3(256), 0, st>>>(p, m);
    return hipGetLastError();
}

// Zeroes `bytes` (a multiple of 16) at the 16-byte aligned p.
hipError_t launch_zero(void *p, size_t bytes, hipStream_t st) {
    if (bytes == 0) return hipSuccess;
    const int64_t n4 = static_cast<int64_t>(bytes / 16);
    const int64_t blocks = std::min<int64_t>((n4 + 255) / 256, 4096);
    k_zero_u128<<<dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, st>>>(static_cast<uint4 *>(p), n4);
    return hipGetLastError();
}

// Zeroes as launch_zero does and writes `n` (at most kPutBytes) bytes at `src`,
// host memory, to the 16-byte aligned dst, up to 15 bytes more behind them.
hipError_t launch_zero_put(void *p, size_t bytes, void *dst, const void *src, size_t n, hipStream_t st) {
    if (n > kPutBytes) return hipErrorInvalidValue;
    PutData d = {};
    if (n) memcpy(&d, src, n);
    const int64_t n4 = static_cast<int64_t>(bytes / 16);
    const int64_t blocks = std::min<int64_t>(std::max<int64_t>((n4 + 255) / 256, 1), 4096);
    k_zero_put<<<dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, st>>>(
        static_cast<uint4 *>(p), n4, static_cast<uint4 *>(dst), static_cast<int>((n + 15) / 16), d);
    return hipGetLastError();
}

// dst[w] += sum over s < n_copies of src[s * n + w], w < n (one thread per word)
__global__ void __launch_bounds__(256) k_add_copies(unsigned long long *__restrict__ dst,
                                                    const unsigned long long *__restrict__ src, int64_t n,
                                                    int32_t n_copies) {
    const int64_t w = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (w >= n) return;
    unsigned long long v = 0;
    for (int32_t s = 0; s < n_copies; ++s) v += src[static_cast<int64_t>(s) * n + w];
    dst[w] += v;
}

hipError_t launch_add_copies(unsigned long long *dst, const unsigned long long *src, int64_t n, int32_t n_copies,
                             hipStream_t st) {
    if (n <= 0 || n_copies <= 0) return hipSuccess;
    const int64_t blocks = (n + 255) / 256;
    k_add_copies<<<dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, st>>>(dst, src, n, n_copies);
    return hipGetLastError();
}

// In-place exclusive prefix sum of a[0, m), a 16-byte aligned; sums:
// scan_sums_words(m) words.
hipError_t launch_exclusive_scan(uint32_t *a, int64_t m, uint32_t *sums, hipStream_t st) {
    if (m <= 0) return hipSuccess;
    const int64_t nb = (m + kScanChunk - 1) / kScanChunk;
    k_scan_local<<<dim3(static_cast<uint32_t>(nb)), dim3(kScanBlock), 0, st>>>(a, m, sums);
    k_scan_sums<<<dim3(1), dim3(kSumsBlock), 0, st>>>(sums, nb);
    k_scan_add<<<dim3(static_cast<uint32_t>(nb)), dim3(kScanBlock), 0, st>>>(a, m, sums);
    return hipGetLastError();
}

int64_t convert_blocks(int64_t n) { return (n + 256 * convert_per(n) - 1) / (256 * convert_per(n)); }
int64_t order_blocks(int64_t n) { return (n + 256 * kKeysPer - 1) / (256 * kKeysPer); }

// Converts the sources (blk0 = running sum of convert_blocks(n); n > 0 each).
hipError_t launch_convert(const SrcDesc *srcs, int n_srcs, int64_t blocks, hipStream_t st) {
    if (n_srcs <= 0) return hipSuccess;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    k_convert<<<dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, st>>>(srcs, n_srcs);
    return hipGetLastError();
}

// Spatially ordered copies of the views (blk0 = running sum of
// order_blocks(n); n > 0 each).  hist: the views' counters one after the
// other, `buckets` words, zeroed; sums: scan_sums_words(buckets) words.
hipError_t launch_order(const ViewDesc *views, int n_views, int64_t blocks, uint32_t *hist, int64_t buckets,
                        uint32_t *sums, hipStream_t st) {
    if (n_views <= 0) return hipSuccess;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    const int64_t nb = (buckets + kScanChunk - 1) / kScanChunk;
    const dim3 grid(static_cast<uint32_t>(blocks));
    k_keys<<<grid, dim3(256), 0, st>>>(views, n_views);
    k_scan_local<<<dim3(static_cast<uint32_t>(nb)), dim3(kScanBlock), 0, st>>>(hist, buckets, sums);
    k_scan_sums<<<dim3(1), dim3(kSumsBlock), 0, st>>>(sums, nb);
    k_scatter<<<grid, dim3(256), 0, st>>>(views, n_views, sums);
    return hipGetLastError();
}

#endif  // tile-independent part

// ------------------------------------------------ per tile size

namespace PC_TILE_NS {

// ---------------------------------------------------------------- bounds

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, kWave));
    return v;
}

// One wave per tile of kTile sorted points: centre = normalised mean, radius
// = largest distance from the centre, rounded outward.  Written as
// (cx, cy, cz, r).  The same for each of the tile's kSubs sub-blocks of kSub
// points (the r-th point of every lane: sub-block r), into sub[kSubs t + r].
// Each point is also written in Gram form centred on the tile's centre:
// b' = RN32(b - c) (difference in binary64), (-2 b'_x, -2 b'_y, -2 b'_z,
// |b'|^2) with |b'|^2 formed in binary32 as z*z + (y*y + x*x) by fused
// multiply-adds.
__device__ __forceinline__ double4 ball_of(const double4 *p, const bool *ok, int rows, double sx, double sy,
                                           double sz, double4 fallback) {
    const double norm = sqrt(sx * sx + sy * sy + sz * sz);
    double cx, cy, cz;
    if (norm > 1e-6) {
        cx = sx / norm;
        cy = sy / norm;
        cz = sz / norm;
    } else {
        cx = fallback.x;
        cy = fallback.y;
        cz = fallback.z;
    }
    double m = 0.0;
    for (int r = 0; r < rows; ++r) {
        if (ok[r]) {
            const double dx = p[r].x - cx, dy = p[r].y - cy, dz = p[r].z - cz;
            m = fmax(m, dx * dx + dy * dy + dz * dz);
        }
    }
    m = wave_max(m);
    return make_double4(cx, cy, cz, sqrt(m) * (1.0 + 0x1p-40) + 0x1p-60);
}

__global__ void __launch_bounds__(kWave) k_bounds(const ViewDesc *__restrict__ views, int n_views) {
    static_assert(kSub == kWave, "a sub-block is one point per lane");
    // the view of this tile (its first tile is tile0 of the launch)
    int lo = 0, hi = n_views - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (views[mid].tile0 <= static_cast<int64_t>(blockIdx.x)) lo = mid;
        else hi = mid - 1;
    }
    const ViewDesc &vw = views[lo];
    const double4 *__restrict__ a64s = vw.a64s;
    const int64_t n = vw.n;
    double4 *__restrict__ bounds = vw.bounds;
    double4 *__restrict__ sub = bounds + vw.tiles;
    float4 *__restrict__ g32s = vw.g32s;
    const int64_t t = static_cast<int64_t>(blockIdx.x) - vw.tile0;
    const int lane = threadIdx.x;
    const int64_t b = t * kTile;
    double sx = 0, sy = 0, sz = 0;
    double4 p[kR];
    bool ok[kR];
    double4 rs[kR];
#pragma unroll
    for (int r = 0; r < kR; ++r) {
        const int64_t i = b + r * kWave + lane;
        ok[r] = i < n;
        p[r] = a64s[ok[r] ? i : b];
        // every lane takes part in the reductions; lanes past the end add 0
        rs[r] = make_double4(wave_sum(ok[r] ? p[r].x : 0.0), wave_sum(ok[r] ? p[r].y : 0.0),
                             wave_sum(ok[r] ? p[r].z : 0.0), 0.0);
        sx += rs[r].x;
        sy += rs[r].y;
        sz += rs[r].z;
    }
    const double4 first = a64s[b];
    const double4 tb = ball_of(p, ok, kR, sx, sy, sz, first);
    if (lane == 0) bounds[t] = tb;
#pragma unroll
    for (int r = 0; r < kR; ++r) {
        // an empty sub-block (past a ragged end) gets the tile's ball; it is
        // never split from
        const bool any = __ballot(ok[r]) != 0ull;
        const double4 sb = any ? ball_of(&p[r], &ok[r], 1, rs[r].x, rs[r].y, rs[r].z, first) : tb;
        if (lane == 0) sub[t * kSubs + r] = sb;
    }
    if (!g32s) return;
    const double cx = tb.x, cy = tb.y, cz = tb.z;
#pragma unroll
    for (int r = 0; r < kR; ++r) {
        if (ok[r]) {
            const float x = static_cast<float>(p[r].x - cx);
            const float y = static_cast<float>(p[r].y - cy);
            const float z = static_cast<float>(p[r].z - cz);
            g32s[b + r * kWave + lane] =
                make_float4(-2.0f * x, -2.0f * y, -2.0f * z, __builtin_fmaf(z, z, __builtin_fmaf(y, y, x * x)));
        }
    }
}

// ----------------------------------------------------------------- prune


template <typename P>
__device__ __forceinline__ uint32_t count_le(P e, int32_t n, double c) {
    int32_t lo = 0, hi = n;
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (e[mid] <= c) lo = mid + 1;
        else hi = mid;
    }
    return static_cast<uint32_t>(lo);
}

// The prune decision for one tile pair.  The chord of every pair of a tile
// pair lies in [d - rI - rJ, d + rI + rJ] (triangle inequality in R^3, d =
// distance of the centres); when the squared interval, widened by 1e-12
// relative for the rounding of these bounds and of the binary64 chord itself,
// sits inside one bin, all the item's pairs belong to that bin (bin >= 0).
// Otherwise the item survives (bin = -1) with its tags: k0 = edges at or below
// the interval, m = edges inside (kept when m <= PC_FEWCUT), and the Gram /
// matrix-core eligibility.
struct PruneOut {
    int32_t bin;
    uint64_t pairs;
    uint64_t tags;  // bits 40..63 of the survivor entry (block kernel: bits 32..53)
    uint64_t sub;   // sub-block word of a split item, else 0
};

// Squared-chord interval of the pairs between two balls (centre, radius):
// [c_lo, c_hi], and the chord lower bound lo.
__device__ __forceinline__ void chord_interval(const double4 &bi, const double4 &bj, double &lo, double &c_lo,
                                               double &c_hi) {
    // outward-rounded bounds: distance of the centres (+-2^-45 relative),
    // radii (+2^-45), absolute 2^-50 for the subtraction, then the squared
    // chord interval widened by 1e-12 relative and 1e-300 absolute
    const double dx = bi.x - bj.x, dy = bi.y - bj.y, dz = bi.z - bj.z;
    const double d = sqrt(dx * dx + dy * dy + dz * dz);
    const double rs = (bi.w + bj.w) * (1.0 + 0x1p-45);
    lo = fmax(0.0, d * (1.0 - 0x1p-45) - rs - 0x1p-50);
    const double hi = d * (1.0 + 0x1p-45) + rs + 0x1p-50;
    // (a squared chord is never negative, so an edge at 0 always lies at or
    // below the interval: few-edge items never hold it)
    c_lo = fmax(lo * lo * (1.0 - 1e-12) - 1e-300, 0.0);
    c_hi = hi * hi * (1.0 + 1e-12) + 1e-300;
}

// far_l: a chord length past the last edge, sqrt(e[n_edges - 1]) * (1 +
// 1e-12) in binary64.  A tile pair whose squared centre distance d2 exceeds
// (far_l + r_I + r_J)^2 (1 + 1e-12) has every chord past the last edge: the
// computed d2 is at most 5 ulp above the true squared distance D^2 and the
// bound at most 4 ulp below its value, so D - r_I - r_J > far_l (1 + 0.49e-12);
// every pair is at least that far apart, and its binary64 squared chord
// (5 ulp) stays above e[n_edges - 1].
template <bool BLOCKS, typename P>
__device__ __forceinline__ PruneOut prune_item(const SegDesc &sd, int64_t t, int64_t u, const double4 &bi,
                                               const double4 &bj, P e, int32_t n_edges, double far_l,
                                               int32_t mfma_ok, int32_t split_ok) {
    PruneOut o;
    o.sub = 0;
    constexpr int kT = BLOCKS ? kBlockTile : kTile;
    const int64_t ni = min<int64_t>(kT, sd.ni - t * kT);
    const int64_t nj = min<int64_t>(kT, sd.nj - u * kT);
    const bool diag = sd.tri && t == u;
    o.pairs = diag ? static_cast<uint64_t>(ni * (ni - 1) / 2) : static_cast<uint64_t>(ni * nj);
    {
        // past the last edge without the square root (most tile pairs of a
        // wide field)
        const double dx = bi.x - bj.x, dy = bi.y - bj.y, dz = bi.z - bj.z;
        const double reach = far_l + (bi.w + bj.w);
        if (dx * dx + dy * dy + dz * dz > reach * reach * (1.0 + 1e-12)) {
            o.bin = n_edges;
            o.tags = 0;
            return o;
        }
    }
    double lo, c_lo, c_hi;
    chord_interval(bi, bj, lo, c_lo, c_hi);
    if (c_lo > e[n_edges - 1]) {
        // the whole interval lies past the last edge (most tile pairs of a
        // wide field): the bin above it, without the two searches
        o.bin = n_edges;
        o.tags = 0;
        return o;
    }
    const uint32_t k_lo = count_le(e, n_edges, c_lo);
    const uint32_t k_hi = count_le(e, n_edges, c_hi);
    if (k_lo == k_hi) {
        o.bin = static_cast<int32_t>(k_lo);
        o.tags = 0;
        return o;
    }
    o.bin = -1;
    // edges inside the interval: k_lo .. k_hi-1; few of them are compared one
    // by one instead of through the cell table
    const uint32_t m = k_hi - k_lo;
    if (BLOCKS) {
        o.tags = (static_cast<uint64_t>(k_lo) << 32) | (static_cast<uint64_t>(m) << 43);
        return o;
    }
    static_assert(PC_FEWCUT >= 1 && PC_FEWCUT <= kFewMax, "few-edge cut");
    const bool is_few = m <= static_cast<uint32_t>(PC_FEWCUT);
    // few-edge full tiles whose chord lower bound is at least twice the
    // smaller bounding radius: eligible for the matrix-core path (bit 63),
    // centred on the j-tile when that one is smaller (bit 62); otherwise the
    // vector path forms Gram chords centred on the j-tile (bit 61) under the
    // same condition on the j radius
    const bool full = ni == kTile && nj == kTile;
    const bool mfma = mfma_ok && is_few && !diag && full && 2.0 * fmin(bi.w, bj.w) <= lo;
    const bool gram_j = !mfma && is_few && !diag && 2.0 * bj.w <= lo;
    o.tags = (static_cast<uint64_t>(k_lo) << kItemBits) |
             (static_cast<uint64_t>(is_few ? m : 0u) << (kItemBits + 11)) | (mfma ? (1ull << 63) : 0ull) |
             ((mfma && bj.w < bi.w) ? (1ull << 62) : 0ull) | (gram_j ? (1ull << 61) : 0ull);
    if (split_ok && !mfma && !diag && full) {
        // the same decision for each sub-block of the j-tile; the Gram form
        // stays centred on the whole j-tile, so its condition keeps the
        // j-tile's radius against the sub-block's chord lower bound
        uint64_t w = 0;
#pragma unroll
        for (int s = 0; s < kSubs; ++s) {
            const double4 bs = sd.jb_sub[u * kSubs + s];
            double lo_s, cl, ch;
            chord_interval(bi, bs, lo_s, cl, ch);
            const uint32_t kl = count_le(e, n_edges, cl);
            const uint32_t kh = count_le(e, n_edges, ch);
            uint32_t f;
            if (kl == kh) {
                f = kl | kSubWhole;
            } else {
                const uint32_t ms = kh - kl;
                const bool few = ms <= static_cast<uint32_t>(PC_FEWCUT);
                f = kl | ((few ? ms : 0u) << 11) | ((few && 2.0 * bj.w <= lo_s) ? kSubGram : 0u);
            }
            w |= static_cast<uint64_t>(f) << (16 * s);
        }
        o.sub = w;
        o.tags |= 1ull << kSplitBit;
    }
    return o;
}

// Sub-blocks of a split item left for the counting kernel.
__device__ __forceinline__ uint32_t open_subs(uint64_t w) {
    uint32_t n = 0;
#pragma unroll
    for (int s = 0; s < kSubs; ++s) n += (((w >> (16 * s)) & kSubWhole) == 0u) ? 1u : 0u;
    return n;
}

// (t, u) and item number of column c of prune row r (map_item's fold for a
// triangle: row r holds (r, r..T-1) then (T-1-r, T-1-r..T-1))
__device__ __forceinline__ bool row_item(const SegDesc &sd, int64_t r, int64_t c, int64_t &t, int64_t &u,
                                         uint64_t &q) {
    const int64_t T = sd.tiles_i;
    if (sd.tri) {
        q = static_cast<uint64_t>(r * (T + 1) + c);
        if (c < T - r) {
            t = r;
            u = r + c;
        } else {
            t = T - 1 - r;
            u = t + (c - (T - r));
        }
        return c < T + 1 && q < sd.n_items;
    }
    t = r;
    u = c;
    q = static_cast<uint64_t>(r * sd.tiles_j + c);
    return c < sd.tiles_j;
}

constexpr int kPruneThreads = 256;     // threads per prune workgroup
constexpr int kPruneMaskSteps = 128;  // steps of 256 columns whose survivor ballots are kept (4 KB)

// Column c of prune row r with the bounds of its two tiles; a column past the
// row's end (valid false) loads the bounds of tile 0, which every segment has.
struct PruneCol {
    int64_t t, u;
    uint64_t q;
    bool valid;
    double4 bi, bj;
};

__device__ __forceinline__ void load_col(const SegDesc &sd, int64_t r, int64_t c, PruneCol &k) {
    k.valid = row_item(sd, r, c, k.t, k.u, k.q);
    k.bi = sd.ib[k.valid ? k.t : 0];
    k.bj = sd.jb[k.valid ? k.u : 0];
}

// One workgroup per row of tile pairs (one i-tile, or the two i-tiles of a
// folded triangle row), threads across its columns: (t, u) and the item
// number come without divisions, and the edges of the row's table sit in LDS.
// Whole tile pairs are added to an LDS histogram and survivors counted in a
// first pass; the workgroup then reserves its survivors' slots with one global
// atomic and writes them in a second pass (the decision is recomputed), and
// flushes its histogram and statistics with one atomic per non-zero entry --
// global atomics on a few shared counters would otherwise serialise the pass.
//
// BLOCKS: for the block kernel, which looks at every survivor block by block
// itself: survivors carry their segment, edges and tiles, no sub-blocks are
// judged here and no statistics kept but the number of survivors.
template <bool BLOCKS>
__global__ void __launch_bounds__(kPruneThreads) k_prune(const SegDesc *__restrict__ segs, int32_t n_segs,
                                               const TableDesc *__restrict__ tabs,
                                               uint64_t *__restrict__ survivors, uint64_t *__restrict__ sub_out,
                                               unsigned long long *__restrict__ meta, int32_t mfma_ok,
                                               int32_t split_ok) {
    // meta[0] = survivors (the slot counter).  Statistics, summed over the
    // kPruneStripes stripes at meta[kPruneStatBase + stripe * kPruneStripeWords
    // + k] (k as in s_stat): k = 1 pairs left for the counting kernel, 2
    // survivors marked for the matrix cores; work units (a survivor, or an
    // open sub-block of a split one): 3 with at most PC_FEWCUT edges in their
    // chord interval, 4 with vector-path chords in Gram form; 5 split
    // survivors; pairs left for the counting kernel by the path it takes them
    // through (the same decisions as k_count): 6 + m binned against m edges
    // one by one (m = 1..3), 6 through the cell table; 10 pairs whose chords
    // the vector path forms in Gram form, 11 pairs on the matrix cores.
    __shared__ double e_lds[kMaxEdges];
    __shared__ unsigned long long h_lds[kMaxEdges + 1];
    // survivors, pairs, matrix-core, few-edge, Gram, split; pairs by m (4),
    // Gram-form pairs, matrix-core pairs
    static_assert(kPruneStats <= kPruneStripeWords, "statistics per stripe");
    constexpr int kStats = kPruneStats;
    __shared__ unsigned long long s_stat[kStats];
    __shared__ unsigned long long s_base;
    __shared__ unsigned int s_cursor;
    // survivor ballots of the first kPruneMaskSteps steps of each wave
    __shared__ uint64_t s_mask[kPruneMaskSteps][kPruneThreads / kWave];
    const int64_t row_g = blockIdx.x;
    int s = 0;  // last segment with prow0 <= row_g
    {
        int lo = 0, hi = n_segs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (segs[mid].prow0 <= row_g) lo = mid;
            else hi = mid - 1;
        }
        s = lo;
    }
    const SegDesc &sd = segs[s];
    const TableDesc &td = tabs[sd.tab];
    const int32_t n_edges = td.n_edges;
    const int tid = static_cast<int>(threadIdx.x);
    const int lane = tid & (kWave - 1);
    for (int32_t k = tid; k < n_edges; k += blockDim.x) e_lds[k] = td.e64[k];
    for (int32_t k = tid; k <= n_edges; k += blockDim.x) h_lds[k] = 0ull;
    if (tid < kStats) s_stat[tid] = 0ull;
    if (tid == 0) s_cursor = 0u;
    __syncthreads();
    const int64_t r = row_g - sd.prow0;
    const int64_t cols = sd.tri ? sd.tiles_i + 1 : sd.tiles_j;
    const double far_l = sqrt(e_lds[n_edges - 1]) * (1.0 + 1e-12);
    constexpr unsigned long long kSubPairs = static_cast<unsigned long long>(kTile) * kSub;

    // pass 1: histogram of whole tile pairs and sub-blocks, statistics of
    // survivors.  Whole tile pairs past the last edge (most of them in a wide
    // field) and the statistics add up in registers over the row and are
    // reduced once at its end; other whole tile pairs go to the LDS histogram.
    unsigned long long above = 0;
    // survivors, pairs left, matrix-core items, few-edge work units, Gram
    // work units, split items; pairs by the counting kernel's path: by edges
    // compared one by one (index m, 0 = cell table), Gram-form chords, matrix
    // cores (the layout of s_stat)
    unsigned long long st[kStats];
#pragma unroll
    for (int k = 0; k < kStats; ++k) st[k] = 0ull;
    // the next column's tiles load while this one is judged; each wave keeps
    // the ballot of its survivors per step for the second pass
    PruneCol cur, nxt;
    load_col(sd, r, tid, cur);
    nxt = cur;
    const int wave = tid / kWave;
    for (int64_t c0 = 0, it = 0; c0 < cols; c0 += kPruneThreads, ++it) {
        if (c0 + kPruneThreads < cols) load_col(sd, r, c0 + kPruneThreads + tid, nxt);
        bool survive = false;
        if (cur.valid) {
            const PruneOut o =
                prune_item<BLOCKS>(sd, cur.t, cur.u, cur.bi, cur.bj, e_lds, n_edges, far_l, mfma_ok, split_ok);
            survive = o.bin < 0;
            if (o.bin == n_edges) {
                above += o.pairs;
            } else if (o.bin >= 0) {
                atomicAdd(&h_lds[o.bin], static_cast<unsigned long long>(o.pairs));
            } else if (BLOCKS) {
                st[0] += 1ull;
                survive = true;
            } else if (o.sub) {
                // the kernel forms a split item's chords in Gram form when
                // every open sub-block allows it
                bool gram_all = true;
#pragma unroll
                for (int k = 0; k < kSubs; ++k) {
                    const uint32_t f = static_cast<uint32_t>(o.sub >> (16 * k)) & 0xFFFFu;
                    if (!(f & kSubWhole) && !(f & kSubGram)) gram_all = false;
                }
                unsigned long long left = 0;
#pragma unroll
                for (int k = 0; k < kSubs; ++k) {
                    const uint32_t f = static_cast<uint32_t>(o.sub >> (16 * k)) & 0xFFFFu;
                    if (f & kSubWhole) {
                        atomicAdd(&h_lds[f & 2047u], kSubPairs);
                    } else {
                        const uint32_t m = (f >> 11) & 3u;
                        left += kSubPairs;
                        st[3] += m != 0u ? 1ull : 0ull;
                        st[4] += (f & kSubGram) != 0u ? 1ull : 0ull;
                        st[6 + m] += kSubPairs;
                        st[10] += gram_all ? kSubPairs : 0ull;
                    }
                }
                st[0] += left != 0 ? 1ull : 0ull;
                st[1] += left;
                st[5] += left != 0 ? 1ull : 0ull;
                survive = left != 0;
            } else {
                const uint32_t m = static_cast<uint32_t>((o.tags >> (kItemBits + 11)) & 3u);
                const bool mc = (o.tags >> 63) != 0;
                const bool gram = ((o.tags >> 61) & 1u) != 0;
                st[0] += 1ull;
                st[1] += o.pairs;
                st[2] += mc ? 1ull : 0ull;
                st[3] += m != 0u ? 1ull : 0ull;
                st[4] += gram ? 1ull : 0ull;
                st[6 + m] += o.pairs;
                st[10] += (!mc && gram && m != 0u) ? o.pairs : 0ull;
                st[11] += mc ? o.pairs : 0ull;
            }
        }
        const uint64_t sm = __ballot(survive);
        if (it < kPruneMaskSteps && lane == 0) s_mask[it][wave] = sm;
        cur = nxt;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        above += __shfl_xor(above, o, kWave);
#pragma unroll
        for (int k = 0; k < kStats; ++k) st[k] += __shfl_xor(st[k], o, kWave);
    }
    if (lane == 0) {
        if (above) atomicAdd(&h_lds[n_edges], above);
#pragma unroll
        for (int k = 0; k < kStats; ++k)
            if (st[k]) atomicAdd(&s_stat[k], st[k]);
    }
    __syncthreads();
    if (tid == 0) s_base = s_stat[0] ? atomicAdd(meta + 0, s_stat[0]) : 0ull;
    __syncthreads();

    // pass 2: the survivors, written into the workgroup's reserved slots
    if (s_stat[0]) {
        const int wave = tid / kWave;
        for (int64_t c0 = 0, it = 0; c0 < cols; c0 += kPruneThreads, ++it) {
            // steps whose ballot the first pass kept: only their survivors
            // are judged again
            const uint64_t kept = it < kPruneMaskSteps ? s_mask[it][wave] : ~0ull;
            if (kept == 0) continue;
            bool survive = false;
            uint64_t tags = 0, sub = 0, q = 0, tu = 0;
            if ((kept >> lane) & 1u) {
                PruneCol k;
                load_col(sd, r, c0 + tid, k);
                if (k.valid) {
                    const PruneOut o =
                        prune_item<BLOCKS>(sd, k.t, k.u, k.bi, k.bj, e_lds, n_edges, far_l, mfma_ok, split_ok);
                    survive = o.bin < 0 && (o.sub == 0 || open_subs(o.sub) != 0);
                    tags = o.tags;
                    sub = o.sub;
                    q = k.q;
                    tu = static_cast<uint64_t>(k.t) | (static_cast<uint64_t>(k.u) << 32);
                }
            }
            const uint64_t sm = __ballot(survive);
            if (sm) {
                const uint64_t below = sm & ((lane == 0) ? 0ull : (~0ull >> (kWave - lane)));
                unsigned int at = 0;
                if (lane == __ffsll(static_cast<long long>(sm)) - 1)
                    at = atomicAdd(&s_cursor, static_cast<unsigned int>(__popcll(sm)));
                at = __shfl(at, __ffsll(static_cast<long long>(sm)) - 1, kWave);
                if (survive) {
                    const uint64_t slot = s_base + at + __popcll(below);
                    survivors[slot] = (BLOCKS ? static_cast<uint64_t>(s) : sd.item0 + q) | tags;
                    if (sub_out) sub_out[slot] = BLOCKS ? tu : sub;
                }
            }
        }
    }

    // flush: one atomic per non-zero bin and per statistic, into one of
    // kPruneStripes copies (by workgroup) of the counters and statistics
    unsigned long long *pc = sd.pcounts + static_cast<int64_t>(blockIdx.x % kPruneStripes) * sd.pstride;
    for (int32_t k = tid; k <= n_edges; k += blockDim.x) {
        const unsigned long long v = h_lds[k];
        if (v) atomicAdd(pc + k, v);
    }
    if (tid > 0 && tid < kStats && s_stat[0] && s_stat[tid])
        atomicAdd(meta + kPruneStatBase + (blockIdx.x % kPruneStripes) * kPruneStripeWords + tid, s_stat[tid]);
}

// Tile bounds of the ordered views: bounds[0, T) for a view's T tiles, then
// bounds[T, T + kSubs T) for their sub-blocks, and (where asked for) the
// Gram-form copy g32s.  tiles: over all views (tile0 = running sum).
hipError_t launch_bounds(const ViewDesc *views, int n_views, int64_t tiles, hipStream_t st) {
    if (n_views <= 0 || tiles <= 0) return hipSuccess;
    if (tiles > 0x7FFFFFFF) return hipErrorInvalidValue;
    k_bounds<<<dim3(static_cast<uint32_t>(tiles)), dim3(kWave), 0, st>>>(views, n_views);
    return hipGetLastError();
}

hipError_t launch_prune(const SegDesc *segs, int32_t n_segs, const TableDesc *tabs, int64_t total_rows,
                        uint64_t *survivors, uint64_t *sub, unsigned long long *meta, int32_t mfma_ok,
                        int32_t split_ok, bool blocks, hipStream_t st) {
    if (total_rows <= 0) return hipSuccess;
    if (total_rows > 0x7FFFFFFF) return hipErrorInvalidValue;
#if PC_R == 4
    const auto k = blocks ? k_prune<true> : k_prune<false>;
#else
    if (blocks) return hipErrorInvalidValue;  // the block kernel's pass is in the 256-point build
    const auto k = k_prune<false>;
#endif
    k<<<dim3(static_cast<uint32_t>(total_rows)), dim3(kPruneThreads), 0, st>>>(segs, n_segs, tabs, survivors, sub, meta,
                                                                                mfma_ok, split_ok);
    return hipGetLastError();
}

}  // namespace PC_TILE_NS

}  // namespace pc
