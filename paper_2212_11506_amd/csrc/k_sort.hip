// Bounding box, Morton codes and the sort of the codes (gfx950).
//
// Quadtree Building (Algorithm 1 and the paragraph on Morton codes): the
// square domain is centred on the bounding box with half-side r_span, each
// coordinate is quantised to 32 bits and the two are bit-interleaved with
// dimension 0 in the even bits.  Sorting the codes puts points of a cell next
// to each other, which is what the tree build and the repulsive traversal
// rely on.
//
// The sort orders the pairs (code, index), which are distinct, so it need not be
// stable.  Three ways, by the number of points:
//  - up to kRankSortMax a key's place is counted, all against all, in one launch;
//  - up to kSampleSortMax a sample sort: every 64th code, taken while the codes
//    are formed, is ranked among the sampled ones, every fourth of those splits the
//    pairs into buckets of about 256, and a key's place is counted in its bucket:
//    four launches, each pair moved twice;
//  - beyond, an LSD radix sort over 8-bit digits: eight passes, each a kernel that
//    ranks a tile in LDS, finds the tile's global offsets with a decoupled
//    look-back over the tiles before it, and writes the tile out digit by digit;
//    its digit histograms are accumulated while the codes are formed.
// A radix pass takes 9.5 us however few points there are (its look-back is a chain
// of tiles), so eight of them are latency up to some 100k points; comparisons grow
// with n, and faster.  us of the kernels that make the codes and sort them, by
// rank / sample / radix: 1500 points 11 / 27 / -, 3000 16 / 33 / 89, 8000 27 / 32 / -,
// 10k 32 / 31 / 99, 70k - / 48 / 118, 300k - / 124 / 162, 600k - / 227 / 245, 1.3M
// - / 535 / 430.  The first line lies where they meet, the second at the last power of
// two before they do, near 800k points: whole steps by sample / radix, us, beside the
// sliced attraction 600k 637 / 661, 700k 702 / 721, 900k 866 / 856, 1.3M 1218 / 1156, beside
// the windows 600k 934 / 961, 700k 1010 / 1026, 900k 1341 / 1358, 1.3M 2046 / 2013.
#include "common.hpp"
#include "kernels.hpp"
#include <algorithm>

namespace bht {

// ------------------------------------------------------------------ bbox
// T: float (the path) or double (the fp64 variant); each block writes
// {min x, max x, min y, max y, non-finite flag} as 8 T.
template <typename T>
__global__ __launch_bounds__(256) void bbox_partial_kernel(const vec2_t<T> *__restrict__ Y, int64_t n,
                                                           T *__restrict__ part)
{
    T mnx = INFINITY, mny = INFINITY, mxx = -INFINITY, mxy = -INFINITY;
    uint32_t bad = 0;
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += int64_t(gridDim.x) * blockDim.x) {
        const vec2_t<T> y = Y[i];
        bad |= !(isfinite(y.x) && isfinite(y.y));
        mnx = vmin(mnx, y.x);
        mxx = vmax(mxx, y.x);
        mny = vmin(mny, y.y);
        mxy = vmax(mxy, y.y);
    }
    mnx = wave_min(mnx);
    mny = wave_min(mny);
    mxx = wave_max(mxx);
    mxy = wave_max(mxy);
    bool anybad = ballot(bad != 0) != 0;
    __shared__ T s[4][4];
    __shared__ uint32_t sb[4];
    int w = threadIdx.x / kWave;
    if (lane_id() == 0) {
        s[w][0] = mnx;
        s[w][1] = mxx;
        s[w][2] = mny;
        s[w][3] = mxy;
        sb[w] = anybad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        T r[4] = {s[0][0], s[0][1], s[0][2], s[0][3]};
        uint32_t b = sb[0];
        for (int k = 1; k < 4; ++k) {
            r[0] = vmin(r[0], s[k][0]);
            r[1] = vmax(r[1], s[k][1]);
            r[2] = vmin(r[2], s[k][2]);
            r[3] = vmax(r[3], s[k][3]);
            b |= sb[k];
        }
        T *o = part + 8 * blockIdx.x;
        o[0] = r[0];
        o[1] = r[1];
        o[2] = r[2];
        o[3] = r[3];
        reinterpret_cast<uint32_t *>(o + 4)[0] = b;
    }
}

// The per-call scalars and counters, reset by the box kernel that starts a call.
__device__ inline void reset_call_state(Header *hdr, uint32_t nonfinite)
{
    hdr->flags = nonfinite ? kErrNonFinite : 0u;
    hdr->Z = 0.0;
    hdr->interactions = 0;
    for (int k = 0; k < kSortPasses; ++k) hdr->tile_counter[k] = 0;
    hdr->ticket_bbox = 0;
    hdr->ticket_rep = 0;
    hdr->attract_next = 0;
    hdr->max_depth = 0;
}

// The box from its parts by a block of 256 threads, and from it the quantisation
// parameters in fp64: s_root = {root of either axis, scale}.  `write`: leave them
// in the header as well and reset the per-call counters.
template <typename T>
__device__ inline void finish_box(const T *__restrict__ part, int nparts, Header *__restrict__ hdr, bool write,
                                  double *s_root)
{
    T mnx = INFINITY, mny = INFINITY, mxx = -INFINITY, mxy = -INFINITY;
    uint32_t bad = 0;
    for (int k = threadIdx.x; k < nparts; k += blockDim.x) {
        const T *p = part + 8 * k;
        mnx = vmin(mnx, p[0]);
        mxx = vmax(mxx, p[1]);
        mny = vmin(mny, p[2]);
        mxy = vmax(mxy, p[3]);
        bad |= reinterpret_cast<const uint32_t *>(p + 4)[0];
    }
    mnx = wave_min(mnx);
    mny = wave_min(mny);
    mxx = wave_max(mxx);
    mxy = wave_max(mxy);
    bool anybad = ballot(bad != 0) != 0;
    __shared__ T s[4][4];
    __shared__ uint32_t sb[4];
    int w = threadIdx.x / kWave;
    if (lane_id() == 0) {
        s[w][0] = mnx;
        s[w][1] = mxx;
        s[w][2] = mny;
        s[w][3] = mxy;
        sb[w] = anybad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        T r[4] = {s[0][0], s[0][1], s[0][2], s[0][3]};
        uint32_t b = sb[0];
        for (int k = 1; k < 4; ++k) {
            r[0] = vmin(r[0], s[k][0]);
            r[1] = vmax(r[1], s[k][1]);
            r[2] = vmin(r[2], s[k][2]);
            r[3] = vmax(r[3], s[k][3]);
            b |= sb[k];
        }
        // fp64, fixed operation order: the codes depend on these bits
        double c0 = (double(r[0]) + double(r[1])) * 0.5;
        double c1 = (double(r[2]) + double(r[3])) * 0.5;
        double e0 = double(r[1]) - double(r[0]);
        double e1 = double(r[3]) - double(r[2]);
        double rs = 0.5 * (e0 > e1 ? e0 : e1);
        s_root[0] = c0 - rs;
        s_root[1] = c1 - rs;
        s_root[2] = rs > 0.0 ? 2147483648.0 / rs : 0.0;
        if (write) {
            hdr->bmin[0] = float(r[0]);
            hdr->bmax[0] = float(r[1]);
            hdr->bmin[1] = float(r[2]);
            hdr->bmax[1] = float(r[3]);
            hdr->cent[0] = c0;
            hdr->cent[1] = c1;
            hdr->rspan = rs;
            hdr->yroot[0] = c0 - rs;
            hdr->yroot[1] = c1 - rs;
            hdr->scale = s_root[2];
            reset_call_state(hdr, b);
        }
    }
    __syncthreads();
}

// One block: the box and the histograms' clearing, before the radix sort's codes.
template <typename T>
__global__ __launch_bounds__(256) void bbox_final_kernel(const T *__restrict__ part, int nparts,
                                                         Header *__restrict__ hdr, uint32_t *__restrict__ hist)
{
    __shared__ double s_root[3];
    for (int k = threadIdx.x; k < kHistCopies * kHistWords; k += blockDim.x) hist[k] = 0;
    finish_box(part, nparts, hdr, true, s_root);
}

// ------------------------------------------------------------------ Morton
template <typename T> __device__ inline uint32_t quantise(T y, double yroot, double scale)
{
    double q = (double(y) - yroot) * scale;
    if (!(q > 0.0)) return 0u; // also catches NaN
    if (q >= 4294967295.0) return 0xffffffffu;
    return uint32_t(q); // truncation toward zero
}

// Interleaving by its definition: bit k of a grid coordinate goes to bit 2k
// of its spread word, and dimension d is then shifted to bit 2k + d.  The
// spread is taken a byte at a time: entry b of a 256-entry table holds byte b
// with each bit k moved to bit 2k (built from that rule, one entry per
// thread), and byte j of the coordinate lands at bit 16 j of the word.
__device__ inline uint32_t spread_byte_rule(uint32_t b)
{
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) s |= ((b >> k) & 1u) << (2 * k);
    return s;
}

__device__ inline uint64_t spread_by_bytes(const uint16_t *__restrict__ tab, uint32_t v)
{
    return uint64_t(tab[v & 0xffu]) | (uint64_t(tab[(v >> 8) & 0xffu]) << 16) |
           (uint64_t(tab[(v >> 16) & 0xffu]) << 32) | (uint64_t(tab[v >> 24]) << 48);
}

// The digit counts of a tile (radix sort): cleared with the tile's look-back
// words of every pass, counted, and added to the global ones by the block.
__device__ inline void clear_tile(uint32_t *sh, uint32_t *__restrict__ status, int64_t tiles)
{
    for (int k = threadIdx.x; k < kSortPasses * kRadix; k += kSortBlock) {
        sh[k] = 0;
        status[(int64_t(k / kRadix) * tiles + blockIdx.x) * kRadix + k % kRadix] = 0;
    }
}

__device__ inline void count_digits(uint32_t *sh, uint64_t code)
{
#pragma unroll
    for (int p = 0; p < kSortPasses; ++p)
        atomicAdd(&sh[p * kRadix + int((code >> (p * kRadixBits)) & (kRadix - 1))], 1u);
}

__device__ inline void add_digits(const uint32_t *sh, uint32_t *__restrict__ hist)
{
    __syncthreads();
    uint32_t *hc = hist + (blockIdx.x % kHistCopies) * kHistWords;
    for (int k = threadIdx.x; k < kSortPasses * kRadix; k += kSortBlock)
        if (sh[k]) atomicAdd(&hc[k], sh[k]);
}

// Codes of one tile of points, the private copy of Y (in the caller's order,
// or in a layout order when `perm` is given: position i holds the point
// perm[i], gathered, which costs less than scattering each point to its
// position), and what the sort wants: its samples (kRadixSort = false) or the 8
// global digit histograms and cleared look-back words of this tile; also clears the
// per-position tree masks.  Without the radix sort every block finishes the box for
// itself (2-4 us of a launch for at most 16 KB read again, 32 KB in fp64) and takes
// one point a thread: eight, the radix sort's tile, leave 70k points in 35 blocks.
// 70k points: the box's last launch and this one took 5.4 + 10.8 us, now 4.8; 1500
// points 2.9 + 7.0, now 4.1.
template <typename T, bool kRadixSort>
__global__ __launch_bounds__(kSortBlock) void morton_kernel(
    const vec2_t<T> *__restrict__ Y, int64_t n, const T *__restrict__ part, int nparts, Header *__restrict__ hdr,
    uint64_t *__restrict__ codes, vec2_t<T> *__restrict__ ycopy, const uint32_t *__restrict__ perm,
    uint32_t *__restrict__ hist, uint32_t *__restrict__ levelmask, uint32_t *__restrict__ status, int64_t tiles,
    SampleSort sample)
{
    __shared__ uint32_t sh[kRadixSort ? kSortPasses * kRadix : 1];
    __shared__ uint16_t s_spread[256];
    __shared__ double s_root[3];
    static_assert(kSortBlock == 256, "one spread-table entry per thread");
    s_spread[threadIdx.x] = uint16_t(spread_byte_rule(threadIdx.x));
    if (kRadixSort) {
        clear_tile(sh, status, tiles);
        __syncthreads();
    } else {
        finish_box(part, nparts, hdr, blockIdx.x == 0, s_root);
    }
    const double yr0 = kRadixSort ? hdr->yroot[0] : s_root[0], yr1 = kRadixSort ? hdr->yroot[1] : s_root[1];
    const double sc = kRadixSort ? hdr->scale : s_root[2];
    constexpr int kItems = kRadixSort ? kSortItems : 1;
    const int64_t base = int64_t(blockIdx.x) * kItems * kSortBlock;
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        int64_t i = base + r * kSortBlock + threadIdx.x;
        if (i < n) {
            const vec2_t<T> y = Y[i];
            if (perm) {
                const uint32_t p = perm[i];
                if (p < uint32_t(n)) ycopy[i] = Y[p];
            } else {
                ycopy[i] = y;
            }
            uint64_t code = spread_by_bytes(s_spread, quantise(y.x, yr0, sc)) |
                            (spread_by_bytes(s_spread, quantise(y.y, yr1, sc)) << 1);
            codes[i] = code;
            levelmask[i] = 0;
            if (kRadixSort)
                count_digits(sh, code);
            else if (sample.code)
                take_sample(i, code, n, sample);
        }
    }
    if (kRadixSort) add_digits(sh, hist);
}

// ------------------------------------------------------------------ 3-D box and codes
// A 3-D embedding: the domain is the cube centred on the box with half-side
// r_span (the widest half extent); each coordinate is quantised to 21 bits,
// trunc((y - y_root) * 2^20 / r_span) clamped to [0, 2^21 - 1], in fp64 in
// a fixed order, and bit k of dimension d goes to bit 3k + d of the code
// (63 bits; the top bit stays 0).
__global__ __launch_bounds__(256) void bbox3_partial_kernel(const float3 *__restrict__ Y, int64_t n,
                                                            float *__restrict__ part)
{
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    uint32_t bad = 0;
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) {
        const float3 y = Y[i];
        bad |= !(isfinite(y.x) && isfinite(y.y) && isfinite(y.z));
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            mn[d] = fminf(mn[d], coord(y, d));
            mx[d] = fmaxf(mx[d], coord(y, d));
        }
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        mn[d] = wave_min(mn[d]);
        mx[d] = wave_max(mx[d]);
    }
    const bool anybad = ballot(bad != 0) != 0;
    __shared__ float s[4][6];
    __shared__ uint32_t sb[4];
    const int w = threadIdx.x / kWave;
    if (lane_id() == 0) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            s[w][2 * d] = mn[d];
            s[w][2 * d + 1] = mx[d];
        }
        sb[w] = anybad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float *o = part + 8 * blockIdx.x; // {min x, max x, min y, max y, min z, max z, flag}
        uint32_t b = 0;
        for (int d = 0; d < 3; ++d) {
            float lo = s[0][2 * d], hi = s[0][2 * d + 1];
            for (int k = 1; k < 4; ++k) {
                lo = fminf(lo, s[k][2 * d]);
                hi = fmaxf(hi, s[k][2 * d + 1]);
            }
            o[2 * d] = lo;
            o[2 * d + 1] = hi;
        }
        for (int k = 0; k < 4; ++k) b |= sb[k];
        reinterpret_cast<uint32_t *>(o + 6)[0] = b;
    }
}

// finish_box for a 3-D embedding: s_root = {root of each axis, scale}
__device__ inline void finish_box3(const float *__restrict__ part, int nparts, Header *__restrict__ hdr, bool write,
                                   double *s_root)
{
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    uint32_t bad = 0;
    for (int k = threadIdx.x; k < nparts; k += blockDim.x) {
        const float *p = part + 8 * k;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            mn[d] = fminf(mn[d], p[2 * d]);
            mx[d] = fmaxf(mx[d], p[2 * d + 1]);
        }
        bad |= reinterpret_cast<const uint32_t *>(p + 6)[0];
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        mn[d] = wave_min(mn[d]);
        mx[d] = wave_max(mx[d]);
    }
    const bool anybad = ballot(bad != 0) != 0;
    __shared__ float s[4][6];
    __shared__ uint32_t sb[4];
    const int w = threadIdx.x / kWave;
    if (lane_id() == 0) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            s[w][2 * d] = mn[d];
            s[w][2 * d + 1] = mx[d];
        }
        sb[w] = anybad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t b = 0;
        for (int k = 0; k < 4; ++k) b |= sb[k];
        double c[3], widest = 0.0;
        for (int d = 0; d < 3; ++d) {
            float lo = s[0][2 * d], hi = s[0][2 * d + 1];
            for (int k = 1; k < 4; ++k) {
                lo = fminf(lo, s[k][2 * d]);
                hi = fmaxf(hi, s[k][2 * d + 1]);
            }
            if (write) {
                hdr->bmin[d] = lo;
                hdr->bmax[d] = hi;
            }
            // fp64, fixed operation order: the codes depend on these bits
            c[d] = (double(lo) + double(hi)) * 0.5;
            const double ext = double(hi) - double(lo);
            widest = ext > widest ? ext : widest;
        }
        const double rs = 0.5 * widest;
        for (int d = 0; d < 3; ++d) s_root[d] = c[d] - rs;
        s_root[3] = rs > 0.0 ? 1048576.0 / rs : 0.0;
        if (write) {
            for (int d = 0; d < 3; ++d) {
                hdr->cent[d] = c[d];
                hdr->yroot[d] = s_root[d];
            }
            hdr->rspan = rs;
            hdr->scale = s_root[3];
            reset_call_state(hdr, b);
        }
    }
    __syncthreads();
}

__global__ __launch_bounds__(256) void bbox3_final_kernel(const float *__restrict__ part, int nparts,
                                                          Header *__restrict__ hdr, uint32_t *__restrict__ hist)
{
    __shared__ double s_root[4];
    for (int k = threadIdx.x; k < kHistCopies * kHistWords; k += blockDim.x) hist[k] = 0;
    finish_box3(part, nparts, hdr, true, s_root);
}

__device__ inline uint32_t quantise21(float y, double yroot, double scale)
{
    double q = (double(y) - yroot) * scale;
    if (!(q > 0.0)) return 0u; // also catches NaN
    if (q >= 2097151.0) return 2097151u;
    return uint32_t(q); // truncation toward zero
}

// Three-way spread by the interleaving rule: entry b of the table holds byte
// b with each bit k moved to bit 3k; byte j of a 21-bit coordinate lands at
// bit 24 j of the word.
__device__ inline uint32_t spread3_byte_rule(uint32_t b)
{
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) s |= ((b >> k) & 1u) << (3 * k);
    return s;
}

__device__ inline uint64_t spread3_by_bytes(const uint32_t *__restrict__ tab, uint32_t v)
{
    return uint64_t(tab[v & 0xffu]) | (uint64_t(tab[(v >> 8) & 0xffu]) << 24) | (uint64_t(tab[v >> 16]) << 48);
}

template <bool kRadixSort>
__global__ __launch_bounds__(kSortBlock) void morton3_kernel(
    const float3 *__restrict__ Y, int64_t n, const float *__restrict__ part, int nparts, Header *__restrict__ hdr,
    uint64_t *__restrict__ codes, float3 *__restrict__ ycopy, const uint32_t *__restrict__ perm, uint32_t *__restrict__ hist,
    uint32_t *__restrict__ levelmask, uint32_t *__restrict__ status, int64_t tiles, SampleSort sample)
{
    __shared__ uint32_t sh[kRadixSort ? kSortPasses * kRadix : 1];
    __shared__ uint32_t s_spread[256];
    __shared__ double s_root[4];
    static_assert(kSortBlock == 256, "one spread-table entry per thread");
    s_spread[threadIdx.x] = spread3_byte_rule(threadIdx.x);
    if (kRadixSort) {
        clear_tile(sh, status, tiles);
        __syncthreads();
    } else {
        finish_box3(part, nparts, hdr, blockIdx.x == 0, s_root);
    }
    const double yr0 = kRadixSort ? hdr->yroot[0] : s_root[0], yr1 = kRadixSort ? hdr->yroot[1] : s_root[1];
    const double yr2 = kRadixSort ? hdr->yroot[2] : s_root[2], sc = kRadixSort ? hdr->scale : s_root[3];
    constexpr int kItems = kRadixSort ? kSortItems : 1;
    const int64_t base = int64_t(blockIdx.x) * kItems * kSortBlock;
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const int64_t i = base + r * kSortBlock + threadIdx.x;
        if (i < n) {
            const float3 y = Y[i];
            const uint32_t p = perm ? perm[i] : uint32_t(i); // a layout's order, or the caller's
            ycopy[i] = p == uint32_t(i) ? y : Y[p < uint32_t(n) ? p : uint32_t(i)];
            const uint64_t code = spread3_by_bytes(s_spread, quantise21(y.x, yr0, sc)) |
                                  (spread3_by_bytes(s_spread, quantise21(y.y, yr1, sc)) << 1) |
                                  (spread3_by_bytes(s_spread, quantise21(y.z, yr2, sc)) << 2);
            codes[i] = code;
            levelmask[i] = 0;
            if (kRadixSort)
                count_digits(sh, code);
            else if (sample.code)
                take_sample(i, code, n, sample);
        }
    }
    if (kRadixSort) add_digits(sh, hist);
}

// ------------------------------------------------------------------ onesweep pass
// Block-wide exclusive scan of one value per thread (256 threads).
__device__ inline uint32_t block_exclusive_scan256(uint32_t v, uint32_t *s_wave /*[4]*/,
                                                   uint32_t *total)
{
    int lane = lane_id(), w = threadIdx.x / kWave;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        uint32_t y = __shfl_up(x, o, kWave);
        if (lane >= o) x += y;
    }
    if (lane == kWave - 1) s_wave[w] = x;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint32_t t = s_wave[k];
        off += (k < w) ? t : 0u;
        tot += t;
    }
    if (total) *total = tot;
    return off + x - v;
}

__device__ inline void publish(uint32_t *p, uint32_t word)
{
    __hip_atomic_store(p, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline uint32_t peek(const uint32_t *p)
{
    return __hip_atomic_load(const_cast<uint32_t *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

static_assert(kSortBlock == kRadix, "thread t owns digit t in the scans and the look-back");

// V: the point type gathered by the last pass (float2, double2 or float3)
template <bool kFirst, bool kLast, typename V = float2>
__global__ __launch_bounds__(kSortBlock) void onesweep_kernel(
    const uint64_t *__restrict__ keys_in, const uint32_t *__restrict__ idx_in,
    uint64_t *__restrict__ keys_out, uint32_t *__restrict__ idx_out,
    uint32_t *__restrict__ status, const uint32_t *__restrict__ hist, Header *__restrict__ hdr,
    int pass, int64_t n, const V *__restrict__ ysrc, V *__restrict__ ys)
{
    constexpr int kWaves = kSortBlock / kWave;
    constexpr int kSeg = kWave * kSortItems; // keys per wave segment
    __shared__ uint32_t s_tile;
    __shared__ uint32_t s_wcnt[kWaves][kRadix];
    __shared__ uint32_t s_lstart[kRadix];
    __shared__ uint32_t s_gofs[kRadix];
    __shared__ uint32_t s_scan[4];
    __shared__ uint64_t s_keys[kSortTile];
    __shared__ uint32_t s_idx[kSortTile];

    const int t = threadIdx.x, w = t / kWave, lane = lane_id();
    const int shift = pass * kRadixBits;
    if (t == 0) s_tile = atomicAdd(&hdr->tile_counter[pass], 1u);
    for (int k = t; k < kWaves * kRadix; k += kSortBlock) (&s_wcnt[0][0])[k] = 0;
    __syncthreads();
    const uint32_t tile = s_tile;
    const int64_t base = int64_t(tile) * kSortTile;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));

    uint64_t key[kSortItems];
    uint32_t rank[kSortItems], ixv[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        int64_t p = base + w * kSeg + r * kWave + lane;
        bool valid = p < n;
        key[r] = valid ? keys_in[p] : ~0ull;
        // the payload is loaded with the key, so its latency is not exposed after the look-back
        ixv[r] = kFirst ? uint32_t(p) : (valid ? idx_in[p] : 0u);
        uint32_t d = uint32_t(key[r] >> shift) & (kRadix - 1);
        uint64_t peers = ballot(valid);
#pragma unroll
        for (int b = 0; b < kRadixBits; ++b) {
            bool bit = (d >> b) & 1u;
            uint64_t m = ballot(bit);
            peers &= bit ? m : ~m;
        }
        int leader = peers ? __ffsll((unsigned long long)peers) - 1 : lane;
        uint32_t old = 0;
        if (valid && lane == leader) {
            old = s_wcnt[w][d];
            s_wcnt[w][d] = old + uint32_t(__popcll(peers));
        }
        old = __shfl(old, leader, kWave);
        rank[r] = old + uint32_t(__popcll(peers & lt_mask));
    }
    __syncthreads();

    // thread t owns digit t: per-wave offsets, tile count, look-back
    const uint32_t d = t;
    uint32_t c[kWaves], tot = 0;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        c[k] = s_wcnt[k][d];
        s_wcnt[k][d] = tot;
        tot += c[k];
    }
    uint32_t *my = status + int64_t(tile) * kRadix + d;
    publish(my, (tile == 0 ? kFlagInclusive : kFlagAggregate) | tot);
    uint32_t lstart = block_exclusive_scan256(tot, s_scan, nullptr);
    s_lstart[d] = lstart;
    // global start of digit d: exclusive scan of the histogram
    uint32_t h = 0;
#pragma unroll
    for (int c = 0; c < kHistCopies; ++c) h += hist[c * kHistWords + pass * kRadix + d];
    __syncthreads();
    uint32_t dbase = block_exclusive_scan256(h, s_scan, nullptr);
    uint32_t excl = 0;
    if (tile > 0) {
        // look back kLook predecessors per round trip: add their aggregates
        // until an inclusive prefix; stop at a tile that has not published yet
        // and read again from there
        constexpr int kLook = 8;
        int64_t tt = int64_t(tile) - 1;
        uint32_t spins = 0;
        for (;;) {
            uint32_t sv[kLook];
#pragma unroll
            for (int k = 0; k < kLook; ++k) sv[k] = tt - k >= 0 ? peek(status + (tt - k) * kRadix + d) : 0u;
            int used = 0;
            bool found = false;
#pragma unroll
            for (int k = 0; k < kLook; ++k) {
                if (used != k || tt - k < 0 || (sv[k] & ~kValueMask) == 0) continue; // stopped earlier
                excl += sv[k] & kValueMask;
                used = k + 1;
                if (sv[k] & kFlagInclusive) {
                    found = true;
                    used = kLook + 1; // stop consuming
                }
            }
            if (found) break;
            tt -= used;
            if (tt < 0) break; // cannot happen: tile 0 publishes an inclusive prefix
            if (used < kLook) { // tile tt has not published yet
                if (++spins > kSpinLimit) { // a predecessor never published: give up loudly
                    atomicOr(&hdr->flags, kErrLookback);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        publish(my, kFlagInclusive | (excl + tot));
    }
    s_gofs[d] = dbase + excl;
    __syncthreads();

    // rank -> position inside the tile, staged through LDS
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        int64_t p = base + w * kSeg + r * kWave + lane;
        if (p < n) {
            uint32_t dd = uint32_t(key[r] >> shift) & (kRadix - 1);
            uint32_t lp = s_lstart[dd] + s_wcnt[w][dd] + rank[r];
            s_keys[lp] = key[r];
            s_idx[lp] = ixv[r];
        }
    }
    __syncthreads();
    const int tile_n = int(n - base < kSortTile ? n - base : kSortTile);
    for (int j = t; j < tile_n; j += kSortBlock) {
        uint64_t k = s_keys[j];
        uint32_t dd = uint32_t(k >> shift) & (kRadix - 1);
        uint32_t out = s_gofs[dd] + (uint32_t(j) - s_lstart[dd]);
        if (out < uint32_t(n)) {
            keys_out[out] = k;
            uint32_t ix = s_idx[j];
            idx_out[out] = ix;
            if (kLast) ys[out] = ix < uint32_t(n) ? ysrc[ix] : V{};
        } else {
            atomicOr(&hdr->flags, kErrRange);
        }
    }
}

// ------------------------------------------------------------------ ranks and sample sort
// (code, index) order of two pairs
__device__ inline bool pair_less(uint64_t ca, uint32_t ia, uint64_t cb, uint32_t ib)
{
    return ca < cb || (ca == cb && ia < ib);
}

// The number of pairs before the pair (code, ix) at position own + lane, counted by
// the block's kWaves waves together, valid in wave 0.  own is a multiple of 64; what
// lies below lo is before all 64 pairs, what lies from hi on after all of them.
// idx null: a key's index is its position.  Every wave takes each kWaves-th run of
// 64 keys, as scalar loads (addresses are uniform): three vector instructions a
// comparison, no LDS and no barrier but the one of the sum.
template <int kWaves, bool kIndexed>
__device__ inline uint32_t pairs_before(const uint64_t *__restrict__ codes, const uint32_t *__restrict__ idx, uint32_t n,
                                        uint32_t lo, uint32_t hi, uint32_t own, uint64_t code, uint32_t ix)
{
    __shared__ uint32_t s_count[kWaves][kWave];
    const uint32_t w = uniform(threadIdx.x / kWave), lane = uint32_t(lane_id()), low = uint32_t(code);
    auto index = [&](uint32_t k) { return kIndexed ? idx[k] : k; };
    lo &= ~uint32_t(kWave - 1);
    uint32_t r = 0;
    for (uint32_t k0 = lo + w * kWave; k0 < hi; k0 += kWaves * kWave) {
        if (k0 + kWave > n) {
            for (uint32_t k = k0; k < n; ++k) r += pair_less(codes[k], index(k), code, ix) ? 1u : 0u;
        } else if (k0 == own) {
#pragma unroll 8
            for (int k = 0; k < kWave; ++k) r += pair_less(codes[k0 + k], index(k0 + k), code, ix) ? 1u : 0u;
        } else {
            // equal codes are looked for by their low words and counted apart
            bool tie = false;
#pragma unroll
            for (int k = 0; k < kWave; ++k) {
                const uint64_t c = codes[k0 + k];
                r += c < code ? 1u : 0u;
                tie |= uint32_t(c) == low;
            }
            if (ballot(tie))
                for (int k = 0; k < kWave; ++k) r += codes[k0 + k] == code && index(k0 + k) < ix ? 1u : 0u;
        }
    }
    s_count[w][lane] = r;
    __syncthreads();
    if (w == 0) {
        r += lo;
#pragma unroll
        for (int k = 1; k < kWaves; ++k) r += s_count[k][lane];
    }
    return r;
}

// All pairs in order, each key's place counted among all of them: n^2 comparisons,
// spread over the chip.  2000 points: 8 us, where a bitonic sort in one block's LDS
// took 28 and the eight radix passes 63.
constexpr int kRankWaves = 16;

template <typename V>
__global__ __launch_bounds__(kRankWaves *kWave) void rank_sort_kernel(const uint64_t *__restrict__ codes, int64_t n,
                                                                      uint64_t *__restrict__ keys,
                                                                      uint32_t *__restrict__ idx,
                                                                      const V *__restrict__ ysrc, V *__restrict__ ys)
{
    const uint32_t own = blockIdx.x * kWave, x = own + uint32_t(lane_id());
    const bool live = int64_t(x) < n;
    const uint64_t code = live ? codes[x] : 0;
    const uint32_t r = pairs_before<kRankWaves, false>(codes, nullptr, uint32_t(n), 0, uint32_t(n), own, code, x);
    if (threadIdx.x >= kWave || !live || int64_t(r) >= n) return;
    keys[r] = code;
    idx[r] = x;
    ys[r] = ysrc[x];
}

// Waits until the block's global atomics are done (they take effect where every
// XCD sees them, and the last block reads them back with atomic loads), so that
// the ticket drawn after it counts them; a fence would write back the whole L2.
__device__ inline void adds_done()
{
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
}

// 1. The splitters: every kSamplesPerBucket-th of the sampled keys in order (their
// indices increase with their positions).
__global__ __launch_bounds__(kRankWaves *kWave) void sample_split_kernel(const uint64_t *__restrict__ code, SampleSort s,
                                                                         int64_t n)
{
    const uint32_t own = blockIdx.x * kWave, x = own + uint32_t(lane_id());
    const bool live = int64_t(x) < s.samples;
    const uint64_t c = live ? code[x] : 0;
    const uint32_t r = pairs_before<kRankWaves, false>(code, nullptr, uint32_t(s.samples), 0, uint32_t(s.samples), own, c, x);
    if (threadIdx.x >= kWave || !live) return;
    const uint32_t b = r / kSamplesPerBucket;
    if (r % kSamplesPerBucket == kSamplesPerBucket - 1 && int64_t(b) < s.buckets - 1) {
        s.split[b] = c;
        s.split_idx[b] = uint32_t(sample_position(x, n));
    }
}

// 2. Every key's bucket, the number of splitters at or below it (binary search
// in LDS), and its place in the bucket: a tile counts its keys per bucket in LDS
// and takes its places from the buckets' counters, in any order (the buckets are
// sorted afterwards).  The last block turns the counts into offsets.
constexpr int kBucketBlock = 1024, kBucketItems = 4;
constexpr int kBucketTile = kBucketBlock * kBucketItems;

__global__ __launch_bounds__(kBucketBlock) void sample_bucket_kernel(const uint64_t *__restrict__ codes, int64_t n,
                                                                     SampleSort s, Header *__restrict__ hdr)
{
    extern __shared__ uint64_t s_mem[]; // splitters' keys, their indices, the tile's counts
    const int splits = int(s.buckets) - 1;
    uint64_t *s_code = s_mem;
    uint32_t *s_idx = reinterpret_cast<uint32_t *>(s_code + s.buckets), *s_cnt = s_idx + s.buckets;
    __shared__ bool s_last;
    __shared__ uint32_t s_wave[kBucketBlock / kWave];
    for (int k = threadIdx.x; k < int(s.buckets); k += kBucketBlock) {
        if (k < splits) {
            s_code[k] = s.split[k];
            s_idx[k] = s.split_idx[k];
        }
        s_cnt[k] = 0;
    }
    __syncthreads();
    const int64_t base = int64_t(blockIdx.x) * kBucketTile + threadIdx.x;
    uint64_t key[kBucketItems];
    uint32_t at_or_below[kBucketItems], local[kBucketItems];
#pragma unroll
    for (int q = 0; q < kBucketItems; ++q) {
        const int64_t i = base + q * kBucketBlock;
        key[q] = i < n ? codes[i] : 0;
        at_or_below[q] = 0;
    }
    int top = 1;
    while (2 * top <= splits) top *= 2;
    for (int w = top; w > 0; w >>= 1) {
#pragma unroll
        for (int q = 0; q < kBucketItems; ++q) {
            const int k = int(at_or_below[q]) + w - 1; // the splitter that decides on this step
            if (k < splits && !pair_less(key[q], uint32_t(base + q * kBucketBlock), s_code[k], s_idx[k]))
                at_or_below[q] += uint32_t(w);
        }
    }
#pragma unroll
    for (int q = 0; q < kBucketItems; ++q)
        local[q] = base + q * kBucketBlock < n ? atomicAdd(&s_cnt[at_or_below[q]], 1u) : 0u;
    __syncthreads();
    for (int k = threadIdx.x; k < int(s.buckets); k += kBucketBlock)
        if (s_cnt[k]) s_cnt[k] = atomicAdd(&s.count[k], s_cnt[k]);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kBucketItems; ++q) {
        const int64_t i = base + q * kBucketBlock;
        if (i < n) {
            s.bucket[i] = uint16_t(at_or_below[q]);
            s.pos[i] = s_cnt[at_or_below[q]] + local[q];
        }
    }
    adds_done();
    if (threadIdx.x == 0) s_last = atomicAdd(&hdr->tile_counter[0], 1u) == gridDim.x - 1;
    __syncthreads();
    if (!s_last) return;
    // exclusive scan of the counts, a contiguous run a thread
    const int per = (int(s.buckets) + kBucketBlock - 1) / kBucketBlock, first = int(threadIdx.x) * per;
    uint32_t sum = 0;
    for (int k = first; k < first + per && k < int(s.buckets); ++k) sum += s_cnt[k] = peek(&s.count[k]);
    uint32_t x = sum;
    const int lane = lane_id(), wave = threadIdx.x / kWave;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, kWave);
        if (lane >= o) x += y;
    }
    if (lane == kWave - 1) s_wave[wave] = x;
    __syncthreads();
    uint32_t run = x - sum;
    for (int k = 0; k < wave; ++k) run += s_wave[k];
    for (int k = first; k < first + per && k < int(s.buckets); ++k) {
        s.offset[k] = run;
        run += s_cnt[k];
    }
    if (threadIdx.x == 0) s.offset[s.buckets] = uint32_t(n);
}

// 3. The pairs to their buckets.
__global__ __launch_bounds__(256) void sample_scatter_kernel(const uint64_t *__restrict__ codes, int64_t n,
                                                             SampleSort s, uint64_t *__restrict__ keys_out,
                                                             uint32_t *__restrict__ idx_out)
{
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    const uint32_t o = s.offset[s.bucket[i]] + s.pos[i];
    if (o < uint32_t(n)) {
        keys_out[o] = codes[i];
        idx_out[o] = uint32_t(i);
    }
}

// The bucket that position x lies in: 64 offsets are looked at at a time.
__device__ inline uint32_t bucket_of(const uint32_t *__restrict__ offset, uint32_t buckets, uint32_t x)
{
    uint32_t lo = 0, hi = buckets;
    while (hi - lo > 1) {
        const uint32_t step = (hi - lo + kWave - 1) / kWave, k = lo + uint32_t(lane_id()) * step;
        const uint32_t c = uint32_t(__popcll(ballot(k < hi && offset[k] <= x)));
        lo += (c ? c - 1 : 0) * step;
        hi = lo + step < hi ? lo + step : hi;
    }
    return lo;
}

// 4. The pairs in order: 64 of them a block, each counted among the buckets that
// any of the 64 lies in (what is before those is before all of them): about 400
// comparisons a key, 1.6 times the mean bucket.  No bucket is too large: one that
// held all of the 2^19 points, which the sample's places make unlikely for any
// input, would cost some 40 ms.  70k points: 16 us; the buckets sorted by bitonic
// networks in LDS, a block each, took 53, by runs of 64 merged in LDS 60.
constexpr int kPlaceWaves = 4;

template <typename V>
__global__ __launch_bounds__(kPlaceWaves *kWave) void bucket_sort_kernel(
    const uint64_t *__restrict__ keys_in, const uint32_t *__restrict__ idx_in, const uint32_t *__restrict__ offset,
    uint32_t buckets, int64_t n, uint64_t *__restrict__ keys, uint32_t *__restrict__ idx, const V *__restrict__ ysrc,
    V *__restrict__ ys)
{
    const uint32_t own = blockIdx.x * kWave, x = own + uint32_t(lane_id());
    const bool live = int64_t(x) < n;
    const uint64_t code = live ? keys_in[x] : 0;
    const uint32_t ix = live ? idx_in[x] : 0;
    const uint32_t last = int64_t(own) + kWave <= n ? own + kWave - 1 : uint32_t(n - 1);
    const uint32_t lo = uniform(offset[bucket_of(offset, buckets, own)]);
    const uint32_t hi = uniform(offset[bucket_of(offset, buckets, last) + 1]);
    const uint32_t r = pairs_before<kPlaceWaves, true>(keys_in, idx_in, uint32_t(n), lo, hi, own, code, ix);
    if (threadIdx.x >= kWave || !live || int64_t(r) >= n) return;
    keys[r] = code;
    idx[r] = ix;
    ys[r] = ix < uint32_t(n) ? ysrc[ix] : V{};
}

// ------------------------------------------------------------------ launchers
static SampleSort samples_of(int64_t n, void *ws, const Layout &L)
{
    return sort_mode(n) == SortMode::kSample ? sample_sort(ws, L) : SampleSort{};
}

static int box_parts(int64_t n) { return int(std::min<int64_t>((n + 255) / 256, kBBoxBlocks)); }

// blocks of the kernels that make the codes: the radix sort's tiles, or a point a thread
static unsigned code_blocks(int64_t n, const Layout &L)
{
    return unsigned(sort_mode(n) == SortMode::kRadix ? L.sort_tiles : (n + kSortBlock - 1) / kSortBlock);
}

template <typename T> void launch_bbox(const T *Y, int64_t n, void *ws, const Layout &L, hipStream_t st)
{
    bbox_partial_kernel<T><<<box_parts(n), 256, 0, st>>>(reinterpret_cast<const vec2_t<T> *>(Y), n,
                                                         at<T>(ws, L.bbox_part));
    if (sort_mode(n) == SortMode::kRadix)
        bbox_final_kernel<T><<<1, 256, 0, st>>>(at<T>(ws, L.bbox_part), box_parts(n), at<Header>(ws, L.header),
                                                at<uint32_t>(ws, L.hist));
}
template void launch_bbox<float>(const float *, int64_t, void *, const Layout &, hipStream_t);
template void launch_bbox<double>(const double *, int64_t, void *, const Layout &, hipStream_t);

void launch_bbox_morton3(const float *Y, int64_t n, const uint32_t *perm, void *ws, const Layout &L, hipStream_t st)
{
    const float3 *y3 = reinterpret_cast<const float3 *>(Y);
    bbox3_partial_kernel<<<box_parts(n), 256, 0, st>>>(y3, n, at<float>(ws, L.bbox_part));
    const bool radix = sort_mode(n) == SortMode::kRadix;
    if (radix)
        bbox3_final_kernel<<<1, 256, 0, st>>>(at<float>(ws, L.bbox_part), box_parts(n), at<Header>(ws, L.header),
                                              at<uint32_t>(ws, L.hist));
    auto *kernel = radix ? morton3_kernel<true> : morton3_kernel<false>;
    kernel<<<code_blocks(n, L), kSortBlock, 0, st>>>(
        y3, n, at<float>(ws, L.bbox_part), box_parts(n), at<Header>(ws, L.header), sort_input(ws, L),
        at<float3>(ws, L.ycopy), perm, at<uint32_t>(ws, L.hist), at<uint32_t>(ws, L.levelmask),
        at<uint32_t>(ws, L.status), L.sort_tiles, samples_of(n, ws, L));
}

template <typename T>
void launch_morton(const T *Y, int64_t n, const uint32_t *perm, void *ws, const Layout &L, hipStream_t st)
{
    auto *kernel = sort_mode(n) == SortMode::kRadix ? morton_kernel<T, true> : morton_kernel<T, false>;
    kernel<<<code_blocks(n, L), kSortBlock, 0, st>>>(
        reinterpret_cast<const vec2_t<T> *>(Y), n, at<T>(ws, L.bbox_part), box_parts(n), at<Header>(ws, L.header),
        sort_input(ws, L), at<vec2_t<T>>(ws, L.ycopy), perm, at<uint32_t>(ws, L.hist), at<uint32_t>(ws, L.levelmask),
        at<uint32_t>(ws, L.status), L.sort_tiles, samples_of(n, ws, L));
}
template void launch_morton<float>(const float *, int64_t, const uint32_t *, void *, const Layout &, hipStream_t);
template void launch_morton<double>(const double *, int64_t, const uint32_t *, void *, const Layout &,
                                    hipStream_t);

// the last pass also gathers the points in sorted order (from `ysrc`, in the
// order the codes were made)
template <typename V> void launch_sort_points(int64_t n, const V *ysrc, void *ws, const Layout &L, hipStream_t st)
{
    uint64_t *k[2] = {at<uint64_t>(ws, L.codes0), at<uint64_t>(ws, L.codes1)};
    uint32_t *x[2] = {at<uint32_t>(ws, L.idx0), at<uint32_t>(ws, L.idx1)};
    Header *hdr = at<Header>(ws, L.header);
    const uint32_t *hist = at<uint32_t>(ws, L.hist);
    V *ys = at<V>(ws, L.ys);
    const unsigned groups = unsigned((n + kWave - 1) / kWave);
    if (sort_mode(n) == SortMode::kRank) {
        rank_sort_kernel<V><<<groups, kRankWaves * kWave, 0, st>>>(k[1], n, k[0], x[0], ysrc, ys);
        return;
    }
    if (sort_mode(n) == SortMode::kSample) {
        const SampleSort s = sample_sort(ws, L);
        sample_split_kernel<<<unsigned((s.samples + kWave - 1) / kWave), kRankWaves * kWave, 0, st>>>(s.code, s, n);
        sample_bucket_kernel<<<unsigned((n + kBucketTile - 1) / kBucketTile), kBucketBlock, size_t(s.buckets) * 16,
                               st>>>(k[0], n, s, hdr);
        sample_scatter_kernel<<<unsigned((n + 255) / 256), 256, 0, st>>>(k[0], n, s, k[1], x[1]);
        bucket_sort_kernel<V><<<groups, kPlaceWaves * kWave, 0, st>>>(k[1], x[1], s.offset, uint32_t(s.buckets), n, k[0],
                                                                     x[0], ysrc, ys);
        return;
    }
    for (int p = 0; p < kSortPasses; ++p) {
        uint32_t *status = at<uint32_t>(ws, L.status) + int64_t(p) * L.sort_tiles * kRadix;
        int src = p & 1, dst = src ^ 1;
        dim3 g(unsigned(L.sort_tiles));
        if (p == 0)
            onesweep_kernel<true, false, V><<<g, kSortBlock, 0, st>>>(k[src], nullptr, k[dst], x[dst], status, hist,
                                                                     hdr, p, n, nullptr, nullptr);
        else if (p == kSortPasses - 1)
            onesweep_kernel<false, true, V><<<g, kSortBlock, 0, st>>>(k[src], x[src], k[dst], x[dst], status,
                                                                     hist, hdr, p, n, ysrc, ys);
        else
            onesweep_kernel<false, false, V><<<g, kSortBlock, 0, st>>>(k[src], x[src], k[dst], x[dst], status,
                                                                      hist, hdr, p, n, nullptr, nullptr);
    }
}
template void launch_sort_points<float3>(int64_t, const float3 *, void *, const Layout &, hipStream_t);

template <typename T> void launch_sort(int64_t n, const T *ysrc, void *ws, const Layout &L, hipStream_t st)
{
    launch_sort_points(n, reinterpret_cast<const vec2_t<T> *>(ysrc), ws, L, st);
}
template void launch_sort<float>(int64_t, const float *, void *, const Layout &, hipStream_t);
template void launch_sort<double>(int64_t, const double *, void *, const Layout &, hipStream_t);

} // namespace bht
