// Repulsive (Barnes-Hut) and attractive forces, gradient and update (gfx950).
//
// Repulsive Force Computation: every point walks the tree depth first; a
// cell whose side is small against its distance (side^2 < theta^2 d^2) is
// replaced by its summary, otherwise its children are visited; leaves are
// taken point by point, excluding the point itself.  The normaliser Z (the
// q_ij definition) is the sum of all the kernel values used.
//
// GPU design: points are processed in Morton order, one lane per point, and a
// wavefront walks the pre-order node array together.  The current node index
// is wave-uniform (scalar loads of the 24-byte node record); a lane that
// summarises a cell parks itself until the walk reaches the cell's skip
// index, so its own interaction list is exactly the depth-first one, while the
// wave only descends where some lane needs it.  No stack is needed.
//
// Attractive Force Computation (Algorithm 2): a group of lanes per CSR row,
// coalesced column/value reads, fused with the gradient assembly
// g = 4 (alpha F_attr - F_rep / Z) and the gains/momentum update.
#include "common.hpp"
#include "kernels.hpp"

#include <algorithm>

namespace bht {

__device__ inline float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// Lane masks straight from the vector compares (one instruction each, no
// conversion through a boolean per lane): predicates as in LLVM's icmp/fcmp.
constexpr int kCmpUge = 35, kCmpNe = 33, kCmpOgt = 2;
__device__ inline uint64_t mask_uge(uint32_t a, uint32_t b) { return __builtin_amdgcn_uicmp(a, b, kCmpUge); }
__device__ inline uint64_t mask_ne(uint32_t a, uint32_t b) { return __builtin_amdgcn_uicmp(a, b, kCmpNe); }
__device__ inline uint64_t mask_ogt(float a, float b) { return __builtin_amdgcn_fcmpf(a, b, kCmpOgt); }

// The interaction with one node in the lanes of `take` only: EXEC is narrowed
// to the mask for the block and restored after it, so lanes outside keep their
// sums and resume offsets and no per-lane select is needed.  The instruction
// between the reciprocal and its first use gives the one wait state that a
// transcendental result needs before another VALU reads it on gfx950.
__device__ inline void take_node(uint64_t take, float d2, float dx, float dy, float cnt, uint32_t next, float &z,
                                 float &fx, float &fy, uint32_t &resume)
{
    float w, t;
    uint64_t saved;
    asm volatile("s_and_saveexec_b64 %[sv], %[take]\n\t"
                 "v_add_f32 %[w], 1.0, %[d2]\n\t"
                 "v_rcp_f32 %[w], %[w]\n\t"
                 "v_mov_b32 %[res], %[next]\n\t"
                 "v_mul_f32 %[t], %[cnt], %[w]\n\t"
                 "v_fmac_f32 %[z], %[cnt], %[w]\n\t"
                 "v_mul_f32 %[t], %[t], %[w]\n\t"
                 "v_fmac_f32 %[fx], %[t], %[dx]\n\t"
                 "v_fmac_f32 %[fy], %[t], %[dy]\n\t"
                 "s_mov_b64 exec, %[sv]"
                 : [z] "+v"(z), [fx] "+v"(fx), [fy] "+v"(fy), [res] "+v"(resume), [w] "=&v"(w), [t] "=&v"(t),
                   [sv] "=&s"(saved)
                 : [take] "s"(take), [d2] "v"(d2), [cnt] "s"(cnt), [dx] "v"(dx), [dy] "v"(dy), [next] "s"(next)
                 : "scc");
}

typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));

// 32 bytes at a record: one scalar load
__device__ inline u32x8 load_record(const char *nbase, uint32_t at)
{
    return *reinterpret_cast<const u32x8 *>(nbase + at);
}

// The words of a record that a visit does not read count as read when it
// starts: their registers would be given to other values while the load that
// fills them is in flight, and the wave would wait for it there.  After a loop
// they keep its last load from being moved behind the exit test.
__device__ inline void keep_loaded(const u32x8 &r) { asm volatile("" ::"s"(r[5]), "s"(r[6]), "s"(r[7])); }

// One lane per point.  Every visit runs the same code on a 24-byte record read
// with one scalar load: a single point is a node whose threshold (-1) every
// lane passes, and a bucket of identical points is a cell whose children are
// its points.  The acceptance test gives the lanes that take the node; the
// interaction terms are accumulated in those lanes only, which also park until
// the walk reaches the node's next offset.  The next node is the first child
// when some active lane descends, else the node's next offset.
//
// The lane's own point: with theta^2 <= 0.49 no point accepts a cell that
// contains it (the centre of mass lies in the cell's square, so the squared
// distance is at most 2 side^2, below side^2 / theta^2), so every lane reaches
// its own leaf and takes it once with d2 = 0: a weight of exactly 1 in z and
// nothing in the force, removed after the walk.  Larger theta compares the
// leaf's position with the lane's.
//
// A visit is a chain: the record's scalar load, the compares, the choice of the
// next record.  With kAhead the next record is loaded as soon as it is chosen,
// before the accumulation of the one in hand, which takes as long as the
// compares; two visits a round alternate between two sets of registers, and only
// the second asks for the end, so nothing is moved (with an exit after either the
// sums were, at three vector instructions a visit): the record at `end` is one that
// no lane takes and whose successor lies past it, and the load after that reads at
// most 32 bytes into the array that follows.  (Loading ahead: 3-D 150k points 718 ->
// 622 us, fp64 400k 451 -> 424, 2-D fp32 150k 151 -> 139.  One exit a round: whole
// steps at 70k points 205 -> 195 us.  With 8 waves a SIMD the 2-D fp32 walk is bound
// by issue, and the simple loop, which picks the next record last, serves there.)
//
// The walk goes from `cur` (a byte offset) to `end`.  kPart: `end` may lie before the
// last record; the second visit of a round then takes nothing when it is past it.
template <bool kSelf, bool kAhead, bool kPart = false>
__device__ inline void repulsive_walk(const char *nbase, uint32_t cur, uint32_t end, float2 yi, uint32_t si,
                                      uint32_t &resume, float &fx, float &fy, float &z, uint32_t &inter)
{
    if (cur >= end) return;
    auto visit = [&](const u32x8 &r, u32x8 &after, bool live) {
        if (kAhead) keep_loaded(r);
        const float cx = __uint_as_float(r[0]), cy = __uint_as_float(r[1]);
        const float cnt = __uint_as_float(r[2]), thr = __uint_as_float(r[3]);
        const uint32_t next = r[4];
        const float dx = yi.x - cx, dy = yi.y - cy;
        const float d2 = fmaf(dx, dx, dy * dy);
        const uint64_t act = live ? mask_uge(cur, resume) : 0;
        uint64_t take = act & mask_ogt(d2, thr);
        if (kSelf) take &= mask_ne(r[5], si);
        // the first child follows its cell; no lane descends: jump past the subtree
        if (kAhead) {
            cur = take != act ? cur + kNodeBytes : next;
            after = load_record(nbase, cur);
            __builtin_amdgcn_sched_barrier(0);
        }
        inter += uint32_t(__builtin_popcountll(take));
        take_node(take, d2, dx, dy, cnt, next, z, fx, fy, resume);
        if (!kAhead) cur = take != act ? cur + kNodeBytes : next;
    };
    if (!kAhead) {
        u32x8 none;
        do {
            visit(load_record(nbase, cur), none, true);
        } while (cur < end);
        return;
    }
    u32x8 a = load_record(nbase, cur), b;
    do {
        visit(a, b, true);
        visit(b, a, !kPart || cur < end);
    } while (cur < end);
    keep_loaded(a);
    keep_loaded(b);
}

// The 3-D interaction with one node in the lanes of `take` (see take_node).
__device__ inline void take_node3(uint64_t take, float d2, float dx, float dy, float dz, float cnt, uint32_t next,
                                  float &z, float &fx, float &fy, float &fz, uint32_t &resume)
{
    float w, t;
    uint64_t saved;
    asm volatile("s_and_saveexec_b64 %[sv], %[take]\n\t"
                 "v_add_f32 %[w], 1.0, %[d2]\n\t"
                 "v_rcp_f32 %[w], %[w]\n\t"
                 "v_mov_b32 %[res], %[next]\n\t"
                 "v_mul_f32 %[t], %[cnt], %[w]\n\t"
                 "v_fmac_f32 %[z], %[cnt], %[w]\n\t"
                 "v_mul_f32 %[t], %[t], %[w]\n\t"
                 "v_fmac_f32 %[fx], %[t], %[dx]\n\t"
                 "v_fmac_f32 %[fy], %[t], %[dy]\n\t"
                 "v_fmac_f32 %[fz], %[t], %[dz]\n\t"
                 "s_mov_b64 exec, %[sv]"
                 : [z] "+v"(z), [fx] "+v"(fx), [fy] "+v"(fy), [fz] "+v"(fz), [res] "+v"(resume), [w] "=&v"(w),
                   [t] "=&v"(t), [sv] "=&s"(saved)
                 : [take] "s"(take), [d2] "v"(d2), [cnt] "s"(cnt), [dx] "v"(dx), [dy] "v"(dy), [dz] "v"(dz),
                   [next] "s"(next)
                 : "scc");
}

// The walk over a 3-D embedding's octree: the same visit order and lane
// masks on 32-byte records {com.x, com.y, com.z, count, thr, next, self, 0},
// each exactly one 32-byte scalar load.  With theta^2 <= 0.33 no point
// accepts a cell containing it (the centre of mass lies in the cell's cube,
// so the squared distance is at most 3 side^2, below side^2 / theta^2), and
// the lane's own leaf is taken once with weight 1 as in 2-D.
template <bool kSelf, bool kPart = false>
__device__ inline void repulsive_walk3(const char *nbase, uint32_t cur, uint32_t end, float3 yi, uint32_t si,
                                       uint32_t &resume, float &fx, float &fy, float &fz, float &z, uint32_t &inter)
{
    if (cur >= end) return;
    auto visit = [&](const u32x8 &r, u32x8 &after, bool live) {
        keep_loaded(r);
        const float dx = yi.x - __uint_as_float(r[0]), dy = yi.y - __uint_as_float(r[1]);
        const float dz = yi.z - __uint_as_float(r[2]);
        const float cnt = __uint_as_float(r[3]), thr = __uint_as_float(r[4]);
        const uint32_t next = r[5];
        const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
        const uint64_t act = live ? mask_uge(cur, resume) : 0;
        uint64_t take = act & mask_ogt(d2, thr);
        if (kSelf) take &= mask_ne(r[6], si);
        cur = take != act ? cur + kNodeBytes3 : next;
        after = load_record(nbase, cur);
        __builtin_amdgcn_sched_barrier(0);
        inter += uint32_t(__builtin_popcountll(take));
        take_node3(take, d2, dx, dy, dz, cnt, next, z, fx, fy, fz, resume);
    };
    u32x8 a = load_record(nbase, cur), b;
    do { // (two visits a round, as in 2-D)
        visit(a, b, true);
        visit(b, a, !kPart || cur < end);
    } while (cur < end);
    keep_loaded(a);
    keep_loaded(b);
}

// 1/x in fp64 for x >= 1: the hardware's approximate reciprocal (measured on
// gfx950 within 2^-24.4 relative over x in [1, 1e8]) refined by one
// Newton-Raphson step r <- r + r (1 - x r), which squares the relative error:
// within 2^-48.7 (11 ulps) of the quotient, so a weight and its square carry
// below 5e-15 relative error, and Z, a sum of positive weights, no more (the
// IEEE division sequence costs three times the instructions); 1/inf stays 0.
__device__ inline double recip(double x)
{
    const double r = __builtin_amdgcn_rcp(x);
    return x != __builtin_huge_val() ? fma(r, fma(-x, r, 1.0), r) : 0.0;
}
__device__ inline float recip(float x) { return fast_rcp(x); }

// The fp64 variant of the walk: the same visit order and acceptance test on
// 40-byte records with fp64 centres and thresholds; the lanes that take a
// node accumulate under the compiler's own EXEC mask.
template <bool kSelf>
__device__ inline void repulsive_walk64(const char *nbase, uint32_t cur, uint32_t end, double2 yi, uint32_t si,
                                        uint32_t &resume, double &fx, double &fy, double &z, uint32_t &inter)
{
    struct Rec {
        double cx, cy, thr;
        uint32_t cnt, next, self, pad;
    };
    static_assert(sizeof(Rec) == kNodeBytes64, "the record as it is stored");
    if (cur >= end) return; // cur: byte offset of the current record
    auto load = [&](uint32_t at) { return *reinterpret_cast<const Rec *>(nbase + at); };
    auto visit = [&](const Rec &r, Rec &after) {
        const double cnt = double(__uint_as_float(r.cnt));
        const uint32_t next = r.next;
        const double dx = yi.x - r.cx, dy = yi.y - r.cy;
        const double d2 = fma(dx, dx, dy * dy);
        const bool act = cur >= resume;
        bool tk = act & (d2 > r.thr);
        if (kSelf) tk &= r.self != si;
        const uint64_t take = ballot(tk);
        const uint64_t rej = ballot(act & !tk);
        cur = rej ? cur + kNodeBytes64 : next;
        after = load(cur);
        __builtin_amdgcn_sched_barrier(0);
        inter += uint32_t(__builtin_popcountll(take));
        if (tk) {
            const double wgt = recip(1.0 + d2);
            const double nw = cnt * wgt;
            z += nw;
            const double nw2 = nw * wgt;
            fx = fma(nw2, dx, fx);
            fy = fma(nw2, dy, fy);
            resume = next;
        }
        return cur < end;
    };
    Rec a = load(cur), b = a;
    while (visit(a, b) && visit(b, a)) {
    }
    asm volatile("" ::"s"(a.cx), "s"(b.cx)); // as keep_loaded
}

// a record's centre, threshold and next offset
template <int D, typename T> struct Cell {
    T c[D], thr;
    uint32_t next;
};

template <int D, typename T> __device__ inline Cell<D, T> load_cell(const char *__restrict__ r)
{
    Cell<D, T> x;
    const T *f = reinterpret_cast<const T *>(r);
#pragma unroll
    for (int d = 0; d < D; ++d) x.c[d] = f[d];
    const uint32_t *u = reinterpret_cast<const uint32_t *>(r);
    if constexpr (sizeof(T) == 8) {
        x.thr = f[2];
        x.next = u[7];
    } else {
        x.thr = f[D + 1];
        x.next = u[D + 2];
    }
    return x;
}

// From the root to the first record of the wave's part, over the cells that
// contain it: lanes that accept one of them park until its end (and the wave
// that owns it counts it).  The cells before the part are stepped over, so
// this costs a few records per level.  Returns where the part's walk starts,
// which is past `from` when every lane has parked.  Every step advances.
template <int D, typename T>
__device__ inline uint32_t walk_to(const char *nbase, uint32_t from, const point_t<D, T> &yi, uint32_t &resume)
{
    uint32_t cur = 0;
    while (cur < from) {
        const Cell<D, T> c = load_cell<D, T>(nbase + cur);
        if (c.next <= from) {
            cur = c.next;
            continue;
        }
        const T dx = coord(yi, 0) - c.c[0], dy = coord(yi, 1) - c.c[1];
        T d2;
        if constexpr (D == 3) {
            const T dz = coord(yi, 2) - c.c[2];
            d2 = fma(dx, dx, fma(dy, dy, dz * dz));
        } else {
            d2 = fma(dx, dx, dy * dy);
        }
        const bool act = cur >= resume, take = act && d2 > c.thr;
        resume = take ? c.next : resume;
        cur = ballot(act && !take) ? cur + uint32_t(node_bytes<D, T>()) : c.next;
    }
    return cur;
}

// Bounds of part q of `parts` of the records [0, total) for the points around
// record `mid`.  A group visits about as many records at each doubling of the
// distance from its own place in the array (simulated on early and late
// embeddings of 2k to 1M points: some 100 within its own 64 points, then 50 a
// doubling, nearest first), so the bounds are evenly spaced in log2(1 +
// distance / kPartNear).  Every wave of a group computes the same bounds.
constexpr uint32_t kLine = 128, kTouchLines = 32768;
constexpr float kPartNear = 16.0f;
__device__ inline uint32_t part_bound(uint32_t q, uint32_t parts, uint32_t mid, uint32_t total)
{
    if (q == 0) return 0;
    if (q >= parts) return total;
    const float left = log2f(1.0f + float(mid) / kPartNear), right = log2f(1.0f + float(total - mid) / kPartNear);
    const float t = (left + right) * (float(q) / float(parts));
    const float far = kPartNear * (exp2f(fabsf(left - t)) - 1.0f);
    const uint32_t d = uint32_t(far);
    return t < left ? (d < mid ? mid - d : 0u) : (d < total - mid ? mid + d : total);
}

// ---- fp32 groups shared by several waves
// The waves of a group list what their parts of the records contribute, an entry
// {centre, count; mask of the lanes that take it}, and the group's first wave then
// adds the entries up in the order of the records: the same sums, bit for bit, as
// one wave's walk.  (Partial sums of the parts would round differently, which
// where attraction and repulsion nearly cancel shows in single points a step
// later.)  Listing leaves out the reciprocal and the sums, 10 vector instructions
// a visit instead of 14, and adding up has no chain but the sums.
constexpr int kListRoom = 256; // entries of a wave's list
// Half the widest box whose entries are listed.  In a wider one an entry may be
// infinitely far in fp32 from a lane that does not take it, and counting it 0 times
// would make the lane's sums NaN; the group's first wave walks alone there.
constexpr double kWidest = 1e38;

struct Lists { // in LDS, `waves` lists of kListRoom entries
    float4 *c;
    uint32_t *lo, *hi;
    uint32_t *resume, *cur, *end; // where a part's listing stopped
    int *len;
    static size_t bytes(int waves) { return size_t(waves) * (kListRoom * 24 + kWave * 4 + 12); }
    __device__ Lists(char *m, int waves)
    {
        c = reinterpret_cast<float4 *>(m);
        lo = reinterpret_cast<uint32_t *>(c + waves * kListRoom);
        hi = lo + waves * kListRoom;
        resume = hi + waves * kListRoom;
        cur = resume + waves * kWave;
        end = cur + waves;
        len = reinterpret_cast<int *>(end + waves);
    }
};

// Walks on from `cur` until the part ends or the list holds `room` entries (a multiple
// of 64); returns the list's length.
template <int D, bool kSelf>
__device__ inline int walk_list(const char *nbase, uint32_t &cur, uint32_t end, const point_t<D, float> &yi, uint32_t si,
                                uint32_t &resume, uint32_t &inter, const Lists &l, int first, int room)
{
    constexpr uint32_t kBytes = uint32_t(node_bytes<D, float>());
    uint32_t rec = 0, lo = 0, hi = 0; // the last up to 64 entries, one a lane
    int fill = 0, len = 0;
    auto visit = [&](const u32x8 &r, u32x8 &after) {
        keep_loaded(r);
        asm volatile("" ::"s"(r[D])); // (the count)
        const float dx = coord(yi, 0) - __uint_as_float(r[0]), dy = coord(yi, 1) - __uint_as_float(r[1]);
        float d2;
        if constexpr (D == 3) {
            const float dz = coord(yi, 2) - __uint_as_float(r[2]);
            d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
        } else {
            d2 = fmaf(dx, dx, dy * dy);
        }
        const float thr = __uint_as_float(r[D + 1]);
        const uint32_t next = r[D + 2], at = cur;
        const uint64_t act = mask_uge(cur, resume);
        uint64_t take = act & mask_ogt(d2, thr);
        if (kSelf) take &= mask_ne(r[D + 3], si);
        cur = take != act ? cur + kBytes : next;
        after = load_record(nbase, cur);
        __builtin_amdgcn_sched_barrier(0);
        inter += uint32_t(__builtin_popcountll(take));
        // the lanes that take it park, and lane `fill` keeps the entry (a record that no
        // lane takes is overwritten by the next)
        uint64_t saved;
        asm volatile("s_and_saveexec_b64 %[sv], %[take]\n\t"
                     "v_mov_b32 %[res], %[next]\n\t"
                     "s_lshl_b64 exec, 1, %[fill]\n\t"
                     "v_mov_b32 %[rec], %[at]\n\t"
                     "v_mov_b32 %[lo], %[tlo]\n\t"
                     "v_mov_b32 %[hi], %[thi]\n\t"
                     "s_mov_b64 exec, %[sv]"
                     : [res] "+v"(resume), [sv] "=&s"(saved), [rec] "+v"(rec), [lo] "+v"(lo), [hi] "+v"(hi)
                     : [take] "s"(take), [next] "s"(next), [fill] "s"(fill), [at] "s"(at), [tlo] "s"(uint32_t(take)),
                       [thi] "s"(uint32_t(take >> 32))
                     : "scc");
        fill += take != 0 ? 1 : 0;
        return cur < end && fill < kWave;
    };
    while (cur < end && len + kWave <= room) {
        u32x8 a = load_record(nbase, cur), b = a;
        while (visit(a, b) && visit(b, a)) {
        }
        keep_loaded(a);
        keep_loaded(b);
        asm volatile("" ::"s"(a[D]), "s"(b[D]));
        if (lane_id() < fill) {
            const int to = first + len + lane_id();
            const float *r = reinterpret_cast<const float *>(nbase + rec);
            l.c[to] = make_float4(r[0], r[1], r[2], D == 3 ? r[3] : 0.0f);
            l.lo[to] = lo;
            l.hi[to] = hi;
        }
        len += fill;
        fill = 0;
    }
    return len;
}

// Adds up `len` listed entries in their order.  An entry is read by all lanes at
// once; a lane outside its mask counts it 0 times, which leaves its sums as they
// are.  (The distance must be finite in fp32: see kWidest.)
template <int D>
__device__ inline void add_list(const Lists &l, int first, int len, const point_t<D, float> &yi, float &fx, float &fy,
                                float &fz, float &z)
{
    const float4 *c = l.c + first;
    const uint32_t *mask = (lane_id() < 32 ? l.lo : l.hi) + first;
    const uint32_t bit = lane_id() & 31;
    auto add = [&](const float4 &e, uint32_t m) {
        const float cnt = (m >> bit) & 1u ? (D == 3 ? e.w : e.z) : 0.0f;
        const float dx = coord(yi, 0) - e.x, dy = coord(yi, 1) - e.y;
        float dz = 0.0f, d2;
        if constexpr (D == 3) {
            dz = coord(yi, 2) - e.z;
            d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
        } else {
            d2 = fmaf(dx, dx, dy * dy);
        }
        const float w = fast_rcp(1.0f + d2);
        float t = cnt * w;
        z = fmaf(cnt, w, z);
        t = t * w;
        fx = fmaf(t, dx, fx);
        fy = fmaf(t, dy, fy);
        if constexpr (D == 3) fz = fmaf(t, dz, fz);
    };
    constexpr int kAtOnce = 8;
    int k = 0;
    for (; k + kAtOnce <= len; k += kAtOnce) {
        float4 e[kAtOnce];
        uint32_t m[kAtOnce];
#pragma unroll
        for (int q = 0; q < kAtOnce; ++q) {
            e[q] = c[k + q];
            m[q] = mask[k + q];
        }
#pragma unroll
        for (int q = 0; q < kAtOnce; ++q) add(e[q], m[q]);
    }
    for (; k < len; ++k) add(c[k], mask[k]);
}

// The walk of a block's waves, which share one group of points: every wave lists its
// part until it ends or its list is full, then the first adds the lists up in order,
// and walks what is left of a part itself, from where its listing stopped.  (Before,
// lists were filled and added up in turns until every part ended, one of the two
// waiting for the other, which long runs of taken records showed.  Walk in us, one wave
// a group by the simple loop / in turns / now: 30k points, 27k of them in three places,
// 1380 / 1622 / 1182; 20k in one place 2973 / 3508 / 2578; 30k at theta 0.05 2473 / 2367
// / 1659; 3-D 8192 at theta 0.2 1057 / 906 / 636.)
template <int D, bool kSelf>
__device__ inline void walk_shared(const char *nbase, uint32_t cur, uint32_t end, const point_t<D, float> &yi,
                                   uint32_t si, int me, int parts, int room, uint32_t &resume, float &fx, float &fy,
                                   float &fz, float &z, uint32_t &inter, const Lists &l)
{
    const int len = walk_list<D, kSelf>(nbase, cur, end, yi, si, resume, inter, l, me * kListRoom, room);
    l.resume[me * kWave + lane_id()] = resume;
    if (lane_id() == 0) {
        l.len[me] = len;
        l.cur[me] = cur;
        l.end[me] = end;
    }
    __syncthreads();
    if (me != 0) return;
    for (int p = 0; p < parts; ++p) {
        add_list<D>(l, p * kListRoom, int(uniform(uint32_t(l.len[p]))), yi, fx, fy, fz, z);
        cur = uniform(l.cur[p]);
        end = uniform(l.end[p]);
        if (cur >= end) continue;
        resume = l.resume[p * kWave + lane_id()];
        if constexpr (D == 3)
            repulsive_walk3<kSelf, true>(nbase, cur, end, yi, si, resume, fx, fy, fz, z, inter);
        else
            repulsive_walk<kSelf, true, true>(nbase, cur, end, yi, si, resume, fx, fy, z, inter);
    }
}

// D = 2, T = float: the path (24-byte records); T = double: the fp64
// variant; D = 3: 3-D embeddings (32-byte records).  kForm: one wave walks for a
// group of 64 points, by the simple loop (2-D fp32, blocks of kRepBlock) or loading
// ahead, or 2^log_waves waves of a block share the group, each walking a part of
// the records (in fp32 all waves of the block).  Each is a kernel of its own: with
// the simple and the load-ahead loop in one kernel, which chose at run time, the
// simple one's walk took 0.5 to 0.8% longer (700k points 382.2 us, now 378.8; 1M at
// theta 0.2 1397.7, now 1389.0).
enum WalkForm { kSimple, kAhead, kShared };

template <int D, typename T, int kForm>
__global__ __launch_bounds__(kRepBlock) void repulsive_kernel(
    const char *__restrict__ nodes, const point_t<D, T> *__restrict__ ys, const uint32_t *__restrict__ perm,
    const uint32_t *__restrict__ base, Header *__restrict__ hdr, int64_t n, int self_test, int log_waves,
    point_t<D, T> *__restrict__ frep, double *__restrict__ zpart, unsigned long long *__restrict__ ipart)
{
    constexpr bool kSplit = kForm == kShared;
    using V = point_t<D, T>;
    const uint32_t nb = gridDim.x;
    const uint32_t lb = xcd_contiguous(blockIdx.x, nb);
    const int w = threadIdx.x / kWave;
    const uint32_t threads = kForm == kSimple ? kRepBlock : blockDim.x; // at most kRepBlock
    const int waves = int(threads) / kWave;
    uint32_t me = 0; // this wave's number among those of its group
    int64_t s64 = int64_t(lb) * threads + threadIdx.x;
    if (kSplit) {
        me = uniform(uint32_t(w)) & ((1u << log_waves) - 1u);
        s64 = int64_t(lb) * (threads >> log_waves) + int64_t(w >> log_waves) * kWave + lane_id();
    }
    const bool valid = s64 < n;
    const uint32_t si = uint32_t(s64);
    const V yi = valid ? ys[s64] : V{};
    uint32_t resume = valid ? 0u : 0xffffffffu;
    T fx = 0, fy = 0, fz = 0, z = 0;
    uint32_t total = uniform(hdr->nodes);
    const uint32_t cap = uint32_t(2 * n);
    total = total < cap ? total : cap;
    // Every record's next offset lies past the record (the tree kernel checks
    // it and flags the call otherwise), so each visit advances and the walk
    // ends after at most `total` visits.  A flagged tree is not walked.
    if (uniform(hdr->flags) & (kErrLookback | kErrRange)) total = 0;
    const uint32_t all = total * uint32_t(node_bytes<D, T>());
    uint32_t cur = 0, end = all;
    [[maybe_unused]] uint32_t touched = 0;
    if constexpr (kSplit) {
        // The records were written through other XCDs' caches.  Where they fit
        // this XCD's (4 MB) its blocks fetch them together, one load a line,
        // before the waves miss them one by one (2k points 42 -> 34 us).
        const uint32_t lines = (end + kLine - 1) / kLine, stride = (nb >> 3) * threads;
        if (lines <= kTouchLines)
            for (uint32_t q = (blockIdx.x >> 3) * threads + threadIdx.x; q < lines; q += stride)
                touched ^= *reinterpret_cast<const uint32_t *>(nodes + size_t(q) * kLine);
        const int64_t first = s64 - lane_id();
        if (first < n && total) {
            // record of the group's middle point, at most `total`
            uint32_t mid = uniform(base[first + kWave / 2 < n ? first + kWave / 2 : first]);
            mid = mid < total ? mid : total;
            const uint32_t from = uniform(part_bound(me, 1u << log_waves, mid, total));
            const uint32_t to = uniform(part_bound(me + 1, 1u << log_waves, mid, total));
            end = to * uint32_t(node_bytes<D, T>());
            cur = from < to ? walk_to<D, T>(nodes, from * uint32_t(node_bytes<D, T>()), yi, resume) : end;
        } else {
            end = 0;
        }
        cur = uniform(cur);
        end = uniform(end);
    }

    uint32_t inter = 0; // this wave's interactions (a launch has fewer than 2^32 per wave)
    if constexpr (kSplit && sizeof(T) == 4) {
        extern __shared__ float4 s_lists[];
        const Lists lists(reinterpret_cast<char *>(s_lists), waves); // one group a block: me is the wave's number
        int room = kListRoom;
        if (uniform(hdr->rspan < kWidest ? 0u : 1u)) { // the first wave takes all records
            room = 0;
            cur = 0;
            end = me == 0 ? all : 0;
        }
        if (self_test)
            walk_shared<D, true>(nodes, cur, end, yi, si, int(me), waves, room, resume, fx, fy, fz, z, inter, lists);
        else
            walk_shared<D, false>(nodes, cur, end, yi, si, int(me), waves, room, resume, fx, fy, fz, z, inter, lists);
    } else if constexpr (D == 3) {
        if (self_test)
            repulsive_walk3<true>(nodes, cur, end, yi, si, resume, fx, fy, fz, z, inter);
        else
            repulsive_walk3<false>(nodes, cur, end, yi, si, resume, fx, fy, fz, z, inter);
    } else if constexpr (sizeof(T) == 8) {
        if (self_test)
            repulsive_walk64<true>(nodes, cur, end, yi, si, resume, fx, fy, z, inter);
        else
            repulsive_walk64<false>(nodes, cur, end, yi, si, resume, fx, fy, z, inter);
    } else {
        if (self_test)
            repulsive_walk<true, kForm == kAhead>(nodes, cur, end, yi, si, resume, fx, fy, z, inter);
        else
            repulsive_walk<false, kForm == kAhead>(nodes, cur, end, yi, si, resume, fx, fy, z, inter);
    }
    if constexpr (kSplit) asm volatile("" ::"v"(touched)); // the loads above are wanted, not their values
    bool lead = true; // this wave finishes its group's points
    if constexpr (kSplit) {
        lead = me == 0;
        if constexpr (sizeof(T) == 8) {
            // the group's sums, added in the order of its waves by the first of them
            // (in fp64 another rounding of the sums shows nowhere)
            __shared__ T s_part[3][kRepBlock];
            s_part[0][threadIdx.x] = fx;
            s_part[1][threadIdx.x] = fy;
            s_part[2][threadIdx.x] = z;
            __syncthreads();
            if (lead) {
                for (uint32_t q = 1; q < 1u << log_waves; ++q) {
                    const int at = int(threadIdx.x + q * kWave);
                    fx += s_part[0][at];
                    fy += s_part[1][at];
                    z += s_part[2][at];
                }
            }
        }
    }
    if (!self_test && lead) {
        // each valid lane took its own leaf once, with weight 1
        if (valid) z -= T(1);
        inter -= uint32_t(__builtin_popcountll(ballot(valid))); // (the group's total is not negative)
    }

    if (valid && lead) {
        const uint32_t p = perm[si];
        const T f[3] = {fx, fy, fz};
        if (p < uint32_t(n)) frep[p] = make_point(f, static_cast<V *>(nullptr));
    }
    // deterministic Z: wave -> block partial -> fixed-order sum in the last block
    double zw = wave_sum(lead ? double(z) : 0.0);
    __shared__ double s_z[kRepBlock / kWave];
    __shared__ unsigned long long s_i[kRepBlock / kWave];
    __shared__ bool s_last;
    if (lane_id() == 0) {
        s_z[w] = zw;
        s_i[w] = static_cast<unsigned long long>(int64_t(int32_t(inter))); // split: the lead's own may be below 0
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double zb = 0.0;
        unsigned long long ib = 0;
        for (int k = 0; k < waves; ++k) {
            zb += s_z[k];
            ib += s_i[k];
        }
        zpart[lb] = zb;
        ipart[lb] = ib;
        __threadfence();
        s_last = atomicAdd(&hdr->ticket_rep, 1u) == nb - 1;
    }
    __syncthreads();
    if (!s_last) return;
    __threadfence();
    // last block: each thread sums a fixed contiguous chunk, then a fixed tree
    const uint32_t per = (nb + threads - 1) / threads;
    double zs = 0.0;
    unsigned long long is = 0;
    for (uint32_t k = threadIdx.x * per; k < (threadIdx.x + 1) * per && k < nb; ++k) {
        zs += zpart[k];
        is += ipart[k];
    }
    zs = wave_sum(zs);
    is = wave_sum(is);
    __syncthreads();
    if (lane_id() == 0) {
        s_z[w] = zs;
        s_i[w] = is;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double Z = 0.0;
        unsigned long long I = 0;
        for (int k = 0; k < waves; ++k) {
            Z += s_z[k];
            I += s_i[k];
        }
        hdr->Z = Z;
        hdr->interactions = I;
    }
}


constexpr int kAttB = 4;

// D = 2, T = float: the path's plain-CSR attraction; T = double: the fp64
// variant; D = 3: 3-D embeddings.  Coordinates are handled component by
// component (unrolled).
template <int G, bool kUpdate, int D, typename T>
__global__ __launch_bounds__(256) void attract_kernel(
    const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col, const T *__restrict__ val,
    const point_t<D, T> *__restrict__ ycopy, const point_t<D, T> *__restrict__ frep, Header *__restrict__ hdr,
    int64_t n, int64_t nnz, StepArgsT<T> a, point_t<D, T> *__restrict__ Y, point_t<D, T> *__restrict__ upd,
    point_t<D, T> *__restrict__ gains, point_t<D, T> *__restrict__ grad)
{
    using V = point_t<D, T>;
    const int sub = lane_id() % G;
    constexpr int kRows = 256 / G;
    const T inv_z = T(1.0 / hdr->Z);
    for (int64_t row0 = int64_t(blockIdx.x) * kRows; row0 < n; row0 += int64_t(gridDim.x) * kRows) {
        const int64_t i = row0 + threadIdx.x / G;
        const bool valid = i < n;
        T f[D];
#pragma unroll
        for (int d = 0; d < D; ++d) f[d] = T(0);
        V yi{};
        if (valid) {
            yi = ycopy[i];
            int64_t s = row_ptr[i], e = row_ptr[i + 1];
            if (s < 0 || e > nnz) { // malformed row: skip what lies outside the arrays
                if (sub == 0) atomicOr(&hdr->flags, kErrRange);
                s = s < 0 ? 0 : s;
                e = e > nnz ? nnz : e;
            }
            // kAttB entries per lane at a time: their loads, then their gathers,
            // are in flight together
            for (int64_t k0 = s + sub; k0 < e; k0 += kAttB * G) {
                int32_t j[kAttB];
                T p[kAttB];
#pragma unroll
                for (int u = 0; u < kAttB; ++u) {
                    const int64_t k = k0 + u * G;
                    // P is streamed once per call: keep it out of the caches that hold Y
                    j[u] = k < e ? __builtin_nontemporal_load(col + k) : 0;
                    p[u] = k < e ? __builtin_nontemporal_load(val + k) : T(0);
                    if (uint32_t(j[u]) >= uint32_t(n)) {
                        atomicOr(&hdr->flags, kErrRange);
                        j[u] = 0;
                        p[u] = T(0);
                    }
                }
                V yj[kAttB];
#pragma unroll
                for (int u = 0; u < kAttB; ++u) yj[u] = ycopy[j[u]];
#pragma unroll
                for (int u = 0; u < kAttB; ++u) {
                    T dv[D];
#pragma unroll
                    for (int d = 0; d < D; ++d) dv[d] = coord(yi, d) - coord(yj[u], d);
                    T d2 = dv[D - 1] * dv[D - 1];
#pragma unroll
                    for (int d = D - 2; d >= 0; --d) d2 = fma(dv[d], dv[d], d2);
                    const T pw = p[u] * recip(T(1) + d2);
#pragma unroll
                    for (int d = 0; d < D; ++d) f[d] = fma(pw, dv[d], f[d]);
                }
            }
        }
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) {
#pragma unroll
            for (int d = 0; d < D; ++d) f[d] += __shfl_xor(f[d], o, kWave);
        }
        if (valid && sub == 0) {
            const V fr = frep[i];
            T g[D];
#pragma unroll
            for (int d = 0; d < D; ++d) g[d] = T(4) * (a.alpha * f[d] - coord(fr, d) * inv_z);
            if (grad) grad[i] = make_point(g, static_cast<V *>(nullptr));
            if (kUpdate) {
                const V u0 = upd[i], g0 = gains[i];
                T u[D], gn[D], y[D];
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    const T ud = coord(u0, d);
                    T gd = (ud * g[d] < T(0)) ? coord(g0, d) + T(0.2) : coord(g0, d) * T(0.8);
                    gd = vmax(gd, a.min_gain);
                    u[d] = a.momentum * ud - a.learning_rate * gd * g[d];
                    gn[d] = gd;
                    y[d] = coord(yi, d) + u[d];
                }
                Y[i] = make_point(y, static_cast<V *>(nullptr));
                upd[i] = make_point(u, static_cast<V *>(nullptr));
                gains[i] = make_point(gn, static_cast<V *>(nullptr));
            }
        }
    }
}

// ------------------------------------------------------------------ launchers
// How a walk is launched: its form, log2 of the waves that share a group of 64
// points, and the threads of a block.
//
// A walk is a chain of dependent record loads (some 300 ns a record alone on a
// SIMD, 500 to 900 records a group), so few groups leave the chip waiting, and
// several waves share one: in fp64 4, 8 or 16 as long as all are resident at
// once (about 4096), and 2 up to a point where the launch is bound by issue and
// the scalar cache, which waves in different places of the tree share less
// well.  In fp32 the listed entries are added up by one wave of a group, so
// sharing pays only where the walks themselves are many times longer than that.
// Blocks of consecutive points share records through the scalar cache, 1024
// points best where every CU has several blocks; smaller ones reach more CUs and
// end sooner.  Walk in us, gfx950, theta 0.5, in brackets one wave a group by the
// simple loop in blocks of 1024 threads:
//   fp32  8 waves a group: 2k points (94) 52, 10k (115) 65, 30k (112) 82;
//         1 wave, ahead, 256 threads: 2k 81, 10k 98, 30k 89, 70k (165) 134, 150k (151)
//         141, 300k (226) 200, 500k 256; 1024 threads, simple: 500k 235, 1M 447
//   fp64  5k (203) 41 with 16 waves, 50k (237) 79 with 4, 200k (281) 198 with 2, 400k
//         (451) 374 with 2; 600k 503 with 1 and 512 threads, 562 with 1024
//   3-D   5k (328) 168 with 16 waves, 225 with 1; 20k 203 against 208; 1 wave, 256
//         threads: 50k (397) 299, 150k (718) 539, 300k (930) 664, 800k (1717) 1380 early
//         and (1371) 1119 late in a run, 1.3M (2503) 2049
struct WalkLaunch {
    WalkForm form;
    int log_waves, threads;
};

// (fp32: kWave << log_waves threads a block that shares, one group)
template <int D, typename T> static WalkLaunch walk_launch(int64_t n)
{
    const int64_t groups = (n + kWave - 1) / kWave;
    if (D == 3) return groups <= 128 ? WalkLaunch{kShared, 4, 1024} : WalkLaunch{kAhead, 0, 256};
    if (sizeof(T) == 8) {
        for (int lw = 4; lw > 1; --lw)
            if (groups << lw <= 4096) return {kShared, lw, std::max(512, kWave << lw)};
        return groups <= 8192 ? WalkLaunch{kShared, 1, 512} : WalkLaunch{kAhead, 0, 512};
    }
    if (groups <= 480) return {kShared, 3, 512};
    if (groups <= 6400) return {kAhead, 0, 256};
    return {kSimple, 0, kRepBlock};
}

template <int D, typename T>
void launch_repulsive(int64_t n, bool self_test, void *ws, const Layout &L, hipStream_t st, int form)
{
    using V = point_t<D, T>;
    WalkLaunch c = walk_launch<D, T>(n);
    if (form >= 0) c = form == kSimple ? WalkLaunch{kSimple, 0, kRepBlock} : WalkLaunch{kAhead, 0, 256};
    const int64_t per = c.threads >> c.log_waves;
    const int64_t blocks = ((n + per - 1) / per + 7) / 8 * 8; // a multiple of 8 for the XCD-contiguous remap
    // the blocks' partials go to the sort's second key array, free by now: 16
    // bytes for at least 64 points, in 8 bytes a point (and 256 at the least)
    double *zpart = at<double>(ws, L.codes1);
    auto *kernel = c.form == kShared ? repulsive_kernel<D, T, kShared> : repulsive_kernel<D, T, kAhead>;
    if constexpr (D == 2 && sizeof(T) == 4)
        if (c.form == kSimple) kernel = repulsive_kernel<D, T, kSimple>;
    const size_t lds = c.form == kShared && sizeof(T) == 4 ? Lists::bytes(c.threads / kWave) : 0;
    kernel<<<unsigned(blocks), unsigned(c.threads), lds, st>>>(
        at<char>(ws, L.nodes), at<V>(ws, L.ys), at<uint32_t>(ws, L.idx0), at<uint32_t>(ws, L.base),
        at<Header>(ws, L.header), n, self_test ? 1 : 0, c.log_waves, at<V>(ws, L.frep), zpart,
        reinterpret_cast<unsigned long long *>(zpart + blocks));
}
template void launch_repulsive<2, float>(int64_t, bool, void *, const Layout &, hipStream_t, int);
template void launch_repulsive<2, double>(int64_t, bool, void *, const Layout &, hipStream_t, int);
template void launch_repulsive<3, float>(int64_t, bool, void *, const Layout &, hipStream_t, int);

template <int D, typename T>
void launch_attract(const int64_t *row_ptr, const int32_t *col, const T *val, int64_t n, int64_t nnz,
                    const StepArgsT<T> &a, T *Y, T *upd, T *gains, T *grad, void *ws, const Layout &L, hipStream_t st)
{
    constexpr int G = 64; // one wave per row: rows hold ~100-200 entries
    int64_t blocks = (n + (256 / G) - 1) / (256 / G);
    if (blocks > 65535 * 8) blocks = 65535 * 8;
    using V = point_t<D, T>;
    const V *yc = at<V>(ws, L.ycopy);
    const V *fr = at<V>(ws, L.frep);
    Header *hdr = at<Header>(ws, L.header);
    if (a.update)
        attract_kernel<G, true, D, T><<<unsigned(blocks), 256, 0, st>>>(
            row_ptr, col, val, yc, fr, hdr, n, nnz, a, reinterpret_cast<V *>(Y), reinterpret_cast<V *>(upd),
            reinterpret_cast<V *>(gains), reinterpret_cast<V *>(grad));
    else
        attract_kernel<G, false, D, T><<<unsigned(blocks), 256, 0, st>>>(row_ptr, col, val, yc, fr, hdr, n, nnz, a,
                                                                       nullptr, nullptr, nullptr,
                                                                       reinterpret_cast<V *>(grad));
}
template void launch_attract<2, float>(const int64_t *, const int32_t *, const float *, int64_t, int64_t,
                                       const StepArgsT<float> &, float *, float *, float *, float *, void *,
                                       const Layout &, hipStream_t);
template void launch_attract<2, double>(const int64_t *, const int32_t *, const double *, int64_t, int64_t,
                                        const StepArgsT<double> &, double *, double *, double *, double *, void *,
                                        const Layout &, hipStream_t);
template void launch_attract<3, float>(const int64_t *, const int32_t *, const float *, int64_t, int64_t,
                                       const StepArgsT<float> &, float *, float *, float *, float *, void *,
                                       const Layout &, hipStream_t);

} // namespace bht
