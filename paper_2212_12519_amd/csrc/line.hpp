// Forward projection of ray lists in which many consecutive rays lie on one transaxial line (sinograms
// with the ring pairs fastest, densely presorted events).
//
// The rays of a line (bitwise-equal principal axis p in {0, 1}, U0 and dU) meet the image in the same two
// columns per plane, so a workgroup interpolates the columns once, sheet[k][j] = (1 - fu) img[k][i0][j] +
// fu img[k][i0 + 1][j], and keeps this sheet in LDS: a sample is then two neighbouring LDS words instead of
// four global gathers with their index arithmetic and bounds (the rows carry a zero at either end).
// Consecutive groups on one line share the sheet.  Rays of short runs, or along axis 2, gather from the
// image.
#pragma once

#include <hip/hip_runtime.h>

#include "joseph.hpp"

namespace ppmi {

constexpr int kLineMaxBlock = 1024;
constexpr int kLineBlock = 512;  // rays of a group of k_fwd_lines and k_back_lines
// Shortest run that gets a sheet.  TOF forward: one that keeps nearly half a workgroup's waves busy (clinical grid, 157
// rays a line: 0.58 ms with a sheet for every run, 0.28 ms by gathers); where the groups have long runs but at
// their ends (line_group): what the sheet's entries cost
constexpr int kLineMinRun = 96, kLineMinRunTof = 224;
constexpr int kLineHeads = 32;  // forward: a group with more runs than its rays / kLineHeads gathers them all

// What a group of kLineBlock rays looks like at its sixteen points, by their transaxial end points: how many of the fifteen
// stretches between them begin and end on different lines, and how many points lie on the line of the first and of
// the last one without a break.  The stretches' lengths have no common divisor: a list that returns to a line every so
// many rays is not taken for one that stays on it.
constexpr int kLineLanes = 16;

struct LineProbe {
    bool ok;                 // every point's ends are known
    int other, lead, trail;
    float ax, ay, bx, by;    // this lane's point's ends
};

// The points 0 .. 15 of a group: rays 0, 31, 68, 97, 138, 173, 206, 242, 274, 312, 342, 381, 409, 443, 478, 511
__device__ __forceinline__ int line_point(int q) { return 34 * q + (int)(0x6766c7b797870525ull >> (4 * q) & 15) - 5; }

// The bits of b in this lane's group of kLineLanes (called by whole waves)
__device__ __forceinline__ unsigned line_bits(bool b) {
    return (unsigned)(__ballot(b) >> (threadIdx.x & 63 & ~(kLineLanes - 1))) & 0xffffu;
}

// Called by whole waves, kLineLanes neighbouring lanes for a group, all of which get its answer.
__device__ inline LineProbe line_probe(const RaySrc& src, int64_t i0, int64_t n) {
    static_assert(kLineBlock == 512, "the points");
    const int lane = (int)threadIdx.x & 63, group = lane & ~(kLineLanes - 1);
    const float *s, *e;
    const bool ok = src.ends(min(i0 + line_point(lane - group), n - 1), s, e);
    LineProbe p{false, 0, 0, 0, 0.0f, 0.0f, 0.0f, 0.0f};
    if (ok) p.ax = s[0], p.ay = s[1], p.bx = e[0], p.by = e[1];
    auto like = [&](int from) {  // this lane's ray lies on the line of lane `from`'s (every lane shuffles: no short circuit)
        const float sx = __shfl(p.ax, from, 64), sy = __shfl(p.ay, from, 64);
        const float ex = __shfl(p.bx, from, 64), ey = __shfl(p.by, from, 64);
        return sx == p.ax && sy == p.ay && ex == p.bx && ey == p.by;
    };
    p.ok = line_bits(!ok) == 0;
    p.other = __popc(line_bits(!like(min(lane + 1, group + 15))));
    p.lead = __ffs((int)~line_bits(like(group))) - 1;
    p.trail = __clz((int)~(line_bits(like(group + 15)) << 16));
    return p;
}

// Both line kernels take no group with more than some 70 rays in short runs (kLineOther stretches), which they would
// scatter or gather one by one: a line of 340 rays and 22 of 8 in turn took 57 ms where k_back_runs takes 15 ms, one of 400
// and 7 of 16 forward 2.9 ms where gathers take 1.7 ms.
constexpr int kLineOther = 2;

// The rule of k_fwd_lines: the first or the last nine points (nine sixteenths of the group) on one line.  (Much shorter
// runs would be walked one after the other by a few of the waves.)
__device__ inline bool line_group(const RaySrc& src, int64_t i0, int64_t n) {
    const LineProbe p = line_probe(src, i0, n);
    return p.ok && p.other <= kLineOther && (p.lead >= 9 || p.trail >= 9);
}

// The rule of k_back_lines besides:
// - the line of those nine points is longer than kLineLong rays (shorter ones change sheets too often: TOF lines of 480
//   rays 1.9 ms by k_back_runs, 2.2 by lines; of 600 rays 2.5 and 1.8 ms);
// - regular: the rays' mid points move by the same step from ray to ray, as in a sinogram, whose neighbours meet in few
//   entries of the sheet.  Without TOF those meetings bound the kernel (40 M presorted events 11.8 ms by k_back_runs, 18.8
//   by lines; lines of 1200 rays of random slices 1.25 and 1.63 ms); with TOF the lines are the faster all the same
//   (lines of 1200 presorted rays 1.9 and 0.7 ms).
constexpr int kLineRegular = 11, kLineLong = 500;

__device__ inline bool back_lines_group(const RaySrc& src, int64_t i0, int64_t n, bool regular) {
    const LineProbe p = line_probe(src, i0, n);
    const int lane = (int)threadIdx.x & 63, q = lane & (kLineLanes - 1);
    // a ray kLineLong before the last point of the first line, and after the first point of the last one
    const int64_t far = q == 0 ? i0 + line_point(p.lead - 1) - kLineLong : i0 + line_point(kLineLanes - p.trail) + kLineLong;
    const float *s, *e;
    bool on = false;
    if ((q == 0 || q == 15) && far >= 0 && far < n && src.ends(far, s, e))
        on = s[0] == p.ax && s[1] == p.ay && e[0] == p.bx && e[1] == p.by;
    const unsigned out = line_bits(on);
    bool take = p.ok && p.other <= kLineOther && ((p.lead >= 9 && out & 1) || (p.trail >= 9 && out >> 15));
    if (regular) {
        // from this point's ray to the next, or the list's last one's from the one before it
        const int64_t i = min(i0 + line_point(q), n - 1), by = i + 1 < n ? 1 : -1;
        float step = 0.0f;
        if (src.ends(max(i + by, (int64_t)0), s, e)) {
            const float z = s[2] + e[2];
            if (src.ends(i, s, e)) step = (z - (s[2] + e[2])) * (float)by;
        }
        auto steps = [&](int from) {  // how many of the steps are point `from`'s
            const float d = __shfl(step, lane - q + from, 64);
            const int alike = __popc(line_bits(fabsf(step - d) <= 0.02f * fabsf(d)));
            return d != 0.0f ? alike : 0;
        };
        const int a = steps(2), b = steps(9);
        take = take && max(a, b) >= kLineRegular;
    }
    return take;
}

// Whether ray i lies on the line of the one before it, by their transaxial end points
__device__ inline bool line_goes_on(const RaySrc& src, int64_t i, int64_t n) {
    const float *s0, *e0, *s1, *e1;
    if (i >= n || !src.ends(i - 1, s0, e0) || !src.ends(i, s1, e1)) return false;
    return s0[0] == s1[0] && s0[1] == s1[1] && e0[0] == e1[0] && e0[1] == e1[1];
}

// Rows of the sheet: planes 0 .. n_p - 1, nw + 2 entries each (slices -1 .. nw)
__host__ __device__ inline int line_stride(const GeomK& g) { return g.n[2] + 2; }
__host__ __device__ inline int line_planes(const GeomK& g) { return g.n[0] > g.n[1] ? g.n[0] : g.n[1]; }
// Words of a sheet with a guard entry on either side, and of its planes' records (LinePlane)
__host__ __device__ inline int line_words(const GeomK& g) { return line_planes(g) * line_stride(g) + 2; }
__host__ __device__ inline int line_plane_words(const GeomK& g) { return 3 * line_planes(g); }

// Trim the (conservative) plane range to the planes whose stencil has its first voxel in [-1, n): W then
// addresses the sheet's row without further checks.
__device__ __forceinline__ void line_trim(RayK& r) {
    auto out = [&](int k) {
        const int i = (int)floor(fma((double)k, r.dU, r.U0)), j = (int)floor(fma((double)k, r.dW, r.W0));
        return i < -1 || i >= r.nu || j < -1 || j >= r.nw;
    };
    while (r.k_lo <= r.k_hi && out(r.k_lo)) ++r.k_lo;
    while (r.k_lo <= r.k_hi && out(r.k_hi)) --r.k_hi;
}

// The sheet of line (p, U0, dU) over all planes (every thread of the workgroup; zeros where a column lies
// outside the grid).  The planes' column offsets and weights are worked out once; a thread keeps its slice and
// takes every rows-th plane, four planes' loads in flight together: with one at a time the load's latency, not
// the rays' samples, was most of the kernel's time.  *odd: an entry is infinite, a NaN or so large that a difference
// of two may be infinite.
struct LinePlane {
    unsigned a, b;  // byte offsets of the two columns; out of the image's range outside the grid
    float fu;
};
constexpr unsigned kLineOutside = 0xC0000000u;  // beyond every grid whose sheet fits the LDS

__device__ __forceinline__ void line_load(float* sheet, LinePlane* planes, __amdgpu_buffer_rsrc_t ib, const GeomK& g, int p,
                                 double U0, double dU, int* odd) {
    const int np = g.n[p], nu = g.n[1 - p], nw = g.n[2], zs = line_stride(g);
    const int sp = g.stride[p], su = g.stride[1 - p];
    const int T = blockDim.x, lanes = min(nw, T), rows = T / lanes;
    for (int k = threadIdx.x; k < np; k += T) {
        const double U = fma((double)k, dU, U0), fi = floor(U);
        const int i0 = (int)fmin(fmax(fi, -2.0), (double)nu);
        const unsigned at = (unsigned)(k * sp + i0 * su) * 4u;
        planes[k] = {(unsigned)i0 < (unsigned)nu ? at : kLineOutside,
                     (unsigned)(i0 + 1) < (unsigned)nu ? at + (unsigned)su * 4u : kLineOutside, (float)(U - fi)};
    }
    if (threadIdx.x == 0) *odd = 0;
    __syncthreads();
    const int kr = (int)threadIdx.x / lanes;
    constexpr int kBatch = 4;
    if (kr >= rows) return;
    for (int j = (int)threadIdx.x - kr * lanes; j < nw; j += lanes) {
        for (int k0 = kr; k0 < np; k0 += kBatch * rows) {
            float a[kBatch], b[kBatch], fu[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const LinePlane q = planes[min(k0 + u * rows, np - 1)];
                fu[u] = q.fu;
                a[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ib, q.a + 4u * j, 0, 0));
                b[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ib, q.b + 4u * j, 0, 0));
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int k = k0 + u * rows;
                const float v = fmaf(fu[u], b[u], (1.0f - fu[u]) * a[u]);
                if (k < np) sheet[k * zs + j + 1] = v;
                if (!(fabsf(v) <= 1e38f)) *odd = 1;
            }
        }
    }
}

// The samples of a ray through the sheet: f(v, k) with the interpolated value v at plane k, and with Four also
// f4(v) for four planes at once.  Z(k) = W(k) + 1 + k zs is the position in the sheet as one array: its integer
// part addresses the pair of entries (row and slice at once), its remainder is fw.  (Z keeps 38 bits behind the
// point; a rounding across an integer at the grid's faces reads the neighbouring row's zero or the guard entry
// beside the sheet.)
template <bool Four, class F, class F4>
__device__ __forceinline__ void line_walk(const float* sheet, int zs, const RayK& r, F f, F4 f4) {
    const double dZ = r.dW + (double)zs, Z0 = r.W0 + 1.0, d2 = dZ + dZ, d3 = d2 + dZ;
    auto at = [&](double Z) {
        const int i = (int)Z;
        const float a = sheet[i], b = sheet[i + 1];
        const float fw = (float)__builtin_amdgcn_fract(Z);
        return fmaf(fw, b, (1.0f - fw) * a);  // not a + fw (b - a): an infinite voxel stays infinite
    };
    int k = r.k_lo;
    if (Four)
        for (; k + 3 <= r.k_hi; k += 4) {
            const double Z = fma((double)k, dZ, Z0);
            const float v[4] = {at(Z), at(Z + dZ), at(Z + d2), at(Z + d3)};
            f4(v);
        }
    for (; k <= r.k_hi; ++k) f(at(fma((double)k, dZ, Z0)), k);
}

// The runs of a group of blockDim.x consecutive rays, one per thread (line: p in {0, 1} and U0, dU; p < 0: a
// ray on no line).  heads[w]: the positions of wave w where a new run begins.  Returns the number of runs.
// Every thread of the workgroup calls it; it synchronises once before and once after writing.
__device__ inline int line_runs(int p, double U0, double dU, unsigned long long* heads, double* last) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    int pp = __shfl_up(p, 1, 64);
    double pU = __shfl_up(U0, 1, 64), pd = __shfl_up(dU, 1, 64);
    __syncthreads();  // the previous group's readers are done
    if (lane == 63) {
        last[3 * wave] = (double)p;
        last[3 * wave + 1] = U0;
        last[3 * wave + 2] = dU;
    }
    __syncthreads();
    if (lane == 0 && wave > 0) {
        pp = (int)last[3 * wave - 3];
        pU = last[3 * wave - 2];
        pd = last[3 * wave - 1];
    }
    const bool head = threadIdx.x == 0 || p != pp || (p >= 0 && (U0 != pU || dU != pd));
    const unsigned long long b = __ballot(head);
    if (lane == 0) heads[wave] = b;
    __syncthreads();
    int count = 0;
    for (int w = 0; w < waves; ++w) count += __popcll(heads[w]);
    return count;
}

// First position after `at` where a run begins (blockDim.x if none)
__device__ __forceinline__ int line_next(const unsigned long long* heads, int at) {
    const int waves = blockDim.x >> 6;
    int w = (at + 1) >> 6;
    if (w >= waves) return blockDim.x;
    unsigned long long m = heads[w] & (~0ull << ((at + 1) & 63));
    while (m == 0) {
        if (++w >= waves) return blockDim.x;
        m = heads[w];
    }
    return w * 64 + __ffsll((long long)m) - 1;
}

// The workgroup's state in LDS.
struct LineShared {
    unsigned long long heads[kLineMaxBlock / 64];
    double last[3 * (kLineMaxBlock / 64)];
    double line[2];
    int p, odd;
};

// Walks `groups` groups of blockDim.x rays from position `first` on, but those with their bit set in `left`.  setup(i, r) prepares the ray at position i
// (false: it contributes nothing; r.p, r.U0 and r.dU stay valid if it has a line); walk(r, sheet, on), called by
// whole waves, projects this thread's ray if on (sheet nullptr: by gathers; a ray without planes is never on);
// end(i0, count) follows every group.  plane_mem: LDS words for the planes' records, free to use in walk and end.
template <class Setup, class Walk, class End>
__device__ __forceinline__ void line_groups(const GeomK& g, __amdgpu_buffer_rsrc_t ib, float* mem, float* plane_mem, int min_run, int64_t first,
                            int groups, unsigned left, int64_t n, LineShared& sh, Setup setup, Walk walk, End end) {
    const int T = blockDim.x, tid = threadIdx.x, zs = line_stride(g);
    float* const sheet = mem + 1;  // [-1] and the entry past the end: guards
    LinePlane* const planes = reinterpret_cast<LinePlane*>(plane_mem);
    for (int e = tid; e < line_planes(g) * 2; e += T) sheet[(e >> 1) * zs + (e & 1 ? zs - 1 : 0)] = 0.0f;
    if (tid < 2) mem[tid * (line_planes(g) * zs + 1)] = 0.0f;
    int cur_p = -1;  // the sheet's line (block-uniform)
    double cur_U = 0.0, cur_d = 0.0;
    for (int grp = 0; grp < groups; ++grp) {
        const int64_t i0 = first + (int64_t)grp * T;
        if (i0 >= n) break;  // block-uniform
        if (left >> grp & 1) continue;
        RayK r;
        r.p = -1;
        r.U0 = r.dU = 0.0;
        r.k_lo = 0, r.k_hi = -1;
        const bool ok = setup(i0 + tid, r);
        if (ok) line_trim(r);
        else r.k_lo = 0, r.k_hi = -1;
        const int lp = (r.p == 0 || r.p == 1) ? r.p : -1;
        const int runs = line_runs(lp, r.U0, r.dU, sh.heads, sh.last);
        bool done = r.k_lo > r.k_hi;
        if (runs * kLineHeads <= T) {
            for (int h = 0; h < T;) {  // block-uniform
                const int e = line_next(sh.heads, h);
                if (tid == h) {
                    sh.p = lp;
                    sh.line[0] = r.U0;
                    sh.line[1] = r.dU;
                }
                __syncthreads();
                const int p = sh.p;
                const double U0 = sh.line[0], dU = sh.line[1];
                const bool same = p >= 0 && p == cur_p && U0 == cur_U && dU == cur_d;
                if (p >= 0 && !same && e - h >= min_run) {
                    line_load(sheet, planes, ib, g, p, U0, dU, &sh.odd);
                    cur_p = p, cur_U = U0, cur_d = dU;
                }
                __syncthreads();
                const bool on = !done && tid >= h && tid < e && p == cur_p && p >= 0 && U0 == cur_U && dU == cur_d;
                if (__ballot(on)) walk(r, (const float*)sheet, on);
                done |= on;
                h = e;
                if (h < T) __syncthreads();  // before the sheet or the run's line is written again
            }
        }
        if (__ballot(!done)) walk(r, (const float*)nullptr, !done);
        end(i0, (int)(n - i0 < T ? n - i0 : T));
    }
}

}  // namespace ppmi
