// Back projection of ray lists in which many consecutive rays lie on one transaxial line: the transpose of the
// forward's line walk (line.hpp), one ray per lane.
//
// The rays of a line add their samples to an LDS sheet (planes x slices, 32-bit fixed point, as in sheet.hpp: a
// power-of-two scale from the run's bound, rounding remainders carried along the ray), which is then added
// to the line's two image columns per plane.  With a ray per lane a sample takes its two LDS adds and some 15
// instructions (in a sinogram neighbouring rays differ in their slices, so the lanes of a plane mostly meet different
// entries); the run/sheet kernel's half-wave per ray needs as many again to read, bound and place every ray, which
// pays for short runs and for rays of nearly the same slices (back_lines_group).
#pragma once

#include <hip/hip_runtime.h>

#include "line.hpp"
#include "sheet.hpp"

namespace ppmi {

// A sheet's fixed point is as fine as its first run allows (the run's bound between half of kSheetCap and kSheetCap) and
// is coarsened, by at most kLineCoarse bits in all, for later runs of the line that do not fit; a run that still does
// not is preceded by a flush.  Values are left to the direct scatter below kSheetBits + what coarsening may still take:
// the bits that sheet.hpp keeps at least.  The beginning of a line that goes on in the next group is scaled with room
// for that group.  (A first run scaled to 28 bits, without coarsening, gave TOF sinograms with values over three decades
// 2.9e-7 against float64 where k_back_runs gives 1.7e-7; now 1.2 to 1.6e-7.  335 M LORs: 22.9 -> 23.5 ms.)
constexpr int kLineCoarse = 3;

// Every word of the sheet divided by 2^sft and rounded, the remainder carried into the thread's next word (every thread
// of the workgroup; the caller synchronises before and after).  Entries stay within kSheetCap, so 32 bits hold the sums.
__device__ inline void line_coarsen(int* words, int count, int sft) {
    int rem = 0;
    const int half = 1 << (sft - 1);
    auto one = [&](int v) {
        const int t = v + rem, c = (t + half) >> sft;
        rem = t - (c << sft);
        return c;
    };
    int4* const quads = reinterpret_cast<int4*>(words);
    for (int e = threadIdx.x; e < count / 4; e += blockDim.x) {
        int4 v = quads[e];
        v.x = one(v.x), v.y = one(v.y), v.z = one(v.z), v.w = one(v.w);
        quads[e] = v;
    }
    for (int e = count / 4 * 4 + (int)threadIdx.x; e < count; e += blockDim.x) words[e] = one(words[e]);
}

struct LineBackNonTof {
    static constexpr bool kRegular = true;  // the lists it takes (back_lines_group)
    const float* __restrict__ p;
    __device__ bool value(int64_t l, const RayK& r, float& cv, float& bound) const {
        const float pl = p[l];
        cv = r.ell * pl;
        bound = fabsf(cv);
        return pl != 0.0f;
    }
    // f(k, value) for the planes of the rays that are on, called by whole waves; `uniform`: the wave's rays are
    // of one line
    template <class F>
    __device__ __forceinline__ void walk(const RayK& r, int64_t, float cv, bool on, bool, F f) const {
        if (on)
            for (int k = r.k_lo; k <= r.k_hi; ++k) f(k, cv);
    }
};

// One Gaussian for all rays: the value at a sample is ell times the sum of its bins' values with the weights of
// tof_edge_weights.  The bins a wave's rays reach are kept in registers, one window of 2 R + 2 for the wave
// (k_fwd_tof_sino_lines), the next bin's value loaded ahead.
template <int R>
struct LineBackTofSino {
    static constexpr bool kRegular = false;
    const float* __restrict__ p;  // [n][nb]
    TofEdgeK t;
    int nb;
    __device__ bool value(int64_t l, const RayK& r, float& cv, float& bound) const {
        const float* row = p + l * nb;
        float top = 0.0f, nan = 0.0f;
        for (int b = 0; b < nb; ++b) top = fmaxf(top, fabsf(row[b])), nan += row[b] * 0.0f;
        cv = r.ell;
        bound = r.ell * top * (1.0f + 1e-5f) + nan;  // a sample's weights sum to at most 1 (their rounding added)
        return !(bound == 0.0f);
    }
    __device__ float bin(const float* row, int b) const { return (unsigned)b < (unsigned)nb ? row[b] : 0.0f; }
    template <class F>
    __device__ __forceinline__ void walk(const RayK& r, int64_t l, float cv, bool on, bool uniform, F f) const {
        const double B0 = fma(r.s0, t.inv_bw, t.B0), dB = r.ds * t.inv_bw;
        const float* row = p + l * nb;
        float w[2 * R + 1];
        if (uniform) {
            const int k0 = __builtin_amdgcn_readfirstlane(wave_min(on ? r.k_lo : INT_MAX));
            const int k1 = __builtin_amdgcn_readfirstlane(wave_max(on ? r.k_hi : INT_MIN));
            const double Ba = fma((double)k0, dB, B0), Bb = fma((double)k1, dB, B0);
            const int first = __ffsll((long long)__ballot(on)) - 1;
            const double Ba0 = __shfl(Ba, first, 64), Bb0 = __shfl(Bb, first, 64);
            // the window moves one way only: a line's rays in both directions (bitwise the same U0 and dU) walk alone
            const int dir = __builtin_amdgcn_readfirstlane(__shfl(dB, first, 64) > 0.0 ? 1 : -1);
            const bool near = (dB > 0.0) == (dir > 0) && fabs(Ba - Ba0) < 0.49 && fabs(Bb - Bb0) < 0.49 &&
                              fabs(Ba0) < 4096.0 && fabs(Bb0) < 4096.0;
            if (__ballot(on && !near) == 0ull) {
                if (!on) return;
                // cur: the lowest bin a lane lies in (wave-uniform; the others lie in cur or cur + 1)
                int cur = __builtin_amdgcn_readfirstlane((int)rint(Ba0)) - dir;
                float y[2 * R + 2];  // bins cur - R .. cur + R + 1
#pragma unroll
                for (int i = 0; i <= 2 * R + 1; ++i) y[i] = bin(row, cur - R + i);
                float ahead = bin(row, dir > 0 ? cur + R + 2 : cur - R - 1);
                double kd = (double)k0;
                for (int k = k0; k <= k1; ++k, kd += 1.0) {
                    const double B = fma(kd, dB, B0), fb = rint(B);
                    const int q = (int)fb;
                    if (dir > 0) {
                        while (__ballot(q <= cur) == 0ull) {
#pragma unroll
                            for (int i = 0; i <= 2 * R; ++i) y[i] = y[i + 1];
                            y[2 * R + 1] = ahead;
                            ++cur;
                            ahead = bin(row, cur + R + 2);
                        }
                    } else {
                        while (__ballot(q < cur)) {
#pragma unroll
                            for (int i = 2 * R + 1; i > 0; --i) y[i] = y[i - 1];
                            y[0] = ahead;
                            --cur;
                            ahead = bin(row, cur - R - 1);
                        }
                    }
                    tof_edge_weights<R>((float)(B - fb), t, w);
                    float c = 0.0f;
                    if (__ballot(q != cur)) {
                        const bool hi = q != cur;
#pragma unroll
                        for (int i = 0; i <= 2 * R; ++i) c = fmaf(w[i], hi ? y[i + 1] : y[i], c);
                    } else {
#pragma unroll
                        for (int i = 0; i <= 2 * R; ++i) c = fmaf(w[i], y[i], c);
                    }
                    if (k >= r.k_lo && k <= r.k_hi) f(k, c * cv);
                }
                return;
            }
        }
        if (!on) return;
        for (int k = r.k_lo; k <= r.k_hi; ++k) {
            const double B = fma((double)k, dB, B0), fb = rint(B);
            const int q = (int)fmin(fmax(fb, -1e6), 1e6);
            tof_edge_weights<R>((float)(B - fb), t, w);
            float c = 0.0f;
#pragma unroll
            for (int i = 0; i <= 2 * R; ++i) c = fmaf(w[i], bin(row, q - R + i), c);
            f(k, c * cv);
        }
    }
};

constexpr int kLineApart = 24;  // rays of a wave that are scattered one by one; with more of them all at once

__device__ __forceinline__ int lane_value(int x, int j) { return __builtin_amdgcn_readlane(x, j); }
__device__ __forceinline__ double lane_value(double x, int j) {
    const long long b = __double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, j);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), j);
    return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}

// The ray of lane j, for the whole wave
__device__ __forceinline__ RayK ray_of_lane(const RayK& r, int j) {
    RayK o;
    o.U0 = lane_value(r.U0, j), o.dU = lane_value(r.dU, j), o.W0 = lane_value(r.W0, j), o.dW = lane_value(r.dW, j);
    o.s0 = lane_value(r.s0, j), o.ds = lane_value(r.ds, j);
    o.ell = __uint_as_float((unsigned)lane_value((int)__float_as_uint(r.ell), j));
    o.k_lo = lane_value(r.k_lo, j), o.k_hi = lane_value(r.k_hi, j), o.p = lane_value(r.p, j);
    o.sp = lane_value(r.sp, j), o.su = lane_value(r.su, j), o.sw = lane_value(r.sw, j);
    o.nu = lane_value(r.nu, j), o.nw = lane_value(r.nw, j);
    return o;
}

// The groups of kLineBlock rays that back_lines_group takes (the others: k_back_runs)
template <class Mode>
__global__ void __launch_bounds__(kLineBlock, 4) k_back_lines(Mode m, RaySrc src, int64_t n, GeomK g,
                                                              float* __restrict__ img, int groups) {
    constexpr int T = kLineBlock;
    extern __shared__ __attribute__((aligned(16))) int line_sheet[];
    __shared__ LineShared sh;
    __shared__ unsigned left, on;  // groups left to k_back_runs; groups whose last line goes on after them
    __shared__ float part[T / 64];
    typedef __attribute__((address_space(3))) int lds_int;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, zs = line_stride(g), nw = g.n[2];
    const int words = line_words(g);
    int* const sheet = line_sheet + 1;
    LinePlane* const planes = reinterpret_cast<LinePlane*>(line_sheet + words);
    if (tid == 0) left = on = 0;
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * groups * T;
    {
        const int at = tid / kLineLanes;  // groups <= T / kLineLanes
        const int64_t ia = first + (int64_t)at * T;
        const bool some = at < groups && ia < n, take = back_lines_group(src, some ? ia : 0, n, Mode::kRegular);
        if (some && tid % kLineLanes == 0) {
            if (!take) atomicOr(&left, 1u << at);
            if (line_goes_on(src, ia + T, n)) atomicOr(&on, 1u << at);
        }
    }
    __syncthreads();
    const unsigned skip = left, follow = on;
    const int64_t here = (n - first + T - 1) / T;  // groups with rays
    if (__popc(skip) >= (here < groups ? here : groups)) return;
    for (int e = tid; e < words; e += T) line_sheet[e] = 0;
    int cur_p = -1;  // the sheet's line, its scale and the bounds added to it (block-uniform)
    double cur_U = 0.0, cur_d = 0.0;
    float scale = 1.0f, used = 0.0f;
    int coarse = 0;  // bits that the fixed point has been coarsened by
    // the sheet into the image's columns of its line, and cleared (every thread; synchronises before and after)
    auto flush = [&]() {
        const int np = g.n[cur_p], nu = g.n[1 - cur_p], sp = g.stride[cur_p], su = g.stride[1 - cur_p];
        __syncthreads();
        for (int k = tid; k < np; k += T) {
            const double U = fma((double)k, cur_d, cur_U), fi = floor(U);
            const int i0 = (int)fmin(fmax(fi, -2.0), (double)nu);
            const unsigned at = (unsigned)(k * sp + i0 * su);
            planes[k] = {(unsigned)i0 < (unsigned)nu ? at : kLineOutside,
                         (unsigned)(i0 + 1) < (unsigned)nu ? at + (unsigned)su : kLineOutside, (float)(U - fi)};
        }
        __syncthreads();
        const float inv_scale = 1.0f / scale, inv = 1.0f / (float)nw;
        for (int e = tid; e < np * nw; e += T) {  // consecutive threads on consecutive slices
            const int k = (int)(((float)e + 0.5f) * inv), j = e - k * nw;
            int* const at = sheet + k * zs + j + 1;
            const int q = *at;
            if (q == 0) continue;
            *at = 0;
            const float v = (float)q * inv_scale;
            const LinePlane c = planes[k];
            if (c.a != kLineOutside) unsafeAtomicAdd(img + c.a + j, (1.0f - c.fu) * v);
            if (c.b != kLineOutside) unsafeAtomicAdd(img + c.b + j, c.fu * v);
        }
        __syncthreads();
    };
    __syncthreads();
    for (int grp = 0; grp < groups; ++grp) {
        const int64_t i0 = first + (int64_t)grp * T;
        if (i0 >= n) break;  // block-uniform
        if (skip >> grp & 1) continue;
        const int64_t l = i0 + tid;
        RayK r;
        r.p = -1;
        r.U0 = r.dU = 0.0;
        float cv = 0.0f, bound = 0.0f;
        bool todo = l < n && ray_setup(src, l, g, r);
        if (todo) todo = m.value(l, r, cv, bound);
        if (todo) line_trim(r);
        todo = todo && r.k_lo <= r.k_hi;
        bound *= 1.0f + 0x1p-8f;  // margin for the rounding of the bounds
        const int lp = (r.p == 0 || r.p == 1) ? r.p : -1;
        const int runs = line_runs(lp, r.U0, r.dU, sh.heads, sh.last);
        for (int h = 0; h < T;) {  // block-uniform
            const int e = line_next(sh.heads, h);
            // among many runs the short ones between the group's first and last are left to the scatter unseen
            if (runs * kLineHeads > T && h > 0 && e < T && e - h < kLineMinRun) {
                h = e;
                continue;
            }
            const bool mine = todo && tid >= h && tid < e && lp >= 0 && bound <= FLT_MAX;
            float b = mine ? bound : 0.0f;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) b += __shfl_xor(b, off, 64);
            if (lane == 0) part[wave] = b;
            if (tid == h) {
                sh.p = lp;
                sh.line[0] = r.U0;
                sh.line[1] = r.dU;
            }
            __syncthreads();
            const int p = sh.p;
            const double U0 = sh.line[0], dU = sh.line[1];
            float sum = 0.0f;
            for (int w = 0; w < T / 64; ++w) sum += part[w];
            sum *= 1.0f + 0x1p-12f;
            const bool same = p >= 0 && p == cur_p && U0 == cur_U && dU == cur_d;
            // the beginning of a line that goes on in the next group, however short
            const bool goes_on = e == T && (follow >> grp & 1) && grp + 1 < groups && !(skip >> (grp + 1) & 1);
            const bool take = p >= 0 && sum > 0.0f && sum <= 1e37f && (same || goes_on || e - h >= kLineMinRun);
            if (take && same && used + sum * scale > kSheetCap) {
                int sft = 1;
                while (sft <= kLineCoarse && ldexpf(used + sum * scale, -sft) + 1.0f > kSheetCap) ++sft;
                if (coarse + sft <= kLineCoarse && scale >= 0x1p-120f) {
                    line_coarsen(line_sheet, words, sft);
                    __syncthreads();
                    coarse += sft;
                    scale = ldexpf(scale, -sft);
                    used = ldexpf(used, -sft) + 1.0f;  // each entry's rounding adds at most 1/2
                }
            }
            if (take && !(same && used + sum * scale <= kSheetCap)) {
                if (cur_p >= 0) flush();
                cur_p = p, cur_U = U0, cur_d = dU;
                int ex = 0;
                frexpf(sum, &ex);  // sum < 2^ex
                // room for another group of the line
                const int room = !goes_on ? 0 : e - h == T ? 1 : 2 * (e - h) >= T ? 2 : 3;
                scale = ldexpf(1.0f, min(max(31 - room - ex, -126), 126));
                if (sum * scale > kSheetCap) scale *= 0.5f;
                used = 0.0f;
                coarse = 0;
            }
            if (take) {
                used += sum * scale;
                // a ray of far smaller values than the run's is left to the direct scatter
                const bool in = mine && bound * scale >= (float)(1 << (kSheetBits + kLineCoarse - coarse));
                if (__ballot(in)) {
                    const double dZ = r.dW + (double)zs, Z0 = r.W0 + 1.0;
                    float res = 0.0f;
                    m.walk(r, l, cv * scale, in, true, [&](int k, float v) {
                        const double Z = fma((double)k, dZ, Z0);
                        lds_int* const at = (lds_int*)sheet + (int)Z;
                        const float fw = (float)__builtin_amdgcn_fract(Z);
                        // the value with the carried remainder, rounded; the first entry gets its own share rounded, the
                        // second the rest
                        const float tv = v + res, qt = rintf(tv);
                        res = tv - qt;
                        const int q0 = round_half_up(fmaf(-fw, v, v));
                        __hip_atomic_fetch_add(at, q0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        __hip_atomic_fetch_add(at + 1, (int)qt - q0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    });
                    todo = todo && !in;
                }
            }
            h = e;
            __syncthreads();  // before part[] and the line are written again
        }
        // Rays left out of their run's sheet (values of 1e-6 of the run's sum, as at a body's rim): the lanes of the
        // wave take a ray's planes.  With the wave's combined scatter for one such ray the clinical sinogram of a
        // phantom (335 M LORs) took 38.3 ms, with lanes on its planes 19.7 ms, now 21.0 (with TOF 82 and 59.8, now 61.1).
        while (const unsigned long long some = __ballot(todo)) {
            if (__popcll(some) > kLineApart) break;
            const int j = __builtin_amdgcn_readfirstlane(__ffsll((long long)some) - 1);
            const RayK one = ray_of_lane(r, j);
            const float c1 = __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(cv), j));
            for (int k = one.k_lo + lane; k <= one.k_hi; k += 64) {
                RayK at = one;
                at.k_lo = at.k_hi = k;
                float v = 0.0f;
                m.walk(at, i0 + (wave << 6) + j, c1, true, false, [&](int, float x) { v = x; });
                const Stencil st = stencil_at(one, k);
                const float gu = 1.0f - st.fu, gw = 1.0f - st.fw;
                float* const to = img + st.base;
                if (v == 0.0f) continue;
                if (st.i0ok && st.j0ok) unsafeAtomicAdd(to, gu * gw * v);
                if (st.i0ok && st.j1ok) unsafeAtomicAdd(to + one.sw, gu * st.fw * v);
                if (st.i1ok && st.j0ok) unsafeAtomicAdd(to + one.su, st.fu * gw * v);
                if (st.i1ok && st.j1ok) unsafeAtomicAdd(to + one.su + one.sw, st.fu * st.fw * v);
            }
            if (lane == j) todo = false;
        }
        if (__ballot(todo)) {  // float atomics, combined over the wave
            const int dlo = todo ? r.k_lo : INT_MAX, dhi = todo ? r.k_hi : INT_MIN;
            const int k0 = wave_min(dlo), k1 = wave_max(dhi);
            int k = k0;
            float v = 0.0f;
            // the lanes' values plane by plane: every lane walks its planes through one slot of the wave's loop
            for (; k <= k1; ++k) {
                Stencil st{};
                v = 0.0f;
                const bool act = todo && k >= dlo && k <= dhi;
                if (act) st = stencil_at(r, k);
                RayK one = r;
                one.k_lo = one.k_hi = k;
                m.walk(one, l < n ? l : 0, cv, act, false, [&](int, float x) { v = x; });
                wave_stencil_scatter(img, act && v != 0.0f, r, st, v);
            }
        }
    }
    if (cur_p >= 0) flush();
}

}  // namespace ppmi
