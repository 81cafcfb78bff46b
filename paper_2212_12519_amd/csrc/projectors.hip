// Joseph forward / back projection kernels for gfx950 (non-TOF, TOF sinogram,
// TOF listmode).  One thread per ray; 256-thread workgroups (4 wave64s) in
// plain workgroup order.  See joseph.hpp for the traversal itself.
#include <hip/hip_runtime.h>

#include "joseph.hpp"
#include "back_lines.hpp"
#include "launch.hpp"
#include "line.hpp"
#include "sheet.hpp"

namespace ppmi {

constexpr int kBlock = 256;
constexpr int kParts = 4;  // lanes that share a ray where rays are few (split_rays)
constexpr int kSinoBlock = 512;  // k_fwd_tof_sino_lines, at most

// ------------------------------------------------------------- non-TOF ----

// Ray processed by this thread: position i of the processing order (identity,
// or a permutation such as the one pp_lm_presort produces).  Entries outside
// [0, n) are skipped.
template <int Parts = 1>
__device__ __forceinline__ int64_t ray_index(const int32_t* __restrict__ order, int64_t n) {
    const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / Parts;
    if (i >= n) return -1;
    if (!order) return i;
    const int64_t l = order[i];
    return (l >= 0 && l < n) ? l : -1;
}

// The sum of the Parts neighbouring lanes that share a ray
template <int Parts>
__device__ __forceinline__ float sum_parts(float v) {
#pragma unroll
    for (int off = 1; off < Parts; off <<= 1) v += __shfl_xor(v, off, 64);
    return v;
}

template <int Parts, int Walk>
__global__ void __launch_bounds__(kBlock) k_fwd(RaySrc src,
                                                int64_t n, GeomK g, const float* __restrict__ img,
                                                float* __restrict__ p, const int32_t* __restrict__ order) {
    const int64_t l = ray_index<Parts>(order, n);
    const int part = (int)threadIdx.x % Parts;
    const __amdgpu_buffer_rsrc_t ib = img_buffer(img, g);
    RayK r;
    float acc = 0.0f;
    if (l >= 0 && ray_setup(src, l, g, r)) ray_walk<Parts, Walk, true>(ib, r, [&](double, float v) { acc += v; }, part);
    else r.ell = 0.0f;
    acc = sum_parts<Parts>(acc) * r.ell;
    if (l >= 0 && part == 0) p[l] = acc;
}

// The groups of kLineBlock rays that k_fwd_lines leaves (line_group), half a group at a time; a workgroup looks at
// `batch` halves.
constexpr int kLeftBatch = 32;

template <int Walk>
__global__ void __launch_bounds__(kBlock) k_fwd_left(RaySrc src, int64_t n, GeomK g, const float* __restrict__ img,
                                                     float* __restrict__ p, int batch) {
    static_assert(kLineBlock == 2 * kBlock, "halves of a group");
    static_assert(kLeftBatch / 2 * kLineLanes == kBlock, "lanes for every group");
    __shared__ bool left[kLeftBatch / 2];
    const int64_t h0 = (int64_t)blockIdx.x * batch;  // (batch is even: whole groups)
    const int at = (int)threadIdx.x / kLineLanes;
    const int64_t i = (h0 / 2 + at) * kLineBlock;
    const bool take = line_group(src, i < n ? i : 0, n);
    if (threadIdx.x % kLineLanes == 0) left[at] = i < n && !take;
    __syncthreads();
    const __amdgpu_buffer_rsrc_t ib = img_buffer(img, g);
    for (int q = 0; q < batch; ++q) {
        if (!left[q / 2]) continue;  // block-uniform
        const int64_t l = (h0 + q) * kBlock + threadIdx.x;
        if (l >= n) continue;
        RayK r;
        float acc = 0.0f;
        if (ray_setup(src, l, g, r)) {
            ray_walk<1, Walk, true>(ib, r, [&](double, float v) { acc += v; });
            acc *= r.ell;
        }
        p[l] = acc;
    }
}

// The rays in list order, through line sheets where many rays share a line (line.hpp).
__global__ void __launch_bounds__(kLineBlock) k_fwd_lines(RaySrc src, int64_t n, GeomK g, const float* __restrict__ img,
                                                             float* __restrict__ p, int min_run, int groups) {
    extern __shared__ float sheet[];
    __shared__ LineShared sh;
    const __amdgpu_buffer_rsrc_t ib = img_buffer(img, g);
    const int zs = line_stride(g);
    // the groups whose runs are too short are left to k_fwd_left
    __shared__ unsigned left;
    if (threadIdx.x == 0) left = 0;
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * groups * blockDim.x;
    const int at = (int)threadIdx.x / kLineLanes;  // groups <= kLineBlock / kLineLanes
    const int64_t ia = first + (int64_t)at * blockDim.x;
    const bool some = at < groups && ia < n, take = line_group(src, some ? ia : 0, n);
    if (some && !take && threadIdx.x % kLineLanes == 0) atomicOr(&left, 1u << at);
    __syncthreads();
    const int64_t here = (n - first + blockDim.x - 1) / blockDim.x;  // groups with rays
    if (__popc(left) >= (here < groups ? here : groups)) return;
    float acc = 0.0f;
    line_groups(
        g, ib, sheet, sheet + line_words(g), min_run, first, groups, left, n, sh,
        [&](int64_t i, RayK& r) {
            acc = 0.0f;
            return i < n && ray_setup(src, i, g, r);
        },
        [&](const RayK& r, const float* sheet, bool on) {
            if (!on) return;
            if (sheet) {
                line_walk<true>(sheet, zs, r, [&](float v, int) { acc += v; },
                                [&](const float (&v)[4]) { acc += (v[0] + v[1]) + (v[2] + v[3]); });
            } else {
                // the few rays beside the long runs (the walk that looks at its wave costs this kernel registers: 16.2
                // against 15.9 ms for 335 M LORs)
                ray_walk(ib, r, [&](double, float v) { acc += v; });
            }
            acc *= r.ell;
        },
        [&](int64_t i0, int cnt) {
            if ((int)threadIdx.x < cnt) p[i0 + threadIdx.x] = acc;
        });
}

// ------------------------------------------------------- TOF listmode ----

// PerRay: per-ray sigma / centre offset arrays are set (TofRay in joseph.hpp).  Presorted
// events of one wave share their TOF bin, so their plane windows nearly coincide and the lanes
// of a wave gather from the same planes at each step; with per-ray parameters the windows start
// at different planes, so the loop runs over absolute planes instead (wave-synchronous: all
// lanes at plane k, each active inside its own window), keeping the gathers of a step coherent.
// Emit: also write the events and their projections in processing order (thread i: the event order[i];
// an order entry outside [0, n) gives event i with the value 0), for a back projection that then walks
// them without an order array.
template <int Form, bool PerRay, bool Emit = false>
__global__ void __launch_bounds__(kBlock) k_fwd_tof_lm(RaySrc src,
                                                       const int16_t* __restrict__ bins, int64_t n, GeomK g,
                                                       TofK t, const float* __restrict__ img,
                                                       float* __restrict__ p, const int32_t* __restrict__ order,
                                                       EventsOut eo) {
    constexpr bool kWaveSync = PerRay;
    const __amdgpu_buffer_rsrc_t ib = img_buffer(img, g);
    const int64_t l = ray_index(order, n);
    // every load of the ray issued together (no short circuit); a thread past the end reads ray 0
    const int64_t lc = l >= 0 ? l : 0;
    const int b = bins[lc];
    float acc = 0.0f;
    RayK r;
    TofRay q;
    // Emit: the event is copied from the registers of its setup, before the plane loop (coordinate
    // events only; an order entry outside [0, n) copies event i)
    bool geo;
    if constexpr (Emit) {
        float ev[6];
        const float *ps = src.xs + 3 * lc, *pe = src.xe + 3 * lc;
        ev[0] = ps[0], ev[1] = ps[1], ev[2] = ps[2], ev[3] = pe[0], ev[4] = pe[1], ev[5] = pe[2];
        geo = ray_setup(ev, ev + 3, g, r);
        const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
        if (i < n) {
            if (l < 0) {
                const float *qs = src.xs + 3 * i, *qe = src.xe + 3 * i;
                ev[0] = qs[0], ev[1] = qs[1], ev[2] = qs[2], ev[3] = qe[0], ev[4] = qe[1], ev[5] = qe[2];
            }
            eo.xs[3 * i] = ev[0];
            eo.xs[3 * i + 1] = ev[1];
            eo.xs[3 * i + 2] = ev[2];
            eo.xe[3 * i] = ev[3];
            eo.xe[3 * i + 1] = ev[4];
            eo.xe[3 * i + 2] = ev[5];
            eo.bins[i] = l >= 0 ? (int16_t)b : bins[i];
        }
    } else {
        geo = ray_setup(src, lc, g, r);
    }
    const bool tr = tof_ray<PerRay>(t, lc, q);
    bool on = l >= 0 && b >= 0 && b < t.nb && tr && geo;
    if (on) {
        if (PerRay) r.s0 -= q.shift;
        on = tof_window_rel(r, t.c0 + b * t.bw, q.lo, q.hi);
    }
    if (kWaveSync) {  // every lane of the wave reaches this point
        const int lo = on ? r.k_lo : (1 << 30), hi = on ? r.k_hi : -(1 << 30);
        const int k0 = wave_min(lo), k1 = wave_max(hi);
        for (int k = k0; k <= k1; ++k) {
            if (k >= lo && k <= hi) {
                const float w = tof_weight_unscaled<Form, true>(fma((double)k, r.ds, r.s0), t, q.inv);
                acc = fmaf(w, stencil_gather<false>(ib, r, stencil_at(r, k)), acc);  // per-ray: arithmetic-bound
            }
        }
    } else if (on) {
        ray_walk(ib, r, [&](double kd, float v) {
            acc = fmaf(tof_weight_unscaled<Form, true>(fma(kd, r.ds, r.s0), t, q.inv), v, acc);
        });
    }
    if (on) acc *= r.ell * kTofScale<Form>;
    if (l >= 0) p[l] = acc;
    if constexpr (Emit) {
        const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
        if (i < n) eo.p[i] = l >= 0 ? acc : 0.0f;
    }
}

// Batched listmode forward: the same events through `nimg` images of the grid (imgs[b] at b * voxels,
// at most kFwdBatch per launch), p[b * n + l] for image b.  Ray setup, TOF window, plane positions,
// stencils and TOF weights are computed once per sample for all images; only the four gathers and the
// accumulation are per image, in the order of k_fwd_tof_lm, so each image's result is that kernel's.
constexpr int kFwdBatch = 8;

template <int Form, bool PerRay>
__global__ void __launch_bounds__(kBlock) k_fwd_tof_lm_batch(RaySrc src, const int16_t* __restrict__ bins, int64_t n,
                                                             GeomK g, TofK t, const float* __restrict__ imgs,
                                                             int nimg, float* __restrict__ p,
                                                             const int32_t* __restrict__ order) {
    constexpr bool kWaveSync = PerRay;
    const __amdgpu_buffer_rsrc_t ib = img_buffer_n(imgs, g, nimg);
    const int nv = g.n[0] * g.n[1] * g.n[2];
    const int64_t l = ray_index(order, n);
    // every load of the ray issued together (no short circuit); a thread past the end reads ray 0
    const int64_t lc = l >= 0 ? l : 0;
    const int b = bins[lc];
    float acc[kFwdBatch];
#pragma unroll
    for (int q = 0; q < kFwdBatch; ++q) acc[q] = 0.0f;
    RayK r;
    TofRay tq;
    const bool geo = ray_setup(src, lc, g, r);
    const bool tr = tof_ray<PerRay>(t, lc, tq);
    bool on = l >= 0 && b >= 0 && b < t.nb && tr && geo;
    if (on) {
        if (PerRay) r.s0 -= tq.shift;
        on = tof_window_rel(r, t.c0 + b * t.bw, tq.lo, tq.hi);
    }
    auto sample = [&](int k) {
        const float w = tof_weight_unscaled<Form, true>(fma((double)k, r.ds, r.s0), t, tq.inv);
        const Stencil st = stencil_at(r, k);
#pragma unroll
        for (int q = 0; q < kFwdBatch; ++q)
            if (q < nimg) {  // uniform
                const float v = PerRay ? stencil_gather_at<false>(ib, r, st, q * nv)
                                       : edge_gather(ib, r, st, st.base + q * nv);
                acc[q] = fmaf(w, v, acc[q]);
            }
    };
    if (kWaveSync) {  // every lane of the wave reaches this point
        const int lo = on ? r.k_lo : (1 << 30), hi = on ? r.k_hi : -(1 << 30);
        const int k0 = wave_min(lo), k1 = wave_max(hi);
        for (int k = k0; k <= k1; ++k)
            if (k >= lo && k <= hi) sample(k);
    } else if (on) {
        int ka, kb;
        inner_planes(r, ka, kb);
        edge_planes(r, ka, kb, sample);
        unsigned plane = (unsigned)(ka * r.sp);
        double kd = (double)ka;
        for (int k = ka; k <= kb; ++k, kd += 1.0, plane += (unsigned)r.sp) {
            float fu, fw;
            const unsigned off = inner_at(r, kd, plane, fu, fw);
            const float w = tof_weight_unscaled<Form, true>(fma(kd, r.ds, r.s0), t, tq.inv);
#pragma unroll
            for (int q = 0; q < kFwdBatch; ++q)
                if (q < nimg) {
                    const unsigned at = (off + (unsigned)(q * nv)) * 4u;
                    const auto a = __builtin_amdgcn_raw_buffer_load_b64(ib, at, 0, 0);
                    const auto c = __builtin_amdgcn_raw_buffer_load_b64(ib, at + (unsigned)r.su * 4u, 0, 0);
                    acc[q] = fmaf(w, inner_value(__uint_as_float(a[0]), __uint_as_float(a[1]), __uint_as_float(c[0]),
                                                 __uint_as_float(c[1]), fu, fw), acc[q]);
                }
        }
    }
    if (l < 0) return;
    const float scale = on ? r.ell * kTofScale<Form> : 0.0f;
#pragma unroll
    for (int q = 0; q < kFwdBatch; ++q)
        if (q < nimg) p[(int64_t)q * n + l] = on ? acc[q] * scale : 0.0f;
}

// imgs[0 .. count) of nv voxels -> out[voxel][B], zeros for images count .. B - 1
template <int B>
__global__ void __launch_bounds__(kBlock) k_interleave(const float* __restrict__ imgs, int count, int64_t nv,
                                                       float* __restrict__ out) {
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < nv; v += (int64_t)gridDim.x * kBlock) {
        float x[B];
#pragma unroll
        for (int q = 0; q < B; ++q) x[q] = q < count ? imgs[q * nv + v] : 0.0f;
#pragma unroll
        for (int q = 0; q < B; q += 2) *reinterpret_cast<float2*>(out + v * B + q) = make_float2(x[q], x[q + 1]);
    }
}

// A voxel of all B images from the interleaved copy, `at` its byte offset
template <int B>
__device__ __forceinline__ void load_images(__amdgpu_buffer_rsrc_t ib, unsigned at, float (&v)[B]) {
    if constexpr (B == 2) {
        const auto a = __builtin_amdgcn_raw_buffer_load_b64(ib, at, 0, 0);
        v[0] = __uint_as_float(a[0]), v[1] = __uint_as_float(a[1]);
    } else {
#pragma unroll
        for (int q = 0; q < B; q += 4) {
            const auto a = __builtin_amdgcn_raw_buffer_load_b128(ib, at + q * 4u, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[q + i] = __uint_as_float(a[i]);
        }
    }
}

// k_fwd_tof_lm_batch over images interleaved voxel by voxel (k_interleave).  With the images apart a sample asks for
// two cache lines of every image, and the lines of eight images, not one, have to stay in an L2 of 4 MB: 10 M
// presorted events through eight images of 128 x 128 x 64 took 0.95 G misses, 17.8 ms.  Interleaved, a column's two
// slices of all images are 64 bytes together: 0.45 G misses, 6.9 ms, the address units busy for most of it.  The same
// arithmetic in the same order per image.
template <int Form, int B>
__global__ void __launch_bounds__(kBlock) k_fwd_tof_lm_mixed(RaySrc src, const int16_t* __restrict__ bins, int64_t n,
                                                             GeomK g, TofK t, const float* __restrict__ mixed,
                                                             int nimg, float* __restrict__ p,
                                                             const int32_t* __restrict__ order) {
    const __amdgpu_buffer_rsrc_t ib = img_buffer_n(mixed, g, B);
    const int64_t l = ray_index(order, n);
    const int64_t lc = l >= 0 ? l : 0;
    const int b = bins[lc];
    float acc[B];
#pragma unroll
    for (int q = 0; q < B; ++q) acc[q] = 0.0f;
    RayK r;
    const bool geo = ray_setup(src, lc, g, r);
    const bool on = l >= 0 && b >= 0 && b < t.nb && geo && tof_window_rel(r, t.c0 + b * t.bw, t.lo, t.hi);
    if (on) {
        int ka, kb;
        inner_planes(r, ka, kb);
        edge_planes(r, ka, kb, [&](int k) {
            const Stencil st = stencil_at(r, k);
            const float w = tof_weight_unscaled<Form, true>(fma((double)k, r.ds, r.s0), t, t.u_per_mm);
            const unsigned at = (unsigned)st.base * (B * 4u), su = (unsigned)r.su * (B * 4u), sw = (unsigned)r.sw * (B * 4u);
            float v00[B], v01[B], v10[B], v11[B];
            load_images<B>(ib, st.i0ok && st.j0ok ? at : 0xFFFFFF00u, v00);
            load_images<B>(ib, st.i0ok && st.j1ok ? at + sw : 0xFFFFFF00u, v01);
            load_images<B>(ib, st.i1ok && st.j0ok ? at + su : 0xFFFFFF00u, v10);
            load_images<B>(ib, st.i1ok && st.j1ok ? at + su + sw : 0xFFFFFF00u, v11);
#pragma unroll
            for (int q = 0; q < B; ++q)
                acc[q] = fmaf(w, inner_value(v00[q], v01[q], v10[q], v11[q], st.fu, st.fw), acc[q]);
        });
        unsigned plane = (unsigned)(ka * r.sp);
        double kd = (double)ka;
        for (int k = ka; k <= kb; ++k, kd += 1.0, plane += (unsigned)r.sp) {
            float fu, fw, a0[B], a1[B], c0[B], c1[B];
            const unsigned at = inner_at(r, kd, plane, fu, fw) * (B * 4u), at1 = at + (unsigned)r.su * (B * 4u);
            load_images<B>(ib, at, a0);
            load_images<B>(ib, at + B * 4u, a1);
            load_images<B>(ib, at1, c0);
            load_images<B>(ib, at1 + B * 4u, c1);
            const float w = tof_weight_unscaled<Form, true>(fma(kd, r.ds, r.s0), t, t.u_per_mm);
#pragma unroll
            for (int q = 0; q < B; ++q) acc[q] = fmaf(w, inner_value(a0[q], a1[q], c0[q], c1[q], fu, fw), acc[q]);
        }
    }
    if (l < 0) return;
    const float scale = on ? r.ell * kTofScale<Form> : 0.0f;
#pragma unroll
    for (int q = 0; q < B; ++q)
        if (q < nimg) p[(int64_t)q * n + l] = on ? acc[q] * scale : 0.0f;
}

// ------------------------------------------------------- TOF sinogram ----
//
// Each thread keeps its n_bins accumulators in LDS (column per thread, so a
// wave touching the same bin hits 64 distinct banks).  Per plane sample only
// the bins inside the TOF window are evaluated; neighbouring bins share their
// edge, so a window of m bins costs m + 1 erf evaluations.  The block's
// [rays][bins] output tile is contiguous in memory and is written with
// coalesced stores at the end.  PerRay: per-ray sigma / centre offset arrays are set.

template <bool PerRay>
__global__ void k_fwd_tof_sino(RaySrc src, int64_t n, GeomK g,
                               TofK t, const float* __restrict__ img, float* __restrict__ p) {
    extern __shared__ float lds[];  // [nb][blockDim]
    const int nt = blockDim.x;
    const int64_t l0 = (int64_t)blockIdx.x * nt;
    const int64_t l = l0 + threadIdx.x;
    for (int b = 0; b < t.nb; ++b) lds[b * nt + threadIdx.x] = 0.0f;
    const __amdgpu_buffer_rsrc_t ib = img_buffer(img, g);
    RayK r;
    TofRay q;
    if (l < n && tof_ray<PerRay>(t, l, q) && ray_setup(src, l, g, r)) {
        if (PerRay) r.s0 -= q.shift;
        float* mine = lds + threadIdx.x;
        for (int k = r.k_lo; k <= r.k_hi; ++k) {
            const float v = stencil_gather<false>(ib, r, stencil_at(r, k));  // arithmetic-bound
            if (v == 0.0f) continue;
            const double s = fma((double)k, r.ds, r.s0);
            int b_lo, b_hi;
            tof_bin_range(s, t, q.lo, q.hi, b_lo, b_hi);
            if (t.lut) {
                for (int b = b_lo; b <= b_hi; ++b) mine[b * nt] += tof_lut(s - (t.c0 + b * t.bw), t) * v;
                continue;
            }
            // upper edge argument of bin b_lo; the next edges follow in float steps of bw
            const float x_hi0 = (float)(s - (t.c0 + b_lo * t.bw) + 0.5 * t.bw), bwf = (float)t.bw;
            float e_hi = tof_erf(x_hi0, q.inv, t);
            for (int b = b_lo; b <= b_hi; ++b) {
                const float e_lo = tof_erf(x_hi0 - (float)(b - b_lo + 1) * bwf, q.inv, t);
                mine[b * nt] += 0.5f * (e_hi - e_lo) * v;
                e_hi = e_lo;
            }
        }
        const float ell = r.ell;
        for (int b = 0; b < t.nb; ++b) mine[b * nt] *= ell;
    }
    __syncthreads();
    const int64_t nrays = (n - l0 < nt) ? (n - l0) : nt;
    const int64_t total = nrays * t.nb;
    float* out = p + l0 * t.nb;
    for (int64_t i = threadIdx.x; i < total; i += nt) {
        const int ray = (int)(i / t.nb), b = (int)(i - (int64_t)ray * t.nb);
        out[i] = lds[b * nt + ray];
    }
}

// A ray's row of TOF bins, filled in order (rising or falling): a bin's value waits in the thread's LDS slots until
// its block of eight is complete, which then goes out as two 16-byte stores.  `next` and `dir` are the
// wave's in the uniform walk, a lane's own otherwise.
struct alignas(4) Float4u {
    float v[4];
};

struct BinRow {
    float* out;   // the ray's row of nb bins
    float* slot;  // eight LDS floats, `step` apart
    int step, nb;
    __device__ __forceinline__ void emit(float v, int& next, int dir) {
        const int s = next & 7;
        slot[s * step] = v;
        if (dir > 0 ? (s == 7 || next == nb - 1) : s == 0) {
            const int b = next & ~7;
            float x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = slot[i * step];
            if (b + 8 <= nb) {
                *reinterpret_cast<Float4u*>(out + b) = Float4u{{x[0], x[1], x[2], x[3]}};
                *reinterpret_cast<Float4u*>(out + b + 4) = Float4u{{x[4], x[5], x[6], x[7]}};
            } else {
#pragma unroll
                for (int i = 0; i < 7; ++i)
                    if (b + i < nb) out[b + i] = x[i];
            }
        }
        next += dir;
    }
    // bin b of the row (ignored outside it); the bins since the last one are 0
    __device__ __forceinline__ void put(int b, float v, int& next, int dir) {
        if ((unsigned)b >= (unsigned)nb) return;
        while (next != b) emit(0.0f, next, dir);
        emit(v, next, dir);
    }
    __device__ __forceinline__ void finish(int& next, int dir) {
        while ((unsigned)next < (unsigned)nb) emit(0.0f, next, dir);
    }
};

// TOF sinogram forward with one Gaussian for all rays: samples through line sheets, weights from the fitted
// edge polynomials.  The 2 R + 1 bins a sample reaches are accumulated in registers; when the ray moves on to
// the next bin, the one it leaves behind is complete and goes out through BinRow (whose slots leave the LDS
// for two workgroups per CU beside their sheets).  The rays of a line move through the bins nearly together:
// where they stay less than a bin apart, the wave keeps one window of 2 R + 2 bins and all its lanes
// leave a bin in one step; with a window per lane, moving it took as many instructions as the samples.
template <int R>
__global__ void __launch_bounds__(kSinoBlock, 4) k_fwd_tof_sino_lines(RaySrc src, int64_t n, GeomK g, TofEdgeK t, int nb,
                                                                   const float* __restrict__ img,
                                                                   float* __restrict__ p, int min_run, int groups) {
    extern __shared__ float line_mem[];
    __shared__ LineShared sh;
    float* const slots = line_mem + line_words(g);  // eight per thread (or the planes' records, between the walks)
    const int zs = line_stride(g);
    const __amdgpu_buffer_rsrc_t ib = img_buffer(img, g);
    BinRow row{nullptr, slots + threadIdx.x, (int)blockDim.x, nb};
    bool walked = false;
    if constexpr (R <= 3) tof_edge_to_vgprs<R>(t);  // (more would not fit 128 registers)
    line_groups(
        g, ib, line_mem, slots, min_run, (int64_t)blockIdx.x * groups * blockDim.x, groups, 0u, n, sh,
        [&](int64_t i, RayK& r) {
            walked = false;
            row.out = p + i * nb;
            return i < n && ray_setup(src, i, g, r);
        },
        [&](const RayK& r, const float* sheet, bool on) __attribute__((always_inline)) {
            const double B0 = fma(r.s0, t.inv_bw, t.B0), dB = r.ds * t.inv_bw;
            const float ell = r.ell;
            float w[2 * R + 1];
            if (sheet && !sh.odd) {  // a sheet with an infinity: a window per ray, which keeps it to its bins
                const int k0 = __builtin_amdgcn_readfirstlane(wave_min(on ? r.k_lo : INT_MAX));
                const int k1 = __builtin_amdgcn_readfirstlane(wave_max(on ? r.k_hi : INT_MIN));
                // the lanes' positions in bins at both ends (linear between): how far they lie apart there
                const double Ba = fma((double)k0, dB, B0), Bb = fma((double)k1, dB, B0);
                const int first = __ffsll((long long)__ballot(on)) - 1;
                const double Ba0 = __shfl(Ba, first, 64), Bb0 = __shfl(Bb, first, 64);
                // the window moves one way only: a line's rays in both directions (bitwise the same U0 and dU) walk alone
                const int dir = __builtin_amdgcn_readfirstlane(__shfl(dB, first, 64) > 0.0 ? 1 : -1);
                const bool near = (dB > 0.0) == (dir > 0) && fabs(Ba - Ba0) < 0.49 && fabs(Bb - Bb0) < 0.49 &&
                                  fabs(Ba0) < 4096.0 && fabs(Bb0) < 4096.0;
                if (__ballot(on && !near) == 0ull) {
                    if (!on) return;
                    walked = true;
                    const double dZ = r.dW + (double)zs, Z0 = r.W0 + 1.0;
                    float acc[2 * R + 2];  // bins cur - R .. cur + R + 1
#pragma unroll
                    for (int i = 0; i <= 2 * R + 1; ++i) acc[i] = 0.0f;
                    int next = dir > 0 ? 0 : nb - 1;
                    // cur: the lowest bin a lane lies in (wave-uniform; the others lie in cur or cur + 1)
                    int cur = __builtin_amdgcn_readfirstlane((int)rint(Ba0)) - dir;
                    auto up = [&]() __attribute__((always_inline)) {
                        row.put(cur - R, acc[0] * ell, next, 1);
#pragma unroll
                        for (int i = 0; i <= 2 * R; ++i) acc[i] = acc[i + 1];
                        acc[2 * R + 1] = 0.0f;
                        ++cur;
                    };
                    auto down = [&]() __attribute__((always_inline)) {
                        row.put(cur + R + 1, acc[2 * R + 1] * ell, next, -1);
#pragma unroll
                        for (int i = 2 * R + 1; i > 0; --i) acc[i] = acc[i - 1];
                        acc[0] = 0.0f;
                        --cur;
                    };
                    double kd = (double)k0;
                    for (int k = k0; k <= k1; ++k, kd += 1.0) {
                        float v = 0.0f;
                        if (k >= r.k_lo && k <= r.k_hi) {
                            const double Z = fma(kd, dZ, Z0);
                            const int i = (int)Z;
                            const float a = sheet[i], b = sheet[i + 1];
                            v = fmaf((float)__builtin_amdgcn_fract(Z), b - a, a);
                        }
                        if (__ballot(v != 0.0f) == 0ull) continue;
                        const double B = fma(kd, dB, B0), fb = rint(B);
                        const int q = (int)fb;
                        tof_edge_weights<R>((float)(B - fb), t, w);
                        if (__ballot(q != cur)) {
                            if (dir > 0)
                                while (__ballot(q <= cur) == 0ull) up();
                            else
                                while (__ballot(q < cur)) down();
                            const bool hi = q != cur;
                            acc[0] = fmaf(hi ? 0.0f : w[0], v, acc[0]);
#pragma unroll
                            for (int i = 1; i <= 2 * R; ++i) acc[i] = fmaf(hi ? w[i - 1] : w[i], v, acc[i]);
                            acc[2 * R + 1] = fmaf(hi ? w[2 * R] : 0.0f, v, acc[2 * R + 1]);
                        } else {
#pragma unroll
                            for (int i = 0; i <= 2 * R; ++i) acc[i] = fmaf(w[i], v, acc[i]);
                        }
                    }
#pragma unroll 1
                    for (int i = 0; i <= 2 * R + 1; ++i) {
                        if (dir > 0) up();
                        else down();
                    }
                    row.finish(next, dir);
                    return;
                }
            }
            if (!on) return;
            walked = true;
            float acc[2 * R + 1];
#pragma unroll
            for (int i = 0; i <= 2 * R; ++i) acc[i] = 0.0f;
            const bool up = dB > 0.0;
            const int dir = up ? 1 : -1;
            int next = up ? 0 : nb - 1;
            int cur = (int)rint(fma((double)r.k_lo, dB, B0));
            // the bin the ray leaves behind goes out, the others move up
            auto advance = [&]() __attribute__((always_inline)) {
                row.put(up ? cur - R : cur + R, (up ? acc[0] : acc[2 * R]) * ell, next, dir);
                float a[2 * R + 1];
#pragma unroll
                for (int i = 0; i <= 2 * R; ++i)
                    a[i] = up ? (i < 2 * R ? acc[i + 1] : 0.0f) : (i > 0 ? acc[i - 1] : 0.0f);
#pragma unroll
                for (int i = 0; i <= 2 * R; ++i) acc[i] = a[i];
                cur += dir;
            };
            auto sample = [&](float v, int k) __attribute__((always_inline)) {
                if (__ballot(v != 0.0f) == 0ull) return;
                const double B = fma((double)k, dB, B0), fb = rint(B);
                const int q = (int)fb;
                for (int i = 0; cur != q; ++i) {
                    if (i > 2 * R) cur = q;  // further than the window reaches: it is empty by now
                    else advance();
                }
                tof_edge_weights<R>((float)(B - fb), t, w);
                // only into the bins that the sample reaches, which are all but an outer one (R - 1 < reach <= R bins):
                // v may be infinite
                if (w[0] != 0.0f) acc[0] = fmaf(w[0], v, acc[0]);
                if (w[2 * R] != 0.0f) acc[2 * R] = fmaf(w[2 * R], v, acc[2 * R]);
#pragma unroll
                for (int i = 1; i < 2 * R; ++i) acc[i] = fmaf(w[i], v, acc[i]);
            };
            if (sheet) {
                line_walk<false>(sheet, zs, r, sample, [](const float (&)[4]) {});
            } else {
                for (int k = r.k_lo; k <= r.k_hi; ++k) sample(stencil_gather<false>(ib, r, stencil_at(r, k)), k);
            }
#pragma unroll 1
            for (int i = 0; i <= 2 * R; ++i) advance();
            row.finish(next, dir);
        },
        [&](int64_t, int cnt) {
            if (!walked && (int)threadIdx.x < cnt)
                for (int b = 0; b < nb; ++b) row.out[b] = 0.0f;
        });
}

// ------------------------------------------------------- work counter ----
//
// Plane samples per ray whose 2x2 stencil has at least one voxel inside the
// grid; for TOF listmode (bins != nullptr) only samples strictly inside the
// event's TOF window (non-zero weight).  Same traversal as the projectors.

__global__ void __launch_bounds__(kBlock) k_count(RaySrc src,
                                                  const int16_t* __restrict__ bins, int64_t n, GeomK g, TofK t,
                                                  int32_t* __restrict__ counts) {
    const int64_t l = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (l >= n) return;
    int cnt = 0;
    RayK r;
    TofRay q{};
    bool ok = ray_setup(src, l, g, r);
    double centre = 0.0;
    if (ok && bins) {
        const int b = bins[l];
        ok = b >= 0 && b < t.nb && tof_ray<true>(t, l, q);
        r.s0 -= q.shift;
        centre = t.c0 + b * t.bw;
        ok = ok && tof_window(r, centre, q.lo, q.hi);
    }
    if (ok) {
        for (int k = r.k_lo; k <= r.k_hi; ++k) {
            const Stencil st = stencil_at(r, k);
            if (!((st.i0ok || st.i1ok) && (st.j0ok || st.j1ok))) continue;
            if (bins) {
                const double x = fma((double)k, r.ds, r.s0) - centre;
                if (!(x > q.lo && x < q.hi)) continue;
            }
            ++cnt;
        }
    }
    counts[l] = cnt;
}

// --------------------------------------------------------------- launch ----

static unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

static int device_cus() {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) !=
                                                 hipSuccess || cus <= 0)
        cus = 256;
    return cus;
}

// Groups of T rays per workgroup of a line kernel: about `rays` consecutive rays (a clinical sinogram's line has 2204),
// unless that leaves CUs idle.
static int line_groups_of(int64_t n, int T, int rays) {
    const int64_t groups = n / ((int64_t)T * 8 * device_cus());
    return (int)(groups < 1 ? 1 : groups > rays / T ? rays / T : groups);
}

constexpr int kLineMaxWords = 20 * 1024;  // largest sheet (two workgroups of a smaller one share a CU's LDS)
constexpr int64_t kCuLds = 160 * 1024;
constexpr int64_t kLineStaticLds = sizeof(LineShared) + 256;  // what the line kernels hold beside the sheet and the planes

// Dynamic LDS of k_fwd_lines and k_back_lines (64 bits: the extents of a long flat grid overflow an int)
static int64_t line_lds_bytes(const GeomK& g) {
    const int64_t planes = line_planes(g);
    return (planes * line_stride(g) + 2 + 3 * planes) * (int64_t)sizeof(float);
}

// Whether a CU's LDS holds the grid's sheet with its planes' records
static bool lines_fit(const GeomK& g) {
    return (int64_t)line_planes(g) * line_stride(g) + 2 <= kLineMaxWords && line_lds_bytes(g) + kLineStaticLds <= kCuLds;
}

// Fewest rays the non-TOF line kernel is launched for: below, the second launch and the look at the groups are felt
// where the lines turn out short (561,600 rays of 39 a line: 62 us by one kernel, 79 by two)
constexpr int64_t kLineRays = 11 << 19;
constexpr int64_t kLineRaysTof = 1 << 20;  // TOF back projection

// Lanes that share a ray in the ray-per-thread forwards: kParts of them while that leaves lanes of the chip idle.
// A small call's time is one ray's, a wait for memory per plane, of which each lane has a quarter (64,512 rays: 22.2 -> 15.9
// us; four planes read at a time 17.2).  Only where rays are sinograms' or sorted: 100,001 unsorted TOF events stay at 61 us,
// bound by their 20 M requests for cache lines.
static bool split_rays(int64_t n) { return n <= (int64_t)device_cus() * (kBlock * 8 / kParts); }

hipError_t launch_fwd(const RaySrc& src, int64_t n, const GeomK& g, const float* img, float* p,
                      const int32_t* order, hipStream_t s) {
    // Planes read at a time: while the image fits an XCD's L2 four (128 x 128 x 64, 5 M presorted rays 655 -> 599 us),
    // in a larger one, whose lines more samples in flight only drive out, one (215 x 215 x 71, 1 M unsorted rays: 2.86 ms
    // with four, 2.2 with one)
    const bool walk4 = (int64_t)g.n[0] * g.n[1] * g.n[2] * 4 <= (4 << 20);
    if (!order && n >= kLineRays && lines_fit(g)) {
        constexpr int T = kLineBlock;
        const size_t lds = (size_t)line_lds_bytes(g);
        const hipError_t e = hipFuncSetAttribute((const void*)k_fwd_lines, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)lds);
        if (e != hipSuccess) return e;
        const int groups = line_groups_of(n, T, 16384);
        const int64_t per = n / ((int64_t)kBlock * 64 * device_cus()) / 2 * 2;
        const int batch = (int)(per < 2 ? 2 : per > kLeftBatch ? kLeftBatch : per);
        hipLaunchKernelGGL(walk4 ? k_fwd_left<kWalk> : k_fwd_left<1>, dim3(grid_for(n, kBlock * batch)), dim3(kBlock), 0, s, src,
                           n, g, img, p, batch);
        hipLaunchKernelGGL(k_fwd_lines, dim3(grid_for(n, T * groups)), dim3(T), lds, s, src, n, g, img, p, kLineMinRun,
                           groups);
        return hipGetLastError();
    }
    if (split_rays(n))
        hipLaunchKernelGGL((k_fwd<kParts, 1>), dim3(grid_for(n * kParts, kBlock)), dim3(kBlock), 0, s, src, n, g, img, p, order);
    else
        hipLaunchKernelGGL((walk4 ? k_fwd<1, kWalk> : k_fwd<1, 1>), dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, src, n, g,
                           img, p, order);
    return hipGetLastError();
}

// Back projections of ray lists go through the run/sheet kernel (sheet.hpp): kLeftRuns: only what k_back_lines leaves of a
// list without an order; kRunsOrTiles: where the device has not chosen the tiles.
enum Runs : int { kAllRuns, kLeftRuns, kRunsOrTiles };

struct RunsOrTiles {
    const int* changes;  // the tiles where *changes >= need
    int need;
};

template <Runs Kind = kAllRuns, class Mode>
static hipError_t launch_runs(const Mode& m, const RaySrc& src, int64_t n, const GeomK& g, float* img,
                              const int32_t* order, hipStream_t s, int n_img = 1, int64_t img_stride = 0,
                              bool regular = false, RunsOrTiles choice = {nullptr, 0}) {
    const int nw = (g.n[2] <= kSheetMaxW) ? g.n[2] : 0;
    const size_t lds = SheetLayout::bytes(nw, g);
    const void* k;
    if constexpr (Kind == kLeftRuns) k = (const void*)k_back_runs_left<Mode>;
    else if constexpr (Kind == kRunsOrTiles) k = (const void*)k_back_runs_else<Mode>;
    else k = (const void*)k_back_runs<Mode>;
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    // enough workgroups for about 4 per CU (small subsets), at most kSheetGroups groups each
    const int cus = device_cus();
    int64_t groups = (n + (int64_t)kSheetBlock * 4 * cus - 1) / ((int64_t)kSheetBlock * 4 * cus);
    groups = groups < 1 ? 1 : (groups > kSheetGroups ? kSheetGroups : groups);
    // as many more as leave each of the two workgroups that a CU holds eight and sixteen in turn: with fewer the last ones
    // run alone (9.7 M TOF rays in lines of 64: 0.98 of k_back_runs' speed with 8 groups, 0.92 with 16)
    if (Kind == kLeftRuns && n > (int64_t)kLeftGroups / 2 * kSheetBlock * 16 * cus)
        groups = n > (int64_t)kLeftGroups * kSheetBlock * 32 * cus ? kLeftGroups : kLeftGroups / 2;
    const dim3 grid(grid_for(n, kSheetBlock * groups));
    if constexpr (Kind == kLeftRuns)
        hipLaunchKernelGGL(k_back_runs_left<Mode>, grid, dim3(kSheetBlock), lds, s, m, src, n, g, img, nw, (int)groups,
                           regular);
    else if constexpr (Kind == kRunsOrTiles)
        hipLaunchKernelGGL(k_back_runs_else<Mode>, grid, dim3(kSheetBlock), lds, s, m, src, n, g, img, order, nw, (int)groups,
                           n_img, img_stride, choice.changes, choice.need);
    else
        hipLaunchKernelGGL(k_back_runs<Mode>, grid, dim3(kSheetBlock), lds, s, m, src, n, g, img, order, nw, (int)groups,
                           n_img, img_stride);
    return hipGetLastError();
}

// The groups of rays with long runs by k_back_lines, the others by the run/sheet kernel (first: their sums meet a small
// image, where a float addition rounds less)
template <class LineMode, class Mode>
static hipError_t launch_back_lines(const LineMode& lm, const Mode& m, const RaySrc& src, int64_t n, const GeomK& g,
                                    float* img, hipStream_t s) {
    const size_t lds = (size_t)line_lds_bytes(g);
    hipError_t e = hipFuncSetAttribute((const void*)k_back_lines<LineMode>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
    e = launch_runs<kLeftRuns>(m, src, n, g, img, nullptr, s, 1, 0, LineMode::kRegular);
    if (e != hipSuccess) return e;
    const int groups = line_groups_of(n, kLineBlock, 16384);
    hipLaunchKernelGGL(k_back_lines<LineMode>, dim3(grid_for(n, kLineBlock * groups)), dim3(kLineBlock), lds, s, lm, src, n,
                       g, img, groups);
    return hipGetLastError();
}

hipError_t launch_back(const RaySrc& src, int64_t n, const GeomK& g, float* img, const float* p,
                       const int32_t* order, hipStream_t s) {
    ModeNonTof m{p};
    if (!order && n >= kLineRays && lines_fit(g))
        return launch_back_lines(LineBackNonTof{p}, m, src, n, g, img, s);
    return launch_runs(m, src, n, g, img, order, s);
}

hipError_t launch_fwd_tof_lm(const RaySrc& src, const int16_t* bins, int64_t n, const GeomK& g,
                             const TofK& t, const float* img, float* p, const int32_t* order, hipStream_t s) {
    const bool per = t.sig_ray || t.off_ray;
    const int form = tof_form(t);
    auto* k = form == kFormLut    ? (per ? k_fwd_tof_lm<kFormLut, true> : k_fwd_tof_lm<kFormLut, false>)
              : form == kFormPoly ? (per ? k_fwd_tof_lm<kFormPoly, true> : k_fwd_tof_lm<kFormPoly, false>)
                                  : (per ? k_fwd_tof_lm<kFormErf, true> : k_fwd_tof_lm<kFormErf, false>);
    hipLaunchKernelGGL(k, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, src, bins, n, g, t, img, p, order,
                       EventsOut{});
    return hipGetLastError();
}

hipError_t launch_fwd_tof_lm_gather(const RaySrc& src, const int16_t* bins, int64_t n, const GeomK& g,
                                    const TofK& t, const float* img, float* p, const int32_t* order,
                                    const EventsOut& eo, hipStream_t s) {
    const int form = tof_form(t);
    auto* k = form == kFormLut    ? k_fwd_tof_lm<kFormLut, false, true>
              : form == kFormPoly ? k_fwd_tof_lm<kFormPoly, false, true>
                                  : k_fwd_tof_lm<kFormErf, false, true>;
    hipLaunchKernelGGL(k, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, src, bins, n, g, t, img, p, order, eo);
    return hipGetLastError();
}

// Images interleaved per launch of k_fwd_tof_lm_mixed for a batch of n_img: 8, 4 or 2; 0 where the images stay apart.
// The copy costs two passes over the images (eight of 128 x 128 x 64: 14 us).  At n = voxels / 16 the events already
// repay it twice over (two images 46 -> 32 us, eight 392 -> 63 us; 12 mm bins, unsorted), below voxels / 32 two
// images would gain nothing.
static int mixed_images(int64_t n, const GeomK& g, const TofK& t, int n_img) {
    const int64_t nv = (int64_t)g.n[0] * g.n[1] * g.n[2];
    if (n_img < 2 || t.sig_ray || t.off_ray || n < nv / 32) return 0;
    int B = n_img > 4 ? 8 : n_img > 2 ? 4 : 2;
    while (B > 1 && nv * B * 4 >= 0xFFFFFF00ll) B /= 2;
    return B > 1 ? B : 0;
}

size_t fwd_batch_bytes(int64_t n, const GeomK& g, const TofK& t, int n_img) {
    return (size_t)g.n[0] * g.n[1] * g.n[2] * mixed_images(n, g, t, n_img) * sizeof(float);
}

template <int B>
static hipError_t launch_mixed(const RaySrc& src, const int16_t* bins, int64_t n, const GeomK& g, const TofK& t,
                               const float* imgs, int cnt, float* p, const int32_t* order, float* ws, hipStream_t s) {
    const int64_t nv = (int64_t)g.n[0] * g.n[1] * g.n[2];
    const int64_t blocks = (nv + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_interleave<B>, dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(kBlock), 0, s, imgs, cnt,
                       nv, ws);
    const int form = tof_form(t);
    auto* k = form == kFormLut    ? k_fwd_tof_lm_mixed<kFormLut, B>
              : form == kFormPoly ? k_fwd_tof_lm_mixed<kFormPoly, B>
                                  : k_fwd_tof_lm_mixed<kFormErf, B>;
    hipLaunchKernelGGL(k, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, src, bins, n, g, t, ws, cnt, p, order);
    return hipGetLastError();
}

// ws: fwd_batch_bytes of device memory, or nullptr
hipError_t launch_fwd_tof_lm_batch(const RaySrc& src, const int16_t* bins, int64_t n, const GeomK& g, const TofK& t,
                                   const float* imgs, int n_img, float* p, const int32_t* order, float* ws,
                                   hipStream_t s) {
    const bool per = t.sig_ray || t.off_ray;
    const int form = tof_form(t);
    auto* k = form == kFormLut    ? (per ? k_fwd_tof_lm_batch<kFormLut, true> : k_fwd_tof_lm_batch<kFormLut, false>)
              : form == kFormPoly ? (per ? k_fwd_tof_lm_batch<kFormPoly, true> : k_fwd_tof_lm_batch<kFormPoly, false>)
                                  : (per ? k_fwd_tof_lm_batch<kFormErf, true> : k_fwd_tof_lm_batch<kFormErf, false>);
    // images per launch: at most kFwdBatch, and their bytes within the 32-bit buffer range
    const int64_t nv = (int64_t)g.n[0] * g.n[1] * g.n[2];
    const int most = ws ? mixed_images(n, g, t, n_img) : 0;
    int64_t per_launch = ((int64_t(1) << 32) - 1) / (nv * 4);
    if (per_launch > kFwdBatch) per_launch = kFwdBatch;
    if (most) per_launch = most;
    for (int b0 = 0; b0 < n_img; b0 += (int)per_launch) {
        const int cnt = (n_img - b0 < per_launch) ? (n_img - b0) : (int)per_launch;
        const float* im = imgs + b0 * nv;
        float* pb = p + b0 * n;
        hipError_t e = hipSuccess;
        if (most && cnt > 4) e = launch_mixed<8>(src, bins, n, g, t, im, cnt, pb, order, ws, s);
        else if (most && cnt > 2) e = launch_mixed<4>(src, bins, n, g, t, im, cnt, pb, order, ws, s);
        else if (most && cnt == 2) e = launch_mixed<2>(src, bins, n, g, t, im, cnt, pb, order, ws, s);
        else {
            hipLaunchKernelGGL(k, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, src, bins, n, g, t, im, cnt, pb, order);
            e = hipGetLastError();
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <Runs Kind = kAllRuns>
static hipError_t back_tof_lm_runs(const RaySrc& src, const int16_t* bins, int64_t n, const GeomK& g, const TofK& t,
                                   float* img, const float* p, const int32_t* order, hipStream_t s,
                                   RunsOrTiles choice = {nullptr, 0}) {
    const int form = tof_form(t);
    auto runs = [&](const auto& m) { return launch_runs<Kind>(m, src, n, g, img, order, s, 1, 0, false, choice); };
    if (t.sig_ray || t.off_ray) {
        if (form == kFormLut) return runs(ModeTofLm<kFormLut, true>{p, bins, t});
        if (form == kFormPoly) return runs(ModeTofLm<kFormPoly, true>{p, bins, t});
        return runs(ModeTofLm<kFormErf, true>{p, bins, t});
    }
    if (form == kFormLut) return runs(ModeTofLm<kFormLut>{p, bins, t});
    if (form == kFormPoly) return runs(ModeTofLm<kFormPoly>{p, bins, t});
    return runs(ModeTofLm<kFormErf>{p, bins, t});
}

hipError_t launch_back_tof_lm(const RaySrc& src, const int16_t* bins, int64_t n, const GeomK& g,
                              const TofK& t, float* img, const float* p, const int32_t* order, hipStream_t s) {
    return back_tof_lm_runs(src, bins, n, g, t, img, p, order, s);
}

// Images per launch of the batched listmode back projection (each launch walks the events once)
constexpr int kBackBatch = 16;

template <Runs Kind = kAllRuns>
static hipError_t back_tof_lm_batch_runs(const RaySrc& src, const int16_t* bins, int64_t n, const GeomK& g, const TofK& t,
                                         float* imgs, int n_img, const float* p, const int32_t* order, hipStream_t s,
                                         RunsOrTiles choice = {nullptr, 0}) {
    const int64_t nv = (int64_t)g.n[0] * g.n[1] * g.n[2];
    const int form = tof_form(t);
    const bool per = t.sig_ray || t.off_ray;
    for (int b0 = 0; b0 < n_img; b0 += kBackBatch) {
        const int cnt = (n_img - b0 < kBackBatch) ? (n_img - b0) : kBackBatch;
        float* im = imgs + (int64_t)b0 * nv;
        const float* pb = p + (int64_t)b0 * n;
        auto runs = [&](const auto& m) { return launch_runs<Kind>(m, src, n, g, im, order, s, cnt, nv, false, choice); };
        hipError_t e;
        if (per) {
            if (form == kFormLut) e = runs(ModeTofLm<kFormLut, true, true>{pb, bins, t});
            else if (form == kFormPoly) e = runs(ModeTofLm<kFormPoly, true, true>{pb, bins, t});
            else e = runs(ModeTofLm<kFormErf, true, true>{pb, bins, t});
        } else {
            if (form == kFormLut) e = runs(ModeTofLm<kFormLut, false, true>{pb, bins, t});
            else if (form == kFormPoly) e = runs(ModeTofLm<kFormPoly, false, true>{pb, bins, t});
            else e = runs(ModeTofLm<kFormErf, false, true>{pb, bins, t});
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_back_tof_lm_batch(const RaySrc& src, const int16_t* bins, int64_t n, const GeomK& g,
                                    const TofK& t, float* imgs, int n_img, const float* p, const int32_t* order,
                                    hipStream_t s) {
    return back_tof_lm_batch_runs(src, bins, n, g, t, imgs, n_img, p, order, s);
}

hipError_t launch_back_runs_or_tiles(const RaySrc& src, const int16_t* bins, int64_t n, const GeomK& g, const TofK* t,
                                     float* imgs, int n_img, const float* p, const int32_t* order, const int* changes,
                                     int need, hipStream_t s) {
    const RunsOrTiles choice{changes, need};
    if (!bins) return launch_runs<kRunsOrTiles>(ModeNonTof{p}, src, n, g, imgs, order, s, 1, 0, false, choice);
    if (n_img == 1) return back_tof_lm_runs<kRunsOrTiles>(src, bins, n, g, *t, imgs, p, order, s, choice);
    return back_tof_lm_batch_runs<kRunsOrTiles>(src, bins, n, g, *t, imgs, n_img, p, order, s, choice);
}

static int sino_block(int nb) { return nb <= 64 ? 256 : 64; }  // LDS tile <= 64 KiB

// Threads of a k_fwd_tof_sino_lines workgroup: as many as leave two workgroups room in a CU's LDS, fewer where n would
// leave CUs idle; 0 if the grid's sheet does not fit
static int sino_lines_block(const GeomK& g, int64_t n) {
    const int64_t room = (80 * 1024 - (int)sizeof(LineShared) - 64) / 4 - ((int64_t)line_planes(g) * line_stride(g) + 2);
    if (room < 8 * 64) return 0;
    const int words = (int)room;
    if (words < line_plane_words(g)) return 0;
    int rays = words / 8 / 64 * 64;
    rays = rays > kSinoBlock ? kSinoBlock : rays;
    while (rays > 64 && n < (int64_t)rays * 2 * device_cus()) rays = (rays / 2 + 63) / 64 * 64;
    return rays;
}

template <int R>
static hipError_t launch_sino_lines(const RaySrc& src, int64_t n, const GeomK& g, const TofEdgeK& t, int nb, int T,
                                    const float* img, float* p, hipStream_t s) {
    const int extra = 8 * T > line_plane_words(g) ? 8 * T : line_plane_words(g);
    const size_t lds = (size_t)(line_words(g) + extra) * sizeof(float);
    const hipError_t e = hipFuncSetAttribute((const void*)k_fwd_tof_sino_lines<R>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int groups = line_groups_of(n, T, 16384);
    hipLaunchKernelGGL(k_fwd_tof_sino_lines<R>, dim3(grid_for(n, T * groups)), dim3(T), lds, s, src, n, g, t, nb, img, p,
                       kLineMinRunTof, groups);
    return hipGetLastError();
}

hipError_t launch_fwd_tof_sino(const RaySrc& src, int64_t n, const GeomK& g, const TofK& t, const TofEdgeK* te,
                               const float* img, float* p, hipStream_t s) {
    const int T = te && te->R ? sino_lines_block(g, n) : 0;
    if (T) {
        switch (te->R) {
            case 1: return launch_sino_lines<1>(src, n, g, *te, t.nb, T, img, p, s);
            case 2: return launch_sino_lines<2>(src, n, g, *te, t.nb, T, img, p, s);
            case 3: return launch_sino_lines<3>(src, n, g, *te, t.nb, T, img, p, s);
            case 4: return launch_sino_lines<4>(src, n, g, *te, t.nb, T, img, p, s);
            default: return launch_sino_lines<5>(src, n, g, *te, t.nb, T, img, p, s);
        }
    }
    const int blk = sino_block(t.nb);
    const size_t lds = (size_t)t.nb * blk * sizeof(float);
    hipLaunchKernelGGL((t.sig_ray || t.off_ray) ? k_fwd_tof_sino<true> : k_fwd_tof_sino<false>, dim3(grid_for(n, blk)),
                       dim3(blk), lds, s, src, n, g, t, img, p);
    return hipGetLastError();
}

hipError_t launch_back_tof_sino(const RaySrc& src, int64_t n, const GeomK& g, const TofK& t, const TofEdgeK* te,
                                float* img, const float* p, hipStream_t s) {
    if (te && te->R && n >= kLineRaysTof && lines_fit(g)) {
        const ModeTofSino<false> m{p, t};
        switch (te->R) {
            case 1: return launch_back_lines(LineBackTofSino<1>{p, *te, t.nb}, m, src, n, g, img, s);
            case 2: return launch_back_lines(LineBackTofSino<2>{p, *te, t.nb}, m, src, n, g, img, s);
            case 3: return launch_back_lines(LineBackTofSino<3>{p, *te, t.nb}, m, src, n, g, img, s);
            case 4: return launch_back_lines(LineBackTofSino<4>{p, *te, t.nb}, m, src, n, g, img, s);
            default: return launch_back_lines(LineBackTofSino<5>{p, *te, t.nb}, m, src, n, g, img, s);
        }
    }
    // the run/sheet kernel carries ray indices in 32 bits: the C ABI takes n < 2^31
    if (t.sig_ray || t.off_ray) {
        if (t.lut) return launch_runs(ModeTofSino<true, true>{p, t}, src, n, g, img, nullptr, s);
        return launch_runs(ModeTofSino<false, true>{p, t}, src, n, g, img, nullptr, s);
    }
    if (t.lut) return launch_runs(ModeTofSino<true>{p, t}, src, n, g, img, nullptr, s);
    return launch_runs(ModeTofSino<false>{p, t}, src, n, g, img, nullptr, s);
}

// The Gaussian bin weight w(x) = (erf(clip(x + bw/2) / (sqrt2 sigma)) - erf(clip(x - bw/2) /
// (sqrt2 sigma))) / 2, clip at +-trunc, at x_i = x0 + i dx, in float64 (the device library's erf).
__global__ void __launch_bounds__(kBlock) k_tof_gauss_table(float* __restrict__ lut, int n, double x0, double dx,
                                                           double hbw, double trunc, double inv_s2) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const double x = fma((double)i, dx, x0);
    const double a = fmin(fmax(x + hbw, -trunc), trunc), b = fmin(fmax(x - hbw, -trunc), trunc);
    lut[i] = (float)(0.5 * (erf(a * inv_s2) - erf(b * inv_s2)));
}

hipError_t launch_tof_gauss_table(float* lut, int n, double x0, double dx, double bw, double sigma, double n_sigmas,
                                  hipStream_t s) {
    hipLaunchKernelGGL(k_tof_gauss_table, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, lut, n, x0, dx, 0.5 * bw,
                       n_sigmas * sigma, 1.0 / (sqrt(2.0) * sigma));
    return hipGetLastError();
}

hipError_t launch_count(const RaySrc& src, const int16_t* bins, int64_t n, const GeomK& g,
                        const TofK& t, int32_t* counts, hipStream_t s) {
    hipLaunchKernelGGL(k_count, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, src, bins, n, g, t, counts);
    return hipGetLastError();
}

}  // namespace ppmi
