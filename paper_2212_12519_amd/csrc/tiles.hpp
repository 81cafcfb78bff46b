// Tile back projection for listmode events with few events per transaxial line.
//
// The run/sheet kernel (sheet.hpp) pays a flush per line; below some ten events per line the flush's
// memory-side float atomics are most of its time (about 21 G cache-line requests per second on this GPU,
// whatever the scope or buffer), and unsorted events pay four of them per plane sample.  Here every
// event's plane range is cut at the borders of image tiles (kTileMax^2 columns or fewer, all slices or a
// part of them), the pieces are collected per tile, and workgroups add a tile's pieces into an LDS copy of
// the tile, which is then added to the image once: the order of the events does not matter, and the image
// traffic is a few passes over the tiles instead of one request per sample pair.
//
// The LDS copy is fixed point in 64-bit integers (ds_add_u64: 5.7 lanes per cycle and CU at random
// addresses; ds_add_f64 3.0, ds_add_f32 0.33).  A unit's scale keeps its largest possible sum below 2^63
// and its largest value below 2^50, so values down to 2^-26 of the largest are added as exactly as a
// float holds them, in any order.  A piece whose values would keep fewer than kTileBits bits, or are not
// finite, is added to the image directly.
//
//   k_tile_zero    clears the per-tile counters
//   k_tile_probe   (where it is open whether the tiles pay) counts the line changes from event to event
//   k_tile_bin     one event per thread: ray setup, the event's record (64 B), its pieces counted per tile
//                  (an LDS histogram per workgroup); rays along axis 2 are scattered directly
//   k_tile_scan    one workgroup: first piece of every tile, and the work units (a tile's pieces split so
//                  that the units have similar sizes)
//   k_tile_fill    the pieces written in their tile's range (the workgroup reserves one range per tile)
//   k_tile_add     units: pieces -> LDS tile -> image
#pragma once

#include <hip/hip_runtime.h>

#include "joseph.hpp"
#include "sheet.hpp"

namespace ppmi {

constexpr int kTileMax = 24;                 // largest tile edge (columns)
constexpr int kTileMinEdge = 12;             // smallest edge before the slices are split
constexpr size_t kTileLds = 150 * 1024;      // LDS copy of a tile; one k_tile_add workgroup per CU
constexpr int kTileMaxTiles = 8192;          // LDS histogram of k_tile_bin / k_tile_fill
constexpr int kTileMaxDim = 32767;           // planes are packed in 15 bits
constexpr int kBinBlock = 256, kBinRays = 4;  // at most 1024 events of one k_tile_bin / k_tile_fill workgroup
constexpr int kAddBlock = 1024;
constexpr int kUnitMin = 2048;               // fewest pieces a unit is cut to
constexpr int kRound = 4096;                 // pieces ordered by length at a time
constexpr int kTileBits = 20;                // fewest bits a piece's largest value keeps in a tile
constexpr int kTileImages = 16;              // images of one pass over the events (batch modes)

// A tile holds the samples whose first voxel (i, j, k) (the stencil's lowest corner, from -1 on) lies in
// it: edge x edge columns by zc slices, and one more column and slice for the corner's neighbours.
struct TileGeom {
    int edge, zc;          // first-voxel range of a tile
    int zs;                // entries of a column: zc + 1
    int nt0, nt1, ntz;     // tiles per axis
    float inv_edge, inv_zc;
    __host__ __device__ int count() const { return nt0 * nt1 * ntz; }
    __host__ __device__ size_t lds_bytes() const { return (size_t)(edge + 1) * (edge + 1) * zs * 8; }
    // a / edge for 0 <= a <= 2^15: (a + 1/2) / edge stays at least 1/48 from an integer, the product's
    // rounding is below 2^-9
    __device__ int tile_of(int a) const { return (int)(((float)a + 0.5f) * inv_edge); }
    __device__ int slab_of(int a) const { return (int)(((float)a + 0.5f) * inv_zc); }
};

// An event prepared for the tile kernels.  kk: k_lo | k_hi << 15 | axis << 30 (planes whose stencil has
// its first voxel in [-1, n)), or kNoPlanes.
struct alignas(16) TileRec {
    double U0, dU, W0, dW, s0, ds;
    float cv;
    int aux;
    int l;
    uint32_t kk;
};
static_assert(sizeof(TileRec) == 64, "TileRec layout");
constexpr uint32_t kNoPlanes = 0xffffffffu;

// The workspace's parts (device pointers)
struct TileWork {
    int* head;    // [0] pieces, [1] units, [2] pieces per unit, [3] the weights' bound (float bits), [4 + b] largest |value| of image b (float
                  // bits), then the next unit to take, then the line changes that k_tile_probe found
    int* count;   // [tiles] pieces of a tile
    int* first;   // [tiles] its first piece
    int* cursor;  // [tiles] next free piece of the tile's range
    int* unit0;   // [tiles] its first unit
    TileRec* rec; // [events]
    uint2* piece; // [capacity] (record, k0 | (k1 - k0) << 16 | axis << 31)
    float* value; // [images][events of the pass] batch modes: cv times the event's value, in processing order
    int64_t capacity;
    int need;     // fewest line changes among the probed events for which the tiles are the better way (0: not asked)
    __device__ bool on() const { return need == 0 || head[5 + kTileImages] >= need; }
};

// The first plane after k (whose coordinate lies in `tile`) where the coordinate A0 + k dA has left the tile, at
// most khi + 1: the crossing by the reciprocal slope, then the exact test.
template <class F>
__device__ __forceinline__ int tile_next(double A0, double dA, double inv_dA, int tile, int size, int k, int khi,
                                         F tile_at) {
    const double edge = (double)((dA > 0.0 ? tile + 1 : tile) * size - 1);
    int kc = (int)fmin(fmax((edge - A0) * inv_dA, (double)k + 1.0), (double)khi + 1.0);  // (NaN, dA == 0: k + 1)
    while (kc > k + 1 && tile_at(kc - 1) != tile) --kc;
    while (kc <= khi && tile_at(kc) == tile) ++kc;
    return kc;
}

// The pieces of a record's plane range: f(tile, k0, k1) for each stretch inside one tile.  The first voxel of
// a sample is floor(fma(k, dU, U0)), the expression k_tile_add evaluates.  A crossing is looked up again only
// when the ray has passed it.
template <class F>
__device__ __forceinline__ void tile_walk(const TileGeom& tg, double U0, double dU, double W0, double dW, uint32_t kk,
                                          F f) {
    if (kk == kNoPlanes) return;
    const int khi = (kk >> 15) & 0x7fff;
    const bool p1 = (kk >> 30) & 1;
    auto tu_at = [&](int k) { return tg.tile_of((int)floor(fma((double)k, dU, U0)) + 1); };
    auto tz_at = [&](int k) { return tg.slab_of((int)floor(fma((double)k, dW, W0)) + 1); };
    const double inv_dU = 1.0 / dU, inv_dW = tg.ntz > 1 ? 1.0 / dW : 0.0;
    auto next_u = [&](int k, int t) {
        if (tu_at(khi) == t) return khi + 1;  // (every slope of 0 among them)
        return tile_next(U0, dU, inv_dU, t, tg.edge, k, khi, tu_at);
    };
    auto next_z = [&](int k, int t) {
        if (tg.ntz == 1 || tz_at(khi) == t) return khi + 1;
        return tile_next(W0, dW, inv_dW, t, tg.zc, k, khi, tz_at);
    };
    int k = kk & 0x7fff;
    int tp = tg.tile_of(k + 1), tu = tu_at(k), tz = tg.ntz > 1 ? tz_at(k) : 0;
    int kp = (tp + 1) * tg.edge - 1, ku = next_u(k, tu), kz = next_z(k, tz);
    while (true) {
        const int ke = min(min(kp, khi + 1), min(ku, kz));
        const int t0 = p1 ? tu : tp, t1 = p1 ? tp : tu;
        f((t0 * tg.nt1 + t1) * tg.ntz + tz, k, ke - 1);
        k = ke;
        if (k > khi) break;
        if (k == kp) ++tp, kp += tg.edge;
        if (k == ku) tu = tu_at(k), ku = next_u(k, tu);
        if (k == kz) tz = tz_at(k), kz = next_z(k, tz);
    }
}

// The cnt events from place `first` of the processing order on -> records and per-tile counts.  Batch modes: the
// record's cv is for a value of 1; n_img images (img_stride apart) receive the rays along axis 2.
template <class Mode>
__global__ void __launch_bounds__(kBinBlock) k_tile_bin(Mode m, RaySrc src, int64_t n, GeomK g, TileGeom tg,
                                                        float* __restrict__ img, const int32_t* __restrict__ order,
                                                        int64_t first, int cnt, int rays, TileWork w, int n_img,
                                                        int64_t img_stride) {
    extern __shared__ int hist[];
    __shared__ float red[4];
    __shared__ unsigned top[kTileImages];
    if (!w.on()) return;
    const int nt = tg.count();
    for (int t = threadIdx.x; t < nt; t += kBinBlock) hist[t] = 0;
    if (threadIdx.x < kTileImages) top[threadIdx.x] = 0;
    static_assert(kBinBlock == kSheetBlock, "weight_bound reduces over kSheetBlock threads");
    const float wb = m.weight_bound(red);
    __syncthreads();
    // OSEM projects here: neighbouring events, in the same L2, share the image's lines (125,000 events of a subset,
    // 13 MB image: 158 -> 143 us; without image reads the plain order is the faster, 52 against 56 us)
    const unsigned block = Mode::kReads ? xcd_block() : blockIdx.x;
    for (int e = 0; e < rays; ++e) {
        const int q = (block * rays + e) * kBinBlock + threadIdx.x;
        if ((int64_t)(block * rays + e) * kBinBlock >= cnt) break;  // block-uniform
        int64_t l = -1;
        if (q < cnt) {
            l = order ? (int64_t)order[first + q] : first + q;
            if (l < 0 || l >= n) l = -1;
        }
        RayK r;
        float cv = 0.0f;
        int ax = 0;
        const bool ok = l >= 0 && m.setup(l, src, g, r, cv, ax);
        // rays along axis 2 (none in a cylindrical scanner's data): float atomics, combined over the wave
        const bool direct = ok && r.p == 2;
        if (__ballot(direct)) {
            const int dlo = direct ? r.k_lo : (1 << 30), dhi = direct ? r.k_hi : -(1 << 30);
            const int k0 = wave_min(dlo), k1 = wave_max(dhi);
            for (int b = 0; b < n_img; ++b) {
                float c = cv;
                if constexpr (Mode::kBatch) c = direct ? cv * m.value(l, b, n) : 0.0f;
                for (int k = k0; k <= k1; ++k) {
                    const bool act = k >= dlo && k <= dhi;
                    Stencil st{};
                    float v = 0.0f;
                    if (act) {
                        st = stencil_at(r, k);
                        v = m.sample(fma((double)k, r.ds, r.s0), c, ax);
                    }
                    wave_stencil_scatter(img + b * img_stride, act && v != 0.0f, r, st, v);
                }
            }
        }
        for (int b = 0; b < n_img; ++b) {  // largest finite |value|, per image
            float c = ok ? cv : 0.0f;
            if constexpr (Mode::kBatch) {
                c = ok ? cv * m.value(l, b, n) : 0.0f;
                if (q < cnt) w.value[(int64_t)b * cnt + q] = c;
            }
            float a = m.mag(c, ax) * wb;
            if (!(a <= FLT_MAX)) a = 0.0f;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) a = fmaxf(a, __shfl_xor(a, off, 64));
            if (__lane_id() == 0) atomicMax(&top[b], __float_as_uint(a));
        }
        if (q < cnt) {
            TileRec rec{};
            rec.kk = kNoPlanes;
            if (ok && !direct) {
                // the planes whose first voxel lies in [-1, n): the conservative end planes may lie outside
                auto out = [&](int k) {
                    const int i = (int)floor(fma((double)k, r.dU, r.U0)), j = (int)floor(fma((double)k, r.dW, r.W0));
                    return i < -1 || i >= r.nu || j < -1 || j >= r.nw;
                };
                int lo = r.k_lo, hi = r.k_hi;
                while (lo <= hi && out(lo)) ++lo;
                while (lo <= hi && out(hi)) --hi;
                if (lo <= hi) {
                    rec.U0 = r.U0, rec.dU = r.dU, rec.W0 = r.W0, rec.dW = r.dW, rec.s0 = r.s0, rec.ds = r.ds;
                    rec.cv = cv;
                    rec.aux = ax;
                    rec.l = (int)l;
                    rec.kk = (uint32_t)lo | ((uint32_t)hi << 15) | ((uint32_t)r.p << 30);
                    tile_walk(tg, rec.U0, rec.dU, rec.W0, rec.dW, rec.kk,
                              [&](int t, int, int) { atomicAdd(&hist[t], 1); });
                }
            }
            w.rec[q] = rec;
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < nt; t += kBinBlock)
        if (hist[t]) atomicAdd(&w.count[t], hist[t]);
    if (blockIdx.x == 0 && threadIdx.x == 0) w.head[3] = __float_as_int(wb);
    if (threadIdx.x < n_img && top[threadIdx.x])
        atomicMax(reinterpret_cast<unsigned*>(w.head) + 4 + threadIdx.x, top[threadIdx.x]);
}

constexpr double kMagic = 6755399441055744.0;  // 1.5 * 2^52

// A sample of a piece that does not use the LDS tile: its four values into the image.
__device__ inline void tile_direct(float* __restrict__ img, const GeomK& g, bool p1, double kd, const TileRec& r,
                                   float v) {
    const double U = fma(kd, r.dU, r.U0), W = fma(kd, r.dW, r.W0), fi = floor(U), fj = floor(W);
    const float fu = (float)(U - fi), fw = (float)(W - fj), gu = 1.0f - fu, gw = 1.0f - fw;
    const int i = (int)fi, j = (int)fj;
    const int su = p1 ? g.stride[0] : g.stride[1], nu = p1 ? g.n[0] : g.n[1], nw = g.n[2];
    float* at = img + (int)kd * (p1 ? g.stride[1] : g.stride[0]) + i * su + j;
    const bool i0 = i >= 0 && i < nu, i1 = i + 1 < nu, j0 = j >= 0 && j < nw, j1 = j + 1 < nw;
    if (i0 && j0) unsafeAtomicAdd(at, gu * gw * v);
    if (i0 && j1) unsafeAtomicAdd(at + 1, gu * fw * v);
    if (i1 && j0) unsafeAtomicAdd(at + su, fu * gw * v);
    if (i1 && j1) unsafeAtomicAdd(at + su + 1, fu * fw * v);
}

// Units taken from a counter: the unit's pieces into the LDS tile, the tile into the image.  1.5 M clinical TOF
// events (142 M plane samples, 15 M pieces): 0.45 ms, of which the vector ALU is busy about 60% (54
// instructions per 64 samples of a wave, all lanes on) and the LDS 50% (bank conflicts are two thirds of it);
// the rest is the barriers of the rounds and the flush.  Without the ordering by length 0.50 ms, with float64
// entries 0.68 ms.
// The lanes of a wave take pieces of one length that lie far apart in the unit (neighbouring events,
// which a presort puts on nearly the same line, would meet in the same LDS entries).
template <class Mode>
__global__ void __launch_bounds__(kAddBlock) k_tile_add(Mode m, int64_t cnt_events, GeomK g, TileGeom tg, TileWork w,
                                                        float* __restrict__ img, int n_img, int64_t img_stride) {
    extern __shared__ unsigned long long tile[];
    if (!w.on()) return;
    typedef __attribute__((address_space(3))) unsigned long long lds_u64;
    const int T1 = tg.edge + 1, zs = tg.zs, nt = tg.count();
    const int total = T1 * T1 * zs;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    lds_u64* const lt = (lds_u64*)tile;
    __shared__ int bin[kTileMax + 1], s_job;
    __shared__ unsigned short sorted[kRound];
    for (int e = threadIdx.x; e < total; e += kAddBlock) tile[e] = 0;
    Mode ms = m;
    ms.to_vgprs();
    const int n_units = w.head[1], per = w.head[2];
    const float weight = __int_as_float(w.head[3]);
    const float inv_zs = 1.0f / (float)zs, inv_t1 = 1.0f / (float)T1;
    __syncthreads();
    while (true) {
        if (threadIdx.x == 0) s_job = atomicAdd(&w.head[4 + kTileImages], 1);
        __syncthreads();
        const int64_t job = (unsigned)s_job;
        if (job >= (int64_t)n_units * n_img) break;
        const int b = (int)(job / n_units), unit = (int)(job - (int64_t)b * n_units);
        int lo = 0, hi = nt - 1;  // the tile whose units hold this one (block-uniform)
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (w.unit0[mid] <= unit) lo = mid; else hi = mid - 1;
        }
        const int t0 = lo / (tg.nt1 * tg.ntz), rest = lo - t0 * tg.nt1 * tg.ntz;
        const int t1 = rest / tg.ntz, tz = rest - t1 * tg.ntz;
        const int o0 = t0 * tg.edge - 1, o1 = t1 * tg.edge - 1, oz = tz * tg.zc - 1;
        const int all = w.count[lo], nu = (all + per - 1) / per, each = (all + nu - 1) / nu;
        const int skip = (unit - w.unit0[lo]) * each, first = w.first[lo] + skip, cnt = min(each, all - skip);
        const int origin = (o0 * T1 + o1) * zs + oz;
        float* const out = img + b * img_stride;
        // a voxel takes at most one value of a piece: scale = 2^sx with top * scale <= 2^50, cnt * top * scale < 2^63
        int ex = 0;
        frexpf(__int_as_float(w.head[4 + b]), &ex);  // top < 2^ex (half of that to spare for the bounds' own rounding)
        const int sx = min(max(min(49, 61 - (32 - __clz(cnt))) - ex, -126), 126);
        const float scale = ldexpf(1.0f, sx);
        for (int r0 = 0; r0 < cnt; r0 += kRound) {
            const int nr = min(cnt - r0, kRound);
            // the round's pieces in order of falling length (counting sort), so that the 64 pieces of a wave
            // have the same number of samples
            if (threadIdx.x < kTileMax + 1) bin[threadIdx.x] = 0;
            __syncthreads();
            constexpr int kEach = kRound / kAddBlock;
            int len[kEach], rank[kEach];
#pragma unroll
            for (int j = 0; j < kEach; ++j) {
                const int i = lane * (kRound / 64) + wave * kEach + j;
                if (i < nr) {
                    len[j] = kTileMax - (int)((w.piece[first + r0 + i].y >> 16) & 0x7fff);
                    rank[j] = atomicAdd(&bin[len[j]], 1);
                }
            }
            __syncthreads();
            if (wave == 0) {  // exclusive prefix sums of the bins
                const int v = lane <= kTileMax ? bin[lane] : 0;
                int sum = v;
#pragma unroll
                for (int off = 1; off < 32; off <<= 1) {
                    const int o = __shfl_up(sum, off, 64);
                    if (lane >= off) sum += o;
                }
                if (lane <= kTileMax) bin[lane] = sum - v;
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < kEach; ++j) {
                const int i = lane * (kRound / 64) + wave * kEach + j;
                if (i < nr) sorted[bin[len[j]] + rank[j]] = (unsigned short)i;
            }
            __syncthreads();
            // this thread's pieces of the round, their records loaded one piece ahead
            uint2 pcs[kEach];
#pragma unroll
            for (int j = 0; j < kEach; ++j) {
                // (waves in turn forwards and backwards, so that each gets about the same sum of lengths)
                const int q = ((j & 1 ? kAddBlock / 64 - 1 - wave : wave) + j * (kAddBlock / 64)) * 64 + lane;
                pcs[j] = q < nr ? w.piece[first + r0 + sorted[q]] : make_uint2(0u, kNoPlanes);
            }
            // batch: the values come from k_tile_bin's copy in processing order, of which neighbouring pieces share
            // lines (10 M events, 8 images: 15.4 -> 13.2 ms, 0.81 -> 0.31 G L2 misses against the caller's arrays)
            float value[kEach];
            if constexpr (Mode::kBatch)
#pragma unroll
                for (int j = 0; j < kEach; ++j) value[j] = w.value[b * cnt_events + pcs[j].x];
            TileRec next = w.rec[pcs[0].x];
#pragma unroll
            for (int j = 0; j < kEach; ++j) {
                const uint2 pc = pcs[j];
                const TileRec rec = next;
                if (j + 1 < kEach) next = w.rec[pcs[j + 1 < kEach ? j + 1 : j].x];
                if (pc.y == kNoPlanes) break;
                float cv = rec.cv;
                if constexpr (Mode::kBatch) {
                    cv = value[j];
                    if (cv == 0.0f) continue;
                }
                const float bound = ms.mag(cv, rec.aux) * weight * scale;
                const int k0 = pc.y & 0x7fff, steps = (pc.y >> 16) & 0x7fff;
                const bool p1 = pc.y >> 31;
                double kd = (double)k0;
                if (!(bound >= (float)(1 << kTileBits) && bound <= 0x1p50f)) {
                    for (int c = 0; c <= steps; ++c, kd += 1.0)
                        tile_direct(out, g, p1, kd, rec, ms.sample(fma(kd, rec.ds, rec.s0), cv, rec.aux));
                    continue;
                }
                cv *= scale;
                // entry of the sample's first voxel: (i_p - o_p) sp + (i_u - o_u) su + j - oz, in float64 (exact);
                // added to 1.5 * 2^52 its low word is the integer
                const int sp = p1 ? zs : T1 * zs, su = p1 ? T1 * zs : zs;
                const double su_d = (double)su, sp_d = (double)sp;
                double ad = fma(kd, sp_d, kMagic - (double)origin);
                for (int c = 0; c <= steps; ++c, kd += 1.0, ad += sp_d) {
                    const double U = fma(kd, rec.dU, rec.U0), W = fma(kd, rec.dW, rec.W0);
                    const double fi = floor(U), fj = floor(W), fu = U - fi, fw = W - fj;
                    const double v = (double)ms.sample(fma(kd, rec.ds, rec.s0), cv, rec.aux);
                    lds_u64* const at = lt + __double2loint(fma(fi, su_d, ad + fj));
                    const double vu = fu * v, vg = v - vu, v01 = fw * vg, v11 = fw * vu;
                    auto add = [&](lds_u64* a, double x) {  // x rounded to an integer (|x| < 2^51)
                        __hip_atomic_fetch_add(a, __double_as_longlong(x + kMagic) - __double_as_longlong(kMagic),
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    };
                    add(at, vg - v01);
                    add(at + 1, v01);
                    add(at + su, vu - v11);
                    add(at + su + 1, v11);
                }
            }
            __syncthreads();
        }
        const double inv_scale = ldexp(1.0, -sx);
        for (int e = threadIdx.x; e < total; e += kAddBlock) {
            const long long sum = (long long)tile[e];
            tile[e] = 0;
            if (sum == 0) continue;
            const float v = (float)((double)sum * inv_scale);
            const int c = (int)(((float)e + 0.5f) * inv_zs), j = oz + e - c * zs;
            const int c0 = (int)(((float)c + 0.5f) * inv_t1), i0 = o0 + c0, i1 = o1 + c - c0 * T1;
            if ((unsigned)i0 < (unsigned)g.n[0] && (unsigned)i1 < (unsigned)g.n[1] && (unsigned)j < (unsigned)g.n[2])
                unsafeAtomicAdd(out + i0 * g.stride[0] + i1 * g.stride[1] + j, v);
        }
        __syncthreads();
    }
}

}  // namespace ppmi
