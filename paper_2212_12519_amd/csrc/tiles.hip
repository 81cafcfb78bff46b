// Host side and small kernels of the tile back projection (tiles.hpp).
#include <hip/hip_runtime.h>

#include <cmath>

#include "launch.hpp"
#include "tiles.hpp"

namespace ppmi {

__global__ void k_tile_zero(TileWork w, int nt, bool first) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nt) w.count[i] = 0;
    if (i <= kTileImages + (first ? 1 : 0)) w.head[4 + i] = 0;  // (what k_tile_probe found holds for every pass)
}

// Events of kProbes places of the processing order that lie on another transaxial line than the next one (in either
// direction)
constexpr int kProbes = 16384;

__global__ void __launch_bounds__(256) k_tile_probe(RaySrc src, int64_t n, const int32_t* __restrict__ order, TileWork w) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    const int64_t q = min((int64_t)i * n / kProbes, n - 2);
    const int64_t a = order ? order[q] : q, b = order ? order[q + 1] : q + 1;
    bool same = false;
    const float *s0, *e0, *s1, *e1;
    if (a >= 0 && a < n && b >= 0 && b < n && src.ends(a, s0, e0) && src.ends(b, s1, e1))
        same = (s0[0] == s1[0] && s0[1] == s1[1] && e0[0] == e1[0] && e0[1] == e1[1]) ||
               (s0[0] == e1[0] && s0[1] == e1[1] && e0[0] == s1[0] && e0[1] == s1[1]);
    const unsigned long long other = __ballot(!same);
    if (__lane_id() == 0) atomicAdd(&w.head[5 + kTileImages], __popcll(other));
}

// Exclusive prefix sums over the tiles: every tile's first piece, and its first unit where a unit has at
// most `per` pieces, per chosen so that about `units` units hold them all.
__global__ void __launch_bounds__(1024) k_tile_scan(int nt, int units, TileWork w) {
    __shared__ int part[2][1024];
    if (!w.on()) return;
    const int tid = threadIdx.x;
    const int each = (nt + 1023) / 1024, t_lo = min(nt, tid * each), t_hi = min(nt, t_lo + each);
    auto scan = [&](int v, int* buf) {  // inclusive prefix sum over the workgroup
        buf[tid] = v;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {
            const int o = tid >= off ? buf[tid - off] : 0;
            __syncthreads();
            buf[tid] += o;
            __syncthreads();
        }
        return buf[tid];
    };
    int sum = 0;
    for (int t = t_lo; t < t_hi; ++t) sum += w.count[t];
    int at = scan(sum, part[0]) - sum;
    const int total = part[0][1023];
    const int per = max((total + units - 1) / units, kUnitMin);
    int nu = 0;
    for (int t = t_lo; t < t_hi; ++t) {
        w.first[t] = at;
        w.cursor[t] = at;
        at += w.count[t];
        nu += (w.count[t] + per - 1) / per;
    }
    int ua = scan(nu, part[1]) - nu;
    for (int t = t_lo; t < t_hi; ++t) {
        w.unit0[t] = ua;
        ua += (w.count[t] + per - 1) / per;
    }
    if (tid == 0) {
        w.head[0] = total;
        w.head[1] = part[1][1023];
        w.head[2] = per;
    }
}

// The records' pieces into their tiles' ranges: the workgroup counts its pieces per tile, reserves one
// stretch of each tile's range and writes them there.
__global__ void __launch_bounds__(kBinBlock) k_tile_fill(TileGeom tg, int cnt, int rays, TileWork w) {
    extern __shared__ int hist[];
    if (!w.on()) return;
    const int nt = tg.count();
    for (int t = threadIdx.x; t < nt; t += kBinBlock) hist[t] = 0;
    __syncthreads();
    auto each = [&](auto f) {
        for (int e = 0; e < rays; ++e) {
            const int q = (blockIdx.x * rays + e) * kBinBlock + threadIdx.x;
            if (q >= cnt) break;
            const TileRec& r = w.rec[q];
            const uint32_t kk = r.kk;
            tile_walk(tg, r.U0, r.dU, r.W0, r.dW, kk, [&](int t, int k0, int k1) {
                f(t, make_uint2((unsigned)q, (unsigned)k0 | ((unsigned)(k1 - k0) << 16) | ((kk >> 30) << 31)));
            });
        }
    };
    each([&](int t, uint2) { atomicAdd(&hist[t], 1); });
    __syncthreads();
    for (int t = threadIdx.x; t < nt; t += kBinBlock)
        if (hist[t]) hist[t] = atomicAdd(&w.cursor[t], hist[t]);
    __syncthreads();
    each([&](int t, uint2 piece) {
        const int at = atomicAdd(&hist[t], 1);
        if (at < w.capacity) w.piece[at] = piece;  // always: capacity bounds the pieces of any event
    });
}

// Tile size: the largest edge whose LDS copy fits, with the slices whole if the edge stays at least
// kTileMinEdge (fewer pieces per event and longer rows to flush), else cut in as few parts as allow it.
static bool tile_geom(const GeomK& g, TileGeom& tg) {
    if (g.n[0] > kTileMaxDim || g.n[1] > kTileMaxDim || g.n[2] > kTileMaxDim) return false;
    const int starts = g.n[2] + 1;  // first slices -1 .. n2 - 1
    for (int parts = 1;; ++parts) {
        tg.zc = (starts + parts - 1) / parts;
        tg.zs = tg.zc + 1;
        int e = (int)std::sqrt((double)(kTileLds / 8) / tg.zs) - 1;
        e = e < kTileMax ? e : kTileMax;
        if (e >= kTileMinEdge || tg.zc <= 8) {
            if (e < 4) return false;
            tg.edge = e;
            break;
        }
    }
    tg.nt0 = g.n[0] / tg.edge + 1;
    tg.nt1 = g.n[1] / tg.edge + 1;
    tg.ntz = g.n[2] / tg.zc + 1;
    tg.inv_edge = 1.0f / (float)tg.edge;
    tg.inv_zc = 1.0f / (float)tg.zc;
    return (int64_t)tg.nt0 * tg.nt1 * tg.ntz <= kTileMaxTiles;
}

// An upper bound of one event's pieces: every piece but the first begins where the plane, the in-plane
// coordinate or the slice crosses a tile border, and along a ray none of the three moves further (in mm)
// than the principal coordinate.
static int pieces_bound(const GeomK& g, const TileGeom& tg, const TofK* t) {
    const double h = std::fmin(g.h[0], g.h[1]);
    double planes = g.n[0] > g.n[1] ? g.n[0] : g.n[1];
    if (t && !t->sig_ray) planes = std::fmin(planes, (t->hi - t->lo) / h + 4.0);
    const double mm = planes * std::fmax(g.h[0], g.h[1]);
    const double u = std::fmin(mm / h, (double)(g.n[0] > g.n[1] ? g.n[0] : g.n[1]) + 1.0);
    const double z = tg.ntz > 1 ? std::fmin(mm / g.h[2], (double)g.n[2] + 1.0) / tg.zc + 1.0 : 0.0;
    return (int)std::ceil(planes / tg.edge + 1.0) + (int)std::ceil(u / tg.edge + 1.0) + (int)std::ceil(z) + 1;
}

// Most events the tiles take, on a scanner of 760 crystals a ring (tile_need: on others).  The sheets' cost hardly grows
// with the events while a line has few of them (clinical grid, 58.5 mm TOF, presorted: 3.9 ms at 1.5 M events, 5.6 ms at 15 M), the tiles' is
// proportional to the plane samples (0.71 and 6.3 ms; non-TOF 1.15 and 11 ms against 5.2 and 6.4 ms); both
// limits lie a little below the crossings (serving grid 128 x 128 x 64: 13 M and 8 M).
constexpr int64_t kTileEventsTof = 10'000'000;
constexpr int64_t kTileEventsNonTof = 7'000'000;
// Batches of images: a sheet is flushed at the end of every group and image, so the crossing lies higher (two images
// of 128 x 128 x 64: 7.5 against 9.5 ms at 15 M events, 12.5 against 11.6 at 25 M; eight: 23.5 and 36.7, 40.8 and 46.9)
constexpr int64_t kTileEventsBatch = 20'000'000;
constexpr int64_t kTileRaysList = 5'700'000;

// Below those limits the sheets are still the better way where many events share a line.  Their time is about
// kSheetsMs + line changes * flush + n e, the tiles' n t, and t - e (ns) hardly depends on the scanner: 0.28 with a TOF window of
// 107 planes, 0.2 with 63, 0.62 without TOF in 215 planes, 0.13 an image of a batch; a flush of 215 x 71 entries takes 46
// ns (66 without TOF).  So few events go to the tiles unasked, for more the changes are counted.  Presorted events of a
// ring of 128 crystals (128 x 128 x 64, 6.9 M): tiles 2.25 ms (4.4 without TOF), sheets 1.66 (2.1); of 360 crystals (215 x
// 215 x 71, 6.9 M) 3.0 (5.4) and 2.3 (2.5) ms, of 760 crystals 2.9 and 4.6 ms, 1 M of 360 crystals 0.47 and 1.5 ms.
constexpr double kSheetsMs = 0.9;

// TileWork::need for n events
static int tile_need(int64_t n, const GeomK& g, const TofK* t, int n_img) {
    if (g.n[2] > kSheetMaxW || n < 2) return 0;  // no sheets
    double planes = g.n[0] > g.n[1] ? g.n[0] : g.n[1];
    const double flush = (t ? 46.0 : 66.0) * planes * g.n[2] / (215.0 * 71.0);
    if (t && !t->sig_ray) planes = std::fmin(planes, (t->hi - t->lo) / std::fmin(g.h[0], g.h[1]));
    const double more = n_img > 1 ? 0.13 : t ? 0.12 + 0.0015 * planes : 0.3 + 0.0015 * planes;  // t - e, ns
    const double share = (more - kSheetsMs * 1e6 / (double)n) / flush;  // line changes an event
    return share <= 0.0 ? 0 : (int)std::fmin(std::ceil(share * kProbes), kProbes + 1.0);
}

static size_t up256(size_t b) { return (b + 255) & ~size_t(255); }

static size_t tile_layout(int64_t events, int tiles, int bound, int n_img, char* base, TileWork& w) {
    size_t at = 0;
    auto take = [&](size_t bytes) {
        char* p = base + at;
        at += up256(bytes);
        return p;
    };
    w.need = 0;
    w.head = reinterpret_cast<int*>(take((6 + kTileImages) * 4));
    w.count = reinterpret_cast<int*>(take((size_t)tiles * 4));
    w.first = reinterpret_cast<int*>(take((size_t)tiles * 4));
    w.cursor = reinterpret_cast<int*>(take((size_t)tiles * 4));
    w.unit0 = reinterpret_cast<int*>(take((size_t)tiles * 4));
    w.rec = reinterpret_cast<TileRec*>(take((size_t)events * sizeof(TileRec)));
    w.piece = reinterpret_cast<uint2*>(take((size_t)events * bound * 8));
    w.value = n_img > 1 ? reinterpret_cast<float*>(take((size_t)events * (n_img < kTileImages ? n_img : kTileImages) * 4))
                        : nullptr;
    w.capacity = events * bound;
    return at;
}

constexpr int64_t kTileEventsMost = 40'000'000;

// Events of one pass over the tiles: as many as kTilePassBytes of workspace hold, in passes of equal size.  A pass costs
// its launches and a flush of every tile, some 60 us beside the 5 ms and more that so many events take.
constexpr size_t kTilePassBytes = size_t(4) << 30;

static int64_t tile_pass(int64_t n, const TileGeom& tg, int bound, int n_img) {
    TileWork w;
    const size_t bytes = tile_layout(n, tg.count(), bound, n_img, nullptr, w);
    const int64_t passes = (int64_t)((bytes + kTilePassBytes - 1) / kTilePassBytes);
    return (n + passes - 1) / passes;
}

// 0: a grid the tiles do not suit, or more events than their counts (32 bits) or 16 GB of records and pieces hold
size_t tile_bytes(int64_t n, const GeomK& g, const TofK* t, int n_img) {
    TileGeom tg;
    if (n <= 0 || n > kTileEventsMost || !tile_geom(g, tg)) return 0;
    TileWork w;
    const int bound = pieces_bound(g, tg, t);
    const size_t bytes = tile_layout(n, tg.count(), bound, n_img, nullptr, w);
    if (w.capacity > INT32_MAX || bytes > (size_t(16) << 30)) return 0;
    return tile_layout(tile_pass(n, tg, bound, n_img), tg.count(), bound, n_img, nullptr, w);
}

// Grids of more slices than a sheet holds have no other way than float atomics (12 M presorted TOF events, 160
// slices: 28 ms), so the tiles take all they can there, of a ray list what is left below the line kernels' size.
size_t tile_workspace_bytes(int64_t n, const GeomK& g, const TofK* t, bool listmode, int n_img) {
    const bool sheets = g.n[2] <= kSheetMaxW;
    const int64_t most = !sheets ? (listmode ? kTileEventsMost : kTileRaysList) : !listmode ? 0
                         : n_img > 1 ? kTileEventsBatch : t ? kTileEventsTof : kTileEventsNonTof;
    return n <= most ? tile_bytes(n, g, t, n_img) : 0;
}

// all_img: the images of the whole call, for which the workspace was laid out
template <class Mode>
static hipError_t launch_tiles(const Mode& m, const RaySrc& src, int64_t n, const GeomK& g, const TofK* t, float* img,
                               int n_img, int all_img, const int32_t* order, void* ws, int cus, hipStream_t s, int need,
                               TileWork& w) {
    TileGeom tg;
    if (!tile_geom(g, tg)) return hipErrorInvalidValue;
    const int nt = tg.count(), bound = pieces_bound(g, tg, t);
    const int64_t pass = tile_pass(n, tg, bound, all_img);
    tile_layout(pass, nt, bound, all_img, static_cast<char*>(ws), w);
    w.need = need;
    const size_t lds = tg.lds_bytes(), hist = (size_t)nt * 4;
    hipError_t e = hipFuncSetAttribute((const void*)k_tile_add<Mode>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
    const int64_t stride = (int64_t)g.n[0] * g.n[1] * g.n[2];
    for (int64_t first = 0; first < n; first += pass) {
        const int cnt = (int)(n - first < pass ? n - first : pass);
        // four workgroups per CU where there are events for them, up to kBinRays events per thread
        const int each = (cnt + 4 * cus * kBinBlock - 1) / (4 * cus * kBinBlock);
        const int rays = each < kBinRays ? each : kBinRays;
        const dim3 bins((unsigned)((cnt + kBinBlock * rays - 1) / (kBinBlock * rays)));
        hipLaunchKernelGGL(k_tile_zero, dim3((nt + 255) / 256), dim3(256), 0, s, w, nt, first == 0);
        if (need && first == 0) hipLaunchKernelGGL(k_tile_probe, dim3(kProbes / 256), dim3(256), 0, s, src, n, order, w);
        hipLaunchKernelGGL(k_tile_bin<Mode>, bins, dim3(kBinBlock), hist, s, m, src, n, g, tg, img, order, first, cnt, rays,
                           w, n_img, stride);
        // about three units per CU: a unit's flush writes its whole tile (some 15 us at 320 G values/s for the
        // chip), more units balance better (400 k events: 158 us of adding with 2 or 3 per CU, 206 with 6)
        hipLaunchKernelGGL(k_tile_scan, dim3(1), dim3(1024), 0, s, nt, 3 * cus, w);
        hipLaunchKernelGGL(k_tile_fill, bins, dim3(kBinBlock), hist, s, tg, cnt, rays, w);
        hipLaunchKernelGGL(k_tile_add<Mode>, dim3(cus), dim3(kAddBlock), lds, s, m, (int64_t)cnt, g, tg, w, img, n_img,
                           stride);
    }
    return hipGetLastError();
}

// The tiles, and where it is open whether they pay the run/sheet kernel too, one of which then does nothing
template <class Mode>
static hipError_t launch_either(const Mode& m, const RaySrc& src, const int16_t* bins, int64_t n, const GeomK& g,
                                const TofK* t, float* imgs, int n_img, int all_img, const float* p,
                                const int32_t* order, void* ws, int cus, hipStream_t s) {
    TileWork w;
    const int need = tile_need(n, g, t, all_img);
    const hipError_t e = launch_tiles(m, src, n, g, t, imgs, n_img, all_img, order, ws, cus, s, need, w);
    if (e != hipSuccess || !need) return e;
    return launch_back_runs_or_tiles(src, bins, n, g, t, imgs, n_img, p, order, w.head + 5 + kTileImages, need, s);
}

template <int Form, bool PerRay>
static hipError_t launch_tiles_lm(const RaySrc& src, const int16_t* bins, int64_t n, const GeomK& g, const TofK& t,
                                  float* imgs, int n_img, const float* p, const int32_t* order, void* ws, int cus,
                                  hipStream_t s) {
    if (n_img == 1)
        return launch_either(ModeTofLm<Form, PerRay>{p, bins, t}, src, bins, n, g, &t, imgs, 1, 1, p, order, ws, cus, s);
    const int64_t nv = (int64_t)g.n[0] * g.n[1] * g.n[2];
    for (int b = 0; b < n_img; b += kTileImages) {
        const float* pb = p + (int64_t)b * n;
        const hipError_t e = launch_either(ModeTofLm<Form, PerRay, true>{pb, bins, t}, src, bins, n, g, &t, imgs + b * nv,
                                           n_img - b < kTileImages ? n_img - b : kTileImages, n_img, pb, order, ws, cus,
                                           s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_back_tiles(const RaySrc& src, const int16_t* bins, int64_t n, const GeomK& g, const TofK* t,
                             float* imgs, int n_img, const float* p, const int32_t* order, void* ws, int cus,
                             hipStream_t s) {
    if (!bins) return launch_either(ModeNonTof{p}, src, nullptr, n, g, nullptr, imgs, 1, 1, p, order, ws, cus, s);
    const int form = tof_form(*t);
    if (t->sig_ray || t->off_ray) {
        if (form == kFormLut) return launch_tiles_lm<kFormLut, true>(src, bins, n, g, *t, imgs, n_img, p, order, ws, cus, s);
        if (form == kFormPoly) return launch_tiles_lm<kFormPoly, true>(src, bins, n, g, *t, imgs, n_img, p, order, ws, cus, s);
        return launch_tiles_lm<kFormErf, true>(src, bins, n, g, *t, imgs, n_img, p, order, ws, cus, s);
    }
    if (form == kFormLut) return launch_tiles_lm<kFormLut, false>(src, bins, n, g, *t, imgs, n_img, p, order, ws, cus, s);
    if (form == kFormPoly) return launch_tiles_lm<kFormPoly, false>(src, bins, n, g, *t, imgs, n_img, p, order, ws, cus, s);
    return launch_tiles_lm<kFormErf, false>(src, bins, n, g, *t, imgs, n_img, p, order, ws, cus, s);
}

hipError_t launch_osem_tiles(const RaySrc& src, const int16_t* bins, int64_t n, const GeomK& g, const TofK& t,
                             const float* x, float bg, float* acc, void* ws, int cus, hipStream_t s) {
    const int form = tof_form(t);
    TileWork w;
    auto tiles = [&](const auto& m) { return launch_tiles(m, src, n, g, &t, acc, 1, 1, nullptr, ws, cus, s, 0, w); };
    if (form == kFormLut) return tiles(ModeOsem<kFormLut>{x, bins, bg, t});
    if (form == kFormPoly) return tiles(ModeOsem<kFormPoly>{x, bins, bg, t});
    return tiles(ModeOsem<kFormErf>{x, bins, bg, t});
}

}  // namespace ppmi
