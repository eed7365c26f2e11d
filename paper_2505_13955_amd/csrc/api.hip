// C ABI of libxct.so: argument validation, per-geometry device tables and
// dispatch of the filter, back-projection, forward-projection and reduction
// kernels.  See include/xct.h for the contract of every entry point.
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstring>
#include <limits>
#include <memory>
#include <mutex>
#include <string>
#include <unordered_map>
#include <vector>

#include "xct_internal.h"

using namespace xct;

namespace {

thread_local int g_last_hip = 0;

int hip_fail(hipError_t e)
{
    g_last_hip = (int)e;
    return XCT_EHIP;
}

// Stream-ordered scratch: the forward projector's four-slice copies and the
// back-projector's split tables take at most kQuadBytes at a time, partial
// images at most kPartBytes, and the device's default pool keeps up to both
// between calls instead of returning them at each synchronisation.
constexpr int64_t kQuadBytes = (int64_t)1 << 30;
constexpr int64_t kPartBytes = (int64_t)1 << 28;

std::mutex g_pool_mu;
std::vector<int> g_pool_seen, g_pool_raised;  // devices

// Raises the current device's default pool to that, once; a larger threshold
// of the caller's stays.
void keep_stream_pool()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return;
    std::lock_guard<std::mutex> lock(g_pool_mu);
    if (std::find(g_pool_seen.begin(), g_pool_seen.end(), dev) != g_pool_seen.end()) return;
    g_pool_seen.push_back(dev);
    hipMemPool_t pool;
    uint64_t held = 0, keep = (uint64_t)(kQuadBytes + kPartBytes);
    if (hipDeviceGetDefaultMemPool(&pool, dev) != hipSuccess) return;
    if (hipMemPoolGetAttribute(pool, hipMemPoolAttrReleaseThreshold, &held) != hipSuccess || held >= keep) return;
    if (hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep) == hipSuccess) g_pool_raised.push_back(dev);
}

// Gives back what those pools hold without use.
void trim_stream_pools()
{
    std::lock_guard<std::mutex> lock(g_pool_mu);
    for (int dev : g_pool_raised) {
        hipMemPool_t pool;
        if (hipDeviceGetDefaultMemPool(&pool, dev) == hipSuccess) (void)hipMemPoolTrimTo(pool, 0);
    }
}

bool dtype_ok(int t) { return t == XCT_F32 || t == XCT_F16 || t == XCT_BF16; }
size_t dtype_size(int t) { return t == XCT_F32 ? 4 : 2; }

// ---------------------------------------------------------------- validation

int check_geometry(const xct_geometry *g, bool need_angles)
{
    if (!g) return XCT_EINVAL;
    if (g->n_angles <= 0 || g->n_det <= 0 || g->nx <= 0 || g->ny <= 0) return XCT_EINVAL;
    if (!std::isfinite(g->det_pitch) || !(g->det_pitch > 0)) return XCT_EINVAL;
    if (!std::isfinite(g->pixel_size) || !(g->pixel_size > 0)) return XCT_EINVAL;
    if (!std::isfinite(g->center)) return XCT_EINVAL;
    if (need_angles) {
        if (!g->angles) return XCT_EINVAL;
        for (int k = 0; k < g->n_angles; ++k)
            if (!std::isfinite(g->angles[k])) return XCT_EINVAL;
    }
    if (g->n_det > 65536 || g->nx > 65536 || g->ny > 65536 || g->n_angles > (1 << 20))
        return XCT_ETOOBIG;
    const double ratio = g->pixel_size / g->det_pitch;
    if (ratio > 16.0 || ratio < 1.0 / 16.0) return XCT_ETOOBIG;
    if (std::fabs(g->center) > 1e6) return XCT_ETOOBIG;
    return XCT_OK;
}

int check_slices(const xct_geometry *g, int32_t n_slices)
{
    if (n_slices <= 0) return XCT_EINVAL;
    const double lim = 4.0e18;
    if ((double)n_slices * g->n_angles * g->n_det > lim) return XCT_ETOOBIG;
    if ((double)n_slices * g->nx * g->ny > lim) return XCT_ETOOBIG;
    return XCT_OK;
}

// ---------------------------------------------------------------- device tables
//
// Per-geometry tables (trigonometry, filter spectra, forward-projector plans,
// blur taps, redundancy weights) are built on the host in FP64 and cached on
// the device.  One cache entry is one device allocation holding its tables at
// 256-byte offsets.  Its upload is ordered on the stream of the call that
// creates it (an asynchronous copy from pinned host staging, kept with the
// entry), and an event marks its completion so that calls on other streams
// wait for it.  The cache is bounded: past kCacheEntries entries or
// kCacheBytes bytes the least recently used entries that no call is using are
// freed (hipFree, which waits for the device).

constexpr size_t kCacheBytes = (size_t)1 << 30;
constexpr size_t kCacheEntries = 256;

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Entry {
    char *dev = nullptr;        // device allocation (all tables of the entry)
    void *host = nullptr;       // pinned staging of the upload
    hipEvent_t ready = nullptr; // recorded after the upload, on the creating call's stream
    bool done = false;          // the upload is known to be complete
    size_t bytes = 0;
    uint64_t tick = 0;
    size_t off[2] = {0, 0};     // offsets of the entry's tables in `dev`
    // forward-projector plan metadata
    int n_blocks = 0;
    bool fp_four = false;  // every angle block has a four-slice staging shape
    // filter length
    int L = 0, lg = 0;
    template <typename T>
    T *table(int i) const { return reinterpret_cast<T *>(dev + off[i]); }
};
typedef std::shared_ptr<Entry> EntryRef;

std::mutex g_mu;
std::unordered_map<std::string, EntryRef> g_cache;
size_t g_cache_bytes = 0;
uint64_t g_tick = 0;

void entry_release(Entry &e)
{
    if (e.dev) (void)hipFree(e.dev);
    if (e.host) (void)hipHostFree(e.host);
    if (e.ready) (void)hipEventDestroy(e.ready);
    e.dev = nullptr;
    e.host = nullptr;
    e.ready = nullptr;
}

// Evict least recently used entries held by no call until `incoming` more
// bytes fit (called with g_mu held).
void cache_make_room(size_t incoming)
{
    while (!g_cache.empty() &&
           (g_cache.size() + 1 > kCacheEntries || g_cache_bytes + incoming > kCacheBytes)) {
        auto victim = g_cache.end();
        for (auto it = g_cache.begin(); it != g_cache.end(); ++it)
            if (it->second.use_count() == 1 && (victim == g_cache.end() || it->second->tick < victim->second->tick))
                victim = it;
        if (victim == g_cache.end()) return;  // every entry is in use: grow past the bound
        (void)hipDeviceSynchronize();         // kernels of earlier calls may still read it
        g_cache_bytes -= victim->second->bytes;
        entry_release(*victim->second);
        g_cache.erase(victim);
    }
}

// Look up `key`; on a hit whose upload may still be in flight, make
// `stream` wait for it.  *out is empty on a miss.  Called with g_mu held.
int cache_find(const std::string &key, hipStream_t stream, EntryRef *out)
{
    auto it = g_cache.find(key);
    if (it == g_cache.end()) {
        out->reset();
        return XCT_OK;
    }
    Entry &e = *it->second;
    e.tick = ++g_tick;
    if (!e.done) {
        hipError_t q = hipEventQuery(e.ready);
        if (q == hipSuccess) {
            e.done = true;
        } else if (q == hipErrorNotReady) {
            hipError_t w = hipStreamWaitEvent(stream, e.ready, 0);
            if (w != hipSuccess) return hip_fail(w);
        } else {
            return hip_fail(q);
        }
    }
    *out = it->second;
    return XCT_OK;
}

// Create and upload an entry from host tables `parts` (up to two), ordered on
// `stream`.  Called with g_mu held.
int cache_insert(const std::string &key, const void *const parts[2], const size_t sizes[2],
                 hipStream_t stream, const Entry &meta, EntryRef *out)
{
    EntryRef e = std::make_shared<Entry>(meta);
    size_t total = 0;
    for (int i = 0; i < 2; ++i) {
        e->off[i] = total;
        total += align256(sizes[i]);
    }
    total = std::max<size_t>(total, 256);
    cache_make_room(total);
    hipError_t r = hipMalloc(reinterpret_cast<void **>(&e->dev), total);
    if (r == hipSuccess) r = hipHostMalloc(&e->host, total, hipHostMallocDefault);
    if (r == hipSuccess) {
        for (int i = 0; i < 2; ++i)
            if (sizes[i]) std::memcpy(static_cast<char *>(e->host) + e->off[i], parts[i], sizes[i]);
        r = hipMemcpyAsync(e->dev, e->host, total, hipMemcpyHostToDevice, stream);
    }
    if (r == hipSuccess) r = hipEventCreateWithFlags(&e->ready, hipEventDisableTiming);
    if (r == hipSuccess) r = hipEventRecord(e->ready, stream);
    if (r != hipSuccess) {
        entry_release(*e);
        return hip_fail(r);
    }
    e->bytes = total;
    e->tick = ++g_tick;
    g_cache.emplace(key, e);
    g_cache_bytes += total;
    *out = e;
    return XCT_OK;
}

template <typename T>
void key_append(std::string &k, const T &v)
{
    k.append(reinterpret_cast<const char *>(&v), sizeof(T));
}

int current_device(int *dev)
{
    hipError_t e = hipGetDevice(dev);
    return e == hipSuccess ? XCT_OK : hip_fail(e);
}

// Key prefix: kind, device.
int cache_key(char kind, std::string &key)
{
    int dev;
    if (int rc = current_device(&dev)) return rc;
    key.clear();
    key.push_back(kind);
    key_append(key, dev);
    return XCT_OK;
}

// cos/sin of every angle times pixel/pitch, in FP32 (inner loops, table 0) and
// FP64 (window anchors, table 1), rounded once from FP64 host trigonometry.
int geo_tables(const xct_geometry *g, hipStream_t stream, EntryRef *out)
{
    std::string key;
    if (int rc = cache_key('g', key)) return rc;
    const double r = g->pixel_size / g->det_pitch;
    key_append(key, r);
    key.append(reinterpret_cast<const char *>(g->angles), sizeof(double) * g->n_angles);
    std::lock_guard<std::mutex> lock(g_mu);
    if (int rc = cache_find(key, stream, out)) return rc;
    if (*out) return XCT_OK;
    const int n = g->n_angles;
    std::vector<float2> cs(n);
    std::vector<double2> csd(n);
    for (int k = 0; k < n; ++k) {
        const double c = std::cos(g->angles[k]) * r, s = std::sin(g->angles[k]) * r;
        csd[k] = make_double2(c, s);
        cs[k] = make_float2((float)c, (float)s);
    }
    const void *parts[2] = {cs.data(), csd.data()};
    const size_t sizes[2] = {sizeof(float2) * n, sizeof(double2) * n};
    return cache_insert(key, parts, sizes, stream, Entry(), out);
}

// Unit-sum sampled Gaussian of standard deviation sigma over -R..R,
// R = int(4 sigma + 0.5), in FP64 rounded once to FP32.
int blur_taps(float sigma, int radius, hipStream_t stream, EntryRef *out)
{
    std::string key;
    if (int rc = cache_key('b', key)) return rc;
    key_append(key, sigma);
    std::lock_guard<std::mutex> lock(g_mu);
    if (int rc = cache_find(key, stream, out)) return rc;
    if (*out) return XCT_OK;
    std::vector<double> g(2 * radius + 1);
    double sum = 0.0;
    for (int m = -radius; m <= radius; ++m) {
        const double t = (double)m / (double)sigma;
        g[m + radius] = std::exp(-0.5 * t * t);
        sum += g[m + radius];
    }
    std::vector<float> g32(g.size());
    for (size_t i = 0; i < g.size(); ++i) g32[i] = (float)(g[i] / sum);
    const void *parts[2] = {g32.data(), nullptr};
    const size_t sizes[2] = {sizeof(float) * g32.size(), 0};
    return cache_insert(key, parts, sizes, stream, Entry(), out);
}

// Virtual detector of a full-turn scan: the physical bins and their mirror
// images about the axis (bin 2c - n), renumbered from 0.  `first` is the
// virtual bin of physical bin 0.  Needs 2c integral and the axis on the
// detector.
void offset_virtual(const xct_geometry *g, int *nv, double *cv, int *first)
{
    const int nc = g->n_det;
    const int two_c = (int)std::nearbyint(2.0 * g->center);
    if ((nc - 1) - g->center >= g->center) {  // longer side to the right of the axis
        const int lo = two_c - (nc - 1);
        *nv = nc - lo;
        *cv = g->center - lo;
        *first = -lo;
    } else {
        *nv = two_c + 1;
        *cv = g->center;
        *first = 0;
    }
}

// Redundancy weights of a full-turn scan (offset scan, Section V-A b): with
// t = (n - c) / overlap, positive on the detector's longer side,
// w = 0 (t <= -1), sin^2(pi (1 + t) / 4) (|t| < 1), 1 (t >= 1), so that the
// two measurements of every ray, bins n and 2c - n half a turn apart, weigh
// one together.  FP64 on the host, rounded once.
int offset_weights(const xct_geometry *g, double overlap, hipStream_t stream, EntryRef *out)
{
    std::string key;
    if (int rc = cache_key('o', key)) return rc;
    key_append(key, g->n_det);
    key_append(key, g->center);
    key_append(key, overlap);
    std::lock_guard<std::mutex> lock(g_mu);
    if (int rc = cache_find(key, stream, out)) return rc;
    if (*out) return XCT_OK;
    const int nc = g->n_det;
    const double side = ((nc - 1) - g->center >= g->center) ? 1.0 : -1.0;
    std::vector<float> w(nc);
    for (int n = 0; n < nc; ++n) {
        const double t = side * ((double)n - g->center) / overlap;
        double v = 1.0;
        if (t <= -1.0) v = 0.0;
        else if (t < 1.0) {
            const double sn = std::sin(0.25 * M_PI * (1.0 + t));
            v = sn * sn;
        }
        w[n] = (float)v;
    }
    const void *parts[2] = {w.data(), nullptr};
    const size_t sizes[2] = {sizeof(float) * nc, 0};
    return cache_insert(key, parts, sizes, stream, Entry(), out);
}

// Checks shared by the offset-scan entry points.
int check_offset(const xct_geometry *g, double overlap)
{
    const double m = 2.0 * g->center;
    if (std::fabs(m - std::nearbyint(m)) > 1e-9) return XCT_EINVAL;
    if (g->center < 0.0 || g->center > g->n_det - 1) return XCT_EINVAL;
    const double short_side = std::min(g->center, (g->n_det - 1) - g->center);
    if (!std::isfinite(overlap) || !(overlap > 0.0) || overlap > short_side + 1e-9) return XCT_EINVAL;
    return XCT_OK;
}

// Forward-projector plan of a geometry (angle table 0, angle blocks 1, the
// staging shapes for one and four slices per workgroup).
int fp_tables(const xct_geometry *g, hipStream_t stream, EntryRef *out)
{
    std::string key;
    if (int rc = cache_key('f', key)) return rc;
    key_append(key, g->pixel_size / g->det_pitch);
    key_append(key, g->center);
    key_append(key, g->nx);
    key_append(key, g->ny);
    key_append(key, g->n_det);
    key.append(reinterpret_cast<const char *>(g->angles), sizeof(double) * g->n_angles);
    std::lock_guard<std::mutex> lock(g_mu);
    if (int rc = cache_find(key, stream, out)) return rc;
    if (*out) return XCT_OK;
    std::vector<FPAngle> ang;
    std::vector<FPBlock> blocks;
    Entry meta;
    // four slices per workgroup when their staging fits (not for strips many
    // pixels wide)
    if (int rc = fp_plan(g, ang, blocks, &meta.fp_four)) return rc;
    meta.n_blocks = (int)blocks.size();
    const void *parts[2] = {ang.data(), blocks.data()};
    const size_t sizes[2] = {sizeof(FPAngle) * ang.size(), sizeof(FPBlock) * blocks.size()};
    return cache_insert(key, parts, sizes, stream, meta, out);
}

// Spatial ramp kernel taps h_W[n] (inverse DTFT of |nu| W(nu) on |nu| <= 1/2).
double ramp_tap(int window, long n)
{
    auto rl = [](long m) -> double {
        if (m == 0) return 0.25;
        if (m % 2 == 0) return 0.0;
        return -1.0 / (M_PI * M_PI * (double)m * (double)m);
    };
    if (window == XCT_RAM_LAK) return rl(n);
    if (window == XCT_SHEPP_LOGAN) return 2.0 / (M_PI * M_PI * (1.0 - 4.0 * (double)n * (double)n));
    return 0.5 * rl(n) + 0.25 * (rl(n - 1) + rl(n + 1));
}

// In-place iterative radix-2 FFT in FP64 (forward, e^{-2 pi i k n / L}).
void host_fft(std::vector<std::complex<double>> &a)
{
    const size_t L = a.size();
    for (size_t i = 1, j = 0; i < L; ++i) {
        size_t bit = L >> 1;
        for (; j & bit; bit >>= 1) j ^= bit;
        j ^= bit;
        if (i < j) std::swap(a[i], a[j]);
    }
    for (size_t len = 2; len <= L; len <<= 1) {
        const size_t h = len >> 1;
        for (size_t k = 0; k < h; ++k) {
            const double ang = -2.0 * M_PI * (double)k / (double)len;
            const std::complex<double> w(std::cos(ang), std::sin(ang));
            for (size_t i = 0; i < L; i += len) {
                const std::complex<double> u = a[i + k], v = a[i + k + h] * w;
                a[i + k] = u + v;
                a[i + k + h] = u - v;
            }
        }
    }
}

int fft_length(int nc, int *log2L)
{
    int L = 64, lg = 6;
    while (L < 2 * nc - 1) {
        L <<= 1;
        ++lg;
    }
    *log2L = lg;
    return L;
}

// Twiddles exp(-2 pi i e / L) (table 0) and the filter spectrum H =
// DFT_L(h_W placed circularly) / (L pitch) (table 1), both rounded once from
// FP64.
int filter_tables(int nc, int window, double pitch, hipStream_t stream, EntryRef *out)
{
    std::string key;
    if (int rc = cache_key('h', key)) return rc;
    key_append(key, nc);
    key_append(key, window);
    key_append(key, pitch);
    std::lock_guard<std::mutex> lock(g_mu);
    if (int rc = cache_find(key, stream, out)) return rc;
    if (*out) return XCT_OK;
    Entry meta;
    const int L = fft_length(nc, &meta.lg);
    meta.L = L;
    std::vector<std::complex<double>> h(L, 0.0);
    for (long d = -(long)(nc - 1); d <= (long)(nc - 1); ++d)
        h[(size_t)((d % L + L) % L)] = ramp_tap(window, d);
    host_fft(h);
    std::vector<float> H(L);
    for (int k = 0; k < L; ++k) H[k] = (float)(h[k].real() / ((double)L * pitch));
    std::vector<float2> tw(L);
    for (int e = 0; e < L; ++e) {
        const double ang = 2.0 * M_PI * (double)e / (double)L;
        tw[e] = make_float2((float)std::cos(ang), (float)-std::sin(ang));
    }
    const void *parts[2] = {tw.data(), H.data()};
    const size_t sizes[2] = {sizeof(float2) * L, sizeof(float) * L};
    return cache_insert(key, parts, sizes, stream, meta, out);
}

// ---------------------------------------------------------------- back-projection plan

// Window entries per angle for a 64-pixel tile: the detector footprint of the
// tile spans 63 (|C| + |S|) <= 63 sqrt(2) pixel/pitch bins; 3 more cover the
// floor, the right tap and the one-bin margin of the anchor.
int window_entries(double ratio) { return (int)std::ceil((kTile - 1) * std::sqrt(2.0) * ratio + 1e-3) + 3; }

// Half-turn sets of a symmetric angle set: 1 when angle k + N_p/2 is angle k
// plus a quarter turn for every k < N_p/2 (a half turn); 2 when each half of
// the angles is such a set (a full turn, as in offset scans); 0 otherwise,
// or when the slice is not square and even, 2c is not integral, or the
// windows do not fit the symmetric kernel.
int symmetric_sets(const xct_geometry *g)
{
    if (g->nx != g->ny || (g->nx & 1) || (g->n_angles & 1)) return 0;
    if (!bp_sym_window(window_entries(g->pixel_size / g->det_pitch))) return 0;
    const double m = 2.0 * g->center;
    if (std::fabs(m - std::nearbyint(m)) > 1e-9) return 0;
    auto quarter_closed = [g](int k_begin, int n) {
        const int H = n / 2;
        for (int k = 0; k < H; ++k)
            if (std::fabs(g->angles[k_begin + k + H] - g->angles[k_begin + k] - 0.5 * M_PI) > 1e-9)
                return false;
        return true;
    };
    const int np = g->n_angles;
    if (quarter_closed(0, np)) return 1;
    if (np % 4 == 0 && quarter_closed(0, np / 2) && quarter_closed(np / 2, np / 2)) return 2;
    return 0;
}

// Kernel path of a geometry: the quarter-turn + mirror symmetric kernel when
// it applies; otherwise the mirror kernel when 2c is integral (detector bin
// 2c - n exists for every bin n) and its windows fit; otherwise the generic
// kernel.
int choose_path(const xct_geometry *g, int *sets)
{
    *sets = symmetric_sets(g);
    if (*sets) return kPathSymmetric;
    const double m = 2.0 * g->center;
    if (std::fabs(m - std::nearbyint(m)) <= 1e-9 && bp_sym_window(window_entries(g->pixel_size / g->det_pitch)))
        return kPathMirror;
    return kPathGeneric;
}

struct BPJob {
    const xct_geometry *g;  // geometry the rows are back-projected with
    EntryRef t;             // its trigonometry tables
    int32_t n_slices;
    const void *sino;
    void *image;
    float scale;
    int32_t accumulate;
    int cus = device_cus();  // (once per job: plans weigh some hundred forms)
    int path;
    int sets = 0;           // half-turn sets of the symmetric path
    int32_t out_u16 = 0;
    float code_a = 0.0f, code_b = 0.0f;
    // Vector kernels: the parts that the job's angles (pairs) are split into
    // where there is room for the parts' copies of the image (partial).
    int32_t parts = 1, part_len = 0;
    float *partial = nullptr;
};

#ifndef XCT_SYM_MAX_SLICES
#define XCT_SYM_MAX_SLICES 2  // slices per work item of the symmetric kernel (1 or 2)
#endif
// Slices (pairs of slices) per work item of a job alone; 3 where three slices
// go as a pair and one.
int item_slices(const BPJob &j)
{
    if (j.path == kPathGeneric) return 1;
    if (j.path == kPathPairs && j.n_slices == 3) return 3;
    return std::min(j.path == kPathPairs ? (j.n_slices + 1) / 2 : j.n_slices, XCT_SYM_MAX_SLICES);
}

// Work items by which the entry points limit a call (kMaxItems to a launch):
// those of the path that the geometry gives, one generic item per slice and
// tile also where slices go in pairs or the matrix cores take the slab.
constexpr int64_t kMaxItems = (int64_t)1 << 31;
int64_t plan_tiles(const BPJob &j, int sl, int *tx, int *ty);

int64_t limit_items(BPJob j)
{
    if (j.path == kPathPairs) j.path = kPathGeneric;
    int tx, ty;
    return plan_tiles(j, item_slices(j), &tx, &ty);
}

// Slices of any geometry go two at a time where the call may round otherwise
// than xct_backproject_u16 does (which keeps the generic kernel's bits) and
// the windows fit.
void pair_slices(BPJob &j)
{
    if (j.path == kPathGeneric && !j.out_u16 && j.n_slices >= 2 && bp_sym_window(window_entries(j.g->pixel_size / j.g->det_pitch)))
        j.path = kPathPairs;
}

// Tiles per slice as the kernel indexes them (tiles_x, tiles_y) and the work
// items of the whole slab.
int64_t plan_tiles(const BPJob &j, int sl, int *tx, int *ty)
{
    if (j.path == kPathGeneric) {
        *tx = (j.g->nx + kTile - 1) / kTile;
        *ty = (j.g->ny + kTile - 1) / kTile;
        return (int64_t)*tx * *ty * j.n_slices;
    }
    if (j.path == kPathPairs) {
        *tx = (j.g->nx + kTile - 1) / kTile;
        *ty = (j.g->ny + kTile - 1) / kTile;
        const int64_t spi = sl == 3 ? 3 : 2 * sl;  // slices per item
        return (int64_t)*tx * *ty * ((j.n_slices + spi - 1) / spi);
    }
    if (j.path == kPathMirror) {  // the upper ceil(N_y/2) rows
        *tx = (j.g->nx + kTile - 1) / kTile;
        *ty = ((j.g->ny + 1) / 2 + kTile - 1) / kTile;
        return (int64_t)*tx * *ty * (((int64_t)j.n_slices + sl - 1) / sl);
    }
    const int q = (j.g->nx / 2 + kTile - 1) / kTile;  // tiles along a quadrant edge
    *tx = *ty = q;
    return (int64_t)q * q * (((int64_t)j.n_slices + sl - 1) / sl);
}

// LDS bytes of one angle stage: the symmetric kernel takes 6 angle pairs of
// 8 FP32 windows of 96 entries per slice (four 256-thread or two 512-thread
// workgroups per CU fit in 160 KiB).
#ifndef XCT_SYM2_STAGE_KB
#define XCT_SYM2_STAGE_KB 74
#endif
constexpr size_t kGenericStageBytes = 32 * 1024;
constexpr size_t kSymStageBytes = 37 * 1024;
constexpr size_t kSym2StageBytes = XCT_SYM2_STAGE_KB * 1024;
// (three 512-thread workgroups per CU, or six of 256, whose registers the
// mirror kernels leave: three slices of 1600^2, 1500 angles 1.74 ms with two,
// 1.35 with three; where there are items for them also the others: 8 x 2048^2 x
// 1801 5.24 to 5.33 ms and 4.90 to 5.23, one slice of 3000^2, 2001 angles, 2.73
// and 1.91, while 512 items of 1001^2 take 1 to 2 % longer in shorter stages)
constexpr size_t kMirrorStageBytes = 49 * 1024;
constexpr int kPartStages = 1;  // LDS stages of the shortest part of a split job

// Window, angles (pairs) per stage and LDS bytes of a vector kernel whose
// widest window needs W entries, for `items` items of `spi` slices.
struct VectorShape { int win, kb; size_t lds; };

VectorShape vector_shape(int path, int W, int spi, int64_t items, int cus)
{
    VectorShape v;
    // (the wide windows only where the shorter stages save a round: 8 x 1300^2,
    // pixel 1.2, 924 items 1.07 times as long in them, 693 items 0.91)
    const bool narrow = bp_sym_window(W) <= 96;
    auto shorter = [&](int more) { return path != kPathSymmetric && items > (more - (more == 6 ? 2 : 1)) * (int64_t)cus && (narrow || items <= more * (int64_t)cus); };
    const bool three = spi == 3 || (spi == 2 && shorter(3)), six = spi == 1 && shorter(6);
    const size_t budget = three ? kMirrorStageBytes : six ? kMirrorStageBytes / 2 : spi == 2 ? kSym2StageBytes : kSymStageBytes;
    v.win = path == kPathGeneric ? W : bp_sym_window(W);  // choose_path only routes windows that fit here
    if (path == kPathSymmetric) {
        v.kb = (int)std::max<size_t>(1, budget / (4 * (size_t)v.win * spi * sizeof(float4) + 24));
        v.lds = bp_sym_lds_bytes(v.win, v.kb, spi);
    } else if (path == kPathMirror || path == kPathPairs) {
        v.kb = (int)std::max<size_t>(1, budget / bp_mirror_lds_bytes(v.win, 1, spi));
        v.lds = bp_mirror_lds_bytes(v.win, v.kb, spi);
    } else {
        // (more than four items per CU: stages that let eight workgroups share
        // it; 8 x 2048^2 x 1025 angles 4.67 ms with the longer stages, 3.83)
        const size_t bytes = items > 4 * (int64_t)cus ? kGenericStageBytes * 3 / 5 : kGenericStageBytes;
        v.kb = (int)std::max<size_t>(1, std::min<size_t>(64, bytes / (8 * (size_t)v.win + 16)));
        v.lds = bp_generic_lds_bytes(v.win, v.kb);
    }
    return v;
}

// Work items of a job alone on the vector kernels, with its slices per item.
int64_t vector_items(const BPJob &j, int *spi)
{
    *spi = item_slices(j);
    int tx, ty;
    return plan_tiles(j, *spi, &tx, &ty);
}

// Times of the vector kernels as measured (ns per angle that a round of work
// items takes, with every slot of the device taken and with one item per CU,
// and ns for the stores that end a full round's items; shapes of 24 to 600
// angles, and 8192^2), by the workgroups that vector_shape lets share a CU:
//  * symmetric, two slices per item: two, 1260 (2048^2 1180, 1024^2 and 512^2
//    1350) and 770; one slice: four, 1400 and 710; stores 17 us.
//  * mirror (and slices in pairs), two slices (pairs): two, 820 and 600, or
//    three, 1140; one: four, 1270 and 630, or six, 1300; stores 11 us.
//  * a pair and one slice: three, 870 and 465.
//  * generic: four, 640 and 510, or eight, 980 over many rounds and 1200 over
//    one or two; stores 5 us.
// The others' windows of 192 bins take 1.13 times as long (mirror, 16 x 1024^2 x
// 300 angles: 517 us at pixel 1.2, 459 at 1).
struct KernelTimes { int per_cu; double full, alone, store; };

KernelTimes vector_times(int path, int spi, int64_t items, int cus)
{
    if (path == kPathGeneric && items > 4 * (int64_t)cus) return {8, items > 16 * (int64_t)cus ? 980.0 : 1200.0, 510, 5000};
    if (path == kPathGeneric) return {4, 640, 510, 5000};
    if (path == kPathSymmetric) return spi == 2 ? KernelTimes{2, 1260, 770, 17000} : KernelTimes{4, 1400, 710, 17000};
    if (spi == 3) return {3, 870, 465, 11000};
    if (spi == 2) return items > 2 * (int64_t)cus ? KernelTimes{3, 1140, 600, 11000} : KernelTimes{2, 820, 600, 11000};
    return items > 4 * (int64_t)cus ? KernelTimes{6, 1300, 630, 11000} : KernelTimes{4, 1270, 630, 11000};
}

// Time of n items of `angles` angles that store `stores` times each.  The last
// round takes as long as the CUs that hold most of its items, which up to three
// large workgroups a CU show in steps.
double rounds_ns(const KernelTimes &t, int64_t n, int64_t cus, double angles, double stores)
{
    const double full = t.full * angles + t.store * stores;
    const double alone = t.alone * angles + (t.per_cu > 1 ? 0.6 : 1.0) * t.store * stores;
    const int64_t slots = t.per_cu * cus, rest = n % slots;
    const double held = t.per_cu <= 3 ? (double)((rest + cus - 1) / cus) : (double)rest / cus;
    return (n / slots) * full + (rest == 0 ? 0.0 : held <= 1.0 ? alone : alone + (full - alone) * (held - 1.0) / (t.per_cu - 1.0));
}

// Angles that a work item of a job walks.
int item_angles(const BPJob &j) { return j.parts < 2 ? j.g->n_angles : j.part_len * (j.path == kPathSymmetric ? 2 : 1); }

// The share of a job's whole walks in rounds that fill the device.
double vector_share_ns(const BPJob &j)
{
    int spi;
    const int64_t items = vector_items(j, &spi);
    const KernelTimes t = vector_times(j.path, spi, std::numeric_limits<int64_t>::max(), j.cus);  // (in a batch that fills the device)
    return (double)items / (t.per_cu * (double)j.cus) * (t.full * j.g->n_angles + t.store);
}

size_t image_bytes(const BPJob &j) { return sizeof(float) * (size_t)j.n_slices * j.g->nx * j.g->ny; }

// Adding up parts: a launch and its scratch, and the passes over the images at 4 TB/s.
double sum_ns(const BPJob &j, int64_t parts) { return 14000.0 + (parts + 1) * (double)image_bytes(j) / 4000.0; }

// (stores: 0 where whole walks and parts are weighed against each other)
double bp_vector_ns(const BPJob &j, double stores)
{
    int spi;
    const int64_t items = vector_items(j, &spi);
    const int64_t n = j.parts < 2 ? items : items * j.parts;
    KernelTimes t = vector_times(j.path, spi, n, j.cus);
    if (j.path != kPathGeneric && bp_sym_window(window_entries(j.g->pixel_size / j.g->det_pitch)) > 96) t.full *= 1.13, t.alone *= 1.13;
    if (j.parts < 2) return rounds_ns(t, n, j.cus, j.g->n_angles, stores);
    return rounds_ns(t, n, j.cus, item_angles(j), stores) + sum_ns(j, j.parts);
}

// At most `want` parts of whole LDS stages, as equal as these allow.
void set_parts(BPJob &j, int64_t want)
{
    int spi;
    const int64_t items = vector_items(j, &spi);
    const int kb = vector_shape(j.path, window_entries(j.g->pixel_size / j.g->det_pitch), spi, items, j.cus).kb;
    const int64_t units = j.path == kPathSymmetric ? j.g->n_angles / 2 : j.g->n_angles;
    j.part_len = (int)(((units + want - 1) / want + kb - 1) / kb * kb);
    j.parts = (int)((units + j.part_len - 1) / j.part_len);
}

// Parts of a small job's angles: a workgroup walks all angles of its tile, so
// a call with fewer items than the device has slots leaves some idle and takes
// the time of one walk (one 256^2 slice, 360 angles: four items, 194 us).  Its
// angles are split into the parts, of kPartStages LDS stages or more, whose
// rounds and sum take least, each part a work item with its own copy of the
// image, and the copies are added up.  (Parts added up inside an item, without
// copies, cost a pass over the item's pixels each: 64 slabs of one 512^2 slice,
// 720 angles, in one batch 2.53 ms, 1.98 in whole walks.)
void plan_parts(BPJob &j)
{
    int spi;
    const int64_t items = vector_items(j, &spi);
    if (j.out_u16 || items >= vector_times(j.path, spi, 0, j.cus).per_cu * (int64_t)j.cus) return;
    const VectorShape v = vector_shape(j.path, window_entries(j.g->pixel_size / j.g->det_pitch), spi, items, j.cus);
    const int units = j.path == kPathSymmetric ? j.g->n_angles / 2 : j.g->n_angles;
    const int64_t most = std::min<int64_t>(units / (kPartStages * v.kb), kPartBytes / image_bytes(j));
    BPJob t = j;
    double least = 0.95 * bp_vector_ns(j, 0);
    for (int64_t want = 2; want <= most && want <= 64; want += 1 + want / 8) {
        set_parts(t, want);
        const double ns = t.parts < 2 ? least : bp_vector_ns(t, 0);
        if (ns < least) {
            least = ns;
            j.part_len = t.part_len;
            j.parts = t.parts;
        }
    }
}

// A job alone: the parts of its angles, and slices in pairs only where that is
// faster.  A call that leaves the device idle anyway ends sooner in the generic
// kernel's more and shorter items (16 x 142^2 x 28 angles 35 us, 42 in pairs).
void plan_alone(BPJob &j)
{
    BPJob single = j;
    plan_parts(j);
    if (j.path != kPathPairs) return;
    single.path = kPathGeneric;
    plan_parts(single);
    if (bp_vector_ns(single, 1) < bp_vector_ns(j, 1)) j = single;
}

// Partial images of a split job that takes one item per part (0: too large, or not split).
size_t part_bytes(const BPJob &j)
{
    const size_t b = j.parts * image_bytes(j);
    return j.parts > 1 && b <= (size_t)kPartBytes ? align256(b) : 0;
}

// Launch one back-projection over jobs that all take the same kernel path.
// `counters` (kXcds zeroed words on the stream) makes it persistent; `table`
// is device memory for the slab descriptors, needed when there are more than
// kInlineSlabs jobs.  A non-persistent launch whose grid would exceed 2^32
// work-items is split into several launches over consecutive item ranges.
int launch_bp_jobs(std::vector<BPJob> jobs, int dtype, unsigned int *counters, BPSlab *table,
                   hipStream_t s, const uint32_t *gate = nullptr)
{
    if (jobs.empty()) return XCT_OK;
    const int path = jobs[0].path;
    // longest items first (those of one slab cost the same; a split slab's are short)
    std::stable_sort(jobs.begin(), jobs.end(),
                     [](const BPJob &a, const BPJob &b) { return item_angles(a) > item_angles(b); });
    // two slices (pairs) per work item when every slab has at least two
    int spi = item_slices(jobs[0]);
    bool split = gate != nullptr;
    for (const BPJob &j : jobs) {
        spi = std::min(spi, item_slices(j));
        split = split || j.partial;
    }
    std::vector<BPSlab> desc(jobs.size());
    int W = 0;
    int64_t items = 0;
    for (size_t i = 0; i < jobs.size(); ++i) {
        const BPJob &j = jobs[i];
        BPSlab &sl = desc[i];
        std::memset(&sl, 0, sizeof(sl));
        int tx, ty;
        const int64_t n_items = plan_tiles(j, spi, &tx, &ty);
        sl.sino = j.sino;
        sl.image = j.image;
        sl.cs = j.t->table<float2>(0);
        sl.csd = j.t->table<double2>(1);
        sl.center = j.g->center;
        sl.item_begin = items;
        sl.n_angles = j.g->n_angles;
        sl.n_det = j.g->n_det;
        sl.nx = j.g->nx;
        sl.ny = j.g->ny;
        sl.n_slices = j.n_slices;
        sl.tiles_x = tx;
        sl.tiles_y = ty;
        sl.mirror = path == kPathSymmetric || path == kPathMirror ? (int32_t)std::nearbyint(2.0 * j.g->center) : 0;
        sl.sets = path == kPathSymmetric ? j.sets : 1;
        sl.scale = j.scale;
        sl.accumulate = j.accumulate;
        sl.part_len = j.part_len;
        sl.partial = j.partial;
        sl.out_u16 = j.out_u16;
        sl.code_a = j.code_a;
        sl.code_b = j.code_b;
        items += j.partial ? n_items * j.parts : n_items;
        W = std::max(W, window_entries(j.g->pixel_size / j.g->det_pitch));
    }
    if (items >= kMaxItems) return XCT_ETOOBIG;
    BPBatch b;
    std::memset(&b, 0, sizeof(b));
    b.n_slabs = (int32_t)jobs.size();
    b.total_items = items;
    b.counter = counters;
    b.gate = gate;
    const VectorShape v = vector_shape(path, W, spi, items, jobs[0].cus);
    W = v.win;
    b.kb = v.kb;
    const size_t lds = v.lds;
    b.win = W;
    if (lds > 160 * 1024) return XCT_ETOOBIG;
    if (jobs.size() > (size_t)kInlineSlabs) {
        if (!table) return XCT_ETOOBIG;
        hipError_t e = write_slab_table(table, desc.data(), (int)desc.size(), s);
        if (e != hipSuccess) return hip_fail(e);
        b.table = table;
    } else {
        std::memcpy(b.slab, desc.data(), sizeof(BPSlab) * desc.size());
    }
    if (counters) {
        const int per_cu = bp_max_blocks_per_cu(path, dtype, W, spi, split, lds);
        const int grid = (int)std::min<int64_t>(items, (int64_t)per_cu * jobs[0].cus);
        hipError_t e = launch_bp(path, b, dtype, spi, split, grid, lds, s);
        return e == hipSuccess ? XCT_OK : hip_fail(e);
    }
    const int64_t threads = bp_block_threads(path, spi);
    const int64_t max_items = ((((int64_t)1 << 32) - 1) / threads) & ~(int64_t)7;
    for (int64_t base = 0; base < items; base += max_items) {
        const int64_t count = std::min(max_items, items - base);
        b.item_base = base;
        b.xcd_remap = (count % 8 == 0) ? 1 : 0;
        hipError_t e = launch_bp(path, b, dtype, spi, split, (int)count, lds, s);
        if (e != hipSuccess) return hip_fail(e);
    }
    return XCT_OK;
}

// A split job, one work item per part.
int launch_bp_parts(BPJob j, int dtype, float *partial, hipStream_t s)
{
    j.partial = partial;
    if (int rc = launch_bp_jobs({j}, dtype, nullptr, nullptr, s)) return rc;
    const hipError_t e = launch_sum_parts(static_cast<float *>(j.image), partial, j.parts, (int64_t)j.n_slices * j.g->nx * j.g->ny,
                                          j.accumulate, nullptr, s);
    return e == hipSuccess ? XCT_OK : hip_fail(e);
}

// ---------------------------------------------------------------- matrix-core back-projection

// How a job takes the matrix-core kernel: the kind (what a coordinate
// serves), columns per item (0: it does not), and the angles per launch.
struct MXPlan {
    int kind = kMXPlain, cols = 0;
    double ns = 0;     // its time, estimated
    int angles = 0;    // per launch (of one quarter turn for kMXQuarter)
    int part_len = 0;  // angles added up at a time (see MXArgs)
    int per_launch = 0;   // angles of a launch
    int parts = 1;        // of a launch
    bool spread = false;  // one workgroup per item and part
};

// The split table of one launch is held to this much scratch; a table that
// needs more is made and used angle range by angle range, the image
// accumulating.
constexpr int64_t kMXTableBytes = kQuadBytes;

// xct_backproject keeps the vector kernels below this many voxel updates
// (about a millisecond), so that there its images are to the bit what
// xct_backproject_u16 quantises.
constexpr double kMXLeastUpdates = 1.5e10;

// Angle k of a half turn is angle k pi / N_p: reflection pairs angle k with N_p - k.
bool reflected_set(const xct_geometry *g)
{
    if (std::fabs(g->angles[0]) > 1e-9) return false;
    for (int k = 1; k < g->n_angles; ++k)
        if (std::fabs(g->angles[k] + g->angles[g->n_angles - k] - M_PI) > 1e-9) return false;
    return true;
}

size_t mx_words_bytes(int n_slices) { return align256(sizeof(uint32_t) * (2 * (size_t)n_slices + 1)); }

int mx_ops(int kind)
{
    return kind == kMXPlain ? 1 : kind == kMXMirror ? 2 : kind == kMXQuarter2 ? 8 : 4;
}

// Work items of a job on the matrix cores, and their tiles.
int64_t mx_items(const BPJob &j, int kind, int cols, int *tiles_x, int *tiles_y)
{
    const bool all_x = kind == kMXPlain || kind == kMXMirror, all_y = kind == kMXPlain;
    *tiles_x = ((all_x ? j.g->nx : (j.g->nx + 1) / 2) + kMXTile - 1) / kMXTile;
    *tiles_y = ((all_y ? j.g->ny : (j.g->ny + 1) / 2) + kMXTile - 1) / kMXTile;
    const int64_t tiles = kind == kMXQuarter2 ? (int64_t)*tiles_x * (*tiles_x + 1) / 2 : (int64_t)*tiles_x * *tiles_y;
    const int spi = cols / mx_ops(kind);
    return tiles * ((j.n_slices + spi - 1) / spi);
}

// Which kernels a job takes is decided by their times as measured: the vector
// kernels' above; the matrix kernel's ns per angle are 610 for a round of one
// 64-column item per CU, and for two items per CU (one) 680 (430) with 32
// columns and 415 (270) with 16 (16 x 2048^2 x 1800 angles in 64 columns 4.94
// ms; 32 x 1024^2 x 1025 in 32 columns 1.57 ms; 4 x 4096^2 x 1023 in 16 columns
// 3.63 ms; 4 x 4096^2 x 3072, 2080 items of 32 columns or 4096 of 16: 9.1 and
// 9.7 ms).  Every part's stores add 59, 46 and 23 us to a round in which all
// columns are slices (16 x 1024^2, 64 x 512^2 and 4 x 2048^2 in two parts: 118
// to 121, 92 to 97 and 46 to 51 us apart from the angles), which decides calls
// of few angles: 104 x 1950^2 x 20 take 3.7 ms in matrix form, 0.94 in vector
// form.  The matrix path's own passes over the rows (magnitudes, split table)
// are added at the 4.5 TB/s they reach, with 30 us for their launches (4 x 512^2
// x 721 angles: 102 us in matrix form, 94 in vector form).
double bp_matrix_ns(const BPJob &j, const MXPlan &p, int64_t items, int dtype)
{
    const double rows = (double)j.n_slices * j.g->n_angles * j.g->n_det;
    const double launches = (j.g->n_angles + p.per_launch - 1) / p.per_launch;
    const double angles = p.spread ? (double)p.part_len / p.per_launch * j.g->n_angles : j.g->n_angles;
    const int spi = p.cols / mx_ops(p.kind);
    const double used = (double)j.n_slices / ((j.n_slices + spi - 1) / spi * spi);
    const KernelTimes t = p.cols == 64   ? KernelTimes{1, 610, 610, 59000}
                          : p.cols == 32 ? KernelTimes{2, 680, 430, 46000}
                                         : KernelTimes{2, 415, 270, 23000};
    double ns = rounds_ns(t, (p.spread ? p.parts : 1) * items, j.cus, angles, launches * (p.spread ? 1 : p.parts) * used);
    ns += rows * (2 * dtype_size(dtype) + 4) / 4500.0 + 30000.0;
    if (p.spread) ns += sum_ns(j, p.parts);
    return ns;
}

// The parts of a matrix launch: two at least where one launch covers all
// angles (its three roundings per product pair would otherwise leave more
// error in the sums than the vector kernels' one).  They are work items of
// their own where that fills the last round of items better by more than
// adding them up costs.
void mx_parts(const BPJob &j, MXPlan &p, int64_t items, int dtype)
{
    const int n = p.per_launch, whole = n == j.g->n_angles ? 2 : 1;
    const int64_t most = std::min<int64_t>(std::min<int64_t>(64, n / 16), kPartBytes / (int64_t)image_bytes(j));
    auto split = [&](int64_t parts, bool spread) {
        MXPlan q = p;
        q.part_len = (int)((n + parts - 1) / parts + kMXAngles - 1) & ~(kMXAngles - 1);
        q.parts = (n + q.part_len - 1) / q.part_len;
        q.spread = spread && q.parts > 1;
        return q;
    };
    p = split(whole, false);
    double least = bp_matrix_ns(j, p, items, dtype);
    for (int64_t parts = 2; parts <= most; parts += 1 + parts / 8) {
        const MXPlan q = split(parts, true);
        const double ns = bp_matrix_ns(j, q, items, dtype);
        if (ns < least) {
            least = ns;
            p = q;
        }
    }
}

MXPlan mx_plan(const BPJob &j, int dtype)
{
    MXPlan best;
    const xct_geometry *g = j.g;
    // (uint16 images keep the vector kernels' rounding; windows cover
    // kMXMaxRatio; slice groups are a grid dimension)
    if (j.out_u16 || g->pixel_size / g->det_pitch > kMXMaxRatio || j.n_slices > 4 * 65535) return best;
    // (below some 50 us of the vector kernels the extra launches cost more than is saved)
    if ((double)j.n_slices * g->n_angles * g->nx * g->ny < 3e8) return best;
    const int64_t angle_bytes = (int64_t)((j.n_slices + 3) / 4) * g->n_det * 16;
    const int64_t fit = kMXTableBytes / angle_bytes;
    // the reflected kinds read rows k and N_p - k together: whole tables only
    const bool refl = (j.path == kPathSymmetric || j.path == kPathMirror) && fit >= g->n_angles && reflected_set(g);
    double least = 0.95 * bp_vector_ns(j, 1);
    auto consider = [&](int kind) {
        MXPlan p;
        p.kind = kind;
        const int run = kind == kMXQuarter ? g->n_angles / j.sets / 2 : g->n_angles;
        const int64_t cap = (kind == kMXQuarter ? fit / 2 : fit) & ~(int64_t)(kMXAngles - 1);
        if (fit < g->n_angles && cap <= 0) return;
        // (equal ranges)
        const int64_t ranges = fit >= g->n_angles ? 1 : (run + cap - 1) / cap;
        p.angles = ranges == 1 ? run : (int)((run + ranges - 1) / ranges + kMXAngles - 1) & ~(kMXAngles - 1);
        p.per_launch = kind == kMXQuarter ? 2 * p.angles : p.angles;
        for (p.cols = kind == kMXQuarter2 ? 32 : 16; p.cols <= 64; p.cols *= 2) {
            int tx, ty;
            const int64_t items = mx_items(j, kind, p.cols, &tx, &ty);
            if (items >= (int64_t)1 << 22) continue;  // (grid of workgroups of 1024 below 2^32)
            mx_parts(j, p, items, dtype);
            const double ns = bp_matrix_ns(j, p, items, dtype);
            if (ns < least) {
                least = p.ns = ns;
                best = p;
            }
        }
    };
    consider(j.path == kPathSymmetric ? kMXQuarter : j.path == kPathMirror ? kMXMirror : kMXPlain);
    if (refl) consider(j.path == kPathSymmetric ? kMXQuarter2 : kMXMirror2);
    return best;
}

// Scratch of a job: the slices' magnitudes, the split table of one launch, and
// the parts' images where each part is a work item of its own.
size_t mx_scratch_bytes(const BPJob &j, const MXPlan &p)
{
    const size_t rows = (size_t)p.angles * (p.kind == kMXQuarter ? 2 : 1);
    return mx_words_bytes(j.n_slices) + align256((size_t)((j.n_slices + 3) / 4) * rows * j.g->n_det * 16) +
           (p.spread ? align256(p.parts * image_bytes(j)) : 0);
}

// The slices' magnitudes, then for each range of angles its split table and
// its back-projection, and last the vector kernels, whose launch does nothing
// unless some row element is not finite or some slice's range too wide.
int launch_bp_matrix(const BPJob &j, const MXPlan &p, int dtype, void *scratch, hipStream_t s)
{
    const xct_geometry *g = j.g;
    uint32_t *amax = static_cast<uint32_t *>(scratch);
    char *table = static_cast<char *>(scratch) + mx_words_bytes(j.n_slices);
    hipError_t e = launch_absmax(j.sino, dtype, j.n_slices, (int64_t)g->n_angles * g->n_det, amax, s);
    if (e != hipSuccess) return hip_fail(e);
    MXArgs a{};
    a.table = reinterpret_cast<int64_t>(table);
    a.image = static_cast<float *>(j.image);
    a.csd = j.t->table<double2>(1);
    a.amax = amax;
    a.center = g->center;
    a.n_det = g->n_det;
    a.nx = g->nx;
    a.ny = g->ny;
    a.n_slices = j.n_slices;
    a.mirror = p.kind == kMXPlain ? 0 : (int32_t)std::nearbyint(2.0 * g->center);
    a.scale = j.scale;
    a.accumulate = j.accumulate;
    a.part_len = p.part_len;
    if (p.spread)  // the parts' images end the scratch
        a.partial = reinterpret_cast<float *>(static_cast<char *>(scratch) + mx_scratch_bytes(j, p) - align256(p.parts * image_bytes(j)));
    const int64_t items = mx_items(j, p.kind, p.cols, &a.tiles_x, &a.tiles_y);
    const int sets = p.kind == kMXQuarter ? j.sets : 1;
    const int h = g->n_angles / sets / 2;                       // quarter turn
    const int run = p.kind == kMXQuarter ? h : g->n_angles;     // angles that one set's launches cover
    SplitArgs t{};
    t.sino = j.sino;
    t.table = reinterpret_cast<uint4 *>(table);
    t.amax = amax;
    t.n_angles = g->n_angles;
    t.n_det = g->n_det;
    t.n_slices = j.n_slices;
    for (int set = 0; set < sets; ++set) {
        for (int k0 = 0; k0 < run; k0 += p.angles) {
            const int n = std::min(p.angles, run - k0);
            a.k_first = t.k_first = set * 2 * h * (p.kind == kMXQuarter) + k0;
            a.half_set = p.kind == kMXQuarter ? n : p.kind == kMXQuarter2 ? h : 0;
            a.k_jump = t.k_jump = p.kind == kMXQuarter ? h - n : 0;
            a.n_angles = t.rows = p.kind == kMXQuarter ? 2 * n : n;
            t.split = p.kind == kMXQuarter ? n : t.rows;
            a.items = (int32_t)items;
            e = launch_split(t, dtype, s);
            const int parts = (a.n_angles + a.part_len - 1) / a.part_len;
            if (e == hipSuccess) e = launch_bp_mfma(a, p.cols, p.kind, (int)(p.spread ? items * parts : items), s);
            if (e == hipSuccess && p.spread)
                e = launch_sum_parts(a.image, a.partial, parts, (int64_t)j.n_slices * g->nx * g->ny, a.accumulate, amax, s);
            if (e != hipSuccess) return hip_fail(e);
            a.accumulate = 1;
        }
    }
    return launch_bp_jobs({j}, dtype, nullptr, nullptr, s, amax);
}

}  // namespace

// ================================================================ C ABI

extern "C" {

const char *xct_status_string(int status)
{
    switch (status) {
    case XCT_OK: return "ok";
    case XCT_EINVAL: return "invalid argument";
    case XCT_EDTYPE: return "unsupported dtype or window";
    case XCT_EWORKSPACE: return "workspace missing, misaligned or too small";
    case XCT_ETOOBIG: return "size beyond the supported limits";
    case XCT_EHIP: return "HIP runtime error";
    default: return "unknown status";
    }
}

int xct_version(void) { return XCT_VERSION; }

int xct_last_hip_error(void) { return g_last_hip; }

void xct_cache_clear(void)
{
    std::lock_guard<std::mutex> lock(g_mu);
    for (auto &kv : g_cache) entry_release(*kv.second);
    g_cache.clear();
    g_cache_bytes = 0;
    trim_stream_pools();
}

int xct_filter(const xct_geometry *g, int32_t n_slices, const void *sino, int32_t sino_t,
               void *filtered, int32_t filtered_t, int32_t window, xct_stream stream)
{
    if (int rc = check_geometry(g, false)) return rc;
    if (int rc = check_slices(g, n_slices)) return rc;
    if (!sino || !filtered) return XCT_EINVAL;
    if (!dtype_ok(sino_t) || !dtype_ok(filtered_t)) return XCT_EDTYPE;
    if (window < XCT_RAM_LAK || window > XCT_HANN) return XCT_EDTYPE;
    if (sino == filtered && sino_t != filtered_t) return XCT_EINVAL;
    if (g->n_det > kMaxFFT / 2) return XCT_ETOOBIG;
    hipStream_t s = (hipStream_t)stream;
    EntryRef ft;
    if (int rc = filter_tables(g->n_det, window, g->det_pitch, s, &ft)) return rc;
    FilterArgs a{};
    a.in = sino;
    a.out = filtered;
    a.tw = ft->table<float2>(0);
    a.H = ft->table<float>(1);
    a.rows = (int64_t)n_slices * g->n_angles;
    a.nc = g->n_det;
    a.in_len = g->n_det;
    a.L = ft->L;
    a.log2L = ft->lg;
    hipError_t e = launch_filter(a, sino_t, filtered_t, s);
    return e == hipSuccess ? XCT_OK : hip_fail(e);
}

int xct_offset_detector(const xct_geometry *g, int32_t *n_virtual, double *center_virtual)
{
    if (int rc = check_geometry(g, false)) return rc;
    if (!n_virtual || !center_virtual) return XCT_EINVAL;
    const double m = 2.0 * g->center;
    if (std::fabs(m - std::nearbyint(m)) > 1e-9) return XCT_EINVAL;
    if (g->center < 0.0 || g->center > g->n_det - 1) return XCT_EINVAL;
    int nv, first;
    double cv;
    offset_virtual(g, &nv, &cv, &first);
    *n_virtual = nv;
    *center_virtual = cv;
    return XCT_OK;
}

int xct_filter_offset(const xct_geometry *g, int32_t n_slices, const void *sino, int32_t sino_t,
                      void *filtered, int32_t filtered_t, int32_t window, double overlap,
                      xct_stream stream)
{
    if (int rc = check_geometry(g, false)) return rc;
    if (int rc = check_slices(g, n_slices)) return rc;
    if (!sino || !filtered || sino == filtered) return XCT_EINVAL;
    if (!dtype_ok(sino_t) || !dtype_ok(filtered_t)) return XCT_EDTYPE;
    if (window < XCT_RAM_LAK || window > XCT_HANN) return XCT_EDTYPE;
    if (int rc = check_offset(g, overlap)) return rc;
    int nv, first;
    double cv;
    offset_virtual(g, &nv, &cv, &first);
    if (nv > kMaxFFT / 2) return XCT_ETOOBIG;
    hipStream_t s = (hipStream_t)stream;
    EntryRef ft, w;
    if (int rc = filter_tables(nv, window, g->det_pitch, s, &ft)) return rc;
    if (int rc = offset_weights(g, overlap, s, &w)) return rc;
    FilterArgs a{};
    a.in = sino;
    a.out = filtered;
    a.tw = ft->table<float2>(0);
    a.H = ft->table<float>(1);
    a.weight = w->table<float>(0);
    a.in_first = first;
    a.in_len = g->n_det;
    a.rows = (int64_t)n_slices * g->n_angles;
    a.nc = nv;
    a.L = ft->L;
    a.log2L = ft->lg;
    hipError_t e = launch_filter(a, sino_t, filtered_t, s);
    return e == hipSuccess ? XCT_OK : hip_fail(e);
}

int xct_preprocess_filter(const xct_geometry *g, int32_t n_rows, int32_t row_begin, int32_t n_slices,
                          const void *proj, int32_t proj_t, const float *dark, const float *flat,
                          float floor, float blur_sigma, void *filtered, int32_t filtered_t,
                          int32_t window, xct_stream stream)
{
    if (int rc = check_geometry(g, false)) return rc;
    if (int rc = check_slices(g, n_slices)) return rc;
    if (n_rows < 1 || row_begin < 0 || (int64_t)row_begin + n_slices > n_rows) return XCT_EINVAL;
    if (!proj || !dark || !flat || !filtered) return XCT_EINVAL;
    if ((proj_t != XCT_U16 && proj_t != XCT_F32) || !dtype_ok(filtered_t)) return XCT_EDTYPE;
    if (window < XCT_RAM_LAK || window > XCT_HANN) return XCT_EDTYPE;
    if (!std::isfinite(floor) || !(floor >= std::numeric_limits<float>::min())) return XCT_EINVAL;
    if (!std::isfinite(blur_sigma) || blur_sigma < 0.0f) return XCT_EINVAL;
    if (g->n_det > kMaxFFT / 2) return XCT_ETOOBIG;
    if ((double)g->n_angles * n_rows * g->n_det > 4.0e18) return XCT_ETOOBIG;
    const int radius = blur_sigma == 0.0f ? 0 : (int)(4.0 * (double)blur_sigma + 0.5);
    if (radius > 64) return XCT_ETOOBIG;
    // the output must not overlap the projection stack
    const char *pb = static_cast<const char *>(proj), *fb = static_cast<const char *>(filtered);
    const size_t pbytes = (size_t)g->n_angles * n_rows * g->n_det * dtype_size(proj_t);
    const size_t fbytes = (size_t)n_slices * g->n_angles * g->n_det * dtype_size(filtered_t);
    if (pb < fb + fbytes && fb < pb + pbytes) return XCT_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    EntryRef ft, taps;
    if (int rc = filter_tables(g->n_det, window, g->det_pitch, s, &ft)) return rc;
    if (radius > 0)
        if (int rc = blur_taps(blur_sigma, radius, s, &taps)) return rc;
    FilterArgs a{};
    a.in = proj;
    a.out = filtered;
    a.tw = ft->table<float2>(0);
    a.H = ft->table<float>(1);
    a.rows = (int64_t)n_slices * g->n_angles;
    a.nc = g->n_det;
    a.L = ft->L;
    a.log2L = ft->lg;
    a.pre.dark = dark;
    a.pre.flat = flat;
    a.pre.taps = taps ? taps->table<float>(0) : nullptr;
    a.pre.radius = radius;
    a.pre.n_rows = n_rows;
    a.pre.row_begin = row_begin;
    a.pre.n_angles = g->n_angles;
    a.pre.floor = floor;
    hipError_t e = launch_front_end_filter(a, proj_t, filtered_t, s);
    return e == hipSuccess ? XCT_OK : hip_fail(e);
}

// Back-projection of one slab (all entry points but the batch).  `least`:
// voxel updates from which the matrix cores are considered.
static int backproject_one(const xct_geometry *g, int32_t n_slices, const void *sino, int32_t sino_t,
                           void *image, float scale, int32_t accumulate, int out_u16, float code_a,
                           float code_b, double least, hipStream_t s)
{
    BPJob j;
    j.g = g;
    j.n_slices = n_slices;
    j.sino = sino;
    j.image = image;
    j.scale = scale;
    j.accumulate = accumulate ? 1 : 0;
    j.path = choose_path(g, &j.sets);
    j.out_u16 = out_u16;
    j.code_a = code_a;
    j.code_b = code_b;
    if (limit_items(j) >= kMaxItems) return XCT_ETOOBIG;
    if (int rc = geo_tables(g, s, &j.t)) return rc;
    const double updates = (double)n_slices * g->n_angles * g->nx * g->ny;
    if (updates >= least) pair_slices(j);
    if (least == 0.0) plan_alone(j);
    MXPlan p;
    if (updates >= least) p = mx_plan(j, sino_t);
    // Scratch in stream-ordered memory.  A stream under capture, or no memory,
    // takes whole walks of the vector kernels, which need none.
    const size_t bytes = p.cols ? mx_scratch_bytes(j, p) : part_bytes(j);
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    void *scratch = nullptr;
    if (bytes && hipStreamIsCapturing(s, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone) {
        keep_stream_pool();
        if (hipMallocAsync(&scratch, bytes, s) != hipSuccess) scratch = nullptr;
    }
    (void)hipGetLastError();
    if (!scratch) return launch_bp_jobs({j}, sino_t, nullptr, nullptr, s);
    const int rc = p.cols ? launch_bp_matrix(j, p, sino_t, scratch, s) : launch_bp_parts(j, sino_t, static_cast<float *>(scratch), s);
    const hipError_t e = hipFreeAsync(scratch, s);
    return rc ? rc : e == hipSuccess ? XCT_OK : hip_fail(e);
}

int xct_backproject(const xct_geometry *g, int32_t n_slices, const void *sino, int32_t sino_t,
                    float *image, float scale, int32_t accumulate, xct_stream stream)
{
    if (int rc = check_geometry(g, true)) return rc;
    if (int rc = check_slices(g, n_slices)) return rc;
    if (!sino || !image) return XCT_EINVAL;
    if (!dtype_ok(sino_t)) return XCT_EDTYPE;
    if (!std::isfinite(scale)) return XCT_EINVAL;
    return backproject_one(g, n_slices, sino, sino_t, image, scale, accumulate, 0, 0.0f, 0.0f,
                           kMXLeastUpdates, (hipStream_t)stream);
}

int xct_backproject_u16(const xct_geometry *g, int32_t n_slices, const void *sino, int32_t sino_t,
                        uint16_t *image, float scale, double mu_water, double hu_min, double hu_max,
                        xct_stream stream)
{
    if (int rc = check_geometry(g, true)) return rc;
    if (int rc = check_slices(g, n_slices)) return rc;
    if (!sino || !image) return XCT_EINVAL;
    if (!dtype_ok(sino_t)) return XCT_EDTYPE;
    if (!std::isfinite(scale) || !std::isfinite(mu_water) || !std::isfinite(hu_min) ||
        !std::isfinite(hu_max) || !(mu_water > 0.0) || !(hu_max > hu_min))
        return XCT_EINVAL;
    // code = A mu + B: HU = 1000 (mu - mu_water) / mu_water, [hu_min, hu_max] -> [0, 65535]
    const double span = 65535.0 / (hu_max - hu_min);
    const double A = 1000.0 / mu_water * span;
    const double B = (-1000.0 - hu_min) * span;
    const float a32 = (float)A, b32 = (float)B;
    if (!std::isfinite(a32) || !std::isfinite(b32)) return XCT_EINVAL;
    return backproject_one(g, n_slices, sino, sino_t, image, scale, 0, 1, a32, b32, kMXLeastUpdates,
                           (hipStream_t)stream);
}

// Parts of a forward projection of `triples` workgroups walking `side` steps
// each, `bytes` of sinogram, `room` for parts of it.  Fewer workgroups than the device holds (four per
// CU) take the time of one workgroup's walk (one 512^2 slice, 720 angles: 180
// workgroups, 450 us), so walks are split until there are about two rounds of
// them, down to 32 steps; then halved to 16 while one round holds them all, and
// to 8 (four slices: shorter than one slice's stages) while each has a CU's LDS
// to itself.  Three 64^2 slices, 90 angles: 58 us with 32 steps, 41 with 16, 37
// with 8; five 256^2 slices, 360 angles: 87 us in eight parts of 32 steps (768
// workgroups), 93 in ten, 95 in sixteen.
static int fp_parts(int64_t triples, int side, int sl, size_t bytes, size_t room)
{
    const int64_t cus = device_cus(), slots = 4 * cus;
    if (triples >= slots) {
        // More than one round ends with a tail of some 0.9 rounds of whole
        // walks (1024^2, 1440 angles, 4 to 32 slices: 1.45 ms a round of 1024
        // workgroups and 1.3 ms besides).  Parts shorten it, for some 16 steps
        // each and the passes over their sums: 8 slices 2.88 ms whole, 2.30 in
        // two parts, 2.08 in four; 64 slices of 512^2, 720 angles: 2.28, 2.18,
        // 2.30; 8 of 2048^2, 1024 angles: 11.9, 9.3, 8.4.
        double best = 0.0;
        int parts = 1;
        for (int64_t p = 1; p <= 4 && side / p >= 64 && (p == 1 || (size_t)p * bytes <= room); ++p) {
            const double us = 1.41 * (side + 16.0 * p) * triples / slots + 1.27 * side / p +
                              (p > 1 ? 15.0 + p * bytes / 2e6 : 0.0);
            if (p == 1 || us < best) best = us, parts = (int)p;
        }
        return parts;
    }
    // (more than half a round: parts of up to 64 steps at least, as whole walks
    // leave less idle; 64^2, 384 angles, 152 slices, 912 workgroups, 119 us whole
    // and 162 in two parts, 200^2, 768 workgroups 318 and 285 in three)
    const double filled = std::max(1.0, 2.0 * triples / slots);
    const int steps = (int)std::min(64.0, 32.0 * filled * filled);
    int64_t p = std::max<int64_t>(1, std::min<int64_t>((2 * slots + triples - 1) / triples, side / steps));
    while (side / (2 * p) >= 16 && triples * 2 * p <= slots) p *= 2;
    while (sl == 4 && side / (2 * p) >= 8 && triples * 2 * p <= cus) p *= 2;
    return p * bytes <= (size_t)kPartBytes ? (int)p : 1;
}

// Angle k is k pi / N_p, N_p even.
static bool uniform_half_turn(const xct_geometry *g)
{
    if (g->n_angles & 1) return false;
    for (int k = 0; k < g->n_angles; ++k)
        if (std::fabs(g->angles[k] - k * (M_PI / g->n_angles)) > 1e-9) return false;
    return true;
}

// P = (pixel^2 / pitch) A, the projector of the least-squares problem.
static double projector_scale(const xct_geometry *g) { return g->pixel_size * g->pixel_size / g->det_pitch; }

}  // extern "C"

// Square slices under a uniform half turn: the projections of one slice at
// angles k, k + H, N - k and H - k (H = N_p / 2) are those of the slice, and of
// the slice turned, reflected and transposed, at angle k, so the first quarter
// of the angles of four copies gives all rows, each weight shared by four
// values as in a group of four slices.  That saves three quarters of one or two
// slices' walks, and of more slices the walks of the last group's absent ones;
// it costs the copies, 64 bytes of traffic per pixel, some 50 angles' worth of
// three quarters of a walk.  1024^2, one slice: 16 angles 114 us against 122
// without, 64 angles 148 against 274, 1440 angles 320 against 634; three
// slices: 16 angles 212 against 204, 1440 angles 858 against 1057; seven
// slices: 64 angles 831 against 823, 1440 angles 1815 against 2800.  Below
// 512^2 a call is as long as its launches: one 256^2 slice, 360 angles, 46 us
// against 43.
static bool fp_turns(const xct_geometry *g, int n_slices)
{
    if (n_slices % 4 == 0 || g->nx != g->ny || g->nx < 512) return false;
    const int64_t saved = n_slices <= 2 ? 3 * n_slices : 4 - n_slices % 4;
    return saved * g->n_angles >= (int64_t)144 * n_slices && uniform_half_turn(g);
}

// sino = (base ? base : accumulate ? sino : 0) + alpha P image; `scratch`:
// with turned copies and split walks where they are faster.
static int forward_form(const xct_geometry *g, int32_t n_slices, const float *image, const float *base,
                        float *sino, float alpha, int32_t accumulate, bool scratch, hipStream_t s)
{
    // (the whole set's plan also where the turned copies need a quarter's alone:
    // a later call under capture takes it, and may not be its geometry's first)
    EntryRef t;
    if (int rc = fp_tables(g, s, &t)) return rc;
    // one workgroup per (slice group, bin block, angle block), indexed in 32 bits
    const int64_t bin_blocks = (g->n_det + kFPBins - 1) / kFPBins;
    const int whole = n_slices >= 3 && t->fp_four ? 4 : 1;
    if (t->n_blocks * bin_blocks * ((n_slices + whole - 1) / whole) >= ((int64_t)1 << 31)) return XCT_ETOOBIG;
    bool turned = scratch && fp_turns(g, n_slices);
    if (turned) {
        xct_geometry quarter = *g;
        quarter.n_angles = g->n_angles / 4 + 1;
        EntryRef q;
        if (int rc = fp_tables(&quarter, s, &q)) return rc;
        turned = q->fp_four;
        if (turned) t = q;
    }
    FPArgs a{};
    a.turned = turned;
    a.image = image;
    a.sino = sino;
    a.base = base;
    a.ang = t->table<FPAngle>(0);
    a.blocks = t->table<FPBlock>(1);
    a.n_blocks = t->n_blocks;
    a.bin_blocks = (int32_t)bin_blocks;
    // four slices per workgroup share coordinates and weights; a call with
    // one or two slices, without turned copies, keeps one per workgroup
    const int sl = turned || (n_slices >= 3 && t->fp_four) ? 4 : 1;
    const int64_t groups = turned ? n_slices : (n_slices + sl - 1) / sl;
    const int64_t triples = a.n_blocks * bin_blocks * groups;
    if (triples >= ((int64_t)1 << 31)) return forward_form(g, n_slices, image, base, sino, alpha, accumulate, false, s);
    a.scale = (float)((double)alpha * projector_scale(g));
    a.accumulate = accumulate ? 1 : 0;
    a.n_angles = g->n_angles;
    a.n_det = g->n_det;
    a.nx = g->nx;
    a.ny = g->ny;
    a.n_slices = n_slices;
    a.parts = 1;
    const size_t sino_bytes = sizeof(float) * (size_t)n_slices * g->n_angles * g->n_det;
    // Four slices per workgroup read four-slice copies of the image and of
    // its transpose, made chunk by chunk of slice groups in stream-ordered
    // memory (kQuadBytes, or one group when a group needs more); what is left
    // of the memory that the pool keeps is room for parts.
    const int64_t plane = (int64_t)g->nx * g->ny;
    const int64_t group_bytes = sl == 4 ? 2 * plane * (int64_t)sizeof(float4) : 0;
    const int64_t per = sl == 4 ? std::max<int64_t>(1, std::min<int64_t>(groups, kQuadBytes / group_bytes)) : groups;
    const int64_t room = std::max<int64_t>(kPartBytes, kQuadBytes + kPartBytes - per * group_bytes);
    if (scratch && per == groups) a.parts = fp_parts(triples, std::min(g->nx, g->ny), sl, sino_bytes, (size_t)room);
    if (sl == 1 && a.parts == 1) {
        const hipError_t e = launch_forward(a, 1, s);
        return e == hipSuccess ? XCT_OK : hip_fail(e);
    }
    keep_stream_pool();
    char *buf = nullptr;
    const size_t part_bytes = a.parts > 1 ? align256(a.parts * sino_bytes) : 0;
    hipError_t e = hipMallocAsync(reinterpret_cast<void **>(&buf), part_bytes + (size_t)(per * group_bytes), s);
    if (e != hipSuccess && (turned || a.parts > 1)) {  // no memory for these: the form that needs the least
        (void)hipGetLastError();
        return forward_form(g, n_slices, image, base, sino, alpha, accumulate, false, s);
    }
    if (e != hipSuccess) return hip_fail(e);
    a.partial = reinterpret_cast<float *>(buf);
    if (sl == 1) {
        e = launch_forward(a, 1, s);
    } else {
        float4 *quad = reinterpret_cast<float4 *>(buf + part_bytes), *quad_t = quad + per * plane;
        for (int64_t g0 = 0; g0 < groups && e == hipSuccess; g0 += per) {
            const int64_t z = turned ? g0 : 4 * g0;
            const int ns = (int)std::min<int64_t>(n_slices - z, turned ? per : 4 * per);
            e = turned ? launch_forward_turned(image + z * plane, ns, g->nx, quad, quad_t, s)
                       : launch_forward_quads(image + z * plane, ns, g->nx, g->ny, quad, quad_t, s);
            if (e != hipSuccess) break;
            FPArgs c = a;
            c.image = image + z * plane;
            c.sino = sino + z * (int64_t)g->n_angles * g->n_det;
            if (base) c.base = base + z * (int64_t)g->n_angles * g->n_det;
            c.n_slices = ns;
            c.quad = quad;
            c.quad_t = quad_t;
            e = launch_forward(c, 4, s);
        }
    }
    const hipError_t f = hipFreeAsync(buf, s);
    if (e == hipSuccess) e = f;
    return e == hipSuccess ? XCT_OK : hip_fail(e);
}

static int forward_project(const xct_geometry *g, int32_t n_slices, const float *image, const float *base,
                           float *sino, float alpha, int32_t accumulate, xct_stream stream)
{
    if (int rc = check_geometry(g, true)) return rc;
    if (int rc = check_slices(g, n_slices)) return rc;
    if (!image || !sino) return XCT_EINVAL;
    if (!std::isfinite(alpha)) return XCT_EINVAL;
    if (n_slices > 65535) return XCT_ETOOBIG;
    // under capture one or two slices take no scratch
    hipStream_t s = (hipStream_t)stream;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    const bool scratch = hipStreamIsCapturing(s, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone;
    if (!scratch) (void)hipGetLastError();
    return forward_form(g, n_slices, image, base, sino, alpha, accumulate, scratch, s);
}

extern "C" {

int xct_forward_project(const xct_geometry *g, int32_t n_slices, const float *image, float *sino,
                        float alpha, int32_t accumulate, xct_stream stream)
{
    return forward_project(g, n_slices, image, nullptr, sino, alpha, accumulate, stream);
}

int xct_forward_residual(const xct_geometry *g, int32_t n_slices, const float *image, const float *y,
                         float *r, float alpha, xct_stream stream)
{
    if (!y) return XCT_EINVAL;
    return forward_project(g, n_slices, image, y, r, alpha, 0, stream);
}

int xct_project_adjoint(const xct_geometry *g, int32_t n_slices, const float *sino, float *image,
                        float alpha, int32_t accumulate, xct_stream stream)
{
    if (int rc = check_geometry(g, true)) return rc;
    if (int rc = check_slices(g, n_slices)) return rc;
    if (!sino || !image) return XCT_EINVAL;
    if (!std::isfinite(alpha)) return XCT_EINVAL;
    return backproject_one(g, n_slices, sino, XCT_F32, image, (float)((double)alpha * projector_scale(g)),
                           accumulate, 0, 0.0f, 0.0f, 0.0, (hipStream_t)stream);
}

// Detector bins of a slab's filtered rows: the virtual (mirrored) detector
// for an offset scan, the physical one otherwise.
static int filtered_bins(const xct_slab &sl)
{
    if (sl.offset_overlap == 0.0) return sl.geom.n_det;
    int nv, first;
    double cv;
    offset_virtual(&sl.geom, &nv, &cv, &first);
    return nv;
}

static int check_slabs(const xct_slab *slabs, int32_t n_slabs, bool need_data)
{
    if (!slabs || n_slabs <= 0) return XCT_EINVAL;
    if (n_slabs > kMaxSlabs) return XCT_ETOOBIG;
    for (int i = 0; i < n_slabs; ++i) {
        if (int rc = check_geometry(&slabs[i].geom, true)) return rc;
        if (int rc = check_slices(&slabs[i].geom, slabs[i].n_slices)) return rc;
        if (slabs[i].offset_overlap != 0.0)
            if (int rc = check_offset(&slabs[i].geom, slabs[i].offset_overlap)) return rc;
        if (filtered_bins(slabs[i]) > kMaxFFT / 2) return XCT_ETOOBIG;
        if (need_data && (!slabs[i].sino || !slabs[i].image)) return XCT_EINVAL;
    }
    return XCT_OK;
}

// Workspace layout of xct_fbp_batch: 256 bytes of work counters (kXcds per
// launch group), the slab descriptor table, then the filtered rows of every
// slab, each region 256-byte aligned.
static size_t table_bytes(int32_t n_slabs) { return align256(sizeof(BPSlab) * (size_t)n_slabs); }

// Back-projection job of a batch's slab over its filtered rows `filt`: the
// slab's geometry (`virt`: its copy with the virtual detector of an offset
// scan) and weight.
static BPJob slab_job(const xct_slab &sl, xct_geometry *virt)
{
    BPJob j;
    j.g = &sl.geom;
    double weight = M_PI / sl.geom.n_angles;
    if (sl.offset_overlap != 0.0) {
        int first;
        *virt = sl.geom;
        offset_virtual(&sl.geom, &virt->n_det, &virt->center, &first);
        j.g = virt;
        weight = 2.0 * M_PI / sl.geom.n_angles;
    }
    j.n_slices = sl.n_slices;
    j.image = sl.image;
    j.scale = (float)weight;
    j.accumulate = 0;
    j.path = choose_path(j.g, &j.sets);
    pair_slices(j);
    return j;
}

// Filtered rows of a slab in the workspace, and the bytes of the workspace's
// counters, table and filtered rows.
static size_t rows_bytes(const xct_slab &sl, int32_t filtered_t)
{
    return align256((size_t)sl.n_slices * sl.geom.n_angles * filtered_bins(sl) * dtype_size(filtered_t));
}

static size_t base_bytes(const xct_slab *slabs, int32_t n_slabs, int32_t filtered_t)
{
    size_t bytes = 256 + table_bytes(n_slabs);
    for (int i = 0; i < n_slabs; ++i) bytes += rows_bytes(slabs[i], filtered_t);
    return bytes;
}

// How a batch takes its slabs (in their order): each slab's job (its rows not
// yet set) and, where it takes the matrix cores, its plan there.
struct BatchPlan {
    std::vector<xct_geometry> virt;  // virtual detectors of offset slabs
    std::vector<BPJob> jobs;
    std::vector<MXPlan> mx;
    size_t scratch = 0;  // bytes behind the base: the matrix-core launches use them in turn, then the split slabs' copies
};

// Launch groups of a batch: the generic kernel; slices in pairs, the mirror and
// the symmetric kernel, each with one slice (pair) per item or two.
enum { kGroupGeneric = 0, kGroupPairs1, kGroupPairs2, kGroupPairs3, kGroupMirror1, kGroupMirror2, kGroupSym1, kGroupSym2, kGroups };

static int launch_group(const BPJob &j)
{
    const int spi = item_slices(j), two = spi == 2;
    return j.path == kPathGeneric  ? kGroupGeneric
           : j.path == kPathPairs  ? (spi == 3 ? kGroupPairs3 : two ? kGroupPairs2 : kGroupPairs1)
           : j.path == kPathMirror ? (two ? kGroupMirror2 : kGroupMirror1)
                                   : (two ? kGroupSym2 : kGroupSym1);
}

static void batch_jobs(const xct_slab *slabs, int32_t n_slabs, BatchPlan &b)
{
    b.virt.resize(n_slabs);
    b.jobs.reserve(n_slabs);
    for (int i = 0; i < n_slabs; ++i) b.jobs.push_back(slab_job(slabs[i], &b.virt[i]));
}

// The limit on the items of a launch, for each kernel's slabs together (one
// slice per item apart from two).
static int check_batch_items(const BatchPlan &b)
{
    int64_t items[4][2] = {};
    for (const BPJob &j : b.jobs)
        if ((items[j.path == kPathPairs ? (int)kPathGeneric : j.path][j.path != kPathPairs && item_slices(j) == 2] += limit_items(j)) >= kMaxItems)
            return XCT_ETOOBIG;
    return XCT_OK;
}

// Estimated time of the jobs' launches in turn, a group at a time, and of the
// sum of the split jobs' copies.  A group of items that the device holds at once,
// or of items that are all alike, takes its rounds; else the items' shares of the
// device and for the tail part of a mean walk, or what the longest walk, begun
// at the rate of a full device, has left.
static double launches_ns(const std::vector<BPJob> &jobs)
{
    struct Group { int64_t items = 0; double least = 0, most = 0, share = 0, walks = 0; KernelTimes t; } groups[kGroups];
    double sums = 0, ns = 0;
    auto angles = [](const BPJob &j) { return (double)item_angles(j); };
    int spi;
    for (const BPJob &j : jobs) {
        Group &grp = groups[launch_group(j)];
        grp.least = grp.items ? std::min(grp.least, angles(j)) : angles(j);
        grp.most = std::max(grp.most, angles(j));
        grp.items += vector_items(j, &spi) * j.parts;
    }
    for (const BPJob &j : jobs) {
        Group &grp = groups[launch_group(j)];
        const double n = (double)vector_items(j, &spi) * j.parts;
        grp.t = vector_times(j.path, spi, grp.items, j.cus);
        const double walk = grp.t.full * angles(j) + grp.t.store;
        grp.share += n / (grp.t.per_cu * (double)j.cus) * walk;
        grp.walks += n * walk;
        if (j.parts > 1) sums += 1000.0 + (j.parts + 1) * (double)image_bytes(j) / 6700.0;
    }
    for (const Group &grp : groups) {
        if (!grp.items) continue;
        const int cus = jobs[0].cus;
        const double left = std::max(0.0, grp.most - grp.share / grp.t.full) * grp.t.alone;
        ns += 6000.0 + (grp.items <= grp.t.per_cu * (int64_t)cus || grp.least == grp.most
                            ? rounds_ns(grp.t, grp.items, cus, grp.most, 1)
                            : grp.share + std::max(left, 0.4 * grp.walks / grp.items));
    }
    return ns + (sums > 0 ? 5000.0 + sums : 0.0);
}

// How the vector kernels take a batch's slabs, given as they are taken alone,
// with an estimate of the time.  Either that way, with no more parts for a slab
// than cut the longest walks into four, three or two, where that saves 5 %, and
// the room for copies to the longest walks first (8 slabs of 1 to 2 x 68^2 to
// 1540 x 1138, 76 to 1484 angles: 1.22 ms, 2.26 where copies larger than the room
// left every slab whole).  Or in whole walks, where slices of any geometry go in
// pairs only if that is worth launches of their own behind the generic kernel's
// (25 slabs of 1 to 30 slices of 63^2 to 1588^2: triples, pairs, single pairs and
// the rest in four launches 2.15 ms, in one 0.90).  Whole walks are preferred up to 3 %.
static double plan_vector(std::vector<BPJob> &jobs)
{
    std::vector<int> order;
    int longest = 0;
    bool generic = false;
    for (size_t i = 0; i < jobs.size(); ++i) {
        generic = generic || jobs[i].path == kPathPairs || jobs[i].path == kPathGeneric;
        if (jobs[i].parts < 2) continue;
        order.push_back((int)i);
        longest = std::max(longest, jobs[i].g->n_angles);
    }
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return jobs[x].g->n_angles > jobs[y].g->n_angles; });

    std::vector<BPJob> apart, whole;
    double apart_ns = 0, whole_ns = 0;
    for (int most : {0, 4, 3, 2}) {
        std::vector<BPJob> v = jobs;
        size_t room = (size_t)kPartBytes;
        for (int i : order) {
            BPJob &j = v[i];
            if (most) set_parts(j, std::min<int64_t>(j.parts, ((int64_t)j.g->n_angles * most + longest - 1) / longest));
            const size_t bytes = part_bytes(j);
            if (bytes <= room) room -= bytes;
            else j.parts = 1;
        }
        const double ns = launches_ns(v);
        if (!most || ns < 0.95 * apart_ns) {
            apart_ns = ns;
            apart.swap(v);
        }
        if (order.empty()) break;
    }
    for (int pairs = 0; pairs < (generic ? 8 : 1); ++pairs) {  // a bit for each of the groups in pairs
        std::vector<BPJob> v = jobs;
        for (BPJob &j : v) {
            j.parts = 1;
            if (j.path == kPathPairs) j.path = kPathGeneric;
            BPJob two = j;
            pair_slices(two);
            if (two.path == kPathPairs && (pairs >> (launch_group(two) - kGroupPairs1) & 1)) j.path = kPathPairs;
        }
        const double ns = launches_ns(v);
        if (!pairs || ns < whole_ns) {
            whole_ns = ns;
            whole.swap(v);
        }
    }
    jobs.swap(whole_ns < 1.03 * apart_ns ? whole : apart);
    return std::min(whole_ns, apart_ns);
}

// A slab alone is split, or goes to the matrix cores, partly because it leaves
// the device idle otherwise.  In a batch that is no reason where the slabs fill
// the device together: slabs that the matrix cores are not faster for per
// share of the device join the vector launches when those are estimated to take
// less than the slabs' launches in turn (64 slabs of one 512^2 slice, 720
// angles: 1.9 ms, and 2.5 on the matrix cores; 32 of four slices 2.4 and 3.3).
static void plan_batch(int32_t n_slabs, int32_t filtered_t, BatchPlan &b)
{
    b.mx.resize(n_slabs);
    std::vector<int> joins;
    double turns = 0;
    std::vector<BPJob> apart, joined;  // the vector kernels' jobs without and with those slabs
    for (int i = 0; i < n_slabs; ++i) {
        BPJob &j = b.jobs[i];
        plan_alone(j);
        b.mx[i] = mx_plan(j, filtered_t);
        const bool may_join = n_slabs > 1 && b.mx[i].cols && b.mx[i].ns >= vector_share_ns(j);
        if (may_join) {
            joins.push_back(i);
            turns += b.mx[i].ns;
        }
        if (!b.mx[i].cols) apart.push_back(j);
        if (may_join || !b.mx[i].cols) joined.push_back(j);
    }
    if (n_slabs > 1) {
        turns += plan_vector(apart);
        if (!joins.empty() && plan_vector(joined) < turns) {
            for (int i : joins) b.mx[i] = MXPlan();
            apart.swap(joined);
        }
    }
    size_t parts = 0, next = 0;
    for (int i = 0; i < n_slabs; ++i) {
        if (b.mx[i].cols) {
            b.scratch = std::max(b.scratch, mx_scratch_bytes(b.jobs[i], b.mx[i]));
        } else {
            b.jobs[i] = apart[next++];
            parts += part_bytes(b.jobs[i]);
        }
    }
    b.scratch = std::max(b.scratch, parts);
}

size_t xct_fbp_workspace_bytes(const xct_slab *slabs, int32_t n_slabs, int32_t filtered_t)
{
    if (check_slabs(slabs, n_slabs, false) || !dtype_ok(filtered_t)) return 0;
    BatchPlan b;
    batch_jobs(slabs, n_slabs, b);
    plan_batch(n_slabs, filtered_t, b);
    return base_bytes(slabs, n_slabs, filtered_t) + b.scratch;
}

int xct_fbp_batch(const xct_slab *slabs, int32_t n_slabs, int32_t sino_t, int32_t window,
                  int32_t filtered_t, void *workspace, size_t workspace_bytes, xct_stream stream)
{
    static_assert(8 * kXcds * sizeof(unsigned int) <= 256, "work counters exceed their region");
    if (int rc = check_slabs(slabs, n_slabs, true)) return rc;
    if (!dtype_ok(sino_t) || !dtype_ok(filtered_t)) return XCT_EDTYPE;
    if (window < XCT_RAM_LAK || window > XCT_HANN) return XCT_EDTYPE;
    const size_t base = base_bytes(slabs, n_slabs, filtered_t);
    if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < base) return XCT_EWORKSPACE;
    BatchPlan b;
    batch_jobs(slabs, n_slabs, b);
    if (int rc = check_batch_items(b)) return rc;
    hipStream_t s = (hipStream_t)stream;

    char *ws = static_cast<char *>(workspace);
    unsigned int *counters = reinterpret_cast<unsigned int *>(ws);
    BPSlab *table = reinterpret_cast<BPSlab *>(ws + 256);
    std::vector<char *> rows(n_slabs);  // of each slab
    rows[0] = ws + 256 + table_bytes(n_slabs);
    for (int i = 1; i < n_slabs; ++i) rows[i] = rows[i - 1] + rows_bytes(slabs[i - 1], filtered_t);
    auto filter_slab = [&](int i) {
        const xct_slab &sl = slabs[i];
        // (an offset scan's redundancy-weighted rows are filtered on the virtual detector)
        return sl.offset_overlap != 0.0 ? xct_filter_offset(&sl.geom, sl.n_slices, sl.sino, sino_t, rows[i], filtered_t, window, sl.offset_overlap, stream)
                                        : xct_filter(&sl.geom, sl.n_slices, sl.sino, sino_t, rows[i], filtered_t, window, stream);
    };
    // The host weighs the back-projections' forms (some 3 us a slab) while
    // filters run: the first slab's, so that a matrix-core launch of the others
    // finds its rows in cache (three slabs of up to 4 x 2048^2: 3.57 ms, 3.60
    // with all filters first), or of many slabs all of them.
    const int ahead = n_slabs > 8 ? n_slabs : 1;
    for (int i = 0; i < ahead; ++i)
        if (int rc = filter_slab(i)) return rc;
    plan_batch(n_slabs, filtered_t, b);
    // without the scratch every slab takes whole walks of the vector kernels
    if (workspace_bytes < base + b.scratch) {
        std::fill(b.mx.begin(), b.mx.end(), MXPlan());
        for (BPJob &j : b.jobs) j.parts = 1;
        plan_vector(b.jobs);
    }
    float *partial = reinterpret_cast<float *>(ws + base);
    std::vector<BPJob> groups[kGroups];
    for (int i = 0; i < n_slabs; ++i) {
        if (i >= ahead)
            if (int rc = filter_slab(i)) return rc;
        BPJob &j = b.jobs[i];
        j.sino = rows[i];
        if (int rc = geo_tables(j.g, s, &j.t)) return rc;
        if (b.mx[i].cols) {
            if (int rc = launch_bp_matrix(j, b.mx[i], filtered_t, ws + base, s)) return rc;
            continue;
        }
        if (part_bytes(j)) {
            j.partial = partial;
            partial += part_bytes(j) / sizeof(float);
        } else {
            j.parts = 1;
        }
        groups[launch_group(j)].push_back(j);
    }
    // A group whose items all fit on the device at once is launched with one
    // workgroup per item: no counters, and no workgroup that asks every XCD's
    // counter in turn before it ends (some 10 us of a call with one item each).
    // So is one of less than a millisecond whose items all walk as many angles (26 x
    // 780^2 x 33 angles 118 us, 166 with counters; longer, their order keeps rows
    // in cache: 46 x 1554^2 x 660, pixel 1.3, 7.5 ms with them, 8.0 without).
    bool persistent[kGroups], any = false;
    for (int grp = 0; grp < kGroups; ++grp) {
        int64_t items = 0;
        int spi = 1;
        bool alike = true;
        for (const BPJob &j : groups[grp]) {
            items += vector_items(j, &spi) * j.parts;
            alike = alike && item_angles(j) == item_angles(groups[grp][0]);
        }
        persistent[grp] = false;
        if (!items) continue;
        const BPJob &j = groups[grp][0];
        const KernelTimes t = vector_times(j.path, spi, items, j.cus);
        persistent[grp] = items > t.per_cu * (int64_t)j.cus &&
                          (!alike || rounds_ns(t, items, j.cus, item_angles(j), 1) >= 1e6);
        any = any || persistent[grp];
    }
    hipError_t e = any ? launch_fill_u32(counters, kGroups * kXcds, 0u, s) : hipSuccess;
    if (e != hipSuccess) return hip_fail(e);
    // each group reads its descriptors from its own part of the table
    BPSlab *group_table[kGroups];
    size_t first = 0;
    for (int grp = kGroups - 1; grp >= 0; --grp) {
        group_table[grp] = table + first;
        first += groups[grp].size();
    }
    for (int grp = kGroups - 1; grp >= 0; --grp)
        if (int rc = launch_bp_jobs(groups[grp], filtered_t, persistent[grp] ? counters + grp * kXcds : nullptr, group_table[grp], s))
            return rc;
    std::vector<SumJob> sums;
    for (const auto &grp : groups)
        for (const BPJob &j : grp)
            if (j.partial)
                sums.push_back({static_cast<float *>(j.image), j.partial, (int64_t)j.n_slices * j.g->nx * j.g->ny, j.parts});
    // (one image: four elements a thread where it is large)
    if (sums.size() == 1)
        e = launch_sum_parts(sums[0].image, sums[0].partial, (int)sums[0].parts, sums[0].n, 0, nullptr, s);
    else
        e = launch_sum_jobs(sums.data(), (int)sums.size(), s);
    return e == hipSuccess ? XCT_OK : hip_fail(e);
}

size_t xct_reduce_workspace_bytes(int64_t n)
{
    if (n <= 0) return 0;
    return sizeof(double) * (size_t)reduce_blocks(n);
}

static int reduce_common(const float *a, const float *b, int64_t n, double *result, void *workspace,
                         size_t workspace_bytes, int sqdist, xct_stream stream)
{
    if (!a || !b || !result || n <= 0) return XCT_EINVAL;
    if (!workspace || ((uintptr_t)workspace & 7) || workspace_bytes < xct_reduce_workspace_bytes(n))
        return XCT_EWORKSPACE;
    hipError_t e = launch_reduce(a, b, n, result, static_cast<double *>(workspace), reduce_blocks(n),
                                 sqdist, (hipStream_t)stream);
    return e == hipSuccess ? XCT_OK : hip_fail(e);
}

int xct_dot_f64(const float *a, const float *b, int64_t n, double *result, void *workspace,
                size_t workspace_bytes, xct_stream stream)
{
    return reduce_common(a, b, n, result, workspace, workspace_bytes, 0, stream);
}

int xct_sqdist_f64(const float *a, const float *b, int64_t n, double *result, void *workspace,
                   size_t workspace_bytes, xct_stream stream)
{
    return reduce_common(a, b, n, result, workspace, workspace_bytes, 1, stream);
}

int xct_dot_f64_noalloc(const float *a, const float *b, int64_t n, double *result, xct_stream stream)
{
    if (!a || !b || !result || n <= 0) return XCT_EINVAL;
    const int nb = reduce_blocks(n);
    if (nb > reduce_scratch_doubles()) return XCT_ETOOBIG;  // cannot happen: the partial count is capped
    double *partials = nullptr;
    hipError_t e = reduce_scratch(&partials);
    if (e != hipSuccess) return hip_fail(e);
    e = launch_reduce(a, b, n, result, partials, nb, 0, (hipStream_t)stream);
    return e == hipSuccess ? XCT_OK : hip_fail(e);
}

}  // extern "C"

// Compute units of the current device (cached per device).
int xct::device_cus()
{
    static int cus[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (!cus[dev]) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        cus[dev] = n;
    }
    return cus[dev];
}
