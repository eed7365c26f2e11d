// Back-projection on the matrix cores, for calls with many slices.
//
// At one angle, the value that a pixel takes from a row is the row's samples
// times the two hat weights of the pixel's detector coordinate, so for a block
// of pixels and a set of rows (the columns: slices, and the rows that the
// slice's symmetries let the same coordinates read) the back-projection is a
// product A B, A [pixel][angle, bin] holding the weights (two adjacent
// non-zeros per angle) and B [angle, bin][column] the samples.  The vector
// kernels (bp.hip) read 8 bytes of LDS and issue some three instructions per
// update and are bound by the LDS; here a weight is formed once for all
// columns and a sample is read once per 16 pixels.
//
// Precision.  FP32 operands are split into two FP16 halves: samples scaled by
// a power of two (per slice, so that its largest magnitude lies in
// [2^14, 2^15)) as high + low with at most 2^-23 of the sample or 2^-39 of the
// slice's largest magnitude left over (kMXRange bounds the latter), weights as a
// multiple of 2^-11 and a remainder of at most 2^-12 held to 2^-24.  The
// products high high, low high and high low are accumulated in FP32 (low low is
// below 2^-23 of the sample a tap).  Coordinates
// are formed relative to an FP64 window anchor as in bp.hip, over windows half
// as wide.  Measured against the FP64 values the images are closer than the
// vector kernels' (white noise rows: 2e-6 against 5e-6 relative).
//
// Split table.  One pass writes the rows of four slices side by side, a
// 16-byte record (four high halves, four low halves) per angle and bin, so
// that a window of one slice group is one run of memory that is copied into
// LDS without registers and without instructions per sample.
//
// Workgroup: a 32 x 32 pixel tile (and its images under the symmetries) for
// COLS = 16, 32 or 64 columns, 1024 threads; a wavefront owns an 8 x 8 block as
// four 4 x 4 quarters, COLS / 16 accumulators of 16 x 16 each.  A stage is four
// angles: windows of 52 bins (31 sqrt 2 pixels of footprint and a quarter's
// reads past it) of every column, in one of three LDS buffers: while stage s is
// added up, stage s + 1 is complete and stage s + 2 in flight.  A quarter reads
// 7 bins from its own window start b at each angle, as two groups of four bins
// b .. b + 3 and b + 3 .. b + 6: the groups overlap by one bin, so a pixel's two
// taps always lie in one group and fit the matrix unit's 2:4 sparse form
// (v_smfmac_f32_16x16x32: two stored weights of every four bins, with their
// positions; 16 pixels x four angles' two groups x 16 columns).  Samples reach
// the operand layout through transposing LDS reads, which need no alignment of
// b.  Up to 32 columns two workgroups share a CU (64 registers, 80 KB of LDS);
// with 64 columns the accumulators alone take 64.
//
// What bounds it: with 64 columns the matrix cores, the vector instructions and
// the LDS together (0.52 of the matrix units' cycles, 0.39 vector instructions a
// cycle and CU, LDS 0.73 at 2.07 GHz; 16 x 2048^2 x 1800 angles: 4.94 ms, 24,450
// GUPS; the vector kernels 8.4 ms; the instruction does half the products of
// the unit's longest, 16 x 16 x 64 in the same cycles); with 32 and 16 columns
// the vector instructions that form the weights (0.84 and 0.87; 4 x 4096^2 x 1023 angles
// with 16 columns: 3.63 ms, 18,900 GUPS, the vector kernels 5.90 ms).
// Blocks of 8 x 8 pixels with four groups of four bins and 32 x 32 tiles took
// half the LDS reads but twice the cycles of the matrix unit and two more
// selects a weight: 5.44 ms, and 4.50 ms with 16 columns.  LDS passes without
// bank conflicts (half of the LDS cycles are conflicts, as only high halves are
// read together) gained 1 to 2 % for 64 columns, less than their addressing
// costs in the others.
#include <type_traits>

#include "xct_internal.h"

namespace xct {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef __fp16 g4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_char;

constexpr int kMXThreads = 1024; // 16 wavefronts, one 8 x 8 block each
constexpr int kRec = 16;         // bytes of a table record
constexpr int kMXWindow = 52;    // window bins per angle
// LDS bytes of a window: 16 dwords more than a multiple of the 64 banks, so
// the 16 lanes of one angle's transposing read (4 bins of 4 windows) meet
// distinct banks
constexpr int kRegion = kMXWindow * kRec;
static_assert(kRegion % 256 == 64, "window stride");
constexpr int kOutCols = 8;      // columns that go out through LDS together
// A quarter's reads stay inside the window: it starts at the bin below 28 sqrt(2)
// r + 2 at most (r bins per pixel) and reads 7 bins; and its pixels' coordinates
// stay below 6 bins after its start.
static_assert(28 * 1.41422 * kMXMaxRatio + 2 < kMXWindow - 6, "window covers the last quarter");
static_assert(3 * 1.41422 * kMXMaxRatio + 1.02 < 6, "quarter footprint");

template <int COLS>
constexpr int mx_buf_bytes() { return kMXAngles * (COLS / 4) * kRegion; }
template <int COLS>
constexpr int mx_lds_bytes()
{
    const int stage = 3 * mx_buf_bytes<COLS>(), out = kOutCols * kMXTile * (kMXTile + 1) * 4;
    return stage > out ? stage : out;
}

// What the split holds: the low halves end 2^-39 below the slice's largest
// magnitude, so a sample far smaller than that maximum keeps fewer bits than in
// FP32.  A slab is split only where every run of kMXRun samples of a slice
// (rows following each other) that is not all zero reaches kMXRange of the
// slice's largest magnitude; there the halves leave 2^-19 of the run's at
// most.  Pixels that see nothing but runs at the limit are 2.2e-6 off the FP64
// values (2.05e-6 far from it), the vector kernels' 5.3e-6; at 2^-22 4.9e-6, at
// 2^-24 1.8e-5.  Detector rows come nowhere near the limit: the least run of
// noise-free phantom rows of 8192 bins is 2^-14 of the largest, of rows with
// noise 2^-9.
constexpr int kMXRun = 32;
constexpr float kMXRange = 0x1p-20f;

constexpr uint32_t kBeyondRow = 0x40000000u;  // past any row: the buffer unit returns zeros there

__device__ __forceinline__ uint32_t pack_h2(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2){a, b}, h2));
}

// Scale (a power of two) that brings the slice's largest magnitude into
// [2^14, 2^15), and its inverse.
__device__ __forceinline__ void mx_scale(uint32_t amax_bits, float &s, float &inv)
{
    int e = amax_bits == 0 ? 0 : 14 - ((int)(amax_bits >> 23) - 127);
    e = e > 126 ? 126 : e;
    s = __uint_as_float((uint32_t)(127 + e) << 23);
    inv = __uint_as_float((uint32_t)(127 - e) << 23);
}

// Workgroup barrier that orders LDS accesses but leaves copies into LDS in
// flight (__syncthreads would wait for them).
__device__ __forceinline__ void mx_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// 16 bytes a lane from a buffer (zeros out of its range) straight into LDS at
// `to` + 16 lane.  Written as assembly because the compiler waits for every
// copy in flight before the next read of LDS, whichever bytes that reads;
// the waits are the kernel's own (s_waitcnt vmcnt and a barrier before a
// buffer is read).  It has no register result.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // m0 is reserved; nothing else here uses it
__device__ __forceinline__ void copy_to_lds(uint32_t to, uint32_t off, u4 rsrc)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(to), "v"(off), "s"(rsrc)
                 : "memory", "m0");
}
#pragma clang diagnostic pop

// Operations a pixel's coordinate serves (its columns per slice), by kind:
//   kMXPlain    Q
//   kMXMirror   Q, R^2 Q (detector mirror)
//   kMXQuarter  Q, R^2 Q, R^3 Q, R Q (rows a quarter turn on)
//   kMXMirror2, kMXQuarter2: the same after the reflection F (x -> -x), which
//   sees angle k's coordinate at angle pi - th_k, row N_p - k (row 0: its own
//   mirror).
constexpr int mx_ops(int kind)
{
    return kind == kMXPlain ? 1 : kind == kMXMirror ? 2 : kind == kMXQuarter2 ? 8 : 4;
}

template <int COLS, int KIND>
__global__ __launch_bounds__(kMXThreads, COLS < 64 ? 8 : 4) void bp_mfma_kernel(MXArgs a)
{
    constexpr int G = mx_ops(KIND);
    constexpr int kMXChunk = COLS == 64 ? 64 : 32;  // angles whose parameters are formed at a time
    constexpr bool kQuarter = KIND == kMXQuarter || KIND == kMXQuarter2;
    constexpr bool kReflect = KIND == kMXMirror2 || KIND == kMXQuarter2;
    constexpr int NT = COLS / 16;           // 16-column tiles
    constexpr int R = COLS / 4;             // windows per angle: window r is operation r % G of slice group r / G
    constexpr int GPI = R / G;              // groups of four slices per item
    constexpr int kBuf = mx_buf_bytes<COLS>();
    static_assert(R % G == 0, "whole slice groups per item");
    __shared__ __attribute__((aligned(16))) char buf[mx_lds_bytes<COLS>()];
    __shared__ float4 par[2 * kMXChunk];
    __shared__ int wst[2 * kMXChunk];
    if (a.amax[0] != 0) return;  // a row element is not finite: the vector kernels take the slab

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroup i runs on XCD i mod 8: each XCD takes a contiguous run of
    // items, whose windows overlap in its L2
    const int n_wg = (int)gridDim.x, xcd = (int)blockIdx.x & 7, jx = (int)blockIdx.x >> 3;
    const int qx = n_wg >> 3, rx = n_wg & 7;
    int item = xcd * qx + min(xcd, rx) + jx;
    // The angles are added up in parts of part_len, each stored or added to
    // the image on its own: one after the other in this workgroup, or
    // (partial) one workgroup per item and part, part slowest.
    int part = 0, part_end = (a.n_angles + a.part_len - 1) / a.part_len;
    if (a.partial) {
        part = item / a.items;
        item -= part * a.items;
        part_end = part + 1;
    }
    const int tiles = KIND == kMXQuarter2 ? a.tiles_x * (a.tiles_x + 1) / 2 : a.tiles_x * a.tiles_y;
    const int zg = item / tiles, t = item - zg * tiles;
    int ty, tx;
    if (KIND == kMXQuarter2) {  // the tiles on and above the quadrant's diagonal
        tx = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
        while (tx * (tx + 1) / 2 > t) --tx;
        while ((tx + 1) * (tx + 2) / 2 <= t) ++tx;
        ty = t - tx * (tx + 1) / 2;
    } else if (a.tiles_x % 4 == 0 && a.tiles_y % 4 == 0) {  // 4 x 4 groups of neighbouring tiles
        const int grp = t >> 4, in = t & 15, gy = grp / (a.tiles_x >> 2);
        ty = gy * 4 + (in >> 2);
        tx = (grp - gy * (a.tiles_x >> 2)) * 4 + (in & 3);
    } else {
        ty = t / a.tiles_x;
        tx = t - ty * a.tiles_x;
    }
    const int i0 = ty * kMXTile, j0 = tx * kMXTile;
    const int Np = a.n_angles;
    int l0 = part * a.part_len, l1 = min(Np, l0 + a.part_len);  // angles of the part
    const int g0 = zg * GPI, n_groups = (a.n_slices + 3) >> 2;
    const int64_t row_bytes = (int64_t)a.n_det * kRec, group_bytes = row_bytes * Np;

    // Per angle of the launch: the tile's first pixel's coordinate above the
    // window start, C, S, the window start of a quarter at the tile's corner
    // (with 1/64 bin of margin), and the window start itself.
    auto make_params = [&](int chunk) {
        if (lane >= kMXChunk) return;
        const int l = l0 + chunk * kMXChunk + lane, slot = (chunk & 1) * kMXChunk + lane;
        float4 p = make_float4(2.0f, 0.0f, 0.0f, 2.0f - 0.015625f);
        int B = 0;
        if (l < l1) {
            const double2 cd = a.csd[a.k_first + l + (kQuarter && l >= a.half_set ? a.k_jump : 0)];
            const double U = (j0 - 0.5 * (a.nx - 1)) * cd.x + (i0 - 0.5 * (a.ny - 1)) * cd.y + a.center;
            const double Bd = floor(U + (kMXTile - 1) * (fmin(cd.x, 0.0) + fmin(cd.y, 0.0))) - 1.0;
            p.x = (float)(U - Bd);
            p.y = (float)cd.x;
            p.z = (float)cd.y;
            p.w = p.x + 3.0f * (fminf(p.y, 0.0f) + fminf(p.z, 0.0f)) - 0.015625f;
            B = (int)Bd;
        }
        par[slot] = p;
        wst[slot] = B;
    };

    // Staging: this wavefront copies the windows su, su + 4, ... of angle sa
    // of a stage.  An angle past the last, or a slice group past the slab's,
    // copies zeros (an empty buffer).
    const int sa = wave & 3, su = wave >> 2;
    int64_t from[R / 4];
    uint32_t len[R / 4];
#pragma unroll
    for (int i = 0; i < R / 4; ++i) {
        const int g = g0 + (su + 4 * i) / G;
        from[i] = a.table + (g < n_groups ? g : 0) * group_bytes;
        len[i] = g < n_groups ? (uint32_t)row_bytes : 0u;
    }
    // row and direction that operation su (reflected or not) reads at angle l
    auto source = [&](int l, bool reflected, int &row, bool &flip) {
        row = l;
        flip = false;
        if (reflected) {
            flip = l == 0;
            row = l == 0 ? 0 : Np - l;
        }
        if (kQuarter && su >= 2) {
            const bool upper = row >= a.half_set;
            row += upper ? -a.half_set : a.half_set;
            flip = flip != upper;
        }
        if (G > 1 && (su & 1)) flip = !flip;
    };
    auto stage = [&](int s, int B, lds_char *dst) {
        const int l = l0 + kMXAngles * s + sa;
        const bool live = l < l1;
        constexpr int kRows = KIND == kMXQuarter2 ? 2 : 1;  // distinct rows among this wavefront's operations
        int64_t at[kRows];
        uint32_t off[kRows];
#pragma unroll
        for (int f = 0; f < kRows; ++f) {
            int row;
            bool flip;
            source(live ? l : 0, KIND == kMXQuarter2 ? f == 1 : kReflect && su >= 2, row, flip);
            at[f] = (int64_t)row * row_bytes;
            off[f] = min((uint32_t)((flip ? a.mirror - B - lane : B + lane) * kRec), kBeyondRow);
        }
        const uint32_t to = (uint32_t)(uintptr_t)(dst + (sa * R + su) * kRegion);
        if (lane < kMXWindow) {
#pragma unroll
            for (int i = 0; i < R / 4; ++i) {
                const int64_t base = from[i] + at[i % kRows];
                const u4 rsrc = {(uint32_t)base, (uint32_t)(base >> 32), live ? len[i] : 0u, 0x00020000u};
                copy_to_lds(to + 4 * i * kRegion, off[i % kRows], rsrc);
            }
        }
    };

    const int c = lane & 15, quad = lane >> 4;
    const float px = (float)(c & 3), py = (float)(c >> 2);  // pixel of a 4 x 4 quarter of the block
    // a transposing read: lane c of 16 supplies bin c / 4 of window c % 4 of
    // this lane's angle of the four
    const int lane_off = (c >> 2) * kRec + (quad * R + (c & 3)) * kRegion;
    const float bx = (float)((wave & 3) * 8), by = (float)((wave >> 2) * 8);  // block's corner in the tile

    // Weights of 16 pixels (4 x 4) at the coordinate t in [0, 6) above the
    // quarter's window start: group floor(t / 3) of the two holds 1 - f and f at
    // its bins r = floor(t) mod 3 and r + 1.
    struct Weights {
        h4 hi, lo;
        int ix;
    };
    auto weights = [&](float t) {
        Weights w;
        const float f = __builtin_amdgcn_fractf(t);
        const float hi = (f + 6144.0f) - 6144.0f;  // to a multiple of 2^-11
        const float lo = f - hi;
        const uint32_t ph = pack_h2(1.0f - hi, hi);
        uint32_t pl;  // (-lo, lo)
        asm("v_cvt_pk_f16_f32 %0, -%1, %1" : "=v"(pl) : "v"(lo));
        const bool c3 = t < 3.0f;
        w.hi = __builtin_bit_cast(h4, (u2){c3 ? ph : 0u, c3 ? 0u : ph});
        w.lo = __builtin_bit_cast(h4, (u2){c3 ? pl : 0u, c3 ? 0u : pl});
        // positions r and r + 1 in both groups: byte floor(t) of 44 99 ee 44 99 ee
        w.ix = (int)__builtin_amdgcn_perm(0xee99u, 0x44ee9944u, (uint32_t)t);
        return w;
    };
    typedef const lds_char *ldsp;
    auto rd = [&](ldsp p, int off) {
        return __builtin_bit_cast(u2, __builtin_amdgcn_ds_read_tr16_b64_v4f16(
                                          (__attribute__((address_space(3))) g4 *)(p + off)));
    };

    f4v acc[4][NT];  // the block's 4 x 4 quarters
    for (;;) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n) acc[m][n] = (f4v){0.0f, 0.0f, 0.0f, 0.0f};

        if (wave < 2) make_params(wave);
        __syncthreads();
        stage(0, __builtin_amdgcn_readfirstlane(wst[sa]), (lds_char *)buf);
        stage(1, __builtin_amdgcn_readfirstlane(wst[kMXAngles + sa]), (lds_char *)buf + kBuf);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        mx_barrier();

        const int nst = (l1 - l0 + kMXAngles - 1) / kMXAngles;
        int cur = 0, nxt = kBuf, far = 2 * kBuf;  // buffers of stages s, s + 1 and s + 2
        for (int s = 0; s < nst;) {
            // at each chunk: the parameters of the one after it (in the slots of
            // the one before it)
            constexpr int kRun = kMXChunk / kMXAngles;
            if (s > 0 && wave == (s / kRun & 15)) make_params(s / kRun + 1);
            const int s_end = min(nst, s + kRun);
            for (; s < s_end; ++s) {
                const int slot0 = (kMXAngles * s) & (2 * kMXChunk - 1);
                const int slot2 = (kMXAngles * (s + 2)) & (2 * kMXChunk - 1);
                stage(s + 2, __builtin_amdgcn_readfirstlane(wst[slot2 + sa]), (lds_char *)buf + far);
                const float4 p = par[slot0 + quad];
                const float u = fmaf(bx + px, p.y, fmaf(by + py, p.z, p.x));
                const float v = fmaf(bx, p.y, fmaf(by, p.z, p.w));
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const float ux = m & 1 ? fmaf(4.0f, p.y, u) : u, vx = m & 1 ? fmaf(4.0f, p.y, v) : v;
                    const float fl = floorf(m & 2 ? fmaf(4.0f, p.z, vx) : vx);
                    const Weights w = weights((m & 2 ? fmaf(4.0f, p.z, ux) : ux) - fl);
                    const ldsp at = (ldsp)buf + cur + (int)fl * kRec + lane_off;
                    // (the 64-column kernel's registers hold all tiles' samples at once)
                    constexpr int kGroup = COLS == 64 ? NT : 1;
#pragma unroll
                    for (int n0 = 0; n0 < NT; n0 += kGroup) {
                        h8 hi[kGroup], lo[kGroup];
#pragma unroll
                        for (int n = 0; n < kGroup; ++n) {
                            const int q = (n0 + n) * 4 * kRegion;
                            const u2 x0 = rd(at, q), x1 = rd(at, q + 3 * kRec), y0 = rd(at, q + 8), y1 = rd(at, q + 8 + 3 * kRec);
                            hi[n] = __builtin_bit_cast(h8, (u4){x0[0], x0[1], x1[0], x1[1]});
                            lo[n] = __builtin_bit_cast(h8, (u4){y0[0], y0[1], y1[0], y1[1]});
                        }
#pragma unroll
                        for (int n = 0; n < kGroup; ++n)
                            acc[m][n0 + n] = __builtin_amdgcn_smfmac_f32_16x16x32_f16(w.hi, hi[n], acc[m][n0 + n], w.ix, 0, 0);
#pragma unroll
                        for (int n = 0; n < kGroup; ++n)
                            acc[m][n0 + n] = __builtin_amdgcn_smfmac_f32_16x16x32_f16(w.lo, hi[n], acc[m][n0 + n], w.ix, 0, 0);
#pragma unroll
                        for (int n = 0; n < kGroup; ++n)
                            acc[m][n0 + n] = __builtin_amdgcn_smfmac_f32_16x16x32_f16(w.hi, lo[n], acc[m][n0 + n], w.ix, 0, 0);
                    }
                }
                const int old = cur;
                cur = nxt;
                nxt = far;
                far = old;
                // stage s + 1 has arrived (its copies were issued a stage ago);
                // s + 2's, the newest R / 4, may be in flight
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(R / 4) : "memory");
                mx_barrier();
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the copies past the last stage have landed

        // Output through LDS, kOutCols columns at a time ([column][row][33]), so
        // that the stores run along the image rows that a column's operation gives.
        float *out = reinterpret_cast<float *>(buf);
        const bool add = a.partial ? false : a.accumulate || part > 0;
        constexpr int kPitch = kMXTile + 1;
        const int NX = a.nx, NY = a.ny;
        const int lim_i = KIND == kMXPlain ? NY : (NY + 1) >> 1;
        const int lim_j = KIND == kMXPlain || KIND == kMXMirror ? NX : (NX + 1) >> 1;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
#pragma unroll 1
            for (int c0 = 0; c0 < 16; c0 += kOutCols) {
                if (g0 + (4 * n + c0 / 4) / G >= n_groups) break;
                __syncthreads();
                if (c >= c0 && c < c0 + kOutCols) {
                    float *o = out + ((c - c0) * kMXTile + (int)by + quad) * kPitch + (int)bx;
#pragma unroll
                    for (int m = 0; m < 4; ++m)
#pragma unroll
                        for (int r = 0; r < 4; ++r) o[4 * (m >> 1) * kPitch + 4 * (m & 1) + r] = acc[m][n][r];
                }
                __syncthreads();
#pragma unroll 1
                for (int cc = 0; cc < kOutCols; ++cc) {
                    const int r = 4 * n + (c0 + cc) / 4, op = r % G;
                    const int z = 4 * (g0 + r / G) + (cc & 3);
                    const bool reflected = KIND == kMXQuarter2 ? op >= 4 : kReflect && op >= 2;
                    const int turn = kQuarter ? op & 3 : op & 1;  // 0: Q, 1: R^2, 2: R^3, 3: R
                    if (z >= a.n_slices) continue;
                    // a tile on the diagonal is its own reflection
                    if (KIND == kMXQuarter2 && reflected && ty == tx) continue;
                    float sc, inv;
                    mx_scale(a.amax[1 + z], sc, inv);
                    float *img = (a.partial ? a.partial + (int64_t)part * a.n_slices * NX * NY : a.image) + (int64_t)z * NX * NY;
                    const int e = tid;
                    const int di = turn >= 2 ? e & 31 : e >> 5, dj = turn >= 2 ? e >> 5 : e & 31;
                    const int i = i0 + di, j = j0 + dj;
                    bool store = i < lim_i && j < lim_j;
                    // pixels of a middle row or column that another operation stores
                    const bool mid_i = 2 * i + 1 >= NY, mid_j = 2 * j + 1 >= NX;
                    if (KIND == kMXMirror) store = store && !(turn == 1 && mid_i);
                    if (KIND == kMXMirror2)
                        store = store && !(turn == 1 && mid_i) && !(turn == 1 && !reflected && mid_j) && !(turn == 0 && reflected && mid_j);
                    if (!store) continue;
                    const int fj = reflected ? NX - 1 - j : j;
                    const int ri = turn == 0 ? i : turn == 1 ? NY - 1 - i : turn == 2 ? fj : NX - 1 - fj;
                    const int rj = turn == 0 ? fj : turn == 1 ? NX - 1 - fj : turn == 2 ? NX - 1 - i : i;
                    float *at = img + (int64_t)ri * NX + rj;
                    float v = a.scale * (out[(cc * kMXTile + di) * kPitch + dj] * inv);
                    if (add) v += *at;
                    *at = v;
                }
            }
        }

        if (++part == part_end) break;
        l0 += a.part_len;
        l1 = min(Np, l0 + a.part_len);
        __syncthreads();  // the output's readers are done with the buffers
    }
}

// Largest magnitude over groups of LANES lanes (a power of two up to 32), in
// every lane of the group.
template <int LANES>
__device__ __forceinline__ uint32_t group_max(uint32_t m)
{
    auto dpp = [&](auto ctrl) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, decltype(ctrl)::value, 0xf, 0xf, true); };
    if constexpr (LANES >= 2) m = max(m, dpp(std::integral_constant<int, 0xB1>()));    // lanes 1 0 3 2
    if constexpr (LANES >= 4) m = max(m, dpp(std::integral_constant<int, 0x4E>()));    // lanes 2 3 0 1
    if constexpr (LANES >= 8) m = max(m, dpp(std::integral_constant<int, 0x141>()));   // mirrored in 8 lanes
    if constexpr (LANES >= 16) m = max(m, dpp(std::integral_constant<int, 0x140>()));  // mirrored in 16 lanes
    if constexpr (LANES >= 32) m = max(m, (uint32_t)__shfl_xor((int)m, 16, 64));
    return m;
}

// Magnitudes of every slice: the largest (as float bits) in amax[1 + z], minus
// the least magnitude that a run of kMXRun samples reaches, of those that are
// not all zero, in amax[1 + n_slices + z] (0: none), and amax[0] != 0 when some
// element is not finite.  Bound by memory (64 x 1800 x 2900 FP32: 225 us, 5.9
// TB/s), and where the rows are still in cache by the workgroups' atomics on one
// line: 16 bytes a load where every slice is so aligned (VEC), eight in flight,
// and few, large workgroups (4 x 2048 x 2898: 16 us with 256 workgroups of 1024
// threads, 33 with 1024 of 256; 24 x 720 x 727: 11 us, 4.7 TB/s).
constexpr int kMagThreads = 1024;
template <typename T, bool VEC>
__global__ __launch_bounds__(kMagThreads) void absmax_kernel(const T *sino, int64_t per_slice, uint32_t *amax, int z0, int n_slices)
{
    const int z = z0 + blockIdx.y;
    const T *p = sino + z * per_slice;
    const int64_t stride = (int64_t)gridDim.x * kMagThreads;
    constexpr int kPer = VEC ? 16 / (int)sizeof(T) : 1;  // samples of a lane's load
    uint32_t m = 0, least = 0;
    // magnitudes: of an FP16 element its bits, of the others float bits
    auto bits = [](T v) -> uint32_t {
        if constexpr (sizeof(T) == 4) return __float_as_uint(v) & 0x7fffffffu;
        else if constexpr (__is_same(T, f16_t)) return __builtin_bit_cast(uint16_t, v) & 0x7fffu;
        else return ((uint32_t)v.bits << 16) & 0x7fffffffu;
    };
    auto bits4 = [](u4 v) -> uint32_t {
        uint32_t r = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (sizeof(T) == 4) r = max(r, v[j] & 0x7fffffffu);
            else if constexpr (__is_same(T, f16_t)) r = max(r, max(v[j] & 0x7fffu, v[j] >> 16 & 0x7fffu));
            else r = max(r, max(v[j] << 16 & 0x7fffffffu, v[j] & 0x7fff0000u));
        }
        return r;
    };
    auto load = [&](int64_t i) {
        if constexpr (VEC) return reinterpret_cast<const u4 *>(p)[i];
        else return p[i];
    };
    auto take = [&](auto v) {
        uint32_t r;
        if constexpr (VEC) r = bits4(v);
        else r = bits(v);
        r = group_max<kMXRun / kPer>(r);
        m = max(m, r);
        least = max(least, 0u - r);
    };
    const int64_t n = per_slice / kPer;
    int64_t i = (int64_t)blockIdx.x * kMagThreads + threadIdx.x;
    const int lane = threadIdx.x & 63;
    // (whole wavefronts at a time: the runs' maxima are taken across lanes)
    for (; i - lane < n; i += 8 * stride) {
        decltype(load(0)) v[8];
        if (i - lane + 63 + 7 * stride < n) {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = load(i + j * stride);
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const decltype(load(0)) zero{};
                v[j] = zero;
                if (i + j * stride < n) v[j] = load(i + j * stride);
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) take(v[j]);
    }
    if constexpr (__is_same(T, f16_t)) {
        m = __float_as_uint((float)__builtin_bit_cast(f16_t, (uint16_t)m));
        least = 0u - __float_as_uint((float)__builtin_bit_cast(f16_t, (uint16_t)(0u - least)));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
        least = max(least, (uint32_t)__shfl_xor((int)least, off, 64));
    }
    __shared__ uint32_t part[2][kMagThreads / 64];
    if (lane == 0) {
        part[0][threadIdx.x >> 6] = m;
        part[1][threadIdx.x >> 6] = least;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        uint32_t v = 0;
#pragma unroll
        for (int w = 0; w < kMagThreads / 64; ++w) v = max(v, part[threadIdx.x][w]);
        if (v) atomicMax(amax + 1 + z + threadIdx.x * n_slices, v);
        if (threadIdx.x == 0 && v >= 0x7f800000u) atomicOr(amax, 1u);
    }
}

hipError_t launch_absmax(const void *sino, int dtype, int n_slices, int64_t per_slice, uint32_t *amax, hipStream_t s)
{
    hipError_t e = launch_fill_u32(amax, 1 + 2 * n_slices, 0u, s);
    if (e != hipSuccess) return e;
    // 8 loads a thread; one workgroup per CU, or two (2 per slice at least) where
    // whole numbers per slice come close to that
    const int64_t size = dtype == XCT_F32 ? 4 : 2;
    const bool vec = (reinterpret_cast<uintptr_t>(sino) & 15) == 0 && (per_slice * size & 15) == 0;
    const int64_t loads = vec ? per_slice * size / 16 : per_slice, want = (loads + kMagThreads * 8 - 1) / (kMagThreads * 8);
    const int64_t cap = n_slices < 16 ? (256 + n_slices - 1) / n_slices : n_slices < 256 ? 512 / n_slices : 2;
    for (int z = 0; z < n_slices; z += 65535) {
        const dim3 grid((unsigned)(want < cap ? want : cap), (unsigned)(n_slices - z < 65535 ? n_slices - z : 65535));
        auto go = [&](auto *p, auto kernel, auto kernel_vec) {
            if (vec) hipLaunchKernelGGL(kernel_vec, grid, dim3(kMagThreads), 0, s, p, per_slice, amax, z, n_slices);
            else hipLaunchKernelGGL(kernel, grid, dim3(kMagThreads), 0, s, p, per_slice, amax, z, n_slices);
        };
        if (dtype == XCT_F32) go((const float *)sino, absmax_kernel<float, false>, absmax_kernel<float, true>);
        else if (dtype == XCT_F16) go((const f16_t *)sino, absmax_kernel<f16_t, false>, absmax_kernel<f16_t, true>);
        else go((const bf16_t *)sino, absmax_kernel<bf16_t, false>, absmax_kernel<bf16_t, true>);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// The split table of the rows k_first .. of every slice: [group][row][bin] of
// 16-byte records (four slices' high halves, then their low halves) of the
// scaled samples.  Row l of the table is row k_first + l of the slab, plus
// k_jump from row `split` on.  One thread per record, rows read and written
// along bins: bound by memory (16 x 3072 x 4096: 0.37 ms, 4.4 TB/s).  A slice
// whose range is wider than the halves hold sends the slab to the vector
// kernels: the launches behind this one see amax[0].
template <typename T>
__global__ __launch_bounds__(256) void split_kernel(SplitArgs a)
{
    if (a.amax[0] != 0) return;
    const int n = blockIdx.x * 256 + threadIdx.x, g = blockIdx.z;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 4 && 4 * g + (int)threadIdx.x < a.n_slices) {
        const uint32_t *w = a.amax + 1 + 4 * g + threadIdx.x;
        const uint32_t least = 0u - w[a.n_slices];
        if (least != 0 && __uint_as_float(least) < __uint_as_float(w[0]) * kMXRange) atomicOr(a.amax, 1u);
    }
    if (n >= a.n_det) return;
    for (int l = blockIdx.y; l < a.rows; l += gridDim.y) {
        const int64_t row = a.k_first + l + (l >= a.split ? a.k_jump : 0);
        float x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int z = 4 * g + j;
            x[j] = 0.0f;
            if (z < a.n_slices) {
                float s, inv;
                mx_scale(a.amax[1 + z], s, inv);
                const T v = static_cast<const T *>(a.sino)[((int64_t)z * a.n_angles + row) * a.n_det + n];
                if constexpr (sizeof(T) == 4) x[j] = v * s;
                else if constexpr (__is_same(T, f16_t)) x[j] = (float)v * s;
                else x[j] = __uint_as_float((uint32_t)v.bits << 16) * s;
            }
        }
        uint4 o;
        o.x = pack_h2(x[0], x[1]);
        o.y = pack_h2(x[2], x[3]);
        const h2 p = __builtin_bit_cast(h2, o.x), q = __builtin_bit_cast(h2, o.y);
        o.z = pack_h2(x[0] - (float)p[0], x[1] - (float)p[1]);
        o.w = pack_h2(x[2] - (float)q[0], x[3] - (float)q[1]);
        a.table[((int64_t)g * a.rows + l) * a.n_det + n] = o;
    }
}

hipError_t launch_split(const SplitArgs &a, int dtype, hipStream_t s)
{
    (void)hipGetLastError();
    SplitArgs c = a;
    const int groups = (a.n_slices + 3) / 4;
    // grids stay below 2^32 work-items; (slice groups over 65535 are not routed here)
    const unsigned bx = (unsigned)((a.n_det + 255) / 256);
    int64_t by = (((int64_t)1 << 31) / 256) / ((int64_t)bx * groups);
    by = by < 1 ? 1 : by > a.rows ? a.rows : by;
    by = by > 65535 ? 65535 : by;
    const dim3 grid(bx, (unsigned)by, (unsigned)groups);
    if (dtype == XCT_F32) hipLaunchKernelGGL(split_kernel<float>, grid, dim3(256), 0, s, c);
    else if (dtype == XCT_F16) hipLaunchKernelGGL(split_kernel<f16_t>, grid, dim3(256), 0, s, c);
    else hipLaunchKernelGGL(split_kernel<bf16_t>, grid, dim3(256), 0, s, c);
    return hipGetLastError();
}

template <int COLS>
static hipError_t launch_mx(const MXArgs &a, int kind, int grid, hipStream_t s)
{
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kMXThreads), 0, s, a);
        return hipGetLastError();
    };
    switch (kind) {
    case kMXPlain: return go(bp_mfma_kernel<COLS, kMXPlain>);
    case kMXMirror: return go(bp_mfma_kernel<COLS, kMXMirror>);
    case kMXMirror2: return go(bp_mfma_kernel<COLS, kMXMirror2>);
    case kMXQuarter: return go(bp_mfma_kernel<COLS, kMXQuarter>);
    default: return go(bp_mfma_kernel<COLS == 16 ? 32 : COLS, kMXQuarter2>);  // (32 columns at least)
    }
}

hipError_t launch_bp_mfma(const MXArgs &a, int cols, int kind, int grid, hipStream_t s)
{
    (void)hipGetLastError();
    return cols == 64 ? launch_mx<64>(a, kind, grid, s) : cols == 32 ? launch_mx<32>(a, kind, grid, s)
                                                                     : launch_mx<16>(a, kind, grid, s);
}

}  // namespace xct
