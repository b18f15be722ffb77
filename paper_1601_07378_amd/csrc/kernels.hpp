// kernels.hpp -- launch interface of the three transform kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cstdint>

namespace vloc {

// APPLY_DENSITY: the application and, from the same real-space values, the
// weighted density of the launch's bands (one pass instead of two).
enum PlaneMode {
    MODE_APPLY = 0,
    MODE_G2R = 1,
    MODE_R2G = 2,
    MODE_DENSITY = 3,
    MODE_APPLY_DENSITY = 4
};

// Tables and sizes shared by the kernels of one plan (device pointers).
struct DevTables {
    const int4 *slot_info;  // per slot: {offset, count, lmin mod N3, plane position}
    const int2 *groups;     // per group: {first slot, number of sticks}
    const int2 *cols;       // per occupied x-plane: {first k mod N2, number of k}
    const void *twx, *twy, *twz; // exp(-2 pi i n2 k1 / L) at [n2][k1] (L = L1 L2, k1 < L1),
                                 // complex of the plan precision
    const double2 *twx64;        // exp(-2 pi i j / N1) in FP64 (quad x pass)
    double *partial;             // density: [nsub][N3][N2][N1] partial sums (FP64)
    const double *wts;           // density: band weights (FP64)
    // real mode, per slot: {source offset in the half-sphere arrays, kind
    // (0 = stick of the half sphere, 1 = its mirror, 2 = the (0, 0) stick),
    // -lmin of the (0, 0) stick, index in the group of the mirror stick}
    const int4 *gam;
    // whole-plane layout, per occupied x-plane hc and row y (hc-major, N2 per
    // hc): the slot of stick (hmin + hc, y), or -1
    const int *yslot;
    // plane positions that lie inside an occupied x-plane's k span but hold no
    // stick (zero in the y pass's input); rows [hole_off, hole_off + nholes)
    // of a segment
    const int *holes;
    // parted plane: per workgroup of the plane grid, nxo x N2 values [hc][yp]
    // (rows of the parts not in the row buffer)
    void *parts;
};

struct Geometry {
    int N1, N2, N3;
    int L1x, L2x, L1y, L2y, L1z, L2z;
    int nxo;        // occupied x-planes
    unsigned long long nxo_magic; // ceil(2^40 / nxo): v / nxo = (v nxo_magic) >> 40, v < 2^16
    int hmin_mod;   // hmin mod N1
    int ldy, ldx, ldz;
    int rb, rl;     // x rows per wavefront batch, padded row length in the plane kernel
    int xw;         // wavefronts taking part in the x pass
    int xq;         // > 0: quad x pass with N1 = 4 xq (no row buffer)
    int zx, zy, zz; // zero masks of the first-stage input groups per axis (0 = none)
    int fx;         // x stage-A groups whose every position is occupied
    int full;       // plane kernel holds the whole plane, x pass in place: 1 = spread
                    // over the workgroup, 2 = rows owned by wavefronts, 3 = row blocks;
                    // 4 = parted plane (0 = row buffers or lane quads)
    int parts;      // parted plane: x-pass parts of N2 / parts rows
    int parts_elems; // parted plane: LDS elements of the columns / row buffer region
    int resident_plane_wgs; // plane workgroups resident at once on the device
    int nsub;       // density: band subsets per launch
    int group_cap;  // most sticks in one group (over all segments)
    int gamma;      // real mode: a launch band is a pair of real bands
    double inv_n;   // 1 / (N1 N2 N3)
};

// Threads of a whole-plane launch: no more than the plane's widest stage has
// tasks for, in steps of four waves (one per SIMD).  24^3 (144 tasks): 256 instead
// of 512 or 1024 threads, and as many more workgroups per CU.
inline int plane_launch_threads(const Geometry &g, int threads)
{
    if (g.full != 1) return threads;
    const int tasks = std::max(g.nxo * std::max(g.L1y, g.L2y), g.N2 * std::max(g.L1x, g.L2x));
    return std::min(threads, std::max(256, (tasks + 255) / 256 * 256));
}

// Lane-quad plane kernel (application and density; q = 0: the layout's own kernel
// runs them) of the plans that share a route.  Known zeros, and tests in the place of
// loads known to be needed, change which products the compiler fuses, so q, cls and
// ysplit decide the last bits of a result: they follow from a plan's own sphere, and
// only plans that agree in them share launches.
struct LaneQuads {
    int q;    // x axis of 4 q points
    int nxo;  // most occupied x-planes of any plan
    int cus;  // compute units of the device
    int planes; // planes per workgroup of the launch
    int cls;    // class of occupied and empty x points (lq_mask)
    int ysplit; // the y split compiled with its zero mask (VLOC_LQ_YSPLITS)
    // (the size decides where a launch's segments lie among the kernel arguments: 12
    // bytes less, with the potential's buffer allocated later, took 1% off batches of
    // small k-points: seven on 40 x 36 x 32 73.5 against 72.7 us)
    int pad[3];
};

// One launch covers the bands of up to kMaxSeg k-points ("segments") that
// share the grid and the occupied-plane geometry.  Segment s owns launch bands
// [band_lo, band_lo + nb), its stick buffer at S + s_off ([band][z][slot],
// nst slots), its rows of the device tables, and blocks
// [blk_lo, blk_lo + nb * ngroups) of the stick kernels (group fastest).
constexpr int kMaxSeg = 8;
struct Seg {
    const void *in;   // stick forward input: c of the segment's first band
    void *out;        // stick backward output: out of the segment's first band
    long long s_off;  // element offset of the segment's stick buffer in S
    int nst, npw, ngroups;
    int slot_off, group_off, col_off; // first row in slot_info, groups, cols
    int band_lo, nb, blk_lo;
    int nbr;          // real mode: real bands from `in` / `out` (2 nb or 2 nb - 1)
    int hole_off, nholes; // rows of the segment in the hole table
    // the segment's occupied x-planes (a batch with a whole-plane layout plans
    // each k-point on its own occupied range): count, ceil(2^40 / count) and
    // first x-plane mod N1
    int nxo, hmin_mod;
    unsigned long long nxo_magic;
};
struct Launch {
    int nseg;  // segments in use (1 .. kMaxSeg)
    int nbt;   // bands of all segments
    int nblk;  // stick-kernel blocks of all segments
    Seg seg[kMaxSeg];
};

// Arrangement of the potential in the plane kernel's order, next to K1's work.
struct ArrangeV {
    const void *V;
    void *VT;
    int blocks;   // workgroups that arrange (the first of the launch)
    int L1x, L2x;
};
// K1: stick z-transforms (G -> r direction) from each segment's c into the
// stick buffer S.  With V, the launch also writes VT[z][k1][yp][k2] =
// V[z][y][k1 + L1x k2], yp the row's position after the y pass (the order of the
// whole-plane, parted and lane-quad kernels).
template <typename T>
hipError_t launch_stick_fwd(const Geometry &g, const LaneQuads &lq, const DevTables &t,
                            const Launch &L, void *S, const void *V, void *VT, int threads,
                            hipStream_t st);
// K2: plane kernel over the planes of every segment.  APPLY: S -> S in place.
// G2R: S -> psi rows; R2G: psi -> S; DENSITY: weighted |psi|^2 into the
// partial planes; APPLY_DENSITY: both APPLY and DENSITY.  The last three take one segment; psi and the weights are
// indexed from band band0 (the launch's first band in the caller's arrays).
template <typename T>
hipError_t launch_plane(const Geometry &g, const LaneQuads &lq, const DevTables &t, const Launch &L, int mode, void *S,
                        const void *V, void *psi, int64_t band0, int threads, int lds_bytes,
                        hipStream_t st);
// The plane-kernel launchers of the two layouts (whole plane in LDS; occupied
// x-planes with row buffers or lane quads), called by launch_plane.
template <typename T, int MODE>
hipError_t launch_plane_full_mode(const Geometry &g, const DevTables &t, const Launch &L, void *S,
                                  const void *V, void *psi, int64_t band0, int threads, int lds,
                                  hipStream_t st);
template <typename T, int MODE>
hipError_t launch_plane_rows_mode(const Geometry &g, const DevTables &t, const Launch &L, void *S,
                                  const void *V, void *psi, int64_t band0, int threads, int lds,
                                  hipStream_t st);
// Lane-quad plane kernel (FP64, x pass in registers): application, density, or
// both.
template <int MODE>
hipError_t launch_plane_lq_mode(const Geometry &g, const LaneQuads &lq, const DevTables &t,
                                const Launch &L, void *S, const void *VT, int64_t band0,
                                hipStream_t st);
// Register codelets Q of the lane-quad kernel (x axis of 4 Q points).
#define VLOC_LQ_SIZES(X)                                                                           \
    X(8) X(9) X(10) X(12) X(15) X(16) X(18) X(20) X(24) X(25) X(27) X(30) X(32)
// Compiled y splits {Q, L1y, L2y, zero mask}, for at most two stage-A tasks per thread.
#define VLOC_LQ_YSPLITS(X)                                                                         \
    X(24, 8, 12, 0x38) X(18, 8, 12, 0x38) X(32, 16, 8, 0xFE0) X(20, 8, 10, 0x38)
// Masks of a class of spheres (LaneQuads::cls), bit n for the points 4 n .. 4 n + 3:
// 2 = for a reach ext on the x axis from N1/4 - 1 to N1/4 (the grid that holds V psi
// exactly), 1 = from 0.19 to 0.32 N1, 0 = any.  `what`: 0 = points left empty, for every
// k-point with |h + k| <= ext and |k| <= 1; 1 / 2 = points occupied with x <= hmax / x >=
// N1 + hmin, for most k (classes 3 and 4 are 2 and 1 without them).
constexpr unsigned lq_mask(int Q, int cls, int what)
{
    const int N = 4 * Q;
    const bool quarter = cls == 2 || cls == 3;
    const int in = quarter ? N / 4 - 1 : (int)(0.18 * N);
    const int out = quarter ? N / 4 + 1 : (int)(0.32 * N) + 1;
    unsigned m = 0;
    for (int n = 0; n < Q && cls && (what == 0 || cls < 3); ++n) {
        const int a = 4 * n, b = 4 * n + 3;
        const bool on = what == 0 ? (a > out && b < N - out) : what == 1 ? b <= in : a >= N - in;
        if (on) m |= 1u << n;
    }
    return m;
}
// Waves per SIMD the kernel is compiled for: a lane holds four registers per
// point of its Q, and in the density alone two more for the sums; y codelets of
// 15 and 16 points need more than the 128 registers that four waves leave.
constexpr int lq_wpe(int mode, int q, int ymax)
{
    const int groups = (q + 3) / 4;
    const int regs = 16 * groups + 56 + (mode == MODE_DENSITY ? 8 * groups : 0);
    const int wpe = regs <= 128 ? 4 : regs <= 168 ? 3 : 2;
    return ymax > 12 && wpe > 3 ? 3 : wpe;
}
inline int lq_ymax(const Geometry &g)
{
    return std::max(g.L1y, g.L2y) <= 12 ? 12 : 16;
}
// Column stride in LDS: odd, so that lanes along columns fall on distinct banks.
__host__ __device__ constexpr int lq_ldy(int n2)
{
    return n2 | 1;
}
inline int lq_lds_bytes(int q, int n2, int nxo, int planes)
{
    return (planes * nxo * lq_ldy(n2) + n2 + 3 * q + 1) * 16;
}
// Shape of a lane-quad launch over `bands` bands (density: band subsets): planes
// per workgroup, threads, LDS bytes and resident workgroups.  A wavefront takes
// a block of 16 rows.  A workgroup's waves are dealt to the four SIMDs in turn
// from the first, so that one whose waves are no multiple of four leaves slots
// that the next cannot use (96 rows: six waves, one workgroup per CU at three
// waves per SIMD).  Several planes share a workgroup where that puts more
// wavefronts on a CU and shortens the launch: rounds of resident workgroups,
// times 1 + 0.75 (planes - 1) for a workgroup's time (96^3: 26.4k cycles with one
// plane, 46k with two).  Where workgroups of one plane fill the CU, they stay:
// 60 x 60 x 100, 37 bands 90 us, against 101 us with four planes each.
struct LqLaunch {
    int planes, threads, lds, resident;
};
inline LqLaunch lq_launch(const Geometry &g, const LaneQuads &lq, int mode, int64_t bands,
                          int max_planes = 4)
{
    const int wpe = lq_wpe(mode, lq.q, lq_ymax(g)), cap = 4 * wpe;
    const int blocks = (g.N2 + 15) / 16;
    LqLaunch best{};
    double least = 0.0;
    int most = 0; // wavefronts on a CU
    for (int p = 1; p <= max_planes && (p == 1 || p <= bands); ++p) {
        const int lds = lq_lds_bytes(lq.q, g.N2, lq.nxo, p);
        const int units = p * blocks, rounds = (units + cap - 1) / cap;
        const int waves = (units + rounds - 1) / rounds;
        if (p > 1 && (lds > 160 * 1024 || rounds > 1)) break;
        const int per_cu = std::max(1, std::min(160 * 1024 / lds, wpe / ((waves + 3) / 4)));
        int res = lq.cus * per_cu;
        if (res >= 8) res &= ~7;
        const int64_t items = (bands + p - 1) / p * g.N3;
        const double cost = (double)((items + res - 1) / res) * (1.0 + 0.75 * (p - 1));
        if (p > 1 && (per_cu * waves <= most || cost >= least)) continue;
        least = cost;
        most = per_cu * waves;
        best = LqLaunch{p, 64 * waves, lds, res};
    }
    return best;
}
// Is the lane-quad kernel faster than the layout's own, for a sphere of reach ext on
// the x axis?  The layout's own kernels come with codelets of at most 12 points, or
// with those of 15 and 16 too, which spill; the parted plane goes through a device
// scratch.  Without masks of occupied points (class 0) every point of a row is tested,
// and from Q = 15 on the lane quads spill as well (56 registers per lane; 120 and more
// at Q = 24 to 27), except in the density alone.  Whole calls on the layout's kernel ->
// on lane quads, FP64 (many bands; a ratio where they are faster):
//   reach 0.40 of each axis: 80^3 x 78 bands 516 -> 915 us, 96 x 72 x 96 x 60 541 -> 1093,
//     64^3 x 152 442 -> 718, 128 x 64 x 128 x 38 723 -> 978; but 48^3 0.74 of the time,
//     and with codelets of 15 or 16 points 64 x 150 x 64 0.90, 72 x 135 x 64 0.73, 128 x
//     18 x 64 0.75;
//   reach 0.12: 96 x 72 x 96 252 -> 344, 108 x 90 x 64 223 -> 328, 120 x 80 x 64 229 ->
//     309, parted 108^2 x 64 300 -> 421; but 80^3 0.91, 64^3 0.60, 96 x 32 x 64 0.70,
//     128^2 x 16 0.79, 120^2 x 64 0.90;
//   density alone, reach 0.40: 72^3 0.87 of the time on the layout's kernel, 80^3 0.84,
//     120 x 80 x 64 0.82; on lane quads 60^3 0.78, 100^3 0.79, 128 x 64 x 128 0.88.
// With masks, two waves per SIMD want workgroups that fill them: 120 x 80 x 64 x 65 bands,
// reach 0.25, five waves on a CU, 1.18 times the time.
inline bool lq_pays(const Geometry &g, const LaneQuads &lq, double ext, int mode)
{
    const int codelet = std::max(std::max(g.L1x, g.L2x), std::max(g.L1y, g.L2y));
    const bool two = lq_wpe(MODE_APPLY, lq.q, lq_ymax(g)) == 2; // 256 registers
    const bool parted = g.full == 4, dens = mode == MODE_DENSITY;
    if (lq.cls) {
        const LqLaunch l = lq_launch(g, lq, MODE_APPLY, 4);
        const int waves = l.threads / 64 * std::max(1, l.resident / std::max(1, lq.cus));
        return parted || codelet > 12 || !two || 3 * waves > 16;
    }
    if (ext < 0.25 * g.N1)
        return dens || lq.q <= 20 || codelet > 12 || g.N2 <= 32 || (parted && two);
    if (dens) return lq.q <= 16 || codelet > 12 || parted;
    return lq.q <= 12 || (codelet > 12 && (lq.q <= 18 || g.N2 <= 24));
}
// Whole-plane kernels with a compiled x split and the y split at run time; hit =
// false where none applies.
template <typename T, int MODE>
hipError_t launch_plane_xline(const Geometry &g, const DevTables &t, const Launch &L, void *S,
                              const void *VT, int64_t band0, int threads, int lds,
                              hipStream_t st, bool &hit);
// Compiled specialisations of the whole-plane application kernel for the
// splits the schedule tuner tries; hit = false where none applies.
template <typename T>
hipError_t launch_plane_full_tuned(const Geometry &g, const DevTables &t, const Launch &L,
                                   void *S, const void *VT, int threads, int lds, hipStream_t st,
                                   bool &hit);
// ... those of workload geometry G (one compiled part each)
template <typename T, int G>
hipError_t launch_plane_full_tuned_g(const Geometry &g, const DevTables &t, const Launch &L,
                                     void *S, const void *VT, int threads, int lds,
                                     hipStream_t st, bool &hit);
// Density helpers (reduce.hip): FP64 reductions and band scaling.
hipError_t launch_fill_f64(double *x, int64_t n, double v, hipStream_t st);
// y[i] = factor * s * x[i], s = scale[0] (or 1 if scale is NULL); y may equal x.
hipError_t launch_scale_real(const double *x, int64_t n, const double *scale, double factor,
                             double *y, hipStream_t st);
// partial planes in [z][y][x] order, or with full != 0 in the full-plane
// kernel's [z][x][yp] order
hipError_t launch_density_reduce(const Geometry &g, const LaneQuads &lq, const double *partial,
                                 int nsub, const double *scale, double *rho, hipStream_t st);
template <typename T>
hipError_t launch_band_dot(const void *a, const void *b, int64_t npw, int64_t nb, double *out,
                           hipStream_t st);
hipError_t launch_weighted_sum(const double *x, const double *w, int64_t n, double *out,
                               hipStream_t st);
template <typename T>
hipError_t launch_scale_bands(const void *x, int64_t npw, int64_t nb, const double *w,
                              const double *scale, double factor, void *y, hipStream_t st);

// K3: stick z-transforms (r -> G direction) with 1/N, gathering into each
// segment's out.
template <typename T>
hipError_t launch_stick_bwd(const Geometry &g, const DevTables &t, const Launch &L, const void *S,
                            int threads, hipStream_t st);

} // namespace vloc
