// kernel_common.h -- device helpers and launch helpers shared by the transform
// kernels (stick kernels, plane kernels).
#pragma once
#include <algorithm>
#include <type_traits>

#include "dft_codelets.h"
#include "kernels.hpp"

namespace vloc {

template <typename T>
struct Cx;
template <>
struct Cx<double> {
    using type = double2;
};
template <>
struct Cx<float> {
    using type = float2;
};
template <typename T>
using cx = typename Cx<T>::type;

template <typename T>
__device__ __forceinline__ cx<T> mk(T a, T b)
{
    cx<T> v;
    v.x = a;
    v.y = b;
    return v;
}

// Calls f with a compile-time codelet size equal to the runtime r.  Sizes
// above MAXR are not compiled (workgroups of more than 512 threads have too
// few registers for them, and a kernel that holds the paths of larger sizes
// carries their register pressure into every other size); the launchers never
// run such a kernel with them.
template <int MAXR = 32, typename F>
__device__ __forceinline__ void with_codelet(int r, F &&f)
{
    if constexpr (MAXR > 16) {
        switch (r) {
        case 18: f(std::integral_constant<int, 18>{}); return;
        case 20: f(std::integral_constant<int, 20>{}); return;
        case 24: f(std::integral_constant<int, 24>{}); return;
        case 25: f(std::integral_constant<int, 25>{}); return;
        case 27: f(std::integral_constant<int, 27>{}); return;
        case 30: f(std::integral_constant<int, 30>{}); return;
        case 32: f(std::integral_constant<int, 32>{}); return;
        default: break;
        }
    }
    switch (r) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 9: f(std::integral_constant<int, 9>{}); break;
    case 10:
        if constexpr (MAXR >= 10) f(std::integral_constant<int, 10>{});
        break;
    case 12:
        if constexpr (MAXR >= 12) f(std::integral_constant<int, 12>{});
        break;
    case 15:
        if constexpr (MAXR >= 15) f(std::integral_constant<int, 15>{});
        break;
    case 16:
        if constexpr (MAXR >= 16) f(std::integral_constant<int, 16>{});
        break;
    default: break;
    }
}

// Compile-time size CT if non-zero, else the runtime r through the switch.
template <int CT, int MAXR = 32, typename F>
__device__ __forceinline__ void with_size(int r, F &&f)
{
    if constexpr (CT > 0)
        f(std::integral_constant<int, CT>{});
    else
        with_codelet<MAXR>(r, f);
}

// Bit n1 of a zero mask ZM is set when every input x[n2 + L2 n1] of stage A
// is zero for every task (positions that no sphere point reaches); stage A
// then skips those loads, the codelet folds the zeros, and the reverse stage
// A' skips computing and storing those outputs, which nothing reads.
template <int ZM>
__device__ __forceinline__ constexpr bool masked(int n1)
{
    return ZM != 0 && ((ZM >> n1) & 1);
}

// x[k1] *= W_L^{S n2 k1}, L = R L2; the table holds W_L^{n2 k1} =
// exp(-2 pi i n2 k1 / L) at [n2][k1] (R entries per n2), so a task's
// twiddles are one contiguous run.
template <int R, int S, typename T>
__device__ __forceinline__ void twiddle(T *xr, T *xi, int n2, const cx<T> *__restrict__ tw)
{
    const cx<T> *w_n2 = tw + n2 * R;
#pragma unroll
    for (int k1 = 1; k1 < R; ++k1) {
        cx<T> w = w_n2[k1];
        T wr = w.x, wi = (S < 0) ? w.y : -w.y;
        T a = xr[k1], b = xi[k1];
        xr[k1] = a * wr - b * wi;
        xi[k1] = a * wi + b * wr;
    }
}

// The same with fewer table reads.  For an 8-point first stage only w^1, w^2
// and w^4 are read; w^3, w^5, w^6 and w^7 are their products (one or two
// roundings from the tabulated values): four complex multiplies instead of four
// reads; a 16-point stage (FP64) also reads w^8 and forms the rest likewise.  Used where reads are the scarcer resource: the FP64 whole-plane
// kernel (its LDS traffic is as long as its arithmetic) and, with ANY, the
// forward stick kernel in both precisions (its twiddle loads were a third of
// its vector-memory instructions).
template <int R, int S, typename T, bool ANY = false>
__device__ __forceinline__ void twiddle_pw(T *xr, T *xi, int n2, const cx<T> *__restrict__ tw)
{
    if constexpr (R == 8 && (ANY || std::is_same<T, double>::value)) {
        const cx<T> *w_n2 = tw + n2 * R;
        const cx<T> a = w_n2[1], b = w_n2[2], d = w_n2[4];
        auto mul = [](cx<T> u, cx<T> v) {
            return mk<T>(u.x * v.x - u.y * v.y, u.x * v.y + u.y * v.x);
        };
        cx<T> w[R];
        w[1] = a;
        w[2] = b;
        w[3] = mul(a, b);
        w[4] = d;
        w[5] = mul(a, d);
        w[6] = mul(b, d);
        w[7] = mul(w[3], d);
#pragma unroll
        for (int k1 = 1; k1 < R; ++k1) {
            T wr = w[k1].x, wi = (S < 0) ? w[k1].y : -w[k1].y;
            T u = xr[k1], v = xi[k1];
            xr[k1] = u * wr - v * wi;
            xi[k1] = u * wi + v * wr;
        }
        return;
    }
    if constexpr (R == 16 && (ANY || std::is_same<T, double>::value)) {
        // w^1, w^2, w^4, w^8 read; w^3 and w^5..w^7 products of them (at most
        // two roundings), w^9..w^15 = w^(k - 8) w^8 (at most three): 4 reads
        // and 11 complex multiplies instead of 15 reads, and 8 twiddles live
        const cx<T> *w_n2 = tw + n2 * R;
        const cx<T> w1 = w_n2[1], w2 = w_n2[2], w4 = w_n2[4], w8 = w_n2[8];
        auto mul = [](cx<T> u, cx<T> v) {
            return mk<T>(u.x * v.x - u.y * v.y, u.x * v.y + u.y * v.x);
        };
        auto app = [&](int k1, cx<T> w) {
            T wr = w.x, wi = (S < 0) ? w.y : -w.y;
            T u = xr[k1], v = xi[k1];
            xr[k1] = u * wr - v * wi;
            xi[k1] = u * wi + v * wr;
        };
        cx<T> lo[8];
        lo[0] = mk<T>(T(1), T(0));
        lo[1] = w1;
        lo[2] = w2;
        lo[3] = mul(w1, w2);
        lo[4] = w4;
        lo[5] = mul(w1, w4);
        lo[6] = mul(w2, w4);
        lo[7] = mul(lo[3], w4);
#pragma unroll
        for (int k = 1; k < 8; ++k) app(k, lo[k]);
        app(8, w8);
#pragma unroll
        for (int k = 1; k < 8; ++k) app(8 + k, mul(lo[k], w8));
        return;
    }
    twiddle<R, S, T>(xr, xi, n2, tw);
}

// Segment of a launch by a uniform key (stick-kernel block or launch band):
// the last segment whose first key is <= v.  The descriptor is read from the
// kernel-argument segment with a uniform index (scalar loads), not held in
// registers across the kernel.
__device__ __forceinline__ Seg seg_by_block(const Launch &L, int v)
{
    int s = 0;
    for (int i = 1; i < L.nseg; ++i)
        if (v >= L.seg[i].blk_lo) s = i;
    return L.seg[s];
}
// Block numbering of K3: consecutive workgroups go to the eight XCDs in turn,
// so renumber them to give each XCD one contiguous range of (band, group)
// items; the output cache lines shared by neighbouring groups (the ends of
// their coefficient runs) then meet in one L2 instead of being written back
// partially from two.  A bijection on [0, nblk) for any nblk.  (K1 keeps the
// hardware order, measured faster for its S writes.)
__device__ __forceinline__ int xcd_block(int nblk)
{
    const int b = blockIdx.x, x = b & 7, q = nblk >> 3, r = nblk & 7;
    return x * q + min(x, r) + (b >> 3);
}
__device__ __forceinline__ int seg_index_by_band(const Launch &L, int v)
{
    int s = 0;
    for (int i = 1; i < L.nseg; ++i)
        if (v >= L.seg[i].band_lo) s = i;
    return s;
}
__device__ __forceinline__ Seg seg_at(const Launch &L, int s)
{
    return L.seg[s];
}

// Real mode: the value at position i of a stick's run for the band pair
// (a, b), d = A + i B, where A, B are the coefficients of bands a, b at that
// g; a mirror stick (-h, -k) reads the half-sphere run of its partner in
// reverse, conjugated (c(-g) = conj c(g)); the (0, 0) stick reads l >= 0
// directly and l < 0 mirrored, with Im c(0) taken as 0.
template <typename T>
__device__ __forceinline__ cx<T> gamma_pair(const cx<T> *__restrict__ ca,
                                            const cx<T> *__restrict__ cb, int4 gm, int i)
{
    int idx;
    bool mir, zero = false;
    if (gm.y == 0) {
        idx = gm.x + i;
        mir = false;
    } else if (gm.y == 1) {
        idx = gm.x - i;
        mir = true;
    } else {
        const int l = i - gm.z;
        mir = l < 0;
        zero = l == 0;
        idx = gm.x + (mir ? -l : l);
    }
    cx<T> a = ca[idx];
    cx<T> b = cb ? cb[idx] : mk<T>(T(0), T(0));
    T ai = mir ? -a.y : a.y, bi = mir ? -b.y : b.y;
    if (zero) ai = bi = T(0);
    return mk<T>(a.x - bi, ai + b.x);
}

// Orders LDS accesses of one wavefront (LDS executes a wave's operations in
// issue order; this keeps the compiler from moving accesses across).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Persistent plane grid: the workgroups that are resident at once (a
// multiple of 8 so that the XCD schedule applies), never more than the planes.
[[maybe_unused]] static unsigned plane_blocks(const Geometry &g, int nb)
{
    long long total = (long long)nb * g.N3;
    long long res = (long long)g.resident_plane_wgs;
    if (res >= 8) res &= ~7LL;
    if (res < 1) res = 1;
    return (unsigned)(total < res ? total : res);
}

template <typename K>
static hipError_t allow_lds(K kernel, size_t bytes)
{
    if (bytes <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

} // namespace vloc
