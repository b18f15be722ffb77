// plane_quads.hip -- the plane kernel K2 with the whole x pass in registers.
//
// Four lanes of one wavefront hold an x row of N1 = 4 Q points.  Lane q of the
// quad takes the points x = q + 4 n (n < Q) from the occupied columns in LDS,
// runs a Q-point register DFT over n, exchanges with the other three lanes, and
// then owns, for every k1 = 4 j + q, all four values that the last radix-4 step
// of frequency k1 + Q k2 needs:
//
//   X[k1 + Q k2] = sum_q W_4^{q k2} W_N1^{q k1} Y_q[k1],  Y_q = DFT_Q(x[q + 4 n]).
//
// Twiddle, radix 4, the potential, the inverse radix 4 and the conjugate
// twiddle are done group by group in registers; a second exchange and the
// inverse Q-point DFT give back the occupied points, which overwrite the
// columns.  The four lanes of a quad are 16 lanes apart (q = lane / 16), so the
// exchange is a 4 x 4 transposition of registers against lane bits 4 and 5:
// v_permlane32_swap and v_permlane16_swap, one instruction per 32-bit register
// and exchange, no LDS.
//
// What bounds it.  The whole-plane kernel (rows in LDS) moves every point of the
// plane through LDS four times in its x pass, and an FP64 plane is bound by LDS
// writes and vector issue with little overlap.  Here the occupied columns are
// the only x traffic (half the LDS bytes of a plane), only they live in LDS (two
// 96 x 96 planes fit one CU, and a 128 x 128 plane fits without parts), and what
// is left is vector issue (10.5k wave instructions per 96 x 96 plane, a lane swap
// taking two slots: 62% of a CU's busy cycles) and waits: at four registers per point
// two or three waves fit a SIMD beyond Q = 16, four up to there.  The y split is
// compiled for four planes only (VLOC_LQ_YSPLITS); elsewhere the y sizes are runtime
// values, and the x pass, two thirds of the arithmetic, is compiled for every Q.
// Whole applications, quarter sphere, rows in LDS -> lane quads (with the other steps
// of a call as they are now): 36^3 x 2572 bands 2204 -> 948 us, 48^3 x 1085 1496 -> 759,
// 60^3 x 555 1289 -> 684, 64^3 x 457 1114 -> 689, 72^3 x 321 1112 -> 949, 80^3 x 1001
// 3013 -> 2896, 96^3 x 256 1188 -> 1177, 100^3 x 120 1222 -> 1047, 120^3 x 69 1234 -> 932,
// 128^3 x 96 (parted plane before) 1894 -> 1240; density 1.05 - 3.7 times, energy and
// gradients 1.04 - 2.9 times.
// FP32 planes are bound by vector issue at two workgroups per CU already and
// gained nothing (96^3 x 256 bands 696 -> 699 us), so FP32 keeps rows in LDS.
// Measured and left out: y stage B inside the row blocks' wavefronts (two
// barriers per plane instead of four, fewer lanes in use: 128^3 x 96 1242 -> 1286
// us); sticks scattered into and gathered from the columns in slot order
// (coalesced, but two more LDS passes: 1242 -> 1301 us); two workgroups of four
// or eight waves instead of one of twelve (96^3: 931 -> 1103 us in the plane
// kernel; at 128 registers spills, 1515 us).
#include "kernel_common.h"

namespace vloc {

// Registers a and b of a lane: exchanges a of the lanes with bit BIT set with b
// of the lanes with it clear.
template <int BIT>
__device__ __forceinline__ void lane_swap(unsigned &a, unsigned &b)
{
    if constexpr (BIT == 5) {
        const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    }
}
template <int BIT>
__device__ __forceinline__ void lane_swap(double &a, double &b)
{
    unsigned al = (unsigned)__double2loint(a), ah = (unsigned)__double2hiint(a);
    unsigned bl = (unsigned)__double2loint(b), bh = (unsigned)__double2hiint(b);
    lane_swap<BIT>(al, bl);
    lane_swap<BIT>(ah, bh);
    a = __hiloint2double((int)ah, (int)al);
    b = __hiloint2double((int)bh, (int)bl);
}
// r[i] of quad lane q becomes r[q] of quad lane i.
__device__ __forceinline__ void quad_transpose(double *r)
{
    lane_swap<5>(r[0], r[2]);
    lane_swap<5>(r[1], r[3]);
    lane_swap<4>(r[0], r[1]);
    lane_swap<4>(r[2], r[3]);
}

// One workgroup runs P planes (bands) of one z at a time: a wavefront takes a
// block of 16 rows of one of them in the x pass, and P is chosen on the host to
// fill the SIMDs with whole wavefronts.
//
// ZM, LO, HI: bit n set where the points q + 4 n of every quad lane are
// unoccupied, occupied with x <= hmax, or occupied with x >= N1 + hmin; the
// others are tested per lane.  CY1, CY2, ZY: the y split and its zero mask
// (0: runtime sizes, codelets of at most MR points).  YT: y stage-A tasks per
// thread whose stick values are prefetched into registers during the reverse y
// pass (compiled y split only; 0: loaded by the stage itself).
template <int MODE, int Q, unsigned ZM, unsigned LO, unsigned HI, int CY1, int CY2, int ZY, int YT,
          int MR, int MAXT, int WPE>
__global__ __attribute__((amdgpu_flat_work_group_size(64, MAXT), amdgpu_waves_per_eu(WPE)))
void k_plane_lq(Geometry g, LaneQuads lq, DevTables t, Launch L, double2 *__restrict__ S,
                const double *__restrict__ VT, long long band0)
{
    using T = double;
    constexpr int N1 = 4 * Q, G = (Q + 3) / 4, QP = 4 * G;
    constexpr bool DENS = (MODE == MODE_DENSITY || MODE == MODE_APPLY_DENSITY);
    constexpr bool POT = (MODE == MODE_APPLY || MODE == MODE_APPLY_DENSITY);
    extern __shared__ unsigned char smem_raw[];
    cx<T> *plane = reinterpret_cast<cx<T> *>(smem_raw);
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int lane = tid & 63, nwaves = nthr >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L1y = CY1 ? CY1 : g.L1y, L2y = CY2 ? CY2 : g.L2y;
    const int N2 = CY1 ? CY1 * CY2 : g.N2;
    const int ldy = lq_ldy(N2);
    const int P = lq.planes, psz = lq.nxo * ldy;  // LDS elements of one plane
    const int nrb = (N2 + 15) >> 4;               // blocks of 16 rows
    const int q = lane >> 4;
    // LDS: the planes' occupied columns, y twiddles, x twiddles W_N1^{s k1} at
    // [k1][s - 1] (s = 1..3), one zero
    cx<T> *twy = plane + P * psz;
    cx<T> *twx = twy + N2;
    const int izero = P * psz + N2 + 3 * Q;
    for (int i = tid; i < N2; i += nthr) twy[i] = reinterpret_cast<const cx<T> *>(t.twy)[i];
    for (int i = tid; i < 3 * Q; i += nthr) twx[i] = t.twx64[(i / 3) * (i % 3 + 1)];
    if (tid == 0) plane[izero] = mk<T>(T(0), T(0));

    // Persistent XCD-aware schedule as in the other plane kernels.  Work items:
    // (z, P bands of one segment) for the application; for the density (z, P
    // band subsets), step k taking the k-th band of each subset.
    const int nb = L.nbt;
    const int nsub = DENS ? g.nsub : 1;
    const int bps = DENS ? (nb + nsub - 1) / nsub : 1; // bands of a subset
    int per_z = 0;
    if constexpr (DENS)
        per_z = (nsub + P - 1) / P;
    else
        for (int s = 0; s < L.nseg; ++s) per_z += (L.seg[s].nb + P - 1) / P;
    const int total = per_z * g.N3;
    int j0 = blockIdx.x, jstep = gridDim.x, jend = total;
    if ((gridDim.x & 7) == 0 && (total & 7) == 0) {
        const int share = total >> 3, xcd = blockIdx.x & 7;
        j0 = xcd * share + (blockIdx.x >> 3);
        jstep = gridDim.x >> 3;
        jend = (xcd + 1) * share;
    }
    // step k of item j: z, segment, launch band of plane 0, planes in use
    // (plane p holds band b + p bps)
    auto item_of = [&](int j, int k, int &z, int &si, int &b, int &np) {
        z = j / per_z;
        int r = j - z * per_z;
        si = 0;
        if constexpr (DENS) {
            b = r * P * bps + k;
            np = 0;
            for (int p = 0; p < P; ++p)
                if (r * P + p < nsub && b + p * bps < nb) np = p + 1;
        } else {
            for (int s = 0; s < L.nseg; ++s) {
                const int n = (L.seg[s].nb + P - 1) / P;
                if (r < n) {
                    si = s;
                    break;
                }
                r -= n;
            }
            b = L.seg[si].band_lo + r * P;
            np = min(P, L.seg[si].nb - r * P);
        }
    };
    // next non-empty step of this workgroup's sequence; false at the end
    auto advance = [&](int &j, int &k) -> bool {
        for (;;) {
            if (DENS && k + 1 < bps)
                ++k;
            else {
                j += jstep;
                k = 0;
            }
            if (j >= jend) return false;
            if constexpr (!DENS) return true;
            int z, si, b, np;
            item_of(j, k, z, si, b, np);
            if (np > 0) return true;
            k = bps;
        }
    };

    // the current segment's occupied columns
    int nxo = 0, hx = 0, cur_seg = -1, col_off = 0, pstride = 0;
    unsigned long long nxo_magic = 0;
    auto div_nxo = [&](int v) {
        return (int)(((unsigned long long)(unsigned)v * nxo_magic) >> 40);
    };
    // y task `task` of a stage of `per` tasks per column: plane, index, column
    auto y_task = [&](int task, int per, int &p, int &idx, int &hc) {
        const int v = div_nxo(task);
        hc = task - v * nxo;
        p = 0;
        idx = v;
        for (int i = 1; i < P; ++i)
            if (idx >= per) {
                idx -= per;
                ++p;
            }
    };
    // y stage-A tasks tid + u nthr: LDS position, n2, start of their plane's slice
    // of S counted from plane 0's, and the slots of their points in it
    constexpr bool PRE = YT > 0 && CY1 > 0;
    constexpr int NU = PRE ? YT : 1, RY = PRE ? CY1 : 1;
    // (two 16-bit slots to a register, 0xFFFF where no stick)
    int yn2[NU], ycol[NU], yoff[NU];
    unsigned slots[(NU * RY + 1) / 2];
    cx<T> pre[NU * RY];
    int nT = 0, nV = 0; // this lane's points n >= nT lie at x >= N1 + hmin, n < nV at x <= hmax
    auto load_seg = [&](int si) {
        nxo = L.seg[si].nxo;
        hx = L.seg[si].hmin_mod;
        nxo_magic = L.seg[si].nxo_magic;
        col_off = L.seg[si].col_off;
        pstride = bps * g.N3 * L.seg[si].nst;
        cur_seg = si;
        nT = (hx - q + 3) >> 2;
        nV = (hx + nxo - N1 - q + 3) >> 2;
        if constexpr (PRE) {
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int task = tid + u * nthr;
                int p, hc;
                y_task(task, L2y, p, yn2[u], hc);
                const bool mine = task < P * nxo * L2y;
                ycol[u] = mine ? p * psz + hc * ldy + yn2[u] : -1;
                yoff[u] = p * pstride;
                const int *ys = t.yslot + (long long)(col_off + hc) * N2 + yn2[u];
#pragma unroll
                for (int n1 = 0; n1 < RY; ++n1) {
                    const int i = u * RY + n1;
                    const unsigned sl =
                        (mine && !masked<ZY>(n1)) ? (unsigned)ys[L2y * n1] & 0xFFFFu : 0xFFFFu;
                    slots[i / 2] = (i & 1) ? slots[i / 2] | (sl << 16) : sl;
                }
            }
        }
    };
    auto slot_at = [&](int i) { return (int)((slots[i / 2] >> (16 * (i & 1))) & 0xFFFFu); };
    auto slice = [&](int z, int si, int b) {
        const Seg &sg = L.seg[si];
        return S + sg.s_off + ((long long)(b - sg.band_lo) * g.N3 + z) * sg.nst;
    };
    // positions of planes not in use (p >= np) are left out
    auto prefetch = [&](int z, int si, int b, int np) {
        if constexpr (PRE) {
            const cx<T> *Sj = slice(z, si, b);
#pragma unroll
            for (int i = 0; i < NU * RY; ++i) {
                const int u = i / RY;
                if (masked<ZY>(i % RY)) continue;
                pre[i] = mk<T>(T(0), T(0));
                if (slot_at(i) != 0xFFFF && ycol[u] < np * psz) pre[i] = Sj[yoff[u] + slot_at(i)];
            }
        }
    };
    // (so that no register carries the old values across the x pass)
    auto prefetch_none = [&]() {
#pragma unroll
        for (int i = 0; i < NU * RY; ++i) pre[i] = mk<T>(T(0), T(0));
    };
    // The density alone sums w_b |psi_b|^2 over the bands of a work item in
    // registers; next to the application there are none left for that, and each
    // band adds to its subset's partial plane.
    constexpr bool SUMS = MODE == MODE_DENSITY;
    double dacc[SUMS ? QP : 1];
    if constexpr (SUMS) {
#pragma unroll
        for (int i = 0; i < QP; ++i) dacc[i] = 0.0;
    }

    int rot = 0;
    int jc = j0, kc = 0, z = 0, si = 0, b = 0, np = 0;
    bool have = jc < jend;
    if (have) {
        item_of(jc, kc, z, si, b, np);
        if (np == 0) {
            have = advance(jc, kc);
            if (have) item_of(jc, kc, z, si, b, np);
        }
    }
    if (have) {
        load_seg(si);
        prefetch(z, si, b, np);
    }
    __syncthreads(); // twiddles and the zero in LDS

    while (have) {
        int jn = jc, kn = kc, zn = z, sn = si, bn = b, npn = np;
        const bool more = advance(jn, kn);
        if (more) item_of(jn, kn, zn, sn, bn, npn);
        cx<T> *Sz = slice(z, si, b);

        // y forward, stage A, from the stick values (zero where no stick)
        if constexpr (PRE) {
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                if (ycol[u] < 0 || ycol[u] >= np * psz) continue;
                cx<T> *col = plane + ycol[u];
                T xr[RY], xi[RY];
#pragma unroll
                for (int n1 = 0; n1 < RY; ++n1) {
                    xr[n1] = masked<ZY>(n1) ? T(0) : pre[u * RY + n1].x;
                    xi[n1] = masked<ZY>(n1) ? T(0) : pre[u * RY + n1].y;
                }
                Dft<RY, -1, T>::run(xr, xi);
                twiddle_pw<RY, -1, T>(xr, xi, yn2[u], twy);
#pragma unroll
                for (int k1 = 0; k1 < RY; ++k1) col[L2y * k1] = mk<T>(xr[k1], xi[k1]);
            }
        } else {
            with_size<CY1, MR>(L1y, [&](auto RC) {
                constexpr int R = decltype(RC)::value;
                for (int task = tid; task < np * nxo * L2y; task += nthr) {
                    int p, n2, hc;
                    y_task(task, L2y, p, n2, hc);
                    const int *ys = t.yslot + (long long)(col_off + hc) * N2 + n2;
                    const cx<T> *Sp = Sz + (long long)p * pstride;
                    int sl[R];
#pragma unroll
                    for (int n1 = 0; n1 < R; ++n1) sl[n1] = masked<ZY>(n1) ? -1 : ys[L2y * n1];
                    T xr[R], xi[R];
#pragma unroll
                    for (int n1 = 0; n1 < R; ++n1) {
                        cx<T> v = mk<T>(T(0), T(0));
                        if (!masked<ZY>(n1) && sl[n1] >= 0) v = Sp[sl[n1]];
                        xr[n1] = v.x;
                        xi[n1] = v.y;
                    }
                    Dft<R, -1, T>::run(xr, xi);
                    twiddle_pw<R, -1, T>(xr, xi, n2, twy);
                    cx<T> *col = plane + p * psz + hc * ldy + n2;
#pragma unroll
                    for (int k1 = 0; k1 < R; ++k1) col[L2y * k1] = mk<T>(xr[k1], xi[k1]);
                }
            });
        }
        __syncthreads();
        // y stage B of either direction
        auto y_stage_b = [&](auto SC) {
            constexpr int SGN = decltype(SC)::value;
            with_size<CY2, MR>(L2y, [&](auto RC) {
                constexpr int R = decltype(RC)::value;
                for (int task = tid; task < np * nxo * L1y; task += nthr) {
                    int p, k1, hc;
                    y_task(task, L1y, p, k1, hc);
                    cx<T> *col = plane + p * psz + hc * ldy + L2y * k1;
                    T xr[R], xi[R];
#pragma unroll
                    for (int i = 0; i < R; ++i) {
                        cx<T> v = col[i];
                        xr[i] = v.x;
                        xi[i] = v.y;
                    }
                    Dft<R, SGN, T>::run(xr, xi);
#pragma unroll
                    for (int i = 0; i < R; ++i) col[i] = mk<T>(xr[i], xi[i]);
                }
            });
        };
        y_stage_b(std::integral_constant<int, -1>{});
        __syncthreads();

        // x pass: a wavefront per block of 16 rows of a plane, lane = 16 q + row; the
        // deal goes on from where the last plane's ended, so that a remainder does
        // not fall on the same SIMDs on every plane
        const T *VTz = POT ? VT + (long long)z * N1 * N2 : nullptr;
        const int first = wave >= rot ? wave - rot : wave - rot + nwaves;
        if constexpr (!DENS) rot = (rot + P * nrb) % nwaves;
        for (int unit = first; unit < P * nrb; unit += nwaves) {
            const int p = unit / nrb, rb = unit - p * nrb;
            using V4 = double __attribute__((ext_vector_type(4)));
            // partial plane of the band's subset, as VT [k1][yp][k2]
            const int sub = DENS ? (b - kc) / bps + p : 0;
            V4 *part = DENS ? reinterpret_cast<V4 *>(t.partial) +
                                  ((long long)sub * g.N3 + z) * Q * N2
                            : nullptr;
            // lanes past the last row repeat it: same reads, same values written
            const int yp = min(16 * rb + (lane & 15), N2 - 1);
            if (p < np) {
                const int lo = p * psz + (q - hx + N1) * ldy + yp;
                int step = 4 * ldy, wrap = N1 * ldy;
                // runtime sizes: keeps the multiples of the stride out of the scalar registers
                if constexpr (CY1 == 0) asm volatile("" : "+s"(step), "+s"(wrap));
                // the potential of group j: values k2 of k1 = 4 j + q (the last
                // group of a Q that 4 does not divide re-reads k1 = Q - 1)
                auto at_k1 = [&](int j) {
                    const int k1 = (Q % 4 && j == G - 1) ? min(4 * j + q, Q - 1) : 4 * j + q;
                    return k1 * N2 + yp;
                };
                const V4 *Vz = reinterpret_cast<const V4 *>(VTz);
                // groups whose potential is loaded ahead
                constexpr int AH = DENS ? 1 : 2;
                V4 vq[AH];
                if constexpr (POT) {
#pragma unroll
                    for (int j = 0; j < AH && j < G; ++j) vq[j] = Vz[at_k1(j)];
                }
                T xr[QP], xi[QP];
                int at = lo; // of point n with x <= hmax; those at x >= N1 + hmin lie wrap lower
#pragma unroll
                for (int n = 0; n < QP; ++n) {
                    cx<T> v = mk<T>(T(0), T(0));
                    if (n < Q && !((ZM >> n) & 1)) {
                        if ((LO >> n) & 1)
                            v = plane[at];
                        else if ((HI >> n) & 1)
                            v = plane[at - wrap];
                        else
                            v = plane[n >= nT ? at - wrap : n < nV ? at : izero];
                    }
                    xr[n] = v.x;
                    xi[n] = v.y;
                    at += step;
                }
                Dft<Q, -1, T>::run(xr, xi);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < G; ++j) {
                    T *zr = xr + 4 * j, *zi = xi + 4 * j;
                    V4 d = V4(T(0));
                    if constexpr (DENS && !SUMS) d = part[at_k1(j)];
                    quad_transpose(zr);
                    quad_transpose(zi);
                    const int k1 = (Q % 4 && j == G - 1) ? min(4 * j + q, Q - 1) : 4 * j + q;
                    cx<T> w[3];
#pragma unroll
                    for (int s = 0; s < 3; ++s) {
                        w[s] = twx[3 * k1 + s];
                        const T u = zr[s + 1], v = zi[s + 1];
                        zr[s + 1] = u * w[s].x - v * w[s].y;
                        zi[s + 1] = u * w[s].y + v * w[s].x;
                    }
                    Dft<4, -1, T>::run(zr, zi);
                    if constexpr (DENS) {
                        const double wb = t.wts[band0 + b + p * bps];
#pragma unroll
                        for (int k2 = 0; k2 < 4; ++k2) {
                            const double v = wb * (zr[k2] * zr[k2] + zi[k2] * zi[k2]);
                            if constexpr (SUMS)
                                dacc[4 * j + k2] += v;
                            else
                                d[k2] += v;
                        }
                        if constexpr (!SUMS) {
                            if (Q % 4 == 0 || j < G - 1 || 4 * j + q < Q) part[at_k1(j)] = d;
                        }
                    }
                    if constexpr (POT) {
                        const V4 v = vq[j % AH];
                        if (j + AH < G) vq[j % AH] = Vz[at_k1(j + AH)];
#pragma unroll
                        for (int k2 = 0; k2 < 4; ++k2) {
                            zr[k2] *= v[k2];
                            zi[k2] *= v[k2];
                        }
                        Dft<4, +1, T>::run(zr, zi);
#pragma unroll
                        for (int s = 0; s < 3; ++s) {
                            const T u = zr[s + 1], y = zi[s + 1];
                            zr[s + 1] = u * w[s].x + y * w[s].y;
                            zi[s + 1] = y * w[s].x - u * w[s].y;
                        }
                        quad_transpose(zr);
                        quad_transpose(zi);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (POT) {
                    Dft<Q, +1, T>::run(xr, xi);
                    int to = lo;
#pragma unroll
                    for (int n = 0; n < Q; ++n) {
                        if (!((ZM >> n) & 1)) {
                            if ((LO >> n) & 1)
                                plane[to] = mk<T>(xr[n], xi[n]);
                            else if ((HI >> n) & 1)
                                plane[to - wrap] = mk<T>(xr[n], xi[n]);
                            else if (n >= nT || n < nV)
                                plane[n >= nT ? to - wrap : to] = mk<T>(xr[n], xi[n]);
                        }
                        to += step;
                    }
                }
            }
            if constexpr (SUMS) {
                // the sums go to the subset's partial plane when the work item ends
                // (or after every band where a wavefront has several row blocks)
                if ((P * nrb > nwaves || !more || jn != jc) && sub < nsub) {
#pragma unroll
                    for (int j = 0; j < G; ++j) {
                        if (Q % 4 == 0 || j < G - 1 || 4 * j + q < Q) {
                            V4 &d = part[(4 * j + q) * N2 + yp];
                            d += V4{dacc[4 * j], dacc[4 * j + 1], dacc[4 * j + 2], dacc[4 * j + 3]};
                        }
#pragma unroll
                        for (int k2 = 0; k2 < 4; ++k2) dacc[4 * j + k2] = 0.0;
                    }
                }
            }
        }
        // the next planes' stick values, loaded behind the reverse y pass
        prefetch_none();
        if (more && sn == cur_seg) prefetch(zn, sn, bn, npn);
        __syncthreads();
        if constexpr (POT) {
            y_stage_b(std::integral_constant<int, 1>{});
            __syncthreads();
            // y reverse, stage A', stick positions stored straight to S; stage A of
            // the next planes writes only the thread's own positions, so no barrier
            if constexpr (PRE) {
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    if (ycol[u] < 0 || ycol[u] >= np * psz) continue;
                    cx<T> *col = plane + ycol[u];
                    T xr[RY], xi[RY];
#pragma unroll
                    for (int k1 = 0; k1 < RY; ++k1) {
                        cx<T> v = col[L2y * k1];
                        xr[k1] = v.x;
                        xi[k1] = v.y;
                    }
                    twiddle_pw<RY, +1, T>(xr, xi, yn2[u], twy);
                    Dft<RY, +1, T>::run(xr, xi);
#pragma unroll
                    for (int n1 = 0; n1 < RY; ++n1) {
                        if (masked<ZY>(n1)) continue;
                        const int sl = slot_at(u * RY + n1);
                        if (sl != 0xFFFF) Sz[yoff[u] + sl] = mk<T>(xr[n1], xi[n1]);
                    }
                }
            } else {
                with_size<CY1, MR>(L1y, [&](auto RC) {
                    constexpr int R = decltype(RC)::value;
                    for (int task = tid; task < np * nxo * L2y; task += nthr) {
                        int p, n2, hc;
                        y_task(task, L2y, p, n2, hc);
                        const int *ys = t.yslot + (long long)(col_off + hc) * N2 + n2;
                        cx<T> *Sp = Sz + (long long)p * pstride;
                        int sl[R];
#pragma unroll
                        for (int n1 = 0; n1 < R; ++n1)
                            sl[n1] = masked<ZY>(n1) ? -1 : ys[L2y * n1];
                        cx<T> *col = plane + p * psz + hc * ldy + n2;
                        T xr[R], xi[R];
#pragma unroll
                        for (int k1 = 0; k1 < R; ++k1) {
                            cx<T> v = col[L2y * k1];
                            xr[k1] = v.x;
                            xi[k1] = v.y;
                        }
                        twiddle_pw<R, +1, T>(xr, xi, n2, twy);
                        Dft<R, +1, T>::run(xr, xi);
#pragma unroll
                        for (int n1 = 0; n1 < R; ++n1)
                            if (!masked<ZY>(n1) && sl[n1] >= 0)
                                Sp[sl[n1]] = mk<T>(xr[n1], xi[n1]);
                    }
                });
            }
        }
        if (more && sn != cur_seg) {
            // another segment: its columns are dealt to the threads anew
            __syncthreads();
            load_seg(sn);
            prefetch(zn, sn, bn, npn);
        }
        have = more;
        jc = jn;
        kc = kn;
        z = zn;
        si = sn;
        b = bn;
        np = npn;
    }
}

// ------------------------------------------------------------- launcher

// Planes per workgroup whose offsets from the first one's slice of S, counted in
// values, stay within 31 bits (a density workgroup's planes are a whole band subset
// apart).
template <int MODE>
static int lq_max_planes(const Geometry &g, const Launch &L)
{
    long long nst = 0, step = 1;
    for (int s = 0; s < L.nseg; ++s) nst = std::max<long long>(nst, L.seg[s].nst);
    if (MODE != MODE_APPLY) step = (L.nbt + g.nsub - 1) / g.nsub;
    const long long most = 0x7FFFFFFFLL / std::max(1LL, step * g.N3 * nst);
    return (int)std::max(1LL, std::min(4LL, most));
}

template <int MODE, int Q, int CLS, int CY1, int CY2, int ZY, int YT, int MR>
static hipError_t launch_lq_kernel(const Geometry &g, LaneQuads lq, const DevTables &t,
                                   const Launch &L, void *S, const void *VT, int64_t band0,
                                   hipStream_t st)
{
    constexpr int WPE = lq_wpe(MODE, Q, MR), MAXT = 256 * WPE;
    auto kern = k_plane_lq<MODE, Q, lq_mask(Q, CLS, 0), lq_mask(Q, CLS, 1), lq_mask(Q, CLS, 2),
                           CY1, CY2, ZY, YT, MR, MAXT, WPE>;
    const LqLaunch ll = lq_launch(g, lq, MODE, MODE == MODE_APPLY ? L.nbt : g.nsub,
                                  lq_max_planes<MODE>(g, L));
    lq.planes = ll.planes;
    hipError_t e = allow_lds(kern, (size_t)ll.lds);
    if (e != hipSuccess) return e;
    long long per_z = 0;
    if (MODE == MODE_APPLY)
        for (int s = 0; s < L.nseg; ++s) per_z += (L.seg[s].nb + ll.planes - 1) / ll.planes;
    else
        per_z = (g.nsub + ll.planes - 1) / ll.planes;
    const long long blocks = std::min<long long>(per_z * g.N3, ll.resident);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(ll.threads), (size_t)ll.lds, st, g, lq,
                       t, L, reinterpret_cast<double2 *>(S), reinterpret_cast<const double *>(VT),
                       (long long)band0);
    return hipGetLastError();
}

// Mask class and y split of one Q.
template <int MODE, int Q>
static hipError_t launch_lq_q(const Geometry &g, const LaneQuads &lq, const DevTables &t,
                              const Launch &L, void *S, const void *VT, int64_t band0,
                              hipStream_t st)
{
    // the compiled y splits, where the plans' rows leave the zero mask empty
#define VLOC_LQ_YC(C, Y1, Y2, ZY)                                                                  \
    if (lq.cls == C)                                                                              \
        return launch_lq_kernel<MODE, Q, C, Y1, Y2, ZY, 2, 16>(g, lq, t, L, S, VT, band0, st);
#define VLOC_LQ_Y(QQ, Y1, Y2, ZY)                                                                  \
    if constexpr (Q == QQ)                                                                         \
        if (lq.ysplit && g.L1y == Y1 && g.L2y == Y2) {                                            \
            VLOC_LQ_YC(1, Y1, Y2, ZY)                                                             \
            VLOC_LQ_YC(2, Y1, Y2, ZY)                                                             \
            VLOC_LQ_YC(3, Y1, Y2, ZY)                                                             \
            VLOC_LQ_YC(4, Y1, Y2, ZY)                                                             \
            return hipErrorInvalidValue;                                                          \
        }
    VLOC_LQ_YSPLITS(VLOC_LQ_Y)
#undef VLOC_LQ_Y
#undef VLOC_LQ_YC
    // runtime y sizes
    auto sized = [&](auto cls) {
        constexpr int C = decltype(cls)::value;
        return lq_ymax(g) <= 12
                   ? launch_lq_kernel<MODE, Q, C, 0, 0, 0, 0, 12>(g, lq, t, L, S, VT, band0, st)
                   : launch_lq_kernel<MODE, Q, C, 0, 0, 0, 0, 16>(g, lq, t, L, S, VT, band0, st);
    };
    switch (lq.cls) {
    case 0: return sized(std::integral_constant<int, 0>{});
    case 1: return sized(std::integral_constant<int, 1>{});
    case 4: return sized(std::integral_constant<int, 4>{});
    default: return hipErrorInvalidValue;
    }
}

template <int MODE>
hipError_t launch_plane_lq_mode(const Geometry &g, const LaneQuads &lq, const DevTables &t,
                                const Launch &L, void *S, const void *VT, int64_t band0,
                                hipStream_t st)
{
    switch (lq.q) {
#define VLOC_LQ_CASE(Q)                                                                            \
    case Q: return launch_lq_q<MODE, Q>(g, lq, t, L, S, VT, band0, st);
    VLOC_LQ_SIZES(VLOC_LQ_CASE)
#undef VLOC_LQ_CASE
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_plane_lq_mode<VLOC_LQ_MODE>(const Geometry &, const LaneQuads &,
                                                       const DevTables &, const Launch &, void *,
                                                       const void *, int64_t, hipStream_t);

} // namespace vloc
