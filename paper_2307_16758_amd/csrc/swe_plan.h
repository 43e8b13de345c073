// Tile plan of the tiled stage kernels: for every tile (at most TILE
// consecutive cells), the cells its edges read and the edges themselves,
// built once per mesh on the device.
//
// A tile's cells have the slots 0 .. TILE-1; the cells outside it that its
// edges need (those across an edge and, for MUSCL and WAF, their other
// neighbours) are its halo, slots TILE .. TILE + hs - 1, listed once each in
// ascending order.  Every edge of the tile's cells is one entry in canonical
// orientation (L the cell of smaller global id, L's outward normal): inside
// edges first, then edges leaving the tile (each side's tile has its own
// entry), then boundary edges.  The stage kernels then need no neighbour
// table: all addresses are known before the first load returns, the states
// are gathered once per tile, and everything an edge reads is in LDS or in
// one contiguous stream.
//
// Entry (two words):
//   x: L slot (10) | R slot (10) | mL (2) | mR (2) | low 8 bits of Rb
//   y: La (10) | Lb (10) | Ra (10) | high 2 bits of Rb
// mL, mR: the edge's local number in L and R; La, Lb (Ra, Rb): the two other
// neighbours of L (R).  Where one of them is missing its place holds the
// other, so their mean is the existing one; where both are, both hold the last
// halo slot, which no cell takes and the kernels keep dry: the side then stays
// first order (with the cell itself there, a zero slope, its bed would come
// back as eta - h, a rounding away from b).  A boundary edge has R = kNoCell,
// its cell as L and minus its tag in the last byte of x.
#pragma once

#include <hip/hip_runtime.h>

#include "swe_internal.h"
#include "swe_kernels.h"

namespace swe {

constexpr unsigned kNoCell = 1023u;
constexpr int kMaxSlots = 1023;  // 10-bit slots, kNoCell excluded
constexpr int kDeepHalo = 132;   // largest plain halo (with its dry slot) of a tile of a DEEP plan

// One block per tile, threads = min(TILE, 256).  desc[tile] comes in with x:
// the tile's first cell and y: its cells.  write == 0: z becomes the halo's
// cells and w the tile's edges; otherwise z becomes the scenario (-1 when the
// tile holds several), w the edges to other cells and, from bit 16, the
// boundary edges, and the tile's halo list (-1 after its end) and entries are
// written.  ring2: list the far cells' other neighbours too.
//
// DEEP: the plan of a whole two-stage step in one launch.  The cells are the
// tile's and, in the slots from TILE on, those of its plain halo (base, base_hs
// places, -1 after its end): their first stage is computed too.  The halo is
// theirs, in the slots from TILE + base_hs on, and the entries are all of
// their edges.
template <int TILE, bool DEEP>
__global__ void __launch_bounds__(TILE < 256 ? TILE : 256)
k_tile_plan(const int4 *nbr, int ring2, int write, int hs, int es, int4 *desc, int *halo, uint2 *ent,
            const int *base, int base_hs)
{
    constexpr int NT = TILE < 256 ? TILE : 256, CELLS = TILE + (DEEP ? kDeepHalo : 0);
    constexpr int CAP = CELLS * 9 <= 1024 ? 1024 : (CELLS * 9 <= 2048 ? 2048 : (CELLS * 9 <= 4096 ? 4096 : 8192));
    __shared__ int sBase[DEEP ? kDeepHalo : 1];
    __shared__ int sNb;
    __shared__ int sC[CAP];
    __shared__ int sScan[NT];
    __shared__ unsigned long long sScan64[NT];
    __shared__ int sCnt, sUniq;
    const int t = threadIdx.x, tile = blockIdx.x, c0 = desc[tile].x, c1 = c0 + desc[tile].y;
    const int nown = c1 - c0;
    if (t == 0) { sCnt = 0; sNb = 0; }
    __syncthreads();
    if constexpr (DEEP) {
        int mine = 0;
        for (int i = t; i < base_hs; i += NT) {
            const int k = base[(size_t)tile * base_hs + i];
            sBase[i] = k;
            mine += k >= 0;
        }
        atomicAdd(&sNb, mine);
        __syncthreads();
    }
    const int nbase = sNb, ncell = nown + nbase;
    // place of cell k in an ascending list, -1 if it is not there
    const auto find = [](const int *list, int m, int k) {
        int lo = 0, hi = m;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (list[mid] < k) lo = mid + 1;
            else hi = mid;
        }
        return lo < m && list[lo] == k ? lo : -1;
    };
    // slot of a cell of the tile, -1 outside
    const auto inner = [&](int k) {
        if (k >= c0 && k < c1) return k - c0;
        const int j = DEEP ? find(sBase, nbase, k) : -1;
        return j < 0 ? -1 : TILE + j;
    };
    const auto inside = [&](int k) { return inner(k) >= 0; };
    const auto cell_at = [&](int i) { return i < nown ? c0 + i : sBase[DEEP ? i - nown : 0]; };
    const int per = (ncell + NT - 1) / NT;  // cells of a thread, contiguous
    const auto third = [](const int4 &v, int m) { return m == 0 ? v.x : (m == 1 ? v.y : v.z); };
    for (int ic = t; ic < ncell; ic += NT) {
        const int4 q = nbr[cell_at(ic)];
        for (int m = 0; m < 3; ++m) {
            const int k = third(q, m);
            if (k < 0 || inside(k)) continue;
            sC[atomicAdd(&sCnt, 1)] = k;
            if (!ring2) continue;
            const int4 p = nbr[k];
            const int jb = ((unsigned)q.w >> (2 * m)) & 3;
            for (int j = 1; j < 3; ++j) {
                const int kk = third(p, (jb + j) % 3);
                if (kk >= 0 && !inside(kk)) sC[atomicAdd(&sCnt, 1)] = kk;
            }
        }
    }
    __syncthreads();
    const int cnt = sCnt;
    int P = NT;
    while (P < cnt) P <<= 1;
    for (int i = cnt + t; i < P; i += NT) sC[i] = 0x7fffffff;
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1)  // bitonic sort, ascending
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = t; i < P; i += NT) {
                const int l = i ^ j;
                if (l > i) {
                    const int x = sC[i], y = sC[l];
                    if ((x > y) == ((i & k) == 0)) { sC[i] = y; sC[l] = x; }
                }
            }
            __syncthreads();
        }
    // unique: every thread owns a contiguous run of P / NT values; a scan of
    // the runs' counts gives the places
    const int run = P / NT, r0 = t * run;
    int heads = 0;
    for (int i = r0; i < r0 + run; ++i)
        heads += sC[i] != 0x7fffffff && (i == 0 || sC[i] != sC[i - 1]);
    sScan[t] = heads;
    __syncthreads();
    for (int d = 1; d < NT; d <<= 1) {
        const int v = t >= d ? sScan[t - d] : 0;
        __syncthreads();
        sScan[t] += v;
        __syncthreads();
    }
    const int at0 = sScan[t] - heads;
    if (t == NT - 1) sUniq = sScan[t];
    int prev = r0 > 0 ? sC[r0 - 1] : -1;
    __syncthreads();  // the run before is read before its owner moves values
    // compaction in place moves values to the left only; runs are handled in
    // thread order by going through registers first
    {
        int keep[CAP / NT];
#pragma unroll 1
        for (int i = 0; i < run; ++i) {
            const int v = sC[r0 + i];
            keep[i] = v != 0x7fffffff && v != prev ? v : -1;
            prev = v;
        }
        __syncthreads();
        int at = at0;
#pragma unroll 1
        for (int i = 0; i < run; ++i)
            if (keep[i] >= 0) sC[at++] = keep[i];
    }
    __syncthreads();
    const int nh = sUniq;
    // edges: counts per cell (inside | outside | boundary, 21 bits each)
    unsigned long long mine = 0;
    int smin = 0x7fffffff, smax = -1;
    for (int i = t * per; i < (t + 1) * per && i < ncell; ++i) {
        const int4 q = nbr[cell_at(i)];
        const int s = (int)((unsigned)q.w >> kScenShift);
        smin = s < smin ? s : smin;
        smax = s > smax ? s : smax;
        for (int m = 0; m < 3; ++m) {
            const int k = third(q, m);
            if (k < 0) mine += 1ull << 42;
            else if (!inside(k)) mine += 1ull << 21;
            else if (((unsigned)q.w >> (6 + m)) & 1u) mine += 1ull;
        }
    }
    sScan64[t] = mine;
    sScan[t] = smin;
    __syncthreads();
    for (int d = 1; d < NT; d <<= 1) {
        const unsigned long long v = t >= d ? sScan64[t - d] : 0ull;
        __syncthreads();
        sScan64[t] += v;
        __syncthreads();
    }
    const unsigned long long all = sScan64[NT - 1], before = sScan64[t] - mine;
    const int ni = (int)(all & 0x1fffff), no = (int)((all >> 21) & 0x1fffff), nb = (int)(all >> 42);
    if (!write) {
        if (t == 0) {
            desc[tile].z = nh;
            desc[tile].w = ni + no + nb;
        }
        return;
    }
    // one scenario in the whole tile?  (sScan holds the threads' minima)
    const int first = sScan[0];
    const int mixed = __syncthreads_or(smax >= 0 && (smin != first || smax != first));
    if (t == 0) desc[tile] = make_int4(c0, c1 - c0, mixed ? -1 : first, (ni + no) | (nb << 16));
    for (int i = t; i < hs; i += NT) halo[(size_t)tile * hs + i] = i < nh ? sC[i] : -1;
    const auto slot = [&](int k) -> unsigned {
        const int in = inner(k);
        return (unsigned)(in >= 0 ? in : TILE + (DEEP ? base_hs : 0) + find(sC, nh, k));
    };
    uint2 *e = ent + (size_t)tile * es;
    int ai = (int)(before & 0x1fffff), ao = ni + (int)((before >> 21) & 0x1fffff),
        ab = ni + no + (int)(before >> 42);
    for (int i = t * per; i < (t + 1) * per && i < ncell; ++i) {
        const int c = cell_at(i);
        const unsigned sc = (unsigned)(i < nown ? i : TILE + i - nown);
        const int4 q = nbr[c];
        for (int m = 0; m < 3; ++m) {
            const int k = third(q, m);
            if (k < 0) {
                e[ab++] = make_uint2(sc | (kNoCell << 10) | ((unsigned)m << 20) |
                                         ((unsigned)(-k) << 24), 0u);
                continue;
            }
            const bool in = inside(k), isL = ((unsigned)q.w >> (6 + m)) & 1u;
            if (in && !isL) continue;
            const int4 p = nbr[k];
            const int jb = ((unsigned)q.w >> (2 * m)) & 3;
            int ca = third(q, (m + 1) % 3), cb = third(q, (m + 2) % 3);
            int ka = third(p, (jb + 1) % 3), kb = third(p, (jb + 2) % 3);
            if (ca < 0) ca = cb;
            if (cb < 0) cb = ca;
            if (ka < 0) ka = kb;
            if (kb < 0) kb = ka;
            const unsigned sk = slot(k), dry = (unsigned)(TILE + (DEEP ? base_hs : 0) + hs - 1);
            unsigned xa = sc, xb = sc, ya = sk, yb = sk;
            if (ring2) {
                xa = ca < 0 ? dry : slot(ca);
                xb = cb < 0 ? dry : slot(cb);
                ya = ka < 0 ? dry : slot(ka);
                yb = kb < 0 ? dry : slot(kb);
            }
            const unsigned L = isL ? sc : sk, R = isL ? sk : sc, mL = isL ? m : jb, mR = isL ? jb : m;
            const unsigned La = isL ? xa : ya, Lb = isL ? xb : yb, Ra = isL ? ya : xa, Rb = isL ? yb : xb;
            e[in ? ai++ : ao++] = make_uint2(L | (R << 10) | (mL << 20) | (mR << 22) | ((Rb & 255u) << 24),
                                             La | (Lb << 10) | (Ra << 20) | ((Rb >> 8) << 30));
        }
    }
}

// Geometry of the entries, from the per-half-edge arrays of the mesh
// (edge-major): the unit normal of L and, where asked for, the MUSCL weights
// (L's backward and forward, R's backward and forward), the learned
// limiter's central weights of L and R, and WAF's centroid distance.  One
// block per tile.
template <typename T>
__global__ void __launch_bounds__(256)
k_plan_geometry(int n, int TILE, const int4 *desc, const int *halo, const uint2 *ent, int hs, int es,
                const int *base, int base_hs,
                const typename V4<T>::type *he_co, const T *he_gam, const T *he_dfw,
                typename V2<T>::type *nrm, typename V4<T>::type *wgt, typename V2<T>::type *gam, T *dfw)
{
    const int tile = blockIdx.x, c0 = desc[tile].x, nt = (desc[tile].w & 0xffff) + (desc[tile].w >> 16);
    // base: a DEEP plan (base_hs is 0 otherwise)
    const auto cell = [&](int slot) {
        if (slot < TILE) return c0 + slot;
        slot -= TILE;
        return slot < base_hs ? base[(size_t)tile * base_hs + slot] : halo[(size_t)tile * hs + slot - base_hs];
    };
    for (int i = threadIdx.x; i < nt; i += blockDim.x) {
        const size_t at = (size_t)tile * es + i;
        const unsigned x = ent[at].x;
        const int L = x & 1023u, R = (x >> 10) & 1023u, mL = (x >> 20) & 3u, mR = (x >> 22) & 3u;
        const int cL = cell(L);
        const auto a = he_co[(size_t)mL * n + cL];
        typename V2<T>::type v;
        v.x = a.x; v.y = a.y;
        nrm[at] = v;
        if (R == (int)kNoCell) continue;
        const int cR = cell(R);
        if (wgt) {
            const auto b = he_co[(size_t)mR * n + cR];
            typename V4<T>::type w;
            w.x = a.z; w.y = a.w; w.z = b.z; w.w = b.w;
            wgt[at] = w;
        }
        if (dfw) dfw[at] = he_dfw[(size_t)mL * n + cL];
        if (gam) {
            v.x = he_gam[(size_t)mL * n + cL];
            v.y = he_gam[(size_t)mR * n + cR];
            gam[at] = v;
        }
    }
}

}  // namespace swe
