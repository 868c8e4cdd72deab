// Patch kernel of the reduced two-dimensional problems (cylindrical orders,
// k_z points, Bloch-periodic x): one block carries one channel through clear,
// kick, start and all its steps in a single launch, with every field value in
// a register.
//
// A thread owns a patch of CX x B cells (columns x rows); LX x LY patches
// cover the grid, of which those with a cell that can change are listed (open
// runs: all).  Inside the patch a neighbour is a register; the patch's
// lowest row and first column of E and highest row and last column of H go
// through LDS, one entry of S values per thread, read by the threads below /
// left (E) and above / right (H).  A neighbour index is formed once per
// thread: beyond a wall it points at an entry of zeros, across a periodic
// edge at the wrapped thread, so the half steps hold no edge tests.  The entry
// stride S is odd, so that the 64 lanes' reads of one value fall on different
// banks.  Two barriers per step: E and H entries have buffers of their own,
// so a write is separated from the last reads of its buffer by the other half
// step's barrier.
//
// Coefficients: x <- a x -/+ b curl has one a per field group outside
// conductors (1, or the conductivity's factor), where b = 0 the field is 0 and
// stays 0 whatever a is; so a is a scalar and a cell looks up only its three
// b values, by its coefficient class, in LDS.
//
// What bounds it: VALU issue (about 40 instructions per cell-update and part)
// and the register file, which caps the cells of a CU: 6 (12 complex) values
// per cell of 512 KB.  The kernel with one cell list per thread (k_red_regs)
// reads four neighbours and writes three values in LDS per cell and half step
// and recomputes every cell's coordinates; a patch of 5 x 5 cells reads and
// writes 1.6 and computes none.  k_z piston (80 x 40, 1856 channels, 2000
// steps, FP32): 56.5 -> 14.7 ms on the device (17.3 with the H coefficients
// looked up, see HU; 15.4 with copies of updated fields, see upd_h), 8.8 with the
// patches left out that hold only conductor (half of this grid); Bloch grating
// (48 x 60, 4096 complex channels, 2000 steps, FP32): 177.7 -> 54.4 ms (59.7 with
// the copies).
#pragma once

#include <algorithm>
#include <type_traits>

#include "../../include/casimir_fdtd.h"
#include "device.hpp"
#include "red_common.hpp"
#include "red_patch.hpp"
#include "yee_common.hpp"

namespace cf {

namespace {

using yee::as_global;

// LDS of a block, byte offsets into the dynamic array.
struct PatchLds {
    int tab[2];    // b values of the H and the E classes, 4 (3 used) per class
    int sw, sb;    // surface weights and basis row (FP64)
    int xe, xh;    // exchange entries of E and H
    int rows;      // row factors (cylindrical)
    int stage;     // measured (and at the start the kicked) component inside its box
    int so;        // surface point offsets into the stage
    int ez;        // LZ: E_z entries
    int prof;      // open: CPML (b, c) pairs, [x half, x whole, y half, y whole][position]
    int psi;       // open: psi of the x differences, one entry per thread with x-layer cells
    int pol;       // open: E, then the polarizations' share of its update, per dispersive cell and component
    int prow;      // and its Lorentz row
    int lrow, lor; // open: Lorentz row of each E class and component; the rows (row 0: no term)
    int total;
};
// What an open (CPML) or dispersive run adds to a launch.
struct OpenSizes {
    int prof = 0;        // profile pairs
    int psi = 0;         // values of all x psi entries
    int pol = 0;         // dispersive cells times 3
    int n_lor = 0, lor_rows = 0;
};
__host__ __device__ inline PatchLds patch_lds(int nt, int S, int ZS, bool overlay, int tsz, int n_h, int n_e,
                                              int n_rows, const PatchSizes& z, const OpenSizes& os) {
    PatchLds l;
    int at = 0;
    auto take = [&](int bytes) {
        const int p = at;
        at += (bytes + 15) & ~15;
        return p;
    };
    l.tab[0] = take(n_h * 4 * tsz);
    l.tab[1] = take(n_e * 4 * tsz);
    l.sw = take(z.samples * z.points * 8);
    l.sb = take(z.samples * 8);
    // entries: one per patch, the zero entry, and one for threads without a patch
    l.ez = take((nt + 2) * ZS * tsz);
    l.xe = take((nt + 2) * S * tsz);
    l.xh = overlay ? l.xe : take((nt + 2) * S * tsz);
    l.rows = take(n_rows * kRowFactors * tsz);
    l.stage = take(z.box * tsz);
    l.so = take(z.samples * z.points * 2);
    l.prof = take(os.prof * 2 * tsz);
    l.psi = take(os.psi * tsz);
    l.pol = take(os.pol * tsz);
    l.prow = take(os.pol);
    l.lrow = take(os.lor_rows ? n_e * 4 : 0);
    l.lor = take(os.lor_rows * (1 + 3 * os.n_lor) * tsz);
    l.total = at;
    return l;
}

// Entry strides (odd): E and H exchange (one stride for both, so that the two
// have one zero entry when they share a buffer), E_z storage (LZ).
constexpr int patch_stride(int CX, int B, int NP) { return (2 * (CX + B) * NP) | 1; }
constexpr int patch_zs(int CX, int B) { return (CX * B) | 1; }

struct PatchArgs {
    int LX, LY;
    // patches in use, and their list [patch column and row, list indices of the
    // patches right, left, above, below (np: none)], or null: all LX LY of them
    int np;
    const uint16_t* list;
    PatchLds lds;
    // open: patch columns [0, xlo) and [xhi, LX), rows [0, ylo) and [yhi, LY)
    // hold layer cells; psi of the y differences in memory, a region of
    // `scratch_stride` values per block; Lorentz rows as in Grid2D::lor
    int xlo, xhi, ylo, yhi;
    int n_lor, lor_rows, items;
    const double* prof[2];
    void* scratch;
    int64_t scratch_stride;
    double lor[4][13];           // [row][1 / eps, (c1, c2, c3) per term]
    uint8_t lrow[kPatchClasses][3];
};

// A uniform value the compiler cannot see through.
__device__ __forceinline__ int opaque(int v) {
    int r;
    asm volatile("s_mov_b32 %0, %1" : "=s"(r) : "s"(__builtin_amdgcn_readfirstlane(v)));
    return r;
}

// (b0, b1, b2) of a class
template <typename T>
struct B3 {
    T x, y, z;
};
template <typename T>
__device__ __forceinline__ B3<T> class_b(const char* tab, uint32_t cls) {
    const T* q = static_cast<const T*>(__builtin_assume_aligned(tab + cls * (4 * sizeof(T)), 4 * sizeof(T)));
    return B3<T>{q[0], q[1], q[2]};
}

// x <- a x -/+ b d in x's own register (MODE 0), or the consistent start's
// (b / 2) d.  The three-source form matters: with v_fmac the compiler forms
// the sum in the product's register and copies all 6 values of a cell back
// every step.
template <typename T, int MODE>
__device__ __forceinline__ void upd_h(T& x, T a, T b, T d) {
    if constexpr (MODE == 0) yee::sub_into(x, a, b, d);
    else x = yee::half(b, d);
}
template <typename T, int MODE>
__device__ __forceinline__ void upd_e(T& x, T a, T b, T d) {
    if constexpr (MODE == 0) yee::add_into(x, a, b, d);
    else x = yee::half(b, d);
}

constexpr bool patch_packs(bool lz, bool open) { return lz && !open; }

// HU: every cell of the grid has the same H class, so the H half step takes its
// three b values as scalars (cells of a patch beyond the grid then keep
// H = 0 because E is 0 there and above and to the right of them).
// MW: waves per SIMD the register budget is sized for (the launch keeps the
// block within 4 MW waves).
// LZ: E_z lives in LDS instead of registers, one entry per thread, from which
// the neighbours read it too; the E and H exchange entries then share one
// buffer, with two more barriers per step.  For the largest grids: 8400 cells
// in FP64 need 18 per thread, 216 registers of field values, 180 without E_z
// (cylindrical piston, 400 x 21, 126 channels, FP64, 6000 base steps: 291 ms
// on the global-memory kernel, 57.3 ms here).
// OPEN (k_z runs): in-plane CPML and Lorentz polarizations.  Each psi and
// polarization belongs to one cell and so to one thread: psi of the x
// differences and the polarizations in LDS, psi of the y differences in
// memory (L2), loaded one row ahead, in a scratch region per block.  Two
// waveguides (130 x 90, CPML of 20 cells on four sides, one Lorentz term, 1024
// channels, 1000 steps, FP32): 476 ms on the split kernels, which move every
// field through memory twice a step, 51.8 ms here (107.6 with row-major threads
// and each polarization advanced by its patch's thread: the few waves with
// dispersive cells then held up every step for 15 us).
template <typename T, int CX, int B, bool CYL, bool CPLX, int MW, bool LZ, bool OPEN, bool HU>
__global__ __launch_bounds__(256 * MW) __attribute__((amdgpu_waves_per_eu(MW)))
void k_red_patch(T* __restrict__ fields, const ChanDev* __restrict__ ch, const int* __restrict__ slots, int first,
                 int nslots, Grid2D g, RedOrders ord, RedSpan sp, SurfTables t, PatchClasses pc, PatchArgs pa, double dA,
                 double* __restrict__ acc, double* __restrict__ gamma, int gamma_stride) {
    constexpr int NP = CPLX ? 2 : 1;
    constexpr int S = patch_stride(CX, B, NP), ZS = patch_zs(CX, B);
    constexpr int PS = 2 * (CX + B);               // values of one part in an H entry
    constexpr int PE = LZ ? CX + B : PS;           // and in an E entry: rows (E_z, E_x), columns (E_z, E_y)
    constexpr int OEX = LZ ? 0 : CX;               // offsets of the E_x row, the E_z and E_y columns
    constexpr int OZC = 2 * CX, OYC = LZ ? CX : 2 * CX + B;
    constexpr int NC = CX * B;
    constexpr bool OVERLAY = LZ;
    constexpr int XS = (4 * NC) | 1;               // x psi entry: slots H_y, H_z, E_y, E_z of every cell
    static_assert(NC <= 32, "one mask bit per cell of the patch");
    static_assert(!(LZ && CPLX) && !(OPEN && (CYL || CPLX)), "real runs only; open ones without an axis");
    extern __shared__ __align__(16) char lds[];
    __shared__ int s_box[8];                       // source box (min x, min y, max x, max y), measured box
    __shared__ int s_lor;                          // dispersive cells, numbered patch by patch as they come
    __shared__ double s_acc[2];                    // the channel's compensated accumulator
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int LX = pa.LX, LY = pa.LY;
    // orders are listed from the first; a cylindrical launch takes the last
    // (longest) ones first
    const int item = first + (int)blockIdx.x;
    const int slot = slots ? slots[CYL ? nslots - 1 - item : item] : item;
    const ChanDev d = ch[slot];
    const int m = d.order;
    const int s0 = sp.s0[m], s1 = sp.s1[m];
    const bool resume_later = s1 < ord.steps[m];
    const double dt = ord.dt[m];
    const auto ktab = as_global(ord.ktab + m * ord.ktab_stride);
    const int nx = g.nx, ny = g.ny;
    const bool act = tid < pa.np;
    int tx = tid % LX, ty = tid / LX;
    const bool listed = !OPEN && pa.list != nullptr;
    uint32_t link[2] = {0, 0};                     // right | left << 16, above | below << 16
    if (listed && act) {
        const auto q = reinterpret_cast<yee::gmem<const uint32_t>>(as_global(pa.list)) + 3 * tid;
        tx = q[0] & 0xffff;
        ty = q[0] >> 16;
        link[0] = q[1];
        link[1] = q[2];
    }
    // Open runs: the threads are sorted by what their patches hold, corners
    // of both layers first, then x layers, y layers and the rest, so that few
    // waves carry CPML work, the heaviest one on each SIMD beside a light one.
    const int nxl = OPEN ? pa.xlo + LX - pa.xhi : 0, nyl = OPEN ? pa.ylo + LY - pa.yhi : 0;
    if constexpr (OPEN) {
        const bool in_x = tid < nxl * LY;
        int k = in_x ? tid : tid - nxl * LY;
        const int w = in_x ? nxl : LX - nxl;
        const bool in_y = k < w * nyl;
        if (!in_y) k -= w * nyl;
        const int cx = k % max(w, 1), cy = k / max(w, 1);
        tx = in_x ? (cx < pa.xlo ? cx : pa.xhi + cx - pa.xlo) : pa.xlo + cx;
        ty = in_y ? (cy < pa.ylo ? cy : pa.yhi + cy - pa.ylo) : pa.ylo + cy;
    }
    const int patch = OPEN ? ty * LX + tx : tid;   // its exchange entry
    const int x0 = tx * CX, y0 = ty * B;

    T* const XE = reinterpret_cast<T*>(lds + pa.lds.xe);
    T* const XH = reinterpret_cast<T*>(lds + pa.lds.xh);
    T* const EZ = reinterpret_cast<T*>(lds + pa.lds.ez);
    const int zero = pa.np;                        // the entry of zeros
    T* const stage = reinterpret_cast<T*>(lds + pa.lds.stage);
    T* const rows = reinterpret_cast<T*>(lds + pa.lds.rows);
    double* const sw = reinterpret_cast<double*>(lds + pa.lds.sw);
    double* const sb = reinterpret_cast<double*>(lds + pa.lds.sb);
    uint16_t* const so = reinterpret_cast<uint16_t*>(lds + pa.lds.so);

    // ---- tables -------------------------------------------------------
    {
        const auto lk = as_global(static_cast<const T*>(ord.lut) + m * ord.lut_stride + d.kind * 6 * 256 * 2);
        for (int k = tid; k < (pc.n[0] + pc.n[1]) * 4; k += nthr) {
            const int grp = k >= pc.n[0] * 4, kk = k - (grp ? pc.n[0] * 4 : 0), c = kk >> 2, q = kk & 3;
            T b = T(0);
            if (q < 3 && c > 0) b = lk[(((grp ? CF_EX : CF_HX) + q) * 256 + pc.id[grp][c][q]) * 2 + 1];
            reinterpret_cast<T*>(lds + pa.lds.tab[grp])[kk] = b;
        }
        if (CYL)
            for (int k = tid; k < kRowFactors * ny; k += nthr) rows[k] = as_global(static_cast<const T*>(ord.rows))[k];
        for (int k = tid; k < S; k += nthr) XE[zero * S + k] = XH[zero * S + k] = T(0);
        if (LZ)
            for (int k = tid; k < ZS; k += nthr) EZ[zero * ZS + k] = T(0);
        if (tid < 8) s_box[tid] = (tid & 2) ? -1 : 0x7fffffff;
        if constexpr (OPEN) {
            // (b, c) pairs: H positions, then E positions, of x and then y;
            // (1, 0) on an axis without layers
            T* q = reinterpret_cast<T*>(lds + pa.lds.prof);
            for (int k = tid; k < 2 * (nx + ny); k += nthr) {
                const int ax = k >= 2 * nx, kk = ax ? k - 2 * nx : k, n = ax ? ny : nx;
                const int grp = kk >= n, pos = grp ? kk - n : kk;
                const double* tab = pa.prof[ax];
                q[2 * k] = tab ? T(as_global(tab)[2 * grp * n + pos]) : T(1);
                q[2 * k + 1] = tab ? T(as_global(tab)[(2 * grp + 1) * n + pos]) : T(0);
            }
            if (tid == 0) s_lor = 0;
            for (int k = tid; k < pa.lor_rows * (1 + 3 * pa.n_lor); k += nthr)
                reinterpret_cast<T*>(lds + pa.lds.lor)[k] = T(pa.lor[k / (1 + 3 * pa.n_lor)][k % (1 + 3 * pa.n_lor)]);
            if (pa.lor_rows > 1)
                for (int k = tid; k < pc.n[1] * 4; k += nthr)
                    reinterpret_cast<uint8_t*>(lds + pa.lds.lrow)[k] = (k & 3) < 3 ? pa.lrow[k >> 2][k & 3] : 0;
        }
        __syncthreads();
        for (int k = tid; k < d.n_uniq; k += nthr) {
            const int c = as_global(t.uidx)[d.u_off + k], i = c % nx, j = c / nx;
            atomicMin(&s_box[0], i);
            atomicMin(&s_box[1], j);
            atomicMax(&s_box[2], i);
            atomicMax(&s_box[3], j);
        }
        for (int k = tid; k < d.nsamp * d.P; k += nthr) {
            const int c = as_global(t.gidx)[d.g_off + k], i = c % nx, j = c / nx;
            atomicMin(&s_box[4], i);
            atomicMin(&s_box[5], j);
            atomicMax(&s_box[6], i);
            atomicMax(&s_box[7], j);
        }
        __syncthreads();
    }
    const int mx0 = s_box[4], my0 = s_box[5], mbw = s_box[6] - mx0 + 1;
    for (int k = tid; k < d.nsamp * d.P; k += nthr) {
        const int c = as_global(t.gidx)[d.g_off + k];
        so[k] = (uint16_t)((c / nx - my0) * mbw + (c % nx - mx0));
        sw[k] = as_global(t.gw)[d.g_off + k];
    }
    for (int k = tid; k < d.nsamp; k += nthr) sb[k] = as_global(t.basis)[d.basis_off + k];

    // ---- the patch's classes, neighbours and masks ---------------------
    // the cells' classes, H and E in 16 bits; where the registers are short (LZ)
    // and one H class needs no lookup, 4 bits of E class each (cylindrical
    // piston, 400 x 21, FP64: 62.5 -> 57.3 ms, 56.3 with its 7 % of conductor left
    // out; elsewhere the words cost less than
    // their extraction: k_z piston 14.7 against 15.3 ms)
    constexpr bool C4 = HU && patch_packs(LZ, OPEN);
    constexpr int CPW = C4 ? 8 : 2, CB = 32 / CPW, NW = (NC + CPW - 1) / CPW;
    uint32_t cw[NW];
    uint32_t in_m = 0;                             // cells inside the measured component's box
    const int sx0 = s_box[0], sy0 = s_box[1], sbw = s_box[2] - sx0 + 1, sbh = s_box[3] - sy0 + 1;
    uint32_t in_s = 0;                             // cells inside the source's box
#pragma unroll
    for (int k = 0; k < NW; ++k) cw[k] = 0;
#pragma unroll
    for (int r = 0; r < B; ++r)
#pragma unroll
        for (int j = 0; j < CX; ++j) {
            const int k = r * CX + j, x = x0 + j, y = y0 + r;
            if (act && x < nx && y < ny) {
                const uint32_t c = as_global(pc.cls)[y * nx + x];
                cw[k / CPW] |= (C4 ? c >> 8 : c) << (CB * (k % CPW));
                if (x >= mx0 && x <= s_box[6] && y >= my0 && y <= s_box[7]) in_m |= 1u << k;
                if (x >= sx0 && x <= s_box[2] && y >= sy0 && y <= s_box[3]) in_s |= 1u << k;
            }
        }
    const int n_r = !act ? zero : listed ? link[0] & 0xffff : tx + 1 < LX ? patch + 1 : g.perx ? patch + 1 - LX : zero;
    const int n_l = !act ? zero : listed ? link[0] >> 16 : tx > 0 ? patch - 1 : g.perx ? patch + LX - 1 : zero;
    const int n_u = !act ? zero : listed ? link[1] & 0xffff : ty + 1 < LY ? patch + LX : !CYL && g.pery ? tx : zero;
    const int n_d = !act ? zero : listed ? link[1] >> 16 : ty > 0 ? patch - LX : !CYL && g.pery ? tx + (LY - 1) * LX : zero;
    const T* const er = XE + n_r * S;             // E columns of the patch to the right
    const T* const eu = XE + n_u * S;             // E rows of the patch above
    const T* const hl = XH + n_l * S + 2 * CX;    // H_y, H_z columns of the patch to the left
    const T* const hd = XH + n_d * S;             // H_x, H_z rows of the patch below
    const T* const zr = EZ + n_r * ZS;             // LZ: E_z of the patches to the right and above
    const T* const zu = EZ + n_u * ZS;
    const int me = act ? patch : zero + 1;
    T* const xe = XE + me * S;
    T* const xh = XH + me * S;
    T* const zme = EZ + me * ZS;
    const bool edge_r = CPLX && tx + 1 == LX, edge_l = CPLX && tx == 0;
    const T M = T(ord.coup[m]), la = T(ord.la[m]);
    const T a_e = d.kind == 0 ? la : T(1), a_h = d.kind == 0 ? T(1) : la;
    const T ph_c = CPLX ? T(ord.ph_c[m]) : T(1), ph_s = CPLX ? T(ord.ph_s[m]) : T(0);
    const char* const tab_h = lds + pa.lds.tab[0];
    B3<T> hb{T(0), T(0), T(0)};                    // HU: the b values of class 1
    if constexpr (HU) {
        const auto lk = as_global(static_cast<const T*>(ord.lut) + m * ord.lut_stride + d.kind * 6 * 256 * 2);
        hb = B3<T>{yee::lane_value(lk[(CF_HX * 256 + pc.id[0][1][0]) * 2 + 1], 0),
                   yee::lane_value(lk[(CF_HY * 256 + pc.id[0][1][1]) * 2 + 1], 0),
                   yee::lane_value(lk[(CF_HZ * 256 + pc.id[0][1][2]) * 2 + 1], 0)};
    }
    const char* const tab_e = lds + pa.lds.tab[1];

    T e0[NP][B][CX], e1[NP][B][CX], e2[LZ ? 1 : NP][LZ ? 1 : B][CX], h0[NP][B][CX], h1[NP][B][CX], h2[NP][B][CX];
    // E_z of row r (this patch) as a row of values
    auto ez_row = [&](int p, int r, T (&v)[CX]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < CX; ++j) {
            if constexpr (LZ) v[j] = zme[r * CX + j];
            else v[j] = e2[p][r][j];
        }
    };

    // ---- open runs: the patch's layers and dispersive cells --------------
    int xi = -1, yi = -1, li = -1;                 // entry of x psi, column of y psi, first dispersive cell
    bool any_x = false, any_y = false, any_l = false;
    T* px = nullptr;
    T* const pol = reinterpret_cast<T*>(lds + pa.lds.pol);
    uint8_t* const prow = reinterpret_cast<uint8_t*>(lds + pa.lds.prow);
    __attribute__((address_space(1))) T* py = nullptr;   // y psi
    __attribute__((address_space(1))) T* pq = nullptr;   // polarizations: [term][P^m, P^{m-1}][cell and component]
    int ny_t = 0;                                  // threads with y-layer cells (stride of the y psi)
    uint32_t yv = 0, lmask = 0;                    // lmask: the patch's dispersive cells
    int xq = x0, yq = y0;
    const T* const prof = reinterpret_cast<const T*>(lds + pa.lds.prof);
    const uint8_t* const lrow = reinterpret_cast<const uint8_t*>(lds + pa.lds.lrow);
    const T* const lor = reinterpret_cast<const T*>(lds + pa.lds.lor);
    const int n_lor = pa.n_lor;
    T ya[OPEN ? CX : 1], yb[OPEN ? CX : 1];        // y psi of the next row (two differences)
    if constexpr (OPEN) {
        if (tid < nxl * LY) xi = tid;
        if (act && (ty < pa.ylo || ty >= pa.yhi)) yi = tid < nxl * LY ? tid : tid - nxl * (LY - nyl);
        ny_t = nyl * LX;
        if (pa.lor_rows > 1) {
            for (int k = 0; k < NC; ++k) {
                const int x = x0 + k % CX, y = y0 + k / CX;
                if (act && x < nx && y < ny) {
                    const uint8_t* q = lrow + (as_global(pc.cls)[y * nx + x] >> 8) * 4;
                    if (q[0] | q[1] | q[2]) lmask |= 1u << k;
                }
            }
            if (lmask) li = atomicAdd(&s_lor, __popc(lmask));
            int n = li;
            for (int k = 0; k < NC; ++k)
                if ((lmask >> k) & 1u) {
                    const uint8_t* q = lrow + (as_global(pc.cls)[(y0 + k / CX) * nx + x0 + k % CX] >> 8) * 4;
                    for (int c = 0; c < 3; ++c) prow[3 * n + c] = q[c];
                    ++n;
                }
        }
        px = reinterpret_cast<T*>(lds + pa.lds.psi) + max(xi, 0) * XS;
        py = as_global(static_cast<T*>(pa.scratch) + blockIdx.x * pa.scratch_stride);
        pq = py + (int64_t)4 * NC * ny_t;
        yv = (uint32_t)max(yi, 0);
        if (xi >= 0)
            for (int k = 0; k < 4 * NC; ++k) px[k] = T(0);
        if (yi >= 0)
            for (int k = 0; k < 4 * NC; ++k) (py + k * ny_t)[yv] = T(0);
        for (int q = 0; q < 2 * n_lor; ++q)
            for (int i = tid; i < pa.items; i += nthr) pq[q * pa.items + i] = T(0);
        any_x = __builtin_amdgcn_readfirstlane(__any(xi >= 0)) != 0;
        any_y = __builtin_amdgcn_readfirstlane(__any(yi >= 0)) != 0;
        any_l = __builtin_amdgcn_readfirstlane(__any(li >= 0)) != 0;
    }
    // y psi of row r, group grp (0: H, 1: E), into ya / yb
    auto load_y = [&](int grp, int r) __attribute__((always_inline)) {
        if constexpr (OPEN) {
            if (any_y) {
                const int yst = opaque(ny_t);      // no addresses kept across rows
                if (yi >= 0) {
#pragma unroll
                    for (int j = 0; j < CX; ++j) {
                        ya[j] = (py + ((2 * grp) * NC + r * CX + j) * yst)[yv];
                        yb[j] = (py + ((2 * grp + 1) * NC + r * CX + j) * yst)[yv];
                    }
                }
            }
        }
    };
    // The four differences of row r stretched inside the layers: psi <- b psi
    // + c D, D <- D + psi (outside them b = 1, c = 0 and psi = 0).  xa, xb:
    // the x differences in the group's first and second psi slot; da, db: the
    // y differences.  The next row's y psi are loaded before this row's
    // arithmetic.
    auto stretch = [&](int grp, int r, T (&xa)[CX], T (&xb)[CX], T (&da)[CX], T (&db)[CX]) __attribute__((always_inline)) {
        if constexpr (OPEN) {
            asm volatile("" : "+v"(xq), "+v"(yq));
            if (any_y) {
                T pa_[CX], pb_[CX];
#pragma unroll
                for (int j = 0; j < CX; ++j) {
                    pa_[j] = ya[j];
                    pb_[j] = yb[j];
                }
                if (r + 1 < B) load_y(grp, r + 1);
                const int yst = opaque(ny_t);
                if (yi >= 0) {
                    const T* q = prof + 2 * ((grp ? 2 * nx + ny : 2 * nx) + min(yq + r, ny - 1));
                    const T b = q[0], c = q[1];
#pragma unroll
                    for (int j = 0; j < CX; ++j) {
                        const T u = fma(b, pa_[j], c * da[j]), v = fma(b, pb_[j], c * db[j]);
                        (py + ((2 * grp) * NC + r * CX + j) * yst)[yv] = u;
                        (py + ((2 * grp + 1) * NC + r * CX + j) * yst)[yv] = v;
                        da[j] = da[j] + u;
                        db[j] = db[j] + v;
                    }
                }
            }
            if (any_x) {
                if (xi >= 0) {
#pragma unroll
                    for (int j = 0; j < CX; ++j) {
                        const T* q = prof + 2 * ((grp ? nx : 0) + min(xq + j, nx - 1));
                        const T b = q[0], c = q[1];
                        T* s0_ = px + (2 * grp) * NC + r * CX + j;
                        T* s1_ = s0_ + NC;
                        const T u = fma(b, *s0_, c * xa[j]), v = fma(b, *s1_, c * xb[j]);
                        *s0_ = u;
                        *s1_ = v;
                        xa[j] = xa[j] + u;
                        xb[j] = xb[j] + v;
                    }
                }
            }
        }
    };
    // Polarizations.  The threads whose patches hold dispersive cells put E of
    // those cells into `pol`; behind the next barrier all threads share the
    // (cell, component) items, advance their P from E^m and leave there what
    // the E update of D = eps_inf E + sum P subtracts (the operations of
    // yee::lorentz_step).
    auto share_e = [&]() __attribute__((always_inline)) {
        if constexpr (OPEN) {
            if (any_l) {
#pragma unroll
                for (int k = 0; k < NC; ++k)
                    if ((lmask >> k) & 1u) {
                        T* at = pol + 3 * (li + __popc(lmask & ((1u << k) - 1u)));
                        at[0] = e0[0][k / CX][k % CX];
                        at[1] = e1[0][k / CX][k % CX];
                        if constexpr (LZ) at[2] = zme[k];
                        else at[2] = e2[0][k / CX][k % CX];
                    }
            }
        }
    };
    auto polarize = [&]() __attribute__((always_inline)) {
        if constexpr (OPEN) {
            const int items = pa.items;
            constexpr int G = 4;                   // items of a thread in flight
#pragma nounroll
            for (int i0 = 0; i0 < items; i0 += G * nthr) {
                T now[G], next[G];
#pragma unroll
                for (int u = 0; u < G; ++u) now[u] = next[u] = T(0);
#pragma nounroll
                for (int q = 0; q < n_lor; ++q) {
                    T cur[G], prev[G];
                    const auto a_ = pq + (2 * q) * items;
                    const auto b_ = a_ + items;
#pragma unroll
                    for (int u = 0; u < G; ++u) {
                        const uint32_t i = min(i0 + u * nthr + tid, items - 1);
                        cur[u] = a_[i];
                        prev[u] = b_[i];
                    }
#pragma unroll
                    for (int u = 0; u < G; ++u) {
                        const uint32_t i = i0 + u * nthr + tid;
                        if (i < (uint32_t)items) {
                            const T* row = lor + prow[i] * (1 + 3 * n_lor);
                            const T nxt = fma(row[1 + 3 * q], cur[u], fma(-row[2 + 3 * q], prev[u], row[3 + 3 * q] * pol[i]));
                            now[u] += cur[u];
                            next[u] += nxt;
                            b_[i] = cur[u];
                            a_[i] = nxt;
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    const uint32_t i = i0 + u * nthr + tid;
                    if (i < (uint32_t)items) pol[i] = (next[u] - a_e * now[u]) * lor[prow[i] * (1 + 3 * n_lor)];
                }
            }
        }
    };

    auto cls = [&](int k, int grp) {
        return C4 ? (cw[k / CPW] >> (CB * (k % CPW))) & 15u : (cw[k / CPW] >> (CB * (k % CPW) + 8 * grp)) & 255u;
    };
    // the class words pass through an empty asm statement in every half step,
    // and rows through a scheduling barrier: otherwise the compiler keeps the
    // coefficients' addresses of every cell in registers across the steps, or
    // loads many rows' coefficients ahead, and spills
    auto half_h = [&](auto mode) __attribute__((always_inline)) {
        constexpr int MODE = decltype(mode)::value;
#pragma unroll
        for (int k = 0; k < NW; ++k) asm volatile("" : "+v"(cw[k]));
#pragma unroll
        for (int r = 0; r < B; ++r) {
            __builtin_amdgcn_sched_barrier(0);
            T ezR[NP], eyR[NP], ezC[NP][CX], ezU[NP][CX], exU[NP][CX];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                ez_row(p, r, ezC[p]);
                if (r + 1 < B) ez_row(p, r + 1, ezU[p]);
                eyR[p] = er[p * PE + OYC + r];
                if constexpr (LZ) ezR[p] = zr[r * CX];
                else ezR[p] = er[p * PE + OZC + r];
#pragma unroll
                for (int j = 0; j < CX; ++j) {
                    exU[p][j] = r + 1 < B ? e0[p][(r + 1) % B][j] : eu[p * PE + OEX + j];
                    if (r + 1 == B) {
                        if constexpr (LZ) ezU[p][j] = zu[j];
                        else ezU[p][j] = eu[p * PE + j];
                    }
                }
            }
            if constexpr (CPLX) {                  // across the Bloch-periodic edge
                const T z0 = ezR[0], z1 = ezR[1], q0 = eyR[0], q1 = eyR[1];
                ezR[0] = edge_r ? bloch_fwd(z0, z1, 0, ph_c, ph_s) : z0;
                ezR[1] = edge_r ? bloch_fwd(z1, z0, 1, ph_c, ph_s) : z1;
                eyR[0] = edge_r ? bloch_fwd(q0, q1, 0, ph_c, ph_s) : q0;
                eyR[1] = edge_r ? bloch_fwd(q1, q0, 1, ph_c, ph_s) : q1;
            }
            T rA, rB, rC, rD;
            if (CYL) {
                const T* rw = rows + kRowFactors * min(y0 + r, ny - 1);
                rA = rw[RA];
                rB = rw[RB];
                rC = rw[RC];
                rD = rw[RD];
            }
            const bool axis = CYL && r == 0 && y0 == 0;
            // undivided differences of cell j: d_x e_z, d_x e_y, d_y e_z, d_y e_x
            auto dxz = [&](int p, int j) { return (j + 1 < CX ? ezC[p][(j + 1) % CX] : ezR[p]) - ezC[p][j]; };
            auto dxy = [&](int p, int j) { return (j + 1 < CX ? e1[p][r][(j + 1) % CX] : eyR[p]) - e1[p][r][j]; };
            auto dyz = [&](int p, int j) { return ezU[p][j] - ezC[p][j]; };
            auto dyx = [&](int p, int j) { return exU[p][j] - e0[p][r][j]; };
            T sxz[CX], sxy[CX], syz[CX], syx[CX];  // stretched (open runs)
            if constexpr (OPEN) {
#pragma unroll
                for (int j = 0; j < CX; ++j) {
                    sxz[j] = dxz(0, j);
                    sxy[j] = dxy(0, j);
                    syz[j] = dyz(0, j);
                    syx[j] = dyx(0, j);
                }
                stretch(0, r, sxz, sxy, syz, syx);
            }
#pragma unroll
            for (int j = 0; j < CX; ++j) {
                const B3<T> b = HU ? hb : class_b<T>(tab_h, cls(r * CX + j, 0));
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const T ex = e0[p][r][j], ey = e1[p][r][j];
                    const T xz = OPEN ? sxz[j] : dxz(p, j), xy = OPEN ? sxy[j] : dxy(p, j);
                    const T yx = OPEN ? syx[j] : dyx(p, j);
                    T cz, cr;
                    if (CYL) {
                        cz = ((rA * ezU[p][j] - rB * ezC[p][j]) - M * ey) * rC;
                        cr = (M * ex) * rD - xz;
                        if (r == 0) cz = axis ? T(4) * ezU[p][j] : cz;   // h_z on the axis: the disk circulation
                    } else {
                        cz = (OPEN ? syz[j] : dyz(p, j)) - M * ey;
                        cr = M * ex - xz;
                    }
                    const T cp = xy - yx;
                    T &vx = h0[p][r][j], &vy = h1[p][r][j], &vz = h2[p][r][j];
                    upd_h<T, MODE>(vx, a_h, b.x, cz);
                    upd_h<T, MODE>(vy, a_h, b.y, cr);
                    upd_h<T, MODE>(vz, a_h, b.z, cp);
                    if (CYL && r == 0) {
                        // order 0 alone has h_z on the axis; h_r lies outside, h_phi is 0
                        vx = axis && M != T(0) ? T(0) : vx;
                        vy = axis ? T(0) : vy;
                        vz = axis ? T(0) : vz;
                    }
                    // computed here: between the branches of an open row the
                    // compiler would put the updates off to the last one
                    if constexpr (OPEN) asm volatile("" : "+v"(vx), "+v"(vy), "+v"(vz));
                }
            }
        }
    };
    auto half_e = [&](auto mode) __attribute__((always_inline)) {
        constexpr int MODE = decltype(mode)::value;
#pragma unroll
        for (int k = 0; k < NW; ++k) asm volatile("" : "+v"(cw[k]));
#pragma unroll
        for (int r = 0; r < B; ++r) {
            __builtin_amdgcn_sched_barrier(0);
            T hyL[NP], hzL[NP], hxD[NP][CX], hzD[NP][CX];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                hyL[p] = hl[p * PS + r];
                hzL[p] = hl[p * PS + B + r];
                if (r == 0)
#pragma unroll
                    for (int j = 0; j < CX; ++j) {
                        hxD[p][j] = hd[p * PS + j];
                        hzD[p][j] = hd[p * PS + CX + j];
                    }
            }
            if constexpr (CPLX) {
                const T q0 = hyL[0], q1 = hyL[1], z0 = hzL[0], z1 = hzL[1];
                hyL[0] = edge_l ? bloch_bwd(q0, q1, 0, ph_c, ph_s) : q0;
                hyL[1] = edge_l ? bloch_bwd(q1, q0, 1, ph_c, ph_s) : q1;
                hzL[0] = edge_l ? bloch_bwd(z0, z1, 0, ph_c, ph_s) : z0;
                hzL[1] = edge_l ? bloch_bwd(z1, z0, 1, ph_c, ph_s) : z1;
            }
            T rP, rQ, rC, rD;
            if (CYL) {
                const T* rw = rows + kRowFactors * min(y0 + r, ny - 1);
                rP = rw[RP];
                rQ = rw[RQ];
                rC = rw[RC];
                rD = rw[RD];
            }
            const bool axis = CYL && r == 0 && y0 == 0;
            // undivided differences of cell j: d_x h_z, d_x h_y, d_y h_z, d_y h_x
            auto dxz = [&](int p, int j) { return h2[p][r][j] - (j > 0 ? h2[p][r][(j + CX - 1) % CX] : hzL[p]); };
            auto dxy = [&](int p, int j) { return h1[p][r][j] - (j > 0 ? h1[p][r][(j + CX - 1) % CX] : hyL[p]); };
            auto hzd = [&](int p, int j) { return r > 0 ? h2[p][(r + B - 1) % B][j] : hzD[p][j]; };
            auto dyx = [&](int p, int j) {
                return h0[p][r][j] - (r > 0 ? h0[p][(r + B - 1) % B][j] : hxD[p][j]);
            };
            T sxz[CX], sxy[CX], syz[CX], syx[CX];
            if constexpr (OPEN) {
#pragma unroll
                for (int j = 0; j < CX; ++j) {
                    sxz[j] = dxz(0, j);
                    sxy[j] = dxy(0, j);
                    syz[j] = h2[0][r][j] - hzd(0, j);
                    syx[j] = dyx(0, j);
                }
                stretch(1, r, sxz, sxy, syz, syx);
            }
            T ezN[NP][CX];                         // E_z of the row, updated below
#pragma unroll
            for (int p = 0; p < NP; ++p)
                if constexpr (LZ) ez_row(p, r, ezN[p]);
#pragma unroll
            for (int j = 0; j < CX; ++j) {
                const B3<T> b = class_b<T>(tab_e, cls(r * CX + j, 1));
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const T hx = h0[p][r][j], hy = h1[p][r][j], hz = h2[p][r][j];
                    const T xz = OPEN ? sxz[j] : dxz(p, j), xy = OPEN ? sxy[j] : dxy(p, j);
                    const T yx = OPEN ? syx[j] : dyx(p, j);
                    T cz, cr;
                    if (CYL) {
                        cz = ((rP * hz - rQ * hzd(p, j)) + M * hy) * rD;
                        cr = -((M * hx) * rC) - xz;
                    } else {
                        cz = (OPEN ? syz[j] : hz - hzd(p, j)) + M * hy;
                        cr = -(M * hx) - xz;
                    }
                    const T cp = xy - yx;
                    T lx = T(0), ly = T(0), lz = T(0);
                    if constexpr (OPEN && MODE == 0)
                        if (any_l) {
                            if ((lmask >> (r * CX + j)) & 1u) {
                                const T* at = pol + 3 * (li + __popc(lmask & ((1u << (r * CX + j)) - 1u)));
                                lx = at[0];
                                ly = at[1];
                                lz = at[2];
                            }
                        }
                    T &vx = e0[p][r][j], &vy = e1[p][r][j], &vz = LZ ? ezN[p][j] : e2[LZ ? 0 : p][LZ ? 0 : r][j];
                    upd_e<T, MODE>(vx, a_e, b.x, cz);
                    upd_e<T, MODE>(vy, a_e, b.y, cr);
                    upd_e<T, MODE>(vz, a_e, b.z, cp);
                    if constexpr (OPEN && MODE == 0) {
                        vx -= lx;
                        vy -= ly;
                        vz -= lz;
                    }
                    if (CYL && r == 0) {           // e_z, e_phi outside, e_r kept at 0 on the axis
                        vx = axis ? T(0) : vx;
                        vy = axis ? T(0) : vy;
                        vz = axis ? T(0) : vz;
                    }
                    if constexpr (OPEN) asm volatile("" : "+v"(vx), "+v"(vy), "+v"(vz));
                    if constexpr (LZ) zme[r * CX + j] = vz;
                }
            }
        }
    };
    auto publish_e = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
#pragma unroll
            for (int j = 0; j < CX; ++j) {
                if constexpr (!LZ) xe[p * PE + j] = e2[p][0][j];
                xe[p * PE + OEX + j] = e0[p][0][j];
            }
#pragma unroll
            for (int r = 0; r < B; ++r) {
                if constexpr (!LZ) xe[p * PE + OZC + r] = e2[p][r][0];
                xe[p * PE + OYC + r] = e1[p][r][0];
            }
        }
    };
    auto publish_h = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
#pragma unroll
            for (int j = 0; j < CX; ++j) {
                xh[p * PS + j] = h0[p][B - 1][j];
                xh[p * PS + CX + j] = h2[p][B - 1][j];
            }
#pragma unroll
            for (int r = 0; r < B; ++r) {
                xh[p * PS + 2 * CX + r] = h1[p][r][CX - 1];
                xh[p * PS + 2 * CX + B + r] = h2[p][r][CX - 1];
            }
        }
    };

    // ---- the state at the first step: kick and start, or the fields in memory
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int r = 0; r < B; ++r)
#pragma unroll
            for (int j = 0; j < CX; ++j) {
                e0[p][r][j] = e1[p][r][j] = h0[p][r][j] = h1[p][r][j] = h2[p][r][j] = T(0);
                if constexpr (LZ) zme[r * CX + j] = T(0);
                else e2[p][r][j] = T(0);
            }
    if (s0 == 0) {
        const int src = (int)((d.src_off - d.field_off) / g.ncell);   // slot of the source component
        for (int k = tid; k < sbw * sbh; k += nthr) stage[k] = T(0);
        __syncthreads();
        for (int u = tid; u < d.n_uniq; u += nthr) {
            const int k0 = as_global(t.uoff)[d.u_off + u], k1 = as_global(t.uoff)[d.u_off + u + 1];
            double s = 0.0;
            for (int k = k0; k < k1; ++k)
                s += as_global(t.uw)[k] * as_global(t.basis)[d.basis_off + as_global(t.usamp)[k]];
            const int c = as_global(t.uidx)[d.u_off + u];
            stage[(c / nx - sy0) * sbw + (c % nx - sx0)] = T(d.kick_scale * s);
        }
        __syncthreads();
        const int base = (y0 - sy0) * sbw + (x0 - sx0);
#pragma unroll
        for (int r = 0; r < B; ++r)
#pragma unroll
            for (int j = 0; j < CX; ++j) {
                T v = T(0);
                if ((in_s >> (r * CX + j)) & 1u) v = stage[base + r * sbw + j];
                e0[0][r][j] = src == 0 ? v : T(0);
                e1[0][r][j] = src == 1 ? v : T(0);
                if constexpr (LZ) zme[r * CX + j] = src == 2 ? v : T(0);
                else e2[0][r][j] = src == 2 ? v : T(0);
                h0[0][r][j] = src == 3 ? v : T(0);
                h1[0][r][j] = src == 4 ? v : T(0);
                h2[0][r][j] = src == 5 ? v : T(0);
            }
        if (d.kind == 0) publish_e();
        else publish_h();
        load_y(d.kind, 0);
        __syncthreads();
        if (d.kind == 0) half_h(std::integral_constant<int, 1>{});
        else half_e(std::integral_constant<int, 1>{});
        if (OVERLAY) __syncthreads();
    } else {
        const auto F = as_global(fields + d.field_off);
        const int n = (int)g.ncell;
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int r = 0; r < B; ++r)
#pragma unroll
                for (int j = 0; j < CX; ++j)
                    if (act && x0 + j < nx && y0 + r < ny) {
                        const int c = p * 6 * n + (y0 + r) * nx + x0 + j;
                        e0[p][r][j] = F[c];
                        e1[p][r][j] = F[c + n];
                        if constexpr (LZ) zme[r * CX + j] = F[c + 2 * n];
                        else e2[p][r][j] = F[c + 2 * n];
                        h0[p][r][j] = F[c + 3 * n];
                        h1[p][r][j] = F[c + 4 * n];
                        h2[p][r][j] = F[c + 5 * n];
                    }
    }
    if (OVERLAY || s0 > 0 || d.kind == 1) publish_e();   // else the E kick's entries are there already
    share_e();
    load_y(0, 0);

    // ---- steps ----------------------------------------------------------
    // The measured component's cells inside its box go to the stage with the
    // half step's exchange values; after the barrier the block's last wave
    // forms the surface sum alone while the others go on.  The next write of
    // the stage lies behind the barrier after that.
    const bool meas_h = d.meas_slot >= 3;
    const int ms = d.meas_slot % 3;
    int mbase = (y0 - my0) * mbw + (x0 - mx0);
    uint32_t wave_m = 0;                           // cells some lane of the wave measures
#pragma unroll
    for (int k = 0; k < NC; ++k) wave_m |= __any((in_m >> k) & 1u) ? 1u << k : 0u;
    wave_m = __builtin_amdgcn_readfirstlane(wave_m);
    const bool has_m = wave_m != 0;
    const bool summing = tid >= nthr - 64;
    const int lane = tid & 63;
    const int nsamp = d.nsamp, P = d.P;
    if (summing && lane == 0) {
        s_acc[0] = acc[2 * slot];
        s_acc[1] = acc[2 * slot + 1];
    }
    auto put = [&](auto grp) __attribute__((always_inline)) {                     // 0: an H component, 1: an E component
        asm volatile("" : "+v"(in_m), "+v"(mbase));   // no masks or addresses kept across steps
#pragma unroll
        for (int r = 0; r < B; ++r)
#pragma unroll
            for (int j = 0; j < CX; ++j)
                if ((wave_m >> (r * CX + j)) & 1u) {
                    T a, b, c;
                    if constexpr (decltype(grp)::value == 0) {
                        a = h0[0][r][j];
                        b = h1[0][r][j];
                        c = h2[0][r][j];
                    } else {
                        a = e0[0][r][j];
                        b = e1[0][r][j];
                        if constexpr (LZ) c = zme[r * CX + j];
                        else c = e2[0][r][j];
                    }
                    if ((in_m >> (r * CX + j)) & 1u) stage[mbase + r * mbw + j] = ms == 0 ? a : ms == 1 ? b : c;
                }
    };
    auto measure = [&](int step) __attribute__((always_inline)) {
        const double kt = ktab[step];
        // partial v: the samples of the threads 64 v .. 64 v + 63 of the
        // block sum the other kernels take, added in the same order
        double total = 0.0;
#pragma nounroll
        for (int v = 0; v * 64 < min(nsamp, yee::kSurfThreads); ++v) {
            double s = 0.0;
#pragma nounroll
            for (int i = v * 64 + lane; i < nsamp; i += yee::kSurfThreads) {
                double x = 0.0;
#pragma nounroll
                for (int q = 0; q < P; ++q) x += sw[i * P + q] * (double)stage[so[i * P + q]];
                s += sb[i] * x;
            }
            s = yee::wave_total(s);
            total = v == 0 ? s : total + s;
        }
        if (lane == 0) {
            const double G = dA * total;
            double sum = s_acc[0], comp = s_acc[1];
            yee::neumaier(sum, comp, (dt * kt) * G);
            s_acc[0] = sum;
            s_acc[1] = comp;
            if (gamma) as_global(gamma)[(int64_t)step * gamma_stride + slot] = G;
        }
    };
    __syncthreads();
    for (int step = s0; step < s1; ++step) {
        polarize();
        half_h(std::integral_constant<int, 0>{});
        load_y(1, 0);
        if (OVERLAY) __syncthreads();
        publish_h();
        if (meas_h && has_m) put(std::integral_constant<int, 0>{});
        __syncthreads();
        if (meas_h && summing) measure(step);
        half_e(std::integral_constant<int, 0>{});
        load_y(0, 0);
        if (OVERLAY) __syncthreads();
        publish_e();
        share_e();
        if (!meas_h && has_m) put(std::integral_constant<int, 1>{});
        __syncthreads();
        if (!meas_h && summing) measure(step);
    }
    if (summing && lane == 0) {
        acc[2 * slot] = s_acc[0];
        acc[2 * slot + 1] = s_acc[1];
    }
    if (resume_later) {   // a later launch resumes from memory
        const auto F = as_global(fields + d.field_off);
        const int n = (int)g.ncell;
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int r = 0; r < B; ++r)
#pragma unroll
                for (int j = 0; j < CX; ++j)
                    if (act && x0 + j < nx && y0 + r < ny) {
                        const int c = p * 6 * n + (y0 + r) * nx + x0 + j;
                        F[c] = e0[p][r][j];
                        F[c + n] = e1[p][r][j];
                        if constexpr (LZ) F[c + 2 * n] = zme[r * CX + j];
                        else F[c + 2 * n] = e2[p][r][j];
                        F[c + 3 * n] = h0[p][r][j];
                        F[c + 4 * n] = h1[p][r][j];
                        F[c + 5 * n] = h2[p][r][j];
                    }
    }
}

// Patch shapes (columns, rows, waves per SIMD of the register budget, E_z in
// LDS).  The registers of a lane hold 6 (12 complex) values per cell of its
// patch and 50 to 90 more (class words, neighbour values, addresses); the step
// loop of none spills.
struct PatchShape {
    int cx, b, mw;
    bool lz;
    bool any;   // also built for grids of several H classes (HU = false)
};
template <typename T, bool CPLX, bool OPEN>
struct PatchShapes;
template <>
struct PatchShapes<float, false, false> {
    static constexpr int n = 7;
    static constexpr PatchShape s[n] = {{5, 5, 2, false, true}, {8, 3, 2, false, true}, {6, 4, 2, false, false},
                                        {4, 4, 3, false, true}, {5, 2, 4, false, true}, {3, 3, 4, false, false},
                                        {2, 2, 4, false, true}};
};
template <>
struct PatchShapes<double, false, false> {
    static constexpr int n = 7;
    static constexpr PatchShape s[n] = {{6, 3, 2, true, true},   {5, 3, 2, false, false}, {6, 2, 2, false, false},
                                        {4, 3, 2, false, true},  {4, 2, 3, false, false}, {3, 2, 3, false, true},
                                        {2, 2, 4, false, true}};
};
template <>
struct PatchShapes<float, true, false> {
    static constexpr int n = 6;
    static constexpr PatchShape s[n] = {{4, 3, 2, false, true},  {6, 2, 2, false, false}, {3, 3, 2, false, false},
                                        {4, 2, 3, false, false}, {3, 2, 3, false, true},  {2, 2, 4, false, true}};
};
template <>
struct PatchShapes<double, true, false> {
    static constexpr int n = 3;
    static constexpr PatchShape s[n] = {{3, 2, 2, false, true}, {2, 2, 2, false, true}, {2, 1, 4, false, true}};
};
template <>
struct PatchShapes<float, false, true> {
    static constexpr int n = 4;
    static constexpr PatchShape s[n] = {{5, 5, 2, true, true}, {4, 4, 2, false, true}, {3, 3, 3, false, false},
                                        {2, 2, 4, false, true}};
};
template <>
struct PatchShapes<double, false, true> {
    static constexpr int n = 3;
    static constexpr PatchShape s[n] = {{4, 3, 2, false, true}, {3, 2, 2, false, false}, {2, 2, 3, false, true}};
};

constexpr int kCUs = 256;

// one H class, and few enough E classes for a shape that packs them
inline bool patch_hu(const PatchClasses& pc, const PatchShape& q, bool open) {
    return pc.h_uniform && (pc.n[1] <= 16 || !patch_packs(q.lz, open));
}

struct PatchPlan {
    int shape = -1;
    PatchArgs args{};
    int threads = 0, blocks = 0;
    double cost = 0, cells = 0;                    // cells: of its patches, inside the grid
};

// Issue slots of a lane per step (the cost model's unit): the updates, the
// exchange, and the fixed part.
inline double patch_issue(const PatchShape& q, int np) {
    return np * ((q.lz ? 44.0 : 38.0) * q.cx * q.b + 10.0 * (q.cx + q.b)) + (q.lz ? 160.0 : 80.0);
}

// The open part of a launch: layer columns / rows of patches, sizes of the
// LDS entries, scratch values per block.
inline void plan_open(const PatchShape& q, const Grid2D& g, const PatchOpen& op, PatchArgs& a, OpenSizes& os) {
    auto split = [](int P, int n, int w, int L, int* lo, int* hi) {
        *lo = P > 0 ? std::min(L, (P + w - 1) / w) : 0;
        *hi = P > 0 ? std::max(*lo, (n - P) / w) : L;
    };
    split(g.pml[0], g.nx, q.cx, a.LX, &a.xlo, &a.xhi);
    split(g.pml[1], g.ny, q.b, a.LY, &a.ylo, &a.yhi);
    const int nc = q.cx * q.b;
    os.prof = 2 * (g.nx + g.ny);
    os.psi = (a.xlo + a.LX - a.xhi) * a.LY * ((4 * nc) | 1);
    a.scratch_stride = (int64_t)4 * nc * (a.ylo + a.LY - a.yhi) * a.LX;
    a.prof[0] = g.pml[0] > 0 ? g.pml_tab[0] : nullptr;
    a.prof[1] = g.pml[1] > 0 ? g.pml_tab[1] : nullptr;
    a.n_lor = op.n_lor;
    a.lor_rows = op.lor_rows;
    os.n_lor = op.n_lor;
    os.lor_rows = op.lor_rows;
    if (op.lor_rows > 1) {
        std::copy(&op.lor[0][0], &op.lor[0][0] + 4 * 13, &a.lor[0][0]);
        std::copy(&op.lrow[0][0], &op.lrow[0][0] + kPatchClasses * 3, &a.lrow[0][0]);
        int n = 0;   // dispersive cells
        for (int64_t k = 0; k < g.ncell; ++k) {
            const int c = op.cls[k] >> 8;
            n += (op.lrow[c][0] | op.lrow[c][1] | op.lrow[c][2]) != 0;
        }
        os.pol = 3 * n;
        a.items = 3 * n;
        a.scratch_stride += (int64_t)2 * op.n_lor * a.items;
    }
}

// The list (see PatchArgs) of the patches of cx x b cells with a cell that can
// change: E of a class that holds a field, H where an E value of its curl is of
// such a one.
inline std::vector<uint16_t> live_list(const uint16_t* cls, const Grid2D& g, bool pery, int cx, int b) {
    const int LX = (g.nx + cx - 1) / cx, LY = (g.ny + b - 1) / b;
    std::vector<int> at((size_t)LX * LY, -1);
    for (int y = 0; y < g.ny; ++y)
        for (int x = 0; x < g.nx; ++x) {
            if ((cls[(size_t)y * g.nx + x] >> 8) == 0) continue;
            const int xl = (x > 0 ? x - 1 : g.perx ? g.nx - 1 : x) / cx, yd = (y > 0 ? y - 1 : pery ? g.ny - 1 : y) / b;
            at[(y / b) * LX + x / cx] = at[(y / b) * LX + xl] = at[yd * LX + x / cx] = 0;
        }
    int n = 0;
    for (int& v : at)
        if (v == 0) v = n++;
    auto ref = [&](int i, int j) -> uint16_t {
        if (i < 0 || i >= LX) {
            if (!g.perx) return (uint16_t)n;
            i = (i + LX) % LX;
        }
        if (j < 0 || j >= LY) {
            if (!pery) return (uint16_t)n;
            j = (j + LY) % LY;
        }
        return (uint16_t)(at[j * LX + i] < 0 ? n : at[j * LX + i]);
    };
    std::vector<uint16_t> out;
    for (int j = 0; j < LY; ++j)
        for (int i = 0; i < LX; ++i)
            if (at[j * LX + i] >= 0)
                for (uint16_t v : {(uint16_t)i, (uint16_t)j, ref(i + 1, j), ref(i - 1, j), ref(i, j + 1), ref(i, j - 1)})
                    out.push_back(v);
    return out;
}

// The shape that takes the least modelled time for nslots channels on an
// nx x ny grid: steps of a CU's resident blocks at the waves its fullest SIMD
// holds, times the rounds of blocks.  shape -1 when none covers the grid.
// live: the list of the best shape lands in `list` (empty: every patch).
template <typename T, bool CPLX, bool OPEN>
PatchPlan plan_patch(bool cyl, const Grid2D& g, int nslots, const PatchClasses& pc, const PatchSizes& z,
                     const PatchOpen* op, size_t lds_cap, const PatchLive* live, std::vector<uint16_t>& list) {
    using SH = PatchShapes<T, CPLX, OPEN>;
    constexpr int np = CPLX ? 2 : 1;
    PatchPlan best;
    for (int k = 0; k < SH::n; ++k) {
        const PatchShape& q = SH::s[k];
        if (!q.any && !patch_hu(pc, q, OPEN)) continue;
        // a periodic axis wraps at a patch edge
        if ((g.perx && g.nx % q.cx) || (!cyl && g.pery && g.ny % q.b)) continue;
        PatchArgs a{};
        a.LX = (g.nx + q.cx - 1) / q.cx;
        a.LY = (g.ny + q.b - 1) / q.b;
        int64_t need = (int64_t)a.LX * a.LY;
        std::vector<uint16_t> l;
        if (live && need <= 4 * 1024) l = live_list(live->cls, g, !cyl && g.pery, q.cx, q.b);
        // without room for it, or with nothing to leave out, no list
        if (l.size() * sizeof(l[0]) > (live ? live->room : 0) || (int64_t)l.size() == 6 * need) l.clear();
        if (!l.empty()) need = (int64_t)l.size() / 6;
        if (need > 256 * q.mw || need > 1024) continue;
        a.np = (int)need;
        const int threads = (int)((need + 63) / 64) * 64, waves = threads / 64;
        OpenSizes os;
        if (OPEN) plan_open(q, g, *op, a, os);
        a.lds = patch_lds((int)need, patch_stride(q.cx, q.b, np), q.lz ? patch_zs(q.cx, q.b) : 0, q.lz, (int)sizeof(T), pc.n[0], pc.n[1], cyl ? g.ny : 0, z, os);
        const size_t lds = a.lds.total + 128;      // and the static part
        if (lds > lds_cap) continue;
        const int fit = std::max(1, std::min({4 * q.mw / waves, (int)(lds_cap / lds), (nslots + kCUs - 1) / kCUs}));
        int blocks = OPEN ? std::min(nslots, kCUs * fit) : nslots;
        if (OPEN && a.scratch_stride > 0)
            blocks = (int)std::min<int64_t>(blocks, op->scratch_bytes / (a.scratch_stride * (int64_t)sizeof(T)));
        if (blocks < 1) continue;
        const int at_once = std::min(blocks, kCUs * fit);
        const int rounds = (nslots + at_once - 1) / at_once;
        const double per_simd = (fit * waves + 3) / 4;
        const double cost = rounds * (per_simd * patch_issue(q, np) + 150.0);
        if (best.shape < 0 || cost < best.cost) {
            best.shape = k;
            best.args = a;
            best.threads = threads;
            best.blocks = blocks;
            best.cost = cost;
            list = std::move(l);
        }
    }
    if (best.shape >= 0) {
        const PatchShape& q = SH::s[best.shape];
        best.cells = list.empty() ? (double)g.ncell : 0;
        for (size_t k = 0; k < list.size(); k += 6)
            best.cells += (double)std::min(q.cx, g.nx - list[k] * q.cx) * std::min(q.b, g.ny - list[k + 1] * q.b);
    }
    return best;
}

template <typename T, bool CYL, bool CPLX, bool OPEN>
hipError_t patch_dispatch(T* fields, const ChanDev* ch, const int* slots, int nslots, const Grid2D& g,
                          const RedOrders& ord, const RedSpan& sp, const SurfTables& t, const PatchClasses& pc,
                          const PatchSizes& z, const PatchOpen* op, PatchLive* live, double dA, double* acc,
                          double* gamma, int gamma_stride, hipStream_t s, PatchRan* ran) {
    using SH = PatchShapes<T, CPLX, OPEN>;
    hipError_t e = hipSuccess;
    PatchPlan pl;
    if (!OPEN && live && live->plan_slots == nslots) {
        pl = *static_cast<const PatchPlan*>(live->plan.get());
    } else {
        std::vector<uint16_t> list;
        pl = plan_patch<T, CPLX, OPEN>(CYL, g, nslots, pc, z, op, device_lds_limit(), OPEN ? nullptr : live, list);
        if (OPEN) pl.args.scratch = op->scratch;
        if (!list.empty()) {
            live->keep->push_back(std::move(list));
            const std::vector<uint16_t>& l = live->keep->back();
            pl.args.list = reinterpret_cast<const uint16_t*>(live->dev);
            e = hipMemcpyAsync(live->dev, l.data(), l.size() * sizeof(l[0]), hipMemcpyHostToDevice, s);
            if (e != hipSuccess) return e;
        }
        if (!OPEN && live) {
            live->plan = std::make_shared<PatchPlan>(pl);
            live->plan_slots = nslots;
        }
    }
    if (pl.shape < 0) return hipSuccess;
    auto attempt = [&](auto v) {
        constexpr int V = decltype(v)::value;
        if constexpr (V < SH::n) {
            constexpr PatchShape q = SH::s[V];
            if (V != pl.shape) return;
            const auto run = [&](auto kernel) {
                if (!lds_allow(reinterpret_cast<const void*>(kernel), pl.args.lds.total)) return;
                ran->launched = true;
                ran->cells = pl.cells;
                // an open run's launches take as many channels as there are scratch regions
                for (int first = 0; first < nslots && e == hipSuccess; first += pl.blocks) {
                    hipLaunchKernelGGL(kernel, dim3(std::min(pl.blocks, nslots - first)), dim3(pl.threads),
                                       pl.args.lds.total, s, fields, ch, slots, first, nslots, g, ord, sp, t, pc,
                                       pl.args, dA, acc, gamma, gamma_stride);
                    e = hipGetLastError();
                }
            };
            if (patch_hu(pc, q, OPEN)) run(&k_red_patch<T, q.cx, q.b, CYL, CPLX, q.mw, q.lz, OPEN, true>);
            else if constexpr (q.any) run(&k_red_patch<T, q.cx, q.b, CYL, CPLX, q.mw, q.lz, OPEN, false>);
        }
    };
    attempt(std::integral_constant<int, 0>{});
    attempt(std::integral_constant<int, 1>{});
    attempt(std::integral_constant<int, 2>{});
    attempt(std::integral_constant<int, 3>{});
    attempt(std::integral_constant<int, 4>{});
    attempt(std::integral_constant<int, 5>{});
    attempt(std::integral_constant<int, 6>{});
    static_assert(SH::n <= 7, "one attempt per shape");
    return e;
}

}  // namespace

template <typename T>
hipError_t launch_red_patch(T* fields, const ChanDev* ch, const int* slots, int nslots, const Grid2D& g,
                            const RedOrders& ord, const RedSpan& span, const SurfTables& t, const PatchClasses& pc,
                            const PatchSizes& ps, const PatchOpen* op, PatchLive* live, double dA, double* acc,
                            double* gamma, int gamma_stride, hipStream_t s, PatchRan* ran) {
    *ran = PatchRan();
    if (nslots <= 0 || pc.cls == nullptr) return hipSuccess;
    if (op) {
        if (ord.axis || ord.cplx) return hipSuccess;
        return patch_dispatch<T, false, false, true>(fields, ch, slots, nslots, g, ord, span, t, pc, ps, op, live, dA, acc,
                                                     gamma, gamma_stride, s, ran);
    }
    if (ord.axis)
        return patch_dispatch<T, true, false, false>(fields, ch, slots, nslots, g, ord, span, t, pc, ps, op, live, dA, acc,
                                                     gamma, gamma_stride, s, ran);
    if (ord.cplx)
        return patch_dispatch<T, false, true, false>(fields, ch, slots, nslots, g, ord, span, t, pc, ps, op, live, dA, acc,
                                                     gamma, gamma_stride, s, ran);
    return patch_dispatch<T, false, false, false>(fields, ch, slots, nslots, g, ord, span, t, pc, ps, op, live, dA, acc,
                                                  gamma, gamma_stride, s, ran);
}

}  // namespace cf
