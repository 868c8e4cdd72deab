// Patch kernel of the reduced two-dimensional problems (cylindrical orders,
// k_z points, Bloch-periodic x): one block carries one channel through clear,
// kick, start and all its steps in a single launch, with every field value in
// a register.
//
// A thread owns a patch of CX x B cells (columns x rows); LX x LY threads
// cover the grid.  Inside the patch a neighbour is a register; the patch's
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
// steps, FP32): 56.5 -> 17.3 ms on the device; Bloch grating (48 x 60, 4096
// complex channels, 2000 steps, FP32): 177.7 -> 62.0 ms.
#include <algorithm>
#include <mutex>
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
    int xe, xh;    // exchange entries of E and H: threads + 1 (the zero entry) of S values
    int rows;      // row factors (cylindrical)
    int stage;     // measured (and at the start the kicked) component inside its box
    int so;        // surface point offsets into the stage
    int total;
};
__host__ __device__ inline PatchLds patch_lds(int nt, int S, int tsz, int n_h, int n_e, int n_rows,
                                              const PatchSizes& z) {
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
    l.xe = take((nt + 1) * S * tsz);
    l.xh = take((nt + 1) * S * tsz);
    l.rows = take(n_rows * kRowFactors * tsz);
    l.stage = take(z.box * tsz);
    l.so = take(z.samples * z.points * 2);
    l.total = at;
    return l;
}

constexpr int patch_stride(int CX, int B, int NP) { return (2 * (CX + B) * NP) | 1; }

struct PatchArgs {
    int LX, LY;
    PatchLds lds;
};

// s of lane l plus s of lane l + off for off = 32 .. 1, as
// yee::wave_partial_store orders it: the wave's sum in lane 0.
template <int N>
__device__ __forceinline__ double row_shl(double v) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    return __hiloint2double(__builtin_amdgcn_mov_dpp(hi, 0x100 | N, 0xf, 0xf, true),
                            __builtin_amdgcn_mov_dpp(lo, 0x100 | N, 0xf, 0xf, true));
}
__device__ __forceinline__ double wave_total(double s) {
    s += __shfl_down(s, 32, 64);
    s += __shfl_down(s, 16, 64);
    s += row_shl<8>(s);
    s += row_shl<4>(s);
    s += row_shl<2>(s);
    s += row_shl<1>(s);
    return s;
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

template <typename T, int MODE>
__device__ __forceinline__ T upd_h(T a, T x, T b, T d) {
    return MODE == 0 ? yee::sub(a, x, b, d) : yee::half(b, d);
}
template <typename T, int MODE>
__device__ __forceinline__ T upd_e(T a, T x, T b, T d) {
    return MODE == 0 ? yee::add(a, x, b, d) : yee::half(b, d);
}

// MW: waves per SIMD the register budget is sized for (the launch keeps the
// block within 4 MW waves).
template <typename T, int CX, int B, bool CYL, bool CPLX, int MW>
__global__ __launch_bounds__(256 * MW) __attribute__((amdgpu_waves_per_eu(MW)))
void k_red_patch(T* __restrict__ fields, const ChanDev* __restrict__ ch, const int* __restrict__ slots, int nslots,
                 Grid2D g, RedOrders ord, RedSpan sp, SurfTables t, PatchClasses pc, PatchArgs pa, double dA,
                 double* __restrict__ acc, double* __restrict__ gamma, int gamma_stride) {
    constexpr int NP = CPLX ? 2 : 1;
    constexpr int S = patch_stride(CX, B, NP);
    constexpr int PS = 2 * (CX + B);               // values of one part in an entry
    constexpr int NC = CX * B;
    static_assert(NC <= 32, "one mask bit per cell of the patch");
    extern __shared__ __align__(16) char lds[];
    __shared__ int s_box[8];                       // source box (min x, min y, max x, max y), measured box
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int LX = pa.LX, LY = pa.LY;
    // orders are listed from the first; a cylindrical launch takes the last
    // (longest) ones first
    const int slot = slots[CYL ? nslots - 1 - (int)blockIdx.x : (int)blockIdx.x];
    const ChanDev d = ch[slot];
    const int m = d.order;
    const int s0 = sp.s0[m], s1 = sp.s1[m];
    const bool resume_later = s1 < ord.steps[m];
    const double dt = ord.dt[m];
    const auto ktab = as_global(ord.ktab + m * ord.ktab_stride);
    const int nx = g.nx, ny = g.ny;
    const bool act = tid < LX * LY;
    const int tx = tid % LX, ty = tid / LX;
    const int x0 = tx * CX, y0 = ty * B;

    T* const XE = reinterpret_cast<T*>(lds + pa.lds.xe);
    T* const XH = reinterpret_cast<T*>(lds + pa.lds.xh);
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
        for (int k = tid; k < S; k += nthr) XE[nthr * S + k] = XH[nthr * S + k] = T(0);
        if (tid < 8) s_box[tid] = (tid & 2) ? -1 : 0x7fffffff;
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
    uint32_t cw[(NC + 1) / 2];
    uint32_t in_m = 0;                             // cells inside the measured component's box
    const int sx0 = s_box[0], sy0 = s_box[1], sbw = s_box[2] - sx0 + 1, sbh = s_box[3] - sy0 + 1;
    uint32_t in_s = 0;                             // cells inside the source's box
#pragma unroll
    for (int k = 0; k < (NC + 1) / 2; ++k) cw[k] = 0;
#pragma unroll
    for (int r = 0; r < B; ++r)
#pragma unroll
        for (int j = 0; j < CX; ++j) {
            const int k = r * CX + j, x = x0 + j, y = y0 + r;
            if (act && x < nx && y < ny) {
                cw[k >> 1] |= (uint32_t)as_global(pc.cls)[y * nx + x] << (16 * (k & 1));
                if (x >= mx0 && x <= s_box[6] && y >= my0 && y <= s_box[7]) in_m |= 1u << k;
                if (x >= sx0 && x <= s_box[2] && y >= sy0 && y <= s_box[3]) in_s |= 1u << k;
            }
        }
    const int zero = nthr;
    const int n_r = !act ? zero : tx + 1 < LX ? tid + 1 : g.perx ? tid + 1 - LX : zero;
    const int n_l = !act ? zero : tx > 0 ? tid - 1 : g.perx ? tid + LX - 1 : zero;
    const int n_u = !act ? zero : ty + 1 < LY ? tid + LX : !CYL && g.pery ? tx : zero;
    const int n_d = !act ? zero : ty > 0 ? tid - LX : !CYL && g.pery ? tx + (LY - 1) * LX : zero;
    const T* const er = XE + n_r * S + 2 * CX;     // Ez, Ey columns of the thread to the right
    const T* const eu = XE + n_u * S;              // Ez, Ex rows of the thread above
    const T* const hl = XH + n_l * S + 2 * CX;     // Hy, Hz columns of the thread to the left
    const T* const hd = XH + n_d * S;              // Hx, Hz rows of the thread below
    T* const xe = XE + tid * S;
    T* const xh = XH + tid * S;
    const bool edge_r = CPLX && tx + 1 == LX, edge_l = CPLX && tx == 0;
    const T M = T(ord.coup[m]), la = T(ord.la[m]);
    const T a_e = d.kind == 0 ? la : T(1), a_h = d.kind == 0 ? T(1) : la;
    const T ph_c = CPLX ? T(ord.ph_c[m]) : T(1), ph_s = CPLX ? T(ord.ph_s[m]) : T(0);
    const char* const tab_h = lds + pa.lds.tab[0];
    const char* const tab_e = lds + pa.lds.tab[1];

    T e0[NP][B][CX], e1[NP][B][CX], e2[NP][B][CX], h0[NP][B][CX], h1[NP][B][CX], h2[NP][B][CX];

    auto cls = [&](int k, int grp) { return (cw[k >> 1] >> (16 * (k & 1) + 8 * grp)) & 255u; };
    // the class words pass through an empty asm statement in every half step,
    // and rows through a scheduling barrier: otherwise the compiler keeps the
    // coefficients' addresses of every cell in registers across the steps, or
    // loads many rows' coefficients ahead, and spills
    auto half_h = [&](auto mode) {
        constexpr int MODE = decltype(mode)::value;
#pragma unroll
        for (int k = 0; k < (NC + 1) / 2; ++k) asm volatile("" : "+v"(cw[k]));
#pragma unroll
        for (int r = 0; r < B; ++r) {
            __builtin_amdgcn_sched_barrier(0);
            T ezR[NP], eyR[NP], ezU[NP][CX], exU[NP][CX];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                ezR[p] = er[p * PS + r];
                eyR[p] = er[p * PS + B + r];
                if (r + 1 == B)
#pragma unroll
                    for (int j = 0; j < CX; ++j) {
                        ezU[p][j] = eu[p * PS + j];
                        exU[p][j] = eu[p * PS + CX + j];
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
#pragma unroll
            for (int j = 0; j < CX; ++j) {
                const B3<T> b = class_b<T>(tab_h, cls(r * CX + j, 0));
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const T ex = e0[p][r][j], ey = e1[p][r][j], ez = e2[p][r][j];
                    const T ezu = r + 1 < B ? e2[p][(r + 1) % B][j] : ezU[p][j];
                    const T exu = r + 1 < B ? e0[p][(r + 1) % B][j] : exU[p][j];
                    const T ezr = j + 1 < CX ? e2[p][r][(j + 1) % CX] : ezR[p];
                    const T eyr = j + 1 < CX ? e1[p][r][(j + 1) % CX] : eyR[p];
                    T cz, cr;
                    if (CYL) {
                        cz = ((rA * ezu - rB * ez) - M * ey) * rC;
                        cr = (M * ex) * rD - (ezr - ez);
                        if (r == 0) cz = axis ? T(4) * ezu : cz;   // h_z on the axis: the disk circulation
                    } else {
                        cz = (ezu - ez) - M * ey;
                        cr = M * ex - (ezr - ez);
                    }
                    const T cp = (eyr - ey) - (exu - ex);
                    T vx = upd_h<T, MODE>(a_h, h0[p][r][j], b.x, cz);
                    T vy = upd_h<T, MODE>(a_h, h1[p][r][j], b.y, cr);
                    T vz = upd_h<T, MODE>(a_h, h2[p][r][j], b.z, cp);
                    if (CYL && r == 0) {
                        // order 0 alone has h_z on the axis; h_r lies outside, h_phi is 0
                        vx = axis && M != T(0) ? T(0) : vx;
                        vy = axis ? T(0) : vy;
                        vz = axis ? T(0) : vz;
                    }
                    h0[p][r][j] = vx;
                    h1[p][r][j] = vy;
                    h2[p][r][j] = vz;
                }
            }
        }
    };
    auto half_e = [&](auto mode) {
        constexpr int MODE = decltype(mode)::value;
#pragma unroll
        for (int k = 0; k < (NC + 1) / 2; ++k) asm volatile("" : "+v"(cw[k]));
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
#pragma unroll
            for (int j = 0; j < CX; ++j) {
                const B3<T> b = class_b<T>(tab_e, cls(r * CX + j, 1));
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const T hx = h0[p][r][j], hy = h1[p][r][j], hz = h2[p][r][j];
                    const T hxd = r > 0 ? h0[p][(r + B - 1) % B][j] : hxD[p][j];
                    const T hzd = r > 0 ? h2[p][(r + B - 1) % B][j] : hzD[p][j];
                    const T hyl = j > 0 ? h1[p][r][(j + CX - 1) % CX] : hyL[p];
                    const T hzl = j > 0 ? h2[p][r][(j + CX - 1) % CX] : hzL[p];
                    T cz, cr;
                    if (CYL) {
                        cz = ((rP * hz - rQ * hzd) + M * hy) * rD;
                        cr = -((M * hx) * rC) - (hz - hzl);
                    } else {
                        cz = (hz - hzd) + M * hy;
                        cr = -(M * hx) - (hz - hzl);
                    }
                    const T cp = (hy - hyl) - (hx - hxd);
                    T vx = upd_e<T, MODE>(a_e, e0[p][r][j], b.x, cz);
                    T vy = upd_e<T, MODE>(a_e, e1[p][r][j], b.y, cr);
                    T vz = upd_e<T, MODE>(a_e, e2[p][r][j], b.z, cp);
                    if (CYL && r == 0) {           // e_z, e_phi outside, e_r kept at 0 on the axis
                        vx = axis ? T(0) : vx;
                        vy = axis ? T(0) : vy;
                        vz = axis ? T(0) : vz;
                    }
                    e0[p][r][j] = vx;
                    e1[p][r][j] = vy;
                    e2[p][r][j] = vz;
                }
            }
        }
    };
    auto publish_e = [&]() {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
#pragma unroll
            for (int j = 0; j < CX; ++j) {
                xe[p * PS + j] = e2[p][0][j];
                xe[p * PS + CX + j] = e0[p][0][j];
            }
#pragma unroll
            for (int r = 0; r < B; ++r) {
                xe[p * PS + 2 * CX + r] = e2[p][r][0];
                xe[p * PS + 2 * CX + B + r] = e1[p][r][0];
            }
        }
    };
    auto publish_h = [&]() {
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
            for (int j = 0; j < CX; ++j)
                e0[p][r][j] = e1[p][r][j] = e2[p][r][j] = h0[p][r][j] = h1[p][r][j] = h2[p][r][j] = T(0);
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
                e2[0][r][j] = src == 2 ? v : T(0);
                h0[0][r][j] = src == 3 ? v : T(0);
                h1[0][r][j] = src == 4 ? v : T(0);
                h2[0][r][j] = src == 5 ? v : T(0);
            }
        if (d.kind == 0) publish_e();
        else publish_h();
        __syncthreads();
        if (d.kind == 0) half_h(std::integral_constant<int, 1>{});
        else half_e(std::integral_constant<int, 1>{});
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
                        e2[p][r][j] = F[c + 2 * n];
                        h0[p][r][j] = F[c + 3 * n];
                        h1[p][r][j] = F[c + 4 * n];
                        h2[p][r][j] = F[c + 5 * n];
                    }
    }
    if (s0 > 0 || d.kind == 1) publish_e();   // an E kick's entries are there already

    // ---- steps ----------------------------------------------------------
    // The measured component's cells inside its box go to the stage with the
    // half step's exchange values; after the barrier the block's last wave
    // forms the surface sum alone while the others go on.  The next write of
    // the stage lies behind the barrier after that.
    const bool meas_h = d.meas_slot >= 3;
    const int ms = d.meas_slot % 3;
    int mbase = (y0 - my0) * mbw + (x0 - mx0);
    const bool has_m = __any(in_m != 0);
    const bool summing = tid >= nthr - 64;
    const int lane = tid & 63;
    const int nsamp = d.nsamp, P = d.P;
    double sum = 0.0, comp = 0.0, kt = 0.0;
    if (summing && lane == 0) {
        sum = acc[2 * slot];
        comp = acc[2 * slot + 1];
    }
    auto put = [&](const T (&f)[B][CX]) {
        asm volatile("" : "+v"(in_m), "+v"(mbase));   // no masks or addresses kept across steps
#pragma unroll
        for (int r = 0; r < B; ++r)
#pragma unroll
            for (int j = 0; j < CX; ++j)
                if ((in_m >> (r * CX + j)) & 1u) stage[mbase + r * mbw + j] = f[r][j];
    };
    auto measure = [&](int step) {
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
            s = wave_total(s);
            total = v == 0 ? s : total + s;
        }
        if (lane == 0) {
            const double G = dA * total;
            yee::neumaier(sum, comp, (dt * kt) * G);
            if (gamma) as_global(gamma)[(int64_t)step * gamma_stride + slot] = G;
        }
    };
    __syncthreads();
    for (int step = s0; step < s1; ++step) {
        if (summing) kt = ktab[step];
        half_h(std::integral_constant<int, 0>{});
        publish_h();
        if (meas_h && has_m) {
            if (ms == 0) put(h0[0]);
            else if (ms == 1) put(h1[0]);
            else put(h2[0]);
        }
        __syncthreads();
        if (meas_h && summing) measure(step);
        half_e(std::integral_constant<int, 0>{});
        publish_e();
        if (!meas_h && has_m) {
            if (ms == 0) put(e0[0]);
            else if (ms == 1) put(e1[0]);
            else put(e2[0]);
        }
        __syncthreads();
        if (!meas_h && summing) measure(step);
    }
    if (summing && lane == 0) {
        acc[2 * slot] = sum;
        acc[2 * slot + 1] = comp;
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
                        F[c + 2 * n] = e2[p][r][j];
                        F[c + 3 * n] = h0[p][r][j];
                        F[c + 4 * n] = h1[p][r][j];
                        F[c + 5 * n] = h2[p][r][j];
                    }
    }
}

// Patch shapes (columns, rows, waves per SIMD of the register budget).  The
// registers of a lane hold 6 (12 complex) values per cell of its patch and
// about 50 more (class words, neighbour values, addresses); none spills.
struct PatchShape {
    int cx, b, mw;
};
template <typename T, bool CPLX>
struct PatchShapes;
template <>
struct PatchShapes<float, false> {
    static constexpr int n = 7;
    static constexpr PatchShape s[n] = {{5, 5, 2}, {8, 3, 2}, {6, 4, 2}, {4, 4, 3}, {5, 2, 4}, {3, 3, 4}, {2, 2, 4}};
};
template <>
struct PatchShapes<double, false> {
    static constexpr int n = 6;
    static constexpr PatchShape s[n] = {{5, 3, 2}, {6, 2, 2}, {4, 3, 2}, {4, 2, 3}, {3, 2, 3}, {2, 2, 4}};
};
template <>
struct PatchShapes<float, true> {
    static constexpr int n = 6;
    static constexpr PatchShape s[n] = {{4, 3, 2}, {6, 2, 2}, {3, 3, 2}, {4, 2, 3}, {3, 2, 3}, {2, 2, 4}};
};
template <>
struct PatchShapes<double, true> {
    static constexpr int n = 3;
    static constexpr PatchShape s[n] = {{3, 2, 2}, {2, 2, 2}, {2, 1, 4}};
};

constexpr int kCUs = 256;

struct PatchPlan {
    int shape = -1;
    PatchArgs args{};
    int threads = 0;
    double cost = 0;
};

// Issue slots of a lane per step (the cost model's unit): the updates, the
// exchange, and the fixed part.
inline double patch_issue(const PatchShape& q, int np) {
    return np * (38.0 * q.cx * q.b + 10.0 * (q.cx + q.b)) + 80.0;
}

// The shape that takes the least modelled time for nslots channels on an
// nx x ny grid: steps of a CU's resident blocks at the waves its fullest SIMD
// holds, times the rounds of blocks.  shape -1 when none covers the grid.
template <typename T, bool CPLX>
PatchPlan plan_patch(bool cyl, const Grid2D& g, int nslots, const PatchClasses& pc, const PatchSizes& z, size_t lds_cap) {
    using SH = PatchShapes<T, CPLX>;
    constexpr int np = CPLX ? 2 : 1;
    PatchPlan best;
    for (int k = 0; k < SH::n; ++k) {
        const PatchShape& q = SH::s[k];
        // a periodic axis wraps at a patch edge
        if ((g.perx && g.nx % q.cx) || (!cyl && g.pery && g.ny % q.b)) continue;
        const int LX = (g.nx + q.cx - 1) / q.cx, LY = (g.ny + q.b - 1) / q.b;
        const int64_t need = (int64_t)LX * LY;
        if (need > 256 * q.mw || need > 1024) continue;
        const int threads = (int)((need + 63) / 64) * 64, waves = threads / 64;
        const PatchLds l = patch_lds(threads, patch_stride(q.cx, q.b, np), (int)sizeof(T), pc.n[0], pc.n[1],
                                     cyl ? g.ny : 0, z);
        if ((size_t)l.total + 128 > lds_cap) continue;
        const int fit = std::max(1, std::min({4 * q.mw / waves, (int)(lds_cap / (l.total + 128)),
                                              (nslots + kCUs - 1) / kCUs}));
        const int rounds = (nslots + kCUs * fit - 1) / (kCUs * fit);
        const double per_simd = (fit * waves + 3) / 4;
        const double cost = rounds * (per_simd * patch_issue(q, np) + 150.0);
        if (best.shape < 0 || cost < best.cost) {
            best.shape = k;
            best.args = PatchArgs{LX, LY, l};
            best.threads = threads;
            best.cost = cost;
        }
    }
    return best;
}

// Dynamic LDS above 64 KB needs the kernel's attribute raised first (a cap,
// only ever raised, under a lock); false when the runtime refuses.
template <typename T, int CX, int B, bool CYL, bool CPLX, int MW>
bool patch_lds_ok(size_t lds) {
    if (lds <= 65536) return true;
    static std::mutex mu;
    static size_t cap = 65536;
    std::lock_guard<std::mutex> lk(mu);
    if (lds <= cap) return true;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_red_patch<T, CX, B, CYL, CPLX, MW>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    cap = lds;
    return true;
}

template <typename T, bool CYL, bool CPLX>
hipError_t patch_dispatch(T* fields, const ChanDev* ch, const int* slots, int nslots, const Grid2D& g,
                          const RedOrders& ord, const RedSpan& sp, const SurfTables& t, const PatchClasses& pc,
                          const PatchSizes& z, double dA, double* acc, double* gamma, int gamma_stride, hipStream_t s,
                          bool* launched) {
    using SH = PatchShapes<T, CPLX>;
    const PatchPlan pl = plan_patch<T, CPLX>(CYL, g, nslots, pc, z, device_lds_limit());
    if (pl.shape < 0) return hipSuccess;
    hipError_t e = hipSuccess;
    auto attempt = [&](auto v) {
        constexpr int V = decltype(v)::value;
        if constexpr (V < SH::n) {
            constexpr PatchShape q = SH::s[V];
            if (V != pl.shape || !patch_lds_ok<T, q.cx, q.b, CYL, CPLX, q.mw>(pl.args.lds.total)) return;
            *launched = true;
            hipLaunchKernelGGL((k_red_patch<T, q.cx, q.b, CYL, CPLX, q.mw>), dim3(nslots), dim3(pl.threads),
                               pl.args.lds.total, s, fields, ch, slots, nslots, g, ord, sp, t, pc, pl.args, dA, acc,
                               gamma, gamma_stride);
            e = hipGetLastError();
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
                            const PatchSizes& ps, double dA, double* acc, double* gamma, int gamma_stride,
                            hipStream_t s, bool* launched) {
    *launched = false;
    if (nslots <= 0 || pc.cls == nullptr) return hipSuccess;
    if (ord.axis)
        return patch_dispatch<T, true, false>(fields, ch, slots, nslots, g, ord, span, t, pc, ps, dA, acc, gamma,
                                              gamma_stride, s, launched);
    if (ord.cplx)
        return patch_dispatch<T, false, true>(fields, ch, slots, nslots, g, ord, span, t, pc, ps, dA, acc, gamma,
                                              gamma_stride, s, launched);
    return patch_dispatch<T, false, false>(fields, ch, slots, nslots, g, ord, span, t, pc, ps, dA, acc, gamma,
                                           gamma_stride, s, launched);
}
template hipError_t launch_red_patch<float>(float*, const ChanDev*, const int*, int, const Grid2D&, const RedOrders&,
                                            const RedSpan&, const SurfTables&, const PatchClasses&, const PatchSizes&,
                                            double, double*, double*, int, hipStream_t, bool*);
template hipError_t launch_red_patch<double>(double*, const ChanDev*, const int*, int, const Grid2D&, const RedOrders&,
                                             const RedSpan&, const SurfTables&, const PatchClasses&,
                                             const PatchSizes&, double, double*, double*, int, hipStream_t, bool*);

}  // namespace cf
