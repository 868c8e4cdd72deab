// Patch kernel of the Cartesian 2D problems: one block advances one channel,
// every field value in a register.
#include <algorithm>
#include <type_traits>

#include "../../include/casimir_fdtd.h"
#include "lds.hpp"
#include "patch2d.hpp"
#include "yee_common.hpp"

namespace cf {

namespace {

using yee::as_global;

// Exchange entry of a patch: its edge row (CX values) and edge column (B
// values), whole 16-byte words of both first, then what remains of each.  The
// stride is an odd number of such words: the 16-byte accesses of consecutive
// threads then fall into different banks.  (As 4-byte accesses at a stride of 12
// values they kept the LDS busy for 60 % of the time, three quarters of it
// bank conflicts: 400 x 200 piston 37.4 -> 27.4 ms.)
template <typename T, int CX, int B>
struct P2Entry {
    static constexpr int V = 16 / (int)sizeof(T);
    static constexpr int row_full = CX / V * V, col_full = B / V * V;
    static constexpr int row = 0, col = row_full, row_rest = row_full + col_full, col_rest = row_rest + CX - row_full;
    static constexpr int words = (col_rest + B - col_full + V - 1) / V;
    static constexpr int stride = (words | 1) * V;
};

template <typename T, int C>
using P2Vec = T __attribute__((ext_vector_type(C)));
// Values I .. E - 1 of v from or to entry e at offset AT + I, in the widest
// accesses their alignment allows.
template <int C, typename T>
__device__ __forceinline__ void p2_get1(const T* e, T* v) {
    if constexpr (C == 1) {
        v[0] = e[0];
    } else {
        const P2Vec<T, C> x = *reinterpret_cast<const P2Vec<T, C>*>(__builtin_assume_aligned(e, C * sizeof(T)));
#pragma unroll
        for (int k = 0; k < C; ++k) v[k] = x[k];
    }
}
template <int C, typename T>
__device__ __forceinline__ void p2_put1(T* e, const T* v) {
    if constexpr (C == 1) {
        e[0] = v[0];
    } else {
        P2Vec<T, C> x;
#pragma unroll
        for (int k = 0; k < C; ++k) x[k] = v[k];
        *reinterpret_cast<P2Vec<T, C>*>(__builtin_assume_aligned(e, C * sizeof(T))) = x;
    }
}
template <int AT, int I, int E, bool PUT, typename T, int N>
__device__ __forceinline__ void p2_move(T* e, T (&v)[N]) {
    if constexpr (I < E) {
        constexpr int V = 16 / (int)sizeof(T), at = AT + I, left = E - I;
        constexpr int C = V >= 4 && left >= 4 && at % 4 == 0 ? 4 : left >= 2 && at % 2 == 0 ? 2 : 1;
        if constexpr (PUT) p2_put1<C>(e + at, v + I);
        else p2_get1<C>(e + at, v + I);
        p2_move<AT, I + C, E, PUT>(e, v);
    }
}
template <bool PUT, typename X, typename T, int N>
__device__ __forceinline__ void p2_row(T* e, T (&v)[N]) {
    p2_move<X::row, 0, X::row_full, PUT>(e, v);
    p2_move<X::row_rest - X::row_full, X::row_full, N, PUT>(e, v);
}
template <bool PUT, typename X, typename T, int N>
__device__ __forceinline__ void p2_col(T* e, T (&v)[N]) {
    p2_move<X::col, 0, X::col_full, PUT>(e, v);
    p2_move<X::col_rest - X::col_full, X::col_full, N, PUT>(e, v);
}

// Row of a patch in memory, in accesses of 16 bytes (aligned as its values are).
// With an access per value, CX values apart in neighbouring threads, every line
// was read and written several times over: a launch of 16 steps of 260 x 200
// cells in two parts (8 x 4 cells, 16 waves, FP32) took 114 us, 44 of them the
// steps; it takes 63.
template <int C, typename T>
using P2Mem = T __attribute__((ext_vector_type(C), aligned(sizeof(T))));
template <int I, typename P, typename T, int N>
__device__ __forceinline__ void p2_load_row(P p, T (&v)[N]) {
    if constexpr (I < N) {
        constexpr int left = N - I, V = 16 / (int)sizeof(T), C = V >= 4 && left >= 4 ? 4 : left >= 2 ? 2 : 1;
        const P2Mem<C, T> x = *reinterpret_cast<yee::gmem<const P2Mem<C, T>>>(p + I);
#pragma unroll
        for (int k = 0; k < C; ++k) v[I + k] = x[k];
        p2_load_row<I + C>(p, v);
    }
}
template <int I, typename P, typename T, int N>
__device__ __forceinline__ void p2_store_row(P p, const T (&v)[N]) {
    if constexpr (I < N) {
        constexpr int left = N - I, V = 16 / (int)sizeof(T), C = V >= 4 && left >= 4 ? 4 : left >= 2 ? 2 : 1;
        P2Mem<C, T> x;
#pragma unroll
        for (int k = 0; k < C; ++k) x[k] = v[I + k];
        *reinterpret_cast<yee::gmem<P2Mem<C, T>>>(p + I) = x;
        p2_store_row<I + C>(p, v);
    }
}

struct P2Lds {
    int xe, xh, stage, sw, sb, so, total;
};
// stride: values of an exchange entry
template <typename T>
P2Lds p2_lds(int stride, int n, const Patch2DSizes& z) {
    P2Lds l{};
    int off = 0;
    auto take = [&](size_t bytes) {
        const int at = off;
        off = (int)((off + bytes + 15) / 16 * 16);
        return at;
    };
    const size_t entries = (size_t)(n + 2) * stride * sizeof(T);   // + zeros, + a spare to write to
    l.xe = take(entries);
    l.xh = take(entries);
    l.stage = take((size_t)z.box * sizeof(T));
    l.sw = take((size_t)z.samples * z.points * 8);
    l.sb = take((size_t)z.samples * 8);
    l.so = take((size_t)z.samples * z.points * 2);
    l.total = off;
    return l;
}

// v where bit k of `bits` is set, else 0 (one bit-field extract and one and).
__device__ __forceinline__ float masked(float v, uint32_t bits, int k) {
    return __int_as_float(__float_as_int(v) & __builtin_amdgcn_sbfe((int)bits, k, 1));
}
__device__ __forceinline__ double masked(double v, uint32_t bits, int k) {
    const int m = __builtin_amdgcn_sbfe((int)bits, k, 1);
    return __hiloint2double(__double2hiint(v) & m, __double2loint(v) & m);
}

// v where bit k of `bits` is set, else w: an extract and a bit-field insert (as
// asm: the compiler makes a test and a conditional move of it, one more)
__device__ __forceinline__ int bfi(int m, int v, int w) {
    int r;
    asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "v"(m), "v"(v), "v"(w));
    return r;
}
__device__ __forceinline__ float selected(float v, float w, uint32_t bits, int k) {
    return __int_as_float(bfi(__builtin_amdgcn_sbfe((int)bits, k, 1), __float_as_int(v), __float_as_int(w)));
}
__device__ __forceinline__ double selected(double v, double w, uint32_t bits, int k) {
    const int m = __builtin_amdgcn_sbfe((int)bits, k, 1);
    return __hiloint2double(bfi(m, __double2hiint(v), __double2hiint(w)), bfi(m, __double2loint(v), __double2loint(w)));
}

// x <- a x - b d and x <- a x + b d, or (START) the consistent start's (b / 2) d
template <bool START, typename T>
__device__ __forceinline__ void p2_sub(T& x, T a, T b, T v) {
    if constexpr (START) x = yee::half(b, v);
    else yee::sub_into(x, a, b, v);
}
template <bool START, typename T>
__device__ __forceinline__ void p2_add(T& x, T a, T b, T v) {
    if constexpr (START) x = yee::half(b, v);
    else yee::add_into(x, a, b, v);
}

// One block advances one channel; thread k holds patch k of the channel's list,
// CX x B cells with every field value in registers, over all steps of the
// launch.  Only patches with a cell that can change are listed, so conductors
// cost nothing; a neighbour that is not listed holds 0 and is read from an
// entry of zeros.  Per half step a patch writes one edge row and one edge
// column to LDS and reads its neighbours' (E: bottom row and left column; H:
// top row and right column), with one barrier.
//
// Coefficients: b != 0 holds one a per field group (1, or the conductivity's
// factor), and where b = 0 the field is 0 whatever a is, so a is a scalar.
// Patch2DCoef says where b comes from.
//
// What bounds it: VALU issue (11 instructions per cell-update, 2 more per
// masked component) and the register file, which caps a channel's cells: 3
// to 6 values per cell of 512 KB.  The tiles (k_rb2d) compute 64 x 64 cells
// for 52 x 52, whole waves of conductor but not less, and reload everything
// every 6 steps.  400 x 200 piston (14000 live cells, 448 channels, 10000
// steps, FP32): 108.4 -> 27.4 ms on the device.  Small grids are bound by the
// latency of a step (two LDS exchanges, two barriers): 80 x 40 piston (1040
// live cells, FP64) 2.9 -> 0.5 us per step.  The surface sum has a wave of its
// own, a step behind the others, with the lane's offsets and weights in
// registers: read from LDS by an ordinary wave they took 0.9 us per step.
template <typename T, int POL, int CX, int B, int COEF>
__device__ __forceinline__ void p2_advance(const ChanDev& d, const InstDev& g, const Patch2DInst& hd, int part, int m0,
                                           int ksteps, int src, int dst, const P2Lds& l) {
    constexpr bool TM = POL == CF_POL_TM;
    constexpr int C0 = TM ? CF_EZ : CF_EX, C1 = TM ? CF_HX : CF_EY, C2 = TM ? CF_HY : CF_HZ;
    constexpr int NE = TM ? 1 : 2, NH = 3 - NE, NC = CX * B;
    using X = P2Entry<T, CX, B>;
    constexpr int S = X::stride;
    static_assert(NC <= 32, "one mask bit per cell of the patch");
    extern __shared__ __align__(16) char lds[];
    __shared__ int s_box[8];                       // box of the measured points (x0, y0, x1, y1), of the kicked ones
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const SurfTables& t = g.t;
    const int n = hd.n[TM ? 0 : 1];
    // small shapes: the block's own kick and consistent start at step 0; else the
    // fields are in memory
    const bool start = patch2d_small(NC, sizeof(T)) && hd.start != 0 && m0 == 0;
    const bool surf = part == hd.surf_part[TM ? 0 : 1];   // this block takes the surface sums
    const int nx = g.nx, ny = g.ny;
    const auto lk = as_global(static_cast<const T*>(g.lut)) + d.kind * 6 * 256 * 2;   // (a, b) of (comp, id)

    T* const XE = reinterpret_cast<T*>(lds + l.xe);
    T* const XH = reinterpret_cast<T*>(lds + l.xh);
    T* const stage = reinterpret_cast<T*>(lds + l.stage);
    double* const sw = reinterpret_cast<double*>(lds + l.sw);
    double* const sb = reinterpret_cast<double*>(lds + l.sb);
    uint16_t* const so = reinterpret_cast<uint16_t*>(lds + l.so);

    // ---- surface tables and the zero entries ---------------------------
    const int npt = surf ? d.nsamp * d.P : 0;
    if (tid < 8) s_box[tid] = (tid & 2) ? -1 : 0x7fffffff;
    for (int k = tid; k < S; k += nthr) XE[n * S + k] = XH[n * S + k] = T(0);
    __syncthreads();
    for (int k = tid; k < npt; k += nthr) {
        const int c = as_global(t.gidx)[d.g_off + k], i = c % nx, j = c / nx;
        atomicMin(&s_box[0], i);
        atomicMin(&s_box[1], j);
        atomicMax(&s_box[2], i);
        atomicMax(&s_box[3], j);
    }
    if (start)
        for (int u = tid; u < d.n_uniq; u += nthr) {
            const int c = as_global(t.uidx)[d.u_off + u], i = c % nx, j = c / nx;
            atomicMin(&s_box[4], i);
            atomicMin(&s_box[5], j);
            atomicMax(&s_box[6], i);
            atomicMax(&s_box[7], j);
        }
    __syncthreads();
    const int mx0 = s_box[0], my0 = s_box[1], mx1 = s_box[2], my1 = s_box[3], mbw = mx1 - mx0 + 1;
    for (int k = tid; k < npt; k += nthr) {
        const int c = as_global(t.gidx)[d.g_off + k];
        so[k] = (uint16_t)((c / nx - my0) * mbw + (c % nx - mx0));
        sw[k] = as_global(t.gw)[d.g_off + k];
    }
    for (int k = tid; k < d.nsamp; k += nthr) sb[k] = as_global(t.basis)[d.basis_off + k];

    // ---- the kick (as k_kick), in the stage array -------------------------
    const int kx0 = s_box[4], ky0 = s_box[5], kx1 = s_box[6], ky1 = s_box[7], kbw = kx1 - kx0 + 1;
    if (start) {
        for (int k = tid; k < kbw * (ky1 - ky0 + 1); k += nthr) stage[k] = T(0);
        __syncthreads();
        for (int u = tid; u < d.n_uniq; u += nthr) {
            const int k0 = as_global(t.uoff)[d.u_off + u], k1 = as_global(t.uoff)[d.u_off + u + 1];
            double v = 0.0;
            for (int k = k0; k < k1; ++k)
                v += as_global(t.uw)[k] * as_global(t.basis)[d.basis_off + as_global(t.usamp)[k]];
            const int c = as_global(t.uidx)[d.u_off + u];
            stage[(c / nx - ky0) * kbw + c % nx - kx0] = T(d.kick_scale * v);
        }
        __syncthreads();
    }

    if (wave == (nthr >> 6) - 1) {
        if (start) {                               // the barriers of the others' start
            __syncthreads();
            __syncthreads();
        }
        // ---- the block's last wave: surface sum and accumulation of every
        // step, while the others take the next one (the samples before their
        // H half, the total before their E half)
        if (!surf) {
            __syncthreads();
            for (int step = 0; step < ksteps; ++step) {
                __syncthreads();
                __syncthreads();
            }
            return;
        }
        const auto acc = as_global(g.acc + 2 * d.local);
        const auto ktab = as_global(g.ktab) + m0;
        const int nsamp = d.nsamp, P = d.P;
        double acc_s = acc[0], acc_c = acc[1];
        // partial v: the samples of the threads 64 v .. 64 v + 63 of the block
        // sum the other kernels take
        auto advance = [&](auto gather, auto& part) __attribute__((always_inline)) {
            auto total = [&](int step, double kt) __attribute__((always_inline)) {
                double sum = yee::wave_total(part[0]);
#pragma unroll
                for (int v = 1; v < (int)(sizeof(part) / sizeof(part[0])); ++v)
                    if (v * 64 < nsamp) sum += yee::wave_total(part[v]);
                const double G = g.dA * sum;
                yee::neumaier(acc_s, acc_c, (g.dt * kt) * G);
                if (lane == 0 && g.gamma) as_global(g.gamma)[(int64_t)(m0 + step) * g.gamma_stride + d.local] = G;
            };
            for (int step = 0; step < ksteps; ++step) {
                const double kt = ktab[max(step - 1, 0)];
                if (step > 0) gather();
                __syncthreads();
                if (step > 0) total(step - 1, kt);
                __syncthreads();
            }
            const double kt = ktab[ksteps - 1];
            gather();
            total(ksteps - 1, kt);
        };
        __syncthreads();
        constexpr int NV = kPatchSamples / 64, NPT = kPatchPoints;
        // the lane's samples: offsets, weights and basis values in registers
        double w[NV][NPT], b[NV], part[NV];
        uint32_t at[NV][NPT];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int i = v * 64 + lane;
            b[v] = i < nsamp ? sb[i] : 0.0;
#pragma unroll
            for (int q = 0; q < NPT; ++q) {
                const bool in = i < nsamp && q < P;
                at[v][q] = in ? so[i * P + q] : 0u;
                w[v][q] = in ? sw[i * P + q] : 0.0;
            }
        }
        advance(
            [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    if (v * 64 >= nsamp) break;
                    T f[NPT];
#pragma unroll
                    for (int q = 0; q < NPT; ++q) f[q] = stage[at[v][q]];
                    double x = 0.0;
#pragma unroll
                    for (int q = 0; q < NPT; ++q)
                        if (q < P) x += w[v][q] * (double)f[q];
                    part[v] = v * 64 + lane < nsamp ? 0.0 + b[v] * x : 0.0;
                }
            },
            part);
        if (lane == 0) {
            acc[0] = acc_s;
            acc[1] = acc_c;
        }
        return;
    }

    // ---- the patch: neighbours, coefficients, fields ----------------------
    Patch2DCell pc{};
    if (tid < n) {
        const auto q = reinterpret_cast<yee::gmem<const uint64_t>>(as_global(hd.cells[TM ? 0 : 1])) +
                       (int64_t)4 * (part * n + tid);
        const uint64_t w[4] = {q[0], q[1], q[2], q[3]};
        __builtin_memcpy(&pc, w, sizeof(pc));
    }
    const bool act = (pc.flags & kPatchUsed) != 0;
    const int x0 = pc.x0, y0 = pc.y0;
    const bool whole = act && x0 + CX <= nx && y0 + B <= ny;   // no cell beyond the grid
    T* const er = XE + (act ? pc.right : n) * S;   // E column of the patch to the right
    T* const eu = XE + (act ? pc.up : n) * S;      // E row of the patch above
    T* const hl = XH + (act ? pc.left : n) * S;    // H column of the patch to the left
    T* const hb = XH + (act ? pc.down : n) * S;    // H row of the patch below
    T* const xe = XE + (act ? tid : n + 1) * S;
    T* const xh = XH + (act ? tid : n + 1) * S;
    // a, b of the materials the cells share
    const T a_e = lk[(C0 * 256 + hd.id_e) * 2], a_h = lk[(C2 * 256 + hd.id_h) * 2];
    const T be = yee::lane_value(lk[(C0 * 256 + hd.id_e) * 2 + 1], 0);
    const T bh = yee::lane_value(lk[(C2 * 256 + hd.id_h) * 2 + 1], 0);

    const T bh2 = yee::lane_value(lk[(C2 * 256 + hd.id_h2) * 2 + 1], 0);   // kMaskH
    constexpr bool MASK_E = COEF == kMaskB || COEF == kMaskH, MASK_H = COEF == kMaskH;

    T f0[B][CX], f1[B][CX], f2[B][CX];
    uint32_t live[NE], high[NH];                   // the masks of kMaskB and kMaskH
    constexpr int KE = MASK_E ? 1 : NC, KH = COEF == kRegAll ? NC : 1;
    T ke[NE][KE], kh[NH][KH];                      // kRegE, kRegAll: b of the cells
    uint32_t in_m = 0;                             // cells inside the measured box
#pragma unroll
    for (int e = 0; e < NE; ++e) live[e] = pc.live[e];
#pragma unroll
    for (int h = 0; h < NH; ++h) high[h] = pc.high[h];
    {
        const auto F0 = as_global(static_cast<const T*>(src ? g.fb : g.fa)) + d.field_off;
        const auto F1 = F0 + g.ncell;
        const auto F2 = F1 + g.ncell;
        const int kick = (int)((d.src_off - d.field_off) / g.ncell);   // slot of the kicked component
        const auto I0 = as_global(g.ids[C0]), I1 = as_global(g.ids[C1]), I2 = as_global(g.ids[C2]);
        if (whole && !start) {
#pragma unroll
            for (int r = 0; r < B; ++r) {
                const uint32_t c = (uint32_t)((y0 + r) * nx + x0);
                p2_load_row<0>(F0 + c, f0[r]);
                p2_load_row<0>(F1 + c, f1[r]);
                p2_load_row<0>(F2 + c, f2[r]);
            }
        } else {
#pragma unroll
            for (int r = 0; r < B; ++r) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < CX; ++j) {
                    const int x = x0 + j, y = y0 + r;
                    const bool in = act && x < nx && y < ny;
                    const uint32_t c = in ? (uint32_t)(y * nx + x) : 0u;
                    if (start) {
                        const bool at = in && x >= kx0 && x <= kx1 && y >= ky0 && y <= ky1;
                        const T v = at ? stage[(y - ky0) * kbw + x - kx0] : T(0);
                        f0[r][j] = kick == 0 ? v : T(0);
                        f1[r][j] = kick == 1 ? v : T(0);
                        f2[r][j] = kick == 2 ? v : T(0);
                    } else {
                        const T v0 = F0[c], v1 = F1[c], v2 = F2[c];
                        f0[r][j] = in ? v0 : T(0);
                        f1[r][j] = in ? v1 : T(0);
                        f2[r][j] = in ? v2 : T(0);
                    }
                }
            }
        }
#pragma unroll
        for (int r = 0; r < B; ++r) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < CX; ++j) {
                const int x = x0 + j, y = y0 + r, k = r * CX + j;
                const bool in = act && x < nx && y < ny;
                const uint32_t c = in ? (uint32_t)(y * nx + x) : 0u;
                if constexpr (COEF == kRegE) {
                    ke[0][k % KE] = masked(be, pc.live[0], k);
                    if constexpr (!TM) ke[NE - 1][k % KE] = masked(be, pc.live[1], k);
                    if (!hd.masks) {
                        ke[0][k % KE] = lk[(C0 * 256 + (in ? I0[c] : kNullId)) * 2 + 1];
                        if constexpr (!TM) ke[NE - 1][k % KE] = lk[(C1 * 256 + (in ? I1[c] : kNullId)) * 2 + 1];
                    }
                }
                if constexpr (COEF == kRegAll) {
                    const uint32_t i0 = in ? I0[c] : kNullId, i1 = in ? I1[c] : kNullId, i2 = in ? I2[c] : kNullId;
                    ke[0][k % KE] = lk[(C0 * 256 + i0) * 2 + 1];
                    if constexpr (!TM) ke[NE - 1][k % KE] = lk[(C1 * 256 + i1) * 2 + 1];
                    if constexpr (TM) kh[0][k % KH] = lk[(C1 * 256 + i1) * 2 + 1];
                    kh[NH - 1][k % KH] = lk[(C2 * 256 + i2) * 2 + 1];
                }
                if (surf && in && x >= mx0 && x <= mx1 && y >= my0 && y <= my1) in_m |= 1u << k;
            }
        }
    }
    const int mbase = (y0 - my0) * mbw + x0 - mx0;
    // the wave's cells inside the box, as a scalar
    uint32_t wave_m = in_m;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) wave_m |= __shfl_xor(wave_m, off, 64);
    wave_m = __builtin_amdgcn_readfirstlane(wave_m);
    const int ms = d.meas_slot;

    auto b_e = [&](int e, int k) __attribute__((always_inline)) -> T {
        if constexpr (MASK_E) return masked(be, live[e], k);
        else return ke[e][k % KE];
    };
    auto b_h = [&](int h, int k) __attribute__((always_inline)) -> T {
        if constexpr (COEF == kRegAll) return kh[h][k % KH];
        else if constexpr (MASK_H) return selected(bh2, bh, high[h], k);
        else return bh;
    };
    // large patches take their rows in turn, so that the registers hold one row's
    // temporaries; small ones interleave them to hide the arithmetic's latency
    constexpr bool rows_in_turn = NC > 8;
    // a half step, or (START) its part of the consistent start, the (b / 2) curl
    auto half_h = [&](auto mode) __attribute__((always_inline)) {
        constexpr bool START = decltype(mode)::value;
        if constexpr (MASK_H)
#pragma unroll
            for (int h = 0; h < NH; ++h) asm volatile("" : "+v"(high[h]));
        T eR[B], eU[CX];
        p2_col<false, X>(er, eR);
#pragma unroll
        for (int r = 0; r < B; ++r) {
            if (rows_in_turn) __builtin_amdgcn_sched_barrier(0);
            if (r + 2 == B || B == 1)
                p2_row<false, X>(eu, eU);
#pragma unroll
            for (int j = 0; j < CX; ++j) {
                const int k = r * CX + j;
                if constexpr (TM) {
                    const T ez = f0[r][j];
                    const T ezr = j + 1 < CX ? f0[r][(j + 1) % CX] : eR[r];
                    const T ezu = r + 1 < B ? f0[(r + 1) % B][j] : eU[j];
                    p2_sub<START>(f1[r][j], a_h, b_h(0, k), ezu - ez);
                    p2_sub<START>(f2[r][j], a_h, b_h(NH - 1, k), ez - ezr);
                } else {
                    const T ex = f0[r][j], ey = f1[r][j];
                    const T eyr = j + 1 < CX ? f1[r][(j + 1) % CX] : eR[r];
                    const T exu = r + 1 < B ? f0[(r + 1) % B][j] : eU[j];
                    p2_sub<START>(f2[r][j], a_h, b_h(0, k), (eyr - ey) - (exu - ex));
                }
            }
        }
    };
    auto half_e = [&](auto mode) __attribute__((always_inline)) {
        constexpr bool START = decltype(mode)::value;
        if constexpr (MASK_E)   // no b values kept across steps
#pragma unroll
            for (int e = 0; e < NE; ++e) asm volatile("" : "+v"(live[e]));
        T hL[B], hD[CX];
        p2_row<false, X>(hb, hD);
        p2_col<false, X>(hl, hL);
        // the row and column that wait for the neighbours' values last
#pragma unroll
        for (int r = B - 1; r >= 0; --r) {
            if (rows_in_turn) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = CX - 1; j >= 0; --j) {
                const int k = r * CX + j;
                if constexpr (TM) {
                    const T hx = f1[r][j], hy = f2[r][j];
                    const T hyl = j > 0 ? f2[r][(j + CX - 1) % CX] : hL[r];
                    const T hxd = r > 0 ? f1[(r + B - 1) % B][j] : hD[j];
                    p2_add<START>(f0[r][j], a_e, b_e(0, k), (hy - hyl) - (hx - hxd));
                } else {
                    const T hz = f2[r][j];
                    const T hzl = j > 0 ? f2[r][(j + CX - 1) % CX] : hL[r];
                    const T hzd = r > 0 ? f2[(r + B - 1) % B][j] : hD[j];
                    p2_add<START>(f0[r][j], a_e, b_e(0, k), hz - hzd);
                    p2_sub<START>(f1[r][j], a_e, b_e(NE - 1, k), hz - hzl);
                    if (START) f1[r][j] = -f1[r][j];   // E_y <- -(b / 2) d
                }
            }
        }
    };
    // bottom E row and left E column; top H row and right H column
    auto publish_e = [&]() __attribute__((always_inline)) {
        T c[B];
#pragma unroll
        for (int r = 0; r < B; ++r) c[r] = TM ? f0[r][0] : f1[r][0];
        p2_row<true, X>(xe, f0[0]);
        p2_col<true, X>(xe, c);
    };
    auto publish_h = [&]() __attribute__((always_inline)) {
        T c[B];
#pragma unroll
        for (int r = 0; r < B; ++r) c[r] = f2[r][CX - 1];
        p2_row<true, X>(xh, TM ? f1[B - 1] : f2[B - 1]);
        p2_col<true, X>(xh, c);
    };
    auto put = [&]() __attribute__((always_inline)) {
        asm volatile("" : "+v"(in_m));             // no masks kept across steps
#pragma unroll
        for (int r = 0; r < B; ++r)
#pragma unroll
            for (int j = 0; j < CX; ++j)
                if ((wave_m >> (r * CX + j)) & 1u) {
                    const T a = f0[r][j], b = f1[r][j], c = f2[r][j];
                    if ((in_m >> (r * CX + j)) & 1u) stage[mbase + r * mbw + j] = ms == 0 ? a : ms == 1 ? b : c;
                }
    };
    using Step = std::false_type;
    using Start = std::true_type;
    if (start) {
        // E-current runs set H^{-1/2}, H-current runs E^{+1/2}
        if (d.kind == 0) publish_e();
        else publish_h();
        __syncthreads();
        if (d.kind == 0) half_h(Start{});
        else half_e(Start{});
        __syncthreads();
    }
    publish_e();
    __syncthreads();
    for (int step = 0; step < ksteps; ++step) {
        half_h(Step{});
        publish_h();
        __syncthreads();
        half_e(Step{});
        publish_e();
        if (wave_m) put();
        __syncthreads();
    }
    const auto F0 = as_global(static_cast<T*>(dst ? g.fb : g.fa)) + d.field_off;
    const auto F1 = F0 + g.ncell;
    const auto F2 = F1 + g.ncell;
    if (!(pc.flags & kPatchStored)) return;
    if (whole) {
#pragma unroll
        for (int r = 0; r < B; ++r) {
            const uint32_t c = (uint32_t)((y0 + r) * nx + x0);
            p2_store_row<0>(F0 + c, f0[r]);
            p2_store_row<0>(F1 + c, f1[r]);
            p2_store_row<0>(F2 + c, f2[r]);
        }
        return;
    }
#pragma unroll
    for (int r = 0; r < B; ++r)
#pragma unroll
        for (int j = 0; j < CX; ++j)
            if (x0 + j < nx && y0 + r < ny) {
                const uint32_t c = (uint32_t)((y0 + r) * nx + x0 + j);
                F0[c] = f0[r][j];
                F1[c] = f1[r][j];
                F2[c] = f2[r][j];
            }
}

// POL 0: items of both polarizations (small shapes only: the registers of the
// larger ones leave no room for two bodies)
template <typename T, int POL, int CX, int B, int MW, int COEF>
__global__ __launch_bounds__(256 * MW) __attribute__((amdgpu_waves_per_eu(MW)))
void k_patch2d(const ChanDev* __restrict__ ch, const int* __restrict__ items, const InstDev* __restrict__ insts,
               const Patch2DInst* __restrict__ heads, int kmax, int mclock, int src, int dst, P2Lds l) {
    const int item = items[blockIdx.x], part = item >> kPartShift;
    const ChanDev d = ch[item & ((1 << kPartShift) - 1)];
    const InstDev g = insts[d.inst];
    const Patch2DInst hd = heads[d.inst];
    const int m0 = mclock - g.start;               // instance's own step
    const int ksteps = min(kmax, g.nsteps - m0);
    if (m0 < 0 || ksteps <= 0) return;             // not started / finished
    if constexpr (POL != 0) p2_advance<T, POL, CX, B, COEF>(d, g, hd, part, m0, ksteps, src, dst, l);
    else if (d.pol == CF_POL_TM) p2_advance<T, CF_POL_TM, CX, B, COEF>(d, g, hd, part, m0, ksteps, src, dst, l);
    else p2_advance<T, CF_POL_TE, CX, B, COEF>(d, g, hd, part, m0, ksteps, src, dst, l);
}

// Shapes (columns, rows, waves per SIMD of the register budget, coefficients).
// None spills in the step loop; 128 registers hold up to 32 cells with masks,
// 20 with E values, 12 with all values (12, 8, 6 in FP64).  Twelve pistons of
// 400 x (84 .. 160) with mu = 5 sidewalls (FP32, 1000 steps): 246 ms with kMaskH,
// 328 on tiles, where kRegAll holds only the smallest.
template <typename T>
struct P2Shapes;
template <>
struct P2Shapes<float> {
    static constexpr int n = 14;
    static constexpr Patch2DShape s[n] = {{8, 4, 4, kMaskB},  {6, 5, 4, kMaskB}, {5, 5, 4, kMaskB}, {5, 4, 4, kRegE},
                                          {4, 4, 4, kRegE},   {4, 2, 4, kRegE},  {2, 2, 4, kRegE},  {4, 3, 4, kRegAll},
                                          {3, 2, 4, kRegAll}, {2, 2, 4, kRegAll}, {2, 1, 4, kRegE},  {8, 4, 4, kMaskH},
                                          {5, 5, 4, kMaskH},  {4, 4, 4, kMaskH}};
};
template <>
struct P2Shapes<double> {
    static constexpr int n = 9;
    static constexpr Patch2DShape s[n] = {{4, 3, 4, kMaskB}, {4, 2, 4, kRegE},   {3, 2, 4, kRegE},
                                          {2, 2, 4, kRegE},  {3, 2, 4, kRegAll}, {2, 2, 4, kRegAll},
                                         {2, 1, 4, kRegE},  {4, 3, 4, kMaskH},  {3, 3, 4, kMaskH}};
};

template <typename T, int V = 0>
int p2_stride_of(const Patch2DShape& q) {
    if constexpr (V < P2Shapes<T>::n) {
        constexpr Patch2DShape c = P2Shapes<T>::s[V];
        if (c.cx == q.cx && c.b == q.b) return P2Entry<T, c.cx, c.b>::stride;
        return p2_stride_of<T, V + 1>(q);
    } else {
        return 0;
    }
}

template <typename T, int V>
hipError_t p2_launch(int shape, int pol, int threads, const P2Lds& l, const ChanDev* ch, const int* items, int nitems,
                     const InstDev* inst, const Patch2DInst* heads, int kmax, int m, int src, int dst, hipStream_t s) {
    if constexpr (V >= P2Shapes<T>::n) {
        return hipErrorInvalidValue;
    } else {
        if (shape != V)
            return p2_launch<T, V + 1>(shape, pol, threads, l, ch, items, nitems, inst, heads, kmax, m, src, dst, s);
        constexpr Patch2DShape q = P2Shapes<T>::s[V];
        if (threads > 256 * q.mw) return hipErrorInvalidValue;
        auto run = [&](auto kernel) -> hipError_t {
            if (!lds_allow(reinterpret_cast<const void*>(kernel), (size_t)l.total)) return hipErrorInvalidValue;
            hipLaunchKernelGGL(kernel, dim3(nitems), dim3(threads), l.total, s, ch, items, inst, heads, kmax, m, src,
                               dst, l);
            return hipGetLastError();
        };
        if (pol == CF_POL_TM) return run(&k_patch2d<T, CF_POL_TM, q.cx, q.b, q.mw, q.coef>);
        if (pol == CF_POL_TE) return run(&k_patch2d<T, CF_POL_TE, q.cx, q.b, q.mw, q.coef>);
        if constexpr (patch2d_small(q.cx * q.b, sizeof(T))) return run(&k_patch2d<T, 0, q.cx, q.b, q.mw, q.coef>);
        return hipErrorInvalidValue;
    }
}

}  // namespace

template <typename T>
int patch2d_shapes(Patch2DShape* out, int max) {
    const int n = std::min(P2Shapes<T>::n, max);
    for (int k = 0; k < n; ++k) out[k] = P2Shapes<T>::s[k];
    return n;
}

template <typename T>
size_t patch2d_lds(const Patch2DShape& q, int n, const Patch2DSizes& z) {
    // the static part: s_box, once per polarization a kernel holds
    return (size_t)p2_lds<T>(p2_stride_of<T>(q), n, z).total + 2 * 8 * sizeof(int);
}

template <typename T>
hipError_t launch_patch2d(int shape, int pol, const ChanDev* ch, const int* items, int nitems, const InstDev* inst,
                          const Patch2DInst* heads, int n, const Patch2DSizes& z, int kmax, int m, int src, int dst,
                          hipStream_t s) {
    if (nitems <= 0) return hipSuccess;
    if (shape < 0 || shape >= P2Shapes<T>::n || n < 0 || kmax < 1) return hipErrorInvalidValue;
    const Patch2DShape& q = P2Shapes<T>::s[shape];
    // a wave of its own takes the surface sums
    const int threads = (n + 63) / 64 * 64 + 64;
    return p2_launch<T, 0>(shape, pol, threads, p2_lds<T>(p2_stride_of<T>(q), n, z), ch, items, nitems, inst, heads,
                           kmax, m, src, dst, s);
}

#define CF_INSTANTIATE(T)                                                                                          \
    template int patch2d_shapes<T>(Patch2DShape*, int);                                                            \
    template size_t patch2d_lds<T>(const Patch2DShape&, int, const Patch2DSizes&);                                 \
    template hipError_t launch_patch2d<T>(int, int, const ChanDev*, const int*, int, const InstDev*,               \
                                          const Patch2DInst*, int, const Patch2DSizes&, int, int, int, int,        \
                                          hipStream_t);
CF_INSTANTIATE(float)
CF_INSTANTIATE(double)
#undef CF_INSTANTIATE

}  // namespace cf
