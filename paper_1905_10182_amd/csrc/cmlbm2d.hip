// Two-dimensional D2Q9 central-moment lattice Boltzmann solver with Hermite
// forcing for gfx950 (MI355X): the model of App. B of De Rosis, Huang &
// Coreixas, PRE 2019.  C ABI: include/cmlbm2d.h.  The per-cell collision is in
// d2q9.hpp; this file holds the kernels and the host side.
//
// Data layout in HBM: every population in rows of nx values padded to 256
// bytes; FP32 and 16-bit storage keep the nine population rows of one lattice
// row together (row blocks, [ny][9][row]), FP64 keeps nine planes of ny rows
// kPlanePad bytes apart beyond their rows; values stored shifted (f_i - w_i rho0) in the storage type; two such
// buffers alternate (read one, write the other).  The stored array A_i(y)
// holds the population that the next pull gather moves to y + c_i, so
// f_i(x, t) = A_i(x - c_i): a step is gather (streaming), collision and a
// store at the cell's own index.
//
// Kernels: k2_step one step; k2_march and k2_tile several steps of FP64 and
// FP32 storage in one launch (large and small planes); k2_init, k2_gather the
// state's import and export.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <new>
#include <string>
#include <type_traits>

#include "cmlbm2d.h"
#include "d2q9.hpp"

using namespace cmlbm2d;

// Cells per lane of the step kernel for each storage type (overridable for
// tuning builds); a value above 1 is used only when it divides nx.
#ifndef CMLBM2D_LANES_FP64
#define CMLBM2D_LANES_FP64 1
#endif
#ifndef CMLBM2D_LANES_FP32
#define CMLBM2D_LANES_FP32 2
#endif
#ifndef CMLBM2D_LANES_16
#define CMLBM2D_LANES_16 4
#endif

namespace {

constexpr int kBlock = 256;         // threads per workgroup
constexpr size_t kPlanePad = 4096;  // bytes between consecutive FP64 population planes (a multiple of 256)

// ---------------------------------------------------------------------------
// storage types: S is stored, T is the arithmetic type

template <int ST>
struct storage2;
template <>
struct storage2<CMLBM2D_FP64> {
    typedef double S;
    typedef double T;
    static __device__ __forceinline__ T load(S v) { return v; }
    static __device__ __forceinline__ S pack(T v) { return v; }
};
template <>
struct storage2<CMLBM2D_FP32> {
    typedef float S;
    typedef float T;
    static __device__ __forceinline__ T load(S v) { return v; }
    static __device__ __forceinline__ S pack(T v) { return v; }
};
// FP16 carries a factor 2^8 so that the small shifted populations stay in
// its normal range.
template <>
struct storage2<CMLBM2D_FP16> {
    typedef _Float16 S;
    typedef float T;
    static __device__ __forceinline__ T load(S v) { return (float)v * 0.00390625f; }
    static __device__ __forceinline__ S pack(T v) { return (_Float16)(v * 256.0f); }
};
template <>
struct storage2<CMLBM2D_BF16> {
    typedef __bf16 S;
    typedef float T;
    static __device__ __forceinline__ T load(S v) { return (float)v; }
    static __device__ __forceinline__ S pack(T v) { return (__bf16)v; }
};

size_t storage_bytes(int st) { return st == CMLBM2D_FP64 ? 8 : st == CMLBM2D_FP32 ? 4 : 2; }

struct Geom2 {
    int nx, ny;
    int nxp;           // padded row length (elements)
    int V;             // cells per lane of the step kernel
    int segs;          // 64-lane segments per row in the step kernel
    int nblk;          // step workgroups
    uint64_t pstride;  // elements from population i to i + 1 of one row
    uint64_t rstride;  // elements from one row of a population to the next row
    uint64_t ncell;    // ny * nx
};

__device__ __forceinline__ int wrap(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// lane l receives the value of lane l - 1 (mod 64) / lane l + 1 (mod 64)
__device__ __forceinline__ int from_prev_lane(int v) { return __builtin_amdgcn_mov_dpp(v, 0x13C, 0xF, 0xF, false); }
__device__ __forceinline__ int from_next_lane(int v) { return __builtin_amdgcn_mov_dpp(v, 0x134, 0xF, 0xF, false); }

template <typename S>
__device__ __forceinline__ S shift_lane(S v, bool prev)
{
    if constexpr (sizeof(S) == 8) {
        const int2 w = __builtin_bit_cast(int2, v);
        int2 r;
        r.x = prev ? from_prev_lane(w.x) : from_next_lane(w.x);
        r.y = prev ? from_prev_lane(w.y) : from_next_lane(w.y);
        return __builtin_bit_cast(S, r);
    } else if constexpr (sizeof(S) == 4) {
        const int w = __builtin_bit_cast(int, v);
        return __builtin_bit_cast(S, prev ? from_prev_lane(w) : from_next_lane(w));
    } else {
        const int w = (int)__builtin_bit_cast(unsigned short, v);
        const int r = prev ? from_prev_lane(w) : from_next_lane(w);
        return __builtin_bit_cast(S, (unsigned short)r);
    }
}

template <typename X>
__device__ __forceinline__ X load_at(const void* base, uint32_t byte_off)
{
    return *(const X*)((const char*)base + byte_off);
}

// Non-temporal store: the post-collision populations are not read again in
// this step.
template <typename X>
__device__ __forceinline__ void store_nt(void* base, uint32_t byte_off, X v)
{
    X* p = (X*)((char*)base + byte_off);
    if constexpr (sizeof(X) == 16) {
        typedef int i4 __attribute__((ext_vector_type(4)));
        __builtin_nontemporal_store(__builtin_bit_cast(i4, v), (i4*)p);
    } else if constexpr (sizeof(X) == 8) {
        __builtin_nontemporal_store(__builtin_bit_cast(unsigned long long, v), (unsigned long long*)p);
    } else if constexpr (sizeof(X) == 4) {
        __builtin_nontemporal_store(__builtin_bit_cast(unsigned, v), (unsigned*)p);
    } else {
        __builtin_nontemporal_store(__builtin_bit_cast(unsigned short, v), (unsigned short*)p);
    }
}

// ---------------------------------------------------------------------------
// the hot path: one fused time step
//
// Wave w owns segment (w mod segs) of row (w / segs): 64 lanes x V cells.
// Every cell pulls its nine populations from x - c_i (periodic), collides
// (cmlbm2d::collide) and stores the nine post-collision values at its own
// index.  With V > 1 each lane reads every plane as one aligned V-element
// vector; the six planes with c_x = +-1 need the row shifted by one cell,
// done in registers: the element crossing a lane boundary comes from the
// neighbouring lane by a DPP wave rotation (which is also the periodic wrap
// when a row is exactly one wave), and the end lanes of a segment otherwise
// reload that element.  Row addressing is wave-uniform (scalar registers);
// each access is a scalar base plus a 32-bit per-lane byte offset.

template <int ST, int V, bool FIELD>
__global__ __launch_bounds__(kBlock) void k2_step(const typename storage2<ST>::S* __restrict__ src,
                                                   typename storage2<ST>::S* __restrict__ dst, Geom2 g,
                                                   typename storage2<ST>::T omega, typename storage2<ST>::T rho0,
                                                   typename storage2<ST>::T fx, typename storage2<ST>::T fy,
                                                   const typename storage2<ST>::T* __restrict__ field)
{
    using SS = storage2<ST>;
    using S = typename SS::S;
    using T = typename SS::T;
    typedef S vt __attribute__((ext_vector_type(V == 1 ? 2 : V)));
    const int blk = (int)blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(blk * (kBlock / 64) + (int)(threadIdx.x >> 6));
    const int row = wave / g.segs;
    if (row >= g.ny) return;  // whole wave
    const int seg = wave - row * g.segs;
    const int x0 = (seg * 64 + lane) * V;
    const bool active = x0 < g.nx;
    const S* srow[3];  // [c_y + 1]: source row y - c_y
#pragma unroll
    for (int b = 0; b < 3; ++b) srow[b] = src + (uint64_t)wrap(row - (b - 1), g.ny) * g.rstride;
    T h[V][9];
    if constexpr (V == 1) {
        if (!active) return;
        const uint32_t bx[3] = {(uint32_t)wrap(x0 + 1, g.nx) * (uint32_t)sizeof(S), (uint32_t)x0 * (uint32_t)sizeof(S),
                                (uint32_t)wrap(x0 - 1, g.nx) * (uint32_t)sizeof(S)};
#pragma unroll
        for (int i = 0; i < 9; ++i)
            h[0][i] = SS::load(load_at<S>(srow[vel_y(i) + 1] + (uint64_t)i * g.pstride, bx[vel_x(i) + 1]));
    } else {
        const bool whole = g.nx == 64 * V;
        const bool prev_in_reg = whole || lane > 0;
        const bool next_in_reg = whole || (lane < 63 && x0 + V < g.nx);
        const uint32_t bxm = (uint32_t)(x0 == 0 ? g.nx - 1 : x0 - 1) * (uint32_t)sizeof(S);
        const uint32_t bxp = (uint32_t)(x0 + V >= g.nx ? 0 : x0 + V) * (uint32_t)sizeof(S);
        const uint32_t bx0 = (uint32_t)x0 * (uint32_t)sizeof(S);
        vt v[9];
#pragma unroll
        for (int i = 0; i < 9; ++i)
            v[i] = active ? load_at<vt>(srow[vel_y(i) + 1] + (uint64_t)i * g.pstride, bx0) : vt(0);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            if (vel_x(i) == 0) {
#pragma unroll
                for (int c = 0; c < V; ++c) h[c][i] = SS::load(v[i][c]);
                continue;
            }
            // cell c of a c_x = +1 plane reads element c - 1, of a c_x = -1 plane element c + 1
            const bool prev = vel_x(i) == 1;
            S e = shift_lane<S>(prev ? v[i][V - 1] : v[i][0], prev);
            if (!(prev ? prev_in_reg : next_in_reg) && active)
                e = load_at<S>(srow[vel_y(i) + 1] + (uint64_t)i * g.pstride, prev ? bxm : bxp);
#pragma unroll
            for (int c = 0; c < V; ++c) {
                const S s = prev ? (c == 0 ? e : v[i][c - 1]) : (c == V - 1 ? e : v[i][c + 1]);
                h[c][i] = SS::load(s);
            }
        }
        if (!active) return;
    }
    T Fx[V], Fy[V];
#pragma unroll
    for (int c = 0; c < V; ++c) {
        if (FIELD) {
            const uint64_t lin = (uint64_t)row * (uint64_t)g.nx + (uint64_t)(x0 + c);
            Fx[c] = field[lin];
            Fy[c] = field[g.ncell + lin];
        } else {
            Fx[c] = fx;
            Fy[c] = fy;
        }
    }
#pragma unroll
    for (int c = 0; c < V; ++c) {
        T drho, ux, uy;
        if constexpr (sizeof(S) == 2)
            joined::collide<T>(h[c], Fx[c], Fy[c], omega, rho0, drho, ux, uy);
        else
            lockstep::collide<T>(h[c], Fx[c], Fy[c], omega, rho0, drho, ux, uy);
    }
    const uint32_t own = (uint32_t)x0 * (uint32_t)sizeof(S);
    const uint64_t orow = (uint64_t)row * g.rstride;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        S* plane_row = dst + (uint64_t)i * g.pstride + orow;
        if constexpr (V == 1) {
            store_nt<S>(plane_row, own, SS::pack(h[0][i]));
        } else {
            vt o;
#pragma unroll
            for (int c = 0; c < V; ++c) o[c] = SS::pack(h[c][i]);
            store_nt<vt>(plane_row, own, o);
        }
    }
}

// ---------------------------------------------------------------------------
// several steps in one pass
//
// K steps of a strip of 64 V cells, one wave, marching up y.  At source row r
// of the state, stage 1 pulls from the stored populations and finishes row
// r - 1 of the next time; stage k takes the numbers that stage k - 1 finished
// (rho - rho0, u, s4, s5: with the force they determine the post-collision
// populations), reconstructs that row and finishes row r - k, k steps on; the
// last stage's row is reconstructed and stored.  The x shift is a DPP rotation
// of the wave; the y shift stays in a lane's registers: of a row, class
// c_y = -1 goes to the row below, 0 to the row itself, +1 to the row above, as
// three row sums each.  No barrier: waves are independent.
// The stages are kept apart in the schedule: left to itself the compiler moves
// parts of later stages up until the registers are full (K = 6 with a field:
// 256 and spills instead of 195; K = 4 on 3001 x 3000 358 -> 283 us).
// A strip loses one cell at each end per stage, so strips overlap by 2 H >= 2 K
// cells (none where a strip is exactly a periodic row), and a chunk of rows
// starts and ends K rows outside.
// What bounds it: K = 2 HBM, 72 bytes per cell (FP32) and 8 with a field, at 5.1
// TB/s; K = 8 the issue of vector instructions, 148 lane-operations per cell and
// step (the overlap included) at 85% of the rate at 2.4 GHz.  Per step at 8192^2 with a force field: FP32 k2_step 890, K = 2 524,
// 4 320, 6 299, 8 270 us; FP64 1870, 1100, 592, 518, 489.
// H: for K = 2, 8 cells make strips of whole 64-byte pieces, where 2 leave each
// end in pieces that two waves write (FP32 8192^2 1260 -> 1050 us a pass);
// longer passes lose more to the overlap than that gains (K = 4 on 2048^2 97 /
// 101 us, FP64 on 4096^2 592 / 650).
constexpr int march_halo(int K) { return K == 2 ? 8 : K; }

template <typename X>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const X* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)bytes, 0x00020000);
}

template <int ST, int V, int K, bool FIELD>
__global__ __launch_bounds__(kBlock, K >= 6 ? 2 : 1) void k2_march(const typename storage2<ST>::S* __restrict__ src,
                                                   typename storage2<ST>::S* __restrict__ dst, Geom2 g, int strips,
                                                   int rows, typename storage2<ST>::T omega,
                                                   typename storage2<ST>::T rho0, typename storage2<ST>::T fx,
                                                   typename storage2<ST>::T fy,
                                                   const typename storage2<ST>::T* __restrict__ field)
{
    using T = typename storage2<ST>::T;
    static_assert(std::is_same<T, typename storage2<ST>::S>::value, "FP64 and FP32 storage");
    constexpr int H = march_halo(K);
    static_assert(H >= K && H % V == 0 && V * sizeof(T) <= 8, "a lane's cells are one vector of 4 or 8 bytes");
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)));
    const int chunk = wave / strips, strip = wave - chunk * strips;
    const int ys = chunk * rows, ye = ys + rows < g.ny ? ys + rows : g.ny;
    if (ys >= g.ny) return;  // whole wave
    // cells of this lane: position i0 in the strip, x (periodic); stored are the
    // positions [H, 64 V - H) of an overlapping strip that lie in the row
    const bool ring = g.nx == 64 * V;
    const int stride = ring ? 64 * V : 64 * V - 2 * H, i0 = lane * V;
    const int xr = strip * stride + i0 - (ring ? 0 : H);
    const int x = ((xr % g.nx) + g.nx) % g.nx;
    const bool stored = ring || (i0 >= H && i0 < 64 * V - H && xr < g.nx);
    constexpr uint32_t kNone = 0xffffff00u;  // past every range: the store is dropped
    const uint32_t rowb = (uint32_t)g.nxp * (uint32_t)sizeof(T), off = (uint32_t)x * (uint32_t)sizeof(T);
    const uint32_t fieldb = (uint32_t)g.nx * (uint32_t)sizeof(T);
    auto ld = [&](const T* row, uint32_t bytes, T v[V]) {
        if constexpr (V * sizeof(T) == 4) {
            v[0] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(rsrc_of(row, bytes), off, 0, 0));
            return;
        }
        const u2 w = __builtin_amdgcn_raw_buffer_load_b64(rsrc_of(row, bytes), off, 0, 0);
        if constexpr (sizeof(T) == 8) {
            v[0] = __builtin_bit_cast(T, w);
        } else {
            const uint32_t w0 = w.x, w1 = w.y;
            v[0] = __builtin_bit_cast(T, w0);
            v[V - 1] = __builtin_bit_cast(T, w1);
        }
    };

    // Forces of the K rows that the stages work on: each is loaded once and kept
    // in the wave's own ring of LDS rows until the last stage has used it.
    typedef T tv __attribute__((ext_vector_type(V == 1 ? 2 : V)));
    using FV = std::conditional_t<V == 1, T, tv>;
    __shared__ FV ring_f[FIELD ? kBlock / 64 : 1][FIELD ? K : 1][2][64];
    FV(*const my_f)[2][64] = ring_f[FIELD ? threadIdx.x >> 6 : 0];
    int slot = 0;  // of the row that stage 1 works on

    T nh[9][V], nf[2][V];  // populations of the next source row, force of the current one
    auto load_row = [&](int r, int fr) {
        const T* p = src + (uint64_t)r * g.rstride;
#pragma unroll
        for (int i = 0; i < 9; ++i) ld(p + (uint64_t)i * g.pstride, rowb, nh[i]);
        if (FIELD) {
            ld(field + (uint64_t)fr * g.nx, fieldb, nf[0]);
            ld(field + g.ncell + (uint64_t)fr * g.nx, fieldb, nf[1]);
        }
    };
    T Z[K][V][3], P[K][2][V][3];  // row sums of c_y = 0 (last row) and +1 (last two rows) of each stage
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int c = 0; c < V; ++c)
#pragma unroll
            for (int j = 0; j < 3; ++j) Z[k][c][j] = P[k][0][c][j] = P[k][1][c][j] = T(0);
    const T om1 = T(1) - omega;

    int y[K + 1];  // row of stage k's target, periodic (y[0]: the source row)
    y[0] = (((ys - K) % g.ny) + g.ny) % g.ny;
#pragma unroll
    for (int k = 1; k <= K; ++k) y[k] = y[k - 1] == 0 ? g.ny - 1 : y[k - 1] - 1;
    load_row(y[0], y[1]);
#pragma unroll
    for (int c = 0; c < V; ++c) {  // arrived: not counted in the loop
#pragma unroll
        for (int i = 0; i < 9; ++i) asm volatile("" : "+v"(nh[i][c]));
        if (FIELD) asm volatile("" : "+v"(nf[0][c]), "+v"(nf[1][c]));
    }
    auto advance = [&](int r, auto parity) {
        constexpr int q = decltype(parity)::value;
        T h[V][9], Fx[V], Fy[V];
#pragma unroll
        for (int i = 0; i < 9; ++i)
#pragma unroll
            for (int c = 0; c < V; ++c) h[c][i] = nh[i][c];
        if constexpr (FIELD) {
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                FV w;
                if constexpr (V == 1)
                    w = nf[a][0];
                else
                    for (int c = 0; c < V; ++c) w[c] = nf[a][c];
                my_f[slot][a][lane] = w;
            }
        }
        load_row(y[0] + 1 == g.ny ? 0 : y[0] + 1, y[0]);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            T X[V][3][3];  // row sums of this row, by c_y class
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const int ip = vel_index(1, b - 1), i0 = vel_index(0, b - 1), im = vel_index(-1, b - 1);
                const T from_prev = shift_lane<T>(h[V - 1][ip], true), from_next = shift_lane<T>(h[0][im], false);
#pragma unroll
                for (int c = 0; c < V; ++c)
                    lockstep::row_sums<T>(c < V - 1 ? h[c + 1][im] : from_next, h[c][i0],
                                          c > 0 ? h[c - 1][ip] : from_prev, X[c][b]);
            }
#pragma unroll
            for (int c = 0; c < V; ++c) {
                Fx[c] = fx;
                Fy[c] = fy;
                if constexpr (FIELD) {
                    const FV w0 = my_f[slot >= k ? slot - k : slot - k + K][0][lane];
                    const FV w1 = my_f[slot >= k ? slot - k : slot - k + K][1][lane];
                    if constexpr (V == 1) {
                        Fx[c] = w0;
                        Fy[c] = w1;
                    } else {
                        Fx[c] = w0[c];
                        Fy[c] = w1[c];
                    }
                }
                T drho, ux, uy, k4, k5;
                lockstep::moments_of_sums<T>(X[c][0], Z[k][c], P[k][q][c], Fx[c], Fy[c], rho0, drho, ux, uy, k4, k5);
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    Z[k][c][j] = X[c][1][j];
                    P[k][q][c][j] = X[c][2][j];
                }
                const T s4 = om1 * k4, s5 = om1 * k5;
                lockstep::reconstruct<T>(drho, ux, uy, Fx[c], Fy[c], s4, s5, rho0, h[c]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        const int yt = r - K;  // the row just finished, K steps on
        T* out = dst + (uint64_t)y[K] * g.rstride;
        const uint32_t so = stored && yt >= ys ? off : kNone;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            if constexpr (V * sizeof(T) == 4) {
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, h[0][i]),
                                                      rsrc_of(out + (uint64_t)i * g.pstride, rowb), so, 0, 2);
                continue;
            }
            u2 w;
            if constexpr (sizeof(T) == 8) {
                w = __builtin_bit_cast(u2, h[0][i]);
            } else {
                w.x = __builtin_bit_cast(uint32_t, h[0][i]);
                w.y = __builtin_bit_cast(uint32_t, h[V - 1][i]);
            }
            __builtin_amdgcn_raw_buffer_store_b64(w, rsrc_of(out + (uint64_t)i * g.pstride, rowb), so, 0, 2);
        }
#pragma unroll
        for (int k = 0; k <= K; ++k) y[k] = y[k] + 1 == g.ny ? 0 : y[k] + 1;
        slot = slot + 1 == K ? 0 : slot + 1;
    };
    int r = ys - K;
    const int end = ye + K;  // one past the last source row
    for (; r + 1 < end; r += 2) {
        advance(r, std::integral_constant<int, 0>{});
        advance(r + 1, std::integral_constant<int, 1>{});
    }
    if (r < end) advance(r, std::integral_constant<int, 0>{});
}

// K steps of a small lattice: a workgroup of kTileRows waves, one row of 64
// cells each, advances its rows K steps in registers.  Per step a wave forms
// the row sums of its populations, hands those of c_y = +1 and -1 to the rows
// above and below through LDS (two buffers in turn, one barrier), and finishes
// its own row.  A row at each end and a cell at each side are lost per step, so
// kTileRows - 2 K rows by 64 - 2 K cells (64 where that is the periodic row)
// are stored.  A launch and the loads cost as much as several of these steps,
// which is what a step of k2_step pays on such a lattice.
constexpr int kTileRows = 16;

template <int ST, bool FIELD>
__global__ __launch_bounds__(kTileRows * 64) void k2_tile(const typename storage2<ST>::S* __restrict__ src,
                                                          typename storage2<ST>::S* __restrict__ dst, Geom2 g, int K,
                                                          int strips, typename storage2<ST>::T omega,
                                                          typename storage2<ST>::T rho0,
                                                          typename storage2<ST>::T fx, typename storage2<ST>::T fy,
                                                          const typename storage2<ST>::T* __restrict__ field)
{
    using T = typename storage2<ST>::T;
    static_assert(std::is_same<T, typename storage2<ST>::S>::value, "FP64 and FP32 storage");
    __shared__ T up[2][kTileRows][3][64], down[2][kTileRows][3][64];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int tile = (int)blockIdx.x / strips, strip = (int)blockIdx.x - tile * strips;
    const bool ring = g.nx == 64;
    const int xr = strip * (ring ? 64 : 64 - 2 * K) + lane - (ring ? 0 : K);
    const int x = ((xr % g.nx) + g.nx) % g.nx;
    const int yr = tile * (kTileRows - 2 * K) + w - K;
    const int y = ((yr % g.ny) + g.ny) % g.ny;
    T h[9], Fx = fx, Fy = fy;
    const T* row = src + (uint64_t)y * g.rstride + x;
#pragma unroll
    for (int i = 0; i < 9; ++i) h[i] = row[(uint64_t)i * g.pstride];
    if (FIELD) {
        const uint64_t lin = (uint64_t)y * (uint64_t)g.nx + (uint64_t)x;
        Fx = field[lin];
        Fy = field[g.ncell + lin];
    }
    const T om1 = T(1) - omega;
    for (int t = 0; t < K; ++t) {
        const int q = t & 1;
        T X[3][3];  // row sums by c_y class
        if (w >= t && w < kTileRows - t) {
#pragma unroll
            for (int b = 0; b < 3; ++b)
                lockstep::row_sums<T>(shift_lane<T>(h[vel_index(-1, b - 1)], false), h[vel_index(0, b - 1)],
                                      shift_lane<T>(h[vel_index(1, b - 1)], true), X[b]);
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                down[q][w][j][lane] = X[0][j];
                up[q][w][j][lane] = X[2][j];
            }
        }
        __syncthreads();
        if (w > t && w < kTileRows - 1 - t) {
            T Xm[3], Xp[3], drho, ux, uy, k4, k5;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                Xm[j] = down[q][w + 1][j][lane];
                Xp[j] = up[q][w - 1][j][lane];
            }
            lockstep::moments_of_sums<T>(Xm, X[1], Xp, Fx, Fy, rho0, drho, ux, uy, k4, k5);
            const T s4 = om1 * k4, s5 = om1 * k5;
            lockstep::reconstruct<T>(drho, ux, uy, Fx, Fy, s4, s5, rho0, h);
        }
    }
    if (w < K || w >= kTileRows - K || yr >= g.ny) return;
    if (!ring && (lane < K || lane >= 64 - K || xr >= g.nx)) return;
    T* out = dst + (uint64_t)y * g.rstride + x;
#pragma unroll
    for (int i = 0; i < 9; ++i) out[(uint64_t)i * g.pstride] = h[i];
}

// ---------------------------------------------------------------------------
// cell-parallel kernels (one thread per cell, 1D grid over the N cells)

enum InitSrc { INIT_EQ_F64 = 0, INIT_EQ_F32 = 1, INIT_POPS_F64 = 2 };

// Write a pre-collision state through the inverse of the pull gather:
// A_i(x - c_i) = h_i(x).  The complete equilibrium is the reconstruction with
// zero force and zero shear moments (all its central moments are those of
// the post-collision state of a force-free, fully relaxed cell).
template <int ST, int SRC>
__global__ __launch_bounds__(kBlock) void k2_init(typename storage2<ST>::S* __restrict__ dst, Geom2 g, double rho0,
                                                  const void* __restrict__ rho_in, const void* __restrict__ u_in,
                                                  const double* __restrict__ pops)
{
    using SS = storage2<ST>;
    using T = typename SS::T;
    const uint64_t n = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (n >= g.ncell) return;
    const int x = (int)(n % (uint64_t)g.nx), y = (int)(n / (uint64_t)g.nx);
    T e[9];
    if constexpr (SRC == INIT_POPS_F64) {
#pragma unroll
        for (int i = 0; i < 9; ++i) e[i] = (T)(pops[(uint64_t)i * g.ncell + n] - weight(i) * rho0);
    } else {
        T drho = T(0), ux = T(0), uy = T(0);
        if constexpr (SRC == INIT_EQ_F64) {
            const double* R = (const double*)rho_in;
            const double* U = (const double*)u_in;
            if (R) drho = (T)(R[n] - rho0);
            if (U) {
                ux = (T)U[n];
                uy = (T)U[g.ncell + n];
            }
        } else {
            const float* R = (const float*)rho_in;
            const float* U = (const float*)u_in;
            if (R) drho = (T)((double)R[n] - rho0);
            if (U) {
                ux = (T)U[n];
                uy = (T)U[g.ncell + n];
            }
        }
        joined::reconstruct<T>(drho, ux, uy, T(0), T(0), T(0), T(0), (T)rho0, e);
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const uint64_t d = (uint64_t)i * g.pstride + (uint64_t)wrap(y - vel_y(i), g.ny) * g.rstride +
                           (uint64_t)wrap(x - vel_x(i), g.nx);
        dst[d] = SS::pack(e[i]);
    }
}

// Gather the pre-collision state of every cell: rho and the half-force
// velocity (FP64 or FP32 out), and/or the unshifted FP64 populations.
template <int ST>
__global__ __launch_bounds__(kBlock) void k2_gather(const typename storage2<ST>::S* __restrict__ src, Geom2 g,
                                                    double rho0, double fx, double fy, const void* __restrict__ field,
                                                    void* __restrict__ rho_out, void* __restrict__ u_out, int out_f64,
                                                    double* __restrict__ pops)
{
    using SS = storage2<ST>;
    const uint64_t n = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (n >= g.ncell) return;
    const int x = (int)(n % (uint64_t)g.nx), y = (int)(n / (uint64_t)g.nx);
    double h[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const uint64_t s = (uint64_t)i * g.pstride + (uint64_t)wrap(y - vel_y(i), g.ny) * g.rstride +
                           (uint64_t)wrap(x - vel_x(i), g.nx);
        h[i] = (double)SS::load(src[s]);
    }
    if (pops) {
#pragma unroll
        for (int i = 0; i < 9; ++i) pops[(uint64_t)i * g.ncell + n] = h[i] + weight(i) * rho0;
    }
    if (!rho_out && !u_out) return;
    double Fx = fx, Fy = fy;
    if (field) {
        if (ST == CMLBM2D_FP64) {
            Fx = ((const double*)field)[n];
            Fy = ((const double*)field)[g.ncell + n];
        } else {
            Fx = ((const float*)field)[n];
            Fy = ((const float*)field)[g.ncell + n];
        }
    }
    double drho = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        drho += h[i];
        jx += vel_x(i) * h[i];
        jy += vel_y(i) * h[i];
    }
    const double rho = rho0 + drho;
    const double ux = (jx + 0.5 * Fx) / rho, uy = (jy + 0.5 * Fy) / rho;
    if (out_f64) {
        if (rho_out) ((double*)rho_out)[n] = rho;
        if (u_out) {
            ((double*)u_out)[n] = ux;
            ((double*)u_out)[g.ncell + n] = uy;
        }
    } else {
        if (rho_out) ((float*)rho_out)[n] = (float)rho;
        if (u_out) {
            ((float*)u_out)[n] = (float)ux;
            ((float*)u_out)[g.ncell + n] = (float)uy;
        }
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// host side

struct cmlbm2d_lattice {
    cmlbm2d_params p;
    Geom2 g;
    void* pop[2];
    int cur;  // buffer holding the state
    int cus;  // compute units of the lattice's device
    int force_mode;
    double fu[2];  // UNIFORM force
    const void* field;
    bool initialized;
    bool graph;  // a call has been captured: even calls end in the buffer they start in
    int64_t t;
    std::string err;
};

namespace {

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

int lanes_for(int storage, int nx)
{
    int want = storage == CMLBM2D_FP64 ? CMLBM2D_LANES_FP64
                                        : storage == CMLBM2D_FP32 ? CMLBM2D_LANES_FP32 : CMLBM2D_LANES_16;
    const int vmax = 16 / (int)storage_bytes(storage);  // vectors of at most 16 bytes
    if (want > vmax) want = vmax;
    if (want > 4) want = 4;  // the step kernel is instantiated for 1, 2 and 4 cells per lane
    for (int v = want; v > 1; v /= 2)
        if (nx % v == 0) return v;
    return 1;
}

// Population layout: row blocks (the nine population rows of one lattice row
// stored together) for FP32 and 16-bit storage, planes (population i of every
// row together, 4 KiB apart) for FP64.  Measured at 8192^2 against planes: FP32
// +10%, FP16 +2.5%, FP64 -2.5% (against its spaced planes).
bool row_blocks2(int storage) { return storage != CMLBM2D_FP64; }

int make_geom(const cmlbm2d_params* p, Geom2* g, size_t* pop_bytes)
{
    if (!p) return CMLBM2D_EINVAL;
    if (p->nx < 1 || p->ny < 1) return CMLBM2D_EINVAL;
    if (!(p->tau > 0.5) || !std::isfinite(p->tau)) return CMLBM2D_EINVAL;
    if (!(p->rho0 > 0.0) || !std::isfinite(p->rho0)) return CMLBM2D_EINVAL;
    if (p->storage < CMLBM2D_FP64 || p->storage > CMLBM2D_BF16) return CMLBM2D_EINVAL;
    if (p->flags != 0) return CMLBM2D_EINVAL;
    const size_t sb = storage_bytes(p->storage);
    g->nx = p->nx;
    g->ny = p->ny;
    g->nxp = (int)(align256((size_t)p->nx * sb) / sb);
    // FP64 planes kPlanePad bytes apart beyond their rows (at power-of-two plane sizes the
    // nine plane streams otherwise share HBM channels); measured on 8192^2 it raises FP64 by
    // 6% (dense planes lowered FP16/BF16 by 6% with it, before their row blocks)
    const size_t pad = p->storage == CMLBM2D_FP64 ? kPlanePad : 0;
    const uint64_t plane = (uint64_t)p->ny * (uint64_t)g->nxp + pad / sb;
    if (plane * sb >= (1ULL << 32)) return CMLBM2D_EINVAL;  // one population's byte offsets are 32-bit
    const bool blocks = row_blocks2(p->storage);
    g->pstride = blocks ? (uint64_t)g->nxp : plane;
    g->rstride = blocks ? 9ull * g->nxp : (uint64_t)g->nxp;
    g->ncell = (uint64_t)p->ny * (uint64_t)p->nx;
    g->V = lanes_for(p->storage, p->nx);
    g->segs = (p->nx + 64 * g->V - 1) / (64 * g->V);
    const uint64_t waves = (uint64_t)p->ny * (uint64_t)g->segs;
    const uint64_t nblk = (waves + kBlock / 64 - 1) / (kBlock / 64);
    if (nblk > 0x7fffffffULL || (g->ncell + kBlock - 1) / kBlock > 0x7fffffffULL) return CMLBM2D_EINVAL;
    g->nblk = (int)nblk;
    if (pop_bytes) *pop_bytes = align256(blocks ? (uint64_t)p->ny * g->rstride * sb : 9 * plane * sb);
    return CMLBM2D_OK;
}

int fail(cmlbm2d_lattice* lat, int code, const std::string& msg)
{
    if (lat) lat->err = msg;
    return code;
}

int launch_check(cmlbm2d_lattice* lat, const char* what)
{
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess) return CMLBM2D_OK;
    return fail(lat, CMLBM2D_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

dim3 cell_grid(const Geom2& g) { return dim3((unsigned)((g.ncell + kBlock - 1) / kBlock)); }

// Strips of k2_march (and k2_tile: V = 1) across a row, with H cells of halo at each end.
int march_strips(const Geom2& g, int V, int H)
{
    return g.nx == 64 * V ? 1 : (g.nx + 64 * V - 2 * H - 1) / (64 * V - 2 * H);
}

// Waves that a SIMD holds of k2_march, by its registers (K = 4 about 150, 6 and 8 about 200 to 250).
constexpr int march_waves(int K) { return K >= 6 ? 2 : K == 4 ? 3 : 4; }

// Rows per wave of k2_march, and the waves that a SIMD then runs: the least of
// that number (a SIMD is bound by their instructions) times the rows of each
// and the 2 K it starts and ends with.
int march_rows2(const Geom2& g, int strips, int K, int cus, int* waves_per_simd)
{
    const int simds = 4 * cus;
    int best = g.ny, best_w = (strips + simds - 1) / simds;
    uint64_t best_cost = (uint64_t)best_w * (uint64_t)(g.ny + 2 * K);
    for (int w = 1; w <= march_waves(K); ++w) {
        const int n = std::min(g.ny, simds * w / strips);
        if (n < 1) continue;
        const int rows = (g.ny + n - 1) / n;
        const uint64_t cost = (uint64_t)w * (uint64_t)(rows + 2 * K);
        if (cost < best_cost) {
            best_cost = cost;
            best = rows;
            best_w = w;
        }
    }
    if (waves_per_simd) *waves_per_simd = best_w;
    return best;
}

template <int ST, int V>
void launch_step_v(cmlbm2d_lattice* lat, hipStream_t s)
{
    using SS = storage2<ST>;
    using T = typename SS::T;
    const Geom2& g = lat->g;
    const auto* src = (const typename SS::S*)lat->pop[lat->cur];
    auto* dst = (typename SS::S*)lat->pop[1 - lat->cur];
    const T om = (T)(1.0 / lat->p.tau), r0 = (T)lat->p.rho0;
    if (lat->force_mode == CMLBM2D_FORCE_FIELD)
        k2_step<ST, V, true><<<dim3(g.nblk), dim3(kBlock), 0, s>>>(src, dst, g, om, r0, T(0), T(0),
                                                                    (const T*)lat->field);
    else
        k2_step<ST, V, false><<<dim3(g.nblk), dim3(kBlock), 0, s>>>(src, dst, g, om, r0, (T)lat->fu[0],
                                                                     (T)lat->fu[1], nullptr);
}

template <int ST>
void launch_step_st(cmlbm2d_lattice* lat, hipStream_t s)
{
    // vectors of at most 16 bytes per lane
    if constexpr (sizeof(typename storage2<ST>::S) <= 4) {
        if (lat->g.V == 4) return launch_step_v<ST, 4>(lat, s);
    }
    if (lat->g.V == 2) return launch_step_v<ST, 2>(lat, s);
    launch_step_v<ST, 1>(lat, s);
}

void launch_step(cmlbm2d_lattice* lat, hipStream_t s)
{
    switch (lat->p.storage) {
        case CMLBM2D_FP64: launch_step_st<CMLBM2D_FP64>(lat, s); break;
        case CMLBM2D_FP32: launch_step_st<CMLBM2D_FP32>(lat, s); break;
        case CMLBM2D_FP16: launch_step_st<CMLBM2D_FP16>(lat, s); break;
        default: launch_step_st<CMLBM2D_BF16>(lat, s); break;
    }
}

// K steps in one pass of k2_march.
template <int ST, int V, int K>
void launch_march_k(cmlbm2d_lattice* lat, hipStream_t s)
{
    using T = typename storage2<ST>::T;
    const Geom2& g = lat->g;
    const int strips = march_strips(g, V, march_halo(K)), rows = march_rows2(g, strips, K, lat->cus, nullptr);
    const uint64_t waves = (uint64_t)strips * (uint64_t)((g.ny + rows - 1) / rows);
    const dim3 grid((unsigned)((waves + kBlock / 64 - 1) / (kBlock / 64)));
    const T* src = (const T*)lat->pop[lat->cur];
    T* dst = (T*)lat->pop[1 - lat->cur];
    const T om = (T)(1.0 / lat->p.tau), r0 = (T)lat->p.rho0;
    if (lat->force_mode == CMLBM2D_FORCE_FIELD)
        k2_march<ST, V, K, true><<<grid, dim3(kBlock), 0, s>>>(src, dst, g, strips, rows, om, r0, T(0), T(0),
                                                               (const T*)lat->field);
    else
        k2_march<ST, V, K, false><<<grid, dim3(kBlock), 0, s>>>(src, dst, g, strips, rows, om, r0, (T)lat->fu[0],
                                                                (T)lat->fu[1], nullptr);
}

// Most steps of a k2_march pass: eight, and six with one FP32 cell a lane, which
// eight do not make faster (next_pass).
constexpr int march_most(bool f64, int V) { return f64 || V == 2 ? 8 : 6; }

// One pass of that many steps; false if there is none.
template <int ST, int V, int K = 2>
bool launch_march_v(cmlbm2d_lattice* lat, int steps, hipStream_t s)
{
    if constexpr (K <= march_most(ST == CMLBM2D_FP64, V)) {
        if (steps != K) return launch_march_v<ST, V, K + 2>(lat, steps, s);
        launch_march_k<ST, V, K>(lat, s);
        return true;
    }
    return false;
}

template <int ST>
void launch_tile(cmlbm2d_lattice* lat, int K, hipStream_t s)
{
    using T = typename storage2<ST>::T;
    const Geom2& g = lat->g;
    const int strips = march_strips(g, 1, K), R = kTileRows - 2 * K;
    const dim3 grid((unsigned)(strips * ((g.ny + R - 1) / R)));
    const T* src = (const T*)lat->pop[lat->cur];
    T* dst = (T*)lat->pop[1 - lat->cur];
    const T om = (T)(1.0 / lat->p.tau), r0 = (T)lat->p.rho0;
    if (lat->force_mode == CMLBM2D_FORCE_FIELD)
        k2_tile<ST, true><<<grid, dim3(kTileRows * 64), 0, s>>>(src, dst, g, K, strips, om, r0, T(0), T(0),
                                                                (const T*)lat->field);
    else
        k2_tile<ST, false><<<grid, dim3(kTileRows * 64), 0, s>>>(src, dst, g, K, strips, om, r0, (T)lat->fu[0],
                                                                 (T)lat->fu[1], nullptr);
}

// The next launch of a call with n steps left: how many steps, in which kernel.
struct Pass {
    enum Kind { STEP, MARCH, TILE } kind;
    int steps, V;
    double t;  // estimated us
};

// The first of the launches that take n steps in the least time, by estimates
// of each kernel's launch in us (measured, FP64 / FP32; the four-rolls mill on
// n x n cells):
//   k2_step   3.0 + 160 (80) bytes per cell at 5.6 TB/s (by 256 CUs);
//   k2_march  2.5 + waves per SIMD x (rows + 2 K) x the time of a row: K = 2
//             1.45 / 1.65 (HBM-bound), 4 1.75 / 2.15, 6 2.15 / 2.95, 8 2.6 / 3.8
//             (3.4 with two waves); FP32 with one cell a lane 0.97, 1.26, 1.69
//             and, no better than 6, 2.19;
//   k2_tile   with x = workgroups per CU: up to 1, 4.6 + 0.59 K + 3.7 x / 3.6 +
//             0.53 K + 3.7 x; beyond, 3.5 + 7.5 x / 3.5 + 3.9 x.
// The best rate decides while many steps are left, the best way to end exactly
// (6 + 4 for ten steps where 8 + 2 has the better start) over the last sixteen.
// parity 0 or 1: those n steps shall take an even or odd number of passes of an
// even number of steps (see cmlbm2d_step); -1: any.
// us per step, k2_step / chosen: FP64 16^2 3.06 / 1.23 (tile), 64^2 3.18 / 1.25
// (tile), 256^2 4.9 / 2.3 (tile), 500^2 9.3 / 5.8, 1024^2 30.9 / 11.8 (march),
// 4096^2 495 / 127, 8192^2 1873 / 489; FP32 64^2 3.4 / 1.04, 300^2 4.2 / 1.9, 1024^2
// 16.8 / 10.1, 4096^2 223 / 78 (march), 8192^2 890 / 270.
Pass next_pass(const cmlbm2d_lattice* lat, int n, int parity)
{
    constexpr int kMost = 8, kLast = 16;
    const Geom2& g = lat->g;
    const bool f64 = lat->p.storage == CMLBM2D_FP64;
    Pass of[kMost + 1];  // the fastest launch of k steps
    of[1] = Pass{Pass::STEP, 1, g.V, 3.0 + (double)g.ncell * (f64 ? 160.0 : 80.0) / (5.6e6 / 256.0 * lat->cus)};
    if ((!f64 && lat->p.storage != CMLBM2D_FP32) || n < 2) return of[1];
    for (int K = 2; K <= kMost; ++K) of[K] = Pass{Pass::STEP, 0, 1, 1e300};
    auto consider = [&](Pass::Kind kind, int K, int V, double t) {
        if (t < of[K].t) of[K] = Pass{kind, K, V, t};
    };
    const int V = f64 || g.nx % 2 ? 1 : 2;
    for (int K = 2; K <= march_most(f64, V); K += 2) {
        int w = 1;
        const int rows = march_rows2(g, march_strips(g, V, march_halo(K)), K, lat->cus, &w);
        const double per_row = f64      ? (K == 2 ? 1.45 : K == 4 ? 1.75 : K == 6 ? 2.15 : 2.6)
                               : V == 1 ? (K == 2 ? 0.97 : K == 4 ? 1.26 : 1.69)
                                        : (K == 2 ? 1.65 : K == 4 ? 2.15 : K == 6 ? 2.95 : w > 1 ? 3.4 : 3.8);
        consider(Pass::MARCH, K, V, 2.5 + w * (double)(rows + 2 * K) * per_row);
    }
    for (int K = 2; K <= 7; ++K) {
        const int R = kTileRows - 2 * K;
        const double x = (double)march_strips(g, 1, K) * ((g.ny + R - 1) / R) / lat->cus;
        if (x > 8192) break;  // far beyond its range, and near a launch's work-items
        const double t = x > 1.0 ? 3.5 + (f64 ? 7.5 : 3.9) * x : (f64 ? 4.6 + 0.59 * K : 3.6 + 0.53 * K) + 3.7 * x;
        consider(Pass::TILE, K, 1, t);
    }
    int first = 1;
    if (n > kLast) {
        for (int K = 2; K <= kMost; ++K)
            if (of[K].t * first < of[first].t * K) first = K;
        return of[first];
    }
    // least[m][q]: m steps, q the parity of their even passes (q = 0 where it is free)
    const int layers = parity < 0 ? 1 : 2;
    double least[kLast + 1][2] = {{0.0, 1e300}};
    for (int m = 1; m <= n; ++m)
        for (int q = 0; q < layers; ++q) {
            least[m][q] = 1e300;
            for (int K = 1; K <= kMost && K <= m; ++K) {
                const double t = of[K].t + least[m - K][layers == 2 && K % 2 == 0 ? 1 - q : q];
                if (t < least[m][q]) {
                    least[m][q] = t;
                    if (m == n && (layers == 1 || q == parity)) first = K;
                }
            }
        }
    return of[first];
}

// Whether calls on this lattice are in a HIP graph: noted by every entry that
// reads or writes the state on s (the null stream cannot be captured).
bool in_graph(cmlbm2d_lattice* lat, hipStream_t s)
{
    if (!lat->graph && s) {
        hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &status) != hipSuccess) (void)hipGetLastError();
        lat->graph = status == hipStreamCaptureStatusActive;
    }
    return lat->graph;
}

template <int ST>
bool launch_pass_st(cmlbm2d_lattice* lat, const Pass& p, hipStream_t s)
{
    if (p.kind == Pass::TILE) return launch_tile<ST>(lat, p.steps, s), true;
    if constexpr (ST == CMLBM2D_FP32) {
        if (p.V == 2) return launch_march_v<ST, 2>(lat, p.steps, s);
    }
    return launch_march_v<ST, 1>(lat, p.steps, s);
}

bool launch_pass(cmlbm2d_lattice* lat, const Pass& p, hipStream_t s)
{
    if (p.kind == Pass::STEP) return launch_step(lat, s), true;
    if (lat->p.storage == CMLBM2D_FP64) return launch_pass_st<CMLBM2D_FP64>(lat, p, s);
    return launch_pass_st<CMLBM2D_FP32>(lat, p, s);
}

template <int ST>
void launch_init_st(cmlbm2d_lattice* lat, int src_kind, const void* rho, const void* u, const double* pops,
                    hipStream_t s)
{
    using SS = storage2<ST>;
    auto* dst = (typename SS::S*)lat->pop[lat->cur];
    const Geom2& g = lat->g;
    if (src_kind == INIT_EQ_F64)
        k2_init<ST, INIT_EQ_F64><<<cell_grid(g), dim3(kBlock), 0, s>>>(dst, g, lat->p.rho0, rho, u, nullptr);
    else if (src_kind == INIT_EQ_F32)
        k2_init<ST, INIT_EQ_F32><<<cell_grid(g), dim3(kBlock), 0, s>>>(dst, g, lat->p.rho0, rho, u, nullptr);
    else
        k2_init<ST, INIT_POPS_F64><<<cell_grid(g), dim3(kBlock), 0, s>>>(dst, g, lat->p.rho0, nullptr, nullptr,
                                                                         pops);
}

void launch_init(cmlbm2d_lattice* lat, int src_kind, const void* rho, const void* u, const double* pops, hipStream_t s)
{
    switch (lat->p.storage) {
        case CMLBM2D_FP64: launch_init_st<CMLBM2D_FP64>(lat, src_kind, rho, u, pops, s); break;
        case CMLBM2D_FP32: launch_init_st<CMLBM2D_FP32>(lat, src_kind, rho, u, pops, s); break;
        case CMLBM2D_FP16: launch_init_st<CMLBM2D_FP16>(lat, src_kind, rho, u, pops, s); break;
        default: launch_init_st<CMLBM2D_BF16>(lat, src_kind, rho, u, pops, s); break;
    }
}

template <int ST>
void launch_gather_st(cmlbm2d_lattice* lat, void* rho, void* u, int out_f64, double* pops, hipStream_t s)
{
    using SS = storage2<ST>;
    const Geom2& g = lat->g;
    const void* field = lat->force_mode == CMLBM2D_FORCE_FIELD ? lat->field : nullptr;
    k2_gather<ST><<<cell_grid(g), dim3(kBlock), 0, s>>>((const typename SS::S*)lat->pop[lat->cur], g, lat->p.rho0,
                                                        lat->fu[0], lat->fu[1], field, rho, u, out_f64, pops);
}

void launch_gather(cmlbm2d_lattice* lat, void* rho, void* u, int out_f64, double* pops, hipStream_t s)
{
    switch (lat->p.storage) {
        case CMLBM2D_FP64: launch_gather_st<CMLBM2D_FP64>(lat, rho, u, out_f64, pops, s); break;
        case CMLBM2D_FP32: launch_gather_st<CMLBM2D_FP32>(lat, rho, u, out_f64, pops, s); break;
        case CMLBM2D_FP16: launch_gather_st<CMLBM2D_FP16>(lat, rho, u, out_f64, pops, s); break;
        default: launch_gather_st<CMLBM2D_BF16>(lat, rho, u, out_f64, pops, s); break;
    }
}

bool aligned256(const void* p) { return ((uintptr_t)p & 255u) == 0; }

}  // namespace

extern "C" {

int cmlbm2d_required_bytes(const cmlbm2d_params* params, size_t* pop_buffer_bytes)
{
    Geom2 g;
    size_t bytes = 0;
    const int rc = make_geom(params, &g, &bytes);
    if (rc) return rc;
    if (pop_buffer_bytes) *pop_buffer_bytes = bytes;
    return CMLBM2D_OK;
}

int cmlbm2d_create(const cmlbm2d_params* params, void* pop_a, size_t pop_a_bytes, void* pop_b, size_t pop_b_bytes,
                   cmlbm2d_lattice** out)
{
    if (!out) return CMLBM2D_EINVAL;
    *out = nullptr;
    Geom2 g;
    size_t bytes = 0;
    const int rc = make_geom(params, &g, &bytes);
    if (rc) return rc;
    if (!pop_a || !pop_b || pop_a == pop_b) return CMLBM2D_EINVAL;
    if (!aligned256(pop_a) || !aligned256(pop_b)) return CMLBM2D_EINVAL;
    if (pop_a_bytes < bytes || pop_b_bytes < bytes) return CMLBM2D_ENOMEM;
    cmlbm2d_lattice* lat = new (std::nothrow) cmlbm2d_lattice();
    if (!lat) return CMLBM2D_ENOMEM;
    lat->p = *params;
    lat->g = g;
    lat->pop[0] = pop_a;
    lat->pop[1] = pop_b;
    lat->cur = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&lat->cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        lat->cus < 1)
        lat->cus = 256;
    lat->force_mode = CMLBM2D_FORCE_NONE;
    lat->fu[0] = lat->fu[1] = 0.0;
    lat->field = nullptr;
    lat->initialized = false;
    lat->graph = false;
    lat->t = 0;
    *out = lat;
    return CMLBM2D_OK;
}

int cmlbm2d_set_force(cmlbm2d_lattice* lat, int mode, const double* host_values, const void* dev_field, int io_dtype,
                      void* hip_stream)
{
    (void)hip_stream;
    if (!lat) return CMLBM2D_EINVAL;
    switch (mode) {
        case CMLBM2D_FORCE_NONE:
            lat->fu[0] = lat->fu[1] = 0.0;
            lat->field = nullptr;
            break;
        case CMLBM2D_FORCE_UNIFORM:
            if (!host_values) return fail(lat, CMLBM2D_EINVAL, "UNIFORM force needs host_values[2]");
            if (!std::isfinite(host_values[0]) || !std::isfinite(host_values[1]))
                return fail(lat, CMLBM2D_EINVAL, "non-finite force");
            lat->fu[0] = host_values[0];
            lat->fu[1] = host_values[1];
            lat->field = nullptr;
            break;
        case CMLBM2D_FORCE_FIELD: {
            const int need = lat->p.storage == CMLBM2D_FP64 ? CMLBM2D_FP64 : CMLBM2D_FP32;
            if (!dev_field) return fail(lat, CMLBM2D_EINVAL, "FIELD force needs dev_field[2][N]");
            if (io_dtype != need)
                return fail(lat, CMLBM2D_EINVAL, "FIELD force dtype must be FP64 for FP64 storage, FP32 otherwise");
            if ((uintptr_t)dev_field & (need == CMLBM2D_FP64 ? 7u : 3u))
                return fail(lat, CMLBM2D_EINVAL, "FIELD force pointer misaligned");
            lat->fu[0] = lat->fu[1] = 0.0;
            lat->field = dev_field;
            break;
        }
        default: return fail(lat, CMLBM2D_EINVAL, "unknown force mode");
    }
    lat->force_mode = mode;
    return CMLBM2D_OK;
}

int cmlbm2d_init(cmlbm2d_lattice* lat, const void* dev_rho, const void* dev_u, int io_dtype, void* hip_stream)
{
    if (!lat) return CMLBM2D_EINVAL;
    if (io_dtype != CMLBM2D_FP64 && io_dtype != CMLBM2D_FP32)
        return fail(lat, CMLBM2D_EINVAL, "io_dtype must be FP64 or FP32");
    in_graph(lat, (hipStream_t)hip_stream);
    launch_init(lat, io_dtype == CMLBM2D_FP64 ? INIT_EQ_F64 : INIT_EQ_F32, dev_rho, dev_u, nullptr,
                (hipStream_t)hip_stream);
    const int rc = launch_check(lat, "init");
    if (rc) return rc;
    lat->initialized = true;
    lat->t = 0;
    return CMLBM2D_OK;
}

int cmlbm2d_step(cmlbm2d_lattice* lat, int32_t nsteps, void* hip_stream)
{
    if (!lat) return CMLBM2D_EINVAL;
    if (nsteps < 0) return fail(lat, CMLBM2D_EINVAL, "nsteps must be >= 0");
    if (!lat->initialized) return fail(lat, CMLBM2D_ESTATE, "step before init");
    hipStream_t s = (hipStream_t)hip_stream;
    // A graph keeps the buffers of its capture, so once a call is in one, the state
    // has to be where the number of steps alone puts it: an even number of steps
    // ends in the buffer it starts in.  A pass changes buffers once, so the passes
    // of an even number of steps then come in pairs.
    int parity = in_graph(lat, s) ? 0 : -1;
    for (int32_t k = 0; k < nsteps;) {
        const Pass p = next_pass(lat, nsteps - k, parity);
        if (parity >= 0 && p.steps % 2 == 0) parity = 1 - parity;
        if (!launch_pass(lat, p, s)) return fail(lat, CMLBM2D_EINVAL, "no kernel for a pass of these steps");
        const int rc = launch_check(lat, "step");
        if (rc) return rc;
        lat->cur = 1 - lat->cur;
        lat->t += p.steps;
        k += p.steps;
    }
    return CMLBM2D_OK;
}

int cmlbm2d_moments(cmlbm2d_lattice* lat, void* dev_rho, void* dev_u, int io_dtype, void* hip_stream)
{
    if (!lat) return CMLBM2D_EINVAL;
    if (io_dtype != CMLBM2D_FP64 && io_dtype != CMLBM2D_FP32)
        return fail(lat, CMLBM2D_EINVAL, "io_dtype must be FP64 or FP32");
    if (!lat->initialized) return fail(lat, CMLBM2D_ESTATE, "moments before init");
    if (!dev_rho && !dev_u) return CMLBM2D_OK;
    in_graph(lat, (hipStream_t)hip_stream);
    launch_gather(lat, dev_rho, dev_u, io_dtype == CMLBM2D_FP64, nullptr, (hipStream_t)hip_stream);
    return launch_check(lat, "moments");
}

int cmlbm2d_populations(cmlbm2d_lattice* lat, double* dev_out, void* hip_stream)
{
    if (!lat || !dev_out) return CMLBM2D_EINVAL;
    if (!lat->initialized) return fail(lat, CMLBM2D_ESTATE, "populations before init");
    in_graph(lat, (hipStream_t)hip_stream);
    launch_gather(lat, nullptr, nullptr, 1, dev_out, (hipStream_t)hip_stream);
    return launch_check(lat, "populations");
}

int cmlbm2d_load_populations(cmlbm2d_lattice* lat, const double* dev_in, void* hip_stream)
{
    if (!lat || !dev_in) return CMLBM2D_EINVAL;
    in_graph(lat, (hipStream_t)hip_stream);
    launch_init(lat, INIT_POPS_F64, nullptr, nullptr, dev_in, (hipStream_t)hip_stream);
    const int rc = launch_check(lat, "load populations");
    if (rc) return rc;
    lat->initialized = true;
    return CMLBM2D_OK;
}

int cmlbm2d_get_time(const cmlbm2d_lattice* lat, int64_t* t)
{
    if (!lat || !t) return CMLBM2D_EINVAL;
    *t = lat->t;
    return CMLBM2D_OK;
}

int cmlbm2d_destroy(cmlbm2d_lattice* lat)
{
    delete lat;
    return CMLBM2D_OK;
}

const char* cmlbm2d_last_error(const cmlbm2d_lattice* lat) { return lat ? lat->err.c_str() : ""; }

const char* cmlbm2d_status_string(int status)
{
    switch (status) {
        case CMLBM2D_OK: return "CMLBM2D_OK";
        case CMLBM2D_EINVAL: return "CMLBM2D_EINVAL";
        case CMLBM2D_ENOMEM: return "CMLBM2D_ENOMEM";
        case CMLBM2D_EHIP: return "CMLBM2D_EHIP";
        case CMLBM2D_ESTATE: return "CMLBM2D_ESTATE";
        default: return "CMLBM2D_UNKNOWN";
    }
}

}  // extern "C"
