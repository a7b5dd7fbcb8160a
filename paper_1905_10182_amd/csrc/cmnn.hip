// libcmnn: gfx950 kernels of the learned warm start (C ABI in include/cmnn.h).
//
// Convolutions are implicit GEMMs on v_mfma_f32_16x16x32_bf16.  Operand
// layout of that instruction (checked on the hardware): lane l holds
// A[l % 16][(l / 16) * 8 + i] and B[(l / 16) * 8 + i][l % 16] for i < 8, and
// receives D[(l / 16) * 4 + i][l % 16] for i < 4.
//
//   k_conv_fwd      y[v][co] = act(sum_t sum_ci x[v + s*off(t)][ci] w[t][co][ci] + b[co])
//                   (s = +1; the data gradient is the same kernel with s = -1 and
//                   the transposed weights).  A = 16 voxels x 32 input channels,
//                   one 16-byte load per lane; B = 32 channels x 16 outputs.
//   k_conv_bwd_w    dw[t][co][ci] = sum_v dy[v][co] x[v + off(t)][ci]: the voxel
//                   axis is the MFMA K axis, so 32-voxel tiles of dy and x are
//                   staged through LDS transposed (channel-major) and read back
//                   as 16-byte fragments; per-chunk partials, fixed-order sum.
#include <hip/hip_runtime.h>

#include <type_traits>

#include <cstdint>
#include <mutex>

#include "cmnn.h"

namespace {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

constexpr float kLeak = 0.1f;

struct G {
    int n, d, h, w;
    int per[3];
    long long nvox;
};

G make_g(const cmnn_geom* g)
{
    G r;
    r.n = g->n;
    r.d = g->d;
    r.h = g->h;
    r.w = g->w;
    for (int a = 0; a < 3; ++a) r.per[a] = g->periodic[a];
    r.nvox = (long long)g->n * g->d * g->h * g->w;
    return r;
}

// Positive extents and at most 2^31 - 1 voxels, so that every launch grid and
// per-voxel index fits the kernels' arithmetic.
bool geom_ok(const cmnn_geom* g)
{
    if (!g || g->n <= 0 || g->d <= 0 || g->h <= 0 || g->w <= 0) return false;
    return (long long)g->n * g->d * g->h * g->w <= 0x7fffffffLL;
}
bool chan_ok(int c) { return c > 0 && c % CMNN_CALIGN == 0; }
bool al16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

__device__ __forceinline__ bool shift_axis(int v, int dv, int n, int periodic, int& out)
{
    int s = v + dv;
    if (s < 0 || s >= n) {
        if (!periodic) return false;
        s = s < 0 ? s + n : s - n;
    }
    out = s;
    return true;
}

// Neighbour voxel of linear voxel m along tap t (sign s = +1 or -1); false if
// it falls into zero padding.
__device__ __forceinline__ bool neighbour(const G& g, long long m, int t, int s, long long& out)
{
    const int w = (int)(m % g.w);
    long long r = m / g.w;
    const int h = (int)(r % g.h);
    r /= g.h;
    const int d = (int)(r % g.d);
    const long long n = r / g.d;
    const int dz = s * (t / 9 - 1), dy = s * ((t / 3) % 3 - 1), dx = s * (t % 3 - 1);
    int nd, nh, nw;
    if (!shift_axis(d, dz, g.d, g.per[0], nd)) return false;
    if (!shift_axis(h, dy, g.h, g.per[1], nh)) return false;
    if (!shift_axis(w, dx, g.w, g.per[2], nw)) return false;
    out = ((n * g.d + nd) * g.h + nh) * g.w + nw;
    return true;
}

#define GRID_STRIDE(i, total) \
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < (total); i += (long long)gridDim.x * blockDim.x)

// The same with the index type I: the elementwise kernels below take 32-bit
// unsigned index arithmetic (a quarter of the 64-bit division's work) when
// every element index of the call fits, 64-bit otherwise.
#define GRID_STRIDE_I(I, i, total) \
    for (I i = (I)blockIdx.x * blockDim.x + threadIdx.x; i < (I)(total); i += (I)gridDim.x * blockDim.x)

__device__ __forceinline__ void unpack8(u4 v, float (&f)[8])
{
    const bf16x8 b = __builtin_bit_cast(bf16x8, v);
#pragma unroll
    for (int i = 0; i < 8; ++i) f[i] = (float)b[i];
}

__device__ __forceinline__ u4 pack8(const float (&f)[8])
{
    bf16x8 b;
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = (bf16)f[i];
    return __builtin_bit_cast(u4, b);
}

__device__ __forceinline__ bf16x8 ld8(const bf16* p) { return __builtin_bit_cast(bf16x8, *(const u4*)p); }

// Raw buffer loads of 16 bytes: a descriptor in four scalar registers
// (wave-uniform base, stride 0, size in bytes, the gfx9 raw-buffer format
// word) plus a 32-bit per-lane offset and a wave-uniform offset, added by the
// memory unit instead of by 64-bit VALU arithmetic.
constexpr int kRawBufferWord3 = 0x00020000;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, kRawBufferWord3);
}
__device__ __forceinline__ bf16x8 ldb8(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t uniform_off)
{
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, uniform_off, 0));
}

// ---------------------------------------------------------------------------
// forward convolution (and, with SIGN = -1, the data gradient)
//
// Workgroup = 4 waves = 64 consecutive voxels x (16 * NB) output channels;
// wave w owns voxels [16w, 16w + 16) and NB 16-channel output blocks.

// Epilogue of the convolution kernels.  SIGN = +1 (forward): v + bias, then
// the activation.  SIGN = -1 (data gradient) with ACT = LEAKY: the gradient is
// multiplied by the leaky-ReLU slope at the activation output `gate` (0.1
// where gate <= 0), i.e. it leaves as the producing layer's pre-activation
// gradient (the rule of k_act_bwd, applied before the BF16 rounding).
template <int SIGN, int ACT>
__device__ __forceinline__ float conv_out(float v, float bias, const bf16* __restrict__ gate, long long idx)
{
    if (SIGN > 0) {
        v += bias;
        if (ACT == CMNN_ACT_LEAKY) v = v > 0.f ? v : kLeak * v;
    } else if (ACT == CMNN_ACT_LEAKY) {
        if ((float)gate[idx] <= 0.f) v *= kLeak;
    }
    return v;
}

template <int NB, int SIGN, int ACT>
__global__ __launch_bounds__(256) void k_conv_fwd(G g, const bf16* __restrict__ x, int cin, const bf16* __restrict__ wt,
                                                  const float* __restrict__ bias, int cout, bf16* __restrict__ y,
                                                  const bf16* __restrict__ gate)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long m0 = (long long)blockIdx.x * 64 + wave * 16;
    const int co0 = blockIdx.y * 16 * NB;
    const long long mrow = m0 + (lane & 15);  // voxel of this lane's A row
    const int kq = lane >> 4;
    f4 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f4{0.f, 0.f, 0.f, 0.f};
    for (int t = 0; t < 27; ++t) {
        long long src = 0;
        const bool valid = mrow < g.nvox && neighbour(g, mrow, t, SIGN, src);
        const bf16* xp = x + src * cin + kq * 8;
        const bf16* wp = wt + ((long long)t * cout + co0 + (lane & 15)) * cin + kq * 8;
        for (int c0 = 0; c0 < cin; c0 += 32) {
            bf16x8 a;
            if (valid)
                a = ld8(xp + c0);
            else
                a = __builtin_bit_cast(bf16x8, u4{0u, 0u, 0u, 0u});
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const bf16x8 bw = ld8(wp + (long long)b * 16 * cin + c0);
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bw, acc[b], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int co = co0 + 16 * b + (lane & 15);
        const float bb = bias ? bias[co] : 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const long long m = m0 + kq * 4 + i;
            if (m >= g.nvox) continue;
            y[m * cout + co] = (bf16)conv_out<SIGN, ACT>(acc[b][i], bb, gate, m * cout + co);
        }
    }
}

// ---------------------------------------------------------------------------
// brick-tiled forward convolution (and data gradient), for extents that are
// multiples of the 4 x 4 x 16 (d, h, w) brick
//
// Workgroup = one brick of 256 output voxels x (16 * NB) output channels.
// Per 32-channel input chunk the brick's 6 x 6 x 18 halo is staged once in LDS
// (voxel stride 80 bytes: 16 consecutive voxels of a 16-byte fragment read
// land on distinct bank groups), and every one of the 27 taps takes its A
// fragments from there: each input value is fetched from memory once per
// brick instead of once per tap, and each halo row is read from LDS once for
// its three x taps (the x - 1 and x + 1 fragments are lane shifts of it).  Wave w owns the 4 brick rows (d, h) =
// (w, 0..3), i.e. 4 MFMA row blocks of 16 x-consecutive voxels, and keeps
// 4 x NB accumulator tiles: each B fragment (weights, through L1) feeds 4
// MFMAs and each A fragment (LDS) feeds NB.  The weight fragments are raw
// buffer loads (a loop-invariant lane offset plus a wave-uniform tap offset,
// no per-load address arithmetic); a tap group's second and third taps are
// loaded before its LDS reads and the next group's first tap during its first
// tap's MFMAs, so the load latency overlaps work.

// The A operand of v_mfma_f32_16x16x32_bf16 holds voxel row (lane % 16), so
// the fragment of the neighbouring x tap is the same fragment shifted by one
// lane within each 16-lane DPP row; the lane left without a source keeps
// `edge` (update_dpp with bound_ctrl off leaves it unwritten).
// rows_from_lower: lane l takes lane l - 1 (voxel x - 1), lane 0 keeps edge.
// rows_from_upper: lane l takes lane l + 1 (voxel x + 1), lane 15 keeps edge.
__device__ __forceinline__ bf16x8 rows_from_lower(bf16x8 edge, bf16x8 v)
{
    const u4 e = __builtin_bit_cast(u4, edge), a = __builtin_bit_cast(u4, v);
    u4 r;
    r.x = (unsigned)__builtin_amdgcn_update_dpp((int)e.x, (int)a.x, 0x111, 0xF, 0xF, false);  // row_shr:1
    r.y = (unsigned)__builtin_amdgcn_update_dpp((int)e.y, (int)a.y, 0x111, 0xF, 0xF, false);
    r.z = (unsigned)__builtin_amdgcn_update_dpp((int)e.z, (int)a.z, 0x111, 0xF, 0xF, false);
    r.w = (unsigned)__builtin_amdgcn_update_dpp((int)e.w, (int)a.w, 0x111, 0xF, 0xF, false);
    return __builtin_bit_cast(bf16x8, r);
}

__device__ __forceinline__ bf16x8 rows_from_upper(bf16x8 edge, bf16x8 v)
{
    const u4 e = __builtin_bit_cast(u4, edge), a = __builtin_bit_cast(u4, v);
    u4 r;
    r.x = (unsigned)__builtin_amdgcn_update_dpp((int)e.x, (int)a.x, 0x101, 0xF, 0xF, false);  // row_shl:1
    r.y = (unsigned)__builtin_amdgcn_update_dpp((int)e.y, (int)a.y, 0x101, 0xF, 0xF, false);
    r.z = (unsigned)__builtin_amdgcn_update_dpp((int)e.z, (int)a.z, 0x101, 0xF, 0xF, false);
    r.w = (unsigned)__builtin_amdgcn_update_dpp((int)e.w, (int)a.w, 0x101, 0xF, 0xF, false);
    return __builtin_bit_cast(bf16x8, r);
}

constexpr int kTD = 4, kTH = 4, kTW = 16;
constexpr int kHD = kTD + 2, kHH = kTH + 2, kHW = kTW + 2;
constexpr int kHalo = kHD * kHH * kHW;  // 648 voxels
constexpr int kVStride = 40;            // bf16 per staged voxel (32 channels + 8 pad)
constexpr uint32_t kVBytes = kVStride * 2;

constexpr int kStageIters = (kHalo * 4 + 255) / 256;

__device__ __forceinline__ void stage_halo_load(const G& g, const bf16* __restrict__ x, int cin, int c0, long long n,
                                                int d0, int h0, int x0, int tid, u4 stage[kStageIters])
{
#pragma unroll
    for (int it = 0; it < kStageIters; ++it) {
        const int p = tid + it * 256;
        const int hv = p >> 2, part = p & 3;
        const int hx = hv % kHW, hh = (hv / kHW) % kHH, hd = hv / (kHW * kHH);
        int sd = 0, sh = 0, sw = 0;
        stage[it] = u4{0u, 0u, 0u, 0u};
        if (p < kHalo * 4 && shift_axis(d0, hd - 1, g.d, g.per[0], sd) && shift_axis(h0, hh - 1, g.h, g.per[1], sh) &&
            shift_axis(x0, hx - 1, g.w, g.per[2], sw))
            stage[it] = *(const u4*)(x + (((n * g.d + sd) * g.h + sh) * g.w + sw) * cin + c0 + part * 8);
    }
}

template <int NB, int SIGN, int ACT>
__global__ __launch_bounds__(256) void k_conv_tile(G g, const bf16* __restrict__ x, int cin,
                                                   const bf16* __restrict__ wt, const float* __restrict__ bias,
                                                   int cout, bf16* __restrict__ y, unsigned xcd_span,
                                                   const bf16* __restrict__ gate)
{
    __shared__ __attribute__((aligned(16))) bf16 sx[kHalo * kVStride];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // blocks are dealt round-robin to the 8 XCDs: give each XCD a contiguous
    // run of bricks so that halo overlaps and weights share its L2
    unsigned bid = blockIdx.x;
    if (xcd_span) bid = (bid & 7u) * xcd_span + (bid >> 3);
    const int nbw = g.w / kTW, nbh = g.h / kTH, nbd = g.d / kTD;
    int r = (int)bid;
    const int x0 = (r % nbw) * kTW;
    r /= nbw;
    const int h0 = (r % nbh) * kTH;
    r /= nbh;
    const int d0 = (r % nbd) * kTD;
    const long long n = r / nbd;
    const int co0 = blockIdx.y * 16 * NB;
    f4 acc[4][NB];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[m][b] = f4{0.f, 0.f, 0.f, 0.f};
    // weights: one descriptor over the [27][cout][cin] tensor, this lane's
    // row / channel part as a loop-invariant lane offset, the tap, output
    // block and channel chunk as a wave-uniform offset
    const __amdgpu_buffer_rsrc_t wr = buf_rsrc(wt, 27u * (uint32_t)cout * (uint32_t)cin * 2u);
    const uint32_t wlane = ((uint32_t)(co0 + (lane & 15)) * (uint32_t)cin + (uint32_t)(lane >> 4) * 8u) * 2u;
    // halo staging: thread tid moves the 16-byte parts tid, tid + 256, ... of
    // the 648 x 4; all its loads are in flight together
    u4 stage[kStageIters];
    // LDS fragment reads: lane part of the centre row (voxel x = lane % 16 + 1
    // of the halo row) and of its edge voxel, 16-byte channel group lane / 16
    const char* sxb = (const char*)sx;
    const uint32_t lane_a = ((uint32_t)(lane & 15) + 1u) * kVBytes + (uint32_t)(lane >> 4) * 16u;
    const uint32_t lane_e = ((lane & 15) < 8 ? 0u : (uint32_t)(kHW - 1) * kVBytes) + (uint32_t)(lane >> 4) * 16u;
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    for (int c0 = 0; c0 < cin; c0 += 32) {
        stage_halo_load(g, x, cin, c0, n, d0, h0, x0, tid, stage);
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kStageIters; ++it) {
            const int p = tid + it * 256;
            if (p < kHalo * 4) *(u4*)&sx[(p >> 2) * kVStride + (p & 3) * 8] = stage[it];
        }
        __syncthreads();
        // weight fragments of tap t (NB output blocks); the first tap of the
        // next group is loaded one group ahead
        auto wload = [&](int t, bf16x8 bw[NB]) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
                bw[b] = ldb8(wr, wlane, (((uint32_t)t * (uint32_t)cout + 16u * b) * (uint32_t)cin + (uint32_t)c0) * 2u);
        };
        bf16x8 bnext[NB];
        wload(0, bnext);
#pragma unroll 1
        for (int t9 = 0; t9 < 9; ++t9) {
            const int dz = SIGN * (t9 / 3 - 1), dy = SIGN * (t9 % 3 - 1);
            bf16x8 bw[3][NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) bw[0][b] = bnext[b];
            wload(t9 * 3 + 1, bw[1]);
            wload(t9 * 3 + 2, bw[2]);
            // A fragments of the three x taps (index dx + 1) of each brick row:
            // 32-bit LDS byte offsets, the tap's row wave-uniform, the brick row
            // m an immediate
            const uint32_t trow = (uint32_t)(((wv + 1 + dz) * kHH + 1 + dy) * kHW) * kVBytes;
            bf16x8 af[4][3];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const uint32_t mrow = trow + (uint32_t)(m * kHW) * kVBytes;
                const bf16x8 a0 = *(const bf16x8*)(sxb + lane_a + mrow);
                const bf16x8 e = *(const bf16x8*)(sxb + lane_e + mrow);
                af[m][0] = rows_from_lower(e, a0);
                af[m][1] = a0;
                af[m][2] = rows_from_upper(e, a0);
            }
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int k = SIGN > 0 ? j : 2 - j;  // dx = SIGN * (j - 1)
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        acc[m][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[m][k], bw[j][b], acc[m][b], 0, 0, 0);
                if (j == 0 && t9 < 8) wload(t9 * 3 + 3, bnext);
            }
        }
    }
    // D[row][col]: row = voxel (lane / 16) * 4 + i of the block's x-row, col = output channel lane % 16.
    // The NB bias values are loaded together, before the stores (one wait instead of one per store group).
    float bbv[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) bbv[b] = bias ? bias[co0 + 16 * b + (lane & 15)] : 0.f;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const long long vrow = ((n * g.d + d0 + wave) * g.h + h0 + m) * g.w + x0;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int co = co0 + 16 * b + (lane & 15);
            const float bb = bbv[b];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const long long idx = (vrow + (lane >> 4) * 4 + i) * cout + co;
                y[idx] = (bf16)conv_out<SIGN, ACT>(acc[m][b][i], bb, gate, idx);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// row-tiled forward convolution (and data gradient), for extents that are
// multiples of 4 x 8 x 16 (d, h, w)
//
// Workgroup = a brick of 512 output voxels x 32 output channels; wave w owns
// depth slice w, eight rows of 16 x-consecutive voxels.  Per 32-channel input
// chunk the 6 x 10 x 18 halo is staged in LDS, 64 bytes per voxel with the
// 16-byte channel groups XOR-swizzled by (x / 2) mod 4 (eight consecutive
// voxels of a fragment read then cover all banks without padding, and two
// workgroups fit a CU).  For each of the three depth taps a wave holds the nine
// (dy, dx) weight fragments in registers and walks down the ten halo rows once:
// a row is read once per x tap and feeds up to 18 MFMAs, those of the three
// output rows it is a neighbour of.
// Against the 4 x 4 x 16 brick kernel, which is bound by its weight reads from
// L1 and by the vector instructions between MFMAs, this reads the weights half
// as often per voxel and the halo 0.83 times, finds the halo rows' sources once
// per workgroup instead of once per thread and part, and writes four
// consecutive channels of a voxel per lane (8-byte stores: the weights are the
// first MFMA operand).  The x - 1 and x + 1 fragments are LDS reads of their
// own: built from the centre one by lane shifts they cost as much issue time as
// the MFMAs (75 us instead of 66).  Each output adds its products in the order
// of the brick kernel: same bits.
// What waits on memory at the start of a workgroup is issued together: the gates
// and the first row's weights with the halo (forward 65 -> 60 us; all nine
// weights early, or the gates kept with them, run out of registers: 87 us).
// us, brick kernel / this, repeated on the same tensors, 16 x 32 x 32 x 64: 32 -> 32
// forward 77 / 52, data gradient 76 / 50, gated 81 / 57; 96 -> 32 201 / 153; 32 -> 96
// 187 / 147; 160 -> 64 at half extents 79 / 64 and its data gradient 131 / 78.  In a
// training step 32 -> 32 takes 59 forward and 61 gated (950 TFLOP/s).
constexpr int kRH = 8, kRHH = kRH + 2, kRRows = kHD * kRHH;  // 60 halo rows of 18 voxels
constexpr uint32_t kRRow = kHW * 64;                          // bytes of a halo row
constexpr int kRParts = kHW * 4;                              // 16-byte parts of a halo row: 72
constexpr int kRIters = kRRows / 3;                           // three rows are staged at a time, by 216 threads
constexpr uint32_t kNone = 0xffffff00u;                       // past every buffer range: loads give 0

// f > 0 ? f : kLeak f, as the larger of the two (0 < kLeak < 1)
__device__ __forceinline__ float leaky(float f)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(f), "v"(kLeak * f));
    return r;
}

template <int SIGN, int ACT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_conv_rows(
    G g, const bf16* __restrict__ x, int cin, const bf16* __restrict__ wt, const float* __restrict__ bias, int cout,
    bf16* __restrict__ y, unsigned xcd_span, const bf16* __restrict__ gate)
{
    typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    __shared__ __attribute__((aligned(128))) char sx[kRRows * kRRow];
    __shared__ uint32_t row_off[kRRows];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // blocks are dealt round-robin to the 8 XCDs: each XCD gets a contiguous
    // run of (brick, output block) pairs, the blocks of a brick together
    unsigned bid = blockIdx.x;
    if (xcd_span) bid = (bid & 7u) * xcd_span + (bid >> 3);
    const int ncb = cout / 32;
    const int co0 = (int)(bid % ncb) * 32;
    int r0 = (int)(bid / ncb);
    const int nbw = g.w / kTW, nbh = g.h / kRH, nbd = g.d / kTD;
    const int x0 = (r0 % nbw) * kTW;
    r0 /= nbw;
    const int h0 = (r0 % nbh) * kRH;
    r0 /= nbh;
    const int d0 = (r0 % nbd) * kTD;
    const long long n = r0 / nbd;
    // halo staging: the source offset of each row within the sample (kNone
    // where it is padding) once per workgroup; a thread keeps one voxel column
    // and channel part
    auto source = [](int v, int q, int ext, int periodic, bool& out) -> int {
        const int t = v + q - 1, w = t < 0 ? t + ext : t >= ext ? t - ext : t;
        out |= t != w && !periodic;
        return w;
    };
    if (tid < kRRows) {
        bool out = false;
        const int sd = source(d0, tid / kRHH, g.d, g.per[0], out), sh = source(h0, tid % kRHH, g.h, g.per[1], out);
        row_off[tid] = out ? kNone : (uint32_t)(sd * g.h + sh) * (uint32_t)g.w * (uint32_t)cin * 2u;
    }
    const int trow = tid / kRParts, hx = (tid - trow * kRParts) >> 2, part = tid & 3;
    uint32_t col_off;
    {
        bool out = trow >= 3;
        const int sw = source(x0, hx, g.w, g.per[2], out);
        col_off = out ? kNone : ((uint32_t)sw * (uint32_t)cin + (uint32_t)part * 8u) * 2u;
    }
    char* const put = sx + trow * kRRow + hx * 64 + ((part ^ ((hx >> 1) & 3)) << 4);
    const uint32_t sample = (uint32_t)g.d * (uint32_t)g.h * (uint32_t)g.w * (uint32_t)cin * 2u;
    const __amdgpu_buffer_rsrc_t xr = buf_rsrc(x + n * (long long)(sample / 2u), sample);
    const __amdgpu_buffer_rsrc_t wr = buf_rsrc(wt, 27u * (uint32_t)cout * (uint32_t)cin * 2u);
    const uint32_t wlane = ((uint32_t)(co0 + (lane & 15)) * (uint32_t)cin + (uint32_t)(lane >> 4) * 8u) * 2u;
    // this lane's output channels co + 16 b + i
    const int co = co0 + (lane >> 4) * 4;
    f4 bb[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
    if (SIGN > 0 && bias) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) bb[b][i] = bias[co + 16 * b + i];
    }
    // D[row][col]: row = output channel (lane / 16) * 4 + i, col = voxel lane % 16;
    // a lane offset and a wave-uniform offset within the sample.  The gates are
    // read ahead of the products.
    const uint32_t sample_y = (uint32_t)g.d * (uint32_t)g.h * (uint32_t)g.w * (uint32_t)cout * 2u;
    const __amdgpu_buffer_rsrc_t yr = buf_rsrc(y + n * (long long)(sample_y / 2u), sample_y);
    const __amdgpu_buffer_rsrc_t gr = buf_rsrc(gate + n * (long long)(sample_y / 2u), sample_y);
    const uint32_t ylane = ((uint32_t)(lane & 15) * (uint32_t)cout + (uint32_t)co) * 2u;
    auto yrow = [&](int m) { return (uint32_t)(((d0 + wv) * g.h + h0 + m) * g.w + x0) * (uint32_t)cout * 2u; };
    u2 gt[kRH][2];
    if (SIGN < 0 && ACT == CMNN_ACT_LEAKY) {
#pragma unroll
        for (int m = 0; m < kRH; ++m)
#pragma unroll
            for (int b = 0; b < 2; ++b) gt[m][b] = __builtin_amdgcn_raw_buffer_load_b64(gr, ylane, yrow(m) + 32u * b, 0);
    }
    f4 acc[kRH][2];
#pragma unroll
    for (int m = 0; m < kRH; ++m) acc[m][0] = acc[m][1] = f4{0.f, 0.f, 0.f, 0.f};
    // LDS fragment reads: voxel x = lane % 16 + dx of a halo row, dx = 0, 1, 2
    uint32_t lane_a[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const uint32_t vx = (uint32_t)(lane & 15) + (uint32_t)k, grp = (uint32_t)(lane >> 4);
        lane_a[k] = vx * 64u + ((grp ^ ((vx >> 1) & 3u)) << 4);
    }
    __syncthreads();
    for (int c0 = 0; c0 < cin; c0 += 32) {
        u4 stage[kRIters];
#pragma unroll
        for (int it = 0; it < kRIters; ++it) {
            const uint32_t row = row_off[(it * 3 + trow) % kRRows];
            stage[it] = __builtin_bit_cast(u4, ldb8(xr, __builtin_elementwise_add_sat(row, col_off), (uint32_t)c0 * 2u));
        }
        // weight fragments of (depth tap tz, row tap ty): reloaded in place for
        // tz + 1 as soon as the last row that needs them is done, so that a
        // row or two of MFMAs covers the load.  The order is pinned per row:
        // left to itself the compiler sinks each load to its first use.
        bf16x8 bw[9][2];
        auto wload = [&](int tz, int ty) {
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    bw[ty * 3 + j][b] = ldb8(wr, wlane, (((uint32_t)(tz * 9 + ty * 3 + j) * (uint32_t)cout + 16u * b) * (uint32_t)cin + (uint32_t)c0) * 2u);
        };
        wload(0, 0);  // the first row's, behind the halo's loads
        __syncthreads();
        if (trow < 3) {
#pragma unroll
            for (int it = 0; it < kRIters; ++it) *(u4*)(put + it * 3 * kRRow) = stage[it];
        }
        __syncthreads();
        wload(0, 1);
        wload(0, 2);
        bf16x8 af[2][3];
        auto row_load = [&](int s30) {  // row s30 % 10 of depth tap s30 / 10
            const int dz = SIGN * (s30 / kRHH - 1), r = SIGN > 0 ? s30 % kRHH : kRHH - 1 - s30 % kRHH;
            const char* row = sx + (uint32_t)((wv + 1 + dz) * kRHH + r) * kRRow;
#pragma unroll
            for (int k = 0; k < 3; ++k) af[s30 & 1][k] = *(const bf16x8*)(row + lane_a[k]);
        };
        row_load(0);
#pragma unroll
        for (int s30 = 0; s30 < 3 * kRHH; ++s30) {
            const int tz = s30 / kRHH, rr = s30 % kRHH, r = SIGN > 0 ? rr : kRHH - 1 - rr;
            if (s30 + 1 < 3 * kRHH) row_load(s30 + 1);
            if (tz < 2 && rr >= kRH) wload(tz + 1, rr - kRH);  // ty = 0 after its last row, 1 after its last
            if (tz > 0 && rr == 0) wload(tz, 2);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int ty = 0; ty < 3; ++ty) {
                    const int m = r - 1 - SIGN * (ty - 1);
                    if (m < 0 || m >= kRH) continue;
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        acc[m][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            bw[ty * 3 + j][b], af[s30 & 1][SIGN > 0 ? j : 2 - j], acc[m][b], 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int m = 0; m < kRH; ++m) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            bf16x4 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float f = acc[m][b][i];
                if (SIGN > 0) {
                    f += bb[b][i];
                    if (ACT == CMNN_ACT_LEAKY) f = leaky(f);
                } else if (ACT == CMNN_ACT_LEAKY) {
                    if ((float)__builtin_bit_cast(bf16x4, gt[m][b])[i] <= 0.f) f *= kLeak;
                }
                o[i] = (bf16)f;
            }
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, o), yr, ylane, yrow(m) + 32u * b, 0);
        }
    }
}

// ---------------------------------------------------------------------------
// forward convolution (and data gradient) for grids that leave CUs idle
//
// Workgroup = a 4 x 4 x 16 brick x 32 output channels; wave w owns depth slice w
// and walks down the halo rows as in the row kernel.  Here the weights go through
// LDS: read from L1 by every wave, the nine taps' 32 rows of a depth tap (half
// lines where cin is a multiple of 64) do not fit it, and each wave fetches them
// from L2.  With one workgroup on a CU nothing else covers a load, so the
// weights of a depth tap are loaded two taps ahead and the next channels' halo
// a chunk ahead; two buffers each, one barrier per depth tap.  No load is under
// a branch: what there is not to load has an offset past its buffer's range.
// Products are added in the order of the brick kernel: same bits.
// us, brick kernel / this: 192 -> 96 channels at 16 x 8 x 8 x 16 47 / 28, 64 -> 96 19.5 /
// 11.9, 96 -> 96 21 / 16; 64 -> 64 at 4 x 16 x 16 x 32 20.5 / 13.0, at 1 x 16 x 16 x 32 12.7 /
// 11.2; 32 -> 32 at 1 x 32 x 32 x 64 10.5 / 8.7.  The same with the weights read from L1
// into two register sets, or with twelve waves a brick: 47 and 47.
constexpr int kFH = kTH + 2, kFRows = kHD * kFH, kFIters = kFRows / 3;

template <int SIGN, int ACT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2))) void k_conv_few(
    G g, const bf16* __restrict__ x, int cin, const bf16* __restrict__ wt, const float* __restrict__ bias, int cout,
    bf16* __restrict__ y, const bf16* __restrict__ gate)
{
    typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    __shared__ __attribute__((aligned(128))) char sx[2][kFRows * kRRow];
    __shared__ __attribute__((aligned(128))) char sw[2][9 * 32 * 64];
    __shared__ uint32_t row_off[kFRows];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ncb = cout / 32;
    const int co0 = (int)(blockIdx.x % ncb) * 32;
    int r0 = (int)(blockIdx.x / ncb);
    const int nbw = g.w / kTW, nbh = g.h / kTH, nbd = g.d / kTD;
    const int x0 = (r0 % nbw) * kTW;
    r0 /= nbw;
    const int h0 = (r0 % nbh) * kTH;
    r0 /= nbh;
    const int d0 = (r0 % nbd) * kTD;
    const long long n = r0 / nbd;
    auto source = [](int v, int q, int ext, int periodic, bool& out) -> int {
        const int t = v + q - 1, w = t < 0 ? t + ext : t >= ext ? t - ext : t;
        out |= t != w && !periodic;
        return w;
    };
    if (tid < kFRows) {
        bool out = false;
        const int sd = source(d0, tid / kFH, g.d, g.per[0], out), sh = source(h0, tid % kFH, g.h, g.per[1], out);
        row_off[tid] = out ? kNone : (uint32_t)(sd * g.h + sh) * (uint32_t)g.w * (uint32_t)cin * 2u;
    }
    const int trow = tid / kRParts, hx = (tid - trow * kRParts) >> 2, part = tid & 3;
    uint32_t col_off;
    {
        bool out = trow >= 3;
        const int sw = source(x0, hx, g.w, g.per[2], out);
        col_off = out ? kNone : ((uint32_t)sw * (uint32_t)cin + (uint32_t)part * 8u) * 2u;
    }
    const uint32_t put = trow * kRRow + hx * 64 + ((part ^ ((hx >> 1) & 3)) << 4);
    const uint32_t sample = (uint32_t)g.d * (uint32_t)g.h * (uint32_t)g.w * (uint32_t)cin * 2u;
    const __amdgpu_buffer_rsrc_t xr = buf_rsrc(x + n * (long long)(sample / 2u), sample);
    const __amdgpu_buffer_rsrc_t wr = buf_rsrc(wt, 27u * (uint32_t)cout * (uint32_t)cin * 2u);
    const int co = co0 + (lane >> 4) * 4;  // this lane's output channels co + 16 b + i
    const uint32_t sample_y = (uint32_t)g.d * (uint32_t)g.h * (uint32_t)g.w * (uint32_t)cout * 2u;
    const __amdgpu_buffer_rsrc_t yr = buf_rsrc(y + n * (long long)(sample_y / 2u), sample_y);
    const __amdgpu_buffer_rsrc_t gr = buf_rsrc(gate + n * (long long)(sample_y / 2u), sample_y);
    const uint32_t ylane = ((uint32_t)(lane & 15) * (uint32_t)cout + (uint32_t)co) * 2u;
    auto yrow = [&](int m) { return (uint32_t)(((d0 + wv) * g.h + h0 + m) * g.w + x0) * (uint32_t)cout * 2u; };
    uint32_t lane_a[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const uint32_t vx = (uint32_t)(lane & 15) + (uint32_t)k, grp = (uint32_t)(lane >> 4);
        lane_a[k] = vx * 64u + ((grp ^ ((vx >> 1) & 3u)) << 4);
    }
    u4 stage[kFIters];
    auto halo = [&](int c) {
        const uint32_t col = c < cin ? col_off : kNone;
#pragma unroll
        for (int it = 0; it < kFIters; ++it)
            stage[it] = __builtin_bit_cast(u4, ldb8(xr, __builtin_elementwise_add_sat(row_off[(it * 3 + trow) % kFRows], col), (uint32_t)c * 2u));
    };
    // weights: rows (tap of the depth tap, output channel) of 32 input channels,
    // four threads a row, parts swizzled as the halo's are
    constexpr int kWIters = (9 * 32 * 4 + 255) / 256;
    u4 ws[kWIters];
    const int wco = tid >> 2 & 31, wt0 = tid >> 7;  // tap wt0 + 2 it
    const uint32_t wthr = ((uint32_t)(wt0 * cout + co0 + wco) * (uint32_t)cin + (uint32_t)part * 8u) * 2u;
    const uint32_t wput = (uint32_t)((tid >> 2) * 64) + ((uint32_t)(part ^ (wco >> 1 & 3)) << 4);
    auto weights = [&](int c, int tz) {
#pragma unroll
        for (int it = 0; it < kWIters; ++it)
            ws[it] = __builtin_bit_cast(u4, ldb8(wr, c < cin && wt0 + 2 * it < 9 ? wthr : kNone,
                                                 ((uint32_t)((tz * 9 + 2 * it) * cout) * (uint32_t)cin + (uint32_t)c) * 2u));
    };
    auto put_weights = [&](int set) {
#pragma unroll
        for (int it = 0; it < kWIters; ++it)
            if (wt0 + 2 * it < 9) *(u4*)(sw[set] + wput + it * (2 * 32 * 64)) = ws[it];
    };
    uint32_t lane_w[2];  // fragment reads: output channel lane % 16 of each block
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const uint32_t c = (uint32_t)(lane & 15) + 16u * b;
        lane_w[b] = c * 64u + ((((uint32_t)lane >> 4) ^ (c >> 1 & 3u)) << 4);
    }
    __syncthreads();
    halo(0);
    weights(0, 0);
    f4 bb[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
    if (SIGN > 0 && bias) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) bb[b][i] = bias[co + 16 * b + i];
    }
    u2 gt[kTH][2];
    if (SIGN < 0 && ACT == CMNN_ACT_LEAKY) {
#pragma unroll
        for (int m = 0; m < kTH; ++m)
#pragma unroll
            for (int b = 0; b < 2; ++b) gt[m][b] = __builtin_amdgcn_raw_buffer_load_b64(gr, ylane, yrow(m) + 32u * b, 0);
    }
    f4 acc[kTH][2];
#pragma unroll
    for (int m = 0; m < kTH; ++m) acc[m][0] = acc[m][1] = f4{0.f, 0.f, 0.f, 0.f};
    auto store = [&](char* to) {
        if (trow < 3) {
#pragma unroll
            for (int it = 0; it < kFIters; ++it) *(u4*)(to + put + it * 3 * kRRow) = stage[it];
        }
    };
    store(sx[0]);
    put_weights(0);
    weights(0, 1);
    __syncthreads();
    auto chunk = [&](int c0, auto par) {  // par: the set of its first depth tap, and its LDS buffer
        constexpr int P = decltype(par)::value;
#pragma unroll
        for (int tz = 0; tz < 3; ++tz) {
            const int dz = SIGN * (tz - 1);
            put_weights((P + tz + 1) & 1);  // of the next depth tap
            weights(tz == 0 ? c0 : c0 + 32, tz == 0 ? 2 : tz - 1);
            if (tz == 0) halo(c0 + 32);
            bf16x8 bw[9][2];
            auto frag = [&](int ty) {
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int b = 0; b < 2; ++b) bw[ty * 3 + j][b] = *(const bf16x8*)(sw[(P + tz) & 1] + (ty * 3 + j) * (32 * 64) + lane_w[b]);
            };
            frag(0);
            bf16x8 af[2][3];
            auto row_load = [&](int rr) {
                const int r = SIGN > 0 ? rr : kFH - 1 - rr;
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    af[rr & 1][k] = *(const bf16x8*)(sx[P] + (uint32_t)((wv + 1 + dz) * kFH + r) * kRRow + lane_a[k]);
            };
            row_load(0);
            frag(1);
            frag(2);
#pragma unroll
            for (int rr = 0; rr < kFH; ++rr) {
                const int r = SIGN > 0 ? rr : kFH - 1 - rr;
                if (rr + 1 < kFH) row_load(rr + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int ty = 0; ty < 3; ++ty) {
                        const int m = r - 1 - SIGN * (ty - 1);
                        if (m < 0 || m >= kTH) continue;
#pragma unroll
                        for (int b = 0; b < 2; ++b)
                            acc[m][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                bw[ty * 3 + j][b], af[rr & 1][SIGN > 0 ? j : 2 - j], acc[m][b], 0, 0, 0);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (tz == 2) store(sx[P ^ 1]);
            __syncthreads();
        }
    };
    for (int c0 = 0; c0 < cin; c0 += 64) {
        chunk(c0, std::integral_constant<int, 0>{});
        if (c0 + 32 >= cin) break;
        chunk(c0 + 32, std::integral_constant<int, 1>{});
    }
#pragma unroll
    for (int m = 0; m < kTH; ++m) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            bf16x4 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float f = acc[m][b][i];
                if (SIGN > 0) {
                    f += bb[b][i];
                    if (ACT == CMNN_ACT_LEAKY) f = leaky(f);
                } else if (ACT == CMNN_ACT_LEAKY) {
                    if ((float)__builtin_bit_cast(bf16x4, gt[m][b])[i] <= 0.f) f *= kLeak;
                }
                o[i] = (bf16)f;
            }
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, o), yr, ylane, yrow(m) + 32u * b, 0);
        }
    }
}

// ---------------------------------------------------------------------------
// weight gradient
//
// Workgroup (chunk, tap, co tile of 32, ci tile of 32) accumulates over the
// chunk's voxels in steps of 32: 128 threads stage dy[32 voxels][32 co] and
// 128 stage x[32 shifted voxels][32 ci] into LDS transposed ([channel][voxel],
// rows padded to 40 elements = 80 bytes, 16-byte aligned); wave w then
// computes the 16 x 16 block (co block w / 2, ci block w % 2).

constexpr int kLdsRow = 40;

__global__ __launch_bounds__(256) void k_conv_bwd_w(G g, const bf16* __restrict__ x, int cin,
                                                    const bf16* __restrict__ dy, int cout, long long chunk,
                                                    float* __restrict__ part)
{
    __shared__ __attribute__((aligned(16))) bf16 sdy[32 * kLdsRow];
    __shared__ __attribute__((aligned(16))) bf16 sx[32 * kLdsRow];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ct = cout / 32, it = cin / 32;
    int bid = blockIdx.x;
    const int cit = bid % it;
    bid /= it;
    const int cot = bid % ct;
    bid /= ct;
    const int t = bid % 27;
    const long long ch = bid / 27;
    const long long v0 = ch * chunk;
    const long long v1 = v0 + chunk < g.nvox ? v0 + chunk : g.nvox;
    // staging role: threads 0..127 load dy, 128..255 load x; each 16 bytes (8 channels) of one voxel
    const int st = tid & 127, sv = st >> 2, sc = (st & 3) * 8;
    f4 acc = f4{0.f, 0.f, 0.f, 0.f};
    const int cob = wave >> 1, cib = wave & 1;
    for (long long vb = v0; vb < v1; vb += 32) {
        const long long v = vb + sv;
        bf16x8 e = __builtin_bit_cast(bf16x8, u4{0u, 0u, 0u, 0u});
        if (tid < 128) {
            if (v < v1) e = ld8(dy + v * cout + cot * 32 + sc);
#pragma unroll
            for (int i = 0; i < 8; ++i) sdy[(sc + i) * kLdsRow + sv] = e[i];
        } else {
            long long s;
            if (v < v1 && neighbour(g, v, t, 1, s)) e = ld8(x + s * cin + cit * 32 + sc);
#pragma unroll
            for (int i = 0; i < 8; ++i) sx[(sc + i) * kLdsRow + sv] = e[i];
        }
        __syncthreads();
        const bf16x8 a = *(const bf16x8*)&sdy[(cob * 16 + (lane & 15)) * kLdsRow + (lane >> 4) * 8];
        const bf16x8 b = *(const bf16x8*)&sx[(cib * 16 + (lane & 15)) * kLdsRow + (lane >> 4) * 8];
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
        __syncthreads();
    }
    // D[co][ci]: row (lane/16)*4 + i, column lane % 16
    float* p = part + ((ch * 27 + t) * (long long)cout) * cin;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int co = cot * 32 + cob * 16 + (lane >> 4) * 4 + i;
        const int ci = cit * 32 + cib * 16 + (lane & 15);
        p[(long long)co * cin + ci] = acc[i];
    }
}

// ---------------------------------------------------------------------------
// brick-tiled weight gradient (extents multiples of the 4 x 4 x 16 brick)
//
// Workgroup (chunk of bricks, 32 output channels, 32 input channels), all 27
// taps, 12 waves (three per SIMD).  The MFMA K axis is the voxel axis: a
// fragment is 8 consecutive voxels of one channel.  Per brick, dy (256 voxels)
// and the 6 x 6 x 18 halo of x are staged in LDS as they lie in memory, voxel by
// voxel, 16 channels (32 bytes) apart in two halves, and the fragments are read
// by the transposing LDS read (four voxels of 16 channels per 16 lanes: 128
// consecutive bytes, at any x shift).  A wave owns a depth
// tap, a 16-channel half of x and two of the brick's depth slices (K = the two
// slices' rows), and walks down the six halo rows: each is read once, its
// three x taps are byte shifts of the 12 voxels read, and it meets the up to
// three dy rows it is a neighbour of, 18 MFMAs.  The two waves that share taps
// add up through LDS at the end.  The bias gradient is summed from
// the dy fragments of two of the waves.
// What bounds it: the matrix cores run 52% of the time; the rest is LDS reads (17
// KB a wave and brick, half of the MFMAs' time) and the one barrier a brick.  Two
// buffers alternate and the next brick's loads are in flight meanwhile.
// Against staging channel-major (an 8 x 8 register transpose per task, 16-byte
// LDS stores with bank conflicts, eight waves with 3, 3, 2, .. units each), with
// the chunk sums: 16 x 32 x 32 x 64, 32 x 32 channels 78 -> 64 us, 96 x 32 215 -> 171 us
// (1015 TFLOP/s), 160 x 64 at half extents 103 -> 84 us.

constexpr int kBwThreads = 768;
// Voxels 8 and up of a row lie four slots further on: the two octets of a row
// that 32 lanes read at a time then fall on different banks.
constexpr uint32_t kBwXRow = 22 * 32, kBwYRow = 20 * 32;          // bytes of a row: 18 and 16 voxels
constexpr uint32_t kBwXHalf = kHD * kHH * kBwXRow + 64;           // halves 64 bytes out of step with the banks;
constexpr uint32_t kBwYHalf = kTD * kTH * kBwYRow + 64;           // (also the two voxels read past the last row)
constexpr uint32_t kBwBuf = 2 * kBwXHalf + 2 * kBwYHalf;
constexpr int kBwRows = kHD * kHH;                                // halo rows: 36
constexpr int kBwStep = kBwThreads / (kHW * 4);                   // halo rows staged at a time: 10

__global__ __launch_bounds__(kBwThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_conv_bwd_w_tile(G g, const bf16* __restrict__ x, int cin,
                                                                const bf16* __restrict__ dy, int cout,
                                                                int bricks_per_chunk, float* __restrict__ part,
                                                                long long pstride, bool bias)
{
    typedef short s4 __attribute__((ext_vector_type(4)));
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) s4 lds_s4;
    __shared__ __attribute__((aligned(128))) char lds[2 * kBwBuf];
    __shared__ uint32_t row_off[2][kBwRows];
    static_assert((6 * 18 + 2) * 64 * sizeof(f4) <= sizeof(lds), "the sums of half the waves");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ct = cout / 32, it = cin / 32;
    int bid = blockIdx.x;
    const int cit = bid % it;
    bid /= it;
    const int cot = bid % ct;
    const int ch = bid / ct;
    const int nbw = g.w / kTW, nbh = g.h / kTH, nbd = g.d / kTD;
    const long long nbricks = (long long)g.n * nbd * nbh * nbw;
    const long long b0 = (long long)ch * bricks_per_chunk;
    const long long b1 = b0 + bricks_per_chunk < nbricks ? b0 + bricks_per_chunk : nbricks;
    // Staging: five 16-byte parts per thread, four consecutive threads a voxel.
    // Rounds 0 to 3 are ten halo rows each (round 3: the last six), the waves
    // from 7 on in round 3 and the first eleven in round 4 take dy.  The halo rows' sources
    // (byte offset within the sample, kNone where it is padding) are found once
    // per brick, by one wave, a brick ahead of their use.
    const int trow = tid / (kHW * 4), hx = tid % (kHW * 4) >> 2, tp = tid & 3;
    const bool all4 = trow < kBwStep, r3x = trow < kBwRows - 3 * kBwStep, r3y = wave >= 7, r4 = wave < 11;
    auto slot = [](int v) { return (uint32_t)(v + (v >= 8 ? 4 : 0)) * 32u; };
    const uint32_t put_x = (uint32_t)(tp >> 1) * kBwXHalf + (uint32_t)trow * kBwXRow + slot(hx) + (uint32_t)(tp & 1) * 16u;
    const int yv3 = r3y ? (tid - 448) >> 2 : 0, yv4 = r4 ? 80 + (tid >> 2) : 0;  // dy voxels of rounds 3 and 4
    auto put_y = [&](int v) {
        return 2 * kBwXHalf + (uint32_t)(tp >> 1) * kBwYHalf + (uint32_t)(v >> 4) * kBwYRow + slot(v & 15) + (uint32_t)(tp & 1) * 16u;
    };
    const uint32_t put3 = r3y ? put_y(yv3) : put_x + 3 * kBwStep * kBwXRow, put4 = put_y(yv4);
    const uint32_t xc = (uint32_t)(cit * 32 + tp * 8) * 2u;
    auto yrel = [&](int v) {  // of a voxel of the brick
        return ((uint32_t)(((v >> 6) * g.h + (v >> 4 & 3)) * g.w + (v & 15)) * (uint32_t)cout + (uint32_t)(cot * 32 + tp * 8)) * 2u;
    };
    const uint32_t yrel3 = yrel(yv3), yrel4 = yrel(yv4);
    const uint32_t xsample = (uint32_t)g.d * (uint32_t)g.h * (uint32_t)g.w * (uint32_t)cin * 2u;
    const uint32_t ysample = (uint32_t)g.d * (uint32_t)g.h * (uint32_t)g.w * (uint32_t)cout * 2u;
    auto axis = [](int v, int ext, int periodic, bool& out) {
        const int w = v < 0 ? v + ext : v >= ext ? v - ext : v;
        out |= w != v && !periodic;
        return w;
    };
    struct Brick {
        int x, h, d, n;
    };
    auto after = [&](Brick b) {
        b.x += kTW;
        if (b.x == g.w) {
            b.x = 0;
            b.h += kTH;
            if (b.h == g.h) {
                b.h = 0;
                b.d += kTD;
                if (b.d == g.d) {
                    b.d = 0;
                    ++b.n;
                }
            }
        }
        return b;
    };
    Brick next;  // the next brick to load (bricks are loaded in order b0, b0 + 1, ...)
    {
        int r = (int)b0;
        next.x = (r % nbw) * kTW;
        r /= nbw;
        next.h = (r % nbh) * kTH;
        r /= nbh;
        next.d = (r % nbd) * kTD;
        next.n = r / nbd;
    }
    auto find_rows = [&](const Brick& b, uint32_t* rows) {
        if (lane < kBwRows) {
            bool out = false;
            const int sd = axis(b.d + lane / kHH - 1, g.d, g.per[0], out);
            const int sh = axis(b.h + lane % kHH - 1, g.h, g.per[1], out);
            rows[lane] = out ? kNone : (uint32_t)(sd * g.h + sh) * (uint32_t)g.w * (uint32_t)cin * 2u;
        }
    };
    u4 st[5];
    auto load = [&](const Brick& b, const uint32_t* rows) {
        const __amdgpu_buffer_rsrc_t xr = buf_rsrc((const char*)x + (uint64_t)b.n * xsample, xsample);
        const __amdgpu_buffer_rsrc_t yr = buf_rsrc((const char*)dy + (uint64_t)b.n * ysample, ysample);
        bool out = !all4;
        const int sw = axis(b.x + hx - 1, g.w, g.per[2], out);
        const uint32_t col = out ? kNone : (uint32_t)sw * (uint32_t)cin * 2u + xc;
        const uint32_t ybase = (uint32_t)((b.d * g.h + b.h) * g.w + b.x) * (uint32_t)cout * 2u;
#pragma unroll
        for (int i = 0; i < 3; ++i)
            st[i] = __builtin_bit_cast(u4, ldb8(xr, __builtin_elementwise_add_sat(rows[trow % kBwStep + i * kBwStep], col), 0));
        // one load for both kinds: a wave is of one kind
        const __amdgpu_buffer_rsrc_t r3 = r3y ? yr : xr;
        const uint32_t o3 = __builtin_elementwise_add_sat(rows[r3x ? trow + 3 * kBwStep : 0], r3x ? col : kNone);
        st[3] = __builtin_bit_cast(u4, ldb8(r3, r3y ? yrel3 : o3, r3y ? ybase : 0));
        st[4] = __builtin_bit_cast(u4, ldb8(yr, yrel4, ybase));
    };
    auto store = [&](uint32_t buf) {
        if (all4) {
#pragma unroll
            for (int i = 0; i < 3; ++i) *(u4*)(lds + buf + put_x + i * kBwStep * kBwXRow) = st[i];
        }
        if (r3x || r3y) *(u4*)(lds + buf + put3) = st[3];
        if (r4) *(u4*)(lds + buf + put4) = st[4];
    };
    // this wave's depth tap, x half and pair of depth slices
    const int dz = wave % 3, ib = wave / 3 & 1, dp = wave / 6;
    const int j = lane >> 4, l16 = lane & 15;
    // fragment reads: slice j / 2 of the pair, voxels 8 (j mod 2) + 0..7; a lane
    // addresses four channels of one voxel, and gets four voxels of one channel
    const uint32_t lane_at = (uint32_t)(j & 1) * slot(8) + (uint32_t)(l16 >> 2) * 32u + (uint32_t)(l16 & 3) * 8u;
    const uint32_t get_x = (uint32_t)ib * kBwXHalf + (uint32_t)((2 * dp + dz + (j >> 1)) * kHH) * kBwXRow + lane_at;
    const uint32_t get_x8 = get_x + ((j & 1) ? 256u : slot(8));  // four voxels 8 further on
    const uint32_t get_y = 2 * kBwXHalf + (uint32_t)((2 * dp + (j >> 1)) * kTH) * kBwYRow + lane_at;
    auto tr = [&](uint32_t at) -> u2 {
        return __builtin_bit_cast(u2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(lds + at)));
    };
    const bool ones = bias && cit == 0 && dz == 0 && ib == 0;
    float bsum[2] = {0.f, 0.f};  // this lane's voxels of channel l16 of each co block
    f4 acc[3][3][2];             // [dy tap][x tap][co block]
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[t / 3][t % 3][b] = f4{0.f, 0.f, 0.f, 0.f};
    }
    Brick following = after(next);
    if (wave == 0) find_rows(next, row_off[0]);
    if (wave == 1) find_rows(following, row_off[1]);
    __syncthreads();
    if (b0 < b1) {
        load(next, row_off[0]);
        store(0);
    }
    __syncthreads();
    uint32_t cur = 0;
    for (long long br = b0; br < b1; ++br) {
        const bool more = br + 1 < b1;
        const int odd = (int)(br - b0) & 1;
        next = following;
        following = after(next);
        if (more) load(next, row_off[odd ^ 1]);
        if (wave == 11) find_rows(following, row_off[odd]);
        u2 xt[2][3], yt[4][2][2];
        auto read_row = [&](int r) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                xt[r & 1][k] = tr(cur + (k == 2 ? get_x8 : get_x + 128u * k) + (uint32_t)r * kBwXRow);
            if (r < 4) {
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        yt[r][b][k] = tr(cur + get_y + (uint32_t)b * kBwYHalf + (uint32_t)r * kBwYRow + 128u * k);
            }
        };
        read_row(0);
#pragma unroll
        for (int r = 0; r < 6; ++r) {
            const u2 t0 = xt[r & 1][0], t1 = xt[r & 1][1], t2 = xt[r & 1][2];
            const u4 f[3] = {u4{t0.x, t0.y, t1.x, t1.y},
                             u4{__builtin_amdgcn_alignbyte(t0.y, t0.x, 2), __builtin_amdgcn_alignbyte(t1.x, t0.y, 2),
                                __builtin_amdgcn_alignbyte(t1.y, t1.x, 2), __builtin_amdgcn_alignbyte(t2.x, t1.y, 2)},
                             u4{t0.y, t1.x, t1.y, t2.x}};
            // the dy row that this halo row is neighbour ty - 1 of; the next rows are
            // read once the oldest dy row is done with
#pragma unroll
            for (int ty = 2; ty >= 0; --ty) {
                const int h = r - ty;
                if (h >= 0 && h < 4) {
#pragma unroll
                    for (int cx = 0; cx < 3; ++cx)
#pragma unroll
                        for (int b = 0; b < 2; ++b) {
                            const u4 a = u4{yt[h][b][0].x, yt[h][b][0].y, yt[h][b][1].x, yt[h][b][1].y};
                            acc[ty][cx][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                __builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, f[cx]), acc[ty][cx][b], 0, 0, 0);
                        }
                }
                __builtin_amdgcn_sched_barrier(0);
                if (ty == 2 && r < 5) read_row(r + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (ones && r < 4) {
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int k = 0; k < 2; ++k)
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            const unsigned w = yt[r][b][k][e];
                            bsum[b] += __builtin_bit_cast(float, w << 16);
                            bsum[b] += __builtin_bit_cast(float, w & 0xffff0000u);
                        }
            }
        }
        cur ^= kBwBuf;
        if (more) store(cur);
        __syncthreads();
    }
    // the waves of the second pair of slices hand their sums over
    f4* sum = (f4*)lds + (wave % 6) * 18 * 64 + lane;
    float* bs = (float*)((f4*)lds + 6 * 18 * 64) + l16;
    if (ones) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            bsum[b] += __shfl_xor(bsum[b], 16);
            bsum[b] += __shfl_xor(bsum[b], 32);
        }
    }
    if (dp == 1) {
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int b = 0; b < 2; ++b) sum[(t * 2 + b) * 64] = acc[t / 3][t % 3][b];
        if (ones && j == 0) {
            bs[0] = bsum[0];
            bs[16] = bsum[1];
        }
    }
    __syncthreads();
    if (dp == 1) return;
    // D[co][ci]: row (lane / 16) * 4 + i, column lane % 16
    float* const out = part + (long long)ch * pstride;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        float* p = out + ((long long)(dz * 9 + t) * cout) * cin;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const f4 s = acc[t / 3][t % 3][b] + sum[(t * 2 + b) * 64];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int co = cot * 32 + b * 16 + j * 4 + i;
                const int ci = cit * 32 + ib * 16 + l16;
                p[(long long)co * cin + ci] = s[i];
            }
        }
    }
    if (ones && j == 0) {
#pragma unroll
        for (int b = 0; b < 2; ++b) out[27LL * cin * cout + cot * 32 + b * 16 + l16] = bsum[b] + bs[16 * b];
    }
}

// Element e of the chunk sums, e < n0 + n1: out0[e] (e < n0) or out1[e - n0]
// = sum over chunks c of part[c * pstride + e], in a fixed order: wave s of a
// workgroup of W waves sums chunks s, s + W, s + 2 W, ... for 64 consecutive
// elements, then the wave sums are added in wave order.  The sum is bound by
// the latency of its loads: 16 waves pay off from about 128 chunks.
template <int W>
__global__ __launch_bounds__(64 * W) void k_sum_chunks(const float* __restrict__ part, long long pstride, long long n0,
                                                       long long n1, int nchunk, float* __restrict__ out0,
                                                       float* __restrict__ out1)
{
    __shared__ float sh[W][64];
    const int e = threadIdx.x & 63, sl = threadIdx.x >> 6;
    const long long i = (long long)blockIdx.x * 64 + e;
    const long long n = n0 + n1;
    float acc = 0.f;
    if (i < n)
        for (int c = sl; c < nchunk; c += W) acc += part[(long long)c * pstride + i];
    sh[sl][e] = acc;
    __syncthreads();
    if (sl == 0 && i < n) {
        float v = sh[0][e];
        for (int k = 1; k < W; ++k) v += sh[k][e];
        if (i < n0)
            out0[i] = v;
        else
            out1[i - n0] = v;
    }
}

// Per-chunk column sums of a [rows][cols] BF16 matrix (cols <= 256): thread t
// sums column t % cols over every (256 / cols)-th row of the block's chunk,
// then the row groups are added in LDS in a fixed order.
constexpr int kColSumBlocks = 1024;

__global__ __launch_bounds__(256) void k_colsum_part(const bf16* __restrict__ a, long long rows, int cols,
                                                     long long chunk, float* __restrict__ part)
{
    __shared__ float sh[256];
    const int t = threadIdx.x;
    const int rpi = 256 / cols;
    const int c = t % cols, roff = t / cols;
    const long long r0 = (long long)blockIdx.x * chunk;
    const long long r1 = r0 + chunk < rows ? r0 + chunk : rows;
    float s = 0.f;
    if (roff < rpi)
        for (long long r = r0 + roff; r < r1; r += rpi) s += (float)a[r * cols + c];
    sh[t] = s;
    __syncthreads();
    if (t < cols) {
        float q = 0.f;
        for (int k = 0; k < rpi; ++k) q += sh[k * cols + t];
        part[(long long)blockIdx.x * cols + t] = q;
    }
}

// ---------------------------------------------------------------------------
// elementwise

__global__ void k_act_bwd(const bf16* __restrict__ y, const bf16* __restrict__ dy, bf16* __restrict__ dp, long long n,
                          int act)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        float d = (float)dy[i];
        if (act == CMNN_ACT_LEAKY && (float)y[i] <= 0.f) d *= kLeak;
        dp[i] = (bf16)d;
    }
}

__global__ void k_pool2_fwd(G g, const bf16* __restrict__ x, int c, bf16* __restrict__ y)
{
    const int d2 = g.d / 2, h2 = g.h / 2, w2 = g.w / 2;
    const long long total = (long long)g.n * d2 * h2 * w2 * c;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        const int ch = (int)(i % c);
        long long r = i / c;
        const int w = (int)(r % w2);
        r /= w2;
        const int h = (int)(r % h2);
        r /= h2;
        const int d = (int)(r % d2);
        const long long n = r / d2;
        float s = 0.f;
        for (int k = 0; k < 8; ++k) {
            const long long v = ((n * g.d + 2 * d + (k >> 2)) * g.h + 2 * h + ((k >> 1) & 1)) * g.w + 2 * w + (k & 1);
            s += (float)x[v * c + ch];
        }
        y[i] = (bf16)(0.125f * s);
    }
}

__global__ void k_pool2_bwd(G g, const bf16* __restrict__ dy, int c, bf16* __restrict__ dx)
{
    const long long total = g.nvox * c;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        const int ch = (int)(i % c);
        long long r = i / c;
        const int w = (int)(r % g.w);
        r /= g.w;
        const int h = (int)(r % g.h);
        r /= g.h;
        const int d = (int)(r % g.d);
        const long long n = r / g.d;
        const long long v = ((n * (g.d / 2) + d / 2) * (g.h / 2) + h / 2) * (g.w / 2) + w / 2;
        dx[i] = (bf16)(0.125f * (float)dy[v * c + ch]);
    }
}

// coarse geometry g; fine voxel (2d + a, 2h + b, 2w + e) copies coarse (d, h, w)
__global__ void k_up2_fwd(G g, const bf16* __restrict__ x, int c, bf16* __restrict__ y)
{
    const int D = 2 * g.d, H = 2 * g.h, W = 2 * g.w;
    const long long total = (long long)g.n * D * H * W * c;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        const int ch = (int)(i % c);
        long long r = i / c;
        const int w = (int)(r % W);
        r /= W;
        const int h = (int)(r % H);
        r /= H;
        const int d = (int)(r % D);
        const long long n = r / D;
        const long long v = ((n * g.d + d / 2) * g.h + h / 2) * g.w + w / 2;
        y[i] = x[v * c + ch];
    }
}

__global__ void k_up2_bwd(G g, const bf16* __restrict__ dy, int c, bf16* __restrict__ dx)
{
    const int H = 2 * g.h, W = 2 * g.w;
    const long long total = g.nvox * c;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        const int ch = (int)(i % c);
        long long r = i / c;
        const int w = (int)(r % g.w);
        r /= g.w;
        const int h = (int)(r % g.h);
        r /= g.h;
        const int d = (int)(r % g.d);
        const long long n = r / g.d;
        float s = 0.f;
        for (int k = 0; k < 8; ++k) {
            const long long v = ((n * (2 * g.d) + 2 * d + (k >> 2)) * H + 2 * h + ((k >> 1) & 1)) * W + 2 * w + (k & 1);
            s += (float)dy[v * c + ch];
        }
        dx[i] = (bf16)s;
    }
}

__global__ void k_concat_fwd(long long nvox, const bf16* __restrict__ a, int ca, const bf16* __restrict__ b, int cb,
                             bf16* __restrict__ y)
{
    const int c = ca + cb;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nvox * c;
         i += (long long)gridDim.x * blockDim.x) {
        const long long v = i / c;
        const int ch = (int)(i % c);
        y[i] = ch < ca ? a[v * ca + ch] : b[v * cb + ch - ca];
    }
}

__global__ void k_concat_bwd(long long nvox, const bf16* __restrict__ dy, int ca, int cb, bf16* __restrict__ da,
                             bf16* __restrict__ db)
{
    const int c = ca + cb;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nvox * c;
         i += (long long)gridDim.x * blockDim.x) {
        const long long v = i / c;
        const int ch = (int)(i % c);
        if (ch < ca) {
            if (da) da[v * ca + ch] = dy[i];
        } else if (db) {
            db[v * cb + ch - ca] = dy[i];
        }
    }
}

__global__ void k_add(long long n, const bf16* __restrict__ a, const bf16* __restrict__ b, bf16* __restrict__ y)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
        y[i] = (bf16)((float)a[i] + (float)b[i]);
}

// 16-byte variants of the elementwise kernels (8 channels per thread), used when
// the channel counts are multiples of 8 and the pointers 16-byte aligned

__global__ void k_act_bwd8(const u4* __restrict__ y, const u4* __restrict__ dy, u4* __restrict__ dp, long long n8, int act)
{
    GRID_STRIDE(i, n8)
    {
        float fy[8], fd[8];
        unpack8(y[i], fy);
        unpack8(dy[i], fd);
        if (act == CMNN_ACT_LEAKY)
#pragma unroll
            for (int k = 0; k < 8; ++k) fd[k] = fy[k] <= 0.f ? kLeak * fd[k] : fd[k];
        dp[i] = pack8(fd);
    }
}

template <typename I>
__global__ void k_pool2_fwd8(G g, const bf16* __restrict__ x, int c, bf16* __restrict__ y)
{
    const I d2 = g.d / 2, h2 = g.h / 2, w2 = g.w / 2, q8 = c / 8;
    GRID_STRIDE_I(I, i, (long long)g.n * d2 * h2 * w2 * q8)
    {
        const I q = i % q8;
        I r = i / q8;
        const I w = r % w2;
        r /= w2;
        const I h = r % h2;
        r /= h2;
        const I d = r % d2;
        const I n = r / d2;
        float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, f[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const I v = ((n * g.d + 2 * d + (k >> 2)) * g.h + 2 * h + ((k >> 1) & 1)) * g.w + 2 * w + (k & 1);
            unpack8(*(const u4*)(x + v * c + 8 * q), f);
#pragma unroll
            for (int e = 0; e < 8; ++e) s[e] += f[e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] *= 0.125f;
        *(u4*)(y + i * 8) = pack8(s);
    }
}

__global__ void k_pool2_bwd8(G g, const bf16* __restrict__ dy, int c, bf16* __restrict__ dx)
{
    const int q8 = c / 8;
    GRID_STRIDE(i, g.nvox * q8)
    {
        const int q = (int)(i % q8);
        long long r = i / q8;
        const int w = (int)(r % g.w);
        r /= g.w;
        const int h = (int)(r % g.h);
        r /= g.h;
        const int d = (int)(r % g.d);
        const long long n = r / g.d;
        const long long v = ((n * (g.d / 2) + d / 2) * (g.h / 2) + h / 2) * (g.w / 2) + w / 2;
        float f[8];
        unpack8(*(const u4*)(dy + v * c + 8 * q), f);
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] *= 0.125f;
        *(u4*)(dx + i * 8) = pack8(f);
    }
}

__global__ void k_up2_fwd8(G g, const bf16* __restrict__ x, int c, bf16* __restrict__ y)
{
    const int D = 2 * g.d, H = 2 * g.h, W = 2 * g.w, q8 = c / 8;
    GRID_STRIDE(i, (long long)g.n * D * H * W * q8)
    {
        const int q = (int)(i % q8);
        long long r = i / q8;
        const int w = (int)(r % W);
        r /= W;
        const int h = (int)(r % H);
        r /= H;
        const int d = (int)(r % D);
        const long long n = r / D;
        const long long v = ((n * g.d + d / 2) * g.h + h / 2) * g.w + w / 2;
        *(u4*)(y + i * 8) = *(const u4*)(x + v * c + 8 * q);
    }
}

__global__ void k_up2_bwd8(G g, const bf16* __restrict__ dy, int c, bf16* __restrict__ dx)
{
    const int H = 2 * g.h, W = 2 * g.w, q8 = c / 8;
    GRID_STRIDE(i, g.nvox * q8)
    {
        const int q = (int)(i % q8);
        long long r = i / q8;
        const int w = (int)(r % g.w);
        r /= g.w;
        const int h = (int)(r % g.h);
        r /= g.h;
        const int d = (int)(r % g.d);
        const long long n = r / g.d;
        float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, f[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const long long v = ((n * (2 * g.d) + 2 * d + (k >> 2)) * H + 2 * h + ((k >> 1) & 1)) * W + 2 * w + (k & 1);
            unpack8(*(const u4*)(dy + v * c + 8 * q), f);
#pragma unroll
            for (int e = 0; e < 8; ++e) s[e] += f[e];
        }
        *(u4*)(dx + i * 8) = pack8(s);
    }
}

__global__ void k_concat_fwd8(long long nvox, const bf16* __restrict__ a, int ca, const bf16* __restrict__ b, int cb,
                              bf16* __restrict__ y)
{
    const int qa = ca / 8, q8 = (ca + cb) / 8;
    GRID_STRIDE(i, nvox * q8)
    {
        const long long v = i / q8;
        const int q = (int)(i % q8);
        *(u4*)(y + i * 8) = q < qa ? *(const u4*)(a + v * ca + 8 * q) : *(const u4*)(b + v * cb + 8 * (q - qa));
    }
}

__global__ void k_concat_bwd8(long long nvox, const bf16* __restrict__ dy, int ca, int cb, bf16* __restrict__ da,
                              bf16* __restrict__ db)
{
    const int qa = ca / 8, q8 = (ca + cb) / 8;
    GRID_STRIDE(i, nvox * q8)
    {
        const long long v = i / q8;
        const int q = (int)(i % q8);
        const u4 e = *(const u4*)(dy + i * 8);
        if (q < qa) {
            if (da) *(u4*)(da + v * ca + 8 * q) = e;
        } else if (db) {
            *(u4*)(db + v * cb + 8 * (q - qa)) = e;
        }
    }
}

__global__ void k_add8(long long n8, const u4* __restrict__ a, const u4* __restrict__ b, u4* __restrict__ y)
{
    GRID_STRIDE(i, n8)
    {
        float fa[8], fb[8];
        unpack8(a[i], fa);
        unpack8(b[i], fb);
#pragma unroll
        for (int e = 0; e < 8; ++e) fa[e] += fb[e];
        y[i] = pack8(fa);
    }
}

// Skip-connection joins of the U-Net: one pass over the fine level each, in
// place of the separate upsampling or pooling, concatenation, sum and
// activation-gradient passes.  Channel counts are multiples of 32 and channel
// strides multiples of 8, so every thread moves 8 channels (16 bytes).

// y = [skip | up2(x)] at the fine level; g is the coarse geometry of x.
template <typename I>
__global__ void k_up2_concat_fwd8(G g, const bf16* __restrict__ skip, int cs, const bf16* __restrict__ x, int cx,
                                  bf16* __restrict__ y)
{
    const I D = 2 * g.d, H = 2 * g.h, W = 2 * g.w, qs = cs / 8, q8 = (cs + cx) / 8;
    GRID_STRIDE_I(I, i, 8 * g.nvox * q8)
    {
        const I q = i % q8;
        const I v = i / q8;
        u4 e;
        if (q < qs) {
            e = *(const u4*)(skip + v * cs + 8 * q);
        } else {
            const I w = v % W;
            I r = v / W;
            const I h = r % H;
            r /= H;
            const I d = r % D;
            const I n = r / D;
            const I p = ((n * g.d + d / 2) * g.h + h / 2) * g.w + w / 2;
            e = *(const u4*)(x + p * cx + 8 * (q - qs));
        }
        *(u4*)(y + i * 8) = e;
    }
}

// Leaky-ReLU slope at the activation output, applied to an FP32 gradient.
__device__ __forceinline__ void act_grad8(const bf16* __restrict__ gate, int act, float (&f)[8])
{
    if (act != CMNN_ACT_LEAKY) return;
    float t[8];
    unpack8(*(const u4*)gate, t);
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = t[e] <= 0.f ? kLeak * f[e] : f[e];
}

// dx = act'(gate) * (up2 gradient of dy): dy is the upsampled part of a
// concatenation's gradient (channel stride ldy), g the coarse geometry.
template <typename I>
__global__ void k_up2_bwd_act8(G g, const bf16* __restrict__ dy, int ldy, int c, const bf16* __restrict__ gate,
                               int act, bf16* __restrict__ dx)
{
    const I H = 2 * g.h, W = 2 * g.w, q8 = c / 8;
    GRID_STRIDE_I(I, i, g.nvox * q8)
    {
        const I q = i % q8;
        I r = i / q8;
        const I w = r % g.w;
        r /= g.w;
        const I h = r % g.h;
        r /= g.h;
        const I d = r % g.d;
        const I n = r / g.d;
        float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, f[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const I v = ((n * (2 * g.d) + 2 * d + (k >> 2)) * H + 2 * h + ((k >> 1) & 1)) * W + 2 * w + (k & 1);
            unpack8(*(const u4*)(dy + v * ldy + 8 * q), f);
#pragma unroll
            for (int e = 0; e < 8; ++e) s[e] += f[e];
        }
        act_grad8(gate + i * 8, act, s);
        *(u4*)(dx + i * 8) = pack8(s);
    }
}

// dx = act'(gate) * (pool2 gradient of dy + skip): g is the fine geometry, dy
// coarse, skip the skip part of a concatenation's gradient (channel stride
// ldskip) or NULL.
template <typename I>
__global__ void k_pool2_bwd_add_act8(G g, const bf16* __restrict__ dy, int c, const bf16* __restrict__ skip,
                                     int ldskip, const bf16* __restrict__ gate, int act, bf16* __restrict__ dx)
{
    const I q8 = c / 8;
    GRID_STRIDE_I(I, i, g.nvox * q8)
    {
        const I q = i % q8;
        const I v = i / q8;
        const I w = v % g.w;
        I r = v / g.w;
        const I h = r % g.h;
        r /= g.h;
        const I d = r % g.d;
        const I n = r / g.d;
        const I p = ((n * (g.d / 2) + d / 2) * (g.h / 2) + h / 2) * (g.w / 2) + w / 2;
        float f[8], t[8];
        unpack8(*(const u4*)(dy + p * c + 8 * q), f);
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] *= 0.125f;
        if (skip) {
            unpack8(*(const u4*)(skip + v * ldskip + 8 * q), t);
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] += t[e];
        }
        act_grad8(gate + i * 8, act, f);
        *(u4*)(dx + i * 8) = pack8(f);
    }
}

// masked MSE: per-block partial (sum wt * sq, sum wt), then a single-block final
constexpr int kMseBlocks = 1024;

__global__ __launch_bounds__(256) void k_mse_part(long long nvox, const bf16* __restrict__ pred, int c, int creal,
                                                  const float* __restrict__ tgt, const float* __restrict__ wt,
                                                  float* __restrict__ part)
{
    __shared__ float s0[256], s1[256];
    float a = 0.f, b = 0.f;
    for (long long v = (long long)blockIdx.x * 256 + threadIdx.x; v < nvox; v += (long long)gridDim.x * 256) {
        const float w = wt[v];
        float q = 0.f;
        for (int k = 0; k < creal; ++k) {
            const float d = (float)pred[v * c + k] - tgt[(long long)k * nvox + v];
            q += d * d;
        }
        a += w * q;
        b += w;
    }
    s0[threadIdx.x] = a;
    s1[threadIdx.x] = b;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            s0[threadIdx.x] += s0[threadIdx.x + s];
            s1[threadIdx.x] += s1[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = s0[0];
        part[2 * blockIdx.x + 1] = s1[0];
    }
}

// One workgroup of 256: thread t adds partials t, t + 256, ... in order, then
// the 256 sums are added pairwise in LDS (a fixed order: deterministic).
__global__ __launch_bounds__(256) void k_mse_final(const float* __restrict__ part, int nb, int creal,
                                                   float* __restrict__ out)
{
    __shared__ float sa[256], sb[256];
    const int t = threadIdx.x;
    float a = 0.f, b = 0.f;
    for (int i = t; i < nb; i += 256) {
        a += part[2 * i];
        b += part[2 * i + 1];
    }
    sa[t] = a;
    sb[t] = b;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h) {
            sa[t] += sa[t + h];
            sb[t] += sb[t + h];
        }
        __syncthreads();
    }
    if (t == 0) {
        out[0] = sb[0] > 0.f ? sa[0] / (sb[0] * creal) : 0.f;  // loss
        out[1] = sb[0] * creal;                                 // normaliser, read by k_mse_grad
    }
}

__global__ void k_mse_grad(long long nvox, const bf16* __restrict__ pred, int c, int creal,
                           const float* __restrict__ tgt, const float* __restrict__ wt,
                           const float* __restrict__ norm, bf16* __restrict__ dpred)
{
    const float scale = norm[1] > 0.f ? 2.f / norm[1] : 0.f;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nvox * c;
         i += (long long)gridDim.x * blockDim.x) {
        const long long v = i / c;
        const int k = (int)(i % c);
        float d = 0.f;
        if (k < creal) d = scale * wt[v] * ((float)pred[i] - tgt[(long long)k * nvox + v]);
        dpred[i] = (bf16)d;
    }
}

// 8 channels per thread: channels below creal get the gradient, the padded
// ones zeros (their prediction is not read)
template <typename I>
__global__ void k_mse_grad8(long long nvox, const bf16* __restrict__ pred, int c, int creal,
                            const float* __restrict__ tgt, const float* __restrict__ wt,
                            const float* __restrict__ norm, bf16* __restrict__ dpred)
{
    const float scale = norm[1] > 0.f ? 2.f / norm[1] : 0.f;
    const I q8 = c / 8, nv = (I)nvox;
    GRID_STRIDE_I(I, i, nvox * q8)
    {
        const I q = i % q8;
        const I v = i / q8;
        float f[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if ((int)(8 * q) < creal) {
            float p[8];
            unpack8(*(const u4*)(pred + i * 8), p);
            const float sw = scale * wt[v];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if ((int)(8 * q) + e < creal) f[e] = sw * (p[e] - tgt[(8 * q + e) * nv + v]);
        }
        *(u4*)(dpred + i * 8) = pack8(f);
    }
}

__global__ void k_adam(long long n, float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, float lr, float b1, float b2, float eps, float wd, float c1, float c2)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        const float mh = mi / c1, vh = vi / c2;
        p[i] -= lr * (mh / (sqrtf(vh) + eps) + wd * p[i]);
    }
}

// Global gradient-norm clipping: per-block partial sums of g^2, one workgroup
// that sums them and forms the norm and the scale min(1, max_norm / norm) (0 for a
// non-finite norm, which turns the update into a no-gradient step), then an
// in-place scale read from device memory (no host round trip).
constexpr int kClipBlocks = 512;

__global__ __launch_bounds__(256) void k_sumsq_part(long long n, const float* __restrict__ g, float* __restrict__ part)
{
    __shared__ float sh[256];
    float a = 0.f;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256) {
        const float x = g[i];
        a += x * x;
    }
    sh[threadIdx.x] = a;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// One workgroup of 256, FP64 sums in a fixed order (as k_mse_final).
__global__ __launch_bounds__(256) void k_clip_final(const float* __restrict__ part, int nb, float max_norm,
                                                    float* __restrict__ out)
{
    __shared__ double sh[256];
    const int t = threadIdx.x;
    double a = 0.0;
    for (int i = t; i < nb; i += 256) a += part[i];
    sh[t] = a;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h) sh[t] += sh[t + h];
        __syncthreads();
    }
    if (t != 0) return;
    const float norm = (float)sqrt(sh[0]);
    float scale = 1.f;
    if (!(norm < INFINITY)) scale = 0.f;
    else if (max_norm > 0.f && norm > max_norm) scale = max_norm / norm;
    out[0] = norm;
    out[1] = scale;
}

__global__ void k_scale(long long n, float* __restrict__ g, const float* __restrict__ sc)
{
    const float a = sc[1];
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
        g[i] = a == 0.f ? 0.f : g[i] * a;
}

__global__ void k_pack_w(const float* __restrict__ w, int cin, int cout, bf16* __restrict__ wf, bf16* __restrict__ wtr)
{
    const long long total = 27LL * cin * cout;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        const int ci = (int)(i % cin);
        long long r = i / cin;
        const int co = (int)(r % cout);
        const int t = (int)(r / cout);
        const bf16 b = (bf16)w[i];
        wf[i] = b;
        wtr[((long long)t * cin + ci) * cout + co] = b;
    }
}

// Several layers' packing in one launch: each workgroup belongs to one layer
// (first_block ranges), so the layer's parameters are wave-uniform.
struct PackJobs {
    const float* w[CMNN_PACK_MAX];
    bf16* wf[CMNN_PACK_MAX];
    bf16* wt[CMNN_PACK_MAX];
    int cin[CMNN_PACK_MAX], cout[CMNN_PACK_MAX];
    int first_block[CMNN_PACK_MAX + 1];
    int n;
};

__global__ __launch_bounds__(256) void k_pack_w_batch(const PackJobs J)
{
    int l = 0;
    while (l + 1 < J.n && (int)blockIdx.x >= J.first_block[l + 1]) ++l;
    const int cin = J.cin[l], cout = J.cout[l];
    const long long i = (long long)((int)blockIdx.x - J.first_block[l]) * 256 + threadIdx.x;
    if (i >= 27LL * cin * cout) return;
    const int ci = (int)(i % cin);
    const long long r = i / cin;
    const int co = (int)(r % cout), t = (int)(r / cout);
    const bf16 b = (bf16)J.w[l][i];
    J.wf[l][i] = b;
    J.wt[l][((long long)t * cin + ci) * cout + co] = b;
}

__global__ void k_pack_ch(long long nvox, const float* __restrict__ src, int cs, bf16* __restrict__ dst, int c)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nvox * c;
         i += (long long)gridDim.x * blockDim.x) {
        const long long v = i / c;
        const int k = (int)(i % c);
        dst[i] = k < cs ? (bf16)src[(long long)k * nvox + v] : (bf16)0.f;
    }
}

// Minibatch gathers from sample-major planes src [np][nsrc][nvs]: output
// sample b is source sample idx[b] (b itself when idx is NULL); an index
// outside [0, nsrc) gives zeros.
__device__ __forceinline__ long long pick(const int* __restrict__ idx, long long b, int nsrc)
{
    const long long s = idx ? (long long)idx[b] : b;
    return s >= 0 && s < nsrc ? s : -1;
}

// BF16 NDHWC [nsel * nvs][c] (channels from cs on zero), 8 channels per thread
template <typename I>
__global__ void k_gather_pack8(int nsel, const int* __restrict__ idx, long long nvs, const float* __restrict__ src,
                               int nsrc, int cs, bf16* __restrict__ dst, int c)
{
    const I q8 = c / 8, nv = (I)nvs;
    GRID_STRIDE_I(I, i, (long long)nsel * nvs * q8)
    {
        const I q = i % q8;
        const I r = i / q8, v = r % nv;
        const long long s = pick(idx, (long long)(r / nv), nsrc);
        float f[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (s >= 0 && (int)(8 * q) < cs)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if ((int)(8 * q) + e < cs) f[e] = src[((8 * q + e) * (I)nsrc + (I)s) * nv + v];
        *(u4*)(dst + i * 8) = pack8(f);
    }
}

// FP32 [np][nsel][nvs], 4 values per thread (nvs a multiple of 4)
__global__ void k_gather4(int nsel, const int* __restrict__ idx, long long nvs4, const float4* __restrict__ src,
                          int nsrc, int np, float4* __restrict__ dst)
{
    GRID_STRIDE(i, (long long)np * nsel * nvs4)
    {
        const long long v = i % nvs4, r = i / nvs4, b = r % nsel, p = r / nsel, s = pick(idx, b, nsrc);
        dst[i] = s >= 0 ? src[(p * nsrc + s) * nvs4 + v] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

__global__ void k_gather1(int nsel, const int* __restrict__ idx, long long nvs, const float* __restrict__ src,
                          int nsrc, int np, float* __restrict__ dst)
{
    GRID_STRIDE(i, (long long)np * nsel * nvs)
    {
        const long long v = i % nvs, r = i / nvs, b = r % nsel, p = r / nsel, s = pick(idx, b, nsrc);
        dst[i] = s >= 0 ? src[(p * nsrc + s) * nvs + v] : 0.f;
    }
}

__global__ void k_unpack_ch(long long nvox, const bf16* __restrict__ src, int c, float* __restrict__ dst, int cs)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nvox * cs;
         i += (long long)gridDim.x * blockDim.x) {
        const int k = (int)(i / nvox);
        const long long v = i % nvox;
        dst[i] = (float)src[v * c + k];
    }
}

// Per-sample channel means broadcast back over the voxels:
// y[n][v][c] = (1/V) sum_v' x[n][v'][c].  The operator is a symmetric
// projection, so the same two kernels also give its gradient.
__global__ __launch_bounds__(256) void k_chmean_part(const bf16* __restrict__ x, int ldx, long long vps, int c,
                                                     int parts, float* __restrict__ part)
{
    // block (n, p): voxels [p * chunk, (p + 1) * chunk) of sample n; thread t sums channel t % c
    // (voxel rows ldx channels apart)
    __shared__ float sh[256];
    const int n = blockIdx.x / parts, p = blockIdx.x % parts;
    const long long chunk = (vps + parts - 1) / parts;
    const long long v0 = p * chunk, v1 = v0 + chunk < vps ? v0 + chunk : vps;
    const int t = threadIdx.x, rpi = 256 / c, ch = t % c, roff = t / c;
    float s = 0.f;
    if (roff < rpi)
        for (long long v = v0 + roff; v < v1; v += rpi) s += (float)x[((long long)n * vps + v) * ldx + ch];
    sh[t] = s;
    __syncthreads();
    if (t < c) {
        float q = 0.f;
        for (int k = 0; k < rpi; ++k) q += sh[k * c + t];
        part[((long long)n * parts + p) * c + t] = q;
    }
}

__global__ void k_chmean_final(const float* __restrict__ part, long long vps, int c, int nsamp, int parts,
                               float* __restrict__ mean)
{
    GRID_STRIDE(i, (long long)nsamp * c)
    {
        const long long n = i / c;
        const int ch = (int)(i % c);
        float s = 0.f;
#pragma unroll 16
        for (int p = 0; p < parts; ++p) s += part[(n * parts + p) * c + ch];  // loads in flight together
        mean[i] = s / (float)vps;
    }
}

__global__ void k_chmean_bcast8(const float* __restrict__ mean, long long vps, int c, bf16* __restrict__ y,
                                long long total8)
{
    const int q8 = c / 8;
    GRID_STRIDE(i, total8)
    {
        const int q = (int)(i % q8);
        const long long n = i / q8 / vps;
        float f[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = mean[n * c + 8 * q + e];
        *(u4*)(y + i * 8) = pack8(f);
    }
}

// Joins of the U-Net bottleneck's global context (channel counts multiples of
// 32): y = [x | broadcast mean] for the forward concatenation, and
// y = act'(gate) * (skip + broadcast mean) for its gradient.
__global__ void k_chmean_concat8(const float* __restrict__ mean, long long vps, int c, const bf16* __restrict__ x,
                                 bf16* __restrict__ y, long long total8)
{
    const int qc = c / 8, q8 = 2 * qc;
    GRID_STRIDE(i, total8)
    {
        const int q = (int)(i % q8);
        const long long v = i / q8;
        if (q < qc) {
            *(u4*)(y + i * 8) = *(const u4*)(x + v * c + 8 * q);
        } else {
            const long long n = v / vps;
            float f[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = mean[n * c + 8 * (q - qc) + e];
            *(u4*)(y + i * 8) = pack8(f);
        }
    }
}

__global__ void k_chmean_add_act8(const float* __restrict__ mean, long long vps, int c,
                                  const bf16* __restrict__ skip, int ldskip, const bf16* __restrict__ gate, int act,
                                  bf16* __restrict__ y, long long total8)
{
    const int q8 = c / 8;
    GRID_STRIDE(i, total8)
    {
        const int q = (int)(i % q8);
        const long long v = i / q8, n = v / vps;
        float f[8], t[8];
        unpack8(*(const u4*)(skip + v * ldskip + 8 * q), t);
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = mean[n * c + 8 * q + e] + t[e];
        act_grad8(gate + i * 8, act, f);
        *(u4*)(y + i * 8) = pack8(f);
    }
}

__global__ void k_chmean_bcast(const float* __restrict__ part, long long vps, int c, int nsamp, int parts,
                               bf16* __restrict__ y)
{
    const long long total = (long long)nsamp * vps * c;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        const int ch = (int)(i % c);
        const long long n = i / c / vps;
        float s = 0.f;
        for (int p = 0; p < parts; ++p) s += part[(n * parts + p) * c + ch];
        y[i] = (bf16)(s / (float)vps);
    }
}

constexpr int kMeanParts = 64;

int launched() { return hipGetLastError() == hipSuccess ? CMNN_OK : CMNN_EHIP; }

int sum_chunks(const float* part, long long pstride, long long n0, long long n1, int nchunk, float* out0, float* out1,
               hipStream_t s)
{
    const unsigned nblk = (unsigned)((n0 + n1 + 63) / 64);
    if (nchunk >= 128)
        k_sum_chunks<16><<<nblk, 1024, 0, s>>>(part, pstride, n0, n1, nchunk, out0, out1);
    else
        k_sum_chunks<8><<<nblk, 512, 0, s>>>(part, pstride, n0, n1, nchunk, out0, out1);
    return launched();
}

dim3 grid_for(long long n)
{
    long long b = (n + 255) / 256;
    if (b > 65536) b = 65536;
    if (b < 1) b = 1;
    return dim3((unsigned)b);
}

bool brick_ok(const G& g) { return g.d % kTD == 0 && g.h % kTH == 0 && g.w % kTW == 0; }
// The brick weight-gradient kernel addresses x and dy with 32-bit byte offsets.
bool bwd_w_brick(const G& g, int cin, int cout)
{
    return brick_ok(g) && g.nvox * 2LL * (cin > cout ? cin : cout) < (1LL << 32);
}

// Voxel chunks of the weight gradient (partials summed in a fixed order).
// Brick path: at most 256 workgroups (one per CU), whole bricks
// per chunk.  Generic path: >= 4096 voxels per chunk.
int bwd_w_chunks(const G& g, int cin, int cout)
{
    if (bwd_w_brick(g, cin, cout)) {
        // one workgroup per CU (143 KB of LDS): at most 256 (chunk, tile)
        // workgroups, so that none waits for a second round; then the bricks
        // per chunk with the least time, at about 1.6 us a brick and 0.028 us to
        // write and sum a workgroup's partials.  One brick each where 256 CUs
        // take 256: 24.4 us, two each 21.1; 64 -> 64 on 128 bricks 2 / 3: 23.3 / 20.8;
        // 1024 bricks 4 / 6: 29.4 / 30.4.
        const long long bricks = g.nvox / (kTD * kTH * kTW);
        const long long tiles = (long long)(cin / 32) * (cout / 32);
        long long c = 256 / tiles;
        if (c < 1) c = 1;
        if (c > bricks) c = bricks;
        long long per = (bricks + c - 1) / c;
        auto chunks = [&](long long p) { return (bricks + p - 1) / p; };
        auto cost = [&](long long p) { return 1.6 * (double)p + 0.028 * (double)(chunks(p) * tiles); };
        while (per < bricks && cost(per + 1) < cost(per)) ++per;
        return (int)chunks(per);
    }
    long long c = (g.nvox + 4095) / 4096;
    return (int)(c < 64 ? c : 64);
}

template <int NB, int SIGN, int ACT>
int conv_tile_launch(const G& g, const bf16* x, int cin, const bf16* w, const float* bias, int cout, bf16* y,
                     const bf16* gate, hipStream_t s)
{
    const unsigned bricks = (unsigned)(g.nvox / (kTD * kTH * kTW));
    const unsigned span = bricks % 8 == 0 ? bricks / 8 : 0;
    k_conv_tile<NB, SIGN, ACT><<<dim3(bricks, cout / (16 * NB)), 256, 0, s>>>(g, x, cin, w, bias, cout, y, span, gate);
    return launched();
}

template <int SIGN, int ACT>
int conv_rows_launch(const G& g, const bf16* x, int cin, const bf16* w, const float* bias, int cout, bf16* y,
                     const bf16* gate, hipStream_t s)
{
    const unsigned blocks = (unsigned)(g.nvox / (kTD * kRH * kTW)) * (unsigned)(cout / 32);
    k_conv_rows<SIGN, ACT><<<dim3(blocks), 256, 0, s>>>(g, x, cin, w, bias, cout, y, blocks % 8 == 0 ? blocks / 8 : 0, gate);
    return launched();
}

template <int SIGN, int ACT>
int conv_dispatch(const G& g, const bf16* x, int cin, const bf16* w, const float* bias, int cout, bf16* y,
                  const bf16* gate, hipStream_t s)
{
    // the brick kernel addresses the weights with 32-bit byte offsets
    if (brick_ok(g) && 27LL * cout * cin * 2 < (1LL << 32)) {
        // widest output tile that still leaves >= 512 workgroups (two per CU)
        const long long bricks = g.nvox / (kTD * kTH * kTW);
        const int c16 = cout / 16;
        // The row kernel's workgroup does the work of four 16-channel bricks in
        // one pass, so it needs workgroups for three quarters of the CUs to win:
        // 192 -> 25 us against 29 (bricks), 256 -> 24 / 33, 512 -> 20 / 26; at 128
        // it is 11.6 / 10.6 and at 96 22 / 20.  It has 32-bit offsets within a
        // sample and stores 8 bytes at a time; its grid is one-dimensional, and a
        // launch has fewer than 2^32 work-items.
        const long long row_blocks = bricks / 2 * (c16 / 2), most_blocks = (1LL << 32) / 256 - 1;
        const bool rows32 = g.nvox / g.n * 2 * (cin > cout ? cin : cout) < (long long)kNone;
        if (g.h % kRH == 0 && row_blocks >= 192 && row_blocks <= most_blocks && rows32 && ((uintptr_t)y & 7u) == 0)
            return conv_rows_launch<SIGN, ACT>(g, x, cin, w, bias, cout, y, gate, s);
        // One workgroup of k_conv_few runs on a CU (120 KB of LDS).  While 256 of
        // them take all there is to do, it wins over the brick kernel (us, bricks /
        // this: 192 workgroups 32 -> 32 channels 9.2 / 7.5, 96 -> 96 18.5 / 14.2), but
        // not with one chunk of input channels for at most 128 workgroups, which
        // leaves it no weights to load ahead and half the workgroups of 16-channel
        // bricks (128, 32 -> 64: forward 7.5 / 7.6, data gradient 7.3 / 7.7, gated 7.8 /
        // 8.6).  In more rounds the several brick workgroups of a CU are better,
        // unless input channels in 64s make their weight rows whole lines, which
        // do not stay in L1 (64 -> 64: 768 workgroups 44 / 36, 7168 358 / 278; 128 ->
        // 128: 14336 1406 / 939; 192 -> 96: 1152 192 / 123; against 96 -> 96: 576 37 /
        // 43, 10752 481 / 595; 160 -> 64: 768 64 / 68; 32 -> 32: 288 13.5 / 15.3).
        const long long few_blocks = bricks * (c16 / 2);
        const bool few = few_blocks <= 256 ? cin > 32 || few_blocks > 128 : cin % 64 == 0;
        if (few && few_blocks <= most_blocks && rows32 && ((uintptr_t)y & 7u) == 0) {
            k_conv_few<SIGN, ACT><<<dim3((unsigned)few_blocks), 256, 0, s>>>(g, x, cin, w, bias, cout, y, gate);
            return launched();
        }
        if (c16 % 6 == 0 && bricks * (c16 / 6) >= 512) return conv_tile_launch<6, SIGN, ACT>(g, x, cin, w, bias, cout, y, gate, s);
        if (c16 % 4 == 0 && bricks * (c16 / 4) >= 512) return conv_tile_launch<4, SIGN, ACT>(g, x, cin, w, bias, cout, y, gate, s);
        // a grid of fewer workgroups than CUs takes 16-channel tiles (twice the workgroups)
        if (bricks * (c16 / 2) < 256) return conv_tile_launch<1, SIGN, ACT>(g, x, cin, w, bias, cout, y, gate, s);
        return conv_tile_launch<2, SIGN, ACT>(g, x, cin, w, bias, cout, y, gate, s);
    }
    const unsigned mb = (unsigned)((g.nvox + 63) / 64);
    if (cout % 64 == 0)
        k_conv_fwd<4, SIGN, ACT><<<dim3(mb, cout / 64), 256, 0, s>>>(g, x, cin, w, bias, cout, y, gate);
    else
        k_conv_fwd<2, SIGN, ACT><<<dim3(mb, cout / 32), 256, 0, s>>>(g, x, cin, w, bias, cout, y, gate);
    return launched();
}

// Device scratch of the entry points that allocate nothing: a file-scope
// array of fixed size, one copy per GPU, found once per device through
// hipGetSymbolAddress (host code never uses the array's name as an address).
constexpr size_t kStaticScratchBytes = size_t(64) << 20;
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// The current device's copy of `scratch`, looked up on the first call on that device.
int static_scratch(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return CMNN_EHIP;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return CMNN_EHIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return CMNN_OK;
}

// every element index a call's kernel forms is below 2^32: its 32-bit index variant
bool idx32(long long elements) { return elements < (1LL << 32); }

void gather_pack(long long nsel, const int* idx, long long nvs, const float* src, int nsrc, int cs, bf16* dst, int c,
                 hipStream_t s)
{
    const long long n8 = nsel * nvs * c / 8;
    if (idx32(nsel * nvs * c) && idx32((long long)cs * nsrc * nvs))
        k_gather_pack8<uint32_t><<<grid_for(n8), 256, 0, s>>>((int)nsel, idx, nvs, src, nsrc, cs, dst, c);
    else
        k_gather_pack8<uint64_t><<<grid_for(n8), 256, 0, s>>>((int)nsel, idx, nvs, src, nsrc, cs, dst, c);
}

// the fine level of a coarse geometry must fit the voxel limit too
bool coarse_ok(const cmnn_geom* g) { return geom_ok(g) && 8LL * g->n * g->d * g->h * g->w <= 0x7fffffffLL; }
bool ld_ok(int ld, int c) { return ld >= c && ld % 8 == 0; }
bool gate_ok(const void* gate, int act)
{
    if (act == CMNN_ACT_NONE) return true;
    return act == CMNN_ACT_LEAKY && gate && al16(gate);
}

// Per-sample channel means of x (voxel rows ldx channels apart) into
// workspace: partial sums, then the means after them; returns the means.
const float* channel_means(const cmnn_geom* g, const void* x, int ldx, int c, void* workspace, hipStream_t s)
{
    const long long vps = (long long)g->d * g->h * g->w;
    k_chmean_part<<<(unsigned)(g->n * kMeanParts), 256, 0, s>>>((const bf16*)x, ldx, vps, c, kMeanParts,
                                                                 (float*)workspace);
    if (launched()) return nullptr;
    float* mean = (float*)workspace + (size_t)g->n * kMeanParts * c;
    k_chmean_final<<<grid_for((long long)g->n * c), 256, 0, s>>>((const float*)workspace, vps, c, g->n, kMeanParts,
                                                                 mean);
    return launched() ? nullptr : mean;
}

}  // namespace

extern "C" {

int cmnn_conv3d_fwd(const cmnn_geom* g, const void* x, int32_t cin, const void* w, const float* bias, int32_t cout,
                    int32_t act, void* y, void* hip_stream)
{
    if (!geom_ok(g) || !chan_ok(cin) || !chan_ok(cout) || !x || !w || !y) return CMNN_EINVAL;
    if (!al16(x) || !al16(w) || act < CMNN_ACT_NONE || act > CMNN_ACT_LEAKY) return CMNN_EINVAL;
    const G gg = make_g(g);
    hipStream_t s = (hipStream_t)hip_stream;
    if (act == CMNN_ACT_LEAKY)
        return conv_dispatch<1, CMNN_ACT_LEAKY>(gg, (const bf16*)x, cin, (const bf16*)w, bias, cout, (bf16*)y, nullptr,
                                                s);
    return conv_dispatch<1, CMNN_ACT_NONE>(gg, (const bf16*)x, cin, (const bf16*)w, bias, cout, (bf16*)y, nullptr, s);
}

int cmnn_conv3d_bwd_data(const cmnn_geom* g, const void* dy, int32_t cout, const void* w_t, int32_t cin, void* dx,
                         void* hip_stream)
{
    if (!geom_ok(g) || !chan_ok(cin) || !chan_ok(cout) || !dy || !w_t || !dx) return CMNN_EINVAL;
    if (!al16(dy) || !al16(w_t)) return CMNN_EINVAL;
    const G gg = make_g(g);
    // the data gradient is the forward kernel with negated tap offsets, input dy
    // (cout channels), transposed weights [27][cin][cout] and cin outputs
    return conv_dispatch<-1, CMNN_ACT_NONE>(gg, (const bf16*)dy, cout, (const bf16*)w_t, nullptr, cin, (bf16*)dx,
                                            nullptr, (hipStream_t)hip_stream);
}

int cmnn_conv3d_bwd_data_act(const cmnn_geom* g, const void* dy, int32_t cout, const void* w_t, int32_t cin,
                             const void* gate, int32_t act, void* dx, void* hip_stream)
{
    if (!geom_ok(g) || !chan_ok(cin) || !chan_ok(cout) || !dy || !w_t || !dx) return CMNN_EINVAL;
    if (!al16(dy) || !al16(w_t) || act < CMNN_ACT_NONE || act > CMNN_ACT_LEAKY) return CMNN_EINVAL;
    if (act == CMNN_ACT_LEAKY && (!gate || !al16(gate) || gate == dx)) return CMNN_EINVAL;
    const G gg = make_g(g);
    if (act == CMNN_ACT_NONE)
        return conv_dispatch<-1, CMNN_ACT_NONE>(gg, (const bf16*)dy, cout, (const bf16*)w_t, nullptr, cin, (bf16*)dx,
                                                nullptr, (hipStream_t)hip_stream);
    return conv_dispatch<-1, CMNN_ACT_LEAKY>(gg, (const bf16*)dy, cout, (const bf16*)w_t, nullptr, cin, (bf16*)dx,
                                             (const bf16*)gate, (hipStream_t)hip_stream);
}

int cmnn_conv3d_bwd_weight_workspace(const cmnn_geom* g, int32_t cin, int32_t cout, size_t* bytes)
{
    if (!geom_ok(g) || !chan_ok(cin) || !chan_ok(cout) || !bytes) return CMNN_EINVAL;
    const G gg = make_g(g);
    const size_t nc = (size_t)bwd_w_chunks(gg, cin, cout);
    *bytes = nc * 27 * (size_t)cin * cout * sizeof(float) + (size_t)kColSumBlocks * cout * sizeof(float);
    return CMNN_OK;
}

int cmnn_conv3d_bwd_weight(const cmnn_geom* g, const void* x, int32_t cin, const void* dy, int32_t cout, float* dw,
                           float* dbias, void* workspace, size_t workspace_bytes, void* hip_stream)
{
    size_t need = 0;
    if (cmnn_conv3d_bwd_weight_workspace(g, cin, cout, &need) != CMNN_OK) return CMNN_EINVAL;
    if (!x || !dy || !dw || !workspace || workspace_bytes < need || !al16(x) || !al16(dy)) return CMNN_EINVAL;
    if (cout > 256) return CMNN_EINVAL;
    const G gg = make_g(g);
    hipStream_t s = (hipStream_t)hip_stream;
    const int nc = bwd_w_chunks(gg, cin, cout);
    float* part = (float*)workspace;
    const long long per = 27LL * cin * cout;
    float* bpart = part + (long long)nc * per;
    if (bwd_w_brick(gg, cin, cout)) {
        const long long bricks = gg.nvox / (kTD * kTH * kTW);
        const int per_chunk = (int)((bricks + nc - 1) / nc);
        const unsigned nblk = (unsigned)(nc * (cout / 32) * (cin / 32));
        // per chunk: the 27 x cout x cin weight partials, then the cout bias partials,
        // summed over the chunks by one launch; nc <= 256 <= kColSumBlocks, so the
        // nc * (per + cout) floats fit the workspace
        const long long pst = per + cout, nb = dbias ? cout : 0;
        k_conv_bwd_w_tile<<<nblk, kBwThreads, 0, s>>>(gg, (const bf16*)x, cin, (const bf16*)dy, cout, per_chunk, part,
                                                      pst, dbias != nullptr);
        if (launched()) return CMNN_EHIP;
        return sum_chunks(part, pst, per, nb, nc, dw, dbias, s);
    } else {
        const long long chunk = (gg.nvox + nc - 1) / nc;
        const unsigned nblk = (unsigned)(nc * 27 * (cout / 32) * (cin / 32));
        k_conv_bwd_w<<<nblk, 256, 0, s>>>(gg, (const bf16*)x, cin, (const bf16*)dy, cout, chunk, part);
    }
    if (launched()) return CMNN_EHIP;
    if (sum_chunks(part, per, per, 0, nc, dw, nullptr, s)) return CMNN_EHIP;
    if (dbias) {
        long long nb = (gg.nvox + 1023) / 1024;
        if (nb > kColSumBlocks) nb = kColSumBlocks;
        const long long bchunk = (gg.nvox + nb - 1) / nb;
        k_colsum_part<<<(unsigned)nb, 256, 0, s>>>((const bf16*)dy, gg.nvox, cout, bchunk, bpart);
        if (launched()) return CMNN_EHIP;
        if (sum_chunks(bpart, cout, cout, 0, (int)nb, dbias, nullptr, s)) return CMNN_EHIP;
    }
    return CMNN_OK;
}

int cmnn_conv3d_bwd_weight_noalloc(const cmnn_geom* g, const void* x, int32_t cin, const void* dy, int32_t cout,
                                   float* dw, float* dbias, void* hip_stream)
{
    size_t need = 0;
    if (cmnn_conv3d_bwd_weight_workspace(g, cin, cout, &need) != CMNN_OK) return CMNN_EINVAL;
    if (need > kStaticScratchBytes) return CMNN_EINVAL;  // beyond the fixed scratch: nothing enqueued
    if (!x || !dy || !dw || !al16(x) || !al16(dy) || cout > 256) return CMNN_EINVAL;
    void* ws = nullptr;
    const int rc = static_scratch(&ws);
    if (rc != CMNN_OK) return rc;
    // every partial the kernels read is written first in the same call, so the
    // previous call's contents need no clearing
    return cmnn_conv3d_bwd_weight(g, x, cin, dy, cout, dw, dbias, ws, kStaticScratchBytes, hip_stream);
}

int cmnn_act_bwd(const void* y, const void* dy, void* dpre, size_t n, int32_t act, void* hip_stream)
{
    if (!y || !dy || !dpre || act < CMNN_ACT_NONE || act > CMNN_ACT_LEAKY) return CMNN_EINVAL;
    if (n % 8 == 0 && al16(y) && al16(dy) && al16(dpre)) {
        k_act_bwd8<<<grid_for((long long)n / 8), 256, 0, (hipStream_t)hip_stream>>>(
            (const u4*)y, (const u4*)dy, (u4*)dpre, (long long)n / 8, act);
        return launched();
    }
    k_act_bwd<<<grid_for((long long)n), 256, 0, (hipStream_t)hip_stream>>>((const bf16*)y, (const bf16*)dy,
                                                                         (bf16*)dpre, (long long)n, act);
    return launched();
}

int cmnn_pool2_fwd(const cmnn_geom* g, const void* x, int32_t c, void* y, void* hip_stream)
{
    if (!geom_ok(g) || c <= 0 || !x || !y || (g->d | g->h | g->w) & 1) return CMNN_EINVAL;
    const G gg = make_g(g);
    if (c % 8 == 0 && al16(x) && al16(y))
    {
        if (idx32(gg.nvox * c))
            k_pool2_fwd8<uint32_t><<<grid_for(gg.nvox * c / 64), 256, 0, (hipStream_t)hip_stream>>>(gg, (const bf16*)x,
                                                                                                   c, (bf16*)y);
        else
            k_pool2_fwd8<uint64_t><<<grid_for(gg.nvox * c / 64), 256, 0, (hipStream_t)hip_stream>>>(gg, (const bf16*)x,
                                                                                                   c, (bf16*)y);
    }
    else
        k_pool2_fwd<<<grid_for(gg.nvox * c / 8), 256, 0, (hipStream_t)hip_stream>>>(gg, (const bf16*)x, c, (bf16*)y);
    return launched();
}

int cmnn_pool2_bwd(const cmnn_geom* g, const void* dy, int32_t c, void* dx, void* hip_stream)
{
    if (!geom_ok(g) || c <= 0 || !dy || !dx || (g->d | g->h | g->w) & 1) return CMNN_EINVAL;
    const G gg = make_g(g);
    if (c % 8 == 0 && al16(dy) && al16(dx))
        k_pool2_bwd8<<<grid_for(gg.nvox * c / 8), 256, 0, (hipStream_t)hip_stream>>>(gg, (const bf16*)dy, c, (bf16*)dx);
    else
        k_pool2_bwd<<<grid_for(gg.nvox * c), 256, 0, (hipStream_t)hip_stream>>>(gg, (const bf16*)dy, c, (bf16*)dx);
    return launched();
}

int cmnn_up2_fwd(const cmnn_geom* g, const void* x, int32_t c, void* y, void* hip_stream)
{
    if (!geom_ok(g) || c <= 0 || !x || !y) return CMNN_EINVAL;
    const G gg = make_g(g);
    if (c % 8 == 0 && al16(x) && al16(y))
        k_up2_fwd8<<<grid_for(gg.nvox * c), 256, 0, (hipStream_t)hip_stream>>>(gg, (const bf16*)x, c, (bf16*)y);
    else
        k_up2_fwd<<<grid_for(gg.nvox * c * 8), 256, 0, (hipStream_t)hip_stream>>>(gg, (const bf16*)x, c, (bf16*)y);
    return launched();
}

int cmnn_up2_bwd(const cmnn_geom* g, const void* dy, int32_t c, void* dx, void* hip_stream)
{
    if (!geom_ok(g) || c <= 0 || !dy || !dx) return CMNN_EINVAL;
    const G gg = make_g(g);
    if (c % 8 == 0 && al16(dy) && al16(dx))
        k_up2_bwd8<<<grid_for(gg.nvox * c / 8), 256, 0, (hipStream_t)hip_stream>>>(gg, (const bf16*)dy, c, (bf16*)dx);
    else
        k_up2_bwd<<<grid_for(gg.nvox * c), 256, 0, (hipStream_t)hip_stream>>>(gg, (const bf16*)dy, c, (bf16*)dx);
    return launched();
}

int cmnn_concat_fwd(size_t nvox, const void* a, int32_t ca, const void* b, int32_t cb, void* y, void* hip_stream)
{
    if (!a || !b || !y || ca <= 0 || cb <= 0) return CMNN_EINVAL;
    if (ca % 8 == 0 && cb % 8 == 0 && al16(a) && al16(b) && al16(y))
        k_concat_fwd8<<<grid_for((long long)nvox * (ca + cb) / 8), 256, 0, (hipStream_t)hip_stream>>>(
            (long long)nvox, (const bf16*)a, ca, (const bf16*)b, cb, (bf16*)y);
    else
        k_concat_fwd<<<grid_for((long long)nvox * (ca + cb)), 256, 0, (hipStream_t)hip_stream>>>(
            (long long)nvox, (const bf16*)a, ca, (const bf16*)b, cb, (bf16*)y);
    return launched();
}

int cmnn_concat_bwd(size_t nvox, const void* dy, int32_t ca, int32_t cb, void* da, void* db, void* hip_stream)
{
    if (!dy || ca <= 0 || cb <= 0) return CMNN_EINVAL;
    if (ca % 8 == 0 && cb % 8 == 0 && al16(dy) && al16(da) && al16(db))
        k_concat_bwd8<<<grid_for((long long)nvox * (ca + cb) / 8), 256, 0, (hipStream_t)hip_stream>>>(
            (long long)nvox, (const bf16*)dy, ca, cb, (bf16*)da, (bf16*)db);
    else
        k_concat_bwd<<<grid_for((long long)nvox * (ca + cb)), 256, 0, (hipStream_t)hip_stream>>>(
            (long long)nvox, (const bf16*)dy, ca, cb, (bf16*)da, (bf16*)db);
    return launched();
}

int cmnn_up2_concat_fwd(const cmnn_geom* g, const void* skip, int32_t cs, const void* x, int32_t cx, void* y,
                        void* hip_stream)
{
    if (!coarse_ok(g) || !chan_ok(cs) || !chan_ok(cx) || !skip || !x || !y || !al16(skip) || !al16(x) || !al16(y))
        return CMNN_EINVAL;
    const G gg = make_g(g);
    if (idx32(8 * gg.nvox * (cs + cx)))
        k_up2_concat_fwd8<uint32_t><<<grid_for(8 * gg.nvox * (cs + cx) / 8), 256, 0, (hipStream_t)hip_stream>>>(
            gg, (const bf16*)skip, cs, (const bf16*)x, cx, (bf16*)y);
    else
        k_up2_concat_fwd8<uint64_t><<<grid_for(8 * gg.nvox * (cs + cx) / 8), 256, 0, (hipStream_t)hip_stream>>>(
            gg, (const bf16*)skip, cs, (const bf16*)x, cx, (bf16*)y);
    return launched();
}

int cmnn_up2_bwd_act(const cmnn_geom* g, const void* dy, int32_t ldy, int32_t c, const void* gate, int32_t act,
                     void* dx, void* hip_stream)
{
    if (!coarse_ok(g) || !chan_ok(c) || !ld_ok(ldy, c) || !dy || !dx || !al16(dy) || !al16(dx) || !gate_ok(gate, act))
        return CMNN_EINVAL;
    const G gg = make_g(g);
    if (idx32(8 * gg.nvox * ldy))
        k_up2_bwd_act8<uint32_t><<<grid_for(gg.nvox * c / 8), 256, 0, (hipStream_t)hip_stream>>>(
            gg, (const bf16*)dy, ldy, c, (const bf16*)gate, act, (bf16*)dx);
    else
        k_up2_bwd_act8<uint64_t><<<grid_for(gg.nvox * c / 8), 256, 0, (hipStream_t)hip_stream>>>(
            gg, (const bf16*)dy, ldy, c, (const bf16*)gate, act, (bf16*)dx);
    return launched();
}

int cmnn_pool2_bwd_add_act(const cmnn_geom* g, const void* dy, int32_t c, const void* skip, int32_t ldskip,
                           const void* gate, int32_t act, void* dx, void* hip_stream)
{
    if (!geom_ok(g) || (g->d | g->h | g->w) & 1 || !chan_ok(c) || !dy || !dx || !al16(dy) || !al16(dx) ||
        !gate_ok(gate, act))
        return CMNN_EINVAL;
    if (skip && (!al16(skip) || !ld_ok(ldskip, c))) return CMNN_EINVAL;
    const G gg = make_g(g);
    if (idx32(gg.nvox * (skip && ldskip > c ? ldskip : c)))
        k_pool2_bwd_add_act8<uint32_t><<<grid_for(gg.nvox * c / 8), 256, 0, (hipStream_t)hip_stream>>>(
            gg, (const bf16*)dy, c, (const bf16*)skip, ldskip, (const bf16*)gate, act, (bf16*)dx);
    else
        k_pool2_bwd_add_act8<uint64_t><<<grid_for(gg.nvox * c / 8), 256, 0, (hipStream_t)hip_stream>>>(
            gg, (const bf16*)dy, c, (const bf16*)skip, ldskip, (const bf16*)gate, act, (bf16*)dx);
    return launched();
}

int cmnn_add(size_t n, const void* a, const void* b, void* y, void* hip_stream)
{
    if (!a || !b || !y) return CMNN_EINVAL;
    if (n % 8 == 0 && al16(a) && al16(b) && al16(y))
        k_add8<<<grid_for((long long)n / 8), 256, 0, (hipStream_t)hip_stream>>>((long long)n / 8, (const u4*)a,
                                                                               (const u4*)b, (u4*)y);
    else
        k_add<<<grid_for((long long)n), 256, 0, (hipStream_t)hip_stream>>>((long long)n, (const bf16*)a,
                                                                         (const bf16*)b, (bf16*)y);
    return launched();
}

int cmnn_channel_mean_workspace(const cmnn_geom* g, int32_t c, size_t* bytes)
{
    if (!geom_ok(g) || c <= 0 || c > 256 || !bytes || (long long)g->n * kMeanParts > 0x7fffffffLL) return CMNN_EINVAL;
    *bytes = (size_t)g->n * (kMeanParts + 1) * c * sizeof(float);
    return CMNN_OK;
}

int cmnn_channel_mean(const cmnn_geom* g, const void* x, int32_t c, void* y, void* workspace, size_t workspace_bytes,
                      void* hip_stream)
{
    size_t need = 0;
    if (cmnn_channel_mean_workspace(g, c, &need) != CMNN_OK || !x || !y || !workspace || workspace_bytes < need)
        return CMNN_EINVAL;
    const G gg = make_g(g);
    hipStream_t s = (hipStream_t)hip_stream;
    const long long vps = (long long)g->d * g->h * g->w;
    k_chmean_part<<<(unsigned)(g->n * kMeanParts), 256, 0, s>>>((const bf16*)x, c, vps, c, kMeanParts,
                                                                 (float*)workspace);
    if (launched()) return CMNN_EHIP;
    if (c % 8 == 0 && al16(y)) {
        float* mean = (float*)workspace + (size_t)g->n * kMeanParts * c;
        k_chmean_final<<<grid_for((long long)g->n * c), 256, 0, s>>>((const float*)workspace, vps, c, g->n,
                                                                     kMeanParts, mean);
        if (launched()) return CMNN_EHIP;
        k_chmean_bcast8<<<grid_for(gg.nvox * c / 8), 256, 0, s>>>(mean, vps, c, (bf16*)y, gg.nvox * c / 8);
        return launched();
    }
    k_chmean_bcast<<<grid_for(gg.nvox * c), 256, 0, s>>>((const float*)workspace, vps, c, g->n, kMeanParts, (bf16*)y);
    return launched();
}

int cmnn_channel_mean_concat(const cmnn_geom* g, const void* x, int32_t c, void* y, void* workspace,
                             size_t workspace_bytes, void* hip_stream)
{
    size_t need = 0;
    if (cmnn_channel_mean_workspace(g, c, &need) != CMNN_OK || !chan_ok(c) || !x || !y || !al16(x) || !al16(y) ||
        !workspace || workspace_bytes < need)
        return CMNN_EINVAL;
    hipStream_t s = (hipStream_t)hip_stream;
    const float* mean = channel_means(g, x, c, c, workspace, s);
    if (!mean) return CMNN_EHIP;
    const long long total8 = make_g(g).nvox * 2 * c / 8;
    k_chmean_concat8<<<grid_for(total8), 256, 0, s>>>(mean, (long long)g->d * g->h * g->w, c, (const bf16*)x,
                                                      (bf16*)y, total8);
    return launched();
}

int cmnn_channel_mean_add_act(const cmnn_geom* g, const void* dy, int32_t ldy, int32_t c, const void* skip,
                              int32_t ldskip, const void* gate, int32_t act, void* dx, void* workspace,
                              size_t workspace_bytes, void* hip_stream)
{
    size_t need = 0;
    if (cmnn_channel_mean_workspace(g, c, &need) != CMNN_OK || !chan_ok(c) || !ld_ok(ldy, c) || !ld_ok(ldskip, c) ||
        !dy || !skip || !dx || !al16(dy) || !al16(skip) || !al16(dx) || !gate_ok(gate, act) || !workspace ||
        workspace_bytes < need)
        return CMNN_EINVAL;
    hipStream_t s = (hipStream_t)hip_stream;
    const float* mean = channel_means(g, dy, ldy, c, workspace, s);
    if (!mean) return CMNN_EHIP;
    const long long total8 = make_g(g).nvox * c / 8;
    k_chmean_add_act8<<<grid_for(total8), 256, 0, s>>>(mean, (long long)g->d * g->h * g->w, c, (const bf16*)skip,
                                                       ldskip, (const bf16*)gate, act, (bf16*)dx, total8);
    return launched();
}

int cmnn_mse_workspace(size_t nvox, size_t* bytes)
{
    if (!bytes || nvox == 0) return CMNN_EINVAL;
    *bytes = 2 * kMseBlocks * sizeof(float);
    return CMNN_OK;
}

int cmnn_mse(size_t nvox, const void* pred, int32_t c, int32_t creal, const float* target, const float* weight,
             float* loss_out, void* dpred, void* workspace, size_t workspace_bytes, void* hip_stream)
{
    if (!pred || !target || !weight || !loss_out || !workspace || nvox == 0) return CMNN_EINVAL;
    if (c <= 0 || creal <= 0 || creal > c || workspace_bytes < 2 * kMseBlocks * sizeof(float)) return CMNN_EINVAL;
    hipStream_t s = (hipStream_t)hip_stream;
    float* part = (float*)workspace;
    k_mse_part<<<kMseBlocks, 256, 0, s>>>((long long)nvox, (const bf16*)pred, c, creal, target, weight, part);
    if (launched()) return CMNN_EHIP;
    // loss_out[0] = loss, loss_out[1] = normaliser (callers pass two floats)
    k_mse_final<<<1, 256, 0, s>>>(part, kMseBlocks, creal, loss_out);
    if (launched()) return CMNN_EHIP;
    if (dpred && c % 8 == 0 && al16(pred) && al16(dpred)) {
        if (idx32((long long)nvox * c))
            k_mse_grad8<uint32_t><<<grid_for((long long)nvox * c / 8), 256, 0, s>>>(
                (long long)nvox, (const bf16*)pred, c, creal, target, weight, loss_out, (bf16*)dpred);
        else
            k_mse_grad8<uint64_t><<<grid_for((long long)nvox * c / 8), 256, 0, s>>>(
                (long long)nvox, (const bf16*)pred, c, creal, target, weight, loss_out, (bf16*)dpred);
        if (launched()) return CMNN_EHIP;
    } else if (dpred) {
        k_mse_grad<<<grid_for((long long)nvox * c), 256, 0, s>>>((long long)nvox, (const bf16*)pred, c, creal, target,
                                                               weight, loss_out, (bf16*)dpred);
        if (launched()) return CMNN_EHIP;
    }
    return CMNN_OK;
}

int cmnn_clip_grad_norm_workspace(size_t n, size_t* bytes)
{
    if (!bytes || n == 0) return CMNN_EINVAL;
    *bytes = kClipBlocks * sizeof(float);
    return CMNN_OK;
}

int cmnn_clip_grad_norm(size_t n, float* grad, float max_norm, float* norm_out, void* workspace,
                        size_t workspace_bytes, void* hip_stream)
{
    if (!grad || !norm_out || !workspace || n == 0 || workspace_bytes < kClipBlocks * sizeof(float) ||
        !(max_norm >= 0.f))
        return CMNN_EINVAL;
    hipStream_t s = (hipStream_t)hip_stream;
    float* part = (float*)workspace;
    k_sumsq_part<<<kClipBlocks, 256, 0, s>>>((long long)n, grad, part);
    if (launched()) return CMNN_EHIP;
    k_clip_final<<<1, 256, 0, s>>>(part, kClipBlocks, max_norm, norm_out);
    if (launched()) return CMNN_EHIP;
    k_scale<<<grid_for((long long)n), 256, 0, s>>>((long long)n, grad, norm_out);
    return launched();
}

int cmnn_adam(size_t n, float* param, const float* grad, float* m, float* v, float lr, float beta1, float beta2,
              float eps, float weight_decay, int32_t step, void* hip_stream)
{
    if (!param || !grad || !m || !v || step < 1) return CMNN_EINVAL;
    const float c1 = 1.f - powf(beta1, (float)step), c2 = 1.f - powf(beta2, (float)step);
    k_adam<<<grid_for((long long)n), 256, 0, (hipStream_t)hip_stream>>>((long long)n, param, grad, m, v, lr, beta1,
                                                                      beta2, eps, weight_decay, c1, c2);
    return launched();
}

int cmnn_pack_weights(const float* w, int32_t cin, int32_t cout, void* w_fwd, void* w_t, void* hip_stream)
{
    if (!w || !w_fwd || !w_t || cin <= 0 || cout <= 0) return CMNN_EINVAL;
    k_pack_w<<<grid_for(27LL * cin * cout), 256, 0, (hipStream_t)hip_stream>>>(w, cin, cout, (bf16*)w_fwd, (bf16*)w_t);
    return launched();
}

int cmnn_pack_weights_batch(int32_t n, const cmnn_pack_job* jobs, void* hip_stream)
{
    if (n <= 0 || n > CMNN_PACK_MAX || !jobs) return CMNN_EINVAL;
    PackJobs J = {};
    long long blocks = 0;
    for (int l = 0; l < n; ++l) {
        const cmnn_pack_job& j = jobs[l];
        if (!j.w || !j.w_fwd || !j.w_t || j.cin <= 0 || j.cout <= 0) return CMNN_EINVAL;
        J.w[l] = j.w;
        J.wf[l] = (bf16*)j.w_fwd;
        J.wt[l] = (bf16*)j.w_t;
        J.cin[l] = j.cin;
        J.cout[l] = j.cout;
        J.first_block[l] = (int)blocks;
        blocks += (27LL * j.cin * j.cout + 255) / 256;
        if (blocks > 0x7fffffffLL) return CMNN_EINVAL;
    }
    J.first_block[n] = (int)blocks;
    J.n = n;
    k_pack_w_batch<<<(unsigned)blocks, 256, 0, (hipStream_t)hip_stream>>>(J);
    return launched();
}

int cmnn_pack_channels(size_t nvox, const float* src, int32_t cs, void* dst, int32_t c, void* hip_stream)
{
    if (!src || !dst || cs <= 0 || c < cs) return CMNN_EINVAL;
    if (c % 8 == 0 && al16(dst)) {
        // one "sample" of nvox voxels, taken in place
        gather_pack((long long)1, nullptr, (long long)nvox, src, 1, cs, (bf16*)dst, c, (hipStream_t)hip_stream);
        return launched();
    }
    k_pack_ch<<<grid_for((long long)nvox * c), 256, 0, (hipStream_t)hip_stream>>>((long long)nvox, src, cs, (bf16*)dst,
                                                                                c);
    return launched();
}

int cmnn_gather_pack_channels(int32_t nsel, const int32_t* idx, size_t nvs, const float* src, int32_t nsrc,
                              int32_t cs, void* dst, int32_t c, void* hip_stream)
{
    if (nsel <= 0 || !idx || nvs == 0 || !src || nsrc <= 0 || cs <= 0 || c < cs || c % 8 != 0 || !dst || !al16(dst))
        return CMNN_EINVAL;
    gather_pack(nsel, idx, (long long)nvs, src, nsrc, cs, (bf16*)dst, c, (hipStream_t)hip_stream);
    return launched();
}

int cmnn_gather_samples(int32_t nsel, const int32_t* idx, size_t nvs, const float* src, int32_t nsrc, int32_t np,
                        float* dst, void* hip_stream)
{
    if (nsel <= 0 || !idx || nvs == 0 || !src || nsrc <= 0 || np <= 0 || !dst) return CMNN_EINVAL;
    if (nvs % 4 == 0 && al16(src) && al16(dst))
        k_gather4<<<grid_for((long long)np * nsel * nvs / 4), 256, 0, (hipStream_t)hip_stream>>>(
            nsel, idx, (long long)nvs / 4, (const float4*)src, nsrc, np, (float4*)dst);
    else
        k_gather1<<<grid_for((long long)np * nsel * nvs), 256, 0, (hipStream_t)hip_stream>>>(nsel, idx, (long long)nvs,
                                                                                          src, nsrc, np, dst);
    return launched();
}

int cmnn_unpack_channels(size_t nvox, const void* src, int32_t c, float* dst, int32_t cs, void* hip_stream)
{
    if (!src || !dst || cs <= 0 || c < cs) return CMNN_EINVAL;
    k_unpack_ch<<<grid_for((long long)nvox * cs), 256, 0, (hipStream_t)hip_stream>>>((long long)nvox, (const bf16*)src,
                                                                                   c, dst, cs);
    return launched();
}

}  // extern "C"
