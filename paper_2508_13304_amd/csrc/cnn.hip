// Learned pose proposal: the layers of a small strided CNN on BF16 matrix
// cores (MFMA) with FP32 accumulation.  The network regresses a 6-DoF pose
// offset from a pair of DRRs rendered by the forward projector; its output
// initialises the analytic-gradient registration.
//
// Layout: activations are NHWC (row m = (n, y, x), column = channel), so a
// 3x3 strided convolution is
//   col  = im2col(x)            [M = N Ho Wo][K = 9 Ci], K index (ky, kx, ci)
//   z    = col . W^T            W [Co][K]                  (GEMM, MFMA)
//   y    = relu(z + b)          fused epilogue, BF16 out
// and its backward is
//   dz   = dy * (y > 0)
//   dW   = dz^T . col           [Co][K]                    (GEMM, MFMA)
//   db   = column sums of dz
//   dcol = dz . W               [M][K]                     (GEMM, MFMA)
//   dx   = col2im(dcol)         gather of the overlapping windows.
//
// GEMM: C[M][N] (FP32) = op(A) op(B) (+ C if accumulate), A/B BF16.  A block
// computes a 128x128, 128x64 or 64x64 tile with 2 x 2 wavefronts, or a 128x32 or
// 64x32 one with 4 x 1 (MFMA 16x16x32 tiles); K advances by 64 through LDS.  Operand lane layout of
// v_mfma_f32_16x16x32_bf16: lane l supplies row (l % 16) of A and column
// (l % 16) of B, each with the 8 consecutive k = 8 (l / 16) .. +7; it receives
// D rows 4 (l / 16) .. +3 of column (l % 16).
#include <algorithm>
#include <type_traits>

#include "dp_internal.h"
#include "gemm_plan.h"

namespace dp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kGT = 64;          // smallest block tile (M and N)
constexpr int kBK = 64;          // K step (two MFMA steps)
constexpr int kKP = kBK + 8;     // pitch of a k-major tile S[row][k]: rows 4 banks apart
// pitch of a row-major tile T[k][row] of R rows: the four k rows one 16-lane
// group of a transpose read touches start 8 banks apart
constexpr int t_pitch(int R) { return R + 16; }

__device__ inline __bf16 to_bf16(float x) { return (__bf16)x; }

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef short i16x8 __attribute__((ext_vector_type(8)));

// MFMA operand fragment of rows rb .. rb + 15 at step k of a tile: lane l gets
// row rb + (l % 16), k + 8 (l / 16) .. + 7.  From a k-major tile that is one
// 16-byte read.  From a row-major tile of R rows it is two transpose reads
// (ds_read_b64_tr_b16): within each 16-lane group, the lane i' = 4 j + q
// addresses the four rows 4 q .. 4 q + 3 at one k (8 bytes) and lane i
// receives, as element j, the element i % 4 of lane 4 j + i / 4's four; so
// lane i gets row i at the four k the group's lanes addressed.
template <bool KC, int R>
__device__ inline bf16x8 load_frag(const __bf16* S, int rb, int k, int lane)
{
    if constexpr (KC) {
        return *(const bf16x8*)&S[(rb + (lane & 15)) * kKP + k + (lane >> 4) * 8];
    } else {
        const int i = lane & 15, kk = k + (lane >> 4) * 8 + (i >> 2);
        typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
        const __bf16* p = S + kk * t_pitch(R) + rb + 4 * (i & 3);
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)p);
        const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p + 4 * t_pitch(R)));
        const i16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8, v);
    }
}

// Exact unsigned division by a divisor fixed at launch (multiply-high and
// shift; Granlund and Montgomery's method with a 33-bit magic number split
// into a 32-bit multiplier and an add-and-halve step).  Valid for every
// 32-bit dividend.
struct FastDiv {
    unsigned d, mul, sh;
    FastDiv() = default;
    explicit FastDiv(unsigned div) : d(div), mul(0), sh(0)
    {
        while ((1ull << sh) < div) ++sh;  // sh = ceil(log2 d)
        if (sh > 0) mul = (unsigned)((((1ull << sh) - div) << 32) / div + 1);
    }
    __device__ unsigned div(unsigned n) const
    {
        if (sh == 0) return n;
        const unsigned t = __umulhi(n, mul);
        return (t + ((n - t) >> 1)) >> (sh - 1);
    }
};

// ---------------------------------------------------------------------------
// Operand sources.  A block stages the R x 64 (rows x k) tile of an operand in
// chunks of 8 elements, R / 32 per thread: k-major tiles S[row][k] if KC (the
// operand is k-contiguous), else row-major tiles T[k][row] (row-contiguous; the
// transpose happens when the fragments are read).  A thread's chunks share
// their k (KC: rows 32 apart) or their rows (else: k apart), so a source keeps
// what it can over the K loop (init):
//   fetch(st, k0, kend, tid, out): the thread's chunks at step k0, zero outside
//   [0, rows) x [k0, kend).
// ---------------------------------------------------------------------------

template <bool KC, int R>
struct Chunk {
    static constexpr int N = R / 32;
    // first row and k (relative to the tile) of a thread's chunk u
    __device__ static int row(int tid, int u) { return KC ? (tid >> 3) + 32 * u : (tid % (R / 8)) * 8; }
    __device__ static int k(int tid, int u) { return KC ? (tid & 7) * 8 : tid / (R / 8) + (2048 / R) * u; }
    __device__ static int at(int tid, int u)
    {
        return KC ? row(tid, u) * kKP + k(tid, u) : k(tid, u) * t_pitch(R) + row(tid, u);
    }
};

// Chunks are read with raw buffer loads: a 32-bit byte offset per lane from a
// wave-uniform base, and kOut, past the descriptor's end, where there is
// nothing to read (the load returns zeros): no branches around the loads.
constexpr unsigned kOut = 0xFFFFFFFFu;

__device__ inline __amdgpu_buffer_rsrc_t tile_rsrc(const __bf16* base)
{
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)kOut, 0x00020000);
}

__device__ inline uint4 load8(__amdgpu_buffer_rsrc_t r, unsigned off)
{
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

// A dense BF16 matrix (k-contiguous if KC).
template <bool KC_, Vec VEC>
struct DenseSrc {
    static constexpr bool KC = KC_, kGuarded = VEC != kWhole;
    const __bf16* P;
    int ld, rows;
    template <int R>
    struct St { int row0; unsigned off[R / 32]; };
    template <int R>
    __device__ St<R> init(int row0, int tid) const
    {
        St<R> st;
        st.row0 = row0;
#pragma unroll
        for (int u = 0; u < R / 32; ++u) {
            const int r = Chunk<KC, R>::row(tid, u), k = Chunk<KC, R>::k(tid, u);
            // (read for kWhole only: ld < kWholeLd there, or the operand has less than 2^31 elements)
            st.off[u] = row0 + r < rows ? 2u * (KC ? (unsigned)r * (unsigned)ld + (unsigned)k : (unsigned)k * (unsigned)ld + (unsigned)r)
                                        : kOut;
        }
        return st;
    }
    template <int R>
    __device__ void fetch(const St<R>& st, int k0, int kend, int tid, uint4 (&o)[R / 32]) const
    {
        if constexpr (VEC == kWhole) {
            const __amdgpu_buffer_rsrc_t r = tile_rsrc(P + (KC ? (size_t)st.row0 * ld + k0 : (size_t)k0 * ld + st.row0));
#pragma unroll
            for (int u = 0; u < R / 32; ++u)
                o[u] = load8(r, k0 + Chunk<KC, R>::k(tid, u) < kend ? st.off[u] : kOut);
            return;
        }
#pragma unroll
        for (int u = 0; u < R / 32; ++u) {
            const int row = st.row0 + Chunk<KC, R>::row(tid, u), k = k0 + Chunk<KC, R>::k(tid, u);
            const __bf16* p = P + (KC ? (size_t)row * ld + k : (size_t)k * ld + row);
            // how many of the chunk's 8 elements exist
            const int n = KC ? (row < rows ? kend - k : 0) : (k < kend ? rows - row : 0);
            union { uint4 v; __bf16 h[8]; } c;
            if (VEC == kRagged && n >= 8) {
                c.v = *(const uint4*)p;
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) c.h[j] = j < n ? p[j] : to_bf16(0.f);
            }
            o[u] = c.v;
        }
    }
};

// 3x3 convolution geometry (padding 1, stride s) on NHWC BF16 input with C
// channels, C a multiple of 8: output pixel m = (n, yo, xo), column
// k = (3 ky + kx) C + ci of the implicit im2col matrix; column 9 C is the
// ones column if `ones`, further columns are zero.
struct ConvGeo {
    int H, W, C, s, Ho, Wo, M;  // M = N Ho Wo output pixels
    int ones;
    FastDiv hw, w, c;            // by Ho Wo, Wo, C
};

// A row offset that takes every row (fewer than 2^28: at least 8 channels, 2^31
// elements) out of the image: chunks beyond the reduction.
constexpr int kNoRow = -(1 << 30);

// The im2col matrix of the input x as the GEMM's A (rows = output pixels,
// KC): a thread keeps its rows' first tap, and per step the tap of its k.
struct Im2colA {
    static constexpr bool KC = true, kGuarded = false;
    const __bf16* x;  // (below 2^32 bytes)
    ConvGeo g;
    template <int R>
    struct St { unsigned off[R / 32]; int y[R / 32], x[R / 32]; };
    template <int R>
    __device__ St<R> init(int row0, int tid) const
    {
        St<R> st;
#pragma unroll
        for (int u = 0; u < R / 32; ++u) {
            const int m = row0 + Chunk<true, R>::row(tid, u);
            const unsigned n = g.hw.div((unsigned)m), r = (unsigned)m - n * (unsigned)(g.Ho * g.Wo);
            const unsigned yo = g.w.div(r);
            const int y0 = (int)yo * g.s - 1, x0 = ((int)r - (int)yo * g.Wo) * g.s - 1;
            st.off[u] = 2u * (((n * (unsigned)g.H + (unsigned)y0) * (unsigned)g.W + (unsigned)x0) * (unsigned)g.C);
            st.y[u] = m < g.M ? y0 : -4;  // (no tap of a row beyond the last is inside)
            st.x[u] = x0;
        }
        return st;
    }
    template <int R>
    __device__ void fetch(const St<R>& st, int k0, int kend, int tid, uint4 (&o)[R / 32]) const
    {
        const unsigned k = (unsigned)(k0 + Chunk<true, R>::k(tid, 0));  // the chunks' common k
        const unsigned t = g.c.div(k);
        const int ky = (int)k < kend ? (int)t / 3 : kNoRow, kx = (int)t - 3 * ((int)t / 3);
        const unsigned tap = 2u * (((t / 3) * (unsigned)g.W + (unsigned)kx) * (unsigned)g.C + (k - t * (unsigned)g.C));
        const __amdgpu_buffer_rsrc_t r = tile_rsrc(x);
#pragma unroll
        for (int u = 0; u < R / 32; ++u) {
            const bool in = (unsigned)(st.y[u] + ky) < (unsigned)g.H && (unsigned)(st.x[u] + kx) < (unsigned)g.W;
            o[u] = load8(r, in ? st.off[u] + tap : kOut);
        }
    }
};

// The im2col matrix as the B of the weight gradient dW = dz^T . col: rows =
// im2col columns (the GEMM's N), k = output pixels (row-major tile): a thread
// keeps its columns' tap.
struct Im2colB {
    static constexpr bool KC = false, kGuarded = false;
    const __bf16* x;
    ConvGeo g;  // (columns past the product's are zero and not stored)
    template <int R>
    struct St { int dy, dx; unsigned ci, fill; bool tap; };
    template <int R>
    __device__ St<R> init(int row0, int tid) const
    {
        const int col = row0 + Chunk<false, R>::row(tid, 0), K9 = 9 * g.C;
        St<R> st;
        const unsigned t = g.c.div((unsigned)min(col, K9 - 1));
        st.dy = (int)t / 3 - 1;
        st.dx = (int)t - 3 * ((int)t / 3) - 1;
        st.ci = (unsigned)col - t * (unsigned)g.C;
        st.tap = col < K9;
        st.fill = g.ones && col == K9 ? 0x3F80u : 0u;  // BF16 1.0 in the low half
        return st;
    }
    template <int R>
    __device__ void fetch(const St<R>& st, int k0, int kend, int tid, uint4 (&o)[R / 32]) const
    {
        const __amdgpu_buffer_rsrc_t rs = tile_rsrc(x);
#pragma unroll
        for (int u = 0; u < R / 32; ++u) {
            const int m = k0 + Chunk<false, R>::k(tid, u);
            const unsigned n = g.hw.div((unsigned)m), r = (unsigned)m - n * (unsigned)(g.Ho * g.Wo);
            const int yo = (int)g.w.div(r), xo = (int)r - yo * g.Wo;
            const int y = yo * g.s + st.dy, xx = xo * g.s + st.dx;
            const bool in = m < kend && st.tap && (unsigned)y < (unsigned)g.H && (unsigned)xx < (unsigned)g.W;
            o[u] = load8(rs, in ? 2u * (((n * (unsigned)g.H + (unsigned)y) * (unsigned)g.W + (unsigned)xx) * (unsigned)g.C + st.ci)
                                : kOut);
            if (!st.tap && m < kend) o[u].x = st.fill;
        }
    }
};

// The same for a two-channel input (the network's image pair; one pixel is one
// 32-bit load): a chunk holds four taps, the third one tap 8 and the ones column.
struct Im2colB2 {
    static constexpr bool KC = false, kGuarded = false;
    const __bf16* x;
    ConvGeo g;
    template <int R>
    struct St { int t0; };
    template <int R>
    __device__ St<R> init(int row0, int tid) const { return {(row0 + Chunk<false, R>::row(tid, 0)) / 2}; }
    template <int R>
    __device__ void fetch(const St<R>& st, int k0, int kend, int tid, uint4 (&o)[R / 32]) const
    {
        const __amdgpu_buffer_rsrc_t rs = tile_rsrc(x);
#pragma unroll
        for (int u = 0; u < R / 32; ++u) {
            const int m = k0 + Chunk<false, R>::k(tid, u);
            const unsigned n = g.hw.div((unsigned)m), r = (unsigned)m - n * (unsigned)(g.Ho * g.Wo);
            const int yo = (int)g.w.div(r), xo = (int)r - yo * g.Wo;
            o[u] = taps2(g, rs, (int)n, yo * g.s - 1, xo * g.s - 1, st.t0, m < kend);
            if (st.t0 == 8 && m < kend && g.ones) o[u].y = 0x3F80u;  // BF16 1.0 in column 18
        }
    }
    // taps t0 .. t0 + 3 of the window at (y0, x0) of image n (zero beyond tap 8 or outside)
    __device__ static uint4 taps2(const ConvGeo& g, __amdgpu_buffer_rsrc_t rs, int n, int y0, int x0,
                                  int t0, bool ok)
    {
        unsigned v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int t = t0 + j, ky = t / 3, y = y0 + ky, xx = x0 + t - 3 * ky;
            const bool in = ok && t < 9 && (unsigned)y < (unsigned)g.H && (unsigned)xx < (unsigned)g.W;
            v[j] = (unsigned)__builtin_amdgcn_raw_buffer_load_b32(
                rs, in ? 4u * (((unsigned)n * (unsigned)g.H + (unsigned)y) * (unsigned)g.W + (unsigned)xx) : kOut, 0, 0);
        }
        return make_uint4(v[0], v[1], v[2], v[3]);
    }
};

// Input gradient of a 3x3 convolution, one parity class (py, px) of input
// pixels y = s y' + py, x = s x' + px at a time: such a pixel receives tap
// (ky, kx) exactly when s divides py + 1 - ky and px + 1 - kx, from output
// pixel (y' + (py + 1 - ky) / s, x' + (px + 1 - kx) / s).  So the class is
// the product dx[m'][ci] = sum_{(t, co)} dz[pixel(m', t)][co] W[co][tap t][ci]
// over its taps t, with no overlap between classes (no col2im).
// Tap j of an axis: ky0 + j s from output offset dy0 - j.
struct DgradClass {
    int py, px, Hc, Wc, M;      // class pixels: N Hc Wc
    int nky, nkx;               // taps of the class
    int ky0, kx0, dy0, dx0;
    FastDiv hw, w, nkxd;        // by Hc Wc, Wc, nkx
};
struct DgradGeo {
    int H, W, Ci, Co, s, Ho, Wo;
    FastDiv co;                 // by Co
};

struct DgradA {
    static constexpr bool KC = true, kGuarded = false;
    const __bf16* dz;  // [N][Ho][Wo][Co]
    DgradGeo g;
    DgradClass c;
    template <int R>
    struct St { unsigned off[R / 32]; int y[R / 32], x[R / 32]; };
    template <int R>
    __device__ St<R> init(int row0, int tid) const
    {
        St<R> st;
#pragma unroll
        for (int u = 0; u < R / 32; ++u) {
            const int m = row0 + Chunk<true, R>::row(tid, u);
            const unsigned n = c.hw.div((unsigned)m), r = (unsigned)m - n * (unsigned)(c.Hc * c.Wc);
            const unsigned yc = c.w.div(r), xc = r - yc * (unsigned)c.Wc;
            st.off[u] = 2u * (((n * (unsigned)g.Ho + yc) * (unsigned)g.Wo + xc) * (unsigned)g.Co);
            st.y[u] = m < c.M ? (int)yc : kNoRow / 2;
            st.x[u] = (int)xc;
        }
        return st;
    }
    template <int R>
    __device__ void fetch(const St<R>& st, int k0, int kend, int tid, uint4 (&o)[R / 32]) const
    {
        const unsigned k = (unsigned)(k0 + Chunk<true, R>::k(tid, 0));
        const unsigned t = g.co.div(k), ty = c.nkxd.div(t), tx = t - ty * (unsigned)c.nkx;
        const int dy = (int)k < kend ? c.dy0 - (int)ty : kNoRow, dx = c.dx0 - (int)tx;
        const unsigned tap = 2u * (((unsigned)(c.dy0 - (int)ty) * (unsigned)g.Wo + (unsigned)dx) * (unsigned)g.Co +
                                   (k - t * (unsigned)g.Co));
        const __amdgpu_buffer_rsrc_t r = tile_rsrc(dz);
#pragma unroll
        for (int u = 0; u < R / 32; ++u) {
            const bool in = (unsigned)(st.y[u] + dy) < (unsigned)g.Ho && (unsigned)(st.x[u] + dx) < (unsigned)g.Wo;
            o[u] = load8(r, in ? st.off[u] + tap : kOut);
        }
    }
};

// The weights as the class's B: element (k = (t, co), ci) = W[co][tap t][ci]
// of the [Co][ldw] weight rows (row-major tile).
struct DgradB {
    static constexpr bool KC = false, kGuarded = false;
    const __bf16* w;
    int ldw;
    DgradGeo g;
    DgradClass c;
    template <int R>
    struct St { int ci; };
    template <int R>
    __device__ St<R> init(int row0, int tid) const { return {row0 + Chunk<false, R>::row(tid, 0)}; }
    template <int R>
    __device__ void fetch(const St<R>& st, int k0, int kend, int tid, uint4 (&o)[R / 32]) const
    {
        const __amdgpu_buffer_rsrc_t r = tile_rsrc(w);
#pragma unroll
        for (int u = 0; u < R / 32; ++u) {
            const unsigned k = (unsigned)(k0 + Chunk<false, R>::k(tid, u));
            const unsigned t = g.co.div(k), co = k - t * (unsigned)g.Co;
            const unsigned ty = c.nkxd.div(t), tx = t - ty * (unsigned)c.nkx;
            const unsigned tap = (unsigned)(3 * (c.ky0 + (int)ty * g.s) + c.kx0 + (int)tx * g.s);
            const bool in = (int)k < kend && st.ci < g.Ci;  // Ci % 8 == 0
            o[u] = load8(r, in ? 2u * (co * (unsigned)ldw + tap * (unsigned)g.Ci + (unsigned)st.ci) : kOut);
        }
    }
};

// ---------------------------------------------------------------------------
// Epilogues.  FP32 results: store4(z, m, n, v, N) of split z receives v[q] = C[m][n + q] for
// the four consecutive columns n .. n + 3 (n a multiple of 4, n < N) a lane
// holds.  BF16 results (kBf16): value4(n, v, N) gives the lane's four values,
// the block's tile is gathered in LDS, and store8(m, n, v, N) writes eight
// consecutive columns (n a multiple of 8): whole lines of 128 bytes instead
// of 32-byte pieces.
// ---------------------------------------------------------------------------

// C (+ C if accumulating), FP32; v4: rows 16-byte aligned (one vector store).
struct EpF32 {
    static constexpr bool kBf16 = false;
    float* C;
    int ldc, accumulate, v4;
    __device__ void store4(int, int m, int n, const f32x4& v, int N) const
    {
        float* c = C + (size_t)m * ldc + n;
        if (v4 && n + 3 < N) {
            float4 o = make_float4(v[0], v[1], v[2], v[3]);
            if (accumulate) {
                const float4 a = *(const float4*)c;
                o.x += a.x; o.y += a.y; o.z += a.z; o.w += a.w;
            }
            *(float4*)c = o;
            return;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (n + q < N) c[q] = accumulate ? c[q] + v[q] : v[q];
    }
};

// This block's split-K partial tile into the workspace [splits][M][N].
struct EpPartial {
    static constexpr bool kBf16 = false;
    float* ws;
    int M, N;
    __device__ void store4(int z, int m, int n, const f32x4& v, int) const
    {
        float* c = ws + ((size_t)z * M + m) * N + n;
        if ((N & 3) == 0) {
            *(float4*)c = make_float4(v[0], v[1], v[2], v[3]);
            return;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (n + q < N) c[q] = v[q];
    }
};

union Bf16x8 {
    uint4 u;
    __bf16 h[8];
};

// act(C + bias) to BF16 (the forward convolution's epilogue); v8: rows of Y
// 16-byte aligned.
struct EpBiasAct {
    static constexpr bool kBf16 = true;
    const float* bias;  // bias of column n at bias[n * bias_stride]
    int bias_stride, relu;
    __bf16* Y;
    int ldy, v8;
    __device__ void value4(int n, const f32x4& v, int N, float (&y)[4]) const
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            y[q] = v[q] + bias[(size_t)min(n + q, N - 1) * bias_stride];
            if (relu) y[q] = fmaxf(y[q], 0.f);
        }
    }
    __device__ void store8(int m, int n, const Bf16x8& v, int N) const
    {
        __bf16* p = Y + (size_t)m * ldy + n;
        if (v8 && n + 8 <= N) {
            *(uint4*)p = v.u;
            return;
        }
        // unrolled: an array indexed at run time lives in LDS or scratch, and the
        // LDS form reads its place from the dispatch packet in host memory, which
        // cost every launch of enough blocks about 10 us
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (n + q < N) p[q] = v.h[q];
    }
};

// Input gradient of one parity class, with the ReLU backward of the layer
// below applied (dz_below = dx where y_below > 0) and written as BF16 at the
// class pixel's place in [N][H][W][Ci] (Ci a multiple of 8).
struct EpDgradAct {
    static constexpr bool kBf16 = true;
    DgradGeo g;
    DgradClass c;
    const __bf16* y;  // activation of the layer below (NULL: no activation)
    int relu;
    __bf16* out;
    __device__ void value4(int, const f32x4& v, int, float (&o)[4]) const
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = v[q];
    }
    __device__ void store8(int m, int n, Bf16x8 v, int) const
    {
        const unsigned b = c.hw.div((unsigned)m), r = (unsigned)m - b * (unsigned)(c.Hc * c.Wc);
        const int yc = (int)c.w.div(r), xc = (int)r - yc * c.Wc;
        const size_t p = ((size_t)(((int)b * g.H + g.s * yc + c.py) * g.W + g.s * xc + c.px)) * g.Ci + n;
        if (relu) {
            Bf16x8 a;
            a.u = *(const uint4*)(y + p);
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (!((float)a.h[q] > 0.f)) v.h[q] = to_bf16(0.f);
        }
        *(uint4*)(out + p) = v.u;
    }
};

// C tile (m0, n0) of A B over k in [kbeg, kend): BM x BN with 2 x 2 wavefronts
// (BN = 32: 4 x 1).
// The next step's chunks are on their way to registers while the products of
// this step run, and every step's products come in the same order (ascending
// k, 32 at a time) whatever the tile, so its size does not change the result.
// Bound by the wait for the next step's chunks and by LDS reads and writes, not
// by the matrix cores: 256 x 64^2 x 64 to 32^2 x 128 channels: forward 117 -> 75 us
// (matrix cores 18 % busy), weight gradient 166 -> 124 (14 %), input gradient
// 222 -> 117 (15 %), with 64x64 tiles, K steps of 32, per-chunk index arithmetic and branches, 8-byte stores
// of the results and blocks spread over the XCDs in launch order before.
template <int BM, int BN, class AS, class BS, class EP>
__device__ inline void gemm_tile(int M, int N, int z, int m0, int n0, int kbeg, int kend, const AS& as,
                                 const BS& bs, const EP& ep)
{
    constexpr int WN = BN >= 64 ? 2 : 1, WM = 4 / WN;       // wavefronts per axis
    constexpr int FM = BM / (16 * WM), FN = BN / (16 * WN);  // MFMA tiles per wavefront
    constexpr int ea = AS::KC ? BM * kKP : kBK * t_pitch(BM), eb = BS::KC ? BN * kKP : kBK * t_pitch(BN);
    typedef Chunk<AS::KC, BM> CA;
    typedef Chunk<BS::KC, BN> CB;
    constexpr int ec = EP::kBf16 ? BM * (BN + 8) : 0;  // the result tile takes the operands' place
    __shared__ __attribute__((aligned(16))) __bf16 smem[ea + eb > ec ? ea + eb : ec];
    __bf16 *const As = smem, *const Bs = smem + ea;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave / WN) * (BM / WM), wn = (wave % WN) * (BN / WN);
    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const auto sa = as.template init<BM>(m0, tid);
    const auto sb = bs.template init<BN>(n0, tid);
    uint4 ra[CA::N], rb[CB::N];
    const auto fetch = [&](int k0) {
        as.template fetch<BM>(sa, k0, kend, tid, ra);
        bs.template fetch<BN>(sb, k0, kend, tid, rb);
    };
    fetch(kbeg);
    for (int k0 = kbeg; k0 < kend; k0 += kBK) {
#pragma unroll
        for (int u = 0; u < CA::N; ++u) *(uint4*)&As[CA::at(tid, u)] = ra[u];
#pragma unroll
        for (int u = 0; u < CB::N; ++u) *(uint4*)&Bs[CB::at(tid, u)] = rb[u];
        __syncthreads();
        if (k0 + kBK < kend) fetch(k0 + kBK);
#pragma unroll
        for (int k = 0; k < kBK; k += 32) {
            bf16x8 a[FM], b[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) a[i] = load_frag<AS::KC, BM>(As, wm + i * 16, k, lane);
#pragma unroll
            for (int j = 0; j < FN; ++j) b[j] = load_frag<BS::KC, BN>(Bs, wn + j * 16, k, lane);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    // B's fragment as the instruction's first operand: the
                    // result is the transposed tile, so a lane holds four
                    // consecutive columns n of one row m (vector stores)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    }
    if constexpr (EP::kBf16) {
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                const int m = wm + i * 16 + (lane & 15), n = wn + j * 16 + (lane >> 4) * 4;
                float y[4];
                ep.value4(n0 + n, acc[i][j], N, y);
                union { uint2 u; __bf16 h[4]; } o;
#pragma unroll
                for (int q = 0; q < 4; ++q) o.h[q] = to_bf16(y[q]);
                *(uint2*)&smem[m * (BN + 8) + n] = o.u;
            }
        __syncthreads();
        for (int t = tid; t < BM * BN / 8; t += 256) {
            const int m = t / (BN / 8), n = (t % (BN / 8)) * 8;
            if (m0 + m < M && n0 + n < N) {
                Bf16x8 v;
                v.u = *(const uint4*)&smem[m * (BN + 8) + n];
                ep.store8(m0 + m, n0 + n, v, N);
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int m = m0 + wm + i * 16 + (lane & 15);
                const int n = n0 + wn + j * 16 + (lane >> 4) * 4;
                if (m < M && n < N) ep.store4(z, m, n, acc[i][j], N);
            }
    }
}

__device__ inline unsigned block_id() { return blockIdx.y * gridDim.x + blockIdx.x; }

// With splits > 1 (split-K) each split covers its own contiguous k range.
template <int BM, int BN, class AS, class BS, class EP>
__global__ __launch_bounds__(256, BM * BN >= 128 * 128 ? 3 : 4) void gemm_kernel(int M, int N, int K, TileMap map,
                                                                                int splits, AS as, BS bs, EP ep)
{
    int tm, tn, z;
    if (!map.get(block_id(), tm, tn, z)) return;
    const int ksplit = (K + splits - 1) / splits, per = (ksplit + 31) / 32 * 32;
    const int kbeg = z * per, kend = min(K, kbeg + per);
    gemm_tile<BM, BN>(M, N, z, tm * BM, tn * BN, kbeg, kend, as, bs, ep);
}

constexpr int kDgradClasses = 4;  // parity classes per launch (all of them for s <= 2)
struct DgradClasses {
    DgradClass c[kDgradClasses];
};

template <int BM, int BN>
__global__ __launch_bounds__(256, BM * BN >= 128 * 128 ? 3 : 4) void dgrad_kernel(DgradGeo geo, DgradClasses all,
                                                                                 Groups gr, int mixed,
                                                                                 const __bf16* dz,
                                                                                 const __bf16* w, int ldw,
                                                                                 const __bf16* y, int relu,
                                                                                 __bf16* out)
{
    int g, tn, cls;
    if (mixed) {
        int t;
        if (!gr.get(blockIdx.x, g, t)) return;
        tn = t / mixed;
        cls = t - tn * mixed;
    } else {
        cls = (int)((blockIdx.x >> 3) / (unsigned)(gr.per * gr.size));
        if (!gr.get(blockIdx.x, g, tn, cls)) return;
    }
    const DgradClass& c = all.c[cls];
    const int m0 = g * BM;
    if (m0 >= c.M) return;
    gemm_tile<BM, BN>(c.M, geo.Ci, 0, m0, tn * BN, 0, c.nky * c.nkx * geo.Co, DgradA{dz, geo, c},
                      DgradB{w, ldw, geo, c}, EpDgradAct{geo, c, y, relu, out});
}

// The block tile of an M x N product with z reductions side by side: the largest
// that still gives two blocks per CU (training step at 256 x 256^2: 1.59 ms of
// kernels; with half as many blocks asked for 3 % more, twice as many 2 % more),
// split reductions, whose blocks only read and multiply, four (1.66 / 1.60 / 1.58 ms
// with one / two / four).
// Products of at most 32 columns never take a tile of 64 (43264 x 8 x 72: 6.5 us with
// 64x64, 5.4 with 64x32).
constexpr long long kMinBlocks = 512;
template <class F>
static void with_tile(long long M, long long N, long long z, F&& f, long long least = kMinBlocks)
{
    const auto blocks = [&](int bm, int bn) { return (M + bm - 1) / bm * ((N + bn - 1) / bn) * z; };
    typedef std::integral_constant<int, 32> I32;
    typedef std::integral_constant<int, 64> I64;
    typedef std::integral_constant<int, 128> I128;
    if (N <= 32 && M > 64 && blocks(128, 32) >= least) f(I128(), I32());
    else if (N <= 32) f(I64(), I32());
    else if (M > 64 && N > 64 && blocks(128, 128) >= least) f(I128(), I128());
    else if (M > 64 && N > 32 && blocks(128, 64) >= least) f(I128(), I64());
    else f(I64(), I64());
}

template <class AS, class BS, class EP>
static void launch_gemm(int M, int N, int K, int z, const AS& as, const BS& bs, const EP& ep, hipStream_t st)
{
    const auto go = [&](auto bm, auto bn) {
        constexpr int BM = decltype(bm)::value, BN = decltype(bn)::value;
        const TileMap map((M + BM - 1) / BM, (N + BN - 1) / BN, z);
        const Grid grid = gemm_grid(map.gr.blocks());
        gemm_kernel<BM, BN><<<dim3(grid.x, grid.y), 256, 0, st>>>(M, N, K, map, z, as, bs, ep);
    };
    // (operands with guarded loads: the loads are what takes the time)
    if constexpr (AS::kGuarded || BS::kGuarded)
        go(std::integral_constant<int, 64>(), std::integral_constant<int, 64>());
    else
        with_tile(M, N, z, go, z > 1 ? 2 * kMinBlocks : kMinBlocks);
}

// 3x3 convolution of a two-channel input with bias and activation: K = 18 is a
// single MFMA step, so there is nothing to stage: a wavefront takes 16 output
// pixels x 32 channels at a time, every lane gathers the four taps of its
// fragment (lanes l / 16 = 0, 1: taps 0 .. 7, 2: tap 8) straight from the image,
// and the weights stay in registers.  Channel 8 q + 4 j + e sits in column
// 4 q + e of product j, so a lane ends with eight consecutive channels and a
// wavefront writes 16 pixels x 64 bytes in one piece.  Bound by the output's
// writes: 256 images of 256^2 to 128^2 x 32 in 0.104 ms (0.34 GB, 3.2 TB/s), against
// 0.39 ms for an im2col matrix and its product.
__global__ __launch_bounds__(256) void conv2_fwd_kernel(ConvGeo g, int Co, const __bf16* __restrict__ x,
                                                        const __bf16* __restrict__ w, int ldw,
                                                        const float* __restrict__ bias, int bias_stride,
                                                        int relu, __bf16* __restrict__ y)
{
    const int lane = threadIdx.x & 63, i16 = lane & 15, q = lane >> 4;
    const int wave = blockIdx.x * 4 + (threadIdx.x >> 6), waves = gridDim.x * 4;
    const int c0 = blockIdx.y * 32;
    bf16x8 b[2];
    float bs[8];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const __bf16* wr = w + (size_t)(c0 + 8 * (i16 >> 2) + 4 * j + (i16 & 3)) * ldw + 8 * q;
#pragma unroll
        for (int e = 0; e < 8; ++e) b[j][e] = 8 * q + e < 18 ? wr[e] : to_bf16(0.f);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) bs[e] = bias[(size_t)(c0 + 8 * q + e) * bias_stride];
    const __amdgpu_buffer_rsrc_t rs = tile_rsrc(x);
    constexpr int U = 4;  // pixel groups whose loads are in flight together
    for (int m0 = wave * 16 * U; m0 < g.M; m0 += waves * 16 * U) {
        uint4 a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int m = m0 + 16 * u + i16;
            const unsigned n = g.hw.div((unsigned)m), r = (unsigned)m - n * (unsigned)(g.Ho * g.Wo);
            const int yo = (int)g.w.div(r), xo = (int)r - yo * g.Wo;
            a[u] = Im2colB2::taps2(g, rs, (int)n, yo * g.s - 1, xo * g.s - 1, 4 * q, m < g.M);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int m = m0 + 16 * u + i16;
            const bf16x8 av = __builtin_bit_cast(bf16x8, a[u]);
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            const f32x4 r0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[0], av, zero, 0, 0, 0);
            const f32x4 r1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[1], av, zero, 0, 0, 0);
            Bf16x8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float v = (e < 4 ? r0[e & 3] : r1[e & 3]) + bs[e];
                if (relu) v = fmaxf(v, 0.f);
                o.h[e] = to_bf16(v);
            }
            if (m < g.M) *(uint4*)(y + (size_t)m * Co + c0 + 8 * q) = o.u;
        }
    }
}

// C (+)= the sum of the split-K partial tiles, in split order (the result
// does not depend on which block finished first).
__global__ __launch_bounds__(256) void splitk_reduce_kernel(int M, int N, int S,
                                                            const float* __restrict__ ws,
                                                            float* __restrict__ C, int ldc,
                                                            int accumulate)
{
    const size_t total = (size_t)M * N;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
        float v = 0.f;
        for (int z = 0; z < S; ++z) v += ws[(size_t)z * total + i];
        float* c = C + (i / N) * ldc + i % N;
        *c = accumulate ? *c + v : v;
    }
}

// The same sum for many splits: a block covers 16 consecutive outputs with
// 16 threads each; thread g sums its contiguous range of splits in order,
// and the 16 range sums are added in range order (fixed order, so still
// independent of block timing).
constexpr int kRedOut = 16, kRedGroups = 16;
__global__ __launch_bounds__(256) void splitk_reduce_grouped_kernel(int M, int N, int S,
                                                                    const float* __restrict__ ws,
                                                                    float* __restrict__ C, int ldc,
                                                                    int accumulate)
{
    __shared__ float part[kRedGroups][kRedOut];
    const size_t total = (size_t)M * N;
    const int o = threadIdx.x % kRedOut, grp = threadIdx.x / kRedOut;
    const size_t i = (size_t)blockIdx.x * kRedOut + o;
    const int per = (S + kRedGroups - 1) / kRedGroups;
    const int z0 = grp * per, z1 = min(S, z0 + per);
    float v = 0.f;
    if (i < total)
        for (int z = z0; z < z1; ++z) v += ws[(size_t)z * total + i];
    part[grp][o] = v;
    __syncthreads();
    if (grp == 0 && i < total) {
        float t = part[0][o];
        for (int q = 1; q < kRedGroups; ++q) t += part[q][o];
        float* c = C + (i / N) * ldc + i % N;
        *c = accumulate ? *c + t : t;
    }
}

// Split-K for few output tiles and a long reduction (the weight gradients):
// about 1024 tiles of 64 x 64, each reducing at least 1024 rows.
static int gemm_splits(int M, int N, int K)
{
    const long long tiles = (long long)((M + kGT - 1) / kGT) * ((N + kGT - 1) / kGT);
    if (tiles < 512 && K >= 2048)
        return (int)std::max<long long>(1, std::min<long long>((1024 + tiles - 1) / tiles, K / 1024));
    return 1;
}

size_t gemm_ws_bytes(int M, int N, int K)
{
    const int s = gemm_splits(M, N, K);
    return s > 1 ? (size_t)s * M * N * sizeof(float) : 0;
}

// Runs C (+)= A B with the split-K decision of gemm_splits: the partial
// tiles go to ws and are reduced in split order (one pass if ws is too
// small or NULL).
template <class AS, class BS>
static void run_gemm_f32(int M, int N, int K, const AS& as, const BS& bs, float* C, int ldc,
                         bool accumulate, float* ws, size_t ws_bytes, hipStream_t st)
{
    int splits = gemm_splits(M, N, K);
    // (partial tiles take 16-byte stores: the workspace must be aligned)
    if (splits > 1 && (!ws || ws_bytes < gemm_ws_bytes(M, N, K) || ((uintptr_t)ws & 15)))
        splits = 1;
    if (splits > 1) {
        launch_gemm(M, N, K, splits, as, bs, EpPartial{ws, M, N}, st);
        const size_t total = (size_t)M * N;
        if (splits >= 2 * kRedGroups) {
            const size_t blocks = (total + kRedOut - 1) / kRedOut;
            splitk_reduce_grouped_kernel<<<(unsigned)blocks, 256, 0, st>>>(M, N, splits, ws, C, ldc,
                                                                          accumulate ? 1 : 0);
        } else {
            const int blocks = (int)std::min<size_t>((total + 255) / 256, 65536);
            splitk_reduce_kernel<<<blocks, 256, 0, st>>>(M, N, splits, ws, C, ldc,
                                                         accumulate ? 1 : 0);
        }
    } else {
        const int v4 = ldc % 4 == 0 && ((uintptr_t)C & 15) == 0;
        launch_gemm(M, N, K, 1, as, bs, EpF32{C, ldc, accumulate ? 1 : 0, v4}, st);
    }
}

// Dense operands: A stored [M][K] unless ta ([K][M]), B stored [K][N] unless
// tb ([N][K]).
template <Vec VEC, class F>
static void with_dense(bool ta, bool tb, const __bf16* a, int lda, int M, const __bf16* b, int ldb,
                       int N, F&& f)
{
    if (!ta && !tb) f(DenseSrc<true, VEC>{a, lda, M}, DenseSrc<false, VEC>{b, ldb, N});
    else if (!ta && tb) f(DenseSrc<true, VEC>{a, lda, M}, DenseSrc<true, VEC>{b, ldb, N});
    else if (ta && !tb) f(DenseSrc<false, VEC>{a, lda, M}, DenseSrc<false, VEC>{b, ldb, N});
    else f(DenseSrc<false, VEC>{a, lda, M}, DenseSrc<true, VEC>{b, ldb, N});
}

void launch_gemm_bf16(bool ta, bool tb, int M, int N, int K, const void* A, int lda, const void* B,
                      int ldb, float* C, int ldc, bool accumulate, float* ws, size_t ws_bytes,
                      hipStream_t st)
{
    const __bf16* a = (const __bf16*)A;
    const __bf16* b = (const __bf16*)B;
    auto go = [&](const auto& as, const auto& bs) {
        run_gemm_f32(M, N, K, as, bs, C, ldc, accumulate, ws, ws_bytes, st);
    };
    const Vec v = std::min(dense_vec(!ta, M, K, lda, (uintptr_t)A), dense_vec(tb, N, K, ldb, (uintptr_t)B));
    if (v == kWhole) with_dense<kWhole>(ta, tb, a, lda, M, b, ldb, N, go);
    else if (v == kRagged) with_dense<kRagged>(ta, tb, a, lda, M, b, ldb, N, go);
    else with_dense<kElems>(ta, tb, a, lda, M, b, ldb, N, go);
}

void launch_gemm_bias_act(int M, int N, int K, const void* A, int lda, const void* B, int ldb,
                          const float* bias, int bias_stride, bool relu, void* Y, int ldy,
                          hipStream_t st)
{
    const EpBiasAct ep{bias, bias_stride, relu ? 1 : 0, (__bf16*)Y, ldy,
                       ldy % 8 == 0 && ((uintptr_t)Y & 15) == 0};
    const __bf16* a = (const __bf16*)A;
    const __bf16* b = (const __bf16*)B;
    const auto go = [&](const auto& as, const auto& bs) { launch_gemm(M, N, K, 1, as, bs, ep, st); };
    const Vec v = std::min(dense_vec(true, M, K, lda, (uintptr_t)A), dense_vec(true, N, K, ldb, (uintptr_t)B));
    if (v == kWhole) go(DenseSrc<true, kWhole>{a, lda, M}, DenseSrc<true, kWhole>{b, ldb, N});
    else if (v == kRagged) go(DenseSrc<true, kRagged>{a, lda, M}, DenseSrc<true, kRagged>{b, ldb, N});
    else go(DenseSrc<true, kElems>{a, lda, M}, DenseSrc<true, kElems>{b, ldb, N});
}

// ---------------------------------------------------------------------------
// Implicit-GEMM 3x3 convolutions (C a multiple of 8; no im2col matrix)
// ---------------------------------------------------------------------------

static ConvGeo conv_geo(int N, int H, int W, int C, int s, bool ones)
{
    ConvGeo g;
    g.H = H; g.W = W; g.C = C; g.s = s;
    g.Ho = (H - 1) / s + 1;
    g.Wo = (W - 1) / s + 1;
    g.M = N * g.Ho * g.Wo;
    g.ones = ones ? 1 : 0;
    g.hw = FastDiv((unsigned)(g.Ho * g.Wo));
    g.w = FastDiv((unsigned)g.Wo);
    g.c = FastDiv((unsigned)C);
    return g;
}

void launch_conv_fwd(int N, int H, int W, int Ci, int Co, int s, const void* x, const void* w,
                     int ldw, const float* bias, int bias_stride, bool relu, void* y, hipStream_t st)
{
    const ConvGeo g = conv_geo(N, H, W, Ci, s, false);
    launch_gemm(g.M, Co, 9 * Ci, 1, Im2colA{(const __bf16*)x, g}, DenseSrc<true, kWhole>{(const __bf16*)w, ldw, Co},
                EpBiasAct{bias, bias_stride, relu ? 1 : 0, (__bf16*)y, Co,
                          Co % 8 == 0 && ((uintptr_t)y & 15) == 0}, st);
}

size_t conv_wgrad_ws_bytes(int N, int H, int W, int Ci, int Co, int s, int ldw)
{
    const ConvGeo g = conv_geo(N, H, W, Ci, s, false);
    return gemm_ws_bytes(Co, ldw, g.M);
}

void launch_conv_wgrad(int N, int H, int W, int Ci, int Co, int s, const void* x, const void* dz,
                       int ldw, bool ones, float* dw, float* ws, size_t ws_bytes, hipStream_t st)
{
    const ConvGeo g = conv_geo(N, H, W, Ci, s, ones);
    run_gemm_f32(Co, ldw, g.M, DenseSrc<false, kWhole>{(const __bf16*)dz, Co, Co},
                 Im2colB{(const __bf16*)x, g}, dw, ldw, false, ws, ws_bytes, st);
}

void launch_conv2_fwd(int N, int H, int W, int Co, int s, const void* x, const void* w, int ldw,
                      const float* bias, int bias_stride, bool relu, void* y, hipStream_t st)
{
    const ConvGeo g = conv_geo(N, H, W, 2, s, false);
    const int groups = (g.M + 4 * 4 * 16 - 1) / (4 * 4 * 16);  // blocks that take one round
    conv2_fwd_kernel<<<dim3(std::min(groups, 2048), Co / 32), 256, 0, st>>>(
        g, Co, (const __bf16*)x, (const __bf16*)w, ldw, bias, bias_stride, relu ? 1 : 0, (__bf16*)y);
}

void launch_conv2_wgrad(int N, int H, int W, int Co, int s, const void* x, const void* dz, int ldw,
                        float* dw, float* ws, size_t ws_bytes, hipStream_t st)
{
    const ConvGeo g = conv_geo(N, H, W, 2, s, true);
    run_gemm_f32(Co, ldw, g.M, DenseSrc<false, kWhole>{(const __bf16*)dz, Co, Co},
                 Im2colB2{(const __bf16*)x, g}, dw, ldw, false, ws, ws_bytes, st);
}

void launch_conv_dgrad_act(int N, int H, int W, int Ci, int Co, int s, const void* dz,
                           const void* w, int ldw, const void* y, bool relu, void* out,
                           hipStream_t st)
{
    DgradGeo g;
    g.H = H; g.W = W; g.Ci = Ci; g.Co = Co; g.s = s;
    g.Ho = (H - 1) / s + 1;
    g.Wo = (W - 1) / s + 1;
    g.co = FastDiv((unsigned)Co);
    DgradClasses all{};
    int n = 0, most = 0;
    const auto flush = [&]() {
        with_tile(most, Ci, n, [&](auto bm, auto bn) {
            constexpr int BM = decltype(bm)::value, BN = decltype(bn)::value;
            // One class after the other, those with the most taps first; but pixels
            // of less than a 128-byte line are written by all classes of a row
            // tile side by side, so that the lines of neighbouring columns'
            // classes meet in the XCD's L2 (128^2 x 32 channels: 0.30 -> 0.19 ms;
            // wider pixels gain nothing and lose to the uneven blocks, 64^2 x 64:
            // 0.11 -> 0.14 ms).
            const int mixed = 2 * Ci < 128 ? n : 0, tm = (most + BM - 1) / BM, tn = (Ci + BN - 1) / BN;
            const Groups gr(tm, mixed ? tn * n : tn);
            std::sort(all.c, all.c + n, [](const DgradClass& a, const DgradClass& b) {
                return a.nky * a.nkx > b.nky * b.nkx;
            });
            dgrad_kernel<BM, BN><<<(unsigned)gr.blocks() * (mixed ? 1 : n), 256, 0, st>>>(
                g, all, gr, mixed, (const __bf16*)dz, (const __bf16*)w, ldw, (const __bf16*)y, relu ? 1 : 0, (__bf16*)out);
        });
        n = most = 0;
    };
    for (int py = 0; py < s && py < H; ++py)
        for (int px = 0; px < s && px < W; ++px) {
            DgradClass& c = all.c[n];
            c.py = py; c.px = px;
            c.Hc = (H - py + s - 1) / s;
            c.Wc = (W - px + s - 1) / s;
            c.M = N * c.Hc * c.Wc;
            c.nky = c.nkx = 0;
            for (int k = 2; k >= 0; --k) {  // (the first tap of each axis is set last)
                if ((py + 1 - k) % s == 0) { c.ky0 = k; c.dy0 = (py + 1 - k) / s; ++c.nky; }
                if ((px + 1 - k) % s == 0) { c.kx0 = k; c.dx0 = (px + 1 - k) / s; ++c.nkx; }
            }
            c.hw = FastDiv((unsigned)(c.Hc * c.Wc));
            c.w = FastDiv((unsigned)c.Wc);
            c.nkxd = FastDiv((unsigned)std::max(c.nkx, 1));
            most = std::max(most, c.M);
            if (++n == kDgradClasses) flush();
        }
    if (n) flush();
}

// im2col of a 3x3 convolution (stride s, padding 1) on NHWC BF16 input:
// col[m][t C + c] = x[n][yo s + ky - 1][xo s + kx - 1][c] (zero outside),
// t = 3 ky + kx.  One thread per (output pixel m, tap t, group of G
// channels); G = 8 copies 16 bytes at a time.  Index math is 32-bit (the
// host checks that every index space fits).
template <int G>
__global__ __launch_bounds__(256) void im2col_kernel(int N, int H, int W, int C, int s, int Ho,
                                                     int Wo, const __bf16* __restrict__ x,
                                                     __bf16* __restrict__ col, int ld)
{
    const unsigned groups = (unsigned)(C / G);
    const unsigned total = (unsigned)N * Ho * Wo * 9u * groups;
    for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
        const unsigned g = i % groups, r = i / groups;
        const unsigned t = r % 9u, m = r / 9u;
        const int xo = (int)(m % (unsigned)Wo);
        const unsigned q = m / (unsigned)Wo;
        const int yo = (int)(q % (unsigned)Ho), n = (int)(q / (unsigned)Ho);
        const int ky = (int)t / 3, kx = (int)t - 3 * ky;
        const int yi = yo * s + ky - 1, xi = xo * s + kx - 1;
        __bf16* dst = col + (size_t)m * ld + t * C + g * G;
        const bool in = yi >= 0 && yi < H && xi >= 0 && xi < W;
        const __bf16* src = x + (((size_t)n * H + yi) * W + xi) * C + g * G;
        if constexpr (G == 8) {
            *reinterpret_cast<uint4*>(dst) = in ? *reinterpret_cast<const uint4*>(src) : make_uint4(0, 0, 0, 0);
        } else {
#pragma unroll
            for (int c = 0; c < G; ++c) dst[c] = in ? src[c] : to_bf16(0.f);
        }
    }
}

// Columns [9 C, ld) of each im2col row: 1 in column 9 C when `ones` (so that
// the weight-gradient product dz^T col also yields the bias gradient, the
// column sums of dz), 0 elsewhere.
__global__ __launch_bounds__(256) void col_tail_kernel(unsigned rows, int K9, int ld, int ones,
                                                       __bf16* __restrict__ col)
{
    const unsigned w = (unsigned)(ld - K9), total = rows * w;
    for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
        const unsigned m = i / w, c = i - m * w;
        col[(size_t)m * ld + K9 + c] = to_bf16(ones && c == 0 ? 1.f : 0.f);
    }
}

// dx = col2im(dcol): each input element gathers the window entries that read
// it (taps in ky, kx order).  One thread per (n, yi, xi, group of G
// channels); G = 4 moves float4.
// ACT: the result is the gradient of the layer below's BF16 activation y, and
// the kernel applies that layer's ReLU backward and writes the BF16 operand
// dz = dx * (y > 0) instead of FP32 dx.
template <int G, bool ACT>
__global__ __launch_bounds__(256) void col2im_kernel(int N, int H, int W, int C, int s, int Ho,
                                                     int Wo, const float* __restrict__ dcol,
                                                     float* __restrict__ dx,
                                                     const __bf16* __restrict__ y, int relu,
                                                     __bf16* __restrict__ dz)
{
    const unsigned groups = (unsigned)(C / G);
    const unsigned total = (unsigned)N * H * W * groups;
    const int K = 9 * C;
    for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
        const unsigned g = i % groups, p = i / groups;
        const int xi = (int)(p % (unsigned)W);
        const unsigned q = p / (unsigned)W;
        const int yi = (int)(q % (unsigned)H), n = (int)(q / (unsigned)H);
        float acc[G];
#pragma unroll
        for (int c = 0; c < G; ++c) acc[c] = 0.f;
        for (int ky = 0; ky < 3; ++ky) {
            const int ty = yi + 1 - ky;  // = yo * s
            if (ty < 0 || ty % s) continue;
            const int yo = ty / s;
            if (yo >= Ho) continue;
            for (int kx = 0; kx < 3; ++kx) {
                const int tx = xi + 1 - kx;
                if (tx < 0 || tx % s) continue;
                const int xo = tx / s;
                if (xo >= Wo) continue;
                const float* src = dcol + ((size_t)((n * Ho + yo) * Wo + xo)) * K + (ky * 3 + kx) * C + g * G;
                if constexpr (G == 4) {
                    const float4 v = *reinterpret_cast<const float4*>(src);
                    acc[0] += v.x; acc[1] += v.y; acc[2] += v.z; acc[3] += v.w;
                } else {
#pragma unroll
                    for (int c = 0; c < G; ++c) acc[c] += src[c];
                }
            }
        }
        if constexpr (ACT) {
            const size_t o = (size_t)p * C + g * G;
            union { uint2 u; __bf16 h[4]; } yv, dv;
            if constexpr (G == 4) {
                yv.u = *reinterpret_cast<const uint2*>(y + o);
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    dv.h[c] = to_bf16(relu ? ((float)yv.h[c] > 0.f ? acc[c] : 0.f) : acc[c]);
                *reinterpret_cast<uint2*>(dz + o) = dv.u;
            } else {
#pragma unroll
                for (int c = 0; c < G; ++c)
                    dz[o + c] = to_bf16(relu ? ((float)y[o + c] > 0.f ? acc[c] : 0.f) : acc[c]);
            }
        } else {
            float* dst = dx + (size_t)p * C + g * G;
            if constexpr (G == 4) {
                *reinterpret_cast<float4*>(dst) = make_float4(acc[0], acc[1], acc[2], acc[3]);
            } else {
#pragma unroll
                for (int c = 0; c < G; ++c) dst[c] = acc[c];
            }
        }
    }
}

// y = relu(z + b) -> BF16 (and FP32 copy for the head); z [M][C] FP32.
__global__ __launch_bounds__(256) void bias_relu_kernel(size_t total, int C, const float* __restrict__ z,
                                                        const float* __restrict__ b, int relu,
                                                        __bf16* __restrict__ y)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
        float v = z[i] + b[i % C];
        if (relu) v = fmaxf(v, 0.f);
        y[i] = to_bf16(v);
    }
}

// dz = dy * (y > 0) -> BF16 operand for the GEMMs; y is the layer's BF16 output.
__global__ __launch_bounds__(256) void relu_bwd_kernel(size_t total, const float* __restrict__ dy,
                                                       const __bf16* __restrict__ y, int relu,
                                                       __bf16* __restrict__ dz)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
        const float g = dy[i];
        dz[i] = to_bf16(relu ? ((float)y[i] > 0.f ? g : 0.f) : g);
    }
}

// db[c] = sum over rows of dz (BF16 operand as used by the weight GEMM).
// Grid-stride over rows with consecutive threads on consecutive elements:
// for C < 256 a block covers R = 256 / C rows per pass (thread t: column
// t % C, row offset t / C), for C >= 256 strips of 256 columns.  Each block
// adds its column sums to db with FP32 atomics (db zeroed first), so the
// summation order, and the last bits, vary from run to run.
__global__ __launch_bounds__(256) void colsum_kernel(int M, int C, const __bf16* __restrict__ dz,
                                                     float* __restrict__ db)
{
    __shared__ float red[256];
    const int t = threadIdx.x;
    const bool narrow = C < 256;
    const int R = narrow ? 256 / C : 1;
    for (int c0 = 0; c0 < C; c0 += 256) {
        const int c = narrow ? t % C : c0 + t;
        const int ro = narrow ? t / C : 0;
        const bool act = narrow ? t < R * C : c < C;
        float acc = 0.f;
        if (act)
            for (size_t r = (size_t)blockIdx.x * R + ro; r < (size_t)M; r += (size_t)gridDim.x * R)
                acc += (float)dz[r * C + c];
        if (narrow) {
            red[t] = acc;
            __syncthreads();
            if (t < C) {
                float sum = 0.f;
                for (int k = 0; k < R; ++k) sum += red[k * C + t];
                atomicAdd(db + t, sum);
            }
            __syncthreads();
        } else if (act) {
            atomicAdd(db + c, acc);
        }
    }
}

// One Adam step over a flat parameter buffer (every layer at once): moments
// m, v and the FP32 master p updated in place, and p rounded to BF16 for the
// next products.  c1, c2: the bias corrections 1 - beta^t.
__global__ __launch_bounds__(256) void adam_kernel(size_t n, float* __restrict__ p,
                                                   const float* __restrict__ g, float* __restrict__ m,
                                                   float* __restrict__ v, __bf16* __restrict__ pb,
                                                   float lr, float b1, float b2, float eps, float c1,
                                                   float c2)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = fmaf(b1, m[i], (1.f - b1) * gi);
        const float vi = fmaf(b2, v[i], (1.f - b2) * gi * gi);
        m[i] = mi;
        v[i] = vi;
        const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
        p[i] = pi;
        pb[i] = to_bf16(pi);
    }
}

__global__ __launch_bounds__(256) void fill_zero_kernel(int n, float* __restrict__ p)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.f;
}

static int grid_for(size_t total)
{
    const size_t b = (total + 255) / 256;
    return (int)(b < 65536 ? (b == 0 ? 1 : b) : 65536);
}

void launch_im2col(int N, int H, int W, int C, int s, int Ho, int Wo, const void* x, void* col,
                   int ld, bool ones, hipStream_t st)
{
    const bool vec = C % 8 == 0 && ld % 8 == 0 && (uintptr_t)x % 16 == 0 && (uintptr_t)col % 16 == 0;
    const size_t total = (size_t)N * Ho * Wo * 9 * (vec ? C / 8 : C);
    if (vec)
        im2col_kernel<8><<<grid_for(total), 256, 0, st>>>(N, H, W, C, s, Ho, Wo, (const __bf16*)x,
                                                          (__bf16*)col, ld);
    else
        im2col_kernel<1><<<grid_for(total), 256, 0, st>>>(N, H, W, C, s, Ho, Wo, (const __bf16*)x,
                                                          (__bf16*)col, ld);
    if (ld > 9 * C) {
        const unsigned rows = (unsigned)N * Ho * Wo;
        col_tail_kernel<<<grid_for((size_t)rows * (ld - 9 * C)), 256, 0, st>>>(rows, 9 * C, ld, ones ? 1 : 0,
                                                                              (__bf16*)col);
    }
}

void launch_col2im(int N, int H, int W, int C, int s, int Ho, int Wo, const float* dcol, float* dx,
                   const void* y, bool relu, void* dz, hipStream_t st)
{
    const bool act = y != nullptr;
    const bool vec = C % 4 == 0 && (uintptr_t)dcol % 16 == 0 &&
                     (act ? ((uintptr_t)y % 8 == 0 && (uintptr_t)dz % 8 == 0) : (uintptr_t)dx % 16 == 0);
    const size_t total = (size_t)N * H * W * (vec ? C / 4 : C);
    const __bf16* yb = (const __bf16*)y;
    __bf16* dzb = (__bf16*)dz;
    const int r = relu ? 1 : 0;
    if (act) {
        if (vec)
            col2im_kernel<4, true><<<grid_for(total), 256, 0, st>>>(N, H, W, C, s, Ho, Wo, dcol, dx, yb, r, dzb);
        else
            col2im_kernel<1, true><<<grid_for(total), 256, 0, st>>>(N, H, W, C, s, Ho, Wo, dcol, dx, yb, r, dzb);
    } else {
        if (vec)
            col2im_kernel<4, false><<<grid_for(total), 256, 0, st>>>(N, H, W, C, s, Ho, Wo, dcol, dx, yb, r, dzb);
        else
            col2im_kernel<1, false><<<grid_for(total), 256, 0, st>>>(N, H, W, C, s, Ho, Wo, dcol, dx, yb, r, dzb);
    }
}

void launch_adam(size_t n, float* p, const float* g, float* m, float* v, void* pb, float lr,
                 float b1, float b2, float eps, float c1, float c2, hipStream_t st)
{
    adam_kernel<<<grid_for(n), 256, 0, st>>>(n, p, g, m, v, (__bf16*)pb, lr, b1, b2, eps, c1, c2);
}

void launch_bias_relu(size_t total, int C, const float* z, const float* b, bool relu, void* y,
                      hipStream_t st)
{
    bias_relu_kernel<<<grid_for(total), 256, 0, st>>>(total, C, z, b, relu ? 1 : 0, (__bf16*)y);
}

void launch_relu_bwd(size_t total, const float* dy, const void* y, bool relu, void* dz,
                     hipStream_t st)
{
    relu_bwd_kernel<<<grid_for(total), 256, 0, st>>>(total, dy, (const __bf16*)y, relu ? 1 : 0,
                                                     (__bf16*)dz);
}

void launch_colsum(int M, int C, const void* dz, float* db, hipStream_t st)
{
    const int R = C < 256 ? 256 / C : 1;
    const int blocks = (int)std::min<long long>(1024, ((long long)M + R - 1) / R);
    fill_zero_kernel<<<(C + 255) / 256, 256, 0, st>>>(C, db);
    colsum_kernel<<<blocks, 256, 0, st>>>(M, C, (const __bf16*)dz, db);
}

}  // namespace dp
