// FDK pre-filter and image-sharpness loss for motion-compensated
// reconstruction (the paper's motion-compensated FBP task, Sec. III-B).
//
// Pre-filter: the projections are referred to a virtual detector through
// the isocentre (pitch tau = du SAD/SDD), multiplied by the cosine weight
// SAD / sqrt(SAD^2 + u'^2 + v'^2), and each row is convolved with the
// band-limited ramp (Ram-Lak) kernel
//   h[0] = 1/(4 tau^2),  h[k] = -1/(pi^2 k^2 tau^2) for odd k,  0 for even k != 0,
//   q[a] = scale tau sum_n p_w[n] h[a - n]      (rows zero outside the detector).
// The sums are FP64 (the ramp's cancellation between h[0] and the odd taps
// would cost FP32 several digits on smooth rows).  Odd k couples the outputs
// of one column parity with the inputs of the other, so rows of up to 2048
// pixels are two Toeplitz products of half the size on the FP64 matrix cores, or
// the same sums a row per block where there are few rows; longer ones take one
// block per row and two LDS reads per pair of taps.
//
// Sharpness: S = -sum over x, y, z forward differences d of d^2 (pairs
// inside the grid); dS/dmu_j = sum over axes of 2 (mu[j+e] - mu_j) where j+e
// exists, minus 2 (mu_j - mu[j-e]) where j-e exists.  FP32 per voxel, FP32
// block sums, FP64 fixed-order total.
//
// Gradient entropy (the sharpness criterion of the paper's motion-compensated
// FBP experiment): g_j = sqrt(dx^2 + dy^2 + dz^2 + eps) from the same forward
// differences, Z = sum g, GE = -sum (g/Z) log(g/Z) = log Z - (sum g log g) / Z.
// Pass 1 reduces sum g and sum g log g per block; a one-block kernel forms Z
// and GE in FP64; pass 2 writes dGE/dmu_i = sum over axes of
// c_{i-e} d_{i-e} - c_i d_i with c_j = -(log g_j - log Z + GE) / (Z g_j),
// recomputing g at i and at its three backward neighbours.
#include <algorithm>
#include <climits>
#include <cmath>

#include "dp_internal.h"

namespace dp {

constexpr int kFdkThreads = 256;
constexpr int kFdkMaxNu = 4000;  // LDS: 3 nu floats + nu/2 doubles <= 64 KiB

// Entries of the matrix kernel's table: d = alpha - nuu (+ 0 or -1) with alpha
// up to a tile of 16 and nuu up to 3 beyond the row.
__host__ __device__ inline int fdk_table(int nu) { return nu + 32; }

// Inputs of one parity, to a multiple of 4.
__host__ __device__ inline int fdk_half(int nu) { return ((nu + 1) / 2 + 3) / 4 * 4; }

typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ inline float fdk_weighted(float p, double uu, double vv, double sad)
{
    // (explicit fma: the same rounding in every kernel)
    return (float)((double)p * sad / sqrt(fma(vv, vv, fma(uu, uu, sad * sad))));
}

// 16 detector rows per block.  The 8 wavefronts share the tiles of 16 outputs
// of one parity, NT each (nu <= 128 NT), and walk the inputs of the other
// parity 4 at a time (v_mfma_f64_16x16x4: lane l supplies row l % 16, input
// l / 16 of the first operand and input l / 16, output l % 16 of the second;
// it receives rows l / 16 + 4 v of output l % 16).  The rows are staged in
// LDS kFdkChunk inputs at a time; outputs stay in registers until every input
// was read (proj == out is allowed).
// Bound by the FP64 matrix rate: nu / 2 FMAs per output, 0.46 ms at 78.6 TFLOP/s for
// 360 views of 512 x 384; 0.74 ms measured, 2.99 ms with a block per row and two
// LDS reads, two conversions, an addition and an FMA per pair of taps.
constexpr int kFdkRows = 16, kFdkChunk = 512, kFdkWaves = 8;
constexpr int kFdkPitch = kFdkChunk + 8;  // rows 8 banks apart

template <int NT>
__global__ __launch_bounds__(64 * kFdkWaves) void fdk_filter_mfma_kernel(
    int nu, int nv, int rows, double cu, double cv, double du_iso, double dv_iso, double sad,
    double tau, double scale, const float* proj, float* out)
{
    // row[16][kFdkPitch], then h[2 d + 1] for d = -off .. (table entry d + off)
    extern __shared__ __align__(16) unsigned char smem[];
    float* row = reinterpret_cast<float*>(smem);
    double* h = reinterpret_cast<double*>(smem + sizeof(float) * kFdkRows * kFdkPitch);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r0 = blockIdx.x * kFdkRows;
    const int off = nu / 2 + 8, ntab = fdk_table(nu);
    const double pi2tau2 = M_PI * M_PI * tau * tau, h0 = 1.0 / (4.0 * tau * tau);
    for (int t = tid; t < ntab; t += 64 * kFdkWaves) {
        const double k = 2.0 * (t - off) + 1.0;
        h[t] = -1.0 / (pi2tau2 * k * k);
    }
    const int e = wave & 1;                  // parity of this wavefront's outputs
    const int n_out = (nu - e + 1) / 2;      // outputs a = 2 alpha + e
    const int n_in = (nu + e) / 2;           // inputs n = 2 nuu + 1 - e
    const int i16 = lane & 15, q = lane >> 4;
    f64x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = (f64x4){0.0, 0.0, 0.0, 0.0};
    for (int c0 = 0; c0 < nu; c0 += kFdkChunk) {
        const int nc = min(kFdkChunk, nu - c0);
        __syncthreads();
        for (int x = tid; x < kFdkRows * kFdkPitch; x += 64 * kFdkWaves) {
            const int j = x / kFdkPitch, c = x - j * kFdkPitch, r = r0 + j;
            float v = 0.0f;
            if (c < nc && r < rows)
                v = fdk_weighted(proj[(size_t)r * nu + c0 + c], ((double)(c0 + c) - cu) * du_iso,
                                 ((double)(r % nv) - cv) * dv_iso, sad);
            row[x] = v;
        }
        __syncthreads();
        // this chunk's inputs: c0 even, so input nuu sits at row[..][2 (nuu - c0 / 2) + 1 - e]
        const int k1 = min(n_in - c0 / 2, kFdkChunk / 2);
        const float* in = row + i16 * kFdkPitch + 2 * q + 1 - e;
        // h[a - n]: a - n = 2 (alpha - nuu) + 2 e - 1, entry alpha - nuu + e - 1 + off
        const double* hk = h + (off + e - 1 + i16 - q - c0 / 2);
        for (int k = 0; k < k1; k += 4) {
            const double p = (double)in[2 * k];  // (zero from the row's end on)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int alpha0 = 16 * ((wave >> 1) + (kFdkWaves / 2) * t);
                if (alpha0 >= n_out) break;
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(p, hk[alpha0 - k], acc[t], 0, 0, 0);
            }
        }
        // the chunk's own outputs: h[0] times their input
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int a = 2 * (16 * ((wave >> 1) + (kFdkWaves / 2) * t) + i16) + e - c0;
            if (a >= 0 && a < nc)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    acc[t][v] = fma(h0, (double)row[(q + 4 * v) * kFdkPitch + a], acc[t][v]);
        }
    }
    // through LDS for whole-row stores, a chunk at a time
    for (int c0 = 0; c0 < nu; c0 += kFdkChunk) {
        const int nc = min(kFdkChunk, nu - c0);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int a = 2 * (16 * ((wave >> 1) + (kFdkWaves / 2) * t) + i16) + e - c0;
            if (a >= 0 && a < nc)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    row[(q + 4 * v) * kFdkPitch + a] = (float)(scale * tau * acc[t][v]);
        }
        __syncthreads();
        for (int j = wave; j < kFdkRows && r0 + j < rows; j += kFdkWaves)
            for (int c = lane; c < nc; c += 64)
                out[(size_t)(r0 + j) * nu + c0 + c] = row[j * kFdkPitch + c];
    }
}

// One detector row per block, for launches of few rows: the same sums, in the same
// order and hence to the same bits, on the vector units (the matrix instruction
// adds its four products one fma after the other, in ascending k; padding adds
// zeros).  A wavefront takes 64 neighbouring outputs of one parity, NJ times (nu <=
// NJ threads), and walks the inputs of the other parity: per tap an FP64 table
// read and fma, the inputs (as FP64 in LDS) are wave-uniform reads.
template <int NJ>
__global__ __launch_bounds__(1024) void fdk_filter_row_kernel(
    int nu, int nv, double cu, double cv, double du_iso, double dv_iso, double sad, double tau,
    double scale, const float* proj, float* out)  // proj == out allowed (row staged first)
{
    // in[e][n / 2]: the inputs n of parity e (zeros to a multiple of 4), then the table
    extern __shared__ __align__(16) unsigned char smem[];
    const int half = fdk_half(nu), off = nu / 2 + 8, ntab = fdk_table(nu);
    double* in = reinterpret_cast<double*>(smem);
    double* h = in + 2 * half;
    const int tid = threadIdx.x, threads = blockDim.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = blockIdx.x;  // row index over all views: v * nv + b
    const float* src = proj + (size_t)r * nu;
    const double vv = ((double)(r % nv) - cv) * dv_iso;
    const double pi2tau2 = M_PI * M_PI * tau * tau, h0 = 1.0 / (4.0 * tau * tau);
    for (int t = tid; t < ntab; t += threads) {
        const double k = 2.0 * (t - off) + 1.0;
        h[t] = -1.0 / (pi2tau2 * k * k);
    }
    for (int c = tid; c < 2 * half; c += threads)
        in[(c & 1) * half + (c >> 1)] =
            c < nu ? (double)fdk_weighted(src[c], ((double)c - cu) * du_iso, vv, sad) : 0.0;
    __syncthreads();
    const int e = wave & 1, n_out = (nu - e + 1) / 2, n_in = (nu + e) / 2;
    const double* p = in + (1 - e) * half;
    const double* own = in + e * half;
    const int stride = threads / 2;  // outputs of a parity per round
    double acc[NJ];
    const double* hk[NJ];
    int alpha[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        acc[j] = 0.0;
        alpha[j] = (wave >> 1) * 64 + lane + j * stride;
        hk[j] = h + (off + e - 1 + min(alpha[j], n_out - 1));
    }
    for (int c0 = 0; c0 < nu; c0 += kFdkChunk) {
        const int k1 = min(n_in, (c0 + kFdkChunk) / 2);
        for (int k = c0 / 2; k < k1; k += 4)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int j = 0; j < NJ; ++j) acc[j] = fma(p[k + q], hk[j][-(k + q)], acc[j]);
        // the chunk's own outputs: h[0] times their input
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            if (alpha[j] < n_out && alpha[j] >= c0 / 2 && alpha[j] < (c0 + kFdkChunk) / 2)
                acc[j] = fma(h0, own[alpha[j]], acc[j]);
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j)
        if (alpha[j] < n_out) out[(size_t)r * nu + 2 * alpha[j] + e] = (float)(scale * tau * acc[j]);
}

__global__ __launch_bounds__(kFdkThreads) void fdk_filter_kernel(
    int nu, int nv, double cu, double cv, double du_iso, double dv_iso, double sad, double tau,
    double scale, const float* proj, float* out)  // proj == out allowed (row staged first)
{
    // row[nu .. 2 nu) holds the weighted row; nu zeros on either side
    extern __shared__ __align__(16) unsigned char smem[];
    double* hodd = reinterpret_cast<double*>(smem);            // h[2 i + 1], i < nu / 2
    float* row = reinterpret_cast<float*>(smem + sizeof(double) * (nu / 2 + 1));
    const int r = blockIdx.x;  // row index over all views: v * nv + b
    const int b = r % nv;
    const float* src = proj + (size_t)r * nu;
    const double vv = ((double)b - cv) * dv_iso;
    for (int i = threadIdx.x; i < 3 * nu; i += kFdkThreads) {
        const int a = i - nu;
        float val = 0.0f;
        if (a >= 0 && a < nu) {
            const double uu = ((double)a - cu) * du_iso;
            val = fdk_weighted(src[a], uu, vv, sad);
        }
        row[i] = val;
    }
    const double pi2tau2 = M_PI * M_PI * tau * tau;
    for (int i = threadIdx.x; i < (nu + 1) / 2; i += kFdkThreads) {
        const double k = 2.0 * i + 1.0;
        hodd[i] = -1.0 / (pi2tau2 * k * k);
    }
    __syncthreads();
    const double h0 = 1.0 / (4.0 * tau * tau);
    float* dst = out + (size_t)r * nu;
    for (int a = threadIdx.x; a < nu; a += kFdkThreads) {
        const float* c = row + nu + a;
        double acc = h0 * (double)c[0];
        // odd offsets k = 2 i + 1 < nu: both neighbours a - k and a + k (zero padded)
        for (int i = 0; 2 * i + 1 < nu; ++i) {
            const int k = 2 * i + 1;
            acc = fma(hodd[i], (double)c[-k] + (double)c[k], acc);
        }
        dst[a] = (float)(scale * tau * acc);
    }
}

// Rows (of all views) from which the matrix kernel is faster: it takes 16 rows a
// block, 8 wavefronts, so that a thousand rows are needed to fill the chip, and it
// computes whole tiles of 128 outputs.  Kernel us, row by row against matrix: 512
// pixels 16 rows 7.9 / 27.1, 600 20.9 / 28.0, 1200 32.3 / 28.5, 60000 1246 / 321;
// 100 pixels 4800 rows 9.6 / 12.0, 20000 28.5 / 23.3; 2048 pixels 600 rows 222 / 297,
// 1200 355 / 302; 16 pixels never.
static int fdk_row_limit(int nu)
{
    return nu < 64 ? INT_MAX : nu <= 128 ? 8192 : nu <= 256 ? 1600 : nu <= 512 ? 1000 : nu <= 768 ? 900 : 700;
}

size_t fdk_filter_lds_bytes(int nu)
{
    return sizeof(double) * (nu / 2 + 1) + sizeof(float) * 3 * (size_t)nu;
}

void launch_fdk_filter(const GeoScalars& s, int V, const float* proj, float* out, double scale,
                       hipStream_t st)
{
    const double mag = s.sad / s.sdd;
    const double du_iso = s.du * mag, dv_iso = s.dv * mag;
    // up to 2048 pixels a block's registers hold 16 rows of FP64 outputs; longer
    // rows keep the direct kernel
    if (s.nu <= 2048) {
        const int rows = V * s.nv;
        if (rows < fdk_row_limit(s.nu)) {
            const int threads = std::min(1024, (s.nu + 127) / 128 * 128);
            const size_t lds = sizeof(double) * (2 * fdk_half(s.nu) + fdk_table(s.nu));
            const auto k = s.nu <= 1024 ? fdk_filter_row_kernel<1> : fdk_filter_row_kernel<2>;
            k<<<(unsigned)rows, threads, lds, st>>>(s.nu, s.nv, s.cu, s.cv, du_iso, dv_iso, s.sad, du_iso, scale,
                                                    proj, out);
            return;
        }
        const size_t lds = sizeof(float) * kFdkRows * kFdkPitch + sizeof(double) * fdk_table(s.nu);
        const auto k = s.nu <= 512 ? fdk_filter_mfma_kernel<4>
                                   : s.nu <= 1024 ? fdk_filter_mfma_kernel<8> : fdk_filter_mfma_kernel<16>;
        k<<<(unsigned)((rows + kFdkRows - 1) / kFdkRows), 64 * kFdkWaves, lds, st>>>(
            s.nu, s.nv, rows, s.cu, s.cv, du_iso, dv_iso, s.sad, du_iso, scale, proj, out);
        return;
    }
    const size_t lds = fdk_filter_lds_bytes(s.nu);
    fdk_filter_kernel<<<(unsigned)(V * s.nv), kFdkThreads, lds, st>>>(
        s.nu, s.nv, s.cu, s.cv, du_iso, dv_iso, s.sad, du_iso, scale, proj, out);
}

int fdk_max_nu() { return kFdkMaxNu; }

// ---------------------------------------------------------------------------
// Sharpness
// ---------------------------------------------------------------------------

constexpr int kShThreads = 256;

__global__ __launch_bounds__(kShThreads) void sharpness_kernel(int nx, int ny, int nz,
                                                               const float* __restrict__ vol,
                                                               float* __restrict__ grad,
                                                               double* __restrict__ partial)
{
    __shared__ float red[kShThreads];
    const size_t n = (size_t)nx * ny * nz;
    const size_t i = (size_t)blockIdx.x * kShThreads + threadIdx.x;
    float s = 0.0f;
    if (i < n) {
        const int x = (int)(i % nx), y = (int)((i / nx) % ny), z = (int)(i / ((size_t)nx * ny));
        const float m = vol[i];
        float g = 0.0f;
        const size_t sx = 1, sy = (size_t)nx, sz = (size_t)nx * ny;
        if (x + 1 < nx) { const float d = vol[i + sx] - m; s += d * d; g += 2.0f * d; }
        if (y + 1 < ny) { const float d = vol[i + sy] - m; s += d * d; g += 2.0f * d; }
        if (z + 1 < nz) { const float d = vol[i + sz] - m; s += d * d; g += 2.0f * d; }
        if (x > 0) g -= 2.0f * (m - vol[i - sx]);
        if (y > 0) g -= 2.0f * (m - vol[i - sy]);
        if (z > 0) g -= 2.0f * (m - vol[i - sz]);
        if (grad) grad[i] = g;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = kShThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = (double)red[0];
}

// One block: fixed-order FP64 sum of the block partials, negated.
__global__ __launch_bounds__(kShThreads) void sharpness_total_kernel(int n_part,
                                                                     const double* __restrict__ partial,
                                                                     double* __restrict__ loss)
{
    __shared__ double red[kShThreads];
    double s = 0.0;
    for (int i = threadIdx.x; i < n_part; i += kShThreads) s += partial[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = kShThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = -red[0];
}

size_t sharpness_partials(int nx, int ny, int nz)
{
    return ((size_t)nx * ny * nz + kShThreads - 1) / kShThreads;
}

void launch_sharpness(int nx, int ny, int nz, const float* vol, float* grad, double* loss,
                      double* partial, hipStream_t st)
{
    const size_t blocks = sharpness_partials(nx, ny, nz);
    sharpness_kernel<<<(unsigned)blocks, kShThreads, 0, st>>>(nx, ny, nz, vol, grad, partial);
    sharpness_total_kernel<<<1, kShThreads, 0, st>>>((int)blocks, partial, loss);
}

// ---------------------------------------------------------------------------
// Gradient entropy
// ---------------------------------------------------------------------------

struct GeDiffs {
    float dx, dy, dz, g;
};

__device__ inline GeDiffs ge_at(const float* __restrict__ vol, int x, int y, int z, int nx, int ny,
                                int nz, float eps)
{
    const size_t i = ((size_t)z * ny + y) * nx + x;
    const float m = vol[i];
    GeDiffs d;
    d.dx = x + 1 < nx ? vol[i + 1] - m : 0.0f;
    d.dy = y + 1 < ny ? vol[i + nx] - m : 0.0f;
    d.dz = z + 1 < nz ? vol[i + (size_t)nx * ny] - m : 0.0f;
    d.g = sqrtf(d.dx * d.dx + d.dy * d.dy + d.dz * d.dz + eps);
    return d;
}

__global__ __launch_bounds__(kShThreads) void ge_sums_kernel(int nx, int ny, int nz, float eps,
                                                             const float* __restrict__ vol,
                                                             double* __restrict__ partial)
{
    __shared__ float r1[kShThreads], r2[kShThreads];
    const size_t n = (size_t)nx * ny * nz;
    const size_t i = (size_t)blockIdx.x * kShThreads + threadIdx.x;
    float s1 = 0.0f, s2 = 0.0f;
    if (i < n) {
        const int x = (int)(i % nx), y = (int)((i / nx) % ny), z = (int)(i / ((size_t)nx * ny));
        const float g = ge_at(vol, x, y, z, nx, ny, nz, eps).g;
        s1 = g;
        s2 = g * logf(g);
    }
    r1[threadIdx.x] = s1;
    r2[threadIdx.x] = s2;
    __syncthreads();
    for (int w = kShThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            r1[threadIdx.x] += r1[threadIdx.x + w];
            r2[threadIdx.x] += r2[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = (double)r1[0];
        partial[2 * blockIdx.x + 1] = (double)r2[0];
    }
}

// scal[0] = Z, scal[1] = GE, scal[2] = log Z; *loss = GE.
__global__ __launch_bounds__(kShThreads) void ge_total_kernel(int n_part, const double* __restrict__ partial,
                                                              double* __restrict__ scal,
                                                              double* __restrict__ loss)
{
    __shared__ double r1[kShThreads], r2[kShThreads];
    double s1 = 0.0, s2 = 0.0;
    for (int i = threadIdx.x; i < n_part; i += kShThreads) {
        s1 += partial[2 * i];
        s2 += partial[2 * i + 1];
    }
    r1[threadIdx.x] = s1;
    r2[threadIdx.x] = s2;
    __syncthreads();
    for (int w = kShThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            r1[threadIdx.x] += r1[threadIdx.x + w];
            r2[threadIdx.x] += r2[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double Z = r1[0], lz = log(Z), ge = lz - r2[0] / Z;
        scal[0] = Z;
        scal[1] = ge;
        scal[2] = lz;
        loss[0] = ge;
    }
}

__global__ __launch_bounds__(kShThreads) void ge_grad_kernel(int nx, int ny, int nz, float eps,
                                                             const float* __restrict__ vol,
                                                             const double* __restrict__ scal,
                                                             float* __restrict__ grad)
{
    const size_t n = (size_t)nx * ny * nz;
    const size_t i = (size_t)blockIdx.x * kShThreads + threadIdx.x;
    if (i >= n) return;
    const int x = (int)(i % nx), y = (int)((i / nx) % ny), z = (int)(i / ((size_t)nx * ny));
    const float invZ = (float)(1.0 / scal[0]);
    const float shift = (float)(scal[1] - scal[2]);  // GE - log Z
    // c_j = -(log g_j + GE - log Z) / (Z g_j)
    const GeDiffs d0 = ge_at(vol, x, y, z, nx, ny, nz, eps);
    const float c0 = -(logf(d0.g) + shift) * invZ / d0.g;
    float acc = -c0 * (d0.dx + d0.dy + d0.dz);
    if (x > 0) {
        const GeDiffs d = ge_at(vol, x - 1, y, z, nx, ny, nz, eps);
        acc += -(logf(d.g) + shift) * invZ / d.g * d.dx;
    }
    if (y > 0) {
        const GeDiffs d = ge_at(vol, x, y - 1, z, nx, ny, nz, eps);
        acc += -(logf(d.g) + shift) * invZ / d.g * d.dy;
    }
    if (z > 0) {
        const GeDiffs d = ge_at(vol, x, y, z - 1, nx, ny, nz, eps);
        acc += -(logf(d.g) + shift) * invZ / d.g * d.dz;
    }
    grad[i] = acc;
}

void launch_gradient_entropy(int nx, int ny, int nz, float eps, const float* vol, float* grad,
                             double* loss, double* ws, hipStream_t st)
{
    const size_t blocks = sharpness_partials(nx, ny, nz);
    double* partial = ws;                 // [blocks][2]
    double* scal = ws + 2 * blocks;       // Z, GE, log Z
    ge_sums_kernel<<<(unsigned)blocks, kShThreads, 0, st>>>(nx, ny, nz, eps, vol, partial);
    ge_total_kernel<<<1, kShThreads, 0, st>>>((int)blocks, partial, scal, loss);
    if (grad)
        ge_grad_kernel<<<(unsigned)blocks, kShThreads, 0, st>>>(nx, ny, nz, eps, vol, scal, grad);
}

size_t gradient_entropy_ws_doubles(int nx, int ny, int nz)
{
    return 2 * sharpness_partials(nx, ny, nz) + 4;
}

}  // namespace dp
