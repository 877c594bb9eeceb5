// Full-volume reference mode (paper: Eq. 2 and the paragraph after it, the
// "default implementation"): the dense volume C = F1 . F2^T / sqrt(D) for all
// pixel pairs, a pyramid made by 2x2 average pooling of the volume's last two
// dimensions, then bilinear sampling of the pooled volumes with zero padding.
// fp32's precision throughout.  Memory is quadratic in pixels; the caller checks the size.
#include "corr_internal.h"

namespace {

constexpr size_t MAX_BLOCKS = 1u << 22;     // of 256 threads: 2^30 threads per launch, the kernels stride over the rest

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// C[p][q] = scale * sum_d A[p][d] * B[q][d].  fp32 precision on v_mfma_f32_16x16x32_bf16: an operand is the sum of three bf16
// values (24 significand bits), and the six of the nine partial products that reach 2^-24 are accumulated in fp32.
// A workgroup makes 128 x 64 elements (a wave 64 x 32), 32 channels a step: its 192 rows are split once, by the thread that
// loads them, into LDS planes [3][192 rows][32 channels], the next step's rows on their way into registers meanwhile.
// 16-byte pieces of a row lie at piece ^ (row / 4 & 3), so that 16 rows' reads of one piece meet every bank once.
// 28 x 64, D = 256: 19 us, against 61 on the vector ALU; 64 x 64: 55, where the 1.3 PFLOP/s that a large bf16 product reaches would
// give 40.  Splitting, LDS reads and matrix instructions each fill about half of the time.  64 x 64 tiles take 21 / 64 us,
// 128 x 128 ones (196 workgroups on 28 x 64) 18 / 52, and deeper prefetching changes nothing.
constexpr int TP = 128, TQ = 64, V_PLANE = (TP + TQ) * 64;
__global__ __launch_bounds__(256, 2) void vol_gemm_kernel(const float* __restrict__ A, const float* __restrict__ Bm,
                                                          float* __restrict__ C, int N, int D, float scale) {
    __shared__ __align__(16) unsigned char smem[3 * V_PLANE];
    const int b = blockIdx.z;
    A += (size_t)b * N * D; Bm += (size_t)b * N * D; C += (size_t)b * N * N;
    const int p0 = blockIdx.y * TP, q0 = blockIdx.x * TQ;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lg = lane >> 4;
    // staging: eight lanes to a row's 128 bytes, 32 rows at a time, first A's, then B's; a row past the end is the last one
    // again (its products are not stored)
    constexpr int NS = (TP + TQ) / 32;
    const float* src[NS];
    unsigned dst[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int row = 32 * i + (tid >> 3), piece = tid & 7;
        src[i] = (row < TP ? A + (size_t)min(p0 + row, N - 1) * D : Bm + (size_t)min(q0 + row - TP, N - 1) * D) + 4 * piece;
        dst[i] = (unsigned)(row * 64 + (((piece >> 1) ^ (row >> 2 & 3)) << 4) + (piece & 1) * 8);
    }
    f32x4 x[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) x[i] = *reinterpret_cast<const f32x4*>(src[i]);
    const int wp = (wave & 1) * 64, wq = (wave >> 1) * 32;       // the wave's part
    const unsigned sw = (unsigned)((lg ^ (lr >> 2 & 3)) << 4);
    const unsigned fa = (unsigned)((wp + lr) * 64) + sw, fb = (unsigned)((TP + wq + lr) * 64) + sw;
    f32x4 acc[4][2] = {};
    for (int k0 = 0; k0 < D; k0 += 32) {
        __syncthreads();                                 // the previous step's fragments have been read
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            f32x2 lo = {x[i][0], x[i][1]}, hi = {x[i][2], x[i][3]};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const bf16x2 cl = __builtin_convertvector(lo, bf16x2), ch = __builtin_convertvector(hi, bf16x2);
                *reinterpret_cast<u32x2*>(smem + k * V_PLANE + dst[i]) = u32x2{__builtin_bit_cast(unsigned, cl), __builtin_bit_cast(unsigned, ch)};
                lo -= __builtin_convertvector(cl, f32x2); hi -= __builtin_convertvector(ch, f32x2);
            }
        }
        const int kn = min(k0 + 32, D - 32);             // the last step loads its own again
#pragma unroll
        for (int i = 0; i < NS; ++i) x[i] = *reinterpret_cast<const f32x4*>(src[i] + kn);
        __syncthreads();
        bf16x8 fa3[4][3], fb3[2][3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
#pragma unroll
            for (int j = 0; j < 2; ++j) fb3[j][k] = *reinterpret_cast<const bf16x8*>(smem + k * V_PLANE + fb + j * 1024);
#pragma unroll
            for (int i = 0; i < 4; ++i) fa3[i][k] = *reinterpret_cast<const bf16x8*>(smem + k * V_PLANE + fa + i * 1024);
        }
        // small products first
        constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int m = 0; m < 6; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa3[i][PA[m]], fb3[j][PB[m]], acc[i][j], 0, 0, 0);
    }
    // An infinity, a NaN or a value beyond bf16's range has no three parts (its remainder is infinity - infinity): what is not finite
    // here is taken from fp32 instructions instead, four channels of a row per lane and 16 a step.
    float none = 0.f;                                    // NaN if any sum is not finite
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) none = fmaf(acc[i][j][e], 0.f, none);
    if (__any(none != 0.f)) {
        f32x4 plain[4][2] = {};
        for (int k0 = 0; k0 < D; k0 += 16) {
            f32x4 xa[4], xb[2];
#pragma unroll
            for (int i = 0; i < 4; ++i) xa[i] = *reinterpret_cast<const f32x4*>(A + (size_t)min(p0 + wp + 16 * i + lr, N - 1) * D + k0 + 4 * lg);
#pragma unroll
            for (int j = 0; j < 2; ++j) xb[j] = *reinterpret_cast<const f32x4*>(Bm + (size_t)min(q0 + wq + 16 * j + lr, N - 1) * D + k0 + 4 * lg);
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) plain[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[i][c], xb[j][c], plain[i][j], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (!(fabsf(acc[i][j][e]) < INFINITY)) acc[i][j][e] = plain[i][j][e];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int p = p0 + wp + 16 * i + 4 * lg + e, q = q0 + wq + 16 * j + lr;
                if (p < N && q < N) C[(size_t)p * N + q] = acc[i][j][e] * scale;
            }
}

// Every pooled level in one pass over the volume: dst_l[v][u] = 0.25 * (((s[2v][2u] + s[2v][2u+1]) + s[2v+1][2u]) + s[2v+1][2u+1])
// of the level before.  A wave takes 8 rows x 32 columns of one query's image: a lane 2 x 2 of them (4 x 16 lanes), the
// deeper levels from the neighbouring lanes.  Bound by the traffic: the volume is read once, instead of each level after it was
// written, and two launches go away.  28 x 64: 6 us, against three times 5; 64 x 64: 19.5 us = 4.5 TB/s.
struct PoolArgs {
    const float* src;
    float* dst[CORR_MAX_L];                  // levels 1 ..
    int Hl[CORR_MAX_L], Wl[CORR_MAX_L];
    int L;
    size_t rows;                             // images
};
__global__ __launch_bounds__(256) void vol_pool_kernel(PoolArgs a) {
    const int H = a.Hl[0], W = a.Wl[0], lane = threadIdx.x & 63, lx = lane & 15, ly = lane >> 4;
    const int tx = (W + 31) / 32, tiles = tx * ((H + 7) / 8);
    const size_t total = a.rows * (size_t)tiles, step = (size_t)gridDim.x * 4;
    for (size_t w = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6); w < total; w += step) {
        const size_t image = w / (unsigned)tiles;
        const int tile = (int)(w - image * (unsigned)tiles), ty = tile / tx;
        int y = ty * 4 + ly, x = (tile - ty * tx) * 16 + lx;                   // of level 1
        const float* s = a.src + image * (size_t)H * W;
        float v = 0.f;
        if (y < a.Hl[1] && x < a.Wl[1]) {
            const float* t = s + (size_t)(2 * y) * W + 2 * x;
            v = 0.25f * (((t[0] + t[1]) + t[W]) + t[W + 1]);
            a.dst[1][image * (size_t)a.Hl[1] * a.Wl[1] + (size_t)y * a.Wl[1] + x] = v;
        }
#pragma unroll
        for (int l = 2; l < CORR_MAX_L; ++l) {
            if (l >= a.L) break;
            // lanes whose place is even in both axes at every level so far hold a value of level l - 1
            const int d = 1 << (l - 2);
            const float right = __shfl_down(v, d), below = __shfl_down(v, 16 * d), across = __shfl_down(v, 17 * d);
            v = 0.25f * (((v + right) + below) + across);
            y >>= 1; x >>= 1;
            if ((lx & (2 * d - 1)) == 0 && (ly & (2 * d - 1)) == 0 && y < a.Hl[l] && x < a.Wl[l])
                a.dst[l][image * (size_t)a.Hl[l] * a.Wl[l] + (size_t)y * a.Wl[l] + x] = v;
        }
    }
}

struct FvArgs {
    const float* vol[CORR_MAX_L];
    const float* coords;
    float* out;
    int B, HW, L, r;
    int tap_stride, pix_stride;      // layout of out
    int Hl[CORR_MAX_L], Wl[CORR_MAX_L];
};

// A workgroup = one level of 16 consecutive queries of a batch item, 16 lanes a query: lane x reads column x of the footprint
// (2r + 2 columns and rows), so a load's lanes lie on four queries' rows and all of a thread's loads are in flight at once; the column to the
// right comes from the next lane.  The taps leave through LDS, in runs of 64 bytes along the pixels (the taps, channels-last).
// Bound by latency: launch, coordinates, footprint, output.  One thread per tap with four loads of its own and 64-bit
// divisions took 10 us on 28 x 64; this takes 4.
constexpr int SQ = 16, SKK = (2 * CORR_R + 1) * (2 * CORR_R + 1);
__global__ __launch_bounds__(256) void vol_sample_kernel(FvArgs a) {
    __shared__ float taps[SKK * (SQ + 1)];
    const int K = 2 * a.r + 1, KK = K * K, l = blockIdx.y, b = blockIdx.z;
    const int H = a.Hl[l], W = a.Wl[l];
    const int q = threadIdx.x >> 4, i = threadIdx.x & 15, pix0 = blockIdx.x * SQ, pix = min(pix0 + q, a.HW - 1);
    const float cx0 = a.coords[((size_t)b * 2 + 0) * a.HW + pix];
    const float cy0 = a.coords[((size_t)b * 2 + 1) * a.HW + pix];
    const bool ok = fabsf(cx0) <= CORR_COORD_LIMIT && fabsf(cy0) <= CORR_COORD_LIMIT;
    const float inv = __uint_as_float((uint32_t)(127 - l) << 23);
    const float cx = ok ? cx0 * inv : 0.f, cy = ok ? cy0 * inv : 0.f;
    const float flx = floorf(cx), fly = floorf(cy);
    const float fx = cx - flx, fy = cy - fly;
    const int x = (int)flx - a.r + i, y0 = (int)fly - a.r;
    const bool col = ok && i <= K && x >= 0 && x < W;
    const float* vp = a.vol[l] + ((size_t)b * a.HW + pix) * (size_t)H * W + (col ? x : 0);
    float v[2 * CORR_R + 2];
#pragma unroll
    for (int j = 0; j < 2 * CORR_R + 2; ++j)
        v[j] = j <= K && col && y0 + j >= 0 && y0 + j < H ? vp[(size_t)(unsigned)(y0 + j) * (unsigned)W] : 0.f;
    const float w00 = (1.f - fx) * (1.f - fy), w01 = fx * (1.f - fy), w10 = (1.f - fx) * fy, w11 = fx * fy;
    float right[2 * CORR_R + 2];
#pragma unroll
    for (int j = 0; j < 2 * CORR_R + 2; ++j) right[j] = __shfl_down(v[j], 1);
    if (i < K) {
#pragma unroll
        for (int j = 0; j < 2 * CORR_R + 1; ++j)
            if (j < K) taps[(i * K + j) * (SQ + 1) + q] = w00 * v[j] + w01 * right[j] + w10 * v[j + 1] + w11 * right[j + 1];
    }
    __syncthreads();
    float* out = a.out + (size_t)b * a.L * KK * a.HW + (size_t)(l * KK) * a.tap_stride + (size_t)pix0 * a.pix_stride;
    if (a.pix_stride == 1) {
        for (int t = q; t < KK; t += 16)
            if (pix0 + i < a.HW) out[(size_t)t * a.tap_stride + i] = taps[t * (SQ + 1) + i];
    } else {
        for (int t = i; t < KK; t += 16)
            if (pix0 + q < a.HW) out[(size_t)q * a.pix_stride + t] = taps[t * (SQ + 1) + q];
    }
}

}  // namespace

hipError_t launch_fullvol_build(const corr_pyramid* p, hipStream_t s) {
    const int N = p->H * p->W;
    dim3 grid((N + TQ - 1) / TQ, (N + TP - 1) / TP, p->B);
    hipLaunchKernelGGL(vol_gemm_kernel, grid, dim3(256), 0, s, p->f1_nhwc, p->f2_nhwc[0], p->vol[0], N, p->D,
                       1.0f / sqrtf((float)p->D));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (p->L > 1) {
        PoolArgs a;
        a.src = p->vol[0]; a.L = p->L; a.rows = (size_t)p->B * N;
        for (int l = 0; l < CORR_MAX_L; ++l) { a.dst[l] = l < p->L ? p->vol[l] : nullptr; a.Hl[l] = p->Hl[l]; a.Wl[l] = p->Wl[l]; }
        const size_t blocks = (a.rows * ((p->H + 7) / 8) * ((p->W + 31) / 32) + 3) / 4;
        hipLaunchKernelGGL(vol_pool_kernel, dim3((unsigned)(blocks < MAX_BLOCKS ? blocks : MAX_BLOCKS)), dim3(256), 0, s, a);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_fullvol_sample(const corr_pyramid* p, const LookupArgs& q, hipStream_t s) {
    FvArgs a;
    for (int l = 0; l < CORR_MAX_L; ++l) {
        a.vol[l] = l < p->L ? p->vol[l] : nullptr;
        a.Hl[l] = p->Hl[l]; a.Wl[l] = p->Wl[l];
    }
    a.coords = q.coords; a.out = q.out; a.B = p->B; a.HW = p->H * p->W; a.L = p->L; a.r = q.r;
    a.tap_stride = corr_tap_stride(p, q); a.pix_stride = corr_pix_stride(p, q);
    const dim3 grid((unsigned)(a.HW + SQ - 1) / SQ, (unsigned)p->L, (unsigned)p->B);
    hipLaunchKernelGGL(vol_sample_kernel, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}
