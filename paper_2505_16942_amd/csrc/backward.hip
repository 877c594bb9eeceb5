// Gradient of the lookup with respect to the two feature maps (the paper leaves the backward pass as future
// work, Sec. "Conclusion"; what it computes follows from Eq. 1).  Coordinates are constants.
//
// For one query p and level l the 81 tap gradients fold into a (K+1) x (K+1) footprint of weights
//     G[v][u] = sum over the up to four taps whose bilinear stencil touches footprint point (u, v) of
//               d_out[tap] * (corner weight),
// because all taps of a query share one fractional part.  Then
//     d f1(p)       += G[v][u] / sqrt(D) * f2_l(origin + (u, v))
//     d f2_l(q)     += G[v][u] / sqrt(D) * f1(p)          (q = origin + (u, v), inside the level)
// and the levels' gradients go down the pyramid by the adjoint of the 2x2 mean.
//
// Both forms below read the fp32 channels-last representation of the pyramid (CORR_REP_F32), accumulate the
// gradients channels-last in a caller-provided workspace and bring them to NCHW at the end.  Summation order of
// the atomics on d f2_l is not fixed: d_fmap2 agrees between calls to rounding, not bit for bit.
//
// The first form is the plain one: one wave per query, fp32 vector ALU, channels across lanes, a hardware float
// atomic per (footprint point, channel) for d f2_l.  The second, further down, is what the entry point runs.
#include "corr_internal.h"

namespace {

constexpr int BQ = 4;                       // queries (waves) per workgroup
constexpr int MAXK = 2 * CORR_R + 1;
constexpr int MAX_NK = 1024 / 64;           // channel slots per lane at the largest D

struct BwdArgs {
    const float* f1;                        // [B*HW][D]
    const float* f2[CORR_MAX_L];            // [B*Hl*Wl][D]
    float* d_f1;                            // [B*HW][D], written
    float* d_f2[CORR_MAX_L];                // [B*Hl*Wl][D], zero on entry, accumulated
    const float* coords;                    // [B][2][HW]
    const float* d_out;                     // [B][L*K*K][HW]
    int B, HW, D, L, r;
    int Hl[CORR_MAX_L], Wl[CORR_MAX_L];
    float scale;
};

// Weight of footprint point (pu, pv): of the taps (i, j) = (pu - du, pv - dv), du, dv in {0, 1}, with their corner weights.  Tap
// (i, j), i the x offset, is taps[(i * K + j) * stride].
__device__ __forceinline__ float footprint_weight(const float* taps, int stride, int K, int pu, int pv, float fx, float fy) {
    float g = 0.f;
#pragma unroll
    for (int dv = 0; dv < 2; ++dv)
#pragma unroll
        for (int du = 0; du < 2; ++du) {
            const int i = pu - du, j = pv - dv;
            if (i >= 0 && i < K && j >= 0 && j < K)
                g += taps[(size_t)(i * K + j) * stride] * (du ? fx : 1.f - fx) * (dv ? fy : 1.f - fy);
        }
    return g;
}

__global__ __launch_bounds__(64 * BQ) void bwd_query_kernel(BwdArgs a) {
    __shared__ float s_taps[BQ][MAXK * MAXK];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int K = 2 * a.r + 1, KK = K * K, NK = (a.D + 63) / 64;
    const long long q = (long long)blockIdx.x * BQ + wave;
    const bool real = q < (long long)a.B * a.HW;          // waves past the end stay for the barriers
    const int b = real ? (int)(q / a.HW) : 0, p = real ? (int)(q - (long long)b * a.HW) : 0;
    const float cx = a.coords[((size_t)b * 2 + 0) * a.HW + p], cy = a.coords[((size_t)b * 2 + 1) * a.HW + p];
    // comparisons are false for NaN: non-finite or huge coordinates give the constant 0, no gradient
    const bool live = real && fabsf(cx) <= CORR_COORD_LIMIT && fabsf(cy) <= CORR_COORD_LIMIT;
    float f1r[MAX_NK], acc[MAX_NK];
#pragma unroll
    for (int k = 0; k < MAX_NK; ++k) {
        const int ch = lane + 64 * k;
        f1r[k] = (k < NK && ch < a.D && real) ? a.f1[(size_t)q * a.D + ch] : 0.f;
        acc[k] = 0.f;
    }
    for (int l = 0; l < a.L; ++l) {
        __syncthreads();                                   // the previous level's taps are no longer read
        for (int t = lane; t < KK; t += 64)
            s_taps[wave][t] = live ? a.d_out[((size_t)b * a.L * KK + (size_t)l * KK + t) * a.HW + p] : 0.f;
        __syncthreads();
        if (!live) continue;                               // uniform per wave; the barriers above are outside
        const float inv = __uint_as_float((uint32_t)(127 - l) << 23);
        const float cxl = cx * inv, cyl = cy * inv;
        const float flx = floorf(cxl), fly = floorf(cyl);
        const float fx = cxl - flx, fy = cyl - fly;
        const int x0 = (int)flx - a.r, y0 = (int)fly - a.r;
        const int Hl = a.Hl[l], Wl = a.Wl[l];
        for (int pv = 0; pv <= K; ++pv) {
            const int v = y0 + pv;
            if (v < 0 || v >= Hl) continue;
            for (int pu = 0; pu <= K; ++pu) {
                const int u = x0 + pu;
                if (u < 0 || u >= Wl) continue;
                const float g = footprint_weight(s_taps[wave], 1, K, pu, pv, fx, fy) * a.scale;
                const size_t row = ((size_t)b * Hl * Wl + (size_t)v * Wl + u) * a.D;
                const float* f2p = a.f2[l] + row;
                float* dp = a.d_f2[l] + row;
#pragma unroll
                for (int k = 0; k < MAX_NK; ++k) {
                    const int ch = lane + 64 * k;
                    if (k < NK && ch < a.D) {
                        acc[k] += g * f2p[ch];
                        unsafeAtomicAdd(dp + ch, g * f1r[k]);
                    }
                }
            }
        }
    }
    if (real) {
#pragma unroll
        for (int k = 0; k < MAX_NK; ++k) {
            const int ch = lane + 64 * k;
            if (k < NK && ch < a.D) a.d_f1[(size_t)q * a.D + ch] = acc[k];
        }
    }
}

// ---------------------------------------------------------------------------------------------------------
// The item form: the same work items as the forward block kernel (a target cell and up to 128 of its queries, at every
// level the window of points their footprints cover), and both gradients as dense contractions on the matrix cores.
// For one item and level, with G[point][query] the footprint weights of every query scattered over the window
// (zero outside the query's footprint) and 1/sqrt(D) folded in:
//     d f1[query][:]       += sum over points  G[point][query] * f2_l[point][:]       (M = queries, K = points)
//     d f2_l[point][:]     += sum over queries G[point][query] * f1[query][:]         (M = points,  K = queries)
// fp32 in, fp32 accumulation, at fp32's precision on v_mfma_f32_16x16x32_bf16: every operand is the sum of three bf16
// values (hi + mid + lo hold all 24 bits of an fp32 significand), and of the nine partial products the six that reach
// 2^-24 are accumulated (hi*hi, hi*mid, mid*hi, mid*mid, hi*lo, lo*hi).  Six products at 16 times the rate of
// v_mfma_f32_16x16x4_f32, which this replaced; the error against fp64 is the same (rms 1.8e-7 of d f1's).
// Queries are ranked by target column and points are numbered column by column, so a tile of 16 queries and a run of 32
// points meet only if the tile's footprints reach those columns; the others are skipped (about half of them at level
// 0, where a full item's window is 25 columns wide and a tile's footprints are 11 or 12).
// G is built CH points at a time from the tap gradients (a footprint point collects up to four taps) in LDS, three bf16
// planes [point][query], 32-byte blocks XOR-swizzled by the point.  The second contraction reads its fragments along the
// queries as they lie, the first one through the transposing LDS read.  The feature rows are the B operands: lane =
// (channel, 8 consecutive points or queries), loaded as fp32 in that layout and split in registers; f1's fragments stay in
// registers for the whole item.  d f1 stays in accumulators over all levels and is stored once (a query belongs to one
// item, so its bits are the same on every call); the window's d f2_l rows go out through float atomics once per item and
// pass, instead of once per query and footprint point.
// Measured, D = 256: the call takes 1.21 ms on a 270 x 480 map and 0.205 ms on two 46 x 62 ones, against 1.62 and 0.28 ms with fp32
// instructions, every tile against every point, and one 64-byte row piece per atomic.  An item's 156 us on 270 x 480 are 55 and 56
// in the two contractions (matrix pipes 38 of both together), 17 in the scatter (serial work per footprint column), 14 waiting
// for tap gradients and 8 clearing G; 30 of the second contraction's are its atomics, which all execute beyond the L2.  Half
// of the waves on each contraction at the same time, the window's rows warmed into the L2 during the scatter, and loads
// two runs ahead (spills) were no faster.
// Eight waves, two per SIMD: a wave owns 32 channels of a 256-channel group (16 of a 128-channel group for D <= 128).
// Feature rows come through buffer resources: an offset past the end reads zero and an atomic there is dropped, so rows
// outside the level and empty query slots need no branch inside the loops.
constexpr int NTI = 512;
constexpr int CH = 144;                     // window points per pass: level 2's window in one pass, level 0's in three
constexpr int QT = CORR_GROUP / 16;         // 16-query tiles
constexpr int G_PLANE = CORR_GROUP * 2;     // bytes of a point in one plane
constexpr int G_ROW = 3 * G_PLANE;
constexpr int MAXKK = MAXK * MAXK;
constexpr int TAB = CH + 16;                // the last run of 32 points ends past the pass: invalid entries
// LDS layout (bytes)
constexpr int I_G = 0;                                  // [CH][3][128] bf16
constexpr int I_ROW = I_G + CH * G_ROW;                 // [TAB] byte offset of each point's feature row; BAD_OFF: outside the level
constexpr int I_Q = I_ROW + TAB * 4;                    // [128] by rank: byte offset of the query's feature row; BAD_OFF: empty
constexpr int I_CX = I_Q + CORR_GROUP * 4;              // [128] each by rank: coordinates, pixel * 4 (BAD_OFF: empty), target column inside the cell
constexpr int I_CY = I_CX + CORR_GROUP * 4;
constexpr int I_PIX = I_CY + CORR_GROUP * 4;
constexpr int I_COL = I_PIX + CORR_GROUP * 4;
constexpr int I_HIST = I_COL + CORR_GROUP * 4;          // [16] queries per column
constexpr int I_NEXT = I_HIST + 16 * 4;                 // the workgroup's next queue position
constexpr int I_TAPS = I_HIST + 32 * 4;                 // [K*K][128] tap gradients of the level in work, by rank
constexpr int ITEM_LDS = I_TAPS + MAXKK * CORR_GROUP * 4;
static_assert(ITEM_LDS <= 160 * 1024 && I_ROW % 16 == 0 && I_Q % 16 == 0, "LDS layout");
constexpr unsigned BAD_OFF = 0x80000000u;   // beyond every buffer here (each is below 2 GiB)

struct BwdItemArgs {
    const float* f1;
    const float* f2[CORR_MAX_L];
    float* d_f1;                            // zero on entry (queries without an item keep the zero)
    float* d_f2[CORR_MAX_L];                // zero on entry, accumulated
    const float* d_out;
    const int* perm;
    const float2* sorted_c;
    const int4* items;
    const int* n_items;
    int* queue;                             // [8] next queue position per XCD, zero on entry
    int parts;                              // 1, 2 or L: small inputs run an item's levels in workgroups of their own, each with
                                            // a d_f1 array of its own (part p at d_f1 + p * B*HW*D), summed in order at the end
    int B, HW, D, L, r;
    int Hl[CORR_MAX_L], Wl[CORR_MAX_L];
    CellGrid g;
    float scale;
#ifdef CORR_TRACE
    long long* trace;
#endif
};

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
typedef __attribute__((address_space(3))) u32x4* lds_u32x4;
typedef __attribute__((address_space(3))) __bf16* lds_bf16;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const float* base, size_t floats) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, (int)(unsigned)(floats * 4), 0x00020000);
}
typedef int i32x4 __attribute__((ext_vector_type(4)));
// 4 bytes per lane from a buffer straight into LDS at lds_base + lane * 4 (lds_base, the resource and soff uniform).
// A lane whose offset lies beyond the resource's size writes zero.
__device__ __forceinline__ void dma4(i32x4 rsrc, unsigned lds_base, unsigned voff, int soff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds"
                 :: "s"(lds_base), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
__device__ __forceinline__ float buf_load(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}

// three bf16 values whose sum is the fp32 value: rounded, the rounded remainder, and the rest
struct Split3 { bf16x8 p[3]; };
__device__ __forceinline__ void split2(f32x2 v, bf16x2 (&p)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        p[k] = __builtin_convertvector(v, bf16x2);
        v -= __builtin_convertvector(p[k], f32x2);
    }
}
__device__ __forceinline__ Split3 split8(const float (&v)[8]) {
    Split3 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        bf16x2 p[3];
        split2(f32x2{v[2 * i], v[2 * i + 1]}, p);
#pragma unroll
        for (int k = 0; k < 3; ++k) { r.p[k][2 * i] = p[k][0]; r.p[k][2 * i + 1] = p[k][1]; }
    }
    return r;
}
// acc += a * b to fp32's precision: the six partial products down to 2^-24, small ones first
__device__ __forceinline__ f32x4 mma6(const Split3& a, const Split3& b, f32x4 c) {
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[2], b.p[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[0], b.p[2], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[1], b.p[1], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[1], b.p[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[0], b.p[1], c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[0], b.p[0], c, 0, 0, 0);
}
// LDS byte of (point, plane 0, block of 16 query ranks) of G: 32-byte blocks, XOR-swizzled by the point so that reads along
// the points (8 of them, one block each) and along the queries spread over all banks
__device__ __forceinline__ unsigned g_at(int row, int block) { return (unsigned)(row * G_ROW + ((block ^ (row & 7)) << 5)); }

#ifdef CORR_TRACE
// trace builds: thread 0 adds up the 100 MHz wall clock per phase (a barrier in front of every reading, so a phase's
// time is that of its slowest wave) and leaves the item's seven sums and its tile count in trace[item][8]
#define BT(slot) do { __builtin_amdgcn_s_barrier(); if (tid == 0) { long long now = (long long)wall_clock64(); tacc[slot] += now - tlast; tlast = now; } } while (0)
#else
#define BT(slot) do {} while (0)
#endif
// One item, levels lv_lo .. lv_hi - 1, d f1 into share `part` (whole items: all levels, share 0).
// KT: the footprint's taps per axis, 2r + 1, as a constant (the largest radius, the usual one), or 0: taken from the arguments
// NTW: 16-channel tiles per wave: 2 (a workgroup covers 256 channels at a time), or 1 for D <= 128, so that all
// eight waves have channels to work on
template <int KT, int NTW>
__device__ __forceinline__ void bwd_item_body(const BwdItemArgs& a, unsigned char* smem, const int4 item, const int k,
                                              const int lv_lo, const int lv_hi, const int part) {
    unsigned* rowoff = reinterpret_cast<unsigned*>(smem + I_ROW);
    unsigned* q_off = reinterpret_cast<unsigned*>(smem + I_Q);
    float* q_cx = reinterpret_cast<float*>(smem + I_CX);
    float* q_cy = reinterpret_cast<float*>(smem + I_CY);
    unsigned* q_pix = reinterpret_cast<unsigned*>(smem + I_PIX);
    int* q_col = reinterpret_cast<int*>(smem + I_COL);
    int* hist = reinterpret_cast<int*>(smem + I_HIST);
    float* taps = reinterpret_cast<float*>(smem + I_TAPS);
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    const int n = item.z;
#ifdef CORR_TRACE
    long long tacc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    long long tlast = (long long)wall_clock64();
#endif
    int b, u, v;
    corr_cell_coords(a.g, item.x, &b, &u, &v);
    const int cell_x = (u + a.g.u_min) * (1 << CORR_LOG_CX), cell_y = (v + a.g.v_min) * (1 << CORR_LOG_CY);
    const int K = KT ? KT : 2 * a.r + 1, KK = K * K, D = a.D;
    const int R = (K - 1) / 2;
    // the item's queries, ranked by target column
    {
        const bool real = tid < n;
        int rx = 0, rank = 0;
        unsigned pix = 0;
        float2 xy = {0.f, 0.f};
        if (real) {
            xy = a.sorted_c[item.y + tid];
            pix = (unsigned)(a.perm[item.y + tid] - b * a.HW);
            rx = ((int)floorf(xy.x) - cell_x) & ((1 << CORR_LOG_CX) - 1);
        }
        if (tid < CORR_GROUP) { q_pix[tid] = BAD_OFF; q_off[tid] = BAD_OFF; }
        if (tid >= NTI - 16) hist[tid - (NTI - 16)] = 0;
        __syncthreads();
        if (real) rank = atomicAdd(&hist[rx], 1);
        __syncthreads();
        if (real) {
#pragma unroll
            for (int i = 0; i < 16; ++i) rank += i < rx ? hist[i] : 0;
            q_cx[rank] = xy.x; q_cy[rank] = xy.y; q_pix[rank] = pix * 4u;
            q_col[rank] = rx; q_off[rank] = pix * (unsigned)D * 4u;
        }
        __syncthreads();
    }
    const int tiles = (n + 15) >> 4;
    // lane t: leftmost and rightmost target column of tile t
    const int tx0 = q_col[min(16 * (lane & (QT - 1)), n - 1)], tx1 = q_col[min(16 * (lane & (QT - 1)) + 15, n - 1)];
    BT(0);
    const __amdgpu_buffer_rsrc_t r_f1 = rsrc_of(a.f1 + (size_t)b * a.HW * D, (size_t)a.HW * D);
    const __amdgpu_buffer_rsrc_t r_d1 = rsrc_of(a.d_f1 + ((size_t)part * a.B + b) * a.HW * D, (size_t)a.HW * D);

    for (int cg = 0; cg < D; cg += 128 * NTW) {                  // channel groups of 128 * NTW: 16 * NTW per wave
        const int ch = cg + wave * (16 * NTW) + lr;              // this lane's channel of tile nt: ch + 16 * nt
        const unsigned ch4 = (unsigned)ch * 4u;
        // the first contraction deals a wave's channels out alternately (tile nt, column lr: channel NTW * lr + nt), so that a lane's
        // are next to each other in memory
        const unsigned ca4 = (unsigned)(cg + wave * (16 * NTW) + NTW * lr) * 4u;
        const bool wave_on = cg + wave * (16 * NTW) < D;         // uniform; D is a multiple of 32
        f32x4 acc1[QT][NTW];
#pragma unroll
        for (int t = 0; t < QT; ++t)
#pragma unroll
            for (int nt = 0; nt < NTW; ++nt) acc1[t][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
        // f1 as the second contraction's B operand: queries 32 * s + 8 * lg + i of this lane's channels
        Split3 f1f[QT / 2][NTW];
        if (wave_on) {
#pragma unroll
            for (int s = 0; s < QT / 2; ++s) {
                float x[NTW][8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const unsigned off = q_off[32 * s + 8 * lg + i] + ch4;
#pragma unroll
                    for (int nt = 0; nt < NTW; ++nt) x[nt][i] = buf_load(r_f1, off + 64u * nt);
                }
#pragma unroll
                for (int nt = 0; nt < NTW; ++nt) f1f[s][nt] = split8(x[nt]);
            }
        }

        // Tap gradients of one level, from d_out straight into LDS (no registers in between, so the loads can fly
        // under a contraction): wave = (half of the queries, every fourth tap), lane = query.  The level's K*K
        // planes of this batch item are one buffer: the lane's pixel is the vector offset (an empty slot's lies
        // past the end and lands as zero), the tap's plane a scalar offset; a wave's 64 values land at
        // taps[t][64 * half + lane].
        const unsigned tq_off = q_pix[tid & (CORR_GROUP - 1)];   // pixel * 4
        int tv_level = -1;
        auto load_taps = [&](int lv) {
            const uint64_t base = reinterpret_cast<uint64_t>(a.d_out + ((size_t)(b * a.L + lv) * KK) * a.HW);
            i32x4 rs;
            rs[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)base);
            rs[1] = __builtin_amdgcn_readfirstlane((int)((base >> 32) & 0xffffu));
            rs[2] = __builtin_amdgcn_readfirstlane(KK * a.HW * 4);
            rs[3] = __builtin_amdgcn_readfirstlane(0x00020000);
            const unsigned to = __builtin_amdgcn_readfirstlane(lds0 + (unsigned)I_TAPS + (unsigned)(wave & 1) * 256u);
            for (int t = wave >> 1; t < KK; t += NTI / CORR_GROUP)
                dma4(rs, __builtin_amdgcn_readfirstlane(to + (unsigned)t * (CORR_GROUP * 4)), tq_off,
                     __builtin_amdgcn_readfirstlane(t * a.HW * 4));
            tv_level = lv;
        };
        for (int l = lv_lo; l < lv_hi; ++l) {
            const int Hl = a.Hl[l], Wl = a.Wl[l];
            // the cell's window: points are numbered the same way whatever queries the item holds, so that a query's sums do
            // not depend on its company (bits)
            const int xs = (cell_x >> l) - R, ys = (cell_y >> l) - R;
            const int wx = max((1 << CORR_LOG_CX) >> l, 1) + K, wy = max((1 << CORR_LOG_CY) >> l, 1) + K;
            if (!(xs + wx - 1 >= 0 && xs <= Wl - 1 && ys + wy - 1 >= 0 && ys <= Hl - 1)) continue;   // all padding (uniform)
            const __amdgpu_buffer_rsrc_t r_f2 = rsrc_of(a.f2[l] + (size_t)b * Hl * Wl * D, (size_t)Hl * Wl * D);
            const __amdgpu_buffer_rsrc_t r_d2 = rsrc_of(a.d_f2[l] + (size_t)b * Hl * Wl * D, (size_t)Hl * Wl * D);
            const float iwy = 1.0f / (float)wy;
            // this level's tap gradients: on their way into LDS since the previous level's last pass, or loaded now
            // (the first level, or one after a level that was all padding)
            if (tv_level != l) {
                __syncthreads();                                 // the previous level's last pass no longer reads taps
                load_taps(l);
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this wave's part has landed; the passes' barriers cover the others'
            BT(1);
            // lane t: the points that the footprints of tile t reach, columns of the window from its leftmost to its rightmost one
            const int first_pt = (tx0 >> l) * wy, end_pt = (lane & (QT - 1)) < tiles ? ((tx1 >> l) + K + 1) * wy : 0;
            // bit t: tile t's footprints reach points p .. p + len - 1 (uniform)
            auto reached = [&](int p, int len) { return (unsigned)__ballot(p < end_pt && p + len > first_pt) & ((1u << QT) - 1u); };
            const int begin = __builtin_amdgcn_readlane(first_pt, 0), npts = __builtin_amdgcn_readlane(end_pt, tiles - 1);   // of the whole item
            for (int r0 = begin / CH * CH; r0 < npts; r0 += CH) {
                __syncthreads();                                 // the previous pass no longer reads G or rowoff
                {
                    u32x4* g4 = reinterpret_cast<u32x4*>(smem + I_G);
                    const int used = (min(CH, npts - r0) + 31 & ~31) < CH ? min(CH, npts - r0) + 31 & ~31 : CH;   // whole runs of points
                    for (int i = tid; i < used * (G_ROW / 16); i += NTI) g4[i] = u32x4{0u, 0u, 0u, 0u};
                    if (tid < TAB) {
                        const int p = r0 + tid, px = (int)(((float)p + 0.5f) * iwy), py = p - px * wy;     // p < 512: exact
                        const int y = ys + py, x = xs + px;
                        rowoff[tid] = (tid < CH && p < npts && y >= 0 && y < Hl && x >= 0 && x < Wl) ? (unsigned)(y * Wl + x) * (unsigned)D * 4u : BAD_OFF;
                    }
                }
                __syncthreads();
                BT(2);
                const int rows = min(CH, npts - r0), nks = (rows + 31) >> 5;
                // f2 rows of a run of 32 points as the first contraction's B operand: points 8 * lg .. + 7 of this lane's channels.
                typedef unsigned raw_t __attribute__((ext_vector_type(NTW)));
                raw_t x[8];
                auto load_b = [&](int ks) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const u32x4 off = *reinterpret_cast<const u32x4*>(rowoff + 32 * ks + 8 * lg + 4 * h);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            if constexpr (NTW == 2) x[4 * h + i] = __builtin_amdgcn_raw_buffer_load_b64(r_f2, (int)(off[i] + ca4), 0, 0);
                            else x[4 * h + i] = __builtin_amdgcn_raw_buffer_load_b32(r_f2, (int)(off[i] + ca4), 0, 0);
                        }
                    }
                };
                {
                    // footprint weights into G: thread = (query, every fourth footprint column).  Point (pu, pv)
                    // collects the taps (pu - du, pv - dv), du, dv in {0, 1}, with their corner weights; every
                    // element of G has one writer, so G (and with it d f1) is the same bits on every call.
                    const int q = tid & (CORR_GROUP - 1), quarter = tid >> 7;
                    if (q < n) {
                        const float inv = __uint_as_float((uint32_t)(127 - l) << 23);
                        const float cxl = q_cx[q] * inv, cyl = q_cy[q] * inv;
                        const float flx = floorf(cxl), fly = floorf(cyl);
                        const float fx = cxl - flx, fy = cyl - fly;
                        const int rx = (int)flx - R - xs, ry = (int)fly - R - ys;
                        const float wx1 = fx * a.scale, wx0 = a.scale - wx1;
                        const float* dp = taps + q;
                        const unsigned gq = lds0 + (unsigned)(I_G + (q & 15) * 2);
                        for (int pu = quarter; pu <= K; pu += 4) {
                            const int row0 = (rx + pu) * wy + ry - r0;                   // of the column's first point
                            if (row0 <= -(K + 1) || row0 >= CH) continue;                // none in this pass
                            // the column's horizontally weighted taps first (all LDS reads in flight at once), then its K + 1 points
                            const float w0 = pu < K ? wx0 : 0.f, w1 = pu >= 1 ? wx1 : 0.f;
                            const float* c0 = dp + min(pu, K - 1) * K * CORR_GROUP;
                            const float* c1 = dp + max(pu - 1, 0) * K * CORR_GROUP;
                            float t[MAXK + 2];
                            t[0] = 0.f;
#pragma unroll
                            for (int j = 0; j < MAXK; ++j) {
                                const int jj = min(j, K - 1);
                                t[j + 1] = j < K ? c0[jj * CORR_GROUP] * w0 + c1[jj * CORR_GROUP] * w1 : 0.f;
                            }
                            t[MAXK + 1] = 0.f;
#pragma unroll
                            for (int pv = 0; pv <= MAXK; pv += 2) {
                                bf16x2 p[3];
                                split2(f32x2{t[pv + 1] + fy * (t[pv] - t[pv + 1]), t[pv + 2] + fy * (t[pv + 1] - t[pv + 2])}, p);
#pragma unroll
                                for (int e = 0; e < 2; ++e) {
                                    const int row = row0 + pv + e;
                                    if (pv + e <= K && (unsigned)row < (unsigned)CH) {
                                        lds_bf16 to = (lds_bf16)(uintptr_t)(gq + g_at(row, q >> 4));
#pragma unroll
                                        for (int k = 0; k < 3; ++k) to[k * (G_PLANE / 2)] = p[k][e];
                                    }
                                }
                            }
                        }
                    }
                }
                __syncthreads();
                BT(3);
                if (wave_on) {
                    // d f1 += G^T x f2 rows, 32 points at a time.  A operand: 16 ranks x 8 consecutive points per lane group
                    // through the transposing read (lane i of 16 addresses 4 ranks of point i / 4, twice).
                    Split3 bf[NTW];
                    auto split_b = [&]() {
#pragma unroll
                        for (int nt = 0; nt < NTW; ++nt) {
                            float f[8];
#pragma unroll
                            for (int i = 0; i < 8; ++i) { const unsigned w = x[i][nt]; f[i] = __uint_as_float(w); }
                            bf[nt] = split8(f);
                        }
                    };
                    load_b(0);
                    split_b();
#pragma unroll 1
                    for (int ks = 0; ks < nks; ++ks) {
                        load_b(min(ks + 1, nks - 1));            // always: a load that may not be issued would be waited for early
                        const unsigned on = reached(r0 + 32 * ks, 32);
                        // rows past the pass (the last run is half a one) meet zeros of f2: any finite row will do
                        const int ra = min(32 * ks + 8 * lg, CH - 8) + (lr >> 2);
                        // blocks are 32-byte parts of an aligned 256 bytes: the swizzle is one exclusive or
                        const unsigned ga0 = lds0 + (unsigned)(I_G + ra * G_ROW + 8 * (lr & 3)) + ((unsigned)(lr >> 2) << 5);
                        const unsigned ga1 = lds0 + (unsigned)(I_G + (ra + 4) * G_ROW + 8 * (lr & 3)) + ((unsigned)(4 + (lr >> 2)) << 5);
#pragma unroll
                        for (int t = 0; t < QT; ++t) {
                            if (on >> t & 1u) {
                                Split3 af;
#pragma unroll
                                for (int k = 0; k < 3; ++k) {
                                    const s16x4 u0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)((ga0 ^ (unsigned)(t << 5)) + k * G_PLANE));
                                    const s16x4 u1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)((ga1 ^ (unsigned)(t << 5)) + k * G_PLANE));
                                    const bf16x4 v0 = __builtin_bit_cast(bf16x4, u0), v1 = __builtin_bit_cast(bf16x4, u1);
                                    af.p[k] = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
                                }
#pragma unroll
                                for (int nt = 0; nt < NTW; ++nt) acc1[t][nt] = mma6(af, bf[nt], acc1[t][nt]);
                            }
                        }
                        split_b();
                    }
                }
                BT(4);
                // the next level's tap gradients start to move under the second contraction of this level's last
                // pass (every wave is past the pass's scatter, the last reader of the current ones)
                if (r0 + CH >= npts && l + 1 < lv_hi) load_taps(l + 1);
                if (wave_on) {
                    // d f2_l rows of this pass = G x f1, 16 points at a time, then out through atomics
                    const int ntile = (rows + 15) >> 4;
                    const unsigned sw = (unsigned)(lr & 7);
#pragma unroll 1
                    for (int m = 0; m < ntile; ++m) {
                        const unsigned on = reached(r0 + 16 * m, 16);
                        if (on == 0) continue;
                        const unsigned ga = lds0 + (unsigned)(I_G + (16 * m + lr) * G_ROW + (lg & 1) * 16) + (((unsigned)(lg >> 1) ^ sw) << 5);
                        f32x4 acc2[NTW];
#pragma unroll
                        for (int nt = 0; nt < NTW; ++nt) acc2[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int s = 0; s < QT / 2; ++s) {
                            if (on >> (2 * s) & 3u) {
                                Split3 af;
#pragma unroll
                                for (int k = 0; k < 3; ++k)
                                    af.p[k] = __builtin_bit_cast(bf16x8, *(lds_u32x4)(uintptr_t)((ga ^ (unsigned)(s << 6)) + k * G_PLANE));
#pragma unroll
                                for (int nt = 0; nt < NTW; ++nt) acc2[nt] = mma6(af, f1f[s][nt], acc2[nt]);
                            }
                        }
                        if constexpr (NTW == 2) {
                            // lane groups 2g and 2g + 1 hold 16 channels each of different points: they swap a tile, so that one
                            // atomic covers 128 bytes of each of two rows (a whole line) instead of 64 of each of four
                            const u32x4 off0 = *reinterpret_cast<const u32x4*>(rowoff + 16 * m + 4 * (lg & 2));
                            const u32x4 off1 = *reinterpret_cast<const u32x4*>(rowoff + 16 * m + 4 * (lg & 2) + 4);
                            const unsigned c4 = (unsigned)(cg + wave * 32 + 16 * (lg & 1) + lr) * 4u;
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const auto two = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc2[0][e]), __float_as_uint(acc2[1][e]), false, false);
                                __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(__uint_as_float(two[0]), r_d2, (int)(off0[e] + c4), 0, 0);
                                __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(__uint_as_float(two[1]), r_d2, (int)(off1[e] + c4), 0, 0);
                            }
                        } else {
                            const u32x4 off = *reinterpret_cast<const u32x4*>(rowoff + 16 * m + 4 * lg);
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(acc2[0][e], r_d2, (int)(off[e] + ch4), 0, 0);
                        }
                    }
                }
                BT(5);
            }
        }
        if (wave_on) {
#pragma unroll
            for (int t = 0; t < QT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const unsigned off = q_off[16 * t + 4 * lg + e] + ca4;
                    if constexpr (NTW == 2)
                        __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(acc1[t][0][e]), __float_as_uint(acc1[t][1][e])}, r_d1, (int)off, 0, 0);
                    else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc1[t][0][e]), r_d1, (int)off, 0, 0);
                }
        }
    }
    // a prefetch for a level that turned out to be all padding may still be in flight: nothing may land in LDS after the end
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#ifdef CORR_TRACE
    BT(6);
    if (tid == 0 && a.trace) { for (int i = 0; i < 7; ++i) a.trace[(size_t)k * 8 + i] = tacc[i]; a.trace[(size_t)k * 8 + 7] = tiles; }
#endif
}

// One workgroup per compute unit, each taking items from a queue until it is empty.  Workgroup w runs on XCD
// w % 8 and serves that XCD's share of the item list in list order (runs of CORR_XCD_RUN consecutive items, as in
// the forward kernel: neighbouring cells share window rows, so they should share an L2 and run at about the same
// time); a workgroup whose queue has run out goes on with the next XCD's.  So no compute unit spends time on
// workgroups that find nothing to do (one of this kernel's workgroups needs most of a unit's LDS, so even an empty
// one waits for a unit of its own), and the end of the launch is shared out item by item.  Handing out the full
// items first and the small ones last was measured too: it costs more in L2 misses than it gains at the end.
__global__ __launch_bounds__(NTI, 2) void bwd_item_kernel(BwdItemArgs a) {
    extern __shared__ __align__(256) unsigned char smem[];
    int& s_next = *reinterpret_cast<int*>(smem + I_NEXT);
    int xcd = (int)blockIdx.x & 7, tried = 0;
    const int n_items = *a.n_items;
    const int share = (n_items + 8 * CORR_XCD_RUN - 1) / (8 * CORR_XCD_RUN) * CORR_XCD_RUN;   // item positions per queue
    for (;;) {
        __syncthreads();                                   // the previous item's last LDS reads; s_next has been read
        if (threadIdx.x == 0) s_next = atomicAdd(a.queue + xcd, 1);
        __syncthreads();
        const int pos = s_next;                            // uniform
        if (pos >= share * a.parts) {                  // this queue is empty: help the next XCD's, until all eight are
            if (++tried == 8) break;
            xcd = (xcd + 1) & 7;
            continue;
        }
        // with parts > 1 consecutive positions are the levels of one item
        const int part = pos % a.parts, ipos = pos / a.parts;
        const int k = corr_item_of_workgroup(ipos * 8 + xcd);
        if (k >= n_items) continue;
        const int4 item = a.items[k];
        // parts = L: one level each; parts = 2 (and L > 2): level 0, and the rest
        const int lv_lo = a.parts > 1 ? part : 0;
        const int lv_hi = a.parts == 1 || (a.parts == 2 && part == 1) ? a.L : part + 1;
        if (a.D <= 128) {
            if (a.r == CORR_R) bwd_item_body<MAXK, 1>(a, smem, item, k, lv_lo, lv_hi, part);
            else bwd_item_body<0, 1>(a, smem, item, k, lv_lo, lv_hi, part);
        } else {
            if (a.r == CORR_R) bwd_item_body<MAXK, 2>(a, smem, item, k, lv_lo, lv_hi, part);
            else bwd_item_body<0, 2>(a, smem, item, k, lv_lo, lv_hi, part);
        }
    }
}

// Channels-last gradients to NCHW, and for fmap2 the levels' gradients down the pyramid in the same pass.
// Adjoint of the 2x2 mean: a pixel of level l - 1 receives a quarter of its parent's gradient at level l, if it
// has a parent (a trailing odd row or column that the pooling dropped has none, and then none at the deeper
// levels either).  For a level-0 pixel that is the nested sum d0 + (d1 + (d2 + d3 / 4) / 4) / 4 along its chain
// of parents, evaluated from the deepest level.  With L = 1 this is a plain transposition (d_fmap1).
// A workgroup moves 64 pixels x 64 channels through LDS: 16-byte loads along the channels (a wave reads four
// pixels' 256 bytes), 256-byte runs along the pixels on the way out.
struct GatherOne {
    const float* d[CORR_MAX_L];
    float* dst;
    int L;                      // levels to fold (1: a plain transposition)
    int parts;                  // d[0] is the sum of this many arrays, part_stride floats apart (d_fmap1 of a small input)
    size_t part_stride;
};
struct GatherArgs {
    GatherOne out[2];           // blockIdx.z = which * B + batch item; 0: d_fmap1, 1: d_fmap2
    int Hl[CORR_MAX_L], Wl[CORR_MAX_L];
    int B, D, W, HW;
    // for what the item form left not finite (set for that form only)
    bool mend;
    int r, L;
    float scale;
    CellGrid grid;
    const float *f1, *f2[CORR_MAX_L], *coords, *d_out;
    const int *bin_off, *n_items, *perm;
    const float2* sorted_c;
};
// An infinity, a NaN or a value beyond bf16's range (3.39e38) has no three bf16 parts: the item form's contractions make NaN of it,
// and 0 * NaN carries that over the whole window, into sums whose footprints hold nothing of the kind.  So what comes out not finite is
// summed again here over the footprints alone, in fp32, by the wave that found it.  Where there is nothing to mend that costs the
// check (the call on 270 x 480, D = 256: 1.23 ms with and without); detected in the item kernel instead, by its operands or by
// its sums, it cost that kernel 2 to 10 us a call.  The same call with one pixel of each map NaN takes 86 ms, everything NaN 33: a
// level 3 point is the sum over 6400 queries.
//
// A wave's 64 lanes are 16 channels x 4 rows at a time.  s += weight * row for the lanes' rows (`hit`: the lane has one), row numbers
// and weights one per lane
__device__ __forceinline__ float add_rows(float s, const float* rows, int D, int ch, bool hit, float weight, int row) {
    if (!__any(hit)) return s;
    const float* from = rows + min(ch, D - 1);
    row = hit ? row : -1;
#pragma unroll
    for (int i = 0; i < 64; i += 4) {                      // all loads in flight
        const int lane = i + ((threadIdx.x & 63) >> 4), r = __shfl(row, lane);
        const float w = __shfl(weight, lane), v = from[(size_t)max(r, 0) * D];
        s = r >= 0 ? fmaf(w, v, s) : s;
    }
    return s;
}
__device__ __forceinline__ float add_groups(float s) {
    s += __shfl_xor(s, 16);
    return s + __shfl_xor(s, 32);
}
// d_fmap1 of query p, channel ch
__device__ __forceinline__ float query_again(const GatherArgs& g, int b, int p, int ch) {
    const int lane = threadIdx.x & 63, K = 2 * g.r + 1, points = (K + 1) * (K + 1);
    const float cx = g.coords[((size_t)b * 2 + 0) * g.HW + p], cy = g.coords[((size_t)b * 2 + 1) * g.HW + p];
    float s = 0.f;
    if (!(fabsf(cx) <= CORR_COORD_LIMIT && fabsf(cy) <= CORR_COORD_LIMIT)) return s;     // uniform
    for (int l = 0; l < g.L; ++l) {
        const float inv = __uint_as_float((uint32_t)(127 - l) << 23);
        const float cxl = cx * inv, cyl = cy * inv, flx = floorf(cxl), fly = floorf(cyl);
        const float* taps = g.d_out + (size_t)(b * g.L + l) * K * K * g.HW + p;
        for (int i0 = 0; i0 < points; i0 += 64) {
            const int i = i0 + lane, pu = i / (K + 1), pv = i - pu * (K + 1), x = (int)flx - g.r + pu, y = (int)fly - g.r + pv;
            const bool hit = i < points && x >= 0 && x < g.Wl[l] && y >= 0 && y < g.Hl[l];
            const float w = hit ? footprint_weight(taps, g.HW, K, pu, pv, cxl - flx, cyl - fly) * g.scale : 0.f;
            s = add_rows(s, g.f2[l], g.D, ch, hit, w, hit ? (b * g.Hl[l] + y) * g.Wl[l] + x : 0);
        }
    }
    return add_groups(s);
}
// gradient of point (x, y) of level l, channel ch: over the queries whose footprints hold it, from the cells their targets can lie in
__device__ __forceinline__ float point_again(const GatherArgs& g, int b, int l, int y, int x, int ch) {
    const int lane = threadIdx.x & 63, K = 2 * g.r + 1;
    const float inv = __uint_as_float((uint32_t)(127 - l) << 23);
    // floor(target) >> l is in x - r - 1 .. x + r
    const int u0 = max(((x - g.r - 1) * (1 << l)) >> CORR_LOG_CX, g.grid.u_min) - g.grid.u_min;
    const int v0 = max(((y - g.r - 1) * (1 << l)) >> CORR_LOG_CY, g.grid.v_min) - g.grid.v_min;
    const int u1 = min((((x + g.r + 1) * (1 << l) - 1) >> CORR_LOG_CX) - g.grid.u_min, g.grid.nbx - 1);
    const int v1 = min((((y + g.r + 1) * (1 << l) - 1) >> CORR_LOG_CY) - g.grid.v_min, g.grid.nby - 1);
    const int last = g.B * CORR_TILE_CELLS * g.grid.tnx * g.grid.tny - 1;
    const float* taps = g.d_out + (size_t)(b * g.L + l) * K * K * g.HW;
    float s = 0.f;
    for (int v = v0; v <= v1; ++v)
        for (int u = u0; u <= u1; ++u) {
            const int cell = corr_cell_id(g.grid, b, u, v);
            const int begin = g.bin_off[cell * CORR_SUB], end = cell < last ? g.bin_off[(cell + 1) * CORR_SUB] : g.n_items[1];
            for (int i0 = begin; i0 < end; i0 += 64) {
                const int i = min(i0 + lane, end - 1);
                const float2 c = g.sorted_c[i];
                const float cxl = c.x * inv, cyl = c.y * inv, flx = floorf(cxl), fly = floorf(cyl);
                const int pu = x - ((int)flx - g.r), pv = y - ((int)fly - g.r);
                const bool hit = i0 + lane < end && (unsigned)pu <= (unsigned)K && (unsigned)pv <= (unsigned)K;
                const int q = g.perm[i];                           // of the whole batch
                const float w = hit ? footprint_weight(taps + (q - b * g.HW), g.HW, K, pu, pv, cxl - flx, cyl - fly) * g.scale : 0.f;
                s = add_rows(s, g.f1, g.D, ch, hit, w, q);
            }
            if (__all(s != s || ch >= g.D)) return s;              // NaN for good
        }
    return add_groups(s);
}
// Bound by the traffic (270 x 480, D = 256: 119 us), which takes all eight waves a SIMD can hold: with seven, for the scalar registers
// of the mending, it took 136.
constexpr int TP = 64, TC = 64;
__global__ __launch_bounds__(256, 8) void bwd_gather_nchw_kernel(GatherArgs g) {
    __shared__ float tile[TC][TP + 1];
    const int which = (int)blockIdx.z / g.B, b = (int)blockIdx.z - which * g.B;
    const GatherOne& o = g.out[which];
    const int p0 = blockIdx.x * TP, d0 = blockIdx.y * TC;
#pragma unroll
    for (int k = 0; k < TP * TC / 4 / 256; ++k) {
        const int idx = threadIdx.x + 256 * k, c4 = idx & (TC / 4 - 1), pr = idx / (TC / 4);
        const int p = p0 + pr, ch = d0 + 4 * c4;
        if (p < g.HW && ch < g.D) {                        // D is a multiple of 4
            const int y = p / g.W, x = p - y * g.W;
            float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int l = o.L - 1; l >= 1; --l) {
                const int yy = y >> l, xx = x >> l;
                if (yy < g.Hl[l] && xx < g.Wl[l]) {
                    const float4 v = *reinterpret_cast<const float4*>(o.d[l] + (((size_t)b * g.Hl[l] + yy) * g.Wl[l] + xx) * g.D + ch);
                    t = make_float4(v.x + 0.25f * t.x, v.y + 0.25f * t.y, v.z + 0.25f * t.z, v.w + 0.25f * t.w);
                }
            }
            const float* src = o.d[0] + ((size_t)b * g.HW + p) * g.D + ch;
            float4 v = *reinterpret_cast<const float4*>(src);
            for (int part = 1; part < o.parts; ++part) {
                const float4 w = *reinterpret_cast<const float4*>(src + part * o.part_stride);
                v = make_float4(v.x + w.x, v.y + w.y, v.z + w.z, v.w + w.w);
            }
            tile[4 * c4 + 0][pr] = v.x + 0.25f * t.x;
            tile[4 * c4 + 1][pr] = v.y + 0.25f * t.y;
            tile[4 * c4 + 2][pr] = v.z + 0.25f * t.z;
            tile[4 * c4 + 3][pr] = v.w + 0.25f * t.w;
        }
    }
    __syncthreads();
    float sum = 0.f;                                       // not finite if any element is not
#pragma unroll
    for (int k = 0; k < TP * TC / 256; ++k) {
        const int idx = threadIdx.x + 256 * k, px = idx & (TP - 1), chn = idx / TP;
        if (d0 + chn < g.D && p0 + px < g.HW) {
            const float v = tile[chn][px];
            o.dst[((size_t)b * g.D + d0 + chn) * g.HW + p0 + px] = v;
            sum += v;
        }
    }
    if (!g.mend || !__any(!(fabsf(sum) < INFINITY))) return;
    // the wave's channels of the tile: d0 + wave + 4 * i
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, chn = wave + 4 * (lane & 15), ch = d0 + chn;
    bool spoiled = false;
    for (int i = 0; i < TC / 4; ++i)
        spoiled |= p0 + lane < g.HW && d0 + wave + 4 * i < g.D && !(fabsf(tile[wave + 4 * i][lane]) < INFINITY);
    const uint64_t pixels = __ballot(spoiled);
    auto write = [&](int p, float v) {                     // what was finite stays
        if (lane < 16 && ch < g.D && !(fabsf(tile[chn][p - p0]) < INFINITY)) o.dst[((size_t)b * g.D + ch) * g.HW + p] = v;
    };
    if (which == 0) {
        for (uint64_t left = pixels; left; left &= left - 1) {
            const int p = p0 + __builtin_ctzll(left);
            write(p, query_again(g, b, p, ch));
        }
        return;
    }
    // the levels' gradients first, in place (a wave of another tile that needs the same point writes the same value), then the fold again
    for (int l = 0; l < o.L; ++l)
        for (uint64_t left = pixels; left; left &= left - 1) {
            const int p = p0 + __builtin_ctzll(left), y = p / g.W >> l, x = p % g.W >> l;
            if (y >= g.Hl[l] || x >= g.Wl[l]) continue;
            float* d = const_cast<float*>(o.d[l]) + (((size_t)b * g.Hl[l] + y) * g.Wl[l] + x) * g.D + ch;
            const bool bad = ch < g.D && !(fabsf(__hip_atomic_load(d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < INFINITY);
            if (!__any(bad)) continue;
            const float v = point_again(g, b, l, y, x, ch);
            if (bad && lane < 16) __hip_atomic_store(d, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __threadfence_block();                         // the next pixel may have the same point
        }
    for (uint64_t left = pixels; left; left &= left - 1) {
        const int p = p0 + __builtin_ctzll(left), y = p / g.W, x = p % g.W;
        float v = 0.f;
        for (int l = o.L - 1; l >= 0; --l)
            if ((y >> l) < g.Hl[l] && (x >> l) < g.Wl[l] && ch < g.D)
                v = __hip_atomic_load(o.d[l] + (((size_t)b * g.Hl[l] + (y >> l)) * g.Wl[l] + (x >> l)) * g.D + ch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 0.25f * v;
        write(p, v);
    }
}

}  // namespace

// Small inputs run an item's levels in workgroups of their own (a map of a few thousand queries has fewer items
// than the chip has compute units, and the call's time is one item's latency); each level then adds into a d f1
// array of its own and the final gather sums them in level order, so the result stays the same bits on every call.
#ifndef CORR_BACKWARD_SPLIT_MAX_QUERIES
#define CORR_BACKWARD_SPLIT_MAX_QUERIES 32000   // measured: the split gains up to about 28000 queries and costs 8 % at 45000
#endif
#ifndef CORR_BACKWARD_HALVE_MAX_QUERIES
#define CORR_BACKWARD_HALVE_MAX_QUERIES 40000   // up to here an item is two pieces: level 0 (three passes) and the other levels (four); measured: -7 % at 32400 queries, nothing from 45000 on
#endif
static int backward_parts(int B, int H, int W, int L) {
    const long long BN = (long long)B * H * W;
    return BN <= CORR_BACKWARD_SPLIT_MAX_QUERIES ? L : (BN <= CORR_BACKWARD_HALVE_MAX_QUERIES && L > 1) ? 2 : 1;
}
size_t corr_backward_workspace_floats(int B, int H, int W, int D, int L) {
    size_t px = 0;
    for (int l = 0; l < L; ++l) px += (size_t)(H >> l) * (W >> l);
    return ((size_t)backward_parts(B, H, W, L) * B * H * W + (size_t)B * px) * D;
}

// gradient arrays (rounded up to 256 bytes), then a planning workspace like the pyramid's (the call bins the
// queries itself and leaves the pyramid's own workspace alone)
static size_t grad_bytes(int B, int H, int W, int D, int L) {
    return (corr_backward_workspace_floats(B, H, W, D, L) * sizeof(float) + 255) & ~(size_t)255;
}
size_t corr_backward_workspace_bytes_internal(int B, int H, int W, int D, int L) {
    CellGrid g;
    corr_fill_grid(&g, H, W, L);
    return grad_bytes(B, H, W, D, L) + corr_ws_layout(B * H * W, corr_ncells(g, B)).total;
}

#ifdef CORR_TRACE
static long long* g_bwd_trace = nullptr;
extern "C" void corr_debug_set_backward_trace(long long* p) { g_bwd_trace = p; }
#endif
hipError_t launch_backward(const corr_pyramid* p, const float* coords, const float* d_out, int r,
                           float* d_fmap1, float* d_fmap2, float* ws, int form, int split_max, hipStream_t s) {
    const int HW = p->H * p->W;
    float* cur = ws;
    // the test hook can switch the splitting of levels off (a setting of 0; the workspace is laid out for the default)
    const bool split = split_max != 0;
    const int parts = form == CORR_BACKWARD_ITEMS && split ? backward_parts(p->B, p->H, p->W, p->L) : 1;
    float* d_f1 = cur; cur += (size_t)backward_parts(p->B, p->H, p->W, p->L) * p->B * HW * p->D;
    float* d_f2[CORR_MAX_L] = {nullptr, nullptr, nullptr, nullptr};
    size_t lev_floats = 0;
    for (int l = 0; l < p->L; ++l) {
        d_f2[l] = cur;
        const size_t n = (size_t)p->B * p->Hl[l] * p->Wl[l] * p->D;
        cur += n; lev_floats += n;
    }
    const float scale = 1.0f / sqrtf((float)p->D);
    const long long BN = (long long)p->B * HW;
    hipError_t e;
    GatherArgs ga{};
    if (form == CORR_BACKWARD_ITEMS) {
        // Everything accumulates or keeps its zero; in the planning workspace the bin counters, the item counters and
        // the item kernel's queues (kept in the statistics slots) start at zero, the rest is written before it is
        // read.  Fill kernels, so the call can be graph-captured.  A small input's whole workspace is cleared in one
        // launch: there the call's time is launches and one item's latency.
        const size_t gbytes = grad_bytes(p->B, p->H, p->W, p->D, p->L);
        const int ncells = corr_ncells(p->grid, p->B);
        const BinWs bws = corr_ws_carve(reinterpret_cast<char*>(ws) + gbytes, (int)BN, ncells);
        if (backward_parts(p->B, p->H, p->W, p->L) > 1) {
            const size_t all = gbytes + corr_ws_layout((int)BN, ncells).total;
            if ((e = launch_fill_i32(reinterpret_cast<int*>(ws), 0, all / 4, s)) != hipSuccess) return e;
        } else {
            if ((e = launch_fill_i32(reinterpret_cast<int*>(ws), 0, (size_t)(cur - ws), s)) != hipSuccess) return e;
            if ((e = launch_fill_i32(bws.bin_count, 0, (size_t)bws.nbins, s)) != hipSuccess) return e;
            // item counters and, right behind them, the statistics slots
            const size_t tail = (size_t)(reinterpret_cast<int*>(bws.stats) + 2 * CORR_NSTATS - bws.n_items);
            if ((e = launch_fill_i32(bws.n_items, 0, tail, s)) != hipSuccess) return e;
        }
        LookupArgs q{coords, nullptr, r, 0, 0, 0};
        if ((e = launch_binning(p, bws, q, s)) != hipSuccess) return e;
        static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(bwd_item_kernel),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, ITEM_LDS);
        if (attr != hipSuccess) return attr;
        BwdItemArgs a;
#ifdef CORR_TRACE
        a.trace = g_bwd_trace;
#endif
        a.f1 = p->f1_nhwc; a.d_f1 = d_f1; a.d_out = d_out;
        a.perm = bws.perm; a.sorted_c = bws.sorted_c; a.items = bws.items; a.n_items = bws.n_items; a.queue = reinterpret_cast<int*>(bws.stats); a.parts = parts;
        a.B = p->B; a.HW = HW; a.D = p->D; a.L = p->L; a.r = r; a.g = p->grid; a.scale = scale;
        for (int l = 0; l < CORR_MAX_L; ++l) {
            a.f2[l] = l < p->L ? p->f2_nhwc[l] : nullptr; a.d_f2[l] = d_f2[l];
            a.Hl[l] = p->Hl[l]; a.Wl[l] = p->Wl[l];
        }
        ga.mend = true;
        ga.bin_off = bws.bin_off; ga.n_items = bws.n_items; ga.perm = bws.perm; ga.sorted_c = bws.sorted_c;
        hipLaunchKernelGGL(bwd_item_kernel, dim3(CORR_NUM_CU), dim3(NTI), ITEM_LDS, s, a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else {
        BwdArgs a;
        a.f1 = p->f1_nhwc; a.coords = coords; a.d_out = d_out;
        a.B = p->B; a.HW = HW; a.D = p->D; a.L = p->L; a.r = r; a.scale = scale;
        a.d_f1 = d_f1;
        for (int l = 0; l < CORR_MAX_L; ++l) {
            a.f2[l] = l < p->L ? p->f2_nhwc[l] : nullptr; a.d_f2[l] = d_f2[l];
            a.Hl[l] = p->Hl[l]; a.Wl[l] = p->Wl[l];
        }
        if ((e = launch_fill_i32(reinterpret_cast<int*>(d_f2[0]), 0, lev_floats, s)) != hipSuccess) return e;
        hipLaunchKernelGGL(bwd_query_kernel, dim3((unsigned)((BN + BQ - 1) / BQ)), dim3(64 * BQ), 0, s, a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // both gradients to NCHW in one launch: d_fmap1 (a small input's per-level shares summed), d_fmap2 (levels folded)
    for (int l = 0; l < CORR_MAX_L; ++l) {
        ga.Hl[l] = p->Hl[l]; ga.Wl[l] = p->Wl[l];
        ga.out[0].d[l] = nullptr; ga.out[1].d[l] = d_f2[l];
    }
    ga.out[0].d[0] = d_f1; ga.out[0].dst = d_fmap1; ga.out[0].L = 1;
    ga.out[0].parts = parts; ga.out[0].part_stride = (size_t)p->B * HW * p->D;
    ga.out[1].dst = d_fmap2; ga.out[1].L = p->L; ga.out[1].parts = 1; ga.out[1].part_stride = 0;
    ga.B = p->B; ga.D = p->D; ga.W = p->W; ga.HW = HW;
    ga.r = r; ga.L = p->L; ga.scale = scale; ga.grid = p->grid; ga.f1 = p->f1_nhwc; ga.coords = coords; ga.d_out = d_out;
    for (int l = 0; l < CORR_MAX_L; ++l) ga.f2[l] = l < p->L ? p->f2_nhwc[l] : nullptr;
    hipLaunchKernelGGL(bwd_gather_nchw_kernel, dim3((HW + TP - 1) / TP, (p->D + TC - 1) / TC, 2 * p->B), dim3(256), 0, s, ga);
    return hipGetLastError();
}
