// smol_jpeg_kernels.hip -- the GPU part of partial JPEG decoding (section 6.4, "ROI
// decoding"): dequantisation and the 8 x 8 inverse DCT of the blocks of a
// 4:2:0 frame that meet a rectangle, written to I420 planes. The entropy
// decoding that produces the coefficients is the CPU decoder's.
//
// Each 1-D transform x(n) = sum_k c(k, n) D(k) is evaluated through the parity
// of the cosine basis, c(k, 7 - n) = (-1)^k c(k, n): for n < 4 the
// even-frequency sum E and the odd-frequency sum O (each in increasing
// frequency), then x(n) = E + O and x(7 - n) = E - O (T.81 A.3.3 evaluated
// separably), each product and sum rounded on its own (no contraction). Every
// c(k, n) is one of seven magnitudes with a sign (c(2, 3) = -c(2, 0), and so
// on), so the even frequencies need 6 products for the four E instead of 16:
// the products are the same numbers up to an exact negation.
//
// A job is the rectangle's blocks among sixteen adjacent ones of a block row
// (aligned to sixteen in the plane), decoded by one wave in two halves of
// eight. Pass 1: lane l loads coefficient row v = l % 8
// of block b = l / 8 (16 contiguous bytes) and forms G(v, x) for all x. After an
// exchange through LDS, pass 2: lane l forms column x = l % 8 of block b, adds
// 128, clamps to [0, 255] and rounds to nearest even. The bytes of the sixteen
// blocks go through LDS once more, so that a lane stores 16 bytes of a picture
// row and eight lanes 128, a whole line of the plane where its rows are.
//
// Bound by memory: the rectangles of 128 720p frames are 157 MB of coefficients
// and 81 MB of pixels, 47 us at a large copy's 5.05 TB/s. 59.5 us with one
// group of eight per job, 4-byte stores of 64-byte row pieces and every
// output's products formed on their own (194 vector and 110 scalar instructions
// per group), 48 us now (170 and 84); with nontemporal coefficient loads
// the planes stay cached for the preprocessing that reads them next (2 us of
// the pair of launches; nontemporal stores cost it 1.5).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "smol_internal.h"

namespace smol {
namespace {

constexpr int kBlocksPerWave = 8;
// LDS words of a block's G: eight more than its 64, so that the columns of the
// eight blocks read together (pass 2) lie in different banks.
constexpr int kBlockWords = 72;

// x = the 1-D transform of d; c[k] = C(k)/2 cos(k pi / 16).
__device__ __forceinline__ void idct8(const float (&c)[8], const float (&d)[8], float (&x)[8])
{
    const float p0 = c[0] * d[0], p4 = c[4] * d[4];
    const float a2 = c[2] * d[2], b2 = c[6] * d[2], a6 = c[6] * d[6], b6 = c[2] * d[6];
    const float e[4] = {((p0 + a2) + p4) + a6, ((p0 + b2) - p4) - b6, ((p0 - b2) - p4) + b6,
                        ((p0 - a2) + p4) - a6};
    const float o[4] = {((c[1] * d[1] + c[3] * d[3]) + c[5] * d[5]) + c[7] * d[7],
                        ((c[3] * d[1] - c[7] * d[3]) - c[1] * d[5]) - c[5] * d[7],
                        ((c[5] * d[1] - c[1] * d[3]) + c[7] * d[5]) + c[3] * d[7],
                        ((c[7] * d[1] - c[5] * d[3]) + c[3] * d[5]) - c[1] * d[7]};
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        x[n] = e[n] + o[n];
        x[7 - n] = e[n] - o[n];
    }
}

// The 32-bit word at a 4-byte aligned field, and its two 16-bit halves.
__device__ __forceinline__ uint32_t word_of(const int16_t *p)
{
    uint32_t w;
    __builtin_memcpy(&w, p, 4);
    return w;
}
__device__ __forceinline__ int lo16(uint32_t w) { return (int)(int16_t)(w & 0xffffu); }
__device__ __forceinline__ int hi16(uint32_t w) { return (int)(int16_t)(w >> 16); }

// floor(n / d) from the run's m = ceil(2^s / d) (exact for n < 2^31)
__device__ __forceinline__ uint32_t magic_div(uint32_t n, uint32_t m, uint32_t s)
{
    return (uint32_t)(((uint64_t)n * m) >> s);
}

__global__ void __launch_bounds__(64) jpeg_idct_kernel(JpegArgs a)
{
    // G(v, x) of block b at word b * kBlockWords + 8 v + x; pixel (y, x) of the
    // sixteen blocks' 8 x 128 at byte 128 y + x
    __shared__ __attribute__((aligned(16))) float g[kBlocksPerWave * kBlockWords];
    __shared__ __attribute__((aligned(16))) uint8_t pix[2 * kBlocksPerWave * 64];
    const int l = threadIdx.x;
    const int b = l >> 3, row = l & 7;  // block of the group; row v (pass 1), column x (pass 2)
    float c[8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
        c[k] = a.c[k];
    // job indices stay below 2^31 (the host splits launches), so the job
    // mapping runs in 32-bit unsigned arithmetic, its divisions by the run's
    // divisors as multiplications (JpegRun)
    const uint32_t jobs = a.run[a.runs - 1].jobs_end;
    int ri = 0;  // run of the current job (jobs ascend within a workgroup)
    for (uint32_t job = blockIdx.x; job < jobs; job += gridDim.x) {
        while (a.run[ri].jobs_end <= job)
            ++ri;
        const JpegRun &r = a.run[ri];
        // jobs along each block row of the rectangle
        const uint32_t lg = r.jobs_row & 0xffffu, cg = r.jobs_row >> 16;
        const uint32_t lum = r.lum, chr = r.chr, per_frame = lum + 2 * chr;
        const uint32_t local = job - (ri ? a.run[ri - 1].jobs_end : 0);
        const uint32_t f = magic_div(local, r.m_pf, r.shifts & 0xffu);
        uint32_t k = local - f * per_frame;
        // the 16-bit fields in pairs, as the words that hold them (a 16-bit
        // field read alone becomes a vector load that the wave waits for)
        const uint32_t wxy = word_of(&r.wx0), wm = word_of(&r.wmx);
        int comp, by, bx0, nbx, gi, gw, ox, oy, pw, ph;  // (ox, oy): the stored grid's first block
        long long cbase, pbase;
        if (k < lum) {
            comp = 0;
            const uint32_t kr = magic_div(k, r.m_lg, (r.shifts >> 8) & 0xffu);
            const uint32_t lb = word_of(&r.lbx0);
            by = hi16(lb) + (int)kr;
            gi = (int)(k - kr * lg);
            bx0 = lo16(lb);
            nbx = lo16(word_of(&r.lnbx));
            gw = 2 * lo16(wm);
            ox = 2 * lo16(wxy);
            oy = 2 * hi16(wxy);
            cbase = 0;
            pbase = 0;
            pw = r.W;
            ph = r.H;
        } else {
            k -= lum;
            comp = k < chr ? 1 : 2;
            k -= comp == 1 ? 0 : chr;
            const uint32_t kr = magic_div(k, r.m_cg, (r.shifts >> 16) & 0xffu);
            const uint32_t cb = word_of(&r.cbx0);
            by = hi16(cb) + (int)kr;
            gi = (int)(k - kr * cg);
            bx0 = lo16(cb);
            nbx = lo16(word_of(&r.cnbx));
            gw = lo16(wm);
            ox = lo16(wxy);
            oy = hi16(wxy);
            cbase = 64LL * lo16(wm) * hi16(wm) * (comp == 1 ? 4 : 5);
            pbase = comp == 1 ? r.cboff : r.croff;
            pw = (r.W + 1) >> 1;
            ph = (r.H + 1) >> 1;
        }
        // the job's blocks: begin .. end - 1 of the plane's block row
        const int first = (bx0 / kJpegJobBlocks + gi) * kJpegJobBlocks;
        const int begin = max(bx0, first), end = min(bx0 + nbx, first + kJpegJobBlocks);
        const int16_t *blocks = a.coef + r.coef + f * r.coef_stride + cbase +
                                64LL * ((long long)(by - oy) * gw - ox);
        // the lane's 8 table entries
        const uint64_t q = *(const uint64_t *)&a.q[r.shifts >> 24][comp == 0 ? 0 : 1][8 * row];
        uint8_t *const plane = a.out + r.out + f * r.out_stride + pbase;
        typedef short short8 __attribute__((ext_vector_type(8)));
        // coefficient row of the lane's block in the eight from block b0 on;
        // lanes of blocks outside the job repeat one inside
        auto load = [&](int b0) {
            const short8 *p = (const short8 *)(
                blocks + (uint32_t)(64 * min(max(b0 + b, begin), end - 1) + 8 * row));
            return __builtin_nontemporal_load(p);  // read once: keeps the planes cached
        };
        const short8 raw[2] = {load(first), load(first + kBlocksPerWave)};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int b0 = first + h * kBlocksPerWave;
            if (b0 + kBlocksPerWave <= begin || b0 >= end)
                continue;  // none of these eight is in the job
            float d[8], x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                d[u] = (float)((int)raw[h][u] * (int)(uint8_t)(q >> (8 * u)));  // exact: < 2^24
            // horizontal pass for row v = row
            idct8(c, d, x);
            typedef float f32x4 __attribute__((ext_vector_type(4)));
            f32x4 *grow = (f32x4 *)&g[b * kBlockWords + 8 * row];
            grow[0] = f32x4{x[0], x[1], x[2], x[3]};
            grow[1] = f32x4{x[4], x[5], x[6], x[7]};
            __syncthreads();
            // vertical pass for column x = row
#pragma unroll
            for (int v = 0; v < 8; ++v)
                d[v] = g[b * kBlockWords + 8 * v + row];
            idct8(c, d, x);
#pragma unroll
            for (int y = 0; y < 8; ++y)
                // clamped to [0, 255] and rounded to nearest even
                pix[128 * y + 64 * h + l] =
                    (uint8_t)__builtin_amdgcn_cvt_pk_u8_f32(x[y] + 128.0f, 0u, 0u);
            __syncthreads();
        }
        // lane l stores 16 bytes of row l / 8 of the sixteen blocks
        const int gx = 8 * first + 16 * row, gy = 8 * by + b;
        const int x_end = min(8 * end, pw);
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        const u32x4 px = *(const u32x4 *)&pix[16 * l];
        if (gy < ph) {
            uint8_t *dst = plane + (uint32_t)gy * (uint32_t)pw;
            if (gx >= 8 * begin && gx + 16 <= x_end) {
                typedef uint32_t Unaligned __attribute__((ext_vector_type(4), aligned(1)));
                *(Unaligned *)(dst + (uint32_t)gx) = px;
            } else {
                for (int x = max(gx, 8 * begin); x < min(gx + 16, x_end); ++x)
                    dst[x] = pix[16 * l + x - gx];
            }
        }
        __syncthreads();
    }
}

}  // namespace

int launch_jpeg_idct(const JpegArgs &a, int grid, void *stream)
{
    hipLaunchKernelGGL(jpeg_idct_kernel, dim3((unsigned)grid), dim3(64), 0, (hipStream_t)stream,
                       a);
    return (int)hipGetLastError();
}

}  // namespace smol
