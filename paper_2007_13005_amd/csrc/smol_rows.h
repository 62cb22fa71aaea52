// smol_rows.h -- the pieces the row-streaming kernels (RGB in smol_rows_rgb.h,
// I420 in smol_rows_yuv.h) share: the row walk over waves, the vertical tap
// cursor, row staging and tap reads for RGB rows, normalisation, output
// packing and stores. Each smol_rows_*.hip file instantiates one part of the
// kernels (input, output type, row walk, output layout), so the parts build
// in parallel.
#pragma once

#include <limits.h>

#include "smol_device.h"

namespace smol {
namespace {

// ---------------------------------------------------------------------------
// RGB, row streaming: independent waves, no barriers.
//
// Work items are output rows (image, row), image-major. On the contiguous walk
// wave g takes the range [g*T/G, (g+1)*T/G) of the T rows; on the strided walk
// it takes rows q, q + G, q + 2G, ... (q: g remapped so the waves of one XCD
// take neighbouring rows), so the rows in flight on the chip at any moment
// form one band of the output. For each output row the wave loads the two
// source rows its vertical taps read -- only the crop's source column span, as
// the 16-byte chunks that hold it, aligned in the global address space, one
// coalesced 16-byte load per lane and 64 chunks -- into registers, one or two
// rows ahead of the row it interpolates, and writes a row's chunks into its
// LDS slot right after interpolating the previous row. The bytes in flight
// live in registers, so a compute unit keeps more loads outstanding than its
// LDS could stage, and the compiler orders each LDS write after exactly the
// loads it needs.
//
// A wide crop, or one whose source span is long, runs as column strips side by
// side (strip_start); a wave keeps to one strip.
//
// Only images whose chunks all lie inside src come here; the host sends the
// others to the direct kernel. Lanes past a row's last chunk load that chunk
// again (their copy lands past the row in the slot and is never read).
//
// The contiguous walk computes its rows' vertical taps 64 at a time, a row per
// lane (row_records); the strided walk steps the vertical half-pixel map with
// exact integer arithmetic (the numerator grows by a precomputed constant per
// step): no division per row but the one for the weight.
//
// Lane l computes J pairs of output columns (pair_col); their taps (byte
// offset in the staged span, weight) stay in registers while the horizontal
// geometry is unchanged. Each pixel's two horizontal taps are 6 bytes of a
// staged row, read as three aligned dwords and realigned.
//
// The three lerps are always evaluated as defined, every product and sum
// rounded on its own. EXACT selects the rest: 1 forms the normalisation as
// the correctly rounded quotient and rounds to fp16 from that fp32 value,
// bit-identical to a scalar fp32 evaluation of the definition; 0 multiplies
// the same difference v - mean by RN(1/std), at most one fp32 ulp from the
// quotient, and lets the fp16 conversion fuse with that product (fp16 output
// within one fp16 ulp of the definition's).
// ---------------------------------------------------------------------------
struct RowImg {
    long long off;
    int W, H, pitch, Wr, Hr, left, top, xf, span;
};

// The descriptor table is read-only for the whole launch: read it through the
// constant address space so the wave uses scalar loads, which do not count
// against (or wait for) the vector-memory counter.
typedef __attribute__((address_space(4))) const Desc ConstDesc;

// The first crop column of column strip `strip` of a launch: strips of
// a.strip_w columns side by side, the last one ending at the crop's last
// column (where it overlaps its neighbour, both store the same values).
__device__ __forceinline__ int strip_start(const BatchArgs &a, int strip)
{
    return min(strip * a.strip_w, a.Cw - a.strip_w);
}

__device__ __forceinline__ RowImg row_img(const BatchArgs &a, int img, int strip)
{
    RowImg g;
    if (a.table) {
        const ConstDesc *t = (const ConstDesc *)a.table + img;
        g.off = t->off[0];
        g.W = t->W;
        g.H = t->H;
        g.pitch = t->pitch;
        g.Wr = t->Wr;
        g.Hr = t->Hr;
        g.left = t->left;
        g.top = t->top;
        g.xf = t->xf;
        g.span = t->span;
    } else {
        g.off = a.uni.off[0] + (long long)img * a.stride;
        g.W = a.uni.W;
        g.H = a.uni.H;
        g.pitch = a.uni.pitch;
        g.Wr = a.uni.Wr;
        g.Hr = a.uni.Hr;
        g.left = a.uni.left;
        g.top = a.uni.top;
        g.xf = a.uni.xf;
        g.span = a.uni.span;
    }
    if (a.strips > 1) {
        // the strip's own columns of the crop and the source span they read
        g.left += strip_start(a, strip);
        g.xf = axis_tap(g.left, g.W, g.Wr).x0;
        g.span = 3 * (axis_tap(g.left + a.strip_w - 1, g.W, g.Wr).x1 - g.xf + 1);
    }
    return g;
}

// Column px of column pair j that lane `lane` computes. QUADS (J = 2): four
// consecutive columns from 4 lane on, so that a plane's store is 4 columns wide;
// else pair j is the columns from 2 lane + 128 j on, so that an interleaved
// (NHWC) row's stores of pair j lie side by side (fp32 pixels of four columns
// per lane, stored 48 bytes apart, took twice as long: 101 upscales 110 -> 224
// 48.8 against 21.6 us). Clamped so that the columns end at the strip's last
// (cols >= 2J, or cols = 1 with J = 1). Lanes past the strip thus compute and
// store columns that other lanes store as well, the same values to the same
// addresses: every lane runs the same stores, with no branch around them, and
// the compiler can count the memory operations in flight exactly (a branch that
// might skip the stores would make it wait for them before every write to LDS).
template <int J, bool QUADS>
__device__ __forceinline__ int pair_col(int lane, int j, int cols)
{
    return QUADS ? min(2 * J * lane, max(cols - 2 * J, 0)) + 2 * j
                 : min(2 * lane + 128 * j, max(cols - 2, 0));
}

// A column's floor quotient and remainder of num = (2 (left + c) + 1) W - Wr by
// den = 2 Wr (-den < num < 2^39; the double quotient's truncation is the exact
// floor: a non-integer quotient is at least 1 / den from the next integer).
__device__ __forceinline__ void col_divmod(const RowImg &g, int c, int den, int &q, int &rem)
{
    const long long num = (long long)(2 * (g.left + c) + 1) * g.W - g.Wr;
    q = num < 0               ? -1
        : num < 0x7fffffffLL ? (int)((unsigned)num / (unsigned)den)
                             : (int)((double)num / (double)den);
    rem = (int)(num - (long long)q * den);
}

// Column taps of a lane's columns: one division per run of consecutive columns
// and exact integer steps within it. The weight rem / den rounded to nearest
// fp32 comes from an fp64 product with RN(1 / den): the product is within 2^-52
// (relative) of the quotient, and no such quotient (0 < rem < den <= 2^24) lies
// within 2^-49 (relative) of a midpoint between fp32 values, so both round to
// the same fp32 value. (A tap computed on its own costs about 60 instructions,
// and a wave of a ragged batch walks only a dozen rows with them.)
template <int J, bool QUADS>
__device__ __forceinline__ void row_taps(const RowImg &g, const int cols, int (&cx)[J][2],
                                         float (&cw)[J][2], int lane)
{
    const int den = 2 * g.Wr;
    const double rcp = 1.0 / (double)den;
    // a crop of one column computes it twice
    const int step = cols > 1 ? 2 * g.W : 0;
    const int qs = step / den, rs = step - qs * den;
    int q, rem;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        if (j == 0 || !QUADS)
            col_divmod(g, pair_col<J, QUADS>(lane, j, cols), den, q, rem);
#pragma unroll
        for (int px = 0; px < 2; ++px) {
            const bool low = q < 0, high = q >= g.W - 1;
            cx[j][px] = 3 * ((low ? 0 : high ? g.W - 1 : q) - g.xf);
            cw[j][px] = low || high ? 0.0f : (float)((double)rem * rcp);
            q += qs;
            rem += rs;
            const bool carry = rem >= den;
            rem -= carry ? den : 0;
            q += carry ? 1 : 0;
        }
    }
}

// Pixels x0 (bytes 0..2) and x0 + 1 (bytes 3..5) of an 8-byte window, as
// a = value at x0 and d = (value at x0 + 1) - a per channel; d is an exact
// small integer, so a + w * d is the definition's a + w * (b - a).
#define SMOL_CVT_UBYTE(N)                                                                     \
    __device__ __forceinline__ float cvt_ubyte##N(uint32_t x)                                 \
    {                                                                                         \
        float f;                                                                              \
        asm("v_cvt_f32_ubyte" #N " %0, %1" : "=v"(f) : "v"(x));                               \
        return f;                                                                             \
    }
SMOL_CVT_UBYTE(0)
SMOL_CVT_UBYTE(1)
SMOL_CVT_UBYTE(2)
SMOL_CVT_UBYTE(3)
#undef SMOL_CVT_UBYTE

__device__ __forceinline__ void unpack_ad(uint64_t v, float (&a)[3], float (&d)[3])
{
    // One conversion per byte (the compiler's own selection extracts some
    // bytes with extra shifts first).
    const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    a[0] = cvt_ubyte0(lo);
    a[1] = cvt_ubyte1(lo);
    a[2] = cvt_ubyte2(lo);
    d[0] = cvt_ubyte3(lo) - a[0];  // exact: small integers
    d[1] = cvt_ubyte0(hi) - a[1];
    d[2] = cvt_ubyte1(hi) - a[2];
}

// a + w * d with the product and the sum rounded on their own.
__device__ __forceinline__ float lerp_ad(float a, float d, float w) { return a + w * d; }

// Normalisation constants of the three channels.
struct NormK {
    float mean[3], stdv[3], rcp[3];
};

__device__ __forceinline__ NormK norm_consts(const BatchArgs &a)
{
    NormK k;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        k.mean[ch] = a.mean[ch];
        k.stdv[ch] = a.stdv[ch];
        k.rcp[ch] = a.rcp[ch];
    }
    return k;
}

// (v - mean) / std: the correctly rounded quotient (EXACT), or the product
// of the same difference with RN(1/std), which is within one fp32 ulp of it.
template <int EXACT>
__device__ __forceinline__ float normalize_k(const NormK &k, int ch, float v)
{
    return EXACT ? normalize(v, k.mean[ch], k.stdv[ch], k.rcp[ch]) : (v - k.mean[ch]) * k.rcp[ch];
}

// The value an output element holds: normalised (fp32 / fp16 output, OUT 0 /
// 1), or the resized value itself (uint8 output, OUT 2; rounded when packed).
template <int OUT, int EXACT>
__device__ __forceinline__ float out_value(const NormK &k, int ch, float v)
{
    return OUT == 2 ? v : normalize_k<EXACT>(k, ch, v);
}


typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// One output row's two source rows in registers (G chunk loads each), with
// the offset of each row's first byte in its first chunk and the vertical
// weight.
template <int G>
struct StagedRows {
    u32x4 c0[G], c1[G];
    int sh0, sh1;
    float wy;
};

// The rows a wave of the strided walk takes: batch rows q, q + G, q + 2G, ...
// (G waves) as (image, crop row) pairs, which advance by (G / Ch, G % Ch) per
// step, so at any moment the waves work on a band of consecutive output rows,
// close together in memory.
struct RowStep {
    int di, dr, Ch;
};

// First row and row count of wave `w`: the host splits the n * Ch rows as
// rows_q * grid + rows_r, so every wave walks rows_q rows and waves
// w < rows_r one more. STRIDE = 1: wave w starts at row w; STRIDE = 0: at the
// end of the ranges of waves 0 .. w - 1.
template <int STRIDE>
__device__ __forceinline__ void wave_rows(const BatchArgs &a, int w, long long &r0, int &n_rows)
{
    n_rows = a.rows_q + (w < a.rows_r ? 1 : 0);
    r0 = STRIDE ? (long long)w : (long long)w * a.rows_q + min(w, a.rows_r);
}

// Image and crop row of batch row r. (A 64-bit division takes about 140 scalar
// instructions before a wave's first load, so it stands aside for rows past
// 2^32.)
__device__ __forceinline__ void split_row(long long r, int Ch, int &img, int &rr)
{
    if ((unsigned long long)r >> 32 == 0)
        img = (int)((unsigned)r / (unsigned)Ch);
    else
        img = (int)(r / Ch);
    rr = (int)(r - (long long)img * Ch);
}

// Workgroups are dealt to the 8 XCDs round-robin; remap so the waves of one
// XCD take consecutive rows (neighbouring output rows share source rows when
// the vertical scale is below 2, and share the XCD's L2).
__device__ __forceinline__ int xcd_position(int g, int G)
{
    return G % 8 == 0 ? (g % 8) * (G / 8) + g / 8 : g;
}

// A workgroup holds a.wpg independent waves (no barriers), each with its own
// LDS slot of `slot_bytes`; several waves per workgroup cut the cost of
// dispatching the grid. Returns the wave's slot and sets its lane and rows.
// (The wave count comes from the arguments: blockDim would be a memory read
// that every wave waits for before its first address is known.)
template <int STRIDE>
__device__ __forceinline__ uint8_t *rows_wave(uint8_t *lds_all, int slot_bytes, const BatchArgs &a,
                                              int &lane, long long &r0, int &n_rows)
{
    const int wpg = a.wpg;
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    lane = (int)(threadIdx.x & 63);
    const int g = STRIDE ? xcd_position((int)blockIdx.x, (int)gridDim.x) : (int)blockIdx.x;
    wave_rows<STRIDE>(a, g * wpg + wid, r0, n_rows);
    return lds_all + wid * slot_bytes;
}

// floor(n / d) and n - d floor(n / d) for d > 0: one truncating division (a
// 32-bit one when n fits), then the correction for negative n.
__device__ __forceinline__ void floor_divmod(long long n, int d, int &q, int &r)
{
    long long qq = (n >= INT_MIN && n <= INT_MAX) ? (long long)((int)n / d) : n / d;
    long long rr = n - qq * d;
    if (rr < 0) {
        --qq;
        rr += d;
    }
    q = (int)qq;
    r = (int)rr;
}

// Vertical half-pixel taps along a strided walk over rows of one geometry:
// num(rr) = (2 * (top + rr) + 1) * H - Hr, den = 2 * Hr, q = floor(num / den),
// rem = num - q * den. A step moves rr by dr, or by dr - Ch when it wraps to
// the next image of the same geometry, so num by one of two constants whose
// floor quotients and remainders are precomputed: exact integer arithmetic,
// no division per row. (num <= 0 exactly when q < 0 or q == rem == 0.)
struct VCursor {
    int q, rem, den, H;
    int qs, rs;    // step within an image
    int qw, rw;    // step that wraps (a uniform batch)
};

__device__ __forceinline__ void vcursor_init(VCursor &v, const BatchArgs &a, const RowImg &g, int rr,
                                             const RowStep &s)
{
    const int den = 2 * g.Hr;
    int q, rem, qs, rs, qw = 0, rw = 0;
    floor_divmod((long long)(2 * (g.top + rr) + 1) * g.H - g.Hr, den, q, rem);
    if (!a.table) {
        // one geometry for the whole launch: the host computed the steps
        qs = a.vq_s;
        rs = a.vr_s;
        qw = a.vq_w;
        rw = a.vr_w;
    } else {
        // a walk over a table reads the next image's descriptor on a wrap
        floor_divmod(2LL * g.H * s.dr, den, qs, rs);
    }
    // (every field stored on every path: stores that differ by branch can be
    // merged into one store to a chosen field, which keeps the cursor in
    // memory)
    v = VCursor{q, rem, den, g.H, qs, rs, qw, rw};
}

__device__ __forceinline__ void vcursor_add(VCursor &v, int dq, int dr)
{
    v.q += dq;
    v.rem += dr;
    if (v.rem >= v.den) {
        v.rem -= v.den;
        ++v.q;
    }
}

__device__ __forceinline__ void vcursor_tap(const VCursor &v, int &y0, int &y1, float &w)
{
    if (v.q < 0 || (v.q == 0 && v.rem == 0)) {
        y0 = y1 = 0;
        w = 0.0f;
    } else if (v.q >= v.H - 1) {
        y0 = y1 = v.H - 1;
        w = 0.0f;
    } else {
        y0 = v.q;
        y1 = y0 + 1;
        w = (float)v.rem / (float)v.den;  // IEEE division, both operands exact
    }
}

// Load cursor of the strided RGB walk: image, crop row, vertical map and the
// image's row addressing.
struct RowCursor {
    int img, rr;
    VCursor v;
    uintptr_t base;  // first staged byte of source row 0
    int pitch, span;
};

__device__ __forceinline__ void cursor_image(RowCursor &c, const BatchArgs &a, int img, int rr,
                                             const RowStep &s)
{
    const RowImg g = row_img(a, img, (int)blockIdx.y);
    c.img = img;
    c.rr = rr;
    vcursor_init(c.v, a, g, rr, s);
    c.base = (uintptr_t)(a.src + g.off) + 3 * (uintptr_t)g.xf;
    c.pitch = g.pitch;
    c.span = g.span;
}

// Next row of the walk. A strided walk over a uniform batch (one geometry,
// images `stride` bytes apart) moves the base address and steps the vertical
// map; over a table it reads the new image's descriptor when the image
// changes.
__device__ __forceinline__ void cursor_next(RowCursor &c, const BatchArgs &a, const RowStep &s)
{
    const int img0 = c.img;
    c.img += s.di;
    c.rr += s.dr;
    const bool wrapped = c.rr >= s.Ch;
    if (wrapped) {
        c.rr -= s.Ch;
        ++c.img;
    }
    if (!a.table) {
        c.base += (uintptr_t)(c.img - img0) * (uintptr_t)a.stride;
        vcursor_add(c.v, wrapped ? c.v.qw : c.v.qs, wrapped ? c.v.rw : c.v.rs);
    } else if (c.img != img0) {
        cursor_image(c, a, c.img, c.rr, s);
    } else {
        vcursor_add(c.v, c.v.qs, c.v.rs);
    }
}

// `repeat`: the row was loaded already (past the end of the wave's range);
// every lane then loads the rows' first chunk, so the instruction stream is
// unchanged but almost nothing is fetched.
// Nontemporal loads: the strided walk of large frames reads each source row
// once.
template <int G>
__device__ __forceinline__ void load_rows(StagedRows<G> &st, const RowCursor &c, int lane,
                                          bool repeat)
{
    int y0, y1;
    vcursor_tap(c.v, y0, y1, st.wy);
    const uintptr_t r0 = c.base + (uintptr_t)y0 * (uintptr_t)c.pitch;
    const uintptr_t r1 = c.base + (uintptr_t)y1 * (uintptr_t)c.pitch;
    st.sh0 = (int)(r0 & 15);
    st.sh1 = (int)(r1 & 15);
    const int last0 = repeat ? 0 : (st.sh0 + c.span - 1) >> 4;
    const int last1 = repeat ? 0 : (st.sh1 + c.span - 1) >> 4;
    // global address space: a generic (flat) load would also count against
    // the LDS counter and make every LDS access wait for it
    // (a uniform base and a 32-bit lane offset: the loads take the base from
    // scalar registers)
    typedef __attribute__((address_space(1))) const uint8_t GlobalByte;
    GlobalByte *p0 = (GlobalByte *)(r0 - (uintptr_t)st.sh0);
    GlobalByte *p1 = (GlobalByte *)(r1 - (uintptr_t)st.sh1);
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const uint32_t o0 = 16u * (uint32_t)min(64 * g + lane, last0);
        const uint32_t o1 = 16u * (uint32_t)min(64 * g + lane, last1);
        typedef const __attribute__((address_space(1))) u32x4 GlobalChunk;
        st.c0[g] = __builtin_nontemporal_load((GlobalChunk *)(p0 + o0));
        st.c1[g] = __builtin_nontemporal_load((GlobalChunk *)(p1 + o1));
    }
}

template <int G>
__device__ __forceinline__ void write_rows(uint8_t *slot, const StagedRows<G> &st, int lane)
{
#pragma unroll
    for (int g = 0; g < G; ++g) {
        ((u32x4 *)slot)[64 * g + lane] = st.c0[g];
        ((u32x4 *)(slot + 1024 * G))[64 * g + lane] = st.c1[g];
    }
}

// LDS byte address of a pointer into the dynamic LDS array.
__device__ __forceinline__ uint32_t lds_addr(const uint8_t *p)
{
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t *)p;
}

// Tap pairs (6 bytes at LDS byte address A) are read as the three dwords at
// A & ~3 and realigned with v_alignbyte, which takes its shift from the low
// bits of A (an unaligned LDS access is split lane by lane). The reads of a
// row's tap pairs are issued together from inline assembly, then waited for
// once: the compiler would wait after every pixel.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

#define SMOL_RD3(D2, D1, A) "ds_read2_b32 " D2 ", " A " offset1:1\n\tds_read_b32 " D1 ", " A " offset:8\n\t"
__device__ __forceinline__ void lds_read_taps4(const uint32_t (&ad)[4], u32x2 (&lo)[4],
                                               uint32_t (&hi)[4])
{
    asm volatile(SMOL_RD3("%0", "%4", "%8") SMOL_RD3("%1", "%5", "%9") SMOL_RD3("%2", "%6", "%10")
                 SMOL_RD3("%3", "%7", "%11") "s_waitcnt lgkmcnt(0)"
                 : "=&v"(lo[0]), "=&v"(lo[1]), "=&v"(lo[2]), "=&v"(lo[3]), "=&v"(hi[0]),
                   "=&v"(hi[1]), "=&v"(hi[2]), "=&v"(hi[3])
                 : "v"(ad[0]), "v"(ad[1]), "v"(ad[2]), "v"(ad[3])
                 : "memory");
}
__device__ __forceinline__ void lds_read_taps8(const uint32_t (&ad)[8], u32x2 (&lo)[8],
                                               uint32_t (&hi)[8])
{
    asm volatile(SMOL_RD3("%0", "%8", "%16") SMOL_RD3("%1", "%9", "%17")
                 SMOL_RD3("%2", "%10", "%18") SMOL_RD3("%3", "%11", "%19")
                 SMOL_RD3("%4", "%12", "%20") SMOL_RD3("%5", "%13", "%21")
                 SMOL_RD3("%6", "%14", "%22") SMOL_RD3("%7", "%15", "%23")
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(lo[0]), "=&v"(lo[1]), "=&v"(lo[2]), "=&v"(lo[3]), "=&v"(lo[4]),
                   "=&v"(lo[5]), "=&v"(lo[6]), "=&v"(lo[7]), "=&v"(hi[0]), "=&v"(hi[1]),
                   "=&v"(hi[2]), "=&v"(hi[3]), "=&v"(hi[4]), "=&v"(hi[5]), "=&v"(hi[6]),
                   "=&v"(hi[7])
                 : "v"(ad[0]), "v"(ad[1]), "v"(ad[2]), "v"(ad[3]), "v"(ad[4]), "v"(ad[5]),
                   "v"(ad[6]), "v"(ad[7])
                 : "memory");
}
__device__ __forceinline__ void lds_read_taps2(const uint32_t (&ad)[2], u32x2 (&lo)[2],
                                               uint32_t (&hi)[2])
{
    asm volatile(SMOL_RD3("%0", "%2", "%4") SMOL_RD3("%1", "%3", "%5") "s_waitcnt lgkmcnt(0)"
                 : "=&v"(lo[0]), "=&v"(lo[1]), "=&v"(hi[0]), "=&v"(hi[1])
                 : "v"(ad[0]), "v"(ad[1])
                 : "memory");
}
#undef SMOL_RD3

// The 2J tap pairs of one staged row (pixel c and c + 1 of every column
// iteration), realigned to 8-byte values: tap 2j + px.
template <int J>
__device__ __forceinline__ void read_row_taps(uint32_t row, const int (&cx)[J][2],
                                              uint64_t (&v)[2 * J])
{
    constexpr int N = 2 * J;
    uint32_t A[N], ad[N], hi[N];
    u32x2 lo[N];
#pragma unroll
    for (int t = 0; t < N; ++t) {
        A[t] = row + (uint32_t)cx[t / 2][t & 1];
        ad[t] = A[t] & ~3u;
    }
    static_assert(N == 2 || N == 4, "lerps are kept for one or two pairs per lane");
    if constexpr (N == 4)
        lds_read_taps4(ad, lo, hi);
    else
        lds_read_taps2(ad, lo, hi);
#pragma unroll
    for (int t = 0; t < N; ++t)
        v[t] = (uint64_t)__builtin_amdgcn_alignbyte(lo[t].y, lo[t].x, A[t]) |
               ((uint64_t)__builtin_amdgcn_alignbyte(hi[t], lo[t].y, A[t]) << 32);
}

// The tap pairs of column iterations j0 .. j0 + N/4 - 1 (pixel c, c + 1 of
// rows 0 and 1 each), realigned to 8-byte values.
template <int J, int N>
__device__ __forceinline__ void read_taps(uint32_t row0, uint32_t row1, const int (&cx)[J][2],
                                          int j0, uint64_t (&v)[N])
{
    uint32_t A[N], ad[N], hi[N];
    u32x2 lo[N];
#pragma unroll
    for (int t = 0; t < N; ++t) {
        const int j = j0 + t / 4, px = t & 1;
        A[t] = ((t & 2) ? row1 : row0) + (uint32_t)cx[j][px];
        ad[t] = A[t] & ~3u;
    }
    if constexpr (N == 8)
        lds_read_taps8(ad, lo, hi);
    else
        lds_read_taps4(*(const uint32_t(*)[4])ad, *(u32x2(*)[4])lo, *(uint32_t(*)[4])hi);
#pragma unroll
    for (int t = 0; t < N; ++t)
        v[t] = (uint64_t)__builtin_amdgcn_alignbyte(lo[t].y, lo[t].x, A[t]) |
               ((uint64_t)__builtin_amdgcn_alignbyte(hi[t], lo[t].y, A[t]) << 32);
}

// One output row's values of a lane, ready to store: per column iteration
// and channel the pair (c, c + 1) as one dword (fp16) or two (fp32).
//
// A row's stores are issued after the next row's chunks are written to LDS,
// not before: the wait for those chunks' loads then never includes the
// completion of this row's stores (the compiler cannot count stores among
// the loads they may overtake, so a wait for a load issued before a store
// lasts until the store is done as well).
// Output form of a row-streaming kernel instance (its FORM template
// parameter): NHWC layout, crops of a single column, rows stored as whole
// lines.
constexpr int kFormNhwc = 1;
constexpr int kFormOne = 2;
constexpr int kFormLines = 4;

// A lane's output pairs of one row: per channel, for every column pair, two
// fp32 words (F16 0), one word of two fp16 (F16 1) or the low half-word of one
// word holding two uint8 (F16 2, uint8 output). (One vector, not an array:
// vector stores gathered from an array's elements keep the array in memory.)
template <int F16, int J>
struct RowOut {
    static constexpr int kWords = F16 ? J : 2 * J;  // per channel
    uint32_t __attribute__((ext_vector_type(3 * kWords))) w;
    // word k of pair j (k = 0 unless fp32)
    __device__ __forceinline__ uint32_t word(int ch, int j, int k = 0) const
    {
        return w[ch * kWords + (F16 ? j : 2 * j + k)];
    }
    __device__ __forceinline__ void set(int ch, int j, int k, uint32_t v)
    {
        w[ch * kWords + (F16 ? j : 2 * j + k)] = v;
    }
};

template <int F16, int EXACT, int J>
__device__ __forceinline__ void pack_pair(RowOut<F16, J> &out, int j, const float (&o)[3][2])
{
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        if (F16 == 2) {
            // clamped to [0, 255] and rounded to nearest even, into bytes 0
            // and 1 (v_cvt_pk_u8_f32 does clamp, round, convert and insert)
            out.set(ch, j, 0,
                    __builtin_amdgcn_cvt_pk_u8_f32(
                        o[ch][1], 1u, __builtin_amdgcn_cvt_pk_u8_f32(o[ch][0], 0u, 0u)));
        } else if (F16 && !EXACT) {
            // The conversion may fuse with the last product (one rounding
            // to fp16 instead of two).
            typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
            const f16x2 h = {(_Float16)o[ch][0], (_Float16)o[ch][1]};
            out.set(ch, j, 0, __builtin_bit_cast(uint32_t, h));
        } else if (F16) {
            out.set(ch, j, 0, f16_bits(o[ch][0]) | (f16_bits(o[ch][1]) << 16));
        } else {
            out.set(ch, j, 0, __builtin_bit_cast(uint32_t, o[ch][0]));
            out.set(ch, j, 1, __builtin_bit_cast(uint32_t, o[ch][1]));
        }
    }
}

// Store a lane's columns (pair_col) of one output row: per plane (NCHW) or
// interleaved (NHWC), in the widest stores that hold them (4 columns of fp16:
// 8 bytes per plane). The addresses are aligned to an element only: crop
// widths and strips are arbitrary, and global stores take any alignment.
// ONE (a crop of one column) is a template parameter so that the stores are
// straight-line code: the compiler then counts them exactly in the vmcnt waits
// of the row loop (with a branch here it waits for them as well when it waits
// for the next rows' loads).
// Stores are nontemporal: on their own, 308 MB of 448-byte rows take 77 us as
// 4-byte stores, 68 as 8-byte ones and 57 as 16-byte stores of whole 128-byte
// lines; ordinary stores are as fast alone but 1.5 times slower beside the
// loads. uint8 output is stored ordinarily: it is small, and the
// low-resolution op reads it back at once (step 2 of 256 images: 24.3 us, 29.7
// after nontemporal stores).
template <int N, bool NT>
__device__ __forceinline__ void store_words(uint8_t *dst,
                                            uint32_t __attribute__((ext_vector_type(N))) v)
{
    typedef uint32_t Unaligned __attribute__((ext_vector_type(N), aligned(1)));
    if (NT)
        __builtin_nontemporal_store(v, (Unaligned *)dst);
    else
        *(Unaligned *)dst = v;
}

template <bool NT>
__device__ __forceinline__ void store_half(uint8_t *dst, uint32_t v)
{
    typedef uint16_t __attribute__((aligned(1))) Unaligned;
    if (NT)
        __builtin_nontemporal_store((uint16_t)v, (Unaligned *)dst);
    else
        *(Unaligned *)dst = (uint16_t)v;
}

template <int F16, int J, int ONE, bool QUADS, bool NT>
__device__ __forceinline__ void store_row(uint8_t *orow, long long plane, int cols, int lane,
                                          const RowOut<F16, J> &out, int nhwc)
{
    static_assert(!(QUADS && J > 2), "four columns side by side at most");
    constexpr int kEsz = F16 == 2 ? 1 : F16 ? 2 : 4;
    constexpr bool FOUR = QUADS && J == 2;  // the lane's columns lie side by side
    if constexpr (ONE) {
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            uint8_t *dst = orow + (nhwc ? ch * kEsz : ch * plane);
            if (F16 == 2)
                *dst = (uint8_t)out.word(ch, 0);
            else if (F16)
                *(uint16_t *)dst = (uint16_t)out.word(ch, 0);
            else
                *(uint32_t *)dst = out.word(ch, 0);
        }
        return;
    }
    if (!nhwc) {
#pragma unroll
        for (int j = 0; j < (FOUR ? 1 : J); ++j) {
            const uint32_t lo = (uint32_t)pair_col<J, QUADS>(lane, j, cols) * kEsz;
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                uint8_t *dst = orow + ch * plane + lo;
                if constexpr (F16 == 2 && !FOUR)
                    store_half<NT>(dst, out.word(ch, j));
                else if constexpr (F16 == 2)
                    store_words<1, NT>(dst, (out.word(ch, 0) & 0xffffu) |
                                                   (out.word(ch, J - 1) << 16));
                else if constexpr (F16 && !FOUR)
                    store_words<1, NT>(dst, out.word(ch, j));
                else if constexpr (F16)
                    store_words<2, NT>(dst, u32x2{out.word(ch, 0), out.word(ch, J - 1)});
                else if constexpr (!FOUR)
                    store_words<2, NT>(dst, u32x2{out.word(ch, j), out.word(ch, j, 1)});
                else
                    store_words<4, NT>(dst, u32x4{out.word(ch, 0), out.word(ch, 0, 1),
                                              out.word(ch, J - 1), out.word(ch, J - 1, 1)});
            }
        }
        return;
    }
    typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
    if constexpr (F16 == 2) {
        // a pair is r0 g0 b0 r1 g1 b1, the bytes of a word being pixels c, c + 1
        uint32_t lo[J], hi[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const uint32_t r = out.word(0, j), g = out.word(1, j), b = out.word(2, j);
            lo[j] = (r & 0xffu) | (g & 0xffu) << 8 | (b & 0xffu) << 16 | (r & 0xff00u) << 16;
            hi[j] = (g >> 8 & 0xffu) | (b & 0xff00u);
        }
        if constexpr (!FOUR) {
#pragma unroll
            for (int j = 0; j < J; ++j) {
                uint8_t *dj = orow + 3u * (uint32_t)pair_col<J, QUADS>(lane, j, cols);
                store_words<1, NT>(dj, lo[j]);
                store_half<NT>(dj + 4, hi[j]);
            }
        } else {
            store_words<3, NT>(orow + 3u * (uint32_t)pair_col<J, true>(lane, 0, cols),
                                  u32x3{lo[0], hi[0] | lo[J - 1] << 16,
                                        lo[J - 1] >> 16 | hi[J - 1] << 16});
        }
    } else {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            // two pixels: r g b r g b
            uint8_t *dj = orow + 3u * (uint32_t)pair_col<J, false>(lane, j, cols) * kEsz;
            if constexpr (F16) {
                const uint32_t w0 = out.word(0, j), w1 = out.word(1, j), w2 = out.word(2, j);
                store_words<3, NT>(dj, u32x3{(w0 & 0xffffu) | (w1 << 16),
                                         (w2 & 0xffffu) | (w0 & 0xffff0000u),
                                         (w1 >> 16) | (w2 & 0xffff0000u)});
            } else {
                store_words<2, NT>(dj, u32x2{out.word(0, j), out.word(1, j)});
                store_words<2, NT>(dj + 8, u32x2{out.word(2, j), out.word(0, j, 1)});
                store_words<2, NT>(dj + 16, u32x2{out.word(1, j, 1), out.word(2, j, 1)});
            }
        }
    }
}

// Interpolate, normalise and store one output row from its staged rows
// (row 0 at byte `row0` of lds, row 1 at `row1`, both including the offset
// of the first byte in its chunk).
template <int F16, int J, int EXACT>
__device__ __forceinline__ void rows_compute(const NormK &nk, uint32_t row0, uint32_t row1,
                                             float wy, const int (&cx)[J][2],
                                             const float (&cw)[J][2], RowOut<F16, J> &out)
{
    // tap pairs, 4 per column iteration: pixel c and c + 1 of row 0, then row 1
    constexpr int kN = J == 1 ? 4 : 8;
    uint64_t v[J * 4];
#pragma unroll
    for (int j0 = 0; j0 < J; j0 += kN / 4)
        read_taps<J, kN>(row0, row1, cx, j0, *(uint64_t(*)[kN]) & v[4 * j0]);
#pragma unroll
    for (int j = 0; j < J; ++j) {
        float o[3][2];
#pragma unroll
        for (int px = 0; px < 2; ++px) {
            float pa[3], pd[3], qa[3], qd[3];
            unpack_ad(v[4 * j + px], pa, pd);
            unpack_ad(v[4 * j + 2 + px], qa, qd);
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                const float top = lerp_ad(pa[ch], pd[ch], cw[j][px]);
                const float bot = lerp_ad(qa[ch], qd[ch], cw[j][px]);
                o[ch][px] = out_value<F16, EXACT>(nk, ch, lerp(top, bot, wy));
            }
        }
        pack_pair<F16, EXACT, J>(out, j, o);
    }
}

// Horizontal lerps of one staged row at the lane's columns: h[j][px][ch].
template <int J>
__device__ __forceinline__ void rows_horizontal(uint32_t row, const int (&cx)[J][2],
                                                const float (&cw)[J][2], float (&h)[J][2][3])
{
    uint64_t v[2 * J];
    read_row_taps<J>(row, cx, v);
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int px = 0; px < 2; ++px) {
            float pa[3], pd[3];
            unpack_ad(v[2 * j + px], pa, pd);
#pragma unroll
            for (int ch = 0; ch < 3; ++ch)
                h[j][px][ch] = lerp_ad(pa[ch], pd[ch], cw[j][px]);
        }
}

// Vertical lerp of two rows of horizontal lerps, normalise, store.
template <int F16, int J, int EXACT>
__device__ __forceinline__ void rows_vertical(const NormK &nk, const float (&h0)[J][2][3],
                                              const float (&h1)[J][2][3], float wy,
                                              RowOut<F16, J> &out)
{
#pragma unroll
    for (int j = 0; j < J; ++j) {
        float o[3][2];
#pragma unroll
        for (int px = 0; px < 2; ++px)
#pragma unroll
            for (int ch = 0; ch < 3; ++ch)
                o[ch][px] = out_value<F16, EXACT>(nk, ch,
                                                  lerp(h0[j][px][ch], h1[j][px][ch], wy));
        pack_pair<F16, EXACT, J>(out, j, o);
    }
}

// The rows of a contiguous walk, one per lane: up to 64 rows' vertical taps
// and addresses are computed at once, each lane its own row, and read back
// lane by lane as scalars, so a row costs a few scalar moves instead of a
// cursor's steps, a division and 64-bit addresses in every lane.
constexpr int kRowNew = 0;    // both source rows differ from the previous row's
constexpr int kRowShift = 1;  // y0 is the previous row's y1
constexpr int kRowSame = 2;   // the previous row's source rows
struct RowRecs {
    uint32_t lo, hi;  // address of the row's first staged byte in source row y0
    uint32_t d1;      // bytes from there to the same column of source row y1
    float wy;
    uint32_t kind;    // span << 2 | relation to the previous row
};

// Records of the next `count` rows, at most 64, from crop row rr of image img
// on. An image's first row and the first record are kRowNew. (Only the images
// of those rows are visited: a ragged batch's descriptors come over the bus.)
__device__ __forceinline__ void row_records(RowRecs &t, const BatchArgs &a, int img, int rr,
                                            int count, int lane, int strip)
{
    const int Ch = a.Ch;
    int first = 0;  // the record of crop row rr of image img
    int y0 = 0, y1 = 0;
    bool fresh = lane == 0;
    while (true) {
        const RowImg g = row_img(a, img, strip);
        const int r = rr + lane - first;
        const Tap ty = axis_tap(g.top + r, g.H, g.Hr);
        if (lane >= first && r < Ch) {
            const uint64_t base = (uint64_t)(uintptr_t)(a.src + g.off) + 3u * (uint64_t)g.xf;
            const uint64_t addr = base + (uint64_t)(uint32_t)ty.x0 * (uint32_t)g.pitch;
            t.lo = (uint32_t)addr;
            t.hi = (uint32_t)(addr >> 32);
            t.d1 = ty.x1 > ty.x0 ? (uint32_t)g.pitch : 0u;
            t.wy = ty.w;
            t.kind = (uint32_t)g.span << 2;
            y0 = ty.x0;
            y1 = ty.x1;
            fresh = fresh || r == 0;
        }
        first += Ch - rr;
        rr = 0;
        if (first >= min(count, 64))
            break;
        ++img;
    }
    const int p0 = __shfl_up(y0, 1, 64), p1 = __shfl_up(y1, 1, 64);
    t.kind |= fresh                    ? kRowNew
              : y0 == p0 && y1 == p1 ? kRowSame
              : y0 == p1             ? kRowShift
                                     : kRowNew;
}

}  // namespace
}  // namespace smol
