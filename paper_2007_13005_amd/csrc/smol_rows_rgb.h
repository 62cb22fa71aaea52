// smol_rows_rgb.h -- the RGB row-streaming kernels (rgb_stride_kernel,
// rgb_range_kernel) and the choice of their instance for a plan. The
// smol_rows_rgb_*.hip files instantiate their parts.
#pragma once

#include "smol_rows.h"

namespace smol {
namespace {

// Strided walk: wave q takes rows q, q + G, ... (G waves). FORM: kFormNhwc,
// kFormOne.
template <int F16, int J, int EXACT, int G, int P, int FORM>
__global__ void __launch_bounds__(64 * kRowsMaxWavesPerGroup) rgb_stride_kernel(BatchArgs a)
{
    constexpr int NHWC = FORM & kFormNhwc, ONE = (FORM & kFormOne) ? 1 : 0;
    constexpr bool QUADS = (!NHWC || F16 == 2) && J <= 2;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_all[];
    int lane;
    long long r0;
    int n_rows;
    const int Ch = a.Ch;
    uint8_t *const lds = rows_wave<1>(lds_all, 2048 * G, a, lane, r0, n_rows);
    // The host launches at most one wave per row, so every wave has rows (an
    // early exit here would hold the remaining argument loads behind it).
    __builtin_assume(n_rows > 0);
    const int strip = (int)blockIdx.y;
    const RowStep step{a.step_di, a.step_dr, Ch};
    constexpr int kEsz = F16 == 2 ? 1 : F16 ? 2 : 4;
    int c_img, c_rr;  // row to interpolate
    split_row(r0, Ch, c_img, c_rr);
    RowCursor lc;  // next row to load
    cursor_image(lc, a, c_img, c_rr, step);

    // The load cursor stops at the wave's last row: past the end the loads
    // repeat that row (fetching one chunk), so every step issues the same
    // loads and the compiler can count exactly what is outstanding when a
    // row is written to LDS.
    int lrow = 0;
    bool at_end = false;  // the cursor sits on the wave's last row, already loaded
    auto advance = [&]() {
        if (lrow + 1 < n_rows) {
            cursor_next(lc, a, step);
            ++lrow;
        } else {
            at_end = true;
        }
    };
    // The first row (two with P = 2) is requested before the column taps
    // and the rest of the set-up are computed.
    StagedRows<G> A, B, C;
    load_rows<G>(A, lc, lane, false);
    advance();
    if (P == 2) {
        load_rows<G>(B, lc, lane, at_end);
        advance();
    }

    // Output row pointer of the row to interpolate: a step adds 3 Ch di + dr
    // rows, plus 2 Ch (planes 1 and 2 of the image left) when it wraps.
    // bytes between an image's output rows: Cw elements per plane (NCHW) or
    // 3 Cw (NHWC); a wrap to the next image skips the rest of the image.
    const long long rb = (long long)a.Cw * kEsz, rowb = NHWC ? 3 * rb : rb;
    const long long imgb = 3LL * Ch * rb;
    uint8_t *orow = (uint8_t *)a.out + (long long)(a.img_base + c_img) * imgb + c_rr * rowb +
                    (long long)strip_start(a, strip) * (NHWC ? 3 : 1) * kEsz;
    const long long ostep = step.di * imgb + step.dr * rowb, owrap = imgb - Ch * rowb;
    int cx[J][2];
    float cw[J][2];
    int cW, cWr, cleft;
    {
        const RowImg g = row_img(a, c_img, strip);
        row_taps<J, QUADS>(g, a.strip_w, cx, cw, lane);
        cW = g.W;
        cWr = g.Wr;
        cleft = g.left;
    }
    const NormK nk = norm_consts(a);
    const uint32_t lds0 = lds_addr(lds);

    // P = 2: a step loads row k + 2 into FUT, interpolates row k (staged in
    // LDS), writes row k + 1 (in NXT) into the slot; the three register sets
    // rotate over three steps without copies. P = 1: one register set, loaded
    // with row k + 1 before row k is interpolated. The loop runs the n_rows - 1
    // steps that stage a next row and leaves only at its end, with nothing
    // outstanding but the prefetched row; the last row is interpolated after
    // it.
    write_rows<G>(lds, A, lane);
    int csh0 = A.sh0, csh1 = A.sh1;
    float cwy = A.wy;
    const long long plane = (long long)Ch * a.Cw * kEsz;
    RowOut<F16, J> out;
    auto compute = [&]() {
        rows_compute<F16, J, EXACT>(nk, lds0 + (uint32_t)csh0, lds0 + (uint32_t)(1024 * G + csh1),
                                    cwy, cx, cw, out);
    };
#define SMOL_ROWS_STEP(NXT, FUT)                                                              \
    {                                                                                         \
        load_rows<G>(FUT, lc, lane, at_end);                                                  \
        advance();                                                                            \
        compute();                                                                            \
        write_rows<G>(lds, NXT, lane);                                                        \
        store_row<F16, J, ONE, QUADS, true>(orow, plane, a.strip_w, lane, out, NHWC);         \
        csh0 = NXT.sh0;                                                                       \
        csh1 = NXT.sh1;                                                                       \
        cwy = NXT.wy;                                                                         \
        const int pimg = c_img;                                                               \
        c_img += step.di;                                                                     \
        c_rr += step.dr;                                                                      \
        orow += ostep;                                                                        \
        if (c_rr >= Ch) {                                                                     \
            c_rr -= Ch;                                                                       \
            ++c_img;                                                                          \
            orow += owrap;                                                                    \
        }                                                                                     \
        if (c_img != pimg) {                                                                  \
            const RowImg g = row_img(a, c_img, strip);                                        \
            if (g.W != cW || g.Wr != cWr || g.left != cleft) {                                \
                cW = g.W;                                                                     \
                cWr = g.Wr;                                                                   \
                cleft = g.left;                                                               \
                row_taps<J, QUADS>(g, a.strip_w, cx, cw, lane);                               \
            }                                                                                 \
        }                                                                                     \
    }
    int left = n_rows - 1;
    if (P == 2) {
        for (; left >= 3; left -= 3) {
            SMOL_ROWS_STEP(B, C)
            SMOL_ROWS_STEP(C, A)
            SMOL_ROWS_STEP(A, B)
        }
        if (left >= 1)
            SMOL_ROWS_STEP(B, C)
        if (left >= 2)
            SMOL_ROWS_STEP(C, A)
    } else {
        for (; left > 0; --left)
            SMOL_ROWS_STEP(A, A)
    }
#undef SMOL_ROWS_STEP
    compute();
    store_row<F16, J, ONE, QUADS, true>(orow, plane, a.strip_w, lane, out, NHWC);
}

// Contiguous walk: wave w takes a range of consecutive output rows. The wave's
// rows come from row_records; the next row's chunks are loaded into registers
// while a row is interpolated, and written to the wave's LDS slot after it.
// Consecutive rows share source rows when the vertical scale is below 2, so the
// horizontal lerps of the last two source rows stay in registers (A, B; `swap`
// says which one is y0's): a row whose y0 was the previous row's y1 computes
// one source row, a row of the same source rows none, and nothing is copied.
//
// LINES (fp16 NCHW whole crops whose rows are not whole 128-byte lines): a
// wave's rows are consecutive in each plane, so they are gathered in LDS and
// leave as the whole lines they complete, 16 bytes per lane; a row's own 8-byte
// stores leave partial lines at both ends, which the memory takes one by one.
//
// What bounds it: upscales issue VALU instructions for 51 of their 72 us (1024
// images of 128 x 128 to 224 x 224 without stores) and store for 57; larger
// sources are bound by memory, whose reads and writes do not overlap (512 x 512
// to 224 x 224: 33 us without stores, 25 without loads, 52 together). 1024
// thumbnails: 81.3 us with a vertical cursor per wave, copied lerps and 4-byte
// stores, 75.6 with row records, 72 with whole lines as well. A second row in
// flight costs registers and time (77.8 against 75.0 us), so only one is.
template <int F16, int J, int EXACT, int G, int FORM>
__global__ void __launch_bounds__(64 * kRowsMaxWavesPerGroup) rgb_range_kernel(BatchArgs a)
{
    constexpr int NHWC = FORM & kFormNhwc, ONE = (FORM & kFormOne) ? 1 : 0;
    // Long staged rows are large shrinks, whose lanes' taps lie far apart (four
    // columns side by side at a shrink by 5.3: 16 words, 4 of the 64 LDS banks;
    // pairs: 8 words and 8 banks).
    constexpr bool QUADS = (!NHWC || F16 == 2) && G <= 2 && J <= 2;
    constexpr bool LINES = (FORM & kFormLines) != 0;
    constexpr bool NT = F16 != 2 || G >= 4;
    static_assert(!LINES || (F16 == 1 && !NHWC && !ONE), "whole lines: fp16 NCHW");
    constexpr int kEsz = F16 == 2 ? 1 : F16 ? 2 : 4;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_all[];
    int lane;
    long long r0;
    int n_rows;
    const int Ch = a.Ch;
    uint8_t *const lds = rows_wave<0>(lds_all, 2048 * G + (LINES ? 3 * kLineRing : 0), a, lane, r0,
                                      n_rows);
    // The host launches at most one wave per row, so every wave has rows (an
    // early exit here would hold the remaining argument loads behind it).
    __builtin_assume(n_rows > 0);
    const int strip = (int)blockIdx.y;
    int c_img, c_rr;  // row to interpolate
    split_row(r0, Ch, c_img, c_rr);

    RowRecs recs;
    row_records(recs, a, c_img, c_rr, n_rows, lane, strip);
    // A row's scalars: offset of each source row's first byte in its first
    // chunk, vertical weight, relation to the previous row.
    struct RowS {
        uint32_t sh0, sh1;
        float wy;
        uint32_t rel;
    };
    struct Chunks {
        u32x4 c0[G], c1[G];
    };
    RowS nxt;
    int li = 0;  // next row to load
    const uint32_t lane16 = 16u * (uint32_t)lane;
    // Loads row li into registers and moves on. Past the wave's last row the
    // loads repeat its first chunks (fetching almost nothing), so every step
    // issues the same loads and the compiler can count what is outstanding
    // when a row is written to LDS.
    auto load_next = [&](Chunks &st) {
        const bool past = li >= n_rows;
        if (!past && li != 0 && (li & 63) == 0) {
            int img, rr;
            split_row(r0 + li, Ch, img, rr);
            row_records(recs, a, img, rr, n_rows - li, lane, strip);
        }
        const int i = min(li, n_rows - 1) & 63;
        const uint32_t lo = __builtin_amdgcn_readlane(recs.lo, i);
        const uint32_t hi = __builtin_amdgcn_readlane(recs.hi, i);
        const uint32_t d1 = __builtin_amdgcn_readlane(recs.d1, i);
        const uint32_t kind = __builtin_amdgcn_readlane(recs.kind, i);
        nxt.wy = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(recs.wy), i));
        nxt.rel = kind & 3u;
        const uint64_t p0 = (uint64_t)hi << 32 | lo, p1 = p0 + d1;
        nxt.sh0 = (uint32_t)p0 & 15u;
        nxt.sh1 = (uint32_t)p1 & 15u;
        // (lanes past a row's last chunk load that chunk again)
        const uint32_t span1 = (kind >> 2) - 1;
        const uint32_t last0 = past ? 0u : (nxt.sh0 + span1) & ~15u;
        const uint32_t last1 = past ? 0u : (nxt.sh1 + span1) & ~15u;
        // global address space, a uniform base and a 32-bit lane offset: the
        // loads take the base from scalar registers and do not count against
        // the LDS counter. Ordinary loads: rows met again hit in the caches.
        typedef __attribute__((address_space(1))) const uint8_t GlobalByte;
        typedef __attribute__((address_space(1))) const u32x4 GlobalChunk;
        GlobalByte *q0 = (GlobalByte *)(p0 & ~(uint64_t)15), *q1 = (GlobalByte *)(p1 & ~(uint64_t)15);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            st.c0[g] = *(GlobalChunk *)(q0 + min(lane16 + 1024u * g, last0));
            st.c1[g] = *(GlobalChunk *)(q1 + min(lane16 + 1024u * g, last1));
        }
        ++li;
    };
    auto stage = [&](const Chunks &st) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            ((u32x4 *)lds)[64 * g + lane] = st.c0[g];
            ((u32x4 *)(lds + 1024 * G))[64 * g + lane] = st.c1[g];
        }
    };
    // The first row is requested before the column taps and the rest of the
    // set-up are computed.
    Chunks ahead;
    load_next(ahead);
    RowS cur = nxt;

    // bytes between an image's output rows: Cw elements per plane (NCHW) or
    // 3 Cw (NHWC); a wrap to the next image skips the rest of the image.
    const long long rb = (long long)a.Cw * kEsz, rowb = NHWC ? 3 * rb : rb;
    const long long plane = Ch * rb, imgb = 3 * plane;
    uint8_t *orow = (uint8_t *)a.out + (long long)(a.img_base + c_img) * imgb + c_rr * rowb +
                    (long long)strip_start(a, strip) * (NHWC ? 3 : 1) * kEsz;
    const long long owrap = NHWC ? 0 : 2 * plane;
    int cx[J][2];
    float cw[J][2];
    int cW, cWr, cleft;
    {
        const RowImg g = row_img(a, c_img, strip);
        row_taps<J, QUADS>(g, a.strip_w, cx, cw, lane);
        cW = g.W;
        cWr = g.Wr;
        cleft = g.left;
    }
    const NormK nk = norm_consts(a);
    const uint32_t lds0 = lds_addr(lds), lds1 = lds0 + 1024 * G;
    float hA[J][2][3], hB[J][2][3];
    bool swap = false;  // hB holds y0's lerps, hA y1's
    RowOut<F16, J> out;
    auto compute = [&](const RowS &row) {
        if constexpr (J > 2) {  // (kept lerps would take 48 registers more)
            rows_compute<F16, J, EXACT>(nk, lds0 + row.sh0, lds1 + row.sh1, row.wy, cx, cw, out);
        } else {
            if (row.rel == kRowNew) {
                swap = false;
                rows_horizontal<J>(lds0 + row.sh0, cx, cw, hA);
                rows_horizontal<J>(lds1 + row.sh1, cx, cw, hB);
            } else if (row.rel == kRowShift) {
                // (the differing empty asm keeps the branches apart: merged into
                // one with a chosen array, the arrays would live in memory)
                swap = !swap;
                if (swap) {
                    rows_horizontal<J>(lds1 + row.sh1, cx, cw, hA);
                    asm volatile("; row into A");
                } else {
                    rows_horizontal<J>(lds1 + row.sh1, cx, cw, hB);
                    asm volatile("; row into B");
                }
            }
            if (swap) {
                rows_vertical<F16, J, EXACT>(nk, hB, hA, row.wy, out);
                asm volatile("; rows B, A");
            } else {
                rows_vertical<F16, J, EXACT>(nk, hA, hB, row.wy, out);
                asm volatile("; rows A, B");
            }
        }
    };
    // Whole lines: the ring holds byte b of the wave's rows (counted from
    // `pos0`, the offset of the first row in its 128-byte line; the planes'
    // sizes are whole lines, so all three share it) at b modulo its size.
    uint8_t *const ring = lds + 2048 * G;
    uint32_t pos = LINES ? (uint32_t)(uintptr_t)orow & 127u : 0u;  // the row's first byte
    uint32_t done = pos;                                          // bytes stored so far
    const uint32_t lane_out = LINES ? 2u * (uint32_t)pair_col<J, QUADS>(lane, 0, a.strip_w) : 0u;
    const uint32_t lane_out1 =
        LINES ? 2u * (uint32_t)pair_col<J, QUADS>(lane, J - 1, a.strip_w) : 0u;
    // store the row; `last`: the wave's last row
    auto store = [&](bool last) {
        if constexpr (!LINES) {
            store_row<F16, J, ONE, QUADS, NT>(orow, plane, a.strip_w, lane, out, NHWC);
        } else {
            const uint32_t wo = (pos + lane_out) & (kLineRing - 1);
            const uint32_t w1 = (pos + lane_out1) & (kLineRing - 1);
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                if constexpr (J == 1 || !QUADS) {
                    *(uint32_t *)(ring + ch * kLineRing + wo) = out.word(ch, 0);
                    if constexpr (J == 2)
                        *(uint32_t *)(ring + ch * kLineRing + w1) = out.word(ch, J - 1);
                } else
                    *(u32x2 *)(ring + ch * kLineRing + wo) = u32x2{out.word(ch, 0), out.word(ch, J - 1)};
            }
            const uint32_t end = pos + (uint32_t)rb;
            // (an image ends at a line's end)
            const uint32_t to = last ? end : end & ~127u;
            const uint32_t off = min(lane16, to - done - 16u);
            const uint32_t ro = (done + off) & (kLineRing - 1);
            uint8_t *dst = orow - (pos - done);
#pragma unroll
            for (int ch = 0; ch < 3; ++ch)
                store_words<4, true>(dst + ch * plane + off, *(const u32x4 *)(ring + ch * kLineRing + ro));
            done = to;
            pos = end;
        }
    };
    stage(ahead);
    for (int left = n_rows - 1; left > 0; --left) {
        load_next(ahead);
        compute(cur);
        stage(ahead);
        cur = nxt;
        store(false);
        orow += rowb;
        if (++c_rr == Ch) {
            c_rr = 0;
            ++c_img;
            orow += owrap;
            const RowImg g = row_img(a, c_img, strip);
            if (g.W != cW || g.Wr != cWr || g.left != cleft) {
                cW = g.W;
                cWr = g.Wr;
                cleft = g.left;
                row_taps<J, QUADS>(g, a.strip_w, cx, cw, lane);
            }
        }
    }
    compute(cur);
    store(true);
}

// Column pairs per lane, output form and (strided walk) prefetch depth from
// the launch arguments.
template <int F16, int EXACT, int G, int STRIDE, int FORM, int J>
const void *rgb_rows_k(const BatchArgs &a)
{
    if constexpr (STRIDE)
        return a.prefetch == 1 ? (const void *)rgb_stride_kernel<F16, J, EXACT, G, 1, FORM>
                               : (const void *)rgb_stride_kernel<F16, J, EXACT, G, 2, FORM>;
    else
        return (const void *)rgb_range_kernel<F16, J, EXACT, G, FORM>;
}

template <int F16, int EXACT, int G, int STRIDE, int NHWC>
const void *rgb_rows_g(const BatchArgs &a)
{
    if constexpr (F16 == 1 && !STRIDE && !NHWC)
        if (a.lines)
            return a.col_iters > 1 ? rgb_rows_k<F16, EXACT, G, STRIDE, kFormLines, 2>(a)
                                   : rgb_rows_k<F16, EXACT, G, STRIDE, kFormLines, 1>(a);
    // (the forms that the host's plan takes to one wide strip)
    if constexpr (STRIDE || F16 == 2 ? G == 4 : F16 == 0 && NHWC && G <= 2)
        if (a.col_iters > 2)
            return rgb_rows_k<F16, EXACT, G, STRIDE, NHWC, kRowsWidePairs>(a);
    return a.col_iters > 1 ? rgb_rows_k<F16, EXACT, G, STRIDE, NHWC, 2>(a)
           : a.Cw > 1      ? rgb_rows_k<F16, EXACT, G, STRIDE, NHWC, 1>(a)
                           : rgb_rows_k<F16, EXACT, G, STRIDE, NHWC | kFormOne, 1>(a);
}

template <int F16, int EXACT, int STRIDE, int NHWC>
const void *rgb_rows_f(const BatchArgs &a)
{
    return a.row_groups <= 1   ? rgb_rows_g<F16, EXACT, 1, STRIDE, NHWC>(a)
           : a.row_groups <= 2 ? rgb_rows_g<F16, EXACT, 2, STRIDE, NHWC>(a)
                               : rgb_rows_g<F16, EXACT, 4, STRIDE, NHWC>(a);
}

template <int F16, int STRIDE, int NHWC>
const void *rgb_rows_table(const BatchArgs &a)
{
    return a.exact ? rgb_rows_f<F16, 1, STRIDE, NHWC>(a) : rgb_rows_f<F16, 0, STRIDE, NHWC>(a);
}
}  // namespace
}  // namespace smol
