// Polyphase formulation of the WTConv operator on the gfx950 matrix cores:
// device building blocks shared by the forward and the kernel-gradient
// kernels. Internal; not part of the public ABI.
//
// Operands. The matrix cores take 16-bit operands and accumulate in float32.
// A float32 value is split into three bfloat16 pieces h + m + l (8 bits each,
// exactly from 2^-110 on), and a product keeps the six piece products down to
// 2^-16 of it; the dropped ones are below 2^-24 together, about one float32
// rounding. bfloat16 and float16 storage needs one piece for the input itself
// (bfloat16 / float16 matrix instructions) and three for the float32 weights;
// the block means of deeper stages are split in three. The matrix instructions
// round their sums down: an error of one direction, which the kernel gradients
// have to cancel (see wtconv_phase_grad.hip).
#pragma once

#include <type_traits>

#include "wtconv_fused.h"
#include "wtconv_phase_args.h"

namespace wtc {
namespace {

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) uint16_t u16x2;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// Matrix-core operand scheme of stage 0 by storage type.
template <typename ST>
struct Scheme;
template <>
struct Scheme<float> {
    static constexpr int NX = 3, NW = 3;
    static constexpr bool F16 = false;
};
template <>
struct Scheme<uint16_t> {
    static constexpr int NX = 1, NW = 3;
    static constexpr bool F16 = false;
};
template <>
struct Scheme<_Float16> {
    static constexpr int NX = 1, NW = 3;
    static constexpr bool F16 = true;
};
struct DeepScheme {  // stages >= 1, every storage type
    static constexpr int NX = 3, NW = 3;
    static constexpr bool F16 = false;
};

DEV uint32_t pk_bf16(float a, float b)
{
    const bf16x2 v = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, v);
}
DEV uint32_t pk_f16(float a, float b)
{
    const f16x2 v = {(_Float16)a, (_Float16)b};
    return __builtin_bit_cast(uint32_t, v);
}
DEV float bf_lo(uint32_t u) { return __uint_as_float(u << 16); }
DEV float bf_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// Two finite floats -> packed bfloat16 pieces h, m, l with v = h + m + l, exactly
// from 2^-110 on (below it l, then m, falls under bfloat16's smallest subnormal:
// an error of up to 2^-134). h is rounded, which halves m and with it what the
// dropped products leave out (2^-24.2 of a product at most over 2^24 random
// pairs; with h cut off 2^-23.2), but never to infinity: next to the largest
// float (a mask's lowest value) 0 * inf would reach outputs that do not depend on
// the pixel.
DEV void split2(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l)
{
    constexpr float top = 0x1.fep127f;  // the largest bfloat16
    h = pk_bf16(__builtin_amdgcn_fmed3f(a, -top, top), __builtin_amdgcn_fmed3f(b, -top, top));
    const float ra = a - bf_lo(h), rb = b - bf_hi(h);
    m = pk_bf16(ra, rb);
    l = pk_bf16(ra - bf_lo(m), rb - bf_hi(m));
}

// Mean of four values, finite for finite ones (their sum need not be).
DEV float mean4(float a, float b, float c, float d)
{
    return __builtin_fmaf(0.25f, d, __builtin_fmaf(0.25f, c, __builtin_fmaf(0.25f, b, 0.25f * a)));
}

template <bool F16>
DEV f32x4 mfma(u32x4 a, u32x4 b, f32x4 c)
{
    if constexpr (F16)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                      0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                       0, 0, 0);
}

// ----------------------------------------------------------------------------
// 4 x 4 pixel blocks as raw storage words. fetch_raw only loads, without a
// branch, from positions clamped into the plane, so that a batch's blocks
// stay in flight while the previous batch is computed (a load under a branch
// was waited for where the branches join); mask_raw then puts zeros in the
// place of the pixels outside.
// ----------------------------------------------------------------------------
template <typename ST>
struct RawBlock {
    static constexpr int NW = sizeof(ST);  // 32-bit words per row: 4 (float32) or 2 (16-bit pairs)
    uint32_t w[4][NW];
};

// Rows off, off + W, ... (elements, clamped to `last`) of the planes at `base`,
// W >= 4: one 16- or 8-byte load each at any element alignment (global loads
// take unaligned addresses).
template <typename ST>
DEV void fetch_raw(const ST* __restrict__ base, uint32_t off, uint32_t last, int W, RawBlock<ST>& v)
{
#pragma unroll
    for (int r = 0; r < 4; ++r)
        __builtin_memcpy(v.w[r], reinterpret_cast<const char*>(base) + (uint32_t)sizeof(ST) * min(off + r * W, last),
                         4 * sizeof(ST));
}

// edge = (-W) mod 4: how far the last block of a row reaches past the plane.
template <typename ST>
DEV void mask_raw(int H, int W, int y0, int x0, int edge, RawBlock<ST>& v)
{
    const bool shifted = x0 + 4 > W && x0 < W;  // the row was read from column W - 4
    const bool in_x = x0 >= 0 && x0 < W;
    if constexpr (sizeof(ST) == 4) {
        auto shift = [&](int r, auto e) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                v.w[r][c] = shifted ? (c + e.value < 4 ? v.w[r][(c + e.value) & 3] : 0u) : v.w[r][c];
        };
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (edge == 1) shift(r, std::integral_constant<int, 1>{});
            if (edge == 2) shift(r, std::integral_constant<int, 2>{});
            if (edge == 3) shift(r, std::integral_constant<int, 3>{});
        }
    } else {
        const int sh = shifted ? 16 * edge : 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint64_t u = (((uint64_t)v.w[r][1] << 32) | v.w[r][0]) >> sh;
            v.w[r][0] = (uint32_t)u;
            v.w[r][1] = (uint32_t)(u >> 32);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const bool in = in_x && y0 + r >= 0 && y0 + r < H;
#pragma unroll
        for (int i = 0; i < RawBlock<ST>::NW; ++i) v.w[r][i] = in ? v.w[r][i] : 0u;
    }
}

// Whether a block holds an infinity or NaN.
template <typename ST>
DEV bool nonfinite(const RawBlock<ST>& v)
{
    if constexpr (sizeof(ST) == 4) {
        float m = 0.f;  // maximum() keeps NaN
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                m = __builtin_elementwise_maximum(m, __builtin_fabsf(__uint_as_float(v.w[r][c])));
        return !(m < __builtin_inff());
    } else {
        constexpr uint16_t inf = Scheme<ST>::F16 ? 0x7c00 : 0x7f80;
        u16x2 m = {0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < 2; ++i)
                m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, v.w[r][i] & 0x7fff7fffu));
        return m.x >= inf || m.y >= inf;
    }
}

// Whether a block holds an infinity.
template <typename ST>
DEV bool infinite(const RawBlock<ST>& v)
{
    bool any = false;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < RawBlock<ST>::NW; ++i) {
            if constexpr (sizeof(ST) == 4) {
                any = any || (v.w[r][i] & 0x7fffffffu) == 0x7f800000u;
            } else {
                constexpr uint32_t inf = Scheme<ST>::F16 ? 0x7c00 : 0x7f80;
                any = any || (v.w[r][i] & 0x7fffu) == inf || ((v.w[r][i] >> 16) & 0x7fffu) == inf;
            }
        }
    return any;
}

// Zero the infinities and NaNs of row r, columns 2 j and 2 j + 1; whether
// there was one.
template <typename ST>
DEV bool drop_nonfinite(RawBlock<ST>& v, int r, int j)
{
    if constexpr (sizeof(ST) == 4) {
        const bool b0 = (v.w[r][2 * j] & 0x7f800000u) == 0x7f800000u;
        const bool b1 = (v.w[r][2 * j + 1] & 0x7f800000u) == 0x7f800000u;
        if (b0) v.w[r][2 * j] = 0;
        if (b1) v.w[r][2 * j + 1] = 0;
        return b0 || b1;
    } else {
        constexpr uint32_t inf = Scheme<ST>::F16 ? 0x7c00 : 0x7f80;
        const bool b0 = (v.w[r][j] & inf) == inf, b1 = ((v.w[r][j] >> 16) & inf) == inf;
        if (b0) v.w[r][j] &= 0xffff0000u;
        if (b1) v.w[r][j] &= 0x0000ffffu;
        return b0 || b1;
    }
}

// A raw block's values.
template <typename ST>
DEV void raw_values(const RawBlock<ST>& b, float (&v)[4][4])
{
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if constexpr (sizeof(ST) == 4)
                v[r][c] = __uint_as_float(b.w[r][c]);
            else
                v[r][c] = to_f32(__builtin_bit_cast(ST, (uint16_t)(b.w[r][c / 2] >> (16 * (c & 1)))));
        }
}

// Signed sum (band q of the Haar butterfly) of the 2^l x 2^l block (j, i) of a
// plane, zero-extended, at its true values.
template <typename ST>
DEV double block_sum(const ST* __restrict__ plane, int H, int W, int l, int q, int j, int i)
{
    const int half = 1 << (l - 1);
    double sum = 0.0;
#pragma unroll 1
    for (int y = j << l; y < min((j + 1) << l, H); y += 2)
#pragma unroll 1
        for (int x = i << l; x < min((i + 1) << l, W); x += 2) {
            double v[2][2];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int yy = y + (e >> 1), xx = x + (e & 1);
                const bool neg = ((q & 1) && (yy & half)) != ((q >> 1) && (xx & half));
                const double f = to_f32(plane[(long)min(yy, H - 1) * W + min(xx, W - 1)]);
                v[e >> 1][e & 1] = yy < H && xx < W ? (neg ? -f : f) : 0.0;
            }
            sum += (v[0][0] + v[0][1]) + (v[1][0] + v[1][1]);
        }
    return sum;
}

// ----------------------------------------------------------------------------
// weights
// ----------------------------------------------------------------------------
// The channel's folded kernels in float64 in LDS, where the tables are built
// from: s0 W0 [k k], then per level the four phase combinations
//   E[al][be] = 1/4 (LL +- LH +- HL +- HH), LH with the sign of al, HL of be,
// HH of al ^ be, [2][2][k k] (taps reversed with rot). The products of two
// float32 values and their sums are exact to float64. False if this thread met a
// kernel that is not finite.
template <int K>
constexpr int staged_doubles(int L) { return (1 + 4 * L) * K * K; }
template <int K>
DEV bool stage_kernels(const ParamPtrs& p, int c, int L, double* st, int tid)
{
    constexpr int KK = K * K;
    const bool rot = p.rot != 0;
    bool finite = true;
    for (int e = tid; e < (1 + L) * KK; e += kThreads) {
        const int l = e / KK, t = e - l * KK, tap = rot ? KK - 1 - t : t;
        if (l == 0) {
            st[t] = (double)p.s0[c] * p.w0[(long)c * KK + tap];
            finite = finite && __builtin_fabsf((float)st[t]) < __builtin_inff();
        } else {
            const float* w = p.lw[l - 1] + (long)4 * c * KK + tap;
            const float* s = p.ls[l - 1] + 4 * c;
            const double f0 = 0.25 * s[0] * w[0], f1 = 0.25 * s[1] * w[KK];
            const double f2 = 0.25 * s[2] * w[2 * KK], f3 = 0.25 * s[3] * w[3 * KK];
            const double m = (__builtin_fabs(f0) + __builtin_fabs(f1)) + (__builtin_fabs(f2) + __builtin_fabs(f3));
            finite = finite && (float)m < __builtin_inff();
            double* o = st + KK + 4 * (l - 1) * KK + t;
            o[0] = (f0 + f1) + (f2 + f3);
            o[KK] = (f0 + f1) - (f2 + f3);
            o[2 * KK] = (f0 - f1) + (f2 - f3);
            o[3 * KK] = (f0 - f1) - (f2 - f3);
        }
    }
    return finite;
}

// Coefficient of input column kc (counted from the tile's first column minus
// the margin) of window row (pr, ap) for output phase (a, cb) in the tile's
// first column pair: level s + 1's, and with `base` the base kernel's.
template <int K>
DEV double phase_coeff(const double* st, int s, bool base, int a, int cb, int pr, int ap, int kc)
{
    constexpr int R = K / 2, KK = K * K, M = kPhaseMargin;
    double v = 0.0;
    const int t = (kc >> 1) - M / 2 + R;
    if (t >= 0 && t < K) v = st[KK + (4 * s + 2 * (a ^ ap) + (cb ^ (kc & 1))) * KK + pr * K + t];
    if (base) {
        const int dy = 2 * pr + ap - R - a, dx = kc - M - cb + R;
        if (dy >= 0 && dy < K && dx >= 0 && dx < K) v += st[dy * K + dx];
    }
    return v;
}

// Table row of (a, cb, window row (pr, ap)). With the base kernel (BASE, stage
// 0) every (a, ap) has a row of its own; a stage of bands alone depends on
// a ^ ap only.
template <int K, bool BASE>
DEV int tab_row(int a, int cb, int pr, int ap)
{
    return BASE ? ((a * 2 + cb) * K + pr) * 2 + ap : ((a ^ ap) * 2 + cb) * K + pr;
}
template <int K, bool BASE>
constexpr int tab_rows() { return (BASE ? 8 : 4) * K; }

// Fill the table of stage s from the staged kernels: piece i at i * tab_rows *
// kPhaseTabPitch, row element u is the coefficient of input column kc = u - 6 (a
// tile's column pair j reads from u = 6 - 2 j on). A thread fills two elements.
// float16 pieces: `scale` (a power of two) takes the channel's largest
// coefficient to 2^14 or more, and the second and third piece are another 2^11
// larger (kF16Step). Together they hold 33 bits, and weights down to 2^-26 of the
// largest to float32's 24; below that the error is 2^-50 of the largest.
constexpr float kF16Step = 2048.f;
template <int K, bool BASE, bool F16>
DEV void fill_table(const double* st, int s, bool base, char* tab, float scale, int tid)
{
    constexpr int NR = tab_rows<K, BASE>(), P = kPhaseTabPitch / 2;
    uint32_t* t32 = reinterpret_cast<uint32_t*>(tab);
    for (int e = tid; e < NR * P; e += kThreads) {
        const int row = e / P, u = 2 * (e - row * P);
        int pa, cb, pr, ap;
        if (BASE) {
            ap = row & 1, pr = (row >> 1) % K, cb = (row / (2 * K)) & 1, pa = row / (4 * K);
        } else {
            ap = 0, pr = row % K, cb = (row / K) & 1, pa = row / (2 * K);
        }
        const double v0 = phase_coeff<K>(st, s, BASE && base, pa, cb, pr, ap, u - 6);
        const double v1 = phase_coeff<K>(st, s, BASE && base, pa, cb, pr, ap, u - 5);
        if constexpr (F16) {
            const double a = v0 * scale, b = v1 * scale;
            const uint32_t h = pk_f16((float)a, (float)b);
            const f16x2 hv = __builtin_bit_cast(f16x2, h);
            const float ra = (float)(a - (double)hv.x) * kF16Step, rb = (float)(b - (double)hv.y) * kF16Step;
            const uint32_t m = pk_f16(ra, rb);
            const f16x2 mv = __builtin_bit_cast(f16x2, m);
            t32[e] = h;
            t32[NR * P + e] = m;
            t32[2 * NR * P + e] = pk_f16(ra - (float)mv.x, rb - (float)mv.y);
        } else {
            const uint32_t h = pk_bf16((float)v0, (float)v1);
            const float ra = (float)(v0 - (double)bf_lo(h)), rb = (float)(v1 - (double)bf_hi(h));
            const uint32_t m = pk_bf16(ra, rb);
            t32[e] = h;
            t32[NR * P + e] = m;
            t32[2 * NR * P + e] = pk_bf16(ra - bf_lo(m), rb - bf_hi(m));
        }
    }
}

// The weight operand of one stage: fragment p holds window rows 2p, 2p + 1.
// Lane m = lane & 15 is output (a, column c) = (m >> 3, m & 7); the lane group
// lane >> 4 = (ap, seg) its eight input columns 8 seg .. 8 seg + 7 of row ap.
// Only fragments P0 .. P1 are loaded.
template <int K, bool BASE, int NW, int P0 = 0, int P1 = K - 1>
DEV void load_weights(const char* tab, int lane, u32x4 (&A)[K][3])
{
    constexpr int N = tab_rows<K, BASE>() * kPhaseTabPitch;
    const int a = (lane >> 3) & 1, c = lane & 7, ap = lane >> 5, seg = (lane >> 4) & 1;
    const int u = 8 * seg - 2 * (c >> 1) + 6;
#pragma unroll
    for (int p = P0; p <= P1; ++p)
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const uint32_t* t = reinterpret_cast<const uint32_t*>(
                tab + 2 * (i * N + tab_row<K, BASE>(a, c & 1, p, ap) * kPhaseTabPitch + u));
            A[p][i] = u32x4{t[0], t[1], t[2], t[3]};
        }
}

// ----------------------------------------------------------------------------
// one vertical run of JS tiles (row pairs) in each of the wavefront's 16
// columns: acc[J] += sum_p A[p] * window row pair J + p. off: this lane's
// first 16 bytes in LDS (its window row ap, columns 8 seg .. 8 seg + 7) of
// piece 0.
// ----------------------------------------------------------------------------
// With several pieces of x, and in float16, the products of the largest pieces
// come last, in a second pass over the rows: the small products then round against small sums,
// and only k roundings of full size are left (measured against 64 bits at k =
// 5, float32: 1.7e-7 with all products of a row together).
template <int K, int JS, typename SC, int NA, bool BIG, bool SMALL, bool WHOLE>
DEV void run_pass(const char* lds, int off, int rp_bytes, int psz, const u32x4 (&A)[K][3], f32x4 (&acc)[NA])
{
    constexpr int NX = SMALL ? SC::NX : 1;  // pieces read
    // row pairs read: with WHOLE (the run is the plane's whole height) only the
    // plane's own, the others are zero
    constexpr int R0 = WHOLE ? K / 2 : 0, N = WHOLE ? JS : JS + K - 1;
    // Rows in flight ahead of the products (no more: the scheduler would
    // otherwise hoist every read and spill). A row of the big pass alone is
    // few products, so it reads further ahead (k = 5: by one row less, for the
    // registers; 256 x 256 B8 C128 L3 f16 forward 271 -> 243 us).
    constexpr int D = NX > 1 ? 2 : (K > 3 ? 3 : 4);
    u32x4 b[D][NX];
    // (opaque: the runs of every length would share, and keep, their addresses)
    asm volatile("" : "+v"(off));
    if (R0) off += R0 * rp_bytes;
    auto read = [&](int r) {
#pragma unroll
        for (int i = 0; i < NX; ++i) b[r % D][i] = *reinterpret_cast<const u32x4*>(lds + off + i * psz);
        off += rp_bytes;
    };
#pragma unroll
    for (int r = 0; r < D - 1 && r < N; ++r) read(r);
#pragma unroll
    for (int r = 0; r < N; ++r) {
        if (r + D - 1 < N) read(r + D - 1);
#pragma unroll
        for (int i = NX - 1; i >= 0; --i)
#pragma unroll
            for (int j = SC::NW - 1; j >= 0; --j) {
                if (i + j > 2) continue;  // 2^-25 of the product or less each
                if (i + j == 0 ? !BIG : !SMALL) continue;
#pragma unroll
                for (int J = 0; J < JS; ++J) {
                    const int p = R0 + r - J;
                    if (p >= 0 && p < K) acc[J] = mfma<SC::F16>(A[p][j], b[r % D][i], acc[J]);
                }
            }
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int K, int JS, typename SC, int NA, bool WHOLE = false>
DEV void run_tiles(const char* lds, int off, int rp_bytes, int psz, const u32x4 (&A)[K][3], f32x4 (&acc)[NA])
{
    static_assert(JS <= NA, "");
    if constexpr (SC::NX > 1 || SC::F16) {
        run_pass<K, JS, SC, NA, false, true, WHOLE>(lds, off, rp_bytes, psz, A, acc);
        if constexpr (SC::F16) {  // (the small pieces are held kF16Step larger)
#pragma unroll
            for (int J = 0; J < JS; ++J) acc[J] *= 1.f / kF16Step;
        }
        run_pass<K, JS, SC, NA, true, false, WHOLE>(lds, off, rp_bytes, psz, A, acc);
    } else {
        run_pass<K, JS, SC, NA, true, true, WHOLE>(lds, off, rp_bytes, psz, A, acc);
    }
}

}  // namespace
}  // namespace wtc
