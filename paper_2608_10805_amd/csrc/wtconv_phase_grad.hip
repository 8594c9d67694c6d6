// Kernel gradients of WTConv on the gfx950 matrix cores (see wtconv_phase.h
// for the formulation).
//
// Stage s computes R_s = A_s * (windows of X_s): its 16 x (16 k) weight matrix
// maps the window of a 2 x 8 tile to the tile. The gradient of that matrix is
// the sum over all tiles of dR_s (tile) times X_s (window), a matrix product
// with the tiles as its contraction, 32 of them per v_mfma_f32_16x16x32. dR_s
// is the sum of dy over each 2^s x 2^s block, 4^s times the mean D_s. Summed
// over a workgroup's planes, the matrix is projected on the kernels: every
// tap of the base kernel and of each subband kernel is a signed sum of its
// entries (eq. foldgrad of Section 4.3 applied to the polyphase matrix).
//
// One workgroup (four wavefronts) owns channel c and a run of batch planes.
// Per batch of PP planes the threads turn their 4 x 4 blocks of x and dy into
// 16-bit pieces of the stages in LDS, row-major as in the forward; both
// operands are then read with the transposing LDS loads (ds_read_b64_tr_b16:
// four tiles' rows of 16 values become four values per lane of one column),
// and the fine wavefronts accumulate stage 0, the others the deeper stages.
// The accumulators stay in registers for the workgroup's life.
//
// 16-bit storage only: stage 0 is then one exact product per term (float32
// would take six). The vector pass is bound by FMA issue (56 x 56 B128 C96 L1
// bf16 104 us); here stage 0 is 10 matrix instructions per 512 pixels and the
// pass is bound by building the deeper stages (means, splits) and, at L >= 3,
// by the wavefront of stage 1. Training steps, vector / polyphase kernels on one
// card: 56 x 56 B128 C96 bf16 L1 287 -> 121 us, L3 397 -> 236, L5 471 -> 400; 14 x
// 14 B128 C384 L2 214 -> 101; 63 x 95 B32 C128 L3 477 -> 206; 224 x 224 B16 C64 L1
// (region tiles) 469 -> 210.
//
// The matrix instructions round their sums down, and a tap adds up many of them
// (the LL band 64): the odd rows of x are stored negated, so that half of the
// errors point up. Error of the kernel gradients against 64 bits 0.6-1.4e-7
// (vector pass 1.1-3.5e-7); 56 x 56 B128 C96 L3 levels 2 and 3 3.6e-7 and 4.1e-7
// without it, 1.2e-7 and 0.9e-7 with it (vector pass 3.5e-7 and 1.2e-7).
//
// The stages hold non-finite values as zeros; the workgroup sums the planes that
// have any once more at its end, tap by tap (plain_sum()).
#include "wtconv_phase.h"

namespace wtc {
namespace {

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// Transposing read: lane i of each 16 addresses four values of row i / 4
// (columns 4 (i % 4) ..), and receives column i of the four rows.
DEV uint2 read_tr(const char* p)
{
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p)));
}

// One run of JS row pairs in each of the wavefront's 32 tile columns:
//   acc[2 p + ap] += dy tiles (row pair J) * x window rows 2 (J + p) + ap.
// x0, x1 / d0, d1: byte offsets in LDS of the values this lane addresses for
// the transposing reads (tiles lane / 16 * 8 + lane % 16 / 4, and that + 4).
// mask: clears the tiles past the last one from the dy operand.
template <int K, int JS, int NX, int ND, bool F16, bool BIAS>
DEV void corr_run(const char* lds, int x0, int x1, int d0, int d1, int xrow, int xpsz, int drp, int dpsz, bool masked,
                  u32x4 mask, f32x4 (&acc)[2 * K], f32x4& accb)
{
    u32x4 d[JS][ND];
#pragma unroll
    for (int J = 0; J < JS; ++J)
#pragma unroll
        for (int i = 0; i < ND; ++i) {
            const uint2 u = read_tr(lds + d0 + J * drp + i * dpsz), v = read_tr(lds + d1 + J * drp + i * dpsz);
            d[J][i] = u32x4{u.x, u.y, v.x, v.y};
        }
    if (masked) {
#pragma unroll
        for (int J = 0; J < JS; ++J)
#pragma unroll
            for (int i = 0; i < ND; ++i) d[J][i] &= mask;
    }
    if constexpr (BIAS) {  // the sum of dy: one more column of ones
        const uint32_t one = F16 ? 0x3c003c00u : 0x3f803f80u;
#pragma unroll
        for (int i = ND - 1; i >= 0; --i)
#pragma unroll
            for (int J = 0; J < JS; ++J) accb = mfma<F16>(d[J][i], u32x4{one, one, one, one}, accb);
    }
    asm volatile("" : "+v"(x0), "+v"(x1));
#pragma unroll
    for (int r = 0; r < 2 * (JS + K - 1); ++r) {
        u32x4 b[NX];
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const uint2 u = read_tr(lds + x0 + i * xpsz), v = read_tr(lds + x1 + i * xpsz);
            b[i] = u32x4{u.x, u.y, v.x, v.y};
        }
        x0 += xrow;
        x1 += xrow;
#pragma unroll
        for (int J = 0; J < JS; ++J) {
            const int p = (r >> 1) - J;
            if (p < 0 || p >= K) continue;
            f32x4& o = acc[2 * p + (r & 1)];
            if constexpr (NX * ND == 1) {
                o = mfma<F16>(d[J][0], b[0], o);
            } else {
                // a term's piece products are summed on their own, smallest
                // first, so that the long-lived sums take one rounding each
                f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = NX - 1; i >= 0; --i)
#pragma unroll
                    for (int j = ND - 1; j >= 0; --j)
                        if (i + j <= 2) t = mfma<F16>(d[J][j], b[i], t);
                o += t;
            }
        }
    }
}

// Stage s of every resident plane by wavefronts w0 .. of nw of them.
template <int K, int JS, int NX, int ND, bool F16, bool BIAS>
DEV void corr_stage_js(const PhaseGradArgs& a, const char* lds, int s, int first, int step, int lane,
                       f32x4 (&acc)[2 * K], f32x4& accb)
{
    constexpr int R = K / 2, M = kPhaseMargin;
    asm volatile("" : "+v"(lane));  // no addresses kept across the batch loop
    const int vct = a.V[s] * a.ct[s], nslots = a.PP * vct;
    const int xp = 2 * a.sx.pitch[s], dp = 2 * a.sd.pitch[s];
    const int grp = lane >> 4, q = (lane & 15) >> 2, ch = lane & 3;
    for (int s0 = first; s0 < nslots; s0 += step) {
        int xo[2], d_o[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int slot = min(s0 + 8 * grp + 4 * e + q, nslots - 1);
            const int p = fdiv(slot, a.r_vct[s]), rem = slot - p * vct;
            const int v = fdiv(rem, a.r_ct[s]), I = rem - v * a.ct[s];
            const int row = 2 * v * JS;
            xo[e] = p * a.plane_bytes + a.sx.off[s] + (row + M - 2 * R) * xp + 2 * (8 * I + 4 * ch);
            d_o[e] = p * a.plane_bytes + a.sd.off[s] + (row + (ch >> 1)) * dp + 2 * (8 * I + 4 * (ch & 1));
        }
        const bool masked = s0 + 32 > nslots;
        u32x4 mask = {~0u, ~0u, ~0u, ~0u};
        if (masked) {
            const int left = nslots - s0 - 8 * grp;  // tiles of this lane's eight that exist
#pragma unroll
            for (int i = 0; i < 4; ++i)
                mask[i] = left >= 2 * i + 2 ? ~0u : (left >= 2 * i + 1 ? 0xffffu : 0u);
        }
        corr_run<K, JS, NX, ND, F16, BIAS>(lds, xo[0], xo[1], d_o[0], d_o[1], xp, a.sx.psz[s], 2 * dp, a.sd.psz[s], masked,
                                           mask, acc, accb);
    }
}

// A deeper stage (three pieces on both sides), by one wavefront.
template <int K>
DEV void corr_deep(const PhaseGradArgs& a, const char* lds, int s, int lane, f32x4 (&acc)[2 * K])
{
    f32x4 none = {0.f, 0.f, 0.f, 0.f};
    // (runs of two row pairs read fewer rows but spill: 14 x 14 L2 102.6 us
    // per training step against 97.8)
    corr_stage_js<K, 1, 3, 3, false, false>(a, lds, s, 0, 32, lane, acc, none);
}

// One block's pieces and block means on one side. With X (the x side) odd rows
// are stored negated, and project() turns their sums back: the matrix
// instructions round their sums down, and over the 64 entries that the LL band
// adds up these errors met in one direction (56 x 56 B128 C96 L3 bf16, kernel
// gradients of level 3 against 64 bits 4.1e-7, the vector pass 1.2e-7; B1024 C16
// L1 f16, level 1 4.2e-7 and 3.6e-7). Now half of them point the other way.
template <typename ST, bool DEEP, bool X>
DEV void put_side(const PhaseSide& g, int L, int w2, char* plane, int y0, int x0, const RawBlock<ST>& raw)
{
    const int M = g.margin;
    char* o = plane + g.off[0] + 2 * ((y0 + M) * g.pitch[0] + x0 + M);
#pragma unroll
    for (int r = 0; r < 4; ++r)
        *reinterpret_cast<uint2*>(o + 2 * r * g.pitch[0]) =
            X && r % 2 ? make_uint2(raw.w[r][0] ^ 0x80008000u, raw.w[r][1] ^ 0x80008000u)
                       : make_uint2(raw.w[r][0], raw.w[r][1]);
    if constexpr (!DEEP) return;
    float v[4][4];
    raw_values<ST>(raw, v);
    float s1[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
            s1[i][j] = mean4(v[2 * i][2 * j], v[2 * i][2 * j + 1], v[2 * i + 1][2 * j], v[2 * i + 1][2 * j + 1]);
        uint32_t h, m, l;
        const bool neg = X && i == 1;
        split2(neg ? -s1[i][0] : s1[i][0], neg ? -s1[i][1] : s1[i][1], h, m, l);
        char* q = plane + g.off[1] + 2 * (((y0 >> 1) + i + M) * g.pitch[1] + (x0 >> 1) + M);
        *reinterpret_cast<uint32_t*>(q) = h;
        *reinterpret_cast<uint32_t*>(q + g.psz[1]) = m;
        *reinterpret_cast<uint32_t*>(q + 2 * g.psz[1]) = l;
    }
    if (L < 3) return;
    const float s2 = mean4(s1[0][0], s1[0][1], s1[1][0], s1[1][1]);
    uint32_t h, m, l;
    split2(X && (y0 & 4) ? -s2 : s2, 0.f, h, m, l);
    uint16_t* q = reinterpret_cast<uint16_t*>(plane + g.off[2]) + ((y0 >> 2) + M) * g.pitch[2] + (x0 >> 2) + M;
    q[0] = (uint16_t)h;
    q[g.psz[2] / 2] = (uint16_t)m;
    q[g.psz[2]] = (uint16_t)l;
    if (L >= 4) reinterpret_cast<float*>(plane + g.mf[2])[(y0 >> 2) * w2 + (x0 >> 2)] = s2;
}

// The means of stage s >= 3 on one side, from stage s - 1's, by one wavefront.
template <bool X>
DEV void deepen_side(const PhaseGradArgs& a, const PhaseSide& g, char* lds, int s, int lane)
{
    asm volatile("" : "+v"(lane));
    const int h = a.h[s], w = a.w[s], ph = a.h[s - 1], pw = a.w[s - 1], per = h * w;
    const float r_per = 1.0f / (float)per, r_w = 1.0f / (float)w;
    for (int e = lane; e < a.PP * per; e += 64) {
        const int p = fdiv(e, r_per), r = e - p * per;
        const int j = fdiv(r, r_w), i = r - j * w;
        char* plane = lds + p * a.plane_bytes;
        const float* src = reinterpret_cast<const float*>(plane + g.mf[s - 1]) + 2 * j * pw + 2 * i;
        const bool bx = 2 * i + 1 < pw, by = 2 * j + 1 < ph;
        const float v00 = src[0], v01 = bx ? src[1] : 0.f;
        const float v10 = by ? src[pw] : 0.f, v11 = (bx && by) ? src[pw + 1] : 0.f;
        const float v = mean4(v00, v01, v10, v11);
        if (s + 1 < a.L) reinterpret_cast<float*>(plane + g.mf[s])[j * w + i] = v;
        uint32_t hh, m, l;
        split2(X && (j & 1) ? -v : v, 0.f, hh, m, l);
        uint16_t* o = reinterpret_cast<uint16_t*>(plane + g.off[s]) + (j + g.margin) * g.pitch[s] + i + g.margin;
        o[0] = (uint16_t)hh;
        o[g.psz[s] / 2] = (uint16_t)m;
        o[g.psz[s]] = (uint16_t)l;
    }
}

// Level-1 carrier sites of a 4 x 4 block at (y0, x0) of a plane: half of each
// 2 x 2 sum (pixels outside the plane are zero), rounded to the storage type;
// the sums and their order are the carrier kernel's.
template <typename ST>
DEV void put_carrier(ST* __restrict__ out, int H1, int W1, int y0, int x0, const RawBlock<ST>& raw)
{
    float v[4][4];
    raw_values<ST>(raw, v);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int j = (y0 >> 1) + a, i = (x0 >> 1) + b;
            if (j < H1 && i < W1) {
                const float s = (v[2 * a][2 * b] + v[2 * a][2 * b + 1]) + (v[2 * a + 1][2 * b] + v[2 * a + 1][2 * b + 1]);
                out[(long)j * W1 + i] = from_f32<ST>(__builtin_ldexpf(s, -1));
            }
        }
}

// Matrix-gradient entry of window row rho, window column kc, tile position m.
DEV int entry(int rho, int kc, int m) { return (rho * 16 + kc) * 16 + m; }

template <int K>
DEV void put_acc(float* cm, const f32x4 (&acc)[2 * K], int lane, bool add)
{
#pragma unroll
    for (int r = 0; r < 2 * K; ++r) {
        f32x4* o = reinterpret_cast<f32x4*>(cm + entry(r, lane & 15, 4 * (lane >> 4)));
        *o = add ? *o + acc[r] : acc[r];
    }
}

// Whether [p, p + n) holds an infinity or NaN, for a whole wavefront.
template <typename ST>
DEV bool any_nonfinite(const ST* __restrict__ p, long n, int lane)
{
#pragma unroll 1
    for (long i = 0; i < n; i += 64)
        if (__ballot(i + lane < n && !(__builtin_fabsf(to_f32(p[min(i + lane, n - 1)])) < __builtin_inff()))) return true;
    return false;
}

// One kernel-gradient sum per lane of a workgroup in plain arithmetic, over the
// pixels [ya, ye) x [xa, xe) of nplanes planes: tap (pr, t) of the base kernel
// (l = 0) or of band q of level l. The matrix products multiply the positions of
// a tile outside the plane, and every phase of a band, by themselves: an
// infinity or NaN in x or dy then reaches taps that do not pair with it, and the
// band's infinities cancel to NaN. Sums that came out non-finite (`bad`) are
// therefore formed again here, over the planes that hold such a value first:
// the others only count where the sum is finite without them. As in the vector
// kernels, dy meets the zeros around x (but on planes of at most 8 x 8, whose
// vector kernel skips them). Called by whole wavefronts; cold.
template <int K, typename ST>
DEV float plain_sum(const ST* __restrict__ x, const ST* __restrict__ dy, int H, int W, int ya, int ye, int xa, int xe,
                    int nplanes, long step, int l, int q, int pr, int t, bool bad, int lane)
{
    constexpr int R = K / 2;
    const bool halo = H > kTinyMaxEdge || W > kTinyMaxEdge;
    const int h = (H + (1 << l) - 1) >> l, w = (W + (1 << l) - 1) >> l;
    const int j0 = ya >> l, j1 = (ye + (1 << l) - 1) >> l, i0 = xa >> l, i1 = (xe + (1 << l) - 1) >> l;
    const int top = max(ya - 2 * R, 0), bottom = min(ye + 2 * R, H);  // rows of x that meet them (l <= 1 in regions)
    double sum = 0.0;
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
        const bool open = bad && __builtin_fabs(sum) < __builtin_inf();
        if (__ballot(open) == 0) break;
#pragma unroll 1
        for (int b = 0; b < nplanes; ++b) {
            const ST *xb = x + b * step, *db = dy + b * step;
            const bool first = any_nonfinite<ST>(xb + (long)top * W, (long)(bottom - top) * W, lane) ||
                               any_nonfinite<ST>(db + (long)ya * W, (long)(ye - ya) * W, lane);
            if (first == (pass != 0) || !open) continue;
#pragma unroll 1
            for (int j = j0; j < j1; ++j) {
                const int u = j + pr - R;
                const bool row = u >= 0 && u < h;
                if (sum != sum || (!row && !halo)) continue;
                if (l == 0) {
#pragma unroll 4
                    for (int i = i0; i < i1; ++i) {
                        const int v = i + t - R;
                        const bool in = row && v >= 0 && v < w;
                        const double d = to_f32(db[(long)j * W + i]);
                        const double m = to_f32(xb[(long)min(max(u, 0), h - 1) * W + min(max(v, 0), w - 1)]);
                        if (in || halo) sum += d * (in ? m : 0.0);
                    }
                } else {
#pragma unroll 1
                    for (int i = i0; i < i1; ++i) {
                        const int v = i + t - R;
                        const bool in = row && v >= 0 && v < w;
                        if (!in && !halo) continue;
                        const double m = in ? block_sum<ST>(xb, H, W, l, q, u, v) : 0.0;
                        sum += block_sum<ST>(db, H, W, l, q, j, i) * m;
                    }
                }
            }
        }
    }
    return (float)sum;
}

// Wavefronts per SIMD: three, but two for two block rounds on both sides or
// with two stages' accumulators in one wavefront (L = 4 and 5).
template <int NR, int ND>
constexpr int grad_waves() { return ND > 2 || NR == 2 ? 2 : 3; }

// NR: rounds of 4 x 4 blocks per thread and side. ND: deeper stages (0: L = 1,
// 1: L = 2, 2: L = 3, 4: L = 4 and 5).
template <int K, typename ST, int NR, bool RGN, int ND>
__global__ void __launch_bounds__(kThreads, (grad_waves<NR, ND>())) phase_grad_kernel(const PhaseGradArgs a)
{
    using SC = Scheme<ST>;
    constexpr int R = K / 2, M = kPhaseMargin, KK = K * K;
    static_assert(SC::NX == 1, "16-bit storage");
    constexpr int JS0 = 4;  // row pairs per run of stage 0
    constexpr bool DEEP = ND > 0;
    extern __shared__ float4 lds4[];
    char* lds = reinterpret_cast<char*>(lds4);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int C = a.C, H = a.H, W = a.W, HW = H * W;
    const int c = (int)blockIdx.x % C, ct = (int)blockIdx.x / C;
    const int ntiles = RGN ? a.rg_ntx * a.rg_nty : 1;
    const int chunk = ct / ntiles, tile = ct - chunk * ntiles;
    const int b_begin = chunk * a.nb, b_end = min(a.B, b_begin + a.nb);
    const int oy = RGN ? (tile / a.rg_ntx) * a.rg_T : 0;
    const int ox = RGN ? (tile % a.rg_ntx) * a.rg_T : 0;
    const int top = RGN ? 4 : 0;
    const ST* xs = reinterpret_cast<const ST*>(a.x);
    const ST* ds = reinterpret_cast<const ST*>(a.dy);

    // this thread's blocks of x and dy: as in the forward kernel
    RawBlock<ST> vx[NR], vd[NR];
    int xp[NR], xy[NR], xx[NR], dp[NR], dy[NR], dx[NR];
    uint32_t xoff[NR], xlast[NR], doff[NR], dlast[NR];
    const int nxb = a.xbx * a.xby, ndb = a.dbx * a.dby;
    auto place = [&](int e, int nblk, int bx, float r_b, float r_bx, int margin, int& p, int& y0, int& x0, uint32_t& off,
                     uint32_t& last) {
        p = fdiv(e, r_b);
        const int r = e - p * nblk, j = fdiv(r, r_bx);
        y0 = 4 * j - margin;
        x0 = 4 * (r - j * bx) - margin;
        const int yc = min(max(oy + y0, 0), H - 1), xc = min(max(ox + x0, 0), W - 4);
        const uint32_t pb = (uint32_t)min(p, a.PP - 1) * C * HW;
        off = pb + yc * W + xc;
        last = pb + (H - 1) * W + xc;
    };
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        place(tid + i * kThreads, nxb, a.xbx, a.r_xb, a.r_xbx, top, xp[i], xy[i], xx[i], xoff[i], xlast[i]);
        if constexpr (RGN)
            place(tid + i * kThreads, ndb, a.dbx, a.r_db, a.r_dbx, 0, dp[i], dy[i], dx[i], doff[i], dlast[i]);
    }
    auto fetch = [&](int b0) {
        if (b0 >= b_end) return;
        const long base = ((long)b0 * C + c) * HW;
        const bool part = b0 + a.PP > b_end;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            uint32_t off = xoff[i], last = xlast[i];
            if (part && b0 + xp[i] >= b_end) off = last = 0;
            fetch_raw<ST>(xs + base, off, last, W, vx[i]);
            if constexpr (RGN)
                fetch_raw<ST>(ds + base, doff[i], dlast[i], W, vd[i]);
            else
                fetch_raw<ST>(ds + base, off, last, W, vd[i]);
        }
    };
    const int edge = (4 - (W & 3)) & 3;
    const bool ragged = RGN || edge != 0 || (H & 3) != 0;
    const int ye = RGN ? min(oy + a.rg_T, H) : H, xe = RGN ? min(ox + a.rg_T, W) : W;
    auto put = [&](int b0) {
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            int y0 = xy[i], x0 = xx[i];
            asm volatile("" : "+v"(y0), "+v"(x0));  // no per-row addresses kept across the batch loop
            if (xp[i] < a.PP) {
                char* plane = lds + xp[i] * a.plane_bytes;
                const bool have = b0 + xp[i] < b_end;
                if (have) {
                    if (ragged) mask_raw<ST>(H, W, oy + y0, ox + x0, edge, vx[i]);
                    put_side<ST, DEEP, true>(a.sx, a.L, a.w[ND > 1 ? 2 : 0], plane, y0, x0, vx[i]);
                    if constexpr (RGN)
                        if (a.cx && y0 >= 0 && y0 < a.rg_T && x0 >= 0 && x0 < a.rg_T)
                            put_carrier<ST>(reinterpret_cast<ST*>(a.cx) + ((long)(b0 + xp[i]) * C + c) * a.cH * a.cW,
                                            a.cH, a.cW, oy + y0, ox + x0, vx[i]);
                }
                if constexpr (!RGN) {
                    if (have) {
                        if (ragged) mask_raw<ST>(H, W, y0, x0, edge, vd[i]);
                    } else {  // a last, partial batch: planes that do not exist count nothing
#pragma unroll
                        for (int r = 0; r < 4; ++r)
#pragma unroll
                            for (int j = 0; j < RawBlock<ST>::NW; ++j) vd[i].w[r][j] = 0;
                    }
                    put_side<ST, DEEP, false>(a.sd, a.L, a.w[ND > 1 ? 2 : 0], plane, y0, x0, vd[i]);
                }
            }
            if constexpr (RGN) {
                int v0 = dy[i], u0 = dx[i];
                asm volatile("" : "+v"(v0), "+v"(u0));
                if (dp[i] < 1) {
                    mask_raw<ST>(H, W, oy + v0, ox + u0, edge, vd[i]);
                    put_side<ST, false, false>(a.sd, 1, 0, lds, v0, u0, vd[i]);
                    if (a.cdy)
                        put_carrier<ST>(reinterpret_cast<ST*>(a.cdy) + ((long)b0 * C + c) * a.cH * a.cW, a.cH, a.cW,
                                        oy + v0, ox + u0, vd[i]);
                }
            }
        }
    };

    fetch(b_begin);
    for (int i = tid; i < a.lds_bytes / 16; i += kThreads) lds4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();

    const int NP = partial_floats_per_channel(K, a.L);
    float* dst = a.partial + ((long)ct * C + c) * NP;
    float* cm = reinterpret_cast<float*>(lds);
    // Stage s's matrix gradient in cm -> its kernel gradients. Thread (q, tap):
    // band q of level s + 1; the last k k threads the base taps (stage 0).
    auto project = [&](int s) {
        for (int e0 = 64 * wave; e0 < 5 * KK; e0 += kThreads) {
            const int e = e0 + lane, q = e / KK, tap = e - q * KK, pr = tap / K, t = tap - pr * K;
            const bool band = q < 4, base = q == 4 && s == 0;
            double sum = 0.0;  // (64 terms: their rounding would show)
            if (band) {
                for (int m = 0; m < 16; ++m) {
                    const int pa = m >> 3, cb = m & 1, kc = 2 * (t + M / 2 - R + ((m & 7) >> 1));
                    for (int ap = 0; ap < 2; ++ap)
                        for (int be = 0; be < 2; ++be) {
                            const float v = cm[entry(2 * pr + ap, kc + be, m)];
                            const int neg = ((q & 1) & (pa ^ ap)) ^ ((q >> 1) & (cb ^ be)) ^ ap;
                            sum += neg ? -v : v;
                        }
                }
            } else if (base) {
                for (int m = 0; m < 16; ++m) {
                    const float v = cm[entry(pr + R + (m >> 3), t + M - R + (m & 7), m)];
                    sum += (pr + R + (m >> 3)) & 1 ? -v : v;
                }
                if (a.skip_base) sum = 0.0;
            }
            float g = band ? __builtin_ldexpf((float)sum, 4 * s) : (float)sum;
            const bool bad = !(__builtin_fabsf(g) < __builtin_inff());
            if (__builtin_expect(__ballot(bad) != 0, 0)) {
                const long at = ((long)b_begin * C + c) * HW;
                const float v = plain_sum<K, ST>(xs + at, ds + at, H, W, oy, ye, ox, xe, b_end - b_begin, (long)C * HW,
                                                 band ? s + 1 : 0, q, pr, t, bad, lane);
                g = bad ? v : g;
            }
            if (band)
                dst[KK + (4 * s + q) * KK + tap] = g;
            else if (base)
                dst[tap] = g;
        }
    };
    const bool fine = !DEEP || wave < a.fine_waves;

    if (fine) {
        // a batch's sums are formed on their own and then added: the chains stay
        // short, and the error below the vector kernels'
        f32x4 tot[2 * K], totb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 2 * K; ++r) tot[r] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int b0 = b_begin; b0 < b_end; b0 += a.PP) {
            put(b0);
            __syncthreads();
            fetch(b0 + a.PP);
            f32x4 acc[2 * K], accb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < 2 * K; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
            corr_stage_js<K, JS0, 1, 1, SC::F16, true>(a, lds, 0, 32 * wave, 32 * a.fine_waves, lane, acc, accb);
#pragma unroll
            for (int r = 0; r < 2 * K; ++r) tot[r] += acc[r];
            totb += accb;
            __syncthreads();
        }
        // the fine wavefronts' sums, added in their order
        for (int w = 0; w < a.fine_waves; ++w) {
            if (w == wave) put_acc<K>(cm, tot, lane, w > 0);
            __syncthreads();
        }
        project(0);
        float sb = (totb[0] + totb[1]) + (totb[2] + totb[3]);
        sb += __shfl_xor(sb, 16, 64);
        sb += __shfl_xor(sb, 32, 64);
        __syncthreads();
        if (lane == 0) cm[wave] = sb;
        __syncthreads();
        if (tid == 0) {
            float t = cm[0];
            for (int w = 1; w < a.fine_waves; ++w) t += cm[w];
            dst[NP - 1] = t;
        }
        if constexpr (DEEP) {
            for (int s = 1; s < a.L; ++s) {
                __syncthreads();
                __syncthreads();  // (a deeper wavefront writes its stage between the two)
                project(s);
            }
        }
    } else if constexpr (DEEP) {
        // one wavefront per deeper stage; with ND = 4 the last takes two
        const int lo = wave - a.fine_waves + 1;
        constexpr int NS = ND > 2 ? 2 : 1;
        f32x4 acc[NS][2 * K];
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
            for (int r = 0; r < 2 * K; ++r) acc[i][r] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int b0 = b_begin; b0 < b_end; b0 += a.PP) {
            put(b0);
            __syncthreads();
            fetch(b0 + a.PP);
            if (lo < 3) {
                corr_deep<K>(a, lds, lo, lane, acc[0]);
            } else if constexpr (ND > 2) {
#pragma unroll
                for (int i = 0; i < NS; ++i)
                    if (3 + i < a.L) {
                        asm volatile("" ::: "memory");
                        deepen_side<true>(a, a.sx, lds, 3 + i, lane);
                        deepen_side<false>(a, a.sd, lds, 3 + i, lane);
                        asm volatile("" ::: "memory");
                        corr_deep<K>(a, lds, 3 + i, lane, acc[i]);
                    }
            }
            __syncthreads();
        }
        for (int w = 0; w < a.fine_waves; ++w) __syncthreads();
        project(0);
        __syncthreads();
        __syncthreads();
        for (int s = 1; s < a.L; ++s) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NS; ++i)
                if (s == lo + i && (i == 0 || lo == 3)) put_acc<K>(cm, acc[i], lane, false);
            __syncthreads();
            project(s);
        }
    }
}

template <int K, typename ST, int NR, bool RGN, int ND>
hipError_t launch_v(const PhaseGradArgs& a, int grid, hipStream_t s)
{
    static std::atomic<unsigned long long> lds_done{0};
    const hipError_t e = allow_full_lds(reinterpret_cast<const void*>(&phase_grad_kernel<K, ST, NR, RGN, ND>), lds_done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((phase_grad_kernel<K, ST, NR, RGN, ND>), dim3(grid), dim3(kThreads), a.lds_bytes, s, a);
    return hipGetLastError();
}

template <int K, typename ST, int NR>
hipError_t launch_l(const PhaseGradArgs& a, int grid, hipStream_t s)
{
    switch (a.L) {
        case 1: return launch_v<K, ST, NR, false, 0>(a, grid, s);
        case 2: return launch_v<K, ST, NR, false, 1>(a, grid, s);
        case 3: return launch_v<K, ST, NR, false, 2>(a, grid, s);
        case 4:
        case 5: return launch_v<K, ST, NR, false, 4>(a, grid, s);
    }
    return hipErrorInvalidValue;
}

template <int K, typename ST>
hipError_t launch_t(const PhaseGradArgs& a, int grid, int rounds, hipStream_t s)
{
    if (a.rg_ntx > 0) return launch_v<K, ST, 1, true, 0>(a, grid, s);
    return rounds > 1 ? launch_l<K, ST, 2>(a, grid, s) : launch_l<K, ST, 1>(a, grid, s);
}

template <int K>
hipError_t launch_k(wtconv_dtype dt, const PhaseGradArgs& a, int grid, int rounds, hipStream_t s)
{
    switch (dt) {
        case WTCONV_F32: break;  // (not offered)
        case WTCONV_BF16: return launch_t<K, uint16_t>(a, grid, rounds, s);
        case WTCONV_F16: return launch_t<K, _Float16>(a, grid, rounds, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_phase_grad(int k, wtconv_dtype dt, const PhaseGradArgs& a, int grid, int block_rounds, hipStream_t s)
{
    switch (k) {
        case 3: return launch_k<3>(dt, a, grid, block_rounds, s);
        case 5: return launch_k<5>(dt, a, grid, block_rounds, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace wtc
