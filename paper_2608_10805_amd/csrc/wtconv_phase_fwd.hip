// Polyphase forward of WTConv on the gfx950 matrix cores (see wtconv_phase.h
// for the formulation). With rotated taps it is dx.
//
// One workgroup (four wavefronts) owns channel c and a run of batch planes, PP
// of them resident. Per batch:
//   1. every thread turns its prefetched 4 x 4 pixel blocks into 16-bit pieces
//      of X_0 and of the block means X_1, X_2 (float32 sums) in LDS;
//   2. the next batch's blocks are requested; the fine wavefronts run stage 0
//      over their columns of tiles and keep the sums in registers, while the
//      fourth wavefront (when L > 1) runs the deeper stages, coarsest first,
//      each adding the coarser result, into a float32 array in LDS;
//   3. the fine wavefronts add the coarse result and store y.
// Two barriers per batch.
//
// What bounds it, and why this split. The vector kernels issue k^2 (1 + c(L))
// FMAs per pixel and are bound by that issue (56 x 56 B128 C96 k5 L1 bf16 115
// us). Here a 2 x 8 tile is k matrix instructions of 16 cycles per operand
// pair for 16 tiles: 62 % of the weight matrix is non-zero at k = 5, and a
// third of the vector kernels' VALU instructions remain (splitting the
// pixels, addresses, the epilogue). Tiles of 16 columns would be 42 % full; a
// run of row pairs keeps its sums in registers and reads each window row
// once. 16-bit storage (three operand pairs per term: the weight's pieces) ends
// up between the VALU and HBM, vector / polyphase on one card: 56 x 56 B128 C96
// L1 bf16 94.5 -> 48 us (3.2 TB/s of algorithmic traffic), L3 118 -> 77, L5 133
// -> 113, 63 x 95 B32 C128 L3 142 -> 70. float16 sums its pieces in two passes
// and pays for it in registers: 56 x 56 B128 C96 L1 89 -> 44, 256 x 256 B8 C128
// L3 371 -> 233. In float32 (six pairs) matrix and VALU time are about equal and
// share the SIMDs: 63 x 95 L3 127 -> 87 (one launch, rows of odd width in whole
// 16-byte loads), 48 x 48 B64 C96 L3 60 -> 49, 128 x 128 B8 C64 L1 42 -> 30.
//
// A tile's window holds zeros of the weight matrix next to its taps, and
// 0 * inf is NaN: a non-finite input pixel would reach every output of the
// tiles whose window holds it. Such pixels are zeroed and marked as they are
// loaded, and the outputs that depend on one, and only they, become NaN. Where
// one was an infinity (or a kernel of the channel is not finite), the workgroup
// goes over these outputs once more at its end: an infinity remains where every
// term of it has the same sign.
#include "wtconv_phase.h"

namespace wtc {
namespace {

// Deeper stage s of every resident plane, by one wavefront; carry: on top of
// stage s + 1's result, which this wavefront formed.
template <int K, int JS, bool WHOLE = false>
DEV void coarse_stage_js(const PhaseArgs& a, char* lds, int s, bool carry, int lane, const u32x4 (&A)[K][3])
{
    constexpr int R = K / 2, M = kPhaseMargin;
    const PhaseStage& g = a.st[s];
    asm volatile("" : "+v"(lane));  // no addresses kept across the batch loop
    const int n = lane & 15, grp = lane >> 4;
    const int vct = g.V * g.ct, nslots = a.PP * vct;
    const int jt = (g.h + 1) >> 1;
    for (int s0 = 0; s0 < nslots; s0 += 16) {
        const bool live = s0 + n < nslots;
        const int slot = live ? s0 + n : 0;
        const int p = fdiv(slot, g.r_vct), rem = slot - p * vct;
        const int v = fdiv(rem, g.r_ct), I = rem - v * g.ct;
        char* plane = lds + a.planes_off + p * a.plane_bytes;
        const int J0 = v * JS;
        const int bp = a.planes_off + p * a.plane_bytes + g.poff +
                       2 * ((2 * J0 + M - 2 * R + (grp >> 1)) * g.pitch + 8 * I + 8 * (grp & 1));
        f32x4 acc[JS];
#pragma unroll
        for (int J = 0; J < JS; ++J) {
            if (carry) {
                const PhaseStage& gn = a.st[s + 1];
                const int j = min(J0 + J, jt - 1);
                const float2 r = *reinterpret_cast<const float2*>(plane + gn.roff +
                                                                  4 * (j * gn.rpitch + 4 * I + 2 * (grp & 1)));
                acc[J] = f32x4{r.x, r.x, r.y, r.y};
            } else {
                acc[J] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
        run_tiles<K, JS, DeepScheme, JS, WHOLE>(lds, bp, 4 * g.pitch, g.psz, A, acc);
        const int x = 8 * I + 4 * (grp & 1);
#pragma unroll
        for (int J = 0; J < JS; ++J)
            if (live)
                *reinterpret_cast<f32x4*>(plane + g.roff + 4 * ((2 * (J0 + J) + (grp >> 1)) * g.rpitch + x)) = acc[J];
    }
}

// Stage s with its weights in A (all fragments).
template <int K>
DEV void coarse_stage(const PhaseArgs& a, char* lds, int s, bool carry, int lane, const u32x4 (&A)[K][3])
{
    if (a.st[s].js == 1)
        coarse_stage_js<K, 1>(a, lds, s, carry, lane, A);
    else if (a.st[s].js == 2)
        coarse_stage_js<K, 2>(a, lds, s, carry, lane, A);
    else
        coarse_stage_js<K, 4>(a, lds, s, carry, lane, A);
}

// Stage s, reading its weights anew. A grid of at most four rows is one run
// over its own rows alone, with the few fragments those meet.
template <int K>
DEV void coarse_stage_load(const PhaseArgs& a, char* lds, int s, bool carry, int lane)
{
    constexpr int R = K / 2;
    const PhaseStage& g = a.st[s];
    u32x4 A[K][3];
    if (g.h <= 2) {
        load_weights<K, false, 3, R, R>(lds + g.tab, lane, A);
        coarse_stage_js<K, 1, true>(a, lds, s, carry, lane, A);
    } else if (g.h <= 4) {
        load_weights<K, false, 3, R - 1, R + 1>(lds + g.tab, lane, A);
        coarse_stage_js<K, 2, true>(a, lds, s, carry, lane, A);
    } else {
        load_weights<K, false, 3>(lds + g.tab, lane, A);
        coarse_stage<K>(a, lds, s, carry, lane, A);
    }
}

// X_s of every resident plane for s >= 3 (float32 block means of X_{s-1},
// zero-extended), by one wavefront.
DEV void build_deep(const PhaseArgs& a, char* lds, int s, int lane)
{
    const PhaseStage& g = a.st[s];
    const PhaseStage& gp = a.st[s - 1];
    asm volatile("" : "+v"(lane));
    const int per = g.h * g.w;
    const float r_per = 1.0f / (float)per, r_w = 1.0f / (float)g.w;
    for (int e = lane; e < a.PP * per; e += 64) {
        const int p = fdiv(e, r_per), r = e - p * per;
        const int j = fdiv(r, r_w), i = r - j * g.w;
        char* plane = lds + a.planes_off + p * a.plane_bytes;
        const float* src = reinterpret_cast<const float*>(plane + gp.mf) + 2 * j * gp.w + 2 * i;
        const bool bx = 2 * i + 1 < gp.w, by = 2 * j + 1 < gp.h;
        const float v00 = src[0], v01 = bx ? src[1] : 0.f;
        const float v10 = by ? src[gp.w] : 0.f, v11 = (bx && by) ? src[gp.w + 1] : 0.f;
        const float v = mean4(v00, v01, v10, v11);
        if (s + 1 < a.L) reinterpret_cast<float*>(plane + g.mf)[j * g.w + i] = v;
        uint32_t h, m, l;
        split2(v, 0.f, h, m, l);
        uint16_t* o = reinterpret_cast<uint16_t*>(plane + g.poff) + (j + kPhaseMargin) * g.pitch + i + kPhaseMargin;
        o[0] = (uint16_t)h;
        o[g.psz / 2] = (uint16_t)m;
        o[g.psz] = (uint16_t)l;
    }
}

template <typename ST>
DEV uint32_t pk_storage(float a, float b)
{
    if constexpr (sizeof(ST) == 2 && Scheme<ST>::F16)
        return pk_f16(a, b);
    else
        return pk_bf16(a, b);
}

// One loaded 4 x 4 block -> the pieces of X_0, X_1 and X_2 of its plane.
template <typename ST, bool DEEP>
DEV void put_block(const PhaseArgs& a, char* plane, int y0, int x0, const RawBlock<ST>& raw)
{
    constexpr int M = kPhaseMargin;
    const PhaseStage& g = a.st[0];
    char* o = plane + g.poff + 2 * ((y0 + M) * g.pitch + x0 + M);
    if constexpr (Scheme<ST>::NX == 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r)  // the storage type's own values
            *reinterpret_cast<uint2*>(o + 2 * r * g.pitch) = make_uint2(raw.w[r][0], raw.w[r][1]);
        if constexpr (!DEEP) return;
    }
    float v[4][4];
    raw_values<ST>(raw, v);
    if constexpr (Scheme<ST>::NX == 3) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            uint2 h, m, l;
            split2(v[r][0], v[r][1], h.x, m.x, l.x);
            split2(v[r][2], v[r][3], h.y, m.y, l.y);
            *reinterpret_cast<uint2*>(o) = h;
            *reinterpret_cast<uint2*>(o + g.psz) = m;
            *reinterpret_cast<uint2*>(o + 2 * g.psz) = l;
            o += 2 * g.pitch;
            __builtin_amdgcn_sched_barrier(0);  // row by row, within the register budget
        }
    }
    if constexpr (!DEEP) return;
    const PhaseStage& g1 = a.st[1];
    float s1[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
            s1[i][j] = mean4(v[2 * i][2 * j], v[2 * i][2 * j + 1], v[2 * i + 1][2 * j], v[2 * i + 1][2 * j + 1]);
        uint32_t h, m, l;
        split2(s1[i][0], s1[i][1], h, m, l);
        char* q = plane + g1.poff + 2 * (((y0 >> 1) + i + M) * g1.pitch + (x0 >> 1) + M);
        *reinterpret_cast<uint32_t*>(q) = h;
        *reinterpret_cast<uint32_t*>(q + g1.psz) = m;
        *reinterpret_cast<uint32_t*>(q + 2 * g1.psz) = l;
    }
    if (a.L < 3) return;
    const PhaseStage& g2 = a.st[2];
    const float s2 = mean4(s1[0][0], s1[0][1], s1[1][0], s1[1][1]);
    uint32_t h, m, l;
    split2(s2, 0.f, h, m, l);
    uint16_t* q = reinterpret_cast<uint16_t*>(plane + g2.poff) + ((y0 >> 2) + M) * g2.pitch + (x0 >> 2) + M;
    q[0] = (uint16_t)h;
    q[g2.psz / 2] = (uint16_t)m;
    q[g2.psz] = (uint16_t)l;
    if (a.L >= 4) reinterpret_cast<float*>(plane + g2.mf)[(y0 >> 2) * g2.w + (x0 >> 2)] = s2;
}

// Four outputs of one lane at element `off` of the planes at `base`, the first
// of them column x, cropped to column xe.
template <typename ST>
DEV void store4(ST* __restrict__ base, uint32_t off, int x, int xe, const float (&v)[4])
{
    ST* q = reinterpret_cast<ST*>(reinterpret_cast<char*>(base) + (uint32_t)sizeof(ST) * off);
    if (x + 4 <= xe) {  // one 16- or 8-byte store at any element alignment
        if constexpr (sizeof(ST) == 4) {
            __builtin_memcpy(q, v, 16);
        } else {
            const uint32_t u[2] = {pk_storage<ST>(v[0], v[1]), pk_storage<ST>(v[2], v[3])};
            __builtin_memcpy(q, u, 8);
        }
    } else {
#pragma unroll
        for (int c = 0; c < 3; ++c)
            if (x + c < xe) q[c] = from_f32<ST>(v[c]);
    }
}

// Marks of non-finite input pixels (LDS, 16-bit): one per resident plane, then
// one per cell of its loaded blocks (2 x 2 pixels for L = 1, else 4 x 4). A
// mark holds twice the number of the last batch that set it, so nothing is
// cleared, plus one if the batch before set it too: a wavefront may mark batch
// n + 1 while another still stores batch n (never n - 1: two barriers apart).
DEV void set_mark(uint16_t& m, uint16_t epoch)
{
    const int last = m >> 1;
    if (last != epoch) m = (uint16_t)(2 * epoch + (last + 1 == epoch));
}
DEV bool marked(uint16_t m, uint16_t epoch) { return (m >> 1) == epoch || m == 2 * (epoch + 1) + 1; }
DEV int mark_cells(const PhaseArgs& a) { return a.L == 1 ? 4 * a.bx * a.by : a.bx * a.by; }
// After the marks: whether any batch so far held an infinity, or the channel has
// a kernel that is not finite.
DEV uint16_t& infinity_flag(const PhaseArgs& a, char* lds)
{
    return reinterpret_cast<uint16_t*>(lds + a.mark_off)[a.PP * (1 + mark_cells(a))];
}

// Zeroes the non-finite pixels of block e of plane p and marks their cells.
template <typename ST>
DEV void mark_block(const PhaseArgs& a, char* lds, int p, int e, uint16_t epoch, RawBlock<ST>& v)
{
    uint16_t* marks = reinterpret_cast<uint16_t*>(lds + a.mark_off);
    uint16_t* cell = marks + a.PP + p * mark_cells(a);
    set_mark(marks[p], epoch);
    if (infinite<ST>(v)) infinity_flag(a, lds) = 1;
    const int j = fdiv(e, a.r_bx), i = e - j * a.bx;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (drop_nonfinite<ST>(v, r, h))
                set_mark(cell[a.L == 1 ? (2 * j + (r >> 1)) * 2 * a.bx + 2 * i + h : e], epoch);
}

// Whether a pixel (in the loaded area's coordinates) depends on a marked one:
// on the 2^L x 2^L blocks within k / 2 of its own.
DEV bool depends_on_mark(const PhaseArgs& a, const char* lds, int R, int p, int y, int x, uint16_t epoch)
{
    const int sh = a.L == 1 ? 1 : 2, L = a.L;
    const int cw = a.L == 1 ? 2 * a.bx : a.bx, ch = a.L == 1 ? 2 * a.by : a.by;
    const uint16_t* cell = reinterpret_cast<const uint16_t*>(lds + a.mark_off) + a.PP + p * mark_cells(a);
    const int j0 = max((((y >> L) - R) << L) >> sh, 0), j1 = min(((((y >> L) + R + 1) << L) - 1) >> sh, ch - 1);
    const int i0 = max((((x >> L) - R) << L) >> sh, 0), i1 = min(((((x >> L) + R + 1) << L) - 1) >> sh, cw - 1);
#pragma unroll 1
    for (int j = j0; j <= j1; ++j)
#pragma unroll 1
        for (int i = i0; i <= i1; ++i)
            if (marked(cell[j * cw + i], epoch)) return true;
    return false;
}

// Terms of the operator that pixel (py, px) of value f (an infinity or NaN)
// adds to output (y, x), as the vector kernels multiply and add them: bit 0,
// +inf among them; bit 1, -inf; both, NaN.
template <int K>
DEV int nonfinite_terms(const PhaseArgs& a, int c, float f, int py, int px, int y, int x)
{
    constexpr int R = K / 2, KK = K * K;
    int cls = 0;
    auto add = [&](const float* w, const float* s, int dy, int dx, bool neg) {
        const int tap = (dy + R) * K + dx + R;
        const float g = *s * w[a.p.rot ? KK - 1 - tap : tap], t = (neg ? -g : g) * f;
        cls |= (t < 0.f ? 0 : 1) | (t > 0.f ? 0 : 2);
    };
    auto within = [](int dy, int dx) { return dy >= -R && dy <= R && dx >= -R && dx <= R; };
    if (!a.skip_base && within(py - y, px - x)) add(a.p.w0 + (long)c * KK, a.p.s0 + c, py - y, px - x, false);
#pragma unroll 1
    for (int l = 1; l <= a.L; ++l) {
        const int dy = (py >> l) - (y >> l), dx = (px >> l) - (x >> l);
        if (!within(dy, dx)) continue;
        const bool ny = ((py ^ y) >> (l - 1)) & 1, nx = ((px ^ x) >> (l - 1)) & 1;
#pragma unroll 1
        for (int q = 0; q < 4; ++q)
            add(a.p.lw[l - 1] + (long)(4 * c + q) * KK, a.p.ls[l - 1] + 4 * c + q, dy, dx,
                ((q & 1) && ny) != ((q >> 1) && nx));
    }
    return cls;
}

// Terms that non-finite folded weights of the channel add to output (y, x) of a
// plane, classed the same way; the pixels around the plane are zeros. On planes
// of at most 8 x 8, whose vector kernel skips those, `rest` is the sum of the
// other terms: the output, if there is none.
template <int K, typename ST>
DEV int weight_terms(const PhaseArgs& a, int c, const ST* __restrict__ plane, int y, int x, float& rest)
{
    constexpr int R = K / 2, KK = K * K;
    const bool skip = a.H <= kTinyMaxEdge && a.W <= kTinyMaxEdge;
    int cls = 0;
#pragma unroll 1
    for (int e = a.skip_base ? KK : 0; e < (1 + 4 * a.L) * KK && cls != 3; ++e) {
        const int r = e / KK, tap = e - r * KK, l = (r + 3) / 4, q = (r + 3) & 3;
        const int t = a.p.rot ? KK - 1 - tap : tap, ch = 4 * c + q;
        const float g = l == 0 ? a.p.s0[c] * a.p.w0[(long)c * KK + t]
                               : a.p.ls[l - 1][ch] * a.p.lw[l - 1][(long)ch * KK + t];
        const bool finite = __builtin_fabsf(g) < __builtin_inff();
        if (finite && !skip) continue;
        const int j = (y >> l) + tap / K - R, i = (x >> l) + tap % K - R;
        const bool in = j >= 0 && i >= 0 && (j << l) < a.H && (i << l) < a.W;
        if (!in && skip) continue;
        float v = 0.f;
        if (in) v = l == 0 ? to_f32(plane[(long)j * a.W + i]) : (float)block_sum<ST>(plane, a.H, a.W, l, q, j, i);
        const bool neg = l > 0 && ((q & 1) && ((y >> (l - 1)) & 1)) != ((q >> 1) && ((x >> (l - 1)) & 1));
        const float s = (neg ? -g : g) * v;
        if (finite) {
            rest += __builtin_ldexpf(s, -2 * l);
            continue;
        }
        cls |= (s < 0.f ? 0 : 1) | (s > 0.f ? 0 : 2);
    }
    return cls;
}

// Whether every folded weight of channel c is finite.
template <int K>
DEV bool finite_weights(const PhaseArgs& a, int c, int lane)
{
    constexpr int KK = K * K;
    bool ok = true;
#pragma unroll 1
    for (int e = lane; e < (1 + 4 * a.L) * KK; e += 64) {
        const int r = e / KK, t = e - r * KK, ch = 4 * c + ((r + 3) & 3);
        const float g = r == 0 ? a.p.s0[c] * a.p.w0[(long)c * KK + t]
                               : a.p.ls[(r - 1) / 4][ch] * a.p.lw[(r - 1) / 4][(long)ch * KK + t];
        ok = ok && __builtin_fabsf(g) < __builtin_inff();
    }
    return __ballot(!ok) == 0;
}

// The wavefront's outputs that became NaN over the planes of its workgroup: an
// infinity where all their non-finite terms (of pixels, kernels, bias and carry)
// have one sign. The wavefront reads 64 pixels at a time. Everything is formed anew from
// the arguments, so that the kernel keeps nothing through its loop for this.
template <int K, typename ST, bool RGN>
DEV void restore_infinities(const PhaseArgs& a, int wave)
{
    const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const int bid = (int)blockIdx.x - a.fin_blocks, c = bid % a.C;
    const int ntiles = RGN ? a.rg_ntx * a.rg_nty : 1, chunk = (bid / a.C) / ntiles, tile = (bid / a.C) - chunk * ntiles;
    const int b_begin = chunk * a.nb, b_end = min(a.B, b_begin + a.nb);
    const int oy = RGN ? (tile / a.rg_ntx) * a.rg_th : 0, ox = RGN ? (tile % a.rg_ntx) * a.rg_tw : 0;
    const int ye = RGN ? min(oy + a.rg_th, a.H) : a.H, xe = RGN ? min(ox + a.rg_tw, a.W) : a.W;
    const int y0 = RGN ? max(oy - 4, 0) : 0, y1 = RGN ? min(ye + 4, a.H) : a.H;  // rows that reach the outputs
    // this lane's outputs, as in the kernel
    const PhaseStage& g = a.st[0];
    const int slot = wave * 16 + (lane & 15), vct = g.V * g.ct, sp = slot < a.PP * vct ? slot / vct : -1;
    const int sv = (slot % vct) / g.ct, I = slot % g.ct, x = ox + 8 * I + 4 * ((lane >> 4) & 1);
    const int y = oy + 2 * sv * g.js + (lane >> 5), nj = min(max((ye - y + 1) >> 1, 0), g.js);
    const float bias = (!a.skip_base && a.p.b0) ? a.p.s0[c] * a.p.b0[c] : 0.f;
    const long HW = (long)a.H * a.W;
    const int L = a.L;
    const bool finite = finite_weights<K>(a, c, lane);
#pragma unroll 1
    for (int b = b_begin; b < b_end; ++b) {
        const long pl = (long)b * a.C + c;
        const ST* ip = reinterpret_cast<const ST*>(a.in) + pl * HW;
        ST* op = reinterpret_cast<ST*>(a.out) + pl * HW;
        const int n = (b - b_begin) % a.PP == sp ? 4 * nj : 0;
        uint32_t open = 0, pos = 0, neg = 0;  // bit e: output e is NaN; has a term +inf, -inf
#pragma unroll 1
        for (int e = 0; e < n; ++e) {
            const int yy = y + 2 * (e >> 2), xx = x + (e & 3);
            if (xx >= xe || to_f32(op[(long)yy * a.W + xx]) == to_f32(op[(long)yy * a.W + xx])) continue;
            open |= 1u << e;
            float extra = bias;
            if (RGN && a.carry)
                extra += 0.5f * to_f32(reinterpret_cast<const ST*>(
                                    a.carry)[(pl * a.carry_H + (yy >> 1)) * a.carry_W + (xx >> 1)]);
            int cls = 0;
            if (!finite) {
                cls = weight_terms<K, ST>(a, c, ip, yy, xx, extra);
                if (cls == 0 && __builtin_fabsf(extra) < __builtin_inff())
                    op[(long)yy * a.W + xx] = from_f32<ST>(extra);
            }
            if ((cls & 1) || !(extra < __builtin_inff())) pos |= 1u << e;
            if ((cls & 2) || !(extra > -__builtin_inff())) neg |= 1u << e;
        }
#pragma unroll 1
        for (long i0 = (long)y0 * a.W; i0 < (long)y1 * a.W && __ballot((open & ~(pos & neg)) != 0) != 0; i0 += 64) {
            const float f = i0 + lane < (long)y1 * a.W ? to_f32(ip[i0 + lane]) : 0.f;
            uint64_t m = __ballot(!(__builtin_fabsf(f) < __builtin_inff()));
#pragma unroll 1
            for (; m != 0; m &= m - 1) {
                const int k = __builtin_ctzll(m), py = (int)((i0 + k) / a.W), px = (int)(i0 + k - (long)py * a.W);
                const float v = __shfl(f, k, 64);
                // the outputs it reaches: those whose 2^L x 2^L block is within k / 2 of its own
                const int yl = max(((((py >> L) - K / 2) << L) - y + 1) >> 1, 0);
                const int yh = min((((((py >> L) + K / 2 + 1) << L) - 1) - y) >> 1, 7);
                const int xl = max((((px >> L) - K / 2) << L) - x, 0), xh = min((((px >> L) + K / 2 + 1) << L) - 1 - x, 3);
                uint32_t left = 0;
                if (yl <= yh && xl <= xh)
                    left = open & ~(pos & neg) & (~0u << 4 * yl) & (~0u >> (28 - 4 * yh)) &
                           (0x11111111u * ((0xfu << xl) & (0xfu >> (3 - xh))));
#pragma unroll 1
                for (; left != 0; left &= left - 1) {
                    const int e = __builtin_ctz(left);
                    const int cls = nonfinite_terms<K>(a, c, v, py, px, y + 2 * (e >> 2), x + (e & 3));
                    pos |= (uint32_t)(cls & 1) << e;
                    neg |= (uint32_t)(cls >> 1) << e;
                }
            }
        }
#pragma unroll 1
        for (uint32_t left = open & (pos ^ neg); left != 0; left &= left - 1) {
            const int e = __builtin_ctz(left);
            op[(long)(y + 2 * (e >> 2)) * a.W + x + (e & 3)] =
                from_f32<ST>((pos >> e) & 1 ? __builtin_inff() : -__builtin_inff());
        }
    }
}

// Wavefronts per SIMD: three (168 registers) but for float32 k = 5 with two block
// rounds in flight, which spills there.
template <int K, typename ST, int NR>
constexpr int phase_waves() { return K == 5 && sizeof(ST) == 4 && NR == 2 ? 2 : 3; }

// NR: rounds of 4 x 4 blocks a thread loads per batch. Three workgroups per
// CU (168 registers): stage 0's weights take 4 k NW registers and stay in them
// for the workgroup's life.
template <int K, typename ST, int NR, bool RGN, bool DEEP>
__global__ void __launch_bounds__(kThreads, (phase_waves<K, ST, NR>())) phase_kernel(const PhaseArgs a)
{
    using SC = Scheme<ST>;
    constexpr int R = K / 2, M = kPhaseMargin, MAXJS = phase_max_js(NR);
    extern __shared__ float4 lds4[];
    char* lds = reinterpret_cast<char*>(lds4);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int C = a.C;
    if ((int)blockIdx.x < a.fin_blocks) {
        const int rows = 1 + 4 * a.fin.L, task = kWaves * (int)blockIdx.x + wave;
        if (task < a.fin.C * rows) reduce_task(a.fin, task / rows, task % rows, lane);
        return;
    }
    const int bid = (int)blockIdx.x - a.fin_blocks;
    const int c = bid % C;
    const int ntiles = RGN ? a.rg_ntx * a.rg_nty : 1;
    const int chunk = (bid / C) / ntiles;
    const int tile = (bid / C) - chunk * ntiles;
    const int b_begin = chunk * a.nb, b_end = min(a.B, b_begin + a.nb);
    const int oy = RGN ? (tile / a.rg_ntx) * a.rg_th : 0;
    const int ox = RGN ? (tile % a.rg_ntx) * a.rg_tw : 0;
    const int H = a.H, W = a.W;
    const int HW = H * W;
    const ST* in = reinterpret_cast<const ST*>(a.in);
    ST* out = reinterpret_cast<ST*>(a.out);

    // This thread's blocks (region mode: the area starts one block before the
    // tile on both axes): plane of the batch, top-left pixel, offset of its
    // first row in the batch's planes and of the plane's last row. Positions
    // outside are clamped (loaded, then masked); threads without a block read
    // the batch's last plane's.
    const int nblk = a.bx * a.by;
    RawBlock<ST> v[NR];
    int blk_p[NR], blk_y[NR], blk_x[NR];
    uint32_t blk_off[NR], blk_last[NR];
    const int top = RGN ? 4 : 0;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int e = tid + i * kThreads;
        const int p = fdiv(e, a.r_bxy), r = e - p * nblk, j = fdiv(r, a.r_bx);
        blk_p[i] = p;
        blk_y[i] = 4 * j - top;
        blk_x[i] = 4 * (r - j * a.bx) - top;
        const int yc = min(max(oy + blk_y[i], 0), H - 1), xc = min(max(ox + blk_x[i], 0), W - 4);
        const uint32_t pb = (uint32_t)min(p, a.PP - 1) * C * HW;
        blk_off[i] = pb + yc * W + xc;
        blk_last[i] = pb + (H - 1) * W + xc;
    }
    auto fetch = [&](int b0) {
        if (b0 >= b_end) return;
        const ST* base = in + ((long)b0 * C + c) * HW;
        // a last, partial batch: planes past the end are read from the first
        const bool part = b0 + a.PP > b_end;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            uint32_t off = blk_off[i], last = blk_last[i];
            if (part && b0 + blk_p[i] >= b_end) off = last = 0;
            fetch_raw<ST>(base, off, last, W, v[i]);
        }
    };
    const int edge = (4 - (W & 3)) & 3;
    const bool ragged = RGN || edge != 0 || (H & 3) != 0;
    uint16_t epoch = 0;  // number of the current batch
    auto put = [&](int b0) {
        ++epoch;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            if (blk_p[i] >= a.PP || b0 + blk_p[i] >= b_end) continue;
            int y0 = blk_y[i], x0 = blk_x[i];
            asm volatile("" : "+v"(y0), "+v"(x0));  // no per-row addresses kept across the batch loop
            if (ragged) mask_raw<ST>(H, W, oy + y0, ox + x0, edge, v[i]);
            if (__builtin_expect(nonfinite<ST>(v[i]), 0))
                mark_block<ST>(a, lds, blk_p[i], tid + i * kThreads - blk_p[i] * nblk, epoch, v[i]);
            put_block<ST, DEEP>(a, lds + a.planes_off + blk_p[i] * a.plane_bytes, y0, x0, v[i]);
        }
    };
    fetch(b_begin);

    // The finalize of an earlier launch's kernel gradients, while the first
    // blocks are on their way: the wavefronts of the whole grid take its
    // (channel, kernel row) tasks in turn.
    if (a.fin_tasks > 0) {
        const int rows = 1 + 4 * a.fin.L;
        for (int task = kWaves * bid + wave; task < a.fin_tasks; task += kWaves * (int)gridDim.x)
            reduce_task(a.fin, task / rows, task % rows, lane);
    }

    // Stage 0's table only lives until its fragments are in registers: it
    // borrows the planes' area (restore_infinities() takes the weights anew).
    char* tab0 = lds + a.planes_off;
    double* st = reinterpret_cast<double*>(tab0 + 2 * SC::NW * tab_rows<K, true>() * kPhaseTabPitch);
    const bool finite = stage_kernels<K>(a.p, c, a.L, st, tid);
    __syncthreads();
    float scale = 1.f, inv = 1.f;  // float16: powers of two that keep the weight pieces in range
    if constexpr (SC::F16) {
        // the largest |E| plus the largest |base| bounds every coefficient: to
        // at most 2^15
        float me = 0.f, mb = 0.f;
        for (int e = lane; e < 5 * K * K; e += 64) {
            const float f = __builtin_fabsf((float)st[e]);
            if (e < K * K)
                mb = __builtin_fmaxf(mb, f);
            else
                me = __builtin_fmaxf(me, f);
        }
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            mb = __builtin_fmaxf(mb, __shfl_xor(mb, m, 64));
            me = __builtin_fmaxf(me, __shfl_xor(me, m, 64));
        }
        const int ex = (int)(__float_as_uint(me + (a.skip_base ? 0.f : mb)) >> 23) - 127;
        const int sh = ex >= 128 ? 0 : min(14 - ex, 100);
        scale = __builtin_ldexpf(1.f, sh);
        inv = __builtin_ldexpf(1.f, -sh);
    }
    fill_table<K, true, SC::F16>(st, 0, !a.skip_base, tab0, scale, tid);
    if constexpr (DEEP)
        for (int s = 1; s < a.L; ++s) fill_table<K, false, false>(st, s, false, lds + a.st[s].tab, 1.f, tid);
    const float bias = (!a.skip_base && a.p.b0) ? a.p.s0[c] * a.p.b0[c] : 0.f;
    __syncthreads();
    auto clear_planes = [&]() {
        __syncthreads();  // the table has been read
        for (int i = a.mark_off / 16 + tid; i < a.lds_bytes / 16; i += kThreads)
            lds4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        __syncthreads();
        if (__builtin_expect(!finite, 0)) infinity_flag(a, lds) = 1;
    };
    // Roles: the first fine_waves wavefronts run stage 0, the others the deeper
    // stages lo .. hi. A wavefront of one stage keeps its weights in registers,
    // one of several reads them anew for each.
    const bool fine = !DEEP || wave < a.fine_waves;
    const bool two = DEEP && a.fine_waves == 2;
    const int lo = two ? wave - 1 : 1, hi = two && wave == 2 ? 1 : a.L - 1;
    if constexpr (DEEP) {
        // (the same barriers as the fine wavefronts below)
        if (!fine && lo == hi) {
            u32x4 A[K][3];
            load_weights<K, false, 3>(lds + a.st[lo].tab, lane, A);
            clear_planes();
            for (int b0 = b_begin; b0 < b_end; b0 += a.PP) {
                put(b0);
                __syncthreads();
                fetch(b0 + a.PP);
                coarse_stage<K>(a, lds, lo, false, lane, A);
                __syncthreads();
            }
            return;
        }
        if (!fine) {
            clear_planes();
            for (int b0 = b_begin; b0 < b_end; b0 += a.PP) {
                put(b0);
                __syncthreads();
                fetch(b0 + a.PP);
                for (int t = 3; t < a.L; ++t) {
                    build_deep(a, lds, __builtin_amdgcn_readfirstlane(t), lane);
                    asm volatile("" ::: "memory");
                }
                for (int t = hi; t >= lo; --t) {
                    const int s = __builtin_amdgcn_readfirstlane(t);
                    coarse_stage_load<K>(a, lds, s, s < hi, lane);
                    asm volatile("" ::: "memory");
                }
                __syncthreads();
            }
            return;
        }
    }
    u32x4 A[K][3];
    load_weights<K, true, SC::NW>(tab0, lane, A);
    clear_planes();
    // this lane's column of tiles (fine wavefronts)
    const PhaseStage& g = a.st[0];
    const int grp = lane >> 4;
    const int vct = g.V * g.ct;
    const int slot = wave * 16 + (lane & 15);
    const bool live = slot < a.PP * vct;
    const int sp = live ? fdiv(slot, g.r_vct) : 0;
    const int rem = live ? slot - sp * vct : 0;
    const int sv = fdiv(rem, g.r_ct), I = rem - sv * g.ct;
    const int J0 = sv * g.js;
    char* plane = lds + a.planes_off + sp * a.plane_bytes;
    const int tp_off = a.planes_off + sp * a.plane_bytes + g.poff + 2 * ((2 * J0 + M - 2 * R + (grp >> 1)) * g.pitch + 8 * I + 8 * (grp & 1));
    // its outputs: columns x .. x + 3 of nj rows, two apart, from ya on
    const int x = 8 * I + 4 * (grp & 1), ya = 2 * J0 + (grp >> 1);
    const int xe = RGN ? min(a.rg_tw, W - ox) : W, ye = RGN ? min(a.rg_th, H - oy) : H;
    const int nj = live && x < xe ? min(max((ye - ya + 1) >> 1, 0), g.js) : 0;
    const uint32_t out_off = (uint32_t)sp * C * HW + (oy + ya) * W + ox + x;

    for (int b0 = b_begin; b0 < b_end; b0 += a.PP) {
        put(b0);
        __syncthreads();
        fetch(b0 + a.PP);
        f32x4 acc[MAXJS];
#pragma unroll
        for (int J = 0; J < MAXJS; ++J) acc[J] = f32x4{0.f, 0.f, 0.f, 0.f};
        switch (g.js) {
            case 1: run_tiles<K, 1, SC>(lds, tp_off, 4 * g.pitch, g.psz, A, acc); break;
            case 2: run_tiles<K, 2, SC>(lds, tp_off, 4 * g.pitch, g.psz, A, acc); break;
            case 3: run_tiles<K, 3, SC>(lds, tp_off, 4 * g.pitch, g.psz, A, acc); break;
            case 4: run_tiles<K, 4, SC>(lds, tp_off, 4 * g.pitch, g.psz, A, acc); break;
            case 5: run_tiles<K, 5, SC>(lds, tp_off, 4 * g.pitch, g.psz, A, acc); break;
            case 6: run_tiles<K, 6, SC>(lds, tp_off, 4 * g.pitch, g.psz, A, acc); break;
            case 7: run_tiles<K, 7, SC>(lds, tp_off, 4 * g.pitch, g.psz, A, acc); break;
            default: run_tiles<K, MAXJS, SC>(lds, tp_off, 4 * g.pitch, g.psz, A, acc); break;
        }
        __syncthreads();
        const int b = b0 + sp;
        if (b >= b_end) continue;
        uint32_t off = out_off;
        int j0 = J0;
        asm volatile("" : "+v"(off), "+v"(j0));  // no per-row addresses kept across the batch loop
        ST* op = out + ((long)b0 * C + c) * HW;
        // the coarser levels' sums for the two column pairs of the row of pair j
        auto coarse = [&](int j, float& r0, float& r1) {
            r0 = r1 = bias;
            if constexpr (DEEP) {
                const PhaseStage& g1 = a.st[1];
                const float2 r = *reinterpret_cast<const float2*>(plane + g1.roff + 4 * (j * g1.rpitch + (x >> 1)));
                r0 += r.x;
                r1 += r.y;
                if (two) {  // stage 2's wavefront is not stage 1's
                    const PhaseStage& g2 = a.st[2];
                    const float q =
                        *reinterpret_cast<const float*>(plane + g2.roff + 4 * ((j >> 1) * g2.rpitch + (x >> 2)));
                    r0 += q;
                    r1 += q;
                }
            }
        };
        // region mode's carry: the values of G rows requested together, clamped
        // (rows and columns past the grid feed pixels that are not stored). All
        // rows' spill in float16 and float32 (256 x 256 B8 C128 L3 f16 forward 285
        // us with all, 271 with four); in bfloat16 they are 1 % faster.
        constexpr int G = SC::F16 || sizeof(ST) == 4 ? 4 : MAXJS;
        const bool carry = RGN && a.carry;
        const ST* cp = nullptr;
        int cx0 = 0, cx1 = 0;
        if constexpr (RGN) {
            cp = reinterpret_cast<const ST*>(a.carry) + ((long)b * C + c) * a.carry_H * a.carry_W;
            cx0 = min((ox + x) >> 1, a.carry_W - 1), cx1 = min(cx0 + 1, a.carry_W - 1);
        }
#pragma unroll
        for (int J1 = 0; J1 < MAXJS; J1 += G) {
            if (J1 >= g.js) break;
            float cr[G][2];
            if constexpr (RGN) {
                if (carry) {
#pragma unroll
                    for (int J = 0; J < G; ++J) {
                        const int cy = min((oy >> 1) + j0 + J1 + J, a.carry_H - 1) * a.carry_W;
                        cr[J][0] = to_f32(cp[cy + cx0]);
                        cr[J][1] = to_f32(cp[cy + cx1]);
                    }
                }
            }
#pragma unroll
            for (int J = J1; J < J1 + G && J < MAXJS; ++J) {
                if (J >= g.js) break;
                if (J < nj) {
                    float o[4] = {acc[J][0], acc[J][1], acc[J][2], acc[J][3]};
                    float r0, r1;
                    coarse(j0 + J, r0, r1);
                    if (carry) {
                        r0 = __builtin_fmaf(0.5f, cr[J - J1][0], r0);
                        r1 = __builtin_fmaf(0.5f, cr[J - J1][1], r1);
                    }
                    if constexpr (SC::F16) {
                        o[0] = __builtin_fmaf(o[0], inv, r0);
                        o[1] = __builtin_fmaf(o[1], inv, r0);
                        o[2] = __builtin_fmaf(o[2], inv, r1);
                        o[3] = __builtin_fmaf(o[3], inv, r1);
                    } else {
                        o[0] += r0;
                        o[1] += r0;
                        o[2] += r1;
                        o[3] += r1;
                    }
                    store4<ST>(op, off, x, xe, o);
                }
                off += 2 * W;
            }
        }
        if (__builtin_expect(marked(reinterpret_cast<const uint16_t*>(lds + a.mark_off)[sp], epoch), 0)) {
            // the plane holds non-finite pixels: NaN for the outputs that see one
            uint32_t o = out_off;
#pragma unroll 1
            for (int e = 0; e < 4 * nj; ++e) {
                const int y = ya + 2 * (e >> 2), xx = x + (e & 3);
                if (xx < xe && depends_on_mark(a, lds, R, sp, y + (RGN ? 4 : 0), xx + (RGN ? 4 : 0), epoch))
                    op[o + (e >> 2) * 2 * W + (e & 3)] = from_f32<ST>(__builtin_nanf(""));
            }
        }
    }
    const PhaseArgs* ap = (const PhaseArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ap));
    if (__builtin_expect(infinity_flag(*ap, lds), 0)) restore_infinities<K, ST, RGN>(*ap, wave);
}

template <int K, typename ST, int NR, bool RGN, bool DEEP>
hipError_t launch_phase_v(const PhaseArgs& a, int grid, hipStream_t s)
{
    static std::atomic<unsigned long long> lds_done{0};
    const hipError_t e = allow_full_lds(reinterpret_cast<const void*>(&phase_kernel<K, ST, NR, RGN, DEEP>), lds_done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((phase_kernel<K, ST, NR, RGN, DEEP>), dim3(grid), dim3(kThreads), a.lds_bytes, s, a);
    return hipGetLastError();
}

template <int K, typename ST>
hipError_t launch_phase_t(const PhaseArgs& a, int grid, int rounds, hipStream_t s)
{
    if (a.rg_ntx > 0) return launch_phase_v<K, ST, 2, true, false>(a, grid, s);
    if (a.L > 1)
        return rounds > 1 ? launch_phase_v<K, ST, 2, false, true>(a, grid, s)
                          : launch_phase_v<K, ST, 1, false, true>(a, grid, s);
    return rounds > 1 ? launch_phase_v<K, ST, 2, false, false>(a, grid, s)
                      : launch_phase_v<K, ST, 1, false, false>(a, grid, s);
}

template <int K>
hipError_t launch_phase_k(wtconv_dtype dt, const PhaseArgs& a, int grid, int rounds, hipStream_t s)
{
    switch (dt) {
        case WTCONV_F32: return launch_phase_t<K, float>(a, grid, rounds, s);
        case WTCONV_BF16: return launch_phase_t<K, uint16_t>(a, grid, rounds, s);
        case WTCONV_F16: return launch_phase_t<K, _Float16>(a, grid, rounds, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_phase_forward(int k, wtconv_dtype dt, const PhaseArgs& a, int grid, int block_rounds, hipStream_t s)
{
    switch (k) {
        case 3: return launch_phase_k<3>(dt, a, grid, block_rounds, s);
        case 5: return launch_phase_k<5>(dt, a, grid, block_rounds, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace wtc
