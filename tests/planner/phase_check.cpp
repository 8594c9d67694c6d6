// Host-only check of the polyphase plans (no GPU, no kernels): includes the
// library's host source with the kernel launchers stubbed out, and for each
// descriptor on stdin ("B C H W k L dtype" per line) verifies what the kernels
// rely on, for the plan of a whole plane, the region plan and the gradient
// plan:
//   - tiles, blocks and batches cover the plane and the batch, within the
//     threads, the wavefronts' slots and the batch numbers there are;
//   - every row and column that a block write, a tile's window, a deeper
//     stage's result or a float32 mean touches lies inside its own array, the
//     arrays do not overlap, and they end inside the workgroup's LDS;
//   - offsets within a batch of planes fit the 32 bits they are held in.
// Prints one line per descriptor: "ok <resident> <region> <gradient>" (0 or 1:
// such a plan exists) or "FAIL <reason>". Built and run by
// tests/test_planner.py.
#include "wtconv_api.cpp"

#include <stdio.h>

namespace wtc {
hipError_t launch_forward(int, wtconv_dtype, const FusedArgs&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_backward(int, wtconv_dtype, const FusedArgs&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_reduce(const ReduceArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_grad(int, wtconv_dtype, const GradArgs&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_carrier(wtconv_dtype, const CarrierArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_tiny(int, wtconv_dtype, bool, const TinyArgs&, hipStream_t) { return hipSuccess; }
int forward_wgs_by_regs(int, wtconv_dtype, bool, int fallback) { return fallback; }
hipError_t launch_forward_mixed(int, wtconv_dtype, const FusedArgs&, int, hipStream_t) { return hipSuccess; }
int mixed_wgs_by_regs(int, wtconv_dtype, int, int fallback) { return fallback; }
hipError_t launch_phase_forward(int, wtconv_dtype, const PhaseArgs&, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_phase_grad(int, wtconv_dtype, const PhaseGradArgs&, int, int, hipStream_t) { return hipSuccess; }
}  // namespace wtc

#define REQUIRE(c) \
    if (!(c)) return #c

constexpr int M = wtc::kPhaseMargin;

static const char* check_forward(const wtconv_desc& d, const PhasePlan& pp)
{
    const wtc::PhaseArgs& a = pp.a;
    const bool rgn = a.rg_ntx > 0;
    const int R = d.k / 2, np0 = d.dtype == WTCONV_F32 ? 3 : 1;
    REQUIRE(a.PP >= 1 && pp.rounds >= 1 && pp.rounds <= 2);
    REQUIRE((long)a.PP * a.bx * a.by <= (long)pp.rounds * wtc::kThreads);
    REQUIRE(a.nb % a.PP == 0 || pp.nchunks == 1);
    REQUIRE((long)a.nb * pp.nchunks >= d.B && (a.nb + a.PP - 1) / a.PP <= 32766);
    REQUIRE((((long)a.PP - 1) * d.C + 1) * d.H * d.W < 1L << 29 || rgn);
    REQUIRE(a.PP * a.st[0].V * a.st[0].ct <= 16 * a.fine_waves);
    REQUIRE(a.st[0].js >= 1 && a.st[0].js <= wtc::phase_max_js(pp.rounds));
    if (rgn) {
        REQUIRE(a.rg_ntx * a.rg_tw >= d.W && a.rg_nty * a.rg_th >= d.H && a.L == 1 && a.PP == 1);
        REQUIRE(4 * a.bx >= a.rg_tw + 8 && 4 * a.by >= a.rg_th + 8);
    } else {
        REQUIRE(4 * a.bx >= d.W && 4 * a.by >= d.H);
    }
    long end = 0;  // of the arrays so far
    for (int s = 0; s < a.L; ++s) {
        const wtc::PhaseStage& g = a.st[s];
        const int rows = g.psz / (2 * g.pitch), np = s == 0 ? np0 : 3, top = rgn ? 4 : 0;
        REQUIRE(g.pitch % 8 == 0 && g.psz % 16 == 0 && 8 * g.ct >= g.w && 2 * g.V * g.js >= g.h);
        REQUIRE(g.poff >= end);
        end = g.poff + (long)np * g.psz;
        REQUIRE(M - 2 * R >= 0 && 2 * g.V * g.js + M + 2 * R <= rows && 8 * g.ct + 8 <= g.pitch);  // windows
        if (s < 3) {  // block writes (stage 2: one value a block)
            REQUIRE(((4 * a.by - top - 1) >> s) + M < rows && ((4 * a.bx - top - 1) >> s) + M < g.pitch);
        } else {
            REQUIRE(g.h - 1 + M < rows && g.w - 1 + M < g.pitch);
        }
        if (s >= 1) {
            REQUIRE(g.js == 1 || g.js == 2 || g.js == 4);
            REQUIRE(g.h > 4 || (g.V == 1 && g.js == (g.h + 1) / 2));  // the runs over a plane's own rows
            REQUIRE(g.roff >= end);
            end = g.roff + 4L * 2 * g.V * g.js * g.rpitch;
            REQUIRE(8 * g.ct <= g.rpitch);
            // what the finer stage reads of this one's result
            const wtc::PhaseStage& f = a.st[s - 1];
            REQUIRE((f.h + 1) / 2 <= 2 * g.V * g.js && 4 * f.ct <= g.rpitch);
            if (s == 2) REQUIRE(((f.h + 1) / 2 <= 2 * g.V * g.js) && 2 * a.st[0].ct <= g.rpitch);
        }
        if (s >= 2 && s + 1 < a.L) {
            REQUIRE(g.mf >= end);
            end = g.mf + 4L * g.h * g.w;
            if (s == 2) REQUIRE(a.by <= g.h && a.bx <= g.w);
        }
    }
    REQUIRE(end <= a.plane_bytes);
    REQUIRE(a.planes_off >= a.mark_off + 2L * (a.PP * (1 + (a.L == 1 ? 4 : 1) * a.bx * a.by) + 1));
    REQUIRE(a.planes_off + (long)a.PP * a.plane_bytes <= a.lds_bytes && a.lds_bytes <= 160 * 1024);
    return nullptr;
}

static const char* check_side(const wtc::PhaseGradArgs& a, const wtc::PhaseSide& g, int s, bool x, int R)
{
    const int rows = g.psz[s] / (2 * g.pitch[s]), bx = x ? a.xbx : a.dbx, by = x ? a.xby : a.dby;
    const int top = x && a.rg_ntx > 0 ? 4 : 0;
    REQUIRE(g.pitch[s] % 8 == 0 && g.psz[s] % 16 == 0);
    REQUIRE(2 * a.V[s] * a.js[s] + (x ? M + 2 * R : 0) <= rows && 8 * a.ct[s] + (x ? 8 : 0) <= g.pitch[s]);
    if (s < 3) {
        REQUIRE(((4 * by - top - 1) >> s) + g.margin < rows && ((4 * bx - top - 1) >> s) + g.margin < g.pitch[s]);
    } else {
        REQUIRE(a.h[s] - 1 + g.margin < rows && a.w[s] - 1 + g.margin < g.pitch[s]);
    }
    if (s == 2 && a.L > 3) REQUIRE(by <= a.h[2] && bx <= a.w[2]);
    return nullptr;
}

static const char* check_grad(const wtconv_desc& d, const PhaseGradPlan& pg)
{
    const wtc::PhaseGradArgs& a = pg.a;
    const int R = d.k / 2;
    REQUIRE((long)a.PP * a.xbx * a.xby <= (long)pg.rounds * wtc::kThreads);
    REQUIRE((((long)a.PP - 1) * d.C + 1) * d.H * d.W < 1L << 29 || a.rg_ntx > 0);
    REQUIRE(a.rg_ntx > 0 || ((long)a.nb * pg.nchunks >= d.B && 4 * a.xbx >= d.W && 4 * a.xby >= d.H));
    long end = 0;
    for (int s = 0; s < a.L; ++s) {
        const int np = s == 0 ? 1 : 3;
        REQUIRE(8 * a.ct[s] >= a.w[s] && 2 * a.V[s] * a.js[s] >= a.h[s] && a.js[s] == (s == 0 ? 4 : 1));
        for (const wtc::PhaseSide* g : {&a.sx, &a.sd}) {
            if (const char* e = check_side(a, *g, s, g == &a.sx, R)) return e;
            REQUIRE(g->off[s] >= end);
            end = g->off[s] + (long)np * g->psz[s];
        }
        if (s >= 2 && s + 1 < a.L)
            for (const wtc::PhaseSide* g : {&a.sx, &a.sd}) {
                REQUIRE(g->mf[s] >= end);
                end = g->mf[s] + 4L * a.h[s] * a.w[s];
            }
    }
    REQUIRE(end <= a.plane_bytes && (long)a.PP * a.plane_bytes <= a.lds_bytes && a.lds_bytes <= 160 * 1024);
    REQUIRE(2 * d.k * 256 * 4 <= a.lds_bytes);
    return nullptr;
}

int main()
{
    int v[7];
    while (scanf("%d %d %d %d %d %d %d", v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6) == 7) {
        const wtconv_desc d = {v[0], v[1], v[2], v[3], v[4], v[5], (wtconv_dtype)v[6]};
        PhasePlan whole, region;
        PhaseGradPlan grad;
        const bool w = make_phase_plan(d, whole), r = make_phase_region_plan(d, region);
        const bool g = d.dtype != WTCONV_F32 && make_phase_grad_plan(d, grad);
        const char* e = w ? check_forward(d, whole) : nullptr;
        if (!e && r) e = check_forward(d, region);
        if (!e && g) e = check_grad(d, grad);
        for (int T = 8; !e && T <= 56; T += 8) {
            PhaseGradPlan t;
            if (make_phase_grad_region(d, T, (d.W + T - 1) / T, (d.H + T - 1) / T, d.B, t)) e = check_grad(d, t);
        }
        if (e)
            printf("FAIL %s\n", e);
        else
            printf("ok %d %d %d\n", w, r, g);
    }
    return 0;
}
