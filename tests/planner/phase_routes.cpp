// Host-only dump of the polyphase dispatch (no GPU, no kernels): includes the
// library's host source with the kernel launchers stubbed out, and for each
// descriptor on stdin ("B C H W k L dtype" per line) prints
//   <forward> <PP> <batches> <last>  <gradient> <PP> <batches> <last>
// forward: 0 vector kernels, 1 polyphase over whole planes, 2 polyphase region
// tiles; gradient: 0 vector, 1 polyphase over whole planes, 2 in region tiles;
// PP: planes of a batch; batches: of the first workgroup of a channel; last: the
// planes in its last one. Built and run by tests/test_planner.py.
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

static void show(int route, int B, int nb, int PP)
{
    const int n = route ? std::min(B, nb) : 0;
    printf("%d %d %d %d  ", route, route ? PP : 0, route ? cdiv(n, PP) : 0, route ? n - (cdiv(n, PP) - 1) * PP : 0);
}

int main()
{
    int v[7];
    while (scanf("%d %d %d %d %d %d %d", v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6) == 7) {
        const wtconv_desc d = {v[0], v[1], v[2], v[3], v[4], v[5], (wtconv_dtype)v[6]};
        const PhaseExec e = choose_phase(d, 0);
        show(e.kind == PhaseExec::None ? 0 : (e.kind == PhaseExec::Resident ? 1 : 2), d.B, e.pl.a.nb, e.pl.a.PP);
        const GradExec g = choose_grad(d);
        GradExec r;
        if (g.use) {
            show(g.phase, d.B, g.pg.a.nb, g.pg.a.PP);
        } else {
            const bool region = region_grad_exec(d, choose(d, true), r) && r.phase;
            show(region ? 2 : 0, d.B, r.pg.a.nb, 1);
        }
        printf("\n");
    }
    return 0;
}
