// The passes' kernels at the limit of their registers (registers_full in
// tlsph_passes.h): compiled with constants formed where they are used.  The
// 64-bit literals of exp, log and the Newton loops, hoisted out of the loops
// as they are elsewhere, take the registers that these kernels do not have.
// (GTN plate 4.1M FP64, force pass 643 us with them hoisted, so 619,
// deformation pass 737 and 719; 200k Voce bar mixed, deformation pass 50.8 and
// 46.0.  The kernels with registers to spare lose by it: the mixed plate's
// deformation pass at 190k 35.0 us hoisted, 36.0 in place; colliding bars
// FP64, two sweeps with four lanes, 41.5 and 46.0; the graded bar unstaged
// 40.7 and 41.9.)
#include "tlsph_passes.h"

namespace tlsph {

hipError_t launch_pipe_fp64(const DevState& s, int parity, hipStream_t st, size_t lds_bytes) {
    k_pass_b_staged<double, 2><<<(unsigned)s.grid_b, s.tile * 2, lds_bytes, st>>>(s, parity);
    return hipGetLastError();
}

const void* pipe_fp64() { return reinterpret_cast<const void*>(&k_pass_b_staged<double, 2>); }

void launch_update_full(const DevState& s, int parity, int block, int model, bool mixed,
                        hipStream_t st) {
    if (!mixed) {
        if (s.flow_general)
            launch_update<double, 3, true>(s, parity, block, st);
        else
            launch_update<double, 3, false>(s, parity, block, st);
    } else if (s.var_h) {
        launch_update<float, -1, true, true>(s, parity, block, st);
    } else {
        switch (model) {
            case 0: launch_update<float, 0, true>(s, parity, block, st); break;
            case 1: launch_update<float, 1, true>(s, parity, block, st); break;
            case 2: launch_update<float, 2, true>(s, parity, block, st); break;
            case 3: launch_update<float, 3, true>(s, parity, block, st); break;
            default: launch_update<float, -1, true>(s, parity, block, st); break;
        }
    }
}

}  // namespace tlsph
