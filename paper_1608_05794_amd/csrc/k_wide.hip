// Wavefront-per-reactor ROS4 for 64 < N <= 112: the whole iteration matrix in one wavefront's tiles
// (N = 112: 392 of its 512 registers, one wavefront per SIMD), two state components per lane.
//
// Against the four-wavefront workgroup (the matrix over four wavefronts, two workgroups per CU): no
// barrier between the 16 pivots of a panel, whose search and broadcasts are a serial chain that the four
// wavefronts ran together, and no panel exchange; four reactors per CU instead of two.  M111 x 4099
// reactors to 1e-13 s: 489 ms with the workgroup, 295 ms here.  Of a step's 472 k cycles in an instrumented
// build the inverse takes 266 k, the Jacobian windows 110 k with 16 k of species and chain rule, the two
// stage source terms 45 k, the four solves 21 k, the controller 6 k.
#include "wave.h"

namespace ck {

// Few reactors are a latency, which four wavefronts on one reactor make shorter: as long as their
// workgroups are all resident at once (two a CU) they finish first where a step is long for one wavefront,
// that is with more than 96 rows (M111 x 256, 20 steps: 2.3 ms, one wavefront 3.4) or with general
// reactions (N = 96, all of 475 general, x 256: 2.2 and 4.3 ms).  Beyond two a CU one wavefront a reactor
// is ahead (M111 x 768: 5.0 and 3.6 ms), with up to 96 rows and pair-form reactions it was never behind.
bool wide_preferred(const DevMech &M, int64_t n, const IntOpts &o) {
    if (M.N <= 64 || M.N > 112) return false;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return true;
    const int64_t resident = int64_t(cus) * (o.blocks_per_cu == 1 ? 1 : 2);
    return n > resident || (M.N <= 96 && M.n_gen == 0);
}

int launch_integrate_wide(const DevMech &M, int64_t n, double *y, int64_t ld, const double *p, const double *t_end,
                          double *t, double *h, const IntOpts &opts, void *ws, int32_t *status, int32_t *nacc,
                          int32_t *nrej, hipStream_t s) {
    unsigned *q = static_cast<unsigned *>(ws);
    IntOpts o = opts;
    // counted in workgroups of the four-wavefront form, of which two fill a CU as four of these do
    if (o.blocks_per_cu > 0) o.blocks_per_cu = o.blocks_per_cu < 2 ? 2 : 4;
    switch ((M.N + 15) / 16 * 16) {
        case 80: return launch_int<Ros4Adapter<80>>(M, n, y, ld, p, t_end, t, h, o, q, status, nacc, nrej, s);
        case 96: return launch_int<Ros4Adapter<96>>(M, n, y, ld, p, t_end, t, h, o, q, status, nacc, nrej, s);
        case 112: return launch_int<Ros4Adapter<112>>(M, n, y, ld, p, t_end, t, h, o, q, status, nacc, nrej, s);
        default: return CK_EUNSUPPORTED;
    }
}

}  // namespace ck
