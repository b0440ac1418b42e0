// small.hpp -- grids up to 64^2: a member's whole time loop in one workgroup.
//
// A launch per pass costs 4-5 us whatever the grid, 16 of them per forward and
// adjoint step, while a 64^2 member's velocity pair (45 KB between the passes)
// fits the LDS of one CU.  So up to 64 points a workgroup owns one member and
// runs any number of steps: the spectral state stays in registers, the row and
// column passes trade the packed half spectra through LDS, and memory sees only
// the stage velocities kept for the adjoint.
//
// Every transform of N = 8 T points is held by a team of T lanes, eight values
// per lane (entry t + T m in register m of lane t): a radix-8 stage on the
// register digit, a trade of its low bits with the lane digit by register
// swaps (no LDS), a radix-T stage.  A team's lanes are the top log2(T) lane
// bits, which v_permlane32_swap, v_permlane16_swap and a DPP rotation by eight
// reach.  N rows take N T threads; the column phase uses 2 (Kc + 1) of the same
// N teams, one per column and signal, as twins on neighbouring lanes that trade
// halves as in col_twin_kernel.
//
// At 64^2 a workgroup (two wavefronts per SIMD) issues vector instructions in
// four cycles of five: 1275 per wavefront and stage, half of them FP64; below,
// one wavefront per SIMD waits on its own chain of transforms.  Measured, a
// launch per pass -> this: one 64^2 member's gradient over 200 steps 19.2 ->
// 11.4 ms (5.2 us per stage); seven 32^2 members over 33 steps 3.43 -> 1.06 ms
// (2.9 us).  Members run side by side, one per CU, so a batch costs no more
// time until it fills the chip.
#pragma once
#include "kernels.hpp"

namespace pa {

struct SmallArgs {
    const cd* tw;            // twiddles exp(-2 pi i m/N)
    const double* invk2;     // [KY][KXP]
    const double* ex2;       // [KXP]
    const double* ey2;       // [KY]
    double h, forcing;
    int nf;
    int B;                   // members of the launch
    int stride_b;            // members between two stage slots of the velocity store
    int steps;               // steps of the launch (0: only what precedes and follows them)
    cd* state;               // compact omega (forward) or lambda (adjoint), [B][KY][KXP]
    cd* ckpt;                // forward: the final state once more, or null
    cd* store;               // velocities z = u + i v, [4 steps (+1)][stride_b][N][N]: forward writes
                             // them if not null, adjoint reads
    cd* z_out;               // forward: z of the final state, [B][N][N], or null
    const double* src_u;     // adjoint: sources r_u, r_v [B][N][N] added at stage n of the last step
    const double* src_v;     // (or null)
    int from_source;         // adjoint: lambda starts as U^T r_u + V^T r_v (steps = 0)
};

// A field through a multiplier on the band.  in and out are the same fields or
// apart from each other: a member's workgroup reads while another writes.
struct SmallFilter {
    const cd* tw;
    const double* in;        // [B][N][N]
    double* out;
    MultSpec spec;           // the table, or with a null table the multiplier itself
    int table_per_member;    // spec.table [B][KY][KXP]
    int B;
};

bool small_grid(int N);
hipError_t launch_small_filter(const Dims& d, const SmallFilter& a, hipStream_t s);
hipError_t launch_small_forward(const Dims& d, const SmallArgs& a, hipStream_t s);
hipError_t launch_small_adjoint(const Dims& d, const SmallArgs& a, hipStream_t s);
// Observations of members [0, nb) from velocities z [nb][N][N] (all pointers at the first member),
// and their residual fields (0 off the probes) or a unit u-impulse (o.slot < 0).
hipError_t launch_small_observe(int N, int nb, const cd* z, const RowObs& o, hipStream_t s);
hipError_t launch_small_source(int N, int nb, const cd* z, const RowObs& o, double* src_u, double* src_v, hipStream_t s);

}  // namespace pa
