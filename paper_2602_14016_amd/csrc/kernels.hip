// kernels.hip -- dispatch of the row / column passes to the per-grid-size
// instantiations (kern_<N>.hip), with host-side argument checks so that a
// launch with a missing buffer is refused before it can touch memory.
#include "kernels.hpp"

#include <algorithm>

namespace pa {

DispatchEvents& dispatch_events() {
    static thread_local DispatchEvents e;
    return e;
}

static bool obs_ok(const RowObs& o) {
    if (o.slot < 0) return true;
    return o.stride >= 1 && o.M >= 1 && o.n_times > o.slot;
}

static bool col_ptrs_ok(int mode, const ColArgs& a) {
    if (!a.invk2 || !a.ex2 || !a.ey2 || !a.tw) return false;
    if (a.nout < 0 || a.nout > 2) return false;
    for (int o = 0; o < a.nout; ++o)
        if (!a.yout[o]) return false;
    switch (mode) {
        case COL_INIT: return a.yin[0] && a.omega;
        case COL_A: case COL_B: case COL_C: case COL_D: return a.yin[0] && a.yin[1] && a.omega && a.acc;
        case COL_FILTER: return a.yin[0] && a.mult;
        case COL_FROM_STATE: return a.state_in != nullptr;
        case COL_FIRST_GUESS: return a.yin[0] && a.yin[1] && a.lowpass >= 0;
        case COL_ADJ_C: case COL_ADJ_B: case COL_ADJ_A: case COL_ADJ_N:
            return a.yin[0] && a.yin[1] && a.lam && a.omb;
        case COL_ADJ_SRC: return a.yin[0] && a.yin[1] && a.lam;
        default: return false;
    }
}

#define PA_DISPATCH_N(CALL)                                   \
    switch (d.N) {                                            \
        case 8: return Launch<8>::CALL;                       \
        case 16: return Launch<16>::CALL;                     \
        case 32: return Launch<32>::CALL;                     \
        case 64: return Launch<64>::CALL;                     \
        case 128: return Launch<128>::CALL;                   \
        case 256: return Launch<256>::CALL;                   \
        case 512: return Launch<512>::CALL;                   \
        case 1024: return Launch<1024>::CALL;                 \
        default: return hipErrorInvalidValue;                 \
    }

int fft_threads(int N, int var) {
    switch (N) {
        case 8: return Launch<8>::threads(var);
        case 16: return Launch<16>::threads(var);
        case 32: return Launch<32>::threads(var);
        case 64: return Launch<64>::threads(var);
        case 128: return Launch<128>::threads(var);
        case 256: return Launch<256>::threads(var);
        case 512: return Launch<512>::threads(var);
        default: return Launch<1024>::threads(var);
    }
}

bool col_twins(const Dims& d) {
    if (d.csplit > 0) return d.csplit > 1;
    const int T = fft_threads(d.N, d.cvar), cb = d.cb_auto ? std::max(1, 64 / T) : d.cb;
    const long waves = (long)(d.KXP / cb) * d.B * ((cb * T + 63) / 64);
    return waves < (d.N <= 256 ? 10L : 8L) * std::max(d.cus, 1);
}

int col_block_auto(const Dims& d) {
    if (!col_twins(d)) return std::max(1, std::min(8, 256 / fft_threads(d.N, d.cvar)));
    return (long)d.KXP / 4 * d.B >= std::max(d.cus, 1) / 2 ? 4 : 2;
}

hipError_t launch_row_r2c(const Dims& d, const double* in, cd* out, const cd* tw, hipStream_t s, const MultSpec* m) {
    if (!in || !out || !tw || (m && !m->table)) return hipErrorInvalidValue;
    PA_DISPATCH_N(row_r2c(d, in, out, tw, m, s));
}
hipError_t launch_row_c2r(const Dims& d, const cd* in, double* out, const cd* tw, hipStream_t s) {
    if (!in || !out || !tw) return hipErrorInvalidValue;
    PA_DISPATCH_N(row_c2r(d, in, out, tw, s));
}
hipError_t launch_row_sq(const Dims& d, const RowArgs& a, hipStream_t s) {
    if (!a.yin[0] || !a.yin[1] || !a.yout[0] || !a.yout[1] || !a.tw) return hipErrorInvalidValue;
    PA_DISPATCH_N(row_sq(d, a, s));
}
hipError_t launch_row_obs(const Dims& d, const RowArgs& a, hipStream_t s) {
    if (!a.yin[0] || !a.yin[1] || !a.tw || a.obs.slot < 0 || !obs_ok(a.obs)) return hipErrorInvalidValue;
    PA_DISPATCH_N(row_obs(d, a, s));
}
hipError_t launch_row_mul(const Dims& d, const RowArgs& a, hipStream_t s) {
    for (int i = 0; i < 4; ++i)
        if (!a.yin[i]) return hipErrorInvalidValue;
    if (!a.yout[0] || !a.yout[1] || !a.tw) return hipErrorInvalidValue;
    PA_DISPATCH_N(row_mul(d, a, s));
}
hipError_t launch_row_src(const Dims& d, const RowArgs& a, int mode, hipStream_t s) {
    if (!a.yout[0] || !a.yout[1] || !a.tw ||
        (mode != SRC_IMPULSE && (!a.yin[0] || !a.yin[1] || !a.obs.values || a.obs.slot < 0 || !obs_ok(a.obs))))
        return hipErrorInvalidValue;
    PA_DISPATCH_N(row_src(d, a, mode, s));
}
hipError_t launch_col(const Dims& d, int mode, const ColArgs& a, hipStream_t s) {
    if (!col_ptrs_ok(mode, a)) return hipErrorInvalidValue;
    PA_DISPATCH_N(col(d, mode, a, s));
}

}  // namespace pa
