// kernels_impl.hpp -- row (physical-space) and column (spectral-space) passes.
//
// Row pass: a team of T threads owns one grid row (or a pair of rows) of one
// member.  It rebuilds full complex rows from the stored half spectra
// (Hermitian extension, two real fields packed as re + i im), inverse
// transforms along x, forms the pointwise products of the method in
// registers, and forward transforms the products back, keeping kx <= Kc.
// Column pass: a team owns one kx column of one member; a workgroup holds CB
// adjacent columns so that every global access is a run of CB contiguous
// complex values.  It transforms along y, applies the spectral operators of
// the step mode by mode, and transforms the derived fields back along y.
//
// Included once per grid size by kern_<N>.hip, which instantiates Launch<N>.
#pragma once
#include <algorithm>
#include <atomic>

#include <hip/hip_ext.h>

#include "device_once.hpp"
#include "kernels.hpp"

namespace pa {

// Launch of a row or column kernel: with timing events pending on this
// thread, the dispatch itself records them (hipExtLaunchKernel), so the
// measured time is the kernel's and not that of separate event packets.
template <class F, class... Args>
inline void launch_kernel(F kernel, dim3 grid, dim3 block, size_t lds, hipStream_t s, Args... args) {
    DispatchEvents& e = dispatch_events();
    if (e.start && !e.used) {
        e.used = true;
        hipExtLaunchKernelGGL(kernel, grid, block, (std::uint32_t)lds, s, e.start, e.stop, 0u, args...);
    } else {
        hipLaunchKernelGGL(kernel, grid, block, lds, s, args...);
    }
}

// Global accesses as uniform base + 32-bit byte offset (element index << 4),
// so the backend can address with a scalar base and one 32-bit lane offset.
__device__ __forceinline__ cd ldc(const cd* base, unsigned i) {
    return *reinterpret_cast<const cd*>(reinterpret_cast<const char*>(base) + (i << 4));
}
__device__ __forceinline__ void stc(cd* base, unsigned i, cd v) {
    *reinterpret_cast<cd*>(reinterpret_cast<char*>(base) + (i << 4)) = v;
}

// The twiddle table is copied into LDS at kernel start, in the stage order of
// the plan: reads after a barrier are not hoisted out of loops, so they do
// not pin registers across the successive transforms of a kernel.
template <int N, int V>
__device__ __forceinline__ const cd* stage_twiddles(cd* lds_tw, const cd* __restrict__ tw) {
    for (int i = threadIdx.x; i < N; i += blockDim.x) lds_tw[i] = tw[twiddle_source<N, V>(i)];
    lds_sync();
    return lds_tw;
}

// Row transforms of a kernel whose rows run several transforms with one set of
// twiddle factors per thread.  Plan (256, 2) (one row per wavefront, four
// values per lane) uses the wavefront-resident transform with lane swaps
// (fft256_wave), whose nine factors per thread come straight from the natural
// table; every other plan runs its Stockham stages with the factors of the
// stage-ordered table (staged in LDS by the workgroup) held in registers.
template <int N, int V>
__host__ __device__ constexpr bool wave256() { return N == 256 && V == 2; }

// The 512-point plan and plan (1024, 3) are wavefront-resident too
// (fft512_wave, fft1024_wave) and read their factors from an LDS table of
// their own.
template <int N, int V>
__host__ __device__ constexpr bool wave_long() { return N == 512 || (N == 1024 && V == 3); }

template <int N, int V, bool LONG = wave_long<N, V>()>
struct RowTw {
    TwReg<N, V> r;
};
template <int N, int V>
struct RowTw<N, V, true> {
    const cd* r;
};
template <>
struct RowTw<256, 2, false> {
    Tw256 r;
};

template <int N, int V>
__device__ __forceinline__ void row_twiddles(RowTw<N, V>& tr, int t, const cd* __restrict__ tw_g, cd* tw_lds) {
    if constexpr (wave256<N, V>()) load_tw256(tr.r, t, tw_g);
    else if constexpr (wave_long<N, V>()) tr.r = stage_wave<N>(tw_lds, tw_g);
    else load_twiddles<N, V>(tr.r, t, stage_twiddles<N, V>(tw_lds, tw_g));
}

template <int N, int V, bool INV, bool WL>
__device__ __forceinline__ void row_fft(cd* v, int t, cd* lds, const RowTw<N, V>& tr) {
    if constexpr (wave256<N, V>()) fft256_wave<INV>(v, t, lds, tr.r);
    else if constexpr (N == 512) fft512_wave<INV>(v, t, lds, tr.r);
    else if constexpr (wave_long<N, V>()) fft1024_wave<INV>(v, t, lds, tr.r);
    else fft<N, V, INV, WL>(v, t, lds, tr.r);
}

// Retained band of a grid of size N: the 2/3 rule keeps |kx|, |ky| <= (N-1)/3.
template <int N>
__host__ __device__ constexpr int band() { return (N - 1) / 3; }
// Row pitch of the half-spectrum layouts: kx = 0..K padded to a multiple of 8.
template <int N>
__host__ __device__ constexpr int kx_pad() { return (band<N>() + 1 + 7) / 8 * 8; }

// Whether register slot m of a T-thread team (elements t + T m, t < T) can
// touch the band kx <= K or kx >= N - K; folded at compile time after
// unrolling, so slots that only see the de-aliased gap issue no loads.
template <int N, int V>
__device__ constexpr bool slot_in_band(int m) {
    constexpr int T = Plan<N, V>::T, K = band<N>();
    return T * m <= K || T * m + T - 1 >= N - K;
}
template <int N, int V>
__device__ constexpr bool slot_low(int m) { return Plan<N, V>::T * m <= band<N>(); }

// z = A_full[e] + i B_full[e] for the Hermitian extensions of half-spectrum
// rows A, B (only kx = 0..K stored, zero beyond): two rows of one field packed
// into one transform (the row pass from a single field to physical space).
// The kx = 0 entry of a real field's half spectrum is real; its imaginary
// round-off is discarded.  Branch-free: the load index is clamped to 0 off the
// band and the result selected, so the loads of all slots issue back to back
// instead of each waiting inside a divergent branch.
template <int N>
__device__ __forceinline__ cd herm_pair(const cd* __restrict__ A, const cd* __restrict__ B, int e) {
    constexpr int K = band<N>();
    const bool lo = e <= K, hi = e >= N - K;
    const unsigned k = lo ? (unsigned)e : (hi ? (unsigned)(N - e) : 0u);
    cd a = ldc(A, k), bb = ldc(B, k);
    if (e == 0) { a.y = 0.0; bb.y = 0.0; }
    if (hi) { a.y = -a.y; bb.y = -bb.y; }
    const cd z = mk(a.x - bb.y, a.y + bb.x);
    return (lo || hi) ? z : czero();
}

// Fills the E register slots of a team with the extension of (A, B).
template <int N, int V>
__device__ __forceinline__ void herm_load(cd* z, const cd* __restrict__ A, const cd* __restrict__ B, int t) {
    constexpr int T = Plan<N, V>::T, E = Plan<N, V>::E;
#pragma unroll
    for (int m = 0; m < E; ++m) z[m] = slot_in_band<N, V>(m) ? herm_pair<N>(A, B, t + T * m) : czero();
}

// z = A_full[e] + i B_full[e] from the packed half spectra P = A + i B and
// Q = A - i B of one row: P[e] on the low band, conj(Q[N - e]) on the high
// band (the Hermitian extension of A and B), zero in the de-aliased gap.  Each
// register slot issues one load; which band its lanes can meet is known at
// compile time from the plan, so all-low and all-high slots carry no select.
template <int N, int V>
__device__ __forceinline__ void packed_load(cd* z, const cd* __restrict__ P, const cd* __restrict__ Q, int t) {
    constexpr int T = Plan<N, V>::T, E = Plan<N, V>::E, K = band<N>();
#pragma unroll
    for (int m = 0; m < E; ++m) {
        const int e = t + T * m;
        const bool all_lo = T * m + T - 1 <= K, all_hi = T * m >= N - K;
        const bool may_lo = T * m <= K, may_hi = T * m + T - 1 >= N - K;
        if (all_lo) {
            z[m] = ldc(P, (unsigned)e);
        } else if (all_hi) {
            const cd q = ldc(Q, (unsigned)(N - e));
            z[m] = mk(q.x, -q.y);
        } else if (may_lo && may_hi) {
            const bool lo = e <= K, hi = e >= N - K;
            const cd p = ldc(P, lo ? (unsigned)e : 0u), q = ldc(Q, hi ? (unsigned)(N - e) : 0u);
            z[m] = lo ? p : (hi ? mk(q.x, -q.y) : czero());
        } else if (may_lo) {
            const bool lo = e <= K;
            const cd p = ldc(P, lo ? (unsigned)e : 0u);
            z[m] = lo ? p : czero();
        } else if (may_hi) {
            const bool hi = e >= N - K;
            const cd q = ldc(Q, hi ? (unsigned)(N - e) : 0u);
            z[m] = hi ? mk(q.x, -q.y) : czero();
        } else {
            z[m] = czero();
        }
    }
}

// Forward transform z of a + i b (a, b real) is split into the half spectra
// of a and b:  Ahat[k] = (Z[k] + conj Z[N-k]) / 2,  Bhat[k] = (Z[k] - conj Z[N-k]) / (2i).
// Stores kx = 0..K of both.  The team's lanes write and read consecutive LDS
// entries (forwards, then backwards).
template <int N, int V>
__device__ __forceinline__ void split_store(const cd* z, int t, cd* lds, cd* __restrict__ outA,
                                            cd* __restrict__ outB) {
    constexpr int T = Plan<N, V>::T, E = Plan<N, V>::E, K = band<N>();
#pragma unroll
    for (int m = 0; m < E; ++m) lds[t + T * m] = z[m];
    wave_lds_sync();
#pragma unroll
    for (int m = 0; m < E; ++m) {
        const int k = t + T * m;
        if (slot_low<N, V>(m) && k <= K) {
            const cd zk = z[m];
            const cd zn = lds[(N - k) & (N - 1)];
            outA[k] = mk(0.5 * (zk.x + zn.x), 0.5 * (zk.y - zn.y));
            outB[k] = mk(0.5 * (zk.y + zn.y), -0.5 * (zk.x - zn.x));
        }
    }
}

// Forward transform z of a + i b (a, b real) stored unsplit for k = 0..K:
// P[k] = Z[k] and Q[k] = conj(Z[N - k]), so that a_hat = (P + Q) / 2 and
// b_hat = (P - Q) / (2i) (the column pass forms them).  Each lane stores the
// values it holds: no exchange.
template <int N, int V>
__device__ __forceinline__ void pair_store(const cd* z, int t, cd* __restrict__ outP, cd* __restrict__ outQ) {
    constexpr int T = Plan<N, V>::T, E = Plan<N, V>::E, K = band<N>();
#pragma unroll
    for (int m = 0; m < E; ++m) {
        const int k = t + T * m;
        if (slot_low<N, V>(m) && k <= K) stc(outP, (unsigned)k, z[m]);
        const bool q_slot = m == 0 || T * m + T - 1 >= N - K;   // holds k = 0 or some k >= N - K
        const int kn = (N - k) & (N - 1);
        if (q_slot && kn <= K) stc(outQ, (unsigned)kn, mk(z[m].x, -z[m].y));
    }
}

// Team sum (fixed order) of one double per thread: a butterfly over the team's
// lanes, the result in every one.
template <int N, int V>
__device__ __forceinline__ double team_sum(double v) {
#pragma unroll
    for (int off = Plan<N, V>::T / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Index of probe (x, y) in the observations of one slot, component u (v is
// M^2 further).  The stride divides N, so it is a power of two.
__device__ __forceinline__ size_t probe_index(const RowObs& o, int b, int y, int x) {
    return (((size_t)b * o.n_times + o.slot) * 2) * o.M * o.M + (size_t)(y >> o.ls) * o.M + (x >> o.ls);
}

__device__ __forceinline__ void store_jpart(const RowObs& o, int b, int y, double s) {
    if (o.jpart && o.values) o.jpart[((size_t)b * o.n_times + o.slot) * o.M + (y >> o.ls)] = 0.5 * s;
}

// The observed velocities of the row's probes that a thread holds (0 where it
// holds none), every load issued at a valid address.
template <int N, int V>
__device__ __forceinline__ void probe_values(const RowObs& o, int b, int y, int t, cd* val) {
    constexpr int T = Plan<N, V>::T, E = Plan<N, V>::E;
#pragma unroll
    for (int m = 0; m < E; ++m) {
        const int x = t + T * m;
        const bool probe = (x & (o.stride - 1)) == 0;
        const size_t i = probe_index(o, b, y, probe ? x : 0);
        const cd q = mk(o.values[i], o.values[i + (size_t)o.M * o.M]);
        val[m] = probe ? q : czero();
    }
}

// LDS entries of a row team's exchange area: the padded one of the Stockham
// plans, or N where the transform is wavefront-resident (four workgroups of
// four 512-point rows, or two of four 1024-point rows, with their tables fill
// a CU's 160 KiB).
template <int N, int V>
__host__ __device__ constexpr int row_area() { return wave_long<N, V>() ? N : lds_team<N>(); }

// A workgroup holds `tpb` teams; the launcher guarantees tpb divides the
// teams per member, so the member index is uniform over the workgroup and
// member base pointers live in scalar registers (32-bit lane offsets).  A
// team of at most 64 threads lies within one wavefront (WL): its exchanges
// synchronise the wave only, and the one workgroup barrier is the twiddle
// staging.
#define PA_TEAM_SETUP(N, V, TEAMS_PER_MEMBER) PA_TEAM_SETUP_AT(N, V, TEAMS_PER_MEMBER, blockIdx.x)
#define PA_TEAM_SETUP_AT(N, V, TEAMS_PER_MEMBER, BLOCK)                 \
    constexpr int T = Plan<N, V>::T, E = Plan<N, V>::E;                 \
    constexpr bool WL = T <= 64 && 64 % T == 0;                         \
    extern __shared__ cd smem[];                                        \
    const int team = threadIdx.x / T, t = threadIdx.x % T;              \
    cd* lds = smem + team * row_area<N, V>();                           \
    const int tpb_ = blockDim.x / T;                                    \
    cd* const tw_lds = smem + tpb_ * row_area<N, V>();                  \
    const int g0 = (int)(BLOCK) * tpb_;                                 \
    const int b = g0 / (TEAMS_PER_MEMBER);                              \
    const int w0 = g0 % (TEAMS_PER_MEMBER);                             \
    const int wi = w0 + team;

// ------------------------------------------------------------ row passes --

// physical rows (y0, y0+1) -> Y rows; team per row pair.  The first `fill`
// workgroups fill the multiplier table of the launch instead: one launch less
// takes a preconditioner call from 19.9 to 18.8 us at 128^2 (the host enqueues a
// launch in about 3 us, and such a call runs no faster than that).
template <int N, int V>
__global__ void __launch_bounds__(256) row_r2c_kernel(Dims d, const double* __restrict__ in, cd* __restrict__ out,
                                                      const cd* __restrict__ tw_g, MultSpec mult, unsigned fill) {
    if (blockIdx.x < fill) {   // uniform over the workgroup
        const int n = d.KY * d.KXP;
        for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < (unsigned)n; i += fill * blockDim.x)
            fill_mult(d, mult, (int)i);
        return;
    }
    PA_TEAM_SETUP_AT(N, V, N / 2, blockIdx.x - fill)
    const double* r0 = in + ((size_t)b * N + 2 * w0) * N;     // block base (uniform)
    const int ro = 2 * team * N;                               // this team's row pair
    cd z[E];
#pragma unroll
    for (int m = 0; m < E; ++m) {
        const int x = t + T * m;
        z[m] = mk(r0[ro + x], r0[ro + N + x]);
    }
    RowTw<N, V> tr;
    row_twiddles<N, V>(tr, t, tw_g, tw_lds);
    row_fft<N, V, false, WL>(z, t, lds, tr);
    cd* o0 = out + ((size_t)b * N + 2 * wi) * kx_pad<N>();
    split_store<N, V>(z, t, lds, o0, o0 + kx_pad<N>());
}

// Y rows (y0, y0+1) -> physical rows.
template <int N, int V>
__global__ void __launch_bounds__(256) row_c2r_kernel(Dims d, const cd* __restrict__ in,
                                                      double* __restrict__ out, const cd* __restrict__ tw_g) {
    PA_TEAM_SETUP(N, V, N / 2)
    const cd* i0 = in + ((size_t)b * N + 2 * wi) * kx_pad<N>();
    cd z[E];
    herm_load<N, V>(z, i0, i0 + kx_pad<N>(), t);
    RowTw<N, V> tr;
    row_twiddles<N, V>(tr, t, tw_g, tw_lds);
    row_fft<N, V, true, WL>(z, t, lds, tr);
    double* r0 = out + ((size_t)b * N + 2 * w0) * N;
    const int ro = 2 * team * N;
#pragma unroll
    for (int m = 0; m < E; ++m) {
        const int x = t + T * m;
        r0[ro + x] = z[m].x;
        r0[ro + N + x] = z[m].y;
    }
}

// The row passes work on velocities only.  With div u = 0 the advection term is
//   u . grad w = (d_xx - d_yy)(u v) + d_xy(v^2 - u^2),
// so a right-hand side needs two fields in physical space instead of the four
// of u w_x + v w_y.  They travel as the one complex signal z = u + i v, whose
// square z^2 = (u^2 - v^2) + i 2 u v holds both products: two transforms per
// row, two fields read and two written (2 + 2 against 4 + 1 and 2.5).  Its
// transpose multiplies by conj(z): with a = (d_yy - d_xx) Lam and
// b = 2 d_xy Lam (as multipliers kx^2 - ky^2 and -2 kx ky of the spectrum),
//   N'(w)^T Lam = U^T(a v + b u) + V^T(a u - b v),
// and (a v + b u) + i (a u - b v) = (b + i a) conj(z).  On the de-aliased band
// both identities hold exactly (every alias of a product falls outside it).
//
// Rounding.  The multipliers kx ky and kx^2 - ky^2 act after the products here
// and so on their rounding too, which is white; in advective form the
// derivatives come before.  Distance of the forward state from a long-double run
// (relative L2, 20 steps unless noted), advective form -> this one: decaying flow with
// its peak at k0 = N/25, 256^2 3.5e-15 -> 3.0e-15, 512^2 9.1e-15 -> 2.3e-15, 1024^2
// 3.3e-14 -> 2.6e-15; Kolmogorov flow (nu = 1/40, k0 = 4), 512^2 40 steps 4.19e-15
// both, 6 steps 6.8e-16 -> 7.7e-16, 1024^2 30 steps 3.2e-15 -> 3.3e-15.  Where the peak lies
// far below the band's edge and little damps that edge it is larger: nu = 1e-4,
// k0 = 4, 256^2 3.7e-15 -> 3.9e-15, 512^2 2.5e-15 -> 3.4e-15, 1024^2 2.4e-15 -> 7.1e-15.
// Gradients are closer in every case: 256^2 k0 = 10 1.4e-14 -> 3.3e-15, 512^2 k0 = 4
// 3.4e-15 -> 3.0e-15, 1024^2 k0 = 41 2.7e-13 -> 1.9e-15, k0 = 4 1.16e-15 -> 1.06e-15.
//
// The passes are bound by HBM traffic at large batches (64 x 256^2: 464 instead
// of 548 bytes per grid point and forward + adjoint step).  Per launch there,
// advective form -> this one: forward rows 27.3 -> 21.6 us (4.2 TB/s), adjoint
// rows 38.7 -> 28.0 us (4.8 TB/s); the tape holds half the fields.

// z^2 and w conj(z)
__device__ __forceinline__ cd csq(cd z) { return mk((z.x - z.y) * (z.x + z.y), 2.0 * z.x * z.y); }

// Right-hand side products of one row.  Inputs yin[0..1] = the packed velocity
// (u, v), outputs yout[0..1] = the row transform Z of z^2, unsplit
// (pair_store): Z and conj Z(-k).  Observations are formed by row_obs_kernel
// from the same field.
template <int N, int V>
constexpr int sq_waves() { return Plan<N, V>::E <= 4 ? 5 : Plan<N, V>::E <= 8 ? 4 : 2; }

template <int N, int V>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sq_waves<N, V>())))
row_sq_kernel(Dims d, RowArgs a) {
    const cd* __restrict__ tw_g = a.tw;
    PA_TEAM_SETUP(N, V, N)
    const size_t roff = ((size_t)b * N + wi) * kx_pad<N>();
    cd z[E];
    packed_load<N, V>(z, a.yin[0] + roff, a.yin[1] + roff, t);
    RowTw<N, V> tr;   // both transforms share the thread's twiddles
    row_twiddles<N, V>(tr, t, tw_g, tw_lds);
    row_fft<N, V, true, WL>(z, t, lds, tr);
#pragma unroll
    for (int m = 0; m < E; ++m) z[m] = csq(z[m]);
    row_fft<N, V, false, WL>(z, t, lds, tr);
    pair_store<N, V>(z, t, a.yout[0] + roff, a.yout[1] + roff);
}

// Observation of one step: team per observed row; yin[0..1] = the packed
// velocity of the state.  A launch of a few rows is one chain of latencies:
// loads, transform, probes, team sum.  The row plans of the products (one LDS
// exchange or none) and shifts in place of divisions in the probe index take
// it from 6.2 to 4.1 us at 128^2 and from 14.7 to 7.8 us at 1024^2 (row_src
// from 6.1 to 4.0 and from 13 to 9.3 us).
template <int N, int V>
__global__ void __launch_bounds__(256) row_obs_kernel(Dims d, RowArgs a) {
    const cd* __restrict__ tw_g = a.tw;
    PA_TEAM_SETUP(N, V, a.obs.M)
    const RowObs& o = a.obs;
    const int y = wi << o.ls;
    const size_t roff = ((size_t)b * N + y) * kx_pad<N>();
    cd z[E], val[E];
    packed_load<N, V>(z, a.yin[0] + roff, a.yin[1] + roff, t);
    if (o.values) probe_values<N, V>(o, b, y, t, val);
    RowTw<N, V> tr;
    row_twiddles<N, V>(tr, t, tw_g, tw_lds);
    row_fft<N, V, true, WL>(z, t, lds, tr);
    double part = 0.0;
#pragma unroll
    for (int m = 0; m < E; ++m) {
        const int x = t + T * m;
        if ((x & (o.stride - 1)) != 0) continue;
        if (o.obs_out) {
            const size_t i = probe_index(o, b, y, x);
            o.obs_out[i] = z[m].x;
            o.obs_out[i + (size_t)o.M * o.M] = z[m].y;
        }
        if (o.values) {
            const double ru = z[m].x - val[m].x, rv = z[m].y - val[m].y;
            part += ru * ru;
            part += rv * rv;
        }
    }
    const double s = team_sum<N, V>(part);
    if (t == 0) store_jpart(o, b, y, s);
}

// Occupancy hint for the adjoint row pass (two signals per thread).
template <int N, int V>
constexpr int mul_waves() { return Plan<N, V>::E <= 4 ? 4 : Plan<N, V>::E <= 8 ? 3 : 1; }

// Adjoint products of one row.  Inputs yin[0..1] = the packed velocity (u, v)
// of the stage state, yin[2..3] = the packed pair (b, a) of the cotangent;
// outputs yout[0..1] = the row transform Z of (b + i a) conj(z), unsplit.
template <int N, int V>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(mul_waves<N, V>())))
row_mul_kernel(Dims d, RowArgs a) {
    const cd* __restrict__ tw_g = a.tw;
    PA_TEAM_SETUP(N, V, N)
    const size_t roff = ((size_t)b * N + wi) * kx_pad<N>();
    cd w[E], z[E];
    packed_load<N, V>(w, a.yin[2] + roff, a.yin[3] + roff, t);
    packed_load<N, V>(z, a.yin[0] + roff, a.yin[1] + roff, t);
    RowTw<N, V> tr;   // the three transforms of the row share the thread's twiddles
    row_twiddles<N, V>(tr, t, tw_g, tw_lds);
    row_fft<N, V, true, WL>(w, t, lds, tr);
    row_fft<N, V, true, WL>(z, t, lds, tr);
#pragma unroll
    for (int m = 0; m < E; ++m) w[m] = cmulc(w[m], z[m]);
    row_fft<N, V, false, WL>(w, t, lds, tr);
    pair_store<N, V>(w, t, a.yout[0] + roff, a.yout[1] + roff);
}

// Adjoint source rows: the row transform Z of r_u + i r_v on the probes of one
// observed step (yin[0..1] = the packed velocity of that state) or of a unit
// u-impulse at (imp_x, imp_y), in the form of the adjoint products, whose
// U^T and V^T it shares.  SRC_WRITE and SRC_IMPULSE cover every row of the
// member; SRC_ADD covers the observed rows (team per observed row) and adds to
// the products already there.
template <int N, int V, int MODE>
__global__ void __launch_bounds__(256) row_src_kernel(Dims d, RowArgs a) {
    constexpr int K = band<N>();
    const cd* __restrict__ tw_g = a.tw;
    PA_TEAM_SETUP(N, V, MODE == SRC_ADD ? a.obs.M : N)
    const RowObs& o = a.obs;
    const int y = MODE == SRC_ADD ? wi << o.ls : wi;
    const size_t roff = ((size_t)b * N + y) * kx_pad<N>();
    const bool row = MODE == SRC_IMPULSE ? y == o.imp_y : (y & (o.stride - 1)) == 0;   // else the row is zero
    cd* const outP = a.yout[0] + roff;
    cd* const outQ = a.yout[1] + roff;
    cd z[E], val[E], p[E], q[E];
    if constexpr (MODE != SRC_IMPULSE) {
        packed_load<N, V>(z, a.yin[0] + roff, a.yin[1] + roff, t);
        probe_values<N, V>(o, b, row ? y : 0, t, val);
    }
    RowTw<N, V> tr;
    row_twiddles<N, V>(tr, t, tw_g, tw_lds);
    if constexpr (MODE != SRC_IMPULSE) row_fft<N, V, true, WL>(z, t, lds, tr);
    if constexpr (MODE == SRC_ADD) {   // the products the sources are added to
#pragma unroll
        for (int m = 0; m < E; ++m) {
            const int k = t + T * m, kn = (N - k) & (N - 1);
            if (slot_low<N, V>(m)) p[m] = ldc(outP, (unsigned)(k <= K ? k : 0));
            if (m == 0 || T * m + T - 1 >= N - K) q[m] = ldc(outQ, (unsigned)(kn <= K ? kn : 0));
        }
    }
#pragma unroll
    for (int m = 0; m < E; ++m) {
        const int x = t + T * m;
        if constexpr (MODE == SRC_IMPULSE) z[m] = mk(row && x == o.imp_x ? 1.0 : 0.0, 0.0);
        else z[m] = row && (x & (o.stride - 1)) == 0 ? mk(z[m].x - val[m].x, z[m].y - val[m].y) : czero();
    }
    row_fft<N, V, false, WL>(z, t, lds, tr);
    if constexpr (MODE == SRC_ADD) {
#pragma unroll
        for (int m = 0; m < E; ++m) {
            const int k = t + T * m, kn = (N - k) & (N - 1);
            if (slot_low<N, V>(m) && k <= K) stc(outP, (unsigned)k, cadd(p[m], z[m]));
            if ((m == 0 || T * m + T - 1 >= N - K) && kn <= K) stc(outQ, (unsigned)kn, cadd(q[m], cconj(z[m])));
        }
    } else {
        pair_store<N, V>(z, t, outP, outQ);
    }
}

// Returns v unchanged, opaquely: index arithmetic derived from it is neither
// hoisted out of a loop nor kept from an earlier phase of a kernel (where its
// results would occupy registers across the transforms) but recomputed.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// ---------------------------------------------------------- column pass --

// Position of workgroup `id` of a one-dimensional grid of `n` in an order in
// which each XCD holds a contiguous run: workgroup id runs on XCD id % XCDS
// (round-robin dispatch), and that XCD's k-th workgroup takes the k-th entry
// of its run.  A bijection of 0..n-1 for any n, so only locality depends on it.
constexpr unsigned XCDS = 8;
__device__ __forceinline__ unsigned xcd_order(unsigned id, unsigned n) {
    const unsigned x = id % XCDS, k = id / XCDS;
    const unsigned q = n / XCDS, r = n % XCDS;   // XCDs below r hold q + 1 workgroups
    return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + k;
}

// Compact outputs and tables of a column launch, at the workgroup's member and
// first column.
struct ColPtrs {
    cd *om, *ac, *ck, *lm, *ob;
    const cd *p0, *p1;       // compact operands: (omega_n, acc) forward, (lambda, omega-bar) adjoint
    const double* ik2;
    double ex, sc;
};

template <int MODE>
struct ColTraits {
    static constexpr bool FWD = MODE >= COL_A && MODE <= COL_D;
    static constexpr bool ADJ = MODE >= COL_ADJ_C && MODE <= COL_ADJ_SRC;
    static constexpr bool PAIR_IN = FWD || ADJ || MODE == COL_FIRST_GUESS;
    static constexpr bool NEED0 = FWD || MODE == COL_FROM_STATE || (ADJ && MODE != COL_ADJ_N && MODE != COL_ADJ_SRC);
    static constexpr bool NEED1 = (FWD && MODE != COL_A) || (ADJ && MODE != COL_ADJ_C && MODE != COL_ADJ_SRC);
};

template <int MODE>
__device__ __forceinline__ ColPtrs col_ptrs(const ColArgs& a, size_t cmem, int b, int kx0, int kx) {
    using M = ColTraits<MODE>;
    ColPtrs q;
    q.om = a.omega ? (MODE == COL_D && a.omega_out ? a.omega_out : a.omega) + cmem : nullptr;
    q.ac = a.acc ? a.acc + cmem : nullptr;
    q.ck = a.ckpt ? a.ckpt + cmem : nullptr;
    q.lm = M::ADJ ? a.lam + cmem : nullptr;
    q.ob = M::ADJ && a.omb ? a.omb + cmem : nullptr;
    q.p0 = M::FWD ? a.omega + cmem : M::ADJ ? a.lam + cmem : a.state_in + cmem;
    q.p1 = M::FWD ? a.acc + cmem : a.omb + cmem;
    q.ik2 = a.invk2 + kx0;
    q.ex = a.ex2[kx];
    q.sc = (M::ADJ || MODE == COL_FROM_STATE) && a.scale ? a.scale[b] : 1.0;
    return q;
}

// What a mode's transformed inputs P, Q give (0 off the band and for the mean):
// the nonlinear term of a forward stage, the cotangent of an adjoint stage, the
// vorticity of probe velocities, or the one input itself.
template <int MODE>
__device__ __forceinline__ cd col_pair_value(const ColArgs& a, bool ins, double ik2, int kx, int ky_, cd P, cd Q) {
    const double dkx = (double)kx, ky = (double)ky_;
    if constexpr (ColTraits<MODE>::FWD) {
        // -P u . grad w = beta (P + Q) + alpha (P - Q)/i with the spectra of z^2,
        // alpha = (kx^2 - ky^2)/4, beta = -kx ky/2
        const double al = 0.25 * (dkx * dkx - ky * ky), be = -0.5 * dkx * ky;
        return ins ? mk(be * (P.x + Q.x) + al * (P.y - Q.y), be * (P.y + Q.y) - al * (P.x - Q.x)) : czero();
    } else if constexpr (ColTraits<MODE>::ADJ) {
        // U^T and V^T of the products, ((kx - i ky) P - (kx + i ky) Q) / (2 |k|^2)
        const double f = 0.5 * ik2;
        return ins ? mk(f * (dkx * (P.x - Q.x) + ky * (P.y + Q.y)), f * (dkx * (P.y - Q.y) - ky * (P.x + Q.x))) : czero();
    } else if constexpr (MODE == COL_FIRST_GUESS) {
        // vorticity of the low-passed probe velocity: i kx v_hat - i ky u_hat on S
        const bool keep = ins && kx <= a.lowpass && ky_ <= a.lowpass && -ky_ <= a.lowpass;
        return keep ? mk(-dkx * Q.y + ky * P.y, dkx * Q.x - ky * P.x) : czero();
    } else {
        return ins ? P : czero();
    }
}

// The rest of a mode's spectral work: its pair value nl and compact operands
// s0, s1 in, compact outputs written at ci (when `on`: the mode lies in the
// band), the value handed to the output transforms returned.  r is the compact
// row, ins: in the band and not the mean.
template <int N, int MODE>
__device__ __forceinline__ cd col_mode_update(const ColArgs& a, const ColPtrs& q, bool on, bool ins, unsigned ci,
                                              int b, int kx, int r, int ky_, double ey2, cd nl, cd s0, cd s1) {
    constexpr int KXP = kx_pad<N>(), KY = 2 * band<N>() + 1;
    const double h = a.h;
    const double e2 = q.ex * ey2, e1 = e2 * e2;
    if constexpr (MODE == COL_INIT) {
        if (on) {
            if (q.om) stc(q.om, ci, nl);
            if (q.ck) stc(q.ck, ci, nl);
        }
        return nl;
    } else if constexpr (MODE == COL_FILTER) {
        const size_t mi = (a.mult_per_member ? (size_t)b * KY * KXP : 0) + (size_t)r * KXP + kx;
        return cscale(nl, a.mult[mi]);
    } else if constexpr (MODE == COL_FIRST_GUESS) {
        return nl;
    } else if constexpr (MODE == COL_FROM_STATE) {
        const cd w = ins ? s0 : czero();
        if (on && q.om) stc(q.om, ci, w);
        return cscale(w, q.sc);
    } else if constexpr (ColTraits<MODE>::FWD) {
        if (a.nf > 0 && kx == 0 && (ky_ == a.nf || ky_ == -a.nf)) nl.x += a.forcing;
        if constexpr (MODE == COL_A) {
            if (on && q.ac) stc(q.ac, ci, cscale(nl, e1));
            return cscale(mk(s0.x + 0.5 * h * nl.x, s0.y + 0.5 * h * nl.y), e2);
        } else if constexpr (MODE == COL_D) {
            const double h6 = h / 6.0;
            const cd w = mk(e1 * s0.x + h6 * (s1.x + nl.x), e1 * s0.y + h6 * (s1.y + nl.y));
            if (on) {
                if (q.om) stc(q.om, ci, w);
                if (q.ck) stc(q.ck, ci, w);
            }
            return w;
        } else {
            if (on && q.ac) stc(q.ac, ci, mk(s1.x + 2.0 * e2 * nl.x, s1.y + 2.0 * e2 * nl.y));
            if constexpr (MODE == COL_B) return mk(e2 * s0.x + 0.5 * h * nl.x, e2 * s0.y + 0.5 * h * nl.y);
            else return mk(e1 * s0.x + h * e2 * nl.x, e1 * s0.y + h * e2 * nl.y);
        }
    } else {
        const cd wb = nl;
        if constexpr (MODE == COL_ADJ_C) {
            if (on && q.ob) stc(q.ob, ci, mk(e1 * (s0.x + wb.x), e1 * (s0.y + wb.y)));
            return mk((h / 3.0) * e2 * s0.x + h * e2 * wb.x, (h / 3.0) * e2 * s0.y + h * e2 * wb.y);
        } else if constexpr (MODE == COL_ADJ_B) {
            if (on && q.ob) stc(q.ob, ci, mk(s1.x + e2 * wb.x, s1.y + e2 * wb.y));
            return mk((h / 3.0) * e2 * s0.x + 0.5 * h * wb.x, (h / 3.0) * e2 * s0.y + 0.5 * h * wb.y);
        } else if constexpr (MODE == COL_ADJ_A) {
            if (on && q.ob) stc(q.ob, ci, mk(s1.x + e2 * wb.x, s1.y + e2 * wb.y));
            return mk((h / 6.0) * e1 * s0.x + 0.5 * h * e2 * wb.x, (h / 6.0) * e1 * s0.y + 0.5 * h * e2 * wb.y);
        } else {   // stage n, COL_ADJ_SRC
            cd ln = wb;
            if constexpr (MODE == COL_ADJ_N) ln = mk(s1.x + wb.x, s1.y + wb.y);
            if (on && q.lm) stc(q.lm, ci, ln);
            return a.final_out ? cscale(ln, q.sc) : cscale(ln, h / 6.0);
        }
    }
}

// Derived fields of a mode: 1_S * multiplier * w / N^2.  The two halves
// A + i B (second = false) and A - i B of a packed pair are formed before the
// transform (it is linear): velocity u +- i v has (+-kx + i ky) / |k|^2, the
// cotangent b +- i a has -2 kx ky +- i (kx^2 - ky^2).
template <int N>
__device__ __forceinline__ cd col_field(int kind, bool second, bool ins, double ik2, int kx, int ky_, cd w) {
    if (!ins) return czero();
    const double dkx = (double)kx, ky = (double)ky_;
    const cd s = cscale(w, 1.0 / ((double)N * (double)N));
    if (kind == F_OMEGA) return s;
    double fr, fi;
    if (kind == F_ZP) {
        fr = (second ? -dkx : dkx) * ik2;
        fi = ky * ik2;
    } else {
        fr = -2.0 * dkx * ky;
        fi = second ? ky * ky - dkx * dkx : dkx * dkx - ky * ky;
    }
    return mk(s.x * fr - s.y * fi, s.x * fi + s.y * fr);
}

// Whether a column plan is the register-trading one (fft_trade): the plans of
// eight values per thread from 128 points.
template <int N, int V>
__host__ __device__ constexpr bool col_trade() { return N >= 128 && Plan<N, V>::E == 8; }

template <int N, int V>
__host__ __device__ constexpr int col_area() { return col_trade<N, V>() ? N : lds_team<N>(); }

template <int N, int V>
__device__ __forceinline__ const cd* col_twiddles(cd* lds_tw, const cd* __restrict__ tw) {
    if constexpr (col_trade<N, V>()) return stage_trade<N>(lds_tw, tw);
    else return stage_twiddles<N, V>(lds_tw, tw);
}

// Where a thread of a column kernel works: column c of its workgroup, thread t of
// the team.  The register-trading plan leaves `low` lane bits to columns and
// t_lo (three, or two beside a twin bit); `id` counts the threads of a signal.
struct ColPlace {
    int c, t;
    TradeSpread spread;
};
template <int N, int V>
__device__ __forceinline__ ColPlace col_place(int CB, int id, int low, int twin) {
    ColPlace p;
    if constexpr (col_trade<N, V>()) {
        const int lane = threadIdx.x & 63, g = (lane & ((1 << low) - 1)) + ((int)(threadIdx.x >> 6) << low);
        p.c = g % CB;
        p.t = g / CB + TradePlan<N>::TL * (lane >> 3);
        const int lc = CB >= (1 << low) ? low : CB == 4 ? 2 : CB == 2 ? 1 : 0;   // column bits in the low lanes
        p.spread.nl = low - lc;
        p.spread.cols = ((p.c & ((1 << lc) - 1)) | (twin << lc)) << (low - lc + 1);
    } else {
        p.c = id % CB;
        p.t = id / CB;
        p.spread = TradeSpread{0, 0};
    }
    return p;
}

// A column transform by the thread at `p`.
template <int N, int V, bool INV>
__device__ __forceinline__ void col_fft(cd* v, const ColPlace& p, cd* lds, const cd* __restrict__ twl) {
    if constexpr (col_trade<N, V>())
        fft_trade<N, INV>(v, p.t % TradePlan<N>::TL, p.t / TradePlan<N>::TL, p.spread, lds, twl);
    else fft<N, V, INV>(v, p.t, lds, twl);
}

// Two forms of the column pass, with the same arithmetic per value, so a
// result does not depend on the form:
//
// col_pass_kernel: a thread runs both signals (P, then Q) of a pair one after
// the other.  A workgroup needs one exchange area per column, so three
// workgroups of eight 256-point columns share a CU: the form for launches that
// fill the chip (64 x 256^2: 28.9 us per forward stage and 27.3 per adjoint
// stage, 4.6 and 4.8 TB/s, against 31.0 and 29.4 on twin teams).
//
// col_twin_kernel: the two signals run on twin teams of one workgroup: thread
// t of column c of twin 0 holds P[t + T m], its twin the same entries of Q.  The
// spectral work of a mode needs both, so between the transforms the twins trade
// halves: pair p of registers (p, E-1-p) is exchanged such that twin 0 holds P
// and Q of entry t + T p (ky >= 0) and twin 1 those of entry t + T (E-1-p)
// (ky < 0).  Each mode is then loaded, combined and written once, and the same
// exchange hands the output pair back to the transforms.  Twins sit 4 lanes
// apart with the register-trading plan (a DPP rotation) and 16 with the others
// (v_permlane16_swap): no LDS; pairs that lie in the de-aliased gap are not exchanged at all.  The chain of a
// launch is two transforms instead of four: the form for launches with too few
// columns to fill the chip (forward stage against one team per column: one
// 256^2 member 8.1 against 11.2 us, 32 members 18.3 against 22.6; eight 512^2
// members 21.9 against 25.6; one 1024^2 member 22.3 against 25.5).
template <int N, int V>
__device__ __forceinline__ void twin_swap(double& a, double& b, int twin, int lanes) {
    if constexpr (col_trade<N, V>()) {
        lane_swap4(a, b);
    } else if constexpr (N >= 64) {
        lane_swap16(a, b);
    } else {   // the smallest grids: teams of fewer than 16 lanes per twin
        const double got = __shfl_xor(twin ? a : b, lanes);
        if (twin) a = got;
        else b = got;
    }
}
template <int N, int V>
__device__ __forceinline__ void twin_swap(cd& a, cd& b, int twin, int lanes) {
    twin_swap<N, V>(a.x, b.x, twin, lanes);
    twin_swap<N, V>(a.y, b.y, twin, lanes);
}

// Most threads of a twin workgroup: plans of up to eight values per thread fit
// 128 VGPRs.
template <int N, int V>
constexpr int twin_threads() { return Plan<N, V>::E <= 8 ? 1024 : 512; }

template <int N, int V>
__host__ __device__ constexpr size_t col_lds(int areas) { return ((size_t)areas * col_area<N, V>() + N) * sizeof(cd); }

// One-dimensional grid of (member, column block), block fastest.  The hardware
// hands workgroups to the XCDs round robin by id; each XCD is given a
// contiguous run of that order instead, so that the column blocks of one
// 128-byte line meet in one L2 rather than fetching and writing the line from
// several.
#define PA_COL_SETUP(N)                                                               \
    constexpr int K = band<N>(), KXP = kx_pad<N>(), KY = 2 * K + 1;                   \
    using MT = ColTraits<MODE>;                                                       \
    const unsigned wg = xcd_order(blockIdx.x, gridDim.x);                             \
    const unsigned nblk = (unsigned)(KXP / CB);                                       \
    const int b = (int)(wg / nblk);                                                   \
    const int kx0 = (int)(wg % nblk) * CB;   /* uniform first column of the block */  \
    const int kx = kx0 + c;                                                           \
    const bool colok = kx <= K;                                                       \
    const size_t ymem = (size_t)b * N * KXP + kx0;                                    \
    const size_t cmem = (size_t)b * KY * KXP + kx0;                                   \
    auto yoff = [&](int m, int t_) { return (unsigned)c + (unsigned)(t_ + T * m) * (unsigned)KXP; };

template <int N, int V, int MODE>
__global__ void __launch_bounds__((twin_threads<N, V>())) col_twin_kernel(Dims d, ColArgs a) {
    constexpr int T = Plan<N, V>::T, E = Plan<N, V>::E, EP = E / 2;
    extern __shared__ cd smem[];
    const int CB = a.cb;
    constexpr bool TRADE = col_trade<N, V>();
    const int lanes = TRADE ? 4 : N >= 64 ? 16 : (CB * T < 16 ? CB * T : 16);   // lanes of one twin in a row
    const int twin = ((int)threadIdx.x / lanes) & 1;
    const ColPlace at =
        col_place<N, V>(CB, (int)threadIdx.x % lanes + (int)threadIdx.x / (2 * lanes) * lanes, 2, twin);
    const int c = at.c, t = at.t;
    cd* lds = smem + (twin * CB + c) * col_area<N, V>();
    PA_COL_SETUP(N)
    // the mode this thread works on in pair p: its entry, whether it lies in the band, its compact row
    auto pair_on = [](int p) { return T * p <= K; };   // folds at compile time
    auto ky_of = [&](int p, int t_) { return twin ? t_ + T * (E - 1 - p) - N : t_ + T * p; };
    auto in_band = [&](int p, int t_) { return colok && ky_of(p, t_) <= K && -ky_of(p, t_) <= K; };
    auto row_of = [&](int p, int t_) { return in_band(p, t_) ? ky_of(p, t_) + (twin ? KY : 0) : 0; };
    auto cidx = [&](int p, int t_) { return (unsigned)c + (unsigned)row_of(p, t_) * (unsigned)KXP; };

    // ---- issue every global load first: the input column and the operands of the
    // thread's modes.  Loads are unconditional at in-bounds addresses (padding
    // columns kx < KXP, compact row 0 for modes off the band) and their results
    // selected, so no load sits in a branch.
    cd v[E];
    if constexpr (MODE != COL_FROM_STATE) {
        const bool has = MT::PAIR_IN || twin == 0;   // a single field: the other twin's signal is zero
        const cd* __restrict__ src = (MT::PAIR_IN && twin ? a.yin[1] : a.yin[0]) + ymem;
#pragma unroll
        for (int m = 0; m < E; ++m) {
            const cd x = ldc(src, yoff(m, t));
            v[m] = colok && has ? x : czero();
        }
    }
    const ColPtrs q = col_ptrs<MODE>(a, cmem, b, kx0, kx);
    cd s0[EP], s1[EP];
    double ik2[EP], ey2[EP];   // 1/|k|^2 and the y factor of the integrating factor: loaded here as well, a
                               // load after the transform would wait for memory once more
#pragma unroll
    for (int p = 0; p < EP; ++p) {
        s0[p] = s1[p] = czero();
        ik2[p] = ey2[p] = 0.0;
        if (!pair_on(p)) continue;
        if constexpr (MT::NEED0) s0[p] = ldc(q.p0, cidx(p, t));
        if constexpr (MT::NEED1) s1[p] = ldc(q.p1, cidx(p, t));
        ik2[p] = q.ik2[cidx(p, t)];
        ey2[p] = a.ey2[row_of(p, t)];
    }
    const cd* twl = col_twiddles<N, V>(smem + 2 * CB * col_area<N, V>(), a.tw);
    if constexpr (MODE != COL_FROM_STATE) {
        col_fft<N, V, false>(v, at, lds, twl);
#pragma unroll
        for (int p = 0; p < EP; ++p)
            if (pair_on(p)) twin_swap<N, V>(v[p], v[E - 1 - p], twin, lanes);
    }
    const int kind = a.nout > 0 ? a.fields[0] : F_OMEGA;
    const int tu = opaque(t);
#pragma unroll
    for (int p = 0; p < EP; ++p) {
        cd& P = v[p];
        cd& Q = v[E - 1 - p];
        if (!pair_on(p)) {
            P = Q = czero();
            continue;
        }
        const bool on = in_band(p, tu);
        const unsigned ci = cidx(p, tu);
        const int r = row_of(p, tu), ky = ky_of(p, tu);
        const bool ins = on && !(kx == 0 && r == 0);
        const cd nl = col_pair_value<MODE>(a, ins, ik2[p], kx, ky, P, Q);
        const cd w = col_mode_update<N, MODE>(a, q, on, ins, ci, b, kx, r, ky, ey2[p], nl, s0[p], s1[p]);
        P = col_field<N>(kind, false, ins, ik2[p], kx, ky, w);
        Q = kind == F_OMEGA ? czero() : col_field<N>(kind, true, ins, ik2[p], kx, ky, w);
    }
    if (a.nout < 1) return;   // uniform over the grid
#pragma unroll
    for (int p = 0; p < EP; ++p)
        if (pair_on(p)) twin_swap<N, V>(v[p], v[E - 1 - p], twin, lanes);
    col_fft<N, V, true>(v, at, lds, twl);
    if (colok && twin < a.nout) {
        cd* __restrict__ out = (twin ? a.yout[1] : a.yout[0]) + ymem;
#pragma unroll
        for (int m = 0; m < E; ++m) stc(out, yoff(m, tu), v[m]);
    }
}

// Occupancy hint for col_pass_kernel: three waves per SIMD (168 VGPRs) for the
// plans of up to eight values per thread; sixteen values per thread are left
// unconstrained (a cap there spills hundreds of bytes).
template <int N, int V>
constexpr int col_waves() { return Plan<N, V>::E <= 8 ? 3 : 1; }

// Up to 512 threads: CB columns of T threads each.
template <int N, int V, int MODE>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(col_waves<N, V>())))
col_pass_kernel(Dims d, ColArgs a) {
    constexpr int T = Plan<N, V>::T, E = Plan<N, V>::E;
    extern __shared__ cd smem[];
    const int CB = a.cb;
    const ColPlace at = col_place<N, V>(CB, (int)threadIdx.x, 3, 0);
    const int c = at.c, t = at.t;
    cd* lds = smem + c * col_area<N, V>();
    PA_COL_SETUP(N)
    auto in_band = [&](int m, int t_) {
        return slot_in_band<N, V>(m) && colok && (t_ + T * m <= K || t_ + T * m >= N - K);
    };
    auto row_of = [&](int m, int t_) { return in_band(m, t_) ? (t_ + T * m <= K ? t_ + T * m : t_ + T * m - N + KY) : 0; };
    auto cidx = [&](int m, int t_) { return (unsigned)c + (unsigned)row_of(m, t_) * (unsigned)KXP; };
    auto ky_of = [&](int m, int t_) { return t_ + T * m <= K ? t_ + T * m : t_ + T * m - N; };
    auto load = [&](cd* v, const cd* yin) {
        const cd* __restrict__ src = yin + ymem;
#pragma unroll
        for (int m = 0; m < E; ++m) {
            const cd x = ldc(src, yoff(m, t));
            v[m] = colok ? x : czero();
        }
    };
    // inputs first, unconditional at in-bounds addresses (as in col_twin_kernel)
    cd v0[E], v1[E];
    if constexpr (MODE != COL_FROM_STATE) load(v0, a.yin[0]);
    if constexpr (MT::PAIR_IN) load(v1, a.yin[1]);
    const ColPtrs q = col_ptrs<MODE>(a, cmem, b, kx0, kx);
    cd s0[E], s1[E];
    auto load_compact = [&]() {
        const int tc = opaque(t);
#pragma unroll
        for (int m = 0; m < E; ++m) {
            if (!slot_in_band<N, V>(m)) continue;
            if constexpr (MT::NEED0) s0[m] = ldc(q.p0, cidx(m, tc));
            if constexpr (MT::NEED1) s1[m] = ldc(q.p1, cidx(m, tc));
        }
    };
#pragma unroll
    for (int m = 0; m < E; ++m) s0[m] = s1[m] = czero();
    const cd* twl = col_twiddles<N, V>(smem + CB * col_area<N, V>(), a.tw);
    // a stage's compact operand is in flight during the second input transform; a stage
    // with two issues them once the inputs are combined (held through a transform, or
    // beside both transformed inputs, they spill under the three-wave cap)
    constexpr bool BOTH = MT::NEED0 && MT::NEED1;
    if constexpr (MODE != COL_FROM_STATE) col_fft<N, V, false>(v0, at, lds, twl);
    if constexpr (!BOTH) load_compact();
    if constexpr (MT::PAIR_IN) col_fft<N, V, false>(v1, at, lds, twl);
    cd w[E];   // spectral values handed to the output transforms
    const int tp = opaque(t);
#pragma unroll
    for (int m = 0; m < E; ++m) {
        const bool ins = in_band(m, tp) && !(kx == 0 && row_of(m, tp) == 0);
        w[m] = MODE != COL_FROM_STATE && slot_in_band<N, V>(m)
                   ? col_pair_value<MODE>(a, ins, MT::ADJ && ins ? q.ik2[cidx(m, tp)] : 0.0, kx, ky_of(m, tp), v0[m],
                                          MT::PAIR_IN ? v1[m] : czero())
                   : czero();
    }
    if constexpr (BOTH) {
        asm volatile("" ::: "memory");
        load_compact();
    }
    const int tu = opaque(t);
#pragma unroll
    for (int m = 0; m < E; ++m) {
        if (!slot_in_band<N, V>(m)) continue;
        const bool on = in_band(m, tu);
        const int r = row_of(m, tu);
        const bool ins = on && !(kx == 0 && r == 0);
        w[m] = col_mode_update<N, MODE>(a, q, on, ins, cidx(m, tu), b, kx, r, ky_of(m, tu), a.ey2[r], w[m], s0[m], s1[m]);
    }
    for (int o = 0; o < a.nout; ++o) {
        cd v[E];
        const int to = opaque(t);
#pragma unroll
        for (int m = 0; m < E; ++m) {
            const bool ins = in_band(m, to) && !(kx == 0 && row_of(m, to) == 0);
            v[m] = slot_in_band<N, V>(m)
                       ? col_field<N>(a.fields[0], o == 1, ins, ins && a.fields[0] == F_ZP ? q.ik2[cidx(m, to)] : 0.0, kx,
                                      ky_of(m, to), w[m])
                       : czero();
        }
        col_fft<N, V, true>(v, at, lds, twl);
        if (colok) {
            cd* __restrict__ out = a.yout[o] + ymem;
#pragma unroll
            for (int m = 0; m < E; ++m) stc(out, yoff(m, to), v[m]);
        }
    }
}

// ---------------------------------------- pipelined row passes (gfx950) --
// Variant 3 of the row passes: the plan of variant 2 run by persistent
// wavefronts.  A wavefront owns G = 64 / T consecutive rows of one member
// (contiguous in the Y layout) at a time and loops over such row groups.
// The half spectra of its next group stream from HBM straight into a
// per-wave LDS stage buffer (global->LDS loads: no registers are held while
// they are in flight) while it transforms the current group.  They are read
// into registers, with the Hermitian extension, just before the current
// group's outputs are stored, so the wait for them never waits on fresh
// stores.  Only the twiddle staging synchronises the workgroup.

constexpr int PIPE_V = 2;   // plan variant run by the pipelined kernels

template <int N>
struct Pipe {
    static constexpr int T = Plan<N, PIPE_V>::T, E = Plan<N, PIPE_V>::E;
    static constexpr int G = (T <= 64 && 64 % T == 0) ? 64 / T : 1;   // rows per wavefront
    // (from 512 points the wavefront plans are faster without the stage buffer: eight 512^2 members
    // 19.4 against 25.2 us per adjoint row launch)
    static constexpr bool OK = T <= 64 && 64 % T == 0 && G <= N && N <= 256;
    static constexpr int KXP = kx_pad<N>();
    static constexpr int SPAN = G * KXP;                   // elements of one field of a row group
    static constexpr int LOADS = (SPAN + 63) / 64;         // 64-lane loads per field
    template <int NF>
    static constexpr int wave_lds() { return NF * SPAN + G * lds_team<N>(); }
    static __host__ __device__ size_t offset(int group) {  // first element of a row group
        constexpr int GPM = N / G;
        return ((size_t)(group / GPM) * N + (size_t)(group % GPM) * G) * KXP;
    }
};

__device__ __forceinline__ void vm_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Global->LDS loads of one row group of NF fields into the wave's stage
// buffer (lane l of a load lands at the load's LDS base + l).  The LDS base
// of these loads goes to M0 and must be uniform over the wavefront: the
// full-wave loads are issued first with no condition, and the partial final
// loads of all fields together in one conditional block, so that the compiler
// never merges a masked load with a load of another LDS base (the merged
// instruction would take one lane's base for every lane).
template <int N, int NF>
__device__ __forceinline__ void pipe_fetch(cd* stage, const cd* (&src)[NF], size_t off, int lane) {
    using P = Pipe<N>;
    constexpr int FULL = P::SPAN / 64, TAIL = P::SPAN % 64;
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int i = 0; i < FULL; ++i)
            __builtin_amdgcn_global_load_lds(src[f] + off + i * 64 + lane,
                                             (__attribute__((address_space(3))) void*)(stage + f * P::SPAN + i * 64),
                                             16, 0, 0);
    if constexpr (TAIL > 0) {
        if (lane < TAIL) {
#pragma unroll
            for (int f = 0; f < NF; ++f)
                __builtin_amdgcn_global_load_lds(src[f] + off + FULL * 64 + lane,
                                                 (__attribute__((address_space(3))) void*)(stage + f * P::SPAN + FULL * 64),
                                                 16, 0, 0);
        }
    }
}

// Both products share the loop: ADJ multiplies by the cotangent pair, else the
// velocity is squared.
template <int N, bool ADJ>
__device__ __forceinline__ void row_pipe_body(const RowArgs& a, int n_groups) {
    using P = Pipe<N>;
    constexpr int V = PIPE_V, T = P::T, E = P::E, KXP = P::KXP, NF = ADJ ? 4 : 2, WL_ = true;
    extern __shared__ cd smem[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, team = lane / T, t0 = lane % T;
    const int wpg = blockDim.x >> 6;
    cd* const stage = smem + wave * P::template wave_lds<NF>();
    cd* const lds = stage + NF * P::SPAN + team * lds_team<N>();
    RowTw<N, V> tr;
    row_twiddles<N, V>(tr, t0, a.tw, smem + wpg * P::template wave_lds<NF>());
    const int nw = gridDim.x * wpg;
    int g = blockIdx.x * wpg + wave;
    const cd* src[NF];   // packed (u, v), then packed (b, a)
#pragma unroll
    for (int f = 0; f < NF; ++f) src[f] = a.yin[f];
    const cd* const row = stage + team * KXP;
    cd w[E], z[E];
    // one signal at a time: LDS latency is short, and the raw values of both
    // in flight at once would double the registers held
    auto read_inputs = [&](int t) {
        packed_load<N, V>(z, row, row + P::SPAN, t);
        wave_lds_sync();
        if constexpr (ADJ) {
            packed_load<N, V>(w, row + 2 * P::SPAN, row + 3 * P::SPAN, t);
            wave_lds_sync();
        }
    };
    if (g < n_groups) {
        pipe_fetch<N, NF>(stage, src, P::offset(g), lane);
        vm_wait();
        read_inputs(t0);
        if (g + nw < n_groups) pipe_fetch<N, NF>(stage, src, P::offset(g + nw), lane);
    }
    for (; g < n_groups; g += nw) {
        const int t = opaque(t0);
        cd q[E];
        if constexpr (ADJ) row_fft<N, V, true, WL_>(w, t, lds, tr);
        row_fft<N, V, true, WL_>(z, t, lds, tr);
#pragma unroll
        for (int m = 0; m < E; ++m) q[m] = ADJ ? cmulc(w[m], z[m]) : csq(z[m]);
        row_fft<N, V, false, WL_>(q, t, lds, tr);
        const int gn = g + nw;
        if (gn < n_groups) {
            vm_wait();
            read_inputs(t);
            if (gn + nw < n_groups) pipe_fetch<N, NF>(stage, src, P::offset(gn + nw), lane);
        }
        const size_t ro = P::offset(g) + team * KXP;
        pair_store<N, V>(q, t, a.yout[0] + ro, a.yout[1] + ro);
    }
}

template <int N>
__global__ void __launch_bounds__(256) row_sq_pipe_kernel(Dims d, RowArgs a, int n_groups) {
    row_pipe_body<N, false>(a, n_groups);
}

template <int N>
__global__ void __launch_bounds__(256) row_mul_pipe_kernel(Dims d, RowArgs a, int n_groups) {
    row_pipe_body<N, true>(a, n_groups);
}

// Persistent grid: as many workgroups as can be resident (occupancy query,
// cached per kernel and workgroup size), at most one row group per wave.
template <int N, int NF, class Kern>
hipError_t pipe_launch(Kern kernel, int teams, const Dims& d, const RowArgs& a, hipStream_t s) {
    using P = Pipe<N>;
    const int n_groups = d.B * (N / P::G);
    const int wpg = teams >= 4 ? 4 : teams >= 2 ? 2 : 1;
    const size_t lds = ((size_t)wpg * P::template wave_lds<NF>() + N) * sizeof(cd);
    static std::atomic<int> per_cu_cache[3];
    std::atomic<int>& slot = per_cu_cache[wpg == 1 ? 0 : wpg == 2 ? 1 : 2];
    int per_cu = slot.load(std::memory_order_relaxed);
    if (per_cu <= 0) {
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, wpg * 64, lds);
        if (e != hipSuccess) return e;
        if (per_cu < 1) return hipErrorInvalidConfiguration;
        slot.store(per_cu, std::memory_order_relaxed);
    }
    const long want = (n_groups + wpg - 1) / wpg;
    const long wgs = std::min<long>(want, (long)per_cu * std::max(d.cus, 1));
    launch_kernel(kernel, dim3((unsigned)wgs), dim3((unsigned)(wpg * 64)), lds, s, d, a, n_groups);
    return hipGetLastError();
}

// ------------------------------------------------------------- launchers --

// Teams per workgroup: must divide the teams per member (the kernels take the
// member index from the workgroup's first team), fit 256 threads and the LDS:
// 64 KiB, or the device's limit for plan 3.
template <int N, int V>
size_t row_lds(int tpb) { return ((size_t)tpb * row_area<N, V>() + N) * sizeof(cd); }

template <int N, int V>
int row_tpb(const Dims& d, int tpb, long teams_per_member) {
    const int cap = 256 / Plan<N, V>::T;
    const size_t most = V == 3 ? (size_t)d.lds_max : 65536;
    if (tpb > cap) tpb = cap;
    if (tpb < 1) tpb = 1;
    while (tpb > 1 && row_lds<N, V>(tpb) > most) tpb >>= 1;
    while (tpb > 1 && teams_per_member % tpb) tpb >>= 1;
    return tpb;
}

// A kernel whose workgroups take more than 64 KiB of LDS: its dynamic limit is
// raised to the device's once per instantiation and device.  (The 1024-point
// rows take 80 KiB by default, wide column blocks up to 144.)
template <auto Kernel>
hipError_t raise_lds(const Dims& d, size_t lds) {
    if (lds <= 65536) return hipSuccess;
    static DeviceOnce raised;
    return raised(d.device, [&] {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(Kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, d.lds_max);
        if (e != hipSuccess) (void)hipGetLastError();   // returned here, not by the next launch too
        return e;
    });
}

template <int N, int V, auto Kernel, class... Args>
hipError_t row_launch(const Dims& d, int teams, long per_member, unsigned more, hipStream_t s, Args... args) {
    const int tpb = row_tpb<N, V>(d, teams, per_member);
    const size_t lds = row_lds<N, V>(tpb);
    const hipError_t e = raise_lds<Kernel>(d, lds);
    if (e != hipSuccess) return e;
    launch_kernel(Kernel, dim3((unsigned)(per_member * d.B / tpb) + more), dim3((unsigned)(tpb * Plan<N, V>::T)), lds, s,
                  d, args...);
    return hipGetLastError();
}

// The plans that differ among variants 0, 1 and 2 of a length are the first
// plans<N>() of them.
template <int N>
__host__ __device__ constexpr int plans() { return N <= 32 || N == 512 ? 1 : N == 64 || N == 1024 ? 2 : 3; }
template <int N>
constexpr int plan_of(int variant) { return std::min(variant, plans<N>() - 1); }
template <int N, int A, int B>
constexpr bool same_plan() {
    using P = Plan<N, A>;
    using Q = Plan<N, B>;
    return P::NS == Q::NS && P::T == Q::T && P::E == Q::E && P::R[0] == Q::R[0] && P::R[1] == Q::R[1] &&
           P::R[2] == Q::R[2] && P::R[3] == Q::R[3];
}

// The grids whose time loop runs in one kernel (small.hpp) launch only the
// transforms of fields and the columns between them.
template <int N>
constexpr bool loop_grid() { return N <= 64; }

// VAR / TPB: the plan variant and rows per workgroup of the launching pass
// (forward rows: d.var, d.tpb; adjoint rows: d.avar, d.atpb).  Variant 3
// (pipelined) runs the plan of variant 2 in the kernels it does not cover.
// Rows of 1024 points run on plan 3 whatever the tiles' variant, four per
// workgroup: the Stockham plans of that length exchange two or three times per
// transform, across two wavefronts where a thread holds eight values.  Per
// launch, best Stockham tiles -> plan 3: one member 14.0 -> 11.9 us (forward
// rows) and 17.4 -> 14.6 (adjoint rows), four 30.8 -> 25.8 and 43.2 -> 37.7,
// eight 53.1 -> 43.9 and 74.6 -> 61.2 (4.1 and 4.4 TB/s).
// Where the variants of a length are one plan (8 to 32 and 512 points; 1 and 2 at
// 64), one of them is instantiated.
// (MORE: workgroups ahead of the rows').
#define PA_ROW_LAUNCH(VAR, TPB, KERNEL, TEAMS_PER_MEMBER, MORE, ...)                                          \
    do {                                                                                                      \
        const long tpm_ = (TEAMS_PER_MEMBER);                                                                 \
        const int v_ = plan_of<N>(VAR);                                                                       \
        if constexpr (N == 1024) return row_launch<N, 3, KERNEL(3)>(d, 4, tpm_, (MORE), s, __VA_ARGS__);      \
        else if (v_ == 0) return row_launch<N, 0, KERNEL(0)>(d, (TPB), tpm_, (MORE), s, __VA_ARGS__);         \
        else if constexpr (plans<N>() > 1) {                                                                  \
            if (v_ == 1) return row_launch<N, 1, KERNEL(1)>(d, (TPB), tpm_, (MORE), s, __VA_ARGS__);          \
            else if constexpr (plans<N>() > 2) return row_launch<N, 2, KERNEL(2)>(d, (TPB), tpm_, (MORE), s, __VA_ARGS__); \
        }                                                                                                     \
        return hipErrorInvalidValue;                                                                          \
    } while (0)

#define PA_K_R2C(V) &row_r2c_kernel<N, V>
#define PA_K_C2R(V) &row_c2r_kernel<N, V>
#define PA_K_SQ(V) &row_sq_kernel<N, V>
#define PA_K_MUL(V) &row_mul_kernel<N, V>
#define PA_K_OBS(V) &row_obs_kernel<N, V>
#define PA_K_SRC_WRITE(V) &row_src_kernel<N, V, SRC_WRITE>
#define PA_K_SRC_IMPULSE(V) &row_src_kernel<N, V, SRC_IMPULSE>
#define PA_K_SRC_ADD(V) &row_src_kernel<N, V, SRC_ADD>

template <int N>
hipError_t Launch<N>::row_r2c(const Dims& d, const double* in, cd* out, const cd* tw, const MultSpec* m, hipStream_t s) {
    const unsigned fill = m ? (unsigned)std::min((d.KY * d.KXP + 63) / 64, 512) : 0;   // a value or so per thread
    PA_ROW_LAUNCH(d.var, d.tpb, PA_K_R2C, N / 2, fill, in, out, tw, m ? *m : MultSpec{}, fill);
}
template <int N>
hipError_t Launch<N>::row_c2r(const Dims& d, const cd* in, double* out, const cd* tw, hipStream_t s) {
    PA_ROW_LAUNCH(d.var, d.tpb, PA_K_C2R, N / 2, 0u, in, out, tw);
}
template <int N>
hipError_t Launch<N>::row_sq(const Dims& d, const RowArgs& a, hipStream_t s) {
    if constexpr (loop_grid<N>()) return hipErrorInvalidValue;
    else {
        if constexpr (Pipe<N>::OK)
            if (d.var == 3) return pipe_launch<N, 2>(row_sq_pipe_kernel<N>, d.tpb, d, a, s);
        PA_ROW_LAUNCH(d.var, d.tpb, PA_K_SQ, N, 0u, a);
    }
}
template <int N>
hipError_t Launch<N>::row_obs(const Dims& d, const RowArgs& a, hipStream_t s) {
    if constexpr (loop_grid<N>()) return hipErrorInvalidValue;
    else PA_ROW_LAUNCH(d.var, d.tpb, PA_K_OBS, a.obs.M, 0u, a);
}
template <int N>
hipError_t Launch<N>::row_mul(const Dims& d, const RowArgs& a, hipStream_t s) {
    if constexpr (loop_grid<N>()) return hipErrorInvalidValue;
    else {
        if constexpr (Pipe<N>::OK)
            if (d.avar == 3) return pipe_launch<N, 4>(row_mul_pipe_kernel<N>, d.atpb, d, a, s);
        PA_ROW_LAUNCH(d.avar, d.atpb, PA_K_MUL, N, 0u, a);
    }
}
template <int N>
hipError_t Launch<N>::row_src(const Dims& d, const RowArgs& a, int mode, hipStream_t s) {
    if constexpr (loop_grid<N>()) return hipErrorInvalidValue;
    else {
        if (mode == SRC_ADD) PA_ROW_LAUNCH(d.avar, d.atpb, PA_K_SRC_ADD, a.obs.M, 0u, a);
        if (mode == SRC_IMPULSE) PA_ROW_LAUNCH(d.avar, d.atpb, PA_K_SRC_IMPULSE, N, 0u, a);
        PA_ROW_LAUNCH(d.avar, d.atpb, PA_K_SRC_WRITE, N, 0u, a);
    }
}

template <auto Kernel>
hipError_t col_launch(const Dims& d, const ColArgs& a, unsigned threads, size_t lds, hipStream_t s) {
    const hipError_t e = raise_lds<Kernel>(d, lds);
    if (e != hipSuccess) return e;
    launch_kernel(Kernel, dim3((unsigned)(d.KXP / a.cb) * (unsigned)d.B), dim3(threads), lds, s, d, a);
    return hipGetLastError();
}

template <int N, int V, int MODE>
hipError_t col_mode(const Dims& d, const ColArgs& a, hipStream_t s) {
    constexpr int T = Plan<N, V>::T;
    ColArgs ak = a;
    ak.cb = d.cb_auto ? col_block_auto(d) : d.cb;
    // the columns that fill the lanes which a team leaves free (per twin)
    const int fill = col_trade<N, V>() ? 64 : N >= 64 ? 16 : 1;
    // a single field in and out has no second signal for a twin
    const bool single = MODE == COL_FILTER || (MODE == COL_FROM_STATE && a.nout < 2);
    if (col_twins(d) && !single) {
        while (ak.cb * T < (col_trade<N, V>() ? 32 : fill)) ak.cb *= 2;
        while (ak.cb > 1 && (2 * ak.cb * T > twin_threads<N, V>() || col_lds<N, V>(2 * ak.cb) > (size_t)d.lds_max))
            ak.cb /= 2;
        return col_launch<&col_twin_kernel<N, V, MODE>>(d, ak, (unsigned)(2 * ak.cb * T), col_lds<N, V>(2 * ak.cb), s);
    }
    if (col_trade<N, V>())
        while (ak.cb * T < fill) ak.cb *= 2;
    return col_launch<&col_pass_kernel<N, V, MODE>>(d, ak, (unsigned)(ak.cb * T), col_lds<N, V>(ak.cb), s);
}

template <int N, int V>
hipError_t col_variant(const Dims& d, int mode, const ColArgs& a, hipStream_t s) {
    switch (mode) {
        case COL_INIT: return col_mode<N, V, COL_INIT>(d, a, s);
        case COL_FILTER: return col_mode<N, V, COL_FILTER>(d, a, s);
        case COL_FROM_STATE: return col_mode<N, V, COL_FROM_STATE>(d, a, s);
        case COL_FIRST_GUESS: return col_mode<N, V, COL_FIRST_GUESS>(d, a, s);
    }
    if constexpr (!loop_grid<N>()) {
        switch (mode) {
            case COL_A: return col_mode<N, V, COL_A>(d, a, s);
            case COL_B: return col_mode<N, V, COL_B>(d, a, s);
            case COL_C: return col_mode<N, V, COL_C>(d, a, s);
            case COL_D: return col_mode<N, V, COL_D>(d, a, s);
            case COL_ADJ_C: return col_mode<N, V, COL_ADJ_C>(d, a, s);
            case COL_ADJ_B: return col_mode<N, V, COL_ADJ_B>(d, a, s);
            case COL_ADJ_A: return col_mode<N, V, COL_ADJ_A>(d, a, s);
            case COL_ADJ_N: return col_mode<N, V, COL_ADJ_N>(d, a, s);
            case COL_ADJ_SRC: return col_mode<N, V, COL_ADJ_SRC>(d, a, s);
        }
    }
    return hipErrorInvalidValue;
}

template <int N>
hipError_t Launch<N>::col(const Dims& d, int mode, const ColArgs& a, hipStream_t s) {
    static_assert((plans<N>() > 1 || same_plan<N, 0, 1>()) && (plans<N>() > 2 || same_plan<N, 1, 2>()));
    const int v = plan_of<N>(d.cvar);
    if (v == 0) return col_variant<N, 0>(d, mode, a, s);
    if constexpr (plans<N>() > 1)
        if (v == 1) return col_variant<N, 1>(d, mode, a, s);
    if constexpr (plans<N>() > 2) return col_variant<N, 2>(d, mode, a, s);
    return hipErrorInvalidValue;
}

template <int N>
int Launch<N>::threads(int var) {
    return var == 0 ? Plan<N, 0>::T : var == 1 ? Plan<N, 1>::T : Plan<N, 2>::T;
}

}  // namespace pa
