// kern_small.hip -- grids up to 64^2: the kernels declared in small.hpp.
#include "small.hpp"

#include "kernels_impl.hpp"

namespace pa {

template <int N>
struct Small {
    static constexpr int E = 8, T = N / E, LT = T == 8 ? 3 : T == 4 ? 2 : T == 2 ? 1 : 0;
    static constexpr int TPW = 64 / T;                              // teams per wavefront
    static constexpr int THREADS = N * T < 64 ? 64 : N * T;
    static constexpr int K = (N - 1) / 3, KX = K + 1, KXP = (KX + 7) / 8 * 8, KY = 2 * K + 1;
    static constexpr int MODES = K / T + 1;                         // modes per twin thread
    // A row of a signal in LDS: columns 0..K, then spare ones that take what a team holds beyond
    // the band, so that no access sits in a branch (SPARE is the last).  The pitch puts teams that
    // access rows side by side on different bank groups (8 rows times 2 lanes: 10 mod 16; 16 rows:
    // odd).  One spare row takes the teams beyond N rows.
    static constexpr int SPARE = T * MODES + 1;
    static constexpr int PITCH = T == 8 ? 26 : (SPARE + 1) | 1, ROWS = N * T < 64 ? N + 1 : N, PLANE = ROWS * PITCH;
    static_assert(PITCH > SPARE, "a row's spare columns");
};

// The neighbouring lane's value (lane bit 0).
__device__ __forceinline__ double lane_next(double a) {
    const unsigned long long ua = __builtin_bit_cast(unsigned long long, a);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)ua, 0xb1, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(ua >> 32), 0xb1, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ void twin_trade(double& a, double& b, bool odd) {
    const double got = lane_next(odd ? a : b);
    a = odd ? got : a;
    b = odd ? b : got;
}
__device__ __forceinline__ void twin_trade(cd& a, cd& b, bool odd) {
    twin_trade(a.x, b.x, odd);
    twin_trade(a.y, b.y, odd);
}

// Transform of a team's N = 8 T points; w[k - 1] = exp(-2 pi i k t / N).  Every
// lane of the wavefront must be active.  Natural order in and out: with
// n = t + T m and k = k1 + 8 k2, the radix-8 stage over m gives k1, the trade
// puts k1 mod T on the lanes, and the radix-T stage over t gives k2, so that
// lane k mod T holds entry k in register k / T.
template <int N, bool INV>
__device__ __forceinline__ void small_fft(cd* v, const cd* w) {
    using S = Small<N>;
    dft8<INV>(v);
    if constexpr (S::T > 1) {
#pragma unroll
        for (int k = 1; k < 8; ++k) v[k] = tw_apply<INV>(v[k], w[k - 1]);
        if constexpr (S::LT == 3) {
            digit_trade<0, 3>(v);
            digit_trade<1, 4>(v);
            digit_trade<2, 5>(v);
        } else if constexpr (S::LT == 2) {
            digit_trade<0, 4>(v);
            digit_trade<1, 5>(v);
        } else {
            digit_trade<0, 5>(v);
        }
        cd o[8];
#pragma unroll
        for (int hi = 0; hi < 8 / S::T; ++hi) {
            cd u[S::T];
#pragma unroll
            for (int j = 0; j < S::T; ++j) u[j] = v[hi * S::T + j];
            dft<S::T, INV>(u);
#pragma unroll
            for (int j = 0; j < S::T; ++j) o[hi + 8 / S::T * j] = u[j];
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = o[r];
    }
}

// A thread's places: its team is row `row` in the row phase, signal `odd` of
// column kx in the column phase, lane t of the team in both.  Teams beyond the
// rows or columns run along on the spare row or column.
template <int N>
struct SmallThread {
    using S = Small<N>;
    int t, row, kx;
    bool odd, row_on, col_on;
    cd* yrow;     // this row's P in LDS (Q a plane further)
    cd* ycol;     // this column's signal in LDS
    cd w[7];
    __device__ __forceinline__ SmallThread(const cd* __restrict__ tw, cd* y) {
        const int lane = threadIdx.x & 63, team = (int)(threadIdx.x >> 6) * S::TPW + (lane & (S::TPW - 1));
        t = lane / S::TPW;
        row_on = S::ROWS == N || team < N;
        row = row_on ? team : N;
        odd = team & 1;
        kx = team >> 1;
        col_on = kx <= S::K;
        yrow = y + row * S::PITCH;
        ycol = y + (odd ? S::PLANE : 0) + (col_on ? kx : S::SPARE);
#pragma unroll
        for (int k = 1; k < 8; ++k) w[k - 1] = tw[(k * t) & (N - 1)];
    }
    __device__ __forceinline__ int ky(int p) const { return odd ? t + S::T * (7 - p) - N : t + S::T * p; }
    __device__ __forceinline__ bool on(int p) const { return col_on && ky(p) <= S::K && -ky(p) <= S::K; }
    __device__ __forceinline__ bool ins(int p) const { return on(p) && !(kx == 0 && ky(p) == 0); }
    __device__ __forceinline__ int cidx(int p) const {   // compact index, 0 off the band
        return on(p) ? (ky(p) + (odd ? S::KY : 0)) * S::KXP + kx : 0;
    }
    // this row's complex signal from the packed half spectra in LDS, and back
    __device__ __forceinline__ void row_read(cd* v) const {
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int e = t + S::T * m;
            v[m] = czero();
            if (S::T * m <= S::K) {
                v[m] = yrow[e];
                if (S::T * (m + 1) - 1 > S::K && e > S::K) v[m] = czero();
            } else if (S::T * (m + 1) - 1 >= N - S::K) {
                v[m] = cconj(yrow[S::PLANE + N - e]);
                if (S::T * m < N - S::K && e < N - S::K) v[m] = czero();
            }
        }
    }
    __device__ __forceinline__ void row_write(const cd* v) const {
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int k = t + S::T * m;
            if (S::T * m <= S::K) yrow[k] = v[m];
            if (m == 0) yrow[S::PLANE + (t == 0 ? 0 : S::SPARE)] = cconj(v[m]);
            else if (S::T * (m + 1) - 1 >= N - S::K) yrow[S::PLANE + N - k] = cconj(v[m]);
        }
    }
    // spectra of the row products -> P and Q of this thread's modes (pair p in v[p], v[7 - p])
    __device__ __forceinline__ void col_in(cd* v) const {
#pragma unroll
        for (int m = 0; m < 8; ++m) v[m] = ycol[(t + S::T * m) * S::PITCH];
        small_fft<N, false>(v, w);
#pragma unroll
        for (int p = 0; p < S::MODES; ++p) twin_trade(v[p], v[7 - p], odd);
    }
    // a pair's signals from the spectral values s of the modes: P = (fr + i fi) s, and Q with the
    // real (FLIP_RE) or the imaginary part of the multiplier negated
    template <bool FLIP_RE>
    __device__ __forceinline__ void col_out(const cd* s, const double* fr, const double* fi) const {
        cd v[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) v[m] = czero();
#pragma unroll
        for (int p = 0; p < S::MODES; ++p) {
            const double gr = FLIP_RE ? -fr[p] : fr[p], gi = FLIP_RE ? fi[p] : -fi[p];
            v[p] = mk(s[p].x * fr[p] - s[p].y * fi[p], s[p].x * fi[p] + s[p].y * fr[p]);
            v[7 - p] = mk(s[p].x * gr - s[p].y * gi, s[p].x * gi + s[p].y * gr);
            twin_trade(v[p], v[7 - p], odd);
        }
        small_fft<N, true>(v, w);
#pragma unroll
        for (int m = 0; m < 8; ++m) ycol[(t + S::T * m) * S::PITCH] = v[m];
    }
};

// A member's element of a velocity store: row y, entry x.
template <int N>
__device__ __forceinline__ unsigned small_at(int row, int t, int m) {
    return (unsigned)(row * N + t + Small<N>::T * m);
}

template <int N>
__global__ void __launch_bounds__(Small<N>::THREADS) small_forward_kernel(SmallArgs a) {
    using S = Small<N>;
    extern __shared__ cd smem[];
    const SmallThread<N> th(a.tw, smem);
    const int b = blockIdx.x;
    const size_t SC = (size_t)S::KY * S::KXP, SZ = (size_t)N * N;
    cd* const st = a.state + (size_t)b * SC;
    cd wn[S::MODES], acc[S::MODES], s[S::MODES];
    // multipliers of the modes, 0 off the band and for the mean: the nonlinear term of a pair
    // (col_pair_value) and the velocity u +- i v (col_field)
    double al[S::MODES], be[S::MODES], fr[S::MODES], fi[S::MODES], e2[S::MODES];
    const double ex = th.col_on ? a.ex2[th.kx] : 0.0, inv_n2 = 1.0 / ((double)N * (double)N);
#pragma unroll
    for (int p = 0; p < S::MODES; ++p) {
        const int ci = th.cidx(p);
        const double dkx = (double)th.kx, dky = (double)th.ky(p), ik2 = th.ins(p) ? a.invk2[ci] : 0.0;
        al[p] = th.ins(p) ? 0.25 * (dkx * dkx - dky * dky) : 0.0;
        be[p] = th.ins(p) ? -0.5 * dkx * dky : 0.0;
        fr[p] = dkx * ik2 * inv_n2;
        fi[p] = dky * ik2 * inv_n2;
        e2[p] = ex * a.ey2[ci / S::KXP];
        wn[p] = st[ci];
        if (!th.on(p)) wn[p] = czero();
        acc[p] = czero();
    }
    const double h = a.h, h6 = h / 6.0;
    cd z[8];
    th.template col_out<true>(wn, fr, fi);
    lds_sync();
    th.row_read(z);
    small_fft<N, true>(z, th.w);
    cd* slot = a.store ? a.store + (size_t)b * SZ : nullptr;
    const size_t slot_step = (size_t)a.stride_b * SZ;
    for (int n = 0; n < a.steps; ++n) {
#pragma unroll 1
        for (int stage = 0; stage < 4; ++stage) {
            if (slot) {
                if (th.row_on) {
#pragma unroll
                    for (int m = 0; m < 8; ++m) stc(slot, small_at<N>(th.row, th.t, m), z[m]);
                }
                slot += slot_step;
            }
#pragma unroll
            for (int m = 0; m < 8; ++m) z[m] = csq(z[m]);
            small_fft<N, false>(z, th.w);
            th.row_write(z);
            lds_sync();
            th.col_in(z);
#pragma unroll
            for (int p = 0; p < S::MODES; ++p) {
                const cd P = z[p], Q = z[7 - p];
                cd nl = mk(be[p] * (P.x + Q.x) + al[p] * (P.y - Q.y), be[p] * (P.y + Q.y) - al[p] * (P.x - Q.x));
                if (a.nf > 0 && th.kx == 0 && th.on(p) && (th.ky(p) == a.nf || th.ky(p) == -a.nf)) nl.x += a.forcing;
                const double g2 = e2[p], g1 = g2 * g2;
                if (stage == 0) {
                    acc[p] = cscale(nl, g1);
                    s[p] = cscale(mk(wn[p].x + 0.5 * h * nl.x, wn[p].y + 0.5 * h * nl.y), g2);
                } else if (stage == 3) {
                    wn[p] = mk(g1 * wn[p].x + h6 * (acc[p].x + nl.x), g1 * wn[p].y + h6 * (acc[p].y + nl.y));
                    s[p] = wn[p];
                } else {
                    acc[p] = mk(acc[p].x + 2.0 * g2 * nl.x, acc[p].y + 2.0 * g2 * nl.y);
                    s[p] = stage == 1 ? mk(g2 * wn[p].x + 0.5 * h * nl.x, g2 * wn[p].y + 0.5 * h * nl.y)
                                      : mk(g1 * wn[p].x + h * g2 * nl.x, g1 * wn[p].y + h * g2 * nl.y);
                }
            }
            th.template col_out<true>(s, fr, fi);
            lds_sync();
            th.row_read(z);
            small_fft<N, true>(z, th.w);
        }
    }
    if (th.row_on) {
        cd* const last = a.z_out ? a.z_out + (size_t)b * SZ : nullptr;
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            if (slot) stc(slot, small_at<N>(th.row, th.t, m), z[m]);
            if (last) stc(last, small_at<N>(th.row, th.t, m), z[m]);
        }
    }
#pragma unroll
    for (int p = 0; p < S::MODES; ++p) {
        if (!th.on(p)) continue;
        if (a.steps > 0) st[th.cidx(p)] = wn[p];
        if (a.ckpt) a.ckpt[(size_t)b * SC + th.cidx(p)] = wn[p];
    }
}

template <int N>
__global__ void __launch_bounds__(Small<N>::THREADS) small_adjoint_kernel(SmallArgs a) {
    using S = Small<N>;
    extern __shared__ cd smem[];
    const SmallThread<N> th(a.tw, smem);
    const int b = blockIdx.x;
    const size_t SC = (size_t)S::KY * S::KXP, SZ = (size_t)N * N;
    cd* const st = a.state + (size_t)b * SC;
    cd lam[S::MODES], omb[S::MODES], s[S::MODES];
    // multipliers of the modes, 0 off the band and for the mean: the cotangent of a pair
    // (col_pair_value) and the signals b +- i a (col_field)
    double fx[S::MODES], fy[S::MODES], fr[S::MODES], fi[S::MODES], e2[S::MODES];
    const double ex = th.col_on ? a.ex2[th.kx] : 0.0, inv_n2 = 1.0 / ((double)N * (double)N);
#pragma unroll
    for (int p = 0; p < S::MODES; ++p) {
        const int ci = th.cidx(p);
        const double dkx = (double)th.kx, dky = (double)th.ky(p), f = th.ins(p) ? 0.5 * a.invk2[ci] : 0.0;
        fx[p] = f * dkx;
        fy[p] = f * dky;
        fr[p] = th.ins(p) ? -2.0 * dkx * dky * inv_n2 : 0.0;
        fi[p] = th.ins(p) ? (dkx * dkx - dky * dky) * inv_n2 : 0.0;
        e2[p] = ex * a.ey2[ci / S::KXP];
        lam[p] = a.from_source ? czero() : st[ci];
        if (!th.on(p)) lam[p] = czero();
        omb[p] = czero();
    }
    auto cotangent = [&](int p, cd P, cd Q) {
        return mk(fx[p] * (P.x - Q.x) + fy[p] * (P.y + Q.y), fx[p] * (P.y - Q.y) - fy[p] * (P.x + Q.x));
    };
    const size_t src0 = (size_t)b * SZ;
    cd v[8];
    if (a.from_source) {   // uniform over the grid
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const unsigned i = small_at<N>(th.row, th.t, m);
            v[m] = th.row_on ? mk(a.src_u[src0 + i], a.src_v[src0 + i]) : czero();
        }
        small_fft<N, false>(v, th.w);
        th.row_write(v);
        lds_sync();
        th.col_in(v);
#pragma unroll
        for (int p = 0; p < S::MODES; ++p)
            if (th.on(p)) st[th.cidx(p)] = cotangent(p, v[p], v[7 - p]);
        return;
    }
    const double h = a.h;
    const size_t slot_step = (size_t)a.stride_b * SZ;
    const cd* slot = a.store + (size_t)b * SZ + slot_step * (size_t)(4 * a.steps - 1);
    cd z[8];
    auto fetch = [&]() {   // the next stage's velocity, in flight during the column phase
#pragma unroll
        for (int m = 0; m < 8; ++m) z[m] = th.row_on ? ldc(slot, small_at<N>(th.row, th.t, m)) : czero();
        slot -= slot_step;
    };
    fetch();
#pragma unroll
    for (int p = 0; p < S::MODES; ++p) s[p] = cscale(lam[p], h / 6.0);
    for (int n = a.steps - 1; n >= 0; --n) {
#pragma unroll 1
        for (int stage = 3; stage >= 0; --stage) {
            th.template col_out<false>(s, fr, fi);
            lds_sync();
            th.row_read(v);
            small_fft<N, true>(v, th.w);
#pragma unroll
            for (int m = 0; m < 8; ++m) v[m] = cmulc(v[m], z[m]);
            if (a.src_u && stage == 0 && n == 0 && th.row_on) {
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    const unsigned i = small_at<N>(th.row, th.t, m);
                    v[m] = cadd(v[m], mk(a.src_u[src0 + i], a.src_v[src0 + i]));
                }
            }
            if (stage > 0 || n > 0) fetch();
            small_fft<N, false>(v, th.w);
            th.row_write(v);
            lds_sync();
            th.col_in(v);
#pragma unroll
            for (int p = 0; p < S::MODES; ++p) {
                const cd wb = cotangent(p, v[p], v[7 - p]), lm = lam[p], ob = omb[p];
                const double g2 = e2[p], g1 = g2 * g2;
                if (stage == 3) {
                    omb[p] = mk(g1 * (lm.x + wb.x), g1 * (lm.y + wb.y));
                    s[p] = mk((h / 3.0) * g2 * lm.x + h * g2 * wb.x, (h / 3.0) * g2 * lm.y + h * g2 * wb.y);
                } else if (stage == 0) {
                    lam[p] = mk(ob.x + wb.x, ob.y + wb.y);
                    s[p] = cscale(lam[p], h / 6.0);
                } else {
                    omb[p] = mk(ob.x + g2 * wb.x, ob.y + g2 * wb.y);
                    s[p] = stage == 2
                               ? mk((h / 3.0) * g2 * lm.x + 0.5 * h * wb.x, (h / 3.0) * g2 * lm.y + 0.5 * h * wb.y)
                               : mk((h / 6.0) * g1 * lm.x + 0.5 * h * g2 * wb.x, (h / 6.0) * g1 * lm.y + 0.5 * h * g2 * wb.y);
                }
            }
        }
    }
#pragma unroll
    for (int p = 0; p < S::MODES; ++p)
        if (th.on(p)) st[th.cidx(p)] = lam[p];
}

// A field, real signal of the packed pair (P = Q = its half spectrum), there and
// back in one launch.  A call is bound by what the host spends on it: 18.6 us
// for a 64^2 field in three launches (the first one filling the table), 11.9 here.
template <int N>
__global__ void __launch_bounds__(Small<N>::THREADS) small_filter_kernel(SmallFilter a) {
    using S = Small<N>;
    extern __shared__ cd smem[];
    const SmallThread<N> th(a.tw, smem);
    const size_t f0 = (size_t)blockIdx.x * N * N;
    cd v[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) v[m] = mk(th.row_on ? a.in[f0 + small_at<N>(th.row, th.t, m)] : 0.0, 0.0);
    double f[S::MODES], none[S::MODES];
    const double inv_n2 = 1.0 / ((double)N * (double)N);
    const double* table = a.spec.table ? a.spec.table + (a.table_per_member ? (size_t)blockIdx.x * S::KY * S::KXP : 0) : nullptr;
#pragma unroll
    for (int p = 0; p < S::MODES; ++p) {
        f[p] = table ? table[th.cidx(p)] : mult_value(a.spec, th.kx, th.ky(p));
        f[p] = th.ins(p) ? f[p] * inv_n2 : 0.0;
        none[p] = 0.0;
    }
    small_fft<N, false>(v, th.w);
    th.row_write(v);
    lds_sync();
    th.col_in(v);
    cd s[S::MODES];
#pragma unroll
    for (int p = 0; p < S::MODES; ++p) s[p] = th.on(p) ? v[p] : czero();
    th.template col_out<false>(s, f, none);
    lds_sync();
    th.row_read(v);
    small_fft<N, true>(v, th.w);
    if (th.row_on) {
#pragma unroll
        for (int m = 0; m < 8; ++m) a.out[f0 + small_at<N>(th.row, th.t, m)] = v[m].x;
    }
}

// Probes of one observed step: a wavefront per probe row and member, in the
// order of the rows' probes.
__global__ void __launch_bounds__(64) small_observe_kernel(int N, const cd* __restrict__ z, RowObs o) {
    const int j = blockIdx.x % o.M, b = blockIdx.x / o.M, y = j * o.stride;
    const cd* row = z + ((size_t)b * N + y) * N;
    double part = 0.0;
    for (int i = threadIdx.x; i < o.M; i += 64) {
        const cd q = row[i * o.stride];
        const size_t k = probe_index(o, b, y, i * o.stride), mm = (size_t)o.M * o.M;
        if (o.obs_out) {
            o.obs_out[k] = q.x;
            o.obs_out[k + mm] = q.y;
        }
        if (o.values) {
            const double ru = q.x - o.values[k], rv = q.y - o.values[k + mm];
            part += ru * ru;
            part += rv * rv;
        }
    }
    for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off, 64);
    if (threadIdx.x == 0) store_jpart(o, b, y, part);
}

__global__ void __launch_bounds__(256) small_source_kernel(int N, int n, const cd* __restrict__ z, RowObs o,
                                                           double* __restrict__ src_u, double* __restrict__ src_v) {
    const int i = blockIdx.x * 256 + threadIdx.x;   // element of [nb][N][N]
    if (i >= n) return;
    const int x = i % N, y = i / N % N, b = i / (N * N);
    double u = 0.0, v = 0.0;
    if (o.slot < 0) {
        if (x == o.imp_x && y == o.imp_y) u = 1.0;
    } else if (y % o.stride == 0 && x % o.stride == 0) {
        const size_t base = (((size_t)b * o.n_times + o.slot) * 2) * o.M * o.M + (size_t)(y / o.stride) * o.M + x / o.stride;
        const cd q = z[i];
        u = q.x - o.values[base];
        v = q.y - o.values[base + (size_t)o.M * o.M];
    }
    src_u[i] = u;
    src_v[i] = v;
}

bool small_grid(int N) { return N <= 64; }

template <int N>
static hipError_t forward_n(const SmallArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(small_forward_kernel<N>, dim3((unsigned)a.B), dim3(Small<N>::THREADS),
                       2 * Small<N>::PLANE * sizeof(cd), s, a);
    return hipGetLastError();
}
template <int N>
static hipError_t adjoint_n(const SmallArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(small_adjoint_kernel<N>, dim3((unsigned)a.B), dim3(Small<N>::THREADS),
                       2 * Small<N>::PLANE * sizeof(cd), s, a);
    return hipGetLastError();
}

template <int N>
static hipError_t filter_n(const SmallFilter& a, hipStream_t s) {
    hipLaunchKernelGGL(small_filter_kernel<N>, dim3((unsigned)a.B), dim3(Small<N>::THREADS),
                       2 * Small<N>::PLANE * sizeof(cd), s, a);
    return hipGetLastError();
}

#define PA_SMALL_N(CALL)                       \
    switch (d.N) {                             \
        case 8: return CALL<8>(a, s);          \
        case 16: return CALL<16>(a, s);        \
        case 32: return CALL<32>(a, s);        \
        case 64: return CALL<64>(a, s);        \
        default: return hipErrorInvalidValue;  \
    }

hipError_t launch_small_forward(const Dims& d, const SmallArgs& a, hipStream_t s) {
    if (!a.tw || !a.invk2 || !a.ex2 || !a.ey2 || !a.state || a.B < 1 || a.stride_b < a.B || a.steps < 0)
        return hipErrorInvalidValue;
    PA_SMALL_N(forward_n);
}
hipError_t launch_small_adjoint(const Dims& d, const SmallArgs& a, hipStream_t s) {
    if (!a.tw || !a.invk2 || !a.ex2 || !a.ey2 || !a.state || a.B < 1 || a.stride_b < a.B || (!a.src_u != !a.src_v) ||
        (a.from_source ? !a.src_u : (!a.store || a.steps < 1)))
        return hipErrorInvalidValue;
    PA_SMALL_N(adjoint_n);
}
hipError_t launch_small_filter(const Dims& d, const SmallFilter& a, hipStream_t s) {
    if (!a.tw || !a.in || !a.out || a.B < 1 || (a.table_per_member && !a.spec.table)) return hipErrorInvalidValue;
    PA_SMALL_N(filter_n);
}
hipError_t launch_small_observe(int N, int nb, const cd* z, const RowObs& o, hipStream_t s) {
    if (!z || nb < 1 || o.slot < 0 || o.stride < 1 || o.M < 1 || o.n_times <= o.slot) return hipErrorInvalidValue;
    hipLaunchKernelGGL(small_observe_kernel, dim3((unsigned)(nb * o.M)), dim3(64), 0, s, N, z, o);
    return hipGetLastError();
}
hipError_t launch_small_source(int N, int nb, const cd* z, const RowObs& o, double* src_u, double* src_v, hipStream_t s) {
    if (!src_u || !src_v || nb < 1 || (o.slot >= 0 && (!z || !o.values || o.stride < 1 || o.n_times <= o.slot)))
        return hipErrorInvalidValue;
    const long n = (long)nb * N * N;
    if (n > 0x7fffff00L) return hipErrorInvalidValue;
    hipLaunchKernelGGL(small_source_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, N, (int)n, z, o, src_u,
                       src_v);
    return hipGetLastError();
}

}  // namespace pa
