// Batched vector kernels on internal-layout vectors: the Gram-Schmidt dot
// products and updates of the GMRES/Arnoldi cycles, norms, quadratic forms
// eta^H Theta y of the trace estimators, precision conversions.
//
// Reductions are per right-hand side and always accumulate in FP64.  A
// workgroup is a 2-D tile: x = RT consecutive right-hand sides (the innermost
// index of the layout, so a wavefront reads one contiguous run), y = CT site
// lanes.  Each workgroup reduces its sites in LDS and writes one partial per
// (vector, workgroup, rhs); a second kernel adds the partials in a fixed order,
// so results are bitwise reproducible (no atomics).
#include <type_traits>

#include "common.h"

namespace {

constexpr int JB = 4;   // basis vectors per thread in the multi-dot

struct Tiling {
    int RT, CT;         // block = RT x CT threads
    int ntile;          // rhs tiles
    int NB;             // site blocks
};

Tiling tiling(const mpmc_ctx *ctx, int N, int groups) {
    Tiling t;
    t.RT = N >= 64 ? 64 : (N >= 32 ? 32 : (N >= 16 ? 16 : (N >= 8 ? 8 : (N >= 4 ? 4 : (N >= 2 ? 2 : 1)))));
    t.CT = 256 / t.RT;
    t.ntile = (N + t.RT - 1) / t.RT;
    const long target = (long)ctx->num_cu * 2048;   // threads in flight
    long nb = target / (256L * t.ntile * (groups > 0 ? groups : 1));
    const long maxnb = (ctx->V + t.CT - 1) / t.CT;
    if (nb < 1) nb = 1;
    if (nb > maxnb) nb = maxnb;
    if (nb > 2048) nb = 2048;
    t.NB = (int)nb;
    return t;
}

template <int P>
__device__ __forceinline__ cpx<double> ldd(const VecRef &v, long e, long si) {
    auto x = Store<P>::ld(v.d, v.sc, e, si);
    return mk((double)x.re, (double)x.im);
}

// partial[j][blk][r] = sum over this block's sites of conj(V_j) Theta w.
// Basis vector j starts vstride_b bytes after vector j-1 and is stored in
// precision PB (FP16S: its scales vscale_off bytes after its data); w in PW.
template <int PB, int PW>
__global__ __launch_bounds__(256) void k_multidot(VecRef Vb, size_t vstride_b, size_t vscale_off, int vN, int nv,
                                                  VecRef w, int N, long V, int theta, double2 *__restrict__ partial,
                                                  int NB) {
    __shared__ double2 red[JB][256];
    const int RT = blockDim.x, CT = blockDim.y;
    const int r = blockIdx.y * RT + threadIdx.x;
    const int j0 = blockIdx.z * JB;
    cpx<double> acc[JB];
#pragma unroll
    for (int q = 0; q < JB; ++q) acc[q] = mk(0.0, 0.0);
    if (r < N) {
        for (long s = (long)blockIdx.x * CT + threadIdx.y; s < V; s += (long)NB * CT) {
            cpx<double> wv[12];
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                wv[k] = ldd<PW>(w, (s * 12 + k) * N + r, s * N + r);
                if (theta && k >= 6) wv[k] = mk(-wv[k].re, -wv[k].im);
            }
#pragma unroll
            for (int q = 0; q < JB; ++q) {
                const int j = j0 + q;
                if (j < nv) {
                    VecRef vj;
                    vj.d = (char *)Vb.d + (size_t)j * vstride_b;
                    vj.sc = PB == MPMC_FP16S ? (float *)((char *)vj.d + vscale_off) : nullptr;
                    const int vr = vN == 1 ? 0 : r;
#pragma unroll
                    for (int k = 0; k < 12; ++k)
                        acc[q] = acc[q] + conjmul(ldd<PB>(vj, (s * 12 + k) * vN + vr, s * vN + vr), wv[k]);
                }
            }
        }
    }
    const int tid = threadIdx.y * RT + threadIdx.x;
#pragma unroll
    for (int q = 0; q < JB; ++q) red[q][tid] = make_double2(acc[q].re, acc[q].im);
    __syncthreads();
    for (int h = CT / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.y < h) {
#pragma unroll
            for (int q = 0; q < JB; ++q) {
                double2 a = red[q][tid], b = red[q][tid + h * RT];
                red[q][tid] = make_double2(a.x + b.x, a.y + b.y);
            }
        }
        __syncthreads();
    }
    if (threadIdx.y == 0 && r < N) {
#pragma unroll
        for (int q = 0; q < JB; ++q) {
            const int j = j0 + q;
            if (j < nv) partial[((long)j * NB + blockIdx.x) * N + r] = red[q][threadIdx.x];
        }
    }
}

// sum_b partial[j][b][r] by a 256-thread workgroup in a fixed order (thread t
// adds b = t, t + 256, ..., then a halving tree); the result is in red[0]
// for every thread after the return.
__device__ __forceinline__ void block_sum_partials(const double2 *__restrict__ partial, int NB, int N, int j, int r,
                                                   double2 *red) {
    double2 a = make_double2(0, 0);
    for (int b = threadIdx.x; b < NB; b += 256) {
        double2 v = partial[((long)j * NB + b) * N + r];
        a.x += v.x;
        a.y += v.y;
    }
    red[threadIdx.x] = a;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            red[threadIdx.x].x += red[threadIdx.x + h].x;
            red[threadIdx.x].y += red[threadIdx.x + h].y;
        }
        __syncthreads();
    }
}

// out[j*N + r] (+)= sum_b partial[j][b][r]; one workgroup per (j, r).
__global__ __launch_bounds__(256) void k_reduce(const double2 *__restrict__ partial, int NB, int N,
                                                double2 *__restrict__ out, int accumulate, int only_real) {
    __shared__ double2 red[256];
    const int jr = blockIdx.x;
    const int j = jr / N, r = jr % N;
    block_sum_partials(partial, NB, N, j, r, red);
    if (threadIdx.x == 0) {
        double2 v = red[0];
        if (only_real) v.y = 0;
        if (accumulate) {
            out[jr].x += v.x;
            out[jr].y += v.y;
        } else {
            out[jr] = v;
        }
    }
}

// w += sign * sum_j h[j*N + r] V_j ; optional partial[blk][r] = sum |w|^2
// OUT kOutHalf (FP16S basis, FP32 w): the result is not written back to w but
// to the FP16S vector hout (half values and per-(site, rhs) scales), for a
// caller that needs it only in that form; partial still receives the norms of
// the FP32 result.
// OUT kOutAdd: sum_j alone (w is not read) is added to the FP64 batch hout: a
// solve's correction without storing, widening and adding it in passes of its
// own (24^4 x 64 FP16S, eleven vectors: 6.7 ms in four passes, 4.0 ms in one).
constexpr int kOutInPlace = 0, kOutHalf = 1, kOutAdd = 2;
__device__ __forceinline__ void add_fp64(void *x, long e, double re, double im) {
    double2 *p = reinterpret_cast<double2 *>(x) + e;
    const double2 v = *p;
    *p = make_double2(re + v.x, im + v.y);
}
template <int PB, int PW, int OUT = kOutInPlace>
__global__ __launch_bounds__(256) void k_multiaxpy(VecRef Vb, size_t vstride_b, size_t vscale_off, int vN, int nv,
                                                   VecRef w, int N, long V, const double2 *__restrict__ h, double sign,
                                                   double2 *__restrict__ partial, int NB, int ldh,
                                                   VecRef hout = VecRef{nullptr, nullptr}) {
    using T = typename Store<PW>::real;
    __shared__ double red[256];
    const int RT = blockDim.x, CT = blockDim.y;
    const int r = blockIdx.y * RT + threadIdx.x;
    double nrm = 0;
    if (r < N) {
        for (long s = (long)blockIdx.x * CT + threadIdx.y; s < V; s += (long)NB * CT) {
            cpx<T> acc[12];
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                if constexpr (OUT == kOutAdd) {
                    acc[k] = mk(T(0), T(0));
                } else {
                    auto v = Store<PW>::ld(w.d, w.sc, (s * 12 + k) * N + r, 0);
                    acc[k] = mk((T)v.re, (T)v.im);
                }
            }
            for (int j = 0; j < nv; ++j) {
                const double2 hj = h[(long)j * ldh + r];
                const cpx<T> c = mk((T)(sign * hj.x), (T)(sign * hj.y));
                const void *vj = (const char *)Vb.d + (size_t)j * vstride_b;
                const float *vsc = PB == MPMC_FP16S ? (const float *)((const char *)vj + vscale_off) : nullptr;
                const int vr = vN == 1 ? 0 : r;
                // all twelve loads first: interleaved with the FMAs the
                // scheduler reuses one register pair and waits for each load
                cpx<T> vv[12];
#pragma unroll
                for (int k = 0; k < 12; ++k) {
                    auto v = Store<PB>::ld(vj, vsc, (s * 12 + k) * vN + vr, s * vN + vr);
                    vv[k] = mk((T)v.re, (T)v.im);
                }
#pragma unroll
                for (int k = 0; k < 12; ++k) acc[k] = acc[k] + c * vv[k];
            }
            if constexpr (OUT == kOutAdd) {
#pragma unroll
                for (int k = 0; k < 12; ++k)
                    add_fp64(hout.d, (s * 12 + k) * N + r, (double)acc[k].re, (double)acc[k].im);
            } else if constexpr (OUT == kOutHalf) {
                float mx = 0.f;
#pragma unroll
                for (int k = 0; k < 12; ++k) {
                    mx = fmaxf(mx, fmaxf(fabsf(acc[k].re), fabsf(acc[k].im)));
                    nrm += (double)acc[k].re * acc[k].re + (double)acc[k].im * acc[k].im;
                }
                const float inv = mx > 0.f ? 1.0f / mx : 0.f;
                __half2 *d = reinterpret_cast<__half2 *>(hout.d);
#pragma unroll
                for (int k = 0; k < 12; ++k)
                    d[(s * 12 + k) * N + r] = __floats2half2_rn(acc[k].re * inv, acc[k].im * inv);
                hout.sc[s * N + r] = mx;
            } else {
#pragma unroll
                for (int k = 0; k < 12; ++k) {
                    Store<PW>::st(w.d, (s * 12 + k) * N + r, acc[k]);
                    nrm += (double)acc[k].re * acc[k].re + (double)acc[k].im * acc[k].im;
                }
            }
        }
    }
    if (!partial) return;
    const int tid = threadIdx.y * RT + threadIdx.x;
    red[tid] = nrm;
    __syncthreads();
    for (int hh = CT / 2; hh > 0; hh >>= 1) {
        if ((int)threadIdx.y < hh) red[tid] += red[tid + hh * RT];
        __syncthreads();
    }
    if (threadIdx.y == 0 && r < N) partial[(long)blockIdx.x * N + r] = make_double2(red[threadIdx.x], 0.0);
}

// The middle of a CGS2 step in one pass over the basis: w += sign * sum_j
// h[j*ldh + r] V_j, then partial[j][blk][r] = sum over the block's sites of
// conj(V_j) w (the second pass's dot products, summed by k_reduce).  Component
// by component, the nv <= NVMAX basis values stay in registers between the
// update and the dot, so the basis is read once instead of twice.
template <int P, int NVMAX>
__global__ __launch_bounds__(256) void k_multiaxpy_dot(VecRef Vb, size_t vstride_b, int nv, VecRef w, int N, long V,
                                                       const double2 *__restrict__ h, double sign, int ldh,
                                                       double2 *__restrict__ partial, int NB) {
    using T = typename Store<P>::real;
    __shared__ double2 red[NVMAX][256];
    const int RT = blockDim.x, CT = blockDim.y;
    const int r = blockIdx.y * RT + threadIdx.x;
    cpx<double> d[NVMAX];
#pragma unroll
    for (int j = 0; j < NVMAX; ++j) d[j] = mk(0.0, 0.0);
    if (r < N) {
        cpx<T> c[NVMAX];
#pragma unroll
        for (int j = 0; j < NVMAX; ++j) {
            const double2 hj = j < nv ? h[(long)j * ldh + r] : make_double2(0.0, 0.0);
            c[j] = mk((T)(sign * hj.x), (T)(sign * hj.y));
        }
        for (long s = (long)blockIdx.x * CT + threadIdx.y; s < V; s += (long)NB * CT) {
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                const long e = (s * 12 + k) * N + r;
                const auto wv = Store<P>::ld(w.d, nullptr, e, 0);
                cpx<T> acc = mk((T)wv.re, (T)wv.im);
                cpx<T> vv[NVMAX];
#pragma unroll
                for (int j = 0; j < NVMAX; ++j) {
                    if (j < nv) {
                        const auto v = Store<P>::ld((const char *)Vb.d + (size_t)j * vstride_b, nullptr, e, 0);
                        vv[j] = mk((T)v.re, (T)v.im);
                    } else {
                        vv[j] = mk(T(0), T(0));
                    }
                }
#pragma unroll
                for (int j = 0; j < NVMAX; ++j)
                    if (j < nv) acc = acc + c[j] * vv[j];
                Store<P>::st(w.d, e, acc);
                const cpx<double> wd = mk((double)acc.re, (double)acc.im);
#pragma unroll
                for (int j = 0; j < NVMAX; ++j)
                    if (j < nv) d[j] = d[j] + conjmul(mk((double)vv[j].re, (double)vv[j].im), wd);
            }
        }
    }
    // the block's sums over its site rows (threadIdx.y), in a fixed order;
    // thread row y writes the partials of vectors j = y, y + CT, ...
    const int tid = threadIdx.y * RT + threadIdx.x;
#pragma unroll
    for (int j = 0; j < NVMAX; ++j) red[j][tid] = make_double2(d[j].re, d[j].im);
    __syncthreads();
    if (r < N) {
        for (int j = threadIdx.y; j < nv; j += CT) {
            double2 a = red[j][threadIdx.x];
            for (int y = 1; y < CT; ++y) {
                a.x += red[j][y * RT + threadIdx.x].x;
                a.y += red[j][y * RT + threadIdx.x].y;
            }
            partial[((long)j * NB + blockIdx.x) * N + r] = a;
        }
    }
}

// y = a * x + b * y   (uniform complex coefficients)
template <int P>
__global__ void k_axpby(VecRef x, VecRef y, long total, double2 a, double2 b) {
    using T = typename Store<P>::real;
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    auto xv = Store<P>::ld(x.d, nullptr, e, 0);
    cpx<T> r = mk((T)a.x, (T)a.y) * mk((T)xv.re, (T)xv.im);
    if (b.x != 0.0 || b.y != 0.0) {   // y is not read when b == 0 (it may be uninitialised)
        auto yv = Store<P>::ld(y.d, nullptr, e, 0);
        r = r + mk((T)b.x, (T)b.y) * mk((T)yv.re, (T)yv.im);
    }
    Store<P>::st(y.d, e, r);
}

// y[e] = coef[r] * x[e] (coef per rhs, FP64) ; invert_sqrt: coef = 1/sqrt(re(c)) (0 if c == 0)
template <int P>
__global__ void k_scale_rhs(VecRef x, VecRef y, long total, int N, const double2 *__restrict__ coef, int mode) {
    using T = typename Store<P>::real;
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const int r = (int)(e % N);
    double2 c = coef[r];
    if (mode == 1) {
        const double q = c.x;
        c = make_double2(q > 0 ? 1.0 / sqrt(q) : 0.0, 0.0);
    } else if (mode == 2) {   // divide by c
        const double d = c.x * c.x + c.y * c.y;
        c = d > 0 ? make_double2(c.x / d, -c.y / d) : make_double2(0.0, 0.0);
    }
    auto xv = Store<P>::ld(x.d, nullptr, e, 0);
    Store<P>::st(y.d, e, mk((T)c.x, (T)c.y) * mk((T)xv.re, (T)xv.im));
}

// precision conversion between two non-FP16S layouts, or from FP16S
template <int PX, int PY>
__global__ void k_convert(VecRef x, VecRef y, long V, int N) {
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= V * N) return;
    const long s = t / N;
    const int r = (int)(t - s * N);
    using TY = typename Store<PY>::real;
    if constexpr (PY == MPMC_FP16S) {
        cpx<float> v[12];
        float mx = 0.f;
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            auto a = Store<PX>::ld(x.d, x.sc, (s * 12 + k) * N + r, s * N + r);
            v[k] = mk((float)a.re, (float)a.im);
            mx = fmaxf(mx, fmaxf(fabsf(v[k].re), fabsf(v[k].im)));
        }
        const float inv = mx > 0.f ? 1.0f / mx : 0.f;
        __half2 *d = reinterpret_cast<__half2 *>(y.d);
#pragma unroll
        for (int k = 0; k < 12; ++k) d[(s * 12 + k) * N + r] = __floats2half2_rn(v[k].re * inv, v[k].im * inv);
        y.sc[s * N + r] = mx;
    } else {
        cpx<TY> v[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            auto a = Store<PX>::ld(x.d, x.sc, (s * 12 + k) * N + r, s * N + r);
            v[k] = mk((TY)a.re, (TY)a.im);
        }
#pragma unroll
        for (int k = 0; k < 12; ++k) Store<PY>::st(y.d, (s * 12 + k) * N + r, v[k]);
    }
}

// y (FP16S) = coef[r] * x (FP32): k_scale_rhs followed by k_convert in one
// pass, with the same arithmetic (the product in FP32, then the per-(site,
// rhs) scale and the half-precision values).
__global__ void k_convert_scaled_h(VecRef x, VecRef y, long V, int N, const double2 *__restrict__ coef) {
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= V * N) return;
    const long s = t / N;
    const int r = (int)(t - s * N);
    const double2 c = coef[r];
    cpx<float> v[12];
    float mx = 0.f;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const auto a = Store<MPMC_FP32>::ld(x.d, nullptr, (s * 12 + k) * N + r, 0);
        v[k] = mk((float)c.x, (float)c.y) * mk(a.re, a.im);
        mx = fmaxf(mx, fmaxf(fabsf(v[k].re), fabsf(v[k].im)));
    }
    const float inv = mx > 0.f ? 1.0f / mx : 0.f;
    __half2 *d = reinterpret_cast<__half2 *>(y.d);
#pragma unroll
    for (int k = 0; k < 12; ++k) d[(s * 12 + k) * N + r] = __floats2half2_rn(v[k].re * inv, v[k].im * inv);
    y.sc[s * N + r] = mx;
}

// y = x / sqrt(re nrm[r]) of an FP64 x in the storage precision of a Krylov
// basis: the narrowing (k_convert), the scaling in the working precision
// (k_scale_rhs, mode 1) and, for FP16S, the packing (k_convert again) in one
// pass with the same arithmetic (24^4 x 64 FP16S: 2.75 ms in three, 0.95 ms in one).
template <int P>
__global__ void k_convert_normalised(VecRef x, VecRef y, long V, int N, const double2 *__restrict__ nrm) {
    using T = typename Store<P>::real;
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= V * N) return;
    const long s = t / N;
    const int r = (int)(t - s * N);
    const double q = nrm[r].x;
    const cpx<T> c = mk((T)(q > 0 ? 1.0 / sqrt(q) : 0.0), T(0));
    cpx<T> v[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const auto a = Store<MPMC_FP64>::ld(x.d, nullptr, (s * 12 + k) * N + r, 0);
        v[k] = c * mk((T)a.re, (T)a.im);
    }
    if constexpr (P == MPMC_FP16S) {
        float mx = 0.f;
#pragma unroll
        for (int k = 0; k < 12; ++k) mx = fmaxf(mx, fmaxf(fabsf(v[k].re), fabsf(v[k].im)));
        const float inv = mx > 0.f ? 1.0f / mx : 0.f;
        __half2 *d = reinterpret_cast<__half2 *>(y.d);
#pragma unroll
        for (int k = 0; k < 12; ++k) d[(s * 12 + k) * N + r] = __floats2half2_rn(v[k].re * inv, v[k].im * inv);
        y.sc[s * N + r] = mx;
    } else {
#pragma unroll
        for (int k = 0; k < 12; ++k) Store<P>::st(y.d, (s * 12 + k) * N + r, v[k]);
    }
}

template <typename F>
int dispatch_prec(mpmc_ctx *ctx, int prec, F &&f) {
    switch (prec) {
        case MPMC_FP64: f(std::integral_constant<int, MPMC_FP64>()); break;
        case MPMC_FP32: f(std::integral_constant<int, MPMC_FP32>()); break;
        default: return set_err(ctx, MPMC_EINVAL, "precision %d not supported by this kernel", prec);
    }
    HIP_OR_RET(ctx, hipGetLastError());
    return MPMC_OK;
}

// acc[r] += sign * c * t[r]
__global__ void k_scale_acc(const double2 *t, int N, double2 c, double sign, double2 *acc) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= N) return;
    const double2 v = t[r];
    acc[r].x += sign * (c.x * v.x - c.y * v.y);
    acc[r].y += sign * (c.x * v.y + c.y * v.x);
}

// ---- single vectors (nrhs == 1): one thread per complex element ----
// partial[j][blk] = sum over this block's elements of conj(V_j) Theta w
template <int P>
__global__ __launch_bounds__(256) void k_multidot1(VecRef Vb, long vstride, int nv, VecRef w, long n, int theta,
                                                   double2 *__restrict__ partial, int NB) {
    using T = typename Store<P>::real;
    __shared__ double2 red[JB][256];
    const int j0 = blockIdx.y * JB;
    cpx<double> acc[JB];
#pragma unroll
    for (int q = 0; q < JB; ++q) acc[q] = mk(0.0, 0.0);
    for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long)NB * 256) {
        cpx<double> wv = ldd<P>(w, e, 0);
        if (theta && (e % 12) >= 6) wv = mk(-wv.re, -wv.im);
        // loads of the JB vectors issued together (index clamped to the last
        // vector, its contribution masked) instead of one guarded load each
        cpx<double> vq[JB];
#pragma unroll
        for (int q = 0; q < JB; ++q) {
            const int j = j0 + q < nv ? j0 + q : nv - 1;
            VecRef vj;
            vj.d = (char *)Vb.d + (size_t)j * vstride * sizeof(T) * 2;
            vj.sc = nullptr;
            vq[q] = ldd<P>(vj, e, 0);
        }
#pragma unroll
        for (int q = 0; q < JB; ++q)
            if (j0 + q < nv) acc[q] = acc[q] + conjmul(vq[q], wv);
    }
#pragma unroll
    for (int q = 0; q < JB; ++q) red[q][threadIdx.x] = make_double2(acc[q].re, acc[q].im);
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
#pragma unroll
            for (int q = 0; q < JB; ++q) {
                red[q][threadIdx.x].x += red[q][threadIdx.x + h].x;
                red[q][threadIdx.x].y += red[q][threadIdx.x + h].y;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < JB; ++q)
            if (j0 + q < nv) partial[(long)(j0 + q) * NB + blockIdx.x] = red[q][0];
    }
}

// w += sign * sum_j h[j*ldh] V_j ; optional partial[blk] = sum |w|^2
template <int P>
__global__ __launch_bounds__(256) void k_multiaxpy1(VecRef Vb, long vstride, int nv, VecRef w, long n,
                                                    const double2 *__restrict__ h, int ldh, double sign,
                                                    double2 *__restrict__ partial, int NB) {
    using T = typename Store<P>::real;
    __shared__ double red[256];
    double nrm = 0;
    for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long)NB * 256) {
        auto v0 = Store<P>::ld(w.d, nullptr, e, 0);
        cpx<T> acc = mk((T)v0.re, (T)v0.im);
        // four basis vectors per iteration, their loads issued together
        int j = 0;
        for (; j + 4 <= nv; j += 4) {
            cpx<T> vq[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const void *vj = (const char *)Vb.d + (size_t)(j + q) * vstride * sizeof(T) * 2;
                auto v = Store<P>::ld(vj, nullptr, e, 0);
                vq[q] = mk((T)v.re, (T)v.im);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double2 hj = h[(long)(j + q) * ldh];
                acc = acc + mk((T)(sign * hj.x), (T)(sign * hj.y)) * vq[q];
            }
        }
        for (; j < nv; ++j) {
            const double2 hj = h[(long)j * ldh];
            const void *vj = (const char *)Vb.d + (size_t)j * vstride * sizeof(T) * 2;
            auto v = Store<P>::ld(vj, nullptr, e, 0);
            acc = acc + mk((T)(sign * hj.x), (T)(sign * hj.y)) * mk((T)v.re, (T)v.im);
        }
        Store<P>::st(w.d, e, acc);
        nrm += (double)acc.re * acc.re + (double)acc.im * acc.im;
    }
    if (!partial) return;
    red[threadIdx.x] = nrm;
    __syncthreads();
    for (int hh = 128; hh > 0; hh >>= 1) {
        if ((int)threadIdx.x < hh) red[threadIdx.x] += red[threadIdx.x + hh];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = make_double2(red[0], 0.0);
}

// End of one single-vector FP64 Arnoldi step, one workgroup: ||w||^2 from the
// partials of the second update (the same sum as k_reduce), then on the first
// wavefront H(:, j) += h2, h_{j+1,j} = ||w||, the breakdown test against the
// running Frobenius norm and the coefficient 1/h of the new basis vector (0
// after a breakdown, which keeps later vectors zero).
__global__ __launch_bounds__(256) void k_arnoldi_finish(const double2 *__restrict__ partial, int NB, double2 *Hcol,
                                                        const double2 *h2, int j, double *state, double2 *scale) {
    // state[0] = running ||H||_F^2, state[1] = d_eff (or -1 while none)
    __shared__ double2 red[256];
    block_sum_partials(partial, NB, 1, 0, 0, red);
    const double wn2 = red[0].x;
    if (threadIdx.x >= 64) return;
    double f = 0.0;
    for (int i = threadIdx.x; i <= j; i += 64) {
        double2 v = Hcol[i];
        v.x += h2[i].x;
        v.y += h2[i].y;
        Hcol[i] = v;
        f += v.x * v.x + v.y * v.y;
    }
    for (int o = 32; o > 0; o >>= 1) f += __shfl_xor(f, o);
    if (threadIdx.x != 0) return;
    double fro = state[0] + f;
    const double hn = sqrt(fmax(wn2, 0.0));
    fro += hn * hn;
    state[0] = fro;
    const bool broken = state[1] >= 0;
    if (broken || hn <= 1e-14 * sqrt(fro) || !(hn == hn)) {
        Hcol[j + 1] = make_double2(0.0, 0.0);
        if (!broken) state[1] = j + 1;
        scale[0] = make_double2(0.0, 0.0);
    } else {
        Hcol[j + 1] = make_double2(hn, 0.0);
        scale[0] = make_double2(1.0 / hn, 0.0);
    }
}

// ---- batches of 2 .. 512 right-hand sides with one basis vector per rhs (a solution's correction: from 1) ----
// A vector is a flat array of rows (site, component) of N elements.  A
// workgroup takes R consecutive rows at a time, R N <= 512 threads, thread t
// element t of them: its right-hand side t % N never changes, and whatever N
// is, a wavefront reads one contiguous run (a (site, rhs) tile reads 64-byte
// pieces at N = 12 and leaves a quarter of its lanes idle).  Bound by HBM: w is
// read once for up to 16 (FP64: 8) basis vectors, all loads of a row group
// issued together.
struct FlatTiling {
    int R;         // rows per workgroup step
    int threads;   // R N rounded up to whole wavefronts
    int NB;        // workgroups per group of basis vectors
};
constexpr int kFlatMaxN = 512;
constexpr size_t kFlatCached = (size_t)640 << 20;   // operands up to here: mostly cached (see blas_multi_dot)

// The flat kernels, or the (site, rhs) tiles?  Tiles read whole lines where 64
// right-hand sides fill a wavefront: there the update gains nothing flat (8^4 x
// 64, ten vectors: 47 us and 53 us), the dot product only from reading w once
// for more than the tiles' four vectors (24^4 x 64 FP16S: four vectors 1,038 us
// in tiles and 1,117 us flat, ten 2,805 us and 2,279 us), and not on small
// lattices, where its workgroups and their partial sums cost more than w (whole
// solves, tiles and flat: 4^4 x 128 FP64 2.75 / 3.10 ms, 4 x 4 x 8 x 8 x 64 5.60 /
// 5.79, 6^4 x 64 5.20 / 5.21 with restarts of 20 and 8.10 / 7.88 of 50; 4 x 4 x 6
// x 8 x 256 15.7 / 15.6).  Nor for FP32 and FP64 vectors of 30 to 60 MB once the
// operands are past kFlatCached: one group of 768 workgroups, whose partial sums
// take 27 us to add and the tiles' 11 (8^4 x 128 FP32 solve 9.09 / 9.28 ms; 75 MB,
// 8^4 x 192, 14.36 / 14.18).  Elsewhere the flat kernels win once a vector is too
// large for its launch to be mere latency (ten vectors and FP32, N = 12: 8^4, 4.7
// MB, 15.8 us in tiles and 17.0 us flat; 12^4, 24 MB, 87.7 us and 53.5 us; 16^4,
// 75 MB, 280 us and 160 us).
bool use_flat(const mpmc_ctx *ctx, int N, int nv, int prec, bool dot) {
    if (N < 2 || N > kFlatMaxN) return false;
    const size_t vb = vec_bytes(ctx, N, prec);
    if (N % 64 != 0) return vb >= (size_t)10000000;
    if (!dot || nv <= JB || (ctx->V < 1200 && ctx->V * N < 150000)) return false;
    return prec == MPMC_FP16S || (nv + 1) * vb <= kFlatCached || vb >= (size_t)60000000;
}

// R near 256 threads' worth, moved to where the fewest lanes of the last
// wavefront idle.  Every workgroup is resident at once, `waves` wavefronts per
// compute unit: a partial second round would run with most of the chip idle
// (16^4 x 12, ten vectors: 161 us with 1,365 workgroups of three wavefronts,
// of which 1,280 fit, 149 us with 1,280).
FlatTiling flat_tiling(const mpmc_ctx *ctx, int N, int groups, int waves = 16) {
    FlatTiling t{1, (N + 63) / 64 * 64, 1};
    for (int R = 1; R * N <= (N <= 128 ? 256 : kFlatMaxN); ++R) {
        const int th = (R * N + 63) / 64 * 64;
        if ((long)R * N * t.threads >= (long)t.R * N * th) {
            t.R = R;
            t.threads = th;
        }
    }
    const long nrb = (ctx->V * 12 + t.R - 1) / t.R;
    const int per_cu = waves * 64 / t.threads;
    long nb = (long)ctx->num_cu * (per_cu > 0 ? per_cu : 1) / groups;
    if (nb < 64) nb = 64;
    const long steps = (nrb + nb - 1) / nb;   // of the busiest workgroup: as few workgroups as it allows
    t.NB = (int)((nrb + steps - 1) / steps);
    return t;
}

// Sums of v[0 .. n-1] over the R threads of each right-hand side (threads r,
// r + N, ...), in a fixed order; the results are thread r's (r < N).  Four at a
// time: the barriers of one sum after the other show on a small lattice
// (6^4 x 12, twelve vectors: 19.2 us one by one, 16.1 us in fours).
constexpr int kFlatSums = 4;
template <int n>
__device__ __forceinline__ void flat_sums(cpx<double> (&v)[n], double2 (*red)[512], int N, int R, int rr, bool live) {
    const int t = threadIdx.x;
#pragma unroll
    for (int q0 = 0; q0 < n; q0 += kFlatSums) {
        if (q0) __syncthreads();
        if (live) {
#pragma unroll
            for (int q = 0; q < kFlatSums; ++q)
                if (q0 + q < n) red[q][t] = make_double2(v[q0 + q].re, v[q0 + q].im);
        }
        __syncthreads();
        for (int h = R; h > 1;) {
            const int half = (h + 1) / 2;
            if (live && rr < h - half) {
#pragma unroll
                for (int q = 0; q < kFlatSums; ++q)
                    if (q0 + q < n) {
                        red[q][t].x += red[q][t + half * N].x;
                        red[q][t].y += red[q][t + half * N].y;
                    }
            }
            __syncthreads();
            h = half;
        }
        if (live && rr == 0) {
#pragma unroll
            for (int q = 0; q < kFlatSums; ++q)
                if (q0 + q < n) v[q0 + q] = mk(red[q][t].x, red[q][t].y);
        }
    }
}

// partial[j][blk][r] = sum over the block's rows of conj(V_j) Theta w for the
// JG basis vectors from blockIdx.y JG on.
template <int P, int JG>
__global__ __launch_bounds__(512) void k_multidot_flat(const void *__restrict__ Vb, size_t vstride_b, int nv,
                                                       const void *__restrict__ w, int N, int R, long rows, int theta,
                                                       double2 *__restrict__ partial, int NB) {
    using E = typename std::conditional<P == MPMC_FP64, double2, float2>::type;
    constexpr int U = JG <= 2 ? (P == MPMC_FP32 ? 4 : 2) : (JG <= 6 && P == MPMC_FP32 ? 2 : 1);   // row groups in flight
    __shared__ double2 red[JG < kFlatSums ? JG : kFlatSums][512];
    const int T = R * N, t = threadIdx.x, rr = t / N;
    const bool live = t < T;
    const int j0 = blockIdx.y * JG;
    cpx<double> acc[JG];
#pragma unroll
    for (int q = 0; q < JG; ++q) acc[q] = mk(0.0, 0.0);
    // rows rb R .. rb R + R - 1; the group's offset is uniform, the lane's is t
    auto group = [&](auto NU, long rb) {
        constexpr int nu = decltype(NU)::value;
        E wv[nu], vv[nu][JG];
#pragma unroll
        for (int u = 0; u < nu; ++u) {
            const size_t off = (size_t)(rb + (long)u * NB) * T * sizeof(E);
            wv[u] = reinterpret_cast<const E *>((const char *)w + off)[t];
#pragma unroll
            for (int q = 0; q < JG; ++q) {   // past the last vector: read again, not used
                const int j = j0 + q < nv ? j0 + q : nv - 1;
                vv[u][q] = reinterpret_cast<const E *>((const char *)Vb + (size_t)j * vstride_b + off)[t];
            }
        }
#pragma unroll
        for (int u = 0; u < nu; ++u) {
            double sg = 1.0;
            if (theta && ((rb + (long)u * NB) * R + rr) % 12 >= 6) sg = -1.0;
            const cpx<double> wd = mk(sg * (double)wv[u].x, sg * (double)wv[u].y);
#pragma unroll
            for (int q = 0; q < JG; ++q)
                acc[q] = acc[q] + conjmul(mk((double)vv[u][q].x, (double)vv[u][q].y), wd);
        }
    };
    if (live) {
        const long full = rows / R;   // whole row groups
        long rb = blockIdx.x;
        for (; rb + (long)(U - 1) * NB < full; rb += (long)U * NB) group(std::integral_constant<int, U>(), rb);
        for (; rb * R + rr < rows; rb += NB) group(std::integral_constant<int, 1>(), rb);
    }
    flat_sums(acc, red, N, R, rr, live);
    if (live && rr == 0) {
#pragma unroll
        for (int q = 0; q < JG; ++q)
            if (j0 + q < nv)
                partial[((long)(j0 + q) * NB + blockIdx.x) * N + t] = make_double2(acc[q].re, acc[q].im);
    }
}

// The same for an FP16S basis and FP32 w: thread = (site, rhs) pair, R sites at
// a time, four components of all JG vectors in flight, so w is read once for
// up to 12 vectors (4 in a (site, rhs) tile with every component in registers).
template <int JG>
__global__ __launch_bounds__(512) void k_multidot_flat_h(const void *__restrict__ Vb, size_t vstride_b,
                                                         size_t vscale_off, int nv, const void *__restrict__ w, int N,
                                                         int R, long V, double2 *__restrict__ partial, int NB) {
    constexpr int KC = 4;
    __shared__ double2 red[JG < kFlatSums ? JG : kFlatSums][512];
    const int T = R * N, t = threadIdx.x, rr = t / N, r = t - rr * N;
    const bool live = t < T;
    const int j0 = blockIdx.y * JG;
    cpx<double> acc[JG];
#pragma unroll
    for (int q = 0; q < JG; ++q) acc[q] = mk(0.0, 0.0);
    const uint32_t lane = (uint32_t)rr * 12u * (uint32_t)N + (uint32_t)r;   // the pair's component 0 within the sites
    if (live) {
        for (long sb = blockIdx.x; sb * R + rr < V; sb += NB) {
            const size_t base = (size_t)sb * T;   // uniform: first pair of the sites
            float sc[JG];
#pragma unroll
            for (int q = 0; q < JG; ++q) {
                const int j = j0 + q < nv ? j0 + q : nv - 1;
                sc[q] = (reinterpret_cast<const float *>((const char *)Vb + (size_t)j * vstride_b + vscale_off) + base)[t];
            }
#pragma unroll 1   // unrolled, all twelve components' loads move up and spill
            for (int kc = 0; kc < 12; kc += KC) {
                float2 wv[KC];
                __half2 vv[KC][JG];
#pragma unroll
                for (int k = 0; k < KC; ++k) {
                    const size_t row = base * 12 + (size_t)(kc + k) * N;
                    wv[k] = (reinterpret_cast<const float2 *>(w) + row)[lane];
#pragma unroll
                    for (int q = 0; q < JG; ++q) {
                        const int j = j0 + q < nv ? j0 + q : nv - 1;
                        vv[k][q] = (reinterpret_cast<const __half2 *>((const char *)Vb + (size_t)j * vstride_b) + row)[lane];
                    }
                }
#pragma unroll
                for (int k = 0; k < KC; ++k) {
                    const cpx<double> wd = mk((double)wv[k].x, (double)wv[k].y);
#pragma unroll
                    for (int q = 0; q < JG; ++q) {
                        const float2 f = __half22float2(vv[k][q]);
                        acc[q] = acc[q] + conjmul(mk((double)(f.x * sc[q]), (double)(f.y * sc[q])), wd);
                    }
                }
            }
        }
    }
    flat_sums(acc, red, N, R, rr, live);
    if (live && rr == 0) {
#pragma unroll
        for (int q = 0; q < JG; ++q)
            if (j0 + q < nv)
                partial[((long)(j0 + q) * NB + blockIdx.x) * N + t] = make_double2(acc[q].re, acc[q].im);
    }
}

// w += sign * sum_j h[j*ldh + r] V_j; optional partial[blk][r] = sum |w|^2.
// NV > 0: exactly NV vectors, coefficients in registers throughout; NV = 0: any
// number, eight at a time with their coefficients read again per row group.
// ADD: as kOutAdd, the sum alone is added to the FP64 batch x.
template <int P, int NV, bool ADD = false>
__global__ __launch_bounds__(512) void k_multiaxpy_flat(const void *__restrict__ Vb, size_t vstride_b, int nv,
                                                        void *__restrict__ w, int N, int R, long rows,
                                                        const double2 *__restrict__ h, int ldh, double sign,
                                                        double2 *__restrict__ partial, int NB,
                                                        void *__restrict__ x = nullptr) {
    using T = typename Store<P>::real;
    using E = typename std::conditional<P == MPMC_FP64, double2, float2>::type;
    constexpr int C = NV > 0 ? NV : 8;
    constexpr int U = C <= 2 ? 4 : (C <= 8 && P == MPMC_FP32 ? 2 : 1);
    __shared__ double2 red[1][512];
    const int Tn = R * N, t = threadIdx.x, rr = t / N, r = t - rr * N;
    const bool live = t < Tn;
    double nrm = 0;
    cpx<T> c[C];
    auto coefs = [&](int j0) {
#pragma unroll
        for (int q = 0; q < C; ++q) {
            const int j = NV > 0 || j0 + q < nv ? j0 + q : nv - 1;
            const double2 hj = h[(long)j * ldh + r];
            c[q] = mk((T)(sign * hj.x), (T)(sign * hj.y));
        }
    };
    auto group = [&](auto NU, long rb) {
        constexpr int nu = decltype(NU)::value;
        cpx<T> acc[nu];
        auto chunk = [&](int j0) {
            E vv[nu][C];
#pragma unroll
            for (int u = 0; u < nu; ++u) {
                const size_t off = (size_t)(rb + (long)u * NB) * Tn * sizeof(E);
#pragma unroll
                for (int q = 0; q < C; ++q) {
                    const int j = NV > 0 || j0 + q < nv ? j0 + q : nv - 1;
                    vv[u][q] = reinterpret_cast<const E *>((const char *)Vb + (size_t)j * vstride_b + off)[t];
                }
            }
#pragma unroll
            for (int q = 0; q < C; ++q)
                if (NV > 0 || j0 + q < nv)
#pragma unroll
                    for (int u = 0; u < nu; ++u) acc[u] = acc[u] + c[q] * mk((T)vv[u][q].x, (T)vv[u][q].y);
        };
#pragma unroll
        for (int u = 0; u < nu; ++u) {
            if constexpr (ADD) {
                acc[u] = mk(T(0), T(0));
            } else {
                const E v = reinterpret_cast<const E *>((const char *)w + (size_t)(rb + (long)u * NB) * Tn * sizeof(E))[t];
                acc[u] = mk((T)v.x, (T)v.y);
            }
        }
        if constexpr (NV > 0) {
            chunk(0);
        } else {
            for (int j0 = 0; j0 < nv; j0 += C) {
                coefs(j0);
                chunk(j0);
            }
        }
#pragma unroll
        for (int u = 0; u < nu; ++u) {
            if constexpr (ADD) {
                add_fp64(x, (rb + (long)u * NB) * Tn + t, (double)acc[u].re, (double)acc[u].im);
                continue;
            }
            E o;
            o.x = acc[u].re;
            o.y = acc[u].im;
            reinterpret_cast<E *>((char *)w + (size_t)(rb + (long)u * NB) * Tn * sizeof(E))[t] = o;
            nrm += (double)acc[u].re * acc[u].re + (double)acc[u].im * acc[u].im;
        }
    };
    if (live) {
        if constexpr (NV > 0) coefs(0);
        const long full = rows / R;
        long rb = blockIdx.x;
        for (; rb + (long)(U - 1) * NB < full; rb += (long)U * NB) group(std::integral_constant<int, U>(), rb);
        for (; rb * R + rr < rows; rb += NB) group(std::integral_constant<int, 1>(), rb);
    }
    if (!partial) return;
    cpx<double> v[1] = {mk(nrm, 0.0)};
    flat_sums(v, red, N, R, rr, live);
    if (live && rr == 0) partial[(long)blockIdx.x * N + r] = make_double2(v[0].re, 0.0);
}

// f(std::integral_constant<int, n>()) for the run-time n in 1 .. MAX
template <int MAX, typename F>
void with_count(int n, F &&f) {
    if constexpr (MAX > 1) {
        if (n < MAX) {
            with_count<MAX - 1>(n, f);
            return;
        }
    }
    f(std::integral_constant<int, MAX>());
}

int nb_single(const mpmc_ctx *ctx, long n, int groups) {
    long nb = (long)ctx->num_cu * 8 / (groups > 0 ? groups : 1);
    const long maxnb = (n + 255) / 256;
    if (nb < 8) nb = 8;
    if (nb > maxnb) nb = maxnb;
    if (nb > 2048) nb = 2048;
    return (int)nb;
}

}  // namespace

int blas_scale_acc(mpmc_ctx *ctx, const double *t, int N, double2 c, double sign, double *acc) {
    k_scale_acc<<<grid_for(N, 64), 64, 0, ctx->stream>>>((const double2 *)t, N, c, sign, (double2 *)acc);
    HIP_OR_RET(ctx, hipGetLastError());
    return MPMC_OK;
}

// h[j*N + r] (+)= V_j^H Theta w for j < nv.  Vb: nv vectors spaced vstride
// elements (complex) apart.
int blas_multi_dot(mpmc_ctx *ctx, const void *Vb, long vstride, int vN, int nv, const void *w, int nrhs, int prec,
                   double *h_dev, int accumulate, int theta) {
    if (nv <= 0) return MPMC_OK;
    const int groups = (nv + JB - 1) / JB;
    if (nrhs == 1 && vN == 1) {
        const int NB = nb_single(ctx, ctx->n, groups);
        double2 *part = (double2 *)ws_get(ctx, WS_PARTIAL, (size_t)nv * NB * sizeof(double2));
        if (!part) return MPMC_ENOMEM;
        int rc = dispatch_prec(ctx, prec, [&](auto P) {
            k_multidot1<decltype(P)::value><<<dim3(NB, groups), 256, 0, ctx->stream>>>(
                vref(ctx, Vb, 1, prec), vstride, nv, vref(ctx, w, 1, prec), ctx->n, theta, part, NB);
        });
        RET_IF(rc);
        k_reduce<<<nv, 256, 0, ctx->stream>>>(part, NB, 1, (double2 *)h_dev, accumulate, 0);
        HIP_OR_RET(ctx, hipGetLastError());
        return MPMC_OK;
    }
    if (vN == nrhs && (prec == MPMC_FP64 || prec == MPMC_FP32) && use_flat(ctx, nrhs, nv, prec, true)) {
        // basis vectors per group, evenly filled: as many as the registers allow,
        // since each group reads w again (16^4 x 64 FP32, 16 vectors: 1,193 us
        // in one group, 1,290 us in four); four where much of it stays in the
        // 256 MB memory-side cache and wavefronts in flight count for more
        // (8^4 x 64, 12 vectors: 66 us in three groups, 75 us in one)
        const size_t vb = (size_t)ctx->n * nrhs * (prec == MPMC_FP64 ? 16 : 8);
        const int most = (nv + 1) * vb <= kFlatCached ? 4 : prec == MPMC_FP64 ? 8 : 16;
        const int ng = (nv + most - 1) / most, per = (nv + ng - 1) / ng;
        const FlatTiling t = flat_tiling(ctx, nrhs, ng, per > 12 ? 12 : 16);
        double2 *part = (double2 *)ws_get(ctx, WS_PARTIAL, (size_t)nv * t.NB * nrhs * sizeof(double2));
        if (!part) return MPMC_ENOMEM;
        const dim3 grd(t.NB, ng);
        if (prec == MPMC_FP64)
            with_count<8>(per, [&](auto JG) {
                k_multidot_flat<MPMC_FP64, decltype(JG)::value><<<grd, t.threads, 0, ctx->stream>>>(
                    Vb, (size_t)vstride * 16, nv, w, nrhs, t.R, ctx->V * 12, theta, part, t.NB);
            });
        else
            with_count<16>(per, [&](auto JG) {
                k_multidot_flat<MPMC_FP32, decltype(JG)::value><<<grd, t.threads, 0, ctx->stream>>>(
                    Vb, (size_t)vstride * 8, nv, w, nrhs, t.R, ctx->V * 12, theta, part, t.NB);
            });
        HIP_OR_RET(ctx, hipGetLastError());
        k_reduce<<<nv * nrhs, 256, 0, ctx->stream>>>(part, t.NB, nrhs, (double2 *)h_dev, accumulate, 0);
        HIP_OR_RET(ctx, hipGetLastError());
        return MPMC_OK;
    }
    Tiling t = tiling(ctx, nrhs, groups);
    double2 *part = (double2 *)ws_get(ctx, WS_PARTIAL, (size_t)nv * t.NB * nrhs * sizeof(double2));
    if (!part) return MPMC_ENOMEM;
    dim3 blk(t.RT, t.CT), grd(t.NB, t.ntile, groups);
    const size_t es = prec == MPMC_FP64 ? 16 : 8;
    int rc = dispatch_prec(ctx, prec, [&](auto P) {
        k_multidot<decltype(P)::value, decltype(P)::value><<<grd, blk, 0, ctx->stream>>>(
            vref(ctx, Vb, nrhs, prec), (size_t)vstride * es, 0, vN, nv, vref(ctx, w, nrhs, prec), nrhs, ctx->V, theta,
            part, t.NB);
    });
    RET_IF(rc);
    k_reduce<<<nv * nrhs, 256, 0, ctx->stream>>>(part, t.NB, nrhs, (double2 *)h_dev, accumulate, 0);
    HIP_OR_RET(ctx, hipGetLastError());
    return MPMC_OK;
}

// FP16S basis (nrhs-wide batches vstride_b bytes apart) against an FP32 w.
int blas_multi_dot_h(mpmc_ctx *ctx, const void *Vb, size_t vstride_b, int nv, const void *w, int nrhs,
                     double *h_dev, int accumulate) {
    if (nv <= 0) return MPMC_OK;
    if (use_flat(ctx, nrhs, nv, MPMC_FP16S, true)) {
        const int most = nv * vstride_b + vec_bytes(ctx, nrhs, MPMC_FP32) <= kFlatCached ? 4 : 12;   // as blas_multi_dot
        const int ng = (nv + most - 1) / most, per = (nv + ng - 1) / ng;
        const FlatTiling t = flat_tiling(ctx, nrhs, ng, per > 10 ? 12 : 16);
        double2 *part = (double2 *)ws_get(ctx, WS_PARTIAL, (size_t)nv * t.NB * nrhs * sizeof(double2));
        if (!part) return MPMC_ENOMEM;
        with_count<12>(per, [&](auto JG) {
            k_multidot_flat_h<decltype(JG)::value><<<dim3(t.NB, ng), t.threads, 0, ctx->stream>>>(
                Vb, vstride_b, fp16s_scale_offset(ctx, nrhs), nv, w, nrhs, t.R, ctx->V, part, t.NB);
        });
        HIP_OR_RET(ctx, hipGetLastError());
        k_reduce<<<nv * nrhs, 256, 0, ctx->stream>>>(part, t.NB, nrhs, (double2 *)h_dev, accumulate, 0);
        HIP_OR_RET(ctx, hipGetLastError());
        return MPMC_OK;
    }
    const int groups = (nv + JB - 1) / JB;
    Tiling t = tiling(ctx, nrhs, groups);
    double2 *part = (double2 *)ws_get(ctx, WS_PARTIAL, (size_t)nv * t.NB * nrhs * sizeof(double2));
    if (!part) return MPMC_ENOMEM;
    dim3 blk(t.RT, t.CT), grd(t.NB, t.ntile, groups);
    k_multidot<MPMC_FP16S, MPMC_FP32><<<grd, blk, 0, ctx->stream>>>(
        VecRef{const_cast<void *>(Vb), nullptr}, vstride_b, fp16s_scale_offset(ctx, nrhs), nrhs, nv,
        vref(ctx, w, nrhs, MPMC_FP32), nrhs, ctx->V, 0, part, t.NB);
    HIP_OR_RET(ctx, hipGetLastError());
    k_reduce<<<nv * nrhs, 256, 0, ctx->stream>>>(part, t.NB, nrhs, (double2 *)h_dev, accumulate, 0);
    HIP_OR_RET(ctx, hipGetLastError());
    return MPMC_OK;
}

int blas_reduce(mpmc_ctx *ctx, const void *part, int NB, int nj, int nrhs, double *out_dev) {
    k_reduce<<<nj * nrhs, 256, 0, ctx->stream>>>((const double2 *)part, NB, nrhs, (double2 *)out_dev, 0, 0);
    HIP_OR_RET(ctx, hipGetLastError());
    return MPMC_OK;
}

int blas_dot(mpmc_ctx *ctx, const void *x, const void *y, int nrhs, int prec, int theta, double *out_dev) {
    return blas_multi_dot(ctx, x, 0, nrhs, 1, y, nrhs, prec, out_dev, 0, theta);
}

int blas_norm2(mpmc_ctx *ctx, const void *x, int nrhs, int prec, double *out_dev) {
    return blas_multi_dot(ctx, x, 0, nrhs, 1, x, nrhs, prec, out_dev, 0, 0);
}

int blas_arnoldi_update(mpmc_ctx *ctx, const void *V, long vstride, int nv, void *w, const double *h2, double *Hcol,
                        int j, double *state, double *scale, int prec) {
    const int NB = nb_single(ctx, ctx->n, 1);
    double2 *part = (double2 *)ws_get(ctx, WS_PARTIAL, (size_t)NB * sizeof(double2));
    if (!part) return MPMC_ENOMEM;
    if (prec == MPMC_FP64)
        k_multiaxpy1<MPMC_FP64><<<NB, 256, 0, ctx->stream>>>(vref(ctx, V, 1, prec), vstride, nv, vref(ctx, w, 1, prec),
                                                             ctx->n, (const double2 *)h2, 1, -1.0, part, NB);
    else if (prec == MPMC_FP32)
        k_multiaxpy1<MPMC_FP32><<<NB, 256, 0, ctx->stream>>>(vref(ctx, V, 1, prec), vstride, nv, vref(ctx, w, 1, prec),
                                                             ctx->n, (const double2 *)h2, 1, -1.0, part, NB);
    else
        return set_err(ctx, MPMC_EINVAL, "Arnoldi vectors are FP64 or FP32");
    HIP_OR_RET(ctx, hipGetLastError());
    k_arnoldi_finish<<<1, 256, 0, ctx->stream>>>(part, NB, (double2 *)Hcol, (const double2 *)h2, j, state,
                                                 (double2 *)scale);
    HIP_OR_RET(ctx, hipGetLastError());
    return MPMC_OK;
}

// w += sign * sum_j h[j*ldh + r] V_j ; if norm2_dev: norm2_dev[r] = ||w_r||^2 (after update)
int blas_multi_axpy(mpmc_ctx *ctx, const void *Vb, long vstride, int vN, int nv, void *w, int nrhs, int prec,
                    const double *h_dev, int ldh, double sign, double *norm2_dev) {
    if (nrhs == 1 && vN == 1) {
        const int NB = nb_single(ctx, ctx->n, 1);
        double2 *part = nullptr;
        if (norm2_dev) {
            part = (double2 *)ws_get(ctx, WS_PARTIAL, (size_t)NB * sizeof(double2));
            if (!part) return MPMC_ENOMEM;
        }
        int rc = dispatch_prec(ctx, prec, [&](auto P) {
            k_multiaxpy1<decltype(P)::value><<<NB, 256, 0, ctx->stream>>>(vref(ctx, Vb, 1, prec), vstride, nv,
                                                                          vref(ctx, w, 1, prec), ctx->n,
                                                                          (const double2 *)h_dev, ldh, sign, part, NB);
        });
        RET_IF(rc);
        if (norm2_dev) {
            k_reduce<<<1, 256, 0, ctx->stream>>>(part, NB, 1, (double2 *)norm2_dev, 0, 1);
            HIP_OR_RET(ctx, hipGetLastError());
        }
        return MPMC_OK;
    }
    if (vN == nrhs && nv > 0 && (prec == MPMC_FP64 || prec == MPMC_FP32) && use_flat(ctx, nrhs, nv, prec, false)) {
        const FlatTiling t = flat_tiling(ctx, nrhs, 1);
        double2 *part = nullptr;
        if (norm2_dev) {
            part = (double2 *)ws_get(ctx, WS_PARTIAL, (size_t)t.NB * nrhs * sizeof(double2));
            if (!part) return MPMC_ENOMEM;
        }
        const size_t vs = (size_t)vstride * (prec == MPMC_FP64 ? 16 : 8);
        auto launch = [&](auto P, auto NV) {
            k_multiaxpy_flat<decltype(P)::value, decltype(NV)::value><<<t.NB, t.threads, 0, ctx->stream>>>(
                Vb, vs, nv, w, nrhs, t.R, ctx->V * 12, (const double2 *)h_dev, ldh, sign, part, t.NB);
        };
        if (prec == MPMC_FP64) {
            const std::integral_constant<int, MPMC_FP64> P;
            if (nv <= 12) with_count<12>(nv, [&](auto NV) { launch(P, NV); });
            else launch(P, std::integral_constant<int, 0>());
        } else {
            const std::integral_constant<int, MPMC_FP32> P;
            // 25 to 30 vectors of 16^4 x 12: 424 us with the count known, 500 without
            if (nv <= 32) with_count<32>(nv, [&](auto NV) { launch(P, NV); });
            else launch(P, std::integral_constant<int, 0>());
        }
        HIP_OR_RET(ctx, hipGetLastError());
        if (norm2_dev) {
            k_reduce<<<nrhs, 256, 0, ctx->stream>>>(part, t.NB, nrhs, (double2 *)norm2_dev, 0, 1);
            HIP_OR_RET(ctx, hipGetLastError());
        }
        return MPMC_OK;
    }
    Tiling t = tiling(ctx, nrhs, 1);
    double2 *part = nullptr;
    if (norm2_dev) {
        part = (double2 *)ws_get(ctx, WS_PARTIAL, (size_t)t.NB * nrhs * sizeof(double2));
        if (!part) return MPMC_ENOMEM;
    }
    dim3 blk(t.RT, t.CT), grd(t.NB, t.ntile, 1);
    const size_t es = prec == MPMC_FP64 ? 16 : 8;
    int rc = dispatch_prec(ctx, prec, [&](auto P) {
        k_multiaxpy<decltype(P)::value, decltype(P)::value><<<grd, blk, 0, ctx->stream>>>(
            vref(ctx, Vb, nrhs, prec), (size_t)vstride * es, 0, vN, nv, vref(ctx, w, nrhs, prec), nrhs, ctx->V,
            (const double2 *)h_dev, sign, part, t.NB, ldh);
    });
    RET_IF(rc);
    if (norm2_dev) {
        k_reduce<<<nrhs, 256, 0, ctx->stream>>>(part, t.NB, nrhs, (double2 *)norm2_dev, 0, 1);
        HIP_OR_RET(ctx, hipGetLastError());
    }
    return MPMC_OK;
}

// w (FP32) += sign * sum_j h[j*ldh + r] V_j with an FP16S basis
int blas_multi_axpy_h(mpmc_ctx *ctx, const void *Vb, size_t vstride_b, int nv, void *w, int nrhs,
                      const double *h_dev, int ldh, double sign, double *norm2_dev, void *out_h) {
    Tiling t = tiling(ctx, nrhs, 1);
    double2 *part = nullptr;
    if (norm2_dev) {
        part = (double2 *)ws_get(ctx, WS_PARTIAL, (size_t)t.NB * nrhs * sizeof(double2));
        if (!part) return MPMC_ENOMEM;
    }
    dim3 blk(t.RT, t.CT), grd(t.NB, t.ntile, 1);
    if (out_h)
        k_multiaxpy<MPMC_FP16S, MPMC_FP32, kOutHalf><<<grd, blk, 0, ctx->stream>>>(
            VecRef{const_cast<void *>(Vb), nullptr}, vstride_b, fp16s_scale_offset(ctx, nrhs), nrhs, nv,
            vref(ctx, w, nrhs, MPMC_FP32), nrhs, ctx->V, (const double2 *)h_dev, sign, part, t.NB, ldh,
            vref(ctx, out_h, nrhs, MPMC_FP16S));
    else
        k_multiaxpy<MPMC_FP16S, MPMC_FP32><<<grd, blk, 0, ctx->stream>>>(
            VecRef{const_cast<void *>(Vb), nullptr}, vstride_b, fp16s_scale_offset(ctx, nrhs), nrhs, nv,
            vref(ctx, w, nrhs, MPMC_FP32), nrhs, ctx->V, (const double2 *)h_dev, sign, part, t.NB, ldh);
    HIP_OR_RET(ctx, hipGetLastError());
    if (norm2_dev) {
        k_reduce<<<nrhs, 256, 0, ctx->stream>>>(part, t.NB, nrhs, (double2 *)norm2_dev, 0, 1);
        HIP_OR_RET(ctx, hipGetLastError());
    }
    return MPMC_OK;
}

// x (FP64) += sum_j y[j*nrhs + r] V_j for a basis in prec (FP64, FP32 or FP16S;
// sums in FP64 or FP32), basis vectors vstride_b bytes apart
int blas_solution_add(mpmc_ctx *ctx, const void *Vb, size_t vstride_b, int nv, int prec, void *x, int nrhs,
                      const double *y_dev) {
    if (nv <= 0) return MPMC_OK;
    const double2 *y = (const double2 *)y_dev;
    // a single vector is one run of elements: flat, a tile's lanes are 12 elements
    // apart (20 FP64 vectors of 16^4: 52 us in tiles, 45 us; solves with restarts
    // of ten at 24^4 21.1 -> 20.7 ms, 8^4 1.44 -> 1.40)
    if (prec != MPMC_FP16S && (nrhs == 1 || use_flat(ctx, nrhs, nv, prec, false))) {
        const FlatTiling t = flat_tiling(ctx, nrhs, 1);
        auto launch = [&](auto P, auto NV) {
            k_multiaxpy_flat<decltype(P)::value, decltype(NV)::value, true><<<t.NB, t.threads, 0, ctx->stream>>>(
                Vb, vstride_b, nv, nullptr, nrhs, t.R, ctx->V * 12, y, nrhs, 1.0, nullptr, t.NB, x);
        };
        if (prec == MPMC_FP64) launch(std::integral_constant<int, MPMC_FP64>(), std::integral_constant<int, 0>());
        else launch(std::integral_constant<int, MPMC_FP32>(), std::integral_constant<int, 0>());
        HIP_OR_RET(ctx, hipGetLastError());
        return MPMC_OK;
    }
    const Tiling t = tiling(ctx, nrhs, 1);
    const dim3 blk(t.RT, t.CT), grd(t.NB, t.ntile, 1);
    const VecRef V{const_cast<void *>(Vb), nullptr}, none{nullptr, nullptr}, xr{x, nullptr};
    if (prec == MPMC_FP64)
        k_multiaxpy<MPMC_FP64, MPMC_FP64, kOutAdd><<<grd, blk, 0, ctx->stream>>>(V, vstride_b, 0, nrhs, nv, none, nrhs,
                                                                                 ctx->V, y, 1.0, nullptr, t.NB, nrhs, xr);
    else if (prec == MPMC_FP32)
        k_multiaxpy<MPMC_FP32, MPMC_FP32, kOutAdd><<<grd, blk, 0, ctx->stream>>>(V, vstride_b, 0, nrhs, nv, none, nrhs,
                                                                                 ctx->V, y, 1.0, nullptr, t.NB, nrhs, xr);
    else
        k_multiaxpy<MPMC_FP16S, MPMC_FP32, kOutAdd><<<grd, blk, 0, ctx->stream>>>(
            V, vstride_b, fp16s_scale_offset(ctx, nrhs), nrhs, nv, none, nrhs, ctx->V, y, 1.0, nullptr, t.NB, nrhs, xr);
    HIP_OR_RET(ctx, hipGetLastError());
    return MPMC_OK;
}

// y (prec) = x (FP64) / sqrt(re nrm[r])
int blas_convert_normalised(mpmc_ctx *ctx, const void *x, void *y, int prec, int nrhs, const double *nrm_dev) {
    const unsigned g = grid_for(ctx->V * nrhs, 256);
    const VecRef xr = vref(ctx, x, nrhs, MPMC_FP64), yr = vref(ctx, y, nrhs, prec);
    const double2 *nrm = (const double2 *)nrm_dev;
    if (prec == MPMC_FP64) k_convert_normalised<MPMC_FP64><<<g, 256, 0, ctx->stream>>>(xr, yr, ctx->V, nrhs, nrm);
    else if (prec == MPMC_FP32) k_convert_normalised<MPMC_FP32><<<g, 256, 0, ctx->stream>>>(xr, yr, ctx->V, nrhs, nrm);
    else k_convert_normalised<MPMC_FP16S><<<g, 256, 0, ctx->stream>>>(xr, yr, ctx->V, nrhs, nrm);
    HIP_OR_RET(ctx, hipGetLastError());
    return MPMC_OK;
}

// w += sign * sum_j h[j*ldh + r] V_j, then h2[j*nrhs + r] = V_j^H w (j < nv):
// one pass over the basis for FP32 storage and nv <= 16 (one basis vector per
// right-hand side), blas_multi_axpy + blas_multi_dot otherwise (an FP64
// version would need twice the registers and spills).
int blas_multi_axpy_dot(mpmc_ctx *ctx, const void *Vb, long vstride, int nv, void *w, int nrhs, int prec,
                        const double *h_dev, int ldh, double sign, double *h2_dev) {
    constexpr int NVMAX = 16;
    if (nv > NVMAX || nrhs < 2 || prec != MPMC_FP32) {
        RET_IF(blas_multi_axpy(ctx, Vb, vstride, nrhs, nv, w, nrhs, prec, h_dev, ldh, sign, nullptr));
        return blas_multi_dot(ctx, Vb, vstride, nrhs, nv, w, nrhs, prec, h2_dev, 0, 0);
    }
    if (nv <= 0) return MPMC_OK;
    Tiling t = tiling(ctx, nrhs, 1);
    double2 *part = (double2 *)ws_get(ctx, WS_PARTIAL, (size_t)nv * t.NB * nrhs * sizeof(double2));
    if (!part) return MPMC_ENOMEM;
    dim3 blk(t.RT, t.CT), grd(t.NB, t.ntile, 1);
    k_multiaxpy_dot<MPMC_FP32, NVMAX><<<grd, blk, 0, ctx->stream>>>(
        vref(ctx, Vb, nrhs, prec), (size_t)vstride * 8, nv, vref(ctx, w, nrhs, prec), nrhs, ctx->V,
        (const double2 *)h_dev, sign, ldh, part, t.NB);
    HIP_OR_RET(ctx, hipGetLastError());
    k_reduce<<<nv * nrhs, 256, 0, ctx->stream>>>(part, t.NB, nrhs, (double2 *)h2_dev, 0, 0);
    HIP_OR_RET(ctx, hipGetLastError());
    return MPMC_OK;
}

int blas_axpby(mpmc_ctx *ctx, const void *x, void *y, int nrhs, int prec, double2 a, double2 b) {
    const long total = ctx->V * 12 * nrhs;
    return dispatch_prec(ctx, prec, [&](auto P) {
        k_axpby<decltype(P)::value><<<grid_for(total, 256), 256, 0, ctx->stream>>>(
            vref(ctx, x, nrhs, prec), vref(ctx, y, nrhs, prec), total, a, b);
    });
}

// y = coef[r] x  (mode 0), y = x / sqrt(re coef[r]) (mode 1), y = x / coef[r] (mode 2)
int blas_scale_rhs(mpmc_ctx *ctx, const void *x, void *y, int nrhs, int prec, const double *coef_dev, int mode) {
    const long total = ctx->V * 12 * nrhs;
    return dispatch_prec(ctx, prec, [&](auto P) {
        k_scale_rhs<decltype(P)::value><<<grid_for(total, 256), 256, 0, ctx->stream>>>(
            vref(ctx, x, nrhs, prec), vref(ctx, y, nrhs, prec), total, nrhs, (const double2 *)coef_dev, mode);
    });
}

// y's per-(site, rhs) scales *= Re coef[r] (FP16S y; its half values stay)
__global__ void k_scale_h(float *__restrict__ sc, long total, int N, const double2 *__restrict__ coef) {
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= total) return;
    sc[t] = sc[t] * (float)coef[t % N].x;
}

int blas_scale_h(mpmc_ctx *ctx, void *y, int nrhs, const double *coef_dev) {
    const long total = ctx->V * nrhs;
    k_scale_h<<<grid_for(total, 256), 256, 0, ctx->stream>>>(vref(ctx, y, nrhs, MPMC_FP16S).sc, total, nrhs,
                                                            (const double2 *)coef_dev);
    HIP_OR_RET(ctx, hipGetLastError());
    return MPMC_OK;
}

int blas_convert_scaled_h(mpmc_ctx *ctx, const void *x, void *y, int nrhs, const double *coef_dev) {
    k_convert_scaled_h<<<grid_for(ctx->V * nrhs, 256), 256, 0, ctx->stream>>>(
        vref(ctx, x, nrhs, MPMC_FP32), vref(ctx, y, nrhs, MPMC_FP16S), ctx->V, nrhs, (const double2 *)coef_dev);
    HIP_OR_RET(ctx, hipGetLastError());
    return MPMC_OK;
}

int blas_convert(mpmc_ctx *ctx, const void *x, int px, void *y, int py, int nrhs) {
    const long work = ctx->V * nrhs;
    VecRef xr = vref(ctx, x, nrhs, px), yr = vref(ctx, y, nrhs, py);
    const unsigned g = grid_for(work, 256);
    hipStream_t st = ctx->stream;
#define CONV(A, B) \
    if (px == A && py == B) k_convert<A, B><<<g, 256, 0, st>>>(xr, yr, ctx->V, nrhs); else
    CONV(MPMC_FP64, MPMC_FP32)
    CONV(MPMC_FP32, MPMC_FP64)
    CONV(MPMC_FP64, MPMC_FP16S)
    CONV(MPMC_FP16S, MPMC_FP64)
    CONV(MPMC_FP32, MPMC_FP16S)
    CONV(MPMC_FP16S, MPMC_FP32)
    CONV(MPMC_FP64, MPMC_FP64)
    CONV(MPMC_FP32, MPMC_FP32)
    return set_err(ctx, MPMC_EINVAL, "blas_convert: %d -> %d unsupported", px, py);
#undef CONV
    HIP_OR_RET(ctx, hipGetLastError());
    return MPMC_OK;
}

int blas_zero(mpmc_ctx *ctx, void *y, int nrhs, int prec) {
    HIP_OR_RET(ctx, hipMemsetAsync(y, 0, vec_bytes(ctx, nrhs, prec), ctx->stream));
    return MPMC_OK;
}
