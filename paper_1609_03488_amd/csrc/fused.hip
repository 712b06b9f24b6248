// Fused ADMM steps for small instances: one workgroup per instance.
//
// A workgroup runs `nsteps` whole HSDE ADMM steps of its instance -- w_y, the
// right-hand side A^T w_y, the conjugate-gradient loop (Section IV-B listing,
// with its data-dependent trip count), the u~_tau solve, relaxation, cone
// projection and dual update (Section V-B) -- and then the termination test,
// with only workgroup barriers: no grid-wide synchronisation and no launch per
// step.  Reductions are fixed-order workgroup sums, so an instance's numbers do
// not depend on the other instances of the launch.  Arithmetic per element is
// the same as in the multi-kernel path; only the reduction trees differ.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>

#include "kernels.hpp"
#include "device_common.hpp"

namespace cgs {

constexpr int FNT = FUSED_THREADS;   // threads per instance workgroup
constexpr int FU = 2;      // elements per thread whose loads are issued together

// Workgroup sum in a fixed order; every thread receives the result.
DEVI double bsum(double v, double* sh) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = 0.0;
#pragma unroll
    for (int i = 0; i < FNT / 64; ++i) r += sh[i];
    return r;
}

// Elementwise pass over [0, len): the thread's elements tid + FNT j, FU at a
// time, with all FU elements' loads (ld) issued before any of their stores
// (st).  Element by element, every load would wait for the previous
// element's stores (the compiler cannot tell the vectors apart), one memory
// round trip each; more than two at a time measured slower (code size).
// Elements are visited in increasing j, so sums that st accumulates keep the
// order of a plain loop.  Indices are 32-bit: an instance on this path has
// n + m <= fused_max.
template <typename R, typename L, typename S>
DEVI void ew(int len, L ld, S st) {
    for (int i0 = threadIdx.x; i0 < len; i0 += FNT * FU) {
        R rg[FU];
#pragma unroll
        for (int u = 0; u < FU; ++u) {
            const int i = i0 + u * FNT;
            if (i < len) ld(rg[u], i);
        }
#pragma unroll
        for (int u = 0; u < FU; ++u) {
            const int i = i0 + u * FNT;
            if (i < len) st(rg[u], i);
        }
    }
}

// Where an instance's vectors live during a fused launch.  Every vector
// starts in the instance's region of global memory; the ones the CG loop and
// the step's other passes touch most are moved into the workgroup's LDS for the
// launch when they fit (a flat pointer reaches either), in the order of
// kResident, and written back at its end.  Only where the values sit changes:
// the arithmetic is the same.
template <typename T>
struct FVecs {
    T* x[NXV];
    T* y[NYV];
    unsigned res;   // bit j: kResident[j] is in LDS
};
// (X vectors below NXV, Y vectors as NXV + their index)
constexpr int kResident[] = {XP, XQ, XR, XZ, XK, NXV + YT, NXV + YA, XH, NXV + YW, NXV + YZ};
constexpr int kNumResident = sizeof(kResident) / sizeof(kResident[0]);
// carried from one launch to the next (the others are written before they are read)
constexpr bool resident_live(int v) { return v == XZ || v == XK || v == NXV + YA; }

template <typename T>
DEVI T*& fv_slot(FVecs<T>& fv, int v) { return v < NXV ? fv.x[v] : fv.y[v - NXV]; }

// Copy every resident vector between LDS and the instance's region: to LDS
// (in = true: only the vectors that hold live values) or back (in = false).
template <typename T>
DEVI void fv_copy(const InstDesc& d, FVecs<T>& fv, bool in) {
#pragma unroll
    for (int j = 0; j < kNumResident; ++j) {
        if (!((fv.res >> j) & 1u)) continue;
        const int v = kResident[j];
        if (in && !resident_live(v)) continue;
        T* lds = fv_slot(fv, v);
        T* glb = v < NXV ? (T*)xvec<T>(d, v) : (T*)yvec<T>(d, v - NXV);
        const int64_t len = v < NXV ? d.n : d.m;
        T* dst = in ? lds : glb;
        const T* src = in ? glb : lds;
        for (int64_t i0 = threadIdx.x; i0 < len; i0 += (int64_t)FNT * 8) {
            T t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t i = i0 + (int64_t)u * FNT;
                if (i < len) t[u] = src[i];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t i = i0 + (int64_t)u * FNT;
                if (i < len) dst[i] = t[u];
            }
        }
    }
    __syncthreads();
}

// out_rows += sigma * scale * W in (W = A or its stored transpose); a wave per row.
template <typename T>
DEVI void dense_rows(const DenseBlock& db, int adj, T* out, const T* in, double sigma) {
    gptr<const T> a = (gptr<const T>)(adj ? db.at : db.a);
    const int64_t ld = adj ? db.ldt() : db.ld();
    const int64_t nrows = adj ? db.cols : db.rows, ncols = adj ? db.rows : db.cols;
    T* o = out + (adj ? db.col0 : db.row0);
    const T* x = in + (adj ? db.row0 : db.col0);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double s = sigma * db.scale;
    for (int64_t r = wave; r < nrows; r += FNT / 64) {
        double acc = 0.0;
        for (int64_t j = lane; j < ncols; j += 64) acc = fma((double)a[r * ld + j], (double)x[j], acc);
        acc = wave_sum(acc);
        if (lane == 0) o[r] = (T)((double)o[r] + s * acc);
    }
}

// out = base (or 0) + the identity blocks' terms, every entry of out: FU
// elements at a time, their base and the inputs of up to four identity blocks
// loaded together, then added block by block in the blocks' order.
template <typename T>
DEVI void f_identity(const Tables& tb, const InstDesc& d, int adj, T* o, const T* src, const T* bs,
                     int64_t len64, double sigma) {
    constexpr int NB = 4;
    const int len = (int)len64;
    for (int i0 = threadIdx.x; i0 < len; i0 += FNT * FU) {
        double v[FU];
#pragma unroll
        for (int u = 0; u < FU; ++u) {
            const int i = i0 + u * FNT;
            v[u] = (bs && i < len) ? (double)bs[i] : 0.0;
        }
        for (int b0 = d.id0; b0 < d.id1; b0 += NB) {
            int r0[NB], c0[NB], ln[NB];
            double sb[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if (b0 + b < d.id1) {
                    const IdBlock ib = tb.ids[b0 + b];
                    r0[b] = (int)(adj ? ib.col0 : ib.row0);
                    c0[b] = (int)(adj ? ib.row0 : ib.col0);
                    ln[b] = (int)ib.len;
                    sb[b] = ib.scale;
                } else {
                    r0[b] = c0[b] = ln[b] = 0;
                    sb[b] = 0.0;
                }
            }
            T x[NB][FU];
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int u = 0; u < FU; ++u) {
                    const int i = i0 + u * FNT;
                    x[b][u] = (i < len && i >= r0[b] && i < r0[b] + ln[b]) ? src[i - r0[b] + c0[b]] : T(0);
                }
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int u = 0; u < FU; ++u) {
                    const int i = i0 + u * FNT;
                    if (i >= r0[b] && i < r0[b] + ln[b]) v[u] += sigma * sb[b] * (double)x[b][u];
                }
        }
#pragma unroll
        for (int u = 0; u < FU; ++u) {
            const int i = i0 + u * FNT;
            if (i < len) o[i] = (T)v[u];
        }
    }
}

// out = base (or 0) + sigma * (A in) (adj = 0) or sigma * (A^T in) (adj = 1).
template <typename T>
DEVI void f_apply(const Tables& tb, const InstDesc& d, int adj, T* o, const T* src, const T* bs,
                  double sigma, int kc, unsigned char* smem) {
    f_identity<T>(tb, d, adj, o, src, bs, adj ? d.n : d.m, sigma);
    constexpr int R = ConvCfg<T>::R;
    const int tid = threadIdx.x;
    for (int c = d.cb0; c < d.cb1; ++c) {
        const ConvBlock cb = tb.cblk[c];
        const int64_t n_out = adj ? cb.n_in : cb.n_in + cb.k - 1;
        T* ob = o + (adj ? cb.col0 : cb.row0);
        const T* ib = src + (adj ? cb.row0 : cb.col0);
        const double s = sigma * cb.scale;
        for (int64_t ot = 0; ot < n_out; ot += (int64_t)FNT * R) {
            T acc[R];
            conv_sums<T, FNT>(cb, adj, ib, ot, kc, smem, acc);   // (its first barrier orders o's writes)
            T ov[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int64_t oi = ot + (int64_t)tid * R + r;
                ov[r] = oi < n_out ? ob[oi] : T(0);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int64_t oi = ot + (int64_t)tid * R + r;
                if (oi < n_out) ob[oi] = (T)((double)ov[r] + s * (double)acc[r]);
            }
        }
    }
    __syncthreads();
    for (int q = d.db0; q < d.db1; ++q) {
        dense_rows<T>(tb.dblk[q], adj, o, src, sigma);
        __syncthreads();
    }
}

// The scalars a fused launch leaves (one thread calls these)
DEVI void record_check(gptr<double> sc, const CheckOut& co) {
    sc[SC_CUX] = co.cux;
    sc[SC_BUY] = co.buy;
    sc[SC_RP] = co.rp;
    sc[SC_RD] = co.rd;
    sc[SC_GAP] = co.gap;
    sc[SC_CX] = co.cx;
    sc[SC_BY] = co.by;
}
DEVI void record_state(gptr<double> sc, const FusedArgs& fa, double tau, double kap, double ut, double iter,
                       double cgtot, double cgmax, double status) {
    sc[SC_TAU] = tau;
    sc[SC_KAPPA] = kap;
    sc[SC_UT] = ut;
    sc[SC_ITER] = iter;
    sc[SC_CGTOT] = cgtot;
    if (fa.check) {
        sc[SC_CGMAXLAST] = cgmax;
        sc[SC_CGMAX] = 0.0;
    } else {
        sc[SC_CGMAX] = cgmax;
    }
    if (status != 0.0) {
        sc[SC_STATUS] = status;
        sc[SC_ACTIVE] = 0.0;
    }
}

// ---------------------------------------------------------------- register form
// The whole-step kernel for the common small instance: one convolution block, no
// dense block, at most one second-order cone, at most two identity blocks to a row
// or column (InstDesc::fused = FUSED_REG + variant; the host checks, fused_reg_variant).
// The general form below is a chain of short passes over vectors in LDS, two barriers
// and a memory round trip each: 13 barriers per CG iteration, window and taps staged
// for every product, the blocks' records read again.  Here thread t owns the elements
// t + FNT j of every vector, as in the general form's passes, and keeps the CG state
// (z, r, p, K z, A z) of them in registers.  LDS holds only what a product reads across
// threads: its input, with zeros around it in place of a staged window, and the
// convolution's sums, which pass to the elements' owners there.  The identity blocks
// that reach an element are looked up once per launch; the taps are uniform scalar
// loads.  Six barriers per CG iteration.  A launch may span several check intervals:
// the test ends an instance inside it.  Arithmetic and order of every sum are those of
// the general form: identical results.

// Dynamic LDS behind the form's own: the cone's tail partials (static LDS the general form
// would lose as well)
constexpr int REG_SCRATCH = FNT * (int)sizeof(double);

template <typename T> using cptr = const __attribute__((address_space(4))) T*;

// N sums over the workgroup, each in the order of bsum, with one barrier; sh: two
// buffers of 6 * FNT / 64, used in turn (a buffer is written again only after the next
// sum's barrier)
template <int N>
DEVI void rsum(double (&s)[N], double* sh, int& turn) {
    constexpr int NWV = FNT / 64;
    double* b = sh + turn * 6 * NWV;
    turn ^= 1;
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const double t = wave_sum(s[j]);
        if ((threadIdx.x & 63) == 0) b[j * NWV + w] = t;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < N; ++j) {
        double r = 0.0;
#pragma unroll
        for (int i = 0; i < NWV; ++i) r += b[j * NWV + i];
        s[j] = r;
    }
}

// acc[r] = sum over kpad taps, in order, of w[t] in[r + t] (in: LDS, the thread's first
// output); eight taps a step, the next step's values and taps fetched ahead of the
// current one's sums
template <typename T, int R>
DEVI void reg_conv(T (&acc)[R], const T* in, cptr<T> w, int kpad) {
    constexpr int U = 8;
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = T(0);
    T c[R], xa[U], xb[U], ta[U], te[U];
    auto fetch = [&](int t, T (&v)[U], T (&tv)[U]) {
#pragma unroll
        for (int j = 0; j < U; ++j) v[j] = in[t + R + j];
#pragma unroll
        for (int j = 0; j < U; ++j) tv[j] = w[t + j];
    };
    auto step = [&](const T (&v)[U], const T (&tv)[U]) {
#pragma unroll
        for (int t = 0; t < U; ++t)
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] = fma(tv[t], r + t < R ? c[(r + t) % R] : v[(r + t - R + U) % U], acc[r]);
        T n[R];
#pragma unroll
        for (int j = 0; j < R; ++j) n[j] = U + j < R ? c[(U + j) % R] : v[(U - R + j + U) % U];
#pragma unroll
        for (int j = 0; j < R; ++j) c[j] = n[j];
    };
#pragma unroll
    for (int j = 0; j < R; ++j) c[j] = in[j];
    const int nu = kpad / U;
    if (nu > 0) fetch(0, xa, ta);
    for (int u = 0; u + 1 < nu; u += 2) {
        fetch((u + 1) * U, xb, te);
        __builtin_amdgcn_sched_barrier(0);
        step(xa, ta);
        fetch((u + 2 < nu ? u + 2 : u) * U, xa, ta);
        __builtin_amdgcn_sched_barrier(0);
        step(xb, te);
    }
    if (nu & 1) step(xa, ta);
    for (int t = nu * U; t < kpad; t += 4) {   // (kpad is a multiple of 4)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const T tv = w[t + j];
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] = fma(tv, in[t + j + r], acc[r]);
        }
    }
}

// LDS elements: the input of A with k - 1 zeros ahead of it, the input of A^T, both
// followed by zeros up to where the last wave's outputs read; the convolution's sums;
// the other columns and rows
struct RegLds {
    int xi, yi, cs, xo, yo, total;   // offsets, elements
};
__host__ __device__ inline RegLds reg_lds(int n, int m, int n_in, int k, int kpad, int R) {
    RegLds l;
    const int no = n_in + k - 1, slack = 64 * R + kpad + 16;
    l.xi = 0;
    l.yi = no + slack;
    l.cs = l.yi + no + slack;
    l.xo = l.cs + no;
    l.yo = l.xo + n - n_in;
    l.total = (l.yo + m - no + 3) & ~3;
    return l;
}

// R: convolution outputs per thread; NX, NY: a thread's most elements of an X / Y vector
template <typename T, int R, int NX, int NY>
DEVI void fused_reg(const Tables& tb, const FusedArgs& fa, const InstDesc& d, T* lds, double* sh, double* idw,
                    double* tails) {
    gptr<double> sc = scal(d);
    const int tid = threadIdx.x;
    const ConvBlock& cbr = tb.cblk[d.cb0];
    const int n = (int)d.n, m = (int)d.m, n_in = (int)cbr.n_in, k = (int)cbr.k, kpad = (int)cbr.kpad;
    const int col0 = (int)cbr.col0, row0 = (int)cbr.row0, no = n_in + k - 1;
    const double cscale = cbr.scale;
    cptr<T> wf = (cptr<T>)cbr.w_fwd, wa = (cptr<T>)cbr.w_adj;
    const RegLds L = reg_lds(n, m, n_in, k, kpad, R);
    const int wave0 = __builtin_amdgcn_readfirstlane(tid & ~63) * R;   // the wave's first output
    // f(slot, index) for the thread's elements.  The thread's number is opaque to the
    // compiler each time: it would otherwise keep every element's addresses in
    // registers for the whole launch (and spill).
    auto opaque_tid = [&]() {
        int t = tid;
        asm volatile("" : "+v"(t));
        return t;
    };
    auto each_x = [&](auto f) {
        const int t = opaque_tid();
#pragma unroll
        for (int q = 0; q < NX; ++q)
            if (q * FNT < n && t + q * FNT < n) f(q, t + q * FNT);
    };
    auto each_y = [&](auto f) {
        const int t = opaque_tid();
#pragma unroll
        for (int q = 0; q < NY; ++q)
            if (q * FNT < m && t + q * FNT < m) f(q, t + q * FNT);
    };
    // LDS offset of an element of a product's input
    auto x_at = [&](int c) { return c >= col0 && c < col0 + n_in ? L.xi + k - 1 + c - col0 : L.xo + (c < col0 ? c : c - n_in); };
    auto y_at = [&](int r) { return r >= row0 && r < row0 + no ? L.yi + r - row0 : L.yo + (r < row0 ? r : r - no); };

    for (int i = tid; i < L.total; i += FNT) lds[i] = T(0);
    // the identity blocks that reach an element, in table order: LDS offset of the
    // input and block, one word each (-1: none)
    int xh[NX][2], yh[NY][2];
#pragma unroll
    for (int s = 0; s < NX; ++s) xh[s][0] = xh[s][1] = -1;
#pragma unroll
    for (int s = 0; s < NY; ++s) yh[s][0] = yh[s][1] = -1;
    for (int b = d.id0; b < d.id1; ++b) {
        const IdBlock ib = tb.ids[b];
        const int r0 = (int)ib.row0, c0 = (int)ib.col0, ln = (int)ib.len, j = b - d.id0;
        if (tid == 0) idw[j] = ib.scale;
        each_x([&](int s, int i) {
            if (i < c0 || i >= c0 + ln) return;
            const int h = y_at(i - c0 + r0) | (j << 24);
            if (xh[s][0] < 0) xh[s][0] = h;
            else xh[s][1] = h;
        });
        each_y([&](int s, int i) {
            if (i < r0 || i >= r0 + ln) return;
            const int h = x_at(i - r0 + c0) | (j << 24);
            if (yh[s][0] < 0) yh[s][0] = h;
            else yh[s][1] = h;
        });
    }
    auto id_add = [&](const int (&h)[2], double sigma, double v) {
#pragma unroll
        for (int e = 0; e < 2; ++e)
            if (h[e] >= 0) v += sigma * idw[h[e] >> 24] * (double)lds[h[e] & 0xffffff];
        return v;
    };
    // the step's vectors, in LDS where they fit (in this order), else in the region
    T* vec[7];
    constexpr int kinds[7] = {NXV + YU, NXV + YV, XU, NXV + YG, XG, NXV + YB, XC};
    int resident = 0;
    {
        int64_t at = L.total;
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            const int v = kinds[j];
            const int64_t len = ((v < NXV ? n : m) + 3) & ~3;
            vec[j] = v < NXV ? (T*)xvec<T>(d, v) : (T*)yvec<T>(d, v - NXV);
            if ((at + len) * (int64_t)sizeof(T) <= fa.lds_reg) {
                const T* g = vec[j];
                T* to = lds + at;
                vec[j] = to;
                at += len;
                resident |= 1 << j;
                if (v < NXV) each_x([&](int, int i) { to[i] = g[i]; });
                else each_y([&](int, int i) { to[i] = g[i]; });
            }
        }
    }
    T *uy = vec[0], *vs = vec[1], *ux = vec[2];
    const T *gy = vec[3], *gx = vec[4], *by = vec[5], *cx = vec[6];
    T z[NX], kz[NX], rx[NX], px[NX], az[NY], ty[NY];
    each_x([&](int s, int i) {
        z[s] = xvec<T>(d, XZ)[i];
        kz[s] = xvec<T>(d, XK)[i];
    });
    each_y([&](int s, int i) { az[s] = yvec<T>(d, YA)[i]; });
    double tau = sc[SC_TAU], kap = sc[SC_KAPPA], ut = sc[SC_UT];
    const double eta = sc[SC_ETA], al = fa.alpha;
    double iter = sc[SC_ITER], cgtot = sc[SC_CGTOT], cgmax = sc[SC_CGMAX];
    int turn = 0;
    const bool soc = d.sg1 > d.sg0;
    const int s0 = soc ? (int)tb.seg[d.sg0].start : m;   // (the cone takes the rows from s0 on)
    const int l = (int)d.l;
    __syncthreads();

    // the sums of A (adj = 0) or A^T over the product's input in LDS, into L.cs
    auto sums = [&](int adj) {
        const int nout = adj ? n_in : no;
        if (wave0 < nout) {
            T acc[R];
            reg_conv<T, R>(acc, lds + (adj ? L.yi : L.xi) + tid * R, adj ? wa : wf, kpad);
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (tid * R + r < nout) lds[L.cs + tid * R + r] = acc[r];
        }
        __syncthreads();
    };
    // out[s] = identity terms + convolution, for the thread's rows
    auto apply_a = [&](T (&out)[NY]) {
        sums(0);
        each_y([&](int s, int i) {
            T o = (T)id_add(yh[s], 1.0, 0.0);
            if (i >= row0 && i < row0 + no) o = (T)((double)o + cscale * (double)lds[L.cs + i - row0]);
            out[s] = o;
        });
    };
    // out[s] = base(s, i) + sigma (identity terms + convolution), for the thread's columns
    auto apply_at = [&](T (&out)[NX], double sigma, auto base) {
        sums(1);
        const double cs = sigma * cscale;
        each_x([&](int s, int i) {
            T o = (T)id_add(xh[s], sigma, base(s, i));
            if (i >= col0 && i < col0 + n_in) o = (T)((double)o + cs * (double)lds[L.cs + i - col0]);
            out[s] = o;
        });
    };

    double status = 0.0;
    for (int step = 0; step < fa.nsteps; ++step) {
        // w_y = u_y + v_s; h = u_x - A^T w_y; r = h - K z, p = r
        each_y([&](int, int i) { lds[y_at(i)] = (T)((double)uy[i] + (double)vs[i]); });
        __syncthreads();
        T q[NX];
        apply_at(q, -1.0, [&](int, int i) { return (double)ux[i]; });
        double s2[2] = {0.0, 0.0};   // ||r||^2, ||h||^2
        each_x([&](int s, int i) {
            const double hi = (double)q[s];
            const T ri = (T)(hi - (double)kz[s]);
            rx[s] = px[s] = ri;
            lds[x_at(i)] = ri;
            s2[0] = fma((double)ri, (double)ri, s2[0]);
            s2[1] = fma(hi, hi, s2[1]);
        });
        rsum<2>(s2, sh, turn);
        double rr = s2[0];
        double rel = fa.zeta > 0.0 ? fa.zeta / pow(iter + 1.0, fa.rate) : 0.0;
        rel = rel > fa.floor_ ? rel : fa.floor_;
        const double tol = sqrt(s2[1]) * rel;
        int cgit = 0;
        bool act = fa.cg_max > 0 && std::isfinite(rr) && sqrt(rr) > tol;
        while (act) {
            apply_a(ty);   // A p
            each_y([&](int s, int i) { lds[y_at(i)] = ty[s]; });
            __syncthreads();
            apply_at(q, 1.0, [&](int s, int) { return (double)px[s]; });   // q = p + A^T A p
            double pq[1] = {0.0};
            each_x([&](int s, int) { pq[0] = fma((double)px[s], (double)q[s], pq[0]); });
            rsum<1>(pq, sh, turn);
            const double a = rr / pq[0];
            if (!(pq[0] > 0.0 && std::isfinite(a))) break;
            double rn[1] = {0.0};
            each_x([&](int s, int) {
                const double qi = (double)q[s];
                z[s] = (T)fma(a, (double)px[s], (double)z[s]);
                const T ri = (T)fma(-a, qi, (double)rx[s]);
                rx[s] = ri;
                kz[s] = (T)fma(a, qi, (double)kz[s]);
                rn[0] = fma((double)ri, (double)ri, rn[0]);
            });
            each_y([&](int s, int) { az[s] = (T)fma(a, (double)ty[s], (double)az[s]); });
            rsum<1>(rn, sh, turn);
            const double be = rr > 0.0 ? rn[0] / rr : 0.0;
            rr = rn[0];
            ++cgit;
            cgtot += 1.0;
            act = std::isfinite(rr) && sqrt(rr) > tol && cgit < fa.cg_max;
            if (act) {
                each_x([&](int s, int i) {
                    px[s] = (T)fma(be, (double)px[s], (double)rx[s]);
                    lds[x_at(i)] = px[s];
                });
                __syncthreads();
            }
        }
        if (cgit > cgmax) cgmax = cgit;
        // z_y = w_y + A z; u~_tau = (tau + kappa + c^T z_x + b^T z_y) / eta
        double s3[2] = {0.0, 0.0};
        each_x([&](int s, int i) { s3[0] = fma((double)cx[i], (double)z[s], s3[0]); });
        each_y([&](int s, int i) {
            ty[s] = z_y<T>(uy[i], vs[i], az[s]);
            s3[1] = fma((double)by[i], (double)ty[s], s3[1]);
        });
        rsum<2>(s3, sh, turn);
        ut = (tau + kap + s3[0] + s3[1]) / eta;
        const double ubar = al * ut + (1.0 - al) * tau;
        const double tnew = ubar - kap > 0.0 ? ubar - kap : 0.0;
        kap = kap - ubar + tnew;
        tau = tnew;
        iter += 1.0;
        // u_bar_y - v_s; the cone's head and tail norm (the general form sums the tail
        // from its first entry on, thread (y - s0 - 1) % FNT: the partials change lanes)
        auto pv_of = [&](int s, int i) {
            const double ut_y = (double)ty[s] - ut * (double)gy[i];
            const double ub = al * ut_y + (1.0 - al) * (double)uy[i];
            return ub - (double)vs[i];
        };
        double nz = 0.0, aa = 0.0;
        int mode = 0;
        if (soc) {
            double s4[1] = {0.0};
            each_y([&](int s, int i) {
                if (i < s0) return;
                const double pv = pv_of(s, i);
                if (i == s0) sh[2 * 6 * (FNT / 64)] = pv;
                else s4[0] = fma(pv, pv, s4[0]);
            });
            tails[(tid - s0 - 1) & (FNT - 1)] = s4[0];
            __syncthreads();
            const double t = sh[2 * 6 * (FNT / 64)];
            s4[0] = tails[tid];
            rsum<1>(s4, sh, turn);
            nz = sqrt(s4[0]);
            if (nz <= t) mode = 0;
            else if (nz <= -t) mode = 1;
            else {
                mode = 2;
                aa = 0.5 * (t + nz);
            }
        }
        // relaxation, projection, dual update
        each_x([&](int s, int i) {
            ux[i] = (T)(al * ((double)z[s] - ut * (double)gx[i]) + (1.0 - al) * (double)ux[i]);
        });
        each_y([&](int s, int i) {
            const double pv = pv_of(s, i);
            double pr;
            if (i < l) pr = pv > 0.0 ? pv : 0.0;
            else if (mode == 0) pr = pv;
            else if (mode == 1) pr = 0.0;
            else pr = i == s0 ? aa : (aa / nz) * pv;
            uy[i] = (T)pr;
            vs[i] = (T)(pr - pv);
        });
        if (!fa.check || ((step + 1) % fa.check_every != 0 && step + 1 != fa.nsteps)) continue;
        // termination test
        each_x([&](int, int i) { lds[x_at(i)] = ux[i]; });
        __syncthreads();
        apply_a(ty);   // A u_x
        each_y([&](int, int i) { lds[y_at(i)] = uy[i]; });
        __syncthreads();
        apply_at(q, 1.0, [](int, int) { return 0.0; });   // A^T u_y
        double r6[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};   // Y: 0-2, X: 3-5
        gptr<const T> dr = yvec<T>(d, YD), ec = xvec<T>(d, XE);
        each_y([&](int s, int i) {
            const double w = 1.0 / (double)dr[i];
            const double e = ((double)ty[s] + (double)vs[i]) * w;
            const double rp = e - tau * (double)by[i] * w;
            r6[0] = fma(rp, rp, r6[0]);
            r6[1] = fma(e, e, r6[1]);
            r6[2] = fma((double)by[i], (double)uy[i], r6[2]);
        });
        each_x([&](int s, int i) {
            const double w = 1.0 / (double)ec[i];
            const double e = (double)q[s] * w;
            const double rd = e + tau * (double)cx[i] * w;
            r6[3] = fma(rd, rd, r6[3]);
            r6[4] = fma(e, e, r6[4]);
            r6[5] = fma((double)cx[i], (double)ux[i], r6[5]);
        });
        rsum<6>(r6, sh, turn);
        const CheckOut co = check_outcome(sc, tau, kap, iter, r6[0], r6[1], r6[2], r6[3], r6[4], r6[5], fa.eps,
                                          fa.max_iters);
        status = co.status;
        if (tid == 0) record_check(sc, co);
        if (status != 0.0) break;
        // exact recomputation of the carried products of the warm start
        each_x([&](int s, int i) { lds[x_at(i)] = z[s]; });
        __syncthreads();
        apply_a(az);
        each_y([&](int s, int i) { lds[y_at(i)] = az[s]; });
        __syncthreads();
        apply_at(kz, 1.0, [&](int s, int) { return (double)z[s]; });
        __syncthreads();
    }
    each_x([&](int s, int i) {
        xvec<T>(d, XZ)[i] = z[s];
        xvec<T>(d, XK)[i] = kz[s];
        if ((resident >> 2) & 1) xvec<T>(d, XU)[i] = ux[i];
    });
    each_y([&](int s, int i) {
        yvec<T>(d, YA)[i] = az[s];
        if (resident & 1) yvec<T>(d, YU)[i] = uy[i];
        if (resident & 2) yvec<T>(d, YV)[i] = vs[i];
    });
    if (tid == 0) record_state(sc, fa, tau, kap, ut, iter, cgtot, cgmax, status);
}

template <typename T>
__global__ __launch_bounds__(FNT) void k_fused(Tables tb, FusedArgs fa) {
    extern __shared__ __align__(16) unsigned char fsmem[];
    __shared__ double sh[2 * 6 * (FNT / 64) + 1];   // (register form: sums, cone head)
    __shared__ double idw[FUSED_REG_IDS];
    static_assert(sizeof sh + sizeof idw <= FUSED_STATIC_LDS, "declared LDS");
    const InstDesc d = tb.inst[blockIdx.x];
    gptr<double> sc = scal(d);
    if (!(sc[SC_ACTIVE] != 0.0 && sc[SC_PHASE] == 2.0)) return;
    if (d.fused >= FUSED_REG && !fa.refresh) {
        T* lds = reinterpret_cast<T*>(fsmem);
        double* tails = reinterpret_cast<double*>(fsmem + fa.lds_reg);
        switch (d.fused - FUSED_REG) {
#define CGS_REG(V) \
    case V: fused_reg<T, kRegVariants[V].r, kRegVariants[V].nx, kRegVariants[V].ny>(tb, fa, d, lds, sh, idw, tails); break
            CGS_REG(0);
            CGS_REG(1);
            CGS_REG(2);
            CGS_REG(3);
            CGS_REG(4);
#undef CGS_REG
            default:
                if constexpr (sizeof(T) == 4)
                    fused_reg<T, kRegVariants[5].r, kRegVariants[5].nx, kRegVariants[5].ny>(tb, fa, d, lds, sh, idw, tails);
        }
        return;
    }
    FVecs<T> fv;
#pragma unroll
    for (int k = 0; k < NXV; ++k) fv.x[k] = (T*)xvec<T>(d, k);
#pragma unroll
    for (int k = 0; k < NYV; ++k) fv.y[k] = (T*)yvec<T>(d, k);
    fv.res = 0u;
    if (fa.refresh) {
        // the same applies as the exact recomputation at a check, so that a
        // refresh between checks leaves the carried products bitwise unchanged
        f_apply<T>(tb, d, 0, fv.y[YA], fv.x[XZ], nullptr, 1.0, fa.kc, fsmem);
        f_apply<T>(tb, d, 1, fv.x[XK], fv.y[YA], fv.x[XZ], 1.0, fa.kc, fsmem);
        return;
    }
    {
        // LDS past the convolution's staging area, vector by vector in the
        // order of kResident while they fit
        unsigned char* p = fsmem + fa.lds_conv;
        int64_t left = fa.lds_res;
#pragma unroll
        for (int j = 0; j < kNumResident; ++j) {
            const int v = kResident[j];
            const int64_t bytes = (((v < NXV ? d.n : d.m) * (int64_t)sizeof(T)) + 15) & ~int64_t(15);
            if (bytes <= left) {
                fv_slot(fv, v) = reinterpret_cast<T*>(p);
                p += bytes;
                left -= bytes;
                fv.res |= 1u << j;
            }
        }
        fv_copy<T>(d, fv, true);
    }
    const int tid = threadIdx.x;
    const int64_t n = d.n, m = d.m;
    double tau = sc[SC_TAU], kap = sc[SC_KAPPA], ut = sc[SC_UT];
    const double eta = sc[SC_ETA];
    double iter = sc[SC_ITER], cgtot = sc[SC_CGTOT], cgmax = sc[SC_CGMAX];
    T *ux = fv.x[XU], *zx = fv.x[XZ], *rx = fv.x[XR], *px = fv.x[XP];
    T *qx = fv.x[XQ], *hx = fv.x[XH], *kz = fv.x[XK];
    const T *gx = fv.x[XG], *cx = fv.x[XC];
    T *uy = fv.y[YU], *vs = fv.y[YV], *wy = fv.y[YW], *zy = fv.y[YZ];
    T *ty = fv.y[YT], *az = fv.y[YA];
    const T *by = fv.y[YB], *gy = fv.y[YG];
    const double al = fa.alpha;

    for (int step = 0; step < fa.nsteps; ++step) {
        // w_y = u_y + v_s; h = u_x - A^T w_y
        struct V2 { T a, b; };
        ew<V2>(m, [&](V2& r, int i) { r.a = uy[i]; r.b = vs[i]; },
               [&](V2& r, int i) { wy[i] = (T)((double)r.a + (double)r.b); });
        __syncthreads();
        f_apply<T>(tb, d, 1, hx, wy, ux, -1.0, fa.kc, fsmem);
        // CG on (I + A^T A) z = h from the warm start (carried K z, A z)
        double s2[2] = {0.0, 0.0};   // ||r||^2, ||h||^2
        ew<V2>(n, [&](V2& r, int i) { r.a = hx[i]; r.b = kz[i]; },
               [&](V2& r, int i) {
                   const double hi = (double)r.a;
                   const T ri = (T)(hi - (double)r.b);
                   rx[i] = ri;
                   px[i] = ri;
                   s2[0] = fma((double)ri, (double)ri, s2[0]);
                   s2[1] = fma(hi, hi, s2[1]);
               });
        block_sumN<FNT, 2>(s2, sh);
        double rr = s2[0];
        const double hh = s2[1];
        double rel = fa.zeta > 0.0 ? fa.zeta / pow(iter + 1.0, fa.rate) : 0.0;
        rel = rel > fa.floor_ ? rel : fa.floor_;
        const double tol = sqrt(hh) * rel;
        int cgit = 0;
        bool act = fa.cg_max > 0 && std::isfinite(rr) && sqrt(rr) > tol;
        while (act) {
            f_apply<T>(tb, d, 0, ty, px, nullptr, 1.0, fa.kc, fsmem);   // A p
            f_apply<T>(tb, d, 1, qx, ty, px, 1.0, fa.kc, fsmem);        // q = p + A^T A p
            double pq = 0.0;
            ew<V2>(n, [&](V2& r, int i) { r.a = px[i]; r.b = qx[i]; },
                   [&](V2& r, int i) { pq = fma((double)r.a, (double)r.b, pq); });
            pq = bsum(pq, sh);
            const double a = rr / pq;
            if (!(pq > 0.0 && std::isfinite(a))) break;
            double rn = 0.0;
            struct V5 { T q, p, z, r, k; };
            ew<V5>(n, [&](V5& r, int i) { r.q = qx[i]; r.p = px[i]; r.z = zx[i]; r.r = rx[i]; r.k = kz[i]; },
                   [&](V5& r, int i) {
                       const double qi = (double)r.q;
                       zx[i] = (T)fma(a, (double)r.p, (double)r.z);
                       const T ri = (T)fma(-a, qi, (double)r.r);
                       rx[i] = ri;
                       kz[i] = (T)fma(a, qi, (double)r.k);
                       rn = fma((double)ri, (double)ri, rn);
                   });
            ew<V2>(m, [&](V2& r, int i) { r.a = ty[i]; r.b = az[i]; },
                   [&](V2& r, int i) { az[i] = (T)fma(a, (double)r.a, (double)r.b); });
            rn = bsum(rn, sh);
            const double be = rr > 0.0 ? rn / rr : 0.0;
            rr = rn;
            ++cgit;
            cgtot += 1.0;
            act = std::isfinite(rr) && sqrt(rr) > tol && cgit < fa.cg_max;
            if (act)
                ew<V2>(n, [&](V2& r, int i) { r.a = px[i]; r.b = rx[i]; },
                       [&](V2& r, int i) { px[i] = (T)fma(be, (double)r.a, (double)r.b); });
            __syncthreads();
        }
        if (cgit > cgmax) cgmax = cgit;
        // z_y = w_y + A z; u~_tau = (tau + kappa + c^T z_x + b^T z_y) / eta
        double s3[2] = {0.0, 0.0};   // c^T z_x, b^T z_y
        ew<V2>(n, [&](V2& r, int i) { r.a = cx[i]; r.b = zx[i]; },
               [&](V2& r, int i) { s3[0] = fma((double)r.a, (double)r.b, s3[0]); });
        struct V3 { T w, a, b; };
        ew<V3>(m, [&](V3& r, int i) { r.w = wy[i]; r.a = az[i]; r.b = by[i]; },
               [&](V3& r, int i) {
                   const T zv = (T)((double)r.w + (double)r.a);
                   zy[i] = zv;
                   s3[1] = fma((double)r.b, (double)zv, s3[1]);
               });
        block_sumN<FNT, 2>(s3, sh);
        const double cz = s3[0], bz = s3[1];
        ut = (tau + kap + cz + bz) / eta;
        const double ubar = al * ut + (1.0 - al) * tau;
        const double tnew = ubar - kap > 0.0 ? ubar - kap : 0.0;
        kap = kap - ubar + tnew;
        tau = tnew;
        iter += 1.0;
        // relaxed point minus v_s of Y entry i, from its u_y, z_y, g_y, v_s
        struct V4 { T u, z, g, v; };
        auto ld4y = [&](V4& r, int i) { r.u = uy[i]; r.z = zy[i]; r.g = gy[i]; r.v = vs[i]; };
        auto pv_of = [&](const V4& r) {
            const double ut_y = (double)r.z - ut * (double)r.g;
            const double ub = al * ut_y + (1.0 - al) * (double)r.u;
            return ub - (double)r.v;
        };
        // second-order cones: head and tail norm of u_bar_y - v_s
        for (int sgi = d.sg0; sgi < d.sg1; ++sgi) {
            const SocSeg sg = tb.seg[sgi];
            double ss = 0.0;
            ew<V4>(sg.len - 1, [&](V4& r, int i) { ld4y(r, sg.start + 1 + i); },
                   [&](V4& r, int) {
                       const double pv = pv_of(r);
                       ss = fma(pv, pv, ss);
                   });
            ss = bsum(ss, sh);
            if (tid == 0) {
                V4 r;
                ld4y(r, sg.start);
                tb.seg_val[2 * sgi] = pv_of(r);
                tb.seg_val[2 * sgi + 1] = ss;
            }
        }
        __syncthreads();
        // relaxation, projection, dual update
        struct V3x { T z, g, u; };
        ew<V3x>(n, [&](V3x& r, int i) { r.z = zx[i]; r.g = gx[i]; r.u = ux[i]; },
                [&](V3x& r, int i) {
                    ux[i] = (T)(al * ((double)r.z - ut * (double)r.g) + (1.0 - al) * (double)r.u);
                });
        ew<V4>(d.l, ld4y, [&](V4& r, int i) {
            const double pv = pv_of(r);
            const double pr = pv > 0.0 ? pv : 0.0;
            uy[i] = (T)pr;
            vs[i] = (T)(pr - pv);
        });
        for (int sgi = d.sg0; sgi < d.sg1; ++sgi) {
            const SocSeg sg = tb.seg[sgi];
            const double t = tb.seg_val[2 * sgi];
            const double nz = sqrt(tb.seg_val[2 * sgi + 1]);
            int mode;
            double aa = 0.0;
            if (nz <= t) mode = 0;
            else if (nz <= -t) mode = 1;
            else {
                mode = 2;
                aa = 0.5 * (t + nz);
            }
            ew<V4>(sg.len, [&](V4& r, int i) { ld4y(r, sg.start + i); },
                   [&](V4& r, int i) {
                       const double pv = pv_of(r);
                       double pr;
                       if (mode == 0) pr = pv;
                       else if (mode == 1) pr = 0.0;
                       else pr = (i == 0) ? aa : (aa / nz) * pv;
                       uy[sg.start + i] = (T)pr;
                       vs[sg.start + i] = (T)(pr - pv);
                   });
        }
        __syncthreads();
    }

    double status = 0.0;
    if (fa.check) {
        f_apply<T>(tb, d, 0, ty, ux, nullptr, 1.0, fa.kc, fsmem);          // A u_x
        f_apply<T>(tb, d, 1, fv.x[XT], uy, nullptr, 1.0, fa.kc, fsmem);    // A^T u_y
        const T* aty = fv.x[XT];
        const T* dr = fv.y[YD];
        const T* ec = fv.x[XE];
        double r6[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};   // Y: 0-2, X: 3-5
        struct V5y { T d, t, v, b, u; };
        ew<V5y>(m, [&](V5y& r, int i) { r.d = dr[i]; r.t = ty[i]; r.v = vs[i]; r.b = by[i]; r.u = uy[i]; },
                [&](V5y& r, int) {
                    const double w = 1.0 / (double)r.d;
                    const double e = ((double)r.t + (double)r.v) * w;
                    const double rp = e - tau * (double)r.b * w;
                    r6[0] = fma(rp, rp, r6[0]);
                    r6[1] = fma(e, e, r6[1]);
                    r6[2] = fma((double)r.b, (double)r.u, r6[2]);
                });
        struct V4x { T e, a, c, u; };
        ew<V4x>(n, [&](V4x& r, int i) { r.e = ec[i]; r.a = aty[i]; r.c = cx[i]; r.u = ux[i]; },
                [&](V4x& r, int) {
                    const double w = 1.0 / (double)r.e;
                    const double e = (double)r.a * w;
                    const double rd = e + tau * (double)r.c * w;
                    r6[3] = fma(rd, rd, r6[3]);
                    r6[4] = fma(e, e, r6[4]);
                    r6[5] = fma((double)r.c, (double)r.u, r6[5]);
                });
        block_sumN<FNT, 6>(r6, sh);
        const double y0 = r6[0], y1 = r6[1], y2 = r6[2], x0 = r6[3], x1 = r6[4], x2 = r6[5];
        const CheckOut co = check_outcome(sc, tau, kap, iter, y0, y1, y2, x0, x1, x2, fa.eps,
                                          fa.max_iters);
        status = co.status;
        if (tid == 0) record_check(sc, co);
        if (status == 0.0) {
            // exact recomputation of the carried products of the warm start
            f_apply<T>(tb, d, 0, az, zx, nullptr, 1.0, fa.kc, fsmem);
            f_apply<T>(tb, d, 1, kz, az, zx, 1.0, fa.kc, fsmem);
        }
    }
    __syncthreads();
    fv_copy<T>(d, fv, false);
    if (tid == 0) record_state(sc, fa, tau, kap, ut, iter, cgtot, cgmax, status);
}

// The CG loop of the setup solve (z = g_x; r, p and the start test from k_cg_init) for
// FP64 instances of the register form whose X vector is one vector tile: one workgroup
// and one launch instead of four launches per iteration and a wait of the host after
// every eight.  Bound by the serial chain of the products (6 us an iteration at n = 1000,
// k = 101): a 60-step solve at that size 4.2 -> 3.6 ms.  Products as in fused_reg; the
// dot products and the update are those of k_cg_dot and k_cg_update, sum for sum
// (256 threads over the tile, ||r'||^2 from the expansion), so the result is theirs.
constexpr int DOT_NT = VEC_NT;
template <typename T, int R, int NX, int NY>
DEVI void setup_cg(const Tables& tb, const InstDesc& d, T* lds, double* sh, int cg_max) {
    gptr<double> sc = scal(d);
    const int tid = threadIdx.x;
    const ConvBlock& cbr = tb.cblk[d.cb0];
    const int n = (int)d.n, m = (int)d.m, n_in = (int)cbr.n_in, k = (int)cbr.k, kpad = (int)cbr.kpad;
    const int col0 = (int)cbr.col0, row0 = (int)cbr.row0, no = n_in + k - 1;
    const double cscale = cbr.scale;
    cptr<T> wf = (cptr<T>)cbr.w_fwd, wa = (cptr<T>)cbr.w_adj;
    const RegLds L = reg_lds(n, m, n_in, k, kpad, R);
    T *lq = lds + L.total, *lr = lq + n;   // q and r, for the dot products
    const int wave0 = __builtin_amdgcn_readfirstlane(tid & ~63) * R;
    auto each_x = [&](auto f) {
#pragma unroll
        for (int q = 0; q < NX; ++q)
            if (q * FNT < n && tid + q * FNT < n) f(q, tid + q * FNT);
    };
    auto x_at = [&](int c) { return c >= col0 && c < col0 + n_in ? L.xi + k - 1 + c - col0 : L.xo + (c < col0 ? c : c - n_in); };
    auto y_at = [&](int r) { return r >= row0 && r < row0 + no ? L.yi + r - row0 : L.yo + (r < row0 ? r : r - no); };
    for (int i = tid; i < L.total; i += FNT) lds[i] = T(0);
    __syncthreads();
    gptr<T> zv = xvec<T>(d, XG);
    T p[NX], r[NX], z[NX], q[NX];
    each_x([&](int s, int i) {
        z[s] = zv[i];
        r[s] = xvec<T>(d, XR)[i];
        p[s] = xvec<T>(d, XP)[i];
        lds[x_at(i)] = p[s];
        lr[i] = r[s];
    });
    __syncthreads();
    auto sums = [&](int adj) {
        const int nout = adj ? n_in : no;
        if (wave0 < nout) {
            T acc[R];
            reg_conv<T, R>(acc, lds + (adj ? L.yi : L.xi) + tid * R, adj ? wa : wf, kpad);
#pragma unroll
            for (int e = 0; e < R; ++e)
                if (tid * R + e < nout) lds[L.cs + tid * R + e] = acc[e];
        }
        __syncthreads();
    };
    // base + identity blocks (in table order) of row / column i, input `at` in LDS
    auto ids = [&](int adj, int i, double v) {
        for (int b = d.id0; b < d.id1; ++b) {
            const IdBlock ib = tb.ids[b];
            const int r0 = (int)(adj ? ib.col0 : ib.row0), c0 = (int)(adj ? ib.row0 : ib.col0);
            if (i >= r0 && i < r0 + (int)ib.len) {
                const int c = i - r0 + c0;
                v += ib.scale * (double)lds[adj ? y_at(c) : x_at(c)];
            }
        }
        return v;
    };
    const double tol = sc[SC_CGTOL];
    double cgit = 0.0, pq = 0.0, al = 0.0, be = 0.0, last = sc[SC_RR];
    bool more = true;
    for (int it = 0; more; ++it) {
        sums(0);
#pragma unroll
        for (int s = 0; s < NY; ++s) {
            const int i = tid + s * FNT;
            if (i >= m) break;
            double v = ids(0, i, 0.0);
            if (i >= row0 && i < row0 + no) v = v + cscale * (double)lds[L.cs + i - row0];
            lds[y_at(i)] = (T)v;
        }
        __syncthreads();
        sums(1);
        each_x([&](int s, int i) {
            double v = ids(1, i, (double)p[s]);
            if (i >= col0 && i < col0 + n_in) v = v + cscale * (double)lds[L.cs + i - col0];
            q[s] = (T)v;
            lq[i] = q[s];
        });
        __syncthreads();
        double s4[4] = {0.0, 0.0, 0.0, 0.0};
        if (tid < DOT_NT) {
            for (int i = tid; i < n; i += DOT_NT) {
                const double pi = (double)lds[x_at(i)], qi = (double)lq[i], ri = (double)lr[i];
                s4[0] = fma(pi, qi, s4[0]);
                s4[1] = fma(ri, ri, s4[1]);
                s4[2] = fma(ri, qi, s4[2]);
                s4[3] = fma(qi, qi, s4[3]);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double t = wave_sum(s4[j]);
                if ((tid & 63) == 0) sh[j * (DOT_NT / 64) + (tid >> 6)] = t;
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < DOT_NT / 64; ++w) t += sh[j * (DOT_NT / 64) + w];
            s4[j] = t;
        }
        pq = s4[0];
        const double rr = s4[1], rq = s4[2], qq = s4[3];
        al = rr / pq;
        const bool ok = pq > 0.0 && std::isfinite(al);
        const double rr1 = fma(al * al, qq, fma(-2.0 * al, rq, rr));
        be = rr > 0.0 ? rr1 / rr : 0.0;
        more = ok && std::isfinite(rr1) && sqrt(rr1) > tol && it + 1 < cg_max;
        last = ok ? rr1 : rr;
        if (ok) cgit += 1.0;
        else al = 0.0;
        each_x([&](int s, int i) {
            if (ok) z[s] = (T)fma(al, (double)p[s], (double)z[s]);
            if (more) {
                r[s] = (T)fma(-al, (double)q[s], (double)r[s]);
                p[s] = (T)fma(be, (double)p[s], (double)r[s]);
                lds[x_at(i)] = p[s];
                lr[i] = r[s];
            }
        });
        __syncthreads();
    }
    each_x([&](int s, int i) { zv[i] = z[s]; });
    if (tid == 0) {
        sc[SC_PQ] = pq;
        sc[SC_ALPHA] = al;
        sc[SC_RR] = last;
        sc[SC_BETA] = be;
        sc[SC_CGIT] += cgit;
        sc[SC_CGTOT] += cgit;
        sc[SC_SETUPIT] += cgit;
        if (sc[SC_CGIT] > sc[SC_CGMAX]) sc[SC_CGMAX] = sc[SC_CGIT];
        sc[SC_CGACT] = 0.0;
    }
}

__host__ __device__ int64_t setup_cg_bytes(const InstDesc& d, const ConvBlock& cb) {
    const int R = kRegVariants[d.fused - FUSED_REG].r;
    return (reg_lds((int)d.n, (int)d.m, (int)cb.n_in, (int)cb.k, (int)cb.kpad, R).total + 2 * d.n) *
           (int64_t)sizeof(double);
}

// lds: bytes of dynamic LDS of the launch (the need of the largest instance taken)
__global__ __launch_bounds__(FNT) void k_setup_cg(Tables tb, int cg_max, int64_t lds_bytes) {
    extern __shared__ __align__(16) unsigned char fsmem[];
    __shared__ double sh[4 * (DOT_NT / 64)];
    const InstDesc d = tb.inst[blockIdx.x];
    if (d.fused < FUSED_REG || !setup_cg_takes(d, tb.cblk[d.cb0], lds_bytes, cg_max) || !gate_ok(scal(d), G_SETUP_CG)) return;
    double* lds = reinterpret_cast<double*>(fsmem);
    switch (d.fused - FUSED_REG) {
#define CGS_SETUP(V) \
    case V: setup_cg<double, kRegVariants[V].r, kRegVariants[V].nx, kRegVariants[V].ny>(tb, d, lds, sh, cg_max); break
        CGS_SETUP(0);
        CGS_SETUP(1);
        CGS_SETUP(2);
        CGS_SETUP(3);
        CGS_SETUP(4);
#undef CGS_SETUP
        default: break;
    }
}

void launch_setup_cg(const Tables& t, int64_t lds, int cg_max, hipStream_t st) {
    if (t.ninst > 0) k_setup_cg<<<t.ninst, FNT, (size_t)lds, st>>>(t, cg_max, lds);
}

int64_t fused_reg_bytes(int prec, int64_t n, int64_t m, const ConvBlock& cb, int R, bool vectors) {
    const int64_t es = prec == 0 ? 8 : 4;
    int64_t e = reg_lds((int)n, (int)m, (int)cb.n_in, (int)cb.k, (int)cb.kpad, R).total;
    if (vectors) e += 3 * ((n + 3) & ~int64_t(3)) + 4 * ((m + 3) & ~int64_t(3));
    return REG_SCRATCH + ((e * es + 15) & ~int64_t(15));
}

size_t fused_smem_bytes(int prec, int kc) {
    const int R = prec == 0 ? CONV_R_F64 : CONV_R_F32;
    return (size_t)(FNT * R + 2 * kc + 2 * R) * (prec == 0 ? 8 : 4);
}

int64_t fused_resident_bytes(int prec, int64_t n, int64_t m) {
    const int64_t es = prec == 0 ? 8 : 4;
    int64_t b = 0;
    for (int j = 0; j < kNumResident; ++j)
        b += (((kResident[j] < NXV ? n : m) * es) + 15) & ~int64_t(15);
    return b;
}

// Dynamic LDS per workgroup that the fused kernels may take on each device (0: not yet queried)
static std::atomic<int> g_fused_lds[64];   // (zero-initialised: static storage)

// (the kernels' attributes belong to the calling thread's current device)
int fused_prepare(int dev) {
    if (dev < 0 || dev >= 64) return 65536 - FUSED_STATIC_LDS;
    if (g_fused_lds[dev].load() == 0) {
        int cur = dev;
        (void)hipGetDevice(&cur);
        if (cur != dev && hipSetDevice(dev) != hipSuccess) return 65536 - FUSED_STATIC_LDS;
        const int fixed = FUSED_STATIC_LDS;
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || v <= 0)
            v = 65536;
        int dyn = v - fixed;
        if (dyn > 65536 - fixed &&
            (hipFuncSetAttribute((const void*)k_fused<double>, hipFuncAttributeMaxDynamicSharedMemorySize, dyn) !=
                 hipSuccess ||
             hipFuncSetAttribute((const void*)k_fused<float>, hipFuncAttributeMaxDynamicSharedMemorySize, dyn) !=
                 hipSuccess ||
             hipFuncSetAttribute((const void*)k_setup_cg, hipFuncAttributeMaxDynamicSharedMemorySize, dyn) !=
                 hipSuccess))
            dyn = 65536 - fixed;
        g_fused_lds[dev].store(dyn);   // (two threads that get here store the same value)
        if (cur != dev) (void)hipSetDevice(cur);
    }
    return g_fused_lds[dev].load();
}

void launch_fused(int prec, const Tables& t, FusedArgs fa, int64_t lds_cap, hipStream_t st) {
    if (t.ninst <= 0) return;
    fa.lds_conv = ((int64_t)fused_smem_bytes(prec, fa.kc) + 15) & ~int64_t(15);
    if (!fa.general) fa.lds_conv = 0;
    fa.lds_res = std::max<int64_t>(0, std::min<int64_t>(fa.res_want, lds_cap - fa.lds_conv));
    const int64_t reg = std::min(std::max(fa.reg_want, fa.lds_conv + fa.lds_res), lds_cap);
    fa.lds_reg = (reg - REG_SCRATCH) & ~int64_t(15);
    const size_t lds = (size_t)std::max(fa.lds_conv + fa.lds_res, reg);
    if (prec == 0) k_fused<double><<<t.ninst, FNT, lds, st>>>(t, fa);
    else k_fused<float><<<t.ninst, FNT, lds, st>>>(t, fa);
}

}  // namespace cgs
