// HIP kernels of the structured-operator conic solver (gfx950 / CDNA4).
//
// Conventions
//  * One workgroup per tile of a tile table (see common.hpp).  Every tile lies
//    in one instance; a workgroup first reads its instance's gate flags and
//    leaves at once when the instance does not take part in this step.
//  * Reductions (dot products, norms) are deterministic: each workgroup folds
//    its tile in a fixed thread/wave order into FP64 partials, and a finalize
//    kernel (one workgroup per instance) sums the instance's partials in tile
//    order and finishes the scalar work (CG alpha and beta, tau/kappa,
//    residuals).  No atomics and no device-wide fences are used inside a
//    kernel (on a multi-XCD part a device-scope fence writes back and
//    invalidates the XCD's L2), so an instance's numbers do not depend on the
//    other instances of a launch.
//  * Vectors are in the working precision T (float or double); every scalar of
//    the method (tau, kappa, eta, CG alpha/beta, norms, residuals) is FP64.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <utility>
#include <vector>

#include "cgs.h"

#include <cmath>
#include <cstdint>

#include "kernels.hpp"
#include "device_common.hpp"

namespace cgs {

// ---------------------------------------------------------------- operator: identity part + base
template <typename T>
__global__ __launch_bounds__(VEC_NT) void k_apply_init(Tables tb, int adj, int out, int in, int base,
                                                       double sigma, int gate) {
    const VecTile tl = adj ? tb.xt[blockIdx.x] : tb.yt[blockIdx.x];
    const InstDesc d = tb.inst[tl.inst];
    if (!gate_ok(scal(d), gate)) return;
    init_tile<T>(tb, d, tl, adj, out, in, base, sigma, true);
}

// Direct convolution: one wave sums 64 R outputs, lane l the R ones from R l, over
// all taps in tap order (the order, and so the result, depends on neither R nor
// the form of the loop).  Two forms (conv_sub chooses):
//  * R = ConvCfg::R (conv_sums): each step of 2 R taps reads its window values and
//    taps from LDS; the other waves of the SIMD cover the reads.
//  * R half of that (NARROW), few tiles and long kernels: the launch is one wave's chain
//    over the taps (n = 3000, k = 1365 in FP64: 18 waves on the chip at R = 4, 25.2 us).
//    The window values of the next 16 taps are read while the current ones are summed,
//    and the taps, which as broadcast reads cost as much LDS time as the window,
//    travel in a register, 16 to a row of lanes, and reach the row's lanes through
//    DPP broadcasts: 17.4 us, bound by the latency of the dependent FP64 sums
//    (about 22 cycles a tap).
constexpr int CONV_U = 16;   // taps per step of the narrow form

// the row's lane N value in every lane of the row of 16 (the builtin's value has
// its operands' width, 64 bits for a double's, whatever type the front end states)
template <int N>
DEVI double row_bcast(double v) {
    const long x = __builtin_bit_cast(long, v);
    const long y = __builtin_amdgcn_update_dpp(x, x, 0x150 + N, 0xf, 0xf, true);
    return __builtin_bit_cast(double, y);
}
template <int N>
DEVI float row_bcast(float v) {
    const int x = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(x, x, 0x150 + N, 0xf, 0xf, true));
}
// acc[r] += tap t * x[r + t], t = 0..15 in order: x[0..R) in c, the rest in v, tap t
// in lane t of each row of tw; c becomes the R values the next 16 taps start with
template <typename T, int R, int... N>
DEVI void conv_row(T (&acc)[R], T (&c)[R], const T (&v)[CONV_U], T tw, std::integer_sequence<int, N...>) {
    auto one = [&](T tv, int t) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            acc[r] = fma(tv, r + t < R ? c[(r + t) % R] : v[(r + t - R + CONV_U) % CONV_U], acc[r]);
    };
    (one(row_bcast<N>(tw), N), ...);
#pragma unroll
    for (int j = 0; j < R; ++j) c[j] = v[CONV_U - R + j];
}

// (the waves a SIMD that the registers are held to, FP64 162 and 89, matter through the
// allocation alone: with no such bound the narrow form took 159 and ran 2 % slower, the wide
// one 87 and ran 4-9 % slower from k = 257 on; a bound of four or six costs 20 and 5 %)
template <typename T, int R>
__global__ __launch_bounds__(CONV_NT, R < ConvCfg<T>::R ? 3 : 5) void k_conv(Tables tb, ConvLaunch cl, int sub,
                                                  int parts, int adj, int out, int in, int base, double sigma, int gate) {
    extern __shared__ __align__(16) unsigned char conv_smem[];
    if ((int)blockIdx.x >= cl.ntiles * sub) {
        // initialisation tiles riding on the launch, in parts: a whole tile on one
        // wave is a chain of 12.5 us, longer than most launches of few tiles
        const int w = (int)blockIdx.x - cl.ntiles * sub, len = VEC_TILE / parts;
        VecTile it = cl.init[w / parts].tile();
        const int p0 = (w % parts) * len;
        if (p0 >= it.len) return;
        it.start += p0;
        it.len = it.len - p0 < len ? it.len - p0 : len;
        const InstDesc di = tb.inst[it.inst];
        // (four elements at a time: eight take 128 registers, the sums 87, FP32 65)
        if (gate_ok(scal(di), gate)) init_tile<T, 4>(tb, di, it, adj, out, in, base, sigma, false);
        return;
    }
    const int tix = (int)blockIdx.x / sub;
    const ConvTile tl = cl.tiles[tix];
    const InstDesc d = tb.inst[tl.inst];
    const ConvBlock cb = cl.blocks[tl.blk];
    if (!gate_ok(scal(d), gate)) return;
    constexpr int TILE = CONV_NT * R, U = CONV_U;
    constexpr bool NARROW = R < ConvCfg<T>::R;
    const int lane = threadIdx.x, li = lane * R;
    const int64_t ot = tl.start + (int64_t)((int)blockIdx.x - tix * sub) * TILE;
    const int64_t n_out = adj ? cb.n_in : cb.n_in + cb.k - 1;
    if (ot >= n_out) return;
    const int64_t n_in = adj ? cb.n_in + cb.k - 1 : cb.n_in;
    const int64_t off = adj ? 0 : -(cb.k - 1), g0 = adj ? cb.col0 : cb.row0;
    gptr<T> o = adj ? xvec<T>(d, out) + cb.col0 : yvec<T>(d, out) + cb.row0;
    gptr<const T> src = adj ? yvec<T>(d, in) + cb.row0 : xvec<T>(d, in) + cb.col0;
    gptr<const T> w = (gptr<const T>)(adj ? cb.w_adj : cb.w_fwd);
    const bool own = (cb.own >> adj) & 1;
    const int no = n_out - ot - li < R ? (int)(n_out - ot - li) : R;   // the lane's outputs (<= 0: none)
    const double s = sigma * cb.scale;
    // what the lane's outputs r0 .. r0 + 3 (of fewer, all) hold besides the sums
    constexpr int NH = R < 4 ? R : 4;
    auto held = [&](int r0, double (&ov)[NH]) {
        if (own) {
            owned_init_n<T, NH>(d, tb.ids, adj, in, base, sigma, g0 + ot + li + r0, no - r0, ov);
        } else {
#pragma unroll
            for (int r = 0; r < NH; ++r) ov[r] = r < no - r0 ? (double)o[ot + li + r0 + r] : 0.0;
        }
    };
    auto write = [&](int r0, const double (&ov)[NH], const T (&acc)[R]) {
#pragma unroll
        for (int r = 0; r < NH; ++r)
            if (r < no - r0) o[ot + li + r0 + r] = (T)(ov[r] + s * (double)acc[r0 + r]);
    };
    T acc[R];
    if constexpr (NARROW) {
        T* taps = reinterpret_cast<T*>(conv_smem);   // kc entries
        T* win = taps + cl.kc;                       // TILE + kc entries
        static_assert(R <= 4, "one piece of outputs");
        double ov[NH];
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] = T(0);
        for (int64_t t0 = 0; t0 < cb.kpad; t0 += cl.kc) {
            const int kc = (int)((cb.kpad - t0) < cl.kc ? (cb.kpad - t0) : cl.kc);
            const int nwin = TILE + kc;
            // the window's positions [qlo, qhi) lie inside the block's inputs
            const int64_t i0 = ot + off + t0;
            const int qlo = i0 < 0 ? (int)-i0 : 0;
            const int qhi = n_in - i0 < nwin ? (int)(n_in - i0) : nwin;
            gptr<const T> sw = src + i0;
            if (t0) __syncthreads();
            constexpr int NB = 16;   // window loads in flight per lane
            for (int b0 = 0; b0 < nwin; b0 += NB * CONV_NT) {
                T v[NB], tv[NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const int i = b0 + j * CONV_NT + lane;
                    v[j] = (i >= qlo && i < qhi) ? sw[i] : T(0);
                    tv[j] = i < kc ? w[t0 + i] : T(0);
                }
                if (t0 == 0 && b0 == 0) held(0, ov);   // (while the window's loads are in flight)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const int i = b0 + j * CONV_NT + lane;
                    if (i < nwin) win[i] = v[j];
                    if (i < kc) taps[i] = tv[j];
                }
            }
            __syncthreads();
            // steps of U taps in two register buffers (the barriers keep the
            // compiler from sinking the next step's reads to where they are
            // used); tap tt + (lane % 16) in every row of 16 lanes
            T c[R], xa[U], xb[U], ta = T(0), te = T(0);
            auto fetch = [&](int u, T (&v)[U], T& tv) {
#pragma unroll
                for (int j = 0; j < U / Vec16<T>::W; ++j) {
                    using V = typename Vec16<T>::type;
                    const V q = *reinterpret_cast<const V*>(win + li + u * U + R + j * Vec16<T>::W);
                    vec_get<T>(q, v + j * Vec16<T>::W);
                }
                tv = taps[u * U + (lane & 15)];
            };
            constexpr auto seq = std::make_integer_sequence<int, U>{};
#pragma unroll
            for (int j = 0; j < R; ++j) c[j] = win[li + j];
            const int nu = kc / U;
            if (nu > 0) fetch(0, xa, ta);
            for (int u = 0; u + 1 < nu; u += 2) {
                fetch(u + 1, xb, te);
                __builtin_amdgcn_sched_barrier(0);
                conv_row<T, R>(acc, c, xa, ta, seq);
                fetch(u + 2 < nu ? u + 2 : u, xa, ta);
                __builtin_amdgcn_sched_barrier(0);
                conv_row<T, R>(acc, c, xb, te, seq);
            }
            if (nu & 1) conv_row<T, R>(acc, c, xa, ta, seq);
            for (int tt = nu * U; tt < kc; tt += 4) {   // (kc is a multiple of 4)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const T tv = taps[tt + t];
#pragma unroll
                    for (int r = 0; r < R; ++r) acc[r] = fma(tv, win[li + tt + t + r], acc[r]);
                }
            }
        }
        write(0, ov, acc);
    } else {
        conv_sums<T, CONV_NT>(cb, adj, src, ot, cl.kc, conv_smem, acc);
#pragma unroll
        for (int r0 = 0; r0 < R; r0 += NH) {   // (all at once: 102 registers in FP32, half a wave fewer)
            double ov[NH];
            held(r0, ov);
            write(r0, ov, acc);
        }
    }
}

// ---------------------------------------------------------------- operator: dense block
// out[row] = v + s * dot(a[row, :], in) for the rows of a tile, v the row's base and
// identity blocks (own: no other block writes the row) or what the output holds.  The
// adjoint walks the stored transpose, so both directions read rows contiguously; FP64
// accumulation, thread t over the 16-byte vectors t + 256 j of the row, then the waves.
// NV > 0: a row is at most 256 NV vectors.  The thread keeps its part of the input in
// registers and the workgroup streams its rows one after the other, each a contiguous
// run of up to 48 KB, with the next row's loads in flight: 35.1 us per product of
// 5000 x 10000 FP32 with its transpose in turn (400 MB, past the last-level cache:
// 5.7 TB/s, where a plain read of 400 MB reaches 6.3), 36.6 with four rows side by side
// and the input loaded again for them.  NV = 0: longer rows, that form.
// Output elements no dense block writes are initialisation tiles of the same launch
// (a launch of its own took 4.7-7.4 us per product).
constexpr int GEMV_NT = 256;
constexpr int GEMV_RB = 4;
template <typename T> using v16u = typename Vec16<T>::type __attribute__((aligned(sizeof(T))));

template <typename T, int NV>
__global__ __launch_bounds__(GEMV_NT) void k_gemv(Tables tb, DenseLaunch dl, int adj, int out, int in, int base,
                                                  double sigma, int gate, int own) {
    using V = typename Vec16<T>::type;
    constexpr int VW = Vec16<T>::W;
    __shared__ double part[DENSE_ROWS_MAX][GEMV_NT / 64];
    if ((int)blockIdx.x >= dl.ntiles) {
        const VecTile it = dl.init[blockIdx.x - dl.ntiles].tile();
        const InstDesc di = tb.inst[it.inst];
        // (two elements at a time: eight take 200 registers, half the products' waves)
        if (gate_ok(scal(di), gate)) init_tile<T, 2>(tb, di, it, adj, out, in, base, sigma, false);
        return;
    }
    const DenseTile tl = dl.tiles[blockIdx.x];
    const InstDesc d = tb.inst[tl.inst];
    const DenseBlock db = dl.blocks[tl.blk];
    if (!gate_ok(scal(d), gate)) return;
    const int tid = threadIdx.x, wave = tid >> 6;
    const int64_t ld = adj ? db.ldt() : db.ld(), ncols = adj ? db.rows : db.cols;
    const int64_t rows = adj ? db.cols : db.rows, per = dense_tile_rows(rows), r0 = (int64_t)tl.t * per;
    const int64_t g0 = (adj ? db.col0 : db.row0) + r0;   // the tile's first output
    gptr<const T> arow = (gptr<const T>)(adj ? db.at : db.a) + r0 * ld;
    gptr<T> o = (adj ? xvec<T>(d, out) : yvec<T>(d, out)) + g0;
    gptr<const T> x = adj ? yvec<T>(d, in) + db.row0 : xvec<T>(d, in) + db.col0;
    const int nr = (int)(rows - r0 < per ? rows - r0 : per);   // <= DENSE_ROWS_MAX
    T v0 = T(0);            // thread r < nr: what row r holds besides the products
    if (tid < nr) v0 = own ? (T)owned_init<T>(d, tb.ids, adj, in, base, sigma, g0 + tid) : o[tid];
    const int64_t nvec = ncols / VW, jt = nvec * VW + tid;   // (jt: the thread's element past the vectors)
    auto wave_part = [&](int r, double acc) {
        if (jt < ncols) acc = fma((double)arow[r * ld + jt], (double)x[jt], acc);
        acc = wave_sum(acc);
        if ((tid & 63) == 0) part[r][wave] = acc;
    };
    if constexpr (NV > 0) {
        // (the longest rows leave the next row's loads to the CU's other workgroups:
        // a second buffer would halve their number)
        constexpr bool AHEAD = NV < 12;
        V xv[NV], cur[NV], nxt[NV];
        const V zero = {};
        const int nv = (int)nvec;
        auto load_row = [&](int r, V (&m)[NV]) {
            gptr<const V> p = (gptr<const V>)(arow + r * ld);
#pragma unroll
            for (int u = 0; u < NV; ++u) m[u] = tid + GEMV_NT * u < nv ? p[tid + GEMV_NT * u] : zero;
        };
        load_row(0, cur);
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int i = tid + GEMV_NT * u;
            xv[u] = i < nv ? (V)*(gptr<const v16u<T>>)(x + (int64_t)i * VW) : zero;
        }
        for (int r = 0; r < nr; ++r) {
            if (AHEAD && r + 1 < nr) load_row(r + 1, nxt);
            double acc = 0.0;
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                if (tid + GEMV_NT * u >= nv) break;
#pragma unroll
                for (int e = 0; e < VW; ++e) acc = fma((double)cur[u][e], (double)xv[u][e], acc);
            }
            if (!AHEAD && r + 1 < nr) load_row(r + 1, cur);
            wave_part(r, acc);
            if (AHEAD) {
#pragma unroll
                for (int u = 0; u < NV; ++u) cur[u] = nxt[u];
            }
        }
    } else {
        for (int rb = 0; rb < nr; rb += GEMV_RB) {
            double acc[GEMV_RB];
#pragma unroll
            for (int r = 0; r < GEMV_RB; ++r) acc[r] = 0.0;
            for (int64_t v = tid; v < nvec; v += GEMV_NT) {
                const V xv = (V)*(gptr<const v16u<T>>)(x + v * VW);
#pragma unroll
                for (int r = 0; r < GEMV_RB; ++r) {
                    if (rb + r >= nr) continue;
                    const V av = *(gptr<const V>)(arow + (rb + r) * ld + v * VW);
#pragma unroll
                    for (int e = 0; e < VW; ++e) acc[r] = fma((double)av[e], (double)xv[e], acc[r]);
                }
            }
#pragma unroll
            for (int r = 0; r < GEMV_RB; ++r)
                if (rb + r < nr) wave_part(rb + r, acc[r]);
        }
    }
    __syncthreads();
    if (tid < nr) {
        double tot = 0.0;
#pragma unroll
        for (int w = 0; w < GEMV_NT / 64; ++w) tot += part[tid][w];
        o[tid] = (T)((double)v0 + sigma * db.scale * tot);
    }
}

// ---------------------------------------------------------------- CG
template <typename T>
__global__ __launch_bounds__(VEC_NT) void k_cg_init(Tables tb, int z, int r, int p, int q, int h,
                                                    int have_q, int gate, double* parts, int stride) {
    __shared__ double sh[VEC_NT / 64];
    const VecTile tl = tb.xt[blockIdx.x];
    const InstDesc d = tb.inst[tl.inst];
    gptr<double> sc = scal(d);
    if (!gate_ok(sc, gate)) return;
    gptr<T> rv = xvec<T>(d, r);
    gptr<T> pv = xvec<T>(d, p);
    gptr<const T> qv = xvec<T>(d, q);
    gptr<const T> hv = xvec<T>(d, h);
    double s0 = 0.0, s1 = 0.0;
    for (int64_t i = tl.start + threadIdx.x; i < tl.start + tl.len; i += VEC_NT) {
        const double hi = (double)hv[i];
        const T ri = (T)(have_q ? hi - (double)qv[i] : hi);
        rv[i] = ri;
        pv[i] = ri;
        s0 += (double)ri * (double)ri;
        s1 += hi * hi;
    }
    s0 = block_sum<VEC_NT>(s0, sh);
    s1 = block_sum<VEC_NT>(s1, sh);
    double* part = parts + stride * (int64_t)blockIdx.x;
    if (threadIdx.x == 0) {
        part[0] = s0;
        part[1] = s1;
    }
}

// Partials of <p, q>, ||r||^2, <r, q> and ||q||^2 (slots 0..3).  The first
// tile's workgroup records the iteration whose products are now in place: the
// update of that iteration runs only if it finds this mark, so the update can
// clear the run flag without racing its own workgroups' gate tests.
template <typename T>
__global__ __launch_bounds__(VEC_NT) void k_cg_dot(Tables tb, int p, int q, int r, int it, int gate) {
    __shared__ double sh[4 * (VEC_NT / 64)];
    const VecTile tl = tb.xt[blockIdx.x];
    const InstDesc d = tb.inst[tl.inst];
    gptr<double> sc = scal(d);
    if (!gate_ok(sc, gate)) return;
    if ((int)blockIdx.x == d.xt0 && threadIdx.x == 0) sc[SC_CGRUN] = (double)it;
    gptr<const T> pv = xvec<T>(d, p);
    gptr<const T> qv = xvec<T>(d, q);
    gptr<const T> rv = xvec<T>(d, r);
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t i = tl.start + threadIdx.x; i < tl.start + tl.len; i += VEC_NT) {
        const double pi = (double)pv[i], qi = (double)qv[i], ri = (double)rv[i];
        s[0] = fma(pi, qi, s[0]);
        s[1] = fma(ri, ri, s[1]);
        s[2] = fma(ri, qi, s[2]);
        s[3] = fma(qi, qi, s[3]);
    }
    block_sum4<VEC_NT>(s, sh);
    if (threadIdx.x == 0) {
        double* part = tb.cpart + 4 * (int64_t)blockIdx.x;
        part[0] = s[0];
        part[1] = s[1];
        part[2] = s[2];
        part[3] = s[3];
    }
}

// The scalar products of u~_tau for one tile (Section V-B: the tau component
// of the subspace projection): c^T z_x over an X tile, or b^T z_y over a Y
// tile with z_y = w_y + A z (the carried product) formed, not stored; FP64 partial in
// slot 0 of the tile in Tables::tpart, and the cone terms of
// the projection that follows (CgStart::tau).
//
// The element work of the update that ends an instance's CG, and of a CG
// update that goes on, in one routine: `upd` = 0 leaves z and A z as they are
// (a step whose CG ran no update) and only does the tau (and cone) work.
// Every thread loads its chunks of every vector it needs before the first
// arithmetic, then stores.
template <typename T>
DEVI void cg_elems(const Tables& tb, const InstDesc& d, const XYTile& xt, gptr<const double> sc,
                   const CgStart& cs, bool upd, double al, double be, bool more, bool track, bool tw,
                   int z, int r, int p, int q, double* sh) {
    // One chunk at a time (all its loads, then the arithmetic, then its
    // stores): holding every chunk of every vector at once needs more
    // registers than let all of a launch's workgroups be resident together.
    const Chunks ck(xt.t.start, xt.t.start + xt.t.len);
    if (!xt.is_y) {
        gptr<T> zp = xvec<T>(d, z);
        gptr<T> rp = xvec<T>(d, r);
        gptr<const T> pp = xvec<T>(d, p);
        gptr<T> pw = xvec<T>(d, cs.pn >= 0 ? cs.pn : p);
        gptr<const T> qp = xvec<T>(d, q);
        gptr<T> kp = xvec<T>(d, XK);
        gptr<const T> cp = xvec<T>(d, XC);
        double s0 = 0.0;
#pragma unroll 1
        for (int j = 0; j < NCH; ++j) {
            if (!ck.any(j)) break;
            const int64_t i = ck.at(j);
            v4<T> zv = ld4<T>(zp, i), qv, pv, rv, kv, cv;
            if (upd) {
                qv = ld4<T>(qp, i);
                pv = ld4<T>(pp, i);
                if (more) rv = ld4<T>(rp, i);
                if (track) kv = ld4<T>(kp, i);
            }
            if (tw) cv = ld4<T>(cp, i);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (upd) {
                    const double qi = (double)qv[e], pi = (double)pv[e];
                    zv[e] = (T)fma(al, pi, (double)zv[e]);
                    if (more) {
                        const T ri = (T)fma(-al, qi, (double)rv[e]);
                        rv[e] = ri;
                        pv[e] = (T)fma(be, pi, (double)ri);
                    }
                    if (track) kv[e] = (T)fma(al, qi, (double)kv[e]);
                }
                if (tw && ck.has(j, e)) s0 = fma((double)cv[e], (double)zv[e], s0);
            }
            if (upd) {
                // (once CG has ended, r is dead: the next solve forms it afresh)
                st4<T>(zp, ck, j, zv);
                if (more) {
                    st4<T>(rp, ck, j, rv);
                    st4<T>(pw, ck, j, pv);
                }
                if (track) st4<T>(kp, ck, j, kv);
            }
        }
        if (tw) {
            s0 = block_sum<VEC_NT>(s0, sh);
            if (threadIdx.x == 0) {
                tb.tpart[xt.index] = s0;
                if (xt.index == d.xt0) {
                    // for the projection: the expansion point and tau + kappa
                    // (it rewrites tau and kappa while its workgroups run)
                    double* part = tb.xpart + 4 * (int64_t)xt.index;
                    const double ex = sc[SC_UT];
                    part[1] = std::isfinite(ex) ? ex : 0.0;
                    part[2] = sc[SC_TAU] + sc[SC_KAPPA];
                }
            }
        }
        return;
    }
    gptr<T> azp = yvec<T>(d, YA);
    gptr<const T> app = yvec<T>(d, YT);
    gptr<const T> wyp = yvec<T>(d, YW);
    gptr<const T> bp = yvec<T>(d, YB);
    gptr<const T> uyp = yvec<T>(d, YU);
    gptr<const T> vsp = yvec<T>(d, YV);
    gptr<const T> gyp = yvec<T>(d, YG);
    const bool cone = tw && xt.t.seg >= 0;
    double e_pt = 0.0;
    int64_t head = -1;
    if (cone) {
        const double ex = sc[SC_UT];
        e_pt = std::isfinite(ex) ? ex : 0.0;
        head = tb.seg[xt.t.seg].start;
    }
    const double alpha = cs.alpha;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int j = 0; j < NCH; ++j) {
        if (!ck.any(j)) break;
        const int64_t i = ck.at(j);
        v4<T> av = ld4<T>(azp, i), apv, wv, bv, uv, vv, gv;
        if (upd) apv = ld4<T>(app, i);
        if (tw) bv = ld4<T>(bp, i);
        if (cone) {
            // w_y = u_y + v_s as the projection (or k_wy) formed it from
            // these stored values: recomputed instead of loaded
            uv = ld4<T>(uyp, i);
            vv = ld4<T>(vsp, i);
            gv = ld4<T>(gyp, i);
#pragma unroll
            for (int e = 0; e < 4; ++e) wv[e] = (T)((double)uv[e] + (double)vv[e]);
        } else if (tw) {
            wv = ld4<T>(wyp, i);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (upd) av[e] = (T)fma(al, (double)apv[e], (double)av[e]);
            if (!tw) continue;
            const T zy = (T)((double)wv[e] + (double)av[e]);
            wv[e] = zy;   // (w_y is not needed again: the register holds z_y)
            if (!ck.has(j, e)) continue;
            s[0] = fma((double)bv[e], (double)zy, s[0]);
            if (cone) {
                const double g = (double)gv[e];
                const double a = alpha * (double)zy + (1.0 - alpha) * (double)uv[e] - (double)vv[e] -
                                 alpha * e_pt * g;
                const double b = alpha * g;
                if (i + e == head) {
                    tb.seg_val[2 * xt.t.seg] = a;
                    tb.seg_val[2 * xt.t.seg + 1] = b;
                } else {
                    s[1] = fma(a, a, s[1]);
                    s[2] = fma(a, b, s[2]);
                    s[3] = fma(b, b, s[3]);
                }
            }
        }
        if (upd) st4<T>(azp, ck, j, av);
        // (z_y is not stored: the projection forms it again from u_y, v_s and A z)
    }
    if (!tw) return;
    const int64_t ntl = tb.ny_tiles, b = (int64_t)tb.nx_tiles + xt.index;
    if (cone) {
        block_sum4<VEC_NT>(s, sh);
        if (threadIdx.x == 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) tb.tpart[j * ntl + b] = s[j];
        }
    } else {
        s[0] = block_sum<VEC_NT>(s[0], sh);
        if (threadIdx.x == 0) tb.tpart[b] = s[0];
    }
}

// One CG step after the products: alpha = ||r||^2 / <p, q>; z += alpha p;
// r' = r - alpha q (and the carried K z, A z when tracking); then the next
// direction p = r' + beta p in the same pass.  beta needs ||r'||^2 before r'
// exists anywhere but in this kernel, so it is taken from the expansion
// ||r - alpha q||^2 = ||r||^2 - 2 alpha <r, q> + alpha^2 ||q||^2 of the FP64
// partials of k_cg_dot (the same quantity the method defines, evaluated
// without a second reduction pass); the stop test uses the same value.  Every
// workgroup sums the partials in the same fixed order.  The first tile's
// workgroup records alpha, beta, the counters and the run flag.
template <typename T>
__global__ __launch_bounds__(VEC_NT) void k_cg_update(Tables tb, int z, int r, int p, int q, int it,
                                                      int cg_max, int gate, int track, int folded,
                                                      int last, CgStart cs) {
    __shared__ double sh[12 * (VEC_NT / 64)];
    const XYTile xt = xy_tile(tb);
    const InstDesc d = tb.inst[xt.t.inst];
    gptr<double> sc = scal(d);
    const double run = sc[SC_CGRUN];
    if (!gate_ok(sc, gate)) return;
    bool act = run == (double)it;
    if (!act && !(cs.tested && run < 0.0)) return;   // (tested, < 0: the start test ahead of the products ended CG)
    const bool rec = !xt.is_y && xt.index == d.xt0 && threadIdx.x == 0;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    double h0 = 0.0, h1 = 0.0;
    if (act) {
        if (folded) inst_csum4(tb, d, s, cs.on != 0, h0, h1, sh);   // partials of the A^T launch(es)
        else inst_xsum4(tb, d, s, cs.on != 0, h0, h1, sh);          // partials of k_cg_dot
    }
    double tol;
    if (cs.on) {
        // the step's CG start test, from the right-hand side launch's partials
        // ||r||^2, ||h||^2 (the products of this first iteration ran whatever
        // its outcome); every workgroup evaluates it
        tol = cg_tolerance(sc[SC_ITER], h1, cs.zeta, cs.rate, cs.floor_);
        act = cg_max > 0 && sqrt(h0) > tol && std::isfinite(h0);
        if (rec) {
            sc[SC_RR] = h0;
            sc[SC_HN] = sqrt(h1);
            sc[SC_CGTOL] = tol;
            sc[SC_CGIT] = 0.0;
            sc[SC_CGACT] = act ? 1.0 : 0.0;
        }
    } else {
        tol = sc[SC_CGTOL];
    }
    if (!act) {
        if (cs.tau) cg_elems<T>(tb, d, xt, sc, cs, false, 0.0, 0.0, false, false, true, z, r, p, q, sh);
        return;
    }
    const double pq = s[0], rr = s[1], rq = s[2], qq = s[3];
    const double al = rr / pq;
    const bool ok = pq > 0.0 && std::isfinite(al);
    const double rr1 = fma(al * al, qq, fma(-2.0 * al, rq, rr));
    const double be = rr > 0.0 ? rr1 / rr : 0.0;
    const bool more = ok && std::isfinite(rr1) && sqrt(rr1) > tol && it + 1 < cg_max;
    if (rec) {
        sc[SC_PQ] = pq;
        sc[SC_ALPHA] = ok ? al : 0.0;
        sc[SC_RR] = ok ? rr1 : rr;
        sc[SC_BETA] = be;
        if (ok) {
            sc[SC_CGIT] += 1.0;
            sc[SC_CGTOT] += 1.0;
            if (sc[SC_CGIT] > sc[SC_CGMAX]) sc[SC_CGMAX] = sc[SC_CGIT];
            if (gate == G_SETUP) sc[SC_SETUPIT] += 1.0;
        }
        // the step's last CG launch, and CG would go on: the step needs more
        // launches than the interval has.  The instance is suspended (phase 3:
        // every later kernel of the interval skips it) until the host restores
        // the interval's snapshot and runs the interval again.
        if (last && more) sc[SC_PHASE] = 3.0;
        sc[SC_CGACT] = more ? 1.0 : 0.0;
    }
    // the step's last CG update also forms the tau products on the final
    // z and A z (cs.tau: every instance's CG ends in an update of this loop)
    const bool tw = cs.tau && !more;
    if ((!ok || (xt.is_y && !track)) && !tw) return;
    cg_elems<T>(tb, d, xt, sc, cs, ok, al, be, more, track != 0, tw, z, r, p, q, sh);
}

template <typename T>
__global__ __launch_bounds__(VEC_NT) void k_wy(Tables tb, int gate) {
    const VecTile tl = tb.yt[blockIdx.x];
    const InstDesc d = tb.inst[tl.inst];
    if (!gate_ok(scal(d), gate)) return;
    gptr<const T> u = yvec<T>(d, YU);
    gptr<const T> v = yvec<T>(d, YV);
    gptr<T> w = yvec<T>(d, YW);
    for (int64_t i = tl.start + threadIdx.x; i < tl.start + tl.len; i += VEC_NT)
        w[i] = (T)((double)u[i] + (double)v[i]);
}

// A thread's elements of a Y tile of u_y, A z, g_y, v_s, loaded at once
// (ahead of a reduction, and ahead of stores into the same vectors, which
// element by element would order each load after the previous stores);
// pv() is ybar_minus_v on them.
template <typename T>
struct YbarTile {
    static constexpr int R = VEC_TILE / VEC_NT;
    T u[R], a[R], g[R], v[R];
    DEVI void load(const InstDesc& d, const VecTile& tl) {
        gptr<const T> pu = yvec<T>(d, YU), pa = yvec<T>(d, YA), pg = yvec<T>(d, YG), pvv = yvec<T>(d, YV);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int64_t o = threadIdx.x + (int64_t)j * VEC_NT;
            const int64_t i = tl.start + (o < tl.len ? o : 0);
            u[j] = pu[i];
            a[j] = pa[i];
            g[j] = pg[i];
            v[j] = pvv[i];
        }
    }
    DEVI bool has(const VecTile& tl, int j) const { return threadIdx.x + (int64_t)j * VEC_NT < tl.len; }
    DEVI int64_t at(const VecTile& tl, int j) const { return tl.start + threadIdx.x + (int64_t)j * VEC_NT; }
    DEVI double pv(int j, double ut, double alpha) const {
        const double uy = (double)u[j];
        const double ut_y = (double)z_y<T>(u[j], v[j], a[j]) - ut * (double)g[j];
        const double ub = alpha * ut_y + (1.0 - alpha) * uy;
        return ub - (double)v[j];
    }
};

template <typename T>
__global__ __launch_bounds__(VEC_NT) void k_project(Tables tb, double alpha) {
    __shared__ double sh[4 * (VEC_NT / 64)];
    const XYTile xt = xy_tile(tb);
    const InstDesc d = tb.inst[xt.t.inst];
    gptr<double> sc = scal(d);
    if (!gate_ok(sc, G_ADMM)) return;
    const int seg = xt.is_y ? xt.t.seg : -1;
    YbarTile<T> yb;
    double ut, t = 0.0, nz = 0.0;
    {
        // u~_tau = (tau + kappa + c^T z_x + b^T z_y) / eta from the slot-0
        // partials (Tables::tpart) of every X and Y tile of the instance, and the cone's head
        // value and tail norm from the cone terms (CgStart::tau), all summed
        // in one fixed order by every workgroup
        const double* xp0 = tb.xpart + 4 * (int64_t)d.xt0;
        const double e_pt = xp0[1], wtau = xp0[2];
        const int64_t ntl = tb.ny_tiles;
        const double* ty = tb.tpart + tb.nx_tiles;   // slot 0 of the Y tiles
        double s[4] = {0.0, 0.0, 0.0, 0.0};
        s[0] = thread_sum<VEC_NT, 4>(tb.tpart, d.xt0, d.xt1, 1) + thread_sum<VEC_NT, 4>(ty, d.yt0, d.yt1, 1);
        double ah = 0.0, bh = 0.0;
        if (seg >= 0) {
            const SocSeg sg = tb.seg[seg];
            ah = tb.seg_val[2 * seg];
            bh = tb.seg_val[2 * seg + 1];
#pragma unroll
            for (int j = 1; j < 4; ++j)
                s[j] = thread_sum<VEC_NT, 4>(ty + j * ntl, sg.yt0, sg.yt0 + sg.ntiles, 1);
        }
        block_sum4<VEC_NT>(s, sh);
        ut = (wtau + s[0]) / sc[SC_ETA];
        if (seg >= 0) {
            const double dl = ut - e_pt;
            t = ah - dl * bh;
            const double n2 = s[1] - 2.0 * dl * s[2] + dl * dl * s[3];
            nz = sqrt(n2 > 0.0 ? n2 : 0.0);
        }
    }
    if (!xt.is_y && xt.index == d.xt0 && threadIdx.x == 0) {
        // tau, kappa of the step (no other workgroup of this kernel reads them)
        sc[SC_UT] = ut;
        const double tau = sc[SC_TAU], kap = sc[SC_KAPPA];
        const double ubar = alpha * ut + (1.0 - alpha) * tau;
        const double tnew = ubar - kap > 0.0 ? ubar - kap : 0.0;
        sc[SC_KAPPA] = kap - ubar + tnew;
        sc[SC_TAU] = tnew;
        sc[SC_ITER] += 1.0;
    }
    const int64_t lo = xt.t.start, hi = xt.t.start + xt.t.len;
    if (!xt.is_y) {
        gptr<T> ux = xvec<T>(d, XU);
        gptr<const T> zx = xvec<T>(d, XZ);
        gptr<const T> gx = xvec<T>(d, XG);
        for (int64_t i = lo + threadIdx.x; i < hi; i += VEC_NT) {
            const double utx = (double)zx[i] - ut * (double)gx[i];
            ux[i] = (T)(alpha * utx + (1.0 - alpha) * (double)ux[i]);
        }
        return;
    }
    gptr<T> uy = yvec<T>(d, YU);
    gptr<T> vs = yvec<T>(d, YV);
    gptr<T> wy = yvec<T>(d, YW);
    if (seg < 0) {
        for (int64_t i = lo + threadIdx.x; i < hi; i += VEC_NT) {
            double ub;
            const double pv = ybar_minus_v<T>(d, i, ut, alpha, ub);
            const double pr = pv > 0.0 ? pv : 0.0;
            const T u = (T)pr, v = (T)(pr - pv);
            uy[i] = u;
            vs[i] = v;
            wy[i] = (T)((double)u + (double)v);
        }
        return;
    }
    const SocSeg sg = tb.seg[seg];
    yb.load(d, xt.t);
    // Pi(t, z): (t, z) if ||z|| <= t; 0 if ||z|| <= -t; ((t+||z||)/2)(1, z/||z||) otherwise
    int mode;
    double a = 0.0;
    if (nz <= t) mode = 0;
    else if (nz <= -t) mode = 1;
    else {
        mode = 2;
        a = 0.5 * (t + nz);
    }
#pragma unroll
    for (int j = 0; j < YbarTile<T>::R; ++j) {
        if (!yb.has(xt.t, j)) continue;
        const int64_t i = yb.at(xt.t, j);
        const double pv = yb.pv(j, ut, alpha);
        double pr;
        if (mode == 0) pr = pv;
        else if (mode == 1) pr = 0.0;
        else pr = (i == sg.start) ? a : (a / nz) * pv;
        const T u = (T)pr, v = (T)(pr - pv);
        uy[i] = u;
        vs[i] = v;
        wy[i] = (T)((double)u + (double)v);   // w_y of the next step
    }
}

// Termination test (relative 2-norm criteria, or the HSDE certificates), in
// the original problem's units: the row sums are divided by D, the column sums
// by E (sums listed at check_outcome).  YT holds A u_x and XT holds A^T u_y on entry.
template <typename T>
__global__ __launch_bounds__(VEC_NT) void k_resid(Tables tb, double eps, int max_iters, int gate) {
    __shared__ double sh[VEC_NT / 64];
    const XYTile xt = xy_tile(tb);
    const InstDesc d = tb.inst[xt.t.inst];
    gptr<double> sc = scal(d);
    if (!gate_ok(sc, gate)) return;
    const double tau = sc[SC_TAU];
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    const int64_t lo = xt.t.start, hi = xt.t.start + xt.t.len;
    if (xt.is_y) {
        gptr<const T> au = yvec<T>(d, YT);
        gptr<const T> vs = yvec<T>(d, YV);
        gptr<const T> b = yvec<T>(d, YB);
        gptr<const T> uy = yvec<T>(d, YU);
        gptr<const T> dr = yvec<T>(d, YD);
        for (int64_t i = lo + threadIdx.x; i < hi; i += VEC_NT) {
            const double w = 1.0 / (double)dr[i];
            const double e = ((double)au[i] + (double)vs[i]) * w;
            const double rp = e - tau * (double)b[i] * w;
            s0 = fma(rp, rp, s0);
            s1 = fma(e, e, s1);
            s2 = fma((double)b[i], (double)uy[i], s2);
        }
    } else {
        gptr<const T> aty = xvec<T>(d, XT);
        gptr<const T> c = xvec<T>(d, XC);
        gptr<const T> ux = xvec<T>(d, XU);
        gptr<const T> ec = xvec<T>(d, XE);
        for (int64_t i = lo + threadIdx.x; i < hi; i += VEC_NT) {
            const double w = 1.0 / (double)ec[i];
            const double e = (double)aty[i] * w;
            const double rd = e + tau * (double)c[i] * w;
            s0 = fma(rd, rd, s0);
            s1 = fma(e, e, s1);
            s2 = fma((double)c[i], (double)ux[i], s2);
        }
    }
    s0 = block_sum<VEC_NT>(s0, sh);
    s1 = block_sum<VEC_NT>(s1, sh);
    s2 = block_sum<VEC_NT>(s2, sh);
    double* part = (xt.is_y ? tb.ypart : tb.xpart) + 4 * (int64_t)xt.index;
    if (threadIdx.x == 0) {
        part[0] = s0;
        part[1] = s1;
        part[2] = s2;
    }
}


// ---------------------------------------------------------------- per-instance finalize
// One workgroup per instance sums the partials of the kernel just before it in
// tile order and finishes the scalar work of the method.
enum FinMode : int {
    FIN_CG_INIT = 0,   // rr = ||r||^2, ||h||; CG tolerance and start flag
    FIN_RESID,         // residuals, gap, certificates, status
    FIN_NORMS,         // ||b||, ||c||
    FIN_ETA            // eta = 1 + c^T g_x + b^T g_y; phase -> iterating
};
struct FinArgs {
    double a0, a1, a2;
    int i0, i1;
};

__global__ __launch_bounds__(VEC_NT) void k_finalize(Tables tb, int mode, int gate, FinArgs fa) {
    __shared__ double sh[VEC_NT / 64];
    const InstDesc d = tb.inst[blockIdx.x];
    gptr<double> sc = scal(d);
    if (!gate_ok(sc, gate)) return;
    double x0 = 0, x1 = 0, x2 = 0, y0 = 0, y1 = 0, y2 = 0;
    const bool use_x = true;
    const bool use_y = mode == FIN_RESID || mode == FIN_NORMS || mode == FIN_ETA;
    const int nslot = (mode == FIN_RESID) ? 3 : (mode == FIN_CG_INIT ? 2 : 1);
    if (use_x) {
        x0 = sum_parts<VEC_NT>(tb.xpart, d.xt0, d.xt1, 0, sh);
        if (nslot > 1) x1 = sum_parts<VEC_NT>(tb.xpart, d.xt0, d.xt1, 1, sh);
        if (nslot > 2) x2 = sum_parts<VEC_NT>(tb.xpart, d.xt0, d.xt1, 2, sh);
    }
    if (use_y) {
        y0 = sum_parts<VEC_NT>(tb.ypart, d.yt0, d.yt1, 0, sh);
        if (nslot > 1) y1 = sum_parts<VEC_NT>(tb.ypart, d.yt0, d.yt1, 1, sh);
        if (nslot > 2) y2 = sum_parts<VEC_NT>(tb.ypart, d.yt0, d.yt1, 2, sh);
    }
    if (threadIdx.x != 0) return;
    switch (mode) {
        case FIN_CG_INIT: {
            const int cg_max = fa.i0;
            const double k = (gate == G_SETUP || gate == G_SETUP_CG) ? 0.0 : sc[SC_ITER];
            const double tol = cg_tolerance(k, x1, fa.a0, fa.a1, fa.a2);
            sc[SC_RR] = x0;
            sc[SC_HN] = sqrt(x1);
            sc[SC_CGTOL] = tol;
            sc[SC_CGIT] = 0.0;
            sc[SC_CGRUN] = -1.0;
            sc[SC_CGACT] = (cg_max > 0 && sqrt(x0) > tol && std::isfinite(x0)) ? 1.0 : 0.0;
            break;
        }
        case FIN_RESID: {
            const CheckOut co = check_outcome(sc, sc[SC_TAU], sc[SC_KAPPA], sc[SC_ITER], y0, y1, y2,
                                              x0, x1, x2, fa.a0, fa.i0);
            sc[SC_CUX] = co.cux;
            sc[SC_BUY] = co.buy;
            sc[SC_CGMAXLAST] = sc[SC_CGMAX];
            sc[SC_CGMAX] = 0.0;
            sc[SC_RP] = co.rp;
            sc[SC_RD] = co.rd;
            sc[SC_GAP] = co.gap;
            sc[SC_CX] = co.cx;
            sc[SC_BY] = co.by;
            if (co.status != 0.0) {
                sc[SC_STATUS] = co.status;
                sc[SC_ACTIVE] = 0.0;
            }
            break;
        }
        case FIN_NORMS:   // of the original b = b^ / (sb D) and c = c^ / (sc E)
            sc[SC_NB] = sqrt(y0) / sc[SC_SB];
            sc[SC_NC] = sqrt(x0) / sc[SC_SC];
            break;
        case FIN_ETA:
            sc[SC_ETA] = 1.0 + x0 + y0;
            sc[SC_PHASE] = d.fused ? 2.0 : 1.0;
            sc[SC_CGACT] = 0.0;
            break;
        default:
            break;
    }
}


// ---------------------------------------------------------------- setup
template <typename T>
__global__ __launch_bounds__(VEC_NT) void k_reset(Tables tb, int only) {
    const XYTile xt = xy_tile(tb);
    if (only >= 0 && xt.t.inst != only) return;
    const InstDesc d = tb.inst[xt.t.inst];
    const int64_t lo = xt.t.start, hi = xt.t.start + xt.t.len;
    if (xt.is_y) {
        gptr<T> uy = yvec<T>(d, YU);
        gptr<T> vs = yvec<T>(d, YV);
        gptr<T> az = yvec<T>(d, YA);
        for (int64_t i = lo + threadIdx.x; i < hi; i += VEC_NT) {
            uy[i] = T(0);
            vs[i] = T(0);
            az[i] = T(0);
        }
    } else {
        gptr<T> ux = xvec<T>(d, XU);
        gptr<T> zx = xvec<T>(d, XZ);
        gptr<T> gx = xvec<T>(d, XG);
        gptr<T> kz = xvec<T>(d, XK);
        for (int64_t i = lo + threadIdx.x; i < hi; i += VEC_NT) {
            ux[i] = T(0);
            zx[i] = T(0);
            gx[i] = T(0);
            kz[i] = T(0);
        }
        if (xt.index == d.xt0 && threadIdx.x == 0) {
            gptr<double> sc = scal(d);
            const double sb = sc[SC_SB], scc = sc[SC_SC];   // data, like b and c
            for (int j = 0; j < NSC; ++j) sc[j] = 0.0;
            sc[SC_SB] = sb;
            sc[SC_SC] = scc;
            sc[SC_TAU] = 1.0;
            sc[SC_KAPPA] = 1.0;
            sc[SC_ACTIVE] = 1.0;
            sc[SC_PHASE] = 0.0;
            int* cn = counters(d);
            for (int j = 0; j < NCNT; ++j) cn[j] = 0;
        }
    }
}

template <typename T>
__global__ __launch_bounds__(VEC_NT) void k_norms(Tables tb, int gate) {
    __shared__ double sh[VEC_NT / 64];
    const XYTile xt = xy_tile(tb);
    const InstDesc d = tb.inst[xt.t.inst];
    gptr<double> sc = scal(d);
    if (!gate_ok(sc, gate)) return;
    gptr<const T> v = xt.is_y ? yvec<T>(d, YB) : xvec<T>(d, XC);
    gptr<const T> w = xt.is_y ? yvec<T>(d, YD) : xvec<T>(d, XE);
    double s0 = 0.0;
    for (int64_t i = xt.t.start + threadIdx.x; i < xt.t.start + xt.t.len; i += VEC_NT) {
        const double e = (double)v[i] / (double)w[i];
        s0 = fma(e, e, s0);
    }
    s0 = block_sum<VEC_NT>(s0, sh);
    double* part = (xt.is_y ? tb.ypart : tb.xpart) + 4 * (int64_t)xt.index;
    if (threadIdx.x == 0) part[0] = s0;
}

// eta = 1 + c^T g_x + b^T g_y; the instance then starts iterating.
template <typename T>
__global__ __launch_bounds__(VEC_NT) void k_eta(Tables tb) {
    __shared__ double sh[VEC_NT / 64];
    const XYTile xt = xy_tile(tb);
    const InstDesc d = tb.inst[xt.t.inst];
    gptr<double> sc = scal(d);
    if (!gate_ok(sc, G_SETUP)) return;
    gptr<const T> a = xt.is_y ? yvec<T>(d, YB) : xvec<T>(d, XC);
    gptr<const T> g = xt.is_y ? yvec<T>(d, YG) : xvec<T>(d, XG);
    double s0 = 0.0;
    for (int64_t i = xt.t.start + threadIdx.x; i < xt.t.start + xt.t.len; i += VEC_NT)
        s0 = fma((double)a[i], (double)g[i], s0);
    s0 = block_sum<VEC_NT>(s0, sh);
    double* part = (xt.is_y ? tb.ypart : tb.xpart) + 4 * (int64_t)xt.index;
    if (threadIdx.x == 0) part[0] = s0;
}

template <typename T>
__global__ __launch_bounds__(VEC_NT) void k_fill(Tables tb, int is_y, int kind, double v, int gate) {
    const VecTile tl = is_y ? tb.yt[blockIdx.x] : tb.xt[blockIdx.x];
    const InstDesc d = tb.inst[tl.inst];
    if (!gate_ok(scal(d), gate)) return;
    gptr<T> o = is_y ? yvec<T>(d, kind) : xvec<T>(d, kind);
    for (int64_t i = tl.start + threadIdx.x; i < tl.start + tl.len; i += VEC_NT) o[i] = (T)v;
}

template <typename T>
__global__ __launch_bounds__(VEC_NT) void k_copy(Tables tb, int is_y, int dst, int src, int gate) {
    const VecTile tl = is_y ? tb.yt[blockIdx.x] : tb.xt[blockIdx.x];
    const InstDesc d = tb.inst[tl.inst];
    if (!gate_ok(scal(d), gate)) return;
    gptr<T> o = is_y ? yvec<T>(d, dst) : xvec<T>(d, dst);
    gptr<const T> s = is_y ? yvec<T>(d, src) : xvec<T>(d, src);
    for (int64_t i = tl.start + threadIdx.x; i < tl.start + tl.len; i += VEC_NT) o[i] = s[i];
}

// Copy of the carried state of every instance that runs one launch per kernel
// (restore = 0: region -> copy; 1: copy -> region).  X tiles copy u_x, z, K z,
// Y tiles u_y, v_s, w_y, A z; the first X tile's workgroup also copies the
// header (scalars and counters).  Instances of the fused path, which runs
// concurrently on another stream, and instances without a copy are left alone.
template <typename T>
__global__ __launch_bounds__(VEC_NT) void k_snapshot(Tables tb, int restore) {
    const XYTile xt = xy_tile(tb);
    const InstDesc d = tb.inst[xt.t.inst];
    if (d.fused || d.snap == nullptr) return;
    gptr<char> region = (gptr<char>)d.base;
    gptr<char> copy = (gptr<char>)d.snap;
    if (!xt.is_y && xt.index == d.xt0) {
        gptr<const int64_t> hs = (gptr<const int64_t>)(restore ? copy : region);
        gptr<int64_t> hd = (gptr<int64_t>)(restore ? region : copy);
        for (int i = threadIdx.x; i < REGION_HDR / 8; i += VEC_NT) hd[i] = hs[i];
    }
    gptr<T> cx = (gptr<T>)(copy + REGION_HDR);
    gptr<T> cy = cx + (int64_t)SNAP_X * d.nxs;
    const int64_t lo = xt.t.start, hi = xt.t.start + xt.t.len;
    const int nv = xt.is_y ? SNAP_Y : SNAP_X;
    for (int v = 0; v < nv; ++v) {
        gptr<T> live = xt.is_y ? yvec<T>(d, v == 0 ? YU : YV) : xvec<T>(d, v == 0 ? XU : XZ);
        gptr<T> kept = xt.is_y ? cy + (int64_t)v * d.nys : cx + (int64_t)v * d.nxs;
        gptr<T> dst = restore ? live : kept;
        gptr<const T> src = restore ? kept : live;
        for (int64_t i = lo + threadIdx.x; i < hi; i += VEC_NT) dst[i] = src[i];
    }
}

// Points of the original problem (what 0: x, 1: y, 2: s; rays scaled by
// -c^T x_ray or -b^T y_ray for certificates) or the raw iterate (3: u_x,
// 4: u_y, 5: v_s) of the scaled problem.
template <typename T>
struct Extract {
    gptr<const T> v, w;
    double scale;
    bool divide;
    DEVI Extract(const InstDesc& d, int what) : w(nullptr), scale(1.0), divide(false) {
        gptr<const double> sc = scal(d);
        const double status = sc[SC_STATUS];
        if (what == 0 || what == 3) v = xvec<T>(d, XU);
        else if (what == 1 || what == 4) v = yvec<T>(d, YU);
        else v = yvec<T>(d, YV);
        if (what > 2) return;
        double ray = sc[SC_TAU];   // x = x_ray / tau, ...
        if (status == 3.0) ray = (what == 1) ? -sc[SC_BUY] : NAN;
        else if (status == 4.0) ray = (what == 1) ? NAN : -sc[SC_CUX];
        if (what == 0) {          // x_ray = E u_x / sb
            w = xvec<T>(d, XE);
            scale = 1.0 / (sc[SC_SB] * ray);
        } else if (what == 1) {   // y_ray = D u_y / sc
            w = yvec<T>(d, YD);
            scale = 1.0 / (sc[SC_SC] * ray);
        } else {                  // s_ray = v_s / (D sb)
            w = yvec<T>(d, YD);
            divide = true;
            scale = 1.0 / (sc[SC_SB] * ray);
        }
    }
    DEVI double at(int64_t i) const {
        double e = (double)v[i];
        if (w) e = divide ? e / (double)w[i] : e * (double)w[i];
        return e * scale;
    }
};
template <typename T>
__global__ void k_extract(const InstDesc* insts, int inst, int what, int64_t off, int64_t len,
                          double* out) {
    const Extract<T> x(insts[inst], what);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < len;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = x.at(off + i);
}
// those of x, y and s (bits 0 to 2 of want) of an instance one after the other, one to
// each blockIdx.y
template <typename T>
__global__ void k_extract_point(const InstDesc* insts, int inst, int want, double* out) {
    const InstDesc d = insts[inst];
    int what = 0;
    for (int left = blockIdx.y;; ++what) {
        if (!((want >> what) & 1)) continue;
        if (left-- == 0) break;
        out += what == 0 ? d.n : d.m;
    }
    const Extract<T> x(d, what);
    const int64_t len = what == 0 ? d.n : d.m;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < len;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = x.at(i);
}
// an instance's scaled data, FP64 [b^ (m) | D (m) | c^ (n) | E (n) | sb, sc], into its region
template <typename T>
__global__ void k_put_data(const double* src, char* base, int64_t n, int64_t m, int64_t nxs, int64_t nys) {
    InstDesc d{};
    d.base = base;
    d.nxs = nxs;
    d.nys = nys;
    const int64_t total = 2 * (n + m);
    gptr<T> b = yvec<T>(d, YB), dr = yvec<T>(d, YD), c = xvec<T>(d, XC), e = xvec<T>(d, XE);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const T v = (T)src[i];
        if (i < m) b[i] = v;
        else if (i < 2 * m) dr[i - m] = v;
        else if (i < 2 * m + n) c[i - 2 * m] = v;
        else e[i - 2 * m - n] = v;
    }
    if (blockIdx.x == 0 && threadIdx.x < 2) scal(d)[threadIdx.x == 0 ? SC_SB : SC_SC] = src[total + threadIdx.x];
}

template <typename T>
__global__ void k_cast(const double* src, T* dst, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = (T)src[i];
}

template <typename S, typename T>
__global__ void k_cast_pad(const S* src, int64_t lds, int64_t rows, int64_t cols, T* dst, int64_t ld) {
    const int64_t total = rows * ld;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = i / ld, c = i - r * ld;
        dst[i] = c < cols ? (T)(double)src[r * lds + c] : T(0);
    }
}

// 32x32 LDS-tiled transpose of a row chunk: dst[c * ldt + r0 + r] = src[r * lds + c]
template <typename S, typename T>
__global__ __launch_bounds__(256) void k_cast_transpose(const S* src, int64_t lds, int64_t rows,
                                                        int64_t cols, T* dst, int64_t ldt,
                                                        int64_t r0) {
    __shared__ double tile[32][33];
    const int64_t c_base = (int64_t)blockIdx.x * 32, r_base = (int64_t)blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
    for (int j = ty; j < 32; j += 8) {
        const int64_t r = r_base + j, c = c_base + tx;
        tile[j][tx] = (r < rows && c < cols) ? (double)src[r * lds + c] : 0.0;
    }
    __syncthreads();
    for (int j = ty; j < 32; j += 8) {
        const int64_t c = c_base + j, r = r_base + tx;
        if (c < cols && r < rows) dst[c * ldt + r0 + r] = (T)tile[tx][j];
    }
}

// Row sums of squares of a device matrix, one thread per row, each summed in
// column order (the host's order for a copied block); a non-finite entry
// raises *bad.  Rows [r0, r0 + nr) into out[0, nr).
template <typename S>
__global__ __launch_bounds__(256) void k_dense_rowsq(const S* a, int64_t lda, int64_t r0, int64_t nr,
                                                     int64_t cols, double* out, int* bad) {
    // products and sums rounded separately, as the host's (which has no FMA)
#pragma clang fp contract(off)
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nr) return;
    const S* row = a + (r0 + r) * lda;
    double s = 0.0;
    bool fin = true;
    for (int64_t c = 0; c < cols; ++c) {
        const double v = (double)row[c];
        fin = fin && isfinite(v);
        s += v * v;
    }
    out[r] = s;
    if (!fin) atomicOr(bad, 1);
}

template <typename T>
__global__ void k_cast_back(const T* src, double* dst, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = (double)src[i];
}

// Gather every instance's scalar block into one contiguous array.
__global__ void k_gather_scalars(const InstDesc* insts, int ninst, double* out) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < ninst * NSC; i += gridDim.x * blockDim.x) {
        const int a = i / NSC, j = i - a * NSC;
        out[i] = reinterpret_cast<const double*>(insts[a].base)[j];
    }
}

// Write one scalar of one instance (host-side state changes).
__global__ void k_set_scalar(const InstDesc* insts, int inst, int slot, double v) {
    if (threadIdx.x == 0 && blockIdx.x == 0) reinterpret_cast<double*>(insts[inst].base)[slot] = v;
}

// ---------------------------------------------------------------- launchers
#define CGS_DISPATCH(prec, KERNEL, grid, block, st, ...)                                 \
    do {                                                                                \
        if ((grid) > 0) {                                                               \
            if ((prec) == 0) KERNEL<double><<<(grid), (block), 0, (st)>>>(__VA_ARGS__);  \
            else KERNEL<float><<<(grid), (block), 0, (st)>>>(__VA_ARGS__);               \
        }                                                                               \
    } while (0)

static int flat_grid(int64_t n, int block) {
    int64_t g = (n + block - 1) / block;
    if (g > 65535) g = 65535;
    return g < 1 ? 1 : (int)g;
}

void launch_apply_init(int prec, const Tables& t, int adj, int out, int in, int base,
                       double sigma, int gate, hipStream_t st) {
    CGS_DISPATCH(prec, k_apply_init, adj ? t.nx_tiles : t.ny_tiles, VEC_NT, st, t, adj, out, in,
                 base, sigma, gate);
}
// Workgroups per tile of the tile tables: two, in the narrow form of k_conv, where a wave's
// own chain bounds the launch: up to 512 tiles (at most two waves per SIMD in the other
// form) and, in FP64, kernels long enough for the chain to outweigh the narrow form's longer
// start, or several identity blocks, whose loads it has in flight with the window's.
// us, wide / narrow, first at 20-30 tiles, then at 490-510: a launch in FP32, A and A^T with
// their initialisation in FP64, of a deconvolution (2 identity blocks) and a lasso (8)
//   FP32 k = 5     5.1 / 4.6    5.5 / 5.0     FP64 deconvolution        FP64 lasso
//        k = 17    5.3 / 4.8    5.7 / 5.2     k = 5     9.2 / 10.3  10.4 / 11.4  12.7 / 12.5  15.5 / 14.7
//        k = 65    5.7 / 5.3    6.0 / 5.8     k = 65   10.6 / 11.2  12.0 / 12.6  14.1 / 13.2  16.2 / 16.1
//        k = 1025 24.8 / 17.3  25.2 / 18.4    k = 129  12.3 / 12.1  13.7 / 13.8  16.0 / 14.3  18.1 / 17.7
// (FP64 launches alone, k = 257 7.6 / 6.3, 8.0 / 7.0 and 782 tiles 8.4 / 8.9; k = 1025 18.8 / 14.0,
// 19.5 / 15.6 and 21.6 / 22.2.)
static int conv_sub(int prec, const ConvLaunch& c) {
    return c.ntiles <= 512 && (prec == 0 ? c.kc >= 128 || c.nid > 4 : c.kc >= 8) ? 2 : 1;
}
// Workgroups per initialisation tile: more where the launch is short
static int conv_init_parts(const ConvLaunch& c) { return c.ntiles <= 512 ? 8 : 2; }

void launch_conv(int prec, const Tables& t, const ConvLaunch& c, int adj, int out, int in, int base,
                 double sigma, int gate, hipStream_t st) {
    const int sub = conv_sub(prec, c), parts = conv_init_parts(c);
    const int grid = c.ntiles * sub + c.ninit * parts;
    if (grid <= 0) return;
    ConvLaunch cl = c;
    if (sub == 1) cl.kc = std::min(c.kc, prec == 0 ? CONV_KC_MAX_F64 : CONV_KC_MAX_F32);
    // taps and window (at the larger R)
    const size_t lds = (size_t)(2 * cl.kc + (prec == 0 ? CONV_TILE_F64 + 2 * CONV_R_F64 : CONV_TILE_F32 + 2 * CONV_R_F32)) *
                       (prec == 0 ? 8 : 4);
#define CGS_CONV(T, R) k_conv<T, R><<<grid, CONV_NT, lds, st>>>(t, cl, sub, parts, adj, out, in, base, sigma, gate)
    if (prec == 0) {
        if (sub == 2) CGS_CONV(double, 2);
        else CGS_CONV(double, 4);
    } else {
        if (sub == 2) CGS_CONV(float, 4);
        else CGS_CONV(float, 8);
    }
#undef CGS_CONV
}
template <typename T>
static void gemv(const Tables& t, const DenseLaunch& d, int adj, int out, int in, int base, double sigma, int gate,
                 int own, hipStream_t st) {
    const int grid = d.ntiles + (own ? d.ninit : 0);
    if (grid <= 0) return;
    const int nv = (int)((d.vecs + GEMV_NT - 1) / GEMV_NT);   // vectors per thread of the longest row
#define CGS_GEMV(NV) k_gemv<T, NV><<<grid, GEMV_NT, 0, st>>>(t, d, adj, out, in, base, sigma, gate, own)
    if (nv <= 2) CGS_GEMV(2);
    else if (nv <= 4) CGS_GEMV(4);
    else if (nv <= 6) CGS_GEMV(6);
    else if (nv <= 8) CGS_GEMV(8);
    else if (nv <= 10) CGS_GEMV(10);
    else if (nv <= 12) CGS_GEMV(12);
    else CGS_GEMV(0);
#undef CGS_GEMV
}
void launch_gemv(int prec, const Tables& t, const DenseLaunch& d, int adj, int out, int in, int base,
                 double sigma, int gate, int own, hipStream_t st) {
    if (prec == 0) gemv<double>(t, d, adj, out, in, base, sigma, gate, own, st);
    else gemv<float>(t, d, adj, out, in, base, sigma, gate, own, st);
}
void launch_cg_init(int prec, const Tables& t, int z, int r, int p, int q, int h, int have_q,
                    double zeta, double rate, double floor_, int cg_max, int gate, hipStream_t st) {
    CGS_DISPATCH(prec, k_cg_init, t.nx_tiles, VEC_NT, st, t, z, r, p, q, h, have_q, gate, t.xpart, 4);
    k_finalize<<<t.ninst, VEC_NT, 0, st>>>(t, FIN_CG_INIT, gate, FinArgs{zeta, rate, floor_, cg_max, 0});
}
void launch_cg_start(int prec, const Tables& t, int z, int r, int p, int q, int h, int gate, hipStream_t st) {
    CGS_DISPATCH(prec, k_cg_init, t.nx_tiles, VEC_NT, st, t, z, r, p, q, h, 1, gate, t.spart, 2);
}
void launch_cg_dot(int prec, const Tables& t, int p, int q, int r, int it, int gate, hipStream_t st) {
    CGS_DISPATCH(prec, k_cg_dot, t.nx_tiles, VEC_NT, st, t, p, q, r, it, gate);
}
void launch_cg_update(int prec, const Tables& t, int z, int r, int p, int q, int it, int cg_max,
                      int gate, int track, hipStream_t st, int folded, int last, CgStart cs) {
    // the update's own gate is the phase test of the CG gate plus the mark of k_cg_dot
    const int g = gate == G_ADMM_CG ? G_ADMM : gate == G_SETUP_CG ? G_SETUP : G_ALL;
    CGS_DISPATCH(prec, k_cg_update, t.nx_tiles + (track ? t.ny_tiles : 0), VEC_NT, st, t, z, r, p, q,
                 it, cg_max, g, track, folded, last, cs);
}
void launch_snapshot(int prec, const Tables& t, int restore, hipStream_t st) {
    CGS_DISPATCH(prec, k_snapshot, t.nx_tiles + t.ny_tiles, VEC_NT, st, t, restore);
}
void launch_wy(int prec, const Tables& t, int gate, hipStream_t st) {
    CGS_DISPATCH(prec, k_wy, t.ny_tiles, VEC_NT, st, t, gate);
}
void launch_project(int prec, const Tables& t, double alpha, hipStream_t st) {
    CGS_DISPATCH(prec, k_project, t.nx_tiles + t.ny_tiles, VEC_NT, st, t, alpha);
}
void launch_resid(int prec, const Tables& t, double eps, int max_iters, int gate, hipStream_t st) {
    CGS_DISPATCH(prec, k_resid, t.nx_tiles + t.ny_tiles, VEC_NT, st, t, eps, max_iters, gate);
    k_finalize<<<t.ninst, VEC_NT, 0, st>>>(t, FIN_RESID, gate, FinArgs{eps, 0, 0, max_iters, 0});
}
void launch_reset(int prec, const Tables& t, int only, hipStream_t st) {
    CGS_DISPATCH(prec, k_reset, t.nx_tiles + t.ny_tiles, VEC_NT, st, t, only);
}
void launch_norms(int prec, const Tables& t, int gate, hipStream_t st) {
    CGS_DISPATCH(prec, k_norms, t.nx_tiles + t.ny_tiles, VEC_NT, st, t, gate);
    k_finalize<<<t.ninst, VEC_NT, 0, st>>>(t, FIN_NORMS, gate, FinArgs{0, 0, 0, 0, 0});
}
void launch_eta(int prec, const Tables& t, hipStream_t st) {
    CGS_DISPATCH(prec, k_eta, t.nx_tiles + t.ny_tiles, VEC_NT, st, t);
    k_finalize<<<t.ninst, VEC_NT, 0, st>>>(t, FIN_ETA, G_SETUP, FinArgs{0, 0, 0, 0, 0});
}
void launch_fill(int prec, const Tables& t, int is_y, int kind, double v, int gate,
                 hipStream_t st) {
    CGS_DISPATCH(prec, k_fill, is_y ? t.ny_tiles : t.nx_tiles, VEC_NT, st, t, is_y, kind, v, gate);
}
void launch_copy(int prec, const Tables& t, int is_y, int dst, int src, int gate, hipStream_t st) {
    CGS_DISPATCH(prec, k_copy, is_y ? t.ny_tiles : t.nx_tiles, VEC_NT, st, t, is_y, dst, src, gate);
}
void launch_extract(int prec, const InstDesc* inst_dev, int inst, int what, int64_t off,
                    int64_t len, double* out64, hipStream_t st) {
    CGS_DISPATCH(prec, k_extract, flat_grid(len, 256), 256, st, inst_dev, inst, what, off, len,
                 out64);
}
void launch_extract_point(int prec, const InstDesc* inst_dev, int inst, int want, int64_t n, int64_t m, double* out,
                          hipStream_t st) {
    const int64_t len = (want & 1) ? std::max(n, (want & 6) ? m : 0) : m;
    const dim3 g((unsigned)flat_grid(len, 256), (unsigned)((want & 1) + ((want >> 1) & 1) + ((want >> 2) & 1)));
    if (prec == 0) k_extract_point<double><<<g, 256, 0, st>>>(inst_dev, inst, want, out);
    else k_extract_point<float><<<g, 256, 0, st>>>(inst_dev, inst, want, out);
}
void launch_put_data(int prec, const double* src, char* base, int64_t n, int64_t m, int64_t nxs, int64_t nys,
                     hipStream_t st) {
    CGS_DISPATCH(prec, k_put_data, flat_grid(2 * (n + m), 256), 256, st, src, base, n, m, nxs, nys);
}
void launch_cast(int prec, const double* src, void* dst, int64_t n, hipStream_t st) {
    if (n <= 0) return;
    if (prec == 0) k_cast<double><<<flat_grid(n, 256), 256, 0, st>>>(src, (double*)dst, n);
    else k_cast<float><<<flat_grid(n, 256), 256, 0, st>>>(src, (float*)dst, n);
}
void launch_cast_pad(int prec, const void* src, int src_dtype, int64_t lds, int64_t rows, int64_t cols,
                     void* dst, int64_t ld, hipStream_t st) {
    if (rows <= 0) return;
    const unsigned g = flat_grid(rows * ld, 256);
    if (src_dtype == 0) {
        const double* s = (const double*)src;
        if (prec == 0) k_cast_pad<double, double><<<g, 256, 0, st>>>(s, lds, rows, cols, (double*)dst, ld);
        else k_cast_pad<double, float><<<g, 256, 0, st>>>(s, lds, rows, cols, (float*)dst, ld);
    } else {
        const float* s = (const float*)src;
        if (prec == 0) k_cast_pad<float, double><<<g, 256, 0, st>>>(s, lds, rows, cols, (double*)dst, ld);
        else k_cast_pad<float, float><<<g, 256, 0, st>>>(s, lds, rows, cols, (float*)dst, ld);
    }
}
void launch_cast_transpose(int prec, const void* src, int src_dtype, int64_t lds, int64_t rows,
                           int64_t cols, void* dst, int64_t ldt, int64_t r0, hipStream_t st) {
    if (rows <= 0 || cols <= 0) return;
    dim3 grid((unsigned)((cols + 31) / 32), (unsigned)((rows + 31) / 32));
    if (src_dtype == 0) {
        const double* s = (const double*)src;
        if (prec == 0) k_cast_transpose<double, double><<<grid, 256, 0, st>>>(s, lds, rows, cols, (double*)dst, ldt, r0);
        else k_cast_transpose<double, float><<<grid, 256, 0, st>>>(s, lds, rows, cols, (float*)dst, ldt, r0);
    } else {
        const float* s = (const float*)src;
        if (prec == 0) k_cast_transpose<float, double><<<grid, 256, 0, st>>>(s, lds, rows, cols, (double*)dst, ldt, r0);
        else k_cast_transpose<float, float><<<grid, 256, 0, st>>>(s, lds, rows, cols, (float*)dst, ldt, r0);
    }
}

int fail(int code, const char* fmt, ...);

// Output of k_dense_rowsq: a fixed device array (no allocation call), one
// user at a time per process (the mutex), addressed through
// hipGetSymbolAddress on the current device.
namespace {
constexpr int64_t ROWSQ_CHUNK = 65536;
__device__ double g_rowsq[ROWSQ_CHUNK];
__device__ int g_rowsq_bad;
std::mutex g_rowsq_mu;
}  // namespace

int dense_frob2_device(const void* a, int dtype, int64_t rows, int64_t cols, int64_t lda, double* frob2) {
    std::lock_guard<std::mutex> lock(g_rowsq_mu);
    double* out = nullptr;
    int* bad = nullptr;
    hipError_t e = hipGetSymbolAddress((void**)&out, HIP_SYMBOL(g_rowsq));
    if (e == hipSuccess) e = hipGetSymbolAddress((void**)&bad, HIP_SYMBOL(g_rowsq_bad));
    if (e != hipSuccess) return fail(CGS_EHIP, "hipGetSymbolAddress failed: %s", hipGetErrorString(e));
    std::vector<double> host((size_t)std::min<int64_t>(rows, ROWSQ_CHUNK));
    int flag = 0;
    e = hipMemcpy(bad, &flag, sizeof(int), hipMemcpyHostToDevice);
    double s = 0.0;
    for (int64_t r0 = 0; e == hipSuccess && r0 < rows; r0 += ROWSQ_CHUNK) {
        const int64_t nr = std::min(ROWSQ_CHUNK, rows - r0);
        const unsigned g = (unsigned)((nr + 255) / 256);
        if (dtype == 0) k_dense_rowsq<double><<<g, 256, 0, 0>>>((const double*)a, lda, r0, nr, cols, out, bad);
        else k_dense_rowsq<float><<<g, 256, 0, 0>>>((const float*)a, lda, r0, nr, cols, out, bad);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipMemcpy(host.data(), out, (size_t)nr * sizeof(double), hipMemcpyDeviceToHost);
        for (int64_t i = 0; e == hipSuccess && i < nr; ++i) s += host[(size_t)i];
    }
    if (e == hipSuccess) e = hipMemcpy(&flag, bad, sizeof(int), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return fail(CGS_EHIP, "dense block check failed: %s", hipGetErrorString(e));
    if (flag) return fail(CGS_EINVAL, "the dense block has a non-finite entry");
    *frob2 = s;
    return CGS_OK;
}
void launch_cast_back(int prec, const void* src, double* dst, int64_t n, hipStream_t st) {
    if (n <= 0) return;
    if (prec == 0) k_cast_back<double><<<flat_grid(n, 256), 256, 0, st>>>((const double*)src, dst, n);
    else k_cast_back<float><<<flat_grid(n, 256), 256, 0, st>>>((const float*)src, dst, n);
}
void launch_gather_scalars(const InstDesc* insts, int ninst, double* out, hipStream_t st) {
    if (ninst > 0) k_gather_scalars<<<flat_grid((int64_t)ninst * NSC, 256), 256, 0, st>>>(insts, ninst, out);
}
void launch_set_scalar(const InstDesc* insts, int inst, int slot, double v, hipStream_t st) {
    k_set_scalar<<<1, 64, 0, st>>>(insts, inst, slot, v);
}

}  // namespace cgs
