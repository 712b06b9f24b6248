// FP32 convolution tiles by FFT (overlap-save), for kernels of up to FFT_KMAX taps.
//
// The correlation form out[o] = sum_t w[t] in[o + off + t] of A x and A^T y
// (taps w of length k, zero beyond) is, for a window u[p] = in[o0 + off + p]
// of FFT_L = L inputs, the circular correlation of u with w at the positions
// p < B = L - k + 1, where no product wraps around.  The circular correlation
// is IDFT(DFT(u) . conj(DFT(w))); conj(DFT(w)) is computed once per block and
// direction when the operator is uploaded.  w is real, so the correlation maps
// real inputs to real outputs: two windows (outputs o0.. and o0 + B..) travel
// as the real and imaginary parts of one complex transform, and the real and
// imaginary parts of the result are their outputs.  The inverse transform is a
// forward one on the conjugate.
//
// Transforms: L = 2048 points in LDS, 256 threads, Stockham self-sorting
// stages of radix 8, 8, 8 and 4 (Govindaraju et al., "High performance
// discrete Fourier transforms on graphics processors", SC 2008); each thread
// keeps the 8 values of its butterflies in registers; the twiddles come from a
// table of roots of unity (sincospi) that each workgroup copies to LDS first.  One workgroup per two output blocks (2B outputs).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "kernels.hpp"
#include "device_common.hpp"

namespace cgs {

namespace {

constexpr int FT = 256;   // threads per transform
static_assert(FFT_L == 2048 && FT * 8 == FFT_L, "transform shape");

struct cf {
    float x, y;
};
DEVI cf cmul(cf a, cf b) { return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
DEVI cf cadd(cf a, cf b) { return {a.x + b.x, a.y + b.y}; }
DEVI cf csub(cf a, cf b) { return {a.x - b.x, a.y - b.y}; }
DEVI cf mul_mi(cf a) { return {a.y, -a.x}; }   // times -i

// 4- and 8-point DFTs (e^{-2 pi i n k / R}) in place, natural order
DEVI void dft4(cf* v) {
    const cf a0 = cadd(v[0], v[2]), a1 = csub(v[0], v[2]);
    const cf a2 = cadd(v[1], v[3]), a3 = mul_mi(csub(v[1], v[3]));
    v[0] = cadd(a0, a2);
    v[2] = csub(a0, a2);
    v[1] = cadd(a1, a3);
    v[3] = csub(a1, a3);
}
DEVI void dft8(cf* v) {
    cf e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft4(e);
    dft4(o);
    const float h = 0.70710678118654752f;
    const cf w1 = {h * (o[1].x + o[1].y), h * (o[1].y - o[1].x)};   // o1 e^{-i pi/4}
    const cf w2 = mul_mi(o[2]);                                     // o2 e^{-i pi/2}
    const cf w3 = {h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y)};  // o3 e^{-3i pi/4}
    v[0] = cadd(e[0], o[0]);
    v[4] = csub(e[0], o[0]);
    v[1] = cadd(e[1], w1);
    v[5] = csub(e[1], w1);
    v[2] = cadd(e[2], w2);
    v[6] = csub(e[2], w2);
    v[3] = cadd(e[3], w3);
    v[7] = csub(e[3], w3);
}
// The transform's LDS array is padded by one entry per 32: the radix-8
// stores of a stage hit addresses 8 or 64 entries apart across the lanes of a
// wave, which without padding fall into the same few LDS banks.
constexpr int LDS_L = FFT_L + FFT_L / 32;
DEVI int lp(int i) { return i + (i >> 5); }

// Twiddle factors e^{-2 pi i m / FFT_L}, stored per stage in the order the
// lanes read them: entry (r - 1) * Ns + k holds the factor of butterfly input
// r for k = thread % Ns, so the lanes of a wave read consecutive entries (a
// table indexed by m would put the lanes of one stage 32 or 256 bytes apart,
// in the same few LDS banks).  Stages Ns = 8 and 64 (radix 8, m = r k FFT_L /
// (8 Ns)) and the radix-4 stage (m = r j, j < 512); every entry is the value
// the m-indexed table would hold.
constexpr int TW8 = 0, TW64 = 7 * 8, TW512 = TW64 + 7 * 64, TW_N = TW512 + 3 * 512;
DEVI int tw_index(int e) {   // entry -> m
    if (e < TW64) return ((e / 8 + 1) * (e % 8) * (FFT_L / 64)) & (FFT_L - 1);
    if (e < TW512) return (((e - TW64) / 64 + 1) * ((e - TW64) % 64) * (FFT_L / 512)) & (FFT_L - 1);
    return (((e - TW512) / 512 + 1) * ((e - TW512) % 512)) & (FFT_L - 1);
}
// The table's values, in device memory (one copy per GPU).  k_conv_spectrum, which an
// operator's upload runs on its device ahead of every product, computes and stores those
// that are not there yet (still zero: once there, no entry is written again).  A workgroup of
// a product copies them to LDS beside its window loads; computing them there (eight
// sincospi per thread) takes 0.7 us of a small launch (n = 20011, k = 201: 7.8 us, with the
// table 7.1) and up to 1.2 at n = 2^20 (A 11.3 and 10.1, A^T 9.8 and 9.3).
__device__ float2 g_twiddles[TW_N];
constexpr int TW_PER = (TW_N + FT - 1) / FT;
struct TwRegs {
    float2 v[TW_PER];
    DEVI void load() {
#pragma unroll
        for (int r = 0; r < TW_PER; ++r) {
            const int e = threadIdx.x + FT * r;
            v[r] = g_twiddles[e < TW_N ? e : 0];
        }
    }
    DEVI void store(cf* tw) const {
#pragma unroll
        for (int r = 0; r < TW_PER; ++r) {
            const int e = threadIdx.x + FT * r;
            if (e < TW_N) tw[e] = {v[r].x, v[r].y};
        }
    }
};
// v[r] *= factor (r - 1) of the stage table `t` (stride n), r = 1 .. R-1
template <int R>
DEVI void twiddle(cf* v, const cf* t, int n) {
#pragma unroll
    for (int r = 1; r < R; ++r) v[r] = cmul(v[r], t[(r - 1) * n]);
}

// Forward DFT of the 2048 values x[t + 256 r] that thread t holds in v[r].
// On return thread t holds X[j + 512 r] (r = 0..3) in v[0..3] for j = t and
// in v[4..7] for j = t + 256.  lds: LDS_L entries (padded, lp); tw: the twiddle table (filled
// before a barrier the first stage passes); ends with a barrier.
DEVI void fft2048(cf* v, cf* lds, const cf* tw) {
    const int t = threadIdx.x;
    dft8(v);   // stage Ns = 1: outputs to 8 t + r
#pragma unroll
    for (int r = 0; r < 8; ++r) lds[lp(8 * t + r)] = v[r];
    __syncthreads();
#pragma unroll
    for (int Ns = 8; Ns <= 64; Ns *= 8) {
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = lds[lp(t + FT * r)];
        const int k = t % Ns;
        twiddle<8>(v, tw + (Ns == 8 ? TW8 : TW64) + k, Ns);
        dft8(v);
        __syncthreads();
        const int base = (t / Ns) * Ns * 8 + k;
#pragma unroll
        for (int r = 0; r < 8; ++r) lds[lp(base + r * Ns)] = v[r];
        __syncthreads();
    }
    // stage Ns = 512, radix 4: butterflies t and t + 256
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int j = t + FT * h;
        cf* w = v + 4 * h;
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = lds[lp(j + 512 * r)];
        twiddle<4>(w, tw + TW512 + j, 512);
        dft4(w);
    }
    __syncthreads();
}

// The identity blocks that reach a workgroup's outputs, in table order: outputs at
// offsets [lo, hi) from its first one (output vector position gw) take the input
// at off + offset.  One lane per block reads the table while the window's loads
// are in flight; walked where they are used, the blocks' records were dependent
// memory round trips (six blocks: 16.7 us per right-hand side launch, two: 11.8).
struct IdRec {
    int lo, hi;   // (lo >= hi: none)
    int64_t off;
    double scale;
};
DEVI IdRec id_rec(const IdBlock& ib, int adj, int64_t gw, int nout) {
    const int64_t r0 = adj ? ib.col0 : ib.row0, c0 = adj ? ib.row0 : ib.col0;
    const int64_t rl = r0 - gw, rh = r0 + ib.len - gw;   // the block's outputs, clamped to [0, nout)
    IdRec r;
    r.lo = rl < 0 ? 0 : rl > nout ? nout : (int)rl;
    r.hi = rh > nout ? nout : rh < 0 ? 0 : (int)rh;
    r.off = c0 - r0 + gw;
    r.scale = ib.scale;
    return r;
}
struct IdList {
    static constexpr int N = 64;
    IdRec rec[N];   // those of the instance's first N blocks with outputs here
    int n, more;    // how many, and the blocks past the first N
    DEVI IdRec at(const Tables& tb, const InstDesc& d, int adj, int64_t gw, int nout, int b) const {
        return b < n ? rec[b] : id_rec(tb.ids[d.id0 + N + (b - n)], adj, gw, nout);
    }
};
// (by the first wave; a barrier follows before the list is read)
DEVI void id_list(const Tables& tb, const InstDesc& d, int adj, int64_t gw, int nout, IdList& l) {
    const int lane = threadIdx.x, nb = d.id1 - d.id0;
    IdRec r{0, 0, 0, 0.0};
    if (lane < nb) r = id_rec(tb.ids[d.id0 + lane], adj, gw, nout);
    const bool hit = r.lo < r.hi;
    const unsigned long long m = __ballot(hit);
    if (hit) l.rec[__popcll(m & ((1ull << lane) - 1))] = r;
    if (lane == 0) {
        l.n = __popcll(m);
        l.more = nb > IdList::N ? nb - IdList::N : 0;
    }
}

// Four consecutive elements at any element alignment
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
// the identity block's inputs for outputs o .. o + 3 (0 where it has none)
DEVI f32x4 id_load(gptr<const float> iw, int o, const IdRec& ib) {
    f32x4 l = {0.0f, 0.0f, 0.0f, 0.0f};
    if (o >= ib.lo && o + 4 <= ib.hi) {
        const f32x4u q = *(gptr<const f32x4u>)(iw + o);
#pragma unroll
        for (int e = 0; e < 4; ++e) l[e] = q[e];
    } else if (o < ib.hi && o + 4 > ib.lo) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (o + e >= ib.lo && o + e < ib.hi) l[e] = iw[o + e];
    }
    return l;
}
// stores v[e] at p[e] for the outputs o + e in [lo, hi); out4: p 16-byte aligned
template <typename V>
DEVI void out4_as(gptr<float> p, int o, int lo, int hi, const f32x4& v) {
    if (o >= lo && o + 4 <= hi) {
        *(gptr<V>)p = v;
    } else if (o < hi && o + 4 > lo) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (o + e >= lo && o + e < hi) p[e] = v[e];
    }
}
DEVI void out4(gptr<float> p, int o, int lo, int hi, const f32x4& v) { out4_as<f32x4>(p, o, lo, hi, v); }
DEVI void out4u(gptr<float> p, int o, int lo, int hi, const f32x4& v) { out4_as<f32x4u>(p, o, lo, hi, v); }

// Partial sums of a CG step folded into an A^T launch:
//   fold 1: ||r||^2, ||h||^2;  fold 2: <p, q>, ||r||^2, <r, q>, ||q||^2
struct Fold4 {
    double a, b, c, d;
};
// The workgroup's partials of a folded CG step (every thread calls this): two or four.
template <int FOLD>
DEVI void fold_partials(double* part, const Fold4& f, double* red) {
    double v[4] = {f.a, f.b, f.c, f.d};
    block_sum4<FT>(v, red);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int j = 0; j < 2 * FOLD; ++j) part[2 * FOLD * (int64_t)blockIdx.x + j] = v[j];
    }
}

}  // namespace

// conj(DFT(w zero-padded to FFT_L)) of k correlation-order taps
__global__ __launch_bounds__(FT) void k_conv_spectrum(const float* w, int k, float2* spec) {
    __shared__ cf lds[LDS_L];
    __shared__ cf tw[TW_N];
    const int t = threadIdx.x;
    TwRegs twr;
    twr.load();
#pragma unroll
    for (int r = 0; r < TW_PER; ++r) {
        const int e = t + FT * r;
        if (twr.v[r].x != 0.0f || twr.v[r].y != 0.0f) continue;   // (no root of unity is 0)
        float sn, cs;
        sincospif(-2.0f * (float)tw_index(e < TW_N ? e : 0) / (float)FFT_L, &sn, &cs);
        twr.v[r] = make_float2(cs, sn);
        if (e < TW_N) g_twiddles[e] = twr.v[r];
    }
    twr.store(tw);
    cf v[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int i = t + FT * r;
        v[r] = {i < k ? w[i] : 0.0f, 0.0f};
    }
    fft2048(v, lds, tw);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) spec[t + FT * h + 512 * r] = make_float2(v[4 * h + r].x, -v[4 * h + r].y);
}

DEVI void conv_windows(cf (&v)[8], cf* lds, const cf* tw, const void* spec) {
    const int t = threadIdx.x;
    fft2048(v, lds, tw);
    // product with conj(DFT(w)), conjugated: the inverse is a forward transform.
    // The thread holds X[t + 256 (h + 2 r)] in v[4 h + r], which is exactly
    // the set x[t + 256 r'] the next transform's first stage takes from it:
    // the products only change register, v'[r'] = p[4 (r' % 2) + r' / 2]
    // (no exchange through LDS; the transform ended with a barrier).
    gptr<const float> sp = (gptr<const float>)spec;   // interleaved (re, im)
    cf pr[8];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = t + FT * h + 512 * r;
            const cf p = cmul(v[4 * h + r], cf{sp[2 * j], sp[2 * j + 1]});
            pr[h + 2 * r] = {p.x, -p.y};
        }
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = pr[r];
    fft2048(v, lds, tw);
}

template <int FOLD>
__global__ __launch_bounds__(FT) void k_conv_fft(Tables tb, ConvLaunch cl, int adj, int out, int in, int base,
                                                 double sigma, int gate) {
    __shared__ cf lds[LDS_L];
    __shared__ cf tw[TW_N];
    __shared__ double red[4 * (FT / 64)];
    __shared__ IdList ids;
    Fold4 f{0.0, 0.0, 0.0, 0.0};
    int bid = (int)blockIdx.x;
    if (FOLD == 0 && cl.pair) {
        // two applies in one launch: the second operand set's transform
        // workgroups follow the first set's, then both sets' initialisation
        // tiles in the same order
        bool second;
        if (bid < 2 * cl.nftiles) {
            second = bid >= cl.nftiles;
            bid -= second ? cl.nftiles : 0;
        } else {
            int w = bid - 2 * cl.nftiles;
            second = w >= cl.ninit;
            w -= second ? cl.ninit : 0;
            bid = cl.nftiles + w;
        }
        if (second) {
            out = cl.out2;
            in = cl.in2;
            base = cl.base2;
        }
    }
    // Workgroups past the transforms write the output elements that no convolution
    // owns (base and identity blocks alone): an initialisation tile goes through
    // the same epilogue with no sums.  Element by element, each behind the last
    // one's loads, such a tile was the longest chain of most launches.
    const int t = threadIdx.x;
    const bool init = bid >= cl.nftiles;
    const VecTile it = init ? cl.init[bid - cl.nftiles].tile() : VecTile{};
    const ConvTile tl = init ? ConvTile{it.inst, 0, 0} : cl.ftiles[bid];
    const InstDesc d = tb.inst[tl.inst];
    ConvBlock cb{};
    if (!init) cb = cl.blocks[tl.blk];   // (loaded beside the instance, ahead of the gate)
    if (!gate_ok(scal(d), gate)) return;
    if (FOLD == 2 && (int)blockIdx.x == d.cp0 && t == 0) scal(d)[SC_CGRUN] = (double)cl.fit;
    const int64_t g0 = adj ? cb.col0 : cb.row0, oa = tl.start;
    const int B = init ? 0 : FFT_L - (int)cb.k + 1;   // outputs per window
    // the workgroup's outputs: nlim of them from position gw of the output vector
    const int64_t gw = init ? it.start : g0 + oa;
    int nlim = it.len;
    cf v[8];
    if (!init) {
        const int64_t n_out = adj ? cb.n_in : cb.n_in + cb.k - 1;
        const int64_t n_in = adj ? cb.n_in + cb.k - 1 : cb.n_in;
        nlim = n_out - oa < 2 * (int64_t)B ? (int)(n_out - oa) : 2 * B;
        gptr<const float> src = adj ? yvec<float>(d, in) + cb.row0 : xvec<float>(d, in) + cb.col0;
        // the pair's inputs as 32-bit offsets q = p (window a) and B + p (window b)
        // from input position i0; valid offsets [qlo, qhi)
        const int64_t i0 = adj ? oa : oa - (cb.k - 1);
        const int qlo = i0 < 0 ? (int)-i0 : 0;
        const int qhi = n_in - i0 < FFT_L + B ? (int)(n_in - i0) : FFT_L + B;
        gptr<const float> sw = src + i0;
        TwRegs twr;
        twr.load();
        // (no load behind a branch: at the block's ends positions are clamped to
        // valid ones, and what was loaded there is dropped)
        float wa[8], wb[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int p = t + FT * r;
            wa[r] = sw[min(max(p, qlo), qhi - 1)];
            wb[r] = sw[min(max(B + p, qlo), qhi - 1)];
        }
        if (t < 64) id_list(tb, d, adj, gw, nlim, ids);   // (while the window's loads are in flight)
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int p = t + FT * r;
            v[r] = {(p >= qlo && p < qhi) ? wa[r] : 0.0f, (B + p >= qlo && B + p < qhi) ? wb[r] : 0.0f};
        }
        twr.store(tw);
        conv_windows(v, lds, tw, adj ? cb.s_adj : cb.s_fwd);
    } else if (t < 64) {
        id_list(tb, d, adj, gw, nlim, ids);
    }
    // conj(result) / L: real part = window a, imaginary part = window b.  Output o
    // (window a: o = j, window b: o = B + j) has position gw + o in the output
    // vector.  They pass through LDS so that a thread's
    // epilogue elements are whole aligned 16-byte chunks of the vectors (LDS entry
    // al + o, the chunk grid's offset al): in the transform's order, 256 apart,
    // every vector cost 16 four-byte accesses a thread, and the epilogue took half
    // of a right-hand side launch (14 of 28 thousand cycles).
    const double s = init ? 0.0 : sigma * cb.scale / (double)FFT_L;
    const bool own = init || ((cb.own >> adj) & 1);
    const int al = (int)(gw & 3);
    float* res = reinterpret_cast<float*>(lds);
    static_assert(2 * LDS_L >= 2 * FFT_L + 4, "outputs in the transform's LDS");
    if (!init) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = t + FT * h + 512 * r;
                if (j < B) {
                    res[al + j] = v[4 * h + r].x;
                    res[al + B + j] = -v[4 * h + r].y;
                }
            }
    }
    __syncthreads();
    const int nid = own ? ids.n + ids.more : 0;   // identity blocks to look at
    gptr<float> xo = (adj ? xvec<float>(d, out) : yvec<float>(d, out)) + (gw - al);
    const int kb = own ? base : out;   // what the sums are added to (-1: nothing)
    gptr<const float> xb = kb >= 0 ? (adj ? xvec<float>(d, kb) : yvec<float>(d, kb)) + (gw - al) : nullptr;
    gptr<const float> isrc = adj ? yvec<float>(d, in) : xvec<float>(d, in);
    const int nchunk = (al + nlim + 3) / 4;
    constexpr int NQ = 4;   // chunks of a thread whose loads are issued together
    for (int c0 = t; c0 < nchunk; c0 += FT * NQ) {
        // every load is at a position inside its (padded) vector: chunks past
        // the last one load the first
        int o0[NQ];   // the chunk's first output (may be < 0)
        f32x4 bl[NQ], sv[NQ], kv[NQ], rv[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int c = c0 + FT * q;
            const int k4 = 4 * (c < nchunk ? c : 0);
            o0[q] = c < nchunk ? 4 * c - al : nlim;
            sv[q] = init ? f32x4{0.0f, 0.0f, 0.0f, 0.0f} : *reinterpret_cast<const f32x4*>(res + k4);
            if (xb != nullptr) bl[q] = *(gptr<const f32x4>)(xb + k4);
            if (FOLD == 1) kv[q] = *(gptr<const f32x4>)(xvec<float>(d, cl.fq) + (gw - al) + k4);
            if (FOLD == 2) {
                kv[q] = cl.fp == kb ? bl[q] : *(gptr<const f32x4>)(xvec<float>(d, cl.fp) + (gw - al) + k4);
                rv[q] = cl.fr == cl.fp ? kv[q] : *(gptr<const f32x4>)(xvec<float>(d, cl.fr) + (gw - al) + k4);
            }
        }
        double bv[NQ][4];   // base + identity blocks, in table order
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) bv[q][e] = xb != nullptr ? (double)bl[q][e] : 0.0;
        for (int b = 0; b < nid; ++b) {
            const IdRec ib = ids.at(tb, d, adj, gw, nlim, b);
            if (ib.lo >= ib.hi) continue;
            const double w = sigma * ib.scale;
            gptr<const float> iw = isrc + ib.off;
            f32x4 l[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) l[q] = id_load(iw, o0[q], ib);
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (o0[q] + e >= ib.lo && o0[q] + e < ib.hi) bv[q][e] += w * (double)l[q][e];
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            f32x4 val;
            double g[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                val[e] = (float)(bv[q][e] + s * (double)sv[q][e]);
                g[e] = (o0[q] + e >= 0 && o0[q] + e < nlim) ? 1.0 : 0.0;   // the output exists
            }
            const int k4 = o0[q] + al;
            if (FOLD == 1) {
                // h = value; r = h - K z (and p = r when fp >= 0) written instead of h
                f32x4 rr;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double hd = (double)val[e];
                    rr[e] = (float)(hd - (double)kv[q][e]);
                    if (g[e] != 0.0) {
                        f.a += (double)rr[e] * (double)rr[e];
                        f.b += hd * hd;
                    }
                }
                out4(xvec<float>(d, cl.fr) + (gw - al) + k4, o0[q], 0, nlim, rr);
                if (cl.fp >= 0) out4(xvec<float>(d, cl.fp) + (gw - al) + k4, o0[q], 0, nlim, rr);
                sv[q] = rr;
            } else {
                out4(xo + k4, o0[q], 0, nlim, val);
                if (FOLD == 2) {
                    // q = value; partials <p, q>, ||r||^2, <r, q>, ||q||^2.  p is the
                    // launch's base (q = p + A^T A p), already loaded; r is p's vector
                    // in a step's first iteration (p = r)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const double pd = (double)kv[q][e], rd = (double)rv[q][e], qd = (double)val[e];
                        if (g[e] == 0.0) continue;
                        f.a = fma(pd, qd, f.a);
                        f.b = fma(rd, rd, f.b);
                        f.c = fma(rd, qd, f.c);
                        f.d = fma(qd, qd, f.d);
                    }
                }
            }
        }
        if (FOLD == 1 && cl.idrows) {
            // A p's identity rows for p = r: A's block maps X column col0 + i
            // to Y row row0 + i (ConvLaunch::idrows)
            gptr<float> yt = yvec<float>(d, cl.idrows - 1);
            for (int b = 0; b < nid; ++b) {
                const IdRec ib = ids.at(tb, d, adj, gw, nlim, b);
                gptr<float> yw = yt + ib.off;
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    f32x4 y;
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] = (float)(0.0 + ib.scale * (double)sv[q][e]);
                    out4u(yw + o0[q], o0[q], ib.lo, ib.hi, y);
                }
            }
        }
    }
    if constexpr (FOLD != 0) fold_partials<FOLD>(cl.part, f, red);
}

void launch_conv_spectrum(const void* w, int64_t k, void* spec, hipStream_t st) {
    k_conv_spectrum<<<1, FT, 0, st>>>((const float*)w, (int)k, (float2*)spec);
}

void launch_conv_fft(const Tables& t, const ConvLaunch& c, int adj, int out, int in, int base, double sigma,
                     int gate, hipStream_t st) {
    const int grid = (c.nftiles + c.ninit) * (c.pair && c.fold == 0 ? 2 : 1);
    if (grid <= 0) return;
    if (c.fold == 1) k_conv_fft<1><<<grid, FT, 0, st>>>(t, c, adj, out, in, base, sigma, gate);
    else if (c.fold == 2) k_conv_fft<2><<<grid, FT, 0, st>>>(t, c, adj, out, in, base, sigma, gate);
    else k_conv_fft<0><<<grid, FT, 0, st>>>(t, c, adj, out, in, base, sigma, gate);
}

}  // namespace cgs
