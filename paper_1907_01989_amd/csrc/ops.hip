// Bandwidth-bound kernels on the sliced (C8) layout: depthwise convolution,
// element-wise add / activation, global average pool, softmax, concat,
// bilinear resize (optionally fused with the per-pixel argmax), argmax, and
// the conversions between NHWC graph I/O and the sliced layout.
//
// Thread order follows the paper's observation (Sec. 4.1) that neighbouring
// threads should read neighbouring cache lines: consecutive lanes take
// consecutive pixels of one 8-channel slice, so a wave's 16-byte loads cover
// 1 KiB of contiguous memory.
#include <cfloat>
#include <cmath>
#include <cstdint>

#include "device.h"

namespace mgi {
namespace kern {

static inline unsigned blocks_for(size_t n, int per) { return (unsigned)((n + per - 1) / per); }

// log2 of the slices of a pixel that neighbouring lanes take where a kernel
// reads or writes NHWC arrays: eight slices unless that would leave more than
// a third of the lanes past the last slice
static int nhwc_slices(int S) {
    int ls = 3;
    while (ls > 0 && ((S + (1 << ls) - 1) >> ls << ls) * 2 > S * 3) --ls;
    return ls;
}

LaunchEvents &launch_events() {
    static thread_local LaunchEvents ev;
    return ev;
}

// ---------------------------------------------------------------------------
// Depthwise 3x3 convolution, column strips.  A thread owns one output column
// of one 8-channel slice of one image and R consecutive output rows: it reads
// the (R-1)*S + 2*D + 1 input rows of its three input columns once (16 bytes
// each), and every input value feeds all the outputs whose
// window covers it, accumulating in fp32 with 16-bit taps (exact products).
// Taps outside the input read a zeroed element instead of branching, so all
// loads are issued unconditionally: all of a strip's before its first FMA, or
// one row ahead of the FMAs for the 32-byte elements of an fp32 input (too
// many registers).
// SRC: where the input lies.  0: sliced, [S][N*H*W]; consecutive lanes take
// consecutive columns, so each load instruction of a wave covers a contiguous
// run of one row.  1 (fp16), 2 (fp32): the NHWC graph input itself, rounded to
// the storage type on the way (as the conversion kernel would), C a multiple
// of 8; 2^ls consecutive lanes take the slices of one pixel and the next ones
// the next column, so with eight slices loads are whole lines of the NHWC
// array and stores eight consecutive elements of each slice.  This saves the
// conversion kernel and its pass over memory (64 x 14 x 14 x 512: fp16 6.8 +
// 8.2 -> 11.0 us, fp32 -> 11.7; one 56 x 56 x 128 image 4.1 + 4.2 -> 4.2 us).
// Launch: 1-D, thread g -> slice of its group g % 2^ls, column, strip, then
// plane (slice group * N + image); the divisions are reciprocal products with
// one correction step (divmod_fast), a few instructions instead of an integer
// division sequence each.
// ---------------------------------------------------------------------------
template <typename E, int SRC>
struct DwElem;   // one element as loaded, and as the storage type
template <typename E>
struct DwElem<E, 0> {
    h8 v;
    __device__ h8 get() const { return v; }
};
template <typename E>
struct DwElem<E, 1> {
    h8 v;
    __device__ h8 get() const {
        if (!E::bf) return v;
        float f[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) f[c] = (float)v[c];
        return E::pack(f);
    }
};
template <typename E>
struct DwElem<E, 2> {
    f4 v[2];
    __device__ h8 get() const {
        const float f[8] = {v[0][0], v[0][1], v[0][2], v[0][3], v[1][0], v[1][1], v[1][2], v[1][3]};
        return E::pack(f);
    }
};

template <typename E, int S_, int D_, int R, int SRC>
__global__ __launch_bounds__(256) void dw3_kernel(DwParams p, int nstrips, DivConsts dc) {
    constexpr int K = 3, NR = (R - 1) * S_ + (K - 1) * D_ + 1;
    constexpr bool AHEAD = SRC != 2;                       // every load first
    typedef DwElem<E, SRC> El;
    int g = blockIdx.x * 256 + threadIdx.x;
    int rest, ox, plane, strip, s, img;
    int sl = 0;
    if (SRC) {
        sl = g & ((1 << p.ls) - 1);
        g >>= p.ls;
    }
    divmod_fast(g, p.OW, dc.inv_ow, rest, ox);
    divmod_fast(rest, nstrips, dc.inv_nstrips, plane, strip);
    divmod_fast(plane, p.N, dc.inv_n, s, img);
    if (SRC) s = (s << p.ls) + sl;
    if (s >= p.S) return;
    if (SRC) plane = s * p.N + img;
    const int oy0 = strip * R;
    const El *xin = SRC ? (const El *)p.xin + (size_t)img * p.H * p.W * p.S + s
                        : (const El *)p.x + (size_t)plane * p.H * p.W;
    const int px = SRC ? p.S : 1;                          // elements between neighbouring pixels
    const h8 *wp = p.w + (size_t)s * (K * K);
    h8 w[K * K];
#pragma unroll
    for (int t = 0; t < K * K; ++t) w[t] = wp[t];
    const int iy0 = oy0 * S_ - p.pt, ix0 = ox * S_ - p.pl;
    int cx[K];
    bool cv[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        cx[k] = ix0 + k * D_;
        cv[k] = cx[k] >= 0 && cx[k] < p.W;
    }
    auto load_row = [&](int r, El *v) {
        const int iy = iy0 + r;
        const bool rv = iy >= 0 && iy < p.H;
#pragma unroll
        for (int k = 0; k < K; ++k)
            v[k] = *((rv && cv[k]) ? xin + ((size_t)iy * p.W + cx[k]) * px : (const El *)p.zero);
    };
    // accumulation per output: bias, then taps ky, kx in window order (the
    // first tap takes the bias as its addend)
    float bias[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) bias[c] = p.bias[s * 8 + c];
    float acc[R][8];
    auto row_fma = [&](int r, const El *e) {
        h8 v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = e[k].get();
#pragma unroll
        for (int ky = 0; ky < K; ++ky) {
            const int t = r - ky * D_;
            if (t >= 0 && t % S_ == 0 && t / S_ < R) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    if (ky == 0 && k == 0) E::fma8_from(acc[t / S_], bias, w[0], v[0]);
                    else E::fma8(acc[t / S_], w[ky * K + k], v[k]);
                }
            }
        }
    };
    if constexpr (AHEAD) {
        El v[NR][K];
#pragma unroll
        for (int r = 0; r < NR; ++r) load_row(r, v[r]);
#pragma unroll
        for (int r = 0; r < NR; ++r) row_fma(r, v[r]);
    } else {
        El v[2][K];
        load_row(0, v[0]);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if (r + 1 < NR) load_row(r + 1, v[(r + 1) & 1]);
            row_fma(r, v[r & 1]);
        }
    }
    // activation as one clamp: [lo, hi] = (-inf, inf), (0, inf) or (0, 6)
    const float lo = p.act == MGI_ACT_NONE ? -INFINITY : 0.0f;
    const float hi = p.act == MGI_ACT_RELU6 ? 6.0f : INFINITY;
    h8 *yout = p.y + (size_t)plane * p.OH * p.OW + ox;
#pragma unroll
    for (int o = 0; o < R; ++o) {
        if (oy0 + o >= p.OH) break;
        float q[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) q[c] = __builtin_amdgcn_fmed3f(acc[o][c], lo, hi);
        yout[(size_t)(oy0 + o) * p.OW] = E::pack(q);
    }
}

// ---------------------------------------------------------------------------
// Depthwise 5x5 convolution from LDS.  A 5x5 strip's loads are too many to
// hold in registers, and loaded a row ahead of their use they expose one
// memory latency per input row (16 x 28 x 28 x 240: 12.4 us; one output per
// thread, as the any-window kernel does, 13.8).  Here a workgroup stages the
// input rows of a band of output rows, for 2^ls slices of one image, all loads
// in flight together, with the zero padding written around them, and computes
// from there: a thread owns four channels (half an element, so that its 25
// taps fit in registers also when bf16 ones are widened to fp32) of one output
// column and R rows.  Bound by vector issue (25 * 8 FMAs per output element,
// 2.1 us of the chip's at this size) and the staging round trip before it:
// 10.2 us from the NHWC input of either type, and nothing for the conversion
// (7.5 us fp16, 10.2 fp32); 11.0 with bf16 storage (16.2); one image 4.9
// (7.7).  SRC as above.
// ---------------------------------------------------------------------------
template <typename E, int S_, int SRC>
__global__ __launch_bounds__(256) void dw5_kernel(DwParams p, DwTile q) {
    constexpr int K = 5, R = 4 / S_, NR = (R - 1) * S_ + K;
    typedef DwElem<E, SRC> El;
    extern __shared__ h8 lds[];
    const int tid = threadIdx.x, TS = 1 << p.ls;
    const int nband = q.nbands, b = blockIdx.x % nband, rest = blockIdx.x / nband;
    const int n = rest % p.N, s0 = (rest / p.N) << p.ls;
    const int nsl = min(TS, p.S - s0);
    const int oy0 = b * q.rb, rows = min(q.rb, p.OH - oy0);
    const int nrb = (rows - 1) * S_ + K, wp = q.wp;         // band: [TS][nrb][wp], first column -pl
    const int iy0 = oy0 * S_ - p.pt;
    h8 *taps = lds + TS * q.nrb * wp;                        // [TS][25]
    float *bias8 = (float *)(taps + TS * K * K);             // [TS][8]
    // taps, biases and the band; cells outside the input are zero
    for (int e = tid; e < nsl * K * K; e += 256) taps[e] = p.w[(size_t)s0 * (K * K) + e];
    if (tid < nsl * 8) bias8[tid] = p.bias[s0 * 8 + tid];
    const El *xin = SRC ? (const El *)p.xin + (size_t)n * p.H * p.W * p.S + s0
                        : (const El *)p.x + ((size_t)s0 * p.N + n) * p.H * p.W;
    const size_t xs = SRC ? 1 : (size_t)p.N * p.H * p.W;     // elements between slices
    const int px = SRC ? p.S : 1;                            // ... and between neighbouring pixels
    const int cells = nsl * nrb * wp;
    constexpr int U = SRC == 2 ? 4 : 8;
    for (int e0 = tid; e0 < cells; e0 += 256 * U) {
        El v[U];
        int at[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = e0 + u * 256;
            int sl, r, c, t;
            if (SRC) {                                       // slice fastest
                divmod_u16(min(e, cells - 1), nsl, q.inv_nsl[nsl == TS ? 0 : 1], t, sl);
                divmod_u16(t, wp, q.inv_wp, r, c);
            } else {                                         // column fastest
                divmod_u16(min(e, cells - 1), wp, q.inv_wp, t, c);
                divmod_u16(t, nrb, rows == q.rb ? q.inv_nrb[0] : q.inv_nrb[1], sl, r);
            }
            const int iy = iy0 + r, ix = c - p.pl;
            const bool in = iy >= 0 && iy < p.H && ix >= 0 && ix < p.W;
            v[u] = *(in ? xin + xs * sl + ((size_t)iy * p.W + ix) * px : (const El *)p.zero);
            at[u] = e < cells ? (sl * nrb + r) * wp + c : -1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (at[u] >= 0) lds[at[u]] = v[u].get();
    }
    __syncthreads();

    const float lo = p.act == MGI_ACT_NONE ? -INFINITY : 0.0f;
    const float hi = p.act == MGI_ACT_RELU6 ? 6.0f : INFINITY;
    const int nstrip = (rows + R - 1) / R, ntask = nsl * nstrip * p.OW * 2;
    for (int t0 = tid; t0 < ntask; t0 += 256) {
        const int half = t0 & 1;
        int t, ox, sl, strip;
        divmod_u16(t0 >> 1, p.OW, q.inv_ow, t, ox);
        divmod_u16(t, nstrip, rows == q.rb ? q.inv_strip[0] : q.inv_strip[1], sl, strip);
        const h4 *w4 = (const h4 *)(taps + sl * (K * K)) + half;
        h4 w[K * K];
#pragma unroll
        for (int i = 0; i < K * K; ++i) w[i] = w4[2 * i];
        const f4 b4 = *((const f4 *)(bias8 + sl * 8) + half);
        const float bias[4] = {b4[0], b4[1], b4[2], b4[3]};
        float acc[R][4];
        const h4 *row = (const h4 *)(lds + (sl * nrb + strip * R * S_) * wp + ox * S_) + half;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            // (rows past the band belong to outputs past it, never stored: they
            // read the band's last row)
            const h4 *rp = row + (size_t)min(r, nrb - 1 - strip * R * S_) * wp * 2;
            h4 v[K];
#pragma unroll
            for (int k = 0; k < K; ++k) v[k] = rp[2 * k];
#pragma unroll
            for (int ky = 0; ky < K; ++ky) {
                const int o = r - ky;
                if (o >= 0 && o % S_ == 0 && o / S_ < R) {
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        if (ky == 0 && k == 0) E::fma4_from(acc[o / S_], bias, w[0], v[0]);
                        else E::fma4(acc[o / S_], w[ky * K + k], v[k]);
                    }
                }
            }
        }
        h4 *yout = (h4 *)(p.y + (((size_t)(s0 + sl) * p.N + n) * p.OH + oy0 + strip * R) * p.OW + ox) + half;
#pragma unroll
        for (int o = 0; o < R; ++o) {
            if (strip * R + o >= rows) break;
            float z[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) z[c] = __builtin_amdgcn_fmed3f(acc[o][c], lo, hi);
            yout[(size_t)o * p.OW * 2] = E::pack4(z);
        }
    }
}

// Any window size: one thread per output pixel of one slice, fp32
// accumulation over the kh x kw window.
template <typename E>
__global__ __launch_bounds__(256) void dw_kernel(DwParams p, int tpp) {
    const int plane = blockIdx.x / tpp;
    const int pix = (blockIdx.x - plane * tpp) * 256 + threadIdx.x;
    const int ohw = p.OH * p.OW;
    if (pix >= ohw) return;
    const int s = plane / p.N;
    const int oy = pix / p.OW, ox = pix - oy * p.OW;
    const h8 *xin = p.x + (size_t)plane * p.H * p.W;
    const h8 *wt = p.w + (size_t)s * p.KH * p.KW;
    float acc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = p.bias[s * 8 + c];
    for (int ky = 0; ky < p.KH; ++ky) {
        const int iy = oy * p.sh + ky * p.dh - p.pt;
        if (iy < 0 || iy >= p.H) continue;
        for (int kx = 0; kx < p.KW; ++kx) {
            const int ix = ox * p.sw + kx * p.dw - p.pl;
            if (ix < 0 || ix >= p.W) continue;
            const h8 v = xin[(size_t)iy * p.W + ix];
            const h8 wk = wt[ky * p.KW + kx];
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[c] = fmaf(E::get(wk, c), E::get(v, c), acc[c]);
        }
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = act_apply(acc[c], p.act);
    p.y[(size_t)plane * ohw + pix] = E::pack(acc);
}

template <typename E, int S_, int D_, int R>
static hipError_t launch_dw3(DwParams p, hipStream_t st) {
    const int nstrips = (p.OH + R - 1) / R;
    p.ls = p.xin ? nhwc_slices(p.S) : 0;
    const size_t slices = ((size_t)p.S + (1 << p.ls) - 1) >> p.ls << p.ls;
    const size_t threads = (size_t)p.OW * nstrips * slices * p.N;
    if (threads > 0x7fffffffull) return hipErrorInvalidValue;
    const DivConsts dc{1.0 / p.OW, 1.0 / nstrips, 1.0 / p.N};
    const dim3 grid((unsigned)((threads + 255) / 256)), block(256);
    if (!p.xin) launch((dw3_kernel<E, S_, D_, R, 0>), grid, block, 0, st, p, nstrips, dc);
    else if (p.xin_fp16) launch((dw3_kernel<E, S_, D_, R, 1>), grid, block, 0, st, p, nstrips, dc);
    else launch((dw3_kernel<E, S_, D_, R, 2>), grid, block, 0, st, p, nstrips, dc);
    return hipGetLastError();
}

// Band of the 5x5 kernel: slices (2^ls) and output rows per workgroup.  Short
// bands of few slices repeat more of their rows and fill fewer threads, tall
// ones of many leave a compute unit one workgroup, whose loads nothing hides.
// The estimate counts, for the workgroups per compute unit, a workgroup's
// staging passes (3 each, of 256 cells, 5 where they read single slices of an
// NHWC input, 16 bytes a pixel; two workgroups' worth is not hidden) and
// computing passes (20 each, of 256 tasks), and 30 for each round of as many
// workgroups as run at a time (by LDS, and by registers five of fp16, two of
// bf16, whose taps are held as floats).  Over 20 sizes of both strides and
// types its choice is 2.4 % over the best of the twelve on average, at most
// 15 %.  (With as many slices and rows as 64 KiB and 512 workgroups allow
// 38 x 55 x 55 x 48 took 23.0 us, now 16.6; 16 x 28 x 28 x 240 11.1, now 10.2;
// bf16 8 x 28 x 28 x 240 11.6, now 7.1; stride 2, 16 x 56 x 56 x 96, 7.2, now
// 7.9.)
static DwTile dw5_tile(int N, int S, int OH, int OW, int sh, bool nhwc, bool bf16, int &ls_out) {
    const int R = 4 / sh, K = 5;
    DwTile best{};
    size_t best_cost = 0;
    for (int ls = nhwc_slices(S); ls >= 0; --ls)
        for (int rb : {R, 2 * R, 4 * R}) {
            if (rb > R && rb >= OH + R) break;
            DwTile t{};
            t.rb = rb;
            t.wp = (OW - 1) * sh + K;
            t.nrb = (rb - 1) * sh + K;
            t.nbands = (OH + rb - 1) / rb;
            const size_t TS = (size_t)1 << ls;
            t.lds = TS * ((size_t)t.nrb * t.wp + K * K) * 16 + TS * 32;
            const size_t wgs = ((size_t)S + TS - 1) / TS * N * t.nbands, cells = TS * t.nrb * t.wp;
            if (t.lds > 65536 || cells >= 65536 || wgs > 0x7fffffffull) continue;
            const size_t nsl = std::min<size_t>(TS, S), per = (wgs + 255) / 256;
            const size_t stage = (nsl * t.nrb * t.wp + 255) / 256, comp = (nsl * (rb / R) * OW * 2 + 255) / 256;
            const size_t conc = std::min<size_t>(bf16 ? 2 : 5, 163840 / t.lds);
            const size_t cost = (per * (nhwc && ls == 0 ? 5 : 3) + 6) * stage + per * comp * 20 + (per + conc - 1) / conc * 30;
            if (best.nbands == 0 || cost < best_cost) {
                best = t;
                best_cost = cost;
                ls_out = ls;
            }
        }
    return best;
}

template <typename E, int S_>
static hipError_t launch_dw5(DwParams p, DwTile t, hipStream_t st) {
    const int R = 4 / S_, last = p.OH - (t.nbands - 1) * t.rb;   // rows of the last band
    const int tail = p.S - ((p.S - 1) >> p.ls << p.ls);          // slices of the last group
    auto inv = [](int d) { return (unsigned)((0x100000000ull + d - 1) / d); };
    t.inv_wp = inv(t.wp);
    t.inv_ow = inv(p.OW);
    t.inv_nsl[0] = inv(1 << p.ls);
    t.inv_nsl[1] = inv(tail);
    t.inv_nrb[0] = inv(t.nrb);
    t.inv_nrb[1] = inv((last - 1) * p.sh + 5);
    t.inv_strip[0] = inv((t.rb + R - 1) / R);
    t.inv_strip[1] = inv((last + R - 1) / R);
    const dim3 grid((unsigned)(t.nbands * p.N * ((p.S + (1 << p.ls) - 1) >> p.ls))), block(256);
    if (!p.xin) launch((dw5_kernel<E, S_, 0>), grid, block, (unsigned)t.lds, st, p, t);
    else if (p.xin_fp16) launch((dw5_kernel<E, S_, 1>), grid, block, (unsigned)t.lds, st, p, t);
    else launch((dw5_kernel<E, S_, 2>), grid, block, (unsigned)t.lds, st, p, t);
    return hipGetLastError();
}

static bool dw3_window(int KH, int KW, int sh, int sw, int dh, int dw) {
    return KH == 3 && KW == 3 && sh == sw && dh == dw && sh >= 1 && sh <= 2 && dh >= 1 && dh <= 2;
}

static bool dw5_window(int KH, int KW, int sh, int sw, int dh, int dw) {
    return KH == 5 && KW == 5 && sh == sw && dh == 1 && dw == 1 && sh >= 1 && sh <= 2;
}

bool depthwise_reads_nhwc(int KH, int KW, int sh, int sw, int dh, int dw, int N, int S, int OH, int OW) {
    int ls;
    return dw3_window(KH, KW, sh, sw, dh, dw) ||
           (dw5_window(KH, KW, sh, sw, dh, dw) && dw5_tile(N, S, OH, OW, sh, true, false, ls).nbands > 0);
}

hipError_t launch_depthwise(const DwParams &p, int rows, hipStream_t st) {
    const int ohw = p.OH * p.OW;
    if (ohw <= 0 || p.N <= 0 || p.S <= 0) return hipSuccess;
    if (dw3_window(p.KH, p.KW, p.sh, p.sw, p.dh, p.dw)) {
        // output rows per thread: 4 at stride 1, 2 at stride 2 unless chosen
        const int R = rows > 0 ? rows : (p.sh == 1 ? 4 : 2);
#define MGI_DW_CASE(S_, D_, R_) \
        if (p.sh == S_ && p.dh == D_ && R == R_) \
            return p.bf16 ? launch_dw3<BF16, S_, D_, R_>(p, st) : launch_dw3<F16, S_, D_, R_>(p, st);
        MGI_DW_CASE(1, 1, 1) MGI_DW_CASE(1, 1, 2) MGI_DW_CASE(1, 1, 4) MGI_DW_CASE(1, 1, 8)
        MGI_DW_CASE(2, 1, 1) MGI_DW_CASE(2, 1, 2) MGI_DW_CASE(2, 1, 4)
        MGI_DW_CASE(1, 2, 1) MGI_DW_CASE(1, 2, 2) MGI_DW_CASE(1, 2, 4) MGI_DW_CASE(1, 2, 8)
        MGI_DW_CASE(2, 2, 1) MGI_DW_CASE(2, 2, 2) MGI_DW_CASE(2, 2, 4)
#undef MGI_DW_CASE
        if (rows > 0) return hipErrorInvalidValue;
    }
    if (dw5_window(p.KH, p.KW, p.sh, p.sw, p.dh, p.dw)) {
        DwParams q = p;
        const DwTile t = dw5_tile(p.N, p.S, p.OH, p.OW, p.sh, p.xin != nullptr, p.bf16, q.ls);
        if (t.nbands > 0) {
            if (p.sh == 1) return p.bf16 ? launch_dw5<BF16, 1>(q, t, st) : launch_dw5<F16, 1>(q, t, st);
            return p.bf16 ? launch_dw5<BF16, 2>(q, t, st) : launch_dw5<F16, 2>(q, t, st);
        }
    }
    if (p.xin) return hipErrorInvalidValue;
    const int tpp = (ohw + 255) / 256;
    const size_t nblk = (size_t)tpp * p.S * p.N;
    if (nblk > 0x7fffffffu) return hipErrorInvalidValue;
    if (p.bf16) launch(dw_kernel<BF16>, dim3((unsigned)nblk), dim3(256), 0, st, p, tpp);
    else launch(dw_kernel<F16>, dim3((unsigned)nblk), dim3(256), 0, st, p, tpp);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Spatial zero padding of a sliced tensor (a PAD that could not be merged into
// a convolution): one thread per output element of 16 bytes.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void pad_kernel(const h8 *x, h8 *y, int N, int H, int W, int OH,
                                                  int OW, int pt, int pl, size_t total) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const size_t plane = i / ((size_t)OH * OW);
    const int r = (int)(i - plane * OH * OW);
    const int oy = r / OW, ox = r - oy * OW;
    const int iy = oy - pt, ix = ox - pl;
    h8 v;
    if (iy >= 0 && iy < H && ix >= 0 && ix < W) {
        v = x[(plane * H + iy) * W + ix];
    } else {
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = (_Float16)0.0f;
    }
    y[i] = v;
}

hipError_t launch_pad(const h8 *x, h8 *y, int N, int S, int H, int W, int OH, int OW, int pt, int pl,
                      hipStream_t st) {
    const size_t total = (size_t)S * N * OH * OW;
    if (!total) return hipSuccess;
    launch(pad_kernel, dim3(blocks_for(total, 256)), dim3(256), 0, st, x, y, N, H, W, OH, OW, pt, pl,
           total);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// element-wise
// ---------------------------------------------------------------------------
template <typename E>
__global__ __launch_bounds__(256) void add_kernel(const h8 *a, const h8 *b, h8 *y, size_t n, int act) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const h8 u = a[i], v = b[i];
    float o[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) o[c] = act_apply(E::get(u, c) + E::get(v, c), act);
    y[i] = E::pack(o);
}

hipError_t launch_add(const h8 *a, const h8 *b, h8 *y, size_t count, int act, bool bf16, hipStream_t st) {
    if (!count) return hipSuccess;
    if (bf16) launch(add_kernel<BF16>, dim3(blocks_for(count, 256)), dim3(256), 0, st, a, b, y, count, act);
    else launch(add_kernel<F16>, dim3(blocks_for(count, 256)), dim3(256), 0, st, a, b, y, count, act);
    return hipGetLastError();
}

template <typename E>
__global__ __launch_bounds__(256) void act_kernel(const h8 *x, h8 *y, size_t n, int act) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const h8 u = x[i];
    float o[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) o[c] = act_apply(E::get(u, c), act);
    y[i] = E::pack(o);
}

hipError_t launch_act(const h8 *x, h8 *y, size_t count, int act, bool bf16, hipStream_t st) {
    if (!count) return hipSuccess;
    if (bf16) launch(act_kernel<BF16>, dim3(blocks_for(count, 256)), dim3(256), 0, st, x, y, count, act);
    else launch(act_kernel<F16>, dim3(blocks_for(count, 256)), dim3(256), 0, st, x, y, count, act);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void zero_words_kernel(unsigned *p, size_t n) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0u;
}

hipError_t launch_zero_words(unsigned *dst, size_t words, hipStream_t st) {
    if (!words) return hipSuccess;
    launch(zero_words_kernel, dim3(blocks_for(words, 256)), dim3(256), 0, st, dst, words);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// global average pool: one 256-thread workgroup per (slice, image); thread t
// sums pixels t, t + 256, ... four loads at a time (all issued before any
// add; pixels past the end read the zero element), then a fixed butterfly in
// each wave and the four wave sums in a fixed order (deterministic).  Output
// is the sliced (n, 1, 1, c) tensor in the storage type.
// ---------------------------------------------------------------------------
template <typename E>
__global__ __launch_bounds__(256) void gap_kernel(const h8 *x, int xp, h8 *y, const h8 *zero, int HW, int N) {
    __shared__ float part[4][8];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // plane b = slice * N + image; NHWC (xp = slices): pixels xp elements apart
    const int b = blockIdx.x, sl = b / N;
    const h8 *xin = xp == 1 ? x + (size_t)b * HW : x + (size_t)(b - sl * N) * HW * xp + sl;
    float acc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = 0.0f;
    for (int p0 = 0; p0 < HW; p0 += 4 * 256) {
        h8 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int px = p0 + u * 256 + tid;
            v[u] = *(px < HW ? xin + (size_t)px * xp : zero);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[c] += E::get(v[u], c);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] += __shfl_xor(acc[c], off, 64);
    if (lane == 0)
#pragma unroll
        for (int c = 0; c < 8; ++c) part[wave][c] = acc[c];
    __syncthreads();
    if (tid == 0) {
        const float inv = 1.0f / (float)HW;
        float m[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) m[c] = ((part[0][c] + part[1][c]) + (part[2][c] + part[3][c])) * inv;
        y[blockIdx.x] = E::pack(m);
    }
}

// Small planes (up to 64 pixels): 8 lanes per (slice, image); lane j sums
// pixels j, j+8, ... with all loads issued at once (pixels past the end read
// the zero element instead of branching), then a 3-step butterfly inside the
// 8-lane group.  Fixed order, so deterministic.
template <typename E>
__global__ __launch_bounds__(256) void gap_small_kernel(const h8 *x, int xp, h8 *y, const h8 *zero,
                                                        int planes, int HW, int N) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    const int idx = t >> 3, j = t & 7;
    const bool live = idx < planes;
    const int b = live ? idx : 0, sl = b / N;
    const h8 *xin = xp == 1 ? x + (size_t)b * HW : x + (size_t)(b - sl * N) * HW * xp + sl;
    h8 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int px = j + 8 * i;
        v[i] = *((live && px < HW) ? xin + (size_t)px * xp : zero);
    }
    float acc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        float a = 0.0f;
#pragma unroll
        for (int i = 0; i < 8; ++i) a += E::get(v[i], c);
        acc[c] = a;
    }
#pragma unroll
    for (int off = 4; off >= 1; off >>= 1)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] += __shfl_xor(acc[c], off, 8);
    if (live && j == 0) {
        const float inv = 1.0f / (float)HW;
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] *= inv;
        y[idx] = E::pack(acc);
    }
}

hipError_t launch_gap(const h8 *x, int xp, h8 *y, const h8 *zero, int N, int HW, int S, bool bf16,
                      hipStream_t st) {
    const size_t planes = (size_t)S * N;
    if (!planes) return hipSuccess;
    if (HW <= 64) {
        if (bf16)
            launch(gap_small_kernel<BF16>, dim3(blocks_for(planes * 8, 256)), dim3(256), 0, st, x, xp, y, zero,
                   (int)planes, HW, N);
        else
            launch(gap_small_kernel<F16>, dim3(blocks_for(planes * 8, 256)), dim3(256), 0, st, x, xp, y, zero,
                   (int)planes, HW, N);
    } else {
        if (bf16) launch(gap_kernel<BF16>, dim3((unsigned)planes), dim3(256), 0, st, x, xp, y, zero, HW, N);
        else launch(gap_kernel<F16>, dim3((unsigned)planes), dim3(256), 0, st, x, xp, y, zero, HW, N);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// softmax over rows of an fp32 (rows x cols) array; one wave per row
// (softmax_row)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void softmax_kernel(const float *z, float *y, int rows, int cols) {
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;  // whole wave
    softmax_row(z + (size_t)row * cols, y + (size_t)row * cols, cols, threadIdx.x & 63);
}

hipError_t launch_softmax(const float *z, float *y, int rows, int cols, hipStream_t st) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    launch(softmax_kernel, dim3(blocks_for(rows, 4)), dim3(256), 0, st, z, y, rows, cols);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// channel concat: one thread per output (slice, pixel)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void concat_kernel(ConcatParams p) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)p.S * p.M) return;
    const int s = (int)(i / p.M);
    const int m = (int)(i - (size_t)s * p.M);
    // 16-bit values are moved as raw bits (the same for fp16 and bf16 storage)
    u16x8 o = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int c = s * 8 + j;
        if (c >= p.C) break;
        int k = 0;
        while (k + 1 < p.nin && c >= p.coff[k + 1]) ++k;
        const int cc = c - p.coff[k];
        o[j] = ((const uint16_t *)p.src[k])[((size_t)(cc >> 3) * p.M + m) * 8 + (cc & 7)];
    }
    p.y[i] = __builtin_bit_cast(h8, o);
}

hipError_t launch_concat(const ConcatParams &p, hipStream_t st) {
    const size_t n = (size_t)p.S * p.M;
    if (!n) return hipSuccess;
    launch(concat_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, p);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// bilinear resize (optionally followed by argmax over the real channels)
// ---------------------------------------------------------------------------
struct Lerp {
    int i0, i1;
    float f;
};

__device__ __forceinline__ Lerp lerp_coord(int d, int in, int out, int align_corners) {
    float src;
    if (align_corners) src = out > 1 ? (float)d * ((float)(in - 1) / (float)(out - 1)) : 0.0f;
    else src = (float)d * ((float)in / (float)out);
    int i0 = (int)floorf(src);
    if (i0 > in - 1) i0 = in - 1;
    const int i1 = i0 + 1 < in ? i0 + 1 : in - 1;
    return Lerp{i0, i1, src - (float)i0};
}

template <typename E>
__global__ __launch_bounds__(256) void resize_kernel(ResizeParams p) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t opix = (size_t)p.N * p.OH * p.OW;
    if (i >= opix * p.S) return;
    const int s = (int)(i / opix);
    const size_t r = i - (size_t)s * opix;
    const int n = (int)(r / ((size_t)p.OH * p.OW));
    const int q = (int)(r - (size_t)n * p.OH * p.OW);
    const int oy = q / p.OW, ox = q - oy * p.OW;
    const Lerp ly = lerp_coord(oy, p.H, p.OH, p.align_corners);
    const Lerp lx = lerp_coord(ox, p.W, p.OW, p.align_corners);
    const h8 *plane = p.x + ((size_t)s * p.N + n) * p.H * p.W;
    const h8 v00 = plane[(size_t)ly.i0 * p.W + lx.i0], v01 = plane[(size_t)ly.i0 * p.W + lx.i1];
    const h8 v10 = plane[(size_t)ly.i1 * p.W + lx.i0], v11 = plane[(size_t)ly.i1 * p.W + lx.i1];
    float o[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const float top = (1.0f - lx.f) * E::get(v00, c) + lx.f * E::get(v01, c);
        const float bot = (1.0f - lx.f) * E::get(v10, c) + lx.f * E::get(v11, c);
        o[c] = (1.0f - ly.f) * top + ly.f * bot;
    }
    ((h8 *)p.y)[i] = E::pack(o);
}

// A thread owns U consecutive rows of an output column.  Bound by vector
// issue: per output and class four operations blend the columns of the two
// source rows, two blend the rows and three keep the maximum, besides widening
// the four source values.  When upsampling, neighbouring rows mostly fall
// between the same two source rows and share all but the last five (21
// classes, 8 x 41 x 41 -> 641 x 641: one row per thread 28.0 us, four 23.6).
template <typename E, int U>
__global__ __launch_bounds__(256) void resize_argmax_kernel(ResizeParams p, int groups) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)p.N * groups * p.OW) return;
    const int t = (int)(i / p.OW), ox = (int)(i - (size_t)t * p.OW);
    const int n = t / groups, oy0 = (t - n * groups) * U;
    const Lerp lx = lerp_coord(ox, p.W, p.OW, p.align_corners);
    Lerp ly[U];
    float best[U];
    int arg[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        ly[u] = lerp_coord(min(oy0 + u, p.OH - 1), p.H, p.OH, p.align_corners);
        best[u] = -FLT_MAX;
        arg[u] = 0;
    }
    for (int s = 0; s < p.S; ++s) {
        const h8 *plane = p.x + ((size_t)s * p.N + n) * p.H * p.W;
        float top[8], bot[8];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u == 0 || ly[u].i0 != ly[u - 1].i0) {
                const h8 *r0 = plane + (size_t)ly[u].i0 * p.W, *r1 = plane + (size_t)ly[u].i1 * p.W;
                const h8 v00 = r0[lx.i0], v01 = r0[lx.i1], v10 = r1[lx.i0], v11 = r1[lx.i1];
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    top[c] = (1.0f - lx.f) * E::get(v00, c) + lx.f * E::get(v01, c);
                    bot[c] = (1.0f - lx.f) * E::get(v10, c) + lx.f * E::get(v11, c);
                }
            }
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int ch = s * 8 + c;
                if (ch >= p.C) break;
                const float v = (1.0f - ly[u].f) * top[c] + ly[u].f * bot[c];
                if (ch == 0 || v > best[u]) {
                    best[u] = v;
                    arg[u] = ch;
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (oy0 + u < p.OH) ((int *)p.y)[((size_t)n * p.OH + oy0 + u) * p.OW + ox] = arg[u];
}

template <typename E, int U>
static hipError_t launch_resize_argmax(const ResizeParams &p, hipStream_t st) {
    const int groups = (p.OH + U - 1) / U;
    launch((resize_argmax_kernel<E, U>), dim3(blocks_for((size_t)p.N * groups * p.OW, 256)), dim3(256), 0, st, p, groups);
    return hipGetLastError();
}

hipError_t launch_resize(const ResizeParams &p, bool argmax, hipStream_t st) {
    const size_t opix = (size_t)p.N * p.OH * p.OW;
    if (!opix) return hipSuccess;
    if (argmax) {
        // as many rows per thread as leave two workgroups per compute unit
        const size_t per = opix / (512 * 256);
        if (per >= 4) return p.bf16 ? launch_resize_argmax<BF16, 4>(p, st) : launch_resize_argmax<F16, 4>(p, st);
        if (per >= 2) return p.bf16 ? launch_resize_argmax<BF16, 2>(p, st) : launch_resize_argmax<F16, 2>(p, st);
        return p.bf16 ? launch_resize_argmax<BF16, 1>(p, st) : launch_resize_argmax<F16, 1>(p, st);
    } else {
        if (p.bf16) launch(resize_kernel<BF16>, dim3(blocks_for(opix * p.S, 256)), dim3(256), 0, st, p);
        else launch(resize_kernel<F16>, dim3(blocks_for(opix * p.S, 256)), dim3(256), 0, st, p);
    }
    return hipGetLastError();
}

template <typename E>
__global__ __launch_bounds__(256) void argmax_kernel(const h8 *x, int *y, int M, int S, int C) {
    const int m = blockIdx.x * 256 + threadIdx.x;
    if (m >= M) return;
    float best = -FLT_MAX;
    int arg = 0;
    for (int s = 0; s < S; ++s) {
        const h8 v = x[(size_t)s * M + m];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int ch = s * 8 + c;
            if (ch >= C) break;
            const float f = E::get(v, c);
            if (ch == 0 || f > best) {
                best = f;
                arg = ch;
            }
        }
    }
    y[m] = arg;
}

hipError_t launch_argmax(const h8 *x, int *y, int M, int S, int C, bool bf16, hipStream_t st) {
    if (M <= 0) return hipSuccess;
    if (bf16) launch(argmax_kernel<BF16>, dim3(blocks_for(M, 256)), dim3(256), 0, st, x, y, M, S, C);
    else launch(argmax_kernel<F16>, dim3(blocks_for(M, 256)), dim3(256), 0, st, x, y, M, S, C);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// NHWC graph input -> sliced tensor, and sliced -> NHWC fp32 output.  Bound by
// memory: a wave covers 2^ls slices of 64 / 2^ls pixels, lane = (pixel, slice)
// with the slice fastest, so that with eight slices both sides move whole
// lines: 128 bytes (fp16) or 256 (fp32) of consecutive channels per pixel on
// the NHWC side, eight consecutive 16-byte elements per slice on the sliced
// side.  A thread takes U pixels, 64 / 2^ls apart, all of its loads in flight
// together.  (With the slice index running over all of a pixel's slices, the
// sliced side was 16-byte pieces a whole slice apart: 64 x 14 x 14 x 512 took
// 11.8 us in and 21.3 us out against 6.8 and 9.4 us here.)
// VEC: whole 16-byte loads and stores (channels and pointer permitting, see
// the launchers); otherwise one value at a time.
// ---------------------------------------------------------------------------
template <int U>
__device__ __forceinline__ void nhwc_place(int ls, unsigned sgroups, int &s, unsigned &m) {
    const unsigned lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned pg = blockIdx.x / sgroups, sg = blockIdx.x - pg * sgroups;
    s = (sg << ls) + (lane & ((1u << ls) - 1));
    m = (pg * 4 + wave) * (U * (64u >> ls)) + (lane >> ls);
}

template <typename E, typename TIN, int U, bool VEC>
__global__ __launch_bounds__(256) void ingest_kernel(const TIN *x, h8 *y, unsigned M, int C, int S, int ls,
                                                     int sgroups) {
    constexpr int VN = 16 / sizeof(TIN), NV = 8 / VN;
    typedef TIN tv __attribute__((ext_vector_type(VN)));
    int s;
    unsigned m0;
    nhwc_place<U>(ls, sgroups, s, m0);
    if (s >= S) return;
    const unsigned step = 64u >> ls;
    if constexpr (VEC) {
        tv v[U][NV];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned m = min(m0 + u * step, M - 1u);      // (loads past the end repeat the last pixel)
            const tv *src = (const tv *)(x + (size_t)m * C + s * 8);
#pragma unroll
            for (int k = 0; k < NV; ++k) v[u][k] = src[k];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float o[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) o[c] = (float)v[u][c / VN][c % VN];
            if (m0 + u * step < M) y[(size_t)s * M + m0 + u * step] = E::pack(o);
        }
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned m = m0 + u * step;
            if (m >= M) break;
            const TIN *src = x + (size_t)m * C + s * 8;
            float o[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) o[c] = s * 8 + c < C ? (float)src[c] : 0.0f;
            y[(size_t)s * M + m] = E::pack(o);
        }
    }
}

template <typename E, int U, bool VEC>
__global__ __launch_bounds__(256) void export_kernel(const h8 *x, float *y, unsigned M, int C, int S, int ls,
                                                     int sgroups) {
    int s;
    unsigned m0;
    nhwc_place<U>(ls, sgroups, s, m0);
    if (s >= S) return;
    const unsigned step = 64u >> ls;
    h8 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = x[(size_t)s * M + min(m0 + u * step, M - 1u)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const unsigned m = m0 + u * step;
        if (m >= M) break;
        float *dst = y + (size_t)m * C + s * 8;
        if constexpr (VEC) {                              // C is a multiple of 4: the last slice may be half
            *(f4 *)dst = f4{E::get(v[u], 0), E::get(v[u], 1), E::get(v[u], 2), E::get(v[u], 3)};
            if (s * 8 + 4 < C) *(f4 *)(dst + 4) = f4{E::get(v[u], 4), E::get(v[u], 5), E::get(v[u], 6), E::get(v[u], 7)};
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c)
                if (s * 8 + c < C) dst[c] = E::get(v[u], c);
        }
    }
}

// Slices of a wave (2^ls) and grid for S slices of M pixels: four pixels per
// thread once one pixel per thread gives more than eight
// workgroups per compute unit (fewer, longer threads below that leave compute
// units idle).  False when the grid does not fit.
static bool nhwc_grid(int M, int S, int &ls, int &U, int &sgroups, unsigned &grid) {
    ls = nhwc_slices(S);
    sgroups = (S + (1 << ls) - 1) >> ls;
    const size_t px = (size_t)4 * (64 >> ls), one = ((size_t)M + px - 1) / px * (size_t)sgroups;
    U = one > 2048 ? 4 : 1;
    const size_t n = ((size_t)M + U * px - 1) / (U * px) * (size_t)sgroups;
    grid = (unsigned)n;
    return n <= 0x7fffffffull;
}

template <typename E, typename TIN>
static hipError_t launch_ingest_t(const TIN *x, h8 *y, int M, int C, hipStream_t st) {
    const int S = (C + 7) / 8;
    if (M <= 0 || S <= 0) return hipSuccess;
    int ls, U, sg;
    unsigned grid;
    if (!nhwc_grid(M, S, ls, U, sg, grid)) return hipErrorInvalidValue;
    // 16-byte loads: every pixel's slices start on 16 bytes
    const bool vec = C % 8 == 0 && ((uintptr_t)x & 15) == 0;
    if (vec && U == 4) launch((ingest_kernel<E, TIN, 4, true>), dim3(grid), dim3(256), 0, st, x, y, M, C, S, ls, sg);
    else if (vec) launch((ingest_kernel<E, TIN, 1, true>), dim3(grid), dim3(256), 0, st, x, y, M, C, S, ls, sg);
    else if (U == 4) launch((ingest_kernel<E, TIN, 4, false>), dim3(grid), dim3(256), 0, st, x, y, M, C, S, ls, sg);
    else launch((ingest_kernel<E, TIN, 1, false>), dim3(grid), dim3(256), 0, st, x, y, M, C, S, ls, sg);
    return hipGetLastError();
}

hipError_t launch_ingest(const void *x, bool fp16_in, h8 *y, int M, int C, bool bf16, hipStream_t st) {
    if (bf16)
        return fp16_in ? launch_ingest_t<BF16>((const _Float16 *)x, y, M, C, st)
                       : launch_ingest_t<BF16>((const float *)x, y, M, C, st);
    return fp16_in ? launch_ingest_t<F16>((const _Float16 *)x, y, M, C, st)
                   : launch_ingest_t<F16>((const float *)x, y, M, C, st);
}

template <typename E>
static hipError_t launch_export_t(const h8 *x, float *y, int M, int C, hipStream_t st) {
    const int S = (C + 7) / 8;
    if (M <= 0 || S <= 0) return hipSuccess;
    int ls, U, sg;
    unsigned grid;
    if (!nhwc_grid(M, S, ls, U, sg, grid)) return hipErrorInvalidValue;
    const bool vec = C % 4 == 0 && ((uintptr_t)y & 15) == 0;
    if (vec && U == 4) launch((export_kernel<E, 4, true>), dim3(grid), dim3(256), 0, st, x, y, M, C, S, ls, sg);
    else if (vec) launch((export_kernel<E, 1, true>), dim3(grid), dim3(256), 0, st, x, y, M, C, S, ls, sg);
    else if (U == 4) launch((export_kernel<E, 4, false>), dim3(grid), dim3(256), 0, st, x, y, M, C, S, ls, sg);
    else launch((export_kernel<E, 1, false>), dim3(grid), dim3(256), 0, st, x, y, M, C, S, ls, sg);
    return hipGetLastError();
}

hipError_t launch_export(const h8 *x, float *y, int M, int C, bool bf16, hipStream_t st) {
    return bf16 ? launch_export_t<BF16>(x, y, M, C, st) : launch_export_t<F16>(x, y, M, C, st);
}

}  // namespace kern
}  // namespace mgi
