// Narrow convolutions (16 / 32 / 64 channels, forward and data-gradient) with the batch-norm passes around them folded in.
//
// A layer of the CIFAR-sized networks moves 0.1 to 16 MB and computes 0.1 to 1.2 GFLOP: 1 to 4 us of the chip.  What such a
// layer costs is the number of dependent launches and, inside a launch, the number of dependent trips to memory.  As
// separate kernels a unit is conv, BN apply (forward) and BN reduce, BN apply, data-gradient (backward), 2 + 3 launches,
// and an implicit GEMM whose k-tiles are loaded one after the other.  Here a unit is one launch each way:
//   * the window of input pixels a tile reads (its rows and a halo) is requested once, all of it; while it is under way
//     the batch-norm coefficients are computed from the summed statistics; then the window is transformed (BN [+ skip]
//     [ReLU], or the BN backward of g and y) and written to LDS.  The tile that owns a pixel also stores the transformed
//     value, which the skip path and the filter gradient need.
//   * the taps read their fragments from the window, the filter's from a ring in LDS that wave-loads fill ahead of them.
//   * the epilogue adds the skip gradient, stores 16-byte vectors, and sums either the statistics of the stored result
//     (forward) or the backward sums of the batch norm(s) the result arrives at.
// Tiles are whole rows of one image.  One kernel serves every width (a tile picks its shape by its problem), so that
// modules of different width share a launch: at most 4096 / BN pixels x BN channels per workgroup of four waves, in the
// ordered tiles of 16 and 32 channels (FConvProb::ordered) 8192 / BN pixels or two images.
#include <algorithm>

#include "lp_kernels.h"
#include "lp_mma.h"
#include "lp_vec.h"

namespace lp {
namespace {

constexpr int FC_NT = 256;
constexpr int FC_COEF = 0;                         // 6 x 64 floats: transform coefficients
constexpr int FC_ECOEF = 6 * 64 * 4;               // 6 x 32 floats: sc, sh, mean, invstd of ey; mean, invstd of ey2
constexpr int FC_FILT = FC_ECOEF + 6 * 32 * 4;     // filter fragments of the tile; behind the contraction: 16 x BN x 4 partial sums
// then the input window, later the result tile
// More k-steps than the ring holds (64 channels; fp32 with 32): its halves of fconv_half(BN) steps are refilled as they are
// done with, so that a tile can have 32 output channels (each column tile transforms the window again) and four workgroups
// (three in fp32) still fit a compute unit.
__host__ __device__ constexpr int fconv_half(int BN) { return BN == 32 ? 5 : 9; }
__host__ __device__ inline int fconv_filt_bytes(int S, int BN) { const int R = 2 * fconv_half(BN), f = (S < R ? S : R) * BN * 64, r = 16 * BN * 16; return f > r ? f : r; }

// floats between the channels of the backward sums of an ordered tile's row lanes: threads of neighbouring channels on distinct banks
__host__ __device__ constexpr int fconv_sum_pitch(int lanes) { return lanes + 4; }

typedef __attribute__((address_space(3))) void* lds_ptr_t;
// The kernel's argument where it lies in constant memory.  (Taken as an ordinary parameter the compiler keeps a private copy
// of all 4 KB in scratch once a kernel has more than 300 uses of it.)
typedef const __attribute__((address_space(4))) FConvProb FConvArg;
typedef const __attribute__((address_space(4))) FConvGroup FConvGroupArg;

// x + (x of the lane N places to the right in the same row of 16 lanes)
template <int N> __device__ __forceinline__ float ror_add(float x) {
    return x + __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), 0x120 | N, 0xf, 0xf, true));
}

// all k-steps of micro-tiles I0 .. I0 + NM of a wave: fragments of the next step are requested ahead of this one's products
template <typename T, bool PAIR, int MT, int NT, int I0, int NM>
__device__ __forceinline__ void fconv_mma_steps(const char* fb, const char* const (&ab)[MT], int atab, int S, int lg, f32x4 (&acc)[MT][NT]) {
    auto fetch = [&](int s, u32x4 (&af)[NM], u32x4 (&bf)[NT]) {
        int off;
        if (PAIR) {
            const int t0 = __builtin_amdgcn_readlane(atab, 2 * s), t1 = __builtin_amdgcn_readlane(atab, 2 * s + 1);
            off = lg >= 2 ? t1 : t0;
        } else off = __builtin_amdgcn_readlane(atab, s);
#pragma unroll
        for (int j = 0; j < NT; ++j) bf[j] = *reinterpret_cast<const u32x4*>(fb + (s * NT + j) * 1024);
#pragma unroll
        for (int i = 0; i < NM; ++i) af[i] = *reinterpret_cast<const u32x4*>(ab[I0 + i] + off);
    };
    auto mma = [&](const u32x4 (&af)[NM], const u32x4 (&bf)[NT]) {
        if constexpr (sizeof(T) == 4) {            // the four products of a k-step go round the accumulators: no chain of dependent ones
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < NM; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        acc[I0 + i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(af[i][e]), __uint_as_float(bf[j][e]), acc[I0 + i][j], 0, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < NM; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) Mma<T, 16>::run(af[i], bf[j], acc[I0 + i][j]);
        }
    };
    u32x4 a0[NM], b0[NT], a1[NM], b1[NT];
    fetch(0, a0, b0);
    int s = 0;
    for (; s + 2 <= S; s += 2) {
        fetch(s + 1, a1, b1);
        mma(a0, b0);
        fetch(min(s + 2, S - 1), a0, b0);
        mma(a1, b1);
    }
    if (s < S) mma(a0, b0);
}
template <typename T, int MT, int NT, int I0, int NM>
__device__ __forceinline__ void fconv_mma(const char* fb, const char* const (&ab)[MT], int atab, int S, bool pair, int lg, f32x4 (&acc)[MT][NT]) {
    if constexpr (sizeof(T) == 2) {
        if (pair) { fconv_mma_steps<T, true, MT, NT, I0, NM>(fb, ab, atab, S, lg, acc); return; }
    }
    fconv_mma_steps<T, false, MT, NT, I0, NM>(fb, ab, atab, S, lg, acc);
}

// ORD (bf16, see FConvProb::ordered; 2: 64 channels): tiles of up to twice the pixels, two images where an image has 64,
// and sums in the order of the passes they replace.
template <typename T, int BN, int ORD>
__device__ __forceinline__ void fconv_tile(FConvArg& P, const int t, const float eps, char* const lds) {
    constexpr int EPV = 16 / (int)sizeof(T);
    constexpr int NT = BN / 16, MT = (ORD == 1 ? 8 : 4) / NT;       // micro-tiles of a wave: MT of pixels (every fourth), NT of channels
    constexpr int CH = 4 * EPV;                    // channels of a k-step
    constexpr int H = fconv_half(BN);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int lr = lane & 15, lg = lane >> 4;

    // ---- tile ----------------------------------------------------------------------------------------
    const int lgt = P.Ncol == BN ? 0 : P.Ncol == 2 * BN ? 1 : 2;     // log2 of the column tiles
    const int tt = t >> lgt, tn = t & ((1 << lgt) - 1);
    const int segs = ORD ? P.segs : 1;             // images of a tile (more than one: whole images)
    const int ti = P.tdiv ? (int)(((unsigned long long)(unsigned)tt * P.tdiv) >> 32) : tt;
    const int n = ti * segs, a0 = (tt - ti * P.tpi) * P.TH;
    const int OB = P.OB, Cin = P.Cin, WW = P.WW, IH = P.IH, IW = P.IW;
    const int nseg = ORD ? min(segs, P.nimg - n) : 1;
    const int spx = min((int)P.TH, P.OA - a0) * OB, px = spx * nseg;      // pixels of a segment, of the tile
    const int n0 = tn * BN;
    const int PB = Cin * (int)sizeof(T) + 16;      // bytes between window pixels: the 16 lanes of a fragment on distinct banks

    float* const s_cf = reinterpret_cast<float*>(lds + FC_COEF);
    float* const s_ec = reinterpret_cast<float*>(lds + FC_ECOEF);
    // ---- filter fragments: straight into LDS, one wave-load per (k-step, 16 output channels): lane -> filter row lr,
    // channels of its k-group, which is also how a fragment is read back (consecutive lanes, 16 bytes each)
    const bool pair = Cin < CH;                    // bf16, 16 channels: a k-step is two taps
    const int ntaps = P.ntr * P.nts;
    const int lgkc = Cin == 2 * CH ? 1 : Cin == 4 * CH ? 2 : 0;
    const int S = fconv_ksteps(ntaps, Cin, (int)sizeof(T));
    const int cl = pair ? (lg & 1) * EPV : lg * EPV;                 // the lane's channel offset inside a k-step
    char* const s_filt = lds + FC_FILT;
    float* const s_red = reinterpret_cast<float*>(s_filt);
    char* const win = s_filt + fconv_filt_bytes(S, BN);
    // Lane u holds where k-step u (pair: tap u) lies in a filter row and in the window, in bytes: 36 steps at most, computed
    // once instead of in every iteration (readlane makes them scalar again).
    int wtab, atab;
    {
        const int u = min(lane, max(pair ? ntaps : S, 1) - 1), tap = u >> lgkc, ch = (u & ((1 << lgkc) - 1)) * (CH * (int)sizeof(T));
        const int nts = P.nts, tr = nts == 3 ? (tap * 11) >> 5 : nts == 2 ? tap >> 1 : tap, ts = tap - tr * nts;
        wtab = ((P.r0 + P.rs * tr) * P.S + (P.s0 + P.ss * ts)) * Cin * (int)sizeof(T) + ch;
        atab = ((P.dh0 + P.dhs * tr - P.dhmin) * WW + (P.dw0 + P.dws * ts - P.dwmin)) * PB + ch;
    }
    auto load_filters = [&](int i0, int i1) __attribute__((always_inline)) {      // wave-loads i0 .. i1 of (k-step, 16 output channels)
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(P.wt), 0, P.Ncol * P.ldw * (int)sizeof(T), 0x00020000);
        const int row = ((n0 + lr) * P.ldw + cl) * (int)sizeof(T);
        for (int i = i0 + wave; i < i1; i += 4) {
            const int s = NT == 2 ? i >> 1 : i, j = NT == 2 ? i & 1 : 0;
            int off = row;
            if (pair) {                            // an odd number of taps: the last one's partner is zeros
                const int o0 = __builtin_amdgcn_readlane(wtab, 2 * s), o1 = __builtin_amdgcn_readlane(wtab, 2 * s + 1);
                off += lg >= 2 ? o1 : o0;
                if (lg >= 2 && 2 * s + 1 >= ntaps) off = (int)0x80000000u;
            } else off += __builtin_amdgcn_readlane(wtab, s);
            int slot = i;
            while (slot >= 2 * H * NT) slot -= 2 * H * NT;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)(s_filt + slot * 1024), 16, off,
                                                     j * 16 * P.ldw * (int)sizeof(T), 0, 0);
        }
    };
    load_filters(0, min(S, 2 * H) * NT);

    // ---- input window: request, coefficients, transform -------------------------------------------------
    const int lgv = Cin == EPV * 2 ? 1 : Cin == EPV * 4 ? 2 : Cin == EPV * 8 ? 3 : 4;   // log2 vectors per pixel
    const int kv = tid & ((1 << lgv) - 1), wp0 = tid >> lgv, wstep = FC_NT >> lgv;
    const int SWH = P.WH, WHW = SWH * WW * nseg;       // window rows of a segment, window pixels
    const int mode = P.mode;
    const bool two = mode >= FX_BN_ADD;
    const size_t img = (size_t)n * IH * IW * Cin;  // this image; offsets inside it fit 32 bits
    const T* __restrict__ in = reinterpret_cast<const T*>(P.in) + img;
    const T* __restrict__ in2 = reinterpret_cast<const T*>(P.in2) + img;
    T* __restrict__ side = tn == 0 && P.side ? reinterpret_cast<T*>(P.side) + img : nullptr;
    const int ihb = a0 * P.imul + P.dhmin, iwb = P.dwmin;
    const int own0 = a0 * P.imul, own1 = min(IH, (a0 + P.TH) * P.imul);
    constexpr int U = sizeof(T) == 4 ? 7 : ORD ? 5 : 4;         // vectors of a trip per thread: a whole window of the usual sizes
    u32x4 r1[U], r2[U];
    unsigned off[U];                               // element offset inside the image
    unsigned inside, owned;                        // per vector: an image pixel, one whose transformed value this tile stores
    auto request = [&](int i0) __attribute__((always_inline)) {
        inside = 0; owned = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if ((i0 + u) * wstep >= WHW) continue;
            const int wp = wp0 + (i0 + u) * wstep;
            int wr = __mul24(wp, P.wdiv) >> 16;
            const int wc = wp - __mul24(wr, WW);
            int seg = 0;
            if (ORD && wr >= SWH) { seg = IH; wr -= SWH; }
            const int ih = ihb + wr, iw = iwb + wc;
            const bool is = wp < WHW && (unsigned)ih < (unsigned)IH && (unsigned)iw < (unsigned)IW;
            off[u] = is ? ((__umul24(seg + ih, IW) + iw) << (lgv + (EPV == 8 ? 3 : 2))) + kv * EPV : 0u;
            inside |= is ? 1u << u : 0u;
            owned |= is && ih >= own0 && ih < own1 ? 1u << u : 0u;
            r1[u] = Vec<T>::load_raw(in + off[u]);
            if (two) r2[u] = Vec<T>::load_raw(in2 + off[u]);
            else r2[u] = u32x4{0u, 0u, 0u, 0u};
        }
        if (!side) owned = 0;
    };
    // A wave each for the sums of a batch norm: their loads go out ahead of the window's (a wave's loads return in order), all
    // stripes at once, and no sum waits for another.
    const double* const sums_of = wave == 0 ? (mode != FX_PLAIN ? P.stats : nullptr) : wave == 1 ? (mode == FX_BN_BN || mode == FX_BWD ? P.stats2 : nullptr)
                                  : wave == 2 ? (P.ey ? P.estats : nullptr) : (P.ey2 ? P.estats2 : nullptr);
    const int sc_C = wave < 2 ? Cin : P.Ncol, sc_c = wave < 2 ? lane : n0 + lane;
    const bool sum_lane = sums_of && lane < (wave < 2 ? Cin : BN);
    StripeLoads sl;
    float ga = 1.f, be = 0.f;
    if (sum_lane) {
        sl.load(sums_of, sc_c, sc_C);
        if (wave != 1 || mode != FX_BWD) {
            const float* const gp = wave == 0 ? P.gamma : wave == 1 ? P.gamma2 : P.egamma;
            const float* const bp = wave == 0 ? P.beta : wave == 1 ? P.beta2 : P.ebeta;
            ga = gp[sc_c]; be = bp[sc_c];
        }
    }
    if (S > 0) request(0);
    // forward: value = (c0*a + c1) + (c2*b + c3), whatever the mode: c = (1, 0) for a tensor taken as it is, (0, 0) for none
    if (wave == 0 && lane < Cin) {
        float sc = 1.f, sh = 0.f, mu = 0.f, is = 1.f;
        if (mode != FX_PLAIN) bn_coeffs(sl, ga, be, P.nimg * IH * IW, eps, sc, sh, mu, is);
        s_cf[lane] = sc; s_cf[64 + lane] = sh;
        if (mode == FX_BWD) { s_cf[128 + lane] = is; s_cf[192 + lane] = mu; }
    }
    if (wave == 1 && lane < Cin) {
        if (mode == FX_BWD) {
            const double inv_m = 1.0 / (double)(P.nimg * IH * IW);
            double rs0, rs1;
            sl.sums(rs0, rs1);
            s_cf[256 + lane] = (float)(rs1 * inv_m); s_cf[320 + lane] = (float)(rs0 * inv_m);
            if (t == 0 && P.side) {
                const_cast<float*>(P.gamma2)[lane] = (float)rs1;
                const_cast<float*>(P.beta2)[lane] = (float)rs0;
            }
        } else {
            float sc = mode == FX_BN_ADD ? 1.f : 0.f, sh = 0.f, mu, is;
            if (mode == FX_BN_BN) bn_coeffs(sl, ga, be, P.nimg * IH * IW, eps, sc, sh, mu, is);
            s_cf[128 + lane] = sc; s_cf[192 + lane] = sh;
        }
    }
    if (wave >= 2 && sum_lane) {                   // of a projection's batch norm (wave 3): no ReLU behind it, scale and shift are not needed
        float sc, sh, mu, is;
        bn_coeffs(sl, ga, be, P.nimg * P.OH * P.OW, eps, sc, sh, mu, is);
        float* const o = wave == 2 ? s_ec + 64 : s_ec + 128;
        if (wave == 2) { s_ec[lane] = sc; s_ec[32 + lane] = sh; }
        o[lane] = mu; o[32 + lane] = is;
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);            // vmcnt(0): this wave's filter fragments are in LDS (the window is needed next anyway)
    __syncthreads();
    if (S > 0) {
        float c0[EPV], c1[EPV], c2[EPV], c3[EPV], c4[EPV];
        auto coef = [&](int q, float (&c)[EPV]) {
#pragma unroll
            for (int e = 0; e < EPV; e += 4) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(s_cf + q * 64 + kv * EPV + e);
                c[e] = v[0]; c[e + 1] = v[1]; c[e + 2] = v[2]; c[e + 3] = v[3];
            }
        };
        coef(0, c0); coef(1, c1); coef(2, c2); coef(3, c3);
        const bool relu = P.relu != 0;
        auto put = [&](int i0, int u, u32x4 v) {
            const int wp = wp0 + (i0 + u) * wstep;
            if (!((inside >> u) & 1u)) v = u32x4{0u, 0u, 0u, 0u};
            if (wp < WHW) *reinterpret_cast<u32x4*>(win + __mul24(wp, PB) + kv * 16) = v;
            if ((owned >> u) & 1u) *reinterpret_cast<u32x4*>(side + off[u]) = v;
        };
        for (int i0 = 0;;) {
            if (mode == FX_BWD) {
                if (i0 == 0) {                     // k1 * g' - k2 * y + k3 from scale, 1 / sigma, mean and the means of the backward sums
                    float f1[EPV], f0[EPV];
                    coef(4, f1); coef(5, f0);
#pragma unroll
                    for (int e = 0; e < EPV; ++e) {
                        const float k2 = c0[e] * c2[e] * f1[e];
                        c4[e] = fmaf(k2, c3[e], -(c0[e] * f0[e]));
                        c2[e] = c0[e]; c3[e] = k2;
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if ((i0 + u) * wstep >= WHW) continue;
                    float a[EPV], b[EPV], o[EPV];
                    Vec<T>::unpack(r1[u], a);
                    Vec<T>::unpack(r2[u], b);
                    if (relu) {
#pragma unroll
                        for (int e = 0; e < EPV; ++e) a[e] = fmaf(c0[e], b[e], c1[e]) > 0.f ? a[e] : 0.f;
                    }
#pragma unroll
                    for (int e = 0; e < EPV; ++e) o[e] = fmaf(c2[e], a[e], -(c3[e] * b[e])) + c4[e];
                    put(i0, u, Vec<T>::pack(o));
                }
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if ((i0 + u) * wstep >= WHW) continue;
                    float a[EPV], b[EPV], o[EPV];
                    Vec<T>::unpack(r1[u], a);
#pragma unroll
                    for (int e = 0; e < EPV; ++e) o[e] = fmaf(c0[e], a[e], c1[e]);
                    if (two) {
                        Vec<T>::unpack(r2[u], b);
#pragma unroll
                        for (int e = 0; e < EPV; ++e) o[e] += fmaf(c2[e], b[e], c3[e]);
                    }
                    if (relu) {
#pragma unroll
                        for (int e = 0; e < EPV; ++e) o[e] = fmaxf(o[e], 0.f);
                    }
                    put(i0, u, Vec<T>::pack(o));
                }
            }
            i0 += U;
            if (i0 * wstep >= WHW) break;
            request(i0);
        }
    }
    __syncthreads();

    // ---- what the epilogue reads from memory, ahead of the contraction ----------------------------------------
    // The result passes through LDS in parts of PART pixels.  A thread has one vector of channels of
    // every ER-th pixel; with ORD the backward sums are added up per thread and then over the ER threads in order, as the
    // separate pass does with its 256 / (Ncol / 8) row lanes, so 64 channels use half of the threads.
    constexpr int LGN = BN / EPV == 2 ? 1 : BN / EPV == 4 ? 2 : 3;                      // log2 vectors per result pixel
    constexpr int ER = ORD == 2 ? 32 : FC_NT >> LGN;
    constexpr int PART = ORD == 2 ? 64 : 4096 / BN, EI = PART / ER;
    const int ev = tid & ((1 << LGN) - 1);
    const int er = tid >> LGN;
    const size_t oimg = (size_t)n * P.OH * P.OW * P.Ncol;
    const T* __restrict__ add0 = reinterpret_cast<const T*>(P.add0) + oimg;
    const T* __restrict__ ey = reinterpret_cast<const T*>(P.ey) + oimg;
    const T* __restrict__ ey2 = reinterpret_cast<const T*>(P.ey2) + oimg;
    u32x4 xa[EI], xe[EI], xf[EI];
    int oo[EI];                                    // element offset of the vector in this image's output; -1: none
    auto ahead = [&](int part) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < EI; ++i) {
            const int p = part * PART + er + i * ER;
            int a = __mul24(p, P.odiv) >> 16;
            const int b = p - __mul24(a, OB);
            if (ORD && a >= P.TH && segs > 1) a += P.OH - P.TH;      // the second image of the tile (TH = OH then)
            oo[i] = p < px && er < ER ? (__mul24((a0 + a) * P.omul + P.ooh, P.OW) + b * P.omul + P.oow) * P.Ncol + n0 + ev * EPV : -1;
            const unsigned o = oo[i] >= 0 ? (unsigned)oo[i] : 0u;
            if (P.add0) xa[i] = Vec<T>::load_raw(add0 + o);
            if (P.ey) xe[i] = Vec<T>::load_raw(ey + o);
            if (P.ey2) xf[i] = Vec<T>::load_raw(ey2 + o);
        }
    };
    ahead(0);

    // ---- contraction ------------------------------------------------------------------------------------------
    f32x4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nmt = (px + 15) >> 4;                // micro-tiles of 16 pixels in this tile
    // micro-tile i of this wave: every fourth, in the ordered tiles MP consecutive ones of every part (a run of the statistics is one
    // wave's, or two neighbours')
    constexpr int NP = ORD ? 2 : 1, MP = MT / NP;
    auto mtile = [&](int i) { return ORD ? i / MP * 4 * MP + wave * MP + i % MP : wave + 4 * i; };
    const char* ab[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int p = min(mtile(i) * 16 + lr, px - 1);
        const int a = __mul24(p, P.odiv) >> 16, b = p - __mul24(a, OB);
        const int seg = ORD && segs > 1 && a >= P.TH ? 1 : 0;
        ab[i] = win + __mul24(__mul24((a - (seg ? P.TH : 0)) * P.imul + (seg ? SWH : 0), WW) + b * P.imul, PB) + cl * (int)sizeof(T);
    }
    const char* const fb = s_filt + lane * 16;
    // micro-tiles of this wave (an ordered tile has one part or both); the loops compute 1, 2 or 4 without a branch per tile
    const int nm = ORD ? (px > PART ? MT : MP) : (nmt - wave + 3) >> 2;
    auto contract = [&](int tab, int slot, int steps) __attribute__((always_inline)) {
        const char* const fs = fb + slot * (NT * 1024);
        if constexpr (MT == 8) {                   // (eight at a time would need 64 registers for fragments)
            if (nm > 4) {
                fconv_mma<T, MT, NT, 0, 4>(fs, ab, tab, steps, pair, lg, acc);
                fconv_mma<T, MT, NT, 4, 4>(fs, ab, tab, steps, pair, lg, acc);
                return;
            }
        }
        if constexpr (MT >= 4) {
            if (nm > 2) { fconv_mma<T, MT, NT, 0, 4>(fs, ab, tab, steps, pair, lg, acc); return; }
        }
        if (nm > 1) fconv_mma<T, MT, NT, 0, 2>(fs, ab, tab, steps, pair, lg, acc);
        else fconv_mma<T, MT, NT, 0, 1>(fs, ab, tab, steps, pair, lg, acc);
    };
    if (S > 0 && S <= 2 * H) contract(atab, 0, S);
    else if (S > 0) {
#pragma unroll 1
        for (int c = 0; c * H < S; ++c) {
            if (c >= 2) {                          // the refill of this half has landed, in every wave
                __builtin_amdgcn_s_waitcnt(0x0f70);
                __syncthreads();
            }
            contract(__builtin_amdgcn_ds_bpermute((lane + H * c) * 4, atab), (c & 1) * H, min(H, S - c * H));
            if ((c + 2) * H < S) {
                __syncthreads();
                load_filters((c + 2) * H * NT, min((c + 3) * H, S) * NT);
            }
        }
    }

    // ---- result tile through LDS, one 16-byte vector per access -------------------------------------------------
    constexpr int SP = BN + 4;
    float* const res = reinterpret_cast<float*>(win);
    T* __restrict__ out = reinterpret_cast<T*>(P.out) + oimg;
    float q1[EPV], q2[EPV], q3[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e) { q1[e] = 0.f; q2[e] = 0.f; q3[e] = 0.f; }
    auto ecoef = [&](int q, float (&c)[EPV]) {
#pragma unroll
        for (int e = 0; e < EPV; e += 4) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(s_ec + q * 32 + ev * EPV + e);
            c[e] = v[0]; c[e + 1] = v[1]; c[e + 2] = v[2]; c[e + 3] = v[3];
        }
    };
    const bool erelu = P.erelu != 0;
    double* const sums = P.ey ? P.ered : P.ostats;
    const bool stat_pass = ORD && !P.ey && sums;   // batch statistics in the order of the implicit-GEMM kernel's epilogue
#pragma unroll
    for (int part = 0; part < NP; ++part) {
        if (part * PART >= px) continue;
        if (part > 0) ahead(part);
        __syncthreads();                           // every wave is done with the window, or with the part before
#pragma unroll
        for (int i = 0; i < MP; ++i) {
            if (mtile(part * MP + i) < nmt) {
                const int row = (ORD ? wave * MP + i : wave + 4 * i) * 16 + lg * 4;
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) res[(row + r) * SP + j * 16 + lr] = acc[part * MP + i][j][r];
            }
        }
        // Statistics in the order of the implicit-GEMM kernel's epilogue: runs of 4 micro-tiles (2 with 64 channels), a lane's rows one after
        // the other, of the values as stored.  They are in this wave's accumulators, the first half of a run in its neighbour's where
        // a wave has half of one: the sums so far go on through LDS.  (Read back from the result's LDS, with a barrier more, the
        // epilogue of a forward layer took 4.9 us of 16, of which 2.)
        constexpr int WR = (ORD == 2 ? 2 : 4) / MP;         // waves of a run
        float s1[NT], s2[NT];
        auto run_sums = [&]() {
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int i = 0; i < MP; ++i)
#pragma unroll
                    for (int r = 0; r < 4; r += 2) {
                        const unsigned v = pack_bf16x2(acc[part * MP + i][j][r], acc[part * MP + i][j][r + 1]);
                        const float lo = __uint_as_float(v << 16), hi = __uint_as_float(v & 0xffff0000u);
                        s1[j] += lo; s2[j] = fmaf(lo, lo, s2[j]);
                        s1[j] += hi; s2[j] = fmaf(hi, hi, s2[j]);
                    }
        };
        float* const hop = s_red + 256 + ((wave >> 1) * NT * 64 + lane) * 2;
        if constexpr (ORD != 0) {
            if (stat_pass && (WR == 1 || !(wave & 1))) {
#pragma unroll
                for (int j = 0; j < NT; ++j) { s1[j] = 0.f; s2[j] = 0.f; }
                run_sums();
                if (WR == 2) {
#pragma unroll
                    for (int j = 0; j < NT; ++j) { hop[j * 128] = s1[j]; hop[j * 128 + 1] = s2[j]; }
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < EI; ++i) {
            if (oo[i] < 0) continue;
            float* const rp = res + (er + i * ER) * SP + ev * EPV;
            float v[EPV];
#pragma unroll
            for (int e = 0; e < EPV; e += 4) {
                const f32x4 q = *reinterpret_cast<const f32x4*>(rp + e);
                v[e] = q[0]; v[e + 1] = q[1]; v[e + 2] = q[2]; v[e + 3] = q[3];
            }
            if (P.add0) {
                float a[EPV];
                Vec<T>::unpack(xa[i], a);
#pragma unroll
                for (int e = 0; e < EPV; ++e) v[e] += a[e];
            }
            const u32x4 st = Vec<T>::pack(v);
            *reinterpret_cast<u32x4*>(out + (unsigned)oo[i]) = st;
            Vec<T>::unpack(st, v);                 // the sums describe the values as stored
            if (P.ey) {
                float y[EPV], c[EPV], d[EPV];
                Vec<T>::unpack(xe[i], y);
                if (P.ey2) {                       // before the mask: there is no ReLU between the sum and a projection's batch norm
                    float y2[EPV];
                    Vec<T>::unpack(xf[i], y2);
                    ecoef(4, c); ecoef(5, d);
#pragma unroll
                    for (int e = 0; e < EPV; ++e) q3[e] += v[e] * ((y2[e] - c[e]) * d[e]);
                }
                if (erelu) {
                    ecoef(0, c); ecoef(1, d);
#pragma unroll
                    for (int e = 0; e < EPV; ++e) v[e] = fmaf(c[e], y[e], d[e]) > 0.f ? v[e] : 0.f;
                }
                ecoef(2, c); ecoef(3, d);
#pragma unroll
                for (int e = 0; e < EPV; ++e) { q1[e] += v[e]; q2[e] += v[e] * ((y[e] - c[e]) * d[e]); }
            } else if (!stat_pass) {
#pragma unroll
                for (int e = 0; e < EPV; ++e) { q1[e] += v[e]; q2[e] += v[e] * v[e]; }
            }
        }
        if constexpr (ORD != 0) {
            if (stat_pass && (WR == 1 || (wave & 1))) {
                if (WR == 2) {
#pragma unroll
                    for (int j = 0; j < NT; ++j) { s1[j] = hop[j * 128]; s2[j] = hop[j * 128 + 1]; }
                    run_sums();
                }
                constexpr int lgrw = ORD == 2 ? 5 : 6;
                const int run = (part * PART >> lgrw) + wave / WR;
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    float a = s1[j], b = s2[j];
                    a += __shfl_xor(a, 16, 64); b += __shfl_xor(b, 16, 64);
                    a += __shfl_xor(a, 32, 64); b += __shfl_xor(b, 32, 64);
                    if (lane < 16) {
                        float* const q = s_red + (run * BN + j * 16 + lane) * 2;
                        q[0] = a; q[1] = b;
                    }
                }
            }
        }
    }
    if (!sums) return;
    const size_t at = (size_t)(blockIdx.x % stat_stripes(P.Ncol)) * 2 * P.Ncol + n0 + tid;          // this workgroup's stripe
    if constexpr (ORD != 0) {
        double d1 = 0.0, d2 = 0.0;
        if (stat_pass) {                           // runs of one tile of the implicit-GEMM kernel in fp32, the tiles in fp64
            __syncthreads();
            if (tid >= BN) return;
            constexpr int lgrw = ORD == 2 ? 5 : 6, per = ORD == 2 ? 2 : 4;
            const int nrun = (px + (1 << lgrw) - 1) >> lgrw;
            for (int r0 = 0; r0 < nrun; r0 += per) {
                float s1 = 0.f, s2 = 0.f;
                for (int w = r0; w < min(r0 + per, nrun); ++w) { s1 += s_red[(w * BN + tid) * 2]; s2 += s_red[(w * BN + tid) * 2 + 1]; }
                d1 += (double)s1; d2 += (double)s2;
            }
        } else {                                   // row lane by row lane, per channel
            __syncthreads();                       // the last part of the result has been read
            // [sum g', sum g' yhat, sum g yhat of the second batch norm][channel][row lane]: a thread each adds up a sum of a channel,
            // four row lanes a read (one thread with three, element by element: 2.5 of a 16-channel tile's 16 us)
            constexpr int RP = fconv_sum_pitch(ER);
            float* const rs = res;
            const int nq = P.ey2 ? 3 : 2;
            if (er < ER) {
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    float* const q = rs + (ev * EPV + e) * RP + er;
                    q[0] = q1[e]; q[BN * RP] = q2[e];
                    if (P.ey2) q[2 * BN * RP] = q3[e];
                }
            }
            __syncthreads();
            const int k = tid / BN, c = tid - k * BN;
            if (k >= nq) return;
            const f32x4* const q = reinterpret_cast<const f32x4*>(rs + tid * RP);
            float sum = 0.f;
#pragma unroll
            for (int l0 = 0; l0 < ER / 4; l0 += 8) {
                f32x4 v[8];
#pragma unroll
                for (int l = 0; l < 8; ++l) v[l] = q[l0 + l];
#pragma unroll
                for (int l = 0; l < 8; ++l) { sum += v[l][0]; sum += v[l][1]; sum += v[l][2]; sum += v[l][3]; }
            }
            const size_t to = (size_t)(blockIdx.x % stat_stripes(P.Ncol)) * 2 * P.Ncol + n0 + c;
            if (k == 2) { atomicAdd(&P.ered2[to + P.Ncol], (double)sum); return; }
            atomicAdd(&sums[to + k * P.Ncol], (double)sum);
            if (k == 0 && P.ey2) atomicAdd(&P.ered2[to], (double)sum);
            return;
        }
        atomicAdd(&sums[at], d1);
        atomicAdd(&sums[at + P.Ncol], d2);
        return;
    }
    // over the pixel rows of 16 lanes by rotation, then 16 partial sums per channel through LDS
#pragma unroll
    for (int e = 0; e < EPV; ++e) {
        q1[e] = ror_add<8>(q1[e]); q2[e] = ror_add<8>(q2[e]);
        if (LGN <= 2) { q1[e] = ror_add<4>(q1[e]); q2[e] = ror_add<4>(q2[e]); }
        if (LGN <= 1) { q1[e] = ror_add<2>(q1[e]); q2[e] = ror_add<2>(q2[e]); }
        if (P.ey2) {
            q3[e] = ror_add<8>(q3[e]);
            if (LGN <= 2) q3[e] = ror_add<4>(q3[e]);
            if (LGN <= 1) q3[e] = ror_add<2>(q3[e]);
        }
    }
    if (lr < (1 << LGN)) {
#pragma unroll
        for (int e = 0; e < EPV; ++e)
            *reinterpret_cast<f32x4*>(s_red + ((wave * 4 + lg) * BN + ev * EPV + e) * 4) = f32x4{q1[e], q2[e], q3[e], 0.f};
    }
    __syncthreads();
    if (tid < BN) {
        f32x4 a = *reinterpret_cast<const f32x4*>(s_red + tid * 4);
#pragma unroll
        for (int w = 1; w < 16; ++w) a += *reinterpret_cast<const f32x4*>(s_red + (w * BN + tid) * 4);
        atomicAdd(&sums[at], (double)a[0]);
        atomicAdd(&sums[at + P.Ncol], (double)a[1]);
        if (P.ey2) {
            atomicAdd(&P.ered2[at], (double)a[0]);
            atomicAdd(&P.ered2[at + P.Ncol], (double)a[2]);
        }
    }
}

template <typename T>
__global__ __launch_bounds__(FC_NT, 3) void fconv_kernel(const FConvGroup) {
    FConvGroupArg& g = *(FConvGroupArg*)__builtin_amdgcn_kernarg_segment_ptr();
    extern __shared__ __attribute__((aligned(16))) char s_lds[];
    int pi = 0;
#pragma unroll
    for (int i = 1; i < kMaxGroup; ++i) pi += (int)blockIdx.x >= g.start[i] ? 1 : 0;
    FConvArg& P = g.p[pi];
    const int t = (int)blockIdx.x - g.start[pi];
    // one field of every cache line of the problem: the lines are fetched together, not one by one where they are first used
    asm volatile("" ::"s"(P.in), "s"(P.stats2), "s"(P.ey), "s"(P.ldw), "s"((int)P.S));
    if constexpr (sizeof(T) == 2) {
        if (P.ordered) {
            if (P.BN == 16) fconv_tile<T, 16, 1>(P, t, g.eps, s_lds);
            else if (P.Ncol == 32) fconv_tile<T, 32, 1>(P, t, g.eps, s_lds);
            else fconv_tile<T, 32, 2>(P, t, g.eps, s_lds);
            return;
        }
    }
    if (P.BN == 16) fconv_tile<T, 16, 0>(P, t, g.eps, s_lds);
    else fconv_tile<T, 32, 0>(P, t, g.eps, s_lds);
}

}  // namespace

size_t fconv_lds_bytes(const FConvProb& p, int esz) {
    const int segs = p.ordered ? p.segs : 1, px = (p.TH * p.OB * segs + 15) & ~15;
    const size_t win = (size_t)p.WH * p.WW * segs * (p.Cin * esz + 16);
    size_t res = (size_t)std::min(px, p.ordered && p.Ncol == 64 ? 64 : fconv_max_px(p.BN)) * (p.BN + 4) * 4;
    if (p.ordered && p.ey) res = std::max(res, (size_t)3 * p.BN * fconv_sum_pitch(p.Ncol == 64 ? 32 : 2048 / p.BN) * 4);
    return FC_FILT + fconv_filt_bytes(fconv_ksteps(p.ntr * p.nts, p.Cin, esz), p.BN) + std::max(win, res);
}

hipError_t launch_fconv(const FConvGroup& g, int dtype, size_t lds, hipStream_t s) {
    if (g.total_tiles <= 0) return hipSuccess;
    static OncePerDevice configured;               // (the windows of stride-2 layers in ordered tiles are the ones beyond 64 KB)
    if (const hipError_t e = raise_lds_limit(configured, {(const void*)fconv_kernel<bf16_t>, (const void*)fconv_kernel<float>}, kFconvMaxLds);
        e != hipSuccess) return e;
    if (dtype == 1) hipLaunchKernelGGL(fconv_kernel<bf16_t>, dim3(g.total_tiles), dim3(FC_NT), lds, s, g);
    else hipLaunchKernelGGL(fconv_kernel<float>, dim3(g.total_tiles), dim3(FC_NT), lds, s, g);
    return hipGetLastError();
}

}  // namespace lp
