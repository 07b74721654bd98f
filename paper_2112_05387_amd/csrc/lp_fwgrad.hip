// Filter gradients of the narrow layers (16 / 32 / 64 channels, and layers that read the 3-channel image):
//   dW[co][r][s][ci] = sum over pixels of dY[pixel][co] * X[pixel + tap][ci]
//
// As an implicit GEMM over (r, s, ci) the input is gathered nine times, in k-tiles of 32 or 64 pixels with a trip to
// memory each: 50 to 115 us for launches that move 60 MB.  Here a workgroup walks over tiles of whole image rows; a tile's
// dY pixels and the ONE window of input pixels its taps read are requested a tile ahead and put into LDS as they are
// stored, [pixel][channel], and all taps take their fragments from there: the reduction runs over pixels, so bf16
// fragments are read with the transposing LDS read (four pixels of a channel per lane), fp32 ones element by element.
// A workgroup owns a block of at most 32 x 32 (co, ci) channels and all taps; a wave owns one 16 x 16 unit of it (nine
// micro-tiles, 36 accumulators) and, where the block has fewer units than there are waves, a share of the pixels.
// Image-facing layers (3 channels): the columns (r, s, ci) of the filter are 27 of two micro-tiles and a lane reads its own
// tap and channel; their operands are put into LDS as fp32 and multiplied as such (exact for bf16 inputs).
// Every layer of every module takes part in the same launches, up to kFwMax of them in one.
// What bounds it: a workgroup adds its whole block (36 KB of 32 x 32 channels) to the gradient with atomics, 25 us of a launch of 1024
// workgroups.  Hence two workgroups per compute unit in bf16 (ResNet-56 of 128 samples 790 us a step with four, 762 with two).  A longer
// walk would be a longer chain of fp32 sums, so a tile's sums start from zero and are added to the workgroup's.
// fp32 is bound by its products (256 clocks a micro-tile of 32 pixels) and wants four workgroups per compute unit (see the launcher); its
// registers hold two at a time.  Products of three bf16 parts on the fast instruction are not precise enough: it cuts what lies
// below 2^-24 of the largest of eight products towards zero, and over operands of one sign that adds up with the pixels (32 x 32 channels, 3x3
// behind a batch norm, 131072 pixels of positive inputs: 2.9e-6 of the gradient's norm against float64, here 4.7e-7).
#include <algorithm>
#include <type_traits>

#include "lp_kernels.h"
#include "lp_mma.h"
#include "lp_vec.h"

namespace lp {
namespace {

constexpr int FW_NT = 256;
// the kernel's argument where it lies in constant memory: indexed per lane, not a copy in scratch
typedef const __attribute__((address_space(4))) FWgradProb FWgradArg;
typedef const __attribute__((address_space(4))) FWgradGroup FWgradGroupArg;
typedef __attribute__((address_space(3))) void* lds_ptr_t;

typedef __attribute__((ext_vector_type(4))) short s16x4;
__device__ __forceinline__ u32x2 tr_read(const char* p) {
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(lds_ptr_t)const_cast<char*>(p)));
}

// NTAP micro-tiles of columns: 9 taps, 1 tap, or (STEM) 2 groups of 16 of the 9 * Cin columns.  SIXTEEN: 16 -> 16 channels
template <typename T, int NTAP, bool STEM, bool SIXTEEN>
__device__ __forceinline__ void fwgrad_body(FWgradArg& P, const int t, char* const lds) {
    typedef typename std::conditional<STEM, float, T>::type E;       // what lies in LDS
    constexpr int EPV = 16 / (int)sizeof(T);
    constexpr int YU = fwgrad_y_vecs((int)sizeof(T)), XU = STEM ? kFwStemElems : fwgrad_x_vecs((int)sizeof(T));
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int lq = lane & 15, lg = lane >> 4;
    const int Cin = SIXTEEN ? 16 : P.Cin, Cout = SIXTEEN ? 16 : P.Cout, CB = min(Cout, 32), CI = STEM ? 4 : min(Cin, 32);
    const int lgco = Cout == 64 ? 1 : 0, lgci = !STEM && Cin == 64 ? 1 : 0;
    const int range = t >> (lgco + lgci), blk = t & ((1 << (lgco + lgci)) - 1);
    const int co0 = (blk & ((1 << lgco) - 1)) * 32, ci0 = (blk >> lgco) * 32;
    const int IH = P.IH, IW = P.IW, OB = P.Wo, WW = P.WW, stride = P.stride;
    const int YP = CB * (int)sizeof(E) + 16, XP = STEM ? 16 : CI * (int)sizeof(E) + 16;      // LDS pitches
    const int pxmax = P.TH * OB, pxpad = (pxmax + 31) & ~31;
    char* const s_y = lds;
    char* const s_x = lds + pxpad * YP;

    // ---- loads of a tile: dY vectors of this channel block, window vectors (STEM: elements) -----------------------
    const int lgy = CB == 32 ? (EPV == 8 ? 2 : 3) : (EPV == 8 ? 1 : 2);
    const int lgx = CI == 32 ? (EPV == 8 ? 2 : 3) : (EPV == 8 ? 1 : 2);
    const int yv = tid & ((1 << lgy) - 1), yp0 = tid >> lgy, yst = FW_NT >> lgy;
    const int xv = tid & ((1 << lgx) - 1), xp0 = tid >> lgx, xst = FW_NT >> lgx;
    const int WHW = P.WH * WW;
    u32x4 yr[YU], xr[STEM ? 1 : XU];
    float xe[STEM ? XU : 1];
    unsigned ylive = 0, xlive = 0;
    auto load_tile = [&](int tile) {
        const int n = P.tdiv ? (int)(((unsigned long long)(unsigned)tile * P.tdiv) >> 32) : tile;
        const int a0 = (tile - n * P.tpi) * P.TH;
        const int px = min((int)P.TH, P.Ho - a0) * OB;
        const T* __restrict__ dy = reinterpret_cast<const T*>(P.dy) + ((size_t)n * P.Ho + a0) * OB * Cout + co0;
        const T* __restrict__ x = reinterpret_cast<const T*>(P.x) + (size_t)n * IH * IW * Cin + ci0;
        ylive = 0; xlive = 0;
#pragma unroll
        for (int u = 0; u < YU; ++u) {
            const int p = yp0 + u * yst;
            const bool is = p < px;
            ylive |= is ? 1u << u : 0u;
            yr[u] = Vec<T>::load_raw(dy + (is ? (unsigned)(p * Cout + yv * EPV) : 0u));
        }
        const int ih0 = a0 * stride - P.pad, iw0 = -P.pad;
        if constexpr (STEM) {
#pragma unroll
            for (int u = 0; u < XU; ++u) {
                const int i = tid + u * FW_NT;                 // element (window pixel, channel)
                const int wp = __mul24(i, P.cdiv) >> 16, ci = i - wp * Cin;
                const int wr = __mul24(wp, P.wdiv) >> 16, wc = wp - __mul24(wr, WW);
                const int ih = ih0 + wr, iw = iw0 + wc;
                const bool is = wp < WHW && (unsigned)ih < (unsigned)IH && (unsigned)iw < (unsigned)IW;
                xlive |= is ? 1u << u : 0u;
                xe[u] = to_float(x[is ? (unsigned)((__mul24(ih, IW) + iw) * Cin + ci) : 0u]);
            }
        } else {
#pragma unroll
            for (int u = 0; u < XU; ++u) {
                const int wp = xp0 + u * xst;
                const int wr = __mul24(wp, P.wdiv) >> 16, wc = wp - __mul24(wr, WW);
                const int ih = ih0 + wr, iw = iw0 + wc;
                const bool is = wp < WHW && (unsigned)ih < (unsigned)IH && (unsigned)iw < (unsigned)IW;
                xlive |= is ? 1u << u : 0u;
                xr[u] = Vec<T>::load_raw(x + (is ? (unsigned)((__mul24(ih, IW) + iw) * Cin + xv * EPV) : 0u));
            }
        }
    };
    auto store_tile = [&]() {
#pragma unroll
        for (int u = 0; u < YU; ++u) {
            const int p = yp0 + u * yst;
            if (p >= pxpad) continue;
            const u32x4 v = (ylive >> u) & 1u ? yr[u] : u32x4{0u, 0u, 0u, 0u};      // pixels that are not there count as zero
            if constexpr (sizeof(E) == sizeof(T)) *reinterpret_cast<u32x4*>(s_y + __mul24(p, YP) + yv * 16) = v;
            else {
                float f[EPV];
                Vec<T>::unpack(v, f);
#pragma unroll
                for (int e = 0; e < EPV; e += 4) *reinterpret_cast<f32x4*>(s_y + __mul24(p, YP) + yv * (EPV * 4) + e * 4) = f32x4{f[e], f[e + 1], f[e + 2], f[e + 3]};
            }
        }
        if constexpr (STEM) {
#pragma unroll
            for (int u = 0; u < XU; ++u) {
                const int i = tid + u * FW_NT;
                const int wp = __mul24(i, P.cdiv) >> 16, ci = i - wp * Cin;
                if (wp < WHW) *reinterpret_cast<float*>(s_x + wp * 16 + ci * 4) = (xlive >> u) & 1u ? xe[u] : 0.f;
            }
        } else {
#pragma unroll
            for (int u = 0; u < XU; ++u) {
                const int wp = xp0 + u * xst;
                if (wp < WHW) *reinterpret_cast<u32x4*>(s_x + __mul24(wp, XP) + xv * 16) = (xlive >> u) & 1u ? xr[u] : u32x4{0u, 0u, 0u, 0u};
            }
        }
    };

    // ---- this wave's unit and pixel share ---------------------------------------------------------------------------
    const int ncot = CB >> 4, ncit = STEM ? 1 : CI >> 4, units = ncot * ncit;
    const int unit = wave & (units - 1), slice = units == 4 ? 0 : units == 2 ? wave >> 1 : wave, nslices = 4 >> (units == 4 ? 2 : units == 2 ? 1 : 0);
    const int cot = unit & (ncot - 1), cit = ncot == 2 ? unit >> 1 : unit;
    int toff[NTAP];                                // LDS offset of a tap (STEM: of this lane's column of a group)
#pragma unroll
    for (int j = 0; j < NTAP; ++j) {
        if constexpr (STEM) {
            const int col = min(j * 16 + lq, 9 * Cin - 1), tap = __mul24(col, P.cdiv) >> 16, r = (tap * 11) >> 5;
            toff[j] = (r * WW + tap - 3 * r) * 16 + (col - tap * Cin) * 4;
        } else {
            const int r = NTAP == 9 ? j / 3 : 0, s = NTAP == 9 ? j % 3 : 0;
            toff[j] = (r * WW + s) * XP;
        }
    }
    f32x4 acc[NTAP];
#pragma unroll
    for (int j = 0; j < NTAP; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto win_pos = [&](int p) {                    // window offset of tap (0, 0) of pixel p of the tile
        p = min(p, pxmax - 1);
        const int a = __mul24(p, P.odiv) >> 16, b = p - __mul24(a, OB);
        return __mul24(__mul24(a * stride, WW) + b * stride, XP);
    };
    auto compute = [&]() {
        if constexpr (sizeof(E) == 2) {
            f32x4 t[NTAP];                         // the sums of a tile
#pragma unroll
            for (int j = 0; j < NTAP; ++j) t[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int c = slice; c < pxpad >> 5; c += nslices) {
                const int p0 = c * 32 + 8 * lg + (lq >> 2);
                const char* const pa = s_y + __mul24(p0, YP) + cot * 32 + (lq & 3) * 8;
                const char* const pb0 = s_x + win_pos(p0) + cit * 32 + (lq & 3) * 8;
                const char* const pb1 = s_x + win_pos(p0 + 4) + cit * 32 + (lq & 3) * 8;
                // fragments one ahead of the products that use them
                const u32x2 alo = tr_read(pa), ahi = tr_read(pa + 4 * YP);
                const u32x4 af = {alo[0], alo[1], ahi[0], ahi[1]};
                u32x2 blo[2], bhi[2];
                blo[0] = tr_read(pb0 + toff[0]); bhi[0] = tr_read(pb1 + toff[0]);
#pragma unroll
                for (int j = 0; j < NTAP; ++j) {
                    const int q = j & 1;
                    if (j + 1 < NTAP) { blo[q ^ 1] = tr_read(pb0 + toff[j + 1]); bhi[q ^ 1] = tr_read(pb1 + toff[j + 1]); }
                    const u32x4 bf = {blo[q][0], blo[q][1], bhi[q][0], bhi[q][1]};
                    t[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, af), __builtin_bit_cast(bf16x8, bf), t[j], 0, 0, 0);
                }
            }
#pragma unroll
            for (int j = 0; j < NTAP; ++j) acc[j] += t[j];
        } else {
            const char* const ya = s_y + cot * 64 + lq * 4;
            const char* const xb = s_x + (STEM ? 0 : cit * 64 + lq * 4);
            f32x4 t[NTAP];
#pragma unroll
            for (int j = 0; j < NTAP; ++j) t[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
            for (int c = slice; c < pxpad >> 2; c += nslices) {
                const int p = c * 4 + lg;
                const float a = *reinterpret_cast<const float*>(ya + __mul24(p, YP));
                const char* const pb = xb + win_pos(p);
#pragma unroll
                for (int j = 0; j < NTAP; ++j)
                    t[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, *reinterpret_cast<const float*>(pb + toff[j]), t[j], 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < NTAP; ++j) acc[j] += t[j];
        }
    };

    const int t0 = range * P.per, t1 = min(P.ntiles, t0 + P.per);
    load_tile(t0);
    for (int i = t0; i < t1; ++i) {
        store_tile();
        __syncthreads();
        if (i + 1 < t1) load_tile(i + 1);
        compute();
        __syncthreads();
    }

    // ---- partial sums -> dW --------------------------------------------------------------------------------------------
    float* __restrict__ dw = P.dw;
    const int Kg = STEM ? 9 * Cin : NTAP * Cin;
    auto add = [&](int co, int j, int c, float v) {        // column c of group j
        const int col = STEM ? j * 16 + c : j * Cin + ci0 + c;
        if (STEM && col >= Kg) return;
        float* dst = dw + (size_t)co * Kg + col;
        if (P.nranges == 1) *dst = v;
        else atomicAdd(dst, v);
    };
    if (nslices == 1) {
#pragma unroll
        for (int j = 0; j < NTAP; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) add(co0 + cot * 16 + 4 * lg + e, j, cit * 16 + lq, acc[j][e]);
        return;
    }
    float* const red = reinterpret_cast<float*>(lds);      // [wave][column group][16 co][16 columns]
#pragma unroll
    for (int j = 0; j < NTAP; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) red[((wave * NTAP + j) * 16 + 4 * lg + e) * 16 + lq] = acc[j][e];
    __syncthreads();
    for (int i = tid; i < units * NTAP * 256; i += FW_NT) {
        float v = red[i];
        for (int s = 1; s < nslices; ++s) v += red[i + s * units * NTAP * 256];
        const int c = i & 15, r = (i >> 4) & 15, uj = i >> 8, u = uj / NTAP, j = uj - u * NTAP;
        add(co0 + (u & (ncot - 1)) * 16 + r, j, (ncot == 2 ? u >> 1 : u) * 16 + c, v);
    }
}

template <typename T>
__global__ __launch_bounds__(FW_NT, sizeof(T) == 4 ? 2 : 3) void fwgrad_kernel(const FWgradGroup) {
    FWgradGroupArg& g = *(FWgradGroupArg*)__builtin_amdgcn_kernarg_segment_ptr();
    extern __shared__ __attribute__((aligned(16))) char s_lds[];
    static_assert(kFwMax <= 64, "an entry of the table a lane");
    const int lane = threadIdx.x & 63, first = g.start[min(lane, kFwMax - 1)];
    const int pi = __popcll(__ballot(lane < kFwMax && (int)blockIdx.x >= first)) - 1;
    FWgradArg& P = g.p[pi];
    const int t = (int)blockIdx.x - g.start[pi];
    fwgrad_form<(int)sizeof(T)>(P.Cin, P.Cout, P.R, [&](auto ntap, auto stem, auto sixteen) __attribute__((always_inline)) {
        fwgrad_body<T, decltype(ntap)::value, decltype(stem)::value, decltype(sixteen)::value>(P, t, s_lds);
    });
}

}  // namespace

size_t fwgrad_lds_bytes(const FWgradProb& p, int esz) {
    const bool stem = p.Cin < 16;
    const int e = stem ? 4 : esz, CB = std::min<int>(p.Cout, 32), CI = std::min<int>(p.Cin, 32);
    const size_t pxpad = ((size_t)p.TH * p.Wo + 31) & ~(size_t)31;
    const size_t tile = pxpad * (CB * e + 16) + (size_t)p.WH * p.WW * (stem ? 16 : CI * e + 16);
    const int units = (CB / 16) * (stem ? 1 : CI / 16);
    int ntap = 0;
    fwgrad_form<4>(p.Cin, p.Cout, p.R, [&](auto n, auto, auto) { ntap = decltype(n)::value; });
    return std::max(tile, units == 4 ? (size_t)0 : (size_t)4 * ntap * 256 * 4);
}

hipError_t launch_fwgrad(const FWgradGroup& g, int dtype, size_t lds, hipStream_t s) {
    if (g.total_tiles <= 0) return hipSuccess;
    if (dtype == 1) hipLaunchKernelGGL(fwgrad_kernel<bf16_t>, dim3(g.total_tiles), dim3(FW_NT), lds, s, g);
    else hipLaunchKernelGGL(fwgrad_kernel<float>, dim3(g.total_tiles), dim3(FW_NT), lds, s, g);
    return hipGetLastError();
}

}  // namespace lp
