// Convolutions that face the image (few input channels: the whole reduction, taps x channels, is at most 32 long), forward.
//
// The stem and the first layer of every auxiliary net read the same small image and write 16, 32 or 64 channels.  Their
// multiplications are nothing (27 products an output) and so is their traffic: the seven of an eight-module ResNet-56 of 128 samples
// read 0.8 MB and write 18 MB, 5 us of the chip.  In the general kernel they were three launches one after another, one per tile width,
// 1024, 384 and 256 workgroups, 19.3 + 15.3 + 11.7 us: every element of a k-tile is gathered from memory by a 2-byte load of its own behind
// a branch, and a layer of one k-tile has nothing to hide that behind.
// Here the input rows that a tile touches, which lie one after another in memory, go to LDS in one asynchronous copy of whole vectors
// (1 to 6 KB), the taps are picked out of LDS into registers (8 elements of k a lane, which is one MFMA of bf16 and two k-steps
// of fp32), and since no operand tile is laid out, the widths share a launch of 14 us: that step 692 -> 665 us, of 8 samples 390 -> 362,
// an iteration 925 -> 897; a step of four modules 749 -> 726.  A stem alone (512 workgroups) 15.6 -> 10.9 us by itself, 5 of them the timing's own; beside other lanes
// the whole pass gains little: pre-activation ResNet-20, 256 samples forward 527 -> 515, and in front of wide layers nothing (build_module).
//
// The tiles are those of the general kernel (256 pixels x 16 or 32 channels with 64-pixel waves; 64 x 64 in four waves of 32 x 32), and
// so is the order of every sum, of a product's terms and of the statistics: the results are the same bits.
#include <algorithm>

#include "lp_kernels.h"
#include "lp_mma.h"

namespace lp {
namespace {

typedef __attribute__((address_space(3))) void* lds_ptr_t;
constexpr int IC_NT = 256;

template <typename T>
__global__ __launch_bounds__(IC_NT) void iconv_kernel(ConvGroup g) {
    constexpr int EPV = 16 / (int)sizeof(T);
    constexpr int OP = 32 * (int)sizeof(T) + 16;       // bytes between the pixels of a wave's result slice
    constexpr int KE = 8;                              // elements of k a lane holds: 32 over the four lane groups
    constexpr int Z = 16 / (int)sizeof(T);             // the window's first elements are zeros: what a tap outside the image reads
    extern __shared__ __attribute__((aligned(16))) char win[];
    __shared__ __attribute__((aligned(16))) char s_out[4 * 16 * OP];
    __shared__ float s_red[256];                       // [wave rows][channels][2]

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
    int pi = 0;
    for (int i = 1; i < g.nprob; ++i)
        if ((int)blockIdx.x >= g.p[i].tile_start) pi = i;
    const ConvProb& P = g.p[pi];
    const int M = P.M, Ncol = P.Ncol, Cin = P.Cin, IH = P.IH, IW = P.IW, OB = P.OB, per = P.OA * OB, imul = P.imul;
    const bool quad = Ncol > 32;                       // 64 x 64 tiles
    const int BM = quad ? 64 : 256, FM = quad ? 2 : 4, FN = Ncol > 16 ? 2 : 1;
    const int wm = quad ? wave >> 1 : wave, col0 = quad ? (wave & 1) * 32 : 0;
    const int m0 = ((int)blockIdx.x - P.tile_start) * BM, mlast = min(m0 + BM, M) - 1;

    // ---- the rows of the image that the tile reads: from the first tap of its first pixel to the last tap of its last one
    unsigned sb;                                       // the copy's first element, from `in`
    {
        const int n0 = m0 / per, a0 = (m0 - n0 * per) / OB, n1 = mlast / per, a1 = (mlast - n1 * per) / OB;
        const int lo = min(max(a0 * imul + P.dh0, 0), IH - 1), hi = min(max(a1 * imul + P.dh0 + P.ntr - 1, 0), IH - 1);
        const size_t total = (size_t)(M / per) * IH * IW * Cin * sizeof(T);
        const size_t b0 = (size_t)(n0 * IH + lo) * IW * Cin * sizeof(T) & ~(size_t)15;
        const size_t b1 = min(((size_t)(n1 * IH + hi + 1) * IW * Cin * sizeof(T) + 3) & ~(size_t)3, total);
        const int bytes = (int)(b1 - b0);
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<void*>(P.in) + b0, 0, bytes, 0x00020000);
        for (int i = wave; i * 1024 < bytes; i += 4)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)(win + 16 + i * 1024), 16, lane * 16, i * 1024, 0, 0);
        sb = (unsigned)(b0 / sizeof(T));
        if (tid == 0) *reinterpret_cast<u32x4*>(win) = u32x4{0u, 0u, 0u, 0u};
    }

    // ---- this lane's elements of k (the chunks of a k-step as every kernel here holds them) and the filter fragments.  Lane u works out
    // element u of k and pixel u of the wave, once, and the others ask it (with every lane's own quotients that launch was 17 us)
    int tr[KE], ts[KE], dq[KE];
    int q_of, pix_at, pix_off;
    {
        const int q = lane & 31, tap = q / Cin, c = q - tap * Cin, r = tap / P.nts;
        q_of = (q < P.Kg ? r : 64) | (tap - r * P.nts) << 8 | c << 16;      // row 64: none of an image (pix_at below)
        const int m = m0 + wm * FM * 16 + min(lane, FM * 16 - 1);
        const int n = m / per, rem = m - n * per, a = rem / OB, b = rem - a * OB;
        const int ih0 = a * imul + P.dh0, iw0 = b * imul + P.dw0;
        pix_at = (m < M ? ih0 : -0x4000) * 0x10000 | (iw0 & 0xffff);
        pix_off = (int)((unsigned)(((n * IH + ih0) * IW + iw0) * Cin) - sb) + Z;
    }
    T bq[2][KE];
    const T* __restrict__ wt = reinterpret_cast<const T*>(P.wt) + (size_t)(col0 + lr) * P.ldw;
#pragma unroll
    for (int e = 0; e < KE; ++e) {
        const int q = (e / EPV) * 4 * EPV + lg * EPV + e % EPV;
        const int at = __shfl(q_of, q, 64), c = at >> 16;
        tr[e] = at & 0xff; ts[e] = at >> 8 & 0xff;
        dq[e] = (tr[e] * IW + ts[e]) * Cin + c;
        const bool ok = tr[e] != 64;
        if (!ok) tr[e] = 1 << 28;
        const T v = wt[ok ? q : 0];
        bq[0][e] = ok ? v : from_float<T>(0.f);
        bq[1][e] = from_float<T>(0.f);
    }
    if (FN == 2) {
#pragma unroll
        for (int e = 0; e < KE; ++e) {
            const bool ok = tr[e] != 1 << 28;
            const T v = wt[16 * P.ldw + (ok ? (e / EPV) * 4 * EPV + lg * EPV + e % EPV : 0)];
            bq[1][e] = ok ? v : from_float<T>(0.f);
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);                // vmcnt(0): this wave's part of the window
    __syncthreads();

    // ---- 16 pixels at a time: fragment from the window, product, result through the wave's slice, statistics
    const T* const w = reinterpret_cast<const T*>(win);
    char* const slice = s_out + wave * (16 * OP);
    T* __restrict__ out = reinterpret_cast<T*>(P.out);
    float cs1[2] = {0.f, 0.f}, cs2[2] = {0.f, 0.f};
    const int lgG = (sizeof(T) == 2 ? 1 : 2) + FN - 1, G = 1 << lgG;      // vectors of a pixel
    for (int i = 0; i < FM; ++i) {
        const int r0 = m0 + (wm * FM + i) * 16;        // first pixel
        T aq[KE];
        {
            const int at = __shfl(pix_at, i * 16 + lr, 64), base = __shfl(pix_off, i * 16 + lr, 64);
            const int ih0 = at >> 16, iw0 = (int)(short)at;
#pragma unroll
            for (int e = 0; e < KE; ++e) {
                const bool ok = (unsigned)(ih0 + tr[e]) < (unsigned)IH && (unsigned)(iw0 + ts[e]) < (unsigned)IW;
                aq[e] = w[ok ? base + dq[e] : 0];
            }
        }
        f32x4 acc[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (j >= FN) break;
            acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < KE / EPV; ++k) {
                u32x4 av, bv;
                __builtin_memcpy(&av, &aq[k * EPV], 16);
                __builtin_memcpy(&bv, &bq[j][k * EPV], 16);
                Mma<T, 16>::run(av, bv, acc[j]);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const T st = from_float<T>(acc[j][r]);
                *reinterpret_cast<T*>(slice + (lg * 4 + r) * OP + (j * 16 + lr) * (int)sizeof(T)) = st;
                if (r0 + lg * 4 + r < M) {
                    const float v = to_float(st);
                    cs1[j] += v;
                    cs2[j] += v * v;
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (int item = lane; item < 16 * G; item += 64) {
            const int row = item >> lgG, v = item & (G - 1);
            if (r0 + row < M)
                *reinterpret_cast<u32x4*>(out + (size_t)(r0 + row) * Ncol + col0 + v * EPV) = *reinterpret_cast<const u32x4*>(slice + row * OP + v * 16);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (!P.stats) return;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (j >= FN) break;
        float s1 = cs1[j], s2 = cs2[j];
#pragma unroll
        for (int sh = 16; sh < 64; sh <<= 1) {
            s1 += __shfl_xor(s1, sh, 64);
            s2 += __shfl_xor(s2, sh, 64);
        }
        if (lane < 16) {
            const int c = wm * Ncol + col0 + j * 16 + lane;
            s_red[c * 2] = s1;
            s_red[c * 2 + 1] = s2;
        }
    }
    __syncthreads();
    if (tid < Ncol) {
        float s1 = 0.f, s2 = 0.f;
        for (int k = 0; k < (quad ? 2 : 4); ++k) { s1 += s_red[(k * Ncol + tid) * 2]; s2 += s_red[(k * Ncol + tid) * 2 + 1]; }
        double* st = P.stats + (size_t)(blockIdx.x % stat_stripes(Ncol)) * 2 * Ncol;
        atomicAdd(&st[tid], (double)s1);
        atomicAdd(&st[Ncol + tid], (double)s2);
    }
}

}  // namespace

hipError_t launch_iconv(const ConvGroup& g, int dtype, int lds_bytes, hipStream_t s) {
    if (g.total_tiles <= 0) return hipSuccess;
    if (dtype == 1) hipLaunchKernelGGL(iconv_kernel<bf16_t>, dim3(g.total_tiles), dim3(IC_NT), lds_bytes, s, g);
    else hipLaunchKernelGGL(iconv_kernel<float>, dim3(g.total_tiles), dim3(IC_NT), lds_bytes, s, g);
    return hipGetLastError();
}

}  // namespace lp
