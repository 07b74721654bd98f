// Wide bf16 convolutions of small mini-batches, and the batch statistics of their results.
//
// The tiles of the wide-layer kernels (512 x 160, 256 x 320, 128 x 160) leave most of the chip idle when a layer has few
// pixels: the 8 x 8 x 640 layers of a wide network have 64 of them per sample, i.e. one or two workgroups for mini-batches
// up to eight, and such a launch is the time ONE workgroup needs for a whole tile (100 us, whatever the mini-batch).  Here a
// workgroup of four waves owns at most 128 pixels x 32 output channels; each wave multiplies one 32 x 32 micro-tile.
// What bounds it is the path from L2 into a compute unit's LDS (a 128-byte line per 4-5 clocks): per slab of 64 channels the
// input window is loaded once for all taps, 100-300 lines, and the filters of 32 output channels, 32 lines per tap.  Groups
// of slabs are double-buffered: all of the next group's lines are requested at once, a group ahead of their use.
// The sum over taps and channels runs in the order of the kernel that would otherwise take the launch (channel slabs of 64
// or 32, taps inside a slab, 16 channels per instruction), and the statistics are added up as that kernel's epilogue does
// (stats_of_tiles_kernel), so the choice between the two changes no bit of any result.
#include <algorithm>

#include "lp_kernels.h"
#include "lp_mma.h"
#include "lp_vec.h"

namespace lp {
namespace {

constexpr int SC_NT = 256;
constexpr unsigned kOOB = 0x80000000u;
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(4))) SConvProb SConvArg;
typedef const __attribute__((address_space(4))) SConvGroup SConvGroupArg;

__global__ __launch_bounds__(SC_NT, 1) void sconv_kernel(const SConvGroup) {
    SConvGroupArg& g = *(SConvGroupArg*)__builtin_amdgcn_kernarg_segment_ptr();
    extern __shared__ __attribute__((aligned(16))) char lds[];
    int pi = 0;
#pragma unroll
    for (int i = 1; i < kMaxGroup; ++i) pi += (int)blockIdx.x >= g.start[i] ? 1 : 0;
    SConvArg& P = g.p[pi];
    const int t = (int)blockIdx.x - g.start[pi];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;

    // ---- tile: TH rows of one image, or `segs` whole images; channels n0 .. n0 + 32 (neighbours share the pixels) --------
    const int ntn = (P.Ncol + 31) >> 5;
    const int tt = __builtin_amdgcn_readfirstlane(t / ntn), n0 = (t - tt * ntn) * 32;
    const int ti = __builtin_amdgcn_readfirstlane(tt / P.tpi);
    const int n = ti * P.segs, a0 = (tt - ti * P.tpi) * P.TH;
    const int OB = P.OB, WW = P.WW, Cin = P.Cin, IH = P.IH, IW = P.IW;
    const int nseg = min((int)P.segs, P.nimg - n);
    const int th = min((int)P.TH, P.OA - a0), px = th * OB * nseg;
    const int ntaps = P.ntr * P.nts;
    const bool single = ntaps == 1;                // one tap: the window is the list of the tile's own source pixels
    const int npx = single ? px : P.WH * WW * nseg;
    const int slab = P.slab, nslab = (Cin + 63) / 64, gs = P.gs, ng = ntaps == 0 ? 0 : (nslab + gs - 1) / gs;
    const int win_bytes = P.win_bytes, slab_bytes = win_bytes + ntaps * 4096, buf_bytes = gs * slab_bytes;

    // ---- addresses of the window pixels this lane fetches: wave-load i of the wave covers pixels 8 * (wave + 4 i) .. + 8,
    // lane l pixel l / 8 of them and the 16-byte chunk that belongs at place l % 8 (chunks of a row are stored XORed with the
    // row, which keeps the fragment reads off each other's banks)
    constexpr int NWL = kSconvMaxPx / 32;
    unsigned wofs[NWL];
    int wswz[NWL];
#pragma unroll
    for (int i = 0; i < NWL; ++i) {
        const int wp = 8 * (wave + 4 * i) + (lane >> 3);
        wswz[i] = ((lane & 7) ^ ((wp >> 1) & 7)) * 16;
        wofs[i] = kOOB;
        if (wp >= npx) continue;
        int seg, ih, iw;
        if (single) {
            int a = __mul24(wp, P.odiv) >> 16;
            const int b = wp - __mul24(a, OB);
            seg = 0;
            while (a >= P.TH) { a -= P.TH; ++seg; }
            ih = (a0 + a) * P.imul + P.dh0; iw = b * P.imul + P.dw0;
        } else {
            int wr = __mul24(wp, P.wdiv) >> 16;
            const int wc = wp - __mul24(wr, WW);
            seg = 0;
            while (wr >= P.WH) { wr -= P.WH; ++seg; }
            ih = a0 * P.imul + P.dhmin + wr; iw = P.dwmin + wc;
        }
        if ((unsigned)ih < (unsigned)IH && (unsigned)iw < (unsigned)IW) wofs[i] = (unsigned)(((n + seg) * IH + ih) * IW + iw) * (unsigned)(Cin * 2);
    }
    const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(P.in), 0, (int)((unsigned)P.nimg * IH * IW * Cin * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(P.wt), 0, (int)((unsigned)P.Ncol * P.ldw * 2), 0x00020000);
    const int frow = 8 * wave + (lane >> 3);       // filter row of this lane (row n0 + frow), four waves cover 32
    const unsigned fofs = n0 + frow < P.Ncol ? (unsigned)((n0 + frow) * P.ldw * 2) + (unsigned)(((lane & 7) ^ ((frow >> 1) & 7)) * 16) : kOOB;
    // lane u holds the filter and window offsets of tap u
    int wtab, atab;
    {
        const int u = min(lane, max(ntaps, 1) - 1), nts = P.nts, tr = nts == 3 ? (u * 11) >> 5 : nts == 2 ? u >> 1 : u, ts = u - tr * nts;
        wtab = ((P.r0 + P.rs * tr) * P.S + (P.s0 + P.ss * ts)) * Cin * 2;
        atab = single ? 0 : (P.dh0 + P.dhs * tr - P.dhmin) * WW + (P.dw0 + P.dws * ts - P.dwmin);
    }
    // channel slabs in the order of the kernel this launch is taken from: with a half last slab its odd workgroups start there
    const int first = P.rot && (((P.row_tile_start + (P.OA * P.OB * n + a0 * OB) / P.row_tile * P.col_tiles + n0 / P.col_tile)) & 1) ? nslab - 1 : 0;
    auto slab_of = [&](int i) { i += first; return i >= nslab ? i - nslab : i; };

    auto issue = [&](int grp) {
        char* const dst = lds + (grp & 1) * buf_bytes;
        for (int q = 0; q < gs && grp * gs + q < nslab; ++q) {
            const int ci = slab_of(grp * gs + q) * 64;
            const bool half = ci + 32 == Cin;      // a half slab: its upper chunks do not exist
            char* const w = dst + q * slab_bytes;
#pragma unroll
            for (int i = 0; i < NWL; ++i)
                if (8 * (wave + 4 * i) < npx) {
                    const unsigned o = wofs[i] == kOOB || (half && wswz[i] >= 64) ? kOOB : wofs[i] + (unsigned)(ci * 2 + wswz[i]);
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, (lds_ptr_t)(w + (wave + 4 * i) * 1024), 16, (int)o, 0, 0, 0);
                }
            const unsigned fo = fofs == kOOB || (half && ((lane & 7) ^ ((frow >> 1) & 7)) >= 4) ? kOOB : fofs + (unsigned)(ci * 2);
            for (int u = 0; u < ntaps; ++u)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_b, (lds_ptr_t)(w + win_bytes + u * 4096 + wave * 1024), 16,
                                                         (int)(fo == kOOB ? kOOB : fo + (unsigned)__builtin_amdgcn_readlane(wtab, u)), 0, 0, 0);
        }
    };

    // ---- this wave's micro-tile: pixels 32 * wave .. + 32 ------------------------------------------------------------
    const int lr = lane & 31, lk = lane >> 5;
    const bool active = wave * 32 < px;
    const int p = min(wave * 32 + lr, px - 1);
    int wrow;                                      // window pixel of tap (0, 0)
    int pa = __mul24(p, P.odiv) >> 16;
    const int pb = p - __mul24(pa, OB);
    int pseg = 0;
    while (pa >= P.TH) { pa -= P.TH; ++pseg; }     // (tiles of several images hold whole images: TH = OA then)
    if (single) wrow = p;
    else wrow = __mul24(pa * P.imul + pseg * P.WH, WW) + pb * P.imul;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    const int brow = lr * 128, bswz = (lr >> 1) & 7;
    auto fetch = [&](const char* w, int u, int lo, u32x4 (&a)[4], u32x4 (&b)[4]) {     // k-steps lo .. of tap u (4 of a whole slab)
        const int row = wrow + __builtin_amdgcn_readlane(atab, u), swz = (row >> 1) & 7;
        const char* const pw = w + row * 128;
        const char* const pf = w + win_bytes + u * 4096 + brow;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int c = lo + 2 * ks + lk;
            a[ks] = *reinterpret_cast<const u32x4*>(pw + ((c & 7) ^ swz) * 16);
            b[ks] = *reinterpret_cast<const u32x4*>(pf + ((c & 7) ^ bswz) * 16);
        }
    };
    if (ng > 0) {
        issue(0);
        for (int grp = 0; grp < ng; ++grp) {
            __builtin_amdgcn_s_waitcnt(0x0f70);    // vmcnt(0): this wave's share of the group has landed
            __syncthreads();                       // ... everyone's, and the other buffer has been read
            if (grp + 1 < ng) issue(grp + 1);
            if (!active) continue;
            for (int q = 0; q < gs && grp * gs + q < nslab; ++q) {
                const char* const w = lds + (grp & 1) * buf_bytes + q * slab_bytes;
                const bool half = slab_of(grp * gs + q) * 64 + 32 == Cin;
                const int nh = slab == 32 && !half ? 2 : 1, nks = slab == 32 || half ? 2 : 4;   // slabs of 32: the halves one after the other
                u32x4 a0r[4], b0r[4], a1r[4], b1r[4];
                auto mma = [&](const u32x4 (&a)[4], const u32x4 (&b)[4]) {
                    Mma<bf16_t, 32>::run(b[0], a[0], acc);
                    Mma<bf16_t, 32>::run(b[1], a[1], acc);
                    if (nks == 4) { Mma<bf16_t, 32>::run(b[2], a[2], acc); Mma<bf16_t, 32>::run(b[3], a[3], acc); }
                };
                const int steps = nh * ntaps;      // (half, tap)
                auto at = [&](int s, u32x4 (&a)[4], u32x4 (&b)[4]) {
                    const int h = s >= ntaps ? 1 : 0;
                    fetch(w, s - h * ntaps, h * 4, a, b);
                };
                at(0, a0r, b0r);
                for (int s = 0;;) {
                    at(min(s + 1, steps - 1), a1r, b1r);
                    mma(a0r, b0r);
                    if (++s == steps) break;
                    at(min(s + 1, steps - 1), a0r, b0r);
                    mma(a1r, b1r);
                    if (++s == steps) break;
                }
            }
        }
    }
    // ---- epilogue: a lane holds four times four consecutive channels of one pixel ------------------------------------
    if (!active || wave * 32 + lr >= px) return;
    const size_t row = ((size_t)(n + pseg) * P.OH + (size_t)((a0 + pa) * P.omul + P.ooh)) * P.OW + (size_t)(pb * P.omul + P.oow);
    bf16_t* __restrict__ out = reinterpret_cast<bf16_t*>(P.out) + row * P.Ncol + n0;
    const bf16_t* __restrict__ add0 = P.add0 ? reinterpret_cast<const bf16_t*>(P.add0) + row * P.Ncol + n0 : nullptr;
    const bf16_t* __restrict__ add1 = P.add1 ? reinterpret_cast<const bf16_t*>(P.add1) + row * P.Ncol + n0 : nullptr;
    uint2 x0[4], x1[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = 8 * r + 4 * lk;
        if (n0 + c >= P.Ncol) continue;
        if (add0) x0[r] = *reinterpret_cast<const uint2*>(add0 + c);
        if (add1) x1[r] = *reinterpret_cast<const uint2*>(add1 + c);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = 8 * r + 4 * lk;
        if (n0 + c >= P.Ncol) continue;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[4 * r + e];
        if (add0) { v[0] += __uint_as_float(x0[r].x << 16); v[1] += __uint_as_float(x0[r].x & 0xffff0000u); v[2] += __uint_as_float(x0[r].y << 16); v[3] += __uint_as_float(x0[r].y & 0xffff0000u); }
        if (add1) { v[0] += __uint_as_float(x1[r].x << 16); v[1] += __uint_as_float(x1[r].x & 0xffff0000u); v[2] += __uint_as_float(x1[r].y << 16); v[3] += __uint_as_float(x1[r].y & 0xffff0000u); }
        uint2 o;
        o.x = pack_bf16x2(v[0], v[1]); o.y = pack_bf16x2(v[2], v[3]);
        *reinterpret_cast<uint2*>(out + c) = o;
    }
}

// Sum and sum of squares per channel of a stored [M, C] tensor, in the order of the wide-layer kernels' epilogue: tiles of BM
// rows; in a tile every wave's 64 rows are three chains (rows q, q + 3, ... of its two groups of 32), the chains of a tile are
// added in fp32, the tiles in fp64.  A workgroup takes one tile and 64 channels; a thread one chain of eight channels.
__global__ __launch_bounds__(SC_NT) void stats_of_tiles_kernel(const TileStatsGroup g) {
    __shared__ float s_red[24 * 64 * 2];
    int pi = 0;
    for (int i = 1; i < g.nprob; ++i)
        if ((int)blockIdx.x >= g.p[i].block_start) pi = i;
    const TileStatsProb& P = g.p[pi];
    const int C = P.C, ncb = (C + 63) / 64;
    const int t = (int)blockIdx.x - P.block_start, tile = t / ncb, c0 = (t - tile * ncb) * 64;
    const int chains = P.BM / 64 * 3;
    const bf16_t* __restrict__ y = reinterpret_cast<const bf16_t*>(P.y);
    const int ncv = min(8, (C - c0) / 8);
    for (int i = threadIdx.x; i < chains * 8; i += SC_NT) {
        const int cv = i & 7, ch = i >> 3, w = ch / 3, q = ch - 3 * w;
        const int r0 = tile * P.BM + w * 64;
        float s1[8], s2[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) { s1[e] = 0.f; s2[e] = 0.f; }
        if (cv < ncv && r0 < P.M) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                u32x4 v[11];
#pragma unroll
                for (int k = 0; k < 11; ++k) {
                    const int row = r0 + h * 32 + q + 3 * k;
                    const bool is = q + 3 * k < 32 && row < P.M;
                    v[k] = Vec<bf16_t>::load_raw(y + (size_t)(is ? row : r0) * C + c0 + cv * 8);
                }
#pragma unroll
                for (int k = 0; k < 11; ++k) {
                    if (!(q + 3 * k < 32 && r0 + h * 32 + q + 3 * k < P.M)) continue;
                    float f[8];
                    Vec<bf16_t>::unpack(v[k], f);
#pragma unroll
                    for (int e = 0; e < 8; ++e) { s1[e] += f[e]; s2[e] = fmaf(f[e], f[e], s2[e]); }
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) { s_red[(ch * 64 + cv * 8 + e) * 2] = s1[e]; s_red[(ch * 64 + cv * 8 + e) * 2 + 1] = s2[e]; }
    }
    __syncthreads();
    const int c = threadIdx.x;
    if (c < 64 && c0 + c < C) {
        float a1 = 0.f, a2 = 0.f;
        for (int k = 0; k < chains; ++k) { a1 += s_red[(k * 64 + c) * 2]; a2 += s_red[(k * 64 + c) * 2 + 1]; }
        double* st = P.stats + (size_t)(tile % stat_stripes(C)) * 2 * C;
        atomicAdd(&st[c0 + c], (double)a1);
        atomicAdd(&st[C + c0 + c], (double)a2);
    }
}

}  // namespace

hipError_t launch_sconv(const SConvGroup& g, size_t lds, hipStream_t s) {
    if (g.total_tiles <= 0) return hipSuccess;
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    static OncePerDevice configured;
    if (const hipError_t e = raise_lds_limit(configured, {(const void*)sconv_kernel}, 160 * 1024); e != hipSuccess) return e;
    hipLaunchKernelGGL(sconv_kernel, dim3(g.total_tiles), dim3(SC_NT), lds, s, g);
    return hipGetLastError();
}
hipError_t launch_tile_stats(const TileStatsGroup& g, hipStream_t s) {
    if (g.total_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(stats_of_tiles_kernel, dim3(g.total_blocks), dim3(SC_NT), 0, s, g);
    return hipGetLastError();
}

}  // namespace lp
