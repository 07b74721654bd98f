// bf16 filter gradient of an image-facing layer (3 input channels, 16 / 32 / 64 output channels, 3 x 3 or 7 x 7) on gfx950.
//
//   dW[co][(r,s,c)] = sum over output pixels (n,ho,wo) of dY[n,ho,wo][co] * X[n, ho*stride - pad + r, wo*stride - pad + s][c]
//
// Three channels are six bytes: the general kernel fetched every element of the im2col matrix with a two-byte load of its own
// (ResNet-50's 7 x 7 stem at 64 samples: 286 us for 122 MB).  Here a workgroup walks over output rows.  The image rows a row of
// dY needs lie in LDS, split by channel and by column modulo the stride, so that eight neighbouring output pixels of one
// (r, s, c) are eight neighbouring elements: a fragment is five dwords shifted by none or one element (v_alignbit by a per-lane
// amount).  Rows stay in a ring of eight; a step to the next output row brings `stride` new ones (requested a row ahead).  The
// dY row goes straight into LDS, a row ahead too, and transposing reads make its fragments.
// Four waves share the columns (groups of 16 of (r,s,c)); every wave has all output channels.  A workgroup is two such sets, each
// with rows of its own, whose sums meet in LDS before the fp32 atomics: those all go to the same few thousand addresses and cost
// 0.1 us a workgroup (ResNet-50 at 64 samples: 512 workgroups of one set 106 us, 256 93; of two sets 256 88, 189 81, 128 92).
#include <algorithm>

#include "lp_kernels.h"
#include "lp_mma.h"

namespace lp {
namespace {

constexpr unsigned kOOB = 0x80000000u;
typedef __attribute__((address_space(3))) void* lds_ptr_t;
constexpr int WS_NT = 256, WS_SETS = 2, WS_SLOTS = 8, WS_U = 4, WS_CG = 3;      // dwords of new image rows a thread holds; column groups of a wave
constexpr int WS_C = 3;

struct StemGeom { int pxp, idxp, plane, ybytes, xbytes, set_bytes; };
__host__ __device__ inline StemGeom stem_geom(const WgradProb& P) {
    StemGeom g;
    g.pxp = (P.Wo + 31) & ~31;
    g.idxp = (g.pxp + P.R / P.stride + 8) & ~7;          // elements of a plane: every pixel of the padded row and every shift, 16-byte rows
    g.plane = WS_C * P.stride * g.idxp * 2;              // bytes of a row slot
    g.ybytes = g.pxp * P.Cout * 2;
    g.xbytes = WS_SLOTS * g.plane;
    g.set_bytes = (2 * g.ybytes + g.xbytes + 1023) & ~1023;
    return g;
}

template <int OFF> __device__ __forceinline__ u32x2 tr_read(unsigned a) {
    u32x2 r;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(a), "i"(OFF));
    return r;
}

}  // namespace

template <int COG>
__global__ __launch_bounds__(WS_SETS * WS_NT) void conv_wgrad_stem_kernel(const WgradGroup g) {
    constexpr int PITCH = COG * 32, CA = PITCH / 16, RPS = 1024 / PITCH;     // bytes of a dY row in LDS, its 16-byte chunks, rows of a wave-load
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_all[];
    const int set = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WS_NT), tid = (int)threadIdx.x - set * WS_NT;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int pi = 0;
    for (int i = 1; i < g.nprob; ++i)
        if ((int)blockIdx.x >= g.p[i].tile_start) pi = i;
    const WgradProb& P = g.p[pi];
    const StemGeom G = stem_geom(P);
    const int Ho = P.Ho, Wo = P.Wo, IH = P.IH, IW = P.IW, S = P.stride, R = P.R, pad = P.pad, Kg = P.Kg;
    const int units = P.M / Wo;                          // output rows
    // this set's output rows; both sets take the same number of steps
    const int steps = (P.kchunk + WS_SETS - 1) / WS_SETS;
    const int b0 = ((int)blockIdx.x - P.tile_start) * P.kchunk, b1 = min(units, b0 + P.kchunk);
    const int u0 = min(b1, b0 + set * steps), u1 = min(b1, u0 + steps);
    unsigned char* const smem = smem_all + set * G.set_bytes;
    unsigned char* const xs = smem + 2 * G.ybytes;
    const __amdgpu_buffer_rsrc_t rsrc_y = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(P.dy), 0, P.M * P.Cout * 2, 0x00020000);

    // ---- dY row of a unit: LDS bytes in order, the 32-byte channel pairs of a row swapped against bank conflicts
    auto load_y = [&](int u, int buf) __attribute__((always_inline)) {
        for (int q = wave; q < G.ybytes / 1024; q += 4) {
            const int px = q * RPS + lane / CA, c = lane % CA;
            const int f = COG == 4 ? ((px >> 1) & 1) | (((px >> 3) & 1) << 1) : COG == 2 ? (px >> 3) & 1 : 0;
            const unsigned off = px < Wo ? (unsigned)(((u * Wo + px) * P.Cout + ((c >> 1) ^ f) * 16 + (c & 1) * 8) * 2) : kOOB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_y, (lds_ptr_t)(smem + buf * G.ybytes + q * 1024), 16, (int)off, 0, 0, 0);
        }
    };
    // ---- image rows: dword i of a row is elements 2i, 2i + 1; element e is channel e % 3 of column e / 3
    const int rowdw = IW * WS_C / 2, maxcol = S * (Wo - 1) + R - 1;
    const unsigned* __restrict__ x = reinterpret_cast<const unsigned*>(P.x);
    auto fetch = [&](int n, int ih, int i) __attribute__((always_inline)) {
        return (unsigned)ih < (unsigned)IH ? x[(size_t)(n * IH + ih) * rowdw + i] : 0u;
    };
    auto put = [&](int ih, int i, unsigned v) __attribute__((always_inline)) {
        unsigned char* const row = xs + ((ih + 8 * pad) & 7) * G.plane;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int e = 2 * i + h, col = (e * 43691) >> 17, c = e - col * 3, cp = col + pad;      // e / 3 (rows of at most 1024 pixels: e < 3072)
            const int idx = cp / S, par = cp - idx * S;
            if (cp <= maxcol) *reinterpret_cast<unsigned short*>(row + ((c * S + par) * G.idxp + idx) * 2) = (unsigned short)(h ? v >> 16 : v);
        }
    };

    // ---- columns of this wave: group wave + 4 * k, lane column (r, s, c)
    const int lq = lane & 15, lg = lane >> 4;
    int cr[WS_CG], cofs[WS_CG], csh[WS_CG];
#pragma unroll
    for (int k = 0; k < WS_CG; ++k) {
        const int j = min((wave + 4 * k) * 16 + lq, Kg - 1), tap = j / WS_C, c = j - tap * WS_C, r = tap / R, s = tap - r * R;
        const int sh = s / S, par = s - sh * S;
        cr[k] = r; csh[k] = (sh & 1) * 16;
        cofs[k] = ((c * S + par) * G.idxp + (sh & ~1) + 8 * lg) * 2;
    }
    const int ncg = (Kg + 15) / 16;
    const int nk = ncg > wave ? (ncg - wave + 3) / 4 : 0;                    // column groups of this wave
    unsigned ya[COG];
    {
        const int r = 8 * lg + (lq >> 2);
        const int f = COG == 4 ? ((r >> 1) & 1) | (((r >> 3) & 1) << 1) : COG == 2 ? (r >> 3) & 1 : 0;
#pragma unroll
        for (int i = 0; i < COG; ++i) ya[i] = (unsigned)(uintptr_t)(lds_ptr_t)smem + r * PITCH + 8 * (lq & 3) + ((i ^ f) << 5);
    }
    f32x4 acc[WS_CG][COG];
#pragma unroll
    for (int k = 0; k < WS_CG; ++k)
#pragma unroll
        for (int i = 0; i < COG; ++i) acc[k][i] = f32x4{0.f, 0.f, 0.f, 0.f};

    // columns outside the image and behind the last pixel stay zero
    for (int i = tid; i < G.xbytes / 16; i += WS_NT) *reinterpret_cast<u32x4*>(xs + i * 16) = u32x4{0u, 0u, 0u, 0u};
    if (u0 < u1) load_y(u0, 0);
    __syncthreads();
    for (int it = 0; it < steps; ++it) {
        const int u = u0 + it;
        const bool live = u < u1;
        const int n = u / Ho, ho = u - n * Ho, ih0 = ho * S - pad;
        if (live && (it == 0 || ho == 0)) {              // all rows of this unit
            for (int i = tid; i < R * rowdw; i += WS_NT) { const int r = i / rowdw, d = i - r * rowdw; put(ih0 + r, d, fetch(n, ih0 + r, d)); }
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);              // vmcnt(0): the dY row is in LDS
        __syncthreads();
        // the next unit's rows are requested ahead of this one's products
        const bool more = u + 1 < u1;
        if (more) load_y(u + 1, (it + 1) & 1);
        const int lo = max(ih0 + R, ih0 + S), nnew = more && ho + 1 < Ho ? ih0 + S + R - lo : 0;
        unsigned nv[WS_U];
#pragma unroll
        for (int q = 0; q < WS_U; ++q) {
            const int i = tid + q * WS_NT, r = i / rowdw, d = i - r * rowdw;
            nv[q] = r < nnew ? fetch(n, lo + r, d) : 0u;
        }
        int base[WS_CG];
#pragma unroll
        for (int k = 0; k < WS_CG; ++k) base[k] = ((ih0 + cr[k] + 8 * pad) & 7) * G.plane + cofs[k];
        const unsigned yb = (unsigned)((it & 1) * G.ybytes);
        if (live && nk > 0) {
            for (int ks = 0; ks < G.pxp / 32; ++ks) {
                u32x2 ar[COG][2];
#pragma unroll
                for (int i = 0; i < COG; ++i) {
                    const unsigned a = ya[i] + yb + (unsigned)(ks * 32 * PITCH);
                    ar[i][0] = tr_read<0>(a); ar[i][1] = tr_read<4 * PITCH>(a);
                }
                unsigned d[WS_CG][5];
#pragma unroll
                for (int k = 0; k < WS_CG; ++k) {
                    const unsigned* const p = reinterpret_cast<const unsigned*>(xs + base[k] + ks * 64);
#pragma unroll
                    for (int e = 0; e < 5; ++e) d[k][e] = p[e];
                }
                __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0)
#pragma unroll
                for (int i = 0; i < COG; ++i) asm volatile("" : "+v"(ar[i][0]), "+v"(ar[i][1]));
#pragma unroll
                for (int k = 0; k < WS_CG; ++k) {
                    if (k >= nk) continue;
                    u32x4 b;
#pragma unroll
                    for (int e = 0; e < 4; ++e) b[e] = __builtin_amdgcn_alignbit(d[k][e + 1], d[k][e], csh[k]);
#pragma unroll
                    for (int i = 0; i < COG; ++i) Mma<bf16_t, 16>::run(u32x4{ar[i][0][0], ar[i][0][1], ar[i][1][0], ar[i][1][1]}, b, acc[k][i]);
                }
            }
        }
        __syncthreads();                                 // the rows of this unit have been read
#pragma unroll
        for (int q = 0; q < WS_U; ++q) {
            const int i = tid + q * WS_NT, r = i / rowdw, d = i - r * rowdw;
            if (r < nnew) put(lo + r, d, nv[q]);
        }
    }

    // (the loop ends with a barrier: nobody reads the operands any more)
    f32x4* const sum = reinterpret_cast<f32x4*>(smem_all) + (wave * WS_CG * COG) * 64 + lane;
    if (set == 1) {
#pragma unroll
        for (int k = 0; k < WS_CG; ++k)
#pragma unroll
            for (int i = 0; i < COG; ++i) sum[(k * COG + i) * 64] = acc[k][i];
    }
    __syncthreads();
    if (set == 1) return;
#pragma unroll
    for (int k = 0; k < WS_CG; ++k)
#pragma unroll
        for (int i = 0; i < COG; ++i) acc[k][i] += sum[(k * COG + i) * 64];
    float* const dw = P.dw;
#pragma unroll
    for (int k = 0; k < WS_CG; ++k) {
        const int col = (wave + 4 * k) * 16 + lq;
        if (col >= Kg) continue;
#pragma unroll
        for (int i = 0; i < COG; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) atomicAdd(dw + (size_t)(i * 16 + 4 * lg + e) * Kg + col, acc[k][i][e]);
    }
}

// The layers this kernel takes: those a network has, 3 x 3 with stride 1, 2 or 4 (modules and AuxNets) and 7 x 7 with stride 2.
// The image has to be aligned to four bytes as well, which the caller sees to.
bool wgrad_stem_ok(const WgradProb& p) {
    if (p.Cin != WS_C || (p.Cout != 16 && p.Cout != 32 && p.Cout != 64)) return false;
    const bool r3 = p.R == 3 && (p.stride == 1 || p.stride == 2 || p.stride == 4), r7 = p.R == 7 && p.stride == 2;
    if (p.R != p.S || !(r3 || r7) || p.pad != p.R / 2 || p.Wo > 256 || p.IW > 1024) return false;
    if ((p.IW * WS_C) % 2 || std::min(p.stride, p.R) * (p.IW * WS_C / 2) > WS_U * WS_NT || (p.Kg + 15) / 16 > 4 * WS_CG) return false;
    if ((double)p.M * p.Cout * 2.0 >= 2.0e9) return false;
    return stem_geom(p).set_bytes <= 64 * 1024;
}

hipError_t launch_wgrad_stem(const WgradGroup& g, hipStream_t s) {
    if (g.total_tiles <= 0) return hipSuccess;
    size_t lds = (size_t)4 * WS_CG * (g.p[0].Cout / 16) * 64 * 16;       // the second set's sums
    for (int i = 0; i < g.nprob; ++i) lds = std::max(lds, (size_t)WS_SETS * stem_geom(g.p[i]).set_bytes);
    static OncePerDevice configured;
    if (const hipError_t e = raise_lds_limit(configured, {(const void*)conv_wgrad_stem_kernel<1>, (const void*)conv_wgrad_stem_kernel<2>,
                                                          (const void*)conv_wgrad_stem_kernel<4>}, WS_SETS * 64 * 1024); e != hipSuccess) return e;
    const dim3 grid(g.total_tiles), block(WS_SETS * WS_NT);
    switch (g.p[0].Cout) {
        case 16: hipLaunchKernelGGL(conv_wgrad_stem_kernel<1>, grid, block, lds, s, g); break;
        case 32: hipLaunchKernelGGL(conv_wgrad_stem_kernel<2>, grid, block, lds, s, g); break;
        default: hipLaunchKernelGGL(conv_wgrad_stem_kernel<4>, grid, block, lds, s, g); break;
    }
    return hipGetLastError();
}

}  // namespace lp
