// bf16 filter gradients of the wide layers that are not 3x3 with stride 1 (1x1, strided, other widths) on gfx950.
//
//   dW[co][j] = sum over output pixels m of dY[m][co] * X[pixel of m at tap(j)][ci(j)],   j = (tap, ci)
//
// The general kernel gathers both operands through registers, 128 columns at a time, and waits for memory every 64 pixels
// (12 % MFMA utilisation on the 1x1 layers of ResNet-50).  Here, as in the kernel of the 3x3 layers, rows of channels go
// from memory straight into LDS as they lie there and transposing LDS reads make the fragments: both operands are stored
// pixel-major and the sum runs over the pixels.
// A block (256 threads, 2 x 2 waves) owns BM (128 or 64) output channels x 128 columns and a chunk of the pixels; its partial
// sums are added to dW with fp32 atomics, or stored where its chunk is the whole sum.  A ring stage is 64 pixels (32 or 24 KB);
// with a ring of two, two blocks (BM = 64: three, by LDS and registers) share a compute unit, and one's atomics and first loads run beside the other's products.
// A lane of a load always serves the same column, so the tap and the channel are found once; per stage it divides its pixel
// into (image, row, column), which a 1x1 layer without stride does not need.
// LDS rows are 256 B (64 channels: 128 B); the 32-byte channel pairs of a row trade places so that the eight rows of a
// half-wave's transposing read lie on distinct banks: pair p of row r sits at p ^ f(r), f = (r & 3) | (r >> 3 & 1) << 2
// (128 B: (r >> 1 & 1) | (r >> 3 & 1) << 1).
#include <algorithm>

#include "lp_kernels.h"
#include "lp_mma.h"
#include "lp_wgsplit.h"

namespace lp {
namespace {

constexpr unsigned kOOB = 0x80000000u;      // byte offset beyond any buffer
typedef __attribute__((address_space(3))) void* lds_ptr_t;

template <int N> __device__ __forceinline__ void wait_vmcnt() {
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
__device__ __forceinline__ unsigned fastdiv(unsigned n, unsigned mul, unsigned shift) { return (__umulhi(n, mul) + n) >> shift; }

// The transposing LDS read as inline assembly, waited for explicitly (see the kernel of the 3x3 layers): nothing may touch the
// result before the wait, and the empty asm behind the wait is where its value becomes usable.
template <int OFF> __device__ __forceinline__ u32x2 tr_read(unsigned a) {
    u32x2 r;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(a), "i"(OFF));
    return r;
}

constexpr int WT_NT = 256, WT_BK = 64, WT_BN = 128, WT_STAGES = 2;

}  // namespace

template <int BM, int STAGES>
__global__ __launch_bounds__(WT_NT, 2) void conv_wgrad_tile_kernel(const WgradGroup g) {
    constexpr int PA = BM * 2, PB = WT_BN * 2;           // bytes of an LDS row
    constexpr int A_BYTES = WT_BK * PA, STAGE = A_BYTES + WT_BK * PB;
    constexpr int LA = A_BYTES / 4096, LB = WT_BK * PB / 4096;        // wave-loads per wave and stage
    constexpr int FM = BM / 32, FN = 4;                  // micro-tiles of a wave
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int pi = 0, L = 0;
    if (!xcd_piece((int)blockIdx.x, g.nprob, [&](int i) { return g.p[i].ntile * g.p[i].ksplit; }, pi, L)) return;
    const WgradProb& P = g.p[pi];
    const int split = __builtin_amdgcn_readfirstlane(L / P.ntile), tile = P.tile0 + L - split * P.ntile;
    const int tile_m = __builtin_amdgcn_readfirstlane(tile / P.tiles_n), tile_n = tile - tile_m * P.tiles_n;
    const int co0 = tile_m * BM, j0 = tile_n * WT_BN;
    const int Cin = P.Cin, Cout = P.Cout, Kg = P.Kg, IH = P.IH, IW = P.IW, Ho = P.Ho, Wo = P.Wo, stride = P.stride;
    const int k_begin = split * P.kchunk, k_end = min(P.M, k_begin + P.kchunk);
    const int nk = (k_end - k_begin + WT_BK - 1) / WT_BK;
    const bool pointwise = P.R == 1 && stride == 1 && P.pad == 0;
    const __amdgpu_buffer_rsrc_t rsrc_y = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(P.dy), 0, P.M * Cout * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(P.x), 0, P.M / (Ho * Wo) * IH * IW * Cin * 2, 0x00020000);
    unsigned mulW = P.mulW, shW = P.shW, mulH = P.mulH, shH = P.shH;
    asm volatile("" : "+s"(mulW), "+s"(shW), "+s"(mulH), "+s"(shH));

    // ---- loads: wave-load q = wave + 4 * i of an operand is 1 KiB of LDS rows; a lane serves 16 bytes of one row, always the
    // same channels (bit 3 of the row is a bit of the wave's number)
    int ya, y_row, xa, x_dh = 0, x_dw = 0;
    bool y_ok, x_ok;
    {
        constexpr int CA = PA / 16;
        const int c = lane % CA, r = lane / CA;
        const int f = BM == 128 ? (r & 3) | (((wave >> 1) & 1) << 2) : ((r >> 1) & 1) | ((wave & 1) << 1);
        const int ch = co0 + ((c >> 1) ^ f) * 16 + (c & 1) * 8;
        y_ok = ch < Cout; y_row = wave * (1024 / PA) + r; ya = ch * 2;
    }
    const int x_row = wave * 4 + (lane >> 4);
    {
        const int c = lane & 15, f = (lane >> 4) | (((wave >> 1) & 1) << 2);
        const int j = j0 + ((c >> 1) ^ f) * 16 + (c & 1) * 8;
        x_ok = j < Kg;
        const int tap = pointwise ? 0 : (x_ok ? j : 0) / Cin, ci = j - tap * Cin, r = tap / P.S;
        x_dh = r - P.pad; x_dw = tap - r * P.S - P.pad;
        xa = ci * 2;
    }
    auto issue = [&](int st, int kt) __attribute__((always_inline)) {
        const int mt = k_begin + kt * WT_BK;             // beyond the chunk: zeros
        unsigned char* const S = smem + st * STAGE + wave * 1024;
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const int m = mt + y_row + i * (4096 / PA);
            const unsigned off = y_ok && m < k_end ? (unsigned)(m * Cout * 2 + ya) : kOOB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_y, (lds_ptr_t)(S + i * 4096), 16, (int)off, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            const int m = mt + x_row + i * 16;
            unsigned off = kOOB;
            if (pointwise) {
                if (x_ok && m < k_end) off = (unsigned)(m * Cin * 2 + xa);
            } else {
                const int t = (int)fastdiv((unsigned)m, mulW, shW), n = (int)fastdiv((unsigned)t, mulH, shH);
                const int ih = (t - n * Ho) * stride + x_dh, iw = (m - t * Wo) * stride + x_dw;
                if (x_ok && m < k_end && (unsigned)ih < (unsigned)IH && (unsigned)iw < (unsigned)IW) off = (unsigned)(((n * IH + ih) * IW + iw) * Cin * 2 + xa);
            }
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_x, (lds_ptr_t)(S + A_BYTES + i * 4096), 16, (int)off, 0, 0, 0);
        }
    };

    // ---- fragments: lane l, l' = l % 16, g = l / 16 supplies rows 8g + l'/4 (+4) and channels 4 * (l' % 4).. of a pair, and
    // receives channel l' of it, pixels 8g..8g+7
    const int wm = wave >> 1, wn = wave & 1, lq = lane & 15, lg = lane >> 4, lr = lq >> 2;
    const unsigned lds0 = (unsigned)(uintptr_t)(lds_ptr_t)smem;
    unsigned aa[FM], ba[FN];
    {
        const int r = 8 * lg + lr;
        const int fa = BM == 128 ? lr | ((lg & 1) << 2) : (lr >> 1) | ((lg & 1) << 1), fb = lr | ((lg & 1) << 2);
#pragma unroll
        for (int i = 0; i < FM; ++i) aa[i] = lds0 + r * PA + 8 * (lq & 3) + (((wm * FM + i) ^ fa) << 5);
#pragma unroll
        for (int j = 0; j < FN; ++j) ba[j] = lds0 + A_BYTES + r * PB + 8 * (lq & 3) + (((wn * FN + j) ^ fb) << 5);
    }
    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x2 a0[FM][2], b0[FN][2], a1[FM][2], b1[FN][2];
    auto read0 = [&](unsigned sb) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FM; ++i) { a0[i][0] = tr_read<0>(aa[i] + sb); a0[i][1] = tr_read<4 * PA>(aa[i] + sb); }
#pragma unroll
        for (int j = 0; j < FN; ++j) { b0[j][0] = tr_read<0>(ba[j] + sb); b0[j][1] = tr_read<4 * PB>(ba[j] + sb); }
    };
    auto read1 = [&](unsigned sb) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FM; ++i) { a1[i][0] = tr_read<32 * PA>(aa[i] + sb); a1[i][1] = tr_read<36 * PA>(aa[i] + sb); }
#pragma unroll
        for (int j = 0; j < FN; ++j) { b1[j][0] = tr_read<32 * PB>(ba[j] + sb); b1[j][1] = tr_read<36 * PB>(ba[j] + sb); }
    };
    auto have = [](u32x2 (&a)[FM][2], u32x2 (&b)[FN][2]) __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(0xc07f);              // lgkmcnt(0)
#pragma unroll
        for (int i = 0; i < FM; ++i) asm volatile("" : "+v"(a[i][0]), "+v"(a[i][1]));
#pragma unroll
        for (int j = 0; j < FN; ++j) asm volatile("" : "+v"(b[j][0]), "+v"(b[j][1]));
    };
    auto mma = [&](const u32x2 (&a)[FM][2], const u32x2 (&b)[FN][2]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int i = 0; i < FM; ++i)
                Mma<bf16_t, 16>::run(u32x4{a[i][0][0], a[i][0][1], a[i][1][0], a[i][1][1]}, u32x4{b[j][0][0], b[j][0][1], b[j][1][0], b[j][1][1]}, acc[i][j]);
    };

    // (every workgroup has at least one stage: k_begin < k_end)
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) issue(s, s);
    wait_vmcnt<(STAGES - 2) * (LA + LB)>();              // this wave's share of stage 0
    __builtin_amdgcn_s_barrier();
    read0(0);
    have(a0, b0);
    int st = 0;
    for (int kt = 0; kt < nk; ++kt) {
        int st_free = st + STAGES - 1;                   // the stage that stage kt - 1 used
        if (st_free >= STAGES) st_free -= STAGES;
        issue(st_free, kt + STAGES - 1);
        read1((unsigned)(st * STAGE));
        __builtin_amdgcn_sched_barrier(0);
        mma(a0, b0);
        __builtin_amdgcn_sched_barrier(0);
        have(a1, b1);                                    // this wave has read all of the stage
        wait_vmcnt<(STAGES - 2) * (LA + LB)>();          // stage kt + 1 landed (this wave's share)
        __builtin_amdgcn_s_barrier();                    // ... everyone's; and stage kt is free
        if (++st == STAGES) st = 0;
        read0((unsigned)(st * STAGE));
        __builtin_amdgcn_sched_barrier(0);
        mma(a1, b1);
        __builtin_amdgcn_sched_barrier(0);
        have(a0, b0);
    }
    wait_vmcnt<0>();                                     // trailing out-of-range loads still write zeros into LDS

    float* const dw = P.dw;
    const bool add = P.ksplit > 1;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int col = j0 + (wn * FN + j) * 16 + lq;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int co = co0 + (wm * FM + i) * 16 + 4 * lg + e;
                if (co < Cout && col < Kg) {
                    float* const dst = dw + (size_t)co * Kg + col;
                    if (add) atomicAdd(dst, acc[i][j][e]);
                    else *dst = acc[i][j][e];
                }
            }
        }
}

int wgrad_tile_rows(int Cout) { return Cout <= 64 ? 64 : 128; }

hipError_t launch_wgrad_tile(const WgradGroup& g, int rows, hipStream_t s) {
    if (g.total_tiles <= 0) return hipSuccess;
    const size_t lds = (size_t)WT_STAGES * WT_BK * (rows + WT_BN) * 2;
    auto k128 = conv_wgrad_tile_kernel<128, WT_STAGES>;
    auto k64 = conv_wgrad_tile_kernel<64, WT_STAGES>;
    static OncePerDevice configured;
    if (const hipError_t e = raise_lds_limit(configured, {(const void*)k128, (const void*)k64}, WT_STAGES * WT_BK * (128 + WT_BN) * 2); e != hipSuccess) return e;
    if (rows == 128) hipLaunchKernelGGL(k128, dim3(xcd_grid(g.total_tiles)), dim3(WT_NT), lds, s, g);
    else hipLaunchKernelGGL(k64, dim3(xcd_grid(g.total_tiles)), dim3(WT_NT), lds, s, g);
    return hipGetLastError();
}

}  // namespace lp
