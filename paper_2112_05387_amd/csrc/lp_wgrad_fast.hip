// bf16 filter-gradient kernel for the wide 3x3 stride-1 layers on gfx950.
//
//   dW[co][r][s][ci] = sum over pixels m=(n,oh,ow) of dY[m][co] * X[n, oh+r-1, ow+s-1][ci]
//
// The reduction runs over pixels, and both operands are stored pixel-major ([pixel][channel]), so a k-tile of
// pixels of either operand is a run of whole channel rows: it is fetched with direct-to-LDS loads of 1 KiB per wave
// instruction (contiguous in memory, not the 64-byte gathers of the forward operand) and lands in LDS in its
// natural [pixel][channel] order.  The MFMA wants the reduction index contiguous inside a lane, i.e. the
// transpose; ds_read_tr16_b64 delivers exactly that: within 16 lanes it reads a 4-pixel x 16-channel block and
// hands lane c the 4 pixels of channel c.
//
// One block (512 threads, 8 waves, two per SIMD) owns a 160 (co) x 160 (ci) filter tile for the three taps of one filter row r
// and a chunk of the pixel range; partial sums are added to dW with fp32 atomics (split-K).  The 30 columns (ten groups of 16
// channels x 3 taps) fall into halves of five channel groups, and a half into a set of 8 columns (two groups, two taps of the
// third) and one of 7 (its third tap, the other two groups): wave (wc, half, set) has 80 co x 8 or 7 columns of 5
// v_mfma_f32_16x16x32_bf16 micro-tiles (160 or 140 accumulators), and the two waves of a SIMD are the two sets of one half.
// The taps of a filter row read the same pixels shifted by one, so a lane reads ten pixels of a channel once (three transposing
// reads) and makes the three fragments of eight from them: tap 0 as they are, tap 2 from the second register on, tap 1 by four
// v_alignbit.  LDS reads per k-step of 32 pixels: 152 instead of the 240 that twelve waves of 80 x 80 with a fragment per tap
// took (LDS bandwidth and the wait for the first fragments were what the matrix cores stood still for).  Five layers of
// 131072 pixels x 160 channels in one launch: 351 -> 282 us (1.07 PFLOP/s); 32768 x 320: 342 -> 275; 8192 x 640: 301 -> 250.
//
// A ring stage holds 64 pixels: the dY rows of pixels m0..m0+63 and ONE window of X shared by the three taps,
// the 66 pixels m0-1+(r-1)W .. m0+64+(r-1)W (flattened pixel index; tap s of pixel m reads window row m-m0+s).
// What the flattened window cannot express is patched in two places: window pixels whose image row is outside the
// image for this filter row are loaded as zeros (out-of-range offsets), and the column wrap of taps 0 and 2 (the
// left neighbour of column 0 is the last pixel of the previous row) is masked in the fragments.  One barrier per
// stage, ahead of the products of its last channel group, so that the first reads of the next stage run under them.
// LDS rows are 320 B; the 32-byte channel pairs of a row swap places in rows with bit 3 set, which keeps the
// transposing reads of a half-wave (pixel rows p..p+3 and p+8..p+11) on distinct banks.
//
// Logical neighbours (the filter-row and channel tiles that read the same pixel chunk) go to one XCD and share its L2, and
// every XCD gets the same number of blocks (lp_wgsplit.h).
#include <algorithm>
#include <type_traits>

#include "lp_kernels.h"
#include "lp_mma.h"
#include "lp_wgsplit.h"

namespace lp {
namespace {

constexpr unsigned kOOB = 0x80000000u;      // byte offset beyond any buffer

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
typedef __attribute__((address_space(3))) void* lds_ptr_t;

template <int N> __device__ __forceinline__ void wait_vmcnt() {
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// n / d for n < 2^31 with the (mul, shift) pair of fastdiv_make
__device__ __forceinline__ unsigned fastdiv(unsigned n, unsigned mul, unsigned shift) {
    return (__umulhi(n, mul) + n) >> shift;
}

constexpr int WF_NW = 8, WF_NT = 512, WF_BK = 64;    // pixels per ring stage (two MFMA k-steps of 32)
constexpr int WF_TILE = 160;                         // channels per operand tile
constexpr int WF_ROW = WF_TILE * 2;                  // bytes per LDS row
constexpr int WF_Y_BYTES = WF_BK * WF_ROW;           // dY rows of a stage: 20 KiB = 20 wave-loads
constexpr int WF_Y_SLABS = WF_Y_BYTES / 1024;
constexpr int WF_X_ROWS = WF_BK + 2;                 // window rows of a stage
constexpr int WF_X_SLABS = (WF_X_ROWS * WF_ROW + 1023) / 1024;     // 21 wave-loads
constexpr int WF_STAGE_BYTES = WF_Y_BYTES + WF_X_SLABS * 1024;
constexpr int WF_STAGES = 3;
constexpr int WF_SLABS = WF_Y_SLABS + WF_X_SLABS;    // 41 wave-loads per stage
constexpr int WF_LPW = (WF_SLABS + WF_NW - 1) / WF_NW;   // at most 6 per wave
constexpr int WF_LDS = WF_STAGES * WF_STAGE_BYTES + 1024;      // (a read's last two window rows, which nobody uses, lie behind the stage)

}  // namespace

// (mul, shift) with n / d == (mulhi(n, mul) + n) >> shift for every n < 2^31 (d >= 1)
void fastdiv_make(unsigned d, unsigned* mul, unsigned* shift) {
    unsigned s = 0;
    while ((1ull << s) < d) ++s;
    *shift = s;
    *mul = (unsigned)((((1ull << s) - d) << 32) / d + 1);
}

// Parameter update of a finished 160 (co) x 3 taps x 160 (ci) gradient tile by the whole workgroup: 480 runs of up to 160
// consecutive channels.  Not inlined: the kernel's registers are allotted for its main loop, and this runs once per
// tile in one workgroup, after the accumulators are dead.
__device__ __attribute__((noinline)) void wgrad_fast_update_tile(void* w, float* vel, float* master, const float* dw, int co0,
                                                                 int ci0, int r, int Cin, int Cout, bool lowp, float lr,
                                                                 float momentum, float wd, int tid) {
    const SgdCoef c{lr, momentum, wd, lowp};
    const int nrows = 3 * min(WF_TILE, Cout - co0), ncols = min(WF_TILE, Cin - ci0);
    sgd_update_tile<WF_NT, 5>(w, vel, master, dw, nrows, ncols, true,
                              [=](int q) { const int co = co0 + q / 3, s = q - (q / 3) * 3; return ((size_t)co * 9 + r * 3 + s) * Cin + ci0; },
                              c, tid);
}

// What a wave reads, multiplies and adds up; see the head of the file.  TY: which of the two column sets (8 or 7 columns of 16
// channels x one tap).
template <int TY> struct WfCols {
    static constexpr int NC = TY == 0 ? 8 : 7;
    static constexpr int group(int gi) { return TY == 0 ? gi : gi + 2; }           // channel group of sixteen inside the half
    static constexpr int tap0(int gi) { return TY == 1 && gi == 0 ? 2 : 0; }       // first tap of the group
    static constexpr int ntap(int gi) { return TY == 0 ? (gi == 2 ? 2 : 3) : (gi == 0 ? 1 : 3); }
    static constexpr int col(int gi) { return TY == 0 ? 3 * gi : (gi == 0 ? 0 : 3 * gi - 2); }     // accumulator column of the first tap
};

// The transposing LDS read as inline assembly with explicit lgkmcnt waits.  Through the compiler's builtin the read carries no
// memory operand, so the waitcnt pass cannot tell it from the in-flight direct-to-LDS loads and puts s_waitcnt vmcnt(0) in
// front of it.  The compiler does not know that the result is pending: nothing may touch it before the wait that covers it,
// and the empty asm behind that wait is where its value becomes usable.  No read is in flight over a back edge.
template <int OFF> __device__ __forceinline__ u32x2 tr_read(unsigned a) {
    u32x2 r;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(a), "i"(OFF));
    return r;
}
template <int N> __device__ __forceinline__ void wait_lgkm() { __builtin_amdgcn_s_waitcnt(0xc07f | (N << 8)); }

template <int TY, class Load>
__device__ __forceinline__ void wgrad_fast_loop(unsigned lds0, int nk, int k_begin, int W, unsigned mulW, unsigned shW, int lane, int wc, int half,
                                                bool six, const Load& issue_load, f32x4 (&acc)[5][WfCols<TY>::NC]) {
    typedef WfCols<TY> C;
    const int lq = lane & 15, lg = lane >> 4;
    const int lrow = 8 * lg + (lq >> 2);                 // this lane's row inside a 32-pixel k-step
    const int sw = (lg & 1) * 32;
    // dY: pairs 5 * wc + i, row bit 3 = lg & 1 in both halves of a fragment; the parity of i = 0 is that of wc
    const unsigned a0 = lds0 + lrow * WF_ROW + 8 * (lq & 3) + 160 * wc;
    const unsigned ae = wc ? a0 - sw : a0 + sw, ao = wc ? a0 + sw : a0 - sw;
    // X: pairs 5 * half + group; rows 0..7 of the lane with row bit 3 = lg & 1, rows 8..11 with the other value
    const unsigned x0 = lds0 + WF_Y_BYTES + lrow * WF_ROW + 8 * (lq & 3) + 160 * half;
    const unsigned xe = half ? x0 - sw : x0 + sw, xo = half ? x0 + sw : x0 - sw;
    const unsigned ye = half ? x0 - (32 - sw) : x0 + (32 - sw), yo = half ? x0 + (32 - sw) : x0 - (32 - sw);

    u32x2 a_lo[5], a_hi[5], x[3], xn[3];
    u32x4 af[5];
    unsigned m0[4], m2[4];                               // column wrap: element k of the lane's 8 is invalid for tap 0 at column 0, for tap 2 at column W - 1
    auto masks = [&](int k0) __attribute__((always_inline)) {
        const int ow = k0 - (int)fastdiv((unsigned)k0, mulW, shW) * W;
        if (W >= 8) {                                    // at most one of the 8 is bad: one half of one register
            int e0 = ow == 0 ? 0 : W - ow;
            const int e2 = W - 1 - ow;
            const unsigned h0 = (e0 & 1) ? 0x0000ffffu : 0xffff0000u, h2 = (e2 & 1) ? 0x0000ffffu : 0xffff0000u;
#pragma unroll
            for (int d = 0; d < 4; ++d) { m0[d] = (e0 >> 1) == d ? h0 : 0xffffffffu; m2[d] = (e2 >> 1) == d ? h2 : 0xffffffffu; }
        } else {
            unsigned b0 = 0, b2 = 0;
            for (int e = ow == 0 ? 0 : W - ow; e < 8; e += W) b0 |= 1u << e;
            for (int e = W - 1 - ow; e < 8; e += W) b2 |= 1u << e;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                m0[d] = ((b0 >> (2 * d)) & 1u ? 0u : 0xffffu) | ((b0 >> (2 * d)) & 2u ? 0u : 0xffff0000u);
                m2[d] = ((b2 >> (2 * d)) & 1u ? 0u : 0xffffu) | ((b2 >> (2 * d)) & 2u ? 0u : 0xffff0000u);
            }
        }
    };
    const bool fixed_masks = 32 % W == 0;                // the same in every k-step
    masks(k_begin + 8 * lg);

#define WF_READ_A(i, sub) do { \
        constexpr int o_ = 32 * (i) + (sub) * 32 * WF_ROW; \
        a_lo[i] = tr_read<o_>(((i) & 1 ? ao : ae) + sb); a_hi[i] = tr_read<o_ + 4 * WF_ROW>(((i) & 1 ? ao : ae) + sb); } while (0)
#define WF_READ_X(dst, gi, sub) do { \
        constexpr int g_ = C::group(gi), o_ = 32 * g_ + (sub) * 32 * WF_ROW; \
        dst[0] = tr_read<o_>((g_ & 1 ? xo : xe) + sb); dst[1] = tr_read<o_ + 4 * WF_ROW>((g_ & 1 ? xo : xe) + sb); \
        dst[2] = tr_read<o_ + 8 * WF_ROW>((g_ & 1 ? yo : ye) + sb); } while (0)
    auto have_x = [](u32x2 (&v)[3]) __attribute__((always_inline)) { asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2])); };
    auto have_a = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            asm volatile("" : "+v"(a_lo[i]), "+v"(a_hi[i]));
            af[i] = u32x4{a_lo[i][0], a_lo[i][1], a_hi[i][0], a_hi[i][1]};
        }
    };
    // the taps of a channel group share the lane's ten pixels: tap 0 takes 0..7, tap 1 1..8, tap 2 2..9
    auto mma_group = [&](const u32x2 (&v)[3], auto gi_) __attribute__((always_inline)) {
        constexpr int gi = decltype(gi_)::value;
#pragma unroll
        for (int q = 0; q < C::ntap(gi); ++q) {
            const int tap = C::tap0(gi) + q;
            u32x4 b;
            if (tap == 0) b = u32x4{v[0][0] & m0[0], v[0][1] & m0[1], v[1][0] & m0[2], v[1][1] & m0[3]};
            else if (tap == 2) b = u32x4{v[0][1] & m2[0], v[1][0] & m2[1], v[1][1] & m2[2], v[2][0] & m2[3]};
            else b = u32x4{__builtin_amdgcn_alignbit(v[0][1], v[0][0], 16), __builtin_amdgcn_alignbit(v[1][0], v[0][1], 16),
                           __builtin_amdgcn_alignbit(v[1][1], v[1][0], 16), __builtin_amdgcn_alignbit(v[2][0], v[1][1], 16)};
#pragma unroll
            for (int i = 0; i < 5; ++i) Mma<bf16_t, 16>::run(af[i], b, acc[i][C::col(gi) + q]);
        }
    };
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    typedef std::integral_constant<int, 2> I2;
#define WF_FENCE __builtin_amdgcn_sched_barrier(0)
#define WF_TIE_A(i) asm volatile("" : "+v"(a_lo[i]), "+v"(a_hi[i]))

    unsigned sb = 0;                                     // the stage being read
    WF_READ_A(0, 0); WF_READ_A(1, 0); WF_READ_A(2, 0); WF_READ_A(3, 0); WF_READ_A(4, 0);
    WF_READ_X(x, 0, 0);
    wait_lgkm<0>();
    have_a(); have_x(x);
    int st = 0;
    for (int kt = 0; kt < nk; ++kt) {
        int st_free = st + WF_STAGES - 1;                // the stage that stage kt - 1 used
        if (st_free >= WF_STAGES) st_free -= WF_STAGES;
        const int kn = kt + WF_STAGES - 1;
        // Six channel groups (three a k-step): one direct-to-LDS load of the stage two ahead, the next group's pixels and a part
        // of the next k-step's dY fragments are requested ahead of a group's products and waited for behind them.
        if (!fixed_masks && kt) masks(k_begin + kt * WF_BK + 8 * lg);
        issue_load(0, st_free, kn);
        WF_READ_X(xn, 1, 0); WF_READ_A(0, 1); WF_READ_A(1, 1); WF_FENCE;
        mma_group(x, I0()); WF_FENCE;
        wait_lgkm<0>(); have_x(xn); WF_TIE_A(0); WF_TIE_A(1);
        issue_load(1, st_free, kn);
        WF_READ_X(x, 2, 0); WF_READ_A(2, 1); WF_READ_A(3, 1); WF_FENCE;
        mma_group(xn, I1()); WF_FENCE;
        wait_lgkm<0>(); have_x(x); WF_TIE_A(2); WF_TIE_A(3);
        issue_load(2, st_free, kn);
        WF_READ_X(xn, 0, 1); WF_READ_A(4, 1); WF_FENCE;
        mma_group(x, I2()); WF_FENCE;
        wait_lgkm<0>(); have_x(xn); have_a();
        if (!fixed_masks) masks(k_begin + kt * WF_BK + 32 + 8 * lg);
        issue_load(3, st_free, kn);
        WF_READ_X(x, 1, 1); WF_FENCE;
        mma_group(xn, I0()); WF_FENCE;
        wait_lgkm<0>(); have_x(x);
        issue_load(4, st_free, kn);
        WF_READ_X(xn, 2, 1); WF_FENCE;
        mma_group(x, I1()); WF_FENCE;
        wait_lgkm<0>(); have_x(xn);                      // this wave has read all it needs of the stage
        issue_load(5, st_free, kn);
        if (six) wait_vmcnt<6>(); else wait_vmcnt<5>();  // stage kt + 1 landed (this wave's share)
        __builtin_amdgcn_s_barrier();                    // ... everyone's; and stage kt is free
        if (++st == WF_STAGES) st = 0;
        sb = (unsigned)(st * WF_STAGE_BYTES);
        WF_READ_A(0, 0); WF_READ_A(1, 0); WF_READ_A(2, 0); WF_READ_A(3, 0); WF_READ_A(4, 0);
        WF_READ_X(x, 0, 0); WF_FENCE;
        mma_group(xn, I2()); WF_FENCE;
        wait_lgkm<0>(); have_a(); have_x(x);
    }
#undef WF_READ_A
#undef WF_READ_X
#undef WF_TIE_A
#undef WF_FENCE
}

// partial sums of a wave -> dW[co][r][s][ci]
template <int TY>
__device__ __forceinline__ void wgrad_fast_store(float* __restrict__ dw, const f32x4 (&acc)[5][WfCols<TY>::NC], int r, int co0, int ci0, int Cin, int Cout,
                                                 bool add, int lane, int wc, int half) {
    typedef WfCols<TY> C;
    const int lq = lane & 15, lg = lane >> 4;
#pragma unroll
    for (int i = 0; i < 5; ++i)
#pragma unroll
        for (int gi = 0; gi < 3; ++gi)
#pragma unroll
            for (int q = 0; q < C::ntap(gi); ++q) {
                const int ci = ci0 + 80 * half + 16 * C::group(gi) + lq, tap = r * 3 + C::tap0(gi) + q;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int co = co0 + 80 * wc + 16 * i + 4 * lg + e;
                    if (co < Cout && ci < Cin) {
                        float* const dst = dw + ((size_t)co * 9 + tap) * Cin + ci;
                        const float v = acc[i][C::col(gi) + q][e];
                        if (add) atomicAdd(dst, v);
                        else *dst = v;
                    }
                }
            }
}

__global__ __launch_bounds__(WF_NT, 2) void conv_wgrad_fast_kernel(const WgradGroup g) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int pi = 0, L = 0;
    if (!xcd_piece((int)blockIdx.x, g.nprob, [&](int i) { return g.p[i].ntile * g.p[i].ksplit; }, pi, L)) return;
    const WgradProb& P = g.p[pi];
    // (block-uniform quotients: the division runs on the vector ALU; readfirstlane puts the results into scalar registers)
    const int split = __builtin_amdgcn_readfirstlane(L / P.ntile), tile = P.tile0 + L - split * P.ntile;
    const int tile_m = __builtin_amdgcn_readfirstlane(tile / P.tiles_n), tile_n = tile - tile_m * P.tiles_n;
    const int r = tile_n % 3, ci0 = (tile_n / 3) * WF_TILE, co0 = tile_m * WF_TILE;
    const int Cin = P.Cin, Cout = P.Cout, H = P.IH, W = P.IW;
    const int k_begin = split * P.kchunk;
    const int k_end = min(P.M, k_begin + P.kchunk);
    const int nk = (k_end - k_begin + WF_BK - 1) / WF_BK;

    const __amdgpu_buffer_rsrc_t rsrc_y = make_rsrc(P.dy, (unsigned)((size_t)P.M * Cout * 2));
    const __amdgpu_buffer_rsrc_t rsrc_x = make_rsrc(P.x, (unsigned)((size_t)P.M * Cin * 2));

    // ---- loads: wave-load q = wave + 8*i; q < 20: bytes [1024*q, +1024) of the dY rows, else of the X window.
    // Lane l supplies the 16 bytes that land at +16*l, i.e. row b/320 and the (swizzled) channel chunk of that row.
    // (Everything is recomputed per stage rather than kept in registers: the accumulators need them.)
    const bool six = wave + WF_NW * (WF_LPW - 1) < WF_SLABS;
    const int Mtot = P.M;
    // the division constants in scalar registers for good (left alone, the compiler re-reads them from the kernel
    // arguments inside the loops and every re-read is a wait on the scalar cache)
    unsigned mulW = P.mulW, shW = P.shW, mulH = P.mulH, shH = P.shH;
    asm volatile("" : "+s"(mulW), "+s"(shW), "+s"(mulH), "+s"(shH));
    auto issue_load = [&](int i, int st, int kt) __attribute__((always_inline)) {
        const int mt = k_begin + kt * WF_BK;                 // first pixel of the stage (beyond k_end: all zeros)
        const bool live = mt < k_end;
        const int q = wave + WF_NW * i;
        if (q >= WF_SLABS) return;
        const bool isx = q >= WF_Y_SLABS;
        const int b = (isx ? q - WF_Y_SLABS : q) * 1024 + lane * 16;
        const int row = b / WF_ROW, cb = b - row * WF_ROW;
        const int ce = ((((cb >> 5) ^ ((row >> 3) & 1)) << 5) | (cb & 31)) >> 1;   // first channel fetched
        unsigned char* dst = smem + st * WF_STAGE_BYTES + q * 1024;
        if (!isx) {
            const bool ok = live && (co0 + ce < Cout) && (mt + row < k_end);
            const unsigned off = ok ? (unsigned)(((mt + row) * Cout + co0 + ce) * 2) : kOOB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_y, (lds_ptr_t)dst, 16, (int)off, 0, 0, 0);
        } else {
            // window pixel p; zero unless it exists and its image row hp has hp-(r-1) inside the image
            const int p = mt + row - 1 + (r - 1) * W;
            const unsigned t = fastdiv((unsigned)p, mulW, shW);
            const int hp = (int)t - (int)fastdiv(t, mulH, shH) * H;
            const bool ok = live && row < WF_X_ROWS && (ci0 + ce < Cin) && p >= 0 && p < Mtot && (unsigned)(hp - (r - 1)) < (unsigned)H;
            const unsigned off = ok ? (unsigned)((p * Cin + ci0 + ce) * 2) : kOOB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_x, (lds_ptr_t)dst, 16, (int)off, 0, 0, 0);
        }
    };
    const int wc = wave & 1, half = (wave >> 1) & 1;     // waves w and w + 4 (one SIMD) have the two column sets
    auto work = [&](auto ty_) __attribute__((always_inline)) {
        constexpr int TY = decltype(ty_)::value;
        f32x4 acc[5][WfCols<TY>::NC];
#pragma unroll
        for (int i = 0; i < 5; ++i)
#pragma unroll
            for (int j = 0; j < WfCols<TY>::NC; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        wgrad_fast_loop<TY>((unsigned)(uintptr_t)(lds_ptr_t)smem, nk, k_begin, W, mulW, shW, lane, wc, half, six, issue_load, acc);
        wait_vmcnt<0>();                 // trailing out-of-range loads still write zeros into LDS
        wgrad_fast_store<TY>(P.dw, acc, r, co0, ci0, Cin, Cout, P.ksplit > 1, lane, wc, half);
    };
    // (every workgroup has at least one stage: k_begin < k_end)
#pragma unroll
    for (int kt = 0; kt < WF_STAGES - 1; ++kt)
#pragma unroll
        for (int i = 0; i < WF_LPW; ++i) issue_load(i, kt, kt);
    // this wave's share of stage 0 landed once at most one stage of its loads is outstanding
    if (six) wait_vmcnt<6>(); else wait_vmcnt<5>();
    __builtin_amdgcn_s_barrier();
    if (wave < 4) work(std::integral_constant<int, 0>());
    else work(std::integral_constant<int, 1>());
    // ---- parameter update by the workgroup that completed this tile (Cin and Cout are multiples of 8: whole vectors)
    if (P.w) {
        __shared__ unsigned s_last;
        // the thread index afresh (not the one of the kernel's head: that would stay live through the main loop)
        const int t2 = wave * 64 + (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        // This workgroup's partial sums must have been added before its ticket is taken: they are device-scope atomics
        // (performed at the memory side, not held in this XCD's L2), so waiting for their acknowledgement is all a release
        // needs here -- a device-scope fence would also write back and invalidate the whole L2 under the other workgroups
        // (measured: the step took 2.4 ms longer).
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __syncthreads();
        if (P.ksplit > 1) {
            if (t2 == 0) s_last = __hip_atomic_fetch_add(P.cnt + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(P.ksplit - 1);
            __syncthreads();
            if (!s_last) return;
        }
        wgrad_fast_update_tile(P.w, P.vel, P.master, P.dw, co0, ci0, r, Cin, Cout, g.lowp != 0, g.lr, g.momentum, g.wd, t2);
    }
}

hipError_t launch_wgrad_fast(const WgradGroup& g, hipStream_t s) {
    if (g.total_tiles <= 0) return hipSuccess;
    const size_t lds = WF_LDS;
    static OncePerDevice configured;
    if (const hipError_t e = raise_lds_limit(configured, {(const void*)conv_wgrad_fast_kernel}, (int)lds); e != hipSuccess) return e;
    hipLaunchKernelGGL(conv_wgrad_fast_kernel, dim3(xcd_grid(g.total_tiles)), dim3(WF_NT), lds, s, g);
    return hipGetLastError();
}

}  // namespace lp
