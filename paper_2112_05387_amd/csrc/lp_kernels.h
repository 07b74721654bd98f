// Device-side problem descriptors and launch entry points of the local-step kernels (gfx950).
// Every kernel is a *grouped* launch: one grid covers the same operation of several modules, the
// per-module problems travel by value in the kernel arguments, and a workgroup finds its problem from
// a prefix table of tile counts.  That is how the K independent local steps of Sec. 4.1 share one GPU.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <initializer_list>

#include "lp_fwform.h"
#include "lp_once.h"

namespace lp {

constexpr int kMaxGroup = 16;   // problems per grouped launch (bounded by the 4 KiB kernel-argument block)

// ---------------------------------------------------------------------------------------------------
// Implicit-GEMM convolution, forward and data-gradient:  OUT[m, col] = sum_q A[m, q] * WT[col, q]
//   m   -> (n, a, b) on a row grid [N][OA][OB];  q -> (tr, ts, ci) with ci fastest
//   A[m,q] = IN[n, a*imul + dh0 + dhs*tr, b*imul + dw0 + dws*ts, ci]      (zero outside the image)
//   WT[col,q] = wt[col*ldw + ((r0 + rs*tr)*S + (s0 + ss*ts))*Cin + ci]
//   OUT pixel = (n, a*omul + ooh, b*omul + oow) of an [N][OH][OW][Ncol] tensor
// Forward conv: imul = stride, dh0 = -pad, dhs = 1, full tap range, omul = 1.
// Data-gradient: IN = dY, wt = filters re-laid-out as [Cin][R][S][Cout]; stride 1: dh0 = pad, dhs = -1;
// stride 2: one problem per output parity class with the taps of matching parity (rs = 2).
struct ConvProb {
    const void* in;
    const void* wt;
    void* out;
    const void* add0;     // optional addends with the layout of out (skip-path gradients)
    const void* add1;
    double* stats;        // optional: [2*Ncol] per-column sum and sum of squares of the fp32 results
    int M, Ncol, Kg, Cin;
    int OA, OB, IH, IW, imul;
    int ntr, nts, dh0, dhs, dw0, dws;
    int r0, rs, s0, ss, S, ldw;
    int OH, OW, omul, ooh, oow;
    int tiles_m, tiles_n, tile_start;
};
struct ConvGroup {
    int nprob, total_tiles;
    ConvProb p[kMaxGroup];
};

// The same contraction for narrow layers (16 / 32 / 64 channels), with the batch-norm passes in front of it and behind it
// folded in (lp_fconv.hip).  What the taps read is a function of one or two stored tensors,
//   FX_PLAIN   in
//   FX_BN      [ReLU] bn(in)
//   FX_BN_ADD  [ReLU] (bn(in) + in2)
//   FX_BN_BN   [ReLU] (bn(in) + bn2(in2))
//   FX_BWD     the batch-norm backward of in = g at y = in2: k1*g' - k2*y + k3
// evaluated while the input window of a tile is copied to LDS, and stored to `side` (layout of in) by the tile that owns
// the pixel.  Behind the sum: optional addend, statistics of the stored result (ostats), and for a data-gradient the
// backward sums of up to two batch norms whose arriving gradient this result is (ey: the tensor they normalise).
enum FxMode { FX_PLAIN = 0, FX_BN, FX_BN_ADD, FX_BN_BN, FX_BWD };
struct FConvProb {
    const void *in, *in2;
    void* side;
    const double* stats; const float *gamma, *beta;          // the batch norm of `in` (FX_BWD: of in2)
    const double* stats2; const float *gamma2, *beta2;       // FX_BN_BN: the batch norm of in2; FX_BWD: its backward sums, and where dgamma / dbeta go
    const void* wt;
    void* out;
    const void* add0;
    double* ostats;
    const void* ey; const double* estats; const float *egamma, *ebeta; double* ered;
    const void* ey2; const double* estats2; double* ered2;
    int nimg, ldw;
    short OA, OB, IH, IW, OH, OW, Cin, Ncol;
    short TH, tpi, WH, WW;                                   // rows of a tile, tiles per image, input window of a tile
    int wdiv, odiv;                                          // 2^16 / WW + 1, 2^16 / OB + 1: quotients of window / tile pixels
    unsigned tdiv;                                           // 2^32 / tpi + 1: quotient of a tile index (0: one tile per image)
    signed char imul, omul, ooh, oow, ntr, nts, dh0, dhs, dw0, dws, r0, rs, s0, ss, S;
    signed char dhmin, dwmin, mode, relu, erelu;
    signed char BN;                                          // output channels of a tile: 16 or 32
    // ordered: the tile is as many pixels as the row lanes of the separate BN-backward reduction take in one trip (512, 256,
    // 128 pixels of 16, 32, 64 channels), and statistics and backward sums are added up in the order of the separate passes,
    // so that a step in bf16 gives the same bits as with separate passes; segs: images of a tile
    signed char ordered, segs;
};
struct FConvGroup {
    int nprob, total_tiles;
    float eps; int pad_;
    int start[kMaxGroup];                                    // first tile of every problem: one cache line, unused entries INT_MAX
    FConvProb p[kMaxGroup];
};
static_assert(sizeof(FConvGroup) <= 4096, "kernel-argument block");
// pixels of a tile with BN output channels: four waves hold at most 4 micro-tiles of 16 x 16 each (ordered tiles of 16 and 32
// channels: 8, in two parts)
constexpr int fconv_max_px(int BN) { return 4096 / BN; }
// k-steps of a tile: 64 bytes of channels of one tap each (bf16 with 16 channels: two taps)
__host__ __device__ inline int fconv_ksteps(int ntaps, int Cin, int esz) { return Cin * esz < 64 ? (ntaps + 1) / 2 : ntaps * (Cin * esz / 64); }
constexpr int kFconvMaxLds = 80 * 1024;                      // two workgroups per compute unit at least
size_t fconv_lds_bytes(const FConvProb& p, int esz);

// A wide bf16 convolution on few pixels (lp_sconv.hip): tiles of TH rows of one image or `segs` whole images (at most 128
// pixels) x 32 output channels, in the summation order of the wide-layer kernel the launch is taken from.
constexpr int kSconvMaxPx = 320;                             // window pixels of a tile
struct SConvProb {
    const void *in, *wt, *add0, *add1;
    void* out;
    int nimg, ldw, wdiv, odiv;
    int win_bytes;                                           // LDS bytes of a window slab of 64 channels
    int row_tile_start, row_tile, col_tiles, col_tile;       // the other kernel's tiles (rot: which workgroup is odd)
    short OA, OB, IH, IW, OH, OW, Cin, Ncol, TH, tpi, segs, WH, WW;
    short slab, gs;                                          // channels of its slabs (64 or 32); slabs of 64 per group here
    signed char imul, omul, ooh, oow, ntr, nts, dh0, dhs, dw0, dws, r0, rs, s0, ss, S, dhmin, dwmin, rot;
};
struct SConvGroup {
    int nprob, total_tiles;
    int pad_[2];
    int start[kMaxGroup];
    SConvProb p[kMaxGroup];
};
static_assert(sizeof(SConvGroup) <= 4096, "kernel-argument block");
// per-channel sums of stored tensors in the order of the wide-layer kernels' epilogue (tiles of BM rows)
struct TileStatsProb { const void* y; double* stats; int M, C, BM, block_start; };
struct TileStatsGroup { int nprob, total_blocks; TileStatsProb p[kMaxGroup]; };

// Weight gradient:  dW[co, (r,s,ci)] (+)= sum_m dY[m, co] * X[n, ho*stride - pad + r, wo*stride - pad + s, ci]
// split over `ksplit` slices of the reduction; partial results are added to dW with fp32 atomics.
struct WgradProb {
    const void* x;
    const void* dy;
    float* dw;
    int M, Cout, Kg, Cin;
    int Ho, Wo, IH, IW, stride, pad, R, S;
    int ksplit, kchunk;
    int tiles_m, tiles_n, tile_start;
    int tile0, ntile;                // wide-layer kernels: the output tiles this entry is about (tiles_m * tiles_n of them in one or two entries)
    unsigned mulW, shW, mulH, shH;   // fast division by IW and IH (lp_wgrad_tile.hip: by Wo and Ho)
    // parameter update in the epilogue (w != NULL): the workgroup that adds the LAST partial sum of an output tile
    // (ticket from cnt[tile], zero before the launch) reads the finished gradient tile back and updates the filter
    void* w;                         // the filter itself, storage type of the activations, layout of dw
    float* vel;                      // momentum buffer (NULL: none)
    float* master;                   // fp32 copy of the filter (NULL: w is read)
    unsigned* cnt;                   // tiles_m * tiles_n tickets
};
struct WgradGroup {
    int nprob, total_tiles;
    float lr, momentum, wd;          // of the update in the epilogue
    int lowp;                        // the filters are bf16
    WgradProb p[kMaxGroup];
};
static_assert(sizeof(WgradGroup) <= 4096, "kernel-argument block");

// Filter gradient of a narrow layer (lp_fwgrad.hip): a workgroup walks over `per` tiles of whole image rows.
struct FWgradProb {
    const void *x, *dy;
    float* dw;
    int ntiles, per, nranges;                                // tiles, tiles of a workgroup, workgroups of a channel block
    int wdiv, odiv, cdiv;                                    // 2^16 / WW + 1, 2^16 / Wo + 1, 2^16 / Cin + 1
    unsigned tdiv;                                           // 2^32 / tpi + 1 (0: one tile per image)
    short Cin, Cout, IH, IW, Ho, Wo, stride, pad, R, TH, tpi, WH, WW;
};
constexpr int kFwMax = 40;                                   // problems of a launch: all layers of a stream lane of most networks
struct FWgradGroup {
    int nprob, total_tiles;
    int pad_[2];
    int start[kFwMax];
    FWgradProb p[kFwMax];
};
static_assert(sizeof(FWgradGroup) <= 4096, "kernel-argument block");
// 16-byte vectors of dY and of the input window a thread holds of a tile; elements of the window of an image-facing layer
__host__ __device__ constexpr int fwgrad_y_vecs(int esz) { return esz == 2 ? 2 : 4; }
__host__ __device__ constexpr int fwgrad_x_vecs(int esz) { return esz == 2 ? 3 : 6; }
constexpr int kFwStemElems = 4;
size_t fwgrad_lds_bytes(const FWgradProb& p, int esz);

// filters [Cout][R][S][Cin] -> [Cin][R][S][Cout]
struct PrepProb {
    const void* src;         // NULL: clear
    void* dst;
    int Cout, RS, Cin;       // filter [Cout][RS][Cin] -> [Cin][RS][Cout]
    int vecs;                // clear: 16-byte vectors; -1: one float at dst and, where there is a src, another there
};
constexpr int kPrepMax = 96;                       // problems of a launch: 3.4 of the 4 KiB of kernel arguments
struct PrepGroup {
    int nprob, total_blocks;
    int start[kPrepMax];                           // first workgroup of a problem; INT_MAX behind the last
    PrepProb p[kPrepMax];
};

// out = act( bn(y) [+ skip] ),  bn(y) = gamma*(y-mean)*invstd + beta from the summed statistics.
// skip_mode 0: none, 1: plain tensor, 2: bn_s(skip) with its own statistics.
// Fused form (the pass that writes a module's output F_k(x_k), inside lp_local_step): with dy != NULL the same pass
// evaluates the local loss and terminal adjoint on the value it stores, as LossProb below describes (xn, lam, dy,
// lam_out, loss), so that F_k(x_k) is not read again.
struct BnApplyProb {
    const void* y; void* out;
    const double* stats; const float* gamma; const float* beta;
    const void* skip; const double* sstats; const float* sgamma; const float* sbeta;
    const void* xn; const void* lam; void* dy; void* lam_out; float* loss; float* r2;
    int M, C, relu, skip_mode;
    int slice, per;       // bn_slice; vectors of a thread, 4 or 8
    int block_start, nblocks;
};
struct BnApplyGroup {
    int nprob, total_blocks; float eps;
    int cmax;             // most channels a workgroup of the group has coefficients of (sizes the arrays in LDS)
    float rho, scale, step;   // fused form: penalty coefficient, loss scale, multiplier step
    BnApplyProb p[kMaxGroup];
};

// Batch-norm backward.  g' = g * [gamma*yhat + beta > 0] when relu is set.
// reduce: red[0..C) += sum g', red[C..2C) += sum g'*yhat.   apply: dy = gamma*invstd*(g' - red0/M - yhat*red1/M),
// and the first workgroup of each problem writes dgamma = red1, dbeta = red0.
struct BnBwdProb {       // add: optional addend of the apply pass with the layout of dy (identity skip of a pre-activation block)
    const void* add;
    const void* g; const void* y; void* dy;
    const double* stats; const float* gamma; const float* beta;
    double* red; float* dgamma; float* dbeta;
    int M, C, relu;
    int slice, per;       // as in BnApplyProb (per: apply pass)
    int parts, lanes, groups;    // reduction: pieces of the rows, their row lanes, and how many of them a workgroup does
    int block_start, nblocks;
};
struct BnBwdGroup {
    int nprob, total_blocks; float eps;
    int cmax;             // as above
    int threads;          // of a workgroup of the reduction
    BnBwdProb p[kMaxGroup];
};

// gm = g * [out > 0]: the gradient through a ReLU behind a residual sum, from the stored block output
struct MaskProb { const void* g; const void* out; void* gm; size_t numel; int block_start, nblocks; };
struct MaskGroup { int nprob, total_blocks; MaskProb p[kMaxGroup]; };

// r = y - x_next;  dy = scale*(rho*r + lam);  loss += scale*(rho/2*sum r^2 + sum lam*r)
struct LossProb {
    const void* y; const void* xn; const void* lam; void* dy; float* loss;
    float* r2;               // != NULL: += sum r^2 (the constraint violation |F_k(x_k) - x_{k+1}|^2 of the interface)
    void* lam_out;           // != NULL: lam + step*(y - x_next) is written there (may be lam itself) after dy took the old lam
    size_t numel; int block_start, nblocks;
};
struct LossGroup { int nprob, total_blocks; float rho, scale, step; LossProb p[kMaxGroup]; };

// lam += step*(y - x_next)
struct MultProb { void* lam; const void* y; const void* xn; size_t numel; int block_start, nblocks; };
struct MultGroup { int nprob, total_blocks; float step; MultProb p[kMaxGroup]; };
// parameter update of one tensor: g' = g + wd*W; v = mu*v + g' (if v); W -= lr*(v or g'); master (fp32 copy) optional
struct SgdProb { void* p; const float* g; float* v; float* master; size_t numel; int lowp; int block_start, nblocks; };
struct SgdGroup { int nprob, total_blocks; float lr, momentum, wd; SgdProb p[kMaxGroup]; };
// correction of an auxiliary variable: x <- x - eta*(scale*(rho*(x - yprev) - lam) + dx), lam may be NULL
struct AuxVarProb {      // gout != NULL: the gradient scale*(rho*(x - yprev) - lam) + dx is written there and x is left as it is
    void* x; const void* yprev; const void* dx; const void* lam; void* gout; size_t numel; int block_start, nblocks;
};
struct AuxVarGroup { int nprob, total_blocks; float rho, scale, eta; AuxVarProb p[kMaxGroup]; };

struct PoolProb {        // max pooling R x R, stride, pad on NHWC
    const void* x; void* y; uint8_t* arg; const void* dy; void* dx;
    int N, H, W, C, Ho, Wo, R, stride, pad;
};

struct HeadProb {        // global average pool + linear
    const void* feat; float* pooled; const float* w; const float* b; float* logits;
    const float* dlogits; float* dw; float* db; void* dfeat;
    const int32_t* labels; float* loss;      // forward with the cross-entropy behind it (head_with_loss): dlogits is written
    int N, HW, C, classes;
};
// Is the head of a step one launch, a workgroup per sample (pooling, linear layer, cross-entropy)?  Where a sample's features fit the LDS
// and every sample can afford to read all weights: three dependent launches of 2 to 6 us otherwise, each of them 4 us of the
// host's time (with the losses cleared in the step's first launch, not one of their own, and the last module's last
// pass in the launch of the others': tiny 81 -> 62 us, ResNet-20 of 3 samples in bf16 192 -> 173, of 16 229 -> 209, 2 in fp32 232 -> 211).
inline bool head_with_loss(const HeadProb& p, int esz) { return (size_t)p.HW * p.C * esz <= 32 * 1024 && (size_t)p.C * p.classes <= 16384; }

// Image-facing convolutions (lp_iconv.hip): bytes of the rows of the image that BM consecutive output pixels read at most, in whole
// wave-loads; 0: not a layer of that kernel.  Up to 24 KB, so that four workgroups and their result slices fit a CU.  The image
// has to end at a whole 4 bytes (the copy's unit; with an odd number of bf16 elements its last one would be lost).
inline int iconv_window(const ConvProb& p, int BM, int esz) {
    if (p.Kg > 32 || p.ntr * p.nts * p.Cin != p.Kg || p.ldw != p.Kg || (p.Ncol != 16 && p.Ncol != 32 && p.Ncol != 64)) return 0;
    if (p.add0 || p.add1 || p.omul != 1 || p.ooh || p.oow || p.dhs != 1 || p.dws != 1 || p.r0 || p.s0 || p.rs != 1 || p.ss != 1) return 0;
    if (p.OH != p.OA || p.OW != p.OB || p.dh0 > 0 || p.dw0 > 0) return 0;
    if (p.IH > 8192 || p.IW > 8192 || p.dh0 < -64 || p.dw0 < -64) return 0;      // 16-bit positions
    const int64_t nimg = p.M / (p.OA * p.OB), elems = nimg * p.IH * p.IW * p.Cin;
    if (elems * esz % 4 || elems > 0x40000000) return 0;
    const int64_t rows = (BM + p.OB - 2) / p.OB + 1;                       // output rows that the pixels lie in
    const int64_t cross = std::min(nimg - 1, (rows - 2 + p.OA) / p.OA);    // ends of images among them
    const int64_t in = std::min(nimg * p.IH, (rows - 1) * p.imul + p.ntr + cross * std::max(0, p.IH - p.OA * p.imul));
    const int64_t bytes = (in * p.IW * p.Cin * esz + 16 + 1023) / 1024 * 1024;
    return bytes <= 24 * 1024 ? (int)bytes + 16 : 0;                       // and a vector of zeros
}

// ---- launchers (host side; return hipError_t of the launch) ----------------------------------------
// tile configuration ids of the implicit-GEMM kernels
enum ConvCfg { CFG_N16 = 0, CFG_N32, CFG_N64, CFG_N128, CFG_N160,
               CFG_N64S,                               // 64 x 64 tiles with twice the k-tile: 33..64 output channels, few pixels (forward / data-gradient only)
               CFG_COUNT,
               FAST_256x320 = 8, FAST_512x160 = 9,     // bf16 wide-layer kernel (lp_conv_fast.hip)
               FAST_128x320 = 10, FAST_128x160 = 11,   // ... its four- and two-wave variants, chosen per launch
               FAST64_256x320 = 12, FAST64_128x320 = 13, FAST64_128x160 = 14,   // ... with k-tiles of 64 channels
               FAST_256x160 = 15, FAST64_256x160 = 16,  // four-wave variants of the 160-wide family
               // (13, 14 and 16 are launched by nets of separate passes only: elsewhere a layer of whole 64-channel k-tiles that would have
               // them takes a tile below or the small ones; they say what bits, and how many rows a partial statistic, those have)
               // ... with waves of 32 pixels: a ring of two k-tiles (two or three workgroups per CU), of three or four (R3, R4)
               MID_128x128 = 17, MID_128x128_R3 = 18, MID_128x32_R4 = 19, MID_64x128_R3 = 20, MID_64x64_R4 = 25, MID_128x64 = 26, MID_128x64_R3 = 27,
               MID_256x128_R3 = 28, MID_256x64_R3 = 29, MID_256x32_R4 = 30,
               WIN64_512x160 = 21, WIN64_256x320 = 23,  // bf16 3x3 stride-1 kernel with the input window in LDS (lp_conv_win.hip)
               SMALL_128x32 = 24,                      // bf16 wide layers on few pixels, recorded only (lp_sconv.hip)
               CONV_IMAGE = 31,                        // image-facing layers, recorded only (lp_iconv.hip)
               WGRAD_FAST = 8,                         // bf16 wide-layer filter-gradient kernel (lp_wgrad_fast.hip)
               WGRAD_TILE = 9,                         // ... of the other wide layers, recorded only (lp_wgrad_tile.hip)
               WGRAD_STEM = 10 };                      // ... of an image-facing layer, recorded only (lp_wgrad_stem.hip)
struct CfgInfo { int BM, BN, BK; };
CfgInfo conv_cfg_info(int cfg, int dtype);
CfgInfo wgrad_cfg_info(int cfg, int dtype);
CfgInfo conv_fast_cfg_info(int cfg);
CfgInfo conv_win_cfg_info(int cfg);
// window slabs (1 KiB wave-loads) a wave of the window kernel can hold addresses for
constexpr int conv_win_max_slabs(int BM, int NW) { return BM == 512 ? 10 : 7; }

// dynamic LDS of up to `bytes` for these kernels, on the current device
inline hipError_t raise_lds_limit(OncePerDevice& once, std::initializer_list<const void*> kernels, int bytes) {
    return once.run([](int* dev) { return hipGetDevice(dev); }, [&] {
        for (const void* k : kernels)
            if (const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); e != hipSuccess) return e;
        return hipSuccess;
    });
}
hipError_t launch_conv(const ConvGroup& g, int dtype, int cfg, bool vec, hipStream_t s);
hipError_t launch_conv_fast(const ConvGroup& g, int cfg, hipStream_t s);
hipError_t launch_iconv(const ConvGroup& g, int dtype, int lds_bytes, hipStream_t s);
hipError_t launch_conv_win(const ConvGroup& g, int cfg, hipStream_t s);
hipError_t launch_sconv(const SConvGroup& g, size_t lds, hipStream_t s);
hipError_t launch_tile_stats(const TileStatsGroup& g, hipStream_t s);
hipError_t launch_fconv(const FConvGroup& g, int dtype, size_t lds, hipStream_t s);
hipError_t launch_fwgrad(const FWgradGroup& g, int dtype, size_t lds, hipStream_t s);
hipError_t launch_wgrad_fast(const WgradGroup& g, hipStream_t s);
int wgrad_tile_rows(int Cout);                             // output channels of a tile of the kernel below: 64 or 128, by 128 columns
hipError_t launch_wgrad_tile(const WgradGroup& g, int rows, hipStream_t s);
bool wgrad_stem_ok(const WgradProb& p);                    // the layers of the image-facing kernel; the image aligned to four bytes as well
hipError_t launch_wgrad_stem(const WgradGroup& g, hipStream_t s);     // kchunk: output rows of a workgroup; tile_start, total_tiles
void fastdiv_make(unsigned d, unsigned* mul, unsigned* shift);
hipError_t launch_wgrad(const WgradGroup& g, int dtype, int cfg, bool vec, hipStream_t s);
hipError_t launch_prep(const PrepGroup& g, int dtype, hipStream_t s);
hipError_t launch_bn_apply(const BnApplyGroup& g, int dtype, bool fused_loss, hipStream_t s);
hipError_t launch_bn_bwd_reduce(const BnBwdGroup& g, int dtype, hipStream_t s);
hipError_t launch_bn_bwd_apply(const BnBwdGroup& g, int dtype, hipStream_t s);
hipError_t launch_relu_mask(const MaskGroup& g, int dtype, hipStream_t s);
hipError_t launch_loss(const LossGroup& g, int dtype, hipStream_t s);
hipError_t launch_mult(const MultGroup& g, int dtype, hipStream_t s);
hipError_t launch_auxvar(const AuxVarGroup& g, int dtype, hipStream_t s);
hipError_t launch_sgd(const SgdGroup& g, hipStream_t s);
// per-channel sum and sum of squares of a stored tensor [M, C] (fields y, red, M, C of BnBwdProb), added to red[2C]
hipError_t launch_bn_stats(const BnBwdGroup& g, int dtype, hipStream_t s);
constexpr int kSgdElemsPerBlock = 4096;
hipError_t launch_bn_bwd_small(const BnBwdGroup& g, hipStream_t s);
hipError_t launch_maxpool_fwd(const PoolProb& p, int dtype, hipStream_t s);
hipError_t launch_maxpool_bwd(const PoolProb& p, int dtype, hipStream_t s);
// does the linear layer of the head run in its tiled kernels (forward, filter gradient)?
bool fc_fwd_tiled(const HeadProb& p);
bool fc_bwd_w_tiled(const HeadProb& p);
hipError_t launch_head_fwd(const HeadProb& p, int dtype, hipStream_t s);
hipError_t launch_head_bwd(const HeadProb& p, int dtype, hipStream_t s);
hipError_t launch_ce(const float* logits, const int32_t* labels, float* loss, float* dlogits,
                     int N, int classes, hipStream_t s);
// v[i] = 0 where bit i of mask is set (i < n), v2 alike with its own mask and number (v2 may be NULL)
hipError_t launch_zero_selected(float* v, uint32_t mask, int n, float* v2, uint32_t mask2, int n2, hipStream_t s);
hipError_t launch_im2col_offsets(const ConvProb& p, const int64_t* m, const int64_t* q, int64_t* out, int count, hipStream_t s);
hipError_t launch_conv_offsets(const ConvProb& p, int kernel, int BM, int bk, int nw, const int64_t* m, const int64_t* q,
                               const int64_t* col, int64_t* in_off, int64_t* w_off, int64_t* out_off, int count, hipStream_t s);

hipError_t launch_mfma_peak(int mode, int blocks, int iters, unsigned long long* clk, float* sink, hipStream_t s);

constexpr int kElemBlock = 256;          // threads per workgroup of the elementwise kernels
// Per-channel sums (batch statistics, BN backward sums) are accumulated with fp64 atomics by every workgroup that holds
// a piece of the tensor.  Atomics on ONE address are performed one after another at the memory side (about 25 ns each
// on this device: 512 workgroups adding to the same 32 addresses cost 13 us), so a sum is kept as several partial sums
// ("stripes", layout [kStatStripes][2][C]); workgroup b adds to stripe b % stat_stripes(C) and readers add the stripes
// up in a fixed order.  Readers pay for every stripe in their prologue (C x stripes loads per workgroup), so the
// number of stripes in use falls with the channel count: narrow layers have many writers per address and cheap readers,
// wide layers the opposite (measured: ResNet-56 step 1.36 -> 1.27 ms with 4-8 stripes; 2048-channel layers lose with 4).
constexpr int kStatStripes = 8;
__host__ __device__ inline int stat_stripes(int C) { return C <= 64 ? 8 : (C <= 320 ? 4 : 1); }
__host__ __device__ inline size_t stat_bytes(int C) { return sizeof(double) * 2 * (size_t)C * kStatStripes; }
constexpr int kBnReduceBlock = 512;      // threads per workgroup of the BN backward reduction (measured: 256 -7 %, 1024 -20 %)
// ... and 256 for launches whose widest tensor has at most 64 channels: with 512 half of the 256 workgroups of a 32 x 32 x 16
// tensor have no trip at all and the others' final sum over the row lanes is twice as long.  The row lanes of whole rows
// follow from it, and the order of the sums from those.
inline int bn_reduce_threads(int cmax) { return cmax <= 64 ? 256 : kBnReduceBlock; }
// Channels of a workgroup of the batch-norm passes (apply, backward), 0: all of them.  A workgroup computes the coefficients of its channels
// from the sums first, 16 bytes a channel, stripe and sum: for 320 to 2048 channels that is as much as its 32 KB of a tensor.
// A small tensor also has few rows a workgroup can share out: 294 rows of 2048 channels were 5 workgroups of the backward reduction
// and are 80.  Slices are whole 128-byte lines of bf16.  ResNet-50 step of 6 samples 1529 -> 1432 us, of 64 5724 -> 5695, WRN-28-10
// in pre-activation order 1942 -> 1892; 160 channels (WRN-28-10's first stage) have no such slice and keep whole rows.
inline int bn_slice(int C) { return C > 128 && C % 128 == 0 ? 128 : C > 64 && C % 64 == 0 ? 64 : 0; }
// How the backward reduction cuts M rows of C channels (epv to a vector): row lanes of a part, and parts, of which each has at least 64
// rows and (one trip being four rows per row lane) no more are made than there are trips.  The order of the sums.
inline void bn_reduce_cut(int M, int C, int epv, int threads, int& lanes, int& parts) {
    lanes = threads / (C / epv) > 1 ? threads / (C / epv) : 1;
    const int most = (M + 63) / 64 < 256 ? (M + 63) / 64 : 256, trips = (M + 4 * lanes - 1) / (4 * lanes);
    parts = most < trips ? most : trips;
    if (parts < 1) parts = 1;
}
// Reduction and apply pass in one launch (bn_bwd_small_kernel): a workgroup for all rows of 64 channels.  It is done in 6 us and a line of
// 128 bytes every 4 to 5 clocks, five lines a row: 49 rows 9 us (timed by itself, with its launch), 196 12, 784 18, 1176 25; the two launches 15 to
// 18 for any of them.  Whole steps, two launches / one: ResNet-50 of 1 / 3 samples 1300 / 1200 and 1370 / 1253 us, WRN-28-10 of 1 / 4 samples
// 848 / 780 and 832 / 800, in pre-activation order of 5 857 / 820; up to 1300 rows ResNet-50 of 6 1398 / 1490, up to 2048 of 9 1568 / 1800.
// Between 449 and 600 rows a step is as long either way, but not the AuxNets' backward pass, which has nothing beside it: iterations of
// WRN-28-10 of 8 / 9 samples (512 / 576 rows) 1517 / 1536 and 1695 / 1713, of ResNet-50 of 3 (588) 1568 / 1581.
constexpr int kBnSmallChannels = 64, kBnSmallThreads = 512;
inline bool bn_bwd_small(int M, int C, int esz) { return esz == 2 && C > 64 && C % kBnSmallChannels == 0 && M <= 448; }
constexpr int kElemVecsPerBlock = 2048;  // 16-byte vectors handled by one workgroup

}  // namespace lp
