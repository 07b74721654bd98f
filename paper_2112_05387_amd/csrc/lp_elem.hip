// Grouped HBM-bound kernels of the local step: batch-norm apply (+ReLU, +skip), batch-norm backward
// (reduce / apply), the local penalty / augmented-Lagrangian loss and terminal adjoint, the multiplier
// update, the classification head, max pooling and buffer clears.  NHWC, 16-byte accesses with the
// channel index fastest, fp32 arithmetic, wavefront/LDS reductions, one atomic per channel per workgroup.
#include <algorithm>

#include "lp_kernels.h"
#include "lp_mma.h"
#include "lp_vec.h"

namespace lp {

namespace {

template <typename G> __device__ __forceinline__ int find_problem(const G& g, int bid) {
    int pi = 0;
    for (int i = 1; i < g.nprob; ++i)
        if (bid >= g.p[i].block_start) pi = i;
    return pi;
}

// Which 16-byte vectors of an [M][C] tensor a thread of a batch-norm apply pass works on: `per` of them, v, v + vstep, ...
// (those below M * C / EPV), and where their channels lie in the workgroup's coefficients (c, c + cstep mod cmod, ...).
// Without slices a workgroup has consecutive vectors and the coefficients of all channels; with slices of `slice` channels
// (bn_slice) it has whole rows of one slice, and every vector of a thread the same channels.
struct BnSpan { size_t v; size_t vstep; unsigned c, cstep, cmod; int ch0, nch; };
template <int EPV> __device__ __forceinline__ BnSpan bn_span(int block, int C, int slice, int per) {
    BnSpan q;
    const unsigned cv = (unsigned)C / EPV;
    if (!slice) {
        q.v = (size_t)block * (per * kElemBlock) + threadIdx.x; q.vstep = kElemBlock;
        q.cmod = cv; q.cstep = (unsigned)kElemBlock % cv; q.c = (unsigned)(q.v % cv);
        q.ch0 = 0; q.nch = C;
    } else {
        const unsigned ns = (unsigned)C / (unsigned)slice, sv = (unsigned)slice / EPV, rl = kElemBlock / sv;
        const unsigned rb = (unsigned)block / ns, sl = (unsigned)block - rb * ns, row = rb * (rl * per) + threadIdx.x / sv;
        q.cmod = sv; q.cstep = 0; q.c = threadIdx.x % sv;
        q.v = (size_t)row * cv + sl * sv + q.c; q.vstep = (size_t)rl * cv;
        q.ch0 = (int)sl * slice; q.nch = slice;
    }
    return q;
}

// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ float block_sum(float v, float* s_tmp);

// FUSE: the pass also evaluates the local loss and terminal adjoint of the interface tensor it writes (exactly the
// arithmetic of loss_kernel, on the value as stored, vector by vector in the same order), of the problems that have one
template <typename T, bool FUSE>
__global__ __launch_bounds__(kElemBlock) void bn_apply_kernel(const BnApplyGroup g) {
    constexpr int EPV = Vec<T>::N;
    // per-channel coefficients: 4 arrays of g.cmax floats (sized by the launch: the LDS footprint limits occupancy)
    extern __shared__ __attribute__((aligned(16))) float s_coef[];
    const int cm = 4 * (g.cmax >> 2);      // written as a multiple of 4 so that the arrays are visibly 16-byte aligned
    float* s_sc = s_coef;
    float* s_sh = s_coef + cm;
    float* s_ssc = s_coef + 2 * cm;
    float* s_ssh = s_coef + 3 * cm;
    const BnApplyProb& P = g.p[find_problem(g, blockIdx.x)];
    const int C = P.C, M = P.M;
    const BnSpan span = bn_span<EPV>(blockIdx.x - P.block_start, C, P.slice, P.per);
    for (int i = threadIdx.x; i < span.nch; i += kElemBlock) {
        const int c = span.ch0 + i;
        float sc, sh, mu, is;
        bn_coeffs(P.stats, P.gamma, P.beta, c, C, M, g.eps, sc, sh, mu, is);
        s_sc[i] = sc; s_sh[i] = sh;
        if (P.skip_mode == 2) {
            bn_coeffs(P.sstats, P.sgamma, P.sbeta, c, C, M, g.eps, sc, sh, mu, is);
            s_ssc[i] = sc; s_ssh[i] = sh;
        }
    }
    __syncthreads();
    const T* __restrict__ y = reinterpret_cast<const T*>(P.y);
    const T* __restrict__ skip = reinterpret_cast<const T*>(P.skip);
    T* __restrict__ out = reinterpret_cast<T*>(P.out);
    const size_t nvec = (size_t)M * C / EPV;
    // four vectors per trip, loads first: up to eight independent 16-byte loads in flight per thread
    constexpr int U = 4;
    unsigned cidx = span.c;
    const T* __restrict__ xn = reinterpret_cast<const T*>(P.xn);
    const T* lam = reinterpret_cast<const T*>(P.lam);
    T* lam_out = reinterpret_cast<T*>(P.lam_out);          // may alias lam: every vector is read before it is written
    T* __restrict__ dyp = reinterpret_cast<T*>(P.dy);
    float lacc = 0.f, racc = 0.f;
    for (int i0 = 0; i0 < P.per; i0 += U) {
        // Unconditional loads (a vector beyond the end re-reads the last one and is dropped): behind a per-lane branch
        // the compiler waits for each pair of loads before it issues the next.
        u32x4 fraw[U], skraw[U], xnraw[FUSE ? U : 1], lmraw[FUSE ? U : 1];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t v = span.v + (i0 + u) * span.vstep;
            ok[u] = v < nvec;
            const size_t vc = ok[u] ? v : nvec - 1;
            fraw[u] = Vec<T>::load_raw(y + vc * EPV);
            if (P.skip_mode) skraw[u] = Vec<T>::load_raw(skip + vc * EPV);
            if constexpr (FUSE) {
                xnraw[u] = Vec<T>::load_raw(xn + vc * EPV);
                if (lam) lmraw[u] = Vec<T>::load_raw(lam + vc * EPV);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c0 = (int)cidx * EPV;
            cidx += span.cstep;
            if (cidx >= span.cmod) cidx -= span.cmod;
            if (!ok[u]) continue;
            const size_t v = span.v + (i0 + u) * span.vstep;
            float f[1][EPV], sk[1][EPV], o[EPV];
            Vec<T>::unpack(fraw[u], f[0]);
            if (P.skip_mode) Vec<T>::unpack(skraw[u], sk[0]);
#pragma unroll
            for (int e = 0; e < EPV; ++e) o[e] = fmaf(s_sc[c0 + e], f[0][e], s_sh[c0 + e]);
            if (P.skip_mode == 2) {
#pragma unroll
                for (int e = 0; e < EPV; ++e) o[e] += fmaf(s_ssc[c0 + e], sk[0][e], s_ssh[c0 + e]);
            } else if (P.skip_mode == 1) {
#pragma unroll
                for (int e = 0; e < EPV; ++e) o[e] += sk[0][e];
            }
            if (P.relu) {
#pragma unroll
                for (int e = 0; e < EPV; ++e) o[e] = fmaxf(o[e], 0.f);
            }
            Vec<T>::store(out + v * EPV, o);
            if constexpr (FUSE) {
                if (!dyp) continue;                         // a problem without a loss
                if constexpr (sizeof(T) == 2) {             // the loss is defined on F_k(x_k) as stored
#pragma unroll
                    for (int e = 0; e < EPV; e += 2) {
                        const unsigned pk = pack_bf16x2(o[e], o[e + 1]);
                        o[e] = __uint_as_float(pk << 16); o[e + 1] = __uint_as_float(pk & 0xffff0000u);
                    }
                }
                float b[EPV], l[EPV], d[EPV];
                Vec<T>::unpack(xnraw[u], b);
                if (lam) Vec<T>::unpack(lmraw[u], l);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    const float r = o[e] - b[e];
                    const float lm = lam ? l[e] : 0.f;
                    lacc += 0.5f * g.rho * r * r + lm * r;
                    racc += r * r;
                    d[e] = g.scale * (g.rho * r + lm);
                }
                Vec<T>::store(dyp + v * EPV, d);
                if (lam && lam_out) {
#pragma unroll
                    for (int e = 0; e < EPV; ++e) l[e] = fmaf(g.step, o[e] - b[e], l[e]);
                    Vec<T>::store(lam_out + v * EPV, l);
                }
            }
        }
    }
    if constexpr (FUSE) {
        if (!dyp) return;
        __shared__ float s_tmp[kElemBlock / 64];
        const float tot = block_sum(lacc, s_tmp);
        if (threadIdx.x == 0 && tot != 0.f) atomicAdd(P.loss, g.scale * tot);
        if (P.r2) {
            const float rt = block_sum(racc, s_tmp);
            if (threadIdx.x == 0 && rt != 0.f) atomicAdd(P.r2, rt);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// red[c] += sum g', red[C+c] += sum g'*yhat over this workgroup's rows.
// S / EPV <= NT channel vectors (S <= 2048): thread t owns channel vector t % cv and is row lane t / cv.  A trip is
// four rows per row lane, i.e. eight independent 16-byte loads per thread.  The rows are cut into `parts`, whose trips are
// interleaved (part b takes trips b, b + parts, ...), so that at any time the parts together read one contiguous, moving
// window of the two tensors instead of as many distant streams.  The first trip is requested before the coefficient prologue
// (it does not depend on it) and every further trip before the previous one is consumed.
// The order of the fp32 sums is that of whole rows, with slices or without: a part has the row lanes that a workgroup has of whole
// rows, they are added up in fp32 one after the other, and the parts meet in fp64.  A workgroup of whole rows is one part; one of
// a slice, whose rows are shorter, holds `groups` of them.  With the row lanes of the slice instead, sums as exact but not
// the same, the bf16 adjoints of wide networks moved by 2e-3 to 8e-3 of their norm, single roundings of the auxiliary
// variables with them, and the gradient of an AuxNet, which is distilled from just those, by 0.02 to 0.10.
// Slices run in workgroups of 256 threads, of which three share a compute unit (155 registers), whole rows in 512: the sliced
// ones in 512 as well, or with three or four trips under way, or one trip and four waves a SIMD, are each the slower choice
// (ResNet-50 step of 6 / 64 samples 1434 / 5576 us; 1450 / 5597, 1457 / 5663, 1494 / 6048; without slices 1448 / 5531).
template <typename T, int NT>
__global__ __launch_bounds__(NT) void bn_bwd_reduce_kernel(const BnBwdGroup g) {
    constexpr int EPV = Vec<T>::N;
    __shared__ float s_red[NT * EPV * 2];
    // per-channel coefficients, computed once per workgroup (4 arrays of g.cmax floats, sized by the launch)
    extern __shared__ __attribute__((aligned(16))) float s_coef[];
    const int cm = 4 * (g.cmax >> 2);
    float* s_sc = s_coef;
    float* s_sh = s_coef + cm;
    float* s_mu = s_coef + 2 * cm;
    float* s_is = s_coef + 3 * cm;
    const BnBwdProb& P = g.p[find_problem(g, blockIdx.x)];
    // S channels (bn_slice, or all of them) from ch0 on; the workgroup's parts are rb * groups, rb * groups + 1, ...
    const int C = P.C, M = P.M, S = P.slice ? P.slice : C, ns = C / S, cv = S / EPV;
    const int b = blockIdx.x - P.block_start, rb = b / ns, ch0 = (b - rb * ns) * S;
    const T* __restrict__ gp = reinterpret_cast<const T*>(P.g);
    const T* __restrict__ y = reinterpret_cast<const T*>(P.y);
    const int rl = P.lanes;                      // row lanes of a part
    const int tcv = threadIdx.x % cv, lane_row = threadIdx.x / cv;
    const int group = P.groups > 1 ? lane_row / rl : lane_row >= rl, trl = lane_row - group * rl;
    const int part = rb * P.groups + group;
    const bool active = group < P.groups && part < P.parts;
    const int c0 = tcv * EPV;                    // in the slice
    const int rows_trip = 4 * rl, stride = P.parts * rows_trip;
    // a trip as loaded (32 registers); rows past the end read the last row and count as zero when consumed
    auto request = [&](u32x4 (&graw)[4], u32x4 (&yraw)[4], int r0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = min(r0 + trl + u * rl, M - 1);
            graw[u] = Vec<T>::load_raw(gp + (size_t)r * C + ch0 + c0);
            yraw[u] = Vec<T>::load_raw(y + (size_t)r * C + ch0 + c0);
        }
    };
    u32x4 ga[4], ya[4], gb[4], yb[4];
    int r0 = part * rows_trip;
    if (active && r0 < M) request(ga, ya, r0);
    for (int c = threadIdx.x; c < S; c += NT) {
        float sc, sh, mu, is;
        bn_coeffs(P.stats, P.gamma, P.beta, ch0 + c, C, M, g.eps, sc, sh, mu, is);
        s_sc[c] = sc; s_sh[c] = sh; s_mu[c] = mu; s_is[c] = is;
    }
    __syncthreads();
    float a1[EPV], a2[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e) { a1[e] = 0.f; a2[e] = 0.f; }
    if (active) {
        float sc[EPV], sh[EPV], mu[EPV], is[EPV];
#pragma unroll
        for (int e = 0; e < EPV; ++e) { sc[e] = s_sc[c0 + e]; sh[e] = s_sh[c0 + e]; mu[e] = s_mu[c0 + e]; is[e] = s_is[c0 + e]; }
        auto consume = [&](const u32x4 (&graw)[4], const u32x4 (&yraw)[4], int rbase) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float gv[EPV], yv[EPV];
                Vec<T>::unpack(graw[u], gv);
                Vec<T>::unpack(yraw[u], yv);
                const bool in = rbase + trl + u * rl < M;
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    float gg = in ? gv[e] : 0.f;
                    if (P.relu && !(fmaf(sc[e], yv[e], sh[e]) > 0.f)) gg = 0.f;
                    a1[e] += gg;
                    a2[e] += gg * ((yv[e] - mu[e]) * is[e]);
                }
            }
        };
        while (r0 < M) {
            int rn = r0 + stride;
            if (rn < M) request(gb, yb, rn);
            __builtin_amdgcn_sched_barrier(0);
            consume(ga, ya, r0);
            if (rn >= M) break;
            r0 = rn; rn = r0 + stride;
            if (rn < M) request(ga, ya, rn);
            __builtin_amdgcn_sched_barrier(0);
            consume(gb, yb, r0);
            r0 = rn;
        }
    }
    if (active) {
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            s_red[((lane_row * cv + tcv) * EPV + e) * 2] = a1[e];
            s_red[((lane_row * cv + tcv) * EPV + e) * 2 + 1] = a2[e];
        }
    }
    __syncthreads();
    const int here = min(P.groups, P.parts - rb * P.groups);     // parts of this workgroup
    for (int i = threadIdx.x; i < cv * EPV; i += NT) {
        double s1 = 0.0, s2 = 0.0;
        for (int q = 0; q < here; ++q) {
            const float* const p = s_red + (q * rl * cv * EPV + i) * 2;
            float f1 = 0.f, f2 = 0.f;
#pragma unroll 8
            for (int l = 0; l < rl; ++l) { f1 += p[l * cv * EPV * 2]; f2 += p[l * cv * EPV * 2 + 1]; }
            s1 += f1; s2 += f2;
        }
        double* red = P.red + (size_t)(rb % stat_stripes(C)) * 2 * C + ch0;
        atomicAdd(&red[i], s1);
        atomicAdd(&red[C + i], s2);
    }
}

// red[c] += sum y, red[C+c] += sum y^2 over this workgroup's rows (batch statistics of a tensor no convolution
// of this module produced: a module input in the pre-activation order)
template <typename T>
__global__ __launch_bounds__(kElemBlock) void bn_stats_kernel(const BnBwdGroup g) {
    constexpr int EPV = Vec<T>::N;
    __shared__ float s_red[kElemBlock * EPV * 2];
    const BnBwdProb& P = g.p[find_problem(g, blockIdx.x)];
    const int C = P.C, M = P.M, cv = C / EPV;
    const int b = blockIdx.x - P.block_start;
    const int rows_pb = (M + P.nblocks - 1) / P.nblocks;
    const int row0 = b * rows_pb, row1 = min(M, row0 + rows_pb);
    const T* __restrict__ y = reinterpret_cast<const T*>(P.y);
    for (int cbase = 0; cbase < cv; cbase += kElemBlock) {
        const int ncv = min(cv - cbase, kElemBlock);
        const int rl = kElemBlock / ncv;
        const int tcv = threadIdx.x % ncv, trl = threadIdx.x / ncv;
        float a1[EPV], a2[EPV];
#pragma unroll
        for (int e = 0; e < EPV; ++e) { a1[e] = 0.f; a2[e] = 0.f; }
        if (trl < rl) {
            const int c0 = (cbase + tcv) * EPV;
            int r = row0 + trl;
            for (; r + 3 * rl < row1; r += 4 * rl) {
                float yv[4][EPV];
#pragma unroll
                for (int u = 0; u < 4; ++u) Vec<T>::load(y + (size_t)(r + u * rl) * C + c0, yv[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int e = 0; e < EPV; ++e) { a1[e] += yv[u][e]; a2[e] += yv[u][e] * yv[u][e]; }
            }
            for (; r < row1; r += rl) {
                float yv[EPV];
                Vec<T>::load(y + (size_t)r * C + c0, yv);
#pragma unroll
                for (int e = 0; e < EPV; ++e) { a1[e] += yv[e]; a2[e] += yv[e] * yv[e]; }
            }
        }
        __syncthreads();
        if (trl < rl) {
#pragma unroll
            for (int e = 0; e < EPV; ++e) {
                s_red[((trl * ncv + tcv) * EPV + e) * 2] = a1[e];
                s_red[((trl * ncv + tcv) * EPV + e) * 2 + 1] = a2[e];
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < ncv * EPV; i += kElemBlock) {
            float s1 = 0.f, s2 = 0.f;
            for (int l = 0; l < rl; ++l) { s1 += s_red[((l * ncv * EPV) + i) * 2]; s2 += s_red[((l * ncv * EPV) + i) * 2 + 1]; }
            const int c = cbase * EPV + i;
            double* red = P.red + (size_t)(blockIdx.x % stat_stripes(C)) * 2 * C;
            atomicAdd(&red[c], (double)s1);
            atomicAdd(&red[C + c], (double)s2);
        }
    }
}

// dy = gamma*invstd*(g' - red0/M - yhat*red1/M)
template <typename T>
__global__ __launch_bounds__(kElemBlock) void bn_bwd_apply_kernel(const BnBwdGroup g) {
    constexpr int EPV = Vec<T>::N;
    // per-channel coefficients: 5 arrays of g.cmax floats (sized by the launch: the LDS footprint limits occupancy)
    extern __shared__ __attribute__((aligned(16))) float s_coef[];
    const int cm = 4 * (g.cmax >> 2);      // written as a multiple of 4 so that the arrays are visibly 16-byte aligned
    float* s_sc = s_coef;
    float* s_sh = s_coef + cm;
    float* s_k1 = s_coef + 2 * cm;
    float* s_k2 = s_coef + 3 * cm;
    float* s_k3 = s_coef + 4 * cm;
    const BnBwdProb& P = g.p[find_problem(g, blockIdx.x)];
    const int C = P.C, M = P.M;
    const BnSpan span = bn_span<EPV>(blockIdx.x - P.block_start, C, P.slice, P.per);
    const bool first = (int)blockIdx.x - P.block_start < (P.slice ? C / P.slice : 1);      // the first rows (of every slice)
    for (int i = threadIdx.x; i < span.nch; i += kElemBlock) {
        const int c = span.ch0 + i;
        float sc, sh, mu, is;
        bn_coeffs(P.stats, P.gamma, P.beta, c, C, M, g.eps, sc, sh, mu, is);
        const double inv_m = 1.0 / (double)M;
        double rs0, rs1;
        stripe_sums(P.red, c, C, rs0, rs1);
        const float r0 = (float)(rs0 * inv_m), r1 = (float)(rs1 * inv_m);
        const float k1 = P.gamma[c] * is;
        const float k2 = k1 * is * r1;
        s_sc[i] = sc; s_sh[i] = sh;
        s_k1[i] = k1; s_k2[i] = k2; s_k3[i] = k2 * mu - k1 * r0;
        if (first) {
            P.dgamma[c] = (float)rs1;
            P.dbeta[c] = (float)rs0;
        }
    }
    __syncthreads();
    const T* __restrict__ gp = reinterpret_cast<const T*>(P.g);
    const T* __restrict__ y = reinterpret_cast<const T*>(P.y);
    T* __restrict__ dy = reinterpret_cast<T*>(P.dy);
    const size_t nvec = (size_t)M * C / EPV;
    const T* __restrict__ ap = reinterpret_cast<const T*>(P.add);
    // U vectors a trip, loads first and unconditional (a vector beyond the end re-reads the last one and is dropped)
    constexpr int U = 4;
    unsigned cidx = span.c;
    for (int i0 = 0; i0 < P.per; i0 += U) {
        u32x4 graw[U], yraw[U], araw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t v = span.v + (i0 + u) * span.vstep, vc = v < nvec ? v : nvec - 1;
            graw[u] = Vec<T>::load_raw(gp + vc * EPV);
            yraw[u] = Vec<T>::load_raw(y + vc * EPV);
            if (ap) araw[u] = Vec<T>::load_raw(ap + vc * EPV);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t v = span.v + (i0 + u) * span.vstep;
            const int c0 = (int)cidx * EPV;
            cidx += span.cstep;
            if (cidx >= span.cmod) cidx -= span.cmod;
            if (v >= nvec) continue;
            float gv[EPV], yv[EPV], o[EPV];
            Vec<T>::unpack(graw[u], gv);
            Vec<T>::unpack(yraw[u], yv);
            // the five coefficient vectors of these EPV channels, as 16-byte LDS reads
            float sc[EPV], sh[EPV], k1[EPV], k2[EPV], k3[EPV];
#pragma unroll
            for (int q4 = 0; q4 < EPV / 4; ++q4) {
                const f32x4 a = *reinterpret_cast<const f32x4*>(s_sc + c0 + 4 * q4), b = *reinterpret_cast<const f32x4*>(s_sh + c0 + 4 * q4);
                const f32x4 c = *reinterpret_cast<const f32x4*>(s_k1 + c0 + 4 * q4), d = *reinterpret_cast<const f32x4*>(s_k2 + c0 + 4 * q4);
                const f32x4 f = *reinterpret_cast<const f32x4*>(s_k3 + c0 + 4 * q4);
#pragma unroll
                for (int e = 0; e < 4; ++e) { sc[4 * q4 + e] = a[e]; sh[4 * q4 + e] = b[e]; k1[4 * q4 + e] = c[e]; k2[4 * q4 + e] = d[e]; k3[4 * q4 + e] = f[e]; }
            }
#pragma unroll
            for (int e = 0; e < EPV; ++e) {
                float gg = gv[e];
                if (P.relu && !(fmaf(sc[e], yv[e], sh[e]) > 0.f)) gg = 0.f;
                o[e] = k1[e] * gg - k2[e] * yv[e] + k3[e];
            }
            if (ap) {
                float av[EPV];
                Vec<T>::unpack(araw[u], av);
#pragma unroll
                for (int e = 0; e < EPV; ++e) o[e] += av[e];
            }
            Vec<T>::store(dy + v * EPV, o);
        }
    }
}

// Both passes of the batch-norm backward on few rows, bf16: a workgroup has all rows of 64 channels, so that the sums need no other
// workgroup.  Two launches of 5 to 8 us, each of them two dependent trips to memory, become one, whose second reading of the two
// tensors comes from its L2.  A thread has eight channels of a row lane of a part, as bn_bwd_reduce_kernel cuts the rows (parts x
// lanes, trips of four rows); 64 of those at a time, round by round, the next trip requested ahead of this one's sums.  The order of
// the fp32 sums is that of the two passes (see there), the parts meet in fp64.
__global__ __launch_bounds__(kBnSmallThreads, 2) void bn_bwd_small_kernel(const BnBwdGroup g) {
    constexpr int S = kBnSmallChannels, EPV = 8, CG = S / EPV, CH = kBnSmallThreads / CG, W = kBnSmallThreads / 64;
    __shared__ __attribute__((aligned(16))) float s_part[CH * S * 2];
    __shared__ double s_sum[W / 2 * S * 2];
    __shared__ __attribute__((aligned(16))) float s_c[7 * S];
    const BnBwdProb& P = g.p[find_problem(g, blockIdx.x)];
    const int C = P.C, M = P.M, rl = P.lanes, parts = P.parts;
    const int tid = threadIdx.x, cg = tid % CG, chain = tid / CG, ch0 = ((int)blockIdx.x - P.block_start) * S, c0 = ch0 + cg * EPV;
    const int pr = CH / rl, my = chain / rl, lane_row = chain - my * rl;         // parts at a time; this thread's part of them and row lane
    const int stride = parts * 4 * rl, trips = (M + stride - 1) / stride, steps = (parts + pr - 1) / pr * trips;
    const bf16_t* gp = reinterpret_cast<const bf16_t*>(P.g) + c0;
    const bf16_t* y = reinterpret_cast<const bf16_t*>(P.y) + c0;
    const bool norelu = P.relu == 0;
    if (tid < S) {
        float sc, sh, mu, is;
        bn_coeffs(P.stats, P.gamma, P.beta, ch0 + tid, C, M, g.eps, sc, sh, mu, is);
        s_c[tid] = sc; s_c[S + tid] = sh; s_c[2 * S + tid] = mu; s_c[3 * S + tid] = is;
    }
    // first row of this thread's trip t of the parts from `first` on; M: it has none.  Rows beyond the end read the last row and count for nothing
    auto row_of = [&](int first, int t) { return my < pr && first + my < parts ? (first + my + t * parts) * 4 * rl + lane_row : M; };
    auto request = [&](u32x4 (&gr)[4], u32x4 (&yr)[4], int row) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const unsigned o = (unsigned)min(row + u * rl, M - 1) * (unsigned)C;
            gr[u] = Vec<bf16_t>::load_raw(gp + o);
            yr[u] = Vec<bf16_t>::load_raw(y + o);
        }
    };
    u32x4 ga[4], ya[4], gb[4], yb[4];
    int row = row_of(0, 0), first = 0, t = 0;
    request(ga, ya, row);
    __syncthreads();
    auto coef = [&](int q, float (&c)[EPV]) {
#pragma unroll
        for (int e = 0; e < EPV; e += 4) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(s_c + q * S + cg * EPV + e);
            c[e] = v[0]; c[e + 1] = v[1]; c[e + 2] = v[2]; c[e + 3] = v[3];
        }
    };
    float sc[EPV], sh[EPV];
    coef(0, sc); coef(1, sh);
    double sum = 0.0;                              // of sum tid % 128 of every fourth part
    {
        float mu[EPV], is[EPV], a1[EPV], a2[EPV];
        coef(2, mu); coef(3, is);
#pragma unroll
        for (int e = 0; e < EPV; ++e) { a1[e] = 0.f; a2[e] = 0.f; }
        auto consume = [&](const u32x4 (&gr)[4], const u32x4 (&yr)[4], int at) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float gv[EPV], yv[EPV];
                Vec<bf16_t>::unpack(gr[u], gv);
                Vec<bf16_t>::unpack(yr[u], yv);
                const bool in = at + u * rl < M;
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    const float gg = in & (norelu | (fmaf(sc[e], yv[e], sh[e]) > 0.f)) ? gv[e] : 0.f;
                    a1[e] += gg;
                    a2[e] += gg * ((yv[e] - mu[e]) * is[e]);
                }
            }
        };
        // one trip: the next one is requested first; behind a chain's last trip the row lanes of its parts are added up in order
        auto step = [&](u32x4 (&gr)[4], u32x4 (&yr)[4], u32x4 (&gn)[4], u32x4 (&yn)[4], bool more) {
            const int at = row, from = first;
            const bool last = t + 1 == trips;
            if (last) { t = 0; first += pr; } else ++t;
            row = row_of(first, t);
            if (more) request(gn, yn, row);
            __builtin_amdgcn_sched_barrier(0);
            consume(gr, yr, at);
            if (!last) return;
            float* const q = s_part + (chain * S + cg * EPV) * 2;
#pragma unroll
            for (int e = 0; e < EPV; e += 2) {
                *reinterpret_cast<f32x4*>(q + 2 * e) = f32x4{a1[e], a2[e], a1[e + 1], a2[e + 1]};
            }
#pragma unroll
            for (int e = 0; e < EPV; ++e) { a1[e] = 0.f; a2[e] = 0.f; }
            __syncthreads();
            const int here = min(pr, parts - from);
            for (int p = tid >> 7; p < here; p += W / 2) {
                const float* const r = s_part + p * rl * (S * 2) + (tid & 127);
                float f = 0.f;
#pragma unroll 8
                for (int l = 0; l < rl; ++l) f += r[l * (S * 2)];
                sum += (double)f;
            }
            __syncthreads();
        };
        for (int k = 0; k < steps; k += 2) {
            step(ga, ya, gb, yb, k + 1 < steps);
            if (k + 1 < steps) step(gb, yb, ga, ya, k + 2 < steps);
        }
    }
    s_sum[tid] = sum;
    __syncthreads();
    if (tid < S) {
        double rs0 = 0.0, rs1 = 0.0;
#pragma unroll
        for (int w = 0; w < W / 2; ++w) { rs0 += s_sum[w * (S * 2) + 2 * tid]; rs1 += s_sum[w * (S * 2) + 2 * tid + 1]; }
        const int c = ch0 + tid;
        const double inv_m = 1.0 / (double)M;
        const float r0 = (float)(rs0 * inv_m), r1 = (float)(rs1 * inv_m);
        const float is = s_c[3 * S + tid], k1 = P.gamma[c] * is;
        const float k2 = k1 * is * r1;
        s_c[4 * S + tid] = k1; s_c[5 * S + tid] = k2; s_c[6 * S + tid] = k2 * s_c[2 * S + tid] - k1 * r0;
        P.dgamma[c] = (float)rs1;
        P.dbeta[c] = (float)rs0;
    }
    __syncthreads();
    float k1[EPV], k2[EPV], k3[EPV];
    coef(4, k1); coef(5, k2); coef(6, k3);
    const bf16_t* const ap = P.add ? reinterpret_cast<const bf16_t*>(P.add) + c0 : nullptr;
    bf16_t* const dy = reinterpret_cast<bf16_t*>(P.dy) + c0;
    for (int r0 = chain; r0 < M; r0 += 4 * CH) {
        u32x4 gr[4], yr[4], ar[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const unsigned o = (unsigned)min(r0 + u * CH, M - 1) * (unsigned)C;
            gr[u] = Vec<bf16_t>::load_raw(gp + o);
            yr[u] = Vec<bf16_t>::load_raw(y + o);
            if (ap) ar[u] = Vec<bf16_t>::load_raw(ap + o);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = r0 + u * CH;
            if (r >= M) continue;
            float gv[EPV], yv[EPV], o[EPV];
            Vec<bf16_t>::unpack(gr[u], gv);
            Vec<bf16_t>::unpack(yr[u], yv);
#pragma unroll
            for (int e = 0; e < EPV; ++e) {
                const float gg = norelu | (fmaf(sc[e], yv[e], sh[e]) > 0.f) ? gv[e] : 0.f;
                o[e] = k1[e] * gg - k2[e] * yv[e] + k3[e];
            }
            if (ap) {
                float av[EPV];
                Vec<bf16_t>::unpack(ar[u], av);
#pragma unroll
                for (int e = 0; e < EPV; ++e) o[e] += av[e];
            }
            Vec<bf16_t>::store(dy + (unsigned)r * (unsigned)C, o);
        }
    }
}

// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ float block_sum(float v, float* s_tmp) {
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) v += __shfl_xor(v, sh, 64);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 0) s_tmp[wave] = v;
    __syncthreads();
    float r = 0.f;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) r += s_tmp[w];
    return r;
}

// local penalty / augmented-Lagrangian term and terminal adjoint
template <typename T>
__global__ __launch_bounds__(kElemBlock) void loss_kernel(const LossGroup g) {
    constexpr int EPV = Vec<T>::N;
    __shared__ float s_tmp[kElemBlock / 64];
    const LossProb& P = g.p[find_problem(g, blockIdx.x)];
    const T* __restrict__ y = reinterpret_cast<const T*>(P.y);
    const T* __restrict__ xn = reinterpret_cast<const T*>(P.xn);
    const T* lam = reinterpret_cast<const T*>(P.lam);
    T* lam_out = reinterpret_cast<T*>(P.lam_out);          // may alias lam: every vector is read before it is written
    T* __restrict__ dy = reinterpret_cast<T*>(P.dy);
    const size_t nvec = P.numel / EPV;
    const size_t base = (size_t)(blockIdx.x - P.block_start) * kElemVecsPerBlock;
    float acc = 0.f, racc = 0.f;
    for (int i = threadIdx.x; i < kElemVecsPerBlock; i += kElemBlock) {
        const size_t v = base + i;
        if (v >= nvec) break;
        float a[EPV], b[EPV], l[EPV], o[EPV];
        Vec<T>::load(y + v * EPV, a);
        Vec<T>::load(xn + v * EPV, b);
        if (lam) Vec<T>::load(lam + v * EPV, l);
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            const float r = a[e] - b[e];
            const float lm = lam ? l[e] : 0.f;
            acc += 0.5f * g.rho * r * r + lm * r;
            racc += r * r;
            o[e] = g.scale * (g.rho * r + lm);
        }
        Vec<T>::store(dy + v * EPV, o);
        if (lam && lam_out) {       // multiplier update of the same interface, from the same y - x_next
#pragma unroll
            for (int e = 0; e < EPV; ++e) l[e] = fmaf(g.step, a[e] - b[e], l[e]);
            Vec<T>::store(lam_out + v * EPV, l);
        }
    }
    const float tot = block_sum(acc, s_tmp);
    if (threadIdx.x == 0 && tot != 0.f) atomicAdd(P.loss, g.scale * tot);
    if (P.r2) {
        const float rt = block_sum(racc, s_tmp);
        if (threadIdx.x == 0 && rt != 0.f) atomicAdd(P.r2, rt);
    }
}

// gradient through the ReLU behind a residual sum: gm = g where the stored block output is positive, else 0
template <typename T>
__global__ __launch_bounds__(kElemBlock) void relu_mask_kernel(const MaskGroup g) {
    constexpr int EPV = Vec<T>::N;
    const MaskProb& P = g.p[find_problem(g, blockIdx.x)];
    const T* __restrict__ gp = reinterpret_cast<const T*>(P.g);
    const T* __restrict__ out = reinterpret_cast<const T*>(P.out);
    T* __restrict__ gm = reinterpret_cast<T*>(P.gm);
    const size_t nvec = P.numel / EPV;
    const size_t base = (size_t)(blockIdx.x - P.block_start) * kElemVecsPerBlock;
    for (int i = threadIdx.x; i < kElemVecsPerBlock; i += kElemBlock) {
        const size_t v = base + i;
        if (v >= nvec) break;
        float a[EPV], o[EPV];
        Vec<T>::load(gp + v * EPV, a);
        Vec<T>::load(out + v * EPV, o);
#pragma unroll
        for (int e = 0; e < EPV; ++e) a[e] = o[e] > 0.f ? a[e] : 0.f;
        Vec<T>::store(gm + v * EPV, a);
    }
}

template <typename T>
__global__ __launch_bounds__(kElemBlock) void mult_kernel(const MultGroup g) {
    constexpr int EPV = Vec<T>::N;
    const MultProb& P = g.p[find_problem(g, blockIdx.x)];
    T* __restrict__ lam = reinterpret_cast<T*>(P.lam);
    const T* __restrict__ y = reinterpret_cast<const T*>(P.y);
    const T* __restrict__ xn = reinterpret_cast<const T*>(P.xn);
    const size_t nvec = P.numel / EPV;
    const size_t base = (size_t)(blockIdx.x - P.block_start) * kElemVecsPerBlock;
    for (int i = threadIdx.x; i < kElemVecsPerBlock; i += kElemBlock) {
        const size_t v = base + i;
        if (v >= nvec) break;
        float a[EPV], b[EPV], l[EPV];
        Vec<T>::load(y + v * EPV, a);
        Vec<T>::load(xn + v * EPV, b);
        Vec<T>::load(lam + v * EPV, l);
#pragma unroll
        for (int e = 0; e < EPV; ++e) l[e] = fmaf(g.step, a[e] - b[e], l[e]);
        Vec<T>::store(lam + v * EPV, l);
    }
}

// parameter update, one tensor per problem (bf16 or fp32 parameter, fp32 gradient / velocity / master copy).
// Every tensor starts on a 16-byte boundary of its buffer: four elements per lane and access, scalar tail.
__device__ __forceinline__ float sgd_elem(const SgdGroup& g, float w, float grad, float* v) {
    float d = fmaf(g.wd, w, grad);
    if (v) { d = fmaf(g.momentum, *v, d); *v = d; }
    return fmaf(-g.lr, d, w);
}
__global__ __launch_bounds__(kElemBlock) void sgd_kernel(const SgdGroup g) {
    const SgdProb& P = g.p[find_problem(g, blockIdx.x)];
    const size_t base = (size_t)(blockIdx.x - P.block_start) * kSgdElemsPerBlock;
    unsigned short* pl = reinterpret_cast<unsigned short*>(P.p);
    float* pf = reinterpret_cast<float*>(P.p);
#pragma unroll
    for (int i = 0; i < kSgdElemsPerBlock / (4 * kElemBlock); ++i) {
        const size_t e = base + 4 * ((size_t)i * kElemBlock + threadIdx.x);
        if (e + 4 <= P.numel) {
            f32x4 w;
            if (P.master) w = *reinterpret_cast<const f32x4*>(P.master + e);
            else if (P.lowp) {
                const u32x2 r = *reinterpret_cast<const u32x2*>(pl + e);
                w[0] = __uint_as_float(r[0] << 16); w[1] = __uint_as_float(r[0] & 0xffff0000u);
                w[2] = __uint_as_float(r[1] << 16); w[3] = __uint_as_float(r[1] & 0xffff0000u);
            } else w = *reinterpret_cast<const f32x4*>(pf + e);
            const f32x4 gr = *reinterpret_cast<const f32x4*>(P.g + e);
            f32x4 v;
            if (P.v) v = *reinterpret_cast<const f32x4*>(P.v + e);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float vq = P.v ? v[q] : 0.f;
                w[q] = sgd_elem(g, w[q], gr[q], P.v ? &vq : nullptr);
                v[q] = vq;
            }
            if (P.v) *reinterpret_cast<f32x4*>(P.v + e) = v;
            if (P.master) *reinterpret_cast<f32x4*>(P.master + e) = w;
            if (P.lowp) {
                u32x2 r; r[0] = pack_bf16x2(w[0], w[1]); r[1] = pack_bf16x2(w[2], w[3]);
                *reinterpret_cast<u32x2*>(pl + e) = r;
            } else *reinterpret_cast<f32x4*>(pf + e) = w;
        } else {
            for (size_t t = e; t < P.numel; ++t) {
                float w = P.master ? P.master[t] : (P.lowp ? bf16_bits_to_float(pl[t]) : pf[t]);
                w = sgd_elem(g, w, P.g[t], P.v ? P.v + t : nullptr);
                if (P.master) P.master[t] = w;
                if (P.lowp) pl[t] = float_to_bf16_bits(w);
                else pf[t] = w;
            }
        }
    }
}

// correction of the auxiliary variables: one gradient step of the relaxed objective with respect to x_k
template <typename T>
__global__ __launch_bounds__(kElemBlock) void auxvar_kernel(const AuxVarGroup g) {
    constexpr int EPV = Vec<T>::N;
    const AuxVarProb& P = g.p[find_problem(g, blockIdx.x)];
    T* __restrict__ x = reinterpret_cast<T*>(P.x);
    const T* __restrict__ yp = reinterpret_cast<const T*>(P.yprev);
    const T* __restrict__ dx = reinterpret_cast<const T*>(P.dx);
    const T* __restrict__ lam = reinterpret_cast<const T*>(P.lam);
    T* __restrict__ gout = reinterpret_cast<T*>(P.gout);
    const size_t nvec = P.numel / EPV;
    const size_t base = (size_t)(blockIdx.x - P.block_start) * kElemVecsPerBlock;
    for (int i = threadIdx.x; i < kElemVecsPerBlock; i += kElemBlock) {
        const size_t v = base + i;
        if (v >= nvec) break;
        float a[EPV], b[EPV], d[EPV], l[EPV];
        Vec<T>::load(x + v * EPV, a);
        Vec<T>::load(yp + v * EPV, b);
        Vec<T>::load(dx + v * EPV, d);
        if (lam) Vec<T>::load(lam + v * EPV, l);
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            const float gr = g.scale * (g.rho * (a[e] - b[e]) - (lam ? l[e] : 0.f)) + d[e];
            a[e] = gout ? gr : a[e] - g.eta * gr;
        }
        Vec<T>::store((gout ? gout : x) + v * EPV, a);
    }
}

// ------------------------------------------------------------------------------------------------
// max pooling (first maximum in row-major window order wins); one thread per pixel and 16-byte channel vector
template <typename T>
__global__ __launch_bounds__(256) void maxpool_fwd_kernel(const PoolProb P) {
    constexpr int EPV = Vec<T>::N;
    const int cv = P.C / EPV;
    const size_t total = (size_t)P.N * P.Ho * P.Wo * cv;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const T* __restrict__ x = reinterpret_cast<const T*>(P.x);
    const int c0 = (int)(i % cv) * EPV;
    unsigned r = (unsigned)(i / cv);
    const int wo = (int)(r % (unsigned)P.Wo); r /= (unsigned)P.Wo;
    const int ho = (int)(r % (unsigned)P.Ho);
    const int n = (int)(r / (unsigned)P.Ho);
    float best[EPV];
    int bi[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e) { best[e] = 0.f; bi[e] = -1; }
    for (int a = 0; a < P.R; ++a) {
        const int hi = ho * P.stride - P.pad + a;
        if (hi < 0 || hi >= P.H) continue;
        for (int b = 0; b < P.R; ++b) {
            const int wi = wo * P.stride - P.pad + b;
            if (wi < 0 || wi >= P.W) continue;
            float v[EPV];
            Vec<T>::load(x + ((size_t)(n * P.H + hi) * P.W + wi) * P.C + c0, v);
#pragma unroll
            for (int e = 0; e < EPV; ++e)
                if (bi[e] < 0 || v[e] > best[e]) { best[e] = v[e]; bi[e] = a * P.R + b; }
        }
    }
    const size_t o = (size_t)(i / cv) * P.C + c0;
    Vec<T>::store(reinterpret_cast<T*>(P.y) + o, best);
    uint8_t arg[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e) arg[e] = (uint8_t)bi[e];
    if constexpr (EPV == 8) *reinterpret_cast<uint2*>(P.arg + o) = *reinterpret_cast<const uint2*>(arg);
    else *reinterpret_cast<unsigned*>(P.arg + o) = *reinterpret_cast<const unsigned*>(arg);
}

template <typename T>
__global__ __launch_bounds__(256) void maxpool_bwd_kernel(const PoolProb P) {
    constexpr int EPV = Vec<T>::N;
    const int cv = P.C / EPV;
    const size_t total = (size_t)P.N * P.H * P.W * cv;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const T* __restrict__ dy = reinterpret_cast<const T*>(P.dy);
    const int c0 = (int)(i % cv) * EPV;
    unsigned r = (unsigned)(i / cv);
    const int wi = (int)(r % (unsigned)P.W); r /= (unsigned)P.W;
    const int hi = (int)(r % (unsigned)P.H);
    const int n = (int)(r / (unsigned)P.H);
    float acc[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e) acc[e] = 0.f;
    // windows (ho, wo) that contain (hi, wi): ho*stride - pad + a = hi
    for (int a = 0; a < P.R; ++a) {
        const int th = hi + P.pad - a;
        if (th < 0 || th % P.stride) continue;
        const int ho = th / P.stride;
        if (ho >= P.Ho) continue;
        for (int b = 0; b < P.R; ++b) {
            const int tw = wi + P.pad - b;
            if (tw < 0 || tw % P.stride) continue;
            const int wo = tw / P.stride;
            if (wo >= P.Wo) continue;
            const size_t o = ((size_t)(n * P.Ho + ho) * P.Wo + wo) * P.C + c0;
            float g[EPV];
            Vec<T>::load(dy + o, g);
            uint8_t arg[EPV];
            if constexpr (EPV == 8) *reinterpret_cast<uint2*>(arg) = *reinterpret_cast<const uint2*>(P.arg + o);
            else *reinterpret_cast<unsigned*>(arg) = *reinterpret_cast<const unsigned*>(P.arg + o);
            const uint8_t me = (uint8_t)(a * P.R + b);
#pragma unroll
            for (int e = 0; e < EPV; ++e)
                if (arg[e] == me) acc[e] += g[e];
        }
    }
    Vec<T>::store(reinterpret_cast<T*>(P.dx) + (size_t)(i / cv) * P.C + c0, acc);
}

// ------------------------------------------------------------------------------------------------
// head: pooled[n,c] = mean_{hw} feat;  logits = pooled W^T + b
template <typename T>
__global__ void avgpool_kernel(const HeadProb P) {           // one thread per (n, 16-byte channel vector)
    constexpr int EPV = Vec<T>::N;
    const int cv = P.C / EPV;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= P.N * cv) return;
    const int n = i / cv, c0 = (i % cv) * EPV;
    const T* __restrict__ f = reinterpret_cast<const T*>(P.feat) + (size_t)n * P.HW * P.C + c0;
    float s[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e) s[e] = 0.f;
    int p = 0;
    constexpr int U = 16;                                // independent loads in flight: the pass is a chain of trips to memory
    for (; p + U <= P.HW; p += U) {
        float v[U][EPV];
#pragma unroll
        for (int u = 0; u < U; ++u) Vec<T>::load(f + (size_t)(p + u) * P.C, v[u]);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < EPV; ++e) s[e] += v[u][e];
    }
    for (; p + 4 <= P.HW; p += 4) {
        float v[4][EPV];
#pragma unroll
        for (int u = 0; u < 4; ++u) Vec<T>::load(f + (size_t)(p + u) * P.C, v[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < EPV; ++e) s[e] += v[u][e];
    }
    for (; p < P.HW; ++p) {
        float v[EPV];
        Vec<T>::load(f + (size_t)p * P.C, v);
#pragma unroll
        for (int e = 0; e < EPV; ++e) s[e] += v[e];
    }
#pragma unroll
    for (int e = 0; e < EPV; ++e) P.pooled[n * P.C + c0 + e] = s[e] / (float)P.HW;
}
__global__ void fc_fwd_kernel(const HeadProb P) {          // one wave per (n, class)
    const int o = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (o >= P.N * P.classes) return;
    const int n = o / P.classes, j = o % P.classes, lane = threadIdx.x & 63;
    float s = 0.f;
    for (int c = lane; c < P.C; c += 64) s += P.pooled[n * P.C + c] * P.w[(size_t)j * P.C + c];
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) s += __shfl_xor(s, sh, 64);
    if (lane == 0) P.logits[o] = s + P.b[j];
}
// The same sums in the same order where one output per wave would read too much from L2, two rows for every output (1 GB for 64
// samples x 1000 classes x 2048 channels): a wave owns 8 samples x 4 classes and reads 12 rows for its 32 outputs.
constexpr int kFcSamples = 8, kFcClasses = 4;
__global__ __launch_bounds__(256) void fc_fwd_tiled_kernel(const HeadProb P) {
    const int ncg = (P.classes + kFcClasses - 1) / kFcClasses;
    const int o = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int ng = o / ncg, n0 = ng * kFcSamples, j0 = (o - ng * ncg) * kFcClasses;
    if (n0 >= P.N) return;
    const float *x[kFcSamples], *w[kFcClasses];
#pragma unroll
    for (int i = 0; i < kFcSamples; ++i) x[i] = P.pooled + (size_t)min(n0 + i, P.N - 1) * P.C;
#pragma unroll
    for (int j = 0; j < kFcClasses; ++j) w[j] = P.w + (size_t)min(j0 + j, P.classes - 1) * P.C;
    float s[kFcSamples][kFcClasses];
#pragma unroll
    for (int i = 0; i < kFcSamples; ++i)
#pragma unroll
        for (int j = 0; j < kFcClasses; ++j) s[i][j] = 0.f;
#pragma unroll 4
    for (int c = lane; c < P.C; c += 64) {
        float xv[kFcSamples], wv[kFcClasses];
#pragma unroll
        for (int i = 0; i < kFcSamples; ++i) xv[i] = x[i][c];
#pragma unroll
        for (int j = 0; j < kFcClasses; ++j) wv[j] = w[j][c];
#pragma unroll
        for (int i = 0; i < kFcSamples; ++i)
#pragma unroll
            for (int j = 0; j < kFcClasses; ++j) s[i][j] += xv[i] * wv[j];
    }
#pragma unroll
    for (int i = 0; i < kFcSamples; ++i)
#pragma unroll
        for (int j = 0; j < kFcClasses; ++j) {
#pragma unroll
            for (int sh = 32; sh > 0; sh >>= 1) s[i][j] += __shfl_xor(s[i][j], sh, 64);
            if (lane == 0 && n0 + i < P.N && j0 + j < P.classes) P.logits[(size_t)(n0 + i) * P.classes + j0 + j] = s[i][j] + P.b[j0 + j];
        }
}
// dW[j,c] = sum_n dz[n,j]*pooled[n,c]; db[j] = sum_n dz[n,j]: one thread per element, the samples in order (no
// partial sums to combine: pooled and dz stay in cache, the whole pass reads 2*N values per thread)
__device__ __forceinline__ void fc_bwd_w(const HeadProb& P, int block) {
    const int i = block * 256 + threadIdx.x;
    if (i >= P.classes * P.C) return;
    const int j = i / P.C, c = i % P.C;
    float s = 0.f, sb = 0.f;
#pragma unroll 8
    for (int n = 0; n < P.N; ++n) {
        const float d = P.dlogits[n * P.classes + j];
        s += d * P.pooled[n * P.C + c];
        sb += d;
    }
    P.dw[i] = s;
    if (c == 0) P.db[j] = sb;
}
// The same sums where those reads are what it takes (36 us for 64 samples x 1000 classes x 2048 channels): one thread per
// channel and four classes, pooled read once for them, 32 samples in flight, their dz through LDS, 128 samples at a time.
// For small layers the longer thread is the slower one: 12 us against 8 for 128 samples x 10 classes x 64 channels.
constexpr int kFcTileSamples = 128;
__device__ __forceinline__ void fc_bwd_w_tiles(const HeadProb& P, int block, float* s_dp) {
    constexpr int NB = kFcTileSamples, U = 32;
    float (*const s_dz)[kFcClasses] = reinterpret_cast<float (*)[kFcClasses]>(s_dp);
    const int jb = (P.classes + kFcClasses - 1) / kFcClasses, j0 = block % jb * kFcClasses, c = block / jb * 256 + threadIdx.x;
    const float* __restrict__ x = P.pooled + min(c, P.C - 1);
    float s[kFcClasses], sb[kFcClasses];
#pragma unroll
    for (int j = 0; j < kFcClasses; ++j) s[j] = sb[j] = 0.f;
    for (int nb = 0; nb < P.N; nb += NB) {
        if (nb) __syncthreads();
        for (int i = threadIdx.x; i < NB * kFcClasses; i += 256) {
            const int n = min(nb + i / kFcClasses, P.N - 1), j = min(j0 + i % kFcClasses, P.classes - 1);
            s_dz[i / kFcClasses][i % kFcClasses] = P.dlogits[(size_t)n * P.classes + j];
        }
        __syncthreads();
        for (int n = nb; n < min(nb + NB, P.N); n += U) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = x[(size_t)min(n + u, P.N - 1) * P.C];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (n + u >= P.N) continue;
#pragma unroll
                for (int j = 0; j < kFcClasses; ++j) {
                    const float d = s_dz[n + u - nb][j];
                    s[j] += d * v[u];
                    sb[j] += d;
                }
            }
        }
    }
    if (c >= P.C) return;
#pragma unroll
    for (int j = 0; j < kFcClasses; ++j) {
        if (j0 + j >= P.classes) continue;
        P.dw[(size_t)(j0 + j) * P.C + c] = s[j];
        if (c == 0) P.db[j0 + j] = sb[j];
    }
}
// dfeat[n,p,c] = (sum_j dz[n,j]*W[j,c]) / HW
template <typename T, bool IN_LDS>
__device__ __forceinline__ void fc_bwd_x(const HeadProb& P, int block, float* s_dp) {
    // One block per sample and chunk of 256 channels: d pooled[c] = sum_j dlogits[j] * w[j][c] (lanes along c: coalesced
    // rows of w, summed in the order of the classes), then the block broadcasts it, divided by the number of pixels, to
    // every pixel of the sample with 16-byte stores.
    constexpr int EPV = Vec<T>::N;
    // s_dp: 256 floats, then (IN_LDS) the sample's `classes` logit gradients
    const int n = block % P.N, cbase = block / P.N * 256, C = P.C, classes = P.classes;
    const int nc = min(256, C - cbase);
    const float inv = 1.f / (float)P.HW;
    float* s_dl = s_dp + 256;
    if (IN_LDS) {
        for (int j = threadIdx.x; j < classes; j += 256) s_dl[j] = P.dlogits[(size_t)n * classes + j];
        __syncthreads();
    }
    auto dl = [&](int j) __attribute__((always_inline)) { return IN_LDS ? s_dl[j] : P.dlogits[(size_t)n * classes + j]; };
    if ((int)threadIdx.x < nc) {
        const int c = cbase + threadIdx.x;
        float acc = 0.f;
        // The chain over the classes is one of trips to L2: 64 rows of w in flight (with 8, 66 us for 1000 classes
        // whatever the mini-batch).  The last rows go 16, 8 and 4 at a time, so that at most three are read in vain (all
        // samples of a large mini-batch together are bound by what they read: with 16 for two classes of 2048 samples and
        // 1024 channels the backward pass of the head took 137 us instead of 125).
        int j = 0;
        for (; j + 63 < classes; j += 64) {
            float w[64];
#pragma unroll
            for (int u = 0; u < 64; ++u) w[u] = P.w[(size_t)(j + u) * C + c];
#pragma unroll
            for (int u = 0; u < 64; ++u) acc += dl(j + u) * w[u];
        }
        for (; j + 15 < classes; j += 16) {
            float w[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) w[u] = P.w[(size_t)(j + u) * C + c];
#pragma unroll
            for (int u = 0; u < 16; ++u) acc += dl(j + u) * w[u];
        }
        if (j + 7 < classes) {
            float w[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) w[u] = P.w[(size_t)(j + u) * C + c];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += dl(j + u) * w[u];
            j += 8;
        }
        for (; j < classes; j += 4) {
            float w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) w[u] = P.w[(size_t)min(j + u, classes - 1) * C + c];
#pragma unroll
            for (int u = 0; u < 4; ++u) if (j + u < classes) acc += dl(j + u) * w[u];
        }
        s_dp[threadIdx.x] = acc * inv;
    }
    __syncthreads();
    T* __restrict__ d = reinterpret_cast<T*>(P.dfeat) + (size_t)n * P.HW * C + cbase;
    const int cvn = nc / EPV;
    for (int i = threadIdx.x; i < P.HW * cvn; i += 256) {
        const int p = i / cvn, v = i - p * cvn;
        float o[EPV];
#pragma unroll
        for (int e = 0; e < EPV; ++e) o[e] = s_dp[v * EPV + e];
        Vec<T>::store(d + (size_t)p * C + v * EPV, o);
    }
}
// Both halves of the linear layer's backward pass: they read the same logit gradients and neither waits for the other, so
// they are one launch, the workgroups of the half that the next launches wait for (dfeat) first.
// The halves' arrays share their LDS, which a workgroup has one of: 40193 to 40704 classes fit a compute unit's 160 KB only so, and
// the logit gradients of more are read from memory.
template <typename T, bool TILED, bool IN_LDS>
__global__ __launch_bounds__(256) void fc_bwd_kernel(const HeadProb P, int xblocks) {
    extern __shared__ __attribute__((aligned(16))) float s_dp[];
    if ((int)blockIdx.x < xblocks) { fc_bwd_x<T, IN_LDS>(P, blockIdx.x, s_dp); return; }
    if (TILED) fc_bwd_w_tiles(P, (int)blockIdx.x - xblocks, s_dp);
    else fc_bwd_w(P, (int)blockIdx.x - xblocks);
}

// softmax cross-entropy of sample n by one workgroup, mini-batch mean; z: its logits
__device__ __forceinline__ void ce_sample(const float* z, const int n, const int lab, float* loss,
                                          float* __restrict__ dlogits, int N, int classes) {
    __shared__ float s_tmp[kElemBlock / 64];
    __shared__ float s_max[kElemBlock / 64];
    float mx = -INFINITY;
    for (int j = threadIdx.x; j < classes; j += kElemBlock) mx = fmaxf(mx, z[j]);
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) mx = fmaxf(mx, __shfl_xor(mx, sh, 64));
    if ((threadIdx.x & 63) == 0) s_max[threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = s_max[0];
    for (int w = 1; w < kElemBlock / 64; ++w) mx = fmaxf(mx, s_max[w]);
    float se = 0.f;
    for (int j = threadIdx.x; j < classes; j += kElemBlock) se += __expf(z[j] - mx);
    se = block_sum(se, s_tmp);
    const float inv = 1.f / se, invN = 1.f / (float)N;
    for (int j = threadIdx.x; j < classes; j += kElemBlock) {
        float p = __expf(z[j] - mx) * inv;
        if (j == lab) p -= 1.f;
        dlogits[(size_t)n * classes + j] = p * invN;
    }
    if (threadIdx.x == 0) atomicAdd(loss, (logf(se) + mx - z[lab]) * invN);
}
__global__ __launch_bounds__(kElemBlock) void ce_kernel(const float* __restrict__ logits, const int32_t* __restrict__ labels,
                                                        float* loss, float* __restrict__ dlogits, int N, int classes) {
    ce_sample(logits + (size_t)blockIdx.x * classes, blockIdx.x, labels[blockIdx.x], loss, dlogits, N, classes);
}
// The head of a small network in one launch, a workgroup per sample: the sums of avgpool_kernel, fc_fwd_kernel and ce_kernel in
// their order, with the sample's features, means and logits in LDS between them.  Bound by its three trips to memory (features,
// then nothing but stores; weights and label are requested with the features).
template <typename T>
__global__ __launch_bounds__(kElemBlock) void head_loss_kernel(const HeadProb P) {
    constexpr int EPV = Vec<T>::N, W = kElemBlock / 64, PRE = 4, CL = 8;
    extern __shared__ __attribute__((aligned(16))) char s_head[];
    const int n = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int HW = P.HW, C = P.C, nvec = HW * (C / EPV);
    T* const s_feat = reinterpret_cast<T*>(s_head);
    float* const s_pool = reinterpret_cast<float*>(s_head + (size_t)nvec * 16);
    float* const s_z = s_pool + C;
    const u32x4* __restrict__ f = reinterpret_cast<const u32x4*>(P.feat) + (size_t)n * nvec;
    u32x4 v[PRE];                                  // this thread's first vectors, and the weights and biases of its wave's first classes
    float w[CL], b[CL];
#pragma unroll
    for (int u = 0; u < PRE; ++u) v[u] = f[min(tid + u * kElemBlock, nvec - 1)];
#pragma unroll
    for (int u = 0; u < CL; ++u) {
        const int j = min(wave + u * W, P.classes - 1);
        w[u] = P.w[(size_t)j * C + min(lane, C - 1)];
        b[u] = P.b[j];
    }
    const int lab = P.labels[n];
#pragma unroll
    for (int u = 0; u < PRE; ++u)
        if (tid + u * kElemBlock < nvec) reinterpret_cast<u32x4*>(s_feat)[tid + u * kElemBlock] = v[u];
    for (int i = tid + PRE * kElemBlock; i < nvec; i += kElemBlock) reinterpret_cast<u32x4*>(s_feat)[i] = f[i];
    __syncthreads();
    for (int c = tid; c < C; c += kElemBlock) {
        float s = 0.f;
#pragma unroll 16
        for (int p = 0; p < HW; ++p) s += to_float(s_feat[p * C + c]);
        s /= (float)HW;
        s_pool[c] = s;
        P.pooled[(size_t)n * C + c] = s;
    }
    __syncthreads();
    // CL classes of a wave at a time, the next ones' weights under way (128 samples x 100 classes x 64 channels with a trip to memory
    // for each class of a wave 19.5 us, so 9.4; ResNet-56 of 128 samples in four modules 733 -> 727)
    for (int j0 = wave; j0 < P.classes; j0 += W * CL) {
        float wn[CL], bn[CL], s[CL];
#pragma unroll
        for (int u = 0; u < CL; ++u) {
            const int j = min(j0 + (CL + u) * W, P.classes - 1);
            wn[u] = P.w[(size_t)j * C + min(lane, C - 1)];
            bn[u] = P.b[j];
            s[u] = lane < C ? s_pool[lane] * w[u] : 0.f;
        }
        for (int c = lane + 64; c < C; c += 64)
#pragma unroll
            for (int u = 0; u < CL; ++u) s[u] += s_pool[c] * P.w[(size_t)min(j0 + u * W, P.classes - 1) * C + c];
#pragma unroll
        for (int sh = 32; sh > 0; sh >>= 1)
#pragma unroll
            for (int u = 0; u < CL; ++u) s[u] += __shfl_xor(s[u], sh, 64);
#pragma unroll
        for (int u = 0; u < CL; ++u) {
            const int j = j0 + u * W;
            if (lane == 0 && j < P.classes) {
                s_z[j] = s[u] + b[u];
                P.logits[(size_t)n * P.classes + j] = s[u] + b[u];
            }
            w[u] = wn[u]; b[u] = bn[u];
        }
    }
    __syncthreads();
    ce_sample(s_z, n, lab, P.loss, const_cast<float*>(P.dlogits), P.N, P.classes);
}

__global__ void zero_selected_kernel(float* v, uint32_t mask, int n, float* v2, uint32_t mask2, int n2) {
    const int i = threadIdx.x;
    if (i < n && ((mask >> i) & 1u)) v[i] = 0.f;
    if (v2 && i < n2 && ((mask2 >> i) & 1u)) v2[i] = 0.f;
}

}  // namespace

// ------------------------------------------------------------------------------------------------
#define LP_DISPATCH_T(dtype, KERNEL, grid, block, stream, ...)                                   \
    do {                                                                                         \
        if ((dtype) == 1) hipLaunchKernelGGL(KERNEL<bf16_t>, grid, block, 0, stream, __VA_ARGS__); \
        else hipLaunchKernelGGL(KERNEL<float>, grid, block, 0, stream, __VA_ARGS__);             \
    } while (0)

hipError_t launch_bn_apply(const BnApplyGroup& g, int dtype, bool fused_loss, hipStream_t s) {
    if (g.total_blocks <= 0) return hipSuccess;
    const size_t lds = (size_t)4 * g.cmax * sizeof(float);
    const dim3 grid(g.total_blocks), block(kElemBlock);
    if (dtype == 1) {
        if (fused_loss) hipLaunchKernelGGL((bn_apply_kernel<bf16_t, true>), grid, block, lds, s, g);
        else hipLaunchKernelGGL((bn_apply_kernel<bf16_t, false>), grid, block, lds, s, g);
    } else {
        if (fused_loss) hipLaunchKernelGGL((bn_apply_kernel<float, true>), grid, block, lds, s, g);
        else hipLaunchKernelGGL((bn_apply_kernel<float, false>), grid, block, lds, s, g);
    }
    return hipGetLastError();
}
hipError_t launch_bn_bwd_reduce(const BnBwdGroup& g, int dtype, hipStream_t s) {
    if (g.total_blocks <= 0) return hipSuccess;
    const size_t lds = (size_t)4 * g.cmax * sizeof(float);
    if (g.threads == 256) {
        if (dtype == 1) hipLaunchKernelGGL((bn_bwd_reduce_kernel<bf16_t, 256>), dim3(g.total_blocks), dim3(256), lds, s, g);
        else hipLaunchKernelGGL((bn_bwd_reduce_kernel<float, 256>), dim3(g.total_blocks), dim3(256), lds, s, g);
        return hipGetLastError();
    }
    if (dtype == 1) hipLaunchKernelGGL((bn_bwd_reduce_kernel<bf16_t, kBnReduceBlock>), dim3(g.total_blocks), dim3(kBnReduceBlock), lds, s, g);
    else hipLaunchKernelGGL((bn_bwd_reduce_kernel<float, kBnReduceBlock>), dim3(g.total_blocks), dim3(kBnReduceBlock), lds, s, g);
    return hipGetLastError();
}
hipError_t launch_bn_stats(const BnBwdGroup& g, int dtype, hipStream_t s) {
    if (g.total_blocks <= 0) return hipSuccess;
    LP_DISPATCH_T(dtype, bn_stats_kernel, dim3(g.total_blocks), dim3(kElemBlock), s, g);
    return hipGetLastError();
}
hipError_t launch_bn_bwd_apply(const BnBwdGroup& g, int dtype, hipStream_t s) {
    if (g.total_blocks <= 0) return hipSuccess;
    const size_t lds = (size_t)5 * g.cmax * sizeof(float);
    if (dtype == 1) hipLaunchKernelGGL(bn_bwd_apply_kernel<bf16_t>, dim3(g.total_blocks), dim3(kElemBlock), lds, s, g);
    else hipLaunchKernelGGL(bn_bwd_apply_kernel<float>, dim3(g.total_blocks), dim3(kElemBlock), lds, s, g);
    return hipGetLastError();
}
hipError_t launch_relu_mask(const MaskGroup& g, int dtype, hipStream_t s) {
    if (g.total_blocks <= 0) return hipSuccess;
    LP_DISPATCH_T(dtype, relu_mask_kernel, dim3(g.total_blocks), dim3(kElemBlock), s, g);
    return hipGetLastError();
}
hipError_t launch_loss(const LossGroup& g, int dtype, hipStream_t s) {
    if (g.total_blocks <= 0) return hipSuccess;
    LP_DISPATCH_T(dtype, loss_kernel, dim3(g.total_blocks), dim3(kElemBlock), s, g);
    return hipGetLastError();
}
hipError_t launch_sgd(const SgdGroup& g, hipStream_t s) {
    if (g.total_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(sgd_kernel, dim3(g.total_blocks), dim3(kElemBlock), 0, s, g);
    return hipGetLastError();
}
hipError_t launch_auxvar(const AuxVarGroup& g, int dtype, hipStream_t s) {
    if (g.total_blocks <= 0) return hipSuccess;
    LP_DISPATCH_T(dtype, auxvar_kernel, dim3(g.total_blocks), dim3(kElemBlock), s, g);
    return hipGetLastError();
}
hipError_t launch_mult(const MultGroup& g, int dtype, hipStream_t s) {
    if (g.total_blocks <= 0) return hipSuccess;
    LP_DISPATCH_T(dtype, mult_kernel, dim3(g.total_blocks), dim3(kElemBlock), s, g);
    return hipGetLastError();
}
hipError_t launch_bn_bwd_small(const BnBwdGroup& g, hipStream_t s) {
    if (g.total_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(bn_bwd_small_kernel, dim3(g.total_blocks), dim3(kBnSmallThreads), 0, s, g);
    return hipGetLastError();
}
hipError_t launch_maxpool_fwd(const PoolProb& p, int dtype, hipStream_t s) {
    const size_t total = (size_t)p.N * p.Ho * p.Wo * (p.C / (dtype == 1 ? 8 : 4));
    LP_DISPATCH_T(dtype, maxpool_fwd_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), s, p);
    return hipGetLastError();
}
hipError_t launch_maxpool_bwd(const PoolProb& p, int dtype, hipStream_t s) {
    const size_t total = (size_t)p.N * p.H * p.W * (p.C / (dtype == 1 ? 8 : 4));
    LP_DISPATCH_T(dtype, maxpool_bwd_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), s, p);
    return hipGetLastError();
}
// The linear layer's tiled kernels do less but take longer chains, a few workgroups of them do not fill the chip.  Forward: the
// tiled kernel takes 17 us until its waves fill it, one output per wave 9 us and 0.1 ns + 0.6 ps * C per output (tiled / plain:
// 128 samples x 100 classes x 640 channels 18.1 / 15.4 us, 256 samples 18.3 / 22.3; 8 x 1000 x 2048 25.6 / 24.3, 12 samples 24.8 /
// 33.7; 4096 x 10 x 128 17.4 / 16.0, 8192 x 10 x 64 17.4 / 20.5).
bool fc_fwd_tiled(const HeadProb& p) { return (size_t)p.N * p.classes * (p.C + 170) >= 18000000u; }
// Filter gradient: a thread of the tiled kernel has four classes, so it wants that many more of them (whole backward pass of the
// head, tiled / plain: 128 samples x 100 classes x 640 channels 20.6 / 15.3 us, 512 x 200 x 1024 68.0 / 60.6, 2048 x 1000 x 64 199 /
// 149, 8192 x 10 x 64 681 / 424; 1024 x 512 x 640 137 / 148, 64 x 1000 x 512 29 / 50, 16 x 1000 x 2048 39 / 79).
bool fc_bwd_w_tiled(const HeadProb& p) {
    return (size_t)p.classes * p.C >= (1u << 18) && (size_t)p.N * p.classes * p.C >= (1u << 22);
}
hipError_t launch_head_fwd(const HeadProb& p, int dtype, hipStream_t s) {
    const int epv = dtype == 1 ? 8 : 4;
    if (p.labels) {
        const size_t lds = (size_t)p.HW * p.C * (dtype == 1 ? 2 : 4) + (p.C + p.classes) * sizeof(float);
        if (dtype == 1) hipLaunchKernelGGL(head_loss_kernel<bf16_t>, dim3(p.N), dim3(kElemBlock), lds, s, p);
        else hipLaunchKernelGGL(head_loss_kernel<float>, dim3(p.N), dim3(kElemBlock), lds, s, p);
        return hipGetLastError();
    }
    LP_DISPATCH_T(dtype, avgpool_kernel, dim3((p.N * (p.C / epv) + 63) / 64), dim3(64), s, p);
    if (fc_fwd_tiled(p)) {
        const size_t waves = (size_t)((p.N + kFcSamples - 1) / kFcSamples) * ((p.classes + kFcClasses - 1) / kFcClasses);
        hipLaunchKernelGGL(fc_fwd_tiled_kernel, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, p);
    } else
        hipLaunchKernelGGL(fc_fwd_kernel, dim3((p.N * p.classes + 3) / 4), dim3(256), 0, s, p);
    return hipGetLastError();
}
template <typename T, bool IN_LDS>
static void head_bwd(const HeadProb& p, hipStream_t s) {
    const int cb = (p.C + 255) / 256, xblocks = p.N * cb;
    const size_t lds = std::max(256 + (IN_LDS ? p.classes : 0), kFcTileSamples * kFcClasses) * sizeof(float);
    if (fc_bwd_w_tiled(p))
        hipLaunchKernelGGL((fc_bwd_kernel<T, true, IN_LDS>), dim3(xblocks + (p.classes + kFcClasses - 1) / kFcClasses * cb), dim3(256), lds, s, p, xblocks);
    else
        hipLaunchKernelGGL((fc_bwd_kernel<T, false, IN_LDS>), dim3(xblocks + (p.classes * p.C + 255) / 256), dim3(256), lds, s, p, xblocks);
}
hipError_t launch_head_bwd(const HeadProb& p, int dtype, hipStream_t s) {
    constexpr int kMostInLds = 160 * 1024 / (int)sizeof(float) - 256;
    if (p.classes <= kMostInLds) {
        if (dtype == 1) head_bwd<bf16_t, true>(p, s);
        else head_bwd<float, true>(p, s);
    } else if (dtype == 1) head_bwd<bf16_t, false>(p, s);
    else head_bwd<float, false>(p, s);
    return hipGetLastError();
}
hipError_t launch_zero_selected(float* v, uint32_t mask, int n, float* v2, uint32_t mask2, int n2, hipStream_t s) {
    hipLaunchKernelGGL(zero_selected_kernel, dim3(1), dim3(64), 0, s, v, mask, n, v2, mask2, n2);
    return hipGetLastError();
}
hipError_t launch_ce(const float* logits, const int32_t* labels, float* loss, float* dlogits, int N, int classes,
                     hipStream_t s) {
    hipLaunchKernelGGL(ce_kernel, dim3(N), dim3(kElemBlock), 0, s, logits, labels, loss, dlogits, N, classes);
    return hipGetLastError();
}

}  // namespace lp
