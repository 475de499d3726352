// Gibbs contractions in the log domain (the absorbed iteration), exact up to
// float rounding.
//
// After the absorption switch the scalings are carried as logs, and one axis
// of a product xi x becomes, per output i of a fibre X of length n,
//     Y[i] = log sum_k exp(X[k] - alpha (i - k)^2),   alpha = 1 / (n^2 gamma)
// (the log of the separable factor K1[i][k] = exp(-(x_i - x_k)^2 / gamma)).
// Each output takes its own shift, the largest term M[i] = max_k (X[k] -
// alpha (i - k)^2), so the largest term is exp(0) = 1 and no term that
// matters to float precision is lost.  No band is assumed: a log input may
// exceed its neighbours by more than the factor's float range, so the max and
// the sum run over windows derived from the fibre's largest value Xmax:
//   - the max starts on |i - k| <= R0 and widens to
//     alpha (i - k)^2 <= Xmax - M (no term beyond can be larger);
//   - the sum runs over alpha (i - k)^2 <= Xmax - M + 40 (every term beyond
//     is below e^-40 of the largest: all 1023 of them together move the sum by
//     less than 5e-15 of it, a millionth of its last float32 bit).
// Exponents are formed in FP64 from the float inputs and rounded to float
// once the shift is taken off.  This is plain ALU work (a max-plus pass and
// exponentials), not a dense contraction, so it does not use MFMA; it runs
// only in the log domain.
//
// Layout: the field is [outer][n][inner] (the contracted axis has stride
// inner); outputs keep that layout, so d passes (contiguous axis first) apply
// xi, the last one handing its values (logs) to the pointwise epilogue.
//
// Split: a work item is 256 outputs (whole rows or a row's chunk of 256 along
// the contiguous axis, 16 x 16 outputs and neighbouring fibres along a strided
// one) whose fibres are staged in LDS; four groups of four waves take every
// fourth distance d of each output, i - d and i + d at once, so the d^2 term is
// shared by the pair and by all lanes.  A 256 x 256 field is 256 items: one
// block of 16 waves on each CU, four waves per SIMD.
// Bound: instruction issue, about 11 slots a term (2 for the max, 9 for the
// sum, of them 4 the exponential) and some 60 to 100 terms an output.  256 x
// 256 at gamma = 2e-4, an iteration of four passes: 46 us; 247 us with a thread
// an output, whole 64-fibre blocks staged and the float band scanned twice.
#include <math.h>

#include <algorithm>

#include "epilogue.h"
#include "logpass.h"

namespace jko {

namespace {

constexpr int kLOut = 256;              // outputs of an item
constexpr int kLSplit = 4;              // groups of waves sharing an output's terms
constexpr int kLThr = kLOut * kLSplit;
constexpr int kLStrided = 16;           // fibres of an item along a strided axis
constexpr int kLMaxBlocks = 1024;       // items beyond are taken in turn (bounds the partial sums' slots)
constexpr double kLog2e = 1.4426950408889634074;
constexpr double kCut = 40.0;           // the sum's reach below the largest term

// Floats as integers of the same order (for the LDS maximum).
__device__ __forceinline__ int ordered(float x) {
    const int b = __float_as_int(x);
    return b >= 0 ? b : b ^ 0x7fffffff;
}
__device__ __forceinline__ float unordered(int k) { return __int_as_float(k >= 0 ? k : k ^ 0x7fffffff); }

template <int EK>
__global__ void __launch_bounds__(kLThr) log_pass_kernel(LogPass L, EpiArgs E) {
    extern __shared__ float xs[];       // the staged fibres
    __shared__ float pmax[kLSplit][kLOut], psum[kLSplit][kLOut];
    __shared__ int xkey[kLOut];         // each fibre's largest value
    __shared__ double shd[kLThr / 64];
    if (E.ctl && E.ctl->done) return;   // the step has stopped (uniform)

    const int tid = threadIdx.x, split = tid / kLOut, out = tid % kLOut;
    const int n = L.n, OI = L.OI, OF = L.OF;
    const bool contig = L.inner == 1;
    const int st = contig ? 1 : kLStrided;            // LDS stride of the axis
    const int f_ = contig ? out / OI : out % kLStrided, il = contig ? out % OI : out / kLStrided;
    const double alpha = L.alpha, a2 = L.alpha * kLog2e;
    EpiAcc acc;
    for (int64_t item = blockIdx.x; item < L.items; item += gridDim.x) {
        const int64_t fb = item / L.chunks;
        const int i0 = (int)(item % L.chunks) * OI;
        // fibre f of this item: contiguous axis: row r0 + f; strided: (o, j0 + f)
        int64_t r0 = 0, o = 0, j0 = 0;
        int nf;
        if (contig) {
            r0 = fb * OF;
            nf = (int)(L.outer - r0 < OF ? L.outer - r0 : OF);
        } else {
            const int64_t jb = (L.inner + kLStrided - 1) / kLStrided;
            o = fb / jb;
            j0 = (fb % jb) * kLStrided;
            nf = (int)(L.inner - j0 < kLStrided ? L.inner - j0 : kLStrided);
        }
        const bool live = f_ < nf && il < OI && i0 + il < n;
        const int f = live ? f_ : 0, i = live ? i0 + il : 0;
        const int64_t idx = contig ? (r0 + f) * n + i : (o * n + i) * L.inner + j0 + f;
        EpiIn in;
        if (EK != EK_STORE && split == 0) in = epi_prefetch<EK, false, false, 1>(E, (int)idx, live ? 1 : 0);

        // stage the fibres and take each one's largest value
        __syncthreads();   // (the previous item's reads are done)
        if (tid < kLOut) xkey[tid] = ordered(-INFINITY);
        __syncthreads();
        if (contig) {
            const int T = L.T, fs = tid / T, q = tid % T;   // T threads per fibre (a power of two)
            float m = -INFINITY;
            if (fs < nf)
                for (int c = q; c < n; c += T) {
                    const float v = L.X[(r0 + fs) * n + c];
                    xs[fs * n + c] = v;
                    m = fmaxf(m, v);
                }
            const int w = T < 64 ? T : 64;
            for (int s = w >> 1; s > 0; s >>= 1) m = fmaxf(m, __shfl_xor(m, s, 64));
            if (fs < nf && (tid & (w - 1)) == 0) atomicMax(&xkey[fs], ordered(m));
        } else {
            const int js = tid % kLStrided;
            float m = -INFINITY;
            for (int c = tid / kLStrided; c < n; c += kLThr / kLStrided) {
                const float v = js < nf ? L.X[(o * n + c) * L.inner + j0 + js] : -INFINITY;
                xs[c * kLStrided + js] = v;
                m = fmaxf(m, v);
            }
            m = fmaxf(m, __shfl_xor(m, 16, 64));
            m = fmaxf(m, __shfl_xor(m, 32, 64));
            if ((tid & 63) < kLStrided) atomicMax(&xkey[js], ordered(m));
        }
        __syncthreads();
        const float xm = unordered(xkey[f]);
        const float* x = xs + (contig ? f * n : f);
        // the two terms at distance d (-inf outside the fibre, and once for d = 0)
        auto up = [&](int d) { return i + d < n ? x[(i + d) * st] : -INFINITY; };
        auto dn = [&](int d) { return i - d >= 0 && d > 0 ? x[(i - d) * st] : -INFINITY; };

        // largest term: a first window, then as far as a term could beat it
        float best = -INFINITY;
#pragma unroll 2
        for (int d = split; d <= L.R0; d += kLSplit) {
            const float ad = (float)(alpha * (double)d * (double)d);
            best = fmaxf(best, fmaxf(up(d), dn(d)) - ad);
        }
        pmax[split][out] = best;
        __syncthreads();
#pragma unroll
        for (int s = 0; s < kLSplit; ++s) best = fmaxf(best, pmax[s][out]);
        int R = 0;
        if (live && xm > -INFINITY) {
            const double reach = (best == -INFINITY) ? (double)n : sqrt((double)(xm - best) / alpha) + 1.0;
            R = (int)fmin(reach, (double)(n - 1));
        }
        if (__syncthreads_or(R > L.R0)) {
            for (int s = 32; s > 0; s >>= 1) R = max(R, __shfl_xor(R, s, 64));
            for (int d = L.R0 + 1 + split; d <= R; d += kLSplit) {
                const float ad = (float)(alpha * (double)d * (double)d);
                best = fmaxf(best, fmaxf(up(d), dn(d)) - ad);
            }
            pmax[split][out] = best;
            __syncthreads();
#pragma unroll
            for (int s = 0; s < kLSplit; ++s) best = fmaxf(best, pmax[s][out]);
        }
        // the sum over every term within e^-kCut of the largest
        const double M = best, M2 = M * kLog2e;
        int R2 = 0;
        if (live && xm > -INFINITY) R2 = (int)fmin(sqrt(((double)xm - M + kCut) / alpha) + 1.0, (double)(n - 1));
        for (int s = 32; s > 0; s >>= 1) R2 = max(R2, __shfl_xor(R2, s, 64));
        float sum = 0.f;
#pragma unroll 2
        for (int d = split; d <= R2; d += kLSplit) {
            const double sh = -((a2 * (double)d) * (double)d + M2);
            sum += __builtin_amdgcn_exp2f((float)__builtin_fma((double)up(d), kLog2e, sh));
            sum += __builtin_amdgcn_exp2f((float)__builtin_fma((double)dn(d), kLog2e, sh));
        }
        psum[split][out] = sum;
        __syncthreads();
        if (split == 0 && live) {
#pragma unroll
            for (int s = 1; s < kLSplit; ++s) sum += psum[s][out];
            const float y = xm > -INFINITY ? (float)(M + (double)logf(sum)) : xm;
            if (EK == EK_STORE) E.y[idx] = y;
            else epi_apply<EK, false, 1>(E, (int)idx, 1, f4{y, 0.f, 0.f, 0.f}, true, in, acc);
        }
    }
    epi_finish<false>(E, acc, (int)blockIdx.x, shd);
}

}  // namespace

LogPass make_log_pass(int64_t outer, int n, int64_t inner, double gamma, const float* X) {
    LogPass L{};
    L.outer = outer;
    L.n = n;
    L.inner = inner;
    L.alpha = 1.0 / ((double)n * (double)n * gamma);
    L.X = X;
    L.R0 = (int)std::min(sqrt(kCut / L.alpha) + 1.0, (double)(n - 1));
    if (inner == 1) {
        L.chunks = (n + kLOut - 1) / kLOut;
        L.OI = (n + L.chunks - 1) / L.chunks;
        L.OF = L.chunks > 1 ? 1 : kLOut / L.OI;
        int p = 1;
        while (p < L.OF) p *= 2;
        L.T = kLThr / p;
        L.items = (outer + L.OF - 1) / L.OF * L.chunks;
    } else {
        L.OI = kLOut / kLStrided;
        L.OF = kLStrided;
        L.T = 0;
        L.chunks = (n + L.OI - 1) / L.OI;
        L.items = outer * ((inner + kLStrided - 1) / kLStrided) * L.chunks;
    }
    return L;
}

int64_t log_pass_blocks(const LogPass& L) { return std::min<int64_t>(L.items, kLMaxBlocks); }

hipError_t launch_log_pass(const LogPass& L, const EpiArgs& epi, int* nblocks, hipStream_t st) {
    const int64_t nb = log_pass_blocks(L);
    if (nb > epi.part.cap && epi.kind != EpiKind::STORE) return hipErrorInvalidValue;
    if (nblocks) *nblocks = (int)nb;
    const dim3 grid((unsigned)nb), block(kLThr);
    const size_t lds = (size_t)L.OF * L.n * sizeof(float);
    switch (ek_of(epi)) {
        case EK_STORE: log_pass_kernel<EK_STORE><<<grid, block, lds, st>>>(L, epi); break;
        case EK_BUPDATE: log_pass_kernel<EK_BUPDATE><<<grid, block, lds, st>>>(L, epi); break;
        case EK_MONITOR: log_pass_kernel<EK_MONITOR><<<grid, block, lds, st>>>(L, epi); break;
        case EK_PROX + JKO_F_ZERO: log_pass_kernel<EK_PROX + JKO_F_ZERO><<<grid, block, lds, st>>>(L, epi); break;
        case EK_PROX + JKO_F_CONGESTION:
            log_pass_kernel<EK_PROX + JKO_F_CONGESTION><<<grid, block, lds, st>>>(L, epi);
            break;
        case EK_PROX + JKO_F_POROUS: log_pass_kernel<EK_PROX + JKO_F_POROUS><<<grid, block, lds, st>>>(L, epi); break;
        case EK_PROX + JKO_F_ENTROPY: log_pass_kernel<EK_PROX + JKO_F_ENTROPY><<<grid, block, lds, st>>>(L, epi); break;
        case EK_PROX + JKO_F_CONGESTION_BINARY:
            log_pass_kernel<EK_PROX + JKO_F_CONGESTION_BINARY><<<grid, block, lds, st>>>(L, epi);
            break;
        case EK_PROX + JKO_F_GEN_ENTROPY:
            log_pass_kernel<EK_PROX + JKO_F_GEN_ENTROPY><<<grid, block, lds, st>>>(L, epi);
            break;
        default: return hipErrorInvalidValue;   // the adjoint has no log domain
    }
    return hipGetLastError();
}

}  // namespace jko
