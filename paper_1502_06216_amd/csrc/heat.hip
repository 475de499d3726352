// Heat-kernel Gibbs operator (Section 4.1, eq. heat-kernel) on a masked 2D
// grid: construction of the dense operator and its application with the
// scaling iteration's pointwise epilogues.
//
// The paper applies xi~ = (Id - (gamma/L) Delta_M)^{-L} by L sparse
// back-substitutions per product, a sequential sweep.  On this device the
// operator of a grid of up to 2^16 cells fits HBM as a dense float32 matrix,
// so it is built once per (domain, gamma, L), and every product of the
// iteration becomes one memory-bound pass over it whose tiles run in
// parallel.  The operator acts on the free cells only, and only its upper
// triangle is stored (xi~ is symmetric): the 9556 free cells of a 100 x 100
// room take 187 MB, which fits the device's 256 MB last-level cache.
//
// Grids of more than 2^16 cells (or on request) take the paper's own form
// instead, nothing stored: each product is (Id - (gamma/L) Delta_M)^-L on the
// grid, as one Chebyshev series of the operator in FP64 (a stencil sweep per
// degree, linear in the grid's size), and its result goes through the same
// epilogues.
//
// Construction: the columns of xi~ are the same series applied to unit
// vectors, a chunk of columns per launch.  M = Id + nu_0 G_0 + nu_1 G_1 is
// symmetric with spectrum in [1, 1 + 4 nu_0 + 4 nu_1] (Gershgorin; G_k is
// positive semi-definite).
#include <math.h>

#include <algorithm>
#include <new>
#include <vector>

#include "heat_tile.h"

namespace jko {

static_assert(HEAT_EK_STORE == EK_STORE && HEAT_EK_BUPDATE == EK_BUPDATE && HEAT_EK_MONITOR == EK_MONITOR &&
                  HEAT_EK_PROX == EK_PROX,
              "heat epilogue codes follow the band contractions' codes");

namespace {

__device__ __forceinline__ bool is_free(const uint8_t* mask, int64_t i) { return !mask || mask[i]; }

// One product (or one column of the stored operator) as a Chebyshev series.
// M has its spectrum in [1, beta], so with u = (x - theta) / delta,
//   x^-L = c_0 / 2 + sum_k c_k T_k(u) + O(tol)          (heat_series)
// and xi~ v = M^-L v takes K sweeps of the recurrence
//   T_0 = v,  T_1 = Mh v,  T_{k+1} = 2 Mh T_k - T_{k-1},   Mh = (M - theta) / delta,
// each one five-point stencil: 325 sweeps for L = 10 and nu = 1 (beta = 9), where
// L successive solves to 1e-13 take 450 and lose more of the tail
// (heat_series_tol).  FP64 throughout.
//
// k_heat_series runs up to kPS sweeps per launch, blocked in time: a block
// holds T_k and T_{k-1} of a kPTileH x kPTileW tile and a halo of kPS cells
// in registers (a wave: one row of 64 cells per register, kPRows rows), and
// the exact region shrinks by one cell per sweep, so that after kPS sweeps
// the tile is still exact.  Left and right neighbours come from the
// neighbouring lanes, the rows above and below from the wave's own registers
// or, at its edge rows, from LDS (double-buffered, one barrier per sweep).
// A cell outside the domain holds zeros in every T_k, so the neighbours'
// weights are the same everywhere and only the diagonal differs by cell.
// 300 x 300 room, one product: 754 us as L solves (60 launches of 11.9 us, eight
// sweeps each through LDS, and 10 of 4.8 us), 260 us as 21 launches of this.
// Bound: launch and load latency (about 4 us of a launch), then FP64 issue:
// 7 FP64 operations and 4 lane moves per cell and sweep, 12 rows per SIMD.
constexpr int kPS = kHeatSweeps;           // sweeps per launch = halo width
constexpr int kPWaves = 16;
constexpr int kPRows = 3;                  // rows per wave
constexpr int kPTileW = 64 - 2 * kPS;      // 32
constexpr int kPTileH = kPWaves * kPRows - 2 * kPS;   // 16
static_assert(kPTileW > 0 && kPTileH > 0, "tile");
constexpr int HEAT_DST_CONT = -1;          // the series goes on in the next launch
constexpr int HEAT_DST_OPERATOR = -2;      // the last launch stores a row of the operator

// The value of the lane to the left (lane - 1) or right (lane + 1); 0 past the ends.
__device__ __forceinline__ double lane_left(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (uint32_t)b, 0x138, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (uint32_t)(b >> 32), 0x138, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double lane_right(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (uint32_t)b, 0x130, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (uint32_t)(b >> 32), 0x130, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

__host__ __device__ __forceinline__ int64_t tile_index(int64_t I, int64_t J, int64_t nT);

// DST: an epilogue code (the last launch of a product), HEAT_DST_CONT or
// HEAT_DST_OPERATOR (the last launch of an operator column; blockIdx.y is the
// column of the batch).
template <int DST>
__global__ void __launch_bounds__(64 * kPWaves)
k_heat_series(HeatSeriesArgs P, HeatGemv G) {
    __shared__ double rowTop[2][kPWaves][64];
    __shared__ double rowBot[2][kPWaves][64];
    const int n0 = P.n0, n1 = P.n1;
    const int tiles_j = (n1 + kPTileW - 1) / kPTileW;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i0 = (int)(blockIdx.x / tiles_j) * kPTileH - kPS + kPRows * wave;   // grid row of this wave's first row
    const int j = (int)(blockIdx.x % tiles_j) * kPTileW - kPS + lane;
    const bool colin = j >= 0 && j < n1;
    const int64_t col = (int64_t)blockIdx.y * P.stride;   // this column's grid vectors
    double T[kPRows], Q[kPRows], y[kPRows], diag[kPRows], f[kPRows];
    // free cells of the wave's rows and of the rows above and below
    bool fr[kPRows + 2];
#pragma unroll
    for (int r = 0; r < kPRows + 2; ++r) {
        const int i = i0 + r - 1;
        fr[r] = colin && i >= 0 && i < n0 && is_free(P.mask, (int64_t)i * n1 + j);
    }
    const bool owncol = lane >= kPS && lane < kPS + kPTileW;
    bool own[kPRows];
#pragma unroll
    for (int r = 0; r < kPRows; ++r) {
        const int i = i0 + r, li = kPRows * wave + r;
        const int g = i * n1 + j;
        const bool c = fr[r + 1];
        own[r] = c && owncol && li >= kPS && li < kPS + kPTileH;
        T[r] = Q[r] = y[r] = 0.0;
        if (c) {
            if (P.first) {
                if (DST == HEAT_DST_OPERATOR || P.unit) T[r] = (P.gidx[P.j0 + blockIdx.y] == g) ? 1.0 : 0.0;
                else {
                    const int32_t x = P.cidx[g];
                    T[r] = x >= 0 ? (double)P.x[x] : 0.0;
                }
                y[r] = P.c0 * T[r];
            } else {
                T[r] = P.Tin[col + g];
                Q[r] = P.Qin[col + g];
                if (own[r]) y[r] = P.Y[col + g];
            }
        }
        f[r] = c ? (P.first ? 0.5 : 1.0) : 0.0;
    }
#pragma unroll
    for (int r = 0; r < kPRows; ++r) {
        // neighbours in the domain, per axis
        const int me = fr[r + 1] ? 1 : 0;
        const int lf = __builtin_amdgcn_update_dpp(0, me, 0x138, 0xf, 0xf, true);
        const int rt = __builtin_amdgcn_update_dpp(0, me, 0x130, 0xf, 0xf, true);
        diag[r] = P.scale * ((1.0 - P.theta) + P.nu0 * (double)((fr[r] ? 1 : 0) + (fr[r + 2] ? 1 : 0)) +
                             P.nu1 * (double)(lf + rt));
    }
    const double w0 = -P.scale * P.nu0, w1 = -P.scale * P.nu1;
    for (int st = 0; st < P.steps; ++st) {
        const int buf = st & 1;
        rowTop[buf][wave][lane] = T[0];
        rowBot[buf][wave][lane] = T[kPRows - 1];
        __syncthreads();
        const double up = wave > 0 ? rowBot[buf][wave - 1][lane] : 0.0;
        const double dn = wave < kPWaves - 1 ? rowTop[buf][wave + 1][lane] : 0.0;
        const double ck = P.c[st];
#pragma unroll
        for (int r = 0; r < kPRows; ++r) {
            const double u = r > 0 ? T[r - 1] : up, d = r < kPRows - 1 ? T[r + 1] : dn;
            double t = diag[r] * T[r];
            t = __builtin_fma(w1, lane_left(T[r]) + lane_right(T[r]), t);
            t = __builtin_fma(w0, u + d, t);
            Q[r] = __builtin_fma(f[r], t, -Q[r]);   // T_{k+1}; swapped with T below
            y[r] = __builtin_fma(ck, Q[r], y[r]);
        }
#pragma unroll
        for (int r = 0; r < kPRows; ++r) {
            const double t = T[r];
            T[r] = Q[r];
            Q[r] = t;
        }
        if (P.first && st == 0)
#pragma unroll
            for (int r = 0; r < kPRows; ++r) f[r] += f[r];
    }
#pragma unroll
    for (int r = 0; r < kPRows; ++r) {
        if (!own[r]) continue;
        const int g = (i0 + r) * n1 + j;
        const int32_t cc = DST == HEAT_DST_CONT ? 0 : P.cidx[g];
        if (cc < 0) continue;
        if constexpr (DST == HEAT_DST_CONT) {
            P.Tout[col + g] = T[r];
            P.Qout[col + g] = Q[r];
            P.Y[col + g] = y[r];
        } else if constexpr (DST == HEAT_DST_OPERATOR) {
            // row j of the operator (xi~ is symmetric: column j), its part in
            // the upper triangle of tiles
            const int64_t row = P.j0 + blockIdx.y;
            const int64_t I = row / kHeatTile, J = cc / kHeatTile;
            if (I <= J)
                P.A[tile_index(I, J, P.nT) * kHeatTileFloats +
                    heat_tile_offset((int)(row - I * kHeatTile), (int)(cc - J * kHeatTile))] = (float)y[r];
        } else {
            heat_epilogue<DST>(G, cc, (float)y[r]);
        }
    }
}

__global__ void k_heat_zero(float* __restrict__ A, int64_t n) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        A[e] = 0.f;
}

// Packed index of the upper-triangular tile (I, J), I <= J, of nT x nT.
__host__ __device__ __forceinline__ int64_t tile_index(int64_t I, int64_t J, int64_t nT) {
    return I * nT - I * (I - 1) / 2 + (J - I);
}

// Free cells in row-major order: each of the 256 threads counts a contiguous
// run of cells, an exclusive scan of the counts gives each run's first free
// index, and the runs are numbered in order.
__global__ void __launch_bounds__(256) k_heat_compact(const uint8_t* __restrict__ mask, int64_t N,
                                                      int32_t* __restrict__ cidx, int32_t* __restrict__ gidx,
                                                      int64_t* __restrict__ count) {
    __shared__ int64_t base[257];
    const int t = threadIdx.x;
    const int64_t per = (N + 255) / 256;
    const int64_t lo = t * per < N ? t * per : N, hi = lo + per < N ? lo + per : N;
    int64_t c = 0;
    for (int64_t i = lo; i < hi; ++i) c += is_free(mask, i) ? 1 : 0;
    base[t + 1] = c;
    __syncthreads();
    if (t == 0) {
        base[0] = 0;
        for (int k = 1; k <= 256; ++k) base[k] += base[k - 1];
        *count = base[256];
    }
    __syncthreads();
    int64_t r = base[t];
    for (int64_t i = lo; i < hi; ++i) {
        if (is_free(mask, i)) {
            cidx[i] = (int32_t)r;
            gidx[r] = (int32_t)i;
            ++r;
        } else {
            cidx[i] = -1;
        }
    }
}

__global__ void k_heat_gather(float* __restrict__ x, const float* __restrict__ src, const int32_t* __restrict__ gidx,
                              int64_t nf, int64_t ld) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < ld; r += (int64_t)gridDim.x * blockDim.x)
        x[r] = r < nf ? src[gidx[r]] : 0.f;
}

// ------------------------------------------------------------------ products

// Tile pass: block b takes the packed tile (I, J), I <= J, and writes
//   part[I][J] = A_IJ x_J             (its row sums, the tile's share of y_I)
//   part[J][I] = A_IJ^T x_I  (I < J)  (its column sums, the share of y_J
//                                      from the transposed lower tile)
// so that every (row block, tile) slot of part is written exactly once.  Wave w
// takes the tile's strips w and w + 4, row by row in turn.  Bound: memory.  The
// operator of a 100 x 100 room stays largely in the last-level cache between
// passes, by plain loads (with the non-temporal hint the room's flow ran 12 %
// slower).  One beyond that cache does not, and the hint (STREAM) saves filling
// it: a product of a 120 x 120 room 117 -> 105 us, 160 x 160 283 -> 253, 200 x 200
// 644 -> 573 (5.6 TB/s); eight waves of a strip each, without it, 117, 296, 692.
// A step runs on the resident kernel (heatres.hip) where the operator suits it;
// this pass serves single products and larger operators.
constexpr int kPassWaves = kHeatWaves / 2;
// 272 MB (a 108 x 108 room) 79 us by plain loads, 82 streamed; 362 MB (116 x 116) 107, 97
constexpr int64_t kCacheBytes = 300000000;

template <bool STREAM>
__global__ void __launch_bounds__(64 * kPassWaves) k_heat_tiles(const float* __restrict__ A,
                                                                const float* __restrict__ x,
                                                                float* __restrict__ part, int nT) {
    constexpr int T = kHeatTile;
    __shared__ float rows[kHeatWaves][T];
    const int b = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, rg = lane >> 2;
    HeatTileRegs a[2];
    const f4* p = reinterpret_cast<const f4*>(A + (int64_t)b * kHeatTileFloats) + wave * 512 + lane;
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f4* q = p + 512 * kPassWaves * h + 64 * k;
            a[h].v[k] = STREAM ? __builtin_nontemporal_load(q) : *q;
        }
    int I = 0, start = 0;
    while (start + (nT - I) <= b) {    // uniform over the block; at most nT steps
        start += nT - I;
        ++I;
    }
    const int J = I + (b - start);
    const f4* xr = reinterpret_cast<const f4*>(x + (int64_t)I * T) + 2 * rg;
    const f4 x0 = xr[0], x1 = xr[1];
    const float xi[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int w = wave + kPassWaves * h;
        const f4 xj = reinterpret_cast<const f4*>(x + (int64_t)J * T)[4 * w + (lane & 3)];
        float rs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        const f4 cs = heat_tile_fma([&](int q) { return a[h].v[q]; }, xj, xi, rs);
        if (I != J) {
            const float v = heat_column_sum(cs);
            if ((lane & 12) == 0) part[((int64_t)J * nT + I) * T + 16 * w + 4 * (lane & 3) + (lane >> 4)] = v;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float v = heat_row_sum(rs[q]);
            if ((lane & 3) == 0) rows[w][8 * rg + q] = v;
        }
    }
    __syncthreads();
    const int t = threadIdx.x;
    if (t < T) {
        float y = rows[0][t];
#pragma unroll
        for (int w = 1; w < kHeatWaves; ++w) y += rows[w][t];
        part[((int64_t)I * nT + J) * T + t] = y;
    }
}

// Finish pass: y_i = the sum of the nT slots of i's row block, split over 8
// slices (slice s takes slots s, s + 8, ...) whose results are added in slice
// order, then the pointwise epilogue of row i.  A block takes 32 consecutive
// cells x 8 slices.
template <int EK>
__global__ void __launch_bounds__(256) k_heat_finish(HeatGemv g) {
    __shared__ float red[8][33];
    const int t = threadIdx.x, c = t & 31, sl = t >> 5;
    const int64_t i = (int64_t)blockIdx.x * 32 + c;
    float y = 0.f;
    if (i < g.N) {
        const int64_t I = i / kHeatTile, il = i - I * kHeatTile;
        const float* __restrict__ p = g.part + I * g.nT * kHeatTile + il;
#pragma unroll 4
        for (int K = sl; K < g.nT; K += 8) y += p[(int64_t)K * kHeatTile];
    }
    red[sl][c] = y;
    __syncthreads();
    if (sl == 0 && i < g.N) {
        float v = red[0][c];
#pragma unroll
        for (int q = 1; q < 8; ++q) v += red[q][c];
        heat_epilogue<EK>(g, i, v);
    }
}

__global__ void k_heat_fill(float* __restrict__ x, float v, int64_t n, int64_t ld) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ld; i += (int64_t)gridDim.x * blockDim.x)
        x[i] = i < n ? v : 0.f;
}

__global__ void __launch_bounds__(1024) k_heat_sums(const double* __restrict__ errrow, int64_t ne,
                                                   const float* __restrict__ p, int64_t np, double* __restrict__ out) {
    __shared__ double sh[16];
    double e = 0.0, m = 0.0, bad = 0.0;
    if (errrow)
#pragma unroll 4
        for (int64_t i = threadIdx.x; i < ne; i += blockDim.x) {
            const double v = errrow[i];
            if (isfinite(v)) e += v;
            else bad += 1.0;
        }
    if (p)
#pragma unroll 4
        for (int64_t i = threadIdx.x; i < np; i += blockDim.x) m += (double)p[i];
    e = block_sum(e, sh);
    if (threadIdx.x == 0) out[0] = e;
    m = block_sum(m, sh);
    if (threadIdx.x == 0) out[1] = m;
    bad = block_sum(bad, sh);
    if (threadIdx.x == 0) out[2] = bad;
}

__global__ void __launch_bounds__(1024) k_heat_input(const float* __restrict__ p, const uint8_t* __restrict__ mask,
                                                    const float* __restrict__ kappa, float kappa_s, int64_t N,
                                                    double* __restrict__ out) {
    __shared__ double sh[16];
    double m = 0.0, cap = 0.0, bad = 0.0;
#pragma unroll 4
    for (int64_t i = threadIdx.x; i < N; i += blockDim.x) {
        const float v = p[i];
        const bool fr = is_free(mask, i);
        if (!(v >= 0.f) || !isfinite(v) || (!fr && v != 0.f)) bad += 1.0;
        else m += (double)v;
        const float k = kappa ? kappa[i] : kappa_s;
        if (!(k >= 0.f)) bad += 1.0;
        else if (fr) cap += (double)k;
    }
    m = block_sum(m, sh);
    if (threadIdx.x == 0) out[0] = m;
    cap = block_sum(cap, sh);
    if (threadIdx.x == 0) out[1] = cap;
    bad = block_sum(bad, sh);
    if (threadIdx.x == 0) out[2] = bad;
}

int grid_for(int64_t n) {
    const int64_t b = (n + 255) / 256;
    return (int)(b < 8192 ? (b > 0 ? b : 1) : 8192);
}

int chunk_log2(int64_t N) {
    int lg = 2;                                   // at least 4 columns
    while (lg < 10 && ((int64_t)1 << lg) < N) ++lg;
    return lg;                                    // at most 1024 columns per chunk
}

// The stencil's weights and the spectrum's end for a domain.
struct Spectrum {
    double nu0, nu1, beta;
    Spectrum(int n0, int n1, double gamma, int L)
        : nu0(n0 > 1 ? gamma * (double)n0 * n0 / L : 0.0), nu1(n1 > 1 ? gamma * (double)n1 * n1 / L : 0.0),
          beta(1.0 + 4.0 * (nu0 + nu1)) {}
};

// The stencil's constants for the launches of the series s.
struct SeriesPlan {
    HeatSeriesArgs a{};
    const HeatSeries& s;
    unsigned tiles = 0;
};
SeriesPlan series_plan(const HeatSeries& s, int n0, int n1, double gamma, int L) {
    SeriesPlan p{HeatSeriesArgs{}, s};
    if (s.c.empty()) return p;
    const auto [nu0, nu1, beta] = Spectrum(n0, n1, gamma, L);
    p.a.n0 = n0;
    p.a.n1 = n1;
    p.a.nu0 = nu0;
    p.a.nu1 = nu1;
    p.a.theta = 0.5 * (beta + 1.0);
    p.a.scale = beta > 1.0 ? 4.0 / (beta - 1.0) : 0.0;   // 2 / delta
    p.a.c0 = 0.5 * p.s.c[0];
    p.tiles = (unsigned)(((n0 + kPTileH - 1) / kPTileH) * ((n1 + kPTileW - 1) / kPTileW));
    return p;
}

// The launches of a series of degree K over `cols` columns; T and Q (T_{k-1})
// alternate between their two buffers (other blocks still read the old ones
// as their halos), the last launch finishes with DST.
template <int DST>
hipError_t run_series(SeriesPlan& p, double* const T[2], double* const Q[2], unsigned cols, const HeatGemv& g,
                      hipStream_t st) {
    const int K = (int)p.s.c.size() - 1;
    if (K < 0) return hipErrorOutOfMemory;   // no series (an operator whose degree could not be run)
    int cur = 0, k = 0;
    do {
        HeatSeriesArgs& a = p.a;
        a.first = k == 0 ? 1 : 0;
        a.steps = std::min(kPS, K - k);
        for (int q = 0; q < a.steps; ++q) a.c[q] = p.s.c[k + 1 + q];
        a.Tin = T[cur];
        a.Qin = Q[cur];
        a.Tout = T[1 - cur];
        a.Qout = Q[1 - cur];
        k += a.steps;
        if (k < K) hipLaunchKernelGGL(k_heat_series<HEAT_DST_CONT>, dim3(p.tiles, cols), dim3(64 * kPWaves), 0, st, a, g);
        else hipLaunchKernelGGL(k_heat_series<DST>, dim3(p.tiles, cols), dim3(64 * kPWaves), 0, st, a, g);
        cur = 1 - cur;
    } while (k < K);
    return hipGetLastError();
}

template <int EK>
hipError_t solve_as(const HeatGemv& g, const HeatSolve& h, hipStream_t st) {
    if (g.N <= 0) return hipSuccess;   // no free cell
    SeriesPlan p = series_plan(h.s, h.n0, h.n1, h.gamma, h.L);
    p.a.mask = h.mask;
    p.a.cidx = h.cidx;
    p.a.x = g.x;
    p.a.Y = h.Y;
    double* T[2] = {h.T0, h.T1};
    double* Q[2] = {h.Q0, h.Q1};
    return run_series<EK>(p, T, Q, 1, g, st);
}

template <int EK>
hipError_t gemv_as(const HeatGemv& g, hipStream_t st) {
    if (g.nT == 0) return hipSuccess;   // no free cell
    const int64_t tiles = (int64_t)g.nT * (g.nT + 1) / 2;
    const dim3 grid((unsigned)tiles), block(64 * kPassWaves);
    if (tiles * (int64_t)(kHeatTileFloats * sizeof(float)) > kCacheBytes)
        hipLaunchKernelGGL(k_heat_tiles<true>, grid, block, 0, st, g.A, g.x, g.part, g.nT);
    else
        hipLaunchKernelGGL(k_heat_tiles<false>, grid, block, 0, st, g.A, g.x, g.part, g.nT);
    hipLaunchKernelGGL(k_heat_finish<EK>, dim3((unsigned)((g.N + 31) / 32)), dim3(256), 0, st, g);
    return hipGetLastError();
}

}  // namespace

// The Chebyshev coefficients of x^-L on [1, beta] (x = theta + delta u), down
// to a tail of tol of the largest value f(1) = 1.  f' = -L f / x gives them
// the three-term recurrence
//   delta (k - 1 + L) c_{k-1} + 2 theta k c_k + delta (k + 1 - L) c_{k+1} = 0,
// of which they are the decaying solution: they are run backwards from a
// degree far in the tail (Miller's algorithm) and scaled so that the series
// is 1 at x = 1, where its terms (-1)^k c_k are all positive.
HeatSeries heat_series(int n0, int n1, double gamma, int L, bool stored) try {
    const double beta = Spectrum(n0, n1, gamma, L).beta, tol = heat_series_tol(L, stored);
    HeatSeries out;
    if (!(beta > 1.0)) {
        out.c = {2.0};   // M is the identity
        return out;
    }
    const double theta = 0.5 * (beta + 1.0), delta = 0.5 * (beta - 1.0);
    const double rho = (sqrt(beta) + 1.0) / (sqrt(beta) - 1.0);   // the terms' final ratio
    constexpr double kMost = (double)(1 << 28);   // far beyond a degree that could be run
    // e^-25 below the cut, where the recurrence's other solution has died out
    const double reach = (25.0 - log(tol)) / log(rho);
    if (!(reach < kMost)) return out;
    int64_t K = (int64_t)reach + 16 + 4 * (int64_t)L;
    std::vector<double> d;   // (-1)^k c_k
    double sum = 0.0;
    for (;;) {
        d.assign((size_t)K + 2, 0.0);
        d[(size_t)K] = 1e-200;
        for (int64_t k = K; k > 0; --k) {
            d[(size_t)k - 1] = (2.0 * theta * (double)k * d[(size_t)k] - delta * (double)(k + 1 - L) * d[(size_t)k + 1]) /
                               (delta * (double)(k - 1 + L));
            if (d[(size_t)k - 1] > 1e150)   // (what is scaled out of range is far below the tail)
                for (int64_t q = k - 1; q <= K; ++q) d[(size_t)q] *= 1e-150;
        }
        sum = 0.5 * d[0];
        for (int64_t k = 1; k <= K; ++k) sum += d[(size_t)k];
        if (d[(size_t)K] <= 1e-10 * tol * sum) break;
        if ((K *= 2) > (int64_t)kMost) return out;
    }
    double tail = 0.0;
    while (K > 0 && tail + d[(size_t)K] <= tol * sum) tail += d[(size_t)K--];
    out.c.resize((size_t)K + 1);
    for (int64_t k = 0; k <= K; ++k) out.c[(size_t)k] = ((k & 1) ? -d[(size_t)k] : d[(size_t)k]) / sum;
    return out;
} catch (const std::bad_alloc&) {
    return HeatSeries{};   // (no exception leaves the C entry points)
}

int64_t heat_build_scratch(int64_t N) { return 4 * N * ((int64_t)1 << chunk_log2(N)); }

hipError_t heat_build_operator(const uint8_t* mask, int n0, int n1, double gamma, int L, const int32_t* cidx,
                               const int32_t* gidx, int64_t nf, float* A, double* scratch, hipStream_t st) {
    const int64_t N = (int64_t)n0 * n1;
    hipLaunchKernelGGL(k_heat_zero, dim3(grid_for(heat_operator_floats(nf))), dim3(256), 0, st, A,
                       heat_operator_floats(nf));
    const HeatSeries s = heat_series(n0, n1, gamma, L, true);
    SeriesPlan p = series_plan(s, n0, n1, gamma, L);
    // columns per chunk: T and Q twice each, and Y
    const int64_t C = std::max<int64_t>(1, 4 * ((int64_t)1 << chunk_log2(N)) / 5);
    p.a.mask = mask;
    p.a.cidx = cidx;
    p.a.gidx = gidx;
    p.a.unit = 1;
    p.a.A = A;
    p.a.nT = heat_ntiles(nf);
    p.a.stride = N;
    p.a.Y = scratch;
    double* T[2] = {scratch + N * C, scratch + 2 * N * C};
    double* Q[2] = {scratch + 3 * N * C, scratch + 4 * N * C};
    for (int64_t j0 = 0; j0 < nf; j0 += C) {
        p.a.j0 = j0;
        const hipError_t e = run_series<HEAT_DST_OPERATOR>(p, T, Q, (unsigned)std::min(C, nf - j0), HeatGemv{}, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_heat_gemv(int ek, const HeatGemv& g, hipStream_t st) {
    switch (ek) {
        case EK_STORE: return gemv_as<EK_STORE>(g, st);
        case EK_BUPDATE: return gemv_as<EK_BUPDATE>(g, st);
        case EK_MONITOR: return gemv_as<EK_MONITOR>(g, st);
        case EK_PROX + JKO_F_ZERO: return gemv_as<EK_PROX + JKO_F_ZERO>(g, st);
        case EK_PROX + JKO_F_CONGESTION: return gemv_as<EK_PROX + JKO_F_CONGESTION>(g, st);
        case EK_PROX + JKO_F_POROUS: return gemv_as<EK_PROX + JKO_F_POROUS>(g, st);
        case EK_PROX + JKO_F_ENTROPY: return gemv_as<EK_PROX + JKO_F_ENTROPY>(g, st);
        case EK_PROX + JKO_F_CONGESTION_BINARY: return gemv_as<EK_PROX + JKO_F_CONGESTION_BINARY>(g, st);
        case EK_PROX + JKO_F_GEN_ENTROPY: return gemv_as<EK_PROX + JKO_F_GEN_ENTROPY>(g, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_heat_solve(int ek, const HeatGemv& g, const HeatSolve& h, hipStream_t st) {
    switch (ek) {
        case EK_STORE: return solve_as<EK_STORE>(g, h, st);
        case EK_BUPDATE: return solve_as<EK_BUPDATE>(g, h, st);
        case EK_MONITOR: return solve_as<EK_MONITOR>(g, h, st);
        case EK_PROX + JKO_F_ZERO: return solve_as<EK_PROX + JKO_F_ZERO>(g, h, st);
        case EK_PROX + JKO_F_CONGESTION: return solve_as<EK_PROX + JKO_F_CONGESTION>(g, h, st);
        case EK_PROX + JKO_F_POROUS: return solve_as<EK_PROX + JKO_F_POROUS>(g, h, st);
        case EK_PROX + JKO_F_ENTROPY: return solve_as<EK_PROX + JKO_F_ENTROPY>(g, h, st);
        case EK_PROX + JKO_F_CONGESTION_BINARY: return solve_as<EK_PROX + JKO_F_CONGESTION_BINARY>(g, h, st);
        case EK_PROX + JKO_F_GEN_ENTROPY: return solve_as<EK_PROX + JKO_F_GEN_ENTROPY>(g, h, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_heat_fill(float* x, float v, int64_t n, int64_t ld, hipStream_t st) {
    hipLaunchKernelGGL(k_heat_fill, dim3(grid_for(ld)), dim3(256), 0, st, x, v, n, ld);
    return hipGetLastError();
}

hipError_t launch_heat_sums(const double* errrow, int64_t ne, const float* p, int64_t np, double* out,
                            hipStream_t st) {
    hipLaunchKernelGGL(k_heat_sums, dim3(1), dim3(1024), 0, st, errrow, ne, p, np, out);
    return hipGetLastError();
}

hipError_t launch_heat_input(const float* p, const uint8_t* mask, const float* kappa, float kappa_s, int64_t N,
                             double* out, hipStream_t st) {
    hipLaunchKernelGGL(k_heat_input, dim3(1), dim3(1024), 0, st, p, mask, kappa, kappa_s, N, out);
    return hipGetLastError();
}

hipError_t launch_heat_compact(const uint8_t* mask, int64_t N, int32_t* cidx, int32_t* gidx, int64_t* count,
                               hipStream_t st) {
    hipLaunchKernelGGL(k_heat_compact, dim3(1), dim3(256), 0, st, mask, N, cidx, gidx, count);
    return hipGetLastError();
}

hipError_t launch_heat_gather(float* x, const float* src, const int32_t* gidx, int64_t nf, int64_t ld,
                              hipStream_t st) {
    hipLaunchKernelGGL(k_heat_gather, dim3(grid_for(ld)), dim3(256), 0, st, x, src, gidx, nf, ld);
    return hipGetLastError();
}

}  // namespace jko
