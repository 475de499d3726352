// Heat-kernel Gibbs operator on a masked 2D grid (Section 4.1, eq. heat-kernel):
// host-side launchers of the kernels in heat.hip.
//
// xi~ = (Id - (gamma/L) Delta_M)^{-L} with Delta_M the no-flux five-point
// Laplacian of the free cells (spacing 1/n_k along axis k), i.e.
// Id + nu_0 G_0 + nu_1 G_1 with nu_k = gamma n_k^2 / L and G_k the graph
// Laplacian of the free axis-k neighbour pairs.  The operator acts on the
// free cells only: they are numbered in row-major order (gidx: free index ->
// grid cell, cidx: grid cell -> free index or -1), and xi~ is stored over
// those Nf indices.  xi~ is symmetric; the library stores its upper triangle
// of kHeatTile x kHeatTile float32 tiles: tile (I, J), I <= J, of the ld x ld
// matrix (ld = Nf rounded up to the tile) at
// packed index I*nT - I*(I-1)/2 + (J - I), each tile in the order of
// heat_tile_offset (heat_tile.h).  Rows and
// columns of the padding are zero.
#pragma once

#include <math.h>

#include <vector>

#include "jko_internal.h"

namespace jko {

constexpr int kHeatTile = 128;

inline int64_t heat_ld(int64_t N) { return (N + kHeatTile - 1) / kHeatTile * kHeatTile; }
inline int64_t heat_ntiles(int64_t N) { return heat_ld(N) / kHeatTile; }
// floats of the packed upper-triangular tiles
inline int64_t heat_operator_floats(int64_t N) {
    const int64_t nT = heat_ntiles(N);
    return nT * (nT + 1) / 2 * kHeatTile * kHeatTile;
}
// floats of the per-pass partial sums (one row block per tile pair)
inline int64_t heat_partial_floats(int64_t N) {
    const int64_t nT = heat_ntiles(N);
    return nT * nT * kHeatTile;
}

// One application of the stored operator, y = A x, with the result of each
// row finished by a pointwise epilogue (EK_STORE, EK_BUPDATE, EK_MONITOR or
// EK_PROX + energy kind, as in the band contractions).
// Row r of the pass is free cell gidx[r]: x, b, a and errrow are indexed by
// r (free-cell vectors), y, q, p and the energy fields by the grid cell.
struct HeatGemv {
    const float* A;          // packed upper-triangular tiles
    float* part;             // heat_partial_floats(N) scratch
    int32_t nT;              // tiles per side
    int64_t ld;              // nT * kHeatTile
    int64_t N;               // rows: free cells
    const int32_t* gidx;     // free index -> grid cell
    const float* x;          // ld floats, padding zero
    float* y;                // STORE: result (grid)
    const float* q;          // BUPDATE / MONITOR: the step's input density (grid)
    float* b;                // BUPDATE: b = q / y (0/0 = 0); MONITOR: read
    double* errrow;          // BUPDATE (when check) / MONITOR: |b_old y - q| per row
    int32_t check;
    float* a;                // PROX: a = p / y (0/0 = 0)
    float* p;                // PROX: p = Prox(y) (grid)
    ProxArgs px;             // fields indexed by grid cell
};

// Numbers the free cells in row-major order: cidx (N), gidx (first Nf
// entries), *count (device int64) = Nf.  One block.
hipError_t launch_heat_compact(const uint8_t* mask, int64_t N, int32_t* cidx, int32_t* gidx, int64_t* count,
                               hipStream_t st);

// x[r] = src[gidx[r]] for r < nf, 0 up to ld.
hipError_t launch_heat_gather(float* x, const float* src, const int32_t* gidx, int64_t nf, int64_t ld,
                              hipStream_t st);

// x^-L on the spectrum [1, beta] of a domain's operator as a Chebyshev series:
// x^-L = c_0 / 2 + sum_k c_k T_k(u), x = theta + delta u, theta = (beta + 1) / 2,
// delta = (beta - 1) / 2, cut where heat_series_tol says; for the columns of the
// stored operator, or for products.  Empty: it has too many terms to be run, or
// for the host's memory.
struct HeatSeries {
    std::vector<double> c;
};
HeatSeries heat_series(int n0, int n1, double gamma, int L, bool stored);

// Where the series is cut.  The cut is absolute, a fraction of the input's
// norm, and the iteration divides by a product (b = q / t), so entries far
// below the norm count as much as any: a series of degree K is exactly zero
// beyond K cells of a point source and wrong some way before, while above its
// cut its entries keep 13 digits (the sweeps, like the entries, spread one cell
// at a time, and so do their rounding errors).
//   - The operator is stored in float32: what lies below float32's smallest
//     value is no entry.
//   - A product's input may span float32's range as well: cut so that what is
//     dropped lies below float32's smallest value for the largest input.
// Small L: L solves, each to 1e-13 of its own right-hand side, lose an entry of
// 1e-14 (20 % off) at L = 1, of 1e-24 (60 %) at L = 3, and are 6 % off there at
// L = 10.  21 decades for each of the L keep more than that everywhere, in no
// more time: at nu = 1 a product of a 1000 x 1000 grid takes 70, 145, 221, 325
// sweeps for L = 1, 2, 3, 10, L solves took 45, 90, 135, 450.
inline double heat_series_tol(int L, bool stored) {
    const int decades = stored ? 46 : 85;
    return pow(10.0, -(double)(21 * (int64_t)L < decades ? 21 * L : decades));
}

// One product y = xi~ x on the grid, nothing stored: x is g's free-cell vector
// and each free row is finished by the epilogue `ek` of g (codes of
// launch_heat_gemv).  T0, T1, Q0, Q1, Y: grid scratch (N doubles each).
struct HeatSolve {
    const uint8_t* mask;     // NULL = no obstacle
    const int32_t* cidx;     // grid cell -> free index or -1
    int n0, n1, L;
    double gamma;
    HeatSeries s;            // the same for all products of a call
    double* T0;
    double* T1;
    double* Q0;
    double* Q1;
    double* Y;
};
hipError_t launch_heat_solve(int ek, const HeatGemv& g, const HeatSolve& h, hipStream_t st);

// Sweeps of the series per launch.
constexpr int kHeatSweeps = 16;

// One launch of the series (kernel argument).
struct HeatSeriesArgs {
    int n0, n1;
    double nu0, nu1, theta;
    double scale;            // 2 / delta
    double c0;               // c_0 / 2
    double c[kHeatSweeps];   // the coefficients of this launch's sweeps
    int steps;
    int first;               // the start: T_0 from x, or from the unit column
    int unit;                // columns of the operator: the vector of blockIdx.y is e_(j0 + blockIdx.y)
    const uint8_t* mask;
    const int32_t* cidx;
    const int32_t* gidx;
    const float* x;
    const double* Tin;
    const double* Qin;
    double* Tout;
    double* Qout;
    double* Y;
    int64_t stride;          // doubles between the grid vectors of two columns
    int64_t j0;              // first column of the batch
    float* A;                // the packed operator and its tiles per side
    int64_t nT;
};

// Scratch doubles heat_build_operator needs for an N-cell grid (4 N C).
int64_t heat_build_scratch(int64_t N);

// Writes the packed tiles of xi~ over the nf free cells (heat_operator_floats(nf)
// floats).  scratch: heat_build_scratch(N) doubles.
hipError_t heat_build_operator(const uint8_t* mask, int n0, int n1, double gamma, int L, const int32_t* cidx,
                               const int32_t* gidx, int64_t nf, float* A, double* scratch, hipStream_t st);

// Epilogue codes of launch_heat_gemv: store, b-update, monitor, and the
// proximal epilogue HEAT_EK_PROX + energy kind (the band contractions' codes).
enum : int { HEAT_EK_STORE = 0, HEAT_EK_BUPDATE = 1, HEAT_EK_MONITOR = 2, HEAT_EK_PROX = 3 };

hipError_t launch_heat_gemv(int ek, const HeatGemv& g, hipStream_t st);

// The products of a step's iteration with the stored operator in one cooperative
// launch (heatres.hip): product 2 (k - 1) is t = A a with the b-update of
// iteration k (record t), product 2 (k - 1) + 1 is s = A b with the proximal
// update (record s, whose p is written where the step may end).
struct HeatResident {
    HeatGemv t, s;
    int32_t last;            // products
    int32_t period;          // a check with every t = A a at a multiple of this (> 0) product; 0: none
    double tol;              // the step ends at a check whose violation is at most this, or not finite
    int32_t spin_limit;      // polls before a wait gives up
    uint32_t* sync;          // heat_resident_sync_words() words, zeroed before the launch; [0] != 0
                             // afterwards: a wait ran out; a HeatOutcome at [kHeatOutcome]
};
constexpr int kHeatOutcome = 2;
struct HeatOutcome {         // of the last check
    int32_t prod;            // its product (0: there was none)
    int32_t bad;             // entries that weren't finite
    double err;              // the sum of the others
};
int64_t heat_resident_sync_words();
bool heat_resident_fits(int nT, int kind, bool check);   // check: with a stop test (period > 0)
hipError_t launch_heat_resident(const HeatResident& r, int kind, hipStream_t st);

// x[0..n) = v, x[n..ld) = 0
hipError_t launch_heat_fill(float* x, float v, int64_t n, int64_t ld, hipStream_t st);


// out[0] = sum of errrow[0..ne) (when errrow != NULL), out[1] = sum of
// p[0..np) (when p != NULL), out[2] = number of non-finite errrow entries.
// One block, fixed order.
hipError_t launch_heat_sums(const double* errrow, int64_t ne, const float* p, int64_t np, double* out,
                            hipStream_t st);

// Input check of a step's density: out[0] = mass, out[1] = capacity over the
// free cells (kappa field or kappa_s; +inf allowed), out[2] = number of
// cells that are negative or non-finite, hold mass on an obstacle, or have a
// negative/NaN capacity.
hipError_t launch_heat_input(const float* p, const uint8_t* mask, const float* kappa, float kappa_s, int64_t N,
                             double* out, hipStream_t st);

}  // namespace jko
