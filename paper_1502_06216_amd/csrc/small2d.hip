// The resident 2D kernel's one-block form: a whole step's iteration on a small
// grid in a single block, with every field of the iteration in LDS.
//
// On a small grid the resident tile kernel spends its time between blocks: a
// phase of four 16 x 16 tiles (32 x 32) takes 2.5 us, nearly all of it the
// store, flag, poll and halo load of a neighbour's tile.  One block needs only
// barriers.  It computes all tiles itself, with the tile kernel's arithmetic
// (tilefrag.h) and its order of sums: Z = X K1_1^T once for all rows (a
// fragment's elements do not depend on the row tile that reads them), the
// 16- or 32-k chunks of Y^T = Z^T K1_0^T each from zero into LDS, their sum in
// chunk order and the epilogue in the tile kernel's lanes, the FP64 partial
// sums wave by wave and tile by tile.  So the bits are those of the tile
// kernel and of the launch path, as long as every product is finite: that
// kernel has zeros past a tile's halo (along a row past the group of four it
// ends in), the rows here go on to the next tile's cells, and a zero of the
// factor cancels a finite value there, not an infinite one.  A product that isn't finite is therefore reported (kResidentRedo), and the
// step runs again on the tile kernel.  (Zeros in place of what lies past the
// halos, selected as the rows are read: 7 to 15 % of an iteration.)
//
// Bound: MFMA issue plus three barriers and two LDS round trips per
// application, about 0.4 us of latency.  The MFMA work of all tiles falls on
// one CU's four matrix units (32 cycles per 16 x 16 x 4 FP32 product), so the
// form is chosen while that work (small2d_fits) stays below what the tile
// kernel spends on synchronisation.  32 x 32 at band 15, per iteration of two
// applications: 5.35 us on the tile kernel, 1.77 us here (split-BF16: 1.56 us).
#include <algorithm>
#include <type_traits>

#include "control.h"
#include "epilogue.h"
#include "tilefrag.h"

namespace jko {

namespace {

constexpr int kSThr = 1024;
constexpr int kSWaves = kSThr / 64;
constexpr int kSTiles = 16;                  // at most this many 16 x 16 tiles (small2d_fits)
constexpr int kSV = kSTiles * 4 / kSWaves;   // tile-kernel waves each wave stands in for
constexpr int kSMostWork = 1792;             // FP32: tiles x k (see small2d_fits)
constexpr int kSUnits = 4;                   // k-chunks of the second contraction per wave, at most
constexpr int kSRow = 68;                    // padded row of a chunk's 64 lanes

// Band of tile t of an axis of n cells: the halo's start (a multiple of 4), its
// extent and the extent padded to whole k-steps, as in the tile kernel.
struct SBand {
    int lo, L, Lp;
};
__host__ __device__ __forceinline__ SBand band_of(int t, int n, int W, int rnd) {
    const int i0 = 16 * t, a = i0 - W > 0 ? i0 - W : 0, e = i0 + 16 + W < n ? i0 + 16 + W : n;
    SBand b;
    b.lo = a & ~3;
    b.L = e - b.lo;
    b.Lp = (b.L + rnd - 1) / rnd * rnd;
    return b;
}

// The longest padded band of an axis.
__host__ __device__ __forceinline__ int max_extent(int n, int W, int rnd) {
    int m = 0;
    for (int t = 0; t < (n + 15) / 16; ++t) {
        const int e = band_of(t, n, W, rnd).Lp;
        m = e > m ? e : m;
    }
    return m;
}

// LDS layout (floats, 16-byte aligned parts).  Rows are an odd number of
// 16-byte units long, so that 16 rows read at once fall in distinct banks.
struct SLayout {
    int T0, T1, NT;          // tiles per axis, in all
    int SX, SZ;              // rows of X ([16 T0][SX], axis 1 along a row) and Z ([16 T1][SZ], axis 0)
    int SK1, SK0;            // factor rows: FP32 floats, or bfloat16 (hi and lo)
    int nch;                 // k-chunks of the second contraction
    int X, Z, K1, K0, red, total;
};
__host__ __device__ __forceinline__ SLayout layout_small(int n0, int n1, int W0, int W1, bool split) {
    const int rnd = split ? 32 : 16;
    SLayout s{};
    s.T0 = (n0 + 15) / 16;
    s.T1 = (n1 + 15) / 16;
    s.NT = s.T0 * s.T1;
    int e0 = 16 * s.T0, e1 = 16 * s.T1;
    for (int t = 0; t < s.T0; ++t) {
        const SBand b = band_of(t, n0, W0, rnd);
        e0 = b.lo + b.Lp > e0 ? b.lo + b.Lp : e0;
    }
    for (int t = 0; t < s.T1; ++t) {
        const SBand b = band_of(t, n1, W1, rnd);
        e1 = b.lo + b.Lp > e1 ? b.lo + b.Lp : e1;
    }
    const int m0 = max_extent(n0, W0, rnd), m1 = max_extent(n1, W1, rnd);
    auto row = [](int floats) { return ((floats + 3) / 4 | 1) * 4; };
    s.SX = row(e1);
    s.SZ = row(e0);
    s.SK1 = split ? m1 + 8 : row(m1);
    s.SK0 = split ? m0 + 8 : row(m0);
    s.nch = m0 / rnd;
    int o = 0;
    auto take = [&](int floats) {
        const int at = o;
        o += (floats + 3) / 4 * 4;
        return at;
    };
    s.X = take(16 * s.T0 * s.SX);
    s.Z = take(16 * s.T1 * s.SZ);
    s.K1 = take(16 * s.T1 * s.SK1);   // (split: hi and lo halves take the FP32 rows' floats)
    s.K0 = take(16 * s.T0 * s.SK0);
    s.red = take(s.NT * s.nch * 4 * kSRow);
    s.total = o;
    return s;
}

template <int PK, bool SPLIT>
__global__ void __launch_bounds__(kSThr)
small2d(Resident2D R) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ Ctl C;
    __shared__ double wsum[2][kSTiles * 4];                // per tile and wave: a sum, a maximum
    __shared__ double perr[kSTiles], pmass[kSTiles], pla[kSTiles], plb[kSTiles];   // tile partials, by slot
    constexpr int RND = SPLIT ? 32 : 16;
    const Band2D& B = R.B;
    const int n0 = B.n0, n1 = B.n1;
    const SLayout L = layout_small(n0, n1, B.W0, B.W1, SPLIT);
    float* const Xs = lds + L.X;
    float* const Zs = lds + L.Z;
    float* const red = lds + L.red;
    float* const K1f = lds + L.K1;
    float* const K0f = lds + L.K0;
    uint16_t* const K1h = reinterpret_cast<uint16_t*>(K1f);
    uint16_t* const K1l = K1h + 16 * L.T1 * L.SK1;
    uint16_t* const K0h = reinterpret_cast<uint16_t*>(K0f);
    uint16_t* const K0l = K0h + 16 * L.T0 * L.SK0;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int T1 = L.T1, NT = L.NT;

    // zeros around the fields, then the factor bands and the initial a
    for (int i = tid; i < L.K1; i += kSThr) lds[i] = 0.f;
    if (tid == 0) C = *R.ctl;
    if (tid < kSTiles) perr[tid] = pmass[tid] = pla[tid] = plb[tid] = 0.0;
    // (an entry depends on |i - k| alone: one of each, in the partial sums' LDS)
    uint32_t* const tab = reinterpret_cast<uint32_t*>(red);
    for (int u = tid; u < n0 + n1; u += kSThr)
        tab[u] = u < n0 ? gibbs_bits<SPLIT>(u, n0, B.gamma) : gibbs_bits<SPLIT>(u - n0, n1, B.gamma);
    __syncthreads();
    for (int u = tid; u < 16 * T1 * L.SK1; u += kSThr) {
        const int j = u / L.SK1, c = u % L.SK1;
        const SBand b = band_of(j / 16, n1, B.W1, RND);
        const uint32_t v = j < n1 && c < b.L ? tab[n0 + abs(j - b.lo - c)] : 0u;
        if (SPLIT) {
            K1h[u] = (uint16_t)v;
            K1l[u] = (uint16_t)(v >> 16);
        } else {
            K1f[u] = __uint_as_float(v);
        }
    }
    for (int u = tid; u < 16 * L.T0 * L.SK0; u += kSThr) {
        const int i = u / L.SK0, c = u % L.SK0;
        const SBand b = band_of(i / 16, n0, B.W0, RND);
        const uint32_t v = i < n0 && c < b.L ? tab[abs(i - b.lo - c)] : 0u;
        if (SPLIT) {
            K0h[u] = (uint16_t)v;
            K0l[u] = (uint16_t)(v >> 16);
        } else {
            K0f[u] = __uint_as_float(v);
        }
    }

    EpiArgs eb{};
    eb.kind = EpiKind::BUPDATE;
    eb.q = R.q;
    eb.b = R.b;
    EpiArgs ep{};
    ep.kind = EpiKind::PROX;
    ep.a = R.a;
    ep.p_out = R.p_out;
    ep.prox = R.prox;

    // the outputs this thread finishes: for the v-th tile-kernel wave it
    // stands in for, tile vw / 4, that wave's row and column of this lane
    int eidx[kSV], ecnt[kSV], exs[kSV], erd[kSV];
    EpiIn inq[kSV], inp[kSV];
#pragma unroll
    for (int v = 0; v < kSV; ++v) {
        const int vw = wave + kSWaves * v, t = vw >> 2, w = vw & 3;
        const int il = 4 * w + (lane >> 4), jl = lane & 15;
        const int i = 16 * (t / T1) + il, j = 16 * (t % T1) + jl;
        ecnt[v] = (t < NT && i < n0 && j < n1) ? 1 : 0;
        eidx[v] = i * n1 + j;
        exs[v] = i * L.SX + j;
        erd[v] = (t * L.nch * 4 + (jl & 3)) * kSRow + il + 16 * (jl >> 2);
        inq[v] = epi_prefetch<EK_BUPDATE, false, false, 1>(eb, eidx[v], ecnt[v]);
        inp[v] = epi_prefetch<PK, false, false, 1>(ep, eidx[v], ecnt[v]);
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < kSV; ++v)
        if (ecnt[v]) Xs[exs[v]] = R.a[eidx[v]];
    __syncthreads();

    float trace = 0.f;   // NaN once a product of this thread's wasn't finite
    float bold[kSV];   // this thread's b (the scaling the violation is taken with)
#pragma unroll
    for (int v = 0; v < kSV; ++v) bold[v] = 0.f;

    // this wave's fragment of Z (tile `wave`) and its chunks of Y
    const int k8 = (SPLIT ? 8 : 4) * (lane >> 4), lr = lane & 15;
    int zx = 0, zk = 0, zL = 0, zw = 0;
    if (wave < NT) {
        const int f = wave / T1, tj = wave % T1;
        const SBand b = band_of(tj, n1, B.W1, RND);
        zx = (16 * f + lr) * L.SX + b.lo + k8;
        zk = (16 * tj + lr) * L.SK1 + k8;
        zL = b.Lp;
        zw = (16 * tj + lr) * L.SZ + 16 * f + 4 * (lane >> 4);
    }
    int yz[kSUnits], yk[kSUnits], yr[kSUnits];
    bool yin[kSUnits], yany[kSUnits];   // the chunk exists; it lies within the band
#pragma unroll
    for (int m = 0; m < kSUnits; ++m) {
        const int u = wave + kSWaves * m;
        yany[m] = u < NT * L.nch;
        const int t = yany[m] ? u / L.nch : 0, c0 = yany[m] ? RND * (u % L.nch) : 0, ti = t / T1, tj = t % T1;
        const SBand b = band_of(ti, n0, B.W0, RND);
        yin[m] = yany[m] && c0 < b.Lp;
        yz[m] = (16 * tj + lr) * L.SZ + b.lo + c0 + k8;
        yk[m] = (16 * ti + lr) * L.SK0 + c0 + k8;
        yr[m] = u * 4 * kSRow + lane;
    }
    const int nch = L.nch;

    // One application of xi to the field in Xs with its epilogue, whose a or b
    // replaces the field.
    using yes = std::true_type;
    using no = std::false_type;
    auto phase = [&](auto ek, auto chkc, EpiArgs& E, const EpiIn (&in)[kSV]) {
        constexpr int EKv = decltype(ek)::value;
        constexpr bool CHK = decltype(chkc)::value;
        E.check = CHK ? 1 : 0;
        if (EKv >= EK_PROX) E.write_p = CHK ? 1 : 0;
        if (wave < NT)
            *reinterpret_cast<f4*>(&Zs[zw]) = z_frag<SPLIT>(&Xs[zx], K1f + (SPLIT ? 0 : zk), K1h + (SPLIT ? zk : 0),
                                                            K1l + (SPLIT ? zk : 0), zL);
        __syncthreads();
#pragma unroll
        for (int m = 0; m < kSUnits; ++m) {
            if (!yany[m]) break;   // (uniform over the wave)
            f4 acc = f4{0.f, 0.f, 0.f, 0.f};
            if (yin[m])
                acc = y_chunk<SPLIT>(&Zs[yz[m]], K0f + (SPLIT ? 0 : yk[m]), K0h + (SPLIT ? yk[m] : 0),
                                     K0l + (SPLIT ? yk[m] : 0), acc);
#pragma unroll
            for (int e = 0; e < 4; ++e) red[yr[m] + e * kSRow] = acc[e];
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < kSV; ++v) {
            const int vw = wave + kSWaves * v;
            if (vw >= 4 * NT) break;   // (uniform over the wave)
            EpiAcc ea;
            if (ecnt[v]) {
                // the chunks' sums in order (the first four read at once; an
                // absent chunk is an exact zero)
                float c[4];
#pragma unroll
                for (int w = 0; w < 4; ++w) c[w] = w < nch ? red[erd[v] + w * 4 * kSRow] : 0.f;
                float y = ((c[0] + c[1]) + c[2]) + c[3];
                for (int w = 4; w < nch; ++w) y += red[erd[v] + w * 4 * kSRow];
                trace = __builtin_fmaf(y, 0.f, trace);
                float out;
                epi_apply<EKv, false, 1, true>(E, eidx[v], 1, f4{y, 0.f, 0.f, 0.f}, false, in[v], ea, &out);
                Xs[exs[v]] = out;
                if (EKv == EK_BUPDATE) bold[v] = out;
            }
            if (CHK) {   // the tile kernel's wave sums (block_sum and block_max)
                double s = EKv == EK_BUPDATE ? ea.err : ea.mass, m = EKv == EK_BUPDATE ? ea.maxlb : ea.maxla;
                for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
                for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
                if (lane == 0) {
                    wsum[0][vw] = s;
                    wsum[1][vw] = m;
                }
            }
        }
        __syncthreads();
        if (CHK) {
            if (tid < NT) {
                double s = 0.0, m = 0.0;
                for (int w = 0; w < 4; ++w) {
                    s += wsum[0][4 * tid + w];
                    m = fmax(m, wsum[1][4 * tid + w]);
                }
                // the slot of the tile's block in the tile kernel's grid
                const int slot = NT % 8 != 0 ? tid : (tid % (NT / 8)) * 8 + tid / (NT / 8);
                if (EKv == EK_BUPDATE) {
                    perr[slot] = s;
                    plb[slot] = m;
                } else {
                    pmass[slot] = s;
                    pla[slot] = m;
                    R.part.mass[slot] = s;       // the closing monitor's check reads them
                    R.part.maxloga[slot] = m;
                }
            }
            __syncthreads();
        }
    };
    const std::integral_constant<int, EK_BUPDATE> ekb;
    const std::integral_constant<int, PK> ekp;
    // where the launch ends: the report, and the scalings to memory
    auto report = [&]() {
        if (trace != 0.f) *R.sync = kResidentRedo;
    };
    auto keep = [&]() {
        report();
#pragma unroll
        for (int v = 0; v < kSV; ++v)
            if (ecnt[v]) {
                R.a[eidx[v]] = Xs[exs[v]];
                R.b[eidx[v]] = bold[v];
            }
    };

    bool due = false;   // the iteration before this one was a candidate: check it now
    for (int k = 1, since = 0; k <= R.K; ++k) {
        // ---- t = xi^T a, b = q / t (and the violation of the previous iterate at checks)
        const bool chk = due;
        due = R.checks && ++since == R.ce;
        if (due) since = 0;
        eb.t_out = R.hist ? R.hist + (2 * (int64_t)(k - 1)) * R.hist_stride : nullptr;
        bool switching = false;
        if (chk) {
            EpiIn ia[kSV];
#pragma unroll
            for (int v = 0; v < kSV; ++v) {
                ia[v] = inq[v];
                ia[v].v[0] = bold[v];
            }
            phase(ekb, yes(), eb, ia);
            if (wave == 0) {
                Partials p{perr, pmass, pla, plb, NT};
                ctl_update<false>(&C, p, NT, k, R.tol, 1, R.absorb, R.a_only);
            }
            __syncthreads();
            if (tid == 0) {
                Ctl* g = R.ctl;
                g->done = C.done;
                g->stop_iter = C.stop_iter;
                g->nonfinite = C.nonfinite;
                g->absorptions = C.absorptions;
                g->absorb_pending = C.absorb_pending;
                g->logmode = C.logmode;
                g->exit_iter = C.absorb_pending ? k : 0;
                g->err = C.err;
                g->mass = C.mass;
                g->maxloga = C.maxloga;
                g->maxlogb = C.maxlogb;
            }
            if (C.done) {   // (the step returns the p of the last candidate)
                report();
                return;
            }
            switching = C.absorb_pending != 0;
        } else {
            phase(ekb, no(), eb, inq);
        }
        // ---- s = xi b, p = prox(s), a = p / s (p kept at candidate iterations)
        const bool cand = due || k == R.K;
        ep.s_out = R.hist ? R.hist + (2 * (int64_t)(k - 1) + 1) * R.hist_stride : nullptr;
        if (cand) phase(ekp, yes(), ep, inp);
        else phase(ekp, no(), ep, inp);
        if (switching) break;   // the rest of the step runs on the log-domain passes
    }
    keep();
}

template <bool SPLIT>
const void* small_kernel_of(int kind) {
    switch (kind) {
        case JKO_F_ZERO: return reinterpret_cast<const void*>(&small2d<EK_PROX + JKO_F_ZERO, SPLIT>);
        case JKO_F_CONGESTION: return reinterpret_cast<const void*>(&small2d<EK_PROX + JKO_F_CONGESTION, SPLIT>);
        case JKO_F_CONGESTION_BINARY:
            return reinterpret_cast<const void*>(&small2d<EK_PROX + JKO_F_CONGESTION_BINARY, SPLIT>);
        case JKO_F_GEN_ENTROPY: return reinterpret_cast<const void*>(&small2d<EK_PROX + JKO_F_GEN_ENTROPY, SPLIT>);
        case JKO_F_POROUS: return reinterpret_cast<const void*>(&small2d<EK_PROX + JKO_F_POROUS, SPLIT>);
        default: return reinterpret_cast<const void*>(&small2d<EK_PROX + JKO_F_ENTROPY, SPLIT>);
    }
}

}  // namespace

bool small2d_fits(int n0, int n1, int W0, int W1, bool split, int kind, int ce) {
    // The epilogues of all tiles and the sums of a check fall on one CU as well,
    // where the tile kernel spreads them.  Where the lines lie, us of 50
    // iterations, this form against the tile kernel, the generalised entropy's
    // Newton steps or the crowd's one, band 5 cells wide:
    //   Newton: 7 tiles 16 x 112 FP32 437 / 409, split 410 / 428, 100 cells on a
    //     line FP32 398 / 454; 8 tiles 32 x 64 FP32 469 / 395, split 424 / 399; 12
    //     tiles 180 cells FP32 639 / 469; 16 tiles 64 x 64 split 754 / 413
    //   no checks: 64 x 64 split 310 / 360
    //   a check every 3 iterations: 10 tiles 16 x 160 FP32 412 / 432, split 358 /
    //     448; 12 tiles 48 x 64 FP32 454 / 415; every iteration split 648 / 610
    //   every 4: 48 x 64 FP32 421 / 406, split 353 / 403; 64 x 64 split 426 / 399
    //   every 10: 64 x 64 split 349 / 375
    const bool newton = kind == JKO_F_POROUS || kind == JKO_F_GEN_ENTROPY;
    const int most = newton ? 7 : ce == 0 ? kSTiles : ce < 4 || !split ? 10 : ce < 10 ? 12 : kSTiles;
    if ((int64_t)((n0 + 15) / 16) * ((n1 + 15) / 16) > most) return false;
    const SLayout L = layout_small(n0, n1, W0, W1, split);
    if (L.NT * L.nch > kSUnits * kSWaves || L.total * (int64_t)sizeof(float) > 144 * 1024) return false;
    // FP32: the tiles' k-steps, NT (Lp0 + Lp1) / 4 products of 32 cycles over
    // four matrix units.  64 x 48 at band 42, 1344: 5.2 / 5.9.
    return split || L.NT * (16 * L.nch + max_extent(n1, W1, 16)) <= kSMostWork;
}

hipError_t launch_small2d(const Resident2D& r, hipStream_t stream) {
    const SLayout L = layout_small(r.B.n0, r.B.n1, r.B.W0, r.B.W1, r.split != 0);
    Resident2D arg = r;
    void* args[] = {&arg};
    return hipLaunchKernel(r.split ? small_kernel_of<true>(r.prox.kind) : small_kernel_of<false>(r.prox.kind), dim3(1),
                           dim3(kSThr), args, (size_t)L.total * sizeof(float), stream);
}

}  // namespace jko
