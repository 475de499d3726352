// The resident heat kernel: the products of a JKO step with the stored
// operator (heat.hip) in one cooperative launch, with the operator on chip.
//
// A pass over the packed operator moves all of it (187 MB for a 100 x 100 room)
// through the memory side, 27.6 us of a product's 32 us, and every product
// needs two launches.  The register files and LDS of 256 CUs hold 100 MB of it:
// block c owns a contiguous range of packed tiles, keeps up to kRegTiles of
// them in registers and kLdsTiles in LDS for the whole launch, and streams only
// the rest, each streamed tile loaded while kept ones are multiplied.  (A fifth
// tile in registers makes the compiler spill 40 of them: 49 us an iteration of
// the 100 x 100 room where four take 39.)
//
// A product y = A x in two phases, each ended by a wait for all blocks:
//   tiles:   every block multiplies its tiles, A_IJ x_J and (off the diagonal)
//            A_IJ^T x_I, and stores the 128-cell shares to the slots (I, J) and
//            (J, I) of `part`; consecutive tiles of one row block I add their
//            row sums in registers and fill the first one's slot, the others'
//            hold zeros from the launch's start;
//   finish:  every block sums the slots of its share of the cells in a fixed
//            order and runs the epilogue of the half-step.
// Values that cross blocks (part, a, b) are stored and loaded at device scope,
// and a block counts its phase once its stores have completed; no
// block starts a phase before all have finished the one before, so nothing is
// overwritten that another still reads.
//
// Stop test: the finish of a check's t = A a stores the cells' violations, block
// 0 sums them once it has seen every block finish, and the word that lets the
// others go on tells them to stop.  64 x 64, 60 iterations with a check after
// each: 1180 us; with a launch up to each check, which loaded the kept tiles again
// and had the host wait twice, 4200; two launches per product 2530.
//
// Bound: streaming of the tiles that are not kept, 4.7 TB/s over a whole step of
// the 100 x 100 room (by plain loads; with the non-temporal hint an iteration took
// 44 us), then the two waits of a product.  An iteration of two products:
// 100 x 100 room 63.4 -> 39.5 us (86 MB of 187 MB streamed), 80 x 80 (all kept)
// 16.1 us, 64 x 64 13.8 us.
#include <algorithm>

#include "epilogue.h"
#include "heat_tile.h"

namespace jko {

namespace {

constexpr int kRegTiles = 4;
constexpr int kLdsTiles = 2;
constexpr int kKept = kRegTiles + kLdsTiles;
constexpr int kMaxTiles = 16;    // tiles of one block
constexpr int kMaxBlocks = 256;
constexpr int kSlotBytes = 4 * kHeatTile;
constexpr int kSlots = 12;       // slots of a cell per wave: nT <= 90 with at most 16 x 256 tiles
// Sync words: [0] abort, the outcome of the last check from kHeatOutcome; the
// blocks' phase counts from kFlag0, packed; from kGo the number of phases all
// blocks have finished, with kStop set where the step ends there, in kGoCopies
// lines.  Block 0
// alone reads the counts and writes the copies, each polled by a sixteenth of
// the blocks: with every block polling every count, or one atomic counter, 256
// requests at a time queue for the same line (6 us a wait; an iteration of the
// 64 x 64 room took 30 and 35 us, and takes 14 us so).
constexpr int kFlag0 = 64;
constexpr int kGo = kFlag0 + kMaxBlocks;
constexpr int kGoCopies = 16;
constexpr int kGoStride = 64;
constexpr uint32_t kStop = 1u << 31;

__device__ __forceinline__ bool poll(const uint32_t* word, uint32_t count, uint32_t* sync, int spin_limit) {
    for (int spins = 0; __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < count; ++spins) {
        if ((spins & 31) == 31 && __hip_atomic_load(sync, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return false;
        if (spins >= spin_limit) {
            __hip_atomic_store(sync, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    return true;
}

// All stores of this block completed, then its count.
__device__ __forceinline__ void publish_phase(uint32_t* sync, int slot, uint32_t count) {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_store(sync + kFlag0 + slot, count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Every block has finished `count` phases (bounded; the abort word is watched).
// CHECK: block 0 decides between the two whether the step ends here (decide(),
// the same in every thread).  Returns whether to go on.
template <bool CHECK, typename Decide>
__device__ __forceinline__ bool wait_all(uint32_t* sync, int slot, int nb, uint32_t count, int spin_limit,
                                         uint32_t* failed, Decide decide) {
    const int t = threadIdx.x;
    if (slot == 0) {
        if (t < nb && !poll(sync + kFlag0 + t, count, sync, spin_limit)) *failed = 1;
        __syncthreads();
        if (*failed != 0) return false;
        const bool stop = CHECK && decide();
        if (t < kGoCopies)
            __hip_atomic_store(sync + kGo + kGoStride * t, count | (stop ? kStop : 0u), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        return !stop;
    }
    if (t == 0) {
        const uint32_t* go = sync + kGo + kGoStride * (slot % kGoCopies);
        // (the word is read again where it may tell to stop: the poll keeps the shorter loop)
        if (!poll(go, count, sync, spin_limit) ||
            (CHECK && (__hip_atomic_load(go, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kStop)))
            *failed = 1;
    }
    __syncthreads();
    return *failed == 0;
}

// Device-scope loads and stores at a lane offset and a scalar offset (bytes).
constexpr int kCoh = 16;
__device__ __forceinline__ float coh_load(__amdgpu_buffer_rsrc_t rs, int voff, int soff) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, voff, soff, kCoh));
}
__device__ __forceinline__ void coh_store(__amdgpu_buffer_rsrc_t rs, int voff, int soff, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rs, voff, soff, kCoh);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const float* p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), (short)0, bytes, 0x00020000);
}

// A tile by buffer loads (one offset register; the tile's place is scalar).  The
// operators taken here are below 2^31 bytes (heat_resident_fits).
__device__ __forceinline__ void load_tile(HeatTileRegs& t, __amdgpu_buffer_rsrc_t rs, int tile, int voff) {
#pragma unroll
    for (int k = 0; k < 8; ++k)
        t.v[k] = __builtin_bit_cast(
            f4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff, tile * (4 * kHeatTileFloats) + 1024 * k, 0));
}

// A value that is the same in every lane, in a scalar register.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// CHECK: with a stop test (R.period > 0); its code alone costs a step without one
// 1 to 3 %.
template <int KIND, bool CHECK>
__global__ void __launch_bounds__(kHeatThr)
heat_resident(HeatResident R) {
    extern __shared__ __attribute__((aligned(16))) float kept[];   // kLdsTiles operator tiles
    __shared__ __attribute__((aligned(16))) float xcol[2 * kMaxTiles][kHeatTile];   // x of the m tiles' columns, then rows
    __shared__ float rows[kHeatWaves][kHeatTile];                               // a run's row sums by wave
    __shared__ float red[kHeatWaves][64];
    __shared__ uint32_t failed;
    __shared__ double shd[kHeatWaves];
    __shared__ uint32_t word;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = (int)gridDim.x, slot = (int)blockIdx.x;
    const HeatGemv& G = R.t;
    const int nT = G.nT;
    const int64_t T = (int64_t)nT * (nT + 1) / 2;
    const int b0 = uniform((int)(T * slot / nb));
    const int m = uniform((int)(T * (slot + 1) / nb)) - b0;   // tiles of this block, <= kMaxTiles
    if (tid == 0) failed = 0;
    int I0 = 0, J0 = 0;   // the first tile's place
    {
        int start = 0;
        while (start + (nT - I0) <= b0) {   // (at most nT steps)
            start += nT - I0;
            ++I0;
        }
        J0 = I0 + (b0 - start);
    }
    I0 = uniform(I0);
    J0 = uniform(J0);
    // this thread's 16-byte shares of x: tile k's columns at k, its rows at m + k
    int xoff[(2 * kMaxTiles * kHeatTile / 4 + kHeatThr - 1) / kHeatThr];
#pragma unroll
    for (int v = 0; v < (int)(sizeof xoff / sizeof xoff[0]); ++v) {
        const int u = tid + v * kHeatThr, k2 = u / (kHeatTile / 4), c = u % (kHeatTile / 4);
        int I = I0, J = J0;
        for (int k = 0; k < (k2 < m ? k2 : k2 - m); ++k)
            if (++J == nT) J = ++I;
        xoff[v] = k2 < 2 * m ? 4 * kHeatTile * (k2 < m ? J : I) + 16 * c : 0;
    }

    // the kept tiles.  All tiles are taken in order, so that runs stay
    // together, the ns streamed ones spread between the nk kept ones: kept
    // tile j has ns j / nk of them before it.
    const int nk = min(m, kKept), ns = m - nk;
    const int voff = 16 * (64 * 8 * wave + lane);
    const __amdgpu_buffer_rsrc_t rs_A = rsrc_of(G.A, (int)(T * (4 * kHeatTileFloats)));
    const __amdgpu_buffer_rsrc_t rs_part = rsrc_of(G.part, nT * nT * kSlotBytes);
    auto kept_at = [&](int j) { return j + uniform(ns * j / nk); };   // (nk > 0 where used)
    auto streamed_at = [&](int s) { return s + uniform(((s + 1) * nk + ns - 1) / ns); };   // (s < ns)
    HeatTileRegs reg[kRegTiles], str;
#pragma unroll
    for (int j = 0; j < kRegTiles; ++j)
        if (j < nk) load_tile(reg[j], rs_A, b0 + kept_at(j), voff);
    for (int j = kRegTiles; j < nk; ++j) {
        load_tile(str, rs_A, b0 + kept_at(j), voff);
        f4* p = reinterpret_cast<f4*>(kept + (j - kRegTiles) * kHeatTileFloats) + wave * 512 + lane;
#pragma unroll
        for (int q = 0; q < 8; ++q) p[64 * q] = str.v[q];
    }
    for (int k = 0, I = I0, J = J0; k < m; ++k) {
        if (k > 0 && J > I && tid < kHeatTile) coh_store(rs_part, 4 * tid, (I * nT + J) * kSlotBytes, 0.f);
        if (++J == nT) J = ++I;
    }
    const int s0 = ns > 0 ? streamed_at(0) : 0;

    // the cells this block finishes, one per lane (at most 64: heat_resident_fits),
    // and what wave 0 needs of them
    const int c0 = (int)(G.N * slot / nb), cn = (int)(G.N * (slot + 1) / nb) - c0;
    const bool mine = lane < cn;
    const int cell = mine ? c0 + lane : 0;
    const int slots = cell / kHeatTile * (nT * kSlotBytes) + 4 * (cell % kHeatTile);
    int gi = 0;
    float q = 0.f, pu = 1.f, pv = 0.f, bold = 0.f;
    if (wave == 0 && mine) {
        gi = G.gidx[cell];
        q = G.q[gi];
        heat_prox_fields<KIND>(R.s.px, gi, pu, pv);
        bold = G.b[cell];
    }
    uint32_t count = 0;
    const int rg = lane >> 2, coff = 4 * (16 * wave + 4 * (lane & 3) + (lane >> 4));

    auto no_decision = []() { return false; };
    // Block 0, after product `prod`: the violation of the iterate before it, in a
    // fixed order; the step ends where it is small enough, or not finite.
    auto outcome = [&](int prod) {
        double e = 0.0, bad = 0.0;
        for (int64_t i = tid; i < G.N; i += kHeatThr) {
            const double v = __hip_atomic_load(G.errrow + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (isfinite(v)) e += v;
            else bad += 1.0;
        }
        e = block_sum(e, shd);
        bad = block_sum(bad, shd);
        if (tid == 0) {   // (every thread's sums are wave 0's: block_sum)
            HeatOutcome* o = reinterpret_cast<HeatOutcome*>(R.sync + kHeatOutcome);
            o->prod = prod;
            o->bad = bad > 0.0 ? 1 : 0;
            o->err = e;
            word = bad > 0.0 || e <= R.tol ? 1u : 0u;
        }
        __syncthreads();
        return word != 0u;
    };

    int to_check = R.period;   // products up to the next check
    for (int prod = 0; prod < R.last; ++prod) {
        const bool bstep = (prod & 1) == 0;   // t = A a, b = q / t; else s = A b, p = Prox(s), a = p / s
        const bool chk = CHECK && to_check == 0;
        if (chk) to_check = R.period;
        if (CHECK) --to_check;
        const float* x = bstep ? R.t.x : R.s.x;
        // ---- tiles
        f4 xv[(2 * kMaxTiles * kHeatTile / 4 + kHeatThr - 1) / kHeatThr];
        {
            const __amdgpu_buffer_rsrc_t rs_x = rsrc_of(x, nT * kSlotBytes);
#pragma unroll
            for (int v = 0; v < (int)(sizeof xv / sizeof xv[0]); ++v)
                xv[v] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, xoff[v], 0, kCoh));
        }
        int sn = 0;   // streamed tile on its way (waves 1 .. 7: since before the wait)
        if (ns > 0 && (wave == 0 || prod == 0)) load_tile(str, rs_A, b0 + s0, voff);
#pragma unroll
        for (int v = 0; v < (int)(sizeof xv / sizeof xv[0]); ++v)
            if (tid + v * kHeatThr < 2 * m * (kHeatTile / 4))
                *reinterpret_cast<f4*>(&(&xcol[0][0])[4 * (tid + v * kHeatThr)]) = xv[v];
        __syncthreads();
        float rs[8], xi[8];
#pragma unroll
        for (int q2 = 0; q2 < 8; ++q2) rs[q2] = xi[q2] = 0.f;
        int k = 0, I = I0, J = J0, Jrun = J0;   // the next tile, and its run's first column
        // the row sums of the run (I, Jrun ..)
        auto close_run = [&]() {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float v = heat_row_sum(rs[e]);
                if ((lane & 3) == 0) rows[wave][8 * rg + e] = v;
                rs[e] = 0.f;
            }
            __syncthreads();
            if (tid < kHeatTile) {
                float v = rows[0][tid];
#pragma unroll
                for (int w = 1; w < kHeatWaves; ++w) v += rows[w][tid];
                coh_store(rs_part, 4 * tid, (I * nT + Jrun) * kSlotBytes, v);
            }
            __syncthreads();
        };
        auto use_tile = [&](auto get) {
            if (J == nT) {   // (uniform) the next row block
                close_run();
                ++I;
                J = Jrun = I;
            }
            if (J == Jrun) {
                const f4 u0 = *reinterpret_cast<const f4*>(&xcol[m + k][8 * rg]);
                const f4 u1 = *reinterpret_cast<const f4*>(&xcol[m + k][8 * rg + 4]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    xi[e] = u0[e];
                    xi[4 + e] = u1[e];
                }
            }
            const f4 xj = *reinterpret_cast<const f4*>(&xcol[k][16 * wave + 4 * (lane & 3)]);
            const f4 cs = heat_tile_fma<true>(get, xj, xi, rs);
            if (I != J) {
                const float v = heat_column_sum(cs);
                if ((lane & 12) == 0) coh_store(rs_part, coff, (J * nT + I) * kSlotBytes, v);
            }
            ++k;
            ++J;
        };
        // the streamed tiles between kept tile j and the next kept one; the
        // one after each is on its way while a kept one is multiplied
        auto use_streamed = [&](int j) {
            const int upto = kept_at(j + 1);
            while (k < upto) {
                use_tile([&](int e) { return str.v[e]; });
                if (++sn < ns) load_tile(str, rs_A, b0 + streamed_at(sn), voff);
            }
        };
#pragma unroll
        for (int j = 0; j < kRegTiles; ++j)
            if (j < nk) {
                use_tile([&](int e) { return reg[j].v[e]; });
                use_streamed(j);
            }
        for (int j = kRegTiles; j < nk; ++j) {
            const f4* p = reinterpret_cast<const f4*>(kept + (j - kRegTiles) * kHeatTileFloats) + wave * 512 + lane;
            use_tile([&](int e) { return p[64 * e]; });
            use_streamed(j);
        }
        close_run();
        publish_phase(R.sync, slot, ++count);
        if (!wait_all<false>(R.sync, slot, nb, count, R.spin_limit, &failed, no_decision)) return;

        // ---- finish: wave w sums slots w, w + 8, ..., wave 0 adds the waves' sums in order
        float y = 0.f;
        if (mine) {
            float v[kSlots];   // (all on their way at once)
#pragma unroll
            for (int e = 0; e < kSlots; ++e) {
                const int K = wave + e * kHeatWaves;
                v[e] = K < nT ? coh_load(rs_part, slots, K * kSlotBytes) : 0.f;
            }
#pragma unroll
            for (int e = 0; e < kSlots; ++e) y += v[e];
        }
        red[wave][lane] = y;
        __syncthreads();
        if (wave == 0 && mine) {
            float v = red[0][lane];
#pragma unroll
            for (int w = 1; w < kHeatWaves; ++w) v += red[w][lane];
            if (bstep) {
                if (chk)
                    __hip_atomic_store(G.errrow + cell, fabs((double)bold * (double)v - (double)q), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                bold = q == 0.f ? 0.f : q / v;
                coh_store(rsrc_of(G.b, nT * kSlotBytes), 4 * cell, 0, bold);
            } else {
                const float p = prox_val<KIND>(R.s.px, v, pu, pv);
                coh_store(rsrc_of(R.s.a, nT * kSlotBytes), 4 * cell, 0, p == 0.f ? 0.f : p / v);
                if ((CHECK && to_check == 0) || prod + 1 == R.last) R.s.p[gi] = p;   // (what a check or the end returns)
            }
        }
        if (prod + 1 == R.last) break;
        publish_phase(R.sync, slot, ++count);
        // (wave 0 polls: its loads would have to land first)
        if (ns > 0 && wave != 0) load_tile(str, rs_A, b0 + s0, voff);
        if (chk) {
            if (!wait_all<true>(R.sync, slot, nb, count, R.spin_limit, &failed, [&]() { return outcome(prod); })) return;
        } else if (!wait_all<false>(R.sync, slot, nb, count, R.spin_limit, &failed, no_decision)) {
            return;
        }
    }
}

template <bool CHECK>
const void* kernel_as(int kind) {
    switch (kind) {
        case JKO_F_ZERO: return reinterpret_cast<const void*>(&heat_resident<JKO_F_ZERO, CHECK>);
        case JKO_F_CONGESTION: return reinterpret_cast<const void*>(&heat_resident<JKO_F_CONGESTION, CHECK>);
        case JKO_F_POROUS: return reinterpret_cast<const void*>(&heat_resident<JKO_F_POROUS, CHECK>);
        case JKO_F_ENTROPY: return reinterpret_cast<const void*>(&heat_resident<JKO_F_ENTROPY, CHECK>);
        case JKO_F_CONGESTION_BINARY:
            return reinterpret_cast<const void*>(&heat_resident<JKO_F_CONGESTION_BINARY, CHECK>);
        case JKO_F_GEN_ENTROPY: return reinterpret_cast<const void*>(&heat_resident<JKO_F_GEN_ENTROPY, CHECK>);
        default: return nullptr;
    }
}
const void* kernel_of(int kind, bool check) { return check ? kernel_as<true>(kind) : kernel_as<false>(kind); }

int blocks_of(int nT) { return (int)std::min<int64_t>((int64_t)nT * (nT + 1) / 2, kMaxBlocks); }
size_t lds_of(int nT) {
    const int64_t T = (int64_t)nT * (nT + 1) / 2, nb = blocks_of(nT);
    return (T + nb - 1) / nb > kRegTiles ? (size_t)kLdsTiles * kHeatTileFloats * sizeof(float) : 0;
}

}  // namespace

int64_t heat_resident_sync_words() { return kGo + kGoStride * kGoCopies; }

bool heat_resident_fits(int nT, int kind, bool check) {
    const void* fn = kernel_of(kind, check);
    // (fewer row blocks leave a block more than 64 cells to finish)
    if (!fn || nT < 3) return false;
    const int64_t T = (int64_t)nT * (nT + 1) / 2, nb = blocks_of(nT);
    if ((T + nb - 1) / nb > kMaxTiles || nT > kSlots * kHeatWaves) return false;
    int dev = 0, coop = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop) return false;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return false;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kHeatThr, lds_of(nT)) != hipSuccess) return false;
    return (int64_t)per_cu * cus >= nb;
}

hipError_t launch_heat_resident(const HeatResident& r, int kind, hipStream_t st) {
    const void* fn = kernel_of(kind, r.period > 0);
    if (!fn) return hipErrorInvalidValue;
    HeatResident arg = r;
    void* args[] = {&arg};
    return hipLaunchCooperativeKernel(fn, dim3((unsigned)blocks_of(r.t.nT)), dim3(kHeatThr), args, lds_of(r.t.nT), st);
}

}  // namespace jko
