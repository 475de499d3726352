// Device code shared by the stored heat operator's kernels (heat.hip,
// heatres.hip): the layout of its 128 x 128 tiles, their products, and the
// epilogue of a free cell's row.
#pragma once

#include "epilogue.h"
#include "heat.h"

namespace jko {

// A tile is spread over eight waves of 64 lanes: wave w holds columns 16 w ..
// 16 w + 15, lane l of it rows 8 (l / 4) .. + 7 of columns 4 (l % 4) .. + 3, as
// eight float4s (one per row).  It is stored in that order, so that each
// float4 load of a wave is 1 KiB of consecutive memory.
constexpr int kHeatThr = 512;
constexpr int kHeatWaves = kHeatThr / 64;
constexpr int kHeatTileFloats = kHeatTile * kHeatTile;

// Position of element (r, c) within its tile.
__host__ __device__ __forceinline__ int heat_tile_offset(int r, int c) {
    const int w = c >> 4, lane = (r >> 3) * 4 + ((c >> 2) & 3);
    return ((w * 8 + (r & 7)) * 64 + lane) * 4 + (c & 3);
}

struct HeatTileRegs {
    f4 v[8];
};

// rs[q] += this lane's share of row 8 (lane / 4) + q of A x_J, and the lane's
// share of the four columns of A^T x_I.  get(q): the lane's float4 of row q.
template <bool BATCH = false, typename Get>
__device__ __forceinline__ f4 heat_tile_fma(Get get, f4 xj, const float (&xi)[8], float (&rs)[8]) {
    f4 cs = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const f4 v = get(q);
        rs[q] += (v[0] * xj[0] + v[1] * xj[1]) + (v[2] * xj[2] + v[3] * xj[3]);
#pragma unroll
        for (int e = 0; e < 4; ++e) cs[e] += v[e] * xi[q];
        if (BATCH && q % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // (no more than four rows loaded ahead)
    }
    return cs;
}

template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
    const int o = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true);
    return v + __int_as_float(o);
}

// The sum of one row over the four lanes that share it (every lane of the four).
__device__ __forceinline__ float heat_row_sum(float v) {
    v = dpp_add<0xB1>(v);      // lane ^ 1
    return dpp_add<0x4E>(v);   // lane ^ 2
}

// The sums of the four columns over the 16 lanes that share them: lane l ends
// with column l / 16 of its group of four.  The halves of the wave trade two
// values each (lanes below 32 keep columns 0 and 1), then the rows of 16 lanes
// one, then two rotations within a row of 16.
__device__ __forceinline__ float heat_column_sum(f4 cs) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    auto swap32 = [](float a, float b) {
        const u2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    };
    const float u0 = swap32(cs[0], cs[2]), u1 = swap32(cs[1], cs[3]);
    const u2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(u0), __float_as_uint(u1), false, false);
    float v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    v = dpp_add<0x128>(v);     // row_ror 8
    return dpp_add<0x124>(v);  // row_ror 4
}

// The fields the proximal map of a grid cell needs (prox_val's pu, pv).
template <int KIND>
__device__ __forceinline__ void heat_prox_fields(const ProxArgs& px, int64_t i, float& pu, float& pv) {
    if (KIND == JKO_F_CONGESTION || KIND == JKO_F_CONGESTION_BINARY) {
        pu = px.g ? px.g[i] : 1.f;
        pv = px.kappa ? px.kappa[i] : px.kappa_s;
    } else if (KIND == JKO_F_ENTROPY || KIND == JKO_F_POROUS) {
        pu = px.kf ? px.kf[i] : px.kf_s;
    } else if (KIND == JKO_F_GEN_ENTROPY) {
        pu = px.kf ? px.kf[i] : px.kf_s;
        pv = px.g ? px.g[i] : px.eps_s;
    }
}

// Finish row r (free cell i = gidx[r]) of y = A x (value v): the epilogue of
// the iteration's half-step.
template <int EK>
__device__ __forceinline__ void heat_epilogue(const HeatGemv& g, int64_t r, float v) {
    const int64_t i = g.gidx[r];
    if constexpr (EK == EK_STORE) {
        g.y[i] = v;
    } else if constexpr (EK == EK_BUPDATE || EK == EK_MONITOR) {
        const float q = g.q[i];
        if (EK == EK_MONITOR || g.check) g.errrow[r] = fabs((double)g.b[r] * (double)v - (double)q);
        if (EK == EK_BUPDATE) g.b[r] = q == 0.f ? 0.f : q / v;
    } else {
        constexpr int KIND = EK - EK_PROX;
        float pu = 1.f, pv = 0.f;
        heat_prox_fields<KIND>(g.px, i, pu, pv);
        const float p = prox_val<KIND>(g.px, v, pu, pv);
        g.a[r] = p == 0.f ? 0.f : p / v;
        g.p[i] = p;
    }
}

}  // namespace jko
