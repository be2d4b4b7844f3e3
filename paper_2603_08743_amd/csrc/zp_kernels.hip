// Unit kernels of libzp.  A unit is one (request, layer, kv head); one workgroup takes a whole unit, or several share it over several
// launches where units are few (split_pays in zp_api.hip).
//
//  * unit_mfma: the (G*w) x T logits are a dense contraction over d, so they run on the matrix cores
//    (v_mfma_f32_32x32x16_bf16, v_mfma_f32_32x32x2_f32) from LDS-staged key tiles.
//  * unit_generic: scoring on the vector ALUs for what does not fit there (more than 16 query heads per kv head,
//    sequences whose scores leave no room for two key tiles in LDS), and the staged select-only / compact-only passes of many units.
//  * unit_sliced: selection and row moving of few units, the rows cut into slices.
//
// Scores follow the appendix "Paged Attention Score": softmax over positions per window
// query, max over the query heads of the group, mean over the window.  The max over heads
// needs the final normaliser of every row, and the (G*w) x T logits do not fit on chip, so
// the keys are swept twice: sweep 1 reduces each row to its log-sum-exp, sweep 2 recomputes
// the logits and reduces them to S[t] = (1/w) sum_u max_g exp(a[g,u,t] - lse[g,u]).
#include "zp_device.h"

namespace zp {

// ------------------------------------------------------------------ generic path

template <int DT> __device__ __forceinline__ float ld_elem(const char *p, int i);
template <> __device__ __forceinline__ float ld_elem<0>(const char *p, int i) { return ((const float *)p)[i]; }
template <> __device__ __forceinline__ float ld_elem<1>(const char *p, int i) {
    return __uint_as_float((unsigned)((const unsigned short *)p)[i] << 16);
}

template <int DT> __device__ __forceinline__ float dot_row(const char *q, const char *k, int d) {
    float acc = 0.f;
    for (int c = 0; c < d; c++) acc = fmaf(ld_elem<DT>(q, c), ld_elem<DT>(k, c), acc);
    return acc;
}

template <int DT>
__device__ void score_generic(const Args &a, const Unit &u, char *smem, const int *tbl) {
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wv = tid >> 6, nw = nt >> 6;
    float *S = (float *)(smem + a.off_S);
    float *lse = (float *)(smem + a.off_union);
    const int G = a.G, w = a.w, rows = G * w;
    const size_t qbase = (((size_t)u.ls * a.M + u.slot) * w) * a.h_q;   // in rows of d elements
    for (int t = tid; t < u.T; t += nt) S[t] = 0.f;
    // sweep 1: log-sum-exp (base 2) of every window row over the keys it may see
    for (int r = wv; r < rows; r += nw) {
        const int g = r / w, uu = r - g * w;
        const char *q = a.q + (qbase + (size_t)uu * a.h_q + u.h * G + g) * a.row_bytes;
        const int jmax = u.Tv - w + uu;                               // causal: keys after the query are hidden
        float m = -1e30f, l = 0.f;
        for (int j = lane; j <= jmax; j += 64) {
            const int t = live_to_pos(u, a, j), blk = div_b(a, t);
            const float x = dot_row<DT>(q, a.k + row_off(a, u.ls, tbl[blk], t - blk * a.b, u.h), a.d) * a.scale_log2;
            if (x > m) { l = l * fexp2(m - x) + 1.f; m = x; }
            else l += fexp2(x - m);
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const float mo = __shfl_xor(m, off), lo = __shfl_xor(l, off);
            const float mm = fmaxf(m, mo);
            l = l * fexp2(m - mm) + lo * fexp2(mo - mm);
            m = mm;
        }
        if (lane == 0) lse[r] = m + flog2(l);
    }
    __syncthreads();
    // sweep 2: S[t] = (1/w) sum_u max_g exp2(x - lse)
    for (int j = tid; j < u.Tv; j += nt) {
        const int t = live_to_pos(u, a, j), blk = div_b(a, t);
        const char *kr = a.k + row_off(a, u.ls, tbl[blk], t - blk * a.b, u.h);
        float acc = 0.f;
        for (int uu = 0; uu < w; uu++) {
            if (j > u.Tv - w + uu) continue;
            float mx = 0.f;
            for (int g = 0; g < G; g++) {
                const char *q = a.q + (qbase + (size_t)uu * a.h_q + u.h * G + g) * a.row_bytes;
                const float x = dot_row<DT>(q, kr, a.d) * a.scale_log2;
                mx = fmaxf(mx, fexp2(x - lse[g * w + uu]));
            }
            acc += mx;
        }
        S[t] = acc / (float)w;
    }
    __syncthreads();
}

template <int DT>
__global__ void __launch_bounds__(256) unit_generic(const Args a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    int *tbl = (int *)(smem + a.off_tbl), *dst = (int *)(smem + a.off_dst);
    Misc *misc = (Misc *)(smem + a.off_misc);
    Unit u;
    if (!unit_setup(a, unit_of_block((int)blockIdx.x, (int)gridDim.x, a.xcd_map), u, tbl, dst, misc)) return;
    if (a.stages & STAGE_SCORE) score_generic<DT>(a, u, smem, tbl);
    unit_tail<0, DT, false, 3, 4, false>(a, u, smem, tbl, dst, misc);
}

hipError_t launch_unit_generic(const Args &a, int units, hipStream_t s) {
    if (units <= 0) return hipSuccess;
    hipError_t e = a.dtype == 0 ? allow_big_lds<unit_generic<0>>() : allow_big_lds<unit_generic<1>>();
    if (e != hipSuccess) return e;
    if (a.dtype == 0) hipLaunchKernelGGL(unit_generic<0>, dim3(units), dim3(256), a.lds_bytes, s, a);
    else hipLaunchKernelGGL(unit_generic<1>, dim3(units), dim3(256), a.lds_bytes, s, a);
    return hipGetLastError();
}

// Selection and row moving with several workgroups per unit, for launches of few units: every workgroup selects for itself
// (nothing to hand over, and the units would leave the other compute units idle) and moves its slice of the rows.
__global__ void __launch_bounds__(1024) unit_sliced(const Args a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    int *tbl = (int *)(smem + a.off_tbl), *dst = (int *)(smem + a.off_dst);
    Misc *misc = (Misc *)(smem + a.off_misc);
    const int v = unit_of_block((int)blockIdx.x, (int)gridDim.x, a.xcd_map);
    Unit u;
    if (!unit_setup<true>(a, v / a.slices, u, tbl, dst, misc)) return;
    unit_tail<0, 1, false, 0, 16, false, true>(a, u, smem, tbl, dst, misc, v % a.slices);
}

hipError_t launch_unit_sliced(const Args &a, int units, hipStream_t s) {
    if (units <= 0) return hipSuccess;
    hipError_t e = allow_big_lds<unit_sliced>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(unit_sliced, dim3(units * a.slices), dim3(1024), a.lds_bytes, s, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------ matrix-core path: geometry and dispatch

size_t mfma_union_bytes(const MfmaGeo &g) {
    const int kt = mfma_tile_keys(g.rowb);
    return 2 * (size_t)kt * (g.rowb + 16) + 2 * (size_t)g.NW * kt * 4 + (size_t)g.NW * g.RB * 32 * 4;
}

// (RB, NW) by the number of 32-row query blocks: small windows use fewer waves, large ones more rows per wave
static void pick_geometry(int NB, int *NW, int *RB) {
    if (NB <= 1) { *NW = 1; *RB = 1; }
    else if (NB <= 2) { *NW = 2; *RB = 1; }
    else if (NB <= 4) { *NW = 4; *RB = 1; }
    else if (NB <= 8) { *NW = 8; *RB = 1; }
    else if (NB <= 16) { *NW = 8; *RB = 2; }
    else if (NB <= 24) { *NW = 8; *RB = 3; }
    else { *NW = 8; *RB = 4; }
}

// bf16 rows of 128 and 256 bytes have kernels of their own; every other row, and windows of more than 32 query blocks, runs
// padded to the next of a few sizes.  Before, those shapes took one dot product per (query row, key) on the vector ALUs with
// one key row per lane (uncoalesced 16-byte steps): fp32, d = 128, G = 4, w = 32, 128 units of 1040 positions 17.6 ms ->
// 0.294 ms; bf16, d = 96, G = 3, w = 20, 72 units of up to 1248 positions 6.98 ms -> 0.154 ms.  A padded k step of
// 32 bytes costs its share of a tile's products, 1/4 of them at 128 bytes and 1/32 at 1024; every further size is another set of
// kernels.
bool mfma_path_available(const Args &a, MfmaGeo *g) {
    if (a.G < 1 || a.G > 16) return false;
    const int UL = 16 / a.G, NB = (a.w + 2 * UL - 1) / (2 * UL);
    g->NP = 1;
    if (a.dtype == 1 && (a.d == 128 || a.d == 64) && NB <= 32) {
        g->pad = false;
        g->rowb = a.row_bytes;
        pick_geometry(NB, &g->NW, &g->RB);
        return true;
    }
    g->pad = true;
    g->RB = 1;
    g->NW = NB <= 2 ? 2 : NB <= 4 ? 4 : 8;
    g->NP = (NB + g->NW - 1) / g->NW;
    static const int sizes_bf16[] = {128, 192, 256, 384, 512, 1024}, sizes_f32[] = {256, 512, 1024};
    for (int r : sizes_bf16) if (a.dtype == 1 && a.row_bytes <= r) { g->rowb = r; return true; }
    for (int r : sizes_f32) if (a.dtype == 0 && a.row_bytes <= r) { g->rowb = r; return true; }
    return false;
}

hipError_t launch_unit_mfma(const Args &a, int units, const MfmaGeo &g, hipStream_t s) {
    if (units <= 0) return hipSuccess;
    if (g.pad) {
        if (a.dtype == 0) return launch_mfma_pad_f32(a, units, g.rowb, g.NW, s);
        return g.rowb <= 256 ? launch_mfma_pad_bf16(a, units, g.rowb, g.NW, s) : launch_mfma_pad_bf16_long(a, units, g.rowb, g.NW, s);
    }
    const bool ref = (a.ex & (EX_GLOBAL | EX_POOL | EX_RED)) != 0, wide = g.NW > 4;
    if (a.d == 128) return (ref ? (wide ? launch_mfma_d128_wide_ref : launch_mfma_d128_ref) : (wide ? launch_mfma_d128_wide : launch_mfma_d128))(a, units, g.NW, g.RB, s);
    return (ref ? (wide ? launch_mfma_d64_wide_ref : launch_mfma_d64_ref) : (wide ? launch_mfma_d64_wide : launch_mfma_d64))(a, units, g.NW, g.RB, s);
}

}  // namespace zp
