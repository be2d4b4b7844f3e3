// Matrix-core unit kernel of libzp and its launcher templates.  The instantiations are spread over several translation
// units (zp_mfma_*.hip) so that they compile in parallel.
#pragma once
#include "zp_device.h"

#include <type_traits>

namespace zp {

// Key tiles: the first sweep loads them normally (the second sweep, which runs the other way, finds the most recent
// ones in L2 / Infinity Cache); the second sweep is their last use by this workgroup and loads them non-temporally.
// Measured on the 8B-like shape: non-temporal in sweep 1 costs 0.5 ms per launch, in sweep 2 it gains 0.1-0.3 ms.
#define ZP_NT1 std::false_type
#define ZP_NT2 std::true_type

// Waves per SIMD the register allocation aims at.  One query block per wave (RB = 1) fits 128 registers: eight such
// waves per workgroup and two workgroups per CU put four waves on every SIMD, which overlaps the matrix-core and
// vector-ALU phases of different waves and gives the row-moving phase sixteen waves per CU to issue memory operations
// from (measured on the 8B-like shape: 15.0 ms per launch against 17.0 ms with four waves of two blocks each).
// Rows above 256 bytes keep 8 more registers of query fragments per 64 bytes, and as many again of tile loads: half the waves.
// Below four waves the compiler is left its own choice: held to 168 registers, one-wave kernels of 256-byte rows take 30 % longer (1344
// units of 3760 positions, G 1, w 32: 1449 -> 1900 us) and two-wave kernels of 512-byte rows spill hundreds of registers.
#define ZP_WPE(NW, RB, ROWB) ((NW) == 8 && (RB) == 1 && (ROWB) <= 256 ? 4 : ((NW) >= 4 ? 2 : 1))

// ------------------------------------------------------------------ matrix-core path
//
// Query rows are laid out so that both reductions of sweep 2 stay inside a lane.  A 32x32 MFMA
// tile gives lane L, register i the element (row 4*(L/32) + 8*(i/4) + i%4, column L%32).  With
// the query block as the row operand, one half-wave (hf = L/32) owns 16 rows of the block per
// key column; those 16 slots hold UL = 16/G window rows u with their G query heads side by side
// (slot i = ul*G + g; left-over slots are zero rows).  Block gb, half hf, slot i therefore is
// window row u = (gb*2 + hf)*UL + i/G, head g = i%G.  NW waves split the NB blocks (RB each) and
// share every key tile through LDS.  In sweep 1 the operands swap, so a lane owns one query row
// and 16 keys per tile and the running (max, sum) of a row never leaves its lane.

//
// Rows are handled as ROWB bytes of either element type (DT: 0 fp32, 1 bf16): a fragment is 16 bytes of a row, i.e. eight
// bf16 values (one v_mfma_f32_32x32x16_bf16) or four fp32 values (four v_mfma_f32_32x32x2_f32, which multiply and add in
// fp32), and both operands take their k index from the same bytes.  PAD: the pool's rows are shorter than ROWB; the
// pieces beyond them are zeros in LDS and in the query fragments and add nothing.

template <int ROWB> struct KTile {
    static constexpr int KT = mfma_tile_keys(ROWB);
    static constexpr int ROW = ROWB + 16;         // padded row stride in bytes: conflict-free 16-byte fragment reads
    static constexpr int BYTES = KT * ROW;
    static constexpr int CPR = ROWB / 16;         // 16-byte pieces per key row
};

// REF: 0 no score refinements in this launch, 1 global score and pooling in the tail, 3 the lightning redundancy as well, 2
// (block size 16, RB = 1, unpadded bf16 rows) its similarity tiles of the live prefix taken from the key tiles of sweep 2
// (with 3 the keys are read a third time in the tail), 4 the redundancy of large blocks (four and eight waves, redundancy_staged).  With the redundancy code in it an eight-wave kernel has no registers
// left, so launches without redundancy do not carry it: 512 units of 4112 positions (d 128, G 4, w 64) with global score and
// pooling took 644 us with 21 spilled registers and take 622 us with none.
// MP: the query blocks take several passes over the keys (NP groups of NW * RB blocks), S collecting their sums.
template <int DT, int ROWB, bool PAD, int RB, int NW, int GT, int REF, bool MP, int PH = 0>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(ZP_WPE(NW, RB, ROWB)))) unit_mfma(const Args a) {
    constexpr bool RED = REF == 2;
    // A segment starts with the maximum of its first 32 keys as reference, not with a subtile that is redone: same bits.  1664 units of
    // up to 912 positions (G 5, w 11) 342 -> 338 us, 272 units of up to 1088 (d 64, w 34) 67.9 -> 65.3 us, 384 of 8208 (G 5, w 128) 1390 ->
    // 1380 us.  Not where the registers are full: 512 units of 4112 with the fused redundancy (REF 2) 659 -> 696 us, 80 units of 4288 with
    // the separate one 356 -> 361 us.
    constexpr bool FIRST_MAX = REF < 2 || (REF >= 3 && RB > 1);
    extern __shared__ __attribute__((aligned(16))) char smem[];
    int *tbl = (int *)(smem + a.off_tbl), *dst = (int *)(smem + a.off_dst);
    Misc *misc = (Misc *)(smem + a.off_misc);
    Unit u;
    int uid = unit_of_block((int)blockIdx.x, (int)gridDim.x, a.xcd_map), part_no = 0;
    if (PH) { part_no = uid % a.parts; uid /= a.parts; }
    else if (a.by_cost) uid = unit_by_cost(a, (int)blockIdx.x, (int)gridDim.x, misc);
    const bool usable = unit_setup<false, PH == 0>(a, uid, u, tbl, dst, misc);
    if (PH == 2 && part_no == 0 && threadIdx.x == 0 && a.unit_out) a.unit_out[uid] = usable ? make_int2(u.vl, u.k) : make_int2(-1, -1);
    if (!usable) return;

    using KTl = KTile<ROWB>;
    constexpr int KT = KTl::KT, CPR = KTl::CPR, NT = NW * 64, KK = ROWB / 32;
    constexpr bool EVEN = NT % CPR == 0 && KT * CPR % NT == 0;   // a thread fetches the same piece of every row it takes
    constexpr int LPT = (KT * CPR + NT - 1) / NT;
    static_assert(NT >= KT && (PAD || EVEN), "unpadded rows divide evenly among the threads");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, l32 = lane & 31, hf = lane >> 5;
    const int G = GT ? GT : a.G, UL = 16 / G, w = a.w;
    float *S = (float *)(smem + a.off_S);
    char *kbuf = smem + a.off_union;
    float *part = (float *)(kbuf + 2 * KTl::BYTES);          // [2][NW][KT] partial sums of sweep 2
    float *lse = part + 2 * NW * KT;                         // [NB*32] per padded query row
    const float c = a.scale_log2;

    const int row_bytes = PAD ? a.row_bytes : ROWB;

    if (!PH) for (int t = tid; t < u.T; t += NT) S[t] = 0.f;   // stale positions stay 0
    const int np = MP ? a.NP : 1;
#pragma unroll 1
    for (int pass = 0; pass < np; pass++) {
    // query fragments: this lane supplies padded row l32 of each of its blocks, 16 bytes per k step
    u32x4 qf[RB][KK];
    int u_col[RB];                                           // window row this lane owns in sweep 1 (-1: zero row)
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
        const int gb = (pass * NW + wv) * RB + rb;
        const int mh = (l32 >> 2) & 1, i = ((l32 >> 3) << 2) | (l32 & 3);
        const int ul = i / G, g = i - ul * G, uu = (gb * 2 + mh) * UL + ul;
        const bool ok = ul < UL && uu < w;
        u_col[rb] = ok ? uu : -1;
        const char *qp = a.q + ((((size_t)u.ls * a.M + u.slot) * w + (ok ? uu : 0)) * a.h_q + u.h * G + g) * (size_t)row_bytes + hf * 16;
#pragma unroll
        for (int kk = 0; kk < KK; kk++) {
            u32x4 raw = {0u, 0u, 0u, 0u};
            if (ok && (!PAD || kk * 32 + hf * 16 < row_bytes)) raw = *(const u32x4 *)(qp + kk * 32);
            qf[rb][kk] = raw;
        }
    }

    const int ntiles = (u.Tv + KT - 1) / KT;
    // this workgroup's tiles [t_lo, t_hi)
    const int nseg = segment_count(ntiles, segments_of(RB));
    int t_lo = 0, t_hi = ntiles;
    int sg_lo = 0;
    if (PH) {                                                 // whole segments
        sg_lo = part_no * nseg / a.parts;
        const int sg_hi = (part_no + 1) * nseg / a.parts;
        if (sg_lo == sg_hi) return;
        t_lo = sg_lo * ntiles / nseg;
        t_hi = sg_hi * ntiles / nseg;
    }
    const int n_here = t_hi - t_lo;
    float2 *seg = a.seg + (size_t)u.unit * ZP_SEGMENTS * (NW * RB * 32);
    // Key tiles travel HBM -> registers -> LDS.  With one query block per wave a tile is requested when the work on the one before it
    // starts: a second register set, with every tile requested two turns ahead, changed nothing from 64 to 2048 units of 4112
    // positions and cost up to 130 registers.  With two or three blocks per wave one workgroup has the compute unit to itself and
    // the second set (DEEP) gives 3 % (160 units of 3440, G 4, w 72: 270 -> 262 us).  Loops of two tiles a turn (TWO) where a wave holds
    // several blocks (44 units of 9136, G 7, w 108: 508 -> 401 us) and with redundancy in the launch (448 units of 5200: 949 -> 921 us);
    // everywhere else two tiles a turn change nothing (182 calls of all kinds: 1.001 times) and cost code.
    constexpr bool TWO = RB > 1 || REF >= 2, DEEP = RB == 2 || (RB == 3 && REF < 3);
    u32x4 stA[LPT], stB[LPT];                                 // named by type: passed by reference, the padded kernels take up to 180 registers more
    using SetA = std::false_type;
    using SetB = std::true_type;
    // a thread always fetches the same 16-byte piece of rows r0, r0 + RSTEP, ...: one 64-bit base, then
    // base + token * (bytes between consecutive tokens) with token = block * b + slot (fits 32 bits, host-checked)
    constexpr int RSTEP = NT / CPR;
    const int r0 = tid / CPR;
    const int piece0 = (tid - r0 * CPR) * 16;
    const char *kbase = a.k + ((size_t)u.ls * a.N_total * a.b * a.h_kv + u.h) * (size_t)row_bytes + (EVEN ? piece0 : 0);
    const unsigned tok_bytes = (unsigned)a.h_kv * row_bytes;
    const int gap = (u.N - 1) * a.b - u.vl;                   // stale positions between the live prefix and the last block
    auto gload = [&](int tile, auto set, auto nt_tag) __attribute__((always_inline)) {   // rows past the end repeat the last key (masked later)
        u32x4 (&st)[LPT] = decltype(set)::value ? stB : stA;
        // Tiles that lie wholly in the live prefix (all but the last one or two) need none of the edge handling when
        // the block size is a power of two: position = live index.  (Eight-wave workgroups only: with fewer waves a
        // thread loads eight or sixteen pieces per tile and the second copy of that code costs registers.)
        if (NW == 8 && EVEN && !PAD && a.b_shift >= 0 && (tile + 1) * KT <= u.vl) {
#pragma unroll
            for (int i = 0; i < LPT; i++) {
                const int j = tile * KT + i * RSTEP + r0;
                const unsigned tok = ((unsigned)tbl[j >> a.b_shift] << a.b_shift) + (unsigned)(j & (a.b - 1));
                if (decltype(nt_tag)::value) st[i] = __builtin_nontemporal_load((const u32x4 *)(kbase + (size_t)tok * tok_bytes));
                else st[i] = *(const u32x4 *)(kbase + (size_t)tok * tok_bytes);
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < LPT; i++) {
            const int pc = tid + i * NT, row = EVEN ? r0 + i * RSTEP : pc / CPR, off = EVEN ? piece0 : (pc - row * CPR) * 16;
            if (PAD) {                                        // pieces past the pool's row, and past the tile, are zeros
                st[i] = u32x4{0u, 0u, 0u, 0u};
                if (off >= row_bytes || (!EVEN && row >= KT)) continue;
            }
            int j = tile * KT + row;
            j = j < u.Tv ? j : u.Tv - 1;
            const int t = j < u.vl ? j : j + gap;
            unsigned tok;
            if (a.b_shift >= 0) {
                const int blk = t >> a.b_shift;
                tok = ((unsigned)tbl[blk] << a.b_shift) + (unsigned)(t & (a.b - 1));
            } else {
                const int blk = t / a.b;
                tok = (unsigned)tbl[blk] * (unsigned)a.b + (unsigned)(t - blk * a.b);
            }
            const char *kp = kbase + (size_t)tok * tok_bytes + (EVEN ? 0 : off);
            if (decltype(nt_tag)::value) st[i] = __builtin_nontemporal_load((const u32x4 *)kp);
            else st[i] = *(const u32x4 *)kp;
        }
    };
    const int lds_st = r0 * KTl::ROW + piece0;
    auto lstore = [&](char *buf, auto set) __attribute__((always_inline)) {
        const u32x4 (&st)[LPT] = decltype(set)::value ? stB : stA;
#pragma unroll
        for (int i = 0; i < LPT; i++) {
            if (EVEN) *(u32x4 *)(buf + lds_st + i * RSTEP * KTl::ROW) = st[i];
            else {
                const int pc = tid + i * NT, row = pc / CPR;
                if (row < KT) *(u32x4 *)(buf + row * KTl::ROW + (pc - row * CPR) * 16) = st[i];
            }
        }
    };
    f32x16 zero16;
#pragma unroll
    for (int i = 0; i < 16; i++) zero16[i] = 0.f;

    // ---------------- sweep 1: per query row, running max and sum of exp2 over the keys it may see
    float rm[RB], rl[RB];
#pragma unroll
    for (int rb = 0; rb < RB; rb++) { rm[rb] = -1e30f; rl[rb] = 0.f; }
    // The sum of exp2(x - ref) is kept against a per-row reference `rm` that only moves when the sum leaves the
    // safe range (first subtile, or logits that jump by more than ~2^100): then the subtile is redone with the
    // proper maximum.  This keeps the common path free of the max reduction: fma, exp2, add per logit.
    auto sweep1_body = [&](const char *buf, int j0, bool fresh, auto edge_tag) __attribute__((always_inline)) {   // fresh: a segment's first tile
        constexpr bool edge = decltype(edge_tag)::value;
#pragma unroll
        for (int sub = 0; sub < KT / 32; sub++) {
            if (PAD && edge && j0 + sub * 32 >= u.Tv) break;  // nothing left of the sequence (unpadded: costs the eight-wave redundancy kernel 13 spills)
            f32x16 acc[RB];
            const char *kp = buf + (sub * 32 + l32) * KTl::ROW + hf * 16;
#pragma unroll
            for (int kk = 0; kk < KK; kk++) {
                const u32x4 kf = *(const u32x4 *)(kp + kk * 32);
#pragma unroll
                for (int rb = 0; rb < RB; rb++) acc[rb] = mma32<DT>(kf, qf[rb][kk], kk ? acc[rb] : zero16);
            }
            // acc[rb][i]: key j0 + sub*32 + 4*hf + 8*(i/4) + i%4, query row = this lane's column
#pragma unroll
            for (int rb = 0; rb < RB; rb++) {
                if (edge) {
                    const int lim = u_col[rb] >= 0 ? u.Tv - w + u_col[rb] : u.Tv - 1;
#pragma unroll
                    for (int i = 0; i < 16; i++) {
                        const int j = j0 + sub * 32 + 4 * hf + 8 * (i >> 2) + (i & 3);
                        if (j > lim) acc[rb][i] = -INFINITY;
                    }
                }
                if (FIRST_MAX && sub == 0 && fresh) {        // the reference that the redo below would find
                    float tm = acc[rb][0];
#pragma unroll
                    for (int i = 1; i < 16; i++) tm = fmaxf(tm, acc[rb][i]);
                    rm[rb] = fmaxf(-1e30f, tm * c);
                }
                float sum = 0.f;
#pragma unroll
                for (int i = 0; i < 16; i++) sum += fexp2(fmaf(acc[rb][i], c, -rm[rb]));
                const float ln = rl[rb] + sum;
                if (__builtin_expect(__any(!(ln < 1e30f)), 0)) {        // wave-uniform, rare
                    float tm = acc[rb][0];
#pragma unroll
                    for (int i = 1; i < 16; i++) tm = fmaxf(tm, acc[rb][i]);
                    const float mn = fmaxf(rm[rb], tm * c);
                    sum = 0.f;
#pragma unroll
                    for (int i = 0; i < 16; i++) sum += fexp2(fmaf(acc[rb][i], c, -mn));
                    rl[rb] = rl[rb] * fexp2(rm[rb] - mn) + sum;
                    rm[rb] = mn;
                } else {
                    rl[rb] = ln;
                }
            }
        }
    };
    // Launches with redundancy in large blocks may have more waves than query blocks (red_waves in zp_api.hip), padded rows take
    // two, four or eight waves: a wave without a block leaves the arithmetic out; its sums of sweep 1 are never read, those of sweep 2 stay zero.
    const bool idle = (REF == 4 || PAD) && RB == 1 && (pass * NW + __builtin_amdgcn_readfirstlane(wv)) * 2 * UL >= w;
    auto sweep1_tile = [&](const char *buf, int j0, bool fresh) __attribute__((always_inline)) {
        if (idle) return;
        if (j0 + KT > u.Tv - w) sweep1_body(buf, j0, fresh, std::true_type());
        else sweep1_body(buf, j0, fresh, std::false_type());
    };
    // end of a segment: the two half-waves hold the same row, different keys; then the segments in ascending order
    float *lsum = part;                                      // [NB*32] sums beside the references in lse (part: sweep 2 only)
    auto merge = [](float &m, float &l, float m2, float l2) {
        const float mm = fmaxf(m, m2);
        l = fmaf(l, fexp2(m - mm), l2 * fexp2(m2 - mm));
        m = mm;
    };
    auto close_segment = [&](int sg) __attribute__((always_inline)) {
        // With eight waves the addresses below stay out of the tile loop (12 spilled registers with REF 2, 26 without).  Fewer waves have
        // the registers, and there the barrier makes the loop wait for its loads: 512 units of 4112 positions with the fused redundancy
        // (one wave, G 4, w 8) 1193 against 1052 us, with the separate one (d 64, two waves, blocks of 32) 176 against 170 us at 528.
        if (NW == 8) asm volatile("" ::: "memory");
#pragma unroll
        for (int rb = 0; rb < RB; rb++) {
            const float mo = __shfl_xor(rm[rb], 32), lo = __shfl_xor(rl[rb], 32);
            const int row = (wv * RB + rb) * 32 + l32;
            if (hf == 0) {
                merge(rm[rb], rl[rb], mo, lo);
                if (PH) seg[sg * (NW * RB * 32) + row] = make_float2(rm[rb], rl[rb]);
                else {
                    float m = rm[rb], l = rl[rb];
                    if (sg) {
                        m = lse[row], l = lsum[row];
                        merge(m, l, rm[rb], rl[rb]);
                    }
                    lse[row] = m;
                    lsum[row] = l;
                }
            }
            rm[rb] = -1e30f;
            rl[rb] = 0.f;
        }
    };
    if constexpr (PH != 2) {
    gload(t_lo, SetA(), ZP_NT1());
    lstore(kbuf, SetA());
    if (DEEP && t_lo + 1 < t_hi) gload(t_lo + 1, SetA(), ZP_NT1());
    __syncthreads();
    int sg = sg_lo, seg_end = (sg + 1) * ntiles / nseg;
    bool fresh = true;
    // a tile of the buffer `odd`; `next` holds the one after it (DEEP: by now, and `far` takes the one after that)
    auto turn1 = [&](int it, int odd, auto next, auto far) __attribute__((always_inline)) {
        if (it + (DEEP ? 2 : 1) < t_hi) gload(it + (DEEP ? 2 : 1), std::conditional_t<DEEP, decltype(far), decltype(next)>(), ZP_NT1());
        sweep1_tile(kbuf + odd * KTl::BYTES, it * KT, fresh);
        if (it + 1 < t_hi) lstore(kbuf + (odd ^ 1) * KTl::BYTES, next);
        fresh = it + 1 == seg_end && it + 1 < t_hi;
        if (fresh) {
            close_segment(sg++);
            seg_end = (sg + 1) * ntiles / nseg;
        }
        __syncthreads();
    };
    if constexpr (TWO) {
#pragma unroll 1
        for (int it = t_lo; it < t_hi; it += 2) {
            turn1(it, 0, SetA(), SetB());
            if (it + 1 < t_hi) turn1(it + 1, 1, std::conditional_t<DEEP, SetB, SetA>(), SetA());
        }
    } else {
#pragma unroll 1
        for (int it = t_lo; it < t_hi; it++) turn1(it, (it - t_lo) & 1, SetA(), SetB());
    }
    close_segment(sg);
    if (PH == 1) return;
    }
    if (hf == 0) {
#pragma unroll
        for (int rb = 0; rb < RB; rb++) {
            const int row = (wv * RB + rb) * 32 + l32;
            float m, l;
            if (PH) {
                const float2 s0 = seg[row];
                m = s0.x, l = s0.y;
                for (int sg = 1; sg < nseg; sg++) {
                    const float2 s = seg[sg * (NW * RB * 32) + row];
                    merge(m, l, s.x, s.y);
                }
            } else {
                m = lse[row], l = lsum[row];
            }
            lse[row] = u_col[rb] >= 0 ? m + flog2(l) : INFINITY;
        }
    }
    __syncthreads();

    // ---------------- sweep 2: S[t] = (1/w) sum_u max_g exp2(x - lse)
    // The products start from -lse / c instead of zero (the accumulator input of the first matrix instruction), so the
    // matrix cores deliver x - lse / c, the logit minus the row's normaliser in units of 1 / c: nothing is left to
    // subtract per logit.  Zero rows have lse = +inf, i.e. start and stay at -inf.
    f32x16 lrn[RB];
    int ub[RB];                                               // first window row of this half-wave's 16 slots
    const float inv_c = 1.0f / c;
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
        const int gb = wv * RB + rb;
        ub[rb] = ((pass * NW * RB + gb) * 2 + hf) * UL;
#pragma unroll
        for (int i = 0; i < 16; i++) lrn[rb][i] = -lse[gb * 32 + 4 * hf + 8 * (i >> 2) + (i & 3)] * inv_c;
    }
    // max_g exp2(x_g - lse_g) = exp2(c max_g (x_g - lse_g) / c): the maximum over the group is taken before the
    // exponential (c > 0), so a window row costs one multiply and one exp2 instead of G of each.
    auto sweep2_body = [&](const char *buf, float *pt, int j0, auto edge_tag) __attribute__((always_inline)) {
        constexpr bool edge = decltype(edge_tag)::value;
#pragma unroll
        for (int sub = 0; sub < KT / 32; sub++) {
            if (PAD && edge && j0 + sub * 32 >= u.Tv) break;  // nothing left of the sequence (unpadded: costs the eight-wave redundancy kernel 13 spills)
            f32x16 acc[RB];
            const char *kp = buf + (sub * 32 + l32) * KTl::ROW + hf * 16;
#pragma unroll
            for (int kk = 0; kk < KK; kk++) {
                const u32x4 kf = *(const u32x4 *)(kp + kk * 32);
#pragma unroll
                for (int rb = 0; rb < RB; rb++) acc[rb] = mma32<DT>(qf[rb][kk], kf, kk ? acc[rb] : lrn[rb]);
            }
            // acc[rb][i]: slot i of this half-wave, key j = j0 + sub*32 + l32
            const int j = j0 + sub * 32 + l32;
            const int thr = j - (u.Tv - w);                   // window rows u < thr come before key j: hidden
            float ps = 0.f;
#pragma unroll
            for (int rb = 0; rb < RB; rb++) {
                const f32x16 &y = acc[rb];                    // (x - lse) / c in base 2; zero rows: -inf
                if (GT) {
#pragma unroll
                    for (int ul = 0; ul < (GT ? 16 / GT : 1); ul++) {
                        float mx = y[ul * GT];
#pragma unroll
                        for (int g = 1; g < GT; g++) mx = fmaxf(mx, y[ul * GT + g]);
                        if (edge && ub[rb] + ul < thr) mx = -INFINITY;
                        ps += fexp2(mx * c);
                    }
                } else {                                      // group size known only at run time
                    float mx = -INFINITY;
                    int g = 0, ul = 0;
#pragma unroll
                    for (int i = 0; i < 16; i++) {
                        const float v = (edge && ub[rb] + ul < thr) ? -INFINITY : y[i];
                        mx = fmaxf(mx, v);
                        if (++g == G) { ps += fexp2(mx * c); mx = -INFINITY; g = 0; ul++; }
                    }
                }
            }
            ps += __shfl_xor(ps, 32);
            if (hf == 0) pt[wv * KT + sub * 32 + l32] = ps;
        }
    };
    // Redundancy (RED, b = 16): a tile holds four blocks of the live prefix, one similarity tile each.  Turning a tile
    // of products into row sums is a chain of dependent lane exchanges which the whole workgroup waits for at the tile
    // barrier, so it runs once per PAIR of tiles, all eight blocks of the pair on the eight waves at once (fewer waves
    // take several blocks in turn).  The first tile of a pair is overwritten while the second is worked on, so the
    // waves that take its blocks compute the products (four registers per block) while it is still theirs to read and
    // hold them across the barrier.  The last block, off the 16-grid of the live sequence, is done in the tail.
    float *rs_red = (float *)(smem + a.off_R);
    const float inv_len = 1.0f / (float)u.Tv;
    constexpr int PER = KT / 16, HOLD = (PER + NW - 1) / NW;  // blocks per tile; first-tile blocks one wave takes
    f32x4 gacc[HOLD];
    auto gram_first = [&](const char *buf, int j0) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < HOLD; h++) {
            const int q = wv + h * NW;
            if (q < PER && j0 + 16 * q < u.vl) gacc[h] = block_gram<ROWB / 2, KTl::ROW>(buf + 16 * q * KTl::ROW, lane);
        }
    };
    // jA: live index of the first tile (products held in gacc); bufB / jB: the second tile, jB < 0 if there is none
    auto gram_finish = [&](int jA, const char *bufB, int jB) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < HOLD; h++) {
            const int q = wv + h * NW;
            if (q < PER && jA + 16 * q < u.vl) block_row_sums(a, u, gacc[h], jA + 16 * q, inv_len, rs_red, lane);
        }
        if (jB >= 0) {
            for (int q = wv; q < 2 * PER; q += NW) {
                const int qq = q - PER;
                if (qq >= 0 && jB + 16 * qq < u.vl)
                    block_row_sums(a, u, block_gram<ROWB / 2, KTl::ROW>(bufB + 16 * qq * KTl::ROW, lane), jB + 16 * qq, inv_len, rs_red, lane);
            }
        }
    };
    auto sweep2_tile = [&](const char *buf, float *pt, int j0) __attribute__((always_inline)) {
        if (idle) return;
        if (j0 + KT > u.Tv - w) sweep2_body(buf, pt, j0, std::true_type());
        else sweep2_body(buf, pt, j0, std::false_type());
    };
    auto reduce_tile = [&](const float *pt, int j0) __attribute__((always_inline)) {         // fixed-order sum over the waves: deterministic
        if (tid < KT) {
            const int jj = j0 + tid;
            if (jj < u.Tv) {
                float s = 0.f;
#pragma unroll
                for (int v = 0; v < NW; v++) s += pt[v * KT + tid];
                const int t = live_to_pos(u, a, jj);
                if (MP && !PH) {                            // (a split call has one pass)
                    s += S[t];
                    if (pass + 1 < np) { S[t] = s; return; }
                }
                if (PH) a.scores_out[(size_t)u.unit * a.T_max + t] = s / (float)w;
                else S[t] = s / (float)w;
            }
        }
    };
    if (idle && lane < KT) part[wv * KT + lane] = part[(NW + wv) * KT + lane] = 0.f;
    // tiles are taken in DESCENDING order (tile number rt = t_hi-1-it): the keys sweep 1 read last are the ones
    // most likely to be still in L2 / Infinity Cache
    gload(t_hi - 1, SetA(), ZP_NT2());
    lstore(kbuf, SetA());
    if (DEEP && n_here > 1) gload(t_hi - 2, SetA(), ZP_NT2());
    __syncthreads();
    auto turn2 = [&](int it, int odd, auto next, auto far) __attribute__((always_inline)) {
        const int rt = t_hi - 1 - it;
        const char *buf = kbuf + odd * KTl::BYTES;
        float *pt = part + odd * (NW * KT);
        if (it + (DEEP ? 2 : 1) < n_here) gload(rt - (DEEP ? 2 : 1), std::conditional_t<DEEP, decltype(far), decltype(next)>(), ZP_NT2());
        sweep2_tile(buf, pt, rt * KT);
        if (RED) {
            if (odd) gram_finish((rt + 1) * KT, buf, rt * KT);
            else {
                gram_first(buf, rt * KT);
                if (it + 1 >= n_here) gram_finish(rt * KT, nullptr, -1);
            }
        }
        if (it + 1 < n_here) lstore(kbuf + (odd ^ 1) * KTl::BYTES, next);
        __syncthreads();
        reduce_tile(pt, rt * KT);
    };
    if constexpr (TWO) {
#pragma unroll 1
        for (int it = 0; it < n_here; it += 2) {
            turn2(it, 0, SetA(), SetB());
            if (it + 1 < n_here) turn2(it + 1, 1, std::conditional_t<DEEP, SetB, SetA>(), SetA());
        }
    } else {
#pragma unroll 1
        for (int it = 0; it < n_here; it++) turn2(it, it & 1, SetA(), SetB());
    }
    if (PH) {                                                // (one pass) the last part, which is never empty, clears what is not live
        if (part_no == a.parts - 1) {
            float *o = a.scores_out + (size_t)u.unit * a.T_max;
            for (int t = u.vl + tid; t < (u.N - 1) * a.b; t += NT) o[t] = 0.f;
            for (int t = u.T + tid; t < a.T_max; t += NT) o[t] = 0.f;
        }
        return;
    }
    __syncthreads();
    }
    unit_tail<ROWB, DT, PAD, REF, NW, ZP_WPE(NW, RB, ROWB) == 4>(a, u, smem, tbl, dst, misc);
}

template <int DT, int ROWB, bool PAD, int RB, int NW, int GT, int REF, bool MP, int PH = 0>
static hipError_t launch_one(const Args &a, int units, hipStream_t s) {
    if constexpr (REF == 0 && PH == 0) {
        if (a.phase == 1) return launch_one<DT, ROWB, PAD, RB, NW, GT, REF, MP, 1>(a, units, s);
        if (a.phase == 2) return launch_one<DT, ROWB, PAD, RB, NW, GT, REF, MP, 2>(a, units, s);
    }
    hipError_t e = allow_big_lds<unit_mfma<DT, ROWB, PAD, RB, NW, GT, REF, MP, PH>>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((unit_mfma<DT, ROWB, PAD, RB, NW, GT, REF, MP, PH>), dim3(PH ? units * a.parts : units), dim3(NW * 64), a.lds_bytes, s, a);
    return hipGetLastError();
}

// ALL_REF: the refinement variants of a geometry (REF 1, 3, and 2 and 4 where they exist); otherwise the plain one
template <int ROWB, int RB, int NW, int GT, bool ALL_REF>
static hipError_t launch_ref(const Args &a, int units, hipStream_t s) {
    if constexpr (!ALL_REF) return launch_one<1, ROWB, false, RB, NW, GT, 0, false>(a, units, s);
    else {
        if constexpr (RB == 1) if (a.ex & EX_RED_FUSED) return launch_one<1, ROWB, false, RB, NW, GT, 2, false>(a, units, s);
        if constexpr (NW >= 4) if (a.ex & EX_RED_STAGED) return launch_one<1, ROWB, false, RB, NW, GT, 4, false>(a, units, s);
        if (a.ex & EX_RED) return launch_one<1, ROWB, false, RB, NW, GT, 3, false>(a, units, s);
        return launch_one<1, ROWB, false, RB, NW, GT, 1, false>(a, units, s);
    }
}

template <int ROWB, int RB, int NW, bool ALL_REF>
static hipError_t launch_g(const Args &a, int units, hipStream_t s) {
    switch (a.G) {
        case 4: return launch_ref<ROWB, RB, NW, 4, ALL_REF>(a, units, s);
        case 5: return launch_ref<ROWB, RB, NW, 5, ALL_REF>(a, units, s);
        case 7: return launch_ref<ROWB, RB, NW, 7, ALL_REF>(a, units, s);
        case 8: return launch_ref<ROWB, RB, NW, 8, ALL_REF>(a, units, s);
        default: return launch_ref<ROWB, RB, NW, 0, ALL_REF>(a, units, s);
    }
}

// the (RB, NW) geometries of unpadded bf16 rows of one size: WIDE = 0 up to four waves, WIDE = 1 eight waves
template <int ROWB, int WIDE, bool ALL_REF>
static hipError_t launch_d(const Args &a, int units, int NW, int RB, hipStream_t s) {
    if constexpr (!WIDE) {
        if (RB == 1 && NW == 1) return launch_g<ROWB, 1, 1, ALL_REF>(a, units, s);
        if (RB == 1 && NW == 2) return launch_g<ROWB, 1, 2, ALL_REF>(a, units, s);
        if (RB == 1 && NW == 4) return launch_g<ROWB, 1, 4, ALL_REF>(a, units, s);
    } else {
        if (RB == 1 && NW == 8) return launch_g<ROWB, 1, 8, ALL_REF>(a, units, s);
        if (RB == 2 && NW == 8) return launch_g<ROWB, 2, 8, ALL_REF>(a, units, s);
        if (RB == 3 && NW == 8) return launch_g<ROWB, 3, 8, ALL_REF>(a, units, s);
        if (RB == 4 && NW == 8) return launch_g<ROWB, 4, 8, ALL_REF>(a, units, s);
    }
    return hipErrorInvalidConfiguration;
}

// every other row: padded to the next size that is instantiated, one query block per wave, up to eight waves, as many
// passes as the window needs, group size at run time
template <int DT, int ROWB>
static hipError_t launch_pad(const Args &a, int units, int NW, hipStream_t s) {
    const bool ref = (a.ex & (EX_GLOBAL | EX_POOL | EX_RED)) != 0;
    if (NW == 2) return ref ? launch_one<DT, ROWB, true, 1, 2, 0, 3, false>(a, units, s) : launch_one<DT, ROWB, true, 1, 2, 0, 0, false>(a, units, s);
    if (NW == 4 && (a.ex & EX_RED_STAGED)) return launch_one<DT, ROWB, true, 1, 4, 0, 4, false>(a, units, s);
    if (NW == 8 && (a.ex & EX_RED_STAGED)) return launch_one<DT, ROWB, true, 1, 8, 0, 4, true>(a, units, s);
    if (NW == 4) return ref ? launch_one<DT, ROWB, true, 1, 4, 0, 3, false>(a, units, s) : launch_one<DT, ROWB, true, 1, 4, 0, 0, false>(a, units, s);
    if (NW == 8) return ref ? launch_one<DT, ROWB, true, 1, 8, 0, 3, true>(a, units, s) : launch_one<DT, ROWB, true, 1, 8, 0, 0, true>(a, units, s);
    return hipErrorInvalidConfiguration;
}

}  // namespace zp
