// Device-side building blocks shared by the unit kernels: per-unit metadata checks, the
// order-preserving score key, radix top-k with the lower-position tie-break, and the
// alias-safe row mover.  A unit is one (request, layer, kv head).
#pragma once
#include "zp_kernels.h"

#include <type_traits>

#ifndef ZP_COMPACT_U
#define ZP_COMPACT_U 4
#endif

namespace zp {

// A workgroup may use the whole 160 KB of LDS; the runtime is told once per kernel (all kernels here are of one type, so the
// kernel itself is the template's parameter).
template <auto Kernel> static hipError_t allow_big_lds() {
    static hipError_t state = hipFuncSetAttribute((const void *)Kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    return state;
}

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

__device__ __forceinline__ float fexp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float flog2(float x) { return __builtin_amdgcn_logf(x); }


struct Misc {            // small LDS block at Args::off_misc
    int hist[256];
    unsigned scan[16];
    int sel_digit, sel_gt, bad, pad;
};

struct Unit {
    int unit, n, ls, h;  // request, layer inside the slab, kv head
    int N, T;            // blocks held, logical positions N*b
    int vl, Tv;          // live prefix length, live sequence length vl + b
    int k;               // keep count
    int slot;            // query slot
};

__device__ __forceinline__ int div_b(const Args &a, int t) { return a.b_shift >= 0 ? (t >> a.b_shift) : (t / a.b); }

// live index -> logical position: the live sequence is [0, vl) followed by the last block
__device__ __forceinline__ int live_to_pos(const Unit &u, const Args &a, int j) {
    return j < u.vl ? j : j + (u.N - 1) * a.b - u.vl;
}

__device__ __forceinline__ size_t row_off(const Args &a, int ls, int blk, int slot, int h) {
    return ((((size_t)ls * a.N_total + blk) * a.b + slot) * a.h_kv + h) * (size_t)a.row_bytes;
}

// logical position -> live index, -1 for a stale position
__device__ __forceinline__ int pos_to_live(const Unit &u, const Args &a, int t) {
    const int lb = (u.N - 1) * a.b;
    return t < u.vl ? t : (t >= lb ? t - lb + u.vl : -1);
}

// element index into the global-score cache F [L_slab][N_total][b][h_kv] (host-checked to fit 32 bits)
__device__ __forceinline__ unsigned f_off(const Args &a, int ls, int blk, int slot, int h) {
    return (((unsigned)ls * (unsigned)a.N_total + (unsigned)blk) * (unsigned)a.b + (unsigned)slot) * (unsigned)a.h_kv + (unsigned)h;
}

__device__ __forceinline__ void report_bad(const Args &a, int unit, int reason) {
    if (a.len_out) a.len_out[unit] = -1;
    if (atomicCAS(&a.status[0], 0, 1) == 0) {
        a.status[1] = unit;
        a.status[2] = reason;
    }
}

// Workgroup -> unit.  The hardware deals consecutive workgroups to the 8 XCDs in turn (workgroup i runs on XCD
// i mod 8, each with its own L2 and address-translation cache).  Neighbouring units are the kv heads of one
// (request, layer): they walk the same physical blocks, 256 bytes apart inside every 2 KiB token row.  The map below
// gives every XCD a contiguous range of units, so that those neighbours run side by side on one XCD.
__device__ __forceinline__ int unit_of_block(int bid, int n, int mode) {
    if (mode == 0 || n < 16) return bid;
    const int q = n >> 3, r = n & 7, x = bid & 7, i = bid >> 3;
    return x < r ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

// Inclusive scan over the 64 lanes with the operation f and its neutral element, on lane shifts of the vector ALU (a row is 16 lanes).
template <typename F> __device__ __forceinline__ unsigned wave_scan(unsigned x, unsigned neutral, F f) {
    auto from = [&](auto ctrl, auto rows) { return (unsigned)__builtin_amdgcn_update_dpp((int)neutral, (int)x, decltype(ctrl)::value, decltype(rows)::value, 0xF, false); };
    using all = std::integral_constant<int, 0xF>;
    x = f(x, from(std::integral_constant<int, 0x111>(), all()));                             // 1, 2, 4, 8 lanes below inside the row
    x = f(x, from(std::integral_constant<int, 0x112>(), all()));
    x = f(x, from(std::integral_constant<int, 0x114>(), all()));
    x = f(x, from(std::integral_constant<int, 0x118>(), all()));
    x = f(x, from(std::integral_constant<int, 0x142>(), std::integral_constant<int, 0xA>()));  // last lane of row 0 (2) into row 1 (3)
    x = f(x, from(std::integral_constant<int, 0x143>(), std::integral_constant<int, 0xC>()));  // lane 31 into rows 2 and 3
    return x;
}
__device__ __forceinline__ unsigned wave_incl_scan(unsigned x) { return wave_scan(x, 0u, [](unsigned p, unsigned q) { return p + q; }); }
__device__ __forceinline__ unsigned last_lane(unsigned x) { return (unsigned)__builtin_amdgcn_readlane((int)x, 63); }

// The unit that a workgroup takes where units differ in length and there are more of them than run at once: the workgroups, which the
// hardware starts in order, take the costliest units first, so that no long unit starts when the others are nearly done.  Costs
// fall into 256 classes, units of a class are taken in order of their number.  A unit's cost: its query blocks times its live
// entries (scoring) and eight times its kept rows (moving).  Every workgroup derives the order from arrays that nothing writes during the launch.
// 384 units of 2064 to 8208 entries (G 5, w 128, one workgroup per compute unit): 1386 us in order of their number, 972 us by cost.
__device__ inline int unit_by_cost(const Args &a, int rank, int n, Misc *misc) {
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
    const unsigned blocks = (unsigned)((a.G * a.w + 31) >> 5);
    const float scale = 256.0f / (float)(blocks * (unsigned)a.T_max + 8u * (unsigned)a.budget + 1u);
    auto cls = [&](int u) {
        const int h = u % a.h_kv, ls = (u / a.h_kv) % a.L_slab, nq = u / (a.h_kv * a.L_slab), idx = (nq * a.L + a.layer0 + ls) * a.h_kv + h;
        unsigned live = a.valid_len ? (unsigned)(a.valid_len[idx] + a.b) : (unsigned)a.num_blocks[nq] * (unsigned)a.b;
        unsigned k = a.keep ? (unsigned)a.keep[idx] : (unsigned)a.budget;
        live = live < (unsigned)a.T_max ? live : (unsigned)a.T_max;      // bad values end in some class, the unit is refused later
        k = k < (unsigned)a.budget ? k : (unsigned)a.budget;
        const int c = (int)((float)(blocks * live + 8u * k) * scale);
        return 255 - (c < 255 ? c : 255);
    };
    for (int i = tid; i < 256; i += nt) misc->hist[i] = 0;
    __syncthreads();
    for (int u = tid; u < n; u += nt) atomicAdd(&misc->hist[cls(u)], 1);
    __syncthreads();
    if (tid < 64) {
        int c[4], sum = 0;
        for (int i = 0; i < 4; i++) sum += c[i] = misc->hist[4 * lane + i];
        int before = (int)wave_incl_scan((unsigned)sum) - sum;
        if (before <= rank && rank < before + sum) {             // one lane
            int i = 0;
            while (rank >= before + c[i]) before += c[i++];
            misc->sel_digit = 4 * lane + i;
            misc->sel_gt = rank - before;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const int want = misc->sel_digit;
        int left = misc->sel_gt;
        for (int u0 = 0; u0 < n; u0 += 64) {
            const unsigned long long m = __ballot(u0 + lane < n && cls(u0 + lane < n ? u0 + lane : 0) == want);
            const int here = __popcll(m);
            if (left < here) {
                if ((m >> lane & 1) && __popcll(m & ((1ull << lane) - 1)) == left) misc->pad = u0 + lane;
                break;
            }
            left -= here;
        }
    }
    __syncthreads();
    return misc->pad;
}

// Decode the unit and check its scalar metadata (identical for every thread and every workgroup
// that looks at the unit).  Returns 0 or the reason the unit must be skipped.
// FIXED: several workgroups of a unit come through here in the launch that writes len_out, and a caller may pass valid_len or keep
// as len_out: the two values are then those an earlier launch of the call has read.
template <bool FIXED>
__device__ inline int unit_scalars(const Args &a, int unit, Unit &u) {
    u.unit = unit;
    u.h = unit % a.h_kv;
    u.ls = (unit / a.h_kv) % a.L_slab;
    u.n = unit / (a.h_kv * a.L_slab);
    // everything is requested before anything is looked at (a workgroup that waits for one value after the other starts 1 us later)
    const int idx = (u.n * a.L + a.layer0 + u.ls) * a.h_kv + u.h;
    const bool fixed = FIXED && a.unit_in, list = a.stages & STAGE_LOAD_LIST, slot = a.stages & (STAGE_SCORE | STAGE_CHECK_SLOT);
    u.N = a.num_blocks[u.n];
    const int2 in = fixed ? a.unit_in[unit] : make_int2(0, 0);
    const int vl_in = !fixed && a.valid_len ? a.valid_len[idx] : 0, k_in = list ? a.len_in[unit] : !fixed && a.keep ? a.keep[idx] : a.budget;
    u.slot = slot ? a.q_slot[u.n] : 0;
    u.T = u.N * a.b;
    u.k = fixed && !list ? in.y : k_in;
    u.vl = fixed ? in.x : a.valid_len ? vl_in : (u.N - 1) * a.b;
    u.Tv = u.vl + a.b;
    if (u.N < a.N_max || u.N > a.max_blocks) return BAD_NUM_BLOCKS;
    if (u.vl < 0 || u.vl > (u.N - 1) * a.b) return BAD_VALID_LEN;
    if (u.Tv < a.w) return BAD_VALID_LEN;
    if (list) {
        if (u.k > a.budget) return BAD_KEEP;
    } else {
        const int cap = a.budget < u.Tv ? a.budget : u.Tv;
        if (u.k < a.w || u.k > cap) return BAD_KEEP;
    }
    if (slot && (u.slot < 0 || u.slot >= a.M)) return BAD_SLOT;
    return 0;
}

// Decode the unit, check its metadata, stage the block tables in LDS (DST: that of the targets too; it is checked in any case, so that
// all launches of a call skip the same units).
// Returns false (for every thread alike) when the unit must be skipped.
template <bool FIXED = false, bool DST = true>
__device__ inline bool unit_setup(const Args &a, int unit, Unit &u, int *tbl, int *dst, Misc *misc) {
    const int tid = threadIdx.x, nt = blockDim.x, n = unit / (a.h_kv * a.L_slab);
    const int *src = a.block_table + (size_t)n * a.max_blocks, *d = a.dst_table ? a.dst_table + (size_t)n * (a.N_max - 1) : src;
    // the first entries are requested together with the scalars that say how many of them count
    const int p0 = tid < a.max_blocks ? src[tid] : 0, d0 = tid < a.N_max - 1 ? d[tid] : 0;
    int bad = unit_scalars<FIXED>(a, unit, u);
    if (tid == 0) misc->bad = bad;
    __syncthreads();
    if (!bad) {
        for (int i = tid; i < u.N; i += nt) {
            int p = i == tid ? p0 : src[i];
            if (p < 0 || p >= a.N_total) { misc->bad = BAD_BLOCK_ID; p = 0; }
            tbl[i] = p;
        }
        for (int i = tid; i < a.N_max - 1; i += nt) {
            int p = i == tid ? d0 : d[i];
            if (p < 0 || p >= a.N_total) { misc->bad = BAD_BLOCK_ID; p = 0; }
            if (DST) dst[i] = p;
        }
    }
    __syncthreads();
    bad = misc->bad;
    if (bad || u.k < 0) {           // k < 0: a unit an earlier stage already skipped
        if (bad && tid == 0) report_bad(a, unit, bad);
        return false;
    }
    return true;
}

// fp32 score -> unsigned key with the same order; NaN ranks with -inf, -0 equals +0.
__device__ __forceinline__ unsigned score_key(float f) {
    unsigned v = __float_as_uint(f);
    if ((v & 0x7fffffffu) > 0x7f800000u) v = 0xff800000u;
    if (v == 0x80000000u) v = 0u;
    return (v & 0x80000000u) ? ~v : (v | 0x80000000u);
}
#define ZP_KEY_NEG_INF 0x007fffffu
#define ZP_KEY_POS_INF 0xff800000u

// Selection (Method, compression pipeline): window +inf, stale -inf, keep the k largest, ties to the
// lower position.  keys: LDS, holds fp32 scores on entry, destroyed.  list: LDS, receives the k kept
// positions in ascending order.  Exact integer work.
// A wave owns a run of positions throughout, so what the waves tell each other is a histogram, a count, and the range of the finite
// keys.  The histograms cut that range (not the key's bits) into 256 equal bins, the next one the bin that holds the k-th largest,
// and so on until all keys of a bin are kept or its keys are equal: scores of one request differ by a few factors of two, so the top byte of
// a key is nearly constant and a histogram of it adds everything to two or three words, one lane after the other.  Two rounds are
// the usual case, with five barriers in all where four rounds of bytes took eighteen.
// 4112 positions on one compute unit: 6.4 us with 16 waves (before: 9.7), 7.3 us with eight (10.9), most of it the five passes over the
// keys; 1040 positions 3.6 us with 16 waves (5.4).
__device__ inline void select_unit(const Args &a, const Unit &u, unsigned *keys, int *list, Misc *misc) {
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), nw = nt >> 6;
    const int T = u.T, k = u.k;
    const int stale_lo = u.vl, stale_hi = (u.N - 1) * a.b;       // [vl, (N-1) b) is stale
    const int win_lo_live = u.Tv - a.w;                          // live indices >= this are the window
    const int run = ((T + nt - 1) / nt) << 6, p0 = wv * run, p1 = p0 + run < T ? p0 + run : T;   // this wave's positions
    unsigned *hist = (unsigned *)misc->hist;                     // two histograms of 256 16-bit counts (a unit has at most 65535 positions)
    unsigned lo = ~0u, hi = 0u, top = 0, fin = 0;
    for (int p = p0; p < p1; p += 64) {
        const int t = p + lane;
        unsigned key = 0u;                                       // past the end: below every key
        if (t < T) {
            if (t >= stale_lo && t < stale_hi) key = ZP_KEY_NEG_INF;
            else {
                const int j = t < stale_lo ? t : t - stale_hi + u.vl;
                key = j >= win_lo_live ? ZP_KEY_POS_INF : score_key(__uint_as_float(keys[t]));
            }
            keys[t] = key;
        }
        const bool finite = key > ZP_KEY_NEG_INF && key < ZP_KEY_POS_INF;
        top += __popcll(__ballot(key == ZP_KEY_POS_INF));
        fin += __popcll(__ballot(finite));
        if (finite) {
            lo = key < lo ? key : lo;
            hi = key > hi ? key : hi;
        }
    }
    const auto min_of = [](unsigned p, unsigned q) { return p < q ? p : q; };
    const auto max_of = [](unsigned p, unsigned q) { return p > q ? p : q; };
    lo = wave_scan(lo, ~0u, min_of);
    hi = wave_scan(hi, 0u, max_of);
    unsigned *stat = hist + 128;                                 // the second histogram's place, until the second round
    if (lane == 63) {
        stat[4 * wv] = lo;
        stat[4 * wv + 1] = hi;
        stat[4 * wv + 2] = top;
        stat[4 * wv + 3] = fin;
    }
    for (int i = tid; i < 128; i += nt) hist[i] = 0u;
    __syncthreads();
    lo = last_lane(wave_scan(lane < nw ? stat[4 * lane] : ~0u, ~0u, min_of));
    hi = last_lane(wave_scan(lane < nw ? stat[4 * lane + 1] : 0u, 0u, max_of));
    top = last_lane(wave_incl_scan(lane < nw ? stat[4 * lane + 2] : 0u));
    fin = last_lane(wave_incl_scan(lane < nw ? stat[4 * lane + 3] : 0u));
    // tau and `remaining`: keys above tau are kept, and of those equal to it `remaining`, lowest positions first
    unsigned tau, remaining = (unsigned)k;
    if (remaining <= top) tau = ZP_KEY_POS_INF;
    else if (remaining - top > fin) {
        tau = ZP_KEY_NEG_INF;
        remaining -= top + fin;
    } else {
        remaining -= top;
        int shift = hi == lo ? 0 : 24 - __builtin_clz(hi - lo);
        shift = shift > 0 ? shift : 0;
#pragma unroll 1
        for (unsigned *h = hist;; h = h == hist ? stat : hist) {
            for (int p = p0; p < p1; p += 64) {
                const unsigned key = p + lane < T ? keys[p + lane] : 0u;
                if (key >= lo && key <= hi) {
                    const unsigned bin = (key - lo) >> shift;
                    atomicAdd(&h[bin >> 1], 1u << ((bin & 1) << 4));
                }
            }
            __syncthreads();
            const unsigned w0 = h[127 - 2 * lane], w1 = h[126 - 2 * lane];   // bins 255 - 4 lane downwards
            const unsigned c[4] = {w0 >> 16, w0 & 0xffffu, w1 >> 16, w1 & 0xffffu};
            const unsigned sum = c[0] + c[1] + c[2] + c[3], incl = wave_incl_scan(sum);
            unsigned above = incl - sum, bin = 255u - 4u * lane, n = c[0];
            const unsigned long long here = __ballot(above < remaining && remaining <= incl);
#pragma unroll
            for (int i = 1; i < 4; i++)
                if (above + n < remaining) { above += n; n = c[i]; bin--; }
            const int src = __builtin_ctzll(here);
            above = (unsigned)__builtin_amdgcn_readlane((int)above, src);
            bin = (unsigned)__builtin_amdgcn_readlane((int)bin, src);
            n = (unsigned)__builtin_amdgcn_readlane((int)n, src);
            remaining -= above;
            lo += bin << shift;
            if (n == remaining) { tau = lo - 1u; remaining = 0u; break; }    // lo is above the key of -inf
            if (shift == 0) { tau = lo; break; }
            const unsigned end = lo + ((1u << shift) - 1u);
            hi = end < hi ? end : hi;
            shift = shift > 8 ? shift - 8 : 0;
            unsigned *next = h == hist ? stat : hist;            // every wave has read it: before the last barrier
            for (int i = tid; i < 128; i += nt) next[i] = 0u;
            __syncthreads();
        }
    }
    unsigned gt = 0, eq = 0;
    for (int p = p0; p < p1; p += 64) {
        const unsigned key = p + lane < T ? keys[p + lane] : 0u;
        gt += __popcll(__ballot(key > tau));
        eq += __popcll(__ballot(key == tau));
    }
    if (lane == 0) misc->scan[wv] = gt | eq << 16;
    __syncthreads();
    const unsigned before = last_lane(wave_incl_scan(lane < wv ? misc->scan[lane] : 0u));
    gt = before & 0xffffu;
    eq = before >> 16;
    for (int p = p0; p < p1; p += 64) {
        const int t = p + lane;
        const unsigned key = t < T ? keys[t] : 0u;
        const unsigned long long mg = __ballot(key > tau), me = __ballot(key == tau);
        const unsigned g = gt + __builtin_amdgcn_mbcnt_hi((unsigned)(mg >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mg, 0u));
        const unsigned e = eq + __builtin_amdgcn_mbcnt_hi((unsigned)(me >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)me, 0u));
        if (key > tau) list[g + (e < remaining ? e : remaining)] = t;
        else if (key == tau && e < remaining) list[g + e] = t;
        gt += __popcll(mg);
        eq += __popcll(me);
    }
    __syncthreads();
}

// Compaction (appendix "KV Cache Compression"): row r of the targets <- source row list[r], K and V.
// Safe in place: kept positions ascend, so list[r] >= r; ranks are taken in ascending chunks, every
// row of a chunk is in registers (loads complete) before the barrier that precedes the chunk's
// stores, and a later chunk only reads positions at or beyond its own ranks, so its loads may be
// issued while the previous chunk's stores are still on their way.  One register set: what makes this
// phase fast is the number of waves per CU that issue memory operations, not the rows a thread holds
// (a second, alternating set cost registers, i.e. resident waves, and was slower).
// Moved rows are touched once: they are loaded and stored with the non-temporal hint, so that they do not push the
// keys of the first sweep, which the second sweep reads again, out of L2 / Infinity Cache (config 2: 15.2 -> 14.7 ms).
#define ZP_NT_LOAD(p) __builtin_nontemporal_load(p)
#define ZP_NT_STORE(v, p) __builtin_nontemporal_store(v, p)

// A row is addressed by its token index `block * b + slot` inside the unit's (layer, head) plane: one 32-bit multiply-add
// per row (host-checked to fit), then one 64-bit multiply-add to the byte address.  Sixteen lanes share a row, so this
// arithmetic is replicated sixteen times per row: it is kept to a dozen instructions.
template <int U, int FM> struct RowSet {   // FM: 0 K/V only, 1 F read back from global memory, 2 F from the on-chip copy
    u32x4 kk[U], vv[U];
    unsigned dtok[U];
    bool mv[U];
    float fv[FM ? U : 1];
};

struct RowBase {
    size_t byte_base;      // byte offset of (layer, block 0, slot 0, head) plus this lane's 16-byte piece
    unsigned tok_bytes;    // bytes between consecutive tokens
    unsigned f_base, f_tok;  // the same for the global-score cache, in elements
};

// KV_APART: a chunk's K rows are all requested before its V rows (small workgroups), instead of K and V row by row.
// The two pools are separate allocations addressed by the same offsets; which order the memory system prefers depends
// on how many waves issue the requests (measured: the paper's own geometry with two-wave workgroups runs 41.8-43.3 ms per
// launch row by row and 35.2-36.8 ms apart; the 8B-like shape with eight-wave workgroups 14.55 ms against 15.16 ms).
template <int U, int FM, bool POW2, bool KV_APART>
__device__ __forceinline__ void rows_load(const Args &a, const RowBase &rb, const int *tbl, const int *dst, const int *list, const float *Sg, int k,
                                          int r0, int rpp, int rsub, bool lead, bool active, RowSet<U, FM> &s) {
    size_t vo[KV_APART ? U : 1];
#pragma unroll
    for (int i = 0; i < U; i++) {
        const int r = r0 + i * rpp + rsub;
        s.mv[i] = false;
        if (active && r < k) {
            const int t = list[r];
            unsigned st, dt;
            if (POW2) {
                st = ((unsigned)tbl[t >> a.b_shift] << a.b_shift) + (unsigned)(t & (a.b - 1));
                dt = ((unsigned)dst[r >> a.b_shift] << a.b_shift) + (unsigned)(r & (a.b - 1));
            } else {
                const int sb = t / a.b, db = r / a.b;
                st = (unsigned)tbl[sb] * (unsigned)a.b + (unsigned)(t - sb * a.b);
                dt = (unsigned)dst[db] * (unsigned)a.b + (unsigned)(r - db * a.b);
            }
            s.dtok[i] = dt;
            if (st != dt) {
                s.mv[i] = true;
                const size_t so = rb.byte_base + (size_t)st * rb.tok_bytes;
                s.kk[i] = ZP_NT_LOAD((const u32x4 *)(a.k + so));
                if (KV_APART) vo[i] = so;
                else s.vv[i] = ZP_NT_LOAD((const u32x4 *)(a.v + so));
                if (FM && lead) s.fv[i] = FM == 2 ? Sg[t] : a.F[rb.f_base + st * rb.f_tok];   // one lane per row carries the cached global score
            }
        }
    }
    if (KV_APART) {
#pragma unroll
        for (int i = 0; i < U; i++)
            if (s.mv[i]) s.vv[i] = ZP_NT_LOAD((const u32x4 *)(a.v + vo[KV_APART ? i : 0]));
    }
}

template <int U, int FM>
__device__ __forceinline__ void rows_store(const Args &a, const RowBase &rb, bool lead, const RowSet<U, FM> &s) {
#pragma unroll
    for (int i = 0; i < U; i++) {
        if (s.mv[i]) {
            const size_t dof = rb.byte_base + (size_t)s.dtok[i] * rb.tok_bytes;
            ZP_NT_STORE(s.kk[i], (u32x4 *)(a.k + dof));
            ZP_NT_STORE(s.vv[i], (u32x4 *)(a.v + dof));
            if (FM && lead) a.F[rb.f_base + s.dtok[i] * rb.f_tok] = s.fv[i];
        }
    }
}

template <int FM, bool POW2, bool KV_APART>
__device__ __forceinline__ void compact_rows(const Args &a, const Unit &u, const int *tbl, const int *dst, const int *list, const float *Sg, int k) {
    const int tid = threadIdx.x;
    const int cpr = a.row_bytes >> 4;                            // 16-byte pieces per row
    const int rpp = blockDim.x / cpr;                            // rows per pass
    const int rsub = tid / cpr, ch = (tid - rsub * cpr) << 4;
    const bool active = rsub < rpp;
    constexpr int U = ZP_COMPACT_U;
    const int CH = U * rpp;                                      // rows per chunk
    RowBase rb;
    rb.tok_bytes = (unsigned)a.h_kv * (unsigned)a.row_bytes;
    rb.byte_base = ((size_t)u.ls * a.N_total * a.b * a.h_kv + u.h) * (size_t)a.row_bytes + ch;
    rb.f_tok = (unsigned)a.h_kv;
    rb.f_base = (unsigned)u.ls * (unsigned)a.N_total * (unsigned)a.b * (unsigned)a.h_kv + (unsigned)u.h;
    RowSet<U, FM> A;
#pragma unroll 1
    for (int r0 = 0; r0 < k; r0 += CH) {
        rows_load<U, FM, POW2, KV_APART>(a, rb, tbl, dst, list, Sg, k, r0, rpp, rsub, ch == 0, active, A);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        rows_store<U, FM>(a, rb, ch == 0, A);
    }
}

template <int FM>
__device__ inline void compact_unit(const Args &a, const Unit &u, const int *tbl, const int *dst, const int *list, const float *Sg, int k) {
    if (a.b_shift < 0) compact_rows<FM, false, false>(a, u, tbl, dst, list, Sg, k);
    else if (blockDim.x <= 128) compact_rows<FM, true, true>(a, u, tbl, dst, list, Sg, k);
    else compact_rows<FM, true, false>(a, u, tbl, dst, list, Sg, k);
}

// Compaction by several workgroups per unit: each moves `slice_bytes` of every row of one pool.  Slices never touch each
// other's bytes, so every workgroup is alias-safe by the argument above, in place as well.
template <int U, bool POW2>
__device__ __forceinline__ void compact_slice(const Args &a, const Unit &u, const int *tbl, const int *dst, const int *list, int k, int slice) {
    const int tid = threadIdx.x;
    const int cpr = a.slice_bytes >> 4, rpp = blockDim.x / cpr, rsub = tid / cpr;
    const bool active = rsub < rpp;
    char *pool = (slice & 1) ? a.v : a.k;
    const size_t base = ((size_t)u.ls * a.N_total * a.b * a.h_kv + u.h) * (size_t)a.row_bytes + (size_t)(slice >> 1) * a.slice_bytes + ((tid - rsub * cpr) << 4);
    const unsigned tok_bytes = (unsigned)a.h_kv * (unsigned)a.row_bytes;
#pragma unroll 1
    for (int r0 = 0; r0 < k; r0 += U * rpp) {
        u32x4 x[U];
        unsigned dt[U];
        bool mv[U];
#pragma unroll
        for (int i = 0; i < U; i++) {
            const int r = r0 + i * rpp + rsub;
            mv[i] = false;
            if (active && r < k) {
                const int t = list[r];
                unsigned st;
                if (POW2) {
                    st = ((unsigned)tbl[t >> a.b_shift] << a.b_shift) + (unsigned)(t & (a.b - 1));
                    dt[i] = ((unsigned)dst[r >> a.b_shift] << a.b_shift) + (unsigned)(r & (a.b - 1));
                } else {
                    const int sb = t / a.b, db = r / a.b;
                    st = (unsigned)tbl[sb] * (unsigned)a.b + (unsigned)(t - sb * a.b);
                    dt[i] = (unsigned)dst[db] * (unsigned)a.b + (unsigned)(r - db * a.b);
                }
                mv[i] = st != dt[i];
                if (mv[i]) x[i] = ZP_NT_LOAD((const u32x4 *)(pool + base + (size_t)st * tok_bytes));
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
#pragma unroll
        for (int i = 0; i < U; i++)
            if (mv[i]) ZP_NT_STORE(x[i], (u32x4 *)(pool + base + (size_t)dt[i] * tok_bytes));
    }
}

// ------------------------------------------------------------------ score refinements
//
// Applied to S (LDS, indexed by logical position) right after scoring, in the paper's order (appendix
// "Combining All These Techniques"): global score -> max pooling -> S - lambda * R.

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// acc += A B over the k values that a 16-byte piece of a row holds, 32 rows times 32 columns: lane L supplies row (column)
// L%32 and the half L/32 of a 32-byte k step.  Register i of lane L holds entry (row 8*(i/4) + 4*(L/32) + i%4, column L%32).
// DT 0: four fp32 values, products and sums in fp32; 1: eight bf16 values.
template <int DT> __device__ __forceinline__ f32x16 mma32(const u32x4 &x, const u32x4 &y, f32x16 acc) {
    if (DT) return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), acc, 0, 0, 0);
    const f32x4 xf = __builtin_bit_cast(f32x4, x), yf = __builtin_bit_cast(f32x4, y);
#pragma unroll
    for (int e = 0; e < 4; e++) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(xf[e], yf[e], acc, 0, 0, 0);
    return acc;
}

// the 16-byte pieces one lane supplies of a row (see mma32); zeros past the pool's row
template <int ROWB, bool PAD> __device__ __forceinline__ void load_row(const char *row, int hf, int row_bytes, u32x4 (&f)[ROWB / 32]) {
#pragma unroll
    for (int kk = 0; kk < ROWB / 32; kk++) {
        f[kk] = u32x4{0u, 0u, 0u, 0u};
        if (!PAD || kk * 32 + hf * 16 < row_bytes) f[kk] = *(const u32x4 *)(row + kk * 32 + hf * 16);
    }
}

// workgroup-wide max and sum of per-thread values, same result in every thread, fixed order
__device__ inline float block_reduce(float v, bool is_max, Misc *misc) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const float o = __shfl_xor(v, off);
        v = is_max ? fmaxf(v, o) : v + o;
    }
    float *sc = (float *)misc->scan;
    __syncthreads();
    if (lane == 0) sc[wv] = v;
    __syncthreads();
    v = sc[0];
    for (int i = 1; i < nw; i++) v = is_max ? fmaxf(v, sc[i]) : v + sc[i];
    return v;
}

// Lightning redundancy, any element type and block size (appendix "Lightning Redundancy"): one thread per
// live key computes its row of the within-block cosine-similarity matrix on the vector ALUs.  The matrix is
// symmetric, so the row of key r is also column r: the thread finds the last entry above p of its column
// there and publishes (row, value); row sums are corrected after a barrier.  rs[j] receives the row sum / Tv.
template <int DT>
__device__ inline void redundancy_valu(const Args &a, const Unit &u, const int *tbl, float *rs, float *inv, int *zl, float *zv) {
    const int tid = threadIdx.x, nt = blockDim.x;
    const int n_el = a.d;
    for (int j = tid; j < u.Tv; j += nt) {
        const int t = live_to_pos(u, a, j), blk = div_b(a, t);
        const char *kr = a.k + row_off(a, u.ls, tbl[blk], t - blk * a.b, u.h);
        float n2 = 0.f;
        for (int e = 0; e < n_el; e++) {
            const float x = DT ? __uint_as_float((unsigned)((const unsigned short *)kr)[e] << 16) : ((const float *)kr)[e];
            n2 = fmaf(x, x, n2);
        }
        inv[j] = n2 > 0.f ? 1.0f / sqrtf(n2) : 0.f;
    }
    __syncthreads();
    for (int j = tid; j < u.Tv; j += nt) {
        const int t = live_to_pos(u, a, j), blk = div_b(a, t), r = t - blk * a.b;
        const char *kb = a.k + row_off(a, u.ls, tbl[blk], 0, u.h);
        const size_t slot_bytes = (size_t)a.h_kv * a.row_bytes;
        const char *kr = kb + r * slot_bytes;
        const float ir = inv[j];
        float acc = 0.f, lastv = 0.f;
        int last = -1;
        for (int c = 0; c < a.b; c++) {
            const int jc = pos_to_live(u, a, blk * a.b + c);
            float val = 0.f;
            if (c != r && jc >= 0) {
                const float ic = inv[jc];
                if (ir != 0.f && ic != 0.f) {
                    const char *kc = kb + c * slot_bytes;
                    float dot = 0.f;
                    for (int e = 0; e < n_el; e++) {
                        const float x = DT ? __uint_as_float((unsigned)((const unsigned short *)kr)[e] << 16) : ((const float *)kr)[e];
                        const float y = DT ? __uint_as_float((unsigned)((const unsigned short *)kc)[e] << 16) : ((const float *)kc)[e];
                        dot = fmaf(x, y, dot);
                    }
                    val = dot * (ir * ic);
                }
            }
            acc += val;
            if (val > a.p_thr) { last = c; lastv = val; }
        }
        rs[j] = acc;
        zl[j] = last;
        zv[j] = lastv;
    }
    __syncthreads();
    const float inv_len = 1.0f / (float)u.Tv;
    for (int j = tid; j < u.Tv; j += nt) {
        const int t = live_to_pos(u, a, j), blk = div_b(a, t), r = t - blk * a.b;
        float corr = 0.f;
        for (int c = 0; c < a.b; c++) {
            const int jc = pos_to_live(u, a, blk * a.b + c);
            if (jc >= 0 && zl[jc] == r) corr += zv[jc];
        }
        rs[j] = (rs[j] - corr) * inv_len;
    }
    __syncthreads();
}

// The same on the matrix cores for a block size that divides 32: K_g K_g^T of 32 consecutive logical positions
// (32/b whole blocks) is one 32x32 tile of the matrix cores, both operands being the same register fragments.
// Lane L, register i holds the entry (row 8*(i/4) + 4*(L/32) + i%4, column L%32); only entries whose row and
// column lie in the same block are used.  A wave owns a group; its 96 words of LDS hold the inverse norms and
// the (row, value) of the entry zeroed in every column.
// last_only: only the rows of the last block are produced (the live prefix was done from the key tiles of sweep 2).
template <int ROWB, int DT, bool PAD>
__device__ inline void redundancy_mfma(const Args &a, const Unit &u, const int *tbl, float *rs, float *wave_scratch, bool last_only) {
    constexpr int KK = ROWB / 32;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nw = blockDim.x >> 6, l32 = lane & 31, hf = lane >> 5;
    float *inv = wave_scratch + wv * 96, *zv = inv + 64;
    int *zr = (int *)(inv + 32);
    const int ngroups = (u.T + 31) >> 5;
    const int stale_hi = (u.N - 1) * a.b;
    const float inv_len = 1.0f / (float)u.Tv;
    const int cblk = l32 >> a.b_shift;                              // block of this lane's column inside the group
    const int dgi = ((l32 >> 3) << 2) | (l32 & 3);              // register that holds the diagonal entry ...
    const bool dg_mine = hf == ((l32 >> 2) & 1);                // ... in this half of the wave
    // groups of this wave in ascending order, wholly stale ones skipped; the fragments of the next group are
    // requested before the current one is worked on
    auto next_group = [&](int g) {
        while (g < ngroups && g * 32 + 32 <= stale_hi && (last_only || g * 32 >= u.vl)) g += nw;
        return g;
    };
    auto live_of = [&](int g) {
        const int p = g * 32 + l32;
        if (p >= u.T || (last_only && p < stale_hi)) return -1;
        return pos_to_live(u, a, p);
    };
    auto load_group = [&](int g, u32x4 (&kf)[KK]) {
        const int pc = live_of(g) >= 0 ? g * 32 + l32 : u.T - 1;  // rows that are not live read a valid row and are masked
        const int blk = div_b(a, pc);
        load_row<ROWB, PAD>(a.k + row_off(a, u.ls, tbl[blk], pc - blk * a.b, u.h), hf, a.row_bytes, kf);
    };
    u32x4 kf[KK], kn[KK];
    int g = next_group(wv);
    if (g < ngroups) load_group(g, kf);
#pragma unroll 1
    while (g < ngroups) {
        const int gn = next_group(g + nw);
        if (gn < ngroups) load_group(gn, kn);
        const int jl = live_of(g);
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; i++) acc[i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; kk++) acc = mma32<DT>(kf[kk], kf[kk], acc);
        float dg = 0.f;
#pragma unroll
        for (int i = 0; i < 16; i++) dg = i == dgi ? acc[i] : dg;
        if (dg_mine) inv[l32] = (jl >= 0 && dg > 0.f) ? 1.0f / sqrtf(dg) : 0.f;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // LDS serves a wave's accesses in order
        const float ic = inv[l32];
        float csum = 0.f, lastv = 0.f;
        int last = -1;
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int row = 8 * (i >> 2) + 4 * hf + (i & 3);
            const float ir = inv[row];
            const bool in_blk = (row >> a.b_shift) == cblk;
            float val = 0.f;
            if (in_blk && row != l32 && ir != 0.f && ic != 0.f) val = acc[i] * (ir * ic);
            csum += val;
            if (in_blk && val > a.p_thr) { last = row; lastv = val; }   // rows ascend with i
        }
        const int o_last = __shfl_xor(last, 32);
        const float o_lastv = __shfl_xor(lastv, 32), o_csum = __shfl_xor(csum, 32);
        const float colsum = hf ? o_csum + csum : csum + o_csum;  // same bits in both halves
        if (hf == 0) {
            zr[l32] = last > o_last ? last : o_last;
            zv[l32] = last > o_last ? lastv : o_lastv;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        // symmetric matrix: the sum of row r before zeroing is the sum of column r; take off what was zeroed in row r
        if (hf == 0 && jl >= 0) {
            float corr = 0.f;
            const int c0 = cblk * a.b;
            for (int c = c0; c < c0 + a.b; c++)
                if (zr[c] == l32) corr += zv[c];
            rs[jl] = (colsum - corr) * inv_len;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // the next group reuses the wave's scratch
#pragma unroll
        for (int kk = 0; kk < KK; kk++) kf[kk] = kn[kk];
        g = gn;
    }
    __syncthreads();
}

// Other block sizes on the matrix cores (those that redundancy_staged does not take).  The similarity matrix of one block is cut into 32-column groups; a wave owns a
// group and goes through the block's 32-row groups, own rows first, each one 32x32 tile (lane L holds column L%32, 16 of the
// rows).  A column's sum and the last row above p stay in its two lanes over all tiles; the matrix is symmetric, so the sum of
// column r is the sum of row r before zeroing, and what was zeroed in row r is taken off in a pass of its own (waves go
// through the columns that have a zeroed entry only).  inv, zr, zv: LDS, by logical position: inverse norm (0: not live),
// row zeroed in the column (-1: none) and its value.
// Row fragments come from L2 (the unit's keys have just been swept), with few waves (FEW) those of the next tile requested
// before the current tile is worked on.  Before, one thread per key took b dot products one element at a time: 345 ms per launch for 1152 units
// of 2304 positions in blocks of 256 (d 128, bf16), now 1.71 ms.  Waves of 128 registers (TIGHT) hold the column
// group only, rows of 192 and 256 bytes come piece by piece (512 units of 4112 positions, d 128, w 64: blocks of 64 1065 -> 1007 us,
// of 256 1540 -> 1522 us against both held and 21 registers spilled; with 256 registers holding both is the faster way: 80 units of 3144
// in blocks of 24, w 69, 372 against 403 us).
template <int ROWB, int DT, bool PAD, bool FEW, bool TIGHT>
__device__ inline void redundancy_blocks(const Args &a, const Unit &u, const int *tbl, float *rs, float *inv, int *zr, float *zv) {
    constexpr int KK = ROWB / 32;
    constexpr bool HOLD = ROWB <= 256;                           // a column group's fragments fit the registers ...
    constexpr bool HOLD_ROWS = HOLD && (!TIGHT || ROWB <= 128);  // ... beside those of a row group (two with FEW)
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nw = blockDim.x >> 6, l32 = lane & 31, hf = lane >> 5;
    const int b = a.b, stale_hi = (u.N - 1) * b;
    const float inv_len = 1.0f / (float)u.Tv;
    auto row_ptr = [&](int p) {                                  // p: a logical position of the request
        const int blk = div_b(a, p);
        return a.k + row_off(a, u.ls, tbl[blk], p - blk * b, u.h);
    };
    f32x16 zero16;
#pragma unroll
    for (int i = 0; i < 16; i++) zero16[i] = 0.f;
    auto gram_stream = [&](const char *rp, const char *cp) {     // long rows: both operands a few pieces at a time
        f32x16 acc = zero16;
#pragma unroll 4
        for (int kk = 0; kk < KK; kk++) {
            u32x4 x = {0u, 0u, 0u, 0u}, y = {0u, 0u, 0u, 0u};
            if (!PAD || kk * 32 + hf * 16 < a.row_bytes) {
                x = *(const u32x4 *)(rp + kk * 32 + hf * 16);
                y = *(const u32x4 *)(cp + kk * 32 + hf * 16);
            }
            acc = mma32<DT>(x, y, acc);
        }
        return acc;
    };
    auto gram_rows = [&](const char *rp, const u32x4 (&col)[HOLD ? KK : 1]) {
        f32x16 acc = zero16;
#pragma unroll
        for (int kk = 0; kk < (HOLD ? KK : 0); kk++) {
            u32x4 x = {0u, 0u, 0u, 0u};
            if (!PAD || kk * 32 + hf * 16 < a.row_bytes) x = *(const u32x4 *)(rp + kk * 32 + hf * 16);
            acc = mma32<DT>(x, col[kk], acc);
        }
        return acc;
    };
    // inverse norms from the diagonals of 32x32 tiles of consecutive positions
    const int dgi = ((l32 >> 3) << 2) | (l32 & 3);
    const bool dg_mine = hf == ((l32 >> 2) & 1);
    for (int g = wv; g * 32 < u.T; g += nw) {
        const int p = g * 32 + l32;
        const bool live = p < u.T && pos_to_live(u, a, p) >= 0;
        if (g * 32 < u.vl || g * 32 + 32 > stale_hi) {
            const char *rp = row_ptr(live ? p : u.T - 1);
            f32x16 acc = zero16;
            if constexpr (HOLD) {
                u32x4 f[KK];
                load_row<ROWB, PAD>(rp, hf, a.row_bytes, f);
#pragma unroll
                for (int kk = 0; kk < KK; kk++) acc = mma32<DT>(f[kk], f[kk], acc);
            } else acc = gram_stream(rp, rp);
            float dg = 0.f;
#pragma unroll
            for (int i = 0; i < 16; i++) dg = i == dgi ? acc[i] : dg;
            if (dg_mine && p < u.T) inv[p] = (live && dg > 0.f) ? 1.0f / sqrtf(dg) : 0.f;
        } else if (hf == 0) inv[p] = 0.f;
    }
    __syncthreads();

    const int ncg = (b + 31) >> 5, items = u.N * ncg;
    auto wanted = [&](int it) {                                  // next column group of this wave that has a live key
        for (; it < items; it += nw) {
            const int blk = it / ncg, p0 = blk * b + (it - blk * ncg) * 32;
            if (p0 < u.vl || blk == u.N - 1) break;
        }
        return it;
    };
    auto load_group = [&](int it, int step, u32x4 (&f)[HOLD_ROWS ? KK : 1]) {   // rows of the group `step` places after the item's own
        const int blk = it / ncg, cg = it - blk * ncg, rg = cg + step < ncg ? cg + step : cg + step - ncg;
        const int r = rg * 32 + l32;
        const char *rp = row_ptr(blk * b + (r < b ? r : b - 1));
        if constexpr (HOLD_ROWS) load_row<ROWB, PAD>(rp, hf, a.row_bytes, f);
        return rp;
    };
    u32x4 cur[HOLD_ROWS ? KK : 1], nxt[HOLD_ROWS ? KK : 1], col[HOLD ? KK : 1];
    int it = wanted(wv);
    const char *cp = nullptr, *rp = nullptr, *rpn = nullptr;
    if (it < items) rp = load_group(it, 0, cur);
#pragma unroll 1
    while (it < items) {
        const int itn = wanted(it + nw);
        const int blk = it / ncg, cg = it - blk * ncg, c = cg * 32 + l32;
        const float *binv = inv + blk * b;
        const float ic = c < b ? binv[c] : 0.f;
        float csum = 0.f, lastv = 0.f;
        int last = -1;
        cp = rp;
        if constexpr (HOLD_ROWS) {
#pragma unroll
            for (int kk = 0; kk < KK; kk++) col[kk] = cur[kk];
        } else if constexpr (HOLD) load_row<ROWB, PAD>(cp, hf, a.row_bytes, col);
#pragma unroll 1
        for (int step = 0; step < ncg; step++) {
            if (FEW) {
                if (step + 1 < ncg) rpn = load_group(it, step + 1, nxt);
                else if (itn < items) rpn = load_group(itn, 0, nxt);
            }
            f32x16 acc = zero16;
            if constexpr (HOLD_ROWS) {
#pragma unroll
                for (int kk = 0; kk < KK; kk++) acc = mma32<DT>(cur[kk], col[kk], acc);
            } else if constexpr (HOLD) acc = gram_rows(rp, col);
            else acc = gram_stream(rp, cp);
            const int rg = cg + step < ncg ? cg + step : cg + step - ncg;
            const int r0 = rg * 32 + 4 * hf;                     // register i: row r0 + 8*(i/4) + i%4
            float mx = -INFINITY;
#pragma unroll
            for (int i = 0; i < 16; i++) {
                const int r = r0 + 8 * (i >> 2) + (i & 3);
                const float ir = r < b ? binv[r] : 0.f;
                const float v = (ir != 0.f && ic != 0.f && r != c) ? acc[i] * (ir * ic) : 0.f;
                acc[i] = v;
                csum += v;
                mx = fmaxf(mx, v);
            }
            if (__any(mx > a.p_thr)) {
#pragma unroll
                for (int i = 0; i < 16; i++) {
                    const int r = r0 + 8 * (i >> 2) + (i & 3);
                    if (acc[i] > a.p_thr && r > last && r < b) { last = r; lastv = acc[i]; }
                }
            }
            if (FEW) {
                rp = rpn;
                if constexpr (HOLD_ROWS) {
#pragma unroll
                    for (int kk = 0; kk < KK; kk++) cur[kk] = nxt[kk];
                }
            } else if (step + 1 < ncg) rp = load_group(it, step + 1, cur);
            else if (itn < items) rp = load_group(itn, 0, cur);
        }
        const int o_last = __shfl_xor(last, 32);
        const float o_lastv = __shfl_xor(lastv, 32), o_csum = __shfl_xor(csum, 32);
        if (hf == 0 && c < b) {
            const int p = blk * b + c, j = pos_to_live(u, a, p);
            if (o_last > last) { last = o_last; lastv = o_lastv; }
            zr[p] = j >= 0 ? last : -1;
            zv[p] = lastv;
            if (j >= 0) rs[j] = csum + o_csum;
        }
        it = itn;
    }
    __syncthreads();

    for (int w0 = wv; w0 < u.N * ((b + 63) >> 6); w0 += nw) {     // 64 rows of one block per wave
        const int nr = (b + 63) >> 6, blk = w0 / nr, r = (w0 - blk * nr) * 64 + lane;
        const int j = r < b ? pos_to_live(u, a, blk * b + r) : -1;
        if (!__any(j >= 0)) continue;
        float corr = 0.f;
        for (int c0 = 0; c0 < b; c0 += 64) {
            int row = -1;
            float val = 0.f;
            // column groups without a live key were not visited
            if (c0 + lane < b && pos_to_live(u, a, blk * b + c0 + lane) >= 0) { row = zr[blk * b + c0 + lane]; val = zv[blk * b + c0 + lane]; }
            unsigned long long m = __ballot(row >= 0);
            while (m) {                                          // columns ascend
                const int l = __builtin_ctzll(m);
                m &= m - 1;
                const float v = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, val), l));
                corr += __builtin_amdgcn_readlane(row, l) == r ? v : 0.f;
            }
        }
        if (j >= 0) rs[j] = (rs[j] - corr) * inv_len;
    }
    __syncthreads();
}

// Large blocks, block by block: every wave holds the fragments of up to CW 32-column groups of the block in registers, the block's rows
// go through LDS (SR at a time, the next ones requested before the current ones are worked on) and all waves read their row fragments
// from there.  Fragments straight from memory touch 32 rows for 32 bytes each, and every row group was fetched once per column
// group: 512 units of 4352 positions in blocks of 256 (d 128, w 64) 1518 -> 859 us, of 4224 in blocks of 128 1148 -> 845.  Four column groups
// per wave need more than 256 registers, two with 256-byte rows fit them.
// A similarity is (product * 1 / row norm) * 1 / column norm; the column's factor is taken out of the sum.  Rows that count as zero (norm 0 or
// infinite, not live) are staged as zeros, columns that do are left out at the end.  inv, zr, zv: LDS, by row of the block.
template <int ROWB, int DT, bool PAD, int NW, int CW>
__device__ inline void redundancy_staged(const Args &a, const Unit &u, const int *tbl, float *rs, float *inv, int *zr, float *zv, char *stage) {
    constexpr int KK = ROWB / 32, CPR = ROWB / 16, SR = mfma_tile_keys(ROWB), ROW = ROWB + 16, NT = NW * 64, LPT = (SR * CPR + NT - 1) / NT;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hf = lane >> 5;
    const int b = a.b, ncg = (b + 31) >> 5;
    const float inv_len = 1.0f / (float)u.Tv;
    const size_t slot_bytes = (size_t)a.h_kv * a.row_bytes;
    const int dgi = ((l32 >> 3) << 2) | (l32 & 3);              // register that holds the diagonal entry ...
    const bool dg_mine = hf == ((l32 >> 2) & 1);                // ... in this half of the wave
    f32x16 zero16;
#pragma unroll
    for (int i = 0; i < 16; i++) zero16[i] = 0.f;
    u32x4 col[CW][KK], st[LPT];
#pragma unroll 1
    for (int blk = 0; blk < u.N; blk++) {
        const int live = blk == u.N - 1 ? b : u.vl - blk * b < b ? u.vl - blk * b : b, j0 = blk == u.N - 1 ? u.vl : blk * b;
        if (live <= 0) continue;
        const char *base = a.k + row_off(a, u.ls, tbl[blk], 0, u.h);
        auto load_cols = [&](int g0) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < CW; c++) {
                const int r = (g0 + wv + c * NW) * 32 + l32;
                load_row<ROWB, PAD>(base + (r < b ? r : b - 1) * slot_bytes, hf, a.row_bytes, col[c]);
            }
        };
        // inverse norms from the diagonals
#pragma unroll 1
        for (int g0 = 0; g0 < ncg; g0 += NW * CW) {
            load_cols(g0);
#pragma unroll
            for (int c = 0; c < CW; c++) {
                const int r = (g0 + wv + c * NW) * 32 + l32;
                f32x16 acc = zero16;
#pragma unroll
                for (int kk = 0; kk < KK; kk++) acc = mma32<DT>(col[c][kk], col[c][kk], acc);
                float dg = 0.f;
#pragma unroll
                for (int i = 0; i < 16; i++) dg = i == dgi ? acc[i] : dg;
                if (dg_mine && r < ncg * 32) inv[r] = (r < live && dg > 0.f) ? 1.0f / sqrtf(dg) : 0.f;
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int g0 = 0; g0 < ncg; g0 += NW * CW) {
            if (ncg > NW * CW) load_cols(g0);
            float ic[CW], csum[CW], lastv[CW];
            int last[CW];
#pragma unroll
            for (int c = 0; c < CW; c++) {
                const int g = g0 + wv + c * NW;
                ic[c] = g < ncg ? inv[g * 32 + l32] : 0.f;
                csum[c] = lastv[c] = 0.f;
                last[c] = -1;
            }
            auto gload = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < LPT; i++) {
                    const int pc = tid + i * NT, row = pc / CPR, off = (pc - row * CPR) * 16, r = r0 + row < b ? r0 + row : b - 1;
                    st[i] = u32x4{0u, 0u, 0u, 0u};
                    if ((SR * CPR % NT == 0 || row < SR) && (!PAD || off < a.row_bytes)) st[i] = *(const u32x4 *)(base + r * slot_bytes + off);
                }
            };
            gload(0);
#pragma unroll 1
            for (int r0 = 0; r0 < b; r0 += SR) {
                __syncthreads();                                 // the rows before these have been read
#pragma unroll
                for (int i = 0; i < LPT; i++) {
                    const int pc = tid + i * NT, row = pc / CPR;
                    const float n = r0 + row < ncg * 32 ? inv[r0 + row] : 0.f;
                    if (SR * CPR % NT == 0 || row < SR) *(u32x4 *)(stage + row * ROW + (pc - row * CPR) * 16) = n != 0.f ? st[i] : u32x4{0u, 0u, 0u, 0u};
                }
                __syncthreads();
                if (r0 + SR < b) gload(r0 + SR);
#pragma unroll 1
                for (int rg = r0; rg < r0 + SR && rg < b; rg += 32) {
                    f32x4 ir[4];
#pragma unroll
                    for (int q = 0; q < 4; q++) ir[q] = *(const f32x4 *)(inv + rg + 4 * hf + 8 * q);
                    const char *rp = stage + (rg - r0 + l32) * ROW + hf * 16;
#pragma unroll
                    for (int c = 0; c < CW; c++) {
                        const int g = g0 + wv + c * NW;
                        if (g >= ncg) break;
                        f32x16 acc = zero16;
#pragma unroll
                        for (int kk = 0; kk < KK; kk++) acc = mma32<DT>(*(const u32x4 *)(rp + kk * 32), col[c][kk], acc);
                        if (g * 32 == rg) {
#pragma unroll
                            for (int i = 0; i < 16; i++) acc[i] = dg_mine && i == dgi ? 0.f : acc[i];
                        }
                        float mx = -INFINITY;
#pragma unroll
                        for (int i = 0; i < 16; i++) {
                            acc[i] *= ir[i >> 2][i & 3];
                            csum[c] += acc[i];
                            mx = fmaxf(mx, acc[i]);
                        }
                        if (__any((ic[c] != 0.f ? mx * ic[c] : 0.f) > a.p_thr)) {
#pragma unroll
                            for (int i = 0; i < 16; i++) {       // rows ascend with i
                                const int r = rg + 4 * hf + 8 * (i >> 2) + (i & 3);
                                const float v = ic[c] != 0.f ? acc[i] * ic[c] : 0.f;
                                if (v > a.p_thr && r < b) { last[c] = r; lastv[c] = v; }
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < CW; c++) {
                const int r = (g0 + wv + c * NW) * 32 + l32;
                const int o_last = __shfl_xor(last[c], 32);
                const float o_lastv = __shfl_xor(lastv[c], 32), sum = csum[c] + __shfl_xor(csum[c], 32);
                if (hf == 0 && r < b) {
                    zr[r] = r < live ? (o_last > last[c] ? o_last : last[c]) : -1;
                    zv[r] = o_last > last[c] ? o_lastv : lastv[c];
                    if (r < live) rs[j0 + r] = ic[c] != 0.f ? sum * ic[c] : 0.f;
                }
            }
        }
        __syncthreads();
        // symmetric matrix: the sum of column r is the sum of row r before zeroing; take off what was zeroed in row r
        for (int r0 = wv * 64; r0 < live; r0 += NT) {
            const int r = r0 + lane;
            float corr = 0.f;
            for (int c0 = 0; c0 < b; c0 += 64) {
                const int row = c0 + lane < b ? zr[c0 + lane] : -1;
                const float val = c0 + lane < b ? zv[c0 + lane] : 0.f;
                unsigned long long m = __ballot(row >= 0);
                while (m) {                                      // columns ascend
                    const int l = __builtin_ctzll(m);
                    m &= m - 1;
                    const float v = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, val), l));
                    corr += __builtin_amdgcn_readlane(row, l) == r ? v : 0.f;
                }
            }
            if (r < live) rs[j0 + r] = (rs[j0 + r] - corr) * inv_len;
        }
        __syncthreads();
    }
}

// Block size 16, live prefix: the similarity matrix of one block from the key tile that sweep 2 holds in LDS anyway
// (rows `rows`, ROWB bytes apart, 16 keys of one block).  K_blk K_blk^T is one 16x16 tile of the matrix cores
// (v_mfma_f32_16x16x32_bf16, both operands the same fragments: lane L supplies key L%16, elements 8*(L/16).. of every
// 32-wide step; register i of lane L holds entry (row 4*(L/16) + i, column L%16)).  j_first: live index of the
// block's first key; rows at or beyond the live prefix are not live.  Everything after the products stays in
// registers: norms and the column rule travel by lane permutes, the row sums by adds across the 16 lanes of a row group
// (this step sits inside the tile loop of sweep 2, where every wait on LDS holds up the whole workgroup's barrier).
// It comes in two parts so that the caller can take the products while the key rows are in LDS and finish later.
// sum over the 16 lanes that share lane/16, the same bits in all of them (a + b and b + a at every step)
__device__ __forceinline__ float row16_sum(float v) {
    auto dpp = [](float x, auto ctrl) { return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xF, 0xF, true)); };
    v += dpp(v, std::integral_constant<int, 0xB1>());      // lane ^ 1 inside every quad
    v += dpp(v, std::integral_constant<int, 0x4E>());      // lane ^ 2
    v += dpp(v, std::integral_constant<int, 0x141>());     // mirror inside every half row: the other quad's sum
    v += dpp(v, std::integral_constant<int, 0x140>());     // mirror inside the row: the other half's sum
    return v;
}

// the products: needs the key rows in LDS only here
template <int D, int ROWB>
__device__ __forceinline__ f32x4 block_gram(const char *rows, int lane) {
    const int c = lane & 15, g = lane >> 4;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const char *kp = rows + c * ROWB + g * 16;
#pragma unroll
    for (int kk = 0; kk < D / 32; kk++) {
        const bf16x8 f = *(const bf16x8 *)(kp + kk * 64);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, f, acc, 0, 0, 0);
    }
    return acc;
}

// from the products to the row sums of the block's live keys: rs[j] = (row sum with the column rule applied) / Tv
__device__ __forceinline__ void block_row_sums(const Args &a, const Unit &u, const f32x4 acc, int j_first, float inv_len, float *rs, int lane) {
    const int c = lane & 15, g = lane >> 4;
    // inverse norm of key c from the diagonal entry (c, c), which sits in lane (column c, group c/4), register c%4
    float dg = acc[0];
#pragma unroll
    for (int i = 1; i < 4; i++) dg = i == (c & 3) ? acc[i] : dg;
    const float own = (j_first + c < u.vl && dg > 0.f) ? 1.0f / sqrtf(dg) : 0.f;    // meaningful in the diagonal lanes only
    const float ic = __shfl(own, (c >> 2) * 16 + c);
    float val[4];
    int last = -1;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const int row = 4 * g + i;
        const float ir = __shfl(ic, g * 16 + row);              // the lane of column `row` in this group holds its inverse norm
        float v = 0.f;
        if (row != c && ir != 0.f && ic != 0.f) v = acc[i] * (ir * ic);
        val[i] = v;
        if (v > a.p_thr) last = row;                            // rows ascend with i
    }
    // the four lanes of a column (rows 0-3, 4-7, 8-11, 12-15) agree on the last entry above p ...
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
        const int ol = __shfl_xor(last, off);
        last = ol > last ? ol : last;
    }
    // ... it is zeroed where it lives, and every row is summed over the 16 columns
    float mine = 0.f;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const float s = row16_sum(4 * g + i == last ? 0.f : val[i]);
        mine = i == c ? s : mine;
    }
    if (c < 4 && j_first + 4 * g + c < u.vl) rs[j_first + 4 * g + c] = mine * inv_len;
}

// ROWB > 0: called from the matrix-core kernel for rows of up to ROWB bytes; ROWB = 0: generic kernel.  Element type DT.
// REF 1: global score and pooling; REF 2: a launch whose similarity tiles came from sweep 2 (EX_RED_FUSED); REF 4: redundancy of large
// blocks (EX_RED_STAGED); REF 3: any other with redundancy.
template <int ROWB, int DT, bool PAD, int REF, int NW, bool TIGHT>
__device__ inline void refine_unit(const Args &a, const Unit &u, char *smem, const int *tbl, Misc *misc) {
    const int tid = threadIdx.x, nt = blockDim.x;
    float *S = (float *)(smem + a.off_S);
    float *tmp = (float *)(smem + a.off_union);
    const bool hist = a.compressed && a.compressed[u.n] != 0;
    if (a.ex & EX_GLOBAL) {
        float *Sg = (float *)(smem + a.off_G);
        for (int j = tid; j < u.Tv; j += nt) {
            const int t = live_to_pos(u, a, j), blk = div_b(a, t);
            const unsigned fi = f_off(a, u.ls, tbl[blk], t - blk * a.b, u.h);
            float v = S[t];
            if (hist && t < u.vl) {                              // the last block holds new tokens: no history
                const float old = a.alpha * a.F[fi];
                if (old > v) v = old;
            }
            a.F[fi] = v;
            S[t] = v;
            if (a.ex & EX_MOVE_F_LDS) Sg[t] = v;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // compaction may write the same cache entries later
        __syncthreads();
    }
    if ((a.ex & EX_POOL) && !((a.ex & EX_POOL_FIRST) && hist)) {
        const int r = a.pool_r;
        for (int j = tid; j < u.Tv; j += nt) {
            const int lo = j - r < 0 ? 0 : j - r, hi = j + r > u.Tv - 1 ? u.Tv - 1 : j + r;
            float m = -INFINITY;
            for (int q = lo; q <= hi; q++) {
                const float x = S[live_to_pos(u, a, q)];
                if (x > m) m = x;
            }
            tmp[j] = m;
        }
        __syncthreads();
        for (int j = tid; j < u.Tv; j += nt) S[live_to_pos(u, a, j)] = tmp[j];
        __syncthreads();
    }
    if constexpr (REF != 1) if (a.ex & EX_RED) {
        if constexpr (REF == 2) {                                // the live prefix was done from the key tiles of sweep 2
            tmp = (float *)(smem + a.off_R);
            redundancy_mfma<ROWB, DT, PAD>(a, u, tbl, tmp, tmp + a.T_max, true);
        } else if constexpr (REF == 4) {
            const int rows = (a.b + 31) & ~31;
            float *inv = tmp + ((a.T_max + 3) & ~3);
            constexpr int CW = ROWB > 256 || TIGHT ? 1 : ROWB > 128 ? 2 : NW > 4 ? 1 : 4;
            redundancy_staged<ROWB, DT, PAD, NW, CW>(a, u, tbl, tmp, inv, (int *)(inv + rows), inv + 2 * rows, (char *)(inv + 3 * rows));
        } else if (ROWB > 0 && 32 % a.b == 0) {
            if constexpr (ROWB > 0) redundancy_mfma<ROWB, DT, PAD>(a, u, tbl, tmp, tmp + a.T_max, false);
        } else {
            float *inv = tmp + a.T_max, *zv = tmp + 3 * (size_t)a.T_max;
            int *zr = (int *)(tmp + 2 * (size_t)a.T_max);
            if constexpr (ROWB > 0) redundancy_blocks<ROWB, DT, PAD, NW <= 4, TIGHT>(a, u, tbl, tmp, inv, zr, zv);
            else redundancy_valu<DT>(a, u, tbl, tmp, inv, zr, zv);
        }
        // R = softmax over the live sequence of (row sum / Tv) / tau, in base 2
        float m = -INFINITY;
        for (int j = tid; j < u.Tv; j += nt) m = fmaxf(m, tmp[j] * a.inv_tau_log2);
        m = block_reduce(m, true, misc);
        float z = 0.f;
        for (int j = tid; j < u.Tv; j += nt) {
            const float e = __builtin_amdgcn_exp2f(tmp[j] * a.inv_tau_log2 - m);
            tmp[j] = e;
            z += e;
        }
        z = block_reduce(z, false, misc);
        const float f = a.lambda / z;
        for (int j = tid; j < u.Tv; j += nt) S[live_to_pos(u, a, j)] -= f * tmp[j];
        __syncthreads();
    }
}

// Everything after S sits in LDS: refinements, optional score output, selection, optional list output, compaction.
// REF: score refinements are compiled in (a launch without them runs a kernel that does not carry their code).
// TIGHT: four waves per SIMD, 128 registers each.
// SLICED: this workgroup is one of a.slices that move the unit's rows; the first of them writes the other outputs.
template <int ROWB, int DT, bool PAD, int REF, int NW, bool TIGHT, bool SLICED = false>
__device__ inline void unit_tail(const Args &a, const Unit &u, char *smem, const int *tbl, const int *dst, Misc *misc, int slice = 0) {
    const int tid = threadIdx.x, nt = blockDim.x;
    float *S = (float *)(smem + a.off_S);
    int *list = (int *)(smem + a.off_union);
    if (a.stages & STAGE_LOAD_SCORES) {
        const float *src = a.scores_in + (size_t)u.unit * a.scores_in_stride;
        for (int t = tid; t < u.T; t += nt) S[t] = src[t];
        __syncthreads();
    }
    if constexpr (REF != 0) {
        if ((a.stages & STAGE_SCORE) && (a.ex & (EX_GLOBAL | EX_POOL | EX_RED))) refine_unit<ROWB, DT, PAD, REF, NW, TIGHT>(a, u, smem, tbl, misc);
    }
    if (a.scores_out && (!SLICED || slice == 0)) {
        float *o = a.scores_out + (size_t)u.unit * a.T_max;
        for (int t = tid; t < a.T_max; t += nt) o[t] = t < u.T ? S[t] : 0.f;
        __syncthreads();
    }
    if (a.stages & STAGE_SELECT) {
        select_unit(a, u, (unsigned *)S, list, misc);
        if (a.keep_idx_out && (!SLICED || slice == 0)) {
            int *o = a.keep_idx_out + (size_t)u.unit * a.budget;
            for (int r = tid; r < a.budget; r += nt) o[r] = r < u.k ? list[r] : -1;
        }
        if (a.len_out && tid == 0 && (!SLICED || slice == 0)) a.len_out[u.unit] = u.k;
    }
    if (a.stages & STAGE_LOAD_LIST) {
        const int *src = a.keep_idx_in + (size_t)u.unit * a.budget;
        for (int r = tid; r < u.k; r += nt) {
            const int t = src[r];
            const int prev = r ? src[r - 1] : -1;
            if (t <= prev || t >= u.T) misc->bad = BAD_KEEP_IDX;
            list[r] = t;
        }
        __syncthreads();
        if (misc->bad) {
            if (tid == 0) report_bad(a, u.unit, misc->bad);
            return;
        }
    }
    if (a.stages & STAGE_COMPACT) {
        if constexpr (SLICED) {
            if (a.b_shift >= 0) compact_slice<8, true>(a, u, tbl, dst, list, u.k, slice);
            else compact_slice<8, false>(a, u, tbl, dst, list, u.k, slice);
            return;
        }
        if (REF != 0 && (a.ex & EX_MOVE_F_LDS)) compact_unit<2>(a, u, tbl, dst, list, (const float *)(smem + a.off_G), u.k);
        else if (REF != 0 && (a.ex & EX_MOVE_F)) compact_unit<1>(a, u, tbl, dst, list, nullptr, u.k);
        else compact_unit<0>(a, u, tbl, dst, list, nullptr, u.k);
    }
}

}  // namespace zp
