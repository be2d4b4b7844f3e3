// C ABI of libzp (see include/zp.h): argument checks, LDS layout, kernel dispatch, the
// host-side block planner and the slow full validator.  No torch types, no hidden allocation
// after zp_create.
#include "../../include/zp.h"
#include "zp_kernels.h"

#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <unordered_set>
#include <vector>

#define ZP_SLOTS 4
static const size_t kSlotBytes = 24u << 20;

struct zp_ctx {
    int device;
    int *d_status;   // 8 words on the device: flag, unit, reason
    int *h_status;   // pinned mirror
    int xcd_map;     // workgroup -> unit map: 1 contiguous ranges per XCD, 0 identity
    int n_cu;        // compute units: every kernel here fits at least one workgroup per CU
    std::atomic<int> launches;   // kernel launches of the last call (zp_last_launches)
    char err[512];
    // Workspaces of the calls that take several launches (partial sums of sweep 1, scores between the launches).  A call takes the
    // one its stream used last, else the next in turn, waits on the device for that one's last call and records an event after
    // its own: calls on different streams stay apart, and one that has to share is merely ordered behind the other.
    struct Slot { char *mem; hipEvent_t done; void *stream; bool used; } slot[ZP_SLOTS];
    int next_slot;
    std::mutex slot_mu;
};

static thread_local char g_err[512] = "";

static zp_status fail(zp_ctx *ctx, zp_status code, const char *fmt, ...) {
    char *dst = ctx ? ctx->err : g_err;
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(dst, 512, fmt, ap);
    va_end(ap);
    return code;
}

extern "C" const char *zp_last_error(const zp_ctx *ctx) { return ctx ? ctx->err : g_err; }

extern "C" zp_status zp_create(zp_ctx **out) {
    if (!out) return fail(nullptr, ZP_EINVAL, "zp_create: out is NULL");
    *out = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(nullptr, ZP_EHIP, "zp_create: no HIP device (%s)", hipGetErrorString(e));
    zp_ctx *c = new (std::nothrow) zp_ctx();
    if (!c) return fail(nullptr, ZP_ENOMEM, "zp_create: out of host memory");
    c->device = dev;
    c->err[0] = 0;
    c->xcd_map = 1;
    c->n_cu = 0;
    (void)hipDeviceGetAttribute(&c->n_cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (c->n_cu <= 0) c->n_cu = 64;
    if ((e = hipMalloc((void **)&c->d_status, 8 * sizeof(int))) != hipSuccess ||
        (e = hipHostMalloc((void **)&c->h_status, 8 * sizeof(int), hipHostMallocDefault)) != hipSuccess ||
        (e = hipMemset(c->d_status, 0, 8 * sizeof(int))) != hipSuccess) {
        zp_status rc = fail(nullptr, ZP_EHIP, "zp_create: %s", hipGetErrorString(e));
        if (c->d_status) (void)hipFree(c->d_status);
        delete c;
        return rc;
    }
    // without workspaces (no memory left for them) every call takes one launch
    char *mem = nullptr;
    bool ok = hipMalloc((void **)&mem, ZP_SLOTS * kSlotBytes) == hipSuccess;
    for (auto &w : c->slot) ok = ok && hipEventCreateWithFlags(&w.done, hipEventDisableTiming) == hipSuccess;
    if (ok) for (int i = 0; i < ZP_SLOTS; i++) c->slot[i].mem = mem + i * kSlotBytes;
    else {
        if (mem) (void)hipFree(mem);
        (void)hipGetLastError();                              // nobody's error
    }
    *out = c;
    return ZP_OK;
}

extern "C" void zp_destroy(zp_ctx *ctx) {
    if (!ctx) return;
    (void)hipFree(ctx->d_status);
    (void)hipHostFree(ctx->h_status);
    if (ctx->slot[0].mem) (void)hipFree(ctx->slot[0].mem);
    for (auto &w : ctx->slot) if (w.done) (void)hipEventDestroy(w.done);
    delete ctx;
}

static int align16(int x) { return (x + 15) & ~15; }
static const int kLdsLimit = 160 * 1024;
static const int kMiscBytes = align16((int)sizeof(int) * (256 + 16 + 4));

enum Path { PATH_GENERIC, PATH_MFMA };

extern "C" zp_status zp_set_option(zp_ctx *ctx, int32_t option, int32_t value) {
    if (!ctx) return ZP_EINVAL;
    if (option == ZP_OPT_SPLIT && value == 1) {
        // Several workgroups per unit that wait for each other inside one kernel: such a kernel existed and its bounded wait
        // expired now and then on MI355X (reported, nothing faulted) with no cause found.  It is gone; the option stays refused.
        snprintf(ctx->err, sizeof(ctx->err), "zp_set_option: the split path is switched off in this build (its rendezvous is not reliable on MI355X yet)");
        return ZP_EUNSUPPORTED;
    }
    if (option == ZP_OPT_SPLIT && value >= -1 && value <= 0) return ZP_OK;
    if (option == ZP_OPT_SPIN_LIMIT && value > 0) return ZP_OK;               // these two were settings of that kernel: accepted, no effect
    if (option == ZP_OPT_STREAMS && value >= 1 && value <= 8) return ZP_OK;
    if (option == ZP_OPT_XCD_MAP && (value == 0 || value == 1)) { ctx->xcd_map = value; return ZP_OK; }
    snprintf(ctx->err, sizeof(ctx->err), "zp_set_option: unknown option %d or bad value %d", option, value);
    return ZP_EINVAL;
}

// Lightning redundancy in blocks of more than 32: a workgroup has at least four waves, above 96 positions eight, also where the window
// gives fewer waves query blocks (the others leave the scoring arithmetic out), and goes block by block with the rows in LDS
// (redundancy_staged) where a block has column groups of 32 for at least half the waves.  Fragments straight from L2 against this,
// in us: paper geometry (two query blocks, blocks of 256, 1152 units of 2304) 1692:951, with two waves 1384; 512 units of 2176 in
// blocks of 128 (one query block) 880:383; 512 units of 4160 in blocks of 64, four waves 1183:884; with eight waves blocks of 64 keep
// two waves busy and stay with redundancy_blocks.
static int red_waves(int b) { return b > 96 ? 8 : b > 32 ? 4 : 1; }
static bool red_staged(int b, int NW) { return b > 32 && NW >= 4 && 2 * ((b + 31) / 32) >= NW; }

// Scalar checks shared by every call, and the kernel argument block.  `need_q`: the call scores.
static zp_status prepare(zp_ctx *ctx, const char *who, const zp_pool *p, const zp_batch *b, bool need_q, zp::Args *a,
                         Path *path, zp::MfmaGeo *geo, const zp_extras *ex = nullptr, bool fused = false) {
    if (!ctx) return fail(nullptr, ZP_EINVAL, "%s: ctx is NULL", who);
    if (!p || !b) return fail(ctx, ZP_EINVAL, "%s: pool or batch is NULL", who);
    if (p->dtype != ZP_F32 && p->dtype != ZP_BF16) return fail(ctx, ZP_EINVAL, "%s: unknown dtype %d", who, p->dtype);
    if (p->L_slab <= 0 || p->layer0 < 0 || p->N_total <= 0 || p->b <= 0 || p->h_kv <= 0 || p->h_q <= 0 || p->d <= 0 ||
        p->M <= 0 || p->w <= 0)
        return fail(ctx, ZP_EINVAL, "%s: pool dimensions must be positive", who);
    if (b->B < 0 || b->N_max < 2 || b->max_blocks < b->N_max || b->L < p->layer0 + p->L_slab)
        return fail(ctx, ZP_EINVAL, "%s: need B >= 0, N_max >= 2, max_blocks >= N_max, L >= layer0 + L_slab", who);
    if (!p->k || !p->v) return fail(ctx, ZP_EINVAL, "%s: k / v pool pointer is NULL", who);
    if (b->B > 0 && (!b->block_table || !b->num_blocks)) return fail(ctx, ZP_EINVAL, "%s: block_table / num_blocks is NULL", who);
    if (need_q && (!p->q || (b->B > 0 && !b->q_slot))) return fail(ctx, ZP_EINVAL, "%s: q / q_slot is NULL", who);
    if (p->h_q % p->h_kv) return fail(ctx, ZP_EUNSUPPORTED, "%s: h_q %d is not a multiple of h_kv %d", who, p->h_q, p->h_kv);
    const int esz = p->dtype == ZP_F32 ? 4 : 2;
    const long long row_bytes = (long long)p->d * esz;
    if (row_bytes % 16 || row_bytes > 1024) return fail(ctx, ZP_EUNSUPPORTED, "%s: row of %lld bytes (need a multiple of 16, at most 1024)", who, row_bytes);
    const long long T_max = (long long)b->max_blocks * p->b, budget = (long long)(b->N_max - 1) * p->b;
    if (budget < p->w) return fail(ctx, ZP_EINVAL, "%s: budget %lld smaller than the window %d", who, budget, p->w);
    if ((long long)p->N_total * p->b > 0x7fffffffLL) return fail(ctx, ZP_EUNSUPPORTED, "%s: N_total*b exceeds 2^31-1 token slots per layer", who);
    if (T_max > 65535) return fail(ctx, ZP_EUNSUPPORTED, "%s: %lld positions per request exceed 65535", who, T_max);
    const long long units = (long long)b->B * p->L_slab * p->h_kv;
    if (units > 0x7fffffffLL) return fail(ctx, ZP_EUNSUPPORTED, "%s: too many units", who);

    memset(a, 0, sizeof(*a));
    a->k = (char *)p->k; a->v = (char *)p->v; a->q = (const char *)p->q;
    a->layer0 = p->layer0; a->L_slab = p->L_slab; a->N_total = p->N_total; a->b = p->b; a->h_kv = p->h_kv; a->h_q = p->h_q;
    a->d = p->d; a->M = p->M; a->w = p->w; a->dtype = p->dtype;
    a->B = b->B; a->N_max = b->N_max; a->max_blocks = b->max_blocks; a->L = b->L;
    a->block_table = b->block_table; a->dst_table = b->dst_table; a->num_blocks = b->num_blocks; a->q_slot = b->q_slot;
    a->valid_len = b->valid_len; a->keep = b->keep;
    a->G = p->h_q / p->h_kv; a->T_max = (int)T_max; a->budget = (int)budget; a->row_bytes = (int)row_bytes;
    a->b_shift = -1;
    for (int s = 0; s < 31; s++) if ((1 << s) == p->b) a->b_shift = s;
    a->scale_log2 = (float)(1.4426950408889634 / std::sqrt((double)p->d));
    a->status = ctx->d_status;
    a->xcd_map = ctx->xcd_map;

    *path = PATH_GENERIC;
    *geo = zp::MfmaGeo{4, 0, 1, 0, false};
    if (need_q && zp::mfma_path_available(*a, geo)) {
        *path = PATH_MFMA;
        a->NP = geo->NP;
    }
    // score refinements (they run in the tail of the one-workgroup-per-unit kernels only)
    if (ex) {
        if (*path == PATH_MFMA && ex->lambda != 0.f && geo->RB == 1 && geo->NW < red_waves(p->b)) geo->NW = red_waves(p->b);
        if (ex->pool_kernel < 1 || !(ex->pool_kernel & 1)) return fail(ctx, ZP_EINVAL, "%s: pool_kernel %d must be odd and >= 1", who, ex->pool_kernel);
        if (ex->lambda != 0.f && !(ex->tau > 0.f && std::isfinite(ex->tau))) return fail(ctx, ZP_EINVAL, "%s: tau must be positive", who);
        if (ex->F && (long long)p->L_slab * p->N_total * p->b * p->h_kv > 0xffffffffLL)
            return fail(ctx, ZP_EUNSUPPORTED, "%s: global-score cache of more than 2^32-1 entries per slab", who);
        // the fused call moves the cached global scores with the rows: from an on-chip copy when targets differ from
        // sources (blocks may be shared inside the batch), read back from F otherwise (in place: every block is private)
        if (ex->F) a->ex |= zp::EX_GLOBAL | (fused ? (b->dst_table ? zp::EX_MOVE_F_LDS : zp::EX_MOVE_F) : 0);
        if (ex->pool_kernel > 1) a->ex |= zp::EX_POOL | (ex->pool_first_only ? zp::EX_POOL_FIRST : 0);
        if (ex->lambda != 0.f) a->ex |= zp::EX_RED;
        a->F = ex->F; a->compressed = ex->compressed; a->alpha = ex->alpha; a->lambda = ex->lambda; a->p_thr = ex->p;
        a->inv_tau_log2 = ex->lambda != 0.f ? (float)(1.4426950408889634 / (double)ex->tau) : 0.f;
        a->pool_r = ex->pool_kernel / 2;
    }
    // LDS of one unit; `worst`: as the fused call with a moved global-score cache would need it
    auto layout = [&](bool worst) {
        const bool mf = *path == PATH_MFMA, move_f = (a->ex & zp::EX_MOVE_F_LDS) || (worst && ex && ex->F && b->dst_table);
        // similarity tiles from sweep 2's key tiles
        if ((a->ex & zp::EX_RED) && mf && !geo->pad && p->b == 16 && geo->RB == 1) a->ex |= zp::EX_RED_FUSED;
        const size_t score_bytes = !need_q ? 0 : mf ? zp::mfma_union_bytes(*geo) : (size_t)a->G * a->w * 4;
        if ((a->ex & zp::EX_RED) && mf && red_staged(p->b, geo->NW)) a->ex |= zp::EX_RED_STAGED;
        else a->ex &= ~zp::EX_RED_STAGED;
        const size_t red_bytes = a->ex & zp::EX_RED_STAGED ? 12 + 12 * (size_t)((p->b + 31) & ~31) + (size_t)zp::mfma_tile_keys(geo->rowb) * (geo->rowb + 16)
                                 : mf && 32 % p->b == 0 ? (size_t)geo->NW * 96 * 4 : (size_t)a->T_max * 12;
        const size_t refine_bytes = ((a->ex & (zp::EX_POOL | zp::EX_RED)) ? (size_t)a->T_max * 4 : 0) + ((a->ex & zp::EX_RED) ? red_bytes : 0);
        const size_t list_bytes = (size_t)a->budget * 4;
        a->off_S = 0;
        a->off_tbl = align16(a->T_max * 4);
        a->off_dst = a->off_tbl + align16(a->max_blocks * 4);
        a->off_misc = a->off_dst + align16((a->N_max - 1) * 4);
        a->off_union = a->off_misc + kMiscBytes;
        size_t union_bytes = score_bytes > list_bytes ? score_bytes : list_bytes;
        if (refine_bytes > union_bytes) union_bytes = refine_bytes;
        a->off_G = a->off_union + align16((int)union_bytes);
        a->off_R = a->off_G + (move_f ? align16(a->T_max * 4) : 0);
        return (size_t)a->off_R + ((a->ex & zp::EX_RED_FUSED) ? (size_t)a->T_max * 4 + (size_t)geo->NW * 96 * 4 : 0);
    };
    // Sequences so long that their scores leave no room for key tiles of this row size go to the vector-ALU kernel (the
    // staged and the fused call decide alike: they give the same bits).
    if (*path == PATH_MFMA && geo->pad && layout(true) > (size_t)kLdsLimit) *path = PATH_GENERIC;
    const size_t total = layout(false);
    if (total > (size_t)kLdsLimit)
        return fail(ctx, ZP_EUNSUPPORTED, "%s: %zu bytes of LDS per unit exceed %d (max_blocks*b too large)", who, total, kLdsLimit);
    a->lds_bytes = (int)align16((int)total);
    return ZP_OK;
}

extern "C" size_t zp_scratch_bytes(const zp_pool *pool, const zp_batch *batch) {
    (void)pool; (void)batch;
    return 0;
}

// With one workgroup per unit, a launch of fewer units than compute units leaves the rest idle, and one unit's two sweeps,
// selection and row moving follow each other on its own.  Row moving (and a selection of its own) is cut into slices up to three
// quarters of the compute units: staged select and compact of 192 units 52 -> 50 us at 272 positions, 437 -> 343 us at 4112.
static bool few_units(const zp_ctx *ctx, long long units) { return units <= ctx->n_cu * 3 / 4; }

// Whether scoring in two launches with several workgroups per unit (`whole`: then selection and row moving in a third) beats one
// launch.  A launch more costs its set-up once per workgroup and its wait for the slowest one, and the wider a unit's workgroup,
// the fewer units fill the chip by themselves.  So the line is drawn on positions against waves in one launch (units x waves per
// workgroup); the measurements below are one launch against three in us, d 128, G 4, bf16, 256 compute units:
//   eight waves (w 64):   64 units   4112           265:122
//                                     768 positions  55: 48      512  39: 46
//                         96         1040            80: 75      768  60: 63
//                        128         2064           151:135     1040  84: 92
//                        160 or 192  up to 8208 never worth it (4112: 298:314, 316:344), but with live lengths from a quarter to
//                                    the whole of the positions, where the longest unit holds up the one launch, 160  4112 257:222,
//                                    2384 156:156;  192  4112 262:253  2384 159:176
//   four (w 32):   128 or fewer 512  52: 51;   160  1040 108: 97  768 78: 82;   192  1040 111:108  768 82: 91
//   two (w 16):    192  768  92: 82   512 63: 67;    one (w 4): 192  512  96: 68
//   several blocks per wave (w 112), four workgroups per unit that fill a compute unit each:
//                   64   512  53: 47;    96  1040 105: 99   768 79: 82;   128  1040 109:107;   160 4112 381:408
//   two staged scoring launches against one, the row moving being sliced either way, need 8/5 of the positions:
//                  128 of eight waves  2064 211:209  1040 118:131;   192 of four  2064 228:219  1040 125:131
// Rows of 128 bytes (d 64) have less to share out; fp32, other long rows and padded rows more (eight waves, 128 units: fp32 512
// 183:172; d 96 1040 96:86, staged 848 74:71).
static bool split_pays(int n_cu, long long units, int T, const zp::MfmaGeo &geo, bool f32, bool whole, bool ragged) {
    const long long u = units * 256 / n_cu;                    // the same share of 256 compute units
    if (T < 512) return false;
    if (geo.RB > 1 && u <= 64) return T >= (geo.rowb <= 128 && geo.RB == 2 ? 768 : 512);
    const bool heavy = geo.RB > 2 || geo.rowb > 256;
    if (u > 128) {                                             // two rounds of row-moving workgroups
        if (geo.NW == 8) {
            if (heavy) return T >= 16 * u;
            if (geo.pad) return (ragged || !whole) && T >= 12 * u;
            return whole ? ragged && T >= 18 * u : T >= 24 * u;
        }
        if (geo.NW > 1 && geo.rowb <= 512 && T < 768) return false;
    }
    int eighths = whole ? 10 : 16;                             // positions per wave of one launch
    if (geo.pad) eighths = f32 && whole ? 5 : 8;
    else if (geo.RB > 1) eighths = whole ? (geo.RB > 2 ? 8 : 10) : 12;
    const bool early = heavy || geo.NW <= 2 || (geo.NW == 4 && geo.rowb > 128 && whole);
    return T >= u * geo.NW * eighths / 8 && T >= (early ? 512 : geo.NW == 8 && geo.rowb <= 128 ? 768 : 640);
}

// Workspace of a call: partial sums of sweep 1, the units' scalars, the scores.
static size_t seg_bytes(const zp::MfmaGeo &geo, long long units) { return (size_t)units * ZP_SEGMENTS * geo.NW * geo.RB * 32 * sizeof(float2); }
static size_t workspace_bytes(const zp::Args &a, const zp::MfmaGeo &geo, long long units) {
    return seg_bytes(geo, units) + (size_t)units * sizeof(int2) + (size_t)units * a.T_max * 4;
}

static bool len_out_meets(const zp::Args &a, long long units, const int *p, long long n) {
    const uintptr_t lo = (uintptr_t)a.len_out, hi = lo + (uintptr_t)units * 4;
    return a.len_out && p && lo < (uintptr_t)p + (uintptr_t)n * 4 && (uintptr_t)p < hi;
}

// len_out inside one of the arrays that every launch of a call reads again
static bool overlaps_tables(const zp::Args &a, long long units) {
    return len_out_meets(a, units, a.num_blocks, a.B) || len_out_meets(a, units, a.q_slot, a.B) ||
           len_out_meets(a, units, a.block_table, (long long)a.B * a.max_blocks) || len_out_meets(a, units, a.dst_table, (long long)a.B * (a.N_max - 1));
}

// len_out inside valid_len or keep: the row-moving launch, where one workgroup of a unit writes it and others read them, takes both
// from the workspace (see unit_scalars; always taking them there costs 1 us of 33 on 32 units of 1296 positions)
static bool overlaps_scalars(const zp::Args &a, long long units) {
    const long long n = (long long)a.B * a.L * a.h_kv;
    return len_out_meets(a, units, a.valid_len, n) || len_out_meets(a, units, a.keep, n);
}

// Whether a call is split.
static bool is_split(const zp_ctx *ctx, const zp::Args &a, Path path, const zp::MfmaGeo &geo, hipStream_t s) {
    const long long units = (long long)a.B * a.L_slab * a.h_kv;
    if (path != PATH_MFMA || geo.NP != 1 || a.ex || !ctx->slot[0].mem || units <= 0 || !few_units(ctx, units) ||
        !split_pays(ctx->n_cu, units, a.T_max, geo, a.dtype == 0, (a.stages & zp::STAGE_SELECT) != 0, a.valid_len != nullptr))
        return false;
    if (workspace_bytes(a, geo, units) > kSlotBytes || overlaps_tables(a, units)) return false;
    int dev = -1;                                              // workspaces and events belong to the context's GPU
    if ((s ? hipStreamGetDevice(s, &dev) : hipGetDevice(&dev)) != hipSuccess) (void)hipGetLastError();
    if (dev != ctx->device) return false;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess) {
        (void)hipGetLastError();                               // not the launch's error
        return false;
    }
    return cap == hipStreamCaptureStatusNone;                  // a graph may run beside anything: no shared workspace
}

// Workgroups per unit of the two scoring launches.  A compute unit takes K = units x parts / compute units of them (the fullest one), in
// as many rounds as its registers and LDS ask for.  A round costs its set-up and first loads, about as much as 21 tiles of one query
// block; a tile costs a compute unit the query blocks of the workgroups on it, but with fewer than six blocks at work there its latency.
// The cheapest number against as many parts as segments, in us: fp32 128 units of 1040 (four waves) 163 against 190, staged 192 units of 2064
// to 4112 (w 32) 193 against 201, one wave 192 units of 4112 284 against 301, 128 units (w 64) 210 against 223, 64 units 119 against 122;
// 128 units of two waves (w 16) keep eight: 174 against 190 with four.
static int pick_parts(const zp_ctx *ctx, const zp::Args &a, const zp::MfmaGeo &geo, long long units, int lds_bytes) {
    const int kt = zp::mfma_tile_keys(geo.rowb), ntiles = (a.T_max + kt - 1) / kt, nseg = zp::segment_count(ntiles, zp::segments_of(geo.RB));
    const int per_simd = geo.RB > 1 || geo.rowb > 512 ? 2 : geo.rowb > 256 ? 3 : 4;
    const int by_regs = 4 * per_simd / geo.NW > 0 ? 4 * per_simd / geo.NW : 1, by_lds = kLdsLimit / lds_bytes, at_once = by_regs < by_lds ? by_regs : by_lds;
    int best = 1;
    long long cost = -1;
    for (int parts = 1; parts <= nseg; parts++) {
        const long long K = (units * parts + ctx->n_cu - 1) / ctx->n_cu, rounds = (K + at_once - 1) / at_once, work = K * geo.NW * geo.RB;
        const long long tiles = (long long)((nseg + parts - 1) / parts) * ((ntiles + nseg - 1) / nseg);
        const long long c = tiles * (work > 6 * rounds ? work : 6 * rounds) + 21 * rounds;
        if (cost < 0 || c < cost) { cost = c; best = parts; }
    }
    return best;
}

// Row-moving workgroups per unit: K and V apart, rows cut into the shortest pieces (from 128 bytes on, 64 where those do not divide
// the row) that make no more workgroups than compute units.  A workgroup of sixteen waves at 67 registers has a compute unit to
// itself, so more of them take turns and every turn pays for the set-up and a selection of its own.  Measured (rows of 256 bytes, d 128,
// G 4, w 32, 1040 positions, whole call) with four pieces against two: 96 units 66 against 59 us, 128 units 77 against 72 us; rows of
// 512 bytes (fp32, 64 units, 512 positions) with eight against two 82 against 80 us; at 64 units of 256 bytes all four pieces
// run at once: 4112 rows of K and V in 64 us with the selection, 3.9 TB/s.  64 registers for two workgroups per
// compute unit gave 6 us at 160 to 192 units below 1040 positions and lost up to 2.7 % at 4112 and more.
static void pick_slices(const zp_ctx *ctx, zp::Args *a, int units) {
    a->slices = 2;
    a->slice_bytes = a->row_bytes;
    const auto fits = [&](int piece) { return a->row_bytes % piece == 0 && a->row_bytes > piece && (long long)units * 2 * (a->row_bytes / piece) <= ctx->n_cu; };
    for (const int piece : {128, 256, 512, 64})
        if (fits(piece)) {
            a->slices = 2 * (a->row_bytes / piece);
            a->slice_bytes = piece;
            break;
        }
}

static hipError_t launch_split(zp_ctx *ctx, zp::Args a, int units, const zp::MfmaGeo &geo, hipStream_t s) {
    std::lock_guard<std::mutex> lock(ctx->slot_mu);
    int i = -1;
    for (int j = 0; j < ZP_SLOTS; j++) if (ctx->slot[j].used && ctx->slot[j].stream == (void *)s) i = j;
    if (i < 0) { i = ctx->next_slot; ctx->next_slot = (i + 1) % ZP_SLOTS; }
    zp_ctx::Slot &w = ctx->slot[i];
    hipError_t e = w.used ? hipStreamWaitEvent(s, w.done, 0) : hipSuccess;
    if (e != hipSuccess) return e;
    const bool whole = (a.stages & zp::STAGE_SELECT) != 0;
    int2 *scalars = (int2 *)(w.mem + seg_bytes(geo, units));
    float *scores = whole ? (float *)(scalars + units) : a.scores_out;
    zp::Args m = a;                                           // scoring
    m.stages = zp::STAGE_SCORE;
    m.keep_idx_out = nullptr;
    m.seg = (float2 *)w.mem;
    m.unit_out = whole && overlaps_scalars(a, units) ? scalars : nullptr;
    m.scores_out = scores;
    m.off_tbl = 0;                                            // the two scoring launches keep no scores and no targets on chip
    m.off_misc = align16(a.max_blocks * 4);
    m.off_union = m.off_misc + kMiscBytes;
    m.lds_bytes = align16(m.off_union + (int)zp::mfma_union_bytes(geo));
    m.parts = pick_parts(ctx, a, geo, units, m.lds_bytes);
    w.used = true;
    w.stream = (void *)s;
    for (m.phase = 1; m.phase <= 2 && e == hipSuccess; m.phase++) e = zp::launch_unit_mfma(m, units, geo, s);
    if (e == hipSuccess && whole) {                           // selection and row moving
        a.stages = zp::STAGE_LOAD_SCORES | zp::STAGE_SELECT | zp::STAGE_COMPACT | zp::STAGE_CHECK_SLOT;
        a.scores_in = scores;
        a.scores_in_stride = a.T_max;
        a.unit_in = m.unit_out;
        a.lds_bytes = a.off_union + align16(a.budget * 4);
        pick_slices(ctx, &a, units);
        e = zp::launch_unit_sliced(a, units, s);
    }
    const hipError_t er = hipEventRecord(w.done, s);
    return e != hipSuccess ? e : er;
}

// Costliest units first (unit_by_cost) where live lengths differ from head to head and some units have to wait for others to end: up to two rounds of
// workgroups, four where a wave holds several query blocks.  With more rounds the short units of the last one even out by themselves,
// and the order costs more than it gives: the kv heads of one (request, layer), which read the same blocks, then run far apart, which
// only launches bound by the scoring arithmetic do not mind.  Measured, in order of number against by cost in us (d 128, bf16; live
// lengths from a quarter of the positions on): several blocks per wave 384 units (1.5 rounds) 1386:972, 768 (3) 1109:923;
// one block, live lengths 640 units 479:425, with all three refinements 768 594:506, four waves 1536 (2) 700:620, but
// 1280 units (2.5) 940:965, 2048 (4) 1165:1224.  Where only the keep counts differ, scoring is alike and little is left to even out:
// 768 units 879:870, f32 637:623, but 672 of seven heads 374:394; requests of different lengths with all heads alike: 1280 units 883:964.
static bool order_by_cost(const zp_ctx *ctx, const zp::Args &a, const zp::MfmaGeo &geo, long long units) {
    if (!a.valid_len || a.T_max < 1024 || overlaps_scalars(a, units) || overlaps_tables(a, units)) return false;
    const int waves = geo.RB == 1 && geo.rowb <= 256 ? 16 : 8, by_regs = waves / geo.NW, by_lds = kLdsLimit / a.lds_bytes;
    const long long at_once = (long long)ctx->n_cu * (by_regs < by_lds ? by_regs : by_lds);
    return units > at_once && units <= (geo.RB > 1 ? 4 : 2) * at_once;
}

extern "C" int32_t zp_last_launches(const zp_ctx *ctx) { return ctx ? ctx->launches.load() : 0; }

static zp_status launch(zp_ctx *ctx, const char *who, zp::Args &a, Path path, const zp::MfmaGeo &geo, void *stream) {
    const int units = a.B * a.L_slab * a.h_kv;
    ctx->launches = units > 0;
    if (is_split(ctx, a, path, geo, (hipStream_t)stream)) {
        ctx->launches = (a.stages & zp::STAGE_SELECT) ? 3 : 2;
        const hipError_t e = launch_split(ctx, a, units, geo, (hipStream_t)stream);
        if (e != hipSuccess) return fail(ctx, ZP_EHIP, "%s: kernel launch failed: %s", who, hipGetErrorString(e));
        return ZP_OK;
    }
    if (path == PATH_GENERIC && !a.ex && !(a.stages & zp::STAGE_SCORE) && few_units(ctx, units)) {   // staged select or compact
        if (a.stages & zp::STAGE_COMPACT) pick_slices(ctx, &a, units);
        else a.slices = 1;
        const hipError_t e = zp::launch_unit_sliced(a, units, (hipStream_t)stream);
        if (e != hipSuccess) return fail(ctx, ZP_EHIP, "%s: kernel launch failed: %s", who, hipGetErrorString(e));
        return ZP_OK;
    }
    a.by_cost = path == PATH_MFMA && order_by_cost(ctx, a, geo, units);
    hipError_t e = path == PATH_MFMA ? zp::launch_unit_mfma(a, units, geo, (hipStream_t)stream)
                                     : zp::launch_unit_generic(a, units, (hipStream_t)stream);
    if (e != hipSuccess) return fail(ctx, ZP_EHIP, "%s: kernel launch failed: %s", who, hipGetErrorString(e));
    return ZP_OK;
}

extern "C" zp_status zp_score(zp_ctx *ctx, const zp_pool *pool, const zp_batch *batch, float *scores, void *stream) {
    zp::Args a; Path path; zp::MfmaGeo geo;
    zp_status rc = prepare(ctx, "zp_score", pool, batch, true, &a, &path, &geo);
    if (rc) return rc;
    if (!scores && batch->B > 0) return fail(ctx, ZP_EINVAL, "zp_score: scores is NULL");
    a.stages = zp::STAGE_SCORE;
    a.scores_out = scores;
    return launch(ctx, "zp_score", a, path, geo, stream);
}

extern "C" zp_status zp_score_ex(zp_ctx *ctx, const zp_pool *pool, const zp_batch *batch, const zp_extras *extras, float *scores,
                                 void *stream) {
    if (!extras) return zp_score(ctx, pool, batch, scores, stream);
    zp::Args a; Path path; zp::MfmaGeo geo;
    zp_status rc = prepare(ctx, "zp_score_ex", pool, batch, true, &a, &path, &geo, extras, false);
    if (rc) return rc;
    if (!scores && batch->B > 0) return fail(ctx, ZP_EINVAL, "zp_score_ex: scores is NULL");
    a.stages = zp::STAGE_SCORE;
    a.scores_out = scores;
    return launch(ctx, "zp_score_ex", a, path, geo, stream);
}

extern "C" zp_status zp_select_topk(zp_ctx *ctx, const float *scores, int32_t T_max, const zp_pool *pool, const zp_batch *batch,
                                    int32_t *keep_idx, int32_t *len_out, void *stream) {
    zp::Args a; Path path; zp::MfmaGeo geo;
    zp_status rc = prepare(ctx, "zp_select_topk", pool, batch, false, &a, &path, &geo);
    if (rc) return rc;
    if ((!scores || !keep_idx || !len_out) && batch->B > 0) return fail(ctx, ZP_EINVAL, "zp_select_topk: scores / keep_idx / len_out is NULL");
    if (T_max < a.T_max) return fail(ctx, ZP_EINVAL, "zp_select_topk: T_max %d smaller than max_blocks*b = %d", T_max, a.T_max);
    a.stages = zp::STAGE_LOAD_SCORES | zp::STAGE_SELECT;
    a.scores_in = scores; a.scores_in_stride = T_max;
    a.keep_idx_out = keep_idx; a.len_out = len_out;
    return launch(ctx, "zp_select_topk", a, PATH_GENERIC, geo, stream);
}

extern "C" zp_status zp_compact_kv(zp_ctx *ctx, const zp_pool *pool, const zp_batch *batch, const int32_t *keep_idx,
                                   const int32_t *len, void *stream) {
    zp::Args a; Path path; zp::MfmaGeo geo;
    zp_status rc = prepare(ctx, "zp_compact_kv", pool, batch, false, &a, &path, &geo);
    if (rc) return rc;
    if ((!keep_idx || !len) && batch->B > 0) return fail(ctx, ZP_EINVAL, "zp_compact_kv: keep_idx / len is NULL");
    a.stages = zp::STAGE_LOAD_LIST | zp::STAGE_COMPACT;
    a.keep_idx_in = keep_idx; a.len_in = len;
    return launch(ctx, "zp_compact_kv", a, PATH_GENERIC, geo, stream);
}

extern "C" zp_status zp_compact_kv_ex(zp_ctx *ctx, const zp_pool *pool, const zp_batch *batch, float *F, const int32_t *keep_idx,
                                      const int32_t *len, void *stream) {
    if (!F) return zp_compact_kv(ctx, pool, batch, keep_idx, len, stream);
    zp::Args a; Path path; zp::MfmaGeo geo;
    zp_status rc = prepare(ctx, "zp_compact_kv_ex", pool, batch, false, &a, &path, &geo);
    if (rc) return rc;
    if ((!keep_idx || !len) && batch->B > 0) return fail(ctx, ZP_EINVAL, "zp_compact_kv_ex: keep_idx / len is NULL");
    if ((long long)pool->L_slab * pool->N_total * pool->b * pool->h_kv > 0xffffffffLL)
        return fail(ctx, ZP_EUNSUPPORTED, "zp_compact_kv_ex: global-score cache of more than 2^32-1 entries per slab");
    a.stages = zp::STAGE_LOAD_LIST | zp::STAGE_COMPACT;
    a.keep_idx_in = keep_idx; a.len_in = len;
    a.F = F; a.ex = zp::EX_MOVE_F;
    return launch(ctx, "zp_compact_kv_ex", a, PATH_GENERIC, geo, stream);
}

extern "C" zp_status zp_compress_ex(zp_ctx *ctx, const zp_pool *pool, const zp_batch *batch, const zp_extras *extras, int32_t *len_out,
                                    float *scores_dbg, int32_t *keep_idx_dbg, void *stream) {
    if (!extras) return zp_compress(ctx, pool, batch, len_out, scores_dbg, keep_idx_dbg, stream);
    zp::Args a; Path path; zp::MfmaGeo geo;
    zp_status rc = prepare(ctx, "zp_compress_ex", pool, batch, true, &a, &path, &geo, extras, true);
    if (rc) return rc;
    if (!len_out && batch->B > 0) return fail(ctx, ZP_EINVAL, "zp_compress_ex: len_out is NULL");
    a.stages = zp::STAGE_SCORE | zp::STAGE_SELECT | zp::STAGE_COMPACT;
    a.scores_out = scores_dbg; a.keep_idx_out = keep_idx_dbg; a.len_out = len_out;
    return launch(ctx, "zp_compress_ex", a, path, geo, stream);
}

extern "C" zp_status zp_compress(zp_ctx *ctx, const zp_pool *pool, const zp_batch *batch, int32_t *len_out, float *scores_dbg,
                                 int32_t *keep_idx_dbg, void *stream) {
    zp::Args a; Path path; zp::MfmaGeo geo;
    zp_status rc = prepare(ctx, "zp_compress", pool, batch, true, &a, &path, &geo);
    if (rc) return rc;
    if (!len_out && batch->B > 0) return fail(ctx, ZP_EINVAL, "zp_compress: len_out is NULL");
    a.stages = zp::STAGE_SCORE | zp::STAGE_SELECT | zp::STAGE_COMPACT;
    a.scores_out = scores_dbg; a.keep_idx_out = keep_idx_dbg; a.len_out = len_out;
    return launch(ctx, "zp_compress", a, path, geo, stream);
}

// ------------------------------------------------------------------ entry point that allocates nothing
//
// The unit kernels report a skipped unit through a few status words in device memory.  zp_create allocates them
// for a context; callers that may not allocate (HIP graph capture, serving loops, harnesses that forbid hipMalloc)
// cannot create a context, so zp_compress_static keeps those words in a file-scope device array instead.  Every GPU
// the library runs on holds its own copy of the array at its own address until the process ends.
#define ZP_STATIC_WORDS 64
static __device__ __align__(256) int scratch[ZP_STATIC_WORDS];

static const int kMaxDevices = 64;
static std::mutex g_static_mu;
static int *g_static_ptr[kMaxDevices];   // device address of `scratch` per device, looked up once (the name itself is only a host-side stand-in)

__global__ void clear_words(int *p, int n) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) p[i] = 0;
}

extern "C" zp_status zp_compress_static(const zp_pool *pool, const zp_batch *batch, int32_t *len_out, void *stream) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(nullptr, ZP_EHIP, "zp_compress_static: no HIP device (%s)", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(nullptr, ZP_EUNSUPPORTED, "zp_compress_static: device index %d outside [0, %d)", dev, kMaxDevices);
    int *words = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_static_mu);
        words = g_static_ptr[dev];
        if (!words) {                                         // first call on this device, with this device current
            e = hipGetSymbolAddress((void **)&words, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !words)
                return fail(nullptr, ZP_EHIP, "zp_compress_static: cannot resolve the status array on device %d (%s)", dev, hipGetErrorString(e));
            g_static_ptr[dev] = words;
        }
    }
    zp_ctx tmp;                                               // host-side only: carries defaults and the error text
    tmp.device = dev; tmp.d_status = words; tmp.h_status = nullptr; tmp.xcd_map = 1; tmp.n_cu = 0; tmp.launches = 0; tmp.err[0] = 0;
    for (auto &w : tmp.slot) w = {};
    tmp.next_slot = 0;
    zp::Args a; Path path; zp::MfmaGeo geo;
    zp_status rc = prepare(&tmp, "zp_compress_static", pool, batch, true, &a, &path, &geo);
    if (rc == ZP_OK && !len_out && batch->B > 0) rc = fail(&tmp, ZP_EINVAL, "zp_compress_static: len_out is NULL");
    if (rc == ZP_OK && batch->B > 0) {
        a.stages = zp::STAGE_SCORE | zp::STAGE_SELECT | zp::STAGE_COMPACT;
        a.len_out = len_out;
        // the array keeps the previous call's contents: the flag must start at zero (a fill kernel, not a memset
        // node, so that the call can be captured in a graph)
        hipLaunchKernelGGL(clear_words, dim3(1), dim3(64), 0, (hipStream_t)stream, words, 8);
        e = hipGetLastError();
        if (e != hipSuccess) rc = fail(&tmp, ZP_EHIP, "zp_compress_static: kernel launch failed: %s", hipGetErrorString(e));
        else rc = launch(&tmp, "zp_compress_static", a, path, geo, stream);
    }
    if (rc != ZP_OK) snprintf(g_err, sizeof(g_err), "%s", tmp.err);
    return rc;
}

extern "C" zp_status zp_decode_attention(zp_ctx *ctx, const zp_pool *p, int32_t B, int32_t table_stride, const int32_t *table,
                                         const int32_t *len, const void *q, float *out, void *stream) {
    if (!ctx) return fail(nullptr, ZP_EINVAL, "zp_decode_attention: ctx is NULL");
    if (!p || !p->k || !p->v) return fail(ctx, ZP_EINVAL, "zp_decode_attention: pool is NULL");
    if (p->dtype != ZP_F32 && p->dtype != ZP_BF16) return fail(ctx, ZP_EINVAL, "zp_decode_attention: unknown dtype %d", p->dtype);
    if (B < 0 || table_stride <= 0 || p->L_slab <= 0 || p->N_total <= 0 || p->b <= 0 || p->h_kv <= 0 || p->h_q <= 0 || p->d <= 0)
        return fail(ctx, ZP_EINVAL, "zp_decode_attention: dimensions must be positive");
    if (p->h_q % p->h_kv) return fail(ctx, ZP_EUNSUPPORTED, "zp_decode_attention: h_q %d is not a multiple of h_kv %d", p->h_q, p->h_kv);
    if (p->d > 256) return fail(ctx, ZP_EUNSUPPORTED, "zp_decode_attention: head dimension %d above 256", p->d);
    if (B > 0 && (!table || !len || !q || !out)) return fail(ctx, ZP_EINVAL, "zp_decode_attention: NULL argument");
    const long long items = (long long)B * p->L_slab * p->h_q;
    if (items > 0x7fffffffLL) return fail(ctx, ZP_EUNSUPPORTED, "zp_decode_attention: too many queries");
    zp::DecodeArgs a;
    a.k = (const char *)p->k; a.v = (const char *)p->v; a.q = (const char *)q; a.out = out; a.table = table; a.len = len;
    a.status = ctx->d_status;
    a.B = B; a.L_slab = p->L_slab; a.N_total = p->N_total; a.b = p->b; a.h_kv = p->h_kv; a.h_q = p->h_q; a.d = p->d;
    a.dtype = p->dtype; a.table_stride = table_stride; a.row_bytes = p->d * (p->dtype == ZP_F32 ? 4 : 2);
    a.scale_log2 = (float)(1.4426950408889634 / std::sqrt((double)p->d));
    hipError_t e = zp::launch_decode_attention(a, (int)items, (hipStream_t)stream);
    if (e != hipSuccess) return fail(ctx, ZP_EHIP, "zp_decode_attention: kernel launch failed: %s", hipGetErrorString(e));
    return ZP_OK;
}

extern "C" zp_status zp_sync_status(zp_ctx *ctx, void *stream) {
    if (!ctx) return fail(nullptr, ZP_EINVAL, "zp_sync_status: ctx is NULL");
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = hipMemcpyAsync(ctx->h_status, ctx->d_status, 8 * sizeof(int), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(ctx, ZP_EHIP, "zp_sync_status: %s", hipGetErrorString(e));
    if (!ctx->h_status[0]) return ZP_OK;
    const int unit = ctx->h_status[1], reason = ctx->h_status[2];
    e = hipMemsetAsync(ctx->d_status, 0, 8 * sizeof(int), s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    static const char *names[] = {"?", "num_blocks outside [N_max, max_blocks]", "valid_len out of range", "keep count out of range",
                                  "query slot out of range", "block id out of range", "keep_idx not ascending or out of range"};
    return fail(ctx, ZP_EINVAL, "a kernel skipped unit %d: %s", unit, reason >= 1 && reason <= 6 ? names[reason] : names[0]);
}

extern "C" zp_status zp_validate_batch(zp_ctx *ctx, const zp_pool *p, const zp_batch *b) {
    zp::Args a; Path path; zp::MfmaGeo geo;
    zp_status rc = prepare(ctx, "zp_validate_batch", p, b, true, &a, &path, &geo);
    if (rc) return rc;
    const int B = b->B, nt = b->N_max - 1;
    const size_t per = (size_t)b->L * p->h_kv;
    std::vector<int> tbl((size_t)B * b->max_blocks), dst, nb(B), slot(B), vl, keep;
    hipError_t e = hipDeviceSynchronize();
    auto pull = [&](std::vector<int> &h, const int *d, size_t n) {
        h.resize(n);
        if (e == hipSuccess && n) e = hipMemcpy(h.data(), d, n * sizeof(int), hipMemcpyDeviceToHost);
    };
    pull(tbl, b->block_table, tbl.size());
    pull(nb, b->num_blocks, B);
    pull(slot, b->q_slot, B);
    if (b->dst_table) pull(dst, b->dst_table, (size_t)B * nt);
    if (b->valid_len) pull(vl, b->valid_len, B * per);
    if (b->keep) pull(keep, b->keep, B * per);
    if (e != hipSuccess) return fail(ctx, ZP_EHIP, "zp_validate_batch: %s", hipGetErrorString(e));
    std::unordered_set<int> sources, targets_seen, slots_seen;
    for (int n = 0; n < B; n++)
        for (int i = 0; i < nb[n] && i < b->max_blocks; i++) sources.insert(tbl[(size_t)n * b->max_blocks + i]);
    for (int n = 0; n < B; n++) {
        const int N = nb[n];
        if (N < b->N_max || N > b->max_blocks) return fail(ctx, ZP_EINVAL, "request %d: num_blocks %d outside [%d, %d]", n, N, b->N_max, b->max_blocks);
        if (slot[n] < 0 || slot[n] >= p->M) return fail(ctx, ZP_EINVAL, "request %d: query slot %d outside [0, %d)", n, slot[n], p->M);
        if (!slots_seen.insert(slot[n]).second) return fail(ctx, ZP_EINVAL, "request %d: query slot %d used twice", n, slot[n]);
        std::unordered_set<int> own;
        for (int i = 0; i < N; i++) {
            const int id = tbl[(size_t)n * b->max_blocks + i];
            if (id < 0 || id >= p->N_total) return fail(ctx, ZP_EINVAL, "request %d: block_table[%d] = %d outside the pool", n, i, id);
            if (!own.insert(id).second) return fail(ctx, ZP_EINVAL, "request %d: block %d appears twice in its table", n, id);
        }
        for (int i = 0; i < nt; i++) {
            const int src = tbl[(size_t)n * b->max_blocks + i];
            const int id = b->dst_table ? dst[(size_t)n * nt + i] : src;
            if (id < 0 || id >= p->N_total) return fail(ctx, ZP_EINVAL, "request %d: dst_table[%d] = %d outside the pool", n, i, id);
            if (id != src && sources.count(id)) return fail(ctx, ZP_EINVAL, "request %d: dst_table[%d] = %d is a source block of the batch but not its own block %d", n, i, id, src);
            if (!targets_seen.insert(id).second) return fail(ctx, ZP_EINVAL, "request %d: target block %d is written by two requests or twice", n, id);
        }
        for (int l = p->layer0; l < p->layer0 + p->L_slab; l++)
            for (int h = 0; h < p->h_kv; h++) {
                const size_t idx = (size_t)n * per + (size_t)l * p->h_kv + h;
                const int v = b->valid_len ? vl[idx] : (N - 1) * p->b;
                if (v < 0 || v > (N - 1) * p->b || v + p->b < p->w) return fail(ctx, ZP_EINVAL, "request %d layer %d head %d: valid_len %d out of range", n, l, h, v);
                const int k = b->keep ? keep[idx] : a.budget;
                const int cap = a.budget < v + p->b ? a.budget : v + p->b;
                if (k < p->w || k > cap) return fail(ctx, ZP_EINVAL, "request %d layer %d head %d: keep %d outside [%d, %d]", n, l, h, k, p->w, cap);
            }
    }
    return ZP_OK;
}

// ------------------------------------------------------------------ host planner
extern "C" zp_status zp_plan(int32_t B, int32_t N_max, int32_t max_blocks, int32_t N_total, const int32_t *block_table,
                             const int32_t *num_blocks, int32_t *refcnt, const int32_t *free_in, int32_t n_free_in,
                             int32_t *n_free_used, int32_t *dst_table, int32_t *new_table, int32_t *freed, int32_t *n_freed) {
    if (B < 0 || N_max < 2 || max_blocks < N_max || N_total <= 0) return fail(nullptr, ZP_EINVAL, "zp_plan: bad scalar argument");
    if (!block_table || !num_blocks || !refcnt || !n_free_used || !dst_table || !new_table || !freed || !n_freed || (n_free_in > 0 && !free_in))
        return fail(nullptr, ZP_EINVAL, "zp_plan: NULL argument");
    const int nt = N_max - 1;
    // pass 1: validate, and decide every target from the counts as they stand at entry
    std::vector<int32_t> targets((size_t)B * nt), reserved(B);
    std::vector<char> is_fresh((size_t)N_total, 0);
    std::vector<int32_t> uses((size_t)N_total, 0);
    int taken = 0;
    for (int n = 0; n < B; n++) {
        const int32_t *row = block_table + (size_t)n * max_blocks;
        const int N = num_blocks[n];
        if (N < N_max || N > max_blocks) return fail(nullptr, ZP_EINVAL, "zp_plan: request %d holds %d blocks, outside [%d, %d]", n, N, N_max, max_blocks);
        for (int i = 0; i < N; i++)
            if (row[i] < 0 || row[i] >= N_total || refcnt[row[i]] < 1)
                return fail(nullptr, ZP_EINVAL, "zp_plan: request %d block_table[%d] = %d is outside the pool or unreferenced", n, i, row[i]);
        for (int i = 0; i < N; i++)
            if (++uses[row[i]] > refcnt[row[i]])
                return fail(nullptr, ZP_EINVAL, "zp_plan: block %d is listed more often than its reference count", row[i]);
        for (int i = 0; i < nt; i++) {
            if (refcnt[row[i]] == 1) { targets[(size_t)n * nt + i] = row[i]; continue; }
            if (taken == n_free_in) return fail(nullptr, ZP_ENOMEM, "zp_plan: free list of %d blocks exhausted at request %d", n_free_in, n);
            const int f = free_in[taken++];
            if (f < 0 || f >= N_total || refcnt[f] != 0 || is_fresh[f]) return fail(nullptr, ZP_EINVAL, "zp_plan: free_in entry %d is not a free block", f);
            is_fresh[f] = 1;
            targets[(size_t)n * nt + i] = f;
        }
        int r = nt;
        while (r < N && refcnt[row[r]] != 1) r++;
        if (r == N) return fail(nullptr, ZP_EINVAL, "zp_plan: request %d has no private block at index >= %d to reserve", n, nt);
        reserved[n] = r;
    }
    // pass 2: commit
    std::vector<char> was_shared((size_t)N_total, 0);
    for (int n = 0; n < B; n++) {
        const int32_t *row = block_table + (size_t)n * max_blocks;
        for (int i = 0; i < num_blocks[n]; i++)
            if (refcnt[row[i]] > 1) was_shared[row[i]] = 1;
    }
    int nf = 0;
    for (int n = 0; n < B; n++) {
        const int32_t *row = block_table + (size_t)n * max_blocks;
        const int N = num_blocks[n];
        for (int i = 0; i < nt; i++) {
            const int32_t t = targets[(size_t)n * nt + i];
            dst_table[(size_t)n * nt + i] = t;
            new_table[(size_t)n * N_max + i] = t;
            if (is_fresh[t]) refcnt[t] = 1;
        }
        new_table[(size_t)n * N_max + nt] = row[reserved[n]];
        for (int i = 0; i < N; i++) {
            const int32_t p = row[i];
            if (was_shared[p]) {
                if (--refcnt[p] == 0) freed[nf++] = p;
            } else if (i >= nt && i != reserved[n]) {
                refcnt[p] = 0;
                freed[nf++] = p;
            }
        }
    }
    *n_free_used = taken;
    *n_freed = nf;
    return ZP_OK;
}
