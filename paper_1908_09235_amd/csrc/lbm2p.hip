// Host side of the lbm2p C ABI (include/lbm2p.h): descriptor validation,
// boundary tables, device memory, launches, checkpoints.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/lbm2p.h"
#include "domain.hpp"
#include "launch.hpp"

using namespace lbm;

namespace {

constexpr uint64_t kStateMagic = 0x6c626d3270737431ULL;  // "lbm2pst1"
constexpr int kProfPool = 1024;
constexpr int kTileH2 = 16;     // rows per segment of the two-step kernel
constexpr int kMinTileH2 = 4;

}  // namespace

namespace lbm {

// Nodes a pull reaches (x_ff of the quadratic interpolation lies two away),
// and a whole step of k_block.
static int block_pull(const lbm_domain* d) { return d->rule == LBM_RULE_IBB_QUADRATIC ? 2 : 1; }
static int block_reach(const lbm_domain* d) {
    return block_pull(d) + (d->eos == EOS_NONE ? 0 : 1);
}

bool domain_blockable(const lbm_domain* d) {
    return d->storage != LBM_STORE_F16NODE && d->rule != LBM_RULE_ZHAO_YONG;
}

long long domain_block_tiles(const lbm_domain* d, int steps, int lanes) {
    const int own = block_side(lanes) - 2 * steps * block_reach(d);
    if (own < 4) return 0;
    return (long long)((d->nx + own - 1) / own) * ((d->ny + own - 1) / own);
}

double single_us(size_t esize, double fluid) {
    return 8.0 + 18.0 * (double)esize * fluid * 1e-6 / (esize == 2 ? 3.7 : 4.6);
}

double block_us(const lbm_domain* d, int steps, long long tiles, int ncu, int lanes) {
    const bool two_phase = d->eos != EOS_NONE;
    struct Cost {
        double launch, step, shared;  // with a CU for each tile; more where tiles share one
        double tile, tile_step;       // each tile more than CUs
    };
    static const Cost costs[2][4] = {{{5.9, 2.1, 7.0, 0.0175, 0.0033},    // single phase: FP64
                                      {5.9, 2.1, 7.0, 0.0115, 0.0043},    // FP32, arithmetic FP64
                                      {5.4, 1.8, 7.0, 0.0135, 0.0014},    // FP32
                                      {5.4, 1.8, 7.0, 0.0059, 0.0033}},   // FP16
                                     {{6.4, 2.45, 4.0, 0.0163, 0.0037},   // two phases
                                      {6.4, 2.45, 4.0, 0.0095, 0.0053},
                                      {5.0, 2.05, 2.0, 0.0115, 0.0018},
                                      {5.0, 2.05, 2.0, 0.0059, 0.0033}}};
    const Cost& c = costs[two_phase][d->esize == 8                   ? 0
                                     : d->storage == LBM_STORE_F32   ? 1
                                     : d->esize == 4                 ? 2
                                                                     : 3];
    double us = (c.launch + c.step * steps) * (lanes == kBlockSmall ? 0.85 : 1.0);
    if (tiles > ncu) us += c.shared + (c.tile + c.tile_step * steps) * (double)(tiles - ncu);
    return us / steps;
}

BlockArgs block_args(const lbm_domain* d) {
    const BlockPlan& p = d->block;
    BlockArgs a{};
    for (int k = 0; k < 2; ++k) {
        a.f[k] = d->f[k];
        a.mom[k] = d->side_mom[k];
    }
    a.flags = d->flags;
    a.psiw = d->psiw;
    a.partial = p.partial[p.set];
    a.tiles = p.tiles;
    a.links = p.links;
    a.nodes = p.nodes;
    a.lc = d->lc;
    a.luw = d->luw;
    a.negrest = d->negrest;
    a.degen = d->degen;
    a.fix = d->fix;
    a.moving = p.moving ? 1 : 0;
    a.chi = d->rule == LBM_RULE_HALFWAY || d->rule == LBM_RULE_FH || d->rule == LBM_RULE_MLS;
    a.max_len = p.max_len;
    a.nx = d->nx;
    a.ny = d->ny;
    a.pitch = d->pitch;
    a.plane = d->plane;
    a.halo = p.halo;
    a.pull = p.pull;
    a.ntiles = p.ntiles;
    a.max_nodes = p.max_nodes;
    a.mom_bytes = (unsigned)(3 * std::max(d->nslots, 1) * 8);
    a.link_bytes = p.link_bytes;
    a.node_bytes = p.node_bytes;
    a.open_x = d->open_x;
    a.inlet_u = d->inlet_u;
    a.mass = d->mass;
    a.hist = d->hist;
    a.cap = d->cap;
    a.unstable = d->unstable;
    a.ph64 = d->ph64;
    a.ph32 = phys_as<float>(d->ph64);
    return a;
}

}  // namespace lbm

namespace {

int dev_alloc(lbm_domain* d, void** p, size_t bytes) {
    if (bytes == 0) bytes = 8;
    if (d->arena) {
        *p = d->arena->alloc(bytes);
        if (!*p) return LBM_ENOMEM;
    } else if (hipMalloc(p, bytes) != hipSuccess) {
        *p = nullptr;
        return LBM_ENOMEM;
    }
    d->allocs.push_back(*p);
    d->bytes += bytes;
    return LBM_OK;
}

void dev_free(lbm_domain* d, void* p, size_t bytes) {
    if (d->arena) d->arena->release(p);
    else (void)hipFree(p);
    d->allocs.erase(std::find(d->allocs.begin(), d->allocs.end(), p));
    d->bytes -= bytes;
}

// host vectors stay alive until the creating call synchronises the stream
template <typename T>
int upload(lbm_domain* d, T** dst, const std::vector<T>& src) {
    int rc = dev_alloc(d, reinterpret_cast<void**>(dst), src.size() * sizeof(T));
    if (rc) return rc;
    if (!src.empty() && hipMemcpyAsync(*dst, src.data(), src.size() * sizeof(T),
                                       hipMemcpyHostToDevice, d->stream) != hipSuccess)
        return LBM_EDEVICE;
    return LBM_OK;
}

void drop_graphs(lbm_domain* d) {
    for (auto& row : d->graphs)
        for (hipGraphExec_t& g : row) {
            if (g) (void)hipGraphExecDestroy(g);
            g = nullptr;
        }
}

void free_domain(lbm_domain* d) {
    if (!d) return;
    // queued work on the domain's stream may still use the memory
    (void)hipStreamSynchronize(d->stream);
    if (d->arena) {
        for (void* p : d->allocs) d->arena->release(p);
    } else {
        for (void* p : d->allocs) (void)hipFree(p);
    }
    for (hipEvent_t e : d->ev) (void)hipEventDestroy(e);
    drop_graphs(d);
    if (d->cap_stream) (void)hipStreamDestroy(d->cap_stream);
    delete d;
}

inline int wrapi(int i, int n) { return ((i % n) + n) % n; }

// Rows per tile.  A tile's rows are worked one after another, in rotations of
// three, so a lattice with few tiles lasts as long as one tile: it is cut into
// as many as the chip holds wavefronts for (4 a SIMD, 4096 in all), each row
// of halos more being a cost only once the chip is full.  Main and boundary
// launch, us a step, 64 columns by 3 / 6 / 9 rows and the former default (9
// rows, the width below), droplet in FP64 storage (FP32): 128^2 11.1 / 13.9 /
// 16.8 and 16.8; 400^2 13.3 / 15.9 / 18.7 and 18.7 (12.2 / 15.2 / 18.4); 600 x
// 500 17.0 / 17.8 / 20.6 and 23.9; 800^2 24.6 / 23.2 / 25.8 and 25.6 (20.8 /
// 21.0 / 24.2 and 24.8); 1024^2 33.0 / 31.4 / 31.9 and 31.7 (26.3 / 24.7 /
// 25.2 and 29.3); 1500 x 1400 77.8 / 73.0 / 72.4 and 71.2.
constexpr long long kSmallNodes = 500000;   // 3 rows
constexpr long long kMediumNodes = 1200000; // 6 rows
// The FP16 per-node form, whose halo rows cost most, takes 15 rows of large
// lattices: 3999 x 2001 9 rows 112.0, 15 rows 111.9; 4096^2 215.2 and 212.1; 6000 x
// 3000 225.2 and 216.7; 8192 x 4096 398.5 and 387.0 (256 columns).
constexpr long long kLargeNodes = 12000000;
int default_tile_h(int nx, int ny, int storage) {
    const long long n = (long long)nx * ny;
    if (storage == LBM_STORE_F16NODE && n > kLargeNodes) return 15;
    return n <= kSmallNodes ? 3 : n <= kMediumNodes ? 6 : 9;
}

// Columns per tile: 64 where there are few tiles (above).  Otherwise the
// widest workgroup whose share of lanes that update a node is within 10 % of
// the best width's (wider strips re-read fewer halo columns and measure
// faster at equal share); within 2 % for the FP16 per-node form, whose rings
// of densities make idle lanes dearer (2048^2: 68.9 us a step with 256 columns
// and a share of 0.89, 62.2 with 128 and 0.94; 3999 x 2001, 0.98 either way:
// 109.1 and 111.4).  Its tiles of 64 columns hold as much LDS as the wider ones,
// for a quarter of the wavefronts, so beyond small lattices a share of theirs
// counts less (64, 128 and 256 columns: 1200 x 1000 by 6 rows 35.3, 30.5 and 31.9;
// 1408^2 by 9 rows 45.3, 38.8 and 39.6 with shares of 0.96, 0.92 and 0.92; 2048^2
// 71.9, 64.2 and 70.2).
int default_tile_w(int nx, int ny, int storage) {
    const bool node = storage == LBM_STORE_F16NODE;
    if ((long long)nx * ny <= (node ? kSmallNodes : kMediumNodes)) return 64;
    double eff[3], best = 0.0;
    const int ws[3] = {256, 128, 64};
    const double near = node ? 0.98 : 0.9;
    for (int k = 0; k < 3; ++k) {
        const int ns = (nx + strip_cols(ws[k]) - 1) / strip_cols(ws[k]);
        eff[k] = (double)nx / ((double)ns * ws[k]);
        if (node && ws[k] == 64) eff[k] *= 0.88;
        best = std::max(best, eff[k]);
    }
    for (int k = 0; k < 3; ++k)
        if (eff[k] >= near * best) return ws[k];
    return 64;
}

inline long long storage_bytes(int storage) {
    return storage == LBM_STORE_F64 ? 8
           : (storage == LBM_STORE_F16DEV || storage == LBM_STORE_F16NODE) ? 2
                                                                            : 4;
}

template <typename R>
Phys<R> make_phys(const lbm_desc* s) {
    Phys<R> p{};
    p.G = R(s->G);
    p.gx = R(s->gravity[0]);
    p.gy = R(s->gravity[1]);
    p.e0 = R(s->eos_param[0]);
    p.e1 = R(s->eos_param[1]);
    p.e2 = R(s->eos_param[2]);
    p.e3 = R(s->eos_param[3]);
    p.p2G = R(s->G != 0.0 ? 2.0 / s->G : 0.0);
    // BGK is the moment-space collision with every rate 1/tau
    for (int i = 0; i < 9; ++i) {
        const double si = s->collision == LBM_COLL_MRT ? s->mrt_s[i] : 1.0 / s->tau;
        p.s[i] = R(si);
        p.h[i] = R(1.0 - 0.5 * si);
    }
    return p;
}

double host_psi(int eos, const Phys<double>& p, double rho) {
    if (eos == EOS_EXP) return psi_of<EOS_EXP, double>(rho, p);
    if (eos == EOS_CS) return psi_of<EOS_CS, double>(rho, p);
    return 0.0;
}

// Whether psi of the Carnahan-Starling EOS is finite at the fluid nodes of a
// row: its square is neither negative nor infinite nor NaN.  (The host's fma is
// a call unless the function is compiled for processors that have it: 24 ms at
// 2048 x 2048 with calls and a square root a node, 3 ms so.)
#if !defined(__HIP_DEVICE_COMPILE__)
__attribute__((target_clones("arch=x86-64-v3", "default")))
#endif
bool cs_psi_finite(const double* rho, const uint8_t* solid, int n, const Phys<double>& p) {
    int bad = 0;
    for (int i = 0; i < n; ++i) {
        const double v = cs_psi_squared<double>(rho[i], p);
        bad |= (solid[i] == 0) & !(v >= 0.0 && v <= DBL_MAX);
    }
    return bad == 0;
}

// ---------------------------------------------------------------- launches
Ctx ctx(lbm_domain* d) {
    Ctx c{};
    c.nx = d->nx;
    c.ny = d->ny;
    c.pitch = d->pitch;
    c.plane = d->plane;
    c.eos = d->eos;
    c.storage = d->storage;
    c.tile_w = d->tile_w;
    c.tile_h = seg_rows(d->tile_h);
    c.nsegs = d->nsegs;
    c.nstrips = d->nstrips;
    c.nblocks = d->nblocks;
    c.flags = d->flags;
    c.side_idx = d->side_idx;
    c.psiw = d->psiw;
    c.side_mom = d->side_mom[d->cur ^ 1];  // a pass writes those of the buffer it fills
    c.side_f = d->side_f;
    c.side_mom_bytes = (unsigned)(3 * std::max(d->nslots, 1) * 8);
    c.side_f_bytes = (unsigned)(9 * (d->save_f ? std::max(d->nslots, 1) : 1) * 8);
    c.save_f = d->save_f;
    c.partial = d->partial;
    c.mass = d->mass;
    const size_t nn = (size_t)d->nx * d->ny;
    for (int k = 0; k < 3; ++k) c.mom_out[k] = d->mom_out ? d->mom_out + k * nn : nullptr;
    c.ref = nullptr;
    c.ph = d->ph64;
    c.stream = d->stream;
    c.tile_h2 = seg_rows(d->tile_h2);
    c.nsegs2 = d->nsegs2;
    c.nstrips2 = d->nstrips2;
    c.nblocks2 = d->nblocks2;
    c.node_link = d->node_link;
    c.tile_order = d->tile_order;
    c.partial2 = d->partial + d->partial_cap;
    c.lmeta = d->lmeta;
    c.lc = d->lc;
    c.luw = d->luw;
    c.negrest = d->negrest;
    c.degen = d->degen;
    c.fix = d->fix;
    return c;
}

// ev: optional start and end events that the launch records itself
void launch_main(lbm_domain* d, const void* src, void* dst, bool moments,
                 const hipEvent_t* ev = nullptr) {
    Ctx c = ctx(d);
    if (ev) {
        c.ev_start = ev[0];
        c.ev_stop = ev[1];
    }
    if (d->storage == LBM_STORE_F64) launch_main_f64(c, src, dst, moments);
    else launch_main_f32(c, src, dst, moments);
}

int link_blocks(const lbm_domain* d) { return (d->nslot_links + 255) / 256; }

MassPass mass_pass(lbm_domain* d) {
    MassPass r{};
    r.steps = d->pending_steps;
    if (d->pending_block) {
        r.partial = d->block.partial[d->block.set];
        r.np = d->block.ntiles;
        r.stride = r.np;
    } else {
        r.partial = d->partial;
        r.np = d->pending_steps == 2 ? d->nblocks2 : d->nblocks;
        r.stride = d->partial_cap;
    }
    r.unit = mass_unit(d->mass.magic);
    r.hist = d->hist;
    r.cap = d->cap;
    r.clock = d->clock;
    r.unstable = d->unstable;
    return r;
}

BndArgs bnd_args(lbm_domain* d) {
    BndArgs b{};
    b.nslot = d->nslot_links;
    b.lnode = d->lnode;
    b.lmeta = d->lmeta;
    b.lghost = d->lghost;
    b.lxf = d->lxf;
    b.lxff = d->lxff;
    b.lslotb = d->lslotb;
    b.lslotf = d->lslotf;
    b.lc = d->lc;
    b.luw = d->luw;
    b.side_mom = d->side_mom[d->cur];
    b.side_f = d->side_f;
    b.plane = d->plane;
    b.rref = d->ph64.rref;
    b.lref = d->lref;
    b.fix = d->fix;
    b.prev = mass_pass(d);
    b.do_reduce = d->pending ? 1 : 0;
    b.force = d->force;
    b.negrest = d->negrest;
    b.degen = d->degen;
    b.nlink_blocks = link_blocks(d);
    b.open_x = d->open_x;
    b.nx = d->nx;
    b.ny = d->ny;
    b.pitch = d->pitch;
    b.inlet_u = d->inlet_u;
    return b;
}

void launch_boundary(lbm_domain* d, void* cur, const hipEvent_t* ev = nullptr) {
    BndArgs b = bnd_args(d);
    // link blocks, then the open rows, then the block that reduces
    const int nbb = b.nlink_blocks + (d->open_x ? (d->ny + 255) / 256 : 0) + 1;
    Ctx c = ctx(d);
    if (ev) {
        c.ev_start = ev[0];
        c.ev_stop = ev[1];
    }
    if (d->storage == LBM_STORE_F64) launch_boundary_f64(c, cur, b, nbb);
    else launch_boundary_f32(c, cur, b, nbb);
    d->pending = false;
    d->force_valid = true;
}

void reduce_pending(lbm_domain* d) {
    if (!d->pending) return;
    launch_reduce(ctx(d), mass_pass(d));
    d->pending = false;
}

int ensure_events(lbm_domain* d) {
    while ((int)d->ev.size() < 4 * kProfPool) {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) return LBM_EDEVICE;
        d->ev.push_back(e);
    }
    return LBM_OK;
}

// add the recorded launch durations to the totals and free the pool
int harvest(lbm_domain* d) {
    if (d->nrec == 0) return LBM_OK;
    if (hipEventSynchronize(d->ev[4 * (d->nrec - 1) + 3]) != hipSuccess) return LBM_EDEVICE;
    for (int i = 0; i < d->nrec; ++i) {
        float a = 0, b = 0;
        if (hipEventElapsedTime(&a, d->ev[4 * i + 0], d->ev[4 * i + 1]) != hipSuccess ||
            hipEventElapsedTime(&b, d->ev[4 * i + 2], d->ev[4 * i + 3]) != hipSuccess)
            return LBM_EDEVICE;
        d->bnd_ms += a;
        d->main_ms += b;
    }
    d->bnd_n += d->nrec;
    d->main_n += d->nrec;
    d->nrec = 0;
    return LBM_OK;
}

// One pass as plain launches: boundary pass on f*(t) (which also records
// the masses of the previous pass), then the main pass f*(t) -> f*(t + 1),
// or with two = true f*(t) -> f*(t + 2).  With rec, HIP events bracket
// both launches.
void launch_pass(lbm_domain* d, bool two, hipEvent_t* rec) {
    void* cur = d->f[d->cur];
    void* nxt = d->f[d->cur ^ 1];
    // with rec, each launch records its own start and end (rec[0..1]: the
    // boundary pass, rec[2..3]: the main pass)
    launch_boundary(d, cur, rec);
    if (two) {
        Ctx c = ctx(d);
        if (rec) {
            c.ev_start = rec[2];
            c.ev_stop = rec[3];
        }
        launch_main2_f32(c, cur, nxt);
    } else {
        launch_main(d, cur, nxt, false, rec ? rec + 2 : nullptr);
    }
    d->cur ^= 1;
    d->t += two ? 2 : 1;
    d->pending = true;
    d->pending_steps = two ? 2 : 1;
    d->pending_block = false;
    d->pending_t = d->t;
    d->last_fused = two;
    d->replay_valid = false;
}

// Runs of steps go through k_block where the domain has a plan for it, also
// with two steps per pass asked for, but for rows per tile asked for with them,
// which name the two-step kernel, and for large two-phase domains, of which a
// step in blocks works the halos twice over (a single phase needs half of them).
// us a step in blocks and in the two-step kernel by its default rows, FP32
// arithmetic (FP32 deviations):
//   without walls   1024^2 14.8 and 22.1, 2048^2 58.6 and 49.1, 8192 x 4096 412
//     and 330: the two-step kernel from three million nodes on;
//   with walls its launch waits for the tiles that hold most of them, until
//   there are enough others, and each link costs it four times as much: 24
//     to 60 cylinders, 4096 x 2048 110 and 126 (114, 126), 4096 x 3000 154 and 155
//     (163, 155), 4096 x 3500 180 and 171 (191, 171), 8192 x 4096 414 and 386 (435,
//     386); 4096^2 with links to 0.3 % of the nodes 207 and 195, 1.1 % 220 and 254,
//     1.6 % 227 and 282;
//   single phase    2048^2 37.2 and 45.4, 8192 x 4096 268 and 322, 4096^2 with
//     pillars 171 and 409: blocks.
bool uses_blocks(const lbm_domain* d) {
    if (d->block.steps == 0) return false;
    if (d->fused != 2) return true;
    if (d->tile_h2_asked) return false;
    if (d->eos == LBM_EOS_NONE) return true;
    if (d->nl == 0) return d->fluid <= 3000000;
    return d->fluid <= 13000000 || 200LL * d->nl >= d->fluid;
}

// k steps in one launch of k_block, which also records the masses of the
// previous one.
void launch_block(lbm_domain* d, int k) {
    BlockPlan& p = d->block;
    BlockKernarg arg{};
    arg.r.cur = d->cur;
    arg.r.steps = k;
    arg.r.prev = mass_pass(d);
    arg.r.do_reduce = d->pending ? 1 : 0;
    p.set ^= 1;
    arg.a = block_args(d);
    const unsigned lds = block_lds(p.max_nodes);
    if (d->storage == LBM_STORE_F64) launch_block_f64(ctx(d), arg, p.lanes, lds);
    else launch_block_f32(ctx(d), arg, p.lanes, lds);
    d->cur ^= 1;
    d->t += k;
    d->pending = true;
    d->pending_steps = k;
    d->pending_block = true;
    d->pending_t = d->t;
    d->last_fused = false;
    d->replay_valid = false;
}

// The passes of n steps: two steps each when the domain fuses them, with
// a single step last if n is odd.
template <typename F>
void for_passes(const lbm_domain* d, int64_t n, F&& pass) {
    for (int64_t i = 0; i < n;) {
        const bool two = d->fused == 2 && n - i >= 2;
        pass(two);
        i += two ? 2 : 1;
    }
}

// Steps with kernel timing: plain launches, events on the passes that
// start at a multiple of prof steps.  (The caller has reduced any pending
// mass.)
int run_steps_profiled(lbm_domain* d, int64_t n) {
    int rc = LBM_OK;
    for_passes(d, n, [&](bool two) {
        if (rc) return;
        const bool rec = (d->t % d->prof) == 0 || (two && ((d->t + 1) % d->prof) == 0);
        if (rec && d->nrec == kProfPool) rc = harvest(d);
        if (rc) return;
        launch_pass(d, two, rec ? &d->ev[4 * d->nrec] : nullptr);
        if (rec) d->nrec++;
    });
    if (rc) return rc;
    reduce_pending(d);
    return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

// The graph of 2^level steps that starts with f*(t) in buffer `parity`:
// the passes' launches and the closing reduction, captured on the
// domain's capture stream (the kernels only read the step from the device
// clock, so every replay continues where the last one stopped).  Null if
// capture is not available.
hipGraphExec_t step_graph(lbm_domain* d, int parity, int level) {
    hipGraphExec_t& g = d->graphs[parity][level];
    if (g || d->graphs_off) return g;
    if (!d->cap_stream &&
        hipStreamCreateWithFlags(&d->cap_stream, hipStreamNonBlocking) != hipSuccess) {
        d->cap_stream = nullptr;
        d->graphs_off = true;
        (void)hipGetLastError();
        return nullptr;
    }
    // replay the bookkeeping of plain launches on a copy of the host state
    const int cur0 = d->cur, ps0 = d->pending_steps;
    const long long t0 = d->t, pt0 = d->pending_t;
    const bool p0 = d->pending, lf0 = d->last_fused, rv0 = d->replay_valid;
    const hipStream_t s0 = d->stream;
    d->cur = parity;
    d->pending = false;
    d->stream = d->cap_stream;
    hipGraph_t graph = nullptr;
    bool ok = hipStreamBeginCapture(d->stream, hipStreamCaptureModeThreadLocal) == hipSuccess;
    if (ok) {
        for_passes(d, 1LL << level, [&](bool two) { launch_pass(d, two, nullptr); });
        reduce_pending(d);
        ok = hipStreamEndCapture(d->stream, &graph) == hipSuccess && graph;
    }
    if (ok) ok = hipGraphInstantiate(&g, graph, nullptr, nullptr, 0) == hipSuccess;
    if (graph) (void)hipGraphDestroy(graph);
    d->cur = cur0;
    d->t = t0;
    d->pending = p0;
    d->pending_steps = ps0;
    d->pending_t = pt0;
    d->last_fused = lf0;
    d->replay_valid = rv0;
    d->stream = s0;
    if (!ok) {
        g = nullptr;
        d->graphs_off = true;
        (void)hipGetLastError();
    }
    return g;
}

// n steps: replays of captured runs of 32, 16, ..., 1 steps (plain
// launches where capture is not available or kernels are being timed).
int run_steps(lbm_domain* d, int64_t n) {
    reduce_pending(d);  // every run below starts with no mass pending
    if (d->prof > 0) return run_steps_profiled(d, n);
    const bool blocks = uses_blocks(d) && !(n > 1 && being_captured(d->stream));
    if (blocks && n > 1) {
        // the last step is a pass of its own: it leaves f*(t - 1) with the
        // ghosts of step t and the wall force, which the read-outs use
        while (n > 1) {
            const int k = (int)std::min<int64_t>(n - 1, d->block.steps);
            // (a launch of one step costs more than a pass, but for the
            // smallest domains, where the launches are the cost)
            if (k == 1 && d->block.lanes == kBlockThreads) launch_pass(d, false, nullptr);
            else launch_block(d, k);
            n -= k;
        }
        launch_pass(d, false, nullptr);
        reduce_pending(d);
        return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
    }
    while (n > 0) {
        int level = lbm_domain::kGraphLevels - 1;
        while ((1LL << level) > n) --level;
        const long long k = 1LL << level;
        if (!d->graphs[d->cur][level] && !d->graphs_off) {
            // all runs for both parities at once, so that later calls of
            // any length replay without capturing
            // (with k_block only single steps come here)
            const int levels = blocks ? 1 : lbm_domain::kGraphLevels;
            for (int par = 0; par < 2; ++par)
                for (int lv = 0; lv < levels; ++lv) (void)step_graph(d, par, lv);
        }
        hipGraphExec_t g = d->graphs_off ? nullptr : d->graphs[d->cur][level];
        if (g) {
            if (hipGraphLaunch(g, d->stream) != hipSuccess) return LBM_EDEVICE;
            // the bookkeeping the captured passes did
            for_passes(d, k, [&](bool two) {
                d->cur ^= 1;
                d->t += two ? 2 : 1;
                d->last_fused = two;
            });
            d->pending_t = d->t;
            d->replay_valid = false;
        } else {
            for_passes(d, k, [&](bool two) { launch_pass(d, two, nullptr); });
            reduce_pending(d);
        }
        n -= k;
    }
    return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

int check_unstable(lbm_domain* d) {
    long long u = -1;
    if (hipMemcpyAsync(&u, d->unstable, sizeof(u), hipMemcpyDeviceToHost, d->stream) != hipSuccess)
        return LBM_EDEVICE;
    if (hipStreamSynchronize(d->stream) != hipSuccess) return LBM_EDEVICE;
    return u >= 0 ? LBM_EUNSTABLE : LBM_OK;
}

// Dispatch order of the two-step pass's tiles: the tiles whose strip and
// rows hold the most boundary nodes first, the others in the XCD order of
// xcd_tile.  A tile that evaluates wall rules in many of its rows lasts
// several times as long as one without walls; started last, such tiles
// would leave the launch waiting on a few of them.  A tile's weight is the
// number of boundary nodes in the rows whose wall rules it evaluates
// (y0 - 1 .. y0 + H) and the 64 columns of its wavefront (x0 - 4 ..
// x0 + 59).  Only the order changes: every tile writes its own partials.
int order_tiles(lbm_domain* d) {
    if (!d->tile_order) return LBM_OK;
    const int ns = d->nstrips2, ng = d->nsegs2, n = d->nblocks2;
    const int H = seg_rows(d->tile_h2);
    const int nx = d->nx, ny = d->ny;
    std::vector<long long> w((size_t)n, 0);
    auto wrap = [](long long v, long long m) { return (int)(((v % m) + m) % m); };
    for (size_t i = 0; i < d->bnd_x.size(); ++i) {
        const int x = d->bnd_x[i], y = d->bnd_y[i];
        const int s0 = (int)((long long)x * ns / nx), g0 = y / H;
        for (int ds = -1; ds <= 1; ++ds) {
            const int s = wrap(s0 + ds, ns);
            const int x0 = (int)((long long)s * nx / ns);
            if (wrap((long long)x - (x0 - kF2Halo), nx) >= kF2Lanes) continue;
            for (int dg = -1; dg <= 1; ++dg) {
                const int g = wrap(g0 + dg, ng);
                const int y0 = g * H, h = std::min(H, ny - y0);
                if (wrap((long long)y - (y0 - 1), ny) >= h + 2) continue;
                w[(size_t)g * ns + s] += 1;
            }
        }
    }
    std::vector<int> nat((size_t)n), pos((size_t)n), order((size_t)n);
    for (int b = 0; b < n; ++b) {
        nat[b] = xcd_tile(b, n);
        pos[b] = b;
    }
    std::stable_sort(pos.begin(), pos.end(),
                     [&](int a, int b) { return w[nat[a]] > w[nat[b]]; });
    for (int b = 0; b < n; ++b) order[b] = nat[pos[b]];
    if (hipMemcpyAsync(d->tile_order, order.data(), (size_t)n * 4, hipMemcpyHostToDevice,
                       d->stream) != hipSuccess ||
        hipStreamSynchronize(d->stream) != hipSuccess)
        return LBM_EDEVICE;
    return LBM_OK;
}

// -------------------------------------------------------------- creation
struct LinkRec {
    int node;  // x_b index in y*nx + x
    int dir;
    int src;   // index in the descriptor
};

// Tables of k_block for `steps` steps per launch: per tile the cut links
// whose fluid node its region pulls, grouped by node in chunks of 64, and the
// nodes whose moments they read.  False if a tile holds more than a workgroup
// has lanes or LDS for.
struct BlockTables {
    int steps = 0, lanes = 0, halo = 0, pull = 0, nstrips = 0, nsegs = 0, max_nodes = 0, max_len = 0;
    std::vector<BlockTile> tiles;
    std::vector<BlockLink> links;
    std::vector<BlockNode> nodes;
};
// What the plan says of them.
void block_plan(lbm_domain* d, const BlockTables& b) {
    BlockPlan& p = d->block;
    p.halo = b.halo;
    p.pull = b.pull;
    p.nstrips = b.nstrips;
    p.nsegs = b.nsegs;
    p.ntiles = b.nstrips * b.nsegs;
    p.max_nodes = b.max_nodes;
    p.max_len = b.max_len;
    p.link_bytes = (unsigned)(b.links.size() * sizeof(BlockLink));
    p.node_bytes = (unsigned)(b.nodes.size() * sizeof(BlockNode));
    p.steps = b.steps;
    p.lanes = b.lanes;
}
bool block_tables(const lbm_domain* d, int steps, int lanes, const LinkTables& lt, BlockTables& b) {
    const std::vector<int>&lnode = lt.node, &lmeta = lt.meta, &lslotb = lt.slotb,
                    &lslotf = lt.slotf;
    const std::vector<double>& lc = lt.c;
    b = BlockTables{};
    b.steps = steps;
    b.lanes = lanes;
    const int W = block_side(lanes);
    b.pull = block_pull(d);
    b.halo = steps * block_reach(d);
    const int own = W - 2 * b.halo;
    if (own < 1) return false;
    b.nstrips = (d->nx + own - 1) / own;
    b.nsegs = (d->ny + own - 1) / own;
    if ((long long)b.nstrips * b.nsegs > kBlockTiles) return false;
    // the regions (and the place in them) that pull a column or row
    auto places = [&](int n, int parts, int width) {
        std::vector<std::vector<std::pair<int, int>>> v((size_t)n);
        for (int s = 0; s < parts; ++s) {
            const int x0 = (int)((long long)s * n / parts);
            for (int l = b.pull; l < width - b.pull; ++l)
                v[(size_t)wrapi(x0 - b.halo + l, n)].push_back({s, l});
        }
        return v;
    };
    const auto X = places(d->nx, b.nstrips, W), Y = places(d->ny, b.nsegs, W);
    auto tile_of = [&](int strip, int seg) {
        const int band = seg / 8, h = std::min(8, b.nsegs - 8 * band);
        return band * 8 * b.nstrips + strip * h + (seg - 8 * band);
    };
    struct Image {
        int k0, at;  // first link of the node, local index
    };
    const int nt = b.nstrips * b.nsegs, P = d->pitch;
    std::vector<int> first((size_t)nt + 1, 0);
    auto images = [&](auto&& take) {
        for (size_t k = 0; k < lnode.size();) {
            if (((lmeta[k] >> 4) & 15) == LK_PAD) {
                ++k;
                continue;
            }
            for (const auto& y : Y[(size_t)(lnode[k] / P)])
                for (const auto& x : X[(size_t)(lnode[k] % P)])
                    take(tile_of(x.first, y.first), (int)k, y.second * W + x.second);
            k += (size_t)((lmeta[k] >> 8) & 15);
        }
    };
    images([&](int tile, int, int) { ++first[(size_t)tile + 1]; });
    for (int i = 0; i < nt; ++i) first[(size_t)i + 1] += first[(size_t)i];
    std::vector<Image> im((size_t)first[(size_t)nt]);
    {
        std::vector<int> at(first.begin(), first.end() - 1);
        images([&](int tile, int k, int l) { im[(size_t)at[(size_t)tile]++] = Image{k, l}; });
    }
    std::vector<int> rec((size_t)W * W, -1);
    b.tiles.resize((size_t)nt);
    for (int i = 0; i < nt; ++i) {
        const int2 g = block_place(i, b.nstrips, b.nsegs);
        const int x0 = (int)((long long)g.x * d->nx / b.nstrips);
        const int y0 = (int)((long long)g.y * d->ny / b.nsegs);
        const int x1 = (int)((long long)(g.x + 1) * d->nx / b.nstrips);
        const int y1 = (int)((long long)(g.y + 1) * d->ny / b.nsegs);
        auto is_own = [&](int l) {
            const int lx = l % W - b.halo, ly = l / W - b.halo;
            return lx >= 0 && lx < x1 - x0 && ly >= 0 && ly < y1 - y0;
        };
        const int link0 = (int)b.links.size(), node0 = (int)b.nodes.size();
        auto record = [&](int l, int slot) {
            if (rec[(size_t)l] < 0) {
                rec[(size_t)l] = (int)b.nodes.size() - node0;
                b.nodes.push_back(BlockNode{slot, (unsigned short)l, (unsigned char)is_own(l), 0});
            }
            return rec[(size_t)l];
        };
        BlockLink pad{};
        pad.meta = LK_PAD << 4 | 1;
        pad.xb = 2 * W + 2;
        for (int e = first[(size_t)i]; e < first[(size_t)i + 1]; ++e) {
            const int k0 = im[(size_t)e].k0, l = im[(size_t)e].at;
            const int len = (lmeta[(size_t)k0] >> 8) & 15;
            b.max_len = std::max(b.max_len, len);
            const int used = ((int)b.links.size() - link0) % 64;
            if (used + len > 64) b.links.resize(b.links.size() + (size_t)(64 - used), pad);
            const int sb = record(l, lslotb[(size_t)k0]);
            b.nodes[(size_t)(node0 + sb)].bnd = 1;
            for (int k = k0; k < k0 + len; ++k) {
                const int a = lmeta[(size_t)k] & 15;
                int sf = 0;
                if (lslotf[(size_t)k] >= 0)
                    sf = record(l - cx(a) - cy(a) * W, lslotf[(size_t)k]);
                BlockLink r{};
                r.meta = lmeta[(size_t)k];
                r.id = k;
                r.xb = (unsigned short)l;
                r.sb = (unsigned short)sb;
                r.sf = (unsigned short)sf;
                r.own = (unsigned short)is_own(l);
                const double* const c = lc.data() + 8 * (size_t)k;
                const bool chi = ((lmeta[(size_t)k] >> 4) & 15) <= LK_CHI_EXT;
                r.k[0] = chi ? c[3] : c[0];
                r.k[1] = chi ? c[4] : c[1];
                b.links.push_back(r);
            }
        }
        const int used = ((int)b.links.size() - link0) % 64;
        if (used) b.links.resize(b.links.size() + (size_t)(64 - used), pad);
        const int chunks = ((int)b.links.size() - link0) / 64;
        const int nn = (int)b.nodes.size() - node0;
        for (int k = node0; k < node0 + nn; ++k) rec[(size_t)b.nodes[(size_t)k].at] = -1;
        if (chunks > kBlockThreads / 64 || nn > kBlockNodes || b.links.size() >= (1u << 25))
            return false;
        b.max_nodes = std::max(b.max_nodes, nn);
        b.tiles[(size_t)i] = BlockTile{link0, chunks, node0, nn, x0, y0, x1 - x0, y1 - y0};
    }
    return true;
}

// (no tables either where the host has no memory for them)
bool try_block_tables(const lbm_domain* d, int steps, int lanes, const LinkTables& lt,
                      BlockTables& b) {
    try {
        return block_tables(d, steps, lanes, lt, b);
    } catch (const std::bad_alloc&) {
        return false;
    }
}

// Whether and how the domain's runs go through k_block: the number of steps
// per launch with the least estimated time, if that is below single steps'
// (the tables of none otherwise).
int plan_blocks(lbm_domain* d, const LinkTables& lt, BlockTables& b) {
    if (d->arena || !domain_blockable(d)) return LBM_OK;
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return LBM_EDEVICE;
    int steps = 0, lanes = kBlockThreads;
    double best = single_us(d->esize, (double)d->fluid);
    for (int n : {2 * kBlockThreads, kBlockSmall})
        for (int k = 2; k <= kBlockSteps; ++k) {
            const long long tiles = domain_block_tiles(d, k, n);
            if (tiles == 0) continue;
            if (n == kBlockSmall && (tiles > ncu || d->eos != EOS_NONE)) continue;
            const int w = tiles <= ncu ? n : kBlockThreads;
            const double us = block_us(d, k, tiles, ncu, w);
            if (us < best) {
                best = us;
                steps = k;
                lanes = w;
            }
        }
    if (steps > 0 && !try_block_tables(d, steps, lanes, lt, b)) b.steps = 0;
    return LBM_OK;
}

// The tables on the device, and moments of its own for each buffer (a launch
// reads those of one time and writes those of another; single steps write
// in place).  Last in the creation, when the initial fields have been given
// back, so that a plan takes no memory that the rest of it needs.  The caller
// waits for the stream before b ends.
int place_blocks(lbm_domain* d, const BlockTables& b) {
    if (b.steps == 0) return LBM_OK;
    BlockPlan& p = d->block;
    const size_t tiles = b.tiles.size() * sizeof(BlockTile);
    const size_t links = b.links.size() * sizeof(BlockLink);
    const size_t nodes = b.nodes.size() * sizeof(BlockNode);
    const size_t part = (size_t)b.steps * b.tiles.size() * sizeof(MassTile);
    const size_t mom = (size_t)3 * std::max(d->nslots, 1) * 8;
    // one piece of memory; a domain that leaves no room for it takes single steps
    char* m = nullptr;
    auto up = [](size_t n) { return (n + 255) & ~size_t(255); };
    const int rc =
        dev_alloc(d, (void**)&m, up(tiles) + up(links) + up(nodes) + 2 * up(part) + up(mom));
    if (rc) {
        (void)hipGetLastError();
        return LBM_OK;
    }
    auto place = [&](auto*& q, size_t n) {
        q = reinterpret_cast<std::remove_reference_t<decltype(q)>>(m);
        m += up(n);
    };
    place(p.tiles, tiles);
    place(p.links, links);
    place(p.nodes, nodes);
    place(p.partial[0], part);
    place(p.partial[1], part);
    place(d->side_mom[1], mom);
    auto put = [&](void* dst, const void* src, size_t n) {
        return n == 0 ||
               hipMemcpyAsync(dst, src, n, hipMemcpyHostToDevice, d->stream) == hipSuccess;
    };
    if (!put(p.tiles, b.tiles.data(), tiles) || !put(p.links, b.links.data(), links) ||
        !put(p.nodes, b.nodes.data(), nodes))
        return LBM_EDEVICE;
    block_plan(d, b);
    return LBM_OK;
}

// The unit of the mass sums (see MassUnit) from the largest initial density.
MassUnit mass_unit_for(const lbm_desc* s, long long n) {
    double mx = 0.0;
    for (long long i = 0; i < n; ++i)
        if (!s->solid[i] && s->rho0[i] > mx) mx = s->rho0[i];
    // (a range in which neither the unit nor its inverse leaves FP64; smaller
    // densities are rests, down to the smallest normal numbers)
    mx = std::min(std::max(mx, std::ldexp(1.0, -980)), 1e200);
    int e = 0;
    (void)std::frexp(mx, &e);  // mx < 2^e
    const double unit = std::ldexp(1.0, e - 40);
    return MassUnit{1.5 * std::ldexp(unit, 52)};
}

int validate_and_build(const lbm_desc* s, lbm_domain* d) {
    const int nx = s->nx, ny = s->ny;
    if (nx < 3 || ny < 3 || !s->solid || !s->rho0) return LBM_EINVAL;
    if (!(s->tau > 0.5) || !std::isfinite(s->tau)) return LBM_EINVAL;
    if (s->rule < 0 || s->rule > 5 || s->fix < 0 || s->fix > 3) return LBM_EINVAL;
    if (s->eos < 0 || s->eos > 2 || s->collision < 0 || s->collision > 1) return LBM_EINVAL;
    if (s->storage < LBM_STORE_F64 || s->storage > LBM_STORE_F16NODE) return LBM_EINVAL;
    if (!(s->rho_ref >= 0.0) || !std::isfinite(s->rho_ref)) return LBM_EINVAL;
    if (s->open_x != 0 && s->open_x != 1) return LBM_EINVAL;
    if (s->open_x) {
        // single phase; the inlet density needs |U| < 1; no wall within
        // three columns of the inlet or the outlet, so that no wall rule
        // reads a slot the open rows write
        if (s->eos != LBM_EOS_NONE || !(std::fabs(s->inlet_u) < 1.0) || nx < 8)
            return LBM_EINVAL;
        for (int y = 0; y < ny; ++y)
            for (int x : {0, 1, 2, nx - 3, nx - 2, nx - 1})
                if (s->solid[(long long)y * nx + x]) return LBM_EINVAL;
    }
    if ((s->fix == LBM_FIX_B || s->fix == LBM_FIX_BAO) && s->rule != LBM_RULE_FH &&
        s->rule != LBM_RULE_MLS)
        return LBM_EINVAL;
    if (s->eos != LBM_EOS_NONE && (s->G == 0.0 || !std::isfinite(s->G))) return LBM_EINVAL;
    if (s->collision == LBM_COLL_MRT) {
        for (int i = 0; i < 9; ++i)
            if (!(s->mrt_s[i] > 0.0 && s->mrt_s[i] < 2.0)) return LBM_EINVAL;
        if (std::fabs(s->mrt_s[7] - 1.0 / s->tau) > 1e-12 ||
            std::fabs(s->mrt_s[8] - 1.0 / s->tau) > 1e-12)
            return LBM_EINVAL;
    }
    if (s->tile_w != 0 && s->tile_w != 64 && s->tile_w != 128 && s->tile_w != 256)
        return LBM_EINVAL;
    if (s->tile_h < 0) return LBM_EINVAL;
    if ((long long)nx * ny >= (1LL << 30)) return LBM_EINVAL;
    {
        // the nine population planes of one buffer are addressed with
        // 32-bit byte offsets
        const long long pitch = (nx + 63) / 64 * 64;
        const long long esz = storage_bytes(s->storage);
        const long long extra = s->storage == LBM_STORE_F16NODE ? 4 * (pitch * ny + 256) : 0;
        // (below the out-of-range lane offset of the kernels)
        if (9 * (pitch * ny + 256) * esz + extra >= (1LL << 32) - 256) return LBM_EINVAL;
    }
    const long long N = (long long)nx * ny;
    auto solid = [&](long long i) { return s->solid[i] != 0; };
    d->ph64 = make_phys<double>(s);
    d->ph32 = make_phys<float>(s);
    // wall densities
    for (long long i = 0; i < N; ++i) {
        if (!solid(i)) continue;
        const double rw = s->rho_wall ? s->rho_wall[i] : s->rho_wall_const;
        if (!std::isfinite(rw)) return LBM_EINVAL;
        if (s->eos != LBM_EOS_NONE) {
            if (!(rw > 0.0) || !std::isfinite(host_psi(s->eos, d->ph64, rw))) return LBM_EINVAL;
        }
    }
    // links
    const long long L = s->nlinks;
    if (L < 0 || (L > 0 && !s->links)) return LBM_EINVAL;
    std::vector<LinkRec> recs((size_t)L);
    bool singular = false;
    for (long long k = 0; k < L; ++k) {
        const lbm_link& l = s->links[k];
        if (l.x < 0 || l.x >= nx || l.y < 0 || l.y >= ny || l.dir < 1 || l.dir > 8 ||
            l.reserved != 0)
            return LBM_EINVAL;
        const long long b = (long long)l.y * nx + l.x;
        const long long xs = (long long)wrapi(l.y + cy(l.dir), ny) * nx + wrapi(l.x + cx(l.dir), nx);
        if (solid(b) || !solid(xs)) return LBM_EINVAL;
        if (!(l.q > 0.0 && l.q <= 1.0)) return LBM_EINVAL;
        if (!std::isfinite(l.uw[0]) || !std::isfinite(l.uw[1])) return LBM_EINVAL;
        const bool moving = l.uw[0] != 0.0 || l.uw[1] != 0.0;
        if (moving && !(s->rule == LBM_RULE_HALFWAY || s->rule == LBM_RULE_FH ||
                        s->rule == LBM_RULE_MLS))
            return LBM_EINVAL;
        if (moving && s->fix == LBM_FIX_BAO) return LBM_EINVAL;
        if (moving) d->block.moving = true;
        if (s->rule == LBM_RULE_FH && l.q < 0.5 && std::fabs(s->tau - 1.0) < 1e-12)
            singular = true;
        recs[k] = LinkRec{(int)b, l.dir, (int)k};
    }
    if (singular) return LBM_ESINGULAR;
    std::sort(recs.begin(), recs.end(), [](const LinkRec& a, const LinkRec& b) {
        return a.node != b.node ? a.node < b.node : a.dir < b.dir;
    });
    for (long long k = 1; k < L; ++k)
        if (recs[k].node == recs[k - 1].node && recs[k].dir == recs[k - 1].dir) return LBM_EINVAL;
    // Solid neighbours of fluid nodes, from the solid nodes of each column of
    // three rows, whose loops vectorise (a division and eight branches a
    // node, 67 ms at 2048 x 2048, was most of the creation; 4 ms now).
    long long count = 0, fluid = 0;
    std::vector<uint8_t> three((size_t)nx + 2);
    for (int y = 0; y < ny; ++y) {
        const uint8_t* const m = s->solid + (long long)y * nx;
        const uint8_t* const u = s->solid + (long long)(y == 0 ? ny - 1 : y - 1) * nx;
        const uint8_t* const b = s->solid + (long long)(y == ny - 1 ? 0 : y + 1) * nx;
        for (int x = 0; x < nx; ++x)
            three[(size_t)x + 1] = (uint8_t)((u[x] != 0) + (m[x] != 0) + (b[x] != 0));
        three[0] = three[(size_t)nx];
        three[(size_t)nx + 1] = three[1];
        const uint8_t* const t = three.data();
        int links = 0, nodes = 0;
        for (int x = 0; x < nx; ++x) {
            const int open = m[x] == 0;
            nodes += open;
            links += open * (t[x] + t[x + 1] + t[x + 2]);
        }
        fluid += nodes;
        count += links;
    }
    if (count != L) return LBM_EINVAL;
    // initial state
    for (long long i = 0; i < N; ++i) {
        if (solid(i)) continue;
        const double r = s->rho0[i];
        const double vx = s->ux0 ? s->ux0[i] : 0.0, vy = s->uy0 ? s->uy0[i] : 0.0;
        if (!(r > 0.0) || !std::isfinite(r) || !std::isfinite(vx) || !std::isfinite(vy))
            return LBM_EINVAL;
    }
    if (s->eos == LBM_EOS_CS)
        for (long long i = 0; i < N; i += nx)
            if (!cs_psi_finite(s->rho0 + i, s->solid + i, nx, d->ph64)) return LBM_EINVAL;
    d->fluid = fluid;
    d->mass = mass_unit_for(s, N);
    if (s->storage == LBM_STORE_F32DEV || s->storage == LBM_STORE_F16DEV) {
        double rref = s->rho_ref;
        if (rref == 0.0 && fluid > 0) {
            double sum = 0.0;
            for (long long i = 0; i < N; ++i)
                if (!solid(i)) sum += s->rho0[i];
            rref = sum / (double)fluid;
        }
        // rounded to FP32 so that the FP32 main kernel and the FP64
        // boundary kernel decode with the same reference
        d->ph64.rref = double(float(rref));
        d->ph32.rref = float(rref);
    }

    // ---- layout
    d->nx = nx;
    d->ny = ny;
    d->pitch = (nx + 63) / 64 * 64;
    d->plane = (long long)d->pitch * ny + 256;  // stagger the nine planes
    d->storage = s->storage;
    d->esize = (size_t)storage_bytes(s->storage);
    d->eos = s->eos;
    d->coll = s->collision;
    d->rule = s->rule;
    d->fix = s->fix;
    d->open_x = s->open_x;
    d->inlet_u = s->open_x ? s->inlet_u : 0.0;
    d->tile_w = s->tile_w ? s->tile_w : default_tile_w(nx, ny, d->storage);
    d->tile_h = s->tile_h ? s->tile_h : default_tile_h(nx, ny, d->storage);
    d->nstrips = (nx + strip_cols(d->tile_w) - 1) / strip_cols(d->tile_w);
    d->nsegs = seg_count(ny, d->tile_h);
    d->nblocks = d->nstrips * d->nsegs;
    // two steps per pass: FP32 or FP16 populations with one reference
    // density, periodic, any rule but Zhao-Yong (which needs the
    // pre-collision populations of the intermediate step) and the
    // quadratic interpolation (whose second fluid node lies outside the
    // pass's three-row rings); not for the instances of a batch, which run
    // the batched kernels
    d->fusable = (s->storage == LBM_STORE_F32 || s->storage == LBM_STORE_F32_ARITH32 ||
                  s->storage == LBM_STORE_F32DEV || s->storage == LBM_STORE_F16DEV) &&
                 !s->open_x && s->rule != LBM_RULE_ZHAO_YONG &&
                 s->rule != LBM_RULE_IBB_QUADRATIC && !d->arena;
    d->fused = 1;  // two steps per pass on request (lbm_set_steps_per_pass)
    d->tile_h2 = kTileH2;
    d->nstrips2 = (nx + kF2Cols - 1) / kF2Cols;
    d->nsegs2 = seg_count(ny, d->tile_h2);
    d->nblocks2 = d->nstrips2 * d->nsegs2;
    d->cap = s->history_capacity > 0 ? s->history_capacity : (1LL << 20);
    d->stream = static_cast<hipStream_t>(s->stream);
    const int P = d->pitch;
    auto pidx = [&](int x, int y) { return y * P + x; };

    // ---- boundary tables
    std::vector<uint8_t> flags((size_t)P * ny, 0);
    std::vector<int> side_idx((size_t)P * ny, -1);
    std::vector<int> node_link((size_t)P * ny, 0);  // first link slot + 1 of a boundary node
    for (long long i = 0; i < N; ++i)
        if (solid(i)) flags[pidx((int)(i % nx), (int)(i / nx))] |= FL_SOLID;
    d->save_f = s->rule == LBM_RULE_ZHAO_YONG;
    int nslots = 0;
    auto slot_of = [&](int x, int y) {
        const int p = pidx(x, y);
        if (side_idx[p] < 0) side_idx[p] = nslots++;
        flags[p] |= FL_SAVE_MOM;
        return side_idx[p];
    };
    // per-link records, grouped by node; a group never straddles a block
    std::vector<int> lnode, lmeta, lghost, lxf, lxff, lslotb, lslotf;
    std::vector<double> lc, luw;
    const double tau = s->tau;
    long long fallbacks = 0;
    int nb = 0;
    auto pad_to = [&](size_t n) {
        while (lnode.size() < n) {
            lnode.push_back(0);
            lmeta.push_back(LK_PAD << 4);
            lghost.push_back(0);
            lxf.push_back(-1);
            lxff.push_back(-1);
            lslotb.push_back(0);
            lslotf.push_back(-1);
            for (int j = 0; j < 8; ++j) lc.push_back(0.0);
            luw.push_back(0.0);
            luw.push_back(0.0);
        }
    };
    for (long long k0 = 0; k0 < L;) {
        long long k1 = k0;
        while (k1 < L && recs[k1].node == recs[k0].node) ++k1;
        const int len = (int)(k1 - k0);
        const size_t used = lnode.size() % 256;
        if (used + len > 256) pad_to(lnode.size() + (256 - used));
        const int x = recs[k0].node % nx, y = recs[k0].node / nx;
        const int sb = slot_of(x, y);
        // the two-step pass keeps (first link slot + 1) << 8 | flags in an int
        if (lnode.size() + 1 >= (size_t(1) << 23)) d->fusable = false;
        node_link[pidx(x, y)] = (int)lnode.size() + 1;
        d->bnd_x.push_back(x);
        d->bnd_y.push_back(y);
        if (d->save_f) flags[pidx(x, y)] |= FL_SAVE_F;
        ++nb;
        for (long long k = k0; k < k1; ++k) {
            const LinkRec& r = recs[k];
            const int a = r.dir;
            const lbm_link& l = s->links[r.src];
            const int xf = wrapi(x - cx(a), nx), yf = wrapi(y - cy(a), ny);
            const int xff = wrapi(x - 2 * cx(a), nx), yff = wrapi(y - 2 * cy(a), ny);
            const bool f_ok = !solid((long long)yf * nx + xf);
            const bool ff_ok = f_ok && !solid((long long)yff * nx + xff);
            const double q = l.q;
            double c[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            int kind = LK_HALFWAY, sf = -1;
            switch (s->rule) {
            case LBM_RULE_HALFWAY:
                kind = LK_HALFWAY;
                break;
            case LBM_RULE_FH:
            case LBM_RULE_MLS:
                if (q < 0.5) {
                    if (s->rule == LBM_RULE_FH) {
                        kind = LK_CHI_UB;
                        c[3] = (2.0 * q - 1.0) / (tau - 1.0);  // Eq. (9)
                    } else {
                        c[3] = (2.0 * q - 1.0) / (tau - 2.0);  // Eq. (11)
                        if (f_ok) {
                            kind = LK_CHI_UF;
                            sf = slot_of(xf, yf);
                        } else {
                            kind = LK_CHI_UB;
                            ++fallbacks;
                        }
                    }
                } else {
                    kind = LK_CHI_EXT;  // Eq. (10)
                    c[3] = (2.0 * q - 1.0) / tau;
                    c[4] = (q - 1.0) / q;
                    c[5] = l.uw[0] / q;
                    c[6] = l.uw[1] / q;
                }
                break;
            case LBM_RULE_IBB_LINEAR:
            case LBM_RULE_IBB_QUADRATIC: {
                const bool quad = s->rule == LBM_RULE_IBB_QUADRATIC;
                if (quad && q < 0.5 && ff_ok) {  // Eq. (13)
                    kind = LK_QUAD_F;
                    c[0] = q * (1.0 + 2.0 * q);
                    c[1] = 1.0 - 4.0 * q * q;
                    c[2] = q * (1.0 - 2.0 * q);
                } else if (quad && q >= 0.5 && f_ok) {
                    kind = LK_QUAD_B;
                    c[0] = 1.0 / (q * (2.0 * q + 1.0));
                    c[1] = (2.0 * q - 1.0) / q;
                    c[2] = (2.0 * q - 1.0) / (2.0 * q + 1.0);
                } else if (q < 0.5 && f_ok) {  // Eq. (12)
                    if (quad) ++fallbacks;
                    kind = LK_LIN_F;
                    c[0] = 2.0 * q;
                    c[1] = 1.0 - 2.0 * q;
                } else {
                    if (quad || q < 0.5) ++fallbacks;
                    kind = LK_LIN_B;
                    c[0] = 1.0 / (2.0 * q);
                    c[1] = (2.0 * q - 1.0) / (2.0 * q);
                }
                break;
            }
            case LBM_RULE_ZHAO_YONG:  // Eq. (14)
                kind = LK_ZY;
                c[0] = 2.0 * q / (1.0 + 2.0 * q);
                c[1] = 1.0 / (1.0 + 2.0 * q);
                break;
            }
            lnode.push_back(pidx(x, y));
            lmeta.push_back(a | (kind << 4) | (len << 8) | ((int)(k - k0) << 12));
            lghost.push_back(pidx(wrapi(x + cx(a), nx), wrapi(y + cy(a), ny)));
            lxf.push_back(f_ok ? pidx(xf, yf) : -1);
            lxff.push_back(ff_ok ? pidx(xff, yff) : -1);
            lslotb.push_back(sb);
            lslotf.push_back(sf);
            for (int j = 0; j < 8; ++j) lc.push_back(c[j]);
            luw.push_back(l.uw[0]);
            luw.push_back(l.uw[1]);
        }
        k0 = k1;
    }
    d->nb = nb;
    d->nl = (int)L;
    d->nslot_links = (int)lnode.size();
    d->nslots = nslots;
    d->fallbacks = fallbacks;

    std::vector<int> lref;
    std::vector<float> rplane;  // FP16 per-node form: initial density plane
    if (s->storage == LBM_STORE_F16NODE) {
        // Each ghost (a solid node receiving incoming populations) is
        // encoded against the density of one boundary node next to it: the
        // first in table order, whose link records it.
        std::vector<int> owner((size_t)P * ny, -1);
        lref.assign(lnode.size(), 0);
        for (size_t k = 0; k < lnode.size(); ++k) {
            if (((lmeta[k] >> 4) & 15) == LK_PAD) continue;
            const int g = lghost[k];
            if (owner[g] < 0) {
                owner[g] = (int)k;
                lmeta[k] |= 1 << 16;
            }
            lref[k] = lslotb[owner[g]];
        }
        rplane.assign((size_t)d->plane, 0.0f);
        for (long long i = 0; i < N; ++i)
            if (!solid(i)) rplane[pidx((int)(i % nx), (int)(i / nx))] = float(s->rho0[i]);
        for (size_t k = 0; k < lnode.size(); ++k)
            if ((lmeta[k] >> 16) & 1) {
                const int n = lnode[k];
                rplane[lghost[k]] = float(s->rho0[(long long)(n / P) * nx + (n % P)]);
            }
    }

    // ---- device memory
    int rc;
    d->fbytes = (size_t)9 * d->plane * d->esize +
                (s->storage == LBM_STORE_F16NODE ? (size_t)4 * d->plane : 0);
    const size_t fbytes = d->fbytes;
    if ((rc = dev_alloc(d, &d->f[0], fbytes))) return rc;
    if ((rc = dev_alloc(d, &d->f[1], fbytes))) return rc;
    if (hipMemsetAsync(d->f[0], 0, fbytes, d->stream) != hipSuccess) return LBM_EDEVICE;
    if (hipMemsetAsync(d->f[1], 0, fbytes, d->stream) != hipSuccess) return LBM_EDEVICE;
    if ((rc = upload(d, &d->flags, flags))) return rc;
    if ((rc = upload(d, &d->side_idx, side_idx))) return rc;
    if (d->esize == 2 && (rc = dev_alloc(d, (void**)&d->psiw, (size_t)P * ny * 4))) return rc;
    if ((rc = dev_alloc(d, (void**)&d->side_mom[0], (size_t)3 * std::max(nslots, 1) * 8)))
        return rc;
    d->side_mom[1] = d->side_mom[0];  // (see place_blocks)
    if ((rc = dev_alloc(d, (void**)&d->side_f,
                        (size_t)9 * (d->save_f ? std::max(nslots, 1) : 1) * 8)))
        return rc;
    // partials for any tile shape down to 64 x 8 (the batched form retunes)
    d->partial_cap = std::max(d->nblocks, ((nx + strip_cols(64) - 1) / strip_cols(64)) * ((ny + 7) / 8));
    if (d->fusable)  // and for two-step tiles down to kMinTileH2 rows
        d->partial_cap = std::max(d->partial_cap,
                                  d->nstrips2 * ((ny + kMinTileH2 - 1) / kMinTileH2));
    const size_t pbytes = (size_t)(d->fusable ? 2 : 1) * d->partial_cap * sizeof(MassTile);
    if (d->arena) {
        // In an arena (batched and served instances) the read-out buffer is
        // part of the footprint, so that reading a finished instance never
        // fails.  The partials share its place: a step's are summed before its
        // fields can be read.
        if ((rc = dev_alloc(d, (void**)&d->mom_out, std::max<size_t>((size_t)3 * N * 8, pbytes))))
            return rc;
        d->partial = reinterpret_cast<MassTile*>(d->mom_out);
    } else if ((rc = dev_alloc(d, (void**)&d->partial, pbytes))) {
        return rc;
    }
    if (d->fusable) {
        if ((rc = upload(d, &d->node_link, node_link))) return rc;
        if ((rc = dev_alloc(d, (void**)&d->tile_order, (size_t)d->partial_cap * 4))) return rc;
        if ((rc = order_tiles(d))) return rc;
        // the replay of the intermediate step (moments and wall force after
        // a two-step pass), held from the start so that reading them never
        // allocates
        if ((rc = dev_alloc(d, &d->frep, fbytes))) return rc;
        if ((rc = dev_alloc(d, (void**)&d->side_mom_rep, (size_t)3 * std::max(nslots, 1) * 8)))
            return rc;
    }
    if ((rc = dev_alloc(d, (void**)&d->hist, (size_t)d->cap * 8))) return rc;
    if ((rc = dev_alloc(d, (void**)&d->unstable, 8))) return rc;
    if ((rc = dev_alloc(d, (void**)&d->clock, 8))) return rc;
    if ((rc = upload(d, &d->lnode, lnode))) return rc;
    if ((rc = upload(d, &d->lmeta, lmeta))) return rc;
    if ((rc = upload(d, &d->lghost, lghost))) return rc;
    if ((rc = upload(d, &d->lxf, lxf))) return rc;
    if ((rc = upload(d, &d->lxff, lxff))) return rc;
    if ((rc = upload(d, &d->lslotb, lslotb))) return rc;
    if ((rc = upload(d, &d->lslotf, lslotf))) return rc;
    if ((rc = upload(d, &d->lc, lc))) return rc;
    if ((rc = upload(d, &d->luw, luw))) return rc;
    if (!lref.empty() && (rc = upload(d, &d->lref, lref))) return rc;
    LinkTables lt{std::move(lnode), std::move(lmeta), std::move(lslotb), std::move(lslotf),
                  std::move(lc)};
    BlockTables blocks;
    if ((rc = plan_blocks(d, lt, blocks))) return rc;
    if (d->arena && domain_blockable(d)) d->links = lt;  // (see domain_make_blocks)
    if ((rc = dev_alloc(d, (void**)&d->force,
                        (size_t)2 * std::max(link_blocks(d), 1) * 8)))
        return rc;

    if ((rc = dev_alloc(d, (void**)&d->negrest, 8))) return rc;
    if (hipMemsetAsync(d->negrest, 0, 8, d->stream) != hipSuccess) return LBM_EDEVICE;
    if ((rc = dev_alloc(d, (void**)&d->degen, 8))) return rc;
    if (hipMemsetAsync(d->degen, 0, 8, d->stream) != hipSuccess) return LBM_EDEVICE;

    // no unstable step yet; the first recorded mass is that of step 0
    static const long long minus1 = -1;
    if (hipMemcpyAsync(d->unstable, &minus1, 8, hipMemcpyHostToDevice, d->stream) != hipSuccess ||
        hipMemcpyAsync(d->clock, &minus1, 8, hipMemcpyHostToDevice, d->stream) != hipSuccess)
        return LBM_EDEVICE;
    if (hipMemsetAsync(d->hist, 0, (size_t)d->cap * 8, d->stream) != hipSuccess)
        return LBM_EDEVICE;

    // ---- initial state: psi at walls, f(0) scattered, f*(0) by one main pass
    // (from the caller's arrays, which the wait at the end outlasts)
    std::vector<double> rw;
    if (!s->rho_wall) rw.assign((size_t)N, s->rho_wall_const);
    double* ini[4] = {nullptr, nullptr, nullptr, nullptr};
    const double* const src[4] = {s->rho_wall ? s->rho_wall : rw.data(), s->rho0, s->ux0, s->uy0};
    for (int k = 0; k < 4; ++k) {
        const size_t bytes = (size_t)N * 8;
        if ((rc = dev_alloc(d, (void**)&ini[k], bytes))) return rc;
        if ((src[k] ? hipMemcpyAsync(ini[k], src[k], bytes, hipMemcpyHostToDevice, d->stream)
                    : hipMemsetAsync(ini[k], 0, bytes, d->stream)) != hipSuccess)
            return LBM_EDEVICE;
    }
    double *drw = ini[0], *dr0 = ini[1], *du0 = ini[2], *dv0 = ini[3];
    if (d->storage == LBM_STORE_F64) launch_init_f64(ctx(d), drw, dr0, du0, dv0, d->f[1], d->f[0]);
    else {
        Ctx c = ctx(d);
        if (!rplane.empty()) {
            // both buffers start with the initial density plane
            const size_t off = (size_t)9 * d->plane * d->esize;
            for (int k = 0; k < 2; ++k)
                if (hipMemcpyAsync(static_cast<char*>(d->f[k]) + off, rplane.data(),
                                   rplane.size() * 4, hipMemcpyHostToDevice, d->stream) != hipSuccess)
                    return LBM_EDEVICE;
            c.ref = reinterpret_cast<const float*>(static_cast<char*>(d->f[1]) + off);
        }
        launch_init_f32(c, drw, dr0, du0, dv0, d->f[1], d->f[0]);
    }
    d->cur = 1;
    launch_main(d, d->f[1], d->f[0], false);
    // the replay buffer starts as a copy, so that its solid nodes hold
    // psi of the wall density in their rest slots as the state buffers do
    if (d->frep && hipMemcpyAsync(d->frep, d->f[0], d->fbytes, hipMemcpyDeviceToDevice,
                                  d->stream) != hipSuccess)
        return LBM_EDEVICE;
    d->cur = 0;
    d->t = 0;
    d->pending = true;
    d->pending_steps = 1;
    d->pending_block = false;
    d->pending_t = 0;
    reduce_pending(d);
    if (hipGetLastError() != hipSuccess) return LBM_EDEVICE;
    if (hipStreamSynchronize(d->stream) != hipSuccess) return LBM_EDEVICE;
    // the initial fields are no longer needed
    for (double* p : {drw, dr0, du0, dv0}) dev_free(d, p, (size_t)N * 8);
    if ((rc = place_blocks(d, blocks))) return rc;
    return check_unstable(d);
}

}  // namespace

namespace lbm {

int domain_create(const lbm_desc* desc, Arena* arena, lbm_domain** out) {
    if (!desc || !out) return LBM_EINVAL;
    lbm_domain* d = new (std::nothrow) lbm_domain();
    if (!d) return LBM_ENOMEM;
    d->arena = arena;
    int rc = validate_and_build(desc, d);
    // (the descriptor is checked before anything touches the device)
    if (rc == LBM_OK && hipGetDevice(&d->device) != hipSuccess) rc = LBM_EDEVICE;
    if (rc != LBM_OK) {
        free_domain(d);
        return rc;
    }
    *out = d;
    return LBM_OK;
}

void domain_free(lbm_domain* d) { free_domain(d); }

int domain_set_tiles(lbm_domain* d, int tile_w, int tile_h) {
    if (tile_w != 64 && tile_w != 128 && tile_w != 256) return LBM_EINVAL;
    if (tile_h < 1) return LBM_EINVAL;
    const int sc = strip_cols(tile_w);
    const int ns = (d->nx + sc - 1) / sc, ng = seg_count(d->ny, tile_h);
    if ((long long)ns * ng > d->partial_cap) return LBM_EINVAL;
    drop_graphs(d);
    d->tile_w = tile_w;
    d->tile_h = tile_h;
    d->nstrips = ns;
    d->nsegs = ng;
    d->nblocks = ns * ng;
    return LBM_OK;
}

bool being_captured(hipStream_t stream) {
    hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &s) == hipSuccess) return s != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

bool domain_make_blocks(lbm_domain* d, int steps, Arena* pool) {
    domain_drop_blocks(d, pool);
    BlockTables b;
    if (!domain_blockable(d) || !try_block_tables(d, steps, kBlockThreads, d->links, b))
        return false;
    BlockPlan& p = d->block;
    const size_t nt = (size_t)b.nstrips * b.nsegs;
    p.tiles = static_cast<BlockTile*>(pool->alloc(nt * sizeof(BlockTile)));
    p.links = static_cast<BlockLink*>(pool->alloc(b.links.size() * sizeof(BlockLink)));
    p.nodes = static_cast<BlockNode*>(pool->alloc(b.nodes.size() * sizeof(BlockNode)));
    p.partial[0] = static_cast<MassTile*>(pool->alloc((size_t)steps * nt * sizeof(MassTile)));
    bool ok = p.tiles && p.links && p.nodes && p.partial[0];
    auto put = [&](void* dst, const void* src, size_t n) {
        if (ok && n)
            ok = hipMemcpyAsync(dst, src, n, hipMemcpyHostToDevice, d->stream) == hipSuccess;
    };
    put(p.tiles, b.tiles.data(), nt * sizeof(BlockTile));
    put(p.links, b.links.data(), b.links.size() * sizeof(BlockLink));
    put(p.nodes, b.nodes.data(), b.nodes.size() * sizeof(BlockNode));
    // (the tables end with this call)
    if (hipStreamSynchronize(d->stream) != hipSuccess) ok = false;
    if (!ok) {
        domain_drop_blocks(d, pool);
        return false;
    }
    p.set = 0;
    block_plan(d, b);
    return true;
}

void domain_drop_blocks(lbm_domain* d, Arena* pool) {
    BlockPlan& p = d->block;
    for (void* q : {(void*)p.tiles, (void*)p.links, (void*)p.nodes, (void*)p.partial[0]})
        pool->release(q);
    const bool moving = p.moving;
    p = BlockPlan{};
    p.moving = moving;
}

Ctx domain_ctx(lbm_domain* d) { return ctx(d); }

const void* moments_source(lbm_domain* d) {
    if (!d->last_fused) return d->f[d->cur ^ 1];
    if (!d->replay_valid) {
        // step t - 1 from f*(t - 2), whose ghosts its boundary pass wrote,
        // into frep; its moments go to the replay's own side slots
        Ctx c = ctx(d);
        c.side_mom = d->side_mom_rep;
        launch_main_f32(c, d->f[d->cur ^ 1], d->frep, false);
        // the ghosts of step t, and the force on the walls during it
        BndArgs b = bnd_args(d);
        b.side_mom = d->side_mom_rep;
        b.do_reduce = 0;
        b.negrest = nullptr;
        b.degen = nullptr;
        launch_boundary_f32(c, d->frep, b, b.nlink_blocks + 1);
        d->force_valid = true;
        d->replay_valid = true;
    }
    return d->frep;
}

// ------------------------------------------------------------------ arena
Arena::~Arena() {
    if (base_) (void)hipFree(base_);
}

int Arena::init(size_t bytes) {
    bytes = (bytes + 255) & ~size_t(255);
    if (bytes == 0 || hipMalloc(reinterpret_cast<void**>(&base_), bytes) != hipSuccess) {
        base_ = nullptr;
        return LBM_ENOMEM;
    }
    cap_ = bytes;
    free_[0] = bytes;
    return LBM_OK;
}

void* Arena::alloc(size_t bytes) {
    bytes = (std::max<size_t>(bytes, 1) + 255) & ~size_t(255);
    for (auto it = free_.begin(); it != free_.end(); ++it) {
        if (it->second < bytes) continue;
        const size_t off = it->first, rest = it->second - bytes;
        free_.erase(it);
        if (rest) free_[off + bytes] = rest;
        live_[off] = bytes;
        used_ += bytes;
        return base_ + off;
    }
    return nullptr;
}

void Arena::release(void* p) {
    if (!p) return;
    const size_t off = static_cast<size_t>(static_cast<char*>(p) - base_);
    auto lv = live_.find(off);
    if (lv == live_.end()) return;
    size_t start = off, len = lv->second;
    live_.erase(lv);
    used_ -= len;
    auto nx = free_.lower_bound(off);
    if (nx != free_.end() && nx->first == off + len) {  // merge with the next block
        len += nx->second;
        nx = free_.erase(nx);
    }
    if (nx != free_.begin()) {  // and with the previous one
        auto pv = std::prev(nx);
        if (pv->first + pv->second == start) {
            start = pv->first;
            len += pv->second;
            free_.erase(pv);
        }
    }
    free_[start] = len;
}

size_t Arena::largest_free() const {
    size_t m = 0;
    for (const auto& kv : free_) m = std::max(m, kv.second);
    return m;
}

}  // namespace lbm

namespace {

// Whether a kernel of the domain can store to a caller's array of n doubles:
// none, or memory of the domain's own GPU, at an address of doubles, whose
// allocation goes on for n of them.  (Other memory -- of another GPU, of the
// host -- is reached by copies, which also refuse an array that ends too soon.)
bool stores_reach(const lbm_domain* d, const void* p, size_t n) {
    if (!p) return true;
    hipPointerAttribute_t at{};
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipPointerGetAttributes(&at, p) != hipSuccess || at.type != hipMemoryTypeDevice ||
        at.device != d->device ||
        hipMemGetAddressRange(&base, &size, const_cast<void*>(p)) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    const uintptr_t at0 = reinterpret_cast<uintptr_t>(p) - reinterpret_cast<uintptr_t>(base);
    return reinterpret_cast<uintptr_t>(p) % 8 == 0 && at0 <= size && n * 8 <= size - at0;
}

// Whether two arrays of n doubles share no byte (where they do, copies one
// after another decide what they hold).
bool apart(const double* p, const double* q, size_t n) {
    if (!p || !q) return true;
    const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(q);
    return (a < b ? b - a : a - b) >= n * 8;
}

}  // namespace

extern "C" {

int lbm_create_domain(const lbm_desc* desc, lbm_domain** out) {
    return domain_create(desc, nullptr, out);
}

int lbm_step_async(lbm_domain* d, int64_t n) {
    if (!d || n < 0) return LBM_EINVAL;
    if (n == 0) return LBM_OK;
    return run_steps(d, n);
}

int lbm_sync(lbm_domain* d) {
    if (!d) return LBM_EINVAL;
    return check_unstable(d);
}

int lbm_step(lbm_domain* d, int64_t n) {
    int rc = lbm_step_async(d, n);
    if (rc != LBM_OK) return rc;
    return lbm_sync(d);
}

int lbm_moments_device(lbm_domain* d, double* rho, double* ux, double* uy) {
    if (!d) return LBM_EINVAL;
    const size_t nn = (size_t)d->nx * d->ny;
    // Into the caller's arrays by the kernel itself where it can store there;
    // through the domain's planes and three copies otherwise (droplet 2048^2
    // in FP32: 54 us for the kernel, 45 for the copies).
    if (stores_reach(d, rho, nn) && stores_reach(d, ux, nn) && stores_reach(d, uy, nn) &&
        apart(rho, ux, nn) && apart(rho, uy, nn) && apart(ux, uy, nn)) {
        const void* src = moments_source(d);
        Ctx c = ctx(d);
        c.mom_out[0] = rho;
        c.mom_out[1] = ux;
        c.mom_out[2] = uy;
        if (d->storage == LBM_STORE_F64) launch_main_f64(c, src, nullptr, true);
        else launch_main_f32(c, src, nullptr, true);
        return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
    }
    if (!d->mom_out) {
        int rc = dev_alloc(d, (void**)&d->mom_out, 3 * nn * 8);
        if (rc) return rc;
    }
    launch_main(d, moments_source(d), nullptr, true);
    double* const outs[3] = {rho, ux, uy};
    for (int k = 0; k < 3; ++k)
        if (outs[k] && hipMemcpyAsync(outs[k], d->mom_out + k * nn, nn * 8,
                                      hipMemcpyDeviceToDevice, d->stream) != hipSuccess) {
            (void)hipGetLastError();  // (a refused array is no error of the next call)
            return LBM_EDEVICE;
        }
    return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

int lbm_moments(lbm_domain* d, double* rho, double* ux, double* uy) {
    if (!d) return LBM_EINVAL;
    const size_t nn = (size_t)d->nx * d->ny;
    if (!d->mom_out) {
        int rc = dev_alloc(d, (void**)&d->mom_out, 3 * nn * 8);
        if (rc) return rc;
    }
    launch_main(d, moments_source(d), nullptr, true);
    if (hipGetLastError() != hipSuccess) return LBM_EDEVICE;
    double* outs[3] = {rho, ux, uy};
    for (int k = 0; k < 3; ++k)
        if (outs[k] && hipMemcpyAsync(outs[k], d->mom_out + k * nn, nn * 8,
                                      hipMemcpyDeviceToHost, d->stream) != hipSuccess)
            return LBM_EDEVICE;
    return hipStreamSynchronize(d->stream) == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

int lbm_total_mass(lbm_domain* d, double* out) {
    if (!d || !out) return LBM_EINVAL;
    double m = 0;
    if (hipMemcpyAsync(&m, d->hist + d->t % d->cap, 8, hipMemcpyDeviceToHost, d->stream) !=
            hipSuccess ||
        hipStreamSynchronize(d->stream) != hipSuccess)
        return LBM_EDEVICE;
    *out = m;
    return LBM_OK;
}

int lbm_wall_force(lbm_domain* d, double out[2]) {
    if (!d || !out) return LBM_EINVAL;
    out[0] = out[1] = 0.0;
    if (d->last_fused) (void)moments_source(d);  // the replay forms the force
    if (!d->force_valid) return LBM_OK;
    const int n = link_blocks(d);
    std::vector<double> part((size_t)2 * std::max(n, 1), 0.0);
    if (n > 0 && hipMemcpyAsync(part.data(), d->force, (size_t)2 * n * 8,
                                hipMemcpyDeviceToHost, d->stream) != hipSuccess)
        return LBM_EDEVICE;
    if (hipStreamSynchronize(d->stream) != hipSuccess) return LBM_EDEVICE;
    // block partials in block order
    for (int k = 0; k < n; ++k) {
        out[0] += part[2 * k];
        out[1] += part[2 * k + 1];
    }
    return LBM_OK;
}

int lbm_time(lbm_domain* d, int64_t* t) {
    if (!d || !t) return LBM_EINVAL;
    *t = d->t;
    return LBM_OK;
}

int lbm_mass_history(lbm_domain* d, double* out, int64_t cap, int64_t* n_written) {
    if (!d || !out || cap < 0 || !n_written) return LBM_EINVAL;
    const long long avail = std::min<long long>(d->t + 1, d->cap);
    const long long n = std::min<long long>(avail, cap);
    std::vector<double> ring((size_t)d->cap);
    if (hipMemcpyAsync(ring.data(), d->hist, (size_t)d->cap * 8, hipMemcpyDeviceToHost,
                       d->stream) != hipSuccess ||
        hipStreamSynchronize(d->stream) != hipSuccess)
        return LBM_EDEVICE;
    const long long first = d->t + 1 - n;
    for (long long i = 0; i < n; ++i) out[i] = ring[(size_t)((first + i) % d->cap)];
    *n_written = n;
    return LBM_OK;
}

int lbm_unstable_step(lbm_domain* d, int64_t* step) {
    if (!d || !step) return LBM_EINVAL;
    long long u = -1;
    if (hipMemcpyAsync(&u, d->unstable, 8, hipMemcpyDeviceToHost, d->stream) != hipSuccess ||
        hipStreamSynchronize(d->stream) != hipSuccess)
        return LBM_EDEVICE;
    *step = u;
    return LBM_OK;
}

static size_t state_bytes(const lbm_domain* d) {
    return 8 * 4 + 2 * d->fbytes + (size_t)3 * std::max(d->nslots, 1) * 8 +
           (size_t)9 * (d->save_f ? std::max(d->nslots, 1) : 1) * 8 + (size_t)d->cap * 8 + 8;
}

int lbm_get_state(lbm_domain* d, void* buf, size_t* bytes) {
    if (!d || !bytes) return LBM_EINVAL;
    const size_t need = state_bytes(d);
    if (!buf) {
        *bytes = need;
        return LBM_OK;
    }
    if (*bytes < need) return LBM_EINVAL;
    if (hipStreamSynchronize(d->stream) != hipSuccess) return LBM_EDEVICE;
    char* p = static_cast<char*>(buf);
    // word 3: the storage form, and whether the last pass made two steps
    const uint64_t hdr[4] = {kStateMagic, (uint64_t)d->t, ((uint64_t)d->nx << 32 | (uint64_t)d->ny),
                             (uint64_t)d->storage | ((uint64_t)(d->last_fused ? 1 : 0) << 32)};
    std::memcpy(p, hdr, sizeof(hdr));
    p += sizeof(hdr);
    const size_t fb = d->fbytes;
    const size_t sm = (size_t)3 * std::max(d->nslots, 1) * 8;
    const size_t sf = (size_t)9 * (d->save_f ? std::max(d->nslots, 1) : 1) * 8;
    if (hipMemcpy(p, d->f[d->cur], fb, hipMemcpyDeviceToHost) != hipSuccess) return LBM_EDEVICE;
    p += fb;
    if (hipMemcpy(p, d->f[d->cur ^ 1], fb, hipMemcpyDeviceToHost) != hipSuccess) return LBM_EDEVICE;
    p += fb;
    if (hipMemcpy(p, d->side_mom[d->cur], sm, hipMemcpyDeviceToHost) != hipSuccess)
        return LBM_EDEVICE;
    p += sm;
    if (hipMemcpy(p, d->side_f, sf, hipMemcpyDeviceToHost) != hipSuccess) return LBM_EDEVICE;
    p += sf;
    if (hipMemcpy(p, d->hist, (size_t)d->cap * 8, hipMemcpyDeviceToHost) != hipSuccess)
        return LBM_EDEVICE;
    p += (size_t)d->cap * 8;
    if (hipMemcpy(p, d->unstable, 8, hipMemcpyDeviceToHost) != hipSuccess) return LBM_EDEVICE;
    *bytes = need;
    return LBM_OK;
}

int lbm_set_state(lbm_domain* d, const void* buf, size_t bytes) {
    if (!d || !buf || bytes != state_bytes(d)) return LBM_EINVAL;
    const char* p = static_cast<const char*>(buf);
    uint64_t hdr[4];
    std::memcpy(hdr, p, sizeof(hdr));
    const bool fused_state = (hdr[3] >> 32) == 1;
    if (hdr[0] != kStateMagic || hdr[2] != ((uint64_t)d->nx << 32 | (uint64_t)d->ny) ||
        (hdr[3] & 0xffffffffULL) != (uint64_t)d->storage || (hdr[3] >> 32) > 1 ||
        (fused_state && !d->fusable))
        return LBM_EINVAL;
    p += sizeof(hdr);
    if (hipStreamSynchronize(d->stream) != hipSuccess) return LBM_EDEVICE;
    const size_t fb = d->fbytes;
    const size_t sm = (size_t)3 * std::max(d->nslots, 1) * 8;
    const size_t sf = (size_t)9 * (d->save_f ? std::max(d->nslots, 1) : 1) * 8;
    d->cur = 0;
    if (hipMemcpy(d->f[0], p, fb, hipMemcpyHostToDevice) != hipSuccess) return LBM_EDEVICE;
    p += fb;
    if (hipMemcpy(d->f[1], p, fb, hipMemcpyHostToDevice) != hipSuccess) return LBM_EDEVICE;
    p += fb;
    if (hipMemcpy(d->side_mom[0], p, sm, hipMemcpyHostToDevice) != hipSuccess) return LBM_EDEVICE;
    p += sm;
    if (hipMemcpy(d->side_f, p, sf, hipMemcpyHostToDevice) != hipSuccess) return LBM_EDEVICE;
    p += sf;
    if (hipMemcpy(d->hist, p, (size_t)d->cap * 8, hipMemcpyHostToDevice) != hipSuccess)
        return LBM_EDEVICE;
    p += (size_t)d->cap * 8;
    if (hipMemcpy(d->unstable, p, 8, hipMemcpyHostToDevice) != hipSuccess) return LBM_EDEVICE;
    if (hipMemset(d->negrest, 0, 8) != hipSuccess || hipMemset(d->degen, 0, 8) != hipSuccess)
        return LBM_EDEVICE;
    const long long tclock = (long long)hdr[1];
    if (hipMemcpy(d->clock, &tclock, 8, hipMemcpyHostToDevice) != hipSuccess) return LBM_EDEVICE;
    d->t = (long long)hdr[1];
    d->last_fused = fused_state;
    d->replay_valid = false;
    d->pending = false;
    d->pending_t = d->t;
    d->force_valid = false;
    return LBM_OK;
}

int lbm_set_profiling(lbm_domain* d, int every) {
    if (!d || every < 0) return LBM_EINVAL;
    int rc = harvest(d);
    if (rc) return rc;
    if (every) {
        rc = ensure_events(d);
        if (rc) return rc;
    }
    d->prof = every;
    d->main_ms = d->bnd_ms = 0;
    d->main_n = d->bnd_n = 0;
    return LBM_OK;
}

int lbm_kernel_times(lbm_domain* d, double* main_ms, int64_t* main_count, double* boundary_ms,
                     int64_t* boundary_count) {
    if (!d) return LBM_EINVAL;
    int rc = harvest(d);
    if (rc) return rc;
    if (main_ms) *main_ms = d->main_ms;
    if (main_count) *main_count = d->main_n;
    if (boundary_ms) *boundary_ms = d->bnd_ms;
    if (boundary_count) *boundary_count = d->bnd_n;
    return LBM_OK;
}

int lbm_negative_rest(lbm_domain* d, int64_t* count) {
    if (!d || !count) return LBM_EINVAL;
    unsigned long long n = 0;
    if (hipMemcpyAsync(&n, d->negrest, 8, hipMemcpyDeviceToHost, d->stream) != hipSuccess ||
        hipStreamSynchronize(d->stream) != hipSuccess)
        return LBM_EDEVICE;
    *count = (int64_t)n;
    return LBM_OK;
}

int lbm_set_steps_per_pass(lbm_domain* d, int32_t steps, int32_t tile_h) {
    if (!d || (steps != 1 && steps != 2) || tile_h < 0) return LBM_EINVAL;
    if (steps == 2 && !d->fusable) return LBM_EINVAL;
    const int th = tile_h ? tile_h : kTileH2;
    if (steps == 2) {
        if (th < kMinTileH2) return LBM_EINVAL;
        const int ng = seg_count(d->ny, th);
        if ((long long)d->nstrips2 * ng > d->partial_cap) return LBM_EINVAL;
        d->tile_h2_asked = tile_h > 0;
        d->tile_h2 = th;
        d->nsegs2 = ng;
        d->nblocks2 = d->nstrips2 * ng;
        const int rc = order_tiles(d);
        if (rc) return rc;
    }
    drop_graphs(d);
    d->fused = steps;
    return LBM_OK;
}

int lbm_get_steps_per_pass(lbm_domain* d, int32_t* steps, int32_t* tile_h) {
    if (!d) return LBM_EINVAL;
    if (steps) *steps = d->fused;
    if (tile_h) *tile_h = d->fused == 2 ? d->tile_h2 : d->tile_h;
    return LBM_OK;
}

int lbm_tune_steps_per_pass(lbm_domain* d, int64_t steps_per_trial, int32_t out[3]) {
    if (!d || !out || steps_per_trial < 2) return LBM_EINVAL;
    struct Cand {
        int steps, tile_h;
    };
    std::vector<Cand> cands{{1, 0}};
    if (d->fusable)
        for (int th : {4, 6, 8, 12, 16, 24})
            if ((long long)d->nstrips2 * ((d->ny + th - 1) / th) <= d->partial_cap)
                cands.push_back({2, th});
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
        if (e0) (void)hipEventDestroy(e0);
        return LBM_EDEVICE;
    }
    // whole runs are timed, so the steps replay their graphs as lbm_step does
    const int prof = d->prof, steps0 = d->fused, tile0 = d->tile_h2;
    const bool asked0 = d->tile_h2_asked;
    d->prof = 0;
    int rc = LBM_OK;
    float best = 0.0f;
    Cand pick = cands[0];
    for (const Cand& c : cands) {
        if ((rc = lbm_set_steps_per_pass(d, c.steps, c.tile_h))) break;
        if ((rc = run_steps(d, steps_per_trial))) break;  // also captures the graphs
        float ms = 0.0f;
        if (hipEventRecord(e0, d->stream) != hipSuccess ||
            (rc = run_steps(d, steps_per_trial)) != LBM_OK ||
            hipEventRecord(e1, d->stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
            hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
            if (!rc) rc = LBM_EDEVICE;
            break;
        }
        if (&c == &cands[0] || ms < best) {
            best = ms;
            pick = c;
        }
    }
    d->prof = prof;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) {
        // the caller's setting again (it was valid when set)
        (void)lbm_set_steps_per_pass(d, steps0, steps0 == 2 ? tile0 : 0);
        d->tile_h2_asked = asked0;
        return rc;
    }
    if ((rc = lbm_set_steps_per_pass(d, pick.steps, pick.tile_h))) return rc;
    out[0] = pick.steps;
    out[1] = pick.steps == 2 ? d->tile_h2 : d->tile_h;
    out[2] = (int32_t)std::lround(1000.0 * best / (double)steps_per_trial);
    return check_unstable(d);
}

int lbm_degenerate_b(lbm_domain* d, int64_t* count) {
    if (!d || !count) return LBM_EINVAL;
    unsigned long long n = 0;
    if (hipMemcpyAsync(&n, d->degen, 8, hipMemcpyDeviceToHost, d->stream) != hipSuccess ||
        hipStreamSynchronize(d->stream) != hipSuccess)
        return LBM_EDEVICE;
    *count = (int64_t)n;
    return LBM_OK;
}

int lbm_info(lbm_domain* d, int64_t out[8]) {
    if (!d || !out) return LBM_EINVAL;
    out[0] = d->fluid;
    out[1] = d->nl;
    out[2] = d->nb;
    out[3] = (int64_t)d->bytes;
    out[4] = d->tile_w;
    out[5] = d->tile_h;
    out[6] = d->nblocks;
    out[7] = d->fallbacks;
    return LBM_OK;
}

int lbm_get_blocks(lbm_domain* d, int32_t out[3]) {
    if (!d || !out) return LBM_EINVAL;
    const bool on = uses_blocks(d) && d->prof == 0;
    out[0] = on ? d->block.steps : 0;
    out[1] = on ? d->block.lanes : 0;
    out[2] = on ? d->block.ntiles : 0;
    return LBM_OK;
}

void lbm_destroy(lbm_domain* d) {
    if (!d) return;
    (void)hipStreamSynchronize(d->stream);
    free_domain(d);
}

const char* lbm_status_string(int status) {
    switch (status) {
    case LBM_OK: return "ok";
    case LBM_EINVAL: return "invalid argument";
    case LBM_ENOMEM: return "out of memory";
    case LBM_EDEVICE: return "HIP runtime error";
    case LBM_ESINGULAR: return "singular boundary parameter (Filippova-Haenel, q < 1/2, tau = 1)";
    case LBM_EUNSTABLE: return "non-finite total mass";
    default: return "unknown status";
    }
}

}  // extern "C"
