// Host-side state of one domain, shared by the single-domain API
// (lbm2p.hip) and the batched and served forms (batch.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <map>
#include <vector>

#include "../../include/lbm2p.h"
#include "launch.hpp"

namespace lbm {

// Device memory carved out of one hipMalloc: first fit over 256-byte
// granules with a coalescing free list.  Bookkeeping is host-only, so
// taking and returning memory never synchronises the device; the caller
// returns a block only once no queued work uses it.
class Arena {
  public:
    ~Arena();
    int init(size_t bytes);  // lbm_status
    void* alloc(size_t bytes);  // nullptr if nothing fits
    void release(void* p);
    size_t capacity() const { return cap_; }
    size_t used() const { return used_; }
    size_t largest_free() const;

  private:
    char* base_ = nullptr;
    size_t cap_ = 0, used_ = 0;
    std::map<size_t, size_t> free_;  // offset -> bytes
    std::map<size_t, size_t> live_;  // offset -> bytes
};

}  // namespace lbm

namespace lbm {

// How a domain's runs of steps are cut into launches of k_block (steps per
// launch; 0: not used), with the tables of its tiles on the device.
struct BlockPlan {
    int steps = 0, halo = 0, pull = 0;
    int nstrips = 0, nsegs = 0, ntiles = 0, max_nodes = 0, max_len = 0;
    unsigned link_bytes = 0, node_bytes = 0;
    bool moving = false;
    int lanes = kBlockThreads;  // per tile (see block_t)
    BlockTile* tiles = nullptr;
    BlockLink* links = nullptr;
    BlockNode* nodes = nullptr;
    MassTile* partial[2] = {nullptr, nullptr};  // [step][tile], used in turn
    int set = 0;                                // the one written last
};

// Host copies of the link tables that k_block's tables are made from.
struct LinkTables {
    std::vector<int> node, meta, slotb, slotf;
    std::vector<double> c;
};

}  // namespace lbm

struct lbm_domain {
    int nx = 0, ny = 0, pitch = 0;
    long long plane = 0;
    int storage = 0, eos = 0, coll = 0, rule = 0, fix = 0;
    int tile_w = 0, tile_h = 0, nstrips = 0, nsegs = 0, nblocks = 0;
    size_t esize = 8;
    size_t fbytes = 0;  // one state buffer: nine planes (+ the FP16 per-node
                        // form's FP32 density plane)
    void* f[2] = {nullptr, nullptr};
    int cur = 0;
    uint8_t* flags = nullptr;
    float* psiw = nullptr;  // FP16 storage: psi_w of solid nodes in FP32
    int* side_idx = nullptr;
    double* side_mom[2] = {nullptr, nullptr};  // moments of the time of f[0], f[1]
    double* side_f = nullptr;
    int nslots = 0;
    bool save_f = false;
    // mass partials of the last pass: one array of partial_cap per step
    lbm::MassTile* partial = nullptr;
    lbm::MassUnit mass{};
    double* hist = nullptr;
    long long* unstable = nullptr;
    double* mom_out = nullptr;
    int* lref = nullptr;   // per link: side slot whose density encodes its ghost
    int open_x = 0;        // velocity inlet at x = 0, outlet at x = nx - 1
    double inlet_u = 0.0;
    double* force = nullptr;   // wall force partials, two per link block
    unsigned long long* negrest = nullptr;  // scheme A: negative rest count
    unsigned long long* degen = nullptr;    // scheme B / Bao: cancelled sums count
    bool force_valid = false;  // a boundary pass has written them
    int nb = 0, nl = 0;
    int nslot_links = 0;
    int *lnode = nullptr, *lmeta = nullptr, *lghost = nullptr, *lxf = nullptr,
        *lxff = nullptr, *lslotb = nullptr, *lslotf = nullptr;
    double *lc = nullptr, *luw = nullptr;
    long long cap = 0, t = 0;
    long long* clock = nullptr;  // device: step of the last recorded mass
    // Two steps per pass (k_main2): fused = 2 when in use (1: every step
    // is its own pass); eligible when the form allows it.
    int fused = 1;
    bool fusable = false;
    bool tile_h2_asked = false;  // by the caller, not the default
    int tile_h2 = 0, nstrips2 = 0, nsegs2 = 0, nblocks2 = 0;
    int* node_link = nullptr;    // per node (pitch layout): first link slot + 1, or 0
    int* tile_order = nullptr;   // tile of each workgroup of the two-step pass
    std::vector<int> bnd_x, bnd_y;  // host: the boundary nodes (tile weights)
    int pending_steps = 0;       // steps of the last pass whose masses are pending
    bool pending_block = false;  // it was a launch of k_block
    lbm::BlockPlan block;
    lbm::LinkTables links;       // instances of a batch: kept for new plans
    // After a two-step pass f*(t - 1) is not in memory: the buffer that
    // held f*(t - 2) still does, with the ghosts of step t - 1, and the
    // moments at t and the wall force of the last step are read from a
    // replay of step t - 1 into these buffers.
    bool last_fused = false;
    bool replay_valid = false;
    void* frep = nullptr;
    double* side_mom_rep = nullptr;
    bool pending = false;
    long long pending_t = 0;
    hipStream_t stream = nullptr;
    int device = 0;              // the GPU the domain lives on
    // Captured runs of 2^k steps (k = 0 .. kGraphLevels - 1), per parity of
    // the buffer that holds f*(t) when the run starts; built on first use
    // on a capture stream of the domain's own and replayed on `stream`.
    static constexpr int kGraphLevels = 6;
    hipGraphExec_t graphs[2][kGraphLevels] = {};
    hipStream_t cap_stream = nullptr;
    bool graphs_off = false;     // capture failed once: plain launches
    lbm::Phys<double> ph64{};
    lbm::Phys<float> ph32{};
    size_t bytes = 0;
    long long fluid = 0, fallbacks = 0;
    std::vector<void*> allocs;
    lbm::Arena* arena = nullptr;  // sub-allocate from it instead of hipMalloc
    int partial_cap = 0;          // partials held (enough for 64 x 8 tiles)
    int prof = 0;                 // record every prof-th step (0: off)
    int nrec = 0;
    std::vector<hipEvent_t> ev;
    double main_ms = 0, bnd_ms = 0;
    long long main_n = 0, bnd_n = 0;
};

namespace lbm {

// Build a domain from a descriptor (all device work on desc->stream, which
// is synchronised before returning).  With an arena, device memory comes
// from it.
int domain_create(const lbm_desc* desc, Arena* arena, lbm_domain** out);
void domain_free(lbm_domain* d);
// The tile shape of the main pass (tile_w 64/128/256, tile_h >= 1 with at
// most partial_cap tiles); the next launch uses it.
int domain_set_tiles(lbm_domain* d, int tile_w, int tile_h);
Ctx domain_ctx(lbm_domain* d);

// k_block (see block.hpp).  Zhao-Yong needs the pre-collision populations of
// the step before, and the FP16 per-node form a second plane: both stay with
// single steps.
bool domain_blockable(const lbm_domain* d);
// Tiles of a launch of `steps` steps (0: its halos leave none).
long long domain_block_tiles(const lbm_domain* d, int steps, int lanes = kBlockThreads);
// The tables of `steps` steps per launch for an instance of a batch, in memory
// of `pool` (false if it has none left or the tables do not fit a tile; the
// instance has no plan then).  Waits for the instance's stream.
bool domain_make_blocks(lbm_domain* d, int steps, Arena* pool);
void domain_drop_blocks(lbm_domain* d, Arena* pool);
BlockArgs block_args(const lbm_domain* d);
// Whether the caller is recording a stream: launches of blocks would be recorded
// with the buffers of that call, so it goes the way of single steps.
bool being_captured(hipStream_t stream);

// Estimated time of a step in us: single steps (boundary and main launch), and
// launches of k_block with `steps` steps on `tiles` tiles.  Fitted to measured
// steps of droplets (64^2 to 2048^2) and of the static channel; what matters
// is where the curves cross.
//   single: two launches and the populations at 4.6 TB/s (FP16 at 3.7);
//     measured in FP64 / FP32 / FP16 storage: 13.3 / 12.2 / 12 at 400^2,
//     31.4 / 24.7 / 20 at 1024^2, 132 / 75 / 48 at 2048^2.
//   k_block: so much a launch and a step while every tile has a CU of its own,
//     then a cost per further tile, of which FP64 arithmetic, the two-phase
//     step and the halos (a step more shrinks the tiles) are the parts.
//     Measured, us a step with the number of steps taken (single steps):
//     droplets, FP64: 3.5 with 6 at 128^2 (11.0), 6.8 with 3 at 400^2 (13.1),
//     24.2 with 2 at 1024^2 (32.4), 91.9 with 2 at 2048^2 (140.7); FP32 with
//     FP64 arithmetic: 22.2 with 2 at 1024^2 (24.6), 79.3 with 2 at 2048^2
//     (77.1: the arithmetic of the halos); FP32: 14.3 and 54.8 (21.5, 75.3);
//     FP16 deviations: 15.0 and 43.6 (20.5, 44.3).  Single phase at 2048^2:
//     FP64 60.0 with 4 (139.6), FP32 with FP64 arithmetic 52.8 with 3 (75.2),
//     FP32 35.0 with 4 (75.1), FP16 deviations 36.6 with 3 (41.0).
double single_us(size_t esize, double fluid);
double block_us(const lbm_domain* d, int steps, long long tiles, int ncu,
                int lanes = kBlockThreads);
// The buffer the moments at the current time are pulled from: f*(t - 1)
// with the ghosts of step t (after a two-step pass, rebuilt by a replay of
// step t - 1 into the domain's replay buffer; also forms the wall force of
// the last step).  Enqueued on the domain's stream; allocates nothing.
const void* moments_source(lbm_domain* d);

}  // namespace lbm
