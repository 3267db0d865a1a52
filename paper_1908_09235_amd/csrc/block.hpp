// Several time steps per launch on blocks of the lattice held in LDS.
//
// A workgroup owns a rectangle of nodes, loads f*(t) of that rectangle and a
// halo around it, advances the whole region by `steps` steps in LDS and
// stores f*(t + steps) of its own nodes: the populations cross HBM once per
// `steps` steps and a step costs no launch.  The halo is worked twice, by its
// own workgroup and by its neighbours; per step it shrinks by the reach of a
// step, one node for the pull (two where the quadratic interpolation reads
// x_ff) and one more for the interaction force.  Each step inside the region
// is the boundary pass and the main pass of kernels.hpp with the same
// functions in the same order, every stored value rounded to the storage
// type as there, so the results are those of single steps bit for bit.
//
// One step in a region, s = 1 .. steps (margins from the region's edge):
//   walls    one lane per cut link (host-built list per tile, one chunk of
//            64 per wavefront) evaluates link_value from LDS and writes the
//            incoming population into the solid neighbour's slot; node sums
//            of schemes A, B and Bao by shuffles in link order;
//   pull     every node takes its populations from its neighbours' slots
//            into registers and publishes psi;
//   collide  force, moments and collision, written back in place (the rest
//            population never leaves its thread), on the last step to HBM.
//
// What bounds it.  Small lattices: latency.  A launch takes about 6 us (its
// start, the loads, the stores) and a step about 2 us on a CU of its own,
// against 9 to 13 us a step for a boundary and a main launch: droplet 128^2 in
// FP64, us a step, single steps 11.0, 2 per launch 5.6, 4 per launch 4.1, 6 per
// launch 3.5.  Large lattices: the wavefronts in flight (FP64 populations of
// two regions fill a CU's LDS) and the arithmetic of the halos, 1.3 times a
// single step's with 2 steps per launch; HBM traffic is halved (331 MB read
// and 283 MB written per 2 steps at 2048^2 in FP64, counted).  At 2048^2, us a
// step before and in blocks: FP64 storage 132 and 89, FP32 with FP64 arithmetic
// 77 and 79 (not used there), FP32 arithmetic 72 and 51; single phase, 4 steps,
// FP64 137 and 51, FP32 arithmetic 73 and 32.
//
// Why 32 x 32: the largest square region of which two fit a CU's 160 KB in
// FP64 (8 x 8 bytes of moving populations and 8 of psi a node; the rest
// population stays in registers), so that one workgroup loads while the other
// computes.  Measured and not kept: 1024 lanes per region where there are
// more tiles than CUs (one workgroup a CU: 96 -> 138 us at 2048^2); a resident
// grid that walks over its tiles (registers: 96 -> 108).
#pragma once

#include "kernels.hpp"

namespace lbm {

constexpr int kBlockSteps = 8;  // at most, per launch
constexpr int kBlockBins = 16;   // LDS bins of a step's mass
constexpr int kBlockThreads = 512;
// the side of the square region that a workgroup of `lanes` threads works on
constexpr int kBlockSmall = 576;  // (24 x 24, one node a lane)
constexpr int block_side(int lanes) { return lanes == kBlockSmall ? 24 : 32; }
// tiles of a launch, at most: a launch has fewer than 2^32 lanes (and one
// workgroup more than tiles)
constexpr int kBlockTiles = (1 << 23) - 2;
static_assert((kBlockTiles + 1ll) * kBlockThreads < 1ll << 32, "lanes of a launch");
constexpr int kBlockNodes = kBlockThreads;  // moment records of a tile: one a thread
// bytes of LDS for n moment records and their leaks
constexpr unsigned block_lds(int n) { return 32u * (unsigned)n; }

// Per tile: records of the cut links whose fluid node lies in the region
// (groups of one node together, none across a chunk of 64) and of the nodes
// whose moments the wall rules read.
struct alignas(32) BlockTile {
    int link0, chunks, node0, nodes;
    int x0, y0, cols, rows;  // its own nodes
};
struct alignas(16) BlockLink {
    int meta;             // as BndArgs::lmeta; LK_PAD: padding
    int id;               // slot in the link tables
    unsigned short xb;    // local index of the fluid node
    unsigned short sb;    // moment record of x_b in this tile
    unsigned short sf;    // ... and of x_f where the rule reads its velocity
    unsigned short own;   // x_b belongs to the tile
    double k[2];          // coefficients: chi and c[4], or c[0] and c[1]
};
struct alignas(8) BlockNode {
    int slot;             // side slot
    unsigned short at;    // local index
    unsigned char own, bnd;
};

// Strip and segment of a tile: bands of 8 segments, strip by strip, so that
// the tiles an XCD runs at a time (64, two per CU) form a patch of about 8 x
// 8 and find most of their halos in its L2.
inline int2 block_place(int tile, int nstrips, int nsegs) {
    const int band = tile / (8 * nstrips), r = tile - band * 8 * nstrips;
    const int h = nsegs - 8 * band < 8 ? nsegs - 8 * band : 8;
    const int strip = r / h;
    return make_int2(strip, 8 * band + (r - strip * h));
}

struct BlockArgs {
    void* f[2];                            // f[cur]: f*(t); f*(t + steps) goes to the other
    double* mom[2];                        // side moments of the times of f[0], f[1]
    const uint8_t* flags;
    const float* psiw;                     // FP16 storage: psi_w of solid nodes
    MassTile* partial;                     // [step][tile]
    const BlockTile* tiles;
    const BlockLink* links;
    const BlockNode* nodes;
    const double* lc;                      // link tables (see BndArgs)
    const double* luw;
    unsigned long long* negrest;
    unsigned long long* degen;
    int fix, moving;                       // moving: some wall has a velocity
    int chi;                               // the rule is of the form of Eq. (7)
    int max_len;                           // links of a node, at most
    int nx, ny, pitch;
    long long plane;
    int halo, pull;                        // pull: margin of a step's pull
    int ntiles;
    int max_nodes;                         // moment records of LDS
    unsigned mom_bytes, link_bytes, node_bytes;
    int open_x;
    double inlet_u;
    MassUnit mass;
    double* hist;                          // (batches: see BInst)
    long long cap;
    long long* unstable;
    Phys<double> ph64;
    Phys<float> ph32;
};

// The value of the next lane (whole-wavefront shift; the last lane gets 0).
__device__ __forceinline__ double next_lane(double v) {
    const uint2_t u = __builtin_bit_cast(uint2_t, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)u.x, 0x130, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)u.y, 0x130, 0xf, 0xf, false);
    return __builtin_bit_cast(double, uint2_t{(unsigned)lo, (unsigned)hi});
}

template <typename R>
__device__ __forceinline__ Phys<R> block_phys(const LBM_CONST_AS BlockArgs& a) {
    if constexpr (sizeof(R) == 8) return a.ph64;
    else return a.ph32;
}

// Wavefronts per SIMD: two workgroups of 512 lanes on a CU (FP64 populations
// fill its LDS), three with FP32 arithmetic, which fits 80 registers.
template <typename R>
constexpr int block_waves(int nt) {
    return nt == kBlockSmall ? 3 : sizeof(R) == 4 && nt == kBlockThreads ? 6 : 4;
}

// `steps` steps of tile `tile` of the domain described at ka (uniform, in
// memory that no launch writes), whose f*(t) lies in f[cur].
template <typename S, typename R, int EOS, int DEV, int NT>
__device__ __forceinline__ void block_tile(const BlockArgs* args, int cur, int steps, int tile) {
    static_assert(DEV == 0 || DEV == 1, "per-node references are not blocked");
    constexpr int RW = block_side(NT), RH = RW, NN = RW * RH, NPT = NN / NT, NW = NT / 64;
    static_assert(NN % NT == 0 && NT % 64 == 0, "every thread has as many nodes");
    constexpr unsigned ES = sizeof(S);
    constexpr int NP = EOS == EOS_NONE ? (NN * 2 + (int)sizeof(R) - 1) / (int)sizeof(R) : NN;
    __shared__ S fs[8][NN];   // moving populations of f*
    __shared__ R psb[NP];     // psi (at first: the moment record of each node)
    __shared__ unsigned long long mq[kBlockSteps][kBlockBins], mfine[kBlockSteps][kBlockBins];
    __shared__ double mbig[kBlockSteps][NW];
    extern __shared__ double dyn[];
    const LBM_CONST_AS BlockArgs& a = *ro(args);
    double* const mom = dyn;                        // [record][3]: rho, u_x, u_y
    double* const leak = dyn + 3 * a.max_nodes;     // scheme A: [record]

    const int t = threadIdx.x;
    const BlockTile bt = ro(a.tiles)[tile];
    const int x0 = bt.x0, y0 = bt.y0, ncols = bt.cols, nrows = bt.rows;
    const int halo = a.halo, pull = a.pull;
    const int fix = a.fix, moving = a.moving, max_len = a.max_len;
    const int open_x = a.open_x, chi = a.chi;
    const int reach = pull + (EOS == EOS_NONE ? 0 : 1);
    const unsigned pitch = (unsigned)a.pitch;
    const unsigned pb = (unsigned)(a.plane * ES);
    const rsrc_t rs = make_rsrc(cur ? a.f[1] : a.f[0], 9u * pb);
    const rsrc_t rfl = make_rsrc(a.flags, pitch * (unsigned)a.ny);
    const rsrc_t rpw = make_rsrc(a.psiw, ES == 2 ? pitch * (unsigned)a.ny * 4u : 0u);
    // local coordinates of the thread's node j, and its place in the lattice
    // (a lattice narrower than the region repeats in it)
    auto lx_at = [](int t, int j) { return (t + j * NT) % RW; };
    auto ly_at = [](int t, int j) { return (t + j * NT) / RW; };
    auto wrap = [](int v, int n, int reach) {
        if (n >= reach) {
            v = v < 0 ? v + n : v;
            return v >= n ? v - n : v;
        }
        v %= n;
        return v < 0 ? v + n : v;
    };
    auto x_at = [&](int t, int j, int nx) { return wrap(x0 - halo + lx_at(t, j), nx, RW); };
    auto at = [&](int t, int j, int nx, int ny) {
        return (unsigned)wrap(y0 - halo + ly_at(t, j), ny, RH) * pitch + (unsigned)x_at(t, j, nx);
    };

    // ---- all loads of the tile: its lists first, then the region of f*(t)
    // (solid nodes' slots come along unread), then the moments that the list
    // names, which so travel with the region.  No branch: a lane without a
    // record reads past its buffer, which yields 0, so each wait leaves the
    // later loads in flight.  (The lists after the region, and the tile's place from
    // four 64-bit divisions instead of its entry: 1700 cycles more a launch;
    // 2048^2 FP64 2110 -> 1997 us per 20 steps, 6 sessile droplets 4780 ->
    // 4490 per 192.)
    const rsrc_t rli = make_rsrc(a.links, a.link_bytes), rno = make_rsrc(a.nodes, a.node_bytes);
    const rsrc_t rmo = make_rsrc(cur ? a.mom[1] : a.mom[0], a.mom_bytes);
    uint4_t l0, l1;
    S f0[NPT];
    // Its place in the lattice, for the stores.  (Worked out again there by FP32
    // arithmetic on 512 lanes, whose registers are counted: kept, 15 spill,
    // 4096 x 2048 115 -> 130 us a step; with FP64 arithmetic, 50 instructions
    // a launch less: 1600 x 1000 25.1 -> 24.7, 2048^2 100 -> 99.)
    constexpr bool KEEP = sizeof(R) == 8 || NT != kBlockThreads;
    unsigned place[KEEP ? NPT : 1];
    // per node, 16 bits: its distance from the region's edge (solid nodes: 0), by
    // which a step decides whether to work it; 16 own (and fluid), 32 scheme
    // A's; (moment record + 1) << 6
    static_assert(NPT <= 2, "two nodes' facts fit a register");
    unsigned info = 0;
    auto fact = [&](int j) { return info >> (16 * j); };
    auto inner = [&](int j) { return (int)(fact(j) & 15); };
    static_assert(RW <= 32 && kBlockNodes < 1024, "four bits and ten");
    {
        const bool has_link = (t >> 6) < bt.chunks, has_node = t < bt.nodes;
        const uint2_t nd =
            bload<uint2_t>(rno, has_node ? (unsigned)(bt.node0 + t) * 8u : kOOB, 0u);
        const unsigned lo =
            has_link ? (unsigned)(bt.link0 + t) * (unsigned)sizeof(BlockLink) : kOOB;
        l0 = bload<uint4_t>(rli, lo, 0u);
        l1 = bload<uint4_t>(rli, lo, 16u);
        S g[NPT][9];
        uint8_t fl[NPT];
        float pw[NPT];
#pragma unroll
        for (int j = 0; j < NPT; ++j) {
            const unsigned o = at(t, j, a.nx, a.ny);
            if constexpr (KEEP) place[j] = o;
            fl[j] = bload<uint8_t>(rfl, o, 0u);
            pw[j] = ES == 2 ? bload<float>(rpw, o * 4u, 0u) : 0.0f;
#pragma unroll
            for (int q = 0; q < 9; ++q) g[j][q] = bload<S>(rs, o * ES, q * pb);
        }
        // the moment record of each node, until psi takes the place
        unsigned short* const rec = reinterpret_cast<unsigned short*>(psb);
#pragma unroll
        for (int j = 0; j < NPT; ++j) rec[t + j * NT] = 0;
        for (int i = t; i < kBlockSteps * kBlockBins; i += NT) {
            (&mq[0][0])[i] = 0;
            (&mfine[0][0])[i] = 0;
        }
        for (int i = t; i < kBlockSteps * NW; i += NT) (&mbig[0][0])[i] = 0.0;
        __syncthreads();
        const unsigned mo = has_node ? nd.x * 24u : kOOB;
        double m[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) m[k] = bload<double>(rmo, mo + 8u * k, 0u);
        if (has_node)
            rec[nd.y & 0xffffu] = (unsigned short)((t + 1) | (nd.y >> 24 ? 0x8000 : 0));
#pragma unroll
        for (int j = 0; j < NPT; ++j) {
            const int lx = lx_at(t, j), ly = ly_at(t, j);
            const bool own = lx >= halo && lx < halo + ncols && ly >= halo && ly < halo + nrows;
            const int in = min(min(lx, RW - 1 - lx), min(ly, RH - 1 - ly));
            if (!(fl[j] & FL_SOLID)) info |= (unsigned)(in | (own ? 16 : 0)) << (16 * j);
            f0[j] = g[j][0];
            if constexpr (ES == 2)
                if (fl[j] & FL_SOLID) f0[j] = S(0);
#pragma unroll
            for (int q = 1; q < 9; ++q) fs[q - 1][t + j * NT] = g[j][q];
        }
        if (has_node) {
#pragma unroll
            for (int k = 0; k < 3; ++k) mom[3 * t + k] = m[k];
        }
        __syncthreads();
        if (bt.chunks > 0) {
#pragma unroll
            for (int j = 0; j < NPT; ++j) {
                const unsigned r = rec[t + j * NT];
                info |= ((r >> 15) << 5 | (r & 0x3ffu) << 6) << (16 * j);
            }
        }
        if constexpr (EOS != EOS_NONE) {
            // psi of solid nodes, which no step changes
            if (bt.chunks > 0) __syncthreads();
#pragma unroll
            for (int j = 0; j < NPT; ++j)
                if (fl[j] & FL_SOLID) psb[t + j * NT] = ES == 2 ? R(pw[j]) : R(f0[j]);
        }
    }
    for (int s = 1; s <= steps; ++s) {
        // The arguments and the thread's place are read anew in every step:
        // kept over the loop, they and what is derived from them would take
        // more registers than there are.
        const BlockArgs* ka = args;
        int t = threadIdx.x;
        asm volatile("" : "+s"(ka));
        asm volatile("" : "+v"(t), "+v"(l0), "+v"(l1), "+v"(info));
        const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
        const LBM_CONST_AS BlockArgs& a = *ro(ka);
        const Phys<R> ph = block_phys<R>(a);
        // ---- walls
        if (bt.chunks > 0) {
            if (wave < bt.chunks) {
                const int meta = (int)l0.x, kind = (meta >> 4) & 15;
                const bool active = kind != LK_PAD;
                const int d = meta & 15, od = lane_opp(d), back = lane_cx(d) + lane_cy(d) * RW;
                const int len = active ? (meta >> 8) & 15 : 0, pos = active ? (meta >> 12) & 15 : 0;
                const int xb = (int)(l0.z & 0xffffu), sb = (int)(l0.z >> 16);
                const int sf = (int)(l0.w & 0xffffu);
                const bool own = l0.w >> 16;
                auto fst = [&](int q, int n) {
                    const double v = double(fs[q - 1][n]);
                    return DEV == 1 ? v + lane_wt(q) * double(ph.rref) : v;
                };
                // what the rule reads from LDS, all at once (padding records
                // point at places that exist)
                const double* const m = mom + 3 * sb;
                double fab = fst(d, xb);
                const double rho_b = m[0], ubx = m[1], uby = m[2];
                double v[4] = {0.0, 0.0, 0.0, 0.0};
                if (chi) {
                    v[0] = mom[3 * sf + 1];
                    v[1] = mom[3 * sf + 2];
                } else {
                    v[0] = fst(od, xb);
                    v[1] = fst(d, xb - back);
                    v[2] = fst(od, xb - back);
                    if (pull > 1) v[3] = fst(d, xb - 2 * back);
                }
                double r = 0.0, ch = 0.0, bk = 0.0, wl = 0.0;
                if (active) {
                    const double k0 = __builtin_bit_cast(double, uint2_t{l1.x, l1.y});
                    const double k1 = __builtin_bit_cast(double, uint2_t{l1.z, l1.w});
                    double c[7] = {k0, k1, 0.0, k0, k1, 0.0, 0.0};
                    if (pull > 1) c[2] = a.lc[8 * (int)l0.y + 2];
                    double uwx = 0.0, uwy = 0.0;
                    if (moving) {
                        c[5] = a.lc[8 * (int)l0.y + 5];
                        c[6] = a.lc[8 * (int)l0.y + 6];
                        uwx = a.luw[2 * (int)l0.y];
                        uwy = a.luw[2 * (int)l0.y + 1];
                    }
                    r = link_value(kind, d, c, uwx, uwy, fab, rho_b, ubx, uby, ch, bk, wl,
                                   [&](int what) -> double {
                                       switch (what) {
                                       case LV_OD_B: case LV_UFX: return v[0];
                                       case LV_D_F: case LV_UFY: return v[1];
                                       case LV_OD_F: return v[2];
                                       case LV_D_FF: return v[3];
                                       default: return 0.0;  // (Zhao-Yong is not blocked)
                                       }
                                   });
                } else {
                    fab = 0.0;
                }
                // node sums in link order: the group's values pass by its
                // first lane, one lane further a turn
                if (fix == 2 || fix == 3) {
                    const bool b = fix == 2;
                    double x = b ? ch * fab : fab, y = b ? ch * bk : bk;
                    double num = 0.0, den = 0.0, mag = 0.0;
                    for (int m = 0; m < max_len; ++m) {
                        num = m < len ? num + x : num;
                        den = m < len ? den + y : den;
                        mag = m < len ? mag + fabs(y) : mag;
                        x = next_lane(x);
                        y = next_lane(y);
                    }
                    const bool ok = den != 0.0 && fabs(den) > 1e-12 * mag;
                    const double rho_s = __shfl(ok ? num / den : NAN, lane - pos, 64);
                    if (active && pos == 0 && own && !ok && mag > 0.0 && a.degen)
                        atomicAdd(a.degen, 1ull);
                    if (!isnan(rho_s)) r = (1.0 - ch) * fab + ch * (rho_s * bk) - wl;
                }
                if (fix == 1) {
                    double x = fab, y = r + wl;
                    double out_sum = 0.0, in_sum = 0.0;
                    for (int m = 0; m < max_len; ++m) {
                        out_sum = m < len ? out_sum + x : out_sum;
                        in_sum = m < len ? in_sum + y : in_sum;
                        x = next_lane(x);
                        y = next_lane(y);
                    }
                    if (active && pos == 0) leak[sb] = out_sum - in_sum;
                }
                if (active)
                    fs[od - 1][xb + back] = S(r - (DEV == 1 ? lane_wt(d) * double(ph.rref) : 0.0));
            }
            __syncthreads();
        }
        // ---- pull and psi
        const int mp = reach * (s - 1) + pull, mc = reach * s;
        constexpr bool SPLIT = sizeof(R) == 8 || DEV != 0;
        // (read here, so that it travels with the pull: read where the sum begins,
        // the step waits for it, 100 x 50 in FP64 152.6 us per 64 steps instead of 149.0)
        MassUnit mass;
        mass.magic = a.mass.magic;
        S g[NPT][9];
#pragma unroll
        for (int j = 0; j < NPT; ++j) {
            const int n = t + j * NT;
            if (inner(j) >= mp) {
                if ((fact(j) & 32) && fix == 1) {
                    // Eq. (18)
                    const double v = double(f0[j]) + leak[(int)(fact(j) >> 6 & 0x3ffu) - 1];
                    f0[j] = S(v);
                    if ((fact(j) & 16) && a.negrest) {
                        const double fr = DEV == 1 ? v + wt(0) * double(ph.rref) : v;
                        if (fr < 0.0) atomicAdd(a.negrest, 1ull);
                    }
                }
                g[j][0] = f0[j];
#pragma unroll
                for (int q = 1; q < 9; ++q) g[j][q] = fs[q - 1][n - cx(q) - cy(q) * RW];
                if constexpr (EOS == EOS_NONE) {
                    if (open_x) {
                        // open x boundaries, as open_rows fills the seam
                        const int x = x_at(t, j, a.nx);
                        auto ref = [&](int q) {
                            return DEV == 1 ? wt(q) * double(ph.rref) : 0.0;
                        };
                        auto ld = [&](int q) { return double(g[j][q]) + ref(q); };
                        if (x == 0) {
                            const double p0 = ld(0), p2 = ld(2), p4 = ld(4);
                            const double p3 = ld(3), p6 = ld(6), p7 = ld(7);
                            const double U = a.inlet_u;
                            const double rho =
                                (p0 + p2 + p4 + 2.0 * (p3 + p6 + p7)) / (1.0 - U);
                            const double hh = 0.5 * (p2 - p4), s6 = 1.0 / 6.0 * rho * U;
                            g[j][1] = S(p3 + 2.0 / 3.0 * rho * U - ref(1));
                            g[j][5] = S(p7 - hh + s6 - ref(5));
                            g[j][8] = S(p6 + hh + s6 - ref(8));
                        } else if (x == a.nx - 1) {
                            g[j][3] = S(double(fs[2][n]) + ref(3) - ref(3));
                            g[j][6] = S(double(fs[5][n - RW]) + ref(6) - ref(6));
                            g[j][7] = S(double(fs[6][n + RW]) + ref(7) - ref(7));
                        }
                    }
                } else {
                    R f[9];
#pragma unroll
                    for (int q = 0; q < 9; ++q) f[q] = R(g[j][q]);
                    const R rho = DEV == 1 ? ph.rref + dens<R>(f) : dens<R>(f);
                    psb[n] = psi_of<EOS, R>(rho, ph);
                }
            }
        }
        __syncthreads();
        // ---- force, moments, collision
        const bool last = s == steps;
        MassSum<SPLIT> msum(mass);
#pragma unroll
        for (int j = 0; j < NPT; ++j) {
            const int n = t + j * NT;
            const bool own = fact(j) & 16;
            if (last ? own : inner(j) >= mc) {
                R fc[9];
#pragma unroll
                for (int q = 0; q < 9; ++q) fc[q] = R(g[j][q]);
                R ps[9];
                if constexpr (EOS != EOS_NONE) {
#pragma unroll
                    for (int q = 0; q < 9; ++q) ps[q] = psb[n + cx(q) + cy(q) * RW];
                }
                R rho, drho, ux, uy, Fx, Fy;
                node_moments<R, EOS, DEV>(fc, ps, ph, rho, drho, ux, uy, Fx, Fy);
                const double rho_d = DEV == 1 ? double(ph.rref) + double(drho) : double(rho);
                msum.add(own, rho_d);
                const int rec = (int)(fact(j) >> 6 & 0x3ffu) - 1;
                if (rec >= 0) {
                    mom[3 * rec] = rho_d;
                    mom[3 * rec + 1] = double(ux);
                    mom[3 * rec + 2] = double(uy);
                }
                R dh[9];
                collide<R>(fc, rho, drho, ux, uy, Fx, Fy, ph, dh);
                if (last) {
                    const rsrc_t rd = make_rsrc(cur ? a.f[0] : a.f[1], 9u * pb);
                    const unsigned vo = (KEEP ? place[KEEP ? j : 0] : at(t, j, a.nx, a.ny)) * ES;
#pragma unroll
                    for (int q = 0; q < 9; ++q) bstore(S(fc[q] + dh[q]), rd, vo, q * pb);
                } else {
                    f0[j] = S(fc[0] + dh[0]);
#pragma unroll
                    for (int q = 1; q < 9; ++q) fs[q - 1][n] = S(fc[q] + dh[q]);
                }
            }
        }
        // into the step's bins, as integers (FP64 atomics in LDS took the
        // droplet at 2048^2 in FP64 from 107 to 120 us a step)
        {
            const double x = SPLIT ? msum.a : msum.a + mass.magic, u = x - mass.magic;
            const double y = SPLIT ? msum.b : msum.a - u;
            const double z = y + mass.magic * kMassFine;
            const bool in = fabs(u) < 0.25 * mass.magic;  // 1.5 * 2^50 units
            const long long q = __builtin_bit_cast(long long, x) -
                                __builtin_bit_cast(long long, mass.magic);
            const long long fn = __builtin_bit_cast(long long, z) -
                                 __builtin_bit_cast(long long, mass.magic * kMassFine);
            if (in && (q | fn) != 0) {
                atomicAdd(&mq[s - 1][t % kBlockBins], (unsigned long long)q);
                atomicAdd(&mfine[s - 1][t % kBlockBins], (unsigned long long)fn);
            }
            if (__builtin_amdgcn_ballot_w64(!in)) {  // not in a stable run
                double v = in ? 0.0 : u + y;
                for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
                if (lane == 0) mbig[s - 1][wave] = v;
            }
        }
        __syncthreads();
    }
    // ---- moments of t + steps and the masses
    if (t < bt.nodes) {
        const BlockNode n = a.nodes[bt.node0 + t];
        double* const out = cur ? a.mom[0] : a.mom[1];
        if (n.own) {
#pragma unroll
            for (int k = 0; k < 3; ++k) out[3 * n.slot + k] = mom[3 * t + k];
        }
    }
    if (t < steps) {
        long long q = 0, fine = 0;
        for (int i = 0; i < kBlockBins; ++i) {
            q += (long long)mq[t][i];
            fine += (long long)mfine[t][i];
        }
        double big = 0.0;
        for (int w = 0; w < NW; ++w) big += mbig[t][w];
        a.partial[(long long)t * a.ntiles + tile] =
            mass_pack(q, fine, big, mass_unit(a.mass.magic));
    }
}

// One domain; the last workgroup reduces the previous launch's masses.
struct BlockRun {
    int cur, steps, do_reduce;
    MassPass prev;
};
struct BlockKernarg {
    BlockArgs a;
    BlockRun r;
};
template <typename S, typename R, int EOS, int DEV, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(block_waves<R>(NT)))) void
k_block(BlockKernarg k) {
    if ((int)blockIdx.x == (int)gridDim.x - 1) {
        if (k.r.do_reduce) reduce_pass<8>(k.r.prev);
        return;
    }
#if defined(__HIP_DEVICE_COMPILE__)
    // (the arguments where they lie, to be read again in every step)
    const BlockArgs* args = (const BlockArgs*)__builtin_amdgcn_kernarg_segment_ptr();
#else
    const BlockArgs* args = &k.a;
#endif
    block_tile<S, R, EOS, DEV, NT>(args, k.r.cur, k.r.steps,
                                   xcd_tile(blockIdx.x, k.a.ntiles));
}

// ---------------------------------------------------------------- batches
// The instances of a batch advance together, up to `steps` steps a launch.
// An instance leaves its last step, and a step that turned out non-finite, to
// single steps, so that it ends as they would leave it: a launch that meets
// a non-finite mass in step j is dropped for that instance (its f*(t) is
// still there), the next one makes j - 1 steps, and single steps go on.
__device__ __forceinline__ int block_steps(long long remaining, int hold, int steps) {
    if (remaining <= 0 || hold < 0) return 0;
    if (hold > 0) return hold;
    return remaining - 1 < steps ? (int)(remaining - 1) : steps;
}

struct BlockBatch {
    const BlockArgs* __restrict__ inst;  // per slot
    BState* __restrict__ state;
    const int2* __restrict__ tiles;      // (instance, tile)
    int ninst, steps;
};

template <typename S, typename R, int EOS, int DEV>
__global__ __launch_bounds__(kBlockThreads)
    __attribute__((amdgpu_waves_per_eu(block_waves<R>(kBlockThreads)))) void k_block_batch(
        BlockBatch b) {
    const int2 te = ro(b.tiles)[xcd_tile(blockIdx.x, gridDim.x)];
    const BState st = ro<BState>(b.state)[te.x];
    const int n = block_steps(st.remaining, st.hold, b.steps);
    if (n <= 0) return;
    block_tile<S, R, EOS, DEV, kBlockThreads>(b.inst + te.x, st.cur, n, te.y);
}

// Per instance: the masses of the launch and the state it leaves.
template <int Unused = 0>
__global__ __launch_bounds__(256) void k_block_reduce(BlockBatch b) {
    __shared__ double m[kBlockSteps];
    for (int i = blockIdx.x; i < b.ninst; i += gridDim.x) {
        BState* st = b.state + i;
        const int n = block_steps(st->remaining, st->hold, b.steps);
        if (n <= 0) continue;
        const auto& I = ro(b.inst)[i];
        sum_masses<16>(I.partial, I.ntiles, n, I.ntiles, mass_unit(I.mass.magic),
                   [&](int s, double v) { m[s] = v; });
        if (threadIdx.x == 0) {
            int bad = 0;
            while (bad < n && isfinite(m[bad])) ++bad;
            if (bad == n) {
                for (int s = 0; s < n; ++s) I.hist[(st->t + 1 + s) % I.cap] = m[s];
                st->t += n;
                st->remaining -= n;
                st->cur ^= 1;
                if (st->hold > 0) st->hold = -1;
            } else {
                st->hold = bad > 0 ? bad : -1;
            }
        }
        __syncthreads();
    }
}

}  // namespace lbm
