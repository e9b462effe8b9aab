// Launchers of the block sweep (ma_fsweep.h) and of the z-stream sweep
// (ma_zsweep.h): the shapes they are built for and the automatic choice
// between them.
#include "ma_fsweep.h"
#include "ma_zsweep.h"

#include <algorithm>

namespace mafas {

namespace {

struct BCfg {
    int tx, ty, tz, nt;
    // z-stream sweeps: -1 chunks chosen by the model below, > 0 about zwg
    // workgroups in all; 0: a block sweep
    int zwg;
};
// Shapes (index = tile_config - 1).  Block sweeps: small blocks keep the
// recomputation cheap in absolute terms and give many workgroups; more
// threads per block cut the rounds of updates per phase, which is what a
// sweep of a small grid waits on.  Z-stream sweeps (tz unused): TX x TY
// columns whose update items (TX TY + 3 (TX + TY) + 14 per step) nearly
// fill the workgroup once or twice; 32 x 24 fills 1024 items with one
// colour per wavefront, which makes the colour's plane and ring slots
// scalars (a step about 2% faster than 32 x 26 with its two mixed
// wavefronts).  The planes are cut into chunks, by the model of zs_chunks
// or into about zwg workgroups (one per compute unit at a time, the ring
// filling most of the LDS).
constexpr BCfg kCfg[] = {{8, 8, 8, 256, 0},   {8, 8, 8, 512, 0},  {8, 8, 8, 1024, 0},
                         {16, 8, 4, 256, 0},  {16, 16, 8, 512, 0}, {8, 8, 4, 512, 0},
                         {8, 8, 4, 256, 0},   {32, 26, 0, 1024, -1}, {32, 26, 0, 512, -1},
                         {32, 26, 0, 1024, 1536}, {40, 20, 0, 1024, -1},
                         {32, 24, 0, 1024, -1}};
constexpr int kZsPureConfig = 11;
// 8-colour block sweeps: enough threads for the first phase (its block grows
// by 5, 3, 1 nodes) in one round.
// Then the first and the last four phases of a sweep, a launch each (u -> t -> u):
// the phases of a launch lie in planes of one parity, so its halo is one plane
// and 4 x 2 nodes, a block recomputes 1.24 x its updates, and a sweep reads u
// twice where eight colour launches read it eight times.
constexpr BCfg kCfg8[] = {{8, 8, 4, 256, 0},  {8, 8, 8, 320, 0}, {16, 8, 8, 512, 0},
                          {32, 8, 8, 512, 0}, {32, 8, 8, 512, 0}};
constexpr int kNumCfg8 = int(sizeof(kCfg8) / sizeof(kCfg8[0]));

const BCfg &shape_of(int order, int cfg) { return order == 0 ? kCfg[cfg] : kCfg8[cfg]; }

// Compute units of the current device (one z-stream workgroup each at a time).
int device_cus()
{
    static int cus = 0;
    if (cus <= 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
            v > 0)
            cus = v;
        else
            cus = 256;
    }
    return cus;
}

// Chunks of a z-stream sweep over `cols` columns of an n grid: a chunk of zc
// planes takes zc + 10 steps (the phases are skewed over 7 planes, plus the
// pipeline's prefetch), and the workgroups run in rounds of one per compute
// unit, so the sweep takes about ceil(cols * chunks / CUs) * (zc + 10) step
// times; the chunk count minimising that (at least 16 planes a chunk).
int zs_chunks(int n, int cols)
{
    const int cus = device_cus();
    int best = 1;
    long best_cost = -1;
    for (int c = 1; c <= std::max(1, (n - 1) / 16); ++c) {
        const int zc = zs_chunk(n, c);
        const int t = (n - 1 + zc - 1) / zc;
        const long rounds = (long(cols) * t + cus - 1) / cus;
        const long cost = rounds * (zc + 10);
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best = t;
        }
    }
    return best;
}
constexpr int kNumCfg = int(sizeof(kCfg) / sizeof(kCfg[0]));

// Automatic z-stream shape of an n grid: 32 x 26 or the one-colour-per-
// wavefront 32 x 24, whichever the chunk model (rounds x (planes + 10) step
// times, the 32 x 24 step counted 2% shorter) gives the shorter sweep.  At
// n = 256 the 88 columns of 32 x 24 make three chunks one workgroup too
// many per compute unit, where the 80 of 32 x 26 fit.
int zs_model_cost100(int n, int cfg)
{
    const BCfg &b = kCfg[cfg];
    const int cols = ((n - 1 + b.tx - 1) / b.tx) * ((n - 1 + b.ty - 1) / b.ty);
    const int zc = zs_chunk(n, zs_chunks(n, cols));
    const long t = (n - 1 + zc - 1) / zc;
    const long rounds = (long(cols) * t + device_cus() - 1) / device_cus();
    return int(rounds * (zc + 10) * (cfg == kZsPureConfig ? 98 : 100));
}

template <int OP, int TX, int TY, int NT>
hipError_t zgo_list(hipStream_t st, const FsList *L, int blocks, unsigned long long *nc, bool pro)
{
    if (pro)
        hipLaunchKernelGGL((k_zsweep<OP, TX, TY, NT, true>), dim3(blocks), dim3(NT), 0, st, L, nc);
    else
        hipLaunchKernelGGL((k_zsweep<OP, TX, TY, NT, false>), dim3(blocks), dim3(NT), 0, st, L, nc);
    return hipGetLastError();
}

template <int OP, int TX, int TY, int NT>
hipError_t zgo_one(hipStream_t st, const FsGrid &G, unsigned long long *nc)
{
    const int blocks = G.tiles_x * G.tiles_y * G.tiles_z;
    hipLaunchKernelGGL((k_zsweep1<OP, TX, TY, NT>), dim3(blocks), dim3(NT), 0, st, G, nc);
    return hipGetLastError();
}

template <int OP, int TX, int TY, int TZ, int NT, int ORDER = 0, int PH = ORDER == 0 ? 4 : 8,
          int GRP = 0>
hipError_t go_list(hipStream_t st, const FsList *L, int blocks, unsigned long long *nc)
{
    hipLaunchKernelGGL((k_bsweep<OP, ORDER, PH, GRP, TX, TY, TZ, NT>), dim3(blocks), dim3(NT), 0, st,
                       L, nc);
    return hipGetLastError();
}

template <int OP, int TX, int TY, int TZ, int NT, int ORDER = 0, int PH = ORDER == 0 ? 4 : 8,
          int GRP = 0>
hipError_t go_one(hipStream_t st, const FsGrid &G, unsigned long long *nc)
{
    const int blocks = G.tiles_x * G.tiles_y * G.tiles_z;
    hipLaunchKernelGGL((k_bsweep1<OP, ORDER, PH, GRP, TX, TY, TZ, NT>), dim3(blocks), dim3(NT), 0,
                       st, G, nc);
    return hipGetLastError();
}

template <int OP>
hipError_t list_op8(int cfg, hipStream_t st, const FsList *L, int blocks, unsigned long long *nc)
{
    switch (cfg) {
    case 0:
        return go_list<OP, 8, 8, 4, 256, 1>(st, L, blocks, nc);
    case 1:
        return go_list<OP, 8, 8, 8, 320, 1>(st, L, blocks, nc);
    case 2:
        return go_list<OP, 16, 8, 8, 512, 1>(st, L, blocks, nc);
    case kGroupConfig8:
        return go_list<OP, 32, 8, 8, 512, 1, 4, 0>(st, L, blocks, nc);
    case kGroupConfig8 + 1:
        return go_list<OP, 32, 8, 8, 512, 1, 4, 1>(st, L, blocks, nc);
    default:
        return hipErrorInvalidValue;
    }
}

template <int OP>
hipError_t one_op8(int cfg, hipStream_t st, const FsGrid &G, unsigned long long *nc)
{
    switch (cfg) {
    case 0:
        return go_one<OP, 8, 8, 4, 256, 1>(st, G, nc);
    case 1:
        return go_one<OP, 8, 8, 8, 320, 1>(st, G, nc);
    case 2:
        return go_one<OP, 16, 8, 8, 512, 1>(st, G, nc);
    case kGroupConfig8:
        return go_one<OP, 32, 8, 8, 512, 1, 4, 0>(st, G, nc);
    case kGroupConfig8 + 1:
        return go_one<OP, 32, 8, 8, 512, 1, 4, 1>(st, G, nc);
    default:
        return hipErrorInvalidValue;
    }
}

// Blocks of the Gauss-Seidel iteration: small ones while they give few
// workgroups.
const BCfg &gs_shape(int order, int n)
{
    if (order == 0)
        return n <= 40 ? kCfg[5] : kCfg[0];
    return n <= 40 ? kCfg8[0] : kCfg8[1];
}

template <int OP>
hipError_t list_op(int cfg, hipStream_t st, const FsList *L, int blocks, unsigned long long *nc,
                   bool pro)
{
    // only the z-stream shapes prolong
    if (pro && kCfg[cfg].zwg == 0)
        return hipErrorInvalidValue;
    switch (cfg) {
    case 0:
        return go_list<OP, 8, 8, 8, 256>(st, L, blocks, nc);
    case 1:
        return go_list<OP, 8, 8, 8, 512>(st, L, blocks, nc);
    case 2:
        return go_list<OP, 8, 8, 8, 1024>(st, L, blocks, nc);
    case 3:
        return go_list<OP, 16, 8, 4, 256>(st, L, blocks, nc);
    case 4:
        return go_list<OP, 16, 16, 8, 512>(st, L, blocks, nc);
    case 5:
        return go_list<OP, 8, 8, 4, 512>(st, L, blocks, nc);
    case 6:
        return go_list<OP, 8, 8, 4, 256>(st, L, blocks, nc);
    case 7:
    case 9:
        return zgo_list<OP, 32, 26, 1024>(st, L, blocks, nc, pro);
    case 8:
        return zgo_list<OP, 32, 26, 512>(st, L, blocks, nc, pro);
    case 10:
        return zgo_list<OP, 40, 20, 1024>(st, L, blocks, nc, pro);
    case 11:
        return zgo_list<OP, 32, 24, 1024>(st, L, blocks, nc, pro);
    default:
        return hipErrorInvalidValue;
    }
}

template <int OP>
hipError_t one_op(int cfg, hipStream_t st, const FsGrid &G, unsigned long long *nc)
{
    switch (cfg) {
    case 0:
        return go_one<OP, 8, 8, 8, 256>(st, G, nc);
    case 1:
        return go_one<OP, 8, 8, 8, 512>(st, G, nc);
    case 2:
        return go_one<OP, 8, 8, 8, 1024>(st, G, nc);
    case 3:
        return go_one<OP, 16, 8, 4, 256>(st, G, nc);
    case 4:
        return go_one<OP, 16, 16, 8, 512>(st, G, nc);
    case 5:
        return go_one<OP, 8, 8, 4, 512>(st, G, nc);
    case 6:
        return go_one<OP, 8, 8, 4, 256>(st, G, nc);
    case 7:
    case 9:
        return zgo_one<OP, 32, 26, 1024>(st, G, nc);
    case 8:
        return zgo_one<OP, 32, 26, 512>(st, G, nc);
    case 10:
        return zgo_one<OP, 40, 20, 1024>(st, G, nc);
    case 11:
        return zgo_one<OP, 32, 24, 1024>(st, G, nc);
    default:
        return hipErrorInvalidValue;
    }
}

} // namespace

int bsweep_num_configs() { return kNumCfg; }

// Automatic shape: 8^3 blocks; the fewer blocks the grid has, the more
// threads each gets (one update per thread and phase at 1024 threads).  A
// launch whose 8^3 blocks (tiles8, over all its grids) would leave most
// compute units idle takes 8 x 8 x 4 blocks of 512 threads instead: twice
// the blocks, each with fewer rounds of updates per phase, for more halo
// recomputation (measured on the level-32 sweeps of one 129^3 solve: 1.7%
// of the solve faster).
int bsweep_pick(int order, int n, long tiles8)
{
    if (order == 1)
        return n >= kGroupN ? kGroupConfig8 : n <= 32 && tiles8 < 256 ? 0 : n <= 64 ? 1 : 2;
    if (n <= 16)
        return 2;
    if (n <= 32)
        return tiles8 < 256 ? 5 : 1;
    // 512 threads while the blocks do not fill the chip twice: n = 64, us: 12.2
    // with 256, 11.0 with 512; 128: 54 / 53
    if (n <= 64)
        return tiles8 < 1024 ? 1 : 0;
    return 4;
}

// Automatic z-stream shape (config index) of an n grid: the cheaper of
// 32 x 26 and 32 x 24 by the chunk model.
int bsweep_zs_pick(int n)
{
    return zs_model_cost100(n, kZsPureConfig) <= zs_model_cost100(n, 7) ? kZsPureConfig : 7;
}

bool bsweep_zs_alone(int n)
{
    const double step = 0.0142, cost = std::min(zs_model_cost100(n, kZsPureConfig), zs_model_cost100(n, 7));
    return n > 256 || step * cost <= 8.5e-6 * n * n * n;
}

void bsweep_grid(int order, int cfg, int n, const double *uin, double *uout, const double *F,
                 int op, int slot, FsGrid *G)
{
    const BCfg &b = shape_of(order, cfg);
    G->uin = uin;
    G->uout = uout;
    G->F = F;
    G->n = n;
    G->tiles_x = (n - 1 + b.tx - 1) / b.tx;
    G->tiles_y = (n - 1 + b.ty - 1) / b.ty;
    if (b.zwg != 0) {
        // chunks of at least 16 planes; the last chunk takes what remains
        const int cols = G->tiles_x * G->tiles_y;
        const int chunks = b.zwg < 0 ? zs_chunks(n, cols)
                                     : std::max(1, std::min((n - 1) / 16,
                                                            (b.zwg + cols - 1) / cols));
        const int zc = zs_chunk(n, chunks);
        G->tiles_z = (n - 1 + zc - 1) / zc;
    } else {
        G->tiles_z = (n - 1 + b.tz - 1) / b.tz;
    }
    G->start = 0;
    G->slot = slot;
    G->s = double(n) * double(n);
    G->s4 = 0.25 * G->s;
    G->hk = op == OP_MA ? 0.5 / G->s : 1.0 / (6.0 * G->s);
    G->cu = G->cw = nullptr;
}

bool bsweep_is_zstream(int order, int cfg)
{
    return order == 0 && cfg >= 0 && cfg < kNumCfg && kCfg[cfg].zwg != 0;
}

hipError_t launch_bsweep(hipStream_t st, int op, int order, int cfg, const FsList *L, int blocks,
                         unsigned long long *nonconvex, bool prolong)
{
    if (cfg < 0 || cfg >= (order == 0 ? kNumCfg : kNumCfg8) || blocks <= 0)
        return hipErrorInvalidValue;
    if (order == 1) {
        if (prolong)
            return hipErrorInvalidValue;
        return op == OP_MA ? list_op8<OP_MA>(cfg, st, L, blocks, nonconvex)
                           : list_op8<OP_LAP>(cfg, st, L, blocks, nonconvex);
    }
    if (op == OP_MA)
        return list_op<OP_MA>(cfg, st, L, blocks, nonconvex, prolong);
    return list_op<OP_LAP>(cfg, st, L, blocks, nonconvex, prolong);
}

hipError_t launch_bsweep_one(hipStream_t st, int op, int order, int cfg, int n,
                             const double *u_in, double *u_out, const double *F,
                             unsigned long long *nonconvex)
{
    if (n < 2)
        return hipErrorInvalidValue;
    if (cfg < 0 || cfg >= (order == 0 ? kNumCfg : kNumCfg8)) {
        cfg = bsweep_pick(order, n, long((n - 1 + 7) / 8) * ((n - 1 + 7) / 8) * ((n - 1 + 7) / 8));
        if (order == 1 && cfg == kGroupConfig8)   // half a sweep: only by name
            cfg = kGroupConfig8 - 1;
    }
    FsGrid G;
    bsweep_grid(order, cfg, n, u_in, u_out, F, op, 0, &G);
    if (order == 1)
        return op == OP_MA ? one_op8<OP_MA>(cfg, st, G, nonconvex)
                           : one_op8<OP_LAP>(cfg, st, G, nonconvex);
    if (op == OP_MA)
        return one_op<OP_MA>(cfg, st, G, nonconvex);
    return one_op<OP_LAP>(cfg, st, G, nonconvex);
}

int gs_blocks(int order, int n)
{
    const BCfg &b = gs_shape(order, n);
    return ((n - 1 + b.tx - 1) / b.tx) * ((n - 1 + b.ty - 1) / b.ty) * ((n - 1 + b.tz - 1) / b.tz);
}

hipError_t launch_gs_step(hipStream_t st, int order, int n, const double *u_in, double *u_out,
                          const double *F, const double *part_in, double *part_out, double *sum,
                          unsigned long long *count, int *stop, int q, double thr)
{
    const BCfg &b = gs_shape(order, n);
    FsGrid G;
    GsStep A;
    bsweep_grid(order, order == 0 ? int(&b - kCfg) : int(&b - kCfg8), n, u_in, u_out, F, OP_MA, 0,
                &G);
    A.part_in = part_in;
    A.part_out = part_out;
    A.sum = sum;
    A.count = count;
    A.stop = stop;
    A.q = q;
    A.thr = thr;
    const dim3 grid(gs_blocks(order, n)), block(b.nt);
    if (&b == &kCfg[5])
        hipLaunchKernelGGL((k_gs_step<0, 8, 8, 4, 512>), grid, block, 0, st, G, A);
    else if (&b == &kCfg[0])
        hipLaunchKernelGGL((k_gs_step<0, 8, 8, 8, 256>), grid, block, 0, st, G, A);
    else if (&b == &kCfg8[0])
        hipLaunchKernelGGL((k_gs_step<1, 8, 8, 4, 256>), grid, block, 0, st, G, A);
    else
        hipLaunchKernelGGL((k_gs_step<1, 8, 8, 8, 320>), grid, block, 0, st, G, A);
    return hipGetLastError();
}

} // namespace mafas
