// lbmp_abi.cpp -- host runtime behind the C ABI of include/lbmp.h.
//
// Responsibilities: parameter validation (pure host), FP64 derivation of the
// FP32 kernel constants, carving of the caller-owned workspace, graph capture
// and replay of step loops, error state.  Every numerical step of the method
// runs in the kernels of d2q9_kernels.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/lbmp.h"
#include "d2q9_launch.hpp"

namespace {

thread_local std::string g_last_error;

lb_status fail(lb_status st, const std::string& msg)
{
    g_last_error = msg;
    return st;
}

lb_status hip_fail(hipError_t e, const char* what)
{
    return fail(LB_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

// Host memory ran out inside an entry point that keeps tables (a short message: storing it
// must not allocate).
lb_status no_memory() { return fail(LB_ENOMEM, "out of memory"); }

constexpr size_t kAlign = 256;
constexpr int kMinStripRows = 3;
constexpr int kBatchPersistentRows = 24;  // measured best (one workgroup walks a whole lattice)
constexpr int kDefaultBand = 1;
constexpr size_t kLastLevelCache = (size_t)256 << 20;
constexpr int kDefaultGraphChunk = 32;
constexpr int kMaxSide = 1 << 20;

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

size_t elem_bytes(int store) { return store == LB_STORE_F32 ? 4 : 2; }

bool local_density(int store) { return store == LB_STORE_F16_LOCAL || store == LB_STORE_BF16_LOCAL; }

// storage-type row slots per lattice row: nine population rows, plus an FP32
// density row (two 16-bit slots) for the local-density encodings, or a bf16
// density-scale row (one slot) for the destination-scaled encoding
int row_slots(int store)
{
    if (local_density(store)) return 11;
    return store == LB_STORE_F16_DEST ? 10 : 9;
}

// bytes per site of the exported density plane (0: none)
size_t density_plane_bytes(int store)
{
    if (local_density(store)) return sizeof(float);
    return store == LB_STORE_F16_DEST ? 2 : 0;
}

// Elements per population row.  The rows are packed without padding: the nine (ten,
// eleven) population rows of a lattice row, and consecutive lattice rows, then form one
// contiguous stream.  Measured on the 512-lattice sweep (sides 64-512): FP32 73.3k
// MLUPS with rows packed against 63.4k with rows padded to 64 elements, whose holes
// break the stream (destination-scaled FP16: 96.9k against 88.9k).  The local-density
// encodings round to an even count so that their FP32 density row stays 4-byte aligned.
int pitch_of(int nx, int store) { return local_density(store) ? (nx + 1) / 2 * 2 : nx; }

// Whether lb_step advances this lattice two steps per launch (an odd last step is a single
// one).  FP32 with the nearest-neighbour stencil, at every size: 8192 x 4096 428 -> 248 us
// per step, 2048 x 1024 28 -> 16 us, 600 x 250 7.2 -> 5.3 us, 128 x 128 7.6 -> 4.2 us.  The
// walk pulls up to four rows beyond a strip and wraps a row or column index once, hence the
// least size.
bool two_step(const lb_params& p)
{
    return p.store == LB_STORE_F32 && p.stencil == LB_STENCIL_NEAREST && p.nx >= 8 && p.ny >= 8;
}

// Output columns per wavefront strip of the one-column kernels for this stencil.
int tile_width(const lb_params& p) { return p.stencil == LB_STENCIL_MULTIRANGE ? lbmp::kMrTileW : lbmp::kTileW; }

// Strip height of the diagnostics and moments passes, a function of the lattice alone (the
// diagnostics' sums are reduced strip by strip): about 4000 strips where the lattice has
// them, since a short walk is short in time (128 x 128: diagnostics 48 us at 32 rows, 7.3 us
// at 4; moments of 200 x 200 30 us and 5 us), and not more than that, since one workgroup
// sums up the strips.
int pass_rows(const lb_params& p)
{
    const int tx = (p.nx + tile_width(p) - 1) / tile_width(p);
    return (int)std::min<long long>(32, std::max<long long>(4, (long long)tx * p.ny / 4096));
}

struct Layout {
    size_t flag_off, dout_off, partial_off, f_off[2], total, buf_bytes;
    int diag_tiles;
};

Layout layout_of(const lb_params& p)
{
    Layout L{};
    const int pitch = pitch_of(p.nx, p.store);
    L.buf_bytes = align_up((size_t)row_slots(p.store) * p.ny * pitch * elem_bytes(p.store), kAlign);
    const int tw = tile_width(p);
    const int tx = (p.nx + tw - 1) / tw;
    const int rows = pass_rows(p);
    const int ty = (p.ny + rows - 1) / rows;
    L.diag_tiles = tx * ty;
    L.flag_off = 0;
    L.dout_off = kAlign;
    L.partial_off = 2 * kAlign;
    size_t off = align_up(L.partial_off + (size_t)L.diag_tiles * lbmp::kDiagFields * sizeof(double), kAlign);
    L.f_off[0] = off;
    L.f_off[1] = off + L.buf_bytes;
    L.total = off + 2 * L.buf_bytes;
    return L;
}

bool finite_all(std::initializer_list<double> v)
{
    for (double x : v)
        if (!std::isfinite(x)) return false;
    return true;
}

bool rate_ok(double s) { return s > 0.0 && s < 2.0; }

lb_status validate(const lb_params* p)
{
    if (!p) return fail(LB_EINVAL, "params is NULL");
    if (p->nx < 3 || p->ny < 3 || p->nx > kMaxSide || p->ny > kMaxSide)
        return fail(LB_EINVAL, "nx and ny must lie in [3, 2^20]");
    if ((long long)p->nx * p->ny > (1LL << 31)) return fail(LB_EINVAL, "nx * ny exceeds 2^31 sites");
    if ((long long)pitch_of(p->nx, p->store) * row_slots(p->store) * (p->store == LB_STORE_F32 ? 4 : 2) >= (1LL << 32))
        return fail(LB_EINVAL, "a lattice row must stay below 4 GiB");
    if (p->bc != LB_BC_PERIODIC && p->bc != LB_BC_WALLS_Y) return fail(LB_EINVAL, "unknown bc");
    if (p->stencil != LB_STENCIL_NEAREST && p->stencil != LB_STENCIL_MULTIRANGE)
        return fail(LB_EINVAL, "unknown stencil");
    if (p->stencil == LB_STENCIL_MULTIRANGE && p->store != LB_STORE_F32)
        return fail(LB_EINVAL, "the 24-site stencil runs with LB_STORE_F32 only");
    if (p->store < LB_STORE_F32 || p->store > LB_STORE_F16_DEST) return fail(LB_EINVAL, "unknown store");
    if (!finite_all({p->a, p->b, p->R, p->T, p->G, p->sigma, p->s_rho, p->s_e, p->s_zeta, p->s_j,
                     p->s_q, p->nu_l, p->nu_g, p->rho_switch, p->rho_ref, p->psi_eps}))
        return fail(LB_EINVAL, "non-finite parameter");
    if (p->psi_form == LB_PSI_CS) {
        if (!(p->b > 0.0) || !(p->T > 0.0) || !(p->R > 0.0) || !(p->a >= 0.0))
            return fail(LB_EINVAL, "need a >= 0, b > 0, R > 0, T > 0");
    } else if (p->psi_form == LB_PSI_SS) {
        if (!(p->psi_eps >= 0.0)) return fail(LB_EINVAL, "need psi_eps >= 0 (Eq. 23)");
    } else {
        return fail(LB_EINVAL, "unknown psi_form");
    }
    if (!(p->G < 0.0)) return fail(LB_EINVAL, "need G < 0 (Eq. 24 radicand)");
    if (!(p->sigma >= 0.0)) return fail(LB_EINVAL, "need sigma >= 0");
    if (!rate_ok(p->s_rho) || !rate_ok(p->s_e) || !rate_ok(p->s_zeta) || !rate_ok(p->s_j) ||
        !rate_ok(p->s_q))
        return fail(LB_EINVAL, "relaxation rates must lie in (0, 2)");
    if (!(p->nu_l > 0.0) || !(p->nu_g > 0.0)) return fail(LB_EINVAL, "viscosities must be > 0");
    if (!(p->rho_switch >= 0.0)) return fail(LB_EINVAL, "rho_switch must be >= 0");
    if ((p->store == LB_STORE_F16_OFFSET || p->store == LB_STORE_BF16_OFFSET) && !(p->rho_ref >= 0.0))
        return fail(LB_EINVAL, "rho_ref must be >= 0");
    return LB_OK;
}

lbmp::PsiConst psi_const(const lb_params& p)
{
    return lbmp::PsiConst{p.b / 4.0, p.R * p.T, p.a, p.G, p.psi_eps, p.psi_form};
}

lbmp::StepConst derive(const lb_params& p, int strip_rows, int band = 1)
{
    lbmp::StepConst k{};
    k.nx = p.nx;
    k.ny = p.ny;
    k.pitch = pitch_of(p.nx, p.store);
    k.strip_rows = strip_rows;
    k.band = band;
    k.tiles_x = (p.nx + tile_width(p) - 1) / tile_width(p);
    k.tiles_y = (p.ny + strip_rows - 1) / strip_rows;
    k.row_stride = (long long)row_slots(p.store) * k.pitch;
    k.b4 = (float)(p.b / 4.0);
    k.RT = (float)(p.R * p.T);
    k.a = (float)p.a;
    k.two_over_G = (float)(2.0 / p.G);
    k.negG = (float)(-p.G);
    k.rho_switch = (float)p.rho_switch;
    k.a_e = (float)(p.s_e / 36.0);
    k.b_e = (float)(6.0 * (1.0 - 0.5 * p.s_e) / 36.0);
    k.a_z = (float)(p.s_zeta / 36.0);
    k.b_z = (float)(6.0 * (1.0 - 0.5 * p.s_zeta) / 36.0);
    k.a_q = (float)(p.s_q / 12.0);
    k.b_q = (float)((1.0 - 0.5 * p.s_q) / 12.0);
    const double s_nu_l = 1.0 / (3.0 * p.nu_l + 0.5), s_nu_g = 1.0 / (3.0 * p.nu_g + 0.5);
    k.a_nu_l = (float)(s_nu_l / 4.0);
    k.b_nu_l = (float)((1.0 - 0.5 * s_nu_l) / 2.0);
    k.a_nu_g = (float)(s_nu_g / 4.0);
    k.b_nu_g = (float)((1.0 - 0.5 * s_nu_g) / 2.0);
    const double G2 = p.G * p.G;
    k.c_e = (float)(12.0 * p.sigma * G2 * p.s_e / 36.0);
    k.c_z = (float)(12.0 * p.sigma * G2 * p.s_zeta / 36.0);
    k.psi_form = p.psi_form;
    k.stencil = p.stencil;
    k.psi_eps = (float)p.psi_eps;
    k.inv_psi_eps = p.psi_eps > 0.0 ? (float)(1.0 / p.psi_eps) : 0.0f;
    static const double w[9] = {4.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9,
                                1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};
    const bool global16 = p.store == LB_STORE_F16_OFFSET || p.store == LB_STORE_BF16_OFFSET;
    for (int a = 0; a < 9; ++a) k.off[a] = global16 ? (float)(w[a] * p.rho_ref) : 0.0f;
    return k;
}

// Constants of the single-step launches of one lattice.  The waves of their workgroups are
// paced (pace) and every other launch runs in descending order (launch_block; back = 1 here, the
// launch sets it) where the two buffers exceed the last-level cache; FP32 lattices run in that
// order up to 512 MiB a state only (one direction and alternating: 2048^2 62.0 and 59.0 us, 4096 x
// 2048 122.7 and 117.6 us, 4096^2 227.7 and 227.1 us, 8192 x 4096 427 and 448 us).  Batches do
// neither: their persistent launch gives the waves of a workgroup different numbers of strips.
lbmp::StepConst derive_single(const lb_params& p, int strip_rows, int band)
{
    lbmp::StepConst k = derive(p, strip_rows, band);
    const size_t bytes = layout_of(p).buf_bytes;
    k.paced = 2 * bytes > kLastLevelCache;
    k.back = k.paced && (p.store != LB_STORE_F32 || bytes <= 2 * kLastLevelCache);
    return k;
}

// Constants of a launch of two steps: 58-column tiles.
lbmp::StepConst derive_two(const lb_params& p, int strip_rows, int band = 1)
{
    lbmp::StepConst k = derive(p, strip_rows, band);
    k.tiles_x = (p.nx + lbmp::kTwoTileW - 1) / lbmp::kTwoTileW;
    return k;
}

int compute_units()
{
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu <= 0)
        return 256;
    return ncu;
}

// Wavefronts per workgroup of the two-step launches: 8 pace a wider stretch of a row
// (8192 x 4096: 250 us per step against 256 us with 4), 4 fill the chip more evenly when
// there are few strips per compute unit (2048 x 1024: 16.0 us against 16.5 us at the best
// height of each, 18.2 us against 21.6 us at 16 rows).
int two_waves(const lb_params& p, int rows)
{
    const lbmp::StepConst k = derive_two(p, rows);
    return (long long)k.tiles_x * k.tiles_y >= 16LL * 4 * compute_units() ? lbmp::kTwoWavesWide : lbmp::kTwoWaves;
}

// Time of a two-step launch of `strips` strips of h rows in workgroups of `waves`, in us per
// step: a strip costs about h + 5 rows of work, and a SIMD that holds w of them (at most four
// at once) needs about 0.36 + 0.17 w per row.  Fitted on 2048 x 1024 at heights 4-24: 16.0 us
// per step at 10 rows, where every strip is resident at once, 18.2 us at 8 rows, 19.9 us at
// 4 rows, 20.5 us at 24 rows.  It holds for batches, whose strips are one list: 40 lattices of
// 200 x 200 at 6 / 8 / 12 / 16 rows 18.1 / 14.2 / 17.7 / 21.3 us (19.1 / 13.5 / 17.7 / 21.8 by
// this).
double two_cost(int h, long long strips, int waves, int ncu)
{
    const long long groups = (strips + waves - 1) / waves;
    const double load = (double)((groups + ncu - 1) / ncu) * (waves / 4.0);
    return (h + 5) * (0.36 * std::ceil(load / 4.0) + 0.17 * load);
}

// Strip height of the two-step launches: the cheapest.  On large lattices the cost falls
// slowly with h and the stride of the resident strips decides: 8192 x 4096 at 8 / 12 / 16 /
// 22 / 36 rows 255 / 248 / 247 / 248 / 268 us.  On small ones the walk itself is the time:
// 128 x 128 at 2 / 3 / 4 / 8 rows 4.1 / 4.9 / 5.2 / 7.8 us.
int auto_two_rows(const lb_params& p)
{
    const int ncu = compute_units();
    int best = 2;
    double least = 1e300;
    for (int h = 2; h <= 18 && h <= p.ny; ++h) {
        const lbmp::StepConst k = derive_two(p, h);
        const double cost = two_cost(h, (long long)k.tiles_x * k.tiles_y, lbmp::kTwoWaves, ncu);
        if (cost < least) {
            least = cost;
            best = h;
        }
    }
    return best;
}

// Wavefronts per workgroup of the step kernel of this lattice, and its workgroups resident at
// once.
int strip_waves(const lb_params& p)
{
    return lbmp::pair_step(p.store, p.nx) ? lbmp::kPairWaves : lbmp::step_waves_per_block(p.store);
}

long long resident_groups(const lb_params& p)
{
    const bool walls = p.bc == LB_BC_WALLS_Y;
    const int nb = lbmp::pair_step(p.store, p.nx) ? lbmp::pair_blocks_per_cu(walls) : lbmp::step_blocks_per_cu(p.store, walls);
    return (long long)std::max(1, nb) * compute_units();
}

// Strip height for the step kernel.  Short strips are fastest on large grids
// even though they re-read two halo rows per strip: the tiles are numbered
// row-band by row-band, so the resident wavefronts work on a narrow band of
// rows at any moment (good DRAM-page and last-level-cache locality, halo rows
// shared by neighbouring strips while they are still cached).  Grids too small
// to give every resident wavefront a strip of kMinStripRows rows use shorter
// strips, down to 2 rows.
int auto_strip_rows(const lb_params& p)
{
    // preferred height (measured on the 8192 x 4096 splash): 3 rows for FP32;
    // the issue-bound 16-bit encodings gain from fewer recomputed halo rows:
    // 4 rows for the source-density ones, 8 for the global offsets and the
    // destination-scaled one with one column per lane, 5 for the latter with two
    const bool pair = lbmp::pair_step(p.store, p.nx);
    int preferred = kMinStripRows;
    if (p.stencil == LB_STENCIL_MULTIRANGE)
        preferred = 8;  // two halo rows a side: taller strips pull fewer extra rows
    else if (pair)
        preferred = 5;
    else if (p.store == LB_STORE_F16_DEST || p.store == LB_STORE_F16_OFFSET || p.store == LB_STORE_BF16_OFFSET)
        preferred = 8;
    else if (p.store == LB_STORE_F16_LOCAL || p.store == LB_STORE_BF16_LOCAL)
        preferred = 4;
    const long long resident = resident_groups(p) * strip_waves(p);
    const int tile_w = pair ? lbmp::kPairTileW : lbmp::kTileW;
    const long long tiles_x = (p.nx + tile_w - 1) / tile_w;
    const long long strips_wanted = (resident + tiles_x - 1) / tiles_x;
    const long long h = std::max<long long>(2, p.ny / strips_wanted);
    return (int)std::min<long long>(h, preferred);
}

// Regions of `steps` steps per compute unit.
double region_load(const lb_params& p, int steps, int ncu)
{
    const long long out = lbmp::region_out(p.stencil, steps);
    return (double)(((p.nx + out - 1) / out) * ((p.ny + out - 1) / out)) / ncu;
}

// Steps per launch by regions (d2q9_region), 0: the lattice is stepped by strips.
//
// Regions win as long as the overlap is computed by units that strips leave idle or waiting.
// Measured, us per step, strips against regions (droplet, CS):
//   FP32       128^2 4.07 / 2.03, 400 x 300 5.07 / 4.35, 512^2 6.45 / 5.79, 768 x 512 6.55 / 7.53
//   FP16 dest  256^2 5.00 / 2.78, 600 x 250 5.91 / 5.05, 640 x 400 6.84 / 6.73, 641 x 640 7.57 / 8.79
//   FP16       256^2 6.19 / 2.57, 1021 x 509 10.75 / 7.82, 2048 x 1024 25.7 / 21.8, 4096 x 1024 37.4 / 40.4
//   FP16 local 200^2 7.37 / 2.59, 1021 x 509 14.27 / 8.65, 2048 x 1024 30.6 / 25.0, 2048 x 1400 31.4 / 31.9
//   24 sites   200^2 7.66 / 3.14, 1021 x 509 14.82 / 11.05, 2048^2 79.3 / 64.0, 8192 x 4096 560 / 496
// (768 x 512 and the like against FP32 strips of two steps per launch).  These are limits only:
// at a given number of sites the strips' time depends on how their workgroups divide among
// the units and the regions' on how many rows and columns of them lie outside the lattice, so
// below the limits region_pays compares the two.
//
// A launch of n regions of `steps` steps takes about 4 + 1.1 steps + l (2.5 + 0.2 steps) us,
// l = n / units - 0.6 where positive (fitted to the sizes above and 20 others for every
// number of steps; the choice is within 9 % of the best one, on average 1 %).
int region_steps(const lb_params& p)
{
    const long long sites = (long long)p.nx * p.ny;
    if ((long long)row_slots(p.store) * pitch_of(p.nx, p.store) * p.ny * 4 >= (1LL << 31)) return 0;
    const int ncu = compute_units();
    long long most = 0;  // sites per compute unit
    if (p.stencil == LB_STENCIL_MULTIRANGE) most = sites;
    else if (p.store == LB_STORE_F32) most = 1200;
    else if (p.store == LB_STORE_F16_DEST) most = 800;
    else if (p.store == LB_STORE_F16_OFFSET || p.store == LB_STORE_BF16_OFFSET) most = 9000;
    else most = 10000;
    if (sites > most * ncu) return 0;
    int best = 0;
    double least = 1e300;
    for (int steps = 1; lbmp::region_out(p.stencil, steps) > 0; ++steps) {
        const double load = region_load(p, steps, ncu);
        const double cost = (4.0 + 1.1 * steps + std::max(0.0, load - 0.6) * (2.5 + 0.2 * steps)) / steps;
        if (cost < least) {
            least = cost;
            best = steps;
        }
    }
    return best;
}

// Times in us of a step by strips and of a launch of `steps` steps by regions:
//   strips   s0 + fill (workgroups per unit, at most as many as are resident and two) +
//            rounds (s1 + s2 rows), the workgroups taking turns in `rounds` of the resident ones;
//   regions  r0 + r1 steps + load (r2 + r3 steps) + r4 where some unit has two regions, for FP16
//            dest (whose registers with walls leave room for one region at a time) also for
//            each further one.
// Fitted on 250 lattices of each kind (3e3 to 4e6 sites, sides 8 to 125000, walls and
// periodic): strips within 8 % and rather too low, regions within 8 %, so that a launch by
// regions is a gain where these say so (of 3500 choices 20 lost more than 2 %, none more than
// 8 %; by the numbers of sites alone 360 did, up to 2.5 times).  Strips against regions, us per step:
// FP16 1984 x 1024 17.5 / 22.1, 992 x 2048 16.0 / 24.1 (one full round of strips), 2048 x 1024 25.7
// / 21.8 (two, the second nearly empty); FP32 37500 x 8 6.6 / 9.9, FP16 125000 x 8 14 / 31 (regions
// mostly off the lattice); 24 sites 1876 x 1823 48.8 / 53.9.  Single steps: FP16 local 525 x 505
// 8.3 / 11.1, 724^2 15.0 / 12.2; 24 sites 641 x 640 9.2 / 12.3, 724^2 16.1 / 13.8.
struct LaunchCost {
    double s0, fill, s1, s2, r0, r1, r2, r3, r4;
    double turns = 1.0;  // times r4 counts at most
};
LaunchCost launch_cost(const lb_params& p, bool pair)
{
    if (p.stencil == LB_STENCIL_MULTIRANGE) return {1.2, 1.2, 2.35, 2.2, 3.5, 1.1, 3.85, 0.0, 0.4};
    if (p.store == LB_STORE_F32) return {0.7, 1.0, 0.8, 2.25, 2.65, 1.07, 6.24, -0.31, 0.64};
    if (p.store == LB_STORE_F16_DEST) {
        LaunchCost c{1.0, 0.8, 3.15, 0.37, 2.58, 1.245, 6.27, -0.89, 5.7, 8.0};
        if (!pair) c.s0 = -0.95, c.s1 = 4.8, c.s2 = 0.2;
        if (p.bc == LB_BC_PERIODIC) c.r1 = 1.19, c.r2 = 6.32, c.r3 = -0.865, c.r4 = 3.47;
        return c;
    }
    if (p.store == LB_STORE_F16_OFFSET || p.store == LB_STORE_BF16_OFFSET)
        return {1.6, 1.2, 2.2, 1.3, 4.4, 0.67, 2.2, 0.55, 1.5};
    return {1.0, 1.2, 3.2, 1.7, 4.75, 0.8, 2.75, 0.45, 0.9};
}

// Whether a launch of `steps` steps by regions takes no longer than the same steps by strips
// (height `rows`, `resident` workgroups of `waves` strips at once).
bool region_pays(const lb_params& p, int steps, int rows, long long resident, int waves)
{
    const int ncu = compute_units();
    const bool pair = lbmp::pair_step(p.store, p.nx);
    // FP32 has strips of two steps per launch: regions win on every lattice below the limit
    // but the flattest (600 x 250 5.1 / 3.7, 4687 x 64 6.4 / 5.6, 9375 x 32 6.5 / 7.2)
    if (p.store == LB_STORE_F32 && p.stencil == LB_STENCIL_NEAREST && steps > 1)
        return p.ny >= 64 || (long long)p.nx * p.ny <= 600LL * ncu;
    // 24 sites, beyond the last-level cache: the strips slow down, the regions do not
    // (1160 x 3206, 255 MiB, 53.2 / 60.1; 1868 x 2040, 262 MiB, 68.7 / 60.9; 2048 x 2048 82 / 64)
    if (p.stencil == LB_STENCIL_MULTIRANGE && steps > 1 && 2 * layout_of(p).buf_bytes > kLastLevelCache) return true;
    const LaunchCost c = launch_cost(p, pair);
    const int tile = pair ? lbmp::kPairTileW : tile_width(p);
    const long long strips = (long long)((p.nx + tile - 1) / tile) * ((p.ny + rows - 1) / rows);
    const long long groups = (strips + waves - 1) / waves;
    double strip = c.s0 + c.fill * std::min(std::min(2.0, (double)resident / ncu), (double)groups / ncu) +
                   (double)((groups + resident - 1) / resident) * (c.s1 + c.s2 * rows);
    // strips with walls take about 7 % longer (periodic and walls: FP16 916 x 517 7.5 and 8.2 us,
    // FP16 local 1021 x 509 14.3 and 15.0, 24 sites 15.0 and 16.1); for FP16 dest that is in the
    // constants, and a single step of source density or of 24 sites would lose by it (FP16 local
    // 151 x 1000 8.1 by strips, 9.0 by regions)
    const bool closest = steps == 1 && p.store != LB_STORE_F16_OFFSET && p.store != LB_STORE_BF16_OFFSET &&
                         (p.store != LB_STORE_F32 || p.stencil == LB_STENCIL_MULTIRANGE);
    if (p.bc == LB_BC_WALLS_Y && p.store != LB_STORE_F16_DEST && !closest) strip *= 1.07;
    const double load = region_load(p, steps, ncu);
    const double region = c.r0 + c.r1 * steps + load * (c.r2 + c.r3 * steps) + c.r4 * std::min(c.turns, std::ceil(load) - 1.0);
    return region * (steps == 1 ? 1.06 : 1.0) <= steps * strip;  // single steps are the closest
}

// The numbers of steps (bits 1 and up) that the lattice takes by regions in one launch.
unsigned region_mask(const lb_params& p, int most)
{
    if (most <= 0) return 0;
    const int rows = auto_strip_rows(p);
    const long long resident = resident_groups(p);
    unsigned mask = 0;
    for (int steps = 1; steps <= most; ++steps)
        if (region_pays(p, steps, rows, resident, strip_waves(p))) mask |= 1u << steps;
    return mask;
}

}  // namespace

namespace lbmp {
// Error reporting shared with the learned-initialiser entry points (the same
// thread-local message is behind lb_last_error()).
lb_status abi_fail(lb_status st, const std::string& msg) { return fail(st, msg); }
lb_status abi_hip_fail(hipError_t e, const char* what) { return hip_fail(e, what); }
}  // namespace lbmp

struct lb_ctx {
    lb_params p;
    Layout L;
    lbmp::StepConst k;   // step launches
    lbmp::StepConst k2;  // launches of two steps (two == true)
    int waves2;          // wavefronts per workgroup of those launches
    bool two;
    int region_steps;      // > 0: advanced by regions, up to that many steps per launch
    unsigned region_mask;  // bit n: a launch that takes n steps is by regions, else these are by strips
    lbmp::StepConst kd;  // moments / diagnostics launches
    char* ws;
    void* f[2];
    int* flag;
    double* dout;
    double* partial;
    int cur;
    int64_t t;
    hipStream_t stream;
    int graph_chunk;
    hipGraph_t graph[2];
    hipGraphExec_t exec[2];
    int graph_end[2];    // buffer that holds the state after the graph captured from each buffer
    bool poisoned;
};

namespace {

// Regions as the rules say; none where no launch would be by regions at the full number of
// steps.
void set_regions(lb_ctx* c)
{
    c->region_steps = region_steps(c->p);
    c->region_mask = region_mask(c->p, c->region_steps);
    if (!(c->region_mask >> c->region_steps & 1)) c->region_steps = 0;
}

void drop_graphs(lb_ctx* c)
{
    for (int i = 0; i < 2; ++i) {
        if (c->exec[i]) (void)hipGraphExecDestroy(c->exec[i]);
        if (c->graph[i]) (void)hipGraphDestroy(c->graph[i]);
        c->exec[i] = nullptr;
        c->graph[i] = nullptr;
    }
}

// One launch from buffer `cur` into the other one: by regions (the steps left spread evenly
// over as few launches as they take) where that number of steps pays, else two steps where
// the lattice is stepped that way and `left` allows it, else one.  *steps receives the number
// of steps taken.
hipError_t launch_some(lb_ctx* c, int cur, int64_t left, int* steps)
{
    const bool walls = c->p.bc == LB_BC_WALLS_Y;
    if (c->region_steps > 0) {
        const int64_t launches = (left + c->region_steps - 1) / c->region_steps;
        *steps = (int)((left + launches - 1) / launches);
        if (c->region_mask >> *steps & 1)
            return lbmp::launch_region(c->p.store, walls, c->f[cur], c->f[cur ^ 1], c->k, *steps, c->flag, c->stream);
        left = *steps;
    }
    *steps = c->two && left >= 2 ? 2 : 1;
    if (*steps == 2) return lbmp::launch_two(walls, c->f[cur], c->f[cur ^ 1], c->k2, c->waves2, c->flag, c->stream);
    lbmp::StepConst k = c->k;
    k.back = k.back ? cur : 0;
    return lbmp::launch_step(c->p.store, walls, c->f[cur], c->f[cur ^ 1], k, c->flag, c->stream);
}

lb_status step_direct(lb_ctx* c, int64_t n)
{
    while (n > 0) {
        int steps = 0;
        const hipError_t e = launch_some(c, c->cur, n, &steps);
        if (e != hipSuccess) {
            c->poisoned = true;
            return hip_fail(e, "step launch");
        }
        c->cur ^= 1;
        c->t += steps;
        n -= steps;
    }
    return LB_OK;
}

lb_status build_graph(lb_ctx* c, int from)
{
    hipError_t e = hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) return hip_fail(e, "hipStreamBeginCapture");
    int cur = from;
    hipError_t le = hipSuccess;
    for (int left = c->graph_chunk; left > 0 && le == hipSuccess;) {
        int steps = 0;
        le = launch_some(c, cur, left, &steps);
        left -= steps;
        cur ^= 1;
    }
    hipGraph_t g = nullptr;
    e = hipStreamEndCapture(c->stream, &g);
    if (le != hipSuccess) {
        if (g) (void)hipGraphDestroy(g);
        return hip_fail(le, "step launch during capture");
    }
    if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
    hipGraphExec_t x = nullptr;
    e = hipGraphInstantiate(&x, g, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        (void)hipGraphDestroy(g);
        return hip_fail(e, "hipGraphInstantiate");
    }
    c->graph[from] = g;
    c->exec[from] = x;
    c->graph_end[from] = cur;
    return LB_OK;
}

lb_status read_flag(lb_ctx* c, int* host_flag)
{
    hipError_t e = hipMemcpyAsync(host_flag, c->flag, sizeof(int), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) {
        c->poisoned = true;
        return hip_fail(e, "reading the device flag");
    }
    return LB_OK;
}

}  // namespace

extern "C" {

lb_status lb_validate_params(const lb_params* p) { return validate(p); }

size_t lb_workspace_bytes(const lb_params* p)
{
    if (validate(p) != LB_OK) return 0;
    return layout_of(*p).total;
}

size_t lb_state_bytes(const lb_params* p)
{
    if (validate(p) != LB_OK) return 0;
    return (size_t)9 * p->nx * p->ny * elem_bytes(p->store) + (size_t)p->nx * p->ny * density_plane_bytes(p->store);
}

}  // extern "C"

namespace {

// Create a context on `workspace` and launch the initial state; with
// sync == false the caller synchronises and checks the flag (batched init).
lb_status init_ctx(lb_ctx** out, const lb_params* p, void* workspace, size_t workspace_bytes,
                   const float* rho0, const float* ux0, const float* uy0, void* stream, bool sync)
{
    if (!out) return fail(LB_EINVAL, "out is NULL");
    *out = nullptr;
    lb_status st = validate(p);
    if (st != LB_OK) return st;
    if (!workspace || !rho0) return fail(LB_EINVAL, "workspace and rho0 must be non-NULL");
    if (reinterpret_cast<uintptr_t>(workspace) % kAlign) return fail(LB_EINVAL, "workspace must be 256-byte aligned");
    Layout L = layout_of(*p);
    if (workspace_bytes < L.total)
        return fail(LB_ENOMEM, "workspace smaller than lb_workspace_bytes");

    lb_ctx* c = new (std::nothrow) lb_ctx{};
    if (!c) return fail(LB_ENOMEM, "host allocation failed");
    c->p = *p;
    c->L = L;
    c->k = derive_single(*p, auto_strip_rows(*p), kDefaultBand);
    c->two = two_step(*p);
    c->k2 = derive_two(*p, auto_two_rows(*p), kDefaultBand);
    c->waves2 = two_waves(*p, c->k2.strip_rows);
    if (sync) set_regions(c);  // a batch steps its lattices itself, by strips
    c->kd = derive(*p, pass_rows(*p));
    c->ws = static_cast<char*>(workspace);
    c->flag = reinterpret_cast<int*>(c->ws + L.flag_off);
    c->dout = reinterpret_cast<double*>(c->ws + L.dout_off);
    c->partial = reinterpret_cast<double*>(c->ws + L.partial_off);
    c->f[0] = c->ws + L.f_off[0];
    c->f[1] = c->ws + L.f_off[1];
    c->stream = static_cast<hipStream_t>(stream);
    c->graph_chunk = kDefaultGraphChunk;

    hipError_t e = hipMemsetAsync(c->flag, 0, kAlign, c->stream);
    if (e == hipSuccess)
        e = lbmp::launch_init(p->store, p->bc == LB_BC_WALLS_Y, rho0, ux0, uy0, c->f[0], c->k,
                              lbmp::InitConst{psi_const(*p)}, c->flag, c->stream);
    if (e != hipSuccess) {
        delete c;
        return hip_fail(e, "init launch");
    }
    if (sync) {
        int hf = 0;
        st = read_flag(c, &hf);
        if (st != LB_OK) {
            delete c;
            return st;
        }
        if (hf & lbmp::kFlagBadInput) {
            delete c;
            return fail(LB_EINVAL, "rho0/u0 out of range (need finite, rho > 0, b rho/4 < 1, psi^2 > 0)");
        }
    }
    c->cur = 0;
    c->t = 0;
    *out = c;
    return LB_OK;
}

}  // namespace

extern "C" {

lb_status lb_init(lb_ctx** out, const lb_params* p, void* workspace, size_t workspace_bytes,
                  const float* rho0, const float* ux0, const float* uy0, void* stream)
{
    lb_status st = init_ctx(out, p, workspace, workspace_bytes, rho0, ux0, uy0, stream, true);
    if (st == LB_OK) g_last_error.clear();
    return st;
}

lb_status lb_step(lb_ctx* c, int64_t n)
{
    if (!c) return fail(LB_EINVAL, "ctx is NULL");
    if (c->poisoned) return fail(LB_ESTATE, "context poisoned by an earlier failure");
    if (n < 0) return fail(LB_EINVAL, "nsteps must be >= 0");
    if (c->stream != nullptr) {
        while (n >= c->graph_chunk) {
            if (!c->exec[c->cur]) {
                lb_status st = build_graph(c, c->cur);
                if (st != LB_OK) {
                    c->poisoned = true;
                    return st;
                }
            }
            hipError_t e = hipGraphLaunch(c->exec[c->cur], c->stream);
            if (e != hipSuccess) {
                c->poisoned = true;
                return hip_fail(e, "hipGraphLaunch");
            }
            n -= c->graph_chunk;
            c->t += c->graph_chunk;
            c->cur = c->graph_end[c->cur];
        }
    }
    return step_direct(c, n);
}

lb_status lb_moments(lb_ctx* c, float* rho, float* ux, float* uy)
{
    if (!c) return fail(LB_EINVAL, "ctx is NULL");
    if (c->poisoned) return fail(LB_ESTATE, "context poisoned by an earlier failure");
    hipError_t e = lbmp::launch_moments(c->p.store, c->p.bc == LB_BC_WALLS_Y, c->f[c->cur], c->kd,
                                        c->flag, rho, ux, uy, c->stream);
    if (e != hipSuccess) return hip_fail(e, "moments launch");
    return LB_OK;
}

static lbmp::DiagConst diag_const(const lb_ctx* c, const lb_region* in, const lb_region* outr)
{
    return lbmp::DiagConst{in->cx, in->cy, in->r_min, in->r_max,
                           outr->cx, outr->cy, outr->r_min, outr->r_max,
                           psi_const(c->p), c->p.bc == LB_BC_PERIODIC ? 1 : 0};
}

// Host lb_diag from the finalised sums [mass, mom_x, mom_y, sum p_in, sum p_out,
// sum rho_in, sum rho_out, n_in, n_out, max|u|, flag word].
static void fill_diag(const lb_ctx* c, const double* h, lb_diag* d)
{
    const int hf = (int)h[lbmp::kDiagFields];
    std::memset(d, 0, sizeof(*d));
    d->mass = h[0];
    d->mom_x = h[1];
    d->mom_y = h[2];
    d->n_in = h[7];
    d->n_out = h[8];
    d->p_in = h[7] > 0 ? h[3] / h[7] : NAN;
    d->p_out = h[8] > 0 ? h[4] / h[8] : NAN;
    d->rho_in = h[7] > 0 ? h[5] / h[7] : NAN;
    d->rho_out = h[8] > 0 ? h[6] / h[8] : NAN;
    d->dp = d->p_in - d->p_out;
    d->max_u = h[9];
    d->unstable = hf & lbmp::kFlagUnstable;
    d->step = c->t;
}

lb_status lb_diagnostics(lb_ctx* c, const lb_region* in, const lb_region* outr, lb_diag* d)
{
    if (!c || !in || !outr || !d) return fail(LB_EINVAL, "NULL argument");
    if (c->poisoned) return fail(LB_ESTATE, "context poisoned by an earlier failure");
    hipError_t e = lbmp::launch_diag(c->p.store, c->p.bc == LB_BC_WALLS_Y, c->f[c->cur], c->kd, c->flag,
                                     diag_const(c, in, outr), c->partial, c->dout, c->stream);
    double h[lbmp::kDiagOut];
    if (e == hipSuccess)
        e = hipMemcpyAsync(h, c->dout, sizeof(h), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) {
        c->poisoned = true;
        return hip_fail(e, "diagnostics");
    }
    fill_diag(c, h, d);
    if (d->unstable) {
        c->poisoned = true;
        return fail(LB_EUNSTABLE, "unstable site (non-finite rho or psi^2 <= 0) since init");
    }
    return LB_OK;
}

lb_status lb_check(lb_ctx* c)
{
    if (!c) return fail(LB_EINVAL, "ctx is NULL");
    if (c->poisoned) return fail(LB_ESTATE, "context poisoned by an earlier failure");
    int hf = 0;
    lb_status st = read_flag(c, &hf);
    if (st != LB_OK) return st;
    if (hf & lbmp::kFlagUnstable) {
        c->poisoned = true;
        return fail(LB_EUNSTABLE, "unstable site (non-finite rho or psi^2 <= 0) since init");
    }
    return LB_OK;
}

int64_t lb_time(const lb_ctx* c) { return c ? c->t : -1; }

// The exported state is [9][ny][nx] (then [ny][nx] FP32 densities for the
// local-density encodings, or [ny][nx] bf16 scales for the destination-scaled
// one); the stored one is [ny][row_slots][pitch].
static hipError_t copy_state(lb_ctx* c, void* dst, const void* src, bool out)
{
    const size_t eb = elem_bytes(c->p.store);
    const size_t nx = c->p.nx, ny = c->p.ny, pitch = c->k.pitch;
    const size_t row = (size_t)row_slots(c->p.store) * pitch * eb;
    char* buf = static_cast<char*>(out ? const_cast<void*>(src) : dst);
    char* ext = static_cast<char*>(out ? dst : const_cast<void*>(src));
    hipError_t e = hipSuccess;
    for (int a = 0; a < 9 && e == hipSuccess; ++a) {
        char* b = buf + a * pitch * eb;
        char* x = ext + a * ny * nx * eb;
        e = out ? hipMemcpy2DAsync(x, nx * eb, b, row, nx * eb, ny, hipMemcpyDeviceToDevice, c->stream)
                : hipMemcpy2DAsync(b, row, x, nx * eb, nx * eb, ny, hipMemcpyDeviceToDevice, c->stream);
    }
    const size_t db = density_plane_bytes(c->p.store);
    if (e == hipSuccess && db) {
        char* b = buf + 9 * pitch * eb;
        char* x = ext + 9 * ny * nx * eb;
        e = out ? hipMemcpy2DAsync(x, nx * db, b, row, nx * db, ny, hipMemcpyDeviceToDevice, c->stream)
                : hipMemcpy2DAsync(b, row, x, nx * db, nx * db, ny, hipMemcpyDeviceToDevice, c->stream);
    }
    return e;
}

lb_status lb_get_state(lb_ctx* c, void* dst)
{
    if (!c || !dst) return fail(LB_EINVAL, "NULL argument");
    hipError_t e = copy_state(c, dst, c->f[c->cur], true);
    if (e != hipSuccess) return hip_fail(e, "lb_get_state copy");
    return LB_OK;
}

lb_status lb_set_state(lb_ctx* c, const void* src, int64_t t)
{
    if (!c || !src) return fail(LB_EINVAL, "NULL argument");
    if (t < 0) return fail(LB_EINVAL, "t must be >= 0");
    hipError_t e = copy_state(c, c->f[0], src, false);
    if (e != hipSuccess) return hip_fail(e, "lb_set_state copy");
    c->cur = 0;
    c->t = t;
    return LB_OK;
}

lb_status lb_set_launch(lb_ctx* c, int32_t strip_rows, int32_t band, int32_t graph_chunk)
{
    if (!c) return fail(LB_EINVAL, "ctx is NULL");
    if (strip_rows < -1 || band < -1 || graph_chunk < 0) return fail(LB_EINVAL, "invalid launch parameter");
    if (graph_chunk != 0 && (graph_chunk < 2 || graph_chunk % 2))
        return fail(LB_EINVAL, "graph_chunk must be even and >= 2");
    drop_graphs(c);
    int rows = c->k.strip_rows, rows2 = c->k2.strip_rows, bd = c->k.band;
    if (strip_rows > 0) rows = rows2 = strip_rows;
    if (strip_rows == -1) {
        rows = auto_strip_rows(c->p);
        rows2 = auto_two_rows(c->p);
    }
    if (band > 0) bd = band;
    if (band == -1) bd = kDefaultBand;
    c->k = derive_single(c->p, rows, bd);
    c->k2 = derive_two(c->p, rows2, bd);
    c->waves2 = two_waves(c->p, rows2);
    if (graph_chunk > 0) c->graph_chunk = graph_chunk;
    if (strip_rows > 0) c->region_steps = 0;  // the caller asks for strips
    if (strip_rows == -1) set_regions(c);
    return LB_OK;
}

lb_status lb_destroy(lb_ctx* c)
{
    if (!c) return LB_OK;
    drop_graphs(c);
    delete c;
    return LB_OK;
}

const char* lb_last_error(void) { return g_last_error.c_str(); }

// ------------------------------------------------------------------ batched lattices

namespace {

// Default strip heights of the stepwise batch, per kernel group, measured on the
// 512-lattice sweep (sides 64-512, packed rows, MI355X), MLUPS by strip rows:
//   FP32, one column per lane:         2: 73.5k  3: 67.6k  5: 59.7k  8: 54.2k
//   destination-scaled FP16 (two columns per lane for even nx, one for odd nx, both
//   groups at the same height):        2: 81.2k  3: 92.1k  5: 98.2k  8: 100.7k
//   source-density FP16:               3: 77.5k  5: 80.1k  8: 79.6k
// A height per lattice-width class, chosen from uniform batches of each width, ran
// slower on the mix (FP32 70.9k): the strips resident at any moment then cover
// different row bands.  lb_batch_tune replaces the defaults by timings on the device
// at hand.
constexpr int kMaxStripRows = 64;
constexpr int kTuneMaxRows = 8;

// Heights that lb_batch_tune tries for the two-step launches.
constexpr int kTuneTwoRows[] = {4, 6, 8, 10, 12, 14, 16, 20};

// Height of equal strips of about `rows` rows.
int even_rows(int ny, int rows)
{
    const int strips = std::max(1, (ny + rows / 2) / rows);
    return (ny + strips - 1) / strips;
}

int default_batch_rows(int store)
{
    if (store == LB_STORE_F16_DEST) return 8;
    if (store == LB_STORE_F16_LOCAL) return 5;
    return 2;
}

// Whether lattice p is stepped two columns per lane in the stepwise batch.
bool batch_pair(const lb_params& p) { return lbmp::pair_step(p.store, p.nx); }

// Upper bound of the workgroups of the stepwise launches (one-row strips, one
// column per lane, the smallest workgroup), per group.
size_t batch_wg_capacity(const lb_params* p, int n)
{
    size_t tiles = 0;
    for (int i = 0; i < n; ++i) tiles += (size_t)((p[i].nx + lbmp::kTileW - 1) / lbmp::kTileW) * p[i].ny;
    const int wpb = std::min(lbmp::batch_waves_per_block(p[0].store, false), lbmp::batch_waves_per_block(p[0].store, true));
    return tiles / wpb + 4;
}

// Whether the stepwise batch advances two steps per launch.
bool batch_two(const lb_params* p, int n)
{
    for (int i = 0; i < n; ++i)
        if (!two_step(p[i])) return false;
    return true;
}

// Upper bound of the workgroups of the two-step launch (one-row strips).
size_t batch_two_capacity(const lb_params* p, int n)
{
    size_t tiles = 0;
    for (int i = 0; i < n; ++i) tiles += (size_t)((p[i].nx + lbmp::kTwoTileW - 1) / lbmp::kTwoTileW) * p[i].ny;
    return tiles / lbmp::kTwoWaves + 1;
}

int batch_diag_tiles(const lb_params* p, int n)
{
    long long tiles = 0;
    for (int i = 0; i < n; ++i) tiles += layout_of(p[i]).diag_tiles;
    return (int)std::min<long long>(tiles, 0x7fffffff);
}

// Offsets of the batch's own part of the workspace, in front of the lattices'.  What the host
// writes comes first, in one piece: the descriptors and tile prefix sums of the launches and
// of the diagnostics, then `tables`, room for the workgroup tables of all of them.
struct BatchLayout {
    size_t desc, two_desc, tile_start, two_start, diag, diag_start, tables;
    size_t table_entries;
    size_t clocks, regions, diag_out, flags, total;
};

BatchLayout batch_layout(const lb_params* p, int n)
{
    BatchLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align_up(bytes, kAlign);
        return at;
    };
    const bool two = batch_two(p, n);
    L.desc = take((size_t)n * sizeof(lbmp::BatchInstance));
    L.two_desc = take(two ? (size_t)n * sizeof(lbmp::BatchInstance) : 0);
    L.tile_start = take((size_t)(n + 2) * sizeof(int));
    L.two_start = take(two ? (size_t)(n + 1) * sizeof(int) : 0);
    L.diag = take((size_t)n * sizeof(lbmp::DiagInstance));
    L.diag_start = take((size_t)(n + 1) * sizeof(int));
    L.table_entries = batch_wg_capacity(p, n) + (two ? batch_two_capacity(p, n) : 0) +
                      (size_t)batch_diag_tiles(p, n) / lbmp::kPassWaves + 1;
    L.tables = take(L.table_entries * sizeof(int));
    L.clocks = take((size_t)n * 16);
    L.regions = take((size_t)n * sizeof(lbmp::DiagConst));
    L.diag_out = take((size_t)n * lbmp::kDiagOut * sizeof(double));
    L.flags = take((size_t)n * sizeof(int));
    L.total = off;
    return L;
}

}  // namespace

struct lb_batch {
    int n;
    int mode;                        // LB_BATCH_STEPWISE or LB_BATCH_PERSISTENT
    int fixed_rows;                  // > 0: every lattice walks strips of this height
    int group_rows[2];               // stepwise heights per kernel group (default or tuned)
    // Stepwise lattices form two groups, each stepped by its own launch: group 0 one
    // column per lane, group 1 two columns per lane (destination-scaled FP16, even
    // nx).  Group g holds dispatch positions [gfirst[g], gfirst[g] + gcount[g]) of
    // `desc` and `order`; its tile prefix sums start at tile_start + gfirst[g] + g and
    // its workgroup table at wg_first + wg_off[g].
    int gfirst[2], gcount[2], ntotal[2];
    size_t wg_off[2];
    // FP32 lattices (all of them group 0) of at least 8 x 8 are stepped two at a time in the
    // stepwise mode, with descriptors and tables of their own (same dispatch order).
    bool two;
    int two_rows, two_waves, two_ntotal;  // two_rows: tuned height, 0: batch_two_rows
    lbmp::BatchInstance* two_desc;
    int *two_start, *two_first;
    int* tile_start;                 // device, n + 2 entries
    int* wg_first;                   // device, lattice of each workgroup's first tile
    char* ws;                        // workspace
    BatchLayout L;
    hipGraph_t graph[2];
    hipGraphExec_t exec[2];
    hipEvent_t ev[2];                // bracket the last lb_batch_step (stepwise mode)
    std::vector<lb_ctx*> inst;       // per-lattice contexts on slices of the workspace
    std::vector<int> order;          // dispatch position -> lattice index
    std::vector<int> rows;           // strip height per lattice (current launch mode)
    lbmp::BatchInstance* desc;       // device descriptors in dispatch order
    unsigned long long* clocks;      // device, 2 per workgroup
    // diagnostics of all lattices together (in lattice order)
    lbmp::DiagInstance* diag;        // device, n
    lbmp::DiagConst* regions;        // device, n
    double* diag_out;                // device, n records of kDiagOut
    int *diag_start, *diag_first;    // device, tile prefix sums (n + 1) and workgroup table
    int* flags;                      // device, n
    int diag_ntotal;
    hipStream_t stream;
    int store, bc, psi;
    bool poisoned;
};

namespace {

void drop_batch_graphs(lb_batch* b)
{
    for (int i = 0; i < 2; ++i) {
        if (b->exec[i]) (void)hipGraphExecDestroy(b->exec[i]);
        if (b->graph[i]) (void)hipGraphDestroy(b->graph[i]);
        b->exec[i] = nullptr;
        b->graph[i] = nullptr;
    }
}

// Dispatch order: in the stepwise mode the one-column lattices, then the
// two-column ones, each largest first (longest-processing-time order); in the
// persistent mode every lattice in one group (one column per lane), largest first.
void order_batch(lb_batch* b)
{
    const int n = b->n;
    std::vector<int> idx(n);
    for (int i = 0; i < n; ++i) idx[i] = i;
    auto area = [&](int i) { return (long long)b->inst[i]->p.nx * b->inst[i]->p.ny; };
    auto grp = [&](int i) { return b->mode == LB_BATCH_STEPWISE && batch_pair(b->inst[i]->p) ? 1 : 0; };
    std::stable_sort(idx.begin(), idx.end(), [&](int x, int y) {
        if (grp(x) != grp(y)) return grp(x) < grp(y);
        return area(x) > area(y);
    });
    b->order = idx;
    b->gcount[0] = b->gcount[1] = 0;
    for (int i = 0; i < n; ++i) ++b->gcount[grp(i)];
    b->gfirst[0] = 0;
    b->gfirst[1] = b->gcount[0];
}

// Strip height of lattice i in the current mode.
int lattice_rows(const lb_batch* b, int i)
{
    if (b->fixed_rows > 0) return b->fixed_rows;
    if (b->mode == LB_BATCH_PERSISTENT) return kBatchPersistentRows;
    return b->group_rows[batch_pair(b->inst[i]->p) ? 1 : 0];
}

// Wavefronts per workgroup of the two-step launches of a batch: with a full chip 8 pace a
// wider stretch of a row (512 lattices of sides 64-512 at 16 rows 424 us per step, 435 us with
// 4); as long as every strip can be resident 4 spread more evenly.
int batch_two_waves(long long strips) { return strips > 16LL * compute_units() ? lbmp::kTwoWavesWide : lbmp::kTwoWaves; }

// Strip height of the two-step launches of a batch: the cheapest for all its strips (two_cost),
// of which the tallest are the longest walk (200 lattices of 32 x 32 have strips of 7 rows at a
// height of 6: 7.5 us per step where that was priced as 6, 6.2 us at 4; 350 of 12 x 12 6.0 / 5.2).
int batch_two_rows(const lb_batch* b)
{
    const int ncu = compute_units();
    int best = 2;
    double least = 1e300;
    for (int h = 2; h <= 20; ++h) {
        long long strips = 0;
        int tallest = 0;
        for (int i = 0; i < b->n; ++i) {
            const lb_params& p = b->inst[i]->p;
            const int rows = even_rows(p.ny, h);
            tallest = std::max(tallest, rows);
            strips += (long long)((p.nx + lbmp::kTwoTileW - 1) / lbmp::kTwoTileW) * ((p.ny + rows - 1) / rows);
        }
        const double cost = two_cost(tallest, strips, batch_two_waves(strips), ncu);
        if (cost < least) {
            least = cost;
            best = h;
        }
    }
    return best;
}

// Copy the launch descriptors (dispatch order), those of the diagnostics (lattice order) and
// their tile tables to the device, in one copy (creating a batch of one lattice took 154 us with
// a copy for each, 104 us so).  trial: two-step launches report unstable sites to words that
// nobody reads, since they also look at the state one step ahead.
hipError_t write_batch_descriptors(lb_batch* b, bool trial = false)
{
    drop_batch_graphs(b);
    const int n = b->n;
    const BatchLayout& L = b->L;
    std::vector<char> image(L.tables, 0);
    std::vector<int> tables;
    auto* host = reinterpret_cast<lbmp::BatchInstance*>(image.data() + L.desc);
    int* const start = reinterpret_cast<int*>(image.data() + L.tile_start);
    // diagnostics
    {
        auto* diag = reinterpret_cast<lbmp::DiagInstance*>(image.data() + L.diag);
        int* st = reinterpret_cast<int*>(image.data() + L.diag_start);
        for (int i = 0; i < n; ++i) {
            const lb_ctx* c = b->inst[i];
            diag[i] = lbmp::DiagInstance{c->kd, {c->f[0], c->f[1]}, c->flag, c->partial};
            st[i + 1] = st[i] + c->kd.tiles_x * c->kd.tiles_y;
        }
        b->diag_ntotal = st[n];
        b->diag_first = reinterpret_cast<int*>(b->ws + L.tables);
        for (int t = 0, i = 0; t < b->diag_ntotal; t += lbmp::kPassWaves) {
            while (t >= st[i + 1]) ++i;
            tables.push_back(i);
        }
    }
    // single steps, both groups
    b->rows.assign(n, 0);
    b->wg_first = reinterpret_cast<int*>(b->ws + L.tables) + tables.size();
    const size_t wg0 = tables.size();
    for (int g = 0; g < 2; ++g) {
        const int j0 = b->gfirst[g], cnt = b->gcount[g];
        int* st = start + j0 + g;
        st[0] = 0;
        for (int j = 0; j < cnt; ++j) {
            const int i = b->order[j0 + j];
            lb_ctx* c = b->inst[i];
            const int rows = lattice_rows(b, i);
            b->rows[i] = rows;
            lbmp::StepConst k = derive(c->p, rows, 1);
            if (g == 1) k.tiles_x = (c->p.nx + lbmp::kPairTileW - 1) / lbmp::kPairTileW;
            host[j0 + j].k = k;
            host[j0 + j].f[0] = c->f[0];
            host[j0 + j].f[1] = c->f[1];
            host[j0 + j].flag = c->flag;
            st[j + 1] = st[j] + k.tiles_x * k.tiles_y;
        }
        b->ntotal[g] = st[cnt];
        const int wpb = lbmp::batch_waves_per_block(b->store, g == 1);
        const int blocks = (b->ntotal[g] + wpb - 1) / wpb;
        b->wg_off[g] = tables.size() - wg0;
        for (int blk = 0, i = 0; blk < blocks; ++blk) {
            const int t = blk * wpb;
            while (t >= st[i + 1]) ++i;
            tables.push_back(i);
        }
    }
    // two steps per launch
    if (b->two && b->mode == LB_BATCH_STEPWISE) {
        auto* host2 = reinterpret_cast<lbmp::BatchInstance*>(image.data() + L.two_desc);
        int* st = reinterpret_cast<int*>(image.data() + L.two_start);
        const int target = b->two_rows > 0 ? b->two_rows : batch_two_rows(b);
        for (int j = 0; j < n; ++j) {
            const lb_params& p = b->inst[b->order[j]]->p;
            host2[j] = host[j];
            host2[j].k = derive_two(p, b->fixed_rows > 0 ? b->fixed_rows : even_rows(p.ny, target));
            if (trial) host2[j].flag = b->flags + j;
            st[j + 1] = st[j] + host2[j].k.tiles_x * host2[j].k.tiles_y;
        }
        b->two_ntotal = st[n];
        b->two_waves = batch_two_waves(b->two_ntotal);
        b->two_first = reinterpret_cast<int*>(b->ws + L.tables) + tables.size();
        for (int t = 0, i = 0; t < b->two_ntotal; t += b->two_waves) {
            while (t >= st[i + 1]) ++i;
            tables.push_back(i);
        }
    }
    if (tables.size() > L.table_entries) return hipErrorInvalidValue;
    const char* const extra = reinterpret_cast<const char*>(tables.data());
    image.insert(image.end(), extra, extra + tables.size() * sizeof(int));
    hipError_t e = hipMemcpyAsync(b->ws, image.data(), image.size(), hipMemcpyHostToDevice, b->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
    return e;
}

// The flag words of all lattices; synchronises.
hipError_t read_batch_flags(lb_batch* b, std::vector<int>& flags)
{
    flags.assign(b->n, 0);
    const int* from = b->inst[0]->flag;  // one lattice: its word, without a launch to gather (20 us, 23 us with it)
    hipError_t e = hipSuccess;
    if (b->n > 1) {
        from = b->flags;
        e = lbmp::launch_batch_flags(b->diag, b->n, b->flags, b->stream);
    }
    if (e == hipSuccess)
        e = hipMemcpyAsync(flags.data(), from, flags.size() * sizeof(int), hipMemcpyDeviceToHost, b->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
    return e;
}

// One step of every lattice (stepwise mode) reading buffer `parity`.
hipError_t batch_flat_launch(lb_batch* b, int parity)
{
    hipError_t e = hipSuccess;
    for (int g = 0; g < 2 && e == hipSuccess; ++g) {
        if (b->gcount[g] == 0) continue;
        e = lbmp::launch_batch_flat(b->store, b->bc == LB_BC_WALLS_Y, b->psi, g == 1, b->desc + b->gfirst[g],
                                    b->tile_start + b->gfirst[g] + g, b->wg_first + b->wg_off[g], b->ntotal[g],
                                    parity, b->stream);
    }
    return e;
}

// One launch reading buffer `parity`: two steps where the batch is stepped that way and
// `left` allows it, else one.  *steps receives the number of steps taken.
hipError_t batch_launch_some(lb_batch* b, int parity, int64_t left, int* steps)
{
    *steps = b->two && left >= 2 ? 2 : 1;
    if (*steps == 1) return batch_flat_launch(b, parity);
    return lbmp::launch_batch_two(b->bc == LB_BC_WALLS_Y, b->psi, b->two_desc, b->two_start, b->two_first, b->two_ntotal,
                                  b->two_waves, parity, b->stream);
}

lb_status build_batch_graph(lb_batch* b, int from)
{
    hipError_t e = hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) return hip_fail(e, "hipStreamBeginCapture");
    hipError_t le = hipSuccess;
    static_assert(kDefaultGraphChunk % 4 == 0, "a graph returns to the buffer it starts from");
    int parity = from;
    for (int left = kDefaultGraphChunk; left > 0 && le == hipSuccess; parity ^= 1) {
        int steps = 0;
        le = batch_launch_some(b, parity, left, &steps);
        left -= steps;
    }
    hipGraph_t g = nullptr;
    e = hipStreamEndCapture(b->stream, &g);
    if (le != hipSuccess) {
        if (g) (void)hipGraphDestroy(g);
        return hip_fail(le, "batch launch during capture");
    }
    if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
    hipGraphExec_t x = nullptr;
    e = hipGraphInstantiate(&x, g, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        (void)hipGraphDestroy(g);
        return hip_fail(e, "hipGraphInstantiate");
    }
    b->graph[from] = g;
    b->exec[from] = x;
    return LB_OK;
}

lb_status validate_batch(const lb_params* p, int32_t n)
{
    if (!p || n < 1) return fail(LB_EINVAL, "need n >= 1 parameter blocks");
    for (int i = 0; i < n; ++i) {
        lb_status st = validate(p + i);
        if (st != LB_OK) return fail(st, "lattice " + std::to_string(i) + ": " + g_last_error);
        if (p[i].store != p[0].store || p[i].bc != p[0].bc || p[i].psi_form != p[0].psi_form)
            return fail(LB_EINVAL, "all lattices of a batch share store, bc and psi_form");
        if (p[i].stencil != LB_STENCIL_NEAREST)
            return fail(LB_EINVAL, "batched lattices use the nearest-neighbour stencil");
    }
    if (p[0].store != LB_STORE_F32 && p[0].store != LB_STORE_F16_LOCAL && p[0].store != LB_STORE_F16_DEST)
        return fail(LB_EINVAL, "batched storage must be LB_STORE_F32, LB_STORE_F16_LOCAL or LB_STORE_F16_DEST");
    return LB_OK;
}

}  // namespace

size_t lb_batch_workspace_bytes(const lb_params* p, int32_t n)
{
    if (validate_batch(p, n) != LB_OK) return 0;
    size_t total = batch_layout(p, n).total;
    for (int i = 0; i < n; ++i) total += layout_of(p[i]).total;
    return total;
}

lb_status lb_batch_init(lb_batch** out, const lb_params* p, int32_t n, void* workspace,
                        size_t workspace_bytes, const float* const* rho0, const float* const* ux0,
                        const float* const* uy0, void* stream)
{
    if (!out) return fail(LB_EINVAL, "out is NULL");
    *out = nullptr;
    lb_status st = validate_batch(p, n);
    if (st != LB_OK) return st;
    if (!workspace || !rho0) return fail(LB_EINVAL, "workspace and rho0 must be non-NULL");
    if (reinterpret_cast<uintptr_t>(workspace) % kAlign) return fail(LB_EINVAL, "workspace must be 256-byte aligned");
    if (workspace_bytes < lb_batch_workspace_bytes(p, n))
        return fail(LB_ENOMEM, "workspace smaller than lb_batch_workspace_bytes");

    lb_batch* b = new (std::nothrow) lb_batch{};
    if (!b) return fail(LB_ENOMEM, "host allocation failed");
    b->n = n;
    b->stream = static_cast<hipStream_t>(stream);
    b->store = p[0].store;
    b->bc = p[0].bc;
    b->psi = p[0].psi_form;
    char* ws = static_cast<char*>(workspace);
    const BatchLayout L = batch_layout(p, n);
    b->ws = ws;
    b->L = L;
    b->two = batch_two(p, n);
    b->two_rows = 0;
    b->desc = reinterpret_cast<lbmp::BatchInstance*>(ws + L.desc);
    b->two_desc = reinterpret_cast<lbmp::BatchInstance*>(ws + L.two_desc);
    b->tile_start = reinterpret_cast<int*>(ws + L.tile_start);
    b->two_start = reinterpret_cast<int*>(ws + L.two_start);
    b->diag = reinterpret_cast<lbmp::DiagInstance*>(ws + L.diag);
    b->diag_start = reinterpret_cast<int*>(ws + L.diag_start);
    b->clocks = reinterpret_cast<unsigned long long*>(ws + L.clocks);
    b->regions = reinterpret_cast<lbmp::DiagConst*>(ws + L.regions);
    b->diag_out = reinterpret_cast<double*>(ws + L.diag_out);
    b->flags = reinterpret_cast<int*>(ws + L.flags);
    b->mode = LB_BATCH_STEPWISE;
    hipError_t ee = hipEventCreate(&b->ev[0]);
    if (ee == hipSuccess) ee = hipEventCreate(&b->ev[1]);
    if (ee != hipSuccess) {
        lb_batch_destroy(b);
        return hip_fail(ee, "hipEventCreate");
    }
    size_t off = L.total;
    auto drop = [&] {
        lb_batch_destroy(b);
        b = nullptr;
    };
    try {
        b->inst.assign(n, nullptr);
        for (int i = 0; i < n; ++i) {
            const size_t bytes = layout_of(p[i]).total;
            st = init_ctx(&b->inst[i], p + i, ws + off, bytes, rho0[i], ux0 ? ux0[i] : nullptr,
                          uy0 ? uy0[i] : nullptr, stream, false);
            if (st != LB_OK) {
                const std::string msg = g_last_error;
                drop();
                return fail(st, "lattice " + std::to_string(i) + ": " + msg);
            }
            off += bytes;
        }
        b->group_rows[0] = b->group_rows[1] = default_batch_rows(b->store);
        order_batch(b);
        hipError_t e = write_batch_descriptors(b);
        std::vector<int> flags;
        if (e == hipSuccess) e = read_batch_flags(b, flags);
        if (e != hipSuccess) {
            drop();
            return hip_fail(e, "batch descriptors");
        }
        for (int i = 0; i < n; ++i) {
            if (!(flags[i] & lbmp::kFlagBadInput)) continue;
            drop();
            return fail(LB_EINVAL, "lattice " + std::to_string(i) + ": rho0/u0 out of range");
        }
        *out = b;
        g_last_error.clear();
        return LB_OK;
    } catch (const std::bad_alloc&) {
        drop();
        return no_memory();
    }
}

lb_status lb_batch_step(lb_batch* b, int64_t nsteps)
{
    if (!b) return fail(LB_EINVAL, "batch is NULL");
    if (b->poisoned) return fail(LB_ESTATE, "batch poisoned by an earlier failure");
    if (nsteps < 0 || nsteps > (1LL << 30)) return fail(LB_EINVAL, "nsteps must lie in [0, 2^30]");
    if (nsteps == 0) return LB_OK;
    int parity = b->inst[0]->cur;
    hipError_t e = hipSuccess;
    if (b->mode == LB_BATCH_PERSISTENT) {
        e = lbmp::launch_batch(b->store, b->bc == LB_BC_WALLS_Y, b->psi, b->desc, b->n, (int)nsteps, parity, b->clocks,
                               b->stream);
        parity ^= (int)(nsteps & 1);
    } else {
        e = hipEventRecord(b->ev[0], b->stream);
        int64_t left = nsteps;
        while (e == hipSuccess && b->stream != nullptr && left >= kDefaultGraphChunk) {
            if (!b->exec[parity]) {
                lb_status st = build_batch_graph(b, parity);
                if (st != LB_OK) {
                    b->poisoned = true;
                    return st;
                }
            }
            e = hipGraphLaunch(b->exec[parity], b->stream);
            left -= kDefaultGraphChunk;  // an even number of launches: the parity is unchanged
        }
        for (; e == hipSuccess && left > 0; parity ^= 1) {
            int steps = 0;
            e = batch_launch_some(b, parity, left, &steps);
            left -= steps;
        }
        if (e == hipSuccess) e = hipEventRecord(b->ev[1], b->stream);
    }
    if (e != hipSuccess) {
        b->poisoned = true;
        return hip_fail(e, "batch launch");
    }
    for (lb_ctx* c : b->inst) {
        c->cur = parity;
        c->t += nsteps;
    }
    return LB_OK;
}

static lb_ctx* batch_member(lb_batch* b, int32_t i)
{
    if (!b || i < 0 || i >= b->n) return nullptr;
    return b->inst[i];
}

lb_status lb_batch_moments(lb_batch* b, int32_t i, float* rho, float* ux, float* uy)
{
    lb_ctx* c = batch_member(b, i);
    if (!c) return fail(LB_EINVAL, "no such lattice");
    return lb_moments(c, rho, ux, uy);
}

lb_status lb_batch_diagnostics(lb_batch* b, int32_t i, const lb_region* in, const lb_region* outr, lb_diag* d)
{
    lb_ctx* c = batch_member(b, i);
    if (!c) return fail(LB_EINVAL, "no such lattice");
    return lb_diagnostics(c, in, outr, d);
}

lb_status lb_batch_diagnostics_all(lb_batch* b, const lb_region* in, const lb_region* outr, lb_diag* d)
try {
    if (!b || !in || !outr || !d) return fail(LB_EINVAL, "NULL argument");
    if (b->poisoned) return fail(LB_ESTATE, "batch poisoned by an earlier failure");
    const int n = b->n;
    std::vector<double> h((size_t)n * lbmp::kDiagOut, 0.0);
    std::vector<lbmp::DiagConst> dg(n);
    for (int i = 0; i < n; ++i) dg[i] = diag_const(b->inst[i], in + i, outr + i);
    hipError_t e = hipMemcpyAsync(b->regions, dg.data(), dg.size() * sizeof(dg[0]), hipMemcpyHostToDevice, b->stream);
    if (e == hipSuccess)
        e = lbmp::launch_batch_diag(b->store, b->bc == LB_BC_WALLS_Y, b->psi, b->diag, b->regions, n, b->diag_start,
                                    b->diag_first, b->diag_ntotal, b->inst[0]->cur, b->diag_out, b->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(h.data(), b->diag_out, h.size() * sizeof(double), hipMemcpyDeviceToHost, b->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
    if (e != hipSuccess) {
        b->poisoned = true;
        return hip_fail(e, "batch diagnostics");
    }
    int bad = 0;
    for (int i = 0; i < n; ++i) {
        lb_ctx* c = b->inst[i];
        double* hi = &h[(size_t)i * lbmp::kDiagOut];
        if (c->poisoned) std::fill(hi, hi + lbmp::kDiagOut, 0.0);  // its fields are meaningless
        fill_diag(c, hi, d + i);
        if (c->poisoned || d[i].unstable) {
            d[i].unstable = 1;
            c->poisoned = true;
            ++bad;
        }
    }
    return bad ? fail(LB_EUNSTABLE, std::to_string(bad) + " lattice(s) flagged an unstable site") : LB_OK;
} catch (const std::bad_alloc&) {
    return no_memory();
}

lb_status lb_batch_get_state(lb_batch* b, int32_t i, void* dst)
{
    lb_ctx* c = batch_member(b, i);
    if (!c) return fail(LB_EINVAL, "no such lattice");
    return lb_get_state(c, dst);
}

lb_status lb_batch_check(lb_batch* b, int32_t* unstable)
try {
    if (!b) return fail(LB_EINVAL, "batch is NULL");
    std::vector<int> flags;
    const hipError_t e = read_batch_flags(b, flags);
    if (e != hipSuccess) {
        for (lb_ctx* c : b->inst) c->poisoned = true;
        return hip_fail(e, "reading the device flags");
    }
    int count = 0;
    for (int i = 0; i < b->n; ++i) {
        if (flags[i] & lbmp::kFlagUnstable) {
            ++count;
            b->inst[i]->poisoned = true;
        }
    }
    if (unstable) *unstable = count;
    return count ? fail(LB_EUNSTABLE, std::to_string(count) + " lattice(s) flagged an unstable site") : LB_OK;
} catch (const std::bad_alloc&) {
    return no_memory();
}

lb_status lb_batch_times(lb_batch* b, double* seconds)
try {
    if (!b || !seconds) return fail(LB_EINVAL, "NULL argument");
    if (b->mode == LB_BATCH_STEPWISE) {
        float ms = 0.0f;
        hipError_t e = hipEventSynchronize(b->ev[1]);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, b->ev[0], b->ev[1]);
        if (e != hipSuccess) return hip_fail(e, "batch events");
        for (int i = 0; i < b->n; ++i) seconds[i] = ms * 1e-3;
        return LB_OK;
    }
    std::vector<unsigned long long> h(2 * (size_t)b->n);
    hipError_t e = hipMemcpyAsync(h.data(), b->clocks, h.size() * sizeof(unsigned long long),
                                  hipMemcpyDeviceToHost, b->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
    int dev = 0, khz = 0;
    if (e == hipSuccess) e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev);
    if (e != hipSuccess) return hip_fail(e, "batch clocks");
    if (khz <= 0) return fail(LB_EHIP, "device reports no wall-clock rate");
    unsigned long long t0 = h[0];
    for (int j = 0; j < b->n; ++j) t0 = std::min(t0, h[2 * j]);
    for (int j = 0; j < b->n; ++j) seconds[b->order[j]] = (double)(h[2 * j + 1] - t0) / (khz * 1e3);
    return LB_OK;
} catch (const std::bad_alloc&) {
    return no_memory();
}

lb_status lb_batch_set_launch(lb_batch* b, int32_t mode, int32_t strip_rows)
try {
    if (!b) return fail(LB_EINVAL, "batch is NULL");
    if (mode != LB_BATCH_STEPWISE && mode != LB_BATCH_PERSISTENT) return fail(LB_EINVAL, "unknown batch mode");
    if (strip_rows < 0 || strip_rows > kMaxStripRows) return fail(LB_EINVAL, "strip_rows must lie in [0, 64]");
    b->mode = mode;
    b->fixed_rows = strip_rows;
    order_batch(b);
    hipError_t e = write_batch_descriptors(b);
    if (e != hipSuccess) return hip_fail(e, "batch descriptors");
    return LB_OK;
} catch (const std::bad_alloc&) {
    b->poisoned = true;  // the descriptors may not be those of the settings
    return no_memory();
}

lb_status lb_batch_tune(lb_batch* b, int32_t trial_steps, int32_t* rows_out)
try {
    if (!b) return fail(LB_EINVAL, "batch is NULL");
    if (b->poisoned) return fail(LB_ESTATE, "batch poisoned by an earlier failure");
    if (trial_steps < 1 || trial_steps > 1000) return fail(LB_EINVAL, "trial_steps must lie in [1, 1000]");
    if (b->mode != LB_BATCH_STEPWISE) return fail(LB_EINVAL, "lb_batch_tune tunes the stepwise mode");
    if (b->stream == nullptr) return fail(LB_EINVAL, "lb_batch_tune needs a stream other than the legacy stream");
    b->fixed_rows = 0;
    const int parity = b->inst[0]->cur;
    // Seconds of `trial_steps` launches that all read buffer `parity` and write the
    // other one: the state (buffer parity) is unchanged, and the other buffer is
    // overwritten in full by the next step.  The least of three repetitions.
    // at_once = 1: single-step launches, 2: two-step launches.
    auto time_launches = [&](int at_once, double& sec) -> hipError_t {
        int steps = 0;
        hipError_t e = write_batch_descriptors(b, true);
        for (int w = 0; w < 2 && e == hipSuccess; ++w) e = batch_launch_some(b, parity, at_once, &steps);
        sec = 1e30;
        for (int rep = 0; rep < 3 && e == hipSuccess; ++rep) {
            e = hipEventRecord(b->ev[0], b->stream);
            for (int t = 0; t < trial_steps && e == hipSuccess; ++t) e = batch_launch_some(b, parity, at_once, &steps);
            if (e == hipSuccess) e = hipEventRecord(b->ev[1], b->stream);
            if (e == hipSuccess) e = hipEventSynchronize(b->ev[1]);
            float ms = 0.0f;
            if (e == hipSuccess) e = hipEventElapsedTime(&ms, b->ev[0], b->ev[1]);
            sec = std::min(sec, ms * 1e-3);
        }
        return e;
    };
    // each kernel group (the larger first) gets the height that runs its share of the
    // batch fastest, with the other group at its current height
    const int first = b->gcount[1] > b->gcount[0] ? 1 : 0;
    for (int gi = 0; gi < 2; ++gi) {
        const int g = gi == 0 ? first : 1 - first;
        if (b->gcount[g] == 0) continue;
        int best_r = b->group_rows[g];
        double best = 1e30;
        hipError_t e = hipSuccess;
        for (int cand = 1; cand <= kTuneMaxRows && e == hipSuccess; ++cand) {
            b->group_rows[g] = cand;
            double sec = 0.0;
            e = time_launches(1, sec);
            if (e == hipSuccess && sec < best) {
                best = sec;
                best_r = cand;
            }
        }
        b->group_rows[g] = best_r;
        if (e != hipSuccess) {
            b->poisoned = true;
            return hip_fail(e, "lb_batch_tune trial launches");
        }
    }
    if (b->two) {
        int best_r = b->two_rows;
        double best = 1e30;
        for (const int cand : kTuneTwoRows) {
            b->two_rows = cand;
            double sec = 0.0;
            const hipError_t e = time_launches(2, sec);
            if (e != hipSuccess) {
                b->poisoned = true;
                return hip_fail(e, "lb_batch_tune trial launches");
            }
            if (sec < best) {
                best = sec;
                best_r = cand;
            }
        }
        b->two_rows = best_r;
    }
    hipError_t e = write_batch_descriptors(b);
    if (e != hipSuccess) return hip_fail(e, "batch descriptors");
    if (rows_out)
        for (int i = 0; i < b->n; ++i) rows_out[i] = b->rows[i];
    return LB_OK;
} catch (const std::bad_alloc&) {
    b->poisoned = true;  // the descriptors may not be those of the settings
    return no_memory();
}

lb_status lb_batch_destroy(lb_batch* b)
{
    if (!b) return LB_OK;
    drop_batch_graphs(b);
    for (int i = 0; i < 2; ++i)
        if (b->ev[i]) (void)hipEventDestroy(b->ev[i]);
    for (lb_ctx* c : b->inst)
        if (c) lb_destroy(c);
    delete b;
    return LB_OK;
}

lb_status lb_copy_probe(const void* src, void* dst, size_t bytes, void* stream)
{
    if (!src || !dst || bytes % 16) return fail(LB_EINVAL, "need non-NULL buffers and bytes % 16 == 0");
    hipError_t e = lbmp::launch_copy_probe(src, dst, (long long)(bytes / 16), static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return hip_fail(e, "copy probe launch");
    return LB_OK;
}

}  // extern "C"
