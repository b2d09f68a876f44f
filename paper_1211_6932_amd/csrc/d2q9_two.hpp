// d2q9_two.hpp -- two D2Q9 time steps in one pass over memory (FP32 storage,
// nearest-neighbour stencil).
#pragma once

#include "d2q9_core.hpp"

namespace lbmp {

// A wavefront walks a strip in direction DIR (+1: up, -1: down in y); when the first step
// collides row r, it passes the post-collision populations of that row straight on to the
// second step, in registers: the populations that move with the walk or stay level belong to
// the second step's rows r + DIR and r, those that move against it complete its row r - DIR,
// and populations that change column come from the neighbouring lane.  Density and psi of
// row r - DIR then allow the second step to collide row r - 2 DIR, which is stored.  The
// state is read and written once per two steps.
// Lane l handles column x0 - 3 + l; the first step needs one halo column a side for psi
// and the second two more (pull, psi), so lanes 3..60 own the 58 output columns.
// Likewise the first step collides two rows more on each side of the strip.  Each site's
// arithmetic is that of strip_walk: the result is bitwise that of two single steps.
//
// What bounds it (8192 x 4096 splash): the single step moves 72 B per site and step and is
// bound by HBM (428 us, 78.4k MLUPS).  Here 36 B and the halo rows remain, 5.5 TB/s or 88 % of
// what a copy reaches, and the vector ALUs are busy for 76 % of the time: 276 instructions
// per wavefront row and pair of steps (with 315 of them, at 90 %, a step took the same 248 us,
// 135k MLUPS; 2048 x 1024 took 2 % longer).  One column per lane: the walk needs 121 VGPRs, so
// four waves per SIMD hide the latency of its loads.
template <bool WALLS, int PSI, int DIR>
__device__ __forceinline__ void two_walk(const float* __restrict__ fin, float* __restrict__ fout,
                                         const StepConst& k, const int ty, const bool live, const bool check,
                                         const unsigned xm, const unsigned xc, const unsigned xp,
                                         int* __restrict__ flag)
{
    const int y0 = ty * k.strip_rows;
    const int y1 = min(y0 + k.strip_rows, k.ny);
    const int n = y1 - y0;
    const int o0 = DIR > 0 ? y0 : y1 - 1;          // first output row of the walk
    const int e0 = DIR > 0 ? 0 : k.ny - 1;         // rows next to the walls in walk order
    const int e1 = DIR > 0 ? k.ny - 1 : 0;
    auto inside = [&](const int y) __attribute__((always_inline)) { return !WALLS || (y >= 0 && y < k.ny); };
    auto wrap = [&](const int y) __attribute__((always_inline)) {
        if (WALLS) return y;
        return y < 0 ? y + k.ny : (y >= k.ny ? y - k.ny : y);
    };
    const Shear nu = in_vectors(k);
    using Win = PsiRow;
    auto window = [](const float v) __attribute__((always_inline)) {
        return psi_row(lane_from_left(v), v, lane_from_right(v));
    };
    auto collide_row = [&](float (&f)[9], const float r, const Sums& sums, const Win& before, const Win& c, const Win& after)
                           __attribute__((always_inline)) {
        const Win& m = DIR > 0 ? before : after;
        const Win& p = DIR > 0 ? after : before;
        float Fx, Fy, Fs2;
        force_stencil(m, c, p, k, Fx, Fy, Fs2);
        float jx, jy;
        momentum(f, jx, jy);
        const float inv_rho = recip(r);
        collide(f, r, sums, fmaf(0.5f, Fx, jx) * inv_rho, fmaf(0.5f, Fy, jy) * inv_rho, Fx, Fy, Fs2, k, nu);
    };
    // populations moving up (into the row above) / down, by column shift
    auto move_up = [](float (&to)[9], const float (&f)[9]) __attribute__((always_inline)) {
        to[2] = f[2];
        to[5] = lane_from_left(f[5]);
        to[6] = lane_from_right(f[6]);
    };
    auto move_down = [](float (&to)[9], const float (&f)[9]) __attribute__((always_inline)) {
        to[4] = f[4];
        to[7] = lane_from_right(f[7]);
        to[8] = lane_from_left(f[8]);
    };
    // the populations a wall reflects into its own row
    auto reflect_up = [](float (&to)[9], const float (&f)[9]) __attribute__((always_inline)) {
        to[2] = f[4]; to[5] = f[7]; to[6] = f[8];
    };
    auto reflect_down = [](float (&to)[9], const float (&f)[9]) __attribute__((always_inline)) {
        to[4] = f[2]; to[7] = f[5]; to[8] = f[6];
    };

    bool bad = false;
    // first step: rows r, r + DIR (pulled) and r + 2 DIR (in flight), psi windows of rows
    // r - DIR, r, r + DIR; second step: rows r - 2 DIR, r - DIR, r, psi windows of rows
    // r - 3 DIR, r - 2 DIR, r - DIR.  The loop is unrolled three times with the roles
    // rotated.
    float fa[9], fb[9], fc[9];
    float ga[9], gb[9], gc[9];
    Win wa{0.0f, 0.0f, 0.0f}, wb{0.0f, 0.0f, 0.0f}, wc{0.0f, 0.0f, 0.0f};
    Win va{0.0f, 0.0f, 0.0f}, vb{0.0f, 0.0f, 0.0f}, vc{0.0f, 0.0f, 0.0f};
    float ra = 0.0f, rb = 0.0f, rc = 0.0f;
    float sa = 0.0f, sb = 0.0f, sc = 0.0f;
    Sums f1{0.0f, 0.0f, 0.0f, 0.0f}, f2{0.0f, 0.0f, 0.0f, 0.0f};  // of rows r and r - 2 DIR
#pragma unroll
    for (int a = 0; a < 9; ++a) ga[a] = gb[a] = gc[a] = 0.0f;

    // walk position i is row o0 + DIR i; the first step starts two rows before the strip
    const int ahead = DIR > 0 ? y0 : k.ny - y1;
    const int is = WALLS ? -min(2, ahead) : -2;
    const int rs = o0 + DIR * is;
    const bool has_h = inside(rs - DIR);
    float pm = 0.0f;
    __builtin_amdgcn_s_setprio(kPrioPrologue);
    if (has_h) {
        pull_row<kStoreF32, WALLS>(fin, k, wrap(rs - DIR), xm, xc, xp, fb);
        pm = pseudopotential<PSI>(density(fb), k, bad);
    }
    pull_row<kStoreF32, WALLS>(fin, k, wrap(rs), xm, xc, xp, fa);
    pull_row<kStoreF32, WALLS>(fin, k, wrap(rs + DIR), xm, xc, xp, fb);
    __builtin_amdgcn_s_setprio(0);
    ra = density(fa, f1);
    const float p0 = pseudopotential<PSI>(ra, k, bad);
    if (!has_h) pm = p0;
    wa = window(pm);
    wb = window(p0);

    // Walk position i, row r.  f, fn, fq: first-step rows r, r + DIR, r + 2 DIR; u, v, w:
    // second-step rows r - 2 DIR, r - DIR, r; b, c, a: psi windows of rows r - DIR, r,
    // r + DIR; e, d, h: of the second step's rows r - 3 DIR, r - 2 DIR, r - DIR; q2, q1:
    // second-step densities of rows r - 2 DIR, r - DIR.
    auto row = [&](const int i, float (&f)[9], float (&fn)[9], float (&fq)[9], const float rho, float& rn,
                   const Win& b, const Win& c, Win& a, float (&u)[9], float (&v)[9], float (&w)[9],
                   const float q2, float& q1, const Win& e, Win& d, Win& h) __attribute__((always_inline)) {
        const int r = o0 + DIR * i;
        // Paces the workgroup: its waves, neighbours in x, stay on the same row, so that the
        // workgroup streams one wide stretch of each row at a time (16-row strips on
        // 8192 x 4096: 250 us per step with it, 285 us without; 8 waves per workgroup, 256 us
        // with 4, 260 us with 16).  No data is exchanged;
        // the hardware barrier counts only waves that have not ended, so waves of one
        // workgroup may walk strips of different heights.
        __builtin_amdgcn_s_barrier();
        Sums fn_sums{0.0f, 0.0f, 0.0f, 0.0f}, v_sums{0.0f, 0.0f, 0.0f, 0.0f};
        if (inside(r)) {
            __builtin_amdgcn_s_setprio(kPrioPrefetch);
            if (i <= n && inside(r + 2 * DIR)) pull_row<kStoreF32, WALLS>(fin, k, wrap(r + 2 * DIR), xm, xc, xp, fq);
            __builtin_amdgcn_s_setprio(0);
            if (inside(r + DIR)) {
                rn = density(fn, fn_sums);
                a = window(pseudopotential<PSI>(rn, k, bad));
            } else {
                a = c;  // mirror beyond a wall
            }
            collide_row(f, rho, f1, b, c, a);
            if (DIR > 0) move_down(v, f); else move_up(v, f);
            w[0] = f[0];
            w[1] = lane_from_left(f[1]);
            w[3] = lane_from_right(f[3]);
            if (WALLS && r == e0) { if (DIR > 0) reflect_up(w, f); else reflect_down(w, f); }
        }
        // second step: row r - DIR is complete
        const int q = r - DIR;
        if (i >= 0 && inside(q)) {
            bool bad2 = false;
            q1 = density(v, v_sums);
            h = window(pseudopotential<PSI>(q1, k, bad2));
            bad = bad || (bad2 && check);
            if (WALLS && q == e0) d = h;
        } else {
            h = d;  // mirror beyond a wall
        }
        if (i >= 2) {
            collide_row(u, q2, f2, e, d, h);
            if (live) {
                float* out = fout + (long long)(q - DIR) * k.row_stride;
#pragma unroll
                for (int a9 = 0; a9 < 9; ++a9) Codec<kStoreF32>::store(out, k, a9, xc, u[a9], 0.0f);
            }
        }
        // the populations of row r that move with the walk start row r + DIR, in the
        // registers that row r - 2 DIR has left
        if (DIR > 0) move_up(u, f); else move_down(u, f);
        if (WALLS && r == e1) { if (DIR > 0) reflect_down(w, f); else reflect_up(w, f); }
        f1 = fn_sums;
        f2 = v_sums;
    };
    for (int i = is; i < n + 2; i += 3) {
        row(i, fa, fb, fc, ra, rb, wa, wb, wc, ga, gb, gc, sa, sb, va, vb, vc);
        if (i + 1 >= n + 2) break;
        row(i + 1, fb, fc, fa, rb, rc, wb, wc, wa, gb, gc, ga, sb, sc, vb, vc, va);
        if (i + 2 >= n + 2) break;
        row(i + 2, fc, fa, fb, rc, ra, wc, wa, wb, gc, ga, gb, sc, sa, vc, va, vb);
    }
    if (bad) flag[0] = kFlagUnstable;
}

// Strip `tile` of a lattice stepped twice (k.tiles_x counts 58-column tiles); tiles in
// bands of `band` strips, as strip_tile.
template <bool WALLS, int PSI>
__device__ __forceinline__ void two_tile(const float* __restrict__ fin, float* __restrict__ fout,
                                         const StepConst& k, const int tile, const int lane, int* __restrict__ flag)
{
    const int band0 = (tile / (k.tiles_x * k.band)) * k.band;
    const int band_h = min(k.band, k.tiles_y - band0);
    const int r = tile - band0 * k.tiles_x;
    const int tx = r / band_h;
    const int ty = band0 + r % band_h;
    const int xs = tx * kTwoTileW - 3 + lane;
    const bool live = (lane >= 3) && (lane < kTwoTileW + 3) && (xs < k.nx);
    // sites whose second-step density is complete here
    const bool check = (lane >= 2) && (lane < kTwoTileW + 4) && (xs <= k.nx);
    int xci = xs < 0 ? xs + k.nx : (xs >= k.nx ? xs - k.nx : xs);
    if (xs > k.nx + 2) xci = 0;  // beyond the right halo: in-range dummy column, never stored
    const unsigned xc = (unsigned)xci * 4u;
    const unsigned xm = (unsigned)((xci == 0) ? k.nx - 1 : xci - 1) * 4u;
    const unsigned xp = (unsigned)((xci == k.nx - 1) ? 0 : xci + 1) * 4u;
    // Strips of odd index walk down and the others up: two strips that share a boundary are
    // at it at about the same time (250 us per step against 254 us walking one way).  A strip whose rows, with the four rows pulled beyond
    // each end, stay off the walls takes the walk without wall handling.
    const int y0 = ty * k.strip_rows;
    const bool off_walls = !WALLS || (y0 >= 4 && y0 + k.strip_rows + 4 <= k.ny);
    if (ty & 1) {
        if (off_walls) two_walk<false, PSI, -1>(fin, fout, k, ty, live, check, xm, xc, xp, flag);
        else two_walk<WALLS, PSI, -1>(fin, fout, k, ty, live, check, xm, xc, xp, flag);
    } else {
        if (off_walls) two_walk<false, PSI, 1>(fin, fout, k, ty, live, check, xm, xc, xp, flag);
        else two_walk<WALLS, PSI, 1>(fin, fout, k, ty, live, check, xm, xc, xp, flag);
    }
}

}  // namespace lbmp
