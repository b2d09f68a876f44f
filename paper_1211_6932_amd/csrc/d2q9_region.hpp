// d2q9_region.hpp -- several D2Q9 time steps in one launch, by regions held in LDS.
#pragma once

#include "d2q9_core.hpp"

namespace lbmp {

// A workgroup loads a region of 32 x 32 sites, one per thread, and advances it `steps` time
// steps with psi and the moving populations exchanged through LDS.  Every step the sites next
// to the region's edge lose a neighbour they need (the pull reaches 1, the force `reach`),
// so after the last step the inner 32 - 2 halo sites a side, halo = (reach + 1) steps - 1,
// are complete and are stored; the regions overlap by the rest.  Each site's arithmetic, and
// for the 16-bit encodings the rounding of every stored population, is that of strip_walk:
// the result is bitwise that of single steps.
//
// What bounds it: a small lattice leaves most of the chip idle, and a step is one launch, one
// round trip to memory and one serial walk; here these are shared by `steps` steps, at the
// price of computing the overlap several times on compute units that had nothing to do.
// Measured on 128 x 128 sites, FP32, per step: 4.07 us by strips of two steps per launch,
// 2.03 us with 6 steps per region launch (12.2 us: about 4 us for the launch and the load,
// the rest the 11 exchanges through LDS, two a step but for the last step's populations,
// each a barrier of 16 wavefronts).
//
// Registers: 64 per lane, so that two workgroups share a compute unit (512 x 512 in 3 steps:
// 5.8 us per step, 6.5 us with 128 registers; a lattice with one region per unit loses 5 %).
// The FP16-dest encoding and the 24-site stencil would spill at 64 and have 128.
constexpr int kRegion = 32;
constexpr int kRegionThreads = kRegion * kRegion;
constexpr int region_waves_per_simd(int store, int stencil)
{
    return store == kStoreF16Dest || stencil == kStencilMultirange ? 4 : 8;
}

template <int S, bool WALLS, int PSI, int STENCIL>
__global__ __launch_bounds__(kRegionThreads, region_waves_per_simd(S, STENCIL)) void d2q9_region(
    const typename Codec<S>::T* __restrict__ fin, typename Codec<S>::T* __restrict__ fout, StepConst k, int steps,
    int* __restrict__ flag)
{
    using C = Codec<S>;
    using T = typename C::T;
    constexpr bool local = S == kStoreF16Local || S == kStoreBF16Local;
    constexpr int reach = STENCIL == kStencilMultirange ? 2 : 1;
    // the density's partial sums kept over the exchange of psi (600 x 250 with walls 3.95 us per
    // step, 4.15 us recomputed); the 24-site stencil needs the registers (400 x 300 4.73 / 4.55 us)
    constexpr bool keep = STENCIL == kStencilNearest;
    // a border around the region's sites keeps every neighbour at a fixed distance (what is
    // read from it is not used)
    constexpr int P = kRegion + 2 * reach, F = kRegion + 2;
    __shared__ float sp_[P][P];                      // psi
    __shared__ float sf_[8][F][F];                   // populations 1 .. 8 on their way
    __shared__ float si_[C::kDestScaled ? F : 1][F];  // 1 / rhohat
    const int lx = threadIdx.x & (kRegion - 1), ly = threadIdx.x / kRegion;
    const int halo = (reach + 1) * steps - 1, out = kRegion - 2 * halo;
    const int tx = blockIdx.x % k.tiles_x, ty = blockIdx.x / k.tiles_x;
    // lattice site of this thread (regions of tiny lattices may wrap around several times)
    int x = (tx * out - halo + lx) % k.nx;
    if (x < 0) x += k.nx;
    int y = ty * out - halo + ly;
    const bool in = !WALLS || (y >= 0 && y < k.ny);  // rows beyond a wall do not exist
    if (WALLS) {
        y = in ? y : 0;
    } else {
        y %= k.ny;
        if (y < 0) y += k.ny;
    }
    const bool bot = WALLS && y == 0, top = WALLS && y == k.ny - 1;
    // rows below and above; beyond a wall the own row
    const int yd = bot ? ly : ly - 1, yu = top ? ly : ly + 1;
    auto sp = [&](const int row, const int col) __attribute__((always_inline)) -> float& { return sp_[row + reach][col + reach]; };
    auto sf = [&](const int a, const int row, const int col) __attribute__((always_inline)) -> float& {
        return sf_[a - 1][row + 1][col + 1];
    };
    auto si = [&](const int row, const int col) __attribute__((always_inline)) -> float& { return si_[row + 1][col + 1]; };

    // Element of population slot a of lattice site (xx, yy), as a byte offset (the host runs
    // this kernel on lattices whose state stays below 2 GiB).
    auto offset = [&](const int yy, const int a, const int xx) __attribute__((always_inline)) {
        return ((unsigned)yy * (unsigned)k.row_stride + (unsigned)(a * k.pitch + xx)) * (unsigned)sizeof(T);
    };
    auto density_offset = [&](const int yy, const int xx) __attribute__((always_inline)) {
        return offset(yy, 9, 0) + (unsigned)xx * (local ? 4u : (unsigned)sizeof(T));
    };
    // stored value of slot a decoded at its source site (the destination-scaled encoding is
    // finished by the puller)
    auto load = [&](const int yy, const int a, const int xx) __attribute__((always_inline)) {
        const float v = static_cast<float>(ld<T>(fin, 0, offset(yy, a, xx)));
        if constexpr (local) return ld<float>(fin, 0, density_offset(yy, xx)) * (lattice_weight(a) + v);
        else if constexpr (S == kStoreF32 || C::kDestScaled) return v;
        else return v + k.off[a];
    };
    auto scale = [&](float (&f)[9], const float sc) __attribute__((always_inline)) {
        const float sw0 = sc * (4.0f / 9.0f), sw1 = sc * (1.0f / 9.0f), sw2 = sc * (1.0f / 36.0f);
        f[0] = fmaf(f[0], sc, sw0);
#pragma unroll
        for (int a = 1; a < 5; ++a) f[a] = fmaf(f[a], sc, sw1);
#pragma unroll
        for (int a = 5; a < 9; ++a) f[a] = fmaf(f[a], sc, sw2);
    };

    float f[9];
    {
        const int xm = x == 0 ? k.nx - 1 : x - 1, xp = x == k.nx - 1 ? 0 : x + 1;
        const int ym = bot ? y : (y == 0 ? k.ny - 1 : y - 1), yp = top ? y : (y == k.ny - 1 ? 0 : y + 1);
        f[0] = load(y, 0, x);
        f[1] = load(y, 1, xm);
        f[3] = load(y, 3, xp);
        f[2] = load(ym, bot ? 4 : 2, x);
        f[5] = load(ym, bot ? 7 : 5, bot ? x : xm);
        f[6] = load(ym, bot ? 8 : 6, bot ? x : xp);
        f[4] = load(yp, top ? 2 : 4, x);
        f[7] = load(yp, top ? 5 : 7, top ? x : xp);
        f[8] = load(yp, top ? 6 : 8, top ? x : xm);
        if constexpr (C::kDestScaled) scale(f, static_cast<float>(ld<__bf16>(fin, 0, density_offset(y, x))));
    }

    // rows of the region this wavefront holds: the first one
    const int row0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * (kWave / kRegion);
    bool bad = false;
    for (int s = 0; s < steps; ++s) {
        // complete populations: m sites or more from the region's edge
        const int m = (reach + 1) * s;
        const bool busy = row0 + kWave / kRegion > m && row0 < kRegion - m;
        float r = 0.0f;
        Sums sums{0.0f, 0.0f, 0.0f, 0.0f};
        if (busy) {
            if constexpr (keep) r = density(f, sums);
            else r = density(f);
            bool b = false;
            sp(ly, lx) = pseudopotential<PSI>(r, k, b);
            bad = bad || (b && in && min(lx, ly) >= m && max(lx, ly) < kRegion - m);
            if constexpr (C::kDestScaled) si(ly, lx) = recip(C::round_scale(r));
        }
        __syncthreads();
        if (busy) {
            float Fx, Fy, Fs2;
            if constexpr (STENCIL == kStencilMultirange) {
                float W[5][5];
#pragma unroll
                for (int j = 0; j < 5; ++j) {
                    int row = ly + j - 2;
                    if (WALLS) row = min(max(row, ly - y), ly + k.ny - 1 - y);
#pragma unroll
                    for (int c = 0; c < 5; ++c) W[j][c] = sp(row, lx + c - 2);
                }
                force_stencil_mr(W, k, Fx, Fy, Fs2);
            } else {
                auto row = [&](const int y9) __attribute__((always_inline)) {
                    return psi_row(sp(y9, lx - 1), sp(y9, lx), sp(y9, lx + 1));
                };
                force_stencil(row(yd), row(ly), row(yu), k, Fx, Fy, Fs2);
            }
            float jx, jy;
            momentum(f, jx, jy);
            const float inv_rho = recip(r);
            const float vx = fmaf(0.5f, Fx, jx) * inv_rho, vy = fmaf(0.5f, Fy, jy) * inv_rho;
            if constexpr (!keep) density(f, sums);
            collide(f, r, sums, vx, vy, Fx, Fy, Fs2, k, Shear{k.a_nu_l, k.a_nu_g, k.b_nu_l, k.b_nu_g});
        }
        // what the encoding stores, still as T
        T g[9];
        if (busy) {
            if constexpr (C::kDestScaled) {
                // 1/rhohat of the site that pulls population a next (as strip_walk)
                const float own = si(ly, lx);
                const float id[9] = {own, si(ly, lx + 1), si(yu, lx), si(ly, lx - 1), si(yd, lx),
                                     top ? own : si(yu, lx + 1), top ? own : si(yu, lx - 1), bot ? own : si(yd, lx - 1),
                                     bot ? own : si(yd, lx + 1)};
#pragma unroll
                for (int a = 0; a < 9; ++a) g[a] = static_cast<T>(fmaf(f[a], id[a], -lattice_weight(a)));
            } else if constexpr (local) {
                const float inv_rho = recip(r);
#pragma unroll
                for (int a = 0; a < 9; ++a) g[a] = static_cast<T>(fmaf(f[a], inv_rho, -lattice_weight(a)));
            } else if constexpr (S == kStoreF32) {
#pragma unroll
                for (int a = 0; a < 9; ++a) g[a] = f[a];
            } else {
#pragma unroll
                for (int a = 0; a < 9; ++a) g[a] = static_cast<T>(f[a] - k.off[a]);
            }
        }
        if (s + 1 == steps) {
            const int xs = tx * out + lx - halo, ys = ty * out + ly - halo;
            if (lx >= halo && lx < halo + out && ly >= halo && ly < halo + out && xs < k.nx && ys < k.ny) {
#pragma unroll
                for (int a = 0; a < 9; ++a) st<T>(fout, 0, offset(y, a, x), g[a]);
                if constexpr (local) st<float>(fout, 0, density_offset(y, x), r);
                if constexpr (C::kDestScaled) st<__bf16>(fout, 0, density_offset(y, x), static_cast<__bf16>(r));
            }
            break;
        }
        if (busy) {
            // decoded as `load` would
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                const float v = static_cast<float>(g[a]);
                if constexpr (local) f[a] = r * (lattice_weight(a) + v);
                else if constexpr (S == kStoreF32 || C::kDestScaled) f[a] = v;
                else f[a] = v + k.off[a];
            }
#pragma unroll
            for (int a = 1; a < 9; ++a) sf(a, ly, lx) = f[a];
        }
        __syncthreads();
        if (busy) {
            f[1] = sf(1, ly, lx - 1);
            f[3] = sf(3, ly, lx + 1);
            f[2] = sf(bot ? 4 : 2, yd, lx);
            f[5] = sf(bot ? 7 : 5, yd, bot ? lx : lx - 1);
            f[6] = sf(bot ? 8 : 6, yd, bot ? lx : lx + 1);
            f[4] = sf(top ? 2 : 4, yu, lx);
            f[7] = sf(top ? 5 : 7, yu, top ? lx : lx + 1);
            f[8] = sf(top ? 6 : 8, yu, top ? lx : lx - 1);
            if constexpr (C::kDestScaled) scale(f, C::round_scale(r));
        }
    }
    if (bad) flag[0] = kFlagUnstable;
}

}  // namespace lbmp
