// Multi-step 2D heat sweep (FP32, fixed halo).  A 2D field of a few hundred
// points per side sits in L2, so a sweep per launch is bound by launch
// latency, not by memory.  Here a workgroup loads its TX x TY tile plus a
// halo of at least R*T points and takes up to T steps; step s is valid on the
// tile grown by R*(T-s) points.  Points outside the interior keep the halo of
// the buffer their level would be in, which is the value two steps back.  The
// tiles overlap by the halo and recompute it (overlapped
// temporal blocking, the related work of Section 7).
//
// The region lives in registers: a lane owns H consecutive rows of C adjacent
// columns, so the y taps are registers except at a lane's first and last
// rows, which it exchanges with the groups above and below through LDS (one
// barrier a step), and the x taps come from the neighbouring lanes by
// wavefront shifts.  A lone wave issues an instruction every 8 cycles, so 16
// waves share a region (few rows each), though fewer would exchange less.
//
// With every point in LDS, a step was five LDS reads and some forty
// instructions of addresses and bounds per point; now nine.  us a step of runs
// of 100, before / now: r = 1, 8 steps on 16 x 16 tiles 256^2 0.67 / 0.61, 16
// steps on 32 x 32 256^2 0.89 / 0.68, 512^2 1.04 / 0.72, 1000^2 2.47 / 1.61; r =
// 2, 8 steps on 32 x 32 512^2 1.35 / 1.11, 1000^2 3.38 / 2.54.  A launch with a
// load and a store takes 2.4 of the 5 us of 8 steps at 256^2.
//
// Each point is evaluated in the canonical order of the plain sweep (centre, y
// pairs, x pairs), so T steps here equal T plain sweeps bit for bit.
#include "strip2d.hpp"

namespace stn {

namespace {

// Lanes across (LX) with C columns each, row groups of H >= R rows per lane,
// waves.  Tiles up to 32 points wide with their halo take half a wave across.
template <int R, int T, int TX, int TY>
struct Heat2dTile {
    static constexpr int EX = TX + 2 * R * T, EY = TY + 2 * R * T;
    static constexpr int LX = EX <= 32 ? 32 : 64, C = EX <= 64 ? 1 : 2;
    static constexpr int WAVES = EX * EY <= 1024 && R > 1 ? 8 : 16;
    static constexpr int G = WAVES * 64 / LX;         // row groups
    static constexpr int H = (EY + G - 1) / G;        // rows per lane
    static constexpr int HX = (LX * C - TX) / 2;      // columns left of the tile
    static constexpr int HY = R * T;                  // rows above it
    static constexpr int W = LX * C;
    static_assert(H >= R && HX >= R * T && G * H >= EY, "a lane's rows reach its neighbours' taps; the halo fits");
};

template <int R, int T, int TX, int TY>
__global__ __launch_bounds__((64 * Heat2dTile<R, T, TX, TY>::WAVES)) void k_heat2d_tb(const float* in, float* out,
                                                                                  const float* halo0, const float* halo1,
                                                                                  Grid3 g, Coefs w, int steps) {
    using Z = Heat2dTile<R, T, TX, TY>;
    constexpr int LX = Z::LX, C = Z::C, G = Z::G, H = Z::H, W = Z::W;
    // the first and last R rows of every group, for two steps
    __shared__ float edge[2][G][2][R][W];
    const int lx = threadIdx.x % LX, grp = threadIdx.x / LX;
    const int nx = g.n[2], ny = g.n[1];
    const int ntx = (nx + TX - 1) / TX;
    const int X0 = (int)(blockIdx.x % ntx) * TX - Z::HX, Y0 = (int)(blockIdx.x / ntx) * TY - Z::HY;
    const int64_t sy = g.s[1];
    const int x = X0 + C * lx, y = Y0 + grp * H;
    const float* U = in + g.origin;
    auto outside = [&](int r, int c) { return y + r < 0 || y + r >= ny || x + c < 0 || x + c >= nx; };
    float v[H][C], hv[2][H][C];
#pragma unroll
    for (int r = 0; r < H; r++)
#pragma unroll
        for (int c = 0; c < C; c++) {
            v[r][c] = hv[0][r][c] = hv[1][r][c] = 0.f;
            if (!outside(r, c)) v[r][c] = U[(int64_t)(y + r) * sy + x + c];
        }
    // where a point lies outside the interior, hv[0] holds its value at this
    // level and every other one after it, hv[1] that of the levels between
    const bool border = X0 < 0 || Y0 < 0 || X0 + W > nx || Y0 + G * H > ny;   // uniform
    bool off[H][C];
#pragma unroll
    for (int r = 0; r < H; r++)
#pragma unroll
        for (int c = 0; c < C; c++) off[r][c] = outside(r, c);
    if (border) {
#pragma unroll
        for (int r = 0; r < H; r++)
#pragma unroll
            for (int c = 0; c < C; c++)
                if (off[r][c] && y + r >= -R && y + r < ny + R && x + c >= -R && x + c < nx + R) {
                    const int64_t o = g.origin + (int64_t)(y + r) * sy + x + c;
                    v[r][c] = hv[0][r][c] = halo0[o];
                    hv[1][r][c] = halo1[o];
                }
    }
    const int up = grp > 0 ? grp - 1 : grp, dn = grp + 1 < G ? grp + 1 : grp;
    // one step; `next` is the parity of the level it makes
    auto step = [&](auto next_c) __attribute__((always_inline)) {
        constexpr int next = decltype(next_c)::value;
        auto& E = edge[next];
#pragma unroll
        for (int k = 0; k < R; k++)
#pragma unroll
            for (int c = 0; c < C; c++) {
                E[grp][0][k][C * lx + c] = v[k][c];
                E[grp][1][k][C * lx + c] = v[H - R + k][c];
            }
        // rows y - R .. y + H - 1 + R of this lane's columns (past the
        // region's ends the group's own rows stand in: not valid any more)
        float q[H + 2 * R][C], n[H][C];
#pragma unroll
        for (int r = 0; r < H; r++)
#pragma unroll
            for (int c = 0; c < C; c++) q[R + r][c] = v[r][c];
        auto row = [&](int r) __attribute__((always_inline)) {
            // columns -R .. C - 1 + R of the row
            float xv[C + 2 * R];
#pragma unroll
            for (int c = 0; c < C; c++) xv[R + c] = q[R + r][c];
            if constexpr (C == 1) {
                float l = q[R + r][0], m = q[R + r][0];
#pragma unroll
                for (int k = 1; k <= R; k++) {
                    xv[R - k] = l = from_left(l);
                    xv[R + k] = m = from_right(m);
                }
            } else {
#pragma unroll
                for (int k = 1; k <= R; k++) {
                    xv[R - k] = from_left(q[R + r][C - k]);
                    xv[R + C - 1 + k] = from_right(q[R + r][k - 1]);
                }
            }
#pragma unroll
            for (int c = 0; c < C; c++) {
                const float ctr = xv[R + c];
                float acc = w.cd0 * ctr, m[R], p[R];
#pragma unroll
                for (int k = 1; k <= R; k++) {
                    m[k - 1] = q[R + r - k][c];
                    p[k - 1] = q[R + r + k][c];
                }
                acc = axis_sum<R>(acc, w, m, p);
#pragma unroll
                for (int k = 1; k <= R; k++) {
                    m[k - 1] = xv[R + c - k];
                    p[k - 1] = xv[R + c + k];
                }
                acc = axis_sum<R>(acc, w, m, p);
                n[r][c] = time_update<MODE_HEAT>(acc, ctr, 0.f, 0.f);
            }
        };
        // the rows that need no other group's go before the barrier
#pragma unroll
        for (int r = R; r < H - R; r++) row(r);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < R; k++)
#pragma unroll
            for (int c = 0; c < C; c++) {
                q[k][c] = E[up][1][k][C * lx + c];
                q[H + R + k][c] = E[dn][0][k][C * lx + c];
            }
#pragma unroll
        for (int r = 0; r < H; r++)
            if (r < R || r >= H - R) row(r);
#pragma unroll
        for (int r = 0; r < H; r++)
#pragma unroll
            for (int c = 0; c < C; c++) v[r][c] = n[r][c];
        if (border) {
#pragma unroll
            for (int r = 0; r < H; r++)
#pragma unroll
                for (int c = 0; c < C; c++)
                    if (off[r][c]) v[r][c] = hv[next][r][c];
        }
    };
    for (int s = 0; s + 1 < steps; s += 2) {
        step(std::integral_constant<int, 1>{});
        step(std::integral_constant<int, 0>{});
    }
    if (steps & 1) step(std::integral_constant<int, 1>{});
    float* O = out + g.origin;
#pragma unroll
    for (int r = 0; r < H; r++)
#pragma unroll
        for (int c = 0; c < C; c++) {
            const int ly = grp * H + r - Z::HY, lxx = C * lx + c - Z::HX;
            if (ly >= 0 && ly < TY && lxx >= 0 && lxx < TX && y + r < ny && x + c < nx)
                O[(int64_t)(y + r) * sy + x + c] = v[r][c];
        }
}

template <int R, int T, int TX, int TY>
hipError_t launch_cfg(const float* in, float* out, const float* halo0, const float* halo1,
                      const Grid3& g, const Coefs& w, int steps, hipStream_t s) {
    const int64_t nb = (int64_t)((g.n[2] + TX - 1) / TX) * ((g.n[1] + TY - 1) / TY);
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL((k_heat2d_tb<R, T, TX, TY>), dim3((unsigned)nb), dim3(64 * Heat2dTile<R, T, TX, TY>::WAVES), 0, s,
                       in, out, halo0, halo1, g, w, steps);
    return hipGetLastError();
}

template <int R>
hipError_t launch_r(int cfg, const float* in, float* out, const float* halo0, const float* halo1,
                      const Grid3& g, const Coefs& w, int steps, hipStream_t s) {
    static_assert(sizeof(kHeat2dCfgs) / sizeof(kHeat2dCfgs[0]) == 4, "one case per configuration");
    switch (cfg) {
        case 0: return launch_cfg<R, kHeat2dCfgs[0].t, kHeat2dCfgs[0].tx, kHeat2dCfgs[0].ty>(in, out, halo0, halo1, g, w, steps, s);
        case 1: return launch_cfg<R, kHeat2dCfgs[1].t, kHeat2dCfgs[1].tx, kHeat2dCfgs[1].ty>(in, out, halo0, halo1, g, w, steps, s);
        case 2: return launch_cfg<R, kHeat2dCfgs[2].t, kHeat2dCfgs[2].tx, kHeat2dCfgs[2].ty>(in, out, halo0, halo1, g, w, steps, s);
        case 3: return launch_cfg<R, kHeat2dCfgs[3].t, kHeat2dCfgs[3].tx, kHeat2dCfgs[3].ty>(in, out, halo0, halo1, g, w, steps, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_heat2d_tb(int cfg, int radius, const float* in, float* out, const float* halo0, const float* halo1,
                            const Grid3& g, const Coefs& w, int steps, hipStream_t s) {
    if (cfg < 0 || cfg >= kNumHeat2dCfgs || steps < 1 || steps > kHeat2dCfgs[cfg].t) return hipErrorInvalidValue;
    if (radius == 1) return launch_r<1>(cfg, in, out, halo0, halo1, g, w, steps, s);
    if (radius == 2) return launch_r<2>(cfg, in, out, halo0, halo1, g, w, steps, s);
    return hipErrorInvalidValue;
}

}  // namespace stn
