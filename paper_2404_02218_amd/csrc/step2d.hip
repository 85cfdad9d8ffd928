// The 2D sweep, one step per launch (k_step2d): a wave computes 1, 2 or 4 rows
// of a strip with every load issued before the first use and the x taps from
// its neighbouring lanes, so a launch on a small grid costs one memory latency.
// In place over prev for the wave (only a point's own prev is read).  The four
// waves of a workgroup take consecutive row groups of one strip.  Sources are
// injected and receivers recorded in the launch: their lists are read beside
// the field, so that no chain of loads follows the arithmetic (counted and
// loaded behind it, a step of 1120 x 1074 with 64 receivers, FP16, r = 4, took
// 5.7 us, now 5.3; 1092 x 1352 with 16, BF16, r = 2, 5.2 and 4.8).
//
// Points take the canonical operation order (device.hpp): the same bits as
// every other kernel.
#include "strip2d.hpp"

namespace stn {

namespace {

constexpr int kStepWaves = 4;

template <int MODE, int R, typename T, int ROWS>
__global__ __launch_bounds__(64 * kStepWaves) void k_step2d(M2View v, Coefs w, FastDiv strips, int row0) {
    using S = Storage<T>;
    using Raw = typename RawGroup<T>::type;
    constexpr int NQ = ROWS + 2 * R;
    constexpr bool WAVE = MODE != MODE_HEAT;
    __shared__ __attribute__((aligned(16))) float recrows[kStepWaves][ROWS][256];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    // the arguments' cache lines, all asked for at once
    asm volatile("" ::"s"(v.u), "s"(v.g.s[0]), "s"(v.nstrips), "s"(v.src.n), "s"(v.rec.n), "s"(w.cd0), "s"(row0));
    const int lb = xcd_remap(blockIdx.x, gridDim.x);
    const int group = (int)fdiv((uint32_t)lb, strips), strip = lb - group * v.nstrips;
    const int nx = v.g.n[2], ny = v.g.n[1];
    const int yb = (group * kStepWaves + wave) * ROWS;
    if (yb >= ny) return;
    const int ye = min(yb + ROWS, ny);
    const int X0 = strip * v.width - v.margin, x0 = X0 + 4 * lane;
    const int64_t sy = v.g.s[1];
    constexpr int kLead = 32;
    const int64_t base = v.g.origin - kLead;
    const T* const U = (const T*)v.u + base;
    const T* const P = (const T*)v.prev + base;
    const T* const B = (const T*)v.beta + base;
    const uint32_t xo = (uint32_t)(min(x0, (int)(v.g.rowlen - v.g.xlead) - 4) + kLead);

    Raw ru[NQ], rp[ROWS], rb[ROWS];
#pragma unroll
    for (int k = 0; k < NQ; k++) ru[k] = load4_raw<T, false>(U + (int64_t)min(yb - R + k, ny + R - 1) * sy + xo);
    if constexpr (WAVE) {
#pragma unroll
        for (int k = 0; k < ROWS; k++) {
            const int64_t o = (int64_t)min(yb + k, ny - 1) * sy;
            rp[k] = load4_raw<T, false>(P + o + xo);
            rb[k] = load4_raw<T, false>(B + o + xo);
        }
    }
    float dgx[4], dgz = 0.f;
    if constexpr (MODE == MODE_WAVE_DAMP) {
        dgz = ld_inv(v.damp);
#pragma unroll
        for (int i = 0; i < 4; i++) dgx[i] = v.damp[v.g.n[0] + ny + min(max(x0 + i, 0), nx - 1)];
    }
    // The strip's sources and receivers, 64 at a time, one per lane, picked by
    // row (-1 before the wave's rows, -2 behind them); the first ones are loaded
    // here, so that their chains of loads (list, entry, amount) run beside the
    // field's.  Of a longer list the wave looks for its own rows next, behind the
    // arithmetic, where it does not hold up the field's loads.  (It walked the
    // whole list before: with 4096 receivers on 1000^2, FP32, r = 4, a step took
    // 7.7 us, now 4.6.)
    int src_begin = 0, src_end = 0, src_row = -1, src_x = 0;
    double src_amt = 0.0;
    auto load_sources = [&](int from) {
        const int4 e = reinterpret_cast<const int4*>(v.src.zyx4)[min(from + lane, src_end - 1)];
        const bool in = from + lane < src_end && e.y >= yb && e.y < ye;
        src_row = in ? e.y - yb : e.y < ye ? -1 : -2;
        src_x = e.z - X0;
        if (in) src_amt = v.src.amp[(int64_t)row0 * v.src.n + e.w] * (v.src.scale ? v.src.scale[e.w] : 1.0);
    };
    if (v.src.n > 0) {
        src_begin = ld_inv(v.src.tile_begin + strip);
        src_end = ld_inv(v.src.tile_begin + strip + 1);
        if (src_begin < src_end) load_sources(src_begin);
    }
    int rec_begin = 0, rec_end = 0, rec_row = -1, rec_x = 0, rec_at = 0;
    auto load_receivers = [&](int from) {
        const int4 e = reinterpret_cast<const int4*>(v.rec.zyx4)[min(from + lane, rec_end - 1)];
        rec_row = from + lane < rec_end && e.y >= yb && e.y < ye ? e.y - yb : e.y < ye ? -1 : -2;
        rec_x = e.z - X0;
        rec_at = e.w;
    };
    if (v.rec.n > 0) {
        rec_begin = ld_inv(v.rec.tile_begin + strip);
        rec_end = ld_inv(v.rec.tile_begin + strip + 1);
        if (rec_begin < rec_end) load_receivers(rec_begin);
    }

    float q[NQ][4], o[ROWS][4];
#pragma unroll
    for (int k = 0; k < NQ; k++) {
        const float4 u = widen4<T>(ru[k]);
#pragma unroll
        for (int i = 0; i < 4; i++) q[k][i] = comp(u, i);
    }
#pragma unroll
    for (int r = 0; r < ROWS; r++) {
        const float(&c)[4] = q[R + r];
        float xv[12];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            xv[i] = from_left(c[i]);
            xv[4 + i] = c[i];
            xv[8 + i] = from_right(c[i]);
        }
        float4 p4 = make_float4(0.f, 0.f, 0.f, 0.f), b4 = p4;
        if constexpr (WAVE) {
            p4 = widen4<T>(rp[r]);
            b4 = widen4<T>(rb[r]);
        }
        float dgy = 0.f;
        if constexpr (MODE == MODE_WAVE_DAMP) dgy = dgz + ld_inv(v.damp + v.g.n[0] + min(yb + r, ny - 1));
#pragma unroll
        for (int i = 0; i < 4; i++) {
            float m[R], n[R];
            float acc = w.cd0 * c[i];
#pragma unroll
            for (int k = 1; k <= R; k++) {
                m[k - 1] = q[R + r - k][i];
                n[k - 1] = q[R + r + k][i];
            }
            acc = axis_sum<R>(acc, w, m, n);
#pragma unroll
            for (int k = 1; k <= R; k++) {
                m[k - 1] = xv[4 + i - k];
                n[k - 1] = xv[4 + i + k];
            }
            acc = axis_sum<R>(acc, w, m, n);
            if constexpr (MODE == MODE_WAVE_DAMP)
                o[r][i] = damped_update(acc, c[i], comp(p4, i), comp(b4, i), dgy + dgx[i]);
            else
                o[r][i] = time_update<MODE>(acc, c[i], comp(p4, i), comp(b4, i));
        }
    }
    // the next entries of a list, or `end`
    auto next = [&](const int* zyx4, int from, int end, int last_row) {
        if (from + 64 >= end || last_row == -2) return end;
        int stop = end;
        return near_first(zyx4, from + 64, stop, 0, yb);
    };
    for (int from = src_begin; from < src_end;
         from = next(v.src.zyx4, from, src_end, __builtin_amdgcn_readlane(src_row, 63))) {
        if (from > src_begin) load_sources(from);
        const int lo = __double2loint(src_amt), hi = __double2hiint(src_amt);
        for (uint64_t mine = __ballot(src_row >= 0); mine; mine &= mine - 1) {   // in the list's order
            const int k = __builtin_ctzll(mine);
            const int r1 = __builtin_amdgcn_readlane(src_row, k), i1 = __builtin_amdgcn_readlane(src_x, k) - 4 * lane;
            const double a = __hiloint2double(__builtin_amdgcn_readlane(hi, k), __builtin_amdgcn_readlane(lo, k));
#pragma unroll
            for (int r = 0; r < ROWS; r++)
                if (r == r1) {
#pragma unroll
                    for (int i = 0; i < 4; i++)
                        if (i == i1) o[r][i] = inject<T>(o[r][i], a);
                }
        }
    }
    bool put = false;
    for (int from = rec_begin; from < rec_end;
         from = next(v.rec.zyx4, from, rec_end, __builtin_amdgcn_readlane(rec_row, 63))) {
        if (from > rec_begin) load_receivers(from);
        if (!__ballot(rec_row >= 0)) continue;
        if (!put) {
#pragma unroll
            for (int r = 0; r < ROWS; r++)
                *reinterpret_cast<float4*>(&recrows[wave][r][4 * lane]) =
                    make_float4(through<T>(o[r][0]), through<T>(o[r][1]), through<T>(o[r][2]), through<T>(o[r][3]));
            wave_lds_fence();
            put = true;
        }
        if (rec_row >= 0) v.rec.trace[(int64_t)row0 * v.rec.n + rec_at] = (double)recrows[wave][rec_row][rec_x];
    }
    if (4 * lane < v.margin || 4 * lane >= v.margin + v.width || x0 >= nx) return;
#pragma unroll
    for (int r = 0; r < ROWS; r++) {
        if (yb + r >= ye) break;
        T* const O = (T*)v.out + base + (int64_t)(yb + r) * sy + xo;
        if (x0 + 3 < nx) {
            S::store4(O, make_float4(o[r][0], o[r][1], o[r][2], o[r][3]));
        } else {
#pragma unroll
            for (int i = 0; i < 4; i++)
                if (x0 + i < nx) S::store(O + i, o[r][i]);
        }
    }
}

template <int MODE, int R, typename T, int ROWS>
hipError_t step_launch(const M2View& v, const Coefs& w, int row0, hipStream_t s) {
    constexpr int rows = ROWS * kStepWaves;
    const int64_t nb = (int64_t)v.nstrips * ((v.g.n[1] + rows - 1) / rows);
    if (nb == 0) return hipSuccess;
    if (nb > INT_MAX) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((k_step2d<MODE, R, T, ROWS>), dim3((unsigned)nb), dim3(64 * kStepWaves), 0, s, v, w,
                       fast_div((uint32_t)v.nstrips), row0);
    return hipGetLastError();
}

// Rows per wave.  While the chip is not full, the rows of a wave are one after
// another on its critical path; once it is, more rows share the y taps.  A
// step of an FP32 / FP16 wave, r = 4, in us with 1, 2 and 4 rows: 256^2 4.9,
// 5.4, 6.0 / 4.9, 5.3, 5.7; 1000^2 6.7, 6.6, 7.1 / 6.5, 6.2, 6.6; 2048^2 13.7,
// 14.1, 14.3 / 12.1, 10.2, 9.3 (each about 1.5 us over a replayed graph).
template <int MODE, int R, typename T>
hipError_t step_rows(const M2View& v, const Coefs& w, int row0, hipStream_t s) {
    const int64_t waves = (int64_t)v.nstrips * v.g.n[1];
    if (waves <= 4096) return step_launch<MODE, R, T, 1>(v, w, row0, s);
    if (waves <= 12288) return step_launch<MODE, R, T, 2>(v, w, row0, s);
    return step_launch<MODE, R, T, 4>(v, w, row0, s);
}

template <int MODE, typename T>
hipError_t step_r(int radius, const M2View& v, const Coefs& w, int row0, hipStream_t s) {
    switch (radius) {
        case 1: return step_rows<MODE, 1, T>(v, w, row0, s);
        case 2: return step_rows<MODE, 2, T>(v, w, row0, s);
        case 3: return step_rows<MODE, 3, T>(v, w, row0, s);
        case 4: return step_rows<MODE, 4, T>(v, w, row0, s);
    }
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t step_m(int mode, int radius, const M2View& v, const Coefs& w, int row0, hipStream_t s) {
    if (mode == MODE_HEAT) return step_r<MODE_HEAT, T>(radius, v, w, row0, s);
    if (mode == MODE_WAVE) return step_r<MODE_WAVE, T>(radius, v, w, row0, s);
    if constexpr (std::is_same<T, float>::value)
        if (mode == MODE_WAVE_DAMP) return step_r<MODE_WAVE_DAMP, T>(radius, v, w, row0, s);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_step2d(int mode, int radius, int dtype, const M2View& v, const Coefs& w, int row0, hipStream_t s) {
    switch (dtype) {
        case DT_F32: return step_m<float>(mode, radius, v, w, row0, s);
        case DT_BF16: return step_m<bf16>(mode, radius, v, w, row0, s);
        case DT_F16: return step_m<f16>(mode, radius, v, w, row0, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace stn
