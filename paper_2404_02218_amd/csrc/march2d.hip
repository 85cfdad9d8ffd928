// The 2D sweep, T steps per launch (k_march2d), one wavefront per strip: for
// grids large enough to fill the chip with long chunks (step2d.hip takes one
// step per launch).
//
// A wave owns 256 consecutive x points (4 per lane) and marches down the rows
// of a chunk.  Stage s of T (step s of the launch) trails stage s - 1 by R
// rows: each stage keeps the last 2R + 1 rows of the level it reads in
// registers (the y taps), and takes the x taps from the neighbouring lanes by
// wavefront shifts, so there is no barrier and no shared plane.  The levels
// between the first and the last two never reach memory: a wave step moves
// 20 / T bytes of FP32 per point instead of 16, a heat step 8 / T.  beta is
// read once and waits in a ring of LDS rows, each lane reading back its own.
//
// The price is overlap: the outermost R T points of a strip on each side, and
// the 2 R T rows around a chunk, are computed again by the neighbours, with
// the same operations and so the same bits.
//
// Points outside the interior keep the halo of the buffer their level would be
// in: even steps that of one level buffer, odd steps that of the other.  That
// is the value two steps back at the same point, so it needs no case of its
// own after the first two levels.
//
// Every point takes the canonical operation order (device.hpp) and every level
// passes through the storage type, so T steps here equal T plain sweeps bit
// for bit.
//
// One thread per point with its taps from the caches, a launch each for the
// sources and the receivers, was bound by 4r + 1 scalar loads a point.  us a
// step before / now: FP32 wave r = 4, 8192^2 326 / 110 (T = 4: 95 VALU
// instructions per 4 points and step, issued 54% of the time at two waves per
// SIMD, 3.6 TB/s); r = 1, 8192^2 265 / 51 (T = 8); FP32 heat r = 1, 8192^2 230 /
// 33.
#include <algorithm>

#include "strip2d.hpp"

namespace stn {

namespace {

template <typename T, int MODE, int R, int NT>
struct March2D {
    static constexpr int Q = 2 * R + 1;
    // LDS of a wave, in 16-byte units: the staged sources and a row for the
    // receivers per stage, and NB rows of beta in the storage type
    static constexpr int NB = MODE != MODE_HEAT && NT > 1 ? (NT - 1) * R + 1 : 0;
    static constexpr int SRC = NT * kMarchRowSources, REC = NT * 64, BETA = NB * 64 * (int)sizeof(T) / 4;
    static constexpr size_t LDS_BYTES = 16 * (size_t)(SRC + REC + BETA);
};

struct StagedSource {
    double amount;
    int x, pad;
};

// One wave per workgroup (waves never meet, and LDS, which bounds the waves
// of a compute unit for deep passes, is handed out wave by wave).
template <int MODE, int R, typename T, int NT>
__global__ __launch_bounds__(64, 2) void k_march2d(M2View v, Coefs w, int row0) {
    using M = March2D<T, MODE, R, NT>;
    using S = Storage<T>;
    using Raw = typename RawGroup<T>::type;
    constexpr int Q = M::Q, NB = M::NB;
    constexpr bool WAVE = MODE != MODE_HEAT;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int lane = threadIdx.x;
    StagedSource* const staged = reinterpret_cast<StagedSource*>(lds);
    float* const recrow = lds + 4 * M::SRC;
    Raw* const bq = reinterpret_cast<Raw*>(recrow + 4 * M::REC) + lane;

    const int lb = xcd_remap(blockIdx.x, gridDim.x);
    const int strip = lb % v.nstrips, chunk = lb / v.nstrips;
    const int nx = v.g.n[2], ny = v.g.n[1];
    const int X0 = strip * v.width - v.margin, x0 = X0 + 4 * lane;
    const int yb = chunk * v.rows, ye = min(yb + v.rows, ny);
    const int64_t sy = v.g.s[1];
    // a lane's position counts from kLead elements before the interior, so
    // that it is a 32-bit offset from a wave-uniform row pointer
    constexpr int kLead = 32;
    const int64_t base = v.g.origin - kLead;
    const T* const U = (const T*)v.u + base;
    const T* const UH = (const T*)v.halo_even + base;
    const T* const P = (const T*)(WAVE ? v.prev : v.halo_odd) + base;
    const T* const PH = (const T*)v.halo_odd + base;
    const T* const B = (const T*)v.beta + base;
    const uint32_t xo = (uint32_t)(min(x0, (int)(v.g.rowlen - v.g.xlead) - 4) + kLead);

    bool in[4];
#pragma unroll
    for (int i = 0; i < 4; i++) in[i] = x0 + i >= 0 && x0 + i < nx;
    const bool edge = X0 < 0 || X0 + 256 > nx;   // some points of the strip lie outside (wave-uniform)
    // the points this wave stores: the strip without its margins
    const bool mine = 4 * lane >= v.margin && 4 * lane < v.margin + v.width && x0 < nx;
    const bool full = x0 + 3 < nx;
    float dgx[4], dgz = 0.f;
    if constexpr (MODE == MODE_WAVE_DAMP) {
        dgz = ld_inv(v.damp);
#pragma unroll
        for (int i = 0; i < 4; i++) dgx[i] = v.damp[v.g.n[0] + ny + min(max(x0 + i, 0), nx - 1)];
    }

    // a row as loaded: inside the interior from `a`, outside from `h`
    struct Pair {
        Raw a, h;
    };
    auto row_off = [&](int y) -> int64_t { return (int64_t)min(max(y, -R), ny + R - 1) * sy; };
    auto load = [&](const T* a, const T* h, int y, Pair& r) {
        const int64_t o = row_off(y);
        const T* const p = (y < 0 || y >= ny) ? h : a;
        r.a = load4_raw<T, false>(p + o + xo);
        if (edge) r.h = load4_raw<T, false>(h + o + xo);
    };
    auto widen = [&](const Pair& r, float (&o)[4]) {
        const float4 a = widen4<T>(r.a);
#pragma unroll
        for (int i = 0; i < 4; i++) o[i] = comp(a, i);
        if (edge) {
            const float4 h = widen4<T>(r.h);
#pragma unroll
            for (int i = 0; i < 4; i++)
                if (!in[i]) o[i] = comp(h, i);
        }
    };
    // heat reads the other buffer only where a point lies outside
    auto need_prev = [&](int y) { return WAVE || edge || y < 0 || y >= ny; };

    // Points of the strip, by row.  Lane s < NT stands for the sources of
    // stage s (margins included), lane 32 + s for the strip's own receivers
    // after that stage: ev_ptr is the next entry of its list and ev_y the
    // value of y (the newest row loaded) in whose iteration it is due.  So an
    // iteration asks once, for all stages, whether anything is due.
    int ev_ptr = 0, ev_y = INT_MAX, ev_cnt = 0;
    int src_end = 0, rec_end = 0;
    if (v.src.n > 0) {
        const int sb = ld_inv(v.src.tile_begin + strip);
        src_end = ld_inv(v.src.tile_begin + strip + 1);
        for (int s = 0; s < NT && sb < src_end; s++) {
            const int k = first_from(v.src.zyx4, sb, src_end, 0, yb - (NT - 1 - s) * R);
            if (lane == s && k < src_end) {
                ev_ptr = k;
                ev_y = v.src.zyx4[4 * k + 1] + (s + 1) * R;
            }
        }
    }
    if (v.rec.n > 0) {
        const int rb = ld_inv(v.rec.tile_begin + strip);
        rec_end = ld_inv(v.rec.tile_begin + strip + 1);
        if (rb < rec_end) {
            const int k = first_from(v.rec.zyx4, rb, rec_end, 0, yb);
            if (lane >= 32 && lane < 32 + NT && k < rec_end && v.rec.zyx4[4 * k + 1] < ye) {
                ev_ptr = k;
                ev_y = v.rec.zyx4[4 * k + 1] + (lane - 31) * R;
            }
        }
    }
    // the due sources of every stage into LDS (at most kMarchRowSources a row)
    auto stage_sources = [&](unsigned due, int y) {
        for (; due; due &= due - 1) {
            const int s = __builtin_ctz(due);
            const int k = __builtin_amdgcn_readlane(ev_ptr, s), e = min(k + lane, src_end - 1);
            const int* q = v.src.zyx4 + 4 * e;
            const bool now = k + lane < src_end && q[1] == y - (s + 1) * R;
            if (now) {
                StagedSource t;
                t.amount = v.src.amp[(int64_t)(row0 + s) * v.src.n + q[3]] * (v.src.scale ? v.src.scale[q[3]] : 1.0);
                t.x = q[2];
                t.pad = 0;
                staged[s * kMarchRowSources + lane] = t;
            }
            const int cnt = __popcll(__ballot(now));
            if (lane == s) {
                ev_cnt = cnt;
                ev_ptr = k + cnt;
                ev_y = k + cnt < src_end ? v.src.zyx4[4 * (k + cnt) + 1] + (s + 1) * R : INT_MAX;
            }
        }
        wave_lds_fence();
    };
    // the due receivers, from the rows the stages left in LDS
    auto record = [&](unsigned due, int y) {
        wave_lds_fence();
        for (; due; due &= due - 1) {
            const int s = __builtin_ctz(due);
            int k = __builtin_amdgcn_readlane(ev_ptr, 32 + s), cnt;
            do {
                const int e = min(k + lane, rec_end - 1);
                const int* q = v.rec.zyx4 + 4 * e;
                const bool now = k + lane < rec_end && q[1] == y - (s + 1) * R;
                if (now) v.rec.trace[(int64_t)(row0 + s) * v.rec.n + q[3]] = (double)recrow[256 * s + q[2] - X0];
                cnt = __popcll(__ballot(now));
                k += cnt;
            } while (cnt == 64);
            if (lane == 32 + s) {
                ev_ptr = k;
                ev_y = k < rec_end && v.rec.zyx4[4 * k + 1] < ye ? v.rec.zyx4[4 * k + 1] + (s + 1) * R : INT_MAX;
            }
        }
        wave_lds_fence();
    };
    auto store = [&](void* out, int y, const float (&o)[4]) {
        if (y < yb || y >= ye) return;
        if (!mine) return;
        T* const O = (T*)out + base + (int64_t)y * sy + xo;
        if (full) {
            S::store4(O, make_float4(o[0], o[1], o[2], o[3]));
        } else {
#pragma unroll
            for (int i = 0; i < 4; i++)
                if (x0 + i < nx) S::store(O + i, o[i]);
        }
    };

    // q[s]: the last Q rows of level s (s steps in); in an iteration the newest
    // row of level s is y - s R
    float q[NT][Q][4];
    Pair pro[2 * R], nu, np;
    Raw nb;
    int y = yb - NT * R + 2 * R;           // newest row of level 0
#pragma unroll
    for (int k = 0; k < 2 * R; k++) load(U, UH, y - 2 * R + k, pro[k]);
    load(U, UH, y, nu);
    if (need_prev(y - R)) load(P, PH, y - R, np);
    if constexpr (WAVE) nb = load4_raw<T, false>(B + row_off(y - R) + xo);
#pragma unroll
    for (int k = 0; k < 2 * R; k++) widen(pro[k], q[0][k]);
#pragma unroll
    for (int s = 1; s < NT; s++)
#pragma unroll
        for (int k = 0; k < Q; k++)
#pragma unroll
            for (int i = 0; i < 4; i++) q[s][k][i] = 0.f;

    const int yend = ye + NT * R;             // the last row loaded is yend - 1
    int bslot = 0;                            // LDS slot of this iteration's beta row
    auto step = [&](auto off_c) __attribute__((always_inline)) {
        // slot of logical row j (0 oldest .. 2R newest): (OFF + 1 + j) % Q
        constexpr int OFF = decltype(off_c)::value;
        auto at = [](int j) constexpr { return (OFF + 1 + j) % Q; };
        widen(nu, q[0][OFF]);
        float prev[4] = {0.f, 0.f, 0.f, 0.f};
        if (need_prev(y - R)) widen(np, prev);
        Raw b1 = {};
        if constexpr (WAVE) b1 = nb;
        // the next row's loads (past the chunk they repeat the last row)
        const int yn = min(y + 1, yend - 1);
        load(U, UH, yn, nu);
        if (need_prev(yn - R)) load(P, PH, yn - R, np);
        if constexpr (WAVE) {
            nb = load4_raw<T, false>(B + row_off(yn - R) + xo);
            if constexpr (NT > 1) bq[bslot * 64] = b1;
        }
        const uint64_t due = __ballot(ev_y == y);
        if ((unsigned)due) stage_sources((unsigned)due, y);
#pragma unroll
        for (int s = 1; s <= NT; s++) {
            const int yo = y - s * R;
            const float(&c)[4] = q[s - 1][at(R)];
            float xv[12];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                xv[i] = from_left(c[i]);
                xv[4 + i] = c[i];
                xv[8 + i] = from_right(c[i]);
            }
            float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
            if constexpr (WAVE) {
                if (s > 1) {
                    int k = bslot - (s - 1) * R;
                    k = k < 0 ? k + NB : k;
                    b = widen4<T>(bq[k * 64]);
                } else {
                    b = widen4<T>(b1);
                }
            }
            float dgy = 0.f;
            if constexpr (MODE == MODE_WAVE_DAMP) dgy = dgz + ld_inv(v.damp + v.g.n[0] + min(max(yo, 0), ny - 1));
            float o[4], before[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                float m[R], p[R];
                float acc = w.cd0 * c[i];
#pragma unroll
                for (int k = 1; k <= R; k++) {
                    m[k - 1] = q[s - 1][at(R - k)][i];
                    p[k - 1] = q[s - 1][at(R + k)][i];
                }
                acc = axis_sum<R>(acc, w, m, p);
#pragma unroll
                for (int k = 1; k <= R; k++) {
                    m[k - 1] = xv[4 + i - k];
                    p[k - 1] = xv[4 + i + k];
                }
                acc = axis_sum<R>(acc, w, m, p);
                before[i] = s == 1 ? prev[i] : q[s < 2 ? 0 : s - 2][at(0)][i];
                if constexpr (MODE == MODE_WAVE_DAMP)
                    o[i] = damped_update(acc, c[i], before[i], comp(b, i), dgy + dgx[i]);
                else
                    o[i] = time_update<MODE>(acc, c[i], before[i], comp(b, i));
            }
            if (due >> (s - 1) & 1) {
                const int cnt = __builtin_amdgcn_readlane(ev_cnt, s - 1);
#pragma nounroll
                for (int k = 0; k < cnt; k++) {
                    const StagedSource t = staged[(s - 1) * kMarchRowSources + k];
                    const int i = t.x - x0;
                    float u = i == 0 ? o[0] : i == 1 ? o[1] : i == 2 ? o[2] : o[3];
                    u = inject<T>(u, t.amount);
                    o[0] = i == 0 ? u : o[0];
                    o[1] = i == 1 ? u : o[1];
                    o[2] = i == 2 ? u : o[2];
                    o[3] = i == 3 ? u : o[3];
                }
            }
#pragma unroll
            for (int i = 0; i < 4; i++) o[i] = through<T>(o[i]);
            const bool yin = yo >= 0 && yo < ny;
            if (edge || !yin) {
#pragma unroll
                for (int i = 0; i < 4; i++) o[i] = yin && in[i] ? o[i] : before[i];
            }
            if (due >> (31 + s) & 1)
                *reinterpret_cast<float4*>(recrow + 256 * (s - 1) + 4 * lane) = make_float4(o[0], o[1], o[2], o[3]);
            if (s == NT) store(v.out, yo, o);
            if (WAVE && s == NT - 1) store(v.out1, yo, o);
            if (s < NT) {
#pragma unroll
                for (int i = 0; i < 4; i++) q[s < NT ? s : 0][OFF][i] = o[i];
            }
        }
        if (due >> 32) record((unsigned)(due >> 32), y);
        if constexpr (WAVE && NT > 1) bslot = bslot + 1 == NB ? 0 : bslot + 1;
        y++;
    };
    // the first iteration's newest row sits in slot 2R
    while (y < yend) {
        step(std::integral_constant<int, 2 * R>{});
        StaticFor<0, Q - 1>::run([&](auto c) __attribute__((always_inline)) {
            if (y < yend) step(c);
        });
    }
}

// waves of a pass the current device holds at once, asked for once per device
template <int MODE, int R, typename T, int NT>
hipError_t m2_resident(int& waves) {
    static std::atomic<int> known[64];   // 0: not yet
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 64 && (waves = known[dev].load()) > 0) return hipSuccess;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(k_march2d<MODE, R, T, NT>), 64,
                                                         March2D<T, MODE, R, NT>::LDS_BYTES);
    waves = std::max(1, cus * per_cu);
    if (e == hipSuccess && dev < 64) known[dev] = waves;
    return e;
}

template <int MODE, int R, typename T, int NT>
hipError_t m2_launch(const M2View& v, const Coefs& w, int row0, hipStream_t s) {
    constexpr size_t lds = March2D<T, MODE, R, NT>::LDS_BYTES;
    if (v.nstrips == 0 || v.g.n[1] == 0) return hipSuccess;
    auto k = k_march2d<MODE, R, T, NT>;
    static std::atomic<uint64_t> lds_on{0};
    const hipError_t attr = allow_lds(k, lds, lds_on);
    if (attr != hipSuccess) return attr;
    // As many chunks of rows as the GPU holds waves: every wave then starts
    // at once and ends with the others, and the 2 R NT rows around a chunk
    // are computed as few times as that allows.  8192^2 FP32 wave, radius 4,
    // NT = 4, us a step: 149 rows (2035 of 2048 waves) 110, 200 rows 133, 99
    // rows 126, 75 rows 116, 50 rows 119.
    int waves = 0;
    const hipError_t known = m2_resident<MODE, R, T, NT>(waves);
    if (known != hipSuccess) return known;
    M2View u = v;
    u.rows = std::max(4, (v.g.n[1] + std::max(1, waves / v.nstrips) - 1) / std::max(1, waves / v.nstrips));
    u.nchunks = (v.g.n[1] + u.rows - 1) / u.rows;
    hipLaunchKernelGGL(k, dim3((unsigned)(v.nstrips * u.nchunks)), dim3(64), lds, s, u, w, row0);
    return hipGetLastError();
}

template <int MODE, int R, typename T>
hipError_t m2_t(int nt, const M2View& v, const Coefs& w, int row0, hipStream_t s) {
    switch (nt) {
        case 4: return m2_launch<MODE, R, T, 4>(v, w, row0, s);
    }
    if constexpr (R == 1 && std::is_same<T, float>::value)
        if (nt == 8) return m2_launch<MODE, R, T, 8>(v, w, row0, s);
    return hipErrorInvalidValue;
}

template <int MODE, typename T>
hipError_t m2_r(int radius, int nt, const M2View& v, const Coefs& w, int row0, hipStream_t s) {
    switch (radius) {
        case 1: return m2_t<MODE, 1, T>(nt, v, w, row0, s);
        case 2: return m2_t<MODE, 2, T>(nt, v, w, row0, s);
        case 3: return m2_t<MODE, 3, T>(nt, v, w, row0, s);
        case 4: return m2_t<MODE, 4, T>(nt, v, w, row0, s);
    }
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t m2_m(int mode, int radius, int nt, const M2View& v, const Coefs& w, int row0, hipStream_t s) {
    if (mode == MODE_HEAT) return m2_r<MODE_HEAT, T>(radius, nt, v, w, row0, s);
    if (mode == MODE_WAVE) return m2_r<MODE_WAVE, T>(radius, nt, v, w, row0, s);
    if constexpr (std::is_same<T, float>::value)
        if (mode == MODE_WAVE_DAMP) return m2_r<MODE_WAVE_DAMP, T>(radius, nt, v, w, row0, s);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_march2d(int mode, int radius, int dtype, int nt, const M2View& v, const Coefs& w, int row0,
                          hipStream_t s) {
    if (nt == 1) return launch_step2d(mode, radius, dtype, v, w, row0, s);
    switch (dtype) {
        case DT_F32: return m2_m<float>(mode, radius, nt, v, w, row0, s);
        case DT_BF16: return m2_m<bf16>(mode, radius, nt, v, w, row0, s);
        case DT_F16: return m2_m<f16>(mode, radius, nt, v, w, row0, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace stn
