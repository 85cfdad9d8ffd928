// The 3D sweep of a box by bricks (k_zbrick): a workgroup
// computes a brick of 64 x 16 x BZ points.  The loads of the brick (the
// threads' own z columns, the in-plane margins, u_prev and beta) come before the
// arithmetic, a single barrier between them, so a workgroup pays the memory
// latency once or twice (the compiler copies a group of the FP32 column's loads
// while the others are under way, and waits for it), where the z-marching
// kernel pays it again on every plane of its chunk.
//
// It serves what the z-march leaves idle: grids with too few xy tiles and
// z-chunks to fill 256 compute units, and boxes (stencil_apply on the boundary
// slabs and the interior of a decomposed grid).  It reads each level
// (BZ + 2R) / BZ times in z, mostly from the caches, so on grids that fill the
// chip the z-march, which reads it once, stays ahead.  Small grids are bound
// by the launch and one memory latency, larger ones by the cache traffic.
//
// One FP32 wave step, radius 4, in us (this kernel / best z-march / one
// thread per point with its taps from the caches, which this replaces):
// 64^3 3.7 / 23 / -, 61 x 75 x 90 with a source and 16 receivers 4.7 / 23 / 6.3
// plus 3.9 of injection and recording, 128^3 7.0 / 24 / 14, 192^3 19 / 26, 256^3
// 47 / 44, 512^3 463 / 372.  FP16 207 x 301 x 259: 31 / 35.
//
// Each point takes the canonical operation order (device.hpp), so the results
// are those of every other sweep kernel bit for bit.
#include "strip2d.hpp"
#include "zmarch.hpp"

namespace stn {

// Number the bricks z first where the planes that z neighbours share pass the
// reach of an XCD's 4 MB L2 otherwise: neighbours in z share 2R of their
// BZ + 2R planes, tiles side by side only their margins.  One FP32 wave step of
// radius 4 in us, x first / z first: 64 x 512 x 512 75 / 46, 207 x 301 x 259 60 /
// 55 (3.1 MB), 256^3 48 / 50 (2.6 MB), 224^3 31 / 37.  Where the fields pass the
// last-level cache the order x first streams as well or better (512^3, BZ = 4:
// 463 / 505).  Radius 1 to 4, FP32 and FP16, 17 boxes of 96^3 to 320^3 and of 8 to
// 128 planes: the order taken is the faster one or within 5%, but for 40 x 384 x
// 384 (10.4 / 9.4) and 8 x 512 x 512 (5.7 / 4.5) in FP16, r = 2 and 1, just below
// the line, where 320^3, r = 4, has 47 / 52.
bool brick_zfast(const int64_t* n, int radius, size_t esize, int bz) {
    return (double)(bz + 2 * radius) * n[1] * n[2] * esize > 2.85e6 && brick_cached(n, esize);
}

namespace {

template <int R, int BZ>
struct ZBrick {
    static constexpr int NT = 256, TX = kBrickTileX, TY = kBrickTileY;
    static constexpr int LDX = TX + 8, LDY = TY + 2 * R, PLANE = LDX * LDY;
    // margin groups of a plane: one each side of every tile row, TX / 4 per
    // row above and below the tile
    static constexpr int NHX = 2 * TY, NHP = NHX + 2 * R * (TX / 4);
    static constexpr int NQ = BZ + 2 * R;   // planes of a thread's own column
    static_assert(TX == 64 && NT == (TX / 4) * TY && NHP <= NT, "one group of the tile, and of a plane's margin, per thread");
};

template <int MODE>
inline constexpr bool kAdj = MODE == MODE_WAVE_ADJ || MODE == MODE_WAVE_ADJ2;

// waves per SIMD the registers are held to (the adjoint spills at 5; the heat
// form would otherwise read the taps of every plane ahead and take 216
// registers at BZ = 4)
template <int MODE, int BZ>
inline constexpr int kBrickWaves = BZ == 2 ? (kAdj<MODE> ? 4 : 5) : kAdj<MODE> ? 3 : 4;

// One workgroup's brick: tile (tile_x, tile_y) and z-chunk zch of the box.
// LONG: a tile may have more than 64 sources.  Such a brick finds the entries of
// its planes by a search and each wave those of its rows; where every brick of
// the column walked the whole list, a gradient of 128^3 with 16384 receivers in
// a plane took 92 us a step, now 64.  A form of its own, because the shorter
// one loses 1% with the search in it.
template <int MODE, int R, typename T, int BZ, bool LONG>
__device__ __forceinline__ void brick(const ZView& v, const Coefs& w, const Box3& box, int tile_x, int tile_y, int zch,
                                      int parity, int arow, float* __restrict__ lds) {
    using Z = ZBrick<R, BZ>;
    using S = Storage<T>;
    constexpr int TX = Z::TX, TY = Z::TY, LDX = Z::LDX, PLANE = Z::PLANE, NQ = Z::NQ;
    constexpr bool WAVE = MODE != MODE_HEAT;
    constexpr bool ADJ = kAdj<MODE>, ADJ2 = MODE == MODE_WAVE_ADJ2;

    const int tid = threadIdx.x, tx = tid % (TX / 4), ty = tid / (TX / 4);
    // the box's x origin rounded down to a 4-element group keeps every access aligned
    const int bx = (int)box.lo[2], by = (int)box.lo[1], bz = (int)box.lo[0];
    const int X0 = (bx & ~3) + tile_x * TX, Y0 = by + tile_y * TY, zb = bz + zch * BZ;
    const int xe = bx + (int)box.n[2], ye = by + (int)box.n[1], ze = min(zb + BZ, bz + (int)box.n[0]);
    const int64_t sz = v.g.s[0], sy = v.g.s[1];

    const T* U = (const T*)(parity ? v.prev : v.u) + v.g.origin;
    const T* P = (const T*)(parity ? v.u : v.prev) + v.g.origin;
    T* O = (T*)(parity ? (void*)v.u : v.out) + v.g.origin;
    const T* B = (const T*)v.beta + v.g.origin;

    // Every load stays inside the field: planes and rows are clamped to the
    // R-deep halo, x groups to the row; clamped values feed no stored point.
    // On a small grid a wave has its SIMD to itself and issues an instruction
    // every 8 cycles, so the addresses are on the critical path: the plane's
    // part is uniform and steps from plane to plane, a lane's is formed once
    // for its own column and once for its margin group.
    const int xmax4 = (int)(v.g.rowlen - v.g.xlead) - 4;
    const int ymax = v.g.n[1] + R - 1, zmax = v.g.n[0] + R - 1;
    const int x0 = X0 + 4 * tx, y = Y0 + ty;
    const int64_t own = (int64_t)min(y, ymax) * sy + min(x0, xmax4);
    int64_t plane[NQ];   // offsets of planes zb - R .. zb + BZ + R - 1
    plane[0] = (int64_t)(zb - R) * sz;
#pragma unroll
    for (int k = 1; k < NQ; k++) plane[k] = plane[k - 1] + (zb - R + k <= zmax ? sz : 0);

    // the thread's own column and the margins of planes zb .. zb + BZ - 1, in
    // the storage type while in flight
    using Raw = typename RawGroup<T>::type;
    Raw hal[BZ], rq[NQ], rp[BZ], rb[BZ];
#pragma unroll
    for (int k = 0; k < NQ; k++) rq[k] = load4_raw<T, false>(U + plane[k] + own);
    // margin group (threads below NHP): a side of a tile row, then the rows
    // above and below
    const bool margin = tid < Z::NHP;
    int hlds = 0;
    {
        const int t2 = tid - Z::NHX, r2 = t2 >> 4, g2 = t2 & 15;
        const bool sides = tid < Z::NHX;
        const int hy = sides ? Y0 + (tid >> 1) : r2 < R ? Y0 - R + r2 : Y0 + TY + (r2 - R);
        const int hx = sides ? ((tid & 1) ? X0 + TX : X0 - 4) : X0 + 4 * g2;
        hlds = sides ? (R + (tid >> 1)) * LDX + ((tid & 1) ? 4 + TX : 0) : (r2 < R ? r2 : TY + r2) * LDX + 4 + 4 * g2;
        const int64_t mo = (int64_t)min(hy, ymax) * sy + min(hx, xmax4);
        if (margin) {
#pragma unroll
            for (int p = 0; p < BZ; p++) hal[p] = load4_raw<T, false>(U + plane[R + p] + mo);
        }
    }
    if constexpr (WAVE) {
#pragma unroll
        for (int p = 0; p < BZ; p++) {
            rp[p] = load4_raw<T, false>(P + plane[R + p] + own);
            rb[p] = load4_raw<T, false>(B + plane[R + p] + own);
        }
    }
    // adjoint: the second differences and the imaging partial, clamped as the
    // levels (a group that the box cuts reads its points at the store instead).
    // Behind a bounds branch they waited for the loads before them: 128^3
    // gradient 2514 us, now 2479
    const bool full = x0 >= bx && x0 + 3 < xe;
    const bool gload = ADJ && !v.gfresh;
    float4 cd[BZ], cg[BZ], cd2[BZ];
    if constexpr (ADJ) {
#pragma unroll
        for (int p = 0; p < BZ; p++) {
            const int64_t o = v.g.origin + plane[R + p] + own;
            cd[p] = Storage<float>::load4_nt(v.dfield + o);
            if constexpr (ADJ2) cd2[p] = Storage<float>::load4_nt(v.dfield2 + o);
            cg[p] = Storage<float>::load4(v.gfield + o);   // of no use, but allocated, where the partial is fresh
        }
    }
    float dgy = 0.f, dgx[4];
    if constexpr (MODE == MODE_WAVE_DAMP) {
        const float* D = v.damp + v.g.n[0];
        dgy = D[min(y, v.g.n[1] - 1)];
#pragma unroll
        for (int i = 0; i < 4; i++) dgx[i] = D[v.g.n[1] + min(x0 + i, v.g.n[2] - 1)];
    }

    // The tile's sources, 64 at a time, one per lane; the first ones are loaded
    // here, so that their chain of loads (list, entry, amount) runs beside the
    // field's.  src_at: the point's place in LDS, -1 outside the brick
    int src_begin = 0, src_end = 0, src_at = -1;
    double src_amt = 0.0;
    auto load_sources = [&](int from) {
        const int4 e = reinterpret_cast<const int4*>(v.src.zyx4)[min(from + (tid & 63), src_end - 1)];
        const bool in = from + (tid & 63) < src_end && e.x >= zb && e.x < ze;
        src_at = in ? (e.x - zb) * PLANE + (R + e.y - Y0) * LDX + 4 + (e.z - X0) : -1;
        if (in) src_amt = v.src.amp[(int64_t)arow * v.src.n + e.w] * (v.src.scale ? v.src.scale[e.w] : 1.0);
    };
    if (v.src.n > 0) {
        const int tile = tile_y * v.ntx + tile_x;
        src_begin = ld_inv(v.src.tile_begin + tile);
        src_end = ld_inv(v.src.tile_begin + tile + 1);
        if constexpr (LONG) {   // the brick's own planes
            src_begin = first_from(v.src.zyx4, src_begin, src_end, zb, INT_MIN);
            src_end = first_from(v.src.zyx4, src_begin, src_end, ze, INT_MIN);
        }
        if (src_begin < src_end) load_sources(src_begin);
    }

    float4 q[NQ];
#pragma unroll
    for (int k = 0; k < NQ; k++) q[k] = widen4<T>(rq[k]);
#pragma unroll
    for (int p = 0; p < BZ; p++)
        *reinterpret_cast<float4*>(&lds[p * PLANE + (R + ty) * LDX + 4 + 4 * tx]) = q[R + p];
    if (margin) {
#pragma unroll
        for (int p = 0; p < BZ; p++) *reinterpret_cast<float4*>(&lds[p * PLANE + hlds]) = widen4<T>(hal[p]);
    }
    __syncthreads();

    float o[BZ][4], dv[BZ][4];
#pragma unroll
    for (int p = 0; p < BZ; p++) {
        const float* L = lds + p * PLANE + (R + ty) * LDX + 4 + 4 * tx;
        const float4 c = q[R + p];
        float acc[4];
#pragma unroll
        for (int i = 0; i < 4; i++) acc[i] = w.cd0 * comp(c, i);
#pragma unroll
        for (int k = 1; k <= R; k++)
#pragma unroll
            for (int i = 0; i < 4; i++) acc[i] = fmaf(w.c[k], comp(q[R + p - k], i) + comp(q[R + p + k], i), acc[i]);
#pragma unroll
        for (int k = 1; k <= R; k++) {
            const float4 m = *reinterpret_cast<const float4*>(L - k * LDX);
            const float4 n = *reinterpret_cast<const float4*>(L + k * LDX);
#pragma unroll
            for (int i = 0; i < 4; i++) acc[i] = fmaf(w.c[k], comp(m, i) + comp(n, i), acc[i]);
        }
        const float4 xl = *reinterpret_cast<const float4*>(L - 4);
        const float4 xr = *reinterpret_cast<const float4*>(L + 4);
        const float xv[12] = {xl.x, xl.y, xl.z, xl.w, c.x, c.y, c.z, c.w, xr.x, xr.y, xr.z, xr.w};
        float4 cp = make_float4(0.f, 0.f, 0.f, 0.f), cb = cp;
        if constexpr (WAVE) {
            cp = widen4<T>(rp[p]);
            cb = widen4<T>(rb[p]);
        }
        float dgz = 0.f;
        if constexpr (MODE == MODE_WAVE_DAMP) dgz = v.damp[min(zb + p, v.g.n[0] - 1)];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            float m[R], n[R];
#pragma unroll
            for (int k = 1; k <= R; k++) {
                m[k - 1] = xv[4 + i - k];
                n[k - 1] = xv[4 + i + k];
            }
            const float a = axis_sum<R>(acc[i], w, m, n);
            if constexpr (MODE == MODE_WAVE_DAMP)
                o[p][i] = damped_update(a, comp(c, i), comp(cp, i), comp(cb, i), (dgz + dgy) + dgx[i]);
            else
                o[p][i] = time_update<MODE>(a, comp(c, i), comp(cp, i), comp(cb, i));
            if constexpr (MODE == MODE_WAVE_D) dv[p][i] = comp(cb, i) * a;
        }
    }

    // Injection: the values go to their places in LDS, where a wave's lanes add
    // the sources of its four rows in parallel.  Those of one point are next to
    // each other in the list and take turns, in its order.  (A receiver line of
    // the adjoint has 32 or 64 of them in one brick, which that brick's wave
    // took one after another before: a 128^3 step 11.6 us, now 7.8.)
    const int chunks = src_end - src_begin;
    if (chunks > 64 || __ballot(src_at >= 0)) {   // the same in all four waves
        __syncthreads();   // the planes have been read
        auto inject_all = [&](float (&val)[BZ][4], auto&& add) __attribute__((always_inline)) {
            float* own = lds + (R + ty) * LDX + 4 + 4 * tx;
#pragma unroll
            for (int p = 0; p < BZ; p++)
                *reinterpret_cast<float4*>(own + p * PLANE) = make_float4(val[p][0], val[p][1], val[p][2], val[p][3]);
            wave_lds_fence();
            const int row0 = __builtin_amdgcn_readfirstlane(ty);
            auto add_from = [&](int begin) __attribute__((always_inline)) {
                for (int from = begin; from < src_end; from += 64) {
                    if (chunks > 64) load_sources(from);
                    const int row = src_at % PLANE / LDX - R - row0;
                    const uint64_t mine = __ballot(src_at >= 0 && row >= 0 && row < 4);
                    const uint64_t next = __ballot(__shfl_up(src_at, 1) == src_at) & ~1ull;   // same point as the one before
                    for (uint64_t todo = mine; todo;) {
                        const uint64_t go = todo & ~(next & (todo << 1));
                        if (go >> (tid & 63) & 1) lds[src_at] = add(lds[src_at], src_amt);
                        wave_lds_fence();
                        todo &= ~go;
                    }
                }
            };
            if (!LONG || chunks <= 64) {
                add_from(src_begin);
            } else {   // the wave's own rows of each plane
                const int end = src_end;
                for (int z = zb, at = src_begin; z < ze; z++, at = src_end) {
                    at = first_from(v.src.zyx4, at, end, z, Y0 + row0);
                    src_end = first_from(v.src.zyx4, at, end, z, Y0 + row0 + 4);
                    add_from(at);
                }
                src_end = end;
            }
#pragma unroll
            for (int p = 0; p < BZ; p++) {
                const float4 r = *reinterpret_cast<const float4*>(own + p * PLANE);
#pragma unroll
                for (int i = 0; i < 4; i++) val[p][i] = comp(r, i);
            }
        };
        inject_all(o, [](float x, double a) { return inject<T>(x, a); });
        if constexpr (MODE == MODE_WAVE_D) inject_all(dv, [](float x, double a) { return (float)((double)x + a); });
    }

    if (y >= ye || x0 >= xe) return;
#pragma unroll
    for (int p = 0; p < BZ; p++) {
        if (zb + p >= ze) break;
        const int64_t off = (int64_t)(zb + p) * sz + (int64_t)y * sy + x0;
        if (full) {
            S::store4(O + off, make_float4(o[p][0], o[p][1], o[p][2], o[p][3]));
        } else {
#pragma unroll
            for (int i = 0; i < 4; i++)
                if (x0 + i >= bx && x0 + i < xe) S::store(O + off + i, o[p][i]);
        }
        if constexpr (MODE == MODE_WAVE_D) {
            float* D = v.dfield + v.g.origin + off;
            if (full) {
                Storage<float>::store4_nt(D, make_float4(dv[p][0], dv[p][1], dv[p][2], dv[p][3]));
            } else {
#pragma unroll
                for (int i = 0; i < 4; i++)
                    if (x0 + i < xe) D[i] = dv[p][i];
            }
        }
        // the input level's term first (ADJ2), as two one-level steps would
        if constexpr (ADJ) {
            float* G = v.gfield + v.g.origin + off;
            if (full) {
                float g[4];
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    g[i] = gload ? comp(cg[p], i) : 0.f;
                    if constexpr (ADJ2) g[i] = fmaf(comp(q[R + p], i), comp(cd2[p], i), g[i]);
                    g[i] = fmaf(o[p][i], comp(cd[p], i), g[i]);
                }
                Storage<float>::store4(G, make_float4(g[0], g[1], g[2], g[3]));
            } else {
                const float* D = v.dfield + v.g.origin + off;
                const float* D2 = v.dfield2 + v.g.origin + off;
#pragma unroll
                for (int i = 0; i < 4; i++)
                    if (x0 + i < xe) {
                        float g = gload ? G[i] : 0.f;
                        if constexpr (ADJ2) g = fmaf(comp(q[R + p], i), D2[i], g);
                        G[i] = fmaf(o[p][i], D[i], g);
                    }
            }
        }
    }
}

// Receivers sample the input level of a launch (nothing writes it there).  They
// have workgroups of their own, in front of the bricks, one for 1024 of them:
// within a brick their two dependent loads would make that brick the last to
// end.  Workgroup k of n takes every nth 256 of them.
__host__ __device__ inline int record_groups(int n) { return (n + 1023) / 1024; }
template <typename T>
__device__ __forceinline__ void record_input(const ZView& v, int parity, int trow, int k, int n) {
    const T* U = (const T*)(parity ? v.prev : v.u) + v.g.origin;
    double* trace = v.rec.trace + (int64_t)trow * v.rec.n;
    for (int r = 256 * k + (int)threadIdx.x; r < v.rec.n; r += 256 * n) trace[r] = (double)Storage<T>::load(U + v.rec.off[r]);
}

// The launch's grid: the workgroups that record receivers, in front, and nb
// bricks numbered x, y, z or (zfast) z, x, y.
struct BrickGrid {
    int nb, zfast;
    FastDiv inner, row;   // by the bricks of an xy plane (zfast: of a column); by v.ntx
};

template <int MODE, int R, typename T, int BZ, bool LONG>
__global__ __launch_bounds__(256, (kBrickWaves<MODE, BZ>)) void k_zbrick(ZView v, Coefs w, Box3 box, BrickGrid grid,
                                                                       int parity, int arow, int trow) {
    __shared__ __attribute__((aligned(16))) float lds[BZ * ZBrick<R, BZ>::PLANE];
    int b = blockIdx.x;
    // the arguments' cache lines, all asked for at once: the loads that the
    // compiler leaves for later then find them in the scalar cache
    asm volatile("" ::"s"(v.u), "s"(v.g.s[0]), "s"(v.src.n), "s"(v.ntx), "s"(box.lo[1]), "s"(v.rec.n), "s"(w.cd0), "s"(grid.nb));
    if (trow >= 0) {
        if constexpr (LONG) {
            const int nrec = record_groups(v.rec.n);
            if (b < nrec) {
                record_input<T>(v, parity, trow, b, nrec);
                return;
            }
            b -= nrec;
        } else {
            if (b == 0) {
                record_input<T>(v, parity, trow, 0, 1);
                return;
            }
            b--;
        }
    }
    const int lb = xcd_remap(b, grid.nb);
    const int q = (int)fdiv((uint32_t)lb, grid.inner), r = lb - q * (int)grid.inner.d;
    const int tile = grid.zfast ? q : r, zch = grid.zfast ? r : q;
    const int tile_y = (int)fdiv((uint32_t)tile, grid.row);
    brick<MODE, R, T, BZ, LONG>(v, w, box, tile - tile_y * (int)grid.row.d, tile_y, zch, parity, arow, lds);
}

// The bricks of a group of shots in one launch: block_map[b] = (shot, tile x,
// tile y, z-chunk) of workgroup b, shot -1 for padding; the host lays it out per
// XCD.  A shot
// of 100^3 has too few bricks to fill the chip and takes 6 us for 2.8 TB/s; all
// shots together fill it.
template <typename T, bool LONG>
__global__ __launch_bounds__(256, (kBrickWaves<MODE_WAVE, kBatchBrick>)) void k_zbrick_batch(
    const ZView* __restrict__ views, const int4* __restrict__ block_map, Coefs w, int parity, int arow, int trow) {
    __shared__ __attribute__((aligned(16))) float lds[kBatchBrick * ZBrick<4, kBatchBrick>::PLANE];
    const int4 e = block_map[blockIdx.x];
    if (e.x < 0) return;
    // the pointers are read as constant memory, where the compiler takes them to
    // be global; as generic ones their loads would count as LDS accesses too and
    // every wait would be for all of them
    const ZView* from = views + e.x;
    ZView v = *from;
    v.u = ld_inv(&from->u);
    v.prev = ld_inv(&from->prev);
    v.out = ld_inv(&from->out);
    v.beta = ld_inv(&from->beta);
    v.src.zyx4 = ld_inv(&from->src.zyx4);
    v.src.amp = ld_inv(&from->src.amp);
    v.src.scale = ld_inv(&from->src.scale);
    v.rec.off = ld_inv(&from->rec.off);
    v.rec.trace = ld_inv(&from->rec.trace);
    Box3 box{};
    for (int a = 0; a < 3; a++) box.n[a] = v.g.n[a];
    brick<MODE_WAVE, 4, T, kBatchBrick, LONG>(v, w, box, e.y, e.z, e.w, parity, arow, lds);
    // (a workgroup in front for this, as in k_zbrick, costs 4% here: it moves
    // the bricks of one XCD against those of the others)
    if (trow >= 0 && (e.y | e.z | e.w) == 0) record_input<T>(v, parity, trow, 0, 1);
}

template <typename T>
hipError_t brick_batch(const ZView* views, const int* block_map, int nblocks, bool long_lists, const Coefs& w,
                       int parity, int arow, int trow, hipStream_t s) {
    if (nblocks == 0) return hipSuccess;
    auto k = long_lists ? k_zbrick_batch<T, true> : k_zbrick_batch<T, false>;
    hipLaunchKernelGGL(k, dim3((unsigned)nblocks), dim3(256), 0, s, views, (const int4*)block_map, w, parity, arow, trow);
    return hipGetLastError();
}

template <int MODE, int R, typename T, int BZ>
hipError_t brick_launch(const ZView& v, const Coefs& w, const Box3& box, int parity, int arow, int trow, hipStream_t s) {
    ZView b = v;
    b.ntx = (int)(((box.lo[2] & 3) + box.n[2] + kBrickTileX - 1) / kBrickTileX);
    b.nty = (int)((box.n[1] + kBrickTileY - 1) / kBrickTileY);
    b.nzc = (int)((box.n[0] + BZ - 1) / BZ);
    const int64_t nb = (int64_t)b.ntx * b.nty * b.nzc;
    if (nb == 0) return hipSuccess;
    if (v.rec.n == 0) trow = -1;
    const int nrec = trow >= 0 ? record_groups(v.rec.n) : 0;
    if (nb >= INT_MAX - nrec) return hipErrorInvalidConfiguration;
    const bool zfast = brick_zfast(box.n, R, sizeof(T), BZ);
    const BrickGrid grid{(int)nb, zfast, fast_div((uint32_t)(zfast ? b.nzc : b.ntx * b.nty)), fast_div((uint32_t)b.ntx)};
    auto k = v.src.longest > 64 || nrec > 1 ? k_zbrick<MODE, R, T, BZ, true> : k_zbrick<MODE, R, T, BZ, false>;
    hipLaunchKernelGGL(k, dim3((unsigned)(nb + nrec)), dim3(256), 0, s, b, w, box, grid, parity, arow, trow);
    return hipGetLastError();
}

template <int MODE, int R, typename T>
hipError_t brick_z(int bz, const ZView& v, const Coefs& w, const Box3& box, int parity, int arow, int trow,
                   hipStream_t s) {
    if (bz == 2) return brick_launch<MODE, R, T, 2>(v, w, box, parity, arow, trow, s);
    if (bz == 4) return brick_launch<MODE, R, T, 4>(v, w, box, parity, arow, trow, s);
    return hipErrorInvalidValue;
}

template <int MODE, typename T>
hipError_t brick_r(int radius, int bz, const ZView& v, const Coefs& w, const Box3& box, int parity, int arow, int trow,
                   hipStream_t s) {
    switch (radius) {
        case 1: return brick_z<MODE, 1, T>(bz, v, w, box, parity, arow, trow, s);
        case 2: return brick_z<MODE, 2, T>(bz, v, w, box, parity, arow, trow, s);
        case 3: return brick_z<MODE, 3, T>(bz, v, w, box, parity, arow, trow, s);
        case 4: return brick_z<MODE, 4, T>(bz, v, w, box, parity, arow, trow, s);
    }
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t brick_m(int mode, int radius, int bz, const ZView& v, const Coefs& w, const Box3& box, int parity, int arow,
                   int trow, hipStream_t s) {
    if (mode == MODE_HEAT) return brick_r<MODE_HEAT, T>(radius, bz, v, w, box, parity, arow, trow, s);
    if (mode == MODE_WAVE) return brick_r<MODE_WAVE, T>(radius, bz, v, w, box, parity, arow, trow, s);
    // the adjoint path and the absorbing layer are FP32 only
    if constexpr (std::is_same<T, float>::value) {
        if (mode == MODE_WAVE_D) return brick_r<MODE_WAVE_D, T>(radius, bz, v, w, box, parity, arow, trow, s);
        if (mode == MODE_WAVE_ADJ) return brick_r<MODE_WAVE_ADJ, T>(radius, bz, v, w, box, parity, arow, trow, s);
        if (mode == MODE_WAVE_ADJ2) return brick_r<MODE_WAVE_ADJ2, T>(radius, bz, v, w, box, parity, arow, trow, s);
        if (mode == MODE_WAVE_DAMP) return brick_r<MODE_WAVE_DAMP, T>(radius, bz, v, w, box, parity, arow, trow, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_brick_batch(int radius, int dtype, const ZView* views, const int* block_map, int nblocks,
                              bool long_lists, const Coefs& w, int parity, int arow, int trow, hipStream_t s) {
    if (radius != 4) return hipErrorInvalidValue;
    switch (dtype) {
        case DT_F32: return brick_batch<float>(views, block_map, nblocks, long_lists, w, parity, arow, trow, s);
        case DT_BF16: return brick_batch<bf16>(views, block_map, nblocks, long_lists, w, parity, arow, trow, s);
        case DT_F16: return brick_batch<f16>(views, block_map, nblocks, long_lists, w, parity, arow, trow, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_brick(int mode, int radius, int dtype, int bz, const ZView& v, const Coefs& w, const Box3& box,
                        int parity, int arow, int trow, hipStream_t s) {
    switch (dtype) {
        case DT_F32: return brick_m<float>(mode, radius, bz, v, w, box, parity, arow, trow, s);
        case DT_BF16: return brick_m<bf16>(mode, radius, bz, v, w, box, parity, arow, trow, s);
        case DT_F16: return brick_m<f16>(mode, radius, bz, v, w, box, parity, arow, trow, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace stn
