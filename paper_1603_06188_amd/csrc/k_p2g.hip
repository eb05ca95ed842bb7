// Transfer to grid (Sec. 3.2) with the force of Sec. 3.3 fused in (lambda = 0).
//
// Every particle of a key (base node) touches the same K^DIM nodes, so one lane
// per key accumulates its particles' contributions to those nodes in registers,
// then the 64 lanes of a tile add their sums into the tile's slab in LDS in
// K^DIM rounds (within a round the lanes hit distinct nodes: plain
// read-modify-write, no atomics), and the slab is stored with plain coalesced
// writes.  2D and multilinear: one wavefront per listed tile holds all sums.
// 3D quadratic and cubic: a block of wavefronts per tile, one plane each.
//
// Per particle, in cell units (r = (x_i - x_p)/dx, grad w in 1/cell):
//   m_i     += w m_p
//   (mv)_i  += w (m_p v_p + Qc r) + Ac grad w
//   Qc = m_p B_p D^{-1} dx        with D = k dx^2 I, 1/k = 4 (quadratic), 3 (cubic)
//   Ac = -dt V_p tau_p / dx       tau = P F^T = mu (F F^T - I) + lambda ln J I
// so Ac grad w is dt times the force contribution -V_p P F^T grad w of Sec. 3.3.
// The K^DIM node terms are factored axis by axis (tensor-product weights).
#include "apic_kernels.h"
#include "p2g_device.h"

namespace apic {

// --- 3D, quadratic and cubic: one block of wavefronts per listed tile ---------------------
// Levels are taken several at a time: each wavefront forms the terms (stress,
// weights, axis factors) of 64 of their particles and leaves them in LDS by key
// and level; then, lane = key, each wavefront adds the terms of all these levels
// to the register sums of one plane of the slab (mass or a momentum component)
// and at the end flushes that plane by itself.
//
// One wavefront per tile has to hold all (1 + 3) K^3 sums of a key: 108
// registers in binary32 quadratic (two wavefronts per SIMD), and more than there
// are in the others, which walked the particles two to four times and formed
// their stress and weights each time.  Here the terms are formed once, a plane's
// K^3 sums leave room for two to four wavefronts per SIMD, and a small scene has
// four times the wavefronts.  Against a wavefront per tile, same box: binary64
// quadratic 512,000 particles 92 -> 45 us, binary64 cubic 1.12M 324 -> 276,
// binary32 cubic 9.0M 784 -> 594 (0.70 of the time VALU issue), binary32
// quadratic 238,328 particles 21 -> 17, 4,096 particles 21 -> 12, 2,097,152
// particles 86 -> 84 (VALU issue 48 us; a tile's chain of loads, barriers and
// flush rounds is 17 us with four blocks on a CU), 80 since the plane addresses
// are scalar adds.
// Vector issue bounds it where tiles are many: the terms by a wavefront per level,
// most lanes without a particle on the later ones, cost a scene of few particles
// per key more than they saved.  By 64 particles at a time: binary32 quadratic 2.4M
// particles at 8 per cell 126 -> 110 us, at 2 219 -> 185, at 1 321 -> 274, at 0.5 522
// -> 459 (a wavefront per tile: 130, 180, 246, 375); cubic 1.0M at 8 79 -> 74;
// binary64 quadratic 1.0M at 8 114 -> 102, cubic 264 -> 250; full levels (the cube at
// rest) as before.  Few tiles of busy keys pay for the branches and counts that the
// other tiles need, with a wavefront per SIMD and nothing beside it: 50,000 particles
// at 27 per cell 57 -> 67 cubic, 81 -> 87 quadratic.
// The mass plane by a loop of its own with half the multiply-adds: 110 -> 116 us (the
// sums move between the two).  The next record's tables loaded ahead: 126 -> 130; the
// flush by LDS atomics: binary32 several times slower, binary64 cubic 1.0M at 1 per
// cell 755 -> 709 but 50,000 at 8 41.6 -> 43.5.
// Binary32 adds by 4x4x1 matrix products (rows: slices, columns: a of one b, 16
// keys a product) need the terms spread over the lanes again: twice the LDS
// traffic, which then bounds the pass (cubic 670 us, quadratic 100).  The next
// tile's tables and particles loaded ahead by 1024 resident blocks: 89 against
// 84 us (cubic 850: three blocks fit a CU and the last ones run alone).
template <typename T, int DEG>
struct LevelTerms {
    static constexpr int K = DEG + 1;
    // FULL: m, the weights, and per component the axis factors X0, Yb, Zc (see
    // p2g_accumulate3).  Else (binary64 cubic, whose LDS they would fill) m, the
    // offsets in the cell and m (v - uref), Qc, Ac, from which the adding
    // wavefront forms them.
    static constexpr bool FULL = !(sizeof(T) == 8 && DEG == 3);
    // WIDE (binary32): a key's terms are 13 units of four words, moved 16 bytes
    // at a time: the weights of axis a in unit a, factor a of component k in unit
    // 3 + 3 k + a, m in unit 12.  An odd number of units per key spreads the
    // lanes of an access over the banks.  Else a row of 64 keys per term.
    static constexpr bool WIDE = sizeof(T) == 4 && DEG == 3;
    static constexpr int UNITS = 13;
    // wavefronts of a block: four, or (binary64 cubic) eight, each plane's 64
    // sums split over two wavefronts by z-slice
    static constexpr int WAVES = FULL ? 4 : 8, CZ = K * 4 / WAVES;
    // the next level's particle is loaded before the current levels are added
    // (cubic has no registers for it beside its sums)
    static constexpr bool AHEAD = DEG == 2;
    static constexpr int W = 1, COMP0 = 1 + 3 * K;
    static constexpr int NF = FULL ? COMP0 + 9 * K : 1 + 3 + 21;
    static constexpr int LEVEL = 64 * (WIDE ? 4 * UNITS : NF);  // elements of a level's terms
    static constexpr int LANE = WIDE ? 4 * UNITS : 1;           // elements between the terms of two keys
};

// K values of unit u of a key's terms.
template <typename T, int DEG>
__device__ __forceinline__ void put_unit(T *s, int u, const T (&x)[DEG + 1]) {
    constexpr int K = DEG + 1;
    using L = LevelTerms<T, DEG>;
    if constexpr (L::WIDE) {
        using V = float __attribute__((ext_vector_type(4)));
        *(V *)(s + 4 * u) = V{x[0], x[1], x[2], K == 4 ? x[K - 1] : 0.f};
    } else {
#pragma unroll
        for (int i = 0; i < K; ++i) s[(L::W + u * K + i) * 64] = x[i];
    }
}
template <typename T, int DEG>
__device__ __forceinline__ void get_unit(const T *s, int u, T (&x)[DEG + 1]) {
    constexpr int K = DEG + 1;
    using L = LevelTerms<T, DEG>;
    if constexpr (L::WIDE) {
        using V = float __attribute__((ext_vector_type(4)));
        const V v = *(const V *)(s + 4 * u);
#pragma unroll
        for (int i = 0; i < K; ++i) x[i] = v[i];
    } else {
#pragma unroll
        for (int i = 0; i < K; ++i) x[i] = s[(L::W + u * K + i) * 64];
    }
}

// Leaves one particle's terms at s (LDS).  A lane without
// a particle (has false) and a particle that must be skipped (flagged) leave
// terms that add nothing.  The stress first, then axis by axis, so that few
// values are live beside the register sums.  Wave-wide.
template <typename T, int DEG, bool ABS>
__device__ __forceinline__ void level_terms(P2GRaw<T, 3> &r, bool has, const int *key, const StepParams<T> &prm,
                                            T inv_dx, uint32_t *flags, const T *uref, T *s) {
    using L = LevelTerms<T, DEG>;
    constexpr int K = DEG + 1;
    int ci[3];
    T off[3], A[6];
    particle_cells<T, 3, ABS>(r.cell, r.off, inv_dx, ci, off);
    bool ok = has && p2g_finite<T, 3>(r);
    if (has && !ok) atomicOr(flags, FLAG_NONFINITE);
    const bool same = base_of<T, DEG>(ci[0], off[0]) == key[0] && base_of<T, DEG>(ci[1], off[1]) == key[1] &&
                      base_of<T, DEG>(ci[2], off[2]) == key[2];
    if (ok && !same) atomicOr(flags, FLAG_UNSORTED);
    ok = ok && same;
    if (~ballot(ok)) {
        // a particle of no mass at rest at the cell's corner
        r.m = ok ? r.m : T(0);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            off[a] = ok ? off[a] : T(0);
            r.v[a] = ok ? r.v[a] : uref[a];
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            r.B[k] = ok ? r.B[k] : T(0);
            r.F[k] = ok ? r.F[k] : (k % 4 == 0 ? T(1) : T(0));
        }
    }
    p2g_force<T, 3>(r.F, r.m, prm, inv_dx, flags, A);
    __builtin_amdgcn_sched_barrier(0);
    const T m = r.m, qs = m * inv_D_factor<T, DEG>() * inv_dx;
    T p[3];
    s[L::WIDE ? 48 : 0] = m;
#pragma unroll
    for (int k = 0; k < 3; ++k) p[k] = m * (r.v[k] - uref[k]);
    constexpr int SYM[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
    if constexpr (L::FULL) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            Axis<T, DEG> ax;
            axis_weights<T, DEG>(ci[a], off[a], ax);
            T Q[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) Q[k] = qs * r.B[k * 3 + a];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                T x[K];
#pragma unroll
                for (int i = 0; i < K; ++i) {
                    x[i] = (ax.w[i] * ax.r[i]) * Q[k] + ax.dw[i] * A[SYM[k][a]];
                    if (a == 0) x[i] += ax.w[i] * p[k];
                }
                put_unit<T, DEG>(s, 3 + 3 * k + a, x);
            }
            put_unit<T, DEG>(s, a, ax.w);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int a = 0; a < 3; ++a) s[(1 + a) * 64] = off[a];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            T *c = s + (4 + 7 * k) * 64;
            c[0] = p[k];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                c[(1 + a) * 64] = qs * r.B[k * 3 + a];
                c[(4 + a) * 64] = A[SYM[k][a]];
            }
        }
    }
}

// Register sums of one plane for the keys of a tile: terms of a level (at s,
// comp 0 mass, 1 + k momentum k) added to them, then flushed into the plane.
// Mass takes the momentum's sums with X0 = m wx and no other factor: one code
// for all wavefronts keeps the sums in place.
template <typename T, int DEG>
struct PlaneSums {
    using L = LevelTerms<T, DEG>;
    static constexpr int K = DEG + 1, CZ = L::CZ;
    T acc[CZ][K][K];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int c = 0; c < CZ; ++c)
#pragma unroll
            for (int b = 0; b < K; ++b)
#pragma unroll
                for (int a = 0; a < K; ++a) acc[c][b][a] = T(0);
    }
    // z-slices [c0, c0 + CZ)
    __device__ __forceinline__ void add(const T *level, int comp, int c0) {
        const T *s = level + lane_id() * L::LANE;
        T w[3][K], f[3][K];  // weights, factors X0, Yb, Zc
        auto slice = [&](const T (&x)[K], int c) { return CZ == K ? x[c] : (c0 == 0 ? x[c] : x[K - CZ + c]); };
        if constexpr (L::FULL) {
#pragma unroll
            for (int a = 0; a < 3; ++a) get_unit<T, DEG>(s, a, w[a]);
            if (comp > 0) {
#pragma unroll
                for (int a = 0; a < 3; ++a) get_unit<T, DEG>(s, 3 * comp + a, f[a]);
            } else {
                const T m = s[L::WIDE ? 48 : 0];
#pragma unroll
                for (int i = 0; i < K; ++i) {
                    f[0][i] = m * w[0][i];
                    f[1][i] = f[2][i] = T(0);
                }
            }
        } else {
            T p, Q[3], A[3];
            if (comp > 0) {
                const T *c = s + (4 + 7 * (comp - 1)) * 64;
                p = c[0];
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    Q[a] = c[(1 + a) * 64];
                    A[a] = c[(4 + a) * 64];
                }
            } else {
                p = s[0];
#pragma unroll
                for (int a = 0; a < 3; ++a) Q[a] = A[a] = T(0);
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                Axis<T, DEG> ax;
                axis_weights<T, DEG>(0, s[(1 + a) * 64], ax);
#pragma unroll
                for (int i = 0; i < K; ++i) {
                    w[a][i] = ax.w[i];
                    const T x = (ax.w[i] * ax.r[i]) * Q[a] + ax.dw[i] * A[a];
                    f[a][i] = a == 0 ? ax.w[i] * p + x : x;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int b = 0; b < K; ++b)
#pragma unroll
            for (int a = 0; a < K; ++a) {
                const T R = w[0][a] * w[1][b], S = f[0][a] * w[1][b] + f[1][b] * w[0][a];
#pragma unroll
                for (int c = 0; c < CZ; ++c) {
                    acc[c][b][a] += slice(w[2], c) * S;
                    acc[c][b][a] += slice(f[2], c) * R;
                }
            }
    }
    // fn(node, value): rounds in each of which the lanes touch distinct nodes
    template <typename Fn>
    __device__ __forceinline__ void flush(int c0, Fn &&fn) {
        using SL = SlabLds<3, DEG>;
        int lc[3];
        local_coords<3>(lane_id(), lc);
        int node0 = SL::at(lc[0], lc[1], lc[2] + c0);
        asm volatile("" : "+v"(node0));  // formed here, not kept in registers over the levels
#pragma unroll
        for (int c = 0; c < CZ; ++c)
#pragma unroll
            for (int b = 0; b < K; ++b)
#pragma unroll
                for (int a = 0; a < K; ++a) fn(node0 + SL::at(a, b, c), acc[c][b][a]);
    }
};

template <typename T, int DEG, bool COMP, bool ABS>
__device__ __forceinline__ void p2g_tile3(const Parts<T> &P, const BinLists &cur, const TileTables &tab,
                                          const Slabs<T> &slabs, const GridState<T> &g, const StepParams<T> &prm_in, uint32_t blk, uint32_t nblk) {
    const StepParams<T> prm = with_step_dt(prm_in);
    using Gm = Geo<3, DEG>;
    using SL = SlabLds<3, DEG>;
    using L = LevelTerms<T, DEG>;
    using U = SlabSum<T, COMP>;
    constexpr bool PAIR = COMP && sizeof(T) == 8;  // sums with an error term beside them
    constexpr int K = Gm::K, RN = Gm::RN, NC = Gm::NC, LP = SL::PLANE, R = (RN + 63) / 64;
    constexpr int NW = L::WAVES, CZ = L::CZ, LEVEL = L::LEVEL;
    constexpr size_t TERMS = NW * LEVEL * sizeof(T), SLAB = NC * (PAIR ? 2 : 1) * LP * sizeof(U);
    // the terms of NW levels; after the last of them the slab planes
    __shared__ __attribute__((aligned(16))) char lds[TERMS > SLAB ? TERMS : SLAB];
    __shared__ T lds_ref[3];
    // key and level in the group of the particles whose terms a wavefront forms
    using Slot = std::conditional_t<NW == 4, uint8_t, uint16_t>;
    __shared__ Slot lds_slot[NW][64];
    const int lane = lane_id(), wv = (int)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int comp = wv & 3, c0 = (wv >> 2) * CZ;  // its plane and z-slices
    Slot *slot = lds_slot[wv];
    // place in LDS of the slab values this lane stores
    int pad[R];
#pragma unroll
    for (int i = 0; i < R; ++i) pad[i] = lane + 64 * i < RN ? kSlabPad<3, DEG>.at[lane + 64 * i] : 0;
    const TileWalk walk = tile_walk(cur);
    T *terms = (T *)lds;
    U *hi = (U *)lds + comp * LP, *lo = (U *)lds + (NC + comp) * LP;
    for (uint32_t r = blk; r < walk.nrec; r += nblk) {
        uint32_t start, cnt, maxc, kstart;
        const uint32_t t = tile_of_record(walk, r, cur, tab, start, cnt, maxc, kstart);
        int origin[3] = {0, 0, 0};
        tile_origin<3>(t, g.d.TN, origin);
        const bool busy = maxc > (uint32_t)kMaxLevels;
        // A group of NW levels from g0 on: its particles follow each other in the
        // tile, from `first` on, `m` of them, and each wavefront forms the terms of 64.
        // (A busy tile's do not: each wavefront forms those of a level, lane = key.)
        // A lane past the last takes the last too: loads under a lane mask would keep
        // the values before them alive.
        uint32_t g0 = 0, first = start, m = 0;
        auto count_group = [&] {
            m = 0;
#pragma unroll
            for (uint32_t i = 0; i < NW; ++i) m += (uint32_t)popc64(ballot(cnt > g0 + i));
        };
        auto place = [&] {  // in the group
            const uint32_t at = (uint32_t)(64 * wv + lane);
            return at < m ? at : m - 1u;
        };
        auto particle = [&] {
            if (busy) return cnt > g0 + (uint32_t)wv ? kstart + g0 + (uint32_t)wv : 0u;
            return first + place();
        };
        auto has_work = [&] { return busy ? g0 + (uint32_t)wv < maxc : (uint32_t)(64 * wv) < m; };
        count_group();
        P2GRaw<T, 3> raw;
        if constexpr (L::AHEAD) {
            if (has_work()) p2g_load<T, 3, ABS>(P, particle(), raw);
        }
        // the tile's reference velocity, from the level-0 particles
        T uref[3];
        if (wv == 0) {
            if constexpr (L::AHEAD) {
                // to the lanes of their keys
                const int from = busy ? lane : popc64(ballot(cnt > 0) & lanes_below(lane));
                T v[3];
#pragma unroll
                for (int a = 0; a < 3; ++a) v[a] = __shfl(raw.v[a], from, 64);
                reference_of_level0<T, 3>(v, cnt > 0, uref);
            } else
                tile_reference<T, 3>(P, start, kstart, cnt, maxc, uref);
            if (lane == 0) {
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    lds_ref[a] = uref[a];
                    g.uref[a * g.d.tiles + t] = uref[a];
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int a = 0; a < 3; ++a) uref[a] = wave_uniform(lds_ref[a]);
        PlaneSums<T, DEG> sums;
        sums.clear();
        while (g0 < maxc) {
            if (has_work()) {
                if constexpr (!L::AHEAD) p2g_load<T, 3, ABS>(P, particle(), raw);
                uint32_t k = (uint32_t)lane, lv = (uint32_t)wv;
                bool has = true;
                if (busy) {
                    has = cnt > g0 + (uint32_t)wv;
                } else if (m < 64u * NW) {  // (else every key has a particle on each level)
                    uint32_t before = 0;
#pragma unroll
                    for (uint32_t i = 0; i < NW; ++i) {
                        const uint64_t mask = ballot(cnt > g0 + i);
                        const uint32_t at = before + (uint32_t)popc64(mask & lanes_below(lane)) - (uint32_t)(64 * wv);
                        if (cnt > g0 + i && at < 64u) slot[at] = (Slot)((uint32_t)lane | i << 6);
                        before += (uint32_t)popc64(mask);
                    }
                    wave_lds_sync();
                    const uint32_t x = slot[place() - (uint32_t)(64 * wv)];
                    k = x & 63u;
                    lv = x >> 6;
                }
                int key[3];
                local_coords<3>((int)k, key);
#pragma unroll
                for (int a = 0; a < 3; ++a) key[a] += origin[a];
                level_terms<T, DEG, ABS>(raw, has, key, prm, g.inv_dx, g.flags, uref,
                                         terms + lv * LEVEL + k * L::LANE);
            }
            const uint32_t g_now = g0;
            first += m;
            g0 += NW;
            count_group();
            if constexpr (L::AHEAD) {
                if (has_work()) p2g_load<T, 3, ABS>(P, particle(), raw);
            }
            __syncthreads();
#pragma unroll 1
            for (uint32_t i = 0; i < NW && g_now + i < maxc; ++i)
                if (cnt > g_now + i) sums.add(terms + i * LEVEL, comp, c0);
            __syncthreads();
        }
        if (c0 == 0) {
#pragma unroll 1
            for (int i = lane; i < LP; i += 64) {
                hi[i] = U(0);
                if constexpr (PAIR) lo[i] = U(0);
            }
        }
        // the two wavefronts of a plane add one after the other
#pragma unroll
        for (int h = 0; h < NW / 4; ++h) {
            if (h > 0) __syncthreads();
            wave_lds_sync();
            if (h * CZ == c0)
                sums.flush(h * CZ, [&](int idx, T x) {
                    const U old = hi[idx], sum = old + (U)x;
                    if constexpr (PAIR) lo[idx] += two_sum_err(old, (U)x, sum);
                    hi[idx] = sum;
                    wave_lds_sync();
                });
        }
        // stored by the wavefront that added last
        if (c0 + CZ == K) {
            T *out = slabs.v + (int64_t)r * slabs.stride + comp * RN;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const int at = lane + 64 * i;
                if (at < RN) {
                    const U sum = hi[pad[i]];
                    const T v = (T)sum;
                    out[at] = v;
                    if constexpr (COMP) out[NC * RN + at] = PAIR ? (T)lo[pad[i]] : (T)(sum - (U)v);
                }
            }
        }
        __syncthreads();
    }
}

template <typename T, int DIM, int DEG, bool COMP, bool ABS = false>
__device__ __forceinline__ void p2g_body(const Parts<T> &P, const BinLists &cur, const TileTables &tab,
                                         const Slabs<T> &slabs, const GridState<T> &g, const StepParams<T> &prm_in, uint32_t blk, uint32_t nblk) {
    const StepParams<T> prm = with_step_dt(prm_in);
    using Gm = Geo<DIM, DEG>;
    using SL = SlabLds<DIM, DEG>;
    using U = SlabSum<T, COMP>;
    constexpr bool PAIR = COMP && sizeof(T) == 8;  // sums with an error term beside them
    constexpr int K = Gm::K, NC = Gm::NC, LP = SL::PLANE;
    constexpr int LSLAB = NC * (PAIR ? 2 : 1) * LP;  // padded planes
    __shared__ U lds_all[4 * LSLAB];
    U *lds = lds_all + (threadIdx.x >> 6) * LSLAB;
    const int lane = lane_id();
    int lcoord[3] = {0, 0, 0};
    local_coords<DIM>(lane, lcoord);
    const TileWalk walk = tile_walk(cur);
    for (uint32_t r = blk * 4 + (threadIdx.x >> 6); r < walk.nrec; r += nblk * 4) {
        uint32_t start, cnt, maxc, kstart;
        const uint32_t t = tile_of_record(walk, r, cur, tab, start, cnt, maxc, kstart);
        int key[3] = {0, 0, 0};
        tile_origin<DIM>(t, g.d.TN, key);
#pragma unroll
        for (int a = 0; a < DIM; ++a) key[a] += lcoord[a];
        // the tile's reference velocity (3D: derived from the level-0
        // particles that the pass loads): the slab holds momenta relative to it
        T uref[DIM];
        for (int i = lane; i < LSLAB; i += 64) lds[i] = U(0);
        wave_lds_sync();
        if constexpr (DIM == 3) {
            p2g_pass3<T, DEG, PAIR, 0, K, false, true, ABS>(P, key, lcoord, start, kstart, cnt, maxc, cnt, maxc, prm,
                                                            g.inv_dx, g.flags, uref, lds);
        } else {
            tile_reference<T, DIM>(P, start, kstart, cnt, maxc, uref);
            T acc_m[K][K], acc_v[2][K][K];
#pragma unroll
            for (int bb = 0; bb < K; ++bb)
#pragma unroll
                for (int a = 0; a < K; ++a) acc_m[bb][a] = acc_v[0][bb][a] = acc_v[1][bb][a] = T(0);
            uint32_t level = 0;
            for (uint32_t jj = 0; jj < maxc; ++jj) {
                const uint64_t mask = ballot(cnt > jj);
                if (cnt > jj) {
                    const int64_t q = particle_at(start, kstart, level, mask, jj, maxc, lane);
                    P2GRaw<T, 2> raw;
                    p2g_load<T, 2, ABS>(P, (uint32_t)q, raw);
                    P2GParticle<T, 2, DEG> pp;
                    if (p2g_prepare<T, 2, DEG, ABS>(raw, key, prm, g.inv_dx, g.flags, uref, pp))
                        p2g_accumulate2<T, DEG>(pp, acc_m, acc_v);
                }
                level += (uint32_t)popc64(mask);
            }
#pragma unroll
            for (int bb = 0; bb < K; ++bb)
#pragma unroll
                for (int a = 0; a < K; ++a) {
                    const int idx = SL::at(lcoord[0] + a, lcoord[1] + bb, 0);
                    const U x[NC] = {(U)acc_m[bb][a], (U)acc_v[0][bb][a], (U)acc_v[1][bb][a]};
                    slab_add_node<U, PAIR, LP, NC>(lds, idx, x);
                    wave_lds_sync();
                }
        }
        if (lane == 0) {
#pragma unroll
            for (int a = 0; a < DIM; ++a) g.uref[a * g.d.tiles + t] = uref[a];
        }
        slab_store_sums<T, DIM, DEG, COMP>(lds, slabs.v + (int64_t)r * slabs.stride);
        wave_lds_sync();
    }
}

template <typename T, int DIM, int DEG, bool COMP, bool ABS>
__device__ __forceinline__ void p2g_any(const Parts<T> &P, const BinLists &cur, const TileTables &tab,
                                        const Slabs<T> &slabs, const GridState<T> &g, const StepParams<T> &prm, uint32_t blk, uint32_t nblk) {
    if constexpr (p2g_block_per_tile(DIM, DEG))
        p2g_tile3<T, DEG, COMP, ABS>(P, cur, tab, slabs, g, prm, blk, nblk);
    else
        p2g_body<T, DIM, DEG, COMP, ABS>(P, cur, tab, slabs, g, prm, blk, nblk);
}

// Threads of a block.
constexpr int p2g_threads(int dim, int deg, size_t elem) {
    return p2g_block_per_tile(dim, deg) && deg == 3 && elem == 8 ? 512 : 256;
}

// Waves per SIMD that the tile blocks are compiled for: as many as their LDS
// lets a CU hold.
template <typename T, int DIM, int DEG>
constexpr int p2g_min_waves() {
    if (!p2g_block_per_tile(DIM, DEG)) return 1;
    return sizeof(T) == 8 ? 2 : (DEG == 3 ? 3 : 4);
}

template <typename T, int DIM, int DEG, bool COMP, bool ABS>
__global__ __launch_bounds__(p2g_threads(DIM, DEG, sizeof(T))) __attribute__((amdgpu_waves_per_eu(p2g_min_waves<T, DIM, DEG>()))) void k_p2g(
    Parts<T> P, BinLists cur, TileTables tab, Slabs<T> slabs, GridState<T> g, StepParams<T> prm) {
    p2g_any<T, DIM, DEG, COMP, ABS>(P, cur, tab, slabs, g, prm, blockIdx.x, gridDim.x);
}

template <typename T, int DIM, int DEG, bool COMP, bool QUEUE>
__global__ __launch_bounds__(p2g_threads(DIM, DEG, sizeof(T))) __attribute__((amdgpu_waves_per_eu(QUEUE ? 1 : p2g_min_waves<T, DIM, DEG>()))) void k_p2g_batch(
    const SceneDesc<T> *descs, const int32_t *start, int n, int k, BatchQueue q) {
    batch_items<QUEUE>(q, [&](uint32_t it) {
        const BatchStep<T> b = batch_step<T>(descs, start, n, k, it);
        const SceneDesc<T> &d = *b.d;
        // the scene's structs as values: read through the table they would be
        // read again after every store the compiler cannot prove apart
        const Parts<T> P = table_struct(d.bufs[b.sp.src]);
        const TileTables tab = table_struct(d.tab[b.sp.cur]);
        const Slabs<T> slabs = table_struct(d.slabs);
        const GridState<T> g = table_struct(d.g);
        const StepParams<T> prm = table_struct(d.prm);
        p2g_any<T, DIM, DEG, COMP, false>(P, b.cur, tab, slabs, g, prm, b.blk, b.nblk);
    });
}

template <typename T, int DIM, int DEG, bool COMP>
void launch_p2g_batch(const SceneDesc<T> *descs, const int32_t *start, int n, int k, const BatchQueue &q, int blocks,
                      hipStream_t st) {
    if (q.ctr)
        hipLaunchKernelGGL((k_p2g_batch<T, DIM, DEG, COMP, true>), dim3((unsigned)blocks), dim3(p2g_threads(DIM, DEG, sizeof(T))), 0, st, descs,
                           start, n, k, q);
    else
        hipLaunchKernelGGL((k_p2g_batch<T, DIM, DEG, COMP, false>), dim3((unsigned)blocks), dim3(p2g_threads(DIM, DEG, sizeof(T))), 0, st, descs,
                           start, n, k, q);
}

template <typename T, int DIM, int DEG, bool COMP, bool ABS>
void launch_p2g(const Parts<T> &P, const BinLists &cur, const TileTables &tab, const Slabs<T> &slabs,
                 const GridState<T> &g, const StepParams<T> &prm, int64_t max_records,
                hipStream_t st) {
    int64_t blocks = p2g_block_per_tile(DIM, DEG) ? max_records : (max_records + 3) / 4;
    if (blocks < 1) blocks = 1;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL((k_p2g<T, DIM, DEG, COMP, ABS>), dim3((unsigned)blocks), dim3(p2g_threads(DIM, DEG, sizeof(T))), 0, st, P, cur, tab,
                       slabs, g, prm);
}

#define APIC_P2G_INST(T, DIM, DEG)                                                                                \
    template void launch_p2g_batch<T, DIM, DEG, false>(const SceneDesc<T> *, const int32_t *, int, int,               \
                                                       const BatchQueue &, int,                                       \
                                                       hipStream_t);                                              \
    template void launch_p2g_batch<T, DIM, DEG, true>(const SceneDesc<T> *, const int32_t *, int, int,                \
                                                      const BatchQueue &, int,                                        \
                                                      hipStream_t);                                               \
    template void launch_p2g<T, DIM, DEG, false, false>(const Parts<T> &, const BinLists &,    \
                                                        const TileTables &, const Slabs<T> &, const GridState<T> &, \
                                                        const StepParams<T> &, int64_t, hipStream_t);            \
    template void launch_p2g<T, DIM, DEG, true, false>(const Parts<T> &, const BinLists &,     \
                                                       const TileTables &, const Slabs<T> &, const GridState<T> &, \
                                                       const StepParams<T> &, int64_t, hipStream_t);
APIC_P2G_INST(float, 2, 1)
APIC_P2G_INST(float, 3, 1)
APIC_P2G_INST(double, 2, 1)
APIC_P2G_INST(double, 3, 1)
APIC_P2G_INST(float, 2, 2)
APIC_P2G_INST(float, 2, 3)
APIC_P2G_INST(float, 3, 2)
APIC_P2G_INST(float, 3, 3)
APIC_P2G_INST(double, 2, 2)
APIC_P2G_INST(double, 2, 3)
APIC_P2G_INST(double, 3, 2)
APIC_P2G_INST(double, 3, 3)

// absolute binary32 positions: binary32, quadratic and cubic
#define APIC_P2G_ABS_INST(DIM, DEG)                                                                                \
    template void launch_p2g<float, DIM, DEG, false, true>(const Parts<float> &, const BinLists &,              \
                                                           const TileTables &,                 \
                                                           const Slabs<float> &, const GridState<float> &,       \
                                                           const StepParams<float> &, int64_t, hipStream_t);     \
    template void launch_p2g<float, DIM, DEG, true, true>(const Parts<float> &, const BinLists &, \
                                                          const TileTables &, const Slabs<float> &,              \
                                                          const GridState<float> &, const StepParams<float> &,   \
                                                          int64_t, hipStream_t);
APIC_P2G_ABS_INST(2, 2)
APIC_P2G_ABS_INST(2, 3)
APIC_P2G_ABS_INST(3, 2)
APIC_P2G_ABS_INST(3, 3)

}  // namespace apic
