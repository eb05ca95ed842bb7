// Transfer to particles (Sec. 3.4) in its lambda = 0 form (Sec. 5.7), with
// the weights of time n, fused with the re-binning of the particles:
//   v_p = sum_i w_ip vt_i
//   B_p = sum_i w_ip vt_i (x_i - x_p)^T
//   F_p = (I + dt sum_i vt_i grad w_ip^T) F_p
//   x_p = x_p + dt v_p          (cell index + offset)
// Both passes take the listed tiles of the current layout, a wavefront or a
// block of four per tile (TileMode).
// Pass 1 (k_bin_keys_moved) finds the particles whose key changes ("movers",
// rare): each takes a place in its new key and is marked in a bit mask of its
// old key's levels.  Pass 2 (k_g2p) stages the grid velocities around the tile
// in LDS, computes the whole update and writes each particle at its place in
// the new layout (within a key the stayers first, in their old order, then the
// movers that entered it); the masks tell a stayer its rank without a count, so
// the tile's chunks are independent of each other.
// Both passes get the new position through the same fixed operation sequence
// (no contraction freedom), so they agree bit for bit on every key.
#include <algorithm>
#include <type_traits>

#include "apic_kernels.h"
#include "g2p_device.h"

namespace apic {

// Tiles of a block that takes several: four, each a wavefront's; two where the grid
// velocities around four would keep blocks off a CU (binary64 3D).
template <typename T, int DIM, int MODE>
constexpr int keys_tiles() {
    return MODE == BLOCK_PER_TILE ? 1 : (MODE == BY_LAYOUT && sizeof(T) == 8 && DIM == 3 ? 2 : 4);
}
template <typename T, int DIM, int DEG, int MODE>
constexpr int g2p_tiles() {
    return MODE == BLOCK_PER_TILE ? 1 : (MODE == BY_LAYOUT && sizeof(T) == 8 && DIM == 3 && DEG == 1 ? 2 : 4);
}

// Waves per SIMD asked for: a wavefront per tile holds the offsets of eight
// chunks (binary32: three).
template <typename T, int MODE>
constexpr int keys_min_waves() {
    return MODE == WAVE_PER_TILE && sizeof(T) == 4 ? 3 : 1;
}

// Waits for the wavefronts that work on a tile (all of a block's, where there are
// several).
__device__ __forceinline__ void tile_sync(uint32_t wpt) {
    if (wpt > 1u)
        __syncthreads();
    else
        wave_lds_sync();
}

// Work items of a pass over a layout: the tiles, a block each (`whole`) or TILES at a
// time, 4 / TILES wavefronts each, then the chunks of dead particles four at a time.
struct TileItems {
    bool whole;
    uint32_t tiles, dead, count;
};
template <typename T, int DIM, int MODE, int TILES>
__device__ __forceinline__ TileItems tile_items(const TileWalk &walk, int64_t n, uint32_t scenes) {
    TileItems it;
    it.whole = MODE == BLOCK_PER_TILE || (MODE == BY_LAYOUT && block_per_tile<T, DIM>(walk.nrec, walk.live, scenes));
    it.tiles = it.whole ? walk.nrec : (walk.nrec + TILES - 1u) / TILES;
    it.dead = dead_chunks(n, walk.live);
    it.count = it.tiles + (it.dead + 3u) / 4u;
    return it;
}

// --- pass 1: new keys ---------------------------------------------------------------------
// The tile's particles in chunks of 64, dealt to its wavefronts in turn.  A
// particle farther from every key boundary than this step can move it keeps its
// key, and only its offsets are read.  The others are queued in LDS and resolved
// 64 at a time from the grid velocities around the tile, staged in LDS.
// Bounded by the latency of that chain (2.1M particles: 28 us for 25 MB read,
// one wavefront per tile at three per SIMD; four per SIMD spill 22 registers:
// 40 us).  With the bound of |vt| per tile and axis instead of one over the grid,
// and marks for the leavers instead of a count of the stayers, 9.0M particles of
// two colliding spheres take 153 us against 278, 2D 1.19M 23 against 31.
// Busy tiles: their keys written by all wavefronts of the tile and read back eight
// at a time, 1.0M particles at 64 per cell 53 -> 42 (with the passes after it; one
// by one and by the first wavefront alone before).
constexpr int kKeyChunks = 8;  // chunks of a tile loaded together

// Resolves queued particles lane < count (indices in the tile): movers take a
// place in their new key (or among the dead) and are marked in `left` (a bit per
// index); a busy tile (more than kMaxLevels levels) has its particles' keys in
// `pkey` and marks its movers there alone.  The grid velocities around tile t
// (first node `origin`) are staged in `reg`.  Wave-wide.
template <typename T, int DIM, int DEG, bool ABS>
__device__ __forceinline__ void resolve_near(const Parts<T> &P, const GridState<T> &g, const StepParams<T> &prm,
                                             const BinLists &nxt, const BinScratch &sc, const uint32_t *queue,
                                             uint32_t count, uint32_t t, uint32_t start, const int *origin,
                                             const T *reg, uint32_t *left, bool busy) {
    const int lane = lane_id();
    const bool act = (uint32_t)lane < count;
    const uint32_t i = act ? queue[lane] : 0u, q = start + i;
    uint32_t nkey = kDeadKey;
    bool mover = false;
    if (act) {
        int ci[3] = {0, 0, 0}, base[3] = {0, 0, 0}, lk[3] = {0, 0, 0}, cn[3] = {0, 0, 0};
        T x[DIM], off[DIM], w[DIM][DEG + 1], vn[DIM], on[DIM];
#pragma unroll
        for (int a = 0; a < DIM; ++a) x[a] = P.off[a * P.s + q];
        particle_cells<T, DIM, ABS>(ABS ? 0u : P.cell[q], x, g.inv_dx, ci, off);
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            base[a] = axis_w_fixed<T, DEG>(ci[a], off[a], w[a]);
            lk[a] = base[a] - origin[a];
        }
        velocity_lds<T, DIM, DEG>(reg, lk, w, vn);
        bool cfl, finite;
        if constexpr (ABS) {
            T xn[DIM];
            move_absolute<T, DIM>(x, vn, prm.dt, g.inv_dx, xn, cn, on, cfl);
        } else {
            move_position<T, DIM>(ci, off, vn, prm.dt * g.inv_dx, cn, on, cfl);
        }
        nkey = key_of<T, DIM, DEG>(cn, on, g.d, finite);
        if (nkey == kDeadKey) atomicOr(g.flags, finite ? FLAG_OUT_OF_DOMAIN : FLAG_NONFINITE);
        mover = nkey != (busy ? sc.pkey[q] : t * 64 + (uint32_t)local_of<DIM>(base));
        if (mover && !busy) atomicOr(left + (i >> 5), 1u << (i & 31u));
    }
    const uint32_t rank = bin_take_slot(nkey, mover, q, tile_order(t, i), nxt, sc);
    if (mover) {
        sc.pkey[q] = nkey;
        sc.prank[q] = rank;
    }
}

constexpr uint32_t kStayer = 0x80000000u;  // prank of a busy tile's stayer: its rank with this bit

template <typename T, int DIM, int DEG, bool ABS, int MODE>
__device__ __forceinline__ void keys_body(const Parts<T> &P, const BinLists &cur, const TileTables &ctab,
                                          const GridState<T> &g, const StepParams<T> &prm_in, const BinLists &nxt,
                                          const BinScratch &sc, uint32_t scenes, uint32_t blk, uint32_t nblk) {
    const StepParams<T> prm = with_step_dt(prm_in);
    using R = VtRegion<DIM>;
    constexpr int U = MODE == WAVE_PER_TILE ? kKeyChunks : kKeyChunks / 4;  // chunks of a wavefront loaded together
    constexpr int TILES = keys_tiles<T, DIM, MODE>();
    __shared__ uint32_t lds_left[TILES][64];  // a bit per particle of a tile that is not busy
    static_assert(kMaxLevels * 64 <= 64 * 32, "a bit for each");
    __shared__ uint32_t lds_queue[4][64 * U];
    __shared__ T lds_vt[TILES * DIM * R::SIZE];
    const int lane = lane_id(), wave = (int)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t *queue = lds_queue[wave];
    const TileWalk walk = tile_walk(cur);
    TileItems items = tile_items<T, DIM, MODE, TILES>(walk, P.n, scenes);
    if (MODE == WAVE_PER_TILE && dense_tiles(walk.nrec, walk.live, scenes)) {
        items.whole = true;
        items.tiles = walk.nrec;
        items.count = walk.nrec + (items.dead + 3u) / 4u;
    }
    const auto walk_tiles = [&](auto w) {
        // the wavefronts of a tile, which of them this one is, and the tile of the block
        constexpr bool whole = decltype(w)::value;
        constexpr uint32_t wpt = whole ? 4u : 4u / TILES;
        const uint32_t wv = (uint32_t)wave & (wpt - 1u);
        const int tl = whole ? 0 : wave / (4 / TILES);
        uint32_t *left = lds_left[tl];
        T *reg = lds_vt + tl * (DIM * R::SIZE);
        for (uint32_t it = blk; it < items.count; it += nblk) {
            if (it >= items.tiles) {
                // particles that could not be binned stay in the dead region
                const int64_t p = (int64_t)walk.live + ((int64_t)(it - items.tiles) * 4 + wave) * 64 + lane;
                if (p < P.n) sc.prank[p] = atomicAdd(nxt.ctr + kCtrDead, 1u);
                continue;
            }
            const uint32_t r = whole ? it : it * TILES + (uint32_t)tl;
            const bool have = whole || r < walk.nrec;
            if (wpt == 1u && !have) continue;
            uint32_t start, cnt, maxc, kstart;
            const uint32_t t = tile_of_record(walk, have ? r : 0u, cur, ctab, start, cnt, maxc, kstart);
            uint32_t total = ctab.tcount[t];
            if (!have) total = cnt = maxc = 0u;  // no second tile: the wavefronts only wait for the others
            const bool busy = maxc > (uint32_t)kMaxLevels;
            int origin[3] = {0, 0, 0};
            tile_origin<DIM>(t, g.d.TN, origin);
            const float4 bounds = load_bounds<T, DIM>(t, g);
            // the tile is claimed in the new layout now (its particles nearly all
            // stay) and appended at the end, so the claim's round trip overlaps
            // the tile's loads; a tile all of whose particles leave is listed
            // empty, which every later pass takes as a tile without particles
            uint32_t claim = nxt.gen;
            if (wv == 0) {
                left[lane] = 0u;
                if (lane == 0 && total > 0u) claim = atomicExch(nxt.tile_gen + t, nxt.gen);
            }
            if (busy)
                for (uint32_t j = wv; j < cnt; j += wpt) sc.pkey[kstart + j] = t * 64 + (uint32_t)lane;
            bool staged = wpt > 1u;  // one wavefront: grid velocities around the tile on first use
            if constexpr (wpt > 1u) stage_velocities<T, DIM, (int)wpt>(t, g, reg, (int)wv);
            tile_sync(wpt);
            for (uint32_t c0 = 64u * wv; c0 < total; c0 += 64u * U * wpt) {
                T off[U][DIM];
                // every load of the group in flight, then its chunks are classified
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t i = c0 + 64u * wpt * u + (uint32_t)lane;
                    if (i < total) {
                        const uint32_t pb = (start + i) * (uint32_t)sizeof(T);
#pragma unroll
                        for (int a = 0; a < DIM; ++a) off[u][a] = *scalar_plane(P.off + a * P.s, pb);
                    }
                }
                T reach[DIM];
                tile_reach<T, DIM, ABS>(bounds, g, prm, reach);
                uint32_t queued = 0;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t i = c0 + 64u * wpt * u + (uint32_t)lane;
                    if (c0 + 64u * wpt * u >= total) break;
                    bool near = false;
                    if (i < total) {
                        T o[DIM];
                        if constexpr (ABS) {
                            int ci[3];
                            particle_cells<T, DIM, true>(0u, off[u], g.inv_dx, ci, o);
                        } else {
#pragma unroll
                            for (int a = 0; a < DIM; ++a) o[a] = off[u][a];
                        }
                        near = !keeps_key<T, DIM, DEG>(o, reach);
                    }
                    const uint64_t nm = ballot(near);
                    if (near) queue[queued + (uint32_t)popc64(nm & lanes_below(lane))] = i;
                    queued += (uint32_t)popc64(nm);
                }
                if (queued > 0u && !staged) {
                    stage_all<T, DIM, MODE == WAVE_PER_TILE ? 1 : 2>(t, g, reg);
                    staged = true;
                }
                wave_lds_sync();
                for (uint32_t q0 = 0; q0 < queued; q0 += 64u) {
                    const uint32_t take = queued - q0 < 64u ? queued - q0 : 64u;
                    resolve_near<T, DIM, DEG, ABS>(P, g, prm, nxt, sc, queue + q0, take, t, start, origin, reg, left, busy);
                }
                wave_lds_sync();
            }
            tile_sync(wpt);
            if (wv == 0 && have) {
                uint32_t stay;
                if (!busy) {
                    // the marks by key and level
                    uint32_t gone = 0u;
                    if (ballot(left[lane] != 0u)) {
                        uint32_t level = 0;
                        for (uint32_t j0 = 0; j0 < maxc; j0 += 4) {
                            // four marks in flight; an absent level reads one that counts for nothing
                            uint32_t word[4], at[4];
#pragma unroll
                            for (uint32_t u = 0; u < 4; ++u) {
                                const uint64_t mask = ballot(cnt > j0 + u);
                                at[u] = level + (uint32_t)popc64(mask & lanes_below(lane));
                                word[u] = left[(at[u] >> 5) & 63u];
                                level += (uint32_t)popc64(mask);
                            }
#pragma unroll
                            for (uint32_t u = 0; u < 4; ++u)
                                if (cnt > j0 + u) gone |= ((word[u] >> (at[u] & 31u)) & 1u) << (j0 + u);
                        }
                    }
                    stay = cnt - (uint32_t)__popc(gone);
                    ctab.kmov[(int64_t)t * 64 + lane] = gone;
                } else {
                    // a busy tile's particles carry their key and rank themselves
                    // (read eight at a time: the compiler must take each store for one
                    // that may change the next read, a round trip per particle)
                    stay = 0;
                    for (uint32_t j0 = 0; j0 < cnt; j0 += 8u) {
                        uint32_t key[8];
#pragma unroll
                        for (uint32_t u = 0; u < 8u; ++u) key[u] = sc.pkey[kstart + (j0 + u < cnt ? j0 + u : j0)];
#pragma unroll
                        for (uint32_t u = 0; u < 8u; ++u)
                            if (j0 + u < cnt && key[u] == t * 64 + (uint32_t)lane)
                                sc.prank[kstart + j0 + u] = kStayer | stay++;
                    }
                }
                sc.scount[(int64_t)t * 64 + lane] = stay;
                if (lane == 0 && claim != nxt.gen) append_tile(t, nxt);
            }
            if (wpt == 1u) wave_lds_sync();
        }
    };
    if constexpr (MODE == BLOCK_PER_TILE) {
        walk_tiles(std::true_type{});
    } else {
        if (items.whole)
            walk_tiles(std::true_type{});
        else
            walk_tiles(std::false_type{});
    }
}

template <typename T, int DIM, int DEG, bool ABS, int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(keys_min_waves<T, MODE>()))) void k_bin_keys_moved(
    Parts<T> P, BinLists cur, TileTables ctab, GridState<T> g, StepParams<T> prm, BinLists nxt, BinScratch sc) {
    keys_body<T, DIM, DEG, ABS, MODE>(P, cur, ctab, g, prm, nxt, sc, 1u, blockIdx.x, gridDim.x);
}

template <typename T, int DIM, int DEG, bool QUEUE, int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(QUEUE ? 1 : keys_min_waves<T, MODE>()))) void k_bin_keys_moved_batch(
    const SceneDesc<T> *descs, const int32_t *start, int n, int k, BatchQueue q) {
    batch_items<QUEUE>(q, [&](uint32_t it) {
        const BatchStep<T> b = batch_step<T>(descs, start, n, k, it);
        const SceneDesc<T> &d = *b.d;
        // the scene's structs as values: read through the table they would be
        // read again after every store the compiler cannot prove apart
        const Parts<T> P = table_struct(d.bufs[b.sp.src]);
        const TileTables ctab = table_struct(d.tab[b.sp.cur]);
        GridState<T> g = table_struct(d.g);
        g.vmax = tile_bounds(table_struct(d.tab[b.sp.nxt].lvl_off));
        const StepParams<T> prm = table_struct(d.prm);
        const BinScratch sc = table_struct(d.sc);
        keys_body<T, DIM, DEG, false, MODE>(P, b.cur, ctab, g, prm, b.nxt, sc, (uint32_t)n, b.blk, b.nblk);
    });
}

// Runs f with the mode as a compile-time constant.
template <typename F>
static void with_keys_mode(int mode, F &&f) {
    if (mode == WAVE_PER_TILE)
        f(std::integral_constant<int, WAVE_PER_TILE>{});
    else if (mode == BLOCK_PER_TILE)
        f(std::integral_constant<int, BLOCK_PER_TILE>{});
    else
        f(std::integral_constant<int, BY_LAYOUT>{});
}

template <typename T, int DIM, int DEG>
void launch_bin_keys_moved_batch(const SceneDesc<T> *descs, const int32_t *start, int n, int k, const BatchQueue &q,
                                 int blocks, int mode, hipStream_t st) {
    with_keys_mode(mode, [&](auto w) {
        constexpr int MODE = decltype(w)::value;
        if (q.ctr)
            hipLaunchKernelGGL((k_bin_keys_moved_batch<T, DIM, DEG, true, MODE>), dim3((unsigned)blocks), dim3(256), 0,
                               st, descs, start, n, k, q);
        else
            hipLaunchKernelGGL((k_bin_keys_moved_batch<T, DIM, DEG, false, MODE>), dim3((unsigned)blocks), dim3(256), 0,
                               st, descs, start, n, k, q);
    });
}

template <typename T, int DIM, int DEG, bool ABS>
void launch_bin_keys_moved(const Parts<T> &P, const BinLists &cur, const TileTables &ctab, const GridState<T> &g,
                           const StepParams<T> &prm, const BinLists &nxt, const BinScratch &sc, int64_t max_records,
                           hipStream_t st) {
    with_keys_mode(key_mode(P.n, few_tiles<T, DIM>((uint32_t)max_records, 1u)), [&](auto w) {
        constexpr int MODE = decltype(w)::value;
        const int64_t items = (MODE == WAVE_PER_TILE ? (max_records + 3) / 4 : max_records) + (P.n + 255) / 256;
        const int64_t blocks = std::min<int64_t>(std::max<int64_t>(items, 1), 4096);
        hipLaunchKernelGGL((k_bin_keys_moved<T, DIM, DEG, ABS, MODE>), dim3((unsigned)blocks), dim3(256), 0, st, P, cur,
                           ctab, g, prm, nxt, sc);
    });
}

// --- pass 2: the transfer, written to the new layout ------------------------------------
// The tile's particles in chunks of 64 (every lane busy), dealt to its
// wavefronts in turn.  A particle's key and level in the old layout and the
// masks of pass 1 give a stayer's rank in its key: its level less the leavers
// below it.  A mover takes the key of pass 1 and its rank there after the key's
// stayers.  At full size it runs at the copy rate of its own traffic (2.1M
// particles: 427 MB in 91 us, 96 before its stayers took their ranks from the
// marks: no counter, no test of the key, and the tile's level tables from LDS
// instead of two dependent loads per particle).  Below it, vector issue counts:
// with the plane addresses by scalar adds and row sums in the sweep a chunk is
// 760 vector instructions, not 915 (quadratic), and four wavefronts fit a SIMD
// in the cubic too (binary32 quadratic 512,000 particles 29.8 -> 26.1 us, cubic
// 9.0M 724 -> 659, binary64 quadratic 512,000 47 -> 42.5).
// ADAPT: the step's dt comes from the device and the CFL bound of the
// written state is folded into g.cfl (adaptive steps); a separate
// instantiation, so that fixed steps carry none of it.
// FINISH: the new layout's bucket tables are found here, and its records numbered
// (g2p_finishes).
template <typename T, int DIM, int DEG, bool ADAPT, bool ABS, int MODE, bool FINISH>
__device__ __forceinline__ void g2p_body(const Parts<T> &src, const Parts<T> &dst, const BinLists &cur,
                                         const TileTables &ctab, const BinLists &nxt, const TileTables &ntab,
                                         const BinScratch &sc, const GridState<T> &g, const StepParams<T> &prm_in,
                                         uint32_t scenes, uint32_t blk, uint32_t nblk) {
    const StepParams<T> prm = ADAPT ? with_step_dt(prm_in) : prm_in;
    using R = VtRegion<DIM>;
    // the grid velocities around the tiles; before them (FINISH) the bucket tables
    constexpr size_t VT = g2p_tiles<T, DIM, DEG, MODE>() * DIM * R::SIZE * sizeof(T);
    __shared__ __attribute__((aligned(16))) char lds_all[FINISH && sizeof(BucketTables) > VT ? sizeof(BucketTables) : VT];
    T *lds_vt = (T *)lds_all;
    __shared__ uint32_t lds_bpre[FINISH ? kBuckets + 1 : 1];
    constexpr int TILES = g2p_tiles<T, DIM, DEG, MODE>();
    __shared__ uint16_t lds_slot[4][64];  // key | level << 6 of the chunk's particles
    __shared__ uint32_t lds_gone[TILES][64], lds_nlo[TILES][kMaxLevels];
    __shared__ uint64_t lds_nmask[TILES][kMaxLevels];
    const int lane = lane_id(), wave = (int)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint16_t *slot = lds_slot[wave];
    const TileWalk walk = tile_walk(cur);
    if constexpr (FINISH) {
        BucketTables &tables = *(BucketTables *)lds_all;
        bucket_tables(nxt, tables, lds_bpre);
        // from the last block on: those of a launch sized for the capacity have no
        // tile, and the records end with the short ones
        finish_layout(nxt, cur, tables, lds_bpre, nblk - 1u - blk, nblk);
        __syncthreads();
    }
    const auto base_at = [&](uint32_t b) {
        if constexpr (FINISH)
            return lds_bpre[b];
        else
            return nxt.bpre[b];
    };
    const uint32_t live_nxt = base_at(kBuckets);
    const T dt_inv_dx = prm.dt * g.inv_dx, gs = prm.dt * g.inv_dx;
    const TileItems items = tile_items<T, DIM, MODE, TILES>(walk, src.n, scenes);
    // the wavefronts of a tile, which of them this one is, and the tile of the block
    const bool whole = items.whole;
    const uint32_t wpt = whole ? 4u : 4u / TILES, wv = (uint32_t)wave & (wpt - 1u);
    const int tl = whole ? 0 : wave / (4 / TILES);
    T *reg = lds_vt + tl * (DIM * R::SIZE);
    uint32_t *gone = lds_gone[tl], *nlo = lds_nlo[tl];
    uint64_t *nmask = lds_nmask[tl];
    const bool ids = src.id != nullptr;
    T cmax = T(0);  // CFL bound of the particles this lane writes (when asked)
    for (uint32_t it = blk; it < items.count; it += nblk) {
        if (it >= items.tiles) {
            const uint32_t c = (it - items.tiles) * 4u + (uint32_t)wave;
            if (c < items.dead) carry_dead<T, DIM>(src, dst, sc, walk.live, live_nxt, c);
            continue;
        }
        const uint32_t r = whole ? it : it * TILES + (uint32_t)tl;
        const bool have = r < walk.nrec;
        if (TILES == 4 && !have) continue;
        const uint32_t t = cur.rec_tile[have ? r : 0u];
        const uint32_t start = walk.bbase[bucket_of(t)] + ctab.off[t], total = ctab.tcount[t], maxc = ctab.maxc[t];
        const uint32_t cnt = ctab.kcount[(int64_t)t * 64 + lane];
        const uint32_t nbase = base_at(bucket_of(t)) + ntab.off[t];  // the tile's place in the new layout
        const bool busy = maxc > (uint32_t)kMaxLevels, nbusy = ntab.maxc[t] > (uint32_t)kMaxLevels;
        int origin[3] = {0, 0, 0};
        tile_origin<DIM>(t, g.d.TN, origin);
        // chunks of 64 start on 32-particle boundaries (128 B in binary32)
        // of the tile's place in the new layout: the particles keep their
        // order there up to the few that change key, so each chunk writes
        // whole cache lines (the writes move twice the bytes of the reads,
        // which now start mid-line), and the next step's transfer to grid
        // reads lines written whole.  The first chunk is in flight while the
        // grid velocities are staged and the tables filled.
        // (no second tile: nothing to do, but the waits for the others)
        const uint32_t head = nbase & 31u, span = have ? total + head : 0u, first = start - head;
        uint32_t e = wv * 64u + (uint32_t)lane;
        G2PRaw<T, DIM> raw;
        if (e >= head && e < span) g2p_load<T, DIM, ABS>(src, first + e, raw);
        if (__builtin_expect(whole, 1))
            stage_velocities<T, DIM, 4>(t, g, reg, wave);
        else if (TILES == 2)
            stage_velocities<T, DIM, 2>(t, g, reg, (int)wv);
        else
            stage_all<T, DIM, 1>(t, g, reg);
        if (wv == 0) gone[lane] = ctab.kmov[(int64_t)t * 64 + lane];
        if (wv == wpt - 1u && lane < kMaxLevels) {
            nlo[lane] = nbase + ntab.lvl_off[(int64_t)t * kMaxLevels + lane];
            nmask[lane] = ntab.lvl_mask[(int64_t)t * kMaxLevels + lane];
        }
        tile_sync(wpt);
        uint32_t lv = 0, lv_off = 0;  // level the next chunk may start in, its first particle
        for (uint32_t c0 = wv * 64u; c0 < span; c0 += 64u * wpt, e += 64u * wpt) {
            // the wavefront's next chunk is in flight while this one is computed
            G2PRaw<T, DIM> raw_n;
            if (e + 64u * wpt < span) g2p_load<T, DIM, ABS>(src, first + e + 64u * wpt, raw_n);
            // key and level of the chunk's particles from the levels it meets
            while (lv < maxc && !busy) {
                const uint64_t mask = ballot(cnt > lv);
                const uint32_t at = head + lv_off + (uint32_t)popc64(mask & lanes_below(lane)) - c0;
                if (cnt > lv && at < 64u) slot[at] = (uint16_t)((uint32_t)lane | lv << 6);
                const uint32_t end = lv_off + (uint32_t)popc64(mask);
                if (head + end > c0 + 64u) break;
                lv_off = end;
                ++lv;
            }
            wave_lds_sync();
            if (e >= head && e < span) {
                const uint32_t p = first + e;
                int cn[3] = {0, 0, 0}, lk[3] = {0, 0, 0};
                T on[DIM], vn[DIM], Bs[DIM * DIM], Fn[DIM * DIM], xs[DIM];
                g2p_update<T, DIM, DEG, ABS>(raw, reg, origin, g, dt_inv_dx, gs, lk, cn, on, vn, Bs, Fn, prm.transfer,
                                             xs, prm.dt);
                bool stays;
                uint32_t key, rank;
                if (!busy) {
                    const uint32_t s = slot[lane], j = s >> 6;
                    key = s & 63u;
                    const uint32_t m = gone[key];
                    stays = !((m >> j) & 1u);
                    rank = j - (uint32_t)__popc(m & ((1u << j) - 1u));
                } else {
                    rank = sc.prank[p];
                    stays = (rank & kStayer) != 0u;
                    rank &= ~kStayer;
                    key = sc.pkey[p] & 63u;
                }
                uint32_t q;
                if (stays && !nbusy) {
                    q = nlo[rank] + (uint32_t)popc64(nmask[rank] & lanes_below((int)key));
                } else if (stays) {
                    q = nbase + ntab.kprefix[(int64_t)t * 64 + key] + rank;
                } else {
                    const uint32_t dkey = sc.pkey[p];
                    const uint32_t drank = sc.prank[p] + (dkey == kDeadKey ? 0u : ntab.kcount[dkey] - ntab.kmov[dkey]);
                    const uint32_t dbase = dkey == kDeadKey ? 0u : base_at(bucket_of(dkey >> 6));
                    q = bin_destination(dkey, drank, ntab, dbase, live_nxt);
                }
                // keep the packed index representable; a particle that left
                // the grid is in the dead region and is not transferred again
#pragma unroll
                for (int a = 0; a < DIM; ++a) cn[a] = cn[a] < 0 ? 0 : (cn[a] > g.d.n[a] - 1 ? g.d.n[a] - 1 : cn[a]);
                g2p_store<T, DIM>(dst, q, pack_cell<DIM>(cn), raw, ids, ABS ? xs : on, vn, Bs, Fn);
                // after the stores, when the particle's other values are dead
                if constexpr (ADAPT) cfl_fold<T, DIM>(vn, Bs, g.cfl_c, cmax);
            }
            raw = raw_n;
            wave_lds_sync();
        }
        tile_sync(wpt);
    }
    if constexpr (ADAPT) cfl_raise(g.cfl, blk * 4 + (uint32_t)wave, (double)cmax);
    (void)cmax;
}

template <typename T, int DIM, int DEG, bool ADAPT, bool ABS, int MODE, bool FINISH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(ADAPT && DIM == 3 ? 1 : g2p_min_waves<T, DIM, DEG>()))) void k_g2p(
    Parts<T> src, Parts<T> dst, BinLists cur, TileTables ctab, BinLists nxt, TileTables ntab, BinScratch sc,
    GridState<T> g, StepParams<T> prm) {
    g2p_body<T, DIM, DEG, ADAPT, ABS, MODE, FINISH>(src, dst, cur, ctab, nxt, ntab, sc, g, prm, 1u, blockIdx.x,
                                                    gridDim.x);
}

template <typename T, int DIM, int DEG, bool ADAPT, bool QUEUE, int MODE, bool FINISH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(QUEUE ? 1 : g2p_min_waves<T, DIM, DEG>()))) void k_g2p_batch(
    const SceneDesc<T> *descs, const int32_t *start, int n, int k, BatchQueue q) {
    batch_items<QUEUE>(q, [&](uint32_t it) {
        const BatchStep<T> b = batch_step<T>(descs, start, n, k, it);
        const SceneDesc<T> &d = *b.d;
        Parts<T> src = table_struct(d.bufs[b.sp.src]), dst = table_struct(d.bufs[b.sp.src ^ 1]);
        if (!src.id || !dst.id) src.id = dst.id = nullptr;
        // the scene's structs as values: read through the table they would be
        // read again after every store the compiler cannot prove apart
        const TileTables ctab = table_struct(d.tab[b.sp.cur]), ntab = table_struct(d.tab[b.sp.nxt]);
        const BinScratch sc = table_struct(d.sc);
        const GridState<T> g = table_struct(d.g);
        const StepParams<T> prm = table_struct(d.prm);
        g2p_body<T, DIM, DEG, ADAPT, false, MODE, FINISH>(src, dst, b.cur, ctab, b.nxt, ntab, sc, g, prm, (uint32_t)n,
                                                          b.blk, b.nblk);
    });
}

// Runs f with the mode and FINISH as compile-time constants.
template <typename T, int DIM, int DEG, typename F>
static void with_g2p_mode(int mode, bool finish, F &&f) {
    using Block = std::integral_constant<int, BLOCK_PER_TILE>;
    using Layout = std::integral_constant<int, BY_LAYOUT>;
    if (finish) {
        if (mode == BLOCK_PER_TILE)
            f(Block{}, std::true_type{});
        else
            f(Layout{}, std::true_type{});
        return;
    }
    if constexpr (g2p_wave_choice<T, DIM, DEG>()) {
        if (mode == WAVE_PER_TILE) {
            f(std::integral_constant<int, WAVE_PER_TILE>{}, std::false_type{});
            return;
        }
    }
    f(Layout{}, std::false_type{});
}

template <typename T, int DIM, int DEG>
void launch_g2p_batch(const SceneDesc<T> *descs, const int32_t *start, int n, int k, const BatchQueue &q, int blocks,
                      bool adapt, int mode, bool finish, hipStream_t st) {
    const dim3 grid((unsigned)blocks), block(256);
    with_g2p_mode<T, DIM, DEG>(mode, finish, [&](auto w, auto f) {
        constexpr int MODE = decltype(w)::value;
        constexpr bool FINISH = decltype(f)::value;
        if (adapt && q.ctr)
            hipLaunchKernelGGL((k_g2p_batch<T, DIM, DEG, true, true, MODE, FINISH>), grid, block, 0, st, descs, start, n,
                               k, q);
        else if (adapt)
            hipLaunchKernelGGL((k_g2p_batch<T, DIM, DEG, true, false, MODE, FINISH>), grid, block, 0, st, descs, start,
                               n, k, q);
        else if (q.ctr)
            hipLaunchKernelGGL((k_g2p_batch<T, DIM, DEG, false, true, MODE, FINISH>), grid, block, 0, st, descs, start,
                               n, k, q);
        else
            hipLaunchKernelGGL((k_g2p_batch<T, DIM, DEG, false, false, MODE, FINISH>), grid, block, 0, st, descs, start,
                               n, k, q);
    });
}

// --- adaptive batched steps (Sec. 4.3) ---------------------------------------------
// One block per scene: zero its bound slots.
template <typename T>
__global__ __launch_bounds__(256) void k_cfl_clear_batch(const SceneDesc<T> *descs) {
    unsigned long long *slots = descs[blockIdx.x].g.cfl;
    for (int i = (int)threadIdx.x; i < kCflSlots; i += (int)blockDim.x) slots[i] = 0ull;
}

// Blocks by particle count (start): each scene's bound over the particles
// it starts the call with, raised into its slots.
template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_cfl_bound_batch(const SceneDesc<T> *descs, const int32_t *start, int n) {
    const int s = scene_of_block(start, n, blockIdx.x);
    const SceneDesc<T> &d = descs[s];
    const Parts<T> P = d.bufs[d.where0];
    const uint32_t b = blockIdx.x - (uint32_t)start[s], nb = (uint32_t)(start[s + 1] - start[s]);
    double m = 0.0;
    for (int64_t p = (int64_t)b * 256 + threadIdx.x; p < P.n; p += (int64_t)nb * 256) {
        T v[DIM], B[DIM * DIM];
#pragma unroll
        for (int a = 0; a < DIM; ++a) v[a] = P.v[a * P.s + p];
#pragma unroll
        for (int q = 0; q < DIM * DIM; ++q) B[q] = P.B[q * P.s + p];
        cfl_fold64<T, DIM>(v, B, d.g.cfl_c, m);
    }
    cfl_raise(d.g.cfl, b * 4 + (threadIdx.x >> 6), m);
}

// One wavefront per scene: dt = min(dt_cap, nu_dx / bound) from its slots
// (bound 0 or NaN: dt_cap), recorded with the running time; slots zeroed.
template <typename T>
__global__ __launch_bounds__(64) void k_adapt_dt_batch(const SceneDesc<T> *descs) {
    const SceneDesc<T> &d = descs[blockIdx.x];
    const int lane = (int)threadIdx.x;
    unsigned long long *slots = d.g.cfl;
    double bnd = 0.0;
    for (int i = lane; i < kCflSlots; i += 64) {
        const double y = __longlong_as_double((long long)slots[i]);
        bnd = y > bnd || y != y ? y : bnd;
        slots[i] = 0ull;
    }
    for (int o = 32; o > 0; o >>= 1) {
        const double y = __shfl_xor(bnd, o, 64);
        bnd = y > bnd || y != y ? y : bnd;
    }
    if (lane == 0) {
        double dt = d.dt_cap;
        if (bnd > 0.0) {
            const double c = d.nu_dx / bnd;
            dt = c < dt ? c : dt;
        }
        double *state = const_cast<double *>(d.prm.dt_dev);
        state[0] = dt;
        state[1] += dt;
    }
}

template <typename T, int DIM>
void launch_adapt_dt_batch(const SceneDesc<T> *descs, const int32_t *copy_start, int n, int copy_blocks, bool first,
                           hipStream_t st) {
    if (first) {
        hipLaunchKernelGGL((k_cfl_clear_batch<T>), dim3((unsigned)n), dim3(256), 0, st, descs);
        hipLaunchKernelGGL((k_cfl_bound_batch<T, DIM>), dim3((unsigned)copy_blocks), dim3(256), 0, st, descs,
                           copy_start, n);
    }
    hipLaunchKernelGGL((k_adapt_dt_batch<T>), dim3((unsigned)n), dim3(64), 0, st, descs);
}

template <typename T, int DIM, int DEG, bool ABS>
void launch_g2p(const Parts<T> &src, const Parts<T> &dst, const BinLists &cur, const TileTables &ctab,
                const BinLists &nxt, const TileTables &ntab, const BinScratch &sc, const GridState<T> &g,
                const StepParams<T> &prm, int64_t max_records, bool finish, hipStream_t st) {
    if (src.n == 0) return;
    Parts<T> s2 = src, d2 = dst;
    if (!src.id || !dst.id) s2.id = d2.id = nullptr;
    const int mode = g2p_mode<T, DIM, DEG>(src.n, few_tiles<T, DIM>((uint32_t)max_records, 1u));
    with_g2p_mode<T, DIM, DEG>(mode, finish, [&](auto w, auto f) {
        constexpr int MODE = decltype(w)::value;
        constexpr bool FINISH = decltype(f)::value;
        const int64_t items = (MODE == WAVE_PER_TILE ? (max_records + 3) / 4 : max_records) + (src.n + 255) / 256;
        const dim3 blocks((unsigned)std::min<int64_t>(std::max<int64_t>(items, 1), 4096));
        if constexpr (!ABS) {
            if (g.cfl) {
                hipLaunchKernelGGL((k_g2p<T, DIM, DEG, true, false, MODE, FINISH>), blocks, dim3(256), 0, st, s2, d2,
                                   cur, ctab, nxt, ntab, sc, g, prm);
                return;
            }
        }
        hipLaunchKernelGGL((k_g2p<T, DIM, DEG, false, ABS, MODE, FINISH>), blocks, dim3(256), 0, st, s2, d2, cur, ctab,
                           nxt, ntab, sc, g, prm);
    });
}

#define APIC_G2P_INST(T, DIM, DEG)                                                                               \
    template void launch_bin_keys_moved_batch<T, DIM, DEG>(const SceneDesc<T> *, const int32_t *, int, int,           \
                                                           const BatchQueue &, int, int,                              \
                                                           hipStream_t);                                          \
    template void launch_g2p_batch<T, DIM, DEG>(const SceneDesc<T> *, const int32_t *, int, int,                      \
                                                const BatchQueue &, int, bool, int, bool,                             \
                                                hipStream_t);                                                     \
    template void launch_bin_keys_moved<T, DIM, DEG, false>(const Parts<T> &, const BinLists &, const TileTables &, \
                                                            const GridState<T> &, const StepParams<T> &,         \
                                                            const BinLists &, const BinScratch &, int64_t,       \
                                                            hipStream_t);                                         \
    template void launch_g2p<T, DIM, DEG, false>(const Parts<T> &, const Parts<T> &, const BinLists &,           \
                                                 const TileTables &, const BinLists &, const TileTables &,       \
                                                 const BinScratch &, const GridState<T> &, const StepParams<T> &, \
                                                 int64_t, bool, hipStream_t);
APIC_G2P_INST(float, 2, 1)
APIC_G2P_INST(float, 3, 1)
APIC_G2P_INST(double, 2, 1)
APIC_G2P_INST(double, 3, 1)
APIC_G2P_INST(float, 2, 2)
APIC_G2P_INST(float, 2, 3)
APIC_G2P_INST(float, 3, 2)
APIC_G2P_INST(float, 3, 3)
APIC_G2P_INST(double, 2, 2)
APIC_G2P_INST(double, 2, 3)
APIC_G2P_INST(double, 3, 2)
APIC_G2P_INST(double, 3, 3)

// absolute binary32 positions: binary32, quadratic and cubic, fixed steps
#define APIC_G2P_ABS_INST(DIM, DEG)                                                                               \
    template void launch_bin_keys_moved<float, DIM, DEG, true>(                                                   \
        const Parts<float> &, const BinLists &, const TileTables &, const GridState<float> &,                    \
        const StepParams<float> &, const BinLists &, const BinScratch &, int64_t, hipStream_t);                  \
    template void launch_g2p<float, DIM, DEG, true>(const Parts<float> &, const Parts<float> &, const BinLists &, \
                                                    const TileTables &, const BinLists &, const TileTables &,    \
                                                    const BinScratch &, const GridState<float> &,                \
                                                    const StepParams<float> &, int64_t, bool, hipStream_t);
APIC_G2P_ABS_INST(2, 2)
APIC_G2P_ABS_INST(2, 3)
APIC_G2P_ABS_INST(3, 2)
APIC_G2P_ABS_INST(3, 3)

template void launch_adapt_dt_batch<float, 2>(const SceneDesc<float> *, const int32_t *, int, int, bool, hipStream_t);
template void launch_adapt_dt_batch<float, 3>(const SceneDesc<float> *, const int32_t *, int, int, bool, hipStream_t);
template void launch_adapt_dt_batch<double, 2>(const SceneDesc<double> *, const int32_t *, int, int, bool,
                                               hipStream_t);
template void launch_adapt_dt_batch<double, 3>(const SceneDesc<double> *, const int32_t *, int, int, bool,
                                               hipStream_t);

}  // namespace apic
