// Binning of particles by base node (apic_sort, and the passes shared with
// the re-binning done by apic_g2p).  Integer work only: counts, prefix sums,
// lists and destinations; nothing here depends on the method's arithmetic.
#include "apic_bin_device.h"
#include "apic_kernels.h"

namespace apic {

static inline int blocks_for(int64_t work, int threads, int cap) {
    int64_t b = (work + threads - 1) / threads;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (int)b;
}

// --- keys of particles at their current position (apic_sort): each takes a
// provisional rank in its key from the key's counter, the order the device runs
// its atomics in; the gather pass orders a key's particles by their index.
// COPY: the particles are also copied to `to` (where the gather reads them when
// it writes over `P`), while the counters' round trips are under way ---------------
template <typename T, int DIM, int DEG, bool ABS, bool COPY>
__global__ __launch_bounds__(256) void k_bin_keys_static(Parts<T> P, Parts<T> to, GridDims d, BinLists nxt,
                                                         BinScratch sc, uint32_t *flags, T inv_dx) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool active = p < P.n;
    uint32_t key = kDeadKey;
    ParticleState<T, DIM> state;
    if (active) {
        int ci[3] = {0, 0, 0};
        T x[DIM], off[DIM];
#pragma unroll
        for (int a = 0; a < DIM; ++a) x[a] = P.off[a * P.s + p];
        const uint32_t cell = ABS ? 0u : P.cell[p];
        if constexpr (COPY) load_particle<T, DIM>(P, (uint32_t)p, P.id != nullptr, state);
        particle_cells<T, DIM, ABS>(cell, x, inv_dx, ci, off);
        bool finite;
        key = key_of<T, DIM, DEG>(ci, off, d, finite);
        if (key == kDeadKey) atomicOr(flags, finite ? FLAG_OUT_OF_DOMAIN : FLAG_NONFINITE);
    }
    uint32_t rank = 0u;
    if (active) rank = atomicAdd(key == kDeadKey ? nxt.ctr + kCtrDead : sc.key_count + key, 1u);
    if (first_lane_of_value(key >> 6, active && key != kDeadKey)) list_tile(key >> 6, nxt);
    if (active) {
        if constexpr (COPY) store_particle<T, DIM>(to, (uint32_t)p, P.id != nullptr, state);
        sc.pkey[p] = key;
        sc.prank[p] = rank;
    }
}

template <typename T, int DIM, int DEG, bool ABS>
void launch_bin_keys_static(const Parts<T> &P, const Parts<T> *to, const GridDims &d, const BinLists &nxt,
                            const BinScratch &sc, uint32_t *flags, T inv_dx, hipStream_t st) {
    if (P.n == 0) return;
    Parts<T> s2 = P, d2 = to ? *to : P;
    if (!s2.id || !d2.id) s2.id = d2.id = nullptr;
    const dim3 blocks((unsigned)((P.n + 255) / 256));
    if (to)
        hipLaunchKernelGGL((k_bin_keys_static<T, DIM, DEG, ABS, true>), blocks, dim3(256), 0, st, s2, d2, d, nxt, sc,
                           flags, inv_dx);
    else
        hipLaunchKernelGGL((k_bin_keys_static<T, DIM, DEG, ABS, false>), blocks, dim3(256), 0, st, s2, d2, d, nxt, sc,
                           flags, inv_dx);
}

// --- per listed tile: counts, prefix sums, tile offset, level table ------------------
__device__ __forceinline__ uint32_t wave_excl_scan(uint32_t x, uint32_t &total) {
    const int lane = lane_id();
    uint32_t inc = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    total = __shfl(inc, 63, 64);
    return inc - x;
}

template <int DIM, bool STATIC = false>
__device__ __forceinline__ void records_body(const BinLists &nxt, const TileTables &tab, const BinScratch &sc,
                                             const GridDims &d, uint32_t blk, uint32_t nblk) {
    __shared__ uint32_t rpre[kBuckets + 4];
    const int lane = lane_id();
    const uint32_t total_recs = block_bucket_prefix(nxt.rec_count, rpre, rpre + kBuckets);
    for (uint32_t r = blk * 4 + (threadIdx.x >> 6); r < total_recs; r += nblk * 4) {
        const uint32_t b = bucket_find(rpre, r);
        const uint32_t t = nxt.rec_list[(int64_t)b * nxt.rcap + (r - rpre[b])];
        const int64_t key = (int64_t)t * 64 + lane;
        const uint32_t mov = sc.key_count[key], stay = sc.scount[key], h = !STATIC && mov ? sc.head[key] : 0u;
        const uint32_t c = mov + stay;
        sc.key_count[key] = 0u;
        sc.scount[key] = 0u;
        if (h) {
            sc.head[key] = 0u;
            rank_movers<DIM == 2 ? 8 : 0>(h, mov, sc);
        }
        uint32_t total;
        const uint32_t kp = wave_excl_scan(c, total);
        const uint32_t mx = wave_max_u32(c);
        tab.kcount[key] = c;
        tab.kmov[key] = mov;
        tab.kprefix[key] = kp;
        if (lane == 0) {
            tab.maxc[t] = mx;
            tab.tcount[t] = total;
            tab.off[t] = atomicAdd(nxt.tot + b, total);
            // rank among the bucket's tiles of its class (high bit: fewer
            // than kFullTile particles); the finalize pass makes it the
            // tile's record number
            nxt.slot[t] = total >= kFullTile ? atomicAdd(nxt.nfull + b, 1u)
                                             : (0x80000000u | atomicAdd(nxt.nsparse + b, 1u));
        }
        if (mx <= (uint32_t)kMaxLevels) {
            // level jj holds the jj-th particle of every key with more than jj
            uint32_t level = 0, my_off = 0;
            uint64_t my_mask = 0;
            for (uint32_t jj = 0; jj < mx; ++jj) {
                const uint64_t mask = ballot(c > jj);
                if ((uint32_t)lane == jj) {
                    my_off = level;
                    my_mask = mask;
                }
                level += (uint32_t)popc64(mask);
            }
            if ((uint32_t)lane < mx) {
                tab.lvl_off[(int64_t)t * kMaxLevels + lane] = my_off;
                tab.lvl_mask[(int64_t)t * kMaxLevels + lane] = my_mask;
            }
        }
    }
}

// STATIC: a build from scratch, whose particles are on no mover lists.
template <int DIM, bool STATIC>
__global__ __launch_bounds__(256) void k_bin_records(BinLists nxt, TileTables tab, BinScratch sc, GridDims d) {
    records_body<DIM, STATIC>(nxt, tab, sc, d, blockIdx.x, gridDim.x);
}

template <typename T, int DIM, bool QUEUE>
__global__ __launch_bounds__(256) void k_bin_records_batch(const SceneDesc<T> *descs, const int32_t *start, int n,
                                                           int k, BatchQueue q) {
    batch_items<QUEUE>(q, [&](uint32_t it) {
        const BatchStep<T> b = batch_step<T>(descs, start, n, k, it);
        const SceneDesc<T> &d = *b.d;
        // the scene's structs as values: read through the table they would be
        // read again after every store the compiler cannot prove apart
        const TileTables tab = table_struct(d.tab[b.sp.nxt]);
        const BinScratch sc = table_struct(d.sc);
        const GridDims dims = table_struct(d.g.d);
        records_body<DIM>(b.nxt, tab, sc, dims, b.blk, b.nblk);
    });
}

template <typename T, int DIM>
void launch_bin_records_batch(const SceneDesc<T> *descs, const int32_t *start, int n, int k, const BatchQueue &q,
                              int blocks, hipStream_t st) {
    if (q.ctr)
        hipLaunchKernelGGL((k_bin_records_batch<T, DIM, true>), dim3((unsigned)blocks), dim3(256), 0, st, descs, start,
                           n, k, q);
    else
        hipLaunchKernelGGL((k_bin_records_batch<T, DIM, false>), dim3((unsigned)blocks), dim3(256), 0, st, descs,
                           start, n, k, q);
}

// copies the particles of every scene that ended in the workspace shadow
// back to the caller's planes
template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_copy_back_batch(const SceneDesc<T> *descs, const int32_t *start, int n,
                                                         int k) {
    const BatchStep<T> b = batch_step<T>(descs, start, n, k, blockIdx.x);
    if (b.sp.src != 1) return;
    const Parts<T> src = table_struct(b.d->bufs[1]), dst = table_struct(b.d->bufs[0]);
    const bool ids = src.id != nullptr && dst.id != nullptr;
    for (int64_t j = (int64_t)b.blk * blockDim.x + threadIdx.x; j < src.n; j += (int64_t)b.nblk * blockDim.x)
        copy_particle<T, DIM>(src, dst, (uint32_t)j, (uint32_t)j, ids);
}

template <typename T, int DIM>
void launch_copy_back_batch(const SceneDesc<T> *descs, const int32_t *start, int n, int k, int blocks,
                            hipStream_t st) {
    hipLaunchKernelGGL((k_copy_back_batch<T, DIM>), dim3((unsigned)blocks), dim3(256), 0, st, descs, start, n, k);
}

// --- prefix tables and record numbers of a finished layout --------------------------
// (bucket_tables, finish_layout)
__global__ __launch_bounds__(256) void k_bin_finalize(BinLists nxt, BinLists other) {
    __shared__ BucketTables tables;
    __shared__ uint32_t bpre[kBuckets + 1];
    bucket_tables(nxt, tables, bpre);
    finish_layout(nxt, other, tables, bpre, blockIdx.x, gridDim.x);
}

void launch_bin_finalize(const BinLists &nxt, const BinLists &other, int64_t max_records, hipStream_t st) {
    hipLaunchKernelGGL(k_bin_finalize, dim3(blocks_for(max_records, 256, 128)), dim3(256), 0, st, nxt, other);
}

template <typename T>
__global__ __launch_bounds__(256) void k_bin_finalize_batch(const SceneDesc<T> *descs, const int32_t *start, int n,
                                                            int k) {
    const BatchStep<T> b = batch_step<T>(descs, start, n, k, blockIdx.x);
    __shared__ BucketTables tables;
    __shared__ uint32_t bpre[kBuckets + 1];
    bucket_tables(b.nxt, tables, bpre);
    finish_layout(b.nxt, b.cur, tables, bpre, b.blk, b.nblk);
}

template <typename T>
void launch_bin_finalize_batch(const SceneDesc<T> *descs, const int32_t *start, int n, int k, int blocks,
                               hipStream_t st) {
    hipLaunchKernelGGL(k_bin_finalize_batch<T>, dim3((unsigned)blocks), dim3(256), 0, st, descs, start, n, k);
}
template void launch_bin_finalize_batch<float>(const SceneDesc<float> *, const int32_t *, int, int, int, hipStream_t);
template void launch_bin_finalize_batch<double>(const SceneDesc<double> *, const int32_t *, int, int, int,
                                                hipStream_t);

template <int DIM>
void launch_bin_records(const GridDims &d, const BinLists &nxt, const TileTables &tab, const BinScratch &sc,
                        int64_t max_records, bool from_scratch, hipStream_t st) {
    const dim3 blocks(blocks_for(max_records, 4, 2048));
    if (from_scratch)
        hipLaunchKernelGGL((k_bin_records<DIM, true>), blocks, dim3(256), 0, st, nxt, tab, sc, d);
    else
        hipLaunchKernelGGL((k_bin_records<DIM, false>), blocks, dim3(256), 0, st, nxt, tab, sc, d);
}

// --- moves every particle to its binned position (apic_sort) ------------------------
// First every key's particles are listed (key after key, in provisional order;
// the dead after all), then a block per tile puts each key's list in order in
// LDS and gathers the tile's particles plane by plane: whole-line writes and one
// scattered read per value, where moving each particle from its old place wrote
// parts of lines that several XCDs' caches held (2.1M binary32 particles in
// lexicographic order: 805 us, the two passes now 18 and 216; 4,096 of them: 17
// us, now 3 and 12, where launches and round trips bound both).
// A tile stored key by key (a key of more than kMaxLevels) is ordered the same way,
// in LDS or, if it has too many for that, in `prank`: gathered key after key by a
// wavefront each, its reads and writes were scattered in time (1.0M particles at 27
// per cell, given in order: 484 us with the passes before it, now 248).
// FINISH: each block finds the bucket tables, and the layout is finished here.
template <bool FINISH>
__global__ __launch_bounds__(256) void k_bin_place(int64_t n, BinLists nxt, BinLists other, TileTables tab,
                                                   BinScratch sc) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t key = p < n ? sc.pkey[p] : kDeadKey, rank = p < n ? sc.prank[p] : 0u;
    const bool dead = key == kDeadKey;
    const uint32_t in_bucket = dead ? 0u : tab.off[key >> 6] + tab.kprefix[key];
    const uint32_t b = dead ? (uint32_t)kBuckets : bucket_of(key >> 6);
    uint32_t base;
    if constexpr (FINISH) {
        __shared__ BucketTables tables;
        __shared__ uint32_t bpre[kBuckets + 1];
        bucket_tables(nxt, tables, bpre);
        finish_layout(nxt, other, tables, bpre, blockIdx.x, gridDim.x);
        base = bpre[b];
    } else {
        base = nxt.bpre[b];
    }
    if (p < n) sc.next[base + in_bucket + rank] = (uint32_t)p;
}

template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_bin_gather(Parts<T> src, Parts<T> dst, BinLists nxt, TileTables tab,
                                                    BinScratch sc) {
    __shared__ uint32_t listed[64 * kMaxLevels], order[64 * kMaxLevels];
    __shared__ uint32_t lvl_off[kMaxLevels];
    __shared__ uint64_t lvl_mask[kMaxLevels];
    const int lane = lane_id(), wv = (int)(threadIdx.x >> 6);
    const TileWalk walk = tile_walk(nxt);
    const uint32_t *src_of = sc.next;
    const bool ids = src.id != nullptr;
    const uint32_t dead = (uint32_t)((src.n - (int64_t)walk.live + 255) / 256);
    for (uint32_t r = blockIdx.x; r < walk.nrec + dead; r += gridDim.x) {
        if (r >= walk.nrec) {
            const uint32_t q = walk.live + (r - walk.nrec) * 256u + threadIdx.x;
            if ((int64_t)q < src.n) copy_particle<T, DIM>(src, dst, src_of[q], q, ids);
            continue;
        }
        uint32_t start, cnt, maxc, kstart;
        const uint32_t t = tile_of_record(walk, r, nxt, tab, start, cnt, maxc, kstart);
        const uint32_t total = tab.tcount[t], kp = tab.kprefix[(int64_t)t * 64 + lane];
        const bool busy = maxc > (uint32_t)kMaxLevels;
        if (total > 64u * (uint32_t)kMaxLevels) {
            // (too many for the LDS; ranks are not needed any more: the order goes there)
            for (uint32_t j = (uint32_t)wv; j < cnt; j += 4u) {
                const uint32_t p = src_of[kstart + j];
                uint32_t rank = 0;
                for (uint32_t i = 0; i < cnt; ++i) rank += src_of[kstart + i] < p ? 1u : 0u;
                sc.prank[kstart + rank] = p;
            }
            __syncthreads();
            for (uint32_t i = threadIdx.x; i < total; i += 256u)
                copy_particle<T, DIM>(src, dst, sc.prank[start + i], start + i, ids);
            continue;
        }
        for (uint32_t i = threadIdx.x; i < total; i += 256u) listed[i] = src_of[start + i];
        if (wv == 0 && lane < kMaxLevels && !busy) {
            lvl_off[lane] = tab.lvl_off[(int64_t)t * kMaxLevels + lane];
            lvl_mask[lane] = tab.lvl_mask[(int64_t)t * kMaxLevels + lane];
        }
        __syncthreads();
        for (uint32_t j = (uint32_t)wv; j < cnt; j += 4u) {
            const uint32_t p = listed[kp + j];
            uint32_t rank = 0;
            for (uint32_t i = 0; i < cnt; ++i) rank += listed[kp + i] < p ? 1u : 0u;
            if (busy)  // key by key: a particle's place is its rank in its key
                order[kp + rank] = p;
            else
                order[lvl_off[rank] + (uint32_t)popc64(lvl_mask[rank] & lanes_below(lane))] = p;
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < total; i += 256u) copy_particle<T, DIM>(src, dst, order[i], start + i, ids);
        __syncthreads();
    }
}

template <typename T, int DIM>
void launch_bin_gather(const Parts<T> &src, const Parts<T> &dst, const BinLists &nxt, const BinLists &other,
                       const TileTables &tab, const BinScratch &sc, int64_t max_records, hipStream_t st) {
    // The placement finishes the layout of a small scene (its blocks wait for the
    // scan: 37k particles 3.4 us and a finalize pass of 4.6 -> 5.8); a large one, and
    // one without particles, has the pass.
    const bool finish = src.n > 0 && src.n < ((int64_t)1 << 18);
    if (!finish) launch_bin_finalize(nxt, other, max_records, st);
    if (src.n == 0) return;
    Parts<T> s2 = src, d2 = dst;
    if (!src.id || !dst.id) s2.id = d2.id = nullptr;
    const dim3 blocks((unsigned)((src.n + 255) / 256));
    if (finish)
        hipLaunchKernelGGL(k_bin_place<true>, blocks, dim3(256), 0, st, src.n, nxt, other, tab, sc);
    else
        hipLaunchKernelGGL(k_bin_place<false>, blocks, dim3(256), 0, st, src.n, nxt, other, tab, sc);
    hipLaunchKernelGGL((k_bin_gather<T, DIM>), dim3(blocks_for(max_records + (src.n + 255) / 256, 1, 8192)), dim3(256),
                       0, st, s2, d2, nxt, tab, sc);
}

// --- instantiations ---------------------------------------------------------------------
template void launch_bin_records<2>(const GridDims &, const BinLists &, const TileTables &, const BinScratch &,
                                    int64_t, bool, hipStream_t);
template void launch_bin_records<3>(const GridDims &, const BinLists &, const TileTables &, const BinScratch &,
                                    int64_t, bool, hipStream_t);

#define APIC_BIN_INST(T, DIM)                                                                                    \
    template void launch_bin_records_batch<T, DIM>(const SceneDesc<T> *, const int32_t *, int, int,                   \
                                                   const BatchQueue &, int,                                           \
                                                   hipStream_t);                                                  \
    template void launch_copy_back_batch<T, DIM>(const SceneDesc<T> *, const int32_t *, int, int, int,            \
                                                 hipStream_t);                                                    \
    template void launch_bin_gather<T, DIM>(const Parts<T> &, const Parts<T> &, const BinLists &, const BinLists &,                 \
                                            const TileTables &, const BinScratch &, int64_t, hipStream_t);        \
    template void launch_bin_keys_static<T, DIM, 1, false>(const Parts<T> &, const Parts<T> *, const GridDims &, const BinLists &,  \
                                                           const BinScratch &, uint32_t *, T, hipStream_t);      \
    template void launch_bin_keys_static<T, DIM, 2, false>(const Parts<T> &, const Parts<T> *, const GridDims &, const BinLists &,  \
                                                           const BinScratch &, uint32_t *, T, hipStream_t);      \
    template void launch_bin_keys_static<T, DIM, 3, false>(const Parts<T> &, const Parts<T> *, const GridDims &, const BinLists &,  \
                                                           const BinScratch &, uint32_t *, T, hipStream_t);
APIC_BIN_INST(float, 2)
APIC_BIN_INST(float, 3)
APIC_BIN_INST(double, 2)
APIC_BIN_INST(double, 3)
template void launch_bin_keys_static<float, 2, 2, true>(const Parts<float> &, const Parts<float> *, const GridDims &, const BinLists &,
                                                        const BinScratch &, uint32_t *, float, hipStream_t);
template void launch_bin_keys_static<float, 2, 3, true>(const Parts<float> &, const Parts<float> *, const GridDims &, const BinLists &,
                                                        const BinScratch &, uint32_t *, float, hipStream_t);
template void launch_bin_keys_static<float, 3, 2, true>(const Parts<float> &, const Parts<float> *, const GridDims &, const BinLists &,
                                                        const BinScratch &, uint32_t *, float, hipStream_t);
template void launch_bin_keys_static<float, 3, 3, true>(const Parts<float> &, const Parts<float> *, const GridDims &, const BinLists &,
                                                        const BinScratch &, uint32_t *, float, hipStream_t);

}  // namespace apic
