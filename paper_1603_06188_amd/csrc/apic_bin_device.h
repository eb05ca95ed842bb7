// Device helpers shared by the binning passes and the kernels that read a
// binned layout.  Wave helpers must be called by all 64 lanes.
#pragma once

#include "apic_common.h"

namespace apic {

__device__ __forceinline__ uint32_t bucket_of(uint32_t tile) { return tile & (kBuckets - 1); }

// Block-wide (every thread of a 256-thread block must call): exclusive
// prefix sums of the per-bucket counts v[0..kBuckets) into the LDS table
// pre[0..kBuckets); returns the total.  Thread i owns buckets [4i, 4i + 4);
// `part` is LDS scratch of 4 words.
__device__ __forceinline__ uint32_t block_bucket_prefix(const uint32_t *v, uint32_t *pre, uint32_t *part) {
    static_assert(kBuckets == 4 * 256, "one uint4 of buckets per thread");
    const int tid = (int)threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint4 q = ((const uint4 *)v)[tid];
    const uint32_t own = q.x + q.y + q.z + q.w;
    uint32_t inc = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    if (lane == 63) part[w] = inc;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) before += k < w ? part[k] : 0u;
    const uint32_t total = part[0] + part[1] + part[2] + part[3];
    const uint32_t e = before + inc - own;
    pre[4 * tid + 0] = e;
    pre[4 * tid + 1] = e + q.x;
    pre[4 * tid + 2] = e + q.x + q.y;
    pre[4 * tid + 3] = e + q.x + q.y + q.z;
    __syncthreads();
    return total;
}

// The same for three tables at once (their loads, scans and barriers shared).
__device__ __forceinline__ void block_bucket_prefix3(const uint32_t *a, const uint32_t *b, const uint32_t *c,
                                                     uint32_t *pa, uint32_t *pb, uint32_t *pc, uint32_t *part,
                                                     uint32_t &ta, uint32_t &tb, uint32_t &tc) {
    const int tid = (int)threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint32_t *v[3] = {a, b, c};
    uint32_t *pre[3] = {pa, pb, pc};
    uint4 q[3];
    uint32_t own[3], inc[3], total[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        q[k] = ((const uint4 *)v[k])[tid];
        own[k] = inc[k] = q[k].x + q[k].y + q[k].z + q[k].w;
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint32_t y = __shfl_up(inc[k], o, 64);
            if (lane >= o) inc[k] += y;
        }
    if (lane == 63) {
#pragma unroll
        for (int k = 0; k < 3; ++k) part[4 * k + w] = inc[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        uint32_t before = 0;
        total[k] = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t p = part[4 * k + i];
            before += i < w ? p : 0u;
            total[k] += p;
        }
        const uint32_t e = before + inc[k] - own[k];
        pre[k][4 * tid + 0] = e;
        pre[k][4 * tid + 1] = e + q[k].x;
        pre[k][4 * tid + 2] = e + q[k].x + q[k].y;
        pre[k][4 * tid + 3] = e + q[k].x + q[k].y + q[k].z;
    }
    __syncthreads();
    ta = total[0];
    tb = total[1];
    tc = total[2];
}

// Bucket of list index r (r below the table's total): the last bucket whose
// exclusive prefix is <= r (it holds r).  Wave-wide, r wave-uniform.
__device__ __forceinline__ uint32_t bucket_find(const uint32_t *pre, uint32_t r) {
    const int lane = lane_id();
    const int grp = popc64(ballot(pre[16 * lane] <= r)) - 1;
    const uint64_t m = ballot(lane < 16 && pre[16 * grp + lane] <= r);
    return (uint32_t)(16 * grp + popc64(m) - 1);
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t y = __shfl_xor(x, o, 64);
        x = x > y ? x : y;
    }
    return x;
}

// The maximum over the wavefront, on its last lane (row shifts and row
// broadcasts in registers; lanes without a source read 0).
__device__ __forceinline__ uint32_t wave_max_last(uint32_t x) {
#define APIC_DPP_MAX(ctrl, rows)                                                                          \
    {                                                                                                     \
        const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, rows, 0xf, true);       \
        x = x > y ? x : y;                                                                                \
    }
    APIC_DPP_MAX(0x111, 0xf)  // row_shr 1, 2, 4, 8
    APIC_DPP_MAX(0x112, 0xf)
    APIC_DPP_MAX(0x114, 0xf)
    APIC_DPP_MAX(0x118, 0xf)
    APIC_DPP_MAX(0x142, 0xa)  // lane 15 of rows 0 and 2 to rows 1 and 3
    APIC_DPP_MAX(0x143, 0xc)  // lane 31 to rows 2 and 3
#undef APIC_DPP_MAX
    return x;
}

// True for exactly one lane among the active lanes holding each value of t.
__device__ __forceinline__ bool first_lane_of_value(uint32_t t, bool active) {
    const int lane = lane_id();
    uint64_t pending = ballot(active);
    bool leader = false;
    while (pending) {
        const int first = __ffsll((unsigned long long)pending) - 1;
        const uint32_t tf = __shfl(t, first, 64);
        pending &= ~ballot(active && t == tf);
        leader = leader || lane == first;
    }
    return leader;
}

// Base of the bucket of `key` from a block table of bucket bases.
__device__ __forceinline__ uint32_t bucket_base_of(uint32_t key, const uint32_t *bases) {
    return key == kDeadKey ? 0u : bases[bucket_of(key >> 6)];
}

// Position of particle (key, rank) in the layout described by `tab`, given
// the base of the key's bucket and the live total (dead particles follow it).
__device__ __forceinline__ uint32_t bin_destination(uint32_t key, uint32_t rank, const TileTables &tab,
                                                    uint32_t base, uint32_t live_total) {
    if (key == kDeadKey) return live_total + rank;
    const uint32_t t = key >> 6, l = key & 63;
    const uint32_t start = base + tab.off[t];
    if (tab.maxc[t] <= (uint32_t)kMaxLevels) {
        const uint64_t mask = tab.lvl_mask[(int64_t)t * kMaxLevels + rank];
        return start + tab.lvl_off[(int64_t)t * kMaxLevels + rank] + (uint32_t)popc64(mask & lanes_below((int)l));
    }
    return start + tab.kprefix[(int64_t)t * 64 + l] + rank;
}

// Appends tile t to its bucket's list of `nxt`.
__device__ __forceinline__ void append_tile(uint32_t t, const BinLists &nxt) {
    const uint32_t b = bucket_of(t);
    const uint32_t j = atomicAdd(nxt.rec_count + b, 1u);
    nxt.rec_list[(int64_t)b * nxt.rcap + j] = t;
}

// Lists tile t in `nxt` unless already listed in this generation.
__device__ __forceinline__ void list_tile(uint32_t t, const BinLists &nxt) {
    if (nxt.tile_gen[t] != nxt.gen && atomicExch(nxt.tile_gen + t, nxt.gen) != nxt.gen) append_tile(t, nxt);
}

// Index of the jj-th particle of a lane's key within a listed tile: level-
// major (start + offset of level jj + rank among the keys present in it,
// given the running level offset and the level's key mask), or key-major
// (kstart + jj) for tiles whose busiest key holds more than kMaxLevels.
__device__ __forceinline__ int64_t particle_at(uint32_t start, uint32_t kstart, uint32_t level, uint64_t mask,
                                               uint32_t jj, uint32_t maxc, int lane) {
    return maxc > (uint32_t)kMaxLevels ? (int64_t)kstart + jj
                                       : (int64_t)start + level + (uint32_t)popc64(mask & lanes_below(lane));
}

// Listed tiles of a finished layout, enumerated as records r = 0, 1, ... in
// bucket order, with the bases of its particle buckets (prefix tables written
// once per layout by the finalize pass).
struct TileWalk {
    const uint32_t *rpre, *bbase;  // [kBuckets] record prefix, particle base per bucket
    uint32_t nrec, live;           // records, live particles
};

__device__ __forceinline__ TileWalk tile_walk(const BinLists &lists) {
    TileWalk w;
    w.rpre = lists.rpre;
    w.bbase = lists.bpre;
    w.nrec = lists.rpre[kBuckets];
    w.live = lists.bpre[kBuckets];
    return w;
}

// Record r of the walk: tile id, first particle and particle count.
__device__ __forceinline__ uint32_t tile_range(const TileWalk &w, uint32_t r, const BinLists &lists,
                                               const TileTables &tab, uint32_t &start, uint32_t &total) {
    const uint32_t t = lists.rec_tile[r];
    start = w.bbase[bucket_of(t)] + tab.off[t];
    total = tab.tcount[t];
    return t;
}

// Record r of the walk: tile id, first particle, this lane's key count,
// busiest key count and (busy tiles) first particle of this lane's key.
__device__ __forceinline__ uint32_t tile_of_record(const TileWalk &w, uint32_t r, const BinLists &lists,
                                                   const TileTables &tab, uint32_t &start, uint32_t &cnt,
                                                   uint32_t &maxc, uint32_t &kstart) {
    const int lane = lane_id();
    const uint32_t t = lists.rec_tile[r];
    start = w.bbase[bucket_of(t)] + tab.off[t];
    cnt = tab.kcount[(int64_t)t * 64 + lane];
    maxc = tab.maxc[t];
    kstart = maxc > (uint32_t)kMaxLevels ? start + tab.kprefix[(int64_t)t * 64 + lane] : 0u;
    return t;
}

// Lists the key's tile in `nxt` on first touch (generation tag + bucketed
// append), takes a provisional rank within the key and pushes the mover (old
// position p, order value ord) on the key's list for its final rank; dead
// particles take a rank in the dead region.  `active` false for lanes
// without a particle.  Wave-wide.
__device__ __forceinline__ uint32_t bin_take_slot(uint32_t key, bool active, uint32_t p, uint64_t ord,
                                                  const BinLists &nxt, const BinScratch &sc) {
    const bool live = active && key != kDeadKey;
    const uint32_t t = key >> 6;
    // the rank and list atomics are issued before the tile listing, whose
    // probe and claim depend on each other, so their round trips overlap
    uint32_t rank = 0u;
    if (active) {
        if (key == kDeadKey) {
            rank = atomicAdd(nxt.ctr + kCtrDead, 1u);
        } else {
            sc.pord[p] = ord;
            const uint32_t nx = atomicExch(sc.head + key, p + 1u);
            rank = atomicAdd(sc.key_count + key, 1u);
            sc.next[p] = nx;
        }
    }
    if (first_lane_of_value(t, live)) list_tile(t, nxt);
    return rank;
}

// Final ranks of the n movers on a key's list (h: first old position + 1): each
// mover's rank is the number of movers on the list with a smaller order value.  The
// list is a chain of loads, walked once for each mover; FIRST: once only where its
// first FIRST are all of it (2D, where a key has longer faces: records pass of
// 1.19M particles 14.8 -> 11.0 us with 8, 14.5 with 4; in 3D, where most lists hold
// one or two, no gain, and 512 bodies 97 -> 102).
template <int FIRST>
__device__ __forceinline__ void rank_movers(uint32_t h, uint32_t n, const BinScratch &sc) {
    if (n == 1u) {
        sc.prank[h - 1] = 0u;
        return;
    }
    if constexpr (FIRST > 0) {
        uint32_t at[FIRST], rest = h;
        uint64_t ord[FIRST];
#pragma unroll
        for (int i = 0; i < FIRST; ++i) {
            at[i] = rest;
            ord[i] = ~0ull;
            if (rest) {
                ord[i] = sc.pord[rest - 1];
                rest = sc.next[rest - 1];
            }
        }
        if (!rest) {
#pragma unroll
            for (int i = 0; i < FIRST; ++i) {
                uint32_t r = 0u;
#pragma unroll
                for (int j = 0; j < FIRST; ++j) r += ord[j] < ord[i] ? 1u : 0u;
                if (at[i]) sc.prank[at[i] - 1] = r;
            }
            return;
        }
    }
    for (uint32_t a = h; a; a = sc.next[a - 1]) {
        const uint64_t oa = sc.pord[a - 1];
        uint32_t r = 0u;
        for (uint32_t b = h; b; b = sc.next[b - 1]) r += sc.pord[b - 1] < oa ? 1u : 0u;
        sc.prank[a - 1] = r;
    }
}

// A particle's values of all planes: loaded all at once, then stored (a load
// after a store to another plane could not be moved above it, so every plane
// would be a round trip of its own).
template <typename T, int DIM>
struct ParticleState {
    uint32_t cell;
    int32_t id;
    T m, off[DIM], v[DIM], B[DIM * DIM], F[DIM * DIM];
};
template <typename T, int DIM>
__device__ __forceinline__ void load_particle(const Parts<T> &src, uint32_t p, bool ids, ParticleState<T, DIM> &x) {
    x.id = ids ? *scalar_plane(src.id, p * 4u) : 0;
    const int64_t step = plane_step<T>(src.s);
    const uint32_t pb = lane_offset(p * (uint32_t)sizeof(T));
    x.cell = *scalar_plane(src.cell, sizeof(T) == 4 ? pb : p * 4u);
    x.m = *scalar_plane(src.m, pb);
    PlaneRun<T> off(src.off, step), v(src.v, step), B(src.B, step), F(src.F, step);
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        x.off[a] = *off.next(pb);
        x.v[a] = *v.next(pb);
    }
#pragma unroll
    for (int k = 0; k < DIM * DIM; ++k) {
        x.B[k] = *B.next(pb);
        x.F[k] = *F.next(pb);
    }
}
template <typename T, int DIM>
__device__ __forceinline__ void store_particle(const Parts<T> &dst, uint32_t q, bool ids,
                                               const ParticleState<T, DIM> &x) {
    if (ids) *scalar_plane(dst.id, q * 4u) = x.id;
    const int64_t step = plane_step<T>(dst.s);
    const uint32_t qb = lane_offset(q * (uint32_t)sizeof(T));
    *scalar_plane(dst.cell, sizeof(T) == 4 ? qb : q * 4u) = x.cell;
    *scalar_plane(dst.m, qb) = x.m;
    PlaneRun<T> off(dst.off, step), v(dst.v, step), B(dst.B, step), F(dst.F, step);
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        *off.next(qb) = x.off[a];
        *v.next(qb) = x.v[a];
    }
#pragma unroll
    for (int k = 0; k < DIM * DIM; ++k) {
        *B.next(qb) = x.B[k];
        *F.next(qb) = x.F[k];
    }
}
template <typename T, int DIM>
__device__ __forceinline__ void copy_particle(const Parts<T> &src, const Parts<T> &dst, uint32_t p, uint32_t q,
                                              bool ids) {
    ParticleState<T, DIM> x;
    load_particle<T, DIM>(src, p, ids, x);
    store_particle<T, DIM>(dst, q, ids, x);
}

// Prefix tables of a layout whose records are counted: per bucket its first record
// number, first full tile and first particle (bpre, [kBuckets + 1]), found by each
// block that asks.
struct BucketTables {
    uint32_t rpre[kBuckets + 1], fpre[kBuckets + 1], part[12];
    uint32_t nfull;
};
__device__ __forceinline__ void bucket_tables(const BinLists &nxt, BucketTables &tb, uint32_t *bpre) {
    uint32_t nrec, nfull, live;
    block_bucket_prefix3(nxt.rec_count, nxt.nfull, nxt.tot, tb.rpre, tb.fpre, bpre, tb.part, nrec, nfull, live);
    if (threadIdx.x == 0) {
        tb.rpre[kBuckets] = nrec;
        bpre[kBuckets] = live;
        tb.nfull = nfull;
    }
    __syncthreads();
}

// Last bucket whose exclusive prefix is <= i (pre[kBuckets] = total > i).
__device__ __forceinline__ uint32_t bucket_search(const uint32_t *pre, uint32_t i) {
    uint32_t lo = 0, hi = kBuckets;
    while (hi - lo > 1u) {
        const uint32_t mid = (lo + hi) >> 1;
        if (pre[mid] <= i)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// Stores them and numbers the records (block `blk` of `nblk` its share of them):
// the tiles of at least kFullTile particles first, in bucket order and then by
// their rank in the bucket, then the others the same way, so that every tile walk
// takes the short tiles last.
// The counters of the other parity's build are not needed once the layout that
// followed it is finished: they are zeroed here, for the build after this one.
__device__ __forceinline__ void finish_layout(const BinLists &nxt, const BinLists &other, const BucketTables &tb,
                                              const uint32_t *bpre, uint32_t blk, uint32_t nblk) {
    if (blk == 0) {
        for (int i = (int)threadIdx.x; i < kBuckets; i += (int)blockDim.x) {
            other.rec_count[i] = 0u;
            other.nfull[i] = 0u;
            other.nsparse[i] = 0u;
            other.tot[i] = 0u;
        }
        for (int i = (int)threadIdx.x; i <= kBuckets; i += (int)blockDim.x) {
            nxt.rpre[i] = tb.rpre[i];
            nxt.bpre[i] = bpre[i];
        }
        if (threadIdx.x < kCtrCount) other.ctr[threadIdx.x] = 0u;
    }
    const uint32_t nrec = tb.rpre[kBuckets];
    for (uint32_t i = blk * blockDim.x + threadIdx.x; i < nrec; i += nblk * blockDim.x) {
        const uint32_t b = bucket_search(tb.rpre, i);
        const uint32_t t = nxt.rec_list[(int64_t)b * nxt.rcap + (i - tb.rpre[b])];
        const uint32_t v = nxt.slot[t];
        const uint32_t rec =
            (v & 0x80000000u) ? tb.nfull + (tb.rpre[b] - tb.fpre[b]) + (v & 0x7FFFFFFFu) : tb.fpre[b] + v;
        nxt.slot[t] = rec;
        nxt.rec_tile[rec] = t;
    }
}

// One scene's view of step k of a batched launch: its descriptor, the lists
// being read and built (with their generations) and its share of blocks.
template <typename T>
struct BatchStep {
    const SceneDesc<T> *d;
    StepParity sp;
    BinLists cur, nxt;
    uint32_t blk, nblk;
};

// Runs fn(item) for the block's work items: item blockIdx.x, or (QUEUE)
// items taken from the device counter until none is left.  The taken item
// passes through LDS behind block barriers, so every thread of the block
// takes part.  (Two kernels rather than one with a run-time test: the loop
// keeps more registers live than the one-item body needs.)
template <bool QUEUE, typename Fn>
__device__ __forceinline__ void batch_items(const BatchQueue &q, Fn &&fn) {
    if constexpr (!QUEUE) {
        fn((uint32_t)blockIdx.x);
    } else {
        __shared__ uint32_t item;
        for (;;) {
            __syncthreads();
            if (threadIdx.x == 0) item = atomicAdd(q.ctr, 1u) - q.base;
            __syncthreads();
            const uint32_t it = (uint32_t)__builtin_amdgcn_readfirstlane((int)item);
            if (it >= q.items) break;
            fn(it);
        }
    }
}

template <typename T>
__device__ __forceinline__ BatchStep<T> batch_step(const SceneDesc<T> *descs, const int32_t *start, int n, int k,
                                                   uint32_t item) {
    BatchStep<T> b;
    // the scene is the same for the whole block: held in scalar registers, and
    // with it every pointer of its table entry
    const int s = __builtin_amdgcn_readfirstlane(scene_of_block(start, n, item));
    b.d = descs + s;
    const uint32_t gen0[2] = {table_struct(b.d->lists[0].gen), table_struct(b.d->lists[1].gen)};
    b.sp = scalar_struct(step_parity(table_struct(b.d->cur0), table_struct(b.d->where0), gen0, k));
    b.cur = table_struct(b.d->lists[b.sp.cur]);
    b.cur.gen = b.sp.gen_cur;
    b.nxt = table_struct(b.d->lists[b.sp.nxt]);
    b.nxt.gen = b.sp.gen_nxt;
    const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane(start[s]);
    b.blk = item - first;
    b.nblk = (uint32_t)__builtin_amdgcn_readfirstlane(start[s + 1]) - first;
    return b;
}

// Key (base node) of a particle at cell `ci`, offset `off`, or kDeadKey when
// its support leaves the grid or the offset is not finite.
template <typename T, int DIM, int DEG>
__device__ __forceinline__ uint32_t key_of(const int *ci, const T *off, const GridDims &d, bool &finite) {
    int base[3] = {0, 0, 0};
    bool inside = true;
    finite = true;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        finite = finite && is_finite(off[a]);
        base[a] = base_of<T, DEG>(ci[a], off[a]);
        inside = inside && base[a] >= 0 && base[a] + DEG <= d.n[a];
    }
    return (finite && inside) ? (uint32_t)node_index<DIM>(base, d.TN) : kDeadKey;
}

}  // namespace apic
