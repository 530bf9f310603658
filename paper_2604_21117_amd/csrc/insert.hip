// Insert batches: sort, deduplicate, locate, plan, check, apply.  Delete
// batches (the last section of this file) share the sort, deduplication
// and locate, then remove keys in place and merge what fell below half full.
//
// The paper searches a static tree (Section V-A); inserts are the dynamic
// counterpart that keeps Section III's invariants: sorted leaves, equal
// leaf depth, every non-root node at least half full.  The batch behaves
// like inserting its pairs one at a time in batch order: a present key is
// overwritten, and the last occurrence of a key in the batch supplies its
// value.
//
//  1. Sort (key, batch index) stably; run heads are the distinct keys; the
//     last element of each run holds the final value.  Every non-head is
//     UPDATED.
//  2. Locate: each distinct key descends the tree (the lookup traversal of
//     traverse.h) recording the inner node and child slot per level; a key
//     found in its leaf is an update, the others are new.
//  3. Plan, read-only, level by level from the leaves up.  Touched leaves
//     are the runs of new keys with the same leaf; a leaf with c old and r
//     new keys gets t = c + r entries and splits into ceil(t/16) pieces when
//     t > 16 (even sizes, so every piece holds >= 8).  Touched parents are
//     the runs of touched children with the same parent; a parent whose
//     children split gains sum(k-1) entries and splits the same way.  Piece
//     counts are scanned into allocation offsets, so new node ids follow key
//     order and repeated runs give the same tree.
//  4. Check: if the node pools cannot hold every new node the device error
//     word gets the capacity bit and nothing below runs (the batch is
//     applied whole or not at all).
//  5. Apply: updates in place; one wave per touched leaf merges its old keys
//     (held in registers) with its new keys and writes the pieces, the first
//     in place, the others to new leaves linked into the chain; then one wave
//     per changed parent, level by level, rebuilds its entry list (old
//     entries shifted, split children replaced by their pieces and piece
//     separators) and writes its own pieces.  A root that splits grows new
//     levels above it, packed with the same even rule.
//  6. Commit the header (key count, pool cursors, height, root) and refresh
//     the top-levels mirror.
#include <atomic>

#include "insert.h"
#include "lanes.h"
#include "mirror.h"
#include "prims.h"
#include "traverse.h"

namespace gt {

constexpr int kBlk = 256;
constexpr uint32_t kSmallInsert = 2048;  // keys of the small path (below)

struct InsState {
    uint32_t U, R;
    uint32_t ok;
    uint32_t height;       // tree height when the batch started
    uint32_t overflow;     // item pool would overflow (internal error)
    uint32_t grow_nodes, grow_levels, new_root;
    uint32_t mirror_dirty;
    uint32_t lvl_count[kMaxLevels];  // items per level (0 = leaves)
    uint32_t lvl_base[kMaxLevels];   // first item of the level in the pool
    uint32_t lvl_new[kMaxLevels];    // new nodes the level's items create
    uint32_t lvl_alloc[kMaxLevels];  // first new id of the level
    uint32_t lvl_psep[kMaxLevels];   // first piece separator of the level
    uint32_t deleted;      // delete batch: keys removed
    uint32_t rebuild;      // delete batch: a parent would fall below half full
    uint32_t merges;       // delete batch: leaf runs left below half full (listed in f1)
    uint32_t gmerges;      // delete batch: parents that would fall below half full (listed in upos)
    uint32_t pad[3];
};

template <class K>
struct Ins {
    InsState* st;
    K* sk; K* sk2; uint32_t* si; uint32_t* si2; void* sort_tmp;
    uint32_t* f0; uint32_t* f1;
    K* uk; K* uv; uint32_t* upos; uint32_t* uleaf; uint8_t* uslot; uint8_t* ufound;
    uint32_t* pn; uint8_t* pi; uint8_t* pc;  // per level: node, child slot taken, node's children
    uint8_t* ulc;                             // per distinct key: its leaf's key count
    K* nk; K* nv; uint32_t* nleaf; uint32_t* nu;
    uint32_t* it_node; uint32_t* it_first; uint32_t* it_end;
    uint32_t* it_cold; uint32_t* it_k; uint32_t* it_off;
    uint8_t* it_cs;  // slot of the item's node in its parent
    K* psep;
    K* gsep0; K* gsep1; uint32_t* gid0; uint32_t* gid1;
    uint64_t Bm, ip_cap, ps_cap;
};

// ------------------------------------------------------------ scratch sizing

static uint64_t al(uint64_t x) { return (x + 255) / 256 * 256; }

static uint64_t item_pool_cap(uint64_t Bm, uint64_t leaf_cap) {
    uint64_t total = 0, lv = leaf_cap;
    for (int d = 0; d < kMaxLevels; ++d) {
        uint64_t bound = lv + 2;
        total += bound < Bm ? bound : Bm;
        lv = lv / 8;
    }
    return total;
}

static uint64_t psep_cap(uint64_t leaf_cap, uint64_t inner_cap) { return leaf_cap + inner_cap + 64; }

// items level d can hold (the item pool's per-level bound)
static uint64_t level_items_bound(uint64_t Bm, uint64_t leaf_cap, int d) {
    uint64_t lv = leaf_cap;
    for (int i = 0; i < d; ++i) lv /= 8;
    return lv + 2 < Bm ? lv + 2 : Bm;
}

template <class K>
static uint64_t carve(Ins<K>* v, uint8_t* base, uint64_t Bm, uint64_t leaf_cap, uint64_t inner_cap) {
    uint64_t off = 0;
    auto take = [&](uint64_t bytes) {
        uint8_t* p = base ? base + off : nullptr;
        off += al(bytes);
        return p;
    };
    const uint64_t ip = item_pool_cap(Bm, leaf_cap), ps = psep_cap(leaf_cap, inner_cap);
    Ins<K> x;
    x.Bm = Bm; x.ip_cap = ip; x.ps_cap = ps;
    x.st = reinterpret_cast<InsState*>(take(sizeof(InsState)));
    x.sk = reinterpret_cast<K*>(take(Bm * sizeof(K)));
    x.sk2 = reinterpret_cast<K*>(take(Bm * sizeof(K)));
    x.si = reinterpret_cast<uint32_t*>(take(Bm * 4));
    x.si2 = reinterpret_cast<uint32_t*>(take(Bm * 4));
    x.sort_tmp = take(sort_tmp_bytes(Bm, sizeof(K)));
    x.f0 = reinterpret_cast<uint32_t*>(take((Bm + 1) * 4));
    x.f1 = reinterpret_cast<uint32_t*>(take((Bm + 1) * 4));
    take(scan_tmp_bytes(Bm + 1));  // (unused: the sizes programs have computed stay)
    x.uk = reinterpret_cast<K*>(take(Bm * sizeof(K)));
    x.uv = reinterpret_cast<K*>(take(Bm * sizeof(K)));
    x.upos = reinterpret_cast<uint32_t*>(take(Bm * 4));
    x.uleaf = reinterpret_cast<uint32_t*>(take(Bm * 4));
    x.uslot = take(Bm);
    x.ufound = take(Bm);
    x.pn = reinterpret_cast<uint32_t*>(take(static_cast<uint64_t>(kMaxLevels) * Bm * 4));
    x.pi = take(static_cast<uint64_t>(kMaxLevels) * Bm);
    x.pc = take(static_cast<uint64_t>(kMaxLevels) * Bm);
    x.ulc = take(Bm);
    x.nk = reinterpret_cast<K*>(take(Bm * sizeof(K)));
    x.nv = reinterpret_cast<K*>(take(Bm * sizeof(K)));
    x.nleaf = reinterpret_cast<uint32_t*>(take(Bm * 4));
    x.nu = reinterpret_cast<uint32_t*>(take(Bm * 4));
    x.it_node = reinterpret_cast<uint32_t*>(take(ip * 4));
    take(ip * 4);  // (unused, as above)
    x.it_first = reinterpret_cast<uint32_t*>(take(ip * 4));
    x.it_end = reinterpret_cast<uint32_t*>(take(ip * 4));
    x.it_cold = reinterpret_cast<uint32_t*>(take(ip * 4));
    x.it_k = reinterpret_cast<uint32_t*>(take(ip * 4));
    x.it_off = reinterpret_cast<uint32_t*>(take(ip * 4));
    x.it_cs = take(ip);
    x.psep = reinterpret_cast<K*>(take(ps * sizeof(K)));
    x.gsep0 = reinterpret_cast<K*>(take(ps * sizeof(K)));
    x.gsep1 = reinterpret_cast<K*>(take(ps * sizeof(K)));
    x.gid0 = reinterpret_cast<uint32_t*>(take(ps * 4));
    x.gid1 = reinterpret_cast<uint32_t*>(take(ps * 4));
    if (v) *v = x;
    return off;
}

uint64_t insert_scratch_bytes(uint64_t max_batch, int key_bytes, uint64_t leaf_cap, uint64_t inner_cap) {
    if (key_bytes == 8) return carve<uint64_t>(nullptr, nullptr, max_batch, leaf_cap, inner_cap);
    return carve<uint32_t>(nullptr, nullptr, max_batch, leaf_cap, inner_cap);
}

// ------------------------------------------------------------------ kernels

__device__ __forceinline__ uint64_t gtid() { return blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; }
__device__ __forceinline__ uint64_t gstride() { return static_cast<uint64_t>(gridDim.x) * blockDim.x; }

// ------------------------------------- chunks of a batch (above 2048 keys)
//
// The plan of a large batch is a row of counts and prefix sums: distinct keys,
// new keys, the items of every level, the pieces of a level's items.  Each is
// a pair of launches over the same chunks, contiguous runs of tiles of
// kChTile entries, one workgroup each: the first leaves the chunk's total (in
// `sums`), the second adds up the totals before it, scans its tiles and writes
// what the prefix is for.  (Flags, a three-kernel scan and a kernel that used
// it, per count and level, were some 70 launches of 2 to 7 us, 300 us of an
// insert of 2^20 keys; these are 13 and take 100.)
constexpr int kChBlock = 512;
constexpr uint32_t kChItems = 4;                         // entries of a tile a thread takes, kChBlock apart
constexpr uint32_t kChTile = kChBlock * kChItems;        // 2048
constexpr uint32_t kChMax = 1024;                        // chunks at most

struct Chunks {
    uint32_t n, tiles;  // chunks, tiles of each
};

static Chunks chunks_for(uint64_t n) {
    const uint64_t all = n ? (n + kChTile - 1) / kChTile : 1;
    Chunks c;
    c.n = static_cast<uint32_t>(all < kChMax ? all : kChMax);
    c.tiles = static_cast<uint32_t>((all + c.n - 1) / c.n);
    return c;
}

// Total of x over the workgroup, in every thread.
__device__ __forceinline__ uint32_t chunk_total(uint32_t x, uint32_t* sh) {
    uint32_t all;
    block_excl_scan<uint32_t>(x, sh, &all);
    return all;
}

// The chunk totals before this chunk, and of all.
__device__ __forceinline__ uint32_t chunk_before(const uint32_t* __restrict__ sums, uint32_t* sh, uint32_t* all) {
    uint32_t pre = 0, tot = 0;
    for (uint32_t i = threadIdx.x; i < gridDim.x; i += kChBlock) {
        const uint32_t x = sums[i];
        tot += x;
        pre += i < blockIdx.x ? x : 0u;
    }
    *all = chunk_total(tot, sh);
    return chunk_total(pre, sh);
}

// Ranks within a tile: entry j * kChBlock + t is thread t's j-th, on[j] says
// whether it counts.  rank[j]: the counted entries before it (entries kChBlock
// apart, so that a wave reads and writes neighbours); returns how many count.
// `cnt` holds a count per wave and j; two barriers.
constexpr uint32_t kChWaves = kChBlock / 64;

__device__ __forceinline__ uint32_t ch_rank(const bool (&on)[kChItems], uint32_t (&rank)[kChItems],
                                            uint32_t (&cnt)[kChItems * kChWaves + 1]) {
    const uint32_t w = threadIdx.x / 64, lane = threadIdx.x & 63;
    uint64_t m[kChItems];
#pragma unroll
    for (uint32_t j = 0; j < kChItems; ++j) {
        m[j] = __ballot(on[j]);
        if (lane == 0) cnt[j * kChWaves + w] = static_cast<uint32_t>(__popcll(m[j]));
    }
    __syncthreads();
    if (w == 0) {
        const uint32_t x = lane < kChItems * kChWaves ? cnt[lane] : 0u, inc = wave_incl_scan(x);
        if (lane < kChItems * kChWaves) cnt[lane] = inc - x;
        if (lane == 63) cnt[kChItems * kChWaves] = inc;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < kChItems; ++j)
        rank[j] = cnt[j * kChWaves + w] + static_cast<uint32_t>(__popcll(m[j] & ((1ull << lane) - 1ull)));
    return cnt[kChItems * kChWaves];
}

// Distinct keys of the sorted batch, counted: the heads of runs.  Repeats get
// `repeat` as their status (the insert: UPDATED, an earlier occurrence exists;
// the delete: ABSENT, an earlier one deleted it).  Also clears the batch state.
template <class K>
__global__ __launch_bounds__(kChBlock) void k_ch_heads(Ins<K> v, const DevHeader* hdr, uint64_t B, uint32_t tiles,
                                                        uint8_t repeat, uint8_t* __restrict__ status,
                                                        uint32_t* __restrict__ sums) {
    __shared__ uint32_t sh[33];
    if (blockIdx.x == 0) {
        uint32_t* s = reinterpret_cast<uint32_t*>(v.st);
        for (uint32_t i = threadIdx.x; i < sizeof(InsState) / 4; i += kChBlock) s[i] = 0;
        __syncthreads();
        if (threadIdx.x == 0) v.st->height = hdr->height;
    }
    uint32_t n = 0;
    for (uint32_t x = 0; x < tiles; ++x) {
        const uint64_t p0 = (static_cast<uint64_t>(blockIdx.x) * tiles + x) * kChTile + threadIdx.x;
#pragma unroll
        for (uint32_t j = 0; j < kChItems; ++j) {
            const uint64_t p = p0 + j * kChBlock;
            if (p >= B) continue;
            if (p == 0 || v.sk[p] != v.sk[p - 1]) ++n;
            else status[v.si[p]] = repeat;
        }
    }
    n = chunk_total(n, sh);
    if (threadIdx.x == 0) sums[blockIdx.x] = n;
}

// ... and written: the key, the place of its first occurrence and (with vals)
// the value of its last.
template <class K>
__global__ __launch_bounds__(kChBlock) void k_ch_unique(Ins<K> v, uint64_t B, uint32_t tiles,
                                                         const K* __restrict__ vals,
                                                         const uint32_t* __restrict__ sums) {
    __shared__ uint32_t sh[33], cnt[kChItems * kChWaves + 1];
    uint32_t all, at = chunk_before(sums, sh, &all);
    if (blockIdx.x == 0 && threadIdx.x == 0) v.st->U = all;
    for (uint32_t x = 0; x < tiles; ++x) {
        const uint64_t p0 = (static_cast<uint64_t>(blockIdx.x) * tiles + x) * kChTile + threadIdx.x;
        K k[kChItems];
        uint32_t rank[kChItems], i[kChItems];
        bool on[kChItems], last[kChItems];
#pragma unroll
        for (uint32_t j = 0; j < kChItems; ++j) {
            const uint64_t p = p0 + j * kChBlock;
            k[j] = p < B ? v.sk[p] : K(0);
            on[j] = p < B && (p == 0 || k[j] != v.sk[p - 1]);
            last[j] = vals && p < B && (p + 1 == B || k[j] != v.sk[p + 1]);
            i[j] = last[j] ? v.si[p] : 0u;
        }
        K val[kChItems];
#pragma unroll
        for (uint32_t j = 0; j < kChItems; ++j) val[j] = last[j] ? vals[i[j]] : K(0);
        const uint32_t n = ch_rank(on, rank, cnt);
#pragma unroll
        for (uint32_t j = 0; j < kChItems; ++j) {
            const uint32_t e = at + rank[j];
            if (on[j]) {
                v.uk[e] = k[j];
                v.upos[e] = static_cast<uint32_t>(p0 + j * kChBlock);
            }
            if (last[j]) v.uv[e + (on[j] ? 1u : 0u) - 1u] = val[j];  // the run's last writer
        }
        at += n;
        __syncthreads();
    }
}

// Locate every distinct key; G lanes per key, QPG keys in flight per group,
// the top levels from LDS; NT threads per workgroup.
template <class K, int G, int QPG, int LV, int NT>
__device__ __forceinline__ void ph_locate(TreeView<K> t, Ins<K> v, uint8_t* __restrict__ status) {
    using T = Trav<K, G>;
    extern __shared__ __align__(16) uint8_t lds[];
    const uint8_t* mir = t.mirror;
    uint32_t mnodes = kMirrorMaxNodes;
    if constexpr (LV > 0) {
        mnodes = mirror_nodes_for_levels(LV);
        stage_mirror<K>(t.mirror, lds, mnodes);
        __syncthreads();
        mir = lds;
    }
    const MirrorHeader* mh = reinterpret_cast<const MirrorHeader*>(mir);
    const bool empty = mh->n_keys == 0;
    const uint64_t U = v.st->U;
    const int lane = lane_id();
    const int gl = lane % G, gbase = lane - gl;
    const uint64_t group = threadIdx.x / G;
    const uint64_t per_block = static_cast<uint64_t>(NT / G) * QPG;
    const uint64_t ntiles = (U + per_block - 1) / per_block;
    for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        K key[QPG];
        const uint64_t u0 = tile * per_block + group * QPG;
#pragma unroll
        for (int j = 0; j < QPG; ++j) key[j] = u0 + j < U ? v.uk[u0 + j] : K(0);
        // lane j of the group writes what is known of key j, so consecutive
        // lanes write consecutive keys' records: one lane's store per key and
        // array bound this kernel (2^20 sorted keys on 2^24: 108 us, now 76)
        const bool mine = gl < QPG && u0 + gl < U;
        const uint64_t u = mine ? u0 + gl : ~0ull;
        uint32_t leaf[QPG];
        descend<K, G, QPG, true>(t, mir, mnodes, LV, key, leaf, gl, gbase, v.pn, v.pi, v.Bm, u, v.pc);
        typename T::KV kv[QPG];
        const uint32_t lf = own_query<QPG>(leaf, gl);
        const uint32_t lcnt = mine ? t.lmeta[lf].x : 0u;
        const uint32_t at = mine ? v.si[v.upos[u]] : 0u;
#pragma unroll
        for (int j = 0; j < QPG; ++j) kv[j] = T::load_keys(t.lkeys + static_cast<uint64_t>(leaf[j]) * kSlots, gl);
        uint32_t slot[QPG];
#pragma unroll
        for (int j = 0; j < QPG; ++j) slot[j] = T::match_slot(kv[j], key[j], gbase);
        const uint32_t sl = own_query<QPG>(slot, gl);
        const bool found = sl < kSlots && !empty;
        if (mine) {
            v.ufound[u] = found ? 1 : 0;
            v.uleaf[u] = lf;
            v.ulc[u] = static_cast<uint8_t>(lcnt);
            v.uslot[u] = static_cast<uint8_t>(found ? sl : 0);
            v.f0[u] = found ? 0u : 1u;
            status[at] = found ? 1 : 0;
        }
    }
}

template <class K, int G, int QPG, int LV>
__global__ __launch_bounds__(kBlk) void k_locate(TreeView<K> t, Ins<K> v, uint8_t* __restrict__ status) {
    ph_locate<K, G, QPG, LV, kBlk>(t, v, status);
}

// A batch of at most kSmallInsert keys, sorted, deduplicated and located in
// one launch.  Every workgroup holds the batch in LDS and 16 lanes take one
// key: they count the keys before it in (key, index) order, each lane a
// sixteenth of the batch, and then descend with it.  A key's records go to
// its rank, repeats included, so no pass compacts the distinct keys first
// (U is the batch size here): a repeat is neither found nor new, it only
// reports what a second occurrence reports, and the first occurrence carries
// the last one's value.  1000 keys on 2^24 take 8.5 us, where the rank sort,
// the compaction in one workgroup and locate took three launches of 4.5, 3.0
// and 7.5.  The first workgroup clears the batch state.
template <class K, int LV, bool INS>
__global__ __launch_bounds__(kBlk) void k_rank_locate(TreeView<K> t, Ins<K> v, const K* __restrict__ keys,
                                                       const K* __restrict__ vals, uint32_t B,
                                                       uint8_t* __restrict__ status) {
    constexpr int G = 16;
    using T = Trav<K, G>;
    extern __shared__ __align__(16) uint8_t lds[];
    __shared__ K s_key[kSmallInsert];
    if (blockIdx.x == 0) {
        uint32_t* st = reinterpret_cast<uint32_t*>(v.st);
        for (uint32_t i = threadIdx.x; i < sizeof(InsState) / 4; i += kBlk)
            st[i] = i == offsetof(InsState, U) / 4 ? B : (i == offsetof(InsState, height) / 4 ? t.hdr->height : 0u);
    }
    for (uint32_t i = threadIdx.x; i < B; i += kBlk) s_key[i] = keys[i];
    const uint8_t* mir = t.mirror;
    uint32_t mnodes = kMirrorMaxNodes;
    if constexpr (LV > 0) {
        mnodes = mirror_nodes_for_levels(LV);
        stage_mirror<K>(t.mirror, lds, mnodes);
        mir = lds;
    }
    __syncthreads();
    const int lane = lane_id();
    const int gl = lane % G, gbase = lane - gl;
    const uint32_t e = (blockIdx.x * kBlk + threadIdx.x) / G;
    const bool mine = e < B && gl == 0;
    K key[1] = {e < B ? s_key[e] : K(0)};
    // lane l takes keys l, l + 16, ...: neighbouring lanes read neighbouring
    // LDS words (no bank conflicts), eight reads in flight
    constexpr uint32_t R = 8;
    uint32_t n = 0;  // smaller keys, and in the upper half smaller or equal ones: at most kSmallInsert
    uint32_t j = static_cast<uint32_t>(gl);
    for (; j + G * (R - 1) < B; j += G * R) {
        K kj[R];
#pragma unroll
        for (uint32_t x = 0; x < R; ++x) kj[x] = s_key[j + G * x];
#pragma unroll
        for (uint32_t x = 0; x < R; ++x) {
            n += kj[x] < key[0] ? 1u : 0u;
            n += kj[x] <= key[0] ? 0x10000u : 0u;
        }
    }
    for (; j < B; j += G) n += (s_key[j] < key[0] ? 1u : 0u) + (s_key[j] <= key[0] ? 0x10000u : 0u);
#pragma unroll
    for (int m = 1; m < G; m <<= 1) n += static_cast<uint32_t>(__shfl_xor(static_cast<int>(n), m, 64));
    uint32_t same = 0, last = e;  // equal keys before, the last equal key
    const uint32_t below = n & 0xFFFFu;
    if ((n >> 16) - below > 1u) {  // the key repeats (the same for its 16 lanes)
        for (j = static_cast<uint32_t>(gl); j < B; j += G)
            if (s_key[j] == key[0]) {
                same += j < e ? 1u : 0u;
                last = j > last ? j : last;
            }
#pragma unroll
        for (int m = 1; m < G; m <<= 1) {
            same += static_cast<uint32_t>(__shfl_xor(static_cast<int>(same), m, 64));
            const uint32_t o = static_cast<uint32_t>(__shfl_xor(static_cast<int>(last), m, 64));
            last = o > last ? o : last;
        }
    }
    const uint32_t u = below + same;
    K val = K(0);
    if constexpr (INS) {
        if (mine) val = vals[last];
    }
    const bool empty = reinterpret_cast<const MirrorHeader*>(mir)->n_keys == 0;
    uint32_t leaf[1];
    descend<K, G, 1, true>(t, mir, mnodes, LV, key, leaf, gl, gbase, v.pn, v.pi, v.Bm, mine ? u : ~0ull, v.pc);
    const uint32_t lcnt = mine ? t.lmeta[leaf[0]].x : 0u;
    const typename T::KV kv = T::load_keys(t.lkeys + static_cast<uint64_t>(leaf[0]) * kSlots, gl);
    const uint32_t slot = T::match_slot(kv, key[0], gbase);
    if (mine) {
        const bool present = slot < kSlots && !empty, first = same == 0;
        v.uk[u] = key[0];
        if constexpr (INS) v.uv[u] = val;
        else v.upos[u] = n >> 16;  // the next key's place
        v.ufound[u] = present && first ? 1 : 0;
        v.uleaf[u] = leaf[0];
        v.ulc[u] = static_cast<uint8_t>(lcnt);
        v.uslot[u] = static_cast<uint8_t>(present ? slot : 0);
        v.f0[u] = first && !present ? 1u : 0u;
        // a repeat: UPDATED (an earlier occurrence exists) or ABSENT (it is gone)
        status[e] = first ? (present ? 1 : 0) : (INS ? 1 : 0);
    }
}

// Entries u < U that count: new keys (not found in their leaf), or, for the
// delete, runs that left their leaf below half full.
template <class K, bool NEW>
__device__ __forceinline__ bool ch_counts(const Ins<K>& v, uint64_t u) {
    if constexpr (NEW) return !v.ufound[u];
    else return v.nu[u] != 0;
}

template <class K, bool NEW>
__global__ __launch_bounds__(kChBlock) void k_ch_count(TreeView<K> t, Ins<K> v, uint32_t tiles,
                                                        uint32_t* __restrict__ sums) {
    __shared__ uint32_t sh[33];
    const uint64_t U = !NEW && (t.hdr->error & kErrInternal) ? 0 : v.st->U;
    uint32_t n = 0;
    for (uint32_t x = 0; x < tiles; ++x) {
        const uint64_t u0 = (static_cast<uint64_t>(blockIdx.x) * tiles + x) * kChTile + threadIdx.x;
#pragma unroll
        for (uint32_t j = 0; j < kChItems; ++j) {
            const uint64_t u = u0 + j * kChBlock;
            n += u < U && ch_counts<K, NEW>(v, u) ? 1u : 0u;
        }
    }
    n = chunk_total(n, sh);
    if (threadIdx.x == 0) sums[blockIdx.x] = n;
}

// NEW: the new keys, in key order, with their leaf.  Else the delete's merge
// list (f1), in key order.
template <class K, bool NEW>
__global__ __launch_bounds__(kChBlock) void k_ch_collect(TreeView<K> t, Ins<K> v, uint32_t tiles,
                                                          const uint32_t* __restrict__ sums) {
    __shared__ uint32_t sh[33], cnt[kChItems * kChWaves + 1];
    const uint64_t U = !NEW && (t.hdr->error & kErrInternal) ? 0 : v.st->U;
    uint32_t all, at = chunk_before(sums, sh, &all);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if constexpr (NEW) v.st->R = all;
        else v.st->merges = all;
    }
    for (uint32_t x = 0; x < tiles; ++x) {
        const uint64_t u0 = (static_cast<uint64_t>(blockIdx.x) * tiles + x) * kChTile + threadIdx.x;
        bool on[kChItems];
        uint32_t rank[kChItems];
#pragma unroll
        for (uint32_t j = 0; j < kChItems; ++j) {
            const uint64_t u = u0 + j * kChBlock;
            on[j] = u < U && ch_counts<K, NEW>(v, u);
        }
        const uint32_t n = ch_rank(on, rank, cnt);
#pragma unroll
        for (uint32_t j = 0; j < kChItems; ++j) {
            if (!on[j]) continue;
            const uint64_t u = u0 + j * kChBlock;
            const uint32_t e = at + rank[j];
            if constexpr (NEW) {
                v.nk[e] = v.uk[u];
                v.nv[e] = v.uv[u];
                v.nleaf[e] = v.uleaf[u];
                v.nu[e] = static_cast<uint32_t>(u);
            } else {
                v.f1[e] = static_cast<uint32_t>(u);
            }
        }
        at += n;
        __syncthreads();
    }
}

// Items of every level, counted: sums[chunk * kMaxLevels + level].  A run of
// new keys through one node at a level is cut wherever a run below it is not,
// so the levels at which key r starts an item, the leaves (level 0) first, are
// 0 .. its depth - 1; the depth goes to f0[r].
template <class K>
__global__ __launch_bounds__(kChBlock) void k_ch_level_count(Ins<K> v, uint32_t tiles, uint32_t* __restrict__ sums) {
    __shared__ uint32_t s_n[kMaxLevels];
    const uint64_t R = v.st->R;
    const int h = static_cast<int>(v.st->height);
    if (threadIdx.x < kMaxLevels) s_n[threadIdx.x] = 0;
    __syncthreads();
    for (uint32_t x = 0; x < tiles; ++x) {
        const uint64_t r0 = (static_cast<uint64_t>(blockIdx.x) * tiles + x) * kChTile + threadIdx.x;
        uint32_t dep[kChItems], u[kChItems], w[kChItems];
        bool on[kChItems];  // still a start at level d
#pragma unroll
        for (uint32_t j = 0; j < kChItems; ++j) {
            const uint64_t r = r0 + j * kChBlock;
            const bool in = r < R, cmp = in && r > 0;
            u[j] = cmp ? v.nu[r] : 0u;
            w[j] = cmp ? v.nu[r - 1] : 0u;
            on[j] = cmp && v.nleaf[r] != v.nleaf[r - 1];
            dep[j] = in && r == 0 ? static_cast<uint32_t>(h) : (on[j] ? 1u : 0u);
        }
        for (int d = 1; d < h; ++d) {
            const uint64_t at = static_cast<uint64_t>(h - 1 - d) * v.Bm;
            uint32_t a[kChItems], b[kChItems];
            bool any = false;
#pragma unroll
            for (uint32_t j = 0; j < kChItems; ++j) {
                any = any || on[j];
                a[j] = on[j] ? v.pn[at + u[j]] : 0u;
                b[j] = on[j] ? v.pn[at + w[j]] : 0u;
            }
            if (!__ballot(any)) break;
#pragma unroll
            for (uint32_t j = 0; j < kChItems; ++j) {
                on[j] = on[j] && a[j] != b[j];
                dep[j] += on[j] ? 1u : 0u;
            }
        }
#pragma unroll
        for (uint32_t j = 0; j < kChItems; ++j)
            if (r0 + j * kChBlock < R) v.f0[r0 + j * kChBlock] = dep[j];
        for (int d = 0; d < h; ++d) {
            uint32_t n = 0;
#pragma unroll
            for (uint32_t j = 0; j < kChItems; ++j)
                n += static_cast<uint32_t>(__popcll(__ballot(dep[j] > static_cast<uint32_t>(d))));
            if (n && (threadIdx.x & 63) == 0) atomicAdd(&s_n[d], n);
        }
    }
    __syncthreads();
    if (threadIdx.x < kMaxLevels) sums[blockIdx.x * kMaxLevels + threadIdx.x] = s_n[threadIdx.x];
}

// ... and written: per item its node, its first child item (leaves: new key),
// the node's entry count and its slot in its
// parent, all recorded by locate; the end of the item before it.  The item
// counts and pool bases of the levels go to the batch state.
template <class K>
__global__ __launch_bounds__(kChBlock) void k_ch_level_items(Ins<K> v, uint32_t tiles,
                                                              const uint32_t* __restrict__ sums) {
    __shared__ uint32_t s_at[kMaxLevels], s_all[kMaxLevels], s_base[kMaxLevels];
    __shared__ uint32_t cnt[kMaxLevels][kChItems * kChWaves];
    __shared__ uint32_t s_tot[kMaxLevels];
    const uint64_t R = v.st->R;
    const int h = static_cast<int>(v.st->height);
    // the totals before this chunk and of all, every level in one pass
    static_assert(kChBlock % kMaxLevels == 0, "a thread stays with its level");
    if (threadIdx.x < kMaxLevels) s_at[threadIdx.x] = s_all[threadIdx.x] = 0;
    __syncthreads();
    {
        uint32_t pre = 0, tot = 0;
        for (uint32_t i = threadIdx.x; i < gridDim.x * kMaxLevels; i += kChBlock) {
            const uint32_t n = sums[i];
            tot += n;
            pre += i / kMaxLevels < blockIdx.x ? n : 0u;
        }
        atomicAdd(&s_at[threadIdx.x % kMaxLevels], pre);
        atomicAdd(&s_all[threadIdx.x % kMaxLevels], tot);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t base = 0;
        for (int d = 0; d < h; ++d) {
            s_base[d] = base;
            if (blockIdx.x == 0) {
                v.st->lvl_count[d] = s_all[d];
                v.st->lvl_base[d] = base;
                // the last item of a level ends where the level below does
                const uint64_t e = static_cast<uint64_t>(base) + s_all[d] - 1;
                if (s_all[d] && e < v.ip_cap) v.it_end[e] = d ? s_all[d - 1] : static_cast<uint32_t>(R);
            }
            base += s_all[d];
        }
        if (blockIdx.x == 0 && base > v.ip_cap) v.st->overflow = 1;
    }
    __syncthreads();
    for (uint32_t x = 0; x < tiles; ++x) {
        const uint64_t r0 = (static_cast<uint64_t>(blockIdx.x) * tiles + x) * kChTile + threadIdx.x;
        const uint32_t w = threadIdx.x / 64, lane = threadIdx.x & 63;
        const uint64_t lt = (1ull << lane) - 1ull;
        uint32_t dep[kChItems];
#pragma unroll
        for (uint32_t j = 0; j < kChItems; ++j)
            dep[j] = r0 + j * kChBlock < R ? v.f0[r0 + j * kChBlock] : 0u;
        // the counts of every level at once (ch_rank's, a wave per level)
        for (int d = 0; d < h; ++d)
#pragma unroll
            for (uint32_t j = 0; j < kChItems; ++j) {
                const uint64_t m = __ballot(dep[j] > static_cast<uint32_t>(d));
                if (lane == 0) cnt[d][j * kChWaves + w] = static_cast<uint32_t>(__popcll(m));
            }
        __syncthreads();
        for (int d = static_cast<int>(w); d < h; d += kChWaves) {
            const uint32_t n = lane < kChItems * kChWaves ? cnt[d][lane] : 0u, inc = wave_incl_scan(n);
            if (lane < kChItems * kChWaves) cnt[d][lane] = inc - n;
            if (lane == 63) s_tot[d] = inc;
        }
        __syncthreads();
        uint32_t below[kChItems];  // the keys' items a level down
        uint32_t u[kChItems], node[kChItems], cold[kChItems], cs[kChItems];
#pragma unroll
        for (uint32_t j = 0; j < kChItems; ++j) {
            below[j] = static_cast<uint32_t>(r0 + j * kChBlock);
            u[j] = dep[j] ? v.nu[below[j]] : 0u;
        }
        for (int d = 0; d < h; ++d) {
            const uint64_t at = static_cast<uint64_t>(d ? h - 1 - d : 0) * v.Bm;
            uint32_t ix[kChItems];
            uint64_t any = 0;
#pragma unroll
            for (uint32_t j = 0; j < kChItems; ++j) {
                const bool head = dep[j] > static_cast<uint32_t>(d);
                const uint64_t m = __ballot(head);
                any |= m;
                ix[j] = s_at[d] + cnt[d][j * kChWaves + w] + static_cast<uint32_t>(__popcll(m & lt));
                node[j] = cold[j] = cs[j] = 0;
                if (head) {
                    node[j] = d ? v.pn[at + u[j]] : v.nleaf[below[j]];
                    cold[j] = d ? v.pc[at + u[j]] : v.ulc[u[j]];
                    if (h - 2 - d >= 0) cs[j] = v.pi[static_cast<uint64_t>(h - 2 - d) * v.Bm + u[j]];
                }
            }
            if (!any) break;  // no key of the wave starts an item here or above
#pragma unroll
            for (uint32_t j = 0; j < kChItems; ++j) {
                const uint64_t e = static_cast<uint64_t>(s_base[d]) + ix[j];
                if (dep[j] > static_cast<uint32_t>(d) && e < v.ip_cap) {
                    v.it_node[e] = node[j];
                    v.it_cold[e] = cold[j];
                    v.it_cs[e] = static_cast<uint8_t>(cs[j]);
                    v.it_first[e] = below[j];
                    if (ix[j] > 0) v.it_end[e - 1] = below[j];
                }
                below[j] = ix[j];
            }
        }
        __syncthreads();
        if (threadIdx.x < static_cast<uint32_t>(h)) s_at[threadIdx.x] += s_tot[threadIdx.x];
        __syncthreads();
    }
}

// Pieces of item i of level d: the entries it had and those it gains -- its
// new keys (leaves), or one per piece beyond the first of its child items, a
// difference of the child level's piece offsets.
template <class K>
__device__ __forceinline__ uint32_t item_pieces(const Ins<K>& v, int d, uint32_t i) {
    const uint32_t at = v.st->lvl_base[d] + i, first = v.it_first[at], end = v.it_end[at];
    uint64_t gain = end - first;
    if (d > 0) {
        const uint32_t bc = v.st->lvl_base[d - 1], nc = v.st->lvl_count[d - 1], all = v.st->lvl_new[d - 1];
        const uint32_t lo = v.it_off[bc + first], hi = end < nc ? v.it_off[bc + end] : all;
        gain = hi - lo;
    }
    return split_pieces(v.it_cold[at] + gain);
}

template <class K>
__global__ __launch_bounds__(kChBlock) void k_ch_pieces(Ins<K> v, int d, uint32_t tiles, uint32_t* __restrict__ sums) {
    __shared__ uint32_t sh[33];
    const uint32_t n = v.st->overflow ? 0u : v.st->lvl_count[d], base = v.st->lvl_base[d];
    uint32_t extra = 0;
    for (uint32_t x = 0; x < tiles; ++x) {
        const uint64_t i0 = (static_cast<uint64_t>(blockIdx.x) * tiles + x) * kChTile;
        if (i0 >= n) break;
#pragma unroll
        for (uint32_t j = 0; j < kChItems; ++j) {
            const uint64_t i = i0 + j * kChBlock + threadIdx.x;
            if (i >= n) continue;
            const uint32_t k = item_pieces<K>(v, d, static_cast<uint32_t>(i));
            v.it_k[base + i] = k;
            extra += k - 1;
        }
    }
    extra = chunk_total(extra, sh);
    if (threadIdx.x == 0) sums[blockIdx.x] = extra;
}

// The scan of one tile's extra pieces from `at` on into it_off.
template <class K, int NT>
__device__ __forceinline__ uint32_t piece_offsets(const Ins<K>& v, uint32_t base, uint64_t i0, uint32_t n, uint32_t at,
                                                  uint32_t* sh) {
    uint32_t f[kChItems], sum = 0;
#pragma unroll
    for (uint32_t j = 0; j < kChItems; ++j) {
        f[j] = i0 + j < n ? v.it_k[base + i0 + j] - 1u : 0u;
        sum += f[j];
    }
    uint32_t tot;
    uint32_t off = at + block_excl_scan<uint32_t>(sum, sh, &tot);
#pragma unroll
    for (uint32_t j = 0; j < kChItems; ++j)
        if (i0 + j < n) {
            v.it_off[base + i0 + j] = off;
            off += f[j];
        }
    return tot;
}

template <class K>
__global__ __launch_bounds__(kChBlock) void k_ch_offsets(Ins<K> v, int d, uint32_t tiles,
                                                          const uint32_t* __restrict__ sums) {
    __shared__ uint32_t sh[33];
    const uint32_t n = v.st->overflow ? 0u : v.st->lvl_count[d], base = v.st->lvl_base[d];
    uint32_t all, at = chunk_before(sums, sh, &all);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        v.st->lvl_new[d] = all;
        v.st->lvl_psep[d] = d ? v.st->lvl_psep[d - 1] + v.st->lvl_new[d - 1] : 0u;
    }
    for (uint32_t x = 0; x < tiles; ++x) {
        const uint64_t i0 = (static_cast<uint64_t>(blockIdx.x) * tiles + x) * kChTile;
        if (i0 >= n) break;
        at += piece_offsets<K, kChBlock>(v, base, i0 + threadIdx.x * kChItems, n, at, sh);
    }
}

// Capacity check and allocation bases (one thread).
template <class K>
__device__ __forceinline__ void ph_check(TreeView<K> t, Ins<K> v, uint64_t tid, uint64_t nth) {
    if (tid != 0) return;
    InsState* st = v.st;
    DevHeader* hdr = t.hdr;
    const int h = static_cast<int>(st->height);
    // root growth: the root is the level-(h-1) item, if touched
    uint32_t gn = 0, gl = 0;
    const int dr = h - 1;
    if (st->lvl_count[dr] > 0) {
        uint64_t cnt = v.it_k[st->lvl_base[dr]];
        while (cnt > 1) {
            const uint64_t nodes = cnt <= kSlots ? 1 : (cnt + kSlots - 1) / kSlots;
            gn += static_cast<uint32_t>(nodes);
            gl += 1;
            cnt = nodes;
        }
    }
    const uint64_t leaf_new = st->lvl_new[0];
    uint64_t inner_new = gn, sep_total = 0;
    for (int d = 0; d < h; ++d) sep_total += st->lvl_new[d];
    for (int d = 1; d < h; ++d) inner_new += st->lvl_new[d];
    bool ok = !st->overflow;
    if (hdr->error & kErrInternal) ok = false;  // e.g. the batch's device sort gave up
    if (hdr->leaf_used + leaf_new > t.leaf_cap) ok = false;
    if (hdr->inner_used + inner_new > t.inner_cap) ok = false;
    if (sep_total + 1 > v.ps_cap) ok = false;
    if (h + gl > kMaxLevels) ok = false;
    if (!ok && !(hdr->error & kErrInternal)) atomicOr(&hdr->error, st->overflow ? kErrInternal : kErrCapacity);
    st->ok = ok ? 1u : 0u;
    st->grow_nodes = gn;
    st->grow_levels = gl;
    st->lvl_alloc[0] = hdr->leaf_used;
    uint32_t cur = hdr->inner_used;
    for (int d = 1; d < h; ++d) {
        st->lvl_alloc[d] = cur;
        cur += st->lvl_new[d];
    }
    st->new_root = cur;  // first growth node id
}

template <class K>
__global__ void k_apply_updates(TreeView<K> t, Ins<K> v) {
    if (!v.st->ok) return;
    const uint64_t U = v.st->U;
    for (uint64_t u = gtid(); u < U; u += gstride())
        if (v.ufound[u]) t.lvals[static_cast<uint64_t>(v.uleaf[u]) * kSlots + v.uslot[u]] = v.uv[u];
}

// part_start and part_of for the splits the rebuilds make: below 2^16
// entries every product j * total fits in 32 bits, and a 32-bit division is
// a few instructions where a 64-bit one is a long sequence (a rebuild makes
// several per entry).  Same results; larger counts take the 64-bit forms.
__device__ __forceinline__ uint32_t pstart(uint64_t j, uint64_t total, uint64_t parts) {
    if (total < (1u << 16)) {
        return static_cast<uint32_t>(j) * static_cast<uint32_t>(total) / static_cast<uint32_t>(parts);
    }
    return static_cast<uint32_t>(part_start(j, total, parts));
}

__device__ __forceinline__ uint32_t ppart(uint64_t pos, uint64_t total, uint64_t parts) {
    if (total < (1u << 16)) {
        const uint32_t p = static_cast<uint32_t>(pos), t = static_cast<uint32_t>(total),
                       n = static_cast<uint32_t>(parts);
        uint32_t j = p * n / t;
        while (j + 1 < n && (j + 1) * t / n <= p) ++j;
        while (j > 0 && j * t / n > p) --j;
        return j;
    }
    return static_cast<uint32_t>(part_of(pos, total, parts));
}

// Lanes that rebuild one node (a leaf or an inner node): one per slot, four
// nodes per wave, so a wave keeps four nodes' reads in flight.
constexpr int kNodeLanes = 16;
static_assert(kNodeLanes == 16, "a node's lane group is one DPP row (row_lane)");

// Merge-split of the touched leaves: kNodeLanes lanes per leaf, group grp
// of ngrp.
// The planned items a rebuild reads: the arrays in device memory, or a copy
// in LDS that the one-workgroup apply makes of every level's items at its
// start (the plan wrote them all before; a rebuild only reads them), so
// that a level's rebuild waits on one round of device memory fewer.
struct ItemView {
    const uint32_t* node;
    const uint32_t* first;
    const uint32_t* end;
    const uint32_t* cold;
    const uint32_t* k;
    const uint32_t* off;
    const uint8_t* cs;
};

template <class K>
__device__ __forceinline__ ItemView items_in(const Ins<K>& v) {
    return ItemView{v.it_node, v.it_first, v.it_end, v.it_cold, v.it_k, v.it_off, v.it_cs};
}

// A leaf that does not split, so holds at most 16 entries in the end, by its
// 16 lanes: lane q holds new pair q, a ballot per new key counts the old keys
// below it, which gives its slot, and the merged lines are stored whole, each
// lane picking the pair that comes to its slot.  (2^20 keys on 2^24: the leaf
// kernel took 145 us when every leaf went the way of a split, whose moves,
// compares and piece bounds, some 480 vector instructions per four leaves,
// were its bound, and takes 104; two kernels, merges with two leaves in flight
// and splits, took 81 + 27.)
template <class K>
__device__ __forceinline__ void merge_leaf(TreeView<K> t, uint32_t leaf, K okey, K oval, uint2 meta, uint32_t c,
                                           const K* nk, const K* nv, uint32_t r, int gl, int gbase) {
    const uint32_t total = c + r;
    K mine = K(0), mval = K(0);
    if (static_cast<uint32_t>(gl) < r) {
        mine = nk[gl];
        mval = nv[gl];
    }
    const bool old = static_cast<uint32_t>(gl) < c;
    uint32_t newpos = 0;  // bit s: a new key comes to slot s
    for (uint32_t q = 0; q < r; ++q) {
        const K kq = static_cast<K>(__shfl(mine, gbase + static_cast<int>(q), 64));
        const uint32_t m = static_cast<uint32_t>(group_bits<kNodeLanes>(__ballot(old && okey < kq), gbase));
        newpos |= 1u << (q + static_cast<uint32_t>(__popc(m)));
    }
    // slot s: the new pair of rank #{new slots below s}, else the old pair of
    // rank s less that; past the count the last pair's key
    const uint32_t s = static_cast<uint32_t>(gl) < total ? static_cast<uint32_t>(gl) : total - 1u;
    const uint32_t nb = static_cast<uint32_t>(__popc(newpos & ((1u << s) - 1u)));
    const bool fresh = (newpos >> s) & 1u;
    const int src = gbase + static_cast<int>(fresh ? nb : s - nb);
    const K ko = static_cast<K>(__shfl(okey, src, 64)), kn = static_cast<K>(__shfl(mine, src, 64));
    const K vo = static_cast<K>(__shfl(oval, src, 64)), vn = static_cast<K>(__shfl(mval, src, 64));
    const uint64_t line = static_cast<uint64_t>(leaf) * kSlots + gl;
    t.lkeys[line] = fresh ? kn : ko;
    t.lvals[line] = static_cast<uint32_t>(gl) < total ? (fresh ? vn : vo) : kmax<K>();
    if (gl == 0) t.lmeta[leaf] = make_uint2(total, meta.y);
}

// first index in a[0..n) whose key is >= k
template <class K>
__device__ __forceinline__ uint32_t lower_bound_dev(const K* a, uint32_t n, K k) {
    uint32_t lo = 0, hi = n;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (a[mid] < k) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

constexpr uint32_t kLongRun = 256;

// Item `it` of the leaf level by its lane group: merge, and split where the
// leaf overflows.  LONG: a run may be longer than kLongRun keys (2^16 keys in
// one leaf 7.1 ms when every chunk counted for the old keys, 6.3 searched;
// 2048 206 us and 187).
template <class K, bool LONG>
__device__ __forceinline__ void apply_leaf(const TreeView<K>& t, const Ins<K>& v, uint64_t it, uint32_t alloc, int gl,
                                           int gbase, const ItemView& iv) {
    const uint32_t leaf = iv.node[it];
    const uint32_t first = iv.first[it];
    const uint32_t r = iv.end[it] - first;
    const uint32_t c = iv.cold[it];
    const uint32_t k = iv.k[it];
    const uint32_t off = iv.off[it];
    const uint32_t total = c + r;  // r is at most the batch size
    const uint32_t base_new = alloc + off;
    const K okey = t.lkeys[static_cast<uint64_t>(leaf) * kSlots + gl];
    const K oval = t.lvals[static_cast<uint64_t>(leaf) * kSlots + gl];
    const uint2 meta = t.lmeta[leaf];
    __threadfence_block();  // the old leaf is in registers before any write
    const K* nk = v.nk + first;
    const K* nv = v.nv + first;
    // the groups of a wave take one of the two ways on their own
    if (k == 1) {
        merge_leaf<K>(t, leaf, okey, oval, meta, c, nk, nv, r, gl, gbase);
        return;
    }
    // one run of new keys (the common case): each lane holds at most one
    // old and one new element, and the group pads the pieces together
    const bool one_run = r <= static_cast<uint32_t>(kNodeLanes);
    auto place = [&](uint32_t pos, K key, K val) {
        const uint32_t j = ppart(pos, total, k);
        const uint32_t s0 = pstart(j, total, k), s1 = pstart(j + 1, total, k);
        const uint32_t slot = pos - s0;
        const uint64_t dest = j == 0 ? leaf : base_new + j - 1;
        t.lkeys[dest * kSlots + slot] = key;
        t.lvals[dest * kSlots + slot] = val;
        if (pos + 1 == s1) {
            const uint32_t cnt = static_cast<uint32_t>(s1 - s0);
            if (!one_run) {
                for (uint32_t s = cnt; s < kSlots; ++s) {
                    t.lkeys[dest * kSlots + s] = key;
                    t.lvals[dest * kSlots + s] = kmax<K>();
                }
            }
            const uint32_t nxt = (j + 1 < k) ? static_cast<uint32_t>(base_new + j) : meta.y;
            t.lmeta[dest] = make_uint2(cnt, nxt);
            if (j + 1 < k) v.psep[off + j] = key;
        }
    };
    // new keys 16 at a time, the next ones' reads in flight: a new key goes
    // behind its smaller old keys, and an old key behind the new keys that it
    // is not below (their ranks tell, where a binary search of the run takes
    // six dependent reads and more; a run above kLongRun keys is searched)
    const bool has_old = gl < static_cast<int>(c);
    const bool long_run = LONG && r > kLongRun;
    uint64_t npos = ~0ull;
    K nkey = K(0);
    uint32_t below = 0;
    K key = static_cast<uint32_t>(gl) < r ? nk[gl] : K(0);
    K val = static_cast<uint32_t>(gl) < r ? nv[gl] : K(0);
    for (uint32_t q0 = 0; q0 < r; q0 += kNodeLanes) {
        const uint32_t q = q0 + gl, qn = q + kNodeLanes;
        const bool act = q < r;
        const K key2 = qn < r ? nk[qn] : K(0), val2 = qn < r ? nv[qn] : K(0);
        uint32_t rank = 0;
        static_for<0, kNodeLanes>([&](auto S) {
            const K ks = row_lane<decltype(S)::value>(okey);
            rank += (static_cast<uint32_t>(decltype(S)::value) < c && ks < key) ? 1u : 0u;
        });
        if (!long_run) {
            const uint32_t rk = act ? rank : kNone;
            static_for<0, kNodeLanes>(
                [&](auto S) { below += row_lane<decltype(S)::value>(rk) <= static_cast<uint32_t>(gl) ? 1u : 0u; });
        }
        if (act) {
            place(q + rank, key, val);
            npos = q + rank;
            nkey = key;
        }
        key = key2;
        val = val2;
    }
    if (long_run && has_old) below = lower_bound_dev(nk, r, okey);
    const uint64_t opos = has_old ? gl + static_cast<uint64_t>(below) : ~0ull;
    if (has_old) place(static_cast<uint32_t>(opos), okey, oval);
    if (one_run) {
        // slots past a piece's count repeat its last key with an all-ones
        // value: the piece's last element sits on one lane, as an old or
        // a new element; lanes past the count write one slot each
        for (uint32_t j = 0; j < k; ++j) {
            const uint64_t s0 = pstart(j, total, k), s1 = pstart(j + 1, total, k);
            const uint32_t cnt = static_cast<uint32_t>(s1 - s0);
            if (cnt >= static_cast<uint32_t>(kSlots)) continue;
            const uint64_t mo = group_bits<kNodeLanes>(__ballot(opos == s1 - 1), gbase);
            const uint64_t mn = group_bits<kNodeLanes>(__ballot(npos == s1 - 1), gbase);
            const K ko = __shfl(okey, gbase + (mo ? __builtin_ctzll(mo) : 0), 64);
            const K kn = __shfl(nkey, gbase + (mn ? __builtin_ctzll(mn) : 0), 64);
            const K lastk = mo ? ko : kn;
            const uint64_t dest = j == 0 ? leaf : base_new + j - 1;
            if (static_cast<uint32_t>(gl) >= cnt) {
                t.lkeys[dest * kSlots + gl] = lastk;
                t.lvals[dest * kSlots + gl] = kmax<K>();
            }
        }
    }
}

template <class K, bool LONG>
__device__ __forceinline__ void apply_leaves_body(TreeView<K> t, Ins<K> v, uint64_t grp, uint64_t ngrp,
                                                  const ItemView& iv) {
    const uint32_t ok = v.st->ok;
    const uint64_t T0 = v.st->lvl_count[0];
    if (!ok || T0 == 0) return;
    const int gl = lane_id() % kNodeLanes, gbase = lane_id() - gl;
    const uint32_t alloc = v.st->lvl_alloc[0];
    for (uint64_t it = grp; it < T0; it += ngrp) apply_leaf<K, LONG>(t, v, it, alloc, gl, gbase, iv);
}

// Rebuild the changed parents of level d: kNodeLanes lanes per parent, group
// grp of ngrp.
template <class K>
__device__ __forceinline__ void apply_inner_body(TreeView<K> t, Ins<K> v, int d, uint64_t grp, uint64_t ngrp,
                                                 const ItemView& iv) {
    const uint32_t ok = v.st->ok;
    const int h = static_cast<int>(v.st->height);
    const int l = h - 1 - d;
    // no child at level d-1 split: no parent at level d changes
    if (!ok || l < 0 || v.st->lvl_new[d - 1] == 0) return;
    const uint64_t n = v.st->lvl_count[d];
    const uint32_t bd = v.st->lvl_base[d], bc = v.st->lvl_base[d - 1];
    const uint32_t alloc = v.st->lvl_alloc[d], alloc_c = v.st->lvl_alloc[d - 1];
    const uint32_t psep_d = v.st->lvl_psep[d], psep_c = v.st->lvl_psep[d - 1];
    const bool child_leaf = d == 1;
    const int gl = lane_id() % kNodeLanes, gbase = lane_id() - gl;
    const uint32_t lane = static_cast<uint32_t>(gl);  // this lane's old slot
    for (uint64_t j = grp; j < n; j += ngrp) {
        const uint32_t node = iv.node[bd + j];
        const uint32_t first = iv.first[bd + j], end = iv.end[bd + j];
        const uint32_t C = iv.cold[bd + j];
        const uint32_t P = iv.k[bd + j];
        const uint32_t off = iv.off[bd + j];
        const K osep = t.ikeys[static_cast<uint64_t>(node) * kSlots + lane];
        const uint32_t ochild = t.ichild[static_cast<uint64_t>(node) * kSlots + lane];
        // the child items (one per changed child node, so at most kSlots),
        // one per lane: slot in this node, piece count, first new piece
        const uint32_t nci = end - first < static_cast<uint32_t>(kNodeLanes) ? end - first : kNodeLanes;
        uint32_t ccs = kNone, cks = 1, cof = 0;
        if (lane < nci) {
            ccs = iv.cs[bc + first + lane];
            cks = iv.k[bc + first + lane];
            cof = iv.off[bc + first + lane];
        }
        // per old slot: shift from split children before it, and its own
        // item (lanes past nci hold no item: slot kNone, one piece, so they
        // add nothing; the moves are row broadcasts)
        uint32_t shift = 0, myk = 1, myoff = 0;
        uint32_t a = 0;  // below 2^21: at most 16 children of at most 2^17 pieces
        static_for<0, kNodeLanes>([&](auto S) {
            constexpr int i = decltype(S)::value;
            const uint32_t cs = row_lane<i>(ccs), ki = row_lane<i>(cks), oi = row_lane<i>(cof);
            a += ki - 1;
            if (cs < lane) shift += ki - 1;
            if (cs == lane) { myk = ki; myoff = oi; }
        });
        __threadfence_block();  // the old node is in registers before any write
        if (a == 0) continue;   // no child split: the parent is unchanged
        const uint32_t newpos = lane + shift;
        const uint32_t Cp = C + a;
        const uint32_t base_new = alloc + off;
        for (uint32_t e0 = 0; e0 < Cp; e0 += kNodeLanes) {
            const uint32_t e = e0 + lane;
            const bool act = e < Cp;
            // old slot whose entries cover e: the last slot with newpos <= e
            uint32_t sf = 0;
            static_for<0, kNodeLanes>([&](auto S) {
                constexpr uint32_t s = decltype(S)::value;
                const uint32_t np = row_lane<s>(newpos);
                if (s < C && np <= e) sf = s;
            });
            const int src = gbase + static_cast<int>(sf);
            const uint32_t np = shfl_u32(newpos, src);
            const uint32_t ks = shfl_u32(myk, src);
            const uint32_t ko = shfl_u32(myoff, src);
            const K os = __shfl(osep, src, 64);
            const uint32_t oc = shfl_u32(ochild, src);
            const uint32_t jj = e - np;
            const K last_sep = (sf + 1 < C) ? os : kmax<K>();
            K sep;
            uint32_t ch;
            if (ks <= 1) {
                sep = last_sep;
                ch = oc;
            } else {
                sep = (jj + 1 < ks) ? v.psep[psep_c + ko + jj] : last_sep;
                if (jj == 0) ch = oc;
                else {
                    const uint32_t id = alloc_c + ko + jj - 1;
                    ch = child_leaf ? (kLeafTag | id) : id;
                }
            }
            if (act) {
                const uint32_t pj = ppart(e, Cp, P);
                const uint32_t s0 = pstart(pj, Cp, P), s1 = pstart(pj + 1, Cp, P);
                const uint32_t slot = e - s0;
                const uint32_t cnt = s1 - s0;
                const uint32_t dest = pj == 0 ? node : base_new + pj - 1;
                t.ikeys[static_cast<uint64_t>(dest) * kSlots + slot] = (slot + 1 < cnt) ? sep : kmax<K>();
                t.ichild[static_cast<uint64_t>(dest) * kSlots + slot] = ch;
                if (e + 1 == s1 && pj + 1 < P) v.psep[psep_d + off + pj] = sep;
            }
        }
        // slots past a piece's count: the largest key and no child, one slot
        // per lane
        for (uint32_t pj = 0; pj < P; ++pj) {
            const uint32_t cnt = pstart(pj + 1, Cp, P) - pstart(pj, Cp, P);
            const uint32_t dest = pj == 0 ? node : base_new + pj - 1;
            if (lane >= cnt) {
                t.ikeys[static_cast<uint64_t>(dest) * kSlots + lane] = kmax<K>();
                t.ichild[static_cast<uint64_t>(dest) * kSlots + lane] = kNone;
            }
        }
    }
}

template <class K>
__global__ __launch_bounds__(kBlk) void k_apply_leaves(TreeView<K> t, Ins<K> v) {
    apply_leaves_body<K, true>(t, v, gtid() / kNodeLanes, gstride() / kNodeLanes, items_in(v));
}

template <class K>
__global__ __launch_bounds__(kBlk) void k_apply_inner(TreeView<K> t, Ins<K> v, int d) {
    apply_inner_body<K>(t, v, d, gtid() / kNodeLanes, gstride() / kNodeLanes, items_in(v));
}

// Root growth: pack the root's pieces into new levels (one workgroup).
template <class K>
__device__ __forceinline__ void grow_body(TreeView<K> t, Ins<K> v) {
    if (!v.st->ok || v.st->grow_levels == 0) return;
    const int h = static_cast<int>(v.st->height);
    const int dr = h - 1;
    const uint32_t item = v.st->lvl_base[dr];
    const uint32_t k0 = v.it_k[item];
    const uint32_t off = v.it_off[item];
    const uint32_t alloc = v.st->lvl_alloc[dr];
    const uint32_t psep0 = v.st->lvl_psep[dr];
    const bool leaf = dr == 0;
    for (uint32_t e = threadIdx.x; e < k0; e += blockDim.x) {
        const uint32_t id = e == 0 ? v.it_node[item] : alloc + off + e - 1;
        v.gid0[e] = leaf ? (kLeafTag | id) : id;
        v.gsep0[e] = (e + 1 < k0) ? v.psep[psep0 + off + e] : kmax<K>();
    }
    __syncthreads();
    K* sa = v.gsep0; K* sb = v.gsep1;
    uint32_t* ia = v.gid0; uint32_t* ib = v.gid1;
    uint64_t cnt = k0;
    uint32_t cursor = v.st->new_root;
    while (cnt > 1) {
        const uint64_t nodes = cnt <= kSlots ? 1 : (cnt + kSlots - 1) / kSlots;
        for (uint64_t e = threadIdx.x; e < cnt; e += blockDim.x) {
            const uint64_t n = part_of(e, cnt, nodes);
            const uint64_t s0 = part_start(n, cnt, nodes), s1 = part_start(n + 1, cnt, nodes);
            const uint64_t slot = e - s0, c = s1 - s0;
            const uint64_t dest = cursor + n;
            t.ikeys[dest * kSlots + slot] = (slot + 1 < c) ? sa[e] : kmax<K>();
            t.ichild[dest * kSlots + slot] = ia[e];
            if (e + 1 == s1) {
                for (uint64_t s = c; s < kSlots; ++s) {
                    t.ikeys[dest * kSlots + s] = kmax<K>();
                    t.ichild[dest * kSlots + s] = kNone;
                }
                sb[n] = sa[e];  // the node's bound is its last entry's separator
                ib[n] = static_cast<uint32_t>(dest);
            }
        }
        __syncthreads();
        cursor += static_cast<uint32_t>(nodes);
        cnt = nodes;
        K* ts = sa; sa = sb; sb = ts;
        uint32_t* ti = ia; ia = ib; ib = ti;
        __syncthreads();
    }
    if (threadIdx.x == 0) v.st->new_root = cursor - 1;
}


template <class K>
__device__ __forceinline__ void ph_commit(TreeView<K> t, Ins<K> v) {
    if (!v.st->ok) return;
    InsState* st = v.st;
    DevHeader* hdr = t.hdr;
    const int h = static_cast<int>(st->height);
    uint32_t inner_new = st->grow_nodes;
    for (int d = 1; d < h; ++d) inner_new += st->lvl_new[d];
    hdr->n_keys += st->R;
    hdr->leaf_used += st->lvl_new[0];
    hdr->inner_used += inner_new;
    if (st->grow_levels) {
        hdr->height = h + st->grow_levels;
        hdr->root = st->new_root;
    }
    hdr->epoch += 1;
    // the mirror (three top inner levels, key count) needs a refresh when the
    // root grew, the tree was empty, or a node of the top three levels was
    // rewritten: parents at tree level l change when their children (item
    // level h-2-l) split
    bool dirty = st->grow_levels > 0 || hdr->n_keys == st->R;
    for (int l = 0; l < 3; ++l) {
        const int dc = h - 2 - l;
        if (dc >= 0 && st->lvl_new[dc] > 0) dirty = true;
    }
    st->mirror_dirty = dirty ? 1u : 0u;
    reinterpret_cast<MirrorHeader*>(t.mirror)->n_keys = hdr->n_keys;
}

// The upper levels of a large batch's plan, from d0 on, and the capacity check
// in one workgroup, tile after tile.  A thread takes kChItems consecutive
// items of a tile, all their reads in flight, and scans their pieces from its
// registers; it is bound by a tile's three dependent reads and its barriers.
// Above a level where nothing splits no level does, and nothing reads their
// items but the check, the root's.  65536 new keys on 2^24 take 5.9 us, 100
// with an item at a time per thread, a second pass for the offsets and every
// level walked; 4096 new keys 13.9, 23.6.
constexpr int kTailBlock = 1024;

template <class K>
__global__ __launch_bounds__(kTailBlock) void k_plan_tail(TreeView<K> t, Ins<K> v, int d0) {
    __shared__ uint32_t sh[33];
    const int h = static_cast<int>(v.st->height);
    uint32_t bc = 0, nc = 0, split = 0, psep = 0;  // the level below: first item, items, new nodes; separators so far
    if (d0 > 0) {
        bc = v.st->lvl_base[d0 - 1];
        nc = v.st->lvl_count[d0 - 1];
        split = v.st->lvl_new[d0 - 1];
        psep = v.st->lvl_psep[d0 - 1] + split;
    }
    for (int d = d0; d < h && !v.st->overflow; ++d) {
        const uint32_t n = v.st->lvl_count[d], base = v.st->lvl_base[d];
        uint32_t at = 0;
        if (d > 0 && split == 0) {
            if (threadIdx.x == 0 && d == h - 1 && n) v.it_k[base] = 1u;
        } else {
            for (uint32_t t0 = 0; t0 < n; t0 += kTailBlock * kChItems) {
                const uint32_t i0 = t0 + threadIdx.x * kChItems;
                uint32_t first[kChItems], end[kChItems], k[kChItems];
#pragma unroll
                for (uint32_t j = 0; j < kChItems; ++j) {
                    const bool in = i0 + j < n;
                    first[j] = in ? v.it_first[base + i0 + j] : 0u;
                    end[j] = in ? v.it_end[base + i0 + j] : 0u;
                    k[j] = in ? v.it_cold[base + i0 + j] : 0u;
                }
                if (d > 0) {  // an item gains a child per piece beyond the first of its child items
#pragma unroll
                    for (uint32_t j = 0; j < kChItems; ++j) {
                        const bool in = i0 + j < n;
                        first[j] = in ? v.it_off[bc + first[j]] : 0u;
                        end[j] = in ? (end[j] < nc ? v.it_off[bc + end[j]] : split) : 0u;
                    }
                }
                uint32_t sum = 0;
#pragma unroll
                for (uint32_t j = 0; j < kChItems; ++j) {
                    k[j] = i0 + j < n ? split_pieces(static_cast<uint64_t>(k[j]) + (end[j] - first[j])) : 1u;
                    sum += k[j] - 1u;
                }
                uint32_t tot;
                uint32_t off = at + block_excl_scan<uint32_t>(sum, sh, &tot);
#pragma unroll
                for (uint32_t j = 0; j < kChItems; ++j)
                    if (i0 + j < n) {
                        v.it_k[base + i0 + j] = k[j];
                        v.it_off[base + i0 + j] = off;
                        off += k[j] - 1u;
                    }
                at += tot;
            }
        }
        if (threadIdx.x == 0) {
            v.st->lvl_new[d] = at;
            v.st->lvl_psep[d] = psep;
        }
        psep += at;
        bc = base;
        nc = n;
        split = at;
        __syncthreads();
    }
    ph_check<K>(t, v, threadIdx.x, kTailBlock);
}

// The batch state from device memory into LDS or back, by threads tid of nth
// (a barrier separates the copy from reads of its destination).
__device__ __forceinline__ void copy_state(InsState* dst, const InsState* src, uint32_t tid, uint32_t nth) {
    static_assert(sizeof(InsState) % 4 == 0, "the state copies as words");
    uint32_t* d = reinterpret_cast<uint32_t*>(dst);
    const uint32_t* s = reinterpret_cast<const uint32_t*>(src);
    for (uint32_t i = tid; i < sizeof(InsState) / 4; i += nth) d[i] = s[i];
}

// Orders one wave's LDS accesses around a point (a workgroup barrier where
// the wave works alone).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Everything after the plan for a batch of at most kFusedMax keys, in one
// workgroup: every level has at most that many touched nodes, one round of
// kNodeLanes-lane groups, and barriers stand where the general path has
// kernel boundaries (leaves, each parent level, growth and commit, mirror).
constexpr int kFusedBlock = 1024;
constexpr uint32_t kFusedMax = kFusedBlock / kNodeLanes;  // 64

// every level's items of a batch of at most kFusedMax keys (at most that
// many runs per level)
constexpr uint32_t kFusedItems = kFusedMax * kMaxLevels;

// Besides the items, two things stay on the chip, so that a level waits on
// fewer rounds of device memory:
//  - the batch state (per-level counts, bases, allocation cursors): from
//    device memory each level, the growth and the commit would wait on its
//    fields one read after another;
//  - the separators a level's splits produce (read by the level above and by
//    the root growth): a level adds at most one piece per new key below it,
//    so a batch of at most kFusedMax keys makes at most kFusedItems of them.
template <class K>
__device__ __forceinline__ void ph_small_apply(TreeView<K> t, Ins<K> v0, int H) {
    __shared__ uint32_t s_node[kFusedItems], s_first[kFusedItems], s_end[kFusedItems];
    __shared__ uint32_t s_cold[kFusedItems], s_k[kFusedItems], s_off[kFusedItems];
    __shared__ uint8_t s_cs[kFusedItems];
    __shared__ K s_psep[kFusedItems];
    __shared__ InsState s_st;
    const uint64_t grp = threadIdx.x / kNodeLanes, ngrp = kFusedBlock / kNodeLanes;
    Ins<K> v = v0;
    v.psep = s_psep;
    copy_state(&s_st, v.st, threadIdx.x, blockDim.x);
    // the planned items of every level, copied once: every slot the plan
    // may have written, so that the copy need not wait for the level counts
    // (it and the state arrive in one round of reads)
    const uint32_t span = v.ip_cap < kFusedItems ? static_cast<uint32_t>(v.ip_cap) : kFusedItems;
    for (uint32_t i = threadIdx.x; i < span; i += kFusedBlock) {
        s_node[i] = v.it_node[i];
        s_first[i] = v.it_first[i];
        s_end[i] = v.it_end[i];
        s_cold[i] = v.it_cold[i];
        s_k[i] = v.it_k[i];
        s_off[i] = v.it_off[i];
        s_cs[i] = v.it_cs[i];
    }
    __syncthreads();
    uint32_t total = 0, pieces = 0;
    for (int d = 0; d < H; ++d) {
        const uint32_t e = s_st.lvl_base[d] + s_st.lvl_count[d];
        total = e > total ? e : total;
        pieces += s_st.lvl_new[d];
    }
    if (total > span || pieces > kFusedItems) {  // cannot happen for at most kFusedMax keys
        if (threadIdx.x == 0) atomicOr(&t.hdr->error, kErrInternal);
        return;
    }
    const ItemView iv{s_node, s_first, s_end, s_cold, s_k, s_off, s_cs};
    // every phase below works on the state's copy (the growth and the
    // commit write only fields that no later kernel reads)
    Ins<K> vr = v;
    vr.st = &s_st;
    apply_leaves_body<K, false>(t, vr, grp, ngrp, iv);
    __syncthreads();
    for (int d = 1; d < H; ++d) {
        if (s_st.lvl_new[d - 1] == 0) break;  // nothing split below: no level above changes
        apply_inner_body<K>(t, vr, d, grp, ngrp, iv);
        __syncthreads();
    }
    grow_body<K>(t, vr);
    __syncthreads();
    if (threadIdx.x == 0) ph_commit<K>(t, vr);
    __syncthreads();
    if (s_st.mirror_dirty) mirror_refresh_body<K, kFusedBlock>(t);
}

template <class K>
__global__ __launch_bounds__(kFusedBlock) void k_small_apply(TreeView<K> t, Ins<K> v, int H) {
    ph_small_apply<K>(t, v, H);
}

// The parent levels from d0 on, the root growth, the commit and the mirror
// in one workgroup: the host starts it at the first level where that is no
// slower than a launch of its own, so the upper levels (and the levels above
// the tree's current height, which the host cannot see) cost none.  The
// workgroup's 64 groups of kNodeLanes walk a level's items in rounds of
// 2 us, a launch costs as much or a little more:
//  - batches of at most kTailItems keys, two rounds a level, go to the tail
//    from the first level on: inserts of 80 keys into 2^24 where nothing
//    splits above the leaves 22.9 us, 27.9 with the levels launched, where
//    every level splits 50.6 and 48.7; of 256 keys 24.3 and 29.5, but 78.0
//    and 51.7;
//  - else the tail starts at the first level that can hold at most kTailNodes
//    nodes.  That bound counts the whole leaf pool and 8 children a node; a
//    level holds nearer a tenth of it, so a round or two (insert, lookup and
//    delete of 1000 keys 88.8 us, 93.7 with the bound at one round).
constexpr uint32_t kTailItems = 128;
constexpr uint32_t kTailNodes = 1024;

template <class K>
__global__ __launch_bounds__(kFusedBlock) void k_apply_tail(TreeView<K> t, Ins<K> v, int d0, int H) {
    __shared__ InsState s_st;
    const uint64_t grp = threadIdx.x / kNodeLanes, ngrp = kFusedBlock / kNodeLanes;
    copy_state(&s_st, v.st, threadIdx.x, blockDim.x);
    __syncthreads();
    Ins<K> vr = v;  // the rebuilds read the state's copy
    vr.st = &s_st;
    for (int d = d0; d < H; ++d) {
        if (s_st.lvl_new[d - 1] == 0) break;  // nothing split below: no level above changes
        apply_inner_body<K>(t, vr, d, grp, ngrp, items_in(v));
        __syncthreads();
    }
    grow_body<K>(t, v);
    __syncthreads();
    if (threadIdx.x == 0) ph_commit<K>(t, v);
    __syncthreads();
    if (v.st->mirror_dirty) mirror_refresh_body<K, kFusedBlock>(t);
}

// ------------------------------------------------------ one key (B = 1)
//
// A batch of one key in one workgroup.  Wave 0 descends from the root,
// keeping each inner node's key and child lines (lane s holds slot s, one
// copy per lane in LDS), and finds the key in its leaf.  A present key gets
// its value.  A new key goes into its leaf; a leaf that held 16 keys splits
// evenly into two, and so does every parent, from the leaves up, that held
// 16 children when a child split; a root that splits grows a new root.
// Node ids, separators, padding, the capacity check and the header commit
// are those the batch path (plan, check and apply above) gives a one-key
// batch, so both leave the same tree.  Every read precedes every write; the
// whole workgroup then refreshes the mirror if the top levels changed.
constexpr int kOneBlock = 256;

template <class K>
__global__ __launch_bounds__(kOneBlock) void k_insert_one(TreeView<K> t, const K* __restrict__ keys,
                                                          const K* __restrict__ vals, uint8_t* __restrict__ status) {
    __shared__ K s_sep[kMaxLevels][64];
    __shared__ uint32_t s_ch[kMaxLevels][64];
    __shared__ uint32_t s_node[kMaxLevels], s_cnt[kMaxLevels], s_slot[kMaxLevels];
    __shared__ uint32_t s_dirty;
    const uint32_t tid = threadIdx.x;
    if (tid < 64) {
        const int s = static_cast<int>(tid) & (kSlots - 1);
        const bool w = tid < static_cast<uint32_t>(kSlots);  // the lanes that write slot s
        DevHeader* hdr = t.hdr;
        const K key = keys[0], val = vals[0];
        const uint32_t h = hdr->height, root = hdr->root, err = hdr->error, epoch = hdr->epoch;
        const uint64_t n0 = hdr->n_keys;
        const uint32_t leaf_used = hdr->leaf_used, inner_used = hdr->inner_used;

        // descent: inner level l (0 = root); slot 15 is never a separator
        uint32_t ref = root;
        for (uint32_t l = 0; l + 1 < h; ++l) {
            const uint64_t at = static_cast<uint64_t>(ref) * kSlots + s;
            const K sp = t.ikeys[at];
            const uint32_t c = t.ichild[at];
            const uint32_t ci = static_cast<uint32_t>(__popcll(__ballot(sp < key) & 0x7FFFull));
            const uint32_t cnt =
                1u + static_cast<uint32_t>(__popcll(__ballot(s < kFirstSlot && sp != kmax<K>()) & 0xFFFFull));
            s_sep[l][tid] = sp;
            s_ch[l][tid] = c;
            s_node[l] = ref;
            s_cnt[l] = cnt;
            s_slot[l] = ci;
            ref = shfl_u32(c, static_cast<int>(ci));
        }
        const uint32_t lf = ref & ~kLeafTag;
        const uint64_t la = static_cast<uint64_t>(lf) * kSlots;
        const K lk = t.lkeys[la + s];
        const K lv = t.lvals[la + s];
        const uint2 meta = t.lmeta[lf];
        __threadfence_block();  // every old line is in registers before any write
        const uint64_t eq = __ballot(lk == key) & 0xFFFFull;
        bool ok = !(err & kErrInternal);
        uint32_t dirty = 0;
        if (eq && n0 != 0) {
            // present: the value in place (padding repeats the last key, so
            // the first equal slot is a real one)
            const uint32_t fs = static_cast<uint32_t>(__builtin_ctzll(eq));
            if (tid == 0) {
                status[0] = 1;
                if (ok) {
                    t.lvals[la + fs] = val;
                    hdr->epoch = epoch + 1;
                    reinterpret_cast<MirrorHeader*>(t.mirror)->n_keys = n0;
                }
            }
        } else {
            const uint32_t c = meta.x, total = c + 1;
            const uint32_t pos =
                static_cast<uint32_t>(__popcll(__ballot(static_cast<uint32_t>(s) < c && lk < key) & 0xFFFFull));
            // levels that split, counted from the leaves (0) up
            uint32_t nsplit = total > static_cast<uint32_t>(kSlots) ? 1u : 0u;
            if (nsplit)
                for (int l = static_cast<int>(h) - 2; l >= 0 && s_cnt[l] + 1 > static_cast<uint32_t>(kSlots); --l)
                    ++nsplit;
            const bool grow = nsplit == h;
            const uint32_t leaf_new = nsplit ? 1u : 0u;
            const uint32_t inner_split = nsplit ? nsplit - 1 : 0u;
            const uint32_t inner_new = inner_split + (grow ? 1u : 0u);
            if (static_cast<uint64_t>(leaf_used) + leaf_new > t.leaf_cap ||
                static_cast<uint64_t>(inner_used) + inner_new > t.inner_cap || h + (grow ? 1u : 0u) > kMaxLevels)
                ok = false;
            if (tid == 0) status[0] = 0;
            if (!ok) {
                if (tid == 0 && !(err & kErrInternal)) atomicOr(&hdr->error, kErrCapacity);
            } else {
                // leaf entry e of the c + 1: old keys below pos, the new key,
                // old keys above
                auto lentry = [&](uint32_t e, K& ke, K& ve) {
                    const int src = static_cast<int>(e <= pos ? e : e - 1);
                    const K ok_ = __shfl(lk, src, 64), ov = __shfl(lv, src, 64);
                    ke = e == pos ? key : ok_;
                    ve = e == pos ? val : ov;
                };
                K sepup = K(0);
                uint32_t newref = 0;
                if (total <= static_cast<uint32_t>(kSlots)) {
                    const uint32_t e = static_cast<uint32_t>(s) < total ? static_cast<uint32_t>(s) : total - 1;
                    K ke, ve;
                    lentry(e, ke, ve);
                    if (w) {
                        t.lkeys[la + s] = ke;
                        t.lvals[la + s] = static_cast<uint32_t>(s) < total ? ve : kmax<K>();
                    }
                    if (tid == 0) t.lmeta[lf] = make_uint2(total, meta.y);
                } else {
                    // 17 entries: [0, 8) stay, [8, 17) go to leaf_used
                    const uint64_t nb = static_cast<uint64_t>(leaf_used) * kSlots;
                    K k0, v0, k1, v1, k7, v7;
                    lentry(s < 8 ? static_cast<uint32_t>(s) : 7u, k0, v0);
                    lentry(8u + (s < 9 ? static_cast<uint32_t>(s) : 8u), k1, v1);
                    lentry(7u, k7, v7);
                    if (w) {
                        t.lkeys[la + s] = k0;
                        t.lvals[la + s] = s < 8 ? v0 : kmax<K>();
                        t.lkeys[nb + s] = k1;
                        t.lvals[nb + s] = s < 9 ? v1 : kmax<K>();
                    }
                    if (tid == 0) {
                        t.lmeta[lf] = make_uint2(8u, leaf_used);
                        t.lmeta[leaf_used] = make_uint2(9u, meta.y);
                    }
                    sepup = k7;
                    newref = kLeafTag | leaf_used;
                }
                // parents from the leaf parents up, while a child split
                uint32_t cursor = inner_used;
                bool split = nsplit > 0;
                for (int l = static_cast<int>(h) - 2; l >= 0 && split; --l) {
                    const uint32_t C = s_cnt[l], cs = s_slot[l], node = s_node[l], E = C + 1;
                    const K osp = s_sep[l][tid];
                    const uint32_t och = s_ch[l][tid];
                    // entry e of the C + 1: the split child's slot holds its
                    // first piece with the piece separator, the next entry its
                    // second piece with the child's old separator
                    auto ientry = [&](uint32_t e, K& se, uint32_t& ce) {
                        const uint32_t src = e <= cs ? e : e - 1;
                        const K sv = __shfl(osp, static_cast<int>(src), 64);
                        const uint32_t cv = shfl_u32(och, static_cast<int>(src));
                        se = e == cs ? sepup : (src + 1 < C ? sv : kmax<K>());
                        ce = e == cs + 1 ? newref : cv;
                    };
                    const uint64_t na = static_cast<uint64_t>(node) * kSlots;
                    if (E <= static_cast<uint32_t>(kSlots)) {
                        K se;
                        uint32_t ce;
                        ientry(static_cast<uint32_t>(s) < E ? static_cast<uint32_t>(s) : 0u, se, ce);
                        if (w) {
                            const bool in = static_cast<uint32_t>(s) < E;
                            t.ikeys[na + s] = in && static_cast<uint32_t>(s) + 1 < E ? se : kmax<K>();
                            t.ichild[na + s] = in ? ce : kNone;
                        }
                        split = false;
                    } else {
                        // 17 entries: [0, 8) stay, [8, 17) go to a new node
                        const uint32_t ni = cursor++;
                        const uint64_t nn = static_cast<uint64_t>(ni) * kSlots;
                        K s0, s1, s7;
                        uint32_t c0, c1, c7;
                        ientry(s < 8 ? static_cast<uint32_t>(s) : 0u, s0, c0);
                        ientry(8u + (s < 9 ? static_cast<uint32_t>(s) : 0u), s1, c1);
                        ientry(7u, s7, c7);
                        if (w) {
                            t.ikeys[na + s] = s + 1 < 8 ? s0 : kmax<K>();
                            t.ichild[na + s] = s < 8 ? c0 : kNone;
                            t.ikeys[nn + s] = s + 1 < 9 ? s1 : kmax<K>();
                            t.ichild[nn + s] = s < 9 ? c1 : kNone;
                        }
                        sepup = s7;
                        newref = ni;
                    }
                }
                uint32_t new_root = root;
                if (split) {
                    // the root split: a new root over its two pieces
                    new_root = cursor;
                    const uint32_t oldref = h == 1 ? (kLeafTag | lf) : s_node[0];
                    const uint64_t ra = static_cast<uint64_t>(new_root) * kSlots;
                    if (w) {
                        t.ikeys[ra + s] = s == 0 ? sepup : kmax<K>();
                        t.ichild[ra + s] = s == 0 ? oldref : (s == 1 ? newref : kNone);
                    }
                }
                if (tid == 0) {
                    hdr->n_keys = n0 + 1;
                    hdr->leaf_used = leaf_used + leaf_new;
                    hdr->inner_used = inner_used + inner_new;
                    if (grow) {
                        hdr->height = h + 1;
                        hdr->root = new_root;
                    }
                    hdr->epoch = epoch + 1;
                    reinterpret_cast<MirrorHeader*>(t.mirror)->n_keys = n0 + 1;
                }
                // the mirror's levels change when the tree was empty, the root
                // grew, or children of its top three levels split
                bool d = grow || n0 == 0;
                for (int l = 0; l < 3; ++l) {
                    const int dc = static_cast<int>(h) - 2 - l;
                    if (dc >= 0 && static_cast<uint32_t>(dc) < nsplit) d = true;
                }
                dirty = d ? 1u : 0u;
            }
        }
        if (tid == 0) s_dirty = dirty;
    }
    __syncthreads();
    if (s_dirty) mirror_refresh_body<K, kOneBlock>(t);
}

// The testing switch of the one-key kernel (on by default).
static std::atomic<int> g_single_key{1};
int set_single_key_insert(int on) { return g_single_key.exchange(on ? 1 : 0, std::memory_order_relaxed); }
static bool single_key_insert_on() { return g_single_key.load(std::memory_order_relaxed) != 0; }

// ------------------------------------------------- small batches (B <= 2048)
//
// One launch over many workgroups ranks and locates the batch
// (k_rank_locate); one workgroup sized to the batch plans every level
// (k_small_plan), and up to kFusedMax keys one more workgroup applies the
// whole batch (k_small_apply).  The results are those of the general
// path: the same item arrays and level counters, the same apply bodies.
// Batches of 2 to kFusedMax keys run all of it in one launch by default
// (k_ins_small, below), with the same results.

constexpr int kSmallBlock = 1024;

// Exclusive scans of W words over the plan's workgroup with one barrier: every
// wave adds up the waves before it by itself.  One wave needs no LDS; else
// `sh` holds W words per wave and a barrier must separate two uses of it.
template <int NT, int W>
__device__ __forceinline__ void plan_scan(uint32_t (&x)[W], uint32_t* sh, uint32_t (&total)[W]) {
    constexpr int nw = NT / 64;
    const int w = static_cast<int>(threadIdx.x >> 6), lane = static_cast<int>(threadIdx.x & 63);
    uint32_t inc[W];
#pragma unroll
    for (int i = 0; i < W; ++i) inc[i] = wave_incl_scan(x[i]);
    if constexpr (nw == 1) {
#pragma unroll
        for (int i = 0; i < W; ++i) {
            total[i] = shfl_u32(inc[i], 63);
            x[i] = inc[i] - x[i];
        }
    } else {
        if (lane == 63) {
#pragma unroll
            for (int i = 0; i < W; ++i) sh[w * W + i] = inc[i];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < W; ++i) {
            const uint32_t s = lane < nw ? sh[lane * W + i] : 0u;
            const uint32_t si = wave_incl_scan(s);
            total[i] = shfl_u32(si, 63);
            x[i] = inc[i] - x[i] + shfl_u32(si - s, w);
        }
    }
}

// Locate's records of a batch of at most kFusedMax distinct keys, by tree
// level l (0 = the leaves' parents) and key: the parent, its entry count
// and the slot taken, and each key's leaf entry count.  The one-launch
// insert stages them in LDS with all its threads before it plans.
struct PlanRecs {
    uint32_t pn[kMaxLevels][kFusedMax];
    uint8_t pc[kMaxLevels][kFusedMax];
    uint8_t pi[kMaxLevels][kFusedMax];
    uint8_t ulc[kFusedMax];
};

// Plan of a small batch, one workgroup of NT threads (NT >= B / 2); thread t
// owns new keys 2t and 2t+1.  Small NT keeps the barriers cheap (one wave
// for B <= 128).
//
// The nodes a new key passes through are known from the locate kernel (its
// leaf and, at every level, its parent, the parent's size and the slot taken),
// so the items (runs of new keys through one node) are cut for kPlanLevels
// levels at once: one round of reads, one scan of the levels' run heads, two
// levels to a word.  The piece counts then follow level after level: an item
// gains the new keys of its run (leaves) or sum(k - 1) over its child items
// (inner nodes), a difference of the child level's piece-offset prefix taken
// by the run's first and last keys; above a level where nothing split there
// is nothing left to count.  It is bound by its chain of barriers and LDS
// round trips: 1000 keys on 2^24 take 15.4 us, 19.8 with the levels cut one
// after another.  Writes the same item arrays and level counters as the general
// path, and then the values of keys already present.
constexpr int kPlanLevels = 6;  // inner levels and leaves of 2^24 keys

template <class K, int NT>
__device__ __forceinline__ void ph_small_plan(TreeView<K> t, Ins<K> v, int H) {
    constexpr int kL = kMaxLevels, Q = kPlanLevels;
    constexpr uint32_t kCap = 2 * NT;  // new keys, items per level
    __shared__ uint32_t sh[Q / 2 * (NT / 64)];
    __shared__ uint32_t s_a[kCap], s_b[kCap];  // key -> distinct key, leaf; later prefix sums at item bounds
    __shared__ uint16_t s_ix[kL * kCap];       // item index of each key, per level
    __shared__ uint32_t s_k[kCap + 1];         // piece-offset prefix of the previous level's items
    __shared__ uint8_t s_C[kL * kCap];         // old entry count of every item
    __shared__ uint32_t s_base[kL + 1];        // first item of each level
    __shared__ uint32_t s_over;
    __shared__ InsState s_st;  // the batch state, written back at the end
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    copy_state(&s_st, v.st, tid, NT);
    if (tid == 0) s_over = 0;
    __syncthreads();
    const uint32_t U = s_st.U;
    const int h = static_cast<int>(s_st.height);
    const int hmax = H < h ? H : h;

    // new keys in key order (locate left f0[u] = 1 for a key not in its leaf)
    uint32_t fl[2];
    for (int j = 0; j < 2; ++j) {
        const uint32_t u = 2 * tid + j;
        fl[j] = u < U ? v.f0[u] : 0u;
    }
    uint32_t o0[1] = {fl[0] + fl[1]}, tot0[1];
    plan_scan<NT, 1>(o0, sh, tot0);
    const uint32_t R = tot0[0];
    for (int j = 0; j < 2; ++j) {
        if (!fl[j]) continue;
        const uint32_t u = 2 * tid + j, r = o0[0] + (j ? fl[0] : 0u);
        const uint32_t leaf = v.uleaf[u];
        v.nk[r] = v.uk[u];
        v.nv[r] = v.uv[u];
        v.nleaf[r] = leaf;
        v.nu[r] = u;
        s_a[r] = u;
        s_b[r] = leaf;
    }
    __syncthreads();
    bool valid[2];
    uint32_t nu[2], leaf[2], ixp[2];
    for (int j = 0; j < 2; ++j) {
        const uint32_t r = 2 * tid + j;
        valid[j] = r < R;
        nu[j] = valid[j] ? s_a[r] : 0u;
        leaf[j] = valid[j] ? s_b[r] : 0u;
        ixp[j] = r;  // at the leaf level an item's range counts keys
    }
    // the key next to the wave's: the one before its first, after its last
    const uint32_t nr = lane == 0 ? 2 * tid - 1 : 2 * tid + 2;
    const bool nb = (lane == 0 && tid > 0 && nr < R) || (lane == 63 && nr < R);
    const uint32_t nbu = nb ? s_a[nr] : 0u, nbleaf = nb ? s_b[nr] : 0u;

    // items of every level: heads and ends of runs, item index per key
    uint32_t hbits = 0, lbits = 0, items = 0;
#pragma unroll 1
    for (int l0 = 0; l0 < hmax; l0 += Q) {
        if (l0 > 0) __syncthreads();  // sh is rewritten
        // per level and key: node, its old entry count and its slot in its
        // parent, all recorded by locate
        uint32_t node[Q][2], cnt[Q][2], cs[Q][2], nbn[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int d = l0 + q;
            const bool on = d < hmax;
            const uint64_t at = d > 0 && on ? static_cast<uint64_t>(h - 1 - d) * v.Bm : 0ull;
            const uint64_t up = on && h - 2 - d >= 0 ? static_cast<uint64_t>(h - 2 - d) * v.Bm : 0ull;
            for (int j = 0; j < 2; ++j) {
                const bool ok = on && valid[j];
                node[q][j] = d == 0 ? leaf[j] : (ok ? v.pn[at + nu[j]] : 0u);
                cnt[q][j] = ok ? (d == 0 ? v.ulc[nu[j]] : v.pc[at + nu[j]]) : 0u;
                cs[q][j] = ok && h - 2 - d >= 0 ? v.pi[up + nu[j]] : 0u;
            }
            nbn[q] = d == 0 ? nbleaf : (on && nb ? v.pn[at + nbu] : 0u);
        }
        uint32_t x[Q / 2], n[Q / 2];
#pragma unroll
        for (int i = 0; i < Q / 2; ++i) x[i] = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int d = l0 + q;
            if (d >= hmax) continue;
            uint32_t before = static_cast<uint32_t>(__shfl_up(static_cast<int>(node[q][1]), 1, 64));
            uint32_t after = static_cast<uint32_t>(__shfl_down(static_cast<int>(node[q][0]), 1, 64));
            if (lane == 0) before = nbn[q];
            if (lane == 63) after = nbn[q];
            const uint32_t r = 2 * tid;
            const uint32_t h0 = valid[0] && (r == 0 || before != node[q][0]) ? 1u : 0u;
            const uint32_t h1 = valid[1] && node[q][1] != node[q][0] ? 1u : 0u;
            const uint32_t e0 = valid[0] && (!valid[1] || node[q][1] != node[q][0]) ? 1u : 0u;
            const uint32_t e1 = valid[1] && (r + 2 == R || after != node[q][1]) ? 1u : 0u;
            hbits |= (h0 | h1 << 1) << (2 * d);
            lbits |= (e0 | e1 << 1) << (2 * d);
            x[q / 2] += (h0 + h1) << (16 * (q & 1));
        }
        plan_scan<NT, Q / 2>(x, sh, n);  // a level has at most 2048 heads: 16 bits hold its sums
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int d = l0 + q;
            if (d >= hmax) continue;
            const uint32_t oh = (x[q / 2] >> (16 * (q & 1))) & 0xFFFFu;
            for (int j = 0; j < 2; ++j) {
                const uint32_t hd = (hbits >> (2 * d + j)) & 1u, hd0 = (hbits >> (2 * d)) & 1u;
                const uint32_t ix = oh + (j ? hd0 : 0u) + hd - 1u;
                const uint64_t e = static_cast<uint64_t>(items) + ix;
                if (valid[j]) s_ix[d * kCap + 2 * tid + j] = static_cast<uint16_t>(ix);
                if (hd) {
                    if (e < v.ip_cap) {
                        v.it_node[e] = node[q][j];
                        v.it_first[e] = ixp[j];
                        v.it_cold[e] = cnt[q][j];
                        v.it_cs[e] = static_cast<uint8_t>(cs[q][j]);
                        s_C[e] = static_cast<uint8_t>(cnt[q][j]);
                    } else {
                        s_over = 1;
                    }
                }
                if (((lbits >> (2 * d + j)) & 1u) && e < v.ip_cap) v.it_end[e] = ixp[j] + 1u;
                ixp[j] = ix;
            }
            if (tid == 0) s_base[d] = items;
            items += (n[q / 2] >> (16 * (q & 1))) & 0xFFFFu;
        }
    }
    if (tid == 0) s_base[hmax] = items;
    __syncthreads();

    const uint32_t total = items < v.ip_cap ? items : static_cast<uint32_t>(v.ip_cap);

    // piece counts, level after level.  An item's gain is its run's key
    // count (leaves) or sum(k - 1) over its child items (inner levels): a
    // difference of the child level's piece-offset prefix (s_k), taken by
    // the run's first and last keys.
    // Every LDS read of a step is issued before any of them is used (the
    // indexes of keys and items past the end are clamped to 0 rather than
    // branched around), and each key's item at the level below stays in a
    // register: a single wave otherwise waits out one LDS round trip per read.
    uint32_t psep = 0;
    uint32_t below[2] = {0u, 0u};  // each key's item index at level d - 1
#pragma unroll 1
    for (int d = 0; d < hmax; ++d) {
        const uint32_t bd = s_base[d], nd = s_base[d + 1] - bd;
        uint32_t ixd[2], c[2], e[2];
        for (int j = 0; j < 2; ++j) {
            const uint32_t r = 2 * tid + j;
            ixd[j] = s_ix[d * kCap + (valid[j] ? r : 0u)];
            c[j] = d == 0 ? r : s_k[below[j]];
            e[j] = d == 0 ? r + 1 : s_k[below[j] + 1];
        }
        for (int j = 0; j < 2; ++j) {
            if (!valid[j]) continue;
            if ((hbits >> (2 * d + j)) & 1u) s_a[ixd[j]] = c[j];
            if ((lbits >> (2 * d + j)) & 1u) s_b[ixd[j]] = e[j];
            below[j] = ixd[j];
        }
        __syncthreads();
        uint32_t kk[2], f[2];
        for (int i = 0; i < 2; ++i) {
            const uint32_t jt = 2 * tid + i;
            const bool in = jt < nd && bd + jt < total;
            const uint32_t at = in ? jt : 0u;
            const uint32_t C = s_C[in ? bd + jt : 0u], hi = s_b[at], lo = s_a[at];
            kk[i] = in ? split_pieces(static_cast<uint64_t>(C) + (hi - lo)) : 1u;
            f[i] = in ? kk[i] - 1u : 0u;
        }
        uint32_t of[1] = {f[0] + f[1]}, nn[1];
        plan_scan<NT, 1>(of, sh, nn);  // (the barriers around s_a, s_k separate its uses of sh)
        const uint32_t nnew = nn[0];
        // s_k now holds this level's piece-offset prefix, s_k[nd] its total
        for (int i = 0; i < 2; ++i) {
            const uint32_t jt = 2 * tid + i;
            const uint32_t o = of[0] + (i ? f[0] : 0u);
            if (jt < nd) s_k[jt] = o;
            if (jt < nd && bd + jt < total) {
                v.it_k[bd + jt] = kk[i];
                v.it_off[bd + jt] = o;
            }
        }
        if (tid == 0) {
            s_k[nd] = nnew;
            s_st.lvl_count[d] = nd;
            s_st.lvl_base[d] = bd;
            s_st.lvl_new[d] = nnew;
            s_st.lvl_psep[d] = psep;
        }
        psep += nnew;
        if (nnew == 0) {  // nothing splits above
            for (uint32_t i = s_base[d + 1] + tid; i < total; i += NT) {
                v.it_k[i] = 1u;
                v.it_off[i] = 0u;
            }
            for (int a = d + 1 + static_cast<int>(tid); a < hmax; a += NT) {
                s_st.lvl_count[a] = s_base[a + 1] - s_base[a];
                s_st.lvl_base[a] = s_base[a];
                s_st.lvl_new[a] = 0;
                s_st.lvl_psep[a] = psep;
            }
            break;
        }
        __syncthreads();
    }
    if (tid == 0) {
        s_st.R = R;
        if (s_over) s_st.overflow = 1;
    }
    __syncthreads();
    // the check reads the level counters one after another: from LDS
    Ins<K> vs = v;
    vs.st = &s_st;
    ph_check<K>(t, vs, tid, NT);
    __syncthreads();
    copy_state(v.st, &s_st, tid, NT);
    // values of keys already present (the batch passed the capacity check;
    // the leaf rewrites that follow read these values)
    // (at most 2 NT distinct keys: each thread's two are read before either
    // is written, so the reads take one round)
    if (s_st.ok) {
        uint32_t found[2], leaf[2], slot[2];
        K val[2];
        for (int j = 0; j < 2; ++j) {
            const uint32_t u = tid + j * NT;
            const bool in = u < U;
            found[j] = in ? v.ufound[u] : 0u;
            leaf[j] = in ? v.uleaf[u] : 0u;
            slot[j] = in ? v.uslot[u] : 0u;
            val[j] = in ? v.uv[u] : K(0);
        }
        for (int j = 0; j < 2; ++j)
            if (found[j]) t.lvals[static_cast<uint64_t>(leaf[j]) * kSlots + slot[j]] = val[j];
    }
}

template <class K, int NT>
__global__ __launch_bounds__(NT) void k_small_plan(TreeView<K> t, Ins<K> v, int H) {
    ph_small_plan<K, NT>(t, v, H);
}

// The plan of a one-launch insert (at most kFusedMax distinct keys, one per
// lane of a wave), by the whole workgroup.  The items of every level are cut
// at once, one wave per level: a level's run heads and each key's item index
// (a wave scan over the heads) depend only on that level's nodes, which
// locate recorded (staged in LDS in `rec`).  The item arrays follow once the
// level bases are known; then one wave takes the piece counts level after
// level (each level's offsets need the level below), the capacity check and
// the values of present keys, as the small path's plan does, with the same
// item arrays and level counters.
template <class K>
__device__ __forceinline__ void ph_fused_plan(TreeView<K> t, Ins<K> v, int H, const PlanRecs& rec) {
    constexpr int kL = kMaxLevels;
    constexpr uint32_t kCap = kFusedMax;
    static_assert(kFusedBlock / 64 >= kL, "a wave per level");
    __shared__ uint32_t s_nu[kCap], s_leaf[kCap];  // new key -> distinct key, leaf
    __shared__ uint8_t s_ix[kL][kCap];              // item index of each new key, per level
    __shared__ uint32_t s_n[kL], s_base[kL + 1];    // items per level, first item of each level
    __shared__ uint32_t s_lo[kCap], s_hi[kCap];     // a level's item bounds in the level below's prefix
    __shared__ uint32_t s_k[kCap + 1];              // piece-offset prefix of the level below
    __shared__ uint8_t s_C[kL * kCap];              // old entry count of every item
    __shared__ uint32_t s_R, s_over;
    __shared__ InsState s_st;                       // the batch state, written back at the end
    const uint32_t tid = threadIdx.x, lane = tid % 64, w = tid / 64;
    copy_state(&s_st, v.st, tid, kFusedBlock);
    __syncthreads();
    const uint32_t U = s_st.U;
    const int h = static_cast<int>(s_st.height);
    const int hmax = H < h ? H : h;

    // new keys in key order (locate left f0[u] = 1 for a key not in its leaf)
    if (w == 0) {
        const uint32_t u = lane;
        const uint32_t f = u < U ? v.f0[u] : 0u;
        const uint32_t inc = wave_incl_scan(f);
        if (f) {
            const uint32_t r = inc - 1u, leaf = v.uleaf[u];
            v.nk[r] = v.uk[u];
            v.nv[r] = v.uv[u];
            v.nleaf[r] = leaf;
            v.nu[r] = u;
            s_nu[r] = u;
            s_leaf[r] = leaf;
        }
        if (lane == 63) {
            s_R = inc;
            s_over = 0;
        }
    }
    __syncthreads();
    const uint32_t R = s_R;

    // each level's items: run heads and ends, item index per key (wave d)
    const int d = static_cast<int>(w);
    const uint32_t r = lane;
    const bool valid = d < hmax && r < R;
    const uint32_t nu = valid ? s_nu[r] : 0u;
    auto node_at = [&](uint32_t x) { return d == 0 ? s_leaf[x] : rec.pn[h - 1 - d][s_nu[x]]; };
    uint32_t node = 0, hd = 0, ls = 0;
    if (valid) {
        node = node_at(r);
        hd = (r == 0 || node_at(r - 1) != node) ? 1u : 0u;
        ls = (r + 1 == R || node_at(r + 1) != node) ? 1u : 0u;
    }
    uint32_t ix = 0;
    if (d < hmax) {
        const uint32_t inc = wave_incl_scan(hd);
        ix = inc - 1u;
        if (valid) s_ix[d][r] = static_cast<uint8_t>(ix);
        if (lane == 63) s_n[d] = inc;
    }
    __syncthreads();
    if (tid == 0) {
        uint32_t items = 0;
        for (int l = 0; l < hmax; ++l) {
            s_base[l] = items;
            items += s_n[l];
        }
        s_base[hmax] = items;
    }
    __syncthreads();
    // the item arrays: node, range of child items (keys at the leaves), old entry count, slot in the parent
    if (valid) {
        const uint64_t e = static_cast<uint64_t>(s_base[d]) + ix;
        const uint32_t ixp = d == 0 ? r : s_ix[d - 1][r];
        if (hd) {
            if (e < v.ip_cap) {
                const uint32_t cnt = d == 0 ? rec.ulc[nu] : rec.pc[h - 1 - d][nu];
                const uint32_t cs = h - 2 - d >= 0 ? rec.pi[h - 2 - d][nu] : 0u;
                v.it_node[e] = node;
                v.it_first[e] = ixp;
                v.it_cold[e] = cnt;
                v.it_cs[e] = static_cast<uint8_t>(cs);
                s_C[e] = static_cast<uint8_t>(cnt);
            } else {
                s_over = 1;
            }
        }
        if (ls && e < v.ip_cap) v.it_end[e] = ixp + 1u;
    }
    __syncthreads();
    if (w != 0) return;

    // piece counts, level after level (one key and one item per lane): an
    // item gains its run's key count (leaves) or sum(k - 1) over its child
    // items, a difference of the level below's piece-offset prefix taken by
    // the run's first and last keys
    const uint32_t total_items = s_base[hmax];
    const uint32_t total = total_items < v.ip_cap ? total_items : static_cast<uint32_t>(v.ip_cap);
    const bool kv = r < R;
    uint32_t psep = 0, below = 0;
#pragma unroll 1
    for (int l = 0; l < hmax; ++l) {
        const uint32_t bd = s_base[l], nd = s_base[l + 1] - bd;
        const uint32_t ixl = kv ? s_ix[l][r] : 0u;
        const uint32_t lo = l == 0 ? r : s_k[below], hi = l == 0 ? r + 1 : s_k[below + 1];
        const bool head = kv && (r == 0 || s_ix[l][r - 1] != ixl);
        const bool end = kv && (r + 1 == R || s_ix[l][r + 1] != ixl);
        if (head) s_lo[ixl] = lo;
        if (end) s_hi[ixl] = hi;
        below = ixl;
        wave_sync();
        const uint32_t jt = lane;
        const bool in = jt < nd && bd + jt < total;
        const uint32_t C = s_C[in ? bd + jt : 0u], ih = s_hi[in ? jt : 0u], il = s_lo[in ? jt : 0u];
        const uint32_t kk = in ? split_pieces(static_cast<uint64_t>(C) + (ih - il)) : 1u;
        const uint32_t f = in ? kk - 1u : 0u;
        const uint32_t inc = wave_incl_scan(f);
        const uint32_t nnew = __shfl(inc, 63, 64), o = inc - f;
        if (jt < nd) s_k[jt] = o;
        if (in) {
            v.it_k[bd + jt] = kk;
            v.it_off[bd + jt] = o;
        }
        if (lane == 0) {
            s_k[nd] = nnew;
            s_st.lvl_count[l] = nd;
            s_st.lvl_base[l] = bd;
            s_st.lvl_new[l] = nnew;
            s_st.lvl_psep[l] = psep;
        }
        psep += nnew;
        wave_sync();
    }
    if (lane == 0) {
        s_st.R = R;
        if (s_over) s_st.overflow = 1;
    }
    wave_sync();
    Ins<K> vs = v;
    vs.st = &s_st;
    ph_check<K>(t, vs, lane, 64);
    wave_sync();
    copy_state(v.st, &s_st, lane, 64);
    // values of keys already present (one per lane, read before written)
    if (s_st.ok && lane < U && v.ufound[lane])
        t.lvals[static_cast<uint64_t>(v.uleaf[lane]) * kSlots + v.uslot[lane]] = v.uv[lane];
}

// Stable rank of a[i] = k0 among a[0..n) in LDS (by key, then position):
// eight reads in flight at a time, where one at a time waits out every
// read's latency.
template <class K>
__device__ __forceinline__ uint32_t stable_rank(const K* a, uint32_t n, K k0, uint32_t i) {
    uint32_t c = 0, j = 0;
    for (; j + 8 <= n; j += 8) {
        K x[8];
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) x[q] = a[j + q];
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) c += (x[q] < k0 || (x[q] == k0 && j + q < i)) ? 1u : 0u;
    }
    for (; j < n; ++j) c += (a[j] < k0 || (a[j] == k0 && j < i)) ? 1u : 0u;
    return c;
}

// A batch of at most kFusedMax keys in one launch: the small path's kernels
// (rank and distinct keys, locate, plan, apply) as phases of one
// kFusedBlock-thread workgroup, with barriers where the small path has
// kernel boundaries.  The batch is ranked in LDS (by key, then by position,
// as the small path ranks it) and planned with the small path's item arrays
// and counters (ph_fused_plan), so the tree it leaves is the small path's.
template <class K>
__global__ __launch_bounds__(kFusedBlock) void k_ins_small(TreeView<K> t, Ins<K> v, const K* __restrict__ keys,
                                                           const K* __restrict__ vals, uint32_t B,
                                                           uint8_t* __restrict__ status, int H) {
    __shared__ K s_rk[kFusedMax];
    __shared__ K s_sk[kFusedMax];
    __shared__ uint32_t s_si[kFusedMax];
    __shared__ uint32_t sh[33];
    const uint32_t tid = threadIdx.x;
    uint32_t* st = reinterpret_cast<uint32_t*>(v.st);
    for (uint32_t i = tid; i < sizeof(InsState) / 4; i += kFusedBlock) st[i] = 0;
    if (tid < B) s_rk[tid] = keys[tid];
    __syncthreads();
    // each key's stable rank in the batch
    if (tid < B) {
        const K k0 = s_rk[tid];
        const uint32_t c = stable_rank(s_rk, B, k0, tid);
        s_sk[c] = k0;
        s_si[c] = tid;
    }
    __syncthreads();
    // the distinct keys, each with the value of its last occurrence; a
    // repeat reports UPDATED (an earlier occurrence inserts the key)
    const bool in = tid < B;
    const bool head = in && (tid == 0 || s_sk[tid] != s_sk[tid - 1]);
    const bool last = in && (tid + 1 == B || s_sk[tid + 1] != s_sk[tid]);
    if (in) {
        v.sk[tid] = s_sk[tid];
        v.si[tid] = s_si[tid];  // locate writes each distinct key's status through it
        if (!head) status[s_si[tid]] = 1;
    }
    uint32_t U;
    const uint32_t pos = block_excl_scan<uint32_t>(head ? 1u : 0u, sh, &U);
    if (head) {
        v.uk[pos] = s_sk[tid];
        v.upos[pos] = tid;
    }
    if (last) v.uv[pos + (head ? 1u : 0u) - 1u] = vals[s_si[tid]];
    if (tid == 0) {
        v.st->U = U;
        v.st->height = t.hdr->height;
    }
    __syncthreads();
    ph_locate<K, 16, 1, 2, kFusedBlock>(t, v, status);
    __syncthreads();
    // the plan's reads of locate's records, in one round by every thread
    __shared__ PlanRecs s_rec;
    {
        const uint32_t h = v.st->height, Ud = v.st->U;
        const uint32_t nl = h >= 2 ? h - 1 : 0;  // levels 0 .. h-2
        for (uint32_t i = tid; i < nl * Ud; i += kFusedBlock) {
            const uint32_t l = i / Ud, u = i % Ud;
            const uint64_t at = static_cast<uint64_t>(l) * v.Bm + u;
            s_rec.pn[l][u] = v.pn[at];
            s_rec.pc[l][u] = v.pc[at];
            s_rec.pi[l][u] = v.pi[at];
        }
        if (tid < Ud) s_rec.ulc[tid] = v.ulc[tid];
    }
    __syncthreads();
    ph_fused_plan<K>(t, v, H, s_rec);
    __syncthreads();
    ph_small_apply<K>(t, v, H);
}

static std::atomic<int> g_one_launch_insert{1};
int set_one_launch_insert(int on) { return g_one_launch_insert.exchange(on ? 1 : 0, std::memory_order_relaxed); }
static bool one_launch_insert_on() { return g_one_launch_insert.load(std::memory_order_relaxed) != 0; }

// ------------------------------------------------------------------ launch

static uint32_t grid_for(uint64_t n, uint32_t per_block) {
    uint64_t g = (n + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > 8192) g = 8192;
    return static_cast<uint32_t>(g);
}

template <class K, int G, int QPG, int LV>
static void launch_locate_t(const TreeView<K>& t, const Ins<K>& v, uint64_t B, uint8_t* status, hipStream_t s) {
    const uint32_t lds = LV > 0 ? MirrorLayout<K>::bytes(mirror_nodes_for_levels(LV)) : 0;
    uint32_t grid = grid_for((B + QPG - 1) / QPG, kBlk / G);
    if (grid > 2048) grid = 2048;
    hipLaunchKernelGGL((k_locate<K, G, QPG, LV>), dim3(grid), dim3(kBlk), lds, s, t, v, status);
}

// Shape by batch size, as for lookups: small batches are latency-bound (16
// lanes, one key per group); large ones are bound by the rate of line
// requests (8 lanes, two keys in flight per group: 75.6 us for 2^20 keys where
// four, with fewer waves, took 77.9).
template <class K, int G, int QPG>
static void launch_locate_lv(const TreeView<K>& t, const Ins<K>& v, const LaunchCfg& cfg, uint64_t B,
                             uint8_t* status, hipStream_t s) {
    switch (cfg.lds_levels) {
        case 0: launch_locate_t<K, G, QPG, 0>(t, v, B, status, s); break;
        case 1: launch_locate_t<K, G, QPG, 1>(t, v, B, status, s); break;
        case 3: launch_locate_t<K, G, QPG, 3>(t, v, B, status, s); break;
        default: launch_locate_t<K, G, QPG, 2>(t, v, B, status, s); break;
    }
}

template <class K>
static void launch_locate(const TreeView<K>& t, const Ins<K>& v, const LaunchCfg& cfg, uint64_t B, uint8_t* status,
                          hipStream_t s) {
    if (B >= kLocateBatch) launch_locate_lv<K, 8, 2>(t, v, cfg, B, status, s);
    else launch_locate_lv<K, 16, 1>(t, v, cfg, B, status, s);
}

template <class K, int LV, bool INS>
static void launch_rank_locate_t(const TreeView<K>& t, const Ins<K>& v, const K* keys, const K* vals, uint32_t B,
                                 uint8_t* status, hipStream_t s) {
    const uint32_t lds = LV > 0 ? MirrorLayout<K>::bytes(mirror_nodes_for_levels(LV)) : 0;
    hipLaunchKernelGGL((k_rank_locate<K, LV, INS>), dim3((B + kBlk / 16 - 1) / (kBlk / 16)), dim3(kBlk), lds, s, t, v,
                       keys, vals, B, status);
}

template <class K, bool INS>
static void launch_rank_locate(const TreeView<K>& t, const Ins<K>& v, const LaunchCfg& cfg, const K* keys,
                               const K* vals, uint32_t B, uint8_t* status, hipStream_t s) {
    switch (cfg.lds_levels) {
        case 0: launch_rank_locate_t<K, 0, INS>(t, v, keys, vals, B, status, s); break;
        case 1: launch_rank_locate_t<K, 1, INS>(t, v, keys, vals, B, status, s); break;
        case 3: launch_rank_locate_t<K, 3, INS>(t, v, keys, vals, B, status, s); break;
        default: launch_rank_locate_t<K, 2, INS>(t, v, keys, vals, B, status, s); break;
    }
}

// highest tree height the pools allow (non-root inner nodes have >= 8
// children, the root >= 2)
static int height_bound(uint64_t leaf_cap) {
    int h = 1;
    uint64_t cover = 2;  // leaves a tree of height h+1 can have at least
    while (cover <= leaf_cap && h < kMaxLevels - 1) {
        ++h;
        cover *= 8;
    }
    return h + 1 < kMaxLevels ? h + 1 : kMaxLevels;
}

// apply, grow, commit, mirror: shared by both paths (the small path's plan
// kernel writes the updates itself)
template <class K>
static void launch_apply(const TreeView<K>& t, const Ins<K>& v, uint64_t B, uint64_t leaf_cap, int H, bool updates,
                         hipStream_t s) {
    const uint32_t gB = grid_for(B, kBlk);
    if (updates) hipLaunchKernelGGL(k_apply_updates<K>, dim3(gB), dim3(kBlk), 0, s, t, v);
    hipLaunchKernelGGL(k_apply_leaves<K>, dim3(grid_for(B, kBlk / kNodeLanes)), dim3(kBlk), 0, s, t, v);
    int d0 = 1;
    while (B > kTailItems && d0 < H && level_items_bound(~0ull, leaf_cap, d0) > kTailNodes) ++d0;
    for (int d = 1; d < d0; ++d)
        hipLaunchKernelGGL(k_apply_inner<K>, dim3(grid_for(B, kBlk / kNodeLanes)), dim3(kBlk), 0, s, t, v, d);
    hipLaunchKernelGGL(k_apply_tail<K>, dim3(1), dim3(kFusedBlock), 0, s, t, v, d0, H);
}

template <class K>
void launch_insert(const TreeView<K>& t, const InsertCtx& c, const K* keys, const K* vals, uint64_t B,
                   uint8_t* status, hipStream_t s) {
    Ins<K> v;
    carve<K>(&v, c.scratch, c.max_batch, c.leaf_cap, c.inner_cap);
    InsState* st = v.st;
    const uint32_t gB = grid_for(B, kBlk);
    const int H = height_bound(c.leaf_cap);

    if (B == 1 && single_key_insert_on()) {
        hipLaunchKernelGGL(k_insert_one<K>, dim3(1), dim3(kOneBlock), 0, s, t, keys, vals, status);
        return;
    }
    if (B <= kFusedMax && one_launch_insert_on()) {
        const uint32_t lds = MirrorLayout<K>::bytes(mirror_nodes_for_levels(2));
        hipLaunchKernelGGL(k_ins_small<K>, dim3(1), dim3(kFusedBlock), lds, s, t, v, keys, vals,
                           static_cast<uint32_t>(B), status, H);
        return;
    }
    if (B <= kSmallInsert) {
        launch_rank_locate<K, true>(t, v, c.cfg, keys, vals, static_cast<uint32_t>(B), status, s);
        if (B <= 128) hipLaunchKernelGGL((k_small_plan<K, 64>), dim3(1), dim3(64), 0, s, t, v, H);
        else if (B <= 512) hipLaunchKernelGGL((k_small_plan<K, 256>), dim3(1), dim3(256), 0, s, t, v, H);
        else hipLaunchKernelGGL((k_small_plan<K, kSmallBlock>), dim3(1), dim3(kSmallBlock), 0, s, t, v, H);
        if (B <= kFusedMax) hipLaunchKernelGGL(k_small_apply<K>, dim3(1), dim3(kFusedBlock), 0, s, t, v, H);
        else launch_apply<K>(t, v, B, c.leaf_cap, H, false, s);  // the plan wrote the updates
        return;
    }
    sort_from<K>(keys, v.sk, v.si, v.sk2, v.si2, B, v.sort_tmp, s, &t.hdr->error, kErrInternal);
    uint32_t* sums = v.f1;  // a word per chunk and level: 16 per 2048 keys at most
    const Chunks cb = chunks_for(B);
    hipLaunchKernelGGL(k_ch_heads<K>, dim3(cb.n), dim3(kChBlock), 0, s, v, t.hdr, B, cb.tiles, uint8_t(1), status, sums);
    hipLaunchKernelGGL(k_ch_unique<K>, dim3(cb.n), dim3(kChBlock), 0, s, v, B, cb.tiles, vals, sums);
    launch_locate<K>(t, v, c.cfg, B, status, s);
    hipLaunchKernelGGL((k_ch_count<K, true>), dim3(cb.n), dim3(kChBlock), 0, s, t, v, cb.tiles, sums);
    hipLaunchKernelGGL((k_ch_collect<K, true>), dim3(cb.n), dim3(kChBlock), 0, s, t, v, cb.tiles, sums);
    hipLaunchKernelGGL(k_ch_level_count<K>, dim3(cb.n), dim3(kChBlock), 0, s, v, cb.tiles, sums);
    hipLaunchKernelGGL(k_ch_level_items<K>, dim3(cb.n), dim3(kChBlock), 0, s, v, cb.tiles, sums);
    // the pieces of the lower levels by chunks, of the others in one workgroup
    // (4 us per 8192 items where the two chunk kernels take 13 a level): a tree
    // level has at most an eighth of the nodes of the one below.  2^20 keys on
    // 2^24: 835 us a pass, 846 with the third level in the workgroup
    const int d0 = B <= 8192 ? 0 : (B <= 65536 ? 1 : 3);
    for (int d = 0; d < d0; ++d) {
        const Chunks cd = chunks_for(level_items_bound(B, c.leaf_cap, d));
        hipLaunchKernelGGL(k_ch_pieces<K>, dim3(cd.n), dim3(kChBlock), 0, s, v, d, cd.tiles, sums);
        hipLaunchKernelGGL(k_ch_offsets<K>, dim3(cd.n), dim3(kChBlock), 0, s, v, d, cd.tiles, sums);
    }
    hipLaunchKernelGGL(k_plan_tail<K>, dim3(1), dim3(kTailBlock), 0, s, t, v, d0);
    launch_apply<K>(t, v, B, c.leaf_cap, H, true, s);
}

template void launch_insert<uint32_t>(const TreeView<uint32_t>&, const InsertCtx&, const uint32_t*,
                                      const uint32_t*, uint64_t, uint8_t*, hipStream_t);
template void launch_insert<uint64_t>(const TreeView<uint64_t>&, const InsertCtx&, const uint64_t*,
                                      const uint64_t*, uint64_t, uint8_t*, hipStream_t);

// ---------------------------------------------------------------- delete
//
// A delete batch (Section III: every node but the root stays at least half
// full) shares the insert's front end: sort, distinct keys, and a locate
// that records each key's path.  Then:
//  1. one thread per touched leaf removes the batch's keys from it in place
//     (survivors moved down, padding rewritten).  If the leaf's largest key
//     went and the leaf stays at least half full, it rewrites the separator
//     that holds that key: on the path, the first node whose child slot is
//     not its last;
//  2. one wave per leaf parent with a child left below half full gathers the
//     parent's keys (at most 16 x 16) and spreads them evenly over
//     max(8, ceil(T / 16)) of its leaves, which borrows and merges in one
//     step.  The leaves no longer needed are cleared (count 0) and dropped
//     from the chain, the parent's line is rewritten, and its new largest
//     key goes into its own separator further up.  A parent that is the
//     root keeps at least two leaves, or becomes the single leaf root when
//     16 keys or fewer remain (the root shrinks);
//  3. a parent that would keep fewer than 64 keys would itself fall below
//     half full; the batch flags it and the host rebuilds the tree from its
//     keys.

constexpr uint32_t kHalf = kSlots / 2;

// A counter that earlier threads raised with atomics (in the L2), read past
// the L1, which may still hold its line from before.
__device__ __forceinline__ uint32_t counter(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Inner nodes at depth < kMirrorDepth (0 = the root) are copied in the
// top-levels mirror: rewriting one, or moving the root, means the mirror
// must be refreshed at the commit (otherwise only its key count changes).
constexpr int kMirrorDepth = 3;

template <class K>
__device__ __forceinline__ void note_inner_write(const Ins<K>& v, int depth) {
    if (depth < kMirrorDepth) v.st->mirror_dirty = 1u;
}
constexpr uint64_t kDelListHere = 2048;   // up to here the leaf kernel lists the merges
static_assert(kDelListHere == kSmallInsert, "its records are k_rank_locate's");
constexpr uint64_t kDelListScan = 16384;  // above: the merge list comes from a scan, in key order

// first distinct key of its leaf's run (keys are sorted, so a leaf's keys
// are consecutive)
template <class K>
__device__ __forceinline__ bool leaf_run_head(const Ins<K>& v, uint64_t u) {
    return u == 0 || v.uleaf[u - 1] != v.uleaf[u];
}

// Or over a row of 16 lanes, in every lane.
__device__ __forceinline__ uint32_t row_or(uint32_t x) {
    x |= __builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x128, 0xf, 0xf, false);  // row_ror:8, 4, 2, 1
    x |= __builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x124, 0xf, 0xf, false);
    x |= __builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x122, 0xf, 0xf, false);
    x |= __builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x121, 0xf, 0xf, false);
    return x;
}

// 16 lanes per touched leaf, lane s on slot s: the lanes read the run's
// distinct keys 16 at a time for the slots to remove, then the kept pairs move
// down (each lane reads the pair its slot gets from the lane that holds it)
// and the leaf's lines are written whole.  A group's first read is its 16
// next keys' records, its second the leaf of its own key, needed or not, so a
// leaf costs two dependent rounds; R keys a group are in flight.  Returns
// how many keys the wave removed.  The leaves left below half full are listed
// for the merges: here (LIST, an atomic for the wave's four groups, in any
// order) or, for larger batches, by the kernels after this one.
// REP: k_rank_locate's records, of which a repeated key has one per occurrence
// (only the first counts) and upos the place after its last one: a run goes on
// from there, so that repeats are not walked (2048 times one key 39 us, 87
// walked).
template <class K, int R, bool LIST, bool REP>
__device__ __forceinline__ uint32_t ph_del_leaf(TreeView<K> t, Ins<K> v) {
    if (t.hdr->error & kErrInternal) return 0;  // e.g. the batch's device sort gave up
    const uint64_t U = v.st->U;
    const int h = static_cast<int>(v.st->height);
    const int lane = static_cast<int>(threadIdx.x) & 63, s = lane & (kSlots - 1), gbase = lane - s;
    const uint64_t g0 = gtid() / kSlots, gs = gstride() / kSlots;
    uint32_t del = 0;  // keys this group removed (lane 0 of the group)
    for (uint64_t ub = g0;; ub += R * gs) {
        if (__ballot(ub < U) == 0) break;  // the wave's four groups are done
        uint32_t le[R], prev[R];  // key u + s: its leaf; the leaf of the key before u
        uint32_t rec[R];          // key u + s: found, and its slot
        uint32_t next[R];         // the record after key u + 15 and its repeats
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint64_t u = ub + r * gs, e = u + static_cast<uint64_t>(s);
            next[r] = REP && u + kSlots <= U ? v.upos[u + kSlots - 1] : 0u;
            const bool in = e < U;
            le[r] = in ? v.uleaf[e] : kNone;
            rec[r] = in ? (v.ufound[e] ? 0x100u : 0u) | v.uslot[e] : 0u;
            prev[r] = u < U && u > 0 ? v.uleaf[u - 1] : kNone;
        }
        K key[R], val[R];
        uint32_t cnt[R], leaf[R];
        bool head[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint64_t u = ub + r * gs;
            leaf[r] = row_lane<0>(le[r]);
            head[r] = u < U && (u == 0 || prev[r] != leaf[r]);  // the same for the group's 16 lanes
            cnt[r] = 0;
            key[r] = val[r] = K(0);
            if (head[r]) {
                cnt[r] = t.lmeta[leaf[r]].x;
                key[r] = t.lkeys[static_cast<uint64_t>(leaf[r]) * kSlots + s];
                val[r] = t.lvals[static_cast<uint64_t>(leaf[r]) * kSlots + s];
            }
            if (u < U && s == 0 && !head[r]) v.nu[u] = 0u;  // only a run left below half full sets 1
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint64_t u = ub + r * gs;
            uint32_t gone = 0, nd = 0;
            {
                uint32_t lx = le[r], rx = rec[r], nx = next[r];
                bool more = head[r];
                for (uint64_t e0 = u; __ballot(more);) {
                    const bool in = more && lx == leaf[r];
                    const bool hit = in && (rx & 0x100u);
                    const uint32_t bits = row_or(hit ? 1u << (rx & 0xFFu) : 0u);
                    gone |= bits;
                    nd += static_cast<uint32_t>(__popcll((__ballot(hit) >> gbase) & 0xFFFFull));
                    more = ((__ballot(in) >> gbase) & 0xFFFFull) == 0xFFFFull;  // else the run ended here
                    if (!__ballot(more)) break;
                    e0 = REP ? nx : e0 + kSlots;
                    const uint64_t e = e0 + static_cast<uint64_t>(s);
                    const bool ok = more && e < U;
                    if (REP) nx = more && e0 + kSlots <= U ? v.upos[e0 + kSlots - 1] : 0u;
                    lx = ok ? v.uleaf[e] : kNone;
                    rx = ok ? (v.ufound[e] ? 0x100u : 0u) | v.uslot[e] : 0u;
                }
            }
            const uint32_t c = cnt[r], w = c - nd;
            const bool under = h > 1 && w < kHalf;
            if (head[r] && s == 0) {
                v.f0[u] = under ? 1u : 0u;
                v.nu[u] = under ? 1u : 0u;
                if constexpr (LIST) {
                    if (under) v.f1[atomicAdd(&v.st->merges, 1u)] = static_cast<uint32_t>(u);
                }
            }
            // slot s gets the pair of the s-th kept slot; past the count the
            // last kept key with an all-ones value
            const uint32_t km = ((1u << c) - 1u) & ~gone;  // c <= 16
            const uint32_t want = static_cast<uint32_t>(s) < w ? static_cast<uint32_t>(s) : (w ? w - 1u : 0u);
            uint32_t src = 0;  // the position of bit number `want` of km
            {
                uint32_t m = km, k = want;
#pragma unroll
                for (int half = 8; half > 0; half >>= 1) {
                    const uint32_t lowc = static_cast<uint32_t>(__popc(m & ((1u << half) - 1u)));
                    if (k >= lowc) {
                        k -= lowc;
                        m >>= half;
                        src += static_cast<uint32_t>(half);
                    }
                }
            }
            const K mk = static_cast<K>(__shfl(key[r], gbase + static_cast<int>(src), 64));
            const K mv = static_cast<K>(__shfl(val[r], gbase + static_cast<int>(src), 64));
            if (head[r] && nd) {
                const uint64_t line = static_cast<uint64_t>(leaf[r]) * kSlots + s;
                t.lkeys[line] = w ? mk : kmax<K>();
                t.lvals[line] = static_cast<uint32_t>(s) < w ? mv : kmax<K>();
                if (static_cast<uint32_t>(s) == kSlots - 1) {  // this lane holds the new largest key
                    t.lmeta[leaf[r]].x = w;
                    del += nd;
                    if (!under && w > 0 && ((gone >> (c - 1)) & 1u)) {
                        for (int l = h - 2; l >= 0; --l) {
                            const uint64_t o2 = static_cast<uint64_t>(l) * v.Bm + u;
                            if (v.pi[o2] + 1u < v.pc[o2]) {
                                t.ikeys[static_cast<uint64_t>(v.pn[o2]) * kSlots + v.pi[o2]] = mk;
                                note_inner_write(v, l);
                                break;
                            }
                        }
                    }
                }
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) del += static_cast<uint32_t>(__shfl_xor(static_cast<int>(del), o));
    return del;
}

// The workgroup's count goes to its own word of parts (the sort's second key
// buffer, at least a word per workgroup), which the commit adds up: one add a
// wave to a single word took 12 ns each, 390 of this kernel's 394 us for 2^20
// keys on 2^24 (88 now).
template <class K, int R, bool LIST, bool REP>
__global__ __launch_bounds__(kBlk) void k_del_leaf(TreeView<K> t, Ins<K> v, uint32_t* __restrict__ parts) {
    __shared__ uint32_t s_del[kBlk / 64];
    const uint32_t del = ph_del_leaf<K, R, LIST, REP>(t, v);
    if ((threadIdx.x & 63) == 0) s_del[threadIdx.x / 64] = del;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t d = 0;
        for (int w = 0; w < kBlk / 64; ++w) d += s_del[w];
        parts[blockIdx.x] = d;
    }
}

// The leaf runs left below half full, listed for the merge pass: batches of
// up to kDelListHere keys list them where they arise, an atomic per wave of
// the leaf kernel (1000 keys on 2^24: 2.7 us of this kernel and its launch
// saved; the counter takes one atomic in 12 ns, so not for more), those up to
// kDelListScan here, an atomic per 64 keys, both in any order; larger ones
// place each run at its prefix-scan position, so the list is in key order.
template <class K>
__global__ void k_del_list(TreeView<K> t, Ins<K> v) {
    if (t.hdr->error & kErrInternal) return;
    const uint64_t U = v.st->U;
    for (uint64_t u = gtid(); u < U; u += gstride())
        if (v.nu[u]) v.f1[atomicAdd(&v.st->merges, 1u)] = static_cast<uint32_t>(u);
}

// A wave's LDS for merging one listed parent.
template <class K>
struct MergeLds {
    K mk[kSlots * kSlots];
    K mv[kSlots * kSlots];
    uint32_t kid[kSlots], cnt[kSlots], pre[kSlots + 1];
    uint32_t next;
};

// Orders a wave's LDS writes before its lanes' later reads (a wave-level
// barrier: the body runs in one wave).
// One wave per listed parent: wave w of nw takes list entries w, w + nw, ...
// with its own LDS slice (the batch kernel: one wave per workgroup; the
// one-launch delete: the waves of its workgroup).
template <class K>
__device__ __forceinline__ void ph_del_merge(TreeView<K> t, Ins<K> v, bool ordered, uint32_t w, uint32_t nw,
                                             MergeLds<K>& sm) {
    if (t.hdr->error & kErrInternal) return;
    const int h = static_cast<int>(v.st->height);
    if (h < 2) return;
    K* const mk = sm.mk;
    K* const mv = sm.mv;
    uint32_t* const kid = sm.kid;
    uint32_t* const cnt = sm.cnt;
    uint32_t* const pre = sm.pre;
    uint32_t& s_next = sm.next;
    const int lane = lane_id();
    const uint64_t lp = static_cast<uint64_t>(h - 2) * v.Bm;  // path level of the leaves' parents
    const uint32_t nlist = counter(&v.st->merges);
    for (uint32_t li = w; li < nlist; li += nw) {
        // a leaf run that left its leaf below half full; the first such run
        // under its parent merges that parent
        const uint64_t u = v.f1[li];
        const uint32_t P = v.pn[lp + u];
        bool first = true;
        if (ordered) {
            // the list is in key order, and a parent's runs are consecutive
            first = li == 0 || v.pn[lp + v.f1[li - 1]] != P;
        } else {
            for (uint64_t e = u; e-- > 0 && v.pn[lp + e] == P;) {
                if (leaf_run_head(v, e) && v.f0[e]) {
                    first = false;
                    break;
                }
            }
        }
        if (!first) continue;
        const uint32_t nc = v.pc[lp + u];
        const K fs = t.ikeys[static_cast<uint64_t>(P) * kSlots + kFirstSlot];
        if (lane < kSlots) {
            uint32_t ref = kNone;
            if (static_cast<uint32_t>(lane) < nc)
                ref = fs != kmax<K>() ? static_cast<uint32_t>(fs) + static_cast<uint32_t>(lane)
                                      : t.ichild[static_cast<uint64_t>(P) * kSlots + lane];
            kid[lane] = ref & ~kLeafTag;
            const uint32_t c = static_cast<uint32_t>(lane) < nc ? t.lmeta[ref & ~kLeafTag].x : 0u;
            cnt[lane] = c < kSlots ? c : kSlots;
        }
        wave_sync();
        if (lane == 0) {
            uint32_t a = 0;
            for (int i = 0; i < kSlots; ++i) {
                pre[i] = a;
                a += cnt[i];
            }
            pre[kSlots] = a;
            s_next = t.lmeta[kid[nc - 1]].y;
        }
        wave_sync();
        const uint32_t T = pre[kSlots];
        const bool root = h == 2;
        if (!root && T < kHalf * kHalf) {
            // the parent would fall below half full: its grandparent merges
            // it with its siblings (marked 2, listed for the next kernel)
            if (lane == 0) {
                v.f0[u] = 2u;
                v.upos[atomicAdd(&v.st->gmerges, 1u)] = static_cast<uint32_t>(u);
            }
            wave_sync();
            continue;
        }
        {
            // 16 lanes per child, slot = lane % 16, four children per round:
            // every load of the gather in flight at once, few registers
            const uint32_t j = static_cast<uint32_t>(lane) % kSlots;
            K kk[4], vv[4];
#pragma unroll
            for (uint32_t r = 0; r < 4; ++r) {
                const uint32_t c = r * 4 + static_cast<uint32_t>(lane) / kSlots;
                if (c < nc && j < cnt[c]) {
                    kk[r] = t.lkeys[static_cast<uint64_t>(kid[c]) * kSlots + j];
                    vv[r] = t.lvals[static_cast<uint64_t>(kid[c]) * kSlots + j];
                }
            }
#pragma unroll
            for (uint32_t r = 0; r < 4; ++r) {
                const uint32_t c = r * 4 + static_cast<uint32_t>(lane) / kSlots;
                if (c < nc && j < cnt[c]) {
                    mk[pre[c] + j] = kk[r];
                    mv[pre[c] + j] = vv[r];
                }
            }
        }
        wave_sync();
        const uint32_t want = (T + kSlots - 1) / kSlots;
        const uint32_t n0 = root ? (T <= kSlots ? 1u : (want > 2u ? want : 2u)) : (want > kHalf ? want : kHalf);
        if (n0 > nc) {  // cannot happen on a tree whose nodes were at least half full
            if (lane == 0) atomicOr(&v.st->rebuild, 1u);
            wave_sync();
            continue;
        }
        const uint32_t q = T / n0, r = T % n0;
        // leaf j (lane j < n0) takes pairs [start, start + len)
        if (static_cast<uint32_t>(lane) < nc) {
            const uint32_t j = static_cast<uint32_t>(lane);
            const uint64_t dst = static_cast<uint64_t>(kid[j]) * kSlots;
            if (j < n0) {
                const uint32_t len = q + (j < r ? 1u : 0u), start = j * q + (j < r ? j : r);
                for (uint32_t s = 0; s < kSlots; ++s) {
                    t.lkeys[dst + s] = s < len ? mk[start + s] : (len ? mk[start + len - 1] : kmax<K>());
                    t.lvals[dst + s] = s < len ? mv[start + s] : kmax<K>();
                }
                t.lmeta[kid[j]] = make_uint2(len, j + 1 < n0 ? kid[j + 1] : s_next);
            } else {
                for (uint32_t s = 0; s < kSlots; ++s) {
                    t.lkeys[dst + s] = kmax<K>();
                    t.lvals[dst + s] = kmax<K>();
                }
                t.lmeta[kid[j]] = make_uint2(0u, kNone);
            }
        }
        if (lane == 0) note_inner_write(v, h - 2);  // P, or the root it replaces
        if (root && n0 == 1) {
            // the root shrinks to its first leaf
            if (lane == 0) {
                t.hdr->root = kid[0] | kLeafTag;
                t.hdr->height = 1;
            }
        } else {
            if (lane < kSlots) {
                const uint32_t s = static_cast<uint32_t>(lane);
                K sep = kmax<K>();
                if (s + 1 < n0) {
                    const uint32_t end = (s + 1) * q + (s + 1 < r ? s + 1 : r);  // start of leaf s + 1
                    sep = mk[end - 1];
                }
                t.ikeys[static_cast<uint64_t>(P) * kSlots + s] = sep;  // slot 15: children from the child line
                t.ichild[static_cast<uint64_t>(P) * kSlots + s] = s < n0 ? (kid[s] | kLeafTag) : kNone;
            }
            if (lane == 0 && !root) {
                const K top = mk[T - 1];
                for (int l = h - 3; l >= 0; --l) {
                    const uint64_t o2 = static_cast<uint64_t>(l) * v.Bm + u;
                    if (v.pi[o2] + 1u < v.pc[o2]) {
                        t.ikeys[static_cast<uint64_t>(v.pn[o2]) * kSlots + v.pi[o2]] = top;
                        note_inner_write(v, l);
                        break;
                    }
                }
            }
        }
        wave_sync();
    }
}

template <class K>
__global__ __launch_bounds__(64) void k_del_merge(TreeView<K> t, Ins<K> v, bool ordered) {
    __shared__ MergeLds<K> sm;
    ph_del_merge<K>(t, v, ordered, blockIdx.x, gridDim.x, sm);
}

// One level up: a leaf parent that would fall below half full (fewer than
// 64 keys) is merged with its siblings.  One workgroup per grandparent G
// gathers every pair below G (at most 16 x 16 x 16) in LDS and lays them out
// again over n1 = max(8, ceil(T / 256)) of G's parents and
// n0 = max(8 n1, ceil(T / 16)) of its leaves, reusing old ids in key order
// (a subtree that was at least half full has enough of both).  A root G
// keeps at least two parents, or the tree loses levels: one parent as root
// at T <= 256, one leaf at T <= 16.  A G left with fewer than 512 keys would
// itself fall below half full; the host rebuilds the tree instead.
constexpr int kBelowG = kSlots * kSlots * kSlots;

template <class K>
__device__ __forceinline__ void ph_del_merge2(TreeView<K> t, Ins<K> v) {
    if (t.hdr->error & kErrInternal) return;
    const int h = static_cast<int>(v.st->height);
    if (h < 3) return;
    __shared__ K mk[kBelowG];
    __shared__ K mv[kBelowG];
    __shared__ uint32_t lid[kSlots * kSlots];  // G's leaves in key order
    __shared__ uint32_t pid[kSlots];           // G's parents in order
    __shared__ uint32_t sh[33];
    __shared__ uint32_t s_first, s_next;
    const int tid = static_cast<int>(threadIdx.x);
    const uint64_t lg = static_cast<uint64_t>(h - 3) * v.Bm;  // path level of the grandparents
    const uint32_t nlist = counter(&v.st->gmerges);
    for (uint32_t li = blockIdx.x; li < nlist; li += gridDim.x) {
        const uint64_t u = v.upos[li];
        const uint32_t G = v.pn[lg + u];
        if (tid == 0) {
            // the first marked run under G merges it
            uint32_t first = 1;
            for (uint64_t e = u; e-- > 0 && v.pn[lg + e] == G;) {
                if (leaf_run_head(v, e) && v.f0[e] == 2u) {
                    first = 0;
                    break;
                }
            }
            s_first = first;
        }
        __syncthreads();
        const bool first = s_first != 0;
        __syncthreads();
        if (!first) continue;
        const uint32_t gc = v.pc[lg + u];
        // thread (p, l), tid < 256: leaf l of parent p, from the child lines
        uint32_t lref = kNone, lc = 0;
        if (tid < kSlots * kSlots) {
            const uint32_t p = static_cast<uint32_t>(tid) / kSlots, l = static_cast<uint32_t>(tid) % kSlots;
            if (p < gc) {
                const uint32_t P = t.ichild[static_cast<uint64_t>(G) * kSlots + p];
                if (l == 0) pid[p] = P;
                const uint32_t r = t.ichild[static_cast<uint64_t>(P) * kSlots + l];
                if (r != kNone) {
                    lref = r & ~kLeafTag;
                    const uint32_t c = t.lmeta[lref].x;
                    lc = c < kSlots ? c : kSlots;
                }
            }
        }
        uint32_t nleaf, T;
        const uint32_t lpos = block_excl_scan<uint32_t>(lref != kNone ? 1u : 0u, sh, &nleaf);
        const uint32_t kpos = block_excl_scan<uint32_t>(lc, sh, &T);
        if (lref != kNone) {
            lid[lpos] = lref;
            const uint64_t src = static_cast<uint64_t>(lref) * kSlots;
            for (uint32_t j = 0; j < lc; ++j) {
                mk[kpos + j] = t.lkeys[src + j];
                mv[kpos + j] = t.lvals[src + j];
            }
        }
        __syncthreads();
        if (tid == 0) s_next = nleaf ? t.lmeta[lid[nleaf - 1]].y : kNone;
        const bool root = h == 3;
        uint32_t n1, n0;
        const uint32_t w0 = (T + kSlots - 1) / kSlots, w1 = (T + kSlots * kSlots - 1) / (kSlots * kSlots);
        if (root && T <= kSlots) {
            n1 = 0;
            n0 = 1;
        } else if (root && T <= kSlots * kSlots) {
            n1 = 1;
            n0 = w0 > 2u ? w0 : 2u;
        } else {
            n1 = w1 > (root ? 2u : kHalf) ? w1 : (root ? 2u : kHalf);
            n0 = w0 > kHalf * n1 ? w0 : kHalf * n1;
        }
        const bool fail = (!root && T < kHalf * kHalf * kHalf) || n1 > gc || n0 > nleaf;
        __syncthreads();
        if (fail) {
            if (tid == 0) atomicOr(&v.st->rebuild, 1u);
            __syncthreads();
            continue;
        }
        // leaves: leaf j (j < n0) takes pairs [j q0 + min(j, r0), + len)
        const uint32_t q0 = T / n0, r0 = T % n0;
        auto leaf_end = [&](uint32_t j) { return (j + 1) * q0 + (j + 1 < r0 ? j + 1 : r0); };
        if (static_cast<uint32_t>(tid) < nleaf) {
            const uint32_t j = static_cast<uint32_t>(tid);
            const uint64_t dst = static_cast<uint64_t>(lid[j]) * kSlots;
            if (j < n0) {
                const uint32_t start = j * q0 + (j < r0 ? j : r0), len = leaf_end(j) - start;
                for (uint32_t s2 = 0; s2 < kSlots; ++s2) {
                    t.lkeys[dst + s2] = s2 < len ? mk[start + s2] : (len ? mk[start + len - 1] : kmax<K>());
                    t.lvals[dst + s2] = s2 < len ? mv[start + s2] : kmax<K>();
                }
                t.lmeta[lid[j]] = make_uint2(len, j + 1 < n0 ? lid[j + 1] : s_next);
            } else {
                for (uint32_t s2 = 0; s2 < kSlots; ++s2) {
                    t.lkeys[dst + s2] = kmax<K>();
                    t.lvals[dst + s2] = kmax<K>();
                }
                t.lmeta[lid[j]] = make_uint2(0u, kNone);
            }
        }
        // parents: parent i (i < n1) takes leaves [i q1 + min(i, r1), + c)
        const uint32_t q1 = n1 ? n0 / n1 : 0, r1 = n1 ? n0 % n1 : 0;
        auto par_first = [&](uint32_t i) { return i * q1 + (i < r1 ? i : r1); };
        if (n1 && tid < kSlots * kSlots) {
            const uint32_t i = static_cast<uint32_t>(tid) / kSlots, s2 = static_cast<uint32_t>(tid) % kSlots;
            if (i < n1) {
                const uint32_t a = par_first(i), c = par_first(i + 1) - a;
                const uint64_t P = pid[i];
                t.ichild[P * kSlots + s2] = s2 < c ? (lid[a + s2] | kLeafTag) : kNone;
                t.ikeys[P * kSlots + s2] = s2 + 1 < c ? mk[leaf_end(a + s2) - 1] : kmax<K>();
            }
        }
        if (n1 >= 2 && tid < kSlots) {
            const uint32_t s2 = static_cast<uint32_t>(tid);
            t.ichild[static_cast<uint64_t>(G) * kSlots + s2] = s2 < n1 ? pid[s2] : kNone;
            t.ikeys[static_cast<uint64_t>(G) * kSlots + s2] =
                s2 + 1 < n1 ? mk[leaf_end(par_first(s2 + 1) - 1) - 1] : kmax<K>();
        }
        if (tid == 0) {
            note_inner_write(v, h - 3);  // G and its parents, or the root that replaces G
            if (root && n1 == 0) {
                t.hdr->root = lid[0] | kLeafTag;
                t.hdr->height = 1;
            } else if (root && n1 == 1) {
                t.hdr->root = pid[0];
                t.hdr->height = 2;
            } else if (!root) {
                const K top = mk[T - 1];
                for (int l = h - 4; l >= 0; --l) {
                    const uint64_t o2 = static_cast<uint64_t>(l) * v.Bm + u;
                    if (v.pi[o2] + 1u < v.pc[o2]) {
                        t.ikeys[static_cast<uint64_t>(v.pn[o2]) * kSlots + v.pi[o2]] = top;
                        note_inner_write(v, l);
                        break;
                    }
                }
            }
        }
        __syncthreads();
    }
}

template <class K>
__global__ __launch_bounds__(1024) void k_del_merge2(TreeView<K> t, Ins<K> v) {
    ph_del_merge2<K>(t, v);
}

// Commit the count d of removed keys and the epoch, then refresh the top-levels mirror if a
// mirrored node changed, else only its key count (one launch).
template <class K, int NT>
__device__ __forceinline__ void ph_del_commit(TreeView<K> t, Ins<K> v, uint32_t d) {
    if (threadIdx.x == 0 && !(t.hdr->error & kErrInternal)) {
        if (d) {
            t.hdr->n_keys -= d;
            t.hdr->epoch += 1;
        }
    }
    __syncthreads();
    if (counter(&v.st->mirror_dirty)) {
        mirror_refresh_body<K, NT>(t);
    } else if (threadIdx.x == 0) {
        reinterpret_cast<MirrorHeader*>(t.mirror)->n_keys = t.hdr->n_keys;
    }
}

constexpr int kDelCommitBlock = 1024;

template <class K>
__global__ __launch_bounds__(kDelCommitBlock) void k_del_commit(TreeView<K> t, Ins<K> v,
                                                                 const uint32_t* __restrict__ parts, uint32_t nparts,
                                                                 uint64_t* host_word, uint32_t seq) {
    __shared__ uint32_t sh[33];
    uint32_t d = 0, all;
    for (uint32_t i = threadIdx.x; i < nparts; i += kDelCommitBlock) d += parts[i];
    block_excl_scan<uint32_t>(d, sh, &all);
    ph_del_commit<K, kDelCommitBlock>(t, v, all);
    // the call's number and the rebuild flag (raised by the merge kernels
    // before this one), in one word, straight into host memory
    if (host_word && threadIdx.x == 0) {
        const uint64_t w = (static_cast<uint64_t>(seq) << 32) | (counter(&v.st->rebuild) ? 1u : 0u);
        __hip_atomic_store(host_word, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// A batch of at most kDelFusedMax keys in one launch: the batch path's
// phases, one after the other in a single 1024-thread workgroup (a grid of
// one workgroup runs each phase's loops over one workgroup), so the tree it
// leaves is the batch path's.  The batch is ranked in LDS (by key, then by
// position, the order of the batch path's sort); the parent merges run one
// per wave, the grandparent merges one after the other on the whole
// workgroup.  The workgroup's waves share one CU and its L1, so a barrier
// with its workgroup-scope fences orders the phases' plain loads and stores;
// the counters raised with atomics are read past the L1 (counter()).  A
// device-scope fence here would write back and invalidate the L2 at every
// phase.
constexpr int kDelOneBlock = 1024;
constexpr uint32_t kDelFusedMax = 64;

__device__ __forceinline__ void phase_boundary() {
    __syncthreads();
}

template <class K>
__global__ __launch_bounds__(kDelOneBlock) void k_del_small(TreeView<K> t, Ins<K> v, const K* __restrict__ keys,
                                                            uint32_t B, uint8_t* __restrict__ status,
                                                            uint64_t* host_word, uint32_t seq) {
    __shared__ K s_rk[kDelFusedMax];
    __shared__ K s_sk[kDelFusedMax];
    __shared__ uint32_t s_si[kDelFusedMax];
    __shared__ uint32_t sh[33];
    __shared__ MergeLds<K> s_merge[kDelOneBlock / 64];
    const uint32_t tid = threadIdx.x;
    uint32_t* st = reinterpret_cast<uint32_t*>(v.st);
    for (uint32_t i = tid; i < sizeof(InsState) / 4; i += kDelOneBlock) st[i] = 0;
    if (tid < B) s_rk[tid] = keys[tid];
    phase_boundary();
    // each key's stable rank in the batch
    if (tid < B) {
        const K k0 = s_rk[tid];
        const uint32_t c = stable_rank(s_rk, B, k0, tid);
        s_sk[c] = k0;
        s_si[c] = tid;
    }
    phase_boundary();
    // the distinct keys; a repeat reports ABSENT (an earlier occurrence
    // deletes the key)
    const bool in = tid < B;
    const bool head = in && (tid == 0 || s_sk[tid] != s_sk[tid - 1]);
    if (in) {
        v.sk[tid] = s_sk[tid];
        v.si[tid] = s_si[tid];  // locate writes each distinct key's status through it
        if (!head) status[s_si[tid]] = 0;
    }
    uint32_t U;
    const uint32_t pos = block_excl_scan<uint32_t>(head ? 1u : 0u, sh, &U);
    if (head) {
        v.uk[pos] = s_sk[tid];
        v.upos[pos] = tid;
    }
    if (tid == 0) {
        v.st->U = U;
        v.st->height = t.hdr->height;
    }
    phase_boundary();
    ph_locate<K, 16, 1, 2, kDelOneBlock>(t, v, status);
    phase_boundary();
    {
        const uint32_t del = ph_del_leaf<K, 1, true, false>(t, v);
        if ((tid & 63) == 0 && del) atomicAdd(&v.st->deleted, del);
    }
    phase_boundary();
    ph_del_merge<K>(t, v, false, tid / 64, kDelOneBlock / 64, s_merge[tid / 64]);
    phase_boundary();
    ph_del_merge2<K>(t, v);
    phase_boundary();
    ph_del_commit<K, kDelOneBlock>(t, v, counter(&v.st->deleted));
    // the call's number and the rebuild flag, in one word, straight into
    // host memory (the merges that raise the flag are behind the barriers
    // above): the host waits for this word rather than for the stream
    if (host_word && tid == 0) {
        const uint64_t w = (static_cast<uint64_t>(seq) << 32) | (counter(&v.st->rebuild) ? 1u : 0u);
        __hip_atomic_store(host_word, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

static std::atomic<int> g_one_launch_delete{1};
int set_one_launch_delete(int on) { return g_one_launch_delete.exchange(on ? 1 : 0, std::memory_order_relaxed); }
static bool one_launch_delete_on() { return g_one_launch_delete.load(std::memory_order_relaxed) != 0; }

// Copy every pair of the leaves that hold keys (cleared leaves hold none).
template <class K>
__global__ void k_del_collect(TreeView<K> t, uint32_t leaves, K* __restrict__ ok, K* __restrict__ ov, uint64_t cap,
                              unsigned long long* __restrict__ n) {
    for (uint64_t l = gtid(); l < leaves; l += gstride()) {
        const uint32_t c = t.lmeta[l].x < kSlots ? t.lmeta[l].x : kSlots;
        if (c == 0) continue;
        const uint64_t at = atomicAdd(n, static_cast<unsigned long long>(c));
        if (at + c > cap) continue;  // more pairs than the tree counts: the host reports it
        for (uint32_t j = 0; j < c; ++j) {
            ok[at + j] = t.lkeys[l * kSlots + j];
            ov[at + j] = t.lvals[l * kSlots + j];
        }
    }
}

template <class K>
const uint32_t* launch_delete(const TreeView<K>& t, const InsertCtx& c, const K* keys, uint64_t B, uint8_t* status,
                              uint64_t* host_word, uint32_t seq, bool* flag_on_host, hipStream_t s) {
    *flag_on_host = false;
    Ins<K> v;
    carve<K>(&v, c.scratch, c.max_batch, c.leaf_cap, c.inner_cap);
    const uint32_t gB = grid_for(B, kBlk);
    const Chunks cb = chunks_for(B);
    uint32_t* sums = reinterpret_cast<uint32_t*>(v.nk);  // (f1 holds the merge list)
    if (B <= kDelFusedMax && one_launch_delete_on()) {
        const uint32_t lds = MirrorLayout<K>::bytes(mirror_nodes_for_levels(2));
        hipLaunchKernelGGL(k_del_small<K>, dim3(1), dim3(kDelOneBlock), lds, s, t, v, keys,
                           static_cast<uint32_t>(B), status, host_word, seq);
        *flag_on_host = host_word != nullptr;
        return &v.st->rebuild;
    }
    if (B <= kSmallInsert) {
        launch_rank_locate<K, false>(t, v, c.cfg, keys, nullptr, static_cast<uint32_t>(B), status, s);
    } else {
        sort_from<K>(keys, v.sk, v.si, v.sk2, v.si2, B, v.sort_tmp, s, &t.hdr->error, kErrInternal);
        hipLaunchKernelGGL(k_ch_heads<K>, dim3(cb.n), dim3(kChBlock), 0, s, v, t.hdr, B, cb.tiles, uint8_t(0), status,
                           sums);
        hipLaunchKernelGGL(k_ch_unique<K>, dim3(cb.n), dim3(kChBlock), 0, s, v, B, cb.tiles,
                           static_cast<const K*>(nullptr), sums);
        launch_locate<K>(t, v, c.cfg, B, status, s);
    }
    // two keys in flight per lane group once every group of the grid has more
    const uint32_t gl = grid_for(B * kSlots, kBlk);
    uint32_t* parts = reinterpret_cast<uint32_t*>(v.sk2);
    if (B <= kDelListHere)
        hipLaunchKernelGGL((k_del_leaf<K, 1, true, true>), dim3(gl), dim3(kBlk), 0, s, t, v, parts);
    else if (B >= 2ull * gl * (kBlk / kSlots))
        hipLaunchKernelGGL((k_del_leaf<K, 2, false, false>), dim3(gl), dim3(kBlk), 0, s, t, v, parts);
    else
        hipLaunchKernelGGL((k_del_leaf<K, 1, false, false>), dim3(gl), dim3(kBlk), 0, s, t, v, parts);
    const bool ordered = B > kDelListScan;
    if (ordered) {
        hipLaunchKernelGGL((k_ch_count<K, false>), dim3(cb.n), dim3(kChBlock), 0, s, t, v, cb.tiles, sums);
        hipLaunchKernelGGL((k_ch_collect<K, false>), dim3(cb.n), dim3(kChBlock), 0, s, t, v, cb.tiles, sums);
    } else if (B > kDelListHere) {
        hipLaunchKernelGGL(k_del_list<K>, dim3(gB), dim3(kBlk), 0, s, t, v);
    }
    const uint32_t gm = B < 16384 ? static_cast<uint32_t>(B) : 16384u;
    hipLaunchKernelGGL(k_del_merge<K>, dim3(gm), dim3(64), 0, s, t, v, ordered);
    hipLaunchKernelGGL(k_del_merge2<K>, dim3(B < 256 ? static_cast<uint32_t>(B) : 256u), dim3(1024), 0, s, t, v);
    hipLaunchKernelGGL(k_del_commit<K>, dim3(1), dim3(kDelCommitBlock), 0, s, t, v, parts, gl, host_word, seq);
    *flag_on_host = host_word != nullptr;
    return &v.st->rebuild;
}

template <class K>
void launch_delete_collect(const TreeView<K>& t, uint32_t leaves, K* ok, K* ov, uint64_t cap,
                           unsigned long long* n, hipStream_t s) {
    const uint32_t g = grid_for(leaves ? leaves : 1, kBlk);
    hipLaunchKernelGGL(k_del_collect<K>, dim3(g < 4096 ? g : 4096), dim3(kBlk), 0, s, t, leaves, ok, ov, cap, n);
}

template const uint32_t* launch_delete<uint32_t>(const TreeView<uint32_t>&, const InsertCtx&, const uint32_t*,
                                                 uint64_t, uint8_t*, uint64_t*, uint32_t, bool*, hipStream_t);
template const uint32_t* launch_delete<uint64_t>(const TreeView<uint64_t>&, const InsertCtx&, const uint64_t*,
                                                 uint64_t, uint8_t*, uint64_t*, uint32_t, bool*, hipStream_t);
template void launch_delete_collect<uint32_t>(const TreeView<uint32_t>&, uint32_t, uint32_t*, uint32_t*, uint64_t,
                                              unsigned long long*, hipStream_t);
template void launch_delete_collect<uint64_t>(const TreeView<uint64_t>&, uint32_t, uint64_t*, uint64_t*, uint64_t,
                                              unsigned long long*, hipStream_t);

}  // namespace gt
