// Lookup and range batches.
//
// Lookup (paper Sections IV-A, IV-E, IV-F): every query descends from the
// root with a group of G lanes (see traverse.h), the top inner levels read
// from the LDS copy of the mirror, the rest from HBM; at the leaf an
// equality ballot over the key line gives the slot, and one lane reads the
// value.  A key that is not found returns all ones with found = 0 (the
// paper's -1 result, Section IV-D).  Results go to the caller's order.
//
// Range (an addition over the linked leaves of Section III): the
// group descends to the leaf of `lo`, then walks the leaf chain, one or a few
// leaves at a time; a ballot marks the slots with lo <= key <= hi and the
// group writes them in order at out[offset + running count], until `max`
// pairs are written, a key above `hi` is seen or the chain ends.
//
// Both kernels are persistent: a grid of at most a few thousand
// workgroups walks tiles of queries, so the mirror is staged once per
// workgroup.
#include "common.h"
#include "traverse.h"
#include "kernels.h"

namespace gt {

constexpr int kLookupBlock = 256;

// Leaf stage shared by the lookup kernels: match the key line, take the
// value (from the co-loaded value line, or by one dependent read), write the
// result of every live query.  NT selects non-temporal loads: bit 0 the key
// line, bit 1 the value line (a lookup reads a value line once, so
// streaming it keeps the lines that are reused -- leaf parents, upper
// levels -- in L2).
template <class K, int G, int QPG, bool VC, int NT>
__device__ __forceinline__ void finish_lookups(const TreeView<K>& t, const K (&key)[QPG], const uint32_t (&leaf)[QPG],
                                               const uint64_t (&qi)[QPG], bool empty, int gl, int gbase,
                                               K* __restrict__ vout, uint8_t* __restrict__ fout) {
    using T = Trav<K, G>;
    typename T::KV kv[QPG];
    typename T::KV vv[QPG];
#pragma unroll
    for (int j = 0; j < QPG; ++j) {
        const K* kl = t.lkeys + static_cast<uint64_t>(leaf[j]) * kSlots;
        const K* vl = t.lvals + static_cast<uint64_t>(leaf[j]) * kSlots;
        if constexpr ((NT & 1) != 0) kv[j] = T::load_keys_nt(kl, gl);
        else kv[j] = T::load_keys(kl, gl);
        if constexpr (VC) {
            if constexpr ((NT & 2) != 0) vv[j] = T::load_keys_nt(vl, gl);
            else vv[j] = T::load_keys(vl, gl);
        }
    }
    uint32_t slot[QPG];
#pragma unroll
    for (int j = 0; j < QPG; ++j) slot[j] = T::match_slot(kv[j], key[j], gbase);
    if constexpr (VC) {
        K val[QPG];
        bool hit[QPG];
#pragma unroll
        for (int j = 0; j < QPG; ++j) {
            hit[j] = slot[j] < kSlots && !empty;
            const K x = T::pick_value(vv[j], hit[j] ? slot[j] : 0u, gbase);
            val[j] = hit[j] ? x : kmax<K>();
        }
#pragma unroll
        for (int j = 0; j < QPG; ++j) {
            if (gl == (j % G) && qi[j] != ~0ull) {
                vout[qi[j]] = val[j];
                fout[qi[j]] = hit[j] ? 1 : 0;
            }
        }
    } else {
        // lane j answers query j, so a wave's values and results go out in one
        // read and two stores
        static_assert(QPG <= G, "one answering lane per query");
        const uint32_t sl = own_query<QPG>(slot, gl), lf = own_query<QPG>(leaf, gl);
        uint64_t q = 0;
#pragma unroll
        for (int j = 0; j < QPG; ++j) q |= qi[j] & (gl == j ? ~0ull : 0ull);
        if (gl < QPG && q != ~0ull) {
            const bool hit = sl < kSlots && !empty;
            K val = kmax<K>();
            if (hit) {
                const K* vp = t.lvals + static_cast<uint64_t>(lf) * kSlots + sl;
                if constexpr ((NT & 2) != 0) val = __builtin_nontemporal_load(vp);
                else val = *vp;
            }
            vout[q] = val;
            fout[q] = hit ? 1 : 0;
        }
    }
}

template <class K, int G, int QPG, int LV, bool VC, int NT>
__global__ __launch_bounds__(kLookupBlock) void k_lookup(TreeView<K> t, const K* __restrict__ q, uint64_t B,
                                                          K* __restrict__ vout, uint8_t* __restrict__ fout,
                                                          uint64_t ntiles) {
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
    const int lane = lane_id();
    const int gl = lane % G, gbase = lane - gl;
    const uint64_t group = threadIdx.x / G;
    const uint64_t tile_q = static_cast<uint64_t>(kLookupBlock / G) * QPG;
    for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        K key[QPG];
        uint64_t qi[QPG];
#pragma unroll
        for (int j = 0; j < QPG; ++j) {
            const uint64_t x = tile * tile_q + group * QPG + j;
            key[j] = x < B ? q[x] : K(0);
            qi[j] = x < B ? x : ~0ull;
        }
        uint32_t leaf[QPG];
        descend<K, G, QPG, false>(t, mir, mnodes, LV, key, leaf, gl, gbase);
        finish_lookups<K, G, QPG, VC, NT>(t, key, leaf, qi, empty, gl, gbase, vout, fout);
    }
}

// Position of the t-th set bit (t counted from 0) of m; m has more than t.
__device__ __forceinline__ int nth_set_bit(uint64_t m, uint32_t t) {
    int pos = 0;
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) {
        const uint32_t c = static_cast<uint32_t>(__popcll(m & ((1ull << w) - 1ull)));
        if (t >= c) {
            t -= c;
            m >>= w;
            pos += w;
        }
    }
    return pos;
}

// XCD-split lookup for large batches.  The dispatcher deals the workgroups
// of a launch to the eight XCDs in turn, so workgroups w and w + 8 share an
// XCD and its L2 (which XCD takes workgroup 0 varies; only the grouping is
// used).  Seven splitter keys cut the key space into eight ranges, and the
// workgroups with w % 8 == x answer the queries of range x only, so the leaf
// parents they read (an eighth of them) stay in one L2.  Every wave of group
// x reads four 64-query chunks of the batch at a time (one coalesced load
// each), keeps the queries of its range with one ballot per chunk, and deals
// them to its eight 8-lane groups, four queries per group per round.  Each
// chunk is read by one wave of every XCD; results go by
// query index, so the output is the plain kernel's.  All lanes stay active
// through a round (the groups' cross-lane reads need their source lanes).
constexpr int kXcdChunks = 4;  // 64-query chunks a wave reads at once

template <class K, bool VC, int NT>
__global__ __launch_bounds__(kLookupBlock) void k_lookup_xcd(TreeView<K> t, const K* __restrict__ q, uint64_t B,
                                                              K* __restrict__ vout, uint8_t* __restrict__ fout,
                                                              uint64_t nchunks) {
    constexpr int G = 8, LV = 2, QPG = kXcdChunks;
    constexpr uint32_t kGroups = 64 / G;
    extern __shared__ __align__(16) uint8_t lds[];
    const uint32_t mnodes = mirror_nodes_for_levels(LV);
    stage_mirror<K>(t.mirror, lds, mnodes);
    const MirrorHeader* gmh = reinterpret_cast<const MirrorHeader*>(t.mirror);
    const K* sp = reinterpret_cast<const K*>(t.mirror + MirrorLayout<K>::split_off());
    const uint32_t nsplit = gmh->nsplit;
    K split[kXcds - 1];
#pragma unroll
    for (int x = 0; x < kXcds - 1; ++x) split[x] = sp[x];
    __syncthreads();
    const bool empty = reinterpret_cast<const MirrorHeader*>(lds)->n_keys == 0;
    const uint32_t xcd = blockIdx.x % kXcds;
    const int lane = lane_id();
    const int gl = lane % G, gbase = lane - gl;
    const uint32_t grp = static_cast<uint32_t>(lane / G);
    constexpr int kWaves = kLookupBlock / 64;
    const uint64_t wave_in_xcd = static_cast<uint64_t>(blockIdx.x / kXcds) * kWaves + threadIdx.x / 64;
    const uint64_t waves_per_xcd = static_cast<uint64_t>(gridDim.x / kXcds) * kWaves;
    const uint64_t nsets = (nchunks + kXcdChunks - 1) / kXcdChunks;
    for (uint64_t set = wave_in_xcd; set < nsets; set += waves_per_xcd) {
        K key[kXcdChunks];
        uint64_t m[kXcdChunks];
#pragma unroll
        for (int k = 0; k < kXcdChunks; ++k) {
            const uint64_t qi = (set * kXcdChunks + k) * 64 + static_cast<uint64_t>(lane);
            const bool valid = qi < B;
            key[k] = valid ? q[qi] : K(0);
            uint32_t b = 0;
            if (nsplit) {
#pragma unroll
                for (int x = 0; x < kXcds - 1; ++x) b += split[x] < key[k] ? 1u : 0u;
            } else {
                b = static_cast<uint32_t>(qi % kXcds);
            }
            m[k] = __ballot(valid && b == xcd);
        }
        uint32_t left = 0;
#pragma unroll
        for (int k = 0; k < kXcdChunks; ++k) left += static_cast<uint32_t>(__popcll(m[k]));
        for (uint32_t r0 = 0; r0 < left; r0 += kGroups * QPG) {  // the same for the whole wave
            // group grp takes the selected queries of rank r0 + grp + 8 j
            K kk[QPG];
            uint64_t qq[QPG];
#pragma unroll
            for (int j = 0; j < QPG; ++j) {
                uint32_t rank = r0 + grp + kGroups * static_cast<uint32_t>(j);
                const bool live = rank < left;
                int chunk = 0, src = 0;
                if (live) {
#pragma unroll
                    for (int k = 0; k < kXcdChunks; ++k) {
                        const uint32_t c = static_cast<uint32_t>(__popcll(m[k]));
                        if (chunk == k && rank >= c) {
                            rank -= c;
                            chunk = k + 1;
                        }
                    }
                    src = nth_set_bit(m[chunk], rank);
                }
                // a cross-lane read returns the source lane's register, so
                // read every chunk's key there and keep the wanted one
                K kx = K(0);
#pragma unroll
                for (int k = 0; k < kXcdChunks; ++k) {
                    const K v = static_cast<K>(__shfl(key[k], src, 64));
                    if (chunk == k) kx = v;
                }
                kk[j] = kx;
                qq[j] = live ? (set * kXcdChunks + static_cast<uint64_t>(chunk)) * 64 + static_cast<uint64_t>(src)
                             : ~0ull;
            }
            uint32_t leaf[QPG];
            descend<K, G, QPG, false>(t, lds, mnodes, LV, kk, leaf, gl, gbase);
            finish_lookups<K, G, QPG, VC, NT>(t, kk, leaf, qq, empty, gl, gbase, vout, fout);
        }
    }
}

// A scan is a chain of dependent reads, the descent and then leaf after leaf.
// Few scans leave the chip idle, so a scan takes 16 AH lanes and reads AH
// leaves at once: the leaf it stands on and, on the guess that they follow,
// the leaves of the next references (a bulk load numbers them so; a split's
// new leaf lies elsewhere).  A leaf read ahead counts only if the links of
// the leaves before it lead to it; one that is not linked is out of the scan,
// its contents never used.  1024 scans of 2^24 u64 keys, 1 to 100 pairs, 7.1
// -> 4.2 us with four leaves at once, up to 400 pairs 16.4 -> 6.1; on a tree
// grown by half with inserts 8.8 -> 7.2 and 20.9 -> 15.6.
template <class K, int AH, int LV>
__global__ __launch_bounds__(kLookupBlock) void k_range(TreeView<K> t, const K* __restrict__ lo,
                                                         const K* __restrict__ hi,
                                                         const uint32_t* __restrict__ maxc,
                                                         const uint64_t* __restrict__ off, uint64_t B,
                                                         K* __restrict__ okeys, K* __restrict__ ovals,
                                                         uint32_t* __restrict__ cnt_out, uint64_t ntiles) {
    constexpr int G = kSlots;    // lanes per leaf: one slot each
    constexpr int W = G * AH;    // lanes per scan
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
    const int lane = lane_id();
    const int gl = lane % G, gbase = lane - gl;         // the 16-lane group of a leaf
    const int wl = lane % W, wbase = lane - wl;         // the lanes of a scan
    const uint32_t sub = static_cast<uint32_t>(wl / G);  // which of the leaves ahead
    const uint64_t below = (1ull << wl) - 1ull;
    const uint64_t group = threadIdx.x / W;
    const uint64_t tile_q = kLookupBlock / W;
    for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const uint64_t qi = tile * tile_q + group;
        const bool live = qi < B;
        K key[1] = {live ? lo[qi] : K(0)};
        const K h = live ? hi[qi] : K(0);
        const uint32_t mx = live ? maxc[qi] : 0u;
        const uint64_t base = live ? off[qi] : 0ull;
        uint32_t leaf[1];
        descend<K, G, 1, false>(t, mir, mnodes, LV, key, leaf, gl, gbase);
        uint32_t c = 0;
        bool done = !live || empty || mx == 0 || key[0] > h;
        uint32_t cur = leaf[0];
        while (!done) {
            // leaves the rest of the scan may reach, the first about half used
            const bool want = sub == 0 || mx - c > kSlots * sub - kSlots / 2;
            const uint64_t guess = static_cast<uint64_t>(cur) + sub;
            const bool on = want && guess < t.leaf_cap;
            const uint64_t at = on ? guess : cur;
            const K kv = t.lkeys[at * kSlots + gl];
            const K vv = t.lvals[at * kSlots + gl];
            const uint2 meta = t.lmeta[at];
            // leaf `sub` counts if every leaf before it is followed by the
            // next reference (and is not empty: a scan ends there)
            const uint64_t linked = group_bits<W>(
                __ballot(on && meta.x != 0 && meta.y == static_cast<uint32_t>(guess) + 1u), wbase);
            bool use = on;
#pragma unroll
            for (int s = 0; s + 1 < AH; ++s)
                use = use && (static_cast<uint32_t>(s) >= sub || ((linked >> (s * G)) & 1ull));
            const bool in = use && static_cast<uint32_t>(gl) < meta.x;
            const bool ok = in && kv >= key[0] && kv <= h;
            const uint64_t bits = group_bits<W>(__ballot(ok), wbase);
            const uint64_t over = group_bits<W>(__ballot(in && kv > h), wbase);
            const uint64_t used = group_bits<W>(__ballot(use), wbase);
            const uint32_t p = c + static_cast<uint32_t>(__popcll(bits & below));
            if (ok && p < mx) {
                okeys[base + p] = kv;
                ovals[base + p] = vv;
            }
            c += static_cast<uint32_t>(__popcll(bits));
            // the last leaf that counted leads on
            const int last = wbase + 63 - static_cast<int>(__builtin_clzll(used));
            const uint32_t cnt = shfl_u32(meta.x, last), next = shfl_u32(meta.y, last);
            done = c >= mx || over != 0 || next == kNone || cnt == 0;
            cur = next;
        }
        if (live && wl == 0) cnt_out[qi] = c < mx ? c : mx;
    }
}

// The scan for large batches: 8 lanes per scan and leaf, two slots per lane,
// so that the resident waves hold twice as many scans and none reads ahead.
template <class K, int LV>
__global__ __launch_bounds__(kLookupBlock) void k_range_many(TreeView<K> t, const K* __restrict__ lo,
                                                              const K* __restrict__ hi,
                                                              const uint32_t* __restrict__ maxc,
                                                              const uint64_t* __restrict__ off, uint64_t B,
                                                              K* __restrict__ okeys, K* __restrict__ ovals,
                                                              uint32_t* __restrict__ cnt_out, uint64_t ntiles) {
    constexpr int G = 8;
    using T = Trav<K, G>;
    constexpr int KPL = T::KPL;
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
    const int lane = lane_id();
    const int gl = lane % G, gbase = lane - gl;
    const uint64_t below_lanes = (1ull << gl) - 1ull;
    const uint64_t group = threadIdx.x / G;
    const uint64_t tile_q = kLookupBlock / G;
    for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const uint64_t qi = tile * tile_q + group;
        const bool live = qi < B;
        K key[1] = {live ? lo[qi] : K(0)};
        const K h = live ? hi[qi] : K(0);
        const uint32_t mx = live ? maxc[qi] : 0u;
        const uint64_t base = live ? off[qi] : 0ull;
        uint32_t leaf[1];
        descend<K, G, 1, false>(t, mir, mnodes, LV, key, leaf, gl, gbase);
        uint32_t c = 0;
        bool done = !live || empty || mx == 0 || key[0] > h;
        uint32_t cur = leaf[0];
        while (!done) {
            typename T::KV kv = T::load_keys(t.lkeys + static_cast<uint64_t>(cur) * kSlots, gl);
            typename T::KV vv = T::load_keys(t.lvals + static_cast<uint64_t>(cur) * kSlots, gl);
            const uint2 meta = t.lmeta[cur];
            bool ok[KPL];
            uint32_t within = 0, lanes_below = 0, total = 0;
            bool beyond = false;
            uint32_t pre[KPL];
#pragma unroll
            for (int e = 0; e < KPL; ++e) {
                const uint32_t slot = static_cast<uint32_t>(gl * KPL + e);
                const bool inl = slot < meta.x;
                ok[e] = inl && kv.v[e] >= key[0] && kv.v[e] <= h;
                const uint64_t bits = group_bits<G>(__ballot(ok[e]), gbase);
                const uint64_t over = group_bits<G>(__ballot(inl && kv.v[e] > h), gbase);
                beyond = beyond || over != 0;
                lanes_below += static_cast<uint32_t>(__popcll(bits & below_lanes));
                total += static_cast<uint32_t>(__popcll(bits));
                pre[e] = within;
                within += ok[e] ? 1u : 0u;
            }
#pragma unroll
            for (int e = 0; e < KPL; ++e) {
                if (ok[e]) {
                    const uint32_t p = c + lanes_below + pre[e];
                    if (p < mx) {
                        okeys[base + p] = kv.v[e];
                        ovals[base + p] = vv.v[e];
                    }
                }
            }
            c += total;
            done = c >= mx || beyond || meta.y == kNone || meta.x == 0;
            cur = meta.y;
        }
        if (live && gl == 0) cnt_out[qi] = c < mx ? c : mx;
    }
}

// ---------------------------------------------------------------- launch

static uint32_t lds_bytes_for(int lv, int key_bytes) {
    if (lv <= 0) return 0;
    uint32_t n = mirror_nodes_for_levels(lv);
    return key_bytes == 8 ? MirrorLayout<uint64_t>::bytes(n) : MirrorLayout<uint32_t>::bytes(n);
}

static uint64_t grid_for(uint64_t ntiles, int lv, int key_bytes) {
    // resident workgroups: 8 per CU when the mirror copy is small, fewer
    // when it takes a large share of the 160 KiB of LDS per CU
    uint32_t lds = lds_bytes_for(lv, key_bytes);
    uint64_t per_cu = 8;
    if (lds > 0) {
        uint64_t fit = (160u * 1024u) / lds;
        if (fit < per_cu) per_cu = fit < 1 ? 1 : fit;
    }
    uint64_t cap = 256 * per_cu;
    return ntiles < cap ? (ntiles < 1 ? 1 : ntiles) : cap;
}

template <class K, int G, int QPG, int LV, bool VC, int NT>
static void launch_lookup_t(const TreeView<K>& t, const K* q, uint64_t B, K* vout, uint8_t* fout, hipStream_t s) {
    const uint64_t tile_q = static_cast<uint64_t>(kLookupBlock / G) * QPG;
    const uint64_t ntiles = (B + tile_q - 1) / tile_q;
    const uint64_t grid = grid_for(ntiles, LV, sizeof(K));
    hipLaunchKernelGGL((k_lookup<K, G, QPG, LV, VC, NT>), dim3(static_cast<uint32_t>(grid)), dim3(kLookupBlock),
                       lds_bytes_for(LV, sizeof(K)), s, t, q, B, vout, fout, ntiles);
}

template <class K, bool VC, int NT>
static void launch_lookup_xcd(const TreeView<K>& t, const K* q, uint64_t B, K* vout, uint8_t* fout, hipStream_t s) {
    const uint64_t nchunks = (B + 63) / 64;
    // per XCD up to 256 workgroups (8 per CU) of four waves; every XCD reads
    // every chunk, four at a time per wave
    uint64_t per_xcd = (nchunks + 4 * kXcdChunks - 1) / (4 * kXcdChunks);
    if (per_xcd > 256) per_xcd = 256;
    if (per_xcd < 1) per_xcd = 1;
    hipLaunchKernelGGL((k_lookup_xcd<K, VC, NT>), dim3(static_cast<uint32_t>(per_xcd * kXcds)), dim3(kLookupBlock),
                       lds_bytes_for(2, sizeof(K)), s, t, q, B, vout, fout, nchunks);
}

constexpr uint64_t kPassBatch = 1u << 16;   // one pass of the grid at one query per group
constexpr uint64_t kStageBatch = 1u << 17;  // from here on the top levels are staged in LDS

// Values are streamed past the caches in large batches over trees loaded with
// leaf lines that outgrow the 256 MB memory-side cache: there few lines are
// read again before they are evicted.  2^20 uniform keys of 2^24 u64 keys (256
// MB of leaf lines) 63.6 us against 64.4 with plain loads, loaded at fill 0.75
// 72.0 and 74.4; below that size the lines are found again, 2^20 keys after
// 2^20 inserts 72.9 us streamed and 60.6 not.  Skewed queries find them at any
// size (Zipf(0.99) ones of 2^24 keys 57.2 us, 43.5 with plain loads): a program
// that makes them turns streaming off.
constexpr uint64_t kStreamLeafBytes = 256ull << 20;

template <class K, int G, int QPG, int LV>
static void launch_lookup_v(const TreeView<K>& t, const LaunchCfg& cfg, const K* q, uint64_t B, K* vout,
                            uint8_t* fout, hipStream_t s) {
    const bool xcd = cfg.xcd_split == 2 || (cfg.xcd_split == 1 && B >= kXcdMinBatch);
    // leaf lines read non-temporally: both (leaf_stream 1), none (2), or by
    // default the values, by the rule above
    const bool big = 2 * cfg.loaded_leaves * kSlots * sizeof(K) >= kStreamLeafBytes;
    const int nt = cfg.leaf_stream == 1 ? 3 : (cfg.leaf_stream == 0 && big && B > kPassBatch ? 2 : 0);
    if (xcd) {
        if (cfg.value_coload) {
            if (nt == 3) launch_lookup_xcd<K, true, 3>(t, q, B, vout, fout, s);
            else if (nt == 2) launch_lookup_xcd<K, true, 2>(t, q, B, vout, fout, s);
            else launch_lookup_xcd<K, true, 0>(t, q, B, vout, fout, s);
        } else {
            if (nt == 3) launch_lookup_xcd<K, false, 3>(t, q, B, vout, fout, s);
            else if (nt == 2) launch_lookup_xcd<K, false, 2>(t, q, B, vout, fout, s);
            else launch_lookup_xcd<K, false, 0>(t, q, B, vout, fout, s);
        }
        return;
    }
    if (cfg.value_coload) {
        if (nt == 3) launch_lookup_t<K, G, QPG, LV, true, 3>(t, q, B, vout, fout, s);
        else if (nt == 2) launch_lookup_t<K, G, QPG, LV, true, 2>(t, q, B, vout, fout, s);
        else launch_lookup_t<K, G, QPG, LV, true, 0>(t, q, B, vout, fout, s);
    } else {
        if (nt == 3) launch_lookup_t<K, G, QPG, LV, false, 3>(t, q, B, vout, fout, s);
        else if (nt == 2) launch_lookup_t<K, G, QPG, LV, false, 2>(t, q, B, vout, fout, s);
        else launch_lookup_t<K, G, QPG, LV, false, 0>(t, q, B, vout, fout, s);
    }
}

template <class K, int G, int QPG>
static void launch_lookup_lv(const TreeView<K>& t, const LaunchCfg& cfg, const K* q, uint64_t B, K* vout,
                             uint8_t* fout, hipStream_t s) {
    switch (cfg.lds_levels) {
        case 0: launch_lookup_v<K, G, QPG, 0>(t, cfg, q, B, vout, fout, s); break;
        case 1: launch_lookup_v<K, G, QPG, 1>(t, cfg, q, B, vout, fout, s); break;
        case 2: launch_lookup_v<K, G, QPG, 2>(t, cfg, q, B, vout, fout, s); break;
        default: launch_lookup_v<K, G, QPG, 3>(t, cfg, q, B, vout, fout, s); break;
    }
}

// Lookup shape by batch size, for the fields the caller did not fix.  The
// 2048 resident workgroups hold 2^16 queries at 8 lanes each.
//  - Below kMidBatch a batch is one latency chain: 16 lanes per query, no LDS
//    staging (the top levels are L2 hits, the staging a barrier on the
//    critical path), the value line read with the key line.
//  - Up to kPassBatch one query per group is one pass of the grid: 65536
//    queries of 2^24 u64 keys 5.4 us, 5.8 with two per group, 6.5 with the
//    top levels staged as well.
//  - Above it a batch is bound by the lines it reads: two queries in flight
//    per group (one is too few to hide the misses; four cost more in
//    registers than they add), and one value read after the match instead of
//    the whole line before it, which an absent key does not read at all: 2^20
//    queries of 2^23 u64 keys, half absent, 47.9 us against 59.2; 2^20
//    present ones of 2^18 u64 keys 33.6 against 36.9.  Also on a tree that
//    took updates, whose searches read child lines too: 2^20 present keys of
//    2^24 after 2^20 inserts 96.9 us, 96.6 with the whole line, half absent
//    88.4 and 96.8, Zipf half absent 65.2 and 85.1; loaded at fill 0.75 72.0
//    and 72.4, 63.1 and 72.3, 47.5 and 53.5.
//  - From kStageBatch on the grid walks its tiles more than once and staging
//    the top two levels is shared: 2^20 queries of 2^22 u64 keys 52.5 us
//    against 53.7; 98304 queries 7.5 against 7.4, of 2^21 keys 6.9 against 6.6.
static LaunchCfg shape_for(const LaunchCfg& cfg, uint64_t B) {
    LaunchCfg c = cfg;
    if (cfg.shape_auto & 1) c.lanes = B < kMidBatch ? 16 : 8;
    if (cfg.shape_auto & 2) c.queries_per_group = B <= kPassBatch ? 1 : 2;
    if (cfg.shape_auto & 4) c.lds_levels = B < kStageBatch ? 0 : 2;
    if (cfg.value_coload == 2) c.value_coload = B <= kPassBatch ? 1 : 0;
    return c;
}

template <class K>
void launch_lookup(const TreeView<K>& t, const LaunchCfg& cfg0, const K* q, uint64_t B, K* vout, uint8_t* fout,
                   hipStream_t s) {
    const LaunchCfg cfg = shape_for(cfg0, B);
    const int qpg = cfg.queries_per_group;
    switch (cfg.lanes) {
        case 4:
            if (qpg >= 4) launch_lookup_lv<K, 4, 4>(t, cfg, q, B, vout, fout, s);
            else if (qpg == 2) launch_lookup_lv<K, 4, 2>(t, cfg, q, B, vout, fout, s);
            else launch_lookup_lv<K, 4, 1>(t, cfg, q, B, vout, fout, s);
            break;
        case 16:
            if (qpg >= 4) launch_lookup_lv<K, 16, 4>(t, cfg, q, B, vout, fout, s);
            else if (qpg == 2) launch_lookup_lv<K, 16, 2>(t, cfg, q, B, vout, fout, s);
            else launch_lookup_lv<K, 16, 1>(t, cfg, q, B, vout, fout, s);
            break;
        default:
            if (qpg >= 4) launch_lookup_lv<K, 8, 4>(t, cfg, q, B, vout, fout, s);
            else if (qpg == 2) launch_lookup_lv<K, 8, 2>(t, cfg, q, B, vout, fout, s);
            else launch_lookup_lv<K, 8, 1>(t, cfg, q, B, vout, fout, s);
            break;
    }
}

template <class K, int AH, int LV>
static void launch_range_t(const TreeView<K>& t, const K* lo, const K* hi, const uint32_t* mx, const uint64_t* off,
                           uint64_t B, K* ok, K* ov, uint32_t* cnt, hipStream_t s) {
    const uint64_t tile_q = kLookupBlock / (kSlots * AH);
    const uint64_t ntiles = (B + tile_q - 1) / tile_q;
    const uint64_t grid = grid_for(ntiles, LV, sizeof(K));
    hipLaunchKernelGGL((k_range<K, AH, LV>), dim3(static_cast<uint32_t>(grid)), dim3(kLookupBlock),
                       lds_bytes_for(LV, sizeof(K)), s, t, lo, hi, mx, off, B, ok, ov, cnt, ntiles);
}

template <class K, int LV>
static void launch_range_many_t(const TreeView<K>& t, const K* lo, const K* hi, const uint32_t* mx,
                                const uint64_t* off, uint64_t B, K* ok, K* ov, uint32_t* cnt, hipStream_t s) {
    const uint64_t tile_q = kLookupBlock / 8;
    const uint64_t ntiles = (B + tile_q - 1) / tile_q;
    const uint64_t grid = grid_for(ntiles, LV, sizeof(K));
    hipLaunchKernelGGL((k_range_many<K, LV>), dim3(static_cast<uint32_t>(grid)), dim3(kLookupBlock),
                       lds_bytes_for(LV, sizeof(K)), s, t, lo, hi, mx, off, B, ok, ov, cnt, ntiles);
}

// Leaves read at once by batch size.  The chip holds 2^13 scans of four
// leaves, 2^14 of two and 2^15 of one; what it has no idle lanes for is only
// more to read: 1024 scans take four (see k_range), 4096 two (1 to 100 pairs
// 5.4 us, four 5.1; 1 pair 3.95, four 4.4, the old 3.9), 8192 one (7.7 us,
// the old 8.2; on a grown tree 9.8 and 11.0).  Above kRangeMany scans 8 lanes
// per scan read as much at once and descend in half as many waves.  64-bit
// keys, 16 lanes and 8: 10000 scans of 1 to 10 pairs 4.52 and 4.58 us, 16384
// 5.05 and 4.86 (1 to 100 pairs 12.2 both).  32-bit keys, whose lines are half
// as long: 20000 scans 4.85 and 4.99 us, 32768 6.45 and 6.17, 131072 of 2^18
// keys 15.3 and 12.3 (1 to 100 pairs 11.2 and 12.3, 13.6 and 15.4, 33 and 37:
// long scans would rather keep 16 lanes, but the call does not know them).
constexpr uint64_t kRangeFour = 1u << 11, kRangeTwo = 1u << 12;
template <class K>
constexpr uint64_t kRangeMany = sizeof(K) == 8 ? 12288 : 24576;

template <class K, int LV>
static void launch_range_lv(const TreeView<K>& t, const K* lo, const K* hi, const uint32_t* mx, const uint64_t* off,
                            uint64_t B, K* ok, K* ov, uint32_t* cnt, hipStream_t s) {
    if (B <= kRangeFour) {
        launch_range_t<K, 4, LV>(t, lo, hi, mx, off, B, ok, ov, cnt, s);
    } else if (B <= kRangeTwo) {
        launch_range_t<K, 2, LV>(t, lo, hi, mx, off, B, ok, ov, cnt, s);
    } else if (B <= kRangeMany<K>) {
        launch_range_t<K, 1, LV>(t, lo, hi, mx, off, B, ok, ov, cnt, s);
    } else {
        launch_range_many_t<K, LV>(t, lo, hi, mx, off, B, ok, ov, cnt, s);
    }
}

template <class K>
void launch_range(const TreeView<K>& t, const LaunchCfg& cfg, const K* lo, const K* hi, const uint32_t* mx,
                  const uint64_t* off, uint64_t B, K* ok, K* ov, uint32_t* cnt, hipStream_t s) {
    switch (cfg.lds_levels) {
        case 0: launch_range_lv<K, 0>(t, lo, hi, mx, off, B, ok, ov, cnt, s); break;
        case 1: launch_range_lv<K, 1>(t, lo, hi, mx, off, B, ok, ov, cnt, s); break;
        case 2: launch_range_lv<K, 2>(t, lo, hi, mx, off, B, ok, ov, cnt, s); break;
        default: launch_range_lv<K, 3>(t, lo, hi, mx, off, B, ok, ov, cnt, s); break;
    }
}

template void launch_lookup<uint32_t>(const TreeView<uint32_t>&, const LaunchCfg&, const uint32_t*, uint64_t,
                                      uint32_t*, uint8_t*, hipStream_t);
template void launch_lookup<uint64_t>(const TreeView<uint64_t>&, const LaunchCfg&, const uint64_t*, uint64_t,
                                      uint64_t*, uint8_t*, hipStream_t);
template void launch_range<uint32_t>(const TreeView<uint32_t>&, const LaunchCfg&, const uint32_t*,
                                     const uint32_t*, const uint32_t*, const uint64_t*, uint64_t, uint32_t*,
                                     uint32_t*, uint32_t*, hipStream_t);
template void launch_range<uint64_t>(const TreeView<uint64_t>&, const LaunchCfg&, const uint64_t*,
                                     const uint64_t*, const uint32_t*, const uint64_t*, uint64_t, uint64_t*,
                                     uint64_t*, uint32_t*, hipStream_t);

}  // namespace gt
