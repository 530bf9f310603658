// Sample sort of (key, payload) pairs: the library's sort above 8192 keys (up to
// there keys are ranked by counting), of bulk loads straight into leaves.
//
// A pass of radix sort moves every pair once per eight key bits (eight
// passes for 64-bit keys).  A sample sort moves a pair twice however wide
// the key is (three times above 2^20 pairs): a sorted sample of the input
// gives G - 1 splitters, every pair is scattered to its group, and each
// group, small enough for one workgroup's LDS, is sorted there.  The groups
// stay balanced whatever the key distribution, also with repeated keys,
// because the splitters are sample pairs (key, position) and all pairs
// differ.  (Frazer and McKellar, "Samplesort: a sampling approach to minimal
// storage tree sorting", J. ACM 17(3), 1970.)
//
//   sample   8 or 16 G pairs at stratified positions, ranked by counting over
//            many workgroups up to 1024 pairs, above merge-sorted in LDS (runs
//            of 512 and a rank kernel); every eighth or sixteenth is a splitter
//   count    each tile classifies its keys by a search of the splitters in
//            LDS and adds its group counts to the global ones
//   scatter  tiles rank their pairs by group in LDS, reserve room in each
//            group with one atomic per tile and group, and write each
//            group's pairs contiguously; the order inside a group is not
//            kept (the group sort compares (key, position))
//   groups   one workgroup per group: keys are dealt to as many LDS bins as
//            the group has pairs by their distance from the group's smallest
//            key, and a pair's rank is its bin's start plus the smaller
//            pairs of its bin (large bins are dealt again first, by their
//            own keys or, of one key, by position); a group whose bins stay
//            too uneven is merge-sorted in LDS, one too large for the LDS (not expected:
//            four times the mean) by a bitonic network in device memory
//
// Above 2^20 pairs a first scatter into 256 segments comes before, and the
// steps above run per segment.
//
// Measured on 2^20 (64-bit key, position) pairs, us: sample 11 and rank 11
// (latency of a few workgroups), count 15, scatter 21, groups 17 and 5; 2^24
// (key, value) pairs of a bulk load: two counts of 39, two scatters of 140
// (512 MiB moved, 3.8 TB/s where a copy reaches 5.1), groups into leaves 193
// (512 MiB, 2.8 TB/s; about 300 vector instructions per 64 pairs are its other
// bound).
//
// No step waits on another workgroup.  A scatter that finds more pairs for a
// group than were counted (the input changed, which no caller may do) writes
// only inside the group and marks the sort failed; the result is then replaced
// by a valid sorted one, every key 0 and index i at position i.  That keeps
// such a sort's writes in bounds where it is noticed; it is no promise.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>
#include <chrono>
#include <type_traits>
#include "common.h"
#include "kernels.h"
#include "prims.h"

namespace gt {

constexpr int kSsThreads = 512;
constexpr uint32_t kSsMaxGroups = 512;                   // groups of one scatter
constexpr uint32_t kSsMaxSample = 4096;                  // sample pairs one workgroup sorts
constexpr uint32_t kSsRun = 512;                         // sample pairs of a run, where several are merged
constexpr uint32_t kSsMaxRuns = 16;
constexpr uint32_t kSsSegments = 256;                    // segments of the first scatter above kSsOneLevel
constexpr uint64_t kSsOneLevel = 1ull << 20;
constexpr uint64_t kSsMax = 1ull << 26;                  // largest input (256 segments of 256 groups)
constexpr uint64_t kSsSmallMean = 512;
constexpr uint32_t kSsRankSample = 1024;                 // largest sample ranked by counting
constexpr uint32_t kSsRankStep = 128;                    // sample pairs a step of k_ss_sample_rank compares

// What one level sorts by: `segs` segments of the input (one for the first
// level), cut into `groups` groups each.
struct SsLevel {
    uint32_t segs, groups, over, runs;  // over: sample pairs per group; runs: of the sample, merged by k_ss_rank
    uint64_t o_sk, o_sp;    // the sample's runs (keys, positions)
    uint64_t o_gk, o_gp;    // splitters: groups - 1 per segment (stride groups)
    uint64_t o_cnt, o_cur;  // group counts and write cursors
    uint64_t o_start;       // group starts, groups + 1 per segment
};

struct SsPlan {
    int levels;
    SsLevel lv[2];
    uint64_t o_fail;
    uint64_t o_list;        // groups too large for the small group sort: count, then the groups
    uint64_t bytes;
};

// The steps' sizes for n pairs (n <= kSsMax) and their places in the
// caller's scratch.
static SsPlan ss_plan(uint64_t n, int key_bytes) {
    SsPlan p{};
    auto al = [](uint64_t x) { return (x + 255) / 256 * 256; };
    auto pow2 = [](uint64_t x) {
        uint32_t r = 1;
        while (r < x) r <<= 1;
        return r;
    };
    uint64_t o = 0;
    p.o_fail = o;
    o += 256;
    auto place = [&](SsLevel& l, uint32_t segs, uint32_t groups, uint32_t over) {
        l.segs = segs;
        l.groups = groups;
        l.over = over;
        const uint64_t S = static_cast<uint64_t>(groups) * over, ng = static_cast<uint64_t>(segs) * groups;
        l.runs = segs == 1 && S > 1024 ? static_cast<uint32_t>(S / kSsRun) : 1u;
        l.o_sk = o;    o += l.runs > 1 ? al(S * key_bytes) : 0;
        l.o_sp = o;    o += l.runs > 1 ? al(S * 4) : 0;
        l.o_gk = o;    o += al(ng * key_bytes);
        l.o_gp = o;    o += al(ng * 4);
        l.o_cnt = o;   o += al(ng * 4);
        l.o_cur = o;   o += al(ng * 4);
        l.o_start = o; o += al((ng + segs) * 4);
    };
    if (n <= kSsOneLevel) {
        // up to 2^16 pairs many small groups (a mean of 512 at most), so that
        // the group sort has work for most CUs; above, 512 groups
        uint32_t g = pow2((n + 511) / 512);
        g = g < 8 ? 8 : (g <= 128 ? g : kSsMaxGroups);
        p.levels = 1;
        place(p.lv[0], 1, g, n > kSsSmallMean * kSsMaxGroups ? 16 : 8);
    } else {
        p.levels = 2;
        place(p.lv[0], 1, kSsSegments, 16);
        const uint32_t g = pow2((n / kSsSegments + 1023) / 1024);
        place(p.lv[1], kSsSegments, g < 8 ? 8 : g, 16);
    }
    p.o_list = o;
    o += al((static_cast<uint64_t>(p.lv[p.levels - 1].segs) * p.lv[p.levels - 1].groups + 1) * 4);
    p.bytes = o;
    return p;
}

// (ka, pa) before (kb, pb); without TIE by key alone
template <bool TIE, class K>
__device__ __forceinline__ bool ss_less(K ka, uint32_t pa, K kb, uint32_t pb) {
    if constexpr (TIE) return ka < kb || (ka == kb && pa < pb);
    else return ka < kb;
}

// a 32-bit mixer (the lowbias32 constants of Chris Wellons' hash prospector)
__device__ __forceinline__ uint32_t ss_hash(uint32_t x) {
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    return x ^ (x >> 16);
}

// Whether the sort is refused already (a repeated key, a failure): what the
// kernels before this one left is then not read.  The same for the whole
// workgroup, though the word may be raised meanwhile.  Only without TIE.
template <bool TIE>
__device__ __forceinline__ bool ss_refused(const uint32_t* refuse) {
    if constexpr (TIE) {
        return false;
    } else {
        __shared__ uint32_t word;
        if (threadIdx.x == 0) word = __hip_atomic_load(refuse, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        return word != 0;
    }
}

// position of sample i of S in a segment of m pairs: one per stratum.  Every
// sort takes another seed, so that no input keeps its sample from telling the
// groups apart (positions that were a fixed hash of i and m let 2^18 keys fall
// into one group, 29 ms for 76 us).
__device__ __forceinline__ uint32_t ss_sample_at(uint32_t i, uint32_t S, uint32_t m, uint32_t seed) {
    const uint64_t a = static_cast<uint64_t>(i) * m / S, b = static_cast<uint64_t>(i + 1) * m / S;
    const uint32_t w = b > a ? static_cast<uint32_t>(b - a) : 1u;
    return static_cast<uint32_t>(a) + ss_hash(ss_hash(i ^ seed) + m) % w;
}

// Bitonic sort of m pairs (any m) by (key, tie): every comparator puts the
// smaller pair at the lower index (the first step of a merge compares
// mirrored indexes), so the missing pairs behind m count as larger than all
// and their comparators are left out.  The whole workgroup; `a` and `b` may
// be LDS or device memory of this workgroup alone.
template <bool TIE, class K, class P>
__device__ void ss_bitonic(K* a, P* b, uint32_t m) {
    uint32_t n2 = 2;
    while (n2 < m) n2 <<= 1;
    for (uint32_t k = 2; k <= n2; k <<= 1) {
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            for (uint32_t q = threadIdx.x; q < n2 / 2; q += blockDim.x) {
                const uint32_t lo = ((q & ~(j - 1)) << 1) | (q & (j - 1));
                const uint32_t hi = j == (k >> 1) ? (lo ^ (k - 1)) : (lo | j);
                if (hi < m) {
                    const K x = a[lo], y = a[hi];
                    const P u = b[lo], w = b[hi];
                    if (ss_less<TIE>(y, static_cast<uint32_t>(w), x, static_cast<uint32_t>(u))) {
                        a[lo] = y; a[hi] = x;
                        b[lo] = w; b[hi] = u;
                    }
                }
            }
            __syncthreads();
        }
    }
}

// Segment `s` of a level: its range of the input (the first level has one,
// the whole input; the second level's are the first level's groups).
__device__ __forceinline__ void ss_segment(const uint32_t* __restrict__ seg_start, uint32_t s, uint32_t n,
                                           uint32_t& b, uint32_t& m) {
    if (seg_start) {
        b = seg_start[s];
        m = seg_start[s + 1] - b;
    } else {
        b = 0;
        m = n;
    }
}

// Merge sort of m pairs (a power of two) by (key, position), by the whole
// workgroup, each thread moving N of them: a round merges neighbouring runs of
// `len` pairs, every pair finding its place by a binary search of the other
// run.  Two buffers in LDS; returns the one the result is in.  (1024 pairs
// took 20 us by a bitonic network, whose 55 rounds each wait for a barrier;
// here 10 rounds of at most 10 dependent LDS reads.)
// An index's place in the buffers: the searches' power-of-two strides would
// otherwise share a bank.
__device__ __forceinline__ uint32_t ss_pad(uint32_t i) { return i + (i >> 5); }
constexpr uint32_t kSsPadded = kSsMaxSample + kSsMaxSample / 32;

template <int N, class K>
__device__ __forceinline__ int ss_merge_sort(K (*a)[kSsPadded], uint32_t (*p)[kSsPadded], uint32_t m) {
    int cur = 0;
    for (uint32_t len = 1; len < m; len <<= 1) {
        K k[N];
        uint32_t q[N], at[N], c[N];
        bool right[N];  // in the right run: pairs equal to it go before it
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const uint32_t i = threadIdx.x + e * blockDim.x;
            const uint32_t x = i < m ? i : 0u;
            k[e] = a[cur][ss_pad(x)];
            q[e] = p[cur][ss_pad(x)];
            right[e] = (x & len) != 0;
            at[e] = (x & ~(2u * len - 1u)) + (right[e] ? 0u : len);  // the other run
            c[e] = 0;
        }
        // pairs of the other run before this one (a sample of a segment
        // smaller than it holds a pair more than once)
        auto before = [&](uint32_t y, int e) {
            const K ky = a[cur][ss_pad(y)];
            if (ky != k[e]) return ky < k[e];
            const uint32_t qy = p[cur][ss_pad(y)];
            return qy < q[e] || (qy == q[e] && right[e]);
        };
        for (uint32_t st = len >> 1; st > 0; st >>= 1) {
#pragma unroll
            for (int e = 0; e < N; ++e) c[e] += before(at[e] + c[e] + st - 1, e) ? st : 0u;
        }
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const uint32_t i = threadIdx.x + e * blockDim.x;
            const bool lt = before(at[e] + c[e], e);
            c[e] += lt ? 1u : 0u;
            if (i < m) {
                const uint32_t to = (i & ~(2u * len - 1u)) + (i & (len - 1u)) + c[e];
                a[cur ^ 1][ss_pad(to)] = k[e];
                p[cur ^ 1][ss_pad(to)] = q[e];
            }
        }
        cur ^= 1;
        __syncthreads();
    }
    return cur;
}

// Sample of segment blockIdx.x (groups * over pairs), run blockIdx.y of
// `runs`.  One run: every `over`-th pair is a splitter; several: the sorted
// runs go to sk, sp for k_ss_rank.  Also clears the level's counters and, on
// the first level, the failure word (`force` is the testing hook that makes
// the sort fail).  Without TIE, equal keys at different positions set bit 0
// of *dup, and the kernels after this one end at once.
template <class K, bool TIE>
__global__ __launch_bounds__(1024) void k_ss_sample(const K* __restrict__ kin, const uint32_t* __restrict__ pin,
                                                     uint32_t n, const uint32_t* __restrict__ seg_start,
                                                     uint32_t groups, uint32_t over, uint32_t runs, uint32_t seed, K* gk,
                                                     uint32_t* gp, K* sk, uint32_t* sp, uint32_t* cnt, uint32_t* cur,
                                                     uint32_t* list, uint32_t* fail, uint32_t force, uint32_t* err,
                                                     uint32_t err_bit, uint32_t* dup) {
    __shared__ K a[2][kSsPadded];
    __shared__ uint32_t p[2][kSsPadded];
    const uint32_t s = blockIdx.x, tid = threadIdx.x, S = groups * over, len = S / runs, first = blockIdx.y * len;
    if (seg_start && ss_refused<TIE>(dup)) return;  // the segments were not written
    if (blockIdx.y == 0)
        for (uint32_t i = tid; i < groups; i += blockDim.x) {
            cnt[static_cast<uint64_t>(s) * groups + i] = 0;
            cur[static_cast<uint64_t>(s) * groups + i] = 0;
        }
    if (s == 0 && blockIdx.y == 0 && tid == 0) {
        list[0] = 0;
        if (!seg_start) {  // the first level
            *fail = force;
            if (force && err) atomicOr(err, err_bit);
        }
    }
    uint32_t b, m;
    ss_segment(seg_start, s, n, b, m);
    for (uint32_t i = tid; i < len; i += blockDim.x) {
        K k = kmax<K>();
        uint32_t q = 0xFFFFFFFFu;
        if (m) {
            const uint32_t at = b + ss_sample_at(first + i, S, m, seed);
            k = kin[at];
            q = pin ? pin[at] : at;
        }
        a[0][ss_pad(i)] = k;
        p[0][ss_pad(i)] = q;
    }
    __syncthreads();
    const int w = len <= blockDim.x ? ss_merge_sort<1>(a, p, len) : ss_merge_sort<4>(a, p, len);
    if (runs > 1) {
        for (uint32_t i = tid; i < len; i += blockDim.x) {
            sk[first + i] = a[w][ss_pad(i)];
            sp[first + i] = p[w][ss_pad(i)];
        }
        return;
    }
    for (uint32_t g = tid; g + 1 < groups; g += blockDim.x) {
        gk[static_cast<uint64_t>(s) * groups + g] = a[w][ss_pad(g * over + over - 1)];
        gp[static_cast<uint64_t>(s) * groups + g] = p[w][ss_pad(g * over + over - 1)];
    }
    if (!TIE && dup)
        for (uint32_t i = tid; i + 1 < len; i += blockDim.x)
            if (m && a[w][ss_pad(i)] == a[w][ss_pad(i + 1)] && p[w][ss_pad(i)] != p[w][ss_pad(i + 1)])
                atomicOr(dup, 1u);
}

// Sample of the first level by counting: every workgroup holds all S sampled
// pairs and ranks a few of them, 16 lanes a pair; a pair whose rank is the
// last of `over` is a splitter.  S^2 comparisons over S / 16 groups of lanes
// are one short chain where sorting the sample in one workgroup is ten rounds
// of dependent LDS reads: for the 1024 pairs of 50000 keys 6 us, 11.6 by
// merging.  Up to kSsRankSample pairs; 4096 take 20 us longer than their runs
// sorted by eight workgroups and ranked by search (the level-wise lookup of
// 65537 keys 52.0 us, so 72.3).  Clears what k_ss_sample clears.
constexpr int kSsRankThreads = 256;

template <class K, bool TIE>
__global__ __launch_bounds__(kSsRankThreads) void k_ss_sample_rank(
    const K* __restrict__ kin, const uint32_t* __restrict__ pin, uint32_t n, uint32_t groups, uint32_t over,
    uint32_t seed, K* gk, uint32_t* gp, uint32_t* cnt, uint32_t* cur, uint32_t* list, uint32_t* fail, uint32_t force, uint32_t* err,
    uint32_t err_bit, uint32_t* dup) {
    constexpr uint32_t G = 16, R = kSsRankStep / G;
    __shared__ K a[kSsRankSample];
    __shared__ uint32_t p[kSsRankSample];
    const uint32_t tid = threadIdx.x, S = groups * over;  // S a multiple of kSsRankStep
    if (blockIdx.x == 0) {
        for (uint32_t i = tid; i < groups; i += kSsRankThreads) {
            cnt[i] = 0;
            cur[i] = 0;
        }
        if (tid == 0) {
            list[0] = 0;
            *fail = force;
            if (force && err) atomicOr(err, err_bit);
        }
    }
    for (uint32_t i = tid; i < S; i += kSsRankThreads) {
        const uint32_t at = ss_sample_at(i, S, n, seed);
        a[i] = kin[at];
        p[i] = pin ? pin[at] : at;
    }
    __syncthreads();
    const uint32_t e = (blockIdx.x * kSsRankThreads + tid) / G, l = tid % G;
    if (e >= S) return;  // whole groups of lanes leave together
    const K ke = a[e];
    uint32_t c = 0;  // smaller keys, and in the upper half smaller or equal ones
    for (uint32_t j = l; j < S; j += G * R) {
        K kj[R];
#pragma unroll
        for (uint32_t u = 0; u < R; ++u) kj[u] = a[j + G * u];
#pragma unroll
        for (uint32_t u = 0; u < R; ++u) {
            c += kj[u] < ke ? 1u : 0u;
            c += kj[u] <= ke ? 0x10000u : 0u;
        }
    }
#pragma unroll
    for (uint32_t m = 1; m < G; m <<= 1) c += __shfl_xor(c, static_cast<int>(m), 64);
    uint32_t rank = c & 0xFFFFu;
    if ((c >> 16) - rank > 1u) {  // equal keys, by position, then by sample (a pair sampled twice)
        const uint32_t pe = p[e];
        uint32_t before = 0, other = 0;
        for (uint32_t j = l; j < S; j += G)
            if (a[j] == ke) {
                before += p[j] < pe || (p[j] == pe && j < e) ? 1u : 0u;
                other |= p[j] != pe ? 1u : 0u;
            }
#pragma unroll
        for (uint32_t m = 1; m < G; m <<= 1) before += __shfl_xor(before, static_cast<int>(m), 64);
        rank += before;
        if (!TIE && dup && other) atomicOr(dup, 1u);
    }
    if (l == 0 && rank % over == over - 1 && rank / over + 1 < groups) {
        gk[rank / over] = ke;
        gp[rank / over] = p[e];
    }
}

// Rank of every pair of the sorted sample runs among all of them (one search
// per run, all in flight together); every `over`-th becomes a splitter.  A
// thread per pair, the runs in LDS.
template <class K, bool TIE, int RUNS>
__global__ __launch_bounds__(256) void k_ss_rank(const K* __restrict__ sk, const uint32_t* __restrict__ sp,
                                                 uint32_t over, K* gk, uint32_t* gp, uint32_t* dup) {
    constexpr uint32_t S = RUNS * kSsRun;
    __shared__ K a[S + S / 32];
    __shared__ uint32_t p[S + S / 32];
    // 16 bytes a load, all of them in flight
    constexpr uint32_t PK = 16 / sizeof(K), LK = S / PK / 256, LP = S / 4 / 256;
    VecN<K, PK> vk[LK];
    VecN<uint32_t, 4> vp[LP];
#pragma unroll
    for (uint32_t j = 0; j < LK; ++j) vk[j] = reinterpret_cast<const VecN<K, PK>*>(sk)[j * 256 + threadIdx.x];
#pragma unroll
    for (uint32_t j = 0; j < LP; ++j) vp[j] = reinterpret_cast<const VecN<uint32_t, 4>*>(sp)[j * 256 + threadIdx.x];
#pragma unroll
    for (uint32_t j = 0; j < LK; ++j)
#pragma unroll
        for (uint32_t u = 0; u < PK; ++u) a[ss_pad((j * 256 + threadIdx.x) * PK + u)] = vk[j].v[u];
#pragma unroll
    for (uint32_t j = 0; j < LP; ++j)
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) p[ss_pad((j * 256 + threadIdx.x) * 4 + u)] = vp[j].v[u];
    __syncthreads();
    const uint32_t i = blockIdx.x * 256 + threadIdx.x, mine = i / kSsRun;
    const K k = a[ss_pad(i)];
    const uint32_t q = p[ss_pad(i)];
    // (no branch on equal keys: the searches' reads would wait for each other)
    auto before = [&](uint32_t y) {
        const K ky = a[ss_pad(y)];
        const uint32_t qy = p[ss_pad(y)];
        return static_cast<uint32_t>(ky < k) | (static_cast<uint32_t>(ky == k) & static_cast<uint32_t>(qy < q));
    };
    // pairs of each run below (k, q); the own run finds the pair's own index
    uint32_t c[RUNS];
#pragma unroll
    for (int r = 0; r < RUNS; ++r) c[r] = 0;
#pragma unroll 1
    for (uint32_t st = kSsRun / 2; st > 0; st >>= 1) {
#pragma unroll
        for (int r = 0; r < RUNS; ++r) c[r] += before(r * kSsRun + c[r] + st - 1) * st;
    }
    uint32_t rank = 0;
    bool twin = false;
#pragma unroll
    for (int r = 0; r < RUNS; ++r) {
        c[r] += before(r * kSsRun + c[r]);
        rank += c[r];
        if (!TIE && static_cast<uint32_t>(r) != mine && c[r] < kSsRun) twin = twin || a[ss_pad(r * kSsRun + c[r])] == k;
    }
    if (!TIE && dup) {
        twin = twin || (i % kSsRun && a[ss_pad(i - 1)] == k);
        if (twin) atomicOr(dup, 1u);
    }
    if (rank % over == over - 1 && rank + 1 < S) {
        gk[rank / over] = k;
        gp[rank / over] = q;
    }
}

// The splitters in LDS as an implicit search tree in breadth-first order
// (node 1 the root, node i's children 2i and 2i + 1): a search of a sorted
// array would read power-of-two strides, one LDS bank; in this order the
// nodes of a level are neighbours.  groups is a power of two.  (Sanders and
// Winkel, "Super Scalar Sample Sort", ESA 2004.)
template <class K>
__device__ __forceinline__ void ss_load_tree(const K* __restrict__ gk, const uint32_t* __restrict__ gp,
                                             uint32_t groups, K* tk, uint32_t* tp) {
    for (uint32_t i = 1 + threadIdx.x; i < groups; i += blockDim.x) {
        const uint32_t lev = 31u - static_cast<uint32_t>(__clz(i));
        const uint32_t at = (2u * (i - (1u << lev)) + 1u) * (groups >> (lev + 1)) - 1u;
        tk[i] = gk[at];
        tp[i] = gp[at];
    }
}

// Group of a pair: the number of splitters below it.
template <bool TIE, int N, class K>
__device__ __forceinline__ void ss_classify(const K* tk, const uint32_t* tp, uint32_t groups, const K (&k)[N],
                                            const uint32_t (&q)[N], uint32_t (&g)[N]) {
#pragma unroll
    for (int e = 0; e < N; ++e) g[e] = 1;
    for (uint32_t d = 1; d < groups; d <<= 1) {
        K x[N];
#pragma unroll
        for (int e = 0; e < N; ++e) x[e] = tk[g[e]];
#pragma unroll
        for (int e = 0; e < N; ++e) {
            bool lt = x[e] < k[e];
            if constexpr (TIE) {
                if (x[e] == k[e]) lt = tp[g[e]] < q[e];
            }
            g[e] = 2u * g[e] + (lt ? 1u : 0u);
        }
    }
#pragma unroll
    for (int e = 0; e < N; ++e) g[e] -= groups;
}

// LDS add of 1 to c[g], returning the old value; a wave whose lanes all hold
// one group (a sorted or nearly sorted input) adds once.
__device__ __forceinline__ uint32_t ss_take(uint32_t* c, uint32_t g, bool valid) {
    const uint64_t act = __ballot(valid);
    if (!act) return 0;
    const int first = __builtin_ctzll(act);
    const uint32_t g0 = shfl_u32(g, first);
    if (__ballot(valid && g == g0) == act) {
        uint32_t old = 0;
        const int lane = lane_id();
        if (lane == first) old = atomicAdd(&c[g0], static_cast<uint32_t>(__popcll(act)));
        return shfl_u32(old, first) + static_cast<uint32_t>(__popcll(act & ((1ull << lane) - 1ull)));
    }
    return valid ? atomicAdd(&c[g], 1u) : 0u;
}

// Group counts: blockIdx.x = segment (consecutive workgroups go to different
// XCDs, so with 256 segments a segment's tiles share one), blockIdx.y and on
// by gridDim.y its tiles of N pairs a thread.
template <class K, bool TIE, int N>
__global__ __launch_bounds__(kSsThreads) void k_ss_count(const K* __restrict__ kin, const uint32_t* __restrict__ pin,
                                                          uint32_t n, const uint32_t* __restrict__ seg_start,
                                                          uint32_t groups, const K* __restrict__ gk,
                                                          const uint32_t* __restrict__ gp, uint32_t* cnt,
                                                          const uint32_t* refuse) {
    constexpr uint32_t kTile = kSsThreads * N;
    if (ss_refused<TIE>(refuse)) return;
    __shared__ K tk[kSsMaxGroups];
    __shared__ uint32_t tp[kSsMaxGroups];
    __shared__ uint32_t h[kSsMaxGroups];
    const uint32_t s = blockIdx.x, tid = threadIdx.x;
    uint32_t b, m;
    ss_segment(seg_start, s, n, b, m);
    if (static_cast<uint64_t>(blockIdx.y) * kTile >= m) return;
    ss_load_tree<K>(gk + static_cast<uint64_t>(s) * groups, gp + static_cast<uint64_t>(s) * groups, groups, tk, tp);
    for (uint32_t i = tid; i < groups; i += kSsThreads) h[i] = 0;
    __syncthreads();
    for (uint64_t t0 = static_cast<uint64_t>(blockIdx.y) * kTile; t0 < m;
         t0 += static_cast<uint64_t>(gridDim.y) * kTile) {
        K k[N];
        uint32_t q[N], g[N];
        bool in[N];
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const uint64_t i = t0 + static_cast<uint32_t>(e) * kSsThreads + tid;
            in[e] = i < m;
            k[e] = in[e] ? kin[b + i] : K(0);
            if constexpr (TIE) q[e] = in[e] ? (pin ? pin[b + i] : static_cast<uint32_t>(b + i)) : 0u;
            else q[e] = 0u;
        }
        ss_classify<TIE, N>(tk, tp, groups, k, q, g);
#pragma unroll
        for (int e = 0; e < N; ++e) ss_take(h, g[e], in[e]);
    }
    __syncthreads();
    for (uint32_t i = tid; i < groups; i += kSsThreads)
        if (h[i]) atomicAdd(&cnt[static_cast<uint64_t>(s) * groups + i], h[i]);
}

// Scatter into the groups; the first workgroup of a segment also writes the
// group starts.  The payload travels with the key (a null `pin` stands for
// the position).  LDS holds one tile, reordered by group, so that a group's
// pairs leave in one run.
template <class K, class P, bool TIE, int N>
__global__ __launch_bounds__(kSsThreads) void k_ss_scatter(const K* __restrict__ kin, const P* __restrict__ pin,
                                                            uint32_t n, const uint32_t* __restrict__ seg_start,
                                                            uint32_t groups, const K* __restrict__ gk,
                                                            const uint32_t* __restrict__ gp,
                                                            const uint32_t* __restrict__ cnt, uint32_t* cur,
                                                            uint32_t* __restrict__ start, K* __restrict__ kout,
                                                            P* __restrict__ pout, uint32_t* fail, uint32_t* err,
                                                            uint32_t err_bit, const uint32_t* refuse) {
    constexpr uint32_t kTile = kSsThreads * N;
    if (ss_refused<TIE>(refuse)) return;
    __shared__ K tk[kSsMaxGroups];
    __shared__ uint32_t tp[kSsMaxGroups];
    __shared__ uint32_t h[kSsMaxGroups];       // the tile's counts
    __shared__ uint32_t ls[kSsMaxGroups];      // the tile's run of a group, in the tile
    __shared__ uint32_t go[kSsMaxGroups];      // and in the output, less the former (wraps)
    __shared__ uint32_t sh[33];
    // one buffer for the keys, then for the payloads: three workgroups a CU
    constexpr int kMax = sizeof(K) > sizeof(P) ? sizeof(K) : sizeof(P);
    __shared__ __align__(16) uint8_t buf[kTile * kMax];
    __shared__ uint16_t lg[kTile];
    K* const lk = reinterpret_cast<K*>(buf);
    P* const lp = reinterpret_cast<P*>(buf);
    const uint32_t s = blockIdx.x, tid = threadIdx.x;
    uint32_t b, m;
    ss_segment(seg_start, s, n, b, m);
    const bool lead = blockIdx.y == 0;
    if (!lead && static_cast<uint64_t>(blockIdx.y) * kTile >= m) return;
    const uint64_t gat = static_cast<uint64_t>(s) * groups;
    ss_load_tree<K>(gk + gat, gp + gat, groups, tk, tp);
    static_assert(kSsMaxGroups <= kSsThreads, "one group per thread");
    const uint32_t mine = tid < groups ? cnt[gat + tid] : 0u;
    uint32_t tot;
    const uint32_t g0 = block_excl_scan<uint32_t>(mine, sh, &tot);
    if (lead) {
        uint32_t* so = start + static_cast<uint64_t>(s) * (groups + 1);
        if (tid < groups) so[tid] = b + g0;
        if (tid == 0) so[groups] = b + m;
    }
    for (uint64_t t0 = static_cast<uint64_t>(blockIdx.y) * kTile; t0 < m;
         t0 += static_cast<uint64_t>(gridDim.y) * kTile) {
        K k[N];
        P p[N];
        uint32_t q[N], g[N], r[N];
        bool in[N];
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const uint64_t i = t0 + static_cast<uint32_t>(e) * kSsThreads + tid;
            in[e] = i < m;
            k[e] = in[e] ? kin[b + i] : K(0);
            p[e] = in[e] ? (pin ? pin[b + i] : static_cast<P>(b + i)) : P(0);
            q[e] = static_cast<uint32_t>(p[e]);  // the position where ties count
        }
        if (tid < groups) h[tid] = 0;
        __syncthreads();
        ss_classify<TIE, N>(tk, tp, groups, k, q, g);
#pragma unroll
        for (int e = 0; e < N; ++e) r[e] = ss_take(h, g[e], in[e]);
        __syncthreads();
        {
            const uint32_t c = tid < groups ? h[tid] : 0u;
            uint32_t all;
            const uint32_t l0 = block_excl_scan<uint32_t>(c, sh, &all);
            if (tid < groups) {
                ls[tid] = l0;
                uint32_t at = 0;
                if (c) {
                    at = atomicAdd(&cur[gat + tid], c);
                    // more pairs than were counted: the input changed under
                    // the sort.  Stay inside the group and give up.
                    if (at > mine || c > mine - at) {
                        atomicOr(fail, 1u);
                        if (err) atomicOr(err, err_bit);
                        at = 0xFFFFFFFFu;
                    }
                }
                go[tid] = g0 + at - l0;
                h[tid] = at;
            }
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < N; ++e)
            if (in[e]) {
                r[e] += ls[g[e]];
                lk[r[e]] = k[e];
                lg[r[e]] = static_cast<uint16_t>(g[e]);
            }
        __syncthreads();
        const uint32_t len = m - t0 < kTile ? static_cast<uint32_t>(m - t0) : kTile;
        uint32_t dst[N];  // place in the segment, all ones to stay put
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const uint32_t i = static_cast<uint32_t>(e) * kSsThreads + tid;
            dst[e] = 0xFFFFFFFFu;
            if (i < len) {
                const uint32_t gr = lg[i];
                if (h[gr] != 0xFFFFFFFFu) {
                    dst[e] = go[gr] + i;
                    kout[b + static_cast<uint64_t>(dst[e])] = lk[i];
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < N; ++e)
            if (in[e]) lp[r[e]] = p[e];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const uint32_t i = static_cast<uint32_t>(e) * kSsThreads + tid;
            if (dst[e] != 0xFFFFFFFFu) pout[b + static_cast<uint64_t>(dst[e])] = lp[i];
        }
        __syncthreads();
    }
}

// Sort of one group, pairs [b, b + m) of kin and pin, by the whole workgroup
// of NT threads; m <= CAP.  On return (after a barrier) L.k holds the sorted
// keys and, with TIE, L.p their payloads (the positions that ties go by);
// without TIE thread t's pairs p[e] have the ranks f[e].
// A bin of more than kSsBinOwn pairs (keys in runs, repeated keys) is ranked by
// a wave, 64 of its pairs at a time: by its pairs' threads it would hold up
// every wave that has one of them.  Above kSsBinMax the merge is cheaper.
constexpr uint32_t kSsBinOwn = 8, kSsBinMax = 256;
// With TIE a group with a bin of more than kSsBinSpread pairs is dealt again,
// up to kSsSpreads times (ss_spread).  Level-wise lookups of 2^20 32-bit keys,
// us, at 64, 32, 24 and 16 pairs (the radix sort before): runs of consecutive
// keys 146, 127, 126, 130 (127), clustered 144, 141, 129, 122 (128), Zipf 134,
// 133, 135, 142 (127), 100 different keys 128, 129, 129, 134 (124).  Without
// TIE equal keys end the sort, and the code would cost the group kernel a wave
// of its four per SIMD.
constexpr uint32_t kSsBinSpread = 24;
constexpr int kSsSpreads = 3;

// The keys of a bin and the positions of its pairs: smallest and largest.
template <class K>
struct SsSpan {
    K lo, hi;
    uint32_t first, last;
};

template <class K, bool TIE, int NT, uint32_t CAP>
struct SsLds {
    union {
        K k[CAP + CAP / 32];            // padded for ss_merge_held
        SsSpan<K> span[CAP / kSsBinOwn];  // before the pairs are placed
    };
    uint32_t p[TIE ? CAP + CAP / 32 : 1];
    uint32_t bin[CAP + CAP / 32];
    uint32_t big[CAP / kSsBinOwn];  // bins of more than kSsBinOwn pairs: start << 16 | pairs
    uint32_t sh[33];
    unsigned long long lo, hi;
    uint32_t worst, nbig;
};

// Smallest and largest over a row of 16 lanes, in every lane of it.
template <bool MAX, class K>
__device__ __forceinline__ K row_extreme(K x) {
    auto step = [&](auto C) {
        constexpr int ctl = decltype(C)::value;
        K y;
        if constexpr (sizeof(K) == 8) {
            const uint32_t l = __builtin_amdgcn_update_dpp(0, static_cast<int>(x), ctl, 0xf, 0xf, false);
            const uint32_t h = __builtin_amdgcn_update_dpp(0, static_cast<int>(x >> 32), ctl, 0xf, 0xf, false);
            y = (static_cast<uint64_t>(h) << 32) | l;
        } else {
            y = static_cast<K>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), ctl, 0xf, 0xf, false));
        }
        x = MAX ? (y > x ? y : x) : (y < x ? y : x);
    };
    step(std::integral_constant<int, 0x128>{});  // row_ror:8, 4, 2, 1
    step(std::integral_constant<int, 0x124>{});
    step(std::integral_constant<int, 0x122>{});
    step(std::integral_constant<int, 0x121>{});
    return x;
}

// The merge sort of ss_merge_sort over a group held in registers, N pairs a
// thread of which pair e starts at index e * NT + t: a pair's index moves on
// with the rounds, one LDS buffer holds the round's order (padded as there,
// plain in the end).  f: the ranks.
template <int NT, int N, class K>
__device__ void ss_merge_held(const K (&k)[N], const uint32_t (&q)[N], uint32_t (&f)[N], uint32_t m, K* a,
                              uint32_t* p) {
    const uint32_t tid = threadIdx.x;
#pragma unroll
    for (int e = 0; e < N; ++e) f[e] = e * NT + tid;
    for (uint32_t len = 1;; len <<= 1) {
        const bool last = len >= m;
#pragma unroll
        for (int e = 0; e < N; ++e)
            if (e * NT + tid < m) {
                const uint32_t at = last ? f[e] : ss_pad(f[e]);
                a[at] = k[e];
                p[at] = q[e];
            }
        __syncthreads();
        if (last) return;
#pragma unroll
        for (int e = 0; e < N; ++e)
            if (e * NT + tid < m) {
                const uint32_t b0 = f[e] & ~(2u * len - 1u), o = b0 + ((f[e] & len) ? 0u : len);
                const uint32_t ol = o >= m ? 0u : (m - o < len ? m - o : len);
                uint32_t c = 0;
                for (uint32_t st = len; st > 0; st >>= 1) {
                    const uint32_t y = ss_pad(o + c + st - 1);
                    if (c + st <= ol && ss_less<true>(a[y], p[y], k[e], q[e])) c += st;
                }
                f[e] = b0 + (f[e] & (len - 1u)) + c;
            }
        __syncthreads();
    }
}

// exclusive scan of nb bins (a power of two, at most CAP) in place, the total
// behind them; lists the bins of more than kSsBinOwn pairs and returns the
// largest of the thread's
template <int NT, uint32_t CAP>
__device__ __forceinline__ uint32_t ss_scan_bins(uint32_t* bin, uint32_t nb, uint32_t* sh, uint32_t* big,
                                                 uint32_t* nbig) {
    constexpr uint32_t E = CAP / NT;
    const uint32_t per = nb < static_cast<uint32_t>(NT) ? 1u : nb / NT, i0 = threadIdx.x * per;
    uint32_t v[E], sum = 0, worst = 0;
#pragma unroll
    for (uint32_t e = 0; e < E; ++e) {
        v[e] = e < per && i0 + e < nb ? bin[i0 + e] : 0u;
        sum += v[e];
        worst = v[e] > worst ? v[e] : worst;
    }
    uint32_t tot;
    uint32_t off = block_excl_scan<uint32_t>(sum, sh, &tot);
#pragma unroll
    for (uint32_t e = 0; e < E; ++e)
        if (e < per && i0 + e < nb) {
            bin[i0 + e] = off;
            if (v[e] > kSsBinOwn) big[atomicAdd(nbig, 1u)] = off << 16 | v[e];
            off += v[e];
        }
    if (threadIdx.x == 0) bin[nb] = tot;
    return worst;
}

template <class K>
__device__ __forceinline__ void lds_min(K* a, K x) {
    if constexpr (sizeof(K) == 8) atomicMin(reinterpret_cast<unsigned long long*>(a), static_cast<unsigned long long>(x));
    else atomicMin(a, x);
}

template <class K>
__device__ __forceinline__ void lds_max(K* a, K x) {
    if constexpr (sizeof(K) == 8) atomicMax(reinterpret_cast<unsigned long long*>(a), static_cast<unsigned long long>(x));
    else atomicMax(a, x);
}

// Deals the pairs of each bin of more than kSsBinOwn among as many bins as it
// has pairs: by their distance from its smallest key, or, where it holds one
// key, from its first position (a key that is repeated many times fills whole
// groups, in which only the positions differ).  bin holds starts before and
// counts after, bn and f a pair's bin and its place there.  Without this such
// groups were merge-sorted, ten rounds and more: the level-wise lookup of 2^20
// u32 keys of which 100 differ 239 us, now 129, of Zipf ones 190 and 135 (120
// where all differ); of 2^15 69 and 39, 70 and 43 (33).
template <class K, int NT, uint32_t CAP>
__device__ __forceinline__ void ss_spread(SsLds<K, true, NT, CAP>& L, uint32_t m, uint32_t nb, const K (&k)[CAP / NT],
                                          const uint32_t (&p)[CAP / NT], uint32_t (&bn)[CAP / NT],
                                          uint32_t (&f)[CAP / NT]) {
    constexpr uint32_t E = CAP / NT;
    const uint32_t tid = threadIdx.x;
    uint32_t b0[E], n[E];
    // (starts of bins above kSsBinOwn lie further apart than kSsBinOwn)
    auto span = [&](uint32_t e) -> SsSpan<K>& { return L.span[b0[e] / kSsBinOwn]; };
#pragma unroll
    for (uint32_t e = 0; e < E; ++e) {
        const bool in = e * NT + tid < m;
        b0[e] = in ? L.bin[bn[e]] : 0u;
        n[e] = in ? L.bin[bn[e] + 1] - b0[e] : 0u;
        if (n[e] > kSsBinOwn && f[e] == 0) span(e) = SsSpan<K>{k[e], k[e], p[e], p[e]};  // one pair of the bin
    }
    __syncthreads();
#pragma unroll
    for (uint32_t e = 0; e < E; ++e)
        if (n[e] > kSsBinOwn) {
            SsSpan<K>& s = span(e);
            if (k[e] < s.lo) lds_min(&s.lo, k[e]);
            if (k[e] > s.hi) lds_max(&s.hi, k[e]);
            if (p[e] < s.first) atomicMin(&s.first, p[e]);
            if (p[e] > s.last) atomicMax(&s.last, p[e]);
        }
    for (uint32_t i = tid; i < nb; i += NT) L.bin[i] = 0;
    if (tid == 0) {
        L.worst = 0;
        L.nbig = 0;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t e = 0; e < E; ++e) {
        uint32_t to = 0;
        if (n[e] > kSsBinOwn) {
            const SsSpan<K>& s = span(e);
            // (conversions and the product round, but keep the order)
            const bool one = s.lo == s.hi;
            const float range = one ? static_cast<float>(s.last - s.first) : static_cast<float>(s.hi - s.lo);
            const float off = one ? static_cast<float>(p[e] - s.first) : static_cast<float>(k[e] - s.lo);
            to = static_cast<uint32_t>(off * (static_cast<float>(n[e]) / (range + 1.0f)));
            to = to < n[e] ? to : n[e] - 1u;
        }
        bn[e] = b0[e] + to;
        f[e] = e * NT + tid < m ? atomicAdd(&L.bin[bn[e]], 1u) : 0u;
    }
    __syncthreads();
}

template <class K, class P, bool TIE, int NT, uint32_t CAP>
__device__ __forceinline__ void ss_sort_group(const K* kin, const P* pin, uint64_t b, uint32_t m,
                                              SsLds<K, TIE, NT, CAP>& L, P (&p)[CAP / NT], uint32_t (&f)[CAP / NT]) {
    constexpr uint32_t E = CAP / NT;
    const uint32_t tid = threadIdx.x;
    K k[E];
    K lo = kmax<K>(), hi = K(0);
    uint32_t nb = 1;
    while (nb < m) nb <<= 1;
#pragma unroll
    for (uint32_t e = 0; e < E; ++e) {
        const uint32_t i = e * NT + tid;
        k[e] = K(0);
        p[e] = P(0);
        if (i < m) {
            k[e] = kin[b + i];
            p[e] = pin[b + i];
        }
    }
    for (uint32_t i = tid; i < nb; i += NT) L.bin[i] = 0;
    if (tid == 0) {
        L.worst = 0;
        L.nbig = 0;
        L.lo = ~0ull;
        L.hi = 0;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t e = 0; e < E; ++e)
        if (e * NT + tid < m) {
            lo = k[e] < lo ? k[e] : lo;
            hi = k[e] > hi ? k[e] : hi;
        }
    lo = row_extreme<false>(lo);
    hi = row_extreme<true>(hi);
    if ((tid & 15) == 0) {
        atomicMin(&L.lo, static_cast<unsigned long long>(lo));
        atomicMax(&L.hi, static_cast<unsigned long long>(hi));
    }
    __syncthreads();
    lo = static_cast<K>(L.lo);
    hi = static_cast<K>(L.hi);
    // a bin is 2^shift keys wide, the first starts at the smallest key: nb of
    // them reach the largest
    const uint64_t range = static_cast<uint64_t>(static_cast<K>(hi - lo));
    const int width = range ? 64 - __clzll(static_cast<long long>(range)) : 0, bits = 31 - __clz(static_cast<int>(nb));
    const int shift = width > bits ? width - bits : 0;
    uint32_t bn[E];
#pragma unroll
    for (uint32_t e = 0; e < E; ++e)
        bn[e] = e * NT + tid < m ? static_cast<uint32_t>(static_cast<uint64_t>(static_cast<K>(k[e] - lo)) >> shift) : 0u;
#pragma unroll
    for (uint32_t e = 0; e < E; ++e) f[e] = e * NT + tid < m ? atomicAdd(&L.bin[bn[e]], 1u) : 0u;
    __syncthreads();
    uint32_t worst;  // the same for the whole workgroup
    for (int round = 0;; ++round) {
        const uint32_t mine = ss_scan_bins<NT, CAP>(L.bin, nb, L.sh, L.big, &L.nbig);
        if (mine > kSsBinSpread) atomicMax(&L.worst, mine);
        __syncthreads();
        worst = L.worst;
        if constexpr (TIE) {
            if (worst > kSsBinSpread && round < kSsSpreads) {
                ss_spread<K, NT, CAP>(L, m, nb, k, p, bn, f);
                continue;
            }
        }
        break;
    }
    if (worst > kSsBinMax) {
        uint32_t q[E];
#pragma unroll
        for (uint32_t e = 0; e < E; ++e) q[e] = TIE ? static_cast<uint32_t>(p[e]) : e * NT + tid;
        if constexpr (TIE) ss_merge_held<NT, E>(k, q, f, m, L.k, L.p);
        else ss_merge_held<NT, E>(k, q, f, m, L.k, L.bin);
        return;
    }
#pragma unroll
    for (uint32_t e = 0; e < E; ++e)
        if (e * NT + tid < m) {
            f[e] += L.bin[bn[e]];
            L.k[f[e]] = k[e];
            if constexpr (TIE) L.p[f[e]] = static_cast<uint32_t>(p[e]);
        }
    __syncthreads();
    // a pair's rank: its bin's start plus the bin's smaller pairs
    uint32_t held = 0;  // bit e: pair e is in a large bin
#pragma unroll
    for (uint32_t e = 0; e < E; ++e) {
        if (e * NT + tid < m) {
            const uint32_t b0 = L.bin[bn[e]], b1 = L.bin[bn[e] + 1];
            if (b1 - b0 > kSsBinOwn) {
                held |= 1u << e;
                continue;
            }
            uint32_t c = b0;
            for (uint32_t x = b0; x < b1; x += 2) {
                const uint32_t x1 = x + 1 < b1 ? x + 1 : x;  // two reads in flight
                const K y0 = L.k[x], y1 = L.k[x1];
                bool lt0 = y0 < k[e], lt1 = y1 < k[e];
                if constexpr (TIE) {
                    const uint32_t q0 = L.p[x], q1 = L.p[x1];
                    lt0 = lt0 | ((y0 == k[e]) & (q0 < static_cast<uint32_t>(p[e])));
                    lt1 = lt1 | ((y1 == k[e]) & (q1 < static_cast<uint32_t>(p[e])));
                } else {
                    lt0 = lt0 || (y0 == k[e] && x < f[e]);
                    lt1 = lt1 || (y1 == k[e] && x1 < f[e]);
                }
                c += (lt0 ? 1u : 0u) + (lt1 && x1 != x ? 1u : 0u);
            }
            f[e] = c;
        }
    }
    const uint32_t nbig = L.nbig;
    __syncthreads();  // the bins are free: large bins' ranks go there, by slot
    if (nbig) {
        const uint32_t lane = tid & 63;
        for (uint32_t i = tid / 64; i < nbig; i += NT / 64) {
            const uint32_t b0 = L.big[i] >> 16, b1 = b0 + (L.big[i] & 0xFFFFu);
            for (uint32_t x = b0 + lane; x - lane < b1; x += 64) {
                const uint32_t own = x < b1 ? x : b0;
                const K kx = L.k[own];
                uint32_t px = own, c = b0;
                if constexpr (TIE) px = L.p[own];
#pragma unroll 4
                for (uint32_t j = b0; j < b1; ++j) {  // one address for the wave
                    const K y = L.k[j];
                    uint32_t py = j;
                    if constexpr (TIE) py = L.p[j];
                    c += static_cast<uint32_t>(y < kx) | (static_cast<uint32_t>(y == kx) & static_cast<uint32_t>(py < px));
                }
                if (x < b1) L.bin[x] = c;
            }
        }
        __syncthreads();
#pragma unroll
        for (uint32_t e = 0; e < E; ++e)
            if ((held >> e) & 1u) f[e] = L.bin[f[e]];
        __syncthreads();
    }
#pragma unroll
    for (uint32_t e = 0; e < E; ++e)
        if (e * NT + tid < m) {
            L.k[f[e]] = k[e];
            if constexpr (TIE) L.p[f[e]] = static_cast<uint32_t>(p[e]);
        }
    __syncthreads();
}

// The groups a group kernel of grid gridDim.x takes: with `list` null group
// x = blockIdx.x (segment x % segs, so that a segment's groups run on the XCD
// whose L2 its scatter wrote through), else the listed groups in turn.
// body(b, m) for each.
template <class F>
__device__ __forceinline__ void ss_each_group(const uint32_t* __restrict__ start, uint32_t segs, uint32_t groups,
                                              const uint32_t* __restrict__ list, F&& body) {
    const uint32_t total = list ? list[0] : segs * groups;
    for (uint32_t i = blockIdx.x; i < total; i += gridDim.x) {
        const uint32_t x = list ? list[1 + i] : i;
        const uint32_t* so = start + static_cast<uint64_t>(x % segs) * (groups + 1) + x / segs;
        body(x, so[0], so[1] - so[0]);
        __syncthreads();
    }
}

// Workgroup shapes of the group kernels.  Small: 256 threads and 2048 pairs,
// for a mean group of at most 1024 (512 with one level, which needs no list
// then); mid: 512 threads and 4096 pairs, two workgroups a CU, for the 512
// groups of up to 2^20 pairs; large: 1024 threads and 8192 pairs, for the
// groups that the others leave to a list.  A group that does not fit is sorted
// in device memory.
constexpr int kSsSmallThreads = 256, kSsMidThreads = 512, kSsLargeThreads = 1024;
constexpr uint32_t kSsSmallCap = 2048, kSsMidCap = 4096, kSsLargeCap = 8192;

// Group sort of (key, position) pairs into kout, iout (which may be kin, pin).
// `later`: the list of groups left to the large workgroups.  `cap`: the
// largest group to sort in LDS, for tests.
template <class K, int NT, uint32_t CAP>
__global__ __launch_bounds__(NT) void k_ss_groups(const K* kin, const uint32_t* pin, const uint32_t* start,
                                                  uint32_t segs, uint32_t groups, const uint32_t* list,
                                                  uint32_t* later, K* kout, uint32_t* iout, const uint32_t* fail,
                                                  uint32_t cap) {
    __shared__ SsLds<K, true, NT, CAP> L;
    const uint32_t tid = threadIdx.x;
    const bool failed = *fail != 0;
    ss_each_group(start, segs, groups, list, [&](uint32_t x, uint32_t b, uint32_t m) {
        if (failed) {  // replaced by a valid result
            for (uint32_t i = tid; i < m; i += NT) {
                kout[b + i] = K(0);
                iout[b + i] = b + i;
            }
            return;
        }
        if (m > CAP || m > cap) {
            if (later) {
                if (tid == 0) later[1 + atomicAdd(&later[0], 1u)] = x;
                return;
            }
            if (kin != kout) {
                for (uint32_t i = tid; i < m; i += NT) {
                    kout[b + i] = kin[b + i];
                    iout[b + i] = pin[b + i];
                }
                __syncthreads();
            }
            ss_bitonic<true>(kout + b, iout + b, m);
            return;
        }
        uint32_t p[CAP / NT], f[CAP / NT];
        ss_sort_group<K, uint32_t, true, NT, CAP>(kin, pin, b, m, L, p, f);
        for (uint32_t i = tid; i < m; i += NT) {
            kout[b + i] = L.k[i];
            iout[b + i] = L.p[i];
        }
    });
}

// Where the pair of rank r goes when n pairs fill L leaves evenly (leaf j
// holds [j n / L, (j + 1) n / L)).  Where every leaf holds `each` pairs a
// multiplication by inv = ceil(2^32 / each) divides exactly (r < 2^26 is off
// by less than 2^-6, a sixteenth is the smallest step).  Else in FP64: n and L
// are at most 2^26, so the products are exact, and a quotient that is no whole
// number is further from one (2^-26) than its rounding error (2^-27).
struct LeafSlot {
    uint32_t leaf, first, end;  // the leaf and its range of ranks
};

__device__ __forceinline__ LeafSlot leaf_slot(uint32_t r, uint32_t n, uint32_t L, uint32_t each, uint32_t inv) {
    LeafSlot s;
    if (each) {
        s.leaf = each == 1 ? r : __umulhi(r, inv);
        s.first = s.leaf * each;
        s.end = s.first + each;
        return s;
    }
    const double dn = n, dl = L;
    s.leaf = static_cast<uint32_t>(ceil((static_cast<double>(r) + 1.0) * dl / dn)) - 1u;
    s.first = static_cast<uint32_t>(floor(static_cast<double>(s.leaf) * dn / dl));
    s.end = static_cast<uint32_t>(floor((static_cast<double>(s.leaf) + 1.0) * dn / dl));
    return s;
}

// Group sort of (key, value) pairs straight into leaves: a pair's rank names
// its leaf and slot, so the sorted pairs are not written and read back.  The
// first pair of a leaf writes its count and link, the last its padding and its
// bound (maxk).  Equal keys lie in one group (ties go by the key alone here)
// and become neighbours: they set bit 0 of *refuse.
template <class K, int NT, uint32_t CAP>
__global__ __launch_bounds__(NT) void k_ss_leaves(K* kin, K* vin, const uint32_t* start, uint32_t segs,
                                                  uint32_t groups, const uint32_t* list, uint32_t* later, K* lkeys,
                                                  K* lvals, uint2* lmeta, uint32_t n, uint32_t nl, uint32_t each,
                                                  K* maxk, uint32_t* refuse, uint32_t cap) {
    __shared__ SsLds<K, false, NT, CAP> L;
    const uint32_t tid = threadIdx.x;
    if (ss_refused<false>(refuse)) return;
    const uint32_t inv = each > 1 ? static_cast<uint32_t>(((1ull << 32) + each - 1) / each) : 0u;
    auto key_out = [&](uint32_t r, K key, bool twin) {
        const LeafSlot s = leaf_slot(r, n, nl, each, inv);
        const uint64_t line = static_cast<uint64_t>(s.leaf) * kSlots;
        lkeys[line + (r - s.first)] = key;
        if (twin) atomicOr(refuse, 1u);
        if (r == s.first) lmeta[s.leaf] = make_uint2(s.end - s.first, s.leaf + 1 < nl ? s.leaf + 1 : kNone);
        if (r + 1 == s.end) {
            maxk[s.leaf] = key;
            for (uint32_t x = s.end - s.first; x < static_cast<uint32_t>(kSlots); ++x) lkeys[line + x] = key;
        }
    };
    auto value_out = [&](uint32_t r, K val) {
        const LeafSlot s = leaf_slot(r, n, nl, each, inv);
        const uint64_t line = static_cast<uint64_t>(s.leaf) * kSlots;
        lvals[line + (r - s.first)] = val;
        if (r + 1 == s.end)
            for (uint32_t x = s.end - s.first; x < static_cast<uint32_t>(kSlots); ++x) lvals[line + x] = kmax<K>();
    };
    ss_each_group(start, segs, groups, list, [&](uint32_t x, uint32_t b, uint32_t m) {
        if (m > CAP || m > cap) {
            if (later) {
                if (tid == 0) later[1 + atomicAdd(&later[0], 1u)] = x;
                return;
            }
            ss_bitonic<false>(kin + b, vin + b, m);
            for (uint32_t i = tid; i < m; i += NT) {
                key_out(b + i, kin[b + i], i > 0 && kin[b + i - 1] == kin[b + i]);
                value_out(b + i, vin[b + i]);
            }
            return;
        }
        K v[CAP / NT];
        uint32_t f[CAP / NT];
        ss_sort_group<K, K, false, NT, CAP>(kin, vin, b, m, L, v, f);
        for (uint32_t i = tid; i < m; i += NT) key_out(b + i, L.k[i], i > 0 && L.k[i - 1] == L.k[i]);
        __syncthreads();  // the values take the keys' place
#pragma unroll
        for (uint32_t e = 0; e < CAP / NT; ++e)
            if (e * NT + tid < m) L.k[f[e]] = v[e];
        __syncthreads();
        for (uint32_t i = tid; i < m; i += NT) value_out(b + i, L.k[i]);
    });
}

// ------------------------------------------------------------- host side

// Testing hooks: the largest input, the largest group sorted in LDS.
static std::atomic<uint64_t> g_ss_max{kSsMax};
static std::atomic<uint32_t> g_ss_group{kSsLargeCap};

uint64_t set_sample_sort_max(uint64_t n) {
    return g_ss_max.exchange(n < kSsMax ? n : kSsMax, std::memory_order_relaxed);
}
uint32_t set_sample_sort_group(uint32_t pairs) {
    return g_ss_group.exchange(pairs < kSsLargeCap ? pairs : kSsLargeCap, std::memory_order_relaxed);
}
uint64_t sample_sort_max() { return g_ss_max.load(std::memory_order_relaxed); }

// The sample's seed: another one for every sort (a captured one keeps its).
static uint32_t ss_next_seed() {
    static std::atomic<uint32_t> next{
        static_cast<uint32_t>(std::chrono::steady_clock::now().time_since_epoch().count())};
    return next.fetch_add(0x9E3779B9u, std::memory_order_relaxed);
}

bool sort_leaves_two_buffers(uint64_t n) { return n > kSsOneLevel; }
uint64_t sample_sort_tmp_bytes(uint64_t n, int key_bytes) { return ss_plan(n, key_bytes).bytes; }

// Sample, count and scatter of every level.  The pairs end in the buffers
// *kr, *pr: ka, pa after one level, kb, pb after two.
template <class K, class P, bool TIE>
static void ss_partition(const SsPlan& pl, uint8_t* tmp, const K* src, const P* pin, uint32_t n, K* ka, P* pa, K* kb,
                         P* pb, uint32_t force, uint32_t* err, uint32_t err_bit, uint32_t* dup, K** kr, P** pr,
                         hipStream_t s) {
    uint32_t* fail = reinterpret_cast<uint32_t*>(tmp + pl.o_fail);
    uint32_t* list = reinterpret_cast<uint32_t*>(tmp + pl.o_list);
    const uint32_t seed = ss_next_seed();
    const K* kin = src;
    const P* in = pin;
    K* kout = ka;
    P* out = pa;
    const uint32_t* seg = nullptr;
    for (int l = 0; l < pl.levels; ++l) {
        const SsLevel& v = pl.lv[l];
        K* gk = reinterpret_cast<K*>(tmp + v.o_gk);
        uint32_t* gp = reinterpret_cast<uint32_t*>(tmp + v.o_gp);
        K* sk = reinterpret_cast<K*>(tmp + v.o_sk);
        uint32_t* sp = reinterpret_cast<uint32_t*>(tmp + v.o_sp);
        uint32_t* cnt = reinterpret_cast<uint32_t*>(tmp + v.o_cnt);
        uint32_t* cur = reinterpret_cast<uint32_t*>(tmp + v.o_cur);
        uint32_t* start = reinterpret_cast<uint32_t*>(tmp + v.o_start);
        // ties go by the position: the payload where it is one
        const uint32_t* tie = nullptr;
        if constexpr (TIE) tie = in;
        const uint32_t S = v.groups * v.over, len = S / v.runs;
        if (v.segs == 1 && S >= kSsRankStep && S <= kSsRankSample) {
            hipLaunchKernelGGL((k_ss_sample_rank<K, TIE>), dim3(S * 16 / kSsRankThreads), dim3(kSsRankThreads), 0, s,
                               kin, tie, n, v.groups, v.over, seed, gk, gp, cnt, cur, list, fail, force, err, err_bit, dup);
        } else {
            hipLaunchKernelGGL((k_ss_sample<K, TIE>), dim3(v.segs, v.runs), dim3(len <= 256 ? 256 : (len <= 512 ? 512 : 1024)),
                               0, s, kin, tie, n, seg, v.groups, v.over, v.runs, seed, gk, gp, sk, sp, cnt, cur, list, fail,
                               force, err, err_bit, dup);
            auto rank = [&](auto R) {
                constexpr int N = decltype(R)::value;
                hipLaunchKernelGGL((k_ss_rank<K, TIE, N>), dim3(N * kSsRun / 256), dim3(256), 0, s, sk, sp, v.over, gk,
                                   gp, dup);
            };
            if (v.runs == 8) rank(std::integral_constant<int, 8>{});
            else if (v.runs == kSsMaxRuns) rank(std::integral_constant<int, kSsMaxRuns>{});
        }
        // tiles: as long as they leave two workgroups for every CU
        auto tiles = [&](auto items) {
            constexpr int N = decltype(items)::value;
            constexpr uint32_t T = kSsThreads * N;
            const uint32_t ty = (n / v.segs + T - 1) / T, gy = v.segs == 1 && ty > 1024 ? 1024 : (ty < 1 ? 1 : ty);
            const dim3 grid(v.segs, gy);
            hipLaunchKernelGGL((k_ss_count<K, TIE, N>), grid, dim3(kSsThreads), 0, s, kin, tie, n, seg, v.groups, gk,
                               gp, cnt, dup);
            hipLaunchKernelGGL((k_ss_scatter<K, P, TIE, N>), grid, dim3(kSsThreads), 0, s, kin, in, n, seg, v.groups,
                               gk, gp, cnt, cur, start, kout, out, fail, err, err_bit, dup);
        };
        if (n > kSsOneLevel) tiles(std::integral_constant<int, 8>{});
        else if (n > (1u << 18)) tiles(std::integral_constant<int, 4>{});
        else tiles(std::integral_constant<int, 2>{});
        kin = kout;
        in = out;
        *kr = kout;
        *pr = out;
        kout = kb;
        out = pb;
        seg = start;
    }
}

// The group kernels of one sort: the shape by the mean group, then the list.
template <class F>
static void ss_launch_groups(F&& groups, int levels, uint32_t total, bool listed, uint32_t* list) {
    if (listed && levels == 1)
        groups(std::integral_constant<int, kSsMidThreads>{}, std::integral_constant<uint32_t, kSsMidCap>{}, total,
               nullptr, list);
    else
        groups(std::integral_constant<int, kSsSmallThreads>{}, std::integral_constant<uint32_t, kSsSmallCap>{}, total,
               nullptr, listed ? list : nullptr);
    if (listed)
        groups(std::integral_constant<int, kSsLargeThreads>{}, std::integral_constant<uint32_t, kSsLargeCap>{}, 256u,
               list, nullptr);
}

template <class K>
void sample_sort_from(const K* src, K* keys, uint32_t* idx, K* keys_alt, uint32_t* idx_alt, uint64_t n, void* tmp,
                      hipStream_t s, uint32_t* err, uint32_t err_bit, bool force_fail) {
    const SsPlan pl = ss_plan(n, sizeof(K));
    uint8_t* b = reinterpret_cast<uint8_t*>(tmp);
    const SsLevel& v = pl.lv[pl.levels - 1];
    uint32_t* fail = reinterpret_cast<uint32_t*>(b + pl.o_fail);
    uint32_t* list = reinterpret_cast<uint32_t*>(b + pl.o_list);
    const uint32_t* start = reinterpret_cast<const uint32_t*>(b + v.o_start);
    const uint32_t cap = g_ss_group.load(std::memory_order_relaxed);
    K* kr;
    uint32_t* pr;
    ss_partition<K, uint32_t, true>(pl, b, src, nullptr, static_cast<uint32_t>(n), keys_alt, idx_alt, keys, idx,
                                    force_fail ? 1u : 0u, err, err_bit, nullptr, &kr, &pr, s);
    auto groups = [&](auto NT, auto CAP, uint32_t grid, const uint32_t* from, uint32_t* later) {
        hipLaunchKernelGGL((k_ss_groups<K, decltype(NT)::value, decltype(CAP)::value>), dim3(grid),
                           dim3(decltype(NT)::value), 0, s, kr, pr, start, v.segs, v.groups, from, later, keys, idx,
                           fail, cap);
    };
    ss_launch_groups(groups, pl.levels, v.segs * v.groups, n > kSsSmallMean * kSsMaxGroups, list);
}

template <class K>
void launch_sort_leaves(const K* keys, const K* vals, uint64_t n64, uint64_t leaves, K* ka, K* va, K* kb, K* vb,
                        void* tmp, K* lkeys, K* lvals, uint2* lmeta, K* maxk, uint32_t* refuse, uint32_t fail_bit,
                        bool force_fail, hipStream_t s) {
    const SsPlan pl = ss_plan(n64, sizeof(K));
    uint8_t* b = reinterpret_cast<uint8_t*>(tmp);
    const uint32_t n = static_cast<uint32_t>(n64), nl = static_cast<uint32_t>(leaves);
    const SsLevel& v = pl.lv[pl.levels - 1];
    const uint32_t each = n % nl == 0 ? n / nl : 0u;
    uint32_t* list = reinterpret_cast<uint32_t*>(b + pl.o_list);
    const uint32_t* start = reinterpret_cast<const uint32_t*>(b + v.o_start);
    const uint32_t cap = g_ss_group.load(std::memory_order_relaxed);
    K *kr, *vr;
    ss_partition<K, K, false>(pl, b, keys, vals, n, ka, va, kb, vb, force_fail ? 1u : 0u, refuse, fail_bit, refuse,
                              &kr, &vr, s);
    auto groups = [&](auto NT, auto CAP, uint32_t grid, const uint32_t* from, uint32_t* later) {
        hipLaunchKernelGGL((k_ss_leaves<K, decltype(NT)::value, decltype(CAP)::value>), dim3(grid),
                           dim3(decltype(NT)::value), 0, s, kr, vr, start, v.segs, v.groups, from, later, lkeys, lvals,
                           lmeta, n, nl, each, maxk, refuse, cap);
    };
    ss_launch_groups(groups, pl.levels, v.segs * v.groups, n64 > kSsSmallMean * kSsMaxGroups, list);
}

template void sample_sort_from<uint32_t>(const uint32_t*, uint32_t*, uint32_t*, uint32_t*, uint32_t*, uint64_t, void*,
                                         hipStream_t, uint32_t*, uint32_t, bool);
template void sample_sort_from<uint64_t>(const uint64_t*, uint64_t*, uint32_t*, uint64_t*, uint32_t*, uint64_t, void*,
                                         hipStream_t, uint32_t*, uint32_t, bool);
template void launch_sort_leaves<uint32_t>(const uint32_t*, const uint32_t*, uint64_t, uint64_t, uint32_t*, uint32_t*,
                                           uint32_t*, uint32_t*, void*, uint32_t*, uint32_t*, uint2*, uint32_t*,
                                           uint32_t*, uint32_t, bool, hipStream_t);
template void launch_sort_leaves<uint64_t>(const uint64_t*, const uint64_t*, uint64_t, uint64_t, uint64_t*, uint64_t*,
                                           uint64_t*, uint64_t*, void*, uint64_t*, uint64_t*, uint2*, uint64_t*,
                                           uint32_t*, uint32_t, bool, hipStream_t);

}  // namespace gt
