// Tile scheduling shared by the forward tile kernels and the adjoint: tile
// lists of kSub sub-lists drained by persistent workgroups through fetch
// counters, per-list tile stamps, dirty-face masks by launch parity, order
// keys and the sampled threshold by which a launch takes the lowest of them
// (ordered scheduling), plus the in-tile geometry and LDS list helpers.
#pragma once

#include <stdint.h>

#include <type_traits>

#include "eik_device.hpp"
#include "eik_internal.hpp"

namespace eik {
namespace {

// Persistent workgroups of a tile launch (eik_options.workgroups, a multiple
// of kSub); group k = blockIdx % kSub drains sub-list k of the launch's tile
// list.  GT is the most a launch takes.
constexpr int GT = kMaxStatBlocks;
constexpr int kSub = kWorkgroupStep;  // sub-lists per tile list
static_assert(GT % kSub == 0, "each sub-list has the same number of workgroups");
constexpr int kPad = 32;      // ints between counters (separate cache lines)
// Dirty-face mask bit meaning "recheck every node of the tile".
constexpr uint32_t kAllFaces = 64u;
// Order keys: monotone 32-bit images of the smallest value that made a tile
// pending; kNoKey marks a tile that is not listed.
constexpr uint32_t kNoKey = 0xffffffffu;

// A tile list: kSub sub-lists of `cap` entries, tile t in sub-list t % kSub.
// count[k * kPad] is the length of sub-list k (appended with atomicAdd by
// producers), fetch[k * kPad] the next entry a consumer of sub-list k takes
// (atomicAdd by consumers).  An entry is the tile and, ordered, the key it was
// first listed with (high half); its key may have dropped since (key arrays).
struct TList {
    unsigned long long* data;
    int* count;
    int* fetch;
    int cap;
};
__device__ __forceinline__ unsigned long long list_entry(int t, uint32_t key) {
    return (static_cast<unsigned long long>(key) << 32) | static_cast<uint32_t>(t);
}

// Scheduling state of a tile launch (shared by the forward kernels and the
// adjoint): the list it drains and the one it fills, tile stamps, dirty-face
// masks, order keys, the control block.
struct Sched {
    uint32_t* tstamp;
    // Per tile dirty faces (bit d) or kAllFaces, double-buffered by launch
    // parity: a launch reads and clears `mask_cur` of the tiles it visits and
    // sets bits only in `mask_next`, which the next launch reads.  A bit set
    // during a launch is therefore never consumed by a visit that may have
    // staged the neighbour's values before the change that set it.
    uint32_t* mask_cur;
    uint32_t* mask_next;
    // ordered scheduling: keys by launch parity
    uint32_t* key_cur;
    uint32_t* key_next;
    int ordered;
    int order_aim;     // ordered: lowest-key tiles a launch takes, about
    TList cur;
    TList next;
    int* zero_count;   // counters of the list two launches ahead: cleared by this launch
    int* zero_fetch;
    Ctl* ctl;
    unsigned long long* blkstat;  // [kStatFields][kMaxStatBlocks], column blockIdx % kMaxStatBlocks
    int* mail;  // where the launch reports the length of the list it found (pinned host word; may be NULL)
    int tag_slot;
    int phase;  // 0 update step, 1 remedy (or adjoint) loop
    int first;  // first launch of its loop
};

__device__ __forceinline__ bool claim_tile(uint32_t* tstamp, int t, uint32_t tag) {
    return atomicMax(tstamp + t, tag) < tag;
}

template <int ND, int TX, int TY, int TZ>
struct Shape {
    static constexpr int LX = TX + 2;
    static constexpr int LY = TY + 2;
    static constexpr int LZ = ND == 3 ? TZ + 2 : 1;
    static constexpr int NT = TX * TY * (ND == 3 ? TZ : 1);
    static constexpr int NL = LX * LY * LZ;
    static constexpr int NPT = (NT + kBlock - 1) / kBlock;
    static constexpr int SY = LX;
    static constexpr int SZ = LX * LY;
};

template <int ND, int TX, int TY, int TZ>
__device__ __forceinline__ int lds_offset(int d) {
    using S = Shape<ND, TX, TY, TZ>;
    switch (d) {
        case 0: return -1;
        case 1: return 1;
        case 2: return -S::SY;
        case 3: return S::SY;
        case 4: return -S::SZ;
        default: return S::SZ;
    }
}

// The neighbour values of LDS node L in direction order (-x, +x, -y, +y, -z, +z).
template <typename T, int ND, int TX, int TY, int TZ>
__device__ __forceinline__ void load_nb(const T* lds, int L, T (&nb)[2 * ND]) {
#pragma unroll
    for (int d = 0; d < 2 * ND; ++d) nb[d] = lds[L + lds_offset<ND, TX, TY, TZ>(d)];
}

template <typename T>
__device__ __forceinline__ int neighbour_tile(const Inst<T>& g, int t, int d) {
    switch (d) {
        case 0: return t - 1;
        case 1: return t + 1;
        case 2: return t - g.ntx;
        case 3: return t + g.ntx;
        case 4: return t - g.ntx * g.nty;
        default: return t + g.ntx * g.nty;
    }
}

// Tag chain: launch with slot p reads tag[p] and stores tag[p] + 1 into
// tag[p ^ 1]; tiles it schedules are claimed with tag[p] + 1.
// The last workgroup of a launch keeps its books: it is the one most likely to
// have no tile to visit, so that nobody waits for its reads of the control
// block.
__device__ __forceinline__ bool book_keeper() { return blockIdx.x == gridDim.x - 1; }
__device__ __forceinline__ uint32_t launch_tag(const Sched& a) {
    const uint32_t tag = static_cast<uint32_t>(a.ctl->tag[a.tag_slot]);
    if (book_keeper() && threadIdx.x == 0) a.ctl->tag[a.tag_slot ^ 1] = static_cast<int>(tag + 1);
    return tag + 1;
}

__device__ __forceinline__ void launch_stats(const Sched& a, int n) {
    if (book_keeper() && threadIdx.x == 0) {
        const unsigned long long un = static_cast<unsigned long long>(n);
        if (n > 0) {
            if (a.phase == 0) {
                a.ctl->iters2 += 1;
                if (un > a.ctl->max_active) a.ctl->max_active = un;
            } else {
                a.ctl->iters3 += 1;
            }
        }
        if (a.first) a.ctl->remedy_init = un;
        if (a.mail) __hip_atomic_store(a.mail, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Claim tile t for the next list and append it to sub-list t % kSub.
__device__ __forceinline__ bool push_tile(const TList& out, uint32_t* tstamp, int t, uint32_t tag) {
    if (!claim_tile(tstamp, t, tag)) return false;
    const int k = t & (kSub - 1);
    const int pos = atomicAdd(out.count + k * kPad, 1);
    out.data[static_cast<size_t>(k) * out.cap + pos] = list_entry(t, 0u);
    return true;
}

// Order key of a value: unsigned integers compare like the (float) values.
template <typename T>
__device__ __forceinline__ uint32_t order_key(T v) {
    const uint32_t b = __float_as_uint(static_cast<float>(v));
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// push_tile with an order key.  In ordered mode the tile's key in the next
// list drops to `key` if lower, and the key array also tells membership: the
// keys of a list start at kNoKey (a tile leaving a list has its key reset,
// a tile carried over to the next list takes its key there), so the push
// that sees kNoKey is the first of t into the next list and appends it.
// Without ordering the tile stamp deduplicates (push_tile).
__device__ __forceinline__ void push_keyed(const Sched& a, int t, uint32_t tag, uint32_t key) {
    if (!a.ordered) {
        push_tile(a.next, a.tstamp, t, tag);
        return;
    }
    if (atomicMin(a.key_next + t, key) != kNoKey) return;
    const int k = t & (kSub - 1);
    const int pos = atomicAdd(a.next.count + k * kPad, 1);
    a.next.data[static_cast<size_t>(k) * a.next.cap + pos] = list_entry(t, key);
}

// Clear the counters of the list two launches ahead (nobody reads or writes
// them during this launch) and return the total length of the current list.
__device__ __forceinline__ int list_open(const Sched& a, int* s_len) {
    if (book_keeper() && threadIdx.x < kSub) {
        a.zero_count[threadIdx.x * kPad] = 0;
        a.zero_fetch[threadIdx.x * kPad] = 0;
    }
    if (threadIdx.x < kSub) s_len[threadIdx.x] = a.cur.count[threadIdx.x * kPad];
    __syncthreads();
    int n = 0;
#pragma unroll
    for (int k = 0; k < kSub; ++k) n += s_len[k];
    return n;
}

// Ordered: the largest key a launch takes, so that it visits about order_aim
// of its n tiles (more than order_aim), or n / kListShare if that is more.  The
// quantile of 64 listed keys, spread over the sub-lists: every workgroup draws the
// same sample (one 8-byte load per lane) and ranks it without LDS.  The count
// taken scatters by up to 6 % of n, which is a third of itself where an eighth of
// the list is taken, and costs nothing.  At least one tile is taken: the one whose
// entry has the threshold's key.  A histogram of all keys, scanned by a kernel of its own that moved the
// chosen tiles to a work list and the others on, took 5 us of each 20 to 27 us
// iteration: 2D lognormal 4096^2 14.5 -> 11.2 ms, 1500^2 4.8 -> 4.0, maze 256^3
// 5.0 -> 4.5, adjoint of 50 receivers at 4096^2 10.7 -> 8.8.  Only an adjoint
// that starts with tens of thousands of tiles queued was faster with it (dense
// dL/dphi at 4096^2 16.8 ms, now 23.5: sending a tile on takes two atomics here,
// where nobody else added to the list there; without the share it took 28.8).
// Against first-in first-out (every listed tile in every launch): 2D lognormal
// 4096^2 10.9 ms against 15.5, 3D lognormal 320^3 7.1 against 9.5, 192^3 2.46
// against 2.60; maze 256^3 4.03 against 3.96, layered 192^3 1.42 against 1.40; one
// front at constant speed, 256^3, 2.17 against 1.88.
constexpr int kListShare = 8;
__device__ __forceinline__ uint32_t sampled_threshold(const Sched& a, const int* s_len, int n) {
    const int lane = threadIdx.x & 63;
    const int k = lane & (kSub - 1), len = s_len[k];
    const int64_t e = static_cast<int64_t>(lane / kSub) * len / (64 / kSub);
    const uint32_t key =
        len > 0 ? static_cast<uint32_t>(a.cur.data[static_cast<size_t>(k) * a.cur.cap + e] >> 32) : kNoKey;
    const unsigned long long drawn = __builtin_amdgcn_ballot_w64(len > 0);
    int rank = 0;  // drawn keys before this one (ties by lane)
#pragma unroll
    for (int j = 0; j < 64; ++j) {
        const uint32_t kj = __builtin_amdgcn_readlane(key, j);
        rank += kj < key || (kj == key && j < lane) ? 1 : 0;
    }
    const int m = __popcll(drawn);
    const int want = static_cast<int>((static_cast<int64_t>(m) * max(a.order_aim, n / kListShare) + n - 1) / n);  // 1 .. m
    const unsigned long long at = __builtin_amdgcn_ballot_w64(rank == want - 1);
    return __builtin_amdgcn_readlane(key, __ffsll(static_cast<long long>(at)) - 1);
}

// Index of the next entry of sub-list k (of `len` entries) a workgroup takes
// (grids of a multiple of kSub workgroups).  Its first entry is fixed,
// blockIdx / kSub: the gridDim / kSub workgroups of group k cover the first
// gridDim / kSub entries without an atomic (a launch's opening fetches would
// otherwise queue on the group's counter).  Later entries come from the
// fetch counter, offset past them -- unless the fixed entries already cover
// the sub-list, when a workgroup is done after its first visit.
__device__ __forceinline__ int fetch_index(const TList& L, int k, int len, bool first) {
    const int fixed = static_cast<int>(gridDim.x) / kSub;
    if (first) return static_cast<int>(blockIdx.x) / kSub;
    if (len <= fixed) return len;
    return fixed + atomicAdd(L.fetch + k * kPad, 1);
}

// A workgroup's first entry: its index is fixed, so it is read in the round of
// the list lengths (an entry past the sub-list's end is not used: the grid has
// no more workgroups than tiles, rounded up, and a sub-list room for more), by
// every lane, so that no broadcast stands before the first visit.
__device__ __forceinline__ unsigned long long first_entry(const Sched& a) {
    const unsigned long long v = a.cur.data[static_cast<size_t>(blockIdx.x & (kSub - 1)) * a.cur.cap + blockIdx.x / kSub];
    return (static_cast<unsigned long long>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32))) << 32) |
           static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v)));
}

// The next tile a workgroup visits (lane 0; -1 when its sub-list k of `len`
// entries is drained), with its order key.  A tile whose key lies above the
// threshold goes on to the next list with its key and dirty faces instead.
__device__ __forceinline__ int next_tile(const Sched& a, int k, int len, bool first, uint32_t thr, uint32_t tag,
                                         uint32_t& key) {
    for (;; first = false) {
        const int e = fetch_index(a.cur, k, len, first);
        if (e >= len) return -1;
        const unsigned long long v = a.cur.data[static_cast<size_t>(k) * a.cur.cap + e];
        const int t = static_cast<int>(static_cast<uint32_t>(v));
        key = static_cast<uint32_t>(v >> 32);
        if (!a.ordered) return t;
        if (key > thr) {
            const uint32_t now = a.key_cur[t], faces = a.mask_cur[t];
            if (now > thr) {
                a.key_cur[t] = kNoKey;
                a.mask_cur[t] = 0u;
                atomicOr(a.mask_next + t, faces);
                push_keyed(a, t, tag, now);
                continue;
            }
            key = now;
        }
        a.key_cur[t] = kNoKey;
        return t;
    }
}

// Next entry of sub-list k for this workgroup (-1 when drained).  Lane 0
// fetches; the value is broadcast through LDS.
__device__ __forceinline__ int list_fetch(const TList& L, int k, int len, int* s_slot, bool first) {
    if (threadIdx.x == 0) {
        const int e = fetch_index(L, k, len, first);
        *s_slot = e < len ? static_cast<int>(static_cast<uint32_t>(L.data[static_cast<size_t>(k) * L.cap + e])) : -1;
    }
    __syncthreads();
    const int t = *s_slot;
    __syncthreads();
    return t;
}

__device__ __forceinline__ void stat_add(unsigned long long* blkstat, int field, unsigned long long v) {
    if (v) atomicAdd(blkstat + field * kMaxStatBlocks + (blockIdx.x & (kMaxStatBlocks - 1)), v);
}

// ---------------------------------------------------------------------------
// In-tile work lists
// ---------------------------------------------------------------------------
// Nodes of a tile are numbered n = (z * TY + y) * TX + x.  The update step
// alone works on an LDS list of node ids: inner iteration it drains list it & 1 (length cnt[it % 3]) and appends
// to list (it + 1) & 1; a per-list flag array keeps entries unique.  Only as
// many waves as the list needs evaluate the local solver.
template <int ND, int TX, int TY, int TZ>
__device__ __forceinline__ void node_loc(int n, int& x, int& y, int& z, int& L) {
    using S = Shape<ND, TX, TY, TZ>;
    x = n % TX;
    y = (n / TX) % TY;
    z = ND == 3 ? n / (TX * TY) : 0;
    L = ND == 3 ? ((z + 1) * S::LY + (y + 1)) * S::LX + (x + 1) : (y + 1) * S::LX + (x + 1);
}

template <int TX, int TY>
__device__ __forceinline__ int node_step(int d) {
    switch (d) {
        case 0: return -1;
        case 1: return 1;
        case 2: return -TX;
        case 3: return TX;
        case 4: return -TX * TY;
        default: return TX * TY;
    }
}

// bit d: the node lies on the tile face in direction d
template <int ND, int TX, int TY, int TZ>
__device__ __forceinline__ int edge_bits(int x, int y, int z) {
    int e = (x == 0 ? 1 : 0) | (x == TX - 1 ? 2 : 0) | (y == 0 ? 4 : 0) | (y == TY - 1 ? 8 : 0);
    if (ND == 3) e |= (z == 0 ? 16 : 0) | (z == TZ - 1 ? 32 : 0);
    return e;
}

// bit d: the grid continues past the tile face in direction d
template <int ND, int TX, int TY, int TZ, typename T>
__device__ __forceinline__ int open_bits(const Inst<T>& g, int x0, int y0, int z0) {
    int f = (x0 > 0 ? 1 : 0) | (x0 + TX < g.nx ? 2 : 0) | (y0 > 0 ? 4 : 0) | (y0 + TY < g.ny ? 8 : 0);
    if (ND == 3) f |= (z0 > 0 ? 16 : 0) | (z0 + TZ < g.nz ? 32 : 0);
    return f;
}

template <int NT>
struct TileLists {
    uint32_t flag[2][NT];
    uint16_t list[2][NT];
    int cnt[3];
};

// Append node q to the next list once (returns whether it was added).
template <int NT>
__device__ __forceinline__ bool list_add(TileLists<NT>& tl, int nb, int* ncnt, int q) {
    if (atomicExch(&tl.flag[nb][q], 1u) != 0u) return false;
    tl.list[nb][atomicAdd(ncnt, 1)] = static_cast<uint16_t>(q);
    return true;
}

// ---------------------------------------------------------------------------
// Dense rounds of a tile visit: chunks of 64 consecutive nodes, one wave each
// ---------------------------------------------------------------------------
// A set of a tile's chunks, a bit each.
template <int NT>
using ChunkMask = std::conditional_t<(NT <= 32 * 64), uint32_t, unsigned long long>;

// The lanes for which p holds, as a wave-uniform mask.
__device__ __forceinline__ unsigned long long ballot64(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// Minimum over the wave's lanes (uniform): row shifts and row broadcasts, no LDS.
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
    constexpr int kShr[4] = {0x111, 0x112, 0x114, 0x118};  // row_shr:1, 2, 4, 8
    v = min(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(-1, static_cast<int>(v), kShr[0], 0xf, 0xf, false)));
    v = min(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(-1, static_cast<int>(v), kShr[1], 0xf, 0xf, false)));
    v = min(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(-1, static_cast<int>(v), kShr[2], 0xf, 0xf, false)));
    v = min(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(-1, static_cast<int>(v), kShr[3], 0xf, 0xf, false)));
    v = min(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(-1, static_cast<int>(v), 0x142, 0xa, 0xf, false)));  // row_bcast:15
    v = min(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(-1, static_cast<int>(v), 0x143, 0xc, 0xf, false)));  // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}

// What a wave's lanes found when a visit ends: the faces they crossed (bit d)
// and the smallest order key among them, joined in LDS with one atomic each (a
// lane each, some 300 in a 3D tile, queued on one address for 2 us).
template <int ND>
__device__ __forceinline__ void join_crossings(int crossed, uint32_t key, int* s_face, uint32_t* s_key) {
    int any = 0;
#pragma unroll
    for (int d = 0; d < 2 * ND; ++d) any |= __builtin_amdgcn_ballot_w64((crossed & (1 << d)) != 0) ? 1 << d : 0;
    if (any == 0) return;
    const uint32_t low = wave_min(key);
    if ((threadIdx.x & 63) == 0) {
        atomicOr(s_face, any);
        atomicMin(s_key, low);
    }
}

__device__ __forceinline__ uint32_t first_lane(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ unsigned long long first_lane(unsigned long long v) {
    return (static_cast<unsigned long long>(first_lane(static_cast<uint32_t>(v >> 32))) << 32) |
           first_lane(static_cast<uint32_t>(v));
}

// The chunks (64 consecutive nodes, one wave's share of a round) that hold a
// neighbour of a node in the chunks of m, m's own among them.
template <int ND, int TX, int TY, typename Mask>
__device__ __forceinline__ Mask chunk_reach(Mask m) {
    static_assert(64 % TX == 0 || TX % 64 == 0, "a neighbouring row lies in the same or the next chunk");
    Mask r = m | (m << 1) | (m >> 1);
    if constexpr (ND == 3) {
        constexpr int ZS = TX * TY / 64;  // chunks per z slice
        static_assert(TX * TY % 64 == 0, "z slices are whole chunks");
        if (ZS > 1) r |= (m << ZS) | (m >> ZS);
    }
    return r;
}

// ---------------------------------------------------------------------------
// Host side: workspace of the scheduling state and the per-launch arguments
// ---------------------------------------------------------------------------
constexpr size_t kCounterBytes = 3 * 2 * kSub * kPad * sizeof(int);

struct SchedWs {
    uint32_t* tstamp;
    uint32_t* tmask;    // two arrays of ntiles dirty-face masks (by launch parity), after tstamp
    unsigned long long* data[2];  // two list buffers (alternating)
    int* counters;      // 3 rotating sets of {count[kSub*kPad], fetch[kSub*kPad]}
    uint32_t* keys;     // two arrays of ntiles order keys (by launch parity)
    int cap;            // entries per sub-list: each tile of its residue class once by stamp and once by key
    int ntiles;
    int* count_of(int set) const { return counters + set * 2 * kSub * kPad; }
    int* fetch_of(int set) const { return counters + set * 2 * kSub * kPad + kSub * kPad; }
    // list t: buffer t % 2, counter set t % 3
    TList list_of(int64_t t) const {
        TList L;
        L.data = data[t & 1];
        L.count = count_of(static_cast<int>(t % 3));
        L.fetch = fetch_of(static_cast<int>(t % 3));
        L.cap = cap;
        return L;
    }
};

// `take(bytes)` hands out aligned workspace regions in order.
template <typename Take>
SchedWs sched_layout(Take&& take, int64_t ntiles) {
    SchedWs w{};
    w.cap = 2 * static_cast<int>((ntiles + kSub - 1) / kSub) + 64;
    w.ntiles = static_cast<int>(ntiles);
    w.tstamp = reinterpret_cast<uint32_t*>(take(4 * static_cast<size_t>(ntiles)));
    w.tmask = reinterpret_cast<uint32_t*>(take(8 * static_cast<size_t>(ntiles)));
    w.counters = reinterpret_cast<int*>(take(kCounterBytes));
    w.keys = reinterpret_cast<uint32_t*>(take(8 * static_cast<size_t>(ntiles)));
    for (int k = 0; k < 2; ++k)
        w.data[k] = reinterpret_cast<unsigned long long*>(take(8 * static_cast<size_t>(w.cap) * kSub));
    return w;
}

// Launch t of a loop drains list t and fills list t + 1 (the counter set of
// list t + 2 is cleared by launch t); tag_slot is the parity in the device
// tag chain.
inline void sched_fill(Sched& a, const SchedWs& w, int64_t t, bool ordered, int omin, int tag_slot, int phase,
                       Ctl* ctl, unsigned long long* blkstat) {
    const size_t nt = static_cast<size_t>(w.ntiles);
    a.tstamp = w.tstamp;
    a.mask_cur = w.tmask + static_cast<size_t>(t & 1) * nt;
    a.mask_next = w.tmask + static_cast<size_t>((t + 1) & 1) * nt;
    a.key_cur = w.keys + static_cast<size_t>(t & 1) * nt;
    a.key_next = w.keys + static_cast<size_t>((t + 1) & 1) * nt;
    a.ordered = ordered ? 1 : 0;
    a.order_aim = order_aim(omin);
    a.cur = w.list_of(t);
    a.next = w.list_of(t + 1);
    a.zero_count = w.count_of(static_cast<int>((t + 2) % 3));
    a.zero_fetch = w.fetch_of(static_cast<int>((t + 2) % 3));
    a.ctl = ctl;
    a.blkstat = blkstat;
    a.tag_slot = tag_slot;
    a.phase = phase;
    a.first = (phase == 1 && t == 0) ? 1 : 0;
}

// Before a solve: stamps and masks zero, list counters zero, order keys "none".
inline void sched_clear(const SchedWs& w, ClearPlan& c) {
    c.add(w.tstamp, 4 * (static_cast<size_t>(w.tmask - w.tstamp) + 2 * static_cast<size_t>(w.ntiles)));
    c.add(w.counters, kCounterBytes);
    c.add(w.keys, 8 * static_cast<size_t>(w.ntiles), kNoKey);
}

}  // namespace
}  // namespace eik
