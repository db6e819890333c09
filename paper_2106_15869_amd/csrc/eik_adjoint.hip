// Adjoint of the converged eikonal solve on gfx950: dL/dF for a loss L(phi).
//
// At the solution every reached non-source node i with F_i > 0 satisfies
// sum_{k in U_i} w_ik^2 = H_i^2 over its upwind axes U_i (a_k < phi_i), with
// w_ik = phi_i - a_k and H_i = h / F_i (Eq 4 / Eq 6 at the fixed point).
// Differentiating gives dphi = M dphi + D dF with M_{i,j_k} = w_ik / W_i,
// W_i = sum_k w_ik, D_i = -H_i^2 / (F_i W_i).  Hence dL/dF = D lambda with
//     lambda = dL/dphi + M^T lambda,
// a triangular system in causal order.
//
//   k_adj_prep   tile by tile: the upwind neighbour on each axis (lower index
//                on a tie), the weights c_ik = w_ik / W_i and D_i; written as
//                what the recurrence pulls, tile-major: for node j and
//                direction d the weight on j of its neighbour there, 0 where j
//                is not upwind of it.  Tiles holding a nonzero dL/dphi are
//                queued.
//   Grids of a batch are tiled back to back (see eik_tile.hpp); every kernel
//   looks up the instance of the tile it works on.
//   k_adj_tile   tile work queues (eik_sched.hpp): a persistent workgroup
//                stages lambda of a tile plus halo in LDS, the pulled weights
//                in registers, and recomputes
//                lambda_j = g_j + sum_d pull_jd lambda_{j+d}
//                in dense rounds (see remedy_visit in eik_tile.hip; 900 x 1100
//                4.4 -> 1.8 ms, 192^3 3.6 -> 1.8 ms against an LDS list of
//                nodes and weights staged as stored) until nothing changes; a node on a tile face whose upwind neighbour
//                lies across it marks that face dirty in the neighbour tile
//                and queues it.
//                lambda starts at 0 and the tiles holding a nonzero dL/dphi
//                start queued, so every node with g_j != 0 changes on its
//                first evaluation and passes its value on, also across a face.
//                Tiles are taken in decreasing arrival time (order keys of
//                -phi), the direction in which lambda flows.  The system is
//                triangular, so the iteration ends at its unique solution
//                whatever the order.
//   k_adj_final  dense: dL/dF = D lambda (0 at sources and unreached nodes).
#include <utility>
#include <vector>

#include "eik_device.hpp"
#include "eik_host.hpp"
#include "eik_seglist.hpp"
#include "eik_batch.hpp"
#include "eik_sched.hpp"
#include "eik_tile.hpp"
#include "eik_walk.hpp"

namespace eik {

namespace {

// stencil byte: bit d set if the node's upwind neighbour on the axis of
// direction d (-x, +x, -y, +y, -z, +z) lies there; 0 for sources, barriers and
// unreached nodes

template <typename T>
struct AdjIter : Sched {
    const T* phi;
    const T* g;      // dL/dphi
    T* lam;
    const uint8_t* up;  // stencil bytes, tile-major
    const T* pull;      // pulled weights, tile-major: [tile][direction][node]
};

// A tile's nodes in the tile-major arrays: the nodes of the grid, tile after
// tile, x fastest within one.  A tile at the grid's end is cut there, so the
// arrays have an entry per node: with whole tiles a 1 x 4096 x 4096 grid had
// eight (3.2 GB of weights in place of 400 MB).
struct TileBlock {
    int first;       // entry of the tile's first node
    int bx, by, bz;  // its extents
    __device__ __forceinline__ int nodes() const { return bx * by * bz; }
    // in-tile position of a node, clamped into the tile
    __device__ __forceinline__ int at(int x, int y, int z) const {
        return (min(z, bz - 1) * by + min(y, by - 1)) * bx + min(x, bx - 1);
    }
};
template <int ND, int TX, int TY, int TZ, typename T>
__device__ __forceinline__ TileBlock tile_block(const Inst<T>& g, int x0, int y0, int z0) {
    TileBlock b;
    b.bx = min(TX, g.nx - x0);
    b.by = min(TY, g.ny - y0);
    b.bz = ND == 3 ? min(TZ, g.nz - z0) : 1;
    b.first = g.node_base + (z0 * g.ny + b.bz * y0) * g.nx + b.bz * b.by * x0;
    return b;
}

// ---------------------------------------------------------------------------
// One workgroup per tile: phi with a halo of two nodes in LDS, from it the
// stencil of the tile's nodes and of a halo of one, from that the weights each
// node pulls.  Also lambda = 0 and the initial list: tiles holding a nonzero
// dL/dphi (all nodes to recompute), keyed by the largest arrival time among
// those nodes.  Written once, the pulled weights spare every visit the staging
// of three weights and a stencil byte per node and halo node (13 bytes each,
// at a stride of 12).
template <typename T, int ND, int TX, int TY, int TZ>
__global__ __launch_bounds__(kBlock) void k_adj_prep(AdjIter<T> a, BatchGeom<T> bg, const T* __restrict__ F, uint8_t* up,
                                                     T* pull, T* D) {
    using S = Shape<ND, TX, TY, TZ>;
    constexpr int PX = TX + 4, PY = TY + 4, PZ = ND == 3 ? TZ + 4 : 1, PN = PX * PY * PZ;
    __shared__ T sphi[PN];
    __shared__ T sw[ND][S::NL];      // weights by axis (x, y, z)
    __shared__ uint8_t sup[S::NL];   // stencil bytes
    __shared__ uint32_t s_key;
    const T inf = pos_inf<T>();
    for (int t = blockIdx.x; t < bg.ntiles; t += gridDim.x) {
        const Inst<T> I = inst_of(bg, t);
        const int lt = t - I.tile_base;
        const int x0 = (lt % I.ntx) * TX, y0 = ((lt / I.ntx) % I.nty) * TY;
        const int z0 = ND == 3 ? (lt / (I.ntx * I.nty)) * TZ : 0;
        auto node = [&](int x, int y, int z) {
            const int cx = min(max(x, 0), I.nx - 1), cy = min(max(y, 0), I.ny - 1), cz = min(max(z, 0), I.nz - 1);
            return I.node_base + (cz * I.ny + cy) * I.nx + cx;
        };
        auto inside = [&](int x, int y, int z) {
            return x >= 0 && x < I.nx && y >= 0 && y < I.ny && z >= 0 && z < I.nz;
        };
        if (threadIdx.x == 0) s_key = kNoKey;
        for (int q = threadIdx.x; q < PN; q += kBlock) {
            const int x = x0 + q % PX - 2, y = y0 + (q / PX) % PY - 2, z = ND == 3 ? z0 + q / (PX * PY) - 2 : 0;
            const T p = a.phi[node(x, y, z)];
            sphi[q] = inside(x, y, z) ? p : inf;
        }
        __syncthreads();
        for (int q = threadIdx.x; q < S::NL; q += kBlock) {
            const int lx = q % S::LX, ly = (q / S::LX) % S::LY, lz = ND == 3 ? q / (S::LX * S::LY) : 0;
            const int x = x0 + lx - 1, y = y0 + ly - 1, z = ND == 3 ? z0 + lz - 1 : 0;
            const int c = ((ND == 3 ? lz + 1 : 0) * PY + ly + 1) * PX + lx + 1;
            const bool ok = inside(x, y, z);
            const T f = F[node(x, y, z)];
            const T p = sphi[c];
            uint8_t u = 0;
            T w[3] = {T(0), T(0), T(0)};
            T W = T(0);
            if (ok && p < inf && f > T(0)) {
                constexpr int st[3] = {1, PX, PX * PY};
#pragma unroll
                for (int k = 0; k < ND; ++k) {
                    const T lo = sphi[c - st[k]], hi = sphi[c + st[k]];  // +inf outside the grid
                    T v = inf;
                    int side = -1;
                    if (lo < v) {
                        v = lo;
                        side = 0;
                    }
                    if (hi < v) {
                        v = hi;
                        side = 1;
                    }
                    if (side >= 0 && v < p) {
                        u |= static_cast<uint8_t>(1u << (2 * k + side));
                        // per-axis spacing weighs axis k by 1 / spacing^2 (axis k = x, y, z
                        // is dims entry ND - 1 - k)
                        const T dk = I.d[ND - 1 - k];
                        w[k] = I.aniso ? (p - v) / (dk * dk) : p - v;
                        W = W + w[k];
                    }
                }
            }
            T d = T(0);
            if (u && W > T(0)) {
                if (I.aniso) {
                    d = -T(1) / (f * f * f * W);
                } else {
                    const T Hh = I.h / f;
                    d = -(Hh * Hh) / (f * W);
                }
#pragma unroll
                for (int k = 0; k < ND; ++k) w[k] = w[k] / W;
            } else {
                u = 0;
#pragma unroll
                for (int k = 0; k < ND; ++k) w[k] = T(0);
            }
            sup[q] = u;
#pragma unroll
            for (int k = 0; k < ND; ++k) sw[k][q] = w[k];
            const bool owned = lx >= 1 && lx <= TX && ly >= 1 && ly <= TY && (ND == 2 || (lz >= 1 && lz <= TZ));
            if (ok && owned) D[node(x, y, z)] = d;
        }
        __syncthreads();
        bool nz = false;
        const TileBlock tb = tile_block<ND, TX, TY, TZ>(I, x0, y0, z0);
        T* const tile_pull = pull + static_cast<size_t>(tb.first) * (2 * ND);
        for (int n = threadIdx.x; n < S::NT; n += kBlock) {
            int x, y, z, L;
            node_loc<ND, TX, TY, TZ>(n, x, y, z, L);
            if (!inside(x0 + x, y0 + y, z0 + z)) continue;
            const int q = tb.at(x, y, z);
            up[tb.first + q] = sup[L];
#pragma unroll
            for (int d = 0; d < 2 * ND; ++d) {
                // the neighbour in direction d pushes to this node if its upwind
                // neighbour on that axis lies in the opposite direction
                const int p = L + lds_offset<ND, TX, TY, TZ>(d);
                tile_pull[d * tb.nodes() + q] = (sup[p] >> (d ^ 1)) & 1u ? sw[d >> 1][p] : T(0);
            }
            const int i = node(x0 + x, y0 + y, z0 + z);
            a.lam[i] = T(0);
            if (a.g[i] != T(0)) {
                nz = true;
                atomicMin(&s_key, order_key(-a.phi[i]));
            }
        }
        if (__syncthreads_or(nz) && threadIdx.x == 0) {
            a.mask_next[t] = kAllFaces;
            push_keyed(a, t, 1u, s_key);
        }
        __syncthreads();
    }
}

// A source has no stencil: nothing pulls from it, and it has no gradient.
template <typename T, int ND, int TX, int TY, int TZ>
__global__ void k_adj_mark_sources(BatchGeom<T> bg, SrcBatch<T> b, uint8_t* up, T* pull, T* D) {
    const int k = threadIdx.x;
    if (k >= b.count) return;
    const Inst<T> g = bg.ninst == 1 ? bg.one : bg.table[b.inst[k]];
    const int i = b.idx[k] - g.node_base;
    const int x = i % g.nx, y = (i / g.nx) % g.ny, z = i / (g.nx * g.ny);
    D[b.idx[k]] = T(0);
    auto block = [&](int X, int Y, int Z) {
        return tile_block<ND, TX, TY, TZ>(g, X / TX * TX, Y / TY * TY, ND == 3 ? Z / TZ * TZ : 0);
    };
    auto pos = [&](const TileBlock& tb, int X, int Y, int Z) { return tb.at(X % TX, Y % TY, ND == 3 ? Z % TZ : 0); };
    const TileBlock own = block(x, y, z);
    up[own.first + pos(own, x, y, z)] = 0;
    constexpr int dx[6] = {-1, 1, 0, 0, 0, 0}, dy[6] = {0, 0, -1, 1, 0, 0}, dz[6] = {0, 0, 0, 0, -1, 1};
    for (int d = 0; d < 2 * ND; ++d) {
        const int X = x + dx[d], Y = y + dy[d], Z = z + dz[d];
        if (X < 0 || X >= g.nx || Y < 0 || Y >= g.ny || Z < 0 || Z >= g.nz) continue;
        const TileBlock tb = block(X, Y, Z);
        // seen from there the source lies the other way
        pull[static_cast<size_t>(tb.first) * (2 * ND) + (d ^ 1) * tb.nodes() + pos(tb, X, Y, Z)] = T(0);
    }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_adj_final(int n, const T* __restrict__ D,
                                                      const T* __restrict__ lam, T* __restrict__ out) {
    for (int64_t i = blockIdx.x * kBlock + threadIdx.x; i < n; i += flat_step(gridDim.x)) out[i] = D[i] * lam[i];
}

// Whether a recomputed lambda differs from the one it replaces: by its bits, so
// that a NaN (from dL/dphi, or from inf - inf in a sum) recomputed from the
// same values is no change.  A changed chunk is evaluated again, so a NaN that
// differed from itself would keep its tile listed for ever.  The system is
// acyclic and a sum of the same values has the same bits, so the iteration
// ends as it does for numbers.  (One instruction, like the comparison of the
// values; testing for two NaNs beside it cost 4 % of a 192^3 training step.)
__device__ __forceinline__ bool lambda_changed(float now, float was) {
    return __float_as_uint(now) != __float_as_uint(was);
}
__device__ __forceinline__ bool lambda_changed(double now, double was) {
    return __double_as_longlong(now) != __double_as_longlong(was);
}

// Resident workgroups per CU: six for 8^3 float tiles, so that all 1536
// default workgroups of a launch are resident at once.  Others unconstrained.
template <int ND, int NPT, typename T>
constexpr int adj_blocks_per_cu() {
    return ND == 3 && NPT == 2 && sizeof(T) == 4 ? 6 : 1;
}

template <typename T, int ND, int TX, int TY, int TZ>
__global__ __launch_bounds__(kBlock, (adj_blocks_per_cu<ND, Shape<ND, TX, TY, TZ>::NPT, T>())) void k_adj_tile(
    AdjIter<T> a, BatchGeom<T> bg, int inner) {
    using S = Shape<ND, TX, TY, TZ>;
    using Mask = ChunkMask<S::NT>;
    constexpr int WAVES = kBlock / 64;
    // LDS step from a lane's node of one round to the next
    constexpr int RSTEP = ND == 2 ? (kBlock / TX) * S::SY : (kBlock / (TX * TY)) * S::SZ;
    static_assert(S::NT % kBlock == 0 && kBlock % TX == 0 && (ND == 2 || kBlock % (TX * TY) == 0),
                  "whole rounds of whole rows (slices)");
    static_assert(S::NPT <= 2, "a lane holds every neighbour value of its nodes");
    __shared__ T slam[S::NL];
    __shared__ Mask s_act[2 * WAVES];  // each wave's chunks that changed in an iteration (by parity)
    __shared__ int s_len[kSub];
    __shared__ int s_slot;
    __shared__ int s_face;
    __shared__ uint32_t s_mask, s_key, s_kmin;
    const uint32_t ntag = launch_tag(a);
    const unsigned long long e0 = first_entry(a);
    const int n = list_open(a, s_len);
    launch_stats(a, n);
    const int k = blockIdx.x & (kSub - 1);
    const int len = s_len[k];
    if (static_cast<int>(blockIdx.x) / kSub >= len) return;  // no first entry: none at all
    const bool all = !a.ordered || n <= a.order_aim;  // the launch takes every tile listed
    const uint32_t thr = !all && threadIdx.x < 64 ? sampled_threshold(a, s_len, n) : kNoKey;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool lane0 = (threadIdx.x & 63) == 0;
    int nx_, ny_, nz_, L0;
    node_loc<ND, TX, TY, TZ>(threadIdx.x, nx_, ny_, nz_, L0);
    unsigned long long visits = 0;
    for (;;) {
        int t;
        if (visits == 0 && all) {
            t = static_cast<int>(static_cast<uint32_t>(e0));
            if (threadIdx.x == 0) {
                if (a.ordered) a.key_cur[t] = kNoKey;  // the tile leaves the list
                s_key = static_cast<uint32_t>(e0 >> 32);
            }
        } else {
            if (threadIdx.x == 0) s_slot = next_tile(a, k, len, visits == 0, thr, ntag, s_key);
            __syncthreads();
            t = s_slot;
            if (t < 0) break;
        }
        if (threadIdx.x == 0) {
            // written by the previous launch; no writer during this one
            s_mask = a.mask_cur[t];
            a.mask_cur[t] = 0u;
            s_kmin = kNoKey;
            s_face = 0;
        }
        ++visits;
        const Inst<T> g = inst_of(bg, t);
        const int lt = t - g.tile_base;
        const int tx = lt % g.ntx, ty = (lt / g.ntx) % g.nty, tz = lt / (g.ntx * g.nty);
        const int x0 = tx * TX, y0 = ty * TY, z0 = tz * (ND == 3 ? TZ : 1);
        const int open = open_bits<ND, TX, TY, TZ>(g, x0, y0, z0);
        // lambda with the halo (0 outside) to LDS; the nodes' pulled weights,
        // dL/dphi, stencil bytes and (on open faces) arrival times to
        // registers: addresses are clamped into the grid so every global load
        // of a lane is issued before its first LDS store
        T c[S::NPT][2 * ND], gv[S::NPT], ph[S::NPT], cur[S::NPT], old[S::NPT];
        uint32_t u[S::NPT];
        bool ok[S::NPT];
        int G[S::NPT], E[S::NPT];
        {
            constexpr int NIT = (S::NL + kBlock - 1) / kBlock;
            T vl[NIT];
            bool in[NIT];
#pragma unroll
            for (int j = 0; j < NIT; ++j) {
                const int q = min(static_cast<int>(threadIdx.x) + j * kBlock, S::NL - 1);
                const int lx = q % S::LX, ly = (q / S::LX) % S::LY, lz = q / (S::LX * S::LY);
                const int gx = x0 + lx - 1, gy = y0 + ly - 1, gz = ND == 3 ? z0 + lz - 1 : 0;
                in[j] = gx >= 0 && gx < g.nx && gy >= 0 && gy < g.ny && gz >= 0 && gz < g.nz;
                const int cx = min(max(gx, 0), g.nx - 1), cy = min(max(gy, 0), g.ny - 1);
                const int cz = min(max(gz, 0), g.nz - 1);
                vl[j] = a.lam[g.node_base + (cz * g.ny + cy) * g.nx + cx];
            }
            const TileBlock tb = tile_block<ND, TX, TY, TZ>(g, x0, y0, z0);
            const T* const tile_pull = a.pull + static_cast<size_t>(tb.first) * (2 * ND);
#pragma unroll
            for (int r = 0; r < S::NPT; ++r) {
                int x, y, z, L;
                node_loc<ND, TX, TY, TZ>(threadIdx.x + r * kBlock, x, y, z, L);
                const int q = tb.at(x, y, z);
                ok[r] = x0 + x < g.nx && y0 + y < g.ny && z0 + z < g.nz;
                E[r] = edge_bits<ND, TX, TY, TZ>(x, y, z) & open;
                G[r] = g.node_base + (min(z0 + z, g.nz - 1) * g.ny + min(y0 + y, g.ny - 1)) * g.nx + min(x0 + x, g.nx - 1);
                gv[r] = a.g[G[r]];
                u[r] = a.up[tb.first + q];
                ph[r] = T(0);
                if (E[r]) ph[r] = a.phi[G[r]];
#pragma unroll
                for (int d = 0; d < 2 * ND; ++d) c[r][d] = tile_pull[d * tb.nodes() + q];
            }
#pragma unroll
            for (int j = 0; j < NIT; ++j) {
                const int q = threadIdx.x + j * kBlock;
                if (q < S::NL) slam[q] = in[j] ? vl[j] : T(0);
            }
        }
        __syncthreads();
        // chunks to recompute: every one with a node in the grid on a first
        // visit, else those with a node on a face whose neighbour tile changed
        const uint32_t m = s_mask;
        Mask todo = 0;
#pragma unroll
        for (int r = 0; r < S::NPT; ++r) {
            cur[r] = old[r] = slam[L0 + r * RSTEP];
            if (ballot64(ok[r] && ((m & kAllFaces) || (E[r] & static_cast<int>(m)))))
                todo |= Mask(1) << (r * WAVES + wave);
        }
        bool pending = false;
        int it = 0;
        for (;; ++it) {
            Mask act[WAVES] = {};
            if (it > 0) {
#pragma unroll
                for (int w = 0; w < WAVES; ++w) act[w] = s_act[((it - 1) & 1) * WAVES + w];
            }
            T l[S::NPT][2 * ND];
#pragma unroll
            for (int r = 0; r < S::NPT; ++r) {
                load_nb<T, ND, TX, TY, TZ>(slam, L0 + r * RSTEP, l[r]);
#pragma unroll
                for (int d = 0; d < 2 * ND; ++d) asm volatile("" : "+v"(l[r][d]));
            }
            if (it > 0) {
                Mask ch = 0;
#pragma unroll
                for (int w = 0; w < WAVES; ++w) ch |= act[w];
                ch = first_lane(ch);
                if (ch == 0) break;
                todo = chunk_reach<ND, TX, TY>(ch);
            }
            if (it == inner) {
                pending = true;
                break;
            }
            Mask changed = 0;
#pragma unroll
            for (int r = 0; r < S::NPT; ++r) {
                const Mask bit = Mask(1) << (r * WAVES + wave);
                if (!(todo & bit)) continue;
                // in direction order; a direction that is not pulled adds 0
                T v = gv[r];
#pragma unroll
                for (int d = 0; d < 2 * ND; ++d) v = v + c[r][d] * (c[r][d] != T(0) ? l[r][d] : T(0));
                const bool diff = ok[r] && lambda_changed(v, cur[r]);
                cur[r] = diff ? v : cur[r];
                slam[L0 + r * RSTEP] = cur[r];  // (only this lane writes it)
                if (ballot64(diff)) changed |= bit;
            }
            if (lane0) s_act[(it & 1) * WAVES + wave] = changed;
            __syncthreads();
        }
        // write back what changed; across an open face it reaches the node's
        // upwind neighbour
        int fm = 0;
        uint32_t kmin = kNoKey;
#pragma unroll
        for (int r = 0; r < S::NPT; ++r) {
            if (!lambda_changed(cur[r], old[r])) continue;
            a.lam[G[r]] = cur[r];
            const int f = static_cast<int>(u[r]) & E[r];
            if (f) {
                fm |= f;
                kmin = min(kmin, order_key(-ph[r]));
            }
        }
        join_crossings<ND>(fm, kmin, &s_face, &s_kmin);
        __syncthreads();
        if (threadIdx.x < 7) {
            const int d = threadIdx.x;
            const int fmask = s_face;
            const uint32_t key = s_kmin;
            if (d == 6) {
                if (pending) {
                    atomicOr(a.mask_next + t, kAllFaces);
                    push_keyed(a, t, ntag, min(key, s_key));
                }
            } else if (d < 2 * ND && (fmask & (1 << d))) {
                const int tn = neighbour_tile(g, t, d);
                atomicOr(a.mask_next + tn, 1u << (d ^ 1));
                push_keyed(a, tn, ntag, key);
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0 && visits) stat_add(a.blkstat, SF_VISITS3, visits);
}

struct AdjWs {
    Ctl* ctl;
    unsigned long long* blkstat;
    uint8_t* up;
    void* pull;
    void* D;
    void* lam;
    SchedWs q;
    void* table;
    int* tile_inst;
    size_t bytes;
};

TileCfg adj_tile(int nd) { return nd == 2 ? TileCfg{16, 16, 1} : TileCfg{8, 8, 8}; }

AdjWs adj_layout(char* base, const Batch& b, size_t esz) {
    AdjWs w{};
    size_t off = 0;
    auto take = [&](size_t n) {
        char* p = base ? base + off : nullptr;
        off = align_up(off + n, 256);
        return p;
    };
    const size_t n = static_cast<size_t>(b.n);
    w.ctl = reinterpret_cast<Ctl*>(take(sizeof(Ctl)));
    w.blkstat = reinterpret_cast<unsigned long long*>(take(8 * static_cast<size_t>(kStatFields) * kMaxStatBlocks));
    w.up = reinterpret_cast<uint8_t*>(take(n));
    w.pull = take(2 * static_cast<size_t>(b.nd) * esz * n);
    w.D = take(esz * n);
    w.lam = take(esz * n);
    w.q = sched_layout(take, b.ntiles);
    if (b.inst.size() > 1) {
        w.table = take((esz == 8 ? sizeof(Inst<double>) : sizeof(Inst<float>)) * b.inst.size());
        w.tile_inst = reinterpret_cast<int*>(take(4 * static_cast<size_t>(b.ntiles)));
    }
    w.bytes = off;
    return w;
}

template <typename T, int ND, int TX, int TY, int TZ>
eik_status adj_run(const Batch& b, const T* F, const T* phi, const T* g, T* out, const eik_options& o, char* ws,
                   hipStream_t s, eik_stats* st) {
    const bool async = (o.flags & EIK_FLAG_ASYNC) != 0;
    const bool ordered = (o.flags & EIK_FLAG_FIFO_REMEDY) == 0;
    AdjWs w = adj_layout(ws, b, sizeof(T));
    const int64_t cap = o.max_iters > 0 ? o.max_iters : 4 * b.n + 64;
    const int inner = o.inner_iters > 0 ? o.inner_iters : 4 * (TX + TY + TZ);
    const int tiles = static_cast<int>(std::min<int64_t>(b.ntiles, 1 << 16));
    const size_t blk_bytes = 8 * static_cast<size_t>(kStatFields) * kMaxStatBlocks;
    int64_t launched = 0;
    Profiler prof;
    prof.start((o.flags & EIK_FLAG_PROFILE) != 0, s);

    BatchGeom<T> G;
    HIP_TRY(timed(prof, EIK_KERNEL_OTHER, [&] { return upload_batch_geom<T>(b, w.table, w.tile_inst, s, G, launched); }));
    ClearPlan clear;
    clear.ctl = w.ctl;
    clear.add(w.blkstat, blk_bytes);
    sched_clear(w.q, clear);
    HIP_TRY(timed(prof, EIK_KERNEL_OTHER, [&] { return launch_clear(clear, s); }));
    // launch t drains list t and fills list t + 1; the seeding fills list 0
    // with tag 1 and the tag chain starts at tag[0] = 1 (claims 2, 3, ...)
    auto iter_args = [&](int64_t t) {
        AdjIter<T> a{};
        sched_fill(a, w.q, t, ordered, order_min_of(ND, o.order_min), static_cast<int>(t & 1), 1, w.ctl, w.blkstat);
        if (!async) a.mail = host_slots().mail + (t & (HostSlots::kMail - 1));
        a.phi = phi;
        a.g = g;
        a.lam = static_cast<T*>(w.lam);
        a.up = w.up;
        a.pull = static_cast<const T*>(w.pull);
        return a;
    };
    {
        AdjIter<T> a0 = iter_args(0);
        a0.next = w.q.list_of(0);
        a0.mask_next = w.q.tmask;  // read by launch 0
        a0.key_next = w.q.keys;
        HIP_TRY(timed(prof, EIK_KERNEL_OTHER, [&] {
            hipLaunchKernelGGL((k_adj_prep<T, ND, TX, TY, TZ>), dim3(tiles), dim3(kBlock), 0, s, a0, G, F, w.up,
                               static_cast<T*>(w.pull), static_cast<T*>(w.D));
            return hipGetLastError();
        }));
        launched += 2;
    }
    for (size_t q = 0; q < b.src.size(); q += kMaxSrcBatch) {
        SrcBatch<T> sb{};
        sb.count = static_cast<int>(std::min<size_t>(kMaxSrcBatch, b.src.size() - q));
        for (int j = 0; j < sb.count; ++j) {
            sb.idx[j] = b.src[q + j].first;
            sb.inst[j] = b.src_inst[q + j];
        }
        HIP_TRY(timed(prof, EIK_KERNEL_OTHER, [&] {
            hipLaunchKernelGGL((k_adj_mark_sources<T, ND, TX, TY, TZ>), dim3(1), dim3(kMaxSrcBatch), 0, s, G, sb, w.up,
                               static_cast<T*>(w.pull), static_cast<T*>(w.D));
            return hipGetLastError();
        }));
        ++launched;
    }
    auto step = [&](int64_t t) {
        const AdjIter<T> a = iter_args(t);
        return timed(prof, EIK_KERNEL_ADJOINT, [&] {
            hipLaunchKernelGGL((k_adj_tile<T, ND, TX, TY, TZ>), dim3(workgroups_of(ND, o.workgroups, b.ntiles)), dim3(kBlock), 0,
                               s, a, G, inner);
            return hipGetLastError();
        });
    };
    int64_t nl = 0;
    auto counts = [&](int64_t t) { return w.q.count_of(static_cast<int>(t % 3)); };
    eik_status rc = async ? run_loop(step, counts, kSub * kPad, cap, true, s, &nl, w.ctl)
                          : run_tile_loop(step, counts, kSub * kPad, 0, cap, s, &nl);
    launched += nl;
    HIP_TRY(timed(prof, EIK_KERNEL_OTHER, [&] {
        hipLaunchKernelGGL(k_adj_final<T>, dim3(flat_blocks(b.n)), dim3(kBlock), 0, s, static_cast<int>(b.n),
                           static_cast<const T*>(w.D), static_cast<const T*>(w.lam), out);
        return hipGetLastError();
    }));
    ++launched;
    if (async) return rc;
    Results res;
    const eik_status rr = read_results(w.ctl, w.blkstat, kMaxStatBlocks, false, s, res);
    if (rr != EIK_OK) return rr;
    if (st) {
        *st = eik_stats{};
        st->step3_iters = static_cast<int64_t>(res.ctl.iters3);
        st->tile_visits_step3 = static_cast<int64_t>(res.sum[SF_VISITS3]);
        st->launches = launched;
        HIP_TRY(prof.collect(st));
    }
    return rc;
}

}  // namespace

size_t adjoint_workspace_bytes(const Batch& b, size_t esz) {
    return adj_layout(nullptr, with_tiles(b, adj_tile(b.nd)), esz).bytes;
}

template <typename T>
eik_status adjoint_solve(const Batch& b0, const T* F, const T* phi, const T* g, T* out, const eik_options& o,
                         char* ws, hipStream_t s, eik_stats* st) {
    const Batch b = with_tiles(b0, adj_tile(b0.nd));
    if (b.nd == 2) return adj_run<T, 2, 16, 16, 1>(b, F, phi, g, out, o, ws, s, st);
    return adj_run<T, 3, 8, 8, 8>(b, F, phi, g, out, o, ws, s, st);
}

template eik_status adjoint_solve<float>(const Batch&, const float*, const float*, const float*, float*,
                                         const eik_options&, char*, hipStream_t, eik_stats*);
template eik_status adjoint_solve<double>(const Batch&, const double*, const double*, const double*, double*,
                                          const eik_options&, char*, hipStream_t, eik_stats*);

}  // namespace eik
