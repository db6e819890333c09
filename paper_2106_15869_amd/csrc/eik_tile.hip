// Tile-activated IFIM for gfx950.
//
// The grid is cut into tiles of TZ x TY x TX nodes.  A launch drains a list
// of tiles with persistent workgroups (256 lanes, four wave64), one tile
// visit at a time.  A visit stages the tile's values plus a one-cell halo in
// LDS (one round of global loads), runs the node rules of Algorithm 2 for
// several inner iterations without touching HBM, writes back what changed and
// schedules the tiles that have to be visited next (eik_sched.hpp: sub-list
// queues, stamps, order keys).
//
//   update step (STEP 2), default: from the sources outward, tile visits by
//     the remedy rule below -- a node takes phi~ = G_i(phi) when that is
//     lower and its neighbours are evaluated again -- lowest keys first.  Values settled
//     from the wrong side are corrected while the front is near (early
//     remedy) instead of after it has passed.
//   update step alone (EIK_FLAG_SKIP_REMEDY; 3D with
//     EIK_FLAG_NO_EARLY_REMEDY): FAR nodes with F > 0 next to a converged or
//     fixed node become active; active nodes take phi~; a node whose value no
//     longer moves (phi - phi~ <= eps) converges and activates its FAR
//     neighbours -- no convergence check of those neighbours (Section 3.3).
//     A node converging on a tile face schedules the tile across that face; a
//     tile that still holds active nodes schedules itself.
//   remedy detection (STEP 3, first part): one dense pass over all tiles;
//     a tile with any node whose phi~ < phi - eps enters the remedy list.
//   remedy loop (STEP 3): the remedy rule of Section 3.1.2 restricted to the
//     tile: evaluate the nodes, take the drops, evaluate again where a
//     neighbour changed, until nothing does (remedy_visit).  A tile enters with
//     all nodes to recheck (first visit) or with those on the faces whose
//     neighbour tile changed; a drop on a tile face marks that face dirty in
//     the tile across it and schedules it with the dropped value as its order
//     key.  By default (ordered) a launch visits only the lowest-key tiles of
//     its list and sends the others on to the next.
// Values are updated in place within an inner iteration (a read racing with
// an update sees either value, both upper bounds of the solution); tiles of
// one launch see each other's values only through the halo staged at the
// start of a visit.
#include <type_traits>
#include <utility>
#include <vector>

#include "eik_device.hpp"
#include "eik_host.hpp"
#include "eik_seglist.hpp"
#include "eik_batch.hpp"
#include "eik_sched.hpp"
#include "eik_tile.hpp"

namespace eik {

namespace {

// LDS label byte: bits 0-1 state, bit 2 passable (F > 0), bit 3 outside grid.
constexpr uint8_t kPass = 4u, kOut = 8u;

template <typename T>
struct TileIter : Sched {
    const T* F;
    T* phi;
    uint8_t* lab;
    const T* cells;  // tile-major cell values (k_tile_init), read by detection and the remedy visits
    int early;       // merged update step: revisits count as early remedy evaluations
};



// Per-node value kept in LDS for the local solve: H = h / F (+inf on a
// barrier), or with per-axis spacing the speed F itself (0 on a barrier).
template <typename T, bool AN>
__device__ __forceinline__ T cell_value(const Inst<T>& g, T f) {
    if (AN) return f > T(0) ? f : T(0);
    return cell_H(g.h, f);
}
template <typename T, bool AN>
__device__ __forceinline__ T dead_value() {
    return AN ? T(0) : pos_inf<T>();
}
// whether the node can take a finite value (not a barrier, inside the grid)
template <typename T, bool AN>
__device__ __forceinline__ bool cell_live(T v) {
    return AN ? v > T(0) : v < pos_inf<T>();
}
// The tile-major cell array marks a fixed (source) node with -1, a value no
// cell_value takes.
template <typename T>
__device__ __forceinline__ T fixed_cell() {
    return T(-1);
}
// whether a cell-array entry belongs to a node the remedy may change
template <typename T, bool AN>
__device__ __forceinline__ bool cell_free(T v) {
    return cell_live<T, AN>(v) && !(v < T(0));
}

// Global index of in-tile node n (clamped into the grid, so that it can be
// loaded unconditionally) and whether the node lies in the grid.
template <typename T, int ND, int TX, int TY, int TZ>
__device__ __forceinline__ int owned_index(const Inst<T>& g, int x0, int y0, int z0, int n, bool& ok) {
    using S = Shape<ND, TX, TY, TZ>;
    const int x = n % TX, y = (n / TX) % TY, z = ND == 3 ? n / (TX * TY) : 0;
    const int gx = x0 + x, gy = y0 + y, gz = z0 + z;
    ok = n < S::NT && gx < g.nx && gy < g.ny && gz < g.nz;
    return g.node_base + (min(gz, g.nz - 1) * g.ny + min(gy, g.ny - 1)) * g.nx + min(gx, g.nx - 1);
}

// F of the nodes a lane owns (n = threadIdx.x + r * kBlock), loaded before
// the staging so that both are in flight together.
template <typename T, int ND, int TX, int TY, int TZ>
__device__ __forceinline__ void load_owned_F(const Inst<T>& g, int x0, int y0, int z0, const T* F,
                                             T (&f)[Shape<ND, TX, TY, TZ>::NPT]) {
    using S = Shape<ND, TX, TY, TZ>;
#pragma unroll
    for (int r = 0; r < S::NPT; ++r) {
        bool ok;
        f[r] = F[owned_index<T, ND, TX, TY, TZ>(g, x0, y0, z0, threadIdx.x + r * kBlock, ok)];
    }
}

// Stage the tile and its halo: values (+inf outside) and labels (kOut outside).
// Addresses are clamped into the grid, so every global load of a lane is
// issued unconditionally, before its first LDS store (one memory round trip).
// Without HALO_LABELS only the tile's own labels are loaded (the halo's are
// set to 0, or kOut outside the grid): the detection pass and the remedy read
// labels of in-tile nodes only, and a halo row of labels is a cache line for
// ten bytes.
// With LABELS false no labels are loaded or stored (sl may be null).
template <typename T, int ND, int TX, int TY, int TZ, bool HALO_LABELS = true, bool LABELS = true>
__device__ __forceinline__ void stage(const Inst<T>& g, int x0, int y0, int z0, const T* phi,
                                      const uint8_t* lab, T* sphi, uint8_t* sl) {
    using S = Shape<ND, TX, TY, TZ>;
    constexpr int NIT = (S::NL + kBlock - 1) / kBlock;
    const T inf = pos_inf<T>();
    T v[NIT];
    uint8_t l[NIT];
    bool in[NIT];
#pragma unroll
    for (int j = 0; j < NIT; ++j) {
        const int q = min(static_cast<int>(threadIdx.x) + j * kBlock, S::NL - 1);
        const int lx = q % S::LX;
        const int ly = (q / S::LX) % S::LY;
        const int lz = q / (S::LX * S::LY);
        const int gx = x0 + lx - 1, gy = y0 + ly - 1, gz = ND == 3 ? z0 + lz - 1 : 0;
        in[j] = gx >= 0 && gx < g.nx && gy >= 0 && gy < g.ny && gz >= 0 && gz < g.nz;
        const int cx = min(max(gx, 0), g.nx - 1), cy = min(max(gy, 0), g.ny - 1), cz = min(max(gz, 0), g.nz - 1);
        const int G = g.node_base + (cz * g.ny + cy) * g.nx + cx;
        v[j] = phi[G];
        const bool inner = lx >= 1 && lx <= TX && ly >= 1 && ly <= TY && (ND == 2 || (lz >= 1 && lz <= TZ));
        l[j] = LABELS && (HALO_LABELS || inner) ? lab[G] : uint8_t(0);
    }
#pragma unroll
    for (int j = 0; j < NIT; ++j) {
        const int q = threadIdx.x + j * kBlock;
        if (q < S::NL) {
            sphi[q] = in[j] ? v[j] : inf;
            if (LABELS) sl[q] = in[j] ? l[j] : static_cast<uint8_t>(kOut);
        }
    }
}

// G_i from the neighbour values (+inf outside the grid).
// v is the node's H = h / F (isotropic) or its speed F (AN: per-axis spacing,
// H_k = spacing_k / F); see cell_value.
template <typename T, int ND, bool AN>
__device__ __forceinline__ T eval_nb(const T (&nb)[2 * ND], T v, const Inst<T>& g) {
    const T inf = pos_inf<T>();
    const T ax = tmin(nb[0], nb[1]);
    const T ay = tmin(nb[2], nb[3]);
    if (AN) {
        if (!(v > T(0))) return inf;
        if (ND == 2) return godunov_aniso<T, 2>(ay, ax, inf, g.d[0] / v, g.d[1] / v, inf);
        const T az = tmin(nb[4], nb[5]);
        return godunov_aniso<T, 3>(az, ay, ax, g.d[0] / v, g.d[1] / v, g.d[2] / v);
    }
    if (ND == 2) return godunov<T, 2>(ay, ax, inf, v);
    const T az = tmin(nb[4], nb[5]);
    return godunov<T, 3>(az, ay, ax, v);
}

// eval_nb for a node with H in the middle of the range (godunov_mid), equal
// spacing.
template <typename T, int ND>
__device__ __forceinline__ T eval_nb_mid(const T (&nb)[2 * ND], T H, T HH) {
    const T ax = vmin(nb[0], nb[1]);
    const T ay = vmin(nb[2], nb[3]);
    if (ND == 2) return godunov_mid<T, 2>(ay, ax, pos_inf<T>(), H, HH);
    return godunov_mid<T, 3>(vmin(nb[4], nb[5]), ay, ax, H, HH);
}

// G_i from the LDS tile (halo holds +inf outside the grid).
template <typename T, int ND, int TX, int TY, int TZ, bool AN>
__device__ __forceinline__ T eval_lds(const T* sphi, int L, T v, const Inst<T>& g) {
    T nb[2 * ND];
    load_nb<T, ND, TX, TY, TZ>(sphi, L, nb);
    return eval_nb<T, ND, AN>(nb, v, g);
}




// ---------------------------------------------------------------------------
// A remedy visit
// ---------------------------------------------------------------------------
// Beside the dirty faces in a visit's mask word: a node of the tile takes the
// general local solve.
constexpr uint32_t kGeneral = 128u;

// LDS of a remedy visit.
template <typename T, typename Mask>
struct RemedyLds {
    T* sphi;           // values with the one-cell halo
    Mask* act;         // [2][waves]: each wave's chunks that changed in an iteration (by parity)
    uint32_t* mask;    // dirty faces the visit starts from, kGeneral (0 between visits)
    int* face;         // faces a drop crossed
    int* evals;        // local-solver evaluations
    uint32_t* kmin;    // ordered: key of the smallest value that crossed a face (the caller sets kNoKey)
    int* unreached;    // whether a free node was +inf at the start (the tile's first visit)
    int* written;      // values written back
};

// The remedy rule on tile t at (x0, y0, z0): every lane owns the NPT nodes
// threadIdx.x + r * kBlock, with their cell values and current values in
// registers; the values with the halo lie in LDS, where neighbours read them.
// An iteration evaluates a node per lane and round, takes the drops in place
// and notes the chunks (64 nodes, one wave) that changed; the next iteration
// leaves out the chunks none of whose neighbours changed.  Iterations run
// until nothing changes or `inner` of them ran (pending).  The first one
// takes the chunks that hold a free node to recheck: any for kAllFaces in the
// dirty faces, else one on a dirty face.
// An iteration is one dependent chain (LDS read, solve, LDS write, barrier)
// whatever the number of active nodes, so evaluating all of a chunk costs no
// more than its few active nodes.  2D lognormal 4096^2: 28.5 ms with an LDS
// list of active nodes (flags and slots claimed by LDS atomics around each
// solve), 17.9 ms with dense rounds at 1000 cycles an iteration, 14.4 ms with
// the chain shortened (godunov_mid, neighbours and masks read in one LDS
// round, a mask word per wave instead of an atomic); maze 256^3 9.07, 6.27,
// 5.03 ms.
// The dirty faces are lane 0's mask_in.  Writes the
// changed values back and leaves the crossed faces, counts and (ordered) the
// crossing key in LDS.  Returns the iterations run.
template <typename T, int ND, int TX, int TY, int TZ, bool AN, typename Mask>
__device__ __forceinline__ int remedy_visit(const T* cells, T* phi, const Inst<T>& g, int t, int x0, int y0,
                                            int z0, int open, T eps, int inner, uint32_t mask_in,
                                            const RemedyLds<T, Mask>& s, bool& pending) {
    using S = Shape<ND, TX, TY, TZ>;
    constexpr int WAVES = kBlock / 64;
    static_assert(S::NT % kBlock == 0 && S::NT / 64 <= 8 * sizeof(Mask), "whole rounds, a chunk per bit");
    // LDS step from a lane's node of one round to the next
    constexpr int RSTEP = ND == 2 ? (kBlock / TX) * S::SY : (kBlock / (TX * TY)) * S::SZ;
    static_assert(kBlock % TX == 0 && (ND == 2 || kBlock % (TX * TY) == 0), "a round is whole rows (slices)");
    const T inf = pos_inf<T>();
    T* sphi = s.sphi;
    T hv[S::NPT];
#pragma unroll
    for (int r = 0; r < S::NPT; ++r) hv[r] = cells[static_cast<size_t>(t) * S::NT + threadIdx.x + r * kBlock];
    stage<T, ND, TX, TY, TZ, false, false>(g, x0, y0, z0, phi, nullptr, sphi, nullptr);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool lane0 = (threadIdx.x & 63) == 0;
    T cur[S::NPT], old[S::NPT], hh[S::NPT];
    constexpr bool AN2 = AN && ND == 2;
    AnisoNode<T> an[AN2 ? S::NPT : 1];
    bool fr[S::NPT], ends = false;
#pragma unroll
    for (int r = 0; r < S::NPT; ++r) {
        fr[r] = cell_free<T, AN>(hv[r]);
        if (!fr[r]) hv[r] = dead_value<T, AN>();  // never solves to a drop
        hh[r] = hv[r] * hv[r];
        if constexpr (AN2) {
            an[r].set(g.d[0], g.d[1], hv[r]);
            ends |= fr[r] && !an[r].fits();
        } else {
            ends |= fr[r] && !mid_range(hv[r]);
        }
    }
    if (ends) atomicOr(s.mask, kGeneral);
    if (threadIdx.x == 0) {
        *s.face = 0;
        *s.evals = 0;
        *s.written = 0;
        *s.unreached = 0;
        atomicOr(s.mask, mask_in);
    }
    __syncthreads();
    const uint32_t m = *s.mask;
    int nx, ny, nz, L0;
    node_loc<ND, TX, TY, TZ>(threadIdx.x, nx, ny, nz, L0);
    int nfree[S::NPT];
    Mask todo = 0;  // chunks to evaluate (the wave looks at its own)
    bool unreached = false;
#pragma unroll
    for (int r = 0; r < S::NPT; ++r) {
        int x, y, z, L;
        node_loc<ND, TX, TY, TZ>(threadIdx.x + r * kBlock, x, y, z, L);
        const int E = edge_bits<ND, TX, TY, TZ>(x, y, z) & open;
        cur[r] = old[r] = sphi[L0 + r * RSTEP];
        nfree[r] = __popcll(ballot64(fr[r]));
        unreached |= fr[r] && !(cur[r] < inf);
        if (ballot64(fr[r] && ((m & kAllFaces) || (E & static_cast<int>(m))))) todo |= Mask(1) << (r * WAVES + wave);
    }
    if (ballot64(unreached) && lane0) *s.unreached = 1;
    pending = false;
    int evals = 0;
    int it = 0;
    // (a loop for each of the two local solves: in one loop the compiler moves
    // parts of both in front of the choice)
    auto iterate = [&](auto mid_c) __attribute__((always_inline)) {
        for (;; ++it) {
            // chunks changed in the previous iteration, and for tiles of one
            // or two nodes per lane every neighbour value in the same LDS round
            // (the empty asm keeps the loads out of the branches that use them)
            constexpr bool AHEAD = S::NPT <= 2;
            T nv[AHEAD ? S::NPT : 1][2 * ND];
            Mask act[WAVES] = {};
            if (it > 0) {
#pragma unroll
                for (int w = 0; w < WAVES; ++w) act[w] = s.act[((it - 1) & 1) * WAVES + w];
            }
            if (AHEAD) {
#pragma unroll
                for (int r = 0; r < S::NPT; ++r) {
                    load_nb<T, ND, TX, TY, TZ>(sphi, L0 + r * RSTEP, nv[AHEAD ? r : 0]);
#pragma unroll
                    for (int d = 0; d < 2 * ND; ++d) asm volatile("" : "+v"(nv[AHEAD ? r : 0][d]));
                }
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
                const int L = L0 + r * RSTEP;
                T(&v)[2 * ND] = nv[AHEAD ? r : 0];
                if (!AHEAD) load_nb<T, ND, TX, TY, TZ>(sphi, L, v);
                T pt;
                if constexpr (decltype(mid_c)::value && AN2) pt = an[r].solve(vmin(v[2], v[3]), vmin(v[0], v[1]));
                else if constexpr (decltype(mid_c)::value) pt = eval_nb_mid<T, ND>(v, hv[r], hh[r]);
                else pt = eval_nb<T, ND, AN>(v, hv[r], g);
                const bool drop = pt < cur[r] - eps;
                cur[r] = drop ? pt : cur[r];
                sphi[L] = cur[r];  // (only this lane writes it)
                if (ballot64(drop)) changed |= bit;
                evals += nfree[r];
            }
            if (lane0) s.act[(it & 1) * WAVES + wave] = changed;
            __syncthreads();
        }
    };
    if constexpr (AN && !AN2) iterate(std::false_type{});
    else if (!(first_lane(m) & kGeneral)) iterate(std::true_type{});  // (the workgroup's choice: each has its own barrier)
    else iterate(std::false_type{});
    // write back what changed; a changed value that lies below the neighbour
    // across an open face crosses it
    int fm = 0, written = 0;
    uint32_t kmin = kNoKey;  // order key of the smallest value that crossed a face
#pragma unroll
    for (int r = 0; r < S::NPT; ++r) {
        const bool changed = cur[r] < old[r];
        written += __popcll(ballot64(changed));
        if (!changed) continue;
        int x, y, z, L;
        node_loc<ND, TX, TY, TZ>(threadIdx.x + r * kBlock, x, y, z, L);
        phi[g.node_base + ((z0 + z) * g.ny + (y0 + y)) * g.nx + (x0 + x)] = cur[r];
        const int E = edge_bits<ND, TX, TY, TZ>(x, y, z) & open;
        int f = 0;
#pragma unroll
        for (int d = 0; d < 2 * ND; ++d)
            if ((E & (1 << d)) && cur[r] < sphi[L + lds_offset<ND, TX, TY, TZ>(d)]) f |= 1 << d;
        if (f) {
            fm |= f;
            kmin = min(kmin, order_key(cur[r]));
        }
    }
    join_crossings<ND>(fm, kmin, s.face, s.kmin);
    if (lane0) {
        if (evals) atomicAdd(s.evals, evals);
        if (written) atomicAdd(s.written, written);
    }
    if (threadIdx.x == 0) *s.mask = 0u;
    __syncthreads();
    return it;
}

// ---------------------------------------------------------------------------
// STEP 2 on tiles
// ---------------------------------------------------------------------------
template <typename T, int ND, int TX, int TY, int TZ, bool AN>
__global__ __launch_bounds__(kBlock) void k_tile_update(TileIter<T> a, BatchGeom<T> bg, T eps, int inner) {
    using S = Shape<ND, TX, TY, TZ>;
    __shared__ T sphi[S::NL];
    __shared__ uint8_t sl[S::NL];
    __shared__ T sH[S::NT];
    __shared__ TileLists<S::NT> tl;
    __shared__ uint8_t schg[2][ND == 2 ? S::NT : 1];  // 2D: inputs changed in phase 1 (by iteration parity)
    __shared__ int s_len[kSub];
    __shared__ int s_slot;
    __shared__ int s_face;
    __shared__ int s_evals;
    __shared__ int s_written;
    const T inf = pos_inf<T>();
    const uint32_t ntag = launch_tag(a);
    const int n = list_open(a, s_len);
    launch_stats(a, n);
    // workgroups of group k take entries of sub-list k one at a time
    const int k = blockIdx.x & (kSub - 1);
    const int len = s_len[k];
    unsigned long long evals = 0, inner_sum = 0, written = 0, visits = 0;
    for (bool first = true;; first = false) {
        const int t = list_fetch(a.cur, k, len, &s_slot, first);
        if (t < 0) break;
        ++visits;
        const Inst<T> g = inst_of(bg, t);
        const int lt = t - g.tile_base;
        const int tx = lt % g.ntx, ty = (lt / g.ntx) % g.nty, tz = lt / (g.ntx * g.nty);
        const int x0 = tx * TX, y0 = ty * TY, z0 = tz * (ND == 3 ? TZ : 1);
        const int open = open_bits<ND, TX, TY, TZ>(g, x0, y0, z0);
        T fv[S::NPT];
        load_owned_F<T, ND, TX, TY, TZ>(g, x0, y0, z0, a.F, fv);
        stage<T, ND, TX, TY, TZ>(g, x0, y0, z0, a.phi, a.lab, sphi, sl);
        bool ok[S::NPT];
        int G[S::NPT], L[S::NPT];
#pragma unroll
        for (int r = 0; r < S::NPT; ++r) {
            const int nn = threadIdx.x + r * kBlock;
            int x, y, z;
            node_loc<ND, TX, TY, TZ>(nn, x, y, z, L[r]);
            G[r] = owned_index<T, ND, TX, TY, TZ>(g, x0, y0, z0, nn, ok[r]);
            if (nn < S::NT) {
                sH[nn] = ok[r] ? cell_value<T, AN>(g, fv[r]) : dead_value<T, AN>();
                tl.flag[0][nn] = 0u;
                tl.flag[1][nn] = 0u;
                if (ND == 2) {
                    schg[0][nn] = 0;
                    schg[1][nn] = 0;
                }
            }
        }
        if (threadIdx.x == 0) {
            s_face = 0;
            s_evals = 0;
            s_written = 0;
            tl.cnt[0] = tl.cnt[1] = tl.cnt[2] = 0;
        }
        __syncthreads();
        uint8_t lab0[S::NPT];
        T phi0[S::NPT];
#pragma unroll
        for (int r = 0; r < S::NPT; ++r) {
            lab0[r] = ok[r] ? sl[L[r]] : uint8_t(0);
            phi0[r] = ok[r] ? sphi[L[r]] : inf;
            if (ok[r] && cell_live<T, AN>(sH[threadIdx.x + r * kBlock])) sl[L[r]] = lab0[r] | kPass;
        }
        __syncthreads();
        // initial active list: active nodes, and FAR nodes next to a converged
        // or fixed node (their activation was requested by a neighbour)
#pragma unroll
        for (int r = 0; r < S::NPT; ++r) {
            if (!ok[r]) continue;
            const uint8_t me = sl[L[r]];
            bool act = (me & 3u) == L_ACTIVE;
            if ((me & 3u) == L_FAR && (me & kPass)) {
#pragma unroll
                for (int d = 0; d < 2 * ND; ++d) {
                    const uint8_t nb = sl[L[r] + lds_offset<ND, TX, TY, TZ>(d)];
                    const uint32_t st = nb & 3u;
                    act |= !(nb & kOut) && (st == L_CONV || st == L_FIXED);
                }
                if (act) sl[L[r]] = (me & ~3u) | L_ACTIVE;
            }
            if (act) tl.list[0][atomicAdd(&tl.cnt[0], 1)] = static_cast<uint16_t>(threadIdx.x + r * kBlock);
        }
        __syncthreads();
        // Inner iterations on the LDS active list, values updated in place.
        // Reads racing with updates see either value, both upper bounds of the
        // solution.  Each iteration has two phases:
        //   1. every listed node is evaluated; a value that does not move
        //      (phi - phi~ <= eps) converges the node, a value that drops is
        //      taken and marks the node's in-tile neighbours "inputs changed";
        //   2. a node whose value dropped in phase 1 while none of its inputs
        //      changed converges at once: its re-evaluation would give the
        //      same value (the convergence test of the next iteration, known
        //      in advance); the others are listed again.
        // A front thus crosses one node per iteration instead of two.  In 3D
        // phase 2 is left out (a dropped value is listed again and confirmed
        // by its next evaluation): the extra phase and its registers cost
        // more there than the shorter crossings save.
        constexpr bool TWO_PHASE = ND == 2;
        bool any_active = false;
        int my_evals = 0, fm = 0;
        int it = 0;
        for (;; ++it) {
            const int ncur = tl.cnt[it % 3];
            if (ncur == 0) break;
            if (it == inner) {
                any_active = true;  // cap reached: the listed nodes stay active
                break;
            }
            const int cb = it & 1, nb = cb ^ 1;
            int* ncnt = &tl.cnt[(it + 1) % 3];
            if (threadIdx.x == 0) tl.cnt[(it + 2) % 3] = 0;
            // the marks of the previous iteration are no longer read
            if (TWO_PHASE) {
#pragma unroll
                for (int r = 0; r < S::NPT; ++r)
                    if (threadIdx.x + r * kBlock < S::NT) schg[nb][threadIdx.x + r * kBlock] = 0;
            }
            // converged node q (LDS index Lq, tile position x, y, z): CONV,
            // its FAR neighbours become active
            auto converge = [&](int q, int Lq, int x, int y, int z) {
                sl[Lq] = (sl[Lq] & ~3u) | L_CONV;
                const int edge = edge_bits<ND, TX, TY, TZ>(x, y, z);
                // the neighbours' labels, read in one round
                uint8_t lbs[2 * ND];
#pragma unroll
                for (int d = 0; d < 2 * ND; ++d) lbs[d] = sl[Lq + lds_offset<ND, TX, TY, TZ>(d)];
#pragma unroll
                for (int d = 0; d < 2 * ND; ++d) {
                    const int Ln = Lq + lds_offset<ND, TX, TY, TZ>(d);
                    const uint8_t lb = lbs[d];
                    if (edge & (1 << d)) {
                        if ((open & (1 << d)) && (lb & 3u) == L_FAR) fm |= 1 << d;
                    } else if (!(lb & kOut) && (lb & 3u) == L_FAR && (lb & kPass)) {
                        if (list_add(tl, nb, ncnt, q + node_step<TX, TY>(d))) sl[Ln] = (lb & ~3u) | L_ACTIVE;
                    }
                }
            };
            constexpr int MAXC = (S::NT + kBlock - 1) / kBlock;
            int cq[MAXC];
            int nc = 0;
            for (int i = threadIdx.x; i < ncur; i += kBlock) {
                const int q = tl.list[cb][i];
                tl.flag[cb][q] = 0u;
                int x, y, z, Lq;
                node_loc<ND, TX, TY, TZ>(q, x, y, z, Lq);
                ++my_evals;
                const T pt = eval_lds<T, ND, TX, TY, TZ, AN>(sphi, Lq, sH[q], g);
                const T cur = sphi[Lq];
                if (pt < inf && cur - pt <= eps) {
                    converge(q, Lq, x, y, z);
                } else if (!(pt < inf)) {
                    sl[Lq] = (sl[Lq] & ~3u) | L_FAR;
                } else {
                    sphi[Lq] = pt;  // pt < cur - eps
                    if (TWO_PHASE) {
                        const int edge = edge_bits<ND, TX, TY, TZ>(x, y, z);
#pragma unroll
                        for (int d = 0; d < 2 * ND; ++d)
                            if (!(edge & (1 << d))) schg[cb][q + node_step<TX, TY>(d)] = 1;
                        cq[nc++] = q;
                    } else {
                        list_add(tl, nb, ncnt, q);
                    }
                }
            }
            if (TWO_PHASE) {
                __syncthreads();
                for (int j = 0; j < nc; ++j) {
                    const int q = cq[j];
                    int x, y, z, Lq;
                    node_loc<ND, TX, TY, TZ>(q, x, y, z, Lq);
                    if (!schg[cb][q]) converge(q, Lq, x, y, z);
                    else list_add(tl, nb, ncnt, q);
                }
            }
            __syncthreads();
        }
        if (fm) atomicOr(&s_face, fm);
        // write back what changed
        int my_written = 0;
#pragma unroll
        for (int r = 0; r < S::NPT; ++r) {
            if (!ok[r]) continue;
            const uint8_t st = sl[L[r]] & 3u;
            if (st != (lab0[r] & 3u)) a.lab[G[r]] = st;
            const T v = sphi[L[r]];
            if (v != phi0[r]) {
                a.phi[G[r]] = v;
                ++my_written;
            }
        }
        if (my_evals) atomicAdd(&s_evals, my_evals);
        if (my_written) atomicAdd(&s_written, my_written);
        __syncthreads();
        // scheduling: lane d < 2*ND handles face d, lane 6 the tile itself,
        // so the device atomics of one visit are in flight together
        if (threadIdx.x < 7) {
            const int d = threadIdx.x;
            const int fmask = s_face;
            if (d == 6) {
                if (any_active) push_tile(a.next, a.tstamp, t, ntag);
            } else if (d < 2 * ND && (fmask & (1 << d))) {
                push_tile(a.next, a.tstamp, neighbour_tile(g, t, d), ntag);
            }
        }
        if (threadIdx.x == 0) {
            evals += static_cast<unsigned long long>(s_evals);
            inner_sum += static_cast<unsigned long long>(it);
            written += static_cast<unsigned long long>(s_written);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0 && visits) {
        stat_add(a.blkstat, SF_EVALS2, evals);
        stat_add(a.blkstat, SF_VISITS2, visits);
        stat_add(a.blkstat, SF_INNER2, inner_sum);
        stat_add(a.blkstat, SF_WRITTEN2, written);
    }
}

// ---------------------------------------------------------------------------
// STEP 3: whole-grid detection, one workgroup per tile
// ---------------------------------------------------------------------------
template <typename T, int ND, int TX, int TY, int TZ, bool AN>
__global__ __launch_bounds__(kBlock) void k_tile_detect(TileIter<T> a, BatchGeom<T> bg, T eps) {
    using S = Shape<ND, TX, TY, TZ>;
    __shared__ T sphi[S::NL];
    __shared__ uint32_t s_key;
    const uint32_t ntag = launch_tag(a);
    for (int t = blockIdx.x; t < bg.ntiles; t += gridDim.x) {
        const Inst<T> g = inst_of(bg, t);
        const int lt = t - g.tile_base;
        const int tx = lt % g.ntx, ty = (lt / g.ntx) % g.nty, tz = lt / (g.ntx * g.nty);
        const int x0 = tx * TX, y0 = ty * TY, z0 = tz * (ND == 3 ? TZ : 1);
        if (threadIdx.x == 0) s_key = kNoKey;  // ordered below the staging barrier
        T hv[S::NPT];
#pragma unroll
        for (int r = 0; r < S::NPT; ++r) {
            const int nn = min(static_cast<int>(threadIdx.x) + r * kBlock, S::NT - 1);
            hv[r] = a.cells[static_cast<size_t>(t) * S::NT + nn];
        }
        stage<T, ND, TX, TY, TZ, false, false>(g, x0, y0, z0, a.phi, nullptr, sphi, nullptr);
        __syncthreads();
        bool flag = false;
        T low = pos_inf<T>();
#pragma unroll
        for (int r = 0; r < S::NPT; ++r) {
            const int nn = threadIdx.x + r * kBlock;
            if (nn >= S::NT || !cell_free<T, AN>(hv[r])) continue;  // outside, barrier or fixed
            int x, y, z, L;
            node_loc<ND, TX, TY, TZ>(nn, x, y, z, L);
            const T pt = eval_lds<T, ND, TX, TY, TZ, AN>(sphi, L, hv[r], g);
            if (pt < sphi[L] - eps) {
                flag = true;
                low = tmin(low, pt);
            }
        }
        if (a.ordered && flag) atomicMin(&s_key, order_key(low));
        if (__syncthreads_or(flag) && threadIdx.x == 0) {
            a.mask_next[t] = kAllFaces;  // one writer: the workgroup of tile t
            push_keyed(a, t, ntag, s_key);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Remedy visits: the correcting update step and the remedy loop
// ---------------------------------------------------------------------------
// Statistics of a workgroup's visits, by the loop it ran in.
__device__ __forceinline__ void visit_stats(const Sched& a, unsigned long long evals, unsigned long long early,
                                            unsigned long long visits, unsigned long long inner,
                                            unsigned long long written) {
    const bool upd = a.phase == 0;
    stat_add(a.blkstat, upd ? SF_EVALS2 : SF_EVALS3, evals);
    stat_add(a.blkstat, SF_CHECK, early);
    stat_add(a.blkstat, upd ? SF_VISITS2 : SF_VISITS3, visits);
    stat_add(a.blkstat, upd ? SF_INNER2 : SF_INNER3, inner);
    stat_add(a.blkstat, upd ? SF_WRITTEN2 : SF_WRITTEN3, written);
}

// Resident workgroups per CU for float tiles (the inner iterations are
// latency-bound; occupancy against spilled registers, measured): eight for
// tiles of one node per lane, six for two (the 8^3 tile: eight spill at
// 64 registers, five or fewer were slower).
template <int NPT, typename T>
constexpr int remedy_blocks_per_cu() {
    return sizeof(T) != 4 ? 1 : NPT == 1 ? 8 : NPT == 2 ? 6 : 1;
}

template <typename T, int ND, int TX, int TY, int TZ, bool AN>
__global__ __launch_bounds__(kBlock, (remedy_blocks_per_cu<Shape<ND, TX, TY, TZ>::NPT, T>())) void k_tile_remedy(
    TileIter<T> a, BatchGeom<T> bg, T eps, int inner) {
    using S = Shape<ND, TX, TY, TZ>;
    __shared__ T sphi[S::NL];
    using Mask = ChunkMask<S::NT>;
    __shared__ Mask s_act[2 * kBlock / 64];
    __shared__ int s_len[kSub];
    __shared__ int s_slot;
    __shared__ int s_face;
    __shared__ int s_evals;
    __shared__ int s_written;
    __shared__ uint32_t s_mask;
    __shared__ uint32_t s_key, s_kmin;
    __shared__ int s_unreached;
    if (threadIdx.x == 0) s_mask = 0u;  // (before the barrier of list_open)
    const uint32_t ntag = launch_tag(a);
    const unsigned long long e0 = first_entry(a);
    const int n = list_open(a, s_len);
    launch_stats(a, n);
    const int k = blockIdx.x & (kSub - 1);
    const int len = s_len[k];
    if (static_cast<int>(blockIdx.x) / kSub >= len) return;  // no first entry: none at all
    const bool all = !a.ordered || n <= a.order_aim;  // the launch takes every tile listed
    const uint32_t thr = !all && threadIdx.x < 64 ? sampled_threshold(a, s_len, n) : kNoKey;
    unsigned long long evals = 0, early = 0, inner_sum = 0, written = 0, visits = 0;
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
            __syncthreads();
            if (t < 0) break;
        }
        ++visits;
        const Inst<T> g = inst_of(bg, t);
        const int lt = t - g.tile_base;
        const int tx = lt % g.ntx, ty = (lt / g.ntx) % g.nty, tz = lt / (g.ntx * g.nty);
        const int x0 = tx * TX, y0 = ty * TY, z0 = tz * (ND == 3 ? TZ : 1);
        const int open = open_bits<ND, TX, TY, TZ>(g, x0, y0, z0);
        uint32_t mask_in = 0;
        if (threadIdx.x == 0) {
            // written by the previous launch; no writer during this one
            mask_in = a.mask_cur[t];
            a.mask_cur[t] = 0u;
            s_kmin = kNoKey;
        }
        const RemedyLds<T, Mask> rl{sphi, s_act, &s_mask, &s_face, &s_evals, &s_kmin, &s_unreached, &s_written};
        bool pending;
        const int it = remedy_visit<T, ND, TX, TY, TZ, AN>(a.cells, a.phi, g, t, x0, y0, z0, open, eps, inner,
                                                           mask_in, rl, pending);
        // scheduling, one lane per target tile (see the update kernel); the
        // targets are read by the next launch
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
                atomicOr(a.mask_next + tn, 1u << (d ^ 1));  // the face of tn shared with t
                push_keyed(a, tn, ntag, key);
            }
        }
        if (threadIdx.x == 0) {
            // a revisit of the merged update step corrects values: early remedy
            (a.early && !s_unreached ? early : evals) += static_cast<unsigned long long>(s_evals);
            inner_sum += static_cast<unsigned long long>(it);
            written += static_cast<unsigned long long>(s_written);
        }
    }
    if (threadIdx.x == 0 && visits) visit_stats(a, evals, early, visits, inner_sum, written);
}


// ---------------------------------------------------------------------------
// STEP 1
// ---------------------------------------------------------------------------
// Tile-major cell values: entry t * NT + n holds the cell value of node n of
// tile t (H = h / F, or F itself with per-axis spacing; +inf / 0 on a barrier),
// -1 for a fixed node (k_tile_sources), the dead value outside the grid.  A
// tile's detection and visits then read one contiguous block instead of a row
// of F per cache line and a label byte per node, and do not divide.  In the same
// pass: every value +inf, and the check of F.
template <typename T, int ND, int TX, int TY, int TZ, bool AN>
__global__ __launch_bounds__(kBlock) void k_tile_init(BatchGeom<T> bg, const T* __restrict__ F, T* __restrict__ phi,
                                                      T* __restrict__ cells, Ctl* ctl) {
    using S = Shape<ND, TX, TY, TZ>;
    static_assert(S::NT % 64 == 0, "a wave's entries must lie in one tile");
    const int64_t total = static_cast<int64_t>(bg.ntiles) * S::NT;
    bool bad = false;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < total;
         i += static_cast<int64_t>(gridDim.x) * kBlock) {
        const int t = static_cast<int>(i / S::NT);
        const int n = static_cast<int>(i - static_cast<int64_t>(t) * S::NT);
        const Inst<T> g = inst_of(bg, t);
        const int lt = t - g.tile_base;
        const int tx = lt % g.ntx, ty = (lt / g.ntx) % g.nty, tz = lt / (g.ntx * g.nty);
        bool ok;
        const int G = owned_index<T, ND, TX, TY, TZ>(g, tx * TX, ty * TY, tz * (ND == 3 ? TZ : 1), n, ok);
        T v = dead_value<T, AN>();
        if (ok) {
            const T f = F[G];
            bad |= !(f >= T(0)) || !(f < pos_inf<T>());
            v = cell_value<T, AN>(g, f);
            phi[G] = pos_inf<T>();
        }
        cells[i] = v;
    }
    if (ballot64(bad) && lane_id() == 0) atomicOr(&ctl->err, 1);
}

// Sources: values and fixed cells.  With `queue`, the tiles holding a grid
// neighbour of a source enter a's next list, every node of them to be
// evaluated, ordered by the source's value.  (cells may be NULL: the update
// step alone takes sources from the labels.)
template <typename T>
__global__ void k_tile_sources(Sched a, BatchGeom<T> bg, int nd, int tx_, int ty_, int tz_, SrcBatch<T> b, T* phi,
                               T* cells, int queue) {
    const int k = threadIdx.x;
    if (k >= b.count) return;
    const Inst<T> g = bg.ninst == 1 ? bg.one : bg.table[b.inst[k]];
    const int i = b.idx[k] - g.node_base;
    const int x = i % g.nx, y = (i / g.nx) % g.ny, z = i / (g.nx * g.ny);
    phi[b.idx[k]] = b.val[k];
    if (cells) {
        const size_t t = g.tile_base + ((z / tz_) * g.nty + (y / ty_)) * g.ntx + (x / tx_);
        cells[t * (tx_ * ty_ * tz_) + ((z % tz_) * ty_ + y % ty_) * tx_ + x % tx_] = fixed_cell<T>();
    }
    if (!queue) return;
    const int dx[6] = {-1, 1, 0, 0, 0, 0}, dy[6] = {0, 0, -1, 1, 0, 0}, dz[6] = {0, 0, 0, 0, -1, 1};
    for (int d = 0; d < 2 * nd; ++d) {
        const int X = x + dx[d], Y = y + dy[d], Z = z + dz[d];
        if (X < 0 || X >= g.nx || Y < 0 || Y >= g.ny || Z < 0 || Z >= g.nz) continue;
        const int t = g.tile_base + ((Z / tz_) * g.nty + (Y / ty_)) * g.ntx + (X / tx_);
        atomicOr(a.mask_next + t, kAllFaces);
        push_keyed(a, t, 1u, order_key(b.val[k]));
    }
}

// Initial tile list holding every tile (the update step alone, many
// sources): tile t is entry t / kSub of sub-list t % kSub.
__global__ void k_seed_all_tiles(int ntiles, uint32_t* tstamp, TList out) {
    for (int t = blockIdx.x * kBlock + threadIdx.x; t < ntiles; t += gridDim.x * kBlock) {
        tstamp[t] = 1u;
        out.data[static_cast<size_t>(t & (kSub - 1)) * out.cap + (t / kSub)] = list_entry(t, 0u);
    }
    if (blockIdx.x == 0 && threadIdx.x < kSub)
        out.count[threadIdx.x * kPad] = (ntiles - static_cast<int>(threadIdx.x) + kSub - 1) / kSub;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct TileWs {
    Ctl* ctl;
    unsigned long long* blkstat;
    uint8_t* lab;
    void* cells;        // tile-major cell values (ntiles x tile nodes)
    SchedWs q;          // lists, stamps, masks, keys
    void* table;        // instance table (batches of more than one instance)
    int* tile_inst;     // instance of every tile (idem)
    void* table_u;      // the same for the update step's tiling (2D, see solve_tile)
    int* tile_inst_u;
    size_t bytes;
};

TileWs tile_layout(char* base, int64_t n, int64_t ntiles, size_t ninst, size_t inst_bytes, bool two_tilings,
                   size_t cell_bytes) {
    TileWs w{};
    size_t off = 0;
    auto take = [&](size_t b) {
        char* p = base ? base + off : nullptr;
        off = align_up(off + b, 256);
        return p;
    };
    w.ctl = reinterpret_cast<Ctl*>(take(sizeof(Ctl)));
    w.blkstat = reinterpret_cast<unsigned long long*>(take(8 * static_cast<size_t>(kStatFields) * kMaxStatBlocks));
    w.lab = reinterpret_cast<uint8_t*>(take(static_cast<size_t>(n)));
    w.cells = take(cell_bytes);
    w.q = sched_layout(take, ntiles);
    if (ninst > 1) {
        w.table = take(inst_bytes * ninst);
        w.tile_inst = reinterpret_cast<int*>(take(4 * static_cast<size_t>(ntiles)));
        if (two_tilings) {  // the update step's tiling has no more tiles than this one
            w.table_u = take(inst_bytes * ninst);
            w.tile_inst_u = reinterpret_cast<int*>(take(4 * static_cast<size_t>(ntiles)));
        }
    }
    w.bytes = off;
    return w;
}

// The 2D update step alone runs on 32 x 32 tiles by default: its launches are bound by the front crossing a tile,
// so bigger tiles need fewer of them (2D lognormal 4096^2: update 18.6 ->
// 17.0 ms), while the remedy is faster on the smaller tiles.
bool update_tiling(const Batch& b, const eik_options& o, TileCfg& cu) {
    const bool def = o.tile[0] == 0 && o.tile[1] == 0 && o.tile[2] == 0;
    if (b.nd != 2 || !def || b.inst[0].aniso || b.cfg.tx != 16 || b.cfg.ty != 16) return false;
    cu = TileCfg{32, 32, 1};
    return true;
}

// Launches of `gt` persistent workgroups (a multiple of kSub, at most GT).
template <typename T, int ND, int TX, int TY, int TZ, bool AN>
struct TileKernels {
    static hipError_t update(const TileIter<T>& a, const BatchGeom<T>& g, T eps, int inner, int gt, hipStream_t s) {
        hipLaunchKernelGGL((k_tile_update<T, ND, TX, TY, TZ, AN>), dim3(gt), dim3(kBlock), 0, s, a, g, eps, inner);
        return hipGetLastError();
    }
    static hipError_t detect(const TileIter<T>& a, const BatchGeom<T>& g, T eps, int gt, hipStream_t s) {
        hipLaunchKernelGGL((k_tile_detect<T, ND, TX, TY, TZ, AN>), dim3(gt), dim3(kBlock), 0, s, a, g, eps);
        return hipGetLastError();
    }
    static hipError_t remedy(const TileIter<T>& a, const BatchGeom<T>& g, T eps, int inner, int gt, hipStream_t s) {
        hipLaunchKernelGGL((k_tile_remedy<T, ND, TX, TY, TZ, AN>), dim3(gt), dim3(kBlock), 0, s, a, g, eps, inner);
        return hipGetLastError();
    }
    static hipError_t init(const BatchGeom<T>& g, const T* F, T* phi, T* cells, Ctl* ctl, hipStream_t s) {
        using S = Shape<ND, TX, TY, TZ>;
        const int64_t total = static_cast<int64_t>(g.ntiles) * S::NT;
        const int blocks = static_cast<int>(std::min<int64_t>((total + kBlock - 1) / kBlock, 8192));
        hipLaunchKernelGGL((k_tile_init<T, ND, TX, TY, TZ, AN>), dim3(blocks), dim3(kBlock), 0, s, g, F, phi, cells, ctl);
        return hipGetLastError();
    }
};

template <typename T>
struct TileOps {
    hipError_t (*update)(const TileIter<T>&, const BatchGeom<T>&, T, int, int, hipStream_t) = nullptr;
    hipError_t (*detect)(const TileIter<T>&, const BatchGeom<T>&, T, int, hipStream_t) = nullptr;
    hipError_t (*remedy)(const TileIter<T>&, const BatchGeom<T>&, T, int, int, hipStream_t) = nullptr;
    hipError_t (*init)(const BatchGeom<T>&, const T*, T*, T*, Ctl*, hipStream_t) = nullptr;
};

template <typename T, int ND, int TX, int TY, int TZ, bool AN = false>
TileOps<T> ops_of() {
    TileOps<T> k;
    k.update = &TileKernels<T, ND, TX, TY, TZ, AN>::update;
    k.detect = &TileKernels<T, ND, TX, TY, TZ, AN>::detect;
    k.remedy = &TileKernels<T, ND, TX, TY, TZ, AN>::remedy;
    k.init = &TileKernels<T, ND, TX, TY, TZ, AN>::init;
    return k;
}

// Supported tile shapes (z, y, x); per-axis spacing only with the default
// shapes (16 x 16 in 2D, 8^3 in 3D).
template <typename T>
bool select_ops(int nd, const TileCfg& c, bool aniso, TileOps<T>& k) {
    if (aniso) {
        if (nd == 2 && c.ty == 16 && c.tx == 16) return k = ops_of<T, 2, 16, 16, 1, true>(), true;
        if (nd == 3 && c.tz == 8 && c.ty == 8 && c.tx == 8) return k = ops_of<T, 3, 8, 8, 8, true>(), true;
        return false;
    }
    if (nd == 2) {
        if (c.ty == 16 && c.tx == 16) return k = ops_of<T, 2, 16, 16, 1>(), true;
        if (c.ty == 32 && c.tx == 32) return k = ops_of<T, 2, 32, 32, 1>(), true;
        if (c.ty == 16 && c.tx == 64) return k = ops_of<T, 2, 64, 16, 1>(), true;
        if (c.ty == 8 && c.tx == 32) return k = ops_of<T, 2, 32, 8, 1>(), true;
        if (c.ty == 64 && c.tx == 64) return k = ops_of<T, 2, 64, 64, 1>(), true;
        return false;
    }
    if (c.tz == 8 && c.ty == 8 && c.tx == 8) return k = ops_of<T, 3, 8, 8, 8>(), true;
    if (c.tz == 4 && c.ty == 8 && c.tx == 8) return k = ops_of<T, 3, 8, 8, 4>(), true;
    if (c.tz == 4 && c.ty == 4 && c.tx == 16) return k = ops_of<T, 3, 16, 4, 4>(), true;
    if (c.tz == 8 && c.ty == 8 && c.tx == 16) return k = ops_of<T, 3, 16, 8, 8>(), true;
    if (c.tz == 16 && c.ty == 16 && c.tx == 16) return k = ops_of<T, 3, 16, 16, 16>(), true;
    return false;
}

}  // namespace

TileCfg pick_tile(int nd, const eik_options& o) {
    TileCfg c{o.tile[2], o.tile[1], o.tile[0]};
    if (nd == 2) {
        c.tz = 1;
        if (c.tx == 0 || c.ty == 0) c = TileCfg{16, 16, 1};
    } else if (c.tx == 0 || c.ty == 0 || c.tz == 0) {
        c = TileCfg{8, 8, 8};
    }
    return c;
}

void batch_add(Batch& b, int nx, int ny, int nz, double h, const double* d) {
    HostInst e{};
    e.nx = nx;
    e.ny = ny;
    e.nz = nz;
    e.ntx = (nx + b.cfg.tx - 1) / b.cfg.tx;
    e.nty = (ny + b.cfg.ty - 1) / b.cfg.ty;
    e.ntz = (nz + b.cfg.tz - 1) / b.cfg.tz;
    e.node_base = static_cast<int>(b.n);
    e.tile_base = static_cast<int>(b.ntiles);
    e.h = h;
    e.aniso = d ? 1 : 0;
    for (int k = 0; k < 3; ++k) e.d[k] = d ? d[k] : 0.0;
    b.inst.push_back(e);
    b.n += static_cast<int64_t>(nx) * ny * nz;
    b.ntiles += static_cast<int64_t>(e.ntx) * e.nty * e.ntz;
}

Batch with_tiles(const Batch& b, const TileCfg& c) {
    Batch r;
    r.nd = b.nd;
    r.cfg = c;
    for (const HostInst& e : b.inst) batch_add(r, e.nx, e.ny, e.nz, e.h, e.aniso ? e.d : nullptr);
    r.src = b.src;
    r.src_inst = b.src_inst;
    return r;
}

// Bytes of the tile-major cell array of a batch's tiling.
static size_t cell_array_bytes(const Batch& b, size_t esz) {
    return static_cast<size_t>(b.ntiles) * static_cast<size_t>(b.cfg.tx) * b.cfg.ty * b.cfg.tz * esz;
}

size_t tile_workspace_bytes(const Batch& b, size_t esz) {
    const size_t ib = esz == 8 ? sizeof(Inst<double>) : sizeof(Inst<float>);
    return tile_layout(nullptr, b.n, b.ntiles, b.inst.size(), ib, b.nd == 2, cell_array_bytes(b, esz)).bytes;
}

template <typename T>
eik_status solve_tile(const Batch& b, const T* F, double eps, T* phi, const eik_options& o, char* ws,
                      hipStream_t s, eik_stats* st) {
    const bool async = (o.flags & EIK_FLAG_ASYNC) != 0;
    const bool pageable = (o.flags & kFlagPageable) != 0;
    const bool skip_remedy = (o.flags & EIK_FLAG_SKIP_REMEDY) != 0;
    // The update step alone (a diagnostic, and 3D solves that ask for it);
    // else the update step corrects values as it goes (see below).
    const bool alone = skip_remedy || (b.nd == 3 && (o.flags & EIK_FLAG_NO_EARLY_REMEDY));
    const TileCfg c = b.cfg;
    TileOps<T> k;
    if (!select_ops<T>(b.nd, c, b.inst[0].aniso != 0, k))
        return fail(EIK_ERR_INVALID_ARGUMENT, b.inst[0].aniso ? "per-axis spacing needs the default tile shape"
                                                              : "unsupported tile shape");
    TileWs w = tile_layout(ws, b.n, b.ntiles, b.inst.size(), sizeof(Inst<T>), b.nd == 2, cell_array_bytes(b, sizeof(T)));
    // the tiling of the update step alone (the same unless update_tiling says otherwise)
    TileCfg cu = c;
    const bool two = alone && update_tiling(b, o, cu);
    const Batch bu = two ? with_tiles(b, cu) : Batch{};
    const Batch& B2 = two ? bu : b;
    TileOps<T> ku = k;
    if (two && !select_ops<T>(b.nd, cu, false, ku)) return fail(EIK_ERR_INVALID_ARGUMENT, "unsupported tile shape");
    const int64_t cap = o.max_iters > 0 ? o.max_iters : 4 * b.n + 64;
    // Launches the correcting update step may take.  It does the work of the
    // update step alone and of the remedy loop, cap launches each, on tiles half
    // as wide in 2D: up to three times the longer of the two (a 4 x 19 grid: 3
    // against 1 and 1; of 1500 random small grids two took more than twice as
    // many; 2D lognormal 1024^2 130 against 64 and 127).  What it leaves over goes to
    // the remedy loop with its cap launches.  An asynchronous call runs every
    // launch of its budget, so there it is cap for each loop.
    const int64_t cap2 = alone || async || cap > INT64_MAX / 2 ? cap : 2 * cap;
    // Inner iterations per tile visit: visits run until their lists empty
    // (4 x the sum of the sides is a safety cap), except in the 2D update step
    // alone, whose visits stop after the iterations a front needs to cross the
    // tile along an axis (the front still advances a tile per launch, and no
    // visit holds its launch for a diagonal crossing).
    const int inner = o.inner_iters > 0 ? o.inner_iters : 4 * (c.tx + c.ty + c.tz);
    const int side_u = std::max(cu.tx, std::max(cu.ty, cu.tz));
    const int inner_upd = o.inner_iters > 0 ? o.inner_iters : (b.nd == 2 ? side_u : inner);
    const int ntiles_u = static_cast<int>(B2.ntiles);
    const int gt = workgroups_of(b.nd, o.workgroups, b.ntiles);
    const int omin = order_min_of(b.nd, o.order_min);
    int64_t launched = 0;

    Profiler prof;
    prof.start((o.flags & EIK_FLAG_PROFILE) != 0, s);
    const size_t blk_bytes = 8 * static_cast<size_t>(kStatFields) * kMaxStatBlocks;
    BatchGeom<T> geom, geom_u;
    HIP_TRY(timed(prof, EIK_KERNEL_OTHER, [&] { return upload_batch_geom<T>(b, w.table, w.tile_inst, s, geom, launched); }));
    if (two)
        HIP_TRY(timed(prof, EIK_KERNEL_OTHER, [&] {
            return upload_batch_geom<T>(bu, w.table_u, w.tile_inst_u, s, geom_u, launched);
        }));
    else
        geom_u = geom;
    ClearPlan clear;
    clear.ctl = w.ctl;
    clear.add(w.blkstat, blk_bytes);
    sched_clear(w.q, clear);
    HIP_TRY(timed(prof, EIK_KERNEL_OTHER, [&] { return launch_clear(clear, s); }));
    // +inf everywhere, cell values for the visits and detection; the update step
    // alone works from labels
    if (alone) {
        HIP_TRY(timed(prof, EIK_KERNEL_OTHER, [&] {
            return launch_init<T>(F, phi, w.lab, nullptr, static_cast<int>(b.n), w.ctl, s);
        }));
        launched += 1;
    }
    if (!skip_remedy) {
        HIP_TRY(timed(prof, EIK_KERNEL_OTHER, [&] { return k.init(geom, F, phi, static_cast<T*>(w.cells), w.ctl, s); }));
        launched += 1;
    }
    launched += 1;
    const bool ordered = (o.flags & EIK_FLAG_FIFO_REMEDY) == 0;
    std::vector<SrcBatch<T>> batches;
    for (size_t q = 0; q < b.src.size(); q += kMaxSrcBatch) {
        SrcBatch<T> sb{};
        sb.count = static_cast<int>(std::min<size_t>(kMaxSrcBatch, b.src.size() - q));
        for (int j = 0; j < sb.count; ++j) {
            sb.idx[j] = b.src[q + j].first;
            sb.inst[j] = b.src_inst[q + j];
            sb.val[j] = static_cast<T>(b.src[q + j].second);
        }
        batches.push_back(sb);
    }
    if (alone) {
        for (auto& sb : batches)
            HIP_TRY(timed(prof, EIK_KERNEL_OTHER, [&] { return launch_seed<T>(phi, w.lab, sb, s); }));
        launched += static_cast<int64_t>(batches.size());
    }

    const T eT = static_cast<T>(eps);
    // The launches of a solve form one chain: launch t drains list t and fills
    // list t + 1; lists alternate two buffers and three counter sets (the set
    // of list t + 2 is cleared by launch t).
    auto iter_args = [&](int64_t t, int phase) {
        TileIter<T> a{};
        sched_fill(a, w.q, t, ordered && !(alone && phase == 0), omin, static_cast<int>(t & 1), phase, w.ctl,
                   w.blkstat);
        if (!async && !pageable) a.mail = host_slots().mail + (t & (HostSlots::kMail - 1));
        a.F = F;
        a.phi = phi;
        a.lab = w.lab;
        a.cells = static_cast<const T*>(w.cells);
        a.early = !alone && phase == 0 && b.nd == 3 && sizeof(T) == 4 ? 1 : 0;
        return a;
    };
    // a kernel that only adds to list t, before launch t drains it (beside
    // launch t - 1, whose tag it claims tiles with)
    auto producer_args = [&](int64_t t, int phase) {
        TileIter<T> a = iter_args(t + 1, phase);
        a.next = w.q.list_of(t);
        a.mask_next = w.q.tmask + static_cast<size_t>(t & 1) * w.q.ntiles;
        a.key_next = w.q.keys + static_cast<size_t>(t & 1) * w.q.ntiles;
        a.ordered = ordered ? 1 : 0;
        a.first = 0;
        return a;
    };
    auto detect = [&](int64_t t) {
        return timed(prof, EIK_KERNEL_DETECT, [&] { return k.detect(producer_args(t, 1), geom, eT, gt, s); });
    };
    auto visits = [&](int64_t t, int phase, bool first) {
        TileIter<T> a = iter_args(t, phase);
        a.first = first ? 1 : 0;
        // The correcting update step takes every drop: with the tolerance a node
        // may keep a value up to eps above its solve (64^2 float64 at eps =
        // 1e-12: 1.3e-15 from the solution instead of 1e-17).
        return timed(prof, phase == 0 ? EIK_KERNEL_UPDATE : EIK_KERNEL_REMEDY,
                     [&] { return k.remedy(a, geom, phase == 0 ? T(0) : eT, inner, gt, s); });
    };
    auto counts = [&](int64_t t) { return w.q.count_of(static_cast<int>(t % 3)); };

    // Sources, and the initial list: the tiles next to them; with many sources a
    // dense pass finds those.  (One launch per 64 sources up to 8 of them, about
    // what the dense pass over a 4 M node grid costs.)
    const bool queue = batches.size() <= 8;
    TileIter<T> a0 = producer_args(0, 0);
    if (alone) a0.ordered = 0;
    auto sources = [&](const BatchGeom<T>& g, const TileCfg& tc, T* cells, bool q) {
        for (auto& sb : batches)
            HIP_TRY(timed(prof, EIK_KERNEL_OTHER, [&] {
                hipLaunchKernelGGL(k_tile_sources<T>, dim3(1), dim3(kMaxSrcBatch), 0, s, static_cast<const Sched&>(a0), g,
                                   b.nd, tc.tx, tc.ty, tc.tz, sb, phi, cells, q ? 1 : 0);
                return hipGetLastError();
            }));
        launched += static_cast<int64_t>(batches.size());
        return EIK_OK;
    };
    // (the update step alone may queue tiles of another shape than the cells')
    eik_status rs = skip_remedy ? EIK_OK : sources(geom, c, static_cast<T*>(w.cells), queue && !alone);
    if (rs == EIK_OK && alone && queue) rs = sources(geom_u, cu, nullptr, true);
    if (rs != EIK_OK) return rs;
    if (!queue && alone) {
        HIP_TRY(timed(prof, EIK_KERNEL_OTHER, [&] {
            hipLaunchKernelGGL(k_seed_all_tiles, dim3(std::min((ntiles_u + kBlock - 1) / kBlock, 1024)), dim3(kBlock),
                               0, s, ntiles_u, w.q.tstamp, w.q.list_of(0));
            return hipGetLastError();
        }));
        launched += 1;
    } else if (!queue) {
        HIP_TRY(detect(0));
        launched += 1;
    }

    // STEP 2.  By default the update step corrects as it goes: from the
    // sources outward, tile visits by the remedy rule (a node that drops lists
    // its neighbours again), lowest keys first, until no tile is queued.  A
    // front that first converged whole tiles without looking back (the update
    // step alone) left 43 evaluations per node to the remedy on a 2D
    // lognormal 4096^2 grid; corrected while the front is near, the same
    // solution takes 36 in all (45.5 -> 28.3 ms; 256^3 maze 13.2 -> 9.1 ms,
    // layered 192^3 5.4 -> 3.3 ms).
    int64_t n2 = 0;
    auto loop = [&](auto step, int64_t first, int64_t most, int64_t* steps, bool report) {
        auto cnt = [&](int64_t t) { return counts(first + t); };
        if (async || pageable)
            return run_loop(step, cnt, kSub * kPad, most, async, s, steps, w.ctl, pageable, report);
        return run_tile_loop(step, cnt, kSub * kPad, first, most, s, steps);
    };
    eik_status rc = loop(
        [&](int64_t t) {
            if (!alone) return visits(t, 0, false);
            return timed(prof, EIK_KERNEL_UPDATE,
                         [&] { return ku.update(iter_args(t, 0), geom_u, eT, inner_upd, gt, s); });
        },
        0, cap2, &n2, alone);
    launched += n2;
    if (rc == EIK_ERR_NO_CONVERGENCE && !alone) {  // the remedy loop takes up what is listed
        g_last_error.clear();
        rc = EIK_OK;
    }
    Results res;
    bool have = false;  // res holds the call's results
    if (rc == EIK_OK && !skip_remedy) {
        // STEP 3: detection adds to the list the next launch drains (what the
        // update step left over is still in it), then the remedy loop.  A
        // synchronous call reads the list's length first, with its results: unless
        // the correcting update step ran out of launches it is empty.
        HIP_TRY(detect(n2));
        launched += 1;
        int64_t n3 = 0;
        if (!async && !alone) {
            rc = read_results(w.ctl, w.blkstat, kMaxStatBlocks, pageable, s, res, counts(n2), kSub * kPad);
            if (rc != EIK_OK) return rc;
            have = res.open == 0;
        }
        if (!have) {
            rc = loop([&](int64_t t) { return visits(n2 + t, 1, t == 0); }, n2, cap, &n3, true);
            launched += n3;
        }
    }
    if (async) return rc;
    if (!have) {
        const eik_status rr = read_results(w.ctl, w.blkstat, kMaxStatBlocks, pageable, s, res);
        if (rr != EIK_OK) return rr;
    }
    if (res.ctl.err & 1) return fail(EIK_ERR_INVALID_ARGUMENT, "F has negative or non-finite values");
    if (st) {
        *st = eik_stats{};
        st->step2_iters = static_cast<int64_t>(res.ctl.iters2);
        st->step3_iters = static_cast<int64_t>(res.ctl.iters3);
        st->evals_step2 = static_cast<int64_t>(res.sum[SF_EVALS2]);
        st->evals_detect = (o.flags & EIK_FLAG_SKIP_REMEDY) ? 0 : b.n - static_cast<int64_t>(b.src.size());
        st->evals_remedy = static_cast<int64_t>(res.sum[SF_EVALS3]);
        st->remedy_initial = static_cast<int64_t>(res.ctl.remedy_init);
        st->max_active = static_cast<int64_t>(res.ctl.max_active);
        st->launches = launched;
        st->tile_visits_step2 = static_cast<int64_t>(res.sum[SF_VISITS2]);
        st->tile_visits_step3 = static_cast<int64_t>(res.sum[SF_VISITS3]);
        st->inner_step2 = static_cast<int64_t>(res.sum[SF_INNER2]);
        st->inner_step3 = static_cast<int64_t>(res.sum[SF_INNER3]);
        st->written_step2 = static_cast<int64_t>(res.sum[SF_WRITTEN2]);
        st->written_step3 = static_cast<int64_t>(res.sum[SF_WRITTEN3]);
        st->evals_early = static_cast<int64_t>(res.sum[SF_CHECK]);
        HIP_TRY(prof.collect(st));
    }
    return rc;
}

template eik_status solve_tile<float>(const Batch&, const float*, double, float*, const eik_options&, char*,
                                      hipStream_t, eik_stats*);
template eik_status solve_tile<double>(const Batch&, const double*, double, double*, const eik_options&, char*,
                                       hipStream_t, eik_stats*);

}  // namespace eik
