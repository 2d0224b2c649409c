// The resident step of one structured Q4 grid (gfx950): a launch of up to
// kResidentMaxSteps time steps whose whole state stays on the chip.
//
// k_step runs one launch per step: every workgroup stages its tile from
// memory, recomputes the element gradients (four divisions per element) and
// hands the pick to the next launch.  On a model of one round of workgroups
// such a step is one chain of latencies, 12 to 14 us on a 40 x 40 plate and on
// a 400 x 400 one alike.  Here every workgroup owns a tile of nodes for the
// whole launch: u lives in LDS, v, 1/m, the gradients at the edge midpoints and
// the smoothing weights in registers (tiles of 768 elements in binary64 spill 16
// values per thread, 57 with sub-cells; of 1 024 in binary32 one or two), the
// lists of free-surface candidates and split elements in LDS.  Per step the
// workgroups exchange the nodes within two of their borders and one candidate
// slot each, as tagged words (mct2d_exchange.h).
//
// What bounds it: the slowest tile's chain of four barriers (latencies of LDS and
// dependent arithmetic with three wavefronts per SIMD; its candidates and split
// pieces) and one exchange through the memory side, 0.7 us there and back.  On the
// 400 x 400 plate with an element splitting in every step a wavefront issues 392
// vector instructions per step, a fifth of what the SIMDs could, and waits for 77 %
// of its cycles.  Per step, before -> after: 400 x 400 plate 13.3 -> 6.1 us
// (binary32 11.9 -> 4.6), 301 x 187 with sub-cells 11.0 -> 5.3, 40 x 40 with cracks
// running 12.4 -> 4.4.
//
// The arithmetic is k_step's, operation for operation, so results are the
// same bits: strains at the four edge midpoints, the smoothed stress of an
// edge by its higher-id intact element, forces, colour-ordered gather, G of
// the candidates, pick and update.
//
// What waits for what in step s:
//   - the pick of step s - 1 acts on the codes and lists; strains of the ring;
//   - barrier, smoothed stresses; barrier, forces, split pieces, candidates
//     (the last wavefront with candidates publishes the tile's slot);
//   - barrier, sum and advance the nodes, send the border nodes;
//   - the first wavefronts receive the halo while the last ones take every
//     tile's slot of step s, one per lane, and reduce them to its pick; barrier.
#include "mct2d_device.h"
#include "mct2d_exchange.h"
#include "mct2d_impl.h"
#include "mct2d_resident.h"

#include <algorithm>
#include <climits>
#include <vector>

namespace mct {

namespace {
using namespace dev;
using namespace res;

template <class T>
struct ResidentArgs {
    StepParamsT<T> p;
    int32_t ntx, nwg;  // tiles per row, tiles
    int32_t n, par0;   // steps of this launch, parity of its first one
    uint32_t epoch0;   // epoch of the state the launch starts from
    uint64_t *xb, *slots;
    uint32_t *err;
};

// Tile shapes, by class: elements of the ring (one thread each) around the
// tile's nodes.
template <int C>
struct ResidentTile;
template <>
struct ResidentTile<256> {
    static constexpr int TXE = 16, TYE = 16;
};
template <>
struct ResidentTile<512> {
    static constexpr int TXE = 22, TYE = 23;
};
template <>
struct ResidentTile<768> {
    static constexpr int TXE = 27, TYE = 28;
};
template <>
struct ResidentTile<1024> {
    static constexpr int TXE = 32, TYE = 32;
};

// Threads of a workgroup: where the registers allow it, four wavefronts more
// than the ring's, which take the candidates, split pieces, outer elements
// and slots while the others do the ring's work.
template <class T, int C>
constexpr int resident_threads() {
    return C == 256 ? 512 : C;
}

// Layout of a tile and its LDS (byte offsets).
template <class T, int C>
struct Res {
    static constexpr int NT = resident_threads<T, C>();
    static constexpr bool HELP = NT > C;
    static constexpr int TXE = ResidentTile<C>::TXE, TYE = ResidentTile<C>::TYE;
    static constexpr int TX = TXE - 1, TY = TYE - 1;  // owned nodes
    static constexpr int HX = TXE + 3, HY = TYE + 3;  // staged nodes
    static constexpr int EX = TXE + 2, EY = TYE + 2;  // staged elements
    static constexpr int NR = TXE * TYE, NH = TXE * (TYE + 1), NS = NH + (TXE + 1) * TYE;
    static constexpr int NO = 2 * (TXE + TYE), HN = HX * HY;
    static constexpr int cap = 4 * (TX + TY);  // nodes sent: stride of the words of one kind
    // the large binary64 tiles keep fewer candidates' normals: their LDS would not
    // fit into 160 KB otherwise
    static constexpr int NC = sizeof(T) == 8 && C > 512 ? 96 : C < 512 ? 384 : 256;  // candidates that keep their normals
    static constexpr int up(int n) { return (n + 15) & ~15; }
    static constexpr int S = (int)sizeof(T);
    static constexpr int u = 0, xy = u + up(2 * HN * S), e = xy + up(2 * HN * S);
    static constexpr int fe = e + up(3 * NS * S), og = fe + up(8 * NR * S), cn = og + up(13 * NO * S);
    static constexpr int ci = cn + up(8 * NC * S), gc = ci + up(32 * NC), bc = gc + up(NR * S), cand = bc + up(4 * cap * S);
    static constexpr int splitl = cand + up(4 * TX * TY * 2), split = splitl + up(NR * 2);
    static constexpr int code = split + up(EX * EY), total = code + up(NT);
    static_assert(total + 5120 <= 160 * 1024, "the LDS of a compute unit (with the static arrays)");
    static_assert(NR <= NT && NO <= NT && 4 * HX + 4 * TY <= NT - 64 * kPickWaves,
                  "one thread per ring and outer element; halo nodes beside the slots");
};

// Position of node (l, m) of a tile of tw x th nodes among the nodes it sends
// (those within two of its border): the two lowest rows, the two highest,
// then four per row between them.
__device__ __forceinline__ int send_index(int l, int m, int tw, int th) {
    if (m < 2) return m * tw + l;
    if (m >= th - 2) return (2 + m - (th - 2)) * tw + l;
    return 4 * tw + (m - 2) * 4 + (l < 2 ? l : 2 + l - (tw - 2));
}


template <class T, int C, bool SC>
__global__ __launch_bounds__((resident_threads<T, C>())) void k_resident(const ResidentArgs<T> A) {
    using R = Res<T, C>;
    constexpr int NT = R::NT;
    constexpr int NW = NT / 64, PW = xch::pair_words<T>();
    constexpr int TX = R::TX, TY = R::TY, TXE = R::TXE, TYE = R::TYE, HX = R::HX, EX = R::EX, EY = R::EY;
    constexpr int NR = R::NR, NH = R::NH, NS = R::NS, NO = R::NO, HN = R::HN, NC = R::NC;
    static_assert(NW >= kPickWaves && kPickWaves * 64 >= kResidentMaxTiles, "one slot per polling lane");
    extern __shared__ char smem[];
    const StepParamsT<T> &p = A.p;
    T *const s_ux = reinterpret_cast<T *>(smem + R::u), *const s_uy = s_ux + HN;
    T *const s_X = reinterpret_cast<T *>(smem + R::xy), *const s_Y = s_X + HN;
    T *const s_e = reinterpret_cast<T *>(smem + R::e);    // per edge slot and component (stride NS)
    T *const s_fe = reinterpret_cast<T *>(smem + R::fe);  // per component of the four nodes (stride NR)
    T *const s_og = reinterpret_cast<T *>(smem + R::og);  // outer elements: gradients at the shared edge, weights, strain
    T *const s_cn = reinterpret_cast<T *>(smem + R::cn);  // path normals of the first NC candidates
    int2 *const s_ci = reinterpret_cast<int2 *>(smem + R::ci);  // and their places: nodes, edge slot, element
    T *const s_gc = reinterpret_cast<T *>(smem + R::gc);  // of the ring elements
    T *const s_bc = reinterpret_cast<T *>(smem + R::bc);  // tractions and prescribed velocities of perimeter nodes
    uint16_t *const s_cand = reinterpret_cast<uint16_t *>(smem + R::cand);
    uint16_t *const s_splitl = reinterpret_cast<uint16_t *>(smem + R::splitl);
    uint8_t *const s_split = reinterpret_cast<uint8_t *>(smem + R::split);  // staged elements, at the start
    uint8_t *const s_code = reinterpret_cast<uint8_t *>(smem + R::code);    // ring elements, kept
    __shared__ int s_ncand, s_ncorner, s_nthru;  // entries of the lists
    __shared__ int s_nred, s_stop;
    __shared__ int s_narr, s_npicks;  // wavefronts that took their slots; splits of the launch (tile 0)
    __shared__ int s_pick;            // the pick: staged element | code << 16, or -1 (none, or elsewhere)
    __shared__ Best<T> s_red[NW], s_pk[kPickWaves];
    __shared__ T s_phi;
    __shared__ int2 s_picks[kResidentMaxSteps];  // tile 0: the launch's splits

    const int tid = threadIdx.x, lane = tid & 63, tile = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nx = p.nx, ny = p.ny;
    const int i0 = (tile % A.ntx) * TX, j0 = (tile / A.ntx) * TY;
    const int tw = min(TX, nx + 1 - i0), th = min(TY, ny + 1 - j0);
    const int64_t base = p.ctl->base;
    const int64_t nsplit0 = p.ctl->nsplit;
    auto corner = [](int n) { return n == 0 ? 0 : n == 1 ? 1 : n == 2 ? HX + 1 : HX; };
    auto edge_slot = [](int ie, int je, int k) {
        return k == 0 ? je * TXE + ie
             : k == 1 ? NH + je * (TXE + 1) + ie + 1
             : k == 2 ? (je + 1) * TXE + ie
                      : NH + je * (TXE + 1) + ie;
    };

    // ---- the state, once per launch ---------------------------------------
    {
        const T *ux = A.par0 ? p.ux1 : p.ux0, *uy = A.par0 ? p.uy1 : p.uy0;
        for (int idx = tid; idx < HN; idx += NT) {
            const int gi = i0 - 2 + idx % HX, gj = j0 - 2 + idx / HX;
            T a = T(0), b = T(0), c = T(0), d = T(0);
            if (gi >= 0 && gi <= nx && gj >= 0 && gj <= ny) {
                const int64_t n = (int64_t)gj * (nx + 1) + gi;
                a = ux[n];
                b = uy[n];
                c = p.X[n];
                d = p.Y[n];
            }
            s_ux[idx] = a;
            s_uy[idx] = b;
            s_X[idx] = c;
            s_Y[idx] = d;
        }
        for (int idx = tid; idx < EX * EY; idx += NT) {
            const int gi = i0 - 2 + idx % EX, gj = j0 - 2 + idx / EX;
            uint8_t code = kAbsent;
            if (gi >= 0 && gi < nx && gj >= 0 && gj < ny) code = p.split[(int64_t)gj * nx + gi];
            s_split[idx] = code;
        }
        if (tid == 0) {
            s_ncand = s_ncorner = s_nthru = s_nred = s_stop = s_narr = s_npicks = 0;
            s_pick = -1;
            s_phi = T(1);
        }
    }
    __syncthreads();

    auto elem_xy = [&](int nb, T x[4], T y[4]) {
        x[0] = s_X[nb]; x[1] = s_X[nb + 1]; x[2] = s_X[nb + HX + 1]; x[3] = s_X[nb + HX];
        y[0] = s_Y[nb]; y[1] = s_Y[nb + 1]; y[2] = s_Y[nb + HX + 1]; y[3] = s_Y[nb + HX];
    };
    auto elem_u = [&](int nb, T ux[4], T uy[4]) {
        ux[0] = s_ux[nb]; ux[1] = s_ux[nb + 1]; ux[2] = s_ux[nb + HX + 1]; ux[3] = s_ux[nb + HX];
        uy[0] = s_uy[nb]; uy[1] = s_uy[nb + 1]; uy[2] = s_uy[nb + HX + 1]; uy[3] = s_uy[nb + HX];
    };
    // (sub-cell) area of the staged element (ex, ey) at its edge k; gi, gj: its grid indices
    auto area_of = [&](int gi, int gj) { return p.area[(int64_t)gj * nx + gi]; };
    auto sub_area = [&](int nb, int k) {
        T x[4], y[4], b[3], c[3];
        elem_xy(nb, x, y);
        return subcell_rt(x, y, static_cast<const T *>(nullptr), static_cast<const T *>(nullptr), k, b, c,
                          static_cast<T *>(nullptr));
    };

    // this thread's ring element
    const bool ring = tid < NR, rings = wave * 64 < NR;
    const int ie = ring ? tid % TXE : 0, je = ring ? tid / TXE : 0;
    const int gi = i0 - 1 + ie, gj = j0 - 1 + je;
    const int e2 = (je + 1) * EX + ie + 1, nb = (je + 1) * HX + ie + 1;
    uint8_t code = ring ? s_split[e2] : kAbsent;
    s_code[tid] = code;
    unsigned nbs = 0;  // bit k: the neighbour across edge k is split or outside the grid
    T gx[4][4], gy[4][4], at[4], c4 = T(0);
    T wb0 = T(0), wb1 = T(0), wl0 = T(0), wl1 = T(0);  // weights (lower id, own) of edges 0 and 3
    if (ring && code != kAbsent) {
        nbs = (s_split[e2 - EX] != 0 ? 1u : 0u) | (s_split[e2 + 1] != 0 ? 2u : 0u) | (s_split[e2 + EX] != 0 ? 4u : 0u) |
              (s_split[e2 - 1] != 0 ? 8u : 0u);
        T x[4], y[4];
        elem_xy(nb, x, y);
        T Ab, Al, A0, A3;
        if constexpr (SC) {
            at[0] = subcell<0>(x, y, static_cast<const T *>(nullptr), static_cast<const T *>(nullptr), gx[0], gy[0],
                               static_cast<T *>(nullptr));
            at[1] = subcell<1>(x, y, static_cast<const T *>(nullptr), static_cast<const T *>(nullptr), gx[1], gy[1],
                               static_cast<T *>(nullptr));
            at[2] = subcell<2>(x, y, static_cast<const T *>(nullptr), static_cast<const T *>(nullptr), gx[2], gy[2],
                               static_cast<T *>(nullptr));
            at[3] = subcell<3>(x, y, static_cast<const T *>(nullptr), static_cast<const T *>(nullptr), gx[3], gy[3],
                               static_cast<T *>(nullptr));
            A0 = at[0];
            A3 = at[3];
            Ab = gj > 0 ? sub_area(nb - HX, 2) : T(0);
            Al = gi > 0 ? sub_area(nb - 1, 1) : T(0);
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) q4_grad(x, y, k, gx[k], gy[k]);
            const T my = area_of(gi, gj);
            c4 = T(0.25) * my;
            A0 = A3 = my;
            Ab = gj > 0 ? area_of(gi, gj - 1) : T(0);
            Al = gi > 0 ? area_of(gi - 1, gj) : T(0);
        }
        s_gc[tid] = p.gc ? p.gc[(int64_t)gj * nx + gi] : p.gc_uniform;
        const T sb = Ab + A0, sl = Al + A3;
        wb0 = Ab / sb;
        wb1 = A0 / sb;
        wl0 = Al / sl;
        wl1 = A3 / sl;
    }
    int sidx[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) sidx[k] = edge_slot(ie, je, k);

    // Elements one further out take part through the edge they share with
    // the ring: the row below, the row above, the column left, the column
    // right.  Below and left are the lower-id side, above and right the higher.
    // fl: what this thread has to do (kept as bits and made opaque in every
    // step, as scalar masks held across the loop would be spilled)
    enum : unsigned { kOuter = 1, kOuterHi = 2, kOuterIn = 4, kOuterNb = 8, kOwn = 16, kSend = 32, kRecv = 64, kEdge = 128,
                     kOddX = 256, kOddY = 512, kFix0 = 1024 };
    unsigned fl = 0;
    const int o = NT - 1 - tid;
    // staged place (rex, rey) of outer element q, its local edge on the ring
    // and that edge's slot
    auto outer_at = [](int q, int &rex, int &rey, int &ork, int &sid) {
        if (q < TXE) {
            rex = q + 1; rey = 0; ork = 2; sid = q;
        } else if ((q -= TXE) < TXE) {
            rex = q + 1; rey = TYE + 1; ork = 0; sid = TYE * TXE + q;
        } else if ((q -= TXE) < TYE) {
            rex = 0; rey = q + 1; ork = 1; sid = NH + q * (TXE + 1);
        } else {
            q -= TYE;
            rex = TXE + 1; rey = q + 1; ork = 3; sid = NH + q * (TXE + 1) + TXE;
        }
    };
    auto across = [](int rex, int rey, int ork, int &nrx, int &nry) {  // the ring element across that edge
        nrx = ork == 1 ? rex + 1 : ork == 3 ? rex - 1 : rex;
        nry = ork == 2 ? rey + 1 : ork == 0 ? rey - 1 : rey;
    };
    int oat = 0;  // node 0 of the outer element | edge slot << 16
    if (o < NO) {
        int rex, rey, ork, osid, nrx, nry;
        outer_at(o, rex, rey, ork, osid);
        across(rex, rey, ork, nrx, nry);
        const bool ohi = ork == 0 || ork == 3;
        const int onb = rey * HX + rex;
        oat = onb | osid << 16;
        const int ogi = i0 - 2 + rex, ogj = j0 - 2 + rey;
        const uint8_t oc = s_split[rey * EX + rex];
        fl |= kOuter | (ohi ? kOuterHi : 0u) | (oc == 0 ? kOuterIn : 0u) |
              (s_split[nry * EX + nrx] != 0 ? kOuterNb : 0u);
        if (oc != kAbsent) {
            T x[4], y[4], dx[4], dy[4], Ao, Alo = T(0);
            elem_xy(onb, x, y);
            const bool lo_in = s_split[nry * EX + nrx] != kAbsent;
            if constexpr (SC) {
                Ao = subcell_rt(x, y, static_cast<const T *>(nullptr), static_cast<const T *>(nullptr), ork, dx, dy,
                                static_cast<T *>(nullptr));
                dx[3] = dy[3] = T(0);
                if (ohi && lo_in) Alo = sub_area(nry * HX + nrx, ork == 0 ? 2 : 1);
            } else {
                q4_grad_rt(x, y, ork, dx, dy);
                Ao = area_of(ogi, ogj);
                if (ohi && lo_in) Alo = area_of(i0 - 2 + nrx, j0 - 2 + nry);
            }
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                s_og[n * NO + o] = dx[n];
                s_og[(4 + n) * NO + o] = dy[n];
            }
            const T sum = Alo + Ao;
            s_og[8 * NO + o] = Alo / sum;
            s_og[9 * NO + o] = Ao / sum;
            if constexpr (SC) {  // the edge's local index, needed for the corner displacements
                s_og[3 * NO + o] = T(ork);
            }
        }
    }

    // this thread's owned node
    const int on_l = tid % TX, on_m = tid / TX;
    const bool own = on_l < tw && on_m < th;
    T n_minv = T(0), n_vx = T(0), n_vy = T(0);
    if (own) {
        const int on_n = (j0 + on_m) * (nx + 1) + (i0 + on_l);
        n_minv = p.minv[on_n];
        n_vx = p.vx[on_n];
        n_vy = p.vy[on_n];
        const int si = send_index(on_l, on_m, tw, th);
        const int pidx = perimeter_index(i0 + on_l, j0 + on_m, nx, ny);
        fl |= kOwn;
        if ((i0 - 1 + on_l) & 1) fl |= kOddX;
        if ((j0 - 1 + on_m) & 1) fl |= kOddY;
        if (pidx >= 0) {  // a border node of its tile
            fl |= kEdge | p.vmask_p[pidx] * kFix0;
            s_bc[4 * si] = p.fext_p[2 * pidx];
            s_bc[4 * si + 1] = p.fext_p[2 * pidx + 1];
            s_bc[4 * si + 2] = p.v0_p[2 * pidx];
            s_bc[4 * si + 3] = p.v0_p[2 * pidx + 1];
        }
        if (on_l < 2 || on_l >= tw - 2 || on_m < 2 || on_m >= th - 2) fl |= kSend;
    }
    // this thread's halo node: two rows below and above, two columns left and right
    int recv_at = 0;  // its word among the sent ones << 11 | its place
    if (tid < 4 * HX + 4 * TY) {
        int hx, hy;
        if (tid < 4 * HX) {
            hx = tid % HX;
            hy = tid / HX;
            if (hy >= 2) hy += TY;
        } else {
            const int q = tid - 4 * HX;
            hy = 2 + (q >> 2);
            hx = q & 3;
            if (hx >= 2) hx += TX;
        }
        const int ni = i0 - 2 + hx, nj = j0 - 2 + hy;
        if (ni >= 0 && ni <= nx && nj >= 0 && nj <= ny) {
            const int ti = ni / TX, tj = nj / TY;
            fl |= kRecv;
            recv_at = (tj * A.ntx + ti) * PW * R::cap +
                      send_index(ni - ti * TX, nj - tj * TY, min(TX, nx + 1 - ti * TX), min(TY, ny + 1 - tj * TY));
            recv_at = recv_at << 11 | (hy * HX + hx);
        }
    }
    // The arguments are read again where they are used (through an opaque
    // pointer to the kernel's arguments): held across the loop they would take
    // more scalar registers than there are.
    using Args = const __attribute__((address_space(4))) ResidentArgs<T> *;
    const Args args = (Args)__builtin_amdgcn_kernarg_segment_ptr();
    auto again = [&]() {
        Args q = args;
        asm volatile("" : "+s"(q));
        return q;
    };
    auto material = [&]() {
        const Args q = again();
        StepParamsT<T> m;
        m.D11 = q->p.D11;
        m.D12 = q->p.D12;
        m.D33 = q->p.D33;
        m.E = q->p.E;
        return m;
    };

    const int pickers = (A.nwg + 63) / 64;  // wavefronts that take the slots
    const bool curve = p.ncurve > 0;
    int curve_i = 0;   // load curve: position of the last step's time
    int ncached = 0;   // candidates whose path normals are in s_cn
    bool stopped = false;

    // Takes the slots of epoch ep (words sw already loaded from at); the last
    // of the wavefronts that do leaves the pick of that step in s_pick, and in
    // tile 0 records it.
    // (by the last wavefronts: the first ones receive the halo)
    const bool picks = NW - 1 - wave < pickers;
    auto take_slots = [&](const uint64_t *at, int count, uint32_t ep, int64_t step, int slot_id, xch::SlotWords &sw) {
        Best<T> g;
        best_none(g);
        bool has = false;
        if (slot_id < count) {
            int e = 0, a = 0, k = 0;
            double G = 0.0, Gm = 0.0;
            if (!xch::take_slot(at, count, ep, sw, has, e, a, k, G, Gm)) s_stop = 1;
            if (has) {
                g.G = T(G);
                g.Gmin = T(Gm);
                g.e = e;
                g.a = a;
                g.k = k;
            }
        }
        const uint64_t hm = __ballot(has);
        if (hm != 0ull) best_wave(g, hm);
        if (pickers > 1) {
            // counted in the low bits; a bit above for each that has a candidate
            int arrived = 0;
            if (lane == 0) {
                const int w = NW - 1 - wave, mine = 1 + (hm != 0ull ? 256 << w : 0);
                if (hm != 0ull) s_pk[w] = g;
                arrived = mine + __hip_atomic_fetch_add(&s_narr, mine, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            arrived = __builtin_amdgcn_readfirstlane(arrived);
            if ((arrived & 255) != pickers) return;
            const int others = (arrived >> 8) & ~(hm != 0ull ? 1 << (NW - 1 - wave) : 0);
            if (others) {
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                for (int w = 0; w < pickers; ++w)
                    if ((others >> w) & 1) best_merge(g, s_pk[w].G, s_pk[w].Gmin, s_pk[w].e, s_pk[w].a, s_pk[w].k);
            }
        }
        if (lane != 0) return;
        s_narr = 0;
        // MCT pick: G* > gamma (G* - G_c) against every other accepted candidate,
        // so against the smallest G
        int local = -1;
        const Args q = again();
        if (g.G >= T(0) && g.G > q->p.gamma * (g.G - g.Gmin)) {
            const int ej = g.e / nx, fy = ej - (j0 - 2), fx = g.e - ej * nx - (i0 - 2);
            const int pc = kSplitFlag | (g.a << 2) | g.k;
            if (fx >= 0 && fx < EX && fy >= 0 && fy < EY) local = (fy * EX + fx) | pc << 16;
            if (tile == 0) {
                const int i = s_npicks;
                s_picks[i] = make_int2(g.e, pc);
                s_npicks = i + 1;
                if (nsplit0 + i < q->p.log_cap) {
                    LogRec r;
                    r.step = (int32_t)step;
                    r.elem = g.e;
                    r.entry = (uint8_t)g.a;
                    r.exit = (uint8_t)g.k;
                    r.pad0 = r.pad1 = 0;
                    r.pad2 = 0;
                    r.G = (double)g.G;
                    q->p.log[nsplit0 + i] = r;
                }
            }
        }
        s_pick = local;
    };

    const int nwg = A.nwg, slot_half = nwg * xch::kSlotWords, xb_half = nwg * (PW * R::cap);
    uint64_t *const slots = A.slots, *const xbuf = A.xb;
    const T gamma = p.gamma, dts = p.dts;
    // The lists only grow within a launch: an (element, edge) pair becomes a
    // candidate once, and the entries of an element that split are skipped.
    // Candidates: owned elements (their node 0 is owned), edges with a split
    // or absent neighbour.  Split ring elements: corner splits from the front
    // of s_splitl (a constant-strain triangle), through splits from the back
    // (two bars).
    auto list_split = [&]() {
        if ((((code & 3) - ((code >> 2) & 3)) & 3) == 2)
            s_splitl[NR - 1 - atomicAdd(&s_nthru, 1)] = (uint16_t)tid;
        else
            s_splitl[atomicAdd(&s_ncorner, 1)] = (uint16_t)tid;
    };
    if (code & kSplitFlag) list_split();
    if (ie >= 1 && je >= 1 && code == 0)
        for (int k = 0; k < 4; ++k)
            if ((nbs >> k) & 1u) s_cand[atomicAdd(&s_ncand, 1)] = (uint16_t)((tid << 2) | k);
    if (code == kAbsent && ring)
        for (int c = 0; c < 8; ++c) s_fe[c * NR + tid] = T(0);

    // every load of the set-up done: a wait for one of them in the loop would
    // also wait for the stores under way there
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : "+v"(n_minv), "+v"(n_vx), "+v"(n_vy) : : "memory");
    const int nsteps = A.n;
    for (int s = 0; s < nsteps; ++s) {
        const uint32_t ep = A.epoch0 + (uint32_t)s;  // of u^k and of step s - 1's slots
        asm volatile("" : "+v"(fl));
        // ---- the pick of the step before acts on the codes from here ------------
        const StepParamsT<T> mat = material();
        if (const int pick = s_pick; pick >= 0) {  // uniform
            const int pe = pick & 0xFFFF;
            const uint8_t pc = (uint8_t)(pick >> 16);
            int tr = tid;
            asm volatile("" : "+v"(tr));
            const int rje = tr / TXE, rie = tr - rje * TXE, re = (rje + 1) * EX + rie + 1;
            if (code == 0) {
                const unsigned nw = ((pe == re - EX ? 1u : 0u) | (pe == re + 1 ? 2u : 0u) | (pe == re + EX ? 4u : 0u) |
                                     (pe == re - 1 ? 8u : 0u)) & ~nbs;
                if (nw) {
                    nbs |= nw;
                    if (rie >= 1 && rje >= 1) s_cand[atomicAdd(&s_ncand, 1)] = (uint16_t)((tid << 2) | __builtin_ctz(nw));
                }
                if (re == pe) {
                    code = pc;
                    s_code[tid] = pc;
                    list_split();
                }
            }
            if (fl & kOuter) {
                int rex, rey, ork, sid, nrx, nry;
                outer_at(NT - 1 - tr, rex, rey, ork, sid);
                across(rex, rey, ork, nrx, nry);
                if (rey * EX + rex == pe) fl &= ~kOuterIn;
                if (nry * EX + nrx == pe) fl |= kOuterNb;
            }
        }

        // ---- strains ------------------------------------------------------------
        T qh0[3], qh3[3];
        if (rings) {  // uniform over the wavefront
            T ux[4], uy[4];
            elem_u(nb, ux, uy);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                T q[3];
                if constexpr (SC) {
                    const int k1 = (k + 1) & 3;
                    const T pu[3] = {ux[k], ux[k1], T(0.25) * (((ux[0] + ux[1]) + ux[2]) + ux[3])};
                    const T pv[3] = {uy[k], uy[k1], T(0.25) * (((uy[0] + uy[1]) + uy[2]) + uy[3])};
                    strain<3>(gx[k], gy[k], pu, pv, q);
                } else {
                    strain<4>(gx[k], gy[k], ux, uy, q);
                }
                if (k == 0) {
                    qh0[0] = q[0]; qh0[1] = q[1]; qh0[2] = q[2];
                } else if (k == 3) {
                    qh3[0] = q[0]; qh3[1] = q[1]; qh3[2] = q[2];
                } else if (code == 0) {  // (what absent elements compute is not used)
#pragma unroll
                    for (int c = 0; c < 3; ++c) s_e[c * NS + sidx[k]] = q[c];
                }
            }
        }
        if (fl & kOuterIn) {
            T ux[4], uy[4], dx[4], dy[4], oq[3];
            const int osid = oat >> 16;
            elem_u(oat & 0xFFFF, ux, uy);
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                dx[n] = s_og[n * NO + o];
                dy[n] = s_og[(4 + n) * NO + o];
            }
            if constexpr (SC) {
                const int k = (int)dx[3];
                const T mu = T(0.25) * (((ux[0] + ux[1]) + ux[2]) + ux[3]);
                const T mv = T(0.25) * (((uy[0] + uy[1]) + uy[2]) + uy[3]);
                const T pu[3] = {k == 0 ? ux[0] : k == 1 ? ux[1] : k == 2 ? ux[2] : ux[3],
                                 k == 0 ? ux[1] : k == 1 ? ux[2] : k == 2 ? ux[3] : ux[0], mu};
                const T pv[3] = {k == 0 ? uy[0] : k == 1 ? uy[1] : k == 2 ? uy[2] : uy[3],
                                 k == 0 ? uy[1] : k == 1 ? uy[2] : k == 2 ? uy[3] : uy[0], mv};
                strain<3>(dx, dy, pu, pv, oq);
            } else {
                strain<4>(dx, dy, ux, uy, oq);
            }
            T *const to = (fl & kOuterHi) ? s_og + 10 * NO + o : s_e + osid;
            const int step_c = (fl & kOuterHi) ? NO : NS;
#pragma unroll
            for (int c = 0; c < 3; ++c) to[c * step_c] = oq[c];
        }
        if (curve && tid == NT - 1) {
            // load_factor, walking on from the last step's place in the curve
            const Args q = again();
            const double *const ct = q->p.curve_t, *const cp = q->p.curve_phi;
            const int nc = q->p.ncurve;
            const double t = (double)(base + s) * q->p.dt;
            double f;
            if (t <= ct[0]) {
                f = cp[0];
            } else if (t >= ct[nc - 1]) {
                f = cp[nc - 1];
            } else {
                while (ct[curve_i + 1] <= t) ++curve_i;
                const double slope = (cp[curve_i + 1] - cp[curve_i]) / (ct[curve_i + 1] - ct[curve_i]);
                f = cp[curve_i] + (t - ct[curve_i]) * slope;
            }
            s_phi = T(f);
        }
        __syncthreads();

        // ---- smoothed stresses ------------------------------------------------
        // the higher-id element of an edge, when intact, forms its stress;
        // otherwise the lower-id one does
        auto lo_of = [&](int sid, T lo[3]) {
#pragma unroll
            for (int c = 0; c < 3; ++c) lo[c] = s_e[c * NS + sid];
        };
        auto sigma_of = [&](bool alone, T w0, T w1, const T lo[3], const T q[3], int sid) {
            T eps[3], sg[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const T both = fmat(w1, q[c], w0 * lo[c]);
                eps[c] = alone ? q[c] : both;
            }
            hooke(mat, eps, sg);
#pragma unroll
            for (int c = 0; c < 3; ++c) s_e[c * NS + sid] = sg[c];
        };
        if (code == 0) {
            T lo0[3], lo3[3];
            lo_of(sidx[0], lo0);
            lo_of(sidx[3], lo3);
            sigma_of((nbs & 1u) != 0, wb0, wb1, lo0, qh0, sidx[0]);
            sigma_of((nbs & 8u) != 0, wl0, wl1, lo3, qh3, sidx[3]);
            if (nbs & 6u) {
#pragma unroll
                for (int k = 1; k < 3; ++k)
                    if ((nbs >> k) & 1u) {
                        T lo[3];
                        lo_of(sidx[k], lo);
                        sigma_of(true, T(0), T(0), lo, lo, sidx[k]);
                    }
            }
        }
        if ((fl & (kOuterIn | kOuterHi)) == (kOuterIn | kOuterHi)) {
            T lo[3], oq[3];
            lo_of(oat >> 16, lo);
#pragma unroll
            for (int c = 0; c < 3; ++c) oq[c] = s_og[(10 + c) * NO + o];
            sigma_of((fl & kOuterNb) != 0, s_og[8 * NO + o], s_og[9 * NO + o], lo, oq, oat >> 16);
        }
        __syncthreads();
        // (the bars start a wavefront of their own)
        const int ncand = s_ncand, ncorner = s_ncorner, bars0 = (ncorner + 63) & ~63, nitems = bars0 + 2 * s_nthru;
        if (ncand == 0 && tid == 0) xch::put_no_slot(slots + ((ep + 1) & 1u) * slot_half + tile, ep + 1);

        // ---- energy release rate and element rule: four lanes per candidate ----
        const int cwave = R::HELP ? NW - 1 - wave : wave;  // place of this wavefront among those with candidates
        int tq = cwave * 64 + lane;
        asm volatile("" : "+v"(tq));
        if (cwave * 16 < ncand) {  // uniform over the wavefront
            Best<T> best;
            best_none(best);
            for (int c0 = 0; c0 + cwave * 16 < ncand; c0 += NT / 4) {
                const int c = c0 + (tq >> 2), j = tq & 3;
                T Gj = T(0);
                bool H = false;
                // the first NC candidates keep their places and path normals
                const bool fresh = c >= ncached;
                int2 ci = make_int2(0, 0);
                if (c < ncand) {
                    if (fresh) {
                        const int ent = s_cand[c], ct = ent >> 2, ca = ent & 3, cie = ct % TXE, cje = ct / TXE;
                        const int nb0 = (cje + 1) * HX + (cie + 1);
                        ci.x = (nb0 + corner(ca)) | (nb0 + corner((ca + 1) & 3)) << 16;
                        ci.y = edge_slot(cie, cje, (ca + 1 + j) & 3) | ct << 16 | ca << 28;
                        if (c < NC) s_ci[4 * c + j] = ci;
                    } else {
                        ci = s_ci[4 * c + j];
                    }
                }
                const int t = (ci.y >> 16) & 0xFFF, a = ci.y >> 28;
                const T gc = s_gc[t];
                if (c < ncand && s_code[t] == 0) {
                    const int o1 = ci.x & 0xFFFF, o2 = ci.x >> 16, sid = ci.y & 0xFFFF;
                    const T X1 = s_X[o1], Y1 = s_Y[o1], X2 = s_X[o2], Y2 = s_Y[o2];
                    const T ux1 = s_ux[o1], uy1 = s_uy[o1], ux2 = s_ux[o2], uy2 = s_uy[o2];
                    const T sg[3] = {s_e[sid], s_e[NS + sid], s_e[2 * NS + sid]};
                    T nxv, nyv;
                    if (fresh) {
                        const int nb0 = (t / TXE + 1) * HX + t % TXE + 1, k = (a + 1 + j) & 3;
                        const int q0 = nb0 + corner(k), q1 = nb0 + corner((k + 1) & 3);
                        T len;
                        path_geom_pts(X1, Y1, X2, Y2, s_X[q0], s_Y[q0], s_X[q1], s_Y[q1], nxv, nyv, len);
                        if (c < NC) {
                            s_cn[4 * c + j] = nxv;
                            s_cn[4 * NC + 4 * c + j] = nyv;
                        }
                    } else {
                        nxv = s_cn[4 * c + j];
                        nyv = s_cn[4 * NC + 4 * c + j];
                    }
                    const T dux = ux2 - ux1, duy = uy2 - uy1;
                    const T x1 = X1 + ux1, y1 = Y1 + uy1;
                    const T x2 = X2 + ux2, y2 = Y2 + uy2;
                    const T lx = x2 - x1, ly = y2 - y1;
                    const T Lx = X2 - X1, Ly = Y2 - Y1;
                    H = (lx * lx + ly * ly) > (Lx * Lx + Ly * Ly);  // else G = 0 on all paths
                    const T spx = fmat(sg[2], nyv, sg[0] * nxv);
                    const T spy = fmat(sg[1], nyv, sg[2] * nxv);
                    if (H) Gj = T(0.5) * fmat(duy, spy, dux * spx);
                }
                if (__ballot(H && Gj > gc) == 0ull) continue;  // no path over Gc in this wavefront
                const T G1 = quad_lane<1>(Gj), G2 = quad_lane<2>(Gj);
                if (H && j == 0) {
                    const T Gv[3] = {Gj, G1, G2};
                    int jb = -1;
                    T gb = T(0);
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        if (Gv[q] > gc && (jb < 0 || Gv[q] > gb)) {
                            jb = q;
                            gb = Gv[q];
                        }
                    if (jb >= 0) {
                        bool ok = true;
#pragma unroll
                        for (int q = 0; q < 3; ++q)
                            if (q != jb && Gv[q] > gc && !(gb > gamma * (gb - Gv[q]))) ok = false;
                        if (ok)
                            best_merge(best, gb, gb, (j0 - 1 + t / TXE) * nx + (i0 - 1 + t % TXE), a, (a + 1 + jb) & 3);
                    }
                }
            }
            const uint64_t hm = __ballot(best.G >= T(0));
            if (hm != 0ull) best_wave(best, hm);
            // the last of the wavefronts with candidates publishes their best
            const int cw = min(NW, (ncand + 15) / 16);
            bool pub = true;
            if (cw > 1) {
                int arrived = 0;
                if (lane == 0) {
                    s_red[cwave] = best;
                    arrived = __hip_atomic_fetch_add(&s_nred, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                pub = __builtin_amdgcn_readfirstlane(arrived) == cw - 1;
                if (pub) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                    best = s_red[lane < cw ? lane : 0];
                    const uint64_t wm = __ballot(lane < cw && best.G >= T(0));
                    if (wm != 0ull) best_wave(best, wm);
                    if (lane == 0) s_nred = 0;
                }
            }
            if (pub && lane == 0) {
                uint64_t *const my = slots + ((ep + 1) & 1u) * slot_half + tile;
                if (best.G >= T(0))
                    xch::put_slot(my, nwg, ep + 1, best.e, best.a, best.k, (double)best.G, (double)best.Gmin);
                else
                    xch::put_no_slot(my, ep + 1);
            }
        }
        ncached = min(ncand, NC);

        // ---- element forces ---------------------------------------------------
        T fe[8];
        if (code == 0) {
            if constexpr (SC) {
                T bb[4][3], cb[4][3], sg[4][3];
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        sg[k][i] = s_e[i * NS + sidx[k]];
                        bb[k][i] = gx[k][i];
                        cb[k][i] = gy[k][i];
                    }
                subcell_force(bb, cb, at, sg, fe);
            } else {
                T sx[4], sy[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const T s0 = s_e[sidx[k]], s1 = s_e[NS + sidx[k]], s2 = s_e[2 * NS + sidx[k]];
#pragma unroll
                    for (int n = 0; n < 4; ++n) {
                        const T tx = fmat(gy[k][n], s2, gx[k][n] * s0);
                        const T ty = fmat(gx[k][n], s2, gy[k][n] * s1);
                        sx[n] = k == 0 ? tx : sx[n] + tx;
                        sy[n] = k == 0 ? ty : sy[n] + ty;
                    }
                }
#pragma unroll
                for (int n = 0; n < 4; ++n) {
                    fe[2 * n] = c4 * sx[n];
                    fe[2 * n + 1] = c4 * sy[n];
                }
            }
        }
        if (code == 0) {
#pragma unroll
            for (int c = 0; c < 8; ++c) s_fe[c * NR + tid] = fe[c];
        }
        // split elements: a constant-strain triangle per corner split, then a
        // bar per piece of a through split
        // (taken by other wavefronts than the candidates)
        int tp = R::HELP ? (tid + NT - C) % NT : NT - 1 - tid;
        asm volatile("" : "+v"(tp));
        for (int it = tp; it < nitems; it += NT) {
            const bool cst = it < bars0;
            if (cst && it >= ncorner) continue;
            const int t = cst ? s_splitl[it] : s_splitl[NR - 1 - ((it - bars0) >> 1)];
            const int sx_ = t % TXE + 1, sy_ = t / TXE + 1;
            const uint8_t scode = s_code[t];
            const int ea = (scode >> 2) & 3, eb = scode & 3;
            const int nb0 = sy_ * HX + sx_;
            const int F = cst ? ((((eb - ea) & 3) == 3) ? ea : eb) : (((it - bars0) & 1) ? eb : ea);
            const int n[4] = {F, (F + 1) & 3, (F + 2) & 3, (F + 3) & 3};
            T x[4], y[4], u[4], v[4], f[8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int oq_ = nb0 + corner(n[q]);
                x[q] = s_X[oq_];
                y[q] = s_Y[oq_];
                u[q] = s_ux[oq_];
                v[q] = s_uy[oq_];
            }
            if (cst) {
                corner_piece(mat, x, y, u, v, f);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    s_fe[(2 * n[q]) * NR + t] = f[2 * q];
                    s_fe[(2 * n[q] + 1) * NR + t] = f[2 * q + 1];
                }
            } else {
                bar_piece(mat, x, y, u, v, f);
#pragma unroll
                for (int q = 1; q < 3; ++q) {
                    s_fe[(2 * n[q]) * NR + t] = f[2 * q];
                    s_fe[(2 * n[q] + 1) * NR + t] = f[2 * q + 1];
                }
            }
        }
        __syncthreads();

        // ---- colour-ordered sums; update; border nodes out, halo in --------------
        const bool last = s + 1 == nsteps;
        uint64_t *const xb = xbuf + ((ep + 1) & 1u) * xb_half;
        asm volatile("" : "+v"(fl));
        int tn = tid;
        asm volatile("" : "+v"(tn));
        const int on_m = tn / TX, on_l = tn - on_m * TX, hidx = (on_m + 2) * HX + (on_l + 2);
        const bool polls = picks && (!last || tile == 0);
        if (fl & kOwn) {
            // forces of its elements, left (0) and right (1) of it in the rows
            // below and above, summed in colour order: colour (i mod 2) +
            // 2 (j mod 2) of element (i, j) puts the even row first and in a row
            // the even column (which matters in the second row only).  An absent
            // element's slot holds zero.
            constexpr int lo0 = 4 * NR, lo1 = 6 * NR + 1, hi0 = 2 * NR + TXE, hi1 = TXE + 1;
            const bool py = (fl & kOddY) != 0, px = (fl & kOddX) != 0;
            const T *const f = s_fe + on_m * TXE + on_l;
            const T *const fa = f + (py ? hi0 : lo0), *const fb = f + (py ? hi1 : lo1);
            const int l2 = py ? lo0 : hi0, r2 = py ? lo1 : hi1;
            const T *const fc = f + (px ? r2 : l2), *const fd = f + (px ? l2 : r2);
            T fx = fa[0] + fb[0], fy = fa[NR] + fb[NR];
            fx = (fx + fc[0]) + fd[0];
            fy = (fy + fc[NR]) + fd[NR];
            const int64_t kabs = base + s;
            const T phi = s_phi;
            T fex = T(0), fey = T(0);
            int si = 0;
            if (fl & (kEdge | kSend)) si = send_index(on_l, on_m, tw, th);
            if (fl & kEdge) {
                fex = s_bc[4 * si];
                fey = s_bc[4 * si + 1];
            }
            T ax = (phi * fex - fx) * n_minv;
            T ay = (phi * fey - fy) * n_minv;
            if (fl & kFix0) ax = T(0);
            if (fl & (2 * kFix0)) ay = T(0);
            const T dtv = (kabs == 0) ? T(0.5) * dts : dts;
            T vx = n_vx + dtv * ax;
            T vy = n_vy + dtv * ay;
            if (fl & (3 * kFix0)) {
                const Args qa = again();
                const double t = ((double)kabs + 0.5) * qa->p.dt, tr = qa->p.t_ramp;
                if (fl & kFix0) vx = prescribed(s_bc[4 * si + 2], t, tr);
                if (fl & (2 * kFix0)) vy = prescribed(s_bc[4 * si + 3], t, tr);
            }
            n_vx = vx;
            n_vy = vy;
            const T ux = s_ux[hidx], uy = s_uy[hidx];
            const T ux1 = ux + dts * vx, uy1 = uy + dts * vy;
            if (!last) {
                if (fl & kSend) xch::put_pair(xb + tile * (PW * R::cap) + si, R::cap, ep + 1, ux1, uy1);
                s_ux[hidx] = ux1;
                s_uy[hidx] = uy1;
            } else {
                // both buffers as k_step would leave them
                const Args qa = again();
                const bool odd = ((qa->par0 + s) & 1) != 0;
                const int on_n = (j0 + on_m) * (nx + 1) + (i0 + on_l);
                T *const cx = odd ? qa->p.ux1 : qa->p.ux0, *const cy = odd ? qa->p.uy1 : qa->p.uy0;
                T *const ox = odd ? qa->p.ux0 : qa->p.ux1, *const oy = odd ? qa->p.uy0 : qa->p.uy1;
                cx[on_n] = ux;
                cy[on_n] = uy;
                ox[on_n] = ux1;
                oy[on_n] = uy1;
                qa->p.vx[on_n] = vx;
                qa->p.vy[on_n] = vy;
            }
        }
        // A poll that comes too early costs a whole round trip, and with many
        // tiles polling the words themselves come later: the first poll waits
        // (400 x 400 plate on 240 tiles: 6.8 us per step without, 6.1 with 1 300
        // cycles, binary32 5.2 and 4.6; 135 tiles 5.4 and 5.2 with 500; none on
        // 9 tiles).
        for (int w = 0; w < nwg / 48; ++w) __builtin_amdgcn_s_sleep(4);
        if (polls) {
            xch::SlotWords sw;
            const int slot_id = NT - 1 - tn;
            const uint64_t *const slot_in = slots + ((ep + 1) & 1u) * slot_half + slot_id;
            if (slot_id < nwg) xch::load_slot(slot_in, nwg, sw);
            take_slots(slot_in, nwg, ep + 1, base + s, slot_id, sw);
        } else if (!last && (fl & kRecv)) {
            T x, y;
            if (!xch::get_pair(xb + (recv_at >> 11), R::cap, ep + 1, x, y)) {
                s_stop = 1;
            } else {
                s_ux[recv_at & 2047] = x;
                s_uy[recv_at & 2047] = y;
            }
        }
        __syncthreads();
        if (s_stop) {  // uniform: set before this barrier, next before the one of the next step
            stopped = true;
            break;
        }
    }

    // A workgroup did not answer.  The others may have stored their nodes (in the last
    // step only one waits for all), so the state in memory is of no use.
    if (stopped) {
        if (tid == 0) atomicOr(A.err, 1u);
        return;
    }
    if (tile != 0) return;
    // ---- tile 0: the last step's pick, split codes and U_d in log order ------
    {
        const int m = s_npicks;
        double *const s_ud = reinterpret_cast<double *>(smem);  // the tile's LDS is free now
        for (int q = tid; q < m; q += NT) {
            const int2 r = s_picks[q];
            p.split[r.x] = (uint8_t)r.y;
            const int64_t n0 = (int64_t)(r.x / nx) * (nx + 1) + r.x % nx;
            const int64_t nd[4] = {n0, n0 + 1, n0 + nx + 2, n0 + nx + 1};
            T x[4], y[4], cx, cy, len;
            for (int i = 0; i < 4; ++i) {
                x[i] = p.X[nd[i]];
                y[i] = p.Y[nd[i]];
            }
            path_geom(x, y, (r.y >> 2) & 3, r.y & 3, cx, cy, len);
            const T gc = p.gc ? p.gc[r.x] : p.gc_uniform;
            s_ud[q] = (double)(gc * len);
        }
        __syncthreads();
        if (tid == 0) {
            Control *ctl = p.ctl;
            double Ud = ctl->Ud;
            for (int q = 0; q < m; ++q) Ud = Ud + s_ud[q];
            ctl->Ud = Ud;
            ctl->nsplit = nsplit0 + m;
            if (nsplit0 + m > p.log_cap) ctl->overflow = 1;
            ctl->base = base + A.n;
        }
    }
}

template <class T, bool SC>
const void *resident_kernel(int c) {
    switch (c) {
        case 256: return reinterpret_cast<const void *>(k_resident<T, 256, SC>);
        case 512: return reinterpret_cast<const void *>(k_resident<T, 512, SC>);
        case 768: return reinterpret_cast<const void *>(k_resident<T, 768, SC>);
    }
    if constexpr (sizeof(T) == 4) return reinterpret_cast<const void *>(k_resident<T, 1024, SC>);
    return nullptr;
}

const void *resident_kernel(const ResidentPlan &r) {
    if (r.f32) return r.subcell ? resident_kernel<float, true>(r.tile) : resident_kernel<float, false>(r.tile);
    return r.subcell ? resident_kernel<double, true>(r.tile) : resident_kernel<double, false>(r.tile);
}

template <class T>
hipError_t launch(const ResidentPlan &r, const StepParamsT<T> &p, int n, int par0, uint32_t &epoch, hipStream_t st) {
    hipError_t e = xch::next_epochs(epoch, n, r.xb, r.words_u, r.slots, r.words_s, st);
    if (e != hipSuccess) return e;
    ResidentArgs<T> a;
    a.p = p;
    a.ntx = r.ntx;
    a.nwg = r.ntx * r.nty;
    a.n = n;
    a.par0 = par0;
    a.epoch0 = epoch;
    a.xb = r.xb;
    a.slots = r.slots;
    a.err = r.err;
    void *args[] = {&a};
    (void)hipGetLastError();
    e = hipLaunchCooperativeKernel(resident_kernel(r), dim3(a.nwg), dim3(r.threads), args, (unsigned)r.lds, st);
    if (e == hipSuccess) epoch += (uint32_t)n;
    return e;
}

}  // namespace

template <class T, int C>
bool tiles_fit(int nx, int ny, int most, ResidentPlan &r) {
    using R = Res<T, C>;
    const int64_t ntx = (nx + R::TXE - 1) / R::TX, nty = (ny + R::TYE - 1) / R::TY;
    if (ntx * nty > most) return false;
    r.tile = C;
    r.threads = R::NT;
    r.ntx = (int)ntx;
    r.nty = (int)nty;
    r.words_u = 2 * ntx * nty * R::cap * xch::pair_words<T>();
    r.words_s = 2 * ntx * nty * xch::kSlotWords;
    r.lds = R::total;
    return true;
}

// The smallest tiles of which there is at most one per compute unit: fewer
// wavefronts are fewer instructions per SIMD and step.  us per step, square grids
// at both ends of a class (per-step kernels in brackets): binary64 class 256 at
// 239 x 239 elements 4.0 (9.5), 512 at 240 and 335 5.0 (10.6) and 5.2 (12.0), 768
// at 336 and 415 6.4 (12.1) and 6.6 (13.0).  Tiles of 1 024 elements, four
// wavefronts per SIMD and 128 registers, spill 93 of them in binary64: 17.8 (13.1)
// at 416, 19.6 (16.7) at 495, so there they are for binary32 only, 4.7 (10.6)
// and 4.7 (11.8).
template <class T>
bool tiles_fit(int nx, int ny, int most, ResidentPlan &r) {
    if (tiles_fit<T, 256>(nx, ny, most, r) || tiles_fit<T, 512>(nx, ny, most, r) || tiles_fit<T, 768>(nx, ny, most, r))
        return true;
    if constexpr (sizeof(T) == 4) return tiles_fit<T, 1024>(nx, ny, most, r);
    return false;
}

bool whole_device(hipStream_t s, int device) {
    if (s == hipStreamLegacy || s == hipStreamPerThread) return true;  // (the query takes streams of their own only)
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return false;
    std::vector<uint32_t> mask((size_t)(cus + 31) / 32, 0u);
    if (hipExtStreamGetCUMask(s, (uint32_t)mask.size(), mask.data()) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    for (int i = 0; i < cus; ++i)
        if (!((mask[i / 32] >> (i % 32)) & 1u)) return false;
    return true;
}

bool resident_plan(int nx, int ny, bool f32, bool subcell, int device, ResidentPlan &r) {
    r = ResidentPlan{};
    r.f32 = f32;
    r.subcell = subcell;
    int cus = 0, coop = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return false;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, device) != hipSuccess || !coop) return false;
    const int most = std::min(cus, kResidentMaxTiles);
    if (!(f32 ? tiles_fit<float>(nx, ny, most, r) : tiles_fit<double>(nx, ny, most, r))) return false;
    const void *k = resident_kernel(r);
    if (r.lds > 65536 &&
        hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, r.lds) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, r.threads, r.lds) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return (int64_t)per_cu * cus >= (int64_t)r.ntx * r.nty;
}

hipError_t launch_resident(const ResidentPlan &r, const Launch &L, int n, int par0, uint32_t &epoch, hipStream_t st) {
    return L.f32 ? launch<float>(r, L.p0f, n, par0, epoch, st) : launch<double>(r, L.p0, n, par0, epoch, st);
}

}  // namespace mct
