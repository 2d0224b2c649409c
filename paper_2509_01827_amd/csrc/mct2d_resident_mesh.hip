// The resident step of an unstructured mesh (gfx950; triangles or
// quadrilaterals, binary64, global pick): many time steps in one cooperative
// launch, the whole state on the chip.
//
// The fused per-step kernel runs patches of some 90 nodes in several rounds of
// workgroups; every step each patch waits for a chain of dependent loads
// (tables, node values, the previous candidates) and recomputes its element
// geometry: 16 us on 320 000 triangles, 20 us on 160 000 quadrilaterals, 10 to
// 12 us on 54 000 triangles.  Here one workgroup per compute unit owns a patch
// of up to 768 nodes for the whole launch: u in LDS, v, 1/m, element gradients
// and smoothing weights in registers (768-thread patches of quadrilaterals spill
// 12 values per thread, 19 with more than eight elements at a node).  Patches are
// equal counts of nodes from a recursive bisection of the coordinates (any node
// numbering).  Border nodes and candidate slots travel as tagged words
// (mct2d_exchange.h).
//
// What bounds it: the slowest patch's chain of a step (barriers, latencies of LDS
// and dependent arithmetic with three wavefronts per SIMD) and the exchange.  Over
// the chip vector issue is busy 35 % of the time on 320 000 triangles and 30 % on
// 160 000 quadrilaterals (460 instructions per wavefront and step); wavefronts wait
// for 69 and 74 % of their cycles.  The strides of the LDS arrays spread a
// wavefront's accesses over the banks; conflicts take 8 to 10 % of the cycles.
// Per step, before -> after: 320 000 triangles 16.2 -> 6.7 us, 160 000
// quadrilaterals 21 -> 7.7, 54 000 triangles with cracks running 11 -> 6.0.
//
// A step, with three barriers (four on quadrilaterals):
//   - the pick of the step before acts on the codes; every element of the patch
//     and of its ring (triangles; on quadrilaterals the ring's shared edges)
//     stores its strains in LDS;
//   - each element smooths its edges with its neighbours' strains, forms its
//     stresses and forces (quadrilaterals: stored over the strains after a
//     barrier); those with a free-surface edge leave stresses and u for the
//     candidates; the last wavefronts form the split pieces;
//   - candidates (last wavefronts first), published; every node sums its forces
//     in colour order, advances and is sent where another patch needs it;
//   - halo (first wavefronts) and slots (last four) received.
// Arithmetic as the per-step kernels', operation for operation: the same bits.
#include <algorithm>
#include <climits>

#include "mct2d_device.h"
#include "mct2d_exchange.h"
#include "mct2d_resident.h"
#include "mct2d_tri.h"

namespace mct {
namespace tri {
namespace {

using namespace res;

constexpr uint32_t kNoAddr = 0xffff;

struct MeshArgs {
    Params p;
    ResidentMesh r;
    int32_t n, par0;
    uint32_t epoch0;
};

// plane-stress Hooke law, engineering shear strain
struct Mat {
    double D11, D12, D33, E;
};
__device__ __forceinline__ void hooke(const Mat &m, const double e[3], double s[3]) {
    s[0] = fma(m.D12, e[1], m.D11 * e[0]);
    s[1] = fma(m.D12, e[0], m.D11 * e[1]);
    s[2] = m.D33 * e[2];
}

__device__ __forceinline__ uint32_t u16_of(uint2 w, int k) {
    return ((k < 2 ? w.x : w.y) >> (16 * (k & 1))) & 0xffffu;
}

// Element gradients: triangles one set (constant), quadrilaterals at the four
// edge midpoints.
template <int NV>
struct Grad {
    double x[NV == 3 ? 1 : 4][NV], y[NV == 3 ? 1 : 4][NV];
};

__device__ __forceinline__ double grads(const double x[3], const double y[3], Grad<3> &g) {
    const double twoA = (x[1] - x[0]) * (y[2] - y[0]) - (x[2] - x[0]) * (y[1] - y[0]);
    const double inv = 1.0 / twoA;
    g.x[0][0] = (y[1] - y[2]) * inv;
    g.x[0][1] = (y[2] - y[0]) * inv;
    g.x[0][2] = (y[0] - y[1]) * inv;
    g.y[0][0] = (x[2] - x[1]) * inv;
    g.y[0][1] = (x[0] - x[2]) * inv;
    g.y[0][2] = (x[1] - x[0]) * inv;
    return 0.5 * twoA;
}
__device__ __forceinline__ double grads(const double x[4], const double y[4], Grad<4> &g) {
#pragma unroll
    for (int k = 0; k < 4; ++k) dev::q4_grad(x, y, k, g.x[k], g.y[k]);
    return 0.5 * ((x[2] - x[0]) * (y[3] - y[1]) - (x[3] - x[1]) * (y[2] - y[0]));
}

// The element rule over the NV - 1 path values G of a candidate; returns the
// chosen path or -1.
template <int NV>
__device__ __forceinline__ int element_rule(const double G[3], double gc, double gamma) {
    int jb = -1;
    double gb = 0.0;
#pragma unroll
    for (int q = 0; q < NV - 1; ++q)
        if (G[q] > gc && (jb < 0 || G[q] > gb)) {
            jb = q;
            gb = G[q];
        }
    if (jb < 0) return -1;
    bool ok = true;
#pragma unroll
    for (int q = 0; q < NV - 1; ++q)
        if (q != jb && G[q] > gc && !(gb > gamma * (gb - G[q]))) ok = false;
    return ok ? jb : -1;
}

// NT threads, up to EPT elements each (slots tid + NT r of the patch's list), up
// to 2 GW elements at a node.
template <int NV, int NT, int EPT, int GW>
__global__ __launch_bounds__(NT) void k_mesh_resident(const MeshArgs A) {
    constexpr int NW = NT / 64, NQ = NV == 3 ? 1 : 4;  // strains per element
    constexpr int PW = xch::pair_words<double>();
    constexpr bool OVER = NV == 4;                // forces stored over the strains
    constexpr int LPC = NV == 3 ? 2 : 4, CPW = 64 / LPC;  // lanes per candidate, candidates per wavefront
    constexpr int NCE = mesh_cands(NT), NC = NCE;  // elements with candidates, candidates that keep their normals
    // strides per element that keep bank groups apart: strains in values of 8
    // bytes, forces of 16 (both then at fixed offsets from one address)
    constexpr int QS = NV == 3 ? kTriStrain : kQuadStrain, FS = NV == 3 ? kTriForce : kQuadForce, RS = kRingGrad;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const Params &p = A.p;
    const ResidentMesh &R = A.r;
    const int NE = R.ne_max, NP = R.np_max;
    double2 *const s_u = reinterpret_cast<double2 *>(smem + R.o_u);
    double2 *const s_x = reinterpret_cast<double2 *>(smem + R.o_x);
    double *const s_q = reinterpret_cast<double *>(smem + R.o_q);  // strains: 3 k + c at QS slot
    double2 *const s_f = reinterpret_cast<double2 *>(smem + R.o_f);  // forces: node n at FS slot + n; last: zero
    uint4 *const s_rt = reinterpret_cast<uint4 *>(smem + R.o_rt);    // the ring's edges: nodes, strain's place, id
    double *const s_rg = reinterpret_cast<double *>(smem + R.o_rg);  // quadrilaterals: gradients of the ring's edges
    double *const s_cd = reinterpret_cast<double *>(smem + R.o_cd);  // stresses and u of elements with candidates
    double *const s_cn = reinterpret_cast<double *>(smem + R.o_cn);  // path normals of the first NC candidates
    int2 *const s_ci = reinterpret_cast<int2 *>(smem + R.o_ci);  // and their places
    double *const s_bc = reinterpret_cast<double *>(smem + R.o_bc);  // loads and prescribed velocities of flagged nodes
    uint16_t *const s_cand = reinterpret_cast<uint16_t *>(smem + R.o_cand);  // element entry | edge << 12
    uint16_t *const s_cslot = reinterpret_cast<uint16_t *>(smem + R.o_cslot);  // slot of an element entry
    double *const s_cgc = reinterpret_cast<double *>(smem + R.o_cgc);  // its Gc
    uint16_t *const s_splitl = reinterpret_cast<uint16_t *>(smem + R.o_split);  // split elements
    uint8_t *const s_code = reinterpret_cast<uint8_t *>(smem + R.o_code);  // by slot, then the ring's edges
    using Args = const __attribute__((address_space(4))) MeshArgs *;
    const Args args = (Args)__builtin_amdgcn_kernarg_segment_ptr();
    // the arguments through a pointer the compiler does not see through: what is
    // read from it in the loop stays out of registers held across the loop
    auto again = [&]() {
        Args q = args;
        asm volatile("" : "+s"(q));
        return q;
    };
    __shared__ int s_ncand, s_ncel, s_ncorner, s_nthru, s_nred, s_ninl, s_stop, s_narr, s_npicks, s_pick, s_pcode, s_hit, s_full, s_nbc;
    __shared__ Best<double> s_red[NW], s_inl[NW * EPT], s_pk[kPickWaves];
    __shared__ double s_phi, s_cv[4];
    __shared__ int2 s_picks[kMeshResidentSteps];

    int tid = threadIdx.x, lane = tid & 63;
    const int b = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const MeshPatch P = R.patch[b];
    const int64_t base = p.ctl->base, nsplit0 = p.ctl->nsplit;
    const int nwg = R.npatch, pickers = (nwg + 63) / 64;

    // ---- the state, once per launch ---------------------------------------
    {
        const double2 *u = A.par0 ? p.u1 : p.u0;
        for (int l = tid; l < P.nown + P.nhalo; l += NT) {
            const int g = R.node_id[P.node0 + l];
            s_u[l] = u[g];
            s_x[l] = p.xy[g];
        }
        if (tid == 0) {
            s_ncand = s_ncel = s_ncorner = s_nthru = s_nred = s_ninl = s_stop = s_narr = s_npicks = s_nbc = 0;
            s_pick = -1;
            s_hit = -1;
            s_phi = 1.0;
            s_cv[0] = 1.0;
            s_cv[1] = -1.0;  // no interval yet
        }
    }
    __syncthreads();

    struct Elem {
        uint32_t eid;    // id (all ones: none)
        uint2 lc, nb;    // nodes, LDS place of the neighbour's strain across each edge (16 bits each)
        unsigned fl;     // bit k: neighbour across k split or absent; 4 + k: this element is the lower-id one
        int ci;          // entry among the elements with candidates, -1 none, -2 they are full
        uint8_t code;
        Grad<NV> g;
        double c, w0[NV], w1[NV];  // force factor; smoothing weights (lower id, higher id)
    };
    constexpr unsigned kOwnedEl = 256;  // its candidates are evaluated here
    Elem el[EPT];
    auto nodes_of = [&](uint2 lc, const double2 *src, double x[NV], double y[NV]) {
#pragma unroll
        for (int n = 0; n < NV; ++n) {
            const double2 v = src[u16_of(lc, n)];
            x[n] = v.x;
            y[n] = v.y;
        }
    };
#pragma unroll
    for (int r = 0; r < EPT; ++r) {
        Elem &E = el[r];
        const int s = tid + NT * r;
        E.eid = 0xffffffffu;
        E.fl = 0;
        E.ci = -1;
        E.code = kAbsent;
        E.lc = E.nb = make_uint2(0, 0);
        if (s < P.nel + P.nring) {
            const int64_t t = P.slot0 + s;
            const uint32_t id = R.slot_eid[t];
            E.eid = id & (uint32_t)(kOwned - 1);
            E.lc = R.slot_lc[t];
            E.code = p.split[E.eid];
            s_code[s] = E.code;
            double x[NV], y[NV];
            nodes_of(E.lc, s_x, x, y);
            const double area = grads(x, y, E.g);
            if (s < P.nel) {
                E.nb = R.slot_nb[t];
                E.c = NV == 3 ? area / 3.0 : 0.25 * area;
                const int4 far = R.slot_far[t];  // the neighbours' ids
                if (id & kOwned) E.fl |= kOwnedEl;
#pragma unroll
                for (int k = 0; k < NV; ++k) {
                    const int nb = k == 0 ? far.x : k == 1 ? far.y : k == 2 ? far.z : far.w;
                    E.w0[k] = E.w1[k] = 0.0;
                    if (nb < 0) {
                        E.fl |= 1u << k;
                        continue;
                    }
                    if (p.split[nb] != 0) E.fl |= 1u << k;
                    const bool lo = (int)E.eid < nb;
                    if (lo) E.fl |= 16u << k;
                    const int4 cn = p.conn[nb];
                    const double2 a0 = p.xy[cn.x], a1 = p.xy[cn.y], a2 = p.xy[cn.z];
                    double An;
                    if constexpr (NV == 3) {
                        An = 0.5 * ((a1.x - a0.x) * (a2.y - a0.y) - (a2.x - a0.x) * (a1.y - a0.y));
                    } else {
                        const double2 a3 = p.xy[cn.w];
                        An = 0.5 * ((a2.x - a0.x) * (a3.y - a1.y) - (a3.x - a1.x) * (a2.y - a0.y));
                    }
                    const double Alo = lo ? area : An, Ahi = lo ? An : area;
                    const double sum = Alo + Ahi;
                    E.w0[k] = Alo / sum;
                    E.w1[k] = Ahi / sum;
                }
            }
        }
    }
    // quadrilaterals: the ring's edges shared with patch elements
    int ro = NT - 1 - tid;
    if constexpr (NV == 4) {
        if (ro < P.nredge) {
            const int64_t t = P.redge0 + ro;
            const uint32_t id = R.redge_eid[t];
            const uint2 rlc = R.redge_lc[t];
            const int k = R.redge_at[t] >> 16;
            s_rt[ro] = make_uint4(rlc.x, rlc.y, R.redge_at[t] & 0xffff, id);
            s_code[NE + ro] = p.split[id];
            double x[NV], y[NV], gx[4], gy[4];
            nodes_of(rlc, s_x, x, y);
            double xx[4] = {x[0], x[1], x[2], x[NV - 1]}, yy[4] = {y[0], y[1], y[2], y[NV - 1]};
            dev::q4_grad_rt(xx, yy, k, gx, gy);
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                s_rg[RS * ro + n] = gx[n];
                s_rg[RS * ro + 4 + n] = gy[n];
            }
        }
    }

    // this thread's node
    enum : unsigned { kOwn = 1, kSend = 2, kBc = 4, kFix0 = 8 };
    constexpr int kBcAt = 8;  // bits from here: its entry of s_bc (kMeshBc: none left, read from memory)
    unsigned nfl = 0;
    double n_minv = 0.0;
    double2 n_v = make_double2(0.0, 0.0);
    int send_at = 0;
    uint32_t gat[GW];
#pragma unroll
    for (int d = 0; d < GW; ++d) gat[d] = 0;
    if (tid < P.nown) {
        const int g = R.node_id[P.node0 + tid];
        nfl = kOwn;
        n_minv = p.minv[g];
        n_v = p.v[g];
        send_at = R.node_send[P.own0 + tid];
        if (send_at >= 0) nfl |= kSend;
        const uint8_t f = p.nflag[g];
        if (f) {
            nfl |= kBc | ((f & kFixX) ? kFix0 : 0u) | ((f & kFixY) ? 2 * kFix0 : 0u);
            const double2 fe = (f & kLoaded) ? p.fext[g] : make_double2(0.0, 0.0);
            const double2 v0 = (f & (kFixX | kFixY)) ? p.v0[g] : make_double2(0.0, 0.0);
            const int i = atomicAdd(&s_nbc, 1);
            if (i < kMeshBc) {
                s_bc[4 * i] = fe.x;
                s_bc[4 * i + 1] = fe.y;
                s_bc[4 * i + 2] = v0.x;
                s_bc[4 * i + 3] = v0.y;
            }
            nfl |= (unsigned)min(i, kMeshBc) << kBcAt;
        }
        const uint32_t *gt = reinterpret_cast<const uint32_t *>(R.node_gather + 16 * (int64_t)(P.own0 + tid));
#pragma unroll
        for (int d = 0; d < GW; ++d) gat[d] = gt[d];
    }
    const int wmax = R.wmax;
    const int xb_half = nwg * PW * R.cap, slot_half = nwg * xch::kSlotWords;
    const double gamma = p.gamma, dt = p.dt;
    const bool curve = p.ncurve > 0;
    int curve_i = 0, ncached = 0;
    bool stopped = false;

    // The lists only grow within a launch (an entry of an element that split is
    // skipped): elements with candidates, their free-surface edges, split
    // elements (quadrilaterals: corner splits from the front, through splits
    // from the back; triangles all from the front).
    auto list_cands = [&](Elem &E, int slot, unsigned bits) {
        if (!(E.fl & kOwnedEl) || !bits) return;
        if (E.ci == -1) {
            const int c = atomicAdd(&s_ncel, 1);
            if (c < NCE) {
                E.ci = c;
                s_cslot[c] = (uint16_t)slot;
                s_cgc[c] = p.gc[E.eid];
            } else {
                E.ci = -2;
            }
        }
        if (E.ci < 0) return;
        for (int k = 0; k < NV; ++k)
            if ((bits >> k) & 1u) s_cand[atomicAdd(&s_ncand, 1)] = (uint16_t)(E.ci | k << 12);
    };
    auto list_split = [&](const Elem &E, int slot) {
        if (slot >= P.nel) return;
        if (NV == 4 && ((((E.code & 3) - ((E.code >> 2) & 3)) & 3) == 2))
            s_splitl[NP - 1 - atomicAdd(&s_nthru, 1)] = (uint16_t)slot;
        else
            s_splitl[atomicAdd(&s_ncorner, 1)] = (uint16_t)slot;
    };
#pragma unroll
    for (int r = 0; r < EPT; ++r) {
        const int s = tid + NT * r;
        if (el[r].code & kSplitFlag) list_split(el[r], s);
        if (el[r].code == 0 && s < P.nel) list_cands(el[r], s, el[r].fl & ((1u << NV) - 1u));
    }

    // Path j (exit edge a + 1 + j) of a tip edge a of the element with nodes lc:
    // unit normal oriented toward the second end of a, and length.
    auto path_of = [&](uint2 lc, int a, int j, double &nx, double &ny, double &len) {
        const int k = (a + 1 + j) % NV;
        const double2 A0 = s_x[u16_of(lc, a)], A1 = s_x[u16_of(lc, (a + 1) % NV)];
        const double2 K0 = s_x[u16_of(lc, k)], K1 = s_x[u16_of(lc, (k + 1) % NV)];
        dev::path_geom_pts(A0.x, A0.y, A1.x, A1.y, K0.x, K0.y, K1.x, K1.y, nx, ny, len);
    };
    // the stretch gate of edge (X1, X2) displaced by (u1, u2)
    auto gate = [](double2 X1, double2 X2, double2 u1, double2 u2) {
        const double x1 = X1.x + u1.x, y1 = X1.y + u1.y;
        const double x2 = X2.x + u2.x, y2 = X2.y + u2.y;
        const double lx = x2 - x1, ly = y2 - y1;
        const double Lx = X2.x - X1.x, Ly = X2.y - X1.y;
        return (lx * lx + ly * ly) > (Lx * Lx + Ly * Ly);
    };

    // Takes the slots of epoch ep; the last of the wavefronts that do leaves the
    // pick in s_pick and s_pcode, and in patch 0 records it.
    const bool picks = NW - 1 - wave < pickers;
    auto take_slots = [&](uint32_t ep, int64_t step, int slot_id) {
        const uint64_t *const at = R.slots + (ep & 1u) * slot_half + slot_id;
        Best<double> g;
        best_none(g);
        bool has = false;
        if (slot_id < nwg) {
            xch::SlotWords sw;
            xch::load_slot(at, nwg, sw);
            int e = 0, a = 0, k = 0;
            double G = 0.0, Gm = 0.0;
            if (!xch::take_slot(at, nwg, ep, sw, has, e, a, k, G, Gm)) s_stop = 1;
            if (has) {
                g.G = G;
                g.Gmin = Gm;
                g.e = e;
                g.a = a;
                g.k = k;
            }
        }
        const uint64_t hm = __ballot(has);
        if (hm != 0ull) best_wave(g, hm);
        if (pickers > 1) {
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
        int pe = -1;
        if (g.G >= 0.0 && g.G > gamma * (g.G - g.Gmin)) {
            const int pc = kSplitFlag | (g.a << 2) | g.k;
            pe = g.e;
            s_pcode = pc;
            if (b == 0) {
                const int i = s_npicks;
                const Args q = again();
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
                    r.G = g.G;
                    q->p.log[nsplit0 + i] = r;
                }
            }
        }
        s_pick = pe;
    };

    if (tid == 0) s_f[FS * NP] = make_double2(0.0, 0.0);  // (never stored over)
    // every load of the set-up done: a wait for one of them in the loop would
    // also wait for the stores under way there
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)"
                 : "+v"(n_minv), "+v"(n_v.x), "+v"(n_v.y), "+v"(send_at), "+v"(nfl)
                 :
                 : "memory");
#pragma unroll
    for (int d = 0; d < GW; ++d) asm volatile("" : "+v"(gat[d]));
#pragma unroll
    for (int r = 0; r < EPT; ++r)
        asm volatile("" : "+v"(el[r].eid), "+v"(el[r].lc.x), "+v"(el[r].lc.y), "+v"(el[r].nb.x), "+v"(el[r].nb.y), "+v"(el[r].fl));
    const int nsteps = A.n;
    for (int s = 0; s < nsteps; ++s) {
        const uint32_t ep = A.epoch0 + (uint32_t)s;  // of u^k
        // (values the compiler must not unpack into registers of their own ahead
        // of the loop)
        asm volatile("" : "+v"(tid), "+v"(nfl), "+v"(send_at));
        lane = tid & 63;
        ro = NT - 1 - tid;
#pragma unroll
        for (int d = 0; d < GW; ++d) asm volatile("" : "+v"(gat[d]));
#pragma unroll
        for (int r = 0; r < EPT; ++r)
            asm volatile(""
                         : "+v"(el[r].lc.x), "+v"(el[r].lc.y), "+v"(el[r].nb.x), "+v"(el[r].nb.y), "+v"(el[r].fl),
                           "+v"(el[r].ci));
        Mat mat;
        {
            const Args q = again();
            mat.D11 = q->p.D11;
            mat.D12 = q->p.D12;
            mat.D33 = q->p.D33;
            mat.E = q->p.E;
        }
        // ---- the pick of the step before ----------------------------------------
        // (whether the candidates' lists are full is decided here, where nothing is
        // added to them: behind the barrier some wavefronts list while others have
        // still to look)
        if (const int pick = s_pick; pick >= 0) {  // uniform
            const uint8_t pc = (uint8_t)s_pcode;
#pragma unroll
            for (int r = 0; r < EPT; ++r)
                if ((int)el[r].eid == pick) {
                    const int slot = tid + NT * r;
                    el[r].code = pc;
                    s_code[slot] = pc;
                    list_split(el[r], slot);
                    s_hit = s;
                    s_full = s_ncel > NCE;
                }
            if (NV == 4 && ro < P.nredge && (int)s_rt[ro].w == pick) {
                s_code[NE + ro] = pc;
                s_hit = s;
                s_full = s_ncel > NCE;
            }
        }
        // ---- strains ------------------------------------------------------------
#pragma unroll
        for (int r = 0; r < EPT; ++r) {
            if (wave * 64 + NT * r >= P.nel + P.nring) continue;  // uniform over the wavefront
            if (el[r].code != 0) continue;
            double ux[NV], uy[NV];
            nodes_of(el[r].lc, s_u, ux, uy);
#pragma unroll
            for (int k = 0; k < NQ; ++k) {
                double q[3];
                dev::strain<NV>(el[r].g.x[k], el[r].g.y[k], ux, uy, q);
#pragma unroll
                for (int c = 0; c < 3; ++c) s_q[QS * (tid + NT * r) + 3 * k + c] = q[c];
            }
        }
        if (NV == 4 && ro < P.nredge && s_code[NE + ro] == 0) {
            const uint4 rt = s_rt[ro];  // nodes, LDS place of its strain
            const uint2 rlc = make_uint2(rt.x, rt.y);
            double ux[NV], uy[NV], gx[NV], gy[NV], rq[3];
            nodes_of(rlc, s_u, ux, uy);
#pragma unroll
            for (int n = 0; n < NV; ++n) {
                gx[n] = s_rg[RS * ro + n];
                gy[n] = s_rg[RS * ro + NV + n];
            }
            dev::strain<NV>(gx, gy, ux, uy, rq);
#pragma unroll
            for (int c = 0; c < 3; ++c) s_q[rt.z + c] = rq[c];
        }
        if (curve && tid == NT - 1) {
            // load factor at t_k; s_cv: the curve's interval and values at hand
            const Args a = again();
            const double t = (double)(base + s) * a->p.dt;
            const double *const ct = a->p.curve_t, *const cp = a->p.curve_phi;
            if (!(t >= s_cv[0] && t < s_cv[1])) {
                const int nc = a->p.ncurve;
                if (t <= ct[0] || t >= ct[nc - 1]) {
                    s_cv[0] = 1.0;
                    s_cv[1] = -1.0;
                    s_cv[2] = t <= ct[0] ? cp[0] : cp[nc - 1];
                } else {
                    while (ct[curve_i + 1] <= t) ++curve_i;
                    s_cv[0] = ct[curve_i];
                    s_cv[1] = ct[curve_i + 1];
                    s_cv[2] = cp[curve_i];
                    s_cv[3] = (cp[curve_i + 1] - cp[curve_i]) / (ct[curve_i + 1] - ct[curve_i]);
                }
            }
            // (t = ct[0] exactly: phi[0] + 0 * slope is phi[0])
            s_phi = s_cv[1] < s_cv[0] ? s_cv[2] : s_cv[2] + (t - s_cv[0]) * s_cv[3];
        }
        __syncthreads();
        if (s_hit == s) {  // uniform: an element of the patch or its ring split
            const bool full = s_full != 0;  // start the lists again, without the entries of split elements
            if (full) {
                if (tid == 0) s_ncel = s_ncand = 0;
                ncached = 0;
                __syncthreads();
            }
#pragma unroll
            for (int r = 0; r < EPT; ++r) {
                const int slot = tid + NT * r;
                if (slot >= P.nel || el[r].code != 0) continue;
                const uint2 cc = R.slot_code[P.slot0 + slot];
                unsigned nw = 0;
#pragma unroll
                for (int k = 0; k < NV; ++k) {
                    const uint32_t at = u16_of(cc, k);
                    if (at != kNoAddr && s_code[at] != 0) nw |= 1u << k;
                }
                if (full)
                    el[r].ci = -1;
                else
                    nw &= ~el[r].fl;
                el[r].fl |= nw;
                if (full) nw = el[r].fl & ((1u << NV) - 1u);
                list_cands(el[r], slot, nw);
            }
        }
        // ---- smoothed stresses, forces ----------------------------------------------
        double2 fe[EPT][NV];
#pragma unroll
        for (int r = 0; r < EPT; ++r) {
            if (wave * 64 + NT * r >= P.nel) continue;  // uniform over the wavefront
            const int slot = tid + NT * r;
            Elem &E = el[r];
            const bool on = slot < P.nel && E.code == 0;
            // smoothed stress of edge k
            auto stress = [&](int k, double w0, double w1, double sig[3]) {
                const double *const own = s_q + QS * slot + (NV == 3 ? 0 : 3 * k), *const nbr = s_q + u16_of(E.nb, k);
                const bool alone = ((E.fl >> k) & 1u) != 0, lo = ((E.fl >> (4 + k)) & 1u) != 0;
                double eps[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const double a = own[c], o = nbr[c];
                    const double both = fma(w1, lo ? o : a, w0 * (lo ? a : o));
                    eps[c] = alone ? a : both;
                }
                hooke(mat, eps, sig);
            };
            if (on) {
                double sx[NV], sy[NV], S[3];
#pragma unroll
                for (int k = 0; k < NV; ++k) {
                    double sig[3];
                    stress(k, E.w0[k], E.w1[k], sig);
                    if (E.ci >= 0) {
#pragma unroll
                        for (int c = 0; c < 3; ++c) s_cd[(3 * k + c) * NCE + E.ci] = sig[c];
                    }
                    if constexpr (NV == 3) {
#pragma unroll
                        for (int c = 0; c < 3; ++c) S[c] = k == 0 ? sig[c] : S[c] + sig[c];
                    } else {
#pragma unroll
                        for (int n = 0; n < NV; ++n) {
                            const double gx = E.g.x[NV == 3 ? 0 : k][n], gy = E.g.y[NV == 3 ? 0 : k][n];
                            const double tx = fma(gy, sig[2], gx * sig[0]);
                            const double ty = fma(gx, sig[2], gy * sig[1]);
                            sx[n] = k == 0 ? tx : sx[n] + tx;
                            sy[n] = k == 0 ? ty : sy[n] + ty;
                        }
                    }
                }
#pragma unroll
                for (int n = 0; n < NV; ++n) {
                    if constexpr (NV == 3)
                        fe[r][n] = make_double2(E.c * fma(E.g.y[0][n], S[2], E.g.x[0][n] * S[0]),
                                                E.c * fma(E.g.x[0][n], S[2], E.g.y[0][n] * S[1]));
                    else
                        fe[r][n] = make_double2(E.c * sx[n], E.c * sy[n]);
                    if (!OVER) s_f[FS * slot + n] = fe[r][n];
                }
                if (E.ci >= 0) {
#pragma unroll
                    for (int n = 0; n < NV; ++n) {
                        const double2 U = s_u[u16_of(E.lc, n)];
                        s_cd[(3 * NV + 2 * n) * NCE + E.ci] = U.x;
                        s_cd[(3 * NV + 2 * n + 1) * NCE + E.ci] = U.y;
                    }
                }
            }
            if (__ballot(on && E.ci == -2) != 0ull) {
                // candidates of elements that found the lists full
                Best<double> inl;
                best_none(inl);
                if (on && E.ci == -2) {
                    const double gc = p.gc[E.eid];
#pragma unroll 1
                    for (int a = 0; a < NV; ++a) {
                        if (!((E.fl >> a) & 1u)) continue;
                        const int i1 = u16_of(E.lc, a), i2 = u16_of(E.lc, (a + 1) % NV);
                        const double2 u1 = s_u[i1], u2 = s_u[i2];
                        if (!gate(s_x[i1], s_x[i2], u1, u2)) continue;
                        double G[3] = {0.0, 0.0, 0.0};
#pragma unroll 1
                        for (int j = 0; j < NV - 1; ++j) {
                            const int k = (a + 1 + j) % NV;
                            double nx, ny, len, sg[3], w0 = E.w0[0], w1 = E.w1[0];
#pragma unroll
                            for (int m = 1; m < NV; ++m)
                                if (m == k) {
                                    w0 = E.w0[m];
                                    w1 = E.w1[m];
                                }
                            path_of(E.lc, a, j, nx, ny, len);
                            stress(k, w0, w1, sg);
                            const double spx = fma(sg[2], ny, sg[0] * nx);
                            const double spy = fma(sg[1], ny, sg[2] * nx);
                            const double Gj = 0.5 * fma(u2.y - u1.y, spy, (u2.x - u1.x) * spx);
                            if (j == 0)
                                G[0] = Gj;
                            else if (j == 1)
                                G[1] = Gj;
                            else
                                G[2] = Gj;
                        }
                        const int jb = element_rule<NV>(G, gc, gamma);
                        if (jb >= 0) {
                            const double gb = jb == 0 ? G[0] : jb == 1 ? G[1] : G[2];
                            best_merge(inl, gb, gb, (int)E.eid, a, (a + 1 + jb) % NV);
                        }
                    }
                }
                const uint64_t im = __ballot(inl.G >= 0.0);
                if (im != 0ull) {
                    best_wave(inl, im);
                    if (lane == 0) s_inl[atomicAdd(&s_ninl, 1)] = inl;
                }
            }
        }
        if constexpr (OVER) {
            __syncthreads();  // every neighbour's strain read
#pragma unroll
            for (int r = 0; r < EPT; ++r)
                if (tid + NT * r < P.nel && el[r].code == 0) {
#pragma unroll
                    for (int n = 0; n < NV; ++n) s_f[FS * (tid + NT * r) + n] = fe[r][n];
                }
        }
        // split elements, from the last wavefront down: triangles a bar and a free
        // node; quadrilaterals a triangle per corner split, then two bars per
        // through split (the bars start a wavefront of their own)
        const int ncorner = s_ncorner;
        const int bars0 = NV == 3 ? 0 : (ncorner + 63) & ~63;
        const int nitems = NV == 3 ? ncorner : bars0 + 2 * s_nthru;
        for (int it = NT - 1 - tid; it < nitems; it += NT) {
            const bool cst = it < bars0;
            if (cst && it >= ncorner) continue;
            const int slot = NV == 3 || cst ? s_splitl[it] : s_splitl[NP - 1 - ((it - bars0) >> 1)];
            const int code = s_code[slot], ea = (code >> 2) & 3, eb = code & 3;
            const uint2 lc = R.slot_lc[P.slot0 + slot];
            if constexpr (NV == 3) {
                // the two-node piece runs from edge F to the edge two on
                const int F = ((eb - ea + 3) % 3) == 2 ? ea : eb, n0 = F, n1 = (F + 1) % 3, n2 = (F + 2) % 3;
                const double2 x0 = s_x[u16_of(lc, n0)], x1 = s_x[u16_of(lc, n1)], x2 = s_x[u16_of(lc, n2)];
                const double2 u1 = s_u[u16_of(lc, n1)], u2 = s_u[u16_of(lc, n2)];
                const double px0 = 0.5 * (x0.x + x1.x), py0 = 0.5 * (x0.y + x1.y);
                const double px3 = 0.5 * (x2.x + x0.x), py3 = 0.5 * (x2.y + x0.y);
                double sa = 0.0;
                sa += (x1.x - px0) * (x2.y - py0) - (x2.x - px0) * (x1.y - py0);
                sa += (x2.x - px0) * (py3 - py0) - (px3 - px0) * (x2.y - py0);
                const double Ap = 0.5 * sa;
                const double dx = x2.x - x1.x, dy = x2.y - x1.y;
                const double L2 = dx * dx + dy * dy;
                const double dux = u2.x - u1.x, duy = u2.y - u1.y;
                const double str = (dx * dux + dy * duy) / L2;
                const double stress = mat.E * str;
                const double coef = Ap * stress / L2;
                s_f[FS * slot + n2] = make_double2(coef * dx, coef * dy);
                s_f[FS * slot + n1] = make_double2(-(coef * dx), -(coef * dy));
                s_f[FS * slot + n0] = make_double2(0.0, 0.0);
            } else {
                const int F = cst ? ((((eb - ea) & 3) == 3) ? ea : eb) : (((it - bars0) & 1) ? eb : ea);
                const int nn[4] = {F, (F + 1) & 3, (F + 2) & 3, (F + 3) & 3};
                double x[4], y[4], u[4], v[4], f[8];
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const double2 X = s_x[u16_of(lc, nn[m])], U = s_u[u16_of(lc, nn[m])];
                    x[m] = X.x;
                    y[m] = X.y;
                    u[m] = U.x;
                    v[m] = U.y;
                }
                StepParams sp;
                sp.D11 = mat.D11;
                sp.D12 = mat.D12;
                sp.D33 = mat.D33;
                sp.E = mat.E;
                if (cst)
                    dev::corner_piece(sp, x, y, u, v, f);
                else
                    dev::bar_piece(sp, x, y, u, v, f);
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    if (cst || m == 1 || m == 2) s_f[FS * slot + nn[m]] = make_double2(f[2 * m], f[2 * m + 1]);
            }
        }
        __syncthreads();

        // ---- energy release rate and element rule of the candidates --------------
        const bool last = s + 1 == nsteps;
        uint64_t *const my_slot = R.slots + ((ep + 1) & 1u) * slot_half + b;
        const int ncand = s_ncand, cwave = NW - 1 - wave;
        if (ncand == 0 && tid == 0) xch::put_no_slot(my_slot, ep + 1);
        if (cwave * CPW < ncand) {  // uniform over the wavefront
            Best<double> best;
            best_none(best);
            int tq = cwave * 64 + lane;
            asm volatile("" : "+v"(tq));
            for (int c0 = 0; c0 + cwave * CPW < ncand; c0 += NT / LPC) {
                const int c = c0 + tq / LPC, j = tq & (LPC - 1);
                double Gj = 0.0, gc = 0.0;
                bool H = false;
                const bool fresh = c >= ncached;
                int2 ci = make_int2(0, 0);
                double nxv = 0.0, nyv = 0.0;
                if (c < ncand) {
                    if (fresh) {
                        const int ent = s_cand[c], a = ent >> 12, i = ent & 0xfff;
                        const uint2 lc = R.slot_lc[P.slot0 + s_cslot[i]];
                        ci.x = (int)(u16_of(lc, a) | u16_of(lc, (a + 1) % NV) << 16);
                        ci.y = i | a << 12 | (int)s_cslot[i] << 16;
                        if (j < NV - 1) {
                            double len;
                            path_of(lc, a, j, nxv, nyv, len);
                        }
                        if (c < NC) {
                            s_ci[LPC * c + j] = ci;
                            s_cn[LPC * c + j] = nxv;
                            s_cn[LPC * NC + LPC * c + j] = nyv;
                        }
                    } else {
                        ci = s_ci[LPC * c + j];
                        nxv = s_cn[LPC * c + j];
                        nyv = s_cn[LPC * NC + LPC * c + j];
                    }
                }
                const int i = ci.y & 0xfff, a = (ci.y >> 12) & 3, slot = ci.y >> 16;
                if (c < ncand && s_code[slot] == 0) {
                    const int a1 = (a + 1) % NV, k = (a + 1 + j) % NV;
                    const double2 X1 = s_x[ci.x & 0xffff], X2 = s_x[(uint32_t)ci.x >> 16];
                    const double2 u1 = make_double2(s_cd[(3 * NV + 2 * a) * NCE + i], s_cd[(3 * NV + 2 * a + 1) * NCE + i]);
                    const double2 u2 = make_double2(s_cd[(3 * NV + 2 * a1) * NCE + i], s_cd[(3 * NV + 2 * a1 + 1) * NCE + i]);
                    const double s0 = s_cd[(3 * k) * NCE + i], s1 = s_cd[(3 * k + 1) * NCE + i], s2 = s_cd[(3 * k + 2) * NCE + i];
                    gc = s_cgc[i];
                    H = gate(X1, X2, u1, u2);
                    const double spx = fma(s2, nyv, s0 * nxv);
                    const double spy = fma(s1, nyv, s2 * nxv);
                    if (H && j < NV - 1) Gj = 0.5 * fma(u2.y - u1.y, spy, (u2.x - u1.x) * spx);
                }
                if (__ballot(H && Gj > gc) == 0ull) continue;  // no path over Gc in this wavefront
                double G[3] = {Gj, 0.0, 0.0};
                if constexpr (LPC == 2) {
                    G[1] = pair_lane(Gj);
                } else {
                    G[1] = quad_lane<1>(Gj);
                    G[2] = quad_lane<2>(Gj);
                }
                if (H && j == 0) {
                    const int jb = element_rule<NV>(G, gc, gamma);
                    if (jb >= 0) {
                        const double gb = jb == 0 ? G[0] : jb == 1 ? G[1] : G[2];
                        const int e = (int)(R.slot_eid[P.slot0 + slot] & (uint32_t)(kOwned - 1));
                        best_merge(best, gb, gb, e, a, (a + 1 + jb) % NV);
                    }
                }
            }
            const uint64_t hm = __ballot(best.G >= 0.0);
            if (hm != 0ull) best_wave(best, hm);
            // the last of the wavefronts with candidates publishes their best
            const int cw = min(NW, (ncand + CPW - 1) / CPW), ninl = s_ninl;
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
                    const uint64_t wm = __ballot(lane < cw && best.G >= 0.0);
                    if (wm != 0ull) best_wave(best, wm);
                    if (lane == 0) s_nred = 0;
                }
            }
            if (pub && lane == 0) {
                for (int w = 0; w < ninl; ++w) best_merge(best, s_inl[w].G, s_inl[w].Gmin, s_inl[w].e, s_inl[w].a, s_inl[w].k);
                if (ninl) s_ninl = 0;
                if (best.G >= 0.0)
                    xch::put_slot(my_slot, nwg, ep + 1, best.e, best.a, best.k, best.G, best.Gmin);
                else
                    xch::put_no_slot(my_slot, ep + 1);
            }
        }
        ncached = min(ncand, NC);

        // ---- colour-ordered sums; update; border nodes out, halo in ------------------
        uint64_t *const xb = R.xb + ((ep + 1) & 1u) * xb_half;
        if (nfl & kOwn) {
            double fx = 0.0, fy = 0.0;
#pragma unroll
            for (int d = 0; d < GW; ++d) {
                if (2 * d >= wmax) break;  // uniform
                const double2 f0 = s_f[gat[d] & 0xffffu], f1 = s_f[gat[d] >> 16];
                fx = (fx + f0.x) + f1.x;
                fy = (fy + f0.y) + f1.y;
            }
            const int64_t kabs = base + s;
            const double phi = s_phi;
            double fex = 0.0, fey = 0.0;
            double v0x = 0.0, v0y = 0.0;
            if (nfl & kBc) {
                const int i = (int)(nfl >> kBcAt);
                if (i < kMeshBc) {
                    fex = s_bc[4 * i];
                    fey = s_bc[4 * i + 1];
                    v0x = s_bc[4 * i + 2];
                    v0y = s_bc[4 * i + 3];
                } else {
                    const Args a = again();
                    const int g = a->r.node_id[P.node0 + tid];
                    if (a->p.nflag[g] & kLoaded) {
                        fex = a->p.fext[g].x;
                        fey = a->p.fext[g].y;
                    }
                    if (nfl & (3 * kFix0)) {
                        v0x = a->p.v0[g].x;
                        v0y = a->p.v0[g].y;
                    }
                }
            }
            double ax = (phi * fex - fx) * n_minv;
            double ay = (phi * fey - fy) * n_minv;
            if (nfl & kFix0) ax = 0.0;
            if (nfl & (2 * kFix0)) ay = 0.0;
            const double dtv = (kabs == 0) ? 0.5 * dt : dt;
            double vx = n_v.x + dtv * ax;
            double vy = n_v.y + dtv * ay;
            if (nfl & (3 * kFix0)) {
                const Args a = again();
                const double t = ((double)kabs + 0.5) * a->p.dt, tr = a->p.t_ramp;
                if (nfl & kFix0) vx = dev::prescribed(v0x, t, tr);
                if (nfl & (2 * kFix0)) vy = dev::prescribed(v0y, t, tr);
            }
            n_v = make_double2(vx, vy);
            const double2 u = s_u[tid];
            const double2 un = make_double2(u.x + dt * vx, u.y + dt * vy);
            if (!last) {
                if (nfl & kSend) xch::put_pair(xb + send_at, R.cap, ep + 1, un.x, un.y);
                s_u[tid] = un;
            } else {
                // both buffers as the per-step kernels would leave them
                const Args a = again();
                const int g = R.node_id[P.node0 + tid];
                const bool odd = ((a->par0 + s) & 1) != 0;
                double2 *const cur = odd ? a->p.u1 : a->p.u0, *const nxt = odd ? a->p.u0 : a->p.u1;
                cur[g] = u;
                nxt[g] = un;
                a->p.v[g] = n_v;
            }
        }
        // As in k_resident the first poll waits, here twice as long: by measurement.
        // us per step at nwg / 48, 32, 24, 16, 12 (plates of nx by
        // 0.4 nx cells): 320 000 triangles 7.1, 6.8, 6.7, 7.3, 7.8; 53 000 on the
        // cylinder 6.3, 6.1, 6.0, 6.1, 6.5; triangles at nx = 400 5.4, 4.7, 4.7,
        // 5.3, 5.8, at 250 4.6, 4.5, 4.1, 4.1, 4.5; quadrilaterals at 258 7.8, 7.7,
        // 7.7, 8.3, 8.9; below 24 patches none waits.  It is the slots' wait that
        // counts: the longer one for the other patches' nodes alone changes nothing.
        for (int w = 0; w < nwg / 24; ++w) __builtin_amdgcn_s_sleep(4);
        if (picks) {
            if (!last || b == 0) take_slots(ep + 1, base + s, NT - 1 - tid);
        } else if (!last) {
            const int nh = NT - 64 * pickers;
            for (int h = tid; h < P.nhalo; h += nh) {
                double x, y;
                if (!xch::get_pair(xb + R.halo_src[P.halo0 + h], R.cap, ep + 1, x, y)) {
                    s_stop = 1;
                    break;
                }
                s_u[P.nown + h] = make_double2(x, y);
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
        if (tid == 0) atomicOr(R.err, 1u);
        return;
    }
    if (b != 0) return;
    // ---- patch 0: split codes and U_d in log order -----------------------------
    const int m = s_npicks;
    double *const s_ud = reinterpret_cast<double *>(smem);  // the patch's LDS is free now
    for (int i = tid; i < m; i += NT) {
        const int2 r = s_picks[i];
        p.split[r.x] = (uint8_t)r.y;
        const int4 c = p.conn[r.x];
        const int nd[4] = {c.x, c.y, c.z, c.w};
        const int a = (r.y >> 2) & 3, k = r.y & 3;
        auto at = [&](int n) {
            const int t = n % NV;
            return p.xy[t == 0 ? nd[0] : t == 1 ? nd[1] : t == 2 ? nd[2] : nd[3]];
        };
        const double2 A0 = at(a), A1 = at(a + 1), K0 = at(k), K1 = at(k + 1);
        double nx, ny, len;
        dev::path_geom_pts(A0.x, A0.y, A1.x, A1.y, K0.x, K0.y, K1.x, K1.y, nx, ny, len);
        s_ud[i] = p.gc[r.x] * len;
    }
    __syncthreads();
    if (tid == 0) {
        Ctl *ctl = p.ctl;
        double Ud = ctl->Ud;
        for (int i = 0; i < m; ++i) Ud = Ud + s_ud[i];
        ctl->Ud = Ud;
        ctl->nsplit = nsplit0 + m;
        if (nsplit0 + m > p.log_cap) ctl->overflow = 1;
        ctl->base = base + A.n;
    }
}

template <int NV, int GW>
const void *mesh_kernel_of(int threads) {
    return threads == 512 ? reinterpret_cast<const void *>(k_mesh_resident<NV, 512, 1, GW>)
                          : reinterpret_cast<const void *>(k_mesh_resident<NV, 768, NV == 3 ? 2 : 1, GW>);
}
// (few elements at a node: fewer registers)
const void *mesh_kernel(int nv, int threads, int wmax) {
    if (nv == 3) return wmax <= 10 ? mesh_kernel_of<3, 5>(threads) : mesh_kernel_of<3, 8>(threads);
    return wmax <= 8 ? mesh_kernel_of<4, 4>(threads) : mesh_kernel_of<4, 8>(threads);
}

}  // namespace

// LDS layout of the plan's patches; false when it does not fit a compute unit
// or the grid not the chip.
bool mesh_resident_fits(ResidentMesh &r, int nv, int device) {
    int cus = 0, coop = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return false;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, device) != hipSuccess || !coop) return false;
    const int lpc = nv == 3 ? 2 : 4, nc = mesh_cands(r.threads);
    int at = 0;
    auto take = [&](int64_t bytes) {
        const int a = at;
        at += (int)((bytes + 15) & ~15ll);
        return a;
    };
    r.o_u = take(16ll * r.nl_max);
    if (nv == 3) {
        r.o_q = take(8ll * kTriStrain * r.ne_max);
        r.o_f = take(16ll * (kTriForce * r.np_max + 1));
    } else {
        // the forces over the strains, the zero force behind both
        r.np_max = std::max<int>(r.np_max, (8 * kQuadStrain * r.ne_max + 16 * kQuadForce - 1) / (16 * kQuadForce));
        r.o_q = r.o_f = take(16ll * (kQuadForce * r.np_max + 1));
    }
    r.o_x = take(16ll * r.nl_max);
    r.o_rt = take(nv == 4 ? 16ll * r.nr_max : 0);
    r.o_rg = take(nv == 4 ? 8ll * kRingGrad * r.nr_max : 0);
    r.o_cd = take(8ll * 5 * nv * nc);
    r.o_cn = take(8ll * 2 * lpc * nc);
    r.o_ci = take(8ll * lpc * nc);
    r.o_bc = take(32ll * kMeshBc);
    r.o_cand = take(2ll * nv * nc);
    r.o_cslot = take(2ll * nc);
    r.o_cgc = take(8ll * nc);
    r.o_split = take(2ll * r.np_max);
    r.o_code = take(r.ne_max + r.nr_max);
    r.lds = at;
    if (r.lds > 160 * 1024 - 6144) return false;  // (the static arrays)
    const void *k = mesh_kernel(nv, r.threads, r.wmax);
    if (r.lds > 65536 && hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, r.lds) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, r.threads, r.lds) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return (int64_t)per_cu * cus >= r.npatch;
}

hipError_t launch_mesh_resident(const Params &p, const ResidentMesh &r, int n, int par0, uint32_t &epoch,
                                hipStream_t st) {
    const size_t words = 2 * (size_t)r.npatch;  // of one kind, both parities
    hipError_t e = xch::next_epochs(epoch, n, r.xb, words * xch::pair_words<double>() * r.cap, r.slots,
                                    words * xch::kSlotWords, st);
    if (e != hipSuccess) return e;
    MeshArgs a;
    a.p = p;
    a.r = r;
    a.n = n;
    a.par0 = par0;
    a.epoch0 = epoch;
    void *args[] = {&a};
    (void)hipGetLastError();
    e = hipLaunchCooperativeKernel(mesh_kernel(p.nv, r.threads, r.wmax), dim3(r.npatch), dim3(r.threads), args,
                                   (unsigned)r.lds, st);
    if (e == hipSuccess) epoch += (uint32_t)n;
    return e;
}

}  // namespace tri
}  // namespace mct
