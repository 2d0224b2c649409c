// Host side of the resident step of an unstructured mesh: its patches and
// their tables.
//
// Patches come from a recursive bisection of the node coordinates into equal
// counts (any node numbering gives compact patches).  The number: meshes that
// fit 512-thread patches use those, larger ones
// one 768-thread patch on every compute unit; a mesh whose patches exceed the
// kernel's threads, tables or LDS keeps the per-step kernels.
#include <algorithm>
#include <cstring>
#include <new>
#include <numeric>
#include <type_traits>

#include "mct2d_impl.h"
#include "mct2d_tri_host.h"

namespace mct {
namespace tri {
namespace {

// Nodes of a 512-thread patch (380 triangles and their ring at 190), in the order
// tried: 160 fit most meshes at once, and 54 000 triangles take the same time per
// step at 107, 130 and 160.
constexpr int kSmallPatch[] = {160, 190, 130};

void bisect(const Model &m, int32_t *ids, int64_t n, int parts, std::vector<int64_t> &sizes) {
    if (parts == 1) {
        std::sort(ids, ids + n);
        sizes.push_back(n);
        return;
    }
    double x0 = m.X[ids[0]], x1 = x0, y0 = m.Y[ids[0]], y1 = y0;
    for (int64_t i = 1; i < n; ++i) {
        x0 = std::min(x0, m.X[ids[i]]);
        x1 = std::max(x1, m.X[ids[i]]);
        y0 = std::min(y0, m.Y[ids[i]]);
        y1 = std::max(y1, m.Y[ids[i]]);
    }
    const std::vector<double> &K = x1 - x0 >= y1 - y0 ? m.X : m.Y;
    const std::vector<double> &L = x1 - x0 >= y1 - y0 ? m.Y : m.X;
    const int pl = parts / 2;
    const int64_t cut = n * pl / parts;
    std::nth_element(ids, ids + cut, ids + n, [&](int32_t a, int32_t b) {
        if (K[a] != K[b]) return K[a] < K[b];
        if (L[a] != L[b]) return L[a] < L[b];
        return a < b;
    });
    bisect(m, ids, cut, pl, sizes);
    bisect(m, ids + cut, n - cut, parts - pl, sizes);
}

struct Tables {
    std::vector<MeshPatch> patch;
    std::vector<int32_t> node_id, node_send, halo_src;
    std::vector<uint16_t> gather;
    std::vector<uint32_t> slot_eid, redge_eid, redge_at;
    std::vector<uint2> slot_lc, slot_nb, slot_code, redge_lc;
    std::vector<int4> slot_far;
};

uint2 pack16(const int v[4]) {
    return make_uint2((uint32_t)v[0] | (uint32_t)v[1] << 16, (uint32_t)v[2] | (uint32_t)v[3] << 16);
}

// Patches of `parts` for kernels of `threads` threads and `slots` element
// slots; false when they exceed the kernel's limits.
bool build(const Model &m, int parts, int threads, int slots, int device, ResidentMesh &r, Tables &t) {
    const int nv = m.nv;
    const int64_t nn = m.nn, ne = m.ne;
    if (nn > (int64_t)parts * threads || ne > (int64_t)parts * slots) return false;  // (before any work on a large mesh)
    r = ResidentMesh{};
    r.threads = threads;
    r.npatch = parts;
    std::vector<int32_t> order((size_t)nn);
    std::iota(order.begin(), order.end(), 0);
    std::vector<int64_t> sizes;
    bisect(m, order.data(), nn, parts, sizes);
    std::vector<int32_t> part((size_t)nn), local((size_t)nn);  // of a node: its patch, its place there
    {
        int64_t at = 0;
        for (int b = 0; b < parts; ++b)
            for (int64_t i = 0; i < sizes[b]; ++i, ++at) {
                part[order[at]] = b;
                local[order[at]] = (int32_t)i;
            }
    }
    for (int64_t i = 0; i < nn; ++i) r.wmax = std::max(r.wmax, m.gnoff[i + 1] - m.gnoff[i]);
    if (r.wmax > 16) return false;
    t = Tables{};
    std::vector<int32_t> epos((size_t)ne, -1), emark((size_t)ne, -1), npos((size_t)nn, -1), nmark((size_t)nn, -1);
    std::vector<int32_t> exported((size_t)nn, -1);  // place among the nodes its patch sends
    std::vector<std::vector<int32_t>> els((size_t)parts), ring((size_t)parts), halo((size_t)parts);
    // per patch: elements, ring, halo; and the strides
    for (int64_t e = 0; e < ne; ++e) {
        int seen[4], ns = 0;
        for (int n = 0; n < nv; ++n) {
            const int b = part[m.conn[nv * e + n]];
            bool dup = false;
            for (int i = 0; i < ns; ++i) dup = dup || seen[i] == b;
            if (dup) continue;
            seen[ns++] = b;
            els[b].push_back((int32_t)e);
        }
    }
    std::vector<int32_t> nredge((size_t)parts, 0);
    for (int b = 0; b < parts; ++b) {
        for (int32_t e : els[b]) emark[e] = b;
        for (int32_t e : els[b])
            for (int k = 0; k < nv; ++k) {
                const int32_t nb = m.nbr[(nv + 1) * (int64_t)e + k];
                if (nb < 0 || emark[nb] == b) continue;
                if (emark[nb] != parts + b) {
                    emark[nb] = parts + b;
                    ring[b].push_back(nb);
                }
                ++nredge[b];
            }
        std::sort(ring[b].begin(), ring[b].end());
        auto add = [&](int32_t e) {
            for (int n = 0; n < nv; ++n) {
                const int32_t g = m.conn[nv * (int64_t)e + n];
                if (part[g] == b || nmark[g] == b) continue;
                nmark[g] = b;
                halo[b].push_back(g);
            }
        };
        for (int32_t e : els[b]) add(e);
        for (int32_t e : ring[b]) add(e);
        std::sort(halo[b].begin(), halo[b].end());
        for (int32_t g : halo[b]) exported[g] = 0;
        const int nel = (int)els[b].size(), nri = (int)ring[b].size();
        const int nslot = nv == 3 ? nel + nri : nel;
        if (sizes[b] > threads || nslot > slots) return false;
        if (nv == 4) {
            if (nredge[b] > threads) return false;
            r.nr_max = std::max(r.nr_max, nredge[b]);
        }
        r.ne_max = std::max(r.ne_max, nv == 3 ? nslot : nel + (nredge[b] + 3) / 4);
        r.np_max = std::max(r.np_max, nel);
        r.nl_max = std::max<int32_t>(r.nl_max, (int32_t)(sizes[b] + (int64_t)halo[b].size()));
    }
    if (!mesh_resident_fits(r, nv, device)) return false;
    const int qs = nv == 3 ? kTriStrain : kQuadStrain, fs = nv == 3 ? kTriForce : kQuadForce;
    if (qs * r.ne_max > 0xffff || fs * r.np_max >= 0xffff) return false;
    std::vector<int32_t> nsent((size_t)parts, 0);
    for (int64_t i = 0; i < nn; ++i)
        if (exported[order[i]] == 0) exported[order[i]] = nsent[part[order[i]]]++;
    r.cap = std::max(1, *std::max_element(nsent.begin(), nsent.end()));
    const int words = 3;  // per node sent
    auto first_word = [&](int32_t g) { return part[g] * words * r.cap + exported[g]; };
    int64_t at = 0;
    for (int b = 0; b < parts; ++b) {
        MeshPatch p{};
        p.node0 = (int32_t)t.node_id.size();
        p.own0 = (int32_t)t.node_send.size();
        p.halo0 = (int32_t)t.halo_src.size();
        p.slot0 = (int32_t)t.slot_eid.size();
        p.redge0 = (int32_t)t.redge_eid.size();
        p.nown = (int32_t)sizes[b];
        p.nhalo = (int32_t)halo[b].size();
        p.nel = (int32_t)els[b].size();
        for (size_t i = 0; i < els[b].size(); ++i) {
            epos[els[b][i]] = (int32_t)i;
            emark[els[b][i]] = b;
        }
        for (size_t i = 0; i < ring[b].size(); ++i) {
            epos[ring[b][i]] = p.nel + (int32_t)i;
            emark[ring[b][i]] = parts + b;
        }
        for (int64_t i = 0; i < sizes[b]; ++i, ++at) {
            const int32_t g = order[at];
            npos[g] = (int32_t)i;
            t.node_id.push_back(g);
            t.node_send.push_back(exported[g] < 0 ? -1 : first_word(g));
            int w = 0;
            for (int32_t q = m.gnoff[g]; q < m.gnoff[g + 1]; ++q, ++w) {
                const int32_t ent = m.gnel[q], e = ent / nv, n = ent % nv;
                t.gather.push_back((uint16_t)(fs * epos[e] + n));
            }
            for (; w < 16; ++w) t.gather.push_back((uint16_t)(fs * r.np_max));
        }
        for (size_t i = 0; i < halo[b].size(); ++i) {
            const int32_t g = halo[b][i];
            npos[g] = p.nown + (int32_t)i;
            t.node_id.push_back(g);
            t.halo_src.push_back(first_word(g));
        }
        auto nodes = [&](int32_t e) {
            int v[4] = {0, 0, 0, 0};
            for (int n = 0; n < nv; ++n) v[n] = npos[m.conn[nv * (int64_t)e + n]];
            return pack16(v);
        };
        for (int32_t e : els[b]) {
            const int32_t *nb = &m.nbr[(nv + 1) * (int64_t)e];
            int pl[4] = {0, 0, 0, 0}, cd[4] = {0xffff, 0xffff, 0xffff, 0xffff}, far[4] = {-1, -1, -1, -1};
            for (int k = 0; k < nv; ++k) {
                if (nb[k] < 0) continue;
                far[k] = nb[k];
                const int loc = (nb[nv] >> (2 * k)) & 3;
                if (nv == 3) {
                    pl[k] = qs * epos[nb[k]];
                    cd[k] = epos[nb[k]];
                } else if (emark[nb[k]] == b) {
                    pl[k] = qs * epos[nb[k]] + 3 * loc;
                    cd[k] = epos[nb[k]];
                } else {
                    const int i = p.nredge++;
                    pl[k] = qs * (p.nel + (i >> 2)) + 3 * (i & 3);
                    cd[k] = r.ne_max + i;
                    t.redge_eid.push_back((uint32_t)nb[k]);
                    t.redge_lc.push_back(nodes(nb[k]));
                    t.redge_at.push_back((uint32_t)pl[k] | (uint32_t)loc << 16);
                }
            }
            const bool owned = part[m.conn[nv * (int64_t)e]] == b;
            t.slot_eid.push_back((uint32_t)e | (owned ? (uint32_t)kOwned : 0u));
            t.slot_lc.push_back(nodes(e));
            t.slot_nb.push_back(pack16(pl));
            t.slot_code.push_back(pack16(cd));
            t.slot_far.push_back(make_int4(far[0], far[1], far[2], far[3]));
        }
        if (nv == 3) {
            p.nring = (int32_t)ring[b].size();
            for (int32_t e : ring[b]) {
                t.slot_eid.push_back((uint32_t)e);
                t.slot_lc.push_back(nodes(e));
                t.slot_nb.push_back(make_uint2(0, 0));
                t.slot_code.push_back(make_uint2(0, 0));
                t.slot_far.push_back(make_int4(-1, -1, -1, -1));
            }
        }
        t.patch.push_back(p);
    }
    return true;
}

hipError_t plan(Model &m, hipStream_t stream);

}  // namespace

void free_resident(Model &m) {
    if (m.res.tables) (void)hipFree(m.res.tables);
    m.res = ResidentMesh{};
    m.res_epoch = 0;  // (new buffers are cleared)
}

// Builds the resident step's patches where it applies (automatic kernels, the
// global pick of every tip); leaves m.res.threads 0 otherwise.
hipError_t plan_resident(Model &m, hipStream_t stream) {
    free_resident(m);
    try {
        return plan(m, stream);
    } catch (const std::bad_alloc &) {  // no memory for the tables: the per-step kernels need none of them
        return hipSuccess;
    }
}

namespace {

hipError_t plan(Model &m, hipStream_t stream) {
    if (m.kernels != 0 || m.sct || m.front_rho > 0 || m.ne == 0) return hipSuccess;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (!whole_device(stream, dev)) return hipSuccess;
    ResidentMesh r;
    Tables t;
    bool ok = false;
    for (int P : kSmallPatch) {
        const int64_t parts = (m.nn + P - 1) / P;
        if (parts > kMeshResidentPatches) continue;
        if ((ok = build(m, (int)parts, 512, 512, dev, r, t))) break;
    }
    if (!ok && m.nn >= kMeshResidentPatches)
        ok = build(m, kMeshResidentPatches, 768, m.nv == 3 ? 1536 : 768, dev, r, t);
    if (!ok) return hipSuccess;
    // one allocation: tables, exchange words, slots
    size_t bytes = 0;
    auto place = [&](size_t n) {
        const size_t at = bytes;
        bytes += (n + 15) & ~(size_t)15;
        return at;
    };
    auto of = [&](const auto &v) { return place(v.size() * sizeof(v[0])); };
    const size_t o_patch = of(t.patch), o_id = of(t.node_id), o_send = of(t.node_send), o_gather = of(t.gather),
                 o_halo = of(t.halo_src), o_eid = of(t.slot_eid), o_lc = of(t.slot_lc), o_nb = of(t.slot_nb),
                 o_code = of(t.slot_code), o_far = of(t.slot_far), o_re = of(t.redge_eid), o_rl = of(t.redge_lc),
                 o_ra = of(t.redge_at);
    const size_t table_bytes = bytes;
    const size_t o_xb = place(sizeof(uint64_t) * 2 * 3 * (size_t)r.npatch * r.cap);
    const size_t o_sl = place(sizeof(uint64_t) * 2 * 4 * (size_t)r.npatch);
    std::vector<char> blob(table_bytes);
    auto copy = [&](size_t at, const auto &v) {
        if (!v.empty()) std::memcpy(blob.data() + at, v.data(), v.size() * sizeof(v[0]));
    };
    copy(o_patch, t.patch);
    copy(o_id, t.node_id);
    copy(o_send, t.node_send);
    copy(o_gather, t.gather);
    copy(o_halo, t.halo_src);
    copy(o_eid, t.slot_eid);
    copy(o_lc, t.slot_lc);
    copy(o_nb, t.slot_nb);
    copy(o_code, t.slot_code);
    copy(o_far, t.slot_far);
    copy(o_re, t.redge_eid);
    copy(o_rl, t.redge_lc);
    copy(o_ra, t.redge_at);
    char *d = nullptr;
    if (hipMalloc((void **)&d, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return hipSuccess;  // the per-step kernels need none of it
    }
    r.tables = d;
    if ((e = hipMemcpyAsync(d, blob.data(), table_bytes, hipMemcpyHostToDevice, stream)) == hipSuccess)
        e = hipMemsetAsync(d + o_xb, 0, bytes - o_xb, stream);
    const hipError_t e2 = hipStreamSynchronize(stream);
    if (e == hipSuccess) e = e2;
    if (e != hipSuccess) {
        (void)hipFree(d);
        return e;
    }
    auto at = [&](auto *&p, size_t o) { p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(d + o); };
    at(r.patch, o_patch);
    at(r.node_id, o_id);
    at(r.node_send, o_send);
    at(r.node_gather, o_gather);
    at(r.halo_src, o_halo);
    at(r.slot_eid, o_eid);
    at(r.slot_lc, o_lc);
    at(r.slot_nb, o_nb);
    at(r.slot_code, o_code);
    at(r.slot_far, o_far);
    at(r.redge_eid, o_re);
    at(r.redge_lc, o_rl);
    at(r.redge_at, o_ra);
    at(r.xb, o_xb);
    at(r.slots, o_sl);
    r.err = reinterpret_cast<uint32_t *>(m.dctl + 1);
    m.res = r;
    return hipSuccess;
}

}  // namespace
}  // namespace tri
}  // namespace mct
