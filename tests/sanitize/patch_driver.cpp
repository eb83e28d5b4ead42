// Sanitizer harness of the host code that cuts patches in two, counts each patch's working set, and forms the units and
// chunks of the row-owned evaluation (built with g++ under AddressSanitizer + UndefinedBehaviorSanitizer and,
// separately, ThreadSanitizer by test_patch_driver.py beside it). Exits non-zero on the first violated invariant.
// Test infrastructure: not part of the library.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "mad_internal.hpp"
#include "mlp.hpp"

namespace mad {
// the library's error reporting lives with the C ABI (api.cpp), which this harness does not link
static std::string g_err;
void set_error(const std::string& msg) { g_err = msg; }
int fail(int code, const std::string& msg) {
    g_err = msg;
    return code;
}
}  // namespace mad

using namespace mad;

#define CHECK(cond)                                                                 \
    do {                                                                            \
        if (!(cond)) {                                                              \
            std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #cond); \
            std::exit(2);                                                           \
        }                                                                           \
    } while (0)

struct MeshIn {
    std::string name;
    int64_t nv = 0;
    std::vector<int32_t> tris;
    std::vector<int64_t> comp;   // empty: one component
};

static void add_grid(MeshIn& m, int n) {
    const int32_t base = (int32_t)m.nv;
    for (int j = 0; j + 1 < n; ++j)
        for (int i = 0; i + 1 < n; ++i) {
            const int32_t v00 = base + j * n + i, v10 = v00 + 1, v01 = v00 + n, v11 = v01 + 1;
            m.tris.insert(m.tris.end(), {v00, v10, v11, v00, v11, v01});
        }
    m.nv += (int64_t)n * n;
}

static void add_fan(MeshIn& m, int k) {
    const int32_t b = (int32_t)m.nv;
    for (int i = 0; i < k; ++i) {
        const int32_t p = b + 1 + i, q = b + 1 + (i + 1) % k;
        m.tris.insert(m.tris.end(), {b, p, q, b + k + 1, q, p});
    }
    m.nv += k + 2;
}

static std::vector<MeshIn> meshes() {
    std::vector<MeshIn> out;
    MeshIn a{"grid 170x170"};   // groups of more than 4096 faces: cut level by level, by several threads
    add_grid(a, 170);
    out.push_back(a);
    MeshIn b{"components, one of them without a face"};
    b.comp.push_back(0);
    for (int n : {7, 12, 0, 5, 20, 2}) {
        if (n) add_grid(b, n);
        else b.nv += 3;
        b.comp.push_back(b.nv);
    }
    add_fan(b, 90);
    b.comp.push_back(b.nv);
    out.push_back(b);
    MeshIn c{"fan of valence 300, vertices on no face"};
    c.nv = 70;
    add_fan(c, 300);
    c.nv += 5;
    out.push_back(c);
    MeshIn d{"non-manifold"};
    d.tris = {0, 1, 2, 1, 0, 3, 0, 1, 4, 2, 1, 5, 5, 1, 6};
    d.nv = 8;
    out.push_back(d);
    MeshIn e{"loose faces"};
    for (int32_t f = 0; f < 40; ++f) e.tris.insert(e.tris.end(), {3 * f, 3 * f + 1, 3 * f + 2});
    e.nv = 120;
    out.push_back(e);
    return out;
}

static void make(const MeshIn& in, mad_mesh& mesh, mad_problem& P) {
    mesh.nv = in.nv;
    mesh.nt = (int64_t)in.tris.size() / 3;
    mesh.tris = in.tris;
    mesh.comp_off = in.comp.empty() ? std::vector<int64_t>{0, in.nv} : in.comp;
    mesh.batched = !in.comp.empty();
    CHECK(build_topology(mesh) == MAD_OK);
    P.mesh = &mesh;
    P.d = 3;
    P.prec = MAD_F32;
    for (int kind : {(int)MAD_STVK, (int)MAD_BENDING}) {
        Term t;
        t.kind = kind;
        t.ns = kind_stencil(kind);
        t.d = 3;
        t.stencil = kind == MAD_STVK ? mesh.tris : mesh.diamonds;
        t.n = (int64_t)t.stencil.size() / t.ns;
        P.terms.push_back(std::move(t));
    }
}

// the faces of every patch, sorted, after checking that the patches are a partition that keeps components apart
static std::vector<std::vector<int32_t>> faces_of(const mad_mesh& m, const Patches& P) {
    CHECK((int32_t)P.start.size() == P.n + 1 && P.start[0] == 0 && P.start[P.n] == m.nt);
    CHECK((int64_t)P.order.size() == m.nt && (int64_t)P.face_patch.size() == m.nt);
    auto comp = [&](int32_t f) {
        return (int)(std::upper_bound(m.comp_off.begin(), m.comp_off.end(), (int64_t)m.tris[3 * (int64_t)f]) - m.comp_off.begin()) - 1;
    };
    std::vector<std::vector<int32_t>> out;
    std::vector<uint8_t> seen((size_t)m.nt, 0);
    CHECK(P.comp_patch_ptr.size() == m.comp_off.size() && P.comp_patch_ptr.back() == P.n);
    for (int32_t p = 0; p < P.n; ++p) {
        CHECK(P.start[p + 1] > P.start[p]);
        std::vector<int32_t> f(P.order.begin() + P.start[p], P.order.begin() + P.start[p + 1]);
        for (int32_t x : f) {
            CHECK(!seen[x] && P.face_patch[x] == p && comp(x) == comp(f[0]));
            seen[x] = 1;
        }
        CHECK(p >= P.comp_patch_ptr[comp(f[0])] && p < P.comp_patch_ptr[comp(f[0]) + 1]);
        std::sort(f.begin(), f.end());
        out.push_back(std::move(f));
    }
    return out;
}

static void check_halving(const MeshIn& in, int target, int every) {
    mad_mesh mesh;
    mad_problem P;
    make(in, mesh, P);
    build_patches(mesh, target, P.patches);
    const auto before = faces_of(mesh, P.patches);
    std::vector<uint8_t> which(before.size(), 0);
    for (size_t p = 0; p < which.size(); ++p) which[p] = p % every == 0;
    halve_patches(mesh, which, P.patches);
    const auto after = faces_of(mesh, P.patches);
    // in order: an unmarked patch as it was, a marked one as two halves (one face cannot be cut)
    size_t q = 0;
    for (size_t p = 0; p < before.size(); ++p) {
        CHECK(q < after.size());
        if (!which[p] || before[p].size() == 1) {
            CHECK(after[q] == before[p]);
            ++q;
            continue;
        }
        CHECK(q + 1 < after.size());
        CHECK(after[q].size() == before[p].size() / 2);
        std::vector<int32_t> both(after[q]);
        both.insert(both.end(), after[q + 1].begin(), after[q + 1].end());
        std::sort(both.begin(), both.end());
        CHECK(both == before[p]);
        q += 2;
    }
    CHECK(q == after.size());
    // each patch's working set, counted with sets
    order_terms(&P);
    int32_t mv = 0, mb = 0;
    std::vector<std::pair<int32_t, int32_t>> each;
    patch_extent(&P, &mv, &mb, &each);
    CHECK((int32_t)each.size() == P.patches.n);
    int32_t top_v = 0, top_b = 0;
    for (int32_t p = 0; p < P.patches.n; ++p) {
        std::set<int32_t> verts;
        std::set<std::pair<int32_t, int32_t>> blocks;
        for (const Term& t : P.terms)
            for (int32_t i = t.elem_ptr[p]; i < t.elem_ptr[p + 1]; ++i)
                for (int a = 0; a < t.ns; ++a)
                    for (int b = 0; b < t.ns; ++b) {
                        const int32_t u = t.stencil[(int64_t)t.perm[i] * t.ns + a], v = t.stencil[(int64_t)t.perm[i] * t.ns + b];
                        verts.insert(u);
                        if (u <= v) blocks.insert({u, v});
                    }
        CHECK(each[p].first == (int32_t)verts.size() && each[p].second == (int32_t)blocks.size());
        top_v = std::max(top_v, each[p].first);
        top_b = std::max(top_b, each[p].second);
    }
    CHECK(top_v == mv && top_b == mb);
    // another target after a halving starts over from the kept cuts
    build_patches(mesh, std::max(1, target / 2), P.patches);
    faces_of(mesh, P.patches);
    std::printf("%s, target %d: %zu patches, %zu after halving every %d\n", in.name.c_str(), target, before.size(), after.size(), every);
}

static void check_rows(const MeshIn& in, int step, int64_t wanted) {
    mad_mesh mesh;
    mad_problem P;
    make(in, mesh, P);
    std::vector<int32_t> rowptr(1, 0);
    std::vector<std::set<int32_t>> rows((size_t)mesh.nv);
    for (int64_t v = 0; v < mesh.nv; ++v) rows[v].insert((int32_t)v);
    for (int64_t e = 0; e < mesh.ne(); ++e) {
        rows[mesh.edges[2 * e]].insert(mesh.edges[2 * e + 1]);
        rows[mesh.edges[2 * e + 1]].insert(mesh.edges[2 * e]);
    }
    for (const auto& r : rows) rowptr.push_back(rowptr.back() + (int32_t)r.size());
    std::vector<int32_t> unit, chunk, comp_chunk;
    row_units(rowptr, mesh.comp_off, step, wanted, unit, chunk, comp_chunk);
    const int64_t nu = (int64_t)unit.size() - 1, nc = (int64_t)chunk.size() - 1, ncomp = (int64_t)mesh.comp_off.size() - 1;
    CHECK(unit[0] == 0 && unit[nu] == mesh.nv && chunk[0] == 0 && chunk[nc] == nu);
    CHECK((int64_t)comp_chunk.size() == ncomp + 1 && comp_chunk[0] == 0 && comp_chunk[ncomp] == nc);
    auto comp = [&](int32_t row) {
        return (int64_t)(std::upper_bound(mesh.comp_off.begin(), mesh.comp_off.end(), (int64_t)row) - mesh.comp_off.begin()) - 1;
    };
    for (int64_t u = 0; u < nu; ++u) {
        CHECK(unit[u] < unit[u + 1] && comp(unit[u]) == comp(unit[u + 1] - 1));
        // at most 64 blocks, or one row; and no more rows than lanes (a row has at least its diagonal block)
        CHECK(rowptr[unit[u + 1]] - rowptr[unit[u]] <= 64 || unit[u + 1] - unit[u] == 1);
        CHECK(unit[u + 1] - unit[u] <= 64);
        // as full as the next row allows
        if (u + 1 < nu && comp(unit[u + 1]) == comp(unit[u])) CHECK(rowptr[unit[u + 1] + 1] - rowptr[unit[u]] > 64);
    }
    const int64_t per = step * std::min<int64_t>(4, std::max<int64_t>(1, nu / (step * std::max<int64_t>(wanted, 1))));
    for (int64_t c = 0; c < ncomp; ++c)
        for (int32_t k = comp_chunk[c]; k < comp_chunk[c + 1]; ++k) {
            CHECK(chunk[k] < chunk[k + 1] && chunk[k + 1] - chunk[k] <= per);
            CHECK(comp(unit[chunk[k]]) == c && comp(unit[chunk[k + 1]] - 1) == c);
            if (k + 1 < comp_chunk[c + 1]) CHECK(chunk[k + 1] - chunk[k] == per);   // full but for a component's last
        }
    std::printf("%s: %lld units, %lld chunks of at most %lld\n", in.name.c_str(), (long long)nu, (long long)nc, (long long)per);
}

int main() {
    for (const MeshIn& m : meshes()) {
        for (int target : {1, 7, 64, 500, 3000})
            for (int every : {1, 3}) check_halving(m, target, every);
        for (int64_t wanted : {0, 1, 20, 2048}) check_rows(m, 4, wanted);
    }
    // training workgroups: one for four samples, at least one, at most what the device has room for
    for (int most : {2, 64, 512})
        for (int64_t n : {0ll, 1ll, 4ll, 5ll, 8ll * most, 4000000000ll}) {
            const int r = train_rows(n, most);
            CHECK(r >= 1 && r <= most && (r == most || (int64_t)r * 4 >= n));
            CHECK(r == 1 || (int64_t)(r - 1) * 4 < n);
        }
    std::printf("patch and row checks passed\n");
    return 0;
}
