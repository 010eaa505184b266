// Binned-SAH BVH2 construction on the host (Wald, "On fast construction of
// SAH-based bounding volume hierarchies", 2007: 32 bins per axis over the
// centroid bounds), flattened into 64-byte two-child nodes (which stay on the
// host), collapsed into 128-byte four-wide nodes that the traversals read with
// 16-byte loads, and the placement of the pyramid of traversal entry points.
#include "bvh_build.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>

#include "entry.hpp"

namespace hyb {
namespace {

constexpr int kBins = 32;
constexpr float kTraversalCost = 1.0f;
constexpr float kTriangleCost = 1.0f;

// x, y, z and a lane that stays out of every result.
typedef float Vec4 __attribute__((vector_size(16)));
typedef int Int4 __attribute__((vector_size(16)));

struct Box {
    Vec4 lo, hi;
    void reset() {
        const float inf = std::numeric_limits<float>::infinity();
        lo = Vec4{inf, inf, inf, inf};
        hi = -lo;
    }
    void grow(const Box& b) {
        lo = b.lo < lo ? b.lo : lo;
        hi = hi < b.hi ? b.hi : hi;
    }
    float area() const {
        const Vec4 d = hi - lo, zero = {};
        const Vec4 e = zero < d ? d : zero;
        return 2.0f * (e[0] * e[1] + e[1] * e[2] + e[2] * e[0]);
    }
};

struct Prim {
    Box box;
    Vec4 c;
};

struct TmpNode {
    Box box;
    int child[2] = {-1, -1};  // indices into the temporary node array
    int first = 0, count = 0; // leaf range in the index array (count > 0 => leaf)
};

struct Builder {
    const std::vector<Prim>& prims;
    std::vector<int> idx;
    std::vector<TmpNode> nodes;
    int max_depth = 0;

    explicit Builder(const std::vector<Prim>& p) : prims(p), idx(p.size()) {
        for (size_t i = 0; i < p.size(); ++i) idx[i] = static_cast<int>(i);
        nodes.reserve(2 * p.size());
    }

    int make_leaf(const Box& b, int first, int count) {
        TmpNode n;
        n.box = b;
        n.first = first;
        n.count = count;
        nodes.push_back(n);
        return static_cast<int>(nodes.size()) - 1;
    }

    // Bins of a centroid along each axis, scale = bins per unit.
    static Int4 bins_of(const Prim& p, Vec4 lo, Vec4 scale) {
        const Int4 b = __builtin_convertvector((p.c - lo) * scale, Int4);
        const Int4 last = {kBins - 1, kBins - 1, kBins - 1, kBins - 1}, zero = {};
        const Int4 m = b < last ? b : last;
        return m > zero ? m : zero;
    }

    // Builds the subtree over idx[first, first+count); returns its node index.
    int build(int first, int count, int depth) {
        max_depth = std::max(max_depth, depth);
        Box bounds, cbounds;
        bounds.reset();
        cbounds.reset();
        for (int i = first; i < first + count; ++i) {
            const Prim& p = prims[idx[i]];
            bounds.grow(p.box);
            cbounds.grow(Box{p.c, p.c});
        }
        if (count == 1) return make_leaf(bounds, first, count);

        // The bins of all three axes in one pass, min and max on whole boxes; `used`
        // has a bit per bin that holds a triangle: near the leaves, where most nodes
        // are, few of the 96 do.  A mesh of 1,052 triangles and its 32^3 grid are
        // ready in 663 us instead of 1,021 with scalar sweeps over every bin; 188,572
        // triangles are built in 0.19 s instead of 0.32 s.
        Box bins[3][kBins];
        int cnt[3][kBins] = {};
        for (int b = 0; b < 3 * kBins; ++b) bins[b / kBins][b % kBins].reset();
        uint32_t used[3] = {0, 0, 0};
        const Vec4 ext = cbounds.hi - cbounds.lo;
        Vec4 scale = {};
        for (int a = 0; a < 3; ++a)
            if (ext[a] > 0.0f) scale[a] = kBins / ext[a];
        for (int i = first; i < first + count; ++i) {
            const Prim& p = prims[idx[i]];
            const Int4 bin = bins_of(p, cbounds.lo, scale);
            for (int a = 0; a < 3; ++a) {
                const int b = bin[a];
                used[a] |= 1u << b;
                bins[a][b].grow(p.box);
                ++cnt[a][b];
            }
        }

        // SAH sweep over the used bins of every axis with a nonzero centroid
        // extent (a split after an empty bin is the split after the used one
        // before it).
        float best_cost = std::numeric_limits<float>::infinity();
        int best_axis = -1, best_split = -1;
        const float parent_area = bounds.area();
        for (int a = 0; a < 3; ++a) {
            if (!(ext[a] > 0.0f)) continue;
            int at[kBins], n_used = 0;
            for (uint32_t left = used[a]; left; left &= left - 1) at[n_used++] = __builtin_ctz(left);
            float right_area[kBins];
            Box acc = bins[a][at[n_used - 1]];
            for (int k = n_used - 1; k > 0; --k) {
                acc.grow(bins[a][at[k]]);
                right_area[k] = acc.area();
            }
            acc.reset();
            int n = 0;
            for (int k = 0; k + 1 < n_used; ++k) {
                acc.grow(bins[a][at[k]]);
                n += cnt[a][at[k]];
                float cost = kTraversalCost +
                             kTriangleCost * (acc.area() * n + right_area[k + 1] * (count - n)) /
                                 std::max(parent_area, 1e-30f);
                if (cost < best_cost) {
                    best_cost = cost;
                    best_axis = a;
                    best_split = at[k];
                }
            }
        }

        const float leaf_cost = kTriangleCost * count;
        if (count <= kLeafMax && leaf_cost <= best_cost) return make_leaf(bounds, first, count);

        int mid;
        if (best_axis < 0) {
            mid = first + count / 2;  // all centroids coincide: split by position in the list
        } else {
            int* m = std::partition(idx.data() + first, idx.data() + first + count, [&](int i) {
                return bins_of(prims[i], cbounds.lo, scale)[best_axis] <= best_split;
            });
            mid = static_cast<int>(m - idx.data());
            if (mid == first || mid == first + count) mid = first + count / 2;
        }
        TmpNode inner;
        inner.box = bounds;
        nodes.push_back(inner);
        int self = static_cast<int>(nodes.size()) - 1;
        int l = build(first, mid - first, depth + 1);
        int r = build(mid, first + count - mid, depth + 1);
        nodes[self].child[0] = l;
        nodes[self].child[1] = r;
        return self;
    }
};

inline float bits_as_float(int32_t v) {
    float f;
    std::memcpy(&f, &v, 4);
    return f;
}

constexpr int kEntryRes = 64;

// Placement of the entry pyramid over the mesh bounds.
void place_entries(BvhHost* out) {
    out->entry.clear();
    out->entry_res = 0;
    out->entry_levels = 0;
    float ext = 0.0f;
    for (int a = 0; a < 3; ++a) ext = std::max(ext, out->hi[a] - out->lo[a]);
    if (out->nodes4.empty() || !(ext > 0.0f)) return;
    const int E = kEntryRes;
    const float size = ext / static_cast<float>(E) * (1.0f + 1e-4f);
    for (int a = 0; a < 3; ++a) out->entry_lo[a] = out->lo[a] - 0.5f * (size * E - (out->hi[a] - out->lo[a]));
    // bounds too far apart for FP32: no pyramid, traversals start at the root
    if (!std::isfinite(size) || !std::isfinite(out->entry_lo[0] + out->entry_lo[1] + out->entry_lo[2])) return;
    out->entry_size = size;
    out->entry_res = E;
    for (int e = E; e >= 1; e >>= 1) ++out->entry_levels;
}

// Entry points of BvhHost (see the header): the finest level by a box query
// per voxel, the coarser ones as the common ancestor of their 8 children.
void build_entries(BvhHost* out) {
    if (out->entry_res == 0) return;
    const size_t n4 = out->nodes4.size() / 32;
    const float* nd = out->nodes4.data();
    auto lca = [&](int32_t a, int32_t b) { return entry_lca(nd, out->tris.data(), a, b); };
    out->entry.assign(static_cast<size_t>(entry_total(out->entry_res)), kEmptyRef);
    // every leaf joins each finest half-cell its box overlaps
    int H = 2 * out->entry_res;
    std::vector<int32_t> cells(static_cast<size_t>(H) * H * H, kEmptyRef);
    for (size_t i = 0; i < n4; ++i)
        for (int c = 0; c < 4; ++c) {
            const float* q = nd + 32 * i;
            const int32_t r = entry_word(q + 24 + c);
            if (r == kEmptyRef || r >= 0) continue;
            int v0[3], v1[3];
            for (int a = 0; a < 3; ++a)
                entry_range(q[8 * a + c], q[8 * a + 4 + c], out->entry_lo[a], out->entry_size, out->entry_res, v0[a],
                            v1[a]);
            for (int z = v0[2]; z <= v1[2]; ++z)
                for (int y = v0[1]; y <= v1[1]; ++y)
                    for (int x = v0[0]; x <= v1[0]; ++x) {
                        int32_t& slot = cells[x + static_cast<size_t>(H) * (y + static_cast<size_t>(H) * z)];
                        slot = lca(slot, r);
                    }
        }
    size_t off = 0;
    for (int l = 0; l < out->entry_levels; ++l) {
        // windows of 2 x 2 x 2 half-cells of this level
        const int W = H - 1;
        for (int z = 0; z < W; ++z)
            for (int y = 0; y < W; ++y)
                for (int x = 0; x < W; ++x) {
                    int32_t acc = kEmptyRef;
                    for (int c = 0; c < 8; ++c) {
                        const int cx = x + (c & 1), cy = y + ((c >> 1) & 1), cz = z + (c >> 2);
                        acc = lca(acc, cells[cx + static_cast<size_t>(H) * (cy + static_cast<size_t>(H) * cz)]);
                    }
                    out->entry[off + x + static_cast<size_t>(W) * (y + static_cast<size_t>(W) * z)] = acc;
                }
        off += static_cast<size_t>(W) * W * W;
        if (l + 1 == out->entry_levels) break;
        // the next level's half-cells: 2 x 2 x 2 of this level's
        const int h = H / 2;
        std::vector<int32_t> up(static_cast<size_t>(h) * h * h, kEmptyRef);
        for (int z = 0; z < h; ++z)
            for (int y = 0; y < h; ++y)
                for (int x = 0; x < h; ++x) {
                    int32_t acc = kEmptyRef;
                    for (int c = 0; c < 8; ++c) {
                        const int cx = 2 * x + (c & 1), cy = 2 * y + ((c >> 1) & 1), cz = 2 * z + (c >> 2);
                        acc = lca(acc, cells[cx + static_cast<size_t>(H) * (cy + static_cast<size_t>(H) * cz)]);
                    }
                    up[x + static_cast<size_t>(h) * (y + static_cast<size_t>(h) * z)] = acc;
                }
        cells.swap(up);
        H = h;
    }
}

}  // namespace

int build_bvh_host(const float* verts, int64_t n_verts, const int32_t* tris, int64_t n_tris, BvhHost* out,
                   bool entries) {
    if (n_verts < 0 || n_tris < 0 || (n_verts > 0 && !verts) || (n_tris > 0 && !tris) || !out) return 1;
    if (n_tris > (int64_t(1) << 28)) return 4;
    for (int64_t i = 0; i < 3 * n_verts; ++i)
        if (!std::isfinite(verts[i])) return 1;
    for (int64_t i = 0; i < 3 * n_tris; ++i)
        if (tris[i] < 0 || tris[i] >= n_verts) return 1;

    std::vector<Prim> prims(static_cast<size_t>(n_tris));
    Box all;
    all.reset();
    for (int64_t t = 0; t < n_tris; ++t) {
        Prim& p = prims[t];
        p.box.reset();
        for (int k = 0; k < 3; ++k) {
            const float* v = verts + 3 * static_cast<int64_t>(tris[3 * t + k]);
            const Vec4 pt = {v[0], v[1], v[2], 0.0f};
            p.box.grow(Box{pt, pt});
        }
        p.c = 0.5f * (p.box.lo + p.box.hi);
        all.grow(p.box);
    }
    for (int a = 0; a < 3; ++a) {
        out->lo[a] = n_tris ? all.lo[a] : 0.0f;
        out->hi[a] = n_tris ? all.hi[a] : 0.0f;
    }

    Builder b(prims);
    int root = -1;
    if (n_tris > 0) root = b.build(0, static_cast<int>(n_tris), 1);
    if (b.max_depth > kMaxDepth) return 4;

    // Flatten depth-first: internal nodes get consecutive output indices, leaves
    // become references into the leaf-ordered triangle array.
    out->nodes.clear();
    out->tris.clear();
    out->tris.reserve(static_cast<size_t>(12 * n_tris + 4));  // the library appends four words
    out->tris.resize(static_cast<size_t>(12 * n_tris), 0.0f);
    int64_t tri_cursor = 0;
    auto leaf_ref = [&](const TmpNode& n) -> int32_t {
        int32_t first = static_cast<int32_t>(tri_cursor);
        for (int i = 0; i < n.count; ++i) {
            int t = b.idx[n.first + i];
            float* dst = out->tris.data() + 12 * tri_cursor;
            for (int k = 0; k < 3; ++k) {
                const float* v = verts + 3 * static_cast<int64_t>(tris[3 * static_cast<int64_t>(t) + k]);
                dst[4 * k + 0] = v[0];
                dst[4 * k + 1] = v[1];
                dst[4 * k + 2] = v[2];
                dst[4 * k + 3] = k == 0 ? bits_as_float(t) : 0.0f;
            }
            ++tri_cursor;
        }
        return ~((first << 3) | n.count);
    };
    std::vector<int32_t> leaf_refs(b.nodes.size(), 0);
    std::vector<char> leaf_done(b.nodes.size(), 0);
    auto leaf_of = [&](int tn) -> int32_t {  // each leaf's triangles are written once
        if (!leaf_done[tn]) {
            leaf_refs[tn] = leaf_ref(b.nodes[tn]);
            leaf_done[tn] = 1;
        }
        return leaf_refs[tn];
    };
    const float far = 1e30f;
    Box empty_box;
    empty_box.lo = empty_box.hi = Vec4{far, far, far, far};

    out->nodes.reserve(8 * b.nodes.size() + 16);
    out->nodes4.clear();
    out->nodes4.reserve(16 * b.nodes.size() + 32);
    auto alloc = [&]() {
        out->nodes.resize(out->nodes.size() + 16, 0.0f);
        return static_cast<int32_t>(out->nodes.size() / 16 - 1);
    };
    auto write_children = [&](int32_t slot, const Box& l, int32_t lref, const Box& r, int32_t rref) {
        float* n = out->nodes.data() + 16 * static_cast<size_t>(slot);
        n[0] = l.lo[0]; n[1] = l.hi[0]; n[2] = l.lo[1]; n[3] = l.hi[1];
        n[4] = r.lo[0]; n[5] = r.hi[0]; n[6] = r.lo[1]; n[7] = r.hi[1];
        n[8] = l.lo[2]; n[9] = l.hi[2]; n[10] = r.lo[2]; n[11] = r.hi[2];
        n[12] = bits_as_float(lref); n[13] = bits_as_float(rref); n[14] = 0.0f; n[15] = 0.0f;
    };

    // BVH4 for the trace kernels: each node takes the children of its BVH2
    // node and replaces the inner child of largest surface area by that
    // child's two children until it has four (or only leaves are left).
    auto emit4 = [&]() {
        out->nodes4.clear();
        auto alloc4 = [&]() {
            out->nodes4.resize(out->nodes4.size() + 32, 0.0f);
            return static_cast<int32_t>(out->nodes4.size() / 32 - 1);
        };
        auto write4 = [&](int32_t slot, const int* kids, int nk) {
            float* q = out->nodes4.data() + 32 * static_cast<size_t>(slot);
            for (int c = 0; c < 4; ++c) {
                const Box& bx = c < nk ? b.nodes[kids[c]].box : empty_box;
                q[0 + c] = bx.lo[0]; q[4 + c] = bx.hi[0];
                q[8 + c] = bx.lo[1]; q[12 + c] = bx.hi[1];
                q[16 + c] = bx.lo[2]; q[20 + c] = bx.hi[2];
            }
        };
        out->depth4 = 1;
        out->stack4 = 0;
        if (root < 0 || b.nodes[root].count > 0) {
            int32_t s = alloc4();
            int kid = root;
            write4(s, &kid, root < 0 ? 0 : 1);
            float* q = out->nodes4.data() + 32 * static_cast<size_t>(s);
            for (int c = 0; c < 4; ++c) q[24 + c] = bits_as_float(c == 0 && root >= 0 ? leaf_of(root) : kEmptyRef);
            q[kNode4Parent] = bits_as_float(-1);
            if (root >= 0) out->tris[kTriLeafParent] = bits_as_float(0);
            return;
        }
        // `pushed`: stack entries a traversal can hold on arrival at the node
        // (the nearer-first order pushes the other hit children of every
        // ancestor), so its maximum bounds the traversal stack.
        struct Item { int tn; int32_t slot; int depth; int pushed; };
        std::vector<Item> st;
        st.push_back({root, alloc4(), 1, 0});
        out->nodes4[kNode4Parent] = bits_as_float(-1);
        while (!st.empty()) {
            const Item it = st.back();
            st.pop_back();
            out->depth4 = std::max(out->depth4, it.depth);
            int kids[4] = {b.nodes[it.tn].child[0], b.nodes[it.tn].child[1], -1, -1};
            int nk = 2;
            while (nk < 4) {
                int best = -1;
                float best_area = -1.0f;
                for (int c = 0; c < nk; ++c) {
                    const TmpNode& ch = b.nodes[kids[c]];
                    if (ch.count == 0 && ch.box.area() > best_area) {
                        best_area = ch.box.area();
                        best = c;
                    }
                }
                if (best < 0) break;
                const TmpNode& ch = b.nodes[kids[best]];
                kids[best] = ch.child[0];
                kids[nk++] = ch.child[1];
            }
            write4(it.slot, kids, nk);
            out->stack4 = std::max(out->stack4, it.pushed + nk - 1);
            int32_t refs[4] = {kEmptyRef, kEmptyRef, kEmptyRef, kEmptyRef};
            Item pending[4];
            int np = 0;
            for (int c = 0; c < nk; ++c) {
                if (b.nodes[kids[c]].count > 0) {
                    refs[c] = leaf_of(kids[c]);
                    out->tris[12 * static_cast<size_t>((~refs[c]) >> 3) + kTriLeafParent] = bits_as_float(it.slot);
                } else {
                    refs[c] = alloc4();
                    float* child = out->nodes4.data() + 32 * static_cast<size_t>(refs[c]);
                    child[kNode4Parent] = bits_as_float(it.slot);
                    child[kNode4Depth] = bits_as_float(it.depth);
                    pending[np++] = {kids[c], refs[c], it.depth + 1, it.pushed + nk - 1};
                }
            }
            float* q = out->nodes4.data() + 32 * static_cast<size_t>(it.slot);
            for (int c = 0; c < 4; ++c) q[24 + c] = bits_as_float(refs[c]);
            for (int c = np - 1; c >= 0; --c) st.push_back(pending[c]);
        }
    };

    if (root < 0) {
        int32_t s = alloc();
        write_children(s, empty_box, kEmptyRef, empty_box, kEmptyRef);
        out->depth = 1;
        emit4();
        place_entries(out);
        if (entries) build_entries(out);
        return 0;
    }
    if (b.nodes[root].count > 0) {
        int32_t s = alloc();
        int32_t lr = leaf_of(root);
        write_children(s, b.nodes[root].box, lr, empty_box, kEmptyRef);
        out->depth = 1;
        emit4();
        place_entries(out);
        if (entries) build_entries(out);
        return 0;
    }
    // iterative pre-order so the left child usually follows its parent in memory
    std::vector<std::pair<int, int32_t>> stack;
    stack.push_back({root, alloc()});
    while (!stack.empty()) {
        auto [tn, slot] = stack.back();
        stack.pop_back();
        const TmpNode& n = b.nodes[tn];
        int32_t refs[2];
        int32_t pending_slot[2] = {-1, -1};
        for (int c = 0; c < 2; ++c) {
            const TmpNode& ch = b.nodes[n.child[c]];
            if (ch.count > 0) {
                refs[c] = leaf_of(n.child[c]);
            } else {
                pending_slot[c] = alloc();
                refs[c] = pending_slot[c];
            }
        }
        write_children(slot, b.nodes[n.child[0]].box, refs[0], b.nodes[n.child[1]].box, refs[1]);
        for (int c = 1; c >= 0; --c)
            if (pending_slot[c] >= 0) stack.push_back({n.child[c], pending_slot[c]});
    }
    out->depth = b.max_depth;
    emit4();
    if (out->stack4 > kStackDepth4) return 4;
    place_entries(out);
    if (entries) build_entries(out);
    return 0;
}

}  // namespace hyb
