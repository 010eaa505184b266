// The stack of traversals of a four-wide tree, for the test: reads triangles (9 floats
// each) from stdin; writes the build's status, its bound of a traversal that enters the
// nearest child and pushes the others, the most entries of one that pushes every child
// (found by walking the tree), the entries that such a traversal has, and whether the
// four words that the library appends to the triangles have room.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <utility>
#include <vector>

#include "bvh_build.hpp"

int main() {
    std::vector<float> v(9 << 16);
    v.resize(fread(v.data(), 4, v.size(), stdin));
    const int n = (int)(v.size() / 9);
    std::vector<int32_t> t(3 * n);
    for (int i = 0; i < 3 * n; ++i) t[i] = i;
    hyb::BvhHost b;
    const int rc = hyb::build_bvh_host(v.data(), 3 * n, t.data(), n, &b, false);
    int most = 0;
    std::vector<std::pair<int32_t, int>> todo = {{0, 0}};  // node, entries on arrival at it
    while (!todo.empty() && !b.nodes4.empty()) {
        const auto [node, held] = todo.back();
        todo.pop_back();
        int32_t refs[4], kids = 0;
        for (int c = 0; c < 4; ++c) {
            std::memcpy(&refs[kids], &b.nodes4[32 * (size_t)node + 24 + c], 4);
            kids += refs[kids] != hyb::kEmptyRef;
        }
        most = held + kids > most ? held + kids : most;
        for (int c = 0; c < kids; ++c)
            if (refs[c] >= 0) todo.push_back({refs[c], held + kids - 1});
    }
    const int32_t out[5] = {rc, b.stack4, most, hyb::kStackAll4, b.tris.capacity() >= 12 * (size_t)n + 4};
    fwrite(out, 4, 5, stdout);
    return 0;
}
