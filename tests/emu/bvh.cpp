// Host build of a tree, for the test: reads triangles (9 floats each) from stdin,
// writes the two-child nodes (16 words each) and each triangle slot's index.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

#include "bvh_build.hpp"

int main() {
    std::vector<float> v(9 << 16);
    v.resize(fread(v.data(), 4, v.size(), stdin));
    const int n = (int)(v.size() / 9);
    std::vector<int32_t> t(3 * n);
    for (int i = 0; i < 3 * n; ++i) t[i] = i;
    hyb::BvhHost b;
    if (hyb::build_bvh_host(v.data(), 3 * n, t.data(), n, &b, false) != 0) return 1;
    const int32_t head[2] = {(int32_t)(b.nodes.size() / 16), b.depth};
    fwrite(head, 4, 2, stdout);
    fwrite(b.nodes.data(), 4, b.nodes.size(), stdout);
    for (int i = 0; i < n; ++i) fwrite(&b.tris[12 * i + 3], 4, 1, stdout);
    return 0;
}
