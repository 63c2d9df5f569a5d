// Prints a hash of the tree that build_bvh_host makes of meshes of the sizes
// and leaf widths given as argument pairs. Built twice, once with the threads
// on for every mesh and once without them: the lines have to agree.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "../../paper_2606_05581_amd/csrc/msk_internal.h"

int main(int argc, char** argv) {
  for (int a = 1; a + 2 < argc; a += 3) {
    const int nf = std::atoi(argv[a]), leaf = std::atoi(argv[a + 1]), kind = std::atoi(argv[a + 2]);
    std::mt19937 rng(nf);
    std::uniform_real_distribution<float> U(-1.0f, 1.0f);
    std::vector<float> V(9 * (size_t)nf);
    std::vector<int32_t> F(3 * (size_t)nf);
    for (int t = 0; t < nf; ++t) {
      float c[3];
      for (float& x : c) x = U(rng);
      if (kind == 1) c[2] = 0.0f;                  // no extent along one axis
      if (kind == 2) c[0] = c[1] = c[2] = 0.25f;   // coincident centroids
      if (kind == 3) c[0] = std::ldexp(c[0], -(t % 40));  // crowded into one bin
      for (int j = 0; j < 3; ++j) {
        for (int k = 0; k < 3; ++k) V[9 * (size_t)t + 3 * j + k] = c[k] + (j == k ? 0.01f : -0.005f);
        F[3 * (size_t)t + j] = 3 * t + j;
      }
    }
    msk::HostBvh b;
    const std::string err = msk::build_bvh_host(V.data(), 3 * (int64_t)nf, F.data(), nf, leaf, b);
    unsigned long long h = 1469598103934665603ull;
    auto mix = [&](const void* p, size_t n) {
      for (size_t i = 0; i < n; ++i) h = (h ^ ((const unsigned char*)p)[i]) * 1099511628211ull;
    };
    mix(b.nodes.data(), b.nodes.size() * sizeof(msk::Node4));
    mix(b.slot_of_tri.data(), b.slot_of_tri.size() * sizeof(int32_t));
    std::printf("%d %d %d: %zu nodes, depth %d, %016llx %s\n", nf, leaf, kind, b.nodes.size(), b.depth, h, err.c_str());
  }
  return 0;
}
