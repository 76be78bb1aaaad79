// Build-time generator of the operand images of the sample-domain channel
// mixing (gtp_mixq_tables.hpp), degrees 1..8: device arrays, so that a plan
// neither computes nor uploads them.
#include <cstdio>

#include "gtp_mixq_tables.hpp"

int main(int argc, char** argv) {
  if (argc != 2) {
    std::fprintf(stderr, "usage: %s <output>\n", argv[0]);
    return 2;
  }
  std::FILE* f = std::fopen(argv[1], "w");
  if (!f) {
    std::perror(argv[1]);
    return 1;
  }
  std::fprintf(f, "// generated from gtp_mixq_tables.cpp\ntemplate <int L> struct MixqImages;\n");
  for (int L = 1; L <= 8; ++L) {
    const std::vector<uint16_t> v = gtp::build_mixq_images(L);
    std::fprintf(f, "__device__ const uint32_t kMixqImages%d[%zu] __attribute__((aligned(16))) = {", L, v.size() / 2);
    for (size_t i = 0; i < v.size(); i += 2)
      std::fprintf(f, "%s%uu,", i % 24 ? "" : "\n", unsigned(v[i]) | unsigned(v[i + 1]) << 16);
    std::fprintf(f, "\n};\n");
    std::fprintf(f,
                 "template <> struct MixqImages<%d> {\n"
                 "  static __device__ const uint32_t* get() { return kMixqImages%d; }\n};\n",
                 L, L);
  }
  if (std::fclose(f) != 0) {
    std::perror(argv[1]);
    return 1;
  }
  return 0;
}
