// Every layer of a network, every batch up to max_batch: the chunks of the
// weight gradients against the bounds that size their workspace at max_batch,
// and the positions that the chunks cover.
//
//   wgrad_chunks_check <width> <positions per window> <embedding columns> <head rows> <largest max_batch>
// prints the number of batches whose chunks exceed the bound of their
// max_batch, of those with more chunks than max_batch itself has, and of those
// whose chunks do not cover all positions exactly once.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "wgrad_chunks.hpp"

int main(int argc, char** argv) {
  if (argc != 6) return 2;
  const int C = std::atoi(argv[1]), Lpos = std::atoi(argv[2]), E = std::atoi(argv[3]), H = std::atoi(argv[4]),
            most = std::atoi(argv[5]);
  struct Layer {
    int M, Cin, Kr;
  };
  const Layer layers[] = {{C, E, E}, {C, C, 3 * C}, {H, C, C}};
  long over = 0, more = 0, uncovered = 0;
  for (const Layer& L : layers)
    for (int form = 0; form < 2; ++form) {
      auto bound = [&](int N) { return form ? wsn::direct_bound(L.M, L.Cin, N) : wsn::wgrad_bound(L.M, L.Kr, N); };
      auto plan = [&](int N) { return form ? wsn::direct_chunks(L.M, L.Cin, N) : wsn::wgrad_chunks(L.M, L.Kr, N); };
      int largest = 0;   // most chunks of any batch so far
      for (int n = 1; n <= most; ++n) {
        const int N = n * Lpos;
        const wsn::Chunks c = plan(N);
        largest = largest > c.count ? largest : c.count;
        over += largest > bound(N);
        more += largest > c.count;
        uncovered += !(c.chunk > 0 && (c.count - 1) * long(c.chunk) < N && c.count * long(c.chunk) >= N);
      }
    }
  std::printf("%ld %ld %ld\n", over, more, uncovered);
  return 0;
}
