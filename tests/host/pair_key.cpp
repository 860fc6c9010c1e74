// Packing of the pair keys, with and without the species, up to the largest
// atom index a batch may hold: fields come back, the order of the keys is that of
// (shell, [species,] j, n), and a key without its species is the plain key.
#include <stdint.h>
#include <stdio.h>

#include <tuple>
#include <vector>

#define __host__
#define __device__
#include "../../paper_2303_12980_amd/csrc/pair_key.h"

using namespace gmp;

int main() {
  const int64_t top = 0x7ffffff0LL;  // atoms a batch may hold
  std::vector<int64_t> atoms;
  for (int b = 0; b <= 31; ++b)
    for (int64_t j : {((int64_t)1 << b) - 1, (int64_t)1 << b, ((int64_t)1 << b) + 1})
      if (j < top) atoms.push_back(j);
  atoms.push_back(top - 1);
  int bad = 0;
  for (int species = 0; species < 2; ++species) {
    using Fields = std::tuple<int, int, int64_t, int, int, int>;
    std::vector<std::pair<Fields, uint64_t>> all;
    for (int64_t j : atoms) {
      if (species && j >= kKeySpeciesAtoms) continue;
      for (int sh : {0, 7, 15})
        for (int e : {0, 1, 63}) {
          if (!species && e) continue;
          for (int n1 : {-126, 0, 126})
            for (int n3 : {-126, -1, 126}) {
              const uint64_t plain = make_key(j, n1, -n1, n3, sh);
              const uint64_t k = plain | (species ? (uint64_t)e << kKeySpecies : 0);
              const int64_t back = species ? key_atom_below_species(k) : key_atom(k);
              if (back != j || key_shell(k) != sh || key_shift(k, 0) != n1 || key_shift(k, 1) != -n1 ||
                  key_shift(k, 2) != n3 || (species && key_species(k) != e) || key_atom(plain) != j ||
                  (species && (k & ~kKeySpeciesMask) != plain)) {
                if (bad++ < 5) printf("j %lld shell %d species %d: wrong fields\n", (long long)j, sh, e);
              }
              all.push_back({Fields(sh, e, j, n1, -n1, n3), k});
            }
        }
    }
    for (size_t a = 0; a < all.size(); a += 7)
      for (size_t b = 0; b < all.size(); ++b)
        if ((all[a].first < all[b].first) != (all[a].second < all[b].second) && bad++ < 5)
          printf("order of %zu and %zu\n", a, b);
  }
  return bad ? 1 : 0;
}
