// Packed key of a pair: (shell, j, n), the order of a bucket's entries and what
// the reverse-index search compares.
//   bits 60-63 shell, 24-54 atom index j, 16-23, 8-15, 0-7 image shifts + 128
// (atom indices stay below 2^31, image shifts within -126..126, shells below 16).
// While a list of up to 2^30 atoms is sorted, j ends at bit 53 and the species
// takes bits 54-59: the keys of a list then grow from bucket to bucket, and the
// species need not be looked up.  Larger batches sort without it.
#pragma once

#include <stdint.h>

namespace gmp {

constexpr int kKeyAtom = 24, kKeySpecies = 54, kKeyShell = 60;
constexpr uint64_t kKeySpeciesMask = (uint64_t)63 << kKeySpecies;
constexpr int64_t kKeySpeciesAtoms = (int64_t)1 << (kKeySpecies - kKeyAtom);

__host__ __device__ inline uint64_t make_key(int64_t j, int n1, int n2, int n3, int shell = 0) {
  return ((uint64_t)shell << kKeyShell) | ((uint64_t)j << kKeyAtom) | ((uint64_t)(n1 + 128) << 16) |
         ((uint64_t)(n2 + 128) << 8) | (uint64_t)(n3 + 128);
}
__host__ __device__ inline int key_shell(uint64_t key) { return (int)(key >> kKeyShell); }
__host__ __device__ inline int key_species(uint64_t key) { return (int)(key >> kKeySpecies) & 63; }
// the atom index of a key without and with the species beside it
__host__ __device__ inline int64_t key_atom(uint64_t key) { return (int64_t)(key >> kKeyAtom) & 0x7fffffff; }
__host__ __device__ inline int64_t key_atom_below_species(uint64_t key) {
  return (int64_t)(key >> kKeyAtom) & (kKeySpeciesAtoms - 1);
}
// image shift along axis 0, 1 or 2
__host__ __device__ inline int key_shift(uint64_t key, int axis) { return (int)(key >> (16 - 8 * axis) & 0xff) - 128; }

}  // namespace gmp
