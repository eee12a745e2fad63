// Lists of runs as they lie in memory (ft_pieces.h: find_base, pack_pieces), read back as the kernels read them: a tile's block by
// the first tiles of the blocks, its piece by the tiles of the block's pieces. Every first and last tile of a piece must find it.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../paper_2411_01830_amd/csrc/ft_pieces.h"

using namespace ft;

#define CHECK(x)                                             \
  do {                                                       \
    if (!(x)) {                                              \
      std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x);    \
      return 1;                                              \
    }                                                        \
  } while (0)

static uint64_t g_state = 1;
static uint64_t rnd(uint64_t n) {
  g_state = g_state * 6364136223846793005ull + 1442695040888963407ull;
  return (g_state >> 17) % n;
}

static int one(uint32_t n, uint64_t reach, uint32_t tile, bool by_source, bool close) {
  std::vector<PieceSides> at(n);
  std::vector<uint32_t> first(n), len(n);
  PieceTables t;
  t.at = at.data();
  t.first = first.data();
  t.len = len.data();
  t.n = n;
  t.tile = tile;
  for (uint32_t i = 0; i < n; ++i) {
    at[i] = PieceSides{(1ull << 40) + rnd(reach), (3ull << 40) + rnd(reach)};
    if (i + 1 == n) at[i] = PieceSides{(1ull << 40) + reach, 3ull << 40};
    if (i == 0) at[i] = PieceSides{1ull << 40, (3ull << 40) + reach};
    const uint64_t most[] = {1, 16, 130, tile, 3 * tile, 1u << 20};
    len[i] = 1 + (uint32_t)rnd(most[rnd(6)]);
    first[i] = t.ntiles;
    t.ntiles += run_tiles(by_source ? at[i].src : at[i].dst, len[i], tile);
  }
  find_base(&t);
  CHECK(t.close == close);
  std::vector<char> packed(packed_bytes(t) + 1, 0x5a);
  pack_pieces(t, packed.data());
  CHECK(packed.back() == 0x5a);
  const uint32_t *words = reinterpret_cast<const uint32_t *>(packed.data());
  for (uint32_t i = 0; i < n; ++i) {
    const uint32_t last = (i + 1 < n ? first[i + 1] : t.ntiles) - 1;
    for (uint32_t tile_no : {first[i], last}) {
      uint32_t b = 0;
      while ((b + 1) * kPieceBlock < n && first[(b + 1) * kPieceBlock] <= tile_no) ++b;
      uint32_t begins = first[b * kPieceBlock], x = ~0u, its = 0;
      PieceSides s{};
      uint32_t bytes = 0;
      for (uint32_t j = b * kPieceBlock; j < n && j < (b + 1) * kPieceBlock && begins <= tile_no; ++j) {
        if (t.close) {
          s = PieceSides{t.src0 + words[j], t.dst0 + words[n + j]};
          bytes = words[2 * n + j];
        } else {
          std::memcpy(&s, packed.data() + j * sizeof(PieceSides), sizeof(s));
          std::memcpy(&bytes, packed.data() + n * sizeof(PieceSides) + j * 4, 4);
        }
        x = j;
        its = begins;
        begins += run_tiles(by_source ? s.src : s.dst, bytes, tile);
      }
      CHECK(x == i && its == first[i] && s.src == at[i].src && s.dst == at[i].dst && bytes == len[i]);
    }
  }
  return 0;
}

int main() {
  for (uint32_t n : {1u, 2u, 63u, 64u, 65u, 241u, 1024u, 1025u, 4096u, 4097u, 16384u})
    for (uint32_t tile : {1024u, 8192u, 16384u})
      for (bool by_source : {false, true}) {
        if (one(n, (1ull << 31) - 1, tile, by_source, true)) return 1;
        if (n > 1 && one(n, (1ull << 31) + 1, tile, by_source, false)) return 1;
        if (n > 1 && one(n, 1ull << 38, tile, by_source, false)) return 1;
      }
  std::printf("done\n");
  return 0;
}
