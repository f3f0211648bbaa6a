// Tiles of the moment step where solid cells exist (host code, plain C++).
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

namespace tlbk {

// Rows y0 .. y1 - 1 of one strip. `linked`: some stored node has a solid link
// other than those of the flat walls.
struct MomentTile {
  int strip, y0, y1, linked;
};

struct MomentTileRule {
  int lx, ly, strips, strip;        // lattice; strips of `strip` stored columns
  int rows;                         // chunk height of the launch
  bool fixed;                       // the caller's: not to be changed
  long long slots, simds;           // wavefronts the chunks are cut for; SIMDs
  uint16_t from_below, from_above;  // masks of the flat walls' links
};

// Rows more than its own that a tile costs (two of equilibria, four of psi),
// and the cost of a linked row in plain ones (measured on lattices full of
// posts: 1.25 FP32, 1.4 FP64, 1.85 FP16 storage).
constexpr int kTileHalo = 3;
constexpr double kLinkedRow = 1.5;
// Height of plain tiles where the tiles do not all fit in the slots at once and
// are taken up as others end. Per step of 4096 x 2048, tiles of 12 / 24 / 48 /
// 100 rows: posts over the lower third FP32 178 / 172 / 195 / 242 us, FP64 269 /
// 257 / 272 / 315, FP16 208 / 205 / 222 / 287; single nodes one in 2000 FP32 166
// / 168 / 180 / 210; large discs FP32 181 / 173 / 190 / 241.
constexpr int kQueuedRows = 24;

// A row of a strip is linked where a stored node's mask is not the flat walls'
// one; runs of linked rows (with gaps of up to three others) are cut into tiles
// of half the chunk height (at most 8 rows: a linked row takes longer). The
// other runs are cut into tiles of the chunk height, or, where that makes more
// tiles than slots, of the height at which all are resident at once, unless
// that leaves tiles so tall that the last of them run alone: then of
// kQueuedRows. (Posts over the lower third, 4096 x 2048, FP32: 2027 us a step
// in tiles of a run each, 158 in queued ones; over the lower tenth 232 resident
// at 270 rows, 140 queued. Posts along the bottom wall stay resident, 79 rows
// each: FP32 / FP64 / FP16 119 / 176 / 124 us, queued 115 / 181 / 124.)
inline std::vector<MomentTile> moment_tiles(const MomentTileRule& r, const uint16_t* link,
                                            int* nlinked) {
  std::vector<MomentTile> linked, plain;
  auto cut = [](std::vector<MomentTile>& to, int strip, int y0, int y1, int most, int flag) {
    const int n = (y1 - y0 + most - 1) / most;
    for (int k = 0; k < n; ++k)
      to.push_back({strip, y0 + (int)((long long)(y1 - y0) * k / n),
                    y0 + (int)((long long)(y1 - y0) * (k + 1) / n), flag});
  };
  std::vector<MomentTile> runs;  // of rows without links
  std::vector<char> marked((size_t)r.ly);
  for (int s = 0; s < r.strips; ++s) {
    const int x0 = s * r.strip, x1 = std::min(x0 + r.strip, r.lx);
    for (int y = 0; y < r.ly; ++y) {
      const uint16_t flat = (y == 0 ? r.from_below : 0u) | (y == r.ly - 1 ? r.from_above : 0u);
      const uint16_t* row = link + (size_t)y * r.lx;
      uint16_t other = 0;
      for (int x = x0; x < x1; ++x) other |= row[x] ^ flat;
      marked[y] = other != 0;
    }
    for (int y = 0; y < r.ly;) {
      int e = y;
      if (marked[y]) {
        for (int k = y; k < r.ly && k < e + 4; ++k)
          if (marked[k]) e = k + 1;
        cut(linked, s, y, e, std::min(8, std::max(1, r.rows / 2)), 1);
      } else {
        while (e < r.ly && !marked[e]) ++e;
        runs.push_back({s, y, e, 0});
      }
      y = e;
    }
  }
  int rows = r.rows;
  auto count = [&](int h) {
    long long n = 0;
    for (const auto& t : runs) n += (t.y1 - t.y0 + h - 1) / h;
    return n;
  };
  const long long room = r.slots - (long long)linked.size();
  if (!r.fixed && count(rows) > room) {
    const int queued = std::min(rows, kQueuedRows);
    int tall = rows;  // the longest run
    for (const auto& t : runs) tall = std::max(tall, t.y1 - t.y0);
    if (count(tall) > room) {
      rows = queued;
    } else {
      int lo = rows;  // the lowest height at which all fit lies in (lo, tall]
      while (lo + 1 < tall) {
        const int mid = lo + (tall - lo) / 2;
        (count(mid) > room ? lo : tall) = mid;
      }
      // time of either in rows that a SIMD marches: its share of all rows, at
      // least the tallest tile; queued, about half a tile more at the end
      double work = 0;
      for (const auto& t : linked) work += kLinkedRow * (t.y1 - t.y0 + kTileHalo);
      for (const auto& t : runs) work += t.y1 - t.y0;
      auto share = [&](int h) { return (work + (double)kTileHalo * count(h)) / r.simds; };
      rows = std::max(share(tall), (double)tall + kTileHalo) <= share(queued) + 0.5 * queued ? tall : queued;
    }
  }
  for (const auto& t : runs) cut(plain, t.strip, t.y0, t.y1, rows, 0);
  // strip fastest: neighbouring strips at the same height run together
  auto lower = [](const MomentTile& u, const MomentTile& v) { return u.y0 < v.y0; };
  std::stable_sort(plain.begin(), plain.end(), lower);
  std::stable_sort(linked.begin(), linked.end(), lower);
  *nlinked = (int)linked.size();
  linked.insert(linked.end(), plain.begin(), plain.end());
  return linked;
}

}  // namespace tlbk
