// Host check of the LDS stage layout of the pipelined W4A4 kernel (pipe_stage.h): over all threads of a workgroup, every
// byte that a wave reads has exactly one writer, it carries what the reader expects, and the stores stay inside their row.
#include <cstdio>
#include <cstring>
#include <vector>

#include "pipe_stage.h"

using namespace dirotq::pipe;

static int failures = 0;

// what a byte holds: 0 = never written, else a tag of its content; writers counted
struct Byte {
  int tag = 0, writers = 0;
};

constexpr int JUNK = -1;

// copied byte b (0..31) of a row; expanded byte d (0..47) of a row: 12 per 16-channel part, parts in channel order
static int copied(int b) { return 1000 + b; }
static int expanded(int d) { return 2000 + d; }

template <int GS>
static void check(bool narrow, bool copy) {
  constexpr int ROWS = 512;
  std::vector<Byte> lds(ROWS * SB);
  auto put = [&](int row, int at, const std::vector<int>& tags) {
    if (at < row * SB || at + (int)tags.size() > (row + 1) * SB) failures++, std::printf("store outside its row\n");
    for (size_t i = 0; i < tags.size(); i++) {
      Byte& b = lds[at + i];
      b.writers++;
      b.tag = tags[i];
    }
  };
  auto bytes = [&](bool is_copy, int first, int n) {   // n tags from `first` on
    std::vector<int> v(n);
    for (int i = 0; i < n; i++) v[i] = is_copy ? copied(first + i) : expanded(first + i);
    return v;
  };
  auto junk = [](int n) { return std::vector<int>(n, JUNK); };
  auto padded = [](std::vector<int> v) {               // 12 bytes and a zero dword (any value: the operand's unused end)
    v.resize(16, JUNK);
    return v;
  };
  auto cat = [](std::vector<int> a, const std::vector<int>& b) {
    a.insert(a.end(), b.begin(), b.end());
    return a;
  };
  for (int row = 0; row < ROWS; row++)
    for (int half = 0; half < 2; half++) {
      const RowPart p = row_part<GS>(row, half);
      const int e = 24 * half, c = 16 * half;          // first expanded / copied byte of the row half
      if (!narrow) {
        const Stores s = wide_stores<GS>(p, copy);
        if (GS == 32) {
          put(row, s.second, copy ? junk(16) : padded(bytes(false, e + 12, 12)));
          put(row, s.first, copy ? bytes(true, c, 16) : padded(bytes(false, e, 12)));
        } else {
          put(row, s.first, copy ? bytes(true, c, 16) : bytes(false, e, 16));
          put(row, s.second, copy ? junk(8) : bytes(false, e + 16, 8));
        }
        continue;
      }
      for (int part = 0; part < 2; part++) {
        const Stores s = narrow_stores<GS>(p, part, copy);
        const std::vector<int> d = bytes(false, e + 12 * part, 12);
        if (GS == 32) {
          put(row, s.first, copy ? bytes(true, c + 8 * part, 8) : std::vector<int>(d.begin(), d.begin() + 8));
          put(row, s.second, copy ? junk(8) : cat(std::vector<int>(d.begin() + 8, d.end()), junk(4)));
        } else {                                       // part 0: dwords 0 1 and 2; part 1: dwords 1 2 and 0
          put(row, s.second, copy ? junk(4) : part ? std::vector<int>(d.begin(), d.begin() + 4) : std::vector<int>(d.begin() + 8, d.end()));
          put(row, s.first, copy ? bytes(true, c + 8 * part, 8) : part ? std::vector<int>(d.begin() + 4, d.end()) : std::vector<int>(d.begin(), d.begin() + 8));
        }
      }
    }
  auto expect = [&](int at, int tag) {
    const Byte& b = lds[at];
    if (b.writers != 1 || (tag && b.tag != tag)) {
      if (failures++ < 20)
        std::printf("GS=%d narrow=%d copy=%d byte %d of row %d: %d writers, holds %d, wanted %d\n", GS, narrow, copy, at % SB, at / SB, b.writers, b.tag, tag);
    }
  };
  for (int row = 0; row < ROWS; row++)
    for (int h = 0; h < 2; h++) {
      const int lo = read_lo<GS>(row, h), hi = read_hi<GS>(row, h);
      if (copy) {                                      // k-half h of the bf16 operand
        for (int i = 0; i < 16; i++) expect(lo + i, copied(16 * h + i));
      } else if (GS == 32) {                           // group 0 then group 1: k-half h of each
        for (int i = 0; i < 12; i++) expect(lo + i, expanded(12 * h + i)), expect(hi + i, expanded(24 + 12 * h + i));
      } else {
        for (int i = 0; i < 16; i++) expect(lo + i, expanded(24 * h + i));
        for (int i = 0; i < 8; i++) expect(hi + i, expanded(24 * h + 16 + i));
      }
    }
}

int main() {
  for (int narrow = 0; narrow < 2; narrow++)
    for (int copy = 0; copy < 2; copy++) check<32>(narrow, copy), check<64>(narrow, copy), check<128>(narrow, copy);
  std::printf("%d failure(s)\n", failures);
  return failures != 0;
}
