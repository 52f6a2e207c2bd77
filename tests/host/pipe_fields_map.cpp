// Host check of the stores of the pipelined W4A4 kernel (pipe_stage.h) for activations in field form, 8 bytes a thread: every byte
// that a wave reads of the 4-bit part has exactly one writer and is the byte of the FP6 dword that the reader expects.
#include <cstdio>
#include <vector>

#include "pipe_stage.h"

using namespace dirotq::pipe;

static int failures = 0;

template <int GS>
static void check(bool copy) {
  constexpr int ROWS = 128, FIRST = 256;               // the token rows behind the weights'
  std::vector<int> tag((FIRST + ROWS) * SB, -1), writers((FIRST + ROWS) * SB, 0);
  // content in dwords of a row half: 0..5 the expanded ones, 10..13 the copied ones, 20 anything
  auto put = [&](int row, int at, std::vector<int> dwords) {
    for (size_t i = 0; i < dwords.size() * 4; i++) {
      const int b = at + (int)i;
      if (b < row * SB || b >= (row + 1) * SB) { failures++; continue; }
      writers[b]++;
      tag[b] = dwords[i / 4] * 4 + (int)i % 4;
    }
  };
  for (int row = FIRST; row < FIRST + ROWS; row++)
    for (int half = 0; half < 2; half++)
      for (int part = 0; part < 2; part++) {
        const RowPart p = row_part<GS>(row, half);
        const Stores s = narrow_fields_stores<GS>(p, part, copy);
        const int h = half * 100;
        std::vector<int> raw = {h + 10 + 2 * part, h + 11 + 2 * part};
        if (GS == 32) {
          put(row, s.first, copy ? raw : part ? std::vector<int>{h + 3, h + 4} : std::vector<int>{h, h + 1});
          put(row, s.second, copy ? std::vector<int>{h + 20, h + 20} : part ? std::vector<int>{h + 2, h + 20} : std::vector<int>{h + 5, h + 20});
        } else {
          put(row, s.first, copy ? raw : part ? std::vector<int>{h + 2, h + 3} : std::vector<int>{h, h + 1});
          put(row, s.second, {copy ? h + 20 : part ? h + 4 : h + 5});
        }
      }
  auto expect = [&](int at, int dwords, int first) {
    for (int i = 0; i < 4 * dwords; i++)
      if (writers[at + i] != 1 || tag[at + i] != first * 4 + i) {
        if (failures++ < 20) std::printf("GS=%d copy=%d byte %d of row %d: %d writers, holds %d, wanted %d\n", GS, copy, (at + i) % SB, at / SB, writers[at + i], tag[at + i], first * 4 + i);
      }
  };
  for (int row = FIRST; row < FIRST + ROWS; row++)
    for (int h = 0; h < 2; h++) {
      const int lo = read_lo<GS>(row, h), hi = read_hi<GS>(row, h);
      if (copy) {
        if (GS == 32) expect(lo, 4, 100 * h + 10);
        else expect(lo, 4, 100 * h + 10);
      } else if (GS == 32) {                           // half h of group 0, then of group 1: three dwords of row half 0, 1
        expect(lo, 3, 3 * h), expect(hi, 3, 100 + 3 * h);
      } else {
        expect(lo, 4, 100 * h), expect(hi, 2, 100 * h + 4);
      }
    }
}

int main() {
  for (int copy = 0; copy < 2; copy++) check<32>(copy), check<64>(copy), check<128>(copy);
  std::printf("%d failure(s)\n", failures);
  return failures != 0;
}
