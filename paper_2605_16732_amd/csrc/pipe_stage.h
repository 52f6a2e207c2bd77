// LDS layout of a stage of the pipelined kernel B (w4a4_gemm_pipe.hip): which bytes a thread's stores go to and which
// bytes a wave reads.  Plain constexpr functions, so that a host test can check that no byte that is read has two writers
// (the order of two lanes' stores is nothing that the source could promise).
//
// A row has 64 bytes in four chunks of 16.  A stage of the 4-bit part holds the FP6 codes of 64 channels: 24 bytes per
// row half, in chunk 2 half and in 8 bytes of chunk 2 half + 1 (groups of 32: four parts of 12 bytes, one per chunk).  A
// stage of the 16-bit branch holds 16 bf16 numbers, copied: row half in chunk 2 half (groups of 32: in chunk half).
// The kind of a stage selects addresses, not code: every thread makes the same stores for both, and on a 16-bit stage
// sends what means nothing then to a chunk that is not read.
#pragma once

namespace dirotq {
namespace pipe {

constexpr int SB = 64;                       // bytes per row and stage in LDS

// 16-B chunk c of row r sits in slot c ^ ((r >> 2) & 3): the 16 rows that a 16-byte LDS access serves per cycle
// fall into 16 different slots of a 256-byte bank line
constexpr int stage_off(int row, int chunk) { return row * SB + ((chunk ^ ((row >> 2) & 3)) << 4); }
// the chunk behind the one at `lo` (groups of 64 and 128: the 8 bytes in it, alternating within the chunks: all banks)
template <int GS>
constexpr int hi_off(int lo, int row) { return (lo ^ 16) + (GS == 32 ? 0 : 8 * ((row >> 4) & 1)); }

struct RowPart {                             // offsets of a row half: expanded (first and second store), copied
  int at, at_hi, at_copy;
};
template <int GS>
constexpr RowPart row_part(int row, int half) {
  const int at = stage_off(row, 2 * half);
  return {at, hi_off<GS>(at, row), GS == 32 ? stage_off(row, half) : at};
}

struct Stores {                              // offsets of a thread's two stores
  int first, second;
};
// 16 staged bytes (a row half).  Groups of 64 and 128: 16 bytes (codes or copy), then 8; groups of 32: 16 and 16
template <int GS>
constexpr Stores wide_stores(RowPart p, bool copy) {
  if (GS != 32) return {p.at, p.at_hi};
  return {copy ? p.at_copy : p.at, copy ? p.at_copy ^ 32 : p.at_hi};
}
// 8 staged bytes (part 0 or 1 of a row half).  Groups of 64 and 128: 8 bytes, then 4; groups of 32: 8 and 8
template <int GS>
constexpr Stores narrow_stores(RowPart p, int part, bool copy) {
  if (GS != 32) return {copy ? p.at_copy + 8 * part : part ? p.at_hi : p.at, (copy ? p.at ^ 16 : p.at) + (part ? 12 : 8)};
  const int at = copy ? p.at_copy + 8 * part : part ? p.at ^ 16 : p.at;
  return {at, copy ? (p.at_copy ^ 32) + 8 * part : at + 8};
}

// the same of the field form.  Part 0 expands to dwords 0 1 | 5 of the row half's six, part 1 to 2 3 | 4.  Groups of 64 and 128: 8
// bytes (dwords 0 1, 2 3), then 4; groups of 32: 8 (0 1, 3 4) and 8 (5 0, 2 0)
template <int GS>
constexpr Stores narrow_fields_stores(RowPart p, int part, bool copy) {
  if (GS != 32) return {p.at + 8 * part, copy ? (p.at ^ 16) + (part ? 12 : 8) : p.at_hi + (part ? 0 : 4)};
  return {copy ? p.at_copy + 8 * part : part ? p.at ^ 16 : p.at, copy ? (p.at_copy ^ 32) + 8 * part : part ? p.at + 8 : (p.at ^ 16) + 8};
}

// what lane half h reads of a row: 16 bytes, then 8 (groups of 32: 16); of a 16-bit stage only the first 16 are used
template <int GS>
constexpr int read_lo(int row, int h) { return stage_off(row, GS == 32 ? h : 2 * h); }
template <int GS>
constexpr int read_hi(int row, int h) { return GS == 32 ? stage_off(row, 2 + h) : hi_off<GS>(stage_off(row, 2 * h), row); }

}  // namespace pipe
}  // namespace dirotq
