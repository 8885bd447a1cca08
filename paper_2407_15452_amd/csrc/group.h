// Grouping of records by rows (group.hip).
#pragma once

#include "common.h"

namespace gs {

constexpr uint32_t kNoGroupRow = 0xffffffffu;  // (rows are below 2^31)
// device counters: pieces of split buckets, rows of split buckets, long rows, records of both kinds
enum : int { kGroupPieces, kGroupSplitRows, kGroupLong, kGroupRecords, kGroupCounters };

struct GroupArgs {
  // records of the first kind (rows below 2^31) and the list of rows of the second kind (-1: no record)
  const uint32_t* rows;
  const uint2* vals;
  int64_t n;
  const int32_t* second;
  int64_t second_n;
  uint32_t second_word;          // a record of the second kind: (place in the list, this)
  uint32_t second_key;           // key of its row 0; a row of the first kind is its own key
  uint32_t* rows_mid;            // [n + second_n] in between
  uint2* vals_mid;
  uint32_t* keys_out;            // the result, in ascending order of the keys: counters[kGroupRecords] records, the
  uint2* vals_out;               // first n of the first kind
  // rows of more than 2^seg_shift records: their slots of `dim` numbers, (position of the row's first record) >> seg_shift, are set to 0 and
  // (key, slot) goes to long_rows, in any order
  int32_t seg_shift;
  int32_t dim;
  long long* long_acc;           // [((n + second_n) >> seg_shift) + 1][dim]
  // taken from the caller's memory by group_take
  uint2* long_rows;
  uint2* further;                // [((n + second_n) >> seg_shift) + 2] entry w: the one position of [w << seg_shift, (w + 1) << seg_shift) at which a
                                 // segment of a row other than its first starts, and the row's first position; else kNoGroupRow
  uint32_t* counters;            // [kGroupCounters]
  uint8_t* named;                // null, or marks: entry r is 1 if row r of the first kind has a record, entry second_named + r
  uint32_t second_named;         // the same of the second kind
  uint32_t* counts;              // [tiles][buckets] of one kind, then of the other
  uint32_t *totals, *starts;     // [digits] records of a bucket, and the first of them
  uint4* pieces;                 // of the buckets to split: bucket, place of its rows in the next two, piece, pieces of the bucket
  uint32_t* row_counts;          // of the rows of the buckets to split: their records, and
  uint32_t* row_taken;           // those that pieces have taken places for
  uint32_t digits;               // buckets of both kinds
  // set by group_rows
  int row_bits, second_row_bits;
  uint32_t buckets;              // of the first kind
  uint32_t most;                 // records that one workgroup takes
  uint32_t first_scans;          // workgroups of the prefix sums for the first kind
  int64_t first_tiles, tiles, tiles_per_xcd;
};

bool can_group(int64_t rows);
bool group_crowded(int64_t n, int64_t rows);                              // whether sorting is faster, since most buckets are split
constexpr int kBucketRowBits = 14;             // rows of a bucket: their counters fit a workgroup's LDS
int64_t group_border(int64_t rows, bool second, int bits);
void group_take(GroupArgs& a, Carver& cv, int64_t n, int64_t second_n, int64_t rows, int32_t seg_shift, bool marks);
int32_t group_rows(GroupArgs a, int64_t rows, hipStream_t stream);       // n >= 1, n + second_n < 2^32

}  // namespace gs
