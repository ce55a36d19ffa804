// Work lists of the certified key-to-anchor assignment (assign.hip), shared by
// the kernels and the host-side stage sequencing.  All pointers are device
// arrays for one chunk of P pairs.
#pragma once
#include <stdint.h>

namespace arckv {

constexpr int kAssignStats = 8;

// Pool survivors per float64-pass entry: a key and 31 candidates fill one
// batch of 32 vectors.  A key with more pool survivors is queued as several
// entries, so its batches can run on different workgroups.
constexpr int kPassDSplit = 31;

// Entries for at most Tp queued keys whose pool candidates number at most
// pool_per_key * Tp: one per key, plus one per kPassDSplit candidates of a
// split key.
inline int64_t pass_d_capacity(int64_t Tp, int64_t pool_per_key) {
  return Tp + (pool_per_key * Tp + kPassDSplit - 1) / kPassDSplit + 1;
}

// Query ranges into which a work item of the refine and of the float64 pass is
// cut, by the numbers of queries and keys, so that decisions do not depend on how
// many pairs run together: a pair of few keys has a few dozen items, each a serial
// sweep over its queries, on 256 CUs.  More than four cost more in setting the items
// up than they gain, and a pair of many keys has items enough for two: both passes with
// 1, 2 and 4 ranges, in us: T = 8192, n = 4096, 8 pairs 455, 264, 177, 128 pairs 3349, 2182,
// 1732; T = 15001, n = 3000, 8 pairs 379, 236, 239; T = 16384, n = 2100, 32 pairs 732, 676,
// 762; T = 32768, n = 4096, 16 pairs 1016, 1034, 1104, 64 pairs 3723, 3660, 3922.
inline int query_ranges(int64_t n, int64_t T) {
  const int64_t tiles = (n + 127) / 128;
  return tiles >= 16 && T < 16384 ? 4 : tiles >= 2 ? 2 : 1;
}

struct AssignLists {
  int32_t *fcnt;    // [P] keys queued for the refine pass
  int32_t *fkey;    // [P][cap]
  int32_t *foff;    // [P][cap] first candidate of the queued key in the pool
  int32_t *fn;      // [P][cap] its number of candidates
  // [P] candidates of all queued keys, in the pool or not: up to T t, which 32 bits do not hold (a count
  // that wraps gives out places in the pool twice)
  unsigned long long *pcnt;
  int32_t *pool;    // [P][pcap] candidate anchors, contiguous per queued key
  double *psim;     // [P][2 nspl][pcap]: the first nspl arrays the parts of their refined similarities, then
                    // (float64 pass) array 2 i the part i of a candidate's dot product, 2 i + 1 of its
                    // squared norm
  int64_t pcap;     // pool capacity per pair
  int32_t nspl;     // query ranges (query_ranges)
  int32_t *dcnt;    // [P] entries queued for the float64 pass (a key with many pool survivors is split
                    // into several entries of consecutive survivors)
  int32_t *dkey;    // [P][dcap] the entry's key
  int32_t *dn;      // [P][dcap] candidates of the entry
  int32_t *doff;    // [P][dcap] its first candidate in the pool (-1: all t anchors)
  int32_t *stats;   // [P][kAssignStats] (assign.hip): flagged after the first pass, sent to the float64
                    // pass, candidates of the flagged keys, undecided (sum of the next two), undecided
                    // in the first pass, undecided in the refine pass (kept at 0: survivors of any
                    // number go to the float64 pass), sent to the refine pass, keys whose pass-A
                    // candidates include a whole anchor tile
  int64_t cap;      // key capacity per pair
  int32_t *goff;    // [P][gcap] pass C work items: first (group of 64 queued keys, candidate chunk) item of each
                    // group, then the pair's item count
  int64_t gcap;     // >= cap / 64 + 1
  int32_t *dgrp;    // [P][dcap] first entry of the entry's key when the key is split, else -1
  int32_t *dgn;     // [P][dcap] entries of the entry's key
  int32_t *ditem;   // [P][dcap + 2] pass D work items: count, first entry of each item, then dcnt
  int64_t dcap;     // entry capacity per pair
};

}  // namespace arckv
