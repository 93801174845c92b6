// ploc.h -- what the host makes of a group of clustering rounds (no HIP: the
// CPU tests compile it by itself).
#pragma once

// clusters that one block takes to the end (k_ploc_tail)
#define PLOC_TAIL 1024

enum PlocStep { PLOC_DONE, PLOC_MORE, PLOC_STALLED };

// A group of rounds and the tail block after it began with `before` clusters
// and left `clusters` and the next internal node `next`.  Every merge takes
// one cluster and one node.  The tail block runs for any count up to
// PLOC_TAIL and keeps its merges in LDS, so a count of 2 to PLOC_TAIL means
// that it met a round without a merge (boxes whose merged areas are not
// finite), and that the clusters in memory are older than the count: another
// group would merge them again into nodes that are taken.
inline PlocStep ploc_step(int before, int clusters, int next) {
  if (clusters < 1 || clusters >= before || next != clusters - 2) return PLOC_STALLED;
  if (clusters == 1) return PLOC_DONE;
  return clusters <= PLOC_TAIL ? PLOC_STALLED : PLOC_MORE;
}
