// Which workgroup a block of a launch takes, for the 8 XCDs that receive blocks
// in turn, and the launches' grids.  -1: none.
#pragma once

#include <cstdint>

#include "mf_internal.hpp"

namespace mf {
namespace wave {

// Each XCD works through one contiguous chunk of the natural order:
// neighbouring strips then share that XCD's L2.
MF_HD int xcd_wg_at(int block, int nwg) {
  const int chunk = (nwg + kXCD - 1) / kXCD;
  const int k = block % kXCD, j = block / kXCD;
  if (j >= chunk) return -1;
  const int n = k * chunk + j;
  return n < nwg ? n : -1;
}
MF_HD int xcd_grid(int nwg) { return kXCD * ((nwg + kXCD - 1) / kXCD); }

// The same for launches of at least `from` workgroups with runs of 2^shift
// consecutive workgroups dealt to the XCDs in turn: neighbours still share an
// L2, and the launch as a whole moves through memory in one front instead of
// eight.  Smaller launches (whose data the caches hold) keep one chunk per XCD.
struct XcdRuns {
  int from, shift;
};
constexpr XcdRuns kNoRuns{0x7fffffff, 0};
MF_HD int xcd_wg_at(int block, int nwg, XcdRuns r) {
  if (nwg < r.from) return xcd_wg_at(block, nwg);
  const int k = block % kXCD, j = block / kXCD;
  const int n = (((j >> r.shift) * kXCD + k) << r.shift) + (j & ((1 << r.shift) - 1));
  return n < nwg ? n : -1;
}
inline int xcd_grid_runs(int nwg, XcdRuns r) {
  if (nwg < r.from) return xcd_grid(nwg);
  const int per = kXCD << r.shift;
  return (nwg + per - 1) / per * per;
}

// The same, and in smaller launches the first `lead` workgroups and the next
// `lead2` in chunks of their own.  They hold tiles of other kinds (copies of shared
// DoFs, other boundary points) that take longer than the walk's; at the head of the
// first chunk they all fall to one XCD (512 triangles at level 6: FP64 apply 10.2
// us, 14.9 so; P2 10.4 and 23; 32 at level 9, two FP32 sweeps 32.4 and 38.5).  Up
// to kLeadMin of them, one for each CU of that XCD, stay there, and so do up to one
// in kLeadShare (a fifth of the chunk): they share their CUs with fewer others than
// anywhere else (two triangles at level 11, eight of them: FP32 P2 9.8 us, 11.4 dealt
// out; 13 at level 10, 48 of 2,100: 13.6 and 15.2).
constexpr int kLeadMin = 32, kLeadShare = 40;
// In larger launches, where runs deal them out, leading workgroups of one in
// kLeadSpread or more are spread evenly among the others: the lines they share with
// the walk are then in the caches (3,200 triangles at level 7, 4.9 %, FP64 apply 168 ->
// 149 us, two sweeps 490 -> 445; 32 at level 10, 1.7 %, apply 51.0 -> 52.0).  Not with
// a second kind (P2, 512 triangles at level 7, FP32 16.8 -> 19.1).
constexpr int kLeadSpread = 24;
MF_HD int xcd_spread(int p, int nwg, int lead) {
  const int before = (int)((int64_t)p * lead / nwg), upto = (int)((int64_t)(p + 1) * lead / nwg);
  return upto > before ? before : lead + p - before;
}
MF_HD int xcd_head(int nwg, int lead) {
  return lead > kLeadMin && (int64_t)lead * kLeadShare > nwg ? kXCD * ((lead + kXCD - 1) / kXCD) : 0;
}
MF_HD int xcd_wg_at(int block, int nwg, int lead, int lead2, XcdRuns r) {
  // Few of them stay where they are under every rule (runs start at more than
  // kLeadMin * kLeadSpread workgroups).  Asked first: 0.1 us of the smallest P2 applies.
  if (lead <= kLeadMin && lead2 <= kLeadMin) return xcd_wg_at(block, nwg, r);
  if (nwg >= r.from) {
    const int p = xcd_wg_at(block, nwg, r);
    return p < 0 || lead2 > 0 || (int64_t)lead * kLeadSpread < nwg ? p : xcd_spread(p, nwg, lead);
  }
  int first = 0;
  for (int l : {lead, lead2}) {
    const int head = xcd_head(nwg, l);
    if (block < head) {
      const int n = xcd_wg_at(block, l);
      return n < 0 ? -1 : first + n;
    }
    block -= head;
    if (head > 0) first += l;
    else if (l > 0) break;  // (it stays before what follows)
  }
  const int n = xcd_wg_at(block, nwg - first);
  return n < 0 ? -1 : first + n;
}
inline int xcd_grid(int nwg, int lead, int lead2, XcdRuns r) {
  if (nwg >= r.from) return xcd_grid_runs(nwg, r);
  const int h = xcd_head(nwg, lead), h2 = lead == 0 || h > 0 ? xcd_head(nwg, lead2) : 0;
  return h + h2 + xcd_grid(nwg - (h > 0 ? lead : 0) - (h2 > 0 ? lead2 : 0));
}

// Dynamic LDS (unused) that lets at most n workgroups of a kernel with `own` bytes
// of LDS share a CU, in launches of at least `from` workgroups: fewer waves at once
// keep the front of a launch that streams from memory compact, which the memory
// rewards more than further loads in flight.  n workgroups and a half would fill
// the CU, so that the steps LDS is granted in do not matter (up to n = 8).
constexpr int kLdsPerCu = 160 * 1024, kLdsStep = 1280;
inline int lds_cap(int nwg, int from, int n, int own) {
  const int bytes = 2 * kLdsPerCu / (2 * n + 1);
  return nwg < from || n <= 0 || own >= bytes ? 0 : bytes - own;
}

}  // namespace wave
}  // namespace mf
