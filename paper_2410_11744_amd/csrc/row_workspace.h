// The greedy builder's workspace, per row (kRowSumDoubles doubles): the totals of kSums runs of kRun tokens, the row maximum
// (already divided by the temperature), from kDrawnOffset on the tokens drawn at this position, two bytes each in the
// order of the draws (their weights are no longer in the totals), at kMadeOffset a draw made but not asked for, at kMailOffset a mailbox.
// Host code as well as device code.
#pragma once
#include <stddef.h>

#include "../../include/dyspec.h"

namespace dyspec {

constexpr int kRun = 128;
constexpr int kSums = DYSPEC_MAX_VOCAB / kRun;
constexpr int kRowSumDoubles = 24 + DYSPEC_MAX_VOCAB / 64;
constexpr int kDrawnOffset = kSums + 2;
// A node's draws have ranks up to DYSPEC_MAX_BUILD_NODES: each of the tree's other rows may be a child, the last pop asks for the
// draw after the last child's, and the one after that is made ahead.
constexpr int kDrawnEntries = DYSPEC_MAX_BUILD_NODES + 1;
constexpr int kMadeOffset = kDrawnOffset + (kDrawnEntries + 3) / 4;
constexpr int kMadeDoubles = 3;
// Draws of a node made by another workgroup (helper): a mailbox in the row of the helper's number, and a ring, 16 bytes a draw, from the back
// of the tree: a node's children are later rows, so that one of the last rows has hardly a draw, and the places of its tokens of ranks
// kMailRanks and on are free.  (In the node's own row they are not: a helper may come when the node's wave is past those ranks.)
constexpr int kMailOffset = kMadeOffset + kMadeDoubles;
constexpr int kMailDoubles = 3;
constexpr int kMailRing = 64;
constexpr int kMailRanks = 512;
constexpr int kMailRingOffset = kDrawnOffset + kMailRanks / 4;
static_assert(kRowSumDoubles >= kMailOffset + kMailDoubles, "room for every draw of a row, one that is put aside, and a mailbox");
static_assert(kMailRingOffset + 2 * kMailRing <= kMadeOffset && kMailRingOffset % 2 == 0 && kRowSumDoubles % 2 == 0, "16-byte entries among the drawn tokens");

__host__ __device__ inline double* ws_totals(double* ws, int row) { return ws + (size_t)row * kRowSumDoubles; }
__host__ __device__ inline double* ws_rowmax(double* ws, int row) { return ws_totals(ws, row) + kSums; }
__host__ __device__ inline unsigned short* ws_drawn(double* ws, int row) { return reinterpret_cast<unsigned short*>(ws_totals(ws, row) + kDrawnOffset); }
__host__ __device__ inline double* ws_made(double* ws, int row) { return ws_totals(ws, row) + kMadeOffset; }
__host__ __device__ inline double* ws_mail(double* ws, int row) { return ws_totals(ws, row) + kMailOffset; }
// of helper k of the tree whose N rows begin at `base`
__host__ __device__ inline double* ws_mail_ring(double* ws, int base, int N, int k) { return ws_totals(ws, base + N - 1 - k) + kMailRingOffset; }

}  // namespace dyspec
