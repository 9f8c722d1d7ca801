// Schedule of the attention pass and its merge: which key tiles of which (head, query
// tile) item each workgroup runs.  Plain C++, shared by the device code and a CPU build.
//
// The key tiles of every item, items head-major, form one range of `work` tile-steps cut
// into G contiguous shares, one per workgroup, numbered so that each XCD gets consecutive
// shares (the query tiles of a head share its K/V in that XCD's L2).  With cuts the shares
// are equal: a share covers the end of one item, whole items and the start of another, and
// an item covered by several shares is a cut item whose pieces the merge pass combines.  A
// share w holds at most two pieces of cut items: the continuation of an item begun in an
// earlier share (scratch slot 2w) and the first piece of an item that goes on into later
// shares (slot 2w + 1; when that item starts at the share's start there is no continuation
// and slot 2w stays unused).  Without cuts every share boundary is rounded up to the next
// item start.
#pragma once

#include <stdint.h>

#include "fd_rules.h"

namespace fd {

constexpr int kXcds = 8;
constexpr int kKeyTile = 64;   // keys per tile
constexpr int kMaxSchedRequests = 1024;

// Per-request prefix tables: wpre[b] = tile-steps (query tiles x key tiles, one head) of the
// requests before b, tpre[b] = their query tiles; entry B holds the totals.
struct SchedTables {
  long long wpre[kMaxSchedRequests + 1];
  int tpre[kMaxSchedRequests + 1];
};

// A wave-uniform value read from LDS, moved to a scalar register so that the loop
// bounds and branches derived from it stay scalar.
FD_RULE int uniform(int v) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_readfirstlane(v);
#else
  return v;
#endif
}
FD_RULE long long uniform(long long v) {
  const uint32_t lo = static_cast<uint32_t>(uniform(static_cast<int>(v)));
  const uint32_t hi = static_cast<uint32_t>(uniform(static_cast<int>(v >> 32)));
  return static_cast<long long>((static_cast<uint64_t>(hi) << 32) | lo);
}

// q / d for 0 <= q, 1 <= d.  Tile-steps number less than 2^32 but for single requests of a
// million tokens and more, and a workgroup runs about ten divisions before its first load: as
// 32-bit ones they take 1.2 us less per attention pass than as 64-bit ones (head dim 128, 1 request
// of 1024 tokens), and a multiplication by the reciprocal in 64-bit floating point took as long as
// those.  Larger values go bit by bit, in little code.
FD_RULE long long div_steps(long long q, long long d) {
  if (((q | d) >> 32) == 0) return static_cast<uint32_t>(q) / static_cast<uint32_t>(d);
  long long r = 0, rem = 0;
#ifdef __HIP_DEVICE_COMPILE__
#pragma unroll 1
#endif
  for (int b = 62; b >= 0; --b) {
    rem = 2 * rem + ((q >> b) & 1);
    if (rem >= d) {
      rem -= d;
      r |= 1LL << b;
    }
  }
  return r;
}

// QB: queries per tile.  TABLES: requests are found by binary search in prefix tables, else
// they are walked.  CUT: the shares may cut items; without it they are runs of whole items.
template <int QB, int DH, bool TABLES, bool CUT>
struct AttnSched {
  const SchedTables* t;         // TABLES
  const int32_t* cu_q;          // else
  const int32_t* req_tok_off;
  int B, G;               // G: shares, a multiple of the XCDs when they cut
  int tiles;              // query tiles over all requests
  long long work_head;    // tile-steps of one head (key tiles summed over every query tile)
  long long work;         // ... of every head
  long long per;          // work = per * G + extra; little work: shares of per, those past the work empty
  int extra;
  uint32_t inv;           // 2^32 / G, rounded up: x / G = (x * inv) >> 32 for 0 <= x <= G * G, 8 <= G <= 1024
  bool cut;
  bool narrow;            // work for the whole grid (head dim <= 64: pieces then store O in bf16)

  FD_RULE AttnSched(const SchedTables* tab, const int32_t* cq, const int32_t* rto, int B_, int H, int G_, int nkv_max)
      : t(tab), cu_q(cq), req_tok_off(rto), B(B_), G(G_), tiles(0), work_head(0), cut(false), narrow(false) {
    if constexpr (TABLES) {
      tiles = uniform(t->tpre[B]);
      work_head = uniform(t->wpre[B]);
    } else {
      for (int b = 0; b < B; ++b) {
        const int nt = (cu_q[b + 1] - cu_q[b] + QB - 1) / QB;
        tiles += nt;
        work_head += static_cast<long long>(nt) * ((req_tok_off[b + 1] - req_tok_off[b] + kKeyTile - 1) / kKeyTile);
      }
    }
    work = work_head * H;
    per = div_steps(work, G);
    extra = static_cast<int>(work - per * G);
    inv = 0xffffffffu / static_cast<uint32_t>(G) + 1;
    if constexpr (CUT) {
      narrow = work >= G;
      cut = G % kXcds == 0 && attn_cuts(DH, tiles * H, H, work_head, tiles, per + (extra > 0), nkv_max, G, 0);
      if (cut) {   // little work on as many workgroups as give each kMinShareSteps tile-steps
        const long long up = ((work + kMinShareSteps - 1) / kMinShareSteps + kXcds - 1) / kXcds * kXcds;
        if (up < G) {   // whole: items of a multiple of it are cut at share bounds only
          G = static_cast<int>(up);
          per = kMinShareSteps;
          extra = 0;
        }
      }
    }
  }
  // the share run by workgroup `blk` (G: none)
  FD_RULE int share(int blk) const {
    const int per_xcd = G / kXcds;
    if (G % kXcds != 0) return blk;
    return blk / kXcds < per_xcd ? (blk % kXcds) * per_xcd + blk / kXcds : G;
  }
  // tile-step q < work: its item's first tile-step and key tiles, head, request,
  // the request's first query tile and the query tile
  FD_RULE void locate(long long q, long long& i_start, int& nkv, int& head, int& b, int& first, int& tau) const {
    head = static_cast<int>(div_steps(q, work_head));
    long long r = q - static_cast<long long>(head) * work_head;
    if constexpr (!TABLES) {   // requests without tile-steps are passed over
      b = 0;
      first = 0;
      nkv = 1;
      for (; b < B; ++b) {
        const int nt = (cu_q[b + 1] - cu_q[b] + QB - 1) / QB;
        nkv = (req_tok_off[b + 1] - req_tok_off[b] + kKeyTile - 1) / kKeyTile;
        const long long span = static_cast<long long>(nt) * nkv;
        if (r < span) break;
        r -= span;
        first += nt;
      }
    } else {
      // the request: the largest b < B with wpre[b] <= r, which has tile-steps
      // (wpre[b + 1] > r); requests without any are passed over
      int lo = 0, hi = B - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (uniform(t->wpre[mid]) <= r) lo = mid; else hi = mid - 1;
      }
      b = lo;
      first = uniform(t->tpre[b]);
      const long long w0 = uniform(t->wpre[b]);
      nkv = static_cast<int>(div_steps(uniform(t->wpre[b + 1]) - w0, uniform(t->tpre[b + 1]) - first));
      r -= w0;
    }
    const long long y = div_steps(r, nkv);
    tau = first + static_cast<int>(y);
    i_start = q - (r - y * nkv);
  }
  FD_RULE long long bound(long long x) const {   // first tile-step of share x (x <= G)
    if (x >= G) return work;
    // floor(x * work / G)
    const long long q = x * per + static_cast<long long>((static_cast<uint64_t>(static_cast<uint32_t>(x) * extra) * inv) >> 32);
    if (q >= work) return work;
    if (cut) return q;
    long long i_start;
    int nkv, head, b, first, tau;
    locate(q, i_start, nkv, head, b, first, tau);
    return i_start == q ? q : i_start + nkv;
  }
  // Scratch slot of share w's piece of key tiles [kt0, kt1) of an item of nkv: -1 for a whole item.
  FD_RULE static int slot_of(int w, int kt0, int kt1, int nkv) { return kt0 > 0 ? 2 * w : kt1 < nkv ? 2 * w + 1 : -1; }
  // slot of piece j of a cut item whose first piece is in share x
  FD_RULE static int slot_at(int x, int j) { return 2 * (x + j) + (j == 0); }
  // last share that holds a piece of the item that ends at tile-step i_end and goes on past share x
  FD_RULE int last_share(int x, long long i_end) const {
    while (bound(x + 1) < i_end) ++x;
    return x;
  }
};

}  // namespace fd
