// How a workgroup of score_mfma_wide.hip goes through the 32-key tiles of its key chunk: which tile is requested when, what is
// waited for, which tiles the pipelined loop takes and which the plain one, when parked column sums are added up.  Apart from
// the kernel, and written against its operations, so that the same code also runs on the host against a model of the LDS ring
// (tests/sanitize/launch_stubs.cpp): a request of rows past the sequence's end or into a slot that is still read shows on the
// GPU as a memory fault or as a wrong sum now and then.
#pragma once
#include "common.h"

namespace skv {

#define SKV_HD __host__ __device__ inline __attribute__((always_inline))

template <int V> using IntC = std::integral_constant<int, V>;

template <int PASS>
struct TileChunk {
  int key0, nsub;     // first key, tiles
  int ni, n_full;     // keys of the sequence, keys that every row sees
  int causal;
  // first key of the s-th tile: pass 1 goes forwards, pass 2 backwards (what pass 1 left in L2 is the end of every chunk)
  SKV_HD int key(int s) const { return key0 + 32 * (PASS == 2 ? nsub - 1 - s : s); }
  SKV_HD bool whole(int s) const { return key(s) + 32 <= ni; }   // all of its rows exist
  // whether request s is followed by one of another tile: past the chunk's end the last tile is requested again
  SKV_HD bool more(int s) const { return s + 1 < nsub; }
  // whether the pipelined loop can take the `count` tiles from s on: they exist, every row sees them whole, and what is requested
  // meanwhile, `ahead` tiles further, is whole too
  SKV_HD bool clean(int s, int count, int ahead) const {
    if (s + count > nsub) return false;
    if (PASS == 2) return !causal || key(s) + 32 <= n_full;
    const int last = s + count + ahead < nsub ? s + count + ahead : nsub - 1;
    return key(s + count - 1) + 32 <= n_full && whole(last);
  }
};

// the operations of go_through_chunk, mostly lambdas
template <class Wait, class Barrier, class Request, class RequestWhole, class Begin, class Step, class Any, class Park, class AddOne, class AddEach>
struct ChunkOps {
  Wait wait; Barrier barrier; Request request; RequestWhole request_whole; Begin begin; Step step; Any any; Park park; AddOne add_one; AddEach add_each;
};
template <class... T>
SKV_HD ChunkOps<T...> chunk_ops(T... t) { return ChunkOps<T...>{t...}; }

// The whole chunk, its first PD tiles already requested.  fast: with the pipelined loop.  PARKS: the waves' column sums of a tile
// are parked and added up later, the first `unflushed` tiles' have been.  Operations, by all waves:
//   wait(IntC<N>)     at most N tiles' requests are outstanding, and no LDS operation
//   barrier()
//   request(s)        request s; request_whole(s): of a tile that is whole
//   begin(s)          reads tile s and starts its first unit
//   step(s)           computes a begun tile s, reading tile s + 1 (whatever the slot holds behind the chunk's end) and starting its first unit
//   any(s)            reads and computes tile s
//   park(s)
//   add_one(s)        adds up tile s's parked sums; add_each(s): those of tiles s to s + NW - 1
template <int PD, int NW, bool PARKS, int PASS, class Ops>
SKV_HD void go_through_chunk(const TileChunk<PASS>& c, bool fast, int& unflushed, Ops& ops) {
  constexpr int GROUP = 2;   // tiles of one run
  static_assert(PD == 3, "a tile is waited for with up to two later ones outstanding");
  // Tile s ready: a wave's share of it has landed when at most the later requests (PD - 1 tiles) are outstanding, and its reads of
  // tile s - 1 are done; then the barrier.  After it everybody's share of tile s is in LDS and everybody is done reading tile
  // s - 1's slot, which the next request overwrites.
  auto ready_any = [&](int s) __attribute__((always_inline)) {
    const int left = c.nsub - 1 - s;
    if (left >= 2) ops.wait(IntC<2>{});
    else if (left == 1) ops.wait(IntC<1>{});
    else ops.wait(IntC<0>{});
    ops.barrier();
    if (s + PD < c.nsub) ops.request(s + PD);
  };
  // inside the loop: always one request, past the chunk's end the last tile again (nobody reads it; it keeps the count of
  // outstanding loads, and with it the step, free of conditions)
  auto ready_whole = [&](int s) __attribute__((always_inline)) {
    ops.wait(IntC<PD - 1>{});
    ops.barrier();
    ops.request_whole(s + PD);
  };
  auto step = [&](int s) __attribute__((always_inline)) {
    ready_whole(s + 1);
    ops.step(s);
    ops.park(s);
  };
  int ready = 0;   // tiles made ready
  for (int s = 0; s < c.nsub;) {
    if (fast && s + PD <= c.nsub && c.clean(s, GROUP, PD)) {   // (PD requests are outstanding)
      if (ready <= s) ready_whole(s);
      ops.begin(s);
      do {   // one straight run of instructions
        step(s);
        step(s + 1);
        s += GROUP;
        if (PARKS && s >= unflushed + NW + 1) { ops.add_each(unflushed); unflushed += NW; }
      } while (c.clean(s, GROUP, PD));
      if (c.clean(s, 1, PD)) { step(s); ++s; }   // (half of another run)
      ready = s + 1;
    } else {
      if (ready <= s) { ready_any(s); ready = s + 1; }   // (else behind the loop, whose last step has)
      for (; unflushed + 2 <= s; ++unflushed)            // (parked before the barrier of tile s)
        if (PARKS) ops.add_one(unflushed);
      ops.any(s);
      ops.park(s);
      ++s;
    }
  }
  ops.wait(IntC<0>{});   // (the requests past the chunk's end)
}

}  // namespace skv
