// Stand-ins for the kernel launchers of libstructkv, for the host-only sanitizer build of its C ABI:
// api.cpp is compiled with -fsanitize=address,undefined and linked against these instead of the HIP
// kernels, so that argument validation, work planning and workspace carving run under the sanitizers
// on a machine without a GPU.  The stubs launch nothing and count the calls; those that stand in for the scoring
// kernels also check the plan they are handed against what those kernels assume about it (tilings that are
// instantiated, key chunks within the LDS capacity, chunk bookkeeping) and keep it for the tests to look at, and those of
// the selection follow its forms by length.
#include "../../paper_2604_06746_amd/csrc/score_schedule.h"

#include <algorithm>
#include <deque>

namespace skv {

static int g_launches = 0;
static int32_t g_last_plan[8];
static int32_t g_last_selection[3];
static int g_last_wide;
static int g_last_copy[2];
extern "C" int structkv_stub_launch_count(void) { return g_launches; }
// RB, NW, KC, planes, stream_k, RC, grid_chunks, path of the latest scoring launch
extern "C" void structkv_stub_last_plan(int32_t* out) { for (int i = 0; i < 8; ++i) out[i] = g_last_plan[i]; }

// whether that one was for the kernels of score_mfma_wide.hip
extern "C" int structkv_stub_last_wide(void) { return g_last_wide; }
// of the latest fused layer step: the form its scoring prepared (-1: none), the form of its selection, whether that also
// sums the scoring's planes
extern "C" void structkv_stub_last_selection(int32_t* out) { for (int i = 0; i < 3; ++i) out[i] = g_last_selection[i]; }
// of the latest layer step's selection: workgroups per sequence that copy the kept rows (0: the gather kernel does), and the most
// 16-byte units that one of them moves
extern "C" void structkv_stub_last_copy(int32_t* out) { for (int i = 0; i < 2; ++i) out[i] = g_last_copy[i]; }
// the division of the copy's units by their (tensor, head) pairs: quotients that come out wrong, over all that a workgroup may see
extern "C" int structkv_stub_copy_division_faults(int kv_heads, int tensors) {
  alignas(16) static unsigned char rows[16];
  CopyWork c;
  if (!make_copy_work(rows, tensors == 2 ? rows : nullptr, 16, 16, rows, tensors == 2 ? rows : nullptr, 16, 16, kv_heads, 16, &c)) return -1;
  int bad = c.planes != (uint32_t)(kv_heads * tensors);
  for (uint32_t q = 0; q < (uint32_t)kCopyRows * c.planes; ++q)
    bad += (c.recip ? (uint32_t)(((uint64_t)q * c.recip) >> 32) : q) != q / c.planes;
  return bad;
}
static bool chunks_fit(const ScorePlan& p, const SeqTable& seq, int64_t total) {
  bool ok = seq.batch >= 1 && seq.batch <= kMaxBatch && seq.chunk_start[0] == 0 && seq.chunk_start[seq.batch] == p.grid_chunks;
  for (int b = 0; ok && b < seq.batch; ++b) {
    const int64_t n = seq.cu[b + 1] - seq.cu[b];
    ok = n >= 0 && seq.chunk_start[b + 1] - seq.chunk_start[b] == (n + p.KC - 1) / p.KC && seq.cu[b + 1] <= total;
  }
  return ok;
}
static void keep_plan(const ScorePlan& p) {
  ++g_launches;
  const int32_t plan[8] = {p.RB, p.NW, p.KC, p.planes, p.stream_k, p.RC, (int32_t)p.grid_chunks, p.path};
  for (int i = 0; i < 8; ++i) g_last_plan[i] = plan[i];
  g_last_wide = p.wide;
}

// The bins of the mid-sized selection for one centre: how many keys the two directions of the mapping disagree on, how many
// bins do not follow on the one before, and whether they end with the last key.
extern "C" int structkv_stub_bin_faults(uint32_t centre) {
  int bad = 0;
  uint32_t next = 0;
  const BinTiers tiers = bins_around(centre);
  for (uint32_t bin = 0; bin < (uint32_t)kUsedBins; ++bin) {
    uint32_t lo, width;
    fine_range(bin, tiers, &lo, &width);
    const uint32_t hi = lo + ((1u << width) - 1u);
    bad += lo != next || hi < lo || width < (uint32_t)kSubBits;
    const uint32_t keys[4] = {lo, lo + (hi - lo) / 3, lo + (hi - lo) / 2, hi};
    for (uint32_t key : keys) bad += fine_bin(key, tiers) != bin;
    next = hi + 1;
  }
  return bad + (next != 0);
}
// The same for the bins of the pivot detector's rows and the keys of non-negative scores; no bin may leave its octave.
extern "C" int structkv_stub_row_bin_faults(uint32_t centre) {
  int bad = 0;
  uint32_t next = 0x80000000u;
  const uint32_t at = row_bins_at(centre);
  for (uint32_t bin = 0; bin < 1024u + kRowExtra; ++bin) {
    uint32_t lo, width;
    row_bin_range(bin, at, &lo, &width);
    const uint32_t hi = lo + ((1u << width) - 1u);
    bad += lo != next || hi < lo || (lo >> 23) != (hi >> 23);
    const uint32_t keys[4] = {lo, lo + (hi - lo) / 3, lo + (hi - lo) / 2, hi};
    for (uint32_t key : keys) bad += row_bin(key, at) != bin;
    next = hi + 1;
  }
  return bad + (next != 0);
}

// score_mfma_wide.hip's way through a key chunk, run against a model of one wave's requests, the LDS ring and the slots for parked
// sums.  All waves run the same program, so what one of them has done before a barrier all have; what lies between two barriers
// is in no order between the waves.  Counts what would be a fault: rows outside the sequence requested, a slot requested while some wave
// may still read it, a tile read before it has landed for everybody, sums parked over others that were not added up or may still be
// read, sums added up before every wave has parked them; tiles left out, taken twice or by a loop that cannot mask.
template <int PASS>
struct RingModel {
  static constexpr int NBUF = 4, PARKED = 8;
  struct Parked { int tile = -1; bool added = true; int at = -1; };
  TileChunk<PASS> c;
  bool parks;
  int faults = 0, barriers = 0, next = 0, computed = 0, added = 0;
  struct Request { int tile, slot; };
  std::deque<Request> out, waited;        // not waited for, oldest first; waited for by this wave, but not yet behind a barrier
  int content[NBUF], read_at[NBUF];       // tile that has landed for everybody (-1: unknown); barrier count of the slot's last read
  Parked parked[PARKED];
  RingModel(const TileChunk<PASS>& chunk, bool p) : c(chunk), parks(p) {
    for (int i = 0; i < NBUF; ++i) { content[i] = -1; read_at[i] = -1; }
  }
  void check(bool ok) { faults += !ok; }
  void request(int s, bool whole) {
    const int tile = next;                // (the kernel's pointer to the next tile's first row)
    check(tile >= 0 && tile < c.nsub && c.key(tile) >= c.key0 && (whole ? c.whole(tile) : c.key(tile) < c.ni));
    check(read_at[s % NBUF] < barriers);
    content[s % NBUF] = -1;
    out.push_back({tile, s % NBUF});
    if (c.more(s)) ++next;
  }
  void request_any(int s) { check(next == s); request(s, c.whole(s)); }
  void wait(int tiles) { while ((int)out.size() > tiles) { waited.push_back(out.front()); out.pop_front(); } }
  void barrier() {
    ++barriers;
    for (const Request& r : waited) content[r.slot] = r.tile;
    waited.clear();
  }
  void read(int s) {
    if (s < c.nsub) check(content[s % NBUF] == s);
    read_at[s % NBUF] = barriers;
  }
  void compute(int s, bool masks) {
    check(s == computed++);
    const bool visible = c.key(s) + 32 <= c.n_full;
    check(masks || visible || (PASS == 2 && !c.causal));   // (pass 2 writes no key past the sequence's end)
  }
  void park(int s) {
    if (!parks) return;
    Parked& p = parked[s % PARKED];
    check(p.added && p.at < barriers);
    p = {s, false, barriers};
  }
  void add(int s) {
    Parked& p = parked[s % PARKED];
    check(p.tile == s && !p.added && p.at < barriers);
    p.added = true;
    p.at = barriers;
    ++added;
  }
  int run(bool fast) {
    constexpr int PD = NBUF - 1, NW = 4;
    int unflushed = 0;
    for (int s = 0; s < PD && s < c.nsub; ++s) request_any(s);
    auto ops = chunk_ops([&](auto n) { wait(decltype(n)::value); }, [&]() { barrier(); }, [&](int s) { request_any(s); },
                         [&](int s) { request(s, true); }, [&](int s) { read(s); }, [&](int s) { compute(s, false); read(s + 1); },
                         [&](int s) { read(s); compute(s, true); }, [&](int s) { park(s); }, [&](int s) { add(s); },
                         [&](int s) { for (int i = 0; i < NW; ++i) add(s + i); });
    if (parks) go_through_chunk<PD, NW, PASS == 2>(c, fast, unflushed, ops);
    else go_through_chunk<PD, NW, false>(c, fast, unflushed, ops);
    check(computed == c.nsub && out.empty());
    if (parks) {
      barrier();
      for (int s = unflushed; s < c.nsub; ++s) add(s);
      check(added == c.nsub);
    }
    return faults;
  }
};
// faults of both passes over one key chunk: keys of the sequence, the chunk's first key, most keys of a chunk, causal window or 0
extern "C" int structkv_stub_chunk_faults(int ni, int key0, int kc, int window) {
  const int key_end = ni < key0 + kc ? ni : key0 + kc, nsub = (key_end - key0 + 31) / 32, n_full = ni - window, causal = window > 0;
  int faults = 0;
  for (int fast = 0; fast < 2; ++fast) {
    faults += RingModel<1>({key0, nsub, ni, n_full, causal}, false).run(fast);
    for (int parks = 0; parks < 2; ++parks) faults += RingModel<2>({key0, nsub, ni, n_full, causal}, parks).run(fast);
  }
  return faults;
}

hipError_t launch_score_mfma_ring(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq, const void*,
                                  const void*, int64_t, int64_t, float, float*, const float*, float*, int64_t total,
                                  float* probs, int pass, hipStream_t) {
  keep_plan(p);
  if (p.grid_chunks == 0) return hipSuccess;
  bool ok = p.path == 0 && (s.head_dim == 64 || s.head_dim == 128) && (pass == 1 || pass == 2);
  ok = ok && ((p.RB == 2 && p.NW == 4) || (p.RB == 1 && p.NW == 4) || (p.RB == 2 && p.NW == 1) || (p.RB == 1 && p.NW == 1));
  ok = ok && p.RPC == 32 * p.RB && p.R == (s.n_q_heads / s.n_kv_heads) * s.window && p.RC == (p.R + p.RPC - 1) / p.RPC;
  ok = ok && (p.NW == 4 || p.RC == 1);                          // one-wave workgroups hold a KV group's only row-chunk
  ok = ok && (!p.wide || (p.RB == 2 && p.NW == 4 && s.head_dim == 128));
  const int planes = pass == 2 && probs == nullptr ? p.planes : 0;
  ok = ok && (planes == 0 || planes == 1 || (planes == 2 && p.RB == 2)) && (p.split == 1 || ((p.split == 2 || p.split == 4) && p.planes == p.RB));
  ok = ok && (planes == 0 || p.CP == s.n_q_heads / s.n_kv_heads);
  const int cap = planes ? planes_key_cap(p.NW, planes * p.split) : ring_key_cap(p.NW);   // keys whose sums fit the LDS
  ok = ok && p.KC >= 32 && p.KC % 32 == 0 && (pass == 1 || p.KC <= cap);
  ok = ok && (int64_t)s.n_kv_heads * ((p.RC + p.NW - 1) / p.NW) * p.grid_chunks < ((int64_t)1 << 31);
  return ok && chunks_fit(p, seq, total) ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_score_f32(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq, const void*, const void*,
                            int64_t, int64_t, float, float*, const float*, float*, int64_t total, float*, int pass,
                            hipStream_t) {
  keep_plan(p);
  if (p.grid_chunks == 0) return hipSuccess;
  bool ok = p.path == 1 && s.head_dim <= 256 && (pass == 1 || pass == 2) && p.planes == 0;
  ok = ok && p.RPC == 32 && p.R == (s.n_q_heads / s.n_kv_heads) * s.window && p.RC == (p.R + 31) / 32;
  ok = ok && (p.NW == 1 || p.NW == 2 || p.NW == 4) && p.CP == (p.RC + p.NW - 1) / p.NW;
  ok = ok && p.KC >= 32 && p.KC % 32 == 0 && p.KC <= kF32KeyCap;
  ok = ok && (int64_t)s.n_kv_heads * p.CP * p.grid_chunks < ((int64_t)1 << 31);
  return ok && chunks_fit(p, seq, total) ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_score_short(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq, const void*, const void*,
                              int64_t, int64_t, float, float*, float*, int64_t total, hipStream_t) {
  keep_plan(p);
  const bool bf16 = s.dtype == STRUCTKV_DTYPE_BF16;
  bool ok = p.path == 2 && (s.head_dim == 64 || s.head_dim == 128) && (p.RPC == 16 || (bf16 && p.RPC == 32));
  ok = ok && p.R == (s.n_q_heads / s.n_kv_heads) * s.window && p.RC == (p.R + p.RPC - 1) / p.RPC && p.CP == p.RC;
  ok = ok && s.n_kv_heads * p.RC <= kReduceShortPlanes && seq.batch >= 1 && seq.batch * s.n_kv_heads * p.RC <= 256;
  for (int b = 0; ok && b < seq.batch; ++b)
    ok = seq.cu[b + 1] >= seq.cu[b] && seq.cu[b + 1] - seq.cu[b] <= (bf16 ? 2048 : 1024) && seq.cu[b + 1] <= total;
  return ok ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_score_combine(const structkv_shape&, const ScorePlan&, const SeqTable&, const float*, float*,
                                float*, uint32_t*, int64_t, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_score_reduce(const structkv_shape&, const ScorePlan&, const SeqTable&, const float*, int64_t,
                               float*, const float*, float*, float*, float*, float, float, const SelectFusion* fuse,
                               hipStream_t) {
  ++g_launches;
  g_last_selection[0] = fuse ? fuse->mode : -1;
  return !fuse || (fuse->hist && fuse->idx_out && (fuse->mode == kSelMid || fuse->mode == kSelLong)) ? hipSuccess : hipErrorInvalidValue;
}
void topk_plan(const SeqTable& seq_in, int keep_tail, void* wsp, SeqTable* plan, TopkWs* ws, unsigned* blocks) {
  *plan = seq_in;
  *blocks = 1;
  int64_t longest = 0;
  for (int b = 0; b < seq_in.batch; ++b)
    if (seq_in.k[b] > 0 && seq_in.cu[b + 1] - seq_in.cu[b] - keep_tail > longest) longest = seq_in.cu[b + 1] - seq_in.cu[b] - keep_tail;
  ws->mode = selection_mode(longest);
  ws->mass = 0.f;
  ws->red = nullptr;
  ws->hist = ws->state = ws->suf = ws->meta = (uint32_t*)wsp;
  g_last_selection[0] = -1;
}
hipError_t launch_topk_rest(const float*, const SeqTable& plan, int keep_tail, const TopkWs& ws, unsigned, int32_t*, hipStream_t) {
  ++g_launches;
  g_last_selection[1] = ws.mode;
  g_last_selection[2] = ws.red != nullptr;
  bool ok = ws.hist && ws.mass > 0.f;
  g_last_copy[0] = ws.copy ? ws.copy_parts : 0;
  g_last_copy[1] = 0;
  for (int b = 0; ws.copy && b < plan.batch; ++b) {   // what a workgroup has room for
    const int64_t rows = ceil_div(plan.k[b] + keep_tail, ws.copy_parts), units = (rows * ws.copy->planes) << ws.copy->upr_shift;
    ok = ok && ws.mode == kSelShort && ws.copy_parts >= 1 && rows <= kCopyRows;
    g_last_copy[1] = std::max(g_last_copy[1], (int)units);
  }
  for (int b = 0; ws.red && b < plan.batch; ++b)   // the selection sums the planes: at most two tokens a thread
    ok = ok && ws.mode == kSelShort && ws.red->planes <= kReduceShortPlanes && plan.cu[b + 1] - plan.cu[b] <= kReduceShortSeq && keep_tail >= 0;
  return ok ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_group_sums(const structkv_shape&, const ScorePlan&, const float*, int64_t, float*, hipStream_t) {
  ++g_launches; return hipSuccess;
}
hipError_t launch_accumulate(float*, const float*, int64_t, float, float, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_topk(const float*, const SeqTable&, int, int32_t*, void*, hipStream_t) { ++g_launches; return hipSuccess; }
size_t topk_workspace_bytes(int batch, int64_t total_tokens) {
  return 256 * (size_t)(batch > 0 ? batch : 1) + 4 * (size_t)(total_tokens > 0 ? total_tokens : 0) + 256;
}
bool topk_static_fits(int, int64_t total_tokens) { return total_tokens <= 2 * (int64_t)STRUCTKV_STATIC_TOPK_MAX_TOKENS; }
hipError_t topk_static_scratch(void** ptr, size_t* bytes) {
  alignas(256) static unsigned char host_stand_in[(size_t)4 << 20];   // never touched: the launchers are stubs
  *ptr = host_stand_in;
  *bytes = sizeof(host_stand_in);
  return hipSuccess;
}
static uint32_t g_row_bins_at;
hipError_t launch_pivot_planes(const ReduceWork& r, uint32_t at, uint32_t* hist, float* var_part, hipStream_t) {
  ++g_launches;
  g_row_bins_at = at;
  return r.colsum && r.planes == r.Hq && r.Hq <= kMaxBatch && hist && var_part && at == row_bins_of(r.w, r.total) ? hipSuccess : hipErrorInvalidValue;
}
// all buffers lie behind each other: the partial sums in Hq x n words (var_part, part_above, sums), the kernels on the same bins
hipError_t launch_pivot_mass(const ReduceWork& r, uint32_t kk, uint32_t at, uint32_t*, uint32_t*, float*, float* part_above, const float* var_part,
                             float* sums, float*, float*, hipStream_t) {
  ++g_launches;
  const int64_t parts = (int64_t)r.Hq * pivot_shares(r.total);
  bool ok = kk >= 1 && kk <= r.total && r.total <= ((int64_t)1 << 24) && at == g_row_bins_at;
  ok = ok && part_above - var_part == parts && sums - part_above == parts && (sums - var_part) + 2 * r.Hq <= r.Hq * r.total;
  return ok ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_pivot_heads(const float*, int, int64_t, const int32_t*, int64_t, float, float*, hipStream_t) {
  ++g_launches; return hipSuccess;
}
hipError_t launch_zero_floats(float*, int, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_pivot_finish(const float*, int, int64_t, float, int, float*, float*, hipStream_t) {
  ++g_launches; return hipSuccess;
}
hipError_t launch_block_scores(const float*, const SeqTable&, int, float*, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_positions(const int64_t*, const SeqTable&, const int32_t*, int64_t*, hipStream_t) {
  ++g_launches; return hipSuccess;
}
hipError_t launch_gather(const void*, const void*, int64_t, int64_t, void*, void*, int64_t, int64_t, int, int,
                         const SeqTable&, const int32_t*, hipStream_t) { ++g_launches; return hipSuccess; }

}  // namespace skv
