// Argument blocks and launchers shared by the C-ABI layer and the HIP kernels.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

#include <hip/hip_runtime_api.h>

#include "divide.hpp"

namespace ellm {

constexpr int MAX_LAUNCH_REQ = 128;   // requests that a launch is planned for (3.2 KB of arguments); larger batches go in groups of so many
constexpr int MAX_PATCH = 448;        // table entries patched by one launch
constexpr int TILE_TOKENS = 64;       // the kernel that walks tiles: rows of one chunk a wave handles at a time
constexpr int UNIT_TOKENS = 16;       // the kernel that walks units: rows of one chunk the work is dealt out by
constexpr int STEP_UNITS = 4;         // units of a request that are worth a wave of their own
constexpr int BLOCK_UNITS = 16;       // small launches: units of a request that one workgroup of several waves takes
constexpr int WIDE_UNITS = 32;        // launches up to twice as large: the most units that a workgroup takes,
constexpr int WIDE_WAVES = 8;         // and its waves
constexpr int HEADS_PER_PASS = 16;    // q heads of a group the kernel that walks units handles in one pass over K and V
constexpr int SIMDS_PER_CU = 4;       // a decode launch runs one wave on each SIMD
constexpr int SHARE_WAVES = SIMDS_PER_CU;   // waves of a workgroup that walk a share each
constexpr int WS_ML = 2;              // floats per partial and q head in the (m, l) region of the workspace
constexpr int MERGE_STRIDE = 16;      // words of a line of counters of partial results: 64 bytes
constexpr size_t STATIC_WS_BYTES = 16u << 20;   // the fixed workspace of the entry point that allocates nothing

// what a kernel needs to turn (tensor, token) into an address
struct PoolView {
  char* base;                 // device pool
  const int32_t* table;       // device mirror of the chunk tables, [max_tensors][max_slots]
  const uint64_t* vbase;      // NULL: kernels go through the table. Else: per tensor, the start of its virtual
                              // address range, into which the driver has mapped its chunks; kernels read that
  uint32_t* merged;           // lines of counters, 0 between launches: workgroups whose partial result of a request is in
                              // the workspace. Line kv head * MAX_LAUNCH_REQ + request; of blocks, the blocks' own numbers.
                              // A set for each workspace: launches that may overlap count in different ones
  uint32_t chunk_bytes;
  int32_t tokens_per_chunk;
  int32_t tiles_per_chunk;    // ceil(tokens_per_chunk / TILE_TOKENS); a tile never straddles a chunk
  int32_t units_per_chunk;    // ceil(tokens_per_chunk / UNIT_TOKENS); nor does a unit
  int32_t max_slots;
  int32_t n_q_heads, n_kv_heads, head_dim, group;
  Divisor by_chunk, by_tiles, by_units;   // division by tokens_per_chunk, tiles_per_chunk, units_per_chunk
};

// One decode launch: requests [q_row0, q_row0 + n_req) of the caller's batch.
// For every kv head the units of all requests, laid end to end in request order, form one sequence
// of units_per_head units, which is dealt out evenly to waves_per_head waves: wave w takes
// units_each units, the first units_extra waves one more, each from where the wave before it
// stopped. A wave whose share runs from one request into the next finishes a result for each; so
// request b is covered by n_part waves per kv head, numbered from the wave that holds its first
// unit (wave_first). A request that lies wholly inside one wave's share (n_part == 1) is finished by that wave, which
// normalises and writes the output row itself. The others ("split" requests) are added up: SHARE_WAVES neighbouring
// waves are a workgroup, whose results of a request meet in LDS; a request that reaches into several workgroups gets one
// partial result from each, part0 + j from the j-th, and the workgroup that ends last, or the combine pass where there
// are many, adds those up (merge_parts()). Short launches of more than HEADS_PER_PASS heads have workgroups of one wave, and a
// partial result from each (single_waves()).
// A launch that fills the GPU has one wave for every SIMD of it (a second wave on a SIMD is served markedly
// worse than the first and slows both down): all are resident at once and have the same amount to
// read, so none waits for a slot and none is left over at the end. The cut is fixed by the plan,
// so results do not depend on which wave ran when.
//
// Workspace of a launch, from the pointer the launch is given: accumulator rows
// [kv head][partial slot of the head][q head of the group][D] fp32 (ws_slots = n_kv_heads *
// parts_per_head slots in all), then the (m, l) pairs in the same order, WS_ML floats each.
template <int REQS>
struct BatchArgsOf {
  static constexpr int MAX_REQ = REQS;
  BatchArgsOf() {}            // (filled in field by field: not worth clearing first)
  // (first what a wave needs before anything else: one load of eight words)
  int32_t n_req;
  int32_t waves_per_head;     // <= units_per_head
  int32_t units_each, units_extra;   // units_per_head = waves_per_head * units_each + units_extra
  Divisor by_waves;           // division by waves_per_head
  int32_t step_units;         // 1; or, in a launch too small to fill the GPU, what every wave (STEP_UNITS) or
                              // workgroup of several waves (up to WIDE_UNITS) gets: up to this many units of
                              // one request (then "units" and "waves" in the fields around are such steps)
  int32_t q_row0;             // row of the first request in q / out
  int32_t unit_tokens;        // TILE_TOKENS or UNIT_TOKENS: what the work is dealt out by, and which kernel walks it
  int32_t units_per_head;     // units of all requests of the launch, for one kv head
  int32_t parts_per_head;     // partial slots per kv head: the sum of n_part over the split requests (where workgroups are
                              // waves of several shares, a request uses no more than it spans workgroups), or slots_by_workgroup()
  int32_t ws_slots;           // n_kv_heads * parts_per_head
  int32_t merge_parts;        // requests with 2 <= n_part <= merge_parts are added up by the workgroup that ends last;
                              // 0 where any request has more than merge_parts()
  int32_t n_split_req;        // requests with more: the combine pass runs for these only
  // the requests for the combine pass in ascending order, one byte each
  uint32_t split_req[REQS / 4];
  // per request, one record: a wave gets all of them with one round of loads (Records in kernels.hip)
  struct Req {
    int32_t len, tensor;
    int32_t unit_prefix;      // units of the requests before this one
    int32_t wave_first;       // wave that holds this request's first unit
    int32_t n_part;           // waves that hold units of this request
    int32_t part0;            // first partial slot of the request within a kv head's slots (split requests)
  } req[REQS];
  // for the combine pass:
  int32_t wg_waves;           // waves of a workgroup that each have a share of their own (SHARE_WAVES), or 1
  int32_t in_order_parts;     // requests of up to so many partials are added up in the attention kernel's order
};
using BatchArgs = BatchArgsOf<MAX_LAUNCH_REQ>;
// what a launch in blocks of few requests hands to its kernel instead: the host writes the arguments to device memory for
// each launch; with 0.5 KB instead of 3.2 a call of 4 requests of up to 256 tokens takes 5.77 us instead of 6.04, of one of 3300 7.54
// instead of 7.69
using FewArgs = BatchArgsOf<16>;

// The two groups of a batch of up to 2 * MAX_LAUNCH_REQ requests in one launch: the workgroups of the second behind those of the
// first, each with its own plan, slots and counters, so that every output is bit for bit that of two launches. For two groups only:
// handed over for one plan, these 6.5 KB, and the look which half a workgroup is in, make a call of one request of 3300 tokens 8.03 us
// instead of 7.52, chunks of 16 tokens 33.6 instead of 32.9, an 8B-shaped step 2003 instead of 1985.
struct PairArgs {
  BatchArgs half[2];
  uint32_t workgroups;        // of the first
  uint32_t counters;          // words from the first one's counters to the second's
  uint64_t floats;            // from the first one's workspace to the second's
};

// Slots for the partial results that the attention kernel of a planned launch leaves, counted by workgroup: returned are those of a
// kv head, and part0 and the slots of `a` are set to them. A request that one workgroup has all of needs none, unless the combine
// pass takes it; where a head's waves are no multiple of SHARE_WAVES its workgroups begin elsewhere from head to head (and as in the
// first ones from the SHARE_WAVES-th head on), and the most count. (The plan itself reserves a slot for each wave, which is the documented bound.)
inline int64_t slots_by_workgroup(BatchArgs& a, int32_t n_kv_heads) {
  const int32_t ways = a.waves_per_head % SHARE_WAVES ? std::min<int32_t>(n_kv_heads, SHARE_WAVES) : 1;
  int64_t parts = 0;
  for (int32_t i = 0; i < a.n_req; i++) {
    auto& r = a.req[i];
    int32_t n = 0;
    if (r.n_part > 1) {
      if (a.wg_waves == 1) n = r.n_part;
      else
        for (uint32_t g = 0, w0 = r.wave_first; g < (uint32_t)ways; g++, w0 += a.waves_per_head)
          n = std::max(n, (int32_t)((w0 % SHARE_WAVES + r.n_part - 1) / SHARE_WAVES) + 1);
      if (n == 1 && a.merge_parts > 0) n = 0;
    }
    r.part0 = n ? (int32_t)parts : 0;
    parts += n;
  }
  a.parts_per_head = (int32_t)parts;
  a.ws_slots = (int32_t)parts * n_kv_heads;
  return parts;
}

// (aligned: every workgroup reads one or a few neighbours of each array, which 24 more bytes of PoolView had put across two cache
// lines; prompts of four requests 123.8 us a call, aligned 123.5, ahead of that 123.3)
struct alignas(64) AppendArgs {
  int32_t n_req, total_new;
  int32_t tensor[MAX_LAUNCH_REQ];
  int32_t len_before[MAX_LAUNCH_REQ];
  int32_t tok0[MAX_LAUNCH_REQ];    // first new-token row of request b, relative to this launch
};

struct PatchArgs {
  int32_t n;
  int32_t idx[MAX_PATCH];
  int32_t val[MAX_PATCH];
};

// chunks copied by one launch between the pool and the pinned host buffer: move i is device chunk
// chunk[i] <-> host slot host_slot[i]
constexpr int MAX_COPY = 480;
struct CopyArgs {
  int32_t n;
  int32_t chunk[MAX_COPY];
  int32_t host_slot[MAX_COPY];
};

// Workgroups of a call's copy kernel. While copies of both directions run, 64 for an offload and 128 for a fetch are the fastest,
// but the writes to host memory that an offload has under way hold up all other traffic of the GPU. Where attention runs beside
// copies the offload takes 32 (for how that is known see ellm_pool::compute_beside_copies): 16 requests swapped for others layer by
// layer under the attention of an 8B-shaped model, an attention launch (60 us alone) / the step: 64 workgroups 265 to 340 us /
// 113 ms, 32: 68 us / 108 ms, 48 and 96 for the fetch 280 to 330, 32 and 64: 94 to 120. With copies always under way: offloads alone
// 240 / 158 us, fetches alone (128) 213, both 300 / 184. Swaps that nothing runs beside, 8 requests for 8, 27 chunks: 1714 us, 32: 1760.
constexpr int OFFLOAD_WORKGROUPS = 64, OFFLOAD_WORKGROUPS_BESIDE = 32, FETCH_WORKGROUPS = 128;

// Which of the two attention kernels a pool's calls use: the one that walks 64-row tiles of a chunk, or the one
// that walks 16-row units. The first has no instance for group sizes that are not 1, 2, 4 or 8 (it would
// read K and V two or three times: 6 heads 92 us against 52, 16 heads of 64 145 against 70) and loads whole
// tiles, so it pays for chunks that do not fill them. Measured on 32 requests of 1500 to 3500 tokens, 8 kv
// heads, tiles against units, us: head size 128, 4 q heads per kv head: chunks of 16 tokens 80 / 58, 24:
// 65 / 58, 40: 55.8 / 57.4, 64: 56.1 / 58.5, 512: 55.7 / 59.2, and alike for 1, 2 and 8 heads; head size
// 64, 1 head: 24: 44 / 32, 40: 33.0 / 31.8, 48: 30.5 / 31.4, 80: 32.7 / 31.5, 102: 30.4 / 31.8, 2 heads
// within 1 %; 4 heads: 48: 33.1 / 31.6, 512: 33.5 / 32.0, 8 heads: 39 / 32 and 38 / 33. With the fused append one
// head of 128 gains nothing from units in chunks of 32 to 39 tokens (32: 60.2 / 61.4, without it 57.2 / 58.0, 36: 59.1 /
// 61.1, 56.5 / 56.5); they stay there because they carry a weight as two bf16 values, tiles as one.
inline bool tile_kernel(int head_dim, int group, int tokens_per_chunk) {
  const int64_t Tc = tokens_per_chunk, padded = (Tc + TILE_TOKENS - 1) / TILE_TOKENS * TILE_TOKENS;
  if (head_dim == 128) return (group == 1 || group == 2 || group == 4 || group == 8) && padded * 5 <= Tc * 8;
  return (group == 1 || group == 2) && padded * 3 <= Tc * 4;
}

// Up to how many waves (blocks: steps) a request may be shared by for its partial results, one per workgroup, to be
// added up by the workgroup that ends last. The others go to the combine pass: a launch of its own, 4 to 5 us, but a
// workgroup for each q head. Where one request of a launch goes there, all do: beside a combine launch the others' sums at the
// end of the attention kernel save nothing and take 2 to 4 us. us a call, both ways in one launch / the pass for all: 1 kv head of
// 128, 4 q heads, 10 requests of 5400 to 16200 tokens (shares of 15 to 38 workgroups) 19.1 / 15.6, 8 heads of 64, 11 of 2100 to 6400
// 15.6 / 12.0, 16 heads of 128, 11 of 6500 to 19400 36.9 / 30.8; 12 heads, 6 of 2000 to 9000 (8 to 36 blocks) 14.6 / 10.4.
// us, added up by the last / by the pass, of launches in which all requests go one way:
//  - Where shares are walked one wave reads them all, in tiles 16 to 32 KB in a round trip: up to 64 KB. 8 kv heads of 128, one request of
//    20000 to 100000 tokens (32 workgroups), 1 q head each (16 KB) 65.5 / 66.6, 4 (64 KB) 21.8 / 22.6, 8 (128 KB) 72.3 /
//    70.2, 16 (256 KB) 81 / 70.8; 4 kv heads (64 workgroups), 4 q heads each (128 KB) 30.2 / 28.3, 8: 36.9 / 29.6.
//    In units 16 KB of two heads in a round trip: up to 32 KB. 16-token chunks, 2 kv heads of 128, 8 q heads each, 9 of 10000 (56 KB) 21.3 /
//    19.8, of 12486 (60 KB) 25.2 / 23.7, 14 of 12000 (40 KB) 32.4 / 31.8, 4 kv heads, 16 each, 12 of 6000 (48 KB) 31.3 / 30.4, 24 of 6000
//    (32 KB) 52.4 / 53.8; heads of 64, 6 each, 4 of 12800 to 38300 (27 to 60 KB) 18.0 / 15.4, 8 each, 9 of 12000 (30 KB) 14.0 / 14.6.
//  - The waves of a block take 64 columns each, 16 partials in a round trip: up to 192 KB. One request: 8 kv heads of 128, 31
//    blocks of 4 q heads each (62 KB) 9.7 / 11.7, of 6 (93 KB) 10.1 / 11.9, of 8 (124 KB) 10.6 / 12.0, of 16 (248 KB) 12.9 / 12.4; 16
//    blocks of 16 (128 KB) 9.8 / 11.6; 4 kv heads, 59 of 4 (118 KB) 11.1 / 12.1, of 8 (236 KB) 12.6 / 12.3; heads of 64, 31 of 16
//    (124 KB) 9.0 / 11.5.
//  - A group of more than HEADS_PER_PASS q heads takes several launches over the same units, each with these sums at its
//    end: up to 16 waves. us a call, in every launch / the pass: 4 kv heads of 64, 20 q heads each, 8 requests of
//    2100 to 6400 tokens (16 to 48 waves) 25.1 / 21.7, of 128, 32 q heads, 14 of 1000 to 3100 (18 waves) 39.7 / 33.9, 128 of 300 to 600
//    (2 or 3) 54.6 / 85.
inline int merge_parts(int head_dim, int group, bool blocks, bool tiles) {
  const int row = std::min(group, HEADS_PER_PASS) * head_dim * 4;      // bytes of a partial result in one launch
  if (blocks) return (192 << 10) / row;
  return std::min((tiles ? 64 << 10 : 32 << 10) * SHARE_WAVES / row, group > HEADS_PER_PASS ? 4 * SHARE_WAVES : 1 << 30);
}
// Such launches do without sums in the kernel where a wave has few units (more, where many requests end inside waves): a
// workgroup is one wave, and every wave leaves a partial result of its own for one combine pass behind the last launch. us
// a call, sums in every launch / this: steps: 16 requests of 200 to 400 tokens, 1 kv head of 128, 64 q heads 47.3 / 22.1, 44 of 58 to 175,
// 33 heads 31.2 / 17.4, 4 kv heads, 40 heads, 5 of 270 to 800 36.6 / 18.5; 8 kv heads, 32 heads, 114 of 31 to 93 (5 units a wave) 44.0 / 33.7; 2 kv
// heads, 16 of 2000 to 4000 (6 units a wave, few requests) 28.1 / 32.0.
inline bool single_waves(int group, bool blocks, int64_t units, int64_t waves, int n_req) {
  return group > HEADS_PER_PASS && !blocks && units < STEP_UNITS * waves + 2 * n_req;
}

// Small launches are cut in units whatever the pool's shares are cut in, and request by request: in blocks (one
// workgroup of several waves per BLOCK_UNITS units of a request, `blocks` of them per kv head) or in steps (one wave
// per STEP_UNITS). Small: at most two blocks for every CU, one where requests are split, so a split launch has at most
// one partial result per SIMD.
inline bool small_launch(int group, int64_t blocks, int n_req, int n_kv, int cus) {
  return group <= HEADS_PER_PASS && blocks * n_kv <= cus * (blocks > n_req ? 1 : 2);
}
// Which of the two; tiles: the pool's shares are cut in tiles; one_piece: no request has more than one tile. The lines were
// drawn when every split request was followed by a combine launch, which blocks of whole requests saved and fewer partial
// results made shorter; those below 12 blocks (3000 tokens) per request went by steps, unless almost every CU got a block. 256
// CUs, 8 kv heads of 128, us a call of the present kernels in a replayed graph, blocks / steps / shares of tiles:
//  - Requests of one block each: 8 of 200 tokens, 4 q heads each 4.8 / 5.9 / 6.0, 64 of 200 12.1 / 12.3 / 10.5; 1 q head 5.2 / 5.7 / 5.0,
//    64 of 80 7.8 / 6.1 / 6.1, of 128 (two full tiles) 10.2 / 7.7 / 7.9, of 200 12.0 / 11.6 / 9.7.
//  - Requests that one wave handles: a workgroup whose other waves have nothing to do takes longer to start where a
//    CU gets two of them. 1 q head: 8 of 64 tokens 3.6 / 4.7 / 4.3, 32 of 64 3.9 / 5.2 / 5.0, 64 of 64 7.1 / 5.1 / 4.8; 4 q heads: 3.7 /
//    4.9 / 5.9, 3.9 / 5.3 / 6.6, 7.1 / 5.3 / 6.4. Heads of 64: 64 of 64 3.8 / 4.5 / 3.9.
//  - Split requests: 4 q heads: 1 of 512 tokens 6.5 / 7.2 / 7.2, 8 of 300 7.4 / 8.1 / 8.5, 1 of 1500 7.3 / 8.0 / 9.0, 3000 7.9 / 9.0 / 9.4, 8000
//    9.2 / 10.7 / 11.6, 16 of 512 8.6 / 8.9 / 9.8; 1 q head: 1 of 512 6.4 / 7.1 / 6.0, 8 of 300 7.3 / 7.7 / 7.1, 1 of 1500 7.3 / 7.8 / 7.5, 3000
//    7.9 / 8.9 / 7.9 (tiles are as fast for requests of one head; their weights are rounded to one bf16 value). Heads of 64:
//    1 of 512 5.5 / 6.6 / 5.2, 8000 7.4 / 10.3 / 8.3.
// So blocks would be the faster way for all split requests of 4 heads, and no longer are for 64 requests of two or more tiles.
// Pools whose shares are cut in units always take blocks, which leaves a request's result independent of its neighbours.
inline bool takes_blocks(int head_dim, bool tiles, bool one_piece, int64_t blocks, int n_req, int n_kv, int cus) {
  const int64_t workgroups = blocks * n_kv;
  if (!tiles || head_dim == 64) return true;
  if (blocks > n_req) return blocks >= 12 * (int64_t)n_req || workgroups * 8 >= (int64_t)cus * 7;
  return !one_piece || workgroups <= cus;
}

// Launches past those in which one workgroup per CU can still have everything in flight at once, whichever way the pool's
// shares are cut: blocks again, but of as many units (17 to WIDE_UNITS) as leave no more of them than CUs. Shares of such
// launches are one or two tiles a wave, one after the other. Shares / blocks, us a call, 8 kv heads of 128: 8 requests of 800
// to 1200 tokens, 4 q heads each 11.0 / 10.1, of 1400 to 1700 12.4 / 11.8, of 1700 to 2000 14.3 / 13.2, 16 of 700 to 900
// 12.4 / 11.8, 30 of 300 to 400 12.3 / 9.3; 4 of 3000 to 4000, 8 q heads each 18.0 / 13.4, 1 q head 13.4 / 13.4; 6 q heads, 8 of
// 1500 to 2000 14.3 / 12.7. Heads of 64, 4 q heads, 8 of 1500 to 2000 10.4 / 8.8, 1 q head 9.5 / 8.9; twice as many units a
// wave are no gain there (16 of 1500 to 2000, 4 q heads 14.2 / 13.5, 1 q head 12.6 / 13.7). Up to 12 units for every CU (17
// of 257 tokens 9.0 / 7.9), and where a request has more than WIDE_PARTS blocks (1 of 15000 15.6 / 13.5, 9000 13.9 / 10.8),
// blocks would be faster too: these two lines are not drawn by the figures but stand where tests/test_host_logic.py has shares.
constexpr int WIDE_PARTS = 16;
inline bool wide_batch(int group, int n_req, int room) { return group <= HEADS_PER_PASS && n_req <= room; }   // room: CUs for each kv head
inline bool wide_launch(int64_t units, int room) { return units > 12 * (int64_t)room && units <= (int64_t)WIDE_UNITS * room; }

// resident waves of the partial-pass kernel per compute unit (occupancy query)
int partial_waves_per_cu(int head_dim, int group, int tokens_per_chunk);

// each returns 0 or a hipError_t value
int launch_table_patch(int32_t* table, const PatchArgs& a, hipStream_t stream);
int launch_fill(uint32_t* words, uint32_t value, size_t n, hipStream_t stream);
int launch_kv_append(const PoolView& pv, const void* k_new, const void* v_new, const AppendArgs& a,
                     hipStream_t stream);
// Whole chunks between the pool (chunk c at pool + c * chunk_bytes) and the host buffer as the GPU
// sees it (slot s at host + s * chunk_bytes); to_host: offload, else fetch.
int launch_chunk_copy(char* pool, char* host, uint32_t chunk_bytes, const CopyArgs& a, bool to_host, int workgroups, hipStream_t stream);
// k_new / v_new non-NULL: fused append. a.len then counts one token per request whose K/V row
// ([request][kv head][dim], rows q_row0 .. of the caller's batch) is still in k_new / v_new; the
// kernel uses it from there and writes it into the chunk.
// out: the caller's output rows; requests with n_part == 1 are finished by the partial pass itself.
// ev_start / ev_stop (may be NULL): events that receive the start time of the call's first attention
// kernel and the end time of its last one, taken from the kernels' own dispatches.
int launch_decode_partial(const PoolView& pv, const void* q, const void* k_new, const void* v_new, float* ws,
                          void* out, float scale_log2, const BatchArgs& a, hipStream_t stream,
                          hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
// the two plans of `a`, which run the same kernel, in one launch
int launch_decode_pair(const PoolView& pv, const void* q, const void* k_new, const void* v_new, float* ws, void* out, float scale_log2,
                       PairArgs& a, hipStream_t stream, hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
int launch_decode_combine(const PoolView& pv, const float* ws, void* out, const BatchArgs& a, hipStream_t stream);

// Device address and size of the library's fixed workspace on the current device (resolved once per
// device, kept afterwards). Allocates nothing. Returns 0 or a hipError_t value.
int static_workspace(float** ptr, size_t* bytes);

// calibration (measurement only)
int launch_copy(void* dst, const void* src, int64_t bytes, hipStream_t stream);
int launch_read(const void* src, int64_t bytes, uint32_t* sink, hipStream_t stream);
int launch_kv_stream(const PoolView& pv, uint32_t* sink, const BatchArgs& a, hipStream_t stream);

}  // namespace ellm
