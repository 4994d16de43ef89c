// HIP kernels for gfx950 (MI355X): table patch, KV append, split-K decode attention, combine.
//
// Decode attention is a streaming read of every cached K and V row once per step (the paper calls
// auto-regressive generation memory-bound, Introduction and Sec. 2.2.1), so the kernels are built
// around 128-bit coalesced loads from the scattered chunks. With one query token per request the
// arithmetic is G (q heads per kv head) flops per byte read. Two kernels share the work cut, the
// workspace and the combine pass: one walks 64-row tiles of a chunk, with an instance per group size (1
// and 2 heads on ordinary vector lanes; 4 and 8, where the lanes of a wave could no longer keep up with
// the bytes, on 4x4x4 matrix instructions); the other walks 16-row units and takes any group size and
// any chunk size with 16x16x32 matrix instructions. Which is used where: tile_kernel() in kernels.hpp.
//
// Per-launch metadata (which tensors, their lengths, how the tiles are dealt out) is passed by value
// in the kernel arguments, so a launch needs no host-to-device copy and no staging buffer whose
// lifetime would have to be tracked. The chunk tables live in a device mirror that is patched, also
// through kernel arguments, whenever the host changes an entry.
#include "kernels.hpp"

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

namespace ellm {

// ---------------------------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------------------------
// fp32 -> bf16 bits, round to nearest even; NaN stays NaN
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0u;
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}

// v + (v of lane ^ 16), v + (v of lane ^ 32): gfx950's row and half-wave swaps exchange the odd rows
// (upper half) of one register with the even rows (lower half) of another; fed the same value
// twice they return the two partners side by side, with no trip through the LDS crossbar
__device__ __forceinline__ float add_xor16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_xor32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// DPP lane permutations inside a row of 16 lanes
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
constexpr int DPP_QUAD_XOR1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int DPP_QUAD_XOR2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int DPP_ROW_HALF_MIRROR = 0x141; // lane i <-> 7 - i within each 8 lanes
constexpr int DPP_ROW_MIRROR = 0x140;      // lane i <-> 15 - i within each 16 lanes

__device__ __forceinline__ float max_xor16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max_xor32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// reductions over the 64 lanes, result in every lane: four steps inside the rows of 16 lanes (DPP),
// then the two swaps across rows
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_f32<DPP_QUAD_XOR1>(v));
  v = fmaxf(v, dpp_f32<DPP_QUAD_XOR2>(v));
  v = fmaxf(v, dpp_f32<DPP_ROW_HALF_MIRROR>(v));
  v = fmaxf(v, dpp_f32<DPP_ROW_MIRROR>(v));
  return max_xor32(max_xor16(v));
}

__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_f32<DPP_QUAD_XOR1>(v);
  v += dpp_f32<DPP_QUAD_XOR2>(v);
  v += dpp_f32<DPP_ROW_HALF_MIRROR>(v);
  v += dpp_f32<DPP_ROW_MIRROR>(v);
  return add_xor32(add_xor16(v));
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef short __attribute__((ext_vector_type(4))) bf16x4_bits_t;     // four bf16 values as the matrix instructions take them
typedef float __attribute__((ext_vector_type(4))) f32x4_t;

typedef __attribute__((ext_vector_type(2))) float f32x2_t;
// two floats rounded to nearest-even bf16, the first in the low half
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{a, b}), bf16x2_t));
}

// c + a.lo * b.lo + a.hi * b.hi on packed bf16 pairs, fp32 accumulate
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c, false);
}

// The same, with the first operand taken from lane N of this lane's row of 16 (a DPP broadcast
// folded into the instruction): lets 16 lanes share one register of query values.
template <int N>
__device__ __forceinline__ float dot2_bf16_rowlane(uint32_t row_shared, uint32_t b, float c) {
  asm("v_dot2c_f32_bf16_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
      : "+v"(c) : "v"(row_shared), "v"(b), "n"(N));
  return c;
}

// The compiler cannot see that the inline-asm instruction above is a dot product, so it does not
// insert the wait states the hardware needs between a dot product's result and its first use by a
// different instruction (nor between a register write and its first use as a DPP source). Passing
// the value through this makes the gap explicit.
__device__ __forceinline__ void settle(float& v) { asm volatile("s_nop 3" : "+v"(v)); }
__device__ __forceinline__ void settle(uint32_t& v) { asm volatile("s_nop 1" : "+v"(v)); }

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// 16-byte load of data that is read once (the K/V stream): marked non-temporal, so that it does not
// displace what is reused (partials, queries, tables) from the caches on its way through
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_stream16(const void* p) {
  const u32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
  return make_uint4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ void store_stream16(void* p, uint4 v) {
  const u32x4_t t = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(t, reinterpret_cast<u32x4_t*>(p));
}

// cache-policy operand of the buffer and load-to-LDS builtins: non-temporal; coherent across the GPU (past the L2
// of the wave's own XCD)
constexpr int CPOL_NT = 2, CPOL_DEVICE = 16;

typedef __attribute__((ext_vector_type(4))) uint32_t words4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t words2_t;

// memory from `base` on (the same for all lanes; said so, because the descriptor has to be in scalar registers) as a
// buffer: loads past its end return zeros, stores past it are dropped
constexpr int BUFFER_RAW = 0x00027000;    // last word of a buffer descriptor: raw dwords, range check on the byte offset
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_at(const void* base, int32_t bytes) {
  const uint64_t b = (uint64_t)base;
  const uint64_t bs = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b) |
                      (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32)) << 32;
  return __builtin_amdgcn_make_buffer_rsrc((void*)bs, 0, __builtin_amdgcn_readfirstlane(bytes), BUFFER_RAW);
}

typedef const __attribute__((address_space(1))) void* global_cptr_t;
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const int32_t __attribute__((address_space(4)))* const_i32_ptr;
typedef const uint64_t __attribute__((address_space(4)))* const_u64_ptr;

// How a kernel gets from (tensor, slot) to the chunk's bytes. With the software table the slot's
// entry names a chunk of the pool. DIRECT is the paper's own arrangement (Sec. 2.1.1, Sec. 3.2): the
// tensor is a contiguous virtual address range into which the driver has mapped the chunks, so a
// slot's bytes sit at base + slot * chunk_bytes and no table is read.
struct TensorWalk {
  const_i32_ptr trow;      // table row of the tensor (table addressing)
  const char* tbase;       // start of the tensor's virtual range (direct addressing)
};
template <bool DIRECT>
__device__ __forceinline__ TensorWalk tensor_walk(const PoolView& pv, int32_t tensor) {
  TensorWalk w;
  if (DIRECT) {
    w.trow = nullptr;
    w.tbase = reinterpret_cast<const char*>(((const_u64_ptr)pv.vbase)[tensor]);
  } else {
    w.trow = (const_i32_ptr)(pv.table + (int64_t)tensor * pv.max_slots);
    w.tbase = nullptr;
  }
  return w;
}
template <bool DIRECT>
__device__ __forceinline__ const char* chunk_addr(const PoolView& pv, const TensorWalk& w, int32_t slot) {
  if (DIRECT) return w.tbase + (uint64_t)slot * pv.chunk_bytes;
  return pv.base + (uint64_t)w.trow[slot] * pv.chunk_bytes;
}

// s_waitcnt immediates (gfx9 encoding): vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8
constexpr int waitcnt_vm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }

constexpr float NEG_BIG = -1.0e30f;   // finite stand-in for "no score yet"; exp2(NEG_BIG - x) == 0

__global__ __launch_bounds__(256) void fill_kernel(uint32_t* words, uint32_t value, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) words[i] = value;
}

// ---------------------------------------------------------------------------------------------
// table patch: device_table[idx[i]] = val[i]
// ---------------------------------------------------------------------------------------------
__global__ void table_patch_kernel(int32_t* table, PatchArgs a) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < a.n) table[a.idx[i]] = a.val[i];
}

// ---------------------------------------------------------------------------------------------
// KV append: copy rows of D bf16 from the dense [token][Hkv][D] inputs to their chunk rows
// ---------------------------------------------------------------------------------------------
template <int D, bool DIRECT>
__global__ __launch_bounds__(256) void kv_append_kernel(PoolView pv, const uint4* __restrict__ k_new,
                                                        const uint4* __restrict__ v_new, AppendArgs a) {
  // One workgroup per new token: which request it belongs to, its position and its chunk are the
  // same for every lane, so they are found once with scalar loads. The lanes then copy the token's
  // 2 * n_kv_heads rows (K and V of every head), 16 bytes each per turn.
  constexpr int LPR = D * 2 / 16;            // 16-byte pieces per row
  const int32_t tau = blockIdx.x;            // index of the new token in the launch
  int lo = 0, hi = a.n_req - 1;              // request that owns it: largest b with tok0[b] <= tau
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.tok0[mid] <= tau) lo = mid; else hi = mid - 1;
  }
  const int b = lo;
  const int64_t pos = (int64_t)a.len_before[b] + (tau - a.tok0[b]);
  const int32_t slot = (int32_t)(pos / pv.tokens_per_chunk);
  const int32_t r = (int32_t)(pos - (int64_t)slot * pv.tokens_per_chunk);
  const TensorWalk walk = tensor_walk<DIRECT>(pv, a.tensor[b]);
  char* chunk = const_cast<char*>(chunk_addr<DIRECT>(pv, walk, slot)) + (uint64_t)r * (D * 2);
  const uint64_t plane_bytes = (uint64_t)pv.tokens_per_chunk * (D * 2);
  const int n16 = pv.n_kv_heads * LPR;       // 16-byte pieces of the token's K (and of its V)
  const uint4* ks = k_new + (int64_t)tau * n16;
  const uint4* vs = v_new + (int64_t)tau * n16;
  for (int i = threadIdx.x; i < n16; i += 256) {
    const int h = i / LPR, sub = i - h * LPR;
    char* dst = chunk + (uint64_t)(h * 2) * plane_bytes + sub * 16;
    const uint4 kv = load_stream16(ks + i), vv = load_stream16(vs + i);     // read once, written once
    store_stream16(dst, kv);
    store_stream16(dst + plane_bytes, vv);
  }
}

// ---------------------------------------------------------------------------------------------
// offload / fetch (paper Sec. 2.2.2): whole chunks between the pool and pinned host memory, which the
// GPU reads and writes directly over PCIe. One launch moves all chunks of a call, wherever they are:
// per chunk a copy call of the runtime costs about 10 us of a 46 us transfer (2 MiB at a time go at
// 44-45 GB/s on this machine, one large copy at 57); a kernel that gathers the chunks itself moves calls of 27
// chunks at 55 / 56 GB/s out / in, the host's wait for their end included (engines 45 / 45). Both directions at once, call by
// call with nothing to wait for, 31 each, calls of 3 chunks 28 (engines 48, and 12 to 25).
// WPC workgroups share a chunk; the loads and stores are streaming ones (the data passes through once), one of each a
// lane at a time: while calls of both directions run beside each other, what an offload has in flight holds up the
// fetch's reads. Requests of 1 to 5 chunks swapped for others, 27 chunks each way, us: 4 loads a lane, 64 workgroups for a
// call 1893; 1 load, 64: 1819, 128: 1839, 192: 1829, 64 for an offload and 128 for a fetch 1702 to 1748, the other way round
// 1920, 64 and 256: 1773, 32 and 128: 1747. One direction alone goes at 50 to 56 GB/s in all of these.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void chunk_copy_kernel(char* __restrict__ pool, char* __restrict__ host, uint32_t chunk_bytes,
                                                         int32_t wpc, int32_t to_host, CopyArgs a) {
  const int32_t c = blockIdx.x / wpc, part = blockIdx.x - c * wpc;
  if (c >= a.n) return;
  char* dev_p = pool + (size_t)a.chunk[c] * chunk_bytes;
  char* host_p = host + (size_t)a.host_slot[c] * chunk_bytes;
  const uint4* src = reinterpret_cast<const uint4*>(to_host ? dev_p : host_p);
  uint4* dst = reinterpret_cast<uint4*>(to_host ? host_p : dev_p);
  const uint32_t nv = chunk_bytes / 16;                 // chunk_bytes is a multiple of 256
  for (uint32_t i = (uint32_t)part * 256u + threadIdx.x; i < nv; i += (uint32_t)wpc * 256u) store_stream16(dst + i, load_stream16(src + i));
}

// ---------------------------------------------------------------------------------------------
// work partition shared by the partial pass, the combine pass and the calibration kernel
// ---------------------------------------------------------------------------------------------
// number of units (tiles) of a sequence of len tokens (neither straddles a chunk)
__device__ __forceinline__ int32_t units_of(int32_t len, const PoolView& pv, int32_t units_per_chunk, int32_t unit_tokens = UNIT_TOKENS) {
  const int32_t Tc = pv.tokens_per_chunk, full = divide(len, pv.by_chunk), rest = len - full * Tc;
  return full * units_per_chunk + (rest + unit_tokens - 1) / unit_tokens;
}

// Kernel arguments that a wave needs early. Named in one place, they are asked for together when it starts; left to
// itself the compiler puts loads of them behind waits for other loads and behind branches, and no cache holds them yet.
// (eight to an asm statement: across such statements loads are not made into wider ones)
template <class A, class B, class C, class D, class E, class F, class G, class H>
__device__ __forceinline__ void wanted(A a, B b, C c, D d, E e, F f, G g, H h) {
  asm volatile("" :: "s"(a), "s"(b), "s"(c), "s"(d), "s"(e), "s"(f), "s"(g), "s"(h));
}

// A kernel argument as a value of its own, which is not loaded again later and from which nothing is derived earlier
template <class T>
__device__ __forceinline__ T held(T v) {
  asm volatile("" : "+s"(v));
  return v;
}

// The records of a launch's requests, spread over the lanes of a wave: lane l has those of requests l, l + 64, .. Where a
// wave begins used to be found in three dependent steps (header, a table of the waves' requests, the record), about a third
// of a microsecond each from the L2 and more from memory, which no cache holds the arguments of. Now all records are asked for
// at once, together with the header, when the wave starts. One request of 3300 tokens 8.25 -> 7.99 us a call, 8 requests, 4
// layers 52.3 -> 51.6, four short ones 7.38 -> 7.11; shares no different (8B-shaped step 1992, 1994).
template <class Args>
struct Records {
  using Req = typename Args::Req;
  static constexpr int N = (Args::MAX_REQ + 63) / 64;
  int32_t len[N], tensor[N], unit_prefix[N], wave_first[N], n_part[N], part0[N];
  __device__ __forceinline__ Records(const Args& a, int lane) {
    static_for<0, N>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      const Req& r = a.req[min(64 * k + lane, Args::MAX_REQ - 1)];
      len[k] = r.len; tensor[k] = r.tensor; unit_prefix[k] = r.unit_prefix;
      wave_first[k] = r.wave_first; n_part[k] = r.n_part; part0[k] = r.part0;
    });
  }
  // request whose units include unit number pos of a kv head's sequence: the last b with unit_prefix[b] <= pos
  __device__ __forceinline__ int32_t find(int32_t n_req, int32_t pos, int lane) const {
    int32_t cnt = 0;
    static_for<0, N>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      cnt += __popcll(__builtin_amdgcn_ballot_w64(64 * k + lane < n_req && unit_prefix[k] <= pos));
    });
    return cnt - 1;
  }
  __device__ __forceinline__ Req of(int32_t b) const {      // b: the same in all lanes
    return {get(len, b), get(tensor, b), get(unit_prefix, b), get(wave_first, b), get(n_part, b), get(part0, b)};
  }

 private:
  static __device__ __forceinline__ int32_t get(const int32_t (&field)[N], int32_t b) {
    int32_t v = field[0];
    // (values, not places, to choose from: a choice of places makes the compiler put the records into LDS and scratch memory)
    static_for<1, N>([&](auto kc) {
      const int32_t w = field[decltype(kc)::value];
      v = b >= 64 * decltype(kc)::value ? w : v;
    });
    return __builtin_amdgcn_readlane(v, b & 63);
  }
};

// what a wave (in blocks: a workgroup) handles: kv head g, wave w of that head, n_units steps of the head's
// sequence from step u_lo on, the first of which belongs to request b. A step is a unit (a tile in the
// kernel that walks tiles) or, where every wave gets one step, up to step_units units of one request
template <class Args>
struct Share { int32_t g, w, u_lo, n_units, b; typename Args::Req first; };

template <class Args>
__device__ __forceinline__ Share<Args> locate_share(const Args& a, const Records<Args>& records, int32_t index, int lane) {
  Share<Args> s;
  const int32_t W = a.waves_per_head, each = a.units_each, extra = a.units_extra;
  s.g = divide(index, a.by_waves);
  s.w = index - s.g * W;
  s.u_lo = s.w * each + min(s.w, extra);
  s.n_units = each + (s.w < extra ? 1 : 0);
  s.b = records.find(a.n_req, s.u_lo, lane);
  s.first = records.of(s.b);
  return s;
}

// Calls body(pool, workspace, plan, number of this workgroup in the plan): of a pair, with what belongs to this workgroup's half.
template <class Args, class Body>
__device__ __forceinline__ void in_launch(const PoolView& pv, float* ws, const Args& a, Body body) {
  if constexpr (std::is_same_v<Args, PairArgs>) {
    const bool second = blockIdx.x >= a.workgroups;
    PoolView mine = pv;
    mine.merged += second ? a.counters : 0u;
    body(mine, ws + (second ? a.floats : 0u), a.half[second ? 1 : 0], (int32_t)(blockIdx.x - (second ? a.workgroups : 0u)));
  } else {
    body(pv, ws, a, (int32_t)blockIdx.x);
  }
}

// which four dims of a head piece f of a partial result's row holds: rows keep the dims in the order in which the
// lanes of the kernel that wrote them store neighbouring pieces
template <int D>
__device__ __forceinline__ int32_t partial_dim(int32_t unit_tokens, int32_t f) {
  constexpr int LPR = D / 8, E = D / 16;
  return unit_tokens == TILE_TOKENS ? 8 * (f % LPR) + 4 * (f / LPR) : E * (4 * (f & 3) + f / E) + (f % E) / 4 * 4;
}

// ---------------------------------------------------------------------------------------------
// Requests that several waves share. The SHARE_WAVES waves of a workgroup (one per SIMD of a CU) walk neighbouring
// shares; a request that such a wave begins or ends in the middle of has its results of that wave put into LDS, and
// when all four are done the results of one request are added up there, the requests dealt out to the waves. What
// lies wholly inside the workgroup is finished by that. A request that reaches into other workgroups leaves one partial
// result in the workspace, written past the L2 of the XCD, and its workgroup counts itself in once it is there; the last
// to do so adds up all of them. Which one that is depends on who ends last, but the sum is taken in the order of the
// partials, so the result does not. Nobody waits for another workgroup, and the counter goes back to 0 by itself
// (an increment that wraps).
// This took the place of a combine launch behind every call, 4.6 us of which 3.4 are the launch: 8B-shaped step 2087 ->
// 2003 us, 8 requests of it, 4 layers 67.5 -> 63.7, 48 requests of 6 q heads each 52.2 -> 49.4, 64 of 16 heads of 64 68.2 ->
// 66.6, chunks of 16 tokens 36.9 -> 33.8. By single waves, without the sum in LDS, it was no faster than the pass: up to 29
// partials for one wave to add up, 6 us. A workgroup's chain behind its last wave is 2.2 to 3.3 us now (where the results go 0.6, LDS
// sum 0.3 and store 0.3, count 0.3, adding up 0.7 to 1.5).
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void store_partial(__amdgpu_buffer_rsrc_t rows, int32_t at, float4 v) {
  const words4_t w = {__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)};
  __builtin_amdgcn_raw_buffer_store_b128(w, rows, at, 0, CPOL_DEVICE);
}
__device__ __forceinline__ void store_partial(__amdgpu_buffer_rsrc_t pairs, int32_t at, float2 v) {
  __builtin_amdgcn_raw_buffer_store_b64(words2_t{__float_as_uint(v.x), __float_as_uint(v.y)}, pairs, at, 0, CPOL_DEVICE);
}
// this wave's stores have arrived where every XCD sees them
__device__ __forceinline__ void stores_done() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
  asm volatile("" ::: "memory");
}
// One more of n_part workgroups has its results in memory (asked by one lane): how many had before? `line`: of the counters,
// `k`: which in that line.
__device__ __forceinline__ uint32_t count_in(const PoolView& pv, int32_t line, int32_t k, int32_t n_part) {
  return atomicInc(pv.merged + (int64_t)line * MERGE_STRIDE + k, (uint32_t)n_part - 1u);
}

// sums of one 16-byte piece of a head's row over some partials: running maximum, normaliser, weighted sum
struct Sum { float M, L; float4 A; };
__device__ __forceinline__ void add(Sum& s, float L, const float4& v, float w) {
  s.L += L * w;
  s.A.x += v.x * w; s.A.y += v.y * w; s.A.z += v.z * w; s.A.w += v.w * w;
}
__device__ __forceinline__ void rescale(Sum& s, float M) {
  const float w = fast_exp2(s.M - M);
  s.M = M;
  s.L *= w;
  s.A.x *= w; s.A.y *= w; s.A.z *= w; s.A.w *= w;
}

// The partials of a request for n_heads q heads of kv head g from head g_first of the group on. Columns: the pieces of
// the heads' rows in order.
template <int D>
struct Partials {
  static constexpr int F = D / 4;
  __amdgpu_buffer_rsrc_t rows, pairs;
  int32_t group;
  // slot0: the first one's slot; ws_slots: all slots of the workspace
  __device__ __forceinline__ Partials(const float* ws, int32_t ws_slots, int64_t slot0, int32_t n_part, int32_t group, int32_t g_first,
                                      int32_t n_heads) : group(group) {
    const int64_t row0 = slot0 * group + g_first;
    const int32_t n_rows = (n_part - 1) * group + n_heads;
    rows = buffer_at(ws + row0 * D, n_rows * (D * 4));
    pairs = buffer_at(ws + (int64_t)ws_slots * group * D + row0 * WS_ML, n_rows * (WS_ML * 4));
  }
  // columns x, x + step, .. (KB of them) over partials j0 .. j1 - 1, FEW or MANY of them asked for at a time
  template <int KB, int FEW, int MANY>
  __device__ __forceinline__ void sum(Sum (&sums)[KB], int32_t x, int32_t step, int32_t j0, int32_t j1) const {
    asm volatile("" ::: "memory");     // nothing of this is read before the last one has counted itself in
#pragma unroll
    for (int k = 0; k < KB; k++) sums[k] = {NEG_BIG, 0.f, make_float4(0.f, 0.f, 0.f, 0.f)};
    auto some = [&](auto ahead) __attribute__((always_inline)) {
      constexpr int N = decltype(ahead)::value;
      words4_t v[KB][N];
      words2_t ml[KB][N];
#pragma unroll
      for (int u = 0; u < N; u++)
#pragma unroll
        for (int k = 0; k < KB; k++) {
          // (all of the offset lies in the lanes: it is what the buffer's range is compared with, while a part of it in a
          // scalar register is taken off the range first, of which rows past the last would leave less than nothing)
          const int32_t xk = x + k * step, row = (j0 + u) * group + xk / F;
          ml[k][u] = __builtin_amdgcn_raw_buffer_load_b64(pairs, row * (WS_ML * 4), 0, CPOL_DEVICE);
          v[k][u] = __builtin_amdgcn_raw_buffer_load_b128(rows, row * (D * 4) + xk % F * 16, 0, CPOL_DEVICE);
        }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < KB; k++) {
        float M = sums[k].M;
#pragma unroll
        for (int u = 0; u < N; u++) M = j0 + u < j1 ? fmaxf(M, __uint_as_float(ml[k][u].x)) : M;
        rescale(sums[k], M);
#pragma unroll
        for (int u = 0; u < N; u++) {
          // (a row that is not there came back as zeros; a branch around each would make a chain of them)
          const words4_t t = v[k][u];
          add(sums[k], __uint_as_float(ml[k][u].y), make_float4(__uint_as_float(t.x), __uint_as_float(t.y), __uint_as_float(t.z), __uint_as_float(t.w)),
              j0 + u < j1 ? fast_exp2(__uint_as_float(ml[k][u].x) - M) : 0.f);
        }
      }
    };
    for (; j0 + FEW < j1; j0 += MANY) some(std::integral_constant<int, MANY>{});
    if (j0 < j1) some(std::integral_constant<int, FEW>{});
  }
};

// column x of request b's output: the four dims that piece x % (D / 4) of the rows holds, of head g_first + x / (D / 4)
template <int D, class Args>
__device__ __forceinline__ void write_out(const PoolView& pv, uint16_t* __restrict__ out, const Args& a, int32_t b, int32_t g,
                                          int32_t g_first, int32_t x, const Sum& s) {
  constexpr int F = D / 4;
  const float inv = 1.f / s.L;
  uint16_t* o = out + ((int64_t)(a.q_row0 + b) * pv.n_q_heads + g * pv.group + g_first + x / F) * D + partial_dim<D>(a.unit_tokens, x % F);
  *reinterpret_cast<uint2*>(o) = make_uint2(pack_bf16(s.A.x * inv, s.A.y * inv), pack_bf16(s.A.z * inv, s.A.w * inv));
}

// Where a request's partial results are: the workgroups it reaches into, for kv head g, are numbered from 0 on
struct Parts { int32_t first, n; };    // workgroup of its first wave, how many
__device__ __forceinline__ Parts parts_of(int32_t wave_first, int32_t n_part, int32_t waves_per_head, int32_t g, int32_t wg_waves) {
  const int32_t w0 = g * waves_per_head + wave_first;
  if (wg_waves == 1) return {w0, n_part};     // a workgroup is one of the request's steps
  return {w0 / SHARE_WAVES, (w0 + n_part - 1) / SHARE_WAVES - w0 / SHARE_WAVES + 1};
}

// results of the workgroup's waves: slot 2 w of wave w's first request, 2 w + 1 of its last one, if it is another
template <int D, int HEADS>
struct Results {
  static constexpr int SLOTS = 2 * SHARE_WAVES, NONE = SLOTS;      // slot NONE: what takes part in a sum and adds nothing
  float4 rows[SLOTS + 1][HEADS][D / 4 + 1];    // (padded against bank conflicts)
  float2 ml[SLOTS + 1][HEADS];
  int32_t whose[SLOTS];      // request and kv head, -1: no result, or one that needs no other
  // by all waves, a slot in whose each, before their first results
  __device__ __forceinline__ void clear(int32_t wave, int32_t lane) {
    if (lane < 2) whose[2 * wave + lane] = -1;
    for (int32_t h = wave; h < HEADS; h += SHARE_WAVES) {
      if (lane < D / 4) rows[NONE][h][lane] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (lane == 0) ml[NONE][h] = make_float2(-INFINITY, 0.f);
    }
  }
};

// column x of a request's result of this workgroup becomes partial result `part` of the request
template <int D, class Args>
__device__ __forceinline__ void leave_partial(const PoolView& pv, float* ws, const Args& a, int32_t part, int32_t g, int32_t g_first,
                                              int32_t n_heads, int32_t x, const Sum& s) {
  constexpr int F = D / 4;
  const int64_t row0 = ((int64_t)g * a.parts_per_head + part) * pv.group + g_first;
  store_partial(buffer_at(ws + row0 * D, n_heads * (D * 4)), x * 16, s.A);
  if (x % F == 0)
    store_partial(buffer_at(ws + (int64_t)a.ws_slots * pv.group * D + row0 * WS_ML, n_heads * (WS_ML * 4)), x / F * (WS_ML * 4), make_float2(s.M, s.L));
}

// All waves of the workgroup have ended their shares. What follows is a chain of latencies with nothing beside it, so what
// it needs is in registers (`records`, the arguments) before the barrier, LDS is read without a branch, and the heads of a
// request are dealt out to the waves, in up to four pieces that are stored, counted in and added up each by itself: one
// request, four waves; two, two waves each; more, a wave each. (A piece is whole heads: their (m, l) pairs belong to it.) With one
// wave for a request and branches around the parts of each sum: 48 requests of 6 q heads each 49.95 -> 49.3 us, 64 of 16
// heads of 64 66.4 -> 65.7, chunks of 16 tokens 33.6 -> 33.3, the 8B-shaped step 1995 -> 1985.
template <int D, int HEADS, class Args>
__device__ __forceinline__ void end_shares(const PoolView& pv, float* ws_, uint16_t* __restrict__ out, const Args& a, const Records<Args>& records,
                                           const Results<D, HEADS>& res, int32_t g_first, int32_t n_heads, int32_t workgroup, int32_t wave, int32_t lane) {
  constexpr int F = D / 4, SLOTS = Results<D, HEADS>::SLOTS, NONE = Results<D, HEADS>::NONE;
  float* const ws = held(ws_);
  const int32_t waves_per_head = held(a.waves_per_head), parts_per_head = held(a.parts_per_head), ws_slots = held(a.ws_slots),
                merge_parts = held(a.merge_parts);
  __syncthreads();
  const int32_t whose = res.whose[lane % SLOTS];
  uint32_t left = (uint32_t)__builtin_amdgcn_ballot_w64(whose >= 0) & ((1u << SLOTS) - 1u);
  int32_t n_requests = 0;
  for (uint32_t l = left; l; n_requests++)
    l &= ~(uint32_t)__builtin_amdgcn_ballot_w64(whose == __builtin_amdgcn_readlane(whose, __builtin_ctz(l)));
  // pieces of 1, 2 or 4 heads; those that a wave has: piece p0 on, n_pieces of them
  const int32_t shift = n_heads <= 4 ? 0 : n_heads <= 8 ? 1 : 2, pieces = (n_heads + (1 << shift) - 1) >> shift;
  const int32_t each = n_requests == 1 ? 1 : n_requests == 2 ? 2 : 4, p0 = n_requests == 1 ? wave : n_requests == 2 ? wave & ~1 : 0;
  const int32_t n_pieces = min(each, pieces - p0), h0 = p0 << shift, h1 = min(n_heads, (p0 + each) << shift);
  if (n_pieces <= 0) return;
  for (int32_t nth = 0; left; nth++) {
    const int32_t id = __builtin_amdgcn_readlane(whose, __builtin_ctz(left));
    uint32_t mine = (uint32_t)__builtin_amdgcn_ballot_w64(whose == id) & ((1u << SLOTS) - 1u);      // the slots of one request
    left &= ~mine;
    if (n_requests == 2 ? nth != (wave & 1) : n_requests > 2 && nth % SHARE_WAVES != wave) continue;
    const int32_t b = id % MAX_LAUNCH_REQ, g = id / MAX_LAUNCH_REQ, group = held(pv.group);
    const typename Args::Req rq = records.of(b);
    const int32_t n = __builtin_popcount(mine);      // at most one slot of every wave
    int32_t slot[SHARE_WAVES];
#pragma unroll
    for (int i = 0; i < SHARE_WAVES; i++) {
      slot[i] = mine ? __builtin_ctz(mine) : NONE;
      mine &= mine - 1;
    }
    // (a request for the combine pass goes there also where no other workgroup has a part of it)
    const bool whole = n == rq.n_part && rq.n_part <= merge_parts;
    const Parts parts = parts_of(rq.wave_first, rq.n_part, waves_per_head, g, SHARE_WAVES);
    const int64_t slot0 = (int64_t)g * parts_per_head + rq.part0;
    const int64_t row0 = (slot0 + (workgroup - parts.first)) * group + g_first;
    // (stores past this wave's heads are dropped by the buffers' range)
    const auto rows = buffer_at(ws + row0 * D, h1 * (D * 4));
    const auto pairs = buffer_at(ws + (int64_t)ws_slots * group * D + row0 * WS_ML, h1 * (WS_ML * 4));
    for (int32_t x = h0 * F + lane; x - lane < h1 * F; x += 64) {
      const int32_t h = min(x / F, HEADS - 1), f = x % F;
      float2 ml[SHARE_WAVES];
      float4 v[SHARE_WAVES];
#pragma unroll
      for (int i = 0; i < SHARE_WAVES; i++) {
        ml[i] = res.ml[slot[i]][h];
        v[i] = res.rows[slot[i]][h][f];
      }
      Sum s = {ml[0].x, 0.f, make_float4(0.f, 0.f, 0.f, 0.f)};
#pragma unroll
      for (int i = 1; i < SHARE_WAVES; i++) s.M = fmaxf(s.M, ml[i].x);
#pragma unroll
      for (int i = 0; i < SHARE_WAVES; i++) add(s, ml[i].y, v[i], fast_exp2(ml[i].x - s.M));
      if (whole) {
        if (x < h1 * F) write_out<D>(pv, out, a, b, g, g_first, x, s);
      } else {
        store_partial(rows, x * 16, s.A);
        if (f == 0) store_partial(pairs, x / F * (WS_ML * 4), make_float2(s.M, s.L));
      }
    }
    if (whole || rq.n_part > merge_parts) continue;
    stores_done();
    uint32_t before = 0;
    if (lane < n_pieces) before = count_in(pv, g * MAX_LAUNCH_REQ + b, p0 + lane, parts.n);
    const Partials<D> all(ws, ws_slots, slot0, parts.n, held(pv.group), g_first, h1);
    // (all of a wave's pieces or none, as a rule)
    const uint32_t last = (uint32_t)__builtin_amdgcn_ballot_w64(lane < n_pieces && before == (uint32_t)parts.n - 1u);
    if (!last) continue;
    auto done = [&](int32_t x, const Sum& s) __attribute__((always_inline)) {
      if (x < h1 * F && (last >> ((x / F >> shift) - p0) & 1u)) write_out<D>(pv, out, a, b, g, g_first, x, s);
    };
    const int32_t x = h0 * F + lane;
    if ((h1 - h0) * F <= 64) {
      Sum s[1];
      all.template sum<1, 4, 16>(s, x, 0, 0, parts.n);
      done(x, s[0]);
    } else {
      for (int32_t at = x; at - lane < h1 * F; at += 128) {
        Sum s[2];
        all.template sum<2, 4, 8>(s, at, 64, 0, parts.n);
        done(at, s[0]);
        done(at + 64, s[1]);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// decode attention, partial pass (split-K), for 1, 2, 4 and 8 q heads per kv head and chunks that whole
// tiles fill (see tile_kernel): one wave per equal share of a kv head's tiles
//
// A tile is up to 64 consecutive rows of one chunk of one (request, kv head). A wave walks its
// share tile by tile; where a request ends inside the share it writes that request's partial
// result, takes the next request's query, and goes on without letting its loads run dry: the next
// request's first K tile is already in flight by then. Per tile:
//   K  64 rows are fetched with coalesced 128-bit loads (LPR = D/8 lanes per row) that write straight
//      into LDS (no staging registers), then read back transposed: lane t owns token t and reads
//      its whole row, so a score needs no cross-lane reduction. The query values of the G heads of
//      the group stay in registers, one packed bf16 pair per lane and 16 lanes per row sharing a
//      register; v_dot2_f32_bf16 with a DPP row broadcast multiplies two pairs per lane-op.
//   softmax  one score per lane and head; the tile maximum is a wave reduction; weights are
//      rounded to bf16 (the running sum l uses the rounded weights, so they still sum to one)
//      and handed to the PV layout by cross-lane reads.
//   V  is consumed straight from registers in the load layout (lane = 8 dims of one row, RPW rows
//      per wave-wide load): rows of two consecutive loads are interleaved with v_perm_b32 so that
//      one v_dot2_f32_bf16 adds two tokens' contributions to a dim.
// V of the tile is in flight while its scores are computed, K of the next tile while V is multiplied.
// Scores are kept in log2 units (scale_log2 = scale * log2 e).
// ---------------------------------------------------------------------------------------------
template <int D, int G, bool APPEND, bool DIRECT, class Args>
__device__ __forceinline__ void decode_tile_body(const PoolView& pv, const uint16_t* __restrict__ q,
                                                    const uint4* __restrict__ k_new, const uint4* __restrict__ v_new,
                                                    float* __restrict__ ws, uint16_t* __restrict__ out, float scale_log2,
                                                    int32_t g_first, const Args& a, int32_t workgroup) {
  constexpr int NW = SHARE_WAVES;
  constexpr int LPR = D / 8;             // lanes per row = 16-byte pieces per row
  constexpr int RPW = 64 / LPR;          // rows per wave-wide load
  constexpr int NL = 64 / RPW;           // wave-wide loads per 64-row tile and plane
  constexpr int ROWB = D * 2;            // bytes per row
  constexpr int QR = D / 32;             // registers holding one head's query (16 lanes x 1 pair each)
  // With 4 or 8 q heads per kv head the two products of a tile are small dense contractions, [G x D] by
  // [D x 64 tokens] and [G x 64 tokens] by [64 x D], and on ordinary lanes, with one wave per SIMD, the
  // 8-head instance's arithmetic takes longer than the tile's bytes take to arrive (70B-shaped layer:
  // 1.07 ms, against 0.86 ms with either product switched off, which is also what a kernel that only
  // reads the same tiles takes). Those instances form both products on the matrix cores, 4 heads by 4
  // tokens (or dims) by 4 at a time; the 1- and 2-head instances, which are not short of lane time,
  // keep the dot products on ordinary lanes. The softmax is on ordinary lanes in all of them.
  constexpr bool MFMA_QK = (G % 4 == 0);
  // For the weighted sum of V a lane then owns NL consecutive rows of the tile instead of every RPW-th
  // one, so that four of its rows at a time are the contraction index of one product; the tile's
  // weights reach it through a small transposed copy in LDS.
  constexpr bool MFMA_PV = (G % 4 == 0);
  __shared__ __attribute__((aligned(16))) uint16_t sm_p_all[NW][MFMA_PV ? G * 64 : 8];   // weights [head][token], bf16
  __shared__ __attribute__((aligned(16))) char sm_k_all[NW][64 * ROWB];      // the K tile being scored
  __shared__ __attribute__((aligned(16))) Results<D, G> results;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Records<Args> records(a, lane);
  wanted(a.n_req, a.waves_per_head, a.units_each, a.units_extra, a.by_waves.mul, a.by_waves.shift, a.q_row0, g_first);
  wanted(pv.chunk_bytes, pv.tokens_per_chunk, pv.tiles_per_chunk, pv.max_slots, pv.n_q_heads, pv.n_kv_heads, pv.group, q);
  wanted(pv.base, pv.table, pv.vbase, k_new, pv.by_chunk.mul, pv.by_chunk.shift, pv.by_tiles.mul, pv.by_tiles.shift);
  uint16_t* const sm_p = sm_p_all[wave];
  char* const sm_k = sm_k_all[wave];
  const int sub = lane % LPR, rg = lane / LPR;
  const int32_t Tc = pv.tokens_per_chunk;
  const uint64_t plane = (uint64_t)Tc * ROWB;        // V plane follows the K plane of the same head

  // Tile loads. Lane (rg, sub) handles piece `sub` of tile rows RPW*u + rg, u = 0 .. NL-1. Rows past
  // nv are replaced by row nv - 1, so every load is in bounds and returns finite data; those
  // rows are masked later (score -inf, weight 0).
  // K goes straight from global memory into LDS (one 16-byte slot per lane, slots in lane order, so a
  // wave-wide load fills RPW consecutive LDS rows). To make the transposed reads conflict-free the
  // swizzle is applied on the source side: LDS slot (row, c) receives piece c ^ (row % LPR).
  const int sx = sub ^ rg;    // (RPW*u + rg) % LPR == ((RPW*u) % LPR) | rg
  const int kswz = lane % LPR;
#define ELLM_LOAD_K_TILE(base, nvalid)                                                              \
  _Pragma("unroll") for (int u = 0; u < NL; u++) {                                                  \
    const uint32_t off_ = (uint32_t)min(RPW * u + rg, (nvalid) - 1) * ROWB +                        \
                          (uint32_t)((sx ^ ((RPW * u) % LPR)) * 16);                                \
    __builtin_amdgcn_global_load_lds((global_cptr_t)((base) + off_),                                \
                                     (lds_ptr_t)(sm_k + u * (RPW * ROWB)), 16, 0, CPOL_NT);         \
  }
// V: tile row that lane (rg, sub) holds in register u of a tile
#define ELLM_VROW(u) (MFMA_PV ? NL * rg + (u) : RPW * (u) + rg)
#define ELLM_LOAD_TILE(dst, base, nvalid)                                                           \
  _Pragma("unroll") for (int u = 0; u < NL; u++) {                                                  \
    const uint32_t off_ = (uint32_t)min(ELLM_VROW(u), (nvalid) - 1) * ROWB + sub * 16;              \
    dst[u] = load_stream16((base) + off_);                                                          \
  }
// Move the cursor to the next tile of the share and compute its address and valid rows. `left`
// counts the tiles of the cursor's request from the cursor tile on; when it is 1 the next tile is
// the first one of the next request.
#define ELLM_NEXT_TILE()                                                                            \
  if (left == 1) {                                                                                  \
    cb += 1;                                                                                        \
    const typename Args::Req nx_ = a.req[cb];                                                           \
    len = nx_.len;                                                                                  \
    left = units_of(len, pv, pv.tiles_per_chunk, TILE_TOKENS);                                                   \
    c_np = nx_.n_part;                                                                              \
    walk = tensor_walk<DIRECT>(pv, nx_.tensor);                                                     \
    slot = 0;                                                                                       \
    r = 0;                                                                                          \
  } else {                                                                                          \
    left -= 1;                                                                                      \
    r += TILE_TOKENS;                                                                               \
    if (r >= Tc) { r = 0; slot += 1; }                                                              \
  }                                                                                                 \
  nv_c = min(TILE_TOKENS, min(Tc - r, len - (slot * Tc + r)));                                      \
  kb = chunk_addr<DIRECT>(pv, walk, slot) + ((uint64_t)(g * 2) * Tc + r) * ROWB;
// scores of one tile (lane = token) and online softmax: leaves the tile's weights, rounded to bf16,
// in pu[] (one per head, for this lane's token). Consecutive dot products go to different heads'
// accumulators, so no instruction waits for the one before it.
#define ELLM_TILE_SCORES(nvalid)                                                                    \
  float s[G];                                                                                       \
  uint32_t pu[G];                                                                                   \
  bf16x4_bits_t wa[MFMA_PV ? NL / 4 : 1];                                                           \
  {                                                                                                 \
    if constexpr (MFMA_QK) {                                                                        \
      /* v_mfma_f32_4x4x4 (16 blocks of 4 lanes): block b computes D[i][j] = sum_k A[i][k] B[k][j] */ \
      /* with A[i][.] in lane 4b + i, B[.][j] in lane 4b + j and D[i][j] in register i of lane    */ \
      /* 4b + j. B = this lane's K row, four dims at a time, so column j of block b is token      */ \
      /* 4b + j = lane; A = the query rows of four heads, taken by all blocks from the block that */ \
      /* holds them (lanes 0..3: heads 0..3, lanes 4..7: heads 4..7). D: register i = score of    */ \
      /* head i for this lane's token, the layout the softmax below expects.                      */ \
      f32x4_t sacc[G / 4];                                                                          \
      _Pragma("unroll") for (int h = 0; h < G / 4; h++) sacc[h] = f32x4_t{0.f, 0.f, 0.f, 0.f};      \
      static_for<0, LPR>([&](auto jc) {                                                             \
        constexpr int j = decltype(jc)::value;                                                      \
        const uint4 kp = *reinterpret_cast<const uint4*>(sm_k + lane * ROWB + ((j ^ kswz) * 16));   \
        const bf16x4_bits_t k0 = __builtin_bit_cast(bf16x4_bits_t, make_uint2(kp.x, kp.y));         \
        const bf16x4_bits_t k1 = __builtin_bit_cast(bf16x4_bits_t, make_uint2(kp.z, kp.w));         \
        static_for<0, G / 4>([&](auto hc) {                                                         \
          constexpr int h = decltype(hc)::value;                                                    \
          sacc[h] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(qa[2 * j], k0, sacc[h], 4, h, 0);        \
        });                                                                                         \
        static_for<0, G / 4>([&](auto hc) {                                                         \
          constexpr int h = decltype(hc)::value;                                                    \
          sacc[h] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(qa[2 * j + 1], k1, sacc[h], 4, h, 0);    \
        });                                                                                         \
      });                                                                                           \
      _Pragma("unroll") for (int h = 0; h < G / 4; h++) {                                           \
        s[4 * h + 0] = sacc[h][0]; s[4 * h + 1] = sacc[h][1];                                       \
        s[4 * h + 2] = sacc[h][2]; s[4 * h + 3] = sacc[h][3];                                       \
      }                                                                                             \
    } else {                                                                                        \
      _Pragma("unroll") for (int i = 0; i < G; i++) s[i] = 0.f;                                     \
      static_for<0, LPR>([&](auto jc) {                                                             \
        constexpr int j = decltype(jc)::value;                                                      \
        const uint4 kp = *reinterpret_cast<const uint4*>(sm_k + lane * ROWB + ((j ^ kswz) * 16));   \
        _Pragma("unroll") for (int i = 0; i < G; i++)                                               \
          s[i] = dot2_bf16_rowlane<4 * (j % 4) + 0>(qreg[i][j / 4], kp.x, s[i]);                    \
        _Pragma("unroll") for (int i = 0; i < G; i++)                                               \
          s[i] = dot2_bf16_rowlane<4 * (j % 4) + 1>(qreg[i][j / 4], kp.y, s[i]);                    \
        _Pragma("unroll") for (int i = 0; i < G; i++)                                               \
          s[i] = dot2_bf16_rowlane<4 * (j % 4) + 2>(qreg[i][j / 4], kp.z, s[i]);                    \
        _Pragma("unroll") for (int i = 0; i < G; i++)                                               \
          s[i] = dot2_bf16_rowlane<4 * (j % 4) + 3>(qreg[i][j / 4], kp.w, s[i]);                    \
      });                                                                                           \
      _Pragma("unroll") for (int i = 0; i < G; i++) settle(s[i]);                                   \
    }                                                                                               \
    _Pragma("unroll") for (int i = 0; i < G; i++) {                                                 \
      const float sc = lane < (nvalid) ? s[i] * scale_log2 : -INFINITY;                             \
      /* the running maximum is the same in every lane: it lives in a scalar register */           \
      const float mn = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(fmaxf(m[i], wave_max(sc))))); \
      const float alpha = fast_exp2(m[i] - mn);                                                     \
      m[i] = mn;                                                                                    \
      pu[i] = __float_as_uint(fast_exp2(sc - mn));                                                  \
      pu[i] = (pu[i] + 0x7fffu + ((pu[i] >> 16) & 1u)) & 0xffff0000u; /* nearest even */            \
      l[i] = l[i] * alpha + __uint_as_float(pu[i]);                                                 \
      if constexpr (MFMA_PV) { _Pragma("unroll") for (int e = 0; e < 8; e++) accv[i / 4][e][i % 4] *= alpha; } \
      else { _Pragma("unroll") for (int e = 0; e < 8; e++) acc[i][e] *= alpha; }                    \
    }                                                                                               \
    if constexpr (MFMA_PV) {                                                                        \
      /* the tile's weights through LDS, transposed to [head][token], so that lane (rg, sub) gets  */ \
      /* the weights of its own NL consecutive rows for head sub % G. Done here, while no          */ \
      /* load-to-LDS is pending, so that these LDS reads do not have to wait for one.              */ \
      _Pragma("unroll") for (int i = 0; i < G; i++) sm_p[i * 64 + lane] = (uint16_t)(pu[i] >> 16);  \
      __builtin_amdgcn_wave_barrier();                                                              \
      const uint2* src_ = reinterpret_cast<const uint2*>(sm_p + (sub % G) * 64 + NL * rg);          \
      _Pragma("unroll") for (int mm = 0; mm < NL / 4; mm++) wa[mm] = __builtin_bit_cast(bf16x4_bits_t, src_[mm]); \
      __builtin_amdgcn_wave_barrier();                                                              \
    }                                                                                               \
  }
// weighted V: the PV lane (rg, sub) fetches the weights of its rows RPW*u + rg from the lanes that
// own those tokens (a cross-lane read, no LDS memory), packs two of them into one register, and
// adds two tokens per dot2
#define ELLM_TILE_PV(VR)                                                                            \
  if constexpr (MFMA_PV) {                                                                          \
    /* wa[mm] (set up with the scores): for head sub % G, the weights of rows 4 mm .. 4 mm + 3 of  */ \
    /* this lane's NL rows = one A operand. A[i][k] is looked up in lane 4b + i of the block named */ \
    /* by abid within each group of LPR / 4 blocks (the lanes of one row-group): block 0 holds     */ \
    /* heads 0..3, block 1 heads 4..7.                                                             */ \
    /* B[k][j] = four rows' values of one dim of lane 4b + j; D[i][j] = head i, that dim.          */ \
    constexpr int CB = (LPR == 16) ? 2 : 1;     /* log2 of the blocks that share one A */          \
    static_for<0, NL / 4>([&](auto mc) {                                                            \
      constexpr int mm = decltype(mc)::value;                                                       \
      const uint4 r0 = VR[4 * mm], r1 = VR[4 * mm + 1], r2 = VR[4 * mm + 2], r3 = VR[4 * mm + 3];   \
      static_for<0, 8>([&](auto ec) {                                                               \
        constexpr int e = decltype(ec)::value;                                                      \
        constexpr uint32_t sel = (e % 2) ? 0x07060302u : 0x05040100u;                               \
        const uint32_t w0 = e / 2 == 0 ? r0.x : e / 2 == 1 ? r0.y : e / 2 == 2 ? r0.z : r0.w;       \
        const uint32_t w1 = e / 2 == 0 ? r1.x : e / 2 == 1 ? r1.y : e / 2 == 2 ? r1.z : r1.w;       \
        const uint32_t w2 = e / 2 == 0 ? r2.x : e / 2 == 1 ? r2.y : e / 2 == 2 ? r2.z : r2.w;       \
        const uint32_t w3 = e / 2 == 0 ? r3.x : e / 2 == 1 ? r3.y : e / 2 == 2 ? r3.z : r3.w;       \
        const bf16x4_bits_t vb = __builtin_bit_cast(                                                \
            bf16x4_bits_t, make_uint2(__builtin_amdgcn_perm(w1, w0, sel), __builtin_amdgcn_perm(w3, w2, sel))); \
        static_for<0, G / 4>([&](auto hc) {                                                         \
          constexpr int h = decltype(hc)::value;                                                    \
          accv[h][e] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(wa[mm], vb, accv[h][e], CB, h, 0);    \
        });                                                                                         \
      });                                                                                           \
    });                                                                                             \
  } else {                                                                                          \
  _Pragma("unroll") for (int i = 0; i < G; i++) {                                                   \
    uint32_t pp[NL / 2];                                                                            \
    _Pragma("unroll") for (int v = 0; v < NL / 2; v++) {                                            \
      const uint32_t pa = __builtin_amdgcn_ds_bpermute((RPW * (2 * v) + rg) * 4, pu[i]);            \
      const uint32_t pb = __builtin_amdgcn_ds_bpermute((RPW * (2 * v + 1) + rg) * 4, pu[i]);        \
      pp[v] = __builtin_amdgcn_perm(pb, pa, 0x07060302u);                                           \
    }                                                                                               \
    _Pragma("unroll") for (int v = 0; v < NL / 2; v++) {                                            \
      const uint4 A = VR[2 * v], Bv = VR[2 * v + 1];                                                \
      acc[i][0] = dot2_bf16(__builtin_amdgcn_perm(Bv.x, A.x, 0x05040100u), pp[v], acc[i][0]);       \
      acc[i][1] = dot2_bf16(__builtin_amdgcn_perm(Bv.x, A.x, 0x07060302u), pp[v], acc[i][1]);       \
      acc[i][2] = dot2_bf16(__builtin_amdgcn_perm(Bv.y, A.y, 0x05040100u), pp[v], acc[i][2]);       \
      acc[i][3] = dot2_bf16(__builtin_amdgcn_perm(Bv.y, A.y, 0x07060302u), pp[v], acc[i][3]);       \
      acc[i][4] = dot2_bf16(__builtin_amdgcn_perm(Bv.z, A.z, 0x05040100u), pp[v], acc[i][4]);       \
      acc[i][5] = dot2_bf16(__builtin_amdgcn_perm(Bv.z, A.z, 0x07060302u), pp[v], acc[i][5]);       \
      acc[i][6] = dot2_bf16(__builtin_amdgcn_perm(Bv.w, A.w, 0x05040100u), pp[v], acc[i][6]);       \
      acc[i][7] = dot2_bf16(__builtin_amdgcn_perm(Bv.w, A.w, 0x07060302u), pp[v], acc[i][7]);       \
    }                                                                                               \
  }                                                                                                 \
  }

// query of request b_. Lanes: lane keeps pair (16 c + lane % 16) of each head in qreg[.][c]. Matrix
// cores: lane i < G keeps the whole row of head i, four dims per entry of qa (the other lanes' copies
// are never looked at; they read the last head's row, which is in bounds)
#define ELLM_LOAD_Q(b_)                                                                             \
  if constexpr (MFMA_QK) {                                                                          \
    const uint4* qsrc = reinterpret_cast<const uint4*>(                                             \
        q + ((int64_t)(a.q_row0 + (b_)) * pv.n_q_heads + hq0 + min(lane, G - 1)) * D);              \
    _Pragma("unroll") for (int c = 0; c < LPR; c++) {                                               \
      const uint4 t_ = qsrc[c];                                                                     \
      qa[2 * c] = __builtin_bit_cast(bf16x4_bits_t, make_uint2(t_.x, t_.y));                        \
      qa[2 * c + 1] = __builtin_bit_cast(bf16x4_bits_t, make_uint2(t_.z, t_.w));                    \
    }                                                                                               \
  } else {                                                                                          \
    const uint32_t* qsrc =                                                                          \
        reinterpret_cast<const uint32_t*>(q + ((int64_t)(a.q_row0 + (b_)) * pv.n_q_heads + hq0) * D); \
    _Pragma("unroll") for (int i = 0; i < G; i++)                                                   \
      _Pragma("unroll") for (int c = 0; c < QR; c++) qreg[i][c] = qsrc[i * (D / 2) + c * 16 + (lane & 15)]; \
  }
// Fused append: len counts the new token already, but its K/V row is still in k_new / v_new. The wave
// that reaches the end of a request's sequence takes that row from there (lane's 16-byte piece `sub`
// of each), puts it where the last tile's loads would have found it, and writes it to the chunk.
#define ELLM_LOAD_NEW_ROW(b_)                                                                       \
  if (APPEND) {                                                                                     \
    const int64_t row16 = ((int64_t)(a.q_row0 + (b_)) * pv.n_kv_heads + g) * LPR + sub;             \
    kn = k_new[row16];                                                                              \
    vn = v_new[row16];                                                                              \
  }

  results.clear(wave, lane);             // (behind the first loads it is slower: LDS writes wait for loads to LDS)
  const int32_t index = workgroup * NW + wave;
  if (index < a.waves_per_head * pv.n_kv_heads) {
    const Share<Args> sh = locate_share(a, records, index, lane);
    const int32_t g = sh.g, n_tiles = sh.n_units;
    const int hq0 = g * pv.group + g_first;            // first q head handled here
    // cursor: the tile whose K is in LDS or on its way there. cb: its request; len, walk: that
    // request's length and its table row or base address (read-only for the kernel's lifetime: uniform loads)
    int32_t cb = sh.b;
    const typename Args::Req& first = sh.first;
    int32_t len = first.len;
    TensorWalk walk = tensor_walk<DIRECT>(pv, first.tensor);
    const int32_t tile0 = sh.u_lo - first.unit_prefix;
    int32_t left = units_of(len, pv, pv.tiles_per_chunk, TILE_TOKENS) - tile0;
    int32_t slot = divide(tile0, pv.by_tiles);
    int32_t r = (tile0 - slot * pv.tiles_per_chunk) * TILE_TOKENS;
    int32_t nv_c = min(TILE_TOKENS, min(Tc - r, len - (slot * Tc + r)));
    const char* kb = chunk_addr<DIRECT>(pv, walk, slot) + ((uint64_t)(g * 2) * Tc + r) * ROWB;
    ELLM_LOAD_K_TILE(kb, nv_c)

    // the request being accumulated, and how many waves share it (c_np: the same for the cursor's
    // request, which runs one tile ahead)
    int32_t b = cb, b_np = first.n_part, c_np = b_np;
    uint32_t qreg[MFMA_QK ? 1 : G][QR];
    bf16x4_bits_t qa[MFMA_QK ? 2 * LPR : 1];
    uint4 kn, vn;
    ELLM_LOAD_Q(b)
    ELLM_LOAD_NEW_ROW(b)

    float m[G], l[G], acc[G][8];
    f32x4_t accv[MFMA_PV ? G / 4 : 1][8];      // matrix cores: accv[h][e][i] = head 4h + i, dim 8 sub + e
#pragma unroll
    for (int i = 0; i < G; i++) {
      m[i] = NEG_BIG; l[i] = 0.f;
#pragma unroll
      for (int e = 0; e < 8; e++) acc[i][e] = 0.f;
    }
#pragma unroll
    for (int h = 0; h < (MFMA_PV ? G / 4 : 1); h++)
#pragma unroll
      for (int e = 0; e < 8; e++) accv[h][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    bool q_settled = false;

    for (int32_t it = 0; it < n_tiles; it++) {
      // the K tile (and, after a change of request, the query) is all that is outstanding here:
      // wait until it has landed in LDS, then start this tile's V, which stays in flight while the
      // scores are computed
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
      __builtin_amdgcn_wave_barrier();
      const int32_t nv = nv_c;
      const bool last = left == 1;         // this tile ends its request
      const bool more = it + 1 < n_tiles;
      uint4 vr[NL];
      ELLM_LOAD_TILE(vr, kb + plane, nv)
      if (APPEND && last) {
        // the new token is row nv - 1 of this tile: K goes into the LDS tile (same swizzle as the
        // loads) and both rows go to the chunk; V replaces what the loads fetched for that row once
        // they have arrived
        const int rl = nv - 1;
        if (rg == 0) {
          *reinterpret_cast<uint4*>(sm_k + rl * ROWB + ((sub ^ (rl % LPR)) * 16)) = kn;
          char* dst = const_cast<char*>(kb) + (uint32_t)rl * ROWB + sub * 16;
          *reinterpret_cast<uint4*>(dst) = kn;
          *reinterpret_cast<uint4*>(dst + plane) = vn;
        }
      }
      if (!MFMA_QK && !q_settled) {
#pragma unroll
        for (int i = 0; i < G; i++)
#pragma unroll
          for (int c = 0; c < QR; c++) settle(qreg[i][c]);
        q_settled = true;
      }
      ELLM_TILE_SCORES(nv)
      // where the next tile is: scalar work, done while V is still on its way
      if (more) {
        ELLM_NEXT_TILE()
      }
      // V of this tile must have arrived now (it is the only load outstanding); then the K tile,
      // which has been consumed, is replaced by the next one while V is multiplied
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
      if (APPEND && last) {
#pragma unroll
        for (int u = 0; u < NL; u++)
          if (ELLM_VROW(u) >= nv - 1) vr[u] = vn;
      }
      if (more) {
        ELLM_LOAD_K_TILE(kb, nv_c)
      }
      __builtin_amdgcn_sched_barrier(0);
      ELLM_TILE_PV(vr)

      if (last || !more) {
        // request b ends here, or the share does: write partial j of pair (b, g).
        // Every row-group holds the same dims for different tokens under one common maximum: add them up
        if constexpr (MFMA_PV) {
#pragma unroll
          for (int i = 0; i < G; i++)
#pragma unroll
            for (int e = 0; e < 8; e++) acc[i][e] = accv[i / 4][e][i % 4];
        }
#pragma unroll
        for (int i = 0; i < G; i++) {
#pragma unroll
          for (int e = 0; e < 8; e++) {
            if (LPR < 16) acc[i][e] += __shfl_xor(acc[i][e], 8);
            acc[i][e] = add_xor32(add_xor16(acc[i][e]));
          }
          l[i] = wave_sum(l[i]);
        }
        if (b_np == 1) {
          // the whole request lay inside this wave's share: this is the final result. Normalise, round
          // and write the output rows
          if (rg == 0) {
#pragma unroll
            for (int i = 0; i < G; i++) {
              const float li = l[i];
              uint32_t w[4];
#pragma unroll
              for (int e = 0; e < 4; e++)
                w[e] = f32_to_bf16_bits((acc[i][2 * e] + 0.f) / li) | (f32_to_bf16_bits((acc[i][2 * e + 1] + 0.f) / li) << 16);
              uint16_t* o = out + ((int64_t)(a.q_row0 + b) * pv.n_q_heads + hq0 + i) * D + sub * 8;
              *reinterpret_cast<uint4*>(o) = make_uint4(w[0], w[1], w[2], w[3]);
            }
          }
        } else {
          // one of several waves of the request: its results meet the others' in LDS
          // (dims in the order in which the lanes of a row store neighbouring 16-byte pieces)
          const int32_t to = 2 * wave + (b == sh.b ? 0 : 1);
          if (rg == 0) {
#pragma unroll
            for (int i = 0; i < G; i++)
#pragma unroll
              for (int h = 0; h < 2; h++)
                results.rows[to][i][h * LPR + sub] = make_float4(acc[i][4 * h], acc[i][4 * h + 1], acc[i][4 * h + 2], acc[i][4 * h + 3]);
            float mm = m[0], ll = l[0];       // lane `sub` writes head sub's pair
#pragma unroll
            for (int i = 1; i < G; i++)
              if (sub == i) { mm = m[i]; ll = l[i]; }
            if (sub < G) results.ml[to][sub] = make_float2(mm, ll);
            if (sub == 0) results.whose[to] = g * MAX_LAUNCH_REQ + b;
          }
        }
        if (more) {
          // the cursor is already in the next request, whose first tile this wave holds
          b = cb;
          b_np = c_np;
          ELLM_LOAD_Q(b)
          ELLM_LOAD_NEW_ROW(b)
          q_settled = false;
#pragma unroll
          for (int i = 0; i < G; i++) {
            m[i] = NEG_BIG; l[i] = 0.f;
#pragma unroll
            for (int e = 0; e < 8; e++) acc[i][e] = 0.f;
          }
#pragma unroll
          for (int h = 0; h < (MFMA_PV ? G / 4 : 1); h++)
#pragma unroll
            for (int e = 0; e < 8; e++) accv[h][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
  }
  end_shares<D, G>(pv, ws, out, a, records, results, g_first, G, workgroup, wave, lane);
#undef ELLM_LOAD_Q
#undef ELLM_LOAD_NEW_ROW
#undef ELLM_LOAD_TILE
#undef ELLM_VROW
#undef ELLM_LOAD_K_TILE
#undef ELLM_NEXT_TILE
#undef ELLM_TILE_SCORES
#undef ELLM_TILE_PV
}

// Launched with one wave per SIMD, so a wave may use the SIMD's whole register file. The instances
// for 1 and 2 q heads per kv head fit the budget of two waves per SIMD with room to spare and keep
// that cap (it is what their schedule was tuned under); the 4- and 8-head instances, which keep the
// whole query rows and the matrix-core accumulators in registers, are compiled without it and do
// not spill.
template <int D, int G, bool APPEND, bool DIRECT, class Args>
__global__ __launch_bounds__(64 * SHARE_WAVES) __attribute__((amdgpu_waves_per_eu(2))) void decode_tile_kernel(
    PoolView pv, const uint16_t* __restrict__ q, const uint4* __restrict__ k_new, const uint4* __restrict__ v_new,
    float* __restrict__ ws, uint16_t* __restrict__ out, float scale_log2, int32_t g_first, Args a) {
  in_launch(pv, ws, a, [&](const PoolView& pv, float* ws, const auto& a, int32_t workgroup) __attribute__((always_inline)) {
    decode_tile_body<D, G, APPEND, DIRECT>(pv, q, k_new, v_new, ws, out, scale_log2, g_first, a, workgroup);
  });
}
template <int D, int G, bool APPEND, bool DIRECT, class Args>
__global__ __launch_bounds__(64 * SHARE_WAVES) __attribute__((amdgpu_waves_per_eu(1, 1))) void decode_tile_kernel_wide(
    PoolView pv, const uint16_t* __restrict__ q, const uint4* __restrict__ k_new, const uint4* __restrict__ v_new,
    float* __restrict__ ws, uint16_t* __restrict__ out, float scale_log2, int32_t g_first, Args a) {
  in_launch(pv, ws, a, [&](const PoolView& pv, float* ws, const auto& a, int32_t workgroup) __attribute__((always_inline)) {
    decode_tile_body<D, G, APPEND, DIRECT>(pv, q, k_new, v_new, ws, out, scale_log2, g_first, a, workgroup);
  });
}

// ---------------------------------------------------------------------------------------------
// decode attention, partial pass (split-K), for every other group and chunk size: one wave per equal share
// of a kv head's units
//
// A unit is up to UNIT_TOKENS = 16 consecutive rows of one chunk of one (request, kv head); a tile is
// up to U units of one request, not necessarily of one chunk. A wave walks its share tile by tile:
// the next tile's K is asked for as soon as this one's scores are formed, its V as soon as this one's
// weighted sum is, so that one of the two is on its way at any time.
//   scores   S^T = K Q^T by 16x16x32 matrix instructions, one unit by up to 16 q heads: A = the unit's
//      rows (lane 16 g + c: 16 bytes of one row per product), B = the query rows (lane: head c, the same
//      bytes of it). To load whole cache lines a wave-wide load takes 128 bytes of each of 8 rows instead
//      of 64 of 16: with c1 the second-lowest bit of c, load j of a half row gives lane (g, c) piece
//      g + 4 (c1 ^ j) of row 4 (c & 1) + (c >> 2) + 8 j. Product x takes, per lane, load c1 ^ x: the same
//      piece g + 4 x in every lane, of row 4 (c & 1) + (c >> 2) + 8 (c1 ^ x). A's lane c = 4 g + i becomes
//      register i of lane group g, so product 0 leaves the score of token 4 i + g for head c in register i of
//      lane (g, c), and product 1 the score of token 4 (i ^ 2) + g: an exchange of registers i and i ^ 2.
//   softmax  a lane owns one head (c) and four tokens of every unit: the tile's maximum is lane-local up
//      to two cross-lane swaps, and the weights are already where the next product wants them: as the sum
//      of two bf16 values, the next one below the weight and the rest (to 2^-16 of the weight; both
//      positive, so an infinite V stays infinite), one product each. With the weights rounded to one bf16
//      value the result is as far from 64 bits as the tile kernels' (2.1e-3 instead of 1.6e-3, the
//      rounding of the result included), and further where those cut a request more finely.
//   PV       O^T = V^T P^T, two units at a time: contraction index of lane group g = its four tokens of
//      either unit. A = V, loaded as whole rows (lane (g, c): dims E c .. E c + E - 1 of rows 4 i + g) and
//      transposed in registers by v_perm_b32, one product per e = dim % E; B = the weights.
//      Register i of product e in lane (g, c) is dim E (4 g + i) + e of head c: every per-head quantity
//      (m, l, the rescaling) sits in the lanes that need it, and a lane ends with 4 E consecutive dims.
// K, V and the weights do not go through LDS (results that several waves share do). The cost per byte does not depend on the number of q heads up to 16, so every
// group size up to that is one pass over K and V. Bound by HBM: 48 requests of 6 q heads per kv head (278 MB
// of K and V) 92.4 -> 51.8 us with a combine pass (the tile kernels read K and V twice), 64 requests of 16
// heads of 64 (398 MB) 144 -> 69.8, 16-token chunks (187 MB) 50.8 -> 36.4.
// Tried on these and on the 8B-shaped layer: two or three tiles in registers (no faster, and what does not
// fit 256 registers goes through accumulation registers: 2 to 4 % slower); tiles of 64 tokens (pages
// 37.4); K in 64-byte pieces of 16 rows (16 heads of 64: 77), in whole rows of 4 (no change, more
// exchanges); an exit between a tile's loads (the compiler then waits for everything in flight).
// Scores are kept in log2 units (scale_log2 = scale * log2 e).
// ---------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef const __attribute__((address_space(1))) char* gptr_t;
typedef __attribute__((address_space(1))) char* gwptr_t;

__device__ __forceinline__ f32x4_t mfma16(words4_t a, words4_t b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

enum : uint32_t { T_FIRST = 1, T_LAST = 2, T_FIN = 4 };   // a tile starts a request here, ends it, ends the share
// the largest bf16 value below a positive float, as a float's bits; 0 for 0, NaN for NaN
__device__ __forceinline__ uint32_t bf16_below(float p) {
  return __builtin_elementwise_sub_sat(__float_as_uint(p), 1u) & 0xffff0000u;
}

template <int U>
struct TileInfo {                    // what is known of a tile before its loads are issued (uniform)
  int32_t n, b, part;                // units, request, partial slot of the request in this wave (-1: finished here)
  uint32_t flags;                    // T_*
  int32_t tail;                      // rows of its last unit
  int32_t nv[U];                     // rows of each unit (0: the tile has no such unit)
  int32_t r[U];                      // first row of the unit in its chunk
  uint32_t at[U];                    // its chunk (table entry, or slot of the tensor's own range)
  const char* base;                  // start of the pool, or of the tensor's range
};

// units per tile: 8 KB of K and 8 KB of V for either head size
template <int D> constexpr int tile_units = D == 128 ? 2 : 4;

// NW == 0: a wave walks its share, SW of them are a workgroup; SW == 1: single_waves(). NW > 0 (small launches): NW waves share a step of up to NW * U units of one
// request, one tile each, everything asked for at once, and add up through LDS.
template <int D, int U, bool APPEND, bool DIRECT, int NW, int SW, class Args>
__device__ __forceinline__ void decode_unit_body(const PoolView& pv, const uint16_t* __restrict__ q,
                                            const char* __restrict__ k_new, const char* __restrict__ v_new,
                                            float* __restrict__ ws, uint16_t* __restrict__ out, float scale_log2,
                                            int32_t g_first, int32_t n_heads, const Args& a, int32_t workgroup) {
  constexpr int P = D / 32;          // products along a row = 16-byte pieces of K, dwords of a V row, per lane
  constexpr int ROWB = D * 2, E = D / 16, VB = E * 2;
  static_assert(U % 2 == 0, "PV takes two units at a time");
  const int lane = threadIdx.x & 63, c = lane & 15, g16 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Records<Args> records(a, lane);
  wanted(a.n_req, a.waves_per_head, a.units_each, a.units_extra, a.by_waves.mul, a.by_waves.shift, a.step_units, a.q_row0);
  // (what only the table's way reads stays out of the others: kept in registers with its neighbours it made
  // decode_unit_kernel<64, 4, 4, append, direct> spill 20 scalar registers; 64 requests of 100 to 900 tokens 20.80 -> 20.68 us a call)
  wanted(pv.chunk_bytes, pv.tokens_per_chunk, pv.units_per_chunk, DIRECT ? 0 : pv.max_slots, pv.n_q_heads, pv.n_kv_heads, pv.group, g_first);
  wanted(DIRECT ? nullptr : pv.base, DIRECT ? nullptr : pv.table, pv.vbase, q, pv.by_chunk.mul, pv.by_chunk.shift, pv.by_units.mul, pv.by_units.shift);
  const int32_t Tc = pv.tokens_per_chunk;
  const uint64_t plane = (uint64_t)Tc * ROWB;        // V plane follows the K plane of the same head

  const int32_t index = NW ? workgroup : workgroup * SW + wave;
  const Share<Args> sh = locate_share(a, records, NW ? index : min(index, a.waves_per_head * pv.n_kv_heads - 1), lane);
  const int32_t g = sh.g;
  const int32_t hq0 = g * pv.group + g_first;        // first q head handled here
  const int32_t head = min(c, n_heads - 1);          // lanes beyond the last head repeat it and write nothing

  // ---- cursor: the next tile to be asked for ----
  int32_t cb = sh.b, rem_share = sh.n_units, len, slot, r, rem_req, part;
  uint32_t first = T_FIRST;
  TensorWalk walk;
  const typename Args::Req& first_rq = sh.first;
  {
    const typename Args::Req& rq = first_rq;
    len = rq.len;
    walk = tensor_walk<DIRECT>(pv, rq.tensor);
    constexpr int32_t STEP_WAVES = NW ? NW : 1;
    const int32_t mine = NW ? wave * a.step_units / STEP_WAVES : 0;     // (at most U apart from one wave to the next)
    const int32_t u0 = (sh.u_lo - rq.unit_prefix) * a.step_units + mine;
    rem_req = units_of(len, pv, pv.units_per_chunk) - u0;
    if (NW) rem_share = min((wave + 1) * a.step_units / STEP_WAVES - mine, rem_req);
    else if (a.step_units > 1) rem_share = min(rem_share * a.step_units, rem_req);
    slot = divide(u0, pv.by_units);
    r = (u0 - slot * pv.units_per_chunk) * UNIT_TOKENS;
    part = rq.n_part == 1 ? -1 : rq.part0 + (sh.w - rq.wave_first);    // (which slot: only where a workgroup is a step)
  }
  auto advance = [&](TileInfo<U>& t) __attribute__((always_inline)) {
    t.n = min(U, min(rem_share, rem_req));
    t.b = cb;
    t.part = part;
    t.flags = first;
    t.base = DIRECT ? walk.tbase : pv.base;
#pragma unroll
    for (int u = 0; u < U; u++) {
      if (u == 0 || u < t.n) {
        t.at[u] = DIRECT ? (uint32_t)slot : (uint32_t)walk.trow[slot];
        t.r[u] = r;
        t.nv[u] = min(UNIT_TOKENS, min(Tc - r, len - (slot * Tc + r)));
        t.tail = t.nv[u];
        if (u < t.n - 1 || (t.n > 0 && rem_req > t.n)) {   // there is a next unit of this request
          r += UNIT_TOKENS;
          if (r >= Tc) { r = 0; slot += 1; }
        }
      } else {
        t.at[u] = t.at[u - 1];
        t.r[u] = t.r[u - 1];
        t.nv[u] = 0;
      }
    }
    if (t.n == 0) t.nv[0] = 0;                       // past the end of the share
    rem_req -= t.n;
    rem_share -= t.n;
    first = 0;
    if (rem_req == 0) {
      t.flags |= T_LAST;
      first = T_FIRST;
    }
    if (rem_share == 0) t.flags |= T_FIN;
    if (rem_req == 0 && rem_share > 0) {
      cb += 1;
      const typename Args::Req rq = a.req[cb];
      len = rq.len;
      rem_req = units_of(len, pv, pv.units_per_chunk);
      walk = tensor_walk<DIRECT>(pv, rq.tensor);
      slot = 0;
      r = 0;
      part = rq.n_part == 1 ? -1 : rq.part0;
    }
  };
  auto unit_base = [&](const TileInfo<U>& t, int u) __attribute__((always_inline)) {
    return const_cast<char*>(t.base) + (uint64_t)t.at[u] * pv.chunk_bytes + ((uint64_t)(g * 2) * Tc + t.r[u]) * ROWB;
  };
  // the rows of a unit as a buffer of their own
  auto rows_of = [&](char* base, int32_t rows) __attribute__((always_inline)) {
    return buffer_at(base, rows * ROWB);
  };
  // how many of them are in the chunk: all but the one that a fused append is about to put there
  auto there = [&](const TileInfo<U>& t, int u) __attribute__((always_inline)) {
    return t.nv[u] - (APPEND && (t.flags & T_LAST) && u == t.n - 1 ? 1 : 0);
  };

  // ---- loads ----
  // Buffer loads with the unit's rows as their range: rows past its end, and units that the tile does not
  // have, come back as zeros without a memory access. So the addresses of a lane are the same for every
  // tile, a wave's last round costs no traffic for the tile after it, V rows that are not there have the
  // value their weight 0 needs, and the number of loads does not depend on the tile (the waits count them).
  words4_t k[U][P], qr[P], kn[P / 2];
  uint32_t v[U][4][P], vn[P];
  const int c1 = (c >> 1) & 1;
  // of a unit's K, load j of a half row gives this lane row krow + 8 j, 16 bytes at kpiece(j) of the half
  const int krow = 4 * (c & 1) + (c >> 2), voff = g16 * ROWB + c * VB;
  auto kpiece = [&](int32_t j) __attribute__((always_inline)) { return (uint32_t)(g16 + 4 * (c1 ^ j)) * 16; };
  // Before a tile's own rows, so that waiting for these does not mean waiting for what is asked for later:
  // with the first tile of a request its query (the one before it has had its last scores formed), and,
  // fused append, with the last one the new rows. There len counts the new token already, but its row is
  // still in k_new / v_new; the wave that reaches the end of a request's sequence takes it from there, puts
  // it where the last tile's loads would have found it, and writes it to the chunk.
  auto new_row = [&](const TileInfo<U>& t) __attribute__((always_inline)) {
    return ((int64_t)(a.q_row0 + t.b) * pv.n_kv_heads + g) * ROWB;
  };
  auto load_row = [&](__amdgpu_buffer_rsrc_t rows, int32_t at, uint32_t (&dst)[P]) __attribute__((always_inline)) {
    if constexpr (P == 4) {
      const words4_t w = __builtin_amdgcn_raw_buffer_load_b128(rows, at, 0, CPOL_NT);
      dst[0] = w.x; dst[1] = w.y; dst[2] = w.z; dst[3] = w.w;
    } else {
      const words2_t w = __builtin_amdgcn_raw_buffer_load_b64(rows, at, 0, CPOL_NT);
      dst[0] = w.x; dst[1] = w.y;
    }
  };
  auto issue_k = [&](const TileInfo<U>& t) __attribute__((always_inline)) {
    if (t.flags & T_FIRST) {
      const gptr_t qp = (gptr_t)(q + ((int64_t)(a.q_row0 + t.b) * pv.n_q_heads + hq0 + head) * D) + g16 * 16;
#pragma unroll
      for (int p = 0; p < P; p++) qr[p] = *(const __attribute__((address_space(1))) words4_t*)(qp + p * 64);
    }
    if (APPEND && (t.flags & T_LAST)) {
      const gptr_t kp = (gptr_t)(k_new + new_row(t)) + kpiece((t.tail - 1) >> 3 & 1);
#pragma unroll
      for (int h = 0; h < P / 2; h++) kn[h] = *(const __attribute__((address_space(1))) words4_t*)(kp + h * 128);
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      const auto rows = rows_of(unit_base(t, u), there(t, u));
#pragma unroll
      for (int j = 0; j < 2; j++)
#pragma unroll
        for (int h = 0; h < P / 2; h++)
          k[u][2 * h + j] = __builtin_amdgcn_raw_buffer_load_b128(rows, (krow + 8 * j) * ROWB + kpiece(j) + h * 128, 0, CPOL_NT);
    }
  };
  auto issue_v = [&](const TileInfo<U>& t) __attribute__((always_inline)) {
    if (APPEND && (t.flags & T_LAST)) load_row(rows_of(const_cast<char*>(v_new) + new_row(t), 1), c * VB, vn);
#pragma unroll
    for (int u = 0; u < U; u++) {
      const auto rows = rows_of(unit_base(t, u) + plane, there(t, u));
#pragma unroll
      for (int i = 0; i < 4; i++) load_row(rows, voff + 4 * i * ROWB, v[u][i]);
    }
  };

  // ---- arithmetic ----
  float m = NEG_BIG, l = 0.f;
  f32x4_t acc[E], s[U];
  auto scores = [&](const TileInfo<U>& t) __attribute__((always_inline)) {
    if (APPEND && (t.flags & T_LAST)) {
      // the new token's K row replaces what the loads found in its place, and goes into the chunk (a unit that
      // the tile does not have has the address of the one before it)
      const int32_t rl = t.tail - 1;
#pragma unroll
      for (int u = 0; u < U; u++)
#pragma unroll
        for (int j = 0; j < 2; j++) {
          const bool mine = u == t.n - 1 && krow + 8 * j == rl;
#pragma unroll
          for (int h = 0; h < P / 2; h++) k[u][2 * h + j] = mine ? kn[h] : k[u][2 * h + j];
        }
      if (krow == (rl & 7)) {
        const gwptr_t dst = (gwptr_t)unit_base(t, U - 1) + (uint32_t)(rl * ROWB) + kpiece(rl >> 3);
#pragma unroll
        for (int h = 0; h < P / 2; h++) *(__attribute__((address_space(1))) words4_t*)(dst + h * 128) = kn[h];
      }
    }
    const bool odd = c1 != 0;
#pragma unroll
    for (int u = 0; u < U; u++) {
      f32x4_t d0 = {0.f, 0.f, 0.f, 0.f}, d1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int h = 0; h < P / 2; h++) {
        const words4_t k0 = k[u][2 * h], k1 = k[u][2 * h + 1];
        d0 = mfma16(odd ? k1 : k0, qr[2 * h], d0);
        d1 = mfma16(odd ? k0 : k1, qr[2 * h + 1], d1);
      }
#pragma unroll
      for (int i = 0; i < 4; i++) s[u][i] = (d0[i] + d1[i ^ 2]) * scale_log2;
    }
  };
  auto weigh = [&](const TileInfo<U>& t) __attribute__((always_inline)) {
    if (t.flags & T_FIRST) {
      m = NEG_BIG;
      l = 0.f;
#pragma unroll
      for (int e = 0; e < E; e++) acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    bool full = true;
#pragma unroll
    for (int u = 0; u < U; u++) full &= t.nv[u] == UNIT_TOKENS;
    if (!full) {
      // scores of rows that are not there
#pragma unroll
      for (int u = 0; u < U; u++)
#pragma unroll
        for (int i = 0; i < 4; i++) s[u][i] = 4 * i + g16 < t.nv[u] ? s[u][i] : -INFINITY;
    }
    if (APPEND && (t.flags & T_LAST)) {
      // the new token's V row
      const int32_t rl = t.tail - 1;
#pragma unroll
      for (int u = 0; u < U; u++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const bool mine = u == t.n - 1 && 4 * i + g16 == rl;
#pragma unroll
          for (int w = 0; w < P; w++) v[u][i][w] = mine ? vn[w] : v[u][i][w];
        }
      if (g16 == (rl & 3)) {
        const gwptr_t dst = (gwptr_t)unit_base(t, U - 1) + plane + (uint32_t)(rl * ROWB + c * VB);
        if constexpr (P == 4) *(__attribute__((address_space(1))) words4_t*)dst = words4_t{vn[0], vn[1], vn[2], vn[3]};
        else *(__attribute__((address_space(1))) words2_t*)dst = words2_t{vn[0], vn[1]};
      }
    }
    float mx = fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3]));
#pragma unroll
    for (int u = 1; u < U; u++) mx = fmaxf(mx, fmaxf(fmaxf(s[u][0], s[u][1]), fmaxf(s[u][2], s[u][3])));
    const float mn = fmaxf(m, max_xor32(max_xor16(mx)));
    if (__builtin_amdgcn_ballot_w64(mn > m)) {       // some head has a new maximum
      const float alpha = fast_exp2(m - mn);
      l *= alpha;
#pragma unroll
      for (int e = 0; e < E; e++) acc[e] *= alpha;
      m = mn;
    }
    uint32_t pk[U][2], rest[U][2];
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int h = 0; h < 2; h++) {
        const float p0 = fast_exp2(s[u][2 * h] - m), p1 = fast_exp2(s[u][2 * h + 1] - m);
        l += p0 + p1;
        const uint32_t b0 = bf16_below(p0), b1 = bf16_below(p1);
        pk[u][h] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);
        rest[u][h] = pack_bf16(p0 - __uint_as_float(b0), p1 - __uint_as_float(b1));
      }
#pragma unroll
    for (int u = 0; u < U; u += 2) {
      const words4_t pb = {pk[u][0], pk[u][1], pk[u + 1][0], pk[u + 1][1]};
      const words4_t pr = {rest[u][0], rest[u][1], rest[u + 1][0], rest[u + 1][1]};
#pragma unroll
      for (int e = 0; e < E; e++) {
        const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
        const int w = e / 2;
        const words4_t va = {__builtin_amdgcn_perm(v[u][1][w], v[u][0][w], sel),
                             __builtin_amdgcn_perm(v[u][3][w], v[u][2][w], sel),
                             __builtin_amdgcn_perm(v[u + 1][1][w], v[u + 1][0][w], sel),
                             __builtin_amdgcn_perm(v[u + 1][3][w], v[u + 1][2][w], sel)};
        acc[e] = mfma16(va, pr, mfma16(va, pb, acc[e]));
      }
    }
  };
  if constexpr (NW > 0) {
    constexpr int F = D / 4, ROW = D + 4;              // a row of a head's accumulators, padded against bank conflicts
    __shared__ __attribute__((aligned(16))) float sums[NW][HEADS_PER_PASS][ROW];
    __shared__ float2 ml[NW][HEADS_PER_PASS];
    if (rem_share > 0) {
      TileInfo<U> t;
      advance(t);
      issue_k(t);
      issue_v(t);
      __builtin_amdgcn_sched_barrier(0);
      scores(t);
      weigh(t);
      const float L = add_xor32(add_xor16(l));
      if (c < n_heads) {
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
          for (int e = 0; e < E; e += 4)
            *reinterpret_cast<float4*>(&sums[wave][c][g16 * 4 + (i * E + e) * 4]) = make_float4(acc[e][i], acc[e + 1][i], acc[e + 2][i], acc[e + 3][i]);
        if (g16 == 0) ml[wave][c] = make_float2(m, L);
      }
    } else {
      // nothing left for this wave: zeros, whose weight is 0
      if (lane < n_heads) ml[wave][lane] = make_float2(-INFINITY, 0.f);
      for (int i = lane; i < n_heads * F; i += 64) *reinterpret_cast<float4*>(&sums[wave][i / F][i % F * 4]) = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
    // Every wave takes 64 columns (pieces of the heads' rows in order), in all blocks of a request the same ones, which need
    // no other wave from here on: they are stored, counted in and, by the last, added up by themselves. (All threads
    // together before, with two more barriers around the count and a sum through LDS: one request of 13 blocks 8.66 -> 8.25 us a
    // call, wide blocks 56.0 -> 52.8 for 8 requests, 4 layers. Shares gained nothing from it: no barriers there to save.)
    const int32_t n_cols = n_heads * F, x = threadIdx.x, h = x / F, f = x % F;
    static_assert(HEADS_PER_PASS * F <= NW * 64, "a thread for every column");
    if (wave * 64 >= n_cols) return;
    Sum s = {NEG_BIG, 0.f, make_float4(0.f, 0.f, 0.f, 0.f)};
    if (x < n_cols) {
      // (all rows are read before the first is added, and none is skipped: a branch around each makes a chain of LDS
      // latencies, 0.7 us where this takes 0.45; one request of 3300 tokens 7.99 -> 7.5 us a call with the same in Partials::sum)
      float2 p[NW];
      float4 v4[NW];
#pragma unroll
      for (int w = 0; w < NW; w++) {
        p[w] = ml[w][h];
        v4[w] = *reinterpret_cast<const float4*>(&sums[w][h][f * 4]);
      }
#pragma unroll
      for (int w = 0; w < NW; w++) s.M = fmaxf(s.M, p[w].x);
#pragma unroll
      for (int w = 0; w < NW; w++) add(s, p[w].y, v4[w], fast_exp2(p[w].x - s.M));
      if (part < 0) write_out<D>(pv, out, a, cb, g, g_first, x, s);
      else leave_partial<D>(pv, ws, a, part, g, g_first, n_heads, x, s);
    }
    // one of several blocks of its request: the last of them to get here adds their results up
    const int32_t n_part = first_rq.n_part;
    if (n_part == 1 || n_part > a.merge_parts) return;
    stores_done();
    uint32_t before = 0;
    // counting in one line takes turns (12 ns each; 8 times 8 for 16 heads in 8 blocks): as many lines as there are blocks
    if (lane == 0) before = count_in(pv, g * a.waves_per_head + first_rq.wave_first + wave % n_part, wave, n_part);
    const Partials<D> all(ws, a.ws_slots, (int64_t)g * a.parts_per_head + first_rq.part0, n_part, held(pv.group), g_first, n_heads);
    if (__builtin_amdgcn_readfirstlane(before) != (uint32_t)n_part - 1u) return;
    Sum all_of[1];
    all.template sum<1, 8, 16>(all_of, x, 0, 0, n_part);
    if (x < n_cols) write_out<D>(pv, out, a, cb, g, g_first, x, all_of[0]);
    return;
  }
  __shared__ __attribute__((aligned(16))) Results<D, SW == 1 ? 1 : HEADS_PER_PASS> results;     // (SW == 1: not used)
  auto finish = [&](const TileInfo<U>& t) __attribute__((always_inline)) {
    const float L = add_xor32(add_xor16(l));
    if (c >= n_heads) return;
    if (t.part < 0) {
      // the whole request lay inside this wave's share: this is the final result. Normalise, round and
      // write the output rows
      const float inv = 1.f / L;
      uint16_t* o = out + ((int64_t)(a.q_row0 + t.b) * pv.n_q_heads + hq0 + c) * D + g16 * (4 * E);
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int e = 0; e < E; e += 2)
          *reinterpret_cast<uint32_t*>(o + i * E + e) = pack_bf16(acc[e][i] * inv, acc[e + 1][i] * inv);
    } else if constexpr (SW == 1) {
      // one of several waves of the request: a partial result
      // (dims in the order in which the lanes of a row store neighbouring 16-byte pieces)
      const int64_t row = ((int64_t)g * a.parts_per_head + t.part) * pv.group + g_first + c;
      float* to = ws + row * D + g16 * 4;
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int e = 0; e < E; e += 4)
          *reinterpret_cast<float4*>(to + (i * E + e) * 4) = make_float4(acc[e][i], acc[e + 1][i], acc[e + 2][i], acc[e + 3][i]);
      if (g16 == 0) *reinterpret_cast<float2*>(ws + (int64_t)a.ws_slots * pv.group * D + row * WS_ML) = make_float2(m, L);
    } else {
      // one of several waves of the request: its results meet the others' in LDS
      // (dims in the order in which the lanes of a row store neighbouring 16-byte pieces)
      const int32_t to = 2 * wave + (t.b == sh.b ? 0 : 1);
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int e = 0; e < E; e += 4)
          results.rows[to][c][g16 + i * E + e] = make_float4(acc[e][i], acc[e + 1][i], acc[e + 2][i], acc[e + 3][i]);
      if (g16 == 0) results.ml[to][c] = make_float2(m, L);
      if (lane == 0) results.whose[to] = g * MAX_LAUNCH_REQ + t.b;
    }
  };
  // No exit before the round's last load (the share's last round asks for rows it does not use): what is in
  // flight when a tile is waited for is the same on every path, so the compiler counts the loads exactly.
  if (index < a.waves_per_head * pv.n_kv_heads) {
    TileInfo<U> t, next;
    advance(t);
    issue_k(t);
    issue_v(t);
    __builtin_amdgcn_sched_barrier(0);               // the loads stay where they are asked for
    if constexpr (SW > 1) results.clear(wave, lane);
    advance(next);
    uint32_t done;
    do {
      scores(t);
      issue_k(next);
      __builtin_amdgcn_sched_barrier(0);
      weigh(t);
      if (t.flags & (T_LAST | T_FIN)) finish(t);     // the request ends here, or the share does
      done = t.flags & T_FIN;
      issue_v(next);
      __builtin_amdgcn_sched_barrier(0);
      t = next;
      advance(next);
    } while (!done);
  } else if constexpr (SW > 1) {
    results.clear(wave, lane);
  }
  if constexpr (SW > 1) end_shares<D, HEADS_PER_PASS>(pv, ws, out, a, records, results, g_first, n_heads, workgroup, wave, lane);
}

// Launched with one wave per SIMD. The register cap of two keeps the matrix instructions' results out of
// the accumulation registers, which ordinary instructions cannot read.
template <int D, int U, int SW, bool APPEND, bool DIRECT, class Args>
__global__ __launch_bounds__(64 * SW) __attribute__((amdgpu_waves_per_eu(2, 2))) void decode_unit_kernel(
    PoolView pv, const uint16_t* __restrict__ q, const char* __restrict__ k_new, const char* __restrict__ v_new,
    float* __restrict__ ws, uint16_t* __restrict__ out, float scale_log2, int32_t g_first, int32_t n_heads, Args a) {
  in_launch(pv, ws, a, [&](const PoolView& pv, float* ws, const auto& a, int32_t workgroup) __attribute__((always_inline)) {
    decode_unit_body<D, U, APPEND, DIRECT, 0, SW>(pv, q, k_new, v_new, ws, out, scale_log2, g_first, n_heads, a, workgroup);
  });
}
// Small launches are bound by latency: 4 requests of up to 256 tokens, 8 heads of 64: 12.1 -> 8.5 us a call,
// of which one launch instead of two is 3 us of host time. Launches of 50 MB of K and V, in wide blocks with four units
// a wave: 8 requests of 4 q heads per kv head of 128, 4 layers of map-ahead, append and decode 63.2 -> 57.0 us a pass.
template <int D, int U, int NW, bool APPEND, bool DIRECT, class Args>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2))) void decode_block_kernel(
    PoolView pv, const uint16_t* __restrict__ q, const char* __restrict__ k_new, const char* __restrict__ v_new,
    float* __restrict__ ws, uint16_t* __restrict__ out, float scale_log2, int32_t g_first, int32_t n_heads, Args a) {
  in_launch(pv, ws, a, [&](const PoolView& pv, float* ws, const auto& a, int32_t workgroup) __attribute__((always_inline)) {
    decode_unit_body<D, U, APPEND, DIRECT, NW, 1>(pv, q, k_new, v_new, ws, out, scale_log2, g_first, n_heads, a, workgroup);
  });
}

// ---------------------------------------------------------------------------------------------
// combine pass, for the requests whose partial results are too many for one workgroup (merge_parts): one workgroup
// per (such request, q head). A row of accumulators is read 16 bytes per lane, so the workgroup takes RP = 16
// partials at a time; every lane's rows are asked for before the common maximum is known, so that the pass is one round
// trip to memory for up to 64 partials. The RP sums of a dim are added up through LDS in a fixed order. Twice as many
// waves are slower below 64 partials (32: 11.7 a call, 11.2; of heads of 64 36: 9.5, 8.4), faster for many (256 of heads
// of 64: 19.5, 21.5). In a launch in blocks a request that the attention kernel would have added up, were it not for
// another request, is added up in that kernel's order: its bits do not depend on its neighbours (IN_ORDER; its registers are as many
// as 16 partials ahead take, which launches of many workgroups do not have to pay).
// ---------------------------------------------------------------------------------------------
constexpr int COMBINE_AHEAD = 4;     // rows a lane asks for before it waits

template <int D, int W, bool IN_ORDER = false>
__global__ __launch_bounds__(64 * W) void decode_combine_kernel(const float* __restrict__ ws, uint16_t* __restrict__ out,
                                                                int32_t n_q_heads, int32_t group, BatchArgs a) {
  constexpr int F = D / 4, RP = W * 64 / F, AHEAD = COMBINE_AHEAD;
  __shared__ __attribute__((aligned(16))) float4 sums[RP][F];
  const int h = blockIdx.y, lane = threadIdx.x & 63, f = threadIdx.x % F, row = threadIdx.x / F;
  const int b = (a.split_req[blockIdx.x >> 2] >> ((blockIdx.x & 3) * 8)) & 0xff;   // blockIdx.x-th split request
  const int g = h / group;
  const int n_part = parts_of(a.req[b].wave_first, a.req[b].n_part, a.waves_per_head, g, a.wg_waves).n;
  if (IN_ORDER && n_part <= a.in_order_parts) {
    PoolView pv;
    pv.n_q_heads = n_q_heads;
    pv.group = group;
    if (threadIdx.x >= F) return;
    const Partials<D> all(ws, a.ws_slots, (int64_t)g * a.parts_per_head + a.req[b].part0, n_part, group, h - g * group, 1);
    Sum s[1];
    all.template sum<1, 8, 16>(s, f, 0, 0, n_part);
    write_out<D>(pv, out, a, b, g, h - g * group, f, s[0]);
    return;
  }
  const int64_t row0 = ((int64_t)g * a.parts_per_head + a.req[b].part0) * group + (h - g * group);
  const float4* p = reinterpret_cast<const float4*>(ws + row0 * D) + f;       // accumulator rows of this head
  const float* q0 = ws + (int64_t)a.ws_slots * group * D + row0 * WS_ML;      // their (m, l) pairs
  const int64_t stride = (int64_t)group * F, qstride = (int64_t)group * WS_ML;
  float4 v[AHEAD];
  float mv[AHEAD];
#pragma unroll
  for (int u = 0; u < AHEAD; u++) {
    const int j = row + u * RP;
    mv[u] = -INFINITY;
    v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (j < n_part) {
      mv[u] = q0[j * qstride];
      v[u] = p[j * stride];
    }
  }
  // the common maximum and the normaliser, by every wave for itself, one partial per lane
  float M = NEG_BIG, L = 0.f;
  for (int j = lane; j < n_part; j += 64) M = fmaxf(M, q0[j * qstride]);
  M = wave_max(M);
  for (int j = lane; j < n_part; j += 64) L += q0[j * qstride + 1] * fast_exp2(q0[j * qstride] - M);
  L = wave_sum(L);
  float4 A = make_float4(0.f, 0.f, 0.f, 0.f);
  auto add = [&](const float4& x, float c) __attribute__((always_inline)) {
    A.x += x.x * c; A.y += x.y * c; A.z += x.z * c; A.w += x.w * c;
  };
#pragma unroll
  for (int u = 0; u < AHEAD; u++)
    if (row + u * RP < n_part) add(v[u], fast_exp2(mv[u] - M));
  for (int j = row + AHEAD * RP; j < n_part; j += RP) add(p[j * stride], fast_exp2(q0[j * qstride] - M));
  sums[row][f] = A;
  __syncthreads();
  if (row != 0) return;
  // (eight at a time: all rows at once went through scratch memory, which the runtime allocates at the launch)
#pragma unroll 8
  for (int r = 1; r < RP; r++) add(sums[r][f], 1.f);
  uint16_t* o = out + ((int64_t)(a.q_row0 + b) * n_q_heads + h) * D + partial_dim<D>(a.unit_tokens, f);
  *reinterpret_cast<uint2*>(o) = make_uint2(f32_to_bf16_bits(A.x / L) | (f32_to_bf16_bits(A.y / L) << 16),
                                            f32_to_bf16_bits(A.z / L) | (f32_to_bf16_bits(A.w / L) << 16));
}

// ---------------------------------------------------------------------------------------------
// calibration kernels (measurement only; they compute nothing of the method)
// ---------------------------------------------------------------------------------------------
// plain copy of n 16-byte words: the known-size kernel the HBM byte counters are scaled against
__global__ __launch_bounds__(256) void copy_kernel(uint4* __restrict__ dst, const uint4* __restrict__ src, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * 256 * 4;
  for (int64_t i = (int64_t)blockIdx.x * 256 * 4 + threadIdx.x; i < n; i += stride) {
    uint4 v[4];
#pragma unroll
    for (int u = 0; u < 4; u++) { v[u] = make_uint4(0, 0, 0, 0); if (i + u * 256 < n) v[u] = src[i + u * 256]; }
#pragma unroll
    for (int u = 0; u < 4; u++) if (i + u * 256 < n) dst[i + u * 256] = v[u];
  }
}

// contiguous read of n 16-byte words: the read ceiling of this GPU for a streaming kernel
__global__ __launch_bounds__(256) void read_kernel(const uint4* __restrict__ src, int64_t n, uint32_t* __restrict__ sink) {
  const int64_t stride = (int64_t)gridDim.x * 256 * 8;
  uint32_t x = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 * 8 + threadIdx.x; i < n; i += stride) {
    uint4 v[8];
#pragma unroll
    for (int u = 0; u < 8; u++) { v[u] = make_uint4(0, 0, 0, 0); if (i + u * 256 < n) v[u] = load_stream16(src + i + u * 256); }
#pragma unroll
    for (int u = 0; u < 8; u++) x ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
  }
  if (x == 0x9e3779b9u) sink[0] = x;      // practically never true; keeps the loads alive
}

// the K/V rows a decode over this batch reads, with the same work partition and load shape (one
// wave per share of the same cut, up to 64 rows at a time, 128-bit loads), but no arithmetic
template <int D, bool DIRECT>
__global__ __launch_bounds__(64) void kv_stream_kernel(PoolView pv, uint32_t* __restrict__ sink, BatchArgs a) {
  constexpr int LPR = D / 8, RPW = 64 / LPR, NL = 64 / RPW, ROWB = D * 2;
  const int lane = threadIdx.x;
  const int sub = lane % LPR, rg = lane / LPR;
  const int32_t Tc = pv.tokens_per_chunk;
  uint32_t x = 0;
  {
    const Share<BatchArgs> sh = locate_share(a, Records<BatchArgs>(a, lane), blockIdx.x, lane);
    const int32_t g = sh.g;
    int32_t cb = sh.b;
    BatchArgs::Req rec = sh.first;
    const int32_t ut = a.unit_tokens, upc = (Tc + ut - 1) / ut;
    const int32_t u0 = (sh.u_lo - rec.unit_prefix) * a.step_units;
    int32_t left = units_of(rec.len, pv, upc, ut) - u0, todo = sh.n_units;
    if (a.step_units > 1) todo = min(todo * a.step_units, left);
    int32_t slot = u0 / upc;
    int32_t r = (u0 - slot * upc) * ut;
    while (todo > 0) {
      const TensorWalk walk = tensor_walk<DIRECT>(pv, rec.tensor);
      // up to 64 rows at a time, of one chunk
      const int32_t n = min(min(todo, left), min(64 / ut, upc - r / ut));
      const int32_t nv = min(ut * n, min(Tc - r, rec.len - (slot * Tc + r)));
      const char* kb = chunk_addr<DIRECT>(pv, walk, slot) + ((uint64_t)(g * 2) * Tc + r) * ROWB;
      const char* vb = kb + (uint64_t)Tc * ROWB;
      uint4 kr[NL], vr[NL];
#pragma unroll
      for (int u = 0; u < NL; u++) {
        const uint32_t off = (uint32_t)min(RPW * u + rg, nv - 1) * ROWB + sub * 16;
        kr[u] = load_stream16(kb + off);
        vr[u] = load_stream16(vb + off);
      }
#pragma unroll
      for (int u = 0; u < NL; u++) x ^= kr[u].x ^ kr[u].y ^ kr[u].z ^ kr[u].w ^ vr[u].x ^ vr[u].y ^ vr[u].z ^ vr[u].w;
      todo -= n;
      left -= n;
      if (left > 0) {
        r += ut * n;
        if (r >= Tc) { r = 0; slot += 1; }
      } else if (todo > 0) {
        cb += 1;
        rec = a.req[cb];
        left = units_of(rec.len, pv, upc, ut);
        slot = 0;
        r = 0;
      }
    }
  }
  if (x == 0x9e3779b9u) sink[0] = x;
}

// ---------------------------------------------------------------------------------------------
// A fixed workspace inside the library's own image, for callers that may not allocate: every GPU
// the library runs on holds one copy of this array, at its own address, until the process ends.
// Host code never uses the array's name as an address (on the host it is only a stand-in for the
// symbol); it asks the runtime for the device address once per device and uses that.
// ---------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[STATIC_WS_BYTES];

int static_workspace(float** ptr, size_t* bytes) {
  constexpr int MAX_DEVICES = 64;
  static void* addr[MAX_DEVICES] = {};           // per device: where that device holds the array
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  if (dev < 0 || dev >= MAX_DEVICES) return (int)hipErrorInvalidDevice;
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return (int)e;
    if (!p) return (int)hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = reinterpret_cast<float*>(addr[dev]);
  *bytes = STATIC_WS_BYTES;
  return 0;
}

// ---------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------
// A launch by the kernel's address and the places of its arguments. The launch syntax copies every argument by value twice on
// the way to the same call and takes the launch's shape through thread-local storage: a decode call of one request 2.77 -> 2.52 us
// on the host, of four short ones 2.95 -> 2.70. ev0 / ev1 (either may be NULL): events that take the kernel's own start and end times (the runtime's extended
// launch attaches them to the kernel's dispatch, so no marker of its own goes into the stream and the time between them is the
// kernel's duration).
template <typename... P, typename... A>
static int launch(void (*kernel)(P...), dim3 grid, unsigned threads, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1, const A&... a) {
  static_assert((std::is_same_v<std::remove_cv_t<P>, A> && ...), "the arguments are read as the kernel's own types");
  void* args[] = {const_cast<void*>(static_cast<const void*>(&a))...};
  const hipError_t e = ev0 || ev1 ? hipExtLaunchKernel((const void*)kernel, grid, dim3(threads), args, 0, stream, ev0, ev1, 0)
                                  : hipLaunchKernel((const void*)kernel, grid, dim3(threads), args, 0, stream);
  if (e != hipSuccess) (void)hipGetLastError();      // reported here, and not by the next one who asks
  return (int)e;
}
template <typename... P, typename... A>
static int launch(void (*kernel)(P...), dim3 grid, unsigned threads, hipStream_t stream, const A&... a) {
  return launch(kernel, grid, threads, stream, (hipEvent_t) nullptr, (hipEvent_t) nullptr, a...);
}

int launch_table_patch(int32_t* table, const PatchArgs& a, hipStream_t stream) {
  if (a.n <= 0) return 0;
  return launch(table_patch_kernel, dim3((a.n + 255) / 256), 256, stream, table, a);
}

int launch_fill(uint32_t* words, uint32_t value, size_t n, hipStream_t stream) {
  if (n == 0) return 0;
  return launch(fill_kernel, dim3((unsigned)((n + 255) / 256)), 256, stream, words, value, n);
}

int launch_kv_append(const PoolView& pv, const void* k_new, const void* v_new, const AppendArgs& a,
                     hipStream_t stream) {
  if (a.total_new <= 0) return 0;
  auto go = [&](auto kernel) { return launch(kernel, dim3((unsigned)a.total_new), 256, stream, pv, (const uint4*)k_new, (const uint4*)v_new, a); };
  if (pv.head_dim == 128) return pv.vbase ? go(kv_append_kernel<128, true>) : go(kv_append_kernel<128, false>);
  return pv.vbase ? go(kv_append_kernel<64, true>) : go(kv_append_kernel<64, false>);
}

int launch_chunk_copy(char* pool, char* host, uint32_t chunk_bytes, const CopyArgs& a, bool to_host, int workgroups, hipStream_t stream) {
  if (a.n <= 0) return 0;
  // a workgroup should still have 16 KiB to move
  int32_t wpc = std::max(1, workgroups / a.n);
  wpc = std::max(1, std::min<int>(wpc, (int)(chunk_bytes / (16u << 10))));
  return launch(chunk_copy_kernel, dim3((unsigned)(a.n * wpc)), 256, stream, pool, host, chunk_bytes, wpc, (int32_t)(to_host ? 1 : 0), a);
}

template <int D>
static const void* partial_kernel_ptr(int group, bool tiles) {
  if (!tiles) return (const void*)decode_unit_kernel<D, tile_units<D>, SHARE_WAVES, true, false, BatchArgs>;
  if constexpr (D == 128) {
    if (group == 8) return (const void*)decode_tile_kernel_wide<D, 8, true, false, BatchArgs>;
    if (group == 4) return (const void*)decode_tile_kernel_wide<D, 4, true, false, BatchArgs>;
  }
  return group == 2 ? (const void*)decode_tile_kernel<D, 2, true, false, BatchArgs> : (const void*)decode_tile_kernel<D, 1, true, false, BatchArgs>;
}

int partial_waves_per_cu(int head_dim, int group, int tokens_per_chunk) {
  const bool tiles = tile_kernel(head_dim, group, tokens_per_chunk);
  const void* f = head_dim == 128 ? partial_kernel_ptr<128>(group, tiles) : partial_kernel_ptr<64>(group, tiles);
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, 64 * SHARE_WAVES, 0) != hipSuccess || n < 1) n = 1;
  return n * SHARE_WAVES;
}

// the same launch, described for kernels that take fewer requests (the combine pass, which reads split_req, is not one)
static FewArgs few_of(const BatchArgs& a) {
  FewArgs f;
  f.n_req = a.n_req; f.waves_per_head = a.waves_per_head; f.units_each = a.units_each; f.units_extra = a.units_extra;
  f.by_waves = a.by_waves; f.step_units = a.step_units; f.q_row0 = a.q_row0; f.unit_tokens = a.unit_tokens;
  f.units_per_head = a.units_per_head; f.parts_per_head = a.parts_per_head; f.ws_slots = a.ws_slots;
  f.merge_parts = a.merge_parts; f.n_split_req = a.n_split_req; f.wg_waves = a.wg_waves; f.in_order_parts = a.in_order_parts;
  std::fill_n(f.split_req, FewArgs::MAX_REQ / 4, 0u);
  for (int i = 0; i < FewArgs::MAX_REQ; i++) f.req[i] = {};
  for (int i = 0; i < a.n_req; i++) f.req[i] = {a.req[i].len, a.req[i].tensor, a.req[i].unit_prefix, a.req[i].wave_first, a.req[i].n_part, a.req[i].part0};
  return f;
}

// a: the plan, or one of the two in `args`, which run the same kernel; workgroups: of all of it
template <int D, bool APPEND, bool DIRECT, class Args>
static int launch_partial_i(const PoolView& pv, const void* q, const void* k_new, const void* v_new, float* ws, void* out, float scale_log2,
                            const BatchArgs& a, const Args& args, unsigned workgroups, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop) {
  constexpr bool PAIR = std::is_same_v<Args, PairArgs>;
  if (a.unit_tokens == TILE_TOKENS) {
    auto go = [&](auto kernel) {
      return launch(kernel, dim3(workgroups), 64 * SHARE_WAVES, stream, ev_start, ev_stop, pv, (const uint16_t*)q, (const uint4*)k_new,
                    (const uint4*)v_new, ws, (uint16_t*)out, scale_log2, (int32_t)0, args);
    };
    if constexpr (D == 128) {
      if (pv.group == 4) return go(decode_tile_kernel_wide<D, 4, APPEND, DIRECT, Args>);
      if (pv.group == 8) return go(decode_tile_kernel_wide<D, 8, APPEND, DIRECT, Args>);
    }
    return pv.group == 1 ? go(decode_tile_kernel<D, 1, APPEND, DIRECT, Args>) : go(decode_tile_kernel<D, 2, APPEND, DIRECT, Args>);
  }
  if (a.step_units > STEP_UNITS) {
    auto go = [&](auto kernel, unsigned n_waves, const auto& its) {
      return launch(kernel, dim3(workgroups), 64 * n_waves, stream, ev_start, ev_stop, pv, (const uint16_t*)q, (const char*)k_new,
                    (const char*)v_new, ws, (uint16_t*)out, scale_log2, (int32_t)0, pv.group, its);
    };
    auto in_blocks = [&](const auto& its) {
      using Its = std::decay_t<decltype(its)>;
      constexpr int U = tile_units<D>, NW = BLOCK_UNITS / U;
      if (a.step_units <= BLOCK_UNITS) return go(decode_block_kernel<D, U, NW, APPEND, DIRECT, Its>, NW, its);
      return go(decode_block_kernel<D, WIDE_UNITS / WIDE_WAVES, WIDE_WAVES, APPEND, DIRECT, Its>, WIDE_WAVES, its);
    };
    if constexpr (!PAIR)
      if (a.n_req <= FewArgs::MAX_REQ) return in_blocks(few_of(a));
    return in_blocks(args);
  }
  // a group of more than HEADS_PER_PASS q heads is covered by several launches over the same K/V: the
  // first of them takes the start time, the last one the end time
  for (int done = 0; done < pv.group; done += HEADS_PER_PASS) {
    const int n = std::min(HEADS_PER_PASS, pv.group - done);
    auto go = [&](auto kernel, unsigned threads) {
      return launch(kernel, dim3(workgroups), threads, stream, done == 0 ? ev_start : nullptr, done + n >= pv.group ? ev_stop : nullptr, pv,
                    (const uint16_t*)q, (const char*)k_new, (const char*)v_new, ws, (uint16_t*)out, scale_log2, (int32_t)done, (int32_t)n, args);
    };
    int e = -1;
    if constexpr (!PAIR)               // (single_waves() is for several passes)
      if (a.wg_waves == 1) e = go(decode_unit_kernel<D, tile_units<D>, 1, APPEND, DIRECT, Args>, 64);
    if (e < 0) e = go(decode_unit_kernel<D, tile_units<D>, SHARE_WAVES, APPEND, DIRECT, Args>, 64 * SHARE_WAVES);
    if (e) return e;
  }
  return 0;
}

template <class Args>
static int launch_partial(const PoolView& pv, const void* q, const void* k_new, const void* v_new, float* ws, void* out, float scale_log2,
                          const BatchArgs& a, const Args& args, unsigned workgroups, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop) {
  auto go = [&](auto launch) { return launch(pv, q, k_new, v_new, ws, out, scale_log2, a, args, workgroups, stream, ev_start, ev_stop); };
  auto of_size = [&](auto dim) {
    constexpr int D = decltype(dim)::value;
    if (k_new) return pv.vbase ? go(launch_partial_i<D, true, true, Args>) : go(launch_partial_i<D, true, false, Args>);
    return pv.vbase ? go(launch_partial_i<D, false, true, Args>) : go(launch_partial_i<D, false, false, Args>);
  };
  return pv.head_dim == 128 ? of_size(std::integral_constant<int, 128>{}) : of_size(std::integral_constant<int, 64>{});
}

static unsigned workgroups_of(const PoolView& pv, const BatchArgs& a) {
  return ((unsigned)(a.waves_per_head * pv.n_kv_heads) + a.wg_waves - 1) / a.wg_waves;
}

int launch_decode_partial(const PoolView& pv, const void* q, const void* k_new, const void* v_new, float* ws,
                          void* out, float scale_log2, const BatchArgs& a, hipStream_t stream, hipEvent_t ev_start,
                          hipEvent_t ev_stop) {
  if (a.n_req <= 0 || a.waves_per_head <= 0) return 0;
  return launch_partial(pv, q, k_new, v_new, ws, out, scale_log2, a, a, workgroups_of(pv, a), stream, ev_start, ev_stop);
}

int launch_decode_pair(const PoolView& pv, const void* q, const void* k_new, const void* v_new, float* ws, void* out, float scale_log2,
                       PairArgs& a, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop) {
  a.workgroups = workgroups_of(pv, a.half[0]);
  return launch_partial(pv, q, k_new, v_new, ws, out, scale_log2, a.half[0], a, a.workgroups + workgroups_of(pv, a.half[1]), stream, ev_start, ev_stop);
}

int launch_decode_combine(const PoolView& pv, const float* ws, void* out, const BatchArgs& a, hipStream_t stream) {
  if (a.n_req <= 0 || a.n_split_req <= 0) return 0;
  // where every wave leaves partials there can be few of them each for many requests: as many waves as these fill
  const bool single = a.wg_waves == 1 && a.step_units <= STEP_UNITS;
  const int fill = single ? a.parts_per_head / a.n_split_req * pv.head_dim / (COMBINE_AHEAD * 256) : 4;    // by 1, by 4, more
  auto go = [&](auto kernel, unsigned waves) {
    return launch(kernel, dim3(a.n_split_req, pv.n_q_heads), 64 * waves, stream, ws, (uint16_t*)out, pv.n_q_heads, pv.group, a);
  };
  if (a.in_order_parts) return pv.head_dim == 128 ? go(decode_combine_kernel<128, 8, true>, 8) : go(decode_combine_kernel<64, 4, true>, 4);
  if (pv.head_dim == 128)
    return fill < 1 ? go(decode_combine_kernel<128, 2>, 2) : fill < 4 ? go(decode_combine_kernel<128, 4>, 4) : go(decode_combine_kernel<128, 8>, 8);
  return fill < 1 ? go(decode_combine_kernel<64, 1>, 1) : go(decode_combine_kernel<64, 4>, 4);
}

int launch_copy(void* dst, const void* src, int64_t bytes, hipStream_t stream) {
  const int64_t n = bytes / 16;
  if (n <= 0) return 0;
  const int64_t blocks = std::min<int64_t>((n + 1023) / 1024, 256 * 32);
  return launch(copy_kernel, dim3((unsigned)blocks), 256, stream, (uint4*)dst, (const uint4*)src, n);
}

int launch_read(const void* src, int64_t bytes, uint32_t* sink, hipStream_t stream) {
  const int64_t n = bytes / 16;
  if (n <= 0) return 0;
  const int64_t blocks = std::min<int64_t>((n + 2047) / 2048, 256 * 32);
  return launch(read_kernel, dim3((unsigned)blocks), 256, stream, (const uint4*)src, n, sink);
}

int launch_kv_stream(const PoolView& pv, uint32_t* sink, const BatchArgs& a, hipStream_t stream) {
  const unsigned grid = (unsigned)(a.waves_per_head * pv.n_kv_heads);
  if (a.n_req <= 0 || grid == 0) return 0;
  auto go = [&](auto kernel) { return launch(kernel, dim3(grid), 64, stream, pv, sink, a); };
  if (pv.head_dim == 128) return pv.vbase ? go(kv_stream_kernel<128, true>) : go(kv_stream_kernel<128, false>);
  return pv.vbase ? go(kv_stream_kernel<64, true>) : go(kv_stream_kernel<64, false>);
}

}  // namespace ellm
