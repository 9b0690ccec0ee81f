// libsdnn: Sparse DNN Challenge inference (Kepner et al., 2019) on MI355X (gfx950).
//
// Per layer (Sec. II batched equation, Sec. V listing):
//   z[r][j] = fma chain over the sources k of column j, ascending, of Y[r][k] * W(k, j)
//   Y'[r][j] = (z != 0) ? min(ymax, max(0, z + b[j])) : 0
// followed by dropping rows that became all zero (they stay zero) and, after the last layer, the
// categories: rows with any entry > 0 (Sec. V).
//
// Data layout in HBM
//   Activations: path 0 (widths whose tiles fit LDS, N <= 4096) keeps row-major [M][N] fp32 rows
//   and a list of live row ids; path 1 keeps feature-major tiles of 32 list positions ([N][32] fp32
//   per tile, 128 bytes per source), up to 16384 neurons fp32 rows by list position, or after layer 0
//   one-byte dictionary codes in tiles of 64 or 128 positions (two-byte ones past 32768 neurons), or bit
//   tiles of 16 or 32 positions for binary inputs.
//   Weights: per layer a slot-major ELL table [K][N] of (source offset, fp32 weight), entry [s][j]
//   the s-th smallest source of output j, padded with (0, 0.0f); padding adds fma(y, 0, acc) = acc
//   exactly. Layers with 32 sources per column also get 16-bit source lists with their fp32
//   weights beside them: [32][N] u16 + [32][N] fp32 (path 1, six bytes per edge) and [4][N][8]
//   u16 + [8][N][4] fp32 (path 0, 16-byte loads). Path 1 up to 16384 neurons also keeps every layer's
//   columns as the streams of k_layer_seg. With the opt-in equal-value kernels, a layer whose
//   weights and biases are all equal keeps one weight instead, and where columns share their list
//   only the representative columns' lists.
//
// Kernels (every output is the ascending-source fma chain above, so every path gives the same bits)
//   path 0: k_layer_lds32 (one layer; B rows staged in LDS as [k][B]) and k_layers_lds32 (every remaining
//     layer in one launch, each workgroup's rows resident in LDS) for lists of 32 sources with per-edge
//     weights, loaded ahead; k_layer_lds and k_layers_lds for other lists (and narrow batches); opt-in, layer
//     0 by counts of bit tiles.
//   path 1, layer 0: k_pack_bits, then k_layer_bits (or, opt-in for one-weight layers,
//     k_count_dict + k_layer_count: adder-tree counts of set source bits, decoded by a
//     dictionary); non-binary inputs take k_layer_seg (up to 16384 neurons) or k_to_fm + k_layer_gfm.
//   path 1, later layers: k_layer_gfm_u8 (code tiles in), k_layer_seg (fp32 rows in, up to 16384 neurons),
//     k_layer_gfm (fp32 tiles in), k_layer_gfm_small (at most 8 tiles, whole chains in flight). The
//     tile kernels' workgroups are mapped so that each XCD gathers from its own tile, resident in its L2.
//   Between layers: liveness words per tile (spread over cache lines, or per-workgroup partial
//   words), k_compact (stable compaction of the live list), k_repack / k_repack_u8 (regroup live
//   positions into fewer tiles), k_final_ids.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <exception>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <type_traits>
#include <thread>
#include <unordered_map>
#include <utility>
#include <vector>

#include "sdnn.h"

namespace {

thread_local std::string g_err;

sdnn_status fail(sdnn_status s, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  try {
    g_err = buf;
  } catch (...) {
    g_err.clear();
  }
  return s;
}

// The answer of an entry point in which an allocation on the host failed: no exception crosses the ABI.
sdnn_status no_memory() { return fail(SDNN_ENOMEM, "out of host memory"); }
#define SDNN_CATCH catch (...) { return no_memory(); }

constexpr int kMaxNeurons = 65536;
constexpr int kMaxLayers = 1000000;
constexpr int kMaxDegree = 4096;
constexpr int kLdsTileBytes = 128 * 1024;  // activation tile budget per workgroup
constexpr int kGfmOutputs = 64;            // outputs per work item of k_layer_gfm
constexpr int kPollEvery = 16;             // layers between live-count read-backs
constexpr int64_t kEncodeMinRows = 2048;   // live rows from which a fp32-input layer tries codes

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Run f(i) for i in [0, n) on up to 16 host threads, the caller's among them (used for host-side validation and
// packing). What f throws (out of memory) stops all of them and is thrown on the caller's thread; threads
// that cannot be started are done without.
template <class F>
void parallel_for(int32_t n, F f) {
  const int32_t nt = std::max<int32_t>(1, std::min<int32_t>({n, 16, (int32_t)std::max(1u, std::thread::hardware_concurrency())}));
  std::atomic<int32_t> next{0};
  std::atomic<bool> failed{false};
  std::exception_ptr thrown;  // by the thread that set failed first; read after the joins
  auto work = [&]() noexcept {
    try {
      for (int32_t i = next++; i < n && !failed; i = next++) f(i);
    } catch (...) {
      if (!failed.exchange(true)) thrown = std::current_exception();
    }
  };
  std::vector<std::thread> th;
  try {
    th.reserve((size_t)nt - 1);
    for (int32_t t = 1; t < nt; ++t) th.emplace_back(work);
  } catch (...) {
  }
  work();
  for (auto &x : th) x.join();
  if (thrown) std::rethrow_exception(thrown);
}

// ------------------------------------------------------------------------------------------------
// Device code

__device__ __forceinline__ float activate(float z, float b, float ymax) {
  // Sec. V loop: the bias goes only to nonzero products, then the result is clamped to [0, ymax].
  // Zeros come out as +0: for z != 0 the sum t is never -0 (x + y = -0 needs x = y = -0, and a sum
  // of nonzero values that is zero is +0), so the median of (t, +0, ymax), ymax > 0, is +0 for t <= 0.
  const float t = __builtin_amdgcn_fmed3f(z + b, 0.0f, ymax);
  return z == 0.0f ? 0.0f : t;
}

// Keeps the compiler from moving memory accesses across this point (no instruction is emitted):
// pins the issue order of software-pipelined loads.
__device__ __forceinline__ void mem_fence_compiler() { asm volatile("" ::: "memory"); }

// Barrier of a workgroup that orders LDS accesses only: global loads and stores in flight are not waited for.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Sets bits m in a liveness mask word that many workgroups report to. They report mostly the same
// rows, and hundreds of atomics on one word from workgroups that finish together serialize (several
// us per launch), so only bits not yet set go through an atomic. Within a layer bits are only ever
// set, so a set bit read here is final; a stale read only costs an atomic.
// Liveness words of large layers. Device-scope atomics on one 128-byte line serialize across
// workgroups (2048 workgroups of a launch ORing into one line: tens of us), while atomics on
// different lines proceed in parallel. So mask word t of such a layer is spread over kSpread words
// in lines of their own, spread[(t * kSpread + g) * kLineWords] with g taken from the workgroup
// index, and k_spread_to_masks ORs them into masks[t] before a compaction reads it.
constexpr int kSpread = 8, kLineWords = 32;
__device__ __forceinline__ void or_mask(unsigned *masks, unsigned *spread, int t, unsigned m) {
  if (spread)
    atomicOr(&spread[((size_t)t * kSpread + ((blockIdx.x >> 3) & (kSpread - 1))) * kLineWords], m);
  else
    atomicOr(&masks[t], m);
}

// Ties four values to this point of the instruction stream (no instruction is emitted): the
// computations producing them are scheduled before it.
__device__ __forceinline__ void pin4(float &a, float &b, float &c, float &d) {
  asm volatile("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}

// 16-byte store that streams past the L2 (the data is read by the next kernel, not this one).
__device__ __forceinline__ void store_stream(float4 *p, float4 v) {
  typedef float v4f __attribute__((ext_vector_type(4)));
  const v4f x = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(x, reinterpret_cast<v4f *>(p));
}

__device__ __forceinline__ void store_stream(uint4 *p, uint4 v) {
  typedef unsigned v4u __attribute__((ext_vector_type(4)));
  const v4u x = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(x, reinterpret_cast<v4u *>(p));
}

// 16-byte nontemporal load, for data that is read exactly once (the input rows). Data that other
// workgroups read again (weights, activation tiles) takes plain loads, which measure faster.
__device__ __forceinline__ float4 load_stream_f4(const float4 *p) {
  typedef float v4f __attribute__((ext_vector_type(4)));
  const v4f x = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(p));
  return make_float4(x[0], x[1], x[2], x[3]);
}


// Raw buffer resource over `bytes` bytes at p (stride 0, offsets in bytes): an access past the end
// reads zeros. The third dword is the gfx9 default format word.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void *p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes, 0x00020000);
}

__device__ __forceinline__ bool any_nonzero(float4 v) {
  return v.x != 0.0f || v.y != 0.0f || v.z != 0.0f || v.w != 0.0f;
}

// misc[0]: a layer-0 input is not 0 or 1; misc[kOverflowSlot]: the value dictionary is full;
// misc[3]: first live count of a uniform layer 0; misc[kNposSlot + i]: positions in live list i.
// The value dictionary's initial state (its layout is described with dict_code below): code 0 is
// +0.0, whose key 0 sits in its hash slot 0; every other slot is free and the next code is 1.
constexpr unsigned kDictEmpty = 0x7fc00000u;
constexpr unsigned kNoCode = 0xffffffffu;
constexpr int kDictSlots = 256;       // codes
constexpr int kDictHashSlots = 1024;  // hash table slots
constexpr int kDictKey = kDictSlots, kDictCode = kDictKey + kDictHashSlots, kDictNext = kDictCode + kDictHashSlots,
              kDictWords = kDictNext + 256;
// The two dictionaries: one-byte codes (above) and two-byte codes (4096 values, for layer inputs
// that take more than 256). Words: val[kSlots] | key[kHash] | code[kHash] | next; the hash slot of
// a key is bits kHashShift.. of its 24-bit multiplicative hash, the LDS cache set bits kCacheShift..
template <int CB> struct DictShape;
template <> struct DictShape<1> {
  static constexpr int kSlots = kDictSlots, kHash = kDictHashSlots, kHashShift = 14, kCache = 1024, kCacheShift = 12;
};
template <> struct DictShape<2> {
  static constexpr int kSlots = 4096, kHash = 16384, kHashShift = 10, kCache = 4096, kCacheShift = 10;
};
template <int CB> __host__ __device__ constexpr int dict_key_off() { return DictShape<CB>::kSlots; }
template <int CB> __host__ __device__ constexpr int dict_code_off() { return dict_key_off<CB>() + DictShape<CB>::kHash; }
template <int CB> __host__ __device__ constexpr int dict_next_off() { return dict_code_off<CB>() + DictShape<CB>::kHash; }
template <int CB> __host__ __device__ constexpr int dict_words() { return dict_next_off<CB>() + 256; }
static_assert(dict_words<1>() == kDictWords, "one-byte dictionary layout");
template <int CB = 1>
__device__ __forceinline__ void dict_init(unsigned *dict, int t, int nt) {
  constexpr int KEY = dict_key_off<CB>(), CODE = dict_code_off<CB>(), NEXT = dict_next_off<CB>();
  for (int i = t; i <= NEXT; i += nt)
    dict[i] = i < KEY ? 0u : i < CODE ? (i == KEY ? 0u : kDictEmpty) : i < NEXT ? (i == CODE ? 0u : kNoCode) : 1u;
}

// misc[kPaceSlot + x]: layer that workgroup x < 8 of a fused launch runs (see fetch_lists).
constexpr int kOverflowSlot = 2;
constexpr int kNposSlot = 4;
constexpr int kPaceSlot = 8, kMiscWords = 16;
__global__ void k_init(int *__restrict__ ids, unsigned *__restrict__ masks, unsigned *__restrict__ masks2,
                       unsigned *__restrict__ masks3, int *__restrict__ rownz, int *__restrict__ counts,
                       int *__restrict__ misc, unsigned *__restrict__ dict, int M, int L,
                       unsigned *__restrict__ spread, size_t spread_words) {
  const int st = gridDim.x * blockDim.x;
  // value dictionary (see dict_code): code 0 is +0.0, whose key 0 sits in its hash slot 0; every
  // other slot is free and the next code is 1
  if (blockIdx.x == 0) dict_init(dict, threadIdx.x, blockDim.x);
  if (blockIdx.x == 0 && threadIdx.x < kMiscWords) misc[threadIdx.x] = (threadIdx.x == kNposSlot) ? M : 0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < M; i += st) {
    ids[i] = i;
    masks[i] = 0u;
    masks2[i] = 0u;
    masks3[i] = 0u;
    rownz[i] = 0;
  }
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i <= L; i += st) counts[i] = (i == 0) ? M : 0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < spread_words; i += st) spread[i] = 0u;
}

// Inclusive prefix sum over the 64 lanes of a wave.
__device__ __forceinline__ int wave_inclusive_sum(int v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int u = __shfl_up(v, d, 64);
    if (lane >= d) v += u;
  }
  return v;
}

// Stable compaction over per-tile liveness masks: bit b of masks[t] says that list position
// t*B + b is live. ids_out = the live ids in list order, src_out (unless null) = their positions in
// the input list, *count_out (and *count_out2 unless null) = their number. The masks are cleared for
// the next layer. One workgroup of 1024 threads; tiles are taken 4096 at a time: an exclusive scan
// of their popcounts gives each tile's output offset, then every position is placed.
constexpr int kCompactTiles = 4096;
// masks[t] = OR of the spread words of tile t (see or_mask) for the tiles of the first *npos list
// positions; the spread words are zeroed for the next large layer.
__global__ __launch_bounds__(256) void k_spread_to_masks(unsigned *__restrict__ spread, const int *__restrict__ npos,
                                                         unsigned *__restrict__ masks) {
  const int nt = (*npos + 31) / 32;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < nt; t += gridDim.x * blockDim.x) {
    unsigned m = 0u;
#pragma unroll
    for (int g = 0; g < kSpread; ++g) {
      unsigned *w = &spread[((size_t)t * kSpread + g) * kLineWords];
      m |= *w;
      *w = 0u;
    }
    masks[t] = m;
  }
}

// With notify set, thread 0 finally stores (tag << 40) | (flags << 32) | count into that word of
// coherent host memory, flags = bit 0: misc[0] (a layer-0 input is not 0 or 1), bit 1:
// misc[kOverflowSlot] (the value dictionary is full), bit 2: the sample below took more than
// kDictSlots distinct values; the host waits on it instead of a copy and a stream synchronization.
// With at least sample_min live rows, 4096 values of the layer's output are looked at: of feature-major
// tiles (or, with sample_rows, rows by list position) act, whose segments with a clear seglive bit
// are zero. A layer whose sample holds more values than the dictionary cannot be encoded, and the
// attempt is saved (failed encodings took 0.7-1.2 ms on 16384 x 16384 activations whose values are many,
// longer than a successful one, against 3-5 us for the sample).
constexpr int kSampleValues = 4096;
struct CompactSample {
  const float *act;         // null: no sample
  const unsigned *seglive;  // null: every segment is stored
  int N, rows_major, min_rows;
};
__global__ __launch_bounds__(1024) void k_compact(unsigned *__restrict__ masks, int B, const int *__restrict__ ids_in,
                                                  int *__restrict__ ids_out, int *__restrict__ src_out,
                                                  const int *__restrict__ count_in, int *__restrict__ count_out,
                                                  int *__restrict__ count_out2, const int *__restrict__ misc,
                                                  unsigned long long *__restrict__ notify, unsigned long long tag,
                                                  CompactSample smp) {
  __shared__ int toff[kCompactTiles];
  __shared__ unsigned tmask[kCompactTiles];
  __shared__ int wsum[16];
  const int R = *count_in;
  const int ntiles = (R + B - 1) / B;
  const int sh = __ffs(B) - 1;  // (B is a power of two, at most 32)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int base = 0;
  for (int c0 = 0; c0 < ntiles; c0 += kCompactTiles) {
    unsigned m[4];
    int local = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = c0 + tid * 4 + q;
      m[q] = 0u;
      if (t < ntiles) {
        m[q] = masks[t];
        masks[t] = 0u;
      }
      local += __popc(m[q]);
    }
    const int incl = wave_inclusive_sum(local, lane);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int off = 0, total = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      const int x = wsum[w];
      off += (w < wave) ? x : 0;
      total += x;
    }
    int excl = base + off + incl - local;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      toff[tid * 4 + q] = excl;
      tmask[tid * 4 + q] = m[q];
      excl += __popc(m[q]);
    }
    __syncthreads();
    const int p_end = min(R, (c0 + kCompactTiles) * B);
    // eight ids are loaded at a time: with one, each was waited for (60,000 rows x 120 layers of 1024
    // neurons, 11 compactions: 2.02 -> 1.98 ms a pass)
    constexpr int kIds = 8;
    for (int q0 = c0 * B + tid; q0 < p_end; q0 += kIds * 1024) {
      int id[kIds];
#pragma unroll
      for (int u = 0; u < kIds; ++u) id[u] = ids_in[min(q0 + u * 1024, p_end - 1)];
#pragma unroll
      for (int u = 0; u < kIds; ++u) {
        const int p = q0 + u * 1024;
        if (p >= p_end) break;
        const int tl = (p >> sh) - c0, b = p & (B - 1);
        const unsigned mk = tmask[tl];
        if ((mk >> b) & 1u) {
          const int o = toff[tl] + __popc(mk & ((1u << b) - 1u));
          ids_out[o] = id[u];
          if (src_out) src_out[o] = p;
        }
      }
    }
    base += total;
    __syncthreads();
  }
  // distinct values of the sample: an LDS hash table in place of the tile offsets; at most kDictSlots +
  // 1024 of its slots fill up before every thread sees the count and stops
  __shared__ int distinct;
  static_assert(kDictSlots + 1024 < kCompactTiles, "the table never fills up");
  const bool sampling = smp.act != nullptr && src_out != nullptr && base >= smp.min_rows;
  if (sampling) {
    unsigned *tab = reinterpret_cast<unsigned *>(toff);
    for (int i = tid; i < kCompactTiles; i += 1024) tab[i] = kDictEmpty;
    if (tid == 0) distinct = 0;
    __syncthreads();
    for (int i = tid; i < kSampleValues; i += 1024) {
      if (__hip_atomic_load(&distinct, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > kDictSlots) break;
      const int p = src_out[(int)((long long)i * base / kSampleValues)];
      const unsigned k = (unsigned)(((unsigned long long)((unsigned)i * 0x9E3779B1u) * (unsigned)smp.N) >> 32);
      float v;
      if (smp.rows_major) {
        v = smp.act[(size_t)p * smp.N + k];
      } else {
        const size_t t = (size_t)(p >> 5);
        const bool stored = !smp.seglive || ((smp.seglive[t * ((smp.N + 31) / 32) + (k >> 5)] >> (k & 31)) & 1u);
        v = stored ? smp.act[(t * smp.N + k) * 32 + (p & 31)] : 0.0f;
      }
      const unsigned key = __float_as_uint(v);
      for (unsigned h = (key * 0x9E3779B1u) >> 20;; h = (h + 1) & (kCompactTiles - 1)) {
        const unsigned old = atomicCAS(&tab[h], kDictEmpty, key);
        if (old == kDictEmpty) atomicAdd(&distinct, 1);
        if (old == kDictEmpty || old == key) break;
      }
    }
    __syncthreads();
  }
  if (tid == 0) {
    *count_out = base;
    if (count_out2) *count_out2 = base;
    if (notify) {
      const unsigned long long flags = (misc[0] != 0 ? 1ull : 0ull) | (misc[kOverflowSlot] != 0 ? 2ull : 0ull) |
                                       (sampling && distinct > kDictSlots ? 4ull : 0ull);
      __hip_atomic_store(notify, (tag << 40) | (flags << 32) | (unsigned long long)(unsigned)base, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}

// Zeros into the 128-byte segments of fp32 tiles [0, (*npos + 31) / 32) whose seglive bit is clear
// (segments that a producer skipped because all their rows are zero), for readers that take the
// tiles as they are. 8 lanes write one segment.
__global__ __launch_bounds__(256) void k_fill_dead(float *__restrict__ fm, int N, const unsigned *__restrict__ seglive,
                                                   const int *__restrict__ npos) {
  const int ntiles = (*npos + 31) / 32;
  const int NW = (N + 31) / 32;
  const size_t items = (size_t)ntiles * N * 8;
  for (size_t it = blockIdx.x * (size_t)blockDim.x + threadIdx.x; it < items; it += (size_t)gridDim.x * blockDim.x) {
    const int q = (int)(it & 7);
    const size_t seg = it >> 3;
    const int k = (int)(seg % N);
    const size_t t = seg / N;
    if (!((seglive[t * NW + (k >> 5)] >> (k & 31)) & 1u))
      reinterpret_cast<float4 *>(fm + seg * 32)[q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  }
}

// Copy list positions pos[0..n) of feature-major tiles out as rows: out[i][k] = fm at position
// pos[i], source k. With rowmajor, fm holds whole rows by position instead.
__global__ __launch_bounds__(256) void k_gather_rows(const float *__restrict__ fm, int N, const int *__restrict__ pos,
                                                     int n, float *__restrict__ out, bool rowmajor) {
  const size_t items = (size_t)n * N;
  for (size_t it = blockIdx.x * (size_t)blockDim.x + threadIdx.x; it < items; it += (size_t)gridDim.x * blockDim.x) {
    const int i = (int)(it / N), k = (int)(it % N);
    const int p = pos[i];
    out[it] = rowmajor ? fm[(size_t)p * N + k] : fm[((size_t)(p >> 5) * N + k) * 32 + (p & 31)];
  }
}

// What the host reads after a run, in coherent host memory that the device writes when the host asks: the
// categories' number and (up to kHostIds) ids, the live counts (networks of fewer than kHostCounts
// layers) and the number of nonzero input rows. Reading them costs no copies; each small one from
// device memory takes about 10 us.
constexpr int kHostIds = 4096, kHostCounts = 4096;
struct HostOut {
  long long ids[kHostIds];
  int counts[kHostCounts];
  int count, nonzero;
};

// M: rows of the run (the bound holds whatever a caller has done to the workspace since).
__global__ void k_final_ids(const int *__restrict__ ids, const int *__restrict__ count, int M, long long *__restrict__ out,
                            HostOut *__restrict__ host) {
  const int R = max(0, min(*count, M));
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < R; i += gridDim.x * blockDim.x) {
    out[i] = ids[i];
    if (R <= kHostIds) __hip_atomic_store(&host->ids[i], (long long)ids[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0)
    __hip_atomic_store(&host->count, R, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The live counts and the number of nonzero input rows (rownz, M rows) to the host. One workgroup.
__global__ __launch_bounds__(1024) void k_host_counts(const int *__restrict__ counts, int L, const int *__restrict__ rownz,
                                                      int M, HostOut *__restrict__ host) {
  __shared__ int total;
  if (threadIdx.x == 0) total = 0;
  __syncthreads();
  int n = 0;
  for (int i = threadIdx.x; i < M; i += 1024) n += rownz[i] != 0;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) n += __shfl_xor(n, d, 64);
  if ((threadIdx.x & 63) == 0 && n) atomicAdd(&total, n);
  for (int l = threadIdx.x; l <= L; l += 1024)
    __hip_atomic_store(&host->counts[l], counts[l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(&host->nonzero, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Split a tile's outputs into chunks so that small live counts still spread over the whole grid:
// with many tiles every work item is a whole tile; with few, each tile's outputs are divided.
struct Chunking {
  int nchunks, rounds_per_chunk;
};

// Tile of item w when whole tiles are the items and tpg consecutive tiles share one code group:
// the tpg tiles of a group go to workgroups of the same XCD (workgroup x runs on XCD x % 8), so the
// parts that they write of each code segment meet in that XCD's L2. A bijection of
// [0, gridDim * ceil(n / gridDim)) onto itself; needs gridDim % (8 * tpg) == 0.
__device__ __forceinline__ int code_group_tile(int w, int tpg) {
  const int per_iter = gridDim.x;
  const int k = w / per_iter, x = w % per_iter;
  const int xcd = x & 7, sl = x >> 3;
  const int g = k * (per_iter / tpg) + xcd + 8 * (sl / tpg);
  return tpg * g + sl % tpg;
}
__device__ __forceinline__ Chunking chunking(int ntiles, int rounds, int min_chunks = 1) {
  int nchunks = ntiles > 0 ? (int)gridDim.x / ntiles : 1;
  nchunks = max(min_chunks, min(nchunks, rounds));
  nchunks = min(nchunks, rounds);
  const int rpc = (rounds + nchunks - 1) / nchunks;
  return {(rounds + rpc - 1) / rpc, rpc};
}

// LDS reads in flight ahead of the fmas in the LDS-tile kernels' 32-term chains
#ifndef SDNN_LDS_AHEAD
#define SDNN_LDS_AHEAD 6
#endif
constexpr int kLdsAhead = SDNN_LDS_AHEAD;

// One layer with the activation tile staged in LDS. B rows per tile (4 <= B <= 32, a multiple of 4);
// blockDim 1024. KC is the compile-time ELL width (0: use the runtime K). With cols set (one-weight
// layers through ell16 only), the ncols columns cols[p] alone are computed and written, their
// source lists in ell16 as [4][ncols][8]; the other columns equal one of them (see k_layer_gfm).
// With place set, neuron k is staged at tile row place[k] and ell16 holds tile rows (placed
// sources; see bank_placement), which only changes which LDS banks the reads fall in.
template <int B, int KC>
__global__ __launch_bounds__(1024) void k_layer_lds(const float *__restrict__ yin, float *__restrict__ yout, int N,
                                                    const int2 *__restrict__ ell, int K,
                                                    const uint4 *__restrict__ ell16, const float *__restrict__ w8,
                                                    float wc,
                                                    const float *__restrict__ bias, float ymax,
                                                    const int *__restrict__ ids, const int *__restrict__ count,
                                                    unsigned *__restrict__ masks, int *__restrict__ rownz,
                                                    const int *__restrict__ cols, int ncols,
                                                    const unsigned short *__restrict__ place) {
  extern __shared__ float4 smem[];
  const char *tile = reinterpret_cast<const char *>(smem);
  float *tilef = reinterpret_cast<float *>(smem);
  __shared__ int rowlive[B];
  __shared__ int rowany[B];
  constexpr int LPO = B / 4;    // lanes per output, 4 rows each
  constexpr int OPW = 64 / LPO; // outputs per wave instruction
  const int R = *count;
  const int ntiles = (R + B - 1) / B;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
  const int quad = lane % LPO, jl = lane / LPO;
  const int per_round = nw * OPW;
  const int rounds = (ncols + per_round - 1) / per_round;
  const Chunking ch = chunking(ntiles, rounds);
  const int items = ntiles * ch.nchunks;
  if (tid < B) {
    rowlive[tid] = 0;
    rowany[tid] = 0;
  }
  for (int w = blockIdx.x; w < items; w += gridDim.x) {
    const int t = w / ch.nchunks, c = w % ch.nchunks;
    const int p0 = t * B;
    const int nvalid = min(B, R - p0);
    const bool count_nz = rownz != nullptr && c == 0;
    // ---- stage rows ids[p0 .. p0+nvalid) as tile[k][b]; missing rows are zero
    if ((N & 3) == 0) {
      const int NQ = N >> 2;
      const int nitems = NQ * (B / 4);
      for (int it = tid; it < nitems; it += blockDim.x) {
        const int bq = it % (B / 4), q = it / (B / 4);
        float4 v[4];
#pragma unroll
        for (int c4 = 0; c4 < 4; ++c4) {
          const int b = bq * 4 + c4;
          v[c4] = (b < nvalid) ? reinterpret_cast<const float4 *>(yin + (size_t)ids[p0 + b] * N)[q]
                               : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        // neuron k goes to tile row place[k] (k itself without a placement)
        int rk[4];
#pragma unroll
        for (int c4 = 0; c4 < 4; ++c4) rk[c4] = place ? (int)place[4 * q + c4] : 4 * q + c4;
        float *dst = tilef + bq * 4;
        *reinterpret_cast<float4 *>(dst + (size_t)rk[0] * B) = make_float4(v[0].x, v[1].x, v[2].x, v[3].x);
        *reinterpret_cast<float4 *>(dst + (size_t)rk[1] * B) = make_float4(v[0].y, v[1].y, v[2].y, v[3].y);
        *reinterpret_cast<float4 *>(dst + (size_t)rk[2] * B) = make_float4(v[0].z, v[1].z, v[2].z, v[3].z);
        *reinterpret_cast<float4 *>(dst + (size_t)rk[3] * B) = make_float4(v[0].w, v[1].w, v[2].w, v[3].w);
        if (count_nz) {
#pragma unroll
          for (int c4 = 0; c4 < 4; ++c4)
            if (any_nonzero(v[c4])) rowany[bq * 4 + c4] = 1;
        }
      }
    } else {
      for (int it = tid; it < N * B; it += blockDim.x) {
        const int b = it % B, k = it / B;
        const float v = (b < nvalid) ? yin[(size_t)ids[p0 + b] * N + k] : 0.0f;
        tilef[(size_t)(place ? (int)place[k] : k) * B + b] = v;
        if (count_nz && v != 0.0f) rowany[b] = 1;
      }
    }
    __syncthreads();
    // ---- compute: lane (quad, jl) owns rows 4*quad..4*quad+3 of output j
    int row[4];
#pragma unroll
    for (int c4 = 0; c4 < 4; ++c4) {
      const int b = quad * 4 + c4;
      row[c4] = (b < nvalid) ? ids[p0 + b] : -1;
    }
    const int qoff = quad * 16;
    int live_mask = 0;
    const int r_end = min(rounds, (c + 1) * ch.rounds_per_chunk);
    for (int r = c * ch.rounds_per_chunk; r < r_end; ++r) {
      const int j = r * per_round + wave * OPW + jl;  // output position (the column without cols)
      if (j >= ncols) continue;
      const int col = cols ? cols[j] : j;
      float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, a3 = 0.0f;
      // ELL is slot-major ([s][j]): for a given slot the lanes of a wave read consecutive entries.
      // Terms go in groups of 8 in ascending source order; with KC known, the next group's
      // entries are loaded (unconditionally, so no branch delays the wait counts) while the
      // current group's LDS reads and fma chain run.
      const int2 *ej = ell + j;
      if (ell16) {
        // 32 sources per column, eight per 16-byte load ([4][N][8] u16), with their weights in the
        // grouping of 4 (w8, two 16-byte loads per eight) or the layer's one weight wc; all loads
        // are in flight before the first group's LDS reads
        uint4 ix[4];
        float4 wq[8];
#pragma unroll
        for (int g = 0; g < 4; ++g) ix[g] = ell16[(size_t)g * ncols + j];
        if (w8) {
          const float4 *w4 = reinterpret_cast<const float4 *>(w8);
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            wq[2 * g] = w4[(size_t)(2 * g) * ncols + j];
            wq[2 * g + 1] = w4[(size_t)(2 * g + 1) * ncols + j];
          }
        } else {
#pragma unroll
          for (int i = 0; i < 8; ++i) wq[i] = make_float4(wc, wc, wc, wc);
        }
        // the 32 terms in order, each slot's LDS read issued kLdsAhead slots before its fmas (a
        // rotating buffer, so reads stay in flight across the groups of eight)
        auto src_of = [&](int sl) {
          const uint4 &g = ix[sl / 8];
          const unsigned pr = (sl % 8) < 2 ? g.x : (sl % 8) < 4 ? g.y : (sl % 8) < 6 ? g.z : g.w;
          return (sl & 1) ? (pr >> 16) : (pr & 0xffffu);
        };
        auto w_of = [&](int sl) {
          const float4 &q = wq[sl / 4];
          return (sl % 4) == 0 ? q.x : (sl % 4) == 1 ? q.y : (sl % 4) == 2 ? q.z : q.w;
        };
        auto rd = [&](int sl) { return *reinterpret_cast<const float4 *>(tile + src_of(sl) * (unsigned)(B * 4) + qoff); };
        float4 buf[kLdsAhead];
#pragma unroll
        for (int q = 0; q < kLdsAhead; ++q) buf[q] = rd(q);
#pragma unroll
        for (int sl = 0; sl < 32; ++sl) {
          const float4 v = buf[sl % kLdsAhead];
          if (sl + kLdsAhead < 32) buf[sl % kLdsAhead] = rd(sl + kLdsAhead);
          const float w = w_of(sl);
          a0 = fmaf(v.x, w, a0);
          a1 = fmaf(v.y, w, a1);
          a2 = fmaf(v.z, w, a2);
          a3 = fmaf(v.w, w, a3);
        }
      } else if constexpr (KC > 0) {
        static_assert(KC % 8 == 0, "KC must be a multiple of 8");
        int2 cur[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) cur[q] = ej[(size_t)q * N];
#pragma unroll 1
        for (int g = 0; g < KC - 8; g += 8) {
          int2 nxt[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) nxt[q] = ej[(size_t)(g + 8 + q) * N];
          float4 v[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) v[q] = *reinterpret_cast<const float4 *>(tile + cur[q].x + qoff);
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const float wv = __int_as_float(cur[q].y);
            a0 = fmaf(v[q].x, wv, a0);
            a1 = fmaf(v[q].y, wv, a1);
            a2 = fmaf(v[q].z, wv, a2);
            a3 = fmaf(v[q].w, wv, a3);
          }
#pragma unroll
          for (int q = 0; q < 8; ++q) cur[q] = nxt[q];
        }
        float4 v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = *reinterpret_cast<const float4 *>(tile + cur[q].x + qoff);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const float wv = __int_as_float(cur[q].y);
          a0 = fmaf(v[q].x, wv, a0);
          a1 = fmaf(v[q].y, wv, a1);
          a2 = fmaf(v[q].z, wv, a2);
          a3 = fmaf(v[q].w, wv, a3);
        }
      } else {
        for (int s2 = 0; s2 < K; ++s2) {
          const int2 p = ej[(size_t)s2 * N];
          const float4 v = *reinterpret_cast<const float4 *>(tile + p.x + qoff);
          const float wv = __int_as_float(p.y);
          a0 = fmaf(v.x, wv, a0);
          a1 = fmaf(v.y, wv, a1);
          a2 = fmaf(v.z, wv, a2);
          a3 = fmaf(v.w, wv, a3);
        }
      }
      const float bj = bias[col];
      const float y[4] = {activate(a0, bj, ymax), activate(a1, bj, ymax), activate(a2, bj, ymax),
                          activate(a3, bj, ymax)};
#pragma unroll
      for (int c4 = 0; c4 < 4; ++c4) {
        if (row[c4] >= 0) {
          yout[(size_t)row[c4] * N + col] = y[c4];
          if (y[c4] > 0.0f) live_mask |= 1 << c4;
        }
      }
    }
#pragma unroll
    for (int c4 = 0; c4 < 4; ++c4)
      if (live_mask & (1 << c4)) rowlive[quad * 4 + c4] = 1;
    __syncthreads();
    if (tid < 64) {
      const unsigned long long m = __ballot(tid < nvalid && rowlive[tid] != 0);
      if (tid == 0 && m) atomicOr(&masks[t], (unsigned)m);
      if (count_nz && tid < nvalid && rowany[tid]) rownz[ids[p0 + tid]] = 1;
    }
    if (tid < B) {
      rowlive[tid] = 0;
      rowany[tid] = 0;
    }
    __syncthreads();
  }
}

// A pointer or a number that is the same in every lane, in scalar registers.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <class T>
__device__ __forceinline__ T *uniform(T *p) {
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  return reinterpret_cast<T *>(((unsigned long long)(unsigned)uniform((int)(v >> 32)) << 32) |
                               (unsigned)uniform((int)(unsigned)v));
}
// p[i] of global memory, the base in scalar registers and a 32-bit offset in a vector one
template <class T>
__device__ __forceinline__ T at32(const T *p, unsigned i) {
  typedef const char __attribute__((address_space(1))) *global_bytes;
  typedef const T __attribute__((address_space(1))) *global_t;
  return *(global_t)((global_bytes)p + i * (unsigned)sizeof(T));
}
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// The rows (bits) of a wave in which any lane's flag is set: lane holds rows 4 (lane % LPO) + c, c < RPL,
// flag bit c.
template <int LPO, int RPL>
__device__ __forceinline__ unsigned wave_rows(unsigned flags) {
  constexpr unsigned long long kEvery = LPO == 1   ? ~0ull
                                        : LPO == 2 ? 0x5555555555555555ull
                                        : LPO == 4 ? 0x1111111111111111ull
                                                   : 0x0101010101010101ull;
  unsigned bits = 0u;
#pragma unroll
  for (int c = 0; c < RPL; ++c) {
    const unsigned long long m = __ballot((flags >> c) & 1u);
#pragma unroll
    for (int q = 0; q < LPO; ++q) bits |= ((m >> q) & kEvery) != 0ull ? 1u << (RPL * q + c) : 0u;
  }
  return bits;
}

// k_layer_lds for a layer of 32-source lists with per-edge weights and N % 4 == 0 (the default kernels on
// such layers): same tiles, lanes, sums and placement. The lists of a round are replaced by the next
// round's (or the next item's first) 8 terms at a time as they are summed, and a wave that has
// finished an item loads the next one's rows while the others finish, so that neither latency is
// waited for between the LDS reads.
// Bound: the LDS reads, 64% of the time (60% of that bank conflicts, see bank_placement). 4096 neurons,
// 143,000 rows in 4 layers: 2.49 -> 2.21 ms; 1024 neurons, 10 layers of 60,000 rows and fewer: 1.00 ->
// 0.87 ms. A multiply-add that forms an LDS address in one instruction instead of two changed nothing.
template <int B>
__global__ __launch_bounds__(1024) void k_layer_lds32(const float *__restrict__ yin, float *__restrict__ yout, int N,
                                                      const u32x4 *__restrict__ ell16, const f32x4 *__restrict__ w8,
                                                      const float *__restrict__ bias, float ymax,
                                                      const int *__restrict__ ids, const int *__restrict__ count,
                                                      unsigned *__restrict__ masks, int *__restrict__ rownz,
                                                      const unsigned short *__restrict__ place) {
  static_assert(B == 8 || B == 16 || B == 32, "2 to 8 lanes per output");
  constexpr int LPO = B / 4;    // lanes per output, 4 rows each
  constexpr int OPW = 64 / LPO; // outputs per wave instruction
  constexpr int kPerRound = 16 * OPW;
  constexpr int kAhead = 5;
  constexpr int kStage = kLdsTileBytes / 64 / 1024;  // 4 x 4 blocks of the tile per thread
  extern __shared__ float4 smem[];
  const char *tile = reinterpret_cast<const char *>(smem);
  float *tilef = reinterpret_cast<float *>(smem);
  __shared__ unsigned rowlive, rowany;
  const int R = *count;
  const int ntiles = (R + B - 1) / B;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int quad = lane % LPO, jl = lane / LPO;
  const int rounds = (N + kPerRound - 1) / kPerRound;
  const Chunking ch = chunking(ntiles, rounds);
  const int items = ntiles * ch.nchunks;
  if ((int)blockIdx.x >= items) return;  // uniform over the workgroup
  if (tid == 0) {
    rowlive = 0u;
    rowany = 0u;
  }
  const int NQ = N >> 2;
  // this thread's blocks of the tile: rows 4 quad .., neurons 4 q .. with q = (u 1024 + tid) / LPO
  const int q0 = tid / LPO;
  unsigned rk[kStage][2];  // their tile rows, two per word
#pragma unroll
  for (int u = 0; u < kStage; ++u) {
    const int q = min(q0 + u * (1024 / LPO), NQ - 1);
    if (place) {
      const u32x2 x = at32(reinterpret_cast<const u32x2 *>(place), (unsigned)q);
      rk[u][0] = x.x;
      rk[u][1] = x.y;
    } else {
      rk[u][0] = (unsigned)(4 * q) | ((unsigned)(4 * q + 1) << 16);
      rk[u][1] = (unsigned)(4 * q + 2) | ((unsigned)(4 * q + 3) << 16);
    }
  }
  // row ids of this lane's 4 rows of item w (rows past the list: the last row, never stored)
  auto take_ids = [&](int w, int (&id)[4]) {
    const int p = w / ch.nchunks * B + quad * 4;
#pragma unroll
    for (int c = 0; c < 4; ++c) id[c] = ids[min(p + c, R - 1)];
  };
  float4 v[kStage][4];
  auto load_rows = [&](const int (&id)[4]) {
#pragma unroll
    for (int u = 0; u < kStage; ++u) {
      const int q = min(q0 + u * (1024 / LPO), NQ - 1);
#pragma unroll
      for (int c = 0; c < 4; ++c) v[u][c] = reinterpret_cast<const float4 *>(yin + (size_t)id[c] * N)[q];
    }
  };
  u32x4 ix[4];
  f32x4 wq[8];
  auto load_group = [&](int g, unsigned at) {
    ix[g] = at32(ell16, (unsigned)(g * N) + at);
    wq[2 * g] = at32(w8, (unsigned)(2 * g * N) + at);
    wq[2 * g + 1] = at32(w8, (unsigned)((2 * g + 1) * N) + at);
  };
  // the first position of this lane in item w
  auto first = [&](int w) { return (w % ch.nchunks) * ch.rounds_per_chunk * kPerRound + wave * OPW + jl; };
  int id[4], nid[4];
  take_ids(blockIdx.x, id);
  load_rows(id);
  {
    const unsigned at = (unsigned)min(first(blockIdx.x), N - 1);
#pragma unroll
    for (int g = 0; g < 4; ++g) load_group(g, at);
  }
  lds_barrier();  // the cleared words: a wave reports nonzero inputs before the first item's own barrier
  for (int w = blockIdx.x; w < items; w += gridDim.x) {
    const int t = w / ch.nchunks, c = w % ch.nchunks;
    const int nvalid = min(B, R - t * B);
    const bool count_nz = rownz != nullptr && c == 0;
    // ---- the rows as tile[place[k]][b]
    unsigned any = 0u;
#pragma unroll
    for (int u = 0; u < kStage; ++u) {
      if (q0 + u * (1024 / LPO) < NQ) {
        float *dst = tilef + quad * 4;
        *reinterpret_cast<float4 *>(dst + (rk[u][0] & 0xffffu) * B) = make_float4(v[u][0].x, v[u][1].x, v[u][2].x, v[u][3].x);
        *reinterpret_cast<float4 *>(dst + (rk[u][0] >> 16) * B) = make_float4(v[u][0].y, v[u][1].y, v[u][2].y, v[u][3].y);
        *reinterpret_cast<float4 *>(dst + (rk[u][1] & 0xffffu) * B) = make_float4(v[u][0].z, v[u][1].z, v[u][2].z, v[u][3].z);
        *reinterpret_cast<float4 *>(dst + (rk[u][1] >> 16) * B) = make_float4(v[u][0].w, v[u][1].w, v[u][2].w, v[u][3].w);
        if (count_nz)
#pragma unroll
          for (int b = 0; b < 4; ++b) any |= (any_nonzero(v[u][b]) ? 1u : 0u) << b;
      }
    }
    const int next = min(w + (int)gridDim.x, items - 1);
    take_ids(next, nid);
    if (count_nz) {
      const unsigned rows = wave_rows<LPO, 4>(any);
      if (lane == 0 && rows) atomicOr(&rowany, rows);
    }
    lds_barrier();
    // ---- lane (quad, jl) owns rows 4 quad .. of output j
    const char *tq = tile + quad * 16;
    unsigned lm = 0u;
    const int r_end = min(rounds, (c + 1) * ch.rounds_per_chunk);
    int todo = r_end - c * ch.rounds_per_chunk, j = first(w);
#pragma unroll 1
    for (; todo > 0; --todo) {
      asm volatile("" : "+s"(todo));  // (one body for every round)
      const int jn = todo == 1 ? first(next) : j + kPerRound;
      const unsigned at = (unsigned)min(jn, N - 1);
      const float bj = at32(bias, (unsigned)min(j, N - 1));
      float a[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      auto rd = [&](int sl) {
        const unsigned pr = ix[sl / 8][(sl % 8) / 2];
        return *reinterpret_cast<const float4 *>(tq + ((sl & 1) ? (pr >> 16) : (pr & 0xffffu)) * (unsigned)(B * 4));
      };
      float4 buf[kAhead];
#pragma unroll
      for (int q = 0; q < kAhead; ++q) buf[q] = rd(q);
#pragma unroll
      for (int sl = 0; sl < 32; ++sl) {
        __builtin_amdgcn_sched_barrier(0);
        const float ws = wq[sl / 4][sl % 4];
        const float4 y = buf[sl % kAhead];
        a[0] = fmaf(y.x, ws, a[0]);
        a[1] = fmaf(y.y, ws, a[1]);
        a[2] = fmaf(y.z, ws, a[2]);
        a[3] = fmaf(y.w, ws, a[3]);
        if (sl + kAhead < 32) buf[sl % kAhead] = rd(sl + kAhead);
        if (sl % 8 == 7) {
          // (summed here, also on lanes past the last column, whose sums are not stored)
          pin4(a[0], a[1], a[2], a[3]);
          load_group(sl / 8, at);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (j < N) {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const float y = activate(a[b], bj, ymax);
          if (quad * 4 + b < nvalid) {
            yout[(size_t)id[b] * N + j] = y;
            lm |= (y > 0.0f ? 1u : 0u) << b;
          }
        }
      }
      j = jn;
    }
    // a wave that is done loads the next item's rows while the others finish
    load_rows(nid);
    mem_fence_compiler();
    const unsigned rows = wave_rows<LPO, 4>(lm);
    if (lane == 0 && rows) atomicOr(&rowlive, rows);
    lds_barrier();  // every read of the tile is done
    if (tid < 64) {
      const unsigned m = rowlive, nz = rowany;
      if (tid == 0 && m) atomicOr(&masks[t], m);
      if (count_nz && tid < nvalid && ((nz >> tid) & 1u)) rownz[ids[t * B + tid]] = 1;
      if (tid == 0) {
        rowlive = 0u;
        rowany = 0u;
      }
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) id[b] = nid[b];
    lds_barrier();
  }
}

// Device view of one layer for kernels that run several layers in one launch.
struct LayerPtr {
  const int2 *ell;     // slot-major ELL, offsets in units of 1 << ell_shift bytes per source
  const uint4 *ell16;  // layer with 32 sources per column: [4][D][8] u16 sources, else null
  const float *w8;     // with ell16: the weights, [8][D][4] fp32 (four per 16-byte load); null for a
                       // uniform layer (weight w)
  const float *bias;
  const int *cols;     // with ell16: the D columns computed (null: all N, D = N)
  float w;             // the weight of a one-weight layer
  int K;
  int D;
};

// RPL consecutive fp32 rows of one source, read or written as one LDS access
template <int RPL>
__device__ __forceinline__ void lds_rows_load(const char *p, float (&v)[RPL]) {
  if constexpr (RPL == 4) {
    const float4 t = *reinterpret_cast<const float4 *>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else if constexpr (RPL == 2) {
    const float2 t = *reinterpret_cast<const float2 *>(p);
    v[0] = t.x; v[1] = t.y;
  } else {
    v[0] = *reinterpret_cast<const float *>(p);
  }
}
template <int RPL>
__device__ __forceinline__ void lds_rows_store(float *p, const float (&v)[RPL]) {
  if constexpr (RPL == 4) *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
  else if constexpr (RPL == 2) *reinterpret_cast<float2 *>(p) = make_float2(v[0], v[1]);
  else *p = v[0];
}

// Layers [l0, L) of the live rows listed in ids (count *count), in one launch: workgroup g keeps
// list positions [gB, gB + B) in LDS across all the layers, as two tiles [k][B] (the layer's input
// and its output), so between layers nothing goes through global memory and nothing waits for other
// workgroups (rows are independent, Sec. V). A lane holds RPL = min(B, 4) rows: lane = (quad = lane
// % (B/RPL): rows RPL quad .. RPL quad + RPL - 1, output slot lane / (B/RPL)); each term is one LDS
// read of RPL rows (16, 8 or 4 bytes) and RPL fmas, in ascending source order as everywhere. Small
// B spreads a short list over more CUs. After every layer the workgroup adds its live rows to
// counts[l + 1] and stops once none is left (rows that die stay dead). Rows still live after layer
// L - 1 are written to yout (row-major, by row id) and marked in masks (one bit per list position)
// for the final compaction. A layer with cols computes only those columns (the others are never
// read: the next layer's sources are representatives, and final rows are expanded on the host).
// Dynamic LDS: 2 * N * B floats.
template <int B>
__global__ __launch_bounds__(1024) void k_layers_lds(const float *__restrict__ yin, float *__restrict__ yout, int N,
                                                     const LayerPtr *__restrict__ lp, int l0, int L, float ymax,
                                                     const int *__restrict__ ids, const int *__restrict__ count,
                                                     int *__restrict__ counts, unsigned *__restrict__ masks,
                                                     int ell_shift) {
  static_assert(B == 1 || B == 2 || B == 4 || B == 8 || B == 16, "lanes hold up to 4 rows, at most 4 lanes per output");
  constexpr int RPL = B < 4 ? B : 4;
  extern __shared__ float4 smem[];
  __shared__ unsigned livebits[2];
  float *ta = reinterpret_cast<float *>(smem);
  float *tc = ta + (size_t)N * B;
  const int R = *count;
  const int p0 = blockIdx.x * B;
  if (p0 >= R) return;  // uniform over the workgroup
  const int nvalid = min(B, R - p0);
  const unsigned valid = (1u << nvalid) - 1u;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
  constexpr int LPO = B / RPL, OPW = 64 / LPO;
  const int quad = lane % LPO, jl = lane / LPO;
  const int per_round = nw * OPW;
  // stage the rows as ta[k][b] (reads run along k); positions past the list are zero
  for (int it = tid; it < N * B; it += blockDim.x) {
    const int b = it / N, k = it % N;
    ta[(size_t)k * B + b] = b < nvalid ? yin[(size_t)ids[p0 + b] * N + k] : 0.0f;
  }
  unsigned lb = valid;
  int l = l0;
  for (; l < L; ++l) {
    const LayerPtr P = lp[l];
    // livebits[l & 1] was last read before the barrier at the top of layer l - 1
    if (tid == 0) livebits[l & 1] = 0u;
    __syncthreads();  // ta is complete, and every read of tc (the layer before's input) is done
    unsigned lm = 0u;
    const char *tq = reinterpret_cast<const char *>(ta) + quad * (RPL * 4);
    const int ncols = P.ell16 ? P.D : N;
    const int rounds = (ncols + per_round - 1) / per_round;
    for (int r = 0; r < rounds; ++r) {
      const int jp = r * per_round + wave * OPW + jl;
      if (jp >= ncols) break;
      const int j = P.cols ? P.cols[jp] : jp;
      float a[RPL];
#pragma unroll
      for (int c = 0; c < RPL; ++c) a[c] = 0.0f;
      if (P.ell16) {
        // 32 sources, eight per 16-byte load ([4][D][8] u16), and their weights (eight per two
        // 16-byte loads from w8, or the layer's one weight); every load in flight first
        uint4 ix[4];
        float4 wq[8];
#pragma unroll
        for (int g = 0; g < 4; ++g) ix[g] = P.ell16[(size_t)g * ncols + jp];
        if (P.w8) {
          const float4 *w4 = reinterpret_cast<const float4 *>(P.w8);
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            wq[2 * g] = w4[(size_t)(2 * g) * ncols + jp];
            wq[2 * g + 1] = w4[(size_t)(2 * g + 1) * ncols + jp];
          }
        } else {
#pragma unroll
          for (int i = 0; i < 8; ++i) wq[i] = make_float4(P.w, P.w, P.w, P.w);
        }
        // the 32 terms in order, each slot's LDS read issued kLdsAhead slots before its fmas
        auto src_of = [&](int sl) {
          const uint4 &g = ix[sl / 8];
          const unsigned pr = (sl % 8) < 2 ? g.x : (sl % 8) < 4 ? g.y : (sl % 8) < 6 ? g.z : g.w;
          return (sl & 1) ? (pr >> 16) : (pr & 0xffffu);
        };
        auto w_of = [&](int sl) {
          const float4 &q = wq[sl / 4];
          return (sl % 4) == 0 ? q.x : (sl % 4) == 1 ? q.y : (sl % 4) == 2 ? q.z : q.w;
        };
        float buf[kLdsAhead][RPL];
#pragma unroll
        for (int q = 0; q < kLdsAhead; ++q) lds_rows_load<RPL>(tq + src_of(q) * (unsigned)(B * 4), buf[q]);
#pragma unroll
        for (int sl = 0; sl < 32; ++sl) {
          float v[RPL];
#pragma unroll
          for (int c = 0; c < RPL; ++c) v[c] = buf[sl % kLdsAhead][c];
          if (sl + kLdsAhead < 32) lds_rows_load<RPL>(tq + src_of(sl + kLdsAhead) * (unsigned)(B * 4), buf[sl % kLdsAhead]);
          const float w = w_of(sl);
#pragma unroll
          for (int c = 0; c < RPL; ++c) a[c] = fmaf(v[c], w, a[c]);
        }
      } else {
        for (int sl = 0; sl < P.K; ++sl) {
          const int2 e = P.ell[(size_t)sl * N + j];
          float v[RPL];
          lds_rows_load<RPL>(tq + ((unsigned)e.x >> ell_shift) * (unsigned)(B * 4), v);
          const float wv = __int_as_float(e.y);
#pragma unroll
          for (int c = 0; c < RPL; ++c) a[c] = fmaf(v[c], wv, a[c]);
        }
      }
      const float bj = P.bias[j];
      float y[RPL];
      unsigned bits = 0u;
#pragma unroll
      for (int c = 0; c < RPL; ++c) {
        y[c] = activate(a[c], bj, ymax);
        bits |= (y[c] > 0.0f ? 1u : 0u) << c;
      }
      lds_rows_store<RPL>(tc + (size_t)j * B + quad * RPL, y);
      lm |= bits << (RPL * quad);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) lm |= __shfl_xor(lm, d, 64);
    if (lane == 0 && lm) atomicOr(&livebits[l & 1], lm);
    __syncthreads();
    lb = livebits[l & 1] & valid;
    if (tid == 0 && lb) atomicAdd(&counts[l + 1], __popc(lb));
    float *t = ta;
    ta = tc;
    tc = t;
    if (!lb) break;
  }
  if (l == L && lb) {
    // ta holds the output of layer L - 1
    for (int it = tid; it < N * B; it += blockDim.x) {
      const int b = it / N, k = it % N;
      if ((lb >> b) & 1u) yout[(size_t)ids[p0 + b] * N + k] = ta[(size_t)k * B + b];
    }
    if (tid < B && ((lb >> tid) & 1u)) atomicOr(&masks[(p0 + tid) >> 5], 1u << ((p0 + tid) & 31));
  }
}

// The helper of a fused launch that leaves CUs idle: on the XCD of worker x < 8 a workgroup loads one word of
// each 128-byte line of the layers' lists, at most kFetchAhead layers ahead of that worker, so that the
// XCD's workers find them in its L2 (which holds about 20 layers of 1024 neurons). Every wait ends: the
// worker stores kPaceDone when it ends, and after kFetchPolls polls the helper gives up.
// One layer of 1024 neurons for one row takes 1.84 us with its lists in the L2 and 2.3 from beyond it (1.87 on
// average with the helper); 120 layers, with the final row, 336 -> 280 us a pass; 64 rows x 30 layers of 1000 134 -> 124. Two and
// four helpers per XCD were slower (293 us).
constexpr int kFetchAhead = 12, kPaceEvery = 4, kPaceDone = 0x7fffffff, kFetchPolls = 1 << 14;
__device__ void fetch_lists(const LayerPtr *__restrict__ lp, int l0, int L, int N, const int *__restrict__ pace) {
  __shared__ int at;
  int reached = l0;
  for (int l = l0 + 1; l < L; ++l) {
    if (l > reached + kFetchAhead) {
      if (threadIdx.x == 0) {
        int v = 0;
        for (int i = 0; i < kFetchPolls; ++i) {
          v = __hip_atomic_load(pace, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (l <= v || l - v <= kFetchAhead) break;
          __builtin_amdgcn_s_sleep(8);
          if (i == kFetchPolls - 1) v = kPaceDone;
        }
        at = v;
      }
      __syncthreads();
      reached = at;
      __syncthreads();
      if (reached == kPaceDone) return;  // uniform
    }
    // lines of 128 bytes: the sources (64 bytes per column), the weights (128), columns and biases (4 each)
    const int n1 = (N + 1) / 2, n2 = n1 + N, n3 = n2 + (N + 31) / 32, n4 = n3 + (N + 31) / 32;
    for (int i = threadIdx.x; i < n4; i += 1024) {
      const LayerPtr *q = lp + l;
      const int *a;
      if (i < n1)
        a = reinterpret_cast<const int *>(q->ell16) + (size_t)i * 32;
      else if (i < n2)
        a = reinterpret_cast<const int *>(q->w8) + (size_t)(i - n1) * 32;
      else if (i < n3)
        a = q->cols + (i - n2) * 32;
      else
        a = reinterpret_cast<const int *>(q->bias) + (i - n3) * 32;
      const int v = *a;
      asm volatile("" : : "v"(v));
    }
  }
}

// k_layers_lds for networks whose every layer has 32-source lists in grouped order with per-edge weights
// (the default kernels on such layers): same tiles, lanes and sums. The lists do not depend on the rows,
// so they are loaded a round ahead, also across the end of a layer: the registers of a group of 8
// terms take the next round's group (or the next layer's) as soon as it has been summed. A layer
// ends with one barrier, for LDS alone (a full one would wait for the lists too), and the live rows
// are counted in registers, 64 layers at a time.
// Bound: the LDS reads (random rows; see conflict_grouped_order) and, for one or two rows, the lists, 6
// bytes per edge through one CU's L1. Per layer at 1024 neurons, k_layers_lds -> this: 3.55 -> 2.30 us
// (one row; 1.87 with fetch_lists), 3.48 -> 2.38 (two rows per workgroup), 10.9 -> 8.4 (16 rows); at 4096
// 12.0 -> 9.4 (one row), 9.7 -> 8.6 (two).
template <int B>
__global__ __launch_bounds__(1024) void k_layers_lds32(const float *__restrict__ yin, float *__restrict__ yout, int N,
                                                       const LayerPtr *__restrict__ lp, int l0, int L, float ymax,
                                                       const int *__restrict__ ids, const int *__restrict__ count,
                                                       int *__restrict__ counts, unsigned *__restrict__ masks,
                                                       int *__restrict__ rownz, int *__restrict__ pace, int workers) {
  constexpr int RPL = B < 4 ? B : 4;
  constexpr int LPO = B / RPL, OPW = 64 / LPO;
  constexpr int kAhead = 6;  // LDS reads in flight ahead of their fmas
  extern __shared__ float4 smem[];
  // live rows of layer l in livebits[l % 3]; a word is cleared one layer before its use, when every
  // wave is past its last reading
  __shared__ unsigned livebits[3];
  float *ta = reinterpret_cast<float *>(smem);
  float *tc = ta + (size_t)N * B;
  const int R = *count;
  const int p0 = blockIdx.x * B;
  if ((int)blockIdx.x >= workers) {
    // (workers is a multiple of 8: helper and worker x are on one XCD)
    const int x = (int)blockIdx.x & 7;
    if (x * B < R) fetch_lists(lp, l0, L, N, pace + x);
    return;
  }
  if (p0 >= R) return;  // uniform over the workgroup
  const bool paces = pace != nullptr && blockIdx.x < 8;
  const int nvalid = min(B, R - p0);
  const unsigned valid = (1u << nvalid) - 1u;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int quad = lane % LPO, jl = lane / LPO;
  constexpr int kPerRound = 16 * OPW;
  const int j0 = wave * OPW + jl;  // this lane's output position in a round
  const int rounds = (N + kPerRound - 1) / kPerRound;
  // the lists of the round ahead: sources and weights of 4 groups of 8 terms, and the output column
  u32x4 ix[4];
  f32x4 wq[8];
  int col;
  const u32x4 *q16 = nullptr;
  const f32x4 *q8 = nullptr;
  const int *qcols = nullptr;
  auto take = [&](int l, const float **bias) {
    const LayerPtr *q = lp + l;
    q16 = uniform(reinterpret_cast<const u32x4 *>(q->ell16));
    q8 = uniform(reinterpret_cast<const f32x4 *>(q->w8));
    qcols = uniform(q->cols);
    *bias = uniform(q->bias);
  };
  const float *bias = nullptr, *bias_next = nullptr;
  take(l0, &bias);
  {
    const unsigned at = (unsigned)min(j0, N - 1);
    col = at32(qcols, at);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      ix[g] = at32(q16, (unsigned)(g * N) + at);
      wq[2 * g] = at32(q8, (unsigned)(2 * g * N) + at);
      wq[2 * g + 1] = at32(q8, (unsigned)((2 * g + 1) * N) + at);
    }
  }
  // stage the rows as ta[k][b] (reads run along k); positions past the list are zero
  for (int it = tid; it < N * B; it += 1024) {
    const int b = it / N, k = it % N;
    const float x = b < nvalid ? yin[(size_t)ids[p0 + b] * N + k] : 0.0f;
    ta[(size_t)k * B + b] = x;
    // (layer 0: rows with a nonzero input)
    if (rownz && x != 0.0f) rownz[ids[p0 + b]] = 1;
  }
  if (tid < 3) livebits[tid] = 0u;
  lds_barrier();
  unsigned lb = valid;
  int hist = 0;  // wave 0, lane l % 64: live rows after layer l
  int l = l0;
  for (; l < L; ++l) {
    if (tid == 0) livebits[(l + 1) % 3] = 0u;
    if (paces && tid == 0 && l % kPaceEvery == 0)
      __hip_atomic_store(pace + blockIdx.x, l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned lm = 0u;  // this lane's rows with a positive output: bit c is row RPL quad + c
    const char *tq = reinterpret_cast<const char *>(ta) + quad * (RPL * 4);
    int todo = rounds, jp = j0;
#pragma unroll 1
    for (; todo > 0; --todo) {
      asm volatile("" : "+s"(todo));  // (one body for every round)
      const int j = col;
      const float bj = at32(bias, (unsigned)j);
      // the round ahead: of this layer, or the first of the next (after the last layer: its own, unused)
      if (todo == 1) take(min(l + 1, L - 1), &bias_next);
      const int jn = todo == 1 ? j0 : jp + kPerRound;
      const unsigned at = (unsigned)min(jn, N - 1);
      col = at32(qcols, at);
      float a[RPL];
#pragma unroll
      for (int c = 0; c < RPL; ++c) a[c] = 0.0f;
      auto src_of = [&](int sl) {
        const unsigned pr = ix[sl / 8][(sl % 8) / 2];
        return (sl & 1) ? (pr >> 16) : (pr & 0xffffu);
      };
      float buf[kAhead][RPL];
#pragma unroll
      for (int q = 0; q < kAhead; ++q) lds_rows_load<RPL>(tq + src_of(q) * (unsigned)(B * 4), buf[q]);
#pragma unroll
      for (int sl = 0; sl < 32; ++sl) {
        __builtin_amdgcn_sched_barrier(0);
        const float w = wq[sl / 4][sl % 4];
#pragma unroll
        for (int c = 0; c < RPL; ++c) a[c] = fmaf(buf[sl % kAhead][c], w, a[c]);
        if (sl + kAhead < 32) lds_rows_load<RPL>(tq + src_of(sl + kAhead) * (unsigned)(B * 4), buf[sl % kAhead]);
        if (sl % 8 == 7) {
          // (summed here, also on lanes past the last column, whose sums are not stored)
#pragma unroll
          for (int c = 0; c < RPL; ++c) asm volatile("" : "+v"(a[c]));
          const int g = sl / 8;
          ix[g] = at32(q16, (unsigned)(g * N) + at);
          wq[2 * g] = at32(q8, (unsigned)(2 * g * N) + at);
          wq[2 * g + 1] = at32(q8, (unsigned)((2 * g + 1) * N) + at);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (jp < N) {
        float y[RPL];
#pragma unroll
        for (int c = 0; c < RPL; ++c) {
          y[c] = activate(a[c], bj, ymax);
          lm |= (y[c] > 0.0f ? 1u : 0u) << c;
        }
        lds_rows_store<RPL>(tc + (size_t)j * B + quad * RPL, y);
      }
      jp = jn;
    }
    const unsigned bits = wave_rows<LPO, RPL>(lm);
    if (lane == 0 && bits) atomicOr(&livebits[l % 3], bits);
    lds_barrier();  // tc is complete, every read of ta is done
    lb = livebits[l % 3] & valid;
    if (wave == 0) {
      if (lane == (l & 63)) hist = __popc(lb);
      if ((l & 63) == 63) {
        if (hist) atomicAdd(&counts[l - 63 + lane + 1], hist);
        hist = 0;
      }
    }
    float *t = ta;
    ta = tc;
    tc = t;
    bias = bias_next;
    if (!lb) break;
  }
  if (paces && tid == 0) __hip_atomic_store(pace + blockIdx.x, kPaceDone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // the layers since the last multiple of 64 (a lane whose layer did not run holds 0)
  if (wave == 0 && hist) atomicAdd(&counts[(min(l, L - 1) & ~63) + lane + 1], hist);
  if (l == L && lb) {
    // ta holds the output of layer L - 1
    for (int it = tid; it < N * B; it += 1024) {
      const int b = it / N, k = it % N;
      if ((lb >> b) & 1u) yout[(size_t)ids[p0 + b] * N + k] = ta[(size_t)k * B + b];
    }
    if (tid < B && ((lb >> tid) & 1u)) atomicOr(&masks[(p0 + tid) >> 5], 1u << ((p0 + tid) & 31));
  }
}

// Copy live rows into feature-major tiles of FMR rows: fm[t][k][b] = Y[ids[t*FMR + b]][k], zero
// for positions past the live count.
template <int FMR>
__global__ __launch_bounds__(256) void k_to_fm(const float *__restrict__ yin, float *__restrict__ fm, int N,
                                               const int *__restrict__ ids, const int *__restrict__ count,
                                               int *__restrict__ rownz) {
  const int R = *count;
  const int ntiles = (R + FMR - 1) / FMR;
  const size_t st = (size_t)gridDim.x * blockDim.x;
  if ((N & 3) == 0) {
    const int NQ = N >> 2;
    const size_t items = (size_t)ntiles * NQ * (FMR / 4);
    for (size_t it = blockIdx.x * (size_t)blockDim.x + threadIdx.x; it < items; it += st) {
      const int bq = (int)(it % (FMR / 4));
      const size_t rest = it / (FMR / 4);
      const int q = (int)(rest % NQ);
      const int t = (int)(rest / NQ);
      float4 v[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int p = t * FMR + bq * 4 + c;
        v[c] = (p < R) ? reinterpret_cast<const float4 *>(yin + (size_t)ids[p] * N)[q] : make_float4(0.f, 0.f, 0.f, 0.f);
        if (rownz && p < R && any_nonzero(v[c]) && !rownz[ids[p]]) rownz[ids[p]] = 1;
      }
      float4 *dst = reinterpret_cast<float4 *>(fm + ((size_t)t * N + 4 * q) * FMR + bq * 4);
      dst[0] = make_float4(v[0].x, v[1].x, v[2].x, v[3].x);
      dst[FMR / 4] = make_float4(v[0].y, v[1].y, v[2].y, v[3].y);
      dst[2 * (FMR / 4)] = make_float4(v[0].z, v[1].z, v[2].z, v[3].z);
      dst[3 * (FMR / 4)] = make_float4(v[0].w, v[1].w, v[2].w, v[3].w);
    }
  } else {
    const size_t items = (size_t)ntiles * N * FMR;
    for (size_t it = blockIdx.x * (size_t)blockDim.x + threadIdx.x; it < items; it += st) {
      const int b = (int)(it % FMR);
      const size_t rest = it / FMR;
      const int k = (int)(rest % N);
      const int t = (int)(rest / N);
      const int p = t * FMR + b;
      const float v = (p < R) ? yin[(size_t)ids[p] * N + k] : 0.0f;
      fm[((size_t)t * N + k) * FMR + b] = v;
      if (rownz && v != 0.0f && !rownz[ids[p]]) rownz[ids[p]] = 1;
    }
  }
}

// Weight layouts read by the global-tile kernels:
//   kWEll:  a layer of any width K: the slot-major ELL of (source offset, weight bits), K from the
//           launch (the general fallback);
//   kWOne:  32 sources per column as 16-bit lists src16[slot][column], one weight wc for the whole
//           layer (only with the equal-value kernels);
//   kWEdge: 32 sources per column as 16-bit lists src16[slot][column] and each edge's weight in
//           w32[slot][column] (6 bytes per edge).
constexpr int kWEll = 0, kWOne = 1, kWEdge = 2;

// Stage the 16-bit sources (and, for kWEdge, the weights) of outputs [c0, c0 + nout) of a layer
// into LDS as srcs[slot][CH] and wts[slot][CH], with 16-byte loads where the rows are aligned;
// outputs past nout get source 0 and weight 0 (they are computed but never stored).
template <int WM, int CH>
__device__ __forceinline__ void stage_lists(unsigned short *srcs, float *wts, const unsigned short *__restrict__ src16,
                                            const float *__restrict__ w32, int ncols, int c0, int nout) {
  static_assert(CH % 8 == 0, "whole 16-byte groups");
  for (int i = threadIdx.x; i < 32 * CH / 8; i += blockDim.x) {
    const int sl = i / (CH / 8), pr = (i % (CH / 8)) * 8;
    const unsigned short *sp = src16 + (size_t)sl * ncols + c0 + pr;
    uint4 v;
    if (pr + 7 < nout && (reinterpret_cast<uintptr_t>(sp) & 15) == 0) {
      v = *reinterpret_cast<const uint4 *>(sp);
    } else {
      unsigned o[4] = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int c = 0; c < 8; ++c) o[c >> 1] |= (pr + c < nout ? (unsigned)sp[c] : 0u) << (16 * (c & 1));
      v = make_uint4(o[0], o[1], o[2], o[3]);
    }
    *reinterpret_cast<uint4 *>(srcs + sl * CH + pr) = v;
  }
  if constexpr (WM == kWEdge) {
    for (int i = threadIdx.x; i < 32 * CH / 4; i += blockDim.x) {
      const int sl = i / (CH / 4), pr = (i % (CH / 4)) * 4;
      const float *wp = w32 + (size_t)sl * ncols + c0 + pr;
      float4 v;
      if (pr + 3 < nout && (reinterpret_cast<uintptr_t>(wp) & 15) == 0) {
        v = *reinterpret_cast<const float4 *>(wp);
      } else {
        v = make_float4(pr < nout ? wp[0] : 0.0f, pr + 1 < nout ? wp[1] : 0.0f, pr + 2 < nout ? wp[2] : 0.0f,
                        pr + 3 < nout ? wp[3] : 0.0f);
      }
      *reinterpret_cast<float4 *>(wts + sl * CH + pr) = v;
    }
  }
}

// Work split of one round of a layer on global tiles, tpx tiles per XCD (workgroup x runs on XCD
// x % 8; gridDim.x / 8 must be a multiple of tpx). ntl: tiles left from the round's first tile.
// With more than 8 tiles in the round, XCD x takes its tiles x, x + 8, ..., x + 8 (tpx - 1), one per
// group of its workgroups, each tile's chunks spread over the group; with at most 8 (always for
// tpx = 1), group 0 alone works and each tile's chunks are split over 8 / nt XCDs.
struct RoundSplit {
  int t;             // tile, relative to the round's first
  bool active;
  int cbeg, cend;    // the tile's chunks this XCD (part) covers
  int first, step;   // this workgroup's first chunk and stride
};
__device__ __forceinline__ RoundSplit round_split(int ntl, int tpx, int nchunks) {
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, per_xcd = gridDim.x >> 3;
  const int g = slot % tpx, per_group = per_xcd / tpx;
  const int nt = min(8 * tpx, ntl);
  RoundSplit r;
  if (nt > 8) {
    r.t = xcd + 8 * g;
    r.active = r.t < nt;
    r.cbeg = 0;
  } else {
    const int parts = nt > 0 ? 8 / nt : 1;
    r.t = xcd / parts;
    r.active = nt > 0 && g == 0 && xcd < nt * parts;
    r.cbeg = (xcd % parts) * ((nchunks + parts - 1) / parts);
    r.cend = min(nchunks, r.cbeg + (nchunks + parts - 1) / parts);
  }
  if (nt > 8) r.cend = nchunks;
  if (!r.active) r.cend = 0;
  r.first = r.cbeg + slot / tpx;
  r.step = per_group;
  return r;
}

// One round of a layer on global feature-major tiles of FMR = 32 rows: input tiles fin[t][k][b]
// (source k of list position 32t + b), output tiles fout in the same layout and positions; tiles
// [tile0, tile0 + 8) of the list, one per XCD. blockDim 256 (4 waves); a work item is a chunk of
// kGfmOutputs = 64 outputs. Lane = (row b = lane % 32, h = lane / 32): a source segment of 128
// bytes is read by 32 lanes with 4-byte loads (on gfx950 4-byte lane loads gather a segment three
// times faster than 16-byte ones), so a wave instruction serves 2 outputs; each lane runs the
// chains of the 8 consecutive outputs 16 wave + 8 h .. + 7, one slot ahead, and the results go out
// as 128-byte row segments. gridDim must be a multiple of 8: workgroup x runs on XCD x % 8, and the
// workgroups of XCD x share the output chunks of one tile, which therefore stays in that XCD's L2
// (or, for the widest layers, in the Infinity Cache) for the whole launch. With fewer than 8 tiles
// left, each tile's chunks are split over 8 / ntiles XCDs. With 16-bit lists (WM != kWEll) the
// chunk's sources (and kWEdge weights) are staged in LDS, so the gathers are the only per-output
// memory reads. Slots past the list's end hold zeros in fin and get zeros in fout.
//
// Workgroup 0 of the first round also does the list bookkeeping of the layer sequence: with
// count_out set (a layer that follows one without compaction) it counts the previous layer's live
// rows (masks_prev, complete since that kernel ended) into *count_out, and with masks_clear set it
// clears that buffer, the one the next layer will use (three buffers rotate by layer). With
// count_out set and no live row left (rows that die stay dead), the layer writes nothing.
// Live rows go to masks, or with spread set to the spread words of each tile (see or_mask). With
// cols set (kWOne only), the launch computes the ncols columns cols[p] alone, their source lists in
// src16 as [K][ncols]; the other columns equal one of these and are neither computed nor stored.
template <int WM>
__global__ __launch_bounds__(256) void k_layer_gfm(const float *__restrict__ fin, float *__restrict__ fout, int N,
                                                   const int2 *__restrict__ ell, int K,
                                                   const unsigned short *__restrict__ src16,
                                                   const float *__restrict__ w32, float wc,
                                                   const float *__restrict__ bias, float ymax,
                                                   const int *__restrict__ npos, unsigned *__restrict__ masks,
                                                   int tile0, const unsigned *__restrict__ masks_prev,
                                                   unsigned *__restrict__ masks_clear, int *__restrict__ count_out,
                                                   unsigned *__restrict__ spread, const int *__restrict__ cols,
                                                   int ncols, int tpx) {
  constexpr int FMR = 32, CH = kGfmOutputs, OPL = 8;
  static_assert(CH == 4 * 2 * OPL, "4 waves x 2 halves x OPL outputs");
  constexpr bool LISTS = WM != kWEll;
  __shared__ __align__(16) unsigned short srcs[LISTS ? 32 * CH : 8];
  __shared__ __align__(16) float wts[WM == kWEdge ? 32 * CH : 4];
  __shared__ float bstage[CH];
  __shared__ int cstage[CH];  // output column of each chunk position
  __shared__ unsigned rowmask;
  __shared__ int prev_live;
  const int R = *npos;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid < 64) {
    const int ntl = (R + FMR - 1) / FMR;
    int c = 0;
    if (count_out || (masks_clear && blockIdx.x == 0))
      for (int i = tid; i < ntl; i += 64) {
        if (count_out) c += __popc(masks_prev[i]);
        if (masks_clear && blockIdx.x == 0) masks_clear[i] = 0u;
      }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d, 64);
    if (tid == 0) {
      if (count_out && blockIdx.x == 0) *count_out = c;
      prev_live = count_out ? c : 1;
      rowmask = 0u;
    }
  }
  __syncthreads();
  const int nchunks = (ncols + CH - 1) / CH;
  const RoundSplit rs = round_split((R + FMR - 1) / FMR - tile0, tpx, nchunks);
  const bool active = rs.active && prev_live != 0;  // uniform over the workgroup
  const int t = tile0 + rs.t;
  const int cend = active ? rs.cend : 0;
  const int b = lane & 31, h = lane >> 5;
  const int nvalid = active ? min(FMR, R - t * FMR) : 0;
  const float *tb = fin + (size_t)t * N * FMR + b;
  float *ob = fout + (size_t)t * N * FMR + b;
  const int jl0 = wave * 2 * OPL + h * OPL;  // this lane's outputs in the chunk: jl0 .. jl0 + OPL - 1
  bool live = false;
  for (int chunk = rs.first; chunk < cend; chunk += rs.step) {
    const int c0 = chunk * CH;
    const int nout = min(CH, ncols - c0);
    __syncthreads();  // the previous chunk is done with srcs / wts / bstage / cstage
    for (int i = tid; i < CH; i += blockDim.x) {
      const int col = i < nout ? (cols ? cols[c0 + i] : c0 + i) : 0;
      cstage[i] = col;
      bstage[i] = i < nout ? bias[col] : 0.0f;
    }
    if constexpr (LISTS) stage_lists<WM, CH>(srcs, wts, src16, w32, ncols, c0, nout);
    __syncthreads();
    float acc[OPL];
#pragma unroll
    for (int i = 0; i < OPL; ++i) acc[i] = 0.0f;
    if constexpr (LISTS) {
      // software pipeline kDepth slots deep: a slot's gathers are issued kDepth - 1 slots before
      // its fmas (each gather is one row of one output, so the depth is what keeps enough
      // segments in flight to cover the L2 latency)
      constexpr int kDepth = 4;
      float g[kDepth][OPL];
      auto fetch = [&](int sl, int bf) {
        const unsigned short *sp = srcs + sl * CH + jl0;
#pragma unroll
        for (int i = 0; i < OPL; ++i) g[bf][i] = tb[(unsigned)sp[i] * (unsigned)FMR];
      };
#pragma unroll
      for (int sl = 0; sl < kDepth - 1; ++sl) fetch(sl, sl);
#pragma unroll
      for (int sl = 0; sl < 32; ++sl) {
        if (sl + kDepth - 1 < 32) fetch(sl + kDepth - 1, (sl + kDepth - 1) % kDepth);
        // the slot's weights from LDS (two 16-byte reads), while its gathers are in flight
        float wv[OPL];
        if constexpr (WM == kWEdge) {
          const float4 x = *reinterpret_cast<const float4 *>(wts + sl * CH + jl0);
          const float4 y = *reinterpret_cast<const float4 *>(wts + sl * CH + jl0 + 4);
          wv[0] = x.x; wv[1] = x.y; wv[2] = x.z; wv[3] = x.w;
          wv[4] = y.x; wv[5] = y.y; wv[6] = y.z; wv[7] = y.w;
        } else {
#pragma unroll
          for (int i = 0; i < OPL; ++i) wv[i] = wc;
        }
        mem_fence_compiler();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < OPL; ++i) acc[i] = fmaf(g[sl % kDepth][i], wv[i], acc[i]);
#pragma unroll
        for (int i = 0; i < OPL; i += 4) pin4(acc[i], acc[i + 1], acc[i + 2], acc[i + 3]);
      }
    } else {
      for (int sl = 0; sl < K; ++sl) {
#pragma unroll
        for (int i = 0; i < OPL; ++i) {
          const int2 e = ell[(size_t)sl * N + min(c0 + jl0 + i, N - 1)];
          acc[i] = fmaf(tb[(unsigned)e.x >> 2], __int_as_float(e.y), acc[i]);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < OPL; ++i) {
      const int jl = jl0 + i;
      if (jl < nout) {
        const float y = activate(acc[i], bstage[jl], ymax);
        __builtin_nontemporal_store(y, ob + (size_t)cstage[jl] * FMR);
        live |= y > 0.0f;
      }
    }
  }
  // rows of this tile that stayed live in any of this workgroup's chunks: lanes b and b + 32 are
  // row b
  const unsigned long long bl = __ballot(live);
  const unsigned lm = (unsigned)bl | (unsigned)(bl >> 32);
  __syncthreads();
  if (lane == 0 && lm) atomicOr(&rowmask, lm);
  __syncthreads();
  if (tid == 0) {
    const unsigned valid = nvalid >= 32 ? 0xffffffffu : ((1u << nvalid) - 1u);  // 0 when inactive
    if (active && (rowmask & valid)) or_mask(masks, spread, t, rowmask & valid);
  }
}

// One layer whose activations are fp32 rows in global memory, for widths up to kSegMaxNeurons: a
// workgroup takes 4 rows at a time (list positions 4i .. 4i + 3) and stages their values in LDS as
// [source][4 rows], so that one 16-byte LDS read serves an edge for 4 rows. kSegCap sources fit; a
// wider layer runs in S = 2 segments, [0, kSegCap) and then [N - kSegCap, N), and the sums of all
// the workgroup's outputs stay in registers across them (16 outputs x 4 rows per thread). Every
// column's sources are split between the segments in ascending order, so each sum is the same
// ascending chain as everywhere; the overlap of the segments lets the loader cut almost every
// column of 32 sources into 16 + 16. Columns hold any number of sources: the loader sorts them by
// their groups of 8 terms per segment and pads a block of 64 columns to its longest (padding is
// (row 0 of the segment, weight +0), a no-op term).
//   stream: groups of 8 terms of 64 columns, 3 KiB each: [64 lanes] of 8 u16 sources (within the
//     segment), then [64 lanes] of the first 4 and of the last 4 weights; a wave's groups follow each
//     other, so the next group is loaded while the current one is summed.
//   desc[s * nblk + k]: first group and number of groups of column block k in segment s; block k is
//     taken by wave k % 16 as its output k / 16.
//   colb[64 k + lane]: the column (kNoColumn: none) and its bias.
// Bound: the LDS reads (16 lanes at random rows take 3.06 of the cycles that conflict-free ones take, so
// at most 21 edge-rows per clock and CU; counted: 63-64% of the LDS's active cycles are conflicts, and it is
// active 68-71% of the time), then the rows' way in and out, which every CU takes at about the same time.
// Gathers of 128-byte segments from a resident L2
// (k_layer_gfm) end at 12, and reach 7.3. 15,000 live rows at 16384 neurons: 1.08 ms per layer against
// 1.83 for k_layer_gfm; columns of 1 to 48 sources at 10007 neurons, 3000 rows: 0.13 ms against 0.94.
// Tried: 16-byte loads and stores of the rows (8% slower: their 4-way conflicts in the LDS transposes),
// staggered starts of the workgroups (2%), LDS reads 3 to 8 terms ahead (5 is best by 1-5%), and columns
// regrouped at load time for fewer conflicts (2.7% faster, for 10% of the load time).
// With nsplit > 1 (fewer 4-row groups than CUs) nsplit workgroups share a group's outputs. With
// nsplit = 1 the workgroup knows which of its rows stay live: dead rows are not written, and the
// others go through LDS back into column order. map: the row of yin that holds list position p (null:
// p itself). rownz (layer 0): rows with a nonzero input.
constexpr int kSegThreads = 1024;
constexpr int kSegOutputs = 16;                // outputs per thread
constexpr int kSegMaxNeurons = kSegThreads * kSegOutputs;
constexpr int kSegCap = 10112;                 // sources in LDS: 158 KiB
constexpr int kSegAhead = 5;                   // LDS reads in flight ahead of the fmas
constexpr unsigned kNoColumn = 0x80000000u;
constexpr int kSegGroupWords = 192;            // uint4 words of a group
static_assert(2 * kSegCap >= kSegMaxNeurons && kSegCap * 16 + 1024 <= 160 * 1024, "two segments cover the widest layer");
// f(0), f(1), ..., each with its index as a compile-time constant (arrays indexed by it stay in
// registers whatever loops f holds)
template <class F, int... I>
__device__ __forceinline__ void static_for(F &&f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
// 16 times the low (half = 0) or high u16 of u, in one instruction (a word-select on the operand); four
// holds 4.
template <int HALF>
__device__ __forceinline__ unsigned word_times_16(unsigned u, unsigned four) {
  unsigned r;
  if constexpr (HALF == 0)
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0"
        : "=v"(r) : "v"(four), "v"(u));
  else
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1"
        : "=v"(r) : "v"(four), "v"(u));
  return r;
}

template <int S>
__global__ __launch_bounds__(kSegThreads) void k_layer_seg(
    const float *__restrict__ yin, float *__restrict__ yout, int N, const uint4 *__restrict__ stream,
    const int2 *__restrict__ desc, const uint2 *__restrict__ colb, int nblk, float ymax, const int *__restrict__ map,
    const int *__restrict__ npos, int nsplit, unsigned *__restrict__ masks, unsigned *__restrict__ spread,
    int *__restrict__ rownz, const int *__restrict__ ids) {
  extern __shared__ float4 tile[];  // (the only LDS: the tile starts at address 0, and two words follow it)
  unsigned &livebits = *reinterpret_cast<unsigned *>(tile + min(N, kSegCap));
  unsigned &anybits = *(&livebits + 1);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int R = *npos;
  const int nob = (nblk + 15) / 16;
  const int opw = (nob + nsplit - 1) / nsplit;
  const int items = (R + 3) / 4 * nsplit;
  const char *tb = reinterpret_cast<const char *>(tile);
  unsigned four = 4u;
  asm volatile("" : "+v"(four));
  const std::make_integer_sequence<int, kSegOutputs> outputs{};
  constexpr int kStage = (kSegCap + kSegThreads - 1) / kSegThreads;  // sources of a segment per thread
  const int nk = S == 1 ? N : kSegCap;                               // sources of a segment
  float v[kStage][4];
  const float *row[4];
  // the rows of an item (positions past the list repeat the last one; their sums are not stored)
  auto take_rows = [&](int it) {
    const int q0 = it / nsplit * 4;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int p = min(q0 + b, R - 1);
      // (uniform: the row address stays in scalar registers)
      row[b] = yin + (size_t)(unsigned)__builtin_amdgcn_readfirstlane(map ? map[p] : p) * (unsigned)N;
    }
  };
  // segment s of those rows, into registers (all of them assigned, so that none is live before)
  auto load = [&](int s) {
    const int k0 = s == 0 ? 0 : N - kSegCap;
    int t = tid;
    asm volatile("" : "+v"(t));  // (the offsets are formed here, not kept in registers across the sums)
#pragma unroll
    for (int u = 0; u < kStage; ++u) {
      const unsigned k = (unsigned)(k0 + min(u * kSegThreads + t, nk - 1));
#pragma unroll
      for (int b = 0; b < 4; ++b)
        v[u][b] = u * kSegThreads < nk
                      ? *reinterpret_cast<const float *>(reinterpret_cast<const char *>(row[b]) + k * 4u)
                      : 0.0f;
    }
  };
  if ((int)blockIdx.x >= items) return;  // uniform over the workgroup
  if (tid == 0) {
    livebits = 0u;
    anybits = 0u;
  }
  take_rows(blockIdx.x);
  load(0);
  for (int item = blockIdx.x; item < items; item += gridDim.x) {
    const int part = item % nsplit;
    const int p0 = item / nsplit * 4;
    const int nvalid = min(4, R - p0);
    const int o0 = part * opw;
    const int on = max(0, min(nob - o0, opw));  // outputs of each thread
    float acc[kSegOutputs][4];
#pragma unroll
    for (int o = 0; o < kSegOutputs; ++o)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[o][b] = 0.0f;
    unsigned any = 0u;
    uint2 cb[kSegOutputs];  // column and bias of each output
#pragma unroll
    for (int s = 0; s < S; ++s) {
      // lane o holds the description of this wave's block of output o
      const int blk = (o0 + lane) * 16 + wave;
      int2 d = make_int2(0, 0);
      if (lane < on && blk < nblk) d = desc[s * nblk + blk];
#pragma unroll
      for (int u = 0; u < kStage; ++u) {
        const int k = u * kSegThreads + tid;
        if (k < nk) tile[k] = make_float4(v[u][0], v[u][1], v[u][2], v[u][3]);
        if (rownz && k < nk)
#pragma unroll
          for (int b = 0; b < 4; ++b) any |= (v[u][b] != 0.0f ? 1u : 0u) << b;
      }
      int g = __builtin_amdgcn_readlane(d.x, 0);
      const uint4 *gp = stream + (size_t)g * kSegGroupWords + lane;
      uint4 ix = gp[0], w0 = gp[64], w1 = gp[128], jx, u0, u1;
      lds_barrier();
      static_for([&](auto oc) {
        constexpr int o = decltype(oc)::value;
        if (o >= on) return;
        // (the descriptions are read here, not hoisted: 32 scalar registers would spill)
        asm volatile("" : "+v"(d.x), "+v"(d.y));
        const int ng = __builtin_amdgcn_readlane(d.y, o);
        const int after = o + 1 < kSegOutputs ? __builtin_amdgcn_readlane(d.x, o + 1) : 0;
        // the sums of one group, whose lists are in (ix, w0, w1)
        auto sum = [&](const uint4 &ix, const uint4 &w0, const uint4 &w1) {
          const unsigned q[4] = {ix.x, ix.y, ix.z, ix.w};
          const float w[8] = {__uint_as_float(w0.x), __uint_as_float(w0.y), __uint_as_float(w0.z), __uint_as_float(w0.w),
                              __uint_as_float(w1.x), __uint_as_float(w1.y), __uint_as_float(w1.z), __uint_as_float(w1.w)};
          // LDS reads kSegAhead terms ahead of their fmas
          float4 x[kSegAhead];
          auto rd = [&](int t) {
            return *reinterpret_cast<const float4 *>(
                tb + ((t & 1) ? word_times_16<1>(q[t / 2], four) : word_times_16<0>(q[t / 2], four)));
          };
#pragma unroll
          for (int t = 0; t < kSegAhead; ++t) x[t] = rd(t);
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            __builtin_amdgcn_sched_barrier(0);
            const float4 y = x[t % kSegAhead];
            acc[o][0] = fmaf(y.x, w[t], acc[o][0]);
            acc[o][1] = fmaf(y.y, w[t], acc[o][1]);
            acc[o][2] = fmaf(y.z, w[t], acc[o][2]);
            acc[o][3] = fmaf(y.w, w[t], acc[o][3]);
            if (t + kSegAhead < 8) x[t % kSegAhead] = rd(t + kSegAhead);
          }
          __builtin_amdgcn_sched_barrier(0);
        };
        // a group's lists are loaded while the one before it is summed (the last one's successor is the
        // first group of the wave's next block); two register sets in turn
        auto lists = [&](int gi, uint4 &ix, uint4 &w0, uint4 &w1) {
          const uint4 *np = stream + (size_t)(unsigned)gi * kSegGroupWords;
          ix = np[lane];
          w0 = np[lane + 64];
          w1 = np[lane + 128];
          mem_fence_compiler();
        };
        int i = 0;
        for (; i + 1 < ng; i += 2) {
          lists(g + 1, jx, u0, u1);
          sum(ix, w0, w1);
          g = i + 2 < ng ? g + 2 : after;
          lists(g, ix, w0, w1);
          sum(jx, u0, u1);
        }
        if (i < ng) {
          g = after;
          lists(g, jx, u0, u1);
          sum(ix, w0, w1);
          ix = jx;
          w0 = u0;
          w1 = u1;
        }
      }, outputs);
      // a wave that is done loads what comes next while the others finish
      if (s + 1 < S) {
        load(s + 1);
      } else {
        const uint2 *cp = colb + (size_t)o0 * kSegThreads;
        static_for([&](auto oc) {
          constexpr int o = decltype(oc)::value;
          cb[o] = o < on ? cp[(unsigned)(o * kSegThreads + tid)] : make_uint2(kNoColumn, 0u);
        }, outputs);
      }
      mem_fence_compiler();
      lds_barrier();  // every read of the segment is done
    }
    unsigned lm = 0u;
    static_for([&](auto oc) {
      constexpr int o = decltype(oc)::value;
      if (o >= on) return;
      if (cb[o].x != kNoColumn) {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          acc[o][b] = activate(acc[o][b], __uint_as_float(cb[o].y), ymax);
          lm |= (acc[o][b] > 0.0f ? 1u : 0u) << b;
        }
        if (nsplit > 1) {
#pragma unroll
          for (int b = 0; b < 4; ++b)
            if (b < nvalid) yout[(size_t)(p0 + b) * N + cb[o].x] = acc[o][b];
        }
      }
    }, outputs);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const unsigned l1 = __ballot((lm >> b) & 1u) != 0ull ? 1u << b : 0u;
      const unsigned a1 = rownz && __ballot((any >> b) & 1u) != 0ull ? 1u << b : 0u;
      if (lane == 0 && l1) atomicOr(&livebits, l1);
      if (lane == 0 && a1) atomicOr(&anybits, a1);
    }
    lds_barrier();
    const unsigned live = livebits & ((1u << nvalid) - 1u);
    const unsigned nonzero = anybits;
    const bool write = nsplit == 1 && live != 0u;
    const int H = S == 1 ? N : (N + 1) / 2;  // columns that go through LDS at a time
    auto to_tile = [&](int c0, int nc) {
      static_for([&](auto oc) {
        constexpr int o = decltype(oc)::value;
        if (o >= on) return;
        const unsigned c = cb[o].x - (unsigned)c0;  // (kNoColumn stays past every width)
        if (c < (unsigned)nc) tile[c] = make_float4(acc[o][0], acc[o][1], acc[o][2], acc[o][3]);
      }, outputs);
    };
    auto from_tile = [&](int c0, int nc) {
      for (int k = tid; k < nc; k += kSegThreads) {
        const float4 y = tile[k];
        float *dst = yout + (size_t)p0 * N + c0 + k;
        if (live & 1u) dst[0] = y.x;
        if (live & 2u) dst[(size_t)N] = y.y;
        if (live & 4u) dst[(size_t)2 * N] = y.z;
        if (live & 8u) dst[(size_t)3 * N] = y.w;
      }
    };
    if (write && S == 2) {
      to_tile(0, H);
      lds_barrier();
      from_tile(0, H);
      lds_barrier();
    }
    const int c1 = S == 1 ? 0 : H;
    if (write) to_tile(c1, N - c1);
    // the next item's first segment is loaded while this one's last outputs go out
    take_rows(min(item + (int)gridDim.x, items - 1));
    load(0);
    mem_fence_compiler();
    lds_barrier();
    if (write) from_tile(c1, N - c1);
    if (tid == 0) {
      livebits = 0u;
      anybits = 0u;
      if (live) or_mask(masks, spread, p0 >> 5, live << (p0 & 31));
    }
    if (rownz && tid < nvalid && ((nonzero >> tid) & 1u)) rownz[ids[p0 + tid]] = 1;
    lds_barrier();
  }
}

// The groups of k_layer_seg's stream of one layer from its slot-major ELL (byte offsets of stride per
// source). cut[p]: the column at position p has its first (cut & 0xffff) sources in segment 0, of cut >>
// 16. Workgroup k writes column block k, a group of 8 terms per wave at a time: whole groups, padding
// included. Bound: the ELL's reads and the stream's writes, 7.3 MB per layer at 16384 neurons. The host
// wrote the stream before and uploaded it: making and loading 240 layers of 16384 neurons 0.82 -> 0.66 s.
__global__ __launch_bounds__(256) void k_pack_seg(const int2 *__restrict__ ell, int N, int S, int stride,
                                                  const int2 *__restrict__ desc, const uint2 *__restrict__ colb,
                                                  const unsigned *__restrict__ cut, int nblk,
                                                  uint4 *__restrict__ stream) {
  const int k = blockIdx.x, lane = threadIdx.x & 63;
  const unsigned j = colb[k * 64 + lane].x, c = cut[k * 64 + lane];
  const int2 d0 = desc[k], d1 = S == 2 ? desc[nblk + k] : make_int2(0, 0);
  for (int q = threadIdx.x >> 6; q < d0.y + d1.y; q += 4) {
    const bool second = q >= d0.y;
    const int gi = second ? q - d0.y : q;
    const int base = second ? N - kSegCap : 0;
    const int i0 = (second ? (int)(c & 0xffffu) : 0) + gi * 8, i1 = second ? (int)(c >> 16) : (int)(c & 0xffffu);
    unsigned ix[4] = {0u, 0u, 0u, 0u}, w[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const bool have = j != kNoColumn && i0 + t < i1;
      const int2 x = have ? ell[(size_t)(i0 + t) * N + j] : make_int2(base * stride, 0);
      ix[t / 2] |= (unsigned)(x.x / stride - base) << (t % 2 * 16);
      w[t] = (unsigned)x.y;
    }
    uint4 *g = stream + (size_t)((second ? d1.x : d0.x) + gi) * kSegGroupWords + lane;
    g[0] = make_uint4(ix[0], ix[1], ix[2], ix[3]);
    g[64] = make_uint4(w[0], w[1], w[2], w[3]);
    g[128] = make_uint4(w[4], w[5], w[6], w[7]);
  }
}

// Progress word of few-tile layers, stored by workgroup 0 of each launch into coherent host memory:
// run generation (16 bits) | layer of the launch (20 bits) | live count of the previous layer (28
// bits; all ones when this launch did not count it). The host reads it to follow the device
// without copies or events, and to stop enqueuing layers once no row is live.
constexpr int kProgLayerShift = 28, kProgGenShift = 48;
constexpr unsigned long long kProgCountMask = (1ull << kProgLayerShift) - 1;
constexpr int kProgressAhead = 6;  // layers the host may enqueue ahead of the last reported one

// Partial liveness words of a few-tile layer: workgroup g (in XCD order, see few_tile) of a launch of G
// writes the rows of its tile that stayed live in its chunks to part[g], a plain store (zero or not).
// The tile's mask word is the OR of its workgroups' words. Hundreds of workgroups that finish
// together would otherwise serialize on one atomic word (several us per launch).
constexpr int kPartThreads = 256;
constexpr int kPartLoads = 16;  // words per thread: kPartThreads x kPartLoads >= any launch's slots
constexpr int kMaxPartWords = kPartThreads * kPartLoads;

// Tile of workgroup g of G, nt tiles: the workgroups in XCD order (an XCD's follow each other) are divided
// evenly among the tiles, so that every XCD has its share and gathers from at most two tiles. (Whole
// XCDs per tile left two of eight idle with 3 tiles, three with 5 and one with 7: 12 layers of 65536 neurons,
// read-backs apart, 1.12 -> 1.06, 2.10 -> 1.52 and 2.18 -> 1.99 ms; 1, 2, 4 and 8 tiles the same.)
__device__ __forceinline__ int few_tile(int g, int nt, int G) { return g * nt / G; }

// Mask words m[t] = OR of the partial words of tile t (t < nt), from the kPartLoads of the G
// words each thread of a kPartThreads workgroup loaded (word tid + kPartThreads k). Every thread of
// the workgroup calls it; m: nt <= 8 words of LDS, returned after a barrier.
__device__ void or_partials(const unsigned (&pp)[kPartLoads], int G, int nt, unsigned *m) {
  const int tid = threadIdx.x, lane = tid & 63;
  if (tid < 8) m[tid] = 0u;
  __syncthreads();
  for (int t = 0; t < nt; ++t) {
    unsigned v = 0u;
#pragma unroll
    for (int k = 0; k < kPartLoads; ++k) v |= few_tile(tid + kPartThreads * k, nt, G) == t ? pp[k] : 0u;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v |= __shfl_xor(v, d, 64);
    if (lane == 0 && v) atomicOr(&m[t], v);
  }
  __syncthreads();
}

__device__ __forceinline__ void load_partials(unsigned (&pp)[kPartLoads], const unsigned *part, int words) {
#pragma unroll
  for (int k = 0; k < kPartLoads; ++k) {
    const int i = threadIdx.x + kPartThreads * k;
    pp[k] = i < words ? part[i] : 0u;
  }
}

// The mask words of a few-tile layer from its partial words (before a compaction reads them).
__global__ __launch_bounds__(kPartThreads) void k_finalize_masks(const unsigned *__restrict__ part, int G, int nt,
                                                                 unsigned *__restrict__ masks) {
  __shared__ unsigned m[8];
  unsigned pp[kPartLoads];
  load_partials(pp, part, G);
  or_partials(pp, G, nt, m);
  if (threadIdx.x < nt) masks[threadIdx.x] = m[threadIdx.x];
}

// Layers of few rows (at most 8 tiles, so each XCD works on one tile's share of outputs): the tile
// layout and lane mapping of k_layer_gfm with one output per lane and a whole chain's loads in
// flight at once: the KC ELL entries straight from memory (the 8 lanes of an output read the same
// entry), then all KC gathers, then the fma chain. A work item is a chunk of 32 outputs.
// Such a layer is short, so its time is mostly the latency of dependent loads. The work split
// follows ntiles_h, the host's bound on the tiles, so a lane issues its ELL loads and gathers before
// it has read the list length, which only masks the liveness bits. live_before is the live count two
// layers back (final when the launch starts); at zero every input is zero and the layer neither
// gathers nor stores. Liveness goes to partial words part_out, one per workgroup. Workgroup 0
// turns the previous layer's partial words part_prev (prev_G of them, prev_nt tiles) into its mask words masks_prev, or, with part_prev null, reads those words; then it writes
// their live count to count_out (if set) and to the progress word (if set), and clears masks_clear.
// WM picks the weight layout (kWEll, kWOne, kWEdge; see k_layer_gfm). With cols set (kWOne only),
// only the ncols columns cols[p] are computed (see k_layer_gfm).
template <int KC, int WM>
__global__ __launch_bounds__(kPartThreads) void k_layer_gfm_small(
    const float *__restrict__ fin, float *__restrict__ fout, int N, const int2 *__restrict__ ell,
    const unsigned short *__restrict__ src16, const float *__restrict__ w32, float wc,
    const float *__restrict__ bias, float ymax,
    const int *__restrict__ npos, int ntiles_h, unsigned *__restrict__ part_out,
    const unsigned *__restrict__ part_prev, int prev_G, int prev_nt, unsigned *__restrict__ masks_prev,
    unsigned *__restrict__ masks_clear, int *__restrict__ count_out, const int *__restrict__ live_before,
    unsigned long long *__restrict__ progress, unsigned long long progress_tag, const int *__restrict__ cols,
    int ncols) {
  constexpr int FMR = 32, CH = 32;
  __shared__ unsigned wmask[4];
  __shared__ unsigned pmask[8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int G = gridDim.x;
  const int wg = (blockIdx.x & 7) * (G >> 3) + (blockIdx.x >> 3);  // in XCD order
  const int nchunks = (ncols + CH - 1) / CH;
  const int t = few_tile(wg, ntiles_h, G);
  // the tile's workgroups: first, first + 1, ..., taking its chunks in turn
  const int first = (t * G + ntiles_h - 1) / ntiles_h;
  const int step = ((t + 1) * G + ntiles_h - 1) / ntiles_h - first;
  const int q = lane & 7, h = lane >> 3;
  const char *tbase = reinterpret_cast<const char *>(fin + (size_t)t * N * FMR) + q * 16;
  float *obase = fout + (size_t)t * N * FMR + q * 4;
  const bool wg0 = blockIdx.x == 0;
  // no row was live two layers back: every input is zero, so the layer gathers nothing and stores
  // nothing, and its rows stay dead. The count is read through a per-lane (zero) offset, which keeps
  // it a vector value: used as a scalar it would be waited for before the ELL loads are issued.
  int zero;
  asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
  const int count_before = __hip_atomic_load(live_before + zero, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // workgroup 0: the previous layer's partial words, in flight during its chunk
  unsigned pp[kPartLoads];
  if (wg0 && part_prev) load_partials(pp, part_prev, prev_G);
  int R = 0;           // list length
  unsigned pm = 0u;    // lane i < ntiles_h of workgroup 0: the previous layer's mask word of tile i
  unsigned lm = 0u;
  // FIRST: the workgroup's first chunk, which also issues the loads of the list length and the
  // previous masks
  auto run_chunk = [&](int chunk, auto first) {
    constexpr bool FIRST = decltype(first)::value;
    const int j = chunk * CH + wave * 8 + h;
    const int jj = min(j, ncols - 1);
    const int col = cols ? cols[jj] : jj;  // output column
    // byte offsets of the sources' segments and the weights (16-bit source lists with one weight wc
    // or each edge's weight beside them, or ELL entries)
    unsigned eo[KC];
    float ew[KC];
#pragma unroll
    for (int i = 0; i < KC; ++i) {
      if constexpr (WM != kWEll) {
        eo[i] = (unsigned)src16[(size_t)i * ncols + jj] * (FMR * 4);
        ew[i] = WM == kWEdge ? w32[(size_t)i * ncols + jj] : wc;
      } else {
        const int2 e = ell[(size_t)i * N + jj];
        eo[i] = (unsigned)e.x;
        ew[i] = __int_as_float(e.y);
      }
    }
    const float b = bias[col];
    // taken here, after the ELL loads (the asm keeps the compare from being hoisted above them)
    int cb = count_before;
    asm volatile("" : "+v"(cb));
    const bool dead = cb == 0;
#pragma unroll
    for (int i = 0; i < KC; ++i) eo[i] = dead ? 0u : eo[i];
    float4 g[KC];
#pragma unroll
    for (int i = 0; i < KC; ++i) g[i] = *reinterpret_cast<const float4 *>(tbase + eo[i]);
    if constexpr (FIRST) {
      // after the gathers: vector loads complete in order, so waiting for these waits for nothing
      // the fma chain does not need anyway
      R = __hip_atomic_load(npos, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (wg0 && !part_prev && count_out)
        pm = __hip_atomic_load(masks_prev + min(lane, ntiles_h - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // every gather is issued before the first fma waits on one
    mem_fence_compiler();
    __builtin_amdgcn_sched_barrier(0);
    float a[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < KC; ++i) {
      const float w = ew[i];
      a[0] = fmaf(g[i].x, w, a[0]);
      a[1] = fmaf(g[i].y, w, a[1]);
      a[2] = fmaf(g[i].z, w, a[2]);
      a[3] = fmaf(g[i].w, w, a[3]);
    }
    // the chain is computed for every lane (outputs past N repeat output N - 1), so the loads stay
    // ahead of the branch that stores
    const float4 y = make_float4(activate(a[0], b, ymax), activate(a[1], b, ymax), activate(a[2], b, ymax),
                                 activate(a[3], b, ymax));
    const unsigned bits = (y.x > 0.0f ? 1u : 0u) | (y.y > 0.0f ? 2u : 0u) | (y.z > 0.0f ? 4u : 0u) | (y.w > 0.0f ? 8u : 0u);
    lm |= (j < ncols ? bits : 0u) << (4 * q);
    // positions past the list length (up to the host's tile bound) are stored too: nothing reads them
    if (j < ncols && !dead) store_stream(reinterpret_cast<float4 *>(obase + (size_t)col * FMR), y);
  };
  int chunk = wg - first;
  if (chunk < nchunks) {
    run_chunk(chunk, std::true_type{});
    for (chunk += step; chunk < nchunks; chunk += step) run_chunk(chunk, std::false_type{});
  }
  if (wg0) {
    // (workgroup 0 always runs chunk 0, so R is loaded)
    const int ntiles = min(8, (R + FMR - 1) / FMR);
    if (part_prev) {
      or_partials(pp, prev_G, prev_nt, pmask);
      if (tid < prev_nt) masks_prev[tid] = pmask[tid];
      pm = lane < prev_nt ? pmask[lane] : 0u;
    }
    if (wave == 0) {
      int c = __popc(lane < ntiles ? pm : 0u);
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d, 64);
      if (lane == 0 && count_out) *count_out = c;
      if (lane == 0 && progress)
        __hip_atomic_store(progress, progress_tag | (count_out ? (unsigned long long)c : kProgCountMask),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      if (masks_clear && lane < ntiles) masks_clear[lane] = 0u;
    }
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) lm |= __shfl_xor(lm, d, 64);
  if (lane == 0) wmask[wave] = lm;
  __syncthreads();
  if (tid == 0) {
    const int nvalid = min(FMR, R - t * FMR);
    const unsigned valid = nvalid >= 32 ? 0xffffffffu : (nvalid > 0 ? (1u << nvalid) - 1u : 0u);
    part_out[wg] = count_before == 0 ? 0u : (wmask[0] | wmask[1] | wmask[2] | wmask[3]) & valid;
  }
}

constexpr int kBitsThreads = 1024;  // k_layer_bits workgroup: 16 waves, up to 128 registers each
// k_layer_bits' table that turns 4 input bits into 4 floats: 16 entries of 16 bytes (a 256-entry
// table of 8 bits measured twice as slow: its reads spread over more banks)
constexpr int kLutF4 = 16;
// k_layer_bits' LDS tile: one bit word per neuron, sized for the widest network of its height
// (T = 32 for up to 16384 neurons, 16 for up to 65536); static, so that its address is a constant
// that folds into the LDS instructions' offsets. Beside it: the table, the mask word and the
// dictionary cache (under 9 KiB).
__host__ __device__ constexpr int bits_tile_bytes(int T) { return T == 32 ? 16384 * 4 : 65536 * 2; }
static_assert(bits_tile_bytes(16) + 9 * 1024 <= 160 * 1024, "LDS of k_layer_bits");

// Value dictionary for one-byte activation codes, in device memory (kDictWords words):
//   val[256]   the value (fp32 bit pattern) of each code: decoding is val[code];
//   key[1024]  an open-addressing hash table of the values seen, by dict_hash (four slots per code,
//              so that probes stay short also when the 256 codes run out);
//   code[1024] the code of the value in each hash slot (kNoCode until it is published);
//   next       the next free code.
// Codes are handed out in order 0, 1, 2, ... (code 0 is +0.0, whose key sits in its hash slot 0
// from the start), so a layer's first 32 values decode from distinct LDS banks. A value's slot is
// claimed with compare-and-swap; the lane that claims it takes the next code and publishes it
// (relaxed device-scope atomics: a reader needs the code word itself, and the values are read by
// later kernels only); slots and codes never change afterwards, so a workgroup may cache them in
// LDS. kDictEmpty (a
// NaN pattern, never an activation) marks free slots.
// a value whose slot was claimed by another lane waits this many reads at most for its code (the
// claimer publishes it a few instructions after its compare-and-swap); past the bound the
// dictionary counts as full, which sends the layer to its fp32 outputs
constexpr int kDictWaitReads = 1 << 16;
// Code tiles hold CR list positions (code_rows below): [tile][N][CR] bytes, list position p at tile
// p / CR, byte p % CR.
// The code-tile height goes with the bit tiles that write them: 128 rows after 32-row bit tiles,
// whose counting workgroups then fill each 128-byte segment in 4 parts; 64 rows after 16-row bit
// tiles (4 parts each as well). Taller segments serve more rows per gather request.
__host__ __device__ constexpr int code_rows(int T) { return T == 32 ? 128 : 64; }
// rows per lane of k_layer_gfm_u8 (8: 8-byte gathers, for 64-row codes; 4 for 128-row codes, whose
// lanes would otherwise hold too many accumulators)
#ifndef SDNN_U8_RPL
#define SDNN_U8_RPL 8
#endif
__host__ __device__ constexpr int u8_rows_per_lane(int CR) { return CR == 64 ? SDNN_U8_RPL : 4; }
// outputs per lane of k_layer_gfm_u8 (at most 32 / rows per lane accumulators' worth)
#ifndef SDNN_U8_OPL
#define SDNN_U8_OPL (32 / SDNN_U8_RPL)
#endif
__host__ __device__ constexpr int u8_outs_per_lane(int CR) { return CR == 64 ? SDNN_U8_OPL : 8; }
// outputs per work item: 4 waves x outputs per wave instruction (64 / lanes per code segment) x
// outputs per lane
__host__ __device__ constexpr int u8_outputs(int CR) {
  return 4 * (64 / (CR / u8_rows_per_lane(CR))) * u8_outs_per_lane(CR);
}
// k_layer_gfm_u8's software pipeline: slots whose gathers are in flight (SDNN_U8_DEPTH - 1 ahead),
// code dwords whose dictionary reads run ahead of the fmas (SDNN_U8_LA), waves per SIMD the
// registers are held to at 64-row codes (SDNN_U8_WAVES)
#ifndef SDNN_U8_DEPTH
#define SDNN_U8_DEPTH 2
#endif
#ifndef SDNN_U8_LA
#define SDNN_U8_LA 2
#endif
#ifndef SDNN_U8_WAVES
#define SDNN_U8_WAVES 5
#endif
// One XCD's L2. Two-byte codes are tried only for layers whose fp32 input tile (32 rows of every
// source) is larger: at 65536 sources they gather faster than the fp32 tiles, which live in the
// Infinity Cache, while at 16384 the fp32 tiles stay in L2 and the codes (whose 4096-entry
// dictionary also halves the workgroups per CU) measure slower, encoding included.
constexpr size_t kXcdL2Bytes = (size_t)4 << 20;

template <int CB = 1>
__device__ __forceinline__ unsigned dict_hash(unsigned key) {
  // (low 24 bits of key ^ (key >> 16)) * 0x9E3779, bits kHashShift.. (full-rate 24-bit multiply);
  // key 0 hashes to slot 0
  unsigned h;
  asm("v_mul_u32_u24 %0, 0x9e3779, %1" : "=v"(h) : "v"(key ^ (key >> 16)));
  return (h >> DictShape<CB>::kHashShift) & (unsigned)(DictShape<CB>::kHash - 1);
}

// A workgroup's LDS cache of the dictionary: kCacheEntries (key, code) entries in two-way sets
// (entries 2i and 2i + 1), set chosen by a multiplicative hash (a 24-bit multiply, full rate) that
// spreads the values of a layer well (checked on the workloads' value sets). An entry is claimed
// once, by compare-and-swap of its key from kDictEmpty to kCacheBusy; the claimer writes the code,
// then the key (one wave's LDS operations take effect in order; a compiler barrier keeps the order);
// entries are never replaced. A reader loads the keys before the codes, so a key it sees has its
// code in place; kCacheBusy (a NaN pattern) never matches a value.
constexpr int kCacheEntries = DictShape<1>::kCache;
constexpr unsigned kCacheBusy = 0x7fc00001u;
template <int CB = 1>
__device__ __forceinline__ unsigned cache_set(unsigned key) {  // first entry of the key's set (even)
  // the low 32 bits of (low 24 bits of key ^ (key >> 16)) times 0x9E3779, by the full-rate 24-bit
  // multiply (the compiler would pick the quarter-rate 32-bit one)
  unsigned h;
  asm("v_mul_u32_u24 %0, 0x9e3779, %1" : "=v"(h) : "v"(key ^ (key >> 16)));
  return (h >> DictShape<CB>::kCacheShift) & (unsigned)(DictShape<CB>::kCache - 2);
}

// Code of the value with bits `key` from the global table, claiming a free slot and a code on the
// way, then recorded in the LDS cache (dlk, dlc) if its set has a free entry. A full dictionary
// sets *overflow and returns 0; the caller's output is then not used. Once *overflow is set (by any
// lane) every call returns at its next probe.
template <int CB = 1>
__device__ __forceinline__ unsigned dict_code_slow(unsigned key, unsigned *dlk, unsigned *dlc, unsigned *gd,
                                                   int *overflow) {
  constexpr int SLOTS = DictShape<CB>::kSlots, HASH = DictShape<CB>::kHash;
  unsigned *gkey = gd + dict_key_off<CB>(), *gcode = gd + dict_code_off<CB>();
  unsigned h = dict_hash<CB>(key);
  for (int i = 0; i < HASH; ++i) {
    if (__hip_atomic_load(overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return 0;
    unsigned cur = __hip_atomic_load(&gkey[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bool won = false;
    if (cur == kDictEmpty) {
      const unsigned prev = atomicCAS(&gkey[h], kDictEmpty, key);
      won = prev == kDictEmpty;
      cur = won ? key : prev;
    }
    if (won) {
      // this lane claimed the slot: it takes the next code, records the value, publishes the code
      const unsigned c = atomicAdd(gd + dict_next_off<CB>(), 1u);
      if (c < (unsigned)SLOTS) gd[c] = key;
      __hip_atomic_store(&gcode[h], c < (unsigned)SLOTS ? c : kNoCode - 1u, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
    if (cur == key) {
      unsigned c = kNoCode;
      for (int it = 0; it < kDictWaitReads && c == kNoCode; ++it)
        c = __hip_atomic_load(&gcode[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (c >= (unsigned)SLOTS) break;  // no code left, or none published within the bound
      const unsigned st = cache_set<CB>(key);
      if (dlk[st] != key && dlk[st + 1] != key) {
#pragma unroll
        for (unsigned wy = 0; wy < 2; ++wy) {
          if (atomicCAS(&dlk[st + wy], kDictEmpty, kCacheBusy) == kDictEmpty) {
            dlc[st + wy] = c;
            mem_fence_compiler();
            __hip_atomic_store(&dlk[st + wy], key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            break;
          }
        }
      }
      return c;
    }
    h = (h + 1) & (HASH - 1);
  }
  // device scope, as it is read (a plain store would stay in this XCD's L2 until the kernel ends), and
  // once: a store per lane that fails took a failed repack from 0.10 to 0.29 ms at 65536 neurons
  if (!__hip_atomic_load(overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    __hip_atomic_store(overflow, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return 0;
}
// The cache's answer for `key`: *code, and whether it was there.
template <int CB = 1>
__device__ __forceinline__ bool cache_lookup(unsigned key, const unsigned *dlk, const unsigned *dlc, unsigned *code) {
  const unsigned st = cache_set<CB>(key);
  const uint2 k = *reinterpret_cast<const uint2 *>(dlk + st);
  mem_fence_compiler();  // the keys are read before the codes
  const uint2 c = *reinterpret_cast<const uint2 *>(dlc + st);
  *code = k.x == key ? c.x : c.y;
  return k.x == key || k.y == key;
}
template <int CB = 1>
__device__ __forceinline__ unsigned dict_code(float y, unsigned *dlk, unsigned *dlc, unsigned *gd, int *overflow) {
  const unsigned key = __float_as_uint(y);
  unsigned c;
  if (cache_lookup<CB>(key, dlk, dlc, &c)) return c;
  return dict_code_slow<CB>(key, dlk, dlc, gd, overflow);
}

// waves per SIMD the registers of k_layer_gfm_u8 are held to (with two-byte codes and staged weights,
// 40 KiB of LDS per workgroup leave room for 3)
constexpr int u8_waves(int WM, int CR, int CB) {
  return CB == 2 && WM == kWEdge ? 3 : CR == 64 && CB == 1 ? SDNN_U8_WAVES : 4;
}

// One round of a layer whose input tiles hold CB-byte codes of the activations, cin[t][k][b]
// (source k of list position CR t + b), decoded as dict[code]; the output is fp32 tiles of 32 rows
// as in k_layer_gfm (code tile t covers output tiles ST t .. ST t + ST - 1, ST = CR / 32). Code tiles
// [tile0, tile0 + 8) go one per XCD, as in k_layer_gfm. Two-byte codes (CB = 2, 4096-entry
// dictionary, CR = 64) double the bytes of every gather and leave the rest as it is. A code segment
// is CR codes: RL = CR / RPL lanes read it, RPL codes each (RPL = 4: 4-byte loads; 8: 8-byte loads,
// which halves the gather instructions and their address arithmetic; 16-byte loads for two-byte
// codes), so a wave instruction serves OPI = 64 / RL outputs.
// Lane = (r = lane % RL: rows RPL r .. RPL r + RPL - 1, o = lane / RL); the lane runs the OPL
// consecutive outputs jw + OPL o .. + OPL - 1 of its wave's block of OPI * OPL (4 OPL RPL = 128
// accumulator rows per lane would not fit: OPL RPL = 32), so for every slot its sources come from
// LDS one 16-bit read each and its weights in 16-byte reads. A work item is a chunk of 4 waves'
// outputs. The dictionary and the chunk's lists sit in LDS (kWEdge: 6 bytes per entry, 24 KiB,
// which leaves room for 5 workgroups per CU; 40 KiB with the two-byte codes' dictionary). A 32-row
// output segment that is zero in every row is not stored; its bit in seglive (one bit per fp32
// tile and source) says so. Registers are held to 5 waves per SIMD for one-byte 64-row codes (more
// waves keep more gathers in flight; 6 spill), 4 for 128-row codes and 3 for two-byte codes with
// staged weights (u8_waves). Live rows go to masks, or with spread set to the spread words of each
// fp32 tile (see or_mask). With cols set (kWOne only), the launch computes the ncols columns
// cols[p] alone (see k_layer_gfm), stores every segment of them and leaves seglive untouched.
template <int WM, int CR, int RPL, int OPL, int CB = 1>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(u8_waves(WM, CR, CB)))) void k_layer_gfm_u8(
    const unsigned char *__restrict__ cin, float *__restrict__ fout, int N, const int2 *__restrict__ ell, int K,
    const unsigned short *__restrict__ src16, const float *__restrict__ w32, float wc, const float *__restrict__ bias,
    float ymax, const float *__restrict__ dict, const int *__restrict__ npos, unsigned *__restrict__ masks,
    unsigned *__restrict__ seglive, int tile0, unsigned *__restrict__ spread, const int *__restrict__ cols, int ncols,
    int tpx) {
  static_assert(RPL == 4 || RPL == 8, "4 or 8 rows per lane");
  static_assert(OPL == 2 || OPL % 4 == 0, "weights are read in pairs or quads");
  static_assert(OPL * RPL <= 32, "accumulators per lane");
  constexpr int RL = CR / RPL, OPI = 64 / RL, CH = 4 * OPI * OPL, ST = CR / 32;
  constexpr int DW = RPL * CB / 4;  // code dwords per gather
  constexpr int CPD = 4 / CB;       // codes per dword
  constexpr unsigned CMASK = (unsigned)DictShape<CB>::kSlots - 1u;  // (codes below kSlots)
  constexpr int LPS = 32 / RPL;     // lanes per 32-row output segment
  static_assert(CB == 1 || CB == 2, "one- or two-byte codes");
  constexpr bool LISTS = WM != kWEll;
  static_assert(CR == 64 || CR == 128, "code segments of 64 or 128 rows");
  static_assert(CH % 32 == 0 && CH == u8_outputs(CR), "a chunk covers whole bitmap words");
  static_assert(32 % (OPI * OPL) == 0 || (OPI * OPL) % 32 == 0, "bitmap words");
  static_assert(OPI * OPL <= 32, "a wave's outputs lie within one bitmap word");
  __shared__ float dl[DictShape<CB>::kSlots];
  __shared__ __align__(16) unsigned short srcs[LISTS ? 32 * CH : 8];
  __shared__ __align__(16) float wts[WM == kWEdge ? 32 * CH : 4];
  __shared__ float bstage[CH];
  __shared__ int cstage[CH];  // output column of each chunk position
  __shared__ unsigned segw[ST][CH / 32];
  __shared__ unsigned long long rowmask[CR / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i = tid; i < DictShape<CB>::kSlots; i += blockDim.x) dl[i] = dict[i];
  if (tid < CR / 64) rowmask[tid] = 0ull;
  const int R = *npos;
  const int nchunks = (ncols + CH - 1) / CH;
  const RoundSplit rs = round_split((R + CR - 1) / CR - tile0, tpx, nchunks);
  const bool active = rs.active;
  const int t = tile0 + rs.t;
  const int cend = rs.cend;
  const int r = lane % RL, o = lane / RL;
  const int nvalid = active ? min(CR, R - t * CR) : 0;
  // output rows RPL r .. of the code tile: fp32 tile ST t + RPL r / 32, slots (RPL r) % 32; the
  // list's fp32 tiles end at (R + 31) / 32, so the last code tile may lack some of its fp32 tiles
  const int otile = ST * t + (RPL * r) / 32;
  float *obase = fout + ((size_t)otile * N) * 32 + (RPL * r) % 32;
  const bool has_tile = otile * 32 < R;
  const int NW = (N + 31) / 32;
  // the tile base is uniform, so a gather is one 32-bit offset from it
  const unsigned char *tbs = cin + (size_t)t * N * CR * CB;
  const unsigned lofs = (unsigned)(RPL * r * CB);  // byte offset of the lane's rows in a segment
  // live rows seen by this lane: bit (RPL r + c) % 64 of word (RPL r) / 64
  unsigned long long lm[CR / 64];
#pragma unroll
  for (int h = 0; h < CR / 64; ++h) lm[h] = 0ull;
  const int jw = wave * OPI * OPL;  // first output of this wave in the chunk
  const int jl0 = jw + o * OPL;     // this lane's outputs: jl0 .. jl0 + OPL - 1
  for (int chunk = rs.first; chunk < cend; chunk += rs.step) {
    const int c0 = chunk * CH;
    const int nout = min(CH, ncols - c0);
    __syncthreads();  // the previous chunk is done with srcs / wts / bstage / cstage / segw
    for (int i = tid; i < CH; i += blockDim.x) {
      const int col = i < nout ? (cols ? cols[c0 + i] : c0 + i) : 0;
      cstage[i] = col;
      bstage[i] = i < nout ? bias[col] : 0.0f;
    }
    if (tid < ST * (CH / 32)) segw[tid / (CH / 32)][tid % (CH / 32)] = 0u;
    if constexpr (LISTS) stage_lists<WM, CH>(srcs, wts, src16, w32, ncols, c0, nout);
    __syncthreads();
    float acc[OPL][RPL];
#pragma unroll
    for (int i = 0; i < OPL; ++i)
#pragma unroll
      for (int c = 0; c < RPL; ++c) acc[i][c] = 0.0f;
    if constexpr (LISTS) {
      // software pipeline: a slot's gathers are issued one slot before its fmas (deeper pipelines
      // measure no faster: the gathers are limited by the vector-memory path, not by latency)
      constexpr int kDepth = SDNN_U8_DEPTH;
      unsigned wd[kDepth][OPL][DW];
      auto fetch = [&](int sl, int bf) {
        const unsigned short *sp = srcs + sl * CH + jl0;
#pragma unroll
        for (int i = 0; i < OPL; ++i) {
          const unsigned char *gp = tbs + ((unsigned)sp[i] * (unsigned)(CR * CB) + lofs);
          if constexpr (DW == 4) {
            const uint4 v = *reinterpret_cast<const uint4 *>(gp);
            wd[bf][i][0] = v.x;
            wd[bf][i][1] = v.y;
            wd[bf][i][2] = v.z;
            wd[bf][i][3] = v.w;
          } else if constexpr (DW == 2) {
            const uint2 v = *reinterpret_cast<const uint2 *>(gp);
            wd[bf][i][0] = v.x;
            wd[bf][i][1] = v.y;
          } else {
            wd[bf][i][0] = *reinterpret_cast<const unsigned *>(gp);
          }
        }
      };
#pragma unroll
      for (int sl = 0; sl < kDepth - 1; ++sl) fetch(sl, sl);
#pragma unroll
      for (int sl = 0; sl < 32; ++sl) {
        if (sl + kDepth - 1 < 32) fetch(sl + kDepth - 1, (sl + kDepth - 1) % kDepth);
        mem_fence_compiler();
        __builtin_amdgcn_sched_barrier(0);
        // the slot's weights from LDS (16-byte reads, ahead of the dictionary reads below)
        float wv[OPL];
        if constexpr (WM == kWEdge && OPL == 2) {
          const float2 a = *reinterpret_cast<const float2 *>(wts + sl * CH + jl0);
          wv[0] = a.x; wv[1] = a.y;
        } else if constexpr (WM == kWEdge) {
#pragma unroll
          for (int i = 0; i < OPL; i += 4) {
            const float4 a = *reinterpret_cast<const float4 *>(wts + sl * CH + jl0 + i);
            wv[i] = a.x; wv[i + 1] = a.y; wv[i + 2] = a.z; wv[i + 3] = a.w;
          }
        } else {
#pragma unroll
          for (int i = 0; i < OPL; ++i) wv[i] = wc;
        }
        // dictionary lookups run LA code dwords ahead of the fmas that use them
        constexpr int NQ = OPL * DW;  // code dwords of the slot
        constexpr int LA = SDNN_U8_LA;
        float dv[LA + 1][CPD];
        auto lookup = [&](int q) {
#pragma unroll
          for (int c = 0; c < CPD; ++c)
            dv[q % (LA + 1)][c] = dl[(wd[sl % kDepth][q / DW][q % DW] >> (8 * CB * c)) & CMASK];
        };
#pragma unroll
        for (int q = 0; q < LA; ++q) lookup(q);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          if (q + LA < NQ) lookup(q + LA);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int c = 0; c < CPD; ++c)
            acc[q / DW][CPD * (q % DW) + c] = fmaf(dv[q % (LA + 1)][c], wv[q / DW], acc[q / DW][CPD * (q % DW) + c]);
          __builtin_amdgcn_sched_barrier(0);
        }
        // this slot's fmas complete here, before the slot after next is fetched
#pragma unroll
        for (int i = 0; i < OPL; ++i)
#pragma unroll
          for (int c = 0; c < RPL; c += 4) pin4(acc[i][c], acc[i][c + 1], acc[i][c + 2], acc[i][c + 3]);
      }
    } else {
      const unsigned char *tb = tbs + lofs;
      for (int sl = 0; sl < K; ++sl) {
#pragma unroll
        for (int i = 0; i < OPL; ++i) {
          const int2 e = ell[(size_t)sl * N + min(c0 + jl0 + i, N - 1)];
#pragma unroll
          for (int d = 0; d < DW; ++d) {
            const unsigned word = *reinterpret_cast<const unsigned *>(tb + ((unsigned)e.x >> 7) * (CR * CB) + 4 * d);
#pragma unroll
            for (int c = 0; c < CPD; ++c)
              acc[i][CPD * d + c] = fmaf(dl[(word >> (8 * CB * c)) & CMASK], __int_as_float(e.y), acc[i][CPD * d + c]);
          }
        }
      }
    }
    // segment bits of this wave's outputs (jw .. jw + OPI OPL - 1, within one bitmap word), per fp32 tile
    unsigned seg[ST];
#pragma unroll
    for (int q = 0; q < ST; ++q) seg[q] = 0u;
#pragma unroll
    for (int i = 0; i < OPL; ++i) {
      const int jl = jl0 + i;
      const float b = bstage[jl];
      float y[RPL];
      unsigned bits = 0u;
#pragma unroll
      for (int c = 0; c < RPL; ++c) {
        y[c] = activate(acc[i][c], b, ymax);
        bits |= (jl < nout && y[c] > 0.0f ? 1u : 0u) << c;
      }
      const unsigned long long bal = __ballot(bits != 0u);
      // the LPS lanes of this lane's output segment: lanes (lane & ~(LPS - 1)) .. + LPS - 1
      constexpr unsigned long long kSegLanes = (1ull << LPS) - 1ull;
      if (jl < nout && has_tile && (cols || ((bal >> (lane & ~(LPS - 1))) & kSegLanes) != 0ull)) {
#pragma unroll
        for (int c = 0; c < RPL; c += 4)
          store_stream(reinterpret_cast<float4 *>(obase + (size_t)cstage[jl] * 32 + c),
                       make_float4(y[c], y[c + 1], y[c + 2], y[c + 3]));
      }
#pragma unroll
      for (int h = 0; h < CR / 64; ++h)
        if ((RPL * r) / 64 == h) lm[h] |= (unsigned long long)bits << ((RPL * r) % 64);
      // output jw + OPL oo + i of fp32 tile q is stored by lanes oo RL + LPS q .. + LPS - 1
#pragma unroll
      for (int oo = 0; oo < OPI; ++oo)
#pragma unroll
        for (int q = 0; q < ST; ++q)
          seg[q] |= (((bal >> (oo * RL + LPS * q)) & kSegLanes) != 0ull ? 1u : 0u) << ((jw % 32) + oo * OPL + i);
    }
    if (lane == 0)
#pragma unroll
      for (int q = 0; q < ST; ++q)
        if (seg[q]) atomicOr(&segw[q][jw / 32], seg[q]);
    __syncthreads();
    if (tid < ST * (CH / 32) && !cols) {
      const int q = tid / (CH / 32), wi = tid % (CH / 32);
      if ((ST * t + q) * 32 < R && c0 + 32 * wi < N) seglive[(size_t)(ST * t + q) * NW + c0 / 32 + wi] = segw[q][wi];
    }
  }
  // rows of this code tile that stayed live in any of this workgroup's chunks
#pragma unroll
  for (int h = 0; h < CR / 64; ++h)
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) lm[h] |= __shfl_xor(lm[h], d, 64);
  __syncthreads();
  if (lane == 0)
#pragma unroll
    for (int h = 0; h < CR / 64; ++h)
      if (lm[h]) atomicOr(&rowmask[h], lm[h]);
  __syncthreads();
  if (tid == 0 && active) {
#pragma unroll
    for (int q = 0; q < ST; ++q) {
      const int lo = 32 * q;  // rows lo .. lo + 31 of the code tile
      const unsigned valid = nvalid - lo >= 32 ? 0xffffffffu : (nvalid > lo ? ((1u << (nvalid - lo)) - 1u) : 0u);
      const unsigned m = (unsigned)(rowmask[q / 2] >> (32 * (q & 1))) & valid;
      if (m) or_mask(masks, spread, ST * t + q, m);
    }
  }
}

// Repack of one-byte code tiles (CR positions each) after a compaction: position p of the
// new tiles takes the code at position src[p] of the old ones; positions past *npos get code 0
// (+0.0). A thread writes 4 codes of one source.
template <int CR>
__global__ __launch_bounds__(256) void k_repack_u8(const unsigned char *__restrict__ sfm, unsigned char *__restrict__ dfm,
                                                   int N, const int *__restrict__ src, const int *__restrict__ npos) {
  constexpr int QPS = CR / 4;  // 4-byte quads per source segment
  const int R = *npos;
  const int ntiles = (R + CR - 1) / CR;
  const size_t items = (size_t)ntiles * N * QPS;
  for (size_t it = blockIdx.x * (size_t)blockDim.x + threadIdx.x; it < items; it += (size_t)gridDim.x * blockDim.x) {
    const int qd = (int)(it % QPS);
    const size_t rest = it / QPS;
    const int k = (int)(rest % N);
    const int t = (int)(rest / N);
    unsigned word = 0u;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int p = t * CR + qd * 4 + c;
      if (p < R) {
        const int sp = src[p];
        word |= (unsigned)sfm[((size_t)(sp / CR) * N + k) * CR + sp % CR] << (8 * c);
      }
    }
    *reinterpret_cast<unsigned *>(dfm + ((size_t)t * N + k) * CR + qd * 4) = word;
  }
}

template <int T>
struct BitWord;
template <>
struct BitWord<16> {
  using type = unsigned short;
};
template <>
struct BitWord<32> {
  using type = unsigned int;
};

// The value dictionary back to its initial state (code 0 = +0.0, every other slot free, next code
// 1) and its overflow flag cleared, before a later layer's outputs are encoded into it.
template <int CB>
__global__ void k_dict_reset(unsigned *__restrict__ dict, int *__restrict__ overflow) {
  dict_init<CB>(dict, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
  if (blockIdx.x == 0 && threadIdx.x == 0) *overflow = 0;
}

// Encode the fp32 tiles of a layer's input (32 list positions each) as CB-byte dictionary codes in
// tiles of CR positions, cout[t][k][b] = code of the value at list position CR t + b of source k,
// so that the layer can gather them with k_layer_gfm_u8 (exact: a code decodes to the stored bits).
// A thread encodes 16 positions of one source (16 CB bytes, one or two 16-byte stores). Positions
// at or past *npos get code 0 and are not read. Codes come from gd (the dictionary of CB-byte
// codes) through a per-workgroup LDS cache, as in k_layer_bits; more distinct values than the
// dictionary holds set *overflow, and every thread stops at its next item (the caller then keeps
// the fp32 tiles).
template <int CR, int CB>
__global__ __launch_bounds__(256) void k_encode(const float *__restrict__ fin, unsigned char *__restrict__ cout, int N,
                                                const int *__restrict__ npos, unsigned *__restrict__ gd,
                                                int *__restrict__ overflow) {
  constexpr int CE = DictShape<CB>::kCache;
  __shared__ __align__(8) unsigned dlk[CE];
  __shared__ __align__(8) unsigned dlc[CE];
  for (int i = threadIdx.x; i < CE; i += blockDim.x) dlk[i] = kDictEmpty;
  __syncthreads();
  const int R = *npos;
  constexpr int QPS = CR / 16;  // 16-position groups per source segment
  const size_t items = (size_t)((R + CR - 1) / CR) * N * QPS;
  const size_t step = (size_t)gridDim.x * blockDim.x;
  for (size_t it = (size_t)blockIdx.x * blockDim.x + threadIdx.x; it < items; it += step) {
    if (__hip_atomic_load(overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    const int q = (int)(it % QPS);
    const size_t rest = it / QPS;
    const int k = (int)(rest % N);
    const size_t t = rest / N;
    const int p0 = (int)t * CR + q * 16;  // first list position of the group
    unsigned code[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) code[u] = 0u;
    if (p0 < R) {
      // the group lies in one 32-position fp32 tile (p0 % 16 == 0)
      const float4 *src = reinterpret_cast<const float4 *>(fin + ((size_t)(p0 >> 5) * N + k) * 32 + (p0 & 31));
      float v[16];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 x = src[g];
        v[4 * g] = x.x; v[4 * g + 1] = x.y; v[4 * g + 2] = x.z; v[4 * g + 3] = x.w;
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = p0 + u < R ? v[u] : 0.0f;
      bool miss = false;
#pragma unroll
      for (int u = 0; u < 16; ++u) miss |= !cache_lookup<CB>(__float_as_uint(v[u]), dlk, dlc, &code[u]);
      if (miss) {
#pragma unroll
        for (int u = 0; u < 16; ++u) code[u] = dict_code<CB>(v[u], dlk, dlc, gd, overflow);
      }
    }
    uint4 *dst = reinterpret_cast<uint4 *>(cout + ((t * N + k) * CR + q * 16) * CB);
    if constexpr (CB == 1) {
      uint4 w;
      w.x = code[0] | (code[1] << 8) | (code[2] << 16) | (code[3] << 24);
      w.y = code[4] | (code[5] << 8) | (code[6] << 16) | (code[7] << 24);
      w.z = code[8] | (code[9] << 8) | (code[10] << 16) | (code[11] << 24);
      w.w = code[12] | (code[13] << 8) | (code[14] << 16) | (code[15] << 24);
      store_stream(dst, w);
    } else {
      store_stream(dst, make_uint4(code[0] | (code[1] << 16), code[2] | (code[3] << 16), code[4] | (code[5] << 16),
                                   code[6] | (code[7] << 16)));
      store_stream(dst + 1, make_uint4(code[8] | (code[9] << 16), code[10] | (code[11] << 16),
                                       code[12] | (code[13] << 16), code[14] | (code[15] << 16)));
    }
  }
}

// Reports the overflow flag to the host through the coherent report word (as k_compact does,
// with a count of 0).
__global__ void k_report_overflow(const int *__restrict__ overflow, unsigned long long *__restrict__ notify,
                                  unsigned long long tag) {
  const unsigned long long flags = *overflow != 0 ? 2ull : 0ull;
  __hip_atomic_store(notify, (tag << 40) | (flags << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// After a compaction of the global-tile path: move the live positions of a layer's output tiles
// into fresh tiles, dst[t][k][b] = the value at list position src[32t + b] of the source tiles
// (tile src / 32, slot src % 32; the position itself with src null), for positions below *npos; zero past it. A work item is one new
// tile and kRepackSources sources. The new tile's rows come from at most 32 old tiles (src is
// ascending); for each of them, 8 lanes read a source's whole 128-byte segment (one 16-byte load
// each), keep the rows the new tile takes, and place them in an LDS stage from which the new
// segments are written whole. So each needed old segment is read once, coalesced. With seglive
// set, an old segment whose bit there is clear was never stored (all its rows are zero) and is not
// read. With cols set (tiles of a layer that computed only the columns cols[0..ncols); seglive is
// then null), only those sources are moved.
// With OUT = kRepackRows the live positions are written as rows instead, dfm[p][k] (no position past
// *npos), for k_layer_seg; cols must be null.
// With OUT = kRepackCodes the new tiles are written as one-byte dictionary codes, in code tiles of CR
// positions as k_encode writes them (dcodes; cols must be null): the repack and the encoding of the
// next layer's inputs in one pass. Every position of the last code tile is written (code 0 past
// *npos). A full dictionary sets *overflow, and the workgroups stop at their next work item (the
// caller then repacks the fp32 tiles).
// Bound: waiting, for the list of old tiles (one wave forms it by a ballot; read slot after slot by one
// thread it was a chain of 32 loads per item) and for the segments. Eight workgroups per CU are launched and
// must be resident at once (64 registers: at 70 to 76 the last ones ran alone, 4-7% of a pass more).
// Batches of 4 old tiles beat 8, which read more segments that no slot needs, and 2. 60,000 rows of 16384
// neurons through 20 structured layers, four such repacks: 16.45 -> 15.05 ms a pass (one repack of 65536
// neurons x 16 layers: within the runs' differences).
constexpr int kRepackSources = 256;
constexpr int kRepackTiles = 0, kRepackCodes = 1, kRepackRows = 2;
template <int OUT = kRepackTiles, int CR = 32>
__global__ __launch_bounds__(256, 8) void k_repack(const float *__restrict__ sfm, float *__restrict__ dfm, int N,
                                                const int *__restrict__ src, const int *__restrict__ npos,
                                                const unsigned *__restrict__ seglive, const int *__restrict__ cols,
                                                int ncols, unsigned char *__restrict__ dcodes, unsigned *__restrict__ gd,
                                                int *__restrict__ overflow) {
  constexpr int kSteps = kRepackSources / 32;
  __shared__ int otile[32];            // distinct old tiles of this new tile
  __shared__ unsigned omask[32];       // their slots that this new tile takes
  __shared__ unsigned char bslot[32][32];  // old tile i, old slot s -> new slot
  __shared__ int nold;
  __shared__ unsigned segw[kSteps][32];    // seglive words of the old tiles, per 32 sources
  __shared__ float stages[2][32][33];
  constexpr bool CODES = OUT == kRepackCodes;
  constexpr int CE = CODES ? kCacheEntries : 2;
  __shared__ __align__(8) unsigned dlk[CE];  // the dictionary's LDS cache (CODES)
  __shared__ __align__(8) unsigned dlc[CE];
  __shared__ int stop;
  if constexpr (CODES) {
    for (int i = threadIdx.x; i < CE; i += blockDim.x) dlk[i] = kDictEmpty;
  }
  const int R = *npos;
  // (codes: every 32-position tile of the last code tile, those past the list all zero)
  const int ntiles = CODES ? (R + CR - 1) / CR * (CR / 32) : (R + 31) / 32;
  const int nkc = (ncols + kRepackSources - 1) / kRepackSources;
  const int tid = threadIdx.x, lane = tid & 63, kk = tid >> 3, q = tid & 7;
  const int NW = (N + 31) / 32;
  for (int item = blockIdx.x; item < ntiles * nkc; item += gridDim.x) {
    const int t = item / nkc, k0 = (item % nkc) * kRepackSources;
    const int nb = max(0, min(32, R - t * 32));
    if constexpr (CODES) {
      if (tid == 0) stop = __hip_atomic_load(overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __syncthreads();
      if (stop) return;  // uniform: every thread read the one word
    }
    if (tid < 64) {
      // lane b < nb: the old position of new slot b, and (positions ascend) the number of old tiles up to it
      const int sp = lane < nb ? (src ? src[t * 32 + lane] : t * 32 + lane) : -1;
      const int before = __shfl_up(sp, 1, 64);
      const bool starts = lane < nb && (lane == 0 || (sp >> 5) != (before >> 5));
      const unsigned long long heads = __ballot(starts);
      const int i = __popcll(heads & (~0ull >> (63 - lane))) - 1;
      if (lane < 32) omask[lane] = 0u;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
      if (lane < nb) {
        if (starts) otile[i] = sp >> 5;
        atomicOr(&omask[i], 1u << (sp & 31));
        bslot[i][sp & 31] = (unsigned char)lane;
      }
      if (lane == 0) nold = __popcll(heads);
    }
    __syncthreads();
    const int n = nold;
    const bool zeros = seglive || nb < 32;  // slots that no segment fills (a row of a stage is one wave's)
    // k0 + kb is a multiple of 32: one bitmap word per old tile covers 32 sources
    if (seglive) {
      const int step = tid >> 5, i = tid & 31;
      if (i < n && k0 + 32 * step < N) segw[step][i] = seglive[(size_t)otile[i] * NW + (k0 >> 5) + step];
      __syncthreads();
    }
#pragma unroll 1
    for (int step = 0; step < kSteps; ++step) {
      const int kb = 32 * step;
      float (&stage)[32][33] = stages[step & 1];
      const int kp = k0 + kb + kk;  // source position; the source is cols[kp] with a column list
      const int k = kp < ncols ? (cols ? cols[kp] : kp) : N;
      if (zeros) {
#pragma unroll
        for (int c = 0; c < 4; ++c) stage[kk][4 * q + c] = 0.0f;
      }
      if (k < N) {
        // old tiles in batches of 4: the batch's loads are all issued before the first is used
        for (int i0 = 0; i0 < n; i0 += 4) {
          float4 v[4];
          unsigned mm[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int i = min(i0 + u, n - 1);
            mm[u] = i0 + u < n && (!seglive || ((segw[step][i] >> kk) & 1u)) ? (omask[i] >> (4 * q)) & 15u : 0u;
            // without a branch: a quad that is not needed reads the first one of the old tiles
            // instead (a cache hit), so the loads issue back to back
            const size_t at = mm[u] ? ((size_t)otile[i] * N + k) * 32 : 0;
            v[u] = *(reinterpret_cast<const float4 *>(sfm + at) + q);
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (!mm[u]) continue;
            const float e[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (int c = 0; c < 4; ++c)
              if ((mm[u] >> c) & 1u) stage[kk][bslot[i0 + u][4 * q + c]] = e[c];
          }
        }
      }
      __syncthreads();
      if constexpr (CODES) {
        if (k < N) {
          // codes of rows 4q .. 4q + 3 of this 32-position tile, at its place in its code tile
          unsigned c[4];
          bool miss = false;
#pragma unroll
          for (int u = 0; u < 4; ++u) miss |= !cache_lookup(__float_as_uint(stage[kk][4 * q + u]), dlk, dlc, &c[u]);
          if (miss) {
#pragma unroll
            for (int u = 0; u < 4; ++u) c[u] = dict_code(stage[kk][4 * q + u], dlk, dlc, gd, overflow);
          }
          unsigned char *d = dcodes + ((size_t)(t / (CR / 32)) * N + k) * CR + (t % (CR / 32)) * 32 + 4 * q;
          *reinterpret_cast<unsigned *>(d) = c[0] | (c[1] << 8) | (c[2] << 16) | (c[3] << 24);
        }
      } else if constexpr (OUT == kRepackRows) {
        // row kk of the tile, sources 4q .. 4q + 3 of the 32
        const int ks = k0 + kb + 4 * q;
        if (kk < nb) {
          float *d = dfm + (size_t)(t * 32 + kk) * N + ks;
          if ((N & 3) == 0 && ks < N) {
            *reinterpret_cast<float4 *>(d) =
                make_float4(stage[4 * q][kk], stage[4 * q + 1][kk], stage[4 * q + 2][kk], stage[4 * q + 3][kk]);
          } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
              if (ks + c < N) d[c] = stage[4 * q + c][kk];
          }
        }
      } else if (k < N) {
        *reinterpret_cast<float4 *>(dfm + ((size_t)t * N + k) * 32 + 4 * q) =
            make_float4(stage[kk][4 * q], stage[kk][4 * q + 1], stage[kk][4 * q + 2], stage[kk][4 * q + 3]);
      }
    }
    __syncthreads();
  }
}

// Layer-0 inputs as bits (the challenge inputs are binary images, Sec. IV): pack the live rows into
// feature-major bit tiles, bits[t][k] bit b = (Y[ids[t*T + b]][k] != 0). Any entry other than 0
// and 1 (or not finite) sets *nonbinary, and the bit route is then not used. Rows with a nonzero
// entry are recorded in rownz. One wave per (tile, run of kPackBlocks blocks of sources): with
// N % 4 == 0 a lane takes 4 consecutive sources per block (16-byte loads, 256 sources per block),
// otherwise one (64 per block). The rows' nonzero bits are gathered over the run and stored once.
constexpr int kPackBlocks = 16;
template <int T>
__global__ __launch_bounds__(256) void k_pack_bits(const float *__restrict__ yin, typename BitWord<T>::type *__restrict__ bits,
                                                   int N, const int *__restrict__ ids, const int *__restrict__ count,
                                                   int *__restrict__ rownz, int *__restrict__ nonbinary) {
  using W = typename BitWord<T>::type;
  const int R = *count;
  const int ntiles = (R + T - 1) / T;
  const bool vec = (N & 3) == 0;
  const int per_lane = vec ? 4 : 1;
  const int kblocks = (N + 64 * per_lane - 1) / (64 * per_lane);
  const int runs = (kblocks + kPackBlocks - 1) / kPackBlocks;
  const int lane = threadIdx.x & 63;
  const long long nwaves = (long long)gridDim.x * (blockDim.x >> 6);
  bool bad = false;
  for (long long item = blockIdx.x * (long long)(blockDim.x >> 6) + (threadIdx.x >> 6);
       item < (long long)ntiles * runs; item += nwaves) {
    const int t = (int)(item / runs), run = (int)(item % runs);
    const int nvalid = min(T, R - t * T);
    // row starts in units of 4 floats (vec) or floats: below 2^32 for any row id and width
    unsigned rowq[T];
#pragma unroll
    for (int b = 0; b < T; ++b) rowq[b] = (unsigned)ids[t * T + min(b, nvalid - 1)] * (unsigned)(vec ? N / 4 : N);
    const float4 *y4 = reinterpret_cast<const float4 *>(yin);
    unsigned rows_nz = 0u;
    const int kb_end = min(kblocks, (run + 1) * kPackBlocks);
    for (int kb = run * kPackBlocks; kb < kb_end; ++kb) {
      if (vec) {
        const int k = (kb * 64 + lane) * 4;
        const bool kin = k < N;
        unsigned word[4] = {0u, 0u, 0u, 0u};
        // rows in groups of 16 keep the loads in flight within the register budget
#pragma unroll
        for (int b0 = 0; b0 < T; b0 += 16) {
          float4 v[16];
#pragma unroll
          for (int b = 0; b < 16; ++b)
            v[b] = (b0 + b < nvalid && kin) ? load_stream_f4(y4 + rowq[b0 + b] + (k >> 2)) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
          for (int b = 0; b < 16; ++b) {
            const float e[4] = {v[b].x, v[b].y, v[b].z, v[b].w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const bool nz = e[c] != 0.0f;
              bad |= nz && e[c] != 1.0f;
              word[c] |= (unsigned)nz << (b0 + b);
            }
          }
        }
        rows_nz |= word[0] | word[1] | word[2] | word[3];
        if (kin) {
          W *dst = bits + (size_t)t * N + k;
          if constexpr (sizeof(W) == 2) {
            *reinterpret_cast<uint2 *>(dst) = make_uint2(word[0] | (word[1] << 16), word[2] | (word[3] << 16));
          } else {
            *reinterpret_cast<uint4 *>(dst) = make_uint4(word[0], word[1], word[2], word[3]);
          }
        }
      } else {
        const int k = kb * 64 + lane;
        const bool kin = k < N;
        float v[T];
#pragma unroll
        for (int b = 0; b < T; ++b) v[b] = (b < nvalid && kin) ? yin[(size_t)rowq[b] + k] : 0.0f;
        unsigned word = 0u;
#pragma unroll
        for (int b = 0; b < T; ++b) {
          const bool nz = v[b] != 0.0f;
          bad |= nz && v[b] != 1.0f;
          word |= (unsigned)nz << b;
        }
        rows_nz |= word;
        if (kin) bits[(size_t)t * N + k] = (W)word;
      }
    }
    // rows with a nonzero anywhere in this run: OR over the wave, then lane b stores row b's flag
    unsigned all = rows_nz;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) all |= __shfl_xor(all, d, 64);
    if (lane < nvalid && ((all >> lane) & 1u)) rownz[ids[t * T + lane]] = 1;
  }
  if (__ballot(bad) && lane == 0) *nonbinary = 1;
}

// (byte k of u) & 0xF0 in one instruction: a bitwise and whose first operand is byte k of u (a
// byte-select on the operand); f0 holds 0xF0.
__device__ __forceinline__ unsigned byte_and_f0(unsigned u, int k, unsigned f0) {
  unsigned r;
  switch (k) {
    case 0: return u & 0xF0u;
    case 1:
      asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 src1_sel:DWORD"
          : "=v"(r) : "v"(u), "v"(f0));
      return r;
    case 2:
      asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_2 src1_sel:DWORD"
          : "=v"(r) : "v"(u), "v"(f0));
      return r;
    default:
      asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:DWORD"
          : "=v"(r) : "v"(u), "v"(f0));
      return r;
  }
}

// Layer 0 from bit tiles of T rows (T = 16 or 32): every term is fma(bit, w, acc) with bit 0 or 1,
// the same fp32 chain as the general kernels since 1*w and 0*w are exact. blockDim kBitsThreads. LDS
// holds the tile's N words and a table that turns 4 input bits into as many floats (16
// entries of 4 floats: few distinct entries, so a wave's reads of it are mostly broadcasts). Lane =
// output j; each lane carries the T rows of its output, so one ELL entry and one word serve T
// edge-rows; for 16-row tiles the table reads of a term are issued one term ahead. Results
// go to feature-major tiles of 32 rows (list position p at tile p / 32, slot p % 32): a lane writes
// its T rows of output j as T / 4 16-byte stores. Slots past the list's end get zeros.
// ell is the layer's ELL with source k given as k * sizeof(word), the byte offset of its word in
// the bit tile (LayerDev::ellw).
// KC = 32: the 32 ELL entries of a lane's output are all loaded before the first term is used.
// CODES: instead of fp32 values, write each output's one-byte code in the value dictionary gd
// (same tile layout, one byte per row); a full dictionary sets *overflow. With *skip set (an input
// that is not 0 or 1) the kernel does nothing.
template <int T, int KC, bool CODES>
__global__ __launch_bounds__(kBitsThreads) void k_layer_bits(const typename BitWord<T>::type *__restrict__ bits,
                                                     float *__restrict__ fout, int N, const int2 *__restrict__ ell,
                                                     int K, const float *__restrict__ bias,
                                                     float ymax, const int *__restrict__ count,
                                                     unsigned *__restrict__ masks, unsigned *__restrict__ gd,
                                                     int *__restrict__ overflow, const int *__restrict__ skip) {
  if (*skip) return;  // an input is not 0 or 1 (found by k_pack_bits): the layer goes another way
  constexpr int CR = code_rows(T);
  using W = typename BitWord<T>::type;
  const unsigned f0 = 0xF0u;                            // the byte-select ands' mask, in a register
  // static LDS (addresses known at compile time, so they fold into the instructions' offsets): the
  // table, the tile's live-row mask and the dictionary cache; dynamic LDS: the tile
  // one struct fixes the layout: the table at LDS address 0 and the tile after the small arrays,
  // so that every LDS address here is a register plus a constant that fits the instruction offset
  struct BitsLds {
    float4 lut[kLutF4];
    unsigned dlk[kCacheEntries];
    unsigned dlc[kCacheEntries];
    unsigned tilemask;
    unsigned pad[3];
    W tile[bits_tile_bytes(T) / sizeof(W)];
  };
  __shared__ __align__(16) BitsLds sm;
  float4 *const lut = sm.lut;
  unsigned *const dlk = sm.dlk;
  unsigned *const dlc = sm.dlc;
  unsigned &tilemask = sm.tilemask;
  W *const tile = sm.tile;
  const int R = *count;
  const int ntiles = (R + T - 1) / T;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
  const int blocks = (N + 63) / 64;                 // output blocks of 64
  const int rounds = (blocks + nw - 1) / nw;        // rounds of one block per wave
  // Every tile's outputs in 8 chunks, item w taking chunk w % 8: with the grid a multiple of 8, that
  // is the XCD the workgroup runs on, so each XCD reads one eighth of the layer's ELL (2.1 MB at
  // 65536 neurons), which stays in its L2 while every tile passes; with whole tiles per workgroup
  // each tile re-read the whole ELL (16.8 MB) through the L2s, tens of GB per layer. A tile is then
  // staged 8 times (its bits are 1/16 of the ELL's bytes at 16 rows).
  const Chunking ch = chunking(ntiles, rounds, gridDim.x % 8 == 0 ? 8 : 1);
  // codes with whole tiles as items: keep the tiles of one code group on one XCD
  const bool grouped = CODES && ch.nchunks == 1 && gridDim.x % (8 * (CR / T)) == 0;
  const int items = grouped ? (ntiles + gridDim.x - 1) / gridDim.x * gridDim.x : ntiles * ch.nchunks;
  for (int i = tid; i < kLutF4; i += blockDim.x)
    lut[i] = make_float4((float)(i & 1), (float)((i >> 1) & 1), (float)((i >> 2) & 1), (float)((i >> 3) & 1));
  if (tid == 0) tilemask = 0u;
  if (CODES)
    for (int i = tid; i < kCacheEntries; i += blockDim.x) dlk[i] = kDictEmpty;
  for (int w = blockIdx.x; w < items; w += gridDim.x) {
    const int t = grouped ? code_group_tile(w, CR / T) : w / ch.nchunks;
    const int c = grouped ? 0 : w % ch.nchunks;
    if (t >= ntiles) continue;  // uniform over the workgroup
    const int p0 = t * T;
    const int nvalid = min(T, R - p0);
    {
      const W *src = bits + (size_t)t * N;
      if ((reinterpret_cast<uintptr_t>(src) & 15) == 0) {
        const int n16 = (int)(((size_t)N * sizeof(W)) / 16);
        for (int i = tid; i < n16; i += blockDim.x) reinterpret_cast<int4 *>(tile)[i] = reinterpret_cast<const int4 *>(src)[i];
        for (int k = n16 * (int)(16 / sizeof(W)) + tid; k < N; k += blockDim.x) tile[k] = src[k];
      } else {
        for (int k = tid; k < N; k += blockDim.x) tile[k] = src[k];
      }
    }
    __syncthreads();
    const char *tb = reinterpret_cast<const char *>(tile);
    unsigned live = 0u;
    const int r_end = min(rounds, (c + 1) * ch.rounds_per_chunk);
    const unsigned ell_row = (unsigned)N * (unsigned)sizeof(int2);  // bytes per ELL slot
    const __amdgpu_buffer_rsrc_t ersrc = buffer_rsrc(ell, (unsigned)K * ell_row);
    for (int r = c * ch.rounds_per_chunk; r < r_end; ++r) {
      const int blk = r * nw + wave;
      if (blk >= blocks) break;
      const int j = blk * 64 + lane;
      const bool jin = j < N;
      // ELL entries by buffer loads: the lane's offset in a vector register, the slot's offset
      // (sl * N * 8) in a scalar one, so that no vector instruction forms an address
      const unsigned jo8 = (jin ? (unsigned)j : 0u) * (unsigned)sizeof(int2);
      auto ej = [&](int sl) {
        return __builtin_bit_cast(int2, __builtin_amdgcn_raw_buffer_load_b64(ersrc, jo8, (unsigned)sl * ell_row, 0));
      };
      float acc[T];
#pragma unroll
      for (int b = 0; b < T; ++b) acc[b] = 0.0f;
      // the source's word gives the T input bits; each nibble picks four floats (0 or 1) from the
      // table
      auto expand = [&](unsigned word, float4 (&v)[T / 4]) {
        // byte offset of nibble 2k's entry: byte k of (word << 4) with its low 4 bits cleared; of
        // nibble 2k + 1's: byte k of word, likewise (one byte-select and per nibble)
        const unsigned x = word << 4;
        const char *lb = reinterpret_cast<const char *>(lut);
#pragma unroll
        for (int k = 0; k < T / 8; ++k) {
          v[2 * k] = *reinterpret_cast<const float4 *>(lb + byte_and_f0(x, k, f0));
          v[2 * k + 1] = *reinterpret_cast<const float4 *>(lb + byte_and_f0(word, k, f0));
        }
      };
      auto apply = [&](const float4 (&v)[T / 4], float wv) {
#pragma unroll
        for (int n = 0; n < T / 4; ++n) {
          acc[4 * n] = fmaf(v[n].x, wv, acc[4 * n]);
          acc[4 * n + 1] = fmaf(v[n].y, wv, acc[4 * n + 1]);
          acc[4 * n + 2] = fmaf(v[n].z, wv, acc[4 * n + 2]);
          acc[4 * n + 3] = fmaf(v[n].w, wv, acc[4 * n + 3]);
        }
      };
      if constexpr (KC > 0) {
        // slots go in groups of 16 with the issue order pinned by scheduling barriers: a group's
        // tile words are read while the next group's ELL entries load, then its terms run
        // slots in groups of G (16 rows: 16 with the table reads one term ahead; 32 rows: 8, reads
        // not ahead, which keeps the lane within 128 registers)
        constexpr int G = T == 16 ? 16 : 8;
        constexpr bool AHEAD = T == 16;
        static_assert(KC % G == 0, "KC must be a multiple of the group");
        int2 e[G];
#pragma unroll
        for (int i = 0; i < G; ++i) e[i] = ej(i);
#pragma unroll
        for (int h = 0; h < KC; h += G) {
          mem_fence_compiler();
          unsigned wd[G];
          float wv[G];
#pragma unroll
          for (int i = 0; i < G; ++i) {
            wd[i] = *reinterpret_cast<const W *>(tb + (unsigned)e[i].x);
            wv[i] = __int_as_float(e[i].y);
          }
          if (h + G < KC) {
#pragma unroll
            for (int i = 0; i < G; ++i) e[i] = ej(h + G + i);
          }
          mem_fence_compiler();
          if constexpr (AHEAD) {
            // table reads run one term ahead of the fmas (two buffers by parity: no copies)
            float4 vb[2][T / 4];
            expand(wd[0], vb[0]);
#pragma unroll
            for (int i = 0; i < G; ++i) {
              if (i + 1 < G) expand(wd[i + 1], vb[(i + 1) & 1]);
              apply(vb[i & 1], wv[i]);
              // this term's fmas complete here, and the next table reads are issued after them
#pragma unroll
              for (int b = 0; b < T; b += 4) pin4(acc[b], acc[b + 1], acc[b + 2], acc[b + 3]);
              mem_fence_compiler();
            }
          } else {
#pragma unroll
            for (int i = 0; i < G; ++i) {
              float4 v[T / 4];
              expand(wd[i], v);
              apply(v, wv[i]);
#pragma unroll
              for (int b = 0; b < T; b += 4) pin4(acc[b], acc[b + 1], acc[b + 2], acc[b + 3]);
              mem_fence_compiler();
            }
          }
        }
      } else {
        for (int sl = 0; sl < K; ++sl) {
          const int2 e = ej(sl);
          float4 v[T / 4];
          expand(*reinterpret_cast<const W *>(tb + (unsigned)e.x), v);
          apply(v, __int_as_float(e.y));
        }
      }
      if (jin) {
        // rows past nvalid have all-zero bits, so their outputs are zeros
        const float bj = bias[j];
        if constexpr (CODES) {
          uint4 *dst = reinterpret_cast<uint4 *>(reinterpret_cast<unsigned char *>(fout) +
                                                 ((size_t)(p0 / CR) * N + j) * CR + p0 % CR);
          // every row's value (in place of its accumulator), then per 16 rows the LDS cache's codes;
          // the full lookup (global table included) only on a lane where one of them missed
#pragma unroll
          for (int u = 0; u < T; ++u) {
            acc[u] = activate(acc[u], bj, ymax);
            live |= (acc[u] > 0.0f ? 1u : 0u) << u;
          }
          unsigned cw[T / 4];
          // rows [R0, R0 + 16), R0 a compile-time constant (so that every array index is one)
          auto encode16 = [&](auto r0c) {
            constexpr int R0 = decltype(r0c)::value;
            unsigned code[16];
            bool miss = false;
#pragma unroll
            for (int u = 0; u < 16; ++u) miss |= !cache_lookup(__float_as_uint(acc[R0 + u]), dlk, dlc, &code[u]);
            if (miss) {
#pragma unroll
              for (int u = 0; u < 16; ++u) code[u] = dict_code(acc[R0 + u], dlk, dlc, gd, overflow);
            }
#pragma unroll
            for (int n = 0; n < 4; ++n)
              cw[R0 / 4 + n] = code[4 * n] | (code[4 * n + 1] << 8) | (code[4 * n + 2] << 16) | (code[4 * n + 3] << 24);
          };
          encode16(std::integral_constant<int, 0>{});
          if constexpr (T == 32) encode16(std::integral_constant<int, 16>{});
#pragma unroll
          for (int n = 0; n < T / 16; ++n) dst[n] = make_uint4(cw[4 * n], cw[4 * n + 1], cw[4 * n + 2], cw[4 * n + 3]);
          // the rest of the last code tile gets code 0 (+0.0)
          if (t + 1 == ntiles)
            for (int n = T / 16; n < (CR - p0 % CR) / 16; ++n) dst[n] = make_uint4(0u, 0u, 0u, 0u);
        } else {
          float4 *dst = reinterpret_cast<float4 *>(fout + ((size_t)(p0 >> 5) * N + j) * 32 + (p0 & 31));
#pragma unroll
          for (int n = 0; n < T / 4; ++n) {
            const float4 y = make_float4(activate(acc[4 * n], bj, ymax), activate(acc[4 * n + 1], bj, ymax),
                                         activate(acc[4 * n + 2], bj, ymax), activate(acc[4 * n + 3], bj, ymax));
            dst[n] = y;
            live |= ((y.x > 0.0f ? 1u : 0u) | (y.y > 0.0f ? 2u : 0u) | (y.z > 0.0f ? 4u : 0u) | (y.w > 0.0f ? 8u : 0u))
                    << (4 * n);
          }
          if (T == 16 && (p0 & 31) == 0 && t + 1 == ntiles) {
            // the last 32-row tile has no second half: zero its slots 16..31
#pragma unroll
            for (int n = 0; n < 4; ++n) dst[4 + n] = make_float4(0.f, 0.f, 0.f, 0.f);
          }
        }
      }
    }
    if (live) atomicOr(&tilemask, live);
    __syncthreads();
    if (tid == 0) {
      unsigned m = tilemask;
      tilemask = 0u;
      m &= nvalid >= 32 ? 0xffffffffu : ((1u << nvalid) - 1u);
      if (m) atomicOr(&masks[p0 >> 5], m << (p0 & 31));
    }
    __syncthreads();
  }
}

// Dictionary of a uniform layer on binary inputs (every column K sources, weight w, bias b): a
// column with c sources at 1 has z = z_c, the fp32 chain of c fma(1, w, .) steps from +0 (the steps
// with input 0 leave the accumulator unchanged: fma(0, w, acc) = acc since acc is never -0), so its
// output is dict[c] = activate(z_c, b). Codes c in [0, K]; the other slots are left free.
// misc[kCountMinSlot] receives the smallest c with dict[c] > 0 (K + 1 if none; with w > 0 the
// outputs grow with c, so a row is live exactly when one of its counts reaches it).
constexpr int kCountMinSlot = 3;
__global__ void k_count_dict(unsigned *__restrict__ dict, int *__restrict__ misc, int K, float w, float b,
                             float ymax) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  float z = 0.0f;
  int cmin = K + 1;
  for (int c = 0; c <= K; ++c) {
    const float y = activate(z, b, ymax);
    dict[c] = __float_as_uint(y);
    if (y > 0.0f && cmin > K) cmin = c;
    z = fmaf(1.0f, w, z);
  }
  misc[kCountMinSlot] = cmin;
}

// Carry-save adder on bit-sliced words: per bit position, a + b + c = sum + 2 * carry.
__device__ __forceinline__ void csa(unsigned &carry, unsigned &sum, unsigned a, unsigned b, unsigned c) {
  carry = __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);  // majority
  sum = __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);    // three-way xor
}

// Layer 0 of a uniform layer (K = 32, w > 0) on bit tiles of T rows: for each output, the counts
// of set input bits among its 32 sources, for all rows of a word at once. The 32 source words go
// through a carry-save adder tree (two 16-word blocks), giving the six bit planes of the counts
// (0..32); a bit-sliced comparison with the first live count gives the live rows, and a transpose
// turns the planes into one byte per row: the output's code, decoded by the dictionary of
// k_count_dict. blockDim 1024; lane = output (T = 32) or outputs j and j + 64 in the low and high
// halves of each word (T = 16). LDS holds the tile's N words; the source indices are read 8 per
// 16-byte load from the [4][N][8] u16 table. Codes go to tiles of CR rows, one byte per row. With
// ROWMAJOR (T = 32; widths staged in LDS) the outputs are decoded instead and written as fp32 rows,
// yout[ids[p]][j] = dict[code] (the dictionary is copied after the tile in LDS). With cols set, only
// the ncols columns cols[p] are computed, their source lists in ell16 as [4][ncols][8].
template <int T, bool ROWMAJOR>
__global__ __launch_bounds__(1024) void k_layer_count(const typename BitWord<T>::type *__restrict__ bits,
                                                      unsigned char *__restrict__ cout, int N,
                                                      const uint4 *__restrict__ ell16, const int *__restrict__ misc,
                                                      const int *__restrict__ count, unsigned *__restrict__ masks,
                                                      float *__restrict__ yout, const int *__restrict__ ids,
                                                      const unsigned *__restrict__ dict, const int *__restrict__ cols,
                                                      int ncols, const int *__restrict__ skip) {
  static_assert(!ROWMAJOR || T == 32, "rows of fp32 outputs from 32-row bit tiles");
  if (*skip) return;  // an input is not 0 or 1 (found by k_pack_bits): the layer goes another way
  constexpr int CR = code_rows(T);
  using W = typename BitWord<T>::type;
  constexpr int OPL = T == 16 ? 2 : 1;  // outputs per lane
  extern __shared__ float4 smem[];
  unsigned &tilemask = *reinterpret_cast<unsigned *>(smem);
  W *tile = reinterpret_cast<W *>(smem + 1);
  // ROWMAJOR: the dictionary, then the tile's row ids, after the tile's words
  float *dl = reinterpret_cast<float *>(tile + ((N + 3) / 4) * 4);
  int *rid = reinterpret_cast<int *>(dl + kDictSlots);
  if constexpr (ROWMAJOR)
    for (int i = threadIdx.x; i < kDictSlots; i += blockDim.x) dl[i] = __uint_as_float(dict[i]);
  const int R = *count;
  const int cmin = misc[kCountMinSlot];
  const int ntiles = (R + T - 1) / T;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
  const int blocks = (ncols + 64 * OPL - 1) / (64 * OPL);  // output blocks of one wave
  const int rounds = (blocks + nw - 1) / nw;
  const Chunking ch = chunking(ntiles, rounds);
  // whole tiles as items: keep the tiles of one code group on one XCD
  const bool grouped = ch.nchunks == 1 && gridDim.x % (8 * (CR / T)) == 0;
  const int items = grouped ? (ntiles + gridDim.x - 1) / gridDim.x * gridDim.x : ntiles * ch.nchunks;
  if (tid == 0) tilemask = 0u;
  for (int w = blockIdx.x; w < items; w += gridDim.x) {
    const int t = grouped ? code_group_tile(w, CR / T) : w / ch.nchunks;
    const int c = grouped ? 0 : w % ch.nchunks;
    if (t >= ntiles) continue;  // uniform over the workgroup
    const int p0 = t * T;
    const int nvalid = min(T, R - p0);
    {
      const W *src = bits + (size_t)t * N;
      if ((reinterpret_cast<uintptr_t>(src) & 15) == 0) {
        const int n16 = (int)(((size_t)N * sizeof(W)) / 16);
        for (int i = tid; i < n16; i += blockDim.x) reinterpret_cast<int4 *>(tile)[i] = reinterpret_cast<const int4 *>(src)[i];
        for (int k = n16 * (int)(16 / sizeof(W)) + tid; k < N; k += blockDim.x) tile[k] = src[k];
      } else {
        for (int k = tid; k < N; k += blockDim.x) tile[k] = src[k];
      }
    }
    if constexpr (ROWMAJOR)
      if (threadIdx.x < T) rid[threadIdx.x] = (int)threadIdx.x < nvalid ? ids[p0 + threadIdx.x] : -1;
    __syncthreads();
    unsigned live = 0u;
    const int r_end = min(rounds, (c + 1) * ch.rounds_per_chunk);
    for (int r = c * ch.rounds_per_chunk; r < r_end; ++r) {
      const int blk = r * nw + wave;
      if (blk >= blocks) break;
      int jo[OPL], jc[OPL];  // output position and its column
      bool jin[OPL];
#pragma unroll
      for (int u = 0; u < OPL; ++u) {
        jo[u] = blk * 64 * OPL + u * 64 + lane;
        jin[u] = jo[u] < ncols;
        jc[u] = cols ? cols[min(jo[u], ncols - 1)] : jo[u];
      }
      // the 32 source indices of each output, 8 per load (positions past the last read the last)
      uint4 ix[OPL][4];
#pragma unroll
      for (int u = 0; u < OPL; ++u)
#pragma unroll
        for (int g = 0; g < 4; ++g) ix[u][g] = ell16[(size_t)g * ncols + min(jo[u], ncols - 1)];
      auto word = [&](int sl) -> unsigned {
        unsigned x = 0u;
#pragma unroll
        for (int u = 0; u < OPL; ++u) {
          const uint4 q = ix[u][sl >> 3];
          const unsigned pr = ((sl & 7) < 4) ? ((sl & 7) < 2 ? q.x : q.y) : ((sl & 7) < 6 ? q.z : q.w);
          const unsigned k = (sl & 1) ? (pr >> 16) : (pr & 0xffffu);
          x |= (unsigned)tile[k] << (16 * u);
        }
        return x;
      };
      // carry-save adder tree over two blocks of 16 source words
      unsigned ones = 0u, twos = 0u, fours = 0u, eights = 0u, s16[2];
#pragma unroll
      for (int blk16 = 0; blk16 < 2; ++blk16) {
        const int b0 = 16 * blk16;
        unsigned twosA, twosB, foursA, foursB, eightsA, eightsB;
        csa(twosA, ones, ones, word(b0 + 0), word(b0 + 1));
        csa(twosB, ones, ones, word(b0 + 2), word(b0 + 3));
        csa(foursA, twos, twos, twosA, twosB);
        csa(twosA, ones, ones, word(b0 + 4), word(b0 + 5));
        csa(twosB, ones, ones, word(b0 + 6), word(b0 + 7));
        csa(foursB, twos, twos, twosA, twosB);
        csa(eightsA, fours, fours, foursA, foursB);
        csa(twosA, ones, ones, word(b0 + 8), word(b0 + 9));
        csa(twosB, ones, ones, word(b0 + 10), word(b0 + 11));
        csa(foursA, twos, twos, twosA, twosB);
        csa(twosA, ones, ones, word(b0 + 12), word(b0 + 13));
        csa(twosB, ones, ones, word(b0 + 14), word(b0 + 15));
        csa(foursB, twos, twos, twosA, twosB);
        csa(eightsB, fours, fours, foursA, foursB);
        csa(s16[blk16], eights, eights, eightsA, eightsB);
      }
      const unsigned pl[6] = {ones, twos, fours, eights, s16[0] ^ s16[1], s16[0] & s16[1]};
      // rows whose count reaches cmin (bit-sliced comparison from the top plane down)
      unsigned gt = 0u, eq = 0xffffffffu;
#pragma unroll
      for (int i = 5; i >= 0; --i) {
        if ((cmin >> i) & 1) {
          eq &= pl[i];
        } else {
          gt |= eq & pl[i];
          eq &= ~pl[i];
        }
      }
      const unsigned ge = cmin > 63 ? 0u : (gt | eq);
      // transpose the planes into one byte per row: dword d holds rows 4d..4d+3
      unsigned cw[8];
#pragma unroll
      for (int d = 0; d < 8; ++d) {
        unsigned acc = 0u;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
          const unsigned nib = (pl[i] >> (4 * d)) & 15u;
          acc |= ((nib * 0x00204081u) & 0x01010101u) << i;
        }
        cw[d] = acc;
      }
#pragma unroll
      for (int u = 0; u < OPL; ++u) {
        if (!jin[u]) continue;
        const unsigned rows = T == 16 ? ((ge >> (16 * u)) & 0xffffu) : ge;
        live |= rows;
        if constexpr (ROWMAJOR) {
          // row b's code is byte b % 4 of cw[b / 4]; rows past the list are not written
#pragma unroll
          for (int b = 0; b < T; ++b) {
            const int row = rid[b];
            if (row >= 0) yout[(size_t)row * N + jc[u]] = dl[(cw[b >> 2] >> (8 * (b & 3))) & 255u];
          }
          continue;
        }
        uint4 *dst = reinterpret_cast<uint4 *>(cout + ((size_t)(p0 / CR) * N + jc[u]) * CR + p0 % CR);
        // plain stores: the tiles of one code group fill each segment in parts, merged in L2
        if (T == 32) {
          dst[0] = make_uint4(cw[0], cw[1], cw[2], cw[3]);
          dst[1] = make_uint4(cw[4], cw[5], cw[6], cw[7]);
        } else {
          dst[0] = make_uint4(cw[4 * u], cw[4 * u + 1], cw[4 * u + 2], cw[4 * u + 3]);
        }
        // the rest of the last code tile gets code 0 (+0.0)
        if (t + 1 == ntiles)
          for (int n = T / 16; n < (CR - p0 % CR) / 16; ++n) dst[n] = make_uint4(0u, 0u, 0u, 0u);
      }
    }
    if (live) atomicOr(&tilemask, live);
    __syncthreads();
    if (tid == 0) {
      unsigned m = tilemask;
      tilemask = 0u;
      m &= nvalid >= 32 ? 0xffffffffu : ((1u << nvalid) - 1u);
      if (m) atomicOr(&masks[p0 >> 5], m << (p0 & 31));
    }
    __syncthreads();
  }
}

// The workspace of sdnn_infer_static: a file-scope array in device memory, 64 MiB, of which each
// device that loads the library holds its own copy until the process ends. Host code never passes
// the array's name to a kernel or a copy (on the host it is a stand-in, not a device address): it
// uses the address hipGetSymbolAddress returns for the current device, looked up once per device.
constexpr size_t kStaticWorkspaceBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticWorkspaceBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on `device`, which must be the current device.
sdnn_status scratch_address(int device, void **out) {
  if (device < 0 || device >= kMaxDevices) return fail(SDNN_EINVAL, "device %d out of range", device);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      (void)hipGetLastError();
      return fail(SDNN_EDEVICE, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
    }
    g_scratch_ptr[device] = p;
  }
  *out = g_scratch_ptr[device];
  return SDNN_OK;
}

}  // namespace

// ------------------------------------------------------------------------------------------------
// Host side

struct LayerDev {
  const int2 *ell = nullptr;
  // layer 0 of the global-tile path (bit route): the ELL with each source given as the byte offset
  // of its word in a bit tile (source k * sizeof(word)) instead of its offset in a 32-row fp32 tile
  const int2 *ellw = nullptr;
  const float *bias = nullptr;
  int K = 0;
  // uniform layer (set only with the opt-in equal-value kernels): every column holds exactly K
  // sources, all weights are w and all biases b
  bool uniform = false;
  float w = 0.0f, b = 0.0f;
  // layer with K == 32 on widths staged in LDS, and uniform layer 0 of any width: [K/8][N][8] u16
  // source indices, eight per 16-byte load; unless the layer is uniform, its weights in the same
  // order, [K/4][N][4] fp32 (w8): 16-byte loads of consecutive columns are consecutive (grouped by 8, each
  // load touched every second 16 bytes and the fused launch took up to 6% longer)
  const uint4 *ell16 = nullptr;
  const float *w8 = nullptr;
  // LDS row placement for k_layer_lds (path 0, the first kPlacedLayers layers with ell16): neuron k
  // of the layer's input is staged at tile row place[k], and pell16 is ell16 with every source k
  // replaced by place[k] (see bank_placement)
  const unsigned short *place = nullptr;
  const uint4 *pell16 = nullptr;
  // global-tile path, layer with K == 32 and N <= 65536: [K][N] u16 source indices (the ELL's
  // sources), and unless the layer is uniform its weights [K][N] fp32 beside them (w32)
  const unsigned short *src16 = nullptr;
  const float *w32 = nullptr;
  // distinct columns (uniform layer with K == 32): columns with equal source lists have equal
  // outputs, so only the D representatives cols[0..D) need computing, with their source lists in
  // src16c ([K][D] u16, beside src16) and ell16c ([K/8][D][8], beside ell16). Usable (dedup_ok) once
  // the next layer's sources point to representatives only (or for the last layer).
  const int *cols = nullptr;
  const unsigned short *src16c = nullptr;
  const uint4 *ell16c = nullptr;
  // layer 0 of a uniform layer with K == 32: the lists of ell16 (and ell16c) with each column's
  // sources reordered for the counting kernel, whose counts do not depend on the order
  const uint4 *ell16s = nullptr, *ell16cs = nullptr;
  // widths staged in LDS: the positions of ell16 (and of ell16c) reordered for the fused kernel
  // with tiles of 4 << c rows (c = 0 also serves 1 and 2; see conflict_grouped_order): gcols[c][p]
  // is the column at position p, gell16[c] its sources
  const int *gcols[3] = {}, *gcolsc[3] = {};
  const uint4 *gell16[3] = {}, *gell16c[3] = {};
  const float *gw8[3] = {};  // the weights of gell16's positions (layers with w8)
  int D = 0;
  bool dedup_ok = false;
  // global-tile path, widths up to kSegMaxNeurons, without the equal-value kernels: the layer's
  // columns as k_layer_seg reads them
  const uint4 *seg = nullptr;
  const int2 *segdesc = nullptr;
  const uint2 *segcol = nullptr;  // (null in every layer: no memory for them, the network runs on tiles)
};

// A layer's columns as k_layer_seg reads them: blocks of 64 columns, each with its groups of 8 terms per
// segment. Formed in the pass that writes the layer's ELL, its sources in the caches. Loading without /
// with the streams (ms): 96 layers of 16384 neurons, 32 sources, 211 / 209; 1 to 48 sources 202 / 206; 24
// loads of one such layer of 4100 neurons 9.6 / 11.0 (with passes and a comparison sort of their own: 217, 216, 14.0).
int seg_segments(int N) { return N <= kSegCap ? 1 : 2; }
int seg_blocks(int N) { return (N + 63) / 64; }
int seg_positions(int N) { return (int)align_up((size_t)N, kSegThreads); }

// src(j, i): source i of column j, ascending; deg(j): its number of sources. Written: desc [S][blocks], colb
// and cut [positions] (see k_layer_seg and k_pack_seg). Returns the number of groups.
template <class Src, class Deg>
size_t seg_order(int N, Src src, Deg deg, const float *bias, int2 *desc, uint2 *colb, uint32_t *cut) {
  const int S = seg_segments(N), nb = seg_blocks(N);
  // terms of column j in segment 0 (first) and groups of 8 per segment: sources below N - kSegCap
  // have to be in segment 0, those from kSegCap in segment 1, and the cut is free between them: the
  // fewest groups, then the most even cut (one class of columns is one run length for its waves)
  static_assert(kMaxDegree < 1 << 16, "a cut and a key hold numbers of sources and of groups in 16 bits");
  std::vector<uint32_t> key((size_t)N);  // groups of both segments << 16 | groups of segment 0
  std::vector<uint16_t> first((size_t)N);
  uint32_t most = 0;
  bool one_key = true;
  for (int j = 0; j < N; ++j) {
    const int d = deg(j);
    int n0 = d;
    if (S == 2 && d % 16 == 0 && d > 0 && src(j, d / 2 - 1) < kSegCap && src(j, d / 2) >= N - kSegCap) {
      n0 = d / 2;  // the fewest groups, evenly
    } else if (S == 2) {
      int lo = 0, hi = 0;
      while (lo < d && src(j, lo) < N - kSegCap) ++lo;
      hi = lo;
      while (hi < d && src(j, hi) < kSegCap) ++hi;
      int best = 1 << 30;
      auto take = [&](int n) {
        const int a = (n + 7) / 8, b = (d - n + 7) / 8;
        const int cost = (a + b) * 4096 + std::abs(a - b);
        if (cost < best) { best = cost; n0 = n; }
      };
      take(lo);
      take(hi);
      for (int n = (lo + 7) / 8 * 8; n <= hi; n += 8) take(n);
      for (int n = hi; n >= lo && n > hi - 8; --n)  // the cuts that fill segment 1's last group
        if ((d - n) % 8 == 0) take(n);
    }
    first[(size_t)j] = (uint16_t)n0;
    const uint32_t a = (uint32_t)(n0 + 7) / 8, b = (uint32_t)(d - n0 + 7) / 8;
    key[(size_t)j] = (a + b) << 16 | a;
    most = std::max(most, a + b);
    one_key = one_key && key[(size_t)j] == key[0];
  }
  // longest columns first (blocks go round the waves, so every wave gets some), stable, so that equal
  // columns stay in order and their outputs are consecutive: a place per (a + b, a <= a + b), from the largest
  auto bucket = [](uint32_t k) { return (size_t)(k >> 16) * ((k >> 16) + 1) / 2 + (k & 0xffffu); };
  std::vector<int32_t> place;
  if (!one_key) {
    place.assign((size_t)(most + 1) * (most + 2) / 2, 0);
    for (int j = 0; j < N; ++j) ++place[bucket(key[(size_t)j])];
    int32_t at = 0;
    for (size_t q = place.size(); q-- > 0;) {
      const int32_t n = place[q];
      place[q] = at;
      at += n;
    }
  }
  for (int k = 0; k < S * nb; ++k) desc[k] = make_int2(0, 0);
  for (int j = 0; j < N; ++j) {
    const uint32_t k = key[(size_t)j], a = k & 0xffffu, b = (k >> 16) - a;
    const int p = one_key ? j : place[bucket(k)]++;
    uint32_t bits;
    std::memcpy(&bits, &bias[j], sizeof bits);
    colb[p] = make_uint2((uint32_t)j, bits);
    cut[p] = first[(size_t)j] | ((uint32_t)deg(j) << 16);
    desc[p / 64].y = std::max(desc[p / 64].y, (int)a);
    if (S == 2) desc[nb + p / 64].y = std::max(desc[nb + p / 64].y, (int)b);
  }
  for (int p = N; p < seg_positions(N); ++p) {
    colb[p] = make_uint2(kNoColumn, 0u);
    cut[p] = 0u;
  }
  // a wave's groups in the order it sums them: segment by segment, its blocks in turn (an empty
  // block's first group is that of the next one, which the kernel loads ahead)
  size_t groups = 0;
  for (int w = 0; w < 16; ++w)
    for (int sg = 0; sg < S; ++sg)
      for (int k = w; k < nb; k += 16) {
        int2 &d = desc[sg * nb + k];
        d.x = (int)groups;
        groups += (size_t)d.y;
      }
  return groups;
}

// Layers (from layer 0) that get an LDS row placement: the per-layer kernel runs the first layers
// of a batch, before the fused launch takes over.
constexpr int kPlacedLayers = 64;

// LDS row placement for k_layer_lds. The kernel reads a source's B rows (B * 4 bytes) with 16-byte
// lane reads; an LDS cycle serves 16 lanes (256 bytes, 64 banks), which are the G = 64 / B
// consecutive output columns of a group at one slot. Row r of the tile starts at bank (r B) mod 64,
// so the group's reads of distinct sources collide when their rows agree mod G; the cycles a read
// takes are the largest number of distinct sources on one residue. The sources of a column are
// fixed (and their order, which is the summation order), but the row of each neuron in the tile is
// free: this local search swaps the rows of two neurons whenever the summed cycles of the (group,
// slot) reads that involve them do not grow. h16: the layer's [4][N][8] source groups (ell16).
std::vector<uint16_t> bank_placement(const uint16_t *h16, int N, int B, uint64_t seed, int iters) {
  const int G = std::max(1, 64 / B);
  std::vector<uint16_t> place((size_t)N);
  for (int k = 0; k < N; ++k) place[(size_t)k] = (uint16_t)k;
  if (G < 2 || N < 2 * G) return place;
  auto srcof = [&](int j, int sl) { return (int)h16[((size_t)(sl / 8) * N + j) * 8 + sl % 8]; };
  const int ngroups = (N + G - 1) / G;
  // (group, slot) reads of each neuron, as a CSR over neurons
  std::vector<int> deg((size_t)N + 1, 0);
  for (int j = 0; j < N; ++j)
    for (int sl = 0; sl < 32; ++sl) ++deg[(size_t)srcof(j, sl) + 1];
  for (int k = 0; k < N; ++k) deg[(size_t)k + 1] += deg[(size_t)k];
  std::vector<int> occ((size_t)deg[(size_t)N]), fill(deg.begin(), deg.end() - 1);
  for (int j = 0; j < N; ++j)
    for (int sl = 0; sl < 32; ++sl) occ[(size_t)fill[(size_t)srcof(j, sl)]++] = (j / G) * 32 + sl;
  auto cycles = [&](int gs) {
    const int g = gs / 32, sl = gs % 32;
    int rows[64], n = 0, load[64] = {0}, m = 0;
    for (int j = g * G; j < std::min(N, g * G + G); ++j) {
      const int k = srcof(j, sl);
      bool dup = false;
      for (int t = 0; t < n; ++t) dup |= rows[t] == k;
      if (dup) continue;
      rows[n++] = k;
      m = std::max(m, ++load[place[(size_t)k] % G]);
    }
    return m;
  };
  (void)ngroups;
  uint64_t x = seed;
  auto next = [&]() {  // SplitMix64
    x += 0x9E3779B97F4A7C15ull;
    uint64_t z = x;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
  };
  std::vector<int> touched;
  for (int it = 0; it < iters; ++it) {
    const int a = (int)(next() % (uint64_t)N), c = (int)(next() % (uint64_t)N);
    if (place[(size_t)a] % G == place[(size_t)c] % G) continue;
    touched.clear();
    for (int t = deg[(size_t)a]; t < deg[(size_t)a + 1]; ++t) touched.push_back(occ[(size_t)t]);
    for (int t = deg[(size_t)c]; t < deg[(size_t)c + 1]; ++t) touched.push_back(occ[(size_t)t]);
    std::sort(touched.begin(), touched.end());
    touched.erase(std::unique(touched.begin(), touched.end()), touched.end());
    int before = 0, after = 0;
    for (int gs : touched) before += cycles(gs);
    std::swap(place[(size_t)a], place[(size_t)c]);
    for (int gs : touched) after += cycles(gs);
    if (after > before) std::swap(place[(size_t)a], place[(size_t)c]);
  }
  return place;
}

}  // namespace

struct sdnn_net {
  int32_t N = 0, L = 0;
  float ymax = 32.0f;
  int path = 0;  // 0: LDS tiles, 1: global feature-major tiles
  int B = 0;     // rows per tile: LDS tile (path 0) or global feature-major tile (path 1)
  int bitsT = 0; // rows per layer-0 bit tile (path 1), 0 if the bit route is not available
  int device = -1;
  int cus = 0;
  bool poisoned = false;
  // kernels that exploit layers whose weights and biases are all equal (opt-in, before any load;
  // see sdnn_enable_equal_value_kernels)
  bool equal_value_kernels = false;
  std::vector<LayerDev> layers;
  std::vector<void *> allocations;
  // duplicate columns: representatives of the last layer loaded (rep[j] = smallest column with j's
  // source list), which the next layer's sources are mapped through when it is loaded right after
  std::vector<int32_t> prev_rep;
  int32_t prev_rep_layer = -1;
  std::vector<int32_t> last_rep;  // the same for layer L - 1 (final rows are expanded through it)
  // device tables of the layers, for launches that run several layers: one per fused tile height
  // class (4 << c rows; class 0 also for 1 and 2 rows)
  LayerPtr *lp_dev[3] = {};
  int32_t n_loaded = 0;
  std::vector<void *> streams;  // device allocations of segment streams (LayerDev::seg)
  bool no_streams = false;      // their memory was needed for layers
  int32_t n_edge32 = 0;  // layers with grouped 32-source lists and per-edge weights (see k_layers_lds32)
  // last run
  bool ran = false;
  int64_t M = 0;
  hipStream_t stream = nullptr;
  char *ws = nullptr;
  float *ybuf[2] = {nullptr, nullptr};  // path 0: row-major activations
  float *fm[2] = {nullptr, nullptr};    // path 1: feature-major tiles of 32 list positions
  int *ids[2] = {nullptr, nullptr};     // live lists: row id per position
  int *src[2] = {nullptr, nullptr};     // path 1: position in the previous list, per position
  unsigned *masks = nullptr;               // per-tile liveness bits (path 1: layers l % 3 == 0)
  unsigned *masks_rot[3] = {nullptr, nullptr, nullptr};  // path 1: layer l uses masks_rot[l % 3]
  int *rownz = nullptr, *counts = nullptr;
  int *misc = nullptr;  // device flags and counters: [0] a layer-0 input is not 0 or 1, [2] dictionary full,
                        // [4 + i] positions in list i
  unsigned *dict = nullptr;  // value dictionary of one-byte activation codes (kDictWords words; decoding reads the first 256)
  unsigned *dict16 = nullptr;  // path 1: the dictionary of two-byte codes (dict_words<2>() words)
  unsigned *seglive = nullptr;  // path 1: per fp32 tile, one bit per source: the segment was stored
  unsigned *part[2] = {nullptr, nullptr};  // path 1: partial liveness words of few-tile layers, by layer parity
  unsigned *spread = nullptr;              // path 1: liveness words of large layers, one 128-byte line each
  long long *final_ids = nullptr;
  int final_list = 0;        // which ids buffer holds the final list
  int32_t layers_run = 0;    // layers enqueued by the last infer
  std::vector<int32_t> layer_kernel, layer_launches;  // per layer of the last infer (sdnn_layer_info)
  // ... and whether it ran on k_layer_seg or a list-ahead kernel of that family (sdnn_layer_kernel)
  std::vector<char> layer_ahead;
  const float *final_y = nullptr;   // path 0: final activations, row-major by row id
  const float *final_fm = nullptr;  // path 1: final activation tiles; live row i is at position src[final_list][i]
  bool final_rows_major = false;    // ... or rows by position (k_layer_seg's outputs)
  int32_t *pinned = nullptr; // read-back slots (0-3: polling ring, 6: input-not-binary flag, 7: exact count)
  // progress word of few-tile layers, in coherent host memory written by the device (see
  // progress_word); progress_dev is its device address
  unsigned long long *progress = nullptr, *progress_dev = nullptr;
  // word in coherent host memory where a compaction reports its count and flags (see k_compact);
  // notify_dev is its device address, notify_seq the tag of the last report asked for
  unsigned long long *notify = nullptr, *notify_dev = nullptr;
  uint32_t notify_seq = 0;
  HostOut *host_out = nullptr, *host_out_dev = nullptr;  // see HostOut
  bool finished = false;     // host_out holds the last infer's categories (see finish)
  uint32_t run_gen = 0;      // generation of the current infer, in the progress word's top bits
  std::vector<hipEvent_t> events;
  // profiling
  bool profiling = false;
  int prof_mode = 0;              // 1: every layer, 2: large layers only
  std::vector<char> prof_rec;     // layers recorded by the last infer
  bool pending_times = false;
  std::vector<hipEvent_t> prof_start, prof_end;
  std::vector<double> prof_ms;
  std::vector<int64_t> prof_runs;
};

namespace {

#define HIP_OR_POISON(net, call)                                                                   \
  do {                                                                                             \
    hipError_t e_ = (call);                                                                        \
    if (e_ != hipSuccess) {                                                                        \
      (net)->poisoned = true;                                                                      \
      return fail(SDNN_EDEVICE, "%s failed: %s", #call, hipGetErrorString(e_));                   \
    }                                                                                              \
  } while (0)

struct WsLayout {
  size_t act[2], ids[2], src[2], masks[3], rownz, counts, misc, dict, dict16, seglive, part[2], spread, spread_words,
      final_ids, total;
};

// Two activation buffers: row-major [M][N] (path 0) or feature-major tiles of 32 rows (path 1).
WsLayout layout_for(const sdnn_net *net, int64_t M) {
  WsLayout w{};
  const size_t a = 256;
  size_t off = 0;
  const size_t rows = net->path == 1 ? (size_t)((M + 31) / 32) * 32 : (size_t)M;
  const size_t ybytes = align_up(rows * (size_t)net->N * sizeof(float), a);
  w.act[0] = off; off += ybytes;
  w.act[1] = off; off += ybytes;
  const size_t ib = align_up((size_t)std::max<int64_t>(M, 1) * sizeof(int), a);
  w.ids[0] = off; off += ib;
  w.ids[1] = off; off += ib;
  w.src[0] = off; off += ib;
  w.src[1] = off; off += ib;
  for (int i = 0; i < 3; ++i) { w.masks[i] = off; off += ib; }
  w.rownz = off; off += ib;
  w.counts = off; off += align_up((size_t)(net->L + 1) * sizeof(int), a);
  w.misc = off; off += a;
  w.dict = off; off += align_up(kDictWords * sizeof(unsigned), a);
  w.dict16 = off;
  if (net->path == 1) off += align_up((size_t)dict_words<2>() * sizeof(unsigned), a);
  w.seglive = off;
  if (net->path == 1) off += align_up(rows / 32 * (size_t)((net->N + 31) / 32) * sizeof(unsigned), a);
  for (int i = 0; i < 2; ++i) {
    w.part[i] = off;
    if (net->path == 1) off += align_up((size_t)kMaxPartWords * sizeof(unsigned), a);
  }
  w.spread = off;
  w.spread_words = net->path == 1 ? rows / 32 * kSpread * kLineWords : 0;
  off += align_up(w.spread_words * sizeof(unsigned), a);
  w.final_ids = off; off += align_up((size_t)std::max<int64_t>(M, 1) * sizeof(long long), a);
  w.total = off;
  return w;
}

sdnn_status check_usable(const sdnn_net *net) {
  if (!net) return fail(SDNN_EINVAL, "null handle");
  if (net->poisoned) return fail(SDNN_EDEVICE, "handle is poisoned by an earlier device error");
  return SDNN_OK;
}

// Whether a layer of at most `rows` live rows on widths staged in LDS runs on k_layer_lds32.
bool lists_ahead(const sdnn_net *net, const LayerDev &ld, int64_t rows) {
  if (!ld.ell16 || !ld.w8 || ld.cols || net->N % 4 != 0) return false;
  // k_layer_lds32 has one workgroup per CU, and its threads hold the rows of a tile of kLdsTileBytes: while it
  // stages narrow tiles nothing else runs, and two workgroups of k_layer_lds overlap where a CU has more
  // than one tile (narrower still, always). 60 layers, every row live, k_layer_lds / k_layer_lds32 (ms): 128
  // neurons x 4500 rows (half a tile per CU) 1.15 / 1.47, x 60,000 4.78 / 5.04; 192 x 8000 1.75 / 1.69, x
  // 150,000 (18 tiles per CU) 11.9 / 12.7; 256 x 20,000 2.82 / 3.03, x 60,000 6.09 / 6.22, x 150,000 15.1 / 13.9;
  // 320 x 8300 2.08 / 2.39, x 20,000 3.37 / 3.37, x 60,000 7.50 / 7.15; 448 x 12,000 2.85 / 2.94, x 16,500 3.78 / 3.68.
  const int64_t round = (int64_t)net->B * net->cus;  // rows of one tile per CU
  const bool narrow = net->N <= 128 || (rows > round && (net->N <= 192 || (net->N <= 256 && rows <= 8 * round) ||
                                                         (net->N <= 320 && rows <= 2 * round) ||
                                                         (net->N <= 448 && 2 * rows <= 3 * round)));
  return !narrow;
}

template <int B, int KC>
hipError_t launch_lds(sdnn_net *net, const float *yin, float *yout, const LayerDev &ld, const int *ids,
                      const int *count, int64_t rows, int *rownz) {
  static bool configured = false;
  const size_t lds = (size_t)B * net->N * sizeof(float);
  if (!configured) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_layer_lds<B, KC>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kLdsTileBytes);
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_layer_lds32<B>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, kLdsTileBytes);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const int per_cu = lds <= 64 * 1024 ? 2 : 1;
  // distinct columns only, when the layer's duplicates need not be computed
  const bool dd = ld.ell16 && ld.ell16c && ld.cols && ld.dedup_ok;
  const bool placed = !dd && ld.place && ld.pell16;
  if (lists_ahead(net, ld, rows)) {
    hipLaunchKernelGGL(k_layer_lds32<B>, dim3(net->cus), dim3(1024), lds, net->stream, yin, yout, net->N,
                       reinterpret_cast<const u32x4 *>(placed ? ld.pell16 : ld.ell16),
                       reinterpret_cast<const f32x4 *>(ld.w8), ld.bias, net->ymax, ids, count, net->masks, rownz,
                       placed ? ld.place : nullptr);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((k_layer_lds<B, KC>), dim3(net->cus * per_cu), dim3(1024), lds, net->stream, yin, yout, net->N,
                     ld.ell, ld.K, dd ? ld.ell16c : (placed ? ld.pell16 : ld.ell16), dd ? nullptr : ld.w8, ld.w,
                     ld.bias, net->ymax, ids, count, net->masks, rownz, dd ? ld.cols : nullptr, dd ? ld.D : net->N,
                     placed ? ld.place : nullptr);
  return hipGetLastError();
}

template <int B>
hipError_t launch_lds_k(sdnn_net *net, const float *yin, float *yout, const LayerDev &ld, const int *ids,
                        const int *count, int64_t rows, int *rownz) {
  if (ld.K == 32) return launch_lds<B, 32>(net, yin, yout, ld, ids, count, rows, rownz);
  return launch_lds<B, 0>(net, yin, yout, ld, ids, count, rows, rownz);
}

// A layer of at most 8 tiles with K == 32 (see k_layer_gfm_small). Liveness goes to the partial
// words part_out; *G_out and *nt_out receive their number and the tiles.
hipError_t launch_gfm_small(sdnn_net *net, const LayerDev &ld, const float *fin, float *fout, const int *npos,
                            int64_t max_tiles, unsigned *part_out, const unsigned *part_prev, int prev_G, int prev_nt,
                            unsigned *masks_prev, unsigned *masks_clear, int *count_out, const int *live_before,
                            unsigned long long *progress, unsigned long long progress_tag, int *G_out, int *nt_out) {
  const bool dd = ld.src16 && ld.cols && ld.dedup_ok;  // distinct columns only
  const int ncols = dd ? ld.D : net->N;
  const int nchunks = (ncols + 31) / 32;
  const int ntiles_h = (int)std::max<int64_t>(1, std::min<int64_t>(8, max_tiles));
  // at most kMaxPartWords workgroups, so that the partial words fit their buffer
  const int per_xcd = std::max(1, std::min({kMaxPartWords / 8, 2 * net->cus, (ntiles_h * nchunks + 7) / 8}));
  const dim3 grid(8 * per_xcd);
  *G_out = 8 * per_xcd;
  *nt_out = ntiles_h;
  if (ld.uniform && ld.src16)
    hipLaunchKernelGGL((k_layer_gfm_small<32, kWOne>), grid, dim3(kPartThreads), 0, net->stream, fin, fout, net->N,
                       ld.ell, dd ? ld.src16c : ld.src16, (const float *)nullptr, ld.w, ld.bias, net->ymax, npos,
                       ntiles_h, part_out, part_prev, prev_G, prev_nt, masks_prev, masks_clear, count_out, live_before,
                       progress, progress_tag, dd ? ld.cols : nullptr, ncols);
  else if (ld.src16 && ld.w32)
    hipLaunchKernelGGL((k_layer_gfm_small<32, kWEdge>), grid, dim3(kPartThreads), 0, net->stream, fin, fout, net->N,
                       ld.ell, ld.src16, ld.w32, ld.w, ld.bias, net->ymax, npos, ntiles_h, part_out, part_prev, prev_G,
                       prev_nt, masks_prev, masks_clear, count_out, live_before, progress, progress_tag,
                       (const int *)nullptr, net->N);
  else
    hipLaunchKernelGGL((k_layer_gfm_small<32, kWEll>), grid, dim3(kPartThreads), 0, net->stream, fin, fout, net->N,
                       ld.ell, ld.src16, (const float *)nullptr, ld.w, ld.bias, net->ymax, npos, ntiles_h, part_out,
                       part_prev, prev_G, prev_nt, masks_prev, masks_clear, count_out, live_before, progress,
                       progress_tag, (const int *)nullptr, net->N);
  return hipGetLastError();
}

// One layer of the global-tile path: ceil(tiles / 8) launches of 8 tiles each (rounds), reading fin
// and writing fout at the same list positions; *npos is the list length and max_tiles a host bound
// on its tiles. With count_out set (one round only) the launch first counts the previous layer's
// live rows from masks_prev and clears masks_clear.
// Tiles per XCD and launch for a layer that reads `bytes` of each input tile: as many as fit 2 MiB of
// the XCD's 4 MiB L2, at most 8.
int tiles_per_xcd(size_t bytes) {
  return (int)std::max<size_t>(1, std::min<size_t>(8, ((size_t)2 << 20) / std::max<size_t>(bytes, 1)));
}
// Launches of launch_gfm (fp32 tiles) or launch_gfm_u8 (code tiles of cr rows, cr > 0) for a layer
// over max_tiles fp32 tiles.
int32_t gfm_launches(const sdnn_net *net, const LayerDev &ld, int64_t max_tiles, int cr) {
  const bool dd = ld.K == 32 && ld.src16 && ld.cols && ld.dedup_ok;
  const int ncols = dd ? ld.D : net->N;
  if (cr > 0) max_tiles = (max_tiles + cr / 32 - 1) / (cr / 32);
  const int tpx = dd ? tiles_per_xcd((size_t)ncols * (cr > 0 ? cr : 32 * sizeof(float))) : 1;
  return (int32_t)((max_tiles + 8 * tpx - 1) / (8 * tpx));
}

hipError_t launch_gfm(sdnn_net *net, const LayerDev &ld, const float *fin, float *fout, const int *npos,
                      int64_t max_tiles, unsigned *masks, const unsigned *masks_prev = nullptr,
                      unsigned *masks_clear = nullptr, int *count_out = nullptr, unsigned *spread = nullptr) {
  // distinct columns only, when the layer's duplicates need not be computed
  const bool dd = ld.K == 32 && ld.src16 && ld.cols && ld.dedup_ok;
  const int ncols = dd ? ld.D : net->N;
  const int *cols = dd ? ld.cols : nullptr;
  const unsigned short *s16 = dd ? ld.src16c : ld.src16;
  // the few columns of such a layer touch a small part of each tile, so an XCD can keep several
  // tiles in its L2 and a launch covers 8 tpx of them
  const int tpx = dd ? tiles_per_xcd((size_t)ncols * 32 * sizeof(float)) : 1;
  const int rounds = (int)((max_tiles + 8 * tpx - 1) / (8 * tpx));
  // one workgroup per output chunk of a tile's share when the round has fewer than 8 tiles
  const int nchunks = (ncols + kGfmOutputs - 1) / kGfmOutputs;
  const int64_t parts = 8 / std::max<int64_t>(1, std::min<int64_t>(8, max_tiles));
  const int per_xcd = tpx * std::max(1, (int)std::min<int64_t>(net->cus, (nchunks + parts - 1) / parts));
  const dim3 grid(8 * per_xcd);
  for (int r = 0; r < rounds; ++r) {
    int *cnt = r == 0 ? count_out : nullptr;
    if (ld.K == 32 && ld.src16 && ld.uniform)
      hipLaunchKernelGGL((k_layer_gfm<kWOne>), grid, dim3(256), 0, net->stream, fin, fout, net->N, ld.ell, ld.K, s16,
                         (const float *)nullptr, ld.w, ld.bias, net->ymax, npos, masks, r * 8 * tpx, masks_prev,
                         masks_clear, cnt, spread, cols, ncols, tpx);
    else if (ld.K == 32 && ld.src16 && ld.w32)
      hipLaunchKernelGGL((k_layer_gfm<kWEdge>), grid, dim3(256), 0, net->stream, fin, fout, net->N, ld.ell, ld.K,
                         ld.src16, ld.w32, 0.0f, ld.bias, net->ymax, npos, masks, r * 8, masks_prev, masks_clear, cnt,
                         spread, (const int *)nullptr, net->N, 1);
    else
      hipLaunchKernelGGL((k_layer_gfm<kWEll>), grid, dim3(256), 0, net->stream, fin, fout, net->N, ld.ell, ld.K,
                         (const unsigned short *)nullptr, (const float *)nullptr, 0.0f, ld.bias, net->ymax, npos,
                         masks, r * 8, masks_prev, masks_clear, cnt, spread, (const int *)nullptr, net->N, 1);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// A layer on fp32 rows (see k_layer_seg): reads row map[p] of yin for list position p (null: row p),
// writes row p of yout.
hipError_t launch_seg(sdnn_net *net, const LayerDev &ld, const float *yin, float *yout, const int *map, const int *npos,
                      int64_t rows, unsigned *masks, int *rownz, const int *ids) {
  static std::atomic<bool> configured{false};
  if (!configured.load(std::memory_order_acquire)) {
    for (const void *k : {reinterpret_cast<const void *>(&k_layer_seg<1>), reinterpret_cast<const void *>(&k_layer_seg<2>)}) {
      const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (kSegCap + 1) * (int)sizeof(float4));
      if (e != hipSuccess) return e;
    }
    configured.store(true, std::memory_order_release);
  }
  const int nblk = seg_blocks(net->N), nob = (nblk + 15) / 16;
  const int64_t quads = (rows + 3) / 4;
  // fewer 4-row groups than CUs: split their outputs until the CUs are taken
  int nsplit = 1;
  if (quads < net->cus) nsplit = (int)std::min<int64_t>(nob, net->cus / std::max<int64_t>(1, quads));
  nsplit = std::max(1, nsplit);
  const int opw = (nob + nsplit - 1) / nsplit;
  nsplit = (nob + opw - 1) / opw;
  const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(net->cus, quads * nsplit));
  const size_t lds = ((size_t)std::min(net->N, kSegCap) + 1) * sizeof(float4);  // (+ two words)
  if (seg_segments(net->N) == 1)
    hipLaunchKernelGGL(k_layer_seg<1>, dim3(grid), dim3(kSegThreads), lds, net->stream, yin, yout, net->N, ld.seg,
                       ld.segdesc, ld.segcol, nblk, net->ymax, map, npos, nsplit, masks, net->spread, rownz, ids);
  else
    hipLaunchKernelGGL(k_layer_seg<2>, dim3(grid), dim3(kSegThreads), lds, net->stream, yin, yout, net->N, ld.seg,
                       ld.segdesc, ld.segcol, nblk, net->ymax, map, npos, nsplit, masks, net->spread, rownz, ids);
  return hipGetLastError();
}

hipError_t launch_to_fm(sdnn_net *net, const float *y, float *fm, const int *ids, const int *count, int *rownz) {
  hipLaunchKernelGGL(k_to_fm<32>, dim3(net->cus * 8), dim3(256), 0, net->stream, y, fm, net->N, ids, count, rownz);
  return hipGetLastError();
}

template <int T>
size_t bits_tile_bytes_needed(const sdnn_net *net) {
  using W = typename BitWord<T>::type;
  return (size_t)net->N * sizeof(W);
}

template <int T>
hipError_t launch_pack_bits(sdnn_net *net, const float *yin, void *bits, const int *ids, const int *count) {
  using W = typename BitWord<T>::type;
  hipLaunchKernelGGL(k_pack_bits<T>, dim3(net->cus * 8), dim3(256), 0, net->stream, yin, reinterpret_cast<W *>(bits),
                     net->N, ids, count, net->rownz, net->misc);
  return hipGetLastError();
}

template <int T, int KC, bool CODES>
hipError_t launch_layer_bits_k(sdnn_net *net, const LayerDev &ld, const void *bits, float *fout, const int *count) {
  using W = typename BitWord<T>::type;
  // one workgroup per CU: 16 waves at up to 128 registers fill the register file; LDS is static
  const int per_cu = 1;
  hipLaunchKernelGGL((k_layer_bits<T, KC, CODES>), dim3(net->cus * per_cu), dim3(kBitsThreads), 0, net->stream,
                     reinterpret_cast<const W *>(bits), fout, net->N, ld.ellw, ld.K, ld.bias, net->ymax,
                     count, net->masks, net->dict, net->misc + kOverflowSlot, net->misc);
  return hipGetLastError();
}

// codes: write one-byte dictionary codes instead of fp32 values
template <int T>
hipError_t launch_layer_bits(sdnn_net *net, const LayerDev &ld, const void *bits, float *fout, const int *count,
                             bool codes) {
  if (codes) {
    if (ld.K == 32) return launch_layer_bits_k<T, 32, true>(net, ld, bits, fout, count);
    return launch_layer_bits_k<T, 0, true>(net, ld, bits, fout, count);
  }
  if (ld.K == 32) return launch_layer_bits_k<T, 32, false>(net, ld, bits, fout, count);
  return launch_layer_bits_k<T, 0, false>(net, ld, bits, fout, count);
}

// Source order for the counting kernel. A wave's LDS read of one source slot serves 64 outputs, in
// two halves of 32 lanes (32 consecutive output positions); within a half, reads of different
// 4-byte words in the same one of the 32 banks are served one after another. The count does not
// depend on the order of a column's sources, so for each half the sources are dealt to the 32
// slots greedily: slot by slot, lanes with the fewest distinct remaining banks choose first, each
// taking a remaining source whose bank this slot has used least. src: [4][D][8] u16 lists; wbytes:
// bytes per LDS word of the bit tile (the word of source k is k * wbytes / 4).
std::vector<uint16_t> bank_balanced_lists(const uint16_t *src, int D, int wbytes) {
  std::vector<uint16_t> out((size_t)32 * D);
  const int groups = (D + 31) / 32;
  parallel_for(groups, [&](int32_t g) {
    const int p0 = g * 32, np = std::min(32, D - p0);
    uint16_t rem[32][32];
    int nrem[32];
    for (int i = 0; i < np; ++i) {
      for (int sl = 0; sl < 32; ++sl) rem[i][sl] = src[((size_t)(sl / 8) * D + p0 + i) * 8 + sl % 8];
      nrem[i] = 32;
    }
    auto word = [&](unsigned k) { return (unsigned)((k * (unsigned)wbytes) / 4u); };
    for (int sl = 0; sl < 32; ++sl) {
      int load[32] = {0};
      unsigned used[32][32];  // words of each bank read in this slot
      int order[32], key[32];
      for (int i = 0; i < np; ++i) {
        unsigned seen = 0u;
        for (int q = 0; q < nrem[i]; ++q) seen |= 1u << (word(rem[i][q]) & 31u);
        key[i] = __builtin_popcount(seen);
        order[i] = i;
      }
      std::stable_sort(order, order + np, [&](int a, int b) { return key[a] < key[b]; });
      for (int oi = 0; oi < np; ++oi) {
        const int i = order[oi];
        int best = 0, bcost = 1 << 30;
        for (int q = 0; q < nrem[i]; ++q) {
          const unsigned w = word(rem[i][q]), b = w & 31u;
          bool same = false;
          for (int u = 0; u < load[b]; ++u) same = same || used[b][u] == w;
          const int cost = same ? 0 : load[b] + 1;
          if (cost < bcost) { bcost = cost; best = q; }
        }
        const uint16_t k = rem[i][best];
        rem[i][best] = rem[i][--nrem[i]];
        const unsigned w = word(k), b = w & 31u;
        bool same = false;
        for (int u = 0; u < load[b]; ++u) same = same || used[b][u] == w;
        if (!same) used[b][load[b]++] = w;
        out[((size_t)(sl / 8) * D + p0 + i) * 8 + sl % 8] = k;
      }
    }
  });
  return out;
}

// Column order for the fused LDS kernel: a wave's 16-byte LDS reads of one source slot are served
// 16 lanes at a time, and reads of different rows in the same 16-byte bank group are served one
// after another. With B-row tiles (B = 4, 8, 16) an output takes B / 4 lanes, so a cycle serves
// G = 64 / B consecutive positions, and row k covers bank groups (B / 4) k .. (B / 4) k + B / 4 - 1
// mod 16: two of the G columns collide when their sources agree mod G. The fp32 chain fixes the
// order of a column's sources, but which columns share a read is free, so positions are filled in
// groups of G: each group starts from a remaining column and repeatedly takes, among 128 sampled
// remaining columns, the one whose sources add the fewest collisions over the 32 slots.
// lists: D x 32 sources by position; returns the positions' new order.
std::vector<int32_t> conflict_grouped_order(const std::vector<uint16_t> &lists, int D, int G) {
  std::vector<int32_t> order, rem((size_t)D);
  order.reserve((size_t)D);
  for (int i = 0; i < D; ++i) rem[(size_t)i] = i;
  uint64_t st = 0x5DEECE66Dull + (uint64_t)D;
  auto next = [&]() {  // SplitMix64
    uint64_t z = (st += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
  };
  auto take = [&](size_t idx) {
    const int32_t c = rem[idx];
    rem[idx] = rem.back();
    rem.pop_back();
    return c;
  };
  while (!rem.empty()) {
    uint8_t load[32][16] = {};
    auto add = [&](int32_t c) {
      for (int sl = 0; sl < 32; ++sl) ++load[sl][lists[(size_t)c * 32 + sl] % (unsigned)G];
      order.push_back(c);
    };
    add(take((size_t)(next() % rem.size())));
    for (int g = 1; g < G && !rem.empty(); ++g) {
      size_t best = 0;
      int bcost = 1 << 30;
      for (int t = 0; t < 128; ++t) {
        const size_t idx = (size_t)(next() % rem.size());
        const uint16_t *l = lists.data() + (size_t)rem[idx] * 32;
        int cost = 0;
        for (int sl = 0; sl < 32; ++sl) cost += load[sl][l[sl] % (unsigned)G];
        if (cost < bcost) { bcost = cost; best = idx; }
      }
      add(take(best));
    }
  }
  return order;
}

// Layer 0 of a uniform layer by counting (see k_layer_count): dictionary, then the counts as codes
// (cout) or, with yout set, as fp32 rows yout[ids[p]] (masks: one bit per list position).
template <int T, bool ROWMAJOR>
hipError_t launch_layer_count_k(sdnn_net *net, const LayerDev &ld, const void *bits, unsigned char *cout,
                                const int *count, float *yout, const int *ids, unsigned *masks) {
  using W = typename BitWord<T>::type;
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_layer_count<T, ROWMAJOR>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    configured = true;
  }
  hipLaunchKernelGGL(k_count_dict, dim3(1), dim3(64), 0, net->stream, net->dict, net->misc, ld.K, ld.w, ld.b, net->ymax);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  size_t lds = 16 + ((size_t)net->N * sizeof(W) + 15) / 16 * 16;
  if (ROWMAJOR) lds += kDictSlots * sizeof(float) + T * sizeof(int);
  // distinct columns only, when the layer's duplicates need not be computed
  const bool dd = ld.cols && ld.ell16c && ld.dedup_ok;
  hipLaunchKernelGGL((k_layer_count<T, ROWMAJOR>), dim3(net->cus), dim3(1024), lds, net->stream,
                     reinterpret_cast<const W *>(bits), cout, net->N,
                     dd ? (ld.ell16cs ? ld.ell16cs : ld.ell16c) : (ld.ell16s ? ld.ell16s : ld.ell16), net->misc, count, masks,
                     yout, ids, reinterpret_cast<const unsigned *>(net->dict), dd ? ld.cols : nullptr,
                     dd ? ld.D : net->N, net->misc);
  return hipGetLastError();
}
template <int T>
hipError_t launch_layer_count(sdnn_net *net, const LayerDev &ld, const void *bits, unsigned char *cout,
                              const int *count) {
  return launch_layer_count_k<T, false>(net, ld, bits, cout, count, nullptr, nullptr, net->masks);
}

// A layer whose input tiles hold dictionary codes of CR rows (see k_layer_gfm_u8); rounds of 8 code
// tiles. max_tiles: host bound on the 32-row tiles of the list.
template <int CR, int CB = 1>
hipError_t launch_gfm_u8_cr(sdnn_net *net, const LayerDev &ld, const unsigned char *cin, float *fout, const int *npos,
                            int64_t max_tiles, unsigned *masks, bool *seglive_used) {
  max_tiles = (max_tiles + CR / 32 - 1) / (CR / 32);  // code tiles
  // distinct columns only, when the layer's duplicates need not be computed (every segment of them
  // is then stored and seglive is not written)
  const bool dd = ld.K == 32 && ld.src16 && ld.cols && ld.dedup_ok;
  const int ncols = dd ? ld.D : net->N;
  *seglive_used = !dd;
  const int tpx = dd ? tiles_per_xcd((size_t)ncols * CR * CB) : 1;  // see launch_gfm
  const int nchunks = (ncols + u8_outputs(CR) - 1) / u8_outputs(CR);
  const int64_t parts = 8 / std::max<int64_t>(1, std::min<int64_t>(8, max_tiles));
  const int per_xcd = tpx * std::max(1, (int)std::min<int64_t>(net->cus, (nchunks + parts - 1) / parts));
  const dim3 grid(8 * per_xcd);
  const int rounds = (int)((max_tiles + 8 * tpx - 1) / (8 * tpx));
  const float *dict = reinterpret_cast<const float *>(CB == 1 ? net->dict : net->dict16);
  for (int r = 0; r < rounds; ++r) {
    // (two-byte codes come only from encodings, which the opt-in uniform-layer kernels never use)
    if constexpr (CB == 1) {
      if (ld.K == 32 && ld.src16 && ld.uniform) {
        hipLaunchKernelGGL((k_layer_gfm_u8<kWOne, CR, u8_rows_per_lane(CR), u8_outs_per_lane(CR), CB>), grid, dim3(256), 0, net->stream, cin, fout, net->N, ld.ell, ld.K,
                           dd ? ld.src16c : ld.src16, (const float *)nullptr, ld.w, ld.bias, net->ymax, dict, npos, masks,
                           net->seglive, r * 8 * tpx, net->spread, dd ? ld.cols : nullptr, ncols, tpx);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        continue;
      }
    } else if (ld.uniform) {
      return hipErrorInvalidValue;
    }
    if (ld.K == 32 && ld.src16 && ld.w32)
      hipLaunchKernelGGL((k_layer_gfm_u8<kWEdge, CR, u8_rows_per_lane(CR), u8_outs_per_lane(CR), CB>), grid, dim3(256), 0, net->stream, cin, fout, net->N, ld.ell,
                         ld.K, ld.src16, ld.w32, 0.0f, ld.bias, net->ymax, dict, npos, masks, net->seglive, r * 8,
                         net->spread, (const int *)nullptr, net->N, 1);
    else
      hipLaunchKernelGGL((k_layer_gfm_u8<kWEll, CR, u8_rows_per_lane(CR), u8_outs_per_lane(CR), CB>), grid, dim3(256), 0, net->stream, cin, fout, net->N, ld.ell,
                         ld.K, (const unsigned short *)nullptr, (const float *)nullptr, 0.0f, ld.bias, net->ymax, dict,
                         npos, masks, net->seglive, r * 8, net->spread, (const int *)nullptr, net->N, 1);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
hipError_t launch_gfm_u8(sdnn_net *net, const LayerDev &ld, const unsigned char *cin, float *fout, const int *npos,
                         int64_t max_tiles, unsigned *masks, bool *seglive_used) {
  return code_rows(net->bitsT) == 128 ? launch_gfm_u8_cr<128>(net, ld, cin, fout, npos, max_tiles, masks, seglive_used)
                                      : launch_gfm_u8_cr<64>(net, ld, cin, fout, npos, max_tiles, masks, seglive_used);
}
// A layer whose inputs are two-byte codes (64-row code tiles, dictionary dict16; only layers wider
// than 32768 neurons use them, and those have 64-row code tiles)
hipError_t launch_gfm_u16(sdnn_net *net, const LayerDev &ld, const unsigned char *cin, float *fout, const int *npos,
                          int64_t max_tiles, unsigned *masks, bool *seglive_used) {
  if (code_rows(net->bitsT) != 64) return hipErrorInvalidValue;
  return launch_gfm_u8_cr<64, 2>(net, ld, cin, fout, npos, max_tiles, masks, seglive_used);
}

// Rows per workgroup of k_layers_lds: at most the largest of 16, 8, 4 whose two tiles fit 128 KiB
// of LDS, halved (down to 1) while twice the workgroups still fit one per CU.
int fused_rows_max(const sdnn_net *net) {
  int b = 16;
  while (b > 4 && (size_t)2 * b * net->N * sizeof(float) > (size_t)kLdsTileBytes) b /= 2;
  return b;
}
int fused_rows(const sdnn_net *net, int64_t rows) {
  int b = fused_rows_max(net);
  while (b > 1 && 2 * ((rows + b - 1) / b) <= net->cus) b /= 2;
  return b;
}

template <int B>
hipError_t launch_layers_lds_b(sdnn_net *net, const float *yin, float *yout, int l0, const int *ids, const int *count,
                               int64_t rows, int *rownz) {
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_layers_lds<B>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kLdsTileBytes);
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_layers_lds32<B>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, kLdsTileBytes);
    if (e != hipSuccess) return e;
    configured = true;
  }
  int shift = 0;
  while ((1 << shift) < net->B * (int)sizeof(float)) ++shift;
  const size_t lds = (size_t)2 * net->N * B * sizeof(float);
  const int grid = (int)std::max<int64_t>(1, (rows + B - 1) / B);
  const LayerPtr *lp = net->lp_dev[B >= 16 ? 2 : (B == 8 ? 1 : 0)];  // the table grouped for this height
  if (net->n_edge32 == net->L) {
    // idle CUs fetch the lists ahead, where kFetchAhead layers (200 bytes per neuron) take at most 2.5 MiB of
    // the 4 MiB L2, that is up to 1092 neurons, and more layers than that follow. (1.5 MiB for the layers that
    // the other workers lag behind. Wider layers with a shorter distance have not been measured.)
    const int workers = (grid + 7) / 8 * 8;
    const bool fetch = workers + 8 <= net->cus && (size_t)net->N * 200 * kFetchAhead <= (size_t)5 << 19 &&
                       net->L - l0 > kFetchAhead;
    hipLaunchKernelGGL(k_layers_lds32<B>, dim3(fetch ? workers + 8 : grid), dim3(1024), lds, net->stream, yin, yout,
                       net->N, lp, l0, net->L, net->ymax, ids, count, net->counts, net->masks, rownz,
                       fetch ? net->misc + kPaceSlot : nullptr, fetch ? workers : grid);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_layers_lds<B>, dim3(grid), dim3(1024), lds, net->stream, yin, yout, net->N, lp, l0,
                     net->L, net->ymax, ids, count, net->counts, net->masks, shift);
  return hipGetLastError();
}

// Layers [l0, L) of at most `rows` live rows (list ids, count *count) in one launch (k_layers_lds).
hipError_t launch_layers_lds(sdnn_net *net, const float *yin, float *yout, int l0, const int *ids, const int *count,
                             int64_t rows, int *rownz) {
  switch (fused_rows(net, rows)) {
    case 16: return launch_layers_lds_b<16>(net, yin, yout, l0, ids, count, rows, rownz);
    case 8: return launch_layers_lds_b<8>(net, yin, yout, l0, ids, count, rows, rownz);
    case 4: return launch_layers_lds_b<4>(net, yin, yout, l0, ids, count, rows, rownz);
    case 2: return launch_layers_lds_b<2>(net, yin, yout, l0, ids, count, rows, rownz);
    default: return launch_layers_lds_b<1>(net, yin, yout, l0, ids, count, rows, rownz);
  }
}

// One layer of the LDS-tile path, of at most `rows` live rows.
hipError_t launch_layer(sdnn_net *net, int l, const float *yin, float *yout, const int *ids, const int *count,
                        int64_t rows, int *rownz) {
  const LayerDev &ld = net->layers[l];
  switch (net->B) {
    case 32: return launch_lds_k<32>(net, yin, yout, ld, ids, count, rows, rownz);
    case 16: return launch_lds_k<16>(net, yin, yout, ld, ids, count, rows, rownz);
    default: return launch_lds_k<8>(net, yin, yout, ld, ids, count, rows, rownz);
  }
}

// Gives up the segment streams of all layers, loaded and to come: a layer on rows leaves the liveness words of
// the layer after it as they are, which those of few-row layers of other than 32 sources on tiles must not
// be, so a network has all of its streams or none. (No run reads them: it needs every layer loaded.)
void drop_streams(sdnn_net *net) {
  for (LayerDev &ld : net->layers) {
    ld.seg = nullptr;
    ld.segdesc = nullptr;
    ld.segcol = nullptr;
  }
  for (void *q : net->streams) (void)hipFree(q);
  net->streams.clear();
  net->no_streams = true;
}

// Device memory that a load needs: where there is too little, the segment streams of earlier loads are given up.
hipError_t device_alloc(sdnn_net *net, void **p, size_t bytes) {
  hipError_t e = hipMalloc(p, bytes);
  if (e == hipSuccess || net->streams.empty()) return e;
  (void)hipGetLastError();
  drop_streams(net);
  return hipMalloc(p, bytes);
}

}  // namespace

extern "C" {

const char *sdnn_last_error(void) { return g_err.c_str(); }

sdnn_status sdnn_create(sdnn_net **out, int32_t n_neurons, int32_t n_layers, float ymax) try {
  if (!out) return fail(SDNN_EINVAL, "out is null");
  *out = nullptr;
  if (n_neurons < 1 || n_neurons > kMaxNeurons) return fail(SDNN_EINVAL, "n_neurons %d not in [1, %d]", n_neurons, kMaxNeurons);
  if (n_layers < 1 || n_layers > kMaxLayers) return fail(SDNN_EINVAL, "n_layers %d not in [1, %d]", n_layers, kMaxLayers);
  if (!std::isfinite(ymax) || !(ymax > 0.0f)) return fail(SDNN_EINVAL, "ymax must be finite and > 0");
  auto net = std::make_unique<sdnn_net>();
  net->N = n_neurons;
  net->L = n_layers;
  net->ymax = ymax;
  net->layers.resize((size_t)n_layers);
  // LDS tile of B rows x N fp32 must fit the budget with B >= 8
  if ((size_t)32 * n_neurons * sizeof(float) <= (size_t)kLdsTileBytes) { net->path = 0; net->B = 32; }
  else if ((size_t)16 * n_neurons * sizeof(float) <= (size_t)kLdsTileBytes) { net->path = 0; net->B = 16; }
  else if ((size_t)8 * n_neurons * sizeof(float) <= (size_t)kLdsTileBytes) { net->path = 0; net->B = 8; }
  else {
    // global feature-major tiles of 32 rows (128-byte segments per source); one tile per XCD per
    // launch, held in that XCD's L2 up to 16384 neurons and in the Infinity Cache beyond
    net->path = 1;
    net->B = 32;
    // layer 0 from bit tiles: 32-row tiles while their words fit 64 KiB of LDS, else 16-row tiles
    net->bitsT = (size_t)n_neurons * 4 <= 64 * 1024 ? 32 : ((size_t)n_neurons * 2 <= 128 * 1024 ? 16 : 0);
  }
  *out = net.release();
  g_err.clear();
  return SDNN_OK;
} SDNN_CATCH

int32_t sdnn_kernel_path(const sdnn_net *net) { return net ? net->path : -1; }

sdnn_status sdnn_enable_equal_value_kernels(sdnn_net *net, int32_t enable) {
  sdnn_status st = check_usable(net);
  if (st != SDNN_OK) return st;
  if (enable != 0 && enable != 1) return fail(SDNN_EINVAL, "enable must be 0 or 1");
  if (net->n_loaded > 0) return fail(SDNN_ESTATE, "layers are already loaded");
  net->equal_value_kernels = enable != 0;
  g_err.clear();
  return SDNN_OK;
}

sdnn_status sdnn_load_layers(sdnn_net *net, int32_t l0, int32_t nl, const int64_t *col_ptr, const int32_t *row_idx,
                             const float *val, const float *bias, void *hip_stream) try {
  sdnn_status st = check_usable(net);
  if (st != SDNN_OK) return st;
  if (nl < 1 || l0 < 0 || (int64_t)l0 + nl > net->L) return fail(SDNN_EINVAL, "layers [%d, %d) outside [0, %d)", l0, l0 + nl, net->L);
  if (!col_ptr || !row_idx || !val || !bias) return fail(SDNN_EINVAL, "null array");
  for (int32_t i = 0; i < nl; ++i)
    if (net->layers[(size_t)l0 + i].ell) return fail(SDNN_ESTATE, "layer %d already loaded", l0 + i);
  const int32_t N = net->N;
  for (int32_t i = 1; i < nl; ++i)
    if (col_ptr[(size_t)i * (N + 1)] != col_ptr[(size_t)(i - 1) * (N + 1) + N])
      return fail(SDNN_EINVAL, "layer %d does not start where layer %d ends", l0 + i, l0 + i - 1);
  if (col_ptr[0] < 0) return fail(SDNN_EINVAL, "negative column offset");
  // ---- validate every layer before touching the device (layers in parallel on host threads)
  std::vector<int> K((size_t)nl, 0);
  std::vector<char> uniform((size_t)nl, 0);
  std::vector<std::string> err((size_t)nl);
  parallel_for(nl, [&](int32_t i) {
    const int64_t *cp = col_ptr + (size_t)i * (N + 1);
    char buf[256];
    int kmax = 0, kmin = kMaxDegree + 1;
    bool same_w = true;
    const int64_t e0 = cp[0];
    for (int32_t j = 0; j < N; ++j) {
      const int64_t a = cp[j], b = cp[j + 1];
      if (b < a) { snprintf(buf, sizeof buf, "layer %d column %d: decreasing offsets", l0 + i, j); err[(size_t)i] = buf; return; }
      if (b - a > kMaxDegree) { snprintf(buf, sizeof buf, "layer %d column %d: %lld sources exceed %d", l0 + i, j, (long long)(b - a), kMaxDegree); err[(size_t)i] = buf; return; }
      for (int64_t e = a; e < b; ++e) {
        const int32_t k = row_idx[e];
        if (k < 0 || k >= N) { snprintf(buf, sizeof buf, "layer %d column %d: source %d out of range", l0 + i, j, k); err[(size_t)i] = buf; return; }
        if (e > a && k <= row_idx[e - 1]) { snprintf(buf, sizeof buf, "layer %d column %d: sources not strictly ascending", l0 + i, j); err[(size_t)i] = buf; return; }
        if (!std::isfinite(val[e])) { snprintf(buf, sizeof buf, "layer %d column %d: non-finite weight", l0 + i, j); err[(size_t)i] = buf; return; }
        same_w = same_w && std::memcmp(&val[e], &val[e0], sizeof(float)) == 0;
      }
      kmax = std::max<int>(kmax, (int)(b - a));
      kmin = std::min<int>(kmin, (int)(b - a));
    }
    bool same_b = true;
    for (int32_t j = 0; j < N; ++j) {
      if (!std::isfinite(bias[(size_t)i * N + j])) { snprintf(buf, sizeof buf, "layer %d: non-finite bias", l0 + i); err[(size_t)i] = buf; return; }
      same_b = same_b && std::memcmp(&bias[(size_t)i * N + j], &bias[(size_t)i * N], sizeof(float)) == 0;
    }
    K[(size_t)i] = std::max(kmax, 1);
    // the specialisations that read one weight and one bias per layer are opt-in: by default every
    // layer reads each edge's weight and each neuron's bias from memory, whatever their values
    uniform[(size_t)i] = net->equal_value_kernels && kmax > 0 && kmin == kmax && same_w && same_b;
  });
  for (int32_t i = 0; i < nl; ++i)
    if (!err[(size_t)i].empty()) return fail(SDNN_EINVAL, "%s", err[(size_t)i].c_str());
  // ---- duplicate columns (uniform layers with 32 sources per column): columns
  // with the same source list have the same output, so reps[i][j] = the smallest column with j's
  // list (empty: no duplicates). Grouping uses the sources as given; equal lists stay equal once
  // mapped (below). With the Kronecker-expanded networks of Sec. III every 16 columns of a block
  // share their list.
  std::vector<std::vector<int32_t>> reps((size_t)nl);
  parallel_for(nl, [&](int32_t i) {
    if (N > 65536 || !uniform[(size_t)i] || K[(size_t)i] != 32) return;
    const int64_t *cp = col_ptr + (size_t)i * (N + 1);
    std::unordered_map<uint64_t, std::vector<int32_t>> seen;
    seen.reserve((size_t)N);
    std::vector<int32_t> r((size_t)N);
    int32_t distinct = 0;
    for (int32_t j = 0; j < N; ++j) {
      const int32_t *src = row_idx + cp[j];
      uint64_t h = 0x9E3779B97F4A7C15ull;
      for (int k = 0; k < 32; ++k) {
        h ^= (uint32_t)src[k] + 0x9E3779B97F4A7C15ull + (h << 6) + (h >> 2);
        h *= 0xBF58476D1CE4E5B9ull;
      }
      std::vector<int32_t> &cand = seen[h];
      int32_t found = -1;
      for (int32_t c : cand)
        if (std::memcmp(row_idx + cp[c], src, 32 * sizeof(int32_t)) == 0) { found = c; break; }
      if (found < 0) {
        cand.push_back(j);
        found = j;
        ++distinct;
      }
      r[(size_t)j] = found;
    }
    if (distinct < N) reps[(size_t)i] = std::move(r);
  });
  // ---- a layer loaded right after one with duplicates reads that layer's representatives only:
  // its sources are mapped through them (values are equal), and the earlier layer may then skip
  // its duplicate columns. mapped[i] holds layer i's mapped sources (empty: as given).
  std::vector<std::vector<int32_t>> mapped((size_t)nl);
  std::vector<char> maps_prev((size_t)nl, 0);  // layer l0 + i's sources go through layer l0 + i - 1's reps
  {
    const std::vector<int32_t> *prev = (net->prev_rep_layer == l0 - 1 && !net->prev_rep.empty()) ? &net->prev_rep : nullptr;
    for (int32_t i = 0; i < nl; ++i) {
      if (prev) {
        const int64_t *cp = col_ptr + (size_t)i * (N + 1);
        const int64_t e0 = cp[0], e1 = cp[N];
        std::vector<int32_t> &m = mapped[(size_t)i];
        m.resize((size_t)(e1 - e0));
        for (int64_t e = e0; e < e1; ++e) m[(size_t)(e - e0)] = (*prev)[(size_t)row_idx[e]];
        maps_prev[(size_t)i] = 1;
      }
      prev = reps[(size_t)i].empty() ? nullptr : &reps[(size_t)i];
    }
  }
  // source of entry e of layer i (absolute index into row_idx)
  auto src_at = [&](int32_t i, int64_t e) -> int32_t {
    const std::vector<int32_t> &m = mapped[(size_t)i];
    return m.empty() ? row_idx[e] : m[(size_t)(e - col_ptr[(size_t)i * (N + 1)])];
  };
  // ---- pack: slot-major ELL [K][N] of (byte offset of source row in the tile, weight bits)
  const int stride = net->B * (int)sizeof(float);
  std::vector<size_t> layer_off((size_t)nl + 1, 0);
  for (int32_t i = 0; i < nl; ++i) layer_off[(size_t)i + 1] = layer_off[(size_t)i] + (size_t)N * K[(size_t)i];
  const size_t ell_words = layer_off[(size_t)nl];
  const size_t ell_bytes = align_up(ell_words * sizeof(int2), 256);
  const size_t bias_bytes = (size_t)nl * N * sizeof(float);
  // and, for widths of k_layer_seg, the description of its streams: [nl][seg_dwords] int2, then [nl][seg_cwords]
  // columns with biases and [nl][seg_cwords] cuts (the device writes the streams from the ELL and these)
  const bool seg = net->path == 1 && N <= kSegMaxNeurons && !net->equal_value_kernels;
  const size_t seg_dwords = (size_t)seg_segments(N) * seg_blocks(N), seg_cwords = (size_t)seg_positions(N);
  const size_t seg_colb = align_up((size_t)nl * seg_dwords * sizeof(int2), 256);
  const size_t seg_cut = seg_colb + (size_t)nl * seg_cwords * sizeof(uint2);
  std::vector<char> hseg(seg ? seg_cut + (size_t)nl * seg_cwords * sizeof(uint32_t) : 0);
  std::vector<size_t> groups((size_t)nl, 0);
  std::vector<int2> host_ell(ell_words);
  parallel_for(nl, [&](int32_t i) {
    const int64_t *cp = col_ptr + (size_t)i * (N + 1);
    const int Ki = K[(size_t)i];
    int2 *base = host_ell.data() + layer_off[(size_t)i];
    for (int32_t j = 0; j < N; ++j) {
      int s = 0;
      for (int64_t e = cp[j]; e < cp[j + 1]; ++e, ++s) {
        int wbits;
        std::memcpy(&wbits, &val[e], sizeof(int));
        base[(size_t)s * N + j] = make_int2(src_at(i, e) * stride, wbits);
      }
      for (; s < Ki; ++s) base[(size_t)s * N + j] = make_int2(0, 0);
    }
    if (seg)
      groups[(size_t)i] = seg_order(
          N, [&](int j, int t) { return row_idx[cp[j] + t]; }, [&](int j) { return (int)(cp[j + 1] - cp[j]); },
          bias + (size_t)i * N, reinterpret_cast<int2 *>(hseg.data()) + (size_t)i * seg_dwords,
          reinterpret_cast<uint2 *>(hseg.data() + seg_colb) + (size_t)i * seg_cwords,
          reinterpret_cast<uint32_t *>(hseg.data() + seg_cut) + (size_t)i * seg_cwords);
  });
  // ---- device copy
  if (net->device < 0) {
    HIP_OR_POISON(net, hipGetDevice(&net->device));
    HIP_OR_POISON(net, hipDeviceGetAttribute(&net->cus, hipDeviceAttributeMultiprocessorCount, net->device));
    // the host-side objects sdnn_infer uses (read-back events, pinned read-back slots, the progress
    // word in coherent host memory), created once here so that the timed calls allocate nothing
    net->events.resize(4);
    for (auto &ev : net->events) HIP_OR_POISON(net, hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    HIP_OR_POISON(net, hipHostMalloc(reinterpret_cast<void **>(&net->pinned), 8 * sizeof(int32_t), hipHostMallocDefault));
    HIP_OR_POISON(net, hipHostMalloc(reinterpret_cast<void **>(&net->progress), sizeof(unsigned long long),
                                     hipHostMallocCoherent));
    *net->progress = 0ull;
    HIP_OR_POISON(net, hipHostGetDevicePointer(reinterpret_cast<void **>(&net->progress_dev), net->progress, 0));
    HIP_OR_POISON(net, hipHostMalloc(reinterpret_cast<void **>(&net->notify), sizeof(unsigned long long),
                                     hipHostMallocCoherent));
    *net->notify = 0ull;
    HIP_OR_POISON(net, hipHostGetDevicePointer(reinterpret_cast<void **>(&net->notify_dev), net->notify, 0));
    HIP_OR_POISON(net, hipHostMalloc(reinterpret_cast<void **>(&net->host_out), sizeof(HostOut), hipHostMallocCoherent));
    std::memset(net->host_out, 0, sizeof(HostOut));
    HIP_OR_POISON(net, hipHostGetDevicePointer(reinterpret_cast<void **>(&net->host_out_dev), net->host_out, 0));
    // the device address of the static workspace on this device (sdnn_infer_static)
    void *sw = nullptr;
    st = scratch_address(net->device, &sw);
    if (st != SDNN_OK) return st;
  } else {
    int dev = -1;
    HIP_OR_POISON(net, hipGetDevice(&dev));
    if (dev != net->device) return fail(SDNN_EINVAL, "current device %d differs from the handle's device %d", dev, net->device);
  }
  char *mem = nullptr;
  hipError_t e = device_alloc(net, reinterpret_cast<void **>(&mem), ell_bytes + bias_bytes);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return fail(SDNN_ENOMEM, "hipMalloc of %zu bytes failed: %s", ell_bytes + bias_bytes, hipGetErrorString(e));
  }
  net->allocations.push_back(mem);
  hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
  if (l0 == 0 && net->bitsT > 0 && K[0] <= 32) {
    // layer 0 on the bit route: its ELL again, with source offsets in bit-tile words (k * 128 bytes
    // in a 32-row fp32 tile becomes k * sizeof(word))
    const size_t n0 = (size_t)N * K[0];
    const int wsz = net->bitsT == 32 ? 4 : 2;
    std::vector<int2> hw0(n0);
    for (size_t q = 0; q < n0; ++q) hw0[q] = make_int2(host_ell[q].x / stride * wsz, host_ell[q].y);
    char *m0 = nullptr;
    e = device_alloc(net, reinterpret_cast<void **>(&m0), std::max<size_t>(n0, 1) * sizeof(int2));
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return fail(SDNN_ENOMEM, "hipMalloc of %zu bytes failed: %s", n0 * sizeof(int2), hipGetErrorString(e));
    }
    net->allocations.push_back(m0);
    HIP_OR_POISON(net, hipMemcpy(m0, hw0.data(), n0 * sizeof(int2), hipMemcpyHostToDevice));
    net->layers[0].ellw = reinterpret_cast<const int2 *>(m0);
  }
  // (nothing is allocated on the host while these copies run)
  HIP_OR_POISON(net, hipMemcpyAsync(mem, host_ell.data(), ell_words * sizeof(int2), hipMemcpyHostToDevice, s));
  HIP_OR_POISON(net, hipMemcpyAsync(mem + ell_bytes, bias, bias_bytes, hipMemcpyHostToDevice, s));
  HIP_OR_POISON(net, hipStreamSynchronize(s));
  for (int32_t i = 0; i < nl; ++i) {
    LayerDev &ld = net->layers[(size_t)l0 + i];
    ld.ell = reinterpret_cast<const int2 *>(mem) + layer_off[(size_t)i];
    ld.bias = reinterpret_cast<const float *>(mem + ell_bytes) + (size_t)i * N;
    ld.K = K[(size_t)i];
    ld.uniform = uniform[(size_t)i] != 0;
    if (ld.uniform) {
      ld.w = val[col_ptr[(size_t)i * (N + 1)]];
      ld.b = bias[(size_t)i * N];
    }
  }
  if (net->path == 1 && N <= 65536) {
    // layers with 32 sources per column: 16-bit source lists, [K][N] like the ELL, and unless the
    // layer is uniform its weights [K][N] fp32 (6 bytes per edge for the large-layer kernels)
    std::vector<int32_t> sel;
    for (int32_t i = 0; i < nl; ++i)
      if (net->layers[(size_t)l0 + i].K == 32) sel.push_back(i);
    if (!sel.empty()) {
      const size_t per = (size_t)32 * N;
      std::vector<size_t> woff(sel.size() + 1, 0);  // weight arrays of the non-uniform layers
      for (size_t q = 0; q < sel.size(); ++q)
        woff[q + 1] = woff[q] + (net->layers[(size_t)l0 + sel[q]].uniform ? 0 : per);
      std::vector<uint16_t> hs(per * sel.size());
      std::vector<float> hw(woff[sel.size()]);
      parallel_for((int32_t)sel.size(), [&](int32_t q) {
        const int64_t *cp = col_ptr + (size_t)sel[(size_t)q] * (N + 1);
        uint16_t *dst = hs.data() + per * (size_t)q;
        const bool weights = woff[(size_t)q + 1] > woff[(size_t)q];
        float *wd = hw.data() + woff[(size_t)q];
        for (int32_t j = 0; j < N; ++j) {
          // a column with fewer than 32 sources is padded with (source 0, weight +0), which adds
          // fma(y, +0, acc) = acc exactly, as in the ELL
          const int deg = (int)(cp[j + 1] - cp[j]);
          for (int sl = 0; sl < 32; ++sl) {
            dst[(size_t)sl * N + j] = sl < deg ? (uint16_t)src_at(sel[(size_t)q], cp[j] + sl) : (uint16_t)0;
            if (weights) wd[(size_t)sl * N + j] = sl < deg ? val[cp[j] + sl] : 0.0f;
          }
        }
      });
      const size_t sbytes = align_up(hs.size() * sizeof(uint16_t), 256);
      const size_t wbytes = hw.size() * sizeof(float);
      char *ms = nullptr;
      e = device_alloc(net, reinterpret_cast<void **>(&ms), sbytes + wbytes);
      if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(SDNN_ENOMEM, "hipMalloc of %zu bytes failed: %s", sbytes + wbytes, hipGetErrorString(e));
      }
      net->allocations.push_back(ms);
      HIP_OR_POISON(net, hipMemcpyAsync(ms, hs.data(), hs.size() * sizeof(uint16_t), hipMemcpyHostToDevice, s));
      if (wbytes) HIP_OR_POISON(net, hipMemcpyAsync(ms + sbytes, hw.data(), wbytes, hipMemcpyHostToDevice, s));
      HIP_OR_POISON(net, hipStreamSynchronize(s));
      for (size_t q = 0; q < sel.size(); ++q) {
        LayerDev &ld = net->layers[(size_t)l0 + sel[q]];
        ld.src16 = reinterpret_cast<const unsigned short *>(ms) + per * q;
        if (!ld.uniform) ld.w32 = reinterpret_cast<const float *>(ms + sbytes) + woff[q];
      }
    }
  }
  {
    // 16-bit source indices in groups of 8 per output ([4][N][8] u16, one 16-byte load per group):
    // every layer with 32 sources per column on widths staged in LDS, with its weights grouped the
    // by four ([8][N][4] fp32) unless it is uniform; and layer 0 of a uniform network of any width
    // (for the counting kernel). Columns with fewer than 32 sources are padded with (source 0,
    // weight +0), a no-op term as in the ELL.
    std::vector<int32_t> sel;
    for (int32_t i = 0; i < nl; ++i) {
      const LayerDev &ld = net->layers[(size_t)l0 + i];
      if (ld.K == 32 && N <= 65536 && (net->path == 0 || (ld.uniform && l0 + i == 0))) sel.push_back(i);
    }
    if (!sel.empty()) {
      const size_t per = (size_t)32 * N;
      std::vector<size_t> woff(sel.size() + 1, 0);
      for (size_t q = 0; q < sel.size(); ++q)
        woff[q + 1] = woff[q] + (net->layers[(size_t)l0 + sel[q]].uniform ? 0 : per);
      std::vector<uint16_t> h16(per * sel.size());
      std::vector<float> hw(woff[sel.size()]);
      parallel_for((int32_t)sel.size(), [&](int32_t q) {
        const int64_t *cp = col_ptr + (size_t)sel[(size_t)q] * (N + 1);
        uint16_t *dst = h16.data() + per * (size_t)q;
        const bool weights = woff[(size_t)q + 1] > woff[(size_t)q];
        float *wd = hw.data() + woff[(size_t)q];
        for (int32_t j = 0; j < N; ++j) {
          const int deg = (int)(cp[j + 1] - cp[j]);
          for (int sl = 0; sl < 32; ++sl) {
            dst[((size_t)(sl / 8) * N + j) * 8 + sl % 8] =
                sl < deg ? (uint16_t)src_at(sel[(size_t)q], cp[j] + sl) : (uint16_t)0;
            if (weights) wd[((size_t)(sl / 4) * N + j) * 4 + sl % 4] = sl < deg ? val[cp[j] + sl] : 0.0f;
          }
        }
      });
      const size_t sbytes = align_up(h16.size() * sizeof(uint16_t), 256);
      const size_t wbytes = hw.size() * sizeof(float);
      char *m16 = nullptr;
      e = device_alloc(net, reinterpret_cast<void **>(&m16), sbytes + wbytes);
      if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(SDNN_ENOMEM, "hipMalloc of %zu bytes failed: %s", sbytes + wbytes, hipGetErrorString(e));
      }
      net->allocations.push_back(m16);
      HIP_OR_POISON(net, hipMemcpy(m16, h16.data(), h16.size() * sizeof(uint16_t), hipMemcpyHostToDevice));
      if (wbytes) HIP_OR_POISON(net, hipMemcpy(m16 + sbytes, hw.data(), wbytes, hipMemcpyHostToDevice));
      for (size_t q = 0; q < sel.size(); ++q) {
        LayerDev &ld = net->layers[(size_t)l0 + sel[q]];
        ld.ell16 = reinterpret_cast<const uint4 *>(m16) + (per / 8) * q;
        if (!ld.uniform) ld.w8 = reinterpret_cast<const float *>(m16 + sbytes) + woff[q];
      }
      // LDS row placements of the first layers on widths staged in LDS (bank_placement): per layer
      // place [N] u16 and the placed sources [4][N][8] u16
      std::vector<int32_t> psel;
      for (size_t q = 0; q < sel.size(); ++q)
        if (net->path == 0 && l0 + sel[q] < kPlacedLayers) psel.push_back((int32_t)q);
      if (!psel.empty()) {
        const size_t pbytes = align_up((size_t)N * sizeof(uint16_t), 256);
        const size_t per_layer = pbytes + per * sizeof(uint16_t);
        std::vector<uint16_t> hp(per_layer / sizeof(uint16_t) * psel.size());
        parallel_for((int32_t)psel.size(), [&](int32_t i) {
          const size_t q = (size_t)psel[(size_t)i];
          const uint16_t *src = h16.data() + per * q;
          const std::vector<uint16_t> place =
              bank_placement(src, N, net->B, 0x5DB1ull * (uint64_t)(l0 + sel[q] + 1), 25 * N);
          uint16_t *out = hp.data() + per_layer / sizeof(uint16_t) * (size_t)i;
          std::copy(place.begin(), place.end(), out);
          uint16_t *po = out + pbytes / sizeof(uint16_t);
          for (size_t t = 0; t < per; ++t) po[t] = place[src[t]];
        });
        char *mp = nullptr;
        e = device_alloc(net, reinterpret_cast<void **>(&mp), hp.size() * sizeof(uint16_t));
        if (e != hipSuccess) {
          (void)hipGetLastError();
          return fail(SDNN_ENOMEM, "hipMalloc of %zu bytes failed: %s", hp.size() * sizeof(uint16_t),
                      hipGetErrorString(e));
        }
        net->allocations.push_back(mp);
        HIP_OR_POISON(net, hipMemcpy(mp, hp.data(), hp.size() * sizeof(uint16_t), hipMemcpyHostToDevice));
        for (size_t i = 0; i < psel.size(); ++i) {
          LayerDev &ld = net->layers[(size_t)l0 + sel[(size_t)psel[i]]];
          ld.place = reinterpret_cast<const unsigned short *>(mp + per_layer * i);
          ld.pell16 = reinterpret_cast<const uint4 *>(mp + per_layer * i + pbytes);
        }
      }
    }
  }
  {
    // distinct columns: the representatives and their (mapped) source lists, as [32][D] u16 for the
    // global-tile kernels and as [4][D][8] u16 for the LDS-tile and counting kernels
    std::vector<int32_t> sel;
    for (int32_t i = 0; i < nl; ++i) {
      const LayerDev &ld = net->layers[(size_t)l0 + i];
      if (!reps[(size_t)i].empty() && (ld.src16 || ld.ell16)) sel.push_back(i);
    }
    if (!sel.empty()) {
      std::vector<size_t> off(sel.size() + 1, 0);  // in columns
      std::vector<std::vector<int32_t>> cols(sel.size());
      for (size_t q = 0; q < sel.size(); ++q) {
        const std::vector<int32_t> &r = reps[(size_t)sel[q]];
        for (int32_t j = 0; j < N; ++j)
          if (r[(size_t)j] == j) cols[q].push_back(j);
        off[q + 1] = off[q] + cols[q].size();
      }
      const size_t tot = off[sel.size()];
      std::vector<int32_t> hc(tot);
      std::vector<uint16_t> hs((size_t)32 * tot), hg((size_t)32 * tot);
      parallel_for((int32_t)sel.size(), [&](int32_t q) {
        const int64_t *cp = col_ptr + (size_t)sel[(size_t)q] * (N + 1);
        const size_t D = cols[(size_t)q].size();
        uint16_t *ds = hs.data() + (size_t)32 * off[(size_t)q];
        uint16_t *dg = hg.data() + (size_t)32 * off[(size_t)q];
        for (size_t p = 0; p < D; ++p) {
          const int32_t j = cols[(size_t)q][p];
          hc[off[(size_t)q] + p] = j;
          for (int sl = 0; sl < 32; ++sl) {
            const uint16_t v = (uint16_t)src_at(sel[(size_t)q], cp[j] + sl);
            ds[(size_t)sl * D + p] = v;
            dg[((size_t)(sl / 8) * D + p) * 8 + sl % 8] = v;
          }
        }
      });
      const size_t cbytes = align_up(tot * sizeof(int32_t), 256);
      const size_t sbytes = align_up(hs.size() * sizeof(uint16_t), 256);
      char *mc = nullptr;
      e = device_alloc(net, reinterpret_cast<void **>(&mc), cbytes + 2 * sbytes);
      if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(SDNN_ENOMEM, "hipMalloc of %zu bytes failed: %s", cbytes + 2 * sbytes, hipGetErrorString(e));
      }
      net->allocations.push_back(mc);
      HIP_OR_POISON(net, hipMemcpy(mc, hc.data(), tot * sizeof(int32_t), hipMemcpyHostToDevice));
      HIP_OR_POISON(net, hipMemcpy(mc + cbytes, hs.data(), hs.size() * sizeof(uint16_t), hipMemcpyHostToDevice));
      HIP_OR_POISON(net, hipMemcpy(mc + cbytes + sbytes, hg.data(), hg.size() * sizeof(uint16_t), hipMemcpyHostToDevice));
      for (size_t q = 0; q < sel.size(); ++q) {
        LayerDev &ld = net->layers[(size_t)l0 + sel[q]];
        ld.cols = reinterpret_cast<const int *>(mc) + off[q];
        ld.src16c = ld.src16 ? reinterpret_cast<const unsigned short *>(mc + cbytes) + (size_t)32 * off[q] : nullptr;
        ld.ell16c = ld.ell16 ? reinterpret_cast<const uint4 *>(mc + cbytes + sbytes) + (size_t)4 * off[q] : nullptr;
        ld.D = (int)cols[q].size();
      }
    }
    // layer 0: the lists in the counting kernel's order (words of 4 bytes on the LDS-tile path, of
    // bitsT / 8 bytes on the global-tile path)
    if (l0 == 0 && net->layers[0].ell16 && net->layers[0].w > 0.0f) {
      LayerDev &ld = net->layers[0];
      const int wbytes = net->path == 0 ? 4 : std::max(net->bitsT, 16) / 8;
      const int64_t *cp = col_ptr;
      std::vector<int32_t> c0;
      if (ld.cols)
        for (int32_t j = 0; j < N; ++j)
          if (reps[0][(size_t)j] == j) c0.push_back(j);
      std::vector<uint16_t> full((size_t)32 * N), part((size_t)32 * c0.size());
      for (int32_t j = 0; j < N; ++j)
        for (int sl = 0; sl < 32; ++sl) full[((size_t)(sl / 8) * N + j) * 8 + sl % 8] = (uint16_t)src_at(0, cp[j] + sl);
      const int D0 = (int)c0.size();
      for (int p = 0; p < D0; ++p)
        for (int sl = 0; sl < 32; ++sl)
          part[((size_t)(sl / 8) * D0 + p) * 8 + sl % 8] = (uint16_t)src_at(0, cp[c0[(size_t)p]] + sl);
      const std::vector<uint16_t> bf = bank_balanced_lists(full.data(), N, wbytes);
      const std::vector<uint16_t> bp = D0 ? bank_balanced_lists(part.data(), D0, wbytes) : std::vector<uint16_t>();
      const size_t fb = align_up(bf.size() * sizeof(uint16_t), 256);
      char *mb = nullptr;
      e = device_alloc(net, reinterpret_cast<void **>(&mb), fb + bp.size() * sizeof(uint16_t));
      if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(SDNN_ENOMEM, "hipMalloc of %zu bytes failed: %s", fb + bp.size() * sizeof(uint16_t), hipGetErrorString(e));
      }
      net->allocations.push_back(mb);
      HIP_OR_POISON(net, hipMemcpy(mb, bf.data(), bf.size() * sizeof(uint16_t), hipMemcpyHostToDevice));
      if (D0) HIP_OR_POISON(net, hipMemcpy(mb + fb, bp.data(), bp.size() * sizeof(uint16_t), hipMemcpyHostToDevice));
      ld.ell16s = reinterpret_cast<const uint4 *>(mb);
      ld.ell16cs = D0 ? reinterpret_cast<const uint4 *>(mb + fb) : nullptr;
    }
    // widths staged in LDS: positions in groups for the fused kernel, over all columns and over the
    // distinct columns
    if (net->path == 0) {
      // one order per fused tile-height class the width allows (4 << c rows)
      int nclass = 1;
      while (nclass < 3 && (4 << nclass) <= fused_rows_max(net)) ++nclass;
      std::vector<int32_t> gsel;
      for (int32_t i = 0; i < nl; ++i)
        if (net->layers[(size_t)l0 + i].ell16) gsel.push_back(i);
      const size_t ng = gsel.size() * (size_t)nclass;
      // u = (q * nclass + c) * 2 + v: layer gsel[q], class c, v = 0 all columns / 1 distinct ones
      std::vector<std::vector<int32_t>> gcol(2 * ng);
      std::vector<std::vector<uint16_t>> gl(2 * ng);    // their [4][D][8] lists
      std::vector<std::vector<float>> gw(2 * ng);       // and weights (layers with w8)
      parallel_for((int32_t)(2 * ng), [&](int32_t u) {
        const int32_t i = gsel[(size_t)u / 2 / (size_t)nclass];
        const int cls = (u / 2) % nclass;
        const LayerDev &ld = net->layers[(size_t)l0 + i];
        std::vector<int32_t> pos;
        if (u % 2 == 0) {
          pos.resize((size_t)N);
          for (int32_t j = 0; j < N; ++j) pos[(size_t)j] = j;
        } else if (ld.cols) {
          for (int32_t j = 0; j < N; ++j)
            if (reps[(size_t)i][(size_t)j] == j) pos.push_back(j);
        }
        if (pos.empty()) return;
        const int64_t *cp = col_ptr + (size_t)i * (N + 1);
        const int D = (int)pos.size();
        const bool weights = ld.w8 != nullptr;
        // sources (and weights) by position; short columns padded with (0, +0) as in ell16
        std::vector<uint16_t> lists((size_t)D * 32);
        std::vector<float> wl(weights ? (size_t)D * 32 : 0);
        for (int p = 0; p < D; ++p) {
          const int32_t j = pos[(size_t)p];
          const int deg = (int)(cp[j + 1] - cp[j]);
          for (int sl = 0; sl < 32; ++sl) {
            lists[(size_t)p * 32 + sl] = sl < deg ? (uint16_t)src_at(i, cp[j] + sl) : (uint16_t)0;
            if (weights) wl[(size_t)p * 32 + sl] = sl < deg ? val[cp[j] + sl] : 0.0f;
          }
        }
        const std::vector<int32_t> ord = conflict_grouped_order(lists, D, 16 >> cls);
        std::vector<int32_t> &gc = gcol[(size_t)u];
        std::vector<uint16_t> &g16 = gl[(size_t)u];
        std::vector<float> &g32 = gw[(size_t)u];
        gc.resize((size_t)D);
        g16.resize((size_t)D * 32);
        if (weights) g32.resize((size_t)D * 32);
        for (int p = 0; p < D; ++p) {
          const int32_t q = ord[(size_t)p];
          gc[(size_t)p] = pos[(size_t)q];
          for (int sl = 0; sl < 32; ++sl) {
            g16[((size_t)(sl / 8) * D + p) * 8 + sl % 8] = lists[(size_t)q * 32 + sl];
            if (weights) g32[((size_t)(sl / 4) * D + p) * 4 + sl % 4] = wl[(size_t)q * 32 + sl];
          }
        }
      });
      size_t bytes = 0;
      std::vector<size_t> co(2 * ng), lo(2 * ng), wo(2 * ng);
      for (size_t u = 0; u < 2 * ng; ++u) {
        co[u] = bytes;
        bytes += align_up(gcol[u].size() * sizeof(int32_t), 256);
        lo[u] = bytes;
        bytes += align_up(gl[u].size() * sizeof(uint16_t), 256);
        wo[u] = bytes;
        bytes += align_up(gw[u].size() * sizeof(float), 256);
      }
      if (bytes) {
        char *mg = nullptr;
        e = device_alloc(net, reinterpret_cast<void **>(&mg), bytes);
        if (e != hipSuccess) {
          (void)hipGetLastError();
          return fail(SDNN_ENOMEM, "hipMalloc of %zu bytes failed: %s", bytes, hipGetErrorString(e));
        }
        net->allocations.push_back(mg);
        for (size_t u = 0; u < 2 * ng; ++u) {
          if (gcol[u].empty()) continue;
          HIP_OR_POISON(net, hipMemcpy(mg + co[u], gcol[u].data(), gcol[u].size() * sizeof(int32_t), hipMemcpyHostToDevice));
          HIP_OR_POISON(net, hipMemcpy(mg + lo[u], gl[u].data(), gl[u].size() * sizeof(uint16_t), hipMemcpyHostToDevice));
          if (!gw[u].empty())
            HIP_OR_POISON(net, hipMemcpy(mg + wo[u], gw[u].data(), gw[u].size() * sizeof(float), hipMemcpyHostToDevice));
          LayerDev &ld = net->layers[(size_t)l0 + gsel[u / 2 / (size_t)nclass]];
          const int cls = (int)((u / 2) % (size_t)nclass);
          const int *gc = reinterpret_cast<const int *>(mg + co[u]);
          const uint4 *g16 = reinterpret_cast<const uint4 *>(mg + lo[u]);
          if (u % 2 == 0) {
            ld.gcols[cls] = gc;
            ld.gell16[cls] = g16;
            if (!gw[u].empty()) ld.gw8[cls] = reinterpret_cast<const float *>(mg + wo[u]);
          }
          else { ld.gcolsc[cls] = gc; ld.gell16c[cls] = g16; }
        }
      }
    }
    // a layer whose successor reads its representatives only may skip its duplicates; so may the
    // last layer (the final rows are expanded through its representatives)
    for (int32_t i = 0; i < nl; ++i) {
      if (maps_prev[(size_t)i]) net->layers[(size_t)l0 + i - 1].dedup_ok = true;
      if (l0 + i == net->L - 1 && !reps[(size_t)i].empty()) {
        net->layers[(size_t)l0 + i].dedup_ok = true;
        net->last_rep = reps[(size_t)i];
      }
    }
    net->prev_rep = std::move(reps[(size_t)nl - 1]);
    net->prev_rep_layer = net->prev_rep.empty() ? -1 : l0 + nl - 1;
  }
  // the device tables of layers (for launches that run several layers), one per tile-height class
  if (!net->lp_dev[0]) {
    LayerPtr *t = nullptr;
    e = device_alloc(net, reinterpret_cast<void **>(&t), (size_t)3 * net->L * sizeof(LayerPtr));
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return fail(SDNN_ENOMEM, "hipMalloc of the layer table failed: %s", hipGetErrorString(e));
    }
    net->allocations.push_back(t);
    for (int c = 0; c < 3; ++c) net->lp_dev[c] = t + (size_t)c * net->L;
  }
  {
    // from layer l0 - 1 when this load let it skip its duplicate columns
    const int32_t t0 = (l0 > 0 && net->layers[(size_t)l0 - 1].dedup_ok) ? l0 - 1 : l0;
    std::vector<LayerPtr> hp((size_t)(l0 + nl - t0));
    for (int c = 0; c < 3; ++c) {
      for (int32_t l = t0; l < l0 + nl; ++l) {
        const LayerDev &ld = net->layers[(size_t)l];
        const bool dd = ld.ell16 && ld.ell16c && ld.cols && ld.dedup_ok;
        // the fused kernel reads the positions in their grouped order where there is one
        const uint4 *g16 = dd ? ld.gell16c[c] : ld.gell16[c];
        const uint4 *e16 = g16 ? g16 : (dd ? ld.ell16c : ld.ell16);
        const int *cl = g16 ? (dd ? ld.gcolsc[c] : ld.gcols[c]) : (dd ? ld.cols : nullptr);
        // per-edge weights in the same grouping as the sources (null for a uniform layer)
        const float *w8 = ld.w8 ? (g16 ? ld.gw8[c] : ld.w8) : nullptr;
        hp[(size_t)(l - t0)] = LayerPtr{ld.ell, e16, w8, ld.bias, cl, ld.w, ld.K, dd ? ld.D : N};
      }
      HIP_OR_POISON(net, hipMemcpy(net->lp_dev[c] + t0, hp.data(), hp.size() * sizeof(LayerPtr), hipMemcpyHostToDevice));
    }
  }
  if (seg && !net->no_streams) {
    // the streams of k_layer_seg, last, because the network runs without them where memory does not suffice
    // (one more group after each layer's: the kernel loads one ahead)
    std::vector<size_t> off((size_t)nl + 1, 0);
    for (int32_t i = 0; i < nl; ++i) off[(size_t)i + 1] = off[(size_t)i] + groups[(size_t)i] + 1;
    const size_t gbytes = off[(size_t)nl] * kSegGroupWords * sizeof(uint4);
    net->streams.reserve(net->streams.size() + 1);
    char *mg = nullptr;
    if (hipMalloc(reinterpret_cast<void **>(&mg), gbytes + hseg.size()) != hipSuccess) {
      (void)hipGetLastError();
      drop_streams(net);
    } else {
      net->streams.push_back(mg);
      HIP_OR_POISON(net, hipMemcpyAsync(mg + gbytes, hseg.data(), hseg.size(), hipMemcpyHostToDevice, s));
      for (int32_t i = 0; i < nl; ++i) {
        LayerDev &ld = net->layers[(size_t)l0 + i];
        ld.seg = reinterpret_cast<const uint4 *>(mg) + off[(size_t)i] * kSegGroupWords;
        ld.segdesc = reinterpret_cast<const int2 *>(mg + gbytes) + (size_t)i * seg_dwords;
        ld.segcol = reinterpret_cast<const uint2 *>(mg + gbytes + seg_colb) + (size_t)i * seg_cwords;
        hipLaunchKernelGGL(k_pack_seg, dim3(seg_blocks(N)), dim3(256), 0, s, ld.ell, N, seg_segments(N), stride,
                           ld.segdesc, ld.segcol,
                           reinterpret_cast<const unsigned *>(mg + gbytes + seg_cut) + (size_t)i * seg_cwords,
                           seg_blocks(N), reinterpret_cast<uint4 *>(mg) + off[(size_t)i] * kSegGroupWords);
        HIP_OR_POISON(net, hipGetLastError());
      }
      HIP_OR_POISON(net, hipStreamSynchronize(s));
    }
  }
  for (int32_t i = 0; i < nl; ++i) {
    const LayerDev &ld = net->layers[(size_t)l0 + i];
    net->n_edge32 += ld.ell16 && ld.w8 && ld.gell16[0] && ld.gcols[0] && ld.gw8[0] && !ld.cols;
  }
  net->n_loaded += nl;
  g_err.clear();
  return SDNN_OK;
} SDNN_CATCH

size_t sdnn_workspace_bytes(const sdnn_net *net, int64_t n_rows) {
  if (!net || n_rows < 0) return 0;
  return layout_for(net, n_rows).total;
}

namespace {

// Read-back ring for the live count: every kPollEvery layers the count is copied to pinned host
// memory behind an event; the host checks it two chunks later, so the stream never drains while
// the host waits.
struct PollRing {
  int slot[4], bound[4], n = 0, head = 0, next = 0;
};

// After layer l (every kPollEvery layers), enqueue a poll of counts[idx], a live count known once
// layer l has finished, and consume polls that are two chunks old. *live_bound receives the
// smallest count seen.
hipError_t poll_step(sdnn_net *net, PollRing &ring, int32_t l, int32_t idx, int64_t *live_bound) {
  hipStream_t s = net->stream;
  if ((l + 1) % kPollEvery != 0 || l + 1 >= net->L) return hipSuccess;
  const int slot = ring.next;
  ring.next = (ring.next + 1) % 4;
  hipError_t e = hipMemcpyAsync(net->pinned + slot, net->counts + idx, sizeof(int32_t), hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return e;
  e = hipEventRecord(net->events[(size_t)slot], s);
  if (e != hipSuccess) return e;
  ring.slot[(ring.head + ring.n) % 4] = slot;
  ring.bound[(ring.head + ring.n) % 4] = l + 1;
  ++ring.n;
  while (ring.n > 2) {
    const int sl = ring.slot[ring.head];
    e = hipEventSynchronize(net->events[(size_t)sl]);
    if (e != hipSuccess) return e;
    ring.head = (ring.head + 1) % 4;
    --ring.n;
    *live_bound = std::min<int64_t>(*live_bound, net->pinned[sl]);
  }
  return hipSuccess;
}

// Report of a compaction enqueued with a tag (see k_compact): the live count and the flags.
struct Report {
  int64_t count = 0;
  bool nonbinary = false, overflow = false;
  bool many = false;  // the layer's outputs take more values than the one-byte dictionary holds
};

// Tag for the next reporting compaction (24 bits, never 0: the word starts at 0).
unsigned long long next_report_tag(sdnn_net *net) {
  net->notify_seq = (net->notify_seq + 1) & 0xffffffu;
  if (net->notify_seq == 0) net->notify_seq = 1;
  return net->notify_seq;
}

// Wait for the report tagged `tag`: spin on the word in coherent host memory (no OS wake-up in the
// way); if none arrives within 2 s, wait for the stream and read the count (at count_dev) and the
// flags by copies.
hipError_t wait_report(sdnn_net *net, unsigned long long tag, const int *count_dev, Report *r) {
  const auto t0 = std::chrono::steady_clock::now();
  for (uint32_t it = 1;; ++it) {
    const unsigned long long w = __atomic_load_n(net->notify, __ATOMIC_ACQUIRE);
    if ((w >> 40) == tag) {
      r->count = (int64_t)(w & 0xffffffffull);
      r->nonbinary = ((w >> 32) & 1ull) != 0;
      r->overflow = ((w >> 33) & 1ull) != 0;
      r->many = ((w >> 34) & 1ull) != 0;
      return hipSuccess;
    }
    if ((it & 4095u) == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::seconds(2)) break;
    __builtin_ia32_pause();
  }
  hipError_t e = hipStreamSynchronize(net->stream);
  if (e != hipSuccess) return e;
  int32_t v[3] = {0, 0, 0};
  e = hipMemcpy(&v[0], count_dev, sizeof(int32_t), hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemcpy(&v[1], net->misc, sizeof(int32_t), hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemcpy(&v[2], net->misc + kOverflowSlot, sizeof(int32_t), hipMemcpyDeviceToHost);
  r->count = v[0];
  r->nonbinary = v[1] != 0;
  r->overflow = v[2] != 0;
  r->many = false;
  return e;
}

// LDS-tile path: row-major activations ping-pong between two buffers; the live list is compacted
// after every layer.
sdnn_status infer_lds(sdnn_net *net, const float *y0, int M) {
  hipStream_t s = net->stream;
  const float *yin = y0;
  int cur = 0;
  int32_t l = 0;
  int64_t live_bound = M;
  // One launch runs every remaining layer once the live rows fit one workgroup per CU and either
  // take 4-row tiles or have stopped dying fast (the last two layers, not counting layer 0, each
  // kept 90% of their rows): inside that launch dead rows still occupy their tile's slots, while
  // layer-by-layer launches compact them away. Until the switch the count is read back after each
  // layer (those layers are long).
  const int bmax = fused_rows_max(net);
  int kept = 0;  // consecutive layers after layer 0 that kept at least 90% of their rows
  for (; l < net->L && live_bound > 0; ++l) {
    float *yout = net->ybuf[l & 1];
    const bool fits = (live_bound + bmax - 1) / bmax <= net->cus;
    const bool settled = kept >= 2;
    // (layer 0 too where the kernel marks the nonzero input rows, for at most 4 rows per CU: a launch, a
    // compaction and a wait less, 445 -> 410 us for one row through 120 layers of 1024 neurons. Rows that die
    // in the first layers keep their slots, as they do in later ones, and it still pays: 4096 neurons, layer 0
    // first / fused from it, 1024 rows of which 47 are left, 30 layers 398 / 380 us, 120 layers 1338 / 1318;
    // 1024 rows that all die within 3 layers 107 / 88.)
    const bool from0 = net->n_edge32 == net->L;
    if ((l > 0 || from0) && (live_bound <= 4 * (int64_t)net->cus || (fits && settled))) {
      const bool rec = net->profiling;
      if (rec) HIP_OR_POISON(net, hipEventRecord(net->prof_start[(size_t)l], s));
      HIP_OR_POISON(net, launch_layers_lds(net, yin, yout, l, net->ids[cur], net->counts + l, live_bound,
                                           l == 0 ? net->rownz : nullptr));
      if (rec) HIP_OR_POISON(net, hipEventRecord(net->prof_end[(size_t)l], s));
      if (net->profiling) net->prof_rec[(size_t)l] = rec;
      for (int32_t q = l; q < net->L; ++q) {
        net->layer_kernel[(size_t)q] = SDNN_KERNEL_LDS_FUSED;
        net->layer_ahead[(size_t)q] = net->n_edge32 == net->L;
        net->layer_launches[(size_t)q] = q == l ? 1 : 0;
      }
      // the final list: positions still live after the last layer (bits per 32 positions)
      hipLaunchKernelGGL(k_compact, dim3(1), dim3(1024), 0, s, net->masks, 32, net->ids[cur], net->ids[cur ^ 1],
                         (int *)nullptr, net->counts + l, net->counts + net->L, (int *)nullptr, (const int *)nullptr,
                         (unsigned long long *)nullptr, 0ull, CompactSample{});
      HIP_OR_POISON(net, hipGetLastError());
      cur ^= 1;
      net->layers_run = net->L;
      net->final_list = cur;
      net->final_y = yout;
      net->final_fm = nullptr;
      return SDNN_OK;
    }
    const bool rec = net->profiling && (net->prof_mode == 1 || live_bound > 256);
    if (rec) HIP_OR_POISON(net, hipEventRecord(net->prof_start[(size_t)l], s));
    // layer 0 of a uniform layer on a large batch (from 2^24 inputs, where packing and a read-back
    // cost less than they save): if every input is 0 or 1, by counts of the bit-packed rows (see
    // k_layer_count), written back as fp32 rows; masks then hold one bit per list position
    int mask_rows = net->B;
    bool counted = false;
    const LayerDev &ld0 = net->layers[0];
    if (l == 0 && (int64_t)M * net->N >= (1 << 24) && ld0.uniform && ld0.ell16 && ld0.w > 0.0f && (net->N & 3) == 0 &&
        (uint64_t)M * (uint64_t)net->N / 4 < (1ull << 32)) {
      HIP_OR_POISON(net, launch_pack_bits<32>(net, y0, net->ybuf[1], net->ids[cur], net->counts));
      HIP_OR_POISON(net, hipMemcpyAsync(net->pinned + 6, net->misc, sizeof(int32_t), hipMemcpyDeviceToHost, s));
      HIP_OR_POISON(net, hipStreamSynchronize(s));
      if (net->pinned[6] == 0) {
        HIP_OR_POISON(net, (launch_layer_count_k<32, true>(net, ld0, net->ybuf[1], nullptr, net->counts, yout,
                                                           net->ids[cur], net->masks)));
        counted = true;
        mask_rows = 32;
      }
    }
    if (!counted)
      HIP_OR_POISON(net, launch_layer(net, l, yin, yout, net->ids[cur], net->counts + l, live_bound,
                                      l == 0 ? net->rownz : nullptr));
    if (rec) HIP_OR_POISON(net, hipEventRecord(net->prof_end[(size_t)l], s));
    net->layer_kernel[(size_t)l] = counted ? SDNN_KERNEL_BITS_COUNT : SDNN_KERNEL_LDS_TILE;
    net->layer_ahead[(size_t)l] = !counted && lists_ahead(net, net->layers[(size_t)l], live_bound);
    net->layer_launches[(size_t)l] = counted ? 3 : 1;
    if (net->profiling) net->prof_rec[(size_t)l] = rec;
    const unsigned long long tag = next_report_tag(net);
    hipLaunchKernelGGL(k_compact, dim3(1), dim3(1024), 0, s, net->masks, mask_rows, net->ids[cur], net->ids[cur ^ 1],
                       (int *)nullptr, net->counts + l, net->counts + l + 1, (int *)nullptr, net->misc,
                       net->notify_dev, tag, CompactSample{});
    HIP_OR_POISON(net, hipGetLastError());
    cur ^= 1;
    yin = yout;
    Report rp;
    HIP_OR_POISON(net, wait_report(net, tag, net->counts + l + 1, &rp));
    const int64_t before = live_bound;
    live_bound = std::min<int64_t>(live_bound, rp.count);
    kept = (l > 0 && live_bound * 10 >= before * 9) ? kept + 1 : 0;
  }
  net->layers_run = l;
  net->final_list = cur;
  net->final_y = (l == net->L && net->L > 0) ? net->ybuf[(net->L - 1) & 1] : nullptr;
  net->final_fm = nullptr;
  return SDNN_OK;
}

// Global-tile path: activations stay in feature-major tiles of 32 list positions from layer to
// layer. Large layers are followed by a compaction of the live list (ids plus each live row's old
// position); the tiles are repacked to the compacted list only when that saves tiles, otherwise the
// next layer runs on the old positions, where rows that died hold zeros and stay zero. Small layers
// (one round of tiles) count their live rows themselves, so a layer is one launch; they are
// compacted only when the live bound says that fewer tiles would do, and after the last layer.
// Liveness masks alternate between two buffers by layer parity.
sdnn_status infer_gfm(sdnn_net *net, const float *y0, int M) {
  hipStream_t s = net->stream;
  int *npos = net->misc + kNposSlot;  // npos[i]: positions in list i
  const int64_t one_round = 8 * 32;
  auto tiles = [](int64_t r) { return (r + 31) / 32; };
  auto masks_for = [net](int32_t layer) { return net->masks_rot[layer % 3]; };
  int cur = 0;
  int64_t P = M;           // host bound on the positions of list cur (exact after a read-back)
  int64_t live_bound = M;  // host bound on the live rows
  const float *fin = nullptr;
  float *fout = nullptr;
  bool fin_codes = false, fout_codes = false;  // the tiles hold dictionary codes
  bool fin_wide = false;  // fin's codes are two bytes (k_encode<64, 2>), else one
  bool wide_ok = true;    // a two-byte encoding is worth trying
  // fp32 rows instead of tiles (k_layer_seg): row p of fin, or row fin_map[p], is list position p
  bool fin_rows = false, fout_rows = false;
  const int *fin_map = nullptr;
  // a layer of `rows` live rows runs on rows: more than one round of tiles, or columns of other than 32
  // sources (few-tile layers have kernels for 32 only). 60 layers of 10007 neurons with 1 to 48 sources, the
  // ELL walk of k_layer_gfm polled every 16 layers / rows with a report per layer (us): 1 row 494 / 249, 16
  // rows 2134 / 1658, 64 rows 2650 / 1800, 256 rows 5108 / 2415, 600 rows 11133 / 3192. 8 layers of 32
  // sources and 300 rows, tiles / rows, the library before the rows kernel and with it: 4097 neurons 469 / 328,
  // 10113 neurons 562 / 423. (Layers of 32 sources and fewer rows: k_layer_gfm_small, a launch without a report.)
  auto seg_layer = [&](int32_t layer, int64_t rows) {
    return layer < net->L && net->layers[(size_t)layer].seg && (rows > one_round || net->layers[(size_t)layer].K != 32);
  };
  bool next_tried = false;     // the next layer's one-byte codes were tried, or cannot fit
  bool repacked_codes = false;  // ... and wrote them (else fp32 tiles)
  int last_list = 0;
  bool compacted = true;   // the last layer run has been followed by a compaction
  PollRing ring;
  // few-tile layers leave their liveness in partial words; the next few-tile launch turns them into
  // mask words, any other reader of the masks needs k_finalize_masks first
  bool parts_pending = false;
  int32_t part_layer = -1;
  int part_G = 0, part_nt = 0;
  auto finalize_parts = [&]() -> hipError_t {
    if (!parts_pending) return hipSuccess;
    parts_pending = false;
    hipLaunchKernelGGL(k_finalize_masks, dim3(1), dim3(kPartThreads), 0, s, net->part[part_layer & 1], part_G, part_nt,
                       masks_for(part_layer));
    return hipGetLastError();
  };
  // few-tile layers: the host follows the device through the progress word, staying at most
  // kProgressAhead layers ahead of it, so that it learns within a few layers that no row is left
  const unsigned long long gen = net->run_gen & 0xffffu;
  bool follow = net->progress != nullptr;
  auto follow_progress = [&](int32_t layer) -> hipError_t {
    const int32_t need = layer - kProgressAhead;
    if (!follow || need < 0) return hipSuccess;
    const auto t0 = std::chrono::steady_clock::now();
    for (uint32_t it = 1;; ++it) {
      const unsigned long long w = __atomic_load_n(net->progress, __ATOMIC_ACQUIRE);
      if ((w >> kProgGenShift) == gen && (int32_t)((w >> kProgLayerShift) & 0xfffffu) >= need) {
        const unsigned long long c = w & kProgCountMask;
        if (c != kProgCountMask) live_bound = std::min<int64_t>(live_bound, (int64_t)c);
        return hipSuccess;
      }
      if ((it & 4095u) == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::seconds(2)) {
        // no report from the device: wait for the stream, and poll by copies from now on
        follow = false;
        return hipStreamSynchronize(s);
      }
      __builtin_ia32_pause();
    }
  };
  bool bits_route = false;  // layer 0 went to the bit-tile kernels (unless the report says otherwise)
  int32_t l = 0;
  for (; l < net->L && live_bound > 0; ++l) {
    const bool few = l > 0 && P <= one_round;
    // (a layer on rows or codes, however few, leaves its liveness in the spread words, which only the compaction
    // right after it reads)
    const bool small = few && !fin_rows && !fin_codes;
    bool reported = false;  // this layer's launch writes the progress word
    fout_codes = false;
    fout_rows = false;
    // the columns fout holds, when this layer computed one column per group of equal columns
    const LayerDev &lcur = net->layers[(size_t)l];
    const bool ocols_on = lcur.K == 32 && lcur.src16 && lcur.cols && lcur.dedup_ok;
    const int *fout_cols = nullptr;  // set by the branches whose kernels take the column list
    bool spread_used = false;  // this layer's liveness is in the spread words
    bool seglive_out = false;  // fout's all-zero segments were skipped (net->seglive says which)
    unsigned *mk = masks_for(l);
    const bool rec = net->profiling && (net->prof_mode == 1 || !few);
    if (net->profiling) net->prof_rec[(size_t)l] = rec;
    if (rec) HIP_OR_POISON(net, hipEventRecord(net->prof_start[(size_t)l], s));
    bool encoded = false;  // this layer reads codes that k_encode wrote from fp32 tiles
    int encode_tries = 0;  // launches spent on encodings of this layer's inputs
    const bool tried = next_tried;  // the repack before this layer tried one-byte codes (they overflowed)
    next_tried = false;
    repacked_codes = false;
    if (l > 0 && !fin_codes && !fin_rows && compacted && live_bound >= kEncodeMinRows && !net->equal_value_kernels) {
      // a large layer on fp32 tiles: if its inputs take at most 256 distinct values (saturated rows
      // do), encode them as one-byte codes into the free buffer and gather those instead (unless the
      // repack before this layer found that they do not fit: tried); else, if
      // they take at most 4096 and the fp32 tiles outgrow the L2 (kXcdL2Bytes), as two-byte codes;
      // a full dictionary stops an encoding early, and when both stop the layer reads the fp32 tiles
      unsigned char *cbuf = reinterpret_cast<unsigned char *>((fin == net->fm[1]) ? net->fm[0] : net->fm[1]);
      auto try_encode = [&](int cb) -> hipError_t {
        unsigned *gd = cb == 1 ? net->dict : net->dict16;
        if (cb == 1)
          hipLaunchKernelGGL(k_dict_reset<1>, dim3(1), dim3(256), 0, s, gd, net->misc + kOverflowSlot);
        else
          hipLaunchKernelGGL(k_dict_reset<2>, dim3(16), dim3(256), 0, s, gd, net->misc + kOverflowSlot);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        const int cr = code_rows(net->bitsT);
        const int64_t items = (live_bound + cr - 1) / cr * (int64_t)net->N * (cr / 16);
        const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(net->cus * 8, (items + 255) / 256));
        if (cb == 2 && cr != 64) return hipErrorInvalidValue;
        if (cb == 2)
          hipLaunchKernelGGL((k_encode<64, 2>), dim3(grid), dim3(256), 0, s, fin, cbuf, net->N, npos + cur, gd,
                             net->misc + kOverflowSlot);
        else if (cr == 128)
          hipLaunchKernelGGL((k_encode<128, 1>), dim3(grid), dim3(256), 0, s, fin, cbuf, net->N, npos + cur, gd,
                             net->misc + kOverflowSlot);
        else
          hipLaunchKernelGGL((k_encode<64, 1>), dim3(grid), dim3(256), 0, s, fin, cbuf, net->N, npos + cur, gd,
                             net->misc + kOverflowSlot);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        const unsigned long long tag = next_report_tag(net);
        hipLaunchKernelGGL(k_report_overflow, dim3(1), dim3(1), 0, s, net->misc + kOverflowSlot, net->notify_dev, tag);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        Report rp;
        e = wait_report(net, tag, npos + cur, &rp);
        if (e != hipSuccess) return e;
        encode_tries += 3;
        if (!rp.overflow) {
          fin = reinterpret_cast<const float *>(cbuf);
          fin_codes = true;
          fin_wide = cb == 2;
          encoded = true;
          if (cb == 1) wide_ok = true;
        }
        return hipSuccess;
      };
      if (!tried) HIP_OR_POISON(net, try_encode(1));
      if (!encoded && net->dict16 && wide_ok && (size_t)net->N * 32 * sizeof(float) > kXcdL2Bytes) {
        HIP_OR_POISON(net, try_encode(2));
        // inputs with more than 4096 values: the layers after it are not tried again until the
        // inputs of one of them fit 256 values (values that grow more varied stay so for a while)
        if (!encoded) wide_ok = false;
      }
      if (!encoded && seg_layer(l, P)) {
        // the tiles as rows, into the buffer the encoding left
        const int64_t items = tiles(P) * ((net->N + kRepackSources - 1) / kRepackSources);
        const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(net->cus * 8, items));
        float *rows = reinterpret_cast<float *>(cbuf);
        hipLaunchKernelGGL((k_repack<kRepackRows, 32>), dim3(grid), dim3(256), 0, s, fin, rows, net->N,
                           (const int *)nullptr, npos + cur, (const unsigned *)nullptr, (const int *)nullptr, net->N,
                           (unsigned char *)nullptr, (unsigned *)nullptr, (int *)nullptr);
        HIP_OR_POISON(net, hipGetLastError());
        fin = rows;
        fin_rows = true;
        fin_map = nullptr;
      }
    }
    fout = (fin == net->fm[1]) ? net->fm[0] : net->fm[1];
    if (l == 0) {
      // layer 0 reads the caller's rows; binary inputs go through bit tiles (built in fm[0]), others straight
      // into k_layer_seg or through feature-major tiles in fm[0]; each way also finds the nonzero input rows
      // the pack pass addresses rows with 32-bit offsets (in floats, or float4 when N % 4 == 0)
      const uint64_t units = (uint64_t)M * (uint64_t)net->N / ((net->N & 3) == 0 ? 4 : 1);
      const bool try_bits = net->bitsT > 0 && net->layers[0].K <= 32 && net->layers[0].ellw && units < (1ull << 32) &&
                            (net->bitsT == 32 ? bits_tile_bytes_needed<32>(net) <= bits_tile_bytes(32)
                                              : bits_tile_bytes_needed<16>(net) <= bits_tile_bytes(16));
      if (try_bits) {
        // the bit-tile kernels that follow exit at once if the pack finds an input other than 0 or 1
        // (misc[0]); the host learns of it from the layer's compaction report and then computes
        // layer 0 on fp32 tiles (no host round trip inside the layer)
        HIP_OR_POISON(net, net->bitsT == 32 ? launch_pack_bits<32>(net, y0, net->fm[0], net->ids[cur], npos + cur)
                                            : launch_pack_bits<16>(net, y0, net->fm[0], net->ids[cur], npos + cur));
        bits_route = true;
      }
      const LayerDev &ld0 = net->layers[0];
      if (bits_route && P > one_round && net->L > 1 && ld0.uniform && ld0.ell16 && ld0.w > 0.0f) {
        // a uniform layer: the output of a column is a function of how many of its sources are 1,
        // so the counts are the codes (see k_layer_count)
        fout_codes = true;
        net->layer_kernel[0] = SDNN_KERNEL_BITS_COUNT;
        net->layer_launches[0] = 3;  // pack + dictionary + count
        unsigned char *cout = reinterpret_cast<unsigned char *>(fout);
        HIP_OR_POISON(net, net->bitsT == 32 ? launch_layer_count<32>(net, ld0, net->fm[0], cout, npos + cur)
                                            : launch_layer_count<16>(net, ld0, net->fm[0], cout, npos + cur));
      } else if (bits_route) {
        // outputs of a layer on binary inputs take few distinct values: a large layer 0 writes them
        // as one-byte dictionary codes, which the next layer gathers four times denser
        fout_codes = P > one_round && net->L > 1;
        net->layer_kernel[0] = fout_codes ? SDNN_KERNEL_BITS_TO_CODES : SDNN_KERNEL_BITS;
        net->layer_launches[0] = 2;  // pack + layer
        HIP_OR_POISON(net, net->bitsT == 32
                               ? launch_layer_bits<32>(net, net->layers[0], net->fm[0], fout, npos + cur, fout_codes)
                               : launch_layer_bits<16>(net, net->layers[0], net->fm[0], fout, npos + cur, fout_codes));
      } else if (ld0.seg) {
        // straight from the caller's rows
        HIP_OR_POISON(net, launch_seg(net, ld0, y0, fout, net->ids[cur], npos + cur, P, mk, net->rownz, net->ids[cur]));
        spread_used = true;
        fout_rows = true;
        net->layer_kernel[0] = SDNN_KERNEL_GLOBAL_TILE;
        net->layer_ahead[0] = 1;
        net->layer_launches[0] = 1;
      } else {
        HIP_OR_POISON(net, launch_to_fm(net, y0, net->fm[0], net->ids[cur], npos + cur, try_bits ? nullptr : net->rownz));
        HIP_OR_POISON(net, launch_gfm(net, net->layers[0], net->fm[0], fout, npos + cur, tiles(P), mk, nullptr, nullptr,
                                      nullptr, net->spread));
        spread_used = true;
        fout_cols = ocols_on ? lcur.cols : nullptr;
        net->layer_kernel[0] = SDNN_KERNEL_GLOBAL_TILE;
        net->layer_launches[0] = 1 + gfm_launches(net, net->layers[0], tiles(P), 0) + (try_bits ? 1 : 0);
      }
    } else if (fin_codes) {
      // follows layer 0 or a layer whose outputs were encoded, both compacted: no count to take over
      const unsigned char *cin = reinterpret_cast<const unsigned char *>(fin);
      if (fin_wide)
        HIP_OR_POISON(net, launch_gfm_u16(net, net->layers[(size_t)l], cin, fout, npos + cur, tiles(P), mk, &seglive_out));
      else
        HIP_OR_POISON(net, launch_gfm_u8(net, net->layers[(size_t)l], cin, fout, npos + cur, tiles(P), mk, &seglive_out));
      spread_used = true;
      fout_cols = ocols_on ? lcur.cols : nullptr;
      net->layer_kernel[(size_t)l] = fin_wide ? SDNN_KERNEL_GLOBAL_TILE_CODES16 : SDNN_KERNEL_GLOBAL_TILE_CODES;
      const int st = code_rows(net->bitsT) / 32;  // fp32 tiles per code tile
      // (with the dictionary resets, encodings and their reports when this layer encoded its inputs)
      net->layer_launches[(size_t)l] = gfm_launches(net, net->layers[(size_t)l], tiles(P), st * 32) + encode_tries;
    } else if (fin_rows) {
      HIP_OR_POISON(net, launch_seg(net, lcur, fin, fout, fin_map, npos + cur, P, mk, nullptr, nullptr));
      spread_used = true;
      fout_rows = true;
      net->layer_kernel[(size_t)l] = SDNN_KERNEL_GLOBAL_TILE;
      net->layer_ahead[(size_t)l] = 1;
      net->layer_launches[(size_t)l] = 1 + encode_tries;
    } else {
      // after a layer without compaction, this launch counts that layer's live rows
      const LayerDev &ld = net->layers[(size_t)l];
      int *cnt = compacted ? nullptr : net->counts + l;
      if (small && ld.K == 32) {
        const unsigned *prev = cnt && parts_pending ? net->part[part_layer & 1] : nullptr;
        int G = 0, nt = 0;
        const unsigned long long tag = (gen << kProgGenShift) | ((unsigned long long)l << kProgLayerShift);
        HIP_OR_POISON(net, launch_gfm_small(net, ld, fin, fout, npos + cur, tiles(P), net->part[l & 1], prev, part_G,
                                            part_nt, masks_for(l - 1), masks_for(l + 1), cnt, net->counts + (l - 1),
                                            follow ? net->progress_dev : nullptr, tag, &G, &nt));
        reported = follow;
        fout_cols = ocols_on ? lcur.cols : nullptr;
        parts_pending = true;
        part_layer = l;
        part_G = G;
        part_nt = nt;
        net->layer_kernel[(size_t)l] = SDNN_KERNEL_GLOBAL_TILE_FEW_ROWS;
        net->layer_launches[(size_t)l] = 1;
      } else {
        HIP_OR_POISON(net, finalize_parts());
        // a large layer's liveness goes through spread words (compacted right after)
        HIP_OR_POISON(net, launch_gfm(net, ld, fin, fout, npos + cur, tiles(P), mk, masks_for(l - 1),
                                      masks_for(l + 1), cnt, small ? nullptr : net->spread));
        spread_used = !small;
        fout_cols = ocols_on ? lcur.cols : nullptr;
        net->layer_kernel[(size_t)l] = SDNN_KERNEL_GLOBAL_TILE;
        net->layer_launches[(size_t)l] = gfm_launches(net, ld, tiles(P), 0) + encode_tries;
      }
    }
    if (rec) HIP_OR_POISON(net, hipEventRecord(net->prof_end[(size_t)l], s));
    // compaction of this layer's live rows; with tag != 0 it reports its count and flags
    auto compact = [&](unsigned long long tag = 0) -> hipError_t {
      hipError_t e = finalize_parts();
      if (e != hipSuccess) return e;
      if (spread_used) {
        const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(net->cus, (tiles(P) + 255) / 256));
        hipLaunchKernelGGL(k_spread_to_masks, dim3(grid), dim3(256), 0, s, net->spread, npos + cur, mk);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        spread_used = false;
      }
      hipLaunchKernelGGL(k_compact, dim3(1), dim3(1024), 0, s, mk, 32, net->ids[cur], net->ids[cur ^ 1],
                         net->src[cur ^ 1], npos + cur, net->counts + l + 1, npos + (cur ^ 1), net->misc,
                         tag ? net->notify_dev : nullptr, tag,
                         CompactSample{tag && !fout_codes && !fout_cols && l + 1 < net->L && !net->equal_value_kernels
                                           ? fout : nullptr,
                                       seglive_out ? net->seglive : nullptr, net->N, fout_rows ? 1 : 0,
                                       (int)kEncodeMinRows});
      last_list = cur ^ 1;
      return hipGetLastError();
    };
    // the repack of this layer's outputs as the next layer's one-byte codes (k_repack<kRepackCodes, CR>), into
    // dst; sets repacked_codes when the dictionary held every value
    auto repack_codes = [&](float *dst) -> hipError_t {
      unsigned *gd = net->dict;
      hipLaunchKernelGGL(k_dict_reset<1>, dim3(1), dim3(256), 0, s, gd, net->misc + kOverflowSlot);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      const int cr = code_rows(net->bitsT);
      const int64_t items = (live_bound + cr - 1) / cr * (cr / 32) * ((net->N + kRepackSources - 1) / kRepackSources);
      const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(net->cus * 8, items));
      unsigned char *dc = reinterpret_cast<unsigned char *>(dst);
      const unsigned *sl = seglive_out ? net->seglive : nullptr;
      int *of = net->misc + kOverflowSlot;
      const int *sp = net->src[cur ^ 1], *np = npos + (cur ^ 1);
      if (cr == 128)
        hipLaunchKernelGGL((k_repack<kRepackCodes, 128>), dim3(grid), dim3(256), 0, s, fout, (float *)nullptr, net->N, sp, np, sl,
                           (const int *)nullptr, net->N, dc, gd, of);
      else
        hipLaunchKernelGGL((k_repack<kRepackCodes, 64>), dim3(grid), dim3(256), 0, s, fout, (float *)nullptr, net->N, sp, np, sl,
                           (const int *)nullptr, net->N, dc, gd, of);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
      const unsigned long long tag = next_report_tag(net);
      hipLaunchKernelGGL(k_report_overflow, dim3(1), dim3(1), 0, s, of, net->notify_dev, tag);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
      Report rp;
      e = wait_report(net, tag, np, &rp);
      if (e == hipSuccess && !rp.overflow) repacked_codes = true;
      return e;
    };
    compacted = false;
    bool adopt;
    bool many = false;  // the outputs do not fit the one-byte dictionary
    if (!small) {
      // a large layer: compact, and wait for its exact count (the next layer is large, so the wait
      // is short relative to it)
      unsigned long long tag = next_report_tag(net);
      HIP_OR_POISON(net, compact(tag));
      compacted = true;
      Report rp;
      HIP_OR_POISON(net, wait_report(net, tag, net->counts + l + 1, &rp));
      if (l == 0 && bits_route && rp.nonbinary) {
        // an input is not 0 or 1: the bit-tile kernel exited at once; layer 0 on fp32 tiles
        fout_codes = false;
        if (lcur.seg) {
          HIP_OR_POISON(net, launch_seg(net, lcur, y0, fout, net->ids[cur], npos + cur, P, mk, nullptr, nullptr));
          fout_rows = true;
        } else {
          HIP_OR_POISON(net, launch_to_fm(net, y0, net->fm[0], net->ids[cur], npos + cur, nullptr));
          HIP_OR_POISON(net, launch_gfm(net, net->layers[0], net->fm[0], fout, npos + cur, tiles(P), mk, nullptr,
                                        nullptr, nullptr, net->spread));
        }
        spread_used = true;
        net->layer_kernel[0] = SDNN_KERNEL_GLOBAL_TILE;
        net->layer_ahead[0] = lcur.seg != nullptr;
        net->layer_launches[0] = 2 + (lcur.seg ? 1 : gfm_launches(net, net->layers[0], tiles(P), 0));
        tag = next_report_tag(net);
        HIP_OR_POISON(net, compact(tag));
        HIP_OR_POISON(net, wait_report(net, tag, net->counts + l + 1, &rp));
      } else if (fout_codes && rp.overflow) {
        // more than 256 distinct values: redo layer 0 with fp32 outputs (same liveness)
        fout_codes = false;
        net->layer_kernel[0] = SDNN_KERNEL_BITS;
        net->layer_launches[0] = 3;  // pack + the layer with codes + the layer again with fp32 outputs
        HIP_OR_POISON(net, net->bitsT == 32
                               ? launch_layer_bits<32>(net, net->layers[0], net->fm[0], fout, npos + cur, false)
                               : launch_layer_bits<16>(net, net->layers[0], net->fm[0], fout, npos + cur, false));
        tag = next_report_tag(net);
        HIP_OR_POISON(net, compact(tag));
        HIP_OR_POISON(net, wait_report(net, tag, net->counts + l + 1, &rp));
      }
      live_bound = std::min<int64_t>(live_bound, rp.count);
      many = rp.many;
      // rows move on to the compacted list by its map alone; tiles become rows in the repack
      adopt = live_bound == 0 || tiles(live_bound) * 20 <= tiles(P) * 19 || fout_rows ||
              (!fout_codes && seg_layer(l + 1, live_bound));
    } else {
      adopt = tiles(live_bound) < tiles(P) || seg_layer(l + 1, live_bound);
    }
    next_tried = many;
    bool next_rows = false;
    if (adopt && live_bound > 0 && l + 1 < net->L) {
      if (!compacted) HIP_OR_POISON(net, compact());
      compacted = true;
      float *dst = (fout == net->fm[1]) ? net->fm[0] : net->fm[1];
      const int cr = code_rows(net->bitsT);
      const int64_t items = fout_codes ? (tiles(live_bound) + cr / 32 - 1) / (cr / 32) * net->N * (cr / 4) / 256
                                       : tiles(live_bound) * (((fout_cols ? lcur.D : net->N) + kRepackSources - 1) /
                                                              kRepackSources);
      const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(net->cus * 8, items));
      const bool codes_fit = live_bound >= kEncodeMinRows && !net->equal_value_kernels && !many;  // (perhaps)
      float *next = dst;
      if (fout_rows) {
        if (seg_layer(l + 1, live_bound) && !codes_fit) {
          next_rows = true;
          next = fout;
          fin_map = net->src[cur ^ 1];
        } else {
          // few rows go on in tiles, and the encoder reads tiles
          HIP_OR_POISON(net, launch_to_fm(net, fout, dst, net->src[cur ^ 1], npos + (cur ^ 1), nullptr));
        }
      } else if (fout_codes && cr == 128)
        hipLaunchKernelGGL(k_repack_u8<128>, dim3(grid), dim3(256), 0, s, reinterpret_cast<const unsigned char *>(fout),
                           reinterpret_cast<unsigned char *>(dst), net->N, net->src[cur ^ 1], npos + (cur ^ 1));
      else if (fout_codes)
        hipLaunchKernelGGL(k_repack_u8<64>, dim3(grid), dim3(256), 0, s, reinterpret_cast<const unsigned char *>(fout),
                           reinterpret_cast<unsigned char *>(dst), net->N, net->src[cur ^ 1], npos + (cur ^ 1));
      else {
        // the next layer encodes its inputs if they fit a dictionary (see the start of the loop):
        // the repack writes one-byte codes itself, and falls back to fp32 tiles when they overflow
        // (two-byte codes are then tried by k_encode from the fp32 tiles: written by the repack
        // they measured slower, 30.9 ms per step against 30.4 at 65536 neurons and 60,000 inputs)
        if (codes_fit && !fout_cols) {
          next_tried = true;
          HIP_OR_POISON(net, repack_codes(dst));
          if (repacked_codes) wide_ok = true;
        }
        if (!repacked_codes && seg_layer(l + 1, live_bound)) {
          next_rows = true;
          fin_map = nullptr;
          hipLaunchKernelGGL((k_repack<kRepackRows, 32>), dim3(grid), dim3(256), 0, s, fout, dst, net->N,
                             net->src[cur ^ 1], npos + (cur ^ 1), seglive_out ? net->seglive : nullptr,
                             (const int *)nullptr, net->N, (unsigned char *)nullptr, (unsigned *)nullptr, (int *)nullptr);
        } else if (!repacked_codes)
          hipLaunchKernelGGL((k_repack<kRepackTiles, 32>), dim3(grid), dim3(256), 0, s, fout, dst, net->N, net->src[cur ^ 1],
                             npos + (cur ^ 1), seglive_out ? net->seglive : nullptr, fout_cols,
                             fout_cols ? lcur.D : net->N, (unsigned char *)nullptr, (unsigned *)nullptr, (int *)nullptr);
      }
      HIP_OR_POISON(net, hipGetLastError());
      fin = next;
      cur ^= 1;
      P = live_bound;
    } else {
      if (seglive_out) {
        // the next layer (or the final read-out) takes the tiles as they are
        const int64_t items = tiles(P) * net->N * 8;
        const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(net->cus * 8, (items + 255) / 256));
        hipLaunchKernelGGL(k_fill_dead, dim3(grid), dim3(256), 0, s, fout, net->N, net->seglive, npos + cur);
        HIP_OR_POISON(net, hipGetLastError());
      }
      fin = fout;
    }
    fin_rows = next_rows;
    fin_codes = fout_codes || repacked_codes;  // (one-byte codes: a layer or a repack writes no others)
    fin_wide = false;
    // counts[l] is final once layer l has run (written by a compaction or by layer l's launch)
    if (reported)
      HIP_OR_POISON(net, follow_progress(l));
    else
      HIP_OR_POISON(net, poll_step(net, ring, l, l, &live_bound));
  }
  if (!compacted) {
    // the final list: compaction of the last layer's masks
    const int32_t last = l - 1;
    HIP_OR_POISON(net, finalize_parts());
    hipLaunchKernelGGL(k_compact, dim3(1), dim3(1024), 0, s, masks_for(last), 32, net->ids[cur], net->ids[cur ^ 1],
                       net->src[cur ^ 1], npos + cur, net->counts + last + 1, npos + (cur ^ 1), (const int *)nullptr,
                       (unsigned long long *)nullptr, 0ull, CompactSample{});
    HIP_OR_POISON(net, hipGetLastError());
    last_list = cur ^ 1;
  }
  net->layers_run = l;
  net->final_list = last_list;
  net->final_y = nullptr;
  net->final_fm = (l == net->L && net->L > 0) ? fout : nullptr;
  net->final_rows_major = fout_rows;
  return SDNN_OK;
}

sdnn_status infer_impl(sdnn_net *net, const float *y0, int64_t n_rows, void *workspace, size_t workspace_bytes,
                       void *hip_stream);

}  // namespace

sdnn_status sdnn_infer(sdnn_net *net, const float *y0, int64_t n_rows, void *workspace, size_t workspace_bytes,
                       void *hip_stream) try {
  return infer_impl(net, y0, n_rows, workspace, workspace_bytes, hip_stream);
} SDNN_CATCH

sdnn_status sdnn_infer_static(sdnn_net *net, const float *y0, int64_t n_rows, void *hip_stream) try {
  sdnn_status st = check_usable(net);
  if (st != SDNN_OK) return st;
  if (n_rows < 0) return fail(SDNN_EINVAL, "n_rows %lld out of range", (long long)n_rows);
  const size_t need = sdnn_workspace_bytes(net, n_rows);
  if (need > kStaticWorkspaceBytes)
    return fail(SDNN_ERANGE, "%lld rows need %zu bytes of workspace; the static workspace holds %zu",
                (long long)n_rows, need, kStaticWorkspaceBytes);
  int dev = -1;
  HIP_OR_POISON(net, hipGetDevice(&dev));
  void *ws = nullptr;
  st = scratch_address(dev, &ws);
  if (st != SDNN_OK) return st;
  return infer_impl(net, y0, n_rows, ws, kStaticWorkspaceBytes, hip_stream);
} SDNN_CATCH


namespace {

sdnn_status infer_impl(sdnn_net *net, const float *y0, int64_t n_rows, void *workspace, size_t workspace_bytes,
                       void *hip_stream) {
  sdnn_status st = check_usable(net);
  if (st != SDNN_OK) return st;
  if (net->n_loaded != net->L) return fail(SDNN_ESTATE, "%d of %d layers loaded", net->n_loaded, net->L);
  if (n_rows < 0 || n_rows > (int64_t)0x7fffffff) return fail(SDNN_EINVAL, "n_rows %lld out of range", (long long)n_rows);
  if (n_rows > 0 && !y0) return fail(SDNN_EINVAL, "y0 is null");
  if (!workspace) return fail(SDNN_EINVAL, "workspace is null");
  if (reinterpret_cast<uintptr_t>(workspace) % 256) return fail(SDNN_EINVAL, "workspace is not 256-byte aligned");
  if (n_rows > 0 && reinterpret_cast<uintptr_t>(y0) % 16 && net->N % 4 == 0)
    return fail(SDNN_EINVAL, "y0 must be 16-byte aligned");
  const WsLayout w = layout_for(net, n_rows);
  if (workspace_bytes < w.total) return fail(SDNN_EINVAL, "workspace has %zu bytes, needs %zu", workspace_bytes, w.total);
  int dev = -1;
  HIP_OR_POISON(net, hipGetDevice(&dev));
  if (dev != net->device) return fail(SDNN_EINVAL, "current device %d differs from the handle's device %d", dev, net->device);
  if (n_rows > 0 && hip_stream) {
    // a replay could run on any stream, and sdnn_categories waits for this one once (the kernels that wait
    // for reports cannot be captured at all; the default stream never is)
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(reinterpret_cast<hipStream_t>(hip_stream), &cap) != hipSuccess) (void)hipGetLastError();
    else if (cap != hipStreamCaptureStatusNone) return fail(SDNN_ESTATE, "the stream is being captured");
  }
  char *ws = static_cast<char *>(workspace);
  net->M = n_rows;
  ++net->run_gen;
  net->stream = reinterpret_cast<hipStream_t>(hip_stream);
  net->ws = ws;
  for (int i = 0; i < 2; ++i) {
    float *act = reinterpret_cast<float *>(ws + w.act[i]);
    net->ybuf[i] = net->path == 0 ? act : nullptr;
    net->fm[i] = net->path == 1 ? act : nullptr;
    net->ids[i] = reinterpret_cast<int *>(ws + w.ids[i]);
    net->src[i] = reinterpret_cast<int *>(ws + w.src[i]);
  }
  for (int i = 0; i < 3; ++i) net->masks_rot[i] = reinterpret_cast<unsigned *>(ws + w.masks[i]);
  net->masks = net->masks_rot[0];
  net->rownz = reinterpret_cast<int *>(ws + w.rownz);
  net->counts = reinterpret_cast<int *>(ws + w.counts);
  net->misc = reinterpret_cast<int *>(ws + w.misc);
  net->dict = reinterpret_cast<unsigned *>(ws + w.dict);
  net->dict16 = net->path == 1 ? reinterpret_cast<unsigned *>(ws + w.dict16) : nullptr;
  net->seglive = reinterpret_cast<unsigned *>(ws + w.seglive);
  for (int i = 0; i < 2; ++i) net->part[i] = reinterpret_cast<unsigned *>(ws + w.part[i]);
  net->spread = reinterpret_cast<unsigned *>(ws + w.spread);
  net->final_ids = reinterpret_cast<long long *>(ws + w.final_ids);
  net->ran = false;
  net->finished = false;

  const int M = (int)n_rows;
  hipStream_t s = net->stream;
  hipLaunchKernelGGL(k_init, dim3(std::max(1, std::min(net->cus * 4, (M + 255) / 256 + 1))), dim3(256), 0, s,
                     net->ids[0], net->masks_rot[0], net->masks_rot[1], net->masks_rot[2], net->rownz, net->counts,
                     net->misc, net->dict, M, net->L, net->spread, w.spread_words);
  HIP_OR_POISON(net, hipGetLastError());
  if (net->profiling) net->prof_rec.assign((size_t)net->L, 0);
  net->layer_kernel.assign((size_t)net->L, SDNN_KERNEL_NONE);
  net->layer_launches.assign((size_t)net->L, 0);
  net->layer_ahead.assign((size_t)net->L, 0);
  st = net->path == 0 ? infer_lds(net, y0, M) : infer_gfm(net, y0, M);
  if (st != SDNN_OK) return st;
  net->ran = true;
  net->pending_times = net->profiling;
  g_err.clear();
  return SDNN_OK;
}

}  // namespace

namespace {

// The handle's device as the current one while kernels are launched on its stream (the caller may have
// changed it since sdnn_infer).
struct DeviceGuard {
  int before = -1;
  hipError_t status;
  explicit DeviceGuard(int device) {
    status = hipGetDevice(&before);
    if (status != hipSuccess || before == device) before = -1;
    else status = hipSetDevice(device);
  }
  ~DeviceGuard() {
    if (before >= 0) (void)hipSetDevice(before);
  }
};

// The last infer's number of categories and their ids to the host, and wait for them (once). The host's
// words are the handle's, so only a kernel that the host waits for at once may write them: as the last
// kernel of sdnn_infer, one still queued on another stream would overwrite a later run's answer.
hipError_t finish(sdnn_net *net) {
  if (net->finished) return hipSuccess;
  const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(net->cus, (net->M + 255) / 256 + 1));
  hipLaunchKernelGGL(k_final_ids, dim3(grid), dim3(256), 0, net->stream, net->ids[net->final_list],
                     net->counts + net->layers_run, (int)net->M, net->final_ids, net->host_out_dev);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(net->stream);
  net->finished = e == hipSuccess;
  return e;
}

// The ids of the c categories of a finished run.
hipError_t read_ids(sdnn_net *net, int32_t c, int64_t *ids) {
  if (c <= 0) return hipSuccess;
  if (c > kHostIds) return hipMemcpy(ids, net->final_ids, (size_t)c * sizeof(long long), hipMemcpyDeviceToHost);
  for (int32_t i = 0; i < c; ++i) ids[i] = net->host_out->ids[i];
  return hipSuccess;
}

}  // namespace

sdnn_status sdnn_categories(sdnn_net *net, int64_t *ids, int64_t capacity, int64_t *count) {
  sdnn_status st = check_usable(net);
  if (st != SDNN_OK) return st;
  if (!net->ran) return fail(SDNN_ESTATE, "no inference has run");
  if (!count) return fail(SDNN_EINVAL, "count is null");
  const DeviceGuard dev(net->device);
  HIP_OR_POISON(net, dev.status);
  HIP_OR_POISON(net, finish(net));
  if (net->pending_times) {
    for (int32_t l = 0; l < net->layers_run; ++l) {
      if (!net->prof_rec[(size_t)l]) continue;
      float ms = 0.0f;
      HIP_OR_POISON(net, hipEventElapsedTime(&ms, net->prof_start[(size_t)l], net->prof_end[(size_t)l]));
      net->prof_ms[(size_t)l] += ms;
      net->prof_runs[(size_t)l] += 1;
    }
    net->pending_times = false;
  }
  const int32_t c = net->host_out->count;
  *count = c;
  if (!ids || capacity < c) return fail(SDNN_ERANGE, "need capacity %d", c);
  HIP_OR_POISON(net, read_ids(net, c, ids));
  g_err.clear();
  return SDNN_OK;
}

sdnn_status sdnn_live_counts(sdnn_net *net, int64_t *counts) try {
  sdnn_status st = check_usable(net);
  if (st != SDNN_OK) return st;
  if (!net->ran) return fail(SDNN_ESTATE, "no inference has run");
  if (!counts) return fail(SDNN_EINVAL, "counts is null");
  const DeviceGuard dev(net->device);
  HIP_OR_POISON(net, dev.status);
  if (net->L < kHostCounts) {
    hipLaunchKernelGGL(k_host_counts, dim3(1), dim3(1024), 0, net->stream, net->counts, net->L, net->rownz, (int)net->M,
                       net->host_out_dev);
    HIP_OR_POISON(net, hipGetLastError());
    HIP_OR_POISON(net, hipStreamSynchronize(net->stream));
    counts[0] = net->host_out->nonzero;
    for (int32_t l = 1; l <= net->L; ++l) counts[l] = net->host_out->counts[l];
    g_err.clear();
    return SDNN_OK;
  }
  HIP_OR_POISON(net, hipStreamSynchronize(net->stream));
  std::vector<int32_t> c((size_t)net->L + 1);
  HIP_OR_POISON(net, hipMemcpy(c.data(), net->counts, c.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
  std::vector<int32_t> nz((size_t)std::max<int64_t>(net->M, 1));
  if (net->M > 0) HIP_OR_POISON(net, hipMemcpy(nz.data(), net->rownz, (size_t)net->M * sizeof(int32_t), hipMemcpyDeviceToHost));
  int64_t r0 = 0;
  for (int64_t i = 0; i < net->M; ++i) r0 += nz[(size_t)i] != 0;
  counts[0] = r0;
  for (int32_t l = 1; l <= net->L; ++l) counts[l] = c[(size_t)l];
  g_err.clear();
  return SDNN_OK;
} SDNN_CATCH

sdnn_status sdnn_final_rows(sdnn_net *net, const int64_t *ids, int64_t n, float *out_host) try {
  sdnn_status st = check_usable(net);
  if (st != SDNN_OK) return st;
  if (!net->ran) return fail(SDNN_ESTATE, "no inference has run");
  if (n < 0 || (n > 0 && (!ids || !out_host))) return fail(SDNN_EINVAL, "bad arguments");
  for (int64_t q = 0; q < n; ++q)
    if (ids[q] < 0 || ids[q] >= net->M) return fail(SDNN_EINVAL, "row id %lld out of range", (long long)ids[q]);
  const DeviceGuard dev(net->device);
  HIP_OR_POISON(net, dev.status);
  HIP_OR_POISON(net, finish(net));
  const int32_t c = net->host_out->count;
  std::vector<int64_t> live((size_t)std::max(c, 1));
  HIP_OR_POISON(net, read_ids(net, c, live.data()));
  const size_t rowb = (size_t)net->N * sizeof(float);
  // the final activations: rows by id (LDS-tile path), rows or feature-major tiles by list position
  const float *act = net->path == 0 ? net->final_y : net->final_fm;
  const bool by_row = net->path == 0 || net->final_rows_major;
  // requested rows that are live: where they are in the live list, and their places in the answer
  std::vector<int32_t> at;
  std::vector<int64_t> which;
  for (int64_t q = 0; q < n; ++q) {
    const auto it = std::lower_bound(live.begin(), live.begin() + c, ids[q]);
    if (act && it != live.begin() + c && *it == ids[q]) {
      at.push_back((int32_t)(it - live.begin()));
      which.push_back(q);
    } else {
      std::memset(out_host + (size_t)q * net->N, 0, rowb);
    }
  }
  const size_t nr = at.size();
  bool every = nr == (size_t)c;  // the whole live list, in order
  bool consecutive = true;       // rows that follow each other
  for (size_t i = 0; i < nr; ++i) {
    every = every && (size_t)at[i] == i;
    consecutive = consecutive && live[(size_t)at[i]] == live[(size_t)at[0]] + (int64_t)i;
  }
  const bool direct = nr > 0 && which.back() - which.front() + 1 == (int64_t)nr;  // one run of the answer
  bool done = nr == 0;
  if (!done && net->path == 0 && direct && consecutive) {
    // one copy
    HIP_OR_POISON(net, hipMemcpy(out_host + (size_t)which[0] * net->N, act + (size_t)live[(size_t)at[0]] * net->N,
                                 nr * rowb, hipMemcpyDeviceToHost));
    done = true;
  }
  if (!done) {
    // their places in act, on the device: the final list itself when all of it is asked for, else an
    // uploaded list; then the rows are gathered into the free activation buffer, in batches
    float *const *buf = net->path == 0 ? net->ybuf : net->fm;
    float *stage = act == buf[0] ? buf[1] : buf[0];
    const int *list = net->path == 0 ? net->ids[net->final_list] : net->src[net->final_list];
    std::vector<int32_t> place;
    if (!every) {
      place.resize(nr);
      if (net->path == 0) {
        for (size_t i = 0; i < nr; ++i) place[i] = (int32_t)live[(size_t)at[i]];
      } else {
        std::vector<int32_t> srcpos((size_t)c);
        HIP_OR_POISON(net, hipMemcpy(srcpos.data(), list, (size_t)c * sizeof(int32_t), hipMemcpyDeviceToHost));
        for (size_t i = 0; i < nr; ++i) place[i] = srcpos[(size_t)at[i]];
      }
    }
    int *dpos = net->ids[net->final_list ^ 1];
    const size_t batch = (size_t)std::max<int64_t>(1, net->M);
    std::vector<float> rows;
    for (size_t b0 = 0; b0 < nr; b0 += batch) {
      const int nb = (int)std::min<size_t>(batch, nr - b0);
      const int *pos = list;
      if (!every) {
        HIP_OR_POISON(net, hipMemcpy(dpos, place.data() + b0, (size_t)nb * sizeof(int32_t), hipMemcpyHostToDevice));
        pos = dpos;
      }
      const int64_t items = (int64_t)nb * net->N;
      const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(net->cus * 8, (items + 255) / 256));
      hipLaunchKernelGGL(k_gather_rows, dim3(grid), dim3(256), 0, net->stream, act, net->N, pos, nb, stage, by_row);
      HIP_OR_POISON(net, hipGetLastError());
      HIP_OR_POISON(net, hipStreamSynchronize(net->stream));
      float *dst = out_host + (size_t)which[b0] * net->N;
      if (!direct) {
        rows.resize((size_t)nb * net->N);
        dst = rows.data();
      }
      HIP_OR_POISON(net, hipMemcpy(dst, stage, (size_t)nb * rowb, hipMemcpyDeviceToHost));
      if (!direct)
        for (int i = 0; i < nb; ++i)
          std::memcpy(out_host + (size_t)which[b0 + (size_t)i] * net->N, rows.data() + (size_t)i * net->N, rowb);
    }
  }
  // the last layer may have computed only one column of each group of equal columns
  if (!net->last_rep.empty())
    for (size_t i = 0; i < nr; ++i) {
      float *dst = out_host + (size_t)which[i] * net->N;
      for (int32_t j = 0; j < net->N; ++j) dst[j] = dst[net->last_rep[(size_t)j]];
    }
  g_err.clear();
  return SDNN_OK;
} SDNN_CATCH

sdnn_status sdnn_set_profiling(sdnn_net *net, int32_t enable) try {
  sdnn_status st = check_usable(net);
  if (st != SDNN_OK) return st;
  if (enable < 0 || enable > 2) return fail(SDNN_EINVAL, "profiling mode %d is not 0, 1 or 2", enable);
  net->pending_times = false;
  if (!enable) {
    net->profiling = false;
    g_err.clear();
    return SDNN_OK;
  }
  if (net->prof_start.empty()) {
    net->prof_end.resize((size_t)net->L);
    net->prof_start.resize((size_t)net->L);
    for (int32_t l = 0; l < net->L; ++l) {
      HIP_OR_POISON(net, hipEventCreate(&net->prof_start[(size_t)l]));
      HIP_OR_POISON(net, hipEventCreate(&net->prof_end[(size_t)l]));
    }
  }
  net->prof_ms.assign((size_t)net->L, 0.0);
  net->prof_runs.assign((size_t)net->L, 0);
  net->profiling = true;
  net->prof_mode = enable;
  g_err.clear();
  return SDNN_OK;
} SDNN_CATCH

sdnn_status sdnn_layer_info(sdnn_net *net, int32_t *kernel, int32_t *launches) {
  sdnn_status st = check_usable(net);
  if (st != SDNN_OK) return st;
  if (!net->ran) return fail(SDNN_ESTATE, "no inference has run");
  if (!kernel || !launches) return fail(SDNN_EINVAL, "null array");
  for (int32_t l = 0; l < net->L; ++l) {
    kernel[l] = net->layer_kernel[(size_t)l];
    launches[l] = net->layer_launches[(size_t)l];
  }
  g_err.clear();
  return SDNN_OK;
}

sdnn_status sdnn_layer_kernel(sdnn_net *net, int32_t layer, const char **name) {
  sdnn_status st = check_usable(net);
  if (st != SDNN_OK) return st;
  if (!net->ran) return fail(SDNN_ESTATE, "no inference has run");
  if (!name) return fail(SDNN_EINVAL, "name is null");
  if (layer < 0 || layer >= net->L) return fail(SDNN_EINVAL, "layer %d outside [0, %d)", layer, net->L);
  const bool ahead = net->layer_ahead[(size_t)layer] != 0;
  switch (net->layer_kernel[(size_t)layer]) {
    case SDNN_KERNEL_LDS_TILE: *name = ahead ? "k_layer_lds32" : "k_layer_lds"; break;
    case SDNN_KERNEL_GLOBAL_TILE: *name = ahead ? "k_layer_seg" : "k_layer_gfm"; break;
    case SDNN_KERNEL_GLOBAL_TILE_CODES: *name = "k_layer_gfm_u8"; break;
    case SDNN_KERNEL_GLOBAL_TILE_FEW_ROWS: *name = "k_layer_gfm_small"; break;
    case SDNN_KERNEL_BITS: *name = "k_pack_bits+k_layer_bits"; break;
    case SDNN_KERNEL_BITS_TO_CODES: *name = "k_pack_bits+k_layer_bits(codes)"; break;
    case SDNN_KERNEL_BITS_COUNT: *name = "k_pack_bits+k_layer_count"; break;
    case SDNN_KERNEL_LDS_FUSED: *name = ahead ? "k_layers_lds32" : "k_layers_lds"; break;
    case SDNN_KERNEL_GLOBAL_TILE_CODES16: *name = "k_layer_gfm_u16"; break;
    default: *name = "none"; break;
  }
  g_err.clear();
  return SDNN_OK;
}

sdnn_status sdnn_layer_times(sdnn_net *net, double *ms, int64_t *runs) {
  sdnn_status st = check_usable(net);
  if (st != SDNN_OK) return st;
  if (!ms || !runs) return fail(SDNN_EINVAL, "null array");
  for (int32_t l = 0; l < net->L; ++l) {
    ms[l] = net->prof_ms.empty() ? 0.0 : net->prof_ms[(size_t)l];
    runs[l] = net->prof_runs.empty() ? 0 : net->prof_runs[(size_t)l];
  }
  g_err.clear();
  return SDNN_OK;
}

void sdnn_destroy(sdnn_net *net) {
  if (!net) return;
  for (auto &ev : net->prof_start) (void)hipEventDestroy(ev);
  for (auto &ev : net->prof_end) (void)hipEventDestroy(ev);
  for (void *p : net->allocations) (void)hipFree(p);
  for (void *p : net->streams) (void)hipFree(p);
  for (auto &ev : net->events) (void)hipEventDestroy(ev);
  if (net->pinned) (void)hipHostFree(net->pinned);
  if (net->progress) (void)hipHostFree(net->progress);
  if (net->notify) (void)hipHostFree(net->notify);
  if (net->host_out) (void)hipHostFree(net->host_out);
  delete net;
}

}  // extern "C"
