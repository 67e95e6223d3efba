// Internal helpers shared by the libsrt HIP kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "srt.h"

#define SRT_WAVE 64

namespace srt {

// ---------------------------------------------------------------------------
// Host-side helpers
// ---------------------------------------------------------------------------
inline int hip_status(hipError_t e) { return e == hipSuccess ? SRT_OK : SRT_ERR_HIP; }

inline int launch_status() {
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? SRT_OK : SRT_ERR_HIP;
}

inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

// ---------------------------------------------------------------------------
// Per-prompt cache workspace layout (device memory, caller-owned).
//
// Nodes live in an open-addressing hash table whose slot index is the node
// id: key = (parent_id << 32) | token, roots use parent = kRootParent and
// token = prompt id.  Children of a node form a singly linked list pushed at
// creation time.  A slot is 20 bytes: key (u64), count (u32) and first child
// (u32) in one aligned 16-byte piece, and the next sibling (u32); four slots
// share an 80-byte group (four pieces, then four next words), so a node's
// words lie within 80 bytes.  Every access to a node is a random one into a
// table of up to tens of GB, so what an insertion or a child-list walk costs
// is the memory pages and lines it touches: with the four words in arrays of
// their own a visit touched up to four of each.
// A slot that nothing has used is all ones, so one fill formats the table;
// the stored count is the node's count plus kCountBias (creating a node
// leaves the fill value, which reads as 1).
constexpr uint32_t kMagic = 0x53525432u;  // "SRT2"
constexpr uint64_t kEmptyKey = ~0ull;
constexpr uint32_t kNone = 0xFFFFFFFFu;
constexpr uint32_t kRootParent = 0xFFFFFFFFu;
constexpr uint32_t kCountBias = 2u;  // count = stored count + 2 (mod 2^32)
constexpr uint32_t kMaxSlotsLog2 = 31;  // node ids stay below kRootParent
// Slots a key may lie past its first one.  Up to the capacity (a load of at
// most 0.8) a run of 1000 taken slots is not to be expected in the largest
// table; the bound ends probes of a table that a call fills past its capacity.
constexpr uint64_t kMaxProbes = 4096;

struct alignas(256) WsHeader {
  uint32_t magic;
  uint32_t flags;               // sticky SRT_FLAG_* bits
  int32_t n_prompts;
  int32_t max_streams;
  int32_t max_depth;            // D
  int32_t stream_stride;        // int32 words per stream record
  uint64_t slots;               // power of two
  uint64_t node_limit;          // node_capacity + n_prompts
  unsigned long long used;      // nodes created, roots included
  unsigned long long export_n;  // scratch counter of srt_trie_export
  uint64_t off_roots, off_streams, off_table;
  uint64_t total_bytes;
  int64_t node_capacity;
};

// Stream record: [0] prompt (-1 = unbound), [1] tokens appended so far,
// [2 + j - 1] the node of the stream's suffix of length j, j = 1 ..
// min(appended, D-1) (its active nodes; kNone if the table was full).
constexpr int kStreamHead = 2;

// The 16-byte piece of a slot (first of the words as stored).
struct alignas(16) Slot {
  unsigned long long key;
  uint32_t count;  // plus kCountBias is the node's count
  uint32_t first;
};
constexpr int kGroupSlots = 4;                                            // slots per group
constexpr uint64_t kGroupBytes = kGroupSlots * (sizeof(Slot) + sizeof(uint32_t));  // 80

struct TrieView {
  WsHeader* hdr;
  uint32_t* roots;
  int32_t* streams;
  char* table;
  uint64_t mask;
  uint64_t probes;  // slots a key may lie in: min(slots, kMaxProbes)
  int32_t depth;

  __device__ Slot* slot(uint64_t id) const {
    return reinterpret_cast<Slot*>(table + (id / kGroupSlots) * kGroupBytes + (id % kGroupSlots) * sizeof(Slot));
  }
  __device__ uint32_t* next(uint64_t id) const {
    return reinterpret_cast<uint32_t*>(table + (id / kGroupSlots) * kGroupBytes + kGroupSlots * sizeof(Slot) +
                                       (id % kGroupSlots) * sizeof(uint32_t));
  }
};

__host__ __device__ inline TrieView trie_view(void* ws, const WsHeader& h) {
  char* base = static_cast<char*>(ws);
  TrieView v;
  v.hdr = reinterpret_cast<WsHeader*>(base);
  v.roots = reinterpret_cast<uint32_t*>(base + h.off_roots);
  v.streams = reinterpret_cast<int32_t*>(base + h.off_streams);
  v.table = base + h.off_table;
  v.mask = h.slots - 1;
  v.probes = h.slots < kMaxProbes ? h.slots : kMaxProbes;
  v.depth = h.max_depth;
  return v;
}

__device__ inline TrieView trie_view_dev(const void* ws) {
  const WsHeader* h = static_cast<const WsHeader*>(ws);
  return trie_view(const_cast<void*>(ws), *h);
}

__host__ __device__ inline uint64_t node_key(uint32_t parent, uint32_t token) {
  return (static_cast<uint64_t>(parent) << 32) | static_cast<uint64_t>(token);
}

// 64-bit finaliser (MurmurHash3 fmix64).
__host__ __device__ inline uint64_t mix64(uint64_t k) {
  k ^= k >> 33;
  k *= 0xff51afd7ed558ccdull;
  k ^= k >> 33;
  k *= 0xc4ceb9fe1a85ec53ull;
  k ^= k >> 33;
  return k;
}

__device__ inline void set_flag(const TrieView& t, uint32_t f) { atomicOr(&t.hdr->flags, f); }

// Slot of (parent, token), or kNone; `first` = its list head.  Read-only.  Two
// slots of the probe order are read at a time, so that a wave whose lanes
// look up different keys rarely waits for a third.
__device__ inline uint32_t trie_lookup(const TrieView& t, uint32_t parent, uint32_t token, uint32_t& first) {
  const uint64_t key = node_key(parent, token);
  uint64_t h = mix64(key) & t.mask;
  for (uint64_t probe = 0; probe < t.probes; probe += 2) {
    const uint64_t h1 = (h + 1) & t.mask;
    const Slot s0 = *t.slot(h), s1 = *t.slot(h1);
    if (s0.key == key) {
      first = s0.first;
      return static_cast<uint32_t>(h);
    }
    if (s0.key == kEmptyKey) return kNone;
    if (s1.key == key) {
      first = s1.first;
      return static_cast<uint32_t>(h1);
    }
    if (s1.key == kEmptyKey) return kNone;
    h = (h + 2) & t.mask;
  }
  return kNone;
}

// Slot of `key`, created by this thread (created = true) if absent; kNone
// and the capacity flag if every slot it may lie in is taken.  The probe is the CAS itself
// (a failed one returns the slot's key), one round trip for a new key in a
// free slot.  `beside()` runs once, before the first probe returns.
// Reading first costs more than the failed CASes it spares, also in bulk
// builds, where a quarter of the probes fail or find: 1.2 M tokens of 20-token
// strings into 32 caches took 4.0 ms this way, 4.2 ms reading each slot
// first and 4.2-4.5 ms reading the four keys of a group at once.
template <typename F>
__device__ inline uint32_t trie_find_or_create(const TrieView& t, uint64_t key, bool& created, F beside) {
  uint64_t h = mix64(key) & t.mask;
  beside();
  unsigned long long old = atomicCAS(&t.slot(h)->key, kEmptyKey, (unsigned long long)key);
  for (uint64_t probes = 1; old != kEmptyKey && old != key; ++probes) {
    if (probes >= t.probes) {
      created = false;
      set_flag(t, SRT_FLAG_CAPACITY);
      return kNone;
    }
    h = (h + 1) & t.mask;
    old = atomicCAS(&t.slot(h)->key, kEmptyKey, (unsigned long long)key);
  }
  created = old == kEmptyKey;
  return static_cast<uint32_t>(h);
}

// ---------------------------------------------------------------------------
// Wave helpers
// ---------------------------------------------------------------------------
__device__ inline int lane_id() { return __lane_id(); }

template <typename T>
__device__ inline T shfl_xor(T v, int m) {
  return __shfl_xor(v, m, SRT_WAVE);
}

// Sum over the wave in every lane, by DPP adds (a few cycles each, where a
// shuffle goes through the LDS crossbar): within rows of 16 lanes, then lane 15
// of a row into the next one, then lane 31 into the upper half.
__device__ inline int wave_sum(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return __builtin_amdgcn_readlane(x, SRT_WAVE - 1);
}

__device__ inline uint64_t shfl_xor_u64(uint64_t v, int m) {
  const uint32_t lo = __shfl_xor(static_cast<uint32_t>(v), m, SRT_WAVE);
  const uint32_t hi = __shfl_xor(static_cast<uint32_t>(v >> 32), m, SRT_WAVE);
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

__device__ inline uint64_t shfl_u64(uint64_t v, int src) {
  const uint32_t lo = __shfl(static_cast<uint32_t>(v), src, SRT_WAVE);
  const uint32_t hi = __shfl(static_cast<uint32_t>(v >> 32), src, SRT_WAVE);
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

}  // namespace srt
