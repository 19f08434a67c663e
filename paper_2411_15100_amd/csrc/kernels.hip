// HIP kernels for gfx950 (wave64): token walk / classify, rank->id permute,
// context-dependent lists, batched mask fill, -inf apply.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.hpp"
#include "walk.hpp"

namespace xgm {

namespace {


__device__ __forceinline__ void record_overflow(OverflowLog* log, uint32_t seq, uint32_t a, uint32_t b, uint32_t epoch = 0u) {
  uint32_t slot = atomicAdd(&log->count, 1u) % OverflowLog::kCap;
  log->entry[slot][0] = seq;
  log->entry[slot][1] = a;
  log->entry[slot][2] = b;
  log->entry[slot][3] = epoch;
}

// Copy the staged part of a grammar's table image into LDS, 16 bytes per load
// (all threads of the workgroup call this; a barrier must follow).
__device__ __forceinline__ void stage_tables(const DevTables& tab, unsigned char* smem, int nthreads) {
  uint4* dst = reinterpret_cast<uint4*>(smem);
  for (uint32_t k = threadIdx.x; k < tab.stage_bytes / 16; k += nthreads) dst[k] = tab.image[k];
}
// The same, fetched straight into LDS: all pieces are in flight at once, and no registers hold them.  staged() must come
// before the barrier, and before any wave returns.
__device__ __forceinline__ void stage_tables_async(const DevTables& tab, unsigned char* smem, uint32_t nthreads) {
  const uint32_t n = tab.stage_bytes / 16u, lane = threadIdx.x & 63u;
  for (uint32_t k = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x & ~63u)); k < n; k += nthreads)
    if (k + lane < n)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(tab.image + k + lane),
                                       (__attribute__((address_space(3))) void*)(smem + k * 16u), 16, 0, 0);
}
__device__ __forceinline__ void staged() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The table access of the walk (same answers as CompactTab in walk.hpp) on a
// table image of which bytes [0, lds_end) have been staged by stage_tables().
// Every pointer carries its address space, so that a lookup in a staged
// section is an LDS read and one in an unstaged section a global load (a
// pointer that may point to either would make every access a much slower flat
// one).  Sections are staged whole, so "is it in LDS" is uniform per section.
// kSmallInLds = true: every section in front of the headers is known to be
// staged, so their reads carry no test at all (a lone wave pays for every
// branch of a walk step with its latency).
#define XGM_LDS __attribute__((address_space(3)))
#define XGM_GLOBAL __attribute__((address_space(1)))
#define XGM_CONST __attribute__((address_space(4)))
// kUniform = true: the whole wave asks for the same thing, and what comes back is
// known to be the same for all lanes (see WaveMem): what is not staged is then read
// through the scalar cache.
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
template <bool kSmallInLds, bool kUniform = false>
struct LdsTabT {
  const XGM_LDS unsigned char* lds;     // the staged part of the image
  const XGM_GLOBAL unsigned char* img;  // the whole image
  uint32_t n_near, n_nodes, n_cls, off_shapes, off_targets, off_follow, off_alts, off_hdr, off_first;
  bool cls_lds, shapes_lds, targets_lds, follow_lds, alts_lds;
  __device__ __forceinline__ LdsTabT(const DevTables& t, unsigned char* smem)
      : lds((const XGM_LDS unsigned char*)smem),
        img((const XGM_GLOBAL unsigned char*)reinterpret_cast<const unsigned char*>(t.image)),
        n_near(t.n_near), n_nodes((uint32_t)t.n_nodes), n_cls((uint32_t)t.n_cls), off_shapes(t.off_shapes), off_targets(t.off_targets),
        off_follow(t.off_follow), off_alts(t.off_alts), off_hdr(t.off_hdr), off_first(t.off_first),
        cls_lds(t.lds_end >= 256u), shapes_lds(t.lds_end >= t.off_targets), targets_lds(t.lds_end >= t.off_follow),
        follow_lds(t.lds_end >= t.off_alts), alts_lds(t.lds_end >= t.off_hdr) {}
  // the 32-bit word that holds the bytes at `off`, through the scalar cache
  __device__ __forceinline__ uint32_t scalar_word(uint32_t off) const {
    return *(const XGM_CONST uint32_t*)((const XGM_CONST unsigned char*)(uint64_t)img + (off & ~3u));
  }
  __device__ __forceinline__ uint32_t rd8(uint32_t off, bool in_lds) const {
    if constexpr (kUniform) return (kSmallInLds || in_lds) ? uniform(lds[off]) : (scalar_word(off) >> ((off & 3u) * 8u)) & 0xFFu;
    return (kSmallInLds || in_lds) ? (uint32_t)lds[off] : (uint32_t)img[off];
  }
  __device__ __forceinline__ uint32_t rd16(uint32_t off, bool in_lds) const {
    if constexpr (kUniform)
      return (kSmallInLds || in_lds) ? uniform(*(const XGM_LDS uint16_t*)(lds + off)) : (scalar_word(off) >> ((off & 2u) * 8u)) & 0xFFFFu;
    return (kSmallInLds || in_lds) ? (uint32_t)*(const XGM_LDS uint16_t*)(lds + off)
                                   : (uint32_t)*(const XGM_GLOBAL uint16_t*)(img + off);
  }
  __device__ __forceinline__ uint32_t rd32(uint32_t off, bool in_lds) const {
    if constexpr (kUniform) return (kSmallInLds || in_lds) ? uniform(*(const XGM_LDS uint32_t*)(lds + off)) : scalar_word(off);
    return (kSmallInLds || in_lds) ? *(const XGM_LDS uint32_t*)(lds + off) : *(const XGM_GLOBAL uint32_t*)(img + off);
  }
  __device__ __forceinline__ uint2 header(uint32_t n) const {
    unsigned long long h;  // one 8-byte read
    if constexpr (kUniform) {
      if (n >= n_near) return make_uint2(scalar_word(off_hdr + n * 8u), scalar_word(off_hdr + n * 8u + 4u));
      h = *(const XGM_LDS unsigned long long*)(lds + off_hdr + n * 8u);
      return make_uint2(uniform((uint32_t)h), uniform((uint32_t)(h >> 32)));
    }
    if (!XGM_ANY(n >= n_near)) h = *(const XGM_LDS unsigned long long*)(lds + off_hdr + n * 8u);
    else if (n < n_near) h = *(const XGM_LDS unsigned long long*)(lds + off_hdr + n * 8u);
    else h = *(const XGM_GLOBAL unsigned long long*)(img + off_hdr + (size_t)n * 8u);
    return make_uint2((uint32_t)h, (uint32_t)(h >> 32));
  }
  __device__ __forceinline__ Looked look(uint32_t n, uint32_t c) const {
    const uint2 h = header(n);
    const bool branching = (h.y & 2u) != 0u;
    Looked r{h.x >> 16, c < (h.x & 0xFFu) || c > ((h.x >> 8) & 0xFFu), h.y & 1u, h.y >> 16};
    if (XGM_ANY(branching)) {
      const uint32_t cl = rd8(c, cls_lds);
      const uint32_t si = rd8(off_shapes + (branching ? (h.x & 0xFFFFu) * n_cls : 0u) + cl, shapes_lds);
      const uint32_t a = rd16(off_targets + (branching && si != 0xFFu ? (h.x >> 16) + si : 0u) * 2u, targets_lds);
      r.to = branching ? a : r.to;
      r.none = branching ? si == 0xFFu : r.none;
    }
    return r;
  }
  __device__ __forceinline__ uint32_t alt(uint32_t idx) const { return rd32(off_alts + idx * 4u, alts_lds); }
  __device__ __forceinline__ bool is_final(uint32_t n) const { return header(n).y & 1u; }
  __device__ __forceinline__ bool is_dead_end(uint32_t n) const { return header(n).y & 4u; }
  // can byte c be consumed at node n inside its frame (byte edge, or first byte of a rule it refers to)?
  __device__ __forceinline__ bool can_start(uint32_t n, uint32_t c) const {
    return (*(const XGM_GLOBAL uint32_t*)(img + off_first + ((size_t)n * 8u + (c >> 5)) * 4u) >> (c & 31)) & 1u;
  }
  // can byte c come right after an instance of node n's rule (h = header(n))?
  __device__ __forceinline__ bool can_follow(const uint2& h, uint32_t c) const {
    return (rd32(off_follow + ((h.y >> 16) * 8u + (c >> 5)) * 4u, follow_lds) >> (c & 31)) & 1u;
  }
  // the rule of node n, as the handle of its 256-bit FOLLOW set; is byte c in the set of rule r?
  __device__ __forceinline__ uint32_t follow_of(uint32_t n) const { return header(n).y >> 16; }
  __device__ __forceinline__ uint32_t follows(uint32_t r, uint32_t c) const {
    return (rd32(off_follow + (r * 8u + (c >> 5)) * 4u, follow_lds) >> (c & 31)) & 1u;
  }
};
using LdsTab = LdsTabT<false>;
// are all sections in front of the headers staged?
__device__ __forceinline__ bool small_sections_staged(const DevTables& t) { return t.lds_end >= t.off_hdr; }

// The live frames of a request for the fill kernel: the topmost ones in LDS,
// deeper ones (stacks deeper than the LDS window) in global memory.
struct LiveView {
  const XGM_LDS uint16_t* lds;       // frames [lo, ..) of this stack
  const XGM_GLOBAL uint16_t* glob;   // all frames of this stack
  uint32_t lo;
  __device__ __forceinline__ uint32_t operator[](uint32_t k) const { return k >= lo ? lds[k - lo] : glob[k]; }
};

// ---------------------------------------------------------------- kernel (a)
// Workgroup size of the classify kernels.  A grammar whose staged tables are
// small runs with 256 threads (many workgroups per compute unit, short tails);
// one that needs most of the LDS budget runs with 768, so that two workgroups
// per compute unit still give 6 waves per SIMD.
constexpr int kClassifyThreadsSmall = 256, kClassifyThreadsLarge = 768;
constexpr uint32_t kClassifySmallStage = 32 * 1024;
// Tokens are classified in byte-sorted order, 64 of them (an item) at a time: neighbours mostly share prefixes and
// control flow.  A workgroup of classify_kernel owns up to kClassifyItems items, which its waves draw from a counter in
// LDS, and kClassifyNodes nodes, one for each lane.
// With large tables as many as can be, which are staged for fewer workgroups then (11867-node schema grammar, 151936 tokens,
// with every word written: 533 us with one item per wave, 463 with two, 381 with four or five); with small ones two per
// wave (C/SQL-like grammar, 128256 tokens: 99 us with one, 77 with two, 68 with four; JSON 38, 40, 41).
constexpr int kClassifyNodes = 64, kClassifyItems = 64, kClassifyItemsSmall = 8;
// A run of fewer tokens is not looked at by its prefix: an item of many runs (the tokens that begin with the rarer bytes)
// would take a walk for each of them, one after the other.
constexpr int kPrefixTokens = 16;
constexpr uint32_t kPairNodeBits = 15;  // (XGM_MAX_NODES; the item number takes the bits above)

// What the first byte of a token settles at every node, as bitsets over the nodes: for byte c and the 32 nodes
// of word w, `x` = the node can consume c inside its frame (a walk decides), `y` = it cannot, may end its rule
// here and c can follow that rule in some context (the token leaves the frame at position 0:
// context-dependent), `z` = the same but c follows the rule in no context (context-dependent by section 3.1
// alone, rejected everywhere).  One 16-byte load then tells a thread of the classify kernel what its token's
// first byte means at 32 nodes.
// A wave takes 64 nodes, one in each lane, and 32 byte values.  Bound by the latency of two dependent loads: 3.7 us for JSON's
// 74 nodes and 5.2 for 11867, where a thread that asked 32 nodes one after the other for a byte took 13 and 29.
constexpr int kFirstByteThreads = 512;
__global__ __launch_bounds__(kFirstByteThreads) void first_byte_kernel(DevTables tab, uint32_t n_words, uint4* __restrict__ out) {
  static_assert(kFirstByteThreads / 64 * 32 == 256, "eight waves take all byte values");
  const uint32_t lane = threadIdx.x & 63u, group = uniform(threadIdx.x >> 6), n = blockIdx.x * 64u + lane;
  const unsigned char* img = reinterpret_cast<const unsigned char*>(tab.image);
  uint32_t first = 0u, follow = 0u;
  bool final_ = false;
  if (n < (uint32_t)tab.n_nodes) {
    first = reinterpret_cast<const uint32_t*>(img + tab.off_first)[(size_t)n * 8u + group];
    const uint2 h = reinterpret_cast<const uint2*>(img + tab.off_hdr)[n];
    final_ = h.y & 1u;
    if (final_) follow = reinterpret_cast<const uint32_t*>(img + tab.off_follow)[(h.y >> 16) * 8u + group];
  }
  const uint32_t walks = first, exits = final_ ? ~first & follow : 0u, plain = final_ ? ~first & ~follow : 0u;
  uint4 q = make_uint4(0u, 0u, 0u, 0u);  // lane j: byte value 32 group + j % 32, nodes of the j / 32-th word
  for (uint32_t j = 0; j < 32u; ++j) {
    const unsigned long long x = __ballot((walks >> j) & 1u), y = __ballot((exits >> j) & 1u), z = __ballot((plain >> j) & 1u);
    if ((lane & 31u) == j) q = lane < 32u ? make_uint4((uint32_t)x, (uint32_t)y, (uint32_t)z, 0u) : make_uint4((uint32_t)(x >> 32), (uint32_t)(y >> 32), (uint32_t)(z >> 32), 0u);
  }
  const uint32_t w = blockIdx.x * 2u + (lane >> 5);
  if (w < n_words) out[(size_t)(group * 32u + (lane & 31u)) * n_words + w] = q;
}

// The token of byte-sorted rank r.
struct RankedToken {
  uint4 tk;
  const uint8_t* ext;
  int len;  // 0: no such rank
};
__device__ __forceinline__ RankedToken load_ranked(const DevVocab& voc, int32_t r) {
  RankedToken t{make_uint4(0u, 0u, 0u, 0u), voc.bytes, 0};
  if (r < voc.V) {
    t.tk = voc.tok_by_rank[r];
    t.len = (int)(t.tk.w >> 24);
    if (t.len >= 15) {
      const int32_t id = voc.id_of_rank[r];
      t.ext = voc.bytes + voc.off_by_id[id];
      if (t.len == 255) t.len = (int)(voc.off_by_id[id + 1] - voc.off_by_id[id]);
    }
  }
  return t;
}

// How many bytes two tokens have in common in front of the first that differs, of the 15 that their words hold (behind the end
// of a token these are 0).
__device__ __forceinline__ int same_bytes(const uint4 a, const uint4 b) {
  const uint32_t d0 = a.x ^ b.x, d1 = a.y ^ b.y, d2 = a.z ^ b.z, d3 = (a.w ^ b.w) | 0xFF000000u;
  return (d0 ? __ffs((int)d0) - 1 : d1 ? __ffs((int)d1) + 31 : d2 ? __ffs((int)d2) + 63 : __ffs((int)d3) + 95) / 8;
}

// What a workgroup of the classify kernel keeps beside the tables.
struct ClassifyShared {
  uint32_t next_item, first_pair;
  unsigned long long open[kClassifyItems];  // per item: the nodes at which its tokens have to be walked
  unsigned long long unc[kClassifyItems];   // and those of which it has context-dependent tokens, or may have
};

// Kernel (a), first part: what can be said about an item as a whole.  Lane j of a wave looks at node j.  The first byte
// settles most (item, node) pairs (first_byte_kernel).  Where it does not, the prefix that the item's tokens have in
// common often does: the lane walks the prefix alone, and if no path can consume all of it, every path of every token ends
// where it does, with the same exits from the start frame.  (Where white space may come first - two nodes in ten of a schema
// grammar, and a quarter of the tokens begin with a space - the second byte decides nearly always.)  What is left is
// listed for classify_walks_kernel: 338 K pairs of an 11867-node schema grammar and 151936 tokens, where the first byte
// alone leaves 1.56 M of the 28 M.
// Both kernels write whole words of the rank-space bitsets, 64 tokens of one node, which are lines of their own: only those
// that are not zero (ClassifyArgs::some_acc).  258 us for that grammar (381 with every word written, 451 MB), and 277 us
// for the walks, where one kernel that walked all pairs that the first byte leaves took 1663 us; JSON (128256 tokens) 31 to
// 49 (from run to run) + 34 us, before 163, where a few waves with the walks of whole strings were the last to finish; 32000 tokens 18 + 24, before
// 65; a scripting grammar 64 + 152, before 394; the C/SQL-like grammar, whose identifiers are walked to their ends at a
// hundred nodes, 80 + 940, before 1283.  (Tables fetched straight into LDS as the accept kernel does, and the next item's tokens
// ahead of this one's walk: 258 and 262 us instead of 258, JSON 19.3 and 19.3 instead of 18: the waves wait for each other's
// instructions, not for memory.)
template <class Tab>
__device__ __forceinline__ void classify_body(const Tab& T, ClassifyShared& sm, const DevVocab& voc, const ClassifyArgs& a, int32_t n_items_max) {
  // A workgroup owns a run of up to kClassifyItems items of 64 tokens, and kClassifyNodes nodes; lane j of a wave looks at
  // node j.
  const int32_t item0 = blockIdx.x * n_items_max;
  const int32_t n_items = min(n_items_max, (voc.V + 63) / 64 - item0);
  const int32_t k0 = blockIdx.y * kClassifyNodes, n_own = min(kClassifyNodes, a.n_nodes - k0);
  const uint32_t lane = threadIdx.x & 63u;
  const bool own = (int32_t)lane < n_own;
  const uint32_t own_node = (uint32_t)(a.node0 + k0 + min((int32_t)lane, n_own - 1));
  for (;;) {
    int32_t item = 0;
    if (lane == 0u) item = (int32_t)atomicAdd(&sm.next_item, 1u);
    item = __builtin_amdgcn_readfirstlane(item);
    if (item >= n_items) break;
    const RankedToken t = load_ranked(voc, (item0 + item) * 64 + (int32_t)lane);
    const uint32_t c0 = t.tk.x & 0xFFu;
    const bool too_long = __ballot(t.len > kMaxTokenLen) != 0ull;  // (the walk refuses such a token)
    unsigned long long keep_u = 0ull, keep_p = 0ull, open = 0ull;
    // The tokens come in byte-sorted order: those that begin with the same byte (all of them, in most items) lie side
    // by side and share a prefix.
    for (unsigned long long left = __ballot(t.len > 0); left;) {
      const int first = __ffsll((long long)left) - 1;
      const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)c0, first);
      const unsigned long long run = __ballot(t.len > 0 && c0 == c);
      left &= ~run;
      // what the first byte settles: if the node cannot consume it inside its frame, the token is rejected - or, at a
      // node where the rule may end, leaves the frame at position 0
      const uint4 fb = a.first_byte[(size_t)c * a.n_words + (own_node >> 5)];
      if ((fb.y >> (own_node & 31u)) & 1u) keep_u |= run;
      if ((fb.z >> (own_node & 31u)) & 1u) keep_p |= run;
      bool walk = own && ((fb.x >> (own_node & 31u)) & 1u);
      const unsigned long long needs = __ballot(walk);
      // what the common prefix settles: where no path consumes all of it, every token of the run fares as the prefix does
      if (__popcll(run) >= kPrefixTokens && (needs & (needs - 1ull)) && !too_long) {
        const int last = 63 - __clzll((long long)run);
        auto of = [&](uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); };
        auto token = [&](int l) { return make_uint4(of(t.tk.x, l), of(t.tk.y, l), of(t.tk.z, l), of(t.tk.w, l)); };
        const uint4 pre = token(first);
        const int shortest = (int)min(of((uint32_t)t.len, first), of((uint32_t)t.len, last));
        const int n = min(same_bytes(pre, token(last)), shortest);
        if (n >= 2 && walk) {
          const int res = walk_token<true>(T, pre, voc.bytes, n, own_node, (const uint16_t*)nullptr, 1u, nullptr, T.follow_of(own_node));
          if (res == kUncertain) keep_u |= run;
          if (res == kUncertainPlain) keep_p |= run;
          walk = res == kAccept || res == kOverflow;
        }
      }
      open |= __ballot(walk);
    }
    const unsigned long long unc = __ballot(own && keep_u != 0ull) | open;
    if (lane == 0u) { sm.open[item] = open; sm.unc[item] = unc; }
    if (own && !((open >> lane) & 1ull)) {
      const size_t at = (size_t)(k0 + (int32_t)lane) * voc.WR + (uint32_t)((item0 + item) * 2);  // an even word: 8-byte aligned
      if (!a.some_acc) *reinterpret_cast<uint2*>(a.acc_rank + at) = make_uint2(0u, 0u);
      if (!a.some_unc || keep_u) *reinterpret_cast<uint2*>(a.unc_rank + at) = make_uint2((uint32_t)keep_u, (uint32_t)(keep_u >> 32));
      if (a.plain_rank) *reinterpret_cast<uint2*>(a.plain_rank + at) = make_uint2((uint32_t)keep_p, (uint32_t)(keep_p >> 32));
      if (keep_p) atomicAdd(&a.plain_count[own_node], (uint32_t)__popcll(keep_p));
    }
  }
  __syncthreads();
  // which words of the nodes' rows there are
  if (a.some_acc)
    for (int32_t t = (int32_t)threadIdx.x; t < n_own * (n_items_max / 8); t += (int32_t)blockDim.x) {
      const int32_t j = t / (n_items_max / 8), eight = t % (n_items_max / 8);
      uint32_t acc = 0u, unc = 0u;
#pragma unroll
      for (int32_t i = 0; i < 8; ++i) {
        const int32_t item = eight * 8 + i;
        if (item < n_items) {
          acc |= (uint32_t)((sm.open[item] >> j) & 1ull) << i;
          unc |= (uint32_t)((sm.unc[item] >> j) & 1ull) << i;
        }
      }
      const size_t at = (size_t)(k0 + j) * some_stride(voc) + (uint32_t)(item0 / 8 + eight);
      a.some_acc[at] = (uint8_t)acc;
      a.some_unc[at] = (uint8_t)unc;
    }
  // the (item, node) pairs that are left are listed for classify_walks_kernel
  const uint32_t n_open = (int32_t)lane < n_items ? (uint32_t)__popcll(sm.open[lane]) : 0u;
  uint32_t upto = n_open;  // pairs of the items up to the lane's
#pragma unroll
  for (uint32_t d = 1; d < 64u; d <<= 1) {
    const uint32_t v = __shfl_up(upto, d, 64);
    if (lane >= d) upto += v;
  }
  if (threadIdx.x == 63u) sm.first_pair = upto ? atomicAdd(a.n_pairs, upto) : 0u;
  __syncthreads();
  for (int32_t item = (int32_t)uniform(threadIdx.x >> 6); item < n_items; item += (int32_t)(blockDim.x >> 6)) {
    const unsigned long long open = sm.open[item];
    const uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)(upto - n_open), item);
    if ((open >> lane) & 1ull)
      a.pairs[sm.first_pair + before + (uint32_t)__popcll(open & ((1ull << lane) - 1ull))] = (uint32_t)(item0 + item) << kPairNodeBits | (uint32_t)(k0 + (int32_t)lane);
  }
}

template <int kClassifyThreads>
__global__ __launch_bounds__(kClassifyThreads) void classify_kernel(DevTables tab, DevVocab voc, ClassifyArgs a, int32_t n_items) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ ClassifyShared sm;
  if (threadIdx.x == 0) sm.next_item = 0u;
  stage_tables(tab, smem, kClassifyThreads);
  __syncthreads();
  if (small_sections_staged(tab)) classify_body(LdsTabT<true>(tab, smem), sm, voc, a, n_items);
  else classify_body(LdsTab(tab, smem), sm, voc, a, n_items);
}

// Second part: the pairs that are left, a wave for each; lane j walks token j of the item.  Neighbours in the list (the
// nodes of one item) go to different workgroups, and with several workgroups per place on the chip (small tables) the
// later ones even out what the first ones got: C/SQL-like grammar 1032 us with 4096 workgroups, 1150 with 2048, 1278 with
// 1024.  Large tables are staged once per place: 365 us for the schema grammar above with 512, 400 with 1024.
// Bound by instruction issue: a step takes some 160 instructions.
constexpr uint32_t kWalkBlocksSmall = 4096, kWalkBlocksLarge = 512;
template <int kClassifyThreads>
__global__ __launch_bounds__(kClassifyThreads) void classify_walks_kernel(DevTables tab, DevVocab voc, ClassifyArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const uint32_t n_pairs = *a.n_pairs;
  if (blockIdx.x >= n_pairs) return;
  stage_tables(tab, smem, kClassifyThreads);
  __syncthreads();
  auto body = [&](const auto& T) {
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t q = uniform(threadIdx.x >> 6) * gridDim.x + blockIdx.x; q < n_pairs; q += gridDim.x * (kClassifyThreads / 64)) {
      const uint32_t pair = uniform(a.pairs[q]);
      const uint32_t item = pair >> kPairNodeBits, k = pair & ((1u << kPairNodeBits) - 1u), node = (uint32_t)a.node0 + k;
      const int32_t r = (int32_t)(item * 64u + lane);
      const RankedToken t = load_ranked(voc, r);
      int res = kReject;
      if (t.len > 0) {
        res = walk_token<true>(T, t.tk, t.ext, t.len, node, (const uint16_t*)nullptr, 1u, nullptr, T.follow_of(node));
        if (res == kOverflow) { record_overflow(a.log, a.seq, k, (uint32_t)r); res = kReject; }
      }
      const unsigned long long acc = __ballot(res == kAccept), unc = __ballot(res == kUncertain), plain = __ballot(res == kUncertainPlain);
      if (lane == 0u) {
        const size_t at = (size_t)k * voc.WR + item * 2u;
        *reinterpret_cast<uint2*>(a.acc_rank + at) = make_uint2((uint32_t)acc, (uint32_t)(acc >> 32));
        *reinterpret_cast<uint2*>(a.unc_rank + at) = make_uint2((uint32_t)unc, (uint32_t)(unc >> 32));
        if (a.plain_rank) *reinterpret_cast<uint2*>(a.plain_rank + at) = make_uint2((uint32_t)plain, (uint32_t)(plain >> 32));
        if (plain) atomicAdd(&a.plain_count[node], (uint32_t)__popcll(plain));
      }
    }
  };
  if (small_sections_staged(tab)) body(LdsTabT<true>(tab, smem));
  else body(LdsTab(tab, smem));
}

// Many nodes of a grammar have the same accepted bitset (the inside of a string is
// the inside of a string wherever it occurs), so the cache keeps every distinct
// row once.  The digest only proposes which rows might be equal: the position-
// dependent mix of every word (the finalizer of splitmix64) is summed over the
// row; equality is then checked word for word.
constexpr int kRowThreads = 256;
__device__ __forceinline__ unsigned long long mix64(unsigned long long x) {
  x ^= x >> 30; x *= 0xBF58476D1CE4E5B9ull;
  x ^= x >> 27; x *= 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}
constexpr int kMaxSegs = 128;  // segments of the largest vocabulary (XGM_MAX_VOCAB / kSegTokens), rounded up

// The words of a node's rank-space row (64 tokens each) that are there and not zero, 64 items at a time: each(first item of
// the 64, the lane's word of them or 0).  All lanes of a wave call this together; wave `part` of `parts` takes every
// parts-th 64 items.
typedef unsigned long long u64;
__device__ __forceinline__ u64 word_of_lane(u64 v, int lane) {
  return (u64)(uint32_t)__builtin_amdgcn_readlane((int)v, lane) | (u64)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), lane) << 32;
}
template <class Each>
__device__ __forceinline__ void for_each_word(const DevVocab& voc, const uint32_t* __restrict__ rows, const uint8_t* __restrict__ some,
                                              size_t node, uint32_t part, uint32_t parts, const Each& each) {
  const uint32_t lane = threadIdx.x & 63u, n_items = (uint32_t)voc.WR / 2u, n_blocks = (n_items + 63u) / 64u;
  const u64* const row = reinterpret_cast<const u64*>(rows) + node * n_items;
  const u64* const bits = reinterpret_cast<const u64*>(some + node * some_stride(voc));
  for (uint32_t b0 = 0; b0 < n_blocks; b0 += 64u) {
    const uint32_t b = b0 + lane;
    u64 mine = 0ull;
    if (b < n_blocks) {
      mine = bits[b];
      if (b * 64u + 64u > n_items) mine &= (1ull << (n_items - b * 64u)) - 1ull;
    }
    // four at a time, so that their words are fetched together
    for (u64 left = __ballot(mine != 0ull && b % parts == part); left;) {
      u64 word[4];
      uint32_t first[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        word[q] = 0ull;
        first[q] = 0u;
        if (left) {
          const int j = __ffsll((long long)left) - 1;
          left &= left - 1ull;
          first[q] = (b0 + (uint32_t)j) * 64u;
          if ((word_of_lane(mine, j) >> lane) & 1ull) word[q] = row[first[q] + lane];
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (__ballot(word[q] != 0ull)) each(first[q], word[q]);
    }
  }
}
// The tokens of such words: each(whether the lane has one, its id, how many there are in the wave's lanes before it and in
// all).  With few tokens per item every lane takes those of its own word, with many all lanes those of one word after the
// other; either way several ids are fetched at once.  ORDERED: in byte-sorted order.
template <bool ORDERED, class Each>
__device__ __forceinline__ void for_each_token(const DevVocab& voc, uint32_t item0, u64 word, const Each& each) {
  constexpr int kFew = 4, kAtOnce = 8;
  const uint32_t lane = threadIdx.x & 63u;
  const u64 below = (1ull << lane) - 1ull;
  if (__ballot(__popcll(word) > (ORDERED ? 1 : kFew)) == 0ull) {
    uint32_t id[kFew];
    bool has[kFew];
#pragma unroll
    for (int q = 0; q < (ORDERED ? 1 : kFew); ++q) {
      has[q] = word != 0ull;
      id[q] = has[q] ? (uint32_t)voc.id_of_rank[(item0 + lane) * 64u + (uint32_t)__ffsll((long long)word) - 1u] : 0u;
      word &= word - 1ull;
    }
#pragma unroll
    for (int q = 0; q < (ORDERED ? 1 : kFew); ++q) {
      const u64 all = __ballot(has[q]);
      if (all) each(has[q], id[q], (uint32_t)__popcll(all & below), (uint32_t)__popcll(all));
    }
    return;
  }
  for (u64 left = __ballot(word != 0ull); left;) {
    u64 x[kAtOnce];
    uint32_t id[kAtOnce];
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) {
      x[q] = 0ull;
      id[q] = 0u;
      if (left) {
        const int j = __ffsll((long long)left) - 1;
        left &= left - 1ull;
        x[q] = word_of_lane(word, j);
        id[q] = (uint32_t)voc.id_of_rank[min((int32_t)((item0 + (uint32_t)j) * 64u + lane), voc.V - 1)];
      }
    }
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q)
      if (x[q]) each((bool)((x[q] >> lane) & 1ull), id[q], (uint32_t)__popcll(x[q] & below), (uint32_t)__popcll(x[q]));
  }
}
// What the lanes of a wave have written to LDS in front of this is there for all of them behind it (the hardware keeps a wave's
// LDS operations in order: this is for the compiler).  All lanes of a wave call it together.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// A barrier for what is in LDS: __syncthreads() also waits until what the threads have stored to global memory has got there.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
  for (uint32_t d = 1; d < 64u; d <<= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// The statistics of every node's rows, a workgroup per node: how many tokens it accepts and, if it lists them (a node with
// few of them has no bitset row), how many in each segment; how many are context-dependent.  Nodes with a bitset row are
// collected for bitset_rows_kernel.  Together 62 us for the 11867-node schema grammar and 151936 tokens, where a kernel that
// went through whole rows took 496 (902 MB); 33 for JSON and 128256 tokens, before 53.  (512 threads: 57 us for this kernel
// instead of 30, there are too many nodes that have hardly anything.)
constexpr int kNodeThreads = 256;
__global__ __launch_bounds__(kNodeThreads) void row_stats_kernel(DevVocab voc, RankRows a) {
  __shared__ uint32_t seg[kMaxSegs];
  __shared__ uint32_t sums[2];
  const uint32_t wave = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63u;
  const size_t node = blockIdx.x;
  if (threadIdx.x < kMaxSegs) seg[threadIdx.x] = 0u;
  if (threadIdx.x < 2u) sums[threadIdx.x] = 0u;
  __syncthreads();
  uint32_t acc = 0u, unc = 0u;
  for_each_word(voc, a.acc_rank, a.some_acc, node, wave, kNodeThreads / 64, [&](uint32_t, u64 x) { acc += (uint32_t)__popcll(x); });
  for_each_word(voc, a.unc_rank, a.some_unc, node, wave, kNodeThreads / 64, [&](uint32_t, u64 x) { unc += (uint32_t)__popcll(x); });
  acc = wave_sum(acc);
  unc = wave_sum(unc);
  if (lane == 0u && acc) atomicAdd(&sums[0], acc);
  if (lane == 0u && unc) atomicAdd(&sums[1], unc);
  __syncthreads();
  const uint32_t total = sums[0];
  if (threadIdx.x == 0u) {
    a.acc_counts[node] = total;
    a.unc_counts[node] = sums[1];
    if (!kept_as_list(total, voc.W)) a.bitset_nodes[atomicAdd(a.n_bitset_nodes, 1u)] = (uint32_t)node;
  }
  if (acc && kept_as_list(total, voc.W))
    for_each_word(voc, a.acc_rank, a.some_acc, node, wave, kNodeThreads / 64, [&](uint32_t item0, u64 x) {
      for_each_token<false>(voc, item0, x, [&](bool has, uint32_t id, uint32_t, uint32_t) { if (has) atomicAdd(&seg[id / (uint32_t)kSegTokens], 1u); });
    });
  __syncthreads();
  if ((int32_t)threadIdx.x < voc.n_seg) a.seg_counts[node * voc.n_seg + threadIdx.x] = seg[threadIdx.x];
}

// The accepted rows of the nodes that keep a bitset, in id space (bit id_of_rank[r] of the output = bit r of the row), and
// their digests.  A workgroup builds a row in LDS, of the rarer kind of bit: a row with few set bits starts as zeros
// and gets its set bits, one with many as ones and gets its zeros.
constexpr int kBitsetThreads = 512;
__global__ __launch_bounds__(kBitsetThreads) void bitset_rows_kernel(DevVocab voc, RankRows a, uint32_t* __restrict__ acc_id,
                                                                  unsigned long long* __restrict__ digest) {
  extern __shared__ __align__(16) unsigned char smem[];
  uint32_t* row = reinterpret_cast<uint32_t*>(smem);  // [W]
  __shared__ unsigned long long part[kBitsetThreads / 64];
  const uint32_t n = *a.n_bitset_nodes, n_items = (uint32_t)voc.WR / 2u;
  const uint32_t tail = (voc.V & 31) ? ((1u << (voc.V & 31)) - 1u) : 0xFFFFFFFFu;  // valid bits of the last word
  for (uint32_t k = blockIdx.x; k < n; k += gridDim.x) {
    const size_t node = a.bitset_nodes[k];
    const bool full = a.acc_counts[node] * 2u > (uint32_t)voc.V;
    __syncthreads();
    for (int32_t w = threadIdx.x; w < voc.W; w += kBitsetThreads) row[w] = !full ? 0u : w == voc.W - 1 ? tail : 0xFFFFFFFFu;
    __syncthreads();
    for (uint32_t item0 = uniform(threadIdx.x >> 6) * 64u; item0 < n_items; item0 += kBitsetThreads) {
      const uint32_t item = item0 + (threadIdx.x & 63u);
      u64 x = 0ull;
      if (item < n_items) {
        if ((a.some_acc[node * some_stride(voc) + item / 8u] >> (item & 7u)) & 1u) x = reinterpret_cast<const u64*>(a.acc_rank)[node * n_items + item];
        if (full) {
          x = ~x;
          const int32_t left = voc.V - (int32_t)item * 64;  // ranks from V on do not exist
          if (left < 64) x &= (1ull << left) - 1ull;
        }
      }
      for_each_token<false>(voc, item0, x, [&](bool has, uint32_t id, uint32_t, uint32_t) {
        if (!has) return;
        if (full) atomicAnd(&row[id >> 5], ~(1u << (id & 31)));
        else atomicOr(&row[id >> 5], 1u << (id & 31));
      });
    }
    __syncthreads();
    unsigned long long h = 0ull;
    for (int32_t w = threadIdx.x; w < voc.W; w += kBitsetThreads) {
      const uint32_t x = row[w];
      acc_id[node * voc.W + w] = x;
      h += mix64(((unsigned long long)(uint32_t)w << 32 | x) + 0x9E3779B97F4A7C15ull);
    }
#pragma unroll
    for (uint32_t d = 32; d > 0; d >>= 1) h += __shfl_down(h, d, 64);
    if ((threadIdx.x & 63u) == 0) part[threadIdx.x >> 6] = h;
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned long long t = 0ull;
      for (int q = 0; q < kBitsetThreads / 64; ++q) t += part[q];
      digest[node] = t;
    }
  }
}

// The context-dependent tokens of the nodes with a place in the base lists (first[n] != kNoKey), a workgroup per node; those
// of 4096 neighbours in byte-sorted order stay in that order (the walks of neighbouring lanes then share prefixes, as in
// the classify kernels).  Most nodes have none; a workgroup is large for the few with thousands, which the launch waits for:
// 37 us for the 11867-node schema grammar (151936 tokens), 23 for JSON and 33 for the C/SQL-like grammar (128256), with 256
// threads 61, 43 and 90; lists of whole rows took 68, 18 and 50.
constexpr int kBaseListThreads = 1024;
__global__ __launch_bounds__(kBaseListThreads) void base_lists_kernel(DevVocab voc, RankRows a, const uint32_t* __restrict__ first,
                                                                  uint32_t* __restrict__ ids, uint16_t* __restrict__ nodes) {
  __shared__ uint32_t next;
  const size_t node = blockIdx.x;
  const uint32_t lane = threadIdx.x & 63u, begin = first[node];
  if (begin == kNoKey) return;
  if (threadIdx.x == 0u) next = begin;
  __syncthreads();
  for_each_word(voc, a.unc_rank, a.some_unc, node, uniform(threadIdx.x >> 6), kBaseListThreads / 64, [&](uint32_t item0, u64 x) {
    uint32_t at = 0u;
    const uint32_t total = wave_sum((uint32_t)__popcll(x));
    if (lane == 0u) at = atomicAdd(&next, total);
    at = uniform(at);
    for_each_token<true>(voc, item0, x, [&](bool has, uint32_t id, uint32_t before, uint32_t n) {
      if (has) {
        ids[at + before] = id;
        nodes[at + before] = (uint16_t)node;
      }
      at += n;
    });
  });
}
// The level-0 lists: the accepted tokens of the nodes that list them, by segment.  A workgroup per node.
__global__ __launch_bounds__(kNodeThreads) void level0_lists_kernel(DevVocab voc, RankRows a, const uint32_t* __restrict__ key_off,
                                                                    uint32_t* __restrict__ entries) {
  __shared__ uint32_t next[kMaxSegs];
  const size_t node = blockIdx.x;
  const uint32_t acc = a.acc_counts[node];
  if (acc == 0u || !kept_as_list(acc, voc.W)) return;
  if ((int32_t)threadIdx.x < voc.n_seg) next[threadIdx.x] = key_off[node * voc.n_seg + threadIdx.x];
  __syncthreads();
  for_each_word(voc, a.acc_rank, a.some_acc, node, uniform(threadIdx.x >> 6), kNodeThreads / 64, [&](uint32_t item0, u64 x) {
    for_each_token<false>(voc, item0, x, [&](bool has, uint32_t id, uint32_t, uint32_t) {
      if (has) entries[atomicAdd(&next[id / (uint32_t)kSegTokens], 1u)] = id;
    });
  });
}

// The same from whole rows, for builds that keep what the sparse ones do without (batches of nodes; the context-dependent
// bitsets): bit id_of_rank[r] of the output = bit r of the input.  One workgroup per node builds
// the node's two id-space rows in LDS.  Rows are nearly empty (most nodes reject nearly every token) or nearly
// full (the inside of a string), so only the rarer kind of bit is moved: a row with few set bits starts as zeros
// and gets its set bits, one with many starts as ones and gets its zeros.  With the rows still in LDS the
// workgroup also takes their statistics (the outputs may be null, all together): set bits of the first row per segment,
// its digest, and the number of set bits of both.
__global__ __launch_bounds__(kRowThreads) void permute_kernel(DevVocab voc, const uint32_t* __restrict__ a_rank,
                                                              const uint32_t* __restrict__ b_rank,
                                                              uint32_t* a_id, uint32_t* b_id,  // (may be the same row)
                                                              uint32_t* __restrict__ seg_counts,
                                                              unsigned long long* __restrict__ digest,
                                                              uint32_t* __restrict__ a_counts, uint32_t* __restrict__ b_counts) {
  extern __shared__ __align__(16) unsigned char smem[];
  uint32_t* rows = reinterpret_cast<uint32_t*>(smem);  // [2][W]
  __shared__ uint32_t set_bits[2];
  __shared__ unsigned long long part[kRowThreads / 64];
  __shared__ uint32_t seg[kMaxSegs];
  const size_t node = blockIdx.x;
  const uint32_t* in[2] = {a_rank + node * voc.WR, b_rank + node * voc.WR};
  if (threadIdx.x < 2) set_bits[threadIdx.x] = 0u;
  if (threadIdx.x < kMaxSegs) seg[threadIdx.x] = 0u;
  __syncthreads();
  uint32_t c0 = 0u, c1 = 0u;
  for (int32_t k = threadIdx.x; k < voc.WR; k += kRowThreads) {
    c0 += __popc(in[0][k]);
    c1 += __popc(in[1][k]);
  }
  if (c0) atomicAdd(&set_bits[0], c0);
  if (c1) atomicAdd(&set_bits[1], c1);
  __syncthreads();
  const bool full[2] = {set_bits[0] * 2u > (uint32_t)voc.V, set_bits[1] * 2u > (uint32_t)voc.V};
  const uint32_t tail = (voc.V & 31) ? ((1u << (voc.V & 31)) - 1u) : 0xFFFFFFFFu;  // valid bits of the last word
  for (int32_t w = threadIdx.x; w < voc.W; w += kRowThreads) {
    const uint32_t ones = (w == voc.W - 1) ? tail : 0xFFFFFFFFu;
    rows[w] = full[0] ? ones : 0u;
    rows[voc.W + w] = full[1] ? ones : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    uint32_t* row = rows + (size_t)which * voc.W;
    for (int32_t k = threadIdx.x; k < voc.WR; k += kRowThreads) {
      uint32_t x = in[which][k];
      if (full[which]) {
        x = ~x;
        const int32_t left = voc.V - k * 32;  // ranks from V on do not exist
        if (left < 32) x &= left > 0 ? ((1u << left) - 1u) : 0u;
      }
      while (x) {
        const uint32_t b = (uint32_t)__ffs((int)x) - 1u;
        x &= x - 1u;
        const uint32_t id = (uint32_t)voc.id_of_rank[k * 32 + (int32_t)b];
        if (full[which]) atomicAnd(&row[id >> 5], ~(1u << (id & 31)));
        else atomicOr(&row[id >> 5], 1u << (id & 31));
      }
    }
  }
  __syncthreads();
  unsigned long long h = 0ull;
  for (int32_t w = threadIdx.x; w < voc.W; w += kRowThreads) {
    const uint32_t x = rows[w];
    a_id[node * voc.W + w] = x;
    b_id[node * voc.W + w] = rows[voc.W + w];
    if (seg_counts && x) atomicAdd(&seg[w / kSegWords], (uint32_t)__popc(x));
    h += mix64(((unsigned long long)(uint32_t)w << 32 | x) + 0x9E3779B97F4A7C15ull);
  }
  if (!seg_counts) return;
#pragma unroll
  for (uint32_t d = 32; d > 0; d >>= 1) h += __shfl_down(h, d, 64);
  if ((threadIdx.x & 63u) == 0) part[threadIdx.x >> 6] = h;
  __syncthreads();
  if ((int32_t)threadIdx.x < voc.n_seg) seg_counts[node * voc.n_seg + threadIdx.x] = kept_as_list(set_bits[0], voc.W) ? seg[threadIdx.x] : 0u;
  if (threadIdx.x == 0) {
    unsigned long long t = 0ull;
    for (int k = 0; k < kRowThreads / 64; ++k) t += part[k];
    digest[node] = t;
    a_counts[node] = set_bits[0];
    b_counts[node] = set_bits[1];
  }
}

// Bitset rows (row_words words each) -> lists through cursors.  One workgroup per (segment, row); a thread
// takes four words; a wave reserves room for all its tokens with one atomic.
constexpr int kListThreads = kSegWords / 4;
__global__ __launch_bounds__(kListThreads) void rows_to_lists_kernel(const uint32_t* __restrict__ rows, int32_t row_words,
                                                                     const uint32_t* __restrict__ cursor_of, int32_t per_row,
                                                                     uint32_t* __restrict__ cursor, uint32_t* __restrict__ out,
                                                                     uint16_t* __restrict__ out_row, int32_t row0) {
  const size_t r = blockIdx.y;
  const uint32_t key = cursor_of[r];
  if (key == kNoKey) return;
  const int32_t s = blockIdx.x;
  const int32_t w0 = s * kSegWords + (int32_t)threadIdx.x * 4;
  uint32_t bits[4];
  uint32_t n = 0u;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    bits[k] = w0 + k < row_words ? rows[r * (size_t)row_words + w0 + k] : 0u;
    n += __popc(bits[k]);
  }
  // exclusive prefix of n over the wave, and the wave's total
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t incl = n;
#pragma unroll
  for (uint32_t d = 1; d < 64u; d <<= 1) {
    const uint32_t v = __shfl_up(incl, d, 64);
    if (lane >= d) incl += v;
  }
  const uint32_t total = __shfl(incl, 63, 64);
  if (total == 0u) return;
  uint32_t base = 0u;
  if (lane == 0) base = atomicAdd(&cursor[(size_t)key * per_row + (per_row > 1 ? s : 0)], total);
  base = __shfl(base, 0, 64);
  uint32_t pos = base + incl - n;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint32_t x = bits[k];
    while (x) {
      const uint32_t b = __ffs(x) - 1;
      x &= x - 1;
      if (out_row) out_row[pos] = (uint16_t)(row0 + (int32_t)r);
      out[pos++] = (uint32_t)(w0 + k) * 32u + b;
    }
  }
}

// the first 15 bytes, the length and the remaining bytes of token `id`
struct TokenRef {
  uint4 tk;
  const uint8_t* ext;
  int len;
};
__device__ __forceinline__ TokenRef load_token(const DevVocab& voc, int32_t id) {
  TokenRef t;
  t.tk = voc.tok_by_id[id];
  t.len = (int)(t.tk.w >> 24);
  t.ext = voc.bytes;
  if (t.len >= 15) {
    t.ext = voc.bytes + voc.off_by_id[id];
    if (t.len == 255) t.len = (int)(voc.off_by_id[id + 1] - voc.off_by_id[id]);
  }
  return t;
}

// ---- The per-context lists (section 3.2 per call site; see DevCache), from the base lists: the
// context-dependent (node, token) pairs.  Kernels, tables staged as in the classify kernel:
//   exit_positions_kernel  one thread per pair: the token is walked once more from the node to find the
//                          positions at which it leaves the node's frame;
//   context_open_kernel    which contexts of the node's rule have to be looked at for 64 pairs at all;
//   context_level1_kernel  one lane per (pair, such a context): the rest of the token is
//                          walked from the context node with nothing known below but the frames that this
//                          context forces.  Accepted there: an entry of the (node, context) list.  Leaves all
//                          those frames: a record for the next level;
//   context_deeper_kernel  for level 2, 3, ...: one thread per (record of the level above, a few contexts of
//                          the rule of the last frame left): the same one level further down; what leaves the
//                          frames of the last level becomes a walk entry.
// A frame with a single possible frame below it takes no level of its own: the precedence levels of an
// expression grammar (a dozen frames with one context each between an identifier and the call or bracket it
// stands in) are one level.  With levels of one frame the fill had to walk 48 K tokens over those frames where
// an identifier ends in the C/SQL-like grammar (128256 tokens, one row: 950 us).
// Most (pair, context) combinations end at the first byte of the rest, which the context node cannot
// take.  The walking ones but the first run twice: first they count the entries of every (key, segment), then,
// with the offsets made from the counts, they write them.
constexpr int kContextThreads = 768;
constexpr uint32_t kContextsPerThread = 8;

__global__ __launch_bounds__(kContextThreads) void exit_positions_kernel(DevTables tab, DevVocab voc, ContextListArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  stage_tables(tab, smem, kContextThreads);
  __syncthreads();
  auto body = [&](const auto& T) {
    const uint32_t e = blockIdx.x * kContextThreads + threadIdx.x;
    if (e >= a.total) return;
    const uint32_t node = a.base_node[e];
    const TokenRef t = load_token(voc, (int32_t)a.base_ids[e]);
    uint32_t x = 0u;
    const int res = walk_token<true, true>(T, t.tk, t.ext, t.len, node, (const uint16_t*)nullptr, 1u, nullptr, T.follow_of(node), 0, &x);
    a.exits[e] = res == kOverflow ? 0x80000000u : x;
  };
  if (small_sections_staged(tab)) body(LdsTabT<true>(tab, smem));
  else body(LdsTab(tab, smem));
}

// How an entry reaches its list, counting or writing.
template <bool WRITE>
struct ListSink {
  const DevVocab& voc;
  const ContextListArgs& a;
  // One entry for list `key`.  The lanes of a wave that get here together mostly add to the same list (they hold
  // neighbouring tokens of one node and look at the same context): they are served by one atomic per
  // distinct (list, segment, accepted or not) among them instead of one each - atomics on one address queue up.
  __device__ __forceinline__ void emit(uint32_t id, uint32_t key, uint32_t kind, uint32_t pos) const {
    const uint32_t slot = key * (uint32_t)voc.n_seg + id / (uint32_t)kSegTokens;
    const uint32_t tag = (slot << 1) | (kind == kEntryAccepted ? 0u : 1u);
    const uint32_t lane = threadIdx.x & 63u;
    for (bool pending = true; pending;) {
      const uint32_t lead = __builtin_amdgcn_readfirstlane(tag);
      const bool mine = tag == lead;
      const unsigned long long peers = __ballot(mine);
      if (mine) {
        const uint32_t n = (uint32_t)__popcll(peers), rank = (uint32_t)__popcll(peers & ((1ull << lane) - 1ull));
        const int first = __ffsll((long long)peers) - 1;
        if (!WRITE) {
          if (rank == 0u) atomicAdd(&a.counts[slot], n);
        } else {
          uint32_t base = 0u;
          if (rank == 0u) base = kind == kEntryAccepted ? atomicAdd(&a.front[slot], n) : atomicSub(&a.back[slot], n) - n;
          base = __shfl(base, first, 64);
          a.entries[base + rank] = id | (pos << kEntryPosShift) | (kind << kEntryKindShift);
        }
        pending = false;
      }
    }
  }
};
__device__ __forceinline__ uint32_t outcome_code(uint32_t kind, uint32_t pos) { return (kind + 1u) | (pos << 8); }

// What the list kernels share: the token of one pair, how its entries reach the lists, and one (pair,
// context) step: the rest of the token after it has left the frame above at the positions `ex`, walked
// from context node r.
template <bool WRITE, class Tab>
struct ContextWork {
  const Tab& T;
  const DevVocab& voc;
  const ContextListArgs& a;
  uint32_t e, id;
  TokenRef t;
  // (`outcome`, if not null, also receives what was emitted, as a code; `lds_counts`, if not null, are the
  // workgroup's own counters per segment for this list: the entry is then only counted there)
  __device__ __forceinline__ void emit(uint32_t key, uint32_t kind, uint32_t pos, uint32_t* outcome,
                                       uint32_t* lds_counts) const {
    if (!WRITE && kind != kEntryAccepted) {  // (how many walk entries the cache has, up to kManyWalks)
      const unsigned long long peers = __ballot(true);
      uint32_t* const total = a.res_count + kCtxLevels;
      if ((uint32_t)__ffsll((long long)peers) - 1u == (threadIdx.x & 63u) && *(volatile uint32_t*)total < kManyWalks)
        atomicAdd(total, (uint32_t)__popcll(peers));
    }
    if (!WRITE && lds_counts) atomicAdd(&lds_counts[id / (uint32_t)kSegTokens], 1u);
    else ListSink<WRITE>{voc, a}.emit(id, key, kind, pos);
    if (outcome) *outcome = outcome_code(kind, pos);
  }
  // can the rest of the token from position k on do anything at all at node r?  (its first byte is
  // consumed there, or r may end its rule in front of a byte that can follow the rule)
  __device__ __forceinline__ bool plausible(uint32_t r, uint32_t k) const {
    const uint32_t c = token_byte(t.tk, t.ext, (int)k);
    if (T.can_start(r, c)) return true;
    const uint2 h = T.header(r);
    return (h.y & 1u) && T.can_follow(h, c);
  }
  // Level `level` (1-based), context node r, whose key is `key_local` among its level's keys.  `single`:
  // every frame so far was left at exactly one position.
  __device__ __forceinline__ void step(uint32_t level, uint32_t r, uint32_t key_local, uint32_t ex, bool single,
                                       uint32_t* outcome = nullptr, uint32_t* lds_counts = nullptr) const {
    const uint32_t key = a.key0[level - 1u] + key_local;
    if (ex & 0x80000000u) { emit(key, kEntryWalkTop, 0u, outcome, lds_counts); return; }
    bool accepted = false, over = false, known = false;
    uint4 info = make_uint4(0u, 0u, 0u, 0u);  // the frames that r forces below itself
    uint32_t ex_next = 0u, n_res = 0u;
    for (uint32_t m = ex; m != 0u && !accepted; m &= m - 1u) {
      const uint32_t k = __ffs(m) - 1u;
      if (!plausible(r, k)) continue;
      if (!known) { info = a.rule_info[T.header(r).y >> 16]; known = true; }
      uint32_t x = 0u;
      const int res = walk_token<true, true>(T, t.tk, t.ext, t.len, r, (const XGM_GLOBAL uint16_t*)(a.forced_node + info.x), info.y + 1u,
                                             nullptr, info.z, (int)k, &x);
      if (res == kAccept) accepted = true;
      else if (res == kOverflow) over = true;
      else if (res == kUncertain) { ex_next |= x; ++n_res; }
    }
    if (accepted) { emit(key, kEntryAccepted, 0u, outcome, lds_counts); return; }
    if (over) { emit(key, kEntryWalkTop, 0u, outcome, lds_counts); return; }
    if (ex_next == 0u) return;  // rejected in this context
    // It leaves these frames as well: records for the next level, one per chunk of kContextsPerThread contexts
    // of the last frame's rule (a rule without contexts has nothing below it: the token ends there).
    // The lanes that get here together are taken rule by rule, each group with one atomic.
    const uint32_t rule = info.z;
    const uint32_t n_ch = (a.ctx_off[rule + 1] - a.ctx_off[rule] + kContextsPerThread - 1u) / kContextsPerThread;
    const bool single_next = single && n_res == 1u && (ex_next & (ex_next - 1u)) == 0u;
    if (level == (uint32_t)kCtxLevels || a.k_base[level] == nullptr || (ex_next & 0x80000000u)) {
      // the live stack decides: the walk starts where the way so far is unique
      if (n_ch == 0u) return;
      if (single_next && !(ex_next & 0x80000000u)) emit(key, kEntryWalkTop + level + 1u, (uint32_t)__ffs(ex_next) - 1u, outcome, lds_counts);
      else if (single) emit(key, kEntryWalkTop + level, (uint32_t)__ffs(ex) - 1u, outcome, lds_counts);
      else emit(key, kEntryWalkTop, 0u, outcome, lds_counts);
      return;
    }
    const uint32_t lane = threadIdx.x & 63u;
    for (bool pending = true; pending;) {
      const uint32_t lead = __builtin_amdgcn_readfirstlane(rule);
      const bool mine = rule == lead;
      const unsigned long long peers = __ballot(mine);
      if (mine) {
        if (n_ch != 0u) {
          const uint32_t n = (uint32_t)__popcll(peers), rank = (uint32_t)__popcll(peers & ((1ull << lane) - 1ull));
          const int first = __ffsll((long long)peers) - 1;
          uint32_t base = 0u;
          if (rank == 0u) base = atomicAdd(&a.res_count[level - 1u], n * n_ch);
          base = __shfl(base, first, 64) + rank * n_ch;
          for (uint32_t ch = 0; ch < n_ch; ++ch)
            if (base + ch < a.res_cap)
              a.res[level - 1u][base + ch] = make_uint4(e, key_local, ex_next, rule | (single_next ? 0x10000u : 0u) | (ch << 17));
        }
        pending = false;
      }
    }
  }
};

// Level 1, first part: which contexts the pairs of a tile (see ContextListArgs::tiles) have to be walked on in at all.  A
// wave takes a tile, a pair per lane, and looks at its contexts 64 at a time, a context per lane: pairs that leave the
// node's frame at the same position, in front of the same byte, fare alike in every context whose frames cannot take that
// byte, and in those where no path gets through what the rest of their tokens has in common.  The others are listed, an
// (up to 64 pairs, context) each.
// White space inside an object of a schema grammar has the context of every place where white space may stand: 17072 pairs
// times 2188 contexts of the 44.4 M of the 11867-node grammar at 151936 tokens, of which 9.3 M get past the first byte.
// Both parts and the writing pass: 20 + 111 + 15 us for that grammar, where workgroups of 768 pairs that walked every one
// of 8 contexts took 381 + 63 (8333 times the staging of the tables, 89 MB of outcomes); JSON and 32000 tokens 8 + 20 + 5,
// before 76 + 5; a scripting grammar and 128256 tokens 21 + 187 + 11, before 225 + 12; the C/SQL-like grammar, whose
// pairs get through most contexts, 105 + 900 to 960 (from run to run) + 69, before 970 + 62: there the look at the contexts gains nothing.
// A tile of few contexts is listed as it is (JSON 37 -> 8 us), and so is one of more than a few runs, which would be looked at
// one after the other (schema grammar 58 us with any number of runs, 28 with 8, 20 with 4).
constexpr uint32_t kManyContexts = 8;
constexpr int kMostRuns = 4;
__global__ __launch_bounds__(kContextThreads) void context_open_kernel(DevTables tab, DevVocab voc, ContextListArgs a, uint32_t tile0, uint32_t n_tiles) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr uint32_t kWaves = kContextThreads / 64;
  constexpr int kChunks = kTileContexts / 64;
  __shared__ uint32_t listed[kWaves], first_listed;
  if (blockIdx.x * kWaves >= n_tiles) return;
  stage_tables(tab, smem, kContextThreads);
  __syncthreads();
  auto body = [&](const auto& T) {
    const uint32_t wave = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63u;
    for (uint32_t t0 = blockIdx.x * kWaves; t0 < n_tiles; t0 += gridDim.x * kWaves) {
      u64 open[kChunks] = {};
      uint4 tile = make_uint4(0u, 0u, 0u, 0u);
      if (t0 + wave < n_tiles) {
        tile = a.tiles[tile0 + t0 + wave];
        const uint32_t n_pairs = uniform(tile.y & 0xFFFFu), n_ctx = uniform(tile.y >> 16);
        const uint32_t cb = a.ctx_off[T.header(tile.w).y >> 16] + tile.z;
        TokenRef t{make_uint4(0u, 0u, 0u, 0u), voc.bytes, 0};
        uint32_t ex = 0u;
        const bool look = n_ctx >= kManyContexts;
        if (look && lane < n_pairs) {
          t = load_token(voc, (int32_t)a.base_ids[tile.x + lane]);
          ex = a.exits[tile.x + lane];
        }
        // where the token goes on, if there is only one such place and its byte is among those that the lane holds
        const bool one_exit = ex != 0u && (ex & (ex - 1u)) == 0u && ex < (1u << 15);
        const uint32_t k = one_exit ? (uint32_t)__ffs((int)ex) - 1u : 0u;
        const uint32_t tag = k << 8 | token_byte(t.tk, voc.bytes, (int)k);
        u64 others = __ballot(lane < n_pairs && !one_exit);
        int runs = 0;
        for (u64 left = __ballot(lane < n_pairs && one_exit); left && !others;) {
          const int lead = __ffsll((long long)left) - 1;
          auto of = [&](uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, lead); };
          const uint32_t lead_tag = of(tag), c = lead_tag & 0xFFu;
          const u64 run = __ballot(lane < n_pairs && one_exit && tag == lead_tag);
          left &= ~run;
          if (++runs > kMostRuns) { others = 1ull; break; }
          const uint4 pre = make_uint4(of(t.tk.x), of(t.tk.y), of(t.tk.z), of(t.tk.w));
          // what the tokens of the run have in common with the first of them
          uint32_t same = 15u;
          if ((run >> lane) & 1ull) same = min((uint32_t)same_bytes(t.tk, pre), (uint32_t)t.len);
#pragma unroll
          for (uint32_t d = 1; d < 64u; d <<= 1) same = min(same, (uint32_t)__shfl_xor((int)same, d, 64));
          same = uniform(same);
#pragma unroll
          for (int q = 0; q < kChunks; ++q) {
            if (q * 64u >= n_ctx) break;
            const uint32_t i = q * 64u + lane;
            bool walk = false;
            uint32_t r = 0u;
            if (i < n_ctx) {
              r = a.ctx_node[cb + i];
              const uint2 h = T.header(r);
              walk = T.can_start(r, c) || ((h.y & 1u) && T.can_follow(h, c));
            }
            const u64 needs = __ballot(walk);
            if ((needs & (needs - 1ull)) && same > (lead_tag >> 8) + 1u && __popcll(run) >= kPrefixTokens) {
              if (walk) {
                const uint4 info = a.rule_info[T.header(r).y >> 16];
                walk = walk_token<true, true>(T, pre, voc.bytes, (int)same, r, (const XGM_GLOBAL uint16_t*)(a.forced_node + info.x), info.y + 1u,
                                              nullptr, info.z, (int)(lead_tag >> 8)) != kReject;
              }
            }
            open[q] |= __ballot(walk);
          }
        }
        if (others) {
#pragma unroll
          for (int q = 0; q < kChunks; ++q)
            if (q * 64u < n_ctx) open[q] = n_ctx - q * 64u >= 64u ? ~0ull : (1ull << (n_ctx - q * 64u)) - 1ull;
        }
      }
      uint32_t n = 0u;
#pragma unroll
      for (int q = 0; q < kChunks; ++q) n += (uint32_t)__popcll(open[q]);
      if (lane == 0u) listed[wave] = n;
      __syncthreads();
      uint32_t at = 0u, all = 0u;
      for (uint32_t w = 0; w < kWaves; ++w) {
        if (w < wave) at += listed[w];
        all += listed[w];
      }
      if (threadIdx.x == 0u && all) first_listed = atomicAdd(a.n_open, all);
      __syncthreads();
      at += first_listed;
#pragma unroll
      for (int q = 0; q < kChunks; ++q) {
        if ((open[q] >> lane) & 1ull)
          a.open[at + (uint32_t)__popcll(open[q] & ((1ull << lane) - 1ull))] = make_uint2(tile.x, (tile.y & 0xFFFFu) - 1u | (tile.z + q * 64u + lane) << 6);
        at += (uint32_t)__popcll(open[q]);
      }
      __syncthreads();
    }
  };
  if (small_sections_staged(tab)) body(LdsTabT<true>(tab, smem));
  else body(LdsTab(tab, smem));
}

// Second part: the listed (64 pairs, context), a wave for each (for two neighbours in the list, mostly of the same pairs, if
// there are more than the chip has room for: C/SQL-like grammar 958 us with one, 897 with two, 1064 with four, 1329 with
// eight, side by side).  All entries of a wave go to the lists of one key: they are counted
// per segment in LDS and added to the global counters once.
constexpr uint32_t kOpenBlocks = 512;  // the tables are staged once per place on the chip
template <bool WRITE>
__global__ __launch_bounds__(kContextThreads) void context_level1_kernel(DevTables tab, DevVocab voc, ContextListArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr uint32_t kWaves = kContextThreads / 64;
  __shared__ uint32_t counts[WRITE ? 1 : kWaves][kMaxSegs];
  const uint32_t n_open = *a.n_open;
  if (blockIdx.x >= n_open) return;
  stage_tables(tab, smem, kContextThreads);
  if (!WRITE)
    for (uint32_t t = threadIdx.x; t < kWaves * kMaxSegs; t += kContextThreads) counts[t / kMaxSegs][t % kMaxSegs] = 0u;
  __syncthreads();
  auto body = [&](const auto& T) {
    const uint32_t wave = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63u, n_seg = (uint32_t)voc.n_seg;
    uint32_t* const mine = WRITE ? nullptr : counts[WRITE ? 0 : wave];
    const uint32_t per = n_open > 2u * kOpenBlocks * kWaves ? 2u : 1u;
    uint32_t loaded = 0xFFFFFFFFu, id = 0u, ex = 0u, node = 0u;
    TokenRef t{make_uint4(0u, 0u, 0u, 0u), voc.bytes, 0};
    for (uint32_t q0 = (wave * gridDim.x + blockIdx.x) * per; q0 < n_open; q0 += gridDim.x * kWaves * per)
      for (uint32_t q = q0; q < min(q0 + per, n_open); ++q) {
        const uint2 item = a.open[q];
        const uint32_t e0 = uniform(item.x), n_pairs = (uniform(item.y) & 63u) + 1u, i = uniform(item.y) >> 6;
        if (e0 != loaded) {
          node = uniform(a.base_node[e0]);
          if (lane < n_pairs) {
            id = a.base_ids[e0 + lane];
            ex = a.exits[e0 + lane];
            t = load_token(voc, (int32_t)id);
          }
          loaded = e0;
        }
        const uint32_t r = uniform(a.ctx_node[a.ctx_off[T.header(node).y >> 16] + i]), key = a.k_base[0][node] + i;
        uint32_t outcome = 0u;
        if (lane < n_pairs) {
          const ContextWork<WRITE, std::decay_t<decltype(T)>> w{T, voc, a, e0 + lane, id, t};
          w.step(1u, r, key, ex, (ex & (ex - 1u)) == 0u, &outcome, mine);
        }
        if (WRITE) continue;
        if (a.outcomes) a.outcomes[(size_t)q * 64u + lane] = (uint16_t)outcome;
        if (__ballot(outcome != 0u)) {
          wave_sync();
          for (uint32_t s = lane; s < n_seg; s += 64u) {
            const uint32_t n = mine[s];
            if (n) {
              atomicAdd(&a.counts[(size_t)(a.key0[0] + key) * n_seg + s], n);
              mine[s] = 0u;
            }
          }
          wave_sync();
        }
      }
  };
  if (small_sections_staged(tab)) body(LdsTabT<true>(tab, smem));
  else body(LdsTab(tab, smem));
}
// The writing pass of level 1 when the counting pass kept its outcomes: the same list, no walks, no tables.  A wave
// reserves room in every list once and hands out the places from LDS.
constexpr int kOpenWriteThreads = 256;
__global__ __launch_bounds__(kOpenWriteThreads) void context_level1_write_kernel(DevVocab voc, ContextListArgs a) {
  constexpr uint32_t kWaves = kOpenWriteThreads / 64;
  __shared__ uint32_t next[kWaves][2 * kMaxSegs];  // per segment, accepted and walk entries: how many, then where the next one goes
  const uint32_t wave = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63u, n_seg = (uint32_t)voc.n_seg, n_open = *a.n_open;
  uint32_t* const mine = next[wave];
  for (uint32_t q = blockIdx.x * kWaves + wave; q < n_open; q += gridDim.x * kWaves) {
    const uint32_t code = a.outcomes[(size_t)q * 64u + lane];
    if (__ballot(code != 0u) == 0ull) continue;
    const uint2 item = a.open[q];
    const uint32_t e0 = uniform(item.x), i = uniform(item.y) >> 6;
    const uint32_t key = a.key0[0] + a.k_base[0][a.base_node[e0]] + i;
    const uint32_t id = code ? a.base_ids[e0 + lane] : 0u, kind = (code & 0xFFu) - 1u;
    const uint32_t at = 2u * (id / (uint32_t)kSegTokens) + (kind == kEntryAccepted ? 0u : 1u);
    wave_sync();  // (the places of the round before have been handed out)
    for (uint32_t s = lane; s < 2u * n_seg; s += 64u) mine[s] = 0u;
    wave_sync();
    if (code) atomicAdd(&mine[at], 1u);
    wave_sync();
    for (uint32_t s = lane; s < 2u * n_seg; s += 64u) {
      const uint32_t n = mine[s];
      if (n) {
        const size_t slot = (size_t)key * n_seg + (s >> 1);
        mine[s] = (s & 1u) ? atomicSub(&a.back[slot], n) - n : atomicAdd(&a.front[slot], n);
      }
    }
    wave_sync();
    if (code) a.entries[atomicAdd(&mine[at], 1u)] = id | ((code >> 8) << kEntryPosShift) | (kind << kEntryKindShift);
  }
}

// Level `level` >= 2: a fixed grid walks over the records of level - 1, each of which names a chunk of
// kContextsPerThread contexts.  A wave takes 64 consecutive records (neighbouring tokens of one node and context, as a
// rule) and two contexts of each, one after the other; neighbouring waves the same records.  Where there are records
// enough for all waves anyway it takes all eight.  Two launches of the 11867-node schema grammar (151936 tokens) 127 us with
// eight, 85 with two, 94 with one; JSON (32000) 38, 26, 25; a scripting grammar (128256, 660 K records) 560, 468, 442; the
// C/SQL-like grammar (1.7 M) 1632, 1775, 1811.
constexpr uint32_t kManyRecords = 1u << 20;
template <bool WRITE, class Tab>
__device__ __forceinline__ void context_deeper_body(const Tab& T, const DevVocab& voc, const ContextListArgs& a, uint32_t level) {
  static_assert(kContextsPerThread == 8, "a record's outcomes are eight 16-bit codes in one uint4");
  const uint32_t n_res = min(a.res_count[level - 2u], a.res_cap), per = n_res > kManyRecords ? kContextsPerThread : 2u;
  const uint32_t n_units = (n_res + 63u) / 64u * (kContextsPerThread / per), lane = threadIdx.x & 63u;
  uint16_t* const keep = WRITE ? nullptr : reinterpret_cast<uint16_t*>(a.deep_outcomes[level - 1u]);
  for (uint32_t unit = blockIdx.x * (kContextThreads / 64) + uniform(threadIdx.x >> 6); unit < n_units; unit += gridDim.x * (kContextThreads / 64)) {
    const uint32_t item = unit * per / kContextsPerThread * 64u + lane, q0 = unit * per % kContextsPerThread;
    if (item >= n_res) continue;
    const uint4 rec = a.res[level - 2u][item];
    const uint32_t rule = rec.w & 0xFFFFu, cb = a.ctx_off[rule], m = a.ctx_off[rule + 1] - cb, j0 = (rec.w >> 17) * kContextsPerThread;
    const uint32_t id = a.base_ids[rec.x];
    const ContextWork<WRITE, Tab> w{T, voc, a, rec.x, id, load_token(voc, (int32_t)id)};
    const uint32_t kb = a.k_base[level - 1u][rec.y];
#pragma unroll 1
    for (uint32_t q = q0; q < q0 + per; ++q) {
      uint32_t outcome = 0u;
      if (j0 + q < m) w.step(level, a.ctx_node[cb + j0 + q], kb + j0 + q, rec.z, (rec.w & 0x10000u) != 0u, &outcome);
      if (keep) keep[(size_t)item * kContextsPerThread + q] = (uint16_t)outcome;
    }
  }
}
template <bool WRITE>
__global__ __launch_bounds__(kContextThreads) void context_deeper_kernel(DevTables tab, DevVocab voc, ContextListArgs a, uint32_t level) {
  extern __shared__ __align__(16) unsigned char smem[];
  if (a.res_count[level - 2u] == 0u) return;
  stage_tables(tab, smem, kContextThreads);
  __syncthreads();
  if (small_sections_staged(tab)) context_deeper_body<WRITE>(LdsTabT<true>(tab, smem), voc, a, level);
  else context_deeper_body<WRITE>(LdsTab(tab, smem), voc, a, level);
}

// The writing pass of a deeper level when the counting pass kept its outcomes: the same records, no walks, no tables.
__global__ __launch_bounds__(256) void context_deeper_write_kernel(DevVocab voc, ContextListArgs a, uint32_t level) {
  const uint32_t n_res = min(a.res_count[level - 2u], a.res_cap);
  const ListSink<true> sink{voc, a};
  for (uint32_t item = blockIdx.x * 256u + threadIdx.x; item < n_res; item += gridDim.x * 256u) {
    const uint4 c = a.deep_outcomes[level - 1u][item];
    if ((c.x | c.y | c.z | c.w) == 0u) continue;
    const uint4 rec = a.res[level - 2u][item];
    const uint32_t id = a.base_ids[rec.x];
    const uint32_t key = a.key0[level - 1u] + a.k_base[level - 1u][rec.y] + (rec.w >> 17) * kContextsPerThread;
    const uint32_t codes[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
    for (uint32_t q = 0; q < kContextsPerThread; ++q) {
      const uint32_t code = (codes[q >> 1] >> ((q & 1u) * 16u)) & 0xFFFFu;
      if (code) sink.emit(id, key + q, (code & 0xFFu) - 1u, code >> 8);
    }
  }
}

// The running sum over the slots (see launch_slot_offsets), in two launches: the sum of every block of slots, then the offsets
// in it (a block adds up the sums of all blocks in front of it by itself: 98 of them for the 11867-node schema grammar).
// On the host, with the counts copied there and the offsets copied back, this took 350 us of that grammar's build.  All
// counts of a thread are fetched at once.
constexpr int kSlotThreads = 256, kSlotsPerThread = 16, kSlotBlock = kSlotThreads * kSlotsPerThread;
__device__ __forceinline__ void slot_counts(const SlotCounts& c, uint32_t (&n)[kSlotsPerThread]) {
#pragma unroll
  for (int j = 0; j < kSlotsPerThread; ++j) {
    const size_t k = (size_t)blockIdx.x * kSlotBlock + (uint32_t)(j * kSlotThreads) + threadIdx.x;
    n[j] = k < c.n_level0 ? c.level0[k] : k < c.n_slots ? c.counts[k] : 0u;
  }
}
// the sum over the workgroup, in every thread (64 bits: a grammar's lists may be too long for 32)
__device__ __forceinline__ u64 block_sum(u64 v, u64* part) {
#pragma unroll
  for (uint32_t d = 1; d < 64u; d <<= 1) v += __shfl_xor(v, d, 64);
  if ((threadIdx.x & 63u) == 0u) part[threadIdx.x >> 6] = v;
  __syncthreads();
  u64 sum = 0ull;
  for (int k = 0; k < kSlotThreads / 64; ++k) sum += part[k];
  return sum;
}
__global__ __launch_bounds__(kSlotThreads) void slot_sums_kernel(SlotCounts c, u64* __restrict__ block_sums) {
  __shared__ u64 part[kSlotThreads / 64];
  uint32_t n[kSlotsPerThread];
  slot_counts(c, n);
  u64 v = 0ull;
#pragma unroll
  for (int j = 0; j < kSlotsPerThread; ++j) v += n[j];
  const u64 sum = block_sum(v, part);
  if (threadIdx.x == 0u) block_sums[blockIdx.x] = sum;
}
__global__ __launch_bounds__(kSlotThreads) void slot_offsets_kernel(SlotCounts c, const u64* __restrict__ block_sums, uint32_t* __restrict__ key_off,
                                                                    uint32_t* __restrict__ front, uint32_t* __restrict__ back, u64* __restrict__ total) {
  __shared__ u64 part[kSlotThreads / 64], sums[kSlotsPerThread][kSlotThreads / 64];
  uint32_t n[kSlotsPerThread];
  slot_counts(c, n);
  u64 before = 0ull;
  for (uint32_t k = threadIdx.x; k < blockIdx.x; k += kSlotThreads) before += block_sums[k];
  const u64 base = block_sum(before, part);
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  u64 upto[kSlotsPerThread];  // in the wave, of the thread's j-th slot
#pragma unroll
  for (int j = 0; j < kSlotsPerThread; ++j) {
    upto[j] = n[j];
#pragma unroll
    for (uint32_t d = 1; d < 64u; d <<= 1) {
      const u64 v = __shfl_up(upto[j], d, 64);
      if (lane >= d) upto[j] += v;
    }
    if (lane == 63u) sums[j][wave] = upto[j];
  }
  __syncthreads();
  u64 at = base;
#pragma unroll
  for (int j = 0; j < kSlotsPerThread; ++j) {
    const size_t k = (size_t)blockIdx.x * kSlotBlock + (uint32_t)(j * kSlotThreads) + threadIdx.x;
    u64 end = at + upto[j];
#pragma unroll
    for (uint32_t q = 0; q < (uint32_t)kSlotThreads / 64u; ++q) {
      if (q < wave) end += sums[j][q];
      at += sums[j][q];
    }
    if (k < c.n_slots) {
      key_off[k] = front[k] = (uint32_t)(end - n[j]);
      back[k] = (uint32_t)end;
      if (k + 1 == c.n_slots) {
        key_off[k + 1] = (uint32_t)end;
        *total = end;
      }
    }
  }
}

// What a build has to bring to the device or back, or to clear, before its next kernel (see Moves).  A copy or a fill of the
// runtime's is a launch too, and costs the host more than one of ours does; a build had eight of them and has five launches
// of this kernel.  Builds side by side, JSON x 32000: 343 us with the runtime's, 334 so; 11867-node schema grammar 3256 and 3223.
constexpr int kMoveThreads = 256;
__global__ __launch_bounds__(kMoveThreads) void moves_kernel(Moves m) {
  const uint32_t i0 = blockIdx.x * kMoveThreads + threadIdx.x, step = gridDim.x * kMoveThreads;
#pragma unroll
  for (int k = 0; k < Moves::kMost; ++k)
    for (uint32_t i = i0; i < m.move[k].n; i += step) m.move[k].dst[i] = m.move[k].src ? m.move[k].src[i] : make_uint4(0u, 0u, 0u, 0u);
}

__global__ __launch_bounds__(kRowThreads) void rows_equal_kernel(const uint32_t* __restrict__ rows, int32_t W,
                                                                 const int32_t* __restrict__ rep,
                                                                 uint32_t* __restrict__ equal) {
  __shared__ uint32_t differs;
  if (rep[blockIdx.x] == (int32_t)blockIdx.x) {  // (most nodes are their own)
    if (threadIdx.x == 0) equal[blockIdx.x] = 1u;
    return;
  }
  if (threadIdx.x == 0) differs = 0u;
  __syncthreads();
  const uint32_t* a = rows + (size_t)blockIdx.x * W;
  const uint32_t* b = rows + (size_t)rep[blockIdx.x] * W;
  bool d = false;
  for (int32_t w = threadIdx.x; w < W; w += kRowThreads) d |= a[w] != b[w];
  if (d) differs = 1u;
  __syncthreads();
  if (threadIdx.x == 0) equal[blockIdx.x] = differs ? 0u : 1u;
}
__global__ __launch_bounds__(kRowThreads) void gather_rows_kernel(const uint32_t* __restrict__ rows, int32_t W,
                                                                  const int32_t* __restrict__ unique,
                                                                  uint32_t* __restrict__ out) {
  const uint32_t* src = rows + (size_t)unique[blockIdx.x] * W;
  uint32_t* dst = out + (size_t)blockIdx.x * W;
  for (int32_t w = threadIdx.x; w < W; w += kRowThreads) dst[w] = src[w];
}

__global__ void patch_classes_kernel(DevVocab voc, const uint32_t* __restrict__ items, int32_t n_items,
                                     uint32_t* acc_rank, uint32_t* unc_rank, uint32_t* plain_rank) {
  const int32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n_items) return;
  const size_t node = items[3 * k];
  const uint32_t r = items[3 * k + 1], cls = items[3 * k + 2];
  const uint32_t bit = 1u << (r & 31);
  uint32_t* pa = acc_rank + node * voc.WR + (r >> 5);
  uint32_t* pu = unc_rank + node * voc.WR + (r >> 5);
  if (cls == (uint32_t)kAccept) atomicOr(pa, bit); else atomicAnd(pa, ~bit);
  if (cls == (uint32_t)kUncertain) atomicOr(pu, bit); else atomicAnd(pu, ~bit);
  if (plain_rank) {
    uint32_t* pp = plain_rank + node * voc.WR + (r >> 5);
    if (cls == (uint32_t)kUncertainPlain) atomicOr(pp, bit); else atomicAnd(pp, ~bit);
  }
}

// What a wave stores of 2048 elements of a logits row (section 2.1): -inf where the element's bit is not set.  Lane l
// has the bits of elements 32 l .. 32 l + 31; `p` is the address of element 0, on 16 bytes.  A stretch of 64 groups of
// 16 bytes with nothing allowed is one streaming store per lane (the lines are written whole and not read again here,
// so they need not stay in the caches); any other is stored element by element, 64 at a time, under their bits, which
// lie in the order of the lanes.  The logits are never read: a group that is fetched, blended and stored whole makes
// its wave wait for the fetch, while stores are issued and forgotten.
// Where no lane has more than kApplyFew disallowed elements each stores its own, one after the other (inside a string
// nearly every token is allowed: serving masks have 3 to 7 in the fullest word of such a wave).  One-launch step of 128
// rows, 8.27 us with 8 or 12 of them, 8.9 with 4 and 9.1 with 3, where most of these waves go the other way; a loop over
// the disallowed elements of a lane's group of 16 bytes, for all masks, took 8.81.
constexpr int32_t kApplyWaveWords = 64, kApplyWaveElems = kApplyWaveWords * 32;
constexpr int kApplyFew = 8;
template <int ESIZE>
__device__ __forceinline__ void apply_wave(unsigned char* p, uint32_t allowed, uint32_t neg_inf) {
  typedef uint32_t v4u __attribute__((ext_vector_type(4)));
  constexpr int kStretchWords = 64 * 16 / ESIZE / 32;
  constexpr unsigned long long kOnes = (1ull << kStretchWords) - 1ull;
  const uint32_t lane = threadIdx.x & 63u;
  const unsigned long long none = __ballot(allowed == 0u), all = __ballot(allowed == ~0u);
  const uint32_t fill = ESIZE == 2 ? (neg_inf | (neg_inf << 16)) : neg_inf;
  const v4u val = {fill, fill, fill, fill};
  if (__ballot(__popc(~allowed) > kApplyFew) == 0ull) {
    unsigned char* const q = p + lane * (32u * ESIZE);
    for (uint32_t x = ~allowed; x; x &= x - 1u) {
      const uint32_t h = (uint32_t)__ffs((int)x) - 1u;
      if (ESIZE == 2) reinterpret_cast<uint16_t*>(q)[h] = (uint16_t)neg_inf;
      else reinterpret_cast<uint32_t*>(q)[h] = neg_inf;
    }
    return;
  }
#pragma unroll
  for (int k = 0; k < kApplyWaveWords / kStretchWords; ++k) {
    if (((all >> (k * kStretchWords)) & kOnes) == kOnes) continue;
    unsigned char* const q = p + k * 1024;
    if (((none >> (k * kStretchWords)) & kOnes) == kOnes) {
      __builtin_nontemporal_store(val, reinterpret_cast<v4u*>(q + lane * 16u));
    } else {
#pragma unroll
      for (int h = 0; h < kStretchWords / 2; ++h) {
        const unsigned long long bits = (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)allowed, k * kStretchWords + 2 * h) |
                                        ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)allowed, k * kStretchWords + 2 * h + 1) << 32);
        if (!__builtin_amdgcn_inverse_ballot_w64(bits)) {
          if (ESIZE == 2) reinterpret_cast<uint16_t*>(q)[h * 64 + lane] = (uint16_t)neg_inf;
          else reinterpret_cast<uint32_t*>(q)[h * 64 + lane] = neg_inf;
        }
      }
    }
  }
}

// ---------------------------------------------------------------- kernel (b)
// The per-step stack upload, as a kernel on the caller's stream that reads pinned host memory over the bus
// (for the few tens of kilobytes of a step this takes a fraction of the time a copy-engine transfer with
// its cross-queue synchronisation does).  The stack headers are written out in full on the way: the host
// sends, per stack, the keys of its lists; the offsets of the lists' segments are read from the cache's
// key_off here.  Blocks [0, copy_blocks) copy the row descriptors and the frames, the others expand
// kStacksPerBlock stacks each, whose key words go through LDS (one read over the bus per 16 bytes).
constexpr int kUploadThreads = 256;
constexpr uint32_t kStacksPerBlock = 2;
__global__ __launch_bounds__(kUploadThreads) void upload_stacks_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst,
                                                                       uint32_t plain16, const uint4* __restrict__ src_frames,
                                                                       uint4* __restrict__ dst_frames, uint32_t frames16,
                                                                       uint32_t copy_blocks, const uint4* __restrict__ src_stacks,
                                                                       uint32_t n_stacks, uint32_t n_seg,
                                                                       uint32_t* __restrict__ dst_hdrs) {
  __shared__ uint32_t keys[kStacksPerBlock][kStackKeysWords];
  if (blockIdx.x < copy_blocks) {
    const uint32_t i = blockIdx.x * kUploadThreads + threadIdx.x;
    if (i < plain16) dst[i] = src[i];
    else if (i < plain16 + frames16) dst_frames[i - plain16] = src_frames[i - plain16];
    return;
  }
  const uint32_t s0 = (blockIdx.x - copy_blocks) * kStacksPerBlock;
  constexpr uint32_t kQuads = kStackKeysWords / 4;
  if (threadIdx.x < kStacksPerBlock * kQuads && s0 + threadIdx.x / kQuads < n_stacks) {
    const uint4 q = src_stacks[(size_t)s0 * kQuads + threadIdx.x];
    uint32_t* k = &keys[threadIdx.x / kQuads][(threadIdx.x % kQuads) * 4];
    k[0] = q.x; k[1] = q.y; k[2] = q.z; k[3] = q.w;
  }
  __syncthreads();
  const uint32_t stride = stack_hdr_stride((int32_t)n_seg);
  for (uint32_t t = threadIdx.x; t < kStacksPerBlock * stride; t += kUploadThreads) {
    const uint32_t st = t / stride, w = t % stride;
    if (s0 + st >= n_stacks) break;
    const uint32_t* k = keys[st];
    uint32_t out;
    if (w < kStackHdrWords) out = k[w];
    else {
      const uint32_t sgm = (w - kStackHdrWords) / kStackLists, l = (w - kStackHdrWords) % kStackLists, key = k[kStackHdrWords + l];
      const uint32_t* key_off = reinterpret_cast<const uint32_t*>((uintptr_t)k[kStackHdrWords + kStackLists] |
                                                                  ((uintptr_t)k[kStackHdrWords + kStackLists + 1] << 32));
      out = key == kNoKey ? 0u : key_off[(size_t)key * n_seg + sgm];
    }
    dst_hdrs[(size_t)(s0 + st) * stride + w] = out;
  }
}

// The same in place: the stacks of the states in one slot of some rows of a batch, a workgroup per (stack, row).  The rows'
// scalars are written here too: three copies from the host cost 35 us (a state into a row: 149 us with them, 114 without).
__global__ __launch_bounds__(64) void batch_headers_kernel(DevBatch bt, int32_t row0, int32_t slot, int32_t older) {
  __shared__ uint32_t keys[kStackKeysWords];
  const int32_t b = row0 + (int32_t)blockIdx.y;
  const size_t at = (size_t)b * bt.H + slot;
  if (blockIdx.x == 0u && threadIdx.x == 0u) {
    bt.head[b] = slot;
    bt.older[b] = older;
    bt.status[b] = 0;
  }
  if (blockIdx.x >= bt.meta[at].n_stacks) return;
  const uint32_t stride = stack_hdr_stride(bt.n_seg), n_seg = (uint32_t)bt.n_seg;
  uint32_t* const h = bt.hdrs + (at * kBatchMaxStacks + blockIdx.x) * stride;
  if (threadIdx.x < kStackKeysWords) keys[threadIdx.x] = h[threadIdx.x];
  __syncthreads();
  const uint32_t* key_off = reinterpret_cast<const uint32_t*>((uintptr_t)keys[kStackHdrWords + kStackLists] |
                                                              ((uintptr_t)keys[kStackHdrWords + kStackLists + 1] << 32));
  for (uint32_t w = kStackHdrWords + threadIdx.x; w < stride; w += 64u) {
    const uint32_t sgm = (w - kStackHdrWords) / kStackLists, key = keys[kStackHdrWords + (w - kStackHdrWords) % kStackLists];
    h[w] = key == kNoKey ? 0u : key_off[(size_t)key * n_seg + sgm];
  }
}

// A walk by a whole wave (all lanes do the same): its memory is in LDS, and everything it reads is declared the same
// for all lanes, so that the walk runs in scalar registers with scalar branches.  A lone lane waits for every
// instruction just as long, and needs more of them (each branch turns lanes off and on again; frames and
// alternatives go through scratch memory).
constexpr uint32_t kWaveMemWords = kArenaFrames + 2 * kChoicePoints;
struct WaveMem {
  XGM_LDS uint32_t* arena;    // [kArenaFrames]
  XGM_LDS uint32_t* choices;  // [2 * kChoicePoints]
  __device__ __forceinline__ uint32_t frame(uint32_t k) const { return uniform(arena[k]); }
  __device__ __forceinline__ void set_frame(uint32_t k, uint32_t v) { arena[k] = v; }
  __device__ __forceinline__ uint2 choice(uint32_t k) const { return make_uint2(uniform(choices[2u * k]), uniform(choices[2u * k + 1u])); }
  __device__ __forceinline__ void set_choice(uint32_t k, uint2 v) { choices[2u * k] = v.x; choices[2u * k + 1u] = v.y; }
};
struct UniformFrames {
  const XGM_LDS uint16_t* p;
  __device__ __forceinline__ uint32_t operator[](uint32_t k) const { return uniform(p[k]); }
  __device__ __forceinline__ uint32_t of_lane(uint32_t k) const { return p[k]; }
};
// walk_token (of a live stack) for a wave whose tables (the sections in front of the headers) are in LDS: the same
// paths in the same order, fewer steps.  The token's bytes lie in the lanes, 32 at a time: lane j and lane 32 + j have the
// same one.  A step looks at all of them at once, lane j at node n (the inside of a string stays where it is), lane 32 + j at
// the node that follows n by as many places as the byte does the next one (a literal's nodes are numbered one after the other).
// A byte at which there is nothing to do but a move along an edge is taken in a loop of its own, and where the move stayed at
// its node, or went to the next one, so are all bytes behind it of which the lanes have seen the same.
// Where there is nothing but a return, lane j looks at the frame j below the one returned into, and all frames are
// returned through that can do nothing else with the byte (an operand in an expression grammar sits a dozen precedence
// levels deep).
// Bound by latency: every instruction of a wave that is alone with its walk waits for the one before.  Measured so, in clocks:
// an arithmetic instruction 4, a branch not taken 6 and taken 20, a comparison whose mask goes through scalar registers back
// into a select 28, an LDS read 61 (84 with its value in a scalar register).  So the lookup is arithmetic on vectors with
// three rounds of LDS reads (header, shape and FOLLOW word, target), and one word of it decides whether the step is a move:
// 400 clocks for a move, where the same lookup made of comparisons and masks, with all runs looked for in every step, took
// 1106 (a token of 11 bytes in a keyword of the scripting grammar 13236 and 6870, one of 14 bytes through five frames of a
// schema grammar 34200 and 21900).  Mask and bf16 logits in one launch with that lookup take 1.00 to 1.23 times as long for 24 rows of
// the C/SQL-like grammar and 128256 tokens (six draws of states, 1.12 in the mean), 1.01 to 1.17 for 64 (four), 1.01 to 1.14 for 8
// rows of the scripting grammar and 32000 tokens (six), 1.01 to 1.03 for 32 and 128256 (three).
template <class Note>
__device__ __forceinline__ int walk_wave(const LdsTabT<true, true>& T, WaveMem& mem, const uint4 tk, const uint8_t* ext, const int len,
                                         const uint32_t start_node, const UniformFrames& live, const uint32_t depth, const Note& note,
                                         const int i0 = 0) {
  if (len > kMaxTokenLen) return kOverflow;
  const uint32_t lane = threadIdx.x & 63u, half = lane & 31u, chained = lane < 32u ? 0u : ~0u;
  const uint32_t last_alt = (T.off_hdr - T.off_alts) / 4u - 1u, last_target = (T.off_follow - T.off_targets) / 2u - 1u, last_node = T.n_nodes - 1u;
  const bool all_near = T.n_near >= T.n_nodes;
  uint32_t n = start_node, sp = kLiveBase + depth - 1, f = 1, alt = 0, top = 0, csp = 0, needed = 0;
  int i = i0, steps = 0;
  // the lane's byte, and where its class's column of the shapes and its word of a FOLLOW set begin
  uint32_t byte = 0u, column = 0u, word_of_set = 0u;
  int window = 0, window_end = i0;  // the bytes in the lanes
  auto load_window = [&]() {
    window = i;
    window_end = min(len, i + 32);
    const int at = min(i + (int)half, len - 1);
    byte = token_byte(tk, nullptr, min(at, 14));
    if (len > 15) {
      const uint32_t beyond = ext[at];
      byte = at < 15 ? byte : beyond;
    }
    column = T.off_shapes + T.lds[byte];
    word_of_set = T.off_follow + (byte >> 5) * 4u;
  };
  // What node `node` does with byte `c`, each lane its own: where to (bits 0..15), kNone = there is neither a move nor a call,
  // kReturns = the rule may end there and c can follow it.  Vector arithmetic alone: a comparison whose result goes through a
  // mask in scalar registers costs as much as seven instructions.
  constexpr uint32_t kNone = 0x10000u, kReturns = 0x20000u;
  auto look = [&](uint32_t node, uint32_t c, uint32_t col, uint32_t set) {
    u64 hdr = *(const XGM_LDS u64*)(T.lds + T.off_hdr + (all_near ? node : min(node, T.n_near - 1u)) * 8u);
    if (!all_near && __ballot(node >= T.n_near)) {  // (all lanes fetch, so that none goes a way of its own)
      const u64 far = *(const XGM_GLOBAL u64*)(T.img + T.off_hdr + (size_t)node * 8u);
      hdr = node < T.n_near ? hdr : far;
    }
    const uint32_t hx = (uint32_t)hdr, flags = (uint32_t)(hdr >> 32);
    const uint32_t branching = 0u - ((flags >> 1) & 1u);
    const uint32_t si = T.lds[col + (__umul24(hx & 0xFFFFu, T.n_cls) & branching)];
    const uint32_t follow = *(const XGM_LDS uint32_t*)(T.lds + set + (flags >> 16) * 32u) >> (c & 31u);
    const uint32_t target = *(const XGM_LDS uint16_t*)(T.lds + T.off_targets + min((hx >> 16) + si, last_target) * 2u);
    const uint32_t outside = ((c - (hx & 0xFFu)) | (((hx >> 8) & 0xFFu) - c)) >> 31, dead = (si + 1u) >> 8;
    const uint32_t to = (target & branching) | ((hx >> 16) & ~branching), none = (dead & branching) | (outside & ~branching);
    return to | none << 16 | (flags & follow & 1u) << 17;
  };
  auto of = [](uint32_t v, uint32_t l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l); };
  for (;;) {    // a path
    for (;;) {  // its steps
      uint32_t x, first;
      for (;;) {
        if (__builtin_expect(i == window_end, 0)) {
          if (i == len) break;
          load_window();
        }
        first = (uint32_t)(i - window);
        const uint32_t node = min(n + ((half - first) & chained), last_node);  // (lanes of bytes that have been taken: any node)
        const uint32_t found = look(node, byte, column, word_of_set);
        x = of(found, first);
        // nothing but a move: on with the next byte
        if (x >= 0x8000u || alt != 0u) break;
        ++steps;
        ++i;
        f = 1;
        const uint32_t d = x - n;
        n = x;
        if (d > 1u) continue;
        // it stayed at its node, or went to the next one: for how many bytes more?
        const u64 more = __ballot(found == node - chained);
        const uint32_t run = (uint32_t)__ffs((int)~((uint32_t)(d ? more >> 32 : more) >> first >> 1)) - 1u;
        const uint32_t taken = min(run, (uint32_t)(window_end - i));
        i += (int)taken;
        steps += (int)taken;
        n += d ? taken : 0u;
      }
      if (steps >= kMaxSteps) return kOverflow;
      if (i == len) {
        if constexpr (!Note::kEnumerate) return kAccept;
        note(n, sp, mem, live);
        ++steps;
        break;  // on to the next path
      }
      ++steps;
      // (what has not consumed a byte since the last push cannot return)
      uint32_t can_pop = sp != kLiveBase && (x & kReturns) ? f : 0u;
      if (can_pop && (x & kNone) && alt == 0u) {
        // (frames pushed one after the other lie one after the other, each with the number of the one below)
        const bool pushed = sp < kLiveBase;
        const uint32_t below = pushed ? sp + 1u : sp - kLiveBase, k = min(lane, below - 1u);
        uint32_t word;
        if (pushed) word = mem.arena[sp - k];
        else word = live.of_lane(below - 1u - k);
        const uint32_t there = look(word & 0xFFFFu, of(byte, first), of(column, first), of(word_of_set, first));
        const u64 next = pushed ? __ballot((word >> 16) + 1u == sp - lane) : ~0ull;
        // (frame 0 of the stack is not returned from)
        const uint32_t last = pushed ? below : below - 1u;
        const u64 other = ~(__ballot((there & (kNone | kReturns)) == (kNone | kReturns)) & next & (last < 64u ? (1ull << last) - 1ull : ~0ull));
        const uint32_t through = min((uint32_t)__ffsll((long long)other) - 1u, 63u);  // (none: 0xFFFFFFFF)
        const uint32_t frame = of(word, through);
        n = frame & 0xFFFFu;
        if (pushed && needed <= sp) top = max(sp - through, needed);  // (frames that a pending alternative needs stay)
        sp = pushed ? frame >> 16 : sp - through - 1u;
        steps += (int)through + 1;
        x = of(there, through);
        can_pop = sp != kLiveBase && (x & kReturns) ? 1u : 0u;
      }
      const uint32_t dst = x & 0xFFFFu, k_some = x & kNone ? 0u : 1u;
      const bool pooled = k_some && dst >= 0x8000u;
      // the pool entry: lane j has its word j (a count and the alternatives, or a run of calls)
      const uint32_t base = dst & 0x7FFFu;
      uint32_t word = 0u, word0 = 0u;
      if (pooled) {
        word = *(const XGM_LDS uint32_t*)(T.lds + T.off_alts + min(base + lane, last_alt) * 4u);
        word0 = uniform(word);
      }
      const bool calls = (word0 & kRunFlagD) != 0u;
      const uint32_t k = pooled && !calls ? word0 : k_some, total = k + can_pop;
      if (alt >= total) break;
      if (alt + 1 < total) {
        if (csp == kChoicePoints) return kOverflow;
        mem.set_choice(csp++, make_uint2(n | (sp << 16), (uint32_t)i | ((alt + 1) << 8) | (top << 16) | (f << 24)));
        needed = top;
      }
      if (alt < k) {
        bool consumes;
        if (calls) {
          const uint32_t m = run_frames(word0);
          if (top + m > kArenaFrames) return kOverflow;
          for (uint32_t j = 0; j < m; ++j) {
            mem.set_frame(top, ((T.alt(run_frames_at(word0) + (j >> 1)) >> ((j & 1u) * 16u)) & 0xFFFFu) | (sp << 16));
            sp = top++;
          }
          n = of(word, 1u);
          consumes = (word0 & kRunConsumesD) != 0u;
        } else {
          const uint32_t e = !pooled ? (kMoveTagD << 16) | dst : alt < 63u ? of(word, 1u + alt) : T.alt(base + 1u + alt);
          const uint32_t tag = e >> 16;
          n = e & 0xFFFFu;
          consumes = tag == kMoveTagD;
          if (!consumes && tag != kTailTagD) {
            if (top == kArenaFrames) return kOverflow;
            mem.set_frame(top, tag | (sp << 16));
            sp = top++;
          }
        }
        f = consumes ? 1u : 0u;
        i += consumes ? 1 : 0;
      } else if (sp < kLiveBase) {   // return into a frame pushed during this walk
        const uint32_t fr = mem.frame(sp), old = sp;
        n = fr & 0xFFFFu;
        sp = fr >> 16;
        if (needed <= old) top = old;
      } else {                       // return into a live frame
        n = live[sp - kLiveBase - 1u];
        --sp;
      }
      alt = 0;
    }
    // to the most recent pending alternative
    if (csp == 0) return kReject;
    const uint2 ch = mem.choice(--csp);
    n = ch.x & 0xFFFFu;
    sp = ch.x >> 16;
    i = (int)(ch.y & 0xFFu);
    if (i < window) window_end = i;  // (the lanes hold later bytes)
    alt = (ch.y >> 8) & 0xFFu;
    top = (ch.y >> 16) & 0xFFu;
    f = (ch.y >> 24) & 1u;
    needed = csp ? (mem.choice(csp - 1).y >> 16) & 0xFFu : 0u;
  }
}
// Threads of a workgroup that has a segment to itself.  Where four share one (PARTS: their threads) it is for the walks: see
// part_threads().
constexpr int kFillThreads = 256;
constexpr int fill_threads(int parts) { return parts ? parts : kFillThreads; }
constexpr int kFillFramesLds = 1024;            // live frames kept in LDS (deeper stacks: global memory)

// One workgroup of 4 waves serves one request and one segment of 8192 token
// ids = 256 mask words, which it owns in LDS (PARTS: four workgroups a quarter each):
//   1. every word = OR of the accepted bitsets of the tops of all stacks that
//      keep one (Algorithm 1: the result is the union over the parallel
//      stacks); the stop tokens if the text may end;
//   2. the stacks' token lists for this segment (up to four per stack: the
//      top node's own accepted tokens if it keeps a list instead of a bitset,
//      the tokens accepted given the node below the top frame, those accepted
//      given the two and the three nodes below) are streamed once, coalesced;
//      an accepted entry sets its bit with an LDS atomic, a walk entry is put
//      into a queue in LDS;
//   3. if there are walk entries, they are decided against the live stack: only
//      then are the request's automaton tables and frames copied into LDS;
//   4. the words are stored once, coalesced, and - in the fused instantiation -
//      the logits of the segment are masked straight from them.
// No global atomics, no second pass over the mask.  The launch is bound by
// instruction issue as much as by memory (2432 workgroups of four waves on 1024
// SIMDs): what every thread would do for nothing is kept behind tests that are
// the same for the whole workgroup (an empty list costs a scalar compare).
// COUNT = true additionally sums the automaton steps of all walks into
// *step_counter (instrumentation for the benchmark; never used on the hot path).
// WALKS = false: no mask cache of the batch has a walk entry (a cache knows:
// schema grammars have none) and step 3 is left out; the kernel then fits eight
// workgroups per compute unit (registers, LDS) and needs no scratch memory.
// WALKS = true: up to seven workgroups of 256 threads per compute unit (scalar registers),
// as many as have room for the batch's tables in LDS (four at 31 KB), or three of 512.  With one
// kernel for both the walk was a function of its own, which spilled in its
// inner loop and cost 5 us before its first step: the fill of a
// row that walks a handful of tokens (C/SQL-like grammar, 128256 tokens, one row)
// went from 13.7 to 8.7 us, one that walks 500 steps from 53 to 36, and to 31 with a
// wave for each entry of a short queue; a row of the scripting grammar that walks 50
// steps from 7.8 to 4.8.
template <bool WALKS, int THREADS>
struct FillShared {
  uint32_t words[kSegWords];
};
constexpr uint32_t kWalkQueue = 1024;  // entries; where there are more the lists are gone through again
// a queued entry: its id within the segment, position << 13, kind << 21, stack << 24
__device__ __forceinline__ uint32_t queue_entry(uint32_t e, uint32_t stack, uint32_t seg_id0) {
  static_assert(kSegTokens == 1 << 13 && kEntryWalkTop + kCtxLevels + 1 < 8, "the fields of a queued entry");
  return ((e & kEntryIdMask) - seg_id0) | ((e >> kEntryPosShift) & 0xFFu) << 13 | (e >> kEntryKindShift) << 21 | stack << 24;
}
__device__ __forceinline__ uint32_t list_entry(uint32_t q, uint32_t seg_id0) {
  return ((q & 0x1FFFu) + seg_id0) | ((q >> 13) & 0xFFu) << kEntryPosShift | ((q >> 21) & 7u) << kEntryKindShift;
}
// Up to so many entries for each wave of the workgroup go to the waves (walk_wave): six one after the other cost what a lane's longest walk does in
// a grammar of deep walks (C/SQL-like: 23 -> 17 us for a row with a walk of 79 steps; with up to 64 a row of 4358 steps
// took 137 us instead of 55, with up to 256 as long).  None go to waves in a batch with a cache whose build had walks over
// the limits: such a fill waits for walks of thousands of steps, of which a wave takes longer than a lane each (what a
// wave looks ahead for is not there) and only a few at a time.  Markup grammar, fills of 3 rows x 128256 and of 8 x 151936
// by waves 4.75 and 4.86 ms, by lanes 3.97 and 4.0.
constexpr uint32_t kWaveWalks = 6;  // entries per wave
constexpr uint32_t kPartShift = 2;  // workgroups that share a segment, as a power of two (PARTS)
template <int THREADS>
struct FillShared<true, THREADS> {
  uint32_t words[kSegWords];
  uint16_t live[kFillFramesLds];
  uint32_t queue[kWalkQueue];
  uint32_t n_queued;                  // counts on beyond the queue's room
  uint32_t mem[THREADS / 64][kWaveMemWords];
};

// What the walks need to know about a row, wherever its state came from.
struct WalkRow {
  const XGM_GLOBAL uint32_t* stacks;   // first stack: a header, or kInlineStackWords
  const XGM_GLOBAL uint16_t* frames;
  uint32_t stride, frame0, n_frames, epoch;
};

// One walk entry of a list of a stack: what to walk.  Returns false if the stack does not reach the entry's level.
struct WalkStart { uint32_t f_off, depth, drop; };  // the stack's frames; frames above the one the walk starts in
template <bool INLINE>
__device__ __forceinline__ bool walk_start(const WalkRow& row, uint32_t stack, uint32_t entry, WalkStart& w) {
  const XGM_GLOBAL uint32_t* sh = row.stacks + (size_t)stack * row.stride;
  uint32_t drops;
  if (INLINE) {
    w.depth = sh[5] & 0xFFFFu;
    w.f_off = sh[5] >> 16;
    drops = sh[6];
  } else {
    w.depth = sh[kStackHdrDepth];
    w.f_off = sh[kStackHdrFrames];
    drops = sh[kStackHdrDrops];
  }
  w.drop = stack_drop(drops, (entry >> kEntryKindShift) - kEntryWalkTop);
  return w.depth > w.drop;
}

// Decides walk entries, thread t the entries t, t + THREADS, ... of the queue (list null; neighbours in it go to
// different waves) or of a list of stack `list_stack` (all threads call this).
template <bool COUNT, bool KEEP_UNDECIDED, bool INLINE, int THREADS, class Tab>
__device__ __forceinline__ void fill_walks(const Tab& T, FillShared<true, THREADS>& sm, const WalkRow& row, const int32_t b, const int32_t id0,
                                           const uint32_t n_ids, const XGM_GLOBAL uint32_t* list, const uint32_t list_stack, const uint32_t n,
                                           const DevVocab& voc, OverflowLog* log, uint32_t seq, unsigned long long& my_steps) {
  const bool frames_in_lds = row.n_frames <= kFillFramesLds;
#pragma unroll 1
  for (uint32_t q = list ? threadIdx.x : (threadIdx.x & 63u) * (THREADS / 64) + (threadIdx.x >> 6); q < n; q += THREADS) {
    uint32_t e, stack = list_stack;
    if (list) {
      e = list[q];
      if ((e >> kEntryKindShift) == kEntryAccepted) continue;
    } else {
      e = list_entry(sm.queue[q], (uint32_t)id0 & ~(kSegTokens - 1u));
      stack = sm.queue[q] >> 24;
    }
    const uint32_t id = e & kEntryIdMask, pos = (e >> kEntryPosShift) & 0xFFu;
    const uint32_t rel = id - (uint32_t)id0;
    if (list && rel >= n_ids) continue;                      // another part's
    if ((sm.words[rel >> 5] >> (rel & 31u)) & 1u) continue;  // already allowed
    const TokenRef t = load_token(voc, (int32_t)id);
    WalkStart w;
    if (!walk_start<INLINE>(row, stack, e, w)) continue;
    LiveView live;
    live.lds = (const XGM_LDS uint16_t*)sm.live + (w.f_off - row.frame0);
    live.glob = row.frames + w.f_off;
    live.lo = frames_in_lds ? 0u : 0xFFFFFFFFu;
    uint32_t n_steps = 0;
    const int res = walk_token<false>(T, t.tk, t.ext, t.len, live[w.depth - 1u - w.drop], live, w.depth - w.drop, COUNT ? &n_steps : nullptr, 0u,
                                      w.drop == 0u ? 0 : (int)pos);
    if (COUNT) my_steps += n_steps;
    if (res == kOverflow) record_overflow(log, seq, (uint32_t)b, id, row.epoch);  // decided on the host
    if (res == kAccept || (KEEP_UNDECIDED && res == kOverflow)) atomicOr(&sm.words[rel >> 5], 1u << (rel & 31u));
  }
}
// The same for a short queue, a wave per entry (tables and frames are in LDS).
template <bool KEEP_UNDECIDED, bool INLINE, int THREADS>
__device__ __forceinline__ void fill_walks_by_wave(const LdsTabT<true, true>& T, FillShared<true, THREADS>& sm, const WalkRow& row, const int32_t b,
                                                   const int32_t id0, const uint32_t n, const DevVocab& voc, OverflowLog* log, uint32_t seq) {
  const uint32_t wave = uniform(threadIdx.x >> 6);
  WaveMem mem{(XGM_LDS uint32_t*)sm.mem[wave], (XGM_LDS uint32_t*)sm.mem[wave] + kArenaFrames};
#pragma unroll 1
  for (uint32_t q = wave; q < n; q += THREADS / 64) {
    const uint32_t entry = uniform(sm.queue[q]), e = list_entry(entry, (uint32_t)id0 & ~(kSegTokens - 1u)), stack = entry >> 24;
    const uint32_t id = e & kEntryIdMask, pos = (e >> kEntryPosShift) & 0xFFu;
    const uint32_t rel = id - (uint32_t)id0;
    if ((uniform(sm.words[rel >> 5]) >> (rel & 31u)) & 1u) continue;  // already allowed
    const TokenRef t = load_token(voc, (int32_t)id);
    WalkStart w;
    if (!walk_start<INLINE>(row, stack, e, w)) continue;
    const uint32_t depth = uniform(w.depth), drop = uniform(w.drop);
    const UniformFrames live{(const XGM_LDS uint16_t*)sm.live + (uniform(w.f_off) - row.frame0)};
    const int res = walk_wave(T, mem, t.tk, t.ext, (int)uniform((uint32_t)t.len), live[depth - 1u - drop], live, depth - drop, FirstPathEnds(), drop == 0u ? 0 : (int)pos);
    if ((threadIdx.x & 63u) == 0u) {
      if (res == kOverflow) record_overflow(log, seq, (uint32_t)b, id, row.epoch);  // decided on the host
      if (res == kAccept || (KEEP_UNDECIDED && res == kOverflow)) atomicOr(&sm.words[rel >> 5], 1u << (rel & 31u));
    }
  }
}

// The second launch bound (waves per SIMD): the kernel without walks keeps within the registers that eight workgroups per
// compute unit leave.  With walks the scalar registers are what counts: up to seven waves have 106 of them, eight have 78, for
// which the compiler moved 52 to 109 of them to lanes of vector registers and back (17 to 38 with 106), in walks that wait for
// every instruction.  Where four workgroups of 512 threads share a segment that is three of them per compute unit instead of four,
// and still faster.  Mask and bf16 logits in one launch, V = 128256, us with a bound of eight and of six, three draws of
// states each: 24 rows of the C/SQL-like grammar 23.6, 32.6, 13.8 and 22.5, 32.4, 12.8; 64 rows 31.9, 41.0, 56.6 and 32.4, 40.6,
// 55.7; 16 rows of the scripting grammar (two draws) 12.5, 30 and 10.5, 24.4; 200 C/SQL-like rows x 32000 53.5 and 49.1.
// APPLY = 0: the mask only.  APPLY = 2 / 4 (bytes per logit): the workgroup
// also writes -inf into the logits of its (row, segment) straight from its
// LDS words (section 2.1), which saves a launch and the re-read of the mask.
// A token whose walk exceeded the limits is then left allowed (bit set, logit
// untouched) until the host has decided it.
struct FusedApply {
  unsigned char* logits;  // [B][row_stride] elements of APPLY bytes; 16-byte aligned rows
  int64_t row_stride;     // elements
  int32_t V_logits;
  uint32_t neg_inf;
};

// INLINE != 0: the states came with the launch (InlineStates, the first argument: read where the arguments lie);
// rows, stack_hdrs_ and frames_ are then not used.
template <bool COUNT, int APPLY, uint32_t INLINE, bool WALKS, int PARTS = 0>
__global__ __launch_bounds__(fill_threads(PARTS), WALKS ? (PARTS > kFillThreads ? 6 : 4) : 8) void fill_kernel(const InlineStates<INLINE> states_, const RowDesc* __restrict__ rows,
                                                            const uint32_t* __restrict__ stack_hdrs_,
                                                            const uint16_t* __restrict__ frames_, DevVocab voc,
                                                            uint32_t* __restrict__ out, OverflowLog* log, uint32_t seq,
                                                            unsigned long long* step_counter, FusedApply fa, uint32_t wave_walks) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int kThreads = fill_threads(PARTS);
  __shared__ FillShared<WALKS, kThreads> sm;
  const XGM_GLOBAL uint32_t* stack_hdrs = (const XGM_GLOBAL uint32_t*)stack_hdrs_;
  const uint32_t tid = threadIdx.x;
  const int32_t b = (int32_t)blockIdx.y, seg = (int32_t)blockIdx.x;
  // PARTS: 1 << kPartShift workgroups share the segment, each with its part of the words (the lists are read by all of them)
  const int32_t part_words = PARTS ? kSegWords >> kPartShift : kSegWords;
  const int32_t w_begin = seg * kSegWords + (PARTS ? (int32_t)blockIdx.z * part_words : 0);
  const int32_t n_words = min(part_words, voc.W - w_begin);
  const int32_t id0 = w_begin * 32;
  const uint32_t n_ids = (uint32_t)part_words * 32u;
  // LDS is cleared before anything is fetched (a barrier waits for what its threads have in flight)
  for (int32_t w = tid; w < kSegWords; w += kThreads) sm.words[w] = 0u;
  if constexpr (WALKS)
    if (tid == 0) sm.n_queued = 0u;
  __syncthreads();
  // (in the address space of kernel arguments: what is read from there is known to be the same for all threads)
  const XGM_CONST uint32_t* states = INLINE ? (const XGM_CONST uint32_t*)__builtin_amdgcn_kernarg_segment_ptr() : nullptr;
  const XGM_CONST uint32_t* key_off = nullptr;
  const XGM_GLOBAL uint32_t *acc, *entries;
  uint32_t n_stacks, flags, stack_begin;
  if constexpr (INLINE != 0) {
    const uint32_t r0 = states[2 * b], r1 = states[2 * b + 1];
    const XGM_CONST uint32_t* cache = states + (r1 & 0xFFFFu);
    stack_begin = r0 & 0xFFFFu;
    n_stacks = (r0 >> 16) & 0xFFu;
    flags = r0 >> 24;
    acc = (const XGM_GLOBAL uint32_t*)((uint64_t)cache[0] | ((uint64_t)cache[1] << 32));
    entries = (const XGM_GLOBAL uint32_t*)((uint64_t)cache[2] | ((uint64_t)cache[3] << 32));
    key_off = (const XGM_CONST uint32_t*)((uint64_t)cache[4] | ((uint64_t)cache[5] << 32));
  } else {
    const RowDesc rd = rows[b];
    stack_begin = rd.stack_begin;
    n_stacks = rd.n_stacks;
    flags = rd.flags;
    acc = (const XGM_GLOBAL uint32_t*)rd.acc;
    entries = (const XGM_GLOBAL uint32_t*)rd.entries;
  }
  const uint32_t hdr_stride = stack_hdr_stride(voc.n_seg);
  // may the request end here?  then its stop tokens are allowed (the first kThreads of them are fetched now)
  const bool may_end = flags & 1u;
  const int32_t my_stop = may_end && (int32_t)tid < voc.n_stop ? voc.stop_ids[tid] : -1;
  auto take = [&](uint32_t e, uint32_t stack) {
    const uint32_t rel = (e & kEntryIdMask) - (uint32_t)id0;
    if (PARTS && rel >= n_ids) return;
    if constexpr (WALKS) {
      if ((e >> kEntryKindShift) != kEntryAccepted) {
        const uint32_t at = atomicAdd(&sm.n_queued, 1u);
        if (at < kWalkQueue) sm.queue[at] = queue_entry(e, stack, (uint32_t)(seg * kSegTokens));
        return;
      }
    }
    atomicOr(&sm.words[rel >> 5], 1u << (rel & 31u));
  };
  // where the lists of a stack begin in this segment, and in the next (the same for every thread)
  auto lists_of = [&](uint32_t stack, uint32_t* acc_row, uint2 (&lst)[kStackLists]) {
    if constexpr (INLINE != 0) {
      const XGM_CONST uint32_t* sw = states + stack_begin + stack * kInlineStackWords;
      *acc_row = sw[0] >> 16;
#pragma unroll
      for (uint32_t l = 0; l < kStackLists; ++l) {
        const uint32_t key = sw[1 + l];
        if (key != kNoKey) {
          const XGM_CONST uint32_t* ko = key_off + ((size_t)key * (uint32_t)voc.n_seg + (uint32_t)seg);
          lst[l] = make_uint2(ko[0], ko[1]);
        }
      }
    } else {
      const XGM_GLOBAL uint32_t* sh = stack_hdrs + (size_t)(stack_begin + stack) * hdr_stride;
      *acc_row = sh[kStackHdrTop] >> 16;
      static_assert(kStackLists == 4, "the offsets of a segment's four lists are one 16-byte load");
      const uint4* off = reinterpret_cast<const uint4*>(stack_hdrs_ + (size_t)(stack_begin + stack) * hdr_stride +
                                                        stack_hdr_off((uint32_t)seg, 0u));
      const uint4 o0 = off[0], o1 = off[1];
      lst[0] = make_uint2(o0.x, o1.x);
      lst[1] = make_uint2(o0.y, o1.y);
      lst[2] = make_uint2(o0.z, o1.z);
      lst[3] = make_uint2(o0.w, o1.w);
    }
  };
  // 1 + 2. Two stacks at a time: their headers (the same words for every thread), then, in one go, this
  // thread's words of their bitset rows (Algorithm 1: the union over the parallel stacks) and the first
  // kThreads entries of their lists (most lists are shorter than that); then what is left of the lists.
  constexpr int kWordsPerThread = std::max(1, kSegWords / kThreads);
  for (uint32_t s0 = 0; s0 < n_stacks; s0 += 2u) {
    uint32_t acc_row[2];
    uint2 lst[2][kStackLists];
#pragma unroll
    for (uint32_t q = 0; q < 2u; ++q) {
      acc_row[q] = kNoAccRow;
#pragma unroll
      for (uint32_t l = 0; l < kStackLists; ++l) lst[q][l] = make_uint2(0u, 0u);
      if (s0 + q < n_stacks) lists_of(s0 + q, &acc_row[q], lst[q]);
    }
    uint32_t aw[2][kWordsPerThread], first[2][kStackLists];
    bool have[2][kStackLists];
#pragma unroll
    for (uint32_t q = 0; q < 2u; ++q) {
#pragma unroll
      for (int k = 0; k < kWordsPerThread; ++k) {
        const int32_t w = (int32_t)tid + k * kThreads;
        aw[q][k] = acc_row[q] != kNoAccRow && w < n_words ? acc[(size_t)acc_row[q] * voc.W + w_begin + w] : 0u;
      }
#pragma unroll
      for (uint32_t l = 0; l < kStackLists; ++l) {
        have[q][l] = false;
        first[q][l] = 0u;
        if (lst[q][l].x < lst[q][l].y) {  // (the same for every thread: an empty list costs a scalar compare)
          have[q][l] = lst[q][l].x + tid < lst[q][l].y;
          if (have[q][l]) first[q][l] = entries[lst[q][l].x + tid];
        }
      }
    }
#pragma unroll
    for (uint32_t q = 0; q < 2u; ++q) {
#pragma unroll
      for (int k = 0; k < kWordsPerThread; ++k)
        if (aw[q][k]) atomicOr(&sm.words[tid + k * kThreads], aw[q][k]);
#pragma unroll
      for (uint32_t l = 0; l < kStackLists; ++l) {
        if (lst[q][l].x < lst[q][l].y) {
          if (have[q][l]) take(first[q][l], s0 + q);
          if (lst[q][l].y - lst[q][l].x > (uint32_t)kThreads)
            for (uint32_t j = lst[q][l].x + kThreads + tid; j < lst[q][l].y; j += kThreads) take(entries[j], s0 + q);
        }
      }
    }
  }
  if (may_end)
    for (int32_t k = tid; k < voc.n_stop; k += kThreads) {
      const int32_t rel = (k == (int32_t)tid ? my_stop : voc.stop_ids[k]) - id0;
      if (rel >= 0 && rel < n_words * 32) atomicOr(&sm.words[rel >> 5], 1u << (rel & 31));
    }
  __syncthreads();
  // 3. walk entries, if any
  if constexpr (WALKS) {
    if (sm.n_queued != 0u) {
      WalkRow row;
      DevTables tab;
      if constexpr (INLINE != 0) {
        const XGM_CONST uint32_t* cache = states + (states[2 * b + 1] & 0xFFFFu);
        tab = *(const DevTables*)((uint64_t)cache[6] | ((uint64_t)cache[7] << 32));
        row.stacks = (const XGM_GLOBAL uint32_t*)(uint64_t)(states + stack_begin);
        row.frames = (const XGM_GLOBAL uint16_t*)(uint64_t)states;
        row.stride = kInlineStackWords;
        row.frame0 = states[stack_begin + 5u] >> 16;
        row.n_frames = states[2 * b + 1] >> 16;
        row.epoch = 0u;
      } else {
        tab = rows[b].tab;
        row.stacks = stack_hdrs + (size_t)stack_begin * hdr_stride;
        row.frames = (const XGM_GLOBAL uint16_t*)frames_;
        row.stride = hdr_stride;
        row.frame0 = rows[b].frame_begin;
        row.n_frames = rows[b].n_frames;
        row.epoch = rows[b].epoch;
      }
      unsigned long long my_steps = 0;
      stage_tables_async(tab, smem, kThreads);  // (through registers: launches of 8 to 64 rows that walk take 1.01 to 1.04 times as long)
      if (row.n_frames <= kFillFramesLds) {
#pragma unroll 1
        for (uint32_t k = tid; k < row.n_frames; k += kThreads) sm.live[k] = row.frames[row.frame0 + k];
      }
      staged();
      __syncthreads();
      // the queue, or, if it overflowed, list after list
      const uint32_t n_queued = sm.n_queued;
      const bool again = n_queued > kWalkQueue;
      // (the waves' walk lies right behind: where the lanes' comes in between, a launch of few rows takes 0.2 us longer)
      if (!COUNT && __builtin_expect(n_queued <= wave_walks && small_sections_staged(tab) && row.n_frames <= kFillFramesLds, 1))
        fill_walks_by_wave<APPLY != 0, INLINE != 0, kThreads>(LdsTabT<true, true>(tab, smem), sm, row, b, id0, n_queued, voc, log, seq);
      else
#pragma unroll 1
      for (uint32_t k = 0; k < (again ? n_stacks * kStackLists : 1u); ++k) {
        uint2 list = make_uint2(0u, n_queued);
        if (again) {
          uint32_t acc_row;
          uint2 lst[kStackLists] = {};
          lists_of(k / kStackLists, &acc_row, lst);
          list = k % kStackLists == 0u ? lst[0] : k % kStackLists == 1u ? lst[1] : k % kStackLists == 2u ? lst[2] : lst[3];
        }
        const XGM_GLOBAL uint32_t* from = again ? entries + list.x : nullptr;
        if (small_sections_staged(tab))
          fill_walks<COUNT, APPLY != 0, INLINE != 0, kThreads>(LdsTabT<true>(tab, smem), sm, row, b, id0, n_ids, from, k / kStackLists, list.y - list.x, voc, log, seq, my_steps);
        else
          fill_walks<COUNT, APPLY != 0, INLINE != 0, kThreads>(LdsTab(tab, smem), sm, row, b, id0, n_ids, from, k / kStackLists, list.y - list.x, voc, log, seq, my_steps);
      }
      __syncthreads();
      if (COUNT && my_steps) atomicAdd(step_counter, my_steps);
    }
  }
  // 4. the words, and the logits of the segment; the last segment also takes the columns beyond the vocabulary
  for (int32_t w = tid; w < n_words; w += kThreads) out[(size_t)b * voc.W + w_begin + w] = sm.words[w];
  if constexpr (APPLY != 0) {
    const bool last = seg + 1 == voc.n_seg && (!PARTS || blockIdx.z + 1u == 1u << kPartShift);
    const int32_t e_end = last ? fa.V_logits : min(id0 + (int32_t)n_ids, fa.V_logits), lane = (int32_t)(tid & 63u);
    unsigned char* const logits = fa.logits + (size_t)b * fa.row_stride * APPLY;
    for (int32_t e0 = id0 + (int32_t)uniform(tid >> 6) * kApplyWaveElems; e0 < e_end; e0 += kThreads / 64 * kApplyWaveElems) {
      const int32_t e = e0 + lane * 32;  // (words beyond the vocabulary's are zero, and so are the bits of its last one)
      uint32_t allowed = e < id0 + (int32_t)n_ids ? sm.words[(e - id0) >> 5] : 0u;
      if (e + 32 > e_end) allowed |= e < e_end ? ~0u << (e_end - e) : ~0u;
      apply_wave<APPLY>(logits + (size_t)e0 * APPLY, allowed, fa.neg_inf);
    }
  }
}


// ------------------------------------------------- device-resident states
constexpr int kAcceptThreads = 512;
constexpr int kErrTokenRejected = -6, kErrTerminated = -7, kErrTooManyStacks = -8, kErrTooLarge = -9, kErrBadArg = -1, kErrInternal = -11;

// What the walks of an accept leave behind: for every stack that the token can end in, which of the row's stacks it
// comes from, how many of that one's frames it keeps, and the frames above them (bottom first, the current node
// last).  The frames it keeps are not copied by the lane that walks - it would fetch and store a deep stack frame
// by frame - but by the whole workgroup when the next state is written.
constexpr uint32_t kAcceptHeaders = 1024;  // node headers staged at most
constexpr uint32_t kNewFrames = kArenaFrames + 1;
struct AcceptShared {
  uint16_t live[kBatchRowFrames];                    // the row's frames
  uint16_t fresh[kBatchMaxCandidates][kNewFrames + 1];
  uint32_t from[kBatchMaxCandidates];                // stack it comes from | frames kept << 8 | new frames << 16
  uint32_t less[kBatchMaxCandidates];                // the candidates that come before it, as a bit set
  uint32_t stack[kBatchMaxStacks];                   // the row's stacks: first frame in `live` | frames << 16
  uint32_t common[kBatchMaxStacks][kBatchMaxStacks]; // frames that two of them have in common, from the bottom
  uint32_t slot_of[kBatchMaxStacks];                 // the new stacks in order
  uint32_t mem[kAcceptThreads / 64][kWaveMemWords];
  alignas(DevCache) uint32_t cache[sizeof(DevCache) / 4];  // the row's DevCache
  uint32_t count, overflow, duplicates, can_end, bad_context, n_frames;
  __device__ __forceinline__ uint32_t kept(uint32_t i) const { return (from[i] >> 8) & 0xFFu; }
  __device__ __forceinline__ uint32_t depth(uint32_t i) const { return kept(i) + (from[i] >> 16); }
  __device__ __forceinline__ uint32_t frame(uint32_t i, uint32_t k) const {  // frame k of candidate i, from the bottom
    const uint32_t f = from[i], d = (f >> 8) & 0xFFu;
    return k < d ? live[(stack[f & 0xFFu] & 0xFFFFu) + k] : fresh[i][k - d];
  }
};
// The end policy of the walk (see walk_token): notes where the token can end.  A top node that can only return is
// returned from first, so that equal states get equal stacks.
template <class Tab>
struct NoteStacks {
  static constexpr bool kEnumerate = true;
  const Tab* T;
  AcceptShared* sm;
  uint32_t stack;
  template <class Mem, class Live>
  __device__ __forceinline__ void operator()(uint32_t n, uint32_t sp, const Mem& mem, const Live& live) const {
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t i = 0u;
    if (lane == 0u) i = atomicAdd(&sm->count, 1u);  // (a stack too many or too deep is the end of the accept anyway)
    while (T->is_dead_end(n)) {
      if (sp < kLiveBase) {
        const uint32_t fr = mem.frame(sp);
        n = fr & 0xFFFFu;
        sp = fr >> 16;
      } else {
        const uint32_t d = sp - kLiveBase;
        if (d == 0) break;
        n = live[d - 1];
        sp = kLiveBase + d - 1;
      }
    }
    // lane k: the new frame k + 1 below the top
    static_assert(kArenaFrames <= 64, "the new frames of a stack fit the lanes");
    uint32_t m = 1u, h = sp, mine = 0u;
    for (; h < kLiveBase; ++m) {
      const uint32_t fr = mem.frame(h);
      mine = lane + 1u == m ? fr & 0xFFFFu : mine;
      h = fr >> 16;
    }
    const uint32_t d = h - kLiveBase;  // frames kept
    i = uniform(i);
    if (d + m > kBatchMaxDepth || i >= kBatchMaxCandidates) { sm->overflow = 1u; return; }
    sm->from[i] = stack | (d << 8) | (m << 16);
    sm->fresh[i][m - 1u] = (uint16_t)n;
    if (lane + 1u < m) sm->fresh[i][m - 2u - lane] = (uint16_t)mine;
  }
};
// the order of candidates: element by element from the bottom, the shorter first (the host's order of stacks)
__device__ __forceinline__ int compare_candidates(const AcceptShared& sm, uint32_t i, uint32_t j) {
  const uint32_t si = sm.from[i] & 0xFFu, sj = sm.from[j] & 0xFFu, di = sm.depth(i), dj = sm.depth(j);
  uint32_t k = min(sm.kept(i), sm.kept(j));
  if (si != sj) k = min(k, sm.common[si][sj]);
  for (const uint32_t m = min(di, dj); k < m; ++k) {
    const uint32_t a = sm.frame(i, k), b = sm.frame(j, k);
    if (a != b) return a < b ? -1 : 1;
  }
  return di == dj ? 0 : (di < dj ? -1 : 1);
}

// Section 3.3 on the device: one workgroup per row moves the row's stacks on
// by the row's token.  A wave walks the token from one stack after the other
// and notes every stack it can end in; duplicates are removed, the rest
// is put in the host's order and packed as the next state of the row's ring,
// in the layout the fill kernel reads (stack headers with their lists' segment
// offsets; frames).  A row whose token is not allowed, or whose new state does
// not fit the device limits, keeps its state and gets an error code in `status`.
// Bound by latency: a row is one workgroup, and what it does is one chain - state,
// walk, order, contexts, keys, offsets.  So everything that does not depend on
// the walk is fetched at once in front of it (frames and tables into LDS, by 512
// threads: a pass of 128 schema rows takes 1 us less than with 256, one of a JSON row
// as long), and a wave works out a new stack by itself, its frames and their headers
// one in each lane: what used to be five barriers with a lookup or two between them is
// one memory round for the contexts (DevCache::node_ctx_first), one for each level's
// key and one for the offsets.  A round takes 500 clocks (another kernel wrote the state, so no cache holds it), and the
// compiler makes one of every load that it cannot move in front of a branch: the state, the tables (fetched straight into
// LDS) and the row's DevCache are fetched by all threads alike, each list's offsets along with the next list's key, and
// nothing is stored before the last load has come.  In-kernel clocks, mean of 128 schema rows: 3580 until state and tables
// are there (4940 with the pieces of the tables one after the other), walk 3700 (4580), stacks 4400 (5910, with a wave's sum
// for the first stack too and the DevCache's pointers read one by one where they were needed), the rest 360; a JSON row
// that stays in a string 9280 in all, before 11300.  The launch lasts as long as its slowest row (a twelve-byte token
// through several frames: 17 000 clocks of walk, 27 000 before walk_wave took moves in a loop of their own).  Before all of this
// (walk_wave's part included) a pass of four fills and three accepts of 128 schema rows took 1.11 to 1.20 times as long, one of
// five and four of 8 rows of the scripting grammar 1.09 to 1.15, of one JSON row 1.05 to 1.14 (four draws of states each: 62 to
// 73, 50 to 64 and 44 to 47 us now).  Of that, without the tables straight into LDS 1.00 to 1.02, with the DevCache read where
// it lies 1.02 to 1.04, with __syncthreads() for the last barrier 0.99 to 1.03: no difference beyond the spread.
// With one lane per stack, tables in global memory and stacks copied
// by that lane: 17.9 us for the launch; one JSON row 8.2 us, now 5.7;
// rows of the C/SQL-like grammar, 90 frames deep, 46 us in the mean, now 10.
__global__ __launch_bounds__(kAcceptThreads) void batch_accept_kernel(DevBatch bt, DevVocab voc, uint32_t lds_budget,
                                                                      const int32_t* __restrict__ tokens) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ AcceptShared sm;
  const uint32_t tid = threadIdx.x;
  const int32_t b = blockIdx.x;
  // what the row needs is fetched before anything is decided (a branch in between would make each round wait)
  const int32_t tok = tokens[b];
  const int32_t head = bt.head[b];
  const DevCache& dc = bt.cache[b];
  // (of a large grammar only the first headers: its literals are walked through a few lines of the others)
  const DevTables tab = staged_for(dc.tab, (int32_t)min(lds_budget, dc.tab.off_hdr + kAcceptHeaders * 8u));
  const int32_t first_stop = voc.n_stop > 0 ? voc.stop_ids[0] : -1;
  const uint4 tk = voc.tok_by_id[tok >= 0 && tok < voc.V ? tok : 0];
  const uint32_t hdr_stride = stack_hdr_stride(bt.n_seg);
  const uint32_t at = (uint32_t)b * bt.H + head;
  const SlotMeta cur = bt.meta[at];
  const uint32_t epoch = bt.rows[b].epoch;
  const int32_t older = bt.older[b];
  if (tok < 0) return;  // this row is left alone (its status too)
  // (every thread fetches, whether there is something for it or not: a load under a condition is waited for at its end)
  static_assert(kStackHdrTop == 0 && kStackHdrDepth == 1 && kStackHdrFrames == 2, "a stack's scalars lie side by side");
  static_assert(kAcceptThreads >= sizeof(DevCache) / 4 && sizeof(DevCache) % 8 == 0, "a word of the DevCache for each thread");
  static_assert(alignof(AcceptShared) >= alignof(DevCache) && offsetof(AcceptShared, cache) % alignof(DevCache) == 0, "its pointers are read from there");
  const uint32_t* const frames = reinterpret_cast<const uint32_t*>(bt.frames + (size_t)at * kBatchRowFrames);
  const uint32_t* const h = bt.hdrs + (size_t)(at * kBatchMaxStacks + tid % kBatchMaxStacks) * hdr_stride;
  const uint32_t two = frames[tid], h_depth = h[kStackHdrDepth], h_frames = h[kStackHdrFrames];
  const uint32_t word = reinterpret_cast<const uint32_t*>(&dc)[min(tid, (uint32_t)(sizeof(DevCache) / 4) - 1u)];
  stage_tables_async(tab, smem, kAcceptThreads);
  reinterpret_cast<uint32_t*>(sm.live)[tid] = two;
  if (tid < sizeof(DevCache) / 4) sm.cache[tid] = word;
  if (tid < kBatchMaxStacks) sm.stack[tid] = (h_frames - at * kBatchRowFrames) | (h_depth << 16);
  for (uint32_t k = tid + kAcceptThreads; k * 2u < cur.n_frames; k += kAcceptThreads) reinterpret_cast<uint32_t*>(sm.live)[k] = frames[k];
  if (tid == 0) { sm.count = 0u; sm.overflow = 0u; sm.duplicates = 0u; sm.can_end = 0u; sm.bad_context = 0u; }
  if (tid < kBatchMaxCandidates) sm.less[tid] = 0u;
  int32_t status = 0;
  bool stop = false;
  if (tok >= voc.V) status = kErrBadArg;
  else if (cur.flags & 2u) status = kErrTerminated;
  else {
    stop = tok == first_stop;
    for (int32_t k = 1; k < voc.n_stop; ++k) stop = stop || voc.stop_ids[k] == tok;
    if (stop && !(cur.flags & 1u)) status = kErrTokenRejected;
  }
  int len = (int)(tk.w >> 24);
  if (status == 0 && !stop && len == 0) status = kErrTokenRejected;
  staged();
  if (status != 0) {
    if (tid == 0) bt.status[b] = status;
    return;
  }
  __syncthreads();
  const uint32_t n_off = (uint32_t)bt.n_seg + 1u;
  const int32_t next = head + 1 == bt.H ? 0 : head + 1;
  const uint32_t sb = ((uint32_t)b * bt.H + next) * kBatchMaxStacks;
  const uint32_t fb = ((uint32_t)b * bt.H + next) * kBatchRowFrames;
  uint32_t ns = 0u, n_frames = 0u, can_end = 0u;
  const LdsTab T(tab, smem);
  if (!stop) {
    const uint32_t wave = uniform(tid >> 6), lane = tid & 63u;
    {
      const uint8_t* ext = voc.bytes;
      if (len >= 15) {
        ext = voc.bytes + voc.off_by_id[tok];
        if (len == 255) len = (int)(voc.off_by_id[tok + 1] - voc.off_by_id[tok]);
      }
      const LdsTabT<false, true> U(tab, smem);
      const LdsTabT<true, true> S(tab, smem);
      WaveMem mem{(XGM_LDS uint32_t*)sm.mem[wave], (XGM_LDS uint32_t*)sm.mem[wave] + kArenaFrames};
      for (uint32_t st = wave; st < cur.n_stacks; st += kAcceptThreads / 64) {
        const uint32_t where = uniform(sm.stack[st]), depth = where >> 16;
        const UniformFrames live{(const XGM_LDS uint16_t*)sm.live + (where & 0xFFFFu)};
        int res;
        if (small_sections_staged(tab)) {
          const NoteStacks<LdsTabT<true, true>> note{&S, &sm, st};
          res = walk_wave(S, mem, tk, ext, len, live[depth - 1u], live, depth, note);
        } else {  // (a grammar whose tables are too large)
          const NoteStacks<LdsTabT<false, true>> note{&U, &sm, st};
          res = walk_token_in<false, true>(mem, U, tk, ext, len, live[depth - 1u], live, depth, (uint32_t*)nullptr, 0u, 0, (uint32_t*)nullptr, note);
        }
        if (res == kOverflow) sm.overflow = 1u;
      }
    }
    // what the row's stacks have in common (the last waves get here first)
    if (cur.n_stacks > 1u)
      for (uint32_t p = kAcceptThreads / 64 - 1u - wave; p < cur.n_stacks * cur.n_stacks; p += kAcceptThreads / 64) {
        const uint32_t x = p / cur.n_stacks, y = p % cur.n_stacks;
        if (x >= y) continue;
        const uint32_t sx = sm.stack[x], sy = sm.stack[y], m = min(sx >> 16, sy >> 16);
        uint32_t same = m;
        for (uint32_t k0 = 0; k0 < m; k0 += 64u) {
          const uint32_t k = k0 + lane;
          const unsigned long long differ = __ballot(k < m && sm.live[(sx & 0xFFFFu) + k] != sm.live[(sy & 0xFFFFu) + k]);
          if (differ) { same = k0 + (uint32_t)__ffsll((long long)differ) - 1u; break; }
        }
        if (lane == 0u) sm.common[x][y] = sm.common[y][x] = same;
      }
    __syncthreads();
    const uint32_t nc = sm.count;
    if (sm.overflow) status = kErrTooLarge;
    else if (nc == 0u) status = kErrTokenRejected;
    if (status != 0) {
      if (tid == 0) bt.status[b] = status;
      return;
    }
    // duplicates out, the rest in order: all pairs at once
    if (nc > 1u) {
      for (uint32_t p = tid; p < nc * nc; p += kAcceptThreads) {
        const uint32_t i = p / nc, j = p % nc;
        if (j >= i) continue;
        const int c = compare_candidates(sm, j, i);
        if (c == 0) atomicOr(&sm.duplicates, 1u << i);
        else if (c < 0) atomicOr(&sm.less[i], 1u << j);
        else atomicOr(&sm.less[j], 1u << i);
      }
      __syncthreads();
    }
    const uint32_t dup = sm.duplicates;
    ns = nc - (uint32_t)__popc(dup);
    if (ns > kBatchMaxStacks) {
      if (tid == 0) bt.status[b] = kErrTooManyStacks;
      return;
    }
    if (nc > 1u) {
      if (tid < nc && !((dup >> tid) & 1u)) sm.slot_of[__popc(sm.less[tid] & ~dup)] = tid;
      __syncthreads();
    }
    // A wave writes out a stack, and works out where its lists lie: which context of its rule the frame above each level
    // sits on (a lane per level), the keys (one after the other), the offsets of their segments (a lane per segment).
    for (uint32_t r = wave; r < ns; r += kAcceptThreads / 64) {
      const uint32_t ci = nc > 1u ? uniform(sm.slot_of[r]) : 0u, d = uniform(sm.depth(ci));
      // lane k: the frame k below the top (below the 64th: looked up when they are needed)
      const uint32_t mine = lane < d ? sm.frame(ci, d - 1u - lane) : 0u;
      const uint32_t top = uniform(mine);
      const DevCache& own = *reinterpret_cast<const DevCache*>(sm.cache);  // (its pointers are to global memory: see `fetch`)
      auto fetch = [](const auto* p, size_t k) { return ((const XGM_GLOBAL std::decay_t<decltype(*p)>*)p)[k]; };
      uint32_t child = own.k_base[0] != nullptr ? fetch(own.k_base[0], top) : kNoKey;
      const uint32_t acc_row = fetch(own.acc_row, top);
      const uint32_t flags = T.header(mine).y;
      const uint32_t first = fb + (r ? wave_sum(lane < r ? sm.depth(sm.slot_of[lane]) : 0u) : 0u);
      auto node_at = [&](uint32_t k) { return sm.frame(ci, d - 1u - k); };
      const uint32_t drops = stack_drops(d, [&](uint32_t k) {
        const uint32_t y = k < 64u ? (uint32_t)__builtin_amdgcn_readlane((int)flags, (int)k) : T.header(node_at(k)).y;
        return (uniform(y) >> kHdrChainShift) & kHdrChainMask;
      });
      // which context of its rule the frame above level `lane` + 1 sits on
      const uint32_t from = lane < (uint32_t)kCtxLevels ? stack_drop(drops, lane + 1u) : 255u;
      uint32_t above = (uint32_t)__shfl((int)flags, (int)(from - 1u) & 63, 64), below = (uint32_t)__shfl((int)mine, (int)from & 63, 64);
      uint32_t idx = kNoKey;
      if (from < d) {
        if (from > 64u) above = T.header(node_at(from - 1u)).y;
        if (from > 63u) below = node_at(from);
        const uint32_t rule = above >> 16;
        const u64 both = fetch(reinterpret_cast<const u64*>(own.node_ctx_first), below);
        const uint32_t of_x = (uint32_t)both, of_y = (uint32_t)(both >> 32);
        if ((of_x >> 16) == rule) idx = of_x & 0xFFFFu;
        else if (of_y != kNoKey)
          for (uint32_t k = 1u; k <= fetch(own.node_ctx, of_y); ++k) {
            const uint32_t x = fetch(own.node_ctx, of_y + k);
            if ((x >> 16) == rule) idx = x & 0xFFFFu;
          }
        if (idx == kNoKey) sm.bad_context = 1u;
      }
      // The keys: the top node's own list, then one per level that the stack reaches and the cache keeps.  Each key's number
      // is fetched with what the one before says, and where its list lies (a lane per segment) along with the next key's.
      uint32_t off[kStackLists];
      off[0] = fetch(own.key_off, (size_t)top * (uint32_t)bt.n_seg + min(lane, n_off - 1u));
      uint32_t keys[kStackLists], key0 = (uint32_t)own.n_nodes;
      keys[0] = top;
#pragma unroll
      for (uint32_t l = 1; l <= (uint32_t)kCtxLevels; ++l) {
        const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)idx, (int)l - 1);
        keys[l] = kNoKey;
        off[l] = 0u;
        child = uniform(child);
        if (child != kNoKey && c != kNoKey) {
          keys[l] = key0 + child + c;
          off[l] = fetch(own.key_off, (size_t)keys[l] * (uint32_t)bt.n_seg + min(lane, n_off - 1u));
          child = l < (uint32_t)kCtxLevels && own.k_base[l] != nullptr ? fetch(own.k_base[l], child + c) : kNoKey;
        } else {
          child = kNoKey;
        }
        key0 += own.n_k[l - 1u];
      }
      uint32_t* const h = bt.hdrs + (size_t)(sb + r) * hdr_stride;
      if (lane == 0u) *reinterpret_cast<uint4*>(h) = make_uint4(top | (acc_row << 16), d, first, drops);
      static_assert(kStackLists == 4, "the offsets of a segment's four lists are one 16-byte store");
      if (lane < n_off) *reinterpret_cast<uint4*>(h + stack_hdr_off(lane, 0u)) = make_uint4(off[0], off[1], off[2], off[3]);
      for (uint32_t sgm = lane + 64u; sgm < n_off; sgm += 64u) {
        uint32_t o[kStackLists];
#pragma unroll
        for (uint32_t l = 0; l < kStackLists; ++l) o[l] = keys[l] == kNoKey ? 0u : fetch(own.key_off, (size_t)keys[l] * (uint32_t)bt.n_seg + sgm);
        *reinterpret_cast<uint4*>(h + stack_hdr_off(sgm, 0u)) = make_uint4(o[0], o[1], o[2], o[3]);
      }
      // frames, and whether the stack can end the text: every frame of it may end its rule (behind what had to be
      // fetched: a wait for a load is one for the stores in front of it)
      bool all_final = lane >= d || (flags & 1u) != 0u;
      if (lane < d) bt.frames[first + d - 1u - lane] = (uint16_t)mine;
      for (uint32_t k = lane + 64u; k < d; k += 64u) {
        const uint32_t n = node_at(k);
        bt.frames[first + d - 1u - k] = (uint16_t)n;
        all_final = all_final && T.is_final(n);
      }
      if (__ballot(!all_final) == 0ull && lane == 0u) sm.can_end = 1u;
      if (r + 1u == ns && lane == 0u) sm.n_frames = first + d - fb;
    }
    lds_barrier();
    n_frames = sm.n_frames;
    can_end = sm.can_end;
    if (sm.bad_context) {  // a frame sits on a node that is no context of its rule: never the case for stacks the walk makes
      if (tid == 0) bt.status[b] = kErrInternal;
      return;
    }
  }
  if (tid == 0) {
    SlotMeta m;
    m.n_stacks = ns;
    m.n_frames = n_frames;
    m.flags = stop ? 3u : can_end;
    m.pad = 0u;
    bt.meta[(size_t)b * bt.H + next] = m;
    RowDesc& r = bt.rows[b];  // (its tables and lists stay the same)
    r.stack_begin = sb;
    r.n_stacks = m.n_stacks;
    r.flags = m.flags & 1u;
    r.frame_begin = fb;
    r.n_frames = m.n_frames;
    r.epoch = epoch + 1u;
    bt.head[b] = next;
    bt.older[b] = older + 1 < bt.H - 1 ? older + 1 : bt.H - 1;
    bt.status[b] = 0;
  }
}

// going back: one thread per row
__global__ void batch_rollback_kernel(DevBatch bt, const int32_t* __restrict__ steps) {
  const int32_t b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= bt.B) return;
  const int32_t k = steps[b];
  if (k <= 0) return;
  if (k > bt.older[b]) { bt.status[b] = kErrBadArg; return; }
  const int32_t head = ((bt.head[b] - k) % bt.H + bt.H) % bt.H;
  const SlotMeta m = bt.meta[(size_t)b * bt.H + head];
  RowDesc r = bt.rows[b];
  r.stack_begin = ((uint32_t)b * bt.H + head) * kBatchMaxStacks;
  r.frame_begin = ((uint32_t)b * bt.H + head) * kBatchRowFrames;
  r.n_stacks = m.n_stacks;
  r.n_frames = m.n_frames;
  r.flags = m.flags & 1u;
  r.epoch += 1u;
  bt.rows[b] = r;
  bt.head[b] = head;
  bt.older[b] -= k;
  bt.status[b] = 0;
}

// Forking (section 3.3: one state may be continued in several ways, as in tree
// decoding): row b takes over the current state of row src[b] as its next
// state.  All rows read the states as they were before the call: the first
// kernel only writes next slots, the second moves the rows over.
__global__ __launch_bounds__(256) void batch_fork_copy_kernel(DevBatch bt, const int32_t* __restrict__ src_rows) {
  const int32_t b = blockIdx.x;
  const int32_t src = src_rows[b];
  if (src < 0 || src == b) return;
  if (src >= bt.B || bt.cache[b].acc != bt.cache[src].acc) return;  // reported by the second kernel
  const uint32_t tid = threadIdx.x;
  const uint32_t hdr_stride = stack_hdr_stride(bt.n_seg);
  const uint32_t from = (uint32_t)src * bt.H + bt.head[src], to = (uint32_t)b * bt.H + (bt.head[b] + 1) % bt.H;
  const SlotMeta m = bt.meta[from];
  const uint32_t* sh = bt.hdrs + (size_t)from * kBatchMaxStacks * hdr_stride;
  uint32_t* dh = bt.hdrs + (size_t)to * kBatchMaxStacks * hdr_stride;
  for (uint32_t k = tid; k < m.n_stacks * hdr_stride; k += 256u) {
    uint32_t v = sh[k];
    if (k % hdr_stride == kStackHdrFrames) v = v - from * kBatchRowFrames + to * kBatchRowFrames;
    dh[k] = v;
  }
  for (uint32_t k = tid; k < m.n_frames; k += 256u) bt.frames[(size_t)to * kBatchRowFrames + k] = bt.frames[(size_t)from * kBatchRowFrames + k];
  if (tid == 0) bt.meta[to] = m;
}
__global__ void batch_fork_commit_kernel(DevBatch bt, const int32_t* __restrict__ src_rows) {
  const int32_t b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= bt.B) return;
  const int32_t src = src_rows[b];
  if (src < 0 || src == b) return;
  if (src >= bt.B || bt.cache[b].acc != bt.cache[src].acc) { bt.status[b] = kErrBadArg; return; }
  const int32_t next = (bt.head[b] + 1) % bt.H;
  const SlotMeta m = bt.meta[(size_t)b * bt.H + next];
  RowDesc r = bt.rows[b];
  r.stack_begin = ((uint32_t)b * bt.H + next) * kBatchMaxStacks;
  r.frame_begin = ((uint32_t)b * bt.H + next) * kBatchRowFrames;
  r.n_stacks = m.n_stacks;
  r.n_frames = m.n_frames;
  r.flags = m.flags & 1u;
  r.epoch += 1u;
  bt.rows[b] = r;
  bt.head[b] = next;
  const int32_t o = bt.older[b] + 1;
  bt.older[b] = o < bt.H - 1 ? o : bt.H - 1;
  bt.status[b] = 0;
}

// ---------------------------------------------------------------- kernel (c)
constexpr int kApplyThreads = 256;

// Section 2.1: logits of disallowed tokens become -inf.  One workgroup per (segment of kSegTokens elements, row), a
// quarter of it each wave.  Segments begin on 16 bytes, up to a group less one element in front of a row that does not:
// the bits are then put together from two words of the mask, and elements outside the row count as allowed.
// Bound by the stores: serving masks on 128 rows x 151936 bf16 take 6.9 us, fp32 11.1 (with a loop over the disallowed
// elements of a lane's group of 16 bytes 7.6 and 12.0); rows of 151937, of which every eighth is aligned, 7.6 (one
// element per thread, as such rows went before: 27.8).  16 x 100003: 3.6, before 4.3 (most of it the launch).
// ESIZE = bytes per element.
template <int ESIZE>
__global__ __launch_bounds__(kApplyThreads) void apply_kernel(unsigned char* __restrict__ logits, int64_t row_stride,
                                                              const uint32_t* __restrict__ bitmask, int32_t W_mask,
                                                              int32_t V_logits, int32_t V_mask,
                                                              const int32_t* __restrict__ row_index, uint32_t neg_inf) {
  static_assert(kApplyThreads / 64 * kApplyWaveElems == kSegTokens, "four waves take a segment");
  const int32_t j = blockIdx.y, lane = (int32_t)(threadIdx.x & 63u);
  const int64_t lrow = row_index ? row_index[j] : j;
  unsigned char* row = logits + (size_t)lrow * row_stride * ESIZE;
  const uint32_t* words = bitmask + (size_t)j * W_mask;
  const int32_t ahead = (int32_t)((uint32_t)reinterpret_cast<uintptr_t>(row) % 16u) / ESIZE;
  const int32_t e0 = (int32_t)blockIdx.x * kSegTokens + (int32_t)uniform(threadIdx.x >> 6) * kApplyWaveElems - ahead;
  if (e0 >= V_logits) return;
  const int32_t e = e0 + lane * 32, at = e >> 5;  // the lane's first element
  const uint32_t lo = at >= 0 && at < W_mask ? words[at] : 0u;
  const uint32_t hi = ahead != 0 && at + 1 < W_mask ? words[at + 1] : 0u;
  uint32_t allowed = __builtin_amdgcn_alignbit(hi, lo, (uint32_t)e & 31u);
  if (e + 32 > V_mask) allowed &= e < V_mask ? (1u << (V_mask - e)) - 1u : 0u;
  if (e < 0) allowed |= (1u << -e) - 1u;
  if (e + 32 > V_logits) allowed |= e < V_logits ? ~0u << (V_logits - e) : ~0u;
  apply_wave<ESIZE>(row + (ptrdiff_t)e0 * ESIZE, allowed, neg_inf);
}

// ------------------------------------------------------------ measurement aid
// Chains of dependent LDS reads with every wave slot of the device busy: the
// ceiling for the table lookups of the token walks (each step of a walk is a
// few such reads, each depending on the one before).
constexpr int kLookupThreads = 1024;
__global__ __launch_bounds__(kLookupThreads) void lds_lookup_kernel(uint32_t n_words, uint32_t hops, uint32_t* __restrict__ sink) {
  extern __shared__ __align__(16) unsigned char smem[];
  uint32_t* table = reinterpret_cast<uint32_t*>(smem);
  // a permutation with one long cycle: i -> (i * 5 + 1) mod n_words (n_words is a power of two)
  for (uint32_t k = threadIdx.x; k < n_words; k += kLookupThreads) table[k] = (k * 5u + 1u) & (n_words - 1u);
  __syncthreads();
  uint32_t at = (threadIdx.x * 97u + blockIdx.x) & (n_words - 1u);
  for (uint32_t h = 0; h < hops; ++h) at = table[at];
  if (at == 0xFFFFFFFFu) sink[0] = at;  // never true: keeps the chain alive
}

// ------------------------------------------------------------ static scratch
// Staging memory for the fill entry point that may not allocate: the per-step
// blob (row descriptors, stack headers, frames) goes here instead of into
// a buffer from hipMalloc.  Each device holds its own copy of the array at its
// own address until the process ends.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

}  // namespace

// In host code the array's name is only a stand-in for the symbol: its device
// address is looked up once per device, with that device current, and kept.
hipError_t static_scratch(void** out) {
  constexpr int kMaxDevices = 64;
  static void* ptr_of[kMaxDevices] = {};
  *out = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  if (!ptr_of[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    ptr_of[dev] = p;
  }
  *out = ptr_of[dev];
  return hipSuccess;
}

// ------------------------------------------------------------------ launchers
hipError_t launch_moves(const Moves& moves, hipStream_t stream) {
  uint32_t most = 0u;
  for (int k = 0; k < moves.count; ++k) most = std::max(most, moves.move[k].n);
  if (most == 0u) return hipSuccess;
  hipLaunchKernelGGL(moves_kernel, dim3(std::min((most + kMoveThreads - 1) / kMoveThreads, 1024u)), dim3(kMoveThreads), 0, stream, moves);
  return hipGetLastError();
}
void launch_first_byte(const DevTables& tab, uint4* first_byte, hipStream_t stream) {
  const uint32_t n_words = first_byte_words(tab.n_nodes);
  if (n_words == 0) return;
  hipLaunchKernelGGL(first_byte_kernel, dim3((n_words + 1) / 2), dim3(kFirstByteThreads), 0, stream, tab, n_words, first_byte);
}

void launch_classify(const DevTables& tab, const DevVocab& voc, const ClassifyArgs& args, hipStream_t stream) {
  if (args.n_nodes <= 0 || voc.V <= 0) return;
  const DevTables st = staged_for(tab, kClassifyLdsBudget);
  const bool small = st.stage_bytes <= kClassifySmallStage;
  const int32_t waves = (small ? kClassifyThreadsSmall : kClassifyThreadsLarge) / 64;
  const int32_t items = small ? kClassifyItemsSmall : kClassifyItems;
  static_assert(kClassifyItems % 8 == 0 && kClassifyItemsSmall % 8 == 0, "whole bytes of ClassifyArgs::some_acc");
  const dim3 grid(((voc.V + 63) / 64 + items - 1) / items, (args.n_nodes + kClassifyNodes - 1) / kClassifyNodes);
  const dim3 grid2(small ? kWalkBlocksSmall : kWalkBlocksLarge);
  hipLaunchKernelGGL((small ? classify_kernel<kClassifyThreadsSmall> : classify_kernel<kClassifyThreadsLarge>), grid, dim3(waves * 64), st.stage_bytes,
                     stream, st, voc, args, items);
  hipLaunchKernelGGL((small ? classify_walks_kernel<kClassifyThreadsSmall> : classify_walks_kernel<kClassifyThreadsLarge>), grid2, dim3(waves * 64),
                     st.stage_bytes, stream, st, voc, args);
}

void launch_permute(const DevVocab& voc, int32_t n, const uint32_t* a_rank, const uint32_t* b_rank, uint32_t* a_id,
                    uint32_t* b_id, uint32_t* seg_counts, unsigned long long* digest, uint32_t* a_counts, uint32_t* b_counts, hipStream_t stream) {
  if (n <= 0) return;
  hipLaunchKernelGGL(permute_kernel, dim3(n), dim3(kRowThreads), (size_t)voc.W * 8, stream, voc, a_rank, b_rank, a_id, b_id,
                     seg_counts, digest, a_counts, b_counts);
}

void launch_row_stats(const DevVocab& voc, const RankRows& rows, int32_t n, uint32_t* acc_id, unsigned long long* digest, hipStream_t stream) {
  if (n <= 0) return;
  hipLaunchKernelGGL(row_stats_kernel, dim3(n), dim3(kNodeThreads), 0, stream, voc, rows);
  hipLaunchKernelGGL(bitset_rows_kernel, dim3(std::min(n, 1024)), dim3(kBitsetThreads), (size_t)voc.W * 4, stream, voc, rows, acc_id, digest);
}
void launch_base_lists(const DevVocab& voc, const RankRows& rows, int32_t n, const uint32_t* first, uint32_t* ids, uint16_t* nodes, hipStream_t stream) {
  if (n > 0) hipLaunchKernelGGL(base_lists_kernel, dim3(n), dim3(kBaseListThreads), 0, stream, voc, rows, first, ids, nodes);
}
void launch_level0_lists(const DevVocab& voc, const RankRows& rows, int32_t n, const uint32_t* key_off, uint32_t* entries, hipStream_t stream) {
  if (n > 0) hipLaunchKernelGGL(level0_lists_kernel, dim3(n), dim3(kNodeThreads), 0, stream, voc, rows, key_off, entries);
}

void launch_rows_equal(const uint32_t* rows, int32_t n, int32_t W, const int32_t* rep, uint32_t* equal, hipStream_t stream) {
  if (n > 0) hipLaunchKernelGGL(rows_equal_kernel, dim3(n), dim3(kRowThreads), 0, stream, rows, W, rep, equal);
}
void launch_gather_rows(const uint32_t* rows, int32_t W, const int32_t* unique, int32_t n_unique, uint32_t* out,
                        hipStream_t stream) {
  if (n_unique > 0) hipLaunchKernelGGL(gather_rows_kernel, dim3(n_unique), dim3(kRowThreads), 0, stream, rows, W, unique, out);
}

void launch_rows_to_lists(const uint32_t* rows, int32_t row_words, int32_t n, const uint32_t* cursor_of,
                          int32_t per_row, uint32_t* cursor, uint32_t* out, uint16_t* out_row, hipStream_t stream) {
  const int32_t n_seg = (row_words + kSegWords - 1) / kSegWords;
  for (int32_t r0 = 0; r0 < n; r0 += 32768) {  // grid.y limit
    const int32_t nb = std::min(32768, n - r0);
    hipLaunchKernelGGL(rows_to_lists_kernel, dim3(n_seg, nb), dim3(kListThreads), 0, stream, rows + (size_t)r0 * row_words,
                       row_words, cursor_of + r0, per_row, cursor, out, out_row, r0);
  }
}

size_t slot_blocks(size_t n_slots) { return (n_slots + kSlotBlock - 1) / kSlotBlock; }
void launch_slot_offsets(const SlotCounts& counts, unsigned long long* block_sums, uint32_t* key_off, uint32_t* front, uint32_t* back,
                         unsigned long long* total, hipStream_t stream) {
  const dim3 grid((uint32_t)slot_blocks(counts.n_slots));  // (a grammar has a node, a vocabulary a segment)
  hipLaunchKernelGGL(slot_sums_kernel, grid, dim3(kSlotThreads), 0, stream, counts, block_sums);
  hipLaunchKernelGGL(slot_offsets_kernel, grid, dim3(kSlotThreads), 0, stream, counts, block_sums, key_off, front, back, total);
}

void launch_exit_positions(const DevTables& tab, const DevVocab& voc, const ContextListArgs& args, hipStream_t stream) {
  if (args.total == 0) return;
  const DevTables st = staged_for(tab, kContextLdsBudget);
  hipLaunchKernelGGL(exit_positions_kernel, dim3((args.total + kContextThreads - 1) / kContextThreads), dim3(kContextThreads),
                     st.stage_bytes, stream, st, voc, args);
}

void launch_context_lists(const DevTables& tab, const DevVocab& voc, const ContextListArgs& args, bool write, hipStream_t stream) {
  if (args.total == 0 || args.n_tiles == 0) return;
  const DevTables st = staged_for(tab, kContextLdsBudget);
  const dim3 g2(1024);
  if (write && args.outcomes) {
    // from the kept outcomes: the records of all levels are still there from the counting pass
    hipLaunchKernelGGL(context_level1_write_kernel, dim3(2048), dim3(kOpenWriteThreads), 0, stream, voc, args);
    for (uint32_t level = 2; level <= (uint32_t)kCtxLevels && args.k_base[level - 1] != nullptr; ++level)
      hipLaunchKernelGGL(context_deeper_write_kernel, g2, dim3(256), 0, stream, voc, args, level);
    return;
  }
  // the tiles whose contexts fit the list, if all of them have to be listed, at a time
  for (uint32_t tile0 = 0, k = 0; tile0 < args.n_tiles; ++k) {
    const uint32_t tile1 = args.tile_parts[k];
    if (tile0 > 0) (void)hipMemsetAsync(args.n_open, 0, 4, stream);
    const uint32_t waves = kContextThreads / 64, blocks = std::min((tile1 - tile0 + waves - 1) / waves, kOpenBlocks);
    hipLaunchKernelGGL(context_open_kernel, dim3(blocks), dim3(kContextThreads), st.stage_bytes, stream, st, voc, args, tile0, tile1 - tile0);
    auto kernel = write ? context_level1_kernel<true> : context_level1_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3(kOpenBlocks), dim3(kContextThreads), st.stage_bytes, stream, st, voc, args);
    tile0 = tile1;
  }
  for (uint32_t level = 2; level <= (uint32_t)kCtxLevels && args.k_base[level - 1] != nullptr; ++level) {
    if (write) hipLaunchKernelGGL(context_deeper_kernel<true>, g2, dim3(kContextThreads), st.stage_bytes, stream, st, voc, args, level);
    else hipLaunchKernelGGL(context_deeper_kernel<false>, g2, dim3(kContextThreads), st.stage_bytes, stream, st, voc, args, level);
  }
}

void launch_patch_classes(const DevVocab& voc, const uint32_t* items, int32_t n_items, uint32_t* acc_rank,
                          uint32_t* unc_rank, uint32_t* plain_rank, hipStream_t stream) {
  if (n_items <= 0) return;
  hipLaunchKernelGGL(patch_classes_kernel, dim3((n_items + 255) / 256), dim3(256), 0, stream, voc, items, n_items,
                     acc_rank, unc_rank, plain_rank);
}

void launch_upload_stacks(const void* src, void* dst, size_t plain_bytes, const void* src_stacks, uint32_t n_stacks,
                          int32_t n_seg, void* dst_hdrs, const void* src_frames, void* dst_frames, size_t frames_bytes,
                          hipStream_t stream) {
  static_assert(kStackKeysWords % 4 == 0 && kStackKeysWords >= kStackHdrWords + kStackLists + 2, "the key words of a stack");
  const uint32_t plain16 = (uint32_t)(plain_bytes / 16), frames16 = (uint32_t)((frames_bytes + 15) / 16);
  const uint32_t copy_blocks = (plain16 + frames16 + kUploadThreads - 1) / kUploadThreads;
  const uint32_t stack_blocks = (n_stacks + kStacksPerBlock - 1) / kStacksPerBlock;
  if (copy_blocks + stack_blocks == 0) return;
  hipLaunchKernelGGL(upload_stacks_kernel, dim3(copy_blocks + stack_blocks), dim3(kUploadThreads), 0, stream,
                     reinterpret_cast<const uint4*>(src), reinterpret_cast<uint4*>(dst), plain16,
                     reinterpret_cast<const uint4*>(src_frames), reinterpret_cast<uint4*>(dst_frames), frames16, copy_blocks,
                     reinterpret_cast<const uint4*>(src_stacks), n_stacks, (uint32_t)n_seg, reinterpret_cast<uint32_t*>(dst_hdrs));
}

void launch_batch_headers(const DevBatch& bt, int32_t row0, int32_t n, int32_t slot, int32_t older, hipStream_t stream) {
  static_assert(kStackKeysWords <= stack_hdr_stride(1), "the key words of a stack lie where its header belongs");
  hipLaunchKernelGGL(batch_headers_kernel, dim3(kBatchMaxStacks, n), dim3(64), 0, stream, bt, row0, slot, older);
}

// Walks take long, and few rows of a batch have many: where the segments alone do not fill the chip four workgroups share
// each, if a cache of the batch has many walk entries (C/SQL-like and scripting grammars have 1e4 to 1e6, JSON has
// 23 at 128256 tokens).  Fill of 32 rows of the scripting grammar, 128256 tokens: 51 -> 27 us; 64 rows of the C/SQL-like
// one, three draws: 41, 52, 121 -> 32, 34, 53 us; rows that walk little pay 1 us for reading the lists in every part.
// A workgroup's LDS is what the tables of the batch's caches with walk entries need, so that a full batch whose rows hardly
// ever walk does not run four workgroups per compute unit for it: one launch of 128 JSON rows x 151936, mask and bf16
// logits, 10.83 us with 31 KB for all of them, 9.84 so; 127 schema rows and one JSON row, or one of the scripting
// grammar, 9.3 and 8.46 (8.25 without that row); batches of rows that walk a lot take as long either way.
constexpr uint32_t kFillWalkSlots = 4 * 256;  // workgroups of 256 threads that the chip has room for if each has 31 KB of tables
// Threads of the workgroups that share segments.  With 512 twice the waves take the walks of a part, up to 15 of up to 40 000
// clocks in a row of the C/SQL-like grammar; three such workgroups fit a compute unit (scalar registers: 24 of 28 waves),
// whatever its tables.  Of those with 256 threads seven fit if the tables are small: where there are many times more workgroups
// than the chip holds, that counts for more.  Mask and bf16 logits in one launch, V = 128256, us with 256 and with 512 threads,
// two or three draws of states.  Tables of 10 KB (scripting grammar), by rows: 8: 7.0, 25.6 and 7.0, 21.0; 16: 11.0, 28.3 and
// 10.4, 24.3; 32: 28.7, 28.6 and 26.2, 26.5; 40 (2560 workgroups): 29.0, 28.7 and 29.2, 28.2; 44: 29.6, 31.7 and 29.9, 33.4;
// 64: 35.3, 33.9, 33.2 and 42.7, 40.3, 38.2; 128 rows x 64000: 35.6, 34.5 and 40.5, 37.2.  Tables of 26 KB (C/SQL-like: four
// workgroups of 256 threads, 16 waves): 24: 24 to 32, 38, 12.1 and 22.5, 32.5, 12.9; 40: 36.8, 55.7 and 33.2, 48.4; 64: 28.8
// to 36.7, 41.1, 59.7 and 32.3, 40.6, 55.6; 128 x 64000: 60.0, 61.8 and 56.4, 57.9; 200 x 32000: 56.6 and 49.5.
constexpr uint32_t kManyPartBlocks = 10 * 256;
static int part_threads(uint32_t blocks, uint32_t table_bytes) {
  constexpr uint32_t kLds = 160 * 1024;  // of a compute unit
  static_assert(3 * (sizeof(FillShared<true, 512>) + kFillLdsBudget) <= kLds, "three workgroups of 512 threads per compute unit");
  static_assert(4 * (sizeof(FillShared<true, kFillThreads>) + kFillLdsBudget) <= kLds, "four of 256");
  const uint32_t fit = std::min<uint32_t>(7u, kLds / (uint32_t)(sizeof(FillShared<true, kFillThreads>) + table_bytes));
  return blocks > kManyPartBlocks && fit * kFillThreads > 3u * 512u ? kFillThreads : 512;
}
template <bool COUNT, int APPLY, uint32_t INLINE>
static void launch_fill_of(const InlineStates<INLINE>& st, const RowDesc* rows, const uint32_t* stack_hdrs, const uint16_t* frames, int32_t B,
                           const DevVocab& voc, const FillWalks& walks, uint32_t* out, OverflowLog* log, uint32_t seq, unsigned long long* step_counter,
                           hipStream_t stream, const FusedApply& fa, hipEvent_t done = nullptr) {
  dim3 grid(voc.n_seg, B);
  const bool shared = walks.entries >= kManyWalks && grid.x * grid.y <= kFillWalkSlots;
  const int parts = shared ? part_threads(grid.x * grid.y << kPartShift, walks.table_bytes) : 0;
  if (shared) grid.z = 1u << kPartShift;
  auto kernel = walks.entries == 0u  ? fill_kernel<false, APPLY, INLINE, false>
                : parts == 0         ? fill_kernel<COUNT, APPLY, INLINE, true>
                : parts == 512       ? fill_kernel<COUNT, APPLY, INLINE, true, 512>
                                     : fill_kernel<COUNT, APPLY, INLINE, true, kFillThreads>;
  const dim3 threads(fill_threads(parts));
  const uint32_t wave_walks = walks.long_walks ? 0u : threads.x / 64u * kWaveWalks;
  if (done)
    hipExtLaunchKernelGGL(kernel, grid, threads, walks.table_bytes, stream, nullptr, done, 0, st, rows, stack_hdrs, frames, voc, out, log,
                          seq, step_counter, fa, wave_walks);
  else
    hipLaunchKernelGGL(kernel, grid, threads, walks.table_bytes, stream, st, rows, stack_hdrs, frames, voc, out, log, seq, step_counter, fa,
                       wave_walks);
}
void launch_fill(const RowDesc* rows, const uint32_t* stack_hdrs, const uint16_t* frames, int32_t B, const DevVocab& voc, const FillWalks& walks,
                 uint32_t* out, OverflowLog* log, uint32_t seq, unsigned long long* step_counter, hipStream_t stream,
                 void* logits, int elem_size, uint32_t neg_inf, int32_t V_logits, int64_t row_stride) {
  if (B <= 0) return;
  const FusedApply fa{static_cast<unsigned char*>(logits), row_stride, V_logits, neg_inf};
  auto launch = logits ? (elem_size == 2 ? launch_fill_of<false, 2, 0> : launch_fill_of<false, 4, 0>)
                       : (step_counter ? launch_fill_of<true, 0, 0> : launch_fill_of<false, 0, 0>);
  launch(InlineStates<0>{}, rows, stack_hdrs, frames, B, voc, walks, out, log, seq, step_counter, stream, fa, nullptr);
}
template <uint32_t WORDS>
static void launch_fill_inline_of(const uint32_t* states, uint32_t words, int32_t B, const DevVocab& voc, const FillWalks& walks, uint32_t* out,
                                  OverflowLog* log, uint32_t seq, hipStream_t stream, hipEvent_t done, int elem_size, const FusedApply& fa) {
  InlineStates<WORDS> st;
  std::copy(states, states + words, st.w);
  auto launch = fa.logits ? (elem_size == 2 ? launch_fill_of<false, 2, WORDS> : launch_fill_of<false, 4, WORDS>) : launch_fill_of<false, 0, WORDS>;
  launch(st, nullptr, nullptr, nullptr, B, voc, walks, out, log, seq, nullptr, stream, fa, done);
}
void launch_fill_inline(const uint32_t* states, uint32_t words, int32_t B, const DevVocab& voc, const FillWalks& walks, uint32_t* out, OverflowLog* log,
                        uint32_t seq, hipStream_t stream, hipEvent_t done, void* logits, int elem_size, uint32_t neg_inf, int32_t V_logits,
                        int64_t row_stride) {
  if (B <= 0) return;
  const FusedApply fa{static_cast<unsigned char*>(logits), row_stride, V_logits, neg_inf};
  if (words <= kInlineWordsSmall) launch_fill_inline_of<kInlineWordsSmall>(states, words, B, voc, walks, out, log, seq, stream, done, elem_size, fa);
  else launch_fill_inline_of<kInlineWordsLarge>(states, words, B, voc, walks, out, log, seq, stream, done, elem_size, fa);
}

void launch_lds_lookups(int32_t n_blocks, uint32_t hops, uint32_t* sink, hipStream_t stream) {
  hipLaunchKernelGGL(lds_lookup_kernel, dim3(n_blocks), dim3(kLookupThreads), 8192 * 4, stream, 8192u, hops, sink);
}

void launch_batch_accept(const DevBatch& bt, const DevVocab& voc, const int32_t* d_tokens, hipStream_t stream) {
  hipLaunchKernelGGL(batch_accept_kernel, dim3(bt.B), dim3(kAcceptThreads), kAcceptLdsBudget, stream, bt, voc, (uint32_t)kAcceptLdsBudget, d_tokens);
}

void launch_batch_fork(const DevBatch& bt, const int32_t* d_src_rows, hipStream_t stream) {
  hipLaunchKernelGGL(batch_fork_copy_kernel, dim3(bt.B), dim3(256), 0, stream, bt, d_src_rows);
  hipLaunchKernelGGL(batch_fork_commit_kernel, dim3((bt.B + 255) / 256), dim3(256), 0, stream, bt, d_src_rows);
}

void launch_batch_rollback(const DevBatch& bt, const int32_t* d_steps, hipStream_t stream) {
  hipLaunchKernelGGL(batch_rollback_kernel, dim3((bt.B + 255) / 256), dim3(256), 0, stream, bt, d_steps);
}

void launch_apply(void* logits, int elem_size, uint32_t neg_inf, int32_t V_logits, int64_t row_stride,
                  const uint32_t* bitmask, int32_t V_mask, const int32_t* row_index, int32_t n_rows,
                  hipStream_t stream) {
  if (n_rows <= 0 || V_logits <= 0) return;
  const int32_t W_mask = (V_mask + 31) / 32;
  unsigned char* p = static_cast<unsigned char*>(logits);
  // (a row begins up to a group less one element behind 16 bytes)
  const int32_t ahead = reinterpret_cast<uintptr_t>(logits) % 16 == 0 && row_stride * elem_size % 16 == 0 ? 0 : 16 / elem_size - 1;
  const dim3 grid((V_logits + ahead + kSegTokens - 1) / kSegTokens, n_rows);
  auto launch = elem_size == 2 ? apply_kernel<2> : apply_kernel<4>;
  hipLaunchKernelGGL(launch, grid, dim3(kApplyThreads), 0, stream, p, row_stride, bitmask, W_mask, V_logits, V_mask, row_index, neg_inf);
}

}  // namespace xgm
