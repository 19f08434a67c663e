#include "engine.hpp"

#include <algorithm>

#include "../../include/xgm.h"

namespace xgm {

namespace {
constexpr size_t kMaxConfigs = 1 << 16;   // configurations explored per byte
constexpr size_t kKeptFrames = 1 << 16;   // a larger pool is given back after the call

// All stacks of one advance() as paths in one tree (the persistent stack of section 3.3): a stack is the number of
// its top frame, a frame knows the frame below it, and equal stacks have equal numbers, so that "seen before?" is
// a comparison of a mark.  With a std::set of whole stacks accepting one token took 3 to 10 us, most of it
// allocations; it takes 0.2 to 0.5 us this way.
struct FramePool {
  struct Frame {
    int32_t below, node;
    uint32_t depth;
    uint32_t mark[3];  // last byte step in which the stack was seen: with / without a byte consumed since its last push; reached
  };
  std::vector<Frame> frames;
  std::vector<uint64_t> slots;  // call << 32 | frame number, hashed by (below, node); of earlier calls: empty
  uint32_t call = 0, step = 0;
  std::vector<std::pair<int32_t, bool>> work;
  std::vector<int32_t> cur, next;

  void begin() {
    if (slots.empty() || call == 0xFFFFFFFFu) { slots.assign(256, 0); call = 0; }
    ++call;
    frames.clear();
    step = 0;
  }
  void end() {
    if (frames.capacity() > kKeptFrames) { std::vector<Frame>().swap(frames); std::vector<uint64_t>().swap(slots); call = 0; }
    if (work.capacity() > kKeptFrames) std::vector<std::pair<int32_t, bool>>().swap(work);
    if (next.capacity() > kKeptFrames) { std::vector<int32_t>().swap(next); std::vector<int32_t>().swap(cur); }
  }
  static size_t hash(int32_t below, int32_t node) {
    uint64_t h = ((uint64_t)(uint32_t)below << 32 | (uint32_t)node) * 0x9E3779B97F4A7C15ull;
    return (size_t)(h >> 29);
  }
  int32_t push(int32_t below, int32_t node) {
    if (frames.size() * 2 >= slots.size()) grow();
    size_t at = hash(below, node) & (slots.size() - 1);
    for (; (uint32_t)(slots[at] >> 32) == call; at = (at + 1) & (slots.size() - 1)) {
      const Frame& f = frames[(uint32_t)slots[at]];
      if (f.below == below && f.node == node) return (int32_t)(uint32_t)slots[at];
    }
    const int32_t id = (int32_t)frames.size();
    slots[at] = (uint64_t)call << 32 | (uint32_t)id;
    frames.push_back({below, node, below < 0 ? 1u : frames[below].depth + 1u, {0u, 0u, 0u}});
    return id;
  }
  void grow() {
    std::vector<uint64_t>(slots.size() * 2, 0).swap(slots);
    for (size_t id = 0; id < frames.size(); ++id) {
      size_t at = hash(frames[id].below, frames[id].node) & (slots.size() - 1);
      while ((uint32_t)(slots[at] >> 32) == call) at = (at + 1) & (slots.size() - 1);
      slots[at] = (uint64_t)call << 32 | id;
    }
  }
  bool first_time(int32_t id, int which) {
    if (frames[id].mark[which] == step) return false;
    frames[id].mark[which] = step;
    return true;
  }
  void read(int32_t id, Stack* out) const {
    out->resize(frames[id].depth);
    for (size_t k = out->size(); k-- > 0; id = frames[id].below) (*out)[k] = frames[id].node;
  }
};
thread_local FramePool t_pool;

struct PoolGuard {
  FramePool& p;
  explicit PoolGuard(FramePool& pool) : p(pool) { p.begin(); }
  ~PoolGuard() { p.end(); }
};
}  // namespace

int Engine::advance(const std::vector<Stack>& in, const uint8_t* bytes, int n, std::vector<Stack>* out,
                    int* left_frame, size_t max_out, int32_t follow_rule) const {
  const Automaton& A = *A_;
  PoolGuard guard(t_pool);
  FramePool& P = t_pool;
  auto& cur = P.cur;
  auto& next = P.next;
  auto& work = P.work;
  enum { kConsumed = 0, kEntered = 1, kReached = 2 };
  cur.clear();
  ++P.step;
  for (const Stack& s : in) {
    int32_t id = -1;
    for (int32_t node : s) id = P.push(id, node);
    if (id >= 0 && P.first_time(id, kReached)) cur.push_back(id);
  }
  for (int i = 0; i < n; ++i) {
    const int c = bytes[i];
    next.clear();
    work.clear();
    ++P.step;
    size_t seen = 0;
    // configurations before byte i: (stack, consumed-a-byte-since-last-push)
    auto add = [&](int32_t id, bool consumed) {
      if (!P.first_time(id, consumed ? kConsumed : kEntered)) return;
      ++seen;
      work.emplace_back(id, consumed);
    };
    for (int32_t id : cur) add(id, true);
    while (!work.empty()) {
      const auto [id, consumed] = work.back();
      work.pop_back();
      const int32_t node = P.frames[id].node, below = P.frames[id].below;
      const uint32_t depth = P.frames[id].depth;
      for (auto& e : A.bedges[node])
        if (e.lo <= c && c <= e.hi) {
          const int32_t to = P.push(below, e.to);
          if (P.first_time(to, kReached)) next.push_back(to);
          break;
        }
      for (auto& e : A.redges[node])
        if (A.first[e.rule].test(c)) {
          if ((int)depth + 1 > XGM_MAX_STACK_DEPTH) return XGM_ERR_TOO_LARGE;
          // returning to a dead end = returning to our parent
          const int32_t under = A.node_dead_end[e.to] ? below : P.push(below, e.to);
          add(P.push(under, A.rule_start[e.rule]), false);
        }
      // the rule may end here; an instance must have consumed a byte
      if (A.node_final[node] && consumed && depth >= 2) {
        if (P.frames[below].node == kBottom) {
          if (left_frame) *left_frame |= (follow_rule >= 0 && A.follow[follow_rule].test(c)) ? 3 : 1;
        } else {
          add(below, true);
        }
      }
      if (seen > kMaxConfigs) return XGM_ERR_TOO_LARGE;
    }
    if (next.empty()) return XGM_ERR_TOKEN_REJECTED;
    cur.swap(next);
  }
  // A top node that can only return is returned from right away, so that the
  // stack top is always a node with something of its own to say about the
  // next token (and equal states get equal representations).
  ++P.step;
  next.clear();
  for (int32_t id : cur) {
    while (P.frames[id].depth >= 2 && P.frames[P.frames[id].below].node != kBottom && A.node_dead_end[P.frames[id].node])
      id = P.frames[id].below;
    if (P.first_time(id, kReached)) next.push_back(id);
  }
  if (next.size() > max_out) return XGM_ERR_TOO_MANY_STACKS;
  out->resize(next.size());
  for (size_t k = 0; k < next.size(); ++k) P.read(next[k], &(*out)[k]);
  if (out->size() > 1) std::sort(out->begin(), out->end());
  return XGM_OK;
}

bool Engine::can_terminate(const std::vector<Stack>& stacks) const {
  for (auto& s : stacks) {
    bool all = true;
    for (int32_t n : s)
      if (!A_->node_final[n]) { all = false; break; }
    if (all) return true;
  }
  return false;
}

int Engine::classify(int32_t node, const uint8_t* bytes, int n) const {
  if (n == 0) return 0;
  std::vector<Stack> in{Stack{kBottom, node}}, out;
  int left = 0;
  int rc = advance(in, bytes, n, &out, &left, (size_t)-1, A_->node_rule[node]);
  if (rc == XGM_OK) return 2;
  if (rc == XGM_ERR_TOKEN_REJECTED) return (left & 2) ? 1 : (left & 1) ? 4 : 0;
  return -1;
}

}  // namespace xgm
