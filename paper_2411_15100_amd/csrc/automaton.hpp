// Host-side grammar compilation: EBNF text -> flattened byte-level pushdown
// automaton (arxiv 2411.15100, section 2.2 and Appendix A: one finite
// automaton per rule, character edges and rule-reference edges).
#pragma once
#include <cstdint>
#include <stdexcept>
#include <string>
#include <vector>

namespace xgm {

struct Failure : std::runtime_error {
  int status;
  Failure(int s, const std::string& m) : std::runtime_error(m), status(s) {}
};

struct ByteEdge { uint8_t lo, hi; int32_t to; };
struct RefEdge { int32_t rule; int32_t to; };

// Device header of one node (8 bytes).
//  * plain node (at most one byte edge, no references): [lo, hi] -> target,
//    lo > hi if it has no edge at all;
//  * branching node (kFlagBranching): lo | hi << 8 is its shape id and
//    `target` the start of its outcomes in `targets`; for byte c the outcome
//    is targets[target + shapes[shape * n_cls + cls[c]]] unless that shape
//    entry is kDeadShape.
struct NodeHdr {
  uint8_t lo, hi;
  uint16_t target;
  uint32_t flags;  // kFlagFinal | kFlagBranching | kFlagDeadEnd | frames of the chain << kChainShift | rule index << 16
};
static_assert(sizeof(NodeHdr) == 8, "NodeHdr must be 8 bytes");

constexpr uint32_t kFlagFinal = 1;      // the rule may end at this node
constexpr uint32_t kFlagBranching = 2;
constexpr uint32_t kFlagDeadEnd = 4;    // accepting and without outgoing edges: all it can do is return
constexpr uint32_t kChainShift = 8;     // 8 bits: 1 + the forced frames below a frame of the node's rule
constexpr int kMaxForced = 48;          // forced frames followed per rule (three levels of them stay below 256 frames)
constexpr int kShortWayDown = 2;        // (the levels of a mask cache below the first)
constexpr uint8_t kDeadShape = 0xFF;    // shape entry: nothing to do for this byte class
constexpr uint16_t kAltFlag = 0x8000;   // outcome: index into the alternatives pool (else: move to that node)
constexpr uint32_t kMoveTag = 0xFFFF;   // alternative (tag << 16 | node): consume the byte, go to node
constexpr uint32_t kTailTag = 0xFFFE;   // alternative: enter the callee at `node` without pushing a frame
                                        // (any other tag is the return node to push)
// A run of calls without a choice - entering an expression goes through a dozen precedence levels before the first
// byte of the operand is consumed - is one entry of the alternatives pool instead of a list, of two words: kRunFlag |
// (kRunConsumes if the byte is consumed at its end) | frames to push << kRunFramesShift | where in the pool they are
// (16 bits each, in the order in which they are pushed), and the node it leads to.
constexpr uint32_t kRunFlag = 0x80000000u, kRunConsumes = 0x40000000u, kRunFramesShift = 16, kRunFramesMask = 0x3Fu, kRunAtMask = 0x7FFFu;
constexpr int kShortestRun = 3;         // calls
constexpr int kMaxRun = 32;             // frames pushed by one run

// a set of byte values
struct ByteSet {
  uint32_t w[8] = {};
  bool test(int c) const { return (w[c >> 5] >> (c & 31)) & 1u; }
  void set_range(int lo, int hi) {
    for (int k = lo >> 5; k <= hi >> 5; ++k) {
      const int a = lo > k * 32 ? lo - k * 32 : 0, b = hi < k * 32 + 31 ? hi - k * 32 : 31;
      w[k] |= (0xFFFFFFFFu >> (31 - (b - a))) << a;
    }
  }
  // whether the set has grown
  bool add(const ByteSet& o) {
    uint32_t grown = 0;
    for (int k = 0; k < 8; ++k) { grown |= o.w[k] & ~w[k]; w[k] |= o.w[k]; }
    return grown != 0;
  }
};

// rows of different lengths, one after the other
template <class T>
struct Rows {
  struct Row {
    const T *first, *last;
    const T* begin() const { return first; }
    const T* end() const { return last; }
    size_t size() const { return (size_t)(last - first); }
    bool empty() const { return first == last; }
    const T& operator[](size_t k) const { return first[k]; }
  };
  std::vector<T> items;
  std::vector<uint32_t> off{0};  // row k is items[off[k] .. off[k + 1])
  void end_row() { off.push_back((uint32_t)items.size()); }
  Row operator[](size_t k) const { return {items.data() + off[k], items.data() + off[k + 1]}; }
};

struct Automaton {
  // structured form (host engine)
  int32_t n_nodes = 0;
  std::vector<int32_t> node_rule;
  std::vector<uint8_t> node_final;
  std::vector<uint8_t> node_dead_end;         // accepting and without outgoing edges: all it can do is return
  // The node can be on top of a stack that has other frames: a byte or an instance of a rule leads to it, and it has
  // something of its own to do (a top that can only return is returned from at once).
  std::vector<uint8_t> node_on_top;
  Rows<ByteEdge> bedges;                      // per node: sorted, disjoint
  Rows<RefEdge> redges;                       // per node
  std::vector<int32_t> rule_start;            // per rule: global node id
  std::vector<std::string> rule_names;
  std::vector<ByteSet> first;                 // per rule: bytes an instance can start with
  std::vector<ByteSet> node_first;            // per node: bytes that can be consumed at the node inside its frame
  std::vector<ByteSet> follow;                // per rule: bytes that can come right after an instance, in any context
  // per rule: the nodes that can sit right below a frame of that rule (return nodes of the references to it;
  // a reference in tail position hands on the contexts of the referring rule), sorted
  std::vector<std::vector<int32_t>> contexts;
  // Per rule: the frames that are certain to lie below a frame of that rule, nearest first.  A rule with a single
  // context that can never be at the bottom of a stack has that context below it; if the context's rule is of the
  // same kind, so is its own context, and so on (the precedence levels of an expression grammar).
  std::vector<std::vector<int32_t>> forced;
  int32_t end_rule(int32_t rule) const { return forced[rule].empty() ? rule : node_rule[forced[rule].back()]; }
  int32_t root_rule = 0;
  std::vector<int32_t> path_parent, path_symbol;  // last step of a witness path from the rule start (-1: the start)
  std::vector<int32_t> node_path(int32_t node) const;

  // flattened form (device tables)
  std::vector<NodeHdr> hdr;        // [n_nodes]
  std::vector<uint8_t> cls;        // [256] byte -> class
  int32_t n_cls = 0;
  std::vector<uint8_t> shapes;     // [n_shapes * n_cls]
  int32_t n_shapes = 0;
  std::vector<uint16_t> targets;   // outcomes of the branching nodes, node after node
  std::vector<uint32_t> alts;      // pool: count, then count entries (tag << 16 | node); or a run (kRunFlag)
  int32_t max_alts = 0;
};

// Throws Failure.
Automaton compile_grammar(const std::string& text, const std::string& root);

}  // namespace xgm
