// Grammar text -> per-rule NFA -> per-rule minimal DFA over (bytes + rule
// references) -> flattened tables.  See automaton.hpp and include/xgm.h.
#include "automaton.hpp"

#include <sched.h>

#include <algorithm>
#include <atomic>
#include <exception>
#include <functional>
#include <iterator>
#include <string_view>
#include <system_error>
#include <thread>
#include <unordered_map>

#include "../../include/xgm.h"

namespace xgm {
namespace {

// ------------------------------------------------------------------ lexer
enum TokKind { T_IDENT, T_DEFINE, T_PIPE, T_LP, T_RP, T_STAR, T_PLUS, T_QUEST, T_LIT, T_CLASS, T_END };
struct CpRange { uint32_t lo, hi; };
struct Token {
  TokKind kind;
  size_t pos;
  uint32_t a, b;  // identifier or literal: its bytes are [a, b) of Lexed::text; class: [a, b) of Lexed::ranges
};
struct Lexed {
  std::vector<Token> toks;
  std::string text;
  std::vector<CpRange> ranges;  // classes, normalised and already complemented
  std::string_view text_of(const Token& t) const { return std::string_view(text).substr(t.a, t.b - t.a); }
};

[[noreturn]] void parse_fail(size_t pos, const std::string& why) {
  throw Failure(XGM_ERR_PARSE, "grammar: " + why + " (at byte " + std::to_string(pos) + ")");
}

int hex_digit(char c, size_t pos) {
  if (c >= '0' && c <= '9') return c - '0';
  if (c >= 'a' && c <= 'f') return 10 + c - 'a';
  if (c >= 'A' && c <= 'F') return 10 + c - 'A';
  parse_fail(pos, "bad hex digit");
}

void append_utf8(uint32_t cp, std::string& out) {
  if (cp <= 0x7F) out += (char)cp;
  else if (cp <= 0x7FF) { out += (char)(0xC0 | (cp >> 6)); out += (char)(0x80 | (cp & 0x3F)); }
  else if (cp <= 0xFFFF) { out += (char)(0xE0 | (cp >> 12)); out += (char)(0x80 | ((cp >> 6) & 0x3F)); out += (char)(0x80 | (cp & 0x3F)); }
  else { out += (char)(0xF0 | (cp >> 18)); out += (char)(0x80 | ((cp >> 12) & 0x3F)); out += (char)(0x80 | ((cp >> 6) & 0x3F)); out += (char)(0x80 | (cp & 0x3F)); }
}

std::vector<CpRange> normalise_class(std::vector<CpRange> r, bool negate) {
  std::sort(r.begin(), r.end(), [](const CpRange& a, const CpRange& b) { return a.lo < b.lo; });
  std::vector<CpRange> merged;
  for (auto& x : r) {
    if (!merged.empty() && x.lo <= merged.back().hi + 1) merged.back().hi = std::max(merged.back().hi, x.hi);
    else merged.push_back(x);
  }
  if (negate) {
    std::vector<CpRange> inv;
    uint32_t next = 0;
    for (auto& x : merged) {
      if (x.lo > next) inv.push_back({next, x.lo - 1});
      next = x.hi + 1;
    }
    if (next <= 0x10FFFF) inv.push_back({next, 0x10FFFF});
    merged.swap(inv);
  }
  // drop the surrogate block and anything above the last scalar value
  std::vector<CpRange> out;
  for (auto x : merged) {
    if (x.lo > 0x10FFFF) continue;
    x.hi = std::min<uint32_t>(x.hi, 0x10FFFF);
    if (x.hi < 0xD800 || x.lo > 0xDFFF) { out.push_back(x); continue; }
    if (x.lo < 0xD800) out.push_back({x.lo, 0xD7FF});
    if (x.hi > 0xDFFF) out.push_back({0xE000, x.hi});
  }
  return out;
}

Lexed lex(const std::string& s) {
  Lexed out;
  out.text.reserve(s.size());
  out.toks.reserve(s.size() / 4);
  auto token = [&](TokKind kind, size_t pos) { out.toks.push_back({kind, pos, 0u, 0u}); };
  auto text_token = [&](TokKind kind, size_t pos, size_t a) { out.toks.push_back({kind, pos, (uint32_t)a, (uint32_t)out.text.size()}); };
  size_t i = 0, n = s.size();
  auto ident_start = [](char c) { return (c >= 'a' && c <= 'z') || (c >= 'A' && c <= 'Z') || c == '_'; };
  auto ident_part = [&](char c) { return ident_start(c) || (c >= '0' && c <= '9'); };
  // an escape after a backslash; returns a code point (or raw byte for \x in literals)
  auto escape = [&](bool in_class, bool* raw_byte) -> uint32_t {
    if (i >= n) parse_fail(i, "unterminated escape");
    char k = s[i++];
    *raw_byte = false;
    switch (k) {
      case 'n': return '\n';
      case 't': return '\t';
      case 'r': return '\r';
      case 'b': return '\b';
      case 'f': return '\f';
      case '"': case '\\': case '\'': case '/': return (unsigned char)k;
      case ']': case '[': case '-': case '^':
        if (in_class) return (unsigned char)k;
        break;
      case 'x': {
        if (i + 2 > n) parse_fail(i, "truncated \\x escape");
        uint32_t v = hex_digit(s[i], i) * 16 + hex_digit(s[i + 1], i + 1);
        i += 2;
        *raw_byte = !in_class;
        return v;
      }
      case 'u': {
        if (i + 4 > n) parse_fail(i, "truncated \\u escape");
        uint32_t v = 0;
        for (int k2 = 0; k2 < 4; ++k2) v = v * 16 + hex_digit(s[i + k2], i + k2);
        i += 4;
        return v;
      }
      default: break;
    }
    parse_fail(i - 1, std::string("unknown escape \\") + k);
  };
  while (i < n) {
    char c = s[i];
    if (c == ' ' || c == '\t' || c == '\n' || c == '\r') { ++i; continue; }
    if (c == '#') { while (i < n && s[i] != '\n') ++i; continue; }
    size_t start = i;
    if (ident_start(c)) {
      while (i < n && ident_part(s[i])) ++i;
      const size_t a = out.text.size();
      out.text.append(s, start, i - start);
      text_token(T_IDENT, start, a);
      continue;
    }
    if (c == ':' && s.compare(i, 3, "::=") == 0) { i += 3; token(T_DEFINE, start); continue; }
    if (c == '|') { ++i; token(T_PIPE, start); continue; }
    if (c == '(') { ++i; token(T_LP, start); continue; }
    if (c == ')') { ++i; token(T_RP, start); continue; }
    if (c == '*') { ++i; token(T_STAR, start); continue; }
    if (c == '+') { ++i; token(T_PLUS, start); continue; }
    if (c == '?') { ++i; token(T_QUEST, start); continue; }
    if (c == '"') {
      ++i;
      std::string& bytes = out.text;
      const size_t a = bytes.size();
      for (;;) {
        if (i >= n) parse_fail(start, "unterminated literal");
        char d = s[i++];
        if (d == '"') break;
        if (d != '\\') { bytes += d; continue; }
        bool raw;
        uint32_t v = escape(false, &raw);
        if (raw) bytes += (char)v;
        else {
          if (v >= 0xD800 && v <= 0xDFFF) parse_fail(i, "surrogate code point in literal");
          append_utf8(v, bytes);
        }
      }
      text_token(T_LIT, start, a);
      continue;
    }
    if (c == '[') {
      ++i;
      bool negate = false;
      if (i < n && s[i] == '^') { negate = true; ++i; }
      std::vector<CpRange> ranges;
      auto one = [&]() -> uint32_t {
        if (i >= n) parse_fail(start, "unterminated class");
        unsigned char d = (unsigned char)s[i++];
        if (d == '\\') { bool raw; return escape(true, &raw); }
        if (d < 0x80) return d;
        int extra = d >= 0xF0 ? 3 : d >= 0xE0 ? 2 : d >= 0xC0 ? 1 : -1;
        if (extra < 0) parse_fail(i - 1, "invalid UTF-8 in class");
        uint32_t cp = d & (0x3F >> extra);
        for (int k = 0; k < extra; ++k) {
          if (i >= n || ((unsigned char)s[i] & 0xC0) != 0x80) parse_fail(i, "invalid UTF-8 in class");
          cp = (cp << 6) | ((unsigned char)s[i++] & 0x3F);
        }
        return cp;
      };
      for (;;) {
        if (i >= n) parse_fail(start, "unterminated class");
        if (s[i] == ']') { ++i; break; }
        uint32_t lo = one(), hi = lo;
        if (i + 1 < n && s[i] == '-' && s[i + 1] != ']') { ++i; hi = one(); }
        if (hi < lo) parse_fail(i, "reversed range in class");
        ranges.push_back({lo, hi});
      }
      const uint32_t a = (uint32_t)out.ranges.size();
      for (auto& r : normalise_class(ranges, negate)) out.ranges.push_back(r);
      out.toks.push_back({T_CLASS, start, a, (uint32_t)out.ranges.size()});
      continue;
    }
    parse_fail(i, std::string("unexpected character '") + c + "'");
  }
  token(T_END, n);
  return out;
}

// -------------------------------------------------------------------- NFA
struct NEdge { int kind; int lo, hi; int rule; int to; };  // kind 0 eps, 1 bytes [lo,hi], 2 reference
struct Nfa {
  int add() { return n_++; }
  void eps(int a, int b) { put(a, {0, 0, 0, 0, b}); }
  void bytes(int a, int lo, int hi, int b) { put(a, {1, lo, hi, 0, b}); }
  void ref(int a, int rule, int b) { put(a, {2, 0, 0, rule, b}); }
  int size() const { return n_; }
  void reserve(size_t edges) { edges_.reserve(edges); from_.reserve(edges); }
  // after the last edge: the edges of every state side by side
  void finish() {
    off_.assign(n_ + 1, 0u);
    for (int q : from_) ++off_[q + 1];
    for (int q = 0; q < n_; ++q) off_[q + 1] += off_[q];
    std::vector<uint32_t> at(off_.begin(), off_.end() - 1);
    std::vector<NEdge> sorted(edges_.size());
    for (size_t k = 0; k < edges_.size(); ++k) sorted[at[from_[k]]++] = edges_[k];
    edges_.swap(sorted);
  }
  struct Out {
    const NEdge *first, *last;
    const NEdge* begin() const { return first; }
    const NEdge* end() const { return last; }
  };
  Out out(int q) const { return {edges_.data() + off_[q], edges_.data() + off_[q + 1]}; }

 private:
  void put(int a, const NEdge& e) { from_.push_back(a); edges_.push_back(e); }
  int n_ = 0;
  std::vector<NEdge> edges_;
  std::vector<int> from_;
  std::vector<uint32_t> off_;
};

struct Frag { int in, out; };

class Parser {
 public:
  Parser(const Lexed& lexed, Nfa& nfa) : lexed_(lexed), t_(lexed.toks), nfa_(nfa) {
    for (size_t k = 0; k + 1 < t_.size(); ++k)
      if (t_[k].kind == T_IDENT && t_[k + 1].kind == T_DEFINE) {
        const std::string_view name = lexed_.text_of(t_[k]);
        if (!rule_index_.emplace(name, (int)names_.size()).second) throw Failure(XGM_ERR_PARSE, "grammar: rule '" + std::string(name) + "' defined twice");
        names_.emplace_back(name);
      }
    if (names_.empty()) throw Failure(XGM_ERR_PARSE, "grammar: no rules");
  }
  void run() {
    start_.assign(names_.size(), -1);
    accept_.assign(names_.size(), -1);
    while (t_[p_].kind != T_END) {
      if (!(t_[p_].kind == T_IDENT && t_[p_ + 1].kind == T_DEFINE)) parse_fail(t_[p_].pos, "expected 'name ::='");
      int r = rule_index_[lexed_.text_of(t_[p_])];
      p_ += 2;
      const int before = nfa_.size();
      Frag f = alternatives();
      if (t_[p_].kind == T_RP) parse_fail(t_[p_].pos, "unbalanced ')'");
      start_[r] = f.in;
      accept_[r] = f.out;
      largest_ = std::max(largest_, nfa_.size() - before);
    }
  }
  std::vector<std::string> names_;
  std::unordered_map<std::string_view, int> rule_index_;
  std::vector<int> start_, accept_;
  int largest_ = 1;  // states of the largest rule

 private:
  const Lexed& lexed_;
  const std::vector<Token>& t_;
  Nfa& nfa_;
  size_t p_ = 0;
  std::pair<std::string_view, int> last_of_length_[16] = {};  // (a name is never empty)

  bool at_rule_head() const { return t_[p_].kind == T_IDENT && t_[p_ + 1].kind == T_DEFINE; }
  Frag alternatives() {
    Frag first = sequence();
    if (t_[p_].kind != T_PIPE) return first;
    int in = nfa_.add(), out = nfa_.add();
    nfa_.eps(in, first.in);
    nfa_.eps(first.out, out);
    while (t_[p_].kind == T_PIPE) {
      ++p_;
      Frag f = sequence();
      nfa_.eps(in, f.in);
      nfa_.eps(f.out, out);
    }
    return {in, out};
  }
  Frag sequence() {
    int in = nfa_.add();
    int cur = in;
    for (;;) {
      TokKind k = t_[p_].kind;
      if (k == T_END || k == T_PIPE || k == T_RP || at_rule_head()) break;
      Frag f = item();
      nfa_.eps(cur, f.in);
      cur = f.out;
    }
    return {in, cur};
  }
  Frag item() {
    Frag f = atom();
    for (;;) {
      TokKind k = t_[p_].kind;
      if (k == T_STAR) {
        int hub = nfa_.add();
        nfa_.eps(hub, f.in);
        nfa_.eps(f.out, hub);
        f = {hub, hub};
      } else if (k == T_PLUS) {
        int out = nfa_.add();
        nfa_.eps(f.out, out);
        nfa_.eps(out, f.in);
        f = {f.in, out};
      } else if (k == T_QUEST) {
        int in = nfa_.add(), out = nfa_.add();
        nfa_.eps(in, f.in);
        nfa_.eps(f.out, out);
        nfa_.eps(in, out);
        f = {in, out};
      } else break;
      ++p_;
    }
    return f;
  }
  Frag atom() {
    const Token& tk = t_[p_];
    switch (tk.kind) {
      case T_LIT: {
        ++p_;
        int in = nfa_.add(), cur = in;
        for (unsigned char c : lexed_.text_of(tk)) { int nx = nfa_.add(); nfa_.bytes(cur, c, c, nx); cur = nx; }
        return {in, cur};
      }
      case T_CLASS: {
        ++p_;
        int in = nfa_.add(), out = nfa_.add();
        for (uint32_t k = tk.a; k < tk.b; ++k) add_codepoints(lexed_.ranges[k].lo, lexed_.ranges[k].hi, in, out);
        return {in, out};
      }
      case T_IDENT: {
        ++p_;
        // (a few names, white space above all, are most of the references: the last one of each length is remembered)
        const std::string_view name = lexed_.text_of(tk);
        std::pair<std::string_view, int>& last = last_of_length_[name.size() % 16];
        if (last.first != name) {
          auto it = rule_index_.find(name);
          if (it == rule_index_.end()) throw Failure(XGM_ERR_UNDEFINED_RULE, "grammar: rule '" + std::string(name) + "' is not defined");
          last = *it;
        }
        int in = nfa_.add(), out = nfa_.add();
        nfa_.ref(in, last.second, out);
        return {in, out};
      }
      case T_LP: {
        ++p_;
        Frag f = alternatives();
        if (t_[p_].kind != T_RP) parse_fail(t_[p_].pos, "expected ')'");
        ++p_;
        return f;
      }
      default: parse_fail(tk.pos, "expected a literal, class, rule name or '('");
    }
  }
  // UTF-8 byte sequences for the scalar values lo..hi: cut the range where
  // the encoded length changes, then where a continuation byte would not
  // span its full 0x80..0xBF range, and emit one chain of byte ranges per piece.
  void add_codepoints(uint32_t lo, uint32_t hi, int in, int out) {
    static const uint32_t last_of_len[4] = {0x7F, 0x7FF, 0xFFFF, 0x10FFFF};
    for (int len = 1; len <= 4 && lo <= hi; ++len) {
      if (lo > last_of_len[len - 1]) continue;
      uint32_t top = std::min(hi, last_of_len[len - 1]);
      same_length(lo, top, len, in, out);
      lo = top + 1;
      if (top == 0x10FFFF) break;
    }
  }
  void same_length(uint32_t lo, uint32_t hi, int len, int in, int out) {
    for (int k = 1; k < len; ++k) {
      uint32_t low_bits = (1u << (6 * k)) - 1;
      if ((lo & ~low_bits) != (hi & ~low_bits)) {
        if ((lo & low_bits) != 0) {
          same_length(lo, lo | low_bits, len, in, out);
          same_length((lo | low_bits) + 1, hi, len, in, out);
          return;
        }
        if ((hi & low_bits) != low_bits) {
          same_length(lo, (hi & ~low_bits) - 1, len, in, out);
          same_length(hi & ~low_bits, hi, len, in, out);
          return;
        }
      }
    }
    std::string a, b;
    append_utf8(lo, a);
    append_utf8(hi, b);
    int cur = in;
    for (int k = 0; k < len; ++k) {
      int nx = (k + 1 == len) ? out : nfa_.add();
      nfa_.bytes(cur, (unsigned char)a[k], (unsigned char)b[k], nx);
      cur = nx;
    }
  }
};

// ------------------------------------------------------- per-rule DFA
// Everything from here on is written for grammars of tens of thousands of NFA
// states (a schema with a few hundred properties): every step is linear in the
// edges it looks at, or nearly so, and works on flat arrays that are reused from
// rule to rule.  A new schema is on the path of a request's first token: the
// 36 KB grammar of the largest synthetic schema (11867 nodes) took 84 ms to
// compile with a set or map per state and rounds over all states until nothing
// changed, 2.1 ms this way (another machine), and 1.7 with nothing hashed for states inside a
// literal and for rules whose states cannot be equivalent.

// Finds equal integer sequences: intern() gives every distinct one a number, in the order of first appearance.
class SequenceTable {
 public:
  void clear(size_t expected) {
    size_t cap = 64;
    while (cap < expected * 2) cap *= 2;
    slots_.assign(cap, 0);
    hashed_ = 0;
    pool_.clear();
    off_.assign(1, 0);
  }
  size_t size() const { return off_.size() - 1; }
  const int* begin(int id) const { return pool_.data() + off_[id]; }
  const int* end(int id) const { return pool_.data() + off_[id + 1]; }
  int intern(const int* p, size_t n, bool* is_new = nullptr) {
    if (hashed_ * 2 >= slots_.size()) grow();  // (so that at least half of the slots are free)
    size_t at = hash(p, n) & (slots_.size() - 1);
    for (; slots_[at]; at = (at + 1) & (slots_.size() - 1)) {
      const int id = slots_[at] - 1;
      if (off_[id + 1] - off_[id] == n && std::equal(p, p + n, begin(id))) {
        if (is_new) *is_new = false;
        return id;
      }
    }
    const int id = append(p, n);
    slots_[at] = id + 1;
    ++hashed_;
    if (is_new) *is_new = true;
    return id;
  }
  // a sequence that intern() will never be asked for: it has a number, but no slot
  int append(const int* p, size_t n) {
    const int id = (int)size();
    pool_.insert(pool_.end(), p, p + n);
    off_.push_back((uint32_t)pool_.size());
    return id;
  }

 private:
  static uint64_t hash(const int* p, size_t n) {
    uint64_t h = 0x9E3779B97F4A7C15ull ^ n;
    for (size_t k = 0; k < n; ++k) {
      h = (h ^ (uint32_t)p[k]) * 0xBF58476D1CE4E5B9ull;
      h ^= h >> 29;
    }
    return h;
  }
  void grow() {
    old_.swap(slots_);
    slots_.assign(old_.size() * 2, 0);
    for (int slot : old_) {
      if (!slot) continue;
      const int id = slot - 1;
      size_t at = hash(begin(id), (size_t)(end(id) - begin(id))) & (slots_.size() - 1);
      while (slots_[at]) at = (at + 1) & (slots_.size() - 1);
      slots_[at] = slot;
    }
  }
  std::vector<int> slots_, old_;  // id + 1, or 0
  size_t hashed_ = 0;             // slots in use
  std::vector<int> pool_;
  std::vector<uint32_t> off_{0};
};

// lists of ints by bucket, in the order given
struct Buckets {
  std::vector<uint32_t> off;
  std::vector<int> item;
  template <class Each>  // each(f) calls f(bucket, item) for everything that is to be put in, the same way twice
  void fill(size_t n, const Each& each) {
    off.assign(n + 1, 0u);
    each([&](int b, int) { ++off[b + 1]; });
    for (size_t k = 0; k < n; ++k) off[k + 1] += off[k];
    item.resize(off[n]);
    std::vector<uint32_t>& at = next_;
    at.assign(off.begin(), off.end() - 1);
    each([&](int b, int x) { item[at[b]++] = x; });
  }
  const int* begin(int b) const { return item.data() + off[b]; }
  const int* end(int b) const { return item.data() + off[b + 1]; }

 private:
  std::vector<uint32_t> next_;
};

struct DState {
  bool final_ = false;
  uint32_t b0 = 0, b1 = 0, r0 = 0, r1 = 0;  // its edges: [b0, b1) of Dfa::b (sorted, disjoint), [r0, r1) of Dfa::r (sorted by rule)
};
struct Dfa {  // state 0 is the start
  std::vector<DState> s;
  std::vector<ByteEdge> b;
  std::vector<RefEdge> r;
  void clear() { s.clear(); b.clear(); r.clear(); }
  // neighbouring ranges with the same target become one (the edges of the state being built, from b0 on)
  void merge_byte_edges(size_t b0) {
    size_t out = b0;
    for (size_t k = b0; k < b.size(); ++k) {
      if (out > b0 && b[out - 1].to == b[k].to && (int)b[out - 1].hi + 1 == (int)b[k].lo) b[out - 1].hi = b[k].hi;
      else b[out++] = b[k];
    }
    b.resize(out);
  }
};

// Which rules derive something at all, and which derive the empty text: the states of a rule are entered
// from its start, an edge that refers to a rule once that rule is known to derive what is asked for.
template <class Usable>
std::vector<char> derivable(const Nfa& nfa, const std::vector<int>& start, const std::vector<int>& accept, const Usable& usable_edge) {
  const int R = (int)start.size(), S = nfa.size();
  std::vector<char> done(R, 0), reached(S, 0);
  std::vector<int> accepts(S, -1), work, waiting_head(R, -1), waiting_next;
  std::vector<int> waiting_to;
  for (int r = 0; r < R; ++r) accepts[accept[r]] = r;
  auto enter = [&](int q) { if (!reached[q]) { reached[q] = 1; work.push_back(q); } };
  for (int r = 0; r < R; ++r) enter(start[r]);
  while (!work.empty()) {
    const int q = work.back();
    work.pop_back();
    const int r = accepts[q];
    if (r >= 0 && !done[r]) {
      done[r] = 1;
      for (int k = waiting_head[r]; k >= 0; k = waiting_next[k]) enter(waiting_to[k]);
    }
    for (auto& e : nfa.out(q)) {
      if (!usable_edge(e)) continue;
      if (e.kind != 2 || done[e.rule]) enter(e.to);
      else {
        waiting_next.push_back(waiting_head[e.rule]);
        waiting_head[e.rule] = (int)waiting_to.size();
        waiting_to.push_back(e.to);
      }
    }
  }
  return done;
}

// Subset construction of one rule after the other.
class Determinizer {
 public:
  Determinizer(const Nfa& nfa, const std::vector<char>& productive, const std::vector<char>& nullable)
      : nfa_(nfa), productive_(productive), nullable_(nullable), mark_(nfa.size(), 0u), single_(nfa.size(), -1), alone_(nfa.size(), -1) {}
  void run(int start, int accept, Dfa& d) {
    d.clear();
    sets_.clear(64);
    touched_.clear();
    accept_ = accept;
    closed(&start, 1);
    for (int cur = 0; cur < (int)sets_.size(); ++cur) {
      DState s;
      s.b0 = (uint32_t)d.b.size();
      s.r0 = (uint32_t)d.r.size();
      bytes_.clear();
      refs_.clear();
      for (const int* q = sets_.begin(cur); q != sets_.end(cur); ++q) {
        s.final_ = s.final_ || *q == accept;
        for (auto& e : nfa_.out(*q)) {
          if (e.kind == 1) bytes_.push_back({e.lo, e.hi, e.to});
          else if (e.kind == 2 && productive_[e.rule]) refs_.push_back({e.rule, e.to});
        }
      }
      if (bytes_.size() == 1) {
        d.b.push_back({(uint8_t)bytes_[0].lo, (uint8_t)bytes_[0].hi, closed(&bytes_[0].to, 1)});
      } else if (!bytes_.empty()) {
        cuts_.clear();  // interval starts
        for (auto& e : bytes_) { cuts_.push_back(e.lo); cuts_.push_back(e.hi + 1); }
        std::sort(cuts_.begin(), cuts_.end());
        cuts_.erase(std::unique(cuts_.begin(), cuts_.end()), cuts_.end());
        for (size_t k = 0; k + 1 < cuts_.size(); ++k) {
          const int lo = cuts_[k], hi = cuts_[k + 1] - 1;
          targets_.clear();
          for (auto& e : bytes_)
            if (e.lo <= lo && hi <= e.hi) targets_.push_back(e.to);
          if (!targets_.empty()) d.b.push_back({(uint8_t)lo, (uint8_t)hi, closed(targets_.data(), targets_.size())});
        }
        d.merge_byte_edges(s.b0);
      }
      std::stable_sort(refs_.begin(), refs_.end(), [](const RefEdge& x, const RefEdge& y) { return x.rule < y.rule; });
      for (size_t k = 0; k < refs_.size();) {
        targets_.clear();
        const int rule = refs_[k].rule;
        for (; k < refs_.size() && refs_[k].rule == rule; ++k) targets_.push_back(refs_[k].to);
        d.r.push_back({rule, closed(targets_.data(), targets_.size())});
      }
      s.b1 = (uint32_t)d.b.size();
      s.r1 = (uint32_t)d.r.size();
      d.s.push_back(s);
    }
    for (int q : touched_) single_[q] = alone_[q] = -1;
  }

 private:
  // The DFA state of what can be reached from the seed without consuming anything (epsilon edges, and references
  // to nullable rules skipped); only states with something of their own to say are kept.
  int closed(const int* seed, size_t n) {
    if (n == 1 && single_[*seed] >= 0) return single_[*seed];
    set_.clear();
    if (n == 1 && goes_nowhere(*seed)) set_.push_back(*seed);  // (inside a literal)
    else {
      ++stamp_;
      work_.clear();
      for (size_t k = 0; k < n; ++k)
        if (mark_[seed[k]] != stamp_) { mark_[seed[k]] = stamp_; work_.push_back(seed[k]); }
      while (!work_.empty()) {
        const int q = work_.back();
        work_.pop_back();
        bool says = q == accept_;
        for (auto& e : nfa_.out(q)) {
          if (skips(e) && mark_[e.to] != stamp_) { mark_[e.to] = stamp_; work_.push_back(e.to); }
          says = says || e.kind == 1 || (e.kind == 2 && productive_[e.rule]);
        }
        if (says) set_.push_back(q);
      }
      std::sort(set_.begin(), set_.end());
    }
    int id;
    if (set_.size() == 1) {  // most are: found by their state, not by their hash
      int& a = alone_[set_[0]];
      if (a < 0) { a = sets_.append(set_.data(), 1); touched_.push_back(set_[0]); }
      id = a;
    } else {
      id = sets_.intern(set_.data(), set_.size());
    }
    if (n == 1) { single_[*seed] = id; touched_.push_back(*seed); }
    return id;
  }
  bool skips(const NEdge& e) const { return e.kind == 0 || (e.kind == 2 && productive_[e.rule] && nullable_[e.rule]); }
  bool goes_nowhere(int q) const {
    const auto out = nfa_.out(q);
    return out.last - out.first == 1 && out.first->kind == 1;
  }
  struct Bytes { int lo, hi, to; };
  const Nfa& nfa_;
  const std::vector<char>&productive_, &nullable_;
  std::vector<uint32_t> mark_;
  std::vector<int> single_, alone_, touched_;  // of a single state of the current rule: its closure; the set of it alone
  uint32_t stamp_ = 0;
  int accept_ = -1;
  SequenceTable sets_;
  std::vector<int> set_, work_, cuts_, targets_;
  std::vector<Bytes> bytes_;
  std::vector<RefEdge> refs_;
};

// Trimming (states from which no accepting state can be reached) and minimisation.
class Minimizer {
 public:
  Dfa run(const Dfa& d) {
    n_ = (int)d.s.size();
    d_ = &d;
    if (all_heights_differ()) return d;
    // predecessors
    pred_.fill(n_, [&](auto put) {
      for (int q = 0; q < n_; ++q) {
        for (uint32_t k = d.s[q].b0; k < d.s[q].b1; ++k) put(d.b[k].to, q);
        for (uint32_t k = d.s[q].r0; k < d.s[q].r1; ++k) put(d.r[k].to, q);
      }
    });
    alive_.assign(n_, 0);
    std::vector<int>& work = dirty_;
    work.clear();
    for (int q = 0; q < n_; ++q)
      if (d.s[q].final_) { alive_[q] = 1; work.push_back(q); }
    for (size_t k = 0; k < work.size(); ++k)
      for (const int* p = pred_.begin(work[k]); p != pred_.end(work[k]); ++p)
        if (!alive_[*p]) { alive_[*p] = 1; work.push_back(*p); }
    if (!alive_[0]) throw Failure(XGM_ERR_INTERNAL, "grammar: productive rule lost its start state");
    if (!hash_upwards()) refine();
    // one state per block, in the order in which the blocks first appear
    std::vector<int> renum(sizes_.size(), -1), rep;
    for (int q = 0; q < n_; ++q)
      if (alive_[q] && renum[block_[q]] < 0) { renum[block_[q]] = (int)rep.size(); rep.push_back(q); }
    Dfa m;
    m.s.reserve(rep.size());
    for (int q : rep) {
      DState s;
      s.final_ = d.s[q].final_;
      s.b0 = (uint32_t)m.b.size();
      s.r0 = (uint32_t)m.r.size();
      for (uint32_t k = d.s[q].b0; k < d.s[q].b1; ++k)
        if (alive_[d.b[k].to]) m.b.push_back({d.b[k].lo, d.b[k].hi, renum[block_[d.b[k].to]]});
      m.merge_byte_edges(s.b0);
      for (uint32_t k = d.s[q].r0; k < d.s[q].r1; ++k)
        if (alive_[d.r[k].to]) m.r.push_back({d.r[k].rule, renum[block_[d.r[k].to]]});
      s.b1 = (uint32_t)m.b.size();
      s.r1 = (uint32_t)m.r.size();
      m.s.push_back(s);
    }
    return m;
  }

 private:
  // If there are no loops and no two states have the same longest way to an accepting one, all states are alive and no two
  // are equivalent (an object of a schema: its members come one after the other).
  bool all_heights_differ() {
    constexpr int kNew = -2, kOpen = -1;
    height_.assign(n_, kNew);
    seen_.assign(n_, 0);
    std::vector<int>& work = dirty_;
    work.assign(1, 0);  // (every state is reached from the start)
    while (!work.empty()) {
      const int q = work.back();
      const DState& s = d_->s[q];
      const bool entered = height_[q] == kOpen;
      if (height_[q] >= 0) { work.pop_back(); continue; }
      height_[q] = kOpen;
      int h = s.final_ ? 0 : -1;
      bool waits = false, loop = false;
      auto edge = [&](int to) {
        if (height_[to] >= 0) h = std::max(h, height_[to] + 1);
        else if (height_[to] == kOpen) loop = true;
        else { work.push_back(to); waits = true; }
      };
      for (uint32_t k = s.b0; k < s.b1; ++k) edge(d_->b[k].to);
      for (uint32_t k = s.r0; k < s.r1; ++k) edge(d_->r[k].to);
      if (loop || (entered && waits)) return false;
      if (waits) continue;
      if (h < 0 || seen_[h]) return false;
      seen_[h] = 1;
      height_[q] = h;
      work.pop_back();
    }
    return true;
  }
  // A rule without loops of its own: every state is looked at once, after all
  // its successors, and states with equal signatures are one block.  False if there is a loop.
  bool hash_upwards() {
    block_.assign(n_, -1);
    pending_.assign(n_, 0);
    dirty_.clear();
    for (int q = 0; q < n_; ++q) {
      if (!alive_[q]) continue;
      const DState& s = d_->s[q];
      for (uint32_t k = s.b0; k < s.b1; ++k) pending_[q] += alive_[d_->b[k].to];
      for (uint32_t k = s.r0; k < s.r1; ++k) pending_[q] += alive_[d_->r[k].to];
      if (pending_[q] == 0) dirty_.push_back(q);
    }
    const size_t n_alive = (size_t)std::count(alive_.begin(), alive_.end(), 1);
    table_.clear(n_alive);
    for (size_t k = 0; k < dirty_.size(); ++k) {
      const int q = dirty_[k];
      signature(q);
      sig_.push_back(d_->s[q].final_);
      block_[q] = table_.intern(sig_.data(), sig_.size());
      for (const int* p = pred_.begin(q); p != pred_.end(q); ++p)
        if (alive_[*p] && --pending_[*p] == 0) dirty_.push_back(*p);
    }
    sizes_.assign(table_.size(), 0);  // (how many blocks there are)
    return dirty_.size() == n_alive;
  }
  // Partition refinement on (accepting, outgoing edges by block).  When a block falls apart its largest piece keeps
  // the block's number, so that only the predecessors of the smaller pieces have to be looked at again; the
  // states of a block that need not be looked at again still agree with each other, and one of them stands for all.
  void refine() {
    block_.assign(n_, -1);
    sizes_.assign(2, 0);
    dirty_.clear();
    is_dirty_.assign(n_, 0);
    for (int q = 0; q < n_; ++q)
      if (alive_[q]) {
        block_[q] = d_->s[q].final_ ? 1 : 0;
        ++sizes_[block_[q]];
        dirty_.push_back(q);
        is_dirty_[q] = 1;
      }
    // the states of a block as a linked list (to find one that is not dirty)
    head_.assign(2, -1);
    next_.assign(n_, -1);
    prev_.assign(n_, -1);
    for (int q = n_ - 1; q >= 0; --q)
      if (alive_[q]) link(q, block_[q]);
    while (!dirty_.empty()) {
      std::sort(dirty_.begin(), dirty_.end(), [&](int a, int b) { return block_[a] != block_[b] ? block_[a] < block_[b] : a < b; });
      moved_.clear();
      for (size_t k = 0; k < dirty_.size();) {
        const int blk = block_[dirty_[k]];
        size_t end = k;
        while (end < dirty_.size() && block_[dirty_[end]] == blk) ++end;
        if (sizes_[blk] > 1) split(blk, k, end);
        k = end;
      }
      for (int q : dirty_) is_dirty_[q] = 0;
      dirty_.clear();
      for (int q : moved_)
        for (const int* p = pred_.begin(q); p != pred_.end(q); ++p)
          if (alive_[*p] && !is_dirty_[*p] && sizes_[block_[*p]] > 1) { is_dirty_[*p] = 1; dirty_.push_back(*p); }
    }
  }
  void split(int blk, size_t k0, size_t k1) {
    table_.clear(k1 - k0 + 1);
    group_size_.clear();
    group_of_.clear();
    const int others = sizes_[blk] - (int)(k1 - k0);
    if (others > 0) {  // group 0 holds the states that are not dirty
      int q = head_[blk];
      while (is_dirty_[q]) q = next_[q];
      signature(q);
      table_.intern(sig_.data(), sig_.size());
      group_size_.push_back(others);
    }
    for (size_t k = k0; k < k1; ++k) {
      signature(dirty_[k]);
      const int g = table_.intern(sig_.data(), sig_.size());
      if (g == (int)group_size_.size()) group_size_.push_back(0);
      ++group_size_[g];
      group_of_.push_back(g);
    }
    if (group_size_.size() == 1) return;
    const int keeps = (int)(std::max_element(group_size_.begin(), group_size_.end()) - group_size_.begin());
    number_.assign(group_size_.size(), -1);
    number_[keeps] = blk;
    auto number = [&](int g) {
      if (number_[g] < 0) {
        number_[g] = (int)sizes_.size();
        sizes_.push_back(0);
        head_.push_back(-1);
      }
      return number_[g];
    };
    auto move = [&](int q, int to) {
      if (to == blk) return;
      unlink(q, blk);
      --sizes_[blk];
      block_[q] = to;
      ++sizes_[to];
      link(q, to);
      moved_.push_back(q);
    };
    if (others > 0 && keeps != 0)
      for (int q = head_[blk]; q >= 0;) {
        const int nx = next_[q];
        if (!is_dirty_[q]) move(q, number(0));
        q = nx;
      }
    for (size_t k = k0; k < k1; ++k) move(dirty_[k], number(group_of_[k - k0]));
  }
  void signature(int q) {
    sig_.clear();
    const DState& s = d_->s[q];
    int hi = -2, to = -1;  // the last range that was put down
    for (uint32_t k = s.b0; k < s.b1; ++k) {
      const ByteEdge& e = d_->b[k];
      const int blk = block_[e.to];
      if (blk < 0) continue;  // (trimmed)
      if (blk == to && hi + 1 == (int)e.lo) sig_.back() = e.hi;
      else { sig_.push_back(blk); sig_.push_back(e.lo); sig_.push_back(e.hi); }
      hi = e.hi;
      to = blk;
    }
    sig_.push_back(-2);
    for (uint32_t k = s.r0; k < s.r1; ++k)
      if (block_[d_->r[k].to] >= 0) { sig_.push_back(d_->r[k].rule); sig_.push_back(block_[d_->r[k].to]); }
  }
  void link(int q, int blk) {
    prev_[q] = -1;
    next_[q] = head_[blk];
    if (next_[q] >= 0) prev_[next_[q]] = q;
    head_[blk] = q;
  }
  void unlink(int q, int blk) {
    if (prev_[q] >= 0) next_[prev_[q]] = next_[q];
    else head_[blk] = next_[q];
    if (next_[q] >= 0) prev_[next_[q]] = prev_[q];
  }
  int n_ = 0;
  const Dfa* d_ = nullptr;
  Buckets pred_;
  std::vector<char> alive_, is_dirty_, seen_;
  std::vector<int> block_, sizes_, head_, next_, prev_, dirty_, moved_, sig_, pending_, group_size_, group_of_, number_, height_;
  SequenceTable table_;
};

// The CPUs that this thread, and those that it starts, may run on.
int usable_cpus() {
  cpu_set_t set;
  if (sched_getaffinity(0, sizeof(set), &set) == 0) return CPU_COUNT(&set);
  return std::max(1, (int)std::thread::hardware_concurrency());  // (more CPUs than the set has room for)
}

// Threads that compile: a compile counts itself (the object) and its helpers.
struct Compiling {
  Compiling() { ++threads(); }
  ~Compiling() { --threads(); }
  Compiling(const Compiling&) = delete;
  Compiling& operator=(const Compiling&) = delete;
  static std::atomic<int>& threads() {
    static std::atomic<int> n{0};
    return n;
  }
};

// Threads of one compile, which ends them.  Starting one costs the compile 15 to 20 us, so only large grammars have any, and
// only as long as all that compile in this process are no more than there are CPUs: 36 KB schema grammar on one CPU 3750 us with
// three helpers and 3600 without, eight compiles on eight CPUs 880 to 930 us each and 690 to 740.
class Helpers {
 public:
  ~Helpers() { join(); }
  // starts up to n threads that run `work` and returns how many there are (the caller runs it as well, or instead)
  int start(int n, const std::function<void()>& work) {
    const int cpus = usable_cpus();
    threads_.reserve((size_t)n);
    while ((int)threads_.size() < n) {
      if (++Compiling::threads() > cpus) {
        --Compiling::threads();
        break;
      }
      try {
        threads_.emplace_back(work);
      } catch (const std::exception&) {  // no more threads: those that there are, and the caller, do it all
        --Compiling::threads();
        break;
      }
    }
    return (int)threads_.size();
  }
  void join() {
    for (std::thread& t : threads_) t.join();
    Compiling::threads() -= (int)threads_.size();
    threads_.clear();
  }

 private:
  std::vector<std::thread> threads_;
};

// The minimal DFA of every productive rule.  Rules do not depend on each other: in a large grammar several threads take them
// in turn, as many as the largest rule (of `largest` states) leaves work for.  36 KB schema grammar with 239 rules: 720 of 1660
// us by one thread; the compile takes 890 us with three more, and what does not go into the tables made beside them, where one
// compile follows the other, 1370 instead of 1756 as a part of builds, where the threads' cores have been idle.
constexpr int kManyStates = 8000;  // of the NFA: some 250 us of work
constexpr int kManyNodes = 4000;    // of the automaton: what is made beside the tables takes some 50 us
constexpr int kCompileHelpers = 3;
std::vector<Dfa> determinize(const Nfa& nfa, const std::vector<int>& start, const std::vector<int>& accept, const std::vector<char>& productive,
                             const std::vector<char>& nullable, int largest) {
  const int R = (int)start.size();
  std::vector<Dfa> dfa(R);
  std::atomic<int> next{0};
  std::atomic<bool> failed{false};
  std::exception_ptr failure;
  auto work = [&] {
    try {
      int r = next.fetch_add(1);
      if (r >= R) return;  // (the determinizer is as large as the NFA: made when there is a rule for it)
      Determinizer determinizer(nfa, productive, nullable);
      Minimizer minimizer;
      Dfa d;
      for (; r < R && !failed; r = next.fetch_add(1)) {
        if (!productive[r]) continue;
        determinizer.run(start[r], accept[r], d);
        dfa[r] = minimizer.run(d);
      }
    } catch (...) {
      if (!failed.exchange(true)) failure = std::current_exception();
    }
  };
  Helpers helpers;
  if (nfa.size() >= kManyStates) helpers.start(std::min(kCompileHelpers, nfa.size() / largest - 1), work);
  work();
  helpers.join();
  if (failed) std::rethrow_exception(failure);
  return dfa;
}

}  // namespace

std::vector<int32_t> Automaton::node_path(int32_t node) const {
  std::vector<int32_t> p;
  for (; path_parent[node] >= 0; node = path_parent[node]) p.push_back(path_symbol[node]);
  std::reverse(p.begin(), p.end());
  return p;
}

Automaton compile_grammar(const std::string& text, const std::string& root) {
  const Compiling compiling;
  const Lexed lexed = lex(text);
  Nfa nfa;
  nfa.reserve(lexed.text.size() + lexed.toks.size() * 2);  // (a byte of a literal is an edge, a name or an operator one or two)
  Parser parser(lexed, nfa);
  parser.run();
  nfa.finish();
  const int R = (int)parser.names_.size();
  auto root_it = parser.rule_index_.find(root);
  if (root_it == parser.rule_index_.end())
    throw Failure(XGM_ERR_UNDEFINED_RULE, "grammar: root rule '" + root + "' is not defined");
  const int root_rule = root_it->second;

  // productive rules (derive at least one string) and nullable rules (derive "")
  const std::vector<char> productive = derivable(nfa, parser.start_, parser.accept_, [](const NEdge&) { return true; });
  if (!productive[root_rule]) throw Failure(XGM_ERR_UNPRODUCTIVE, "grammar: the root rule derives no string");
  const std::vector<char> nullable = derivable(nfa, parser.start_, parser.accept_, [](const NEdge& e) { return e.kind != 1; });

  const std::vector<Dfa> dfa = determinize(nfa, parser.start_, parser.accept_, productive, nullable, parser.largest_);

  // rules reachable from the root
  std::vector<int> new_index(R, -1), order;
  {
    std::vector<int> work{root_rule};
    new_index[root_rule] = 0;
    order.push_back(root_rule);
    while (!work.empty()) {
      int r = work.back();
      work.pop_back();
      for (auto& e : dfa[r].r)
        if (new_index[e.rule] < 0) { new_index[e.rule] = (int)order.size(); order.push_back(e.rule); work.push_back(e.rule); }
    }
  }

  // Small rules first: the rules shared by many call sites (strings, numbers,
  // white space) are small, and the kernels keep the headers of the lowest
  // node ids on chip.
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return dfa[a].s.size() < dfa[b].s.size(); });
  for (size_t k = 0; k < order.size(); ++k) new_index[order[k]] = (int)k;

  Automaton A;
  A.root_rule = new_index[root_rule];
  int total = 0;
  for (int r : order) { A.rule_start.push_back(total); total += (int)dfa[r].s.size(); A.rule_names.push_back(parser.names_[r]); }
  if (total > XGM_MAX_NODES) throw Failure(XGM_ERR_TOO_LARGE, "grammar: automaton has " + std::to_string(total) + " nodes (limit 32767)");
  A.n_nodes = total;
  A.node_rule.resize(total);
  A.node_final.resize(total);
  A.node_dead_end.resize(total);
  for (size_t k = 0; k < order.size(); ++k) {
    const int base = A.rule_start[k];
    const Dfa& d = dfa[order[k]];
    for (size_t q = 0; q < d.s.size(); ++q) {
      const int n = base + (int)q;
      const DState& s = d.s[q];
      A.node_rule[n] = (int)k;
      A.node_final[n] = s.final_;
      A.node_dead_end[n] = s.final_ && s.b0 == s.b1 && s.r0 == s.r1;
      for (uint32_t e = s.b0; e < s.b1; ++e) A.bedges.items.push_back({d.b[e].lo, d.b[e].hi, base + d.b[e].to});
      A.bedges.end_row();
      for (uint32_t e = s.r0; e < s.r1; ++e) A.redges.items.push_back({new_index[d.r[e].rule], base + d.r[e].to});
      A.redges.end_row();
    }
  }
  const int NR = (int)order.size();
  A.node_on_top.assign(total, 0);
  for (auto& e : A.bedges.items) A.node_on_top[e.to] = !A.node_dead_end[e.to];
  for (auto& e : A.redges.items) A.node_on_top[e.to] = !A.node_dead_end[e.to];

  // left recursion: a chain of references taken at rule starts that returns to its origin
  std::vector<int> callees_first;  // the rules, those entered at a rule's start before the rule
  {
    std::vector<int> color(NR, 0);
    std::vector<std::pair<int, size_t>> stack;
    for (int s = 0; s < NR; ++s) {
      if (color[s]) continue;
      stack.push_back({s, 0});
      color[s] = 1;
      while (!stack.empty()) {
        auto& top = stack.back();
        const auto refs = A.redges[A.rule_start[top.first]];
        if (top.second < refs.size()) {
          int t = refs[top.second++].rule;
          if (color[t] == 1)
            throw Failure(XGM_ERR_LEFT_RECURSION, "grammar: rule '" + A.rule_names[t] + "' is left-recursive");
          if (color[t] == 0) { color[t] = 1; stack.push_back({t, 0}); }
        } else {
          color[top.first] = 2;
          callees_first.push_back(top.first);
          stack.pop_back();
        }
      }
    }
  }

  // FIRST sets: bytes with which an instance of the rule can begin (no chain of references at rule starts returns to its origin)
  A.first.assign(NR, {});
  auto first_of_node = [&](int n) {
    ByteSet f;
    for (auto& e : A.bedges[n]) f.set_range(e.lo, e.hi);
    for (auto& e : A.redges[n]) f.add(A.first[e.rule]);
    return f;
  };
  for (int r : callees_first) A.first[r] = first_of_node(A.rule_start[r]);
  A.node_first.resize(total);
  for (int n = 0; n < total; ++n) A.node_first[n] = first_of_node(n);

  // What the kernels' tables do not need, or only at their end, is made beside them.
  auto relations = [&] {
    // What one reference hands on: rule e.rule can be followed by what node e.to consumes, and by what follows the
    // referring rule if that may end there; its contexts (see automaton.hpp) are e.to, or the referring rule's if
    // e.to is a dead end.  Both relations between rules are kept as pairs and followed until nothing changes.
    // Nothing follows the root rule itself (end of the text).
    A.follow.assign(NR, {});
    std::vector<std::pair<int, int>> hands_follow, hands_contexts;  // (from rule, to rule)
    Buckets own_contexts;
    own_contexts.fill(NR, [&](auto put) {
      for (int n = 0; n < total; ++n)
        for (auto& e : A.redges[n])
          if (!A.node_dead_end[e.to]) put(e.rule, e.to);
    });
    for (int n = 0; n < total; ++n)
      for (auto& e : A.redges[n]) {
        A.follow[e.rule].add(A.node_first[e.to]);
        if (A.node_final[e.to] && e.rule != A.node_rule[n]) hands_follow.push_back({A.node_rule[n], e.rule});
        if (A.node_dead_end[e.to] && e.rule != A.node_rule[n]) hands_contexts.push_back({A.node_rule[n], e.rule});
      }
    for (auto* pairs : {&hands_follow, &hands_contexts}) {
      std::sort(pairs->begin(), pairs->end());
      pairs->erase(std::unique(pairs->begin(), pairs->end()), pairs->end());
    }
    for (bool changed = true; changed;) {
      changed = false;
      for (auto& p : hands_follow) changed |= A.follow[p.second].add(A.follow[p.first]);
    }
    A.contexts.assign(NR, {});
    for (int r = 0; r < NR; ++r) {
      auto& c = A.contexts[r];
      c.assign(own_contexts.begin(r), own_contexts.end(r));
      std::sort(c.begin(), c.end());
      c.erase(std::unique(c.begin(), c.end()), c.end());
    }
    for (bool changed = true; changed;) {
      changed = false;
      std::vector<int32_t> both;
      for (auto& p : hands_contexts) {
        auto& to = A.contexts[p.second];
        const auto& from = A.contexts[p.first];
        both.clear();
        std::set_union(to.begin(), to.end(), from.begin(), from.end(), std::back_inserter(both));
        if (both.size() != to.size()) { to.assign(both.begin(), both.end()); changed = true; }
      }
    }

    // forced frames: at the bottom of a stack are the root rule and what it (or such a rule) enters by a tail call
    {
      std::vector<char> at_bottom(NR, 0);
      at_bottom[A.root_rule] = 1;
      for (bool changed = true; changed;) {
        changed = false;
        for (auto& p : hands_contexts)
          if (at_bottom[p.first] && !at_bottom[p.second]) { at_bottom[p.second] = 1; changed = true; }
      }
      A.forced.assign(NR, {});
      for (int r = 0; r < NR; ++r) {
        int cur = r;
        while (A.contexts[cur].size() == 1 && !at_bottom[cur] && (int)A.forced[r].size() < kMaxForced) {
          A.forced[r].push_back(A.contexts[cur][0]);
          cur = A.node_rule[A.contexts[cur][0]];
        }
        // a short way down to the bottom is what the levels of a mask cache reach frame by frame
        if (A.contexts[cur].empty() && (int)A.forced[r].size() <= kShortWayDown) A.forced[r].clear();
      }
    }

    // witness paths (breadth-first from each rule start)
    A.path_parent.assign(total, -1);
    A.path_symbol.assign(total, -1);
    {
      std::vector<char> seen(total, 0);
      std::vector<int> q;
      for (int r = 0; r < NR; ++r) {
        q.assign(1, A.rule_start[r]);
        seen[q[0]] = 1;
        for (size_t k = 0; k < q.size(); ++k) {
          const int n = q[k];
          auto step = [&](int to, int symbol) {
            if (seen[to]) return;
            seen[to] = 1;
            A.path_parent[to] = n;
            A.path_symbol[to] = symbol;
            q.push_back(to);
          };
          for (auto& e : A.bedges[n]) step(e.to, e.lo);
          for (auto& e : A.redges[n]) step(e.to, 256 + e.rule);
        }
      }
    }
  };
  std::exception_ptr failure;
  Helpers beside;
  const bool apart = total >= kManyNodes && beside.start(1, [&] {
    try {
      relations();
    } catch (...) {
      failure = std::current_exception();
    }
  }) == 1;
  if (!apart) relations();

  // ---- flatten for the device
  auto plain = [&](int n) { return A.redges[n].empty() && A.bedges[n].size() <= 1; };
  auto byte_target = [&](int n, int c) {
    for (auto& e : A.bedges[n]) if (e.lo <= c && c <= e.hi) return e.to;
    return -1;
  };
  // byte classes: bytes that no node's edges and no FIRST set tell apart.  The sets that tell bytes apart are, for
  // every node, the bytes that lead to the same target, and the FIRST sets; each distinct one is looked at once.
  A.cls.assign(256, 0);
  {
    std::vector<int> cls(256, 0);
    int n_cls = 1;
    auto split_by = [&](const ByteSet& set) {
      int inside[256];  // per class: the class of its bytes that are in the set
      bool has_out[256] = {};
      for (int k = 0; k < n_cls; ++k) inside[k] = -1;
      for (int c = 0; c < 256; ++c)
        if (!set.test(c)) has_out[cls[c]] = true;
      const int n0 = n_cls;
      for (int c = 0; c < 256; ++c) {
        const int k = cls[c];
        if (k >= n0 || !has_out[k] || !set.test(c)) continue;
        if (inside[k] < 0) inside[k] = n_cls++;
        cls[c] = inside[k];
      }
    };
    std::vector<char> range_done(256 * 256, 0);
    SequenceTable sets_done;
    sets_done.clear(256);
    auto split_once = [&](const ByteSet& set) {
      int words[8];
      for (int k = 0; k < 8; ++k) words[k] = (int)set.w[k];
      bool is_new = false;
      sets_done.intern(words, 8, &is_new);
      if (is_new) split_by(set);
    };
    for (int n = 0; n < total; ++n) {
      const auto be = A.bedges[n];
      for (size_t k = 0; k < be.size(); ++k) {
        bool alone = true, seen_before = false;
        for (size_t j = 0; j < be.size(); ++j)
          if (j != k && be[j].to == be[k].to) { alone = false; seen_before = seen_before || j < k; }
        if (seen_before) continue;
        if (alone) {
          char& done = range_done[be[k].lo * 256 + be[k].hi];
          if (done) continue;
          done = 1;
        }
        ByteSet set;
        for (auto& e : be)
          if (e.to == be[k].to) set.set_range(e.lo, e.hi);
        split_once(set);
      }
    }
    for (int r = 0; r < NR; ++r) split_once(A.first[r]);
    // numbered in the order of their first bytes
    std::vector<int> renum(n_cls, -1);
    A.n_cls = 0;
    for (int c = 0; c < 256; ++c) {
      if (renum[cls[c]] < 0) renum[cls[c]] = A.n_cls++;
      A.cls[c] = (uint8_t)renum[cls[c]];
    }
  }
  std::vector<int> cls_rep(A.n_cls, -1);
  for (int c = 255; c >= 0; --c) cls_rep[A.cls[c]] = c;

  // Alternatives of node n on byte c, in the order the walk tries them:
  //  * the byte edge;
  //  * for every reference whose callee can start with c: enter the callee.
  //    - If the return node is a dead end (accepting, no outgoing edges) no
  //      frame is needed: returning there could only be followed by another
  //      return, so the callee returns straight to the caller's parent.
  //    - Otherwise, if the callee does nothing with c but consume it and end (a single
  //      byte edge from its start into a dead end, no reference of its own
  //      that could start with c), the whole call is the move "consume c, go
  //      to the return node"; the frame would be pushed and popped unseen.
  //    Both are exact for the token classes too: neither changes which bytes
  //    are consumed inside the frame the walk started in.
  // per rule: the byte classes that an instance can start with, and whether it then consumes the byte and ends
  std::vector<std::vector<std::pair<uint8_t, bool>>> starts(NR);
  for (int r = 0; r < NR; ++r)
    for (int k = 0; k < A.n_cls; ++k) {
      const int c = cls_rep[k], s = A.rule_start[r];
      if (!A.first[r].test(c)) continue;
      const int m = byte_target(s, c);
      bool callee_refs = false;
      for (auto& e2 : A.redges[s]) callee_refs = callee_refs || A.first[e2.rule].test(c);
      starts[r].push_back({(uint8_t)k, m >= 0 && A.node_dead_end[m] && !callee_refs});
    }

  // Branching nodes: for every byte class one of the node's few outcomes.
  // Which class leads to which outcome index is the node's "shape" (shared by
  // many nodes, e.g. every  ws "," ws  position); the outcomes themselves are
  // the node's own slice of `targets`.
  // A list of alternatives is kept as the number of (the list without its last, its last); 0 is the empty one.
  struct AltList { int before; uint32_t alt; int length; int pool_at; };
  std::vector<AltList> lists{{-1, 0u, 0, -1}};
  SequenceTable list_ids;
  list_ids.clear(1024);
  uint32_t last_single = 0u;  // (a reference has the same alternative for all bytes that its callee can start with)
  int last_single_id = -1;
  auto extend = [&](int list, uint32_t alt) {
    if (list == 0 && last_single_id >= 0 && alt == last_single) return last_single_id;
    for (int k = list; k > 0; k = lists[k].before)
      if (lists[k].alt == alt) return list;
    const int key[2] = {list, (int)alt};
    bool is_new = false;
    const int id = list_ids.intern(key, 2, &is_new) + 1;
    if (is_new) lists.push_back({list, alt, lists[list].length + 1, -1});
    if (list == 0) { last_single = alt; last_single_id = id; }
    return id;
  };
  // what node n does with the byte classes that lead anywhere: (class, list) pairs by class
  std::vector<int> list_of(A.n_cls, 0), classes;
  auto lists_at = [&](int n, std::vector<std::pair<int, int>>* out) {
    classes.clear();
    auto add = [&](int k, uint32_t alt) {
      if (list_of[k] == 0) classes.push_back(k);
      list_of[k] = extend(list_of[k], alt);
    };
    for (auto& e : A.bedges[n])
      for (int c = e.lo; c <= e.hi; ++c)
        if (cls_rep[A.cls[c]] == c) add(A.cls[c], (kMoveTag << 16) | (uint32_t)e.to);
    for (auto& e : A.redges[n])
      for (auto& st : starts[e.rule]) {
        uint32_t alt;
        if (A.node_dead_end[e.to]) alt = (kTailTag << 16) | (uint32_t)A.rule_start[e.rule];
        else if (st.second) alt = (kMoveTag << 16) | (uint32_t)e.to;
        else alt = ((uint32_t)e.to << 16) | (uint32_t)A.rule_start[e.rule];
        add(st.first, alt);
      }
    std::sort(classes.begin(), classes.end());
    out->clear();
    for (int k : classes) { out->push_back({k, list_of[k]}); list_of[k] = 0; }
  };
  std::vector<std::pair<int, int>> at_node;
  std::vector<int> start_lists((size_t)NR * A.n_cls, 0);  // per rule and class: the list at the rule's start
  for (int r = 0; r < NR; ++r) {
    lists_at(A.rule_start[r], &at_node);
    for (auto& kl : at_node) start_lists[(size_t)r * A.n_cls + kl.first] = kl.second;
  }
  auto pool_room = [&] {
    if (A.alts.size() >= 0x7FFF) throw Failure(XGM_ERR_TOO_LARGE, "grammar: alternatives pool is full");
    return (int)A.alts.size();
  };
  // The only alternative at a rule's start for class k is a call: the run of calls that starts with it, in the pool; -1 if it
  // is too short to be worth its place there or if runs are not wanted.  (At other nodes the first call is a step of its
  // own: its return node would make the run another one for every place that refers to the rule, and what the tables
  // grow by is missing on chip.)
  SequenceTable run_ids, run_frames;
  std::vector<int> run_at, frames_at, run;
  bool with_runs = true;
  auto run_of = [&](uint32_t alt, int k) {
    run.clear();  // the frames
    int node = 0, calls = 0;
    bool consumes = false;
    for (;; ++calls) {
      if ((alt >> 16) == kMoveTag) { consumes = true; node = (int)(alt & 0xFFFF); break; }
      if ((alt >> 16) != kTailTag) run.push_back((int)(alt >> 16));
      node = (int)(alt & 0xFFFF);  // the start of the rule that is entered
      const AltList& next = lists[start_lists[(size_t)A.node_rule[node] * A.n_cls + k]];
      if (next.length != 1 || (int)run.size() >= kMaxRun) { ++calls; break; }
      alt = next.alt;
    }
    if (calls < kShortestRun || !with_runs) return -1;
    bool is_new = false;
    const int frames = run_frames.intern(run.data(), run.size(), &is_new);
    if (is_new) {
      frames_at.push_back(pool_room());
      for (size_t j = 0; j < run.size(); j += 2) A.alts.push_back((uint32_t)run[j] | (j + 1 < run.size() ? (uint32_t)run[j + 1] << 16 : 0u));
    }
    const int key[3] = {frames, consumes, node};
    const int id = run_ids.intern(key, 3, &is_new);
    if (is_new) {
      run_at.push_back(pool_room());
      A.alts.push_back(kRunFlag | (consumes ? kRunConsumes : 0u) | (uint32_t)run.size() << kRunFramesShift | (uint32_t)frames_at[frames]);
      A.alts.push_back((uint32_t)node);
    }
    return run_at[id];
  };
  SequenceTable shape_ids;
  std::vector<int> shape, rev;  // shape: (class, outcome) pairs of the classes that lead anywhere
  std::vector<uint16_t> outcomes;
  auto flatten = [&](int n) {
    NodeHdr& h = A.hdr[n];
    h.flags = (A.node_final[n] ? kFlagFinal : 0) | (A.node_dead_end[n] ? kFlagDeadEnd : 0);
    if (plain(n)) {
      if (A.bedges[n].size() == 1) { h.lo = A.bedges[n][0].lo; h.hi = A.bedges[n][0].hi; h.target = (uint16_t)A.bedges[n][0].to; }
      return;
    }
    lists_at(n, &at_node);
    outcomes.clear();
    shape.clear();
    for (auto& kl : at_node) {
      AltList& list = lists[kl.second];
      uint16_t entry;
      if (list.length == 1 && (list.alt >> 16) == kMoveTag) entry = (uint16_t)(list.alt & 0xFFFF);
      else if (const int at = list.length == 1 && n == A.rule_start[A.node_rule[n]] ? run_of(list.alt, kl.first) : -1; at >= 0) entry = (uint16_t)(kAltFlag | at);
      else {
        if (list.length > 250) throw Failure(XGM_ERR_TOO_LARGE, "grammar: too many alternatives at one node");
        if (list.pool_at < 0) {
          list.pool_at = pool_room();
          A.alts.push_back((uint32_t)list.length);
          rev.clear();
          for (int j = kl.second; j > 0; j = lists[j].before) rev.push_back((int)lists[j].alt);
          for (size_t j = rev.size(); j-- > 0;) A.alts.push_back((uint32_t)rev[j]);
        }
        entry = (uint16_t)(kAltFlag | list.pool_at);
        A.max_alts = std::max<int>(A.max_alts, list.length);
      }
      size_t idx = std::find(outcomes.begin(), outcomes.end(), entry) - outcomes.begin();
      if (idx == outcomes.size()) outcomes.push_back(entry);
      if (idx >= kDeadShape) throw Failure(XGM_ERR_TOO_LARGE, "grammar: too many distinct outcomes at one node");
      shape.push_back(kl.first);
      shape.push_back((int)idx);
    }
    bool is_new = false;
    const uint32_t id = (uint32_t)shape_ids.intern(shape.data(), shape.size(), &is_new);
    if (is_new) {
      if (id >= 0xFFFF) throw Failure(XGM_ERR_TOO_LARGE, "grammar: too many node shapes");
      const size_t at = A.shapes.size();
      A.shapes.resize(at + A.n_cls, kDeadShape);
      for (size_t j = 0; j < shape.size(); j += 2) A.shapes[at + shape[j]] = (uint8_t)shape[j + 1];
    }
    if (A.targets.size() + outcomes.size() > 0xFFFF) throw Failure(XGM_ERR_TOO_LARGE, "grammar: outcome table is full");
    h.flags |= kFlagBranching;
    h.lo = (uint8_t)(id & 0xFF);                  // shape id, low and high byte
    h.hi = (uint8_t)(id >> 8);
    h.target = (uint16_t)A.targets.size();        // start of this node's outcomes
    A.targets.insert(A.targets.end(), outcomes.begin(), outcomes.end());
  };
  // (a grammar whose pool has no room for the runs does without them)
  for (bool done = false; !done;) {
    A.hdr.assign(total, NodeHdr{1, 0, 0, 0});
    A.alts.clear();
    A.shapes.clear();
    A.targets.clear();
    shape_ids.clear(256);
    run_ids.clear(256);
    run_frames.clear(64);
    run_at.clear();
    frames_at.clear();
    for (auto& l : lists) l.pool_at = -1;
    try {
      for (int n = 0; n < total; ++n) flatten(n);
      done = true;
    } catch (const Failure&) {
      if (!with_runs) throw;
      with_runs = false;
    }
  }
  A.n_shapes = (int32_t)shape_ids.size();
  beside.join();
  if (failure) std::rethrow_exception(failure);
  for (int n = 0; n < total; ++n)
    A.hdr[n].flags |= (uint32_t)A.node_rule[n] << 16 | (uint32_t)(1 + A.forced[A.node_rule[n]].size()) << kChainShift;
  if (A.alts.empty()) A.alts.push_back(0);
  if (A.shapes.empty()) A.shapes.assign(A.n_cls, kDeadShape);
  if (A.targets.empty()) A.targets.push_back(0);
  return A;
}

}  // namespace xgm
