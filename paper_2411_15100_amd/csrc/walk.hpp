// The token walk shared by the classify and fill kernels.  It is plain C++
// over the flattened tables, so the same code also compiles for the host,
// where the library's tests run it against the CPU oracle without a GPU.
#pragma once
#include <hip/hip_runtime_api.h>
#include <hip/hip_vector_types.h>

#include <cstdint>

#include "kernels.hpp"

#if defined(__HIPCC__) || defined(__HIP__)
#define XGM_HD __host__ __device__ __forceinline__
#else
#define XGM_HD inline
#endif

namespace xgm {

constexpr uint32_t kAltFlagD = 0x8000;
constexpr uint32_t kMoveTagD = 0xFFFF;
constexpr uint32_t kTailTagD = 0xFFFE;
constexpr uint32_t kRunFlagD = 0x80000000u, kRunConsumesD = 0x40000000u;  // a run of calls (see automaton.hpp)
XGM_HD uint32_t run_frames(uint32_t word) { return (word >> 16) & 0x3Fu; }
XGM_HD uint32_t run_frames_at(uint32_t word) { return word & 0x7FFFu; }
constexpr uint32_t kLiveBase = 0x8000;  // stack handles >= this refer to the request's live frames

// Whether any lane of the wave that gets here has it so (on the host: whether it is so).  What stands behind such a test costs a
// wave of which no lane needs it one scalar branch, where a test of every lane by itself turns lanes off and on again.
// (classify_walks_kernel, 11867-node schema grammar x 151936: 301 us with lookups that every lane branched through by itself,
// 284 so; JSON x 32000 24.9 and 23.7; exit_positions_kernel 18.4 and 17.9, context_level1_kernel 111 and 109.)
#if defined(__HIP_DEVICE_COMPILE__)
#define XGM_ANY(condition) (__builtin_amdgcn_ballot_w64(condition) != 0ull)
#else
#define XGM_ANY(condition) (condition)
#endif

// Table access for the walk: what node n does with byte c: `to` = the node that a byte edge leads to, or (kAltFlagD) where in
// the alternatives pool the moves and calls are, `none` = neither; may the rule end at n (fin), and n's rule (for `follows`:
// can c come right after an instance of it at all).
struct Looked {
  uint32_t to;
  bool none;
  uint32_t fin, rule;
};
struct CompactTab {
  TabView v;
  XGM_HD Looked look(uint32_t n, uint32_t c) const {
    const uint2 h = (n < (uint32_t)v.n_near) ? v.hdr_near[n] : v.hdr_far[n];
    Looked r{h.x >> 16, c < (h.x & 0xFFu) || c > ((h.x >> 8) & 0xFFu), h.y & 1u, h.y >> 16};
    if (h.y & 2u) {
      const uint32_t si = v.shapes[(h.x & 0xFFFFu) * v.n_cls + v.cls[c]];
      r.none = si == 0xFFu;
      r.to = r.none ? 0u : v.targets[(h.x >> 16) + si];
    }
    return r;
  }
  XGM_HD uint32_t alt(uint32_t idx) const { return v.alts[idx]; }
  XGM_HD bool is_final(uint32_t n) const { return ((n < (uint32_t)v.n_near) ? v.hdr_near[n] : v.hdr_far[n]).y & 1u; }
  XGM_HD bool is_dead_end(uint32_t n) const { return ((n < (uint32_t)v.n_near) ? v.hdr_near[n] : v.hdr_far[n]).y & 4u; }
  // the rule of node n, as the handle of its 256-bit FOLLOW set; is byte c in the set of rule r?
  XGM_HD uint32_t follow_of(uint32_t n) const { return ((n < (uint32_t)v.n_near) ? v.hdr_near[n] : v.hdr_far[n]).y >> 16; }
  XGM_HD uint32_t follows(uint32_t r, uint32_t c) const { return (v.follow_rules[r * 8 + (c >> 5)] >> (c & 31)) & 1u; }
};

// The first 15 bytes of a token as four plain words (kept in registers: the
// byte at a run-time index is picked with selects, never through memory).
struct TokenWords {
  uint32_t w0, w1, w2, w3;
  XGM_HD explicit TokenWords(const uint4& tk) : w0(tk.x), w1(tk.y), w2(tk.z), w3(tk.w) {}
};
XGM_HD uint32_t token_byte(const TokenWords& t, const uint8_t* ext, int i) {
  if (!XGM_ANY(i >= 15) || i < 15) {
    // bit masks instead of selects: a select between loaded values invites the
    // compiler to index a copy in scratch memory
    const uint32_t m4 = 0u - (((uint32_t)i >> 2) & 1u), m8 = 0u - (((uint32_t)i >> 3) & 1u);
    const uint32_t lo = (t.w1 & m4) | (t.w0 & ~m4), hi = (t.w3 & m4) | (t.w2 & ~m4);
    const uint32_t w = (hi & m8) | (lo & ~m8);
    return (w >> (((uint32_t)i & 3u) * 8u)) & 0xFFu;
  }
  return ext[i];
}
XGM_HD uint32_t token_byte(const uint4& tk, const uint8_t* ext, int i) { return token_byte(TokenWords(tk), ext, i); }

// Depth-first walk of one token through the pushdown automaton (section 2.2,
// Appendix A) from the configuration (node on top, `depth - 1` live frames
// below it).  Alternatives at a configuration, in the order they are tried:
// the byte edge, the rule references whose callee can start with the next
// byte (push the return node, enter the callee), and - if the node is
// accepting and a byte was consumed since the last push - the return to the
// frame below.  A return in front of a byte that can never follow the
// node's rule is not tried at all: it cannot lead anywhere (but out of the bottom
// frame, which is noted: see kUncertainPlain), and leaving it out
// keeps runs like the inside of a string or a name free of pending alternatives.
// (With such returns tried where kUncertainPlain is told from kReject the classify kernel's
// walks took 362 us for an 11867-node schema grammar and 151936 tokens, now 300; exit_positions_kernel
// 45, now 19; for a scripting grammar and 128256 tokens 176 and 59, now 152 and 42.)  Frames pushed during the walk live in a small arena with
// parent links, so that backing up to a pending alternative never copies a
// stack (the persistent stack of section 3.3, in miniature).
//
// BUILD = true:  nothing is known below the bottom frame (the start frame, or
//                `depth` - 1 frames that are certain to lie below it);
//                result kAccept / kUncertain / kReject as in section 3.1,
//                refined by one byte of context (section 3.2 in miniature):
//                leaving the bottom frame while bytes remain only counts if
//                the next byte is in the FOLLOW set of rule `follow` (the bytes
//                that can come right after an instance of the bottom node's rule
//                in any context; `T.follow_of(bottom_node)`); a token that left the frame only in front of other
//                bytes is kUncertainPlain: context-dependent by section 3.1
//                alone, rejected in every context by the refinement.
// BUILD = false: frames below are live[0 .. depth-2]; result kAccept (token
//                allowed) or kReject.
// PRUNE:         returns in front of a byte that can never follow the rule are left out (always when BUILD = false;
//                with BUILD = true kUncertainPlain is then not told from kReject).
// kOverflow: a limit was hit; the caller records the pair.
// `steps_out` (may be null) receives the number of automaton steps taken.
// `i0`: index of the first byte to consume (the walk may start inside the token).
// `exits_out` (BUILD only, may be null): bit min(k, 31) is set for every
// position k at which the bottom frame is left in front of a byte of `follow`.
// `Live` is anything indexable that yields the live frames (a plain pointer,
// or a view that knows which of them sit in LDS).
// `End` decides what the end of the token means.  The default returns kAccept
// at the first path that consumes every byte.  An enumerating End is instead
// called with every configuration (node, stack handle, arena, live frames) in
// which the token can end, and the walk goes on to the next path; the result
// is then kReject (or kOverflow).
// `Mem` keeps the frames pushed by the walk (ret | parent handle << 16) and the
// pending alternatives (x = node | sp << 16 ; y = i | alt << 8 | top << 16 | f << 24).
struct FirstPathEnds {
  static constexpr bool kEnumerate = false;
  template <class Mem, class Live>
  XGM_HD void operator()(uint32_t, uint32_t, const Mem&, const Live&) const {}
};
struct PrivateMem {
  uint32_t arena[kArenaFrames];
  uint2 choices[kChoicePoints];
  XGM_HD uint32_t frame(uint32_t k) const { return arena[k]; }
  XGM_HD void set_frame(uint32_t k, uint32_t v) { arena[k] = v; }
  XGM_HD uint2 choice(uint32_t k) const { return choices[k]; }
  XGM_HD void set_choice(uint32_t k, uint2 v) { choices[k] = v; }
};
template <bool BUILD, bool PRUNE, class Mem, class Tab, class Live, class End>
XGM_HD int walk_token_in(Mem& mem, const Tab& T, const uint4 tk, const uint8_t* ext, const int len,
                         const uint32_t start_node, const Live& live, const uint32_t depth,
                         uint32_t* steps_out, const uint32_t follow, const int i0, uint32_t* exits_out, const End& at_end) {
  if (len > kMaxTokenLen) return kOverflow;
  const TokenWords tw(tk);
  uint32_t n = start_node, sp = kLiveBase + depth - 1, f = 1, alt = 0, top = 0, csp = 0;
  uint32_t needed = 0;           // frames below this are needed by the most recent pending alternative
  int i = i0;
  uint32_t c = i < len ? token_byte(tw, ext, i) : 0u;
  // The stack whose frames were last looked at because of such a return (see below), and how many steps it stands for: they
  // count, so that a text that may be read in many ways is known by its walks (DevCache::long_walks).
  uint32_t looked_at = 0xFFFFu;
  int down = 0;
  uint32_t left_frame = 0u;  // bit 0: the bottom frame was left with bytes remaining, bit 1: in front of a byte of `follow`
  for (int steps = 0;; ++steps) {
    if (steps_out) *steps_out = (uint32_t)steps;
    if (i == len && !End::kEnumerate) return kAccept;
    if (steps >= kMaxSteps) return kOverflow;
    if (i == len) {
      at_end(n, sp, mem, live);      // then on to the next path
    } else {
      const Looked at = T.look(n, c);
      const uint32_t rule = at.rule;
      uint32_t can_pop = at.fin & f;
      if (XGM_ANY(can_pop)) {
        if (sp == kLiveBase) {
          // The bottom frame may end here (nothing is known below it): noted at once instead of kept as a
          // pending alternative, so that a run through a rule that may end after every byte (the inside of
          // a string, a number) leaves nothing to come back to.  (BUILD = false: the end of the root rule.)
          if (BUILD && can_pop) {
            const uint32_t fo = T.follows(follow, c);
            left_frame |= 1u | (fo << 1);
            if (exits_out && fo) *exits_out |= 1u << (i < 31 ? i : 31);
          }
          can_pop = 0u;
        }
        // A return in front of a byte that can never follow the rule leads nowhere, or - if all frames below may end their
        // rules as well - out of the bottom frame in front of a byte that follows it in no context.
        if (can_pop && !T.follows(rule, c)) {
          can_pop = 0u;
          if (BUILD && !PRUNE) {
            if (sp != looked_at) {
              uint32_t h = sp;
              for (down = 1; h < kLiveBase && T.is_final(mem.frame(h) & 0xFFFFu); ++down) h = mem.frame(h) >> 16;
              if (h >= kLiveBase) left_frame |= 1u;
              looked_at = sp;
            }
            steps += down;
          }
        }
      }
      // nothing but a move along a byte edge (most steps inside a string, a number, a name): taken at once
      if (alt == 0u && !can_pop && !at.none && at.to < kAltFlagD) {
        n = at.to;
        f = 1;
        if (++i < len) c = token_byte(tw, ext, i);
        continue;
      }
      const bool pooled = !at.none && at.to >= kAltFlagD;
      const uint32_t base = at.to & ~kAltFlagD;
      uint32_t k = at.none ? 0u : 1u, run = 0u;  // (a run of calls counts as one)
      if (pooled) {
        k = T.alt(base);
        if (k & kRunFlagD) { run = k; k = 1; }
      }
      const uint32_t total = k + can_pop;
      if (alt < total) {
        if (alt + 1 < total) {
          if (csp == kChoicePoints) return kOverflow;
          mem.set_choice(csp++, make_uint2(n | (sp << 16), (uint32_t)i | ((alt + 1) << 8) | (top << 16) | (f << 24)));
          needed = top;
        }
        bool consumes = false;
        looked_at = 0xFFFFu;
        if (alt < k) {
          if (run) {  // several calls, one after the other
            const uint32_t m = run_frames(run);
            if (top + m > kArenaFrames) return kOverflow;
            for (uint32_t j = 0; j < m; ++j) {
              mem.set_frame(top, ((T.alt(run_frames_at(run) + (j >> 1)) >> ((j & 1u) * 16u)) & 0xFFFFu) | (sp << 16));
              sp = top++;
            }
            n = T.alt(base + 1);
            f = 0;
            consumes = (run & kRunConsumesD) != 0u;
          } else {
            const uint32_t e = pooled ? T.alt(base + 1 + alt) : (kMoveTagD << 16) | at.to;
            const uint32_t tag = e >> 16;
            n = e & 0xFFFFu;
            f = 0;
            if (tag == kMoveTagD) consumes = true;
            else if (tag != kTailTagD) {  // (a tail call: enter the callee, it returns to our parent)
              if (top == kArenaFrames) return kOverflow;
              mem.set_frame(top, tag | (sp << 16));
              sp = top++;
            }
          }
          if (consumes) {
            f = 1;
            if (++i < len) c = token_byte(tw, ext, i);
          }
        } else if (sp < kLiveBase) {   // return into a frame pushed during this walk
          const uint32_t fr = mem.frame(sp), old = sp;
          n = fr & 0xFFFFu;
          sp = fr >> 16;
          // frames from `old` upwards are garbage unless a pending alternative still needs them
          if (needed <= old) top = old;
        } else {                       // return into a live frame
          const uint32_t d = sp - kLiveBase;
          n = live[d - 1];
          sp = kLiveBase + d - 1;
        }
        alt = 0;
        continue;
      }
    }
    // back up to the most recent pending alternative
    if (csp == 0) break;
    looked_at = 0xFFFFu;
    const uint2 ch = mem.choice(--csp);
    n = ch.x & 0xFFFFu;
    sp = ch.x >> 16;
    i = (int)(ch.y & 0xFFu);
    alt = (ch.y >> 8) & 0xFFu;
    top = (ch.y >> 16) & 0xFFu;
    f = (ch.y >> 24) & 1u;
    c = token_byte(tw, ext, i);
    needed = csp ? (mem.choice(csp - 1).y >> 16) & 0xFFu : 0u;
  }
  if (BUILD && left_frame) return (left_frame & 2u) ? kUncertain : kUncertainPlain;
  return kReject;
}
template <bool BUILD, bool PRUNE = !BUILD, class Tab, class Live, class End = FirstPathEnds>
XGM_HD int walk_token(const Tab& T, const uint4 tk, const uint8_t* ext, const int len,
                      const uint32_t start_node, const Live& live, const uint32_t depth,
                      uint32_t* steps_out = nullptr, const uint32_t follow = 0u, const int i0 = 0,
                      uint32_t* exits_out = nullptr, const End& at_end = End()) {
  PrivateMem mem;
  return walk_token_in<BUILD, PRUNE>(mem, T, tk, ext, len, start_node, live, depth, steps_out, follow, i0, exits_out, at_end);
}

// End policy of the walk on the host that writes out the stack of every configuration a
// token can end in (section 3.3: the sampled token moves every parallel stack on; the accept
// kernel has one of its own, which notes only the frames above those a stack keeps).  A top
// node that can only return is returned from first, so that equal states get
// equal stacks.  A stack goes to the slot that `sink.claim()` hands out:
//   sink.frames  [capacity][max_depth] uint16, bottom frame first, the current node last
//   sink.depth   [capacity]
// A stack deeper than max_depth, or more stacks than capacity, set *sink.overflow.
// The same stack may be written more than once (several paths): the caller
// removes duplicates.
template <class Tab, class Sink>
struct CollectStacks {
  static constexpr bool kEnumerate = true;
  const Tab* T;
  Sink* sink;
  template <class Mem, class Live>
  XGM_HD void operator()(uint32_t n, uint32_t sp, const Mem& mem, const Live& live) const {
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
    uint32_t depth = 1, h = sp;
    for (; h < kLiveBase; h = mem.frame(h) >> 16) ++depth;
    const uint32_t d = h - kLiveBase;  // live frames kept
    depth += d;
    if (depth > sink->max_depth) { *sink->overflow = 1u; return; }
    const uint32_t idx = sink->claim();
    if (idx >= sink->capacity) { *sink->overflow = 1u; return; }
    auto* out = sink->frames + (size_t)idx * sink->max_depth;
    out[depth - 1] = (uint16_t)n;
    uint32_t k = depth - 1;
    for (h = sp; h < kLiveBase; h = mem.frame(h) >> 16) out[--k] = (uint16_t)(mem.frame(h) & 0xFFFFu);
    for (uint32_t j = 0; j < d; ++j) out[j] = (uint16_t)live[j];
    sink->depth[idx] = depth;
  }
};

}  // namespace xgm
