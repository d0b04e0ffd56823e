// Rules by which the host picks a kernel's shape for a graph and a batch: plain C++, so that they can
// be checked over all sizes without a GPU.
#pragma once

#include <stdint.h>

#include <algorithm>

#include "moc_slices.h"

// ------------------------------------------------------------------ moc_eval_batch_staged
constexpr int kStagedThreads = 512;

// The kernel that holds the copies of a lane's nodes in registers: threads per candidate and nodes a lane (1, 2 or 4:
// nt * nodes >= n).  nodes = 0: the kernel for any size, with kStagedThreads.
struct StagedShape {
  int nt, nodes;
};
// Two nodes a lane (four beyond 2048 nodes), so that no wave is idle in the passes that every wave takes part in.  C = 2,
// microseconds with 64 / 128 / 256 / 512 / 1024 threads (before, with 512 for
// every size): n = 50, 32000 candidates 20 / 30 / 53 / 103 / 202 (115); n = 100, 16384 candidates 17.5 / 19.5 / 30 / 55 / 106 (62);
// n = 200, 8192 candidates 18.8 / 17.8 / 20 / 30 / 55 (35); n = 442, 16384 candidates - / 57 / 58 / 68 / 112 (77); n = 700, 8192 candidates
// - / - / 50 / 52.5 / 64 (56); n = 1000, 16384 candidates - / - / 103 / 98.6 / 127 (105); n = 2000, 4096 candidates - / - / - / 69 / 60
// (85), 512 candidates 13.4 / 11.6 with 512 / 1024 (15.1).
// Up to three candidates to a compute unit wait for the longest lane, and up to 512 threads have one node each.  With two nodes /
// with one (before, with 512 threads for every size): C = 2, n = 100, 256 candidates 5.8 / 5.5 (5.3); n = 442, 256 candidates
// 6.3 / 5.5 (5.3), 768 candidates 7.0 / 6.2 (6.7), n = 200 6.3 / 5.3 (5.8), four to a unit 6.4 / 6.7 (6.7); C = 4, n = 442, every
// copy active, 256 candidates 23.2 / 14.7 (14.7), n = 700 23.9 / 18.9 (24.4), but few active, n = 1000 9.3 / 10.0 (9.4).
inline StagedShape staged_shape(int n, int C, int64_t B, int num_cu) {
  if (C > 4 || n > (C <= 2 ? 4096 : 2048)) return {kStagedThreads, 0};
  if (n > 2048) return {1024, 4};
  int nt = 64;
  while (2 * nt < n) nt *= 2;
  if (nt < n && nt < 512 && B <= 3 * (int64_t)num_cu) nt *= 2;
  return {nt, nt < n ? 2 : 1};
}
struct SfLayout {
  int cur_off, bucket_off, delta_off, red_off;   // word offsets; the copies' records at 0, one node more than the graph has
  int chunk;   // delta entries per thread (odd: conflict-free strided reads)
  int bytes;
};
inline SfLayout sf_layout(int n, int C, int nt) {
  const int T = n * C;
  SfLayout l;
  l.chunk = ((T + 1 + nt - 1) / nt) | 1;
  l.cur_off = T + C;                               // int32 [n]: per stage count, then end of the stage's bucket
  l.bucket_off = l.cur_off + n;                    // uint16 [T]: node places, stage by stage
  l.delta_off = l.bucket_off + (T + 1) / 2;        // int32 [nt * chunk]
  l.red_off = (l.delta_off + nt * l.chunk + 3) & ~3;
  l.bytes = 4 * (l.red_off + 16 + 4 * (nt / 64));
  return l;
}

// ------------------------------------------------------------------ moc_decode_batch
// The largest sizes the call takes: as many words as its first kernels kept in LDS, 2.5 per copy (C = 3:
// starts in four 16-bit entries per node).
inline bool decode_fits(int n, int C, int max_lds) {
  const int T = n * C, T_pad = (T + 4) & ~3, starts = C == 3 ? 2 * n + 2 : T_pad / 2;
  return 4 * (2 * T_pad + starts + 32) <= max_lds;
}

// The kernel for any C.
constexpr int kDecodeThreads = 512;
struct DcLayout {
  int T_pad;   // words in each of the two position arrays (>= T + 1, a multiple of 4); half as many hold the starts
  int bytes;
};
inline DcLayout dc_layout(int n, int C) {
  DcLayout l;
  l.T_pad = (n * C + 4) & ~3;
  l.bytes = 4 * (2 * l.T_pad + l.T_pad / 2 + 2 * (kDecodeThreads / 64) + 16);
  return l;
}

// The kernel for C <= 4.
constexpr int node_slots(int C) { return C <= 2 ? 4 : 2; }   // nodes of a lane (with more copies a lane's positions set the limit)
struct DfLayout {
  int T_pad;                       // > T + 1, a multiple of 8
  int pos_off, list_off, a_off;    // byte offsets; the starts lie at 0
  int told_off;                    // what the waves tell each other
  int bytes;
};
// loop: the running sums have no place of their own but lie in the entries of starts that the first wave writes,
// so that every size of decode_fits has this kernel (the other takes twice as long: n = 8170, C = 2, 1000
// candidates 211 us).
inline DfLayout df_layout(int n, int C, int nt, bool loop) {
  const int T = n * C, waves = nt / 64;
  DfLayout l;
  l.T_pad = (T + 9) & ~7;
  l.pos_off = (2 * starts_stride(C) * (n + 1) + 15) & ~15;
  l.list_off = l.pos_off + 2 * l.T_pad;
  l.a_off = l.list_off + 2 * l.T_pad;
  l.told_off = l.a_off + 4 * l.T_pad;
  l.bytes = l.told_off + 16 + waves * (loop ? 4 : 4 + 8);
  return l;
}

struct DecodeShape {
  int nt;
  bool loop;   // more nodes or positions than a workgroup of 1024 takes at once: in rounds
  DfLayout lay;
};
// As few threads as hold the candidate: a workgroup's waves meet at three barriers per candidate, and
// lanes without a node still take their part of every pass.  By 64 / 128 / 256 / 512 / 1024 threads
// (before: 512 for every size): n = 100, C = 2, 16384 candidates 17.6 / 24.3 / 39.8 / 71.4 / 137 us
// (before 72.1); n = 442, 4096 candidates - / 14.5 / 17.7 / 26.5 / 46.2 (29.8); n = 1000, 4096
// candidates - / - / 24.9 / 31.0 / 49.6 (44.1); n = 2500, 2000 candidates: 1024 threads 35.0 (44.1).  A batch of one
// candidate to a compute unit or less waits for the longest walk of a wave, and gets as many threads as it has nodes: 30
// consumers a node, n = 454, up to 256 candidates 13.5 us with as few as hold it, 8.8 with these (9.1), and as long as the
// launch where nodes have few consumers either way; with two candidates to a compute unit 14.8 and 9.8 (12.6), but
// training graph, n = 1000, 8.7 and 9.9.
// In rounds: n = 4500, C = 2, 2000 candidates 80 us (127); n = 7000, 1000 candidates 64 (95); n = 2500, C = 3,
// 2000 candidates 61 (79); n = 16340, C = 1, 1000 candidates 106 (157).
inline DecodeShape decode_shape(int n, int C, int64_t B = INT64_MAX, int num_cu = 1) {
  int nt = 64;
  const auto holds = [&](int t) { return n <= node_slots(C) * t && df_layout(n, C, t, false).T_pad <= 8 * t; };
  while (nt < 1024 && !holds(nt)) nt *= 2;
  const bool loop = !holds(nt);
  if (B <= num_cu)
    while (nt < 1024 && nt < n) nt *= 2;
  return DecodeShape{nt, loop, df_layout(n, C, nt, loop)};
}

// ------------------------------------------------------------------ a base in LDS (moc_moves.h)
constexpr int kBlk = 8;   // positions per block of the profile's range maxima (two 16-byte reads)

// Word offsets.  The profile begins at 0; `table` holds, at level l and index i <= blocks - 2^l, the
// maximum over the blocks i .. i + 2^l - 1, level behind level (table_level); pre[i] the maximum
// over the blocks before i, suf[i] over the blocks from i on.
constexpr int table_level(int level, int blocks) { return level * (blocks + 1) - (1 << level) + 1; }
struct MvLayout {
  int blocks, levels, bit_words;
  int table, pre, suf, packed, occ1, occ2, peak_bits, peak_before, scratch, extra;
  int lists;   // adjacency lists in LDS, 0 if they are read from global memory
  int bytes;
};

constexpr int kScratchWords = 160;

// extra_words: what the kernel needs beyond the base.  with_lists: the adjacency lists too, if they fit.
inline MvLayout mv_layout(int T, int n, int m, int extra_words, bool with_lists, int max_lds) {
  MvLayout l;
  l.blocks = (T + kBlk - 1) / kBlk;
  l.levels = 1;
  while ((2 << (l.levels - 1)) <= l.blocks) ++l.levels;
  l.bit_words = 2 * ((T + 63) / 64);
  l.table = l.blocks * kBlk;
  l.pre = l.table + table_level(l.levels, l.blocks);
  l.suf = l.pre + l.blocks + 1;
  l.packed = (l.suf + l.blocks + 1 + 3) & ~3;
  l.occ1 = l.packed + ((T + 3) & ~3);
  l.occ2 = l.occ1 + l.bit_words;
  l.peak_bits = l.occ2 + l.bit_words;
  l.peak_before = l.peak_bits + l.bit_words;
  l.scratch = l.peak_before + l.bit_words;
  l.extra = (l.scratch + kScratchWords + 3) & ~3;
  const int words = l.extra + extra_words;
  l.lists = 0;
  l.bytes = 4 * words;
  // sizes and edge pairs as words, the rest in 16 bits (which is why m is bounded)
  const int lists = n + m + (2 * (n + 1) + m + 1) / 2;
  if (with_lists && m < 0xFFFF && 4 * (words + lists) <= max_lds) {
    l.lists = words;
    l.bytes = 4 * (words + lists);
  }
  return l;
}

// The largest T the calls on moves take: as many words per copy as their first kernels kept in LDS
// (4.4 per copy, 4 per 32 copies, and what a workgroup of 16 waves needs).
inline bool moves_fit(int T, int max_lds) {
  const int blocks = (T + 31) / 32;
  int levels = 1;
  while ((2 << (levels - 1)) <= blocks) ++levels;
  const int words = 4 * ((T + 3) & ~3) + 8 + levels * blocks + 4 * blocks + 8 * 16 + 16 + 2 * 64 * 16;
  return 4 * words <= max_lds;
}

// ------------------------------------------------------------------ the best single-field move (moc_best_moves.h)
// The largest T the calls on single-field moves take: what the table's kernel keeps in LDS with 1024 threads.
inline bool neighbours_fit(int T, int max_lds) {
  const int T_pad = (T + 3) & ~3, bits = (T + 31) / 32, masks = 2 * ((T + 63) / 64);
  return 4 * (4 * T_pad + T_pad / 2 + 8 + 2 * bits + 2 * masks + 8 * 16 + 16) <= max_lds;
}

// Word offsets; the profile at 0.
struct BmLayout {
  MvLayout base;   // what the staging of a base needs of it
  int counts, red, queue;
  int cap;         // fields that wait for their scoring, at most
  int bytes;
};
constexpr int kBmCounts = 16;
inline BmLayout bm_layout(int T, int nt) {
  BmLayout l{};
  MvLayout& b = l.base;
  b.blocks = (T + kBlk - 1) / kBlk;
  b.levels = 1;
  b.bit_words = 2 * ((T + 63) / 64);
  b.table = b.blocks * kBlk;
  b.pre = b.table + b.blocks;
  b.suf = b.pre + b.blocks + 1;
  b.packed = (b.suf + b.blocks + 1 + 3) & ~3;
  b.occ1 = b.packed + ((T + 3) & ~3);
  b.occ2 = b.occ1 + b.bit_words;
  b.peak_bits = b.peak_before = b.occ2;   // not used
  b.scratch = b.occ2 + b.bit_words;
  b.extra = l.counts = (b.scratch + kScratchWords + 3) & ~3;
  l.red = l.counts + kBmCounts;
  l.queue = l.red + T;
  l.cap = 2 * nt;
  l.bytes = 4 * (l.queue + l.cap / 2);
  return l;
}

// Threads per base: a chain of short passes, which more waves shorten as long as a base feeds them and the bases
// of a compute unit do not compete.  C = 2, R = 8, microseconds by 256 / 512 / 1024 threads
// (before, with every field that could win scored: 256 to 1024 threads): n = 50, 1024 bases 18 / 26 / 49 (27); n = 442, 16 bases
// 16.0 / 14.5 / 14.7 (25), 512 bases 19.4 / 17.5 / 26.1 (30), 1024 bases 20.2 / 26.7 / 47.4 (43), 4096 bases, R = 4 49 / 73 / 178 (114); n =
// 1000, 300 bases - / 18.5 / 28.0 (48), 1024 bases - / 33.7 / 53.2 (72); n = 2000, 512 bases - / 27.9 / 37.4 (70).  C = 3: n = 300, 300
// bases 17.0 / 15.4 / 23.9 (32), 1024 bases 19.2 / 27.9 / 45.0 (42); n = 600, 100 bases - / 17.6 / 16.3 (32); n = 2500, 100 bases - / 37.1 /
// 28.5 (84), 600 bases - / 109 / 81 (223).  C = 4: n = 250, 300 bases 17.2 / 15.8 / 25.5 (40), 1024 bases 22.7 / 32.2 / 50.6 (57); n =
// 1200, 300 bases - / 35.4 / 45.9 (87); n = 1500, 300 bases, two of which fit no compute unit, - / 63.7 / 52.2 (101).
inline int best_threads(int T, int64_t B, int num_cu, int max_lds) {
  const int64_t share = (B + num_cu - 1) / num_cu;
  if (T <= 1024 && (share > 2 || T <= 256)) return 256;
  if (T <= 2048) return 512;
  // two workgroups of 1024 do not fit a compute unit (80 to 92 registers a thread)
  return share > 1 && T <= 5000 && 2 * bm_layout(T, 512).bytes <= max_lds ? 512 : 1024;
}

// ------------------------------------------------------------------ the descent by cuts (moc_search.hip)
constexpr int kMaxRanges = 65;   // stretches of the profile that are changed together: one per lane and the producer's
constexpr int kCutWords = 6;     // of the chosen move
constexpr int kBuckets = 64;     // of the sieve's histogram of bounds

// Words of LDS beyond the base: a queue of two moves per lane, the stretches, the chosen move.
constexpr int descend_words(int nt) { return (2 * nt + 3 * kMaxRanges + 1 + kCutWords + 1) & ~1; }
// ... and the lists of `cap` moves that pass the sieve.
inline int sift_words(int /*n*/, int cap) { return 3 * cap + cap / 2 + kBuckets + 4; }

struct DescendShape {
  int nt;    // threads per candidate
  int cap;   // moves that pass the sieve, at most
  MvLayout lay;
};

// As many threads per candidate as the candidates that share a compute unit leave room for (a
// thread takes about 96 registers): a step is a chain of short phases, which more waves shorten,
// but a wave with nothing to do in a phase still takes its part of the barriers and the issue
// slots.  C = 2, 32 steps, microseconds with 256 / 512 / 1024 threads: keeping cuts, n = 442, 1024 walkers 539 /
// 850 / 1556, 512 walkers 465 / 437 / 798, 256 walkers 434 / 390 / 413, 32 walkers 423 / 386 / 405; n = 1000, 1024
// walkers 1471 / 1137 / 1859, 32 walkers 693 / 495 / 484; plain cuts, n = 442, 1024 walkers 519 / 851 / 1501, 512
// walkers 454 / 443 / 766, 256 walkers 423 / 399 / 400; n = 1000, 512 walkers 709 / 556 / 1012, 32 walkers 631 / 462
// / 501, training graph 385 / 292 / 276.  (With one walker to a compute unit neither 512 nor 1024 is the better
// one throughout.)  Without the adjacency lists in LDS: 1024.
inline DescendShape descend_shape(int T, int n, int m, int64_t B, int num_cu, int max_lds) {
  const auto layout = [&](int nt, int cap) { return mv_layout(T, n, m, descend_words(nt) + sift_words(n, cap), true, max_lds); };
  const int64_t share = (B + num_cu - 1) / num_cu;
  const int by_lds = max_lds / layout(256, 256).bytes;
  const int nt = !layout(1024, 256).lists || share <= 1 || by_lds <= 1 ? 1024 : share <= 2 || by_lds <= 2 ? 512 : 256;
  // The lists of moves that pass the sieve: as long as costs neither a resident workgroup nor, down to
  // 512, the adjacency lists their place in LDS (32 walkers, 32 plain cuts, with 2048 and without the
  // adjacency lists / with them and what then fits: n = 2500, C = 2 647 / 618 us, 512 walkers 1313 / 1251;
  // n = 3000, training graph, and n = 2790 the same either way).  A list that overflows
  // costs the scoring of every move, a resident workgroup mostly more: 1024 walkers, 32 plain cuts,
  // C = 2, 256 and one more workgroup / 512: n = 590 869 / 1120 us, n = 1320 1294 / 2081, n = 850
  // 1498 / 1422, n = 1400, where most steps overflow, 2379 / 1971.
  const int want = (int)std::min<int64_t>({share, by_lds, 1024 / nt});
  int cap = 2048;
  while (cap > 256 && (layout(nt, cap).bytes * std::max(want, 1) > max_lds || (!layout(nt, cap).lists && layout(nt, 512).lists))) cap /= 2;
  return DescendShape{nt, cap, layout(nt, cap)};
}
