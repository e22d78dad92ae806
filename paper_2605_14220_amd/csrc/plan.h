// Launch shapes chosen from sizes and the device's compute units alone. Pure
// C++: no HIP calls, so the choices can be checked without a GPU. None of them
// changes a result.
#pragma once

#include <cstdint>

namespace tim {

constexpr int kChains = 256;  // partial sums per response, one thread each

// Blocks of 256 threads per response in the sequence scores and the PPO loss,
// one or four, by the tokens a response has on average. Four shorten a
// response's chain of terms but pass them through LDS between barriers, and a
// CU holds two such workgroups against eight: they pay where each response has
// a CU to itself and some length, up to two responses per CU only for long
// ones, and beyond that never (2048 responses of 513 tokens: 6.7 us on one
// block, 17.7 on four; 2000 of 4000: 26 and 33 us).
//   K3 scores, up to one response per CU, 1600 tokens: 4.3 us rejected and 5.4
//     kept on one block, 4.3 and 4.9 on four (1300: 4.0 and 4.7 against 4.2
//     and 4.7; 16384: 30 and 40 against 17 and 22). Two per CU, 4096 tokens:
//     7.2 and 9.8 against 7.5 and 9.7; 6000: 11.4 and 14.6 against 9.4 and 12.5.
//   K1 scores, whose terms are no exponentials: 3072 tokens 4.9 and 6.4 against
//     5.0 and 6.2, 2048: 4.1 and 5.1 against 4.5 and 5.2; two per CU, 6000
//     tokens 7.6 and 11.3 against 7.9 and 11.0.
//   PPO: 1600 tokens 7.6 us against 6.9, 1300 equal, 1024 6.2 against 6.5; two
//     per CU, 16384 tokens 47 against 38-48, 8192 25.9 against 25.9.
enum class ResponseTerm { kK1, kK3, kPpo };
inline int response_blocks(ResponseTerm term, int64_t T, int64_t n_seq, int64_t cus) {
  const int64_t blocks = T / n_seq / kChains;  // whole blocks of 256 tokens
  const bool k1 = term == ResponseTerm::kK1, k3 = term == ResponseTerm::kK3;
  if (n_seq <= cus) return blocks >= (k1 ? 12 : k3 ? 6 : 5) ? 4 : 1;
  if (n_seq <= 2 * cus) return blocks >= (k1 ? 28 : k3 ? 20 : 32) ? 4 : 1;
  return 1;
}

// Decode batches of at most 64 rows over half vocabulary tiles: a wave per half
// with a ring of its own (lmhead_half_stream), for `row_blocks` blocks of 16
// rows (1, 2 or 4), walking its half in groups of `group` W blocks of 16
// entries; or row_blocks = 0 for 64-row tiles of two waves (lmhead_half_partials).
//
// The lone wave does a stage's MFMAs, waits and requests by itself, so it is
// the slower of the two until the stream of W is what bounds the call: with few
// halves per CU it takes the more of them the more rows there are. Calls
// against the two-wave tiles, d = 2560..7168, by halves per CU:
//   up to 16 rows  1.2-1.35 x at 0.06, 0.93-0.96 at 0.25, 0.87-0.93 at 0.5
//   17..32 rows    1.3-1.5 at 0.06, 1.0-1.04 at 0.25, 0.93-0.97 at 0.5
//   33..64 rows    1.6-1.85 at 0.06, 1.1-1.15 at 0.5, 1.0-1.05 at 0.73, 0.85-0.94 at 1
// sooner where W does not stay in the 256 MB memory-side cache from call to
// call (0.77-0.91 at 0.37..0.9 for 295 MB and more). A shorter d moves the
// lines of up to 32 rows: d = 1024 1.02-1.04 and 1.13-1.17 at 0.25, 0.93 and
// 1.02 at 0.5; up to 512 (256 for 17..32 rows) the wave is not slower. Above
// one half per CU the CUs with one more set the time: 33..64 rows stay on the
// two-wave tiles up to two (V = 50257 at d = 4096 100 us against 95), at d <=
// 1024 up to three (1.05-1.1 x), as do fewer rows there up to two. Beyond:
// 0.88-1.0, up to 1.05 just above two.
//
// All the waves start at the same place of their rows, so rows a power of two
// apart meet on the same memory channels; walking fewer W blocks at a time
// spreads them, at the price of reading the hidden block once per group, and
// only helps where the stream is what bounds (V = 32000 at d = 4096, 32 rows:
// 0.83 x by 8 blocks, 1.37 by 4). A bare stream of W at d = 2048 takes 144 us
// by 8, 130 by 4, 118 by 2; at d = 4096 222 and 211 by 8 and 4; at other widths
// the orders are within 3%. Calls against the two-wave tiles, by groups of 8 / 4 / 2:
//   d = 2048, up to 16 rows  V = 57000 0.98 / 1.2 / 1.2, 72000 0.98 / 0.97 / 1.03, 98304 1.01 / 0.97 / 0.87,
//                            151936 1.07 / 1.02 / 0.92
//             17..32 rows    V = 57000 1.0 / 1.15 / 1.1, 90000 1.01 / 1.08 / 1.03, 151936 1.08 / 0.95 / 1.0,
//                            180000 1.15 / 1.05 / 1.04
//             33..64 rows    V = 32000 0.9, 50257 1.0, 151936 1.06 by 8; more by less
//   d = 4096, up to 16 rows  V = 40000 0.9 / 0.85 / 0.84, 98304 0.97 / 0.9 / 0.88, 151936 1.0 / 0.99 / 1.03
//             17..32 rows    V = 50257 0.98 / 1.04 / 1.07, 65536 1.05 / 0.93 / 0.89, 151936 1.0 / 0.98 / 1.15,
//                            165000 1.04 / 1.07 / 1.07
//             33..64 rows    V = 80000 1.08, 151936 0.98, 165000 1.01, 196608 1.03 by 8; more by less
// d = 1024 gains nothing up to three halves per CU (1.0-1.04), multiples of
// 2048 but 2048 itself nothing above five (d = 6144 1.03-1.06, 10240
// 1.02-1.06). Multiples of 8192 lose with any group above one (d = 8192 up to
// 1.25 x, d = 16384 1.3 x; at best 0.92 at some V), and up to 16 rows take
// groups of 4 near one (V = 32000: d = 8192 0.93 against 1.08 by 8).
struct StreamShape {
  int row_blocks, group;
};
constexpr int kStreamPerCU = 6;  // 24 KB of LDS each
inline StreamShape stream_shape(int64_t rows, int32_t d, int n_ht, int cus) {
  constexpr StreamShape kTiles{0, 0};
  if (cus <= 0 || rows > 64 || n_ht > kStreamPerCU * cus) return kTiles;
  const int nb = rows <= 16 ? 1 : rows <= 32 ? 2 : 4;
  if (n_ht <= cus) {
    const bool uncached = (int64_t)n_ht * 256 * d > 280000000;  // bytes of W
    const int least = nb == 1   ? (d <= 512 ? 0 : d < 2048 ? 45 : 22)  // percent of the CUs with a half
                      : nb == 2 ? (d <= 256 ? 0 : d < 1024 ? 90 : d < 1536 ? 70 : 45)
                                : (d < 1024 ? 101 : 90);
    if (!uncached && 100 * n_ht < least * cus) return kTiles;
    return StreamShape{nb, nb == 1 && d % 8192 == 0 && 4 * n_ht > 3 * cus ? 4 : 8};
  }
  if (d % 8192 == 0 || (d % 2048 == 0 && d > 2048 && n_ht > 5 * cus)) return kTiles;
  if (n_ht <= 2 * cus && (nb == 4 || d <= 1024)) return kTiles;
  if (n_ht <= 3 * cus && (d == 1024 || (nb == 4 && d < 1024))) return kTiles;
  if (d != 2048 && d != 4096) return StreamShape{nb, 8};
  if (nb == 1) return StreamShape{1, d == 4096 ? 4 : 4 * n_ht <= 9 * cus ? 8 : 2};
  if (nb == 2 && n_ht < 2 * cus) return StreamShape{2, 8};
  // the groups' second and later reads of the hidden block weigh more the more rows there are
  if (n_ht > 5 * cus || (d == 2048 && (nb == 4 || n_ht <= 4 * cus)) || (nb == 4 && n_ht <= 3 * cus)) return kTiles;
  return StreamShape{nb, nb == 2 ? 4 : 8};
}

// Norm backward at d = 2048 and 4096 with grad_gamma by quarters of 256-row
// blocks: whether the blocks' sums are taken in the grad_x pass, a workgroup per
// block. A 256-CU MI355X holds norm_resident of them at once (two per CU at
// d = 4096, four at 2048) but their time is that of the CUs with the most, so
// the pass is the faster one where the CUs' last blocks are nearly all there,
// from 0.8 of them. Against grad_x and the sums over the same rows in one
// launch, both outputs, us:
//   d = 4096  65536 rows (256 blocks) 543 and 596, 72000 832 and 662, 90000 909 and 818, 105000 (410 of 512) 956 and
//             954, 110000 976 and 997, 131071 1101 and 1185
//   d = 2048  65536 278 and 312, 90000 470 and 424, 105000 486 and 497, 131072 554 and 615, 140000 704 and 657, 160000
//             (625 of 768) 755 and 751, 196608 841 and 917, 210000 (821 of 1024) 1002 and 985, 250000 1080 and 1164
// (grad_gamma alone crosses at the same places). From 256 rows per resident
// block on, the blocks take more rows and always fill the chip.
inline int64_t norm_resident(int32_t d) { return d == 2048 ? 1024 : 512; }
inline bool norm_fused(int64_t T, int32_t d) {
  constexpr int64_t kCUs = 256;
  if (T >= 256 * norm_resident(d)) return true;
  const int64_t blocks = (T + 255) / 256, rounds = (blocks + kCUs - 1) / kCUs;
  return 10 * blocks >= 8 * rounds * kCUs;
}

}  // namespace tim
