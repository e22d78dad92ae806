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

}  // namespace tim
