// Kernel-side shared structures and launcher declarations.
#pragma once
#include "blb_internal.h"

// Per-poly descriptor for batched transforms.  Fields beyond src/dst/mod are used by the
// fused prologue / epilogue variants (rescale, ModDown).
struct PolyDesc {
  const uint64_t* src;
  uint64_t* dst;
  const uint64_t* src2;
  const uint64_t* src3;
  union {
    double aux;         // prologue constant (e.g. the modulus whose residues are lifted)
    const double* cst;  // base-conversion prologue: [Q_D / q_i] mod this modulus, one per source limb
  };
  double aux2;  // epilogue constant (e.g. q_l^-1 or P^-1 mod this modulus); inverse transforms: the
                // scale that takes N^-1's place (0: N^-1)
  int16_t mod;  // modulus index of this poly
  int16_t n_src;  // base-conversion prologue: source limbs, stored back to back from src
  uint32_t gal; // Galois element applied to src3 (0 = none)
  int32_t log_n;
  int32_t flags;  // kAddBoth: src3 is added as it is too, not only under the Galois element
};
constexpr int32_t kAddBoth = 1;
constexpr int32_t kUpperHalf = 2;  // set in a workgroup's own copy: it holds the polynomial's upper half

// Bit-reversal of j over log_n bits
__device__ __forceinline__ uint32_t brv_bits(uint32_t j, int log_n) { return __brev(j) >> (32 - log_n); }

// Evaluation-form automorphism: value j of sigma_g(x) is value perm(j) of x, where slot j
// holds the evaluation at psi^(2 brv(j) + 1).
__device__ __forceinline__ uint32_t gal_perm(uint32_t j, uint32_t g, int log_n) {
  const uint32_t two_n_mask = (2u << log_n) - 1u;
  const uint32_t r = 2u * brv_bits(j, log_n) + 1u;
  const uint32_t rg = (r * g) & two_n_mask;  // g < 2N, r < 2N: product < 2^30 for N <= 2^14
  return brv_bits((rg - 1u) >> 1, log_n);
}

void launch_ntt(blb_ctx* c, const PolyDesc* d_descs, int count, bool fwd);
void launch_ntt_rescale(blb_ctx* c, const PolyDesc* d_descs, int count);
void launch_intt_masked(blb_ctx* c, const PolyDesc* d_descs, int count);
void launch_ntt_rescale_masked(blb_ctx* c, const PolyDesc* d_descs, int count, int level, const double* inv);
// Descriptors that share their sources stand in a row: runs of `group` among the first `split`, of `tail` after them.
struct NttRuns {
  int group, split, tail;
};
// ModUp: source limbs of a digit (y_i = [d_i Qhat_i^-1]_{q_i}, coefficient form) -> evaluation form of
// their base conversion; n_src <= most.  A run is a digit of a source; the digits of fewer limbs come last.
void launch_ntt_modup(blb_ctx* c, const PolyDesc* d_descs, int count, int most, NttRuns runs);
// ModDown: special limbs (y_t = [u_t Phat_t^-1]_{p_t}, coefficient form) -> (u_i - conversion) P^-1 + addend
void launch_ntt_moddown(blb_ctx* c, const PolyDesc* d_descs, int count, int most, NttRuns runs);
void launch_ntt_addto(blb_ctx* c, const PolyDesc* d_descs, int count);
// in-place transform of `count` limb-polys stored back to back at base ([item][nl][N]), no
// descriptor table
void launch_ntt_regular(blb_ctx* c, uint64_t* base, int count, int nl, bool fwd);
