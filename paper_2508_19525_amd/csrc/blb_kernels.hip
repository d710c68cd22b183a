// Elementwise, sampling, key-switching, matmul_cp and encoder kernels for gfx950.
// All modular arithmetic is the FP64 signed-lazy scheme of blb_internal.h.
#include "blb_internal.h"
#include "blb_kernels.h"
#include <algorithm>
#include <type_traits>

// ---------------------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): 10 rounds, multipliers 0xD2511F53 / 0xCD9E8D57,
// key schedule increments 0x9E3779B9 / 0xBB67AE85.  Counter = (coefficient, limb, object,
// tag), key = (seed low word, seed high word).
// ---------------------------------------------------------------------------------------
struct U4 { uint32_t x, y, z, w; };
__device__ __forceinline__ U4 philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t lo0 = 0xD2511F53u * c0, hi0 = __umulhi(0xD2511F53u, c0);
    const uint32_t lo1 = 0xCD9E8D57u * c2, hi1 = __umulhi(0xCD9E8D57u, c2);
    const uint32_t n0 = hi1 ^ c1 ^ k0;
    const uint32_t n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
    k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
  }
  return U4{c0, c1, c2, c3};
}
#define LIMB_INTEGER 0xFFFFFFFFu

// (w3 2^96 + w2 2^64 + w1 2^32 + w0) mod q by Horner steps r <- r*2^32 + w (mod q) on FP64
__device__ __forceinline__ double u128_mod(U4 w, double q, double qi) {
  const double two32 = 4294967296.0;
  double r = (double)w.w;  // < 2^32 < q
  r = canon_full(mulmod_s(r, two32, q, qi) + (double)w.z, q, qi);
  r = canon_full(mulmod_s(r, two32, q, qi) + (double)w.y, q, qi);
  r = canon_full(mulmod_s(r, two32, q, qi) + (double)w.x, q, qi);
  return r;
}

// out[limb][k] = uniform residue mod the limb's modulus; limb counter = mod index
__global__ void k_sample_uniform(uint64_t* out, int n, ModMap map, ModTable mt, uint32_t k0, uint32_t k1, uint32_t obj, uint32_t tag) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const int limb = blockIdx.y;
  if (k >= n) return;
  const int m = map.idx[limb % map.len];
  const U4 w = philox10((uint32_t)k, (uint32_t)m, obj, tag, k0, k1);
  out[(size_t)limb * n + k] = d2u(u128_mod(w, mt.m[m].q, mt.m[m].qinv));
}

// integer samples reduced into every limb of the map.  mode 0: ternary (w0 mod 3) - 1;
// mode 1: Gaussian (CDT); mode F in [32, 48]: uniform integer in [-2^F, 2^F] (the 128-bit
// block mod 2^(F+1) + 1, minus 2^F; |v| <= 2^48 stays below every modulus)
__constant__ uint64_t c_cdt[20];
__global__ void k_sample_int(uint64_t* out, int n, int n_limbs, ModMap map, ModTable mt, uint32_t k0, uint32_t k1, uint32_t obj,
                             uint32_t tag, int mode) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const U4 w = philox10((uint32_t)k, LIMB_INTEGER, obj, tag, k0, k1);
  double v;
  if (mode == 1) {
    const uint64_t r = ((((uint64_t)w.y) << 32) | w.x) >> 1;
    int x = 0;
    while (x < 19 && r >= c_cdt[x]) ++x;
    v = (w.z & 1u) ? -x : x;
  } else if (mode == 0) {
    v = (double)((int)(w.x % 3u) - 1);
  } else {
    const double m = (double)((2ull << mode) + 1ull);
    v = u128_mod(w, m, 1.0 / m) - (double)(1ull << mode);
  }
  for (int l = 0; l < n_limbs; ++l) {
    const double q = mt.m[map.idx[l % map.len]].q;
    out[(size_t)l * n + k] = d2u(v < 0 ? q + v : v);
  }
}

void upload_cdt(const uint64_t* table20) { (void)hipMemcpyToSymbol(HIP_SYMBOL(c_cdt), table20, 20 * sizeof(uint64_t)); }

void launch_sample_uniform(blb_ctx* c, uint64_t* out, int n_limbs, ModMap map, uint64_t seed, uint32_t obj, uint32_t tag) {
  dim3 grid((c->n + 255) / 256, n_limbs);
  emit(c, [=, stream = c->stream] { k_sample_uniform<<<grid, 256, 0, stream>>>(out, c->n, map, c->mt, (uint32_t)seed, (uint32_t)(seed >> 32), obj, tag); });
}
void launch_sample_int(blb_ctx* c, uint64_t* out, int n_limbs, ModMap map, uint64_t seed, uint32_t obj, uint32_t tag, bool gaussian) {
  emit(c, [=, stream = c->stream] {
    k_sample_int<<<(c->n + 255) / 256, 256, 0, stream>>>(out, c->n, n_limbs, map, c->mt, (uint32_t)seed, (uint32_t)(seed >> 32), obj, tag,
                                                    gaussian ? 1 : 0);
  });
}
void launch_sample_flood(blb_ctx* c, uint64_t* out, int n_limbs, ModMap map, uint64_t seed, uint32_t obj, uint32_t tag, int bits) {
  emit(c, [=, stream = c->stream] {
    k_sample_int<<<(c->n + 255) / 256, 256, 0, stream>>>(out, c->n, n_limbs, map, c->mt, (uint32_t)seed, (uint32_t)(seed >> 32), obj, tag, bits);
  });
}

// ---------------------------------------------------------------------------------------
// Elementwise ops over [count][N] u64 arrays (evaluation or coefficient form alike)
// ---------------------------------------------------------------------------------------
__global__ void k_ew(int op, uint64_t* out, const uint64_t* a, const uint64_t* b, const uint64_t* cc, int n, ModMap map, ModTable mt) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const int p = blockIdx.y;
  if (k >= n) return;
  const ModEntry me = mt.m[map.idx[p % map.len]];
  const size_t o = (size_t)p * n + k;
  const double x = u2d(a[o]);
  double r;
  switch (op) {
    case EW_ADD: { r = x + u2d(b[o]); r = r >= me.q ? r - me.q : r; break; }
    case EW_SUB: { r = x - u2d(b[o]); r = r < 0 ? r + me.q : r; break; }
    case EW_MUL: { r = canon(mulmod_s(x, u2d(b[o]), me.q, me.qinv), me.q); break; }
    case EW_NEG: { r = x == 0.0 ? 0.0 : me.q - x; break; }
    case EW_MULADD: { r = mulmod_s(x, u2d(b[o]), me.q, me.qinv) + u2d(cc[o]); r = canon_full(r, me.q, me.qinv); break; }
    default: { r = x; break; }
  }
  out[o] = d2u(r);
}
void launch_ew(blb_ctx* c, int op, uint64_t* out, const uint64_t* a, const uint64_t* b, const uint64_t* cc, int count, ModMap map) {
  if (count <= 0) return;
  dim3 grid((c->n + 255) / 256, count);
  emit(c, [=, stream = c->stream] { k_ew<<<grid, 256, 0, stream>>>(op, out, a, b, cc, c->n, map, c->mt); });
}

// encryption / key combination in evaluation form:
//   out0 = -a*s + e + extra     (extra optional: plaintext or P*s' term, added modularly)
__global__ void k_rlwe_combine(uint64_t* out0, const uint64_t* a, const uint64_t* s, const uint64_t* e, const uint64_t* extra,
                               LimbVals extra_mul, int n, ModMap map, ModTable mt) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const int l = blockIdx.y;
  if (k >= n) return;
  const ModEntry me = mt.m[map.idx[l % map.len]];
  const size_t o = (size_t)l * n + k;
  double r = u2d(e[o]) - mulmod_s(u2d(a[o]), u2d(s[o]), me.q, me.qinv);  // (-q, 2q)
  if (extra) {
    double x = u2d(extra[o]);
    if (extra_mul.use) x = mulmod_s(x, extra_mul.v[l], me.q, me.qinv);
    r += x;
  }
  out0[o] = d2u(canon_full(r, me.q, me.qinv));
}
void launch_rlwe_combine(blb_ctx* c, uint64_t* out0, const uint64_t* a, const uint64_t* s, const uint64_t* e, const uint64_t* extra,
                         LimbVals extra_mul, int n_limbs, ModMap map) {
  dim3 grid((c->n + 255) / 256, n_limbs);
  emit(c, [=, stream = c->stream] { k_rlwe_combine<<<grid, 256, 0, stream>>>(out0, a, s, e, extra, extra_mul, c->n, map, c->mt); });
}

// evaluation-form automorphism of `count` polys
__global__ void k_automorph(uint64_t* out, const uint64_t* in, int n, int log_n, uint32_t g) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const int p = blockIdx.y;
  if (k >= n) return;
  out[(size_t)p * n + k] = in[(size_t)p * n + gal_perm((uint32_t)k, g, log_n)];
}
void launch_automorph(blb_ctx* c, uint64_t* out, const uint64_t* in, int count, uint32_t g) {
  dim3 grid((c->n + 255) / 256, count);
  emit(c, [=, stream = c->stream] { k_automorph<<<grid, 256, 0, stream>>>(out, in, c->n, c->log_n, g); });
}

// ---------------------------------------------------------------------------------------
// Key switching
// ---------------------------------------------------------------------------------------
// Operands reached through descriptors in memory are addressed as global memory explicitly
// (global, not flat, loads and stores: a flat access also counts against the LDS / scalar wait
// counter and takes a 64-bit vector address).
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T* gmem(T* p) {
  return (__attribute__((address_space(1))) T*)p;
}

// Inner product with the switching key, with the automorphism applied to the extended
// digits (hoisted order).  Thread per (o, e, two adjacent k); writes U[o][2][e][k] (evaluation
// form).  For one wave the permuted reads stay inside one aligned block of 64 words: sigma_g
// keeps the low log2(N) - 6 bits of the exponent index, which bit reversal maps to the high
// bits of k.  For the same reason an aligned pair of words stays a pair: one load, swapped or not.
typedef uint64_t u64pair __attribute__((ext_vector_type(2), aligned(8)));  // ciphertexts are 8-byte aligned
__device__ __forceinline__ u64pair ld_pair(const uint64_t* p) { return *(const __attribute__((address_space(1))) u64pair*)p; }
__device__ __forceinline__ void st_pair(uint64_t* p, double a, double b) {
  *(__attribute__((address_space(1))) u64pair*)p = u64pair{d2u(a), d2u(b)};
}
struct KsPair {  // where words k0, k0 + 1 (k0 even) come from under the Galois element
  uint32_t at;
  bool swap;
  __device__ KsPair(uint32_t k0, uint32_t gal, int log_n) {
    const uint32_t kk = gal ? gal_perm(k0, gal, log_n) : k0;
    at = kk & ~1u;
    swap = kk & 1;
  }
};
__device__ __forceinline__ const uint64_t* ks_digit(const KsOut& od, const uint64_t* X, const KsLevelConst* kc, int j, int e, int n_digits, int n_ext,
                                                    int n) {
  return e >= kc->dlo[j] && e < kc->dhi[j] ? od.c1 + (size_t)e * n : X + (((size_t)od.src * n_digits + j) * n_ext + e) * n;
}
__device__ __forceinline__ void ks_madd(double (&acc0)[2], double (&acc1)[2], u64pair w, bool swap, u64pair kb, u64pair ka, const ModEntry& mm) {
  const double x[2] = {u2d(swap ? w[1] : w[0]), u2d(swap ? w[0] : w[1])};
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    acc0[v] += mulmod_s(x[v], u2d(kb[v]), mm.q, mm.qinv);
    acc1[v] += mulmod_s(x[v], u2d(ka[v]), mm.q, mm.qinv);
  }
}
__global__ void k_ks_inner(const KsOut* __restrict__ outs, const uint64_t* __restrict__ X, const KsLevelConst* __restrict__ kc,
                           uint64_t* __restrict__ U, int n, int log_n, int nl, int n_ext, int n_digits, int n_q) {
  const int k0 = (blockIdx.x * blockDim.x + threadIdx.x) * 2;
  const int e = blockIdx.y % n_ext;
  const int o = blockIdx.y / n_ext;
  if (k0 >= n) return;
  const KsOut od = outs[o];
  const KsPair kk((uint32_t)k0, od.gal, log_n);
  const ModEntry mm = kc->ext[e];
  const int key_mod = e < nl ? e : n_q + (e - nl);
  double acc0[2] = {0.0, 0.0}, acc1[2] = {0.0, 0.0};
  for (int j = 0; j < n_digits; ++j) {
    const u64pair w = ld_pair(ks_digit(od, X, kc, j, e, n_digits, n_ext, n) + kk.at);
    const u64pair kb = ld_pair(od.key + (((size_t)j * 2 + 0) * kc->n_key_mod + key_mod) * n + k0);
    const u64pair ka = ld_pair(od.key + (((size_t)j * 2 + 1) * kc->n_key_mod + key_mod) * n + k0);
    ks_madd(acc0, acc1, w, kk.swap, kb, ka, mm);
    if ((j & 3) == 3) {  // keep |acc| < 5q < 2^53
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        acc0[v] = reduce_s(acc0[v], mm.q, mm.qinv);
        acc1[v] = reduce_s(acc1[v], mm.q, mm.qinv);
      }
    }
  }
  st_pair(U + (((size_t)o * 2 + 0) * n_ext + e) * n + k0, canon_full(acc0[0], mm.q, mm.qinv), canon_full(acc0[1], mm.q, mm.qinv));
  st_pair(U + (((size_t)o * 2 + 1) * n_ext + e) * n + k0, canon_full(acc1[0], mm.q, mm.qinv), canon_full(acc1[1], mm.q, mm.qinv));
}
void launch_ks_inner(blb_ctx* c, const KsOut* outs_dev, int n_out, const uint64_t* X, const KsLevelConst* kc_dev, uint64_t* U, int nl,
                     int n_ext, int n_digits) {
  dim3 grid((c->n / 2 + 255) / 256, n_out * n_ext);
  emit(c, [=, stream = c->stream] { k_ks_inner<<<grid, 256, 0, stream>>>(outs_dev, X, kc_dev, U, c->n, c->log_n, nl, n_ext, n_digits, c->n_q); });
}

// The same inner product for a group of outputs that share a switching key and Galois element, modulo
// one prime: the key words of the thread's two coefficients are loaded once (all ND digits, in
// registers) and applied to every output of the group, whose words are loaded while the output before
// it is computed; per output the arithmetic and its order are those of k_ks_inner, so the words are
// identical.  Groups come in the order in which those that read the same digits follow each other.
// Bound by the words written (2 per digit word read) and the L2: 704 outputs of 3 digits and 7 primes at
// N = 16384, 1.3 GB written, 504 us with two 8-byte loads a pair and groups in key order, 422 us so.
template <int ND>
__global__ void k_ks_inner_grp(const KsOut* __restrict__ outs, const int* __restrict__ ord, const KsGroup* __restrict__ groups,
                               const uint64_t* __restrict__ X, const KsLevelConst* __restrict__ kc, uint64_t* __restrict__ U, int n,
                               int log_n, int nl, int n_ext, int n_q) {
  const int k0 = (blockIdx.x * blockDim.x + threadIdx.x) * 2;
  const KsGroup gr = groups[blockIdx.y];
  const int e = gr.ext;
  if (k0 >= n) return;
  int o = ord[gr.first];
  KsOut od = outs[o];
  const KsPair kk((uint32_t)k0, od.gal, log_n);
  const ModEntry mm = kc->ext[e];
  const int key_mod = e < nl ? e : n_q + (e - nl);
  u64pair kb[ND], ka[ND], w[ND];
  auto fetch = [&] {
#pragma unroll
    for (int j = 0; j < ND; ++j) w[j] = ld_pair(ks_digit(od, X, kc, j, e, ND, n_ext, n) + kk.at);
  };
#pragma unroll
  for (int j = 0; j < ND; ++j) {
    kb[j] = ld_pair(od.key + (((size_t)j * 2 + 0) * kc->n_key_mod + key_mod) * n + k0);
    ka[j] = ld_pair(od.key + (((size_t)j * 2 + 1) * kc->n_key_mod + key_mod) * n + k0);
  }
  fetch();
  for (int i = 0; i < gr.count; ++i) {
    u64pair x[ND];
#pragma unroll
    for (int j = 0; j < ND; ++j) x[j] = w[j];
    const int o_now = o;
    o = ord[gr.first + (i + 1 < gr.count ? i + 1 : i)];  // (the last one fetches its own words again)
    od = outs[o];
    fetch();
    double acc0[2] = {0.0, 0.0}, acc1[2] = {0.0, 0.0};
#pragma unroll
    for (int j = 0; j < ND; ++j) ks_madd(acc0, acc1, x[j], kk.swap, kb[j], ka[j], mm);
    if (ND == 4) {
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        acc0[v] = reduce_s(acc0[v], mm.q, mm.qinv);
        acc1[v] = reduce_s(acc1[v], mm.q, mm.qinv);
      }
    }
    st_pair(U + (((size_t)o_now * 2 + 0) * n_ext + e) * n + k0, canon_full(acc0[0], mm.q, mm.qinv), canon_full(acc0[1], mm.q, mm.qinv));
    st_pair(U + (((size_t)o_now * 2 + 1) * n_ext + e) * n + k0, canon_full(acc1[0], mm.q, mm.qinv), canon_full(acc1[1], mm.q, mm.qinv));
  }
}
void launch_ks_inner_grouped(blb_ctx* c, const KsOut* outs_dev, const int* ord_dev, const KsGroup* groups_dev, int n_groups,
                             const uint64_t* X, const KsLevelConst* kc_dev, uint64_t* U, int nl, int n_ext, int n_digits) {
  dim3 grid((c->n / 2 + 255) / 256, n_groups);
  auto go = [&](auto nd) {
    emit(c, [=, stream = c->stream] {
      k_ks_inner_grp<decltype(nd)::value><<<grid, 256, 0, stream>>>(outs_dev, ord_dev, groups_dev, X, kc_dev, U, c->n, c->log_n, nl, n_ext, c->n_q);
    });
  };
  static_assert(kKsMaxDigits == 4, "a kernel for each number of digits");
  switch (n_digits) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 3: go(std::integral_constant<int, 3>{}); break;
    default: go(std::integral_constant<int, 4>{}); break;
  }
}

// ---------------------------------------------------------------------------------------
// matmul_cp inner sums:  inner[bj][p][limb] = sum_{ai} pt[bj][ai][limb] (.) RX[ai][p][limb]
// Thread per (coefficient k, limb) for a tile of TB outputs.  The plaintext stream is read
// exactly once; RX tiles are re-read per output tile (L2 / MALL resident).
// ---------------------------------------------------------------------------------------
typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Words k .. k + CPT - 1 (k even when CPT = 2) of a plan limb-poly in the 50-bit format at p,
// fetched raw (nontemporal: the plan stream is read once per call) and rebuilt as doubles:
// 2^52 + w has the high word 0x43300000 | w >> 32 and the low word w & 0xFFFFFFFF.
template <int CPT>
struct Pt50Raw {
  uint32_t lo[CPT];
  uint32_t mid[(CPT + 1) / 2];  // bits 32..47 of two words per u32 (the even word in the low half)
  uint32_t top;
};
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// Byte offsets of word k's pieces in a limb-poly of n words: one set per work-item, added to the
// (uniform) address of each limb-poly, so a row costs one scalar address, not one per plane (which
// spilled at 8 rows x 4 coefficients).
struct Pt50Off {
  uint32_t lo, mid, top;
};
__device__ __forceinline__ Pt50Off pt50_off(int n, int k) {
  Pt50Off o{4u * (uint32_t)k, 4u * (uint32_t)n + 2u * (uint32_t)k, 6u * (uint32_t)n + ((uint32_t)k >> 2)};
  asm volatile("" : "+v"(o.lo), "+v"(o.mid), "+v"(o.top));  // opaque: kept out of the scalar address
  return o;
}
// (p may come from a descriptor in memory: addressed as global memory explicitly, so the loads are
// global, not flat, ones)
template <int CPT>
__device__ __forceinline__ void pt50_fetch(const uint8_t* __restrict__ p, const Pt50Off& o, Pt50Raw<CPT>& r) {
  typedef __attribute__((address_space(1))) const uint8_t g8;
  typedef __attribute__((address_space(1))) const uint16_t g16;
  typedef __attribute__((address_space(1))) const uint32_t g32;
  typedef __attribute__((address_space(1))) const u32x2 g32x2;
  typedef __attribute__((address_space(1))) const u32x4 g32x4;
  g8* g = (g8*)p;
  if constexpr (CPT == 4) {
    const u32x4 l = __builtin_nontemporal_load((g32x4*)(g + o.lo));
    r.lo[0] = l.x;
    r.lo[1] = l.y;
    r.lo[2] = l.z;
    r.lo[3] = l.w;
    const u32x2 m = __builtin_nontemporal_load((g32x2*)(g + o.mid));
    r.mid[0] = m.x;
    r.mid[1] = m.y;
  } else if constexpr (CPT == 2) {
    const u32x2 l = __builtin_nontemporal_load((g32x2*)(g + o.lo));
    r.lo[0] = l.x;
    r.lo[1] = l.y;
    r.mid[0] = __builtin_nontemporal_load((g32*)(g + o.mid));
  } else {
    r.lo[0] = __builtin_nontemporal_load((g32*)(g + o.lo));
    r.mid[0] = __builtin_nontemporal_load((g16*)(g + o.mid));
  }
  r.top = __builtin_nontemporal_load(g + o.top);  // the byte that holds words k & ~3 .. k | 3 (u32 words, little-endian)
}
__device__ __forceinline__ double pt50_make(uint32_t lo, uint32_t mid16, uint32_t top2) {
  return __hiloint2double((int)(0x43300000u | (top2 << 16) | mid16), (int)lo) - BLB_TWO52;
}
template <int CPT>
__device__ __forceinline__ void pt50_cvt(const Pt50Raw<CPT>& r, int k, double (&v)[CPT]) {
  const uint32_t t = CPT == 4 ? r.top : r.top >> (2 * (k & 3));
#pragma unroll
  for (int j = 0; j < CPT; ++j) v[j] = pt50_make(r.lo[j], (j & 1) ? r.mid[j / 2] >> 16 : r.mid[j / 2] & 0xFFFFu, (t >> (2 * j)) & 3u);
}


// One block's (tile, k-chunk, limb): WAVES waves, each TB output rows x 64 CPT coefficients.
// Bound by HBM (the plaintexts are read once; 7 FP64 instructions per word and poly take a third
// of the issue slots).  What the shape decides is how evenly the stream is spread: every block
// runs as long as its n_ai terms take, so a grid of a few blocks per CU is as slow as the CU that
// got one more.  One-wave blocks (64 threads) spread best; 256-thread blocks of the same tile left
// 3 blocks on some CUs and 2 on others.  SPLIT > 1 divides the terms over the waves of a block
// (their sums meet in LDS), for grids too small to keep enough loads in flight.
// Words of the next term are loaded before the current term is multiplied.  Rows past a partial
// last tile re-read its last row (not stored), so the body has no branches.
template <int TB, int CPT, int SPLIT, int WAVES, bool P50>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2))) void k_cp_mac(
    const uint64_t* __restrict__ pt, const uint64_t* const* __restrict__ rx_tab, uint64_t* __restrict__ inner, int n, int nl, int n_ai,
    int n_bj, ModTable mt, int n_kblk) {
  static_assert(CPT == 2 || CPT == 4, "coefficients per thread");
  static_assert(SPLIT == 1 || SPLIT == WAVES, "every wave of a split block has its own terms");
  typedef __attribute__((address_space(1))) const uint64_t gu64;
  typedef __attribute__((address_space(1))) const u64x2 gu64x2;
  constexpr int LANES = 64 * WAVES / SPLIT;  // work-items over the coefficients
  // Block order: k-chunk fastest, then limb, then output tile.  Consecutive blocks stream
  // consecutive pieces of one plaintext limb-poly (the dispatcher deals them round-robin over the
  // 8 XCDs), and the blocks of one (k-chunk, limb) -- the ones reading the same rotated-input
  // words -- lie n_kblk * nl apart, a multiple of 8 whenever n_kblk is: one XCD, one L2.
  const int kb = blockIdx.x % n_kblk;
  const int limb = (blockIdx.x / n_kblk) % nl;
  const int tile = blockIdx.x / (n_kblk * nl);
  const int part = SPLIT > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / LANES) : 0;
  const int lane = threadIdx.x % LANES;
  const int k0 = (kb * LANES + lane) * CPT;
  const ModEntry me = mt.m[limb];
  const double q = me.q, qi = me.qinv;
  const int bj0 = tile * TB;
  const int rows = min(TB, n_bj - bj0);
  const int ai0 = n_ai * part / SPLIT, ai1 = n_ai * (part + 1) / SPLIT;  // this wave's terms (none if n_ai < SPLIT)
  const size_t pb = pt_poly_bytes(n, P50);
  const size_t stride_ai = (size_t)nl * pb, stride_bj = (size_t)n_ai * stride_ai;
  const uint8_t* pbase = (const uint8_t*)pt + (size_t)bj0 * stride_bj + (size_t)limb * pb;
  size_t row[TB];
#pragma unroll
  for (int t = 0; t < TB; ++t) row[t] = (size_t)min(t, rows - 1) * stride_bj;
  const Pt50Off off50 = pt50_off(n, k0);
  Pt50Raw<CPT> w50[TB];
  u64x2 w64[TB][CPT / 2], r0[CPT / 2], r1[CPT / 2];
  auto fetch = [&](int ai) {
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      const uint8_t* poly = pbase + row[t] + (size_t)ai * stride_ai;
      if constexpr (P50) {
        pt50_fetch<CPT>(poly, off50, w50[t]);
      } else {  // non-temporal: the plan is read once, the rotated inputs by every tile
#pragma unroll
        for (int h = 0; h < CPT / 2; ++h) w64[t][h] = __builtin_nontemporal_load((gu64x2*)((gu64*)poly + k0 + 2 * h));
      }
    }
    gu64* rx = (gu64*)rx_tab[ai];
#pragma unroll
    for (int h = 0; h < CPT / 2; ++h) {
      r0[h] = *(gu64x2*)(rx + (size_t)limb * n + k0 + 2 * h);
      r1[h] = *(gu64x2*)(rx + (size_t)(nl + limb) * n + k0 + 2 * h);
    }
  };
  double a0[TB][CPT], a1[TB][CPT];
#pragma unroll
  for (int t = 0; t < TB; ++t)
#pragma unroll
    for (int c = 0; c < CPT; ++c) a0[t][c] = a1[t][c] = 0.0;
  auto reduce_all = [&] {
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        a0[t][c] = reduce_s(a0[t][c], q, qi);
        a1[t][c] = reduce_s(a1[t][c], q, qi);
      }
  };
  if (ai0 < ai1) fetch(ai0);
  for (int ai = ai0; ai < ai1; ++ai) {
    double w[TB][CPT], x0[CPT], x1[CPT];
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      if constexpr (P50) {
        pt50_cvt<CPT>(w50[t], k0, w[t]);
      } else {
#pragma unroll
        for (int c = 0; c < CPT; ++c) w[t][c] = u2d((c & 1) ? w64[t][c / 2].y : w64[t][c / 2].x);
      }
    }
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      x0[c] = u2d((c & 1) ? r0[c / 2].y : r0[c / 2].x);
      x1[c] = u2d((c & 1) ? r1[c / 2].y : r1[c / 2].x);
    }
    fetch(min(ai + 1, ai1 - 1));  // the last term re-reads itself
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        a0[t][c] += mulmod_s(w[t][c], x0[c], q, qi);
        a1[t][c] += mulmod_s(w[t][c], x1[c], q, qi);
      }
    if (((ai - ai0) & 7) == 7) reduce_all();  // 8 products below 0.875 q on |acc| <= q/2: |acc| < 7.5 q < 2^53
  }
  if constexpr (SPLIT > 1) {
    __shared__ double part_sum[SPLIT - 1][2 * TB * CPT][LANES];
    reduce_all();
    if (part > 0) {
#pragma unroll
      for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
          part_sum[part - 1][t * CPT + c][lane] = a0[t][c];
          part_sum[part - 1][(TB + t) * CPT + c][lane] = a1[t][c];
        }
    }
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int s = 0; s < SPLIT - 1; ++s)
#pragma unroll
      for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
          a0[t][c] += part_sum[s][t * CPT + c][lane];
          a1[t][c] += part_sum[s][(TB + t) * CPT + c][lane];
        }
  }
#pragma unroll
  for (int t = 0; t < TB; ++t) {
    if (t < rows) {
      uint64_t* o0 = inner + (((size_t)(bj0 + t) * 2 + 0) * nl + limb) * n + k0;
      uint64_t* o1 = inner + (((size_t)(bj0 + t) * 2 + 1) * nl + limb) * n + k0;
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        o0[c] = d2u(canon_full(a0[t][c], q, qi));
        o1[c] = d2u(canon_full(a1[t][c], q, qi));
      }
    }
  }
}

// Launch shapes {outputs per wave, coefficients per work-item, waves the terms are divided over,
// waves per block}; none changes a result bit.  Shape 0 is chosen by the size of the product.
struct MacShape {
  int tb, cpt, split, waves;
};
constexpr MacShape kMacShapes[BLB_MAC_VARIANTS] = {
    {0, 0, 0, 0}, {12, 2, 1, 1}, {8, 2, 1, 1}, {8, 2, 2, 2}, {4, 2, 4, 4}, {2, 2, 4, 4}, {8, 4, 1, 4}, {4, 4, 1, 1}, {4, 4, 2, 2},
    {6, 4, 1, 1}, {6, 2, 1, 1}, {4, 2, 1, 1}, {4, 2, 2, 2}, {8, 2, 1, 4}, {4, 2, 1, 4}, {12, 2, 1, 4}, {6, 4, 1, 4}, {4, 4, 1, 4}};

// The shape of a product, by the waves that its outputs give at 8 rows x 2 (64-bit words) or 4 rows
// x 4 (50-bit) coefficients per work-item.  Measured alone, us of the shape taken against its
// neighbour: 64-bit words, 2304 waves (n_ai 192, n_bj 96, 3 limbs, N = 8192): {12,2,1,1} 540, {8,2,1,1}
// 609 (the 256-thread {8,2,1,4}: 682); 1728 waves: {8,2,1,1} 401, {8,2,2,2} 429; 960: {8,2,2,2} 130,
// {8,2,1,1} 139; 576: 245 against 373; 384: {4,2,4,4} 15.2, {8,2,2,2} 19.8; 128: {2,2,4,4} 12.4, {8,2,2,2} 23.
// 50-bit words, 16384 waves: {8,4,1,4} 2386 (5.6 TB/s of packed words), {4,4,1,1} 2814; 3072: {6,4,1,1} 343,
// {4,4,1,1} 370; 2304: {6,4,1,1} 561, {4,4,1,1} 643, {8,4,1,4} 753 and 1728: {4,4,1,4} 418, {4,4,1,1} 438, {6,4,1,1} 465
// (both inside the operator); 960: {4,4,2,2} 119, {4,4,1,1} 154; 384: {4,2,4,4} 15.4, {4,4,2,2} 22; 128:
// {2,2,4,4} 12.6, {4,2,4,4} 14.2.  12 rows only where they pad the outputs by little.
// Larger products, alone: 64-bit words, N = 8192 (n_ai 48) at 4224 / 8256 / 16512 waves: {12,2,1,1} 313 / 610 / 1208,
// {8,2,1,1} 328 / 626 / 1249, {8,2,1,4} 327 / 621 / 1231, {12,2,1,4} 308 / 593 / 1181; N = 16384 (n_ai 32) at 4224 / 9216 /
// 16512: 228-235 / 448 / 852, 233 / 470 / 881, 236 / 469 / 891, 241 / 457 / 846: within 3 % of the best, and of the
// 256-thread blocks that were the rule before.  50-bit words, 4224-4608 waves: {8,4,1,4} 238-242 (N = 16384), 332-338
// (N = 8192), {6,4,1,1} 204-217, 292-307; 8064-8256: 353, 566 against 382, 561; 16512: 736, 1056 against 772, 1117; 1536 waves:
// {4,4,1,4} 120, {4,4,2,2} 112.  So the 50-bit lines at 4096 and 1536 stand too low by these sizes; the points
// inside the operators above put them there.
int64_t mac_waves(int n, int nl, int n_bj) { return (int64_t)n * nl / 128 * ((n_bj + 7) / 8); }
MacShape mac_shape_for(int n, int nl, int n_bj, int p50) {
  const int64_t cols = (int64_t)n * nl;
  if (p50) {
    const int64_t waves = cols / 256 * ((n_bj + 3) / 4);
    if (waves >= 4096) return kMacShapes[6];
    if (waves >= 2048) return kMacShapes[9];
    if (waves >= 1536) return kMacShapes[17];
    if (waves >= 640) return kMacShapes[8];
    return kMacShapes[waves >= 256 ? 4 : 5];
  }
  const int64_t waves = mac_waves(n, nl, n_bj);
  const int pad12 = (n_bj + 11) / 12 * 12, pad8 = (n_bj + 7) / 8 * 8;
  if (waves >= 2048 && pad12 * 16 <= pad8 * 17) return kMacShapes[1];
  if (waves >= 1536) return kMacShapes[2];
  if (waves >= 512) return kMacShapes[3];
  return kMacShapes[waves >= 256 ? 4 : 5];
}

void launch_cp_mac(blb_ctx* c, const uint64_t* pt, const uint64_t* const* rx_tab, uint64_t* inner, int nl, int n_ai, int n_bj, int variant,
                   int p50) {
  const MacShape sh = variant > 0 && variant < BLB_MAC_VARIANTS ? kMacShapes[variant] : mac_shape_for(c->n, nl, n_bj, p50);
  const int n_kblk = c->n / (64 * sh.waves / sh.split * sh.cpt);
  const int blocks = n_kblk * nl * ((n_bj + sh.tb - 1) / sh.tb);
#define CPMAC(tb_, cpt_, split_, waves_)                                                                                            \
  if (sh.tb == tb_ && sh.cpt == cpt_ && sh.split == split_ && sh.waves == waves_) {                                                 \
    if (p50)                                                                                                                        \
      emit(c, [=, stream = c->stream] { k_cp_mac<tb_, cpt_, split_, waves_, true><<<blocks, 64 * waves_, 0, stream>>>(pt, rx_tab, inner, c->n, nl, n_ai, n_bj, c->mt, n_kblk); }); \
    else                                                                                                                            \
      emit(c, [=, stream = c->stream] { k_cp_mac<tb_, cpt_, split_, waves_, false><<<blocks, 64 * waves_, 0, stream>>>(pt, rx_tab, inner, c->n, nl, n_ai, n_bj, c->mt, n_kblk); }); \
    return;                                                                                                                         \
  }
  CPMAC(12, 2, 1, 1)
  CPMAC(8, 2, 1, 1)
  CPMAC(8, 2, 2, 2)
  CPMAC(4, 2, 4, 4)
  CPMAC(2, 2, 4, 4)
  CPMAC(8, 4, 1, 4)
  CPMAC(4, 4, 1, 1)
  CPMAC(4, 4, 2, 2)
  CPMAC(6, 4, 1, 1)
  CPMAC(6, 2, 1, 1)
  CPMAC(4, 2, 1, 1)
  CPMAC(4, 2, 2, 2)
  CPMAC(8, 2, 1, 4)
  CPMAC(4, 2, 1, 4)
  CPMAC(12, 2, 1, 4)
  CPMAC(6, 4, 1, 4)
  CPMAC(4, 4, 1, 4)
#undef CPMAC
}

// out[o] = sum_t src[o * n_terms + t] over whole ciphertexts ([2][nl][N] words), mod q_limb
__global__ void k_sum_cts(const uint64_t* const* __restrict__ srcs, uint64_t* const* __restrict__ dsts, int n_terms, int n, int nl,
                          ModTable mt) {
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  const int o = blockIdx.y;
  if (w >= 2 * nl * n) return;
  const ModEntry me = mt.m[(w / n) % nl];
  double acc = 0.0;
  for (int t = 0; t < n_terms; ++t) {
    acc += u2d(gmem(srcs[(size_t)o * n_terms + t])[w]);
    if ((t & 3) == 3) acc = reduce_s(acc, me.q, me.qinv);
  }
  gmem(dsts[o])[w] = d2u(canon_full(acc, me.q, me.qinv));
}
void launch_sum_cts(blb_ctx* c, const uint64_t* const* srcs, uint64_t* const* dsts, int n_out, int n_terms, int nl) {
  dim3 grid((2 * nl * c->n + 255) / 256, n_out);
  emit(c, [=, stream = c->stream] { k_sum_cts<<<grid, 256, 0, stream>>>(srcs, dsts, n_terms, c->n, nl, c->mt); });
}

// ---------------------------------------------------------------------------------------
// Mask-and-share: r uniform per limb in coefficient form (tag mask, object = ct index),
// share = -r mod q_i; the mask is added to c0 in evaluation form by the caller after an NTT.
// ---------------------------------------------------------------------------------------
__global__ void k_mask_sample(uint64_t* r_out, uint64_t* share, int n, int tl, ModTable mt, uint32_t k0, uint32_t k1,
                              const uint64_t* seed_dev, uint32_t tag) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const int i = blockIdx.y % tl;
  const int t = blockIdx.y / tl;
  if (k >= n) return;
  if (seed_dev) {
    const uint64_t sd = *seed_dev;
    k0 = (uint32_t)sd;
    k1 = (uint32_t)(sd >> 32);
  }
  const ModEntry me = mt.m[i];
  const U4 w = philox10((uint32_t)k, (uint32_t)i, (uint32_t)t, tag, k0, k1);
  const double r = u128_mod(w, me.q, me.qinv);
  const size_t o = ((size_t)t * tl + i) * n + k;
  r_out[o] = d2u(r);
  share[o] = d2u(r == 0.0 ? 0.0 : me.q - r);
}
void launch_mask_sample(blb_ctx* c, uint64_t* r_out, uint64_t* share, int n_ct, int tl, uint64_t seed, const uint64_t* seed_dev,
                        uint32_t tag) {
  dim3 grid((c->n + 255) / 256, n_ct * tl);
  emit(c, [=, stream = c->stream] { k_mask_sample<<<grid, 256, 0, stream>>>(r_out, share, c->n, tl, c->mt, (uint32_t)seed, (uint32_t)(seed >> 32), seed_dev, tag); });
}

__global__ void k_set_u64(uint64_t* dst, uint64_t v) { *dst = v; }
void launch_set_u64(blb_ctx* c, uint64_t* dst, uint64_t value) { emit(c, [=, stream = c->stream] { k_set_u64<<<1, 1, 0, stream>>>(dst, value); }); }

__global__ void k_zero(uint64_t* dst, size_t words) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < words) dst[i] = 0;
}
// a descriptor table from mapped host memory to its device region, 16 bytes per work-item
__global__ void k_stage(uint4* __restrict__ dst, const uint4* __restrict__ src, unsigned n16) {
  const unsigned i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n16) dst[i] = src[i];
}
void launch_stage(hipStream_t stream, void* dst, const void* src_mapped, size_t bytes) {
  const unsigned n16 = (unsigned)(bytes / 16);
  k_stage<<<(n16 + 255) / 256, 256, 0, stream>>>((uint4*)dst, (const uint4*)src_mapped, n16);
}
void launch_zero(blb_ctx* c, uint64_t* dst, size_t words) {
  if (!words) return;
  emit(c, [=, stream = c->stream] { k_zero<<<(unsigned)((words + 255) / 256), 256, 0, stream>>>(dst, words); });
}

// ---------------------------------------------------------------------------------------
// Encoder (eq. ckks_encode) in double-double arithmetic.
//   Slot j sits at zeta^(e_j), e_j = 5^j mod 2N = 4 u_j + 1.  With w_k = p_k + i p_{k+M}
//   (M = N/2), p(zeta^(4u+1)) = sum_k zeta^k w_k eta^(uk), eta = exp(2 pi i / M), so
//   w_k = zeta^-k (1/M) sum_u v_u eta^(-uk) with v_u the (real) slot value at u.
//   Steps: DFT of size M (exp(-i...)) of the slot values placed at their positions u, then
//   finalize (twist, scale, round half away from zero, reduce into the limbs).
// ---------------------------------------------------------------------------------------
struct dd { double hi, lo; };
__device__ __forceinline__ dd two_sum(double a, double b) {
  const double s = a + b;
  const double bb = s - a;
  const double err = (a - (s - bb)) + (b - bb);
  return dd{s, err};
}
__device__ __forceinline__ dd quick_two_sum(double a, double b) {
  const double s = a + b;
  return dd{s, b - (s - a)};
}
__device__ __forceinline__ dd dd_add(dd x, dd y) {
  dd s = two_sum(x.hi, y.hi);
  dd t = two_sum(x.lo, y.lo);
  s.lo += t.hi;
  s = quick_two_sum(s.hi, s.lo);
  s.lo += t.lo;
  return quick_two_sum(s.hi, s.lo);
}
__device__ __forceinline__ dd dd_neg(dd x) { return dd{-x.hi, -x.lo}; }
__device__ __forceinline__ dd dd_mul(dd x, dd y) {
  const double p = x.hi * y.hi;
  double e = __builtin_fma(x.hi, y.hi, -p);
  e += x.hi * y.lo + x.lo * y.hi;
  return quick_two_sum(p, e);
}
__device__ __forceinline__ dd dd_mul_d(dd x, double y) {
  const double p = x.hi * y;
  double e = __builtin_fma(x.hi, y, -p);
  e += x.lo * y;
  return quick_two_sum(p, e);
}
struct cdd { dd re, im; };
__device__ __forceinline__ cdd cdd_mul(cdd a, cdd b) {
  return cdd{dd_add(dd_mul(a.re, b.re), dd_neg(dd_mul(a.im, b.im))), dd_add(dd_mul(a.re, b.im), dd_mul(a.im, b.re))};
}
__device__ __forceinline__ cdd cdd_add(cdd a, cdd b) { return cdd{dd_add(a.re, b.re), dd_add(a.im, b.im)}; }
__device__ __forceinline__ cdd cdd_sub(cdd a, cdd b) { return cdd{dd_add(a.re, dd_neg(b.re)), dd_add(a.im, dd_neg(b.im))}; }
__device__ __forceinline__ cdd ld_cdd(const double* p) { return cdd{dd{p[0], p[1]}, dd{p[2], p[3]}}; }
__device__ __forceinline__ void st_cdd(double* p, cdd v) { p[0] = v.re.hi; p[1] = v.re.lo; p[2] = v.im.hi; p[3] = v.im.lo; }

// Slot values.  Position u of the DFT input holds slot j = slot_inv[u] (u_j = (5^j mod 2N - 1) / 4).
// Dense source: vals[p][j], n_vals per plaintext, one plaintext per complex vector.
// begin(p) gathers what is uniform over complex vector p, (ctx, u) gives the value at u.
struct EncSrcDense {
  const double* vals;
  int n_vals;
  const int32_t* slot_inv;
  __device__ const double* begin(int p) const { return vals + (size_t)p * n_vals; }
  __device__ cdd operator()(const double* v, int u) const {
    const int j = slot_inv[u];
    return cdd{dd{j < n_vals ? v[j] : 0.0, 0.0}, dd{0.0, 0.0}};
  }
};

// The first-block mask: 1 in slots 0 .. block - 1, 0 elsewhere.
struct EncSrcBlock {
  int block;
  const int32_t* slot_inv;
  __device__ int begin(int) const { return block; }
  __device__ cdd operator()(int b, int u) const { return cdd{dd{slot_inv[u] < b ? 1.0 : 0.0, 0.0}, dd{0.0, 0.0}}; }
};

// matmul_cp diagonal plaintexts, two per complex vector (plaintext p0 + 2 pp in the real part,
// p0 + 2 pp + 1 in the imaginary part, split apart after the transform); with the complex-slot
// output packing (g.cplx) one plaintext per complex vector, whose slots hold the diagonal of
// output block 2b in the real and that of block 2b + 1 in the imaginary part; plaintext p = (bj, ai):
//   value at slot s = W{a c + ((u + t) mod c_eff), b c + (u mod c_out)}, u = ((s - r) mod S) / L',
//   t = jB + i, r = j B L' (plaintext pre-rotated right by r).
// L', c, c_eff, c_out and S are powers of two (lLp = log2 L').
// Plaintext diagonals of matmul_cp: diagonal (b, j, a, i) pre-rotated right by j B L' slots,
// block u of the unrotated vector holding W{row, b c + (u mod c_out)} where, with
// u' = (u + j B + i) mod c_eff, row = a c + u' for a spatial-first input (broadcast over the
// L' slots of the block) or, for a diagonal-packed input (dg.tab set), row = h d_v + (r + tau)
// mod d_v' at slot r of the block, (h, tau) being the head and diagonal that block u' of input
// a holds (0 for r >= L or a padded column).
struct EncSrcCp {
  const double* W;
  CpGeom g;
  int p0, count, M, lLp;
  const int32_t* slot_inv;
  CpDiag dg;
  struct Diag {
    int r, t, row0, col0;
    bool used;
    CpDiagIn in;
  };
  struct Pair {
    Diag x, y;
  };
  __device__ Diag diag(int p, int half) const {
    const int n_ai = g.n_in * g.B;
    const int bj = p / n_ai, ai = p % n_ai;
    const int b = g.cplx ? 2 * (bj / g.G) + half : bj / g.G, j = bj % g.G;
    const int a = ai / g.B, i = ai % g.B;
    const bool used = p < p0 + count;
    const CpDiagIn in = (dg.tab && used) ? dg.tab[a] : CpDiagIn{0, 0, 1, 0};
    return Diag{j * g.B * g.Lp, j * g.B + i, a * g.c, b * g.c, used, in};
  }
  __device__ double value(const Diag& d, int s) const {
    if (!d.used) return 0.0;
    const int sr = (s - d.r) & (M - 1);
    const int u = sr >> lLp;
    const int ub = (u + d.t) & (g.c_eff - 1);
    const int col = d.col0 + (u & (g.c_out - 1));
    int row = d.row0 + ub;
    if (dg.tab) {
      const int r = sr & (g.Lp - 1);
      const int h = d.in.h0 + (ub & ((1 << d.in.logH) - 1));
      const int jj = (r + d.in.o * d.in.cg + (ub >> d.in.logH)) & (dg.dvp - 1);
      if (r >= dg.L || jj >= dg.d_v) return 0.0;
      row = h * dg.d_v + jj;
    }
    return (row < g.d_in && col < g.d_out) ? W[(size_t)row * g.d_out + col] : 0.0;
  }
  __device__ Pair begin(int pp) const {
    return g.cplx ? Pair{diag(p0 + pp, 0), diag(p0 + pp, 1)} : Pair{diag(p0 + 2 * pp, 0), diag(p0 + 2 * pp + 1, 0)};
  }
  __device__ cdd operator()(const Pair& pr, int u) const {
    const int s = slot_inv[u];
    return cdd{dd{value(pr.x, s), 0.0}, dd{value(pr.y, s), 0.0}};
  }
};

// The size-M DFT (forward sign) in four steps, M = M1 M2 with M2 = 128, n = M2 n1 + n2,
// k = k1 + M1 k2:
//   Y[k1 + M1 k2] = sum_n2 e^(-2 pi i n2 k2 / M2) [ e^(-2 pi i n2 k1 / M) sum_n1 v[M2 n1 + n2] e^(-2 pi i n1 k1 / M1) ].
// The column pass does the inner M1-point DFTs and the twiddles (Z[k1][n2]), the row pass the
// outer M2-point DFTs, so the transform makes two passes over HBM.  Each small DFT is split once
// more into radix-8 DFTs held in registers (M1 = 8 R2 with R2 = 2, 4 or 8; M2 = 8 x 16), with one
// exchange through LDS in between.
constexpr int kEncM2 = 128;
constexpr int kEncThreads = 128;  // work-items of a column-pass workgroup
constexpr int kEncRB = 8;         // rows (k1) per workgroup in the row pass

// e^(-2 pi i e / M), 0 <= e < M, from the table of eta^k = e^(2 pi i k / M), k < M/2
__device__ __forceinline__ cdd enc_twiddle(const double* tw, int e, int M) {
  const int half = M / 2;
  cdd w = ld_cdd(tw + (size_t)(e >= half ? e - half : e) * 4);
  w.im = dd_neg(w.im);
  if (e >= half) {
    w.re = dd_neg(w.re);
    w.im = dd_neg(w.im);
  }
  return w;
}

// x (-i)
__device__ __forceinline__ cdd cdd_mul_mi(cdd a) { return cdd{a.im, dd_neg(a.re)}; }

// In-place DFT (forward sign) of R = 2, 4 or 8 values in natural order, decimation in frequency:
// stage spans R/2 .. 1, twiddles e^(-2 pi i j / span*2) (1, -i and w8 = e^(-i pi / 4)), then the
// bit-reversed results put back in natural order.
template <int R>
__device__ __forceinline__ void dft_small(cdd (&a)[R], cdd w8) {
#pragma unroll
  for (int span = R / 2; span >= 1; span /= 2) {
#pragma unroll
    for (int b = 0; b < R; b += 2 * span) {
#pragma unroll
      for (int j = 0; j < span; ++j) {
        const cdd x = a[b + j], y = a[b + j + span];
        a[b + j] = cdd_add(x, y);
        cdd d = cdd_sub(x, y);
        // twiddle e^(-2 pi i j / (2 span)) = w8^(j * 4 / span)
        const int e8 = j * (4 / span);  // in units of 1/8 turn: 0..3
        if (e8 & 1) d = cdd_mul(d, w8);
        if (e8 & 2) d = cdd_mul_mi(d);
        a[b + j + span] = d;
      }
    }
  }
  cdd t[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    int r = 0;
#pragma unroll
    for (int bit = 1; bit < R; bit <<= 1) r = (r << 1) | ((k & bit) ? 1 : 0);
    t[r] = a[k];
  }
#pragma unroll
  for (int k = 0; k < R; ++k) a[k] = t[k];
}

// Column pass: CB columns n2 of complex vector p; writes Z[p][k1][n2] (rows of M2).
// M1 = 8 R2: n1 = na + R2 nb, k1 = kb + 8 ka,
//   X[kb + 8 ka] = sum_na e^(-2 pi i na ka / R2) e^(-2 pi i na kb / M1) DFT8_nb(x[na + R2 nb])[kb].
// Step 1 (work-item (c, na)): the DFT8 over nb and its twiddle, into LDS S[kb][na][c]; step 2
// (work-item (c, kb), CB / 16 values of kb each): the DFT of size R2 over na, the four-step twiddle, the
// store.  With CB = 128 / R2 every work-item has a DFT8 of its own (of 16 columns half of the work-items
// have none at N = 8192 and three quarters at N = 4096): right for many vectors.  A few leave most of the GPU
// idle either way, and 16 columns give them more workgroups and each work-item one DFT of step 2 (a single
// vector encoded and waited for, with and without the flag's launch of its own that `clear` saves: N = 4096 53.5
// against 56.8 us, N = 8192 59.8 against 63.9, N = 16384, 16 columns either way, 64.0 against 65.5).
// clear: the overflow flag, zeroed for the row pass (null: it is kept).
template <class Src, int R2, int CB>
__global__ __launch_bounds__(kEncThreads) void k_enc_cols(Src src, double* zbuf, const double* tw, int M, int* clear) {
  constexpr int M1 = 8 * R2, QN = kEncThreads / CB;
  static_assert(QN >= R2 && 8 % QN == 0, "work-items of a column");
  __shared__ cdd S[8 * R2 * CB];
  const int n2_0 = blockIdx.x * CB;
  const int p = blockIdx.y;
  const int t = threadIdx.x;
  const int c = t % CB, q = t / CB;  // q: na in step 1, kb mod QN in step 2
  const cdd w8 = enc_twiddle(tw, M / 8, M);
  const auto ctx = src.begin(p);
  if (clear && (blockIdx.x | blockIdx.y | threadIdx.x) == 0) *clear = 0;
  if (QN == R2 || q < R2) {
    cdd a[8];
#pragma unroll
    for (int nb = 0; nb < 8; ++nb) a[nb] = src(ctx, kEncM2 * (q + R2 * nb) + n2_0 + c);
    dft_small<8>(a, w8);
#pragma unroll
    for (int kb = 0; kb < 8; ++kb) {
      const cdd v = kb == 0 || q == 0 ? a[kb] : cdd_mul(a[kb], enc_twiddle(tw, q * kb * (M / M1), M));
      S[(kb * R2 + q) * CB + c] = v;
    }
  }
  __syncthreads();
  const int n2 = n2_0 + c;
#pragma unroll
  for (int i = 0; i < 8 / QN; ++i) {
    const int kb = q + QN * i;
    cdd b[R2];
#pragma unroll
    for (int na = 0; na < R2; ++na) b[na] = S[(kb * R2 + na) * CB + c];
    dft_small<R2>(b, w8);
#pragma unroll
    for (int ka = 0; ka < R2; ++ka) {
      const int k1 = kb + 8 * ka;
      const cdd z = cdd_mul(b[ka], enc_twiddle(tw, n2 * k1, M));  // n2 k1 < M2 M1 = M
      st_cdd(zbuf + ((size_t)p * M + (size_t)k1 * kEncM2 + n2) * 4, z);
    }
  }
}

__device__ __forceinline__ long long rhaz_dd(dd x, int* overflow) {
  const bool neg = x.hi < 0.0;
  if (neg) x = dd_neg(x);
  if (!(x.hi < 4.0e18)) { *overflow = 1; return 0; }
  const double f = floor(x.hi);
  const double frac = (x.hi - f) + x.lo;
  long long r = (long long)f + (long long)floor(frac + 0.5);
  return neg ? -r : r;
}

// rounding of one transformed value y_k: w = zeta^-k y_k (Delta / M), coefficients k and k + M of the
// plaintext are RHAZ(Re w) and RHAZ(Im w) (|.| < 4e18, else *overflow is set)
__device__ __forceinline__ void enc_round(cdd y, cdd twist, double scale_over_m, long long* out_k, int M, int* overflow) {
  const cdd w = cdd_mul(y, twist);
  int of = 0;
  const long long pr = rhaz_dd(dd_mul_d(w.re, scale_over_m), &of);
  const long long pi = rhaz_dd(dd_mul_d(w.im, scale_over_m), &of);
  if (of) atomicOr(overflow, 1);
  out_k[0] = pr;
  out_k[M] = pi;
}

// Row pass and rounding: kEncRB rows k1 of vector p.  M2 = 128: n2 = na + 16 nb,
// k2 = kb + 8 ka (na, ka < 16; nb, kb < 8),
//   X[kb + 8 ka] = DFT16_na(s_kb)[ka],  s_kb[na] = e^(-2 pi i na kb / 128) DFT8_nb(x[na + 16 nb])[kb].
// Step 1 (work-item (na, r)): the DFT8 over nb and its twiddle, into LDS; step 2 (work-item
// (r, kb, h)): the first decimation-in-frequency stage of the DFT16 (h = 0: s[n] + s[n + 8] for the
// even ka; h = 1: (s[n] - s[n + 8]) e^(-2 pi i n / 16) for the odd ka), then a DFT8.
// The transformed values y_k, k = k1 + M1 k2, are rounded to the plaintext's integer coefficients
// out[p][N] here (a pass of its own read them back, and wrote every limb's residues, which the
// plaintext's transforms now take from the integers).
// PAIRED: vector pp holds FFT(x_{2pp} + i x_{2pp+1}) of two real inputs, whose transforms are
// X1_k = (Y_k + conj Y_{M-k}) / 2 and X2_k = (Y_k - conj Y_{M-k}) / (2i).  M - k lies in row M1 - k1, so a
// workgroup takes four rows and their mirrors (rows 0 and M1/2 are their own) and exchanges the
// values through LDS.
constexpr int kEncRowPad = kEncRB + 1;  // LDS row stride (in cdd) of S[kb][na][r]
template <bool PAIRED>
__global__ __launch_bounds__(kEncRB * 16) void k_enc_rows(const double* zbuf, const double* tw, const double* twist, double scale_over_m,
                                                          long long* out, int count, int* overflow, int M, int M1) {
  __shared__ cdd S[8 * 16 * kEncRowPad];
  const int p = blockIdx.y;
  const int t = threadIdx.x;
  const cdd w8 = enc_twiddle(tw, M / 8, M);
  auto row_of = [&](int r) {
    if (!PAIRED) return (int)blockIdx.x * kEncRB + r;
    const int a = (int)blockIdx.x * (kEncRB / 2) + (r & (kEncRB / 2 - 1));
    if (r < kEncRB / 2) return a;
    return a == 0 ? M1 / 2 : M1 - a;
  };
  {
    const int na = t % 16, r = t / 16;
    const double* row = zbuf + ((size_t)p * M + (size_t)row_of(r) * kEncM2) * 4;
    cdd a[8];
#pragma unroll
    for (int nb = 0; nb < 8; ++nb) a[nb] = ld_cdd(row + (size_t)(na + 16 * nb) * 4);
    dft_small<8>(a, w8);
#pragma unroll
    for (int kb = 0; kb < 8; ++kb) {
      const cdd v = kb == 0 || na == 0 ? a[kb] : cdd_mul(a[kb], enc_twiddle(tw, na * kb * (M / kEncM2), M));
      S[(kb * 16 + na) * kEncRowPad + r] = v;
    }
  }
  __syncthreads();
  const int r = t % kEncRB, q = t / kEncRB;
  const int kb = q % 8, h = q / 8;
  cdd b[8];
#pragma unroll
  for (int n = 0; n < 8; ++n) {
    const cdd s0 = S[(kb * 16 + n) * kEncRowPad + r], s8 = S[(kb * 16 + n + 8) * kEncRowPad + r];
    b[n] = h == 0 ? cdd_add(s0, s8) : (n == 0 ? cdd_sub(s0, s8) : cdd_mul(cdd_sub(s0, s8), enc_twiddle(tw, n * (M / 16), M)));
  }
  dft_small<8>(b, w8);
  const int k1 = row_of(r);
  if constexpr (!PAIRED) {
#pragma unroll
    for (int kp = 0; kp < 8; ++kp) {
      const int k = k1 + M1 * (kb + 8 * (2 * kp + h));
      enc_round(b[kp], ld_cdd(twist + (size_t)k * 4), scale_over_m, out + (size_t)p * 2 * M + k, M, overflow);
    }
  } else {
    __syncthreads();  // every work-item is past its reads of S
#pragma unroll
    for (int kp = 0; kp < 8; ++kp) S[(kb + 8 * (2 * kp + h)) * kEncRowPad + r] = b[kp];
    __syncthreads();
    // the mirror of (k1, k2): row M1 - k1, M2 - 1 - k2; of row 0: M2 - k2 (mod M2)
    const int rm = k1 == 0 || k1 == M1 / 2 ? r : r ^ (kEncRB / 2);
#pragma unroll
    for (int kp = 0; kp < 8; ++kp) {
      const int k2 = kb + 8 * (2 * kp + h), k = k1 + M1 * k2;
      const int k2m = k1 == 0 ? (kEncM2 - k2) % kEncM2 : kEncM2 - 1 - k2;
      const cdd y = b[kp], yc = S[k2m * kEncRowPad + rm];
      const dd half_re1 = dd_add(y.re, yc.re), half_im1 = dd_add(y.im, dd_neg(yc.im));  // Y + conj(Yc)
      const dd half_re2 = dd_add(y.im, yc.im), half_im2 = dd_add(yc.re, dd_neg(y.re));  // (Y - conj(Yc)) / i
      const cdd x1 = cdd{dd_mul_d(half_re1, 0.5), dd_mul_d(half_im1, 0.5)};
      const cdd x2 = cdd{dd_mul_d(half_re2, 0.5), dd_mul_d(half_im2, 0.5)};
      const cdd tws = ld_cdd(twist + (size_t)k * 4);
      enc_round(x1, tws, scale_over_m, out + (size_t)(2 * p) * 2 * M + k, M, overflow);
      if (2 * p + 1 < count) enc_round(x2, tws, scale_over_m, out + (size_t)(2 * p + 1) * 2 * M + k, M, overflow);
    }
  }
}

// integer coefficients -> coefficient-form residues out[p][limb][N] (blb_encode's result; plaintexts
// that go to evaluation form are reduced by their transforms)
__global__ void k_coef_residues(const long long* __restrict__ coef, uint64_t* __restrict__ out, int n, int nl, ModTable mt,
                                const int* __restrict__ overflow) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const int p = blockIdx.y;
  if (k >= n || *overflow) return;
  const uint64_t u = (uint64_t)coef[(size_t)p * n + k];
  for (int i = 0; i < nl; ++i) {
    const ModEntry me = mt.m[i];
    out[((size_t)p * nl + i) * n + k] = d2u(canon_full(i64_mod(u, me.q, me.qinv), me.q, me.qinv));
  }
}
void launch_coef_residues(blb_ctx* c, const uint64_t* coef, uint64_t* out, int count, int nl, const int* overflow) {
  dim3 grid((c->n + 255) / 256, count);
  emit(c, [=, stream = c->stream] { k_coef_residues<<<grid, 256, 0, stream>>>((const long long*)coef, out, c->n, nl, c->mt, overflow); });
}

// Encodes `count` plaintexts into integer coefficients coef[count][N] (int64; the DFT of the slot
// values from src, then twist, scale and rounding).  zbuf: [complex vectors][M][4].  clear: *d_overflow is
// zeroed first.
template <class Src>
int encode_with(blb_ctx* c, const Src& src, int count, double* zbuf, double scale, uint64_t* coef, int* d_overflow, bool paired, bool clear) {
  const int M = c->n / 2, M1 = M / kEncM2;
  if (M1 != 16 && M1 != 32 && M1 != 64) return BLB_EINVAL;  // M1 = 8 R2, R2 = 2, 4, 8; M1 >= kEncRB
  const int n_vec = paired ? (count + 1) / 2 : count;  // complex vectors transformed
  const dim3 gr(M1 / kEncRB, n_vec);
  int* const zero = clear ? d_overflow : nullptr;
  auto cols = [&](auto r2, auto cb) {
    constexpr int R2 = decltype(r2)::value, CB = decltype(cb)::value;
    emit(c, [=, stream = c->stream] {
      k_enc_cols<Src, R2, CB><<<dim3(kEncM2 / CB, n_vec), kEncThreads, 0, stream>>>(src, zbuf, c->d_enc_tw, M, zero);
    });
  };
  typedef std::integral_constant<int, 16> c16;
  const bool few = n_vec <= 32;  // 8 workgroups each: they fit the 256 CUs
  if (M1 == 64) cols(std::integral_constant<int, 8>{}, c16{});
  else if (M1 == 32 && few) cols(std::integral_constant<int, 4>{}, c16{});
  else if (M1 == 32) cols(std::integral_constant<int, 4>{}, std::integral_constant<int, 32>{});
  else if (few) cols(std::integral_constant<int, 2>{}, c16{});
  else cols(std::integral_constant<int, 2>{}, std::integral_constant<int, 64>{});
  const double sm = scale / (double)M;
  long long* out = (long long*)coef;
  if (paired)
    emit(c, [=, stream = c->stream] {
      k_enc_rows<true><<<gr, kEncRB * 16, 0, stream>>>(zbuf, c->d_enc_tw, c->d_enc_twist, sm, out, count, d_overflow, M, M1);
    });
  else
    emit(c, [=, stream = c->stream] {
      k_enc_rows<false><<<gr, kEncRB * 16, 0, stream>>>(zbuf, c->d_enc_tw, c->d_enc_twist, sm, out, count, d_overflow, M, M1);
    });
  return BLB_OK;
}
int run_encode_dense(blb_ctx* c, const double* vals, int n_vals, int count, double* zbuf, double scale, uint64_t* coef, int* d_overflow) {
  return encode_with(c, EncSrcDense{vals, n_vals, c->d_slot_inv}, count, zbuf, scale, coef, d_overflow, false, true);
}
int run_encode_block(blb_ctx* c, int block, double* zbuf, double scale, uint64_t* coef, int* d_overflow) {
  return encode_with(c, EncSrcBlock{block, c->d_slot_inv}, 1, zbuf, scale, coef, d_overflow, false, false);
}
int run_encode_cp(blb_ctx* c, const double* W, CpGeom g, int p0, int count, double* zbuf, double scale, uint64_t* coef, int* d_overflow,
                  CpDiag dg) {
  int lLp = 0;
  while ((1 << lLp) < g.Lp) ++lLp;
  return encode_with(c, EncSrcCp{W, g, p0, count, c->n / 2, lLp, c->d_slot_inv, dg}, count, zbuf, scale, coef, d_overflow, !g.cplx, false);
}

// ---------------------------------------------------------------------------------------
// matmul_cc helpers
// ---------------------------------------------------------------------------------------
// out = x (.) mx + y (.) my over a whole degree-1 ciphertext ([2][nl][N]); masks are
// evaluation-form plaintexts [nl][N] shared by both polys; y may be null.
__global__ void k_mask_pair(const CcPair* __restrict__ pairs, int nl, int n, ModTable mt) {
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= 2 * nl * n) return;
  const CcPair pr = pairs[blockIdx.y];
  const int mw = w % (nl * n);
  const ModEntry me = mt.m[mw / n];
  double r = mulmod_s(u2d(gmem(pr.x)[w]), u2d(gmem(pr.mx)[mw]), me.q, me.qinv);
  if (pr.y) r += mulmod_s(u2d(gmem(pr.y)[w]), u2d(gmem(pr.my)[mw]), me.q, me.qinv);
  gmem(pr.out)[w] = d2u(canon_full(r, me.q, me.qinv));
}
void launch_mask_pair(blb_ctx* c, const CcPair* pairs_dev, int n_pairs, int nl) {
  if (n_pairs <= 0) return;
  dim3 grid((2 * nl * c->n + 255) / 256, n_pairs);
  emit(c, [=, stream = c->stream] { k_mask_pair<<<grid, 256, 0, stream>>>(pairs_dev, nl, c->n, c->mt); });
}

// T3[t] = sum_a A_a (x) R[t][a]: degree-2 output (d0, d1, d2) at nl2 limbs.  A_a is at a
// higher level (nlA limbs per poly) and is used through its first nl2 limbs.
__global__ void k_tensor_sum(const uint64_t* const* __restrict__ A_tab, const uint64_t* const* __restrict__ R_tab,
                             uint64_t* __restrict__ T3, int n_ct, int nlA, int nl2, int n, ModTable mt, int a_per_t) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const int limb = blockIdx.y % nl2;
  const int t = blockIdx.y / nl2;
  if (k >= n) return;
  const ModEntry me = mt.m[limb];
  const double q = me.q, qi = me.qinv;
  double d0 = 0.0, d1 = 0.0, d2 = 0.0;
  for (int a = 0; a < n_ct; ++a) {
    const auto A = gmem(A_tab[a_per_t ? (size_t)t * n_ct + a : (size_t)a]);
    const auto R = gmem(R_tab[(size_t)t * n_ct + a]);
    const double a0 = u2d(A[(size_t)limb * n + k]), a1 = u2d(A[(size_t)(nlA + limb) * n + k]);
    const double r0 = u2d(R[(size_t)limb * n + k]), r1 = u2d(R[(size_t)(nl2 + limb) * n + k]);
    d0 += mulmod_s(a0, r0, q, qi);
    d1 += mulmod_s(a0, r1, q, qi) + mulmod_s(a1, r0, q, qi);
    d2 += mulmod_s(a1, r1, q, qi);
    if ((a & 1) == 1) {
      d0 = reduce_s(d0, q, qi);
      d1 = reduce_s(d1, q, qi);
      d2 = reduce_s(d2, q, qi);
    }
  }
  uint64_t* o = T3 + (size_t)t * 3 * nl2 * n;
  o[(size_t)limb * n + k] = d2u(canon_full(d0, q, qi));
  o[(size_t)(nl2 + limb) * n + k] = d2u(canon_full(d1, q, qi));
  o[(size_t)(2 * nl2 + limb) * n + k] = d2u(canon_full(d2, q, qi));
}
void launch_tensor_sum(blb_ctx* c, const uint64_t* const* A_tab, const uint64_t* const* R_tab, uint64_t* T3, int n_t, int n_ct, int nlA,
                       int nl2, bool a_per_t) {
  dim3 grid((c->n + 255) / 256, n_t * nl2);
  emit(c, [=, stream = c->stream] { k_tensor_sum<<<grid, 256, 0, stream>>>(A_tab, R_tab, T3, n_ct, nlA, nl2, c->n, c->mt, a_per_t ? 1 : 0); });
}

// The same sums for the BSGS schedule, where A'_{j,a} depends on the giant step only and Y_{a,i} on the
// baby step only: t = j Bb + i is a matrix of outputs, and a work-item takes TJ x TI of them, loading
// 2 (TJ + TI) words per a instead of 2 words of each operand per output.  One output at a time was
// bound by the operands' L2 traffic (9 TB/s); 4 x 4 outputs are bound by FP64 issue.  12 heads, 128 tokens,
// N = 16384, four limbs, 16 ciphertexts per operand: 348 us one at a time.
// A: [nj][m][2][nl][N] from the chunk's first giant step, Y: [Bb][m][2][nl][N], T3: [nj Bb][3][nl][N].
template <int TJ, int TI>
__global__ __launch_bounds__(256) void k_tensor_tile(const uint64_t* __restrict__ A, const uint64_t* __restrict__ Y,
                                                     uint64_t* __restrict__ T3, int m, int Bb, int nl, int n, ModTable mt) {
  typedef __attribute__((address_space(1))) const uint64_t gu64;
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const int limb = blockIdx.y % nl;
  const int tile = blockIdx.y / nl, i0 = tile % (Bb / TI) * TI, j0 = tile / (Bb / TI) * TJ;
  const ModEntry me = mt.m[limb];
  const double q = me.q, qi = me.qinv;
  const size_t poly = (size_t)nl * n, ct = 2 * poly;
  gu64* ap = (gu64*)(A + (size_t)j0 * m * ct + (size_t)limb * n);
  gu64* yp = (gu64*)(Y + (size_t)i0 * m * ct + (size_t)limb * n);
  double d0[TJ][TI], d1[TJ][TI], d2[TJ][TI];
#pragma unroll
  for (int j = 0; j < TJ; ++j)
#pragma unroll
    for (int i = 0; i < TI; ++i) d0[j][i] = d1[j][i] = d2[j][i] = 0.0;
  for (int a = 0; a < m; ++a) {
    double a0[TJ], a1[TJ], r0[TI], r1[TI];
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      gu64* x = ap + ((size_t)j * m + a) * ct;
      a0[j] = u2d(x[k]);
      a1[j] = u2d(x[poly + k]);
    }
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      gu64* x = yp + ((size_t)i * m + a) * ct;
      r0[i] = u2d(x[k]);
      r1[i] = u2d(x[poly + k]);
    }
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        d0[j][i] += mulmod_s(a0[j], r0[i], q, qi);
        d1[j][i] += mulmod_s(a0[j], r1[i], q, qi) + mulmod_s(a1[j], r0[i], q, qi);
        d2[j][i] += mulmod_s(a1[j], r1[i], q, qi);
      }
    if ((a & 3) == 3) {  // |d1| <= q/2 + 8 x 0.875 q = 7.5 q < 2^53
#pragma unroll
      for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int i = 0; i < TI; ++i) {
          d0[j][i] = reduce_s(d0[j][i], q, qi);
          d1[j][i] = reduce_s(d1[j][i], q, qi);
          d2[j][i] = reduce_s(d2[j][i], q, qi);
        }
    }
  }
#pragma unroll
  for (int j = 0; j < TJ; ++j)
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      uint64_t* o = T3 + ((size_t)(j0 + j) * Bb + i0 + i) * 3 * poly + (size_t)limb * n + k;
      o[0] = d2u(canon_full(d0[j][i], q, qi));
      o[poly] = d2u(canon_full(d1[j][i], q, qi));
      o[2 * poly] = d2u(canon_full(d2[j][i], q, qi));
    }
}
// false: the step counts are no multiples of a tile (the caller runs k_tensor_sum)
bool launch_tensor_tile(blb_ctx* c, const uint64_t* A, const uint64_t* Y, uint64_t* T3, int m, int nj, int Bb, int nl) {
#define TILE(tj, ti)                                                                                                              \
  if (nj % tj == 0 && Bb % ti == 0) {                                                                                             \
    const dim3 grid(c->n / 256, nj / tj * (Bb / ti) * nl);                                                                        \
    emit(c, [=, stream = c->stream] { k_tensor_tile<tj, ti><<<grid, 256, 0, stream>>>(A, Y, T3, m, Bb, nl, c->n, c->mt); });      \
    return true;                                                                                                                  \
  }
  TILE(4, 4)
  TILE(2, 2)
#undef TILE
  return false;
}

// out[o] (+)= sum over its terms of ct (.) mask, whole degree-1 ciphertexts at nl limbs
__global__ void k_masked_acc(const CcTerm* __restrict__ terms, const int* __restrict__ off, uint64_t* const* __restrict__ outs, int nl,
                             int n, ModTable mt, int accumulate) {
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  const int o = blockIdx.y;
  if (w >= 2 * nl * n) return;
  const int mw = w % (nl * n);
  const ModEntry me = mt.m[mw / n];
  const auto out = gmem(outs[o]);
  double acc = accumulate ? u2d(out[w]) : 0.0;
  int cnt = 0;
  for (int i = off[o]; i < off[o + 1]; ++i) {
    acc += mulmod_s(u2d(gmem(terms[i].ct)[w]), u2d(gmem(terms[i].mask)[mw]), me.q, me.qinv);
    if ((++cnt & 3) == 0) acc = reduce_s(acc, me.q, me.qinv);
  }
  out[w] = d2u(canon_full(acc, me.q, me.qinv));
}
void launch_masked_acc(blb_ctx* c, const CcTerm* terms, const int* off, uint64_t* const* outs, int n_out, int nl, bool accumulate) {
  if (n_out <= 0) return;
  dim3 grid((2 * nl * c->n + 255) / 256, n_out);
  emit(c, [=, stream = c->stream] { k_masked_acc<<<grid, 256, 0, stream>>>(terms, off, outs, nl, c->n, c->mt, accumulate ? 1 : 0); });
}

// ---------------------------------------------------------------------------------------
// Batched matmul_cp MAC over many independent instances (uneven lengths, several plans).
// Work item = (plan group, IB consecutive instances of the group, TB outputs, 256*CPT
// coefficients, one limb).  A persistent grid walks the item list with a grid stride; each
// plaintext word loaded is applied to IB instances' rotated inputs, so instances sharing a
// plan read its diagonals once per IB instances.
// ---------------------------------------------------------------------------------------
// The tile's tail (outputs past n_bj, instances past the group's last) is computed on clamped,
// in-bounds operands and not stored, so the inner loop has no branches.  Operands go through
// the global address space (pointer tables through scalar loads) and the next term's words are
// loaded while the current term is multiplied.
template <int TB, int IB, int CPT, bool P50>
__global__ __launch_bounds__(256) void k_cp_mac_batch(const MacGroup* __restrict__ groups, const MacItem* __restrict__ items, int n_items,
                                                      int n, ModTable mt) {
  typedef __attribute__((address_space(1))) const uint64_t gu64c;
  typedef __attribute__((address_space(1))) const u64x2 gu64x2c;
  typedef __attribute__((address_space(1))) uint64_t gu64;
  typedef __attribute__((address_space(4))) const uint64_t ku64;
  for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
    const MacItem item = items[it];
    const MacGroup gr = groups[item.group];
    const int k0 = (item.kb * 256 + threadIdx.x) * CPT;
    if (k0 >= n) continue;
    const Pt50Off off50 = pt50_off(n, k0);
    for (int limb = item.limb; limb < item.limb + item.n_limb; ++limb) {
    const int nl = gr.nl, n_ai = gr.n_ai, n_bj = gr.n_bj;
    const ModEntry me = mt.m[limb];
    const double q = me.q, qi = me.qinv;
    const int bj0 = item.tile * TB;
    const int ninst = min(IB, gr.n_inst - item.inst0);
    const size_t pb = pt_poly_bytes(n, P50);
    const size_t term = (size_t)nl * pb;  // bytes per (bj, ai) plaintext
    const uint8_t* pt[TB];
#pragma unroll
    for (int t = 0; t < TB; ++t) pt[t] = (const uint8_t*)gr.pt + (size_t)min(bj0 + t, n_bj - 1) * n_ai * term + (size_t)limb * pb;
    const ku64* rxtab[IB];  // row of rotated-input pointers of each instance
#pragma unroll
    for (int u = 0; u < IB; ++u) rxtab[u] = (const ku64*)(gr.rx + (size_t)(item.inst0 + min(u, ninst - 1)) * n_ai);
    Pt50Raw<CPT> rw[TB];
    uint64_t rq[TB][CPT];
    uint64_t rx0[IB][CPT], rx1[IB][CPT];  // raw words of the term in flight
    auto fetch = [&](int ai) {
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        if constexpr (P50) {
          pt50_fetch<CPT>(pt[t] + (size_t)ai * term, off50, rw[t]);
        } else {
          const gu64c* a = (const gu64c*)(pt[t] + (size_t)ai * term) + k0;
          if constexpr (CPT >= 2) {
#pragma unroll
            for (int c = 0; c < CPT; c += 2) {
              const u64x2 w = __builtin_nontemporal_load((const gu64x2c*)(a + c));
              rq[t][c] = w.x;
              rq[t][c + 1] = w.y;
            }
          } else {
            rq[t][0] = __builtin_nontemporal_load(a);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < IB; ++u) {
        const gu64c* x = (const gu64c*)rxtab[u][ai];
        if constexpr (CPT >= 2) {
#pragma unroll
          for (int c = 0; c < CPT; c += 2) {
            const u64x2 w0 = *(const gu64x2c*)(x + (size_t)limb * n + k0 + c);
            const u64x2 w1 = *(const gu64x2c*)(x + (size_t)(nl + limb) * n + k0 + c);
            rx0[u][c] = w0.x;
            rx0[u][c + 1] = w0.y;
            rx1[u][c] = w1.x;
            rx1[u][c + 1] = w1.y;
          }
        } else {
          rx0[u][0] = x[(size_t)limb * n + k0];
          rx1[u][0] = x[(size_t)(nl + limb) * n + k0];
        }
      }
    };
    double a0[IB][TB][CPT], a1[IB][TB][CPT];
#pragma unroll
    for (int u = 0; u < IB; ++u)
#pragma unroll
      for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int c = 0; c < CPT; ++c) { a0[u][t][c] = 0.0; a1[u][t][c] = 0.0; }
    fetch(0);
    for (int ai = 0; ai < n_ai; ++ai) {
      double w[TB][CPT], x0[IB][CPT], x1[IB][CPT];
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        if constexpr (P50) {
          pt50_cvt<CPT>(rw[t], k0, w[t]);
        } else {
#pragma unroll
          for (int c = 0; c < CPT; ++c) w[t][c] = u2d(rq[t][c]);
        }
      }
#pragma unroll
      for (int u = 0; u < IB; ++u)
#pragma unroll
        for (int c = 0; c < CPT; ++c) { x0[u][c] = u2d(rx0[u][c]); x1[u][c] = u2d(rx1[u][c]); }
      fetch(min(ai + 1, n_ai - 1));  // the last term re-reads itself
#pragma unroll
      for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int u = 0; u < IB; ++u)
#pragma unroll
          for (int c = 0; c < CPT; ++c) {
            a0[u][t][c] += mulmod_s(w[t][c], x0[u][c], q, qi);
            a1[u][t][c] += mulmod_s(w[t][c], x1[u][c], q, qi);
          }
      if ((ai & 7) == 7) {  // 8 products below 0.875q each on a reduced |acc| <= q/2: |acc| < 7.5q < 2^53
#pragma unroll
        for (int u = 0; u < IB; ++u)
#pragma unroll
          for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int c = 0; c < CPT; ++c) { a0[u][t][c] = reduce_s(a0[u][t][c], q, qi); a1[u][t][c] = reduce_s(a1[u][t][c], q, qi); }
      }
    }
#pragma unroll
    for (int u = 0; u < IB; ++u) {
      if (u >= ninst) continue;
      gu64* out = (gu64*)gr.inner[item.inst0 + u];
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        if (bj0 + t < n_bj) {
          gu64* o0 = out + (((size_t)(bj0 + t) * 2 + 0) * nl + limb) * n + k0;
          gu64* o1 = out + (((size_t)(bj0 + t) * 2 + 1) * nl + limb) * n + k0;
#pragma unroll
          for (int c = 0; c < CPT; ++c) {
            o0[c] = d2u(canon_full(a0[u][t][c], q, qi));
            o1[c] = d2u(canon_full(a1[u][t][c], q, qi));
          }
        }
      }
    }
    }  // limbs of the item
  }
}

// The MAC of IB instances that share a plan, each plaintext word loaded once for all of them:
// TB outputs x IB instances x one coefficient per work-item.  Bound by FP64 issue from three
// instances on (7.4 instructions per product: 5.9e9 products of 4 instances take 2.6 ms, 2.8 T/s),
// by HBM with two (12 outputs: 5.2 TB/s of plan words).  A group's instances are split into runs of
// 2..4 of near equal size, each size its own launch, so no work-item computes an instance that is
// not there (the run-time tail of a fixed 4 x 2 shape did: 5 instances ran as 6, at 2.1 T/s).
template <int TB, int IB, bool P50>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_cp_mac_multi(const MacGroup* __restrict__ groups,
                                                                                              const MacSeg* __restrict__ segs, int n_seg,
                                                                                              int n, int n_kblk, ModTable mt) {
  typedef __attribute__((address_space(1))) const uint64_t gu64c;
  typedef __attribute__((address_space(1))) uint64_t gu64;
  typedef __attribute__((address_space(4))) const uint64_t ku64;
  int s = 0;
  while (s + 1 < n_seg && (int)blockIdx.x >= segs[s + 1].first) ++s;
  const MacSeg seg = segs[s];
  const MacGroup gr = groups[seg.group];
  const int nl = gr.nl, n_ai = gr.n_ai, n_bj = gr.n_bj;
  const int b = blockIdx.x - seg.first;
  const int kb = b % n_kblk, limb = (b / n_kblk) % nl, bj0 = b / (n_kblk * nl) * TB;
  const int k0 = kb * 256 + threadIdx.x;
  const ModEntry me = mt.m[limb];
  const double q = me.q, qi = me.qinv;
  const Pt50Off off50 = pt50_off(n, k0);
  const size_t pb = pt_poly_bytes(n, P50);
  const size_t term = (size_t)nl * pb;  // bytes per (bj, ai) plaintext
  const uint8_t* pt[TB];                // rows past the last re-read it (not stored)
#pragma unroll
  for (int t = 0; t < TB; ++t) pt[t] = (const uint8_t*)gr.pt + (size_t)min(bj0 + t, n_bj - 1) * n_ai * term + (size_t)limb * pb;
  const ku64* rxtab[IB];
#pragma unroll
  for (int u = 0; u < IB; ++u) rxtab[u] = (const ku64*)(gr.rx + (size_t)(seg.inst0 + u) * n_ai);
  Pt50Raw<1> w50[TB];
  uint64_t w64[TB], r0[IB], r1[IB];
  auto fetch = [&](int ai) {
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      const uint8_t* poly = pt[t] + (size_t)ai * term;
      if constexpr (P50) pt50_fetch<1>(poly, off50, w50[t]);
      else w64[t] = __builtin_nontemporal_load((gu64c*)poly + k0);
    }
#pragma unroll
    for (int u = 0; u < IB; ++u) {
      gu64c* x = (gu64c*)rxtab[u][ai];
      r0[u] = x[(size_t)limb * n + k0];
      r1[u] = x[(size_t)(nl + limb) * n + k0];
    }
  };
  double a0[IB][TB], a1[IB][TB];
#pragma unroll
  for (int u = 0; u < IB; ++u)
#pragma unroll
    for (int t = 0; t < TB; ++t) a0[u][t] = a1[u][t] = 0.0;
  fetch(0);
  for (int ai = 0; ai < n_ai; ++ai) {
    double w[TB], x0[IB], x1[IB];
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      if constexpr (P50) {
        double v[1];
        pt50_cvt<1>(w50[t], k0, v);
        w[t] = v[0];
      } else {
        w[t] = u2d(w64[t]);
      }
    }
#pragma unroll
    for (int u = 0; u < IB; ++u) {
      x0[u] = u2d(r0[u]);
      x1[u] = u2d(r1[u]);
    }
    fetch(min(ai + 1, n_ai - 1));  // the last term re-reads itself
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
      for (int u = 0; u < IB; ++u) {
        a0[u][t] += mulmod_s(w[t], x0[u], q, qi);
        a1[u][t] += mulmod_s(w[t], x1[u], q, qi);
      }
    if ((ai & 7) == 7) {  // 8 products below 0.875 q on |acc| <= q/2: |acc| < 7.5 q < 2^53
#pragma unroll
      for (int u = 0; u < IB; ++u)
#pragma unroll
        for (int t = 0; t < TB; ++t) {
          a0[u][t] = reduce_s(a0[u][t], q, qi);
          a1[u][t] = reduce_s(a1[u][t], q, qi);
        }
    }
  }
#pragma unroll
  for (int u = 0; u < IB; ++u) {
    gu64* out = (gu64*)gr.inner[seg.inst0 + u];
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      if (bj0 + t < n_bj) {
        out[(((size_t)(bj0 + t) * 2 + 0) * nl + limb) * n + k0] = d2u(canon_full(a0[u][t], q, qi));
        out[(((size_t)(bj0 + t) * 2 + 1) * nl + limb) * n + k0] = d2u(canon_full(a1[u][t], q, qi));
      }
    }
  }
}
int mac_multi_rows(int ib) { return ib == 2 ? 12 : 8; }
bool launch_cp_mac_multi(blb_ctx* c, const MacGroup* groups, const MacSeg* segs, int n_seg, int blocks, int ib, int p50) {
#define MULTI(tb_, ib_)                                                                                                        \
  if (ib == ib_) {                                                                                                             \
    if (p50) emit(c, [=, stream = c->stream] { k_cp_mac_multi<tb_, ib_, true><<<blocks, 256, 0, stream>>>(groups, segs, n_seg, c->n, c->n / 256, c->mt); }); \
    else emit(c, [=, stream = c->stream] { k_cp_mac_multi<tb_, ib_, false><<<blocks, 256, 0, stream>>>(groups, segs, n_seg, c->n, c->n / 256, c->mt); }); \
    return true;                                                                                                               \
  }
  MULTI(12, 2)
  MULTI(8, 3)
  MULTI(8, 4)
#undef MULTI
  return false;
}

int batch_mac_shape(int variant, int* tb, int* ib, int* cpt) {
  switch (variant) {
    case 2: *tb = 2; *ib = 4; *cpt = 2; break;
    case 3: *tb = 4; *ib = 4; *cpt = 1; break;
    case 4: *tb = 8; *ib = 2; *cpt = 1; break;
    case 5: *tb = 8; *ib = 4; *cpt = 1; break;
    case 6: *tb = 4; *ib = 8; *cpt = 1; break;
    case 7: *tb = 4; *ib = 4; *cpt = 2; break;
    case 8: *tb = 8; *ib = 2; *cpt = 2; break;
    default: *tb = 4; *ib = 1; *cpt = 2; break;
  }
  return 0;
}

void launch_cp_mac_batch(blb_ctx* c, const MacGroup* groups, const MacItem* items, int n_items, int variant, int grid, int p50) {
  if (n_items <= 0) return;
  int tb, ib, cpt;
  batch_mac_shape(variant, &tb, &ib, &cpt);
  const int blocks = std::min(n_items, grid);
#define MB(a, b, d)                                                                                   \
  do {                                                                                                \
    if (p50) emit(c, [=, stream = c->stream] { k_cp_mac_batch<a, b, d, true><<<blocks, 256, 0, stream>>>(groups, items, n_items, c->n, c->mt); });  \
    else emit(c, [=, stream = c->stream] { k_cp_mac_batch<a, b, d, false><<<blocks, 256, 0, stream>>>(groups, items, n_items, c->n, c->mt); }); \
  } while (0)
  if (tb == 2 && ib == 4) MB(2, 4, 2);
  else if (tb == 4 && ib == 4 && cpt == 1) MB(4, 4, 1);
  else if (tb == 8 && ib == 2 && cpt == 1) MB(8, 2, 1);
  else if (tb == 8 && ib == 4) MB(8, 4, 1);
  else if (tb == 4 && ib == 8) MB(4, 8, 1);
  else if (tb == 4 && ib == 4) MB(4, 4, 2);
  else if (tb == 8 && ib == 2) MB(8, 2, 2);
  else MB(4, 1, 2);
#undef MB
}

// out[o] = sum of its terms (offsets per output), whole ciphertexts of `words` u64 each
__global__ void k_sum_var(const uint64_t* const* __restrict__ srcs, const int* __restrict__ off, uint64_t* const* __restrict__ dsts,
                          int n, int nl, ModTable mt) {
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  const int o = blockIdx.y;
  if (w >= 2 * nl * n) return;
  const ModEntry me = mt.m[(w / n) % nl];
  double acc = 0.0;
  int cnt = 0;
  for (int t = off[o]; t < off[o + 1]; ++t) {
    acc += u2d(gmem(srcs[t])[w]);
    if ((++cnt & 3) == 0) acc = reduce_s(acc, me.q, me.qinv);
  }
  gmem(dsts[o])[w] = d2u(canon_full(acc, me.q, me.qinv));
}
void launch_sum_var(blb_ctx* c, const uint64_t* const* srcs, const int* off, uint64_t* const* dsts, int n_out, int nl) {
  if (n_out <= 0) return;
  dim3 grid((2 * nl * c->n + 255) / 256, n_out);
  emit(c, [=, stream = c->stream] { k_sum_var<<<grid, 256, 0, stream>>>(srcs, off, dsts, c->n, nl, c->mt); });
}

// out[t] = k * in[t] for whole degree-1 ciphertexts (exact integer scalar, every limb); in[t]
// may hold more limbs per poly (nl_in) than out keeps (nl): the extra limbs are dropped
__global__ void k_scale_cts(const uint64_t* const* __restrict__ in, uint64_t* __restrict__ out, int n, int nl, int nl_in, double k,
                            ModTable mt) {
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  const int t = blockIdx.y;
  if (w >= 2 * nl * n) return;
  const int limb = (w / n) % nl, poly = w / (nl * n);
  const ModEntry me = mt.m[limb];
  const size_t src = ((size_t)poly * nl_in + limb) * n + (w % n);
  out[(size_t)t * 2 * nl * n + w] = d2u(canon(mulmod_s(u2d(gmem(in[t])[src]), k, me.q, me.qinv), me.q));
}
void launch_scale_cts(blb_ctx* c, const uint64_t* const* in, uint64_t* out, int count, int nl, double k, int nl_in) {
  if (count <= 0) return;
  dim3 grid((2 * nl * c->n + 255) / 256, count);
  emit(c, [=, stream = c->stream] { k_scale_cts<<<grid, 256, 0, stream>>>(in, out, c->n, nl, nl_in > nl ? nl_in : nl, k, c->mt); });
}
