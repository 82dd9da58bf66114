// Device building blocks of the matrix-core contraction (see apc_gemm.hip for
// the layout of its operands) and of its elementwise epilogues.  Shared by the
// single-plan kernels (apc_gemm.hip) and the persistent batch kernel that mixes
// k-RHS contractions with k = 1 systems (apc_batch.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "apc_internal.h"

namespace apc {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Element type of an FP32 contraction on the bf16 matrix cores (see Split3):
// a float whose V operands are stored split.
struct F32x3 {
  float v;
  F32x3() = default;
  __device__ explicit F32x3(float f) : v(f) {}
};

template <typename T>
struct TnTraits;
template <>
struct TnTraits<F32x3> {
  using Acc = f32x4;
  using Part = float;
};
template <>
struct TnTraits<__bf16> {
  using Acc = f32x4;
  using Part = float;
};
template <>
struct TnTraits<float> {
  using Acc = f32x4;
  using Part = float;
};
template <>
struct TnTraits<double> {
  using Acc = f64x4;
  using Part = double;
};

// MFMA over one 16-byte piece of A (lane's row) and B (lane's right-hand side).
__device__ inline void mma_bf16(const u32x4& a, const u32x4& b, f32x4& c) {
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                              __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ inline void mma_piece(const u32x4& a, const u32x4& b, f32x4& c, __bf16*) { mma_bf16(a, b, c); }
__device__ inline void mma_piece(const u32x4& a, const u32x4& b, f32x4& c, float*) {
  const f32x4 av = __builtin_bit_cast(f32x4, a);
  const f32x4 bv = __builtin_bit_cast(f32x4, b);
#pragma unroll
  for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], bv[e], c, 0, 0, 0);
}
__device__ inline void mma_piece(const u32x4& a, const u32x4& b, f64x4& c, double*) {
  const f64x2 av = __builtin_bit_cast(f64x2, a);
  const f64x2 bv = __builtin_bit_cast(f64x2, b);
#pragma unroll
  for (int e = 0; e < 2; ++e) c = __builtin_amdgcn_mfma_f64_16x16x4f64(av[e], bv[e], c, 0, 0, 0);
}

// FP32 operands on the bf16 matrix cores.  An FP32 value is the exact sum of
// three bf16 values: h and m are the value and the remainder rounded to bf16, l
// is what is left (at most 7 significant bits, so exact).  A product is then
// h h' + h m' + m h' + m m' + h l' + l h' in FP32 accumulation; the three left
// out (m l', l m', l l') are together below 2^-24 of it, which is what rounding
// a product to FP32 may cost: over 4 million random pairs 2^-24.2 at most and
// 2^-27.5 rms.  (h truncated instead leaves an m twice as long, of the value's
// sign: 2^-22.2 and 2^-25.5, and rows of few entries then err by up to 1.6 FP32
// roundings in one direction.)
// Exact from 2^-110 on, below which l falls under bf16's range (2^-112: off by
// 4e-7, 2^-120 by 6e-5): the rows of an operand far from 1 are stored scaled
// (launch_tn_operand).  Infinities, NaN and what rounds to a bf16 infinity
// (from 2^128 - 2^119 on) give NaN.  The FP32 matrix instructions run at 1/16 of the bf16 rate, so six
// products take 3/8 of their time; the errors of long sums against 64 bits
// measured 0.3-0.85 of theirs (fewer roundings per sum).  With 16 right-
// hand sides a pass is bound by reading M, not by its products, and the FP32
// instructions stay (T = float): splitting cost 4-15 % there (5120^2: 18.1
// against 17.3 us).
struct Split3 {
  u32x4 h, m, l;  // eight bf16 each
};
typedef float f32x2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
__device__ inline void split_pair(float x0, float x1, unsigned& h, unsigned& m, unsigned& l) {
  h = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2v{x0, x1}, bf16x2v));
  const float r0 = x0 - __uint_as_float(h << 16);
  const float r1 = x1 - __uint_as_float(h & 0xffff0000u);
  m = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2v{r0, r1}, bf16x2v));
  const float s0 = r0 - __uint_as_float(m << 16);
  const float s1 = r1 - __uint_as_float(m & 0xffff0000u);
  l = __builtin_amdgcn_perm(__float_as_uint(s1), __float_as_uint(s0), 0x07060302u);  // upper halves
}
__device__ inline Split3 split8(const u32x4& a, const u32x4& b) {
  const f32x4 av = __builtin_bit_cast(f32x4, a), bv = __builtin_bit_cast(f32x4, b);
  Split3 s;
  unsigned h, m, l;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    split_pair(av[2 * e], av[2 * e + 1], h, m, l);
    s.h[e] = h;
    s.m[e] = m;
    s.l[e] = l;
    split_pair(bv[2 * e], bv[2 * e + 1], h, m, l);
    s.h[2 + e] = h;
    s.m[2 + e] = m;
    s.l[2 + e] = l;
  }
  return s;
}

// The V operand (one row of K entries per right-hand side).  bf16, FP32 and
// FP64: row-major, 256 bytes per row and step.  F32x3: split when it is written, 384
// bytes per row and step of 64: the h, m and l parts of the step, 128 bytes
// each, every part in the order the lanes take it (chunk kc = 8 q + 4 h + g of
// four entries at 32 q + 8 g + 4 h, so lane group g's eight entries of the
// matrix product q, its pieces 2 q and 2 q + 1 of M, are 16 contiguous bytes).
// A workgroup stages a step in wave loads of kRows rows x 16 kLanes
// contiguous bytes (kParts of them cover a row).
template <typename T>
struct TnOperand {
  static constexpr bool kSplit = std::is_same_v<T, F32x3>;
  static constexpr int kStepBytes = kSplit ? 384 : 256;
  static constexpr int kLanes = kSplit ? 8 : 16;
  static constexpr int kRows = 64 / kLanes;
  static constexpr int kParts = kStepBytes / (16 * kLanes);
};

// V staging of one workgroup: two steps of 16 NCT rows, each row's 16-byte
// chunks + 1 pad (fragment reads, 16 rows at one chunk, are conflict-free).
template <typename T, int NCT>
struct TnStage {
  u32x4 v[2][NCT * 16][TnOperand<T>::kStepBytes / 16 + 1];
};

// Element offset of (row r, column c) in the fragment-packed layout of a
// rows x K operand (rows % 16 == 0, K a multiple of the step).
template <typename T>
__host__ __device__ inline int64_t frag_index(int64_t r, int64_t c, int64_t rows) {
  constexpr int kE = 16 / sizeof(T);
  constexpr int kStep = 16 * kE;
  const int64_t ks = c / kStep;
  const int kc = static_cast<int>((c % kStep) / kE);   // 16-byte chunk in the step
  const int lane = static_cast<int>(r % 16) + 16 * (kc % 4);
  return (ks * (rows / 16) + r / 16) * (16 * kStep) + (64 * (kc / 4) + lane) * kE + c % kE;
}

// What bounds it.  FP32, 16384^2, k = 128: 505 us per pass on the FP32 matrix
// instructions (86 % of their rate), 312-343 us here, bound by power: a launch is
// 579 thousand cycles of an XCD whatever the data, 283 us at the 2.0 GHz of a
// cool chip and up to 375 at the 1.5 GHz that a run of them falls to (1.07 GB of
// M would take 165 us).  8192^2, k = 64: 75 -> 53-63 us (268 MB of M, 4.3-5.1
// TB/s).  bf16 and FP64: HBM, and the FP64 matrix rate from 64 right-hand
// sides on.
//
// Workgroup: W waves (4 or 8), wave w owns RT consecutive 16-row tiles, all
// 16*NCT right-hand sides of its column group.  Grid: (rows / (16 W RT)) x ncg x nsplit,
// with the split index fastest so that, dealt round-robin over the 8 XCDs, one
// XCD works on one split (nsplit | 8) and keeps that split's V in its L2.
template <typename T, int RT, int NCT, int PF, int NT, int W = 4>
__device__ inline void tn_block(const TnArgs& a, int bid, TnStage<T, NCT>& vs) {
  static_assert(W == 4 || W == 8, "waves per workgroup");
  using Op = TnOperand<T>;
  constexpr int kUnits = NCT * 16 / Op::kRows * Op::kParts;  // wave loads per step of V
  constexpr int VU = (kUnits + W - 1) / W;                    // of them each wave's
  using Acc = typename TnTraits<T>::Acc;
  using Part = typename TnTraits<T>::Part;
  constexpr int kE = 16 / sizeof(T);  // elements per 16-byte piece
  constexpr int kStep = 16 * kE;      // elements per row per step (256 bytes)
  const int ncg = a.kp / (16 * NCT);
  int q = bid;
  const int split = q % a.nsplit;
  q /= a.nsplit;
  const int cg = q % ncg;
  const int64_t rtile = q / ncg;
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int li = lane & 15, g = lane >> 4;
  const int64_t kb0 = static_cast<int64_t>(split) * a.klen;
  const int64_t kend = min(a.K, kb0 + a.klen);
  const int nsteps = kend > kb0 ? static_cast<int>((kend - kb0) / kStep) : 0;
  const T* M = static_cast<const T*>(a.M);
  const int64_t vrow = a.ldv / kStep * Op::kStepBytes;  // bytes of one V row
  const char* V = static_cast<const char*>(a.V) + static_cast<int64_t>(cg) * NCT * 16 * vrow +
                  kb0 / kStep * Op::kStepBytes;
  const int64_t rb = rtile * 16 * W * RT + static_cast<int64_t>(wv) * 16 * RT;

  // Fragment-packed M: this wave's tile t of step s starts at
  // ((kb0 / kStep + s) * rows / 16 + rb / 16 + t) * 16 * kStep, and lane L's
  // piece p sits (64 p + L) * kE further on.
  const int64_t sstride = a.rows * kStep;
  const T* mrow[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
    mrow[t] = M + (kb0 / kStep) * sstride + (rb + 16 * t) * kStep + lane * kE;
  // Wave w stages the units w, w + W, ... of a step (the last round repeats a
  // unit where they do not divide evenly): the unit's offset is uniform, a
  // lane adds its row's and its chunk's.
  const int vrl = lane / Op::kLanes, vcl = lane % Op::kLanes;
  const uint32_t vlane = static_cast<uint32_t>(vrl * vrow) + 16 * vcl;
  const int swv = __builtin_amdgcn_readfirstlane(wv);
  int vunit[VU];
#pragma unroll
  for (int u = 0; u < VU; ++u) vunit[u] = min(swv + W * u, kUnits - 1);

  Acc acc[RT][NCT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) acc[t][ct] = Acc{};
  // Units u0 .. u0 + n - 1 of the wave's share of a step of V.
  auto load_v = [&](u32x4* vst, int step, int u0, int n) {
    const char* src = V + static_cast<int64_t>(step) * Op::kStepBytes;
#pragma unroll
    for (int u = 0; u < n; ++u) {
      const int w = vunit[u0 + u];
      const char* unit = src + (w / Op::kParts) * (Op::kRows * vrow) + (w % Op::kParts) * 16 * Op::kLanes;
      vst[u] = *reinterpret_cast<const u32x4*>(unit + vlane);
    }
  };
  auto store_v = [&](const u32x4* vst, int buf, int u0, int n) {
#pragma unroll
    for (int u = 0; u < n; ++u) {
      const int w = vunit[u0 + u];
      vs.v[buf][(w / Op::kParts) * Op::kRows + vrl][(w % Op::kParts) * Op::kLanes + vcl] = vst[u];
    }
  };
  // A split past the end of K (from rounding its length up to whole steps)
  // writes zero partials.
  if constexpr (Op::kSplit) {
    if (nsteps > 0) {
      // A step is two phases (matrix products over 32 of its 64 columns).  In
      // phase k the raw pieces of phase k + 1 are split while the products of
      // phase k run, and those of phase k + R are loaded into the slot that
      // phase k's were split from: R - 1 = 2 PF + 1 phases of M in flight.
      // The loops are unrolled by the ring (PF + 1 steps), so every slot is a
      // compile-time constant.  In the main loop every load is issued without
      // a branch (a load behind one makes the compiler wait for all loads in
      // flight where the paths join); the tail loads only what exists.  With
      // two row tiles and 128 right-hand sides (or four) the tail's branches cost
      // spilled registers: there the main loop runs to the end and a step past
      // the split's end reloads its last one.
      constexpr bool kTail = RT == 1 || (RT == 2 && NCT < 8);
      constexpr int D = PF + 1, R = 2 * D;
      // The next step of V is staged in two halves, one per phase, where its
      // registers are short (128 right-hand sides; VU is even there).
      constexpr int HV = NCT >= 8 ? 2 : 1, VH = VU / HV;
      // Where the registers allow, the small products have sums of their own,
      // added at the end: the large sums are then rounded once per 32 columns
      // instead of six times (the error of long sums falls by about two).
      constexpr bool kLow = RT * NCT <= 8;
      Acc low[kLow ? RT : 1][kLow ? NCT : 1];
#pragma unroll
      for (auto& r : low)
#pragma unroll
        for (auto& v : r) v = Acc{};
      u32x4 raw[R][RT][2], vst[VU];
      Split3 ms[2][RT];
      auto load_m = [&](u32x4 (&dst)[RT][2], int step, int q) {
        const int64_t o = static_cast<int64_t>(step) * sstride;
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            const u32x4* src = reinterpret_cast<const u32x4*>(mrow[t] + o + (2 * q + p) * 64 * kE);
            dst[t][p] = NT ? __builtin_nontemporal_load(src) : *src;
          }
      };
      const int last = nsteps - 1;
      load_v(vst, 0, 0, VU);
#pragma unroll
      for (int k = 0; k < R; ++k) load_m(raw[k], min(k / 2, last), k & 1);
      store_v(vst, 0, 0, VU);
#pragma unroll
      for (int t = 0; t < RT; ++t) ms[0][t] = split8(raw[0][t][0], raw[0][t][1]);
      __syncthreads();
      auto step_body = [&](int step, int i, bool more, bool load_ahead) {
        const int buf = step & 1;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int k = 2 * i + q;
          // V before M: loads complete in order, so the wait for V leaves the
          // M loads behind it in flight.
          if (q < HV && more) load_v(vst, kTail ? step + 1 : min(step + 1, last), q * VH, VH);
          __builtin_amdgcn_sched_barrier(0);
          if (load_ahead) load_m(raw[k], kTail ? step + D : min(step + D, last), q);
          __builtin_amdgcn_sched_barrier(0);
          u32x4 vf[2][3];
#pragma unroll
          for (int e = 0; e < 3; ++e) vf[0][e] = vs.v[buf][li][8 * e + 4 * q + g];
#pragma unroll
          for (int t = 0; t < RT; ++t)
            ms[q ^ 1][t] = split8(raw[(k + 1) % R][t][0], raw[(k + 1) % R][t][1]);
#pragma unroll
          for (int ct = 0; ct < NCT; ++ct) {
            if (ct + 1 < NCT) {
#pragma unroll
              for (int e = 0; e < 3; ++e)
                vf[(ct + 1) & 1][e] = vs.v[buf][(ct + 1) * 16 + li][8 * e + 4 * q + g];
            }
            // The small products first.
            const u32x4* v = vf[ct & 1];
            auto mul = [&](u32x4 Split3::*part, const u32x4& b, bool small) {
#pragma unroll
              for (int t = 0; t < RT; ++t) {
                if constexpr (kLow) {
                  if (small) {
                    mma_bf16(ms[q][t].*part, b, low[t][ct]);
                    continue;
                  }
                }
                mma_bf16(ms[q][t].*part, b, acc[t][ct]);
              }
            };
            mul(&Split3::l, v[0], true);
            mul(&Split3::h, v[2], true);
            mul(&Split3::m, v[1], true);
            mul(&Split3::m, v[0], true);
            mul(&Split3::h, v[1], true);
            mul(&Split3::h, v[0], false);
          }
          // Interleave: the next column tile's LDS reads and a share of the
          // next phase's splitting between the products of each tile.
          constexpr int kValu = (42 * RT + 3 * NCT - 1) / (3 * NCT);
          __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);  // LDS reads
#pragma unroll
          for (int ct = 0; ct < NCT; ++ct) {
            if (ct + 1 < NCT) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
#pragma unroll
            for (int r = 0; r < 3; ++r) {
              __builtin_amdgcn_sched_group_barrier(0x008, 2 * RT, 0);  // matrix products
              __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);  // vector instructions
            }
          }
          __builtin_amdgcn_sched_barrier(0);
          if (more && (HV == 2 || q == 1)) store_v(vst, buf ^ 1, HV == 2 ? q * VH : 0, VH);
        }
        __syncthreads();
      };
      int step0 = 0;
      if constexpr (kTail) {
        for (; step0 + D - 1 + D < nsteps; step0 += D) {
#pragma unroll
          for (int i = 0; i < D; ++i) step_body(step0 + i, i, true, true);
        }
        for (; step0 < nsteps; step0 += D) {
#pragma unroll
          for (int i = 0; i < D; ++i)
            if (step0 + i < nsteps)
              step_body(step0 + i, i, step0 + i + 1 < nsteps, step0 + i + D < nsteps);
        }
      } else {
        for (; step0 < nsteps; step0 += D) {
#pragma unroll
          for (int i = 0; i < D; ++i) {
            if (i > 0 && step0 + i >= nsteps) break;
            step_body(step0 + i, i, true, true);
          }
        }
      }
      if constexpr (kLow) {
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
          for (int ct = 0; ct < NCT; ++ct) acc[t][ct] += low[t][ct];
      }
    }
  } else {
  // Ring of PF + 1 register sets for M: the loads for step s + PF are issued
  // while step s computes.  The step loop is unrolled by the ring size so that
  // every slot index is a compile-time constant.
  constexpr int D = PF + 1;
  u32x4 mr[D][RT][4], vst[VU];
  auto load_m = [&](u32x4 (&dst)[RT][4], int step) {
    const int64_t o = static_cast<int64_t>(step) * sstride;
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const u32x4* src = reinterpret_cast<const u32x4*>(mrow[t] + o + p * 64 * kE);
        dst[t][p] = NT ? __builtin_nontemporal_load(src) : *src;
      }
  };
  // Every load below is issued without a branch, so that the compiler can
  // count the loads in flight (see the main part); a step past the split's
  // end is replaced by its last step.
  if (nsteps > 0) {
#pragma unroll
  for (int s0 = 0; s0 < PF; ++s0) load_m(mr[s0], min(s0, nsteps - 1));
  load_v(vst, 0, 0, VU);
  store_v(vst, 0, 0, VU);
  __syncthreads();
  // One step: V's next step and M's step + PF are loaded, step `step` is
  // multiplied from ring slot i, V's next step goes to the other LDS buffer.
  // V is loaded before M: loads complete in order, so the wait for V at the
  // end of the step does not also wait for the newest M loads, which keep PF
  // steps in flight.
  auto body = [&](int step, int i, bool more, bool load_ahead) {
    const int buf = step & 1;
    if (more) load_v(vst, step + 1, 0, VU);
    if (load_ahead) load_m(mr[(i + PF) % D], step + PF);
    // Keep the loads at the top of the step: moved down among the products
    // they would be waited for as soon as they are issued.
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      u32x4 bf[NCT];
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) bf[ct] = vs.v[buf][ct * 16 + li][4 * p + g];
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct)
          mma_piece(mr[i][t][p], bf[ct], acc[t][ct], static_cast<T*>(nullptr));
    }
    if (more) store_v(vst, buf ^ 1, 0, VU);
    __syncthreads();
  };
  // Main part: every step of the chunk has step + PF < nsteps, so both loads
  // are issued without a branch.  A load behind a branch makes the compiler
  // wait for every load in flight where the paths join (it cannot count the
  // loads issued after V's), which would drain the prefetch each step.
  int step0 = 0;
  // (Both loops are unrolled by the ring size, so every slot index is a
  // compile-time constant.)
  for (; step0 + D - 1 + PF < nsteps; step0 += D) {
#pragma unroll
    for (int i = 0; i < D; ++i) body(step0 + i, i, true, true);
  }
  // Tail: the last steps, loads only where they exist (uniform branches).
  for (; step0 < nsteps; step0 += D) {
#pragma unroll
    for (int i = 0; i < D; ++i)
      if (step0 + i < nsteps) body(step0 + i, i, step0 + i + 1 < nsteps, step0 + i + PF < nsteps);
  }
  }  // nsteps > 0
  }

  // Result layout: f32 accumulators hold D[4 g + q][li]; f64 ones D[g + 4 q][li].
  Part* part = static_cast<Part*>(a.part);
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      const int c = cg * NCT * 16 + ct * 16 + li;
      Part* dst = part + (static_cast<int64_t>(split) * a.kp + c) * a.ldp + rb + 16 * t;
      if constexpr (sizeof(Part) == 8) {
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) dst[g + 4 * qq] = acc[t][ct][qq];
      } else {
        *reinterpret_cast<f32x4*>(dst + 4 * g) = acc[t][ct];
      }
    }
}


template <typename T>
__device__ inline T cvt(double v);
template <>
__device__ inline double cvt<double>(double v) { return v; }
template <>
__device__ inline float cvt<float>(double v) { return static_cast<float>(v); }
template <>
__device__ inline F32x3 cvt<F32x3>(double v) { return F32x3(static_cast<float>(v)); }
template <>
__device__ inline __bf16 cvt<__bf16>(double v) { return static_cast<__bf16>(static_cast<float>(v)); }

// The same, times the row's scale where the operand has one.
template <typename T>
__device__ inline T cvt_scaled(double v, double qs) {
  if constexpr (TnOperand<T>::kSplit) return cvt<T>(v * qs);
  else return cvt<T>(v);
}

template <typename P>
__device__ inline double split_sum(const P* part, int32_t nsplit, int64_t split_stride, int64_t idx) {
  P s = part[idx];
  for (int sp = 1; sp < nsplit; ++sp) s += part[sp * split_stride + idx];
  return static_cast<double>(s);
}

// Four consecutive entries as one or two 16-byte accesses (8 bytes for bf16);
// the address is a multiple of four entries, 16-byte aligned.
template <typename T>
__device__ inline void load4(const T* p, T (&v)[4]) {
  if constexpr (sizeof(T) == 4) {
    const f32x4 w = *reinterpret_cast<const f32x4*>(p);
    __builtin_memcpy(v, &w, 16);
  } else {
    const f64x2 w0 = reinterpret_cast<const f64x2*>(p)[0];
    const f64x2 w1 = reinterpret_cast<const f64x2*>(p)[1];
    v[0] = w0[0];
    v[1] = w0[1];
    v[2] = w1[0];
    v[3] = w1[1];
  }
}
template <typename T>
__device__ inline void store4(T* p, const T (&v)[4]) {
  if constexpr (sizeof(T) == 2) {
    uint2 w;
    __builtin_memcpy(&w, v, 8);
    *reinterpret_cast<uint2*>(p) = w;
  } else if constexpr (sizeof(T) == 4) {
    f32x4 w;
    __builtin_memcpy(&w, v, 16);
    *reinterpret_cast<f32x4*>(p) = w;
  } else {
    reinterpret_cast<f64x2*>(p)[0] = f64x2{v[0], v[1]};
    reinterpret_cast<f64x2*>(p)[1] = f64x2{v[2], v[3]};
  }
}

// Four consecutive entries j .. j + 3 (j % 4 == 0) of row c of a V operand of
// row length ld (a multiple of the step): row-major, or split (F32x3).
template <typename TQ>
__device__ inline void store_operand4(TQ* base, int64_t ld, int64_t c, int64_t j, const TQ (&v)[4]) {
  if constexpr (TnOperand<TQ>::kSplit) {
    unsigned h[2], m[2], l[2];
    split_pair(v[0].v, v[1].v, h[0], m[0], l[0]);
    split_pair(v[2].v, v[3].v, h[1], m[1], l[1]);
    const int kc = static_cast<int>(j >> 2) & 15;
    char* d = reinterpret_cast<char*>(base) + (c * (ld >> 6) + (j >> 6)) * 384 +
              64 * (kc >> 3) + 16 * (kc & 3) + 8 * ((kc >> 2) & 1);
    *reinterpret_cast<uint2*>(d) = make_uint2(h[0], h[1]);
    *reinterpret_cast<uint2*>(d + 128) = make_uint2(m[0], m[1]);
    *reinterpret_cast<uint2*>(d + 256) = make_uint2(l[0], l[1]);
  } else {
    store4(base + c * ld + j, v);
  }
}

// W's row c, entries r .. r + 3 as a V operand: the sum of the split partials
// in split order, for e = c * rows + r (e, rows and ldp multiples of 4: the
// four share one right-hand side).
template <typename P, typename TQ>
__device__ inline void sum_cast4(const P* part, int32_t nsplit, int64_t ldp, int64_t rows,
                                 int64_t stride, TQ* out, int64_t ldo, int64_t e) {
  const int64_t c = e / rows, r = e - c * rows;
  P s[4];
  load4(part + c * ldp + r, s);
  for (int sp = 1; sp < nsplit; ++sp) {
    P t[4];
    load4(part + sp * stride + c * ldp + r, t);
#pragma unroll
    for (int q = 0; q < 4; ++q) s[q] += t[q];
  }
  TQ o[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) o[q] = TQ(s[q]);
  store_operand4(out, ldo, c, r, o);
}

// The (y, x_bar) update, its start, or an anchor update (see TnUpdateArgs)
// for the four entries (c, j .. j + 3), j and the strides multiples of 4, from
// their summed products z.  y1 = (1 - gamma) y + gamma x_bar; an anchor update
// (mode 2, z = m X y1 in FP64) reads the copy y_ref its product was formed
// from and becomes the new anchor, an update in between has
// z = m X~ (y1 - y_ref).  The state is loaded apart from its use, so that a
// contraction can load it before its products.
struct UpdateState {
  double xb[4], x0[4], y[4], yr[4], ur[4];  // y: y_ref in an anchor update
  double2 scale;
};
// kAll: load every field without a branch (absent anchors read y instead, and
// are not used), so that the loads can stay in flight.
template <typename TQ, bool kAll>
__device__ inline void update_load(const TnUpdateArgs& a, int64_t c, int64_t j, UpdateState& s) {
  const int64_t i = c * a.ldx + j;
  const double* y = a.mode == 2 ? a.yref : a.y;
  if constexpr (TnOperand<TQ>::kSplit) s.scale = a.scale[c];
  load4(a.xb + i, s.xb);
  load4(a.x0 + i, s.x0);
  load4(y + i, s.y);
  if (kAll || (a.mode == 0 && a.yref)) {
    load4((kAll && !a.yref ? y : a.yref) + i, s.yr);
    load4((kAll && !a.uref ? y : a.uref) + i, s.ur);
  }
}
template <typename TQ>
__device__ inline void update_quad(const TnUpdateArgs& a, int64_t c, int64_t j, const UpdateState& s,
                                   const double (&z)[4]) {
  TQ* yq = static_cast<TQ*>(a.yq);
  const double g = a.gamma, omg = 1.0 - a.gamma, eta = a.eta, ome = 1.0 - a.eta;
  const int64_t i = c * a.ldx + j;
  TQ qv[4];
  if (a.mode == 1) {
    double x0[4], zero[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      x0[q] = z[q] * a.inv_m;
      qv[q] = cvt_scaled<TQ>(g * x0[q], s.scale.x);
    }
    store4(a.x0 + i, x0);
    store4(a.xb + i, x0);
    store4(a.y + i, zero);
    if (a.yref) {
      store4(a.yref + i, zero);
      store4(a.uref + i, zero);
    }
    store_operand4(yq, a.ldq, c, j, qv);
    return;
  }
  double yo[4], xo[4], uo[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double y1 = a.mode == 2 ? s.y[q] : omg * s.y[q] + g * s.xb[q];
    double u = z[q] * a.inv_m;
    double ref = 0.0;
    if (a.mode == 2) {
      uo[q] = u;
      ref = y1;
    } else if (a.yref) {
      u += s.ur[q];
      ref = s.yr[q];
    }
    const double xn = eta * (s.x0[q] + y1 - u) + ome * s.xb[q];
    yo[q] = y1;
    xo[q] = xn;
    qv[q] = cvt_scaled<TQ>(omg * y1 + g * xn - ref, s.scale.x);
  }
  if (a.mode == 2) store4(a.uref + i, uo);
  store4(a.y + i, yo);
  store4(a.xb + i, xo);
  store_operand4(yq, a.ldq, c, j, qv);
}

// The same for e = c * n + j, from the split partials (n and ldp multiples of 4).
template <typename P, typename TQ>
__device__ inline void update4(const TnUpdateArgs& a, int64_t e) {
  const int64_t stride = static_cast<int64_t>(a.kp) * a.ldp;
  const P* part = static_cast<const P*>(a.part);
  const int64_t c = e / a.n, j = e - c * a.n;
  P zs[4];
  load4(part + c * a.ldp + j, zs);
  for (int sp = 1; sp < a.nsplit; ++sp) {
    P t[4];
    load4(part + sp * stride + c * a.ldp + j, t);
#pragma unroll
    for (int q = 0; q < 4; ++q) zs[q] += t[q];
  }
  UpdateState s;
  update_load<TQ, false>(a, c, j, s);
  const double f = sizeof(P) == 4 && a.scale ? a.scale[c].y : 1.0;
  const double z[4] = {static_cast<double>(zs[0]) * f, static_cast<double>(zs[1]) * f,
                       static_cast<double>(zs[2]) * f, static_cast<double>(zs[3]) * f};
  update_quad<TQ>(a, c, j, s, z);
}

// One reverse step of the (y, x_bar) iteration (see TnAdjointArgs) for the
// four entries (c, j .. j + 3) from their summed products z; adds their shares
// of the dL/dgamma and dL/deta sums.
struct AdjointState {
  double a[4], bh[4], g0[4], y[4], xb[4], xn[4];
  double2 scale;
};
template <typename TQ>
__device__ inline void adjoint_load(const TnAdjointArgs& a, int64_t c, int64_t j, AdjointState& s) {
  const int64_t i = c * a.ldx + j;
  if constexpr (TnOperand<TQ>::kSplit) s.scale = a.scale[c];
  load4(a.a + i, s.a);
  load4(a.bh + i, s.bh);
  load4(a.g0 + i, s.g0);
  load4(a.y_t + i, s.y);
  load4(a.xb_t + i, s.xb);
  load4(a.xb_next + i, s.xn);
}
template <typename TQ>
__device__ inline void adjoint_quad(const TnAdjointArgs& a, int64_t c, int64_t j, AdjointState& s,
                                    const double (&z)[4], double& sg, double& se) {
  const int64_t i = c * a.ldx + j;
  TQ qv[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double zq = TnOperand<TQ>::kSplit ? z[q] * s.scale.y : z[q];
    const double xbh = zq * a.inv_m;  // X b
    const double bh = s.bh[q];
    const double at = s.a[q] + a.eta * (bh - xbh);
    sg += at * (s.xb[q] - s.y[q]);
    se += bh * (s.xn[q] - s.xb[q]);
    s.g0[q] += a.eta * bh;
    s.a[q] = (1.0 - a.gamma) * at;
    s.bh[q] = (1.0 - a.eta) * bh + a.gamma * at;
    qv[q] = cvt_scaled<TQ>(s.bh[q], s.scale.x);
  }
  store4(a.g0 + i, s.g0);
  store4(a.a + i, s.a);
  store4(a.bh + i, s.bh);
  store_operand4(static_cast<TQ*>(a.bq), a.ldq, c, j, qv);
}

}  // namespace

}  // namespace apc
