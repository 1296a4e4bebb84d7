// First-order Shapley values: phi[s, f] accumulated over every root-to-leaf
// path of the ensemble (Theorem 1 with |S| = 1, Eq. 9-10, 8 nodes), and the
// adjoint of phi with respect to the leaf values.
//
// Work mapping (gfx950, wave64):
//   * a workgroup owns a tile of 64 explained samples (one per lane) and a
//     contiguous chunk of rows from one bucket; its wavefronts split the
//     chunk (rows of at most 8 features: one contiguous run per wavefront;
//     longer rows: row by row in turn);
//   * a wavefront processes one row at a time for all 64 samples, so every
//     row quantity (features, bounds, b_j, 1-b_j, slot-0 factor) is uniform
//     across the wave and is fetched with scalar loads;
//   * the sample tile is staged transposed in LDS ([F][65] floats), so the
//     per-lane gather x[s, f_j] is a conflict-free LDS read;
//   * contributions are added into an FP64 LDS accumulator ([F][65] doubles,
//     shared by the workgroup's waves) and flushed to the FP64 global
//     accumulator with one atomic per (sample, feature) at the end.
//
// Per (sample, row) with unique features j = 0..d-1 and nodes m:
//   o_j    = x in [lo_j, hi_j) ? 1 : 0   (NaN: missing_ok_j)            (Eq. 2)
//   c_j    = o_j - b_j, taken as the stored FP64-derived 1 - b_j or as -b_j
//   F_j(m) = b_j (1 - t_m) + o_j t_m = b_j + t_m c_j      (one FMA per node)
//   LOO_j  = sum_m w_m prod_{k != j} F_k(m)    by prefix x suffix products
//   phi[s, f_j] += val c_j LOO_j
// The leaf value is folded into slot 0 (Slot0: F_0 scaled by val, built per
// call in FP64), so a row needs no multiply by val; a merged sibling pair is
// the same form with a combined slot-0 factor.
// At 8 nodes, rows of at most 8 features in FP64 and, with the model's own leaf
// values, longer rows in FP32 are walked by their node products, phi_j = sum_m
// H(m) c_j / F_j(m) with quotients that do not depend on the sample, H summed
// over neighbouring rows that share the slot (values_rows_grouped,
// values_rows_batched).  A few samples take a lane per row
// (values_lane_kernel).  The other calls walk row by row (WALK >= kPerRow):
// rows of at most 8 features reuse the factors and prefix products of the slots
// they share with the previous row (values_rows_shared, adjoint_rows_shared);
// longer rows (values_rows_long, adjoint_paths) run in batches of eight slots:
// slots past the end of a row get c = 0 and b = 1, a factor of exactly 1, so
// whole batches run without branches; the prefix products are kept only at
// batch checkpoints and rebuilt batch by batch in the backward sweep, which
// bounds the registers; NH < NN splits the nodes over several passes (the node
// sum is additive).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "../qts_device.h"

namespace qts {

template <typename T>
__device__ __forceinline__ T fmaT(T a, T b, T c) {
  return __builtin_fma(a, b, c);
}
template <>
__device__ __forceinline__ float fmaT<float>(float a, float b, float c) {
  return __builtin_fmaf(a, b, c);
}

// Copy a wave-uniform value into a VGPR the compiler cannot fold back.
__device__ __forceinline__ float to_vgpr(float v) {
  float r;
  asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "s"(v));
  return r;
}
__device__ __forceinline__ double to_vgpr(double v) {
  double r;
  asm volatile("v_mov_b64 %0, %1" : "=v"(r) : "s"(v));
  return r;
}

// Node m and weight m of the 8-node rule in the walks that hold all 8 nodes
// in one pass: FP32 takes them as instruction literals, FP64 from the kernel
// argument (an FP32 FMA or multiply reading a scalar register issues at about
// half the rate of one with a literal or vector operands; FP64 shows no such
// difference).
template <typename T>
__device__ __forceinline__ T node8_t(const NodeConsts<T>& nc, int m) {
  if constexpr (sizeof(T) == 4) return rule8_t32(m);
  else return nc.t[m];
}
template <typename T>
__device__ __forceinline__ T node8_w(const NodeConsts<T>& nc, int m) {
  if constexpr (sizeof(T) == 4) return rule8_w32(m);
  else return nc.w[m];
}

// Add to a leaf's gradient in memory.  det: grad_leaf is this sample block's
// own row of partial sums, and every leaf belongs to one row, so a plain store
// suffices (and keeps the result independent of scheduling).
__device__ __forceinline__ void leaf_add(double* grad_leaf, int leaf, double v, bool det) {
  if (det) grad_leaf[leaf] = v;
  else if (v != 0.0) unsafeAtomicAdd(&grad_leaf[leaf], v);
}

// Leaf A (which = 0) or B (1) of a row; -1: a single path has no B.
__device__ __forceinline__ int leaf_of(const PathHdr* hdr, const SidePath* side, int row,
                                       int which) {
  if (which == 0) return hdr[row].leaf;
  const int sidx = side == nullptr ? -1 : hdr[row].tree;
  return sidx < 0 ? -1 : side[sidx].leaf_b;
}

// Sums the rows' leaf gradients over the wave's 64 samples and adds them to the workgroup's LDS sums,
// part[2 (row - pb) + which], or without them (part null) to memory.
struct LeafSums {
  double* part;
  double* grad_leaf;
  const PathHdr* hdr;
  const SidePath* side;
  int pb, lane;
  bool det;
  double u_prev = 0.0, w_prev = 0.0;  // rows of the four that wait

  // One row at a time (no registers to let rows wait).
  __device__ __forceinline__ void add_row(double a, double b, int row) const {
    double z = fold16(fold32(a, b), 0.0);
    z += dpp_lanes<0x128>(z);
    z += dpp_lanes<0x141>(z);
    z += dpp_lanes<0xb1>(z);
    z += dpp_lanes<0x4e>(z);
    if ((lane & 31) == 0) put(z, row, lane >> 5);
  }

  __device__ __forceinline__ void put(double z, int row, int which) const {
    if (part != nullptr) {
      __hip_atomic_fetch_add(&part[2 * (row - pb) + which], z, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WORKGROUP);
    } else {
      const int leaf = leaf_of(hdr, side, row, which);
      if (leaf >= 0) leaf_add(grad_leaf, leaf, z, det);
    }
  }

  // Four rows together; a, b: leaf A's and B's terms of row `row`, the i-th of the wave's
  // consecutive rows; last: no row follows
  __device__ __forceinline__ void add(double a, double b, int i, int row, bool last) {
    const double ab = fold32(a, b);
    const int q = i & 3;
    if ((q & 1) == 0 && !last) {
      u_prev = ab;
      return;
    }
    const double w = (q & 1) ? fold16(u_prev, ab) : fold16(ab, 0.0);
    if (q < 2 && !last) {
      w_prev = w;
      return;
    }
    const double z = q < 2 ? wave_sum8(w, 0.0, lane) : wave_sum8(w_prev, w, lane);
    const int v = wave_sum8_index(lane);
    if ((lane & 7) != 0 || (v >> 1) > q) return;
    put(z, row - (q - (v >> 1)), v & 1);
  }
};

// The adjoint's path loop for rows of more than 8 features, and for FP64 tiles
// with an infinite gradient.  NANS: the tile holds a NaN, so the missing-value
// rule is evaluated; otherwise plain interval tests suffice.  phi is linear in the leaf value, so
// d phi[s, f_j] / d val = c_j LOO_j: each lane gathers g[s, f_j] c_j LOO_j from
// the upstream-gradient tile gs, and the wave sums its 64 samples in FP64.
template <typename T, int DMAX, int NH, bool STORE_G, bool NANS, int NN>
__device__ __forceinline__ void adjoint_paths(
    const PathHdr* __restrict__ hdr, const int32_t* __restrict__ feat,
    const float* __restrict__ lo, const float* __restrict__ hi, const T* __restrict__ bb,
    const T* __restrict__ cbb, const SidePath* __restrict__ side,
    const float* xs, const T* gs, LeafSums sums, int pb, int pe, int wave, int nw, int lane,
    const T* tv, const NodeConsts<T>& nc) {
  constexpr int NB = DMAX / 8;  // feature batches
  for (int p = pb + wave; p < pe; p += nw) {
    const int d = ldu(&hdr[p].d);
    const int off = ldu(&hdr[p].off);
    // A merged sibling pair:
    // slot 0 is the parent's split feature L, made inert in the products
    // (b = 1, c = 0), so the sweep yields w Q_j(m) = w prod_{k >= 1, k != j} F_k(m);
    // then
    //   d/dvA = sum_m F_A(m) R(m) + g_L c_A sum_m w Q_0(m),
    //   R(m) = sum_{j >= 1} g_j c_j w Q_j(m)   (shared by A and B),
    // and likewise for B with F_B and c_B.
    const int sidx = side == nullptr ? -1 : ldu(&hdr[p].tree);
    const bool merged = sidx >= 0;  // slot 0 not taken from the row's elements
    T ba = T(0), cba = T(0), bb2 = T(0), cbb2 = T(0);
    float loB = 0.f, hiB = 0.f;
    bool mokB = false;
    if (merged) {
      const SidePath* sp = side + sidx;
      loB = ldu(&sp->lo_b);
      hiB = ldu(&sp->hi_b);
      mokB = ldu(&sp->mok_b) != 0;
      ba = (T)ldu(&sp->b_a);
      cba = (T)ldu(&sp->cb_a);
      bb2 = (T)ldu(&sp->b_b);
      cbb2 = (T)ldu(&sp->cb_b);
    }
    // b_j of slot j (slot 0 of a merged path: 1, inert)
    auto bload = [&](int j) -> T { return (j == 0 && merged) ? T(1) : ldu(bb + off + j); };
    double gacc = 0.0;
    double gaccB = 0.0;          // a merged path: B's gradient
    T oc0A = T(0), oc0B = T(0);  // a merged path: c_A and c_B
    T q0 = T(0);                 // a merged path: sum_m w Q_0(m)
    const int nb = (d + 7) >> 3;  // batches in use; slots [d, 8 nb) are inert

    // c_j per slot, eight slots per batch
    T cf[DMAX];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (b < nb) {
        const int jb = 8 * b;
        int fm[8];
        float l[8], u[8], x[8];
        T bl[8], cbl[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          fm[k] = ldu(feat + off + jb + k);
          l[k] = ldu(lo + off + jb + k);
          u[k] = ldu(hi + off + jb + k);
          bl[k] = ldu(bb + off + jb + k);
          cbl[k] = ldu(cbb + off + jb + k);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = xs[(fm[k] & kFeatureMask) * kTileStride + lane];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          // hi = NaN (no upper bound) makes the upper compare true; a NaN x
          // passes the unordered lower compare iff missing_ok
          bool lower;
          if (NANS) {
            const bool miss = (fm[k] & kMissingOkBit) != 0;
            lower = miss ? !(x[k] < l[k]) : (x[k] >= l[k]);
          } else {
            lower = x[k] >= l[k];
          }
          const bool upper = !(x[k] >= u[k]);
          cf[jb + k] = (lower & upper) ? cbl[k] : -bl[k];
          if (b == 0 && k == 0 && merged) {
            bool lowerB;
            if (NANS) lowerB = mokB ? !(x[0] < loB) : (x[0] >= loB);
            else lowerB = x[0] >= loB;
            const bool upperB = !(x[0] >= hiB);
            oc0A = (lower & upper) ? cba : -ba;
            oc0B = (lowerB & upperB) ? cbb2 : -bb2;
            cf[0] = T(0);
          }
        }
      }
    }

#pragma unroll
    for (int pass = 0; pass < NN / NH; ++pass) {
      const int m0 = pass * NH;
      // checkpoints: ck[b][m] = w_m prod_{k < 8b} F_k(m)
      T ck[NB][NH];
#pragma unroll
      for (int m = 0; m < NH; ++m) ck[0][m] = nc.w[m0 + m];
#pragma unroll
      for (int b = 1; b < NB; ++b) {
        if (b < nb) {
#pragma unroll
          for (int m = 0; m < NH; ++m) ck[b][m] = ck[b - 1][m];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const int j = 8 * (b - 1) + k;
            const T bj = bload(j);
#pragma unroll
            for (int m = 0; m < NH; ++m) ck[b][m] *= fmaT(tv[m0 + m], cf[j], bj);
          }
        }
      }
      // backward sweep, last batch first: rebuild the batch's prefixes from
      // its checkpoint, then suffix products and leave-one-out sums
      T S[NH];
#pragma unroll
      for (int m = 0; m < NH; ++m) S[m] = T(1);
      T R[NH];
#pragma unroll
      for (int m = 0; m < NH; ++m) R[m] = T(0);
#pragma unroll
      for (int b = NB - 1; b >= 0; --b) {
        if (b < nb) {
          const int jb = 8 * b;
          T bj[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) bj[k] = bload(jb + k);
          T Pb[8][NH];
          T Gb[STORE_G ? 8 : 1][NH];
          T run[NH];
#pragma unroll
          for (int m = 0; m < NH; ++m) run[m] = ck[b][m];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
#pragma unroll
            for (int m = 0; m < NH; ++m) {
              const T g = fmaT(tv[m0 + m], cf[jb + k], bj[k]);
              Pb[k][m] = run[m];
              if (STORE_G) Gb[STORE_G ? k : 0][m] = g;
              run[m] *= g;
            }
          }
#pragma unroll
          for (int k = 7; k >= 0; --k) {
            const int j = jb + k;
            if (j < d) {
              const int f = ldu(feat + off + j) & kFeatureMask;
              if (merged) {
                if (j > 0) {
                  const T gc = gs[f * kTileStride + lane] * cf[j];
#pragma unroll
                  for (int m = 0; m < NH; ++m)
                    R[m] = fmaT(gc, Pb[k][m] * S[m], R[m]);
                } else {
#pragma unroll
                  for (int m = 0; m < NH; ++m) q0 = fmaT(Pb[k][m], S[m], q0);
                }
              } else {
                T dot = Pb[k][0] * S[0];
#pragma unroll
                for (int m = 1; m < NH; ++m) dot = fmaT(Pb[k][m], S[m], dot);
                gacc += (double)(gs[f * kTileStride + lane] * cf[j] * dot);
              }
            }
            if (j > 0) {
#pragma unroll
              for (int m = 0; m < NH; ++m) {
                const T g = STORE_G ? Gb[STORE_G ? k : 0][m] : fmaT(tv[m0 + m], cf[j], bj[k]);
                S[m] *= g;
              }
            }
          }
        }
      }
      if (merged) {
        T sa = T(0), sb = T(0);
#pragma unroll
        for (int m = 0; m < NH; ++m) {
          sa = fmaT(fmaT(tv[m0 + m], oc0A, ba), R[m], sa);
          sb = fmaT(fmaT(tv[m0 + m], oc0B, bb2), R[m], sb);
        }
        gacc += (double)sa;
        gaccB += (double)sb;
      }
    }
    if (merged) {
      const T gL = gs[(ldu(feat + off) & kFeatureMask) * kTileStride + lane];
      gacc += (double)(gL * oc0A * q0);
      gaccB += (double)(gL * oc0B * q0);
    }
    sums.add_row(gacc, gaccB, p);
  }
}


// Wide scalar loads of a ShortRow (dword-aligned vectors of 4 and 16 words).
typedef int32_t row_v4 __attribute__((ext_vector_type(4), aligned(4)));
typedef int32_t row_v16 __attribute__((ext_vector_type(16), aligned(4)));
static_assert(offsetof(ShortRow<float>, xoff) == 16 && offsetof(ShortRow<float>, lo) == 80 &&
                  offsetof(ShortRow<float>, b) == 144 && offsetof(ShortRow<float>, cb) == 176 &&
                  offsetof(ShortRow<double>, b) == 144 && offsetof(ShortRow<double>, cb) == 208,
              "ShortRow layout");

// A short row in registers (SGPRs: every field is wave-uniform).
template <typename T>
struct ShortRowRegs {
  int d, share, mok;
  int xo[8], ao[8];
  float l[8], u[8];
  T bl[8], cbl[8];
};

// The record of row p in four wide scalar loads, all issued before any is
// used.
template <typename T>
__device__ __forceinline__ ShortRowRegs<T> load_short_row(const ShortRow<T>* rows, int row0,
                                                          int p) {
  ShortRowRegs<T> r;
  const int32_t* rw = reinterpret_cast<const int32_t*>(rows + (p - row0));
  const row_v4 hd = ldu(reinterpret_cast<const row_v4*>(rw));
  const row_v16 of = ldu(reinterpret_cast<const row_v16*>(rw + 4));
  const row_v16 bd = ldu(reinterpret_cast<const row_v16*>(rw + 20));
  if constexpr (sizeof(T) == 4) {
    const row_v16 bc = ldu(reinterpret_cast<const row_v16*>(rw + 36));
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      r.bl[k] = __int_as_float(bc[k]);
      r.cbl[k] = __int_as_float(bc[8 + k]);
    }
  } else {
    const row_v16 b2 = ldu(reinterpret_cast<const row_v16*>(rw + 36));
    const row_v16 c2 = ldu(reinterpret_cast<const row_v16*>(rw + 52));
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      r.bl[k] = __hiloint2double(b2[2 * k + 1], b2[2 * k]);
      r.cbl[k] = __hiloint2double(c2[2 * k + 1], c2[2 * k]);
    }
  }
  r.d = hd[0];
  r.share = hd[1];
  r.mok = hd[2];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    r.xo[k] = of[k];
    r.ao[k] = of[8 + k];
    r.l[k] = __int_as_float(bd[k]);
    r.u[k] = __int_as_float(bd[8 + k]);
  }
  return r;
}

// First order over rows of at most 8 features with all NH nodes in one pass,
// reusing work between consecutive rows.  Each wave walks a contiguous run of
// rows.  The products are taken over the slots in the order 1, 2, ..., 7, 0,
// so the prefix products and the factors F_j(m) of slots 1..s depend only on
// those slots; when slots 1..s of a row equal the previous row's (share[p] =
// s, from the host), their c_j, F_j(m) and prefix products are still in
// registers and only their suffix products and dot products are formed
// again.  Slot 0 (the row's own factor, from Slot0) and slots past s are
// evaluated as usual, each with the prefix product through it in the same
// step, so the shared count picks one entry into a single straight run of
// code; inert padding slots (b = 1, c = 0) give a factor of exactly 1.
// ND: slots 1..ND of the bucket's rows can be real; the slots past it are inert
// in every row, and leaving out a factor of exactly 1 changes no bit.
// KEEP = false: nothing kept from row to row, so a row is one run of code
// without branches, which a wavefront alone on its SIMD walks faster
// (deterministic FP64 calls: 300 trees of depth 8, 100 features, 5003 rows 50.7
// ms, 59.9 with what is shared kept; 66.3 by values_rows_grouped, whose rows
// wait for scalar loads of their coefficients).
template <typename T, int NH, int ND, bool NANS, bool KEEP>
__device__ __forceinline__ void values_rows_shared(
    const ShortRow<T>* __restrict__ rows, int row0, const Slot0<T>* __restrict__ z0,
    const float* xs, double* as, int pb, int pe, int wave, int nw, int lane, const T* tv,
    const NodeConsts<T>& nc) {
  constexpr bool kScalarT = NH == 8;
  // the last slot whose prefix product is formed: slot 7's is only summed
  constexpr int kLastP = ND < 7 ? ND : 6;
  // 1 in a register the compiler knows nothing of: slot 0's node sum stays a
  // chain of FMAs on the rounded prefix products, as with ND = 7
  T one = T(1);
  asm volatile("" : "+v"(one));
  const int run = (pe - pb + nw - 1) / nw;
  const int p_first = pb + wave * run;
  const int p_last = min(pe, p_first + run);
  T cf[ND + 1];  // c_j of the current row
  T G[ND + 1][NH];  // F_j(m) of the current row
  // prefix products in the order 1..7, 0: P[q] = w prod over the first q
  // slots of that order (slot q + 1 at position q); P[1..s] depend only on
  // shared slots and are kept from the previous row
  T P[ND + 1][NH];
#pragma unroll
  for (int m = 0; m < NH; ++m) P[0][m] = kScalarT ? node8_w(nc, m) : nc.w[m];
  const char* xl = reinterpret_cast<const char*>(xs + lane);
  char* al = reinterpret_cast<char*>(as + lane);
  for (int p = p_first; p < p_last; ++p) {
    // the record and slot 0, all loads issued before any is used.  An empty
    // row (d = 0) is walked too: its slots are inert and its Slot0 factor
    // is 0, so it adds exact zeros.
    const ShortRowRegs<T> r = load_short_row<T>(rows, row0, p);
    const Slot0<T>* z = z0 + p;
    const T bm = ldu(&z->bm);
    const T cA = ldu(&z->ca);
    const T cB = ldu(&z->cb);
    const float loB = ldu(&z->lo_b);
    const float hiB = ldu(&z->hi_b);
    const bool mokB = ldu(&z->mok_b) != 0;
    const int d = r.d;
    const int s = KEEP && p != p_first ? r.share : 0;
    const int mok = r.mok;
    const auto& xo = r.xo;
    const auto& ao = r.ao;
    const auto& l = r.l;
    const auto& u = r.u;
    const auto& bl = r.bl;
    const auto& cbl = r.cbl;
    float x[ND + 1];
#pragma unroll
    for (int k = 0; k <= ND; ++k) x[k] = *reinterpret_cast<const float*>(xl + xo[k]);
#pragma unroll
    for (int k = 0; k <= ND; ++k) {
      if (k == 0 || k > s) {
        bool lower;
        if (NANS) {
          const bool miss = ((mok >> k) & 1) != 0;
          lower = miss ? !(x[k] < l[k]) : (x[k] >= l[k]);
        } else {
          lower = x[k] >= l[k];
        }
        const bool in = lower & !(x[k] >= u[k]);
        // b in a VGPR once: the select's -b and the factor FMAs read it
        // there (a VALU op reads one SGPR, and the select's mask is one)
        const T b = k == 0 ? bm : bl[k];
        const T bv = kScalarT ? to_vgpr(b) : b;
        T c;
        if (k == 0) {
          bool lowerB;
          if (NANS) lowerB = mokB ? !(x[0] < loB) : (x[0] >= loB);
          else lowerB = x[0] >= loB;
          const bool inB = lowerB & !(x[0] >= hiB);
          c = in ? cA : (inB ? cB : -bv);
        } else {
          c = in ? cbl[k] : -bv;
        }
        cf[k] = c;
        if (kScalarT) {
          // t as FP32 literals, or from SGPRs (FP64)
#pragma unroll
          for (int m = 0; m < NH; ++m) G[k][m] = fmaT(node8_t(nc, m), c, bv);
        } else {
#pragma unroll
          for (int m = 0; m < NH; ++m) G[k][m] = fmaT(tv[m], c, b);
        }
        // the prefix through this slot (every later slot is evaluated too)
        if (k >= 1 && k <= kLastP) {
#pragma unroll
          for (int m = 0; m < NH; ++m) P[k][m] = P[k - 1][m] * G[k][m];
        }
      }
    }
    // slot 0, last in the order: its leave-one-out product is that of slots
    // 1..ND (P[6] F_7 for ND = 7)
    {
      T dot = P[kLastP][0] * (ND < 7 ? one : G[ND][0]);
#pragma unroll
      for (int m = 1; m < NH; ++m)
        dot = fmaT(P[kLastP][m], ND < 7 ? one : G[ND][m], dot);
      __hip_atomic_fetch_add(reinterpret_cast<double*>(al + ao[0]), (double)(cf[0] * dot),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    // slots ND..1: suffix products, starting from slot 0's factor.  A full
    // row (most rows of full trees) takes a sweep without the
    // per-slot test of j < d.
    T S[NH];
#pragma unroll
    for (int m = 0; m < NH; ++m) S[m] = G[0][m];
    auto sweep = [&](auto full) __attribute__((always_inline)) {
#pragma unroll
      for (int q = ND - 1; q >= 0; --q) {
        const int j = q + 1;
        if (decltype(full)::value || j < d) {
          T dot = P[q][0] * S[0];
#pragma unroll
          for (int m = 1; m < NH; ++m) dot = fmaT(P[q][m], S[m], dot);
          const double c = (double)(cf[j] * dot);
          __hip_atomic_fetch_add(reinterpret_cast<double*>(al + ao[j]), c, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if (q > 0) {
#pragma unroll
          for (int m = 0; m < NH; ++m) S[m] *= G[j][m];
        }
      }
    };
    if (d == ND + 1) sweep(std::true_type{});
    else sweep(std::false_type{});
  }
}

// A select by a lane mask held in scalar registers (one bit per lane): b
// where the lane's bit is set, else a.
template <typename T>
__device__ __forceinline__ T pick(uint64_t mask, T a, T b) {
  return __builtin_amdgcn_inverse_ballot_w64(mask) ? b : a;
}

// f(integral_constant 0), ..., f(integral_constant N - 1), and downwards.
template <int N, class F, int I = 0>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, F, I + 1>(static_cast<F&&>(f));
  }
}
template <int N, class F>
__device__ __forceinline__ void static_for_down(F&& f) {
  if constexpr (N > 0) {
    f(std::integral_constant<int, N - 1>{});
    static_for_down<N - 1, F>(static_cast<F&&>(f));
  }
}

typedef float acc_v4 __attribute__((ext_vector_type(4)));

// acc[i] += sum_m A[4 (8 G + m) + i] H[m] per lane: block 8 G + m of the
// 4x4x1 product's A operand, broadcast to all 16 blocks of four samples.
template <int G>
__device__ __forceinline__ acc_v4 node_sums4(float A, const float (&H)[8], acc_v4 acc) {
  acc = __builtin_amdgcn_mfma_f32_4x4x1f32(A, H[0], acc, 4, 8 * G + 0, 0);
  acc = __builtin_amdgcn_mfma_f32_4x4x1f32(A, H[1], acc, 4, 8 * G + 1, 0);
  acc = __builtin_amdgcn_mfma_f32_4x4x1f32(A, H[2], acc, 4, 8 * G + 2, 0);
  acc = __builtin_amdgcn_mfma_f32_4x4x1f32(A, H[3], acc, 4, 8 * G + 3, 0);
  acc = __builtin_amdgcn_mfma_f32_4x4x1f32(A, H[4], acc, 4, 8 * G + 4, 0);
  acc = __builtin_amdgcn_mfma_f32_4x4x1f32(A, H[5], acc, 4, 8 * G + 5, 0);
  acc = __builtin_amdgcn_mfma_f32_4x4x1f32(A, H[6], acc, 4, 8 * G + 6, 0);
  acc = __builtin_amdgcn_mfma_f32_4x4x1f32(A, H[7], acc, 4, 8 * G + 7, 0);
  return acc;
}

// First order over rows of at most TOP + 4 <= 8 features at the 8-node rule, in
// FP64.  With H(m) = w_m prod_k F_k(m) over all the row's slots, slot j adds
//   sum_m c_j w_m prod_{k != j} F_k(m) = sum_m H(m) c_j / F_j(m),
// and c_j / F_j depends on the sample only through its follow bit:
//   followed: e_j(m) = (1 - b_j) / (b_j + t_m (1 - b_j)), a table per slot;
//   not:      r(m) = -1 / (1 - t_m), the same for every slot.
// So a row needs the running product, one node sum per slot against
// sample-independent coefficients, and one sum D for all slots not followed;
// no suffix products and no factors kept.
// Slots 1..TOP are the row's root side.  While consecutive rows share all of
// them, their H are summed and slots 1..TOP take their node sums once for
// the run of rows (with full trees of depth TOP + 4: 8 rows); slots TOP + 1
// .. TOP + 3, slot 0 and D are summed for every row.  P[k], the prefix product
// through slot k, is kept from row to row for k >= TOP, so of the slots below
// the root side only those past the shared count are evaluated.
// (FP32 keeps values_rows_shared: a run's H would be summed in FP32, where
// every row's term goes into the FP64 accumulator by itself there, and with
// FP64 sums of H the walk is mostly the slower one.  FP32, ms with FP32 sums,
// with FP64 sums and by values_rows_shared: 500 trees of depth 8, 100 features,
// 100k rows 23.1, 25.6, 23.7; 500 of depth 6, 50 features, 50k rows 2.53, 3.16,
// 2.61; 500 of depth 4 0.65, 0.65, 0.58; 1000 of depth 8 grown on data, 100k
// rows 42.3, 46.7, 49.4.)
//
// The row loop is pipelined by hand.  Scalar loads and LDS reads share one
// wait counter and scalar loads return out of order, so a wait for one is a
// wait for all: the next row's record is loaded once this row's values of x
// are in, and the next row's x are read before this row's sums are added.
//
// Bound by VALU issue: compares, selects and address adds read scalar
// registers, and FP64 takes 1.3 clocks of a CU per wave instruction.  300 trees
// of depth 8, 100 features, 5003 rows: 3.43 ms with suffix products and node
// sums per slot, 2.17 here.
template <int TOP, bool NANS>
__device__ __forceinline__ void values_rows_grouped(
    const WalkRow* __restrict__ rows, const double* __restrict__ coef, int row0,
    const Slot0<double>* __restrict__ z0, const float* xs, double* as, int pb, int pe, int wave,
    int nw, int lane, const NodeConsts<double>& nc) {
  using T = double;
  constexpr int N = 8, ND = TOP + 3;
  const int run = (pe - pb + nw - 1) / nw;
  const int p_first = pb + wave * run;
  const int p_last = min(pe, p_first + run);
  if (p_first >= p_last) return;
  T P[ND + 1][N];
  uint64_t in_k[ND + 1];  // follow bits of slots 1..ND, one per lane
  T Hs[TOP > 0 ? N : 1];  // sum of H over the rows since slots 1..TOP changed
  int xo_top[TOP > 0 ? TOP : 1];
  int d_top = 0, p_top = p_first;
#pragma unroll
  for (int k = 0; k <= ND; ++k) in_k[k] = 0;
#pragma unroll
  for (int m = 0; m < N; ++m) P[0][m] = nc.w[m];
#pragma unroll
  for (int m = 0; m < (TOP > 0 ? N : 1); ++m) Hs[m] = T(0);
  const char* xl = reinterpret_cast<const char*>(xs + lane);
  char* al = reinterpret_cast<char*>(as + lane);
  auto x_at = [&](int off) __attribute__((always_inline)) {
    return *reinterpret_cast<const float*>(xl + off);
  };
  auto add = [&](int xo, T v) __attribute__((always_inline)) {
    __hip_atomic_fetch_add(reinterpret_cast<double*>(al + 2 * xo), v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  // lanes whose x lies in [l, u) (u = NaN: no bound), or is missing and miss
  auto inside = [&](float x, float l, float u, bool miss) __attribute__((always_inline)) {
    uint64_t lower = __builtin_amdgcn_ballot_w64(x >= l);
    if (NANS) lower |= miss ? __builtin_amdgcn_ballot_w64(x != x) : 0;
    return lower & __builtin_amdgcn_ballot_w64(!(x >= u));
  };
  auto flush_top = [&]() __attribute__((always_inline)) {
    if constexpr (TOP > 0) {
      T D = nc.r[0] * Hs[0];
#pragma unroll
      for (int m = 1; m < N; ++m) D = fmaT(nc.r[m], Hs[m], D);
      const T* e = coef + (int64_t)(p_top - row0) * kShortCoef;
#pragma unroll
      for (int k = 0; k < TOP; ++k) {
        if (k + 1 < d_top) {
          T E = ldu(e + 8 * k) * Hs[0];
#pragma unroll
          for (int m = 1; m < N; ++m) E = fmaT(ldu(e + 8 * k + m), Hs[m], E);
          add(xo_top[k], pick(in_k[k + 1], D, E));
        }
      }
    }
  };
  // slot k's prefix product from its bits
  auto extend = [&](int k, T b, T cb) __attribute__((always_inline)) {
    const T bv = to_vgpr(b);
    const T c = pick(in_k[k], -bv, to_vgpr(cb));
#pragma unroll
    for (int m = 0; m < N; ++m) P[k][m] = P[k - 1][m] * fmaT(nc.t[m], c, bv);
  };
  struct Rec {  // the part of a row that every row reads (scalar registers)
    int32_t pack, xo0;
    float lo0, hi0, split;
    int32_t xo[3];
    float lo[3], hi[3];
    T b[3], cb[3], bm, cA, cB;
  };
  auto load = [&](int p) __attribute__((always_inline)) {
    const WalkRow* w = rows + (p - row0);
    Rec r;
    const row_v16 a = ldu(reinterpret_cast<const row_v16*>(w));  // 14 words are the row's
    r.pack = a[0];
    r.xo0 = a[1];
    r.lo0 = __int_as_float(a[2]);
    r.hi0 = __int_as_float(a[3]);
    r.split = __int_as_float(a[4]);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      r.xo[i] = a[5 + i];
      r.lo[i] = __int_as_float(a[8 + i]);
      r.hi[i] = __int_as_float(a[11 + i]);
      r.b[i] = ldu(&w->bl[i]);
      r.cb[i] = ldu(&w->cbl[i]);
    }
    const Slot0<T>* z = z0 + p;
    r.bm = ldu(&z->bm);
    r.cA = ldu(&z->ca);
    r.cB = ldu(&z->cb);
    return r;
  };
  Rec r = load(p_first);
  float x[4] = {x_at(r.xo0), x_at(r.xo[0]), x_at(r.xo[1]), x_at(r.xo[2])};
  for (int p = p_first; p < p_last; ++p) {
    const int d = r.pack & 15;
    const int s = p == p_first ? 0 : (r.pack >> 4) & 15;
    const int mok = r.pack >> 8;
    const int p_next = min(p + 1, p_last - 1);
    // follow bits of slot 0 and of slots TOP + 1 .. ND (shared ones come out
    // as they are), and slot 0's c
    uint64_t in0 = inside(x[0], r.lo0, r.hi0, NANS && (mok & 0x101) != 0);
    uint64_t in0a = __builtin_amdgcn_ballot_w64(!(x[0] >= r.split));
    if (NANS) in0a &= (mok & 0x100) != 0 ? __builtin_amdgcn_ballot_w64(x[0] == x[0]) : ~0ull;
#pragma unroll
    for (int i = 0; i < 3; ++i)
      in_k[TOP + 1 + i] = inside(x[1 + i], r.lo[i], r.hi[i], ((mok >> (TOP + 1 + i)) & 1) != 0);
    if constexpr (TOP > 0) {
      if (s < TOP) {
        if (p != p_first) {
          flush_top();
#pragma unroll
          for (int m = 0; m < N; ++m) Hs[m] = T(0);
        }
        const WalkRow* w = rows + (p - row0);
        float xt[TOP], lt[TOP], ut[TOP];
        T bt[TOP], cbt[TOP];
#pragma unroll
        for (int k = 0; k < TOP; ++k) {
          xo_top[k] = ldu(&w->xot[k]);
          lt[k] = ldu(&w->lot[k]);
          ut[k] = ldu(&w->hit[k]);
          bt[k] = ldu(&w->bt[k]);
          cbt[k] = ldu(&w->cbt[k]);
        }
#pragma unroll
        for (int k = 0; k < TOP; ++k) xt[k] = x_at(xo_top[k]);
#pragma unroll
        for (int k = 0; k < TOP; ++k) {
          in_k[k + 1] = inside(xt[k], lt[k], ut[k], ((mok >> (k + 1)) & 1) != 0);
          extend(k + 1, bt[k], cbt[k]);
        }
        d_top = d;
        p_top = p;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    const Rec rn = load(p_next);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (TOP + 1 + i > s) extend(TOP + 1 + i, r.b[i], r.cb[i]);
    // slot 0 (the row's own factor, leaf values folded in), last in the order
    const T bv0 = to_vgpr(r.bm);
    const T c0 = pick(in0, -bv0, pick(in0a, to_vgpr(r.cB), to_vgpr(r.cA)));
    T H[N];
    T q0 = P[ND][0];
#pragma unroll
    for (int m = 1; m < N; ++m) q0 += P[ND][m];
#pragma unroll
    for (int m = 0; m < N; ++m) H[m] = P[ND][m] * fmaT(nc.t[m], c0, bv0);
    // slots TOP + 1 .. ND, and D
    T E[4];
    E[3] = nc.r[0] * H[0];
#pragma unroll
    for (int m = 1; m < N; ++m) E[3] = fmaT(nc.r[m], H[m], E[3]);
    const T* e = coef + (int64_t)(p - row0) * kShortCoef + 8 * TOP;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      E[i] = ldu(e + 8 * i) * H[0];
#pragma unroll
      for (int m = 1; m < N; ++m) E[i] = fmaT(ldu(e + 8 * i + m), H[m], E[i]);
    }
    __builtin_amdgcn_sched_barrier(0);
    x[0] = x_at(rn.xo0);
#pragma unroll
    for (int i = 0; i < 3; ++i) x[1 + i] = x_at(rn.xo[i]);
    __builtin_amdgcn_sched_barrier(0);
    add(r.xo0, c0 * q0);
    if (d == ND + 1) {
#pragma unroll
      for (int i = 0; i < 3; ++i) add(r.xo[i], pick(in_k[TOP + 1 + i], E[3], E[i]));
    } else {
#pragma unroll
      for (int i = 0; i < 3; ++i)
        if (TOP + 1 + i < d) add(r.xo[i], pick(in_k[TOP + 1 + i], E[3], E[i]));
    }
    if constexpr (TOP > 0) {
#pragma unroll
      for (int m = 0; m < N; ++m) Hs[m] += H[m];
    }
    r = rn;
  }
  flush_top();
}

// First order over rows of more than 8 features in FP32, by the sums of
// values_rows_grouped: slot j adds sum_m H(m) c_j / F_j(m), taken once for a
// run of rows that share it.  Slots 1, 2, ... are taken in batches of 8.  Per
// batch b the wave keeps the prefix product P[b] over the batches before it,
// the follow bits of its slots, and Hs[b], the sum of H over the rows since
// the batch (or one before it) changed and not yet passed on.  When a row
// changes batch b0 first, the batches from the deepest to b0 are closed: each
// adds its slots' node sums of Hs[b] and passes Hs[b] on to batch b - 1; then
// the row's own batches b0, b0 + 1, ... are opened.  So a slot is evaluated and
// added about once per change and not once per row.  A batch's coefficients
// (1 - b_j) / (b_j + t_m (1 - b_j)) are formed when it closes, one per lane:
// lane 4 (8 g + m) + i has slot 4 g + i of the batch at node m, the blocks of
// node_sums4.
// Hs is in FP64: a run may be as long as a subtree has rows, and FP32 sums of
// 4000 like rows lose 2e-5.  Its node sums are FP32's, of the sum rounded once.
// Batches of 8: 148 VGPRs at 32 slots, held to 128 (64 slots: 256 and 88 bytes
// of scratch).  100 trees of up to 32 features and 512 leaves, 10k rows: 7.1
// ms, 6.3 with FP32 sums (99 VGPRs); 12.1 by the suffix products per row and
// slot that this replaces.  Batches of 4 evaluate fewer shared slots again but
// keep twice the state (10.6 ms already with FP32 sums).
template <int DMAX, bool NANS>
__device__ __forceinline__ void values_rows_batched(
    const PathHdr* __restrict__ hdr, const int32_t* __restrict__ feat,
    const float* __restrict__ lo, const float* __restrict__ hi, const float* __restrict__ bb,
    const float* __restrict__ cbb, const Slot0<float>* __restrict__ z0,
    const int32_t* __restrict__ share, const float* xs, double* as, int pb, int pe, int wave,
    int nw, int lane) {
  constexpr int N = 8, BS = 8, NB = DMAX / BS;
  const int run = (pe - pb + nw - 1) / nw;
  const int p_first = pb + wave * run;
  const int p_last = min(pe, p_first + run);
  float P[NB + 1][N];
  double Hs[NB][N];
  uint32_t bits[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    bits[b] = 0;
#pragma unroll
    for (int m = 0; m < N; ++m) Hs[b][m] = 0.0;
  }
#pragma unroll
  for (int m = 0; m < N; ++m) P[0][m] = rule8_w32(m);
  const float t_lane = rule8_t32((lane >> 2) & 7);
  const int slot_lane = (lane >> 5) * 4 + (lane & 3);
  const float* xl = xs + lane;
  double* al = as + lane;
  auto add = [&](int f, float v) __attribute__((always_inline)) {
    __hip_atomic_fetch_add(al + f * kTileStride, (double)v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  auto inside = [&](float x, float l, float u, bool miss) __attribute__((always_inline)) {
    uint64_t lower = __builtin_amdgcn_ballot_w64(x >= l);
    if (NANS) lower |= miss ? __builtin_amdgcn_ballot_w64(x != x) : 0;
    return lower & __builtin_amdgcn_ballot_w64(!(x >= u));
  };
  int off_p = 0, d_p = 0, nb_p = 0;  // the previous row
  // close batch b of the previous row
  auto close = [&](auto bc) __attribute__((always_inline)) {
    constexpr int b = decltype(bc)::value;
    const int j = off_p + BS * b + 1 + slot_lane;
    const float bj = bb[j], cj = cbb[j];
    float h[N];
#pragma unroll
    for (int m = 0; m < N; ++m) h[m] = (float)Hs[b][m];
    const float D0 = [&] {
      float D = rule8_r32(0) * h[0];
#pragma unroll
      for (int m = 1; m < N; ++m) D = __builtin_fmaf(rule8_r32(m), h[m], D);
      return D;
    }();
    const float den = __builtin_fmaf(t_lane, cj, bj);
    const float rc = __builtin_amdgcn_rcpf(den);
    const float e0 = cj * rc;
    // one correction step: e within about an ulp of the quotient (den = 0
    // only where b = 1 - b = 0 cannot be; a slot with b = 0 has den = t)
    const float A = __builtin_fmaf(__builtin_fmaf(-den, e0, cj), rc, e0);
    auto emit = [&](auto full) __attribute__((always_inline)) {
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const acc_v4 E = g == 0 ? node_sums4<0>(A, h, acc_v4{0.f, 0.f, 0.f, 0.f})
                                : node_sums4<1>(A, h, acc_v4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int k = 4 * g + i;
          if (decltype(full)::value || BS * b + 1 + k < d_p) {
            // the follow bit spread over the word selects E or D
            const uint32_t sel = (uint32_t)((int32_t)(bits[b] << (31 - k)) >> 31);
            const uint32_t v = (__float_as_uint(E[i]) & sel) | (__float_as_uint(D0) & ~sel);
            add(ldu(feat + off_p + BS * b + 1 + k) & kFeatureMask, __uint_as_float(v));
          }
        }
      }
    };
    if (BS * b + BS < d_p) emit(std::true_type{});
    else emit(std::false_type{});
    if constexpr (b > 0) {
#pragma unroll
      for (int m = 0; m < N; ++m) Hs[b - 1][m] += Hs[b][m];
    }
#pragma unroll
    for (int m = 0; m < N; ++m) Hs[b][m] = 0.0;
  };
  auto close_from = [&](int b0) __attribute__((always_inline)) {
    static_for_down<NB>([&](auto bc) __attribute__((always_inline)) {
      if (decltype(bc)::value >= b0 && decltype(bc)::value < nb_p) close(bc);
    });
  };
  for (int p = p_first; p < p_last; ++p) {
    const int d = ldu(&hdr[p].d);
    const int off = ldu(&hdr[p].off);
    const Slot0<float>* z = z0 + p;
    const float bm = ldu(&z->bm), cA = ldu(&z->ca), cB = ldu(&z->cb);
    const float loB = ldu(&z->lo_b), hiB = ldu(&z->hi_b);
    const bool mokB = ldu(&z->mok_b) != 0;
    const int f0w = ldu(feat + off);
    const float lo0 = ldu(lo + off), hi0 = ldu(hi + off);
    const int b0 = p == p_first ? 0 : ldu(share + p) / BS;
    const int nb = (d - 1 + BS - 1) / BS;
    const int f0 = f0w & kFeatureMask;
    const float x0 = xl[f0 * kTileStride];
    close_from(b0);
    // open the row's batches from b0 on
    static_for<NB>([&](auto bc) __attribute__((always_inline)) {
      constexpr int b = decltype(bc)::value;
      if (b >= b0 && b < nb) {
        int fw[BS];
        float l[BS], u[BS], bj[BS], cj[BS], x[BS];
        // reads past the row's last slot stay within the padded arrays
#pragma unroll
        for (int k = 0; k < BS; ++k) {
          const int j = off + BS * b + 1 + k;
          fw[k] = ldu(feat + j);
          l[k] = ldu(lo + j);
          u[k] = ldu(hi + j);
          bj[k] = ldu(bb + j);
          cj[k] = ldu(cbb + j);
        }
#pragma unroll
        for (int k = 0; k < BS; ++k) x[k] = xl[(fw[k] & kFeatureMask) * kTileStride];
        uint64_t in[BS];
        uint32_t w = 0;
#pragma unroll
        for (int k = 0; k < BS; ++k) {
          in[k] = inside(x[k], l[k], u[k], (fw[k] & kMissingOkBit) != 0);
          w |= pick(in[k], 0u, 1u) << k;
        }
        bits[b] = w;
        float run_[N];
#pragma unroll
        for (int m = 0; m < N; ++m) run_[m] = P[b][m];
        auto extend = [&](int k) __attribute__((always_inline)) {
          const float bv = to_vgpr(bj[k]);
          const float c = pick(in[k], -bv, to_vgpr(cj[k]));
#pragma unroll
          for (int m = 0; m < N; ++m) run_[m] *= __builtin_fmaf(rule8_t32(m), c, bv);
        };
        if (BS * b + BS < d) {
#pragma unroll
          for (int k = 0; k < BS; ++k) extend(k);
        } else {
#pragma unroll
          for (int k = 0; k < BS; ++k)
            if (BS * b + 1 + k < d) extend(k);
        }
#pragma unroll
        for (int m = 0; m < N; ++m) P[b + 1][m] = run_[m];
      }
    });
    // slot 0 (the row's own factor, leaf values folded in)
    const uint64_t inA = inside(x0, lo0, hi0, (f0w & kMissingOkBit) != 0);
    const uint64_t inB = inside(x0, loB, hiB, mokB);
    const float bv0 = to_vgpr(bm);
    const float c0 = pick(inA, pick(inB, -bv0, to_vgpr(cB)), to_vgpr(cA));
    static_for<NB>([&](auto bc) __attribute__((always_inline)) {
      constexpr int b = decltype(bc)::value;
      if (b == nb - 1) {
        float q0 = P[b + 1][0];
#pragma unroll
        for (int m = 1; m < N; ++m) q0 += P[b + 1][m];
#pragma unroll
        for (int m = 0; m < N; ++m)
          Hs[b][m] += (double)(P[b + 1][m] * __builtin_fmaf(rule8_t32(m), c0, bv0));
        add(f0, c0 * q0);
      }
    });
    off_p = off;
    d_p = d;
    nb_p = nb;
  }
  close_from(0);
}

// First order over rows of more than 8 features in FP64, reusing work between
// consecutive rows.  Each wave walks a contiguous run of rows.  The products
// are taken over the slots in the order 1, 2, ..., d - 1, 0: slot 0 (the
// row's own factor, from Slot0) comes last, so the prefix products over slots
// 1..j-1 depend only on those slots.  When slots 1..s equal the previous
// row's (share[p] = s, from the host), the c_j of the batches of 8 slots that
// lie within them are still in registers, and so are the prefix checkpoints
// ck[b] = w prod_{1 <= k < 8b} F_k(m) of the batches b with 8b - 1 <= s (kept
// across rows when all nodes run in one pass).  The backward sweep is that of
// adjoint_paths with the suffix products started from slot 0's factor; slot 0's own leave-one-out product
// is the full prefix over slots 1..d-1 (inert padding slots are factors 1).
template <typename T, int DMAX, int NH, bool STORE_G, bool NANS, int NN>
__device__ __forceinline__ void values_rows_long(
    const PathHdr* __restrict__ hdr, const int32_t* __restrict__ feat,
    const float* __restrict__ lo, const float* __restrict__ hi, const T* __restrict__ bb,
    const T* __restrict__ cbb, const Slot0<T>* __restrict__ z0,
    const int32_t* __restrict__ share, const float* xs, double* as, int pb, int pe, int wave,
    int nw, int lane, const T* tv, const T* wv) {
  constexpr int NB = DMAX / 8;
  constexpr bool kKeep = NH == NN;
  const int run = (pe - pb + nw - 1) / nw;
  const int p_first = pb + wave * run;
  const int p_last = min(pe, p_first + run);
  T cf[DMAX];     // c_j of the current row
  T ck[NB][NH];   // prefix checkpoints
  int ckv = 0;    // ck[1 .. ckv - 1] are the previous row's
  for (int p = p_first; p < p_last; ++p) {
    const int d = ldu(&hdr[p].d);
    if (d == 0) {
      ckv = 0;
      continue;
    }
    const int off = ldu(&hdr[p].off);
    const int s = p == p_first ? 0 : ldu(share + p);
    const int nb = (d + 7) >> 3;
    const Slot0<T>* z = z0 + p;
    const T bm = ldu(&z->bm);
    const T cA = ldu(&z->ca);
    const T cB = ldu(&z->cb);
    const float loB = ldu(&z->lo_b);
    const float hiB = ldu(&z->hi_b);
    const bool mokB = ldu(&z->mok_b) != 0;

    // c_j of every batch with a slot past s (a batch's shared slots are
    // evaluated again with it, to the same values: one branch per batch)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (b < nb && (b == 0 || 8 * b + 7 > s)) {
        const int jb = 8 * b;
        int fm[8];
        float l[8], u[8], x[8];
        T bl[8], cbl[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          fm[k] = ldu(feat + off + jb + k);
          l[k] = ldu(lo + off + jb + k);
          u[k] = ldu(hi + off + jb + k);
          bl[k] = ldu(bb + off + jb + k);
          cbl[k] = ldu(cbb + off + jb + k);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = xs[(fm[k] & kFeatureMask) * kTileStride + lane];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int j = jb + k;
          bool lower;
          if (NANS) {
            const bool miss = (fm[k] & kMissingOkBit) != 0;
            lower = miss ? !(x[k] < l[k]) : (x[k] >= l[k]);
          } else {
            lower = x[k] >= l[k];
          }
          const bool in = lower & !(x[k] >= u[k]);
          if (j == 0) {
            bool lowerB;
            if (NANS) lowerB = mokB ? !(x[0] < loB) : (x[0] >= loB);
            else lowerB = x[0] >= loB;
            const bool inB = lowerB & !(x[0] >= hiB);
            cf[0] = in ? cA : (inB ? cB : -bm);
          } else {
            cf[j] = in ? cbl[k] : -bl[k];
          }
        }
      }
    }
    const int f0 = ldu(feat + off) & kFeatureMask;

#pragma unroll
    for (int pass = 0; pass < NN / NH; ++pass) {
      const int m0 = pass * NH;
      // checkpoints, recomputed from the first batch whose slots are not all
      // shared with the previous row
#pragma unroll
      for (int m = 0; m < NH; ++m) ck[0][m] = wv[m0 + m];
      bool fresh = !kKeep;
#pragma unroll
      for (int b = 1; b < NB; ++b) {
        if (b < nb) {
          fresh = fresh || b >= ckv || 8 * b - 1 > s;
          if (fresh) {
#pragma unroll
            for (int m = 0; m < NH; ++m) ck[b][m] = ck[b - 1][m];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              const int j = 8 * (b - 1) + k;
              if (j > 0) {
                const T bj = ldu(bb + off + j);
#pragma unroll
                for (int m = 0; m < NH; ++m) ck[b][m] *= fmaT(tv[m0 + m], cf[j], bj);
              }
            }
          }
        }
      }
      // backward sweep, last batch first; S starts from slot 0's factor
      T S[NH];
#pragma unroll
      for (int m = 0; m < NH; ++m) S[m] = fmaT(tv[m0 + m], cf[0], bm);
#pragma unroll
      for (int b = NB - 1; b >= 0; --b) {
        if (b < nb) {
          const int jb = 8 * b;
          T bj[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) bj[k] = jb + k == 0 ? T(1) : ldu(bb + off + jb + k);
          T Pb[8][NH];
          T Gb[STORE_G ? 8 : 1][NH];
          T run[NH];
#pragma unroll
          for (int m = 0; m < NH; ++m) run[m] = ck[b][m];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
#pragma unroll
            for (int m = 0; m < NH; ++m) {
              Pb[k][m] = run[m];
              if (jb + k > 0) {
                const T g = fmaT(tv[m0 + m], cf[jb + k], bj[k]);
                if (STORE_G) Gb[STORE_G ? k : 0][m] = g;
                run[m] *= g;
              }
            }
          }
          if (b == nb - 1) {
            // slot 0: w prod_{k >= 1} F_k(m), the full prefix
            T dot = run[0];
#pragma unroll
            for (int m = 1; m < NH; ++m) dot += run[m];
            __hip_atomic_fetch_add(&as[f0 * kTileStride + lane], (double)(cf[0] * dot),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
#pragma unroll
          for (int k = 7; k >= 0; --k) {
            const int j = jb + k;
            if (j > 0) {
              if (j < d) {
                const int f = ldu(feat + off + j) & kFeatureMask;
                T dot = Pb[k][0] * S[0];
#pragma unroll
                for (int m = 1; m < NH; ++m) dot = fmaT(Pb[k][m], S[m], dot);
                __hip_atomic_fetch_add(&as[f * kTileStride + lane], (double)(cf[j] * dot),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
              }
#pragma unroll
              for (int m = 0; m < NH; ++m) {
                const T g = STORE_G ? Gb[STORE_G ? k : 0][m] : fmaT(tv[m0 + m], cf[j], bj[k]);
                S[m] *= g;
              }
            }
          }
        }
      }
    }
    ckv = kKeep ? nb : 0;
  }
}

// The buckets of a launch over more than one: first rows and output groups of
// the n buckets (n = 1: all rows belong to group grp).
struct BucketIndex {
  const int32_t* begin;
  const int32_t* group;
  int32_t n;
  int32_t grp;
};

// The rows and tile features of one work item.  Work item b is (sample block
// b mod nsb, row chunk b div nsb).  Ordinarily a chunk is `chunk` consecutive
// rows of the bucket and the tile holds every feature; with segments (wide
// feature spaces) chunk c is segment c, whose tile holds its own feature
// list, which the rows' elements index (lfeat).  A launch over several buckets
// (BucketSpan) cuts each bucket into chunks of its own, in bucket order.
struct ItemRows {
  int p0, p1;            // rows [p0, p1)
  int grp;               // their output group
  int nf;                // tile features
  const int32_t* fmap;   // tile feature -> global feature (null: identity)
};

__device__ __forceinline__ ItemRows item_rows(const Segment* segs, const int32_t* seg_feat,
                                              int ch, int32_t path_begin, int32_t path_end,
                                              int32_t chunk, int32_t F, const BucketIndex& bx) {
  ItemRows ir;
  ir.grp = bx.grp;
  if (segs != nullptr) {
    ir.p0 = ldu(&segs[ch].row_begin);
    ir.p1 = ldu(&segs[ch].row_end);
    ir.nf = ldu(&segs[ch].nfeat);
    ir.fmap = seg_feat + ldu(&segs[ch].feat_begin);
    if (bx.n > 1) {
      int b = 0;
      while (b + 1 < bx.n && ir.p0 >= ldu(bx.begin + b + 1)) ++b;
      ir.grp = ldu(bx.group + b);
    }
  } else if (bx.n > 1) {
    int b = 0, c = ch, q0 = path_begin, q1 = path_end;
    for (;; ++b) {
      q1 = b + 1 < bx.n ? ldu(bx.begin + b + 1) : path_end;
      const int n = (q1 - q0 + chunk - 1) / chunk;
      if (c < n || b + 1 >= bx.n) break;
      c -= n;
      q0 = q1;
    }
    ir.p0 = q0 + c * chunk;
    ir.p1 = min(q1, ir.p0 + chunk);
    ir.grp = ldu(bx.group + b);
    ir.nf = F;
    ir.fmap = nullptr;
  } else {
    ir.p0 = path_begin + ch * chunk;
    ir.p1 = min(path_end, ir.p0 + chunk);
    ir.nf = F;
    ir.fmap = nullptr;
  }
  return ir;
}

// tile_f: the features the LDS layout is sized for (F, or kSegFeatures with
// segments); F: phi's row length.
// The walk of a first-order instance: values_rows_grouped with TOP = WALK for
// WALK = 0..4, values_rows_shared with ND = WALK - kPerRow for kPerRow + 3 ..
// kPerRow + 7 and, nothing kept, with ND = WALK - kNoKeep for kNoKeep + 3 ..
// kNoKeep + 7 (short rows), values_rows_long for kPerRow, values_rows_batched
// for kBatched.
constexpr int kPerRow = 16, kNoKeep = 32, kBatched = -2;

// (values_rows_batched at 32 slots: four waves per SIMD with 68 bytes of
// scratch, 7.12 ms, against three with none, 7.38: the case named there.)
template <typename T, int DMAX, int NH, bool STORE_G, int NN, int WALK>
__global__ void __launch_bounds__(512, WALK == kBatched && DMAX == 32 ? 4 : 2)
values_kernel(const PathHdr* __restrict__ hdr, const int32_t* __restrict__ feat,
              const float* __restrict__ lo, const float* __restrict__ hi,
              const T* __restrict__ bb, const T* __restrict__ cbb,
              const Slot0<T>* __restrict__ z0, const int32_t* __restrict__ share,
              const float* __restrict__ X, int64_t M, int64_t ldx, int32_t F, int32_t tile_f,
              int32_t path_begin, int32_t path_end, int32_t chunk, int32_t nsb,
              const Segment* __restrict__ segs, const int32_t* __restrict__ seg_feat,
              int32_t ng, BucketIndex bx, double* __restrict__ acc, void* __restrict__ direct,
              int32_t direct_fp64, int32_t plain_add, const ShortRow<T>* __restrict__ srows,
              const WalkRow* __restrict__ wrows, const double* __restrict__ wcoef,
              NodeConsts<T> nc) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* xs = reinterpret_cast<float*>(smem);
  size_t xs_bytes = ((size_t)tile_f * kTileStride * sizeof(float) + 15) & ~(size_t)15;
  double* as = reinterpret_cast<double*>(smem + xs_bytes);

  // The dispatcher deals workgroups to the 8 XCDs in turn: XCD x gets the
  // workgroups b = x mod 8.  They take the x-th eighth of the work items in
  // order, so each XCD's L2 holds the rows of its own chunks only.
  const int item = xcd_item((int)blockIdx.x, (int)gridDim.x);
  const int sb = item % nsb;
  const int ch = item / nsb;
  int64_t s0 = (int64_t)sb * kSamplesPerBlock;
  ItemRows ir = item_rows(segs, seg_feat, ch, path_begin, path_end, chunk, F, bx);
  int nf = ir.nf;

  // stage the sample tile transposed; zero the accumulator; note any NaN.
  // With segments (wide feature spaces) X is feature-major [F][ldx] and acc
  // [ng][F][M], so consecutive threads take consecutive samples of a feature.
  const bool fmajor = segs != nullptr;
  int tile = kSamplesPerBlock * nf;
  int nan_seen = 0;
  if (fmajor) {
    for (int i = threadIdx.x; i < tile; i += blockDim.x) {
      const int k = i >> 6, r = i & 63;
      const int64_t s = s0 + r;
      const float v = (s < M) ? X[(int64_t)ir.fmap[k] * ldx + s] : 0.0f;
      nan_seen |= (v != v);
      xs[k * kTileStride + r] = v;
      as[k * kTileStride + r] = 0.0;
    }
  } else {
    for (int i = threadIdx.x; i < tile; i += blockDim.x) {
      const int r = i / nf;
      const int k = i - r * nf;
      const int64_t s = s0 + r;
      const float v = (s < M) ? X[s * ldx + k] : 0.0f;
      nan_seen |= (v != v);
      xs[k * kTileStride + r] = v;
      as[k * kTileStride + r] = 0.0;
    }
  }
  const bool any_nan = __syncthreads_or(nan_seen) != 0;

  // The FP64 walk of long rows has no scalar registers to spare: what only the flush
  // needs waits in vector registers, and the weights of up to 16 slots do
  // (32 slots and more: no vector registers).  Otherwise each row reads spilled
  // ones back: 100 trees of up to 14 features, 10k rows, FP64 8.87 ms, 8.64
  // here; up to 32 features, 4000 rows 7.94, 7.80.
  constexpr bool kPark = DMAX > 8 && WALK == kPerRow && sizeof(T) == 8;
  uint32_t parked[kPark ? 5 : 1];
  if constexpr (kPark) {
    const uint64_t fmap = reinterpret_cast<uint64_t>(ir.fmap);
    parked[0] = (uint32_t)nf;
    parked[1] = (uint32_t)ir.grp;
    parked[2] = (uint32_t)sb;
    parked[3] = (uint32_t)fmap;
    parked[4] = (uint32_t)(fmap >> 32);
#pragma unroll
    for (int i = 0; i < 5; ++i) asm volatile("" : "+v"(parked[i]));
  }
  const int lane = threadIdx.x & 63;
  // wave-uniform loop bounds (kept in SGPRs so the path loads are scalar)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = __builtin_amdgcn_readfirstlane(blockDim.x >> 6);
  const int pb = __builtin_amdgcn_readfirstlane(ir.p0);
  const int pe = __builtin_amdgcn_readfirstlane(ir.p1);

  // nodes pinned in VGPRs: a VALU op may read only one SGPR on gfx9-class
  // hardware, and b_j arrives in an SGPR
  T tv[NN];
#pragma unroll
  for (int m = 0; m < NN; ++m) tv[m] = to_vgpr(nc.t[m]);
  T wv[NN];
#pragma unroll
  for (int m = 0; m < NN; ++m)
    wv[m] = DMAX == 16 && sizeof(T) == 8 ? to_vgpr(nc.w[m]) : nc.w[m];

  if constexpr (DMAX == 8 && WALK < kPerRow) {
    if (any_nan)
      values_rows_grouped<WALK, true>(wrows, wcoef, path_begin, z0, xs, as, pb, pe, wave, nw,
                                      lane, nc);
    else
      values_rows_grouped<WALK, false>(wrows, wcoef, path_begin, z0, xs, as, pb, pe, wave, nw,
                                       lane, nc);
  } else if constexpr (WALK == kBatched) {
    if (any_nan)
      values_rows_batched<DMAX, true>(hdr, feat, lo, hi, bb, cbb, z0, share, xs, as, pb, pe,
                                      wave, nw, lane);
    else
      values_rows_batched<DMAX, false>(hdr, feat, lo, hi, bb, cbb, z0, share, xs, as, pb, pe,
                                       wave, nw, lane);
  } else if constexpr (DMAX == 8) {
    constexpr bool kKeep = WALK < kNoKeep;
    constexpr int kNd = WALK - (kKeep ? kPerRow : kNoKeep);
    if (any_nan)
      values_rows_shared<T, NH, kNd, true, kKeep>(srows, path_begin, z0, xs, as, pb, pe, wave, nw,
                                                  lane, tv, nc);
    else
      values_rows_shared<T, NH, kNd, false, kKeep>(srows, path_begin, z0, xs, as, pb, pe, wave,
                                                   nw, lane, tv, nc);
  } else if (any_nan) {
    values_rows_long<T, DMAX, NH, STORE_G, true, NN>(hdr, feat, lo, hi, bb, cbb, z0, share, xs,
                                                     as, pb, pe, wave, nw, lane, tv, wv);
  } else {
    values_rows_long<T, DMAX, NH, STORE_G, false, NN>(hdr, feat, lo, hi, bb, cbb, z0, share, xs,
                                                      as, pb, pe, wave, nw, lane, tv, wv);
  }
  __syncthreads();
  if constexpr (kPark) {
    nf = (int)__builtin_amdgcn_readfirstlane(parked[0]);
    tile = kSamplesPerBlock * nf;
    ir.grp = (int)__builtin_amdgcn_readfirstlane(parked[1]);
    s0 = (int64_t)(int)__builtin_amdgcn_readfirstlane(parked[2]) * kSamplesPerBlock;
    ir.fmap = reinterpret_cast<const int32_t*>(
        (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(parked[3]) |
        (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(parked[4]) << 32);
  }

  // flush: consecutive threads take consecutive features of one sample.
  // direct: this workgroup is the only one of its sample block (one bucket,
  // one chunk), so it writes phi rows outright, in the output precision.
  if (fmajor) {
    // acc[grp, f, s] (segments never write phi directly)
    for (int i = threadIdx.x; i < tile; i += blockDim.x) {
      const int k = i >> 6, r = i & 63;
      const int64_t s = s0 + r;
      if (s < M) {
        const double v = as[k * kTileStride + r];
        const int64_t o = ((int64_t)ir.grp * F + ir.fmap[k]) * M + s;
        if (v != 0.0) {
          if (plain_add) acc[o] += v;
          else unsafeAtomicAdd(&acc[o], v);
        }
      }
    }
    return;
  }
  for (int i = threadIdx.x; i < tile; i += blockDim.x) {
    const int r = i / nf;
    const int k = i - r * nf;
    const int64_t s = s0 + r;
    if (s < M) {
      const double v = as[k * kTileStride + r];
      const int64_t o = (s * ng + ir.grp) * F + k;  // phi[s, grp, f]
      if (direct != nullptr) {
        if (direct_fp64) static_cast<double*>(direct)[o] = v;
        else static_cast<float*>(direct)[o] = (float)v;
      } else if (v != 0.0) {
        // plain_add: the only workgroup of this launch that holds (s, f)
        if (plain_add) acc[o] += v;
        else unsafeAtomicAdd(&acc[o], v);
      }
    }
  }
}


// Adjoint over rows of at most 8 features with all NH nodes in one pass,
// with the reuse of values_rows_shared (contiguous runs, slots 1..s of the
// previous row kept in registers: c_j, F_j(m) and g_j c_j).  Slot 0 (a merged
// pair's split feature, or any one feature of a single path) stays out of the
// products; with Q_j(m) = prod_{k >= 1, k != j} F_k(m), Q_0 = prod_{k >= 1} F_k,
//   R(m) = sum_{j >= 1} g_j c_j w_m Q_j(m),
//   d phi . g / d v_A = sum_m F_A(m) R(m) + g_0 c_A sum_m w_m Q_0(m),
// where F_A = b_A + t c_A is slot 0's factor of leaf A (a single path: its
// own), and likewise for leaf B of a merged pair.  The sum over m of
// F_A(m) R(m) is b_A sum_m R(m) + c_A sum_m t_m R(m).
// ND as in values_rows_shared.
template <typename T, int NH, int ND, bool NANS>
__device__ __forceinline__ void adjoint_rows_shared(
    const ShortRow<T>* __restrict__ rows, int row0, const PathHdr* __restrict__ hdr,
    const SidePath* __restrict__ side, const float* xs, const T* gs, LeafSums sums, int pb, int pe,
    int wave, int nw, int lane, const T* tv, const NodeConsts<T>& nc) {
  constexpr bool kScalarT = NH == 8;
  constexpr int kLastP = ND < 7 ? ND : 6;
  // 1 in a register the compiler knows nothing of: slot 0's node sum stays a
  // chain of FMAs on the rounded prefix products, as with ND = 7
  T one = T(1);
  asm volatile("" : "+v"(one));
  const int run = (pe - pb + nw - 1) / nw;
  const int p_first = pb + wave * run;
  const int p_last = min(pe, p_first + run);
  T gc[ND + 1];     // slots 1..ND: g_j c_j of the current row
  T G[ND + 1][NH];  // slots 1..ND: F_j(m)
  // prefix products over slots 1..q (P[q], q = 0..6; w folded in); P[1..s]
  // depend only on shared slots and are kept from the previous row
  T P[ND + 1][NH];
#pragma unroll
  for (int m = 0; m < NH; ++m) P[0][m] = kScalarT ? node8_w(nc, m) : nc.w[m];
  const char* xl = reinterpret_cast<const char*>(xs + lane);
  const char* gl = reinterpret_cast<const char*>(gs + lane);
  for (int p = p_first; p < p_last; ++p) {
    // the record and the row's leaf and side record, all loads issued
    // before any is used.  An empty row (d = 0) is walked too: its slots are
    // inert, so its leaf's gradient comes out exactly 0.
    const ShortRowRegs<T> r = load_short_row(rows, row0, p);
    const int sidx = side == nullptr ? -1 : ldu(&hdr[p].tree);
    const bool merged = sidx >= 0;
    const int d = r.d;
    const int s = p == p_first ? 0 : r.share;
    // the tile row of slot k's feature: the sample tile is FP32 and the
    // gradient tile T
    const auto& xo = r.xo;
    const auto& go = sizeof(T) == 4 ? r.xo : r.ao;
    const auto& l = r.l;
    const auto& u = r.u;
    const auto& bl = r.bl;
    const auto& cbl = r.cbl;
    float x[ND + 1];
#pragma unroll
    for (int k = 0; k <= ND; ++k) x[k] = *reinterpret_cast<const float*>(xl + xo[k]);
    auto follows = [&](float xv, float lv, float uv, bool miss) -> bool {
      bool lower;
      if (NANS) lower = miss ? !(xv < lv) : (xv >= lv);
      else lower = xv >= lv;
      return lower & !(xv >= uv);
    };
    // slot 0: leaf A's factor (and B's for a merged pair)
    T bA = bl[0], cbA = cbl[0], bB = T(0), cbB = T(0);
    float loB = 0.f, hiB = 0.f;
    bool mokB = false;
    if (merged) {
      const SidePath* sp = side + sidx;
      loB = ldu(&sp->lo_b);
      hiB = ldu(&sp->hi_b);
      mokB = ldu(&sp->mok_b) != 0;
      bA = (T)ldu(&sp->b_a);
      cbA = (T)ldu(&sp->cb_a);
      bB = (T)ldu(&sp->b_b);
      cbB = (T)ldu(&sp->cb_b);
    }
    const T cA = follows(x[0], l[0], u[0], (r.mok & 1) != 0) ? cbA : -bA;
    const T cB = follows(x[0], loB, hiB, mokB) ? cbB : -bB;
    const T g0 = *reinterpret_cast<const T*>(gl + go[0]);
#pragma unroll
    for (int k = 1; k <= ND; ++k) {
      if (k > s) {
        // b in a VGPR once, for the select's -b and the factor FMAs
        const T bv = kScalarT ? to_vgpr(bl[k]) : bl[k];
        const T c = follows(x[k], l[k], u[k], ((r.mok >> k) & 1) != 0) ? cbl[k] : -bv;
        gc[k] = *reinterpret_cast<const T*>(gl + go[k]) * c;
        if (kScalarT) {
#pragma unroll
          for (int m = 0; m < NH; ++m) G[k][m] = fmaT(node8_t(nc, m), c, bv);
        } else {
#pragma unroll
          for (int m = 0; m < NH; ++m) G[k][m] = fmaT(tv[m], c, bl[k]);
        }
        // the prefix through this slot (every later slot is evaluated too)
        if (k <= kLastP) {
#pragma unroll
          for (int m = 0; m < NH; ++m) P[k][m] = P[k - 1][m] * G[k][m];
        }
      }
    }
    // sum_m w_m Q_0(m)
    T q0 = P[kLastP][0] * (ND < 7 ? one : G[ND][0]);
#pragma unroll
    for (int m = 1; m < NH; ++m) q0 = fmaT(P[kLastP][m], ND < 7 ? one : G[ND][m], q0);
    // R(m), slots ND..1
    T S[NH], R[NH];
#pragma unroll
    for (int m = 0; m < NH; ++m) {
      S[m] = T(1);
      R[m] = T(0);
    }
#pragma unroll
    for (int q = ND - 1; q >= 0; --q) {
      const int j = q + 1;
      if (j < d) {
#pragma unroll
        for (int m = 0; m < NH; ++m) R[m] = fmaT(gc[j], P[q][m] * S[m], R[m]);
      }
      if (q > 0) {
#pragma unroll
        for (int m = 0; m < NH; ++m) S[m] *= G[j][m];
      }
    }
    T sR = R[0], stR = (kScalarT ? node8_t(nc, 0) : tv[0]) * R[0];
#pragma unroll
    for (int m = 1; m < NH; ++m) {
      sR += R[m];
      stR = fmaT(kScalarT ? node8_t(nc, m) : tv[m], R[m], stR);
    }
    const T gq = g0 * q0;
    const double gA = (double)fmaT(bA, sR, cA * (stR + gq));
    const double gB = merged ? (double)fmaT(bB, sR, cB * (stR + gq)) : 0.0;
    if constexpr (sizeof(T) == 4) sums.add(gA, gB, p - p_first, p, p + 1 == p_last);
    else sums.add_row(gA, gB, p);
  }
}

// Adjoint over rows of at most TOP + 4 <= 8 features at the 8-node rule, in
// FP64.  With r_j = c_j / F_j as in values_rows_grouped, P = w prod_{k >= 1} F_k and
//   R(m) = P(m) W(m),  W(m) = sum_{j >= 1} g_j r_j(m),
// a leaf A of the row has gradient
//   b_A sum_m R(m) + c_A (sum_m t_m R(m) + g_0 sum_m P(m)),
// and B likewise.  W is linear in the slots' g_j: the followed slots' against
// their coefficients e_j(m), and the sum of the others' against r(m).  The
// root side's part of W is formed once for a run of rows that share it.  The
// row loop is pipelined as in values_rows_grouped.
// (FP32 keeps adjoint_rows_shared: its gradient is returned in FP64 and holds
// the rounding of every row's sums, which this order would change.)
template <int TOP, bool NANS>
__device__ __forceinline__ void adjoint_rows_grouped(
    const WalkRow* __restrict__ rows, const double* __restrict__ coef, int row0,
    const float* xs, const double* gs, LeafSums sums, int pb, int pe, int wave, int nw, int lane,
    const NodeConsts<double>& nc) {
  using T = double;  // offsets of the gradient tile are twice the sample tile's
  constexpr int N = 8, ND = TOP + 3;
  const int run = (pe - pb + nw - 1) / nw;
  const int p_first = pb + wave * run;
  const int p_last = min(pe, p_first + run);
  if (p_first >= p_last) return;
  T P[ND + 1][N];
  uint64_t in_k[ND + 1];
  T Wt[N];          // W over the followed slots 1..TOP
  T gu_top = T(0);  // sum of g over slots 1..TOP not followed
#pragma unroll
  for (int k = 0; k <= ND; ++k) in_k[k] = 0;
#pragma unroll
  for (int m = 0; m < N; ++m) {
    P[0][m] = nc.w[m];
    Wt[m] = T(0);
  }
  const char* xl = reinterpret_cast<const char*>(xs + lane);
  const char* gl = reinterpret_cast<const char*>(gs + lane);
  struct XG {
    float x;
    T g;
  };
  auto xg_at = [&](int off) __attribute__((always_inline)) {
    return XG{*reinterpret_cast<const float*>(xl + off),
              *reinterpret_cast<const T*>(gl + 2 * off)};
  };
  auto inside = [&](float x, float l, float u, bool miss) __attribute__((always_inline)) {
    uint64_t lower = __builtin_amdgcn_ballot_w64(x >= l);
    if (NANS) lower |= miss ? __builtin_amdgcn_ballot_w64(x != x) : 0;
    return lower & __builtin_amdgcn_ballot_w64(!(x >= u));
  };
  auto extend = [&](int k, T b, T cb) __attribute__((always_inline)) {
    const T bv = to_vgpr(b);
    const T c = pick(in_k[k], -bv, to_vgpr(cb));
#pragma unroll
    for (int m = 0; m < N; ++m) P[k][m] = P[k - 1][m] * fmaT(nc.t[m], c, bv);
  };
  struct Rec {
    int32_t pack, xo0;
    float lo0, hi0, split;
    int32_t xo[3];
    float lo[3], hi[3];
    T b[3], cb[3], b0[4];
  };
  auto load = [&](int p) __attribute__((always_inline)) {
    const WalkRow* w = rows + (p - row0);
    Rec r;
    const row_v16 a = ldu(reinterpret_cast<const row_v16*>(w));  // 14 words are the row's
    r.pack = a[0];
    r.xo0 = a[1];
    r.lo0 = __int_as_float(a[2]);
    r.hi0 = __int_as_float(a[3]);
    r.split = __int_as_float(a[4]);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      r.xo[i] = a[5 + i];
      r.lo[i] = __int_as_float(a[8 + i]);
      r.hi[i] = __int_as_float(a[11 + i]);
      r.b[i] = ldu(&w->bl[i]);
      r.cb[i] = ldu(&w->cbl[i]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) r.b0[i] = ldu(&w->b0[i]);
    return r;
  };
  Rec r = load(p_first);
  XG x0 = xg_at(r.xo0);
  XG x[3] = {xg_at(r.xo[0]), xg_at(r.xo[1]), xg_at(r.xo[2])};
  for (int p = p_first; p < p_last; ++p) {
    const int d = r.pack & 15;
    const int s = p == p_first ? 0 : (r.pack >> 4) & 15;
    const int mok = r.pack >> 8;
    const int p_next = min(p + 1, p_last - 1);
    const T* e = coef + (int64_t)(p - row0) * kShortCoef;
    uint64_t in0 = inside(x0.x, r.lo0, r.hi0, NANS && (mok & 0x101) != 0);
    uint64_t in0a = __builtin_amdgcn_ballot_w64(!(x0.x >= r.split));
    if (NANS) in0a &= (mok & 0x100) != 0 ? __builtin_amdgcn_ballot_w64(x0.x == x0.x) : ~0ull;
#pragma unroll
    for (int i = 0; i < 3; ++i)
      in_k[TOP + 1 + i] =
          inside(x[i].x, r.lo[i], r.hi[i], ((mok >> (TOP + 1 + i)) & 1) != 0);
    if constexpr (TOP > 0) {
      if (s < TOP) {
        const WalkRow* w = rows + (p - row0);
        XG xt[TOP];
#pragma unroll
        for (int k = 0; k < TOP; ++k) xt[k] = xg_at(ldu(&w->xot[k]));
        gu_top = T(0);
#pragma unroll
        for (int m = 0; m < N; ++m) Wt[m] = T(0);
#pragma unroll
        for (int k = 0; k < TOP; ++k) {
          in_k[k + 1] = inside(xt[k].x, ldu(&w->lot[k]), ldu(&w->hit[k]),
                               ((mok >> (k + 1)) & 1) != 0);
          extend(k + 1, ldu(&w->bt[k]), ldu(&w->cbt[k]));
          // inert slots past a short row's end have no gradient
          const T g = k + 1 < d ? xt[k].g : T(0);
          const T og = pick(in_k[k + 1], T(0), g);
          gu_top += g - og;
#pragma unroll
          for (int m = 0; m < N; ++m) Wt[m] = fmaT(ldu(e + 8 * k + m), og, Wt[m]);
        }
      }
    }
    // g of the low slots, split by their follow bits
    T og[3], gu = gu_top;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const T g = TOP + 1 + i < d ? x[i].g : T(0);
      og[i] = pick(in_k[TOP + 1 + i], T(0), g);
      gu += g - og[i];
    }
    const T g0 = x0.g;
    __builtin_amdgcn_sched_barrier(0);
    const Rec rn = load(p_next);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (TOP + 1 + i > s) extend(TOP + 1 + i, r.b[i], r.cb[i]);
    T W[N];
#pragma unroll
    for (int m = 0; m < N; ++m) W[m] = fmaT(nc.r[m], gu, Wt[m]);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int m = 0; m < N; ++m) W[m] = fmaT(ldu(e + 8 * (TOP + i) + m), og[i], W[m]);
    T q0 = P[ND][0], sR = P[ND][0] * W[0], stR = nc.t[0] * sR;
#pragma unroll
    for (int m = 1; m < N; ++m) {
      const T R = P[ND][m] * W[m];
      q0 += P[ND][m];
      sR += R;
      stR = fmaT(nc.t[m], R, stR);
    }
    __builtin_amdgcn_sched_barrier(0);
    x0 = xg_at(rn.xo0);
#pragma unroll
    for (int i = 0; i < 3; ++i) x[i] = xg_at(rn.xo[i]);
    __builtin_amdgcn_sched_barrier(0);
    const T bA = to_vgpr(r.b0[0]), bB = to_vgpr(r.b0[2]);
    // not inside: neither leaf is followed
    const T cA = pick(in0 & in0a, -bA, to_vgpr(r.b0[1]));
    const T cB = pick(in0 & ~in0a, -bB, to_vgpr(r.b0[3]));
    const T u = fmaT(g0, q0, stR);
    sums.add(fmaT(bA, sR, cA * u), fmaT(bB, sR, cB * u), p - p_first, p, p + 1 == p_last);
    r = rn;
  }
}

// Adjoint to the leaf values: the tile holds the samples' rows and their
// upstream gradient rows g[s, :].
// Bound by VALU issue.  200 trees of depth 6, 50 features, 20k rows, FP32: 1.6 ms
// with every slot of 8 walked, a wave sum per row and eight wavefronts whatever
// the registers; 0.6 with the inert slots left out (119 VGPRs instead of 136,
// four waves per SIMD), four rows' sums folded together over the wave, and
// the wavefronts chosen by the registers.
// A workgroup takes one chunk of rows and every n_groups-th sample block, and
// keeps the chunk's leaf sums in LDS over them.  Up to items / kAdjItems pairs
// of chunk and block (8192 untuned; at the size above there are 25 x 313) that
// is one block each, and the sums save what the rows' single adds to memory
// cost over one pass of consecutive leaves: that size, values and adjoint, 1.24
// ms without them, 1.18 with.  Beyond it a leaf costs one global atomic per
// workgroup, not one per sample block.
// part_rows = 0: the sums would take other wavefronts' room next to the tiles
// (launch_adj_one); every row adds to memory.  TOP: the bucket's (capacity 8); FP64 at 8 nodes takes the grouped
// walk with it, the others adjoint_rows_shared with ND = TOP + 3.
// Three waves per SIMD (168 VGPRs) where the instance is within a few
// registers of them.
template <typename T, int DMAX, int NH, bool STORE_G, int NN, int TOP>
__global__ void
__launch_bounds__(512, (DMAX == 16 && sizeof(T) == 4) || (DMAX == 8 && NN == 4) ? 3 : 2)
adjoint_kernel(const PathHdr* __restrict__ hdr, const int32_t* __restrict__ feat,
               const float* __restrict__ lo, const float* __restrict__ hi,
               const T* __restrict__ bb, const T* __restrict__ cbb,
               const SidePath* __restrict__ side, const float* __restrict__ X,
               const T* __restrict__ G, int64_t M, int64_t ldx, int32_t F, int32_t tile_f,
               int32_t path_begin, int32_t path_end, int32_t chunk, int32_t part_rows,
               int32_t nsb, int32_t n_groups, const Segment* __restrict__ segs,
               const int32_t* __restrict__ seg_feat, int32_t ng, BucketIndex bx,
               double* __restrict__ grad_leaf, int64_t part_stride,
               const ShortRow<T>* __restrict__ srows, const WalkRow* __restrict__ wrows,
               const double* __restrict__ wcoef, NodeConsts<T> nc) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* xs = reinterpret_cast<float*>(smem);
  const size_t tile_rows = (size_t)tile_f * kTileStride;
  const size_t xs_bytes = (tile_rows * sizeof(float) + 15) & ~(size_t)15;
  T* gs = reinterpret_cast<T*>(smem + xs_bytes);
  double* part = part_rows == 0 ? nullptr
      : reinterpret_cast<double*>(
            smem + ((xs_bytes + tile_rows * sizeof(T) + 15) & ~(size_t)15));

  // work items dealt to the XCDs in contiguous eighths (xcd_item)
  const int item = xcd_item((int)blockIdx.x, (int)gridDim.x);
  const int ch = item / n_groups;
  const int sb_first = item % n_groups;
  const ItemRows ir = item_rows(segs, seg_feat, ch, path_begin, path_end, chunk, F, bx);
  const int n_part = part_rows == 0 ? 0 : 2 * (ir.p1 - ir.p0);
  for (int i = threadIdx.x; i < n_part; i += blockDim.x) part[i] = 0.0;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = __builtin_amdgcn_readfirstlane(blockDim.x >> 6);
  const int pb = __builtin_amdgcn_readfirstlane(ir.p0);
  const int pe = __builtin_amdgcn_readfirstlane(ir.p1);
  T tv[NN];
#pragma unroll
  for (int m = 0; m < NN; ++m) tv[m] = to_vgpr(nc.t[m]);
  // deterministic (one sample block per workgroup): that block's own row of
  // partial sums
  const bool det = part_stride > 0;
  double* gl = det ? grad_leaf + (int64_t)sb_first * part_stride : grad_leaf;
  const LeafSums sums{part, gl, hdr, side, pb, lane, det};
  constexpr bool kGrouped = DMAX == 8 && NN == 8 && sizeof(T) == 8;
  const bool fmajor = segs != nullptr;
  for (int sb = sb_first; sb < nsb; sb += n_groups) {
    // stage the sample rows and gradient rows transposed (padding rows get a
    // zero gradient, so they add nothing); note any NaN.  With segments (wide
    // feature spaces) X is feature-major [F][ldx] and G [ng][F][M].
    const int64_t s0 = (int64_t)sb * kSamplesPerBlock;
    int nan_seen = 0, g_bad = 0;
    // not loop invariants: the walk needs the registers that hoisted index
    // arithmetic would hold
    int tid = threadIdx.x, nf = ir.nf;
    asm volatile("" : "+v"(tid), "+s"(nf));
    const int tile = kSamplesPerBlock * nf;
    if (fmajor) {
      for (int i = tid; i < tile; i += blockDim.x) {
        const int k = i >> 6, r = i & 63;
        const int f = ir.fmap[k];
        const int64_t s = s0 + r;
        const float v = (s < M) ? X[(int64_t)f * ldx + s] : 0.0f;
        nan_seen |= (v != v);
        xs[k * kTileStride + r] = v;
        const T g = (s < M) ? G[((int64_t)ir.grp * F + f) * M + s] : T(0);  // G[grp, f, s]
        if (kGrouped) g_bad |= !(__builtin_fabs(g) < INFINITY);
        gs[k * kTileStride + r] = g;
      }
    } else {
      for (int i = tid; i < tile; i += blockDim.x) {
        const int r = i / nf;
        const int k = i - r * nf;
        const int64_t s = s0 + r;
        const float v = (s < M) ? X[s * ldx + k] : 0.0f;
        nan_seen |= (v != v);
        xs[k * kTileStride + r] = v;
        const T g = (s < M) ? G[(s * ng + ir.grp) * F + k] : T(0);  // G[s, grp, f]
        if (kGrouped) g_bad |= !(__builtin_fabs(g) < INFINITY);
        gs[k * kTileStride + r] = g;
      }
    }
    const bool any_nan = __syncthreads_or(nan_seen | g_bad) != 0;
    if constexpr (kGrouped) {
      if (any_nan && __syncthreads_or(g_bad) != 0)
        // an infinite gradient makes inf - inf and 0 inf of the sums over
        // slots and nodes that the grouped walk regroups; row by row it comes
        // out as the infinity that it is
        adjoint_paths<T, 8, 2, false, true, NN>(hdr, feat, lo, hi, bb, cbb, side, xs, gs, sums, pb,
                                                pe, wave, nw, lane, tv, nc);
      else if (any_nan)
        adjoint_rows_grouped<TOP, true>(wrows, wcoef, path_begin, xs, gs, sums, pb, pe, wave, nw,
                                        lane, nc);
      else
        adjoint_rows_grouped<TOP, false>(wrows, wcoef, path_begin, xs, gs, sums, pb, pe, wave, nw,
                                         lane, nc);
    } else if constexpr (DMAX == 8) {
      if (any_nan)
        adjoint_rows_shared<T, NH, TOP + 3, true>(srows, path_begin, hdr, side, xs, gs, sums, pb,
                                                  pe, wave, nw, lane, tv, nc);
      else
        adjoint_rows_shared<T, NH, TOP + 3, false>(srows, path_begin, hdr, side, xs, gs, sums, pb,
                                                   pe, wave, nw, lane, tv, nc);
    } else if (any_nan) {
      adjoint_paths<T, DMAX, NH, STORE_G, true, NN>(hdr, feat, lo, hi, bb, cbb, side, xs, gs, sums,
                                                    pb, pe, wave, nw, lane, tv, nc);
    } else {
      adjoint_paths<T, DMAX, NH, STORE_G, false, NN>(hdr, feat, lo, hi, bb, cbb, side, xs, gs,
                                                     sums, pb, pe, wave, nw, lane, tv, nc);
    }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < n_part; i += blockDim.x) {
    const int leaf = leaf_of(hdr, side, pb + (i >> 1), i & 1);
    if (leaf >= 0) leaf_add(gl, leaf, part[i], det);
  }
}

namespace {

// Paths per work item: about 32 rounds of the ~512 resident workgroups
// (small tail), chunks of at least 256 paths so the per-item tile load and
// flush stay small next to the path work.
int values_chunk(int n_paths, int nsb, int items) {
  const int64_t want_items = items > 0 ? items : 16384;
  int64_t n_chunks = (want_items + nsb - 1) / nsb;
  n_chunks = std::max<int64_t>(1, std::min<int64_t>(n_chunks, (n_paths + 255) / 256));
  return (int)((n_paths + n_chunks - 1) / n_chunks);
}

}  // namespace

std::vector<BucketSpan> bucket_spans(const std::vector<Bucket>& bks, bool one_each) {
  std::vector<BucketSpan> out;
  for (size_t i = 0; i < bks.size(); ++i) {
    if (!one_each && !out.empty() && out.back().dmax() == bks[i].dmax) ++out.back().n;
    else out.push_back(BucketSpan{&bks[i], 1, (int)i});
  }
  return out;
}

bool values_direct(const std::vector<Bucket>& bks, int64_t M, const ValuesShape& shape) {
  if (bks.size() != 1 || M <= 0) return false;
  const int nsb = (int)((M + kSamplesPerBlock - 1) / kSamplesPerBlock);
  const int n_paths = bks[0].path_end - bks[0].path_begin;
  return values_chunk(n_paths, nsb, shape.items) >= n_paths;
}

namespace {


// The short-row records of a capacity-8 bucket from its first row (null for
// other buckets).
template <typename T>
const ShortRow<T>* short_rows_of(const PathArrays& a, const BucketSpan& sp) {
  const Bucket& bk = sp.list[0];
  if (bk.dmax != 8 || bk.srow_begin < 0) return nullptr;
  const ShortRow<T>* r;
  if constexpr (std::is_same<T, float>::value) r = a.srow32;
  else r = a.srow64;
  if (r == nullptr) fail(QTS_E_INVALID_ARG, "internal: no short-row records");
  return r + bk.srow_begin;
}

// How one launch over a bucket splits its rows: chunks of `chunk` rows with
// the full feature tile, or (wide feature spaces) the bucket's segments with
// their own tiles, the rows' elements read through lfeat.
struct RowSplit {
  const int32_t* feat;   // element features as the kernel indexes its tile
  const Segment* segs;   // null: plain chunks
  int chunk;
  int n_chunks;
  int tile_f;            // features the LDS tile is laid out for
};

// The chunks of `chunk` rows that a span's buckets are cut into.
int n_chunks_of(const BucketSpan& sp, int chunk) {
  int n = 0;
  for (int i = 0; i < sp.n; ++i)
    n += (sp.list[i].path_end - sp.list[i].path_begin + chunk - 1) / chunk;
  return n;
}

BucketIndex bucket_index(const PathArrays& a, const BucketSpan& sp) {
  if (sp.n > 1 && (a.bkt_begin == nullptr || a.bkt_group == nullptr))
    fail(QTS_E_INVALID_ARG, "internal: no bucket index");
  return sp.n > 1 ? BucketIndex{a.bkt_begin + sp.index, a.bkt_group + sp.index, sp.n, 0}
                  : BucketIndex{nullptr, nullptr, 1, sp.list[0].group};
}

RowSplit row_split(const HostTable& h, const PathArrays& a, const BucketSpan& sp, int nsb,
                   const ValuesShape& shape) {
  RowSplit r{a.feat, nullptr, 0, 0, h.F};
  if (a.compact == nullptr) {
    r.chunk = values_chunk(sp.path_end() - sp.path_begin(), nsb, shape.items);
    r.n_chunks = n_chunks_of(sp, r.chunk);
    return r;
  }
  const CompactTable& c = *a.compact;
  for (size_t i = 0; i + 1 < c.bucket_seg.size(); ++i) {
    const int s0 = c.bucket_seg[i];
    int s1 = c.bucket_seg[i + 1];
    if (s1 > s0 && c.segs[(size_t)s0].row_begin == sp.path_begin()) {
      while (s1 < (int)c.segs.size() && c.segs[(size_t)s1].row_begin < sp.path_end()) ++s1;
      r.feat = a.lfeat;
      r.segs = a.segs + s0;
      r.n_chunks = s1 - s0;
      r.tile_f = kSegFeatures;
      return r;
    }
  }
  fail(QTS_E_INVALID_ARG, "internal: bucket without segments");
}

// The grouped walk's rows of a capacity-8 bucket and their coefficients (FP64
// at 8 nodes).
ShortWalk walk_of(const PathArrays& a, const BucketSpan& sp) {
  const Bucket& bk = sp.list[0];
  if (bk.dmax != 8 || bk.srow_begin < 0) return {};
  if (a.walk.rows == nullptr || a.walk.coef == nullptr)
    fail(QTS_E_INVALID_ARG, "internal: no grouped-walk rows");
  return {a.walk.rows + bk.srow_begin, a.walk.coef + (int64_t)bk.srow_begin * kShortCoef};
}

// The first-order kernel's chunk where no timed shape says it: the split with
// the shortest run, in rounds of the workgroups that fit on the chip.  A CU's
// round is, for each of its workgroups, the chunk's rows (170 clocks for a row
// of up to 8 features over 64 samples in FP32, by feature beyond them, 2.5
// times that in FP64) and the tile, staged and passed on with FP64 atomics at
// 270 clocks a feature over 64 samples.  Chunks of 32 rows or more.  Past
// four rounds a gain of less than a fifth is inside the model's error: then
// the chunks stay (20000 rows, 200 trees of depth 6, values and adjoint: 1.17
// ms, 1.20 without this; 8267 rows, 912 of depth 7, 11 features, values: 1.89 and
// 1.86).
// FP32, us a call with chunks of at least 256 rows, and here: 1770 rows, 940
// trees of depth 4, 188 features: 155, 102; 606 rows, 938 of depth 3, 114
// features: 42, 37; 5537 rows, 28 of depth 5, 9 features: 50, 24; 4934 rows, 336
// of depth 7, 65 features: 510, 476.
int chunk_by_rounds(const BucketSpan& sp, int nsb, int F, bool fp64, int groups, int chunk0) {
  const int64_t rows = sp.path_end() - sp.path_begin();
  const int64_t slots = (int64_t)256 * groups;
  const int64_t row = (int64_t)170 * std::max(8, sp.dmax()) / 8 * (fp64 ? 5 : 2) / 2;
  const int64_t tile = (int64_t)270 * F;
  int64_t best = INT64_MAX;
  int out = chunk0;
  auto look = [&](int64_t chunk) {
    const int64_t items = (int64_t)nsb * n_chunks_of(sp, (int)chunk);
    const int64_t cost = ((items + slots - 1) / slots) * (chunk * row + tile);
    if (cost < best) {
      best = cost;
      out = (int)chunk;
    }
  };
  look(chunk0);
  if ((int64_t)nsb * n_chunks_of(sp, chunk0) > 4 * slots) best -= best / 5;
  for (int64_t k : {1, 2, 3, 4, 6, 8, 12, 16}) {
    const int64_t n = k * slots / nsb - (sp.n > 1 ? sp.n / 2 : 0);
    if (n >= 1) look(std::min(rows, std::max<int64_t>(32, (rows + n - 1) / n)));
  }
  return out;
}

template <typename T, int DMAX, int NH, bool STORE_G, int NN, int WALK = kPerRow>
void launch_one(const HostTable& h, const DeviceTable& d, const PathArrays& a,
                const BucketSpan& sp, const float* X, int64_t M, int64_t ldx, const void* slot0, double* acc,
                void* direct, const ValuesShape& shape, hipStream_t s, bool det) {
  const int F = h.F;
  const int nsb = (int)((M + kSamplesPerBlock - 1) / kSamplesPerBlock);
  RowSplit rs = row_split(h, a, sp, nsb, shape);
  const BucketIndex bx = bucket_index(a, sp);
  const int32_t row0 = sp.path_begin(), row1 = sp.path_end();
  const size_t lds = values_lds_bytes(rs.tile_f);
  // deterministic: one wave per workgroup (no LDS atomics between waves), and
  // one launch per chunk, so each launch has one workgroup per (sample, feature)
  const void* fn = (const void*)values_kernel<T, DMAX, NH, STORE_G, NN, WALK>;
  // direct: a sample block has one workgroup, so up to one round of them more
  // wavefronts each are more on the chip (20 trees of depth 4, 200 rows, a call:
  // FP32 36 us with 4, 23 with 8, FP64 45 and 32)
  const bool one_round = direct != nullptr && nsb <= 256 * resident_groups(fn, 512, lds);
  const int threads = det ? 64 : 64 * (shape.tuned ? shape.waves_per_block
                                       : one_round ? 8 : resident_waves(fn, lds));
  // (deterministic: a chunk is a launch; direct: one chunk has all rows)
  if (!det && !shape.tuned && rs.segs == nullptr && direct == nullptr) {
    rs.chunk = chunk_by_rounds(sp, nsb, F, std::is_same<T, double>::value,
                               resident_groups(fn, threads, lds), rs.chunk);
    rs.n_chunks = n_chunks_of(sp, rs.chunk);
  }
  const int64_t grid = (int64_t)nsb * rs.n_chunks;
  if (grid > 0x7fffffff) fail(QTS_E_UNSUPPORTED, "grid too large");
  const T* b = std::is_same<T, float>::value ? (const T*)a.b32 : (const T*)a.b64;
  const T* cb = std::is_same<T, float>::value ? (const T*)a.cb32 : (const T*)a.cb64;
  NodeConsts<T> nc;
  if constexpr (std::is_same<T, float>::value) nc = NN == 8 ? d.n32 : d.n32_4;
  else nc = NN == 8 ? d.n64 : d.n64_4;
  if (lds > raise_lds_limit(fn))
    fail(QTS_E_UNSUPPORTED, "internal: the sample tile does not fit in LDS");
  const ShortRow<T>* srows = short_rows_of<T>(a, sp);
  const ShortWalk walk =
      std::is_same<T, double>::value && NN == 8 ? walk_of(a, sp) : ShortWalk{};
  if (!det) {
    hipLaunchKernelGGL((values_kernel<T, DMAX, NH, STORE_G, NN, WALK>), dim3((unsigned)grid),
                       dim3(threads), lds, s, a.hdr, rs.feat, a.lo, a.hi, b, cb,
                       (const Slot0<T>*)slot0, a.share, X, M, ldx, F, rs.tile_f, row0, row1,
                       rs.chunk, nsb, rs.segs, a.seg_feat, h.n_groups, bx, acc, rs.segs ? nullptr : direct,
                       (int32_t)(std::is_same<T, double>::value ? 1 : 0), 0, srows, walk.rows,
                       walk.coef, nc);
    check_hip(hipGetLastError(), "values_kernel launch");
    return;
  }
  for (int c = 0; c < rs.n_chunks; ++c) {
    const int p0 = rs.segs ? row0 : row0 + c * rs.chunk;
    const int p1 = rs.segs ? row1 : std::min(row1, p0 + rs.chunk);
    hipLaunchKernelGGL((values_kernel<T, DMAX, NH, STORE_G, NN, WALK>), dim3((unsigned)nsb),
                       dim3(threads), lds, s, a.hdr, rs.feat, a.lo, a.hi, b, cb,
                       (const Slot0<T>*)slot0, a.share, X, M, ldx, F, rs.tile_f, p0, p1,
                       rs.chunk, nsb, rs.segs ? rs.segs + c : nullptr, a.seg_feat, h.n_groups,
                       bx, acc, nullptr, (int32_t)(std::is_same<T, double>::value ? 1 : 0),
                       1, srows ? srows + (p0 - row0) : nullptr,
                       walk.rows ? walk.rows + (p0 - row0) : nullptr,
                       walk.coef ? walk.coef + (int64_t)(p0 - row0) * kShortCoef : nullptr,
                       nc);
    check_hip(hipGetLastError(), "values_kernel launch");
  }
}

// A workgroup's chunk is at most kAdjRows rows (their leaf sums in LDS, next to
// the tiles), and the sample blocks are dealt to about items / kAdjItems
// workgroups in all: more than that many take several blocks each.  (200 trees
// of depth 6, 20k rows, values and adjoint: 1.17 ms with 2, where each of 7825
// takes one block; 1.19 and 1.20 with 8 and 32, where they take 4 and 16.)
constexpr int kAdjRows = 512;
constexpr int kAdjItems = 2;

template <typename T, int DMAX, int NH, bool STORE_G, int NN, int TOP = -1>
void launch_adj_one(const HostTable& h, const DeviceTable& d, const PathArrays& a,
                    const BucketSpan& sp, const float* X, const void* G, int64_t M, int64_t ldx,
                    double* grad_leaf, const ValuesShape& shape, hipStream_t s,
                    int64_t part_stride) {
  const int F = h.F;
  const int nsb = (int)((M + kSamplesPerBlock - 1) / kSamplesPerBlock);
  RowSplit rs = row_split(h, a, sp, nsb, shape);
  // a launch that would leave the chip idle (under 4 workgroups per CU) takes
  // chunks of down to 32 rows: its time is a wavefront's walk through its rows
  // one after another
  constexpr int kFill = 1024;
  if (rs.segs == nullptr && nsb * rs.n_chunks < kFill) {
    const int rows = sp.path_end() - sp.path_begin(), n = (kFill + nsb - 1) / nsb;
    rs.chunk = std::min(rs.chunk, std::max(32, (rows + n - 1) / n));
    rs.n_chunks = n_chunks_of(sp, rs.chunk);
  }
  const void* fn = (const void*)adjoint_kernel<T, DMAX, NH, STORE_G, NN, TOP>;
  const size_t limit = raise_lds_limit(fn);
  const size_t tile = (size_t)rs.tile_f * kTileStride;
  const size_t tiles = (((tile * sizeof(float) + 15) & ~(size_t)15) + tile * sizeof(T) + 15) &
                       ~(size_t)15;
  if (tiles > limit + 15) fail(QTS_E_UNSUPPORTED, "internal: the sample tile does not fit in LDS");
  // rows whose leaf sums fit next to the tiles (a chunk of under 128 would
  // load the tiles too often: then the rows add to memory)
  const int fit = tiles >= limit ? 0 : (int)((limit - tiles) / (2 * sizeof(double)));
  int part_rows = 0;
  if (rs.segs != nullptr) {
    // A segment has few rows (50 of 784 features' model), so its sums save
    // few atomics, and they hold 32 KB: 20k rows, 200 trees of depth 8, 784
    // features, values and adjoint, FP32: 19.8 ms with the sums, 16.0 without,
    // 20.7 before; FP64, whose kernel is slower: 22.7 and 24.2, 35.9 before.
    if (sizeof(T) == 8 && fit >= kSegMaxRows)
      part_rows = kSegMaxRows;
  } else if (fit >= 128) {
    // not where their LDS takes wavefronts off the CU.  Values and adjoint, ms
    // without them and with: FP32, 200 trees of depth 6, 152 features, 20k rows
    // 1.62, 2.15; 300 of depth 8, 100 features, 5003 rows 2.37, 2.95; FP64, 60
    // features, 20k rows 14.2, 16.2
    const int chunk = std::min({rs.chunk, kAdjRows, fit});
    auto waves_on = [&](size_t bytes) {
      const int w = shape.tuned ? shape.waves_per_block : resident_waves(fn, bytes);
      return w * resident_groups(fn, 64 * w, bytes);
    };
    if (waves_on(tiles + 2 * (size_t)chunk * sizeof(double)) >= waves_on(tiles)) {
      rs.chunk = chunk;
      rs.n_chunks = n_chunks_of(sp, rs.chunk);
      part_rows = chunk;
    }
  }
  const int64_t want = std::max(1, shape.items / kAdjItems);
  const int n_groups = part_stride > 0 || part_rows == 0
      ? nsb : (int)std::max<int64_t>(1, std::min<int64_t>(nsb, want / rs.n_chunks));
  const int64_t grid = (int64_t)n_groups * rs.n_chunks;
  if (grid > 0x7fffffff) fail(QTS_E_UNSUPPORTED, "grid too large");
  const size_t lds = std::min(limit, tiles + 2 * (size_t)part_rows * sizeof(double));
  const int threads = 64 * (shape.tuned ? shape.waves_per_block : resident_waves(fn, lds));
  const T* b = std::is_same<T, float>::value ? (const T*)a.b32 : (const T*)a.b64;
  const T* cb = std::is_same<T, float>::value ? (const T*)a.cb32 : (const T*)a.cb64;
  NodeConsts<T> nc;
  if constexpr (std::is_same<T, float>::value) nc = NN == 8 ? d.n32 : d.n32_4;
  else nc = NN == 8 ? d.n64 : d.n64_4;
  const ShortWalk w =
      std::is_same<T, double>::value && NN == 8 ? walk_of(a, sp) : ShortWalk{};
  hipLaunchKernelGGL((adjoint_kernel<T, DMAX, NH, STORE_G, NN, TOP>), dim3((unsigned)grid),
                     dim3(threads), lds, s, a.hdr, rs.feat, a.lo, a.hi, b, cb, a.side, X,
                     (const T*)G, M, ldx, F, rs.tile_f, sp.path_begin(), sp.path_end(),
                     rs.chunk, part_rows, nsb, n_groups, rs.segs, a.seg_feat, h.n_groups,
                     bucket_index(a, sp), grad_leaf, part_stride, short_rows_of<T>(a, sp), w.rows, w.coef, nc);
  check_hip(hipGetLastError(), "adjoint_kernel launch");
}

}  // namespace

void launch_adjoint(const HostTable& h, const DeviceTable& d, const PathArrays& a,
                    const BucketSpan& sp, bool fp64, const float* X, const void* G, int64_t M,
                    int64_t ldx, double* grad_leaf, const ValuesShape& shape, int nodes,
                    hipStream_t s, int64_t part_stride) {
  auto go = [&](auto t, auto dmax, auto nh, auto store, auto nn, auto top) {
    launch_adj_one<decltype(t), decltype(dmax)::value, decltype(nh)::value,
                   decltype(store)::value, decltype(nn)::value, decltype(top)::value>(
        h, d, a, sp, X, G, M, ldx, grad_leaf, shape, s, part_stride);
  };
  using std::false_type;
  using std::true_type;
#define QTS_N(n) std::integral_constant<int, n>{}
  if (sp.dmax() == 8) {
    auto short_rows = [&](auto top) {
      if (nodes == 4) {
        if (!fp64) go(0.f, QTS_N(8), QTS_N(4), true_type{}, QTS_N(4), top);
        else go(0.0, QTS_N(8), QTS_N(4), false_type{}, QTS_N(4), top);
      } else if (!fp64) {
        go(0.f, QTS_N(8), QTS_N(8), true_type{}, QTS_N(8), top);
      } else {
        go(0.0, QTS_N(8), QTS_N(8), true_type{}, QTS_N(8), top);
      }
    };
    switch (sp.list[0].top) {
      case 0: short_rows(QTS_N(0)); break;
      case 1: short_rows(QTS_N(1)); break;
      case 2: short_rows(QTS_N(2)); break;
      case 3: short_rows(QTS_N(3)); break;
      default: short_rows(QTS_N(4)); break;
    }
    return;
  }
  if (!fp64) {
    switch (sp.dmax()) {
      case 16: go(0.f, QTS_N(16), QTS_N(8), true_type{}, QTS_N(8), QTS_N(-1)); break;
      case 32: go(0.f, QTS_N(32), QTS_N(8), false_type{}, QTS_N(8), QTS_N(-1)); break;
      default: go(0.f, QTS_N(64), QTS_N(4), false_type{}, QTS_N(8), QTS_N(-1)); break;
    }
  } else {
    switch (sp.dmax()) {
      case 16: go(0.0, QTS_N(16), QTS_N(4), false_type{}, QTS_N(8), QTS_N(-1)); break;
      case 32: go(0.0, QTS_N(32), QTS_N(4), false_type{}, QTS_N(8), QTS_N(-1)); break;
      default: go(0.0, QTS_N(64), QTS_N(1), false_type{}, QTS_N(8), QTS_N(-1)); break;
    }
  }
#undef QTS_N
}

// The grouped walk's rows and node-sum coefficients of one bucket, 64 threads
// per row; entry 8 (j - 1) + m of a row's coefficients is slot j's.
__device__ __forceinline__ void fill_walk_row(const ShortRow<double>& r, const PathHdr& h,
                                              const SidePath* side, int32_t top, WalkRow* o) {
  WalkRow w;
  const int sidx = side == nullptr ? -1 : h.tree;
  int mok_b = 0;
  w.xo0 = r.xoff[0];
  w.lo0 = r.lo[0];
  w.hi0 = w.split = r.hi[0];
  if (r.d > 0 && sidx >= 0) {
    // A [lo, split) and B [split, hi): adjacent, or one of them empty
    w.lo0 = r.lo[0] < side[sidx].lo_b ? r.lo[0] : side[sidx].lo_b;
    w.hi0 = side[sidx].hi_b;
    mok_b = side[sidx].mok_b != 0 ? 1 : 0;
  }
  w.b0[0] = r.b[0];
  w.b0[1] = r.cb[0];
  w.b0[2] = w.b0[3] = 0.0;
  if (r.d > 0 && sidx >= 0) {
    w.b0[0] = side[sidx].b_a;
    w.b0[1] = side[sidx].cb_a;
    w.b0[2] = side[sidx].b_b;
    w.b0[3] = side[sidx].cb_b;
  }
  w.pack = r.d | r.share << 4 | (r.mok & 0xff) << 8 | mok_b << 16;
  for (int i = 0; i < 3; ++i) {
    const int k = top + 1 + i;
    w.xol[i] = r.xoff[k];
    w.lol[i] = r.lo[k];
    w.hil[i] = r.hi[k];
    w.bl[i] = r.b[k];
    w.cbl[i] = r.cb[k];
  }
  for (int i = 0; i < 4; ++i) {
    const int k = i < top ? i + 1 : 0;
    w.xot[i] = r.xoff[k];
    w.lot[i] = r.lo[k];
    w.hit[i] = r.hi[k];
    w.bt[i] = r.b[k];
    w.cbt[i] = r.cb[k];
  }
  *o = w;
}

__global__ void __launch_bounds__(256)
short_walk_kernel(const ShortRow<double>* __restrict__ rows, const PathHdr* __restrict__ hdr,
                  const SidePath* __restrict__ side, int32_t n, int32_t top,
                  NodeConsts<double> nc, WalkRow* __restrict__ out, double* __restrict__ coef) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t row = i >> 6;
  if (row >= n) return;
  const int l = (int)i & 63;
  const ShortRow<double>& r = rows[row];
  const int j = (l >> 3) + 1, m = l & 7;
  // over F as the walks form it
  coef[i] = j > 7 ? 0.0 : r.cb[j] / __builtin_fma(nc.t[m], r.cb[j], r.b[j]);
  if (l == 0) fill_walk_row(r, hdr[row], side, top, out + row);
}

void launch_short_walk(const PathArrays& a, const Bucket& bk, const NodeConsts<double>& nc,
                       hipStream_t s) {
  if (bk.dmax != 8) return;
  constexpr int32_t kRows = 1 << 24;  // a launch's: 2^30 threads
  for (int32_t p = bk.path_begin; p < bk.path_end;) {
    const int32_t n = std::min(bk.path_end - p, kRows);
    const int64_t r = (int64_t)bk.srow_begin + (p - bk.path_begin);
    const unsigned grid = (unsigned)(((int64_t)n * 64 + 255) / 256);
    hipLaunchKernelGGL(short_walk_kernel, dim3(grid), dim3(256), 0, s, a.srow64 + r, a.hdr + p,
                       a.side, n, bk.top, nc, a.walk.rows + r, a.walk.coef + r * kShortCoef);
    check_hip(hipGetLastError(), "short_walk_kernel launch");
    p += n;
  }
}

// First order of a few samples over rows of at most 8 features: a lane takes a
// row, a workgroup one sample and kLaneRows rows.  With samples across lanes a
// call of one sample uses one lane of 64, and is bound by the latency of the
// rows that a wavefront walks one after another; splitting the rows over more
// workgroups runs into their adds to the same few phi entries.
// The arithmetic of a row is values_rows_shared's, operation by operation, so
// a row's terms have the same bits (slot 0's factor is formed here, from the
// current leaf values, and no Slot0 records are needed).
constexpr int kLaneRows = 512;

template <typename T, int ND>
__global__ void __launch_bounds__(kLaneRows)
values_lane_kernel(const PathHdr* __restrict__ hdr, const int32_t* __restrict__ feat,
                   const float* __restrict__ lo, const float* __restrict__ hi,
                   const T* __restrict__ bb, const T* __restrict__ cbb,
                   const double* __restrict__ b64, const double* __restrict__ cb64,
                   const SidePath* __restrict__ side, const double* __restrict__ leaf_val,
                   const float* __restrict__ X, int64_t M, int64_t ldx, int32_t F,
                   int32_t fmajor, int32_t path_begin, int32_t path_end, int32_t ng,
                   BucketIndex bx, double* __restrict__ acc, void* __restrict__ direct,
                   NodeConsts<T> nc) {
  constexpr int N = 8, kLastP = ND < 7 ? ND : 6;
  extern __shared__ __align__(16) unsigned char smem[];
  double* phis = reinterpret_cast<double*>(smem);  // [F]
  float* xrow = reinterpret_cast<float*>(phis + F);
  const int64_t s = (int64_t)blockIdx.x % M;
  const int ch = (int)((int64_t)blockIdx.x / M);
  const ItemRows ir = item_rows(nullptr, nullptr, ch, path_begin, path_end, kLaneRows, F, bx);
  for (int i = threadIdx.x; i < F; i += blockDim.x) {
    xrow[i] = fmajor ? X[(int64_t)i * ldx + s] : X[s * ldx + i];
    phis[i] = 0.0;
  }
  const int p = min(ir.p0 + (int)threadIdx.x, ir.p1 - 1);
  const PathHdr h = hdr[p];
  int fw[ND + 1];
  float l[ND + 1], u[ND + 1];
  T b[ND + 1], cb[ND + 1];
#pragma unroll
  for (int k = 0; k <= ND; ++k) {
    fw[k] = feat[h.off + k];
    l[k] = lo[h.off + k];
    u[k] = hi[h.off + k];
    b[k] = bb[h.off + k];
    cb[k] = cbb[h.off + k];
  }
  // slot 0 as slot0_kernel forms it
  const int sidx = side == nullptr ? -1 : h.tree;
  T bm = T(0), cA = T(0), cB = T(0);
  float loB = l[0], hiB = u[0];
  bool mokB = (fw[0] & kMissingOkBit) != 0;
  if (h.d > 0 && sidx >= 0) {
    const SidePath sp = side[sidx];
    const double va = leaf_val[h.leaf], vb = leaf_val[sp.leaf_b];
    bm = (T)(va * sp.b_a + vb * sp.b_b);
    cA = (T)(va * sp.cb_a - vb * sp.b_b);
    cB = (T)(vb * sp.cb_b - va * sp.b_a);
    loB = sp.lo_b;
    hiB = sp.hi_b;
    mokB = sp.mok_b != 0;
  } else if (h.d > 0) {
    const double v = leaf_val[h.leaf];
    const double vm = v * b64[h.off];
    bm = (T)vm;
    cA = (T)(v * cb64[h.off]);
    cB = (T)(-vm);
  }
  __syncthreads();
  auto follows = [&](float x, float lv, float uv, bool miss) {
    return (miss ? !(x < lv) : (x >= lv)) & !(x >= uv);
  };
  T c[ND + 1], P[ND + 1][N];
#pragma unroll
  for (int m = 0; m < N; ++m) P[0][m] = node8_w(nc, m);
#pragma unroll
  for (int k = 0; k <= ND; ++k) {
    const float x = xrow[fw[k] & kFeatureMask];
    const bool in = follows(x, l[k], u[k], (fw[k] & kMissingOkBit) != 0);
    if (k == 0) {
      c[0] = in ? cA : (follows(x, loB, hiB, mokB) ? cB : -bm);
      b[0] = bm;
    } else {
      c[k] = in ? cb[k] : -b[k];
    }
    if (k >= 1 && k <= kLastP) {
#pragma unroll
      for (int m = 0; m < N; ++m) P[k][m] = P[k - 1][m] * fmaT(node8_t(nc, m), c[k], b[k]);
    }
  }
  T one = T(1);
  asm volatile("" : "+v"(one));
  const bool on = ir.p0 + (int)threadIdx.x < ir.p1;
  auto add = [&](int k, T v) {
    if (on)
      __hip_atomic_fetch_add(&phis[fw[k] & kFeatureMask], (double)v, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  {
    auto g = [&](int m) { return ND < 7 ? one : fmaT(node8_t(nc, m), c[ND], b[ND]); };
    T dot = P[kLastP][0] * g(0);
#pragma unroll
    for (int m = 1; m < N; ++m) dot = fmaT(P[kLastP][m], g(m), dot);
    add(0, c[0] * dot);
  }
  T S[N];
#pragma unroll
  for (int m = 0; m < N; ++m) S[m] = fmaT(node8_t(nc, m), c[0], b[0]);
#pragma unroll
  for (int j = ND; j >= 1; --j) {
    if (j < h.d) {
      T dot = P[j - 1][0] * S[0];
#pragma unroll
      for (int m = 1; m < N; ++m) dot = fmaT(P[j - 1][m], S[m], dot);
      add(j, c[j] * dot);
    }
    if (j > 1) {
#pragma unroll
      for (int m = 0; m < N; ++m) S[m] *= fmaT(node8_t(nc, m), c[j], b[j]);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < F; i += blockDim.x) {
    const double v = phis[i];
    if (direct != nullptr) {
      const int64_t o = (s * ng + ir.grp) * F + i;
      if (sizeof(T) == 8) static_cast<double*>(direct)[o] = v;
      else static_cast<float*>(direct)[o] = (float)v;
    } else if (v != 0.0) {
      const int64_t o = fmajor ? ((int64_t)ir.grp * F + i) * M + s : (s * ng + ir.grp) * F + i;
      unsafeAtomicAdd(&acc[o], v);
    }
  }
}

// The lane kernel's time grows with samples x rows, the others' hardly with up
// to 64 samples.  Microseconds a call (samples in lanes | rows in lanes):
//   1000 trees of depth 8 (128k rows), FP32: 1 sample 64 | 19, 8: 66 | 58,
//   12: 67 | 69, 16: 66 | 82; FP64: 1: 119 | 19, 12: 120 | 101, 16: 120 | 129;
//   500 trees of depth 6 (16k rows), FP32: 1: 26 | 17, 32: 29 | 24, 48: 30 | 29.
bool values_lane(const BucketSpan& sp, int64_t M, int F, int nodes) {
  const int64_t rows = sp.path_end() - sp.path_begin();
  return sp.dmax() == 8 && nodes == 8 && (M <= 12 || (M <= 64 && M * rows <= (int64_t)1 << 19)) &&
         (size_t)F * (sizeof(double) + sizeof(float)) <= (size_t)kMaxLdsBytes;
}

template <typename T, int ND>
static void launch_lane_one(const HostTable& h, const DeviceTable& d, const PathArrays& a,
                            const BucketSpan& sp, const float* X, int64_t M, int64_t ldx,
                            const double* leaf_val, double* acc, void* direct, bool fmajor,
                            hipStream_t s) {
  const void* fn = (const void*)values_lane_kernel<T, ND>;
  const size_t lds = (size_t)h.F * (sizeof(double) + sizeof(float));
  if (lds > raise_lds_limit(fn)) fail(QTS_E_UNSUPPORTED, "internal: n_features too large");
  const int64_t grid = M * n_chunks_of(sp, kLaneRows);
  if (grid > 0x7fffffff) fail(QTS_E_UNSUPPORTED, "grid too large");
  const T *b, *cb;
  NodeConsts<T> nc;
  if constexpr (std::is_same<T, float>::value) {
    b = a.b32;
    cb = a.cb32;
    nc = d.n32;
  } else {
    b = a.b64;
    cb = a.cb64;
    nc = d.n64;
  }
  hipLaunchKernelGGL((values_lane_kernel<T, ND>), dim3((unsigned)grid), dim3(kLaneRows), lds, s,
                     a.hdr, a.feat, a.lo, a.hi, b, cb, a.b64, a.cb64, a.side, leaf_val, X, M, ldx,
                     h.F, (int32_t)fmajor, sp.path_begin(), sp.path_end(), h.n_groups,
                     bucket_index(a, sp), acc, direct, nc);
  check_hip(hipGetLastError(), "values_lane_kernel launch");
}

void launch_values_lane(const HostTable& h, const DeviceTable& d, const PathArrays& a,
                        const BucketSpan& sp, bool fp64, const float* X, int64_t M, int64_t ldx,
                        const double* leaf_val, double* acc, void* direct, bool fmajor,
                        hipStream_t s) {
  auto go = [&](auto nd) {
    constexpr int kNd = decltype(nd)::value;
    if (fp64) launch_lane_one<double, kNd>(h, d, a, sp, X, M, ldx, leaf_val, acc, direct, fmajor, s);
    else launch_lane_one<float, kNd>(h, d, a, sp, X, M, ldx, leaf_val, acc, direct, fmajor, s);
  };
  switch (sp.list[0].top) {
    case 0: go(std::integral_constant<int, 3>{}); break;
    case 1: go(std::integral_constant<int, 4>{}); break;
    case 2: go(std::integral_constant<int, 5>{}); break;
    case 3: go(std::integral_constant<int, 6>{}); break;
    default: go(std::integral_constant<int, 7>{}); break;
  }
}

// Slot 0 of every first-order row with the current leaf values folded in.
template <typename T>
__global__ void __launch_bounds__(256)
slot0_kernel(const PathHdr* __restrict__ hdr, const int32_t* __restrict__ feat,
             const float* __restrict__ lo, const float* __restrict__ hi,
             const double* __restrict__ b64, const double* __restrict__ cb64,
             const SidePath* __restrict__ side, const double* __restrict__ leaf_val, int32_t n,
             Slot0<T>* __restrict__ out) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  const PathHdr h = hdr[r];
  Slot0<T> z{T(0), T(0), T(0), 0.f, 0.f, 0};
  const int sidx = side == nullptr ? -1 : h.tree;
  if (h.d > 0 && sidx >= 0) {
    const SidePath sp = side[sidx];
    const double va = leaf_val[h.leaf];
    const double vb = leaf_val[sp.leaf_b];
    z.bm = (T)(va * sp.b_a + vb * sp.b_b);
    z.ca = (T)(va * sp.cb_a - vb * sp.b_b);
    z.cb = (T)(vb * sp.cb_b - va * sp.b_a);
    z.lo_b = sp.lo_b;
    z.hi_b = sp.hi_b;
    z.mok_b = sp.mok_b;
  } else if (h.d > 0) {
    const double v = leaf_val[h.leaf];
    const double bm = v * b64[h.off];
    z.bm = (T)bm;
    z.ca = (T)(v * cb64[h.off]);
    z.cb = (T)(-bm);
    z.lo_b = lo[h.off];
    z.hi_b = hi[h.off];
    z.mok_b = (feat[h.off] & kMissingOkBit) != 0 ? 1 : 0;
  }
  out[r] = z;
}

size_t slot0_bytes(int32_t n_rows, bool fp64) {
  return (size_t)n_rows * (fp64 ? sizeof(Slot0<double>) : sizeof(Slot0<float>));
}

void launch_slot0(const PathArrays& a, int32_t n_rows, const double* leaf_val, bool fp64,
                  void* out, hipStream_t s) {
  if (n_rows <= 0) return;
  const unsigned grid = (unsigned)((n_rows + 255) / 256);
  if (fp64)
    hipLaunchKernelGGL(slot0_kernel<double>, dim3(grid), dim3(256), 0, s, a.hdr, a.feat, a.lo,
                       a.hi, a.b64, a.cb64, a.side, leaf_val, n_rows, (Slot0<double>*)out);
  else
    hipLaunchKernelGGL(slot0_kernel<float>, dim3(grid), dim3(256), 0, s, a.hdr, a.feat, a.lo,
                       a.hi, a.b64, a.cb64, a.side, leaf_val, n_rows, (Slot0<float>*)out);
  check_hip(hipGetLastError(), "slot0_kernel launch");
}

void launch_values(const HostTable& h, const DeviceTable& d, const PathArrays& a,
                   const BucketSpan& sp, bool fp64, const float* X, int64_t M, int64_t ldx,
                   const void* slot0, double* acc, void* direct, const ValuesShape& shape,
                   int nodes, hipStream_t s, bool per_row, bool deterministic) {
  auto go = [&](auto t, auto dmax, auto nh, auto store, auto nn, auto walk) {
    launch_one<decltype(t), decltype(dmax)::value, decltype(nh)::value, decltype(store)::value,
               decltype(nn)::value, decltype(walk)::value>(
        h, d, a, sp, X, M, ldx, slot0, acc, direct, shape, s, deterministic);
  };
  using std::false_type;
  using std::true_type;
#define QTS_N(n) std::integral_constant<int, n>{}
  if (sp.dmax() == 8) {
    auto short_rows = [&](auto top) {
      const auto walk = QTS_N(kPerRow + 3 + decltype(top)::value);
      if (nodes == 4) {
        if (!fp64) go(0.f, QTS_N(8), QTS_N(4), true_type{}, QTS_N(4), walk);
        else go(0.0, QTS_N(8), QTS_N(4), false_type{}, QTS_N(4), walk);
      } else if (fp64 && deterministic) {
        go(0.0, QTS_N(8), QTS_N(8), true_type{}, QTS_N(8),
           QTS_N(kNoKeep + 3 + decltype(top)::value));
      } else if (fp64) {
        go(0.0, QTS_N(8), QTS_N(8), true_type{}, QTS_N(8), top);
      } else {
        go(0.f, QTS_N(8), QTS_N(8), true_type{}, QTS_N(8), walk);
      }
    };
    switch (sp.list[0].top) {
      case 0: short_rows(QTS_N(0)); break;
      case 1: short_rows(QTS_N(1)); break;
      case 2: short_rows(QTS_N(2)); break;
      case 3: short_rows(QTS_N(3)); break;
      default: short_rows(QTS_N(4)); break;
    }
    return;
  }
  if (!fp64 && !per_row) {
    switch (sp.dmax()) {
      case 16: go(0.f, QTS_N(16), QTS_N(8), true_type{}, QTS_N(8), QTS_N(kBatched)); break;
      case 32: go(0.f, QTS_N(32), QTS_N(8), true_type{}, QTS_N(8), QTS_N(kBatched)); break;
      default: go(0.f, QTS_N(64), QTS_N(8), true_type{}, QTS_N(8), QTS_N(kBatched)); break;
    }
  } else if (!fp64) {
    switch (sp.dmax()) {
      case 16: go(0.f, QTS_N(16), QTS_N(8), true_type{}, QTS_N(8), QTS_N(kPerRow)); break;
      case 32: go(0.f, QTS_N(32), QTS_N(8), false_type{}, QTS_N(8), QTS_N(kPerRow)); break;
      default: go(0.f, QTS_N(64), QTS_N(4), false_type{}, QTS_N(8), QTS_N(kPerRow)); break;
    }
  } else {
    switch (sp.dmax()) {
      case 16: go(0.0, QTS_N(16), QTS_N(4), false_type{}, QTS_N(8), QTS_N(kPerRow)); break;
      case 32: go(0.0, QTS_N(32), QTS_N(4), false_type{}, QTS_N(8), QTS_N(kPerRow)); break;
      default: go(0.0, QTS_N(64), QTS_N(2), false_type{}, QTS_N(8), QTS_N(kPerRow)); break;
    }
  }
#undef QTS_N
}

}  // namespace qts
