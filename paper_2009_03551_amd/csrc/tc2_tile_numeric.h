// Clustered-tile numeric kernel of the TC2 / TC2-CPSCF update for gfx950, and
// its launch for one value type and number of directions (instantiated in the
// tc2_tile_*.hip files, one per pair, so that they compile side by side).
//
// Atoms are grouped into clusters of up to CS = 8 nearby atoms.  A work item
// is a tile of output blocks (I in cluster P) x (J in cluster Q) for P <= Q,
// or a sub-tile of it.
#pragma once
#include "tc2_device.h"
#include "tc2_tile.h"

#include <algorithm>

namespace tc2 {

// ------------------------------------------------------------------ tile numeric
// A work item is a sub-tile of SP rows of cluster P x TQ columns of cluster Q
// (a tile of 8 x 8 output blocks is split into (8/SP)(8/TQ) sub-tiles), which a
// block of NWB waves computes in parts of PS x PT output blocks, or (FINE) one
// part of a sub-tile.  The common columns K of the two panels are found once per
// item.  For each part the block walks them 64 at a time, a column per lane:
// which blocks the outputs need there (a block of a zero matrix, or one without
// a partner, is needed by none) and where they stand in a list of blocks; this
// plan is a word per output and column.  The columns then go through a ring of
// blocks in LDS in stages, as many columns as fit in half of it: while the
// products of a stage run, the next one is copied straight from global memory
// with global_load_lds (16 B per lane, the b stored columns of a block only).
// One barrier per stage.
//
// Measured (MI355X).  Reading the operands from global memory instead (no LDS,
// no barrier) is bound by the fabric behind L2 (9.7 TB/s of operands): 877 ms
// per solve of a 1728-atom lattice in three directions, against 675 here; the
// kernel before, a column and two barriers at a time in blocks of 16 x 16 with
// every matrix of a present block staged, took 1001.  What remains: an FP64 or
// FP32 MFMA leaves no issue slot to the vector ALU of its SIMD (measured with
// two waves, any priority or age), so matrix time (300 ms of that solve) and
// vector time (3.6 instructions per MFMA, about 100) add up; the rest is waits
// of a stage for its busiest wave (1.5 times the mean) and for copies of columns
// too large to stand in the ring beside the stage in use.  Hence the packed
// plan words, scalar addresses and arguments read where they are used, and
// fragments read without conditions while the products before run (with
// conditions the compiler waited at each: 688 ms, and 346 instead of 333 for
// 1000 atoms in one direction).
// Sub-tiles dealt to the XCDs in chunks (L2 hits 10 -> 17 %) and half the blocks
// per CU (-40 %) did not help.
typedef float f2v __attribute__((ext_vector_type(2)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef int i2v __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int KLMAX_ALL = 2048;  // most common columns held in LDS per pass over P's panel
constexpr int KLQ_BITS = 20;  // kl: offset in the pass (12 bits) | offset in Q's panel (20 bits)
static_assert((1 << (32 - KLQ_BITS)) >= KLMAX_ALL && (1 << KLQ_BITS) >= MAX_SYS_BITS, "kl packing");
// Waves per block.  With at most one direction a block of 16 waves has a CU to
// itself and computes a whole sub-tile, 8 x 8 outputs, at a time: columns are
// planned and copied once for all of them (1000-atom lattice in one direction
// 333 -> 320 ms).  With more, an output has 7 products per column, a stage lasts
// longer than its waits, and two blocks of 8 waves fill each other's gaps (1728
// atoms in three directions: 677 ms, with 16 waves 769).
constexpr int waves(bool fine, int D) { return fine || D >= 2 ? 8 : 16; }
// With the network or logging, updates of few sub-tiles run in parts only where a
// sub-tile otherwise takes several parts one after another (FP32 and bfloat16
// values, two or three directions: 343 atoms in three, FP32, logging: 105 ms per
// solve whole, 90 in parts; 600-atom chain 27.6, 19.0).
constexpr bool learn_parts(int D, int SP, int TQ) { return D >= 2 && SP * TQ > 16; }

// the 1 + D block norms of an entry
template <int D>
__device__ __forceinline__ void load_norms(const float* bn, int e, float* n) {
  const float* p = bn + (size_t)e * (1 + D);
  if constexpr (D == 3) {
    const f4v v = *(const f4v*)p;
    n[0] = v[0]; n[1] = v[1]; n[2] = v[2]; n[3] = v[3];
  } else if constexpr (D == 1) {
    const f2v v = *(const f2v*)p;
    n[0] = v[0]; n[1] = v[1];
  } else {
#pragma unroll
    for (int m = 0; m <= D; ++m) n[m] = p[m];
  }
}

// The kernel arguments, read anew where they are used: held in registers over
// the whole kernel they would spill scalar registers in its inner loops.
typedef const __attribute__((address_space(4))) TileArgs* KArgs;
__device__ __forceinline__ KArgs kargs() {
  KArgs k = (KArgs)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(k));
  return k;
}

template <typename T>
__device__ __forceinline__ Acc<T> zero_acc() {
  Acc<T> c;
#pragma unroll
  for (int r = 0; r < 4; ++r) c.v[r] = 0;
  return c;
}
__device__ __forceinline__ void add_wide(AccW& w, const Acc<float>& c) {
#pragma unroll
  for (int r = 0; r < 4; ++r) w.v[r] += (double)c.v[r];
}

// inclusive sum over the lanes of a wave (six data-parallel adds)
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
  return v;
}

// Copy one block of n bytes (a multiple of 16, at most 2048) from global memory
// at src to LDS offset dst, both wave-uniform, 16 B per lane; off = 16 lane.
// The copy bypasses registers; the caller waits for it (vmcnt) before the
// barrier that lets the block be read.  In assembly, because behind the builtin
// the compiler waits for every copy in flight before it reads any LDS address,
// which would end the overlap of the copies of one stage with the products of
// another.  m0 is named as clobbered so that no use of it by the compiler can
// stand across the copy (the compiler warns that the register is reserved, that
// is, not kept across assembly, as is meant).  The s_nop covers an SGPR of src
// written by a readlane just before.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_copy(const char* src, unsigned dst, int off, int n) {
  if (off < n)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(dst), "v"(off), "s"(src) : "memory", "m0");
  if (n > 1024 && off + 1024 < n)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024"
                 :: "s"(dst), "v"(off), "s"(src) : "memory", "m0");
}
#pragma clang diagnostic pop

// the trace sums of a sub-tile from those of its outputs (NQ apart): ng groups of go
__device__ __forceinline__ double sub_sum(const double* row, int ng, int go) {
  double sum = 0.0;
  for (int g = 0; g < ng; ++g) {
    double part = 0.0;
    for (int o = 0; o < go; ++o) part += row[(g * go + o) * NQ];
    sum += part;
  }
  return sum;
}

// W (FP32 values only): the FP32 MFMA product of each column block K is added
// to FP64 accumulators, so that only the short sum inside one block runs in
// FP32 and the long sum over K runs in FP64.
// FK: the block size needs all four K-steps of the padded tile (b > 12).
// WS: the trace sums of a sub-tile are taken over TQ WS groups of SP / WS
// outputs, group (h, v) holding (I_s, J_{(s+v) mod TQ}) for the rows s of part
// h, first within a group, then over the groups: a fixed order, whichever
// wave computed which output.
// A bfloat16 split is made once per staged block, by the wave that copied it, in
// place: h, m and l of the values of lane l's fragment at 8 l in three planes of
// 512 B (split at each of its 4 uses instead: 343 atoms in three directions, two
// thirds of the time in this kind, 134 ms per solve against 128).
// LEARN: with the skip network or feature logging (kept apart, as its code
// would take registers from the products).
template <typename T, int D, int SP, int TQ, bool BF, bool W, bool FK, int WS, bool LEARN, bool FINE>
__device__ __forceinline__ void tile_numeric() {
  constexpr int PER = (1 + D) * BS;                       // elements per entry
  constexpr int NOUT = SP * TQ;                           // outputs of the sub-tile
  KArgs k = kargs();
  // groups of the trace sums and outputs per group (tests compare with WS = 1)
  const int GO = k->column_sums ? SP : SP / WS, NG = NOUT / GO;
  static_assert(SP % WS == 0, "rows of the sub-tile split evenly over its groups");
  // place of output (row r, column q) of the sub-tile in that order
  auto sum_row = [&](int r, int q) { return ((r / GO) * TQ + (q + TQ - r % TQ) % TQ) * GO + r % GO; };
  constexpr int SUBS = (CS / SP) * (CS / TQ);
  // part of a sub-tile in work at a time: with two or more directions 4 x 4
  // outputs, two per wave, else all, at most four (64 accumulator registers in FP64)
  constexpr int NWB = waves(FINE, D), KLMAX = NWB == 8 ? KLMAX_ALL / 2 : KLMAX_ALL;
  constexpr int PS = FINE ? 2 : (D >= 2 ? 4 : SP), PT = FINE || D >= 2 ? 4 : TQ;
  constexpr int NO = PS * PT / NWB;                       // outputs per wave
  constexpr int PARTS = NOUT / (PS * PT);
  constexpr int NE = PS + PT;                             // entries per column
  static_assert(NE <= NWB, "wave x copies entry x of a column");
  constexpr int NM = 1 + D;                               // matrices
  constexpr unsigned MM = (1u << NM) - 1u;
  constexpr int BPE = NM <= 2 ? 2 : 4;                    // plan bits per entry
  constexpr unsigned EM = (1u << BPE) - 1u;
  static_assert(NE * BPE <= 32 && NO >= 1, "plan words");
  constexpr int PLC = NWB * 64;                           // columns planned at once
  constexpr int SROWS = FINE ? PS * PT : NOUT;            // rows of trace sums kept here
  constexpr int FIXED = KLMAX * 4 + SROWS * NQ * 8 + PLC * 4 + PS * PT * 4 + 128;
  constexpr int RING = (160 * 1024 / (16 / NWB) - FIXED) / 64 * 64;     // bytes of staged blocks
  static_assert(RING >= NE * NM * BS * (BF && W ? 6 : (int)sizeof(T)), "a column of 16 x 16 blocks must fit");
  static_assert(!LEARN || RING >= MLP_NP * 4, "the network shares the stage memory");
  __shared__ __attribute__((aligned(16))) char ring[RING + 16];
  __shared__ unsigned kl[KLMAX];
  __shared__ int wcount[NWB];
  __shared__ double spart[SROWS][NQ];
  __shared__ unsigned sown[PS];  // row s: bit t set when output (I_s, J_t) of the part is computed
  __shared__ unsigned s_need[PLC];
  __shared__ int s_np[PS * PT];  // block triples of the outputs of the part
  __shared__ int s_lb;

  constexpr int NT = NWB * 64;
  const T* X = (const T*)k->xv;
  const int b = k->b, ksteps = k->ksteps;
  constexpr bool SPLIT = BF && W;
  const int bbytes = ((LEARN && BF && !W) ? BP : b) * BP * (int)sizeof(T);  // copied of a block
  const int sbytes = SPLIT ? 3 * BS * 2 : (BF ? BP : b) * BP * (int)sizeof(T);  // a slot
  const int nslot = RING / sbytes;                        // blocks the ring holds
  const int rbytes = nslot * sbytes;
  const unsigned ring_lds = (unsigned)(unsigned long long)(lds_void*)ring;  // its LDS offset
  auto wrap = [&](int p) { return p >= rbytes ? p - rbytes : p; };
  unsigned long long nprod = 0;                           // block products issued by this wave
  // A slot holds the b columns of a block; the lanes of the last K-step whose
  // column is beyond them read a zero behind the ring.  Bfloat16 fragments read
  // all 16 columns: the others of a slot are cleared here, and not written by
  // the copies of b columns (the network overwrites them: with it the copies
  // take the zeros along).
  for (int i = threadIdx.x; i < (RING + 16) / 4; i += NT)
    if (BF || i >= RING / 4) ((int*)ring)[i] = 0;
  const bool tail = (threadIdx.x & 63) < (b - 4 * (ksteps - 1)) * BP;  // in the last K-step

  // One sub-tile per block, or (k->work set) a persistent grid in which every
  // block takes the next sub-tile from an atomic counter until all are done;
  // the sub-tile count then comes from the device (tile_rp[nc]).
  int total = (k->n_tiles_dev ? *k->n_tiles_dev : k->n_tiles) * SUBS;
  if ((!LEARN || learn_parts(D, SP, TQ)) && (total <= k->fine_subs) != FINE) return;  // the other split's
  if constexpr (FINE) total *= PARTS;
  for (int it = 0;; ++it) {
    k = kargs();
    int lb;
    if (k->work) {
      if (threadIdx.x == 0) s_lb = atomicAdd(k->work, 1);
      __syncthreads();
      lb = __builtin_amdgcn_readfirstlane(s_lb);
    } else {
      lb = it == 0 ? (int)blockIdx.x : total;
    }
    if (lb >= total) break;
    const int part0 = FINE ? lb % PARTS : 0;
    if constexpr (FINE) lb /= PARTS;
    const int tile = lb / SUBS, sub = lb - tile * SUBS;
    const int ph = (sub / (CS / TQ)) * SP, qh = (sub % (CS / TQ)) * TQ;
    const int P = k->tile_p[tile], Q = k->tile_q[tile];
    // threadIdx-derived values are made opaque per sub-tile, so that the
    // compiler does not hoist per-lane addresses out of the sub-tile loop and
    // keep them live across it (register pressure)
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);  // wave-uniform (scalar)
    // the members of a cluster ascend: no output of a sub-tile below the
    // diagonal of a diagonal tile is an upper block (no work, zero sums)
    if (!FINE && P == Q && ph > qh + TQ - 1) {
      if (t < NQ) k->partial[(size_t)lb * NQ + t] = 0.0;
      __syncthreads();
      continue;
    }
    const int sys = k->clus_sys[P];
    const bool square = k->branch[sys] != 0;
    const double eps = k->eps[sys];
    const int pp0 = k->panel_rp[P], pp1 = k->panel_rp[P + 1];
    const int pq0 = k->panel_rp[Q], nq = k->panel_rp[Q + 1] - pq0;
    for (int i = t; i < SROWS * NQ; i += NT) (&spart[0][0])[i] = 0.0;

    // common columns of the pass [base, end) over P's panel with Q's panel -> kl
    auto build_kl = [&](int base, int end) {
      int nm = 0;
      __syncthreads();  // the readers of the last pass are done
      for (int c0 = base; c0 < end; c0 += NT) {
        const int idx = c0 + t;
        int j = -1;
        if (idx < end) j = (P == Q) ? idx - pp0 : bsearch_eq(k->panel_k + pq0, nq, k->panel_k[idx]);
        const bool found = j >= 0;
        const unsigned long long mask = __ballot(found);
        if (lane == 0) wcount[wave] = __popcll(mask);
        __syncthreads();
        int off = nm, tot = 0;
#pragma unroll
        for (int w = 0; w < NWB; ++w) {
          const int c = wcount[w];
          off += (w < wave) ? c : 0;
          tot += c;
        }
        if (found)
          kl[off + __popcll(mask & ((1ull << lane) - 1ull))] =
              ((unsigned)(idx - base) << KLQ_BITS) | (unsigned)j;
        nm += tot;
        __syncthreads();
      }
      return __builtin_amdgcn_readfirstlane(nm);
    };
    // columns of P's panel taken per pass (a smaller chunk can be forced to
    // test the multi-pass path on small inputs)
    const int KLC = (k->kl_chunk > 0 && k->kl_chunk < KLMAX) ? k->kl_chunk : KLMAX;
    const bool one_pass = pp1 - pp0 <= KLC;
    int nm = 0;
    if (one_pass) nm = build_kl(pp0, pp1);

    for (int part = part0; part < (FINE ? part0 + 1 : PARTS); ++part) {
      const int s0 = (part / (TQ / PT)) * PS, t0 = (part % (TQ / PT)) * PT;  // in the sub-tile
      if (P == Q && ph + s0 > qh + t0 + PT - 1) continue;
      k = kargs();
      const int* rowI = k->clus_atom + P * CS + ph + s0;
      const int* rowJ = k->clus_atom + Q * CS + qh + t0;

      // outputs of this wave: o -> (row so, column to) of the part.  The waves
      // of a SIMD hold one output per row and column of the part.  Lane o
      // holds what belongs to output o: its rows I and J, the entry of the old
      // block (I, J) or -1, and its log slot.
      auto row_of = [&](int o) { return (wave / PT) * NO + o; };
      auto col_of = [&](int o) { return (row_of(o) + wave) % PT; };
      int my_I = -1, my_J = -1, my_e = -1, my_slot = -1;
      if (lane < NO) {
        my_I = rowI[row_of(lane)];
        my_J = rowJ[col_of(lane)];
      }
      // outputs to compute (bit o)
      unsigned own_mask = (unsigned)__ballot(my_I >= 0 && my_J >= 0 && (P != Q || my_I <= my_J));
      if ((own_mask >> lane) & (lane < NO ? 1u : 0u)) {
        const int r0 = k->rp[my_I];
        const int f = bsearch_eq(k->ci + r0, k->rp[my_I + 1] - r0, my_J);
        my_e = f >= 0 ? r0 + f : -1;
      }

      // ---- exact screen: ||C_IJ|| <= sum_K ||A_IK|| ||B_KJ|| (+ 2 ||X_IJ|| on
      // the DOUBLE branch); an off-diagonal output whose bound is below eps
      // for X0 and every X1_d is certainly dropped, so its products are
      // skipped.  The learned screen then evaluates the skip network on
      // features of the remaining outputs and skips those it predicts to be
      // dropped; features and the true outcome can be logged for training.
      if (LEARN || k->skip) {
        float* th = (float*)ring;
        if (LEARN && k->skip == 2) {
          __syncthreads();  // the products of the last part have read the ring
          for (int p = t; p < MLP_NP; p += NT) {
            int q = p;
            if (p >= MLP_W2 && p < MLP_B2) {  // transpose W2 (j, k) -> (k, j)
              const int j = (p - MLP_W2) / MLP_NH, k = (p - MLP_W2) - j * MLP_NH;
              q = MLP_W2 + k * MLP_NH + j;
            }
            th[q] = k->mlp[p];
          }
          __syncthreads();
        }
        double bsum[NO][NM];
        float bmax[NO];
        int bcnt[NO];
#pragma unroll
        for (int o = 0; o < NO; ++o) {
          bmax[o] = 0.f;
          bcnt[o] = 0;
#pragma unroll
          for (int m = 0; m < NM; ++m) bsum[o][m] = 0.0;
        }
        for (int base = pp0; base < pp1; base += KLC) {
          if (!one_pass) nm = build_kl(base, min(pp1, base + KLC));
          for (int c = lane; c < nm; c += 64) {
            // the entries, then the norms of all outputs in flight together
            // (entry 0 stands in for an absent one)
            const unsigned kk = kl[c];
            const int* pa = k->panel_e + (size_t)(base + (int)(kk >> KLQ_BITS)) * CS + ph + s0;
            const int* pb = k->panel_e + (size_t)(pq0 + (int)(kk & ((1u << KLQ_BITS) - 1u))) * CS + qh + t0;
            int eA[NO], eB[NO];
#pragma unroll
            for (int o = 0; o < NO; ++o) {
              eA[o] = pa[row_of(o)];
              eB[o] = pb[col_of(o)];
            }
            float na[NO][NM], nb[NO][NM];
#pragma unroll
            for (int o = 0; o < NO; ++o) {
              load_norms<D>(k->bn, max(eA[o], 0), na[o]);
              load_norms<D>(k->bn, max(eB[o], 0), nb[o]);
            }
#pragma unroll
            for (int o = 0; o < NO; ++o) {
              if (eA[o] < 0 || eB[o] < 0) continue;
              if constexpr (LEARN) {
                bcnt[o] += 1;
                bmax[o] = fmaxf(bmax[o], na[o][0] * nb[o][0]);
              }
              bsum[o][0] += (double)na[o][0] * nb[o][0];
#pragma unroll
              for (int d = 0; d < D; ++d)
                bsum[o][1 + d] += (double)na[o][0] * nb[o][1 + d] + (double)na[o][1 + d] * nb[o][0];
            }
          }
        }
#pragma unroll
        for (int o = 0; o < NO; ++o) {
          const int I = __builtin_amdgcn_readlane(my_I, o), J = __builtin_amdgcn_readlane(my_J, o);
          const int eIJ = __builtin_amdgcn_readlane(my_e, o);
          if (!((own_mask >> o) & 1u) || I == J) continue;
          double bnd[NM];
          bool drop = true;
#pragma unroll
          for (int m = 0; m < NM; ++m) {
            bnd[m] = wave_sum(bsum[o][m]);
            if (!square && eIJ >= 0) bnd[m] += 2.0 * (double)k->bn[(size_t)eIJ * NM + m];
            // a relative margin covers the rounding of the float block norms
            drop = drop && bnd[m] * (1.0 + 1e-6) < eps;
          }
          if (k->skip && drop) {
            own_mask &= ~(1u << o);
            if (lane == 0) atomicAdd(k->screened, 1ull);
            continue;
          }
          if constexpr (LEARN) {
            // features of the candidate (scaled logs relative to eps)
            const int cnt = (int)wave_sum((double)bcnt[o]);
            float mx = bmax[o];
#pragma unroll
            for (int sh = 32; sh > 0; sh >>= 1) mx = fmaxf(mx, __shfl_xor(mx, sh, 64));
            double b1 = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) b1 = fmax(b1, bnd[1 + d]);
            const double le = log10(eps > 0.0 ? eps : 1e-300);
            float feat[MLP_NF];
            feat[0] = (float)(0.1 * (log10(fmax(bnd[0], 1e-300)) - le));
            feat[1] = (float)(0.1 * (log10(fmax(b1, 1e-300)) - le));
            feat[2] = (float)(0.1 * (log10(fmax((double)mx, 1e-300)) - le));
            feat[3] = (float)(0.5 * log10(1.0 + cnt));
            double r = 0.0;
            if (k->xyz) {
              double d2 = 0.0;
              for (int i = 0; i < 3; ++i) {
                const double dd = k->xyz[3 * I + i] - k->xyz[3 * J + i];
                d2 += dd * dd;
              }
              r = sqrt(d2);
            }
            feat[4] = (float)(0.1 * r);
            feat[5] = eIJ >= 0
                          ? (float)(0.1 * (log10(fmax((double)k->bn[(size_t)eIJ * NM], 1e-300)) - le))
                          : -3.f;
            feat[6] = 0.05f * (float)k->iter;
            feat[7] = square ? 1.f : 0.f;
            bool net_skip = false;
            float z = 0.f;
            if (k->skip == 2) {
              z = mlp_logit_wave(th, feat, lane);
              // the network may skip only an output whose exact bound is below
              // mlp_cap * eps for every matrix, and never, on the DOUBLE branch,
              // a stored block whose 2 ||X_IJ|| alone reaches eps
              bool allowed = true;
              double bmx = 0.0;
#pragma unroll
              for (int m = 0; m < NM; ++m) {
                allowed = allowed && bnd[m] < (double)k->mlp_cap * eps;
                if (!square && eIJ >= 0)
                  allowed = allowed && 2.0 * (double)k->bn[(size_t)eIJ * NM + m] < eps;
                bmx = fmax(bmx, bnd[m]);
              }
              net_skip = allowed && z > k->mlp_z;
              if (net_skip && lane == 0) {
                atomicAdd(k->mlp_skipped, 1ull);
                atomicAdd(&k->mlp_bsum[sys], bmx);
              }
            }
            if (k->log_cap > 0) {
              int at = 0;
              if (lane == 0) at = (int)atomicAdd(k->log_count, 1ull);
              at = __builtin_amdgcn_readfirstlane(at);
              if (at >= 0 && at < k->log_cap) {
                float v = z;
#pragma unroll
                for (int i = 0; i < MLP_NF; ++i) v = (lane == i) ? feat[i] : v;
                if (lane < MLP_NF) k->log_x[(long long)at * MLP_NF + lane] = v;
                if (lane == MLP_NF && k->log_z) k->log_z[at] = z;
                // the outcome of an output the network skipped is not known
                if (lane == 0 && net_skip) k->log_y[at] = -1.f;
                if (lane == o) my_slot = at;
              }
            }
            if (net_skip) own_mask &= ~(1u << o);
          }
        }
      }

      // outputs computed by this block, as row masks
      __syncthreads();  // the readers of sown and of the ring are done
      if (t < PS) sown[t] = 0u;
      if (t < PS * PT) s_np[t] = 0;
      __syncthreads();
      own_mask = __builtin_amdgcn_readfirstlane(own_mask);
      if (lane < NO && ((own_mask >> lane) & 1u)) atomicOr(&sown[row_of(lane)], 1u << col_of(lane));
      __syncthreads();
      // the same masks over the bits per entry of the plan: partners of
      // row s among the columns, and of column q among the rows
      unsigned ownA[PS], ownB[PT], own_any = 0u;
#pragma unroll
      for (int q = 0; q < PT; ++q) ownB[q] = 0u;
#pragma unroll
      for (int r = 0; r < PS; ++r) {
        const unsigned w = __builtin_amdgcn_readfirstlane(sown[r]);
        own_any |= w;
        ownA[r] = 0u;
#pragma unroll
        for (int q = 0; q < PT; ++q)
          if ((w >> q) & 1u) {
            ownA[r] |= EM << (BPE * q);
            ownB[q] |= EM << (BPE * r);
          }
      }
      if (!own_any) continue;

      Acc<T> acc[W ? 1 : NO][W ? 1 : NM];
      AccW wacc[W ? NO : 1][W ? NM : 1];
#pragma unroll
      for (int o = 0; o < NO; ++o)
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if constexpr (W) wacc[o][m].v[r] = 0.0;
            else acc[o][m].v[r] = 0;
          }

      // Products of one column for output o: staged blocks of X_IK from ring
      // offset pa and of X_JK from pb on, na and nb the matrices staged there.  A
      // staged matrix is nonzero and has a partner, so the products of the
      // pair are those whose operands are both staged (others would add exact
      // zeros).
      auto column = [&](int o, int pa, int pb, unsigned na, unsigned nb) {
        auto at = [&](int p, unsigned n, int m) { return wrap(p + __popc(n & ((1u << m) - 1u)) * sbytes); };
        nprod += __popc(na & nb & 1u) + ((na & 1u) ? __popc(nb >> 1) : 0) + ((nb & 1u) ? __popc(na >> 1) : 0);
        if constexpr (BF) {
          if constexpr (W) {
            // bfloat16 three-way split: each operand value v = h + m + l; the six
            // cross products above 2^-24 of the leading term (l h, h l, m m, m h,
            // h m, h h, smallest first) run as 16x16x16 bfloat16 MFMAs into an
            // FP32 temporary per column block, which is added to the FP64 sums
            struct Part {
              s4 v[3];
            };
            auto part = [&](int p) {
              Part f;
#pragma unroll
              for (int k = 0; k < 3; ++k) f.v[k] = *(const s4*)(ring + p + k * 512 + lane * 8);
              return f;
            };
            auto prod3 = [&](Acc<float>& c, const Part& u, const Part& v) {
              mfma_bf16(c, u.v[2], v.v[0]);
              mfma_bf16(c, u.v[0], v.v[2]);
              mfma_bf16(c, u.v[1], v.v[1]);
              mfma_bf16(c, u.v[1], v.v[0]);
              mfma_bf16(c, u.v[0], v.v[1]);
              mfma_bf16(c, u.v[0], v.v[0]);
            };
            const Part a0 = part(pa), b0 = part(pb);
            if (na & nb & 1u) {
              Acc<float> tmp = zero_acc<float>();
              prod3(tmp, a0, b0);
              add_wide(wacc[o][0], tmp);
            }
#pragma unroll
            for (int d = 0; d < D; ++d) {
              const Part xb = part(at(pb, nb, 1 + d)), xa = part(at(pa, na, 1 + d));
              asm volatile("" ::: "memory");  // read here, not moved to the products
              const bool p0 = na & (nb >> (1 + d)) & 1u, p1 = (na >> (1 + d)) & nb & 1u;
              if (!(p0 || p1)) continue;
              Acc<float> tmp = zero_acc<float>();
              if (p0) {
                prod3(tmp, a0, xb);
                if (p1) prod3(tmp, xa, b0);
              } else {
                prod3(tmp, xa, b0);
              }
              add_wide(wacc[o][1 + d], tmp);
            }
          } else {
            // bfloat16 operands: one 16x16x16 MFMA per block product
            s4 a0, b0;
            if (na & 1u) a0 = bf16_frag((const float*)(ring + pa), lane);
            if (nb & 1u) b0 = bf16_frag((const float*)(ring + pb), lane);
            if (na & nb & 1u) mfma_bf16(acc[o][0], a0, b0);
#pragma unroll
            for (int d = 0; d < D; ++d) {
              if (na & (nb >> (1 + d)) & 1u)
                mfma_bf16(acc[o][1 + d], a0, bf16_frag((const float*)(ring + at(pb, nb, 1 + d)), lane));
              if ((na >> (1 + d)) & nb & 1u)
                mfma_bf16(acc[o][1 + d], bf16_frag((const float*)(ring + at(pa, na, 1 + d)), lane), b0);
            }
          }
        } else {
          // operand fragments of a staged block: all K-steps at once
          auto frag = [&](int p, T* f) {
            const int q = p + lane * (int)sizeof(T), last = FK ? 3 : ksteps - 1;
            const int ql = tail ? q : RING - last * 64 * (int)sizeof(T);
#pragma unroll
            for (int kk = 0; kk < (FK ? 4 : 3); ++kk)
              if (kk <= last) f[kk] = *(const T*)(ring + (kk == last ? ql : q) + kk * 64 * (int)sizeof(T));
          };
          Acc<T> tmp[W ? NM : 1];
          if constexpr (W) {
#pragma unroll
            for (int m = 0; m < NM; ++m)
#pragma unroll
              for (int r = 0; r < 4; ++r) tmp[m].v[r] = 0.f;
          }
          Acc<T>* dst = W ? tmp : &acc[W ? 0 : o][0];
          auto prod = [&](Acc<T>& cc, const T* ra, const T* rb) {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
              if (!FK && kk >= ksteps) break;
              mfma(cc, ra[kk], rb[kk]);
            }
          };
          // X0's fragments serve all products; those of a direction are read
          // while the products before run.  A matrix not staged is read as well
          // (from a slot behind, unused): between reads under conditions the
          // compiler waits for the ones before.
          T a0[4], b0[4], xa[4], xb[4];
          auto load = [&](int p, T* f) {
            frag(p, f);
            asm volatile("" ::: "memory");  // here, not moved to the products
          };
          load(pa, a0);
          load(pb, b0);
          if constexpr (D > 0) {
            load(at(pb, nb, 1), xb);
            load(at(pa, na, 1), xa);
          }
          if (na & nb & 1u) prod(dst[0], a0, b0);
#pragma unroll
          for (int d = 0; d < D; ++d) {
            if (na & (nb >> (1 + d)) & 1u) prod(dst[1 + d], a0, xb);
            if (d + 1 < D) load(at(pb, nb, 2 + d), xb);
            if ((na >> (1 + d)) & nb & 1u) prod(dst[1 + d], xa, b0);
            if (d + 1 < D) load(at(pa, na, 2 + d), xa);
          }
          if constexpr (W) {
            if (na & nb & 1u) {
#pragma unroll
              for (int r = 0; r < 4; ++r) wacc[o][0].v[r] += (double)tmp[0].v[r];
            }
#pragma unroll
            for (int d = 0; d < D; ++d)
              if (((na & (nb >> (1 + d))) | ((na >> (1 + d)) & nb)) & 1u) {
#pragma unroll
                for (int r = 0; r < 4; ++r) wacc[o][1 + d].v[r] += (double)tmp[1 + d].v[r];
              }
          }
        }
      };

      // ---- plan of the products.  A round of up to PLC columns, 64 per wave, is
      // planned at once, a column per lane: which matrices of which entries its
      // outputs need (BPE bits per entry) and how many blocks that makes, as
      // sums over its 64 columns.  From these two words of a column a wave
      // derives what it needs to know itself: for its outputs, where their
      // operands stand, and for the entries it copies, which blocks to copy.
      //  send: blocks needed up to and including the column (from the chunk start)
      //  word[o]: needed blocks before the column (11 bits) << 18 | offsets of the
      //    blocks of X_IK and X_JK within the column (5 + 5 bits) << 8 | the
      //    matrices staged of X_JK, X_IK (4 + 4 bits); 0: no product
      //  ce, cw: entry this wave copies (waves from NE on: none), and its first
      //    block (chunk) << 4 | matrices needed
      struct Plan {
        int send;
        unsigned word[NO];
        int ce;
        unsigned cw;
      };
      auto plan_round = [&](int base, int r0) {
        KArgs k = kargs();
        const int c = r0 + wave * 64 + lane;
        unsigned mA = 0u, mB = 0u, hA = 0u, hB = 0u;
        __syncthreads();  // the readers of the last round are done
        if (r0 + wave * 64 < nm) {
          if (c < nm) {
            const unsigned kk = kl[c];
            const int* ea = k->panel_e + (size_t)(base + (int)(kk >> KLQ_BITS)) * CS + ph + s0;
            const int* eb = k->panel_e + (size_t)(pq0 + (int)(kk & ((1u << KLQ_BITS) - 1u))) * CS + qh + t0;
            int e[NE];
#pragma unroll
            for (int x = 0; x < PS; x += 2) {
              const i2v v = *(const i2v*)(ea + x);
              e[x] = v[0], e[x + 1] = v[1];
            }
#pragma unroll
            for (int x = 0; x < PT; x += 2) {
              const i2v v = *(const i2v*)(eb + x);
              e[PS + x] = v[0], e[PS + x + 1] = v[1];
            }
            // all masks in flight at once (entry 0 stands in for an absent one)
            unsigned mk[NE];
#pragma unroll
            for (int x = 0; x < NE; ++x) mk[x] = MM;
            if (k->xmask) {
#pragma unroll
              for (int x = 0; x < NE; ++x) mk[x] = k->xmask[max(e[x], 0)];
            }
#pragma unroll
            for (int x = 0; x < NE; ++x) {
              const int ex = e[x];
              const unsigned m = ex >= 0 ? mk[x] & MM : 0u;
              if (x < PS) {
                mA |= m << (BPE * x);
                hA |= (ex >= 0 ? 1u : 0u) << x;
              } else {
                mB |= m << (BPE * (x - PS));
                hB |= (ex >= 0 ? 1u : 0u) << (x - PS);
              }
            }
          }
          // block triples of every output
          int cnt = 0;
#pragma unroll
          for (int r = 0; r < PS; ++r)
#pragma unroll
            for (int q = 0; q < PT; ++q) {
              const int n = __popcll(__ballot(((hA >> r) & (hB >> q) & 1u) != 0u));
              cnt = lane == r * PT + q ? n : cnt;
            }
          if (lane < PS * PT) atomicAdd(&s_np[lane], cnt);
          // needed matrices: X0 with any partner's nonzero matrix, X1_d with a
          // partner's nonzero X0
          static_assert(PS * BPE <= 16 && PT * BPE <= 16, "bits of a side");
          auto fold = [](unsigned u) {
            u |= u >> 8;
            u |= u >> 4;
            if (BPE == 2) u |= u >> 2;
            return u;
          };
          auto wants = [](unsigned u) { return ((u & EM) ? 1u : 0u) | ((u & 1u) ? EM & ~1u : 0u); };
          unsigned nA = 0u, nB = 0u;
#pragma unroll
          for (int r = 0; r < PS; ++r) nA |= wants(fold(mB & ownA[r])) << (BPE * r);
#pragma unroll
          for (int q = 0; q < PT; ++q) nB |= wants(fold(mA & ownB[q])) << (BPE * q);
          nA &= mA;
          nB &= mB;
          const unsigned w = nA | (nB << (PS * BPE));  // 0 past the last column
          s_need[c - r0] = w;
        }
        __syncthreads();
      };
      auto take_chunk = [&](int base, int r0, int c0, Plan& p) {
        KArgs k = kargs();
        const unsigned w = s_need[c0 - r0 + lane];
        p.send = wave_scan(__popc(w));
        const unsigned kk = kl[min(c0 + lane, nm - 1)];
        const int x = wave;
        const size_t row = x < PS ? (size_t)(base + (int)(kk >> KLQ_BITS)) * CS + ph + s0 + x
                                  : (size_t)(pq0 + (int)(kk & ((1u << KLQ_BITS) - 1u))) * CS + qh + t0 + min(x - PS, PT - 1);
        const int at_e = k->panel_e[row];
        const unsigned first = (unsigned)(p.send - __popc(w));
        auto below = [&](int x) { return (unsigned)__popc(w & ((1u << (BPE * x)) - 1u)); };
#pragma unroll
        for (int o = 0; o < NO; ++o) {
          const int so = row_of(o), to = PS + col_of(o);
          const unsigned na = (w >> (BPE * so)) & EM, nb = (w >> (BPE * to)) & EM;
          const bool any = ((na & 1u) && nb) || ((nb & 1u) && na);
          p.word[o] = any && ((own_mask >> o) & 1u)
                          ? (first << 18) | (below(to) << 13) | (below(so) << 8) | (nb << 4) | na
                          : 0u;
        }
        p.cw = x < NE ? ((first + below(x)) << 4) | ((w >> (BPE * x)) & EM) : 0u;
        p.ce = at_e;
        asm volatile("" : "+v"(p.ce));  // loaded before the copies below (the compiler would wait for those too)
      };

      // f(slot offset, matrix, entry) for the blocks that this wave copies of the
      // columns [c0, c1) of plan p, block n of the chunk in slot n + shift
      // (modulo the ring)
      auto each_block = [&](const Plan& p, int c0, int c1, int shift, auto&& f) {
        unsigned long long todo = __ballot(lane >= c0 && lane < c1 && (p.cw & 15u));
        while (todo) {
          const int l = __ffsll((long long)todo) - 1;
          todo &= todo - 1;
          const int e = __builtin_amdgcn_readlane(p.ce, l);
          const unsigned w = (unsigned)__builtin_amdgcn_readlane((int)p.cw, l);
          unsigned n = w & 15u;
          int dst = wrap(((int)(w >> 4) + shift) * sbytes);
          while (n) {
            const int m = __ffs((int)n) - 1;
            n &= n - 1;
            f(dst, m, e);
            dst = wrap(dst + sbytes);
          }
        }
      };
      auto copy = [&](const Plan& p, int c0, int c1, int shift) {
        each_block(p, c0, c1, shift, [&](int dst, int m, int e) {
          lds_copy((const char*)(X + (size_t)e * PER + (size_t)m * BS), ring_lds + dst, lane * 16, bbytes);
        });
      };
      // split the blocks that copy() with the same arguments has put in place
      auto split_own = [&](const Plan& p, int c0, int c1, int shift) {
        each_block(p, c0, c1, shift, [&](int dst, int, int) {
          s4 h, m, l;
          bf16_split3((const float*)(ring + dst), lane, b, h, m, l);
          s4* out = (s4*)(ring + dst) + lane;
          asm volatile("" ::: "memory");  // the block is in registers
          out[0] = h;
          out[64] = m;
          out[128] = l;
        });
      };

      for (int base = pp0; base < pp1; base += KLC) {
        if (!one_pass) nm = build_kl(base, min(pp1, base + KLC));
        // Stages: columns [u0, u1) of the plan words lie in `usize` ring slots
        // from `uat` on, block n of the chunk at n + vshift (modulo the ring);
        // the next stage is copied behind them where it fits.
        Plan nxt;
        unsigned word[NO];
        int cc = -64;          // first column of the chunk of nxt
        int nc0 = 64;          // next column of nxt to stage (64: the chunk is spent)
        int u0 = 0, u1 = 0, uat = 0, usize = 0;
        int v0 = 0, v1 = 0, vsize = 0, vshift = 0;
        // choose and copy the next stage; false when no column is left; v0 ==
        // v1 when none fits beside the stage in use
        auto stage_next = [&]() -> bool {
          for (;;) {
            if (nc0 >= 64) {
              if (cc + 64 >= nm) return false;
              cc += 64;
              if (cc % PLC == 0) plan_round(base, cc);
              take_chunk(base, cc / PLC * PLC, cc, nxt);
              nc0 = 0;
            }
            const int before = nc0 == 0 ? 0 : __builtin_amdgcn_readlane(nxt.send, nc0 - 1);
            if (__builtin_amdgcn_readlane(nxt.send, 63) == before) {  // nothing more is needed
              nc0 = 64;
              continue;
            }
            // send ascends: columns up to half the ring, so that the next stage
            // fits beside this one; a larger column alone where it fits
            const int room = nslot - usize;
            v0 = nc0;
            v1 = __popcll(__ballot(nxt.send <= before + min(room, nslot / 2)));
            if (v1 <= v0) v1 = v0 + (__builtin_amdgcn_readlane(nxt.send, v0) <= before + room ? 1 : 0);
            if (v1 == v0) return true;
            vsize = __builtin_amdgcn_readlane(nxt.send, v1 - 1) - before;
            nc0 = v1;
            if (vsize == 0) continue;  // columns without needed blocks
            int at = uat + usize;
            at = at >= nslot ? at - nslot : at;
            vshift = at - before;
            copy(nxt, v0, v1, vshift);
            return true;
          }
        };
        bool more = stage_next();
        while (more) {
          // stage v becomes the stage in use
#pragma unroll
          for (int o = 0; o < NO; ++o) word[o] = nxt.word[o];
          u0 = v0;
          u1 = v1;
          uat = uat + usize >= nslot ? uat + usize - nslot : uat + usize;
          usize = vsize;
          const int ushift = vshift;
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          if constexpr (SPLIT) split_own(nxt, u0, u1, ushift);
          __syncthreads();
          more = stage_next();
#pragma unroll
          for (int o = 0; o < NO; ++o) {
            unsigned long long todo = __ballot(lane >= u0 && lane < u1 && word[o] != 0u);
            while (todo) {
              const int l = __ffsll((long long)todo) - 1;
              todo &= todo - 1;
              const unsigned w = (unsigned)__builtin_amdgcn_readlane((int)word[o], l);
              const int first = (int)(w >> 18) + ushift;
              column(o, wrap((first + (int)((w >> 8) & 31u)) * sbytes),
                     wrap((first + (int)((w >> 13) & 31u)) * sbytes), w & 15u, (w >> 4) & 15u);
            }
          }
          if (more && v0 == v1) {  // a column too large to stand beside the last stage
            __syncthreads();
            usize = 0;
            more = stage_next();
          }
        }
        __syncthreads();
      }

      // ---- epilogue
      k = kargs();
      EpiCtx E{k->xv, (size_t)PER, k->h_rp, k->h_ci, k->h_v, {k->h1_rp[0], k->h1_rp[1], k->h1_rp[2]},
               {k->h1_ci[0], k->h1_ci[1], k->h1_ci[2]}, {k->h1_v[0], k->h1_v[1], k->h1_v[2]}, k->stage,
               k->kept_ij, k->stage_count, k->stage_cap, k->overflow, k->bad, k->rowcnt};
#pragma unroll
      for (int o = 0; o < NO; ++o) {
        if (!((own_mask >> o) & 1u)) continue;
        const int np = __builtin_amdgcn_readfirstlane(s_np[row_of(o) * PT + col_of(o)]);
        bool kept = false;
        if (np > 0) {
          const int I = __builtin_amdgcn_readlane(my_I, o), J = __builtin_amdgcn_readlane(my_J, o);
          const int eIJ = __builtin_amdgcn_readlane(my_e, o);
          double q[NQ];
#pragma unroll
          for (int k = 0; k < NQ; ++k) q[k] = 0.0;
          if constexpr (W)
            kept = epilogue<T, D, AccW>(E, wacc[o], I, J, eIJ, square, eps, np, sys, q);
          else
            kept = epilogue<T, D>(E, acc[o], I, J, eIJ, square, eps, np, sys, q);
          const int row = FINE ? row_of(o) * PT + col_of(o) : sum_row(s0 + row_of(o), t0 + col_of(o));
          if (lane == 0) {
#pragma unroll
            for (int k = 0; k < NQ; ++k) spart[row][k] = q[k];
          }
        }
        if constexpr (LEARN) {
          const int slot = __builtin_amdgcn_readlane(my_slot, o);
          if (slot >= 0 && lane == 0) k->log_y[slot] = kept ? 0.f : 1.f;  // label: dropped
        }
      }
    }  // parts
    __syncthreads();
    k = kargs();
    if constexpr (FINE) {  // k_sub_sums adds the rows of a sub-tile
      const int s0 = (part0 / (TQ / PT)) * PS, t0 = (part0 % (TQ / PT)) * PT;
      for (int i = t; i < SROWS * NQ; i += NT) {
        const int o = i / NQ;
        k->rows[((size_t)lb * NOUT + sum_row(s0 + o / PT, t0 + o % PT)) * NQ + i % NQ] = (&spart[0][0])[i];
      }
    } else if (t < NQ) {
      k->partial[(size_t)lb * NQ + t] = sub_sum(&spart[0][0] + t, NG, GO);
    }
    __syncthreads();  // spart is free for the next sub-tile
  }  // sub-tiles
  if ((threadIdx.x & 63) == 0 && nprod) atomicAdd(kargs()->exec_pairs, nprod);
}

template <typename T, int D, int SP, int TQ, bool BF, bool W, bool FK, int WS>
__global__ __launch_bounds__(waves(false, D) * 64, 4) void k_tile_numeric(TileArgs) {
  tile_numeric<T, D, SP, TQ, BF, W, FK, WS, false, false>();
}
template <typename T, int D, int SP, int TQ, bool BF, bool W, bool FK, int WS>
__global__ __launch_bounds__(waves(true, D) * 64, 4) void k_tile_fine(TileArgs) {
  tile_numeric<T, D, SP, TQ, BF, W, FK, WS, false, true>();
}
template <typename T, int D, int SP, int TQ, bool BF, bool W, bool FK, int WS>
__global__ __launch_bounds__(waves(false, D) * 64, 4) void k_tile_learn(TileArgs) {
  tile_numeric<T, D, SP, TQ, BF, W, FK, WS, true, false>();
}
template <typename T, int D, int SP, int TQ, bool BF, bool W, bool FK, int WS>
__global__ __launch_bounds__(waves(true, D) * 64, 4) void k_tile_learn_fine(TileArgs) {
  tile_numeric<T, D, SP, TQ, BF, W, FK, WS, true, true>();
}

// Trace sums of the sub-tiles from the rows of their outputs: 16 lanes per sub-tile.
template <int NOUT, int SUBS>
__global__ __launch_bounds__(256) void k_sub_sums(TileArgs a, int go) {
  static_assert(NQ <= 16, "a lane per sum");
  const int total = (a.n_tiles_dev ? *a.n_tiles_dev : a.n_tiles) * SUBS;
  const int q = threadIdx.x & 15, lb = blockIdx.x * 16 + (threadIdx.x >> 4);
  if (total > a.fine_subs || lb >= total || q >= NQ) return;
  double v[NOUT];  // all rows in flight at once
#pragma unroll
  for (int o = 0; o < NOUT; ++o) v[o] = a.rows[((size_t)lb * NOUT + o) * NQ + q];
  double sum = 0.0, part = 0.0;  // as sub_sum
#pragma unroll
  for (int o = 0; o < NOUT; ++o) {
    part += v[o];
    if ((o + 1) % go == 0) {
      sum += part;
      part = 0.0;
    }
  }
  a.partial[(size_t)lb * NQ + q] = sum;
}

// ================================================================== launch
// Blocks of a persistent launch: enough to fill every CU at the kernel's
// occupancy.
static unsigned resident_blocks(const void* kernel, int threads) {
  int dev = 0, n = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, 0) != hipSuccess || n < 1) {
    cus = 256;
    n = 1;
  }
  return (unsigned)(n * cus);
}

template <typename T, int D, int SP, int TQ, bool BF, bool W, bool FK, int WS>
static void tile_go_w(hipStream_t st, const TileArgs& a) {
  constexpr int SUBS = (CS / SP) * (CS / TQ), PARTS = SP * TQ / waves(true, D);
  const bool learn = a.skip == 2 || a.log_cap > 0;
  const unsigned subs = (unsigned)a.n_tiles * SUBS;
  auto go = [&](void (*kernel)(TileArgs), unsigned G, int threads) {
    if (a.work) {  // persistent: never more blocks than items or than fit at once
      const unsigned R = resident_blocks((const void*)kernel, threads);
      G = G < R ? G : R;
    }
    hipLaunchKernelGGL(kernel, dim3(G), dim3(threads), 0, st, a);
  };
  if (learn && !learn_parts(D, SP, TQ))
    return go(k_tile_learn<T, D, SP, TQ, BF, W, FK, WS>, subs, waves(false, D) * 64);
  auto whole = k_tile_numeric<T, D, SP, TQ, BF, W, FK, WS>;
  auto fine = k_tile_fine<T, D, SP, TQ, BF, W, FK, WS>;
  if constexpr (learn_parts(D, SP, TQ)) {
    if (learn) {
      whole = k_tile_learn<T, D, SP, TQ, BF, W, FK, WS>;
      fine = k_tile_learn_fine<T, D, SP, TQ, BF, W, FK, WS>;
    }
  }
  // a.n_tiles bounds the count on the device, where there is one
  if (subs > (unsigned)a.fine_subs) go(whole, subs, waves(false, D) * 64);
  if (a.fine_subs > 0 && (subs <= (unsigned)a.fine_subs || a.n_tiles_dev)) {
    const unsigned few = std::min(subs, (unsigned)a.fine_subs);
    go(fine, few * PARTS, waves(true, D) * 64);
    hipLaunchKernelGGL((k_sub_sums<SP * TQ, SUBS>), dim3((few + 15) / 16), dim3(256), 0, st, a,
                       a.column_sums ? SP : SP / WS);
  }
}

// Groups of the trace sums per sub-tile column (WS): four for the 4 x 4 sub-tile
// with two or three directions (FP64, and the kinds with FP64 sums: FP32
// products and the bfloat16 split), two for the 8 x 8 sub-tile with at most
// one direction (FP64, FP32 with FP64 sums), else one.
template <typename T, int D, int SP, int TQ, bool BF, bool W>
constexpr int groups() {
  return (D >= 2 && SP == 4 && TQ == 4 && (sizeof(T) == 8 || W))            ? 4
         : (D <= 1 && SP == 8 && TQ == 8 && (sizeof(T) == 8 || (W && !BF))) ? 2
                                                                            : 1;
}

template <typename T, int D, bool BF, bool W, int S>
static void tile_go(hipStream_t st, const TileArgs& a) {
  constexpr int SP = SHAPE_SP[S], TQ = SHAPE_TQ[S];
  // bfloat16 products take the whole padded K in one MFMA: no K-step loop
  if constexpr (!BF) {
    if (a.ksteps == 4) return tile_go_w<T, D, SP, TQ, BF, W, true, groups<T, D, SP, TQ, BF, W>()>(st, a);
  }
  tile_go_w<T, D, SP, TQ, BF, W, false, groups<T, D, SP, TQ, BF, W>()>(st, a);
}

// false when the shape does not exist for this kind
template <typename T, int D, bool BF, bool W>
static bool tile_shape_go(hipStream_t st, const TileArgs& a) {
  // the bfloat16 split with FP64 sums has the accumulators of the FP32 kind with FP64 sums
  constexpr int KIND = sizeof(T) == 8 ? K_FP64 : (W ? K_WIDE : (BF ? K_BF16 : K_FP32));
  switch (a.shape) {
    case TS_8x8:
      if constexpr (shape_ok(KIND, D, TS_8x8)) { tile_go<T, D, BF, W, TS_8x8>(st, a); return true; }
      break;
    case TS_4x8:
      if constexpr (shape_ok(KIND, D, TS_4x8)) { tile_go<T, D, BF, W, TS_4x8>(st, a); return true; }
      break;
    case TS_8x4:
      if constexpr (shape_ok(KIND, D, TS_8x4)) { tile_go<T, D, BF, W, TS_8x4>(st, a); return true; }
      break;
    case TS_4x4:
      if constexpr (shape_ok(KIND, D, TS_4x4)) { tile_go<T, D, BF, W, TS_4x4>(st, a); return true; }
      break;
    default: break;
  }
  return false;
}

template <typename T, int D>
bool tile_launch(hipStream_t st, const TileArgs& a) {
  if constexpr (sizeof(T) == 4) {
    if (a.bf16) return a.wide ? tile_shape_go<T, D, true, true>(st, a) : tile_shape_go<T, D, true, false>(st, a);
    if (a.wide) return tile_shape_go<T, D, false, true>(st, a);
  }
  return tile_shape_go<T, D, false, false>(st, a);
}

}  // namespace tc2
