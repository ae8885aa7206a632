// Cluster panels and tiles of the TC2 / TC2-CPSCF update for gfx950, the
// copy-through of stopped systems, block norms, and the choice among the
// instances of the clustered-tile numeric kernel (tc2_tile_numeric.h).
//
// Atoms are grouped into clusters of up to CS = 8 nearby atoms.  A tile holds
// the output blocks (I in cluster P) x (J in cluster Q) for P <= Q; its
// products walk the common columns of the two clusters' row panels, so that an
// operand block staged in LDS feeds up to 8 block products instead of one,
// which cuts the L2/HBM operand traffic of the row-by-row product
// (Algorithm 1) several-fold.
#include "tc2_device.h"
#include "tc2_tile.h"

#include <algorithm>

namespace tc2 {

// ------------------------------------------------------------------ cluster panels
// The symbolic part of an update is three launches (k_panel_count, k_panels,
// k_tiles), each with a block per cluster: of the 230 us of an update of a small
// system (64-atom chain) 130 went to its 23 small kernels, at 4 us or more
// each, so counters are cleared and offsets found by the kernels that need
// them.  A block adds the counts of the clusters before its own itself (nc
// integers from L2) where a scan would be a launch between two others.
//
// Panel of cluster P: sorted union of the columns of its atoms' rows, with the
// entry index of (I_s, K) for every member s (-1 when absent).  The union is
// an LDS bitmap over the system's atoms; k_panels ranks each member entry in it
// (prefix popcounts), so no search is needed.
constexpr int PNT = 1024;         // threads of the panel and tile kernels
constexpr int PNW = PNT / 64;     // waves
static_assert(PNW % CS == 0, "waves split evenly over the members of a cluster");

// sum of v over the threads before this one; *total: over all (sh: PNW ints)
__device__ __forceinline__ int block_exclusive_scan(int v, int* sh, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(inc, o, 64);
    inc += lane >= o ? u : 0;
  }
  __syncthreads();  // readers of sh are done
  if (lane == 63) sh[wave] = inc;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < PNW; ++w) {
    const int x = sh[w];
    before += w < wave ? x : 0;
    all += x;
  }
  *total = all;
  return before + inc - v;
}

// sum of cnt[0 .. P)
__device__ __forceinline__ int sum_before(const int* cnt, int P, int* sh) {
  int v = 0, total = 0;
  for (int i = threadIdx.x; i < P; i += PNT) v += cnt[i];
  (void)block_exclusive_scan(v, sh, &total);
  return total;
}

// f(entry, member) for the entries of the rows of cluster P, members side by side
template <typename F>
__device__ __forceinline__ void each_entry(const PanelArgs& a, int P, F&& f) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, s = wave % CS;
  const int I = a.clus_atom[P * CS + s];
  if (I < 0) return;
  const int end = a.rp[I + 1];
  for (int e = a.rp[I] + (wave / CS) * 64 + lane; e < end; e += PNT / CS) f(e, s);
}

// the LDS bitmap of the union; its words [w0, w1) belong to this thread
__device__ __forceinline__ void panel_bits(const PanelArgs& a, int P, int lo, int nwords, unsigned* bits) {
  for (int w = threadIdx.x; w < nwords; w += PNT) bits[w] = 0u;
  __syncthreads();
  each_entry(a, P, [&](int e, int) {
    const int o = a.ci[e] - lo;
    atomicOr(&bits[o >> 5], 1u << (o & 31));
  });
  __syncthreads();
}

// Columns of every panel; clears the counters of the update.
__global__ __launch_bounds__(PNT) void k_panel_count(PanelArgs a, ClearArgs clear) {
  extern __shared__ unsigned sbits[];
  __shared__ int sh[PNW];
  const int P = blockIdx.x;
  const int sys = a.clus_sys[P];
  const int t = threadIdx.x;
#pragma unroll
  for (int k = 0; k < ClearArgs::N; ++k)
    for (long long i = (long long)P * PNT + t; i < clear.n[k]; i += (long long)gridDim.x * PNT)
      clear.p[k][i] = 0;
  if (!a.active[sys]) {
    if (t == 0) a.panel_cnt[P] = 0;
    return;
  }
  const int lo = a.sys_start[sys], nwords = (a.sys_end[sys] - lo + 31) >> 5;
  panel_bits(a, P, lo, nwords, sbits);
  int cnt = 0, total = 0;
  for (int w = t; w < nwords; w += PNT) cnt += __popc(sbits[w]);
  (void)block_exclusive_scan(cnt, sh, &total);
  if (t == 0) a.panel_cnt[P] = total;
}

// Panels, the triples of the full products (nominal, cleared before), and the
// clusters Q >= P holding an atom J with a column K in common with some atom of
// P (cluster-level symbolic product): their bitmap (tile_bits), count and a
// bound of the number of output blocks of their tiles.
__global__ __launch_bounds__(PNT) void k_panels(PanelArgs a) {
  extern __shared__ unsigned sbits[];  // nwords bits and nwords prefix counts, then the tiles' bits
  __shared__ int sh[PNW];
  __shared__ long long spairs[PNW];
  const int P = blockIdx.x;
  const int sys = a.clus_sys[P];
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const int base = sum_before(a.panel_cnt, P, sh);
  const int np = a.panel_cnt[P];
  if (t == 0) {
    a.panel_rp[P] = base;
    if (P == a.nc - 1) a.panel_rp[a.nc] = base + np;
  }
  if (!a.active[sys]) {
    if (t == 0) {
      a.tile_cnt[P] = 0;
      a.tile_pairs[P] = 0;
    }
    return;
  }
  const int lo = a.sys_start[sys], nwords = (a.sys_end[sys] - lo + 31) >> 5;
  unsigned* pre = sbits + nwords;
  panel_bits(a, P, lo, nwords, sbits);
  {
    const int per = (nwords + PNT - 1) / PNT;
    const int w0 = t * per, w1 = min(nwords, w0 + per);
    int cnt = 0, total = 0;
    for (int w = w0; w < w1; ++w) cnt += __popc(sbits[w]);
    int run = block_exclusive_scan(cnt, sh, &total);
    for (int w = w0; w < w1; ++w) {
      pre[w] = run;
      unsigned x = sbits[w];
      while (x) {
        const int bit = __ffs(x) - 1;
        x &= x - 1;
        const int pos = base + run++;
        a.panel_k[pos] = lo + (w << 5) + bit;
      }
    }
  }
  for (int i = t; i < np * CS; i += PNT) a.panel_e[(size_t)base * CS + i] = -1;
  if (wave == 0) {
    const int I = lane < CS ? a.clus_atom[P * CS + lane] : -1;
    const unsigned long long m = I >= 0 ? (unsigned long long)(a.rp[I + 1] - a.rp[I]) : 0ull;
    unsigned long long sum = m * m;
#pragma unroll
    for (int o = CS / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (lane == 0) atomicAdd(&a.nominal[sys], sum);
  }
  __syncthreads();  // ranks, columns and the -1 fill precede their readers
  each_entry(a, P, [&](int e, int s) {
    const int o = a.ci[e] - lo, w = o >> 5;
    const int rank = (int)pre[w] + __popc(sbits[w] & ((1u << (o & 31)) - 1u));
    a.panel_e[(size_t)(base + rank) * CS + s] = e;
  });
  __syncthreads();  // the ranks are no longer needed
  unsigned* tbits = sbits;
  const int twords = (a.csys_end[sys] - P + 31) >> 5;
  for (int w = t; w < twords; w += PNT) tbits[w] = 0u;
  __syncthreads();
  for (int idx = wave; idx < np; idx += PNW) {
    const int K = a.panel_k[base + idx];
    for (int f = a.rp[K] + lane; f < a.rp[K + 1]; f += 64) {
      const int Q = a.atom_clus[a.ci[f]];
      if (Q >= P) {
        const int o = Q - P;
        atomicOr(&tbits[o >> 5], 1u << (o & 31));
      }
    }
  }
  __syncthreads();
  int nP = 0;
  for (int s = 0; s < CS; ++s) nP += a.clus_atom[P * CS + s] >= 0;
  int cnt = 0, total = 0;
  long long pairs = 0;
  for (int w = t; w < twords; w += PNT) {
    unsigned x = tbits[w];
    a.tile_bits[(size_t)P * a.tile_words + w] = x;
    cnt += __popc(x);
    while (x) {
      const int bit = __ffs(x) - 1;
      x &= x - 1;
      const int Q = P + (w << 5) + bit;
      int nQ = 0;
      for (int s = 0; s < CS; ++s) nQ += a.clus_atom[Q * CS + s] >= 0;
      pairs += (Q == P) ? (long long)nP * (nP + 1) / 2 : (long long)nP * nQ;
    }
  }
  for (int o = 32; o > 0; o >>= 1) pairs += __shfl_xor(pairs, o, 64);
  if (lane == 0) spairs[wave] = pairs;
  (void)block_exclusive_scan(cnt, sh, &total);  // spairs is complete behind its barriers
  if (t == 0) {
    long long all = 0;
    for (int w = 0; w < PNW; ++w) all += spairs[w];
    a.tile_cnt[P] = total;
    a.tile_pairs[P] = all;
  }
}

// The tiles of cluster P from its bitmap, and (mult > 0) the range of work
// items, mult per tile, of every system.
__global__ __launch_bounds__(PNT) void k_tiles(PanelArgs a, int mult, int* sys_lo, int* sys_hi) {
  __shared__ int sh[PNW];
  const int P = blockIdx.x;
  const int sys = a.clus_sys[P];
  const int t = threadIdx.x;
  const int base = sum_before(a.tile_cnt, P, sh);
  if (t == 0) {
    const int end = base + a.tile_cnt[P];
    a.tile_rp[P] = base;
    if (P == a.nc - 1) a.tile_rp[a.nc] = end;
    if (mult > 0 && P == a.csys_start[sys]) sys_lo[sys] = mult * base;
    if (mult > 0 && P == a.csys_end[sys] - 1) sys_hi[sys] = mult * end;
  }
  if (!a.active[sys]) return;
  const int nwords = (a.csys_end[sys] - P + 31) >> 5;
  const unsigned* bits = a.tile_bits + (size_t)P * a.tile_words;
  const int per = (nwords + PNT - 1) / PNT;
  const int w0 = t * per, w1 = min(nwords, w0 + per);
  int cnt = 0, total = 0;
  for (int w = w0; w < w1; ++w) cnt += __popc(bits[w]);
  int pos = base + block_exclusive_scan(cnt, sh, &total);
  for (int w = w0; w < w1; ++w) {
    unsigned x = bits[w];
    while (x) {
      const int bit = __ffs(x) - 1;
      x &= x - 1;
      a.tile_p[pos] = P;
      a.tile_q[pos] = P + (w << 5) + bit;
      ++pos;
    }
  }
}

// ------------------------------------------------------------------ copy-through
// One wave per entry (I, J >= I) of a stopped system: its blocks go to the
// stage unchanged (row-major upper block).
template <typename T>
__global__ void k_copy_through(CopyArgs a) {
  const int lane = threadIdx.x & 63;
  const int nnz = a.rp[a.nb];
  const long long nwaves = ((long long)gridDim.x * blockDim.x) >> 6;
  for (long long w = ((long long)blockIdx.x * blockDim.x + threadIdx.x) >> 6; w < nnz;
       w += nwaves) {
    const int e = (int)w;
    int lo = 0, hi = a.nb;  // row of entry e
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (a.rp[mid] <= e) lo = mid; else hi = mid;
    }
    const int I = lo, J = a.ci[e];
    if (J < I || a.active[a.sys_of[I]]) continue;
    int slot = 0;
    if (lane == 0) slot = atomicAdd(a.stage_count, 1);
    slot = __builtin_amdgcn_readfirstlane(slot);
    if (slot >= a.stage_cap) {
      if (lane == 0) atomicOr(a.overflow, 1);
      continue;
    }
    const int per = (1 + a.D) * BS;
    const T* X = (const T*)a.xv + (size_t)e * per;
    T* st = (T*)a.stage + (size_t)slot * per;
    for (int q = lane; q < per; q += 64) {
      const int m = q / BS, qq = q - m * BS;  // stage index qq = r*16 + c
      const int r = qq >> 4, c = qq & 15;
      st[q] = X[m * BS + c * BP + r];
    }
    if (lane == 0) {
      a.kept_ij[slot] = make_int2(I, J);
      count_kept(a.rowcnt, I, J);
    }
  }
}

// ------------------------------------------------------------------ block norms
// Frobenius norm of every stored block of every matrix (float), one wave per
// entry; used by the screens.
template <typename T>
__global__ void k_block_norms(long long nnz, int D, const T* xv, float* bn, const int* nnz_dev) {
  const int lane = threadIdx.x & 63;
  if (nnz_dev) nnz = min(nnz, (long long)*nnz_dev);
  const long long nwaves = ((long long)gridDim.x * blockDim.x) >> 6;
  for (long long e = ((long long)blockIdx.x * blockDim.x + threadIdx.x) >> 6; e < nnz;
       e += nwaves) {
    for (int m = 0; m <= D; ++m) {
      const T* x = xv + ((size_t)e * (1 + D) + m) * BS;
      double ss = 0.0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double v = (double)x[lane + 64 * j];
        ss += v * v;
      }
      ss = wave_sum(ss);
      if (lane == 0) bn[(size_t)e * (1 + D) + m] = (float)sqrt(ss);
    }
  }
}

void launch_block_norms(hipStream_t st, int prec, long long nnz, int D, const void* xv, float* bn,
                        const int* nnz_dev) {
  if (nnz == 0) return;
  // one wave per entry, waves loop over entries beyond 2^24 blocks of 4 waves
  const long long want = (nnz + 3) / 4;
  const unsigned blocks = (unsigned)(want < (1 << 20) ? want : (1 << 20));
  if (prec == P_FP64)
    hipLaunchKernelGGL(k_block_norms<double>, dim3(blocks), dim3(256), 0, st, nnz, D,
                       (const double*)xv, bn, nnz_dev);
  else
    hipLaunchKernelGGL(k_block_norms<float>, dim3(blocks), dim3(256), 0, st, nnz, D,
                       (const float*)xv, bn, nnz_dev);
}

// ================================================================== launchers
void launch_panel_count(hipStream_t st, const PanelArgs& a, const ClearArgs& clear) {
  if (a.nc == 0) return;
  const size_t words = (size_t)((a.max_sys_atoms + 31) / 32);
  hipLaunchKernelGGL(k_panel_count, dim3(a.nc), dim3(PNT), words * 4, st, a, clear);
}

void launch_panels(hipStream_t st, const PanelArgs& a) {
  if (a.nc == 0) return;
  const size_t words = (size_t)((a.max_sys_atoms + 31) / 32);
  hipLaunchKernelGGL(k_panels, dim3(a.nc), dim3(PNT), std::max(2 * words, (size_t)a.tile_words) * 4, st,
                     a);
}

void launch_tiles(hipStream_t st, const PanelArgs& a, int mult, int* sys_lo, int* sys_hi) {
  if (a.nc == 0) return;
  hipLaunchKernelGGL(k_tiles, dim3(a.nc), dim3(PNT), 0, st, a, mult, sys_lo, sys_hi);
}

bool tile_shape_available(int kind, int D, int shape) {
  return kind >= 0 && kind < 4 && D >= 0 && D <= MAXD && shape >= 0 && shape < TS_N &&
         shape_ok(kind, D, shape);
}

int tile_shape_default(int kind, int D) {
  return ((kind == K_FP64 || kind == K_WIDE) && D >= 2) ? TS_4x4 : TS_8x8;
}

int tile_subs(int shape) { return (CS / SHAPE_SP[shape]) * (CS / SHAPE_TQ[shape]); }

const char* tile_shape_name(int shape) {
  static const char* names[TS_N] = {"8x8", "4x8", "8x4", "4x4"};
  return (shape >= 0 && shape < TS_N) ? names[shape] : "?";
}

extern template bool tile_launch<double, 0>(hipStream_t, const TileArgs&);
extern template bool tile_launch<double, 1>(hipStream_t, const TileArgs&);
extern template bool tile_launch<double, 2>(hipStream_t, const TileArgs&);
extern template bool tile_launch<double, 3>(hipStream_t, const TileArgs&);
extern template bool tile_launch<float, 0>(hipStream_t, const TileArgs&);
extern template bool tile_launch<float, 1>(hipStream_t, const TileArgs&);
extern template bool tile_launch<float, 2>(hipStream_t, const TileArgs&);
extern template bool tile_launch<float, 3>(hipStream_t, const TileArgs&);

template <typename T>
static bool tile_d(hipStream_t st, const TileArgs& a) {
  switch (a.D) {
    case 0: return tile_launch<T, 0>(st, a);
    case 1: return tile_launch<T, 1>(st, a);
    case 2: return tile_launch<T, 2>(st, a);
    default: return tile_launch<T, 3>(st, a);
  }
}

bool launch_tile_numeric(hipStream_t st, int prec, const TileArgs& a) {
  if (a.n_tiles == 0) return true;
  if (prec == P_FP64) return tile_d<double>(st, a);
  return tile_d<float>(st, a);
}

void launch_copy_through(hipStream_t st, int prec, const CopyArgs& a, int nnz) {
  if (nnz == 0) return;
  const long long want = ((long long)nnz + 3) / 4;
  const unsigned blocks = (unsigned)(want < (1 << 20) ? want : (1 << 20));
  if (prec == P_FP64) hipLaunchKernelGGL(k_copy_through<double>, dim3(blocks), dim3(256), 0, st, a);
  else hipLaunchKernelGGL(k_copy_through<float>, dim3(blocks), dim3(256), 0, st, a);
}

}  // namespace tc2
