// Clustered-tile numeric kernel of the TC2 / TC2-CPSCF update for gfx950.
//
// Atoms are grouped into clusters of up to CS = 8 nearby atoms.  A work item
// is a tile of output blocks (I in cluster P) x (J in cluster Q) for P <= Q;
// it walks the common columns K of the two clusters' row panels once and, for
// every K, stages the present blocks X_JK of cluster Q in LDS while each wave
// holds the MFMA fragments of its X_IK in registers.  Every staged block then
// feeds up to 8 block products instead of one, which cuts the L2/HBM operand
// traffic of the row-by-row product (Algorithm 1) several-fold.  The
// accumulators and the fused epilogue (branch combine, Frobenius drop,
// traces and band energies) are the same as in the one-wave-per-block kernel.
#include "tc2_device.h"
#include "tc2_tile.h"

namespace tc2 {

// ------------------------------------------------------------------ cluster panels
// Panel of cluster P: sorted union of the columns of its atoms' rows, with the
// entry index of (I_s, K) for every member s (-1 when absent).  The union is
// an LDS bitmap over the system's atoms; pass 1 ranks each member entry in it
// (prefix popcounts), so no search is needed.
constexpr int PNT = 1024;  // threads of the panel and tile kernels

__device__ __forceinline__ int block_exclusive_scan(int v, int* ssc) {
  const int t = threadIdx.x;
  ssc[t] = v;
  __syncthreads();
  for (int o = 1; o < PNT; o <<= 1) {
    const int u = (t >= o) ? ssc[t - o] : 0;
    __syncthreads();
    ssc[t] += u;
    __syncthreads();
  }
  return ssc[t] - v;  // ssc[PNT-1] holds the total
}

__global__ __launch_bounds__(PNT) void k_panels(int pass, PanelArgs a) {
  extern __shared__ unsigned sbits[];  // nwords bits, then nwords prefix counts
  __shared__ int sscan[PNT];
  const int P = blockIdx.x;
  const int sys = a.clus_sys[P];
  const int t = threadIdx.x;
  if (!a.active[sys]) {
    if (pass == 0 && t == 0) a.panel_cnt[P] = 0;
    return;
  }
  const int lo = a.sys_start[sys], nbits = a.sys_end[sys] - lo;
  const int nwords = (nbits + 31) >> 5;
  unsigned* pre = sbits + nwords;
  for (int w = t; w < nwords; w += PNT) sbits[w] = 0u;
  __syncthreads();
  for (int s = 0; s < CS; ++s) {
    const int I = a.clus_atom[P * CS + s];
    if (I < 0) continue;
    for (int e = a.rp[I] + t; e < a.rp[I + 1]; e += PNT) {
      const int o = a.ci[e] - lo;
      atomicOr(&sbits[o >> 5], 1u << (o & 31));
    }
  }
  __syncthreads();
  const int per = (nwords + PNT - 1) / PNT;
  const int w0 = t * per, w1 = min(nwords, w0 + per);
  int cnt = 0;
  for (int w = w0; w < w1; ++w) cnt += __popc(sbits[w]);
  const int before = block_exclusive_scan(cnt, sscan);
  if (pass == 0) {
    if (t == PNT - 1) a.panel_cnt[P] = sscan[PNT - 1];
    return;
  }
  const int base = a.panel_rp[P];
  int run = before;
  for (int w = w0; w < w1; ++w) {
    pre[w] = run;
    unsigned x = sbits[w];
    while (x) {
      const int bit = __ffs(x) - 1;
      x &= x - 1;
      const int pos = base + run++;
      a.panel_k[pos] = lo + (w << 5) + bit;
#pragma unroll
      for (int s = 0; s < CS; ++s) a.panel_e[(size_t)pos * CS + s] = -1;
    }
  }
  __syncthreads();  // ranks in LDS and the -1 fill precede the entry writes
  for (int s = 0; s < CS; ++s) {
    const int I = a.clus_atom[P * CS + s];
    if (I < 0) continue;
    for (int e = a.rp[I] + t; e < a.rp[I + 1]; e += PNT) {
      const int o = a.ci[e] - lo, w = o >> 5;
      const int rank = (int)pre[w] + __popc(sbits[w] & ((1u << (o & 31)) - 1u));
      a.panel_e[(size_t)(base + rank) * CS + s] = e;
    }
  }
}

// Tiles of cluster P: the clusters Q >= P holding an atom J with a column K in
// common with some atom of P (cluster-level symbolic product).  Pass 0 builds
// the cluster bitmap, keeps it in tile_bits and bounds the number of output
// blocks of the tiles; pass 1 writes the tiles from the kept bitmap.
__global__ __launch_bounds__(PNT) void k_tiles(int pass, PanelArgs a) {
  extern __shared__ unsigned sbits[];
  __shared__ int sscan[PNT];
  __shared__ long long spairs[PNT];
  const int P = blockIdx.x;
  const int sys = a.clus_sys[P];
  const int t = threadIdx.x;
  if (!a.active[sys]) {
    if (pass == 0 && t == 0) {
      a.tile_cnt[P] = 0;
      a.tile_pairs[P] = 0;
    }
    return;
  }
  const int nbits = a.csys_end[sys] - P;
  const int nwords = (nbits + 31) >> 5;
  unsigned* gbits = a.tile_bits + (size_t)P * a.tile_words;
  if (pass == 0) {
    for (int w = t; w < nwords; w += PNT) sbits[w] = 0u;
    __syncthreads();
    const int wave = t >> 6, lane = t & 63, nw = PNT >> 6;
    for (int idx = a.panel_rp[P] + wave; idx < a.panel_rp[P + 1]; idx += nw) {
      const int K = a.panel_k[idx];
      for (int f = a.rp[K] + lane; f < a.rp[K + 1]; f += 64) {
        const int Q = a.atom_clus[a.ci[f]];
        if (Q >= P) {
          const int o = Q - P;
          atomicOr(&sbits[o >> 5], 1u << (o & 31));
        }
      }
    }
    __syncthreads();
    for (int w = t; w < nwords; w += PNT) gbits[w] = sbits[w];
  } else {
    for (int w = t; w < nwords; w += PNT) sbits[w] = gbits[w];
    __syncthreads();
  }
  const int per = (nwords + PNT - 1) / PNT;
  const int w0 = t * per, w1 = min(nwords, w0 + per);
  int cnt = 0;
  for (int w = w0; w < w1; ++w) cnt += __popc(sbits[w]);
  if (pass == 0) {
    int nP = 0;
    for (int s = 0; s < CS; ++s) nP += a.clus_atom[P * CS + s] >= 0;
    long long pairs = 0;
    for (int w = w0; w < w1; ++w) {
      unsigned x = sbits[w];
      while (x) {
        const int bit = __ffs(x) - 1;
        x &= x - 1;
        const int Q = P + (w << 5) + bit;
        int nQ = 0;
        for (int s = 0; s < CS; ++s) nQ += a.clus_atom[Q * CS + s] >= 0;
        pairs += (Q == P) ? (long long)nP * (nP + 1) / 2 : (long long)nP * nQ;
      }
    }
    sscan[t] = cnt;
    spairs[t] = pairs;
    __syncthreads();
    for (int o = PNT / 2; o > 0; o >>= 1) {
      if (t < o) {
        sscan[t] += sscan[t + o];
        spairs[t] += spairs[t + o];
      }
      __syncthreads();
    }
    if (t == 0) {
      a.tile_cnt[P] = sscan[0];
      a.tile_pairs[P] = spairs[0];
    }
    return;
  }
  int pos = a.tile_rp[P] + block_exclusive_scan(cnt, sscan);
  for (int w = w0; w < w1; ++w) {
    unsigned x = sbits[w];
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
    if (lane == 0) a.kept_ij[slot] = make_int2(I, J);
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
void launch_panels(hipStream_t st, int pass, const PanelArgs& a) {
  if (a.nc == 0) return;
  const size_t lds = (size_t)((a.max_sys_atoms + 31) / 32) * 8;  // bitmap + prefix counts
  hipLaunchKernelGGL(k_panels, dim3(a.nc), dim3(PNT), lds, st, pass, a);
}

void launch_tiles(hipStream_t st, int pass, const PanelArgs& a) {
  if (a.nc == 0) return;
  const size_t lds = (size_t)a.tile_words * 4;
  hipLaunchKernelGGL(k_tiles, dim3(a.nc), dim3(PNT), lds, st, pass, a);
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
