// Distinct rows of a window.
//
// A raw prompt repeats its common tokens: 8192 Zipf(1.1) ids over a vocabulary
// of 152064 hold about 2800 different ones, 32768 ids about 8100, a window of
// 2048 that repeats a short template about 150.  Equal rows of X give equal rows
// of Phi, and the operator Phi Phi^T (Eq. 4) then acts on the sums over equal
// rows alone.  With G groups of c_g equal rows the vectors
//   e_g = (sum of the unit vectors of group g) / sqrt(c_g),   g < G,
//   x   = (the part of q_0 orthogonal to every e_g) / its norm
// are orthonormal, the Krylov space of q_0 lies in their span, and on it the
// operator is that of the G + 1 rows sqrt(c_g) phi_g and 0.  Lanczos (Algorithm
// 2) on those rows with the start vector's coordinates gives the same T, the same
// Ritz values, and coordinates from which every token's follow:
//   z_i = z'_g(i) / sqrt(c_g) + z'_x x_i.
// Nothing is approximated; only the order of the sums changes.  The feature map,
// every Lanczos step and the Ritz coordinates shrink by N / (G + 1).
//
//   k_grp_hash    a 64-bit hash per row from 256 bytes of it
//   k_grp_table   one workgroup per window: equal hashes grouped in an LDS table,
//                 groups numbered in the order of their first rows; the counts,
//                 the start vector's coordinates and the rows' own parts x_i
//   k_grp_verify  every row compared with its group's first row, all of it: a
//                 difference anywhere makes the host take the rows as they are
// so that the hash decides only what is compared, never what is equal.  Results
// do not depend on the order of the atomics (minima of row numbers, and sums of
// q_0 in fixed point).
#include "slh_device.h"
#include "slh_internal.h"

namespace slh {

// 16 lanes a row: 64 values from its start and 64 from its middle (two cache
// lines; embedding rows differ everywhere, and rows that agree there but not
// elsewhere are found by k_grp_verify).  2 MB of reads at N = 8192.
__global__ __launch_bounds__(256) void k_grp_hash(const uint16_t* __restrict__ X, int64_t ldx, int D,
                                                  const int* __restrict__ winlist, int L,
                                                  unsigned long long* __restrict__ hash) {
  const int a = blockIdx.y, l = threadIdx.x & 15;
  const int i = blockIdx.x * 16 + (threadIdx.x >> 4);
  const int64_t tok = (int64_t)(winlist ? winlist[a] : a) * L + min(i, L - 1);
  const int c = min((l < 8 ? 0 : ((D / 2) & ~7)) + 8 * (l & 7), D - 8);
  const uint4 v = *(const uint4*)(X + tok * ldx + c);
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  unsigned long long h = 0x9E3779B97F4A7C15ull * (unsigned)(l + 1);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    h = (h ^ w[q]) * 0xD6E8FEB86659FD93ull;
    h ^= h >> 32;
  }
  for (int o = 8; o >= 1; o >>= 1) h += __shfl_xor(h, o, 16);
  h *= 0xD6E8FEB86659FD93ull;
  h ^= h >> 29;
  if (l == 0 && i < L) hash[(int64_t)a * L + i] = h;
}

constexpr int GT = 1024;                 // threads of k_grp_table
constexpr int GSLOT = 16384;             // slots of its table
constexpr int GB = 8;                    // rows of a thread whose loads go out together
constexpr double GFIX = 9007199254740992.0;      // 2^53
constexpr double GFIX2 = 17592186044416.0;       // 2^44: at most 2^43 a row, 2^17 rows

// A table entry as it stands (other waves change it): no volatile, which would
// keep the access from being known as one to LDS.
template <class T>
__device__ __forceinline__ T ld_lds(T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Dynamic LDS: the table (tag and first row per slot, 128 KB) and the bit map of
// first rows, then in its place the groups' sums of q_0 and their counts (12
// bytes a group).  Bound by one CU's LDS atomics and barriers: 4096 rows 19 us,
// 8192 rows 26 us, 32768 rows 97 us (a third of it the probes), and where no two
// rows agree 9, 11 and 33 us (25, 42 and 228 with a limit on the probes of a row in
// place of the count); all windows of a batch run at once.  Summing a wave's most
// frequent groups in registers first did not make it faster (8192 rows: 30 us).
__global__ __launch_bounds__(GT) void k_grp_table(GroupWS w) {
  extern __shared__ unsigned char lds[];
  unsigned* tag = (unsigned*)lds;                      // [GSLOT]
  int* first = (int*)(lds + 4 * GSLOT);                // [GSLOT] first row, then the group's number
  unsigned* bits = (unsigned*)(lds + 8 * GSLOT);       // [ceil(L / 32)] first rows
  long long* qsum = (long long*)lds;                   // [GROUP_MAX]
  int* cnt = (int*)(lds + 8 * GROUP_MAX);              // [GROUP_MAX]
  __shared__ int wtot[GT / 64], made, ngrp;
  __shared__ double red[GT / 64];
  const int a = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int L = w.L, nword = (L + 31) / 32;
  int nslot = 1024;                                    // a power of two, 2 L or GSLOT
  while (nslot < 2 * L && nslot < GSLOT) nslot *= 2;
  const unsigned long long* hash = w.hash + (int64_t)a * L;
  int* gid = w.gid + (int64_t)a * L;
  for (int s = tid; s < nslot; s += GT) {
    tag[s] = 0;
    first[s] = 0x7FFFFFFF;
  }
  for (int s = tid; s < nword; s += GT) bits[s] = 0;
  if (tid == 0) made = 0;
  __syncthreads();
  // More groups than this are not taken: past the table, or so many that they spare
  // too little.  Every new slot is counted, so that whether the limit is passed does
  // not depend on the order of the probes (a limit on a row's probes would: one set
  // of 10000 groups in 40 and three of 12000 in four need more than 64 for some
  // row), and the rows that are left are not looked at.  A full table is past the
  // limit, so every probe ends.
  const int lim = min(GROUP_MAX, 7 * L / 8 - 1);
  int mk = 0;                                          // slots this thread made, not yet added
  auto add_made = [&]() {                              // at most GB a thread: 4 bits
    int n = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) n += __popcll(__ballot((mk >> q) & 1)) << q;
    if (n && lane == __ffsll((long long)__ballot(1)) - 1) atomicAdd(&made, n);
    mk = 0;
  };
  // a slot per hash (open addressing; tag 0 is free); its smallest row number
  for (int i0 = tid; i0 < L && ld_lds(&made) <= lim; i0 += GB * GT) {
    unsigned t[GB], o[GB];
    unsigned sl[GB];
    unsigned pend = 0;
#pragma unroll
    for (int u = 0; u < GB; ++u) {
      const unsigned long long h = hash[min(i0 + u * GT, L - 1)];
      t[u] = (unsigned)(h >> 32) | 1u;
      sl[u] = (unsigned)h & (nslot - 1);
      pend |= i0 + u * GT < L ? 1u << u : 0u;
    }
    // the rows' probes side by side: a round reads every row's slot at once.  The
    // count is looked at after 1, 2, 4, 8, 16, 32, 64, 96, ... rounds.
    for (int p = 1; pend != 0; ++p) {
#pragma unroll
      for (int u = 0; u < GB; ++u) o[u] = ld_lds(&tag[sl[u]]);
#pragma unroll
      for (int u = 0; u < GB; ++u) {
        if ((pend >> u) & 1) {
          if (o[u] == 0) {
            o[u] = atomicCAS(&tag[sl[u]], 0u, t[u]);
            mk += o[u] == 0;
          }
          if (o[u] == 0 || o[u] == t[u]) pend &= ~(1u << u);
          else sl[u] = (sl[u] + 1) & (nslot - 1);
        }
      }
      if ((p & (p - 1)) == 0 || (p & 31) == 0) {
        add_made();
        if (ld_lds(&made) > lim) break;
      }
    }
    add_made();
    if (pend != 0) break;
#pragma unroll
    for (int u = 0; u < GB; ++u) o[u] = (unsigned)ld_lds(&first[sl[u]]);
#pragma unroll
    for (int u = 0; u < GB; ++u) {
      const int i = i0 + u * GT;
      if (i < L) {
        if ((int)o[u] > i) atomicMin(&first[sl[u]], i);
        gid[i] = (int)sl[u];                           // read back by this thread alone
      }
    }
  }
  __syncthreads();
  if (made > lim) {
    if (tid == 0) w.n_dev[a] = w.n_out[a] = -1;
    return;
  }
  for (int s = tid; s < nslot; s += GT) {
    const int f = first[s];
    if (f != 0x7FFFFFFF) atomicOr(&bits[f >> 5], 1u << (f & 31));
  }
  __syncthreads();
  // groups numbered by first row: the bits before it.  A thread owns nper words.
  const int nper = (nword + GT - 1) / GT;
  int mine = 0;
  for (int q = 0; q < nper; ++q) {
    const int s = tid * nper + q;
    if (s < nword) mine += __popc(bits[s]);
  }
  int inc = mine;
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(inc, o);
    if (lane >= o) inc += u;
  }
  if (lane == 63) wtot[wv] = inc;
  __syncthreads();
  int base = 0;
  for (int q = 0; q < wv; ++q) base += wtot[q];
  const int excl = base + inc - mine;                  // groups before this thread's words
  if (tid == GT - 1) ngrp = base + inc;
  // the words' own bases, in the free tags (the numbering below reads them)
  __syncthreads();
  const int n = ngrp;                                  // <= lim
  unsigned* wbase = tag;                               // [nword <= GSLOT]
  {
    int run = excl;
    for (int q = 0; q < nper; ++q) {
      const int s = tid * nper + q;
      if (s < nword) {
        wbase[s] = (unsigned)run;
        run += __popc(bits[s]);
      }
    }
  }
  __syncthreads();
  const int64_t tok0 = (int64_t)(w.winlist ? w.winlist[a] : a) * L;
  int* rowsrc = w.rowsrc + (int64_t)a * L;
  for (int s = tid; s < nslot; s += GT) {
    const int f = first[s];
    if (f != 0x7FFFFFFF) {
      const int g = (int)wbase[f >> 5] + __popc(bits[f >> 5] & ((1u << (f & 31)) - 1u));
      first[s] = g;
      rowsrc[g] = (int)(tok0 + f);
    }
  }
  // the rows past the groups (the orthogonal part's and padding): no row of X
  for (int g = n + tid; g < L; g += GT) rowsrc[g] = ~(int)tok0;
  __syncthreads();
  // the rows' groups, kept in registers up to GB GT rows
  int gr[GB] = {};
  double qr[GB];
  const double* q0 = w.q1 + tok0;
  // f(row, group, q_0) for the rows of this thread
  auto rows = [&](auto f) {
    for (int i0 = tid; i0 < L; i0 += GB * GT) {
      if (L > GB * GT) {
#pragma unroll
        for (int u = 0; u < GB; ++u) {
          const int i = min(i0 + u * GT, L - 1);
          gr[u] = gid[i];
          qr[u] = q0[i];
        }
      }
#pragma unroll
      for (int u = 0; u < GB; ++u)
        if (i0 + u * GT < L) f(i0 + u * GT, gr[u], qr[u]);
    }
  };
  for (int i0 = tid; i0 < L; i0 += GB * GT) {
#pragma unroll
    for (int u = 0; u < GB; ++u) {
      const int i = min(i0 + u * GT, L - 1);
      gr[u] = gid[i];
      qr[u] = q0[i];
    }
#pragma unroll
    for (int u = 0; u < GB; ++u)
      if (i0 + u * GT < L) gid[i0 + u * GT] = gr[u] = first[gr[u]];
  }
  __syncthreads();
  for (int g = tid; g < n; g += GT) {
    qsum[g] = 0;
    cnt[g] = 0;
  }
  __syncthreads();
  // sums of q_0 (|q_0| = 1, so |sum| <= sqrt(L) < 2^9) over the groups in fixed
  // point, the part above 2^-53 and then the rest: the same bits in any order
  rows([&](int, int g, double v) {
    atomicAdd((unsigned long long*)&qsum[g], (unsigned long long)__double2ll_rn(v * GFIX));
    atomicAdd(&cnt[g], 1);
  });
  __syncthreads();
  double hi[(GROUP_MAX + GT - 1) / GT];
#pragma unroll
  for (int u = 0; u < (GROUP_MAX + GT - 1) / GT; ++u) {
    const int g = tid + GT * u;
    hi[u] = g < n ? (double)qsum[g] * (1.0 / GFIX) : 0.0;
    if (g < n) qsum[g] = 0;
  }
  __syncthreads();
  rows([&](int, int g, double v) {                     // the roundings of the first pass
    const double f = v * GFIX;
    atomicAdd((unsigned long long*)&qsum[g], (unsigned long long)__double2ll_rn((f - rint(f)) * GFIX2));
  });
  __syncthreads();
  double* wt = w.wt + (int64_t)a * L;
  double* isq = w.isq + (int64_t)a * L;
  double* q = w.q + (int64_t)a * L;
#pragma unroll
  for (int u = 0; u < (GROUP_MAX + GT - 1) / GT; ++u) {
    const int g = tid + GT * u;
    if (g < n) {
      const double s = fma((double)qsum[g], 1.0 / (GFIX * GFIX2), hi[u]);
      const double c = (double)cnt[g], sc = sqrt(c);
      wt[g] = sc;
      isq[g] = 1.0 / sc;
      q[g] = s / sc;
      ((double*)qsum)[g] = s / c;                      // the group's mean
    }
  }
  __syncthreads();
  // each row's part of q_0 orthogonal to the groups, and its norm
  double* xc = w.xc + (int64_t)a * L;
  double ss = 0.0;
  rows([&](int i, int g, double v) {
    const double d = v - ((double*)qsum)[g];
    xc[i] = d;
    ss = fma(d, d, ss);
  });
  ss = block_sum_f64(ss, red);
  const double nx = sqrt(ss);
  for (int g = n + tid; g < L; g += GT) {
    wt[g] = 0.0;
    isq[g] = g == n && nx > 0.0 ? 1.0 / nx : 0.0;      // x_i = xc_i / nx
    q[g] = g == n ? nx : 0.0;
  }
  if (tid == 0) {
    w.n_dev[a] = n;
    w.n_out[a] = n;
  }
}

// One wave per row that is not its group's first: all D values compared with the
// first row's.  Bound by one read of those rows (39 MB at 8192 x 3584; the first
// rows come from the caches).
__global__ __launch_bounds__(256) void k_grp_verify(GroupWS w, const uint16_t* __restrict__ X,
                                                    int64_t ldx, int D) {
  const int a = blockIdx.y, lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), L = w.L;
  if (i >= L) return;
  const int64_t tok = (int64_t)(w.winlist ? w.winlist[a] : a) * L + i;
  const int n = w.n_dev[a];
  if (n < 0) return;
  const int64_t src = w.rowsrc[(int64_t)a * L + w.gid[(int64_t)a * L + i]];
  if (src == tok) return;
  const uint16_t* x = X + tok * ldx;
  const uint16_t* y = X + src * ldx;
  unsigned diff = 0;
  for (int c0 = 0; c0 < D; c0 += 4 * 512) {
    uint4 u[4], v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = min(c0 + 512 * q + 8 * lane, D - 8);   // past the end: the last 8 again
      u[q] = *(const uint4*)(x + c);
      v[q] = *(const uint4*)(y + c);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      diff |= (u[q].x ^ v[q].x) | (u[q].y ^ v[q].y) | (u[q].z ^ v[q].z) | (u[q].w ^ v[q].w);
  }
  if (__any(diff != 0) && lane == 0) *w.differ = 1;
}

hipError_t launch_group(const GroupWS& w, const uint16_t* X, int64_t ldx, int D, hipStream_t s) {
  (void)hipGetLastError();
  if (w.L < 2 || w.L > GROUP_L_MAX || w.n_act < 1) return hipErrorInvalidValue;
  const size_t table = 8 * GSLOT + 4 * (size_t)((w.L + 31) / 32), sums = 12 * (size_t)GROUP_MAX;
  const size_t bytes = table > sums ? table : sums;
  hipError_t e = hipFuncSetAttribute((const void*)k_grp_table,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_grp_hash, dim3((w.L + 15) / 16, w.n_act), dim3(256), 0, s, X, ldx, D,
                     w.winlist, w.L, w.hash);
  hipLaunchKernelGGL(k_grp_table, dim3(w.n_act), dim3(GT), bytes, s, w);
  hipLaunchKernelGGL(k_grp_verify, dim3((w.L + 3) / 4, w.n_act), dim3(256), 0, s, w, X, ldx, D);
  return hipGetLastError();
}

// Results of the grouped rows for every token.  per = doubles a row; src rows of
// a window lie ld_src apart (doubles), element e of row g at g * rs + e * es.
//   out[a][i] (row i, per values) = isq_g src[g] + isq_x xc_i src[x], x = n[a]
__global__ __launch_bounds__(256) void k_grp_expand(GroupWS w, const double* __restrict__ src,
                                                    int64_t ld_src, int64_t rs, int64_t es, int per,
                                                    double* __restrict__ out, int64_t ld_out,
                                                    int64_t ors, int64_t oes) {
  const int a = blockIdx.y, L = w.L;
  const int64_t o = (int64_t)a * L;
  const int n = w.n_dev[a];
  const double ix = w.isq[o + n];
  const double* sa = src + a * ld_src;
  double* oa = out + a * ld_out;
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < (int64_t)L * per;
       t += (int64_t)gridDim.x * 256) {
    const int i = (int)(oes == 1 ? t / per : t % L), e = (int)(oes == 1 ? t % per : t / L);
    const int g = w.gid[o + i];
    oa[i * ors + e * oes] = fma(w.isq[o + g], sa[g * rs + e * es], (ix * w.xc[o + i]) * sa[n * rs + e * es]);
  }
}
// rows of Phi or entries of the row sums, copied to every token of their group:
// per 32-bit words a row
__global__ __launch_bounds__(256) void k_grp_copy(GroupWS w, const uint32_t* __restrict__ src,
                                                  int64_t ld_src, int per, uint32_t* __restrict__ out) {
  const int a = blockIdx.y, L = w.L;
  const int64_t o = (int64_t)a * L;
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < (int64_t)L * per;
       t += (int64_t)gridDim.x * 256) {
    const int64_t i = t / per, e = t % per;
    out[(o + i) * per + e] = src[a * ld_src + (int64_t)w.gid[o + i] * per + e];
  }
}
hipError_t launch_group_expand(const GroupWS& w, const double* src, int64_t ld_src, int64_t rs,
                               int64_t es, int per, double* out, int64_t ld_out, int64_t ors,
                               int64_t oes, hipStream_t s) {
  (void)hipGetLastError();
  const int64_t b = ((int64_t)w.L * per + 255) / 256;
  hipLaunchKernelGGL(k_grp_expand, dim3((unsigned)(b < 2048 ? b : 2048), w.n_act), dim3(256), 0, s, w,
                     src, ld_src, rs, es, per, out, ld_out, ors, oes);
  return hipGetLastError();
}
hipError_t launch_group_copy(const GroupWS& w, const void* src, int64_t ld_src, int per, void* out,
                             hipStream_t s) {
  (void)hipGetLastError();
  const int64_t b = ((int64_t)w.L * per + 255) / 256;
  hipLaunchKernelGGL(k_grp_copy, dim3((unsigned)(b < 2048 ? b : 2048), w.n_act), dim3(256), 0, s, w,
                     (const uint32_t*)src, ld_src, per, (uint32_t*)out);
  return hipGetLastError();
}

}  // namespace slh
