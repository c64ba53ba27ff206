// Implicit Lanczos with full re-orthogonalization (Algorithm 2; operator of
// Eq. 4, A v = Phi (Phi^T v)) for windows of at most 256 blocks of at most 64 rows
// (res_shapes: 16384 rows, 10240 for m > 1024), held in the register files of the
// device, as one persistent kernel for the whole run.
//
// Block b of a window's nb holds rows [RB b, RB b + RB) of Phi in registers for
// the whole run, loaded once, and its rows of the basis Q in LDS.  Each step is
// the same computation as the pass and the reduction of the streaming path
// (k_lz_step, k_lz_reduce: q_j by the second Gram-Schmidt pass of step j-1 in
// row space, u = A q_j from the row dots with t and the Lanczos relation, z1 by
// the three-term recurrence, then t = Phi^T z1 and h2 = Q_j^T z1), in two phases:
//   rows     every block: its rows of q_j and z1, and its partials of Phi^T z1,
//            of h2 and of |z1|^2 (|t|^2 it sums from the t it holds);
//   columns  block b: t over the columns it owns (written to every copy of t);
//            h2 entries b, b + nb, ... (|z1|^2 among them).
// The scalars of a step (alpha, beta, the breakdown test) are computed by
// every block from the same reduced values in the same order, so all blocks
// agree and leave the loop together.  Results are bitwise reproducible.
//
// The blocks synchronise only through the data they exchange, with no
// barrier: every value passed between blocks is written with an agent-scope
// atomic store (coherent across the device's L2 caches) carrying its step in
// its two lowest mantissa bits (1 + (step & 1); a perturbation of at most
// 3 ulp, the same for every reader), and a reader polls each value it needs
// until the tag is that of the step it waits for.  The buffers are zeroed
// (tag 0, never valid) before the launch; every slot in use is rewritten at
// every step, and no block can rewrite a slot of step e + 1 before every
// reader has consumed step e's value (it first needs values that those
// readers produce after reading), so the two tags suffice.  Every wait is
// bounded: after LR_SPIN polls (or w.spin) a block sets an error word and leaves, and the
// others, seeing it, leave too.  A block's own stores are acknowledged
// before its waves start polling: its polls and its stores share the CU's path
// to memory, and its stores are what the other blocks are waiting for.  The
// host launches the kernel only when all blocks are resident at once (checked
// with the occupancy calculator).
#include "slh_device.h"
#include "slh_internal.h"

#include <algorithm>

namespace slh {

namespace {

constexpr int LR_SPIN = 1 << 20;   // polls before a barrier gives up

__device__ __forceinline__ void st_flag(unsigned* p, unsigned v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned ld_flag(unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// bar: [LR_ERR] error word
constexpr int LR_ERR = LZ_BAR_ERR;
// copies of t~ (T holds [ldq][m] doubles)
__host__ __device__ inline int res_copies(int ldq, int nb) {
  const int c = nb < 32 ? 1 : nb < 64 ? 2 : nb < 128 ? 4 : 8;
  return ldq < c ? ldq : c;
}

// v tagged with step e into *p
__device__ __forceinline__ void st_tag(double* p, double v, int e) {
  const long long x = (__double_as_longlong(v) & ~3LL) | (long long)(1 + (e & 1));
  __hip_atomic_store((long long*)p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// two tagged values into p[0..1] (16-byte aligned) with one coherent 16-byte
// store; each half carries its own tag, so the store need not be atomic as a whole
__device__ __forceinline__ void st_tag2(double* p, double v0, double v1, int e) {
  typedef long long ll2 __attribute__((ext_vector_type(2)));
  ll2 x;
  x.x = (__double_as_longlong(v0) & ~3LL) | (long long)(1 + (e & 1));
  x.y = (__double_as_longlong(v1) & ~3LL) | (long long)(1 + (e & 1));
  // s_nop: a VALU write to the data registers of a store wider than 8 bytes
  // must not follow it directly (the compiler adds this wait state only to
  // stores of its own)
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(p), "v"(x) : "memory");
}
__device__ __forceinline__ long long ld_raw(double* p) {
  return __hip_atomic_load((long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool tag_is(long long x, int e) { return (int)(x & 3) == 1 + (e & 1); }

// x[u] = *addr(u) of step e for the u with bit u of act set, polling until every
// tag matches (the addresses of the others must be readable too: the first
// loads carry no branches, so that they go out together); false after spin
// polls or when the error word is set (the error word is then set)
template <int N, class ADDR>
__device__ __forceinline__ bool ld_wait(ADDR addr, unsigned act, int e, unsigned* bar, int spin,
                                        double (&v)[N]) {
  long long x[N];
#pragma unroll
  for (int u = 0; u < N; ++u) x[u] = ld_raw(addr(u));
  bool ok = true;
  for (int s = 0;; ++s) {
    bool all = true;
#pragma unroll
    for (int u = 0; u < N; ++u) all = all && (((act >> u) & 1) == 0 || tag_is(x[u], e));
    if (all) break;
    if (s > spin || ((s & 63) == 63 && ld_flag(bar + LR_ERR) != 0)) {
      st_flag(bar + LR_ERR, 1u);
      ok = false;
      break;
    }
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (((act >> u) & 1) && !tag_is(x[u], e)) x[u] = ld_raw(addr(u));
  }
#pragma unroll
  for (int u = 0; u < N; ++u) v[u] = ((act >> u) & 1) ? __longlong_as_double(x[u]) : 0.0;
  return ok;
}

// v = p[0], p[1], q[0], q[1] of step e (16-byte aligned pairs), as ld_wait
__device__ __forceinline__ bool ld_wait_pairs(double* p, double* q, int e, unsigned* bar, int spin,
                                              double (&v)[4]) {
  typedef long long ll2 __attribute__((ext_vector_type(2)));
  ll2 x, y;
  bool ok = true;
  for (int s = 0;; ++s) {
    // loads and their wait in one statement: their registers are written when it ends
    asm volatile("global_load_dwordx4 %0, %2, off sc1\n\tglobal_load_dwordx4 %1, %3, off sc1\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(x), "=&v"(y)
                 : "v"(p), "v"(q)
                 : "memory");
    if (tag_is(x.x, e) && tag_is(x.y, e) && tag_is(y.x, e) && tag_is(y.y, e)) break;
    if (s > spin || ((s & 63) == 63 && ld_flag(bar + LR_ERR) != 0)) {
      st_flag(bar + LR_ERR, 1u);
      ok = false;
      break;
    }
  }
  v[0] = __longlong_as_double(x.x);
  v[1] = __longlong_as_double(x.y);
  v[2] = __longlong_as_double(y.x);
  v[3] = __longlong_as_double(y.y);
  return ok;
}

// Sum over the lanes at distances CB, 2 CB, ... 32 (CB a power of two >= 4; the
// same bits in every lane of the sum)
__device__ __forceinline__ double strided_sum(double v, int CB) {
  if (CB <= 32) v = swap32_add(v, v);
  if (CB <= 16) v = swap16_add(v, v);
  if (CB <= 8) v += dpp_f64<DPP_ROR8>(v);
  if (CB <= 4) v += dpp_f64<DPP_ROR4>(v);       // period 8 within the row by now: lane ^ 4
  return v;
}
// Sum over each group of LP consecutive lanes (LP a power of two <= 64)
__device__ __forceinline__ double group_sum(double v, int LP) {
  if (LP >= 64) v = swap32_add(v, v);
  if (LP >= 32) v = swap16_add(v, v);
  if (LP >= 16) v += dpp_f64<DPP_ROR8>(v);
  if (LP >= 8) v += dpp_f64<DPP_HALF_MIRROR>(v);
  if (LP >= 4) v += dpp_f64<DPP_XOR2>(v);
  if (LP >= 2) v += dpp_f64<DPP_XOR1>(v);
  return v;
}

// beta = sqrt(x) and 1 / beta for x > 0: the hardware reciprocal square root,
// two Newton steps, and a last correction of the root (a short chain of
// dependent operations, where sqrt and a division take several times as long)
__device__ __forceinline__ void sqrt_rsqrt(double x, double& r, double& ir) {
  // scaled into the range of the approximation (x = 2^-2k-exact power of two)
  const int ex = __builtin_amdgcn_frexp_exp(x) & ~1;
  const double xs = ldexp(x, -ex);
  double y = __builtin_amdgcn_rsq(xs);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double h = 0.5 * y;
    y = fma(h, fma(-xs * y, y, 1.0), y);
  }
  double s = xs * y;
  s = fma(fma(-s, s, xs), 0.5 * y, s);
  y = fma(fma(-s, y, 1.0), y, y);               // 1 / s from y close to it
  r = ldexp(s, ex >> 1);
  ir = ldexp(y, -(ex >> 1));
}

// Every store this thread issued acknowledged (vmcnt counts stores as well as
// loads here), then a block barrier: the block's polls that follow do not
// compete in the CU's memory path with its own stores, which other blocks are
// waiting for.
__device__ __forceinline__ void stores_done_barrier() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

// The held rows of Phi marked as rewritten (an empty statement, in place), so
// that their fp64 conversions are neither hoisted out of the step loop nor
// shared between a step's two uses (converted once they would need twice the
// registers).  In place: the registers must all be VGPRs, or each one held in
// an accumulation register is moved out and back.
template <int RW>
__device__ __forceinline__ void launder_rows(float4 (&ph)[RW]) {
#pragma unroll
  for (int r = 0; r < RW; ++r)
    asm volatile("" : "+v"(ph[r].x), "+v"(ph[r].y), "+v"(ph[r].z), "+v"(ph[r].w));
}

}  // namespace

// NS = m / 256 column slices and P row subsets: wave (sl, p) of the NW = NS P
// waves holds RW rows of the block's RB = P RW rows, 4 columns a lane, at most 128
// floats a lane.
// Workspace use per window: Spart [m / CB][nb][CB] (CB = 2^cbl: columns per
// owner, the smallest power of two >= 4 with CB nb >= m, so that blocks
// b < m / CB own the columns), H2part [nb][ldq + 1], H2 [ldq + 1], T [C][m] with
// C = res_copies (t written to every copy, block b reading copy b mod C, so that
// the blocks' polls of t spread over C times as many lines); outputs alpha,
// beta, neff, stop and Q[1..] as the streaming path.
// Dynamic LDS: the block's rows of Q, (n_it + 1) (RB + 1) doubles.
//
// t is Phi^T z1 unscaled (the streaming path's t~ times |z1|): in
//   u = (Phi t - Q g - beta h2_last q) / beta,  alpha = (|t|^2 - h2^T g) / beta^2 - 2 h2_last
// |z1| drops out, so that t leaves the block that owns its columns as soon as
// their sums are there, and |z1|^2, needed only by beta, travels with h2.
//
// What bounds it: the serial chain of a step, not Phi (held) or the exchanged
// bytes.  A step is two exchanges between blocks (a store and the poll that
// sees it, about 2000 cycles each) and six block barriers with the dots, sums
// and scalars between them.
// RL: that many more rows a block, in LDS (their float4s are read back once for
// the row dots and once for the column partials), for windows a little past what
// the registers hold.
template <int NS, int P, int RW, int RL, bool SPIN>
__global__ __launch_bounds__(64 * NS * P, 1) void k_lz_resident(LanczosWS w, unsigned* bar,
                                                                const double* __restrict__ q1,
                                                                int nb, int cbl) {
  constexpr int NW = NS * P, NT = 64 * NW, RB = P * RW + RL, QS = RB + 1;   // QS: row stride of Qs (bank spread)
  constexpr int CPT = P <= 4 ? 4 / P : 1;        // columns whose partials a thread stores
  // column partials a thread reads: CB nb is m rounded up to a power of two, or
  // 4 nb <= 4 * 256 at the smallest CB
  constexpr int M2 = NS <= 4 ? 1024 : 2048;
  constexpr int UL = (M2 + NT - 1) / NT;
  constexpr int RS = RB <= 8 ? 8 : RB <= 16 ? 16 : RB <= 32 ? 32 : 64;   // row slots of the row-space sums
  constexpr int KG = NT / RS;
  constexpr int RP = 64 / RS;                    // lanes of wave 0 per row
  constexpr int m = 256 * NS;
  static_assert(RW % 8 == 0 && RL % 8 == 0 && RB <= 64 && NT >= 256 && (RL == 0 || P == 1), "shape");
  const int CB = 1 << cbl;
  // window a, block b of its nb (consecutive blocks on one XCD where n_act is a
  // multiple of 8: the dispatch deals blocks to the XCDs in turn)
  const int a = blockIdx.x % w.n_act, b = blockIdx.x / w.n_act;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int sl = wv % NS, pw = wv / NS;
  const int L = w.L, n_it = w.n_it, ldq = w.ldq, hs = ldq + 1;
  // SPIN: the wait limit from w.spin (SLH_OPT_WAIT_POLLS), else the constant
  const int spin = SPIN ? (w.spin > 0 ? w.spin : LR_SPIN) : LR_SPIN;
  const int r0 = b * RB;
  // the lane's columns: c0, c0 + 1, c1, c1 + 1, so that a wave's 16-byte stores of
  // partials and loads of t cover whole lines (four columns in a row: half of each
  // 32 bytes per instruction; 8192 x 2048 10.6 -> 9.5 us a step)
  const int c0 = 256 * sl + 2 * lane, c1 = c0 + 128;
  extern __shared__ float4 res_dyn[];
  float4* const lrow = res_dyn;                  // [RL][m / 4]
  double* const Qs = (double*)(res_dyn + RL * (m / 4));   // [n_it + 1][QS]
  __shared__ double h2s[256], gs[256], als[256], bes[256];
  __shared__ double prw[NS][RS];
  __shared__ double zs[RS], zw[RS], ws[RS];
  __shared__ double rq[NW][RS + 1], rg[NW][RS + 1];
  __shared__ double red[3][NW], z2s;
  __shared__ double cpart[NT], hw[NW];
  __shared__ double cr[P > 1 ? P : 1][P > 1 ? m : 1];
  __shared__ int bad;
  const int ntc = res_copies(ldq, nb);
  double* Spart = w.Spart + (int64_t)a * nb * m;
  double* Hpart = w.H2part + (int64_t)a * nb * hs;
  double* H2 = w.H2 + (int64_t)a * hs;
  double* Tv = w.T + (int64_t)a * ldq * m;
  double* const Tr = Tv + (int64_t)(b % ntc) * m;   // the copy of t this block reads
  double* Qa = w.Q + (int64_t)a * ldq * L;
  double* alpha_o = w.alpha + (int64_t)a * n_it;
  double* beta_o = w.beta + (int64_t)a * n_it;
  const int lpl = 31 - __builtin_clz(nb);        // LP = nb = 2^lpl threads sum one entry of h2

  // the wave's rows of Phi (rows past L are zero), the block's rows of q_0 and
  // their weights
  float4 ph[RW];
  {
    const float* src = w.Phi + (int64_t)a * L * m + c0;
    auto load4 = [&](int row) {
      const float2 x = *(const float2*)(src + (int64_t)min(row, L - 1) * m);
      const float2 y = *(const float2*)(src + (int64_t)min(row, L - 1) * m + 128);
      return make_float4(x.x, x.y, y.x, y.y);
    };
#pragma unroll
    for (int r = 0; r < RW; ++r) ph[r] = load4(r0 + pw * RW + r);
    if (r0 + RB > L) {
#pragma unroll
      for (int r = 0; r < RW; ++r)
        if (r0 + pw * RW + r >= L) ph[r] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int r = 0; r < RL; ++r) {
      const float4 x = load4(r0 + RW + r);
      lrow[r * (m / 4) + tid] = r0 + RW + r < L ? x : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  if (tid == 0) bad = 0;
  if (RS != RB && tid < RS) zs[tid] = zw[tid] = ws[tid] = 0.0;   // (slots past the rows)
  if (tid < RB) {
    const double q = (r0 + tid < L) ? q1[a * w.ldr + r0 + tid] : 0.0;
    const double wr = (w.wt && r0 + tid < L) ? w.wt[a * w.ldr + r0 + tid] : 1.0;
    Qs[tid] = q;
    zs[tid] = q;
    zw[tid] = wr * q;
    ws[tid] = wr;
  }
  __syncthreads();

  // partials of Phi^T diag(weights) zs over the block's rows, tagged with step e
  auto col_partials = [&](int e) {
    double col[4] = {0.0, 0.0, 0.0, 0.0};
    launder_rows(ph);
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      const double z = zw[pw * RW + r];
      col[0] = fma((double)ph[r].x, z, col[0]);
      col[1] = fma((double)ph[r].y, z, col[1]);
      col[2] = fma((double)ph[r].z, z, col[2]);
      col[3] = fma((double)ph[r].w, z, col[3]);
    }
#pragma unroll
    for (int r = 0; r < RL; ++r) {
      const double z = zw[RW + r];
      const float4 x = lrow[r * (m / 4) + tid];
      col[0] = fma((double)x.x, z, col[0]);
      col[1] = fma((double)x.y, z, col[1]);
      col[2] = fma((double)x.z, z, col[2]);
      col[3] = fma((double)x.w, z, col[3]);
    }
    // column c of block b at ((c / CB) nb + b) CB + c % CB: the partials a block
    // reduces are contiguous
    if constexpr (P == 1) {
      st_tag2(Spart + ((((int64_t)(c0 >> cbl) * nb + b) << cbl) + (c0 & (CB - 1))), col[0], col[1], e);
      st_tag2(Spart + ((((int64_t)(c1 >> cbl) * nb + b) << cbl) + (c1 & (CB - 1))), col[2], col[3], e);
    } else {
      // the row subsets' sums meet in LDS, in order; thread = CPT columns
      cr[pw][c0] = col[0];
      cr[pw][c0 + 1] = col[1];
      cr[pw][c1] = col[2];
      cr[pw][c1 + 1] = col[3];
      __syncthreads();
      const int c = tid * CPT;
      if (P <= 4 || c < m) {
        double v[CPT];
#pragma unroll
        for (int q = 0; q < CPT; ++q) {
          v[q] = cr[0][c + q];
#pragma unroll
          for (int p = 1; p < P; ++p) v[q] += cr[p][c + q];
        }
        double* dst = Spart + ((((int64_t)(c >> cbl) * nb + b) << cbl) + (c & (CB - 1)));
        if constexpr (CPT == 2) st_tag2(dst, v[0], v[1], e);
        else st_tag(dst, v[0], e);
      }
    }
  };
  // The values of step e reduced across the blocks: t over the block's CB
  // columns into every copy (cols), and its entries k = b, b + nb, ... <= last
  // of h2 (k = last: |z1|^2, slot ldq; none for last < 0).  Thread = (column
  // tid % CB, partial lane tid / CB); for h2 (from the last thread down) LP
  // threads over the nb partials of an entry.  The loads of both go out
  // together, so that an entry of h2 costs no round trip of its own.
  auto reduce = [&](int e, bool cols, int last) -> bool {
    // an opaque copy of the thread's index: the addresses below are formed here
    // in every step instead of being held in registers across it
    unsigned td = threadIdx.x;
    asm volatile("" : "+v"(td));
    const unsigned ln = td & 63, wq = td >> 6, th = NT - 1 - td;
    const bool own = cols && (b << cbl) < m;
    const unsigned tot = own ? nb << cbl : 0, endc = (nb << cbl) - 1;
    const int LP = 1 << lpl;
    const unsigned pl = th & (LP - 1);
    double* const src = Spart + (own ? ((int64_t)b * nb) << cbl : 0);
    int k = (int)(th >> lpl) < NT >> lpl ? b + nb * (int)(th >> lpl) : last + 1;
    int slot = k >= last ? ldq : k;
    unsigned act = (k <= last && (int)pl < nb) ? 1u << UL : 0u;
#pragma unroll
    for (int u = 0; u < UL; ++u) act |= (td + u * NT < tot) ? 1u << u : 0u;
    stores_done_barrier();
    double v[UL + 1];
    bool ok = ld_wait<UL + 1>(
        [&](int u) {
          return u < UL ? src + min(td + u * NT, endc) : Hpart + (min(pl, nb - 1u) * (unsigned)hs + slot);
        },
        act, e, bar, spin, v);
    double sm = v[0];
#pragma unroll
    for (int u = 1; u < UL; ++u) sm += v[u];
    // a column's partial lanes within a wave lie CB lanes apart, then the waves'
    // sums (for CB >= 64, the column's lanes) in order
    sm = strided_sum(sm, CB);
    double hv = group_sum(v[UL], LP);
    if ((int)ln < CB) cpart[td] = sm;
    if (LP > 64 && ln == 0) hw[wq] = hv;
    if (!ok) bad = 1;
    __syncthreads();
    if (bad) return false;
    // thread (copy r, column cl) sums the column (the same sum in every copy)
    if (own) {
      const int SD = CB < 64 ? 64 : CB;
      for (int q = td; q < ntc << cbl; q += NT) {
        const int cl = q & (CB - 1), r = q >> cbl;
        double S = cpart[cl];
        for (int p = SD; p < NT; p += SD) S += cpart[p + cl];
        st_tag(Tv + (int64_t)r * m + (b << cbl) + cl, S, e);
      }
    }
    if (pl == 0 && k <= last) {
      for (int q = 1; q < LP >> 6; ++q) hv += hw[wq - q];
      st_tag(H2 + slot, hv, e);
    }
    // entries past the threads' (NT / nb of them were taken above): one per wave
    for (int q = (NT >> lpl) + (int)wq; b + nb * q <= last; q += NW) {
      k = b + nb * q;
      slot = k >= last ? ldq : k;
      hv = 0.0;
      for (unsigned p0 = 0; p0 < (unsigned)nb; p0 += 64) {
        double hx[1];
        if (!ld_wait<1>([&](int) { return Hpart + (min(p0 + ln, nb - 1u) * (unsigned)hs + slot); },
                        p0 + ln < (unsigned)nb ? 1u : 0u, e, bar, spin, hx))
          bad = 1;
        hv += hx[0];
      }
      hv = wave_sum_f64(hv);
      if (ln == 0) st_tag(H2 + slot, hv, e);
    }
    stores_done_barrier();
    return bad == 0;
  };

  double amax = 0.0;
  const int idx = ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1);
  // j = -1: t_0 = Phi^T q_0 only (step 0 of the tags)
  for (int j = -1; j < n_it; ++j) {
    if (j >= 0) {
    // ---- rows: the reduced values of the previous step (tags of step j),
    // those of this step tagged j + 1.  A wave takes its row dots as soon as its
    // own entries of t have arrived (the scalars of the step wait for values
    // of every block).
    double tv[4];
    bool ok = ld_wait_pairs(Tr + c0, Tr + c1, j, bar, spin, tv);
    // Phi t of the block's rows: 4 products per lane and row, summed over the
    // wave 8 rows at a time (into prw), then over the NS slices
    launder_rows(ph);
#pragma unroll
    for (int r8 = 0; r8 < RW; r8 += 8) {
      double d[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float4 y = ph[r8 + e];
        double x = (double)y.x * tv[0];
        x = fma((double)y.y, tv[1], x);
        x = fma((double)y.z, tv[2], x);
        d[e] = fma((double)y.w, tv[3], x);
      }
      const double tot = wave_sum8_f64(d);
      if ((lane & 7) == 0) prw[sl][pw * RW + r8 + idx] = tot;
    }
#pragma unroll
    for (int r8 = 0; r8 < RL; r8 += 8) {
      double d[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float4 y = lrow[(r8 + e) * (m / 4) + tid];
        double x = (double)y.x * tv[0];
        x = fma((double)y.y, tv[1], x);
        x = fma((double)y.z, tv[2], x);
        d[e] = fma((double)y.w, tv[3], x);
      }
      const double tot = wave_sum8_f64(d);
      if ((lane & 7) == 0) prw[sl][RW + r8 + idx] = tot;
    }
    // h2 (threads < j) with the neighbours that the wave's edge lanes need for
    // g, and |z1|^2 (thread j); T_{j-1}'s entries are read while they arrive
    const int tj = min(tid, max(j - 1, 0));
    const double alv = als[tj], bev = bes[tj], bep = bes[max(tj - 1, 0)];
    double h1[2];
    {
      const int nbr = lane == 0 ? tid - 1 : tid + 1;
      const unsigned act = (j > 0 && tid <= j ? 1u : 0u) |
                           (tid < j && (lane == 0 || lane == 63) && nbr >= 0 && nbr < j ? 2u : 0u);
      ok = ld_wait<2>([&](int u) { return H2 + (u == 0 ? (tid < j ? tid : ldq) : max(0, min(nbr, ldq))); },
                      act, j, bar, spin, h1) && ok;
    }
    const double h2v = tid < j ? h1[0] : 0.0;
    if (tid < j) h2s[tid] = h2v;
    if (tid == j) z2s = h1[0];
    if (!ok) bad = 1;
    // g = T_{j-1} h2 (alpha_k on the diagonal, beta_k beside it; beta_{j-1} is
    // not part of T_{j-1}); |h2|^2 and h2^T g; |t|^2 (each column once: the
    // first row subset's waves): every block holds all of t and sums it in the
    // same order, so every block gets the same value
    double hp = dpp_f64<DPP_WAVE_SHR1>(h2v), hn = dpp_f64<DPP_WAVE_SHL1>(h2v);
    if (lane == 0) hp = h1[1];
    if (lane == 63) hn = h1[1];
    double gi = alv * h2v;
    gi = fma(tid > 0 ? bep : 0.0, hp, gi);
    gi = fma(tid + 1 < j ? bev : 0.0, hn, gi);
    if (tid < j) gs[tid] = gi;
    else gi = 0.0;
    {
      double apv = 0.0;
#pragma unroll
      for (int u = 0; u < 4; ++u) apv = fma(tv[u], tv[u], apv);
      // (three sums in one stretch of code, so that their steps overlap)
      const double sa = wave_sum_f64(apv), sh = wave_sum_f64(h2v * h2v), sg = wave_sum_f64(h2v * gi);
      if (lane == 0) {
        red[0][wv] = sa;
        red[1][wv] = sh;
        red[2][wv] = sg;
      }
    }
    __syncthreads();
    if (bad) return;
    // Q_{j-1} h2 and Q_{j-1} g of each row: thread = (row i, k-group kg)
    {
      const int i = tid % RS, kg = tid / RS;
      double aq = 0.0, ag = 0.0;
#pragma unroll 4
      for (int k = (RS == RB || i < RB) ? kg : j; k < j; k += KG) {
        const double qk = Qs[k * QS + i];
        aq = fma(qk, h2s[k], aq);
        ag = fma(qk, gs[k], ag);
      }
      // the wave's k-groups of a row lie RS lanes apart
      if constexpr (RS <= 32) {
        aq = strided_sum(aq, RS);
        ag = strided_sum(ag, RS);
      }
      if (lane < RS) {
        rq[wv][i] = aq;
        rg[wv][i] = ag;
      }
    }
    double alpha = red[0][0];
#pragma unroll
    for (int q = 1; q < NS; ++q) alpha += red[0][q];
    double beta = 0.0, h2last = 0.0, ibeta = 0.0;
    if (j > 0) {
      double hh = red[1][0], hth = red[2][0];
      for (int q = 1; 64 * q < j; ++q) {
        hh += red[1][q];
        hth += red[2][q];
      }
      const double b2 = z2s - hh;
      if (b2 > 0.0) sqrt_rsqrt(b2, beta, ibeta);
      if (!(beta > w.tol * amax)) {             // breakdown: n_eff stays j
        if (b == 0 && tid == 0) {
          beta_o[j - 1] = beta;
          w.stop[a] = 1;
        }
        return;
      }
      h2last = h2s[j - 1];
      alpha = (alpha - hth) * (ibeta * ibeta) - 2.0 * h2last;
    }
    amax = fmax(amax, fabs(alpha));
    if (tid == 64) {
      als[j] = alpha;
      if (j > 0) bes[j - 1] = beta;
      if (b == 0) {
        if (j > 0) beta_o[j - 1] = beta;
        alpha_o[j] = alpha;
        w.neff[a] = j + 1;
      }
    }
    __syncthreads();
    // q_j and z1 of the block's rows: wave 0, RP lanes a row over the waves' sums
    if (tid < 64) {
      const int i = tid % RS, part = tid / RS, row = i < RB ? r0 + i : L;
      double sub = 0.0, sg = 0.0, u = 0.0;
#pragma unroll
      for (int q = 0; q < NW; q += RP) {
        if (NW % RP == 0 || q + part < NW) {
          sub += rq[q + part][i];
          sg += rg[q + part][i];
        }
      }
#pragma unroll
      for (int q = 0; q < NS; q += RP) {
        if (NS % RP == 0 || q + part < NS) u += prw[q + part][i];
      }
      if constexpr (RS <= 32) {
        sub = strided_sum(sub, RS);
        sg = strided_sum(sg, RS);
        u = strided_sum(u, RS);
      }
      const double wr = ws[i];
      u *= wr;
      double q = Qs[min(i, RB - 1)], qm = 0.0;    // j = 0: q_0
      if (j > 0) {
        q = (row < L) ? (zs[i] - sub) * ibeta : 0.0;
        qm = Qs[(j - 1) * QS + min(i, RB - 1)];
        if (part == 0 && (RS == RB || i < RB)) {
          Qs[j * QS + i] = q;
          if (row < L) Qa[(int64_t)j * L + row] = q;
        }
        u = ((u - sg) - beta * h2last * q) * ibeta;
      }
      double z = (u - alpha * q) - beta * qm;
      z = (row < L) ? z : 0.0;
      if (part == 0) {
        zs[i] = z;
        zw[i] = wr * z;
      }
    }
    __syncthreads();
    }
    // partials of Phi^T z1, then of h2 = Q_j^T z1 (k <= j): the h2 partials are
    // formed while the column partials travel
    col_partials(j + 1);
    // four threads per entry k (four lanes of a wave), RB / 4 rows each; the
    // entry after the last is |z1|^2
    for (int t = tid; t < 4 * (j + 2) && j >= 0; t += NT) {
      const int k = t >> 2, p4 = t & 3;
      const double* qk = (k <= j ? Qs + k * QS : zs) + p4 * (RB / 4);
      const double* zq = zs + p4 * (RB / 4);
      double a2[2] = {0.0, 0.0};
#pragma unroll
      for (int i = 0; i < RB / 4; ++i) a2[i & 1] = fma(qk[i], zq[i], a2[i & 1]);
      double v = a2[0] + a2[1];
      v += dpp_f64<DPP_XOR1>(v);
      v += dpp_f64<DPP_XOR2>(v);
      if (p4 == 0) st_tag(Hpart + (int64_t)b * hs + (k <= j ? k : ldq), v, j + 1);
    }
    // ---- t_{j+1}, h2 and |z1|^2 (entry j + 1)
    if (!reduce(j + 1, j + 1 < n_it, j < 0 ? -1 : j + 1)) return;
  }
  // beta of the last step (reported; T does not use it)
  if (b == 0) {
    double hv[1];
    const bool ok = ld_wait<1>([&](int) { return H2 + min(tid, ldq); }, tid < n_it ? 1u : 0u, n_it, bar,
                               spin, hv);
    const double sh = wave_sum_f64(hv[0] * hv[0]);
    if (lane == 0) red[0][wv] = sh;
    if (!ok) bad = 1;
    __syncthreads();
    if (bad) return;
    if (tid == 0) {
      double hh = red[0][0];
      for (int q = 1; q < NW; ++q) hh += red[0][q];
      if (!ld_wait<1>([&](int) { return H2 + ldq; }, 1u, n_it, bar, spin, hv)) return;
      const double b2 = hv[0] - hh;
      beta_o[n_it - 1] = b2 > 0.0 ? sqrt(b2) : 0.0;
    }
  }
}

// Everything the kernel expects before it starts, in one launch: q_0 into
// Q[a][0], alpha, beta, n_eff, the breakdown flag and max |alpha| cleared (the
// streaming path's k_lz_start), and the status word and every buffer of tagged
// values zeroed (tag 0: not yet written).
struct ResClear {
  double* p[5];
  int64_t n[5];   // doubles
};
__global__ void k_lz_res_prep(LanczosWS w, const double* __restrict__ q1, ResClear z) {
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t st = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = t0; i < (int64_t)w.n_act * w.L; i += st) {
    const int64_t a = i / w.L;
    w.Q[a * w.ldq * w.L + i - a * w.L] = q1[a * w.ldr + i - a * w.L];
  }
  for (int64_t i = t0; i < (int64_t)w.n_act * w.n_it; i += st) {
    w.alpha[i] = 0.0;
    w.beta[i] = 0.0;
  }
  for (int64_t a = t0; a < w.n_act; a += st) {
    w.stop[a] = 0;
    w.neff[a] = 0;
    w.amax[2 * a] = 0.0;
    w.amax[2 * a + 1] = 0.0;
  }
#pragma unroll
  for (int q = 0; q < 5; ++q)
    for (int64_t i = t0; i < z.n[q]; i += st) z.p[q][i] = 0.0;
}

namespace {
struct ResShape {
  int p, rw, rl, nb, cbl;   // row subsets, rows per wave, rows in LDS, blocks per window, log2 of the columns per owner
  int nw;               // windows of a launch
};
// Row subsets: those that fill 4 to 8 waves.  m = 1024 takes 8 waves rather than 4
// (us a step, 4 / 8 waves: 1367 rows 6.4 / 6.2, 4096 rows 7.2 / 7.1, a launch of
// 16 windows of 850 rows 10.6 / 8.7, where the blocks are half as many).
constexpr int res_subsets(int ns) { return ns == 1 ? 4 : ns <= 4 ? 2 : 1; }
// The resident kernel's shapes for w in order of preference; returns their number
// (0: it does not qualify).  nb = ceil(L / RB) rounded up to a power of two
// (blocks past the last row hold zeros), at least m / (the most columns a block
// can own), at most 256.
// Preferred: the fewest rows a block (less work per step in each) while the
// exchanged partials, nb m doubles a step and window, stay few: nb <= 128, or
// nb m <= 2^17.  Measured, us a step (rows a block): 5003 x 512 6.1 (32) 6.6
// (64); 1216 x 256 5.2 (32) 5.6 (64); 1367 x 1024 6.2 (16) 6.8 (32) 8.4 (64);
// 4096 x 1024 7.4 (16) 7.0 (32) 8.2 (64); 2788 x 2048 9.0 (16) 8.9 (32); 1367 x 2048 7.3
// (16) 8.1 (32); 3001 x 768 7.2 (16) 7.0 (32) 8.5 (64).
int res_shapes(const LanczosWS& w, int n_cu, ResShape (&out)[4]) {
  if (w.n_act < 1 || w.m % 256 != 0 || w.m < 256 || w.m > 2048 || w.n_it > 256 || w.n_it < 1) return 0;
  const int ns = w.m / 256, p = res_subsets(ns), nt = 64 * ns * p;
  const int cbmax = std::min(nt & -nt, 256);     // a power of two dividing the threads
  ResShape c[4];
  int n = 0, pref = -1;
  for (int q = 0; q < 4; ++q) {
    const int rw = q < 3 ? 8 << q : 32, rl = q < 3 ? 0 : 8, rb = p * rw + rl;
    if (rb > 64 || (rl && ns < 5)) continue;
    int64_t nb = 1;
    while (nb * rb < w.L || nb * cbmax < w.m) nb *= 2;
    if (rl && n > 0 && nb == c[n - 1].nb) continue;      // registers hold as many
    if (nb > 256) continue;
    int cbl = 2;
    while ((nb << cbl) < w.m) ++cbl;
    if (pref < 0 && nb * w.n_act <= n_cu && (nb <= 128 || nb * w.m <= 131072)) pref = n;
    c[n++] = ResShape{p, rw, rl, (int)nb, cbl, 0};
  }
  // the preferred one, then the others from the most rows a block down
  int k = 0;
  if (pref >= 0) out[k++] = c[pref];
  for (int q = n - 1; q >= 0; --q)
    if (q != pref) out[k++] = c[q];
  return k;
}
// per_cu != NULL: only the blocks that one compute unit holds
template <int NS, int P, int RW, int RL, bool SPIN>
hipError_t launch_res_t(const LanczosWS& w, const ResShape& sh, unsigned* bar, const double* q1,
                        int* per_cu, hipStream_t s) {
  auto k = k_lz_resident<NS, P, RW, RL, SPIN>;
  constexpr int NT = 64 * NS * P;
  const size_t lds = (size_t)(w.n_it + 1) * (P * RW + RL + 1) * sizeof(double) + (size_t)RL * 1024 * NS;
  if (lds > 65536) {
    const hipError_t e =
        hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  if (per_cu) return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, (const void*)k, NT, lds);
  hipLaunchKernelGGL(k, dim3(sh.nb * w.n_act), dim3(NT), lds, s, w, bar, q1, sh.nb, sh.cbl);
  return hipGetLastError();
}
template <int NS, bool SPIN>
hipError_t launch_res_n(const LanczosWS& w, const ResShape& sh, unsigned* bar, const double* q1,
                        int* per_cu, hipStream_t s) {
  constexpr int P = res_subsets(NS);
  if (sh.rw == 8) return launch_res_t<NS, P, 8, 0, SPIN>(w, sh, bar, q1, per_cu, s);
  if (sh.rw == 16) return launch_res_t<NS, P, 16, 0, SPIN>(w, sh, bar, q1, per_cu, s);
  if constexpr (NS >= 5)
    if (sh.rl == 8) return launch_res_t<NS, P, 32, 8, SPIN>(w, sh, bar, q1, per_cu, s);
  if constexpr (P <= 2) return launch_res_t<NS, P, 32, 0, SPIN>(w, sh, bar, q1, per_cu, s);
  return hipErrorInvalidValue;
}
template <bool SPIN>
hipError_t launch_res_s(const LanczosWS& w, const ResShape& sh, unsigned* bar, const double* q1,
                        int* per_cu, hipStream_t s) {
  switch (w.m / 256) {
    case 1: return launch_res_n<1, SPIN>(w, sh, bar, q1, per_cu, s);
    case 2: return launch_res_n<2, SPIN>(w, sh, bar, q1, per_cu, s);
    case 3: return launch_res_n<3, SPIN>(w, sh, bar, q1, per_cu, s);
    case 4: return launch_res_n<4, SPIN>(w, sh, bar, q1, per_cu, s);
    case 5: return launch_res_n<5, SPIN>(w, sh, bar, q1, per_cu, s);
    case 6: return launch_res_n<6, SPIN>(w, sh, bar, q1, per_cu, s);
    case 7: return launch_res_n<7, SPIN>(w, sh, bar, q1, per_cu, s);
    case 8: return launch_res_n<8, SPIN>(w, sh, bar, q1, per_cu, s);
  }
  return hipErrorInvalidValue;
}
// a wait limit other than the built-in one (SLH_OPT_WAIT_POLLS) takes an
// instantiation of its own, so that the limit stays a constant in the other
hipError_t launch_res(const LanczosWS& w, const ResShape& sh, unsigned* bar, const double* q1,
                      int* per_cu, hipStream_t s) {
  return w.spin > 0 ? launch_res_s<true>(w, sh, bar, q1, per_cu, s)
                    : launch_res_s<false>(w, sh, bar, q1, per_cu, s);
}
}  // namespace

namespace {
// The first shape whose blocks, of all windows, are resident at once (at most two
// per compute unit), else the one that takes the fewest launches of as many
// windows as are (p = 0: none).  A step of a launch that fills the chip takes
// up to 10 us, one of the streaming path 9 us + its read of Phi at 5.5 TB/s (32
// windows of 850 x 1024: two launches 15.8 us a step against 29).
ResShape res_shape(const LanczosWS& w, int n_cu) {
  ResShape sh[4], best{};
  const int n = res_shapes(w, n_cu, sh);
  int fewest = 0;
  (void)hipGetLastError();
  for (int q = 0; q < n; ++q) {
    int per_cu = 0;
    if (launch_res(w, sh[q], nullptr, nullptr, &per_cu, nullptr) != hipSuccess) continue;
    sh[q].nw = std::min(w.n_act, std::min(per_cu, 2) * n_cu / sh[q].nb);
    if (sh[q].nw == w.n_act) return sh[q];
    if (sh[q].nw < 1) continue;
    const int launches = (w.n_act + sh[q].nw - 1) / sh[q].nw;
    if (best.p == 0 || launches < fewest) {
      best = sh[q];
      fewest = launches;
    }
  }
  (void)hipGetLastError();
  const double phi = 4.0 * w.n_act * w.L * w.m;
  if (best.p && 10.0 * fewest >= 9.0 + phi / 5.5e6) best.p = best.nb = 0;
  if (best.p) best.nw = (w.n_act + fewest - 1) / fewest;   // launches of equal size
  return best;
}
}  // namespace

int lanczos_resident_blocks(const LanczosWS& w, int n_cu) { return res_shape(w, n_cu).nb; }

int lanczos_resident_most_blocks(const LanczosWS& w) {
  // the blocks of every shape grow with the rows; the fewest rows a block give the most
  const int ns = w.m / 256, rb = 8 * res_subsets(ns), nt = 64 * ns * res_subsets(ns);
  const int cbmax = std::min(nt & -nt, 256);
  int nb = 1;
  while (nb < 256 && (nb * rb < w.L || nb * cbmax < w.m)) nb *= 2;
  return nb;
}

size_t lanczos_resident_bar_words() {
  return (size_t)LR_ERR + 32;   // the error word on a line of its own
}

hipError_t launch_lanczos_resident(const LanczosWS& w, const double* q1_act, unsigned* bar,
                                   int n_cu, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  (void)hipGetLastError();
  const ResShape sh = res_shape(w, n_cu);
  if (sh.p == 0) return hipErrorInvalidValue;
  const int64_t hs = w.ldq + 1;
  hipError_t e = hipSuccess;
  for (int a0 = 0; a0 < w.n_act && e == hipSuccess; a0 += sh.nw) {
    // windows a0 .. a0 + na - 1 (Spart, H2part, H2 and T serve every launch)
    const int64_t na = std::min(sh.nw, w.n_act - a0);
    LanczosWS b = w;
    b.n_act = (int)na;
    b.Phi += (int64_t)a0 * w.L * w.m;
    if (b.wt) b.wt += a0 * w.ldr;
    b.Q += (int64_t)a0 * w.ldq * w.L;
    b.alpha += (int64_t)a0 * w.n_it;
    b.beta += (int64_t)a0 * w.n_it;
    b.neff += a0;
    b.stop += a0;
    b.amax += 2 * a0;
    const double* q1 = q1_act + a0 * w.ldr;
    ResClear z;
    double* const bufs[5] = {(double*)bar, b.Spart, b.H2part, b.T, b.H2};
    // the error word is cleared once a run.  T: the copies in use lie at the front
    // of each window's ldq m doubles.
    const int64_t lens[5] = {a0 ? 0 : (int64_t)lanczos_resident_bar_words() / 2, na * sh.nb * w.m,
                             na * sh.nb * hs,
                             ((na - 1) * w.ldq + res_copies(w.ldq, sh.nb)) * w.m, na * hs};
    for (int q = 0; q < 5; ++q) {
      z.p[q] = bufs[q];
      z.n[q] = lens[q];
    }
    hipLaunchKernelGGL(k_lz_res_prep, dim3(256), dim3(256), 0, s, b, q1, z);
    e = hipGetLastError();
    if (e == hipSuccess && e0 && a0 == 0) e = hipEventRecord(e0, s);
    if (e == hipSuccess) e = launch_res(b, sh, bar, q1, nullptr, s);
  }
  if (e == hipSuccess && e1) e = hipEventRecord(e1, s);
  return e;
}

}  // namespace slh
