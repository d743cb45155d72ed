// A whole inner flexible-PCG solve in one launch: the level-2 solve of Algorithm 2 on the
// formed H = C^T C + lam~ W, and SolveM2 of Algorithm 5 (two chained level-3 solves on the
// formed A~^T A~). The steps of such a solve are bound by latency: the s x s operands fit the
// register files of a few compute units and a step is two short products between dot
// products. As launches (k_l2x.hip, k_l2f.hip) a step costs 6 us (one kernel) or 10 to 36 us
// (two), most of it the launch, the fetch of the operands and the host's round trip per
// solve; here the operands are loaded once per solve into registers and stay there.
//
// Work split. A group of nblk blocks solves KC columns; block b keeps 8 RPW rows of both
// s x s operands in the registers of its eight wavefronts (lane l of the wavefront holds the
// columns l, l + 64, ...). Every block keeps all the vectors of its columns (a few elements
// per thread) and evaluates all dots and scalars itself, with the same code on the same data,
// so the blocks agree bit for bit and exchange nothing but the rows of the products. With
// s <= 128 one block holds both operands and a step has no exchange at all; larger s takes
// s / 32 blocks, with few columns s / 16 (after a sweep of a large matrix the operands come from
// HBM, 256 KB per block at s = 512 with s / 32), and s / 16 for s > 512.
//
// Exchange. The rows go through a buffer of 64-bit words, half of a double beside the 32-bit
// number of the exchange: a reader polls the words themselves until the number is right, so a
// step needs no fence, no flag and no barrier between blocks, and a device-scope fence (which
// writes back a whole L2 here) never happens. Words are written and read with relaxed
// agent-scope atomics (one 64-bit access each). Two buffers alternate: a block that writes
// exchange t + 2 has received exchange t + 1 from every block, and each of those had read all
// of exchange t by then. The numbers are never reused while a buffer holds older ones
// (pcg_solve clears it before they would wrap).
//
// The blocks of a launch have to run together: a launch has at most kPcgMaxBlocks blocks, one
// per compute unit, so four launches (the hardware queues a process has) fit the chip. When an
// exchange stays incomplete for kPcgWait ticks (other work holds the compute units;
// MSP_INNER_WAIT_MS in the environment sets another time, a negative one does not wait at all)
// the group's first block solves alone, from the start, with the operands from memory, and the
// others leave: every wait ends, and the launch always delivers. The rows, the dots and the
// scalars are formed by the same code in the same order either way, so the results are the
// same bits whether, and where, a wait ran out (the number of blocks and columns of a group
// does not enter them either). The next kPcgAlone launches do not try to meet: under lasting
// contention a solve pays one wait for so many launches.
//
// Alone a block reads both operands once per step; per step (whole solves): s = 256, one column:
// 18 us (4.5 as a group), 16 columns: 23 us (8.0); s = 512, one column: 60 us (4.8), 8 columns:
// 67 us (7.1); s = 1024, one column: 239 us (5.4).
//
// Measured per step, launch and operand loads included: s = 32, direct form, one block: 1.3 us
// (two kernels per step: 9.9 us); s = 384, recurrence, one column: 3.3 us (6.0 us); s = 512,
// 8 columns, direct, two columns per group: 5.6 us (four per group: 9.8 us; two kernels per
// step: 14.5 us); s = 256, 64 columns, direct, eight columns per group in one launch: 8.3 us
// (four per group in two launches: 13.4 us; the generic step: 42 us).
#include <cstdlib>

#include "msp_internal.h"
#include "wave_ops.h"

// every form of a solve (ONE, GROUP, ALONE) rounds alike: the compiler fuses nothing by itself
#pragma clang fp contract(off)

namespace {

using wave_ops::scatter_sums;
using wave_ops::wave_sum;

constexpr int WAVE = 64;
constexpr int NWV = 8;
constexpr int NT = NWV * WAVE;

__device__ __forceinline__ uint64_t ld_word(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_word(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int ld_mark(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// who solves: one block with both operands in its registers, a group of blocks with a share of
// the rows each, or one block that takes the rows from memory
enum Form { ONE, GROUP, ALONE };

// A block's view of one solve of KC columns: CPL 64-column chunks, RPW rows per wavefront.
template <int CPL, int RPW, int KC, Form FORM>
struct Block {
  static constexpr int SP = CPL * WAVE;              // padded length
  static constexpr int NV = KC * SP;                 // elements of a vector block
  static constexpr int EPT = (NV + NT - 1) / NT;     // per thread: e = tid + q NT
  static constexpr int RC = RPW * KC <= 16 ? RPW : (KC <= 2 ? 8 : 2);  // rows per reduction

  // LDS: xs the staged vector (zero beyond s), zr the product rows (one block), red the dot
  // partials by 64-element chunk, bc per-column scalars
  struct Shared {
    double xs[NV];
    double zr[FORM == GROUP ? 1 : 2 * NV];
    double red[3][2][KC * CPL];
    double bc[2][KC];
    int done[KC];
    int any;
    int stop;
  };

  // rows of M owned by this wavefront, in registers
  static __device__ __forceinline__ void load_rows(const double* __restrict__ M, int s, int row0,
                                                   double (&h)[RPW][CPL]) {
    const int lane = threadIdx.x % WAVE;
#pragma unroll
    for (int i = 0; i < RPW; ++i)
#pragma unroll
      for (int m = 0; m < CPL; ++m) {
        const int c = lane + WAVE * m, r = row0 + i;
        h[i][m] = (r < s && c < s) ? M[(int64_t)r * s + c] : 0.0;
      }
  }

  // out(jj, row) <- M xs_jj for the wavefront's rows: zr[d] in LDS or, in a group, exchange
  // words of number `ep` (ex: the buffer of this number, d the product's index)
  static __device__ __forceinline__ void product(const double (&h)[RPW][CPL], int d, int s, int row0, Shared& sh,
                                                 uint64_t* ex, uint32_t ep) {
    const int lane = threadIdx.x % WAVE;
    constexpr int NVAL = RC * KC;
    constexpr int SHF = wave_ops::log2i(WAVE / NVAL);
#pragma unroll
    for (int i0 = 0; i0 < RPW; i0 += RC) {
      double v[NVAL];
#pragma unroll
      for (int q = 0; q < NVAL; ++q) v[q] = 0.0;
#pragma unroll
      for (int m = 0; m < CPL; ++m)
#pragma unroll
        for (int jj = 0; jj < KC; ++jj) {
          const double x = sh.xs[jj * SP + lane + WAVE * m];
#pragma unroll
          for (int i = 0; i < RC; ++i) v[i * KC + jj] = fma(h[i0 + i][m], x, v[i * KC + jj]);
        }
      const double mine = scatter_sums<NVAL>(v);
      const int val = lane >> SHF;
      if ((lane & ((1 << SHF) - 1)) == 0) {
        const int row = row0 + i0 + val / KC, jj = val % KC;
        if (row < s) {
          if constexpr (FORM == GROUP) {
            uint64_t* w = ex + 2 * ((int64_t)(d * KC + jj) * SP + row);
            const uint64_t tag = (uint64_t)ep << 32;
            st_word(w, tag | (uint32_t)__double2loint(mine));
            st_word(w + 1, tag | (uint32_t)__double2hiint(mine));
          } else {
            sh.zr[(d * KC + jj) * SP + row] = mine;
          }
        }
      }
    }
  }

  // the same for all rows of M, from memory
  static __device__ __forceinline__ void product_all(const double* __restrict__ M, int d, int s, Shared& sh) {
    for (int row0 = threadIdx.x / WAVE * RPW; row0 < s; row0 += NWV * RPW) {
      double h[RPW][CPL];
      load_rows(M, s, row0, h);
      product(h, d, s, row0, sh, nullptr, 0);
    }
  }

  // ND product vectors of exchange `ep`, all rows; false when the wait ran out, or did for
  // another block of the launch
  template <int ND, class Args>
  static __device__ __forceinline__ bool receive(Args& a, Shared& sh, const uint64_t* ex, uint32_t ep,
                                                 double (&out)[ND][EPT]) {
    const int tid = threadIdx.x, s = a.s;
    if constexpr (FORM != GROUP) {
      __syncthreads();
#pragma unroll
      for (int d = 0; d < ND; ++d)
#pragma unroll
        for (int q = 0; q < EPT; ++q) {
          const int e = tid + q * NT;
          out[d][q] = (e < NV && e % SP < s) ? sh.zr[d * NV + e] : 0.0;
        }
      return true;
    } else {
      uint64_t w[ND][EPT][2];
      int64_t t0 = 0;
      if (a.wait < 0) return false;
      for (int spin = 0;; ++spin) {
        bool ok = true;
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
          for (int q = 0; q < EPT; ++q) {
            const int e = tid + q * NT;
            if (e < NV && e % SP < s) {
              const uint64_t* p = ex + 2 * ((int64_t)d * NV + e);
              w[d][q][0] = ld_word(p);
              w[d][q][1] = ld_word(p + 1);
            } else {
              w[d][q][0] = w[d][q][1] = (uint64_t)ep << 32;
            }
          }
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
          for (int q = 0; q < EPT; ++q)
            ok = ok && (uint32_t)(w[d][q][0] >> 32) == ep && (uint32_t)(w[d][q][1] >> 32) == ep;
        if (ok) break;
        if ((spin & 63) == 63) {  // the clock and the mark are read once in 64 polls
          const int64_t now = (int64_t)wall_clock64();
          if (t0 == 0) t0 = now;
          else if (now - t0 > a.wait || ld_mark(&a.ctl->alone) > a.serial) return false;
        }
      }
#pragma unroll
      for (int d = 0; d < ND; ++d)
#pragma unroll
        for (int q = 0; q < EPT; ++q) out[d][q] = __hiloint2double((int)(uint32_t)w[d][q][1], (int)(uint32_t)w[d][q][0]);
      return true;
    }
  }

  // the threads' contributions to ND dots, by chunk: sh.red[slot]; a barrier must follow
  // before totals()
  template <int ND>
  static __device__ __forceinline__ void partials(const double (&v)[ND][EPT], int slot, Shared& sh) {
    const int lane = threadIdx.x % WAVE, w = threadIdx.x / WAVE;
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
      const int chunk = w + q * NWV;
      if (chunk < KC * CPL) {
#pragma unroll
        for (int d = 0; d < ND; ++d) {
          const double t = wave_sum(v[d][q]);
          if (lane == 0) sh.red[slot][d][chunk] = t;
        }
      }
    }
  }
  static __device__ __forceinline__ double total(int slot, int d, int col, const Shared& sh) {
    double t = 0.0;
#pragma unroll
    for (int m = 0; m < CPL; ++m) t += sh.red[slot][d][col * CPL + m];
    return t;
  }
};

// MODE 0 (recurrence): z = Minv r and g = G r (G = H Minv) from one exchange, the operator's
// image of the direction by u_t = g_t + beta_t u_{t-1}. MODE 1 (direct): q = (H + sigma I) p
// and z = Minv r, an exchange each; nsol chained solves. False when a wait ran out.
template <int MODE, int CPL, int RPW, int KC, Form FORM, class Args>
__device__ __forceinline__ bool solve_block(Args& a, typename Block<CPL, RPW, KC, FORM>::Shared& sh) {
  using B = Block<CPL, RPW, KC, FORM>;
  constexpr bool MULTI = FORM == GROUP;
  constexpr int EPT = B::EPT, SP = B::SP, NV = B::NV;
  const int tid = threadIdx.x, s = a.s;
  const int grp = blockIdx.x / a.nblk, blk = blockIdx.x % a.nblk;
  const int k0 = a.col0 + grp * KC;
  const int row0 = (blk * NWV + tid / WAVE) * RPW;
  uint64_t* const exg = a.ex + (int64_t)grp * (MODE == 0 ? 2 : 1) * NV * 2;
  const int64_t exn = (int64_t)a.ex_stride;  // words of one of the two buffers
  uint32_t ep = a.ep0;
  // a thread's elements
  int ecol[EPT];
  int64_t eo[EPT];
  bool ein[EPT];
#pragma unroll
  for (int q = 0; q < EPT; ++q) {
    const int e = tid + q * NT;
    ecol[q] = min(e / SP, KC - 1);
    ein[q] = e < NV && e % SP < s && k0 + ecol[q] < a.k;
    eo[q] = (int64_t)(k0 + ecol[q]) * s + e % SP;
  }
  // per-column scalars: with one column every thread keeps them, with several thread jj does
  // and the values travel through LDS
  const bool owner = KC == 1 || tid < KC;
  const int oc = KC == 1 ? 0 : min(tid, KC - 1);
  if (tid == 0) sh.stop = 0;
  double hm[RPW][CPL], mm[RPW][CPL];  // (not used alone)
  double r[EPT], y[EPT], p[EPT], u[EPT];
  double v2[2][EPT], v1[1][EPT];
#pragma unroll
  for (int q = 0; q < EPT; ++q) y[q] = ein[q] ? a.rhs[eo[q]] : 0.0;
  for (int g = 1; g < a.nrhs; ++g)
#pragma unroll
    for (int q = 0; q < EPT; ++q)
      if (ein[q]) y[q] += a.rhs[(int64_t)g * a.k * s + eo[q]];
  if constexpr (FORM != ALONE) B::load_rows(a.H, s, row0, hm);  // behind the right-hand side: loads return in order

  auto stage = [&](const double(&x)[EPT]) {
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
      const int e = tid + q * NT;
      if (e < NV) sh.xs[e] = x[q];
    }
  };
  // several columns: the owners' scalar v of `slot` and their decision dj go through LDS
  // (one barrier); returns whether any column is active
  auto publish = [&](int slot, double v, int dj) -> bool {
    if constexpr (KC == 1) {
      return dj == 0;
    } else {
      if (tid < KC) {
        sh.done[tid] = dj;
        sh.bc[slot][tid] = v;
      }
      const uint64_t act = __ballot(tid < KC && dj == 0);
      if (tid == 0) sh.any = act != 0;
      __syncthreads();
      return sh.any != 0;
    }
  };
  auto col_done = [&](int q, int dj) -> bool { return KC == 1 ? dj != 0 : sh.done[ecol[q]] != 0; };
  auto scalar = [&](int slot, int q, double v) -> double { return KC == 1 ? v : sh.bc[slot][ecol[q]]; };

  bool failed = false;
  for (int sol = 0; sol < (MODE == 0 ? 1 : a.nsol) && !failed; ++sol) {
    if constexpr (FORM != ALONE) B::load_rows(a.Minv[sol], s, row0, mm);
    auto mul_h = [&](int d, uint64_t* ex) {
      if constexpr (FORM == ALONE) B::product_all(a.H, d, s, sh);
      else B::product(hm, d, s, row0, sh, ex, ep);
    };
    auto mul_m = [&](int d, uint64_t* ex) {
      if constexpr (FORM == ALONE) B::product_all(a.Minv[sol], d, s, sh);
      else B::product(mm, d, s, row0, sh, ex, ep);
    };
    const double sigma = a.sigma[sol];
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
      r[q] = y[q];  // the right-hand side (the previous solution when chained)
      y[q] = 0.0;
      p[q] = u[q] = 0.0;
      v1[0][q] = r[q] * r[q];
    }
    stage(r);
    B::template partials<1>(v1, 2, sh);
    __syncthreads();
    const double bn = sqrt(B::total(2, 0, oc, sh));
    double rz = 0.0, al = 0.0;
    int it = 0;
    const bool pd = k0 + oc >= a.k || (a.parent_done && a.parent_done[k0 + oc] != 0);
    int dj = (pd || bn == 0.0) ? 1 : 0;
    bool any = publish(0, 0.0, dj);
    // the decision on the residual whose partials are in slot 2. With several blocks it is
    // taken after the next product's rows are sent, in the shadow of their way: a product is
    // lost at the end of a solve, a square root and a barrier are won in every step
    bool brk = false;
    auto decide = [&]() {
      if (owner && dj == 0) {
        const double rn = sqrt(B::total(2, 0, oc, sh));
        ++it;
        if (brk || !(rn == rn)) dj = 2;
        else if (rn <= a.tol * bn) dj = 1;
        else if (it >= a.max_iter) dj = 3;
      }
      return publish(1, 0.0, dj);
    };
    if constexpr (MODE == 0) {
      bool first = true;
      while (any) {
        uint64_t* ex = exg + (ep & 1) * exn;
        mul_m(0, ex);
        mul_h(1, ex);
        if (MULTI && !first && !decide()) {
          ep += 2;  // nobody receives the rows just sent: the next exchange takes their buffer
          break;    // (a slow block may still read the other one)
        }
        if (!B::template receive<2>(a, sh, ex, ep, v2)) sh.stop = 1;
        ++ep;
        double zg[2][EPT];
#pragma unroll
        for (int q = 0; q < EPT; ++q) {
          zg[0][q] = v2[0][q];
          zg[1][q] = v2[1][q];
          v2[0][q] = zg[0][q] * r[q];
          v2[1][q] = zg[0][q] * u[q];
        }
        B::template partials<2>(v2, 0, sh);
        __syncthreads();
        if (MULTI && sh.stop) {
          failed = true;
          break;
        }
        double zr = 0.0, beta = 0.0;
        bool rzbad = false;
        if (owner && dj == 0) {
          zr = B::total(0, 0, oc, sh);
          const double zu = B::total(0, 1, oc, sh);
          // beta's denominator <r_{t-1}, z_{t-1}> zero or not finite: no conjugate direction
          // exists; the column stops as a breakdown below (alpha = 0 keeps its iterate)
          rzbad = !first && !(rz != 0.0 && isfinite(rz));
          beta = (first || rzbad) ? 0.0 : -al * zu / rz;
        }
        publish(0, beta, dj);
#pragma unroll
        for (int q = 0; q < EPT; ++q) {
          const double bq = scalar(0, q, beta);
          if (!col_done(q, dj)) {
            p[q] = fma(bq, p[q], zg[0][q]);
            u[q] = fma(bq, u[q], zg[1][q]);
          }
          v1[0][q] = p[q] * u[q];
        }
        B::template partials<1>(v1, 1, sh);
        __syncthreads();
        double alpha = 0.0;
        if (owner && dj == 0) {
          const double pq = B::total(1, 0, oc, sh);
          brk = rzbad || !(pq > 0.0);
          alpha = brk ? 0.0 : zr / pq;
          rz = zr;
          al = alpha;
        }
        publish(1, alpha, dj);
#pragma unroll
        for (int q = 0; q < EPT; ++q) {
          const double aq = scalar(1, q, alpha);
          if (!col_done(q, dj) && aq != 0.0) {  // 0: a breakdown keeps the iterate, p need not be finite
            r[q] = fma(-aq, u[q], r[q]);
            y[q] = fma(aq, p[q], y[q]);
          }
          v1[0][q] = r[q] * r[q];
        }
        stage(r);
        B::template partials<1>(v1, 2, sh);
        __syncthreads();
        first = false;
        if (!MULTI) any = decide();
      }
    } else {
      bool first = true;
      while (any) {
        // z = Minv r (r is staged), then beta and p
        {
          uint64_t* ex = exg + (ep & 1) * exn;
          mul_m(0, ex);
          if (MULTI && !first && !decide()) {
            ep += 2;
            break;
          }
          if (!B::template receive<1>(a, sh, ex, ep, v1)) sh.stop = 1;
          ++ep;
        }
        double z[EPT];
#pragma unroll
        for (int q = 0; q < EPT; ++q) {
          z[q] = v1[0][q];
          v2[0][q] = z[q] * r[q];
          v2[1][q] = z[q] * u[q];  // u holds the previous residual here
        }
        B::template partials<2>(v2, 0, sh);
        __syncthreads();
        if (MULTI && sh.stop) {
          failed = true;
          break;
        }
        double beta = 0.0;
        if (owner && dj == 0) {
          const double zr = B::total(0, 0, oc, sh), zro = B::total(0, 1, oc, sh);
          if (first) {
            rz = zr;
          } else if (rz != 0.0 && isfinite(rz)) {
            beta = (zr - zro) / rz;
            rz = zr;
          } else {
            // beta's denominator <r_{t-1}, z_{t-1}> zero or not finite: no conjugate
            // direction exists; the column stops as a breakdown and keeps its iterate
            dj = 2;
          }
        }
        if (!publish(0, beta, dj)) break;
#pragma unroll
        for (int q = 0; q < EPT; ++q)
          if (!col_done(q, dj)) p[q] = first ? z[q] : fma(scalar(0, q, beta), p[q], z[q]);
        first = false;
        stage(p);
        __syncthreads();
        // q = (H + sigma I) p
        {
          uint64_t* ex = exg + (ep & 1) * exn;
          mul_h(0, ex);
          if (!B::template receive<1>(a, sh, ex, ep, v1)) sh.stop = 1;
          ++ep;
        }
        double qv[EPT];
#pragma unroll
        for (int q = 0; q < EPT; ++q) {
          qv[q] = fma(sigma, p[q], v1[0][q]);
          v1[0][q] = p[q] * qv[q];
        }
        B::template partials<1>(v1, 1, sh);
        __syncthreads();
        if (MULTI && sh.stop) {
          failed = true;
          break;
        }
        double alpha = 0.0;
        if (owner && dj == 0) {
          const double pq = B::total(1, 0, oc, sh);
          brk = !(pq > 0.0);
          alpha = brk ? 0.0 : rz / pq;
        }
        publish(1, alpha, dj);
#pragma unroll
        for (int q = 0; q < EPT; ++q) {
          u[q] = r[q];
          const double aq = scalar(1, q, alpha);
          if (!col_done(q, dj) && aq != 0.0) {  // 0: as above
            y[q] = fma(aq, p[q], y[q]);
            r[q] = fma(-aq, qv[q], r[q]);
          }
          v1[0][q] = r[q] * r[q];
        }
        stage(r);
        B::template partials<1>(v1, 2, sh);
        __syncthreads();
        if (!MULTI) any = decide();
      }
    }
    // the most iterations of any column of the launch
    if (blk == 0 && owner && (KC > 1 || tid == 0)) atomicMax(&a.ctl->it[a.parity][sol], it);
    __syncthreads();  // the next solve reuses the LDS buffers
  }
  if (failed) return false;
  if (blk == 0) {
#pragma unroll
    for (int q = 0; q < EPT; ++q)
      if (ein[q]) a.out[eo[q]] = y[q];
  }
  return true;
}

template <int MODE, int CPL, int RPW, int KC, bool MULTI>
__global__ void __launch_bounds__(NT) k_pcg(PcgArgs a) {
  constexpr Form FORM = MULTI ? GROUP : ONE;
  __shared__ union {
    typename Block<CPL, RPW, KC, FORM>::Shared sh;
    typename Block<CPL, RPW, KC, MULTI ? ALONE : ONE>::Shared alone;
  } lds;
  auto& sh = lds.sh;
  const int tid = threadIdx.x;
  // the iteration counts of the launch before this one join the total
  if (blockIdx.x == 0 && tid == 0) {
    int64_t add = 0;
    for (int q = 0; q < 2; ++q) add += a.ctl->it[a.parity ^ 1][q];
    a.ctl->total += add;
    a.ctl->it[a.parity ^ 1][0] = a.ctl->it[a.parity ^ 1][1] = 0;
  }
  if constexpr (MULTI) {
    if (tid == 0) sh.any = ld_mark(&a.ctl->alone) > a.serial;
    __syncthreads();
    bool alone = sh.any != 0;  // uniform in the block
    __syncthreads();
    if (!alone && !solve_block<MODE, CPL, RPW, KC, FORM>(a, sh)) {
      if (tid == 0)
        __hip_atomic_store(&a.ctl->alone, a.serial + kPcgAlone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      alone = true;
    }
    if (alone && blockIdx.x % a.nblk == 0) {
      if (tid == 0) atomicAdd(&a.ctl->nalone, 1);
      // the arguments anew from the kernel's segment: kept in registers over the group's solve
      // they cost it spills (0.9% of whole solves at n = 10007, s = 320, 16 columns, 265 ms)
      auto seg = (const __attribute__((address_space(4))) PcgArgs*)__builtin_amdgcn_kernarg_segment_ptr();
      asm volatile("" : "+s"(seg));
      __syncthreads();  // the group's LDS is read no more
      solve_block<MODE, CPL, RPW, KC, ALONE>(*seg, lds.alone);
    }
  } else {
    solve_block<MODE, CPL, RPW, KC, FORM>(a, sh);
  }
}

template <int MODE, int CPL, int RPW, int KC, bool MULTI>
hipError_t go(hipStream_t st, const PcgArgs& a, int groups) {
  hipLaunchKernelGGL((k_pcg<MODE, CPL, RPW, KC, MULTI>), dim3((unsigned)(groups * a.nblk)), dim3(NT), 0, st, a);
  return hipGetLastError();
}

template <int MODE>
hipError_t dispatch(hipStream_t st, const PcgArgs& a, const PcgShape& h, int groups) {
  switch (h.cpl * 100 + h.kc) {
    case 101: return go<MODE, 1, 8, 1, false>(st, a, groups);
    case 201: return go<MODE, 2, 16, 1, false>(st, a, groups);
    case 401: return h.rpw == 2 ? go<MODE, 4, 2, 1, true>(st, a, groups) : go<MODE, 4, 4, 1, true>(st, a, groups);
    case 402: return go<MODE, 4, 4, 2, true>(st, a, groups);
    case 404: return go<MODE, 4, 4, 4, true>(st, a, groups);
    case 408: return go<MODE, 4, 4, 8, true>(st, a, groups);
    case 801: return h.rpw == 2 ? go<MODE, 8, 2, 1, true>(st, a, groups) : go<MODE, 8, 4, 1, true>(st, a, groups);
    case 802: return go<MODE, 8, 4, 2, true>(st, a, groups);
    case 804: return go<MODE, 8, 4, 4, true>(st, a, groups);
    case 1601: return go<MODE, 16, 2, 1, true>(st, a, groups);
    case 1602: return go<MODE, 16, 2, 2, true>(st, a, groups);
  }
  return hipErrorInvalidValue;
}

}  // namespace

PcgShape pcg_shape(int64_t s, int64_t k) {
  PcgShape h{};
  if (s < 1 || s > kPcgMaxS || k < 1) return h;
  const int chunks = (int)((s + WAVE - 1) / WAVE);
  h.cpl = chunks <= 1 ? 1 : chunks <= 2 ? 2 : chunks <= 4 ? 4 : chunks <= 8 ? 8 : 16;
  const int rpw = h.cpl == 1 ? 8 : h.cpl == 2 ? 16 : h.cpl == 16 ? 2 : 4;
  h.nblk = (int)((s + NWV * rpw - 1) / (NWV * rpw));
  h.rpw = rpw;
  if (rpw == 4) {  // few columns: twice the blocks, each fetching half as much of the operands
    const int nb2 = (int)((s + NWV * 2 - 1) / (NWV * 2));
    if (k * nb2 <= kPcgMaxBlocks) {
      h.rpw = 2;
      h.nblk = nb2;
    }
  }
  // the fewest columns per group (1, 2, 4, 8) with which the groups fit one launch; at most
  // what the registers hold beside the operands (8 for s <= 256, 4 for s <= 512, else 2)
  const int most = h.cpl <= 2 ? 1 : (h.cpl == 4 ? 8 : (h.cpl == 8 ? 4 : 2));
  h.kc = 1;
  while (h.kc < most && (k + h.kc - 1) / h.kc * h.nblk > kPcgMaxBlocks) h.kc *= 2;
  const int per = kPcgMaxBlocks / h.nblk > 0 ? kPcgMaxBlocks / h.nblk : 1;  // groups per launch
  h.groups = (int)((k + h.kc - 1) / h.kc);
  h.launches = (h.groups + per - 1) / per;
  h.per = per < h.groups ? per : h.groups;
  return h;
}

size_t pcg_words(int64_t s, int64_t k) {
  const PcgShape h = pcg_shape(s, k);
  // two buffers, up to two product vectors per column, two words per element
  return h.nblk > 1 ? (size_t)2 * h.per * 2 * h.kc * h.cpl * WAVE * 2 : 2;
}

PcgRun pcg_carve(WsCarver& w, int64_t s, int64_t k) {
  PcgRun R{};
  R.shape = pcg_shape(s, k);
  R.s = (int)s;
  R.k = (int)k;
  R.words = pcg_words(s, k);
  R.ex = w.take<uint64_t>(R.words);
  R.ctl = w.take<PcgCtl>(1);
  return R;
}

hipError_t pcg_reset(hipStream_t st, PcgRun& R) {
  R.next = 1;
  R.parity = 0;
  R.serial = 0;
  R.wait = kPcgWait;
  if (const char* ms = getenv("MSP_INNER_WAIT_MS")) R.wait = (int64_t)(atof(ms) * 1e5);
  hipError_t e = hipMemsetAsync(R.ctl, 0, sizeof(PcgCtl), st);
  if (e == hipSuccess) e = hipMemsetAsync(R.ex, 0, R.words * sizeof(uint64_t), st);
  return e;
}

hipError_t pcg_solve(hipStream_t st, PcgRun& R, PcgArgs a, int mode) {
  const PcgShape& h = R.shape;
  if (h.cpl == 0 || a.max_iter < 1 || a.max_iter > kPcgMaxIter) return hipErrorInvalidValue;
  // exchange numbers of one launch: two per step, the first and the unreceived last product
  const uint64_t span = (uint64_t)a.nsol * (2 * (uint64_t)a.max_iter + 4);
  if (a.nrhs < 1) a.nrhs = 1;
  a.s = R.s;
  a.k = R.k;
  a.nblk = h.nblk;
  a.ex = R.ex;
  a.ex_stride = (int64_t)(R.words / 2);
  a.ctl = R.ctl;
  a.wait = R.wait;
  for (int g0 = 0; g0 < h.groups; g0 += h.per) {
    if (R.next + span > 0xFFFFFFFFull) {  // before the numbers wrap: a clean buffer
      hipError_t e = hipMemsetAsync(R.ex, 0, R.words * sizeof(uint64_t), st);
      if (e != hipSuccess) return e;
      R.next = 1;
    }
    a.ep0 = (uint32_t)R.next;
    a.parity = R.parity;
    a.serial = R.serial++;
    a.col0 = g0 * h.kc;
    const int groups = h.groups - g0 < h.per ? h.groups - g0 : h.per;
    const hipError_t e = mode == 0 ? dispatch<0>(st, a, h, groups) : dispatch<1>(st, a, h, groups);
    if (e != hipSuccess) return e;
    R.next += span;
    // the launches of one solve share a count (its largest); the next solve takes the other
  }
  R.parity ^= 1;
  return hipSuccess;
}
