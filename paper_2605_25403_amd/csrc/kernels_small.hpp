// Whole Krylov solves of small systems, one block per system: the start, the
// iterations, the confirmation with the true residual and the restarts of
// kernels_krylov.hip in one launch, with the same recurrences, stopping rule,
// statuses and iteration counts (sums are formed in another order). Part of
// kernels_krylov.hip.
//
// Systems of a few thousand rows are bound by launches and polls: an iteration
// of four kernels costs about 22 us whatever it computes. Here an iteration
// is a few block barriers: a thread keeps R rows of the vectors in registers,
// the gathered vector (for BiCGStab also rhat and x) lies in LDS, and the
// matrix in registers too where its rows are short (512 threads of up to 256
// registers); longer rows are streamed from the XCD's L2 (1024 threads, more
// loads in flight). Bound by the LDS gathers and barriers of one CU in the
// register form, about 1.3 us a CG iteration at 16^2 (289 rows) and 2.2 us at
// 44^2, and by one CU's 150 GB/s in the streamed form. Phases before and after
// (ms): 16^2 momentum 0.35 -> 0.06, pressure 0.45 -> 0.11, correction 0.30 ->
// 0.07; 24^2 0.39 -> 0.21, 0.64 -> 0.16, 0.31 -> 0.15; 4^3 0.81 -> 0.31, 0.36 ->
// 0.10, 0.50 -> 0.20; P3-P2 on 16^2 0.43 -> 0.25, 1.05 -> 0.30, 0.29 -> 0.16.
#pragma once

namespace ipcs {

// The R rows of a thread (row e * BS + tid) of the SELL-64 matrix, applied to
// the vector in LDS in the order of sell_row (column by column), streamed from
// the L2; the slice offsets stay in registers.
template <int BS, int R, class VT>
struct SmallRows {
  int base[R], w[R];
  gptr<const VT> val;
  gptr<const int32_t> col;
  __device__ __forceinline__ void load(const KGroup& g) {
    val = G(static_cast<const VT*>(g.val));
    col = G(g.col);
#pragma unroll
    for (int e = 0; e < R; ++e) {
      const int i = e * BS + (int)threadIdx.x, s = i >> 6;   // s: the same in the wavefront
      const bool on = 64 * s < g.n;
      const int b0 = on ? G(g.sptr)[s] : 0, b1 = on ? G(g.sptr)[s + 1] : 0;
      base[e] = i < g.n ? b0 + (i & 63) : 0;
      w[e] = __builtin_amdgcn_readfirstlane((b1 - b0) >> 6);
    }
  }
  // y = A xs; rows past the end read row 0's entries and are discarded by the caller
  __device__ __forceinline__ void apply(const double* xs, double (&y)[R]) const {
#pragma unroll
    for (int e = 0; e < R; ++e) {
      y[e] = 0.0;
      for (int k = 0; k < w[e]; k += 8) {
        int c[8];
        double a[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int at = base[e] + 64 * (k + q < w[e] ? k + q : w[e] - 1);
          c[q] = col[at];
          a[q] = (double)val[at];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) y[e] += k + q < w[e] ? a[q] * xs[c[q]] : 0.0;
      }
    }
  }
};

// The same with the rows' entries, at most W of them, kept in registers for
// the whole solve: values (0 past the row) and 16-bit byte offsets into the
// vector, two to a register. Entries are taken four at a time up to the
// slice's width, which is the same in a wavefront.
template <int BS, int R, int W, class VT>
struct SmallRegs {
  VT a[R][W];
  uint32_t c[R][W / 2];
  int w[R];
  __device__ __forceinline__ void load(const KGroup& g) {
    SmallRows<BS, R, VT> m;
    m.load(g);
#pragma unroll
    for (int e = 0; e < R; ++e) {
      w[e] = m.w[e];
#pragma unroll
      for (int q = 0; q < W; ++q) {
        const int at = q < w[e] ? m.base[e] + 64 * q : m.base[e];
        const VT av = m.val[at];
        a[e][q] = q < w[e] ? av : (VT)0;
        const uint32_t cc = 8u * (uint32_t)m.col[at];
        c[e][q / 2] = q & 1 ? c[e][q / 2] | cc << 16 : cc;
      }
    }
  }
  __device__ __forceinline__ void apply(const double* xs, double (&y)[R]) const {
    const char* xb = reinterpret_cast<const char*>(xs);
#pragma unroll
    for (int e = 0; e < R; ++e) {
      y[e] = 0.0;
#pragma unroll
      for (int q0 = 0; q0 < W; q0 += 4) {
        if (q0 >= w[e]) break;
        double v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          v[q] = *reinterpret_cast<const double*>(
              xb + (q & 1 ? c[e][(q0 + q) / 2] >> 16 : c[e][(q0 + q) / 2] & 0xffffu));
#pragma unroll
        for (int q = 0; q < 4; ++q) y[e] += (double)a[e][q0 + q] * v[q];
      }
    }
  }
};

// Solves system blockIdx.x of group blockIdx.y. One matrix product per turn of
// the loop, whatever it is for (one copy of it in the code and in registers).
// Every thread holds the same scalars (the totals of block_sum_t), so all
// branches on them are uniform.
template <bool PCG, int R, int W, class VT>
__global__ void __launch_bounds__(small_bs(W)) k_small(const KGroup* groups) {
  constexpr int BS = small_bs(W);
  const KGroup& g = groups[blockIdx.y];
  if ((int)blockIdx.x >= g.nsys) return;
  const KVecs& V = g.v[blockIdx.x];
  extern __shared__ double lds[];
  __shared__ double sh[(BS / 64) * 4];
  const int n = g.n, tid = threadIdx.x;
  double* xs = lds;                    // the gathered vector
  double* rh = lds + n;                // BiCGStab: rhat
  double* xl = lds + 2 * (size_t)n;    // BiCGStab: x
  const double tol2 = V.st->tol2, zero2 = V.st->zero2;
  double x[PCG ? R : 1], r[R], p[R], s[R], v[PCG ? 1 : R], di[R];
  std::conditional_t<W != 0, SmallRegs<BS, R, W ? W : 2, VT>, SmallRows<BS, R, VT>> A;
  A.load(g);
  auto row = [&](int e) { return e * BS + tid; };
  // the next gathered vector; every thread is past its last read of the old
  // one after a block sum
  auto put = [&](int e, double val) {
    if (row(e) < n) xs[row(e)] = val;
  };
#pragma unroll
  for (int e = 0; e < R; ++e) {
    const int i = row(e), ic = row_clamp(i, n);
    di[e] = G(g.dinv)[ic];
    const double x0 = G(V.x)[ic];
    if (PCG) x[e] = x0;
    if (i < n) {
      xs[i] = x0;
      if (!PCG) xl[i] = x0;
    }
  }
  __syncthreads();
  enum { START, ITER, SECOND };        // xs holds x; u or phat; shat
  int phase = START, status = KS_RUN, it = 0, nchecks = 0, nstall = 0, launches = 0;
  bool first = true;
  double bb = 0.0, rr = 0.0, rr_best = 0.0, old1 = 0.0, old2 = 0.0;   // PCG: gamma, alpha; else rho, alpha
  for (;;) {
    double y[R];
    A.apply(xs, y);
#pragma unroll
    for (int e = 0; e < R; ++e) y[e] = row(e) < n ? y[e] : 0.0;
    if (phase == START) {
      // the start, or the confirmation of the current iterate
      double t[2] = {0.0, 0.0};
#pragma unroll
      for (int e = 0; e < R; ++e) {
        const double bi = row(e) < n ? G(V.b)[row_clamp(row(e), n)] : 0.0;
        r[e] = bi - y[e];
        t[0] += r[e] * r[e];
        t[1] += bi * bi;
      }
      block_sum_t<BS, 2>(t, sh);
      rr = t[0];
      if (first) bb = t[1];
      else nchecks += 1;
      status = KS_RUN;
      if (bb == 0.0 || bb <= zero2) status = KS_ZERO;
      else if (!finite(rr)) status = KS_NONFINITE;
      else if (rr <= tol2 * bb) status = KS_DONE;
      else if (launches >= g.maxit) status = KS_MAXIT;
      if (first || rr <= 0.81 * rr_best) {
        rr_best = rr;
        nstall = 0;
      } else {
        nstall += 1;
      }
      first = false;
      if (status == KS_RUN && nstall >= KSTALL_CHECKS) status = KS_STALL;
      if (status != KS_RUN) break;
      old1 = PCG ? INFINITY : rr;
      old2 = 1.0;
#pragma unroll
      for (int e = 0; e < R; ++e) {
        p[e] = PCG ? 0.0 : r[e];
        s[e] = 0.0;
        put(e, di[e] * r[e]);
        if (!PCG && row(e) < n) rh[row(e)] = r[e];
      }
      phase = ITER;
    } else if (PCG) {
      double q[3] = {0.0, 0.0, 0.0};   // r.u, r.r, u.w
#pragma unroll
      for (int e = 0; e < R; ++e) {
        const double u = di[e] * r[e];
        q[0] += r[e] * u;
        q[1] += r[e] * r[e];
        q[2] += u * y[e];
      }
      block_sum_t<BS, 3>(q, sh);
      const double gam = q[0], del = q[2];
      rr = q[1];
      const double beta = gam / old1, den = del - beta * gam / old2;
      if (!(finite(gam) && finite(rr) && finite(del))) status = KS_NONFINITE;
      else if (rr <= tol2 * bb) status = KS_PENDING;
      else if (!(den > 0.0)) status = KS_BREAKDOWN;
      if (status == KS_RUN) {
        const double alpha = gam / den;
        it += 1;
        old1 = gam;
        old2 = alpha;
#pragma unroll
        for (int e = 0; e < R; ++e) {
          p[e] = di[e] * r[e] + beta * p[e];
          s[e] = y[e] + beta * s[e];
          x[e] += alpha * p[e];
          r[e] -= alpha * s[e];
          put(e, di[e] * r[e]);
        }
      }
    } else if (phase == ITER) {
      double q[2] = {0.0, 0.0};        // rhat.v, r.r
#pragma unroll
      for (int e = 0; e < R; ++e) {
        v[e] = y[e];
        q[0] += row(e) < n ? rh[row_clamp(row(e), n)] * y[e] : 0.0;
        q[1] += r[e] * r[e];
      }
      block_sum_t<BS, 2>(q, sh);
      rr = q[1];
      old2 = old1 / q[0];
      if (!(finite(q[0]) && finite(rr))) status = KS_NONFINITE;
      else if (rr <= tol2 * bb) status = KS_PENDING;
      else if (!(std::fabs(q[0]) >= 1e-300) || !finite(old2)) status = KS_RESTART;
#pragma unroll
      for (int e = 0; e < R; ++e) {
        s[e] = r[e] - old2 * v[e];
        put(e, di[e] * s[e]);
      }
      phase = SECOND;
    } else {
      double k[4] = {0.0, 0.0, 0.0, 0.0};   // t.s, t.t, rhat.s, rhat.t
#pragma unroll
      for (int e = 0; e < R; ++e) {
        const double h = row(e) < n ? rh[row_clamp(row(e), n)] : 0.0;
        k[0] += y[e] * s[e];
        k[1] += y[e] * y[e];
        k[2] += h * s[e];
        k[3] += h * y[e];
      }
      block_sum_t<BS, 4>(k, sh);
      // t.t == 0 means A shat = 0, so s = 0: x + alpha phat solves the system
      const double omega = k[1] == 0.0 ? 0.0 : k[0] / k[1];
      const double rho = k[2] - omega * k[3];
      const double beta = (rho / old1) * (old2 / omega);
      if (!(finite(k[0]) && finite(k[1]) && finite(k[2]) && finite(k[3]))) {
        status = KS_NONFINITE;
      } else {
        if (k[1] == 0.0) status = KS_PENDING;
        else if (!(std::fabs(omega) >= 1e-300) || !(std::fabs(rho) >= 1e-300) || !finite(beta))
          status = KS_RESTART;
        it += 1;
#pragma unroll
        for (int e = 0; e < R; ++e) {
          if (row(e) < n) xl[row(e)] += di[e] * (old2 * p[e] + omega * s[e]);
          r[e] = s[e] - omega * y[e];
          p[e] = r[e] + beta * (p[e] - omega * v[e]);
          put(e, di[e] * p[e]);
        }
        old1 = rho;
      }
      phase = ITER;
    }
    if (status == KS_PENDING || status == KS_RESTART) {
      phase = START;
#pragma unroll
      for (int e = 0; e < R; ++e) put(e, PCG ? x[e] : xl[row_clamp(row(e), n)]);
    } else if (status != KS_RUN) {
      break;
    } else if (phase == ITER) {
      if (launches >= g.maxit) {
        status = KS_MAXIT;
        break;
      }
      launches += 1;
    }
    __syncthreads();
  }
#pragma unroll
  for (int e = 0; e < R; ++e) {
    const int i = row(e);
    if (i < n) G(V.x)[i] = status == KS_ZERO ? 0.0 : PCG ? x[e] : xl[i];
  }
  if (tid == 0) {
    KState* st = V.st;
    st->bb = bb;
    st->rr = rr;
    st->it = it;
    st->nchecks = nchecks;
    st->nstall = nstall;
    st->rr_best = rr_best;
    st->status = status;
  }
}

// ------------------------------------------------------------------ launchers
template <bool PCG, int R, int W, class VT>
static void small_launch(hipStream_t s, const KLaunch& L, int nmax) {
  const size_t lds = sizeof(double) * (size_t)nmax * (PCG ? 1 : 3);
  over_groups(L.ngroups, [&](int g, int n) {
    launch(k_small<PCG, R, W, VT>, dim3(L.ns, n), dim3(small_bs(W)), (uint32_t)lds, s,
           L.groups + g);
  });
}

template <int W, bool FP32, class F>
static void with_small_rows(int rows, F f) {
  switch (rows) {
    case 1: f(ic<1>{}); return;
    case 2: f(ic<2>{}); return;
    case 3: f(ic<3>{}); return;
    case 4:
      if constexpr (small_rmax(W, FP32) >= 4) return f(ic<4>{});
      break;
    case 5:
      if constexpr (small_rmax(W, FP32) >= 5) return f(ic<5>{});
      break;
  }
  fail(IPCS_E_INVALID, "a one-block solve of that many rows per thread");
}

void small_solve(hipStream_t s, const KLaunch& L, bool pcg, SmallForm f, int nmax) {
  auto width = [&](auto Wc) {
    constexpr int W = decltype(Wc)::value;
    auto go = [&](auto V) {
      using VT = decltype(V);
      with_small_rows<W, sizeof(VT) == 4>(f.rows, [&](auto Rc) {
        constexpr int R = decltype(Rc)::value;
        if (pcg) small_launch<true, R, W, VT>(s, L, nmax);
        else if constexpr (W == 8) fail(IPCS_E_INVALID, "no velocity rows are that short");
        else small_launch<false, R, W, VT>(s, L, nmax);
      });
    };
    if (L.fp32) go(float{});
    else go(double{});
  };
  if (f.width == 8) width(ic<8>{});
  else if (f.width == 20) width(ic<20>{});
  else width(ic<0>{});
}

// The form for a system of n rows, of at most maxw entries and nent SELL
// entries in all, or rows 0 where one block does not pay.
SmallForm small_form(int64_t n, int maxw, int64_t nent, bool pcg, bool fp32) {
  for (int w : {8, 20}) {
    const int64_t r = div_up(n, (int64_t)small_bs(w));
    if (maxw <= w && (pcg || w != 8) && r <= small_rmax(w, fp32)) return SmallForm{(int)r, w};
  }
  const int64_t r = div_up(n, (int64_t)small_bs(0));
  if (nent <= SMALL_STREAM && r <= small_rmax(0, fp32)) return SmallForm{(int)r, 0};
  return SmallForm{};
}

}  // namespace ipcs
