// Multigrid-preconditioned CG of the pressure Poisson system: the kernels of
// the preconditioner's products and of the vector update. Part of
// kernels_krylov.hip, whose start, confirmation and product w = A z it shares.
//
// An iteration (Chronopoulos-Gear CG, u = z = B r in place of D^{-1} r):
//   products: [||r||^2] stop test in the first one; z = B r (three or five
//             sparse products, mesh.hpp MgHierarchy), partial r.z in the last
//   spmv:     w = A z, partial z.w (small hierarchies: formed by the last product
//             from the same gathers, with A times its rows as second values)
//   update:   [gamma = r.z, delta = z.w]; beta = gamma / gamma_old,
//             alpha = gamma / (delta - beta gamma / alpha_old); p = z + beta p,
//             s = w + beta s, x += alpha p, r -= alpha s, partial r.r
// A product gives 2^lg lanes to a row, so that short rows of the finest level
// and the restrictions' long ones both load coalesced, four entries per lane
// in flight; its blocks take about the same number of entries each.
//
// Bound by launches and the latency of rp -> entry -> gather, not by bytes (all
// of it stays in the Infinity Cache): at 512^2 in FP64 the five products take
// 5.8, 5.9 (three times) and 10.1 us for 15, 11, 1, 16 and 31 MB, the update
// 7.6 us and the product w = A z 6.3 us under rocprofv3, 47 us an iteration
// against 9.7 us of the Jacobi form, which needs 80 times as many.
#pragma once

namespace ipcs {

// Sum over aligned groups of 2^LG lanes, the same in every lane of the group.
template <int LG>
__device__ __forceinline__ double lanes_sum(double v) {
  if constexpr (LG == 6) return wave_total(v);
  if constexpr (LG >= 1) v += dpp_d<0xb1>(v);    // quad_perm [1,0,3,2]
  if constexpr (LG >= 2) v += dpp_d<0x4e>(v);    // quad_perm [2,3,0,1]
  if constexpr (LG >= 3) v += dpp_d<0x141>(v);   // mirror within 8 lanes
  if constexpr (LG >= 4) v += dpp_d<0x140>(v);   // mirror within 16 lanes
  if constexpr (LG >= 5) v += __shfl_xor(v, 16, 64);
  return v;
}

// Rows [job.row0, job.row1) of y = X x, 2^LG lanes per row (LG 8: the block).
// put(row, sum, sum2) runs in one lane of each row; TWO: sum2 is the row's sum
// with the second values, else 0.
template <int LG, bool TWO, class VT, class F>
__device__ __forceinline__ void mg_rows(const MgStep& S, const MgJob& job, double* sh, F put) {
  // (three at a time with second values: at four the shared launches of a
  // batch lost a wave per SIMD)
  constexpr int LN = 1 << LG, PER = KBS >> LG, U = TWO ? 3 : 4;
  const gptr<const int32_t> rp = G(S.rp), col = G(S.col);
  const gptr<const VT> val = G(static_cast<const VT*>(S.val));
  const gptr<const double> val2 = G(S.val2);
  const gptr<const double> x = G(S.x);
  const int sub = (int)threadIdx.x & (LN - 1);
  for (int i0 = job.row0; i0 < job.row1; i0 += PER) {
    const int i = i0 + ((int)threadIdx.x >> LG);
    const int ic = i < job.row1 ? i : job.row0;
    const int b = rp[ic], e = rp[ic + 1];
    double acc = 0.0, acc2 = 0.0;
    for (int k = b + sub; k < e; k += LN * U) {
      int c[U];
      double a[U], a2[U], v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int kk = k + u * LN < e ? k + u * LN : k;
        c[u] = col[kk];
        a[u] = (double)val[kk];
        a2[u] = TWO ? val2[kk] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = x[c[u]];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        acc += k + u * LN < e ? a[u] * v[u] : 0.0;
        if (TWO) acc2 += k + u * LN < e ? a2[u] * v[u] : 0.0;
      }
    }
    if constexpr (LG == 8) {
      auto block = [&](double t) {
        t = wave_total(t);
        __syncthreads();
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = t;
        __syncthreads();
        return (sh[0] + sh[1]) + (sh[2] + sh[3]);
      };
      acc = block(acc);
      if (TWO) acc2 = block(acc2);
    } else {
      acc = lanes_sum<LG>(acc);
      if (TWO) acc2 = lanes_sum<LG>(acc2);
    }
    if (sub == 0 && i < job.row1) put(i, acc, acc2);
  }
}

template <bool TWO, class VT, class F>
__device__ __forceinline__ void mg_job(const MgStep& S, const MgJob& job, double* sh, F put) {
  switch (job.lg) {   // the same for the whole block
    case 2: mg_rows<2, TWO, VT>(S, job, sh, put); break;
    case 3: mg_rows<3, TWO, VT>(S, job, sh, put); break;
    case 4: mg_rows<4, TWO, VT>(S, job, sh, put); break;
    case 5: mg_rows<5, TWO, VT>(S, job, sh, put); break;
    case 6: mg_rows<6, TWO, VT>(S, job, sh, put); break;
    default: mg_rows<8, TWO, VT>(S, job, sh, put); break;
  }
}

// One product. KIND 0: the first of an iteration, with the stop test on the
// residual of the last update (block 0 of the group records it; a block that
// finds the new status already there returns as the test would have it);
// KIND 1: between; KIND 2: the last, with the partial sums of r.z; KIND 3: the
// last with w = A z from the same gathers, and the partial sums of r.z and z.w
// (FP64 values in the mixed form too: w has to be A z for this z).
template <int KIND, class VT>
__device__ __forceinline__ void mg_product(const KGroup& g, const MGroup& m, const MgStep& S, int jb,
                                           int par) {
  __shared__ double sh[(KBS / 64) * 2];
  const gptr<const KState> st = G((const KState*)g.v[0].st);
  const int status = st->status;
  const MgJob job = S.job[jb];
  if (KIND == 0) {
    const double lim = st->tol2 * st->bb;
    double rr[1];
    load_partials<1, 1>(g.part_v[par] + g.nblk_v, g.nblk_v, rr);   // value 1 of the records
    block_sum_t<KBS, 1>(rr, sh);
    // after the sum: block 0 may write the status while a block reads it, and
    // a wave that sees it returns where the sum sends the others
    if (status != KS_RUN) return;
    const bool lead = jb == 0 && threadIdx.x == 0;
    if (!finite(rr[0]) || rr[0] <= lim) {
      if (lead) {
        KState* w = g.v[0].st;
        w->rr = rr[0];
        w->status = finite(rr[0]) ? KS_PENDING : KS_NONFINITE;
      }
      return;
    }
    if (lead) g.v[0].st->rr = rr[0];
  } else if (status != KS_RUN) {
    return;
  }
  if (KIND == 3) {
    double dot[2] = {0.0, 0.0};
    mg_job<true, double>(S, job, sh, [&](int i, double z, double w) {
      G(S.y)[i] = z;
      G(g.v[0].w)[i] = w;
      dot[0] += z * G(S.x)[i];   // the residual leads the input vector
      dot[1] += z * w;
    });
    block_sum_t<KBS, 2>(dot, sh);
    if (threadIdx.x == 0) {
      G(m.part_z)[jb] = dot[0];
      G(m.part_z)[m.nz + jb] = dot[1];
    }
  } else if (KIND == 2) {
    double dot[1] = {0.0};
    mg_job<false, VT>(S, job, sh, [&](int i, double v, double) {
      G(S.y)[i] = v;
      dot[0] += v * G(S.x)[i];
    });
    block_sum_t<KBS, 1>(dot, sh);
    if (threadIdx.x == 0) G(m.part_z)[jb] = dot[0];
  } else {
    mg_job<false, VT>(S, job, sh, [&](int i, double v, double) { G(S.y)[i] = v; });
  }
}

template <int KIND, class VT>
__global__ void __launch_bounds__(KBS) k_mg(const KGroup* groups, const MGroup* mgs,
                                            int slot, int par) {
  const MGroup& m = mgs[blockIdx.y];
  if ((int)blockIdx.x >= m.st[slot].njob) return;
  if (KIND == 2 && m.st[slot].val2)
    mg_product<3, VT>(groups[blockIdx.y], m, m.st[slot], blockIdx.x, par);
  else
    mg_product<KIND, VT>(groups[blockIdx.y], m, m.st[slot], blockIdx.x, par);
}

// the same for one group, whose descriptors come with the launch
template <int KIND, class VT>
__global__ void __launch_bounds__(KBS) k_mg1(KGroup g, MGroup m, MgStep S, int par) {
  mg_product<KIND, VT>(g, m, S, blockIdx.x, par);
}

__global__ void __launch_bounds__(KBS) k_mgcg_update(const KGroup* groups, const MGroup* mgs,
                                                     const int2* bmap, int par) {
  GROUP_HEAD(bmap)
  constexpr int EV = kept_v(1);
  __shared__ double sh[(KBS / 64) * 2];
  const KVecs& V = g.v[0];
  const gptr<const KState> st = G((const KState*)V.st);
  const int status = st->status;
  const double g_old = st->sc[par ^ 1], a_old = st->alpha[par ^ 1];
  double xi[EV], ri[EV], pi[EV], si[EV], wi[EV], zi[EV];
#pragma unroll
  for (int e = 0; e < EV; ++e) {
    const int i = row_clamp(row_of<EV>(lb, e), g.n);
    xi[e] = G(V.x)[i];
    ri[e] = G(V.r)[i];
    pi[e] = G(V.p)[i];
    si[e] = G(V.s)[i];
    wi[e] = G(V.w)[i];
    zi[e] = G(V.u)[i];
  }
  double t[2];
  const MGroup& m = mgs[m_.x];
  const bool two = m.st[MG_SLOTS - 1].val2 != nullptr;
  load_partials<1, 1>(m.part_z, m.nz, t);
  load_partials<1, 1>(two ? m.part_z + m.nz : g.part_m, two ? m.nz : g.nblk_m, t + 1);
  block_sum_t<KBS, 2>(t, sh);
  if (status != KS_RUN) return;
  const bool lead = lb == 0 && threadIdx.x == 0;
  const double gam = t[0], del = t[1];
  const double beta = gam / g_old, den = del - beta * gam / a_old;
  if (!(finite(gam) && finite(del)) || !(den > 0.0) || !(gam > 0.0)) {
    if (lead) V.st->status = finite(gam) && finite(del) ? KS_BREAKDOWN : KS_NONFINITE;
    return;
  }
  const double alpha = gam / den;
  if (lead) {
    V.st->sc[par] = gam;
    V.st->alpha[par] = alpha;
    V.st->it += 1;
  }
  double rr[1] = {0.0};
#pragma unroll
  for (int e = 0; e < EV; ++e) {
    const int i = row_of<EV>(lb, e);
    if (i >= g.n) continue;
    const double p = zi[e] + beta * pi[e], s = wi[e] + beta * si[e];
    const double r = ri[e] - alpha * s;
    G(V.x)[i] = xi[e] + alpha * p;
    G(V.r)[i] = r;
    G(V.p)[i] = p;
    G(V.s)[i] = s;
    rr[0] += r * r;
  }
  // value 1 of the records, which the next iteration's stop test reads
  block_sum_t<KBS, 1>(rr, sh);
  if (threadIdx.x == 0) G(g.part_v[par ^ 1])[g.nblk_v + lb] = rr[0];
}

// One product of the preconditioner by itself, for the vector of every group
// (blockIdx.y). LAST: out[g * ld + i] = scale * value (+ add[g * ld + i]).
template <bool LAST>
__global__ void __launch_bounds__(KBS) k_mg_cycle(const MGroup* mgs, int slot, double scale,
                                                  const double* add, double* out, int64_t ld) {
  __shared__ double sh[KBS / 64];
  const MgStep& S = mgs[blockIdx.y].st[slot];
  if ((int)blockIdx.x >= S.njob) return;
  const int64_t o = LAST ? (int64_t)blockIdx.y * ld : 0;
  mg_job<false, double>(S, S.job[blockIdx.x], sh, [&](int i, double v, double) {
    if (LAST) G(out)[o + i] = scale * v + (add ? G(add)[o + i] : 0.0);
    else G(S.y)[i] = v;
  });
}

// ------------------------------------------------------------------ launchers
void mg_cycle(hipStream_t s, const MGroup* groups, int nvec, const int* nblocks, double scale,
              const double* add, double* out, int64_t ld) {
  for (int slot = 0; slot < MG_SLOTS; ++slot) {
    if (nblocks[slot] == 0) continue;
    const dim3 grid(nblocks[slot], nvec);
    if (slot == MG_SLOTS - 1)
      hipLaunchKernelGGL((k_mg_cycle<true>), grid, dim3(KBS), 0, s, groups, slot, scale, add, out,
                         ld);
    else
      hipLaunchKernelGGL((k_mg_cycle<false>), grid, dim3(KBS), 0, s, groups, slot, scale, add, out,
                         ld);
    HIP_LAUNCH_OK();
  }
}

template <int KIND, class VT>
static void mg_launch(hipStream_t s, const KLaunch& L, const MLaunch& M, int slot, int par) {
  if (KIND == 2 && L.ngroups == 1 && M.one.st[slot].val2)
    launch(k_mg1<3, VT>, dim3(M.nblocks[slot]), dim3(KBS), 0, s, M.kone, M.one, M.one.st[slot],
           par);
  else if (L.ngroups == 1 && M.one.part_z)
    launch(k_mg1<KIND, VT>, dim3(M.nblocks[slot]), dim3(KBS), 0, s, M.kone, M.one,
           M.one.st[slot], par);
  else
    over_groups(L.ngroups, [&](int g, int n) {
      launch(k_mg<KIND, VT>, dim3(M.nblocks[slot], n), dim3(KBS), 0, s, L.groups + g,
             M.groups + g, slot, par);
    });
}

template <class VT>
static void mg_product_t(hipStream_t s, const KLaunch& L, const MLaunch& M, int slot, int par) {
  if (slot == 0) mg_launch<0, VT>(s, L, M, slot, par);
  else if (slot + 1 < MG_SLOTS) mg_launch<1, VT>(s, L, M, slot, par);
  else mg_launch<2, VT>(s, L, M, slot, par);
}

void mg_product(hipStream_t s, const KLaunch& L, const MLaunch& M, int slot, int par) {
  if (M.fp32) mg_product_t<float>(s, L, M, slot, par);
  else mg_product_t<double>(s, L, M, slot, par);
}

void mg_update(hipStream_t s, const KLaunch& L, const MLaunch& M, int par) {
  launch(k_mgcg_update, dim3(L.nblocks_v), dim3(KBS), 0, s, L.groups, M.groups, L.bmap_v, par);
}

}  // namespace ipcs
