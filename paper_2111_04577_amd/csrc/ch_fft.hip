// Right-hand side of the fused Cahn-Hilliard solve and its forward x transform in one pass:
// Q - L_N b of eqs. NS25-NS34 (stencil_ch.hip, ch_rhs) formed row by row, transformed in LDS
// (r2c, as k_fft_x_fwd) and written in the spectral layout, so that the right-hand side never
// goes through memory (2 N_f of the 5 N_f + 6 N_c words of the two passes). The halo rows give part of
// that back: a block of TY rows reads TY + 2 of phi^n and phi^{n-1}. At 512 columns in FP64 it holds
// two rows and reads four, 2.75 GB a launch by counter where the pass's own words are 2.02 GB and the
// two passes moved 3.19; in FP32, where it holds four, 1.08, 1.01 and 1.57 GB.
//
// A block owns TY whole x rows and marches up KB layers. Each thread owns 16 bytes of a row (4
// columns in FP32, 2 in FP64): every load of the march is a 16-byte load, the x neighbours are the
// thread's own registers but for one value at either end, and the coarse velocities of eq. dual1
// are loaded once per coarse column and layer instead of once per fine column. phi* and w* = f(phi*)
// - (S/Cn^2) phi* of the column on the layers K-1, K, K+1 stay in registers; only phi* of the
// current layer, with one row of halo in y and none in x (the row is whole and periodic), goes
// through LDS, in two slots so that a layer costs one barrier. w* of the y neighbours is formed
// again from phi* (four operations). The rows of NB layers are then transformed together: with
// four layers every thread has its P points of the transform (lds_fft16.hpp in FP32, lds_fft.hpp in
// FP64).
#include "fine.hpp"
#include "lds_fft.hpp"
#include "lds_fft16.hpp"

namespace drpf {

namespace {

template <typename T, int N>
struct alignas(16) Vec {
  T v[N];
};
// the same in global memory, where a caller's array may be aligned to its elements only
template <typename T, int N>
struct __attribute__((packed, aligned(alignof(T)))) VecU {
  T v[N];
};
template <int N, typename T>
__device__ __forceinline__ Vec<T, N> ld_vec(const T* base, unsigned byte_off) {
  const VecU<T, N> u = *reinterpret_cast<const VecU<T, N>*>(reinterpret_cast<const char*>(base) + byte_off);
  Vec<T, N> r;
#pragma unroll
  for (int i = 0; i < N; ++i) r.v[i] = u.v[i];
  return r;
}

// LOGM: log2(nx / 2) at compile time (FP32), 0 = run-time length (FP64). MODE: 0 dual
// resolution, 1 single resolution, 2 advection given (WENO-Z). RELAX: relaxed walls at rest.
template <typename T, int LOGM, int MODE, bool RELAX, bool Y3D>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4)))
    k_ch_fft(const T* __restrict__ phin, const T* __restrict__ phinm1, Prolonged<T> pv, cx<T>* __restrict__ out,
             const T* __restrict__ advp, int ny, int nz, int logm, int TY, int KB, int NB, T ihx, T ihy, T ihz,
             const cx<T>* __restrict__ twM, const cx<T>* __restrict__ twN, StepConsts c) {
  constexpr int CPT = 16 / sizeof(T);
  constexpr bool sr = MODE == 1, pre = MODE == 2;
  constexpr int NCC = sr ? CPT : CPT / 2;  // coarse columns of a thread
  using VT = Vec<T, CPT>;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lm = LOGM > 0 ? LOGM : logm;
  const int M = 1 << lm, nx = 2 * M;
  const int lv = lm + 1 - (CPT == 4 ? 2 : 1);  // log2 of the threads of a row
  const int tid = threadIdx.x, nth = blockDim.x;
  constexpr bool y3d = Y3D;
  const bool first = c.first != 0;
  const int ty = tid >> lv, X = (tid & ((1 << lv) - 1)) * CPT;
  // consecutive blocks, whose rows are neighbours, on one XCD
  const int b = xcd_block(), cols = ny / TY;
  const int Y0 = (b % cols) * TY, K0 = (b / cols) * KB;
  const int K1 = min(K0 + KB, nz);
  const int J = Y0 + ty;
  // LDS: two slots of phi* ([TY + 2][nx], 2D: one row each), the wall data tile of relaxed walls,
  // the rows of the transform, its twiddles
  const int rows = y3d ? TY + 2 : 1, HP = rows * nx;
  T* sP = reinterpret_cast<T*>(smem);
  T* sB = sP + 2 * HP;
  cx<T>* buf = reinterpret_cast<cx<T>*>(sB + (RELAX ? HP : 0));
  constexpr bool ct = LOGM > 0;
  using F = FftPlan<ct ? LOGM : 1, 3>;
  cx<T>* stw = buf + NB * TY * (ct ? F::LS : M);
  for (int e = tid; e < M; e += nth) stw[e] = twM[e];
  const unsigned own = (unsigned)(J * nx + X) * sizeof(T);
  // halo rows: the first two rows of threads load row Y0 - 1 and row Y0 + TY (TY >= 2 in 3D)
  const bool has_h = y3d && ty < 2;
  const int hr = ty == 0 ? 0 : TY + 1;  // row in the tile
  const unsigned hoff = has_h ? (unsigned)(wrap(ty == 0 ? Y0 - 1 : Y0 + TY, ny) * nx + X) * sizeof(T) : 0u;
  const int me = (y3d ? ty + 1 : 0) * nx;  // the thread's row in the tile
  auto kcl = [&](int K) { return min(max(K, 0), nz - 1); };
  // every access: the array's base plus one 32-bit byte offset (layer and lane parts added), so
  // that no 64-bit address per lane is kept through the march
  const unsigned lbytes = (unsigned)(ny * nx) * sizeof(T);
  auto ldv = [&](const T* a, int K, unsigned off) -> VT {
    return ld_vec<CPT>(a, (unsigned)kcl(K) * lbytes + off);
  };
  auto star = [&](const VT& a, const VT& bb) {
    VT r;
#pragma unroll
    for (int x = 0; x < CPT; ++x) r.v[x] = first ? a.v[x] : (T)2 * a.v[x] - bb.v[x];
    return r;
  };
  auto hat = [&](const VT& a, const VT& bb) {
    VT r;
#pragma unroll
    for (int x = 0; x < CPT; ++x) r.v[x] = first ? a.v[x] : (T)2 * a.v[x] - (T)0.5 * bb.v[x];
    return r;
  };
  const T icn2 = (T)c.inv_cn2, sc = (T)c.s_cn2;
  auto wstar = [&](T p) { return opaque((p * p * p - p) * icn2 - sc * p); };
  auto wvec = [&](const VT& p) {
    VT r;
#pragma unroll
    for (int x = 0; x < CPT; ++x) r.v[x] = wstar(p.v[x]);
    return r;
  };
  const T gb = (T)c.g_bot * ihz, gt = (T)c.g_top * ihz;
  const T kg = RELAX ? (T)(c.relax_kappa * c.inv_gamma0) * ihz : (T)0;
  // wall data of a wall layer from phi* and phi_hat there
  auto bval = [&](bool bottom, T p, T ph) {
    const T s = opaque((bottom ? gb : gt) * fma(-p, p, (T)1));
    return RELAX ? fma(kg, ph, s) : s;
  };
  // ---- face velocities of a coarse layer (eq. dual1)
  const int ic0 = sr ? X : X >> 1;
  const int jc = y3d && !sr ? (J >> 1) : J, jcw = y3d ? wrap(jc - 1, pv.cny) : 0;
  const int cplane = pv.cnx * pv.cny;
  const T h = (T)0.5;
  const bool jodd = J & 1;
  // half the velocity at the CPT + 1 x faces around the thread's columns and at the y faces either
  // side of each coarse column; w at the coarse faces above and below
  T uh[CPT + 1], vhp[NCC], vhm[NCC], wk[NCC], wkm[NCC];
  const unsigned ou = (unsigned)(jc * pv.cnx + ic0) * sizeof(T), oul = (unsigned)(jc * pv.cnx + wrap(ic0 - 1, pv.cnx)) * sizeof(T),
                 ovl = (unsigned)(jcw * pv.cnx + ic0) * sizeof(T);
  auto load_vel = [&](int k, bool next) {
    const unsigned lo = (unsigned)(k * cplane) * sizeof(T);
    // level n and n - 1 of the thread's NCC coarse columns, combined
    auto star2 = [&](const T* a, const T* bm, unsigned o, T* r) {
      const Vec<T, NCC> x = ld_vec<NCC>(a, o), y = ld_vec<NCC>(bm, o);
#pragma unroll
      for (int m = 0; m < NCC; ++m) r[m] = first ? x.v[m] : (T)2 * x.v[m] - y.v[m];
    };
    T us[NCC + 1], v0[NCC], v1[NCC];
    {
      const T x = ld_at(pv.un, lo + oul), y = ld_at(pv.unm1, lo + oul);
      us[0] = first ? x : (T)2 * x - y;
    }
    star2(pv.un, pv.unm1, lo + ou, us + 1);
    star2(pv.vn, pv.vnm1, lo + ou, v0);
    if (y3d) star2(pv.vn, pv.vnm1, lo + ovl, v1);
    // w below: the one above of the layer before, but for the block's first
    if (next) {
#pragma unroll
      for (int m = 0; m < NCC; ++m) wkm[m] = wk[m];
    } else if (k > 0) {
      star2(pv.wn, pv.wnm1, lo - (unsigned)cplane * sizeof(T) + ou, wkm);
    }
    if (k < pv.cnz - 1) star2(pv.wn, pv.wnm1, lo + ou, wk);
#pragma unroll
    for (int m = 0; m < NCC; ++m) {
      if (!y3d) v1[m] = v0[m];
      if (sr || !y3d) {
        vhp[m] = v0[m] * h;
        vhm[m] = v1[m] * h;
      } else {
        const T vc = h * (v1[m] + v0[m]);
        vhp[m] = (jodd ? v0[m] : vc) * h;
        vhm[m] = (jodd ? vc : v1[m]) * h;
      }
      if (k == 0) wkm[m] = (T)0;
      if (k == pv.cnz - 1) wk[m] = (T)0;
    }
#pragma unroll
    for (int x = 0; x <= CPT; ++x) {
      if (sr)
        uh[x] = us[x % (NCC + 1)] * h;
      else
        uh[x] = ((x & 1) ? h * (us[x >> 1] + us[((x >> 1) + 1) % (NCC + 1)]) : us[x >> 1]) * h;
    }
  };
  const T ihx2 = ihx * ihx, ihy2 = ihy * ihy, ihz2 = ihz * ihz;
  // ---- the march
  VT pm, p0, pp, ph0, phm, an, bn, ha, hb;
  {
    const VT a = ldv(phin, K0 - 1, own), a0 = ldv(phin, K0, own);
    const VT bm = ldv(phinm1, K0 - 1, own), b0 = ldv(phinm1, K0, own);
    an = ldv(phin, K0 + 1, own);
    bn = ldv(phinm1, K0 + 1, own);
    if (has_h) {
      ha = ldv(phin, K0, hoff);
      hb = ldv(phinm1, K0, hoff);
    }
    pm = star(a, bm);
    phm = hat(a, bm);
    p0 = star(a0, b0);
    ph0 = hat(a0, b0);
  }
  int kcur = -2;
  for (int Kb = K0; Kb < K1; Kb += NB) {
    const int Ke = min(Kb + NB, K1);
    for (int K = Kb; K < Ke; ++K) {
      const int k = sr ? K : (K >> 1);
      if (!pre && k != kcur) {
        load_vel(k, k == kcur + 1);
        kcur = k;
      }
      // layer K into its slot; the layers to come are in flight meanwhile
      T* P0 = sP + (K & 1) * HP;
      *reinterpret_cast<VT*>(P0 + me + X) = p0;
      const bool wall = K == 0 || K == nz - 1;
      if (has_h) {
        const VT hp = star(ha, hb);
        *reinterpret_cast<VT*>(P0 + hr * nx + X) = hp;
        if (RELAX && wall) {
          const VT hh = hat(ha, hb);
          VT bb;
#pragma unroll
          for (int x = 0; x < CPT; ++x) bb.v[x] = bval(K == 0, hp.v[x], hh.v[x]);
          *reinterpret_cast<VT*>(sB + hr * nx + X) = bb;
        }
      }
      if (RELAX && wall) {
        VT bb;
#pragma unroll
        for (int x = 0; x < CPT; ++x) bb.v[x] = bval(K == 0, p0.v[x], ph0.v[x]);
        *reinterpret_cast<VT*>(sB + me + X) = bb;
      }
      pp = star(an, bn);
      const VT php = hat(an, bn);
      if (K + 1 < K1) {
        an = ldv(phin, K + 2, own);
        bn = ldv(phinm1, K + 2, own);
        if (has_h) {
          ha = ldv(phin, K + 1, hoff);
          hb = ldv(phinm1, K + 1, hoff);
        }
      }
      VT av;
      if (pre) av = ldv(advp, K, own);
      __syncthreads();
      const int xl = (X - 1) & (nx - 1), xr = (X + CPT) & (nx - 1);
      const T pl = P0[me + xl], pr = P0[me + xr];
      const VT pu = y3d ? *reinterpret_cast<const VT*>(P0 + me + nx + X) : p0;
      const VT pd = y3d ? *reinterpret_cast<const VT*>(P0 + me - nx + X) : p0;
      const T wl = wstar(pl), wr = wstar(pr);
      const VT w0 = wvec(p0);
      VT rv;
#pragma unroll
      for (int x = 0; x < CPT; ++x) {
        const T p = p0.v[x], pzp = pp.v[x], pzm = pm.v[x], pyp = pu.v[x], pym = pd.v[x];
        const T pxp = x + 1 < CPT ? p0.v[(x + 1) % CPT] : pr, pxm = x > 0 ? p0.v[(x + CPT - 1) % CPT] : pl;
        const T w = w0.v[x];
        const T wxp = x + 1 < CPT ? w0.v[(x + 1) % CPT] : wr, wxm = x > 0 ? w0.v[(x + CPT - 1) % CPT] : wl;
        const T lapw = (wxp - 2 * w + wxm) * ihx2 + (wstar(pyp) - 2 * w + wstar(pym)) * ihy2 + (wstar(pzp) - 2 * w + wstar(pzm)) * ihz2;
        __builtin_amdgcn_sched_barrier(0);
        T adv;
        if (pre) {
          adv = av.v[x];
        } else {
          // fine z faces of eq. dual1 above and below; the walls carry zero flux
          const int m = sr ? x : x >> 1;
          const T wfp = K == nz - 1 ? (T)0 : (sr || (K & 1) ? wk[m] : h * (wkm[m] + wk[m]));
          const T wfm = K == 0 ? (T)0 : (sr ? wkm[m] : ((K & 1) ? h * (wkm[m] + wk[m]) : wkm[m]));
          // the flux between two of the thread's own columns is formed for each of them (opaque): as a
          // common product it would be rounded before the difference, not fused into it
          adv = (uh[x + 1] * (p + pxp) - (x > 0 ? opaque(uh[x]) : uh[x]) * (pxm + p)) * ihx + (vhp[m] * (p + pyp) - vhm[m] * (pym + p)) * ihy +
                (wfp * h * (p + pzp) - wfm * h * (pzm + p)) * ihz;
        }
        rv.v[x] = (T)c.pe_cn2 * (ph0.v[x] * (T)c.inv_dt - adv) + lapw;
      }
      // minus L_N b of the wall data, on the two layers next to each wall; the layer next to a
      // wall layer carries no data (nz >= 4)
      if (wall) {
        VT bc, bu, bd;
        T bl, br;
        if (RELAX) {
          bc = *reinterpret_cast<const VT*>(sB + me + X);
          bu = y3d ? *reinterpret_cast<const VT*>(sB + me + nx + X) : bc;
          bd = y3d ? *reinterpret_cast<const VT*>(sB + me - nx + X) : bc;
          bl = sB[me + xl];
          br = sB[me + xr];
        } else {
#pragma unroll
          for (int x = 0; x < CPT; ++x) {
            bc.v[x] = opaque(bval(K == 0, p0.v[x], (T)0));
            bu.v[x] = opaque(bval(K == 0, y3d ? P0[me + nx + X + x] : p0.v[x], (T)0));
            bd.v[x] = opaque(bval(K == 0, y3d ? P0[me - nx + X + x] : p0.v[x], (T)0));
          }
          bl = opaque(bval(K == 0, P0[me + xl], (T)0));
          br = opaque(bval(K == 0, P0[me + xr], (T)0));
        }
#pragma unroll
        for (int x = 0; x < CPT; ++x) {
          const T b0 = bc.v[x];
          const T bxp = x + 1 < CPT ? bc.v[(x + 1) % CPT] : br, bxm = x > 0 ? bc.v[(x + CPT - 1) % CPT] : bl;
          T lapb = (bxp - 2 * b0 + bxm) * ihx2 + (bu.v[x] - 2 * b0 + bd.v[x]) * ihy2;
          lapb -= b0 * ihz2;
          rv.v[x] = rv.v[x] - lapb;
        }
      } else if (K == 1 || K == nz - 2) {
#pragma unroll
        for (int x = 0; x < CPT; ++x) {
          T lapb = 0;
          if (K == 1) lapb += opaque(bval(true, pm.v[x], phm.v[x])) * ihz2;
          if (K == nz - 2) lapb += opaque(bval(false, pp.v[x], php.v[x])) * ihz2;
          rv.v[x] = rv.v[x] - lapb;
        }
      }
      // the row as (even, odd) pairs of the half-length complex transform
      const int line = (K - Kb) * TY + ty;
#pragma unroll
      for (int x = 0; x < CPT / 2; ++x) {
        const cx<T> z = mk<T>(rv.v[2 * x], rv.v[2 * x + 1]);
        const int e = (X >> 1) + x;
        if constexpr (ct)
          buf[line * F::LS + F::pad(e)] = z;
        else
          buf[(line << lm) + e] = z;
      }
      pm = p0;
      p0 = pp;
      phm = ph0;
      ph0 = php;
    }
    // ---- the transform of the batch's rows
    const int nl = (Ke - Kb) * TY;
    __syncthreads();
    if constexpr (ct) {
      const int fb = tid >> F::LT, fq = tid & (F::T - 1);
      fft16<T, false, LOGM, 3>(buf + (fb < nl ? fb : 0) * F::LS, fq, fb < nl, stw);
    } else {
      lds_fft<T, false, false>(buf, M, lm, nl, 0, stw);
    }
    const size_t lines = (size_t)(M + 1) * ny;
    const int lty = __ffs(TY) - 1;
    auto mode = [&](int l, int kk) {
      cx<T> zk, zm;
      if constexpr (ct) {
        const cx<T>* row = buf + l * F::LS;
        zk = row[F::pad(kk == M ? 0 : kk)];
        zm = conj(row[F::pad(kk == 0 ? 0 : M - kk)]);
      } else {
        const cx<T>* row = buf + (l << lm);
        zk = row[kk == M ? 0 : kk];
        zm = conj(row[kk == 0 ? 0 : M - kk]);
      }
      const cx<T> E = h * (zk + zm);
      const cx<T> O = h * mul_mi(zk - zm);
      return E + twN[kk] * O;
    };
    for (int e = tid; e < nl << lm; e += nth) {
      const int l = e >> lm, kk = e & (M - 1);
      const int z = Kb + (l >> lty), ky = Y0 + (l & (TY - 1));
      out[z * lines + (size_t)ky * M + kk] = mode(l, kk);
    }
    for (int l = tid; l < nl; l += nth) {
      const int z = Kb + (l >> lty), ky = Y0 + (l & (TY - 1));
      out[z * lines + (size_t)M * ny + ky] = mode(l, M);
    }
    // the next batch's first barrier separates these reads from its writes to buf
  }
}

}  // namespace

// Whether the fused pass takes this grid. A block of 512 threads holds at least two whole rows in
// 3D (the halo rows are loaded by its first two) and one in 2D; the transform takes 16 to 1024
// points; offsets are 32-bit; moving relaxed walls read phi* around the wall cells (ch_rhs). Below
// 16 columns and beyond 1024 there is one thread, or less than one row, per block; measured in
// range, us per step, two passes against one: fine 64 x 64 x 32 FP32 86.2 against 78.9, 512 x 1 x 256
// FP64 63.8 against 57.4, 256 x 256 x 128 FP64 452 against 402, 512 x 512 x 256 FP32 2108 against 1999.
template <typename T>
bool ch_fft_fits(const Dims& f, const StepConsts& k) {
  const bool moving = k.uwb[0] != 0.0 || k.uwb[1] != 0.0 || k.uwt[0] != 0.0 || k.uwt[1] != 0.0;
  const int row = f.nx / (16 / (int)sizeof(T));  // threads of a row
  return f.nx >= 16 && f.nx <= 1024 && row <= (f.ny > 1 ? 256 : 512) && f.cells() * sizeof(T) < ((size_t)1 << 32) &&
         !(moving && k.relax_kappa != 0.0);
}

template <typename T>
hipError_t launch_ch_fft(const Dims& f, const Dims& c, const StepConsts& k, const Tables<T>& tb, ChIn<T> in,
                         cx<T>* spec, hipStream_t st) {
  if (!ch_fft_fits<T>(f, k)) return hipErrorInvalidConfiguration;
  const int single = f.nx == c.nx ? 1 : 0;  // the phase field on the flow grid
  Prolonged<T> pv{in.un, in.unm1, in.vn, in.vnm1, in.wn, in.wnm1, c.nx, c.ny, c.nz,
                  (c.ny == 1 || single) ? 1 : 2, k.first, single};
  constexpr int CPT = 16 / sizeof(T);
  const int row = f.nx / CPT;  // threads of a row
  int TY = 1;
  if (f.ny > 1) {
    TY = 512 / row;
    TY = TY < 2 ? 2 : (TY > 8 ? 8 : TY);
    if (TY > f.ny) TY = f.ny;
  }
  const int nth = TY * row;
  const int mode = in.adv ? 2 : (single ? 1 : 0);
  const bool relax = k.relax_kappa != 0.0;
  const int M = f.nx / 2, rows = f.ny > 1 ? TY + 2 : 1;
  auto go = [&](auto kernel, int ls) {
    auto lds = [&](int NB) {
      return (size_t)(relax ? 3 : 2) * rows * f.nx * sizeof(T) + ((size_t)NB * TY * ls + M) * sizeof(cx<T>);
    };
    // layers per block: one round of resident blocks, at least one block per CU while there are
    // layers; NB = 4 layers give every thread its points of the transform
    const int cols = f.ny / TY;
    int KB = march_layers(kernel, nth, lds(4), cols, f.nz);
    int p = 1;
    while (p < KB) p <<= 1;
    KB = p;
    const int NB = KB < 4 ? KB : 4;
    hipLaunchKernelGGL(kernel, dim3(cols * (f.nz / KB)), dim3(nth), lds(NB), st, in.phin, in.phinm1, pv, spec, in.adv,
                       f.ny, f.nz, f.logx - 1, TY, KB, NB, (T)f.ihx, (T)f.ihy, (T)f.ihz, tb.tw_xm, tb.tw_xn, k);
  };
  auto pick = [&](auto L, int ls) {
    constexpr int LOGM = decltype(L)::value;
#define DRPF_CHF(MODE, RELAX)                                \
  if (f.ny > 1) go(k_ch_fft<T, LOGM, MODE, RELAX, true>, ls); \
  else go(k_ch_fft<T, LOGM, MODE, RELAX, false>, ls)
    if (relax) {
      if (mode == 2) { DRPF_CHF(2, true); } else if (mode == 1) { DRPF_CHF(1, true); } else { DRPF_CHF(0, true); }
    } else {
      if (mode == 2) { DRPF_CHF(2, false); } else if (mode == 1) { DRPF_CHF(1, false); } else { DRPF_CHF(0, false); }
    }
#undef DRPF_CHF
  };
  if constexpr (sizeof(T) == 8) {
    pick(std::integral_constant<int, 0>{}, M);
  } else {
    switch (f.logx - 1) {
#define DRPF_L(N) case N: pick(std::integral_constant<int, N>{}, FftPlan<N, 3>::LS); break
      DRPF_L(3); DRPF_L(4); DRPF_L(5); DRPF_L(6); DRPF_L(7); DRPF_L(8); DRPF_L(9);
#undef DRPF_L
      default: return hipErrorInvalidConfiguration;
    }
  }
  return hipGetLastError();
}

#define INST(T)                                                                                               \
  template bool ch_fft_fits<T>(const Dims&, const StepConsts&);                                               \
  template hipError_t launch_ch_fft<T>(const Dims&, const Dims&, const StepConsts&, const Tables<T>&, ChIn<T>, \
                                       cx<T>*, hipStream_t);
INST(double)
INST(float)
#undef INST

}  // namespace drpf
