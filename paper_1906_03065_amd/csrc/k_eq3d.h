// k_eq3d.h -- the lattice-Boltzmann step on D3Q19 when every relaxation time is 1.
//
// A collision then leaves equilibria, so a node's 57 populations are functions
// of 11 numbers (Macro3), and the steps inside a call pass those on instead:
// 52 B per node in the mixed format against 228.  Two kernels per step:
//   k_mom3d_eq  streams: the moments drho, j, phi, psi of every node from the
//               equilibria of its neighbours, to a moment field (32 B);
//   k_lb3d_eq   the chemical potentials, the force and the collision from the
//               moment field alone, to Macro3 or (a call's last step) to
//               populations.
// A call's first step takes its moments from the populations (k_mom3d_pull).  Every
// value that decides a result is formed by the same operations on both routes
// (explicit fma, contraction off), so a call's division into steps leaves the
// bits alone.
//
// 256^3 with two capsules, moments + update per step: 843 + 2245 us with
// populations between all steps; now 622 (k_mom3d_eq) + 583 (k_lb3d_eq), in a
// call's first step 877 + 583, in its last 622 + 1325.  64^3: 12 + 63 before, 22 +
// 25 now.
#pragma once
#include "common.h"
#include "k_lb.h"
#include "k_lb3d.h"
#include "store.h"

namespace lb {

// Macro2 in three dimensions
template <typename R>
struct Macro3 {
  R dr, w[3], v[3], gm, hm;
  double phi, psi;
};

// c_i . (x, y, z)
template <typename R>
__device__ __forceinline__ R along19(int i, R x, R y, R z) {
#pragma clang fp contract(off)
  using L = Lattice<19>;
  const R sx = L::cx[i] < 0 ? -x : x, sy = L::cy[i] < 0 ? -y : y, sz = L::cz[i] < 0 ? -z : z;
  if (L::cx[i] == 0 && L::cy[i] == 0) return sz;
  if (L::cx[i] == 0) return L::cz[i] == 0 ? sy : sy + sz;
  if (L::cy[i] == 0) return L::cz[i] == 0 ? sx : sx + sz;
  return sx + sy;
}

template <typename R>
__device__ __forceinline__ R speed19(const R* c) {
#pragma clang fp contract(off)
  return R(-1.5) * fma_(c[0], c[0], fma_(c[1], c[1], c[2] * c[2]));
}

// The equilibria at velocity c, q = speed19(c).  Set f (eq. EDF, as deviations
// from w_i rho0): from rr = rho, drs = drho + sp; sets g, h: from the order
// parameter times the weight (a) and 3 Gamma mu times the weight (b).  Population
// i and its opposite share base: the odd one has the positive direction.
template <typename R>
__device__ __forceinline__ R eq19_f(int i, R rr, R drs, R q, const R* c) {
#pragma clang fp contract(off)
  const R cu = along19(i, c[0], c[1], c[2]);
  return R(Lattice<19>::w(i)) * fma_(rr, fma_(R(3), cu, fma_(R(4.5) * cu, cu, q)), drs);
}
template <typename R>
__device__ __forceinline__ R eq19_f0(R rr, R dr, R sp, R q) {
#pragma clang fp contract(off)
  using L = Lattice<19>;
  return fma_(R(L::w(0)), fma_(rr, q, dr), -(R(1.0 - L::w(0)) * sp));
}
template <typename R>
__device__ __forceinline__ R eq19_g(int i, R ph, R gm, R q, const R* c) {
#pragma clang fp contract(off)
  const R cu = along19(i, c[0], c[1], c[2]), w = R(Lattice<19>::w(i)), a = ph * w;
  return fma_(R(3) * a, cu, fma_(a, fma_(R(4.5) * cu, cu, q), gm * w));
}
// all moving populations of g (or h), and its rest population: the order
// parameter less what moves, so that the stored numbers sum to it
template <typename R>
__device__ __forceinline__ void eq19_gall(double phi, R gm, const R* c, R* g, double& g0) {
#pragma clang fp contract(off)
  using L = Lattice<19>;
  const R q = speed19(c), ph = (R)phi;
  const R a1 = ph * R(L::w(1)), a2 = ph * R(L::w(7)), b1 = gm * R(L::w(1)), b2 = gm * R(L::w(7));
  double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 1; i < 19; i += 2) {
    eq_pair(i < 7 ? a1 : a2, R(3) * (i < 7 ? a1 : a2), i < 7 ? b1 : b2, q, along19(i, c[0], c[1], c[2]), g[i], g[i + 1]);
    s[(i / 2) % 3] += (double)g[i] + (double)g[i + 1];
  }
  g0 = phi - ((s[0] + s[1]) + s[2]);
}

// the population buffers' other content: planes of dr, w, v, gm, hm in R, and of
// phi, psi in FP64, read and written through buffer resources as in MixStore
// (32-bit offsets, checked on the host)
template <typename R>
struct MacroStore3 {
  R* p;
  double* r;
  unsigned N;
  double rho0, p0, p1;  // p0, p1: LBParams::psh
  static constexpr bool kMacro = true, kQuantized = false;
  static constexpr int kR = 9;
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rp() const {
    return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)(kR * N * (unsigned)sizeof(R)), 0x00020000);
  }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rr() const {
    return __builtin_amdgcn_make_buffer_rsrc(r, 0, (int)(2 * N * 8u), 0x00020000);
  }
  __device__ __forceinline__ R get(int k, unsigned n) const {
    if constexpr (sizeof(R) == 4)
      return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b32(rp(), (int)(n * 4), (int)(k * N * 4), 0));
    else
      return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b64(rp(), (int)(n * 8), (int)(k * N * 8), 0));
  }
  __device__ __forceinline__ double getd(int k, unsigned n) const {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rr(), (int)(n * 8), (int)(k * N * 8), 0));
  }
  __device__ __forceinline__ void put(int k, unsigned n, R v) const {
    if constexpr (sizeof(R) == 4)
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rp(), (int)(n * 4), (int)(k * N * 4), 0);
    else
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rp(), (int)(n * 8), (int)(k * N * 8), 0);
  }
  __device__ __forceinline__ Macro3<R> node(unsigned n) const {
    return Macro3<R>{get(0, n), {get(1, n), get(2, n), get(3, n)}, {get(4, n), get(5, n), get(6, n)},
                     get(7, n), get(8, n), getd(0, n), getd(1, n)};
  }
  __device__ __forceinline__ void set_node(unsigned n, const Macro3<R>& s) const {
    put(0, n, s.dr);
#pragma unroll
    for (int a = 0; a < 3; a++) {
      put(1 + a, n, s.w[a]);
      put(4 + a, n, s.v[a]);
    }
    put(7, n, s.gm);
    put(8, n, s.hm);
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, s.phi), rr(), (int)(n * 8), 0, 0);
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, s.psi), rr(), (int)(n * 8), (int)(N * 8), 0);
  }
  __device__ __forceinline__ R shift(unsigned n) const {
    return p0 != 0.0 || p1 != 0.0 ? eq_shift<R>(p0, p1, getd(0, n), getd(1, n)) : R(0);
  }
  // single populations, for the kernels that read a few nodes
  template <typename T>
  __device__ __forceinline__ T pull(int set, int i, bool flip, long long nd) const {
#pragma clang fp contract(off)
    const unsigned n = (unsigned)nd;
    const int o = set == 0 ? 1 : 4;
    R c[3] = {get(o, n), get(o + 1, n), get(o + 2, n)};
    const R q = speed19(c);
#pragma unroll
    for (int a = 0; a < 3; a++) c[a] = flip ? -c[a] : c[a];
    if (set == 0) {
      const R dr = get(0, n), sp = shift(n), rr = (R)rho0 + dr;
      return (T)(i == 0 ? eq19_f0(rr, dr, sp, q) : eq19_f(i, rr, dr + sp, q, c));
    }
    return (T)eq19_g(i, (R)getd(set - 1, n), get(6 + set, n), q, c);
  }
  template <typename T>
  __device__ __forceinline__ T load(int set, int i, long long nd) const {
    return pull<T>(set, i, false, nd);
  }
  __device__ __forceinline__ double rest(int set, long long nd) const {
    if (set == 0) return (double)pull<R>(0, 0, false, nd);
    const unsigned n = (unsigned)nd;
    const R c[3] = {get(4, n), get(5, n), get(6, n)};
    R g[19];
    double g0;
    eq19_gall(getd(set - 1, n), get(6 + set, n), c, g, g0);
    return g0;
  }
};

// The moment sums of one node, in shares of the rows its populations come from:
// its own (directions with c_y = 0) and those below and above.
template <typename R>
struct Share19 {
  R d, jx, jz, g, h;
};
template <typename R>
__device__ __forceinline__ R own19(const R* p) {
#pragma clang fp contract(off)
  return (p[5] + p[6]) + ((p[1] + (p[11] + p[13])) + (p[2] + (p[12] + p[14])));
}
template <bool UP, typename R>
__device__ __forceinline__ R side19(const R* p) {
#pragma clang fp contract(off)
  constexpr int a = UP ? 3 : 4, e = UP ? 7 : 9, w = UP ? 10 : 8, t = UP ? 15 : 18, b = UP ? 17 : 16;
  return p[a] + ((p[e] + p[w]) + (p[t] + p[b]));
}
// the shares of f: from the own row, from below, from above
template <typename R>
__device__ __forceinline__ void shares19_f(const R* f, Share19<R>& o, Share19<R>& b, Share19<R>& a) {
#pragma clang fp contract(off)
  const R e = f[1] + (f[11] + f[13]), w = f[2] + (f[12] + f[14]);
  o.d = f[0] + ((f[5] + f[6]) + (e + w));
  o.jx = e - w;
  o.jz = (f[5] - f[6]) + ((f[11] - f[13]) + (f[14] - f[12]));
  b.d = side19<true>(f);
  b.jx = f[7] - f[10];
  b.jz = f[15] - f[17];
  a.d = side19<false>(f);
  a.jx = f[9] - f[8];
  a.jz = f[18] - f[16];
}
template <typename R>
__device__ __forceinline__ void put_moments19(const Moments3<R>& M, long long n, const Share19<R>& o,
                                              const Share19<R>& b, const Share19<R>& a, double g0, double h0) {
#pragma clang fp contract(off)
  M.d[n] = o.d + (b.d + a.d);
  M.jx[n] = o.jx + (b.jx + a.jx);
  M.jy[n] = b.d - a.d;
  M.jz[n] = o.jz + (b.jz + a.jz);
  M.phi[n] = g0 + (double)(o.g + (b.g + a.g));
  M.psi[n] = h0 + (double)(o.h + (b.h + a.h));
}

// the moments node by node: from populations (all nodes), or from Macro3 at the
// nodes next to a wall (BORDER), whose populations bounce back
template <class Src, typename R, bool BORDER>
__global__ __launch_bounds__(256) void k_mom3d_pull(Src src, LBParams P, Moments3<R> M, long long count) {
  long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= count) return;
  const int x = (int)(n % P.nx);
  int y, z;
  if constexpr (BORDER) {
    // the planes next to walls in z, then the rows next to walls in y of the others
    const int zb = P.wall_z ? min(P.nz, 2) : 0, yb = P.wall_y ? min(P.ny, 2) : 0;
    long long r = n / P.nx;
    if (r < (long long)zb * P.ny) {
      y = (int)(r % P.ny);
      z = r < P.ny ? 0 : P.nz - 1;
    } else {
      r -= (long long)zb * P.ny;
      y = (int)(r % yb) ? P.ny - 1 : 0;
      z = (int)(r / yb) + (P.wall_z ? 1 : 0);
    }
    n = ((long long)z * P.ny + y) * P.nx + x;
  } else {
    y = (int)((n / P.nx) % P.ny);
    z = (int)(n / ((long long)P.nx * P.ny));
  }
  R pf[19], pg[19], ph[19];
  double g0, h0;
  pull19(src, P, x, y, z, pf, pg, ph, g0, h0);
  Share19<R> o, b, a;
  shares19_f(pf, o, b, a);
  o.g = own19(pg);
  b.g = side19<true>(pg);
  a.g = side19<false>(pg);
  o.h = own19(ph);
  b.h = side19<true>(ph);
  a.h = side19<false>(ph);
  put_moments19(M, n, o, b, a, g0, h0);
}

// The moments of the nodes away from walls, from Macro3.  A wave of its own owns
// one z plane of a strip in x (one halo lane either side) and marches along y:
// per row it forms the populations that its own row and the rows of the planes
// below and above send, moves them one lane in x, and adds them to the three
// rows that receive them.
//
// What bounds it: VALU issue (some 480 operations per node, each population
// formed once; half of the issue slots at 256^3, with five strips of 52 in 64
// lanes) and memory (84 B per node if every plane were read once).  The next row
// is fetched while one is summed.  The rows of the neighbour planes come out of a
// cache as long as the waves of neighbouring planes keep to the same row: a
// workgroup is four waves of consecutive planes with a barrier per row.  At 256^3
// one wave per workgroup reads 2.8 GB and takes 656 us, four 1.9 GB and 620 us,
// six 1.7 GB and 842 us (they wait for each other, and 12 waves fit a CU).
// Registers: 144, three waves per SIMD; held to 128 for four, 12 of them spill
// and it takes 1152 us.
constexpr int MOM3_WAVES = 4;
template <typename R>
__global__ __launch_bounds__(64 * MOM3_WAVES, sizeof(R) == 4 ? 3 : 2) void k_mom3d_eq(
    MacroStore3<R> src, LBParams P, Moments3<R> M, int width, int nstrip, int seg, int nseg) {
#pragma clang fp contract(off)
  using L = Lattice<19>;
  const int nzg = (P.nz + MOM3_WAVES - 1) / MOM3_WAVES;
  const int l = dealt_index((int)blockIdx.x, nzg * nstrip * nseg, P.nxcd);
  const int zw = (l % nzg) * MOM3_WAVES + (int)(threadIdx.x >> 6), strip = (l / nzg) % nstrip, sg = l / (nzg * nstrip);
  // (a wave past the last plane, or at a wall, goes along with its workgroup)
  const int z = min(zw, P.nz - 1);
  const bool out = zw < P.nz && !(P.wall_z && (z == 0 || z == P.nz - 1));
  const int j = threadIdx.x & 63, xc = strip * width - 1 + j;
  const int x = wrap(xc, P.nx);
  const bool mine = out && j >= 1 && j <= width && xc < P.nx;
  const int y0 = sg * seg, y1 = min(y0 + seg, P.ny);
  const int zs[3] = {z == 0 ? P.nz - 1 : z - 1, z, z == P.nz - 1 ? 0 : z + 1};
  const R rho0 = (R)src.rho0;
  const R w1 = R(L::w(1)), w2 = R(L::w(7));
  auto shift = [&](const Macro3<R>& t) {
    return src.p0 != 0.0 || src.p1 != 0.0 ? eq_shift<R>(src.p0, src.p1, t.phi, t.psi) : R(0);
  };
  Macro3<R> nxt[3];
  auto fetch = [&](int r) {
    const int ry = P.wall_y ? min(max(r, 0), P.ny - 1) : wrap_near(r, P.ny);
#pragma unroll
    for (int a = 0; a < 3; a++) nxt[a] = src.node((unsigned)((zs[a] * P.ny + ry) * P.nx + x));
  };
  Share19<R> below = {}, sent = {}, own = {};
  double og = 0.0, oh = 0.0;
  fetch(y0 - 1);
  for (int r = y0 - 1; r <= y1; r++) {
    Macro3<R> s[3];
#pragma unroll
    for (int a = 0; a < 3; a++) s[a] = nxt[a];
    fetch(min(r + 1, y1));
    // waves of neighbouring planes keep to the same row, so that what they
    // share comes out of the cache
    __builtin_amdgcn_s_barrier();
    // one set after the other, each moved in x and summed before the next
    Share19<R> o, up, dn;
    double g0, h0;
    R p[19];
    auto moved = [&]() {
#pragma unroll
      for (int i = 1; i < 19; i++) p[i] = L::cx[i] > 0 ? west(p[i]) : (L::cx[i] < 0 ? east(p[i]) : p[i]);
    };
    {
      const Macro3<R>& t = s[1];
      const R sp = shift(t), rr = rho0 + t.dr, drs = t.dr + sp, q = speed19(t.w);
      p[0] = eq19_f0(rr, t.dr, sp, q);
#pragma unroll
      for (int i = 1; i < 11; i += 2)
        if (L::cz[i] == 0) eq_pair_f(R(L::w(i)), rr, drs, q, along19(i, t.w[0], t.w[1], t.w[2]), p[i], p[i + 1]);
    }
#pragma unroll
    for (int a = 0; a < 3; a += 2) {  // the planes below (c_z = 1) and above (c_z = -1)
      const Macro3<R>& t = s[a];
      const R rr = rho0 + t.dr, drs = t.dr + shift(t), q = speed19(t.w);
#pragma unroll
      for (int i = 1; i < 19; i++)
        if (L::cz[i] == 1 - a) p[i] = eq19_f(i, rr, drs, q, t.w);
    }
    moved();
    shares19_f(p, o, up, dn);
    // (each set's shares are formed before the next set is begun)
    asm volatile("" : "+v"(o.d), "+v"(o.jx), "+v"(o.jz), "+v"(up.d), "+v"(up.jx), "+v"(up.jz), "+v"(dn.d), "+v"(dn.jx),
                 "+v"(dn.jz));
    __builtin_amdgcn_sched_barrier(0);
    auto order = [&](auto set_c, R& own_, R& up_, R& dn_, double& rest) {
      constexpr int S = decltype(set_c)::value;
      eq19_gall(S == 1 ? s[1].phi : s[1].psi, S == 1 ? s[1].gm : s[1].hm, s[1].v, p, rest);
#pragma unroll
      for (int a = 0; a < 3; a += 2) {
        const Macro3<R>& t = s[a];
        const R q = speed19(t.v), ph = (R)(S == 1 ? t.phi : t.psi), gm = S == 1 ? t.gm : t.hm;
        const R p1 = ph * w1, p2 = ph * w2, b1 = gm * w1, b2 = gm * w2;
#pragma unroll
        for (int i = 1; i < 19; i++)
          if (L::cz[i] == 1 - a) {
            const R cu = along19(i, t.v[0], t.v[1], t.v[2]), ai = i < 7 ? p1 : p2;
            p[i] = fma_(R(3) * ai, cu, fma_(ai, fma_(R(4.5) * cu, cu, q), i < 7 ? b1 : b2));
          }
      }
      moved();
      own_ = own19(p);
      up_ = side19<true>(p);
      dn_ = side19<false>(p);
      asm volatile("" : "+v"(own_), "+v"(up_), "+v"(dn_), "+v"(rest));
      __builtin_amdgcn_sched_barrier(0);
    };
    order(std::integral_constant<int, 1>{}, o.g, up.g, dn.g, g0);
    order(std::integral_constant<int, 2>{}, o.h, up.h, dn.h, h0);
    const int rr = r - 1;  // the row whose shares are complete
    if (rr >= y0 && mine && !(P.wall_y && (rr == 0 || rr == P.ny - 1)))
      put_moments19(M, ((long long)z * P.ny + rr) * P.nx + x, own, below, dn, og, oh);
    below = sent;
    sent = up;
    own = o;
    og = g0;
    oh = h0;
  }
}

// a node's populations, to the store dst
template <class Dst, typename R>
__device__ __forceinline__ void put_pops19(const Dst& dst, R rho0, double p0, double p1, const Macro3<R>& o,
                                           long long node) {
#pragma clang fp contract(off)
  const R sp = p0 != 0.0 || p1 != 0.0 ? eq_shift<R>(p0, p1, o.phi, o.psi) : R(0);
  const R rr = rho0 + o.dr, drs = o.dr + sp, q = speed19(o.w);
  dst.template store<R>(0, 0, node, eq19_f0(rr, o.dr, sp, q));
  R f[19];
#pragma unroll
  for (int i = 1; i < 19; i += 2) {
    eq_pair_f(R(Lattice<19>::w(i)), rr, drs, q, along19(i, o.w[0], o.w[1], o.w[2]), f[i], f[i + 1]);
    dst.template store<R>(0, i, node, f[i]);
    dst.template store<R>(0, i + 1, node, f[i + 1]);
    __builtin_amdgcn_sched_barrier(0);
  }
  double g0;
#pragma unroll
  for (int set = 1; set < 3; set++) {
    __builtin_amdgcn_sched_barrier(0);
    eq19_gall(set == 1 ? o.phi : o.psi, set == 1 ? o.gm : o.hm, o.v, f, g0);
    dst.store_rest(set, node, g0);
#pragma unroll
    for (int i = 1; i < 19; i++) dst.template store<R>(set, i, node, f[i]);
  }
}

// the populations of the state that Macro3 holds (a call that fails between two
// steps leaves populations, as every call does)
template <class St, typename R>
__global__ __launch_bounds__(256) void k_expand3d(MacroStore3<R> src, St dst) {
  const unsigned n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n < src.N) put_pops19(dst, (R)src.rho0, src.p0, src.p1, src.node(n), (long long)n);
}

// The chemical potentials, the force (eqs. ForcingTermLBE, ForceFE + the spread
// membrane force) and the collision, from the moment field.  A workgroup owns a
// TX x TY column of nodes and marches along z; one thread per node of the
// (TX+2) x (TY+2) region where the potentials are formed (the two columns beside
// the tile in a wave of their own).  Per plane the concentrations of the
// (TX+4) x (TY+4) region are staged in LDS, and each thread sums its node's
// in-plane neighbours once: the 3D stencils are put together from the sums of
// three successive planes, kept in registers (9 and 8 LDS reads per plane, field
// and stencil instead of 18).  The potentials of plane k - 2, the sums of plane k
// and the collision of plane k - 3 share an iteration and one barrier.
//
// What bounds it: memory (1.0 GB read, 1.0 GB written at 256^3, 416 us at the rate
// of a copy) and the barrier, with one workgroup per CU at the wide tile (11 waves
// at 168 registers, 8 of which spill, 22 to populations; FP64 14 and 62): 583 us,
// to populations 1325 us (0.9 + 4.2 GB).  The narrow tile gives a small lattice's
// CUs a workgroup each and spills nothing: see EQ3_WIDE.
template <class Dst, typename R, int TX, int TY>
__global__ __launch_bounds__((TX * (TY + 2) + 2 * (TY + 2) + 63) / 64 * 64) void k_lb3d_eq(
    Dst dst, LBParams P, Moments3<R> M, const int* __restrict__ tflag, const int* __restrict__ tstate,
    const double* __restrict__ Ifield, long long* __restrict__ fib, double* __restrict__ force, int ntilex) {
#pragma clang fp contract(off)
  constexpr int TXH = TX + 4, TYH = TY + 4, TXU = TX + 2, TYU = TY + 2;
  constexpr int NT = (TX * TYU + 2 * TYU + 63) / 64 * 64, NH = (TXH * TYH + NT - 1) / NT;
  __shared__ double s_m[2][3][TXH * TYH];  // concentrations
  __shared__ double s_u[2][3][TXU * TYU];  // potentials mu_rho, mu_phi, mu_psi
  const int tid = threadIdx.x;
  int tl, sgm;
  strip_segment((int)(blockIdx.y * gridDim.x + blockIdx.x), (int)gridDim.x, (int)gridDim.y, P.nxcd, tl, sgm);
  const int x0 = (tl % ntilex) * TX, y0 = (tl / ntilex) * TY;
  const int z0 = sgm * P.seg, z1 = min(z0 + P.seg, P.nz);
  const int K = (z1 - z0) + 4;
  const int zbase = z0 - 2;
  const int stamp = tstate[1];
  // this thread's node of the potentials' region
  const int e = tid - TX * TYU;
  const bool live = e < 2 * TYU;
  const int ux = e < 0 ? tid % TX + 1 : (e & 1) * (TXU - 1);
  const int uy = e < 0 ? tid / TX : min(e >> 1, TYU - 1);
  const int gx = x0 - 1 + ux, gy = y0 - 1 + uy;
  const int xw = wrap(gx, P.nx), yw = halo_row(gy, P.ny, P.wall_y);
  const bool own = e < 0 && uy >= 1 && uy <= TY && gx < P.nx && gy < P.ny;
  const int hq = (uy + 1) * TXH + ux + 1, uq = uy * TXU + ux;
  const double km[3] = {P.k1, P.k2, P.k3};
  // offsets in a plane of the staged nodes
  unsigned hoff[NH];
#pragma unroll
  for (int r = 0; r < NH; r++) {
    const int q = min(tid + NT * r, TXH * TYH - 1);
    hoff[r] = (unsigned)(halo_row(y0 - 2 + q / TXH, P.ny, P.wall_y) * P.nx + wrap(x0 - 2 + q % TXH, P.nx));
  }
  const unsigned here = (unsigned)(yw * P.nx + xw);
  const long long plane = (long long)P.ny * P.nx;

  // in flight: the staged moments of the next plane, the profile field of the
  // next potentials, the moments of the next collision
  R nd[NH];
  double nphi[NH], npsi[NH];
  double Inx = 0.0, cphi = 0.0;
  R cd = 0, cjx = 0, cjy = 0, cjz = 0;
  int fl0 = 0, fl1 = 0;  // tile flags of this node in the last plane and the one before
  bool cact = false;
  // sums of the last planes: concentrations c and their in-plane differences
  double c1[3] = {}, s1[3] = {}, acc[3] = {}, lap[3] = {};
  double q2[3] = {};                    // c of the plane of the next potentials
  double psi3 = 0.0;                    // psi of the plane before it
  // sums of the last planes' potentials
  double ax[3] = {}, px[3] = {}, ay[3] = {}, py[3] = {}, t1[3] = {}, t2[3] = {};

  auto stage = [&](int k) {
    const long long zr = (long long)halo_row(zbase + k, P.nz, P.wall_z) * plane;
#pragma unroll
    for (int r = 0; r < NH; r++) {
      nd[r] = (M.d + zr)[hoff[r]];
      nphi[r] = (M.phi + zr)[hoff[r]];
      npsi[r] = (M.psi + zr)[hoff[r]];
    }
  };
  stage(0);
#pragma unroll 1
  for (int k = 0; k <= K; k++) {
    const int b = k & 1;
    // ---- the concentrations of plane k, and the potentials of plane k - 2
#pragma unroll
    for (int r = 0; r < NH; r++) {
      const int q = tid + NT * r;
      const double rho = P.rho0 + (double)nd[r];
      if (q < TXH * TYH) {
        s_m[b][0][q] = fma_(P.cm[0][0], rho, fma_(P.cm[0][1], nphi[r], P.cm[0][2] * npsi[r]));
        s_m[b][1][q] = fma_(P.cm[1][0], rho, fma_(P.cm[1][1], nphi[r], P.cm[1][2] * npsi[r]));
        s_m[b][2][q] = npsi[r];
      }
    }
    {
      double bb[3];
#pragma unroll
      for (int f = 0; f < 3; f++) {
        const double C = q2[f];
        bb[f] = km[f] * fma_(-P.a2, lap[f], (C * (1.0 - C)) * fma_(-2.0, C, 1.0));
      }
      const double mr = fma_(P.cm[0][0], bb[0], P.cm[1][0] * bb[1]);
      const double mp = fma_(P.cm[0][1], bb[0], P.cm[1][1] * bb[1]);
      const double ms = fma_(P.cm[0][2], bb[0], P.cm[1][2] * bb[1]) + fma_(P.kc, q2[2] - Inx, bb[2]);
      if (live) {
        s_u[b][0][uq] = mr;
        s_u[b][1][uq] = mp;
        s_u[b][2][uq] = ms;
      }
    }
    const R d = cd, jx = cjx, jy = cjy, jz = cjz;
    const double phi = cphi, psi = psi3;
    const bool act = cact;
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    // ---- loads of the next iteration
    {
      const long long zi = (long long)halo_row(zbase + k - 1, P.nz, P.wall_z) * plane;
      Inx = 0.0;
      if (k >= 2 && live && fl0 == stamp) Inx = (Ifield + zi)[here];
      const int cz = min(max(zbase + k - 2, 0), P.nz - 1);
      const long long cn = cz * plane;
      cact = own && k >= 4 && k < K && fl1 == stamp;
      const int zf = halo_row(zbase + k, P.nz, P.wall_z);
      fl1 = fl0;
      fl0 = tflag[tile3(P, xw, yw, zf)];
      cd = (M.d + cn)[here];
      cjx = (M.jx + cn)[here];
      cjy = (M.jy + cn)[here];
      cjz = (M.jz + cn)[here];
      cphi = (M.phi + cn)[here];
      stage(min(k + 1, K - 1));
    }
    __builtin_amdgcn_sched_barrier(0);
    // ---- sums of plane k: the Laplacian of plane k - 1 (and, as the next
    // iteration's potentials are of that plane, what they need of it)
    psi3 = q2[2];
#pragma unroll
    for (int f = 0; f < 3; f++) {
      const double* m = s_m[b][f] + hq;
      const double c = m[0];
      const double s = ((m[1] - c) + (m[-1] - c)) + ((m[TXH] - c) + (m[-TXH] - c));
      const double o = ((m[TXH + 1] - c) + (m[TXH - 1] - c)) + ((m[-TXH + 1] - c) + (m[-TXH - 1] - c));
      const double dc = c - c1[f];
      // lap q = 6 sum_i w_i (q(x + c_i) - q(x)): 1/6 (2 s + o of the plane, s of
      // the planes below and above) + the differences to their centres
      lap[f] = fma_(1.0 / 6.0, s, acc[f] + dc);
      acc[f] = fma_(1.0 / 6.0, fma_(2.0, s, o) + s1[f], -dc);
      q2[f] = c1[f];
      c1[f] = c;
      s1[f] = s;
      // formed here, not where they are used: the nine values read would stay
      // in registers until then
      asm volatile("" : "+v"(lap[f]), "+v"(acc[f]), "+v"(s1[f]));
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- sums of the potentials of plane k - 2: the gradient of plane k - 3
    const double rho = P.rho0 + (double)d;
    double F[3];
#pragma unroll
    for (int f = 2; f >= 0; f--) {
      // (nodes at the region's rim sum what they do not use from within the array)
      const double* u = s_u[b][f] + (own ? uq : TXU + 1);
      const double E = u[1], W = u[-1], Nn = u[TXU], S = u[-TXU];
      const double ne = u[TXU + 1], nw = u[TXU - 1], se = u[-TXU + 1], sw = u[-TXU - 1];
      const double dx = E - W, dy = Nn - S;
      const double t = fma_(2.0, u[0], (E + W) + (Nn + S));
      const double gx = ax[f] + dx, gy = ay[f] + dy, gz = t - t2[f];
      F[0] = f == 2 ? psi * gx : fma_(f == 1 ? phi : rho, gx, F[0]);
      F[1] = f == 2 ? psi * gy : fma_(f == 1 ? phi : rho, gy, F[1]);
      F[2] = f == 2 ? psi * gz : fma_(f == 1 ? phi : rho, gz, F[2]);
      ax[f] = fma_(2.0, dx, (ne - nw) + (se - sw)) + px[f];
      ay[f] = fma_(2.0, dy, (ne - se) + (nw - sw)) + py[f];
      px[f] = dx;
      py[f] = dy;
      t2[f] = t1[f];
      t1[f] = t;
      asm volatile("" : "+v"(ax[f]), "+v"(ay[f]), "+v"(t1[f]), "+v"(F[0]), "+v"(F[1]), "+v"(F[2]));
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- the collision of plane k - 3
    if (k >= 5) {
      const int cz = zbase + k - 3;
      const long long node = cz * plane + here;
#pragma unroll
      for (int a = 0; a < 3; a++) F[a] = fma_(-1.0 / 12.0, F[a], P.fext[a]);
      if (act) {
        // (the spread force is loaded here, not ahead: only few planes have one,
        // and six registers more spill)
        long long* fp = fib + 3 * (cz * plane) + 3 * here;
        const long long fx = fp[0], fy = fp[1], fz = fp[2];
        F[0] += from_fix(fx);
        F[1] += from_fix(fy);
        F[2] += from_fix(fz);
#pragma unroll
        for (int a = 0; a < 3; a++) {
          fp[a] = 0;
          (force + 3 * (cz * plane))[3 * here + a] = F[a];
        }
      }
      const double ir = recip(rho);
      const double jd[3] = {(double)jx, (double)jy, (double)jz};
      Macro3<R> o;
      o.dr = d;
#pragma unroll
      for (int a = 0; a < 3; a++) {
        o.w[a] = (R)((jd[a] + F[a]) * ir);             // u + delta u, eq. VelCorrection
        o.v[a] = (R)(fma_(0.5, F[a], jd[a]) * ir);     // eq. ActualFluidVel
      }
      // (the thread's own potentials of the plane, which it alone overwrites)
      o.gm = (R)(3.0 * P.gphi * s_u[b ^ 1][1][uq]);
      o.hm = (R)(3.0 * P.gpsi * s_u[b ^ 1][2][uq]);
      o.phi = phi;
      o.psi = psi;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (Dst::kMacro) {
        dst.set_node(own ? (unsigned)node : 0xffffffffu, o);  // past the buffer: dropped
      } else if (own) {
        put_pops19(dst, (R)P.rho0, P.psh[0], P.psh[1], o, node);
      }
    }
  }
}

}  // namespace lb
