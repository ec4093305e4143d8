// batch.h -- many independent D2Q9 simulations stepped together.
//
// Every phase of the step runs as one launch over all members: the grid
// walks a queue of work items (a membrane, an active tile, a marker, a
// (strip, segment) of a lattice) spread over the members, finds the member
// of each item by binary search over prefix sums, and runs the same device
// code the single-simulation kernels run.  The lattice kernel has one (strip,
// segment) item per wave, and one launch for all members, whether they relax
// (some tau not 1) or not.  All members advance with the same buffer parity and hold the
// same form of the state (populations, or Macro2 between the steps of a call).
#pragma once
#include "common.h"
#include "k_ibm.h"
#include "k_lb.h"

namespace lb {

constexpr int BATCH_MAX = 256;  // members per batch

template <class St, typename R>
struct BMember {
  LBParams P;     // segments for the member's size class
  int relax;      // some relaxation time differs from 1
  int nstrip[2];  // strips when the step reads populations, and when it reads Macro2
  St a, b;        // population buffers (parity 0 reads a, writes b)
  MacroStore2<R> ma, mb;  // the same memory between the steps of a call
  MemDev md;
  TileMap tm;
  CoupArgs ca;
  double* Ifield;
  long long* fib;
  double* force;
};

// The member descriptors live in global memory; every kernel copies the one
// it works on into registers first, so the stores of the step cannot be
// taken to alias it (which would force a reload after each store).

// the buffer a step reads (or, dst, writes) at a parity, in the form MACRO
template <bool MACRO, class St, typename R>
__device__ __forceinline__ auto batch_buffer(const BMember<St, R>& t, bool second) {
  if constexpr (MACRO)
    return second ? t.mb : t.ma;
  else
    return second ? t.b : t.a;
}

// index i in [0, n) with pre[i] <= v < pre[i + 1]
__device__ __forceinline__ int prefix_find(const int* pre, int n, int v) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (pre[mid] <= v)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

template <class St, typename R>
__global__ void kb_begin(BMember<St, R>* T, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    int* ts = T[i].tm.tstate;
    ts[0] = 0;
    ts[1] = ts[1] + 1;
  }
}

// one workgroup per (member, membrane)
template <class St, typename R, int NT>
__global__ __launch_bounds__(NT) void kb_tiles(const BMember<St, R>* T, const int2* mems) {
  const int2 e = mems[blockIdx.x];
  const MemDev md = T[e.x].md;
  const TileMap tm = T[e.x].tm;
  const LBParams P = T[e.x].P;
  const double rc = T[e.x].ca.r_cut;
  tiles_run<NT>(md, tm, P.nx, P.ny, 1, P.wall_y, 0, 2, map_reach(rc), e.y, tm.tstate[1], tm.tstate);
}

// persistent: the active tiles of all members
template <class St, typename R, int NT, bool MACRO>
__global__ __launch_bounds__(NT, 2) void kb_coupling2d(const BMember<St, R>* T, int n, int parity) {
  __shared__ int s_pre[BATCH_MAX + 1];
  for (int i = threadIdx.x; i < n; i += NT) s_pre[i + 1] = T[i].tm.tstate[0];
  if (threadIdx.x == 0) s_pre[0] = 0;
  __syncthreads();
  if (threadIdx.x == 0)
    for (int i = 0; i < n; i++) s_pre[i + 1] += s_pre[i];
  __syncthreads();
  const int total = s_pre[n];
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int i = prefix_find(s_pre, n, item);
    const MemDev md = T[i].md;
    const TileMap tm = T[i].tm;
    const CoupArgs ca = T[i].ca;
    double* Ifield = T[i].Ifield;
    const auto cur = batch_buffer<MACRO>(T[i], parity != 0);
    coupling2d_tile<decltype(cur), R, NT>(md, tm, ca, Ifield, cur, item - s_pre[i]);
  }
}

// markers of all members (mpre: marker prefix, n + 1 entries)
template <class St, typename R>
__global__ void kb_forcespread2d(const BMember<St, R>* T, const int* __restrict__ mpre, int n) {
  const int tid = blockIdx.x * blockDim.x + threadIdx.x;
  const int gf = tid >> 4, k = tid & 15;
  const bool live = gf < mpre[n];
  const int i = live ? prefix_find(mpre, n, gf) : 0;
  const MemDev md = T[i].md;
  long long* fib = T[i].fib;
  const int nx = T[i].P.nx, ny = T[i].P.ny, wy = T[i].P.wall_y;
  forcespread2d_run(md, fib, nx, ny, wy, live ? gf - mpre[i] : 0, k, live);
}

template <class St, typename R, bool MACRO>
__global__ void kb_interp2d(const BMember<St, R>* T, const int* __restrict__ mpre, int n, int parity) {
  const int tid = blockIdx.x * blockDim.x + threadIdx.x;
  const int gf = tid >> 4, k = tid & 15;
  const bool live = gf < mpre[n];
  const int i = live ? prefix_find(mpre, n, gf) : 0;
  const MemDev md = T[i].md;
  const LBParams P = T[i].P;
  const double* force = T[i].force;
  // after the lattice update the current state is in the buffer written
  const auto cur = batch_buffer<MACRO>(T[i], parity == 0);
  interp2d_run<decltype(cur), R>(md, cur, P, force, live ? gf - mpre[i] : 0, k, live);
}

// kinds of batches: no member relaxes, all do, or some
enum { KIND_EQ = 0, KIND_RELAX = 1, KIND_MIXED = 2 };

// one wave per (strip, segment) item of the members (bpre: item prefix, n + 1
// entries); NW as in k_lb2d.  A mixed batch takes one launch too, each wave
// branching on its member: with a launch per kind a step of 15 members of 240 x
// 120, five of which relax, took 120 us instead of 108.
template <class St, typename R, int FORM, bool SM, bool DM, int KIND, int NW>
__global__ __launch_bounds__(64 * NW, step2d_waves<R>()) void kb_lb2d(const BMember<St, R>* T,
                                                                      const int* __restrict__ bpre, int n,
                                                                      int parity) {
  // items dealt to the eight XCDs in contiguous runs, so the neighbouring
  // segments of a member share their halo rows in one L2
  int item = dealt_index((int)blockIdx.x, (int)gridDim.x, 8) * NW;
  if constexpr (NW > 1) {
    item += __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (item >= bpre[n]) return;
  }
  const int i = prefix_find(bpre, n, item);
  const LBParams P = T[i].P;
  const auto src = batch_buffer<SM>(T[i], parity != 0);
  const auto dst = batch_buffer<DM>(T[i], parity == 0);
  const int* tflag = T[i].tm.tflag;
  const int* tstate = T[i].tm.tstate;
  const double* Ifield = T[i].Ifield;
  long long* fib = T[i].fib;
  double* force = T[i].force;
  int strip, sgm;
  strip_segment(item - bpre[i], T[i].nstrip[SM], P.nseg, 1, strip, sgm);
  const int y0 = sgm * P.seg, y1 = min(y0 + P.seg, P.ny);
  auto run = [&](auto relax) {
    step2d_run<St, R, FORM, decltype(src), decltype(dst), decltype(relax)::value, (NW > 1)>(
        src, dst, P, strip, y0, y1, tflag, tstate, Ifield, fib, force);
  };
  if constexpr (KIND == KIND_MIXED) {
    if (T[i].relax)
      run(std::true_type{});
    else
      run(std::false_type{});
  } else {
    run(std::integral_constant<bool, KIND == KIND_RELAX>{});
  }
}

}  // namespace lb
