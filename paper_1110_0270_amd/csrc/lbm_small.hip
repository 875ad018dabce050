// Many time steps of a short D1Q3 lattice in one launch (LBGK, with the
// Ehrenfest and positivity limiters).
//
// The lattice (at most kSmallSites sites) lives in one workgroup's LDS from
// the first step to the last: pull, collision and the Ehrenfest selection are
// separated by barriers instead of kernel boundaries.  A step of such a
// lattice is latency only; as a step kernel and a selection kernel it took
// 18.6 us (800 sites, FP64), of which the arithmetic is a small part; here
// 3.0 us.  One compute unit does the work of the whole lattice, so longer
// lattices stay with the other kernels, which use them all.
//
// The site arithmetic is the step kernel's (the same functions, so the same
// bits), and the selection is exact as there: the k sites of largest
// Delta S > delta, ties to the lower index.  A candidate floor per step
// parity, kept so that 2k to 3.5k sites reach it, keeps the list short; a step
// whose floor turns out too high takes every eligible site again.  The state
// left behind (floors, frames, counts, the last step's list) is what the other
// selection kernels expect.
#include "lbm_collide.h"

namespace lbm {

constexpr int kSmallThreads = 1024;
// Lists of up to this many candidates are ranked by counting, longer ones by an
// MSD radix select.  800 sites FP64, us a step, counting -> radix: k = 8 (16 to
// 28 candidates) 4.9 either way, k = 12 6.1 -> 5.6, k = 20 8.1 -> 5.8, k = 79
// 20.4 -> 6.1.  (A bisection on the key's bits, with three barriers a bit, took
// 37 to 61 us for lists above 512, k above 170 or beyond a tenth of the lattice,
// more than the 23 to 25 of the step and selection kernels; radix 4.9 to 13.1 at
// 300 to 4000 sites.)
constexpr int kSmallRank = 32;

// Bin of a 256-bin LDS histogram where the count from the top reaches `need`
// (at least 1, at most the total): the bin, the count above it and its own.
// Every thread calls it, after a barrier that ends the histogram's updates.
// Out of line: inlined twice it cost the short lists' path 6 % (tube of 800
// sites, 400 steps: 1246 against 1177 us).
struct SmallBin { int bin; unsigned int above, count; };
__device__ __noinline__ SmallBin find_small(const unsigned int* h, unsigned int need, SmallBin* out) {
  if (threadIdx.x < 64) {
    const int lane = (int)threadIdx.x, top = 255 - 4 * lane;
    unsigned int c[4], sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) { c[j] = h[top - j]; sum += c[j]; }
    unsigned int incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned int v = __shfl_up(incl, o);
      if (lane >= o) incl += v;
    }
    unsigned int above = incl - sum;
    if (above < need && need <= incl) {
      int j = 0;
      while (above + c[j] < need) above += c[j++];
      *out = SmallBin{top - j, above, c[j]};
    }
  }
  __syncthreads();
  return *out;
}

template <class S, int SPT>
__global__ __launch_bounds__(kSmallThreads) void k_small(const StepArgs<typename StoreT<S>::R> A,
                                                         const SmallArgs a) {
  using R = typename StoreT<S>::R;
  using K = typename KeyOf<R>::T;
  constexpr bool SH = StoreT<S>::shifted;
  constexpr int CAP = SPT * kSmallThreads;
  __shared__ S lat[3][CAP];
  __shared__ K c_key[CAP];
  __shared__ uint16_t c_site[CAP];
  __shared__ uint8_t taken[CAP];
  __shared__ unsigned int s_nc;
  __shared__ unsigned int dh[256];
  __shared__ SmallBin s_bin;
  __shared__ unsigned int s_nsel;
  __shared__ unsigned long long s_kth;    // the key that the next floor takes
  __shared__ unsigned long long s_top[2]; // largest finite key, per parity
  const int tid = threadIdx.x, n = A.nx;
  const bool per = A.bc == BC_PERIODIC;
  SelState* const st = A.sel;
  const bool ehr = A.ehrenfest != 0;
  const unsigned long long dk = A.ehr_delta <= R(0) ? 0ull : (unsigned long long)key_of<R>(A.ehr_delta);
  unsigned long long floor_key[2] = {st->floor_key[0], st->floor_key[1]};
  int raised[2] = {st->floor_raised[0], st->floor_raised[1]};
  unsigned long long step = st->step;
  unsigned long long cand_total = 0, fallbacks = 0;
  const S* const src = (const S*)A.src;
  S* const dst = (S*)A.dst;
  R om[SPT];
#pragma unroll
  for (int j = 0; j < SPT; ++j) {
    const int x = tid + j * kSmallThreads;
    om[j] = (A.omega_field && x < n) ? A.omega_field[x] : A.omega;
    if (x < n) {
#pragma unroll
      for (int i = 0; i < 3; ++i) lat[i][x] = StoreT<S>::raw(at(src + (long long)i * A.qs, (unsigned)x));
      taken[x] = 0;
    }
  }
  if (tid == 0) { s_nc = 0; s_nsel = 0; s_top[0] = s_top[1] = 0ull; }
  __syncthreads();

  int pos_events = 0;
  for (long long t = 0; t < a.steps; ++t) {
    const int par = (int)(step & 1ull);
    const unsigned long long floor = par ? floor_key[1] : floor_key[0];
    const bool is_raised = (par ? raised[1] : raised[0]) != 0;
    R v[SPT][3], feq[SPT][3], m0[SPT], ux[SPT];
    // pull: f_i(x) = f_i(x - v_i), or halfway bounce-back at the ends
#pragma unroll
    for (int j = 0; j < SPT; ++j) {
      const int x = tid + j * kSmallThreads;
      if (x < n) {
        const int l = x == 0 ? n - 1 : x - 1, r = x == n - 1 ? 0 : x + 1;
        v[j][0] = StoreT<S>::cvt((per || x < n - 1) ? lat[0][r] : lat[2][x]);
        v[j][1] = StoreT<S>::cvt(lat[1][x]);
        v[j][2] = StoreT<S>::cvt((per || x > 0) ? lat[2][l] : lat[0][x]);
      }
    }
    __syncthreads();
    // candidates from `fl` up (screened against it) into the list
    auto append = [&](int j, unsigned long long fl, R screen) {
      const int x = tid + j * kSmallThreads;
      bool is_c = false;
      K key = 0;
      if (x < n) {
        R dx[3], d[3];
        eq_dev6<R>(ux[j], A.eq_kind, dx);
#pragma unroll
        for (int i = 0; i < 3; ++i) d[i] = feq[j][i] - v[j][i];
        const R dS = site_dS_dev<R, 3, SH>(v[j], d, m0[j], A.rho0, dx, dx, dx, screen);
        key = key_of<R>(dS);
        is_c = (dS > A.ehr_delta) && key >= (K)fl;
      }
      const unsigned long long mask = __ballot(is_c);
      if (!mask) return;
      const int lane = __lane_id(), leader = __ffsll((long long)mask) - 1;
      unsigned int base = 0;
      if (lane == leader) base = atomicAdd(&s_nc, (unsigned int)__popcll(mask));
      base = __shfl(base, leader);
      if (is_c) {
        const unsigned int q = base + lanes_below(mask);
        c_key[q] = key;
        c_site[q] = (uint16_t)x;
      }
    };
#pragma unroll
    for (int j = 0; j < SPT; ++j) {
      const int x = tid + j * kSmallThreads;
      if (x < n) {
        R uy;
        moments_v<R, 3, SH>(v[j], A.rho0, m0[j], ux[j], uy);
        equilibrium_v<R, 3, SH>(m0[j], A.rho0, ux[j], R(0), A.eq_kind, feq[j]);
      }
      if (ehr) append(j, floor, value_of_key<R>(floor));
      if (x < n) {
        R d[3], post[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) d[i] = feq[j][i] - v[j][i];
        CollInfo<R> ci;
        collide_site<S, 3, COLL_LBGK>(A, v[j], feq[j], d, om[j], post, ci);
        if (A.positivity) {
          positivity_site<S, 3>(A, feq[j], post, ci);
          pos_events += ci.pos_arg >= 0 ? 1 : 0;
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) lat[i][x] = StoreT<S>::pack(post[i]);
      }
    }
    __syncthreads();
    if (ehr) {
      int nc = (int)s_nc;
      const bool fell_back = nc < a.k && is_raised;
      if (fell_back) {
        __syncthreads();
        if (tid == 0) s_nc = 0;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < SPT; ++j) append(j, dk, R(0));
        __syncthreads();
        nc = (int)s_nc;
        ++fallbacks;
      }
      cand_total += (unsigned long long)nc;
      // the next floor of this parity: kept while 2k to 3.5k sites reach it,
      // else aimed at the 3k-th key; never raised when k is at least a tenth
      // of the lattice
      const bool raises = 10 * a.k < a.n_sites && a.k > 0;
      const bool keep = is_raised && !fell_back && nc >= 2 * a.k && nc <= 7 * a.k / 2;
      const long long aim = (raises && !keep && nc >= 3 * a.k) ? 3 * a.k : 0;   // rank, from 1
      const bool last = t + 1 == a.steps;
      const int take = (int)(a.k < nc ? a.k : nc);
      if (__builtin_expect(nc <= kSmallRank, 1)) {
        // rank of each entry: how many beat it (key, then the lower site)
        for (int q = tid; q < nc; q += kSmallThreads) {
          const K key = c_key[q];
          const uint16_t site = c_site[q];
          int beat = 0;
          for (int e = 0; e < nc; ++e)
            beat += (c_key[e] > key || (c_key[e] == key && c_site[e] < site)) ? 1 : 0;
          if (beat < take) taken[site] = 1;
          if (aim && beat == aim - 1) s_kth = (unsigned long long)key;
        }
        __syncthreads();
      } else {
        // the rank-th entry by (key descending, site ascending): digits of the
        // key from the top, then (sites) those of ~site.  Ends where a digit's
        // bin is taken whole: for distinct keys after three or four.
        auto nth = [&](long long rank, bool sites, K& pk, unsigned int& ps) {
          constexpr int KD = (int)sizeof(K);
          pk = 0;
          ps = 0;
          unsigned int need = (unsigned int)rank;
          for (int d = 0; d < KD + (sites ? 2 : 0); ++d) {
            const bool on_key = d < KD;
            const int sh = 8 * (on_key ? KD - 1 - d : 1 - (d - KD));
            if (tid < 256) dh[tid] = 0;
            __syncthreads();
            for (int b = 0; b < nc; b += kSmallThreads) {
              const int q = b + tid;
              bool on = false;
              unsigned int digit = 0;
              if (q < nc) {
                const K key = c_key[q];
                const unsigned int ns = 0xffffu - c_site[q];
                on = on_key ? d == 0 || ((key ^ pk) >> (sh + 8)) == 0
                            : key == pk && (d == KD || ((ns ^ ps) >> 8) == 0);
                digit = on_key ? (unsigned int)(key >> sh) & 255u : (ns >> sh) & 255u;
              }
              hist_add(dh, digit, on);
            }
            __syncthreads();
            const SmallBin bin = find_small(dh, need, &s_bin);
            need -= bin.above;
            if (on_key) pk |= (K)bin.bin << sh;
            else ps |= (unsigned int)bin.bin << sh;
            if (bin.count == need) break;
          }
        };
        K pk;
        unsigned int ps;
        if (take > 0) {
          nth(take, true, pk, ps);
          for (int q = tid; q < nc; q += kSmallThreads)
            if (c_key[q] > pk || (c_key[q] == pk && 0xffffu - c_site[q] >= ps)) taken[c_site[q]] = 1;
        }
        if (aim) {
          nth(aim, false, pk, ps);
          if (tid == 0) s_kth = (unsigned long long)pk;
        }
        __syncthreads();
      }
      unsigned long long fnext = dk;
      if (raises) {
        if (keep) fnext = floor;
        else if (aim) fnext = s_kth;
        else if (!fell_back && is_raised) fnext = floor > 2 * a.quarter ? floor - 2 * a.quarter : 0ull;
        if (fnext < dk) fnext = dk;
        // an infinite key leaves no room for a frame above it
        if (fnext >= KeyInf<R>::v) fnext = is_raised ? floor : dk;
      }
      if (par) { floor_key[1] = fnext; raised[1] = fnext > dk ? 1 : 0; }
      else { floor_key[0] = fnext; raised[0] = fnext > dk ? 1 : 0; }
      if (t + 2 >= a.steps) {
        // this parity's range, for the frame left behind
        if (tid == 0) s_top[par] = 0ull;
        __syncthreads();
        unsigned long long top = 0ull;
        for (int q = tid; q < nc; q += kSmallThreads) {
          const unsigned long long key = (unsigned long long)c_key[q];
          if (key < KeyInf<R>::v && key > top) top = key;
        }
        if (top) atomicMax(&s_top[par], top);
      }
      // f* at the selected sites
#pragma unroll
      for (int j = 0; j < SPT; ++j) {
        const int x = tid + j * kSmallThreads;
        if (x < n && taken[x]) {
          taken[x] = 0;
#pragma unroll
          for (int i = 0; i < 3; ++i) lat[i][x] = StoreT<S>::pack(feq[j][i]);
          if (last) a.selected[atomicAdd(&s_nsel, 1u)] = x;
        }
      }
      if (tid == 0) s_nc = 0;
      __syncthreads();
    }
    ++step;
  }

#pragma unroll
  for (int j = 0; j < SPT; ++j) {
    const int x = tid + j * kSmallThreads;
    if (x < n) {
#pragma unroll
      for (int i = 0; i < 3; ++i) *at(dst + (long long)i * A.qs, (unsigned)x) = lat[i][x];
    }
  }
  if (A.positivity && A.count_events) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) pos_events += __shfl_xor(pos_events, o);
    if (__lane_id() == 0 && pos_events)
      atomicAdd(A.counters + CNT_POSITIVITY, (unsigned long long)pos_events);
  }
  if (ehr && tid == 0) {
    for (int q = 0; q < 2; ++q) {
      const unsigned long long f = floor_key[q], hi = s_top[q];
      st->floor_key[q] = f;
      st->floor_raised[q] = raised[q];
      // a parity that took no step here keeps its frame
      if (a.steps >= 2 || (int)((step - 1) & 1ull) == q) {
        const unsigned long long span = hi > f ? 2 * (hi - f) : 1ull;
        unsigned int sh = 0;
        while (sh < 62 && (span >> sh) >= (unsigned long long)(kBuckets / 2)) ++sh;
        st->base_key[q] = f;
        st->shift[q] = sh;
      }
    }
    st->step = step;
    st->tape_t += a.steps;
    st->n_sel = (long long)s_nsel;
    st->cand_total += cand_total;
    st->fallbacks += fallbacks;
  }
}

template <class S>
static hipError_t launch_small_t(const void* args, const SmallArgs& a, hipStream_t s) {
  const StepArgs<typename StoreT<S>::R>& A = *(const StepArgs<typename StoreT<S>::R>*)args;
  if (A.nx <= kSmallThreads) hipLaunchKernelGGL((k_small<S, 1>), dim3(1), dim3(kSmallThreads), 0, s, A, a);
  else if (A.nx <= 2 * kSmallThreads) hipLaunchKernelGGL((k_small<S, 2>), dim3(1), dim3(kSmallThreads), 0, s, A, a);
  else hipLaunchKernelGGL((k_small<S, 4>), dim3(1), dim3(kSmallThreads), 0, s, A, a);
  return hipGetLastError();
}

hipError_t launch_small(int storage, const void* args, SmallArgs a, hipStream_t s) {
  a.quarter = storage == 0 ? 1ull << 50 : 1ull << 21;   // a quarter octave of Delta S
  switch (storage) {
    case 0: return launch_small_t<double>(args, a, s);
    case 1: return launch_small_t<float>(args, a, s);
    case 2: return launch_small_t<_Float16>(args, a, s);
    default: return launch_small_t<bf16_t>(args, a, s);
  }
}

}  // namespace lbm
