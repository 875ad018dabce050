// Several time steps of a D2Q9 lattice in one launch (no Ehrenfest selection:
// every step is local), by overlapped tiles.
//
// A workgroup takes a tile of sites with a halo as wide as the steps reach,
// one thread per site of that region, and advances it T steps: the first step
// pulls from the source lattice, the following ones from the post-collision
// populations in LDS, on a region that shrinks by the step's reach (one site;
// two with the median filter, whose neighbourhood adds one), and the last one
// stores the tile.  Halo sites are computed again by the neighbouring tiles.
//
// It serves lattices whose step is latency, not bandwidth: a launch, the
// round trip to the source lattice and a kernel's end per T steps instead of
// per step.  With the median filter one thread per staged site also takes the
// halo's Delta S out of the chain (the step kernel evaluates it after its own
// sites).  LBGK and MRT; the times are at the shapes below.
//
// The arithmetic of a site is the step kernel's (the same functions), so the
// lattice is the same bit for bit.
#include "lbm_collide.h"
#include "lbm_median.h"

namespace lbm {

__device__ __forceinline__ int wrap_into(int g, int n) {
  const int r = g < 0 ? g + n : (g >= n ? g - n : g);
  return (r < 0 || r >= n) ? ((g % n) + n) % n : r;
}

template <class S, int COLL, bool MEDIAN, int T, int RX, int RY>
__global__ __launch_bounds__(RX * RY) void k_multi(const StepArgs<typename StoreT<S>::R> A,
                                                   int tiles_x) {
  using R = typename StoreT<S>::R;
  constexpr int Q = 9;
  constexpr bool SH = StoreT<S>::shifted;
  constexpr int NT = RX * RY, reach = MEDIAN ? 2 : 1;
  constexpr int H = MEDIAN ? 2 * T - 1 : T - 1;      // halo of the region
  constexpr int TX = RX - 2 * H, TY = RY - 2 * H;    // the tile it stores
  static_assert(TX > 0 && TY > 0, "the region must hold a tile");
  __shared__ S pop[Q][NT];
  __shared__ R sdS[MEDIAN ? NT : 1];

  const int NB = (int)gridDim.x, b = (int)blockIdx.x;
  // each XCD takes a contiguous band of tiles (shared halo rows in one L2)
  const int tb = NB % 8 == 0 ? (b % 8) * (NB / 8) + b / 8 : b;
  const int x0 = (tb % tiles_x) * TX, y0 = (tb / tiles_x) * TY;
  const int cell = (int)threadIdx.x, rx = cell % RX, ry = cell / RX;
  const int edge = min(min(rx, RX - 1 - rx), min(ry, RY - 1 - ry));
  int x = x0 + rx - H, y = y0 + ry - H;
  const bool own = edge >= H && x < A.nx && y < A.ny;   // stored (and counted) here
  const bool wrap_x = A.bc == BC_PERIODIC || A.bc == BC_COUETTE, wrap_y = A.bc == BC_PERIODIC;
  if (wrap_x) x = wrap_into(x, A.nx);
  if (wrap_y) y = wrap_into(y, A.ny);
  const bool in = x >= 0 && x < A.nx && y >= 0 && y < A.ny;
  const bool wall = in && on_wall<R>(A, x, y);
  const unsigned o = (unsigned)(y * A.pitch + x);
  const R om = (in && A.omega_field) ? A.omega_field[o] : A.omega;
  int n_pos = 0, n_med = 0;

#pragma unroll 1
  for (int s = 0; s < T; ++s) {
    const bool active = in && edge >= reach * s;
    R v[Q], feq[Q], d[Q], m0, ux, uy, dS = R(0);
    if (active) {
      if (s == 0) {
        pull<S, Q, true>((const S*)A.src, A.qs, A.pitch, A.nx, A.ny, A.bc, x, y, A.lid, v);
      } else {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
          const int sx = x - vx_of<Q>(i), sy = y - vy_of<Q>(i);
          const bool out = (!wrap_x && (sx < 0 || sx >= A.nx)) || (!wrap_y && (sy < 0 || sy >= A.ny));
          const int from = out ? cell : cell - vy_of<Q>(i) * RX - vx_of<Q>(i);
          const R val = StoreT<S>::cvt(pop[out ? Q - 1 - i : i][from]);
          v[i] = (!wrap_y && sy >= A.ny) ? val + A.lid[i] : val;
        }
      }
      if (wall) diffusive_wall<S, Q>(A, x, y, v);
      moments_v<R, Q, SH>(v, A.rho0, m0, ux, uy);
      R dx[3], dy[3];
      equilibrium_v<R, Q, SH>(m0, A.rho0, ux, uy, A.eq_kind, feq, dx, dy);
#pragma unroll
      for (int i = 0; i < Q; ++i) d[i] = feq[i] - v[i];
      if constexpr (MEDIAN) {
        // exact at once: screening it against delta first saves work in a
        // workgroup without a candidate, but one with a candidate, which the
        // launch waits for, would evaluate it twice
        if (!wall) dS = site_dS_dev<R, Q, SH>(v, d, m0, A.rho0, dx, dy, dx, R(0));
      }
    }
    bool post = active;               // sites this step collides
    if constexpr (MEDIAN) {
      post = active && edge >= 2 * s + 1;
      const bool cand = post && !wall && (dS > A.med_delta) && (dS < r_inf<R>());
      // (also the barrier after the pulls)
      if (__syncthreads_or(cand)) {
        sdS[cell] = (active && !wall) ? dS : R(__builtin_nan(""));
        __syncthreads();
        bool acc = false;
        if (post && !wall && __ballot(cand)) {
          const R med = median_of_9<R>([&](int k) { return sdS[cell + (k / 3 - 1) * RX + k % 3 - 1]; });
          acc = cand & (med < dS);
          if (acc) {
            const R c = sqrt(med / dS);
#pragma unroll
            for (int i = 0; i < Q; ++i) {
              v[i] = feq[i] + c * (v[i] - feq[i]);
              d[i] = feq[i] - v[i];
            }
          }
        }
        n_med += (acc && own) ? 1 : 0;
      }
    } else {
      __syncthreads();                // every pull is done
    }
    if (post) {
      R out[Q];
      if (wall) {
#pragma unroll
        for (int i = 0; i < Q; ++i) out[i] = v[i];   // keeps its streamed state
      } else {
        CollInfo<R> ci;
        collide_site<S, Q, COLL>(A, v, feq, d, om, out, ci);
        if (A.positivity) positivity_site<S, Q>(A, feq, out, ci);
        n_pos += (own && ci.pos_arg >= 0) ? 1 : 0;
      }
      if (s + 1 < T) {
#pragma unroll
        for (int i = 0; i < Q; ++i) pop[i][cell] = StoreT<S>::pack(out[i]);
      } else if (own) {
        S* dst = (S*)A.dst;
#pragma unroll
        for (int i = 0; i < Q; ++i) *at(dst + (long long)i * A.qs, o) = StoreT<S>::pack(out[i]);
      }
    }
    __syncthreads();
  }

  if (A.count_events) {
    unsigned long long* const cnt = A.counters + (blockIdx.x % kCntSlots) * CNT_N;
    if (A.positivity) count_sum(n_pos, cnt + CNT_POSITIVITY);
    if constexpr (MEDIAN) count_sum(n_med, cnt + CNT_MEDIAN);
  }
}

// The shapes, smallest region first.  A lattice takes the first whose
// workgroups all run at once (one per CU: a second round would double the
// time of so short a launch); beyond the largest the single steps, which
// neither compute halos nor wait for the slowest of few workgroups, are
// faster.  us per step, single steps -> several (100^2, 256^2, 400^2, 512^2):
//   LBGK FP32    4.2 -> 2.4   3.5 -> 3.4   4.6 -> 3.4   5.5 -> 5.9 (not used)
//   MRT FP32     4.5 -> 2.7   4.7 -> 3.7   5.6 -> 3.9   5.9 -> 6.8 (not used)
//   MRT FP64     4.6 -> 3.3   5.8 -> 4.8   8.9 -> 8.6   9.5 -> 15.7 (not used)
//   median FP32 11.0 -> 5.4   9.4 -> 6.3  11.1 -> 6.1  11.6 -> 11.1 (not used)
//   median FP64 15.9 -> 7.9  14.6 -> 9.0  18.4 -> 16.1 21.0 -> 22.6 (not used)
// FP64 with the median filter takes one step per launch beyond 160^2 (two
// steps of a 24 x 24 region: 12.3 us at 256^2), and gains from the staging
// alone, up to two rounds.  FP64 ELBM is bound by its root solve (256^2: 25 to
// 30 us in every form) and stays with the single steps.
struct Shape { int steps, rx, ry; bool median; int most; };
constexpr Shape kShapes[] = {
    {4, 16, 16, false, 256}, {4, 24, 24, false, 256}, {4, 32, 32, false, 256},
    {2, 16, 16, true, 256},  {2, 24, 24, true, 256},  {2, 32, 32, true, 256},
    {1, 32, 16, true, 512},
};
constexpr int kShapeN = (int)(sizeof(kShapes) / sizeof(kShapes[0]));
constexpr int kFp64MedianWide = 6;   // FP64 with the median filter: shapes 3 and 6

static long long shape_blocks(const Shape& h, int nx, int ny) {
  const int e = h.median ? 2 * h.steps - 1 : h.steps - 1;
  const int tx = h.rx - 2 * e, ty = h.ry - 2 * e;
  return (long long)((nx + tx - 1) / tx) * ((ny + ty - 1) / ty);
}

static int shape_of(int storage, int coll, bool median, int nx, int ny) {
  if (coll == COLL_ELBM) return -1;
  for (int k = 0; k < kShapeN; ++k) {
    if (kShapes[k].median != median) continue;
    if (median && (storage == 0 ? (k == 4 || k == 5) : k == kFp64MedianWide)) continue;
    if (shape_blocks(kShapes[k], nx, ny) <= kShapes[k].most) return k;
  }
  return -1;
}

int multi_steps(int storage, int coll, bool median, int nx, int ny) {
  const int k = shape_of(storage, coll, median, nx, ny);
  return k < 0 ? 0 : kShapes[k].steps;
}

template <class S, int COLL, int K>
static hipError_t launch_m(const StepArgs<typename StoreT<S>::R>& A, hipStream_t s) {
  constexpr Shape h = kShapes[K];
  constexpr int e = h.median ? 2 * h.steps - 1 : h.steps - 1, TX = h.rx - 2 * e;
  const unsigned blocks = (unsigned)shape_blocks(h, A.nx, A.ny);
  hipLaunchKernelGGL((k_multi<S, COLL, h.median, h.steps, h.rx, h.ry>), dim3(blocks),
                     dim3(h.rx * h.ry), 0, s, A, (A.nx + TX - 1) / TX);
  return hipGetLastError();
}

template <class S, int COLL>
static hipError_t launch_multi_c(int shape, const void* args, hipStream_t s) {
  const StepArgs<typename StoreT<S>::R>& A = *(const StepArgs<typename StoreT<S>::R>*)args;
  constexpr bool F64 = sizeof(S) == 8;
  switch (shape) {
    case 0: return launch_m<S, COLL, 0>(A, s);
    case 1: return launch_m<S, COLL, 1>(A, s);
    case 2: return launch_m<S, COLL, 2>(A, s);
    case 3: return launch_m<S, COLL, 3>(A, s);
    case 4: if constexpr (!F64) return launch_m<S, COLL, 4>(A, s); break;
    case 5: if constexpr (!F64) return launch_m<S, COLL, 5>(A, s); break;
    case 6: if constexpr (F64) return launch_m<S, COLL, 6>(A, s); break;
  }
  return hipErrorInvalidValue;
}

hipError_t launch_multi(int storage, int coll, bool median, const void* args, int nx, int ny,
                        hipStream_t s) {
  const int k = shape_of(storage, coll, median, nx, ny);
  const bool mrt = coll == COLL_MRT;
  switch (storage) {
    case 0: return mrt ? launch_multi_c<double, COLL_MRT>(k, args, s) : launch_multi_c<double, COLL_LBGK>(k, args, s);
    case 1: return mrt ? launch_multi_c<float, COLL_MRT>(k, args, s) : launch_multi_c<float, COLL_LBGK>(k, args, s);
    case 2: return mrt ? launch_multi_c<_Float16, COLL_MRT>(k, args, s) : launch_multi_c<_Float16, COLL_LBGK>(k, args, s);
    default: return mrt ? launch_multi_c<bf16_t, COLL_MRT>(k, args, s) : launch_multi_c<bf16_t, COLL_LBGK>(k, args, s);
  }
}

}  // namespace lbm
