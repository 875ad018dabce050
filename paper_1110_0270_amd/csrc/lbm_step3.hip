// The D3Q27 step on a periodic lattice for gfx950:
//   pull-stream (section 2, free flight)
//   -> moments and the product equilibrium (section 6's 1D equilibria)
//   -> median entropy filter over the 27-site neighbourhood (section 4: the
//      14th of the 27 sorted Delta S values)
//   -> LBGK collision (eq. CollisionIntegral) -> positivity rule (section 4)
//   -> store into the second lattice.
// Without the median filter every lane takes one site of a 256-site row
// segment (k_step3).  With it two kernels share the step:
//   k_step3 takes the whole lattice as if no site were filtered, screens each
//   site's Delta S against delta by a bound and flags the chunk (64 x 8 columns
//   of up to 32 layers) of every site not proved below it;
//   k_step3_median takes the flagged chunks again with the filter: a workgroup
//   marches along z through a chunk's layers, keeping Delta S of three layers
//   (the tile plus a one-site halo) in an LDS ring, so that each layer's
//   Delta S is evaluated once per column, not once per neighbour.
// Where most chunks hold such a site the first kernel would be waste: a step
// that finds more than a quarter of the chunks flagged leaves the next one to
// k_step3_median alone, until fewer than an eighth hold a site above 7/8 delta
// (Med3State; the result does not depend on it).  That kernel has Delta S, not
// the bound that flags; at 7/8 it counts what the bound would flag while
// max (f*_i - f_i) / f*_i <= 0.2 (the bound is within 1 + 2/3 of that), so the
// mode does not change back and forth over a flow just under delta.  The first kernel's empty launch then
// costs 17 us; with delta = 0 every site off its equilibrium is a candidate,
// and it is not launched.  256^3 FP32 Taylor-Green vortex, us a step: 1104 ->
// 694 at delta = 1e-3 (no site above it), 1156 -> 1176 at 1e-9 (all above it),
// 1161 -> 1161 at 0.  160^3 FP64: 771 -> 336, 829 -> 841-853, 828 -> 832.
#include <hip/hip_ext.h>

#include "lbm_collide.h"
#include "lbm_internal.h"
#include "lbm_site3.h"

namespace lbm {

// g mod n for the tile and halo coordinates, which lie within one lattice
// width of [0, n) unless the lattice is narrower than a tile (then the
// remainder)
__device__ __forceinline__ int wrap_mod(int g, int n) {
  const int r = g < 0 ? g + n : (g >= n ? g - n : g);
  return (r < 0 || r >= n) ? ((g % n) + n) % n : r;
}

// After the filter: LBGK, the positivity rule (its events to cnt), the store.
template <class S>
__device__ __forceinline__ void finish27(const StepArgs<typename StoreT<S>::R>& A, unsigned off,
                                         bool valid, typename StoreT<S>::R v[27],
                                         typename StoreT<S>::R feq[27], unsigned long long* cnt) {
  using R = typename StoreT<S>::R;
  bool pos_event = false;
  if (valid) {
#pragma unroll
    for (int i = 0; i < 27; ++i) v[i] = v[i] + A.omega * (feq[i] - v[i]);   // collided in place
    if (A.positivity) {
      CollInfo<R> ci;
      positivity_site<S, 27>(A, feq, v, ci);
      pos_event = ci.pos_arg >= 0;
    }
    S* dst = (S*)A.dst;
#pragma unroll
    for (int i = 0; i < 27; ++i) StoreT<S>::st(at(dst + (long long)i * A.qs, off), v[i]);
  }
  if (A.positivity && A.count_events) count_event(pos_event, cnt);
}

constexpr int kM3X = 64, kM3Y = 8;
constexpr double kM3Near = 0.875;
// Every site off its equilibrium is a candidate: the first kernel is not launched
template <class R>
__host__ __device__ inline bool med3_always(R delta) { return !(delta > R(0)); }
// Layers of a chunk: 1.06 layers of Delta S per layer (FP32)
template <class S> constexpr int m3_layers() { return sizeof(typename StoreT<S>::R) == 4 ? 32 : 16; }

// MED: the first of the median step's two kernels.  Bound by HBM: with the
// marching kernel alone every site's Delta S, its halo's and a second pull of
// its own took 1105 us at 256^3 FP32 (delta = 1e-3, no site above it); now
// 650 us (5.6 TB/s).  One segment per workgroup: a loop over four kept 25
// registers more (717 us).
template <class S, bool MED>
__global__ __launch_bounds__(256) void k_step3(const StepArgs<typename StoreT<S>::R> A) {
  using R = typename StoreT<S>::R;
  constexpr bool SH = StoreT<S>::shifted;
  if (MED && A.med3->dense) return;
  // workgroup -> (256-site segment of a row, row z * ny3 + y)
  const int segs = (A.nx + 255) / 256;
  const int row = (int)blockIdx.x / segs, x = ((int)blockIdx.x % segs) * 256 + (int)threadIdx.x;
  const int y = row % A.ny3, z = row / A.ny3;
  const bool valid = x < A.nx;
  R v[27], feq[27];
  bool may = false;
  if (valid) {
    R m0, ux, uy, uz;
    pull27<S>((const S*)A.src, A.qs, A.pitch, A.nx, A.ny3, A.nz, x, y, z, v);
    moments27<R, SH>(v, A.rho0, m0, ux, uy, uz);
    equilibrium27<R, SH>(m0, A.rho0, ux, uy, uz, A.eq_kind, feq);
    if constexpr (MED) may = may_exceed27<R, SH>(v, feq, m0, A.rho0, ux, uy, uz, A.eq_kind, A.med_delta);
  }
  unsigned long long* cnt = A.counters + (blockIdx.x % kCntSlots) * CNT_N + CNT_POSITIVITY;
  if constexpr (MED) {
    // a wavefront's 64 sites of a row lie in one chunk
    const int tx = (A.nx + kM3X - 1) / kM3X, ty = (A.ny3 + kM3Y - 1) / kM3Y;
    Med3Chunk* chunk = med3_chunk(A.med3) + (z / m3_layers<S>() * ty + y / kM3Y) * tx + x / kM3X;
    cnt = &chunk->pos_events;
    const unsigned long long any = __ballot(may);
    if (any && (int)__lane_id() == __ffsll((long long)any) - 1) chunk->flag = 1ull;
  }
  finish27<S>(A, (unsigned)(row * A.pitch + x), valid, v, feq, cnt);
}

template <class R>
__device__ __forceinline__ void cswap(R& a, R& b) {
  const R lo = fmin(a, b), hi = fmax(a, b);
  a = lo;
  b = hi;
}

// The 14th smallest of 27 values by forgetful selection: a window of 15
// values; each round moves the window's minimum to its first slot and its
// maximum to its last, drops both (neither can be the median of the values
// not yet dropped) and takes the next value into the last slot.  After
// twelve rounds three values remain, and their middle one is the median.
// All indices are compile-time, so the array stays in registers.
template <class R>
__device__ __forceinline__ R median27(R a[27]) {
#pragma unroll
  for (int r = 0; r < 13; ++r) {
#pragma unroll
    for (int k = r + 1; k < 15; ++k) cswap(a[r], a[k]);        // minimum -> a[r]
#pragma unroll
    for (int k = r + 1; k < 14; ++k) cswap(a[k], a[14]);       // maximum -> a[14]
    if (r < 12) a[14] = a[15 + r];
  }
  return a[13];
}

// ALL: every chunk is taken (med3_always, or rows past the first kernel's
// launch), without the first kernel and its records.
template <class S, int TX, int TY, int ZC, bool ALL>
__global__ __launch_bounds__(TX * TY, (sizeof(typename StoreT<S>::R) == 4 && TX * TY <= 512) ? 4 : 1) void k_step3_median(const StepArgs<typename StoreT<S>::R> A,
                                                          int tiles_x, int tiles_y) {
  using R = typename StoreT<S>::R;
  constexpr bool SH = StoreT<S>::shifted;
  constexpr int NT = TX * TY, SW = TX + 2, NS = (TX + 2) * (TY + 2);
  __shared__ R ring[3][NS];
  __shared__ int s_near;   // a site near delta or above it in this chunk (not a register of the march)

  // Workgroup -> (tile, chunk of layers).  Consecutive workgroups are dealt
  // round-robin to the 8 XCDs; each XCD takes a contiguous band of tiles
  // (neighbouring rows of tiles in the same layers), whose halos it reads
  // from its own L2.
  const int T = tiles_x * tiles_y * ((A.nz + ZC - 1) / ZC);
  const int b = blockIdx.x;
  const int tb = (T % 8 == 0) ? (b % 8) * (T / 8) + b / 8 : b;
  const int tile_x = tb % tiles_x, tile_y = (tb / tiles_x) % tiles_y, chunk = tb / (tiles_x * tiles_y);
  const int x0 = tile_x * TX, y0 = tile_y * TY, z0 = chunk * ZC;
  const int z1 = min(z0 + ZC, A.nz);
  const int tid = threadIdx.x, lx = tid % TX, ly = tid / TX;
  const int x = x0 + lx, y = y0 + ly;
  const bool valid = x < A.nx && y < A.ny3;
  unsigned long long* const cnt = A.counters + (b % kCntSlots) * CNT_N;

  // Every workgroup reads the mode before it takes its ticket, so the last
  // one may change it; it and the chunk's record are read again after the
  // march, not kept.  Tickets are 64-bit atomics (workgroups done in the low
  // half, chunks flagged or near delta in the high), taken in groups: a thousand on
  // one address, after two dependent loads, cost 11 us of a 705 us step
  // (256^3 FP32).
  auto leave = [&](bool near, bool dense, bool flagged, unsigned long long pos) {
    if (tid != 0) return;
    // the first kernel's positivity events stand where this one did nothing
    Med3Chunk* const chunk_st = med3_chunk(A.med3) + tb;
    if (pos && !dense && !flagged) atomicAdd(cnt + CNT_POSITIVITY, pos);
    if (pos) chunk_st->pos_events = 0ull;
    if (flagged) chunk_st->flag = 0ull;
    const int g = tb % kMed3Groups;
    const unsigned long long mine = 1ull | (((dense ? near : flagged) ? 1ull : 0ull) << 32);
    const unsigned long long in_g = atomicAdd(&A.med3->group[g][0], mine) + mine;
    if ((unsigned int)in_g != (unsigned int)((T - g + kMed3Groups - 1) / kMed3Groups)) return;
    A.med3->group[g][0] = 0ull;
    const unsigned long long sum = (in_g & ~0xffffffffull) | 1ull;
    const unsigned long long all = atomicAdd(&A.med3->tally, sum) + sum;
    if ((unsigned int)all == (unsigned int)min(T, kMed3Groups)) {
      const unsigned long long held = all >> 32;
      A.med3->dense = dense ? (8 * held >= (unsigned long long)T ? 1 : 0)
                            : (4 * held > (unsigned long long)T ? 1 : 0);
      A.med3->tally = 0ull;
    }
  };
  if constexpr (!ALL) {
    // (all three loads before the branch: one round trip)
    const int dense = A.med3->dense;
    const unsigned long long flag = med3_chunk(A.med3)[tb].flag, pos = med3_chunk(A.med3)[tb].pos_events;
    if (!(flag | (unsigned long long)dense)) {
      __syncthreads();   // every wavefront has read the mode: the ticket lets it change
      leave(false, false, false, pos);
      return;
    }
    if (tid == 0) s_near = 0;   // the first layer's barrier is before the first vote
  }

  // Delta S of layer z (periodic) over the tile and its halo into ring slot
  // `slot`; positions beyond the lattice wrap, so ragged tiles need no
  // special case.
  auto layer = [&](int z, int slot) {
    const int zz = wrap_mod(z, A.nz);
#pragma unroll 1
    for (int s = tid; s < NS; s += NT) {
      const int gx = wrap_mod(x0 + s % SW - 1, A.nx), gy = wrap_mod(y0 + s / SW - 1, A.ny3);
      R v[27], d[27], m0, ux, uy, uz;
      pull27<S, true>((const S*)A.src, A.qs, A.pitch, A.nx, A.ny3, A.nz, gx, gy, zz, v);
      moments27<R, SH>(v, A.rho0, m0, ux, uy, uz);
      equilibrium27<R, SH>(m0, A.rho0, ux, uy, uz, A.eq_kind, d);
#pragma unroll
      for (int i = 0; i < 27; ++i) d[i] -= v[i];                      // f* - f
      ring[slot][s] = site_dS_q<R, 27, SH>(v, d, m0, A.rho0, ux, uy, uz, A.eq_kind, R(0));
    }
  };

  layer(z0 - 1, 2);
  layer(z0, 0);
  for (int z = z0; z < z1; ++z) {
    const int sc = (z - z0) % 3, sm = (z - z0 + 2) % 3, sp = (z - z0 + 1) % 3;
    layer(z + 1, sp);
    __syncthreads();
    // The median decision first, from LDS alone (the site's own state is
    // not yet live): median < Delta S exactly when at least 14 of the 27
    // values lie below Delta S; wavefronts without a site above delta skip
    // the count, and only wavefronts with an accepted site select the 14th.
    const R dS = valid ? ring[sc][(ly + 1) * SW + lx + 1] : R(0);
    const bool cand = valid && (dS > A.med_delta) && (dS < r_inf<R>());
    bool acc = false;
    R med = R(0);
    auto nbr = [&](int k) {
      const int dz = k / 9 - 1, dy = (k / 3) % 3 - 1, dx = k % 3 - 1;
      return ring[dz < 0 ? sm : (dz > 0 ? sp : sc)][(ly + 1 + dy) * SW + lx + 1 + dx];
    };
    if constexpr (!ALL) {
      if (__ballot(valid && !(dS <= A.med_delta * R(kM3Near)))) s_near = 1;
    }
    if (__ballot(cand)) {
      int below = 0;
#pragma unroll
      for (int k = 0; k < 27; ++k) below += nbr(k) < dS ? 1 : 0;
      acc = cand && below >= 14;
      if (__ballot(acc)) {
        R nb[27];
#pragma unroll
        for (int k = 0; k < 27; ++k) nb[k] = nbr(k);
        med = median27<R>(nb);
      }
    }
    // every lane pulls (a lane past the lattice edge an in-range site that
    // it does not store), so that nothing stays undefined from one layer to
    // the next: the compiler would otherwise carry those values through the
    // next layer's Delta S and run out of registers
    R v[27], feq[27], m0, ux, uy, uz;
    pull27<S, true>((const S*)A.src, A.qs, A.pitch, A.nx, A.ny3, A.nz, valid ? x : x0, valid ? y : y0, z, v);
    moments27<R, SH>(v, A.rho0, m0, ux, uy, uz);
    equilibrium27<R, SH>(m0, A.rho0, ux, uy, uz, A.eq_kind, feq);
    if (acc) {
      const R c = sqrt(med / dS);
#pragma unroll
      for (int i = 0; i < 27; ++i) v[i] = feq[i] + c * (v[i] - feq[i]);
    }
    if (A.count_events) count_event(acc, cnt + CNT_MEDIAN);
    finish27<S>(A, (unsigned)((z * A.ny3 + y) * A.pitch + x), valid, v, feq, cnt + CNT_POSITIVITY);
    __syncthreads();   // the next layer overwrites the ring slot of z - 1
  }
  if constexpr (!ALL)
    leave(s_near != 0, A.med3->dense != 0, med3_chunk(A.med3)[tb].flag != 0,
          med3_chunk(A.med3)[tb].pos_events);
}

// ---------------------------------------------------------------------------
// Workgroups of the row kernels (k_step3), and whether the median step may use
// them: a launch holds fewer than 2^32 threads, and a narrow lattice pays 256
// of them for each of its rows (64 x 2^12 x 2^12 sites: 2^24 rows).  The
// marching kernel's 512 take 8 rows of 16 or 32 layers.
static long long step3_row_groups(int nx, int ny, int nz) {
  return (nx + 255) / 256 * (long long)ny * nz;
}
bool step3_screens(int nx, int ny, int nz) { return step3_row_groups(nx, ny, nz) * 256 < (1ll << 32); }

template <class S>
static hipError_t launch3(bool median, const void* args, hipStream_t s, hipEvent_t e0,
                          hipEvent_t e1) {
  using R = typename StoreT<S>::R;
  const StepArgs<R>& A = *(const StepArgs<R>*)args;
  const dim3 rows((unsigned)step3_row_groups(A.nx, A.ny3, A.nz));
  if (median) {
    // 64 x 8 columns: 1.29 halo sites per site (FP32 arithmetic: 64 x 16
    // tiles measured no faster)
    constexpr int ZC = m3_layers<S>();
    const int tx = (A.nx + kM3X - 1) / kM3X, ty = (A.ny3 + kM3Y - 1) / kM3Y;
    const dim3 grid(tx * ty * ((A.nz + ZC - 1) / ZC)), block(kM3X * kM3Y);
    auto first = k_step3<S, true>;
    auto second = k_step3_median<S, kM3X, kM3Y, ZC, false>;
    auto alone = k_step3_median<S, kM3X, kM3Y, ZC, true>;
    if (e0) (void)hipEventRecord(e0, s);
    if (med3_always(A.med_delta) || !step3_screens(A.nx, A.ny3, A.nz)) {
      hipLaunchKernelGGL(alone, grid, block, 0, s, A, tx, ty);
    } else {
      hipLaunchKernelGGL(first, rows, dim3(256), 0, s, A);
      hipLaunchKernelGGL(second, grid, block, 0, s, A, tx, ty);
    }
    if (e1) (void)hipEventRecord(e1, s);
  } else {
    auto kern = k_step3<S, false>;
    if (e0 && e1) hipExtLaunchKernelGGL(kern, rows, dim3(256), 0, s, e0, e1, 0, A);
    else hipLaunchKernelGGL(kern, rows, dim3(256), 0, s, A);
  }
  return hipGetLastError();
}

long long med3_chunks(int storage, int nx, int ny, int nz) {
  const int zc = storage == 0 ? m3_layers<double>() : m3_layers<float>();
  return (long long)((nx + kM3X - 1) / kM3X) * ((ny + kM3Y - 1) / kM3Y) * ((nz + zc - 1) / zc);
}

hipError_t launch_step3(int storage, bool median, const void* args, hipStream_t s, hipEvent_t e0,
                        hipEvent_t e1) {
  switch (storage) {
    case 0: return launch3<double>(median, args, s, e0, e1);
    case 1: return launch3<float>(median, args, s, e0, e1);
    case 2: return launch3<_Float16>(median, args, s, e0, e1);
    default: return launch3<bf16_t>(median, args, s, e0, e1);
  }
}

}  // namespace lbm
