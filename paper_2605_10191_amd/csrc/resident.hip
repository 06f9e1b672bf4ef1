// Resident Clenshaw recurrence of a chain operator: the K steps of one column
// (or of two interleaved columns) in ONE launch, by a team of workgroups that
// live on one XCD.
//
// What bounds short chains is not bytes but the launch of every step: at
// L = 18 a step's vectors are 389 KB a column, 0.2 us of HBM time, yet a step
// took 4 to 6 us alone and 17.4 us for 13 columns, whose interleaved block
// outgrows an XCD's 4 MB L2.  Here every member of a team owns a fixed slab
// of rows for the whole recurrence, so
//   - v, b_{i+1}, b_{i+2}, the diagonal and the target of every hop of its
//     rows stay in registers: a step decodes nothing and streams nothing;
//   - the slab of b_{i+1} sits in LDS, where most hops land; the hops that
//     leave the slab gather from the team's vector in global memory, which
//     the team's own L2 holds (copying those rows into LDS first, so that all
//     hops are LDS reads, measured slower: it adds a barrier to each step);
//   - a step ends with a barrier of the team's members (0.9 us for 32 of
//     them; a launch in a replayed graph takes 1.6 us before it does
//     anything) instead of a kernel boundary.
// Measured (FP64, us a step, before -> here): one column at L = 12 3.6 -> 1.0,
// L = 16 3.9 -> 1.9, L = 18 4.5 -> 3.0; 13 columns at L = 14 4.2 -> 1.7; 13 columns
// at L = 18 17.3 -> 4.5, of which the barrier and the gathers' round trip are
// 1.3 and the LDS reads of the hops most of the rest.
// The columns are spread over the eight XCDs, so no data crosses them.
//
// Teams form from the workgroups that are running: a workgroup reads the XCD
// it is on and joins that XCD's next team; the first member closes the team
// when it is full or after a bounded time (see team_join), and a workgroup that
// comes later leaves at once.  So a barrier only ever waits for workgroups that run, no
// matter what else the device executes, and a team with fewer members than
// slabs walks several slabs a member (reloading their state) instead.  Column
// groups are handed out by a counter, so any set of teams finishes them all.
//
// Members exchange data through the L2 of their XCD: a store is in it once
// the writer's vmcnt is zero (the L1 writes through), and the readers' loads
// bypass their L1 (agent scope).
#include <algorithm>

#include <iterator>
#include <memory>
#include <optional>

#include "chain_dev.hpp"
#include "internal.hpp"

namespace polfed {

namespace {

constexpr int kResClosed = 1 << 20;
constexpr int kFieldStride = 33;  // field table of a column: 32 sites, constant
constexpr int kAuxAgent = 16;     // load of agent scope: past the L1

__device__ __forceinline__ int res_load(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int res_add(int* p, int v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void res_store(int* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// the XCD of this workgroup (hardware register XCC_ID, 4 bits)
__device__ __forceinline__ int xcc_id() { return __builtin_amdgcn_s_getreg(20 | (3 << 11)) & 15; }

struct TeamView {
  ResTeam* t;
  int n, rank;
  int step;  // barriers passed
  int failed;
  long long wait;  // of a barrier at most, in ticks
  int* fail;       // LDS: a barrier of this workgroup gave up
};

// Every wait is bounded, so that a kernel ends whatever happens to its team's
// state: a barrier that gives up sets err and lets its member run on to the end
// of the columns it is at, and what the call returns is NaN or an error.

// What a member that cannot go on leaves of n elements of a result.
template <typename T>
__device__ __forceinline__ void poison(T* w, int64_t n) {
  for (int64_t i = threadIdx.x; i < n; i += kResThreads) w[i] = T(NAN);
}

// All members have stored what they wrote before; afterwards all see it.
// between() runs once the workgroup's own LDS reads are done, while the other
// members arrive.  Every member raises its own flag and one wave polls all of
// them with one load.
template <class F>
__device__ __forceinline__ void team_barrier(TeamView& tv, int* err, F&& between) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  ++tv.step;
  if (tv.n > 1 && threadIdx.x == 0) res_store(&tv.t->flag[tv.rank], tv.step);
  between();
  if (tv.n > 1 && threadIdx.x < 64 && !tv.failed) {
    const int* f = &tv.t->flag[min((int)threadIdx.x, tv.n - 1)];
    const long long t0 = wall_clock64();
    while (__ballot(res_load(f) < tv.step)) {
      if (wall_clock64() - t0 >= tv.wait) {
        tv.failed = 1;
        *tv.fail = 1;
        res_store(err, 1);
        break;
      }
    }
  }
  __syncthreads();
}

// Joins the next team of this workgroup's XCD (nslab members); false for a
// workgroup that came too late or is not needed, or (*tv.fail) that waited too
// long for its team to close.
//
// A launch for one column group (steps > 0 of it) needs one team out of the
// eight that its workgroups could form.  Beside other such launches every XCD
// gets a few workgroups of each, and a team that closes with a quarter of its
// members walks four slabs a member, ten times slower (L = 18, four contexts,
// 1,500 steps each: 34 ms a filter instead of 4).  So the teams that are not full
// in time leave, all but that of the home XCD, the one where workgroup `home`
// runs (contexts take different ones): it waits as long as it could lose that
// way, and what the others leave makes room for the rest of its members.  As
// long as the home XCD is not known nobody leaves, and its team is never the one
// to leave, so one team always goes on.
__device__ __forceinline__ bool team_join(ResState* st, int nslab, int teams_per_xcd, int* s_join,
                                          TeamView& tv, int home = 0, int steps = 0) {
  if (threadIdx.x == 0) *tv.fail = 0;
  if (nslab <= 1) return true;
  if (threadIdx.x == 0) {
    constexpr long long kJoin = 10000, kHomeMost = 200000;  // 0.1 and 2 ms
    const int x = xcc_id();
    if (steps > 0 && (int)blockIdx.x == home) res_store(&st->home, x + 1);
    const int slot = res_add(&st->slots[16 * x], 1);
    const int team = slot / nslab;
    int n = 0, rank = 0;
    if (team < teams_per_xcd) {
      ResTeam* t = &st->teams[x * kResTeamsPerXcd + team];
      rank = res_add(&t->joined, 1);
      if (rank == 0) {
        const long long t0 = wall_clock64();
        const long long most =
            steps > 0 ? min(max((long long)steps * 200, kJoin), kHomeMost) : kJoin;
        bool leave = false;
        while (res_load(&t->joined) < nslab) {
          const long long dt = wall_clock64() - t0;
          if (dt >= most) break;
          if (dt < kJoin) continue;
          const int h = res_load(&st->home);
          if (h != 0 && h != x + 1) {
            leave = true;
            break;
          }
        }
        n = __hip_atomic_fetch_or(&t->joined, kResClosed, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
        if (leave && n < nslab) n = -1;
        res_store(&t->n, n);
      } else if (rank < kResClosed) {
        // the first member runs and closes the team within 2 ms
        const long long t0 = wall_clock64();
        while ((n = res_load(&t->n)) == 0 && wall_clock64() - t0 < kResWait)
          __builtin_amdgcn_s_sleep(1);
        if (n == 0) {
          *tv.fail = 1;
          res_store(&st->err, 1);
        }
      }
    }
    s_join[0] = max(n, 0);
    s_join[1] = rank;
    s_join[2] = x * kResTeamsPerXcd + team;
  }
  __syncthreads();
  tv.n = uniform(s_join[0]);
  tv.rank = uniform(s_join[1]);
  if (tv.n == 0 || tv.rank >= nslab) return false;
  tv.n = min(tv.n, nslab);
  tv.t = &st->teams[uniform(s_join[2])];
  return true;
}

template <typename T, int G>
struct Cols {
  T x[G];
};

template <typename T, int G>
__device__ __forceinline__ Cols<T, G> rload(rsrc_t r, uint32_t off) {
  Cols<T, G> c;
  if constexpr (G == 2)
    bload2<T, kAuxAgent>(r, off, 0, c.x[0], c.x[1]);
  else
    c.x[0] = bload<T, kAuxAgent>(r, off, 0);
  return c;
}
template <typename T, int G>
__device__ __forceinline__ void rstore(const Cols<T, G>& c, rsrc_t r, uint32_t off) {
  if constexpr (G == 2)
    bstore2<0>(c.x[0], c.x[1], r, off, 0);
  else
    bstore<0>(c.x[0], r, off, 0);
}
template <typename T, int G>
__device__ __forceinline__ Cols<T, G> lread(const unsigned char* b, uint32_t off) {
  return *reinterpret_cast<const Cols<T, G>*>(b + off);
}

// Row r of slab m of D rows in nslab slabs.
__host__ __device__ __forceinline__ int64_t slab_row(int64_t D, int nslab, int m) {
  return D * m / nslab;
}

// ------------------------------------------------------------ tables ----

// Targets of the hops of a state: f(slot, rank), slot 0 the periodic bond,
// slot b + 1 the bond (b, b + 1).
template <class F>
__device__ __forceinline__ void chain_targets(int L, int periodic, uint32_t s, int64_t r,
                                              const uint32_t* binom, F&& f) {
  int below = 0;
  for (int b = 0; b + 1 < L; ++b) {
    const uint32_t sb = (s >> b) & 1u;
    if (sb != ((s >> (b + 1)) & 1u)) {
      const int64_t d = binom[b * kBinomN + below];
      f(b + 1, sb ? r + d : r - d);
    }
    below += (int)sb;
  }
  if (periodic && (((s >> (L - 1)) ^ s) & 1u)) {
    const uint32_t sp = s ^ (1u | (1u << (L - 1)));
    int k = 0;
    int64_t rk = 0;
    for (int x = 0; x < L; ++x)
      if ((sp >> x) & 1u) rk += binom[x * kBinomN + (++k)];
    f(0, rk);
  }
}

// The slab tables of a chain pattern: FILL = false counts (most hops of a row
// inside its slab, most leaving it), FILL = true writes.
// One workgroup per slab; thread t holds rows t, t + NT, ... of the slab.
template <bool FILL>
__global__ __launch_bounds__(kResThreads) void k_res_build(ResBuild p) {
  __shared__ uint32_t s_binom[(kResMaxL + 1) * kBinomN];
  for (int i = threadIdx.x; i < (kResMaxL + 1) * kBinomN; i += kResThreads) s_binom[i] = p.binom[i];
  __syncthreads();
  const int m = blockIdx.x;
  const int64_t row0 = slab_row(p.D, p.nslab, m), row1 = slab_row(p.D, p.nslab, m + 1);
  for (int j = 0; j < p.R; ++j) {
    const int64_t r = row0 + threadIdx.x + (int64_t)kResThreads * j;
    const bool valid = r < row1;
    uint32_t s = 0, rr = valid ? (uint32_t)r : 0u;
    int k = p.N;
    for (int b = p.L - 1; b >= 0; --b) {
      const uint32_t c = s_binom[b * kBinomN + k];
      if (k > 0 && rr >= c) {
        s |= 1u << b;
        rr -= c;
        --k;
      }
    }
    // entry (m, j, slot, thread): the hops inside the slab (LDS rows), those
    // leaving it (rows), the periodic bond.  A hop takes the slot of its bond
    // among the bonds that stay in (or leave) the slab in this wave, so that
    // the wave's access of a slot is mostly one run of rows: coalesced out of
    // the slab, without bank conflicts in it.  In a wave with more such bonds
    // than slots each lane packs its own.
    const int64_t per = (int64_t)(p.nl + p.nh + 1) * kResThreads;
    const int64_t e = ((int64_t)m * p.R + j) * per + threadIdx.x;
    uint32_t out = 0, in = 0;  // bonds that leave the slab in this row, that do not
    if (valid)
      chain_targets(p.L, p.periodic, s, r, s_binom, [&](int slot, int64_t to) {
        if (to < row0 || to >= row1)
          out |= 1u << slot;
        else
          in |= 1u << slot;
      });
    const uint32_t own = p.sep ? ~1u : ~0u;  // a periodic bond of its own sign
    const int nl = __popc(in & own), nh = __popc(out & own);
    uint32_t any_in = 0, any_out = 0;
    for (int b = 0; b < p.L; ++b) {
      if (__ballot((in & own) >> b & 1u)) any_in |= 1u << b;
      if (__ballot((out & own) >> b & 1u)) any_out |= 1u << b;
    }
    if (FILL && valid) {
      const uint32_t si = __popc(any_in) <= p.nl ? any_in : in & own;
      const uint32_t so = __popc(any_out) <= p.nh ? any_out : out & own;
      chain_targets(p.L, p.periodic, s, r, s_binom, [&](int slot, int64_t to) {
        const bool far = to < row0 || to >= row1;
        const uint32_t below = (1u << slot) - 1u;
        const int k = slot == 0 && p.sep ? p.nl + p.nh
                      : far              ? p.nl + __popc(so & below)
                                         : __popc(si & below);
        p.slot[e + (int64_t)k * kResThreads] = far ? kResFar | (uint32_t)to : (uint32_t)(to - row0);
      });
    }
    if (FILL) {
      if (valid) p.state[r] = s;
    } else {
      atomicMax(&p.counts[0], nl);
      atomicMax(&p.counts[1], nh);
    }
  }
}

__global__ void k_res_fill(int64_t n, uint32_t v, uint32_t* p) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// ------------------------------------------------------- recurrence ----

// A slab's rows in registers: thread t holds rows t, t + NT, ... .  A hop is
// the LDS byte offset of its target (of a zero where there is none) or, out
// of the slab, the byte offset in the group's vector (past its end, which
// reads as 0, where there is none).
template <typename T, int NL, int NH, int R, int G>
struct SlabState {
  uint32_t loc[R][(NL + 1) / 2];  // two 16-bit offsets a register
  uint32_t far[R][NH > 0 ? NH : 1], per[R];
  int nfar[R];  // slots of far that any lane of the wave uses
  Cols<T, G> v[R], b1[R], b2[R], dg[R];
};
constexpr uint32_t kNoRow = 0xFFFFFFF0u;  // an offset past any vector

// hi + lo += x, with the rounding of the sum in lo.
__device__ __forceinline__ void add_exact(double& hi, double& lo, double x) {
  const double t = hi + x, z = t - hi;
  lo += (hi - (t - z)) + (x - z);
  hi = t;
}

template <typename T, int NL, int NH, int R, int G>
__device__ __forceinline__ void res_setup(const ResArgs<T>& p, SlabState<T, NL, NH, R, G>& S,
                                          int c0, int m, const double* s_field, rsrc_t cur,
                                          rsrc_t prev, bool no_prev, unsigned char* s_b) {
  constexpr uint32_t RB = G * sizeof(T);
  const int64_t row0 = slab_row(p.D, p.nslab, m), row1 = slab_row(p.D, p.nslab, m + 1);
  const uint32_t zero = (uint32_t)p.rows_cap;
  // the diagonals first: their sums take registers that the rows' tables fill
  // later (six rows a thread: with the sums among the tables 51 registers of a
  // row's state were spilled instead of 43, L = 19, 8 columns 7.4 us a step, 6.6
  // so)
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int64_t r = row0 + threadIdx.x + kResThreads * j;
    const bool valid = r < row1;
    const uint32_t s = valid ? p.state[r] : 0u;
    const uint32_t top = (s >> (p.L - 1)) & 1u;
    const int n11 = __popc(s & (s >> 1)) + (p.periodic ? (int)(top & s & 1u) : 0);
#pragma unroll
    for (int c = 0; c < G; ++c) {
      const double* f = s_field + c * kFieldStride;
      // the diagonal is rounded once: its error is the same in every step, so
      // it does not average out over them (relative error of KPM moments, plain
      // sums / this: L = 12 2.11e-16 / 1.62e-16, L = 16 2.81e-16 / 2.23e-16; as
      // launches 1.78e-16 and 2.58e-16)
      double d = p.vzz * n11, dlo = fma(p.vzz, (double)n11, -d);
      add_exact(d, dlo, f[32]);
      for (int b = 0; b < p.L; ++b) add_exact(d, dlo, (s >> b) & 1u ? f[b] : 0.0);
      const int col = c0 + c;
      const double sg = (double)p.sc[col], q0 = sg * d;
      double q = q0, qlo = fma(sg, d, -q0) + sg * dlo;
      add_exact(q, qlo, (double)p.sc[p.nb + col]);
      S.dg[j].x[c] = (T)(q + qlo);
    }
  }
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int q = threadIdx.x + kResThreads * j;
    const int64_t r = row0 + q;
    const bool valid = r < row1;
    // a table of fewer rows a thread than this kernel's leaves the rest idle
    const bool have = j < p.R;
    const uint32_t* e =
        p.slot + ((int64_t)m * p.R + (have ? j : 0)) * (p.nl + p.nh + 1) * kResThreads + threadIdx.x;
#pragma unroll
    for (int b = 0; b < NL; ++b) {
      const uint32_t x = have && b < p.nl ? e[(int64_t)b * kResThreads] : kResNone;
      const uint32_t o = (x == kResNone ? zero : x) * RB;  // below 2^16
      S.loc[j][b / 2] = b % 2 ? S.loc[j][b / 2] | o << 16 : o;
    }
    int nfar = 0;
#pragma unroll
    for (int b = 0; b < NH; ++b) {
      const uint32_t x = have && b < p.nh ? e[(int64_t)(p.nl + b) * kResThreads] : kResNone;
      S.far[j][b] = x == kResNone ? kNoRow : (x & ~kResFar) * RB;
      if (__ballot(x != kResNone)) nfar = b + 1;
    }
    S.nfar[j] = uniform(nfar);
    if (p.sep) {  // far targets keep their mark
      const uint32_t x = have ? e[(int64_t)(p.nl + p.nh) * kResThreads] : kResNone;
      S.per[j] = x == kResNone ? zero * RB : (x & kResFar) ? kResFar | (x & ~kResFar) * RB : x * RB;
    }
#pragma unroll
    for (int c = 0; c < G; ++c) {
      const int64_t col = c0 + c;
      S.v[j].x[c] = !valid ? T(0) : p.v ? p.v[col * p.D + r] : T(r == col);
    }
    const uint32_t off = valid ? (uint32_t)r * RB : kNoRow;
    S.b1[j] = rload<T, G>(cur, off);
    S.b2[j] = rload<T, G>(prev, no_prev ? kNoRow : off);
    if (valid) *reinterpret_cast<Cols<T, G>*>(s_b + (uint32_t)q * RB) = S.b1[j];
  }
  __syncthreads();
}

// Wave-uniform value of lane i of a register.
template <typename T>
__device__ __forceinline__ T lane_value(T x, int i) {
  if constexpr (sizeof(T) == 8) {
    int w[2];
    __builtin_memcpy(w, &x, 8);
    w[0] = __builtin_amdgcn_readlane(w[0], i);
    w[1] = __builtin_amdgcn_readlane(w[1], i);
    __builtin_memcpy(&x, w, 8);
  } else {
    int w;
    __builtin_memcpy(&w, &x, 4);
    w = __builtin_amdgcn_readlane(w, i);
    __builtin_memcpy(&x, &w, 4);
  }
  return x;
}

// Sums of the wave's x[0..n) over its lanes, value k in lane k * 64 / n
// (n a power of two): each step halves the values a lane carries until one is
// left, so 2 values take 6 exchanges instead of 12.
template <int n>
__device__ __forceinline__ double wave_sums(double (&x)[n]) {
  const int lane = threadIdx.x & 63;
  int off = 32;
#pragma unroll
  for (int m = n; m > 1; m /= 2, off /= 2) {
    const bool up = lane & off;
#pragma unroll
    for (int k = 0; k < m / 2; ++k) {
      const double give = up ? x[k] : x[k + m / 2];
      const double keep = up ? x[k + m / 2] : x[k];
      x[k] = keep + __shfl_xor(give, off, 64);
    }
  }
  for (; off > 0; off /= 2) x[0] += __shfl_xor(x[0], off, 64);
  return x[0];
}

// MOM: the Chebyshev vectors t_0 = v, t_1 = H~ t_0, t_{n+1} = 2 H~ t_n -
// t_{n-1} instead of the filter (no coefficients), n = i_top - i steps of the
// launch done after step i, with the product <t_0|t_n> of each step: a wave's sums go to
// part[n][column][slab][wave] while the team's other members reach the barrier.
template <typename T, int NL, int NH, int R, int G, bool MOM>
__device__ __forceinline__ void res_group(const ResArgs<T>& p, int c0, TeamView& tv,
                                          unsigned char* s_b, double* s_field, int* err) {
  constexpr uint32_t RB = G * sizeof(T);
  // Leaving out the slots that no lane of a wave uses gains 5-17% of a step
  // with 8-byte rows (L = 18: 3.9 -> 3.4 us); with 16-byte rows or six rows a
  // thread the branches cost more registers than the loads time (L = 18, 13
  // columns: 5.4 -> 6.3 us).
  constexpr bool skip = RB == 8 && R <= 3;
  const int64_t D = p.D;
  const int nslab = p.nslab;
  const bool lda1 = p.lda == 1;  // the same coefficients for every column
  if (threadIdx.x < G * kFieldStride)
    s_field[threadIdx.x] =
        p.fields[p.field_cols > 1 ? (int64_t)c0 * kFieldStride + threadIdx.x
                                  : threadIdx.x % kFieldStride];
  if (threadIdx.x < RB / 4)
    reinterpret_cast<uint32_t*>(s_b + (uint32_t)p.rows_cap * RB)[threadIdx.x] = 0;
  T* cur = p.X + (int64_t)c0 * D;
  T* prev = p.Y + (int64_t)c0 * D;
  if (p.first) {  // b_K = a_K v
    for (int m = tv.rank; m < nslab; m += tv.n)
      for (int64_t r = slab_row(D, nslab, m) + threadIdx.x; r < slab_row(D, nslab, m + 1);
           r += kResThreads)
#pragma unroll
        for (int c = 0; c < G; ++c)
          cur[r * G + c] = (MOM ? T(1) : p.A[(int64_t)p.i_top * p.lda + (lda1 ? 0 : c0 + c)]) *
                           (p.v ? p.v[(int64_t)(c0 + c) * D + r] : T(r == c0 + c));
  }
  team_barrier(tv, err, [] {});
  SlabState<T, NL, NH, R, G> S;
  const bool one = tv.n >= nslab;  // one slab a member: its state is kept
  // hop amplitudes with the column's scale
  T ht[G], hb[G], acf[G];
#pragma unroll
  for (int c = 0; c < G; ++c) {
    const T sg = p.sc[c0 + c];
    ht[c] = sg * (T)p.t_in;
    hb[c] = sg * (T)p.t_pb;
  }
  const int lane = threadIdx.x & 63;
  int row0 = (int)slab_row(D, nslab, tv.rank);
  int rows = (int)slab_row(D, nslab, tv.rank + 1) - row0;
  for (int i = p.i_top - 1; i >= p.i_bot; --i) {
    const bool last = !MOM && i == 0;
    const T half = (MOM ? p.first && i == p.i_top - 1 : last) ? T(0.5) : T(1);
    // 64 steps' coefficients at a time, one a lane
    const int ci = (p.i_top - 1 - i) & 63;
    if (!MOM && ci == 0)
#pragma unroll
      for (int c = 0; c < G; ++c) acf[c] = p.A[(int64_t)max(i - lane, 0) * p.lda + (lda1 ? 0 : c0 + c)];
    T ai[G];
#pragma unroll
    for (int c = 0; c < G; ++c) ai[c] = MOM ? T(0) : lane_value(acf[c], ci);
    double dots[G] = {};
    auto flush = [&](int m) {  // this wave's sums over the rows of slab m
      const double s = wave_sums<G>(dots);
      const int k = lane / (64 / G);  // column k
      if (lane % (64 / G) == 0)
        p.part[(((int64_t)p.i_all - i) * p.nb + c0 + k) * nslab * kResWaves + m * kResWaves +
               (threadIdx.x >> 6)] = s;
#pragma unroll
      for (int q = 0; q < G; ++q) dots[q] = 0;
    };
    const bool bad = last && res_load(err) != 0;
    const rsrc_t rc = make_rsrc(cur, (uint32_t)(D * RB));
    const rsrc_t ro = make_rsrc(prev, (uint32_t)(D * RB));
    // a team of one with one slab exchanges nothing until the chunk's end
    const bool store = nslab > 1 || i <= p.i_bot + 1;
    for (int m = tv.rank; m < nslab; m += tv.n) {
      if (!one) {
        __syncthreads();  // the slab before: its LDS reads are done
        row0 = (int)slab_row(D, nslab, m);
        rows = (int)slab_row(D, nslab, m + 1) - row0;
      }
      if (!one || i == p.i_top - 1)
        res_setup<T, NL, NH, R, G>(p, S, c0, m, s_field, rc, ro, p.first && i == p.i_top - 1, s_b);
#pragma unroll
      for (int j = 0; j < R; ++j) {
        // the hops that leave the slab on their way while the others are summed
        Cols<T, G> g[NH > 0 ? NH : 1], x[NL];
#pragma unroll
        for (int b = 0; b < NH; ++b)
          if (!skip || b < S.nfar[j]) g[b] = rload<T, G>(rc, S.far[j][b]);
#pragma unroll
        for (int b = 0; b < NL; ++b)
          x[b] = lread<T, G>(s_b, b % 2 ? S.loc[j][b / 2] >> 16 : S.loc[j][b / 2] & 0xFFFFu);
        Cols<T, G> acc{}, hp{};
#pragma unroll
        for (int b = 0; b < NL; ++b)
#pragma unroll
          for (int c = 0; c < G; ++c) acc.x[c] += x[b].x[c];
        if (p.sep) {
          const uint32_t o = S.per[j];
          hp = (o & kResFar) ? rload<T, G>(rc, o & ~kResFar) : lread<T, G>(s_b, o);
        }
#pragma unroll
        for (int b = 0; b < NH; ++b)
          if (!skip || b < S.nfar[j]) {
#pragma unroll
            for (int c = 0; c < G; ++c) acc.x[c] += g[b].x[c];
          }
        Cols<T, G> o;
#pragma unroll
        for (int c = 0; c < G; ++c)
          o.x[c] = half * (S.dg[j].x[c] * S.b1[j].x[c] + ht[c] * acc.x[c] + hb[c] * hp.x[c]) -
                   S.b2[j].x[c] + (MOM ? T(0) : ai[c] * S.v[j].x[c]);
        if constexpr (MOM) {  // a row past the slab's end is 0 throughout
#pragma unroll
          for (int c = 0; c < G; ++c) dots[c] += (double)S.v[j].x[c] * (double)o.x[c];
        }
        const int q = threadIdx.x + kResThreads * j;
        if (q < rows) {
          if (last) {
#pragma unroll
            for (int c = 0; c < G; ++c)
              p.w[(int64_t)(c0 + c) * D + row0 + q] = bad ? T(NAN) : o.x[c];
          } else if (store) {
            rstore<T, G>(o, ro, (uint32_t)(row0 + q) * RB);
          }
        }
        S.b2[j] = S.b1[j];
        S.b1[j] = o;
      }
      if (MOM && !one) flush(m);
    }
    if (last) break;
    team_barrier(tv, err, [&] {
      if (!one) return;
      if (MOM) flush(tv.rank);
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const int q = threadIdx.x + kResThreads * j;
        if (q < rows) *reinterpret_cast<Cols<T, G>*>(s_b + (uint32_t)q * RB) = S.b1[j];
      }
    });
    T* t = cur;
    cur = prev;
    prev = t;
  }
}

template <typename T, int NL, int NH, int R, bool MOM>
__global__ __launch_bounds__(kResThreads) void k_chain_res(ResArgs<T> p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ double s_field[2 * kFieldStride];
  __shared__ int s_join[4], s_fail;
  TeamView tv{nullptr, 1, 0, 0, 0, p.wait, &s_fail};
  // all columns' rows, as the ones that are this member's are not known
  auto give_up = [&] {
    if (!MOM) poison(p.w, p.D * p.nb);  // moments: err fails the call
  };
  if (!team_join(p.st, p.nslab, p.teams_per_xcd, s_join, tv, p.home,
                 p.ngrp == 1 ? p.i_top - p.i_bot : 0)) {
    if (s_fail) give_up();
    return;
  }
  for (int round = 0;; ++round) {
    if (threadIdx.x == 0 && tv.rank == 0) {
      const int g = res_add(&p.st->queue, 1);
      if (tv.n > 1)
        res_store(&tv.t->group[round & 1], g);
      else
        s_join[3] = g;
    }
    team_barrier(tv, &p.st->err, [] {});
    if (s_fail) {
      give_up();
      return;
    }
    const int g = uniform(tv.n > 1 ? res_load(&tv.t->group[round & 1]) : s_join[3]);
    if (g >= p.ngrp) return;
    // pairs of columns first, then single ones
    if constexpr (R <= kResMaxPairRows) {
      if (g < p.pairs)
        res_group<T, NL, NH, R, 2, MOM>(p, 2 * g, tv, smem, s_field, &p.st->err);
      else
        res_group<T, NL, NH, R, 1, MOM>(p, p.pairs + g, tv, smem, s_field, &p.st->err);
    } else {
      res_group<T, NL, NH, R, 1, MOM>(p, g, tv, smem, s_field, &p.st->err);
    }
    __syncthreads();
  }
}

// The quantum sun: row = dot state << L | outer bits.  A slab fixes the top
// outer bits, so the whole dot matrix and the rays of the other outer spins
// stay inside it; a ray of a top spin gathers from another slab, at the same
// place for all lanes but the bit.  A thread holds DG dot states of one
// setting of the slab's outer bits (ITEMS settings), so the ND values of a
// setting are read once for DG rows; ND <= 8 keeps the thread's rows of the
// dot matrix in registers (ND = 0: any size, read from LDS).  At 3 + 13 spins
// (FP64) a step takes 4.4 us, 7.6 as a launch: the barrier and the gathers'
// round trip about 2, 1.3 the 2.6 MB that the five top rays gather from one
// XCD's L2, 0.9 the LDS reads.
template <typename T>
struct QsunRes {
  QsunDev q;
  int sbits, i_top, i_bot, first;
  T sigma, tau;
  const T *A, *v;
  T *w, *X, *Y;
  ResState* st;
  int home;
  long long wait;
};

constexpr int kQsunSlabBits = 5;
constexpr int kDenseMaxRows = 2048;  // of a filter applied as a matrix

template <typename T, int DG, int ITEMS, int ND>
__global__ __launch_bounds__(kResThreads) void k_qsun_res(QsunRes<T> p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int s_join[4], s_fail;
  __shared__ T s_amp[kQsunMaxL];
  constexpr uint32_t TB = sizeof(T);
  const int L = p.q.L, nd = 1 << p.q.N, nslab = 1 << p.sbits;
  const int lo = L - p.sbits, nob = 1 << lo;  // outer bits inside a slab
  TeamView tv{nullptr, 1, 0, 0, 0, p.wait, &s_fail};
  if (!team_join(p.st, nslab, 1, s_join, tv, p.home, p.i_top - p.i_bot)) {
    if (s_fail) poison(p.w, p.q.D);
    return;
  }
  // the first team takes the column
  if (threadIdx.x == 0 && tv.rank == 0) {
    const int g = res_add(&p.st->queue, 1);
    if (tv.n > 1)
      res_store(&tv.t->group[0], g);
    else
      s_join[3] = g;
  }
  int* err = &p.st->err;
  team_barrier(tv, err, [] {});
  if (uniform(tv.n > 1 ? res_load(&tv.t->group[0]) : s_join[3]) > 0) return;
  T* s_b = reinterpret_cast<T*>(smem);           // [nd][nob]
  T* s_h = s_b + ((size_t)nd << lo);             // [nd][nd], scaled
  for (int i = threadIdx.x; i < nd * nd; i += kResThreads) s_h[i] = (T)(p.sigma * p.q.hdot[i]);
  if ((int)threadIdx.x < L) s_amp[threadIdx.x] = (T)(p.sigma * p.q.ray_amp[threadIdx.x]);
  T* cur = p.X;
  T* prev = p.Y;
  const int64_t D = p.q.D;
  const int items = (nd / DG) << lo;
  auto row = [&](int m, int d, int o) { return ((uint32_t)d << L) | ((uint32_t)m << lo) | (uint32_t)o; };
  if (p.first) {
    const T a = p.A[p.i_top];
    for (int m = tv.rank; m < nslab; m += tv.n)
      for (int i = threadIdx.x; i < (nd << lo); i += kResThreads) {
        const uint32_t r = row(m, i >> lo, i & (nob - 1));
        cur[r] = a * p.v[r];
      }
  }
  team_barrier(tv, err, [] {});
  T h[ITEMS][DG][ND > 0 ? ND : 1], v[ITEMS][DG], b1[ITEMS][DG], b2[ITEMS][DG], dg[ITEMS], acf = 0;
  const bool one = tv.n >= nslab;
  const int lane = threadIdx.x & 63;
  for (int i = p.i_top - 1; i >= p.i_bot; --i) {
    const bool last = i == 0;
    const T half = last ? T(0.5) : T(1);
    const int ci = (p.i_top - 1 - i) & 63;
    if (ci == 0) acf = p.A[max(i - lane, 0)];
    const T ai = lane_value(acf, ci);
    const bool bad = last && res_load(err) != 0;
    const bool store = nslab > 1 || i <= p.i_bot + 1;
    const rsrc_t rc = make_rsrc(cur, (uint32_t)(D * TB)), ro = make_rsrc(prev, (uint32_t)(D * TB));
    for (int m = tv.rank; m < nslab; m += tv.n) {
      if (!one) __syncthreads();  // the slab before: its LDS reads are done
      if (!one || i == p.i_top - 1) {
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) {
          const int it = threadIdx.x + kResThreads * t, o = it & (nob - 1), d0 = (it >> lo) * DG;
          const bool valid = it < items;
          const uint32_t ob = ((uint32_t)m << lo) | (uint32_t)o;
          const double* f = p.q.ftab;
          const double fs = f[ob & 255u] + f[256 + ((ob >> 8) & 255u)] +
                            f[512 + ((ob >> 16) & 255u)] + f[768 + (ob >> 24)];
          dg[t] = (T)(p.sigma * (p.q.c0 + fs) + p.tau);
#pragma unroll
          for (int d = 0; d < DG; ++d) {
            const uint32_t r = valid ? row(m, d0 + d, o) : 0u, off = valid ? r * TB : kNoRow;
            v[t][d] = valid ? p.v[r] : T(0);
            b1[t][d] = rload<T, 1>(rc, off).x[0];
            b2[t][d] = rload<T, 1>(ro, p.first && i == p.i_top - 1 ? kNoRow : off).x[0];
            if (valid) s_b[((d0 + d) << lo) + o] = b1[t][d];
            if constexpr (ND > 0) {
#pragma unroll
              for (int e = 0; e < ND; ++e) h[t][d][e] = valid ? s_h[(d0 + d) * ND + e] : T(0);
            }
          }
        }
        __syncthreads();
      }
#pragma unroll
      for (int t = 0; t < ITEMS; ++t) {
        const int it = threadIdx.x + kResThreads * t, o = it & (nob - 1), d0 = (it >> lo) * DG;
        const bool valid = it < items;
        const int dv = valid ? d0 : 0;
        T acc[DG];
#pragma unroll
        for (int d = 0; d < DG; ++d) acc[d] = dg[t] * b1[t][d];
        // rays of the top outer spins on their way from other slabs
        T x[kQsunSlabBits][DG];
#pragma unroll
        for (int u = 0; u < kQsunSlabBits; ++u)
#pragma unroll
          for (int d = 0; d < DG; ++d)
            x[u][d] = rload<T, 1>(rc, valid && u < p.sbits
                                          ? (row(m, d0 + d, o) ^ p.q.ray_mask[min(lo + u, L - 1)]) * TB
                                          : kNoRow).x[0];
        // meanwhile the dot matrix and the rays inside the slab
        if constexpr (ND > 0) {
          T y[ND];
#pragma unroll
          for (int e = 0; e < ND; ++e) y[e] = s_b[(e << lo) + o];
#pragma unroll
          for (int d = 0; d < DG; ++d)
#pragma unroll
            for (int e = 0; e < ND; ++e) acc[d] += h[t][d][e] * y[e];
        } else {
#pragma unroll 4
          for (int e = 0; e < nd; ++e) {
            const T y = s_b[(e << lo) + o];
#pragma unroll
            for (int d = 0; d < DG; ++d) acc[d] += s_h[(dv + d) * nd + e] * y;
          }
        }
#pragma unroll 4
        for (int k = 0; k < lo; ++k) {
          const int dm = (int)(p.q.ray_mask[k] >> L);
          const T am = s_amp[k];
          const int oo = o ^ (1 << k);
#pragma unroll
          for (int d = 0; d < DG; ++d) acc[d] += am * s_b[(((dv + d) ^ dm) << lo) + oo];
        }
#pragma unroll
        for (int u = 0; u < kQsunSlabBits; ++u) {
          const T am = s_amp[min(lo + u, L - 1)];
#pragma unroll
          for (int d = 0; d < DG; ++d) acc[d] += am * x[u][d];
        }
#pragma unroll
        for (int d = 0; d < DG; ++d) {
          const T out = half * acc[d] - b2[t][d] + ai * v[t][d];
          if (valid) {
            const uint32_t r = row(m, d0 + d, o);
            if (last)
              p.w[r] = bad ? T(NAN) : out;
            else if (store)
              bstore<0>(out, ro, r * TB, 0);
          }
          b2[t][d] = b1[t][d];
          b1[t][d] = out;
        }
      }
    }
    if (last) break;
    team_barrier(tv, err, [&] {
      if (!one) return;
#pragma unroll
      for (int t = 0; t < ITEMS; ++t) {
        const int it = threadIdx.x + kResThreads * t, o = it & (nob - 1), d0 = (it >> lo) * DG;
#pragma unroll
        for (int d = 0; d < DG; ++d)
          if (it < items) s_b[((d0 + d) << lo) + o] = b1[t][d];
      }
    });
    T* t = cur;
    cur = prev;
    prev = t;
  }
}

// Clears the team state (see res_clears) and writes a chunk's coefficients
// (kernel arguments, so that the call can be captured and needs no copy from
// host memory).
template <typename T>
struct CoefPack {
  static constexpr int kN = 440;
  T a[kN];
};
template <typename T>
__global__ __launch_bounds__(256) void k_res_begin(ResState* st, int first, T* sc, T sigma, T tau,
                                                   int nb) {
  int* p = reinterpret_cast<int*>(st);
  for (int i = blockIdx.x * 256 + threadIdx.x; i < (int)(sizeof(ResState) / 4);
       i += gridDim.x * 256)
    if (res_clears(i, first)) p[i] = 0;
  if (sc && blockIdx.x == 0)
    for (int c = threadIdx.x; c < nb; c += 256) {
      sc[c] = sigma;
      sc[nb + c] = tau;
    }
}
template <typename T>
__global__ __launch_bounds__(512) void k_res_coef(CoefPack<T> c, int n, T* out) {
  if ((int)threadIdx.x < n) out[threadIdx.x] = c.a[threadIdx.x];
}

// A[0 .. top - bot] = a[bot .. top]
template <typename T>
void put_coefs(hipStream_t s, const double* a, int bot, int top, T* A) {
  CoefPack<T> c;
  for (int i = bot; i <= top; i += CoefPack<T>::kN) {
    const int n = std::min(CoefPack<T>::kN, top - i + 1);
    for (int k = 0; k < n; ++k) c.a[k] = (T)a[i + k];
    hipLaunchKernelGGL((k_res_coef<T>), dim3(1), dim3(512), 0, s, c, n, A + (i - bot));
  }
  HIPC(hipGetLastError());
}

// An instantiation that covers a table.
bool res_instance(const ResTable& t) {
  if (t.nh == 0) return t.R <= 2 && t.nl <= 12;
  if (t.R <= 3) return t.nl <= 14 && t.nh <= 10;
  return t.nl <= 15 && t.nh <= 11;
}

template <typename T, bool MOM>
void res_launch(hipStream_t s, const ResTable& t, unsigned grid, size_t shm, const ResArgs<T>& a) {
  const dim3 g(grid), b(kResThreads);
#define POLFED_RES(NL_, NH_, R_)                                             \
  if (t.nl <= NL_ && t.nh <= NH_ && t.R <= R_) {                             \
    hipLaunchKernelGGL((k_chain_res<T, NL_, NH_, R_, MOM>), g, b, shm, s, a); \
    HIPC(hipGetLastError());                                                 \
    return;                                                                  \
  }
  POLFED_RES(12, 0, 1)
  POLFED_RES(12, 0, 2)
  POLFED_RES(10, 6, 1)
  POLFED_RES(14, 10, 1)
  POLFED_RES(14, 10, 2)
  POLFED_RES(14, 10, 3)
  POLFED_RES(15, 11, 6)
#undef POLFED_RES
  fail(POLFED_ERR_INVALID, "resident recurrence: no kernel for this table");
}

std::shared_ptr<ResTable> build_table(hipStream_t s, const polfed_op* op, int nslab) {
  TallyScope untallied(nullptr);  // lives as long as the pattern's operators
  auto t = std::make_shared<ResTable>();
  t->nslab = nslab;
  t->R = res_r(op->D, nslab);
  t->rows = res_rows(op->D, nslab);
  t->sep = op->periodic && op->t_pb != op->t_in ? 1 : 0;
  ResBuild b{};
  b.L = op->L;
  b.N = op->N;
  b.periodic = op->periodic;
  b.sep = t->sep;
  b.nslab = nslab;
  b.R = t->R;
  b.D = op->D;
  b.binom = op->d_binom.as<uint32_t>();
  DevBuf cnt(2 * sizeof(int32_t));
  b.counts = cnt.as<int32_t>();
  hipLaunchKernelGGL(k_res_fill, dim3(1), dim3(64), 0, s, (int64_t)2, 0u, cnt.as<uint32_t>());
  hipLaunchKernelGGL(k_res_build<false>, dim3((unsigned)nslab), dim3(kResThreads), 0, s, b);
  HIPC(hipGetLastError());
  int32_t h[2];
  HIPC(hipMemcpyAsync(h, cnt.get(), sizeof h, hipMemcpyDeviceToHost, s));
  HIPC(hipStreamSynchronize(s));
  t->nl = h[0];
  t->nh = h[1];
  // as many slots inside the slab as the instantiation reads anyway: more waves
  // then find room for every bond of their rows (FP64, us a step, packed by
  // lane / by bond: 13 columns at L = 18 5.15 / 4.70, 32 at L = 17 5.15 / 4.75;
  // the same where the barrier counts).  More slots out of the slab would be
  // more loads.
  if (t->nh == 0 && t->R <= 2 && t->nl <= 12) {
    t->nl = 12;
  } else if (t->R == 1 && t->nl <= 10 && t->nh <= 6) {
    t->nl = 10;
  } else if (t->R <= 3 && t->nl <= 14 && t->nh <= 10) {
    t->nl = 14;
  } else if (t->nl <= 15 && t->nh <= 11) {
    t->nl = 15;
  }
  b.nl = t->nl;
  b.nh = t->nh;
  const size_t n = (size_t)nslab * t->R * (t->nl + t->nh + 1) * kResThreads;
  t->slot.alloc(n * sizeof(uint32_t));
  t->state.alloc((size_t)op->D * sizeof(uint32_t));
  b.slot = t->slot.as<uint32_t>();
  b.state = t->state.as<uint32_t>();
  hipLaunchKernelGGL(k_res_fill, dim3(256), dim3(256), 0, s, (int64_t)n, kResNone, b.slot);
  hipLaunchKernelGGL(k_res_build<true>, dim3((unsigned)nslab), dim3(kResThreads), 0, s, b);
  HIPC(hipGetLastError());
  HIPC(hipStreamSynchronize(s));
  return t;
}

// The table of op's pattern for this many slabs: shared by the operators of
// the pattern on the context, freed with the last of them.  One that op does
// not hold yet is looked up and built only with `build`, and not while the
// stream is captured (null then).
std::shared_ptr<ResTable> res_table(hipStream_t s, const polfed_op* op, int nslab, bool build) {
  polfed_ctx* ctx = op->ctx;
  const std::string key = op->pattern_key + "|" + std::to_string(nslab);
  std::lock_guard<std::mutex> lk(ctx->tune_mu);
  auto& mine = op->res_tables[nslab];
  if (mine || !build) return mine;
  auto& shared = ctx->res_tables[key];
  if ((mine = shared.lock())) return mine;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  HIPC(hipStreamIsCapturing(s, &cs));
  if (cs != hipStreamCaptureStatusNone) return nullptr;
  for (auto it = ctx->res_tables.begin(); it != ctx->res_tables.end();)
    it = it->second.expired() && it->first != key ? ctx->res_tables.erase(it) : std::next(it);
  mine = build_table(s, op, nslab);
  ctx->res_tables[key] = mine;
  return mine;
}

bool res_chain(const polfed_op* op) {
  return op->model == Model::Chain && op->storage == POLFED_MATRIX_FREE && op->split_nseg > 0 &&
         op->L <= kResMaxL && op->D >= 1 && !op->pattern_key.empty();
}

// One chunk after another of a recurrence of order K; put supplies the
// coefficients A of a chunk's steps (and clears the state), done(top, bot)
// follows its launch.
template <bool MOM = false, typename T, class Put, class Done>
void res_run(hipStream_t s, const ResTable& t, const ResShape& x, ResArgs<T> a, int K, int chunk,
             Put&& put, Done&& done) {
  a.sep = t.sep;
  a.nslab = t.nslab;
  a.R = t.R;
  a.nl = t.nl;
  a.nh = t.nh;
  a.rows_cap = t.rows;
  a.slot = t.slot.template as<uint32_t>();
  a.state = t.state.template as<uint32_t>();
  a.pairs = x.pairs;
  a.ngrp = x.ngrp;
  a.teams_per_xcd = t.nslab == 1 ? 1 : std::min(x.teams / 8, (x.ngrp + 7) / 8);
  const unsigned grid = t.nslab == 1 ? (unsigned)std::min(x.ngrp, 1024)
                                     : (unsigned)(8 * a.teams_per_xcd * t.nslab);
  const size_t shm = ((size_t)(t.rows + 1) * (x.pairs ? 2 : 1) * sizeof(T) + 15) / 16 * 16;
  // columns on every XCD, side by side with another such launch 2 to 6 times
  // slower than one after the other (four contexts, 13 columns at L = 18 each:
  // 231 to 400 ms, 58)
  int dev = 0;
  HIPC(hipGetDevice(&dev));
  std::optional<WholeDevice> whole;
  if (x.ngrp > 1 && !res_shares(x)) whole.emplace(dev, s);
  for (int top = K; top > 0;) {
    const int bot = std::max(0, top - chunk);
    a.i_top = top;
    a.i_bot = bot;
    a.first = top == K;
    put(a, top, bot);
    res_launch<T, MOM>(s, t, grid, shm, a);
    done(top, bot);
    if ((top - bot) % 2) std::swap(a.X, a.Y);
    top = bot;
  }
}
template <bool MOM = false, typename T, class Put>
void res_run(hipStream_t s, const ResTable& t, const ResShape& x, const ResArgs<T>& a, int K,
             int chunk, Put&& put) {
  res_run<MOM>(s, t, x, a, K, chunk, put, [](int, int) {});
}

}  // namespace

// A single column: where a thread holds at most three rows (D <= 49,152).
// With six rows a step takes 7.7 us, more than a launch of the step kernel.
static bool chain_res_applies(const polfed_op* op, bool fp32) {
  if (!res_chain(op) || op->forced[fp32 ? 1 : 0]) return false;
  return res_shape(op->D, 1).R <= 3 && res_shape(op->D, 1).nslab > 0;
}

void chain_res_prepare(hipStream_t s, const polfed_op* op, bool fp32) {
  if (chain_res_applies(op, fp32)) (void)res_table(s, op, res_shape(op->D, 1).nslab, true);
}

template <typename T>
static bool chain_res_filter(hipStream_t s, const polfed_op* op, double E_c, double dE,
                             const double* a, int K, const T* v, T* w, T* bufA, T* bufB,
                             void* tail) {
  if (K < kResMinSteps || !chain_res_applies(op, sizeof(T) == 4)) return false;
  const ResShape x = res_shape(op->D, 1);
  if (g_shared_device && !res_shares(x)) return false;
  const auto t = res_table(s, op, x.nslab, false);
  if (!t || !res_instance(*t)) return false;
  const uintptr_t p = res_align(tail ? (uintptr_t)tail : (uintptr_t)(bufA + op->D));
  ResState* st = (ResState*)(p + ResTail::st);
  T* sc = (T*)(p + ResTail::sc);
  T* A = (T*)(p + ResTail::A);
  ResArgs<T> r{};
  r.L = op->L;
  r.N = op->N;
  r.periodic = op->periodic;
  r.nb = 1;
  r.field_cols = 1;
  r.lda = 1;
  r.D = op->D;
  r.t_in = op->t_in;
  r.t_pb = op->t_pb;
  r.vzz = op->vzz;
  r.fields = op->fields();
  r.sc = sc;
  r.v = v;
  r.w = w;
  r.X = bufA;
  r.Y = bufB;
  r.st = st;
  r.wait = op->ctx->team_wait;
  r.home = op->ctx->home;
  const T sigma = (T)(2.0 / dE), tau = (T)(-2.0 * E_c / dE);
  res_run<false>(s, *t, x, r, K, kResChunk, [&](ResArgs<T>& q, int top, int bot) {
    hipLaunchKernelGGL((k_res_begin<T>), dim3(8), dim3(256), 0, s, st, q.first, sc, sigma, tau, 1);
    put_coefs<T>(s, a, bot, top, A);
    q.A = A - bot;  // indexed by the step
  });
  return true;
}

// Quantum sun: slabs so that a thread has one item of DG rows, at most 32 of
// them, then a few items; single-workgroup up to 2,048 rows.  Where the line
// lies, us a step, resident / a launch a step: FP64 N = 3, L = 13 (one item)
// 4.6 / 7.8, N = 2, L = 15 (two) 8.3 / 9.1, N = 4, L = 13 (two) 9.4 / 9.2,
// N = 5, L = 12 (two) 11.6 / 10.7; FP32 N = 5, L = 12 (two) 9.6 / 17.6,
// N = 1, L = 16 (four) 7.8 / 12.8, N = 3, L = 15 (four) 14.7 / 13.8.
static int qsun_slab_bits(const polfed_op* op) {
  const int dg = std::min(2, op->N_dot);
  return std::max(0, std::min({op->N_dot + op->L - 9 - dg, kQsunSlabBits, op->L - 1}));
}
static int qsun_items(const polfed_op* op) {
  const int dg = std::min(2, op->N_dot);
  const int64_t n = (int64_t)1 << (op->N_dot + op->L - qsun_slab_bits(op) - dg);
  return (int)((n + kResThreads - 1) / kResThreads);
}
static bool qsun_res_applies(const polfed_op* op, bool fp32) {
  if (op->model != Model::Qsun || op->storage != POLFED_MATRIX_FREE) return false;
  const int most = fp32 ? (op->N_dot == 1 ? 4 : 2) : (op->N_dot <= 2 ? 2 : 1);
  return qsun_items(op) <= most;
}

bool res_applies(const polfed_op* op, bool fp32) {
  return chain_res_applies(op, fp32) || qsun_res_applies(op, fp32);
}

template <typename T>
bool res_filter(hipStream_t s, const polfed_op* op, double E_c, double dE, const double* a, int K,
                const T* v, T* w, T* bufA, T* bufB, void* tail) {
  if (chain_res_filter<T>(s, op, E_c, dE, a, K, v, w, bufA, bufB, tail)) return true;
  if (K < kResMinSteps || !qsun_res_applies(op, sizeof(T) == 4)) return false;
  if (g_shared_device && (1 << qsun_slab_bits(op)) > kResSharedPerXcd) return false;
  const int items = qsun_items(op), N = op->N_dot;
  QsunRes<T> r{};
  r.q = op->qsun();
  r.sbits = qsun_slab_bits(op);
  r.sigma = (T)(2.0 / dE);
  r.tau = (T)(-2.0 * E_c / dE);
  r.v = v;
  r.w = w;
  r.X = bufA;
  r.Y = bufB;
  const uintptr_t p = res_align(tail ? (uintptr_t)tail : (uintptr_t)(bufA + op->D));
  r.st = (ResState*)(p + ResTail::st);
  r.wait = op->ctx->team_wait;
  r.home = op->ctx->home;
  T* A = (T*)(p + ResTail::A);
  const unsigned grid = r.sbits ? 8u << r.sbits : 1u;
  const size_t nd = (size_t)1 << N;
  const size_t shm = ((nd << (op->L - r.sbits)) + nd * nd) * sizeof(T);
  for (int top = K; top > 0;) {
    const int bot = std::max(0, top - kResChunk);
    r.i_top = top;
    r.i_bot = bot;
    r.first = top == K;
    hipLaunchKernelGGL((k_res_begin<T>), dim3(8), dim3(256), 0, s, r.st, r.first, (T*)nullptr,
                       T(0), T(0), 0);
    put_coefs<T>(s, a, bot, top, A);
    r.A = A - bot;
#define POLFED_QSUN(DG_, IT_, ND_)                                                                \
  hipLaunchKernelGGL((k_qsun_res<T, DG_, IT_, ND_>), dim3(grid), dim3(kResThreads), shm, s, r)
    if (N == 1 && items == 1)
      POLFED_QSUN(2, 1, 2);
    else if (N == 2 && items == 1)
      POLFED_QSUN(4, 1, 4);
    else if (N == 3 && items == 1)
      POLFED_QSUN(4, 1, 8);
    else if (N == 3 && items == 2)
      POLFED_QSUN(4, 2, 8);
    else if (N == 1)
      POLFED_QSUN(2, 4, 0);
    else if (items == 1)
      POLFED_QSUN(4, 1, 0);
    else
      POLFED_QSUN(4, 2, 0);
#undef POLFED_QSUN
    HIPC(hipGetLastError());
    if ((top - bot) % 2) std::swap(r.X, r.Y);
    top = bot;
  }
  return true;
}

// P(H~) as a matrix: its columns are the filter of the unit vectors, a batch
// that fills the chip, and an application is then one product with it.  A
// short chain's filter runs on one workgroup or one XCD however idle the rest
// of the chip is; at L = 12 (D = 924, K = 181) an application takes 195 us,
// the matrix of all 924 columns 0.79 ms and a product 3.4 to 4.7 us; at L = 13
// (D = 1,716, K = 489) 590 us against 9.3 ms and 8 us.  The error of an
// application is that of the columns, each a Clenshaw sum of the same order,
// weighted with v (norm of the error against an 80-bit evaluation, recurrence
// and matrix: L = 12 4.18e-16 and 4.20e-16, L = 13 4.43e-16 and 4.45e-16).
//
// It pays once a solve applies the filter more often than the batch takes in
// applications; M is the expected number of them, of which a solve that
// converges early uses somewhat more than half.  Solves, ms before and after:
// D = 252 8.7 and 6.3, D = 924 22.7 and 10.5, D = 1,716 40.3 and 18.8, D =
// 2,002 44.6 and 21.8; at D = 3,432 the columns would take 40 ms of the 51 that
// the applications take.  The matrix and the two buffers of its columns stay
// below 100 MB.
bool chain_dense_pays(const polfed_op* op, int K, int M) {
  if (K < kResMinSteps || op->D > kDenseMaxRows || !chain_res_applies(op, false)) return false;
  const ResShape all = res_shape(op->D, (int)op->D);
  return all.nslab > 0 && 0.5 * M * res_shape(op->D, 1).us > 2.0 * all.us;
}

size_t chain_dense_bytes(const polfed_op* op) {
  return sizeof(ResState) + 4096 + (2 * (size_t)op->D + kResChunk + 1) * sizeof(double);
}

// P: D x D; X, Y: its two buffers; ws: chain_dense_bytes.
bool chain_dense_build(hipStream_t s, const polfed_op* op, double E_c, double dE, const double* a,
                       int K, double* P, double* X, double* Y, void* ws) {
  const int nb = (int)op->D;
  const ResShape x = res_shape(op->D, nb);
  const auto t = res_table(s, op, x.nslab, true);
  if (!t || !res_instance(*t)) return false;
  ResState* st = (ResState*)ws;
  double* sc = (double*)((unsigned char*)ws + (sizeof(ResState) + 255) / 256 * 256);
  double* A = sc + 2 * nb;
  ResArgs<double> r{};
  r.L = op->L;
  r.N = op->N;
  r.periodic = op->periodic;
  r.nb = nb;
  r.field_cols = 1;
  r.lda = 1;
  r.D = op->D;
  r.t_in = op->t_in;
  r.t_pb = op->t_pb;
  r.vzz = op->vzz;
  r.fields = op->fields();
  r.sc = sc;
  r.w = P;
  r.X = X;
  r.Y = Y;
  r.st = st;
  r.wait = op->ctx->team_wait;
  r.home = op->ctx->home;
  res_run<false>(s, *t, x, r, K, kResChunk, [&](ResArgs<double>& q, int top, int bot) {
    hipLaunchKernelGGL((k_res_begin<double>), dim3(8), dim3(256), 0, s, q.st, q.first, sc,
                       2.0 / dE, -2.0 * E_c / dE, nb);
    put_coefs<double>(s, a, bot, top, A);
    q.A = A - bot;  // indexed by the step
  });
  return true;
}

// y_i = sum_j P[i D + j] x_j: a wave a row (P is symmetric to its rounding, so
// the row is read where the column lies, contiguous), the whole chip at work.
__global__ __launch_bounds__(256) void k_dense_mv(int D, const double* __restrict__ P,
                                                  const double* __restrict__ x,
                                                  double* __restrict__ y) {
  const int i = uniform((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if (i >= D) return;
  const int lane = threadIdx.x & 63;
  const double* row = P + (int64_t)i * D;
  double s0 = 0, s1 = 0;
  int j = lane;
#pragma unroll 8
  for (; j + 64 < D; j += 128) {
    s0 += row[j] * x[j];
    s1 += row[j + 64] * x[j + 64];
  }
  if (j < D) s0 += row[j] * x[j];
  s0 += s1;
  for (int off = 32; off > 0; off >>= 1) s0 += __shfl_down(s0, off, 64);
  if (lane == 0) y[i] = s0;
}

void chain_dense_apply(hipStream_t s, int64_t D, const double* P, const double* x, double* y) {
  hipLaunchKernelGGL(k_dense_mv, dim3((unsigned)((D + 3) / 4)), dim3(256), 0, s, (int)D, P, x, y);
  HIPC(hipGetLastError());
}

// ---- orthogonalization of a short vector in one launch ----

// w <- w - V (V^T w) over k1 basis vectors, twice, beta = ||w||, v_next =
// w / beta, by one team.  For short chains the eight launches that this takes
// otherwise last 40 us whatever they move (D = 924, k1 = 70: 0.5 MB a pass).
// V^T w is split by columns and V c by rows, so every sum lies in one member,
// in an order that does not depend on how many members the team got: virtual
// member m takes the columns m, m + nm, ... and the rows of slab m.  Four
// phases and the norm take five barriers of about 1 us; a pass reads V through
// one XCD's L2.  Measured, us a step with it, launches / this: D = 70, k1 = 30 30 / 20,
// D = 924, k1 = 100 54 / 27, D = 3,432, k1 = 150 88 / 40, k1 = 500 256 / 118.
constexpr int kOrthCols = 8;  // columns of V^T w at a time

__global__ __launch_bounds__(kResThreads) void k_cgs2_team(
    ResState* st, int64_t D, int k1, int nm, const double* V, double* w, double* c, double* norm,
    int* flag, double* alpha, double* beta, double* v_next) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int s_join[4], s_fail;
  __shared__ double s_red[kResWaves * 64];
  double* s_c = reinterpret_cast<double*>(smem);  // [k1]
  TeamView tv{nullptr, 1, 0, 0, 0, kResWait, &s_fail};
  if (!team_join(st, nm, 1, s_join, tv)) {
    if (s_fail) poison(v_next, D);
    return;
  }
  // the first team does it
  if (threadIdx.x == 0 && tv.rank == 0) {
    const int g = res_add(&st->queue, 1);
    if (tv.n > 1)
      res_store(&tv.t->group[0], g);
    else
      s_join[3] = g;
  }
  int* err = &st->err;
  team_barrier(tv, err, [] {});
  if (uniform(tv.n > 1 ? res_load(&tv.t->group[0]) : s_join[3]) > 0) return;
  const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
  const rsrc_t rw = make_rsrc(w, (uint32_t)(D * 8)), rc = make_rsrc(c, (uint32_t)(k1 * 8)),
               rn = make_rsrc(norm, (uint32_t)(nm * 8));
  double a0 = 0;
  for (int pass = 0; pass < 2; ++pass) {
    // c = V^T w, columns m, m + nm, ...: the workgroup's threads share the rows
    for (int m = tv.rank; m < nm; m += tv.n)
      for (int q0 = 0; m + q0 * nm < k1; q0 += kOrthCols) {
        double acc[kOrthCols] = {};
#pragma unroll 2
        for (int64_t r = threadIdx.x; r < D; r += kResThreads) {
          const double wr = bload<double, kAuxAgent>(rw, (uint32_t)(r * 8), 0);
#pragma unroll
          for (int q = 0; q < kOrthCols; ++q) {
            const int j = m + (q0 + q) * nm;
            if (j < k1) acc[q] += V[r + (int64_t)j * D] * wr;
          }
        }
        const double t = wave_sums<kOrthCols>(acc);
        __syncthreads();
        if (lane % (64 / kOrthCols) == 0) s_red[wave * kOrthCols + lane / (64 / kOrthCols)] = t;
        __syncthreads();
        const int j = m + (q0 + (int)threadIdx.x) * nm;
        if ((int)threadIdx.x < kOrthCols && j < k1) {
          double x = 0;
#pragma unroll
          for (int i = 0; i < kResWaves; ++i) x += s_red[i * kOrthCols + threadIdx.x];
          c[j] = x;
          if (j == k1 - 1) {  // adds up to the Lanczos alpha
            a0 += x;
            if (alpha && pass) alpha[0] = a0;
          }
        }
      }
    team_barrier(tv, err, [] {});
    for (int j = threadIdx.x; j < k1; j += kResThreads)
      s_c[j] = bload<double, kAuxAgent>(rc, (uint32_t)(j * 8), 0);
    __syncthreads();
    // w -= V c on the rows of slab m: a wave takes every eighth column
    for (int m = tv.rank; m < nm; m += tv.n) {
      const int64_t row0 = slab_row(D, nm, m), row1 = slab_row(D, nm, m + 1);
      double sq = 0;
      for (int64_t rb = row0; rb < row1; rb += 64) {
        const int64_t r = min(rb + lane, row1 - 1);
        double acc = 0;
#pragma unroll 8
        for (int j = wave; j < k1; j += kResWaves) acc += V[r + (int64_t)j * D] * s_c[j];
        s_red[threadIdx.x] = acc;
        __syncthreads();
        if (wave == 0) {
          double x = 0;
#pragma unroll
          for (int i = 0; i < kResWaves; ++i) x += s_red[64 * i + lane];
          const double y = bload<double, kAuxAgent>(rw, (uint32_t)(r * 8), 0) - x;
          if (rb + lane < row1) {
            w[r] = y;
            sq += y * y;
          }
        }
        __syncthreads();
      }
      if (pass == 1 && wave == 0) {
        for (int off = 32; off > 0; off >>= 1) sq += __shfl_down(sq, off, 64);
        if (lane == 0) norm[m] = sq;
      }
    }
    team_barrier(tv, err, [] {});
  }
  double b = bload<double, kAuxAgent>(rn, (uint32_t)(lane * 8), 0);  // 0 past the last
  for (int off = 32; off > 0; off >>= 1) b += __shfl_xor(b, off, 64);
  b = res_load(err) != 0 ? (double)NAN : sqrt(b);
  const bool ok = b > 1e-300 && isfinite(b);
  const double inv = ok ? 1.0 / b : isnan(b) && res_load(err) != 0 ? b : 0.0;
  if (tv.rank == 0 && threadIdx.x == 0) {
    beta[0] = b;
    if (!ok && flag) flag[0] = 1;
  }
  for (int m = tv.rank; m < nm; m += tv.n)
    for (int64_t r = slab_row(D, nm, m) + threadIdx.x; r < slab_row(D, nm, m + 1);
         r += kResThreads)
      v_next[r] = bload<double, kAuxAgent>(rw, (uint32_t)(r * 8), 0) * inv;
}

// Where it is the faster one.  Below 8,192 rows the launches leave most of the
// chip idle, and the line lies where one XCD's path to V is the longer one (D =
// 3,432: 1.7 M entries 256 us against 118); above, the middle two products go
// in one pass, and the line lies where V outgrows the XCD's L2 (D = 12,870:
// 0.4 M entries 85 against 47, 0.6 M 63 against 82).  With many rows and few
// columns the split by columns is the poor one (D = 24,310, k1 = 2: 52 against
// 69).
static bool orth_team(int64_t D, int k1) {
  return k1 >= 1 && k1 <= 4096 && D >= 1 && D <= 16384 &&
         D * k1 <= (D <= 8192 ? 2000 : 450) * 1000;
}

bool cgs2_team(hipStream_t s, int64_t D, int k1, const double* V, double* w, double* c,
               double* partial, int* flag, double* alpha, double* beta, double* v_next) {
  if (!orth_team(D, k1)) return false;
  // 32 members once a pass is longer than their barrier (0.21 M entries 38.0 us
  // with 16, 31.9; 10 k entries 21.4, 22.4; eight members are no faster there)
  const int nm = D * k1 > 100 * 1000 ? 32 : 16;
  // the team state and the norm's parts lie in the partial sums' 64 KB
  static_assert(sizeof(ResState) + 32 * sizeof(double) <= 8192 * sizeof(double), "partial");
  ResState* st = reinterpret_cast<ResState*>(partial);
  double* norm = reinterpret_cast<double*>(st + 1);
  hipLaunchKernelGGL((k_res_begin<double>), dim3(8), dim3(256), 0, s, st, 1, (double*)nullptr,
                     0.0, 0.0, 0);
  hipLaunchKernelGGL(k_cgs2_team, dim3(8 * nm), dim3(kResThreads), (size_t)k1 * sizeof(double), s,
                     st, D, k1, nm, V, w, c, norm, flag, alpha, beta, v_next);
  HIPC(hipGetLastError());
  return true;
}

template bool res_filter<double>(hipStream_t, const polfed_op*, double, double, const double*, int,
                                 const double*, double*, double*, double*, void*);
template bool res_filter<float>(hipStream_t, const polfed_op*, double, double, const double*, int,
                                const float*, float*, float*, float*, void*);

bool chain_res_batch_shares(const polfed_op* op0, int nb) {
  return res_shares(res_shape(op0->D, nb));
}

bool chain_res_batch_fits(hipStream_t s, const polfed_op* op0, int nb) {
  if (!res_chain(op0)) return false;
  const ResShape x = res_shape(op0->D, nb);
  if (x.nslab == 0) return false;
  const auto t = res_table(s, op0, x.nslab, true);
  return t && res_instance(*t);
}

// Variant 5 of a batch: every column's recurrence of order K (coefficients
// past a column's own order are zero, so its vectors stay zero until there).
template <typename T>
void chain_res_batch(hipStream_t s, const ChainBatch& bt, const T* A, int K, const T* v, T* w,
                     T* bufA, T* bufB) {
  const polfed_op* op0 = bt.ops[0];
  const ResShape x = res_shape(op0->D, bt.nb);
  const auto t = x.nslab ? res_table(s, op0, x.nslab, true) : nullptr;
  REQUIRE(t && res_instance(*t), "batch: no resident recurrence for this chain");
  ResArgs<T> r{};
  r.L = op0->L;
  r.N = op0->N;
  r.periodic = op0->periodic;
  r.nb = bt.nb;
  r.field_cols = bt.nb;
  r.lda = bt.nb;
  r.D = op0->D;
  r.t_in = op0->t_in;
  r.t_pb = op0->t_pb;
  r.vzz = op0->vzz;
  r.fields = bt.fields.template as<double>();
  r.sc = (const T*)(sizeof(T) == 8 ? bt.sc64.get() : bt.sc32.get());
  r.A = A;
  r.v = v;
  r.w = w;
  r.X = bufA;
  r.Y = bufB;
  r.st = bt.res_state.template as<ResState>();
  r.wait = op0->ctx->team_wait;
  r.home = bt.ctx->home;
  res_run<false>(s, *t, x, r, K, kResChunk, [&](ResArgs<T>& q, int, int) {
    hipLaunchKernelGGL((k_res_begin<T>), dim3(8), dim3(256), 0, s, q.st, q.first, (T*)nullptr,
                       T(0), T(0), 0);
    HIPC(hipGetLastError());
  });
}

// out[k] = sum of part[k * n .. k * n + n), one wave a sum; err = st->err.
__global__ __launch_bounds__(256) void k_res_sum(const double* part, int n, int64_t count,
                                                 const ResState* st, double* out, double* err) {
  if (blockIdx.x == 0 && threadIdx.x == 0) err[0] = st->err;
  const int64_t k = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (k >= count) return;
  double x = 0;
  for (int i = threadIdx.x & 63; i < n; i += 64) x += part[k * n + i];
  for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
  if ((threadIdx.x & 63) == 0) out[k] = x;
}

bool chain_res_moments_fit(hipStream_t s, const polfed_op* op, int width) {
  return !op->forced[0] && chain_res_batch_fits(s, op, width);
}

size_t chain_res_moments_bytes(const polfed_op* op, int M, int width) {
  return res_moments_plan(op->D, M, width, width).bytes;
}

// dots[n - 1] = <t_0|t_n> of every column for n = 1 .. M (host, [M][nb] and one
// more, used here); v: D x nb, X and Y: its two buffers; nb
// <= width columns, ws chain_res_moments_bytes of the width.
void chain_res_moments(hipStream_t s, const polfed_op* op, double E_c, double dE, int M, int width,
                       int nb, const double* v, double* X, double* Y, const DevBuf& ws,
                       double* dots) {
  const ResMomentsPlan pl = res_moments_plan(op->D, M, width, nb);
  const ResShape& x = pl.shape;
  REQUIRE(x.nslab > 0 && pl.bytes <= ws.bytes(), "kpm: workspace of another width");
  const auto t = res_table(s, op, x.nslab, true);
  REQUIRE(t && res_instance(*t), "kpm: no resident recurrence for this chain");
  unsigned char* base = ws.as<unsigned char>();
  ResState* st = (ResState*)base;
  double* sc = (double*)(base + pl.sc);
  double* sums = (double*)(base + pl.sums);
  const int64_t count = pl.count;
  ResArgs<double> r{};
  r.L = op->L;
  r.N = op->N;
  r.periodic = op->periodic;
  r.nb = nb;
  r.field_cols = 1;
  r.lda = nb;
  r.D = op->D;
  r.t_in = op->t_in;
  r.t_pb = op->t_pb;
  r.vzz = op->vzz;
  r.fields = op->fields();
  r.sc = sc;
  r.v = v;
  r.X = X;
  r.Y = Y;
  r.st = st;
  r.wait = op->ctx->team_wait;
  r.home = op->ctx->home;
  r.part = (double*)(base + pl.part);
  res_run<true>(
      s, *t, x, r, M, kResMomentSteps,
      [&](ResArgs<double>& q, int top, int) {
        q.i_all = top - 1;
        hipLaunchKernelGGL((k_res_begin<double>), dim3(8), dim3(256), 0, s, q.st, q.first, sc,
                           2.0 / dE, -2.0 * E_c / dE, nb);
        HIPC(hipGetLastError());
      },
      [&](int top, int bot) {
        const int64_t n = (int64_t)(top - bot) * nb;
        hipLaunchKernelGGL(k_res_sum, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, r.part,
                           t->nslab * kResWaves, n, st, sums + (int64_t)(M - top) * nb,
                           sums + count);
        HIPC(hipGetLastError());
      });
  HIPC(hipMemcpyAsync(dots, sums, (size_t)(count + 1) * sizeof(double), hipMemcpyDeviceToHost, s));
  HIPC(hipStreamSynchronize(s));
  if (dots[count] != 0)
    fail(POLFED_ERR_HIP, "kpm: a barrier of the resident recurrence gave up (device without progress?)");
}

template void chain_res_batch<double>(hipStream_t, const ChainBatch&, const double*, int,
                                      const double*, double*, double*, double*);
template void chain_res_batch<float>(hipStream_t, const ChainBatch&, const float*, int,
                                     const float*, float*, float*, float*);

}  // namespace polfed
