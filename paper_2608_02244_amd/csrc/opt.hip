// Exact alpha-fair optimum makespan for tiny instances (n <= 8): one wavefront
// per instance.
//
// Definition (Appendix A's integer program, with release steps and the KV
// budget added): the least makespan over start vectors with s_i >= r_i, at most
// B jobs active per step, reservations within M_kv unless a job runs alone, and
// |s_i - s_j| <= alpha for every pair active at a common step.
//
// Search.  Schedules are enumerated in start order: after placing a job at
// step sigma, the future depends only on (placed set, sigma clipped to the last
// release, progress of every job still active at sigma), because later jobs
// start at or after sigma and jobs that ended before sigma constrain nothing.
// From such a state the next job k starts after a delay d >= 0, bounded by the
// step at which the machine is empty and every job has been released (waiting
// longer with an empty machine can be removed by shifting the rest earlier).
// Among identical unstarted jobs only the lowest index may start next.
// V(state) = min over (k, d) of d + V(child) is computed by a depth-first
// search (depth <= n) whose memo keeps, per state, either the exact value or a
// lower bound, so a child is explored with the bound "best so far - d" and
// children whose lower bound d + LB(child) cannot beat it are skipped
// (LB = max of: longest remaining active job, latest finish of an unstarted job
// if started at once, total remaining work / B).  The root bound is the ISJL
// makespan of the instance (written into T_opt by a simulation launch just
// before this kernel): the search returns a smaller value only if a better
// schedule exists.
//
// Wave organisation: the state and the DFS control are uniform; the 64 lanes
// evaluate candidate (k, d) pairs in parallel (candidate c: d = c / 8,
// k = c % 8) and pick the next one with a wave minimum over packed keys
// (lb << 16 | d << 3 | k); the memo is an LDS hash table probed 64 slots at a
// time; the DFS stack and the per-frame candidate keys live in LDS.
#include <algorithm>

#include "opt_common.hpp"
#include "wave.hpp"

namespace fs {

namespace {

constexpr int NMAX = 8;
constexpr int MEMO_BYTES = 32768;     // LDS memo bytes per wave (first pass)
constexpr int FRAMES = NMAX + 2;      // DFS depth <= n, plus the root
constexpr int FW = 8;                 // words per frame
constexpr int CACHE = 192;            // cached candidate keys per frame (3 per lane)
constexpr uint32_t NOKEY = 0xFFFFFFFFu;
constexpr int GUARD = 1 << 22;        // DFS pushes per search in the first pass
constexpr int PAIR_ENTRIES = 7680;       // two-worker tables: first launch (15 KB)
constexpr int PAIR_ENTRIES_MAX = 32000;  // second launch (64 KB)

// frame word offsets
enum { F_S = 0, F_SIG, F_PLO, F_PHI, F_BOUND, F_BEST, F_THR, F_FLAGS };
// flags: bit 0 entered, bit 1 keys cached, bits 8.. dhi

struct Inst {
  int n, B, alpha, rmax;
  int64_t M;
  int len[NMAX], arr[NMAX];
  uint32_t eqprev[NMAX];
  uint32_t compat[NMAX];  // jobs that may run beside job j under the KV budget
  uint32_t full;
  bool compact;           // B <= 3 and every arrival 0: 64-bit memo entries
};

__device__ __forceinline__ int prog_of(uint32_t plo, uint32_t phi, int j) {
  return (int)(((j < 4 ? plo >> (8 * j) : phi >> (8 * (j - 4)))) & 0xFFu);
}

// Key of candidate c from state (S, sig, progress); NOKEY if inadmissible.
__device__ inline uint32_t cand_key(const Inst& I, uint32_t S, int sig, uint32_t plo,
                                    uint32_t phi, int c, int dhi, int sumU) {
  const int d = c >> 3, k = c & 7;
  if (k >= I.n || d > dhi || ((S >> k) & 1u)) return NOKEY;
  int lk = 0, ak = 0;
  uint32_t eq = 0;
#pragma unroll
  for (int j = 0; j < NMAX; ++j)
    if (j == k) {
      lk = I.len[j];
      ak = I.arr[j];
      eq = I.eqprev[j];
    }
  if ((S & eq) != eq) return NOKEY;  // a lower identical job is still unstarted
  if (d < ak - sig) return NOKEY;    // not released yet
  int cnt = 0, maxp = 0, maxrem = lk, sumrem = lk;
  int64_t sumlen = 0;
#pragma unroll
  for (int j = 0; j < NMAX; ++j) {
    const int p = prog_of(plo, phi, j);
    if (p != 0xFF) {
      const int rem = I.len[j] - p;
      if (rem > d) {
        cnt++;
        maxp = max(maxp, p + d);
        sumlen += I.len[j];
        maxrem = max(maxrem, rem - d);
        sumrem += rem - d;
      }
    }
  }
  if (cnt > I.B - 1) return NOKEY;
  if (cnt > 0 && maxp > I.alpha) return NOKEY;
  if (I.M != 0 && cnt > 0 && sumlen + lk > I.M) return NOKEY;
  const int sig2 = sig + d;
  int maxu = 0;
  uint32_t R = 0;  // jobs with work left after the start of k
#pragma unroll
  for (int j = 0; j < NMAX; ++j) {
    if (j < I.n && j != k && !((S >> j) & 1u)) {
      maxu = max(maxu, max(0, I.arr[j] - sig2) + I.len[j]);
      R |= 1u << j;
    }
    const int p = prog_of(plo, phi, j);
    if (p != 0xFF && I.len[j] - p > d) R |= 1u << j;
  }
  R |= 1u << k;
  // A job that fits beside no other remaining job (KV budget, or B = 1) runs
  // alone: its remaining steps are serial with everything else.
  int alone = 0;
#pragma unroll
  for (int j = 0; j < NMAX; ++j) {
    if (((R >> j) & 1u) && (I.compat[j] & R & ~(1u << j)) == 0u) {
      const int p = prog_of(plo, phi, j);
      int rj = I.len[j];
      if (j != k && p != 0xFF) rj = I.len[j] - p - d;
      alone += rj;
    }
  }
  const int work = sumrem + sumU - lk;
  const int lb = max(max(maxrem, maxu), alone + (work - alone + I.B - 1) / I.B);
  return ((uint32_t)(d + lb) << 16) | ((uint32_t)d << 3) | (uint32_t)k;
}

__device__ __forceinline__ uint32_t mix(uint32_t k0, uint32_t k1, uint32_t k2) {
  uint32_t h = k0 * 0x9E3779B1u ^ (k1 + 0x7F4A7C15u) * 0x85EBCA77u ^ (k2 + 0x165667B1u) * 0xC2B2AE3Du;
  h ^= h >> 15;
  h *= 0x2C1B3C6Du;
  h ^= h >> 12;
  return h;
}

// The memo: a hash table probed 64 slots at a time.  The first pass keeps it in
// LDS; the second pass in its own region of global scratch, read and written
// with agent-scope accesses (they bypass the vector L1, so a lane reads what
// another lane of the wave stored).
struct Memo {
  uint32_t* base;
  bool compact;  // one 64-bit word per entry (LDS only), else 4 words per entry
  bool global;
  int entries;   // power of two

  __device__ uint32_t ld(const uint32_t* p) const {
    if (global) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return *p;
  }
  __device__ void st(uint32_t* p, uint32_t v) const {
    if (global) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
  }
  // every lane sees the stores of the wave before its next probe
  __device__ void sync() const {
    if (global) __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "agent");
    wave_lds_sync();
  }

  // Compact key: valid | S | up to three active (index, progress) pairs in index order.
  __device__ static uint64_t ckey(uint32_t S, uint32_t plo, uint32_t phi) {
    uint64_t slots = 0;
    int c = 0;
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
      const int p = prog_of(plo, phi, j);
      if (p != 0xFF && c < 3) {
        slots |= (uint64_t)((j << 8) | p) << (11 * c);
        c++;
      }
    }
    for (int q = c; q < 3; ++q) slots |= (uint64_t)0x7FFu << (11 * q);
    return (1ull << 63) | ((uint64_t)S << 55) | (slots << 16);
  }

  // value | exact << 31, or NOKEY if absent
  __device__ uint32_t get(uint32_t a, uint32_t b, uint32_t c, uint32_t S, int lane) const {
    if (compact) {
      const uint64_t key = ckey(S, b, c);
      const uint64_t* T = (const uint64_t*)base;
      const uint32_t h = mix((uint32_t)(key >> 32), (uint32_t)key, 0u);
      const int slot = (int)((h + (uint32_t)lane) & (uint32_t)(entries - 1));
      const uint64_t x = T[slot];
      const bool hit = (x >> 16) == (key >> 16);
      const bool empty = x == 0ull;
      const uint64_t mh = ballot(hit), me = ballot(empty);
      if (!mh) return NOKEY;
      const int L = __builtin_ctzll(mh);
      if (me && __builtin_ctzll(me) < L) return NOKEY;
      const uint32_t v = (uint32_t)readlane((int)(uint32_t)(x & 0xFFFFu), L);
      return (v & 0x7FFFu) | ((v & 0x8000u) << 16);
    }
    const uint32_t* k0 = base;
    const uint32_t* k1 = base + entries;
    const uint32_t* k2 = base + 2 * (size_t)entries;
    const uint32_t* val = base + 3 * (size_t)entries;
    const uint32_t h = mix(a, b, c);
    const int slot = (int)((h + (uint32_t)lane) & (uint32_t)(entries - 1));
    const uint32_t x = ld(k0 + slot);
    const bool hit = x == a && ld(k1 + slot) == b && ld(k2 + slot) == c;
    const bool empty = x == 0u;
    const uint64_t mh = ballot(hit), me = ballot(empty);
    if (!mh) return NOKEY;
    const int L = __builtin_ctzll(mh);
    if (me && __builtin_ctzll(me) < L) return NOKEY;  // keys sit before any hole
    return (uint32_t)readlane((int)ld(val + slot), L);
  }

  __device__ void put(uint32_t a, uint32_t b, uint32_t c, uint32_t S, uint32_t v, int lane) {
    if (compact) {
      const uint64_t key = ckey(S, b, c);
      uint64_t* T = (uint64_t*)base;
      const uint32_t h = mix((uint32_t)(key >> 32), (uint32_t)key, 0u);
      const int slot = (int)((h + (uint32_t)lane) & (uint32_t)(entries - 1));
      const uint64_t x = T[slot];
      const bool hit = (x >> 16) == (key >> 16);
      const bool empty = x == 0ull;
      const uint64_t mh = ballot(hit), me = ballot(empty);
      const int L = mh ? __builtin_ctzll(mh) : (me ? __builtin_ctzll(me) : 0);
      const uint64_t e = key | (uint64_t)((v & 0x7FFFu) | ((v >> 16) & 0x8000u));
      if (lane == L) T[slot] = e;
      wave_lds_sync();
      return;
    }
    uint32_t* k0 = base;
    uint32_t* k1 = base + entries;
    uint32_t* k2 = base + 2 * (size_t)entries;
    uint32_t* val = base + 3 * (size_t)entries;
    const uint32_t h = mix(a, b, c);
    const int slot = (int)((h + (uint32_t)lane) & (uint32_t)(entries - 1));
    const uint32_t x = ld(k0 + slot);
    const bool hit = x == a && ld(k1 + slot) == b && ld(k2 + slot) == c;
    const bool empty = x == 0u;
    const uint64_t mh = ballot(hit), me = ballot(empty);
    int L;
    if (mh) L = __builtin_ctzll(mh);
    else if (me) L = __builtin_ctzll(me);
    else L = 0;  // probe window full: replace the home slot
    if (lane == L) {
      st(k0 + slot, a);
      st(k1 + slot, b);
      st(k2 + slot, c);
      st(val + slot, v);
    }
    sync();
  }

  __device__ void clear(int lane) {
    const size_t words = compact ? 2 * (size_t)entries : 4 * (size_t)entries;
    for (size_t i = (size_t)lane; i < words; i += WAVE) st(base + i, 0u);
    sync();
  }
};

struct Dfs {
  const Inst& I;
  Memo& memo;
  uint32_t* F;      // FRAMES * FW words
  uint32_t* keys;   // FRAMES * CACHE candidate keys
  int lane;

  __device__ uint32_t frame(int depth, int f) const { return F[depth * FW + f]; }
  __device__ void set(int depth, int f, uint32_t v) {
    if (lane == 0) F[depth * FW + f] = v;
  }

  // state-dependent scalars
  __device__ void state_info(uint32_t S, int sig, uint32_t plo, uint32_t phi, int& dhi,
                             int& sumU) const {
    int maxrem = 0, late = 0;
    sumU = 0;
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
      const int p = prog_of(plo, phi, j);
      if (p != 0xFF) maxrem = max(maxrem, I.len[j] - p);
      if (j < I.n && !((S >> j) & 1u)) {
        sumU += I.len[j];
        late = max(late, I.arr[j] - sig);
      }
    }
    dhi = max(maxrem, late);
  }

  // smallest candidate key > thr (NOKEY if none)
  __device__ uint32_t pick(int depth, uint32_t S, int sig, uint32_t plo, uint32_t phi,
                           uint32_t flags, uint32_t thr) const {
    const int dhi = (int)(flags >> 8);
    uint32_t best = NOKEY;
    if (flags & 2u) {
      const uint32_t* K = keys + depth * CACHE;
#pragma unroll
      for (int i = 0; i < CACHE / WAVE; ++i) {
        const uint32_t k = K[i * WAVE + lane];
        if (k > thr && k < best) best = k;
      }
    } else {
      int dd, sumU;
      state_info(S, sig, plo, phi, dd, sumU);
      const int nc = (dhi + 1) * 8;
      for (int c0 = 0; c0 < nc; c0 += WAVE) {
        const uint32_t k = cand_key(I, S, sig, plo, phi, c0 + lane, dhi, sumU);
        if (k > thr && k < best) best = k;
      }
    }
    return wave_umin(best);
  }

  // V(root) if it is below `bound`, else a value >= bound; -1 after more than
  // `guard_max` pushes.
  __device__ int run(uint32_t S0, int sig0, uint32_t plo0, uint32_t phi0, int bound0,
                     int guard_max) {
    int depth = 0;
    set(0, F_S, S0);
    set(0, F_SIG, (uint32_t)sig0);
    set(0, F_PLO, plo0);
    set(0, F_PHI, phi0);
    set(0, F_BOUND, (uint32_t)bound0);
    set(0, F_FLAGS, 0u);
    wave_lds_sync();
    int guard = 0;
    while (true) {
      const uint32_t S = frame(depth, F_S);
      const int sig = (int)frame(depth, F_SIG);
      const uint32_t plo = frame(depth, F_PLO), phi = frame(depth, F_PHI);
      const int bound = (int)frame(depth, F_BOUND);
      uint32_t flags = frame(depth, F_FLAGS);
      int ret = -1;
      const uint32_t ka = 1u | (S << 1) | ((uint32_t)min(sig, I.rmax) << 9);
      if (!(flags & 1u)) {
        if (S == I.full) {
          int mr = 0;
#pragma unroll
          for (int j = 0; j < NMAX; ++j) {
            const int p = prog_of(plo, phi, j);
            if (p != 0xFF) mr = max(mr, I.len[j] - p);
          }
          ret = mr;
        } else {
          const uint32_t v = memo.get(ka, plo, phi, S, lane);
          if (v != NOKEY && ((v >> 31) || (int)(v & 0x7FFFFFFFu) >= bound)) {
            ret = (int)(v & 0x7FFFFFFFu);
          } else {
            int dhi, sumU;
            state_info(S, sig, plo, phi, dhi, sumU);
            flags = 1u | ((uint32_t)dhi << 8);
            if ((dhi + 1) * 8 <= CACHE) {
              flags |= 2u;
              uint32_t* K = keys + depth * CACHE;
#pragma unroll
              for (int i = 0; i < CACHE / WAVE; ++i)
                K[i * WAVE + lane] = cand_key(I, S, sig, plo, phi, i * WAVE + lane, dhi, sumU);
            }
            set(depth, F_FLAGS, flags);
            set(depth, F_BEST, (uint32_t)bound);
            set(depth, F_THR, 0u);
            wave_lds_sync();
          }
        }
      }
      if (ret < 0) {
        const int best = (int)frame(depth, F_BEST);
        const uint32_t thr = frame(depth, F_THR);
        const uint32_t key = pick(depth, S, sig, plo, phi, flags, thr);
        if (key != NOKEY && (int)(key >> 16) < best && depth + 1 < FRAMES) {
          const int d = (int)((key >> 3) & 0x1FFFu), k = (int)(key & 7u);
          uint32_t nlo = 0, nhi = 0;
#pragma unroll
          for (int j = 0; j < NMAX; ++j) {
            int p = prog_of(plo, phi, j);
            int q = 0xFF;
            if (j == k) q = 0;
            else if (p != 0xFF && I.len[j] - p > d) q = p + d;
            if (j < 4) nlo |= (uint32_t)q << (8 * j);
            else nhi |= (uint32_t)q << (8 * (j - 4));
          }
          set(depth, F_THR, key);
          set(depth + 1, F_S, S | (1u << k));
          set(depth + 1, F_SIG, (uint32_t)(sig + d));
          set(depth + 1, F_PLO, nlo);
          set(depth + 1, F_PHI, nhi);
          set(depth + 1, F_BOUND, (uint32_t)(best - d));
          set(depth + 1, F_FLAGS, 0u);
          wave_lds_sync();
          depth++;
          if (++guard > guard_max) return -1;
          continue;
        }
        memo.put(ka, plo, phi, S, (uint32_t)best | ((best < bound) ? 0x80000000u : 0u), lane);
        ret = best;
      }
      if (depth == 0) return ret;
      depth--;
      const uint32_t pthr = frame(depth, F_THR);
      const int pd = (int)((pthr >> 3) & 0x1FFFu);
      const int pbest = (int)frame(depth, F_BEST);
      if (ret + pd < pbest) set(depth, F_BEST, (uint32_t)(ret + pd));
      wave_lds_sync();
    }
  }
};

// Read instance `inst` into I.  False (after writing the marker) when a length
// or an arrival is beyond the search's limits.
__device__ bool load_inst(const OptArgs& a, int64_t inst, int lane, Inst& I) {
  const int n = a.n;
  const int64_t row = inst * (int64_t)n;
  int lv = 0, av = 0, bad = 0;
  if (lane < n) {
    lv = a.prompt[row + lane] + a.output[row + lane];
    av = a.arrival[row + lane];
    bad = (lv > OPT_LEN_LIMIT) || (av > OPT_ARR_LIMIT);
  }
  if (ballot(bad != 0)) {
    if (lane == 0) a.T[inst] = FSCHED_T_TOOLARGE;
    return false;
  }
  I.n = n;
  I.B = a.B;
  I.alpha = a.alpha;
  I.M = a.M;
  I.rmax = 0;
#pragma unroll
  for (int j = 0; j < NMAX; ++j) {
    I.len[j] = j < n ? readlane(lv, j) : 0;
    I.arr[j] = j < n ? readlane(av, j) : 0;
    I.rmax = max(I.rmax, I.arr[j]);
  }
#pragma unroll
  for (int k = 0; k < NMAX; ++k) {
    uint32_t e = 0;
#pragma unroll
    for (int j = 0; j < NMAX; ++j)
      if (j < k && k < n && I.len[j] == I.len[k] && I.arr[j] == I.arr[k]) e |= 1u << j;
    I.eqprev[k] = e;
  }
  I.full = (n >= 32) ? 0xFFFFFFFFu : ((1u << n) - 1u);
#pragma unroll
  for (int j = 0; j < NMAX; ++j) {
    uint32_t c = 0;
#pragma unroll
    for (int i = 0; i < NMAX; ++i)
      if (i != j && i < n && j < n && I.B > 1 &&
          (I.M == 0 || (int64_t)I.len[i] + I.len[j] <= I.M))
        c |= 1u << i;
    I.compat[j] = c;
  }
  I.compact = I.B <= 3 && I.rmax == 0;
  return true;
}

// Search instance `inst` below its incumbent (the ISJL makespan in T) and, when
// something better exists, write the optimum and one optimal schedule.  False
// if the search made more than `guard_max` pushes (nothing written then).
__device__ bool solve(const OptArgs& a, int64_t inst, const Inst& I, Memo& memo, uint32_t* frames,
                      uint32_t* keys, int lane, int guard_max) {
  const int64_t row = inst * (int64_t)a.n;
  Dfs dfs{I, memo, frames, keys, lane};
  const uint32_t none = 0xFFFFFFFFu;
  const int bound = (int)a.T[inst];
  const int v = dfs.run(0u, 0, none, none, bound, guard_max);
  if (v < 0) return false;
  if (v >= bound) return true;  // ISJL's schedule (already written) is optimal

  if (lane == 0) a.T[inst] = v;
  if (!a.start) return true;
  // Reconstruct one optimal schedule: from each state take the first candidate
  // (in key order) whose child reaches the state's value.
  uint32_t S = 0u, plo = none, phi = none;
  int sig = 0, val = v;
  int steps = 0;
  while (S != I.full && steps < 2 * NMAX) {
    steps++;
    int dhi, sumU;
    dfs.state_info(S, sig, plo, phi, dhi, sumU);
    const uint32_t flags = 1u | ((uint32_t)dhi << 8);  // no cache: frame 0 is reused below
    uint32_t thr = 0u;
    bool moved = false;
    while (true) {
      const uint32_t key = dfs.pick(FRAMES - 1, S, sig, plo, phi, flags, thr);
      if (key == NOKEY || (int)(key >> 16) > val) break;
      thr = key;
      const int d = (int)((key >> 3) & 0x1FFFu), k = (int)(key & 7u);
      uint32_t nlo = 0, nhi = 0;
#pragma unroll
      for (int j = 0; j < NMAX; ++j) {
        int p = prog_of(plo, phi, j);
        int q = 0xFF;
        if (j == k) q = 0;
        else if (p != 0xFF && I.len[j] - p > d) q = p + d;
        if (j < 4) nlo |= (uint32_t)q << (8 * j);
        else nhi |= (uint32_t)q << (8 * (j - 4));
      }
      const int cv = dfs.run(S | (1u << k), sig + d, nlo, nhi, val - d + 1, guard_max);
      if (cv >= 0 && cv + d == val) {
        if (lane == 0) a.start[row + k] = sig + d;
        S |= 1u << k;
        sig += d;
        plo = nlo;
        phi = nhi;
        val -= d;
        moved = true;
        break;
      }
    }
    if (!moved) break;  // not reachable: some child always attains the value
  }
  return true;
}

// Claim the next entry of a list (counters[0] entries, counters[1] the claim
// counter): its instance, or -1 once the list is exhausted.
__device__ __forceinline__ int64_t claim(const int32_t* list, int32_t* counters, int nlist,
                                         int lane) {
  int idx = 0;
  if (lane == 0) idx = atomicAdd(counters + 1, 1);
  idx = readlane(idx, 0);
  return idx < nlist ? (int64_t)list[idx] : -1;
}

__device__ __forceinline__ void append(int32_t* list, int32_t* counters, int64_t inst, int lane) {
  if (lane == 0) list[atomicAdd(counters, 1)] = (int32_t)inst;
}

// Two workers, every job released at step 0: dynamic program over
//   W(S, s, q)  least remaining time when the jobs S have started and only s
//               runs, with progress q (the other worker is idle)
//   E(S)        the same with both workers idle
// A start of k beside s at progress q needs q <= alpha and the pair within the
// KV budget; then the shorter remainder ends first, which is again a state of
// this kind, so with r = len_s - q, t = min(r, len_k) and S' = S + k
//   W0(S, s, q) = min over k of t + W(S', survivor, its progress)   (start now)
//   W(S, s, q)  = min(W0(S, s, q) if q <= alpha, 1 + W(S, s, q + 1)),
//   W(S, s, len_s) = E(S),  E(S) = min over k of W(S', k, 0),  E(all) = 0,
// and beyond alpha W is len_s - q + E(S), which is not stored.  Identical jobs
// are one class, so S is a mixed-radix number of started jobs per class (a
// superset has the larger number) and s a class: at most 256 rows of
// 1 + sum of min(alpha + 1, len) entries of 16 bits.
//
// The search above visits these states one at a time through its memo, about
// 1.6 M vector instructions per tiny instance at one wave per SIMD (its memo
// fills the LDS); the table has a few thousand entries, each 8 candidates, and
// every entry of one level (number of started jobs) is independent of the
// others, one (S, s) per lane, its q from the largest down.  65,536 tiny
// instances (n = 8, alpha = 2, M_kv = 16): 656 -> 1.8 ms with the ISJL launch
// (0.47 ms) included; 3,000 at alpha = 19, M_kv = 24: 9.0 s -> 1.0 ms.
struct PairDp {
  const Inst& I;
  uint16_t* tab;     // rows of R entries: E(S), then W(S, s, 0..qmax_s) per class
  uint8_t* order;    // rows by number of started jobs, the most first
  uint16_t* info;    // per row: classes with a job left | classes started << 8
  uint32_t* cls;     // per class (by its first job): len | offset of its entries << 16
  int lane;
  int C, NS, R;
  uint32_t reps;     // first jobs of the classes, 4 bits each
  uint32_t first;    // bit j: job j is the first of its class
  int cnt[NMAX], stride[NMAX], off[NMAX];

  __device__ int qmax(int len) const { return min(I.alpha, len - 1); }

  // Row and class tables; false when the rows do not fit `entries`.
  __device__ bool setup(int entries) {
    C = 0;
    NS = 1;
    R = 1;
    reps = first = 0;
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
      cnt[j] = stride[j] = off[j] = 0;
      if (j < I.n && I.eqprev[j] == 0u) {
        int m = 0;
#pragma unroll
        for (int i = 0; i < NMAX; ++i) m += i < I.n && I.len[i] == I.len[j] ? 1 : 0;
        cnt[j] = m;
        stride[j] = NS;
        off[j] = R;
        NS *= m + 1;
        R += qmax(I.len[j]) + 1;
        reps |= (uint32_t)j << (4 * C);
        first |= 1u << j;
        C++;
      }
    }
    if (NS * R > entries) return false;
#pragma unroll
    for (int j = 0; j < NMAX; ++j)
      if (lane == j) cls[j] = (uint32_t)I.len[j] | ((uint32_t)off[j] << 16);
    return true;
  }

  __device__ int fill() {
    // the digits of row r, its class masks, and its place in the level order
    int lev[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = i * WAVE + lane;
      lev[i] = -1;
      if (i * WAVE < NS) {
        int rest = r, l = 0;
        uint32_t left = 0, started = 0;
#pragma unroll
        for (int j = NMAX - 1; j >= 0; --j) {
          if ((first >> j) & 1u) {
            // rest < 256 and stride <= 128: the product is exact
            const int dgt = (int)(((uint32_t)rest * (uint32_t)((65536 + stride[j] - 1) / stride[j])) >> 16);
            rest -= dgt * stride[j];
            l += dgt;
            if (dgt < cnt[j]) left |= 1u << j;
            if (dgt > 0) started |= 1u << j;
          }
        }
        if (r < NS) {
          lev[i] = l;
          info[r] = (uint16_t)(left | (started << 8));
        }
      }
    }
    int begin = 0;
    for (int L = I.n; L >= 0; --L) {
      int end = begin;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (i * WAVE < NS) {
          const uint64_t m = ballot(lev[i] == L);
          if (lev[i] == L) order[end + mbcnt(m)] = (uint8_t)(i * WAVE + lane);
          end += __builtin_popcountll(m);
        }
      }
      wave_lds_sync();
      // one (row, class) per lane; 65536 / C rounded up is exact for products below 2^12
      const int items = L > 0 ? (end - begin) * C : 1;
      const uint32_t inv = (65536u + (uint32_t)C - 1u) / (uint32_t)C;
      for (int it0 = 0; it0 < items; it0 += WAVE) {
        const int it = it0 + lane;
        const int ro = (int)(((uint32_t)it * inv) >> 16);
        const bool in = it < items;
        const int S = in ? order[begin + ro] : 0;
        const int c = (int)((reps >> (4 * (it - ro * C))) & 7u);
        const uint32_t w = in ? info[S] : 0u;
        const uint32_t cw = cls[c];
        const int len = (int)(cw & 0xFFFFu), co = (int)(cw >> 16);
        const int row = S * R;
        const bool on = in & (((w >> (8 + c)) & 1u) != 0u);
        int E = L == I.n ? 0 : 0x7FFF;
#pragma unroll
        for (int k = 0; k < NMAX; ++k)
          if (((first >> k) & 1u) && ((w >> k) & 1u))
            E = min(E, (int)tab[row + stride[k] * R + off[k]]);
        // every lane of a row finds the same value
        if (in) tab[row] = (uint16_t)E;
        const int qm = on ? qmax(len) : -1;
        int best = len - qm + E - 1;
        const int qtop = wave_max(qm);
        for (int q = qtop; q >= 0; --q) {
          if (q <= qm) {
            best++;
            const int r = len - q;
#pragma unroll
            for (int k = 0; k < NMAX; ++k) {
              if (((first >> k) & 1u) && ((w >> k) & 1u) &
                                             ((I.M == 0) | (len + I.len[k] <= I.M))) {
                const int d = r - I.len[k];
                const int t = min(r, I.len[k]);
                const int qq = d > 0 ? q + I.len[k] : r;  // the survivor's progress
                const bool emp = (d == 0) | (qq > I.alpha);
                const int at = emp ? 0 : (d > 0 ? co : off[k]) + qq;
                const int v = (int)tab[row + stride[k] * R + at] + t + (emp ? abs(d) : 0);
                best = min(best, v);
              }
            }
            tab[row + co + q] = (uint16_t)best;
          }
        }
      }
      wave_lds_sync();
      begin = end;
    }
    return (int)tab[0];
  }

  // Value of the state right after k started in the row of `row` (k counted in
  // it), beside job j (-1: none) at progress p.
  __device__ int after_start(int row, int k, int j, int p) const {
    const uint32_t ck = cls[k];
    const int lk = (int)(ck & 0xFFFFu);
    int sl = lk, so = (int)(ck >> 16), qq = 0, t = 0;
    if (j >= 0) {
      const uint32_t cj = cls[j];
      const int r = (int)(cj & 0xFFFFu) - p;
      t = min(r, lk);
      if (r > lk) {
        sl = (int)(cj & 0xFFFFu);
        so = (int)(cj >> 16);
        qq = p + lk;
      } else {
        qq = r;
      }
    }
    if (qq >= sl || qq > I.alpha) return t + (sl - qq) + (int)tab[row * R];
    return t + (int)tab[row * R + so + qq];
  }
};

// Solve instance `inst` by the two-worker table: false when it is not of that
// kind or its table does not fit `entries`.  The schedule is the one that the
// search's reconstruction gives: from each state the first candidate in key
// order that attains the state's value.
__device__ bool solve_pair(const OptArgs& a, int64_t inst, const Inst& I, uint16_t* tab,
                           int entries, uint8_t* order, uint16_t* info, uint32_t* cls, int lane) {
  if (I.B != 2 || I.rmax != 0) return false;
  const int bound = (int)a.T[inst];
  {
    // nothing beats a makespan at the root's lower bound: the longest job, the
    // jobs that fit beside no other one, and half of the rest
    int sum = 0, alone = 0, maxl = 0;
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
      if (j < I.n) {
        sum += I.len[j];
        maxl = max(maxl, I.len[j]);
        if (I.compat[j] == 0u) alone += I.len[j];
      }
    }
    if (bound <= max(maxl, alone + (sum - alone + 1) / 2)) return true;
  }
  PairDp dp{I, tab, order, info, cls, lane};
  if (!dp.setup(entries)) return false;
  wave_lds_sync();
  const int v = uni(dp.fill());
  if (v >= bound) return true;
  if (lane == 0) a.T[inst] = v;
  if (!a.start) return true;
  const int64_t row = inst * (int64_t)a.n;
  const uint32_t none = 0xFFFFFFFFu;
  uint32_t S = 0u, plo = none, phi = none;
  int sig = 0, val = v, at = 0;  // at: the row of S
  for (int step = 0; step < I.n; ++step) {
    int maxrem = 0, sumU = 0;
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
      const int p = prog_of(plo, phi, j);
      if (p != 0xFF) maxrem = max(maxrem, I.len[j] - p);
      if (j < I.n && !((S >> j) & 1u)) sumU += I.len[j];
    }
    uint32_t best = NOKEY;
    for (int c0 = 0; c0 < (maxrem + 1) * 8; c0 += WAVE) {
      const int c = c0 + lane, d = c >> 3, k = c & 7;
      const uint32_t key = cand_key(I, S, sig, plo, phi, c, maxrem, sumU);
      if (key != NOKEY) {
        int j = -1, pj = 0, kc = k, rk = at;
#pragma unroll
        for (int i = 0; i < NMAX; ++i) {
          const int p = prog_of(plo, phi, i);
          if (p != 0xFF && I.len[i] - p > d) {
            j = I.eqprev[i] ? __builtin_ctz(I.eqprev[i]) : i;
            pj = p + d;
          }
          if (i == k && I.eqprev[i]) kc = __builtin_ctz(I.eqprev[i]);
        }
#pragma unroll
        for (int i = 0; i < NMAX; ++i)
          if (i == kc) rk += dp.stride[i];
        if (d + dp.after_start(rk, kc, j, pj) == val) best = min(best, key);
      }
    }
    best = wave_umin(best);
    if (best == NOKEY) break;  // not reachable: some candidate attains the value
    const int d = (int)((best >> 3) & 0x1FFFu), k = (int)(best & 7u);
    uint32_t nlo = 0, nhi = 0;
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
      const int p = prog_of(plo, phi, j);
      int q = 0xFF;
      if (j == k) {
        q = 0;
        const int kc = I.eqprev[j] ? __builtin_ctz(I.eqprev[j]) : j;
#pragma unroll
        for (int i = 0; i < NMAX; ++i)
          if (i == kc) at += dp.stride[i];
      } else if (p != 0xFF && I.len[j] - p > d) {
        q = p + d;
      }
      if (j < 4) nlo |= (uint32_t)q << (8 * j);
      else nhi |= (uint32_t)q << (8 * (j - 4));
    }
    if (lane == 0) a.start[row + k] = sig + d;
    S |= 1u << k;
    sig += d;
    plo = nlo;
    phi = nhi;
    val -= d;
  }
  return true;
}

}  // namespace

// Two-worker instances without releases, one wave (one block) per instance of
// the batch or of src's list; what it does not solve goes to dst's list.
__global__ __launch_bounds__(64) void opt_pair_kernel(OptArgs a, int entries, int32_t* src,
                                                      int32_t* src_n, int32_t* dst,
                                                      int32_t* dst_n) {
  extern __shared__ uint32_t lds_raw[];
  const int lane = lane_id();
  uint32_t* cls = lds_raw;
  uint16_t* info = (uint16_t*)(cls + NMAX);
  uint8_t* order = (uint8_t*)(info + 256);
  uint16_t* tab = (uint16_t*)(order + 256);
  const int nlist =
      src ? __hip_atomic_load(src_n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
  int64_t inst = blockIdx.x;
  while (true) {
    if (src) inst = claim(src, src_n, nlist, lane);
    if (inst < 0) break;
    Inst I;
    if (a.T[inst] >= 0 && load_inst(a, inst, lane, I)) {
      if (!solve_pair(a, inst, I, tab, entries, order, info, cls, lane))
        append(dst, dst_n, inst, lane);
    }
    if (!src) break;
  }
}

// The list counters start at zero (a kernel rather than a memset, which a
// captured graph would not replay reliably).
__global__ __launch_bounds__(64) void opt_clear_kernel(int32_t* counters, int n) {
  if ((int)threadIdx.x < n) counters[threadIdx.x] = 0;
}

// One wave per instance of the batch, or of the list (whose length only the
// device knows: the blocks beyond it end at once).  A loop over the list around
// the search cost it scalar registers and 5-9 % of its time; a constant LDS
// base, which the compiler keeps in scalar registers too (245 instead of 192 of
// them spilled), 3 %.
__global__ __launch_bounds__(64) void opt_kernel(OptArgs a) {
  extern __shared__ uint32_t lds_raw[];
  const int lane = lane_id();
  const int wib = threadIdx.x >> 6;
  uint32_t* base = lds_raw + wib * (MEMO_BYTES / 4 + FRAMES * FW + FRAMES * CACHE);
  uint32_t* frames = base + MEMO_BYTES / 4;
  uint32_t* keys = frames + FRAMES * FW;

  int64_t inst = blockIdx.x;
  if (a.todo_list) {
    if (inst >= *a.todo_count) return;
    inst = a.todo_list[inst];
  }
  if (a.T[inst] < 0) return;  // ISJL's error marker
  Inst I;
  if (!load_inst(a, inst, lane, I)) return;
  Memo memo{base, I.compact, false, I.compact ? MEMO_BYTES / 8 : MEMO_BYTES / 16};
  memo.clear(lane);
  if (!solve(a, inst, I, memo, frames, keys, lane, GUARD)) {
    // the LDS memo was too small for this search: leave it to the second pass
    if (a.fb_list) append(a.fb_list, a.fb_count, inst, lane);
    else if (lane == 0) a.T[inst] = FSCHED_T_INTERNAL;
  }
}

// Second pass: OPT_FB_WAVES persistent waves take the listed instances one at a
// time (claimed with an atomic counter) and search them again with a memo of
// OPT_FB_MEMO_ENTRIES entries in their own region of global scratch.  Every
// wave leaves once the list is exhausted.
__global__ __launch_bounds__(64) void opt_fallback_kernel(OptArgs a) {
  extern __shared__ uint32_t lds_raw[];
  const int lane = lane_id();
  uint32_t* frames = lds_raw;
  uint32_t* keys = frames + FRAMES * FW;
  const int nlist = __hip_atomic_load(a.fb_count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  Memo memo{a.fb_memo + (size_t)blockIdx.x * 4 * (size_t)OPT_FB_MEMO_ENTRIES, false, true,
            OPT_FB_MEMO_ENTRIES};
  while (true) {
    const int64_t inst = claim(a.fb_list, a.fb_count, nlist, lane);
    if (inst < 0) break;
    Inst I;
    if (!load_inst(a, inst, lane, I)) continue;
    memo.clear(lane);
    if (!solve(a, inst, I, memo, frames, keys, lane, OPT_FB_GUARD))
      if (lane == 0) a.T[inst] = FSCHED_T_INTERNAL;
  }
}

static size_t opt_lds_words_per_wave() { return MEMO_BYTES / 4 + FRAMES * FW + FRAMES * CACHE; }

static size_t opt_fallback_lds_words_per_wave() { return FRAMES * FW + FRAMES * CACHE; }

namespace {

// Bytes of the two-worker kernel's LDS beside its table.
constexpr size_t PAIR_LDS_FIXED = NMAX * 4 + 256 * 2 + 256;

hipError_t launch_pair(const OptArgs& a, int64_t blocks, int entries, int32_t* src, int32_t* src_n,
                       int32_t* dst, int32_t* dst_n, hipStream_t s) {
  hipLaunchKernelGGL(opt_pair_kernel, dim3((unsigned)blocks), dim3((unsigned)WAVE),
                     PAIR_LDS_FIXED + ((size_t)entries * 2 + 3) / 4 * 4, s, a, entries, src, src_n,
                     dst, dst_n);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_opt(const OptArgs& a0, hipStream_t s) {
  OptArgs a = a0;
  const size_t lds = (size_t)opt_lds_words_per_wave() * 4;
  if (a.lists) {
    hipLaunchKernelGGL(opt_clear_kernel, dim3(1), dim3((unsigned)WAVE), 0, s, a.counters,
                       OPT_COUNTERS);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    a.fb_list = a.lists;
    a.fb_count = a.counters;
    if (a.B == 2) {
      // Tables of up to 2^n rows of 1 + n (alpha + 1) entries.  The first launch
      // takes those within PAIR_ENTRIES (10 waves share a CU's LDS then; 65,536
      // instances at alpha = 2 took 1.82 ms with it, 1.87 / 1.98 / 3.07 ms with
      // limits of 5,120 / 4,096 / 2,560 entries, which leave more to the second
      // launch); a second one those within PAIR_ENTRIES_MAX, when a table can be
      // larger at all, by 1,024 blocks that claim from the list: two of them share
      // a CU's LDS at the largest table, seven at alpha = 4's (256 blocks took 3.8
      // ms there, 1,024 2.7, 4,096 2.5; at alpha = 7 and 11 10.4 and 13.2 ms, then
      // 4.6 and 6.0 with either).
      const int64_t per_job = (int64_t)std::min(a.alpha, OPT_LEN_LIMIT - 1) + 1;
      const int64_t worst = ((int64_t)1 << a.n) * (1 + a.n * per_job);
      const int first = (int)std::min<int64_t>(worst, PAIR_ENTRIES);
      int32_t* list = a.lists + a.n_inst;
      int32_t* list_n = a.counters + 2;
      e = launch_pair(a, a.n_inst, first, nullptr, nullptr, list, list_n, s);
      if (e != hipSuccess) return e;
      if (worst > PAIR_ENTRIES) {
        int32_t* list2 = list + a.n_inst;
        int32_t* list2_n = a.counters + 4;
        e = launch_pair(a, std::min<int64_t>(a.n_inst, 1024),
                        (int)std::min<int64_t>(worst, PAIR_ENTRIES_MAX), list, list_n, list2,
                        list2_n, s);
        if (e != hipSuccess) return e;
        list = list2;
        list_n = list2_n;
      }
      // the search takes what is left (releases, larger tables)
      a.todo_list = list;
      a.todo_count = list_n;
    }
  }
  hipLaunchKernelGGL(opt_kernel, dim3((unsigned)a.n_inst), dim3((unsigned)WAVE), lds, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !a.lists) return e;
  hipLaunchKernelGGL(opt_fallback_kernel, dim3((unsigned)OPT_FB_WAVES), dim3((unsigned)WAVE),
                     opt_fallback_lds_words_per_wave() * 4, s, a);
  return hipGetLastError();
}

}  // namespace fs
